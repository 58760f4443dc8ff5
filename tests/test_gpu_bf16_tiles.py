"""The bf16-feature kernels in tiles for W of any shape: edges of tiles, remainders of chunks, rows at any alignment, slices of
the contraction, dead workers and values without a three-term split, against fp64.

Bounds.  U of scores that take W exactly: fp32 sums of D products, 2^-24 sqrt(D) of the norm and less; 4e-6 leaves room for expf.
Of scores that round W to bf16 (relative error up to 2^-8 an entry, a random walk in the sum): 2e-2 of the norm.  The update rounds
alpha * u to bf16 once: an entry is off by at most 2^-8 sum |alpha u v| (eight significand bits, half a unit of the last; fp32 sums far less)."""
import pytest
import torch

import paper_1511_08486_amd as sfb

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def strided(x, pad, shift):
    """x with rows `pad` elements longer, starting `shift` elements into its memory; what lies between holds NaN."""
    rows, cols = x.shape
    flat = torch.full((rows * (cols + pad) + shift + 8,), float("nan"), dtype=x.dtype, device=x.device)
    out = flat[shift:shift + rows * (cols + pad)].view(rows, cols + pad)[:, :cols]
    out.copy_(x)
    return out


def batch(J, D, N, seed):
    g = torch.Generator(device=DEV).manual_seed(seed)
    A = (torch.randn((N, D), generator=g, device=DEV) / D ** 0.5).to(torch.bfloat16)
    W = torch.randn((J, D), generator=g, device=DEV)
    return A, W, torch.randint(0, J, (N,), generator=g, device=DEV, dtype=torch.int32), g


def residual(W, A, y):
    u = torch.softmax(A.double() @ W.double().T, 1)
    u[torch.arange(len(y)), y.long()] -= 1.0
    return u


def prox(kind, w, a):
    """The entrywise operators, no larger than the identity in the differences that they leave."""
    return {"none": w, "l2sq": w / (1.0 + a), "l1": torch.sign(w) * (w.abs() - a).clamp(min=0.0)}[kind]


SHAPES = [  # J, D, P, B
    (33, 9, 2, 5), (40, 7, 2, 16), (64, 64, 2, 64), (65, 65, 3, 43), (127, 129, 2, 63), (129, 250, 4, 33), (128, 128, 4, 32),
    (200, 2051, 3, 22), (257, 96, 5, 52), (1000, 31, 2, 65), (2, 2309, 2, 70), (3, 2500, 2, 9), (70, 1, 2, 8), (520, 1056, 4, 32),
    (96, 333, 12, 300), (1300, 1028, 4, 90),
]


@pytest.mark.parametrize("J,D,P,B", SHAPES)
@pytest.mark.parametrize("pad,shift", [(0, 0), (3, 1)])
def test_scores_and_features(J, D, P, B, pad, shift):
    N = P * B
    A, W, y, _ = batch(J, D, N, J + D)
    want = residual(W, A, y)
    ctx = sfb.Sfb("mlr", J, D, P, B, dtype="bf16", device=DEV)
    A2, W2 = strided(A, pad, shift), strided(W, pad, shift)
    U, V = strided(torch.zeros((N, J), device=DEV), pad, shift), strided(torch.zeros_like(A), pad, shift)
    ctx.compute_factors(W2, sfb.SfbBatch(a=A2), y, U, V)
    ctx.sync()
    assert ctx.last_kernel(0)[0] == "scores_bf16_kernel" or J <= 32 and D <= 2048
    assert torch.equal(V, A)
    rounded = N >= 128 and D % 32 == 0 and pad == 0
    err = ((U.double() - want).norm() / want.norm()).item()
    assert err < (2e-2 if rounded else 4e-6), err
    # one worker's rows: W exactly, whatever the batch
    p = P - 1
    U.fill_(float("nan"))
    ctx.compute_factors_worker(W2, sfb.SfbBatch(a=A2[p * B:]), y[p * B:].contiguous(), p, U, V)
    ctx.sync()
    err = ((U[p * B:].double() - want[p * B:]).norm() / want[p * B:].norm()).item()
    assert err < 4e-6, err
    assert torch.isnan(U[:p * B]).all()
    ctx.close()


@pytest.mark.parametrize("J,D,P,B", SHAPES + [(192, 200, 16, 80)])
@pytest.mark.parametrize("pad,shift,dead,kind", [(0, 0, False, "none"), (3, 1, True, "none"), (0, 0, True, "l1"), (3, 1, False, "l2sq")])
def test_update(J, D, P, B, pad, shift, dead, kind):
    N = P * B
    V, W, _, g = batch(J, D, N, J + 2 * D)
    U = torch.randn((N, J), generator=g, device=DEV)
    active = [p != 1 for p in range(P)] if dead else None
    Ul, Vl = U.double(), V.double()
    if dead:
        U[B:2 * B] = float("inf")                        # a dead worker's slot may hold anything
        V[B:2 * B] = float("nan")
        Ul[B:2 * B] = 0.0
        Vl[B:2 * B] = 0.0
    ctx = sfb.Sfb("mlr", J, D, P, B, dtype="bf16", device=DEV)
    W2 = strided(W, pad, shift)
    around = W2.untyped_storage()
    ctx.reconstruct_apply_prox(W2, strided(U, pad, shift), strided(V, pad, shift), 0.25, kind, 0.04, scale=0.5, active=active)
    ctx.sync()
    # (192 x 200, 96 x 333: planes of sums, and the operator in the kernel that adds them)
    name, grid = ctx.last_kernel(2)
    assert name == "update_bf16_kernel" and ((J, D) not in ((192, 200), (96, 333)) or grid > -(-J // 64) * -(-D // 64))
    want = W.double() - 0.125 * (Ul.T @ Vl)
    room = 0.125 * 2.0 ** -8 * (Ul.abs().T @ Vl.abs()) + 2.0 ** -22 * (want.abs() + 1.0)
    assert ((W2.double() - prox(kind, want, 0.25 * 0.04)).abs() <= room).all()
    if pad:                                              # nothing but W's own entries was written
        flat = torch.empty(0, device=DEV).set_(around)
        assert int(torch.isnan(flat).sum()) == flat.numel() - J * D
    ctx.close()


@pytest.mark.parametrize("J,D,P,B,plan", [(J, D, P, B, dict(recon_variant=0)) for J, D, P, B in SHAPES if J > 32 or D > 2048] + [
    (8065, 3715, 4, 60, None), (8064, 3712, 2, 64, None), (4099, 8191, 3, 41, None),          # a W that takes it by itself
])
@pytest.mark.parametrize("pad,shift,dead,kind", [(0, 0, False, "l1"), (3, 1, True, "none"), (0, 0, True, "l2sq")])
def test_update_of_large_w(J, D, P, B, plan, pad, shift, dead, kind):
    """The kernel with tiles of 256 rows and its packed factors: edges, dead workers and the entrywise operators, by the bound of test_update."""
    N = P * B
    V, W, _, g = batch(J, D, N, J + 3 * D)
    U = torch.randn((N, J), generator=g, device=DEV)
    active = [p != 1 for p in range(P)] if dead else None
    Ul, Vl = U.double(), V.double()
    if dead:
        U[B:2 * B] = float("inf")
        V[B:2 * B] = float("nan")
        Ul[B:2 * B] = 0.0
        Vl[B:2 * B] = 0.0
    ctx = sfb.Sfb("mlr", J, D, P, B, dtype="bf16", device=DEV)
    if plan:
        ctx.set_plan(**plan)
    W2 = strided(W, pad, shift)
    around = W2.untyped_storage()
    ctx.reconstruct_apply_prox(W2, strided(U, pad, shift), strided(V, pad, shift), 0.25, kind, 0.04, scale=0.5, active=active)
    ctx.sync()
    assert ctx.last_kernel(2) == ("nt_bf16_kernel", -(-J // 256) * -(-D // 128)) and ctx.plan_info()["recon_grid"] == ctx.last_kernel(2)[1]
    want = W.double() - 0.125 * (Ul.T @ Vl)
    room = 0.125 * 2.0 ** -8 * (Ul.abs().T @ Vl.abs()) + 2.0 ** -22 * (want.abs() + 1.0)
    assert ((W2.double() - prox(kind, want, 0.25 * 0.04)).abs() <= room).all()
    if pad:                                              # nothing but W's own entries was written
        flat = torch.empty(0, device=DEV).set_(around)
        assert int(torch.isnan(flat).sum()) == flat.numel() - J * D
    ctx.close()


def test_slices_of_the_pairs_add_up_and_one_worker_takes_its_own():
    J, D, P, B = 192, 200, 16, 80                        # few tiles, 20 chunks of pairs: planes of sums
    V, W, _, g = batch(J, D, P * B, 3)
    U = torch.randn((P * B, J), generator=g, device=DEV)
    ctx = sfb.Sfb("mlr", J, D, P, B, dtype="bf16", device=DEV)
    W1 = W.clone()
    ctx.reconstruct_apply(W1, U, V, eta=1.0, scale=1.0)
    ctx.sync()
    assert ctx.last_kernel(2)[0] == "update_bf16_kernel" and ctx.last_kernel(2)[1] > 3 * 4
    again = W.clone()
    ctx.reconstruct_apply(again, U, V, eta=1.0, scale=1.0)
    W2 = W.clone()
    for p in range(P):
        ctx.reconstruct_apply_worker(W2, U, V, p, eta=1.0, scale=1.0)
    ctx.sync()
    assert torch.equal(W1, again)
    room = 2.0 ** -20 * (U.abs().T.double() @ V.abs().double()) + 1e-5       # the same rounded factors, other orders of fp32 sums
    assert ((W1 - W2).abs() <= room).all()
    ctx.close()


@pytest.mark.parametrize("J,D,P,B", [(256, 435, 8, 128), (86, 239, 16, 71), (265, 373, 4, 193)])
def test_sliced_update_stays_inside_a_workspace_that_a_plan_has_made_smaller(J, D, P, B):
    """The bytes that the context asks for after a plan of one slice are all that the update writes: what lies behind them in
    the same allocation stays as it was."""
    import ctypes as C
    lib, N, guard = sfb.lib, P * B, 4 << 20
    V, W, _, g = batch(J, D, N, J + D)
    U = torch.randn((N, J), generator=g, device=DEV)
    ctx = sfb.Sfb("mlr", J, D, P, B, dtype="bf16", device=DEV)
    ctx.set_plan(fwd_split_k=1)
    need = ctx.workspace_bytes()
    held = torch.full((need + guard,), 0xA5, dtype=torch.uint8, device=DEV)
    assert held.data_ptr() % 256 == 0 and lib.sfb_set_workspace(ctx._ctx, C.c_void_p(held.data_ptr()), need) == 0
    got = W.clone()
    ctx.reconstruct_apply(got, U, V, eta=0.25, scale=0.5)
    ctx.sync()
    assert (held[need:] == 0xA5).all()
    room = 0.125 * 2.0 ** -8 * (U.double().abs().T @ V.double().abs()) + 2.0 ** -22 * (W.double().abs() + 1.0)
    assert ((got.double() - (W.double() - 0.125 * (U.double().T @ V.double()))).abs() <= room).all()
    ctx.close()


def test_values_without_a_three_term_split():
    """A class switched off by minus infinity scores minus infinity against positive features (the split's second term would
    be NaN), and a finite weight that rounds to an infinity in bf16 stays finite."""
    J, D, P, B = 70, 100, 2, 30
    A, W, y, _ = batch(J, D, P * B, 8)
    A = A.abs() + torch.tensor(0.01, dtype=torch.bfloat16, device=DEV)
    y.clamp_(min=2)
    W[0] = -float("inf")
    W[1] = 0.0
    W[1, 5] = -3.39e38
    want = residual(W, A, y)
    ctx = sfb.Sfb("mlr", J, D, P, B, dtype="bf16", device=DEV)
    U, V = torch.zeros((P * B, J), device=DEV), torch.zeros_like(A)
    ctx.compute_factors(W, sfb.SfbBatch(a=A), y, U, V)
    ctx.sync()
    assert ctx.last_kernel(0)[0] == "scores_bf16_kernel"
    assert ((U.double() - want).norm() / want.norm()).item() < 4e-6
    assert (U[:, :2] == 0).all()
    ctx.close()

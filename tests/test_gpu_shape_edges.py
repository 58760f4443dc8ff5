"""The kernels that a context picks by size, each at the edges of its range, against the fp64 oracle."""
import numpy as np
import pytest
import torch

import oracle
import workloads
from gpu_util import alloc_factors, assert_close, fresh_update, run_chain, to_device

pytestmark = pytest.mark.gpu

TOL32 = 1e-4


def _one_step(wl, active, plan=None, prox=None, update=None):
    """One step with a mask of live workers (and a proximal operator), W and the update alone against the oracle.
    update: the kernel that the step's update has to run."""
    import paper_1511_08486_amd as sfb
    dev = "cuda:0"
    ctx = sfb.Sfb(wl.model, wl.J, wl.D, wl.P, wl.B, dtype=wl.dtype, device=dev)
    if plan:
        ctx.set_plan(**plan)
    db, dy = to_device(wl, wl.batch(0), dev)
    W = torch.from_numpy(wl.W0).to(dev)
    U, V, loss = alloc_factors(wl, dev)
    Uo, Vo, want, fo = oracle.step(wl.model, wl.W0, wl.batch(0), wl.P, wl.B, wl.eta, active=active)
    if prox:
        ctx.step_prox(W, db, dy, U, V, wl.eta, prox[0], prox[1], loss=loss, active=active)
        want = {"l2sq": lambda w: w / (1 + wl.eta * prox[1]),
                "l1": lambda w: np.sign(w) * np.maximum(np.abs(w) - wl.eta * prox[1], 0)}[prox[0]](want)
    else:
        ctx.step(W, db, dy, U, V, wl.eta, loss=loss, active=active)
    ctx.sync()
    if update:
        assert ctx.last_kernel(2)[0] == update
    tol = TOL32 if wl.dtype == "f32" else 2e-2
    for got, exact, what in ((W, want, "W"), (U, Uo, "U"), (V.float(), Vo, "V"), (loss, fo, "loss")):
        assert_close(got.cpu().numpy(), exact, tol, what)
    mag = wl.eta * oracle.delta_w(np.abs(Uo), np.abs(Vo), wl.P, wl.B, active)
    upd = fresh_update(ctx, U, V, wl.eta, W, active=active)
    assert_close(upd.cpu().numpy(), -wl.eta * oracle.delta_w(Uo, Vo, wl.P, wl.B, active), tol, "update", terms=mag)
    ctx.close()


@pytest.mark.parametrize("name,J,D,P,B,active,prox", [
    ("mlr_tiny", 1, 4, 1, 1, None, None),                       # smallest
    ("mlr_tiny", 16, 67, 3, 5, [1, 0, 1], None),                # one workgroup, one block of classes
    ("mlr_tiny", 17, 131, 2, 33, [0, 1], ("l1", 0.05)),         # just over 64 samples: planes; second block of classes
    ("mlr_tiny", 32, 2048, 5, 16, None, ("l2sq", 0.5)),         # most classes, longest rows
    ("mlr_tiny", 10, 784, 7, 613, [1, 1, 0, 1, 1, 1, 1], None),  # many samples, the last workgroup short
    ("dml", 20, 1024, 3, 31, None, None),
    ("dml", 31, 133, 2, 16, [1, 0], None),
])
def test_few_classes(name, J, D, P, B, active, prox):
    _one_step(workloads.make(name, seed=J + D, J=J, D=D, P=P, B=B), active, prox=prox, update="few_step_kernel")


def test_few_classes_bf16():
    _one_step(workloads.make("mlr_large", seed=3, J=19, D=258, P=4, B=37), [1, 1, 0, 1], update="few_step_kernel")


@pytest.mark.parametrize("J,D,P,B,active", [
    (4, 4, 1, 33, None),                                        # smallest, a second chunk of one pair
    (65, 63, 3, 350, [1, 0, 1]),                                # two tiles, slices of the pairs, a dead worker
    (130, 257, 3, 7, None),                                     # every tile ragged, last columns alone in theirs
    (354, 66, 2, 1000, [1, 1]),                                 # slices, an unaligned last pair of columns
    (129, 1030, 1, 2050, None),
])
def test_split_products(J, D, P, B, active):
    _one_step(workloads.make("mlr_tiny", seed=J + D, J=J, D=D, P=P, B=B), active, plan=dict(fwd_dma=13),
              update="reconstruct_split_kernel")


@pytest.mark.parametrize("J,D,P,B,active,density", [
    (33, 65, 1, 1, None, 0.5),                                  # one pair
    (31, 4097, 4, 100, [1, 0, 1, 1], 0.01),                     # empty columns, a dead worker
    (129, 600, 2, 512, None, 0.03),                             # the most pairs, classes over several blocks
])
def test_update_from_the_stored_entries(J, D, P, B, active, density):
    wl = workloads.make("l2svm", seed=J, J=J, D=D, P=P, B=B, density=density)
    _one_step(wl, active, plan=dict(fwd_dma=65), update="sparse_update_kernel")


@pytest.mark.parametrize("J,D,long,repeats", [(600, 4096, 300, 4), (1001, 2003, 64, 2)])
def test_update_from_the_stored_entries_with_row_pointers_that_overlap(J, D, long, repeats):
    """Row pointers that step back share their entries: V then holds more non-zeros than are stored, and the lists have no
    room for some columns.  Nothing is read beyond them, and W is what the rows make it."""
    import paper_1511_08486_amd as sfb
    dev, P, B, eta = "cuda:0", 2, 512, 0.05
    N, rng = P * B, np.random.default_rng(J)
    stored = long * repeats
    rowptr = np.array([long * ((r // 2) % repeats) + (long if r % 2 else 0) for r in range(N + 1)], dtype=np.int32)
    col = np.concatenate([rng.choice(D, size=long, replace=False) for _ in range(repeats)]).astype(np.int32)
    val = np.abs(rng.standard_normal(stored)).astype(np.float32)
    V0 = np.zeros((N, D), np.float32)
    for r in range(N):                                           # (odd rows that step back are empty)
        at = slice(int(rowptr[r]), max(int(rowptr[r]), int(rowptr[r + 1])))
        V0[r, col[at]] = val[at]
    assert np.count_nonzero(V0) > 100 * stored
    W0 = (0.1 * rng.standard_normal((J, D))).astype(np.float32)
    y = rng.integers(0, J, size=N).astype(np.int32)
    ctx = sfb.Sfb("l2svm", J, D, P, B, device=dev)
    up = lambda x: torch.from_numpy(x).to(dev)                   # noqa: E731
    W, U, V = up(W0), torch.empty((N, J), device=dev), torch.empty((N, D), device=dev)
    ctx.step(W, sfb.SfbBatch(rowptr=up(rowptr), col=up(col), val=up(val)), up(y), U, V, eta)
    ctx.sync()
    assert ctx.last_kernel(2)[0] == "sparse_update_kernel"
    assert np.array_equal(V.cpu().numpy(), V0)
    _, Uo = oracle.loss_and_u("l2svm", V0.astype(np.float64) @ W0.astype(np.float64).T, y)
    assert_close(U.cpu().numpy(), Uo, TOL32, "U")
    got, U64, V64 = W.cpu().numpy(), U.cpu().numpy().astype(np.float64), V0.astype(np.float64)
    assert_close(got, W0 - eta / B * (U64.T @ V64), TOL32, "W", terms=eta / B * (np.abs(U64).T @ V64))
    ctx.close()


def test_update_from_the_stored_entries_with_infinite_factors():
    """Infinite factors make NaN against every zero of the features, whether or not it is stored, as in the dense update."""
    import paper_1511_08486_amd as sfb
    wl = workloads.make("l2svm", seed=7, J=600, D=4096, P=2, B=512, density=0.01)
    dev = "cuda:0"
    ctx = sfb.Sfb(wl.model, wl.J, wl.D, wl.P, wl.B, device=dev)
    db, dy = to_device(wl, wl.batch(0), dev)
    W0 = wl.W0.copy()
    W0[40, int(torch.bincount(db.col.cpu()).argmax())] = np.inf  # infinite scores of the samples that have this feature
    W = torch.from_numpy(W0).to(dev)
    U, V, loss = alloc_factors(wl, dev)
    ctx.step(W, db, dy, U, V, wl.eta, loss=loss)
    ctx.sync()
    assert ctx.last_kernel(2)[0] == "sparse_update_kernel"
    U64, V64 = U.cpu().numpy().astype(np.float64), V.cpu().numpy().astype(np.float64)
    assert not np.isfinite(U64[:, 40]).all() and np.isfinite(np.delete(U64, 40, 1)).all()
    with np.errstate(invalid="ignore"):
        want = W0 - wl.eta * ctx.default_scale() * (U64.T @ V64)
    got = W.cpu().numpy()
    assert np.isnan(want[40]).all() and np.isnan(got[40]).all()
    rest = np.arange(wl.J) != 40
    assert_close(got[rest], want[rest], TOL32, "W")
    ctx.close()


@pytest.mark.parametrize("J,D", [(1000, 4100), (600, 4096)])
def test_update_from_the_stored_entries_leaves_out_whatever_a_dead_worker_holds(J, D):
    """NaN and infinities among a dead worker's features: W is what it is with finite values in their place."""
    import paper_1511_08486_amd as sfb
    wl = workloads.make("l2svm", seed=11, J=J, D=D, P=8, B=64, density=0.02)
    active = [1, 1, 0, 1, 1, 1, 1, 1]
    b, got = wl.batch(0), []
    for bad in (False, True):
        val = np.array(b["val"])
        if bad:
            mine = slice(int(b["rowptr"][2 * wl.B]), int(b["rowptr"][3 * wl.B]))
            val[mine] = np.resize(np.float32([np.nan, np.inf, -np.inf]), val[mine].shape)
        ctx = sfb.Sfb(wl.model, J, D, wl.P, wl.B, device="cuda:0")
        db, dy = to_device(wl, dict(b, val=val), "cuda:0")
        W = torch.from_numpy(wl.W0).to("cuda:0")
        U, V, loss = alloc_factors(wl, "cuda:0")
        ctx.step(W, db, dy, U, V, wl.eta, loss=loss, active=active)
        ctx.sync()
        assert ctx.last_kernel(2)[0] == "sparse_update_kernel"
        got.append(W)
        ctx.close()
    _, _, want, _ = oracle.step(wl.model, wl.W0, b, wl.P, wl.B, wl.eta, active=active)
    assert_close(got[0].cpu().numpy(), want, TOL32, "W")
    assert torch.equal(got[0], got[1])


@pytest.mark.parametrize("J,D,P,B,active,prox", [
    (33, 130, 1, 28, None, None),                               # a block of one row, one of two columns
    (64, 4099, 1, 1, None, ("l1", 0.05)),                       # one pair
    (131, 65, 3, 21, [1, 0, 1], None),                          # a dead worker, the last stage short by one
    (97, 1000, 4, 16, None, ("l2sq", 0.5)),                     # four whole stages
    (257, 203, 1, 65, None, None),                              # more than one stage's worth over 64
    (77, 515, 2, 64, None, None),                               # the most pairs
])
def test_few_pairs(J, D, P, B, active, prox):
    _one_step(workloads.make("mlr_tiny", seed=J + D, J=J, D=D, P=P, B=B), active, prox=prox, update="reconstruct_thin_kernel")


def test_many_pairs_on_few_tiles_are_spread_over_the_chip():
    """100 x 192 with 2048 pairs: whole 64-column tiles, but rows that other calls copy into padded ones.  The fp32
    instruction's kernel would walk all pairs in six workgroups there, its slices are for the copies; the costs know."""
    import paper_1511_08486_amd as sfb
    J, D, P, B, dev = 100, 192, 8, 256, "cuda:0"
    rng = np.random.default_rng(1)
    Uh, Vh = rng.standard_normal((P * B, J)).astype(np.float32), rng.standard_normal((P * B, D)).astype(np.float32)
    ctx = sfb.Sfb("dml", J, D, P, B, device=dev)
    W = torch.zeros((J, D), device=dev)
    ctx.reconstruct_apply(W, torch.from_numpy(Uh).to(dev), torch.from_numpy(Vh).to(dev), 0.1, scale=1.0)
    ctx.sync()
    assert ctx.last_kernel(2)[1] >= 64
    U64, V64 = Uh.astype(np.float64), Vh.astype(np.float64)
    assert_close(W.cpu().numpy(), -0.1 * (U64.T @ V64), TOL32, "W", terms=0.1 * (np.abs(U64).T @ np.abs(V64)))
    ctx.close()


@pytest.mark.parametrize("J,D,P,B,masked,kernel", [
    (37, 203, 3, 5, False, "reconstruct_thin_kernel"),          # ragged and small
    (37, 203, 3, 5, True, "reconstruct_thin_kernel"),
    (60, 90, 3, 60, False, "reconstruct_split_kernel"),         # 5 and 3 us less than a copy of the factors and a kernel
    (260, 512, 4, 32, True, "reconstruct_split_kernel"),        # whole, but masked
])
def test_small_calls_leave_no_copies_of_their_factors(J, D, P, B, masked, kernel):
    """Calls that the fp32 instruction's kernels take by way of a copy only: other kernels take them as they are."""
    wl = workloads.make("l2svm", seed=J, J=J, D=D, P=P, B=B, density=0.5)
    _one_step(wl, [p != 1 for p in range(P)] if masked else None, update=kernel)


# Values that no three bf16 terms hold: infinities, and finite ones that round to an infinity in bf16.  What is infinite, or
# as finite as in fp32, stays so; a whole row or column that depends on them is compared with numpy in fp64.
@pytest.mark.parametrize("J,D,N", [(66, 130, 70), (130, 1030, 200), (200, 515, 1030)])
@pytest.mark.parametrize("big", [float("-inf"), -3.4028e38])
def test_split_products_of_unbounded_values(J, D, N, big):
    import paper_1511_08486_amd as sfb
    dev = "cuda:0"
    wl = workloads.make("mlr_tiny", seed=J, J=J, D=D, P=1, B=N)
    ctx = sfb.Sfb("mlr", J, D, 1, N, device=dev)
    ctx.set_plan(fwd_dma=13)
    A = np.abs(np.random.default_rng(J).standard_normal((N, D))).astype(np.float32) / np.float32(np.sqrt(D)) + np.float32(1e-3)
    A[:, 5] = 1.0
    y = torch.zeros(N, dtype=torch.int32, device=dev)
    W0 = wl.W0.copy()
    W0[3, 5] = W0[J - 1, 5] = big                               # classes that are switched off by a feature that is always one
    W, a = torch.from_numpy(W0).to(dev), sfb.SfbBatch(a=torch.from_numpy(A).to(dev))
    U, V, loss = torch.empty((N, J), device=dev), torch.empty((N, D), device=dev), torch.empty(N, device=dev)
    ctx.compute_factors(W, a, y, U, V, loss=loss)
    ctx.sync()
    z = A.astype(np.float64) @ W0.astype(np.float64).T
    p = np.exp(z - z.max(1, keepdims=True))
    want_loss = np.log(p.sum(1)) + z.max(1) - z[:, 0]
    p /= p.sum(1, keepdims=True)
    p[:, 0] -= 1.0
    assert_close(U.cpu().numpy(), p, TOL32, "U")
    assert_close(loss.cpu().numpy(), want_loss, TOL32, "loss")

    V0 = A.copy()
    V0[N - 1, D - 1] = V0[2, 7] = big                            # one entry of each of two columns
    U0 = (np.random.default_rng(N).uniform(0.25, 0.5, (N, J)) / N).astype(np.float32)
    W1 = torch.from_numpy(wl.W0).to(dev)
    ctx.reconstruct_apply(W1, torch.from_numpy(U0).to(dev), torch.from_numpy(V0).to(dev), 0.5, scale=1.0)
    ctx.sync()
    want, got = wl.W0 - 0.5 * (U0.astype(np.float64).T @ V0.astype(np.float64)), W1.cpu().numpy().astype(np.float64)
    cols = np.isin(np.arange(D), [7, D - 1])
    assert_close(got[:, ~cols], want[:, ~cols], TOL32, "W")
    if np.isinf(big):
        assert np.array_equal(got[:, cols], want[:, cols])
    else:
        assert_close(got[:, cols], want[:, cols], TOL32, "columns of large values")
    ctx.close()


def _split_update(J, D, P, B, V0, active=None, seed=0, chosen=True):
    """W after one update formed as split products (chosen by the caller, or by the costs), what it should be (numpy, fp64), and its workgroups."""
    import paper_1511_08486_amd as sfb
    N, rng = P * B, np.random.default_rng(seed)
    U0 = (rng.uniform(0.25, 0.5, (N, J)) / N).astype(np.float32)
    W0 = (0.1 * rng.standard_normal((J, D))).astype(np.float32)
    ctx = sfb.Sfb("mlr", J, D, P, B, device="cuda:0")
    if chosen:
        ctx.set_plan(fwd_dma=13)
    W = torch.from_numpy(W0).to("cuda:0")
    U, V = torch.from_numpy(U0).to("cuda:0"), torch.from_numpy(V0).to("cuda:0")
    ctx.reconstruct_apply(W, U, V, 0.5, scale=1.0, active=active)
    ctx.sync()
    name, grid = ctx.last_kernel(2)
    assert name == "reconstruct_split_kernel"
    ctx.close()
    live = np.repeat(np.ones(P, bool) if active is None else np.asarray(active, bool), B)
    return W.cpu().numpy().astype(np.float64), W0 - 0.5 * (U0[live].astype(np.float64).T @ V0[live].astype(np.float64)), grid


@pytest.mark.parametrize("J,D,P,B,tile,sliced,chosen", [
    (515, 2051, 4, 64, (64, 128), False, True),                 # an odd last column
    (515, 2051, 4, 64, (64, 128), False, False),
    (1001, 4093, 6, 85, (128, 128), False, False),
    (600, 4095, 4, 100, (128, 128), False, False),              # thirteen chunks: one more than whole rounds of three
    (602, 779, 3, 343, (64, 128), True, True),                  # slices of the pairs
    (602, 779, 3, 343, (64, 128), True, False),
    (65, 66, 3, 350, (64, 64), True, True),
    (65, 66, 3, 350, (64, 64), True, False),
])
@pytest.mark.parametrize("masked", [False, True])
def test_split_update_with_infinities_in_one_of_two_neighbouring_columns(J, D, P, B, tile, sliced, chosen, masked):
    """Infinities in single columns, the last one among them, and, with a mask, NaN in everything a dead worker left: the
    neighbours of such a column and every other entry are those of finite features."""
    rng = np.random.default_rng(D)
    V0 = np.abs(rng.standard_normal((P * B, D))).astype(np.float32)
    active = [p != 1 for p in range(P)] if masked else None
    if masked:
        V0[B:2 * B] = np.nan
    V0[2, 6], V0[3, 37], V0[P * B - 1, D - 1] = np.inf, -np.inf, np.inf
    got, want, grid = _split_update(J, D, P, B, V0, active, seed=J, chosen=chosen)
    tiles = -(-J // tile[0]) * -(-D // tile[1])
    assert grid % tiles == 0 and (grid > tiles) == sliced
    cols = np.isin(np.arange(D), [6, 37, D - 1])
    assert np.array_equal(got[:, cols], want[:, cols])
    assert_close(got[:, ~cols], want[:, ~cols], TOL32, "W")


@pytest.mark.parametrize("J,D,N", [(1000, 4096, 512), (520, 1024, 256), (100, 780, 1024)])
def test_split_products_that_were_chosen_keep_the_smaller_terms_apart(J, D, N):
    """Their running sums are rounded once for every sixteen products, as the bits of sfb_set_plan have always given:
    1.4e-7 and 1.3e-7 of the norm at 1000 x 4096, where six roundings leave 2.5e-7 and 2.4e-7."""
    import paper_1511_08486_amd as sfb
    g = torch.Generator().manual_seed(J)
    W, A, U0, V0 = (torch.randn(*s, generator=g).to("cuda:0") for s in ((J, D), (N, D), (N, J), (N, D)))
    ctx = sfb.Sfb("dml", J, D, N // 32, 32, device="cuda:0")
    ctx.set_plan(fwd_dma=13)
    U, V, W1 = torch.empty_like(U0), torch.empty_like(V0), torch.zeros_like(W)
    similar = torch.ones(N, dtype=torch.int32, device="cuda:0")  # u = 2 z
    ctx.compute_factors(W, sfb.SfbBatch(a=A, a2=torch.zeros_like(A)), similar, U, V)
    ctx.reconstruct_apply(W1, U0, V0, -1.0, scale=1.0)
    ctx.sync()
    ctx.close()
    errs = []
    for got, want in ((0.5 * U, A.double() @ W.double().T), (W1, U0.double().T @ V0.double())):
        errs.append(float((got.double() - want).norm() / want.norm()))
    print("error of scores and update", errs)
    assert max(errs) < 1.8e-7


@pytest.mark.parametrize("J,D,N,kernel", [
    (600, 4096, 1024, "reconstruct_split_kernel"),              # stand-ins for the kernel that cuts every sum in four
    (1160, 2048, 1088, "reconstruct_split_kernel"),
    (600, 4096, 128, "reconstruct_thin_kernel"),
    (1000, 4096, 64, "reconstruct_thin_kernel"),                # ... in two
    (1000, 4096, 512, "reconstruct_split_kernel"),
    (300, 1000, 128, "reconstruct_thin_kernel"),                # ... that does not cut them
])
@pytest.mark.parametrize("positive", [False, True])
def test_updates_are_as_accurate_as_with_the_fp32_instruction_kernels(J, D, N, kernel, positive):
    """Error of the default update against fp64, of the norm: no larger than that of the kernels the caller can have instead
    (2 % for the rounding of the result)."""
    import paper_1511_08486_amd as sfb
    g = torch.Generator().manual_seed(J + N)
    draw = (lambda *s: torch.rand(*s, generator=g) + 0.1) if positive else (lambda *s: torch.randn(*s, generator=g))
    U, V = draw(N, J).to("cuda:0"), draw(N, D).to("cuda:0")
    want, errs = U.double().T @ V.double(), []
    for plan in (None, dict(fwd_dma=1)):
        ctx = sfb.Sfb("mlr", J, D, N // 32, 32, device="cuda:0")
        if plan:
            ctx.set_plan(**plan)
        W = torch.zeros((J, D), device="cuda:0")
        ctx.reconstruct_apply(W, U, V, -1.0, scale=1.0)
        ctx.sync()
        assert plan or ctx.last_kernel(2)[0] == kernel
        errs.append(float((W.double() - want).norm() / want.norm()))
        ctx.close()
    print("error: default", errs[0], "fp32 instruction", errs[1])
    assert errs[0] <= 1.02 * errs[1]


def test_classes_switched_off_by_infinite_weights_do_not_stall_the_split_products():
    """One class of a thousand with a weight of minus infinity on a feature that is always one, and one feature that is
    infinite: scores and update are formed again by the fp32 instruction in the tiles concerned.  The bound is eight times
    the time without them (2.1 and 3.7 measured; 22 and 82 where a lane sums such an entry alone)."""
    import paper_1511_08486_amd as sfb
    J, D, P, B, dev = 1000, 4096, 8, 64, "cuda:0"
    rng = np.random.default_rng(0)
    A = torch.from_numpy((rng.standard_normal((P * B, D)) / 64).astype(np.float32)).to(dev)
    A[:, 5] = 1.0
    y = torch.full((P * B,), J - 1, dtype=torch.int32, device=dev)
    ctx = sfb.Sfb("mlr", J, D, P, B, device=dev)
    U, V = torch.empty((P * B, J), device=dev), torch.empty((P * B, D), device=dev)

    def us(call, n=20):
        out = []
        for _ in range(7):
            a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            a.record()
            for _ in range(n):
                call()
            b.record()
            torch.cuda.synchronize()
            out.append(a.elapsed_time(b) * 1e3 / n)
        return sorted(out)[3]

    times = []
    for bad in (False, True):
        W = torch.from_numpy((0.1 * rng.standard_normal((J, D))).astype(np.float32)).to(dev)
        F = A.clone()
        if bad:
            W[3, 5], F[3, 9] = -float("inf"), float("inf")
        Z = torch.zeros((J, D), device=dev)
        scores = us(lambda: ctx.compute_factors(W, sfb.SfbBatch(a=A), y, U, V))
        assert bool(torch.isfinite(U).all()) and (not bad or bool((U[:, 3] == 0).all()))
        times.append((scores, us(lambda: ctx.reconstruct_apply(Z, U, F, 1e-3))))
    print("scores and update, us: finite", times[0], "with infinities", times[1])
    ctx.close()
    assert times[1][0] < 8 * times[0][0] and times[1][1] < 8 * times[0][1]


@pytest.mark.parametrize("J,D,P,B,grid", [
    (1001, 4100, 8, 61, 256),                                   # 256 tiles of 128 x 128 and four columns
    (1030, 4096, 8, 64, 256),                                   # ... and six rows
    (1001, 4129, 4, 130, 256),                                  # ... and 33 columns
    (600, 4096, 4, 128, 224),                                   # tiles of 96 rows
    (1152, 2750, 6, 90, 198),
])
@pytest.mark.parametrize("masked,kind", [(False, "none"), (True, "none"), (False, "l1"), (True, "l2sq")])
def test_updates_whose_last_tiles_are_a_launch_of_their_own(J, D, P, B, grid, masked, kind):
    """Every entry against fp64, with infinities in the last column and row, in rows of W that have words between them.  Sums of
    N products rounded six times for every sixteen: 2^-24 (6 N / 16 + 2) sum |u v|, and the update's own rounding."""
    import paper_1511_08486_amd as sfb
    dev, N, g = "cuda:0", P * B, torch.Generator(device="cuda:0").manual_seed(J)
    U, V = torch.randn((N, J), generator=g, device=dev), torch.randn((N, D), generator=g, device=dev)
    W = torch.randn((J, D + 3), generator=g, device=dev)
    W[:, D:] = float("nan")
    W0, active = W.clone(), [p != 1 for p in range(P)] if masked else None
    U[3, J - 1] = V[5, D - 1] = float("inf")
    if masked:
        U[B:2 * B] = float("nan")
    live = torch.ones(N, dtype=torch.bool, device=dev)
    if masked:
        live[B:2 * B] = False
    ctx = sfb.Sfb("l2svm", J, D, P, B, device=dev)
    ctx.reconstruct_apply_prox(W[:, :D], U, V, 0.5, kind, 0.04, scale=1.0, active=active)
    ctx.sync()
    name, blocks = ctx.last_kernel(2)
    assert name == "reconstruct_split_kernel" and blocks == grid
    Ul, Vl = U[live].double(), V[live].double()
    want, got = W0[:, :D].double() - 0.5 * (Ul.T @ Vl), W[:, :D].double()
    if kind == "l2sq":                                          # entry by entry, differences no larger than before
        want = want / (1.0 + 0.5 * 0.04)
    if kind == "l1":                                            # (what is neither above nor below the threshold is 0, NaN too)
        want = torch.where(want > 0.02, want - 0.02, torch.where(want < -0.02, want + 0.02, torch.zeros_like(want)))
    assert torch.equal(torch.isnan(got), torch.isnan(want)) and torch.equal(got[torch.isinf(want)], want[torch.isinf(want)])
    room = 0.5 * 2.0 ** -24 * (6 * N / 16 + 2) * (Ul.abs().T @ Vl.abs()) + 2.0 ** -23 * want.abs()
    ok = torch.isfinite(want)
    assert ((got - want)[ok].abs() <= room[ok]).all()
    assert torch.isnan(W[:, D:]).all()
    ctx.close()


def test_rows_of_scores_whose_offsets_pass_32_bits():
    """Twelve rows of 90 million classes are more than 2^32 bytes: every row of a block of sixteen, entry by entry, is its own product
    (four columns: four products of 2^-24 each and three sums)."""
    import paper_1511_08486_amd as sfb
    dev, J, D, N = "cuda:0", 89_500_003, 4, 16
    g = torch.Generator(device=dev).manual_seed(1)
    W, A = torch.randn((J, D), generator=g, device=dev), torch.randn((N, D), generator=g, device=dev)
    U, V = torch.full((N, J), float("nan"), device=dev), torch.empty((N, D), device=dev)
    ctx = sfb.Sfb("dml", J, D, 1, N, device=dev)
    ctx.compute_factors(W, sfb.SfbBatch(a=A, a2=torch.zeros_like(A)), torch.ones(N, dtype=torch.int32, device=dev), U, V)
    ctx.sync()                                                   # similar pairs: u = 2 z
    assert ctx.last_kernel(0)[0] == "scores_split_kernel"
    ctx.close()
    for j in range(0, J, 1 << 22):
        w, u = W[j:j + (1 << 22)].double(), U[:, j:j + (1 << 22)].double()
        assert ((0.5 * u - A.double() @ w.T).abs() <= 8 * 2.0 ** -24 * (A.double().abs() @ w.abs().T)).all()

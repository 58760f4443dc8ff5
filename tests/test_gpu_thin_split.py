"""Updates from 17 to 64 pairs, as split products (256 tiles of 64 x 64 and more) and, on a smaller W, by the fp32 instruction: edges of tiles, rows at any alignment, dead workers, infinities, against fp64.

Bound of an entry: what the split drops is below 2^-24 |u v| a product and the leading sums are rounded four times, the small ones
twenty times at 2^-8 of their size: 2^-22 sum |u v|, and a unit in the last place of the result for the update itself."""
import pytest
import torch

import paper_1511_08486_amd as sfb
from test_gpu_bf16_tiles import strided

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


@pytest.mark.parametrize("J,D,P,B", [
    (4, 16450, 2, 9), (16451, 5, 3, 6), (63, 16513, 2, 16), (1025, 1027, 3, 11), (1030, 1090, 2, 17), (1090, 1025, 4, 12), (1000, 2050, 4, 16),
    (2100, 3200, 2, 30), (66, 131, 2, 17), (130, 258, 4, 12),
])
@pytest.mark.parametrize("pad,shift,dead,kind", [(1, 1, False, "none"), (2, 3, True, "l1"), (0, 0, True, "none"), (0, 0, False, "l2sq")])
def test_update(J, D, P, B, pad, shift, dead, kind):
    N = P * B
    g = torch.Generator(device=DEV).manual_seed(J * D + N)
    U, V, W = (torch.randn(*s, generator=g, device=DEV) for s in ((N, J), (N, D), (J, D)))
    Ul, Vl = U.double(), V.double()
    if dead:
        U[B:2 * B], V[B:2 * B] = float("nan"), float("inf")           # a dead worker's slot may hold anything
        Ul[B:2 * B], Vl[B:2 * B] = 0.0, 0.0
    V[0, D - 1] = Vl[0, D - 1] = -float("inf")                          # its column, and nothing else, is not finite
    ctx = sfb.Sfb("mlr", J, D, P, B, device=DEV)
    W2 = strided(W, pad, shift)
    around = W2.untyped_storage()
    active = [p != 1 for p in range(P)] if dead else None
    ctx.reconstruct_apply_prox(W2, strided(U, pad, shift), strided(V, pad, shift), 0.25, kind, 0.02, scale=0.5, active=active)
    ctx.sync()
    assert ctx.last_kernel(2)[0] == "reconstruct_thin_kernel"
    want = W.double() - 0.125 * (Ul.T @ Vl)
    if kind == "l2sq":
        want = want / (1.0 + 0.25 * 0.02)
    if kind == "l1":
        want = torch.sign(want) * (want.abs() - 0.25 * 0.02).clamp(min=0.0)
    room = 2.0 ** -22 * (0.125 * (Ul.abs().T @ Vl[:, :D - 1].abs()) + W[:, :D - 1].double().abs())
    assert ((W2[:, :D - 1].double() - want[:, :D - 1]).abs() <= room).all()
    assert torch.equal(W2[:, D - 1].double(), want[:, D - 1])
    flat = torch.empty(0, device=DEV).set_(around)                      # nothing but W's own entries was written
    assert int(torch.isnan(flat).sum()) == flat.numel() - J * D
    ctx.close()


@pytest.mark.parametrize("J,D,N,blocks", [
    (768, 4096, 64, 768), (832, 4096, 52, 13 * 32), (832, 4096, 48, 832), (1536, 4096, 48, 1536), (1600, 4096, 20, 25 * 32),       # 16-byte rows
    (401, 2000 + 1, 64, 7 * 32), (601, 2001, 20, 10 * 16),                                                           # unaligned ones
])
def test_split_products_begin_where_they_are_the_faster_ones(J, D, N, blocks):
    """64 x 64 tiles by the fp32 instruction, 64 x 128 as split products, one workgroup each."""
    g = torch.Generator(device=DEV).manual_seed(J + N)
    U, V, W = (torch.randn(*s, generator=g, device=DEV) for s in ((N, J), (N, D), (J, D)))
    ctx = sfb.Sfb("mlr", J, D, 4, N // 4, device=DEV)
    W2 = W.clone()
    ctx.reconstruct_apply(W2, U, V, 0.25, scale=0.5)
    ctx.sync()
    assert ctx.last_kernel(2) == ("reconstruct_thin_kernel", blocks)
    want = W.double() - 0.125 * (U.double().T @ V.double())
    assert ((W2.double() - want).abs() <= 2.0 ** -22 * (0.125 * N ** 0.5 * (U.abs().T @ V.abs()).double() + W.double().abs())).all()
    ctx.close()

"""Models of few classes whose batch is too large for the caches: V leaves the kernel while the products run."""
import pytest
import torch

from test_gpu_bf16_tiles import strided

pytestmark = pytest.mark.gpu

DEV = "cuda:0"


@pytest.mark.parametrize("model,J,D,P,B", [
    ("mlr", 10, 784, 4, 1840),              # just over the line, 29 rows to a workgroup: 6 pieces of V to a thread, one batch of loads
    ("mlr", 16, 783, 12, 1001),             # ragged rows
    ("mlr", 3, 101, 7, 9001),               # more rows than factors at a time, more row blocks than wavefronts
    ("mlr", 20, 257, 3, 8203),              # two class blocks, 97 rows
    ("mlr", 16, 2047, 2, 1501),             # long rows, 12 to 16 of them, more pieces than scores and updates have steps
    ("dml", 10, 300, 5, 4001),
    ("dml", 18, 1021, 2, 3003),
])
@pytest.mark.parametrize("pad,shift,dead", [(0, 0, False), (3, 1, True)])
def test_step_and_factors(model, J, D, P, B, pad, shift, dead):
    """V is exact, and so are its copies in both calls.  Scores, entry by entry, within (D + 8) 2^-23 sum |a w|, whatever the order; the softmax is 1-Lipschitz in them, with
    2^-19 for its own exponentials (arguments to 2^7 in an exponential of base two) and divisions.  The update's longest chain is a
    workgroup's rows, sixteen planes and sixteen sums of those."""
    import paper_1511_08486_amd as sfb
    N, g = P * B, torch.Generator(device=DEV).manual_seed(J + D)
    randn = lambda *s: torch.randn(s, generator=g, device=DEV)  # noqa: E731
    A, W = strided(randn(N, D) / D ** 0.5, pad, shift), randn(J, D)
    y = torch.randint(0, J if model == "mlr" else 2, (N,), generator=g, device=DEV, dtype=torch.int32)
    A2 = strided(randn(N, D) / D ** 0.5, pad, shift) if model == "dml" else None
    active = [1] * P
    if dead:
        active[P - 1] = 0
        A[N - 3] = float("inf")             # whatever a dead worker's rows hold
    X = A - A2 if model == "dml" else A
    live = torch.tensor(active, device=DEV, dtype=torch.bool).repeat_interleave(B)
    ctx = sfb.Sfb(model, J, D, P, B, device=DEV)
    U, V, loss = torch.zeros((N, J), device=DEV), strided(torch.zeros((N, D), device=DEV), pad, shift), torch.zeros(N, device=DEV)
    U2, V2 = torch.zeros_like(U), torch.zeros_like(A)
    batch = sfb.SfbBatch(a=A, a2=A2) if model == "dml" else sfb.SfbBatch(a=A)
    W1 = W.clone()
    ctx.step(W1, batch, y, U, V, 0.5, loss=loss, active=active)
    ctx.sync()
    assert ctx.last_kernel(2)[0] == "few_step_kernel"
    ctx.compute_factors(W, batch, y, U2, V2)
    ctx.sync()
    assert torch.equal(V, X) and torch.equal(V2, X)
    x, w, yl = X[live].double(), W.double(), y[live].long()
    z, room = x @ w.T, (D + 8) * 2.0 ** -23 * (x.abs() @ w.abs().T)
    if model == "mlr":
        u, room = torch.softmax(z, 1), room.amax(1, keepdim=True) + 2.0 ** -19
        u[torch.arange(len(yl), device=DEV), yl] -= 1
    else:
        q = (z * z).sum(1, keepdim=True)
        u = torch.where(yl[:, None] != 0, 2 * z, torch.where(q < 1, -2 * z, torch.zeros_like(z)))
        room = 2 * room
        clear = (q - 1).abs()[:, 0] > 1e-3  # (on the edge of the hinge either side is right)
        u, room = u[clear], room[clear]
    for got in (U[live], U2[live]):
        got = got.double() if model == "mlr" else got.double()[clear]
        assert ((got - u).abs() <= room).all()
    ud, rows = U[live].double(), -(-N // 256)
    alpha = 0.5 * ctx.default_scale()
    exact = w - alpha * (ud.T @ x)
    room = (rows + 40) * 2.0 ** -23 * alpha * (ud.abs().T @ x.abs()) + 2.0 ** -23 * w.abs()
    assert ((W1.double() - exact).abs() <= room).all()
    ctx.close()

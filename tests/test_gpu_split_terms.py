"""Split products of two terms: operands whose magnitudes make a workgroup change to three terms at some chunk, or do not."""
import pytest
import torch

pytestmark = pytest.mark.gpu


def _spread(kind, x):
    """x (rows, k) of one scale -> the same with other magnitudes along the contraction."""
    k = x.shape[1]
    if kind == "grows":                     # beyond what the first columns' scale holds, from a middle chunk on
        x[:, (2 * k) // 3:] *= 1e4
    elif kind == "grows at the end":
        x[:, k - 3:] *= 1e6
    elif kind == "zeros first":
        x[:, :100] = 0
    elif kind == "blank but the end":
        x[:, :k - 2] = 0
    elif kind == "magnitudes":
        x *= torch.exp(8 * torch.randn(x.shape, generator=torch.Generator(device=x.device).manual_seed(k), device=x.device))
    elif kind == "small rows":              # far below the largest value, close to it, and none at all
        x[1::7] *= 1e-9
        x[2::7] *= 1e-3
        x[3::7] = 0
    elif kind == "rows in between":         # down to 2^-19 of the largest value, entries of even magnitude
        x.copy_(x.sign() * (1 + 0.5 * x.abs().clamp(max=1)))
        x *= 2.0 ** -(torch.arange(x.shape[0], device=x.device) % 20).float()[:, None]
    elif kind == "large":
        x *= 1e16                           # (twice a sum of 4096 products stays a number)
    elif kind == "small":
        x *= 1e-18
    return x


def _assert_rows_and_columns(got, a, b):
    """got = a b^T, every row and column within 2^-24 (4 + sqrt(k) / 4) of the norm of its products: 4 for the terms of both operands and what
    is left out of their products, and the running sum of an instruction that adds four products, k / 4 roundings of random sign (1.2e-6
    at 4096; the kernels are at 2e-7; without second terms products alone are 3e-4 off)."""
    e, products = got - a @ b.T, (a * a) @ (b * b).T
    for dim in (0, 1):
        assert (e.norm(dim=dim) <= 2.0 ** -24 * (4 + a.shape[1] ** 0.5 / 4) * products.sum(dim=dim).sqrt() + 1e-42).all()


@pytest.mark.parametrize("J,D,P,B", [
    (1000, 4096, 4, 128),                   # 128 x 128 scores, 128 x 128 update
    (600, 4109, 6, 171),                    # ragged D, rows and pairs; 96 x 128 update
    (130, 1503, 4, 63),                     # 64 x 64
    (70, 2001, 10, 321),                    # slices of the pairs
    (2049, 517, 2, 150),
])
@pytest.mark.parametrize("kind", ["grows", "grows at the end", "zeros first", "blank but the end", "magnitudes", "small rows", "rows in between", "large", "small"])
@pytest.mark.parametrize("both", [False, True])
def test_scores_and_updates_over_many_magnitudes(J, D, P, B, kind, both):
    """Row by row and column by column, and entry by entry: sums of K products rounded six times at most for every sixteen, and eight roundings'
    worth for the terms that are left out, 2^-24 (6 K / 16 + 8) sum |a b|; slices of K add theirs within that."""
    import paper_1511_08486_amd as sfb
    dev, N, g = "cuda:0", P * B, torch.Generator(device="cuda:0").manual_seed(J + D)
    randn = lambda *s: torch.randn(s, generator=g, device=dev)  # noqa: E731
    A, A2, W = _spread(kind, randn(N, D)), torch.zeros((N, D), device=dev), randn(J, D)
    if both:
        W = _spread(kind, W)
    y, U, V = torch.ones(N, dtype=torch.int32, device=dev), torch.zeros((N, J), device=dev), torch.full((N, D), float("nan"), device=dev)
    ctx = sfb.Sfb("dml", J, D, P, B, device=dev)
    ctx.compute_factors(W, sfb.SfbBatch(a=A, a2=A2), y, U, V)   # similar pairs: u = 2 z
    ctx.sync()
    assert torch.equal(V, A)
    _assert_rows_and_columns(0.5 * U.double(), A.double(), W.double())
    room = 2.0 ** -24 * (6 * D / 16 + 8) * (A.double().abs() @ W.double().abs().T) + 1e-44
    assert ((0.5 * U.double() - A.double() @ W.double().T).abs() <= room).all()

    Ut, Vt, W1 = _spread(kind, randn(J, N)), randn(D, N), torch.zeros((J, D), device=dev)
    if both:
        Vt = _spread(kind, Vt)
    ctx.reconstruct_apply(W1, Ut.T.contiguous(), Vt.T.contiguous(), -1.0, scale=1.0)
    ctx.sync()
    ctx.close()
    _assert_rows_and_columns(W1.double(), Ut.double(), Vt.double())
    room = 2.0 ** -24 * (6 * N / 16 + 8) * (Ut.double().abs() @ Vt.double().abs().T) + 1e-44
    assert ((W1.double() - Ut.double() @ Vt.double().T).abs() <= room).all()


@pytest.mark.parametrize("k", [32 * 12, 32 * 13 + 5, 32 * 14, 32 * 17 + 31])
def test_the_split_changes_at_any_chunk(k):
    """Walks of every remainder of three chunks, left by one operand's values at each chunk in turn."""
    import paper_1511_08486_amd as sfb
    dev, J, D, N, g = "cuda:0", 1000, 4096, 2048, torch.Generator(device="cuda:0").manual_seed(k)
    randn = lambda *s: torch.randn(s, generator=g, device=dev)  # noqa: E731
    u, v, w, a = randn(k, J), randn(k, D), randn(J, k), randn(N, k)
    update, scores = sfb.Sfb("dml", J, D, 1, k, device=dev), sfb.Sfb("dml", J, k, 1, N, device=dev)
    W1, U, V, y = torch.empty((J, D), device=dev), torch.empty((N, J), device=dev), torch.empty((N, k), device=dev), torch.ones(N, dtype=torch.int32, device=dev)
    for c in range(2, k // 32 + 1):
        for grown, still in ((u, v), (v, u)):
            x = grown.clone()
            x[32 * c:] *= 1e4
            U1, V1 = (x, still) if grown is u else (still, x)
            update.reconstruct_apply(W1.zero_(), U1, V1, -1.0, scale=1.0)
            update.sync()
            _assert_rows_and_columns(W1.double(), U1.double().T, V1.double().T)
        x = a.clone()
        x[:, 32 * c:] *= 1e4
        scores.compute_factors(w, sfb.SfbBatch(a=x, a2=torch.zeros_like(x)), y, U, V.fill_(float("nan")))
        scores.sync()
        assert torch.equal(V, x)
        _assert_rows_and_columns(0.5 * U.double(), x.double(), w.double())
    update.close()
    scores.close()


@pytest.mark.parametrize("chosen,positive,J,D,N,most", [
    (False, True, 1000, 4096, 4096, 2.2e-7),      # 3.0e-7 in one running sum (n roundings of a growing sum), 1.6e-7 in two
    (False, False, 1000, 4096, 4096, 3.5e-7),     # 4.1e-7 and 3.0e-7
    (True, False, 1000, 4096, 512, 1.15e-7),      # 1.3e-7 and 0.94e-7, scores 1.4e-7 and 1.1e-7
    (True, True, 1000, 4096, 4096, 2.2e-7),
])
def test_long_and_chosen_sums_are_added_in_two_halves(chosen, positive, J, D, N, most):
    """Error against fp64, of the norm, half way between what one running sum and two have."""
    import paper_1511_08486_amd as sfb
    dev, g = "cuda:0", torch.Generator(device="cuda:0").manual_seed(1)
    draw = lambda *s: (torch.rand if positive else torch.randn)(s, generator=g, device=dev)  # noqa: E731
    U0, V0, A, W = draw(N, J), draw(N, D), draw(N, D), draw(J, D)
    W1, U, V = torch.zeros((J, D), device=dev), torch.empty((N, J), device=dev), torch.empty((N, D), device=dev)
    ctx = sfb.Sfb("dml", J, D, 4, N // 4, device=dev)
    if chosen:
        ctx.set_plan(fwd_dma=13)
    ctx.reconstruct_apply(W1, U0, V0, -1.0, scale=1.0)
    ctx.compute_factors(W, sfb.SfbBatch(a=A, a2=torch.zeros_like(A)), torch.ones(N, dtype=torch.int32, device=dev), U, V)
    ctx.sync()
    ctx.close()
    for got, want in ((W1, U0.double().T @ V0.double()), (0.5 * U, A.double() @ W.double().T)):
        assert (got.double() - want).norm() <= most * want.norm()


@pytest.mark.parametrize("J,D,N", [(1001, 4096, 512), (600, 4096, 1024), (300, 4096, 512), (130, 1536, 252), (70, 192, 160)])
@pytest.mark.parametrize("off", [-3, -2, -1, 0, 1, 2, 3])
def test_tiles_at_the_end_of_rows_and_columns(J, D, N, off):
    """Rows that end within a lane's words, rows of W apart and not: every entry is its own, and nothing beyond W is written."""
    import paper_1511_08486_amd as sfb
    dev, g = "cuda:0", torch.Generator(device="cuda:0").manual_seed(J)
    D, J = D + off, J + (off & 1)
    U, V = torch.randn((N, J), generator=g, device=dev), torch.randn((N, D), generator=g, device=dev)
    ctx = sfb.Sfb("mlr", J, D, 1, N, device=dev)
    for pitch in (D, D + 5):
        whole = torch.full((J + 2, pitch), 7.0, device=dev)
        W = whole[:J, :D]
        ctx.reconstruct_apply(W, U, V, -1.0, scale=1.0)
        ctx.sync()
        assert ctx.last_kernel(2)[0] == "reconstruct_split_kernel"
        got = W.double() - 7.0
        room = 2.0 ** -24 * (6 * N / 16 + 8) * (U.double().abs().T @ V.double().abs()) + 2.0 ** -21
        assert ((got - U.double().T @ V.double()).abs() <= room).all()
        whole[:J, :D] = 7.0
        assert (whole == 7.0).all()
    # scores of as many classes, and their row of Z's last words
    A, y, U, V = torch.randn((200, 640), generator=g, device=dev), torch.ones(200, dtype=torch.int32, device=dev), torch.full((200, J), float("nan"), device=dev), torch.empty((200, 640), device=dev)
    W = torch.randn((J, 640), generator=g, device=dev)
    ctx.close()
    ctx = sfb.Sfb("dml", J, 640, 1, 200, device=dev)
    ctx.compute_factors(W, sfb.SfbBatch(a=A, a2=torch.zeros_like(A)), y, U, V)
    ctx.sync()
    ctx.close()
    _assert_rows_and_columns(0.5 * U.double(), A.double(), W.double())


@pytest.mark.parametrize("J,D,N", [(1000, 4096, 512), (3326, 376, 532)])
@pytest.mark.parametrize("deviation", [0.1, 3.0, 6.0])
def test_softmax_factors(J, D, N, deviation):
    """Factors of models that are new, half way and done: ones at the labels, which most blocks of many classes meet late, and probabilities
    down to e^-60 elsewhere."""
    import paper_1511_08486_amd as sfb
    dev, g = "cuda:0", torch.Generator(device="cuda:0").manual_seed(J)
    p = torch.softmax(deviation * torch.randn((N, J), generator=g, device=dev), 1)
    U = p.scatter_add(1, torch.multinomial(p, 1, generator=g), torch.full((N, 1), -1.0, device=dev))
    V, W = torch.randn((N, D), generator=g, device=dev) / D ** 0.5, torch.zeros((J, D), device=dev)
    ctx = sfb.Sfb("mlr", J, D, 4, N // 4, device=dev)
    ctx.reconstruct_apply(W, U, V, -1.0, scale=1.0)
    ctx.sync()
    ctx.close()
    _assert_rows_and_columns(W.double(), U.double().T, V.double().T)


# 1 + 2^-12 + 2^-23 has 24 bits: exact in three terms, one bit short in two
_ODD = 1.0 + 2.0 ** -12 + 2.0 ** -23


@pytest.mark.parametrize("J,D,N,blocks", [                      # update tiles and workgroups
    (1000, 4096, 512, 8 * 32),                                  # 128 x 128
    (517, 3618, 482, 6 * 29),                                   # 96 x 128
    (213, 4520, 392, 4 * 36),                                   # 64 x 128
    (1000, 1000, 1400, 256),                                    # 64 x 64, eight splitting wavefronts
    (2908, 647, 291, 46 * 11),                                  # 64 x 64, four
    (907, 755, 3800, None),                                     # with slices of the pairs
    (2775, 135, 1130, None),
    (1101, 76, 5676, None),
    (909, 665, 1224, None),
])
@pytest.mark.parametrize("masked", [False, True])
def test_update_tiles_in_two_terms(J, D, N, blocks, masked):
    """The split that ran, by a value that tells them apart; columns of every magnitude; pairs that end two terms half way, and an infinity
    in the last of them."""
    import paper_1511_08486_amd as sfb
    dev, g = "cuda:0", torch.Generator(device="cuda:0").manual_seed(J)
    P = next(p for p in range(2, 65) if N % p == 0) if masked else 1
    active = [p != 0 for p in range(P)] if masked else None
    live = torch.ones(N, dtype=torch.bool, device=dev)
    ctx, W = sfb.Sfb("mlr", J, D, P, N // P, device=dev), torch.zeros((J, D), device=dev)
    if masked:
        live[:N // P] = False

    def update(U, V):
        ctx.reconstruct_apply(W.zero_(), U, V, -1.0, scale=1.0, active=active)
        ctx.sync()
        assert ctx.last_kernel(2)[0] == "reconstruct_split_kernel" and (blocks is None or ctx.last_kernel(2)[1] == blocks)
        return W.double()

    U, V = torch.zeros((N, J), device=dev), torch.zeros((N, D), device=dev)
    U[N - 1], V[N - 1] = _ODD, 1.0
    got = update(U, V)
    assert ((got - _ODD).abs() <= 2.0 ** -22).all() and (got != _ODD).all()
    U, V = torch.randn((N, J), generator=g, device=dev), torch.randn((N, D), generator=g, device=dev)
    U = _spread("rows in between", U.T.contiguous()).T.contiguous()
    if masked:
        U[~live] = float("nan")
        V[~live] = float("inf")
    _assert_rows_and_columns(update(U, V), U[live].double().T, V[live].double().T)
    V[N // 2:] *= 1e7
    _assert_rows_and_columns(update(U, V), U[live].double().T, V[live].double().T)
    V[N - 1, D - 1] = float("inf")
    got = update(U, V)
    assert torch.equal(got[:, D - 1], torch.sign(U[N - 1].double()) * float("inf"))
    _assert_rows_and_columns(got[:, :D - 1], U[live].double().T, V[live, :D - 1].double().T)
    ctx.close()


@pytest.mark.parametrize("J,D,N,blocks", [                      # score tiles and workgroups
    (2698, 588, 713, 6 * 22),                                   # 128 x 128
    (649, 651, 2779, 22 * 11),                                  # 128 x 64
    (2783, 694, 642, 11 * 22),                                  # 64 x 128
    (75, 2046, 3328, 52 * 2 * 2),                               # 64 x 64, with slices of the columns
    (1000, 4096, 512, 4 * 8 * 8),
])
def test_score_tiles_in_two_terms(J, D, N, blocks):
    import paper_1511_08486_amd as sfb
    dev, g = "cuda:0", torch.Generator(device="cuda:0").manual_seed(J)
    ctx, y = sfb.Sfb("dml", J, D, 1, N, device=dev), torch.ones(N, dtype=torch.int32, device=dev)   # similar pairs: u = 2 z
    U, V = torch.empty((N, J), device=dev), torch.empty((N, D), device=dev)

    def scores(A, W, shift=0.0):
        ctx.compute_factors(W, sfb.SfbBatch(a=A + shift, a2=torch.full_like(A, shift)), y, U, V)
        ctx.sync()
        assert ctx.last_kernel(0)[0] == "scores_split_kernel" and (blocks is None or ctx.last_kernel(0)[1] == blocks)
        return 0.5 * U.double()

    A, W = torch.zeros((N, D), device=dev), torch.zeros((J, D), device=dev)
    A[:, 0], W[:, 0] = _ODD, 1.0
    got = scores(A, W)
    assert ((got - _ODD).abs() <= 2.0 ** -22).all() and (got != _ODD).all()
    A, W = torch.randn((N, D), generator=g, device=dev), torch.randn((J, D), generator=g, device=dev)
    got = scores(A, W, 0.25)
    _assert_rows_and_columns(got, V.double(), W.double())       # (of the differences as they are)
    A = _spread("rows in between", A)
    _assert_rows_and_columns(scores(A, W), A.double(), W.double())
    W[:, D // 2:] *= 1e7
    _assert_rows_and_columns(scores(A, W), A.double(), W.double())
    ctx.close()

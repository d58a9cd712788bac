"""The fp32 contractions on bf16 matrix instructions (three bf16 terms per value): edges of their tiles, blocks of k that do
not divide over the wavefronts, the k-split, values over a wide range, infinities and NaN.

Tolerance: the six products that are taken leave out at most (1 + 2^-9) 2^-24 of a product (values rounded to bf16 leave 2^-9
of them, the second term rounded 2^-17: twice 2^-8 2^-17), and an fp32 sum of k products, in any order, is within k 2^-24 times
the sum of the products' absolute values of the exact one (first order).
"""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu
EPS = 2.0 ** -24


@pytest.fixture(scope="module")
def ctx():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_1409_5705_amd as m
    c = m.Context(0)
    yield c
    c.close()


def normal(seed, *shape):
    return torch.randn(shape, generator=torch.Generator(device="cuda:0").manual_seed(seed), device="cuda:0")


# test_kernel_plans.py asserts that these reach both tile shapes, whole and with a k-split
APPLY_SHAPES = [
    (1619, 4136, 35), (2766, 377, 185),                                # fewer blocks of k than wavefronts; one each
    (785, 4669, 164), (449, 2195, 193), (1003, 2047, 200),             # 128 x 64, one or two blocks of k a wavefront
    (1000, 2048, 801), (641, 2050, 1024),
    (364, 1707, 1148), (262, 899, 1921), (256, 3056, 2848),            # with a k-split
    (642, 2976, 225), (1024, 4096, 512), (2177, 1169, 353),            # 128 x 128
    (1025, 2113, 799),
    (131, 4367, 2491),
]


@pytest.mark.parametrize("J,D,N", APPLY_SHAPES)
def test_apply(ctx, J, D, N):
    print("apply", J, D, N, flush=True)
    U, V, W = normal(1, N, J), normal(2, N, D), 0.1 * normal(3, J, D)
    ref = W.double() - 0.25 * (U.double().t() @ V.double())
    size = 0.25 * (U.abs().double().t() @ V.abs().double())
    ctx.sfb_apply(W, U, V, 0.25)
    assert bool(torch.all((W.double() - ref).abs() <= (N + 4) * EPS * size + 2 * EPS * ref.abs() + 1e-30))


def rms(t):
    return float(t.square().mean().sqrt())


@pytest.mark.parametrize("n", [1, 2, 3, 4])
def test_few_products(ctx, n):
    """Sums with one to four products that are not zero (sparse factors, few active pairs), their positions drawn: no less exact
    than the same products and their sum in fp32.  Of one product at most (1 + 2^-9) 2^-24 is left out and what is taken is
    rounded once, to 2^-24 of it; the sums of the smaller terms, at most 2^-6 of it, five times before that: 2.08 2^-24 in all."""
    J, D, N = 1003, 2047, 300
    place = torch.Generator().manual_seed(20 + n)
    ours, theirs = [], []
    for rep in range(12):
        U, V, W = torch.zeros(N, J, device="cuda:0"), normal(21 + rep, N, D), torch.zeros(J, D, device="cuda:0")
        at = torch.randperm(N, generator=place)[:n].to("cuda:0")
        U[at] = normal(40 + rep, n, J)
        ctx.sfb_apply(W, U, V, -1.0)
        u, v = U[at].double(), V[at].double()
        ref, size = u.t() @ v, u.abs().t() @ v.abs()
        total = torch.zeros(J, D, device="cuda:0")
        for k in range(n):
            total = total + U[at[k]][:, None] * V[at[k]][None, :]
        ours.append(rms((W.double() - ref) / size))
        theirs.append(rms((total.double() - ref) / size))
        if n == 1:
            assert float(((W.double() - ref).abs() / size).max()) <= 2.08 * EPS
    assert sum(ours) <= 1.05 * sum(theirs), (sum(ours) / 12 / EPS, sum(theirs) / 12 / EPS)


@pytest.mark.parametrize("u,v", [(1, 1), (-116, 0), (-125, 0), (-120, 100), (-132, 100), (-140, 100), (100, -140), (62, 55), (110, -120)])
def test_scales(ctx, u, v):
    """Factors of 2^u and 2^v: as exact as those around 1, also below 2^-110 and where they are denormal (2-norm: 7e-8 measured,
    a value rounded to the 2^-149 of the denormals is known to 2^-10 at 2^-140, in the reference too)."""
    J, D, N = 1003, 2047, 300
    U, V = normal(60, N, J) * 2.0 ** (u / 2) * 2.0 ** (u / 2), normal(61, N, D) * 2.0 ** (v / 2) * 2.0 ** (v / 2)
    W = torch.zeros(J, D, device="cuda:0")
    ctx.sfb_apply(W, U, V, -1.0)
    ref = U.double().t() @ V.double()
    assert float((W.double() - ref).norm() / ref.norm()) <= 4e-7
    # and by way of LDS
    import paper_1409_5705_amd as sfb
    J, D, B = 1028, 4004, 517
    W, X = normal(62, J, D) * 2.0 ** (u / 2) * 2.0 ** (u / 2), normal(63, B, D) * 2.0 ** (v / 2) * 2.0 ** (v / 2)
    P, V = torch.empty(B, J, device="cuda:0"), torch.empty(B, D, device="cuda:0")
    ctx.sfb_compute_sf(sfb.SFB_DML, W, X, Y=torch.zeros_like(X), sim=torch.ones(B, dtype=torch.int8, device="cuda:0"), U=P, V=V)
    ref = 2.0 * (X.double() @ W.double().t())
    assert float((P.double() - ref).norm() / ref.norm()) <= 4e-7


def test_wide_range(ctx):
    """Values over 40 orders of magnitude: every product is as exact as fp32 ones, whatever its neighbours."""
    J, D, N = 1003, 2047, 300
    U, V = normal(4, N, J) * torch.exp(12 * normal(5, N, J)), normal(6, N, D) * torch.exp(5 * normal(7, N, D))
    W = torch.zeros(J, D, device="cuda:0")
    ref = -(U.double().t() @ V.double())
    size = U.abs().double().t() @ V.abs().double()
    ctx.sfb_apply(W, U, V, 1.0)
    assert bool(torch.all((W.double() - ref).abs() <= (N + 4) * EPS * size + 2 * EPS * ref.abs()))


def test_not_finite(ctx):
    """Infinities, NaN and the largest values come out as from fp32 products."""
    J, D, N = 1003, 2047, 300
    U, V = normal(8, N, J), normal(9, N, D)
    U[7, 5], U[8, 9], U[299, 999] = float("inf"), float("-inf"), float("nan")
    V[:, 77] = 0.0                                    # inf times 0
    U[:, 500], V[:, 99] = 0.0, 0.0
    U[3, 500], V[3, 99] = torch.finfo(torch.float32).min, 1.0
    W = torch.zeros(J, D, device="cuda:0")
    ref = -(U.double().t() @ V.double())
    ctx.sfb_apply(W, U, V, 1.0)
    for test in (torch.isnan, torch.isposinf, torch.isneginf):
        assert bool(torch.all(test(W[[5, 9, 999]]) == test(ref[[5, 9, 999]]))), test
    rest = torch.ones(J, dtype=torch.bool, device="cuda:0")
    rest[[5, 9, 999, 500]] = False
    assert bool(torch.all(torch.isfinite(W[rest])))
    assert W[500, 99].item() == float(np.finfo(np.float32).max)


# two factors, and whether their product is infinite in fp32: just above the largest value with leading bf16 terms that stay
# below it, the largest value itself, and below
OVERFLOWS = [
    (3.4028234663852886e38, 1.0078124, True), (3e38, 1.137, True), (2e38, 1.7109, True),
    ((1 + 2.0 ** -7 - 2.0 ** -23) * 2.0 ** 64, 1.9921875 * 2.0 ** 63, True),
    (3.4028234663852886e38, 1.0, False), (1e38, 3.4, False), (1.9999 * 2.0 ** 70, 1.00004 * 2.0 ** 57, False),
]
# whole and with a k-split, both tile shapes (test_kernel_plans.py), a partial block of k
NOT_FINITE_APPLY = [(512, 4096, 1024), (364, 1707, 1148), (1025, 2113, 799), (131, 4367, 2491)]
NOT_FINITE_LOGITS = [(512, 4096, 1024), (517, 1028, 4004), (177, 2732, 4148), (770, 2548, 716)]
NANS = [0x7f800001, -0x7fffff, 0x7fc00000, 0x7f80ffff]      # (payloads in the low 16 bits only; -0x7fffff: 0xff800001)


def from_bits(bits):
    return torch.tensor([bits], dtype=torch.int32, device="cuda:0").view(torch.float32)[0]


def extremes(K, M, N):
    """a [K][M], b [K][N] whose contraction has one or two products at the elements that the tests look at."""
    a, b = torch.zeros(K, M, device="cuda:0"), torch.zeros(K, N, device="cuda:0")
    for i, (x, y, _) in enumerate(OVERFLOWS):
        a[101 * i + 3, i], b[101 * i + 3, i] = x, y
        a[101 * i + 4, 64 + i], b[101 * i + 4, 64 + i] = -x, y
    for i, bits in enumerate(NANS):
        a[7 * i, 32 + i], b[7 * i, 32 + i] = from_bits(bits), 1.0
        a[7 * i + 1, 40 + i], b[7 * i + 1, 40 + i] = 1.0, from_bits(bits)
    a[500:502, 50], b[500:502, 50] = 2.0 ** 126 * 1.0039, 2.0             # a sum above the largest value, of products below it
    return a, b


@pytest.mark.parametrize("M,N,K", NOT_FINITE_APPLY)
def test_overflow_and_nan_strided(ctx, M, N, K):
    a, b = extremes(K, M, N)
    C = torch.zeros(M, N, device="cuda:0")
    ctx.sfb_apply(C, a, b, -1.0)
    for i, (x, y, overflow) in enumerate(OVERFLOWS):
        for at, sign in ((i, 1.0), (64 + i, -1.0)):
            got, exact = C[at, at].item(), sign * float(np.float32(x)) * float(np.float32(y))
            assert got == sign * float("inf") if overflow else abs(got - exact) <= 5 * EPS * abs(exact), (i, got, exact)
    for i in range(len(NANS)):
        assert torch.isnan(C[32 + i, 32 + i]) and torch.isnan(C[40 + i, 40 + i]), (i, C[32 + i, 32 + i].item(), C[40 + i, 40 + i].item())
    assert torch.isposinf(C[50, 50])


@pytest.mark.parametrize("B,J,D", NOT_FINITE_LOGITS)
def test_overflow_and_nan_contiguous(ctx, B, J, D):
    """Logits: the softmax of a row with an infinite one or NaN is NaN, with a finite one, however large, it is not."""
    import paper_1409_5705_amd as sfb
    a, b = extremes(D, B, J)
    b[:, 40:40 + len(NANS)] = 0.0                       # (NaN in every row otherwise)
    X, W = a.t().contiguous(), b.t().contiguous()
    U = torch.empty(B, J, device="cuda:0")
    ctx.sfb_compute_sf(sfb.SFB_MLR, W, X, Y=torch.zeros(B, dtype=torch.int32, device="cuda:0"), U=U)
    nan = torch.isnan(U).any(dim=1)
    want = torch.zeros(B, dtype=torch.bool)
    for i, (_, _, overflow) in enumerate(OVERFLOWS):
        want[i] = overflow
    want[32:32 + len(NANS)], want[50] = True, True
    assert torch.equal(nan.cpu(), want), (nan.cpu() != want).nonzero()


def test_not_finite_residual(ctx):
    """The shrink step of samples with infinities and NaN and the residual X - U W (k-contiguous x k-strided) of their codes."""
    import paper_1409_5705_amd as sfb
    J, D, B = 1024, 4096, 512
    W = torch.zeros(J, D, device="cuda:0")
    W[torch.arange(J), torch.arange(J)] = 1.0                # L is 1
    X = torch.zeros(B, D, device="cuda:0")
    X[3, 5], X[4, 6], X[5, 7], X[6, 8] = float("inf"), float("nan"), 3e38, from_bits(0x7f800001)
    U, V = torch.empty(B, J, device="cuda:0"), torch.empty(B, D, device="cuda:0")
    ctx.sfb_compute_sf(sfb.SFB_SC, W, X, U=U, V=V, lam=0.0, ista_iters=1, power_iters=10)
    t = X.double() @ W.double().t()
    codes = torch.where(t > 0, t, torch.where(t < 0, t, torch.zeros_like(t)))       # (NaN: no code)
    for got, want in ((U, codes), (V, X.double() - codes @ W.double())):
        for test in (torch.isnan, torch.isposinf, torch.isneginf):
            assert torch.equal(test(got), test(want)), (test, (test(got) != test(want)).nonzero()[:4])
    assert abs(U[5, 7].item() / 3e38 - 1) <= 1e-5 and float(V[5].abs().max()) <= 1e-5 * 3e38


def test_rows_of_a_larger_matrix_and_alignment(ctx):
    """Factors whose first row starts 4 bytes off 16 (leading dimensions of no particular size)."""
    J, D, N = 1001, 2049, 333
    u, v = normal(10, N * J + 4), normal(11, N * D + 4)
    U, V = u[4:].view(N, J), v[4:].view(N, D)
    W = normal(12, J, D)
    ref = W.double() - 0.5 * (U.double().t() @ V.double())
    size = 0.5 * (U.abs().double().t() @ V.abs().double())
    ctx.sfb_apply(W, U, V, 0.5)
    assert bool(torch.all((W.double() - ref).abs() <= (N + 4) * EPS * size + 2 * EPS * ref.abs() + 1e-30))


# (J, D, B): logits of B samples, projections and shrink steps are J columns over D of k, residuals D columns over J;
# test_kernel_plans.py asserts that each of these epilogues reaches both tile shapes, whole and with a k-split
LOGITS_SHAPES = [(3476, 236, 295), (4096, 1024, 512), (1028, 4004, 517), (2548, 304, 770), (2732, 4148, 177)]
SC_SHAPES = [(4096, 1024, 512), (2196, 2140, 98), (244, 3620, 275), (292, 2752, 714), (4120, 1824, 264), (3476, 236, 295),
             (948, 1828, 648), (644, 44, 2956)]


@pytest.mark.parametrize("J,D,B", LOGITS_SHAPES)
def test_projection(ctx, J, D, B):
    """U = 2 (X - Y) W^T of similar pairs: two k-contiguous operands, stored as they come."""
    import paper_1409_5705_amd as sfb
    print("projection", J, D, B, flush=True)
    W, X = 0.1 * normal(13, J, D), normal(14, B, D)
    U, V = torch.empty(B, J, device="cuda:0"), torch.empty(B, D, device="cuda:0")
    ctx.sfb_compute_sf(sfb.SFB_DML, W, X, Y=torch.zeros_like(X), sim=torch.ones(B, dtype=torch.int8, device="cuda:0"), U=U, V=V)
    ref = 2.0 * (X.double() @ W.double().t())
    size = 2.0 * (X.abs().double() @ W.abs().double().t())
    assert bool(torch.all((U.double() - ref).abs() <= (D + 2) * EPS * size + 1e-30))


@pytest.mark.parametrize("J,D,B", SC_SHAPES)
def test_sparse_codes(ctx, J, D, B):
    """The residual (k-contiguous x k-strided) and shrink epilogues: three ISTA iterations against 64-bit torch."""
    import paper_1409_5705_amd as sfb
    print("sparse codes", J, D, B, flush=True)
    W, X = normal(15, J, D), normal(16, B, D)
    W /= W.norm(dim=1, keepdim=True)
    U, V = torch.empty(B, J, device="cuda:0"), torch.empty(B, D, device="cuda:0")
    lam, iters = 0.1, 3
    ctx.sfb_compute_sf(sfb.SFB_SC, W, X, U=U, V=V, lam=lam, ista_iters=iters, power_iters=10)
    W64, X64 = W.double(), X.double()
    b = torch.full((D,), D ** -0.5, dtype=torch.float64, device="cuda:0")
    for _ in range(10):
        b = W64.t() @ (W64 @ (b / b.norm()))
    L = b.norm()
    a, r = torch.zeros((B, J), dtype=torch.float64, device="cuda:0"), X64
    for _ in range(iters):
        t = a + r @ W64.t() / L
        a = torch.sign(t) * torch.clamp(t.abs() - lam / L, min=0.0)
        r = X64 - a @ W64
    for got, want in ((U, a), (V, r)):
        err = (got.double() - want).abs() / (want.abs() + want.square().mean().sqrt())
        assert float(err.max()) <= 1e-4


# One product per sum, at every k in turn, of factors with 24 significant bits: each of the six bf16 products that are taken is
# worth 2^-18 of it or more, so one that is lost, or a value of k that is, shows (test_few_products: the bound).
ONE = 2.08 * EPS


def one_per_row(seed, rows, columns, count):
    """[rows][columns] with N(0,1) at `count` places, no two of them in one row or column; and these."""
    g = torch.Generator().manual_seed(seed)
    r, c = torch.randperm(rows, generator=g)[:count].to("cuda:0"), torch.randperm(columns, generator=g)[:count].to("cuda:0")
    m = torch.zeros(rows, columns, device="cuda:0")
    m[r, c] = normal(seed, count)
    return m, r, c


@pytest.mark.parametrize("J,D,N", APPLY_SHAPES)
@pytest.mark.parametrize("single", ["U", "V"])
def test_apply_of_single_products(ctx, J, D, N, single):
    print("apply, single", J, D, N, single, flush=True)
    n = J if single == "U" else D
    k = (torch.arange(n, device="cuda:0") * 7 + torch.arange(n, device="cuda:0") // N) % N
    U, V, W = normal(70, N, J), normal(71, N, D), torch.zeros(J, D, device="cuda:0")
    if single == "U":
        u, v = U[k, torch.arange(J)], V[k]
        U = torch.zeros_like(U)
        U[k, torch.arange(J)] = u
        ref = u.double()[:, None] * v.double()
    else:
        u, v = U[k], V[k, torch.arange(D)]
        V = torch.zeros_like(V)
        V[k, torch.arange(D)] = v
        ref = (u.double() * v.double()[:, None]).t()
    ctx.sfb_apply(W, U, V, -1.0)
    assert bool(torch.all((W.double() - ref).abs() <= ONE * ref.abs()))


@pytest.mark.parametrize("J,D,B", LOGITS_SHAPES)
@pytest.mark.parametrize("single", ["W", "X"])
def test_projection_of_single_products(ctx, J, D, B, single):
    import paper_1409_5705_amd as sfb
    print("projection, single", J, D, B, single, flush=True)
    n = J if single == "W" else B
    k = (torch.arange(n, device="cuda:0") * 7 + torch.arange(n, device="cuda:0") // D) % D
    W, X = normal(72, J, D), normal(73, B, D)
    full = W if single == "W" else X
    kept = full[torch.arange(n), k]
    full.zero_()
    full[torch.arange(n), k] = kept
    ref = 2.0 * (X[:, k].double() * kept.double() if single == "W" else kept.double()[:, None] * W[:, k].t().double())
    U, V = torch.empty(B, J, device="cuda:0"), torch.empty(B, D, device="cuda:0")
    ctx.sfb_compute_sf(sfb.SFB_DML, W, X, Y=torch.zeros_like(X), sim=torch.ones(B, dtype=torch.int8, device="cuda:0"), U=U, V=V)
    assert bool(torch.all((U.double() - ref).abs() <= ONE * ref.abs()))


@pytest.mark.parametrize("J,D,B", SC_SHAPES)
def test_sparse_codes_of_single_products(ctx, J, D, B):
    """A dictionary with one value per row and column, no shrinkage: a code is the sample's value there times the dictionary's
    and 1 / L, which is the same for all codes, and the residual one product taken off the sample."""
    import paper_1409_5705_amd as sfb
    print("sparse codes, single", J, D, B, flush=True)
    W, row, col = one_per_row(74, J, D, min(J, D))
    X = normal(75, B, D)
    U, V = torch.empty(B, J, device="cuda:0"), torch.empty(B, D, device="cuda:0")
    ctx.sfb_compute_sf(sfb.SFB_SC, W, X, U=U, V=V, lam=0.0, ista_iters=1, power_iters=10)
    w = W[row, col].double()
    step = X[:, col].double() * w
    big = step.abs() > 1e-3
    ref = step * (U[:, row].double()[big] / step[big]).mean()                  # (1 / L, to much less than 2^-24)
    assert bool(torch.all((U[:, row].double() - ref).abs() <= (ONE + EPS) * ref.abs()))
    assert int((U != 0).sum()) == int((U[:, row] != 0).sum())
    taken = U[:, row].double() * w
    ref = X[:, col].double() - taken
    assert bool(torch.all((V[:, col].double() - ref).abs() <= ONE * taken.abs() + EPS * ref.abs()))
    rest = torch.ones(D, dtype=torch.bool, device="cuda:0")
    rest[col] = False
    assert torch.equal(V[:, rest], X[:, rest])


# few pairs: the 128 x 64 tiles of the fp32 kernel keep these (test_kernel_plans.py)
FP32_SHAPES = [(1104, 1580, 31), (1107, 1583, 30)]


@pytest.mark.parametrize("J,D,N", FP32_SHAPES)
def test_apply_few_pairs(ctx, J, D, N):
    test_apply(ctx, J, D, N)

"""The fp32 contractions on bf16 matrix instructions (three bf16 terms per value): edges of their tiles, blocks of k that do
not divide over the wavefronts, the k-split, values over a wide range, infinities and NaN.

Tolerance: the six products that are taken leave out less than 2^-24 of a product, and an fp32 sum of k products, in any
order, is within k 2^-24 times the sum of the products' absolute values of the exact one (first order).
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


# (J, D, B): logits of B samples and projections are J columns over D of k, residuals D columns over J; test_kernel_plans.py
# asserts that these reach both tile shapes, whole and with a k-split
LOGITS_SHAPES = [(3476, 236, 295), (4096, 1024, 512), (1028, 4004, 517), (2548, 304, 770), (2732, 4148, 177)]
SC_SHAPES = [(4096, 1024, 512), (2196, 2140, 98), (244, 3620, 275), (292, 2752, 714), (4120, 1824, 264), (3476, 236, 295)]


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


# few pairs: the 128 x 64 tiles of the fp32 kernel keep these (test_kernel_plans.py)
FP32_SHAPES = [(1104, 1580, 31), (1107, 1583, 30)]


@pytest.mark.parametrize("J,D,N", FP32_SHAPES)
def test_apply_few_pairs(ctx, J, D, N):
    test_apply(ctx, J, D, N)

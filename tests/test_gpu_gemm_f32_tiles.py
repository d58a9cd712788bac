"""The fp32 contractions at the edges of their tiles: sizes that the cost model gives to each tile shape, with the 16-byte
and the unaligned load path, partial k-slices, fewer rows than a 16-byte load holds, and the k-split over workgroups.

Tolerance: an fp32 sum of k products, in any order, is within k 2^-24 times the sum of the products' absolute values of
the exact one (first order); the update adds one rounding of the product with eta and one of the result.
"""
import numpy as np
import pytest

import sfb_synth as S
from parity import TOL_F32, rel_err

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu
EPS = 2.0 ** -24


@pytest.fixture(scope="module")
def sfb():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_1409_5705_amd as m
    m.lib()
    return m


@pytest.fixture(scope="module")
def ctx(sfb):
    c = sfb.Context(0)
    yield c
    c.close()


def dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).to("cuda:0")


def host(t):
    torch.cuda.synchronize()
    return t.cpu().numpy()


APPLY_SHAPES = [
    (2048, 4096, 96), (2001, 4001, 130),       # 128 x 128 tiles
    (1000, 2048, 300), (1003, 2047, 200),      # 128 x 64
    (700, 800, 300), (701, 803, 300),          # 64 x 64
    (600, 800, 200), (401, 603, 77),           # 32 x 32
    (500, 1000, 260), (501, 603, 100),         # 64 x 32
    (8324, 208, 8), (155, 8287, 4), (174, 5383, 140),      # the large tiles where the three bf16 terms do not take over (few pairs, narrow)
    (400, 600, 200), (16, 10000, 30), (30, 9001, 100), (9000, 20, 64), (64, 4100, 33),   # few slices, several workgroups a CU
    (33, 70, 96), (16, 16, 128), (17, 48, 1),  # 16 x 16
    (3, 2052, 65), (2052, 3, 200), (2, 37, 130), (1, 1, 5), (4, 6, 32),   # rows of fewer floats than a load takes
]


@pytest.mark.parametrize("J,D,N", APPLY_SHAPES)
def test_apply_tiles(ctx, oracle, J, D, N):
    print("apply", J, D, N, flush=True)
    g = np.random.default_rng([21, J, D, N])
    U = g.standard_normal((N, J), dtype=np.float32)
    V = g.standard_normal((N, D), dtype=np.float32)
    W0 = S.normal_matrix(J, D, 0.1, seed=21)
    W = dev(W0)
    ctx.sfb_apply(W, dev(U), dev(V), 0.25)
    ref = oracle.apply(W0, U, V, 0.25)
    size = 0.25 * (np.abs(U).T.astype(np.float64) @ np.abs(V).astype(np.float64))
    assert np.all(np.abs(host(W) - ref) <= (N + 4) * EPS * size + 2 * EPS * np.abs(ref) + 1e-30)


@pytest.mark.parametrize("J,D,B", [
    (512, 4096, 130), (515, 4097, 131),        # 32 x 32 tiles with a k-split; the partial slice in the last split
    (1000, 2048, 256), (1003, 2047, 100),      # 32 x 32; 64 x 32 with a k-split, unaligned
    (96, 8000, 130), (64, 128, 32), (1, 1, 1), (37, 50, 7), (18, 129, 15),   # 16 x 16
    (2100, 100, 1000), (4099, 67, 600),        # large tiles, short k
])
def test_projection_tiles(ctx, sfb, J, D, B):
    """U = 2 V W^T of similar pairs: the contraction of two k-contiguous operands as it is."""
    print("projection", J, D, B, flush=True)
    g = np.random.default_rng([22, J, D, B])
    W0 = S.normal_matrix(J, D, 0.1, seed=22)
    X, Y = g.standard_normal((B, D), dtype=np.float32), np.zeros((B, D), dtype=np.float32)
    U = torch.empty((B, J), dtype=torch.float32, device="cuda:0")
    V = torch.empty((B, D), dtype=torch.float32, device="cuda:0")
    ctx.sfb_compute_sf(sfb.SFB_DML, dev(W0), dev(X), Y=dev(Y), sim=dev(np.ones(B, dtype=np.int8)), U=U, V=V)
    ref = 2.0 * (X.astype(np.float64) @ W0.T.astype(np.float64))
    size = 2.0 * (np.abs(X).astype(np.float64) @ np.abs(W0).T.astype(np.float64))
    assert np.all(np.abs(host(U) - ref) <= (D + 2) * EPS * size + 1e-30)


@pytest.mark.parametrize("J,D,B", [(1000, 300, 100), (1001, 301, 99), (517, 1023, 70), (64, 4, 3), (130, 1030, 300)])
def test_sparse_code_tiles(ctx, sfb, oracle, J, D, B):
    """The residual (k-contiguous x k-strided) and shrink epilogues."""
    print("sparse codes", J, D, B, flush=True)
    W0, X = S.sc_dictionary(J, D, seed=23), S.sc_batch(D, B, seed=23)
    U = torch.empty((B, J), dtype=torch.float32, device="cuda:0")
    V = torch.empty((B, D), dtype=torch.float32, device="cuda:0")
    ctx.sfb_compute_sf(sfb.SFB_SC, dev(W0), dev(X), U=U, V=V, lam=0.1, ista_iters=3, power_iters=10)
    Uo, Vo, _ = oracle.sc_sf(W0, X, lam=0.1, ista_iters=3, power_iters=10)
    assert rel_err(host(U), Uo) <= TOL_F32
    assert rel_err(host(V), Vo) <= TOL_F32


# test_kernel_plans.py asserts that these reach every tile shape, with direct loads and through registers
SC_SHAPES = [
    (100, 112, 16), (106, 105, 16),             # both contractions on 16 x 16 tiles
    (132, 664, 452), (648, 116, 536),           # 32 x 32 and 64 x 32
    (135, 134, 914), (273, 274, 942),           # both 32 x 32; both 64 x 32
    (1416, 1471, 36), (2128, 2196, 17),         # both 64 x 32, both 32 x 32, with a k-split
    (2184, 204, 395), (324, 2144, 233),         # 64 x 64 shrink; residual
    (4212, 133, 100), (139, 4143, 98),
    (3296, 136, 259), (136, 4280, 197),         # 128 x 64
    (4164, 103, 195), (161, 2531, 678),
    (4408, 164, 705), (132, 3780, 515),         # 128 x 128
    (2058, 101, 963), (103, 3662, 533),
    (2204, 2214, 119),                          # both 128 x 64 with a k-split
    (8560, 4, 212), (5004, 4, 276),             # aligned and large, k below 32 (longer ones run on three bf16 terms): 128 x 128
    (4, 8648, 200), (12, 5064, 264), (4, 8416, 130),   # and 128 x 64 shrink; 128 x 128, 128 x 64 and 64 x 64 residual
]


@pytest.mark.parametrize("J,D,B", SC_SHAPES)
def test_sparse_code_and_projection_shapes(ctx, sfb, J, D, B):
    """The shrink, residual and plain-store epilogues against 64-bit torch: two ISTA iterations, and U = 2 X W^T."""
    print("sparse codes, projection", J, D, B, flush=True)
    W0, X0 = S.sc_dictionary(J, D, seed=24), S.sc_batch(D, B, seed=24)
    W, X = dev(W0), dev(X0)
    U = torch.empty((B, J), dtype=torch.float32, device="cuda:0")
    V = torch.empty((B, D), dtype=torch.float32, device="cuda:0")
    lam, iters = 0.1, 2
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
    assert rel_err(host(U), host(a)) <= TOL_F32
    assert rel_err(host(V), host(r)) <= TOL_F32
    ctx.sfb_compute_sf(sfb.SFB_DML, W, X, Y=torch.zeros_like(X), sim=torch.ones(B, dtype=torch.int8, device="cuda:0"), U=U, V=V)
    size = 2.0 * (X64.abs() @ W64.abs().t())
    assert bool(torch.all((U.double() - 2.0 * (X64 @ W64.t())).abs() <= (D + 2) * EPS * size + 1e-30))

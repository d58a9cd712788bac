"""Sums of the k-splits that the row kernels take from the contraction: softmax rows of one to sixteen floats a thread, aligned
and not, and the scaling of the metric's projections; rows at the edges of what a thread holds, and with no split.

Tolerance: a logit is an fp32 sum of D products, within D 2^-24 times the sum of their absolute values of the exact one; the
softmax's exponential turns an error d of two logits into a relative one of at most 2 d, expf and the sum of J exponentials add
(J + 4) 2^-24.
"""
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


# test_kernel_plans.py asserts which of these split k
MLR_SHAPES = [
    (2000, 1, 20000), (2000, 10, 20000), (100, 191, 20000), (600, 256, 4100), (257, 255, 4096),
    (1000, 257, 4100), (600, 1000, 1000), (599, 1001, 2000), (64, 1024, 4000),
    (300, 1025, 2000), (256, 2000, 4000), (256, 4095, 4096), (350, 2048, 2049),
    (100, 1300, 4000), (256, 4097, 2000),                                          # summed by a launch in front
    (100, 191, 64),                                                                # no split
]


@pytest.mark.parametrize("B,J,D", MLR_SHAPES)
def test_mlr(ctx, B, J, D):
    import paper_1409_5705_amd as sfb
    print("mlr", B, J, D, flush=True)
    X, W = normal(1, B, D), normal(2, J, D) / D ** 0.5
    y = torch.randint(0, J, (B,), generator=torch.Generator(device="cuda:0").manual_seed(3), device="cuda:0").to(torch.int32)
    U = torch.full((B, J), 7.0, device="cuda:0")
    ctx.sfb_compute_sf(sfb.SFB_MLR, W, X, Y=y, U=U)
    p = torch.softmax(X.double() @ W.double().t(), dim=1)
    err = 2 * (D * EPS * (X.abs().double() @ W.abs().double().t())).amax(dim=1, keepdim=True) + (J + 4) * EPS
    ref = p.clone()
    ref[torch.arange(B, device="cuda:0"), y.long()] -= 1.0
    assert bool(torch.all((U.double() - ref).abs() <= p * err + 2 * EPS))


DML_SHAPES = [(2000, 1, 20000), (257, 255, 4096), (600, 256, 4100), (100, 601, 5000), (600, 1000, 1024), (70, 1024, 4000),
              (100, 1025, 5000), (100, 300, 64)]


@pytest.mark.parametrize("B,J,D", DML_SHAPES)
def test_dml(ctx, B, J, D):
    import paper_1409_5705_amd as sfb
    print("dml", B, J, D, flush=True)
    X, Y, W = normal(1, B, D), normal(2, B, D), normal(3, J, D) / (J * D) ** 0.5
    sim = (torch.arange(B, device="cuda:0") % 2).to(torch.int8)
    U, V = torch.full((B, J), 7.0, device="cuda:0"), torch.empty(B, D, device="cuda:0")
    n = torch.zeros(1, dtype=torch.int32, device="cuda:0")
    delta = (X - Y).double()
    q = delta @ W.double().t()
    d = (q * q).sum(dim=1)
    margin = float(d[sim == 0].median()) * (1 + 1e-3)            # (between two pairs' distances: at least 1e-3 of them is far from rounding)
    ctx.sfb_compute_sf(sfb.SFB_DML, W, X, Y=Y, sim=sim, U=U, V=V, n_active=n, margin=margin)
    clear = (d - margin).abs() > 1e-4 * margin
    c = torch.where(sim > 0, 2.0, torch.where(d < margin, -2.0, 0.0)).double()[:, None]
    err = 2 * (D + 4) * EPS * (delta.abs() @ W.abs().double().t())
    assert bool(clear.sum() >= B - 2)
    assert bool(torch.all(((U.double() - c * q).abs() <= err + 1e-30)[clear]))
    assert abs(int(n) - int((c != 0).sum())) <= int((~clear).sum())

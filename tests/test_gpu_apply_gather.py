"""sfb_apply_csr over the stored entries: edges of its tiles (64 classes, 128 columns, 32 pairs a step, the largest number of
pairs), every storage of W, densities from nothing to all, signed factors.

Tolerance: bf16 products are exact in fp32, and an fp32 sum of k products, in any order, is within k 2^-24 times the sum of
their absolute values of the exact one (first order); the update adds one rounding of the product with eta and one of the
result.
"""
import ctypes

import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu
EPS = 2.0 ** -24
DEV = "cuda:0"


@pytest.fixture(scope="module")
def sfb():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_1409_5705_amd as m
    m.lib()
    return m


def factors(N, J, D, rho, seed):
    g = torch.Generator(device=DEV).manual_seed(seed)
    U = torch.randn(N, J, generator=g, device=DEV).to(torch.bfloat16)
    V = (torch.randn(N, D, generator=g, device=DEV) * (torch.rand(N, D, generator=g, device=DEV) < rho)).to(torch.bfloat16)
    W = 0.1 * torch.randn(J, D, generator=g, device=DEV)
    at = V.nonzero()
    indptr = torch.zeros(N + 1, dtype=torch.int64, device=DEV)
    indptr[1:] = torch.bincount(at[:, 0], minlength=N).cumsum(0)
    return U, V, W, (indptr, at[:, 1].to(torch.int32), V[at[:, 0], at[:, 1]].contiguous())


def context(sfb, layout, W, route):
    """route of sfb_apply_csr: 0 chosen, 1 dense contraction, 2 over the stored entries"""
    c = sfb.Context(0)
    force = sfb.lib()._ZN3sfb21force_apply_csr_routeEP7sfb_ctxi
    force.restype, force.argtypes = None, [ctypes.c_void_p, ctypes.c_int]
    force(c._h, route)
    if layout == "copy":
        c.sfb_shadow_attach(W)
    elif layout == "planes":
        c.sfb_split_attach(W)
    return c


@pytest.mark.parametrize("layout", ["plain", "copy", "planes"])
@pytest.mark.parametrize("N,J,D,rho,signed", [
    (1, 640, 264, 0.3, False), (33, 72, 24, 0.1, False), (300, 520, 328, 0.01, True), (255, 1096, 1032, 0.004, False),
    (64, 648, 136, 1.0, False), (256, 704, 128, 0.0, False), (1024, 1344, 1160, 0.005, False), (1276, 1488, 264, 0.05, True),
    (1277, 1480, 264, 0.05, False),      # more pairs than it takes: the dense contraction
])
def test_against_64_bits(sfb, N, J, D, rho, signed, layout):
    print("apply_gather", N, J, D, rho, layout, flush=True)
    U, V, W, csr = factors(N, J, D, rho, N + J)
    W0 = W.clone()
    coef = torch.where(torch.arange(N, device=DEV) % 3 == 0, -1.0, 1.0) if signed else None
    c = context(sfb, layout, W, 2)
    ref, size = W0.double(), torch.zeros(J, D, dtype=torch.float64, device=DEV)
    V64 = V.double() * (coef.double()[:, None] if signed else 1.0)
    for eta in (0.01, -0.004):
        c.sfb_apply_csr(W, U, *csr, eta, coef=coef)
        ref = ref - eta * (U.double().t() @ V64)
        size = size + abs(eta) * (U.abs().double().t() @ V64.abs())
    if layout == "planes":
        c.sfb_split_export(W)
    assert bool(torch.all((W.double() - ref).abs() <= (N + 4) * EPS * size + 4 * EPS * (ref.abs() + W0.abs().double())))
    untouched = (V == 0).all(dim=0)
    assert torch.equal(W[:, untouched], W0[:, untouched])
    if layout == "copy":      # the copy is that of the new W: the same logits as from a fresh one
        X, y = V[:8].contiguous(), torch.zeros(min(N, 8), dtype=torch.int32, device=DEV)
        out = []
        for ctx in (c, context(sfb, "copy", W, 1)):
            out.append(torch.empty(X.shape[0], J, dtype=torch.bfloat16, device=DEV))
            ctx.sfb_compute_sf(sfb.SFB_MLR, W, X, Y=y, U=out[-1])
        assert torch.equal(*out)
    c.close()


@pytest.mark.parametrize("N,J,D,rho,gather", [
    (1024, 16384, 2056, 0.005, True), (1024, 16384, 2056, 0.03, False), (200, 16384, 2056, 0.005, False), (1024, 2048, 2056, 0.005, False),
])
def test_picks_its_route(sfb, N, J, D, rho, gather):
    U, V, W, csr = factors(N, J, D, rho, 5)
    W1 = W.clone()
    c = context(sfb, "planes", W, 0)
    c.sfb_profile_enable(True)
    c.sfb_profile_collect()
    c.sfb_apply_csr(W, U, *csr, 0.01)
    ran = c.sfb_profile_collect()
    assert ("apply_gather" in ran) == gather, ran
    c.sfb_split_export(W)
    d = context(sfb, "plain", W1, 1)
    d.sfb_apply_csr(W1, U, *csr, 0.01)
    size = 0.01 * (U.abs().float().t() @ V.abs().float())
    assert bool(torch.all((W - W1).abs() <= 2 * (N + 4) * EPS * size + 4 * EPS * W1.abs()))
    c.close()
    d.close()


@pytest.mark.parametrize("layout", ["plain", "copy", "planes"])
@pytest.mark.parametrize("N,J,D,rho,bad", [
    (1, 72, 24, 0.3, 3), (300, 520, 328, 0.01, 5), (300, 520, 328, 0.01, 4000), (64, 648, 136, 1.0, 9), (256, 704, 136, 0.0, 3),
    (1024, 640, 1160, 0.005, 40), (1276, 520, 264, 0.05, 30), (1274, 520, 264, 0.3, 100),
])
def test_not_finite_factors(sfb, N, J, D, rho, bad, layout):
    """An infinite or NaN factor times the zeros of V is NaN: it reaches every column, as in the dense contraction."""
    print("apply_gather, not finite", N, J, D, rho, bad, layout, flush=True)
    U, V, W, csr = factors(N, J, D, rho, N + J + 1)
    g = torch.Generator().manual_seed(7)
    at, what = torch.randint(N * J, (bad,), generator=g).to(DEV), torch.tensor([float("inf"), -float("inf"), float("nan")], device=DEV)
    U.view(-1)[at] = what[torch.arange(bad, device=DEV) % 3].to(torch.bfloat16)
    out = []
    for route in (1, 2):
        W1 = W.clone()
        c = context(sfb, layout, W1, route)
        c.sfb_apply_csr(W1, U, *csr, 0.01)
        if layout == "copy":      # the copy's rows, by logits of unit samples
            X, y = torch.eye(8, D, device=DEV).to(torch.bfloat16), torch.zeros(8, dtype=torch.int32, device=DEV)
            P = torch.empty(8, J, dtype=torch.bfloat16, device=DEV)
            c.sfb_compute_sf(sfb.SFB_MLR, W1, X, Y=y, U=P)
            out.append(P)
        if layout == "planes":
            c.sfb_split_export(W1)
        out.append(W1)
        c.close()
    ref = W.double() - 0.01 * (U.double().t() @ V.double())
    assert not bool(torch.isfinite(ref).all())
    for got in (out[-1], out[len(out) // 2 - 1]):
        for test in (torch.isnan, torch.isposinf, torch.isneginf):
            assert torch.equal(test(got), test(ref)), (test, (test(got) != test(ref)).nonzero()[:4])
    if layout == "copy":
        assert torch.equal(torch.isnan(out[0]), torch.isnan(out[2]))
    fine = torch.isfinite(ref)
    size = 0.01 * (U.abs().double().t() @ V.abs().double())
    assert bool(torch.all(((out[-1].double() - ref).abs() <= (N + 4) * EPS * size + 4 * EPS * (ref.abs() + W.abs().double()))[fine]))


@pytest.mark.parametrize("route", [0, 1, 2])
@pytest.mark.parametrize("rho,gather", [(0.005, True), (0.05, False)])
def test_the_route_of_the_forward_is_not_the_applys(sfb, rho, gather, route):
    """sfb_set_csr_route is about sfb_mlr_sf_csr: the apply keeps choosing for itself."""
    N, J, D = 1024, 16384, 2056
    U, V, W, csr = factors(N, J, D, rho, 6)
    c = sfb.Context(0)
    c.sfb_split_attach(W)
    c.sfb_set_csr_route(route)
    c.sfb_profile_enable(True)
    c.sfb_profile_collect()
    c.sfb_apply_csr(W, U, *csr, 0.01)
    ran = c.sfb_profile_collect()
    assert ("apply_gather" in ran) == gather, ran
    c.close()

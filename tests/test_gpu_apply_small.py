"""The bf16 apply at the edges of its 128 x 128 tiles and of the rule that picks them: ragged last tiles, one to nine k-slices,
matrices on both sides of every line of the rule, W as fp32, with its bf16 copy and as two planes.

Tolerance: exact products, fp32 sums of N of them (any order: N 2^-24 times the sum of absolute values), the product with
eta and the result rounded once each.  The copy must hold the rounded values bit for bit, the planes the bits of the array.
"""
import numpy as np
import pytest

import sfb_synth as S

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


def dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).to("cuda:0")


def blocked(buf, J, D):
    """The J x D matrix held in blocks of 256 x 64."""
    P = (D + 63) // 64 * 64
    rows = (J + 255) // 256 * 256
    v = buf.view(torch.bfloat16)[:rows * P].view(rows // 256, P // 64, 256, 64)
    return v.permute(0, 2, 1, 3).reshape(rows, P)[:J, :D]


@pytest.mark.parametrize("J,D,N", [
    (8, 8, 1), (128, 128, 64), (136, 120, 65), (120, 136, 128), (264, 248, 129), (1000, 520, 192), (392, 1032, 256),
    (1000, 264, 257), (520, 328, 580),                 # few tiles: any number of pairs
    (2056, 4104, 300), (4104, 4104, 500),              # up to 512 pairs whose V^T fits an L2; just not
    (2048, 4096, 580), (2304, 4096, 580),              # half as many 256 x 256 tiles as CUs; more
])
@pytest.mark.parametrize("eta", [0.5, 1e-4])
def test_apply_small(sfb, J, D, N, eta):
    print("apply small", J, D, N, eta, flush=True)
    g = torch.Generator(device="cuda:0").manual_seed(J + D + N)
    rnd = lambda *s: torch.randn(s, generator=g, device="cuda:0")
    U, V = (rnd(N, J) * 0.1).bfloat16(), rnd(N, D).bfloat16()
    W0 = rnd(J, D) * 0.1
    ctxs = {k: sfb.Context(0) for k in ("plain", "copy", "planes")}
    Ws = {k: W0.clone() for k in ctxs}
    ctxs["copy"].sfb_shadow_attach(Ws["copy"])
    ctxs["planes"].sfb_split_attach(Ws["planes"])
    for k, c in ctxs.items():
        c.sfb_apply(Ws[k], U, V, eta)
    ctxs["planes"].sfb_split_export(Ws["planes"])
    W = Ws["plain"]
    ref = W0.double() - eta * (U.double().T @ V.double())
    size = U.double().abs().T @ V.double().abs()
    bound = eta * (N + 2) * EPS * size + 2 * EPS * (W0.double().abs() + ref.abs())
    assert bool(((W.double() - ref).abs() <= bound).all())
    assert torch.equal(Ws["copy"], W) and torch.equal(Ws["planes"], W)
    assert torch.equal(blocked(ctxs["copy"]._shadow[1], J, D), W.bfloat16())
    for c in ctxs.values():
        c.close()

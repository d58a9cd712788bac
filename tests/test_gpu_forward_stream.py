"""The bf16 logits by the streaming kernel (few 256 x 256 tiles): every tile shape of it, W as fp32 and from its bf16 copy, partial
k-slices, ragged samples and classes, and the k-split whose partial sums the softmax adds up."""
import numpy as np
import pytest

import sfb_synth as S
from parity import TOL_BF16, mlr_u_check

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def sfb():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_1409_5705_amd as m
    m.lib()
    return m


def dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).to("cuda:0")


def dev_bf16(a):
    return dev(S.bf16_bits(a)).view(torch.bfloat16)


# test_kernel_plans.py asserts that these reach every instantiation, with and without the k-split
SHAPES = [
    (8, 8, 1), (72, 136, 17), (264, 72, 64),     # one slice, partial slices; up to 64 samples
    (264, 56, 300), (4096, 32, 40), (40, 24, 5),   # rows narrower than a slice
    (1000, 2056, 65), (1504, 520, 128),          # up to 128 samples
    (1504, 3000, 200), (2040, 1032, 256),        # up to 256, k-split
    (520, 1000, 300), (1000, 4104, 520),         # several tiles of samples, the last one ragged
    (8192, 264, 100), (16400, 72, 40),           # rows at and past the longest that one workgroup keeps in registers
    (8816, 136, 65), (8352, 480, 67),            # samples in tiles of 128: 64 and 128 classes, without and with a k-split
    (8296, 136, 129), (5416, 152, 705),          # in tiles of 256
    (3232, 1840, 142),                           # and with a k-split
    (4208, 400, 67),                             # a k-split of rows of 4097 to 8192 classes
]


@pytest.mark.parametrize("J,D,B", SHAPES)
@pytest.mark.parametrize("layout", ["plain", "copy", "planes"])
def test_stream_forward(sfb, oracle, J, D, B, layout):
    print("stream forward", J, D, B, layout, flush=True)
    ctx = sfb.Context(0)
    W0 = S.normal_matrix(J, D, 0.05, seed=31)
    X, y = S.mlr_batch(J, D, B, seed=31, zero_frac=0.5, bf16=True)
    W = dev(W0)
    if layout == "copy":
        ctx.sfb_shadow_attach(W)
    elif layout == "planes":
        ctx.sfb_split_attach(W)
    U = torch.empty((B, J), dtype=torch.bfloat16, device="cuda:0")
    V = torch.empty((B, D), dtype=torch.bfloat16, device="cuda:0")
    Xd = dev_bf16(X)
    ctx.sfb_compute_sf(sfb.SFB_MLR, W, Xd, Y=dev(y), U=U, V=V)
    torch.cuda.synchronize()
    assert torch.equal(V.view(torch.int16), Xd.view(torch.int16))
    Uo, _ = oracle.mlr_sf(W0, X, y)
    mlr_u_check(U.float().cpu().numpy(), Uo, y, TOL_BF16)
    ctx.close()


def test_workspace_without_room_for_a_split(sfb, oracle):
    """A workspace with one plane of logits is enough: the same call then does not split k."""
    J, D, B = 1504, 3000, 200
    ru = lambda x, a=256: (x + a - 1) // a * a
    planes1 = ru(ru(B, 256) * ru(J, 256) * 4) + ru(ru(B, 256) * ru(D, 64) * 2)
    W0 = S.normal_matrix(J, D, 0.05, seed=35)
    X, y = S.mlr_batch(J, D, B, seed=35, zero_frac=0.5, bf16=True)
    Uo, _ = oracle.mlr_sf(W0, X, y)
    for layout in ("plain", "planes"):
        ctx = sfb.Context(0)
        W = dev(W0)
        if layout == "planes":
            ctx.sfb_split_attach(W)
        U = torch.empty((B, J), dtype=torch.bfloat16, device="cuda:0")
        args = (sfb.SFB_MLR, W, dev_bf16(X))
        ctx.sfb_compute_sf(*args, Y=dev(y), U=U)
        size = planes1 + (sfb.lib().sfb_shadow_bytes(J, D) if layout == "plain" else 0)
        assert size < sfb.lib().sfb_workspace_bytes(sfb.SFB_MLR, J, D, _batch(sfb, B))
        ws = torch.empty(size, dtype=torch.uint8, device="cuda:0")
        assert ws.data_ptr() % 256 == 0
        ctx._ensure_workspace = lambda *a, **k: None
        assert sfb.lib().sfb_set_workspace(ctx._h, ws.data_ptr(), size) == 0
        U2 = torch.empty_like(U)
        ctx.sfb_compute_sf(*args, Y=dev(y), U=U2)
        torch.cuda.synchronize()
        mlr_u_check(U2.float().cpu().numpy(), Uo, y, TOL_BF16)
        assert sfb.lib().sfb_set_workspace(ctx._h, ws.data_ptr(), size - 256) == 0
        with pytest.raises(sfb.SfbError) as e:
            ctx.sfb_compute_sf(*args, Y=dev(y), U=U2)
        assert e.value.code == sfb.SFB_ENOWS
        ctx.close()


def _batch(sfb, B):
    import ctypes
    b = sfb.binding.sfb_batch()
    b.B, b.in_dtype, b.sf_dtype = B, sfb.SFB_BF16, sfb.SFB_BF16
    return ctypes.byref(b)

"""The streaming bf16 forward on samples as they come (whole 64s of features): edges of its sample tiles, fewer k-slices than
stages, with a k-split, W as fp32 and as its bf16 copy; 64 features more or less than whole 64s go through the padded copy.

Tolerance: products of bf16 are exact in fp32; a logit is an fp32 sum of D of them, within D 2^-24 times the sum of their absolute
values; the softmax turns an error d of two logits into a relative one of at most 2 d, its exponentials and their sum add
(J + 4) 2^-24; the factor is rounded to bf16 (2^-8 of it).
"""
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu
EPS = 2.0 ** -24

# test_kernel_plans.py asserts that these take the streaming kernel, with and without a k-split
SHAPES = [(1, 64, 64), (63, 72, 128), (64, 520, 192), (65, 1000, 256), (255, 264, 1024), (256, 1504, 2048), (257, 2000, 1024),
          (513, 520, 2048), (300, 4104, 1088), (100, 520, 8192), (600, 1000, 2048), (300, 8192, 1024), (256, 8192, 2048), (100, 1000, 1000), (257, 264, 1032)]


@pytest.mark.parametrize("copy", [False, True])
@pytest.mark.parametrize("B,J,D", SHAPES)
def test_forward(B, J, D, copy):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_1409_5705_amd as sfb
    print("forward", B, J, D, copy, flush=True)
    g = torch.Generator(device="cuda:0").manual_seed(B + J + D)
    W = torch.randn(J, D, generator=g, device="cuda:0") / D ** 0.5
    X = torch.randn(B, D, generator=g, device="cuda:0").bfloat16()
    y = torch.randint(0, J, (B,), generator=g, device="cuda:0").to(torch.int32)
    U = torch.full((B, J), 7.0, device="cuda:0", dtype=torch.bfloat16)
    c = sfb.Context(0)
    if copy:
        c.sfb_shadow_attach(W)
    c.sfb_compute_sf(sfb.SFB_MLR, W, X, Y=y, U=U)
    Wb, Xd = W.bfloat16().double(), X.double()
    p = torch.softmax(Xd @ Wb.t(), dim=1)
    err = 2 * (D * EPS * (Xd.abs() @ Wb.abs().t())).amax(dim=1, keepdim=True) + (J + 4) * EPS
    ref = p.clone()
    ref[torch.arange(B, device="cuda:0"), y.long()] -= 1.0
    assert bool(torch.all((U.double() - ref).abs() <= p * err + 2.0 ** -8 * ref.abs() + 2 * EPS))
    c.close()

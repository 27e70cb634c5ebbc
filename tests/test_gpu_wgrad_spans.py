"""The weight gradient's staged spans (dilations up to 16, up to 32, beyond) at
their edges, dilations past the image, images of one column or row and pixels
carried over rows and images, against the FP64 reference."""
import numpy as np
import pytest

from oracle import conv_ref as C

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def G():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2404_12968_amd import gabp
    return gabp


def _bf16(a):
    return torch.tensor(a, dtype=torch.float32).to(torch.bfloat16)


CASES = [(2, 40, 70, 16), (2, 40, 70, 17), (1, 50, 90, 32), (1, 50, 90, 33), (2, 3, 1, 5),
         (70, 1, 1, 2), (3, 2, 63, 17), (1, 5, 300, 150), (2, 9, 64, 16), (1, 2, 129, 1000),
         (1, 40, 48, 1), (4, 70, 5, 27)]


@pytest.mark.parametrize("B,H,W,dil", CASES)
@pytest.mark.parametrize("cin,cout,relu", [(16, 16, False), (16, 32, True), (32, 16, True),
                                           (32, 32, False)])
def test_weight_gradient_at_span_edges(G, B, H, W, dil, cin, cout, relu):
    rng = np.random.default_rng(H * W + dil + cout)
    x = _bf16(rng.normal(size=(B, H, W, cin)))
    w = np.zeros((32, 9 * cin))
    w[:cout] = rng.normal(size=(cout, 9 * cin)) * 0.2
    w = _bf16(w)
    y = _bf16(rng.normal(size=(B, H, W, cout)))
    dy = rng.normal(size=(B, H, W, cout)).astype(np.float32)
    dw, db, dx, _ = G.gabp_conv3x3_bwd(x.cuda(), y.cuda(), torch.tensor(dy, device="cuda"),
                                       w.cuda(), cout, dil, relu)
    mask = (y.double().numpy() > 0) if relu else 1.0
    dz = _bf16(dy * mask).double().numpy()
    dxr, dwr, dbr = C.conv3x3_bwd(x.double().numpy(), np.ones_like(dz), dz,
                                  w.double().numpy()[:cout].reshape(cout, 9, cin), dil, relu=False)
    # FP32 sums of exact products, at most 64 accumulations per chunk of 1024
    # pixels and 32 more: their rounding is far below 2e-5 of the sum's scale
    for got, ref in ((dw[:cout].reshape(cout, 9, cin), dwr), (db[:cout], dbr), (dx, dxr)):
        np.testing.assert_allclose(got.cpu().double().numpy(), ref, rtol=0,
                                   atol=2e-5 * (np.abs(ref).max() + 1.0))

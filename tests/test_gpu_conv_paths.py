"""The convolution kernels' dispatch: staged rows against direct loads (bitwise),
dilations past either's staging, and sizes at the edges of their tiles, against
the FP64 reference."""
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


def _weights(rng, cin, cout):
    w = np.zeros((32, 9 * cin))
    w[:cout] = rng.normal(size=(cout, 9 * cin)) * 0.2
    return _bf16(w)


@pytest.mark.parametrize("cin,cout", [(16, 16), (16, 32), (32, 16), (32, 32)])
@pytest.mark.parametrize("dil", [1, 27, 32])
@pytest.mark.parametrize("H,W", [(128, 200), (171, 128), (90, 255)])
def test_staged_rows_equal_direct_loads(G, cin, cout, dil, H, W):
    """A batch large enough for the row kernel against its images one at a
    time, which take the direct kernel: the same order of every sum, so the
    same bits.  Widths of whole and partial segments; an image no taller than
    the dilation's reach on both sides is among them."""
    B = -(-65536 // (H * W))
    assert H * W < 65536 <= B * H * W
    g = torch.Generator(device="cuda").manual_seed(cin + dil + W)
    x = torch.randn((B, H, W, cin), generator=g, device="cuda").to(torch.bfloat16)
    w = _weights(np.random.default_rng(dil), cin, cout).cuda()
    b = torch.randn(32, generator=g, device="cuda")
    yb, yf = G.gabp_conv3x3_fwd(x, w, b, cout, dil, True, want_bf16=True, want_f32=True)
    for k in range(B):
        rb, rf = G.gabp_conv3x3_fwd(x[k:k + 1].contiguous(), w, b, cout, dil, True,
                                    want_bf16=True, want_f32=True)
        assert torch.equal(yf[k], rf[0]) and torch.equal(yb[k], rb[0])


# one pixel, a row, a column, tiles of 32 and 128 pixels and their neighbours,
# images smaller than the dilation, dilations past the staged 32
FWD = [(1, 1, 1, 1), (2, 1, 33, 3), (1, 70, 1, 27), (1, 5, 31, 9), (1, 3, 129, 40),
       (2, 9, 20, 200), (1, 300, 220, 33)]


@pytest.mark.parametrize("B,H,W,dil", FWD)
@pytest.mark.parametrize("cin,cout", [(16, 32), (32, 16)])
def test_forward_at_tile_edges(G, B, H, W, dil, cin, cout):
    rng = np.random.default_rng(H * W + dil)
    x = _bf16(rng.normal(size=(B, H, W, cin)))
    w = _weights(rng, cin, cout)
    b = rng.normal(size=32).astype(np.float32)
    yb, yf = G.gabp_conv3x3_fwd(x.cuda(), w.cuda(), torch.tensor(b, device="cuda"), cout, dil,
                                False, want_bf16=True, want_f32=True)
    _, ref = C.conv3x3_fwd(x.double().numpy(), w.double().numpy()[:cout].reshape(cout, 9, cin),
                           b[:cout], dil, False)
    # FP32 sums of at most 288 exact products of BF16 values: 18 accumulations
    assert np.abs(yf.cpu().double().numpy() - ref).max() <= 2e-5 * (np.abs(ref).max() + 1.0)
    assert torch.equal(yb, yf.to(torch.bfloat16))

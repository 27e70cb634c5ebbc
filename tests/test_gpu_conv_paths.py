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


# one pixel, units of 64 and chunks of 1024 pixels and their neighbours, rows
# that straddle 16-pixel steps, dilations whose column shifts share a staged run
# (up to 32) and those that do not
BWD = [(1, 1, 1, 1), (1, 7, 9, 3), (1, 1, 65, 32), (1, 1025, 1, 9), (2, 16, 32, 33),
       (1, 31, 33, 40), (3, 25, 93, 27), (1, 64, 97, 70)]


@pytest.mark.parametrize("B,H,W,dil", BWD)
@pytest.mark.parametrize("cin,cout,relu", [(16, 16, True), (16, 32, False), (32, 16, False),
                                           (32, 32, True)])
def test_backward_at_unit_edges(G, B, H, W, dil, cin, cout, relu):
    rng = np.random.default_rng(H * W + dil)
    x = _bf16(rng.normal(size=(B, H, W, cin)))
    w = _weights(rng, cin, cout)
    y = _bf16(rng.normal(size=(B, H, W, cout)))
    dy = rng.normal(size=(B, H, W, cout)).astype(np.float32)
    dw, db, dx, _ = G.gabp_conv3x3_bwd(x.cuda(), y.cuda(), torch.tensor(dy, device="cuda"),
                                       w.cuda(), cout, dil, relu)
    mask = (y.double().numpy() > 0) if relu else 1.0
    dz = _bf16(dy * mask).double().numpy()
    dxr, dwr, dbr = C.conv3x3_bwd(x.double().numpy(), np.ones_like(dz), dz,
                                  w.double().numpy()[:cout].reshape(cout, 9, cin), dil, relu=False)
    assert torch.all(dw[cout:] == 0) and torch.all(db[cout:] == 0)
    # FP32 sums of exact products, at most 64 accumulations per chunk of 1024
    # pixels and 32 more: their rounding is far below 2e-5 of the sum's scale
    for got, ref in ((dw[:cout].reshape(cout, 9, cin), dwr), (db[:cout], dbr), (dx, dxr)):
        np.testing.assert_allclose(got.cpu().double().numpy(), ref, rtol=0,
                                   atol=2e-5 * (np.abs(ref).max() + 1.0))
    # without the data gradient: the same weight and bias gradients
    dw2, db2, none, _ = G.gabp_conv3x3_bwd(x.cuda(), y.cuda(), torch.tensor(dy, device="cuda"),
                                           w.cuda(), cout, dil, relu, need_dx=False)
    assert none is None and torch.equal(dw, dw2) and torch.equal(db, db2)


@pytest.mark.parametrize("W,dil", [(93, 9), (64, 1), (70, 40)])
def test_backward_infinite_input_reaches_only_its_taps(G, W, dil):
    """An infinite input pixel at the end of a row enters the weight gradient
    through the taps whose output pixel lies in the image and no others:
    out-of-image taps and padding are no terms of the sums."""
    B, H, cin, cout = 2, 12, 32, 32
    rng = np.random.default_rng(W)
    x = _bf16(rng.normal(size=(B, H, W, cin)))
    yq, xq, ci = 5, W - 1, 7
    x[1, yq, xq, ci] = float("inf")
    dy = torch.tensor(np.abs(rng.normal(size=(B, H, W, cout))) + 0.1, dtype=torch.float32)
    y = torch.ones((B, H, W, cout), dtype=torch.bfloat16)
    dw, _, _, _ = G.gabp_conv3x3_bwd(x.cuda(), y.cuda(), dy.cuda(), _weights(rng, cin, cout).cuda(),
                                     cout, dil, True)
    want = torch.ones(cout, 9, cin, dtype=torch.bool)
    for tap in range(9):
        py, px = yq - (tap // 3 - 1) * dil, xq - (tap % 3 - 1) * dil
        if 0 <= py < H and 0 <= px < W:
            want[:, tap, ci] = False
    assert torch.equal(torch.isfinite(dw[:cout].reshape(cout, 9, cin)).cpu(), want)

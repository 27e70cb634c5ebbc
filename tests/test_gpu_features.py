"""Network input features: repeated and ignored observations, sizes below and
above the observation count, outputs that are not 16-byte aligned."""
import ctypes
import math

import numpy as np
import pytest

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def G():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2404_12968_amd import gabp
    return gabp


@pytest.mark.parametrize("nx,ny,nobs", [(1, 1, 0), (1, 1, 5), (7, 3, 100), (64, 4, 256), (97, 41, 1),
                                        (300, 211, 5000)])
@pytest.mark.parametrize("offset", [0, 1, 8])
def test_features(G, nx, ny, nobs, offset):
    rng = np.random.default_rng(nx + nobs)
    cells = rng.integers(-1, nx * ny + 1, size=nobs)        # some outside: ignored
    y = rng.integers(-8, 9, size=nobs).astype(np.float64)   # sums exact in any order
    c, v = torch.from_numpy(cells).cuda(), torch.from_numpy(y).cuda()
    work = torch.full((2 * nx * ny,), 7.0, device="cuda")
    buf = torch.full((nx * ny * 16 + 32,), 9.0, dtype=torch.bfloat16, device="cuda")
    st = G._lib.gabp_warm_features(ctypes.c_int64(nobs), ctypes.c_void_p(c.data_ptr()),
                                   ctypes.c_void_p(v.data_ptr()), nx, ny, 0.2,
                                   ctypes.c_void_p(work.data_ptr()),
                                   ctypes.c_void_p(buf.data_ptr() + 2 * offset), None)
    torch.cuda.synchronize()
    assert st == G.GABP_OK
    inside = (cells >= 0) & (cells < nx * ny)
    cnt = np.bincount(cells[inside], minlength=nx * ny)
    tot = np.bincount(cells[inside], weights=y[inside], minlength=nx * ny)
    want = torch.zeros(nx * ny, 16)
    want[:, 0] = torch.from_numpy((cnt > 0).astype(np.float32))
    want[:, 1] = torch.from_numpy((tot.astype(np.float32) / np.maximum(cnt, 1).astype(np.float32)))
    want[:, 2] = math.log(0.2) + 2.5
    got = buf.cpu()
    assert torch.equal(got[offset:offset + nx * ny * 16].view(nx * ny, 16), want.to(torch.bfloat16))
    assert (got[:offset] == 9.0).all() and (got[offset + nx * ny * 16:] == 9.0).all()

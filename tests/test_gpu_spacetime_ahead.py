"""The information-only space-time iteration with its loads ahead (grids of
between one and two waves per SIMD) against the form that covers two slices per
workgroup, which has none, bit for bit at the edges of that range."""
import pytest

from paper_2404_12968_amd import inputs as I

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def G():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2404_12968_amd import gabp
    return gabp


N, P = I.BC_NEUMANN, I.BC_PERIODIC


# waves: tiles of 64 columns x rows x slices; 1024 and 2048 on 256 compute units
@pytest.mark.parametrize("nx,ny,nt,bcx,bcy", [
    (64, 128, 8, N, N), (64, 205, 5, P, N), (65, 171, 3, N, P), (130, 85, 8, N, N),
    (128, 128, 8, P, P), (64, 683, 3, N, N), (7, 300, 4, N, P)])
def test_loads_ahead_equal_two_slices_per_workgroup(G, nx, ny, nt, bcx, bcy):
    prob = I.small_spacetime(nx, ny, nt, bc_x=bcx, bc_y=bcy, seed=nx + ny, dtype="f32")
    ctxs = [G.gabp_st_create_problem(prob) for _ in range(2)]
    G.gabp_st_set_theta_slices(ctxs[1], 2)
    for c in ctxs:
        G.gabp_st_set_freeze_tolerance(c, 10**10, 1e9)
        G.gabp_st_iterate(c, 4, 0.4)
        G.gabp_st_residual(c)
        assert G.gabp_st_precision_frozen(c) == 4
        G.gabp_st_iterate(c, 7, 0.4)
    for a, b in zip(G.gabp_st_get_messages(ctxs[0]), G.gabp_st_get_messages(ctxs[1])):
        assert torch.equal(a, b)
    for a, b in zip(G.gabp_st_posterior(ctxs[0]), G.gabp_st_posterior(ctxs[1])):
        assert torch.equal(a, b)

"""Launches of several iterations with a grid spacing and scale other than one (the
couplings of tiles inside the grid are a constant of their own), on a stream of the
caller's: single iterations on the default stream, bit for bit."""
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


@pytest.mark.parametrize("dtype,alpha", [("f32", 2), ("f32", 1), ("f64", 2), ("f64", 1)])
@pytest.mark.parametrize("nx,ny", [(150, 140), (700, 610), (760, 700)])   # 2^19 nodes from the last on
def test_spacing_and_stream(G, dtype, alpha, nx, ny):
    prob = I.small_lattice(nx, ny, alpha, bc_x=I.BC_PERIODIC, kappa=0.31, tau=2.3, frac=0.1,
                           sigma=0.05, seed=nx, hx=0.7, hy=1.3, dtype=dtype)
    side = torch.cuda.Stream()
    with torch.cuda.stream(side):
        a = G.gabp_create_problem(prob)
    b = G.gabp_create_problem(prob)
    G.gabp_set_tile(b, 1, 0)

    def same():
        side.synchronize()
        for x, y in zip(G.gabp_get_messages(b), state()):
            assert torch.equal(x, y)

    def state():
        with torch.cuda.stream(side):
            m = G.gabp_get_messages(a)
        side.synchronize()
        return m

    for c in (a, b):
        G.gabp_iterate(c, 24, 0.5)
        G.gabp_set_freeze_tolerance(c, 10**9, 1e9)
    same()
    assert G.gabp_residual(a) == G.gabp_residual(b)
    assert G.gabp_precision_frozen(a) == G.gabp_precision_frozen(b) == 24
    for n in (33, 3, 5, 4, 2):
        for c in (a, b):
            G.gabp_iterate(c, n, 0.5)
        same()
    for most, check in ((20, 10), (9, 3), (8, 2), (9, 5)):
        assert G.gabp_solve(a, most, 0.5, 0.0, check) == G.gabp_solve(b, most, 0.5, 0.0, check)
        same()

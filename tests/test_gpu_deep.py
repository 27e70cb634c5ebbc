"""Several information-only iterations per launch (the default once the
precision messages froze) against one iteration per launch, bit for bit, and the
state kept after a divergence inside such a launch."""
import numpy as np
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


def _bits(t):
    return t.view(torch.int32 if t.dtype == torch.float32 else torch.int64)


def _same_state(G, a, b):
    pa, ia = G.gabp_get_messages(a)
    pb, ib = G.gabp_get_messages(b)
    return torch.equal(_bits(pa), _bits(pb)) and torch.equal(_bits(ia), _bits(ib))


def _frozen_pair(G, prob):
    """A context on the default launches and one on single iterations, both
    frozen at the same iteration (the tolerance accepts any change)."""
    ctxs = [G.gabp_create_problem(prob) for _ in range(2)]
    G.gabp_set_tile(ctxs[1], 1, 0)
    for c in ctxs:
        G.gabp_set_freeze_tolerance(c, 10**9, 1e9)
        G.gabp_iterate(c, 6, prob.damping)
        G.gabp_residual(c)
        assert G.gabp_precision_frozen(c) == 6
    return ctxs


N, P, D = I.BC_NEUMANN, I.BC_PERIODIC, I.BC_DIRICHLET
# smaller than the stencil's reach, one tile, tiles that end on and next to an
# axis' end, wrapped regions wider than the lattice, each region of each type
CASES = [
    ("f32", 2, 1, 1, N, D), ("f32", 2, 5, 7, P, P), ("f32", 2, 33, 17, P, N),
    ("f32", 2, 64, 64, N, N), ("f32", 2, 129, 40, D, P), ("f32", 2, 380, 390, N, P),
    ("f32", 2, 613, 520, P, D), ("f32", 1, 3, 3, P, P), ("f32", 1, 70, 31, N, P),
    ("f32", 1, 420, 333, P, N), ("f32", 1, 801, 790, D, N), ("f64", 2, 6, 40, P, N),
    ("f64", 2, 150, 70, N, P), ("f64", 2, 520, 500, D, D), ("f64", 1, 64, 64, N, N),
    ("f64", 1, 90, 130, P, D), ("f64", 1, 610, 560, N, P),
]


@pytest.mark.parametrize("dtype,alpha,nx,ny,bcx,bcy", CASES)
def test_deep_launches_equal_single_iterations(G, dtype, alpha, nx, ny, bcx, bcy):
    prob = I.small_lattice(nx, ny, alpha, bc_x=bcx, bc_y=bcy, kappa=0.12, frac=0.1, sigma=0.05,
                           seed=nx + ny, dtype=dtype)
    a, b = _frozen_pair(G, prob)
    before = G.gabp_launch_counts(a)
    for n in (1, 2, 3, 4, 7, 12, 13, 41):
        G.gabp_iterate(a, n, 0.5)
        G.gabp_iterate(b, n, 0.5)
        assert _same_state(G, a, b), n
        # the two buffers hold consecutive iterations
        assert G.gabp_message_change(a) == G.gabp_message_change(b)
    after = G.gabp_launch_counts(a)
    assert after["pair_tiles"] > before["pair_tiles"]
    assert after["theta"] - before["theta"] <= 9      # the last of each call, and n = 2's first
    # chunks of gabp_solve, recorded and replayed, end on launches of several
    for graphs in (True, False):
        G.gabp_set_graph(a, graphs)
        ra = G.gabp_solve(a, 50, 0.5, 0.0, 10)
        rb = G.gabp_solve(b, 50, 0.5, 0.0, 10)
        assert ra == rb and _same_state(G, a, b)
    ma, va = G.gabp_posterior(a)
    mb, vb = G.gabp_posterior(b)
    assert torch.equal(ma, mb) and torch.equal(va, vb)


@pytest.mark.parametrize("alpha,dtype", [(2, "f32"), (1, "f32"), (2, "f64")])
def test_divergence_keeps_the_state_of_two_iteration_launches(G, alpha, dtype):
    """Information messages that overflow after the precisions froze: the same
    status, iteration and kept messages as with two iterations per launch,
    whichever iteration of a launch meets it.  The observations come close to
    the type's largest number; the smaller they are, the later a belief's
    information overflows."""
    largest = 3.4e38 if dtype == "f32" else 1.7e308
    at = set()
    for k in range(30):
        prob = I.small_lattice(70, 50, alpha, kappa=0.05, frac=0.05, sigma=1.0, seed=3, dtype=dtype)
        prob.y = np.abs(prob.y) / np.abs(prob.y).max() * (largest * 10.0 ** (-0.025 * k))
        out = []
        for tile in (None, 4):
            c = G.gabp_create_problem(prob)
            if tile is not None:
                G.gabp_set_tile(c, 1, tile)
            G.gabp_set_freeze_tolerance(c, 10**9, 1e9)
            G.gabp_iterate(c, 6, 0.5)
            try:
                G.gabp_residual(c)
            except G.GabpError:
                break                       # diverged before the freeze
            assert G.gabp_precision_frozen(c) == 6
            G.gabp_iterate(c, 60, 0.5)
            G.gabp_iterate(c, 25, 0.5)
            out.append((G.gabp_iteration_count(c), G.gabp_last_error(c), c))
        if not out:
            continue
        assert out[0][:2] == out[1][:2], k
        assert _same_state(G, out[0][2], out[1][2]), k
        if out[0][0][1] == G.GABP_E_DIVERGED:
            at.add(out[0][1])
    assert len(at) >= 3

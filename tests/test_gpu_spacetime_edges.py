"""Space-time grids at the edges of what an iteration reaches: sides shorter
than the stencil, where every wrapped neighbour is one that does not exist, and
the shortest periodic axes, against the oracle at equal iterations."""
import pytest

from paper_2404_12968_amd import inputs as I
from tests.test_gpu_spacetime import G, S, compare, gpu_state, oracle_for  # noqa: F401

pytestmark = pytest.mark.gpu

N, P = I.BC_NEUMANN, I.BC_PERIODIC


@pytest.mark.parametrize("nx,ny,nt,bcx,bcy", [
    (1, 1, 1, N, N), (1, 9, 2, N, N), (2, 2, 2, N, N), (3, 1, 4, N, N), (4, 3, 1, N, N),
    (2, 70, 3, N, P), (66, 2, 2, P, N), (5, 5, 3, P, P), (65, 5, 2, N, P), (5, 66, 4, P, N)])
def test_short_axes_match_the_oracle(G, S, nx, ny, nt, bcx, bcy):  # noqa: F811
    from oracle import oracle as O
    prob = I.small_spacetime(nx, ny, nt, bc_x=bcx, bc_y=bcy, frac=0.3, seed=nx + 7 * ny + nt)
    og = oracle_for(S, O, prob)
    ctx = G.gabp_st_create_problem(prob)
    done = 0
    for t in (1, 2, 9):
        G.gabp_st_iterate(ctx, t - done, prob.damping)
        og.iterate(t - done, prob.damping)
        done = t
        compare(prob, og, gpu_state(G, ctx), 1e-12)

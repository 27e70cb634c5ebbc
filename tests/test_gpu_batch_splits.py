"""Batched runs of every small length, in changing order: how a run is split into
launches of several iterations and single ones follows its length, and the tiles
follow the longest launch.  Against lone contexts on single iterations, bit for bit."""
import random

import pytest

from paper_2404_12968_amd import inputs as I

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

N, P, D = I.BC_NEUMANN, I.BC_PERIODIC, I.BC_DIRICHLET
SETS = {   # both prior orders in one launch of single iterations, and too many for that
    "few": [(70, 41, 1, P, N), (33, 90, 2, N, D), (130, 17, 2, P, P)],
    "many": [(700, 333, 1, N, N), (520, 400, 2, P, N), (301, 260, 2, D, P)],
    "one order": [(150, 140, 2, N, N), (90, 301, 2, N, P)],
}


@pytest.fixture(scope="module")
def G():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2404_12968_amd import gabp
    return gabp


@pytest.mark.parametrize("dtype", ["f32", "f64"])
@pytest.mark.parametrize("name", SETS)
def test_run_lengths(G, dtype, name):
    probs = [I.small_lattice(nx, ny, a, bc_x=bx, bc_y=by, kappa=0.15, frac=0.1, sigma=0.05,
                             seed=nx + ny, dtype=dtype) for nx, ny, a, bx, by in SETS[name]]
    b = G.gabp_batch_create(probs)
    ctxs = [G.gabp_create_problem(p) for p in probs]
    for c in ctxs:
        G.gabp_set_tile(c, 1, 0)
    lengths = list(range(1, 14)) + [5, 5, 2, 9, 1, 6]
    random.Random(3).shuffle(lengths)

    def run(tag):
        for n in lengths:
            G.gabp_batch_iterate(b, n, 0.5)
            for i, c in enumerate(ctxs):
                G.gabp_iterate(c, n, 0.5)
                for x, y in zip(G.gabp_batch_get_messages(b, i), G.gabp_get_messages(c)):
                    assert torch.equal(x, y), (tag, n, i)
        for n in lengths[:8]:                    # and without a copy between the runs
            G.gabp_batch_iterate(b, n, 0.5)
            for c in ctxs:
                G.gabp_iterate(c, n, 0.5)
        for i, c in enumerate(ctxs):
            for x, y in zip(G.gabp_batch_get_messages(b, i), G.gabp_get_messages(c)):
                assert torch.equal(x, y), (tag, i)

    run("full")
    G.gabp_batch_set_freeze_tolerance(b, 10**9, 1e9)
    _, its, _, _ = G.gabp_batch_solve(b, 3, 0.5, 0.0, 3)
    for i, c in enumerate(ctxs):
        G.gabp_set_freeze_tolerance(c, 10**9, 1e9)
        G.gabp_solve(c, 3, 0.5, 0.0, 3)
        assert G.gabp_precision_frozen(c) == G.gabp_batch_info(b, i)[1] == its[i]
    run("information-only")

"""Chunk graphs of a context with a tile set (only those record and replay): the
results of direct launches bit for bit, and a divergence inside a replayed chunk."""
import numpy as np
import pytest

from paper_2404_12968_amd import inputs as I
from conftest import plane_slot_map

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def G():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2404_12968_amd import gabp
    return gabp


def _same(G, a, b):
    return all(torch.equal(x, y) for x, y in zip(G.gabp_get_messages(a), G.gabp_get_messages(b)))


@pytest.mark.parametrize("dtype,alpha,pair", [("f32", 2, 12), ("f64", 1, 4), ("f32", 1, -4),
                                              ("f64", 2, 0)])
def test_replayed_chunks_equal_direct_launches(G, dtype, alpha, pair):
    """Eager checks, freeze tests and the gain set-up run between the replays; chunks
    of two lengths, before and after the precision messages froze."""
    prob = I.small_lattice(190, 130, alpha, bc_x=I.BC_PERIODIC, kappa=0.1, tracks=5, run=4,
                           sigma=0.05, seed=77, dtype=dtype)
    a, b = G.gabp_create_problem(prob), G.gabp_create_problem(prob)
    for c in (a, b):
        G.gabp_set_tile(c, 2, pair)
        G.gabp_set_freeze_tolerance(c, 64, 1e-6)
    G.gabp_set_graph(b, False)
    for check in (10, 7):
        ra, rb = (G.gabp_solve(c, 300, 0.5, 0.0, check) for c in (a, b))
        assert ra == rb and _same(G, a, b)
        assert G.gabp_precision_frozen(a) == G.gabp_precision_frozen(b) > 0
        assert G.gabp_launch_counts(a) == G.gabp_launch_counts(b)
    # direct iterations of the replaying context go on from its counter
    for c in (a, b):
        G.gabp_iterate(c, 13, 0.5)
    ra, rb = (G.gabp_solve(c, 20, 0.5, 0.0, 10) for c in (a, b))
    assert ra == rb and _same(G, a, b)


@pytest.mark.parametrize("check", [4, 6])
def test_divergence_inside_a_replayed_chunk(G, oracle_mod, check):
    """Reported at the oracle's iteration, numbered from the device's counter."""
    prob = I.small_lattice(16, 16, 2, kappa=0.05, c=2.0, frac=0.05, sigma=0.05, seed=7, dtype="f64")
    og = oracle_mod.OracleGaBP.from_problem(prob)
    assert og.iterate(200, 0.2) == oracle_mod.STATUS_DIVERGED
    for graphs in (True, False):
        c = G.gabp_create_problem(prob)
        G.gabp_set_tile(c, 1, 4)
        G.gabp_set_graph(c, graphs)
        st, it, _ = G.gabp_solve(c, 200, 0.2, 0.0, check)
        assert st == G.GABP_E_DIVERGED and it == og.diverged_at and it > 3 * check
        d, y, x, e = plane_slot_map(prob, og.g)
        p = G.gabp_get_messages(c)[0].cpu().numpy()[d, y, x]
        fin = np.isfinite(p) & np.isfinite(og.lam[e])
        assert fin.sum() > 100
        np.testing.assert_allclose(p[fin], og.lam[e][fin], rtol=1e-9)


@pytest.mark.parametrize("dtype", ["f32", "f64"])
def test_overflow_inside_a_replayed_chunk_after_the_freeze(G, dtype):
    """The state of direct two-iteration launches, whichever replay meets it."""
    largest = 3.4e38 if dtype == "f32" else 1.7e308
    at = set()
    for k in range(24):
        prob = I.small_lattice(70, 50, 2, kappa=0.05, frac=0.05, sigma=1.0, seed=3, dtype=dtype)
        prob.y = np.abs(prob.y) / np.abs(prob.y).max() * (largest * 10.0 ** (-0.025 * k))
        out = []
        for graphs in (True, False):
            c = G.gabp_create_problem(prob)
            G.gabp_set_tile(c, 1, 4)
            G.gabp_set_graph(c, graphs)
            G.gabp_set_freeze_tolerance(c, 10**9, 1e9)
            G.gabp_iterate(c, 6, 0.5)
            try:
                G.gabp_residual(c)
            except G.GabpError:
                break                       # diverged before the freeze
            r = G.gabp_solve(c, 60, 0.5, 0.0, 10)
            out.append((r[:2], G.gabp_last_error(c), c))
        if len(out) < 2:
            continue
        assert out[0][:2] == out[1][:2] and _same_bits(G, out[0][2], out[1][2]), k
        if out[0][0][0] == G.GABP_E_DIVERGED:
            at.add(out[0][0][1])
    assert len(at) >= 2


def _same_bits(G, a, b):
    i = torch.int32 if G.gabp_get_messages(a)[0].dtype == torch.float32 else torch.int64
    return all(torch.equal(x.view(i), y.view(i))
               for x, y in zip(G.gabp_get_messages(a), G.gabp_get_messages(b)))

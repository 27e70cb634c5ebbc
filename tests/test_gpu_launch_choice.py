"""Which launches a context takes, and what its two message buffers then hold."""
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


def _frozen(G, dtype, alpha, tile):
    prob = I.small_lattice(130, 90, alpha, bc_x=I.BC_PERIODIC, kappa=0.12, frac=0.1, sigma=0.05,
                           seed=5, dtype=dtype)
    c = G.gabp_create_problem(prob)
    if tile is not None:
        G.gabp_set_tile(c, *tile)
    G.gabp_set_freeze_tolerance(c, 10**9, 1e9)
    G.gabp_iterate(c, 6, 0.5)
    G.gabp_residual(c)
    assert G.gabp_precision_frozen(c) == 6
    return c


@pytest.mark.parametrize("dtype,alpha", [("f32", 2), ("f32", 1), ("f64", 2), ("f64", 1)])
def test_a_chunk_of_odd_length_ends_on_consecutive_iterations(G, dtype, alpha):
    """gabp_message_change after a solve whose last chunk was odd."""
    a, b = _frozen(G, dtype, alpha, None), _frozen(G, dtype, alpha, (1, 0))
    for most, check in ((25, 10), (7, 7), (3, 10), (1, 10)):
        ra, rb = (G.gabp_solve(c, most, 0.5, 0.0, check) for c in (a, b))
        assert ra == rb
        assert G.gabp_message_change(a) == G.gabp_message_change(b), most
        for x, y in zip(G.gabp_get_messages(a), G.gabp_get_messages(b)):
            assert torch.equal(x, y)


@pytest.mark.parametrize("dtype,alpha", [("f32", 2), ("f64", 1)])
def test_the_autotuner_gives_a_context_its_default_launches(G, dtype, alpha):
    """They are faster than every tile shape, so a set tile ends there."""
    a, b = _frozen(G, dtype, alpha, (4, 4)), _frozen(G, dtype, alpha, None)
    G.gabp_autotune(a, 1, 0.5)
    t, _ = G.gabp_iteration_count(a)
    G.gabp_iterate(b, t - 6, 0.5)
    for c in (a, b):
        before = G.gabp_launch_counts(c)["pair_tiles"]
        G.gabp_iterate(c, 61, 0.5)
        assert G.gabp_launch_counts(c)["pair_tiles"] - before < 25   # 30 of two iterations
    for x, y in zip(G.gabp_get_messages(a), G.gabp_get_messages(b)):
        assert torch.equal(x, y)


def test_the_batch_autotuner_chooses_among_what_it_times(G):
    """Rows per thread belong to the single iterations of instances not frozen:
    with none, the default of one row stays, and the iterations are the same."""
    probs = [I.small_lattice(nx, ny, a, kappa=0.15, frac=0.1, sigma=0.05, seed=nx, dtype="f32")
             for nx, ny, a in ((140, 90, 2), (60, 75, 1), (200, 33, 2))]
    a, b = G.gabp_batch_create(probs), G.gabp_batch_create(probs)
    for x in (a, b):
        G.gabp_batch_set_freeze_tolerance(x, 10**9, 1e9)
        G.gabp_batch_solve(x, 6, 0.5, 0.0, 6)
        assert all(G.gabp_batch_info(x, i) == (6, 6, True) for i in range(3))
    for trials in (3, 5, 4):
        assert G.gabp_batch_autotune(a, trials, 0.5) == 1
        G.gabp_batch_iterate(b, 1 + 8 * trials, 0.5)
        for i in range(3):
            assert G.gabp_batch_info(a, i) == G.gabp_batch_info(b, i)
            for x, y in zip(G.gabp_batch_get_messages(a, i), G.gabp_batch_get_messages(b, i)):
                assert torch.equal(x, y)

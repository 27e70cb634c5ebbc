"""The freeze test stops reading once too many precision messages changed: it
still accepts exactly the tolerance's number of changed messages and refuses
one more, wherever the changes lie."""
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


@pytest.mark.parametrize("dtype,alpha,nx,ny,iters", [
    ("f32", 2, 40, 30, 3), ("f32", 2, 300, 170, 33), ("f32", 1, 65, 700, 25), ("f64", 2, 90, 110, 60),
    ("f64", 1, 50, 40, 70)])
def test_freeze_accepts_exactly_the_tolerated_count(G, dtype, alpha, nx, ny, iters):
    prob = I.small_lattice(nx, ny, alpha, kappa=0.2, frac=0.1, seed=nx, dtype=dtype)
    view = torch.int32 if dtype == "f32" else torch.int64
    # the last of these iterations that still changed more than one message:
    # the fewer changes, the more of the buffers the test has to read
    ref = G.gabp_create_problem(prob)
    G.gabp_set_tile(ref, 1, 0)
    last = None
    for t in range(1, iters + 2):
        G.gabp_iterate(ref, 1, 0.5)
        now, _ = G.gabp_get_messages(ref)
        if t > 2 and int((now.view(view) != last.view(view)).sum()) > 1:
            at, p0, p1 = t, last, now
        last = now
    changed = int((p0.view(view) != p1.view(view)).sum())
    for slots, frozen in ((changed, True), (changed - 1, False), (1, False), (10 * changed, True)):
        c = G.gabp_create_problem(prob)
        G.gabp_set_freeze_tolerance(c, slots, 1e9)
        G.gabp_iterate(c, at, 0.5)
        G.gabp_residual(c)
        assert (G.gabp_precision_frozen(c) == at) == frozen, slots
    # a relative bound just below the largest change refuses, just above accepts
    a, b = p0.double().abs(), p1.double().abs()
    rel = ((p0.double() - p1.double()).abs() / torch.maximum(a, b).clamp(min=1e-300)).max().item()
    for bound, frozen in ((rel * 0.999, False), (rel * 1.001, True)):
        c = G.gabp_create_problem(prob)
        G.gabp_set_freeze_tolerance(c, changed, bound)
        G.gabp_iterate(c, at, 0.5)
        G.gabp_residual(c)
        assert (G.gabp_precision_frozen(c) == at) == frozen, bound


def test_batched_freeze_count_is_per_instance(G):
    """Instances whose changes lie on either side of the tolerance: each
    freezes as it does alone."""
    probs = [I.small_lattice(40 + 17 * k, 70 - 9 * k, 1 + k % 2, kappa=0.1 + 0.05 * k, frac=0.1,
                             seed=k, dtype="f32") for k in range(5)]
    for slots in (0, 20, 1000, 10**6):
        b = G.gabp_batch_create(probs)
        G.gabp_batch_set_freeze_tolerance(b, slots, 1e9)
        G.gabp_batch_solve(b, 60, 0.5, 0.0, 10)
        for k, p in enumerate(probs):
            c = G.gabp_create_problem(p)
            G.gabp_set_freeze_tolerance(c, slots, 1e9)
            G.gabp_solve(c, 60, 0.5, 0.0, 10)
            assert G.gabp_batch_info(b, k)[1] == G.gabp_precision_frozen(c), (slots, k)

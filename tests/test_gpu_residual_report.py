"""The residual at the number of workgroups (64 x 4 tiles) up to which they count
themselves, one below and one above it: |A mu - b| against the oracle's assembled
system, the same at every one of several checks of one state, and after more
iterations again."""
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


@pytest.mark.parametrize("nx,ny,alpha", [
    (5, 4, 1), (64, 64, 2), (60, 124, 1), (64, 128, 1), (64, 128, 2), (61, 129, 1), (64, 132, 2),
    (130, 41, 2), (130, 45, 1),
])
def test_every_check_reports_the_oracles_residual(G, oracle_mod, nx, ny, alpha):
    prob = I.small_lattice(nx, ny, alpha, kappa=0.2, frac=0.1, sigma=0.1, seed=nx + ny,
                           dtype="f64")
    A, b = oracle_mod.posterior_system(prob)
    ctx = G.gabp_create_problem(prob)
    for its in (7, 10):
        G.gabp_iterate(ctx, its, 0.5)
        first = G.gabp_residual(ctx)
        assert [G.gabp_residual(ctx) for _ in range(3)] == [first] * 3
        mu, _ = G.gabp_posterior(ctx, want_var=False)
        want = np.linalg.norm(A @ mu.cpu().numpy().ravel() - b)
        # FP64 sums of some 10^5 terms, as in the other residual tests
        assert first[1] == pytest.approx(want, rel=1e-11)
        assert first[0] == pytest.approx(want / np.linalg.norm(b), rel=1e-11)

"""A grid of one node has no messages, so none can be invalid: whatever its data
term is in message precision, the iterations go on and the mean is the FP64 one."""
import dataclasses

import numpy as np
import pytest

from paper_2404_12968_amd import inputs as I

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

SIGMA = 4.4e-20                     # precision 5e38: infinite in FP32
Y = np.array([2.51, 8.45, 2.16])    # their residual does not round to zero


@pytest.fixture(scope="module")
def G():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2404_12968_amd import gabp
    return gabp


def _one(alpha):
    p = I.small_lattice(1, 1, alpha, bc_x=I.BC_DIRICHLET, kappa=0.3, dtype="f32")
    return dataclasses.replace(p, cells=np.zeros(3, np.int64), y=Y, sigma=SIGMA, var=None)


@pytest.mark.parametrize("alpha", [1, 2])
@pytest.mark.parametrize("tile", [None, (1, 0)])
def test_lattice(G, alpha, tile):
    c = G.gabp_create_problem(_one(alpha))
    if tile is not None:
        G.gabp_set_tile(c, *tile)
    G.gabp_iterate(c, 4, 0.5)
    rel, _ = G.gabp_residual(c)
    assert G.gabp_precision_frozen(c) == 4
    G.gabp_iterate(c, 20, 0.5)
    assert G.gabp_iteration_count(c) == (24, G.GABP_OK)
    assert G.gabp_residual(c)[0] == rel <= 1e-14
    assert G.gabp_posterior(c)[0].item() == pytest.approx(Y.mean(), rel=1e-14)


@pytest.mark.parametrize("alpha", [1, 2])
def test_batch(G, alpha):
    other = I.small_lattice(20, 15, alpha, kappa=0.3, dtype="f32")
    b = G.gabp_batch_create([_one(alpha), other])
    G.gabp_batch_set_freeze_tolerance(b, 10**9, 1e9)
    G.gabp_batch_solve(b, 4, 0.5, 0.0, 4)
    assert G.gabp_batch_info(b, 0) == (4, 4, True)
    _, its, _, sts = G.gabp_batch_solve(b, 20, 0.5, 0.0, 20)
    assert (its[0], sts[0]) == (24, G.GABP_E_NOT_CONVERGED)
    assert G.gabp_batch_posterior(b, 0)[0].item() == pytest.approx(Y.mean(), rel=1e-14)


@pytest.mark.parametrize("slices", [1, 2, 4])
def test_spacetime(G, slices):
    p = I.small_spacetime(1, 1, 1, frac=1.0, dtype="f32")
    p = dataclasses.replace(p, cells=np.zeros(3, np.int64), y=Y, sigma=SIGMA, var=None)
    c = G.gabp_st_create_problem(p)
    G.gabp_st_set_theta_slices(c, slices)
    G.gabp_st_iterate(c, 2, 0.5)
    G.gabp_st_residual(c)
    assert G.gabp_st_precision_frozen(c) == 2
    G.gabp_st_iterate(c, 20, 0.5)
    G.gabp_st_residual(c)
    assert G.gabp_st_posterior(c)[0].item() == pytest.approx(Y.mean(), rel=1e-14)
    prec, info = G.gabp_st_get_messages(c)
    assert not prec.any() and not info.any()

"""Observations in their cells' order (folded as they come) and in any other
(sorted first): the same node terms bit for bit, the same refusals."""
import dataclasses

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


def _observations(n_cells, count, seed):
    """(cells, y, var) with runs of one cell, in a random order, and the same
    observations stably sorted by cell."""
    rng = np.random.default_rng(seed)
    cells = rng.integers(0, n_cells, size=count)
    cells[count // 2:] = cells[:count - count // 2]
    y, var = rng.standard_normal(count), rng.uniform(0.01, 0.5, size=count)
    o = np.argsort(cells, kind="stable")
    return (cells, y, var), (cells[o], y[o], var[o])


def _unique(n_cells, count, seed):
    """The same without repeated cells."""
    rng = np.random.default_rng(seed)
    cells = rng.permutation(n_cells)[:count]
    y, var = rng.standard_normal(count), rng.uniform(0.01, 0.5, size=count)
    o = np.argsort(cells)
    return (cells, y, var), (cells[o], y[o], var[o])


def _with(prob, obs, with_var):
    return dataclasses.replace(prob, cells=obs[0], y=obs[1], var=obs[2] if with_var else None)


def _state(G, prob, prior):
    c = G.gabp_create_problem(prob, prior_mean=prior)
    G.gabp_iterate(c, 3, 0.5)
    return (*G.gabp_get_messages(c), *G.gabp_posterior(c), torch.tensor(G.gabp_residual(c)))


def _equal(a, b):
    return all(torch.equal(x, y) for x, y in zip(a, b))


@pytest.mark.parametrize("count", [1, 2, 255, 257, 5000])
@pytest.mark.parametrize("with_var", [False, True])
@pytest.mark.parametrize("dtype", ["f32", "f64"])
def test_lattice_terms_do_not_depend_on_the_order_of_cells(G, count, with_var, dtype):
    prob = I.small_lattice(70, 45, 2, kappa=0.2, seed=1, dtype=dtype)
    prior = np.random.default_rng(2).standard_normal((45, 70)) if with_var else None
    for draw in (_observations, _unique):
        shuffled, ordered = draw(70 * 45, min(count, 70 * 45), count)
        assert _equal(_state(G, _with(prob, shuffled, with_var), prior),
                      _state(G, _with(prob, ordered, with_var), prior))


@pytest.mark.parametrize("dtype", ["f32", "f64"])
def test_batch_terms_do_not_depend_on_the_order_of_cells(G, dtype):
    probs = []
    for k, (nx, ny) in enumerate([(40, 30), (70, 11), (33, 64)]):
        p = I.small_lattice(nx, ny, 1 + k % 2, kappa=0.2, seed=k, dtype=dtype)
        shuffled, ordered = _observations(nx * ny, 400, k)
        probs.append((_with(p, shuffled, k == 2), _with(p, ordered, k == 2)))
    out = []
    # some instances in order, some not; all in order
    for sel in ((0, 1, 0), (1, 1, 1)):
        b = G.gabp_batch_create([p[s] for p, s in zip(probs, sel)])
        G.gabp_batch_iterate(b, 3, 0.5)
        out.append([t for i in range(3) for t in G.gabp_batch_get_messages(b, i)])
        _, its, rels, _ = G.gabp_batch_solve(b, 10, 0.5, 0.0, 10)
        assert (its == 13).all()
        out[-1].append(torch.tensor(rels))
    assert _equal(out[0], out[1])


@pytest.mark.parametrize("dtype", ["f32", "f64"])
def test_spacetime_terms_do_not_depend_on_the_order_of_cells(G, dtype):
    prob = I.small_spacetime(20, 15, 5, dtype=dtype)
    shuffled, ordered = _observations(20 * 15 * 5, 300, 4)
    out = []
    for obs in (shuffled, ordered):
        c = G.gabp_st_create_problem(_with(prob, obs, True))
        G.gabp_st_iterate(c, 3, 0.5)
        out.append([*G.gabp_st_posterior(c), torch.tensor(G.gabp_st_residual(c))])
    assert _equal(out[0], out[1])


@pytest.mark.parametrize("bad", ["cell", "y", "var"])
@pytest.mark.parametrize("ordered", [False, True])
def test_invalid_observations_are_refused_in_any_order(G, bad, ordered):
    prob = I.small_lattice(30, 20, 2, kappa=0.2, seed=1, dtype="f32")
    cells, y, var = _observations(600, 100, 9)[1 if ordered else 0]
    k = 99 if bad == "cell" else 50
    if bad == "cell":
        cells[k] = 600
    elif bad == "y":
        y[k] = np.inf
    else:
        var[k] = 0.0
    p = _with(prob, (cells, y, var), True)
    with pytest.raises(G.GabpError):
        G.gabp_create_problem(p)
    with pytest.raises(G.GabpError):
        G.gabp_batch_create([p])

"""Observations with cells repeated out of order: given in host memory, a few (sorted
inside the workspace) or more than fit there; the node terms of the same
observations ordered by cell, bit for bit."""
import ctypes

import numpy as np
import pytest

from paper_2404_12968_amd import inputs as I

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

N, A = (90, 41), 2


@pytest.fixture(scope="module")
def G():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2404_12968_amd import gabp
    return gabp


def _obs(count, seed):
    rng = np.random.default_rng(seed)
    cells = rng.integers(0, N[0] * N[1], size=count)
    cells[count // 2:] = cells[:count - count // 2]
    y, var = rng.standard_normal(count), rng.uniform(0.01, 0.5, size=count)
    o = np.argsort(cells, kind="stable")
    return (cells, y, var), (cells[o], y[o], var[o])


def _fill(G, a, obs, device, keep):
    t = [np.ascontiguousarray(v) for v in obs]
    if device:
        t = [torch.from_numpy(v).cuda() for v in t]
    keep.append(t)
    p = [v.data_ptr() if device else v.ctypes.data for v in t]
    a.grid, a.stencil = G._grid(*N), G._stencil(A, 0.2, 1.0, 10.0)
    a.obs = G.gabp_obs(len(obs[0]), p[0], p[1], 1 if device else 0)
    a.noise = G.gabp_noise(0.0, p[2])


def _batch(G, sets, device, dtype):
    """(status, messages and means after three iterations) of a batch."""
    arr, keep, h = (G.gabp_instance * len(sets))(), [], ctypes.c_void_p()
    for a, o, d in zip(arr, sets, device):
        _fill(G, a, o, d, keep)
    opts = G.gabp_opts(dtype, torch.cuda.current_stream().cuda_stream, None, 0, None)
    st = G._lib.gabp_batch_create(len(sets), arr, ctypes.byref(opts), ctypes.byref(h))
    if st != G.GABP_OK:
        return st, None
    b = G.Batch(h, None, [(*N, 12)] * len(sets), dtype, torch.device("cuda"), None)
    G.gabp_batch_iterate(b, 3, 0.5)
    out = []
    for i in range(len(sets)):
        out += [*G.gabp_batch_get_messages(b, i), *G.gabp_batch_posterior(b, i)]
    rels = G.gabp_batch_solve(b, 2, 0.5, 0.0, 2)[2]
    G.gabp_batch_destroy(b)
    return st, out + [torch.tensor(rels)]


def _equal(a, b):
    return all(torch.equal(x, y) for x, y in zip(a, b))


@pytest.mark.parametrize("dtype", [0, 1])
@pytest.mark.parametrize("count", [2, 300, 30000])
def test_batch(G, dtype, count):
    draws = [_obs(count, k) for k in range(4)]
    want = _batch(G, [d[1] for d in draws], [True] * 4, dtype)[1]
    for device in ([False] * 4, [True] * 4, [False, True, False, True]):
        for order in ((0, 0, 0, 0), (0, 1, 1, 0), (1, 0, 0, 1)):
            st, got = _batch(G, [d[o] for d, o in zip(draws, order)], device, dtype)
            assert st == G.GABP_OK and _equal(got, want), (device, order)


@pytest.mark.parametrize("dtype", [0, 1])
@pytest.mark.parametrize("count", [2, 300, 30000])
def test_lattice(G, dtype, count):
    out = []
    for obs, device in zip(2 * _obs(count, 9), (False, False, True, True)):
        inst, keep, h = G.gabp_instance(), [], ctypes.c_void_p()
        _fill(G, inst, obs, device, keep)
        opts = G.gabp_opts(dtype, torch.cuda.current_stream().cuda_stream, None, 0, None)
        r = [ctypes.byref(x) for x in (inst.grid, inst.stencil, inst.obs, inst.noise, opts, h)]
        assert G._lib.gabp_create(*r) == G.GABP_OK
        c = G.Context(h, None, None, *N, dtype, torch.device("cuda"))
        G.gabp_iterate(c, 3, 0.5)
        out.append([*G.gabp_get_messages(c), *G.gabp_posterior(c),
                    torch.tensor(G.gabp_residual(c))])
        G.gabp_iterate(c, 4, 0.5)
        out[-1] += G.gabp_get_messages(c)
    assert all(_equal(out[0], o) for o in out[1:])


@pytest.mark.parametrize("device", [False, True])
@pytest.mark.parametrize("what", ["cell", "y", "var"])
def test_an_invalid_observation_among_repeated_cells_is_refused(G, device, what):
    good, bad = _obs(300, 1)[0], [v.copy() for v in _obs(300, 2)[0]]
    bad[("cell", "y", "var").index(what)][211] = {"cell": N[0] * N[1], "y": np.nan, "var": 0.0}[what]
    assert _batch(G, [good, bad, good], [device] * 3, 0)[0] == G.GABP_E_INVALID

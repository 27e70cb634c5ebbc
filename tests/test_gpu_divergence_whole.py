"""The messages kept after a divergence are one whole iteration, also on a lattice
with more workgroups than run at once: those that start after the first invalid
value was recorded still write theirs."""
import dataclasses
import functools

import numpy as np
import pytest

from paper_2404_12968_amd import inputs as I

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

NX, NY = 1024, 2048     # 8192 tiles of 64 x 4


@pytest.fixture(scope="module")
def G():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2404_12968_amd import gabp
    return gabp


@functools.lru_cache(None)
def _base(alpha):
    return I.small_lattice(NX, NY, alpha, kappa=0.05, frac=0.02, sigma=1.0, seed=3, dtype="f32")


def _problem(alpha, scale):
    """Observed values in the first tile near the largest FP32 number (scale 0: the
    same lattice without them), so that information messages overflow there."""
    p = _base(alpha)
    first = (p.cells % NX < 64) & (p.cells // NX < 4)
    assert first.sum() > 0
    return dataclasses.replace(p, y=np.where(first, 3.4e38 * scale, p.y))


def _frozen(G, p, tile):
    c = G.gabp_create_problem(p)
    if tile is not None:
        G.gabp_set_tile(c, *tile)
    G.gabp_set_freeze_tolerance(c, 10**9, 1e9)
    G.gabp_iterate(c, 6, 0.5)
    try:
        G.gabp_residual(c)
    except G.GabpError:
        return None                         # diverged before the freeze
    assert G.gabp_precision_frozen(c) == 6
    return c


def _same(a, b):
    return torch.equal(a.view(torch.int32), b.view(torch.int32))


def _whole(kept, ref, alpha, it):
    """The rows that the overflow does not reach in `it` iterations are those of a
    run without it, the precision messages are its everywhere."""
    far = 4 + alpha * it
    return _same(kept[0], ref[0]) and _same(kept[1][:, far:], ref[1][:, far:])


SCALES = [10.0 ** (-0.04 * k) for k in range(16)]


@pytest.mark.parametrize("alpha", [1, 2])
def test_information_only_iterations(G, alpha):
    at = set()
    for s in SCALES:
        out = []
        for tile in (None, (1, 4), (1, -2), (4, 0)):
            c = _frozen(G, _problem(alpha, s), tile)
            if c is None:
                break
            G.gabp_iterate(c, 60, 0.5)
            it, st = G.gabp_iteration_count(c)
            if st != G.GABP_E_DIVERGED:
                break
            r = _frozen(G, _problem(alpha, 0.0), (1, 0))
            G.gabp_iterate(r, it - 6, 0.5)
            kept = G.gabp_get_messages(c)
            assert _whole(kept, G.gabp_get_messages(r), alpha, it), (s, tile, it)
            out.append((it, kept))
        if len(out) == 4:
            at.add(out[0][0])
            # as two-iteration launches keep it
            for other in out[1:3]:
                assert out[0][0] == other[0] and all(map(_same, out[0][1], other[1])), s
    assert len(at) >= 2


@pytest.mark.parametrize("alpha", [1, 2])
def test_full_iterations(G, alpha):
    at = set()
    for s in SCALES:
        out = []
        for tile in (None, (1, 0), (8, 4)):
            c = G.gabp_create_problem(_problem(alpha, s))
            if tile is not None:
                G.gabp_set_tile(c, *tile)
            G.gabp_iterate(c, 40, 0.5)
            it, st = G.gabp_iteration_count(c)
            if st != G.GABP_E_DIVERGED:
                break
            r = G.gabp_create_problem(_problem(alpha, 0.0))
            G.gabp_iterate(r, it, 0.5)
            kept = G.gabp_get_messages(c)
            assert _whole(kept, G.gabp_get_messages(r), alpha, it), (s, tile, it)
            out.append((it, kept))
        if len(out) == 3:
            at.add(out[0][0])
            assert out[0][0] == out[1][0] == out[2][0]
            assert all(_same(a, b) for o in out[1:] for a, b in zip(out[0][1], o[1]))
    assert len(at) >= 2


@pytest.mark.parametrize("frozen", [False, True])
@pytest.mark.parametrize("single", [False, True], ids=["several", "single"])
def test_batch(G, frozen, single):
    """`single`: one iteration a call, so that the overflow is met by a launch of
    one iteration."""
    probs = [_problem(2, s) for s in SCALES[::4]] + [_problem(2, 0.0)]
    b = G.gabp_batch_create(probs)
    G.gabp_batch_set_freeze_tolerance(b, 10**9, 1e9)
    start = 6 if frozen else 0
    if frozen:
        G.gabp_batch_solve(b, 6, 0.5, 0.0, 6)
    for n in [1] * 40 if single else [40]:
        G.gabp_batch_iterate(b, n, 0.5)
    _, its, _, sts = G.gabp_batch_solve(b, 1, 0.5, 0.0, 1)
    at = set()
    for i in range(len(probs) - 1):
        was = G.gabp_batch_info(b, i)[1]
        if sts[i] != G.GABP_E_DIVERGED or (was >= 0) != frozen:
            continue
        r = _frozen(G, probs[-1], (1, 0)) if frozen else G.gabp_create_problem(probs[-1])
        G.gabp_iterate(r, int(its[i]) - start, 0.5)
        assert _whole(G.gabp_batch_get_messages(b, i), G.gabp_get_messages(r), 2,
                      int(its[i])), (i, its[i])
        at.add(int(its[i]))
    assert len(at) >= 2

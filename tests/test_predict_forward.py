"""``warm.predict`` takes a network's own ``forward``, whatever defines it."""
import pytest

from paper_2404_12968_amd import build as B

torch = pytest.importorskip("torch")


@pytest.fixture()
def W(monkeypatch):
    import os
    if not os.path.exists(B.LIB):
        pytest.skip("libgabp.so is not built")
    from paper_2404_12968_amd import warm
    monkeypatch.setattr(warm.G, "gabp_warm_features",
                        lambda cells, y, nx, ny, kappa, device: torch.ones(ny, nx, 16))
    return warm


def _problem():
    from paper_2404_12968_amd import inputs as I
    return I.small_lattice(5, 4, 2, kappa=0.2)


def _forward(x):
    assert x.shape == (1, 4, 5, 16)
    return [x], 3.0 * x


def test_predict_calls_the_forward_it_is_given(W):
    class Own(W.WarmNet):
        def forward(self, x):
            return _forward(x)

    class Alone:
        forward = staticmethod(_forward)

    patched = W.WarmNet(device="cpu")
    patched.forward = _forward
    for net in (Own(device="cpu"), Alone(), patched):
        p = W.predict(net, _problem(), device="cpu")
        assert p.shape == (4, 5, 16) and bool((p == 3.0).all())


def test_predict_infers_with_the_library_network(W, monkeypatch):
    monkeypatch.setattr(W.WarmNet, "_infer", lambda self, x: 5.0 * x)
    p = W.predict(W.WarmNet(device="cpu"), _problem(), device="cpu")
    assert p.shape == (4, 5, 16) and bool((p == 5.0).all())

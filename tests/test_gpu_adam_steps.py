"""Adam on a list of tensors against one tensor at a time: lists that fill a
launch, go past one and past two, tensors around a workgroup's size, with and
without a BF16 copy."""
import pytest

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def G():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2404_12968_amd import gabp
    return gabp


@pytest.mark.parametrize("count", [1, 2, 15, 16, 17, 33])
def test_adam_steps_equal_single_steps(G, count):
    sizes = [1, 32, 255, 256, 257, 9216, 4608]
    gen = torch.Generator(device="cuda").manual_seed(count)
    a, b = [], []
    for k in range(count):
        n = sizes[k % len(sizes)]
        w, g, m = (torch.randn(n, generator=gen, device="cuda") for _ in range(3))
        v = torch.rand(n, generator=gen, device="cuda")
        wb = w.to(torch.bfloat16) if k % 3 else None
        a.append((w, g, m, v, wb))
        b.append(tuple(None if t is None else t.clone() for t in a[-1]))
    for step in (1, 2, 50):
        G.gabp_adam_steps(a, 1e-2, 0.9, 0.999, 1e-8, step)
        for w, g, m, v, wb in b:
            G.gabp_adam_step(w, g, m, v, wb, 1e-2, 0.9, 0.999, 1e-8, step)
    for x, y in zip(a, b):
        for s, t in zip(x, y):
            assert s is None or torch.equal(s, t)


def test_adam_steps_refuses_what_a_single_step_refuses(G):
    w = torch.ones(4, device="cuda")
    with pytest.raises(G.GabpError):
        G.gabp_adam_steps([(w, w, w, None, None)], 1e-2, 0.9, 0.999, 1e-8, 1)
    with pytest.raises(G.GabpError):
        G.gabp_adam_steps([(w, w, w, w, None)], 1e-2, 0.9, 0.999, 1e-8, 0)

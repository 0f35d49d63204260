"""The 4-wide traversal against the brute-force closest hit of the same rays (every
triangle through the same triangle test), at the sizes where a node's slots can go
wrong: one leaf, one node, two levels, partly filled nodes; at tmin below, at and
above zero; and rays that run along the axes or hit nothing."""
import sys

import numpy as np
import pytest

torch = pytest.importorskip("torch")

from paper_2012_03939_amd import scenes as S

pytestmark = pytest.mark.gpu


def _say(msg):
    print(msg, flush=True)
    sys.stdout.flush()


@pytest.fixture(scope="module")
def B():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2012_03939_amd import binding
    binding.load()
    return binding


def _rays(n, seed):
    rng = np.random.default_rng(seed)
    o = rng.normal(size=(n, 3))
    o *= (rng.uniform(0.0, 3.0, n) / np.linalg.norm(o, axis=1))[:, None]
    d = 0.8 * rng.normal(size=(n, 3)) - o
    axis = np.eye(3)[rng.integers(0, 3, n)] * rng.choice([-1.0, 1.0], n)[:, None]
    d = np.where(rng.random(n)[:, None] < 0.2, axis, d / np.linalg.norm(d, axis=1, keepdims=True))
    return [torch.from_numpy(x.astype(np.float32)).cuda() for x in (o, d)]


@pytest.mark.parametrize("tmin", [1e-4, 0.0, -0.0, -2.5, -1e38, 0.7])
@pytest.mark.parametrize("nf", [1, 2, 3, 4, 5, 6, 9, 17, 65, 2000])
def test_traversal_equals_brute_force(B, nf, tmin):
    _say(f"case traversal: {nf} faces, tmin {tmin}")
    rng = np.random.default_rng(nf)
    V, F = S.noise_sphere(10, 0.2, noise_seed=3)
    F = F[rng.permutation(F.shape[0])[:nf]]
    g = B.GPUScene(V.astype(np.float32), F, S.random_materials(nf, rng), None, None)
    o, d = _rays(4099, 7 + nf)
    f, t = g.trace(o, d, tmin=tmin)
    fb, tb = g.trace(o, d, tmin=tmin, brute=True)
    torch.cuda.synchronize()
    g.check_errors()
    assert torch.equal(f, fb) and torch.equal(t, tb)


@pytest.mark.parametrize("nf", [1, 3, 500, 20480])
def test_fast_and_counting_traversals_agree(B, nf):
    """Renders and their adjoints with work counters take the 64-bit traversal,
    those without the 32-bit one: the same images bit for bit, the same radiance on
    both sides of every primary edge sample (so the same gradients, up to the
    order of the adjoint's atomic sums)."""
    _say(f"case traversal variants: {nf} faces")
    rng = np.random.default_rng(nf)
    V, F = S.noise_sphere(5 if nf <= 500 else 32, 0.2, noise_seed=3)
    F = F[:nf]
    g = B.GPUScene(V.astype(np.float32), F, S.random_materials(nf, rng), S.hemisphere_lights(1, rng),
                   S.gaussian_lobe_envmap(rng, 32, 16))
    cams = [S.look_at_origin((0.5, 2.0, 2.0), 48, 40), S.look_at_origin((-2.5, 0.4, 1.5), 45, 33)]
    a = g.render(cams, 4, 3, seed=2)
    b = g.render(cams, 4, 3, seed=2, flags=B.ST_COUNT_WORK)
    assert torch.equal(a, b)
    d = torch.randn(a.shape, generator=torch.Generator("cuda").manual_seed(1), device="cuda")
    ga = g.backward(cams, 4, 3, d, seed=2)
    gb = g.backward(cams, 4, 3, d, seed=2, flags=B.ST_ALL_GRADS | B.ST_COUNT_WORK)
    torch.cuda.synchronize()
    g.check_errors()
    for x, y in zip(ga, gb):
        # float32 sums of the same terms in another order
        assert torch.allclose(x, y, rtol=1e-4, atol=1e-4 * float(x.abs().max()))


@pytest.mark.parametrize("size", [(1, 1), (9, 7), (64, 1), (65, 1), (256, 512), (363, 362), (1024, 1024), (1031, 1021)])
def test_tile_counts(B, size):
    """Rays in tiles of 64 over the waves of a launch: fewer tiles than waves, as many,
    one more (2,048 waves in the allocation-free render, 16,384 in the other), and the
    same paths in small chunks, give the same image bit for bit."""
    w, h = size
    _say(f"case tiles: {w}x{h}")
    rng = np.random.default_rng(11)
    V, F = S.noise_sphere(6, 0.2, noise_seed=4)
    g = B.GPUScene(V.astype(np.float32), F, S.random_materials(F.shape[0], rng), S.hemisphere_lights(1, rng),
                   S.gaussian_lobe_envmap(rng, 32, 16))
    cams = [S.look_at_origin((0.5, 2.0, 2.0), w, h)]
    a = g.render(cams, 1, 2, seed=5)
    b = g.render(cams, 1, 2, seed=5, queue_capacity=100000)
    torch.cuda.synchronize()
    assert torch.equal(a, b)
    if w * h <= 1 << 20:
        assert torch.equal(a, g.render_noalloc(cams, 1, 2, seed=5))
    g.check_errors()

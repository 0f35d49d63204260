"""Launches of one to four blocks whose shading points have several shadow entries, so that
the traversal has more tiles of 64 rays than waves: thumbnails, single rows of pixels,
small chunks, short last chunks, several scenes, few edge samples."""
import sys

import numpy as np
import pytest

torch = pytest.importorskip("torch")

from paper_2012_03939_amd import scenes as S
from parity_util import GRAD_RTOL, rel_l2

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


def _scene(nl, env, scene_id=0):
    rng = np.random.default_rng(40 + nl + scene_id)
    V, F = S.noise_sphere(6, 0.2, noise_seed=4 + scene_id)
    return S.Scene(V.astype(np.float32), F, S.random_materials(F.shape[0], rng), S.hemisphere_lights(nl, rng),
                   S.gaussian_lobe_envmap(rng, 32, 16) if env else None, scene_id)


def _close_up(w, h):
    return S.look_at_origin((0.3, 0.8, 1.3), w, h)      # the mesh fills the view


@pytest.mark.parametrize("bounces", [1, 2, 3])
@pytest.mark.parametrize("nl,env", [(2, False), (3, True), (16, True)])
@pytest.mark.parametrize("size", [(8, 8), (16, 8), (16, 16), (257, 1), (16, 32), (24, 32), (769, 1)])
def test_small_views(B, size, nl, env, bounces):
    _say(f"case small view: {size[0]}x{size[1]}, {nl} lights, environment {env}, {bounces} bounces")
    g = B.GPUScene.from_scene(_scene(nl, env))
    cams = [_close_up(*size)]
    # an earlier pass over the same workspace, whose outcomes must not show
    g.render([S.look_at_origin((0.0, -0.4, 2.5), *size)], 1, bounces, seed=8)
    a = g.render(cams, 1, bounces, seed=9)
    m = g.render(cams, 1, bounces, seed=9, flags=B.ST_FORWARD_MEGAKERNEL)
    assert torch.equal(a, g.render_noalloc(cams, 1, bounces, seed=9))
    g.check_errors()
    # at most 17 entries at each of three points: 51 float32 roundings of 6e-8
    assert float(m.max()) > 0 and rel_l2(a.cpu().numpy(), m.cpu().numpy()) < 1e-5


@pytest.mark.parametrize("cap", [64, 128, 256, 512, 768])
@pytest.mark.parametrize("nl", [3, 16])
def test_small_chunks(B, nl, cap):
    _say(f"case small chunks: {nl} lights and an environment, chunks of {cap}")
    g = B.GPUScene.from_scene(_scene(nl, True))
    cams = [_close_up(45, 37)]
    a = g.render(cams, 2, 2, seed=3)
    assert torch.equal(a, g.render(cams, 2, 2, seed=3, queue_capacity=cap))
    # chunks of 2,560 paths and a last one of 770; of cap
    for c in (2560, cap):
        assert torch.equal(a, g.render_noalloc(cams, 2, 2, seed=3, queue_capacity=c))
    g.check_errors()


def test_small_batch(B):
    _say("case small batch: three scenes of 3, 16 and 0 lights, views of 8x8 to 16x16")
    scenes = [B.GPUScene.from_scene(_scene(nl, env, i)) for i, (nl, env) in enumerate([(3, False), (16, True), (0, True)])]
    cams = [_close_up(8, 8), _close_up(16, 16), _close_up(9, 7), _close_up(16, 8)]
    which = [0, 1, 2, 1]
    out = B.render_batch(scenes, cams, which, 1, 2, seed=4)
    got, at = {}, 0
    for c, s in zip(cams, which):
        got.setdefault(s, []).append(out[at:at + c.width * c.height])
        at += c.width * c.height
    for s, parts in got.items():
        mine = [c for c, w in zip(cams, which) if w == s]
        assert torch.equal(torch.cat(parts), scenes[s].render(mine, 1, 2, seed=4))
        scenes[s].check_errors()


@pytest.mark.parametrize("size", [(8, 8), (16, 16), (24, 16)])
@pytest.mark.parametrize("nl", [3, 16])
def test_few_edge_samples(B, nl, size):
    """Side paths of 64 to 384 primary edge samples, and the adjoint of the paths' hit
    records, against the oracle and against tracing again."""
    from test_gpu_parity import _backward_case
    _say(f"case few edge samples: {size[0]}x{size[1]}, {nl} lights and an environment")
    sc = _scene(nl, True)
    cams = [S.look_at_origin((0.3, 0.9, 3.1), *size)]
    d = np.random.default_rng(6).normal(size=(size[0] * size[1], 3)).astype(np.float32)
    _, ef, rv, _, oV, _ = _backward_case(B, sc, cams, 1, 2, d, 2)
    _say(f"  edge flips {ef:.5f} relL2 dV {rv:.2e}")
    assert np.abs(oV).max() > 0
    # of so few samples 0.1 % is none: one may fall the other way (and is masked out)
    assert ef * size[0] * size[1] * (1 + nl) < 1.5 and rv < GRAD_RTOL
    g = B.GPUScene.from_scene(sc)
    dt = torch.from_numpy(d).cuda()
    g.render(cams, 1, 2, seed=2)
    a = [x.cpu().numpy() for x in g.backward(cams, 1, 2, dt, 2, 7)]
    b = [x.cpu().numpy() for x in g.backward(cams, 1, 2, dt, 2, 7 | B.ST_BACKWARD_RETRACE)]
    g.check_errors()
    for x, y in zip(a, b):
        # the recorded hit's distance from its plane, and float32 sums in another order
        assert rel_l2(x, y) < GRAD_RTOL


@pytest.mark.parametrize("cap", [1, 2, 3, 129])
def test_smallest_side_chunks(B, cap):
    """A backward in chunks of the fewest paths: two, the side paths of one edge sample."""
    import ctypes
    _say(f"case smallest side chunks: {cap}")
    g = B.GPUScene.from_scene(_scene(3, False))
    cams = [S.look_at_origin((0.3, 0.9, 3.1), 8, 8)]
    d = torch.ones((64, 3), device="cuda")
    want = g.backward(cams, 1, 1, d, 2, B.ST_EDGE_PRIMARY)[0].cpu().numpy()
    dV, dM = torch.empty((g.nv, 3), device="cuda"), torch.empty((g.ntex, 7), device="cuda")
    o = B.make_opts(flags=B.ST_EDGE_PRIMARY, queue_capacity=cap)
    B._check(B.load().st_render_backward(g.h, B.make_cameras(cams), 1, 1, 1, 2, ctypes.byref(o), B._ptr(d), B._ptr(dV),
                                         B._ptr(dM), B._stream()))
    g.check_errors()
    # float64 sums of the same terms in another order, rounded to float32
    assert np.abs(want).max() > 0 and rel_l2(dV.cpu().numpy(), want) < 1e-6

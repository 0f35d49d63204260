"""The wavefront queues beside a program that holds most of the device's memory: the larger
default chunk is left out, nothing is allocated by later calls of the same shapes, and a
captured graph's workspace is not given up for one that cannot be had."""
import sys

import numpy as np
import pytest

torch = pytest.importorskip("torch")

from paper_2012_03939_amd import scenes as S

pytestmark = pytest.mark.gpu

GB = 1 << 30
SIZE, SPP = 512, 65               # just over 2^24 path samples: two chunks of 2^24, one of 2^25
PATHS = SIZE * SIZE * SPP
PATH_BYTES = 177 * 4 + 17         # queue bytes of a path with 17 shadow entries
LARGE = PATHS * PATH_BYTES * 9 // 8                # with the eighth that a workspace is grown by
SMALL = (PATHS // 2 + 256) * PATH_BYTES * 9 // 8


@pytest.fixture(scope="module")
def B():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2012_03939_amd import binding
    binding.load()
    return binding


def _scene(B):
    rng = np.random.default_rng(5)
    V, F = S.noise_sphere(4, 0.15, noise_seed=2)
    return B.GPUScene.from_scene(S.Scene(V.astype(np.float32), F, S.random_materials(F.shape[0], rng),
                                         S.hemisphere_lights(16, rng), S.gaussian_lobe_envmap(rng, 32, 16)))


def _free():
    torch.cuda.synchronize()
    return torch.cuda.mem_get_info()[0]


def _leave(room):
    """A tensor that leaves `room` bytes of the device's memory free."""
    torch.cuda.empty_cache()
    print(f"  {_free() / GB:.1f} GiB free, taking all but {room / GB:.1f}", flush=True)
    return torch.empty(_free() - room, dtype=torch.uint8, device="cuda")


def test_no_room_for_the_larger_queues(B):
    print(f"case queue memory: {SIZE}^2 at {SPP} spp, 17 shadow entries, 10.5 GiB free", flush=True)
    sys.stdout.flush()
    g = _scene(B)
    cams = [S.look_at_origin((0.4, 1.2, 3.0), SIZE, SIZE)]
    out = torch.empty((SIZE * SIZE, 3), device="cuda")
    room = int(10.5 * GB)
    assert LARGE > room and SMALL + GB < room < 2 * SMALL      # the smaller queues fit, once
    held = _leave(room)
    try:
        side = torch.cuda.Stream()
        side.wait_stream(torch.cuda.current_stream())
        with torch.cuda.stream(side):
            want = g.render(cams, SPP, 1, seed=1, out=out).clone()
        torch.cuda.current_stream().wait_stream(side)
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph):
            g.render(cams, SPP, 1, seed=1, out=out)
        graph.replay()                       # (the runtime's memory of the graph and of the comparison)
        assert torch.equal(out, want)
        before = _free()
        for _ in range(3):
            out.zero_()
            g.render(cams, SPP, 1, seed=1, out=out)
            assert torch.equal(out, want)
            out.zero_()
            graph.replay()
            torch.cuda.synchronize()
            assert torch.equal(out, want)
        assert _free() == before
        g.check_errors()
    finally:
        del held
        torch.cuda.empty_cache()


def test_less_than_half_of_the_memory_free(B):
    print(f"case queue memory: {SIZE}^2 at {SPP} spp, 17 shadow entries, 45 % of the memory free", flush=True)
    sys.stdout.flush()
    g = _scene(B)
    cams = [S.look_at_origin((0.4, 1.2, 3.0), SIZE, SIZE)]
    out = torch.empty((SIZE * SIZE, 3), device="cuda")
    held = _leave(int(0.45 * torch.cuda.mem_get_info()[1]))
    try:
        before = _free()
        want = g.render(cams, SPP, 1, seed=1, out=out).clone()
        after = _free()
        # 1 GiB for radiance, hit records, spill stack and the copy of the image
        assert before - after <= SMALL + GB
    finally:
        del held
        torch.cuda.empty_cache()
    # with the memory back, the same call keeps what it has
    assert torch.equal(out, want)
    before = _free()
    g.render(cams, SPP, 1, seed=1, out=out)
    assert _free() == before and torch.equal(out, want)
    g.check_errors()

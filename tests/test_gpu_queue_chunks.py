"""Chunks of the wavefront queues where a call has more path samples than the default
chunk of a tight memory cap: the call is accepted with as little memory as 2^24 paths'
queues need, and gives the same image and gradients."""
import sys

import numpy as np
import pytest

torch = pytest.importorskip("torch")

from paper_2012_03939_amd import scenes as S
from parity_util import rel_l2

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def B():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2012_03939_amd import binding
    binding.load()
    return binding


@pytest.mark.parametrize("spp", [65, 129])
def test_smaller_chunks_under_a_memory_cap(B, spp):
    print(f"case queue chunks: 512^2, {spp} spp, one light", flush=True)
    sys.stdout.flush()
    V, F = S.noise_sphere(4, 0.15, noise_seed=2)
    lights = np.array([[0.5, 3.0, 1.0, 9.0, 9.0, 9.0]], np.float32)
    g = B.GPUScene(V.astype(np.float32), F, S.uniform_materials(F.shape[0]), lights)
    cams = [S.look_at_origin((0.4, 1.2, 3.0), 512, 512)]
    d = torch.ones((512 * 512, 3), device="cuda")
    want = g.render(cams, spp, 1, seed=1)
    wV, wM = (x.clone() for x in g.backward(cams, spp, 1, d, 1, B.ST_ALL_GRADS))
    lo, hi = 1 << 20, 1 << 40
    img = torch.empty_like(want)
    while hi - lo > 1 << 20:
        mid = (lo + hi) // 2
        try:
            g.render(cams, spp, 1, seed=1, out=img, max_workspace_bytes=mid)
            hi = mid
        except B.StError:
            lo = mid
    # radiance (12 bytes a path), spill stack (48 words for 2^20 threads) and queues of
    # at most 2^24 paths (49 words and a byte each), with 8 MB for what is per launch
    assert hi <= 12 * 512 * 512 * spp + 4 * 48 * (1 << 20) + (4 * 49 + 1) * (1 << 24) + (8 << 20)
    img.zero_()
    g.render(cams, spp, 1, seed=1, out=img, max_workspace_bytes=hi)
    assert torch.equal(img, want)
    lo, hi = 1 << 20, 1 << 40
    while hi - lo > 1 << 30:
        mid = (lo + hi) // 2
        try:
            V2, M2 = g.backward(cams, spp, 1, d, 1, B.ST_ALL_GRADS, max_workspace_bytes=mid)
            hi = mid
        except B.StError:
            lo = mid
    V2, M2 = g.backward(cams, spp, 1, d, 1, B.ST_ALL_GRADS, max_workspace_bytes=hi)
    # float32 sums of the same terms in another order of atomics
    assert rel_l2(V2.cpu().numpy(), wV.cpu().numpy()) < 1e-5
    assert rel_l2(M2.cpu().numpy(), wM.cpu().numpy()) < 1e-5
    g.check_errors()

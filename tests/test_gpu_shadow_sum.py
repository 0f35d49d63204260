"""The sum of a shading point's shadow contributions at the entry counts around the groups
in which it reads them, against the megakernel's running sum."""
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


@pytest.mark.parametrize("nl,env", [(2, False), (3, True), (4, False), (4, True), (8, True), (16, False), (16, True)])
def test_shadow_sum_groups(B, nl, env):
    print(f"case shadow sum: {nl} lights, environment {env}", flush=True)
    sys.stdout.flush()
    rng = np.random.default_rng(nl)
    V, F = S.noise_torus(24, 12, 0.1, noise_seed=3)
    sc = S.Scene(V.astype(np.float32), F, S.random_materials(F.shape[0], rng), S.hemisphere_lights(nl, rng),
                 S.gaussian_lobe_envmap(rng, 32, 16) if env else None)
    g = B.GPUScene.from_scene(sc)
    cams = [S.look_at_origin((0.4, 1.2, 3.0), 48, 40), S.look_at_origin((-2.0, 1.0, 2.2), 33, 17)]
    a = g.render(cams, 4, 2, seed=9).cpu().numpy()
    b = g.render(cams, 4, 2, seed=9, flags=B.ST_FORWARD_MEGAKERNEL).cpu().numpy()
    g.check_errors()
    assert a.max() > 0
    # at most 17 entries at two points of four samples: 136 float32 roundings of 6e-8
    assert rel_l2(a, b) < 1e-5

"""Edges of no weight are never drawn, also where the sums of the edges' CDF round.

The mesh is one part twice, so that its first half has exactly half of the silhouette
length, and the first half ends with the inner edges of a flat patch, which no light sees
as silhouettes.  A sample whose place in the CDF is exactly 1/2 belongs to an edge beside
that run; a CDF that rises by a rounding inside the run would give it one of the run's.
The seeds are such that one sample of the view and light has u0 = 0."""
import collections
import sys

import numpy as np
import pytest

torch = pytest.importorskip("torch")

from paper_2012_03939_amd import scenes as S
from philox_ref import draw4

pytestmark = pytest.mark.gpu

SIZE = 8                       # of a view: 64 samples a light, the 32nd at 1/2
LIGHTS = 16


@pytest.fixture(scope="module")
def B():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2012_03939_amd import binding
    binding.load()
    return binding


def _mesh(k):
    """Twice 20 squares and a patch of 8x8 cells in the plane z = 0; the vertices on the
    patch's boundary come first, so that a run of inner edges ends each half's list."""
    sizes = np.random.default_rng(k).integers(3, 200, (20, 2)) / 256.0
    V, F = [], []
    m = 8
    grid = sorted(((i, j) for i in range(m + 1) for j in range(m + 1)), key=lambda p: (0 < p[0] < m and 0 < p[1] < m, p))
    for half in range(2):
        for j, (a, b) in enumerate(sizes):
            v, x, y = len(V), 4.0 * j, 8.0 * half
            V += [(x, y, 0), (x + a, y + b, 0), (x + a - b, y + b + a, 0), (x - b, y + a, 0)]
            F += [(v, v + 1, v + 2), (v, v + 2, v + 3)]
        at = {p: len(V) + t for t, p in enumerate(grid)}
        V += [(-20.0 + i / 4 - j / 8, 8.0 * half + i / 8 + j / 4, 0) for i, j in grid]
        for i in range(m):
            for j in range(m):
                F += [(at[i, j], at[i + 1, j], at[i + 1, j + 1]), (at[i, j], at[i + 1, j + 1], at[i, j + 1])]
    return np.array(V, np.float32), np.array(F, np.int32)


def _fnv(*words):
    h = 0x811C9DC5
    for w in words:
        for b in range(4):
            h = ((h ^ (w >> (8 * b) & 0xFF)) * 0x01000193) & 0xFFFFFFFF
    return h


@pytest.mark.parametrize("seed,view,light", [(20415, 56, 13), (55289, 46, 9)])
@pytest.mark.parametrize("k", [3, 15, 18, 24])
def test_edges_of_no_weight_are_not_drawn(B, k, seed, view, light):
    print(f"case edge CDF: mesh {k}, seed {seed}, view {view}, light {light}", flush=True)
    sys.stdout.flush()
    n = SIZE * SIZE
    assert draw4(n // 2, view << 16 | light, 3, 3, seed, 0)[0] == 0.0
    V, F = _mesh(k)
    faces = collections.Counter(tuple(sorted((int(t[q]), int(t[(q + 1) % 3])))) for t in F for q in range(3))
    edges = sorted(faces)
    outline = np.array([faces[e] == 1 for e in edges])
    rng = np.random.default_rng(1)
    lights = np.concatenate([rng.uniform(-30, 90, (LIGHTS, 2)), rng.uniform(20, 40, (LIGHTS, 1)),
                             np.full((LIGHTS, 3), 50.0)], axis=1).astype(np.float32)
    g = B.GPUScene(V, F, S.uniform_materials(F.shape[0]), lights)
    assert np.array_equal(g.edges().cpu().numpy()[:, :2], np.array(edges))
    cams = [S.look_at_origin((0.0, 0.0, 60.0 + v), SIZE, SIZE) for v in range(view + 1)]
    h = torch.zeros(B.num_edge_samples(cams, 1, 1.0, LIGHTS), dtype=torch.int32, device="cuda")
    d = torch.ones((n * len(cams), 3), device="cuda")
    g.backward(cams, 1, 1, d, seed, B.ST_EDGE_SHADOW, 1.0, debug_edge_hash=h)
    g.check_errors()
    h = h.cpu().numpy().view(np.uint32)[n * len(cams):].reshape(len(cams), LIGHTS, n)
    # a sample's decisions: its edge, and that the ray past it meets nothing
    edge_of = {_fnv(e, 0xFFFFFFFF): e for e in range(len(edges))}
    drawn = np.array([edge_of[x] for x in h.ravel().tolist()])
    assert outline[drawn].all(), np.flatnonzero(~outline[drawn])
    # the sample at 1/2: the edges of the outline on both sides of it, by the rounding of 1/2
    half = len(edges) // 2
    assert outline[:half].sum() == outline[half:].sum()
    assert edge_of[int(h[view, light, n // 2])] in (np.flatnonzero(outline[:half])[-1], half)

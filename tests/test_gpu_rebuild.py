"""The scene rebuild at the sizes where its tiles and blocks can go wrong: the
radix sort's tiles of 1,024 keys (and the path of more than 512 of them), blocks of
leaves, and the edge CDF's tiles, all against the oracle's tree or a host sum."""
import sys

import numpy as np
import pytest

torch = pytest.importorskip("torch")

import oracle as O
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


@pytest.mark.parametrize("nf", [2, 6, 7, 8, 127, 128, 129, 511, 513, 1023, 1024, 1025, 2049, 9000])
def test_tree_bit_exact(B, nf):
    _say(f"case rebuild: {nf} faces against the oracle's tree")
    rng = np.random.default_rng(nf)
    V, F = S.noise_sphere(22, 0.2, noise_seed=5)
    F = F[rng.permutation(F.shape[0])[:nf]]
    V = V.astype(np.float32)
    g = B.GPUScene(V, F, S.random_materials(nf, rng))
    for got, want in zip(g.lbvh(), O.lbvh(V, F, treelet_rounds=O.TREELET_ROUNDS)):
        got = got.cpu().numpy()
        want = want.view(got.dtype)
        assert np.array_equal(got.reshape(-1).view(np.uint8), want.reshape(-1).view(np.uint8))
    g.check_errors()


@pytest.mark.parametrize("nf", [511 * 1024 + 3, 512 * 1024, 512 * 1024 + 1, 700001])
def test_sort_of_many_tiles(B, nf):
    """Keys sorted and complete around the tile count at which the counts are scanned apart."""
    _say(f"case rebuild: keys of {nf} faces")
    rng = np.random.default_rng(3)
    V = rng.uniform(-1, 1, (3 * nf, 3)).astype(np.float32)
    F = np.arange(3 * nf, dtype=np.int32).reshape(nf, 3)
    g = B.GPUScene(V, F, S.uniform_materials(nf))
    keys = g.lbvh()[0].cpu().numpy().view(np.uint64)
    assert np.all(keys[1:] > keys[:-1])
    assert np.array_equal(np.sort((keys & 0xFFFFFFFF).astype(np.int64)), np.arange(nf))
    g.check_errors()


@pytest.mark.parametrize("nf", [31, 32, 33, 65, 65536, 65537, 131072, 131073, 131137])
def test_tree_bit_exact_at_wave_shares(B, nf):
    """Around the leaf counts of a block and those at which a wave starts from more leaves."""
    _say(f"case rebuild: {nf} faces against the oracle's tree, wave shares")
    V, F = S.noise_sphere(82, 0.2, noise_seed=6)
    F = F[np.random.default_rng(nf).permutation(F.shape[0])[:nf]]
    V = V.astype(np.float32)
    g = B.GPUScene(V, F, S.uniform_materials(nf))
    for got, want in zip(g.lbvh(), O.lbvh(V, F, treelet_rounds=O.TREELET_ROUNDS)):
        got = got.cpu().numpy()
        want = want.view(got.dtype)
        assert np.array_equal(got.reshape(-1).view(np.uint8), want.reshape(-1).view(np.uint8))
    g.check_errors()

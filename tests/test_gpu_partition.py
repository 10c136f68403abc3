"""Large batches go through hash bins (split by hash, then worked on bin by
bin in LDS).  Checked against the oracle, bit for bit, at the sizes where that
path starts and where its ranges, tiles and bins have remainders, and on keys
that strain it: one key throughout, a few keys throughout, and more distinct
keys in one bin than its LDS table holds."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

import synth  # noqa: E402
from tests.test_gpu_parity import check_voxelize  # noqa: E402

VOXEL_MIN = 1 << 18  # points from which a voxelization goes by bins
TILE = 4096          # positions whose copies are dropped together
M64 = (1 << 64) - 1


@pytest.fixture(scope="module")
def ash():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2110_00511_amd as ash_mod
    return ash_mod


def mix64(z):
    z = (z ^ (z >> np.uint64(30))) * np.uint64(0xbf58476d1ce4e5b9)
    z = (z ^ (z >> np.uint64(27))) * np.uint64(0x94d049bb133111eb)
    return z ^ (z >> np.uint64(31))


def key_hash3(k):
    """The hash of int32x3 keys (SplitMix64's output function over the key words)."""
    w = k.astype(np.uint32).astype(np.uint64)
    h = np.full(len(k), (0x9e3779b97f4a7c15 * 3) & M64, np.uint64)
    h = mix64(h ^ (w[:, 0] | (w[:, 1] << np.uint64(32))))
    return mix64(h ^ w[:, 2])


def keys_of_bin(nbins, count, seed=0):
    """`count` distinct int32x3 keys whose hashes all lie in bin 0 of nbins."""
    rng = np.random.default_rng(seed)
    out = []
    have = 0
    while have < count:
        k = rng.integers(-(1 << 20), 1 << 20, size=(1 << 20, 3), dtype=np.int32)
        k = k[((key_hash3(k) >> np.uint64(32)) * np.uint64(nbins)) >> np.uint64(32) == 0]
        out.append(k)
        have += len(k)
    k = np.unique(np.concatenate(out), axis=0)
    assert len(k) >= count
    return k[rng.permutation(len(k))[:count]]


def test_key_hash_is_the_librarys_shape():
    """keys_of_bin fills one bin of 256 and no other (CPU)."""
    k = keys_of_bin(256, 2000)
    assert len(np.unique(k, axis=0)) == 2000
    assert int((key_hash3(k) >> np.uint64(56)).max()) == 0  # 256 bins: the leading 8 bits


@pytest.mark.gpu
@pytest.mark.parametrize("n", [VOXEL_MIN - 1, VOXEL_MIN, VOXEL_MIN + 1, 70 * TILE - 1, 70 * TILE + 63, 1_000_003])
def test_voxelize_at_the_edges_of_its_ranges(ash, n):
    check_voxelize(ash, synth.points(n=n, seed=41), 0.02)


@pytest.mark.gpu
@pytest.mark.parametrize("n,cells", [(VOXEL_MIN, 1), (2_200_000, 1), (2_200_000, 3), (600_000, 700)])
def test_voxelize_few_voxels(ash, n, cells):
    """Few voxels throughout: copies are dropped tile by tile, and a voxel's
    copies in a tile may need several entries."""
    rng = np.random.default_rng(n + cells)
    pts = np.zeros((n, 3), np.float32)
    pts[:, 0] = rng.integers(0, cells, size=n) + 0.5
    pts[rng.integers(0, n, size=7)] = [np.nan, 0.0, np.inf]
    check_voxelize(ash, pts, 1.0)


@pytest.mark.gpu
def test_voxelize_a_bin_fuller_than_its_table(ash):
    """9,500 distinct voxels in one of 256 bins, whose table has 8,192 entries:
    the rest are settled by comparison."""
    rng = np.random.default_rng(3)
    keys = keys_of_bin(256, 9500)
    pick = np.concatenate([np.arange(len(keys)), rng.integers(0, len(keys), size=4000)])
    pts = (keys[pick] + np.float32(0.5)).astype(np.float32)
    rest = rng.integers(-500, 500, size=(VOXEL_MIN, 3)).astype(np.float32) + np.float32(0.5)
    pts = np.concatenate([pts, rest])[rng.permutation(len(pick) + len(rest))]
    check_voxelize(ash, np.ascontiguousarray(pts), 1.0)

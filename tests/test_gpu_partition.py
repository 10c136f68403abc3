"""Large batches go through hash bins (split by hash, then worked on bin by
bin in LDS).  Checked against the oracle, bit for bit, at the sizes where that
path starts and where its ranges, tiles and bins have remainders, and on keys
that strain it: one key throughout, a few keys throughout, and more distinct
keys in one bin than its LDS table holds."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

import synth  # noqa: E402
from tests.test_gpu_parity import Pair, check_voxelize  # noqa: E402

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


INSERT_MIN = 5 << 19  # positions from which an insert goes by bins


def draw(rng, n, key_dim, cells):
    side = max(2, int(round(cells ** (1.0 / key_dim))))
    return rng.integers(-(side // 2), side - side // 2, size=(n, key_dim), dtype=np.int32)


class BinsPair(Pair):
    """Inserts must have gone by bins (the label of their claim)."""

    def __init__(self, *args, **kw):
        super().__init__(*args, **kw)
        self.gpu.profile(True)

    def insert(self, keys, values, by_bins=True):
        self.gpu.profile_collect()
        super().insert(keys, values)
        assert ("claim_bins" in self.gpu.profile_collect()) == by_bins


@pytest.mark.gpu
@pytest.mark.parametrize("key_dim,elems,shape,n", [
    (1, 1, (4, 4, 0.5), INSERT_MIN), (2, 3, (2, 1, 0.85), INSERT_MIN + 1), (3, 8, (2, 1, 0.85), INSERT_MIN + 4095),
    (3, 32, (16, 16, 0.9), INSERT_MIN + 65), (4, 0, (8, 8, 0.7), INSERT_MIN + 100_001)])
def test_insert_by_bins(ash, key_dim, elems, shape, n):
    """Into an empty table, then the general path over what that left: among
    its keys and over tombstones."""
    rng = np.random.default_rng(1000 * key_dim + elems)
    w, g, load = shape
    specs = [(np.float32, elems)] if elems else []
    pair = BinsPair(ash, int(1.4 * n), key_dim, specs, probe_group=g, bucket_width=w, max_load=load)

    def rows(m):
        return [rng.standard_normal((m, elems)).astype(np.float32)] if elems else []

    keys = draw(rng, n, key_dim, 0.8 * n)
    if key_dim == 4:  # goes by bins only after an insert of which most was new
        pair.insert(np.arange(400, dtype=np.int32).reshape(100, 4), rows(100), by_bins=False)
        pair.gpu.clear()
        pair.orc = type(pair.orc)(int(1.4 * n), key_dim, specs)
    pair.insert(keys, rows(n))
    pair.check_state()
    pair.find(keys[: n // 8])
    pair.erase(keys[rng.permutation(n)[: n // 4]])
    more = draw(rng, n // 4, key_dim, 0.8 * n)
    pair.insert(more, rows(len(more)), by_bins=False)
    pair.check_state()
    pair.find(more)


@pytest.mark.gpu
def test_insert_by_bins_overflows(ash):
    """More new keys than indices: nothing changes, and the map goes on."""
    rng = np.random.default_rng(4)
    n = INSERT_MIN + 3
    pair = BinsPair(ash, n // 2, 3, [(np.float32, 1)], max_load=0.9)
    far = rng.integers(-(1 << 20), 1 << 20, size=(n, 3), dtype=np.int32)
    pair.insert(far, [rng.standard_normal((n, 1)).astype(np.float32)])
    pair.check_state()
    keys = draw(rng, n, 3, n // 3)
    pair.insert(keys, [rng.standard_normal((n, 1)).astype(np.float32)], by_bins=False)  # (no new key last time)
    pair.check_state()


@pytest.mark.gpu
def test_insert_by_bins_few_keys(ash):
    """Three keys throughout, and one more at the very end."""
    rng = np.random.default_rng(5)
    n = INSERT_MIN + 17
    keys = rng.integers(0, 3, size=(n, 1), dtype=np.int32) * np.array([[1, 7, -3]], np.int32)
    keys[-1] = [5, 5, 5]
    pair = BinsPair(ash, n, 3, [(np.float32, 1)])
    pair.insert(keys, [np.arange(n, dtype=np.float32)[:, None]])
    pair.check_state()
    pair.find(keys[-1000:])


@pytest.mark.gpu
@pytest.mark.parametrize("shape", [(2, 1, 0.85), (4, 4, 0.5)])
def test_insert_by_bins_one_part_of_the_table(ash, shape):
    """30,000 keys whose homes lie in a 512th of the table, more than a bin's
    LDS table holds and more than that part has slots: the rest are settled
    by comparison and stored in the slots after it."""
    rng = np.random.default_rng(6)
    w, g, load = shape
    crowd = keys_of_bin(512, 30_000, seed=1)
    crowd = crowd[np.concatenate([np.arange(len(crowd)), rng.integers(0, len(crowd), size=9_000)])]
    rest = rng.integers(0, 130, size=(INSERT_MIN, 3), dtype=np.int32)
    keys = np.concatenate([crowd, rest])[rng.permutation(len(crowd) + len(rest))]
    pair = BinsPair(ash, len(keys), 3, [(np.float32, 2)], probe_group=g, bucket_width=w, max_load=load)
    pair.insert(keys, [rng.standard_normal((len(keys), 2)).astype(np.float32)])
    pair.check_state()
    pair.find(crowd)
    pair.find(keys[:100_000])


@pytest.mark.gpu
@pytest.mark.parametrize("key_dim", [1, 2, 3, 4])
def test_insert_by_bins_replayed_from_a_graph(ash, key_dim):
    """An insert captured on an empty map, replayed on an empty one, on one
    that holds keys, on one with tombstones and on one without enough room,
    gives what the general path gives."""
    rng = np.random.default_rng(8 + key_dim)
    n = INSERT_MIN + 5
    cap = int(1.75 * n)

    def batch(cells, shift=0):
        k = draw(rng, n, key_dim, cells) + np.int32(shift)
        return torch.from_numpy(k).cuda(), torch.randn((n, 2), device="cuda")

    batches = [batch(0.8 * n), batch(1.6 * n), batch(1.2 * n, 1 << 20), batch(5 * n, 1 << 21)]
    gone = batches[1][0][:700_001].contiguous()
    eager = ash.HashMap(cap, key_dim, [(torch.float32, 2)])  # inserts in parts too small for the bins
    m = ash.HashMap(cap, key_dim, [(torch.float32, 2)])
    m.insert(torch.arange(key_dim * 64, dtype=torch.int32, device="cuda").view(-1, key_dim),
             [torch.zeros((64, 2), device="cuda")])  # all new: the next one of any width goes by bins
    m.clear()
    m.insert(*[batches[0][0], [batches[0][1]]])  # the workspace is allocated before the capture
    m.clear()
    m.insert(torch.arange(key_dim * 64, dtype=torch.int32, device="cuda").view(-1, key_dim),
             [torch.zeros((64, 2), device="cuda")])
    m.clear()
    torch.cuda.synchronize()
    keys, vals = batches[0][0].clone(), batches[0][1].clone()
    graph = torch.cuda.CUDAGraph()
    m.profile_collect()
    with torch.cuda.graph(graph):
        idx, mask = m.insert(keys, [vals])
    for _ in range(2):
        m.clear()
        eager.clear()
        for j, (k, v) in enumerate(batches):
            keys.copy_(k)
            vals.copy_(v)
            before = eager.size()
            graph.replay()
            torch.cuda.synchronize()
            if j < 3:
                got = [eager.insert(kk, [vv]) for kk, vv in zip(k.split(500_000), v.split(500_000))]
                assert torch.equal(idx, torch.cat([g[0] for g in got]))
                assert torch.equal(mask, torch.cat([g[1] for g in got]))
                assert m.device_status() == 0
            else:  # more new keys than indices
                assert bool((idx == -1).all()) and not bool(mask.any())
                assert m.device_status() == 2 and m.size() == before
            assert m.size() == eager.size()
            if j == 1:
                assert torch.equal(m.erase(gone), eager.erase(gone))
        live = eager.active_indices().long()
        assert torch.equal(m.active_indices().long(), live)
        assert torch.equal(m.key_buffer()[live], eager.key_buffer()[live])
        assert torch.equal(m.value_buffer()[live], eager.value_buffer()[live])
        assert torch.equal(m.heap_buffer(), eager.heap_buffer())

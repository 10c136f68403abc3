"""Large batches at the upper limits of the path by hash bins, just above them,
and where its kernels change over on the way: 1536 bins and more (the second
loop that collects the new keys), more than 2015 bins at key width 3 (the
scatter's smaller tiles), ranges of 65536 positions.  Against the oracle, bit
for bit."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu

from oracle import OracleMap, oracle_voxelize  # noqa: E402
from tests.test_gpu_partition import INSERT_MIN, BinsPair, key_hash3, keys_of_bin  # noqa: E402

INSERT_MOST = 256 * 65536  # positions up to which an insert goes by bins
VOXEL_MOST = 4096 * 3840   # points up to which a voxelization does


@pytest.fixture(scope="module")
def ash():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2110_00511_amd as ash_mod
    return ash_mod


def cells(seed, n, side):
    return np.random.default_rng(seed).integers(0, side, size=(n, 3), dtype=np.int32)


def test_key_hash_is_the_librarys(ash):
    """The hash that these tests fill bins by is the one that places keys: every
    key is stored in its home bucket, or after it with no EMPTY slot between."""
    m = ash.HashSet(4000, 3, bucket_width=4, probe_group=4, max_load=0.5)
    keys = torch.from_numpy(np.random.default_rng(0).integers(-(1 << 31), 1 << 31, size=(1500, 3), dtype=np.int64)
                            .astype(np.int32)).cuda()
    m.activate(keys)
    slots = m.stats()["slots"]
    table, = [t for t in m._alloc.blocks.values() if t.numel() == 16 * slots]
    words = table.cpu().numpy().view(np.uint32).reshape(slots, 4)
    at = np.nonzero(words[:, 3] < 0x80000000)[0]
    assert len(at) == 1500
    home = ((key_hash3(words[at, :3].view(np.int32)) >> np.uint64(32)) * np.uint64(slots // 4) >> np.uint64(32)) * 4
    away = (at - home.astype(np.int64)) % slots
    assert (away < 4).mean() > 0.8 and away.max() < 40
    for p, a in zip(at, away):
        assert (words[[(p - d) % slots for d in range(a + 1)], 3] != 0xFFFFFFFF).all()


def test_insert_of_the_most_positions(ash):
    """The most positions that go by bins (2410 of them, ranges of 65536), and one more."""
    n = INSERT_MOST
    keys = cells(1, n + 1, 190)
    orc = OracleMap(n // 2, 3)
    _, idx, mask = orc.activate(keys)  # in batch order: the first n positions do not depend on the last
    m = ash.HashSet(n // 2, 3, bucket_width=2, probe_group=1, max_load=0.85)
    m.profile()
    k = torch.from_numpy(keys).cuda()
    for count, by_bins in ((n, True), (n + 1, False)):
        m.clear()
        m.profile_collect()
        gi, gm = m.activate(k[:count])
        assert ("claim_bins" in m.profile_collect()) == by_bins
        assert np.array_equal(gi.cpu().numpy(), idx[:count])
        assert np.array_equal(gm.cpu().numpy(), mask[:count].astype(bool))
        assert m.device_status() == 0
        fi, fm = m.find(k[:count])  # every key is where its first position put it
        assert bool(fm.all()) and torch.equal(m.key_buffer()[fi.long()], k[:count])
    m.close()


def test_insert_by_1744_bins(ash):
    """The ten-million-key step's size on the shape W = 4, g = 4, load 0.7."""
    n = 10_000_003
    keys = cells(2, n, 190)
    orc = OracleMap(n, 3)
    _, idx, mask = orc.activate(keys)
    m = ash.HashSet(n, 3, max_load=0.7)
    m.profile()
    k = torch.from_numpy(keys).cuda()
    gi, gm = m.activate(k)
    assert "claim_bins" in m.profile_collect()
    assert np.array_equal(gi.cpu().numpy(), idx) and np.array_equal(gm.cpu().numpy(), mask.astype(bool))
    fi, fm = m.find(k)
    assert bool(fm.all()) and torch.equal(m.key_buffer()[fi.long()], k)
    m.close()


@pytest.mark.parametrize("specs", [[(np.uint8, 3), (np.float16, 1), (np.float32, 2)], [(np.uint8, 1), (np.int64, 9)]])
def test_insert_by_bins_of_several_rows(ash, specs):
    """Several value buffers, rows of 1, 2 and 3 bytes, copied in the commit or
    (80 bytes together) in a pass of their own."""
    rng = np.random.default_rng(5)
    n = INSERT_MIN + 4097
    pair = BinsPair(ash, n, 3, specs)
    rows = [rng.integers(0, 100, size=(n, e)).astype(dt) for dt, e in specs]
    pair.insert(cells(6, n, 120), rows)
    pair.check_state()
    pair.find(cells(7, n // 16, 130))


def test_voxelize_the_most_points(ash):
    """The most points that go by bins (4096 of them), and one more."""
    n = VOXEL_MOST
    rng = np.random.default_rng(8)
    pts = rng.uniform(-8, 8, size=(n + 1, 3)).astype(np.float32)
    pts[rng.integers(0, n, size=9)] = np.nan
    pts[-1] = [100.0, 100.0, 100.0]  # a voxel of its own
    pv, vk, cnt = oracle_voxelize(pts, 0.1)
    p = torch.from_numpy(pts).cuda()
    for count, u in ((n, len(vk) - 1), (n + 1, len(vk))):
        gpv, gvk, gcnt = ash.voxelize(p[:count], 0.1)
        assert np.array_equal(gpv.cpu().numpy(), pv[:count])
        assert np.array_equal(gvk.cpu().numpy(), vk[:u])
        assert np.array_equal(gcnt.cpu().numpy(), cnt[:u])


def test_a_crowded_bin_replayed_on_a_filled_map(ash):
    """A captured insert with 30,000 keys of one bin, replayed on a map that
    holds a third of them: entries beyond the bin's LDS table are looked up in
    the table one by one."""
    rng = np.random.default_rng(9)
    crowd = keys_of_bin(512, 30_000, seed=2)
    n = INSERT_MIN + 30_001
    keys = np.concatenate([crowd, rng.integers(0, 130, size=(n - len(crowd), 3), dtype=np.int32)])[rng.permutation(n)]
    held = np.concatenate([crowd[::3], rng.integers(100, 140, size=(50_000, 3), dtype=np.int32)])
    k, h = torch.from_numpy(keys).cuda(), torch.from_numpy(held).cuda()
    m, eager = (ash.HashSet(n, 3, bucket_width=2, probe_group=1, max_load=0.85) for _ in range(2))
    m.profile()
    m.activate(k)  # (the workspace)
    assert "claim_bins" in m.profile_collect()
    m.profile(False)
    m.clear()
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        idx, mask = m.activate(k)
    for first in (h, h[:7], h[20_000:]):
        for x in (m, eager):
            x.clear()
            x.activate(first)
        graph.replay()
        got = [eager.activate(part) for part in k.split(500_000)]
        assert torch.equal(idx, torch.cat([g[0] for g in got])) and torch.equal(mask, torch.cat([g[1] for g in got]))
        assert m.device_status() == 0 and m.size() == eager.size()
        fi, fm = m.find(k)
        assert bool(fm.all()) and torch.equal(fi, eager.find(k)[0])

"""Small batches run as one block where the table is not crowded for them, and
in the general kernels where it is; both against the oracle, bit for bit.
Captured ones are one block on any table, and their replays are checked."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu

from tests.test_gpu_parity import Pair  # noqa: E402


@pytest.fixture(scope="module")
def ash():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2110_00511_amd as ash_mod
    return ash_mod


def labels(pair, call):
    pair.gpu.profile_collect()
    call()
    return set(pair.gpu.profile_collect())


def distinct(lo, n):
    """Distinct keys: row i of the range [lo, lo + n)."""
    i = np.arange(lo, lo + n, dtype=np.int64)
    return np.stack([i % 31, i // 31, i * 7 % 13], axis=1).astype(np.int32)


@pytest.mark.parametrize("w,g", [(2, 1), (4, 1), (8, 1), (4, 4), (16, 16), (64, 64)])
def test_crowded_tables_take_the_general_kernels(ash, w, g):
    """A table that fills up to 0.85 of its slots: 100 keys and 2000, into
    the nearly empty table and into the full one."""
    rng = np.random.default_rng(w + g)
    c = 60_000
    pair = Pair(ash, c, 3, [(np.float32, 1)], probe_group=g, bucket_width=w, max_load=0.9)
    pair.gpu.profile()
    at = 0
    for upto, small, large in ((1_000, True, g == 1 and w == 2), (c - 3_000, g == 1, False)):
        pair.insert(distinct(at, upto - at), [np.ones((upto - at, 1), np.float32)])
        for n, one in ((100, small), (2000, False)):
            keys = np.concatenate([distinct(upto, n - n // 4), distinct(upto // 2, n // 4)])[rng.permutation(n)]
            vals = [rng.standard_normal((n, 1)).astype(np.float32)]
            got = labels(pair, lambda: pair.insert(keys, vals))
            assert ("insert_small" in got) == one, (upto, n, got)
            pair.check_state()
            got = labels(pair, lambda: pair.erase(distinct(upto, n)))
            assert ("erase_small" in got) == one, (upto, n, got)
            pair.check_state()
        at = upto


def test_a_loaded_map_knows_how_full_it_is(ash, tmp_path):
    """The first small call on a loaded, crowded map takes the general kernels."""
    c = 60_000
    m = ash.HashSet(c, 3, probe_group=16, bucket_width=16, max_load=0.9)
    m.activate(torch.from_numpy(distinct(0, c - 3_000)).cuda())
    m.save(str(tmp_path / "m.ash"))
    m = ash.HashMap.load(str(tmp_path / "m.ash"), probe_group=16, bucket_width=16, max_load=0.9)
    m.profile()
    mask = m.erase(torch.from_numpy(distinct(c - 3_100, 200)).cuda())
    assert mask.sum().item() == 100
    assert "erase_small" not in m.profile_collect()


@pytest.mark.parametrize("n", [300, 2048])
@pytest.mark.parametrize("fill", [0, 20_000, 55_000])
def test_captured_small_batches(ash, n, fill):
    """An insert and an erase of n positions, captured together, replayed on
    changing keys with eager work between, against the same calls on a second
    map in parts that a crowded table sends to the general kernels."""
    rng = np.random.default_rng(n + fill)
    c = 60_000
    specs = [(torch.float32, 3)]
    m = ash.HashMap(c, 3, specs, max_load=0.9)
    eager = ash.HashMap(c, 3, specs, max_load=0.9)
    for x in (m, eager):
        x.insert(torch.from_numpy(distinct(0, fill)).cuda(), [torch.ones((fill, 3), device="cuda")])
        x.erase(torch.from_numpy(distinct(100_000, n)).cuda())  # (scratch of the batch's size)
    keys = torch.zeros((n, 3), dtype=torch.int32, device="cuda")
    gone = torch.zeros((n, 3), dtype=torch.int32, device="cuda")
    vals = torch.zeros((n, 3), device="cuda")
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        idx, mask = m.insert(keys, [vals])
        emask = m.erase(gone)
    for step in range(5):
        pool = np.concatenate([distinct(0, fill), distinct(70_000 + 500 * step, n)])
        k = torch.from_numpy(pool[rng.integers(0, len(pool), size=n)]).cuda()
        g = torch.from_numpy(pool[rng.integers(0, len(pool), size=n)]).cuda()
        keys.copy_(k)
        gone.copy_(torch.cat([g[: n // 2], k[: n - n // 2]]))
        vals.normal_()
        graph.replay()
        got = eager.insert(keys, [vals])
        assert torch.equal(idx, got[0]) and torch.equal(mask, got[1])
        assert torch.equal(emask, eager.erase(gone))
        assert m.size() == eager.size()
        live = eager.active_indices().long()
        assert torch.equal(m.active_indices().long(), live)
        assert torch.equal(m.key_buffer()[live], eager.key_buffer()[live])
        assert torch.equal(m.value_buffer()[live], eager.value_buffer()[live])
        assert torch.equal(m.heap_buffer(), eager.heap_buffer())
        assert m.device_status() == 0
        if step == 2:  # eager calls over what the replays left
            for x in (m, eager):
                x.erase(k)
                x.insert(g, [vals])

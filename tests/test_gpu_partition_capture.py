"""Large inserts under stream capture: what a captured insert may allocate, and
what it goes on using.  Replays are checked against the general path in eager
calls, several times, with eager work between."""
import ctypes

import numpy as np
import pytest

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu

INSERT_MIN = 5 << 19  # positions from which an insert may go by bins


@pytest.fixture(scope="module")
def ash():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2110_00511_amd as ash_mod
    return ash_mod


def draw(seed, n, key_dim, cells):
    side = max(2, int(round(cells ** (1.0 / key_dim))))
    k = np.random.default_rng(seed).integers(0, side, size=(n, key_dim), dtype=np.int32)
    return torch.from_numpy(k).cuda()


def in_parts(m, keys):
    """(idx, mask) of an insert of keys by parts too small for the bins."""
    got = [m.activate(k) for k in keys.split(500_000)]
    return torch.cat([g[0] for g in got]), torch.cat([g[1] for g in got])


def test_a_size_that_has_run_can_be_captured(ash):
    """On the default allocator an insert of a size that has run before (here by
    the general path, as the map's first insert of key width 4) allocates
    nothing, whichever path the next one prefers."""
    from paper_2110_00511_amd import _lib as L
    lib = L.load()
    n, key_dim = INSERT_MIN + 9, 4
    keys = draw(1, n, key_dim, 8 * n)
    other = draw(2, n, key_dim, 8 * n)
    idx = torch.empty(n, dtype=torch.int32, device="cuda")
    mask = torch.empty(n, dtype=torch.bool, device="cuda")
    h = ctypes.c_void_p()

    def stream():
        return ctypes.c_void_p(torch.cuda.current_stream().cuda_stream)

    L.check(lib.ash_create(n, key_dim, 0, None, None, None, None, stream(), ctypes.byref(h)), "ash_create")
    try:
        def activate():
            return lib.ash_activate(h, keys.data_ptr(), n, idx.data_ptr(), mask.data_ptr(), stream())

        L.check(activate(), "ash_activate")
        L.check(lib.ash_clear(h, stream()), "ash_clear")
        torch.cuda.synchronize()
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph):
            status = activate()
        assert status == 0
        eager = ash.HashSet(n, key_dim)
        for k in (keys.clone(), other, keys.clone()):
            keys.copy_(k)
            L.check(lib.ash_clear(h, stream()), "ash_clear")
            graph.replay()
            eager.clear()
            want = in_parts(eager, k)
            assert torch.equal(idx, want[0]) and torch.equal(mask, want[1])
            assert lib.ash_device_status(h, stream()) == 0
        # replayed on a map that has no room for its keys: refused, the map as it was
        size = ctypes.c_int64()
        L.check(lib.ash_clear(h, stream()), "ash_clear")
        L.check(lib.ash_activate(h, other.data_ptr(), n, None, None, stream()), "ash_activate")
        L.check(lib.ash_size(h, ctypes.byref(size), stream()), "ash_size")
        before = size.value
        graph.replay()
        assert bool((idx == -1).all()) and not bool(mask.any())
        assert lib.ash_device_status(h, stream()) == 2
        L.check(lib.ash_size(h, ctypes.byref(size), stream()), "ash_size")
        assert size.value == before > n // 2
        del graph
    finally:
        torch.cuda.synchronize()
        L.check(lib.ash_destroy(h), "ash_destroy")


def test_a_graph_keeps_its_workspace(ash):
    """A captured insert goes on using its workspace after a larger eager insert
    has taken one of its own (the map's other scratch is large enough for both
    from the start, so a graph on it stays valid)."""
    n, big = INSERT_MIN + 11, 2 * INSERT_MIN
    m = ash.HashSet(big, 3)
    m.erase(draw(3, big, 3, 100))  # scratch for the larger batch
    small, large = draw(4, n, 3, 6 * n), draw(5, big, 3, 6 * big)
    m.activate(small)
    m.clear()
    torch.cuda.synchronize()
    held = dict(m._alloc.blocks)
    keys = small.clone()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        idx, mask = m.activate(keys)
    m.profile()
    eager = ash.HashSet(big, 3)
    for seed in (6, 7):
        m.clear()
        m.profile_collect()
        got = m.activate(large)
        assert "claim_bins" in m.profile_collect()
        eager.clear()
        want = in_parts(eager, large)
        assert torch.equal(got[0], want[0]) and torch.equal(got[1], want[1])
        gone = [p for p in held if p not in m._alloc.blocks]
        assert not gone, "a block that the graph may use went back to the allocator"
        keys.copy_(draw(seed, n, 3, 6 * n))
        m.clear()
        graph.replay()
        eager.clear()
        want = in_parts(eager, keys)
        assert torch.equal(idx, want[0]) and torch.equal(mask, want[1])
        assert m.device_status() == 0
    m.close()
    assert not m._alloc.blocks


def test_width_4_replayed(ash):
    """An insert of key width 4 by bins, captured on an empty map and replayed on
    an empty one, on one that holds keys, over tombstones and without enough
    room, gives what the general path gives."""
    n, key_dim = INSERT_MIN + 5, 4
    cap = int(1.75 * n)
    batches = [draw(10, n, key_dim, 0.8 * n), draw(11, n, key_dim, 1.6 * n),
               draw(12, n, key_dim, 1.2 * n) + (1 << 20), draw(13, n, key_dim, 5 * n) + (1 << 21)]
    gone = batches[1][:700_001].contiguous()
    eager = ash.HashSet(cap, key_dim)
    m = ash.HashSet(cap, key_dim)
    first = torch.arange(n, dtype=torch.int32, device="cuda")[:, None].repeat(1, key_dim)
    m.activate(first)  # all new, of the batch's size: the next one goes by bins
    torch.cuda.synchronize()  # (once the host can read its outcome)
    m.profile()
    m.clear()
    m.activate(first)
    assert "claim_bins" in m.profile_collect()
    m.profile(False)
    m.clear()
    torch.cuda.synchronize()
    keys = batches[0].clone()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        idx, mask = m.activate(keys)
    for _ in range(2):
        m.clear()
        eager.clear()
        for j, k in enumerate(batches):
            keys.copy_(k)
            before = eager.size()
            graph.replay()
            torch.cuda.synchronize()
            if j < 3:
                want = in_parts(eager, k)
                assert torch.equal(idx, want[0]) and torch.equal(mask, want[1])
                assert m.device_status() == 0
            else:
                assert bool((idx == -1).all()) and not bool(mask.any())
                assert m.device_status() == 2 and m.size() == before
            assert m.size() == eager.size()
            if j == 1:
                assert torch.equal(m.erase(gone), eager.erase(gone))
        live = eager.active_indices().long()
        assert torch.equal(m.active_indices().long(), live)
        assert torch.equal(m.key_buffer()[live], eager.key_buffer()[live])
        assert torch.equal(m.heap_buffer(), eager.heap_buffer())


@pytest.mark.parametrize("small", [False, True])
def test_the_bound_on_used_slots_does_not_wrap(ash, small):
    """Replays raise the bound on the slots in use by every new key and never
    lower it; past 2^32 it must not read as an empty table, whose parts an
    insert by bins writes whole."""
    n = INSERT_MIN + 13
    m = ash.HashSet(2 * n, 3)
    a, b = draw(20, n, 3, 0.5 * n), draw(21, n, 3, 0.5 * n) + 5000
    few = draw(22, 1000, 3, 10_000) + 100_000
    m.activate(a)  # (the workspace)
    new_a = m.size()
    m.clear()
    new_few = len(torch.unique(few, dim=0))
    torch.cuda.synchronize()
    keys = a.clone()
    graph, graph_few = torch.cuda.CUDAGraph(), torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        m.activate(keys)
    with torch.cuda.graph(graph_few):
        m.activate(few)
    live = draw(23, 3000, 3, 100_000) + 200_000
    m.clear()
    m.activate(live)
    t = m.size()
    meta, = [w for w in (v.view(torch.int32) for v in m._alloc.blocks.values() if v.numel() == 256)
             if w[0].item() == t and w[2].item() == t]
    meta[2] = -(new_few if small else new_a)  # as after as many replays as it takes: 2^32 less the next one's new keys
    torch.cuda.synchronize()
    (graph_few if small else graph).replay()
    keys.copy_(b)
    graph.replay()
    for k in (live, b, few if small else a):
        assert bool(m.find(k)[1].all())
    assert m.device_status() == 0
    assert m.size() == len(torch.unique(torch.cat([live, b, few if small else a]), dim=0))

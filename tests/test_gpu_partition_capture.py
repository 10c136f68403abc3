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

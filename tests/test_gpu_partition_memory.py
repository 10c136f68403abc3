"""The workspace of large inserts: what a map does when it cannot have one, and
when memory is short while it holds one."""
import ctypes

import numpy as np
import pytest

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu

from oracle import OracleMap  # noqa: E402

INSERT_MIN = 5 << 19  # positions from which an insert may go by bins


@pytest.fixture(scope="module")
def ash():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2110_00511_amd as ash_mod
    return ash_mod


class Budget:
    """An allocator of at most `most` bytes in blocks of at most `largest`.  What
    is beyond that fails in the runtime, as an allocator on hipMalloc does, so
    the runtime's last error is set."""

    def __init__(self, L, most=1 << 62, largest=1 << 62):
        self.lib, self.most, self.largest = L.load(), most, largest
        self.blocks, self.refused = {}, 0
        self._alloc = L.AshAllocator._fields_[0][1](self.alloc)
        self._free = L.AshAllocator._fields_[1][1](self.free)
        self.struct = L.AshAllocator(self._alloc, self._free, None)

    def alloc(self, ctx, nbytes, stream):
        if nbytes > self.largest or nbytes + sum(t.numel() for t in self.blocks.values()) > self.most:
            self.refused += 1
            p = ctypes.c_void_p()
            assert self.lib.hipMalloc(ctypes.byref(p), ctypes.c_size_t(1 << 50)) != 0
            return None
        t = torch.empty(int(nbytes), dtype=torch.uint8, device="cuda")
        self.blocks[t.data_ptr()] = t
        return t.data_ptr()

    def free(self, ctx, ptr, stream):
        torch.cuda.synchronize()
        self.blocks.pop(ptr)


def stream():
    return ctypes.c_void_p(torch.cuda.current_stream().cuda_stream)


def create(L, capacity, key_dim, budget):
    h = ctypes.c_void_p()
    L.check(L.load().ash_create(capacity, key_dim, 0, None, None, ctypes.byref(budget.struct), None, stream(),
                                ctypes.byref(h)), "ash_create")
    return h


def activate(L, h, keys):
    n = keys.shape[0]
    idx = torch.empty(n, dtype=torch.int32, device="cuda")
    mask = torch.empty(n, dtype=torch.uint8, device="cuda")
    L.check(L.load().ash_activate(h, keys.data_ptr(), n, idx.data_ptr(), mask.data_ptr(), stream()), "ash_activate")
    return idx.cpu().numpy(), mask.cpu().numpy()


def test_no_workspace_to_be_had(ash):
    """An insert whose workspace is refused goes by the general path."""
    from paper_2110_00511_amd import _lib as L
    n = INSERT_MIN + 21
    keys = np.random.default_rng(1).integers(0, 100, size=(n, 3), dtype=np.int32)
    budget = Budget(L, largest=48 << 20)  # (the workspace takes 20 bytes per position)
    h = create(L, n // 2, 3, budget)
    try:
        got = activate(L, h, torch.from_numpy(keys).cuda())
        assert budget.refused == 1
        _, idx, mask = OracleMap(n // 2, 3).activate(keys)
        assert np.array_equal(got[0], idx) and np.array_equal(got[1], mask)
    finally:
        L.check(L.load().ash_destroy(h), "ash_destroy")
    assert not budget.blocks


def erase(L, h, keys):
    n = keys.shape[0]
    mask = torch.empty(n, dtype=torch.uint8, device="cuda")
    L.check(L.load().ash_erase(h, keys.data_ptr(), n, mask.data_ptr(), stream()), "ash_erase")
    return mask.cpu().numpy()


@pytest.mark.parametrize("call", ["erase", "rehash", "insert"])
def test_short_of_memory_beside_the_workspace(ash, call):
    """What fits beside a map without the workspace of its large inserts fits
    beside one that holds it: it goes back when memory is short."""
    from paper_2110_00511_amd import _lib as L
    n = INSERT_MIN + 21
    rng = np.random.default_rng(2)
    keys = rng.integers(0, 100, size=(n, 3), dtype=np.int32)
    budget = Budget(L)
    h = create(L, n // 2, 3, budget)
    try:
        orc = OracleMap(n // 2, 3)
        got = activate(L, h, torch.from_numpy(keys).cuda())
        _, idx, mask = orc.activate(keys)
        assert np.array_equal(got[0], idx) and np.array_equal(got[1], mask)
        held = max(budget.blocks.values(), key=torch.Tensor.numel).numel()
        assert held >= 20 * n  # the workspace, the largest block of all
        budget.most = sum(t.numel() for t in budget.blocks.values()) + n  # nearly all there is
        more = rng.integers(-50, 90, size=(2 * n, 3), dtype=np.int32)
        if call == "erase":
            assert np.array_equal(erase(L, h, torch.from_numpy(more).cuda()), orc.erase(more)[1])
        elif call == "insert":
            got = activate(L, h, torch.from_numpy(more).cuda())
            st, idx, mask = orc.activate(more)
            assert np.array_equal(got[0], idx) and np.array_equal(got[1], mask)
        else:
            L.check(L.load().ash_rehash(h, n // 2 + 1000, stream()), "ash_rehash")
        assert max(t.numel() for t in budget.blocks.values()) < held
        size = ctypes.c_int64()
        L.check(L.load().ash_size(h, ctypes.byref(size), stream()), "ash_size")
        assert size.value == orc.size
    finally:
        L.check(L.load().ash_destroy(h), "ash_destroy")
    assert not budget.blocks


def test_a_server_allocates_nothing_for_a_batch(ash):
    """A served insert that would go by bins, on an empty map and no larger than
    a full batch: the server's thread does not call the allocator."""
    n = INSERT_MIN + 5
    keys = np.random.default_rng(3).integers(0, 110, size=(n, 3), dtype=np.int32)
    m = ash.HashSet(n // 2, 3)
    srv = ash.Server(m)
    held = set(m._alloc.blocks)
    k = torch.from_numpy(keys).cuda()
    idx = torch.full((n,), -7, dtype=torch.int32, device="cuda")
    mask = torch.full((n,), 7, dtype=torch.uint8, device="cuda")
    r, keep = srv.request(srv.INSERT, k, out_idx=idx, out_mask=mask)
    _, status, _ = srv.replay([r], [0.0])
    assert status[0] == 0
    assert set(m._alloc.blocks) == held
    srv.close()
    orc = OracleMap(n // 2, 3)
    _, oi, om = orc.activate(keys)
    assert np.array_equal(idx.cpu().numpy(), oi) and np.array_equal(mask.cpu().numpy(), om)
    m.clear()
    assert torch.equal(m.activate(k)[0], idx)  # (no longer served: by bins)

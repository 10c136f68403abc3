"""Small and middling batches, whose kernels are spread over more blocks or run
as one, against the oracle, bit for bit, at the sizes where the split changes."""
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


@pytest.mark.parametrize("g,w", [(4, 4), (16, 16), (64, 64)])
@pytest.mark.parametrize("rounds,off", [(2, -1), (2, 1), (3, 0)])
def test_positions_per_block(ash, g, w, rounds, off):
    """256 / g positions at a time per block, and a block takes as many rounds
    as leave about 1024 blocks."""
    n = 256 // g * 1024 * rounds + off
    rng = np.random.default_rng(n)
    side = int(round((0.7 * n) ** (1 / 3)))
    pair = Pair(ash, int(0.95 * n), 3, [(np.float32, 2)], probe_group=g, bucket_width=w)  # (the capacity is checked)

    def batch(lo=0):
        return rng.integers(lo, lo + side, size=(n, 3), dtype=np.int32)

    keys = batch()
    pair.insert(keys, [rng.standard_normal((n, 2)).astype(np.float32)])
    pair.find(batch(side // 3))
    pair.erase(batch(side // 2))
    pair.insert(batch(side // 4)[: n // 2], [rng.standard_normal((n // 2, 2)).astype(np.float32)])
    pair.check_state()


@pytest.mark.parametrize("key_dim,elems,g,w", [(1, 0, 1, 2), (2, 1, 4, 4), (3, 3, 16, 16), (3, 32, 1, 8), (4, 2, 64, 64)])
@pytest.mark.parametrize("n", [1, 64, 65, 1023, 1024, 1025, 2048, 2049])
def test_batches_of_one_block(ash, key_dim, elems, g, w, n):
    """Up to 2048 positions run in one block, more in the general kernels: on a
    crowded table (load 0.9), over tombstones, with repeats in the batch and of
    the map's keys, and beyond the capacity."""
    rng = np.random.default_rng(100 * n + key_dim)
    specs = [(np.float32, elems)] if elems else []
    pair = Pair(ash, int(1.3 * n) + 4, key_dim, specs, probe_group=g, bucket_width=w, max_load=0.9)
    side = max(2, int(round((1.5 * n) ** (1 / key_dim))))

    def batch(m, lo=0):
        return rng.integers(lo, lo + side, size=(m, key_dim), dtype=np.int32)

    def rows(m):
        return [rng.standard_normal((m, elems)).astype(np.float32)] if elems else []

    for step in range(4):
        keys = batch(n, -step)
        pair.insert(keys, rows(n))
        pair.erase(np.concatenate([keys[: n // 2], keys[: n // 3], batch(n - n // 2 - n // 3)]))
        pair.check_state()
    far = batch(2 * n if n <= 1024 else n, 1 << 20)
    pair.insert(far, rows(len(far)))  # (one block or general) more new keys than there may be room for
    pair.find(np.concatenate([keys, far]))
    pair.check_state()
    pair.insert(np.repeat(keys[:1], n, axis=0), rows(n))
    pair.erase(np.repeat(keys[:1], n, axis=0))
    pair.check_state()


def test_one_block_batches_beside_large_ones(ash):
    """Erases by owner entries and by one block in turn, and claims over what both leave."""
    rng = np.random.default_rng(12)
    pair = Pair(ash, 40_000, 3, [(np.float32, 1)], probe_group=1, bucket_width=4)
    for _ in range(3):
        for n in (30_000, 700, 9_000, 2_000):
            k = rng.integers(0, 30, size=(n, 3), dtype=np.int32)
            pair.insert(k, [rng.standard_normal((n, 1)).astype(np.float32)])
            pair.erase(rng.integers(0, 30, size=(n // 2, 3), dtype=np.int32))
        pair.check_state()

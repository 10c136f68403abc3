"""Which inserts and erases leave the general kernels, and that the ones that
must not do not."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu

from tests.test_gpu_partition import BinsPair, INSERT_MIN  # noqa: E402


@pytest.fixture(scope="module")
def ash():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2110_00511_amd as ash_mod
    return ash_mod


@pytest.mark.parametrize("capacity,w,g", [(10, 4, 4), (10, 64, 64), (300, 2, 1), (600, 8, 1)])
def test_large_batch_into_a_tiny_map(ash, capacity, w, g):
    """More distinct keys than a tiny map holds: the general path reports the
    capacity error (the bins of such a table would be far too full)."""
    rng = np.random.default_rng(capacity)
    n = INSERT_MIN + 7
    keys = np.stack([rng.permutation(n), rng.integers(-5, 5, size=n), np.full(n, 3)], axis=1).astype(np.int32)
    pair = BinsPair(ash, capacity, 3, [(np.float32, 1)], probe_group=g, bucket_width=w)
    pair.insert(keys, [np.zeros((n, 1), np.float32)], by_bins=False)
    assert pair.gpu.device_status() == 2
    assert pair.gpu.size() == 0

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

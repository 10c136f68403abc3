"""Large batches of different sizes from two host threads at once, each on a
stream and a map of its own."""
import threading

import numpy as np
import pytest

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu

from oracle import OracleMap, oracle_voxelize  # noqa: E402

INSERT_MIN = 5 << 19  # positions from which an insert may go by bins


@pytest.fixture(scope="module")
def ash():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2110_00511_amd as ash_mod
    return ash_mod


def test_two_threads_with_batches_of_different_sizes(ash):
    rng = np.random.default_rng(9)
    clouds = [rng.uniform(0, 12, size=(n, 3)).astype(np.float32) for n in (300_000, 1_500_000)]
    batches = [rng.integers(0, side, size=(n, 3), dtype=np.int32) for n, side in ((INSERT_MIN + 1, 100),
                                                                                  (2 * INSERT_MIN, 160))]
    want = [(oracle_voxelize(c, 0.1), OracleMap(2 * INSERT_MIN, 3).activate(b)) for c, b in zip(clouds, batches)]
    got, errors = [[], []], []

    def work(i):
        try:
            with torch.cuda.stream(torch.cuda.Stream()):
                pts, keys = torch.from_numpy(clouds[i]).cuda(), torch.from_numpy(batches[i]).cuda()
                m = ash.HashSet(2 * INSERT_MIN, 3)
                for _ in range(4):
                    m.clear()
                    got[i].append((ash.voxelize(pts, 0.1), m.activate(keys)))
                torch.cuda.current_stream().synchronize()
        except Exception as e:  # reported by the test's own thread
            errors.append(e)

    threads = [threading.Thread(target=work, args=(i,)) for i in range(2)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    assert not errors, errors
    for i in range(2):
        (pv, vk, cnt), (_, idx, mask) = want[i]
        for (gpv, gvk, gcnt), (gi, gm) in got[i]:
            assert np.array_equal(gpv.cpu().numpy(), pv)
            assert np.array_equal(gvk.cpu().numpy(), vk)
            assert np.array_equal(gcnt.cpu().numpy(), cnt)
            assert np.array_equal(gi.cpu().numpy(), idx)
            assert np.array_equal(gm.cpu().numpy(), mask.astype(bool))

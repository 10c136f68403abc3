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


def spread(n, new, shift=0):
    """n keys in random order, the given share of them new."""
    rng = np.random.default_rng(int(100 * new) + shift)
    u = int(new * n)
    i = np.concatenate([np.arange(u), rng.integers(0, u, size=n - u)])[rng.permutation(n)] + shift
    return torch.from_numpy(np.stack([i % 1009, i // 1009, i % 7], axis=1).astype(np.int32)).cuda()


def test_tables_large_for_the_batch(ash):
    """The bins write the table whole: with more than four slots per position
    only where the last insert of such a size brought mostly new keys."""
    n = INSERT_MIN + 9
    few, many = spread(n, 0.4), spread(n, 0.9)
    for slots, expect in ((3, [True, True, True]), (7, [False, False, True])):
        m = ash.HashSet(int(slots * n * 0.5), 3)
        m.profile()
        got = []
        for keys in (few, many, few):  # without a word from an insert before; after 40% new; after 90%
            m.clear()
            m.profile_collect()
            idx, mask = m.activate(keys)
            got.append("claim_bins" in m.profile_collect())
            assert m.size() == int(mask.sum()) == len(torch.unique(keys, dim=0))
            assert torch.equal(m.key_buffer()[idx[mask].long()], keys[mask])
        assert got == expect, slots
        m.close()


def test_a_few_keys_say_nothing_of_millions(ash):
    """An insert of ten repeated keys, or of 100 new ones, does not decide how
    the next insert of millions goes."""
    n = INSERT_MIN + 9
    many = spread(n, 0.9)
    for word in (torch.zeros((10, 3), dtype=torch.int32, device="cuda"), spread(100, 1.0)):
        for slots, expect in ((3, True), (7, False)):
            m = ash.HashSet(int(slots * n * 0.5), 3)
            m.activate(word)
            m.clear()
            m.profile()
            torch.cuda.synchronize()
            m.activate(many)
            assert ("claim_bins" in m.profile_collect()) == expect, slots
            m.close()


@pytest.mark.parametrize("w,g", [(4, 4), (8, 8)])
def test_width_4_after_a_few_keys(ash, w, g):
    """Key width 4 takes the word of an insert of 100 new keys on wide buckets only."""
    n = INSERT_MIN + 9
    many = spread(n, 0.9)
    many = torch.cat([many, many[:, :1]], dim=1).contiguous()
    m = ash.HashSet(n, 4, bucket_width=w, probe_group=g)
    m.activate(many[:100])
    m.clear()
    m.profile()
    torch.cuda.synchronize()
    for expect in (w == 8, True):  # then of one of its own size
        m.clear()
        m.profile_collect()
        m.activate(many)
        assert ("claim_bins" in m.profile_collect()) == expect

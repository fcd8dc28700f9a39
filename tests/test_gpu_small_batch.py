"""Batches around the two-launch front end (at most 8192 ids) against the oracle.

Integers bit-exact, sums and updates within the step parity's bounds
(tests/parity.py).  The first batch of a table needs Blocks, so it takes the
general front end at a small size; the later ones find room and take the two
launches, with keys known, new, repeated and hot (hot-key units from 33
occurrences on).  8193 ids take the general front end.
"""
import numpy as np
import pytest
import torch

import oracle as O
from paper_2509_20883_amd import recis as R
from paper_2509_20883_amd import workloads as W
from tests import parity as P

pytestmark = pytest.mark.gpu


def _keys(pattern, n, step, g):
    if pattern == "distinct":
        return g.permutation(n) + n * (step // 2)  # every other step known
    if pattern == "same":
        return np.full(n, 77)
    if pattern == "counts":  # keys of 1, 31, 32, 33, 64, 65 and many ids, interleaved
        k = np.concatenate([np.full(c, 10 * step + j) for j, c in enumerate((1, 31, 32, 33, 64, 65))])
        k = np.concatenate([k, np.full(max(n // 3, 1), 5), g.integers(0, 4 * n, size=n)])[:n]
        return g.permutation(k)
    return np.minimum(g.zipf(1.2, size=n), 1 << 40)


@pytest.mark.parametrize("n", [1, 2, 63, 1024, 1025, 4750, 8191, 8192, 8193])
@pytest.mark.parametrize("pattern", ["distinct", "same", "counts", "zipf"])
def test_small_batches_match_oracle(n, pattern):
    print("small batch", n, pattern, flush=True)
    w = W.workload(0)
    w.mode = W.MEAN if n % 2 else W.SUM
    w.capacity_slots = 1 << 16
    g = np.random.default_rng(n)
    gt, ot = P.gpu_table(w), P.oracle_table(w)
    for step in range(4):
        lens = g.integers(0, 6, size=n)
        cut = np.minimum(np.cumsum(lens), n)
        cut[-1] = n
        off = np.concatenate([[0], cut]).astype(np.int64)
        b = W.Batch(values=_keys(pattern, n, step, g).astype(np.int64), offsets=off, n_features=1, batch=n)
        P.run_step_parity(w, gt, ot, b, g.standard_normal((b.bags, w.dim)).astype(np.float32), step)
    gt.check()
    gt.close()


@pytest.mark.parametrize("mode,pad", [(W.NONE, 7), (W.TAIL, 7)])
def test_small_padded_batches_match_oracle(mode, pad):
    """Ids outside the copied window have no gradient row in the list the pool writes."""
    w = W.workload(5, mini=True)
    w.mode, w.pad_len = mode, pad
    g = np.random.default_rng(3)
    gt, ot = P.gpu_table(w), P.oracle_table(w)
    for step in range(3):
        off = np.concatenate([[0], np.cumsum(g.integers(0, 20, size=300))]).astype(np.int64)
        b = W.Batch(values=g.integers(0, 900, size=off[-1]), offsets=off, n_features=1, batch=300)
        P.run_step_parity(w, gt, ot, b, W.make_grad(w, b, step, nan_in_masked=True), step)
    gt.check()
    gt.close()


def test_small_batch_reserved_keys_evictions_and_find_or_insert():
    """Rejected keys take no part, freed rows are reused top first, clocks are kept: all as the oracle."""
    gt = R.Table(8, R.F32, R.ADAGRAD, capacity_slots=1 << 14, seed=3, block_rows=1 << 13, evictable=True)
    ot = O.Table(8, opt=O.ADAGRAD, seed=3)
    g = np.random.default_rng(9)
    gt.find_or_insert(torch.arange(4000, dtype=torch.int64, device="cuda"))
    ot.find_or_insert(np.arange(4000))
    for it in range(8):
        keys = g.integers(0, 6000, size=3001)
        rows, nins = gt.find_or_insert(torch.from_numpy(keys).cuda())
        st, rref, nref = ot.find_or_insert(keys)
        assert st == O.OK and np.array_equal(rows.cpu().numpy(), rref) and int(nins.item()) == nref, it
        if it % 3 == 2:
            assert gt.evict(1) == ot.evict(1)
    gk, gr = (x.cpu().numpy() for x in gt.export())
    rk, rr = ot.export()
    assert dict(zip(gk.tolist(), gr.tolist())) == dict(zip(rk.tolist(), rr.tolist()))
    gt.check()
    keys = np.array([5, -2 ** 63, 7, -2 ** 63 + 1, 5], dtype=np.int64)
    rows, nins = gt.find_or_insert(torch.from_numpy(keys).cuda())
    with pytest.raises(R.RecisError, match="RS_EKEY"):
        gt.check()
    rows = rows.cpu().numpy()
    assert rows[1] == -1 and rows[3] == -1 and rows[0] == rows[4] >= 0 and rows[2] >= 0
    gt.close()


@pytest.mark.parametrize("max_load,slots,third", [(0.6, 1 << 13, 3000), (0.75, 1 << 13, 5000)])
def test_batch_past_the_small_limit_grows_the_table(max_load, slots, third):
    """A batch of at most 8192 ids that may not fit takes the general front end, which reads the published count
    again: the table still grows and every key gets a row."""
    t = R.Table(8, R.F32, R.ADAGRAD, capacity_slots=slots, max_load=max_load, block_rows=1 << 13, seed=3)
    first = torch.arange(2000, dtype=torch.int64, device="cuda")
    new = torch.arange(10000, 10000 + third, dtype=torch.int64, device="cuda")
    for keys, want in ((first, 2000), (first, 0), (new, third), (new, 0)):
        rows, nins = t.find_or_insert(keys)
        torch.cuda.synchronize()  # the call's count is published before the next one reads it
        print("bound", keys.numel(), int(nins.item()), flush=True)
        assert int(nins.item()) == want and int(rows.min().item()) >= 0
    assert t.size() == 2000 + third and t.capacity() > slots
    t.check()
    t.close()

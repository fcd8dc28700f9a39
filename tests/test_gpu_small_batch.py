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


@pytest.mark.parametrize("dim", [8, 16, 32, 64, 128, 256])
@pytest.mark.parametrize("dtype", [W.F32, W.BF16])
@pytest.mark.parametrize("mode", [W.SUM, W.MEAN, W.NONE, W.TAIL])
def test_small_batch_at_every_width_and_backward_again(dim, dtype, mode):
    """Lane groups of 1 to 64 lanes, fp32 and bf16 rows and gradients; keys of one to ten hot-key units.  A context's
    backward can run again (the counter of a key's finished units starts over): two-call sums twice, then fused."""
    print("small batch width", dim, dtype, mode, flush=True)
    w = W.workload(0)
    w.dim, w.row_dtype, w.mode, w.capacity_slots = dim, dtype, mode, 1 << 14
    w.grad_dtype = dtype if W.padded(mode) else W.F32
    w.pad_len = 13 if W.padded(mode) else 0
    g = np.random.default_rng(dim)
    gt, ot = P.gpu_table(w), P.oracle_table(w)
    for step in range(2):  # the first on the general front end (a new table), the second on the two launches
        off = np.concatenate([[0], np.cumsum(g.integers(0, 20, size=250))]).astype(np.int64)
        n = int(off[-1])
        ids = np.concatenate([np.full(c, 7 + i) for i, c in enumerate((33, 64, 65, 320))] +
                             [g.integers(100, 100 + n, size=n)])[:n]
        b = W.Batch(values=g.permutation(ids), offsets=off, n_features=1, batch=250)
        grad = W.make_grad(w, b, step)
        P.run_step_parity(w, gt, ot, b, grad, step)
        # the same batch again, every key known: sums twice, then the fused update
        _, _, ctx = gt.forward(P.to_dev(b.values), P.to_dev(off), mode, pad_len=w.pad_len)
        _, uniq, inv = O.dedup(b.values)
        U = uniq.size
        ref = O.backward(off, inv, U, dim, mode, w.pad_len, grad)
        mag = O.backward(off, inv, U, dim, mode, w.pad_len, np.abs(grad))
        gd = P.to_dev(grad)
        if w.grad_dtype == W.BF16:
            gd = gd.to(torch.bfloat16)
        for again in range(2):
            P.assert_sum_close(gt.backward(ctx, gd)[:U].cpu().numpy(), ref, mag, what=f"backward {again}")
        w0, s0 = (x.cpu().numpy() for x in gt.read_rows(ctx.rows(U)))
        gt.backward_optimizer(ctx, gd, w.lr, w.eps)
        w1, s1 = (x.cpu().numpy() for x in gt.read_rows(ctx.rows(U)))
        ot.write_rows(uniq, w0, s0)
        _, rows, _ = ot.find_or_insert(uniq)
        ot.optimizer(rows, ref.astype(np.float32), w.lr, w.eps)
        _, w_ref, s_ref = ot.read_rows(uniq)
        dg = 1e-5 * mag + np.abs(ref) * 2.0 ** -23
        P.assert_opt_close(w1, s1, w_ref, s_ref,
                           P.opt_bounds(w.opt, dtype, w0, s0, ref, dg, w.lr, w.eps, w.beta1, w.beta2, ot.t, w_ref),
                           what="fused update")
        ot.write_rows(uniq, w1, s1)
    gt.check()
    gt.close()


@pytest.mark.parametrize("mode", [W.SUM, W.TAIL])
def test_small_batch_with_reserved_keys(mode):
    """A table with room, so the two launches see the rejected ids: no unique id, no row, no place in the list."""
    w = W.workload(0)
    w.mode, w.pad_len, w.capacity_slots = mode, 9 if W.padded(mode) else 0, 1 << 14
    g = np.random.default_rng(2)
    gt, ot = P.gpu_table(w), P.oracle_table(w)
    gt.find_or_insert(torch.arange(8000, dtype=torch.int64, device="cuda"))  # provisions room for more
    ot.find_or_insert(np.arange(8000))
    off = np.concatenate([[0], np.cumsum(g.integers(0, 12, size=400))]).astype(np.int64)
    n = int(off[-1])
    ids = g.integers(0, 400, size=n)
    ids[g.permutation(n)[:300]] = -2 ** 63
    ids[g.permutation(n)[:300]] = -2 ** 63 + 1
    b = W.Batch(values=ids, offsets=off, n_features=1, batch=400)
    grad = W.make_grad(w, b, 0)
    ctx = R.Ctx()
    ctx.ensure(gt.workspace_bytes(n, 400), torch.device("cuda"))
    ctx.ws.fill_(0xA5)
    out, mask, ctx = gt.forward(P.to_dev(ids), P.to_dev(off), mode, pad_len=w.pad_len, ctx=ctx)
    U = int(ctx.scalars()[0].item())
    kept = ids > -2 ** 63 + 1
    st, uniq, kept_inv = O.dedup(ids[kept])  # the oracle refuses a reserved key: the others, deduplicated
    inv = np.full(n, -1, dtype=np.int32)
    inv[kept] = kept_inv
    assert st == O.OK and U == uniq.size and np.array_equal(ctx.unique(U).cpu().numpy(), uniq)
    assert np.array_equal(ctx.inverse().cpu().numpy(), inv)
    rows = np.concatenate([ot.read_rows(uniq)[1], np.zeros((1, w.dim), dtype=np.float32)])  # [-1]: nothing
    o = out.cpu().numpy()
    if W.padded(mode):
        want, m = np.zeros_like(o), np.zeros((400, w.pad_len), dtype=np.uint8)
        for i in range(400):
            last = np.arange(off[i], off[i + 1])[-w.pad_len:]
            want[i, :last.size], m[i, :last.size] = rows[inv[last]], 1
        assert np.array_equal(o, want) and np.array_equal(mask.cpu().numpy(), m)
    else:
        bag = np.repeat(np.arange(400), np.diff(off))
        want, mag = np.zeros(o.shape), np.zeros(o.shape)
        np.add.at(want, bag, rows[inv].astype(np.float64))
        np.add.at(mag, bag, np.abs(rows[inv]).astype(np.float64))
        P.assert_sum_close(o, want, mag, what="pooled")
    gu = gt.backward(ctx, P.to_dev(grad))[:U].cpu().numpy()
    P.assert_sum_close(gu, O.backward(off, inv, U, w.dim, mode, w.pad_len, grad),
                       O.backward(off, inv, U, w.dim, mode, w.pad_len, np.abs(grad)), what="grad_unique")
    with pytest.raises(R.RecisError, match="RS_EKEY"):
        gt.check()
    gt.close()

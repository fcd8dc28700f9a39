"""Ids made to share a dedup partition and every sweep of it, against the oracle.

The partition hash is splitmix64's (invertible) output function, so ids can be
made whose hashes agree in the top 12 bits (the partition) and the low 20 (the
sweeps).  More than 2048 such distinct ids fit no sweep's table, however many
sweeps: they are taken in rounds.  "window": the ids also agree in the eleven
bits that place them in a round's table, so that a round takes 64 of them.
Integers bit-exact, sums and updates within the step parity's bounds
(tests/parity.py).
"""
import functools

import numpy as np
import pytest
import torch

import oracle as O
from paper_2509_20883_amd import recis as R
from paper_2509_20883_amd import workloads as W
from tests import parity as P

M64 = (1 << 64) - 1
SIGN = np.uint64(1 << 63)
PART_SALT, IDMAP_SALT = np.uint64(0x5BD1E9955BD1E995), np.uint64(0x2545F4914F6CDD1D)
MUL = (0xBF58476D1CE4E5B9, 0x94D049BB133111EB)


def _mix(z):
    z = (z ^ (z >> np.uint64(30))) * np.uint64(MUL[0])
    z = (z ^ (z >> np.uint64(27))) * np.uint64(MUL[1])
    return z ^ (z >> np.uint64(31))


def _unshift(z, k):
    x = z
    for _ in range(64 // k):
        x = z ^ (x >> np.uint64(k))
    return x


def _unmix(z):
    z = _unshift(z, 31) * np.uint64(pow(MUL[1], -1, 1 << 64))
    z = _unshift(z, 27) * np.uint64(pow(MUL[0], -1, 1 << 64))
    return _unshift(z, 30)


@functools.lru_cache(None)
def made_ids(count, window=False):
    """`count` distinct ids whose partition hash is j << 20, j < 2^32."""
    j = np.arange(1, 1 + count * (1 << 12 if window else 1), dtype=np.uint64)
    enc = _unmix(j << np.uint64(20)) ^ PART_SALT
    if window:
        enc = enc[(_mix(enc ^ IDMAP_SALT) >> np.uint64(20)) & np.uint64(2047) == 7]
    assert enc.size >= count
    return (enc[:count] ^ SIGN).view(np.int64)


def _batch(count, n, window, g):
    """n ids: every made id, repeats of them, and ordinary ids."""
    made = made_ids(count, window)
    rest = n - count
    ids = np.concatenate([made, made[g.integers(0, count, size=rest // 2)], g.integers(0, n, size=rest - rest // 2)])
    return g.permutation(ids)


@pytest.mark.parametrize("window", [False, True])
def test_made_ids_collide(window):
    ids = made_ids(2100, window)
    h = _mix(ids.view(np.uint64) ^ SIGN ^ PART_SALT)
    assert np.unique(ids).size == 2100 and not (h >> np.uint64(52)).any() and not (h & np.uint64(0xFFFFF)).any()


CASES = [(2100, 2100, False), (2100, 2100, True), (3000, 3000, False), (2049, 9001, False), (6000, 40000, False),
         (2100, 20000, True)]


@pytest.mark.gpu
@pytest.mark.parametrize("count,n,window", CASES)
def test_ids_partition_of_colliding_ids(count, n, window):
    print("colliding ids partition", count, n, window, flush=True)
    vals = _batch(count, n, window, np.random.default_rng(n))
    keys, offs, inv, info = (x.cpu().numpy() for x in R.ids_partition(torch.from_numpy(vals).cuda(), 8, 3))
    ek, eo, ei, _ = O.ids_partition(vals, 8, 3)
    assert int(info[0]) == len(ek) and int(info[1]) == 0 and np.array_equal(keys[:len(ek)], ek)
    assert np.array_equal(offs, eo) and np.array_equal(inv, ei)


@pytest.mark.gpu
@pytest.mark.parametrize("count,n,window", [c for c in CASES if c[1] > 8192])
def test_steps_of_colliding_ids(count, n, window):
    print("colliding ids step", count, n, window, flush=True)
    w = W.workload(0)
    w.mode, w.capacity_slots = W.SUM, 1 << 17
    g = np.random.default_rng(count)
    gt, ot = P.gpu_table(w), P.oracle_table(w)
    for step in range(2):  # new keys, then known ones
        off = np.concatenate([[0], np.sort(g.integers(0, n + 1, size=999)), [n]]).astype(np.int64)
        b = W.Batch(values=_batch(count, n, window, g), offsets=off, n_features=1, batch=1000)
        P.run_step_parity(w, gt, ot, b, g.standard_normal((1000, w.dim)).astype(np.float32), step)
    gt.check()
    gt.close()

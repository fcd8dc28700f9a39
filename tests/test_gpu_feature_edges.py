"""Bucketize and mod where their blocks change path, bit-exact against the oracle.

Boundary counts around powers of two (the shared search step of a block's
elements), at and past the LDS stage; columns so short that a block spans more
columns than it has threads (each element divides), at most as many (one
reciprocal per column), and moduli / ids at the ends of their ranges.
"""
import numpy as np
import pytest
import torch

import oracle as O
from paper_2509_20883_amd import recis as R
from paper_2509_20883_amd import workloads as W

pytestmark = pytest.mark.gpu


def _dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


@pytest.mark.parametrize("nb", [0, 1, 2, 3, 4, 7, 8, 9, 63, 64, 65, 4095, 4096, 4097])
def test_bucketize_boundary_counts(nb):
    print("bucketize", nb, flush=True)
    g = np.random.default_rng(nb)
    b = np.sort(np.round(g.normal(size=2 * nb) * 50) / 4).astype(np.float32)  # repeated boundaries
    bo = np.array([0, nb, 2 * nb], dtype=np.int64)
    b[:nb].sort(), b[nb:].sort()
    co = np.array([0, 2500, 5001], dtype=np.int64)
    v = (np.round(g.normal(size=5001) * 60) / 4).astype(np.float32)
    v[:8] = [np.nan, -np.inf, np.inf, -0.0, 0.0, 3e38, -3e38, np.nan]
    if nb:
        v[100:100 + min(nb, 900)] = b[:min(nb, 900)]  # exact hits
    out = R.fused_bucketize(_dev(v), _dev(co), _dev(b if b.size else np.zeros(1, np.float32)), _dev(bo))
    assert np.array_equal(out.cpu().numpy(), O.bucketize(v, co, b, bo))


@pytest.mark.parametrize("ncols,most", [(1, 4000), (5, 700), (900, 3), (900, 9), (1023, 40), (1024, 2), (3000, 2)])
def test_mod_column_lengths_and_extremes(ncols, most):
    print("mod", ncols, most, flush=True)
    g = np.random.default_rng(ncols)
    size = g.integers(0, most + 1, size=ncols)
    size[0] = most
    co = np.concatenate([[0], np.cumsum(size)]).astype(np.int64)
    n = int(co[-1])
    lo, hi = np.iinfo(np.int64).min, np.iinfo(np.int64).max
    m = np.exp(g.uniform(0, 43, size=ncols)).astype(np.int64).clip(1)
    special = [1, 2, 3, 2 ** 32 - 1, 2 ** 32, 2 ** 32 + 1, 2 ** 62, 2 ** 62 + 7, hi, hi - 1]
    m[:min(ncols, len(special))] = special[:ncols]
    v = g.integers(lo, hi, size=n, dtype=np.int64)
    v[::3] = (g.integers(0, 1000, size=v[::3].size) * np.repeat(m, size)[::3].astype(object) % 2 ** 62).astype(np.int64)
    edge = [lo, lo + 1, -1, 0, 1, hi, hi - 1]
    v[:min(n, len(edge))] = edge[:n]
    out = R.fused_mod(_dev(v), _dev(co), _dev(m))
    assert np.array_equal(out.cpu().numpy(), O.mod(v, co, m))

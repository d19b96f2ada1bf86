"""Digit bases, pass 0's tile prefixes and the plan from the histogram's rows (Sec. 4, Algorithm 4), at the edges of
their splits: rows that do not fit (up to 2047 keys), one tile, 64 ranges of tiles of up to 16 in registers and more,
one launch for the prefixes (up to 4096 tiles) and three."""
import numpy as np
import pytest

import oracle
from gpu_util import assert_bits_equal, require_gpu, to_dev, to_np

pytestmark = pytest.mark.gpu

TILE = 256 * 8


def _keys(kind, n):
    k = np.random.default_rng(n).integers(-2**31, 2**31, n, dtype=np.int64).astype(np.int32)
    if kind == "low_only":   # the last pass is left out, another is not
        return k & np.int32(0x00FF00FF)
    if kind == "constant":   # every pass is left out: the last one copies
        return np.full(n, 7, np.int32)
    return k


@pytest.mark.parametrize("kind", ["full", "low_only", "constant"])
@pytest.mark.parametrize("n", [2, 1023, TILE - 1, TILE, TILE + 1, 63 * TILE, 64 * TILE + 1, 16 * 64 * TILE,
                               16 * 64 * TILE + 1, 4096 * TILE, 4096 * TILE + 1])
def test_digits_from_rows(n, kind):
    import torch

    es = require_gpu()
    keys = _keys(kind, n)
    perm = oracle.stable_perm(keys)
    want = keys[perm]
    p = es.default_params(algo=es.ALGO_RADIX, block_threads=256, items_per_thread=8, fallback_threshold=0)
    dk = to_dev(keys)
    assert es.plan(es.OP_SORT, es.dtype_code(dk.dtype), n, 0, p)["path_name"] == "radix"
    assert_bits_equal(to_np(es.sort(dk, params=p)), want, "keys")
    k2, v2 = es.sort_pairs(dk, torch.arange(n, device="cuda", dtype=torch.int32), params=p)
    assert_bits_equal(to_np(k2), want, "keys")
    assert_bits_equal(to_np(v2), perm.astype(np.int32), "values")
    assert_bits_equal(to_np(es.argsort(dk, params=p)), perm.astype(np.int64), "indices")
    es.sort(dk, params=p, out=dk)  # in place: an odd number of live passes is copied after them
    assert_bits_equal(to_np(dk), want, "keys")


@pytest.mark.parametrize("n", [16383 * TILE + 5, 16384 * TILE + 5])
def test_many_rows_summed_first(n):
    """1024 rows go straight to the digit bases; 4096 are summed to 64 first."""
    es = require_gpu()
    keys = _keys("full", n)
    p = es.default_params(algo=es.ALGO_RADIX, block_threads=256, items_per_thread=8)
    assert_bits_equal(to_np(es.sort(to_dev(keys), params=p)), np.sort(keys), "keys")

"""Small arrays and short segments are sorted by networks in registers and merges in LDS: every length at which the
number of records per thread or of waves changes, for every record size, against the oracle."""
import numpy as np
import pytest

import oracle
import workloads
from gpu_util import assert_bits_equal, require_gpu, to_dev, to_np

pytestmark = pytest.mark.gpu

EDGES = [1, 2, 63, 64, 65, 127, 128, 129, 255, 256, 257, 511, 512, 513, 1023, 1024, 1025, 2047, 2048, 2049, 4095, 4096]
TOPS = {np.int32: [4097, 8191, 8192], np.int64: [4097, 8191, 8192], np.float32: [8192], np.float64: [8192]}


def _keys(dt, n, seed):
    keys = workloads.uniform(dt, n, seed)
    keys[::5] = keys[n // 2]
    if np.dtype(dt).kind == "i":  # the word short records are filled up with
        keys[: n // 9] = np.iinfo(dt).max
    return keys


@pytest.mark.parametrize("desc", [0, 1])
@pytest.mark.parametrize("dt", [np.int32, np.int64, np.float64])
def test_small_arrays(dt, desc):
    import torch

    es = require_gpu()
    # A_code 4: the one-workgroup sort up to its capacity, also where the automatic choice sorts by splitters
    p = es.default_params(algo=es.ALGO_RADIX, descending=desc)
    for n in EDGES + TOPS[dt]:
        keys = _keys(dt, n, n)
        perm = oracle.stable_perm(keys, descending=bool(desc))
        k = to_dev(keys)
        assert_bits_equal(to_np(es.sort(k, params=p)), keys[perm], f"keys {n}")
        for vals in (np.arange(n, dtype=np.int32) * 3, np.arange(n, dtype=np.int64) * 5):
            kin, vin = to_dev(keys), to_dev(vals)
            es.sort_pairs(kin, vin, params=p, keys_out=kin, values_out=vin)  # in place
            assert_bits_equal(to_np(kin), keys[perm], f"pairs({vals.itemsize}) {n} keys")
            assert_bits_equal(to_np(vin), vals[perm], f"pairs({vals.itemsize}) {n} values")
        assert np.array_equal(to_np(es.argsort(k, index_dtype=torch.int32, params=p)), perm), f"argsort {n}"


@pytest.mark.parametrize("vb", [0, 4, 8])
@pytest.mark.parametrize("dt", [np.int32, np.int64, np.float32])
def test_segments_at_every_edge(dt, vb):
    """Each length several times, so that every wave and workgroup sorts segments of changing lengths in turn."""
    es = require_gpu()
    sizes = np.array((EDGES + TOPS[dt]) * 9, dtype=np.int64)
    workloads.rng(1).shuffle(sizes)
    offs = workloads.segment_offsets(sizes)
    n = int(offs[-1])
    keys = _keys(dt, n, 7)
    k = to_dev(keys)
    if not vb:
        es.segmented_sort(k, to_dev(offs), out=k, check=True)  # in place
        assert_bits_equal(to_np(k), oracle.segmented_sort(keys, offs), "keys")
        return
    vals = np.arange(n, dtype=np.int32 if vb == 4 else np.int64)
    v = to_dev(vals)
    es.segmented_sort_pairs(k, v, to_dev(offs), keys_out=k, values_out=v, check=True)
    wk, wv = oracle.segmented_sort_pairs(keys, vals, offs)
    assert_bits_equal(to_np(k), wk, "pairs keys")
    assert_bits_equal(to_np(v), wv, "pairs values")

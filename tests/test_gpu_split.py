"""The splitter sort, which the automatic choice (A_code 0) takes for mid-size arrays (Sec. 4.3, Algorithm 6): every
operation, key type and order against the oracle, element by element, at the edges of its range and of its block
sizes, on inputs that spread well over the buckets and on inputs that do not."""
import numpy as np
import pytest

import oracle
import workloads
from gpu_util import assert_bits_equal, require_gpu, to_dev, to_np

pytestmark = pytest.mark.gpu

RANGE = {4: (8_193, 400_000), 8: (4_097, 262_144)}  # lengths of the route for keys only, by key bytes
DTYPES = [np.int32, np.uint32, np.float32, np.int64, np.float64]


def _split_ran(es, call):
    es.profile_reset()
    es.profile_enable(True)
    try:
        call()
        names = es.profile_collect()
    finally:
        es.profile_enable(False)
    return "split_buckets" in names


def _check(es, keys, desc=0, expect=True):
    import torch

    n = keys.size
    p = es.default_params(descending=desc)
    perm = oracle.stable_perm(keys, descending=bool(desc))
    want = keys[perm]
    k = to_dev(keys)
    assert _split_ran(es, lambda: es.sort(k, params=p)) == expect
    assert_bits_equal(to_np(es.sort(k, params=p, check=True)), want, "keys")
    for vals in ((np.arange(n, dtype=np.int64) * 7 + 1).astype(np.int32), np.arange(n, dtype=np.int64) * 3 - 5):
        ko, vo = es.sort_pairs(k, to_dev(vals), params=p, check=True)
        assert_bits_equal(to_np(ko), want, f"pairs({vals.itemsize}) keys")
        assert_bits_equal(to_np(vo), vals[perm], f"pairs({vals.itemsize}) values")
        kin, vin = to_dev(keys), to_dev(vals)
        es.sort_pairs(kin, vin, params=p, keys_out=kin, values_out=vin, check=True)
        assert_bits_equal(to_np(kin), want, f"pairs({vals.itemsize}) in place: keys")
        assert_bits_equal(to_np(vin), vals[perm], f"pairs({vals.itemsize}) in place: values")
    for idt in (torch.int32, torch.int64):
        assert np.array_equal(to_np(es.argsort(k, index_dtype=idt, params=p, check=True)), perm), f"argsort {idt}"
    es.sort(k, params=p, out=k, check=True)
    assert_bits_equal(to_np(k), want, "in place")


@pytest.mark.parametrize("n", [4_096, 4_097, 8_192, 8_193, 16_383, 16_385, 100_003, 131_072, 131_073, 262_144, 262_145,
                               400_000, 400_001])
@pytest.mark.parametrize("dt", [np.int32, np.float64])
def test_edges_of_the_range(dt, n):
    keys = workloads.float_mix(dt, n, n) if np.dtype(dt).kind == "f" else workloads.uniform(dt, n, n)
    keys[::7] = keys[3]
    low, high = RANGE[np.dtype(dt).itemsize]
    _check(require_gpu(), keys, expect=low <= n <= high)


@pytest.mark.parametrize("desc", [0, 1])
@pytest.mark.parametrize("dt", DTYPES)
def test_key_types(dt, desc):
    keys = workloads.uniform(dt, 50_001, 5)
    if np.dtype(dt).kind == "f":
        keys[:14] = workloads.float_edges(dt)
    else:
        keys[:3] = [np.iinfo(dt).max, np.iinfo(dt).min, np.iinfo(dt).max]  # the word a short block is filled up with
    keys[-5:] = keys[:5]
    _check(require_gpu(), keys, desc)


def _shaped(name, n, dt):
    g = np.random.default_rng(3)
    if name == "one_bucket":  # most keys lie between two neighbouring samples of every block: buckets in many steps
        keys = np.sort(workloads.uniform(dt, n, 3))
        keys = keys.reshape(-1, 512)
        keys[:, 5:500] = 1000 + g.integers(0, 3000, (keys.shape[0], 495))
        return keys.reshape(-1).copy()
    return workloads.make(name, dt, n, 3)


@pytest.mark.parametrize("n", [32_768, 262_144])
@pytest.mark.parametrize("name", ["all_equal", "distinct16", "sorted", "reverse", "nearly_sorted", "zipf", "one_bucket"])
@pytest.mark.parametrize("dt", [np.int32, np.int64])
def test_shapes(dt, name, n):
    _check(require_gpu(), _shaped(name, n, dt))


def test_small_scratch_keeps_the_branch():
    """A scratch that holds the routine of the branch only (here one workgroup: the header) is accepted as before."""
    import torch

    es = require_gpu()
    keys = workloads.uniform(np.int32, 10_000, 8)
    tmp = torch.empty(256, dtype=torch.uint8, device="cuda")
    out = torch.empty(10_000, dtype=torch.int32, device="cuda")
    k = to_dev(keys)
    assert not _split_ran(es, lambda: es.sort(k, out=out, temp=tmp))
    assert_bits_equal(to_np(out), oracle.sort(keys), "keys")

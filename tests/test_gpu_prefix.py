"""Prefix sorts: only the upper digits are passed over, then runs of equal upper digits are sorted in place of
the lower passes (Sec. 4, Algorithms 4 and 5: the result is the stable sort by the whole key).

Every pattern is checked element by element against the oracle for keys, pairs and argsort, and the plan word the
call leaves in its scratch (stages in byte 24, first pass in byte 25, listed long runs in the word at 232) shows
that the route under test is the one that ran.
"""
import numpy as np
import pytest

import oracle
import workloads
from gpu_util import assert_bits_equal, require_gpu, to_dev, to_np

pytestmark = pytest.mark.gpu


def _keys(name, n):
    g = np.random.default_rng(11)
    u = g.integers(0, 2**64, n, dtype=np.uint64)
    if name == "uniform":
        return u.view(np.int64)
    if name == "short_runs":        # about 3 keys per run of equal upper 5 bytes, ties among them
        hi = g.integers(0, n // 3, n, dtype=np.uint64) * np.uint64(2654435761) % np.uint64(2**40)
        return ((hi << np.uint64(24)) | (u & np.uint64(0x010301))).view(np.int64)
    if name == "duplicates":        # 10 copies of every key
        return u[g.integers(0, n // 10, n)].view(np.int64)
    if name == "float":
        return workloads.float_mix(np.float64, n, 5)
    if name == "few_groups":        # 64 upper words, every lower word different
        return (((u >> np.uint64(58)) * np.uint64(0x9E3779B97F4A7C15) & np.uint64(0xFFFFFFFF00000000))
                | (u & np.uint64(0xFFFFFFFF))).view(np.int64)
    if name == "heavy":             # nine of ten keys are one value
        u[g.random(n) < 0.9] = np.uint64(77)
        return u.view(np.int64)
    if name == "zeros":             # one of five keys is zero, alone in its run
        u[g.random(n) < 0.2] = np.uint64(0)
        return u.view(np.int64)
    if name == "strangers":         # the same, and a few other keys in that run, too few for the sample to see
        u[g.random(n) < 0.2] = np.uint64(77)
        u[[1, n // 3, n // 2, n - 2]] = np.array([5, 99, 70, 80], dtype=np.uint64)
        return u.view(np.int64)
    if name == "one_top_byte":      # the upper digits never vary
        return (u & np.uint64(0xFFFF)).view(np.int64)
    raise ValueError(name)


def _run_all(es, keys, prefix, desc=0, params=None, most=None):
    """Every operation on `keys` against the oracle; `prefix`: whether the plan is a prefix sort (None: either);
    `most`: the length its longest run has at least."""
    import torch

    n = keys.size
    p = params or es.default_params(algo=es.ALGO_RADIX, descending=desc)
    perm = oracle.stable_perm(keys, descending=bool(desc))
    want = keys[perm]
    code = es.dtype_code(to_dev(keys[:1]).dtype)

    def temp(op, vb):
        return torch.empty(es.temp_bytes(op, code, n, vb, p), dtype=torch.uint8, device="cuda")

    def check_route(t, what):
        head = t[:256].cpu().numpy()
        first = int(head[25])
        if prefix is not None:
            assert (first > 0) == prefix, f"{what}: first pass {first}"
        if first:  # runs of more than 256 keys are listed
            _, length = np.unique(oracle.order_keys(keys) >> np.uint64(8 * first), return_counts=True)
            listed = int((length > 256).sum())
            assert int(head[232:236].view(np.uint32)[0]) == listed, what
            assert most is None or int(length.max()) >= most

    k = to_dev(keys)
    t = temp(es.OP_SORT, 0)
    assert_bits_equal(to_np(es.sort(k, params=p, temp=t, check=True)), want, "keys")
    check_route(t, "keys")
    for vals in ((np.arange(n, dtype=np.int64) * 7 + 1).astype(np.int32), np.arange(n, dtype=np.int64) * 3 - 5):
        t = temp(es.OP_SORT_PAIRS, vals.itemsize)
        ko, vo = es.sort_pairs(k, to_dev(vals), params=p, temp=t, check=True)
        assert_bits_equal(to_np(ko), want, f"pairs({vals.itemsize}) keys")
        assert_bits_equal(to_np(vo), vals[perm], f"pairs({vals.itemsize}) values")
        check_route(t, f"pairs({vals.itemsize})")
        kin, vin = to_dev(keys), to_dev(vals)
        es.sort_pairs(kin, vin, params=p, keys_out=kin, values_out=vin, check=True)
        assert_bits_equal(to_np(kin), want, f"pairs({vals.itemsize}) in place: keys")
        assert_bits_equal(to_np(vin), vals[perm], f"pairs({vals.itemsize}) in place: values")
    for idt in (torch.int32, torch.int64):
        t = temp(es.OP_ARGSORT, 4 if idt == torch.int32 else 8)
        assert np.array_equal(to_np(es.argsort(k, index_dtype=idt, params=p, temp=t, check=True)), perm), idt
        check_route(t, f"argsort {idt}")
    es.sort(k, params=p, out=k, check=True)
    assert_bits_equal(to_np(k), want, "keys in place")


@pytest.mark.parametrize("desc", [0, 1])
@pytest.mark.parametrize("n", [16_384, 100_003, 1_048_577])
@pytest.mark.parametrize("name, prefix", [("uniform", True), ("short_runs", True), ("duplicates", None),
                                          ("float", True), ("few_groups", None), ("heavy", None),
                                          ("zeros", None), ("strangers", None),
                                          ("one_top_byte", False)])
def test_patterns(name, prefix, n, desc):
    _run_all(require_gpu(), _keys(name, n), prefix, desc)


@pytest.mark.parametrize("length", [255, 256, 257, 600, 1000])
def test_long_runs(length):
    """One run at the longest length sorted beside its neighbours, one longer, and far longer ones (one workgroup
    each), among short runs; the first and the last keys of the array are in such runs too."""
    es = require_gpu()
    n = 2_000_003
    keys = _keys("uniform", n)
    u = keys.view(np.uint64)
    g = np.random.default_rng(3)
    low = np.uint64(0xFFFFFF)
    at = g.permutation(n)[:3 * length]
    for i, top in enumerate((0x8000000000, 0x7FFFFFFFFF, 0x123456789A)):  # smallest, largest and one more as int64
        u[at[i * length:(i + 1) * length]] = (np.uint64(top << 24)
                                              | (g.integers(0, 2**24, length, dtype=np.uint64) & low))
    keys = u.view(np.int64)
    _run_all(es, keys, True, most=length)


def test_run_above_one_workgroup():
    """A run longer than one workgroup's sort holds (merged in pieces) and out of order in four places that the
    sample does not see."""
    _run_all(require_gpu(), _keys("strangers", 100_003), True, most=18_000)


@pytest.mark.parametrize("name,prefix", [("uniform", True), ("one_top_byte", False)])
@pytest.mark.parametrize("tiles", [511, 512])
def test_passes_left_out_before_their_tickets(tiles, name, prefix):
    """From 512 tiles on the lower passes read the plan before they take a ticket."""
    es = require_gpu()
    p = es.default_params(algo=es.ALGO_RADIX, block_threads=256, items_per_thread=8)
    _run_all(es, _keys(name, tiles * 2048), prefix, params=p)

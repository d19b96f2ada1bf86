"""The plan tells where a splitter sort runs instead of the routine of its branch, and a caller's own T_numpy or
T_ins keeps the routine that Algorithm 6 gives for it (Sec. 4.3)."""
import numpy as np
import pytest

import oracle
import workloads

# lengths of the splitter sort by (key bytes, value or index bytes)
RANGE = {(4, 0): (8_193, 400_000), (4, 4): (8_193, 262_144), (4, 8): (8_193, 262_144),
         (8, 0): (4_097, 262_144), (8, 4): (4_097, 262_144), (8, 8): (4_097, 262_144)}


def _es():
    return pytest.importorskip("paper_2505_18681_amd")


@pytest.mark.parametrize("kb,vb", RANGE)
def test_plan_names_the_splitter_sort(kb, vb):
    es = _es()
    code = {4: es.INT32, 8: es.FLOAT64}[kb]
    low, high = RANGE[kb, vb]
    for op in ([es.OP_SORT] if vb == 0 else [es.OP_SORT_PAIRS, es.OP_ARGSORT]):
        for n in (low, high):
            assert es.plan(op, code, n, vb)["split_blocks"] == -(-n // (512 if n <= 131_072 else 1024
                                                                        if n <= 262_144 else 2048))
        for n in (0, 1, low - 1, high + 1):
            assert es.plan(op, code, n, vb)["split_blocks"] == 0
        for params in (dict(algo=es.ALGO_RADIX), dict(algo=es.ALGO_MERGE), dict(digit_bits=7),
                       dict(block_threads=512, items_per_thread=8), dict(debug_flags=es.DEBUG_WIDE_STATUS)):
            assert es.plan(op, code, low, vb, es.default_params(**params))["split_blocks"] == 0, params


# (value bytes, caller's thresholds, length, routine of Algorithm 6 for them)
OWN = [(0, dict(fallback_threshold=1 << 14 | 1), 10_000, "small"), (0, dict(fallback_threshold=9_000), 10_000, "radix"),
       (0, dict(fallback_threshold=0), 10_000, "radix"), (4, dict(fallback_threshold=9_000), 10_000, "radix"),
       (0, dict(insertion_threshold=64), 10_000, "small"), (8, dict(insertion_threshold=64), 100_000, "radix")]


@pytest.mark.parametrize("vb,own,n,routine", OWN)
def test_own_thresholds_decide(vb, own, n, routine):
    es = _es()
    op = es.OP_SORT_PAIRS if vb else es.OP_SORT
    info = es.plan(op, es.INT32, n, vb, es.default_params(**own))
    assert (info["split_blocks"], info["path_name"]) == (0, routine)
    assert es.plan(op, es.INT32, n, vb, es.default_params())["split_blocks"] > 0


def test_own_thresholds_leave_the_choice_to_the_table():
    es = _es()
    from paper_2505_18681_amd import tuner

    for name, n, _lo, _hi, _algo in tuner.auto_table_rows(tuner.packaged_table()):
        for own in (dict(fallback_threshold=0), dict(insertion_threshold=64)):
            info = es.plan(es.OP_SORT, tuner.DTYPE_CODES[name], n, 0, es.default_params(**own))
            assert (info["split_blocks"], info["path_name"]) == (0, "merge"), (name, n, own)


def _ran(es, call):
    es.profile_reset()
    es.profile_enable(True)
    try:
        call()
        return set(es.profile_collect())
    finally:
        es.profile_enable(False)


KERNEL = {"small": "small_sort", "radix": "radix_pass", "merge": "merge_round"}


@pytest.mark.gpu
@pytest.mark.parametrize("vb,own,n,routine", OWN)
def test_own_thresholds_run_their_routine(vb, own, n, routine):
    from gpu_util import assert_bits_equal, require_gpu, to_dev, to_np

    es = require_gpu()
    keys = workloads.uniform(np.int32, n, n)
    keys[::7] = keys[3]
    perm = oracle.stable_perm(keys)
    p = es.default_params(**own)
    out = []
    if vb:
        vals = np.arange(n, dtype=np.int32 if vb == 4 else np.int64)
        names = _ran(es, lambda: out.extend(es.sort_pairs(to_dev(keys), to_dev(vals), params=p, check=True)))
        assert_bits_equal(to_np(out[1]), vals[perm], "values")
    else:
        names = _ran(es, lambda: out.append(es.sort(to_dev(keys), params=p, check=True)))
    assert KERNEL[routine] in names and "split_buckets" not in names, names
    assert_bits_equal(to_np(out[0]), keys[perm], "keys")


@pytest.mark.gpu
def test_table_rows_run_the_mergesort():
    """Every row of the compiled table, at both ends of its range, where the caller's T_numpy leaves it the choice."""
    from gpu_util import assert_bits_equal, require_gpu, to_dev, to_np
    from paper_2505_18681_amd import tuner

    es = require_gpu()
    p = es.default_params(fallback_threshold=0)
    for name, _n, lo, hi, _algo in tuner.auto_table_rows(tuner.packaged_table()):
        for m in (lo, hi - 1):
            keys = workloads.uniform(np.dtype(name), m, m)
            out = []
            names = _ran(es, lambda: out.append(es.sort(to_dev(keys), params=p, check=True)))
            assert "merge_round" in names and "split_buckets" not in names, (name, m, names)
            assert_bits_equal(to_np(out[0]), oracle.sort(keys), f"{name} {m}")

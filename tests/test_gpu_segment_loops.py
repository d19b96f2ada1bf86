"""Batches with several times more short segments of a class than waves or workgroups fit on the GPU: each of them
sorts segments of changing lengths in turn, through the same LDS buffer, for every record size and in place."""
import numpy as np
import pytest

import oracle
import workloads
from gpu_util import assert_bits_equal, require_gpu, to_dev, to_np

pytestmark = pytest.mark.gpu

# a CU holds 32 waves, the GPU 256 CUs: at most 8192 segments of class 0 (a wave each) are sorted at once, 2048 of
# class 1 (four waves), 1024 of class 2 (eight or more) and 512 of class 3 (sixteen)
CLASSES = [(3 * 8192 + 5, [1, 2, 63, 64, 65, 127, 128, 129, 255, 256, 257, 400, 511, 512]),
           (3 * 2048 + 5, [513, 700, 1023, 1024, 1025, 1500, 2047, 2048]),
           (3 * 1024 + 5, [2049, 3000, 4095, 4096, 4097, 6000, 8191, 8192]),
           (3 * 512 + 5, [8193, 12_000, 16_000, 16_383])]


# records of 8 bytes and more have three classes
@pytest.mark.parametrize("kb,vb,cls", [(kb, vb, c) for kb in (4, 8) for vb in (0, 4, 8)
                                       for c in range(4 if kb + vb == 4 else 3)])
def test_segments_in_turn(kb, vb, cls):
    import torch

    es = require_gpu()
    count, lengths = CLASSES[cls]
    if kb + vb > 8:
        lengths = [n for n in lengths if n <= 4096]
    g = workloads.rng(cls)
    sizes = np.array(lengths, dtype=np.int64)[g.integers(0, len(lengths), count)]
    offs = workloads.segment_offsets(sizes)
    n = int(offs[-1])
    dt = np.int32 if kb == 4 else np.int64
    keys = workloads.uniform(dt, n, 7)
    keys[::3] = np.iinfo(dt).max  # ties, and the word short records are filled up with
    code = es.INT32 if kb == 4 else es.INT64
    tmp = torch.empty(es.segmented_temp_bytes(code, n, count, vb), dtype=torch.uint8, device="cuda")
    k = to_dev(keys)
    if vb:
        vals = np.arange(n, dtype=np.int32 if vb == 4 else np.int64)
        v = to_dev(vals)
        es.segmented_sort_pairs(k, v, to_dev(offs), keys_out=k, values_out=v, temp=tmp, check=True)
        want, want_v = oracle.segmented_sort_pairs(keys, vals, offs)
        assert_bits_equal(to_np(v), want_v, "values")
    else:
        es.segmented_sort(k, to_dev(offs), out=k, temp=tmp, check=True)
        want = oracle.segmented_sort(keys, offs)
    assert_bits_equal(to_np(k), want, "keys")
    assert es.segmented_stats(tmp)["block_classes"][cls] == count

"""One captured radix sort replayed over inputs whose plans differ (Sec. 4, Algorithm 4): the launch sequence is the
same, and what the launches do is chosen on the device by every replay.  4-byte keys with 0, 1, 2, 3 and 4 live passes;
8-byte keys that alternate between a prefix sort with short runs, one with a long run out of order (its list and marks
lie in pass 0's look-back words), all passes, one live pass and none.  Eager sorts run between the replays."""
import numpy as np
import pytest

import oracle
from gpu_util import assert_bits_equal, require_gpu, to_np

pytestmark = pytest.mark.gpu

N = 100_003  # a ragged last tile


def _int32(name):
    g = np.random.default_rng(5)
    r = g.integers(0, 2**32, N, dtype=np.uint64)
    return {"none": np.full(N, -7, np.int32), "byte2": ((r & 0xFF) << 16).astype(np.int32),
            "bytes0and3": ((r & 0xFF) | ((r >> 8 & 0x3) << 24)).astype(np.uint32).view(np.int32),
            "low24": (r & 0xFFFFFF).astype(np.int32), "all": r.astype(np.uint32).view(np.int32)}[name]


def _int64(name):
    g = np.random.default_rng(6)
    u = g.integers(0, 2**64, N, dtype=np.uint64)
    if name == "long_run":  # a fifth of the keys are one value, with strangers in its run of equal upper digits
        u[g.random(N) < 0.2] = np.uint64(77)
        u[[1, N // 3, N // 2, N - 2]] = np.array([5, 99, 70, 80], dtype=np.uint64)
    elif name == "low16":
        u &= np.uint64(0xFFFF)
    elif name == "byte5":
        u = (u & np.uint64(0xFF)) << np.uint64(40)
    elif name == "none":
        u[:] = 12345
    return u.view(np.int64)


# pattern -> whether its plan is a prefix sort
INT32 = {"none": False, "byte2": False, "bytes0and3": False, "low24": False, "all": False}
INT64 = {"uniform": True, "long_run": True, "low16": False, "byte5": False, "none": False}
ORDER = {np.int32: ["none", "all", "byte2", "low24", "none", "bytes0and3", "all"],
         np.int64: ["none", "long_run", "uniform", "long_run", "low16", "uniform", "none", "byte5", "long_run"]}


@pytest.mark.parametrize("op", ["keys", "keys in place", "pairs", "pairs in place", "argsort"])
@pytest.mark.parametrize("dt", [np.int32, np.int64])
def test_replays_choose_their_plan(dt, op):
    import torch

    es = require_gpu()
    make, prefix = (_int32, INT32) if dt == np.int32 else (_int64, INT64)
    p = es.default_params(algo=es.ALGO_RADIX, fallback_threshold=0)
    keys = torch.empty(N, dtype=torch.int32 if dt == np.int32 else torch.int64, device="cuda")
    vals = torch.empty(N, dtype=torch.int64, device="cuda")
    in_place = op.endswith("in place")
    out_k, out_v = (keys, vals) if in_place else (torch.empty_like(keys), torch.empty_like(vals))
    code = es.dtype_code(keys.dtype)
    opc, vb = {"k": (es.OP_SORT, 0), "p": (es.OP_SORT_PAIRS, 8), "a": (es.OP_ARGSORT, 8)}[op[0]]
    tmp = torch.empty(es.temp_bytes(opc, code, N, vb, p), dtype=torch.uint8, device="cuda")

    def call():
        if opc == es.OP_SORT:
            es.sort(keys, params=p, out=out_k, temp=tmp)
        elif opc == es.OP_SORT_PAIRS:
            es.sort_pairs(keys, vals, params=p, keys_out=out_k, values_out=out_v, temp=tmp)
        else:
            es.argsort(keys, params=p, out=out_v, temp=tmp)

    def fill(name):
        host, hv = make(name), np.arange(N, dtype=np.int64) * 3 - 5
        host[::9] = host[4]
        keys.copy_(torch.from_numpy(host))
        vals.copy_(torch.from_numpy(hv))
        return host, hv

    def check(name, host, hv, what):
        perm = oracle.stable_perm(host)
        if opc != es.OP_ARGSORT:
            assert_bits_equal(to_np(out_k), host[perm], f"{what} {name}: keys")
        if opc != es.OP_SORT:
            assert_bits_equal(to_np(out_v), hv[perm] if opc == es.OP_SORT_PAIRS else perm, f"{what} {name}: values")
        assert (int(tmp[25].item()) > 0) == prefix[name], f"{what} {name}: plan"
        assert es.check_device_error(tmp) == es.OK

    host, hv = fill(ORDER[dt][1])
    es.profile_reset()
    es.profile_enable(True)
    try:
        call()
        names = es.profile_collect()
    finally:
        es.profile_enable(False)
    assert "radix_pass" in names and "split_buckets" not in names, names
    check(ORDER[dt][1], host, hv, "eager")
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=side):
        call()
    for i, name in enumerate(ORDER[dt]):
        host, hv = fill(name)
        graph.replay()
        torch.cuda.synchronize()
        check(name, host, hv, f"replay {i}")
        if i % 2:  # eager work between replays, on the same scratch
            other = ORDER[dt][i - 1]
            host, hv = fill(other)
            call()
            check(other, host, hv, f"eager after replay {i}")

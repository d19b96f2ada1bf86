"""The calls a user of the sort library makes, as cases that can be timed.

A case is a dict of plain values.  ``prepare`` makes on the GPU what a program has before the call (keys, values,
segment offsets, a server); ``run`` is one pass through the public entry points; ``work`` counts what the call cannot
do without: every input read once and every output written once.  ``draw`` gives further cases of the same ranges.

Kinds: ``sort``, ``pairs`` and ``argsort`` (one array), ``batch`` and ``batch_pairs`` (segments of one buffer),
``merge`` (the mergesort, chosen by the caller) and ``serve`` (a burst of requests to a sort server).
Inputs follow the recipes of ``workloads`` (uniform over every bit pattern; the paper's distributions on
[-1e9, 1e9], widened for 8-byte keys), drawn on the GPU.
"""
import math

import torch

import paper_2505_18681_amd as es

_DTYPES = {"int32": torch.int32, "uint32": torch.uint32, "float32": torch.float32, "int64": torch.int64,
           "float64": torch.float64}
_KEY_BYTES = {"int32": 4, "uint32": 4, "float32": 4, "int64": 8, "float64": 8}
_INT_DISTS = ("uniform", "normal", "exponential", "sparse", "clustered", "nearly_sorted", "duplicates", "zipf")
_FLOAT_DISTS = ("float_mix", "exponential", "nearly_sorted", "duplicates")
# one sort moves about n * (key + value bytes) bytes per digit, and has one digit per key byte; the largest
# listed single array (1e9 int32 keys) is the bound of the drawn ones
_MOST = 4 * 4 * 10**9


def listed():
    return [
        # a served request or a top-k candidate list: the smallest arrays, latency and launches only
        {"name": "sort_int32_1k", "kind": "sort", "dtype": "int32", "dist": "uniform", "n": 1000, "desc": False},
        # the largest array below the fallback threshold
        {"name": "sort_int32_16383", "kind": "sort", "dtype": "int32", "dist": "uniform", "n": 16383, "desc": False},
        # ranking the scores of one model output or query: float keys, 64-bit positions
        {"name": "argsort_float32_100k", "kind": "argsort", "dtype": "float32", "dist": "float_mix", "n": 100_003,
         "vb": 8, "desc": False},
        # a mid-size table column with row numbers, the everyday call
        {"name": "pairs_int32_1m", "kind": "pairs", "dtype": "int32", "dist": "uniform", "n": 1_000_003, "vb": 4,
         "desc": False},
        # one of the paper's distributions at the paper's smallest size, descending
        {"name": "sort_int32_10m_desc", "kind": "sort", "dtype": "int32", "dist": "normal", "n": 10_000_000,
         "desc": True},
        # grouping rows by a 64-bit key with many repeats
        {"name": "argsort_int64_10m", "kind": "argsort", "dtype": "int64", "dist": "duplicates", "n": 10_000_019,
         "vb": 8, "desc": False},
        # float64 measurements with a 64-bit payload
        {"name": "pairs_float64_30m", "kind": "pairs", "dtype": "float64", "dist": "float_mix", "n": 30_000_001,
         "vb": 8, "desc": False},
        # data that is almost in order already (the paper's nearly sorted array)
        {"name": "sort_int32_100m_nearly", "kind": "sort", "dtype": "int32", "dist": "nearly_sorted",
         "n": 100_000_000, "desc": False},
        # the benchmark's sort
        {"name": "sort_int32_1g", "kind": "sort", "dtype": "int32", "dist": "uniform", "n": 1_000_000_000,
         "desc": False},
        # the paper's mergesort, asked for by the caller
        {"name": "merge_int32_100m", "kind": "merge", "dtype": "int32", "dist": "uniform", "n": 100_000_000,
         "desc": False},
        # the benchmark's batch: 100k arrays of log-normal sizes
        {"name": "batch_uint32_100k", "kind": "batch", "dtype": "uint32", "dist": "uniform", "nseg": 100_000,
         "median": 2048.0, "sigma": 2.0, "most": 4_000_000, "desc": False},
        # a burst of requests to the server
        {"name": "serve_48", "kind": "serve", "requests": 48, "low": 1000, "high": 1_000_000},
    ]


def _log_uniform(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(("sort", "sort", "sort", "pairs", "pairs", "argsort", "argsort", "batch", "batch_pairs",
                       "merge", "serve"))
    if kind == "serve":
        low = _log_uniform(rng, 100, 10_000)
        return {"kind": kind, "requests": rng.randint(8, 60), "low": low, "high": low * _log_uniform(rng, 4, 1000)}
    dtype = rng.choice(("int32", "int32", "uint32", "float32", "int64", "float64"))
    kb = _KEY_BYTES[dtype]
    case = {"kind": kind, "dtype": dtype,
            "dist": rng.choice(_FLOAT_DISTS if dtype.startswith("float") else _INT_DISTS),
            "desc": rng.random() < 0.25}
    if kind in ("pairs", "argsort", "batch_pairs"):
        case["vb"] = rng.choice((4, 8))
    most = _MOST // (kb * (kb + case.get("vb", 0)))
    if kind.startswith("batch"):
        case["median"] = float(_log_uniform(rng, 100, 20_000))
        case["sigma"] = round(rng.uniform(0.3, 2.0), 2)
        case["most"] = 4_000_000
        mean = min(case["median"] * math.exp(case["sigma"] ** 2 / 2), case["most"])
        case["nseg"] = _log_uniform(rng, 50, min(100_000, most / (1.5 * mean)))
    else:
        case["n"] = _log_uniform(rng, 200, most if kind != "merge" else most // 10)
    return case


def _generator(seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    return g


def _keys(dtype, dist, n, g):
    """n keys of a dtype: `dist` as in `workloads`, values spread over the dtype's usual range."""
    t = _DTYPES[dtype]
    if dist == "uniform":
        if dtype == "int64":
            lo, hi, draw_as = -2**63, 2**63 - 1, torch.int64
        else:
            lo, hi, draw_as = -2**31, 2**31, torch.int32
        return torch.randint(lo, hi, (n,), generator=g, device="cuda", dtype=draw_as).view(t)
    if dist == "float_mix":
        x = torch.randn(n, generator=g, device="cuda", dtype=t)
        special = torch.tensor([-math.inf, math.inf, -0.0, 0.0], device="cuda", dtype=t)
        r = torch.rand(n, generator=g, device="cuda")
        return torch.where(r < 0.01, special[(r * 400).to(torch.int64).clamp_(max=3)], x)
    lim = 1e9 if _KEY_BYTES[dtype] == 4 else 1e18
    real = torch.float32 if n > 10**8 else torch.float64

    def uniform(k):
        return (torch.rand(k, generator=g, device="cuda", dtype=real) * 2 - 1) * lim

    if dist == "normal":
        x = torch.randn(n, generator=g, device="cuda", dtype=real) * (lim / 10)
    elif dist == "exponential":
        x = torch.empty(n, device="cuda", dtype=real).exponential_(1.0, generator=g) * lim - lim
    elif dist == "sparse":
        x = uniform(n) * (torch.rand(n, generator=g, device="cuda") < 0.1)
    elif dist == "clustered":
        centre = torch.randint(0, 10, (n,), generator=g, device="cuda").to(real) * (2 * lim / 9) - lim
        x = centre + torch.randn(n, generator=g, device="cuda", dtype=real) * (lim / 10)
    elif dist == "nearly_sorted":
        x = torch.linspace(-lim, lim, n, device="cuda", dtype=real)
        x = torch.where(torch.rand(n, generator=g, device="cuda") < 0.1, uniform(n), x)
    elif dist == "duplicates":
        few = uniform(max(1, n // 10))
        x = few[torch.randint(0, few.numel(), (n,), generator=g, device="cuda")]
    elif dist == "zipf":
        weight = torch.arange(1, 1_000_001, device="cuda", dtype=torch.float64) ** -1.1
        cdf = torch.cumsum(weight, 0)
        x = torch.searchsorted((cdf / cdf[-1]).to(real), torch.rand(n, generator=g, device="cuda", dtype=real))
    else:
        raise ValueError(dist)
    if dtype.startswith("float"):
        return x.to(t)
    if x.is_floating_point():
        x = x.clamp_(-lim, lim)
    return x.to(torch.int64 if dtype == "int64" else torch.int32).view(t)


def _sizes(case, g):
    z = torch.randn(case["nseg"], generator=g, device="cuda", dtype=torch.float64)
    sizes = torch.exp(z * case["sigma"] + math.log(case["median"])).round_()
    return sizes.clamp_(16, case["most"]).to(torch.int64)


def prepare(case, seed):
    g = _generator(seed)
    kind = case["kind"]
    if kind == "serve":
        span = math.log(case["high"] / case["low"])
        # every seed has the case's request sizes, as below
        r = torch.rand(case["requests"], generator=_generator(42), device="cuda", dtype=torch.float64)
        sizes = (case["low"] * torch.exp(r * span)).round().to(torch.int64).tolist()
        types = ("int32", "int64", "float32")
        keys = [_keys(types[i % 3], "float_mix" if i % 3 == 2 else "uniform", n, g) for i, n in enumerate(sizes)]
        return {"kind": kind, "server": es.Server(hbm_budget_bytes=4 << 30), "keys": keys}
    state = {"kind": kind, "index_dtype": torch.int32 if case.get("vb") == 4 else torch.int64,
             "params": es.default_params(descending=1) if case["desc"] else None}
    n = case.get("n")
    if kind.startswith("batch"):
        # every seed has the case's number of keys: segment sizes come from one seed, keys from the given one
        sizes = _sizes(case, _generator(42))
        state["offsets"] = torch.cat([sizes.new_zeros(1), torch.cumsum(sizes, 0)])
        n = int(state["offsets"][-1])
    state["keys"] = _keys(case["dtype"], case["dist"], n, g)
    if kind in ("pairs", "batch_pairs"):
        state["values"] = torch.arange(n, device="cuda", dtype=state["index_dtype"])
    if kind == "merge":
        state["params"] = es.default_params(algo=es.ALGO_MERGE, descending=int(case["desc"]))
    return state


def _numbers(t):
    # torch has few operations for uint32: the same bits as int32
    return t.view(torch.int32) if t.dtype == torch.uint32 else t


def run(state):
    kind = state["kind"]
    if kind == "serve":
        server = state["server"]
        ids = [server.submit(k) for k in state["keys"]]
        out = [server.result(i) for i in ids]
        for i in ids:
            server.release(i)
        return out
    keys, params = state["keys"], state["params"]
    if kind in ("sort", "merge"):
        return _numbers(es.sort(keys, params=params))
    if kind == "pairs":
        k, v = es.sort_pairs(keys, state["values"], params=params)
        return _numbers(k), v
    if kind == "argsort":
        return es.argsort(keys, index_dtype=state["index_dtype"], params=params)
    if kind == "batch":
        return _numbers(es.segmented_sort(keys, state["offsets"], params=params))
    k, v = es.segmented_sort_pairs(keys, state["values"], state["offsets"], params=params)
    return _numbers(k), v


def _keys_of(case):
    if "n" in case:
        return case["n"]
    # the segment sizes are the same on every seed; their expected sum is near enough for counting bytes
    m, s, top = math.log(case["median"]), case["sigma"], math.log(case["most"])

    def below(x):
        return 0.5 * (1 + math.erf(x / math.sqrt(2)))

    mean = math.exp(m + s * s / 2) * below((top - m - s * s) / s) + case["most"] * (1 - below((top - m) / s))
    return int(case["nseg"] * max(mean, 16))


def work(case):
    if case["kind"] == "serve":
        span = math.log(case["high"] / case["low"])
        mean = (case["high"] - case["low"]) / span
        return {"bytes": 2 * case["requests"] * mean * (4 + 8 + 4) / 3, "flops": 0}
    n, kb, vb = _keys_of(case), _KEY_BYTES[case["dtype"]], case.get("vb", 0)
    # an argsort reads keys and writes indices; everything else reads and writes keys and values
    return {"bytes": n * (kb + vb) if case["kind"] == "argsort" else 2 * n * (kb + vb), "flops": 0}


def exact(case, seed):
    """Sorted float keys in 64 bits; None for whole numbers (their bytes are the answer) and for the largest."""
    if case["kind"] == "serve" or not case["dtype"].startswith("float") or case["kind"] == "argsort":
        return None
    if _keys_of(case) > 40_000_000:
        return None
    state = prepare(case, seed)
    keys = state["keys"].double().cpu()
    bounds = state["offsets"].tolist() if "offsets" in state else [0, keys.numel()]
    desc = case["desc"]
    out = torch.cat([torch.sort(keys[a:b], descending=desc).values for a, b in zip(bounds, bounds[1:])])
    return (out, None) if "values" in state else out

"""The plan tells where a splitter sort runs instead of the routine of its branch (host only)."""
import pytest

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

"""The installed table of launch shapes (tuned_shapes.json), without a GPU."""
import json

import pytest

from paper_1801_07986_amd import _binding

FP64, MIXED = _binding.PN_FP64, _binding.PN_MIXED


@pytest.fixture(scope="module")
def lib():
    import paper_1801_07986_amd as pn

    pn.load()
    _binding.install_tuned_shapes()
    return pn


@pytest.fixture(scope="module")
def table():
    with open(_binding.TUNED_PATH) as f:
        return json.load(f)


@pytest.mark.parametrize("precision", [FP64, MIXED])
def test_one_launch_stages_only_where_they_win(lib, precision):
    """Up to 2049 bodies: beyond, the chained stages are faster (FP64, us per step,
    one-launch stages of 16 stars and chained: N = 2400 94 and 79, 2739 106 and
    91, 3000 113 and 96, 3505 128 and 115)."""
    for N in (2, 100, 513, 1025, 2049):
        assert lib.pn_query_stage_kernel(precision, N) > 0, N
    for N in (2050, 2400, 2738, 2739, 3000, 3505, 3506, 16384):
        assert lib.pn_query_stage_kernel(precision, N) == 0, N


def test_stage_rows_hold_a_win(table):
    """The autotuner's margin between the two forms: 3 %."""
    for e in table["stage"]:
        assert e["step_ms"] <= 0.97 * e["chain_step_ms"], e


def test_bench_knows_the_timed_kernels(lib):
    """bench.py's measured HBM traffic is for the kernels and split counts that the
    table selects, and a small system's kernel is the one-launch stage."""
    import os
    import sys

    sys.path.insert(0, os.path.dirname(os.path.dirname(os.path.abspath(__file__))))
    import bench

    for name, prec, N in (("plummer_n16384_fp64", FP64, 16384),
                          ("plummer_n65536_mixed", MIXED, 65536)):
        assert (name, *bench.sweep_kernel(lib, prec, N)) in bench.TRAFFIC_BYTES
    assert bench.sweep_kernel(lib, FP64, 1024) == ("k_stage<double,4,false>", 1)
    assert bench.sweep_kernel(lib, FP64, 100) == ("k_stage<double,2,true>", 1)

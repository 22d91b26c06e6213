"""The roofline record of bench.py where the inner solver runs the wave hop."""
import os
import sys

import pytest

sys.path.insert(0, os.path.dirname(os.path.dirname(os.path.abspath(__file__))))
sys.path.insert(0, os.path.dirname(os.path.abspath(__file__)))
import bench  # noqa: E402
from test_bench_record import DIMS, HOP_US, L, LS, S, TUNING, VH, kern_record  # noqa: E402


def tuning(us):
    """As the autotuner reports it: every tile of the sweeps with the time given for it."""
    t = {p: dict(v) for p, v in TUNING.items()}
    t["bf16"]["candidates"] = [[ns, o, "sweep", u] for ns, o, u in us] + [[8, "slab", "dense", 390.0]]
    return t


def test_wave_pair_is_the_record_of_a_solve_that_runs_it():
    t = tuning([(8, "slab", 74.0), (16, "slab", 74.0), (32, "zdom", 74.0)])
    rec = bench.make_roofline(kern_record(HOP_US), t, "bf16", DIMS, LS, S, L, 6000.0)
    nbytes = 5 * S["bf16"] + 2 * L["bf16"]
    flops = VH * LS * (2 * 1320 + 3 * 4 * LS * 12)
    assert rec["kernel"].startswith("wave_hop_kernel<BF16>")
    assert rec["bound"] == "hbm" and rec["unit"] == "GB/s" and rec["peak"] == 8000.0
    assert rec["bytes_per_pair"] == nbytes
    assert rec["frac"] == pytest.approx(nbytes / 74e-6 / 8e12, rel=1e-3)
    assert rec["mfma"]["achieved_tflops"] == pytest.approx(flops / 74e-6 / 1e12, rel=1e-3)
    assert set(rec["per_precision"]) == {"f64", "f32", "bf16"}
    # the site-block hop, which D_bb of larger calls runs, beside it
    plain = bench.make_roofline(kern_record(HOP_US), TUNING, "bf16", DIMS, LS, S, L, 6000.0)
    assert rec["site_block_hop"] == {k: v for k, v in plain.items() if k != "per_precision"}


def test_tiles_of_different_times_are_the_site_block_hop():
    t = tuning([(8, "slab", 80.0), (16, "slab", 74.0), (32, "zdom", 76.0)])
    rec = bench.make_roofline(kern_record(HOP_US), t, "bf16", DIMS, LS, S, L)
    assert rec["kernel"].startswith("hop_mix_kernel") and "site_block_hop" not in rec


def test_committed_wave_counters_match_the_kernel_source():
    # more than the algorithmic bytes (the links come gathered, twice), less than twice
    nbytes = 5 * S["bf16"] + 2 * L["bf16"]
    assert nbytes < bench.measured_wave_traffic("bf16") < 2 * nbytes
    assert bench.measured_wave_traffic("f32") is None


def test_hop_counters_do_not_move_with_the_updates():
    """The hop's source is what precedes the site-local kernels, which hold the CG updates."""
    assert bench._kernel_sha() != bench._source_sha("kcommon.h")
    assert bench._source_sha("kcommon.h", b"#define DWA_SITE_THREAD") == bench._kernel_sha()

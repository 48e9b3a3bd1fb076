"""Host-side tests of libee.so that need no GPU: the library loads and exports the C ABI,
argument validation, blob validation, the exp2 table, and the scheduler against the oracle."""
import ctypes as C
import os
import re
import subprocess
from decimal import Decimal, getcontext

import numpy as np
import pytest

import workloads as W

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.fixture(scope="module")
def ee():
    import paper_2209_13443_amd as ee
    return ee


def test_library_exports_every_declared_symbol(ee):
    header = open(os.path.join(ROOT, "include", "ee.h")).read()
    declared = set(re.findall(r"\b(ee_[a-z0-9_]+)\s*\(", header))
    assert declared, "no declarations found"
    lib = ee.raw()
    for name in sorted(declared):
        assert hasattr(lib, name), f"{name} declared in include/ee.h but not exported"
    assert set(ee.SYMBOLS) <= declared


def test_strerror(ee):
    assert ee.strerror(0) == "ok"
    assert "argument" in ee.strerror(ee.EE_ERR_ARG)
    assert ee.strerror(-99) == "unknown status"


def test_blob_check_matches_oracle_verdicts(ee, orc):
    for name in ("tiny_i8", "resnet50_small_i8", "mobilenetv2_small_i8", "tiny_bf16"):
        b = W.build_net(name)
        assert ee.blob_check(b.buffer()) == ee.EE_OK == orc.blob_check(b)
    b = W.build_net("tiny_i8")
    b.ops[1]["c_in"] = 17
    assert ee.blob_check(b.buffer()) == ee.EE_ERR_SHAPE
    b = W.build_net("tiny_i8")
    b.ops[2]["res"] = 0            # residual of the wrong shape
    assert ee.blob_check(b.buffer()) == ee.EE_ERR_SHAPE == orc.blob_check(b)
    b = W.build_net("tiny_i8")
    b.header[0]["dtype"] = 5
    assert ee.blob_check(b.buffer()) == ee.EE_ERR_UNSUPPORTED
    assert ee.blob_check(np.zeros(64, np.uint8)) == ee.EE_ERR_ARG
    junk = W.build_net("tiny_i8").buffer().copy()
    junk[:8] = 0
    assert ee.blob_check(junk) == ee.EE_ERR_ARG


def test_null_and_range_arguments_are_rejected_without_a_gpu(ee):
    lib = ee.raw()
    assert lib.ee_stage_forward(None, 0, 1, None, None) == ee.EE_ERR_ARG
    assert lib.ee_exit_head(None, 0, 1, None, 0.5, None, None, None, None) == ee.EE_ERR_ARG
    assert lib.ee_autotune(None, 3) == ee.EE_ERR_ARG
    assert lib.ee_config_table(None, 0, None, 0) == ee.EE_ERR_ARG
    assert lib.ee_pair_count(None) == ee.EE_ERR_ARG
    assert lib.ee_pair_mode(None, 1) == ee.EE_ERR_ARG
    assert lib.ee_pair_table(None, 0, None, 0) == ee.EE_ERR_ARG
    assert lib.ee_config_set(None, 0, None, 0) == ee.EE_ERR_ARG
    assert lib.ee_pair_set(None, 0, None, 0) == ee.EE_ERR_ARG
    assert lib.ee_compact_refill(None, 0, 1, None, None, None, None, None, None, None, 0, None, None) == ee.EE_ERR_ARG
    assert lib.ee_serve_stream(None, None, None, None, None, None, None, 0) == ee.EE_ERR_ARG
    assert lib.ee_query(None, None, None, None) == ee.EE_ERR_ARG
    assert lib.ee_measure_lut(None, 1, None) == ee.EE_ERR_ARG
    assert lib.ee_destroy(None) == ee.EE_OK
    h = C.c_void_p()
    blob = W.build_net("tiny_i8").buffer()
    assert lib.ee_create(blob.ctypes.data, blob.size, 0, 0, None, C.byref(h)) == ee.EE_ERR_ARG       # b_max = 0
    assert lib.ee_create(blob.ctypes.data, blob.size, 8, 1, None, C.byref(h)) == ee.EE_ERR_UNSUPPORTED  # dtype mismatch
    assert lib.ee_create(blob.ctypes.data, 100, 8, 0, None, C.byref(h)) == ee.EE_ERR_ARG             # truncated


def test_exp2_table(ee, orc):
    getcontext().prec = 60
    ln2 = Decimal(2).ln()
    t = ee.exp2_table()
    for i in range(256):
        exact = (Decimal(2) ** 30) * (-(Decimal(i) / 256) * ln2).exp()
        assert int(t[i]) == int(exact.to_integral_value(rounding="ROUND_HALF_EVEN"))
    assert np.array_equal(t, orc.exp2_table())


def _case(seed, n=400, n_stages=4, b_max=8, rate=0.02):
    rng = np.random.default_rng(seed)
    arrivals = np.floor(np.cumsum(rng.exponential(1.0 / rate, size=n))).astype(np.int64)
    forced = rng.integers(0, n_stages, size=n).astype(np.int32)
    lut = (rng.integers(40, 120, size=(n_stages, 1)) + np.arange(b_max)[None, :] * rng.integers(0, 9, size=(n_stages, 1))).astype(np.int64)
    return arrivals, forced, lut


@pytest.mark.parametrize("seed", range(8))
def test_scheduler_matches_oracle_bit_for_bit(ee, orc, seed):
    b_max = [8, 8, 3, 64, 1, 16, 8, 8][seed]
    arrivals, forced, lut = _case(seed, b_max=b_max, rate=[0.02, 0.2, 0.05, 0.5, 0.01, 0.1, 0.02, 0.02][seed])
    slo = [-1, -1, 700, 2000, -1, 900, 0, 400][seed]
    min_incr = [1, 1, 1, 4, 1, 2, 1, 1][seed]
    refill = 0 if seed == 4 else 1
    a, sa, ea = orc.serve_stream(None, arrivals, None, b_max, lut, t_slo_ns=slo, min_incr=min_incr, refill=refill,
                                 forced_exit=forced, n_stages=4, max_events=20000)
    b, sb, eb = ee.schedule_sim(4, arrivals, forced, b_max, lut, t_slo_ns=slo, min_incr=min_incr, refill=refill, max_events=20000)
    assert sa == sb
    assert np.array_equal(ea, eb)
    for f in ("exit_idx", "latency_ns"):
        assert np.array_equal(a[f], b[f])


@pytest.mark.parametrize("seed", range(8))
def test_stage_pool_scheduler_matches_oracle_bit_for_bit(ee, orc, seed):
    b_max = [8, 8, 3, 64, 1, 16, 8, 2][seed]
    arrivals, forced, lut = _case(100 + seed, b_max=b_max, rate=[0.02, 0.2, 0.05, 0.5, 0.01, 0.1, 0.03, 0.02][seed])
    if seed == 1:
        arrivals[:] = 0
    slo = [-1, -1, 700, 2000, -1, 900, 900, 400][seed]
    a, sa, ea = orc.serve_stream(None, arrivals, None, b_max, lut, t_slo_ns=slo, refill=2, forced_exit=forced, n_stages=4, max_events=20000)
    b, sb, eb = ee.schedule_sim(4, arrivals, forced, b_max, lut, t_slo_ns=slo, refill=2, max_events=20000)
    assert sa == sb
    assert np.array_equal(ea, eb)
    for f in ("exit_idx", "latency_ns"):
        assert np.array_equal(a[f], b[f])
    if slo >= 0:
        assert sa["preemptions"] > 0                                 # the SLO rule is exercised


def test_scheduler_argument_errors(ee):
    arrivals, forced, lut = _case(0)
    bad = arrivals.copy()
    bad[5] = bad[4] - 1
    with pytest.raises(ee.EEError) as e:
        ee.schedule_sim(4, bad, forced, 8, lut)
    assert e.value.code == ee.EE_ERR_ARG
    res, st, _ = ee.schedule_sim(4, arrivals[:0], forced[:0], 8, lut)
    assert res.size == 0 and st["rounds"] == 0
    with pytest.raises(ee.EEError) as e:
        ee.schedule_sim(4, arrivals, forced, 8, lut, refill=3)
    assert e.value.code == ee.EE_ERR_ARG


def test_timeline_example_through_the_library(ee):
    from test_oracle_sched import read_timeline
    events, samples = read_timeline()
    arrivals = np.array([0, 0, 5, 5, 5, 5, 15], np.int64)
    forced = np.array([s[1] - 1 for s in samples], np.int32)
    res, st, ev = ee.schedule_sim(2, arrivals, forced, 8, np.full((2, 8), 10, np.int64), t_slo_ns=35, max_events=64)
    assert [(int(e["t_ns"]), int(e["kind"]), int(e["stage"]), int(e["b"]), int(e["aux"])) for e in ev] == events
    assert [int(r["latency_ns"] + a) for r, a in zip(res, arrivals)] == [s[2] for s in samples]


# ---- both schedulers against the oracle on generated cases ---------------------------------------------------
from hypothesis import given, settings, strategies as st


@settings(max_examples=120, deadline=None)
@given(seed=st.integers(0, 2**31 - 1), n=st.integers(1, 90), n_stages=st.integers(1, 5), b_max=st.integers(1, 12),
       refill=st.sampled_from([0, 1, 2]), slo_kind=st.sampled_from(["none", "tight", "loose"]), min_incr=st.integers(1, 6),
       burst=st.booleans())
def test_schedulers_match_oracle_on_generated_cases(ee, orc, seed, n, n_stages, b_max, refill, slo_kind, min_incr, burst):
    """Random traces (Poisson or everything at once), exits, latency tables and SLOs: results, statistics and the whole
    event log of the library's scheduler equal the oracle's, bit for bit, for all three policies."""
    rng = np.random.default_rng(seed)
    arrivals = np.zeros(n, np.int64) if burst else np.floor(np.cumsum(rng.exponential(rng.choice([5.0, 40.0, 300.0]), size=n))).astype(np.int64)
    forced = rng.integers(0, n_stages, size=n).astype(np.int32)
    lut = (rng.integers(20, 120, size=(n_stages, 1)) + np.arange(b_max)[None, :] * rng.integers(0, 9, size=(n_stages, 1))).astype(np.int64)
    total = int(lut[:, -1].sum())
    slo = {"none": -1, "tight": total // 2, "loose": 3 * total}[slo_kind]
    a, sa, ea = orc.serve_stream(None, arrivals, None, b_max, lut, t_slo_ns=slo, min_incr=min_incr, refill=refill,
                                 forced_exit=forced, n_stages=n_stages, max_events=8000)
    b, sb, eb = ee.schedule_sim(n_stages, arrivals, forced, b_max, lut, t_slo_ns=slo, min_incr=min_incr, refill=refill, max_events=8000)
    assert sa == sb
    assert np.array_equal(ea, eb)
    assert np.array_equal(a["exit_idx"], b["exit_idx"]) and np.array_equal(a["latency_ns"], b["latency_ns"])
    assert np.array_equal(a["exit_idx"], forced)


def test_random_networks_pass_both_parsers(ee, orc):
    """The generated networks of the parity fuzz test are valid for the oracle's parser and for the library's."""
    lib = ee._lib
    for dtype in (W.DT_I8, W.DT_BF16):
        for seed in range(30):
            blob = W.random_net(seed, dtype)
            buf = blob.buffer()
            assert orc.blob_check(blob) == orc.OK and lib.ee_blob_check(buf.ctypes.data, buf.size) == ee.EE_OK, (dtype, seed)


@pytest.mark.parametrize("lanes", [2, 3, 4])
@pytest.mark.parametrize("seed", range(8))
def test_stage_pools_with_several_steps_in_flight_match_oracle_bit_for_bit(ee, orc, seed, lanes):
    b_max = [8, 8, 3, 64, 1, 16, 8, 2][seed]
    arrivals, forced, lut = _case(200 + seed, b_max=b_max, rate=[0.02, 0.2, 0.05, 0.5, 0.01, 0.1, 0.03, 1.0][seed])
    if seed == 1:
        arrivals[:] = 0
    slo = [-1, -1, 700, 2000, -1, 900, 900, 400][seed]
    a, sa, ea = orc.serve_stream(None, arrivals, None, b_max, lut, t_slo_ns=slo, refill=2, lanes=lanes, forced_exit=forced, n_stages=4, max_events=20000)
    b, sb, eb = ee.schedule_sim(4, arrivals, forced, b_max, lut, t_slo_ns=slo, refill=2, lanes=lanes, max_events=20000)
    assert sa == sb
    assert np.array_equal(ea, eb)
    for f in ("exit_idx", "latency_ns"):
        assert np.array_equal(a[f], b[f])
    assert np.any(eb["aux"][eb["kind"] == 2] > 0) or b_max == 1 or seed in (0, 4)     # a second lane was used


def test_two_lane_timeline_through_the_library(ee):
    lut = np.array([[10 * (s + 1) + b for b in (1, 2)] for s in range(3)], np.int64)
    res, st, ev = ee.schedule_sim(3, np.zeros(6, np.int64), np.array([0, 1, 2, 2, 1, 0], np.int32), 2, lut, refill=2, lanes=2, max_events=64)
    assert res["latency_ns"].tolist() == [12, 46, 100, 100, 68, 36]
    assert [(int(e["t_ns"]), int(e["stage"]), int(e["b"]), int(e["aux"])) for e in ev[ev["kind"] == 2]] == \
        [(0, 0, 2, 0), (12, 0, 2, 0), (24, 1, 2, 0), (24, 0, 2, 1), (46, 1, 2, 0), (68, 2, 2, 0)]
    with pytest.raises(ee.EEError):
        ee.schedule_sim(3, np.zeros(6, np.int64), np.zeros(6, np.int32), 2, lut, refill=2, lanes=5)


@pytest.mark.parametrize("seed", range(6))
def test_adaptive_batching_and_serial_match_oracle_bit_for_bit(ee, orc, seed):
    b_max = [8, 8, 4, 1, 16, 8][seed]
    arrivals, forced, lut = _case(300 + seed, b_max=b_max, rate=[0.02, 0.2, 0.005, 0.01, 0.1, 0.05][seed])
    window = [300, 50, 5000, 100, 10**12, 1][seed]
    a, sa, ea = orc.serve_stream(None, arrivals, None, b_max, lut, refill=0, t_timeout_ns=window, forced_exit=forced, n_stages=4, max_events=20000)
    b, sb, eb = ee.schedule_sim(4, arrivals, forced, b_max, lut, refill=0, t_timeout_ns=window, max_events=20000)
    assert sa == sb and np.array_equal(ea, eb)
    for f in ("exit_idx", "latency_ns"):
        assert np.array_equal(a[f], b[f])


def test_adaptive_batching_timeline_through_the_library(ee):
    arrivals = np.array([0, 3, 50, 51, 52, 53, 54], np.int64)
    res, st, ev = ee.schedule_sim(2, arrivals, np.ones(7, np.int32), 4, np.full((2, 4), 10, np.int64), refill=0, t_timeout_ns=20, max_events=64)
    assert res["latency_ns"].tolist() == [40, 37, 23, 22, 21, 20, 40]
    assert [(int(e["t_ns"]), int(e["b"])) for e in ev[ev["kind"] == 1]] == [(20, 2), (53, 4), (74, 1)]


# Programs of the library's own launchers with the runtime's three calls in their place: the grant of more than 64 KB of LDS answers as told, a launch is only counted.
LAUNCH_PROGRAM = r"""
#include <cstdio>
#include <cstdlib>
#include "ee_internal.hpp"

static hipError_t grant = hipSuccess;
static int launches, lanes;
static size_t lds;
extern "C" hipError_t hipFuncSetAttribute(const void*, hipFuncAttribute, int) { return grant; }
extern "C" hipError_t hipGetLastError() { return hipSuccess; }      // what a failed call leaves has been fetched by somebody
extern "C" hipError_t hipExtLaunchKernel(const void*, dim3, dim3 block, void**, size_t bytes, hipStream_t, hipEvent_t, hipEvent_t, int)
{
    ++launches;
    lanes = (int)block.x;
    lds = bytes;
    return hipSuccess;
}
"""
IR_LAUNCH_PROGRAM = LAUNCH_PROGRAM + r"""
int main(int, char** argv)
{
    grant = (hipError_t)std::atoi(argv[1]);
    int pooled;
    ee::IrArgs a{};
    a.pad = 1;
    while (std::scanf("%d %d %d %d %d %d %d %d %d", &a.B, &a.H, &a.W, &a.Cin, &a.Kx, &a.Ce32, &a.Cout, &a.stride, &pooled) == 9) {
        a.Ho = (a.H + a.stride - 1) / a.stride;
        a.Wo = (a.W + a.stride - 1) / a.stride;
        a.gap_sums = pooled ? (int*)8 : nullptr;
        launches = 0;
        const int first = (int)ee::launch_ir_block(a, nullptr), second = (int)ee::launch_ir_block(a, nullptr);
        std::printf("%d %d %d %zu %d\n", first, second, launches, lds, lanes);
    }
}
"""
# samples, h, w, c_in, c_in in whole 32, expanded in whole 32, c_out, stride, pooled
IR_LAUNCHES = [(1, 14, 14, 96, 96, 576, 160, 2, 0), (2, 14, 14, 160, 160, 960, 160, 2, 0), (1, 7, 7, 160, 160, 960, 160, 1, 0), (1, 7, 7, 160, 160, 960, 160, 1, 1), (1, 28, 28, 32, 32, 192, 32, 1, 0)]


def launch_program(tmp_path, source):
    """Compiles the program against the library; returns run(calls, *arguments): a line of numbers in per call, a tuple of numbers out."""
    csrc = os.path.join(ROOT, "paper_2209_13443_amd", "csrc")
    libdir = os.path.dirname(csrc)
    (tmp_path / "launch.hip").write_text(source)
    exe = str(tmp_path / "launch")
    subprocess.run(["hipcc", "-x", "hip", "--offload-host-only", "-std=c++20", "-I", csrc, str(tmp_path / "launch.hip"), "-o", exe, "-L", libdir, "-lee", "-Wl,-rpath," + libdir], check=True, timeout=120)

    def run(calls, *arguments):
        lines = "".join(" ".join(map(str, c)) + "\n" for c in calls)
        out = subprocess.run([exe, *arguments], input=lines, capture_output=True, text=True, check=True, timeout=60, env={**os.environ, "HIP_VISIBLE_DEVICES": "-1"}).stdout
        return [tuple(map(int, line.split())) for line in out.splitlines()]
    return run


def test_inverted_residual_block_without_its_lds_is_an_error_every_time(ee, tmp_path):
    """A block that needs more than 64 KB of LDS and does not get them: every launch says so, not only the one that asked; and none of them goes out."""
    run = launch_program(tmp_path, IR_LAUNCH_PROGRAM)
    granted, refused = run(IR_LAUNCHES, "0"), run(IR_LAUNCHES, "1")
    large = [g[3] > 64 * 1024 for g in granted]
    assert all(g[:3] == (0, 0, 2) for g in granted) and any(large) and not all(large)
    for big, g, r in zip(large, granted, refused):
        assert r[:3] == ((1, 1, 0) if big else (0, 0, 2)), (g, r)


# h, w, c_in, c_in in whole 32, expanded in whole 32, c_out, stride, the most samples whose tiles the wavefronts share by channel groups: measured edges, and none beyond them
IR_SHARED_EDGES = [(14, 14, 64, 64, 384, 160, 1, 109), (14, 14, 96, 96, 576, 160, 2, 384), (7, 7, 160, 160, 960, 160, 1, 384), (28, 28, 32, 32, 192, 128, 1, 9),
                   (28, 28, 32, 32, 192, 160, 2, 36), (28, 28, 32, 32, 192, 64, 1, 18), (28, 28, 32, 32, 192, 96, 1, 18), (14, 14, 64, 64, 384, 64, 1, 128), (28, 28, 32, 32, 192, 64, 2, 36),
                   (28, 28, 32, 32, 192, 32, 1, 54)]


def test_channel_groups_are_shared_out_only_where_that_was_measured_to_be_faster(ee, tmp_path):
    """Workgroups of eight wavefronts up to the stated number of samples, and of four at any larger one up to 1024."""
    samples = (1, 5, 64, 128, 256, 400, 512, 700, 1024)
    calls = [(b, *shape, 0) for *shape, most in IR_SHARED_EDGES for b in sorted({most, most + 1, *samples})]
    most = [m for *_, m in IR_SHARED_EDGES for b in sorted({m, m + 1, *samples})]
    for (b, *shape, _), m, (first, _, launches, lds, lanes) in zip(calls, most, launch_program(tmp_path, IR_LAUNCH_PROGRAM)(calls, "0")):
        assert first == 0 and launches == 2 and lanes == (512 if b <= m else 256), (b, shape, lds, lanes)


GAP_LAUNCH_PROGRAM = LAUNCH_PROGRAM + r"""
int main()
{
    ee::HeadArgs a{};
    while (std::scanf("%d %d %d", &a.B, &a.HW, &a.C) == 3) {
        launches = 0;
        const int rc = (int)ee::launch_head_gap(a, EE_BF16, nullptr);
        std::printf("%d %d %d\n", rc, launches, ee::head_gap_splits(a.B, a.HW));
    }
}
"""


def test_partial_rows_are_counted_where_the_pooling_keeps_them(ee, tmp_path):
    """bf16 pooling: head_gap_splits, by which the head's scratch memory is sized, says more than one part exactly where a second launch adds partial rows up (which no pooling
    by slices of channels has), and never more rows than a lane's memory for them."""
    calls = [(b, hw, c) for b in (1, 5, 64, 200, 511, 512, 1024) for hw in (1, 15, 17, 49, 784, 4095, 4096, 4097, 112 * 112) for c in (8, 64, 2048)]
    for (b, hw, _), (rc, launches, splits) in zip(calls, launch_program(tmp_path, GAP_LAUNCH_PROGRAM)(calls)):
        assert rc == 0 and launches == (2 if splits > 1 else 1) and splits >= 1 and b * splits <= b + 1024, (b, hw, launches, splits)
        assert splits == 1 or hw > 4096

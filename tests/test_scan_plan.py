"""The rules by which a state scan chooses its launches (csrc/scan_plan.hpp), on the host."""
import ctypes
import os
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2506_05233_amd", "csrc")
WRAPPER = """
#include "scan_plan.hpp"
extern "C" int final_len(int64_t bh, int nc, int dk, int dv, size_t bytes) { return mesa::final_segment_len(bh, nc, dk, dv, bytes); }
extern "C" int wide_scan(int single, int64_t bh, int nc, int64_t elems) {
  const int S = mesa::wide_segments(bh, nc), len = int(mesa::ceil_div(nc, S));
  return mesa::wide_takes_scan(single != 0, bh, nc, elems, int(mesa::ceil_div(nc, len)), len);
}
extern "C" int f32_scan(int64_t bh, int nc, int dk, int dv) { return mesa::f32_takes_scan(bh, nc, dk, dv); }
"""


@pytest.fixture(scope="module")
def plan(tmp_path_factory):
    d = tmp_path_factory.mktemp("scan_plan")
    src, lib = d / "plan.cpp", d / "plan.so"
    src.write_text(WRAPPER)
    subprocess.run(["g++", "-std=c++17", "-O1", "-Wall", "-Werror", "-fPIC", "-shared", "-I" + CSRC, "-o", str(lib), str(src)],
                   check=True)
    p = ctypes.CDLL(str(lib))
    i64, ci, sz = ctypes.c_int64, ctypes.c_int, ctypes.c_size_t
    p.final_len.argtypes, p.final_len.restype = [i64, ci, ci, ci, sz], ci
    p.wide_scan.argtypes, p.wide_scan.restype = [ci, i64, ci, i64], ci
    p.f32_scan.argtypes, p.f32_scan.restype = [i64, ci, ci, ci], ci
    return p


def _cost(bh, nc, dk, dv, length):
    s, elems = -(-nc // length), dk * (dk + dv)
    each, share = -(-2 * bh * s // 256), {(64, 64): 3, (64, 128): 2}.get((dk, dv), 1)
    walk = length * (600 + elems * 132 // 4096) * (4 * each + -(-each // share)) // 5
    return walk + (0 if s == 1 else 3600 + 340 * s + bh * s * elems * 4 // 3100)


def _workspace(bh, nc, elems):
    """mesa_forward_workspace_bytes at chunk 64."""
    extra = min(bh * (nc // 8), 128) * elems * 4 + 512 if bh <= 64 and nc >= 16 else 0
    return bh * nc * elems * 4 + extra


@pytest.mark.parametrize("dk,dv", [(64, 64), (64, 128), (128, 64), (128, 128)])
@pytest.mark.parametrize("bh", [1, 2, 3, 16, 18, 64, 65, 70, 129, 132, 136, 300])
def test_states_only_plan_is_the_best_that_fits(plan, bh, dk, dv):
    """The cheapest plan among those whose totals and decays fit the scratch, for scratch of a whole
    workspace, half of one, and none."""
    elems = dk * (dk + dv)
    for nc in list(range(1, 40)) + [63, 64, 100, 118, 257]:
        for scratch in (_workspace(bh, nc, elems), _workspace(bh, nc, elems) // 2, 0):
            fits = [n for n in sorted({-(-nc // s) for s in range(2, min(128, nc // 2) + 1)})
                    if (bh * -(-nc // n) * (elems + 1)) * 4 <= scratch]
            best = min([_cost(bh, nc, dk, dv, n) for n in fits] + [_cost(bh, nc, dk, dv, nc)])
            got = plan.final_len(bh, nc, dk, dv, scratch)
            assert got == nc or got in fits, (nc, got)
            assert _cost(bh, nc, dk, dv, got) == best, (nc, got, best)


def test_states_only_plan_segments_short_prompts(plan):
    """Even chunk counts from 8 on, few sequences at d 128: two chunks a segment, whose totals and
    decays a whole workspace holds (half of one holds those of three a segment)."""
    for nc in (8, 10, 12, 14):
        assert plan.final_len(4, nc, 128, 128, _workspace(4, nc, 128 * 256)) == 2
        assert plan.final_len(4, nc, 128, 128, _workspace(4, nc, 128 * 256) // 2) == 3


# us of one segment and of the fastest other plan at some of the shapes that were timed
@pytest.mark.parametrize("bh,nc,d,one,more", [(200, 32, 128, 103.8, 117.2), (300, 24, 128, 124.4, 132.7), (130, 64, 128, 196.0, 150.0),
                                              (70, 118, 128, 181.1, 137.0), (48, 10, 128, 20.7, 22.4), (4, 14, 128, 25.6, 12.5),
                                              (2, 8, 128, 16.9, 10.7), (96, 50, 64, 42.5, 33.8), (65, 24, 64, 22.0, 18.8)])
def test_states_only_plan_is_decided_as_measured(plan, bh, nc, d, one, more):
    got = plan.final_len(bh, nc, d, d, _workspace(bh, nc, 2 * d * d))
    assert (got == nc) == (one < more), got


# bf16 chunk states, us of the state pass by the walk and by totals and scan: (single product, sequences, chunks, d_k, d_v)
WIDE = [(False, 4, 32, 128, 128, 38.2, 33.6), (False, 24, 20, 128, 128, 45.3, 42.6), (False, 2, 8, 128, 128, 19.4, 12.3),
        (False, 64, 13, 128, 128, 31.9, 64.3), (False, 8, 128, 128, 128, 53.7, 103.6), (False, 16, 256, 128, 128, 187.3, 455.6),
        (False, 24, 32, 128, 128, 41.4, 61.7), (False, 1, 1000, 64, 64, 64.0, 300.0), (False, 32, 64, 128, 128, 100.8, 193.6),
        (True, 2, 32, 64, 64, 18.5, 12.7), (True, 1, 109, 128, 64, 44.0, 32.5), (True, 2, 64, 128, 128, 33.2, 26.8),
        (True, 16, 13, 128, 128, 21.6, 29.2), (True, 12, 13, 128, 128, 21.2, 26.1), (True, 128, 32, 128, 128, 83.3, 327.1),
        (True, 8, 256, 128, 128, 66.9, 191.8), (True, 24, 20, 128, 64, 32.9, 35.8)]


@pytest.mark.parametrize("single,bh,nc,dk,dv,walk,scan", WIDE)
def test_bf16_state_form_is_decided_as_measured(plan, single, bh, nc, dk, dv, walk, scan):
    assert bool(plan.wide_scan(single, bh, nc, dk * (dk + dv))) == (scan < walk)


# fp32 chunk states, the same: (sequences, chunks, d_k, d_v)
F32 = [(8, 13, 64, 64, 14.4, 10.8), (8, 13, 64, 128, 14.5, 12.1), (2, 256, 64, 64, 221.3, 53.9), (24, 32, 64, 128, 48.7, 41.4), (8, 1000, 64, 64, 864.8, 478.5),
       (2, 13, 128, 128, 14.4, 11.0), (1, 20, 64, 64, 19.8, 10.6), (12, 109, 128, 64, 152.0, 129.0), (2, 8, 64, 64, 9.8, 10.8),
       (32, 32, 64, 64, 31.8, 36.6), (16, 64, 128, 128, 96.2, 133.1), (24, 256, 64, 64, 228.5, 259.0), (24, 128, 128, 64, 328.0, 360.8),
       (8, 512, 128, 64, 454.6, 500.5), (48, 128, 64, 128, 354.0, 377.6)]


@pytest.mark.parametrize("bh,nc,dk,dv,walk,scan", F32)
def test_f32_state_form_is_decided_as_measured(plan, bh, nc, dk, dv, walk, scan):
    assert bool(plan.f32_scan(bh, nc, dk, dv)) == (scan < walk)


def test_scan_ends_where_its_decays_do(plan):
    """One chunk has nothing to scan; past 1024 chunks the scan's decays do not fit its LDS."""
    for single in (0, 1):
        assert not plan.wide_scan(single, 1, 1, 64 * 128) and not plan.wide_scan(single, 1, 1025, 64 * 128)
    assert not plan.f32_scan(1, 1, 64, 64) and plan.f32_scan(1, 1024, 64, 64) and not plan.f32_scan(1, 1025, 64, 64)

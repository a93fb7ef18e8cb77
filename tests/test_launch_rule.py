"""The launch arithmetic of the sweeping kernels (host code, no GPU): compiled here by itself."""
import ctypes
import os
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2209_01877_amd", "csrc")
SOURCE = """
#include "launch_rule.hpp"
extern "C" long long sweep_blocks(long long n, long long fill) { return tetdg::sweep_blocks(n, fill); }
extern "C" long long rising_priority(long long n, long long blocks, int per_cu, long long rounds) {
  return tetdg::rising_priority(n, blocks, per_cu, rounds);
}
"""


@pytest.fixture(scope="module")
def rule(tmp_path_factory):
    d = tmp_path_factory.mktemp("rule")
    (d / "rule.cpp").write_text(SOURCE)
    subprocess.run(["g++", "-std=c++17", "-O1", "-shared", "-fPIC", "-I", CSRC, str(d / "rule.cpp"), "-o",
                    str(d / "rule.so")], check=True)
    lib = ctypes.CDLL(str(d / "rule.so"))
    lib.sweep_blocks.restype = lib.rising_priority.restype = ctypes.c_longlong
    lib.sweep_blocks.argtypes = [ctypes.c_longlong] * 2
    lib.rising_priority.argtypes = [ctypes.c_longlong, ctypes.c_longlong, ctypes.c_int, ctypes.c_longlong]
    return lib


def rounds(ngroups, blocks):
    """Groups that the busiest wavefront sweeps (the kernels' distribution: eighths of the groups if the
    workgroups divide by 8, else one share)."""
    shares = 8 if blocks % 8 == 0 else 1
    per_share = -(-ngroups // shares)
    return -(-per_share // (4 * blocks // shares))


@pytest.mark.parametrize("fill", [1, 5, 8, 100, 256, 304, 512, 768, 1024])
def test_no_round_is_added_by_the_rounding(rule, fill):
    allowed = [b for b in range(1, fill + 1) if b % 8 == 0 or fill < 8]
    most = max(allowed)
    for g in [4 * k for k in range(1, 1200)]:  # meshes are padded to 64 elements: four groups
        b = rule.sweep_blocks(g, fill)
        assert 1 <= b <= fill and (b < 8 or b % 8 == 0)
        if -(-g // 4) < 8:
            assert b == min(-(-g // 4), fill)
        else:
            assert rounds(g, b) == rounds(g, most), (g, b)
            assert b == most or 4 * b < g + 32  # no more workgroups than needed


@pytest.mark.parametrize("per_cu,limit", [(2, 4), (2, 3), (3, 3)])
def test_priorities_where_a_partial_round_fills_every_simd(rule, per_cu, limit):
    cus = 256
    for g in [4 * k for k in range(1, 6000)]:
        blocks = rule.sweep_blocks(g, cus * per_cu)
        full, rest = divmod(g, 4 * blocks)
        # waves of the last round on a SIMD, at least: the workgroups that have one spread over the CUs
        idle_slot = 0 < rest <= 4 * blocks * (per_cu - 1) / per_cu
        assert bool(rule.rising_priority(g, blocks, per_cu, limit)) == (not idle_slot or full < 1 or full >= limit), g

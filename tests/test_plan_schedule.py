"""The schedule behind extend_attention's work plan (host only): a greedy replay of the
dispatch -- 32 workgroup slots per XCD taking its units in plan order -- ends close to
perfect balance, for batches the planner splits and for batches it does not."""

import heapq
import os
import shutil

import numpy as np
import pytest

from paper_2609_32278_amd import kvx
from paper_2609_32278_amd import workloads as wl
from test_abi import _check_plan
from test_sanitizers import ROOT, SAN, _build_and_run


def _replay(items):
    """(end of the last unit, perfect balance), in 64-key iterations."""
    end, total = 0, 0
    for x in range(8):
        slots = [0] * 32
        for it in items[(items["xcd"] == x) & (items["req"] >= 0)]:
            n = -(-(int(it["key_end"]) - int(it["key_begin"])) // 64)
            t = heapq.heappop(slots) + n
            heapq.heappush(slots, t)
            end, total = max(end, t), total + n
    return end, total / 256


@pytest.mark.parametrize("prefix,extend,hq,hkv,d,bound", [
    # few long tiles of very different requests (the one with the least work has the longest tiles)
    ([30000, 9000, 12000, 5000, 22000], [70, 2000, 1500, 1900, 300], 32, 8, 128, 1.12),
    # two KV heads: 26 (request, head) pairs on eight XCDs, unsplit and split
    (list(range(1753, 16554, 1140)), list(range(242, 2107, 144)), 8, 2, 64, 1.2),
    ([40000, 60000, 90000, 100000], [500, 900, 1500, 2300], 8, 2, 64, 1.15),
    ([20000], [3000], 8, 1, 128, 1.25),
])
def test_replayed_schedule_is_balanced(prefix, extend, hq, hkv, d, bound):
    w = wl.make_custom(prefix, extend, hq, hkv, d, seed=3)
    end, ideal = _replay(_check_plan(w))
    assert end <= bound * ideal, (end, ideal)


def test_short_batches_are_split_until_the_start_of_a_unit_dominates():
    """One request of 600 tokens over a 3000-token prefix on one KV head is 19 tiles: the
    planner splits them so that far more of the 256 slots work, but no part is
    shorter than 4 iterations (256 keys)."""
    w = wl.make_custom([3000], [600], 8, 1, 128, seed=3)
    items = _check_plan(w)
    real = items[items["req"] >= 0]
    assert len(real) > 100
    inner = real[real["key_end"] < real["key_end"].max() - 700]
    assert (inner["key_end"] - inner["key_begin"] >= 256).all()


needs_host_build = pytest.mark.skipif(
    shutil.which("g++") is None or not os.path.exists("/opt/rocm/lib/libamdhip64.so"),
    reason="g++ or the HIP runtime library not installed")


def _host_check(tmp_path, name, arg, flags):
    csrc = os.path.join(ROOT, "paper_2609_32278_amd", "csrc")
    exe = str(tmp_path / name)
    cmd = ["g++", "-std=c++17", *flags, "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include",
           "-I" + os.path.join(ROOT, "include"), "-I" + csrc, os.path.join(ROOT, "tests", "sanitize", name + ".cpp"),
           "-L/opt/rocm/lib", "-lamdhip64", "-Wl,-rpath,/opt/rocm/lib", "-o", exe]
    assert "passed" in _build_and_run(cmd, exe, [arg], tmp_path)


@needs_host_build
def test_plans_in_kernel_arguments_expand_to_the_uploaded_units(tmp_path):
    _host_check(tmp_path, "compact_plan", "2000", SAN)


@needs_host_build
@pytest.mark.parametrize("what", ["once", "search", "limits", "fits", "bound"])
def test_planning_of_calls(tmp_path, what):
    _host_check(tmp_path, "plan_calls", what, ["-O2"])

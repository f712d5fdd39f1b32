"""The kernels that bench.py looks counter figures up for are kernels of the built library, and the committed
counter summaries hold them (CPU only)."""
from __future__ import annotations

import json
import os
import re
import sys

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
sys.path.insert(0, ROOT)
import bench  # noqa: E402
from paper_2510_03964_amd import build as lib_build  # noqa: E402

NAMES = {"KERNEL_PLAIN", "KERNEL_FILL", "KERNEL_CACHED", "KERNEL_INCREMENTAL", "KERNEL_EQ7"}


def _mangled(name: str) -> bytes:
    k, op, per_slot, t = re.fullmatch(r"void fwrs::frame_kernel<(\d+), (\d+), (true|false), (\d+)>\(fwrs::FrameDesc\)",
                                      name).groups()
    return f"_ZN4fwrs12frame_kernelILi{k}ELi{op}ELb{int(per_slot == 'true')}ELi{t}EEEvNS_9FrameDescE".encode()


def test_every_kernel_bench_names_is_listed_here():
    assert {n for n in vars(bench) if n.startswith("KERNEL_")} == NAMES
    with open(os.path.join(ROOT, "bench.py")) as f:
        assert len(re.findall(r"frame_kernel<\d", f.read())) == len(NAMES)      # no name outside the constants


@pytest.mark.parametrize("name", sorted(NAMES))
def test_the_library_has_the_kernel(name):
    with open(lib_build.LIB, "rb") as f:
        assert _mangled(getattr(bench, name)) in f.read()


@pytest.mark.parametrize("path,names", [(bench.COUNTERS, ["KERNEL_PLAIN", "KERNEL_FILL", "KERNEL_CACHED"]),
                                        (bench.INC_COUNTERS, ["KERNEL_INCREMENTAL"]), (bench.EQ7_COUNTERS, ["KERNEL_EQ7"]),
                                        (bench.VALU_COUNTERS, ["KERNEL_PLAIN", "KERNEL_CACHED", "KERNEL_EQ7"])])
def test_the_committed_summary_holds_the_kernel(path, names):
    with open(path) as f:
        kernels = json.load(f)["kernels"]
    assert all(getattr(bench, n) in kernels for n in names), sorted(kernels)

"""Plan creation and the launchers agree on which lengths run on which kernels
(csrc/fft_lengths.h), checked on the host for every accepted length: a plan
whose radices only the compile-time kernels know is never handed to the
runtime plan's kernels, which would take them as radix 3."""

import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.fixture(scope="module")
def counts(tmp_path_factory):
    gxx = shutil.which("g++")
    if gxx is None:
        pytest.skip("g++ not available")
    exe = str(tmp_path_factory.mktemp("plan_lengths") / "plan_lengths")
    subprocess.run([gxx, "-std=c++17", "-O1", "-Wall", "-I", os.path.join(ROOT, "paper_1509_07685_amd", "csrc"),
                    os.path.join(ROOT, "tests", "c", "plan_lengths.cpp"), "-o", exe], check=True)
    out = subprocess.run([exe], check=True, capture_output=True, text=True).stdout
    return {tuple(line.split()[:2]): [int(v) for v in line.split()[2:]] for line in out.splitlines()}


LENGTHS = [2 ** a * 3 ** b for a in range(13) for b in range(8) if 2 ** a * 3 ** b <= 4096]
STATIC = [n for n in LENGTHS if 16 <= n <= 512]


@pytest.mark.parametrize("dt", ["f32", "f64"])
def test_every_length_runs_where_plan_creation_meant_it(counts, dt):
    mesh = [n for n in LENGTHS if 2 <= n <= 2048]
    pencils = sum(1 for n in mesh if 32 <= 2 * n <= 512)
    cols = 2 * len(STATIC)
    want = {"x": (sum(1 for n in mesh if n in STATIC and n % 2 == 0 and n <= 256), len(mesh)),
            "pencil": (pencils, len(mesh)), "far_pencil": (0, len(mesh)), "rows": (len(STATIC), len(LENGTHS)),
            "half": (len(STATIC), len(STATIC)), "cols": (cols, 2 * len(LENGTHS)), "far_cols": (0, len(LENGTHS))}
    for role, (fixed, total) in want.items():
        assert counts[dt, role] == [fixed, total - fixed, 0, 0], role


@pytest.mark.parametrize("dt", ["f32", "f64"])
def test_radices_without_kernels_are_refused(counts, dt):
    """Radices of a compile-time plan on another tile, or where 32-bit offsets
    do not reach: no launcher runs them, and the plan check refuses them unless
    the plan is a compile-time one."""
    assert counts[dt, "planted"] == [0, 0, 1, 0]

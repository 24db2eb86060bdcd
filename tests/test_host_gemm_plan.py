"""The dense GEMM's choice of kernel and tile (csrc/gemm_plan.hpp, compiled for the host)."""
import os
import subprocess
from typing import NamedTuple

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


class Plan(NamedTuple):
    few_tokens: bool
    n1: int                # columns of the first of two launches, or 0
    first: str
    rest: str
    first_workgroups: int
    rest_workgroups: int   # (0: the persistent grid)
    splits: int
    split: bool


@pytest.fixture(scope="module")
def plan(tmp_path_factory):
    exe = str(tmp_path_factory.mktemp("host") / "gemm_plan_dump")
    subprocess.run(["g++", "-O1", "-std=c++17", "-Wall", "-Werror", "-I" + os.path.join(ROOT, "paper_2601_18150_amd", "csrc"),
                    os.path.join(ROOT, "tests", "host", "gemm_plan_dump.cpp"), "-o", exe], check=True)

    def run(shapes):
        text = "".join(f"{m} {n} {k}\n" for m, n, k in shapes)
        out = subprocess.run([exe], input=text, capture_output=True, text=True, check=True, timeout=60).stdout
        rows = [ln.split() for ln in out.splitlines()]
        assert len(rows) == len(shapes)
        return [Plan(r[0] == "1", int(r[1]), r[2], r[3], int(r[4]), int(r[5]), int(r[6]), r[7] == "1") for r in rows]
    return run


def test_every_grid_is_one_that_hip_launches(plan):
    """Workgroups of 512 threads: less than 2^32 threads in the grid, whatever valid shape (up to 2^30 tiles of 128x128).
    A few tokens against 2^30 and more weight rows are the ones that fit the memory."""
    sizes = sorted({1, 8, 64, 65, 128, 129, 300, 2047, 8192} | {1 << i for i in range(14, 31)} | {(1 << 31) - 1})
    shapes = [(m, n // 128 * 128, k) for m in sizes for n in sizes for k in (128, 4096)
              if n >= 128 and ((m + 127) // 128) * (n // 128) < 1 << 30]
    assert (8, 1 << 30, 128) in shapes
    for shape, p in zip(shapes, plan(shapes)):
        if not p.few_tokens:
            assert max(p.first_workgroups, p.rest_workgroups) * 512 < 1 << 32, (shape, p)

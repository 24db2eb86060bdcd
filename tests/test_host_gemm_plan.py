"""The dense GEMM's choice of kernel and tile (csrc/gemm_plan.hpp, compiled for the host)."""
import os
import subprocess
from typing import NamedTuple

import pytest

from tests.test_gpu_gemm import SPLIT_CASES, UNSPLIT_CASES
from tests.test_gpu_gemm_tiles import TILE_CASES

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


# (K, N), M, whether the K ranges and their reduction were measured faster than the unsplit tile, by 1 us at least
@pytest.mark.parametrize("k,n,ms,split", [
    (4096, 6144, [65, 72, 80, 100, 128], False), (4096, 4096, [65, 72, 80, 90, 100, 112, 128, 300, 360], False),
    (12288, 4096, [65, 72, 80, 100, 128, 129, 160, 256, 360], True), (8192, 4096, [65, 80, 100, 128], True),
    (8192, 4096, [200], False), (4096, 1024, [100, 128, 300, 512, 800], False), (12288, 1024, [65, 128, 256, 300, 800], True),
    (6144, 2560, [160, 200, 256, 300, 360], False), (16384, 2048, [65, 128, 256, 512], True),
    (2048, 256, [65, 100, 300, 512], False), (28 * 128, 2048, [65, 128, 300], False), (45 * 128, 512, [65, 80, 90, 100], True),
    (12288, 4096, [1, 8, 16, 32, 64], False), (16384, 2048, [40, 48, 64], True), (24576, 1024, [32, 40, 64], True),
    (24576, 4096, [40, 64], True), (24576, 4096, [8, 16, 17, 24], False), (8192, 4096, [8, 33, 64], False), (16384, 1024, [8, 16, 24], False),
])
def test_k_is_split_where_that_was_measured_faster(plan, k, n, ms, split):
    for m, p in zip(ms, plan([(m, n, k) for m in ms])):
        assert p.split == split, (m, n, k, p)
        assert p.splits > 1 or not split


def test_a_split_that_is_run_fits_its_room(plan):
    """Ranges of at least 4 K blocks, tiles x ranges within the 256 CUs, 16 MiB of partial sums at most."""
    shapes = [(m, n, k) for m in (65, 100, 128, 129, 255, 300, 512, 1024, 2047, 5000) for n in (128, 256, 640, 1024, 4096, 16384)
              for k in (512, 1024, 37 * 128, 4096, 12288, 65536)]
    ran = 0
    for (m, n, k), p in zip(shapes, plan(shapes)):
        if p.split:
            ran += 1
            assert k // 128 >= 4 * p.splits and p.splits * ((m + 127) // 128) * (n // 128) <= 256
            assert p.splits * m * n * 4 <= 16 << 20
    assert ran > 20


def test_the_gpu_cases_run_on_the_tiles_they_name(plan):
    for label, shapes in TILE_CASES.items():
        for shape, p in zip(shapes, plan(shapes)):
            assert not p.few_tokens
            assert (p.n1 > 0) == (label == "two launches"), (label, shape, p)
            assert label == "two launches" or p.rest == label, (label, shape, p)
    assert set(TILE_CASES) == {"64x64-short", "64x64", "64x128", "128x64", "128x128", "128x256", "256x128", "256x256", "persistent", "two launches"}


def test_the_gpu_split_cases_are_split(plan):
    for (m, n, k, ranges), p in zip(SPLIT_CASES, plan([c[:3] for c in SPLIT_CASES])):
        assert p.split and p.splits == ranges, (m, n, k, p)
    for shape, p in zip(UNSPLIT_CASES, plan(UNSPLIT_CASES)):
        assert not p.split, (shape, p)
    assert any(r % 2 and k // 128 % r for _, _, k, r in SPLIT_CASES), "an odd number of uneven ranges"

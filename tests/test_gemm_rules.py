"""The GEMM dispatch rules (csrc/gemm_rules.h) in a host build: no GPU needed."""

import os
import shutil
import subprocess

import pytest

import test_gpu_decode_layout
import test_gpu_fp6_ksplit
import test_gpu_ksplit

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.fixture(scope="module")
def routes(tmp_path_factory):
    """The routes of a list of queries (tests/gemm_rules_check.cpp), a list of lines."""
    gxx = shutil.which("g++")
    if not gxx:
        pytest.skip("g++ not available")
    exe = tmp_path_factory.mktemp("rules") / "gemm_rules_check"
    r = subprocess.run([gxx, "-O1", "-std=c++17", "-Wall", "-Werror",
                        "-I" + os.path.join(ROOT, "paper_2606_12487_amd", "csrc"),
                        os.path.join(ROOT, "tests", "gemm_rules_check.cpp"), "-o", str(exe)],
                       capture_output=True, text=True, timeout=300)
    assert r.returncode == 0, r.stderr[-2000:]

    def ask(queries):
        run = subprocess.run([str(exe)], input="\n".join(queries) + "\n", capture_output=True, text=True,
                             timeout=60)
        assert run.returncode == 0, run.stdout[-2000:]
        return run.stdout.rstrip("\n").split("\n")

    return ask


def test_every_shape_has_a_kernel(routes):
    # Sizes far beyond the fitted ones keep to the tile kernels.
    assert routes(["int8 16 4096 4096 4", "int8 17 16 128 8", "int8 1000000 57344 65536 4",
                   "int8 100000 176 8192 8", "fp6 1000000 57344 65536"]) == [
                       "decode", "ksplit 1x2x8", "wide", "tile", "wide"]


def test_shapes_of_the_tile_kernels(routes):
    # Measured 4 to 65% slower on the K-split kernel: short K, and beyond 1024 rows.
    slow = ["int8 512 6144 128 4", "int8 256 11008 256 4", "int8 777 4096 256 4", "int8 256 11008 128 8",
            "int8 160 16384 256 8", "int8 160 11008 128 8", "int8 1024 2576 512 8", "int8 384 6144 512 8",
            "int8 777 2576 256 8", "int8 512 6144 1024 8", "int8 1536 2576 3584 8", "int8 1536 4096 28672 8",
            "int8 2853 1456 9216 8", "int8 2174 1184 2944 8", "int8 21 37760 256 8"]
    fast = ["int8 48 8192 8192 4", "int8 128 6144 4096 8", "int8 333 4096 14336 8", "int8 256 11008 4096 4",
            "int8 33 4096 1024 8", "int8 100 4096 512 4"]
    got = routes(slow + fast)
    assert all(r in ("tile", "wide") for r in got[:len(slow)]), got
    assert all(r.startswith("ksplit") for r in got[len(slow):]), got


def test_fp6_shapes_of_the_tile_kernel(routes):
    # Short K, few channels for many rows, and almost a tile of rows: measured 1.1
    # to 2.3 times slower on the K-split kernel.
    slow = ["fp6 4096 28672 256", "fp6 65536 2576 128", "fp6 65536 160 4096", "fp6 224 28672 4096",
            "fp6 224 57344 512", "fp6 160 28672 2048", "fp6 1024 57344 128"]
    # Many rows of few channels: up to 1.26 times slower there.
    slow += ["fp6 8192 512 2048", "fp6 4096 1024 2048", "fp6 16384 256 1536", "fp6 6144 768 1024",
             "fp6 6144 2048 8192", "fp6 160 28672 8192"]
    fast = ["fp6 500 4096 4096", "fp6 64 2048 14336", "fp6 33 28672 256", "fp6 100 160 4096",
            "fp6 4096 512 2048", "fp6 16384 160 512"]
    got = routes(slow + fast)
    assert got[:len(slow)] == ["wide"] * len(slow)
    assert all(r.startswith("ksplit") for r in got[len(slow):]), got


def test_decode_shapes_of_the_register_kernel(routes):
    # Measured 5 to 18% slower on the K-split kernel: short K, and few tokens on the
    # decode layout; the others up to 1.7 times faster there.
    regs = ["decode 1 28672 128 4 0", "decode 8 4096 384 8 0", "decode 16 6144 384 4 0",
            "decode 1 2560 14336 4 1", "decode 2 1024 28672 4 1", "decode 4 28672 4096 4 1",
            "decode 2 11008 3584 4 1", "decode 1 28672 4096 8 1",
            "decode 4 20480 256 8 1", "decode 8 8192 28672 4 1", "decode 6 2560 28672 4 1"]
    ksplit = ["decode 1 4096 4096 4 0", "decode 16 4096 14336 8 0", "decode 4 16384 128 8 0",
              "decode 16 8192 8192 4 1", "decode 16 4096 14336 8 1", "decode 1 5120 14336 4 1",
              "decode 8 57344 8192 4 1", "decode 8 5120 28672 4 1", "decode 16 8192 28672 4 1"]
    got = routes(regs + ksplit)
    assert all(r.startswith("regs") for r in got[:len(regs)]), got
    assert all(r.startswith("ksplit") for r in got[len(regs):]), got


def test_one_launch_where_it_is_the_faster(routes):
    # Measured: one launch 0.68 to 0.95 of the time of two; two 0.33 to 0.85 of one.
    one = ["fused 1 4096 1 12 4096", "fused 1 4096 1 12 12288", "fused 1 8192 1 12 12288", "fused 1 4096 1 12 16384",
           "fused 1 14336 1 11 4096", "fused 2 4096 1 12 4096", "fused 2 4096 1 7 12288", "fused 2 8192 1 12 4096"]
    two = ["fused 1 14336 1 11 12288", "fused 1 16384 1 13 6144", "fused 1 512 1 9 16384", "fused 1 3584 28 7 4096",
           "fused 2 8192 1 12 12288", "fused 2 5120 1 10 6144", "fused 2 512 1 9 12288", "fused 4 4096 1 12 12288"]
    assert routes(one + two) == ["one"] * len(one) + ["two"] * len(two)


def test_rotation_launches_hold_less_than_2_32_threads(routes):
    # 1024 threads a row in registers, 256 on the general kernel at 28 x 512.
    assert routes(["rotate 65 14336 28 9", "rotate 64 14336 28 9", "rotate 257 28672 28 10", "rotate 256 28672 28 10",
                   "rotate 4194272 14336 28 9", "rotate 4194273 14336 28 9", "rotate 5000000 14336 28 9",
                   "rotate 4096 28672 28 9", "rotate 4096 16384 1 14"]) == [
                       "registers", "general", "registers", "general", "registers", "general", "general",
                       "general", "general"]


def test_every_decode_kernel_has_a_case(routes):
    for layout, cases in ((0, test_gpu_ksplit.CASES), (1, test_gpu_decode_layout.CASES)):
        cases = [c for c in cases if c[0] <= 16]
        got = routes([f"decode {M} {N} {K} {bits} {layout}" for M, K, N, bits in cases])
        seen = {(r, c[3]) for r, c in zip(got, cases)}
        kernels = {"regs 1x4", "regs 2x4", "ksplit 1x1x8", "ksplit 2x1x4", "ksplit 2x1x8"}
        kernels |= {"regs 1x8"} if layout else set()   # long rows of canonical weights are split
        assert seen == {(k, bits) for k in kernels for bits in (4, 8)}, layout
        # two blocks of an odd number, with a last stage of 128 k
        for r in ("ksplit 2x1x4", "ksplit 2x1x8"):
            assert any(g == r and c[2] % 32 == 16 and c[1] % 256 == 128 for g, c in zip(got, cases)), (r, layout)


def test_every_tile_has_a_case(routes):
    # A ragged case each: M and N no multiples of the tile, a last stage of 128 k.
    tiles = {tuple(line.split()) for line in routes(["tiles"]) if line}
    cases = [c for c in test_gpu_ksplit.CASES if c[0] > 16 and c[0] % 16 and c[2] % 32 and c[1] % 256]
    got = routes([f"int8 {M} {N} {K} {bits}" for M, K, N, bits in cases])
    seen = {("int8", str(c[3]), r.split()[1]) for r, c in zip(got, cases) if r.startswith("ksplit")}
    cases = [c for c in test_gpu_fp6_ksplit.CASES if c[0] % 32]
    got = routes([f"fp6 {M} {N} {K}" for M, N, K in cases])
    seen |= {("fp6", "4", r.split()[1]) for r in got if r.startswith("ksplit")}
    assert seen == tiles, (tiles - seen, seen - tiles)
    assert "wide" in got

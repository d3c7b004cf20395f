"""Strips and column tiles in two sets, each fetched by half of the XCDs: which products have them, and that every place of a
launch computes something else.  (No GPU needed: the library's rules are asked, and its function of the places is compiled for the host.)"""
import ctypes
import os
import subprocess

import pytest

import paper_2506_15174_amd as spmm

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(os.path.dirname(HERE), "paper_2506_15174_amd", "csrc")


def test_every_place_once(tmp_path):
    exe = str(tmp_path / "places_in_sets")
    subprocess.run(["g++", "-O2", "-std=c++17", "-Wall", "-I", CSRC, os.path.join(HERE, "places_in_sets.cpp"), "-o", exe], check=True)
    res = subprocess.run([exe], capture_output=True, text=True, timeout=300)
    assert res.returncode == 0 and res.stdout.endswith("ok\n"), res.stdout + res.stderr


def strips_of_set(steps, K, N):
    f = spmm.load().spmm_strips_of_set
    f.restype, f.argtypes = ctypes.c_uint32, [ctypes.c_int64, ctypes.c_int64, ctypes.c_int32]
    return f(steps, K, N)


# 16 strips are the fewest, whole lines (4 strips) to a set, rows of whole lines; 384 bytes of entries a step, less than 8 times B's bytes.
@pytest.mark.parametrize("N,strips,first", [(96, 12, 12), (120, 15, 15), (128, 16, 8), (132, 17, 17), (136, 17, 17), (160, 20, 12), (192, 24, 12),
                                            (256, 32, 16), (288, 36, 20), (2080, 260, 132)])
def test_strips(N, strips, first):
    K = 4096
    limit = 8 * 4 * K * N // 384
    assert strips_of_set(1000, K, N) == first and strips_of_set(limit - 1, K, N) == first
    assert strips_of_set(limit + 1, K, N) == strips


def tiles_of_set(rows, M, K, N, stream_words):
    f = spmm.load().spmm_tiles_of_set
    f.restype, f.argtypes = ctypes.c_uint32, [ctypes.c_int, ctypes.c_int64, ctypes.c_int64, ctypes.c_int32, ctypes.c_int64]
    return f(rows, M, K, N, stream_words)


def column_tiles(rows, M, K, N):
    """Column tiles of a product, and their width."""
    f = spmm.load().spmm_tiles_time
    f.restype, groups = ctypes.c_double, ctypes.c_int(0)
    f(rows, ctypes.c_int64(M), ctypes.c_int64(K), ctypes.c_int64(N), ctypes.c_double(0), ctypes.c_double(0), ctypes.byref(groups))
    return -(-N // (groups.value * rows)), groups.value * rows


# Panels of 16 rows whose blocks have less than 1.5 times B's bytes, rows of whole lines, a line or more to a set.
@pytest.mark.parametrize("M", [16, 512, 3000])
@pytest.mark.parametrize("N", [16, 32, 64, 96, 100, 128, 132, 160, 224, 256, 1056])
def test_tiles(M, N):
    K = 2048
    tiles, cols = column_tiles(16, M, K, N)
    line = max(1, 32 // cols)
    first = -(-((tiles + 1) // 2) // line) * line
    if N % 32 or first >= tiles:
        first = tiles
    limit = 3 * K * N // 2
    assert tiles_of_set(16, M, K, N, limit - 1) == first and tiles_of_set(16, M, K, N, limit) == tiles
    assert N != 128 or M != 512 or (first, tiles) == (4, 8)
    assert tiles_of_set(32, M, K, N, 1) == column_tiles(32, M, K, N)[0]
    assert tiles_of_set(16, M, K, 1 << 24, 1) == -(-(1 << 24) // column_tiles(16, M, K, 1 << 24)[1])  # 64-bit addresses

"""Which of the block route's loads stream (csrc/ds_perm.h): in images that no cache holds those whose lines no other block
reads."""
import ctypes
import os
import subprocess

import numpy as np
import pytest

from test_perm_blocks import _check

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.fixture(scope="module")
def lib(tmp_path_factory):
    so = str(tmp_path_factory.mktemp("perm") / "perm_host.so")
    subprocess.run(["g++", "-O2", "-std=c++17", "-Wall", "-Werror", "-Wno-unknown-pragmas", "-fPIC", "-shared", "-I",
                    os.path.join(ROOT, "paper_2601_16956_amd", "csrc"),
                    os.path.join(ROOT, "tests", "c_abi", "perm_host.cpp"), "-o", so], check=True)
    lib = ctypes.CDLL(so)
    u64, vp = ctypes.c_uint64, ctypes.c_void_p
    lib.perm_host_move.restype = ctypes.c_long
    lib.perm_host_move.argtypes = [vp, u64, u64, u64, u64, u64, ctypes.c_uint32, vp, vp, ctypes.c_int, u64, u64, vp, vp, vp]
    lib.perm_host_loads.restype = lib.perm_host_streamed.restype = u64
    return lib


# (view, do the gather's loads stream?); walks along b: pieces of the tensor on either side of four lines, lines that
# several blocks read, runs of 12 bytes, whole rows of units
GATHERS = [
    ("f32", (3000,), (2,), True), ("u8", (9000,), (3,), True), ("bf16", (40, 300), (800, 2), True),
    ("f32", (20, 64), (1000, 2), True), ("f32", (20, 63), (1000, 2), False),
    ("bf16", (200, 150, 4), (8, 1700, 2), False), ("bf16", (50, 100, 6), (16, 1000, 2), False),
    ("u8", (60, 190, 8), (16, 1200, 2), False), ("bf16", (30, 40, 32), (64, 2000, 2), False),
    ("f32", (40, 30, 4, 3), (16, 700, 4, 1), False), ("f32", (900, 3), (4, 1), True), ("f32", (9, 200, 3), (900, 4, 1), True),
    # walks along a: columns of few lines and of many
    ("bf16", (200, 9), (1, 200), False), ("f32", (512, 9), (1, 512), True)]


@pytest.mark.parametrize("dtype,shape,strides,streams", GATHERS)
def test_the_gather_streams_lines_of_one_block(lib, dtype, shape, strides, streams):
    loads, streamed = lib.perm_host_loads(), lib.perm_host_streamed()
    assert _check(lib.perm_host_move, dtype, shape, strides, 0, 512, np.random.default_rng(1)) > 0
    loads, streamed = lib.perm_host_loads() - loads, lib.perm_host_streamed() - streamed
    assert loads > 0
    assert streamed == (loads if streams else 0)


# (view, image offset, do the scatter's loads stream?): rows on either side of three lines, rows of whole lines, pieces, wide
# blocks
SCATTERS = [
    ("u8", (300, 3283), (1, 301), 512, False), ("bf16", (70, 1031), (1, 77), 512, False), ("f32", (37, 2230), (1, 37), 512, False),
    ("f32", (70, 33, 4, 3), (16, 1120, 4, 1), 512, False), ("bf16", (70, 1024), (1, 77), 512, True),
    ("bf16", (70, 1024), (1, 77), 16, False), ("i64", (50, 362), (1, 58), 64, True), ("i64", (50, 24), (1, 58), 64, False),
    ("f32", (512, 9), (1, 512), 16, True), ("f32", (3000,), (2,), 16, True),
    ("bf16", (64, 257), (1, 72), 512, False), ("bf16", (50, 16), (800, 2), 16, False)]


@pytest.mark.parametrize("dtype,shape,strides,at,streams", SCATTERS)
def test_the_scatter_streams_lines_of_one_block(lib, dtype, shape, strides, at, streams):
    assert _check(lib.perm_host_move, dtype, shape, strides, 0, at, np.random.default_rng(1)) > 0
    assert bool(lib.perm_host_image_streams()) == streams


# (view, bytes of the whole image, do the scatter's loads stream?): narrow blocks along a, image and tensors on either side of
# 7/8 of 256 MiB, with rows of whole lines of 256 MiB, and of batches that lie apart; blocks that are not of that kind, whatever the image has
CACHED = [
    ("i64", (50, 362), (1, 50), 117 * 10**6, True), ("i64", (50, 362), (1, 50), 118 * 10**6, False),
    ("i64", (50, 362), (1, 100), 78 * 10**6, True), ("i64", (50, 362), (1, 100), 79 * 10**6, False),
    ("i64", (33, 512), (1, 33), 134 * 10**6, True), ("i64", (33, 512), (1, 33), 135 * 10**6, False),
    ("i64", (3, 50, 362), (362 * 200, 1, 100), 78 * 10**6, True), ("i64", (3, 50, 362), (362 * 200, 1, 100), 79 * 10**6, False),
    ("f32", (512, 9), (1, 512), 10**9, True), ("f32", (3000,), (2,), 10**9, True)]


@pytest.mark.parametrize("dtype,shape,strides,image_bytes,streams", CACHED)
def test_the_scatter_streams_beside_tensors_that_the_cache_holds(lib, dtype, shape, strides, image_bytes, streams):
    image = ctypes.c_uint64(image_bytes)
    lib.perm_host_image_bytes(image)
    try:
        assert _check(lib.perm_host_move, dtype, shape, strides, 0, 512, np.random.default_rng(1)) > 0
        assert bool(lib.perm_host_image_streams()) == streams
    finally:
        lib.perm_host_image_bytes(ctypes.c_uint64(1 << 20))

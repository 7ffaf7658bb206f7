"""The order in which the blocks of views with short runs are dealt to the XCDs, and the streaming loads of such blocks in
images of more than 64 MiB."""
import ctypes
import os
import subprocess

import numpy as np
import pytest

from oracle import ds_oracle as orc
from workloads.configs import DTYPES, Shard, Workload

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.mark.parametrize("pack", [0, 1])
def test_every_block_is_taken_once(tmp_path, pack):
    so = str(tmp_path / "order_host.so")
    subprocess.run(["g++", "-O2", "-std=c++17", "-Wall", "-Werror", "-Wno-unknown-pragmas", "-fPIC", "-shared", "-I",
                    os.path.join(ROOT, "paper_2601_16956_amd", "csrc"),
                    os.path.join(ROOT, "tests", "c_abi", "order_host.cpp"), "-o", so], check=True)
    deal = ctypes.CDLL(so).order_host_deal
    deal.restype, deal.argtypes = ctypes.c_uint32, [ctypes.c_uint32, ctypes.c_int, ctypes.c_void_p]
    for n in [*range(1, 40), 767, 768, 769, 2047, 2048, 2049, *range(4096, 4110), 100003, (1 << 22) - 1, (1 << 27) - 1]:
        hits = np.zeros(n, dtype=np.uint8)
        launched = deal(n, pack, hits.ctypes.data)
        assert hits.min() == hits.max() == 1
        # at most one block per XCD and stripe too many (a launch of a few blocks has two per XCD)
        assert launched <= max(16, n + 8 * (n // (8 * 48) + 1) + 8)


def test_launches_whose_blocks_share_lines_far_on_have_one_stripe_per_xcd(tmp_path):
    so = str(tmp_path / "order_host.so")
    subprocess.run(["g++", "-O2", "-std=c++17", "-Wall", "-Werror", "-Wno-unknown-pragmas", "-fPIC", "-shared", "-I",
                    os.path.join(ROOT, "paper_2601_16956_amd", "csrc"),
                    os.path.join(ROOT, "tests", "c_abi", "order_host.cpp"), "-o", so], check=True)
    lib = ctypes.CDLL(so)
    stripe, deal = lib.order_host_stripe, lib.order_host_deal_together
    deal.restype, deal.argtypes = ctypes.c_uint32, [ctypes.c_uint32, ctypes.c_int, ctypes.c_void_p]
    for n in (16, 767, 768, 5000, 100003, 8 * 65536, 8 * 65537 + 1, 700001, (1 << 22) - 1, (1 << 27) - 8):
        for pack in (0, 1):
            hits = np.zeros(n, dtype=np.uint8)
            assert deal(n, pack, hits.ctypes.data) == 8 * -(-n // 8)
            assert hits.min() == hits.max() == 1
            assert stripe(n, pack, 1) == -(-n // 8)
    assert stripe(5000, 0, 0) < 64 and stripe(5000, 1, 0) < 128


# lines of the tensor that are one block's own and lines that two blocks share, in each way to walk a block
STREAMED = [("bf16", (1024, 1536), (1, 1024)), ("bf16", (1024, 1531), (1, 1024)), ("f32", (512, 1111), (1, 516)),
            ("u8", (704, 1901), (1, 704)), ("i64", (130, 513), (1, 136)), ("bf16", (2, 512, 768), (512 * 768, 1, 512)),
            ("f32", (300, 300, 9), (2700, 1, 300)), ("f32", (61, 70, 9), (630, 1, 70)), ("f32", (333, 1111), (2222, 2)),
            ("bf16", (700, 64, 6), (1024, 16, 1)), ("u8", (131, 259), (1, 133)), ("bf16", (70, 300), (800, 2))]


@pytest.mark.gpu
@pytest.mark.parametrize("beside", [60 << 20, 70 << 20])
def test_blocks_of_images_that_no_cache_holds(beside):
    """One launch with the other chunks (60 MB) and two (70 MB), whole and in ranges that cut blocks."""
    import gpu_util as gu
    rng = np.random.default_rng(beside >> 20)
    shards, at = [], 0
    for k, (dtype, shape, strides) in enumerate(STREAMED + [("u8", (beside,), (1,))]):
        at = -(-at // 256) * 256 + (0 if k % 3 else DTYPES[dtype][1] * int(rng.integers(0, 3)))
        shards.append(Shard(f"s{k}", dtype, shape, strides, at, k))
        at += (sum((e - 1) * s for e, s in zip(shape, strides)) + 1) * DTYPES[dtype][1]
    w = Workload("streamed", 64, 0, rng.integers(0, 256, size=at + 64, dtype=np.uint8), shards)
    want, offs, tab = gu.oracle_image(w)
    dw = gu.DeviceWorkload(w)
    try:
        print(f"[case] streamed blocks beside {beside} bytes, image={dw.total}", flush=True)
        assert dw.total > 64 << 20
        cuts = [0] + sorted(16 * int(x) for x in rng.integers(1, (dw.total - beside) // 16, 5)) + [dw.total]
        ranges = [(lo, hi) for lo, hi in zip(cuts, cuts[1:]) if lo < hi]
        for lo, hi in [(0, dw.total)] + ranges:
            assert gu.first_mismatch(dw.pack(lo, hi), want[lo:hi]) is None, (lo, hi)
        w.arena[:] = 0x5A
        orc.unpack(tab, len(shards), want)
        for parts in ([(0, dw.total)], ranges):
            dw.arena.fill_(0x5A)
            for lo, hi in parts:
                dw.unpack(want, lo, hi)
            assert gu.first_mismatch(dw.arena_host(), w.arena) is None
    finally:
        dw.close()


@pytest.mark.gpu
@pytest.mark.parametrize("beside", [0, 9 << 20, 12 << 20])
def test_chunks_beside_blocks_in_pieces_and_whole(beside):
    """Up to 640 chunks share the blocks' launch in pieces of 4 KiB, more of them whole: every kind of chunk, ends of shards
    at every place in a piece, and ranges that cut pieces."""
    import gpu_util as gu
    rng = np.random.default_rng(beside >> 20)
    views = [("bf16", (300, 203), (1, 301)), ("u8", (5, 40, 1000), (70000, 1500, 1)), ("u8", (3,), (1,)), ("u8", (41, 513), (700, 1)),
             ("f32", (20, 300, 4), (300 * 8 + 4, 8, 1)), ("u8", (17000,), (1,)), ("i64", (130, 513), (1, 136)), ("u8", (90, 33, 17), (790, 23, 1)),
             ("u8", (4097,), (1,)), ("bf16", (11, 7), (1, 13)), ("u8", (beside // 2 + 5,), (1,)), ("u8", (beside // 3000, 1000), (1012, 1)),
             ("bf16", (beside // 12000, 5, 200), (1100, 216, 1)), ("f32", (333, 111), (222, 2))]
    shards, at = [], 0
    for k, (dtype, shape, strides) in enumerate(v for v in views if v[1][0]):
        es = DTYPES[dtype][1]
        at = -(-at // 64) * 64 + es * int(rng.integers(0, 3))
        shards.append(Shard(f"b{k}", dtype, shape, strides, at, k))
        at += (sum((e - 1) * s for e, s in zip(shape, strides)) + 1) * es
    w = Workload("pieces", 64, 0, rng.integers(0, 256, size=at + 64, dtype=np.uint8), shards)
    want, offs, tab = gu.oracle_image(w)
    dw = gu.DeviceWorkload(w)
    try:
        print(f"[case] pieces beside blocks, {beside} bytes, image={dw.total}", flush=True)
        cuts = [0, 16, 4096, 8208] + sorted(16 * int(x) for x in rng.integers(600, dw.total // 16, 6)) + [dw.total]
        ranges = [(lo, hi) for lo, hi in zip(cuts, cuts[1:]) if lo < hi]
        for lo, hi in [(0, dw.total)] + ranges:
            assert gu.first_mismatch(dw.pack(lo, hi), want[lo:hi]) is None, (lo, hi)
        w.arena[:] = 0x5A
        orc.unpack(tab, len(shards), want)
        for parts in ([(0, dw.total)], ranges):
            dw.arena.fill_(0x5A)
            for lo, hi in parts:
                dw.unpack(want, lo, hi)
            assert gu.first_mismatch(dw.arena_host(), w.arena) is None
    finally:
        dw.close()


@pytest.mark.gpu
@pytest.mark.parametrize("views", [60, 700, 3600])
def test_chunks_that_hold_little_besides_blocks(views):
    """Chunks of the ends of views and of small tensors between them: few, many, and in an image that no cache holds."""
    import gpu_util as gu
    rng = np.random.default_rng(views)
    shards, at = [], 0
    for k in range(views):
        r, c, n = (int(rng.integers(lo, hi)) for lo, hi in ((80, 121), (90, 113), (1, 900)))
        for dtype, shape, strides in (("bf16", (r, c), (1, r + k % 3)), ("u8", (n,), (1,))):
            es = DTYPES[dtype][1]
            at = -(-at // 16) * 16 + es * int(rng.integers(0, 3))
            shards.append(Shard(f"r{len(shards)}", dtype, shape, strides, at, len(shards)))
            at += (sum((e - 1) * s for e, s in zip(shape, strides)) + 1) * es
    w = Workload("rests", 64, 0, rng.integers(0, 256, size=at + 64, dtype=np.uint8), shards)
    want, offs, tab = gu.oracle_image(w)
    dw = gu.DeviceWorkload(w)
    try:
        print(f"[case] rests of {views} views, image={dw.total}", flush=True)
        cuts = [0] + sorted(16 * int(x) for x in rng.integers(1, dw.total // 16, 6)) + [dw.total]
        ranges = [(lo, hi) for lo, hi in zip(cuts, cuts[1:]) if lo < hi]
        for lo, hi in [(0, dw.total)] + ranges:
            assert gu.first_mismatch(dw.pack(lo, hi), want[lo:hi]) is None, (lo, hi)
        w.arena[:] = 0x5A
        orc.unpack(tab, len(shards), want)
        for parts in ([(0, dw.total)], ranges):
            dw.arena.fill_(0x5A)
            for lo, hi in parts:
                dw.unpack(want, lo, hi)
            assert gu.first_mismatch(dw.arena_host(), w.arena) is None
    finally:
        dw.close()

"""Blocks of short rows that are dense along a (16 bytes of neighbours at a time) and runs of 12 bytes, thread by thread on
the CPU and, in one table, on the GPU."""
import ctypes

import numpy as np
import pytest

from oracle import ds_oracle as orc
from test_perm_blocks import _check, host  # noqa: F401  (the fixture)
from test_streaming_loads import lib  # noqa: F401  (the fixture)
from workloads.configs import DTYPES, Shard, Workload

# whole groups and rests of each element size, last blocks of less than a group, one row to a block, batches; runs of 12
# bytes in rows that end anywhere in a unit and in a line, and one behind the other
VIEWS = [
    ("u8", (33, 500), (1, 35)), ("u8", (33, 500), (1, 33)), ("u8", (300, 33), (1, 301)), ("u8", (16, 70), (1, 16)),
    ("bf16", (70, 250), (1, 70)), ("bf16", (65, 9), (1, 67)), ("bf16", (9, 249), (1, 9)), ("bf16", (5, 71, 9), (700, 1, 75)),
    ("f32", (536, 9), (1, 536)), ("f32", (3, 457, 9), (457 * 9, 1, 457)), ("f32", (131, 121), (1, 131)),
    ("i64", (131, 37), (1, 133)), ("i64", (2, 2, 513, 5), (9000, 3000, 1, 513)), ("i64", (3, 63), (1, 3)),
    ("f32", (2, 33, 70, 3), (9900, 290, 4, 1)), ("f32", (700, 3), (8, 1)), ("f32", (41, 90, 3), (400, 4, 1)),
    ("bf16", (1500, 6), (16, 1)), ("f32", (9, 1031, 3), (5000, 4, 1)), ("u8", (5000, 6), (16, 1)), ("f32", (5000,), (2,))]


@pytest.mark.parametrize("k", range(len(VIEWS)))
def test_blocks_move_exactly_the_view(host, k):  # noqa: F811
    dtype, shape, strides = VIEWS[k]
    rng = np.random.default_rng(k)
    for shift, at in ((0, 0), (1, 16), (2, 512), (4, 80)):
        assert _check(host, dtype, shape, strides, shift, at, rng) > 0


# (view, 16 bytes along the columns at a time?): columns that leave 4 banks of LDS or fewer, on either side of the groups per block
# that these serve, and rows of at most 8 bytes
BANKS = [
    ("u8", (3000, 24), (1, 3000), False), ("u8", (3000, 33), (1, 3000), True), ("u8", (3000, 34), (1, 3000), True),
    ("u8", (3000, 60), (1, 3000), False), ("u8", (3000, 72), (1, 3000), False), ("u8", (900, 84), (1, 900), True),
    ("u8", (3000, 76), (1, 3000), False), ("u8", (900, 136), (1, 900), False), ("u8", (900, 200), (1, 900), True),
    ("u8", (9000, 4), (1, 9000), True), ("u8", (9000, 8), (1, 9000), False), ("u8", (9000, 12), (1, 9000), False),
    ("bf16", (5000, 4), (1, 5000), True), ("bf16", (5000, 12), (1, 5000), False), ("bf16", (3000, 28), (1, 3000), False),
    ("bf16", (900, 60), (1, 900), False), ("bf16", (900, 68), (1, 900), True), ("bf16", (3, 900, 20), (18000, 1, 900), False),
    ("f32", (3000, 6), (1, 3000), True), ("i64", (900, 9), (1, 900), True)]


@pytest.mark.parametrize("dtype,shape,strides,groups", BANKS)
def test_groups_where_the_banks_allow(lib, dtype, shape, strides, groups):  # noqa: F811
    lib.perm_host_image_bytes(ctypes.c_uint64(4 << 20))
    assert _check(lib.perm_host_move, dtype, shape, strides, 0, 512, np.random.default_rng(1)) > 0
    assert bool(lib.perm_host_groups()) == groups


@pytest.mark.gpu
@pytest.mark.parametrize("align,beside", [(16, 0), (512, 0), (64, 70 << 20)])
def test_gather_and_scatter(align, beside):
    """Whole and in ranges that cut blocks; with 70 MB beside them the loads stream."""
    import gpu_util as gu
    rng = np.random.default_rng(align)
    shards, at = [], 0
    big = [("f32", (61, 300, 9), (2700, 1, 300)), ("u8", (2003, 267), (1, 2003)), ("bf16", (40000, 6), (16, 1))]
    for k, (dtype, shape, strides) in enumerate(VIEWS + big + ([("u8", (beside,), (1,))] if beside else [])):
        es = DTYPES[dtype][1]
        at = -(-at // 256) * 256 + es * int(rng.integers(0, 3))
        shards.append(Shard(f"g{k}", dtype, shape, strides, at, k))
        at += (sum((e - 1) * s for e, s in zip(shape, strides)) + 1) * es
    w = Workload("groups", align, 0, rng.integers(0, 256, size=at + 64, dtype=np.uint8), shards)
    want, offs, tab = gu.oracle_image(w)
    dw = gu.DeviceWorkload(w)
    try:
        print(f"[case] groups align={align} image={dw.total}", flush=True)
        cuts = [0] + sorted(16 * int(x) for x in rng.integers(1, (dw.total - beside) // 16, 7)) + [dw.total]
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

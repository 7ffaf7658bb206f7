"""How large the blocks of a view with short runs are (csrc/ds_perm.h): smaller in images of up to 2 MiB, none nearly empty for a
few bytes of a row."""
import numpy as np
import pytest

from oracle import ds_oracle as orc
from test_perm_blocks import _check
from test_streaming_loads import lib  # noqa: F401  (the fixture)
from workloads.configs import DTYPES, Shard, Workload

SMALL, LARGE = 2 << 20, (2 << 20) + 16

# (view, blocks in a small image and in a large one): bytes 4 and 8 KiB, other elements 8 KiB; rows up to and above 4608
# bytes, two and three of them to a block; short rows, of which no more than 8 KiB go together; pieces of 8 and 16 KiB
SIZES = [
    ("u8", (40000,), (2,), 10, 5), ("f32", (10000,), (2,), 5, 5), ("f32", (64, 1031), (2063, 2), 32, 32),
    ("f32", (64, 1152), (2400, 2), 32, 32), ("f32", (64, 1153), (2400, 2), 64, 64), ("u8", (40, 1031), (2070, 2), 10, 5),
    ("bf16", (30, 1365), (2800, 2), 10, 10), ("f32", (40, 256, 4), (2100, 8, 2), 20, 20), ("f32", (600, 6), (1, 602), 2, 1),
    ("u8", (400, 60), (1, 401), 4, 2), ("i64", (200, 9), (1, 203), 2, 1), ("bf16", (8192, 3), (1, 8192), 7, 4)]


@pytest.mark.parametrize("dtype,shape,strides,small,large", SIZES)
def test_blocks_of_small_and_large_images(lib, dtype, shape, strides, small, large):  # noqa: F811
    for image, blocks in ((SMALL, small), (LARGE, large)):
        lib.perm_host_image_bytes(image)
        assert _check(lib.perm_host_move, dtype, shape, strides, 0, 512, np.random.default_rng(1)) == blocks
        assert _check(lib.perm_host_move, dtype, shape, strides, 1, 16, np.random.default_rng(2)) > 0


@pytest.mark.gpu
@pytest.mark.parametrize("beside", [0, 2 << 20])
def test_gather_and_scatter(beside):
    """The views in an image of less than 2 MiB, and beside as much, whole and in ranges that cut blocks."""
    import gpu_util as gu
    rng = np.random.default_rng(beside >> 20)
    shards, at = [], 0
    for k, (dtype, shape, strides) in enumerate([v[:3] for v in SIZES] + ([("u8", (beside,), (1,))] if beside else [])):
        es = DTYPES[dtype][1]
        at = -(-at // 256) * 256 + es * int(rng.integers(0, 3))
        shards.append(Shard(f"s{k}", dtype, shape, strides, at, k))
        at += (sum((e - 1) * s for e, s in zip(shape, strides)) + 1) * es
    w = Workload("sizes", 64, 0, rng.integers(0, 256, size=at + 64, dtype=np.uint8), shards)
    want, offs, tab = gu.oracle_image(w)
    dw = gu.DeviceWorkload(w)
    try:
        print(f"[case] block sizes, image={dw.total}", flush=True)
        assert (dw.total <= SMALL) == (not beside)
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

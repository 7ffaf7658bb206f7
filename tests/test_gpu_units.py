"""One unit per thread, 4 KiB per work-group: every kind of chunk, on both sides of the image size up to which the loads
are ordinary ones, whole and in ranges that begin and end at and beside the pieces."""
import numpy as np
import pytest

from oracle import ds_oracle as orc
from workloads.configs import DTYPES, Shard, Workload

pytestmark = pytest.mark.gpu

CACHED = 64 << 20        # kCachedBytes of csrc/ds_kernels.hip
VIEWS = [("u8", (n,), (1,)) for n in (1, 7, 15, 16, 17, 4095, 4097, 12300)] + [
    ("i64", (1,), (1,)), ("bf16", (3,), (1,)), ("f32", (5000,), (1,)),
    ("u8", (300, 17), (23, 1)), ("u8", (41, 513), (700, 1)), ("bf16", (50, 121), (130, 1)), ("f32", (9, 2049), (2050, 1)),
    ("u8", (7, 5, 33), (1000, 170, 1)), ("bf16", (6, 7, 700), (9000, 1100, 1)), ("i64", (3, 4, 5, 9), (900, 200, 20, 1)),
    ("u8", (5, 3), (9, 2)), ("u8", (31, 5), (9, 1)), ("bf16", (11, 7), (1, 13)), ("f32", (4, 3, 3), (50, 11, 1)),
    ("i64", (13, 3), (7, 2)), ("u8", (9, 11), (12, 1))]


@pytest.mark.parametrize("total,align", [(0, 16), (0, 512), (CACHED, 64), (CACHED + 64, 64)])
def test_every_kind_of_chunk(total, align):
    import gpu_util as gu
    rng = np.random.default_rng(align)
    shards, at, image = [], 0, 0

    def add(dtype, shape, strides):
        nonlocal at, image
        es = DTYPES[dtype][1]
        at = -(-at // es) * es + es * int(rng.integers(0, 4))
        shards.append(Shard(f"s{len(shards)}", dtype, shape, strides, at, len(shards)))
        at += (sum((e - 1) * s for e, s in zip(shape, strides)) + 1) * es
        image = -(-(image + int(np.prod(shape)) * es) // align) * align
    for k in rng.permutation(3 * len(VIEWS)):
        add(*VIEWS[k % len(VIEWS)])
    if total:
        add("u8", (total - image - 5,), (1,))
    w = Workload("units", align, 0, rng.integers(0, 256, size=at + 64, dtype=np.uint8), shards)
    want, offs, tab = gu.oracle_image(w)
    dw = gu.DeviceWorkload(w)
    try:
        assert not total or dw.total == total
        print(f"[case] units total={dw.total} align={align}", flush=True)
        last = dw.total // 4096 * 4096
        cuts = [0, 16, 4080, 4096, 8208, 16384, 20464, 32768 + 4096, 65536 - 16, last - 16, last, dw.total]
        ranges = [(lo, hi) for lo, hi in zip(cuts, cuts[1:]) if lo < hi]
        for lo, hi in [(0, dw.total)] + ranges:
            assert gu.first_mismatch(dw.pack(lo, hi), want[lo:hi]) is None, (lo, hi)
        w.arena[:] = 0x5A
        orc.unpack(tab, len(shards), want)
        for parts in ([(0, dw.total)], ranges):
            dw.arena.fill_(0x5A)
            for lo, hi in parts:
                dw.unpack(want, lo, hi)
            assert gu.first_mismatch(dw.arena_host(), w.arena) is None, parts
    finally:
        dw.close()

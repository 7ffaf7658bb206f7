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


DIMS = [("u8", (40, 30, 1000), (31 * 1500, 1500, 1)), ("u8", (90, 33, 17), (33 * 23 + 5, 23, 1)),
        ("bf16", (6, 7, 9, 260), (40000, 5000, 512, 1)), ("f32", (5, 4, 3, 2, 4099), (300000, 70000, 20000, 9000, 1)),
        ("i64", (50, 20, 6), (200, 8, 1)), ("u8", (3, 70000, 16), (2000000, 24, 1)), ("bf16", (3, 2, 40001), (200000, 50000, 1)),
        ("f32", (20, 300, 4), (300 * 8 + 4, 8, 1))]


@pytest.mark.parametrize("blocks", [0, 1, 2])
@pytest.mark.parametrize("large", [0, CACHED])
def test_views_of_several_outer_dimensions(large, blocks):
    """Chunks inside such views (runs of 16 bytes to more than a chunk, units cut by a run's end at every place), alone,
    beside views moved in blocks in the same launch, and in a launch of their own."""
    import gpu_util as gu
    rng = np.random.default_rng(blocks)
    views = DIMS + ([("bf16", (301, 203), (1, 303))] if blocks else [])
    if blocks == 2:
        views = views + [("u8", (70 << 20,), (1,))]     # more chunks than share a launch
    if large:
        views = views + [("u8", (large,), (1,))]
    shards, at = [], 0
    for k, (dtype, shape, strides) in enumerate(views):
        es = DTYPES[dtype][1]
        at = -(-at // es) * es + es * int(rng.integers(0, 4))
        shards.append(Shard(f"d{k}", dtype, shape, strides, at, k))
        at += (sum((e - 1) * s for e, s in zip(shape, strides)) + 1) * es
    w = Workload("dims", 16, 0, rng.integers(0, 256, size=at + 64, dtype=np.uint8), shards)
    want, offs, tab = gu.oracle_image(w)
    dw = gu.DeviceWorkload(w)
    try:
        print(f"[case] several dimensions, blocks={blocks} image={dw.total}", flush=True)
        cuts = [0] + sorted(16 * int(x) for x in rng.integers(1, min(dw.total, 8 << 20) // 16, 9)) + [dw.total]
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


@pytest.mark.parametrize("chunks", [(1 << 22) - 17, (1 << 22) - 16])
def test_the_largest_image_with_one_unit_per_thread_and_the_next(chunks):
    """A launch has less than 2^32 threads: images of up to 2^22 - 17 chunks are moved one unit per thread, larger ones
    several.  One tensor whose last unit is cut, at an odd address, behind a small one."""
    import paper_2601_16956_amd as ds
    import torch
    n = chunks * 16384 - 64 - 5
    arena = torch.empty((n + 4096) // 8 + 8, dtype=torch.int64, device="cuda").random_()
    raw = arena.view(torch.uint8)
    shards = [Shard("a", "u8", (61,), (1,), 3, 0), Shard("b", "u8", (n,), (1,), 129, 1)]
    descs = ds.make_descs(shards, arena.data_ptr())
    total = ds.ds_layout_assign(descs, 2, 64)
    assert -(-total // 16384) == chunks
    plan = ds.ds_plan_create(descs, 2, 64, ds.DS_PLAN_CHECK_MEMORY)
    image = torch.full((total // 8,), -1, dtype=torch.int64, device="cuda")
    img, stream, step = image.view(torch.uint8), torch.cuda.current_stream().cuda_stream, 1 << 30

    def same():
        return (torch.equal(img[:61], raw[3:64]) and not img[61:64].any() and not img[64 + n:].any() and
                all(torch.equal(img[64 + at:64 + min(at + step, n)], raw[129 + at:129 + min(at + step, n)])
                    for at in range(0, n, step)))
    try:
        print(f"[case] {chunks} chunks", flush=True)
        ds.ds_pack(plan, image.data_ptr(), 0, total, stream)
        torch.cuda.synchronize()
        assert same()
        raw[:3].zero_()
        raw[64:129].fill_(7)
        raw[129 + n:].fill_(9)
        kept = [raw[:3].clone(), raw[64:129].clone(), raw[129 + n:].clone()]
        raw[3:64].zero_()
        raw[129:129 + n].zero_()
        ds.ds_unpack(plan, image.data_ptr(), 0, total, stream)
        torch.cuda.synchronize()
        assert same()
        assert all(torch.equal(a, b) for a, b in zip(kept, (raw[:3], raw[64:129], raw[129 + n:])))
    finally:
        torch.cuda.synchronize()
        ds.ds_plan_destroy(plan)

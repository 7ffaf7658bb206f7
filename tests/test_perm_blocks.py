"""The block route for views with runs shorter than 16 bytes (csrc/ds_perm.h): on the CPU thread by thread with
every access counted, and on the GPU against the oracle."""
import ctypes
import mmap
import os
import subprocess

import numpy as np
import pytest

from oracle import ds_oracle as orc
from workloads.configs import DTYPES, Shard, Workload

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

# (dtype, shape, strides in elements): blocks whole and cut on either side, rows that start anywhere in a unit, rows
# shorter than a unit, runs of several granules, batches, both walks, strides that do not nest
VIEWS = [
    ("bf16", (64, 128), (1, 64)), ("bf16", (129, 257), (1, 130)), ("bf16", (65, 1031), (1, 67)),
    ("f32", (64, 64), (1, 64)), ("f32", (63, 129), (1, 63)), ("f32", (200, 9), (1, 200)), ("f32", (7, 500), (1, 9)),
    ("u8", (128, 128), (1, 128)), ("u8", (131, 259), (1, 133)), ("u8", (300, 33), (1, 301)),
    ("i64", (32, 64), (1, 32)), ("i64", (33, 65), (1, 35)), ("i64", (2, 700), (1, 3)),
    ("bf16", (3, 70, 40), (70 * 40, 1, 70)), ("f32", (5, 37, 3, 3), (37 * 9, 1, 111, 37)),
    ("f32", (40, 48, 3, 3), (48 * 9, 1, 144, 48)), ("u8", (2, 3, 2, 25, 2, 60), (20000, 6100, 3000, 1, 1500, 25)),
    ("f32", (2100,), (2,)), ("u8", (5000,), (3,)), ("bf16", (70, 300), (800, 2)), ("i64", (3, 400), (900, 2)),
    ("bf16", (700, 6), (16, 1)), ("u8", (900, 11), (13, 1)), ("f32", (500, 3), (4, 1)), ("bf16", (60, 30, 6), (6, 400, 1)),
    ("u8", (90, 40, 5), (5, 460, 1)), ("f32", (33, 70, 2), (2, 66, 1)), ("u8", (40, 100, 1), (1, 41, 1)),
    ("bf16", (700, 2), (2, 3)), ("bf16", (64, 3, 2, 32), (1, 64, 192, 384)),
    ("bf16", (70, 8, 301), (1, 70, 560)),
    # runs of several granules at odd addresses, in rows that are not whole units
    ("u8", (200, 101, 8), (9, 1800, 1)), ("u8", (64, 300, 15), (15, 961, 1)), ("u8", (128, 101, 8), (8, 1025, 1)),
    ("u8", (130, 131, 12), (13, 1701, 1)), ("bf16", (70, 107, 7), (7, 491, 1)), ("bf16", (70, 203, 3), (3, 211, 1)),
    ("f32", (66, 203, 3), (3, 199, 1)), ("u8", (140, 301, 2), (3, 421, 1)),
]


def _normal(dtype, shape, strides):
    """What the plan makes of a view: outer extents and byte strides, run length."""
    es, dims = DTYPES[dtype][1], []
    for e, s in zip(shape, strides):
        if e == 1:
            continue
        if dims and dims[-1][1] == e * s:
            dims[-1] = (dims[-1][0] * e, s)
        else:
            dims.append((e, s))
    run = es
    if dims and dims[-1][1] == 1:
        run *= dims.pop()[0]
    return [e for e, _ in dims], [s * es for _, s in dims], run


@pytest.fixture(scope="module")
def host(tmp_path_factory):
    so = str(tmp_path_factory.mktemp("perm") / "perm_host.so")
    subprocess.run(["g++", "-O2", "-std=c++17", "-Wall", "-Werror", "-Wno-unknown-pragmas", "-fPIC", "-shared", "-I",
                    os.path.join(ROOT, "paper_2601_16956_amd", "csrc"),
                    os.path.join(ROOT, "tests", "c_abi", "perm_host.cpp"), "-o", so], check=True)
    lib = ctypes.CDLL(so)
    fn, launched = lib.perm_host_move, lib.perm_host_launched
    u64, vp = ctypes.c_uint64, ctypes.c_void_p
    fn.restype = ctypes.c_long
    fn.argtypes = [vp, u64, u64, u64, u64, u64, ctypes.c_uint32, vp, vp, ctypes.c_int, u64, u64, vp, vp, vp]
    launched.restype = u64
    fn.launched = launched
    return fn


def _check(host, dtype, shape, strides, shift, at, rng):
    es = DTYPES[dtype][1]
    extent, stride, run = _normal(dtype, shape, strides)
    ext, st = (ctypes.c_uint64 * 6)(*extent), (ctypes.c_uint64 * 6)(*stride)
    nbytes = int(np.prod(shape)) * es
    idx = np.zeros(shape, dtype=np.int64)
    for j, (e, s) in enumerate(zip(shape, strides)):
        idx += (np.arange(e) * s).reshape([-1 if i == j else 1 for i in range(len(shape))])
    byte = (idx.reshape(-1, 1) * es + np.arange(es)).reshape(-1) + shift * es      # of every image byte
    room = np.empty(int(byte.max()) + 64, dtype=np.uint8)
    start = -room.ctypes.data % 16
    arena = room[start:start + int(byte.max()) + 1]
    whole = nbytes & ~15
    for lo, hi in ((at, at + whole), (0, at + nbytes + 64), (at + 16, at + whole - 16),
                   (at + (whole // 3 & ~15), at + (whole // 2 & ~15))):
        inside = np.arange(max(lo, at), min(hi, at + whole))
        arena[:] = rng.integers(0, 256, arena.size)
        raw = np.empty(hi - lo + 16, dtype=np.uint8)
        img = raw[-raw.ctypes.data % 16:][:hi - lo]
        want_hits = np.zeros(arena.size, dtype=bool)
        want_hits[byte[inside - at]] = True
        for pack in (1, 0):
            ah, ih = np.zeros(arena.size, dtype=np.uint8), np.zeros(hi - lo, dtype=np.uint8)
            if pack:
                img[:] = 0xAA
                want = img.copy()
                want[inside - lo] = arena[byte[inside - at]]
            else:
                img[:] = rng.integers(0, 256, hi - lo)
                want = arena.copy()
                want[byte[inside - at]] = img[inside - lo]
            n = host(arena.ctypes.data, arena.size, shift * es, at, nbytes, run, len(extent), ext, st, pack, lo, hi,
                     img.ctypes.data, ah.ctypes.data, ih.ctypes.data)
            assert n >= 0, "an access out of bounds"
            if n == 0:
                return 0
            if pack:
                assert np.array_equal(img, want)
                assert not ah[np.setdiff1d(np.arange(arena.size), byte)].any(), "read outside the view"
                assert np.array_equal(np.flatnonzero(ih), inside - lo) and ih.max(initial=0) <= 1, "image bytes written once each"
            else:
                assert np.array_equal(arena, want)
                assert np.array_equal(ah > 0, want_hits) and ah.max(initial=0) <= 1, "view bytes written once each"
    return n


@pytest.mark.parametrize("k", range(len(VIEWS)))
def test_blocks_move_exactly_the_view(host, k):
    dtype, shape, strides = VIEWS[k]
    rng = np.random.default_rng(k)
    for shift, at in ((0, 0), (1, 16), (3, 4096)):
        assert _check(host, dtype, shape, strides, shift, at, rng) > 0


# views in wide blocks: the smallest, rows that are whole lines of the image and rows that are not, the last block of a row
# and of the steps along a nearly empty or full, rows at every place in a unit, batches on either side of a
WIDE = [
    ("bf16", (64, 256), (1, 64)), ("bf16", (72, 257), (1, 72)), ("bf16", (136, 1031), (1, 140)), ("bf16", (64, 384), (1, 64)),
    ("bf16", (120, 577), (1, 121)), ("u8", (64, 512), (1, 64)), ("u8", (80, 1031), (1, 81)), ("u8", (144, 737), (1, 144)),
    ("f32", (64, 128), (1, 64)), ("f32", (68, 129), (1, 68)), ("f32", (132, 277), (1, 133)), ("i64", (64, 64), (1, 64)),
    ("i64", (66, 65), (1, 67)), ("i64", (130, 187), (1, 130)), ("bf16", (3, 64, 300), (64 * 300, 1, 64)),
    ("f32", (70, 3, 192), (576, 1, 3)), ("f32", (72, 3, 192), (1, 72, 216)), ("u8", (2, 64, 3, 514), (99000, 1, 32896, 64)),
]


@pytest.mark.parametrize("k", range(len(WIDE)))
def test_wide_blocks_move_exactly_the_view(host, k):
    dtype, shape, strides = WIDE[k]
    rng = np.random.default_rng(k)
    for shift, at in ((0, 0), (1, 16), (3, 4096), (0, 80)):
        assert _check(host, dtype, shape, strides, shift, at, rng) > 0


@pytest.mark.parametrize("dtype,shape,strides", [
    ("bf16", (64, 64), (1, 20000001)), ("bf16", (64, 104), (1, 20000001)), ("u8", (128, 32), (1, 50000001)),
    ("f32", (64, 20), (1, 18000001)), ("i64", (32, 50), (1, 9000001)),
    # on both sides of the distance up to which wide blocks are taken: (129 + 128) columns in 2^31 bytes
    ("bf16", (64, 257), (1, 4177983)), ("bf16", (64, 257), (1, 4177984))])
def test_columns_far_apart(host, dtype, shape, strides):
    """Columns so far apart that 32 bits do not hold the distance over the columns of a usual block: nothing but the
    view is read or written (memory of which only the view's pages exist)."""
    es = DTYPES[dtype][1]
    extent, stride, run = _normal(dtype, shape, strides)
    nbytes, span = int(np.prod(shape)) * es, ((shape[0] - 1) * strides[0] + (shape[1] - 1) * strides[1] + 1) * es
    idx = np.arange(shape[0]).reshape(-1, 1) * strides[0] + np.arange(shape[1]) * strides[1]
    byte = (idx.reshape(-1, 1) * es + np.arange(es)).reshape(-1)
    flags = mmap.MAP_PRIVATE | mmap.MAP_ANONYMOUS | getattr(mmap, "MAP_NORESERVE", 0x4000)
    arena = np.frombuffer(mmap.mmap(-1, span, flags=flags), dtype=np.uint8)
    want = np.random.default_rng(3).integers(0, 256, nbytes, dtype=np.uint8)
    img = np.zeros(nbytes + 16, dtype=np.uint8)
    img = img[-img.ctypes.data % 16:][:nbytes]
    for pack in (1, 0):
        hits = np.frombuffer(mmap.mmap(-1, span, flags=flags), dtype=np.uint8)
        image_hits = np.zeros(nbytes, dtype=np.uint8)
        if pack:
            arena[byte] = want
        else:
            arena[byte] = 0
            img[:] = want
        n = host(arena.ctypes.data, span, 0, 0, nbytes, run, len(extent), (ctypes.c_uint64 * 6)(*extent),
                 (ctypes.c_uint64 * 6)(*stride), pack, 0, nbytes, img.ctypes.data, hits.ctypes.data,
                 image_hits.ctypes.data)
        assert n > 0
        assert np.array_equal(img if pack else arena[byte], want)
        assert hits[byte].all()
        hits[byte] = 0
        assert hits.max() == 0, "an access outside the view"


@pytest.mark.parametrize("dtype,shape,strides", [
    ("bf16", (1200, 1501), (1, 1203)), ("f32", (60, 70, 3, 3), (630, 1, 210, 70)), ("u8", (700001,), (2,)),
    ("bf16", (600, 4, 301), (1, 600, 2400)), ("f32", (300, 900), (2000, 2)), ("u8", (5, 60, 16, 100), (16, 80, 1, 4801))])
def test_blocks_follow_the_range(host, dtype, shape, strides):
    """An image moved in parts has few more blocks than one moved whole, and all its bytes are moved."""
    es = DTYPES[dtype][1]
    extent, stride, run = _normal(dtype, shape, strides)
    nbytes = int(np.prod(shape)) * es
    idx = sum((np.arange(e) * s).reshape([-1 if i == j else 1 for i in range(len(shape))])
              for j, (e, s) in enumerate(zip(shape, strides)))
    byte = (idx.reshape(-1, 1) * es + np.arange(es)).reshape(-1)
    rng = np.random.default_rng(len(shape))
    arena = rng.integers(0, 256, int(byte.max()) + 17, dtype=np.uint8)
    arena = arena[-arena.ctypes.data % 16:][:int(byte.max()) + 1]
    whole, at = nbytes & ~15, 48
    img = np.zeros(nbytes + 64, dtype=np.uint8)
    img = img[-img.ctypes.data % 16:]
    ah, ih = np.zeros(arena.size, dtype=np.uint8), np.zeros(nbytes + 64, dtype=np.uint8)

    def move(lo, hi):
        before = host.launched()
        n = host(arena.ctypes.data, arena.size, 0, at, nbytes, run, len(extent), (ctypes.c_uint64 * 6)(*extent),
                 (ctypes.c_uint64 * 6)(*stride), 1, lo, hi, img.ctypes.data + lo - at, ah.ctypes.data, ih.ctypes.data)
        assert n > 0
        return n, host.launched() - before
    n, all_of_them = move(at, at + whole)
    assert all_of_them == n
    img[:] = 0
    cuts = [at] + sorted({at + 16 * int(x) for x in rng.integers(1, whole // 16, 11)}) + [at + whole]
    total = sum(move(lo, hi)[1] for lo, hi in zip(cuts, cuts[1:]))
    assert np.array_equal(img[:whole], arena[byte[:whole]])
    assert total <= 3 * n, (total, n)


def test_random_permuted_views(host):
    """Slices and permutations of dense parents of one to six dimensions: whatever the route accepts it moves
    exactly; what it leaves to the other paths it does not touch."""
    rng = np.random.default_rng(11)
    taken = 0
    for trial in range(150):
        nd = int(rng.integers(1, 7))
        dtype = list(DTYPES)[trial % 5]
        full = [max(1, int(round((30000 ** (1 / nd)) * rng.uniform(0.3, 2)))) for _ in range(nd)]
        strides = [int(np.prod(full[j + 1:], dtype=np.int64)) for j in range(nd)]
        shape, step = list(full), [int(rng.integers(1, 3)) if rng.random() < 0.3 else 1 for _ in range(nd)]
        shape = [max(1, (e - int(rng.integers(0, max(1, e // 3)))) // s) for e, s in zip(shape, step)]
        strides = [s * t for s, t in zip(strides, step)]
        order = rng.permutation(nd)
        taken += _check(host, dtype, tuple(shape[j] for j in order), tuple(strides[j] for j in order),
                        int(rng.integers(0, 4)), 16 * int(rng.integers(0, 9)), rng) > 0
    assert taken > 30


@pytest.mark.gpu
@pytest.mark.parametrize("chunk_bytes", [16384, 8192, 32768])
def test_gather_and_scatter_of_permuted_views(chunk_bytes):
    """The same views in one table, with a large one of each walk, whole and in ranges that cut blocks."""
    import paper_2601_16956_amd as ds
    import gpu_util as gu
    import torch
    rng = np.random.default_rng(5)
    big = [("bf16", (1000, 1531), (1, 1000)), ("f32", (333, 1111), (2222, 2)), ("u8", (700, 901), (1, 701)),
           ("i64", (130, 513), (1, 131))]
    shards, at = [], 0
    for k, (dtype, shape, strides) in enumerate(VIEWS + big + [("u8", (777,), (1,))]):
        es = DTYPES[dtype][1]
        span = (sum((e - 1) * s for e, s in zip(shape, strides)) + 1) * es
        start = -(-at // 256) * 256 + es * int(rng.integers(0, 4))
        shards.append(Shard(f"p{k}", dtype, shape, strides, start, k))
        at = start + span
    arena = rng.integers(0, 256, size=at + 64, dtype=np.uint8)
    w = Workload("perm", 64, 0, arena, shards)
    want, offs, tab = gu.oracle_image(w)
    old = ds.ds_config_get("chunk_bytes")
    ds.ds_config_set("chunk_bytes", chunk_bytes)
    try:
        dw = gu.DeviceWorkload(w)
        try:
            print(f"[case] permuted views chunk={chunk_bytes} image={dw.total}", flush=True)
            got = dw.pack()
            assert gu.first_mismatch(got, want) is None, gu.first_mismatch(got, want)
            cuts = [0] + sorted(16 * int(x) for x in rng.integers(1, dw.total // 16, 9)) + [dw.total]
            ranges = [(lo, hi) for lo, hi in zip(cuts, cuts[1:]) if lo < hi]
            for lo, hi in ranges:
                assert gu.first_mismatch(dw.pack(lo, hi), want[lo:hi]) is None, (lo, hi)
            out = torch.full((dw.total,), 0xFF, dtype=torch.uint8, device="cuda")
            ds.ds_pack_noalloc(dw.plan, out.data_ptr(), 0, dw.total, torch.cuda.current_stream().cuda_stream)
            assert gu.first_mismatch(out.cpu().numpy(), want) is None
            w.arena[:] = 0x5A
            orc.unpack(tab, len(shards), want)
            for parts in ([(0, dw.total)], ranges):
                dw.arena.fill_(0x5A)
                for lo, hi in parts:
                    dw.unpack(want, lo, hi)
                assert gu.first_mismatch(dw.arena_host(), w.arena) is None
        finally:
            dw.close()
    finally:
        ds.ds_config_set("chunk_bytes", old)


@pytest.mark.gpu
@pytest.mark.parametrize("shift", [0, 1])
def test_gather_and_scatter_in_wide_blocks(shift):
    """Views in wide blocks with columns at multiples of 64 bytes (shift 0: the scatter's stores stream) and at odd
    elements, whole and in ranges that cut blocks."""
    import paper_2601_16956_amd as ds
    import gpu_util as gu
    rng = np.random.default_rng(6)
    big = [("bf16", (1024, 1531), (1, 1024)), ("f32", (512, 1111), (1, 512)), ("u8", (704, 1901), (1, 704)),
           ("i64", (130, 513), (1, 136)), ("bf16", (2, 512, 768), (512 * 768, 1, 512))]
    shards, at = [], 0
    for k, (dtype, shape, strides) in enumerate(WIDE + big):
        es = DTYPES[dtype][1]
        start = -(-at // 256) * 256 + es * shift
        shards.append(Shard(f"w{k}", dtype, shape, strides, start, k))
        at = start + (sum((e - 1) * s for e, s in zip(shape, strides)) + 1) * es
    w = Workload("wide", 64, 0, rng.integers(0, 256, size=at + 64, dtype=np.uint8), shards)
    want, offs, tab = gu.oracle_image(w)
    dw = gu.DeviceWorkload(w)
    try:
        print(f"[case] wide blocks shift={shift} image={dw.total}", flush=True)
        cuts = [0] + sorted(16 * int(x) for x in rng.integers(1, dw.total // 16, 9)) + [dw.total]
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
@pytest.mark.parametrize("beside", [1 << 20, 62 << 20, 70 << 20])
def test_blocks_beside_other_chunks(beside):
    """Blocks and the other chunks in one launch (up to 4096 such chunks; images on both sides of the size read with
    ordinary loads) and in two: tensor ends, rows, padding and views of several dimensions among the other chunks."""
    import gpu_util as gu
    rng = np.random.default_rng(beside >> 20)
    views = [("bf16", (1024, 1531), (1, 1024)), ("u8", (300, 33), (1, 301)), ("u8", (41, 513), (700, 1)),
             ("u8", (beside // 3 + 7,), (1,)), ("f32", (333, 111), (222, 2)), ("i64", (3, 4, 5, 9), (900, 200, 20, 1)),
             ("bf16", (beside // 6 // 1000, 1000), (1012, 1)), ("f32", (512, 4099), (1, 512)), ("bf16", (3,), (1,)),
             ("u8", (beside // 3 + 5,), (1,)), ("u8", (80, 1031), (1, 81)), ("bf16", (11, 7), (1, 13))]
    shards, at = [], 0
    for k, (dtype, shape, strides) in enumerate(views):
        es = DTYPES[dtype][1]
        at = -(-at // 64) * 64 + es * int(rng.integers(0, 3))
        shards.append(Shard(f"b{k}", dtype, shape, strides, at, k))
        at += (sum((e - 1) * s for e, s in zip(shape, strides)) + 1) * es
    w = Workload("beside", 64, 0, rng.integers(0, 256, size=at + 64, dtype=np.uint8), shards)
    want, offs, tab = gu.oracle_image(w)
    dw = gu.DeviceWorkload(w)
    try:
        print(f"[case] blocks beside {beside} bytes, image={dw.total}", flush=True)
        cuts = [0] + sorted(16 * int(x) for x in rng.integers(1, dw.total // 16, 5)) + [dw.total]
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
def test_allocation_free_gather_without_room_for_the_block_tables():
    """Tables that fit the static array only without those of the blocks: the general path moves the views then."""
    import paper_2601_16956_amd as ds
    import gpu_util as gu
    import torch
    rng = np.random.default_rng(9)
    shards, at = [], 0
    for k in range(20000):
        n = 24 if k % 5000 else 190                          # four of them hold whole chunks
        shards.append(Shard(f"p{k}", "bf16", (n, n), (1, n + k % 3), at, k))
        at += 2 * n * (n + 2)
    w = Workload("many views", 64, 0, rng.integers(0, 256, size=at + 64, dtype=np.uint8), shards)
    want, offs, tab = gu.oracle_image(w)
    dw = gu.DeviceWorkload(w)
    try:
        print("[case] noalloc without block tables", flush=True)
        base = 168 * dw.info["n_tiles"] + 36 * dw.info["n_chunks"] + 512
        assert base <= 4 << 20 < base + 176 * len(shards)
        plan = ds.ds_plan_create(dw.descs, dw.n, w.align, ds.DS_PLAN_HOST_ONLY)
        out = torch.full((2, dw.total), 0xFF, dtype=torch.uint8, device="cuda")
        stream = torch.cuda.current_stream().cuda_stream
        ds.ds_pack_noalloc(plan, out[0].data_ptr(), 0, dw.total, stream)
        ds.ds_pack_noalloc(dw.plan, out[1].data_ptr(), 0, dw.total, stream)
        for image in out.cpu().numpy():
            assert gu.first_mismatch(image, want) is None
        ds.ds_plan_destroy(plan)
        assert gu.first_mismatch(dw.pack(), want) is None
    finally:
        dw.close()

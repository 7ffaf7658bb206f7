"""Tables of mostly small tensors with views among them, which the general path takes in the launch of mostly general
chunks: row views, and views of which another launch moves the whole units.  Against the oracle, whole and in ranges."""
import numpy as np
import pytest

from oracle import ds_oracle as orc
from workloads.configs import DTYPES, Shard, Workload

pytestmark = pytest.mark.gpu


def _table(views, rng):
    """6000 tensors of 1 to 900 bytes, each of the views behind some of them."""
    shards, at = [], 0

    def add(name, dtype, shape, strides, gap):
        nonlocal at
        es = DTYPES[dtype][1]
        at = -(-at // es) * es + gap * es
        shards.append(Shard(name, dtype, shape, strides, at, len(shards)))
        at += (sum((e - 1) * s for e, s in zip(shape, strides)) + 1) * es
    every = 6000 // len(views)
    for k in range(6000):
        dtype = ("u8", "bf16", "f32", "i64")[k % 4]
        n = max(1, int(rng.integers(1, 900)) // DTYPES[dtype][1])
        add(f"s{k}", dtype, (n,), (1,), int(rng.integers(0, 3)))
        if k % every == every // 2:
            add(f"v{k}", *views[k // every], int(rng.integers(0, 3)))
    return Workload("mixed", 64, 0, rng.integers(0, 256, size=at + 64, dtype=np.uint8), shards)


VIEWS = {"rows": [("u8", (40 + k, 300 + k), (450 + 3 * k, 1)) for k in range(9)],
         "transposed": [("bf16", (90 + 30 * k, 70 + 11 * k), (1, 95 + 30 * k)) for k in range(9)],
         "small transposed": [("bf16", (24 + k, 23 + k), (1, 30 + k)) for k in range(9)]}


@pytest.mark.parametrize("grid_limit", [0, 40])
@pytest.mark.parametrize("chunk_bytes", [8192, 16384, 32768])
@pytest.mark.parametrize("views", VIEWS)
def test_small_tensors_beside_views(views, chunk_bytes, grid_limit):
    rng = np.random.default_rng(chunk_bytes)
    _check(_table(VIEWS[views], rng), chunk_bytes, grid_limit, f"small tensors beside {views}", rng)


@pytest.mark.parametrize("chunk_bytes", [8192, 16384])
def test_a_large_table_with_one_transposed_view(chunk_bytes):
    """More chunks than a plan always lists, a few of which the blocks cover."""
    rng = np.random.default_rng(chunk_bytes)
    n = 4097 * chunk_bytes + 48
    shards = [Shard("a", "u8", (n,), (1,), 16, 0), Shard("t", "bf16", (301, 203), (1, 303), n + 64, 1),
              Shard("b", "u8", (n,), (1,), n + 64 + 2 * 303 * 203, 2)]
    _check(Workload("large", 64, 0, rng.integers(0, 256, size=2 * n + 200000, dtype=np.uint8), shards), chunk_bytes, 0,
           "one transposed view", rng)


@pytest.mark.parametrize("chunk_bytes", [8192, 16384, 32768])
def test_much_padding_behind_views_of_several_dimensions(chunk_bytes):
    """What is left of a view that is moved in blocks: its cut unit and more than 8 KiB of padding."""
    rng = np.random.default_rng(chunk_bytes)
    shards = [Shard(f"p{k}", "u8", (5 + k % 3, 65 + k, 17), (1400, 1, 80), 10000 * k + k, k) for k in range(9)]
    _check(Workload("padded", 32768, 0, rng.integers(0, 256, size=90000, dtype=np.uint8), shards), chunk_bytes, 0,
           "padding", rng)


def _check(w, chunk_bytes, grid_limit, what, rng):
    import paper_2601_16956_amd as ds
    import gpu_util as gu
    want, offs, tab = gu.oracle_image(w)
    old = [(key, ds.ds_config_get(key)) for key in ("chunk_bytes", "grid_limit")]
    ds.ds_config_set("chunk_bytes", chunk_bytes)
    ds.ds_config_set("grid_limit", grid_limit)
    try:
        dw = gu.DeviceWorkload(w)
        try:
            print(f"[case] {what} chunk={chunk_bytes} grid={grid_limit}", flush=True)
            cuts = [0] + sorted(16 * int(x) for x in rng.integers(1, dw.total // 16, 6)) + [dw.total]
            ranges = [(lo, hi) for lo, hi in zip(cuts, cuts[1:]) if lo < hi]
            for lo, hi in [(0, dw.total)] + ranges:
                assert gu.first_mismatch(dw.pack(lo, hi), want[lo:hi]) is None, (lo, hi)
            w.arena[:] = 0x5A
            orc.unpack(tab, len(w.shards), want)
            for parts in ([(0, dw.total)], ranges):
                dw.arena.fill_(0x5A)
                for lo, hi in parts:
                    dw.unpack(want, lo, hi)
                assert gu.first_mismatch(dw.arena_host(), w.arena) is None, parts
        finally:
            dw.close()
    finally:
        for key, value in old:
            ds.ds_config_set(key, value)


BY_LANES = [("u8", (20, 20), (1, 20)), ("u8", (3, 7), (9, 2)), ("bf16", (5, 7, 9), (1, 50, 5)), ("bf16", (31, 2), (2, 64)),
            ("f32", (10, 20), (40, 2)), ("f32", (3, 3, 3, 3), (200, 1, 31, 5)), ("i64", (7, 5), (1, 8)), ("i64", (2,), (3,)),
            ("u8", (1, 1), (1, 1)), ("bf16", (29, 17), (1, 31))]


@pytest.mark.parametrize("grid_limit", [0, 7])
@pytest.mark.parametrize("chunk_bytes", [8192, 16384, 32768])
def test_units_moved_an_element_per_lane(chunk_bytes, grid_limit):
    """Few views with runs of one element, of every itemsize: many in a wavefront's units and one by itself, with last
    units of every length, and what is left of views that are moved in blocks."""
    rng = np.random.default_rng(chunk_bytes + grid_limit)
    shards, at = [], 0
    views = [BY_LANES[k % len(BY_LANES)] for k in range(150)] + [("u8", (50000,), (1,)), BY_LANES[0], ("u8", (90000,), (1,)),
             ("bf16", (91, 91), (1, 91)), ("u8", (121, 121), (1, 121)), ("f32", (75, 75), (1, 75)),
             ("i64", (33, 41), (1, 33)), ("u8", (11, 300, 3), (3, 40, 1)), BY_LANES[4]]
    for k, (dtype, shape, strides) in enumerate(views):
        es = DTYPES[dtype][1]
        at = -(-at // es) * es + es * int(rng.integers(0, 3))
        shards.append(Shard(f"l{k}", dtype, shape, strides, at, k))
        at += (sum((e - 1) * s for e, s in zip(shape, strides)) + 1) * es
    _check(Workload("lanes", 16, 0, rng.integers(0, 256, size=at + 64, dtype=np.uint8), shards), chunk_bytes, grid_limit,
           "an element per lane", rng)


@pytest.mark.parametrize("nbytes,n,view", [
    (4000, 4500, ("u8", (41, 513), (700, 1))), (4000, 4500, ("bf16", (301, 203), (1, 303))), (9000, 7600, ("f32", (75, 25), (31, 1))),
    (16100, 4700, ("bf16", (31, 25), (1, 33)))])
def test_many_small_tensors_beside_a_view_in_larger_images(nbytes, n, view):
    """The launch of four units per thread: images on both sides of the size read with ordinary loads, in the list beside
    blocks and alone, with tensors below 16 bytes among the others."""
    rng = np.random.default_rng(n)
    shards, at = [], 3
    for k in range(n):
        size = nbytes + k % 61 if k % 100 else 1 + k // 100 % 15
        shards.append(Shard(f"t{k}", "u8", (size,), (1,), at, len(shards)))
        at += size + k % 5
        if k == n // 2:
            dtype, shape, strides = view
            at = -(-at // 8) * 8
            shards.append(Shard("view", dtype, shape, strides, at, len(shards)))
            at += (sum((e - 1) * s for e, s in zip(shape, strides)) + 1) * DTYPES[dtype][1]
    _check(Workload("several", 16, 0, rng.integers(0, 256, size=at + 64, dtype=np.uint8), shards), 16384, 0, "several", rng)

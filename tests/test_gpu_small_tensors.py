"""Plans in which most chunks hold several contiguous tensors and none a strided one: the path without the scan.
Tensors of 1 to 70 bytes around every boundary of a 16-byte unit, up to 1024 of them per chunk (2048 with chunks of
32 KiB, which is more than the path takes), holes, the image's short last chunk and ranges that cut tensors."""
import numpy as np
import pytest

from oracle import ds_oracle as orc
from workloads.configs import DTYPES, Shard, Workload

pytestmark = pytest.mark.gpu


def _table(sizes, align, rng, holes):
    shards, offsets, at, img = [], [], 0, 16 * 5 * align if holes else 0
    for k, size in enumerate(sizes):
        dtype = ("u8", "bf16", "f32", "i64")[k % 4]
        es = DTYPES[dtype][1]
        n = max(1, size // es)
        at = -(-at // es) * es + es * int(rng.integers(0, 3))
        shards.append(Shard(f"s{k}", dtype, (n,), (1,), at, k))
        at += n * es
        offsets.append(img)
        img = -(-(img + n * es) // align) * align + (align * int(rng.integers(0, 4)) if holes and k % 97 == 0 else 0)
    return shards, offsets, at


@pytest.mark.parametrize("chunk_bytes", [8192, 16384, 32768])
@pytest.mark.parametrize("align,sizes,holes", [
    (16, "tiny", False), (16, "units", True), (64, "units", False), (512, "mixed", True), (16, "large", True)])
def test_small_contiguous_tensors(chunk_bytes, align, sizes, holes):
    import paper_2601_16956_amd as ds
    import gpu_util as gu
    rng = np.random.default_rng(align + len(sizes))
    size = {"tiny": rng.integers(1, 17, 9000), "units": rng.integers(1, 71, 9000),
            "mixed": np.exp(rng.uniform(0, np.log(9000), 3000)).astype(int),
            "large": np.exp(rng.uniform(np.log(3000), np.log(30000), 300)).astype(int)}[sizes]
    shards, offsets, span = _table([int(x) for x in size], align, rng, holes)
    w = Workload("small", align, 0, rng.integers(0, 256, size=span + 64, dtype=np.uint8), shards)
    want, offs, tab = gu.oracle_image(w, offsets=offsets)
    old = ds.ds_config_get("chunk_bytes")
    ds.ds_config_set("chunk_bytes", chunk_bytes)
    try:
        dw = gu.DeviceWorkload(w, offsets=offsets)
        try:
            print(f"[case] small tensors {sizes} align={align} chunk={chunk_bytes}", flush=True)
            assert dw.info["n_general_chunks"] * 2 > dw.info["n_chunks"]
            got = dw.pack()
            assert gu.first_mismatch(got, want) is None, gu.first_mismatch(got, want)
            cuts = [0] + sorted(16 * int(x) for x in rng.integers(1, dw.total // 16, 6)) + [dw.total]
            ranges = [(lo, hi) for lo, hi in zip(cuts, cuts[1:]) if lo < hi]
            for lo, hi in ranges:
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
    finally:
        ds.ds_config_set("chunk_bytes", old)


def test_images_beyond_the_size_moved_with_ordinary_loads():
    """The same path in an image of more than 64 MiB, up to which the loads are ordinary ones."""
    import gpu_util as gu
    rng = np.random.default_rng(8)
    shards, offsets, span = _table([int(x) for x in rng.integers(7000, 9500, 8400)], 16, rng, False)
    w = Workload("small", 16, 0, rng.integers(0, 256, size=span + 64, dtype=np.uint8), shards)
    want, offs, tab = gu.oracle_image(w, offsets=offsets)
    dw = gu.DeviceWorkload(w, offsets=offsets)
    try:
        print(f"[case] small tensors, image of {dw.total}", flush=True)
        assert dw.total > 64 << 20 and dw.info["n_general_chunks"] * 2 > dw.info["n_chunks"]
        assert gu.first_mismatch(dw.pack(), want) is None
        w.arena[:] = 0x5A
        orc.unpack(tab, len(shards), want)
        dw.arena.fill_(0x5A)
        dw.unpack(want, 0, dw.total)
        assert gu.first_mismatch(dw.arena_host(), w.arena) is None
    finally:
        dw.close()

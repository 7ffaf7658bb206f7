"""ds_image_compress with blocks larger than the image, up to the largest power of two that 64 bits hold; how
many work-groups look at a block."""
import ctypes
import os
import subprocess

import numpy as np
import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.fixture(scope="module")
def lib(tmp_path_factory):
    so = str(tmp_path_factory.mktemp("blocks") / "blocks_host.so")
    subprocess.run(["g++", "-O2", "-std=c++17", "-Wall", "-Werror", "-fPIC", "-shared", "-I",
                    os.path.join(ROOT, "paper_2601_16956_amd", "csrc"),
                    os.path.join(ROOT, "tests", "c_abi", "blocks_host.cpp"), "-o", so], check=True)
    lib = ctypes.CDLL(so)
    lib.blocks_host_place.restype = None
    lib.blocks_host_place.argtypes = [ctypes.c_uint64, ctypes.c_uint32, ctypes.c_void_p]
    lib.blocks_host_parts_log2.argtypes = [ctypes.c_uint64, ctypes.c_uint32]
    return lib


def test_place_of_a_unit_in_blocks_of_every_size(lib):
    out = (ctypes.c_uint64 * 2)()
    for log2 in range(10, 60):
        for unit in (0, 1, 256, 1024, (1 << 22) - 256, (1 << 22) - 1, 1 << 31, 1 << 32, (1 << 32) + 1024, (1 << 36) + 7):
            lib.blocks_host_place(unit, log2, out)
            assert tuple(out) == divmod(unit, 1 << log2), (unit, log2)


def test_no_work_group_looks_at_more_than_256_KiB(lib):
    for nbytes in (1 << 14, 1 << 20, 16 << 20):
        parts = {b: lib.blocks_host_parts_log2(nbytes, b - 4) for b in range(14, 64)}
        assert {b: p for b, p in parts.items() if p >= 0} == {17: 0, 18: 0, 19: 2, 20: 2}
    for nbytes in ((16 << 20) + 16, 64 << 20, 1 << 40):
        assert all(lib.blocks_host_parts_log2(nbytes, b - 4) == -1 for b in range(14, 64))


@pytest.mark.gpu
@pytest.mark.parametrize("block_log2", [21, 31, 35, 36, 37, 40, 63])
@pytest.mark.parametrize("nbytes", [16, 65536 + 16, (8 << 20) - 16, (9 << 20) + 48, (65 << 20) + 16])
def test_one_block_larger_than_the_image(block_log2, nbytes):
    """One unit per thread (up to 8 MiB), four, and the scan and the pack as launches of their own (more than 64 MiB)."""
    import torch

    import paper_2601_16956_amd as ds
    gen = torch.Generator(device="cuda").manual_seed(nbytes)
    n_blocks = -(-nbytes // (1 << block_log2))
    for constant in (True, False):
        img = torch.randint(0, 256, (nbytes,), dtype=torch.uint8, device="cuda", generator=gen)
        if constant:
            img = img[:16].repeat(nbytes // 16)
        keep = torch.full((n_blocks + 2,), 9, dtype=torch.int32, device="cuda")
        pos = torch.full((n_blocks + 3,), 9, dtype=torch.int32, device="cuda")
        pats = torch.full((n_blocks + 1, 16), 0xCC, dtype=torch.uint8, device="cuda")
        packed = torch.full((nbytes + 64,), 0xCC, dtype=torch.uint8, device="cuda")
        print(f"[case] compress {nbytes} bytes in blocks of 2^{block_log2}, constant={constant}", flush=True)
        ds.ds_image_compress(img.data_ptr(), nbytes, 1 << block_log2, keep.data_ptr(), pos.data_ptr(), pats.data_ptr(),
                             packed.data_ptr(), torch.cuda.current_stream().cuda_stream)
        torch.cuda.synchronize()
        blocks = [img[k << block_log2:(k + 1) << block_log2] for k in range(n_blocks)]
        kept = [int(bool((b.view(-1, 16) != b[:16]).any())) for b in blocks]
        assert keep.tolist() == kept + [9, 9]
        assert pos.tolist() == np.concatenate([[0], np.cumsum(kept)]).tolist() + [9, 9]
        assert torch.equal(pats[:-1], torch.stack([b[:16] for b in blocks])) and bool((pats[-1] == 0xCC).all())
        want = torch.cat([b for b, k in zip(blocks, kept) if k] + [img[:0]])
        assert torch.equal(packed[:want.numel()], want) and bool((packed[want.numel():] == 0xCC).all())


@pytest.mark.gpu
@pytest.mark.parametrize("together", [2, 7])
@pytest.mark.parametrize("block_log2", [16, 17, 18, 19, 20])
def test_the_only_unit_that_differs(block_log2, together):
    """On both sides of the blocks that one work-group looks at and that four do: the first unit behind the reference, those
    around a work-group's first 16 KiB, its steps and its part, the last one; constant blocks between them; a short last block.
    Images of up to 6 MiB and of more."""
    import torch

    import paper_2601_16956_amd as ds
    block, units = 1 << block_log2, 1 << block_log2 - 4
    every = sorted({u for u in (1, 1023, 1024, 4095, 4096, 8191, 8192, 16383, 16384, 17407, 17408, 32768, 49151, units - 1)
                    if u < units})
    rng = np.random.default_rng(block_log2)
    for at in (every[k:k + together] for k in range(0, len(every), together)):
        img = np.repeat(rng.integers(0, 256, (2 * len(at) + 1, 1, 16), dtype=np.uint8), units, axis=1)
        for k, u in enumerate(at):
            img[2 * k, u, int(rng.integers(0, 16))] ^= 1
        n_blocks, nbytes = len(img), img.size - block // 2
        dev = torch.from_numpy(img.reshape(-1)).cuda()
        keep = torch.full((n_blocks + 1,), 9, dtype=torch.int32, device="cuda")
        pos = torch.full((n_blocks + 1,), 9, dtype=torch.int32, device="cuda")
        pats = torch.full((n_blocks, 16), 0xCC, dtype=torch.uint8, device="cuda")
        packed = torch.full((n_blocks * block,), 0xCC, dtype=torch.uint8, device="cuda")
        print(f"[case] compress {n_blocks} blocks of {block}", flush=True)
        ds.ds_image_compress(dev.data_ptr(), nbytes, block, keep.data_ptr(), pos.data_ptr(), pats.data_ptr(), packed.data_ptr(),
                             torch.cuda.current_stream().cuda_stream)
        torch.cuda.synchronize()
        assert keep.tolist() == [1, 0] * len(at) + [0, 9]
        assert pos.tolist() == [(k + 1) // 2 for k in range(2 * len(at))] + [len(at)] * 2
        assert np.array_equal(pats.cpu().numpy(), img[:, 0])
        assert np.array_equal(packed[:len(at) * block].cpu().numpy(), img[:-1:2].reshape(-1))
        assert bool((packed[len(at) * block:] == 0xCC).all())


@pytest.mark.gpu
@pytest.mark.parametrize("nbytes", [(3 << 20) + 16, 12 << 20])
def test_replays_of_a_captured_call(nbytes):
    """Flags that four work-groups leave and one makes whole, again on every replay, for other images in the same buffers."""
    import torch

    import paper_2601_16956_amd as ds
    block = 1 << 19
    n_blocks = -(-nbytes // block)
    img = torch.zeros(nbytes, dtype=torch.uint8, device="cuda")
    keep, pos = (torch.zeros(n_blocks + k, dtype=torch.int32, device="cuda") for k in (0, 1))
    pats = torch.zeros((n_blocks, 16), dtype=torch.uint8, device="cuda")
    packed = torch.zeros(n_blocks * block, dtype=torch.uint8, device="cuda")
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        ds.ds_image_compress(img.data_ptr(), nbytes, block, keep.data_ptr(), pos.data_ptr(), pats.data_ptr(), packed.data_ptr(),
                             torch.cuda.current_stream().cuda_stream)
    rng = np.random.default_rng(5)
    for k in range(4):
        host = np.zeros(nbytes, dtype=np.uint8)
        kept = sorted(int(b) for b in rng.choice(n_blocks - 1, 3, replace=False))
        for b in kept:
            host[b * block + int(rng.integers(16, block))] = 1
        img.copy_(torch.from_numpy(host))
        print(f"[case] replay {k} of {nbytes} bytes", flush=True)
        graph.replay()
        torch.cuda.synchronize()
        assert torch.nonzero(keep).flatten().tolist() == kept and int(keep.max()) == 1 and int(pos[-1]) == 3
        assert np.array_equal(packed[:3 * block].cpu().numpy(), np.concatenate([host[b * block:(b + 1) * block] for b in kept]))

"""ds_image_compress with blocks larger than the image, up to the largest power of two that 64 bits hold."""
import ctypes
import os
import subprocess

import numpy as np
import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_place_of_a_unit_in_blocks_of_every_size(tmp_path):
    so = str(tmp_path / "blocks_host.so")
    subprocess.run(["g++", "-O2", "-std=c++17", "-Wall", "-Werror", "-fPIC", "-shared", "-I",
                    os.path.join(ROOT, "paper_2601_16956_amd", "csrc"),
                    os.path.join(ROOT, "tests", "c_abi", "blocks_host.cpp"), "-o", so], check=True)
    lib = ctypes.CDLL(so)
    lib.blocks_host_place.restype = None
    lib.blocks_host_place.argtypes = [ctypes.c_uint64, ctypes.c_uint32, ctypes.c_void_p]
    out = (ctypes.c_uint64 * 2)()
    for log2 in range(10, 60):
        for unit in (0, 1, 256, 1024, (1 << 22) - 256, (1 << 22) - 1, 1 << 31, 1 << 32, (1 << 32) + 1024, (1 << 36) + 7):
            lib.blocks_host_place(unit, log2, out)
            assert tuple(out) == divmod(unit, 1 << log2), (unit, log2)


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

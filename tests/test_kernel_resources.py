"""What the compiler gave the kernels of the built library: registers, scratch and LDS decide how many wavefronts a SIMD
holds, and the launchers choose kernels by that number.  Read from the library's own code objects (the kernel metadata
that hipcc writes beside the code)."""
import os
import re
import struct
import subprocess

import msgpack
import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
LIB = os.path.join(ROOT, "paper_2601_16956_amd", "libdatastates_hip.so")


def _code_objects(blob):
    """The device ELF images in the clang offload bundles of a host library."""
    magic = b"__CLANG_OFFLOAD_BUNDLE__"
    at = blob.find(magic)
    while at >= 0:
        n, = struct.unpack_from("<Q", blob, at + len(magic))
        p = at + len(magic) + 8
        for _ in range(n):
            off, size, idlen = struct.unpack_from("<QQQ", blob, p)
            target = blob[p + 24:p + 24 + idlen].decode()
            p += 24 + idlen
            if "gfx950" in target and size:
                yield blob[at + off:at + off + size]
        at = blob.find(magic, p)


def _metadata(elf):
    """The kernels of the NT_AMDGPU_METADATA note."""
    phoff, = struct.unpack_from("<Q", elf, 32)
    phsize, phnum = struct.unpack_from("<HH", elf, 54)
    for k in range(phnum):
        kind, _, off, _, _, size = struct.unpack_from("<IIQQQQ", elf, phoff + k * phsize)
        if kind != 4:  # PT_NOTE
            continue
        at = off
        while at < off + size:
            namesz, descsz, ntype = struct.unpack_from("<III", elf, at)
            desc = at + 12 + -(-namesz // 4) * 4
            if ntype == 32 and elf[at + 12:at + 12 + 6] == b"AMDGPU":
                return msgpack.unpackb(elf[desc:desc + descsz], strict_map_key=False)["amdhsa.kernels"]
            at = desc + -(-descsz // 4) * 4
    return []


def _kernels():
    if not os.path.exists(LIB):
        pytest.skip("the library is not built")
    with open(LIB, "rb") as f:
        blob = f.read()
    found = [k for elf in _code_objects(blob) for k in _metadata(elf)]
    names = subprocess.run(["c++filt"], input="\n".join(k[".name"] for k in found), capture_output=True, text=True,
                           check=True).stdout.splitlines()
    out = {}
    for k, name in zip(found, names):
        m = re.search(r"(ds_\w+)(<[^>]*>)?\(", name)
        if m:
            args = [a.strip() for a in (m.group(2) or "<>")[1:-1].split(",")]
            out.setdefault(m.group(1), []).append((args, k))
    return out


def _waves(k):
    """Wavefronts per SIMD that registers and LDS leave room for (512 vector registers in steps of 8, 800 scalar ones in
    steps of 16, 160 KiB per CU)."""
    by_registers = min(512 // (-(-k[".vgpr_count"] // 8) * 8), 800 // (-(-k[".sgpr_count"] // 16) * 16))
    lds = k[".group_segment_fixed_size"]
    groups = (160 * 1024) // lds if lds else 99
    per_group = -(-k[".max_flat_workgroup_size"] // 256)  # wavefronts per SIMD of one work-group
    return min(8, by_registers, groups * per_group)


def test_no_kernel_uses_scratch():
    kernels = _kernels()
    assert len(kernels) >= 10
    for name, variants in kernels.items():
        for args, k in variants:
            assert k[".private_segment_fixed_size"] == 0 and not k.get(".vgpr_spill_count"), (name, args)


def test_the_scatter_has_the_wavefronts_it_is_launched_for():
    """ds_move_kernel<false, threads, units, loads nt, stores nt, buffer stores, WAVES, ...>."""
    scatters = [(a, k) for a, k in _kernels()["ds_move_kernel"] if a[0] == "false"]
    assert any(a[2] == "4" and a[6] == "6" for a, _ in scatters) and any(a[2] == "8" for a, _ in scatters)
    for args, k in scatters:
        assert _waves(k) >= int(args[6]), (args, k[".vgpr_count"])


def test_the_gather_of_mostly_general_chunks_has_six_wavefronts():
    for args, k in _kernels()["ds_move_kernel"]:
        if args[0] == "true" and args[2] in ("2", "4") and args[6] == "6":
            assert _waves(k) >= 6, (args, k[".vgpr_count"])


def test_one_unit_per_thread_runs_at_eight_wavefronts():
    """With one load per thread under way the default kernel is bound by HBM only if eight wavefronts per SIMD fit."""
    units = _kernels()["ds_unit_kernel"]
    assert len(units) >= 8
    for args, k in units:
        assert _waves(k) == 8, (args, k[".vgpr_count"])


def test_blocks_that_are_not_wide_have_seven_work_groups_per_CU():
    """Wide blocks need LDS that leaves room for five; launches without them do not pay for it.  (The gather beside whole
    chunks, ds_mixed_kernel<true, loads nt, 1, ...>, has registers for six.)"""
    for name in ("ds_perm_kernel", "ds_mixed_kernel"):
        for args, k in _kernels()[name]:
            six = name == "ds_mixed_kernel" and args[0] == "true" and args[2] == "1"
            assert _waves(k) >= (5 if args[-1] == "true" else 6 if six else 7), (name, args, k[".vgpr_count"])


def test_the_digest_that_profiles_name_covers_the_flags(monkeypatch):
    import paper_2601_16956_amd as ds
    from paper_2601_16956_amd import build
    before = ds.kernel_source_digest()
    assert ds.kernel_source_digest() == before
    monkeypatch.setattr(build, "HIPCC_FLAGS", [f for f in build.HIPCC_FLAGS if "preload" not in f])
    assert ds.kernel_source_digest() != before

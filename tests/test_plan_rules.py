"""Which route a plan's launches take when it holds views of several kinds: the rules of csrc/ds_plan.cpp, read from
plans made without a device."""
import ctypes
import os
import subprocess
from types import SimpleNamespace

import pytest

import paper_2601_16956_amd as ds
from workloads.configs import DTYPES

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
FACTS = ("n_chunks", "n_general", "n_perm_chunks", "n_perms", "n_blocks", "n_listed", "mostly_general",
         "in_pieces", "n_lanes", "n_dims", "mostly_several", "mostly_columns", "rests_at_once", "rests", "mostly_far")


@pytest.fixture(scope="module")
def facts(tmp_path_factory):
    so = str(tmp_path_factory.mktemp("facts") / "plan_facts.so")
    subprocess.run(["g++", "-O1", "-std=c++17", "-Wall", "-Werror", "-Wno-unknown-pragmas", "-fPIC", "-shared",
                    "-D__HIP_PLATFORM_AMD__", "-isystem", "/opt/rocm/include", "-I", os.path.join(ROOT, "include"), "-I",
                    os.path.join(ROOT, "paper_2601_16956_amd", "csrc"),
                    os.path.join(ROOT, "tests", "c_abi", "plan_facts.cpp"), "-o", so], check=True)
    fn = ctypes.CDLL(so).plan_facts
    fn.argtypes = [ctypes.c_void_p, ctypes.c_void_p]

    def of(views, align=64):
        shards, at = [], 4096
        for k, (dtype, shape, strides) in enumerate(views):
            shards.append(SimpleNamespace(dtype=dtype, shape=shape, strides=strides, byte_offset=at, tensor_id=k))
            at += -(-(sum((e - 1) * s for e, s in zip(shape, strides)) + 1) * DTYPES[dtype][1] // 256) * 256
        descs = ds.make_descs(shards, 1 << 40)
        ds.ds_layout_assign(descs, len(shards), align)
        plan = ds.ds_plan_create(descs, len(shards), align, ds.DS_PLAN_HOST_ONLY)
        out = (ctypes.c_uint64 * len(FACTS))()
        fn(plan, out)
        ds.ds_plan_destroy(plan)
        return SimpleNamespace(**dict(zip(FACTS, [int(x) for x in out])))
    return of


def _small(n, nbytes=1000):
    return [("u8", (nbytes,), (1,))] * n


def _transposed(n, dtype="bf16"):
    return (dtype, (n, n), (1, n))


def test_the_launch_of_the_other_chunks_is_shaped_by_what_it_carries(facts):
    """Tables of small tensors keep the launch of mostly general chunks beside views that another launch moves; and
    such views do not make one of a table of large tensors."""
    assert facts(_small(4000)).mostly_general
    f = facts(_small(4000) + [_transposed(256)])
    assert f.n_perms == 1 and f.n_perm_chunks >= 6 and f.mostly_general
    f = facts([("bf16", (1 << 22,), (1,)), _transposed(4096)])
    assert f.n_perms == 1 and f.n_general * 2 > f.n_chunks and not f.mostly_general
    f = facts([_transposed(512)], 16384)
    assert f.n_perm_chunks == f.n_chunks and not f.mostly_general


def test_the_other_chunks_are_listed_where_it_pays(facts):
    """No second copy of a large table for the sake of one view; a compact list in small plans and where one chunk in
    sixteen is left out."""
    f = facts([("bf16", (1 << 22,), (1,)), _transposed(128)])
    assert (f.n_chunks, f.n_perm_chunks, f.n_listed) == (514, 2, 512)
    rest = [("bf16", (1 << 26,), (1,))]                         # 8192 chunks
    f = facts(rest + [_transposed(128)])
    assert (f.n_chunks, f.n_perm_chunks, f.n_listed) == (8194, 2, 0)
    f = facts(rest + [("bf16", (4096, 1096), (1, 4096))])      # 548 of 8740: one in 15.9
    assert (f.n_chunks, f.n_perm_chunks, f.n_listed) == (8740, 548, 8192)
    f = facts(rest + [("bf16", (4096, 1088), (1, 4096))])      # 544 of 8736: one in 16.1
    assert (f.n_chunks, f.n_perm_chunks, f.n_listed) == (8736, 544, 0)


def test_a_few_KiB_of_short_runs_are_not_worth_a_launch(facts):
    """Views that could be moved in blocks stay with the general path where the other chunks hide them."""
    def blocks(rest, *views):
        f = facts(rest + list(views))
        assert (f.n_perms > 0) == (f.n_blocks > 0)
        return f.n_perms
    long, short = [("bf16", (1600 * 8192,), (1,))], [("bf16", (1500 * 8192,), (1,))]     # 1600 and 1500 chunks
    assert blocks(long, _transposed(24)) == 0 and blocks(short, _transposed(24)) == 1
    assert blocks(long, _transposed(64)) == 0 and blocks(long, _transposed(65)) == 1     # 8192 and 8450 bytes
    assert blocks(long, *[_transposed(32)] * 4) == 0 and blocks(long, *[_transposed(32)] * 5) == 5   # 2048 bytes each
    rows = ("u8", (60, 8), (13, 1))                                                      # 480 bytes, runs of 8
    assert blocks(short + [rows], _transposed(45)) == 0 and blocks(short + [rows], _transposed(46)) == 1
    assert blocks([], _transposed(24)) == 1


@pytest.mark.parametrize("kind,pieces", [
    ("tensor", {100: 1, 384: 1, 450: 0, 700: 0, 1000: 0, 1200: 0, 1536: 0, 1800: 0, 2200: 1, 2500: 0, 3200: 1, 9000: 1}),
    ("rows of 3000", {380: 1, 700: 0, 900: 0, 1100: 0, 1400: 0, 1800: 0, 2200: 1, 9000: 1}),
    ("rows of 256", {380: 1, 700: 0, 900: 0, 1100: 1, 1400: 1, 1800: 0, 2200: 1}),
    ("several dimensions", {380: 1, 450: 1, 700: 1, 1000: 1, 1700: 1, 2500: 1})])
def test_which_scatters_are_cut_into_pieces(facts, kind, pieces):
    """The table of sizes at which one work-group per 8 KiB measured faster than one per 16 KiB, by what is in the
    chunks.  450 to 768 and 1025 to 1536 chunks of one tensor or of long rows were cut, and 2 to 16 % slower for it."""
    for chunks, want in pieces.items():
        n = chunks * 16384
        view = {"tensor": ("u8", (n,), (1,)), "rows of 3000": ("u8", (n // 3000, 3000), (4000, 1)),
                "rows of 256": ("u8", (n // 256, 256), (512, 1)),
                "several dimensions": ("u8", (n // 1280, 5, 256), (2600, 512, 1))}[kind]
        assert facts([view]).in_pieces == want, chunks


def test_few_units_of_views_with_short_runs_are_moved_by_lanes(facts):
    """What is left of a view that is moved in blocks, and views with runs of one element of 1 or 2 bytes, of which
    there are at most 256 KiB; not where those keep the chip busy, nor runs that are few pieces of a unit."""
    assert facts([("u8", (1 << 24,), (1,)), _transposed(20, "u8")]).n_lanes == 1
    f = facts([("u8", (1 << 24,), (1,)), _transposed(91)])                 # 16 562 bytes, moved in blocks
    assert (f.n_perms, f.n_lanes) == (1, 1)
    assert facts([_transposed(16)] * 512).n_lanes == 512                  # 256 KiB
    assert facts([_transposed(16)] * 513).n_lanes == 0
    assert facts([("u8", (40, 9), (13, 1))] * 9).n_lanes == 0
    assert facts([("f32", (10, 9), (40, 2))] * 9).n_lanes == 0
    assert facts([("u8", (40, 16), (23, 1)), ("u8", (1000,), (1,))]).n_lanes == 0


def test_chunks_inside_views_of_several_dimensions_have_records(facts):
    """Whole chunks of a view with several outer dimensions and runs of at least 16 bytes; not those of shorter runs, nor
    the last one with the end of the payload, nor rows that merge into one dimension."""
    view = ("u8", (40, 10, 1000), (20000, 1500, 1))                       # 400 000 bytes = 24 chunks and a part
    assert facts([view]).n_dims == 24
    assert facts([("u8", (5000,), (1,)), view]).n_dims == 23
    assert facts([("u8", (40, 10, 1000), (15000, 1500, 1))]).n_dims == 0  # one outer dimension
    assert facts([("f32", (50, 40, 30, 3), (20000, 400, 10, 1))], 64).n_dims == 0
    assert facts([("f32", (50, 40, 30, 4), (20000, 400, 10, 1))], 64).n_dims == 58


def test_which_plans_of_small_tensors_and_views_keep_four_units_per_thread(facts):
    """Where most chunks hold several contiguous tensors, beside a view, in an image of more than 16 MiB."""
    rows, small = ("u8", (60, 100), (140, 1)), 4096
    assert facts(_small(4200, small) + [rows]).mostly_several
    assert not facts(_small(4000, small) + [rows]).mostly_several                       # 15.6 MiB
    assert not facts(_small(4200, small)).mostly_several                                # contiguous tensors only
    assert facts(_small(4200, small) + [_transposed(512)]).mostly_several               # beside blocks
    assert not facts(([("u8", (small,), (1,))] * 2 + [rows]) * 2500).mostly_several      # chunks that hold views
    assert not facts([("u8", (1 << 25,), (1,)), rows] + _small(100, small)).mostly_several


def test_the_scatter_of_narrow_columns_keeps_one_stripe_per_xcd(facts):
    """Blocks along a that are neither wide nor one piece of the image, when they are most of a launch's."""
    narrow, wide, flat, along_b = (("bf16", (507, 2847), (1, 509)), ("bf16", (512, 2847), (1, 512)),
                                   ("f32", (512, 513, 9), (513 * 9, 1, 513)), ("f32", (500000,), (2,)))
    assert facts([narrow]).mostly_columns
    for other in (wide, flat, along_b):
        assert not facts([other]).mostly_columns
    assert facts([narrow] * 3 + [wide, along_b]).mostly_columns
    assert not facts([narrow, wide, wide, flat]).mostly_columns
    assert not facts([("u8", (5000,), (1,))]).mostly_columns


def test_chunks_that_hold_little_besides_blocks(facts):
    """Ends of views and small tensors between them; not tensors that fill chunks, and where all chunks run at once not one of
    them."""
    view = ("bf16", (100, 102), (1, 100))
    for table in ([view] * 30, [view, ("u8", (1000,), (1,))] * 40, [view] * 1000):
        f = facts(table)
        assert f.n_perms and f.rests and f.rests_at_once
    f = facts([view] * 300 + [("u8", (65000,), (1,))])
    assert f.rests and not f.rests_at_once
    for table in ([view, ("u8", (16000,), (1,))] * 40, [view] * 30 + [("u8", (1 << 20,), (1,))], [view] * 3 + _small(400)):
        f = facts(table)
        assert f.n_perms and not f.rests and not f.rests_at_once
    f = facts(_small(400, 20))
    assert not f.n_perms and not f.rests


def test_the_gather_of_lines_that_blocks_far_on_share_keeps_one_stripe_per_xcd(facts):
    """Walks along b in short pieces, with batches between the pieces of a line: from eight blocks to a batch on."""
    far, near = ("u8", (20, 16384, 9), (18, 400, 2)), ("u8", (20, 3000, 8), (16, 400, 2))
    assert facts([far]).mostly_far and facts([far] * 3 + [("f32", (50000,), (2,))]).mostly_far
    for other in (near, ("f32", (500000,), (2,)), ("bf16", (900, 700), (1500, 2)), ("bf16", (512, 2847), (1, 512)),
                  ("f32", (300, 300, 9), (2700, 1, 300))):
        assert not facts([other]).mostly_far
    assert not facts([far] + [("f32", (2000000,), (2,))]).mostly_far

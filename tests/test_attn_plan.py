"""How the host cuts an attention call into splits (make_attn_plan), through a small program linked with the library: no
GPU needed."""
import itertools
import os
import subprocess

import pytest

from paper_2503_05096_amd import build

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.fixture(scope="module")
def plans(tmp_path_factory):
    exe = str(tmp_path_factory.mktemp("plan") / "plan_driver")
    lib = os.path.dirname(build.LIB_PATH)
    subprocess.check_call(["g++", "-O1", "-std=c++17", "-D__HIP_PLATFORM_AMD__", "-I", "/opt/rocm/include", "-I", build.INCLUDE,
                           os.path.join(ROOT, "tests", "native", "plan_driver.cpp"),
                           "-o", exe, build.LIB_PATH, f"-Wl,-rpath,{lib}"])

    def run(cases, *args):
        text = "\n".join(" ".join(map(str, c)) for c in cases)
        lines = subprocess.run([exe, *args], input=text, capture_output=True, text=True, check=True).stdout.splitlines()
        assert len(lines) == len(cases)
        return [tuple(map(int, l.split())) for l in lines]
    return run


F32, BF16 = 0, 2


def test_the_width_of_the_block_table_does_not_lengthen_splits(plans):
    """The length of a split follows from the number of (request, kv head) pairs; calls without a metadata kernel may take
    a shorter one, down to two blocks per wavefront, but never a longer one, however wide the table; trees always take it."""
    heads = [(32, 8, 128, BF16), (64, 8, 128, BF16), (16, 2, 128, BF16), (32, 32, 128, BF16), (32, 8, 64, BF16), (8, 8, 64, F32)]
    cases = [(B, pages, hq, hkv, d, k, dt) for B, pages, k, (hq, hkv, d, dt) in
             itertools.product((1, 2, 3, 4, 8, 20, 33, 70, 200, 256, 257, 1024), (1, 8, 32, 33, 64, 65, 94, 512, 1024, 2048, 4096), (0, 5, 11), heads)]
    direct_calls = 0
    for c, (split, direct, tree_split, tree_direct, block, chain_bytes, tree_bytes, asked, _) in zip(cases, plans(cases)):
        pairs = c[0] * c[3]
        by_pairs = 2048 if pairs >= 256 else 1024 if pairs >= 128 else 512 if pairs >= 32 else 256
        two_blocks = 2 * 4 * block
        assert (tree_split, tree_direct) == (by_pairs, 0), c
        assert split <= max(by_pairs, two_blocks) if direct else split == by_pairs, (c, split)
        assert asked == max(chain_bytes, tree_bytes), c          # one query serves chains and trees
        direct_calls += direct
    assert direct_calls > len(cases) // 8


def test_the_width_of_the_block_table_does_not_multiply_the_combine(plans):
    """Several wavefronts per (row, head) only while they fit the device beside each other."""
    cases = [(B, pages, 32, 8, 128, k, BF16) for B in (1, 4, 5, 64, 256) for pages in (32, 128, 129, 2048) for k in (0, 5)]
    for c, p in zip(cases, plans(cases)):
        possible, pairs = -(-c[1] * 16 // p[0]), c[0] * (c[5] + 1) * c[2]
        assert p[8] == (4 if possible > 8 and pairs <= 768 else 1), (c, p)


def test_short_contexts_of_many_rows_split_the_rows(plans):
    """More than 32 rows per kv head: a context of a few blocks leaves a ring per wavefront without work for most of them,
    so those calls take the kernel whose wavefronts split the rows; up to 32 rows and other types know no such choice."""
    def kernels(*c):
        return plans([c], "kernels")[0][2:]
    for B in (1, 16, 88, 250):
        for hq, hkv, k in ((64, 8, 4), (64, 8, 5), (28, 4, 7), (64, 8, 8), (16, 1, 7)):       # 40, 48, 56, 72, 128 rows
            assert kernels(B, 2, hq, hkv, 128, k, BF16) == (1, 1), (B, hq, hkv, k)
            assert kernels(B, 128, hq, hkv, 128, k, BF16) == (0, 0), (B, hq, hkv, k)
    assert kernels(88, 12, 64, 8, 128, 7, BF16) == (1, 1)       # 192 tokens: four tiles
    assert kernels(88, 12, 64, 8, 128, 5, BF16) == (0, 0)       # three
    assert kernels(48, 12, 64, 8, 128, 5, BF16) == (1, 1)       # three, two units side by side on a compute unit
    assert kernels(88, 2, 32, 8, 128, 7, BF16) == kernels(88, 2, 64, 8, 64, 7, BF16) == kernels(88, 2, 64, 8, 128, 7, F32) == (0, 0)


def test_two_tiles_of_128_channels_have_their_splits_combined_apart(plans):
    """Their states take the last workgroup of a request longer than a captured launch of the combine kernel."""
    for dtype in (1, BF16, F32):
        tokens = 128 if dtype == F32 else 256
        for splits in (2, 3, 4):
            pages = splits * tokens // 16
            got = plans([(1, pages, 32, 8, 128, 3, dtype), (1, pages, 32, 8, 128, 5, dtype)], "kernels")
            assert [g[:2] for g in got] == [(splits, 1), (splits, 0)], (dtype, splits)
        assert plans([(2, 24 if dtype == F32 else 96, 32, 8, 64, 5, dtype)], "kernels")[0][:2] == (3, 1)       # two tiles of 64


def test_which_splits_are_merged_in_the_main_kernel(plans):
    """The shapes that the GPU tests of the merge are about are merged, and the flag words end the workspace."""
    from tests.test_gpu_attn_merge import APART, MERGED
    for shapes, merged in ((MERGED, 1), (APART, 0)):
        cases = [(len(ctx), -(-max(ctx) // 16), hq, hkv, d, max(spec), {"f32": F32, "f16": 1, "bf16": BF16}[dtype])
                 for ctx, spec, hq, hkv, d, dtype, _ in shapes]
        for s, c, (per_req, is_merged, _, _), p in zip(shapes, cases, plans(cases, "kernels"), plans(cases)):
            assert (p[1], per_req, is_merged) == (1, s[6], merged), c
            assert not merged or p[7] == p[5] >= p[6], c


def test_query_rows_beyond_32_bits_of_offsets_split_the_rows(plans):
    """A unit's rows of Q span (query rows x heads x 256 bytes): from 4 GB on only the row split reaches them all."""
    for hkv, split in ((262143, 0), (262144, 1), (400000, 1)):
        assert plans([(1, 80, hkv, hkv, 128, 63, BF16)], "kernels")[0][2:] == (split, split), hkv

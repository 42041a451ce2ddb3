"""The host's launch rules (csrc/dispatch.hpp), asked by a small program: no GPU."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2607_00466_amd", "csrc")

UP, DOWN = 0, 1
BF16, MXFP4 = 0, 1
QWEN = (8, 128, 2048, 768)       # K, E, H, I
GPT_OSS = (4, 128, 2880, 2880)
FEW_LARGE = (2, 8, 4096, 14336)  # a few large experts

pytestmark = pytest.mark.skipif(shutil.which("g++") is None, reason="needs g++")


@pytest.fixture(scope="module")
def ask(tmp_path_factory):
    """ask(queries) -> one list of numbers a query."""
    exe = str(tmp_path_factory.mktemp("rules") / "dispatch_rules")
    r = subprocess.run(["g++", "-O1", "-std=c++17", "-Wall", "-Werror", "-I", os.path.join(ROOT, "include"), "-I", CSRC,
                        os.path.join(ROOT, "tests", "dispatch_rules.cpp"), "-o", exe],
                       capture_output=True, text=True, timeout=300)
    assert r.returncode == 0, r.stderr[-2000:]

    def run(queries):
        queries = [" ".join(map(str, q)) for q in queries]
        out = subprocess.run([exe], input="\n".join(queries) + "\n", capture_output=True, text=True, timeout=60)
        assert out.returncode == 0, out.stderr
        lines = out.stdout.splitlines()
        assert len(lines) == len(queries)
        return [[int(v) for v in l.split()] for l in lines]

    return run


def test_bucket_in_place_is_one_workgroup(ask):
    # several workgroups would read all the ids while each replaces a stretch of them
    for T, E, K, wgs in [(0, 37, 16, 1), (128, 37, 16, 1), (129, 37, 16, 2), (1024, 128, 8, 4), (4096, 128, 8, 16)]:
        (large, apart, lds), over = ask([("bucket", T, E, K, 0), ("bucket", T, E, K, 1)])
        assert apart == wgs
        assert over == [large, 1, lds]


def test_bucket_threads_an_expert(ask):
    # (few pairs in many tokens are counted faster by one thread an expert)
    for T, E, K, large in [(256, 16, 16, 0), (257, 128, 8, 0), (300, 128, 8, 0), (384, 128, 8, 0), (385, 128, 8, 1),
                           (700, 8, 2, 0), (1536, 8, 2, 0), (1537, 8, 2, 1), (768, 128, 4, 0), (769, 128, 4, 1),
                           (3072, 170, 1, 0), (4096, 128, 1, 1)]:
        assert ask([("bucket", T, E, K, 0)])[0][0] == large, (T, E, K)


def test_gate_tokens_go_by_xcd_while_the_gate_rows_fit_its_cache(ask):
    for T, E, H, tile, by_token in [(128, 128, 2048, 4, 0), (129, 128, 2048, 8, 0), (256, 128, 2048, 8, 0),
                                    (257, 128, 2048, 8, 1), (4096, 1, 32, 8, 1), (4096, 128, 2880, 8, 1),
                                    (257, 256, 4096, 8, 1), (257, 256, 4128, 8, 0), (4096, 256, 7168, 8, 0),
                                    (4096, 256, 16384, 8, 0), (4096, 64, 16384, 8, 1), (4096, 65, 16384, 8, 0)]:
        assert ask([("gate", T, E, H)]) == [[tile, by_token]], (T, E, H)


def _rows(mode, H, I):
    """(output rows, reduction) of a projection."""
    return (I, H) if mode == UP else (H, I)


def _slim(ask, mode, fmt, T, shape):
    K, E, H, I = shape
    return ask([("slim", mode, fmt, T, K, E, *_rows(mode, H, I))])[0][0]


@pytest.mark.parametrize("shape,fmt,up,down", [
    (QWEN, BF16, (1, 1, 1, 1, 0), (1, 0, 0, 0, 0)),
    (QWEN, MXFP4, (1, 1, 1, 1, 0), (1, 1, 1, 1, 0)),
    (GPT_OSS, BF16, (1, 1, 1, 1, 0), (1, 1, 1, 1, 0)),
    (GPT_OSS, MXFP4, (1, 1, 1, 1, 0), (1, 1, 1, 1, 0)),
    ((4, 60, 2048, 1408), BF16, (1, 1, 1, 1, 0), (1, 1, 1, 0, 0)),
    (FEW_LARGE, BF16, (0, 0, 0, 0, 0), (1, 1, 0, 0, 0)),
    (FEW_LARGE, MXFP4, (1, 1, 0, 0, 0), (1, 1, 0, 0, 0)),
    ((6, 64, 4096, 1024), BF16, (1, 1, 1, 1, 0), (1, 0, 0, 0, 0)),
    ((8, 64, 2048, 3072), BF16, (1, 1, 0, 0, 0), (1, 1, 1, 0, 0)),
    ((8, 64, 2048, 3072), MXFP4, (1, 1, 1, 1, 0), (1, 1, 1, 1, 0)),
    ((1, 1, 32, 32), BF16, (1, 1, 1, 1, 0), (1, 1, 1, 1, 0)),
])
def test_one_wave_kernel(ask, shape, fmt, up, down):
    # 1 .. 5 tokens
    assert tuple(_slim(ask, UP, fmt, T, shape) for T in range(1, 6)) == up
    assert tuple(_slim(ask, DOWN, fmt, T, shape) for T in range(1, 6)) == down


def _wide(ask, mode, fmt, T, shape):
    K, E, H, I = shape
    return ask([("wide", mode, fmt, T, K, E, *_rows(mode, H, I))])[0]


def test_wide_kernel_has_a_workgroup_for_each_item_a_round_holds(ask):
    # even buckets of every size, cut to any group the device may choose: there is a
    # workgroup for each of an XCD's items up to the 64 workgroups it holds at once
    for shape, T in [((3, 37, 1056, 544), 1000), (QWEN, 300), (QWEN, 4096), (GPT_OSS, 256), (FEW_LARGE, 200),
                     ((2, 16, 256, 128), 4096), ((1, 1, 32, 32), 65)]:
        K, E, H, I = shape
        for mode in (UP, DOWN):
            _, tiles, slots = _wide(ask, mode, MXFP4, T, shape)
            for U in range(K, E + 1):
                bucket = -(-T * K // U)
                for cap in (128, 64, 32):
                    items = -(-tiles * U * -(-bucket // cap) // 8)
                    assert slots >= min(items, 64), (shape, T, mode, U, cap, items, slots)


@pytest.mark.parametrize("shape,fmt,up,down", [
    # the first batch of each projection the wide kernel takes
    (QWEN, BF16, 320, 192), (QWEN, MXFP4, 65, 128),
    (GPT_OSS, BF16, 640, 384), (GPT_OSS, MXFP4, 128, 256),
    ((4, 60, 2048, 1408), BF16, 300, 180), ((4, 60, 2048, 1408), MXFP4, 65, 480),
    ((3, 37, 1056, 544), BF16, 1067, 1067), ((8, 256, 2048, 256), BF16, 640, 1024),
    ((2, 16, 256, 128), BF16, None, None), ((2, 16, 256, 128), MXFP4, None, None),
])
def test_wide_kernel(ask, shape, fmt, up, down):
    for mode, first in ((UP, up), (DOWN, down)):
        took = [_wide(ask, mode, fmt, T, shape)[0] for T in (1, 64)]
        assert took == [0, 0]
        if first is None:
            assert _wide(ask, mode, fmt, 4096, shape)[0] == 0
        else:
            assert [_wide(ask, mode, fmt, T, shape)[0] for T in (first - 1, first, 2 * first)] == [0, 1, 1], mode


def _groups(ask, fmt, tiles, buckets):
    return ask([("groups", fmt, tiles, *buckets)])[0]


def test_wide_groups(ask):
    # even buckets that give a CU an item or two stay whole
    assert _groups(ask, BF16, 6, [75] * 32 + [60] * 20) == [128, 1, 52]
    assert _groups(ask, MXFP4, 6, [32] * 64) == [128, 1, 64]
    # fewer items than CUs: cut, bf16 to 32 only below 160 items
    assert _groups(ask, BF16, 6, [100] * 32) == [64, 0, 64]
    assert _groups(ask, BF16, 8, [60] * 16) == [32, 0, 32]
    assert _groups(ask, BF16, 8, [60] * 20) == [64, 1, 20]
    # a few items more than CUs: MXFP4 is cut
    assert _groups(ask, MXFP4, 12, [60] * 8 + [68] * 8)[0] == 32
    assert _groups(ask, MXFP4, 8, [40] * 32) == [128, 1, 32]
    # one bucket much longer than the others: MXFP4 is cut to it, and bands are dealt
    skewed = [80, 40, 24] + [6] * 56
    assert _groups(ask, MXFP4, 8, skewed)[:2] == [32, 0]
    assert _groups(ask, BF16, 8, skewed)[:2] == [128, 1]
    # but not where the work of many rounds hides it
    assert _groups(ask, MXFP4, 128, skewed)[0] == 128
    # experts that don't divide among the XCDs are not dealt whole
    assert _groups(ask, MXFP4, 112, [40] * 8)[:2] == [128, 1]
    assert _groups(ask, MXFP4, 112, [40] * 9)[:2] == [128, 0]
    # an empty union, and the largest one
    assert _groups(ask, MXFP4, 1, []) == [32, 1, 0]
    assert _groups(ask, MXFP4, 128, [256] * 256)[0] == 128


def _cases(test):
    """The parameter sets of a parametrised test."""
    return next(m.args[1] for m in test.pytestmark if m.name == "parametrize")


def test_the_one_wave_tests_run_that_kernel(ask):
    from tests import test_gpu_ffn_slim as S
    for fmt, H, I in _cases(S.test_bucket_sizes_and_reductions):
        shape, f = (5, 40, H, I), BF16 if fmt == "bf16" else MXFP4
        assert [_slim(ask, UP, f, T, shape) for T in (1, 2, 3, 4, 8)] == [1, 1, 1, 1, 0], (fmt, H, I)
        assert [_slim(ask, DOWN, f, T, shape) for T in (1, 2, 3, 8)] == [1, 1, 1, 0], (fmt, H, I)


def test_the_wide_tests_run_that_kernel(ask):
    from tests import test_gpu_ffn_wide as W
    for fmt, H, I in _cases(W.test_bucket_sizes_around_every_tile) + _cases(W.test_few_active_experts_take_smaller_groups):
        f = BF16 if fmt == "bf16" else MXFP4
        for mode in (UP, DOWN):
            assert _wide(ask, mode, f, 2080, (4, 248, H, I))[0] == 1, (fmt, H, I, mode)
            assert _wide(ask, mode, f, 64, (4, 248, H, I))[0] == 0


def test_the_choice_tests_run_the_kernels_they_name(ask):
    from tests import test_gpu_kernel_choice as C
    for fmt, E, K, H, I, T in C.SLIM + C.WIDE + C.MIXED:
        f = BF16 if fmt == "bf16" else MXFP4
        slim = [_slim(ask, mode, f, T, (K, E, H, I)) for mode in (UP, DOWN)]
        wide = [_wide(ask, mode, f, T, (K, E, H, I))[0] for mode in (UP, DOWN)]
        assert slim == ([1, 1] if T < 5 else [0, 0]), (fmt, T)
        assert wide == ([0, 0] if T < 5 else [0, 1] if T == 256 else [1, 1]), (fmt, T)
    for fmt, E, K, H, I, T in C.WIDE:
        assert ask([("bucket", T, E, K, 0), ("gate", T, E, H)])[0][:2] == [1, 5]
        assert ask([("gate", T, E, H)])[0] == [8, 1]

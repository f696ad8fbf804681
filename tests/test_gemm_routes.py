"""Which kernel a GEMM launch runs on and how it is dealt out: the host-side
rules of kernels.h, called in the built library (no GPU)."""
import ctypes

import pytest

from paper_2402_15758_amd import binding as B


class StreamPlan(ctypes.Structure):
    _fields_ = [(n, ctypes.c_int) for n in ("row_tiles", "row_blocks", "runs", "run", "long_runs", "mapped")]


def _fn(name, restype):
    f = B.lib()[name]
    f.restype = restype
    return f


def stream_plan(M, nbc, splits):
    mcap = next((c for c in (16, 32, 64) if M <= c), -(-M // 128) * 128)
    return _fn("_Z16gemm_stream_planiiii", StreamPlan)(M, nbc, splits, mcap // 16)


# bf16 launches of two 64-row blocks: 65 to 128 rows of matrices dealt in runs
# of 7 or 8 column blocks (LM head, 13B and 33B gate/up)
@pytest.mark.parametrize("M", [65, 96, 128])
@pytest.mark.parametrize("cols", [27648, 32000, 35840])
def test_two_row_blocks_of_a_run_stay_on_one_die(M, cols):
    p = stream_plan(M, cols // 16, 1)
    assert (p.row_tiles, p.row_blocks) == (4, 2) and p.run in (7, 8) and p.mapped
    # the mapped kernel exists for bf16: <T, row tiles, run, mapped>
    with open(B.LIB_PATH, "rb") as f:
        assert b"gemm_kernelItLi4ELi%dELb1E" % p.run in f.read()


@pytest.mark.parametrize("M", [1, 16, 17, 64, 65, 128, 129, 300, 2048])
def test_a_plan_covers_every_row_and_column_block_once(M):
    for nbc in (1, 4, 100, 255, 256, 768, 1376, 2000, 2560):
        for splits in (1, 2, 8):
            p = stream_plan(M, nbc, splits)
            assert p.long_runs * p.run + (p.runs - p.long_runs) * (p.run - 1) == nbc
            assert 1 <= p.long_runs <= p.runs and 1 <= p.run <= (6 if p.row_tiles == 8 else 8)
            assert 16 * p.row_tiles * (p.row_blocks - 1) < M <= 16 * p.row_tiles * p.row_blocks


F32, SILU, SWIGLU, QKV, PARTIAL, ZIN = 0, 2, 3, 4, 5, 6


def splits_of(bf16, cols, K):
    return _fn("_Z16gemm_pick_splitsiii", ctypes.c_int)(cols, K, bf16)


# Launches of a few rows whose slices meet in one workgroup per column block,
# and those that run their slices side by side on more CUs (measured faster).
@pytest.mark.parametrize("bf16,M,cols,K,one", [
    (1, 1, 64, 2048, True), (1, 1, 64, 4096, False), (1, 1, 64, 32768, False), (1, 4, 1024, 8192, False),
    (1, 1, 2048, 4096, False), (1, 16, 1024, 2048, True), (1, 1, 2560, 3072, True), (1, 1, 4096, 16384, True),
    (1, 1, 4096, 11008, True), (1, 16, 7680, 1280, True), (1, 16, 7680, 1536, False), (1, 1, 5120, 15360, False),
    (0, 5, 1024, 1024, True), (0, 1, 64, 2048, False), (0, 1, 1024, 4096, False), (0, 8, 256, 768, True),
])
def test_few_row_launches_where_one_workgroup_a_block_is_faster(bf16, M, cols, K, one):
    takes = _fn("_Z15gemm_rows_takesiiiiii", ctypes.c_bool)
    for kind in (F32, SILU, ZIN):
        assert takes(bf16, M, cols // 16, K, splits_of(bf16, cols, K), kind) == one
    assert not takes(bf16, M, cols // 16, K, splits_of(bf16, cols, K), PARTIAL)

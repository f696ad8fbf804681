"""Which kernel a GEMM launch runs on and how it is dealt out, and how a top-s
selection is: the host-side rules of kernels.h, called in the built library (no
GPU)."""
import ctypes

import pytest

from gemm_launch import (EPI_F32, EPI_PARTIAL, EPI_QKV, EPI_SILU, EPI_SWIGLU, EPI_ZIN, GemmEpi, GemmShape, launch,
                         fn, mcap, partial_rows, partials, rows_takes, splits_of, stream_plan, wide_takes)
from paper_2402_15758_amd import binding as B


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


# Launches of a few rows whose slices meet in one workgroup per column block,
# and those that run their slices side by side on more CUs (measured faster).
@pytest.mark.parametrize("bf16,M,cols,K,one", [
    (1, 1, 64, 2048, True), (1, 1, 64, 4096, False), (1, 1, 64, 32768, False), (1, 4, 1024, 8192, False),
    (1, 1, 2048, 4096, False), (1, 16, 1024, 2048, True), (1, 1, 2560, 3072, True), (1, 1, 4096, 16384, True),
    (1, 1, 4096, 11008, True), (1, 16, 7680, 1280, True), (1, 16, 7680, 1536, False), (1, 1, 5120, 15360, False),
    (0, 5, 1024, 1024, True), (0, 1, 64, 2048, False), (0, 1, 1024, 4096, False), (0, 8, 256, 768, True),
])
def test_few_row_launches_where_one_workgroup_a_block_is_faster(bf16, M, cols, K, one):
    for kind in (EPI_F32, EPI_SILU, EPI_ZIN):
        assert rows_takes(bf16, M, cols, K, kind) == one
    assert not rows_takes(bf16, M, cols, K, EPI_PARTIAL)


# Launches of more than 128 bf16 rows: the faster of the two kernels (both
# timed), 7B and 13B projections and small or narrow matrices.
@pytest.mark.parametrize("M,cols,K,tiled", [
    (256, 768, 256, False), (512, 2048, 256, False), (2048, 256, 256, False), (256, 64, 16384, False),
    (256, 4096, 256, False), (256, 8192, 4096, False), (129, 8192, 8192, False), (256, 5120, 13824, False),
    (256, 4096, 4096, True), (256, 4096, 11008, True), (256, 22016, 4096, True), (129, 32000, 4096, True),
    (512, 8192, 4096, True), (512, 12288, 4096, True), (2048, 1024, 4096, True), (2048, 4096, 512, True),
    (128, 32000, 4096, False),
])
def test_wide_launches_run_on_the_faster_kernel(M, cols, K, tiled):
    assert wide_takes(1, M, cols, K) == tiled
    assert not wide_takes(0, M, cols, K)


# An epilogue that no kernel of a launch's route applies is refused before any
# launch (there is no GPU here): the few-row epilogue on more rows or an unsplit
# matrix, and values that name none.
@pytest.mark.parametrize("kind", [EPI_ZIN, 1, 7, -1])
@pytest.mark.parametrize("bf16,M,N,K", [(1, 17, 4096, 11008), (1, 256, 4096, 11008), (1, 256, 22016, 4096),
                                        (0, 300, 256, 768), (1, 1, 16384, 4096)])
def test_an_epilogue_without_a_kernel_is_refused(kind, bf16, M, N, K):
    s = GemmShape(M=M, N=N, K=K, x_mtiles=mcap(M) // 16, splits=splits_of(bf16, N, K))
    assert launch(bf16, s, GemmEpi(kind=kind), None) is False


# The workspace of split launches holds every launch of up to max_M rows (the
# input buffer's tiles may exceed a launch's own), and no more than one of them uses
@pytest.mark.parametrize("bf16,cols,K", [(1, 4096, 4096), (1, 4096, 11008), (1, 256, 768), (1, 768, 4096),
                                         (1, 6144, 1024), (1, 5120, 13824), (1, 12288, 4096), (0, 1024, 3072)])
@pytest.mark.parametrize("kind", [EPI_PARTIAL, EPI_F32, EPI_SILU, EPI_SWIGLU, EPI_QKV])
def test_the_split_workspace_covers_every_launch(bf16, cols, K, kind):
    for max_M in (1, 16, 17, 63, 128, 300, 2048):
        most = 0
        for M in range(1, max_M + 1):
            rows = {M * partials(bf16, M, cols, K, kind, t // 16) for t in (mcap(M), mcap(max_M))}
            assert len(rows) == 1
            most = max(most, rows.pop())
        assert partial_rows(bf16, max_M, cols, K, kind) == most


def test_the_split_workspace_of_a_chunk_is_what_its_launches_leave():
    # 7B: a 2048-row chunk's O and down projections add their slices themselves
    # from 1281 rows on, the trigram products too
    assert partial_rows(1, 2048, 4096, 4096, EPI_PARTIAL) <= 4 * 1280
    assert partial_rows(1, 2048, 4096, 12288, EPI_SILU) <= 4 * 1280
    assert partial_rows(1, 2048, 12288, 4096, EPI_QKV) == 0


def test_top_s_rows_are_shared_where_one_workgroup_is_slower():
    splits = fn("_Z11topk_splitsi", ctypes.c_int)
    assert [splits(V) for V in (64, 1024, 1536, 1600, 2048, 4096, 32000)] == [1, 1, 1, 32, 32, 32, 32]

"""How the vocabulary pass launches a batch (host only; 256 compute units without a GPU, as on one)."""
import ctypes as C

import pytest
import torch

import paper_2505_18573_amd as e3

CUS = 256
TILE = 4096
ROWS = [1, 3, 64, 96, 127, 128, 129, 160, 192, 193, 255, 256, 257, 300, 384, 385, 511, 512, 513, 640, 641, 768, 832, 833, 1000, 1024, 1025,
        1280, 1281, 1536, 2048, 2049, 2500, 2560, 2561, 4096, 4097, 5120, 5121, 6144, 6145, 10_000, 32_768]
WIDTHS = [1, 256, 264, 448, 449, 768, 769, 1000, 1024, 1025, 4000, 4096, 4097, 8000, 16_384, 16_385, 20_480, 20_484, 22_528, 22_529,
          24_000, 24_576, 24_577, 27_000, 28_672, 30_000, 32_000, 32_768, 32_769, 40_960, 48_000, 61_440,
          61_441, 70_005, 128_000, 151_936, 262_144, 500_000]


def streamed(rows, V, sample, dtype):
    """Rows of at most eight super-tiles that have no workgroup each (CUS: a row to a compute unit)."""
    tiles, last = -(-V // TILE), V % TILE
    few = 0 < last <= TILE // 2
    if dtype is torch.bfloat16:
        short = not sample and V <= (1024 if rows <= 20 * CUS else 448)
        return short and rows > 10 * CUS or tiles == 8 and rows > 16 * CUS and (sample or few)
    if tiles <= 4:
        return 256 < V <= (1024 if sample else 768) and rows > 10 * CUS
    if tiles <= 6:
        return rows > 2 * CUS and (not sample or rows <= 4 * CUS and last <= TILE // 2 or tiles == 6 and few and rows > 24 * CUS)
    if rows <= CUS:
        return False
    if 4 * rows <= 13 * CUS:
        return last <= TILE // 2 or 2 * rows <= 3 * CUS
    return few and (rows > 16 * CUS and not (tiles == 7 and sample) or tiles == 7 and not sample and 5 * CUS < rows <= 8 * CUS)


@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float32])
@pytest.mark.parametrize("sample", [True, False])
def test_workgroups_cover_the_rows_and_the_cut_follows_their_number(sample, dtype):
    for V in WIDTHS:
        for rows in ROWS:
            cut, waves, per_group, workgroups = e3.e3_launch_plan(rows, V, sample, dtype)
            assert per_group >= 1
            assert workgroups == -(-rows // per_group), (rows, V)
            tiles = -(-V // TILE)
            if not streamed(rows, V, sample, dtype) if tiles <= 8 else dtype is torch.bfloat16 and tiles <= 16 and rows <= CUS:
                # one, two or four waves to a super-tile; their shares, one or two each, have sixteen places
                assert per_group == 1 and waves in (tiles, 2 * tiles, 4 * tiles) and waves <= 16, (rows, V, waves)
            else:
                assert waves in (4, 8), (rows, V, waves)
                # a workgroup never holds more rows than give each wave two items
                assert per_group == 1 or (per_group - 1) * tiles < 2 * waves, (rows, V)
            # rows are cut where whole rows leave half of the compute units without a workgroup
            assert cut == (V > 8 * TILE and rows <= 1024 and 2 * workgroups <= CUS), (rows, V)
            # ... which a batch with a row for more than half of them never does
            assert not (cut and rows > CUS // 2), (rows, V)


@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float32])
@pytest.mark.parametrize("sample", [True, False])
@pytest.mark.parametrize("V", [1, 1000, 4096, 8192, 16_384, 20_000, 32_768])
def test_no_launch_has_more_threads_than_a_grid_may(V, sample, dtype):
    # fewer than 2^32 in all: batches that a workgroup to each row would take beyond go to workgroups of several rows
    tiles = -(-V // TILE)
    for rows in sorted({r + d for e in range(20, 28) for r in (1 << e, (1 << e) // tiles, 3 << (e - 2)) for d in (-1, 0, 1)}):
        _, waves, per_group, workgroups = e3.e3_launch_plan(rows, V, sample, dtype)
        assert workgroups == -(-rows // per_group)
        several = 8 // tiles if tiles <= 8 else 1                      # rows of a streaming workgroup of four waves
        if -(-rows // several) * 256 < 1 << 32:                        # what that kernel can take
            assert workgroups * waves * 64 < 1 << 32, (rows, V, waves, per_group)


def test_the_plan_without_a_type_is_that_of_bf16():
    for rows, V in ((100, 1000), (200, 40_000), (600, 20_000), (4096, 151_936)):
        for sample in (0, 1):
            out = [C.c_int32(), C.c_int32(), C.c_int32(), C.c_int64()]
            assert e3.lib().e3_launch_plan(rows, V, sample, *(C.byref(x) for x in out)) == 0
            assert tuple(x.value for x in out) == e3.e3_launch_plan(rows, V, bool(sample), torch.bfloat16)
            assert e3.lib().e3_launch_plan_of(rows, V, 2, sample, *(C.byref(x) for x in out)) == -3       # E3_ERR_DTYPE


@pytest.mark.parametrize("rows,V,groups", [(512, 4000, 64), (1024, 4000, 128), (512, 1000, 64), (64, 1000, 8)])
def test_small_rows_have_a_workgroup_for_every_group_of_eight(rows, V, groups):
    # advantages ride along with the training-side pass where it has a workgroup for each group
    assert e3.e3_launch_plan(rows, V, False)[3] >= groups


def test_refused_shapes():
    for rows, V in ((0, 1000), (-1, 1000), (10, 0), (10, 1 << 30)):
        with pytest.raises(e3.E3Error) as ei:
            e3.e3_launch_plan(rows, V)
        assert ei.value.status == -2

"""Calls whose time must not leave that of a related call behind: inputs of the same size on which a
kernel takes another route, or another split of the same work.  Only ratios of times taken on the same GPU in the
same test are compared; each bound lies about half way (as a ratio) between what the sound route and the
slow one it guards against measured.
"""
import pytest
import torch

import paper_2505_18573_amd as e3

DEV = "cuda:0"
pytestmark = pytest.mark.gpu


def us(call, n=8):
    """Microseconds per call: the best of five replays of a graph of n calls."""
    stream = torch.cuda.Stream()
    stream.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(stream):
        call()
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=stream):
        for _ in range(n):
            call()
    best = float("inf")
    for _ in range(6):
        start, end = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        start.record()
        graph.replay()
        end.record()
        end.synchronize()
        best = min(best, start.elapsed_time(end) * 1000.0 / n)
    return best


def _objective(lens, cuts):
    soff = torch.zeros(len(lens) + 1, dtype=torch.int64)
    soff[1:] = torch.cumsum(lens, 0)
    T = int(soff[-1])
    g = torch.Generator(device=DEV).manual_seed(T)
    old = -torch.rand(T, generator=g, device=DEV)
    new = old + 0.1 * torch.randn(T, generator=g, device=DEV)
    adv = torch.randn(len(lens), generator=g, device=DEV)
    soff, goff = soff.to(torch.int32).to(DEV), cuts.to(torch.int32).to(DEV)
    return lambda: e3.e3_grpo_objective(new, old, soff, adv, goff, 0.2)


def test_many_questions_cost_their_rounds_only():
    # 20,000 rollouts folded as 20,000 questions or as 1000: 18.8 and 13.7 us with one lane per question
    # (20 rounds and one); 123 and 17.2 us when eight lanes shared every question (157 rounds and eight)
    lens = torch.full((20_000,), 10)
    many = us(_objective(lens, torch.arange(0, 20_001)))
    some = us(_objective(lens, torch.arange(0, 20_001, 20)))
    print(f"objective of 20,000 rollouts: {many:.1f} us as 20,000 questions, {some:.1f} us as 1000")
    assert many < 3.5 * some


def _selection(lg, k=50, p=0.95):
    rows, V = lg.shape
    need = e3.e3_restricted_workspace_bytes(e3.E3_BF16 if lg.dtype == torch.bfloat16 else e3.E3_F32, rows, V, k)
    workspace = torch.empty(need, dtype=torch.uint8, device=DEV) if need else False
    tok = torch.empty(rows, dtype=torch.int32, device=DEV)
    logp = torch.empty(rows, dtype=torch.float32, device=DEV)
    kept = torch.empty(rows, dtype=torch.int32, device=DEV)
    return lambda: e3.e3_sample_restricted(lg, None, 1.0, k, p, 7, 0, tok, logp, kept, workspace)


@pytest.mark.parametrize("rows", [8, 300])
def test_fp32_rows_of_nearly_equal_values_keep_their_bound(rows):
    # values that agree in their upper 16 bits: 22 us as for ordinary rows; 124 us when the selection's bound
    # was held in 16 bits, so that half the row reached it
    g = torch.Generator(device=DEV).manual_seed(3)
    x = torch.randn((rows, 151_936), generator=g, device=DEV)
    ordinary, narrow = us(_selection(3.0 * x)), us(_selection(100.0 + 0.3 * x))
    print(f"{rows} fp32 rows, top-k 50: ordinary {ordinary:.1f} us, nearly equal values {narrow:.1f} us")
    assert narrow < 2.0 * ordinary


@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float32])
def test_rows_that_are_mostly_a_plateau_are_listed_in_one_pass(dtype):
    # 0.13 % of the columns stand out of zeros (bf16 / fp32: ordinary rows 18 / 22 us, these 21 / 30 us;
    # 158 / 202 us when every vector of the plateau was listed first)
    g = torch.Generator(device=DEV).manual_seed(5)
    x = torch.randn((100, 128_000), generator=g, device=DEV) * 3
    ordinary, plateau = us(_selection(x.to(dtype))), us(_selection(torch.relu(x - 9.0).to(dtype)))
    print(f"100 rows {dtype}, top-k 50: ordinary {ordinary:.1f} us, mostly zeros {plateau:.1f} us")
    assert plateau < 3.0 * ordinary


def _nucleus(lg, k=0, p=0.9):
    return _selection(lg.to(torch.bfloat16), k, p)


@pytest.mark.parametrize("rows", [8, 300])
@pytest.mark.parametrize("kind", ["large_late", "all_below", "tiny"])
def test_rows_outside_the_first_window_are_counted_once_more(kind, rows):
    # 1.5 to 2 times an ordinary row (8 rows 25 us: 41, 37 and 48 us; 145, 305 and 154 us when such rows took
    # the wide form)
    g = torch.Generator(device=DEV).manual_seed(9)
    x = torch.randn((rows, 151_936), generator=g, device=DEV) * 3
    ordinary = us(_nucleus(x))
    if kind == "large_late":
        x[:, 75_000:] *= 3000.0
    elif kind == "all_below":
        x = x * 10 - 2000.0
    else:
        x *= 3e-5
    outside = us(_nucleus(x))
    print(f"{rows} rows, top-p 0.9: ordinary {ordinary:.1f} us, {kind} {outside:.1f} us")
    assert outside < 3.0 * ordinary


@pytest.mark.parametrize("rows", [8, 300])
def test_a_count_cut_among_masked_columns_costs_no_sweeps(rows):
    # 100 columns allowed, the others at -1e4: top-k 1000 takes as long as no count cut (8 rows 75 us each; 630
    # and 149 us when the cut sent the row to the wide form)
    g = torch.Generator(device=DEV).manual_seed(9)
    x = torch.full((rows, 151_936), -1e4, device=DEV)
    x[:, ::1520] = torch.randn((rows, 100), generator=g, device=DEV) * 3
    without, with_cut = us(_nucleus(x)), us(_nucleus(x, 1000, 1.0))
    print(f"{rows} masked rows: top-p 0.9 {without:.1f} us, top-k 1000 {with_cut:.1f} us")
    assert with_cut < 2.0 * without


@pytest.mark.parametrize("kind", ["at_most_zero", "tiny_positive", "few_negative"])
def test_few_rows_without_large_positive_values_cost_no_sweeps(kind):
    # 8 rows cut into slices, an ordinary one 16 us: 22, 26 and 24 us (the last counted once more); 268, 154 and 150 us when the
    # slices' window was chosen by the largest value of a sample alone, so that the negative columns lay below it
    g = torch.Generator(device=DEV).manual_seed(9)
    x = torch.randn((8, 151_936), generator=g, device=DEV) * 3
    ordinary = us(_nucleus(x))
    if kind == "at_most_zero":
        x = x.clamp(max=0)
    elif kind == "tiny_positive":
        x = torch.where(x < 0, x, x * 1e-4)
    else:
        x *= 3e-4
        x[:, 3::5000] = -30.0
    other = us(_nucleus(x))
    print(f"8 rows, top-p 0.9: ordinary {ordinary:.1f} us, {kind} {other:.1f} us")
    assert other < 3.0 * ordinary


@pytest.mark.parametrize("rows,V,most", [(8, 32_000, 4.9), (100, 70_000, 5.4)])
def test_rows_that_are_swept_over_all_patterns(rows, V, most):
    # 500 columns of 2^-24 to 2^-60: 42 and 60 us (ordinary rows 11.5 and 15.7); 76 and 124 when a sweep waited for its own
    # requests and every level's counter was looked up twice by half as many threads as before (70 and 108)
    g = torch.Generator(device=DEV).manual_seed(9)
    x = torch.randn((rows, V), generator=g, device=DEV) * 3
    ordinary = us(_nucleus(x))
    for row in x:
        cols = torch.randperm(V, generator=g, device=DEV)[:500]
        row[cols] = 2.0 ** -torch.randint(24, 60, (500,), generator=g, device=DEV).float()
    small = us(_nucleus(x))
    print(f"{rows} x {V}, top-p 0.9: ordinary {ordinary:.1f} us, 500 small columns {small:.1f} us")
    assert small < most * ordinary


def test_levels_without_weight_are_not_searched_among_equals():
    # logits 300 times as large: most kept levels weigh nothing, which many waves' race then ends with.  10.7 us as for ordinary rows; 12.3
    # when the holder of a zero was looked for among all 64 lanes
    g = torch.Generator(device=DEV).manual_seed(9)
    x = torch.randn((100, 5_000), generator=g, device=DEV) * 3
    ordinary, spread = us(_nucleus(x, 1000, 1.0)), us(_nucleus(300.0 * x, 1000, 1.0))
    print(f"100 x 5000, top-k 1000: ordinary {ordinary:.1f} us, 300 times as large {spread:.1f} us")
    assert spread < 1.065 * ordinary


def test_selection_of_negative_rows_looks_at_a_set_once():
    # 12.7 us ordinary and 14.3 us at -30 + 0.3 N(0, 1); 12.4 and 15.6 when every set's maxima were taken as integers first
    g = torch.Generator(device=DEV).manual_seed(9)
    x = torch.randn((300, 40_000), generator=g, device=DEV)
    ordinary, negative = us(_selection((3.0 * x).to(torch.bfloat16), 1, 1.0)), us(_selection((0.3 * x - 30.0).to(torch.bfloat16), 1, 1.0))
    print(f"300 x 40,000 bf16, top-k 1: ordinary {ordinary:.1f} us, negative throughout {negative:.1f} us")
    assert negative < 1.185 * ordinary

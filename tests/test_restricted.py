"""Parity of e3_sample_restricted (top-k / top-p sampling) with the CPU oracle.

Bars: kept counts identical except on rows the oracle flags near_cut (top-p target
within 1e-9 relative of a cumulative level mass); tokens identical except on near_cut
or near_tie rows (two best race scores within 1e-5 relative); logp within 1e-4
relative (it is evaluated in fp64 and stored as fp32).
"""
import numpy as np
import pytest
import torch
from scipy import stats

import paper_2505_18573_amd as e3
from oracle import e3_oracle as o
from paper_2505_18573_amd import workloads as wl

DEV = "cuda:0"
NT = 16


def check(logits, tau_rows, tau_scalar, k, p, seed, row_base, label):
    tok, logp, kept = e3.e3_sample_restricted(logits, tau_rows, tau_scalar, k, p, seed, row_base)
    torch.cuda.synchronize()
    ref = o.sample_restricted(wl.host_bits(logits), None if tau_rows is None else tau_rows.cpu().numpy(),
                              tau_scalar, k, p, seed, row_base, nthreads=NT)
    tok, logp, kept = tok.cpu().numpy(), logp.cpu().numpy(), kept.cpu().numpy()
    V = logits.shape[1]
    assert ((tok >= 0) & (tok < V)).all()
    cut_ok = ref.near_cut == 0
    bad_kept = (kept != ref.kept) & cut_ok
    assert not bad_kept.any(), f"{label}: kept differs on rows {np.flatnonzero(bad_kept)[:8]}: " \
                               f"{kept[bad_kept][:8]} vs {ref.kept[bad_kept][:8]}"
    exempt = (ref.near_cut != 0) | (ref.near_tie != 0)
    bad_tok = (tok != ref.token) & ~exempt
    print(f"[{label}] rows={tok.size} near_cut={int(ref.near_cut.sum())} near_tie={int(ref.near_tie.sum())} "
          f"token mismatches={int((tok != ref.token).sum())} kept range {kept.min()}..{kept.max()}")
    assert not bad_tok.any(), f"{label}: tokens differ on rows {np.flatnonzero(bad_tok)[:8]}"
    same = tok == ref.token
    err = np.abs(logp[same] - ref.logp[same])
    assert (err <= 1e-4 * np.maximum(np.abs(ref.logp[same]), 1e-6)).all(), f"{label}: logp off by {err.max()}"
    return ref


@pytest.mark.gpu
@pytest.mark.parametrize("k,p", [(50, 1.0), (0, 0.9), (50, 0.95), (1, 1.0), (0, 1.0), (3, 0.5)])
def test_decode_rows_full_vocab(k, p):
    w = wl.decode_step(DEV, seed=1, prompts=8, rollouts=8)            # 64 rows x 151,936 bf16
    check(w.logits, w.tau_rows, 1.0, k, p, seed=17, row_base=1000, label=f"decode k={k} p={p}")


@pytest.mark.gpu
def test_cuts_among_negative_values_and_back():
    g = torch.Generator(device=DEV).manual_seed(31)
    lg = (torch.randn((12, 40_000), generator=g, device=DEV) * 3).to(torch.bfloat16)
    tau = (0.6 + 0.8 * torch.rand(12, generator=g, device=DEV)).float()
    # about half of the values are negative: k = 30,000 puts the count cut among them
    check(lg, tau, 1.0, 30_000, 1.0, 5, 0, "k among negatives")
    # ... and the nucleus of that set ends among the non-negative values again (third sweep)
    check(lg, tau, 1.0, 30_000, 0.5, 5, 0, "k among negatives, p back")
    # nucleus that needs negative values: a flat row at a high temperature
    check(lg, None, 50.0, 0, 0.9, 5, 0, "p among negatives")
    check(lg, None, 50.0, 30_000, 0.99, 5, 0, "k and p among negatives")
    # rows without any non-negative value
    neg = (lg.float() - 40.0).to(torch.bfloat16)
    check(neg, tau, 1.0, 40, 0.9, 6, 0, "all negative")
    check(neg, tau, 1.0, 0, 1.0, 6, 0, "all negative, no cut")


@pytest.mark.gpu
@pytest.mark.parametrize("V", [1, 5, 8, 1000, 8200 + 4, 70_001 + 7])
def test_shapes_and_tails(V):
    g = torch.Generator(device=DEV).manual_seed(V)
    pitch = -(-V // 8) * 8
    lg = (torch.randn((9, pitch), generator=g, device=DEV) * 2.5).to(torch.bfloat16)[:, :V]
    check(lg, None, 0.8, 7, 0.9, V, 3, f"V={V}")
    check(lg, None, 0.8, 0, 1.0, V, 3, f"V={V} no cut")


@pytest.mark.gpu
def test_widest_accepted_row():
    V = 1_040_384
    g = torch.Generator(device=DEV).manual_seed(44)
    lg = (torch.randn((2, V), generator=g, device=DEV) * 2.5).to(torch.bfloat16)
    check(lg, None, 0.9, 50, 0.95, 8, 1, "widest row k=50 p=0.95")
    check(lg, None, 0.9, 0, 0.9, 8, 1, "widest row p=0.9")
    same = torch.full((1, V), -1.5, device=DEV).to(torch.bfloat16)     # one level of 1,040,384 columns
    r = check(same, None, 1.0, 3, 0.5, 2, 0, "widest row, all equal")
    assert (r.kept == V).all()


@pytest.mark.gpu
def test_levels_longer_than_a_16_bit_counter():
    # the one-sweep form counts in 16 bits; a level of 65,536 columns or more wraps its counter
    # (into its neighbour when it sits in the low half of a word, into nothing in the high half)
    # and the row must be recognised and recounted in 32 bits.  65,535 still fits.
    V = 200_000
    g = torch.Generator(device=DEV).manual_seed(45)
    even, odd = 0.5, 0.50390625                        # bf16 patterns 0x3F00 and 0x3F01: one LDS word
    base = (torch.randn((6, V), generator=g, device=DEV) * 0.05 - 2.0)
    runs = [(65_536, even, 0, odd), (65_536, odd, 0, even), (65_535, even, 65_535, odd),
            (70_000, odd, 3, even), (131_072, even, 1, odd), (65_537, odd, 65_536, even)]
    for r, (n_a, v_a, n_b, v_b) in enumerate(runs):
        perm = torch.randperm(V, generator=g, device=DEV)
        base[r, perm[:n_a]] = v_a
        base[r, perm[n_a:n_a + n_b]] = v_b
    lg = base.to(torch.bfloat16)
    for k, p in [(0, 0.9), (1000, 1.0), (0, 0.2), (100_000, 0.999), (300, 0.5)]:
        check(lg, None, 1.0, k, p, 21, 5, f"long levels k={k} p={p}")


@pytest.mark.gpu
def test_repeated_values_and_signed_zeros():
    # few distinct values: every level holds many columns, cuts fall inside repeated values
    g = torch.Generator(device=DEV).manual_seed(8)
    vals = torch.tensor([3.0, 2.5, 2.5, 1.0, 0.0, -0.0, -1.0, -1.0, -4.0], device=DEV)
    idx = torch.randint(0, vals.numel(), (16, 5000), generator=g, device=DEV)
    lg = vals[idx].to(torch.bfloat16)
    for k, p in [(10, 1.0), (600, 0.9), (0, 0.7), (3000, 1.0), (3000, 0.999), (0, 1.0)]:
        check(lg, None, 1.2, k, p, 3, 77, f"repeated k={k} p={p}")
    same = torch.full((4, 2048), 0.5, device=DEV).to(torch.bfloat16)
    r = check(same, None, 1.0, 5, 0.3, 1, 0, "all equal")
    assert (r.kept == 2048).all()


@pytest.mark.gpu
def test_top_k_exactly_on_a_level_boundary():
    # every row is a permutation of one multiset, so the cumulative level counts are the same
    # in all rows and k can be put exactly on a boundary, one before and one after it
    counts = [(3.0, 1), (2.5, 37), (1.0, 1200), (0.0, 700), (-0.0, 11), (-1.0, 2500), (-4.0, 551)]
    base = torch.cat([torch.full((n,), v) for v, n in counts])
    V = base.numel()
    g = torch.Generator().manual_seed(3)
    lg = torch.stack([base[torch.randperm(V, generator=g)] for _ in range(6)]).to(torch.bfloat16).to(DEV)
    cum = np.cumsum([n for _, n in counts])
    for j in (0, 1, 2, 3, 4, 5):
        for k in (int(cum[j]) - 1, int(cum[j]), int(cum[j]) + 1):
            if k < 1:
                continue
            r = check(lg, None, 0.9, k, 1.0, 5, 40, f"boundary level {j} k={k}")
            want = int(cum[np.searchsorted(cum, k)])          # first cumulative count >= k
            assert (r.kept == want).all(), (j, k, r.kept, want)


@pytest.mark.gpu
def test_frequencies_follow_the_truncated_softmax():
    vals = torch.tensor([[2.0, 1.5, 2.0, 0.5, 1.5, 1.5, -1.0, 0.5, 0.0, -0.0, 3.0, -2.0, -2.0, 1.0, 0.25, -3.0]],
                        device=DEV)
    n = 40_000
    lg = vals.to(torch.bfloat16).expand(n, 16).contiguous()
    tok, logp, kept = e3.e3_sample_restricted(lg, None, 1.1, 9, 0.97, seed=11, row_base=0)
    tok = tok.cpu().numpy()
    ref = o.sample_restricted(wl.host_bits(lg[:1]), None, 1.1, 9, 0.97, 11, 0)
    assert (kept.cpu().numpy() == ref.kept[0]).all()
    v = vals[0].double().cpu().numpy()
    order = np.sort(v)[::-1]
    keep = v >= order[ref.kept[0] - 1]
    pr = np.where(keep, np.exp((v - v.max()) / np.float32(1.1)), 0.0)
    pr /= pr.sum()
    counts = np.bincount(tok, minlength=16)
    assert counts[~keep].sum() == 0
    chi2, pval = stats.chisquare(counts[keep], pr[keep] * n)
    assert pval > 1e-3, (chi2, pval)


@pytest.mark.gpu
def test_rows_do_not_depend_on_batching():
    w = wl.decode_step(DEV, seed=3, prompts=2, rollouts=4, V=20_000)
    a = e3.e3_sample_restricted(w.logits, w.tau_rows, 1.0, 40, 0.9, seed=5, row_base=50)
    b = e3.e3_sample_restricted(w.logits[3:6], w.tau_rows[3:6].contiguous(), 1.0, 40, 0.9, seed=5, row_base=53)
    for x, y in zip(a, b):
        assert torch.equal(x[3:6], y)


def test_argument_checks_need_no_gpu():
    L = e3.lib()
    call = lambda dtype=1, k=5, p=0.9, tok=0x2000, tau=1.0: L.e3_sample_restricted(
        0x1000, dtype, 4, 64, 64, None, tau, k, p, 1, 0, tok, None, None, None)
    assert call(dtype=0, k=0) == -5       # fp32 rows are served for 1 <= top_k <= 256 only
    assert call(dtype=0, k=257) == -5
    assert call(dtype=7) == -3
    assert call(k=-1) == -5
    assert call(p=0.0) == -5 and call(p=float("nan")) == -5 and call(p=-0.5) == -5
    assert call(tau=0.0) == -5
    assert call(tok=None) == -1
    assert L.e3_sample_restricted(None, 1, 0, 64, 64, None, 1.0, 5, 0.9, 1, 0, None, None, None, None) == 0


def _random_cases(n, seed):
    rng = np.random.default_rng(seed)
    out = []
    for i in range(n):
        V = int(rng.choice([rng.integers(1, 100), rng.integers(100, 9000), rng.integers(9000, 60_000)]))
        rows = int(rng.integers(1, 12))
        k = int(rng.choice([0, 1, 2, rng.integers(3, 200), rng.integers(1, V + 2), V // 2 + 1]))
        p = float(rng.choice([1.0, 0.999, 0.9, 0.5, 0.1, 1e-4]))
        out.append((i, V, rows, k, p, float(rng.choice([0.1, 1.0, 4.0, 60.0])), float(rng.choice([0.3, 3.0, 10.0])),
                    float(rng.choice([0.0, 0.0, -8.0, 8.0]))))
    return out


@pytest.mark.gpu
@pytest.mark.parametrize("i,V,rows,k,p,tau,sigma,shift", _random_cases(32, 77))
def test_seeded_random_settings(i, V, rows, k, p, tau, sigma, shift):
    g = torch.Generator(device=DEV).manual_seed(500 + i)
    pitch = -(-V // 8) * 8 + 8 * (i % 2)
    lg = (torch.randn((rows, pitch), generator=g, device=DEV) * sigma + shift).to(torch.bfloat16)[:, :V]
    tau_rows = None if i % 2 else (tau * (0.5 + torch.rand(rows, generator=g, device=DEV))).float()
    check(lg, tau_rows, tau, k, p, seed=i, row_base=i << 20, label=f"case {i}: {rows}x{V} k={k} p={p} tau={tau}")


# ---------------------------------------------------------------- fp32 rows and the selection path
# top_k <= 256 is served by selection (chunk maxima, a lower bound from the thread maxima, an
# exact radix select) for bf16 and fp32 rows alike; larger k and top-p alone need the bf16 histogram.
@pytest.mark.gpu
@pytest.mark.parametrize("k,p", [(50, 1.0), (50, 0.95), (1, 1.0), (256, 0.9), (3, 0.5), (200, 1e-4)])
def test_fp32_decode_rows_full_vocab(k, p):
    w = wl.decode_step(DEV, seed=2, prompts=8, rollouts=8)
    lg = w.logits.float() + 1e-3 * torch.randn(w.logits.shape, device=DEV,
                                               generator=torch.Generator(device=DEV).manual_seed(k))
    check(lg, w.tau_rows, 1.0, k, p, seed=19, row_base=1 << 35, label=f"fp32 decode k={k} p={p}")


@pytest.mark.gpu
@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float32])
@pytest.mark.parametrize("V", [1, 3, 4, 5, 8, 9, 1000, 4096, 8200 + 4, 70_001 + 7, 300_000])
def test_selection_shapes_and_tails(V, dtype):
    g = torch.Generator(device=DEV).manual_seed(V + 1)
    per = 8 if dtype == torch.bfloat16 else 4
    pitch = -(-V // per) * per
    lg = (torch.randn((5, pitch), generator=g, device=DEV) * 2.5).to(dtype)[:, :V]
    for k, p in ((7, 0.9), (1, 1.0), (256, 1.0), (64, 0.3)):
        check(lg, None, 0.8, k, p, V, 3, f"select V={V} {dtype} k={k} p={p}")


@pytest.mark.gpu
@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float32])
def test_selection_repeated_values_plateaus_and_signed_zeros(dtype):
    g = torch.Generator(device=DEV).manual_seed(9)
    vals = torch.tensor([3.0, 2.5, 2.5, 1.0, 0.0, -0.0, -1.0, -1.0, -4.0], device=DEV)
    idx = torch.randint(0, vals.numel(), (12, 5000), generator=g, device=DEV)
    lg = vals[idx].to(dtype)
    for k, p in [(1, 1.0), (10, 1.0), (200, 0.9), (256, 0.999), (256, 0.2)]:
        check(lg, None, 1.2, k, p, 3, 77, f"select repeated {dtype} k={k} p={p}")
    # zeros of both signs around the cut: +0 ranks above -0
    z = torch.zeros((6, 3000), device=DEV)
    z[:, ::3] = -0.0
    z[:, 5::7] = 0.5
    z[:, 1::11] = -0.25
    check(z.to(dtype), None, 0.9, 256, 1.0, 4, 5, f"select zeros {dtype}")
    check(z.to(dtype), None, 0.9, 255, 0.95, 4, 5, f"select zeros {dtype} p")
    # one level holds the whole row: the cut level is a plateau, its pos-th column is counted out
    same = torch.full((4, 2048), 0.5, device=DEV).to(dtype)
    r = check(same, None, 1.0, 5, 0.3, 1, 0, f"select all equal {dtype}")
    assert (r.kept == 2048).all()
    # the same inside a short candidate list: nothing above the cut level, 200 columns on it
    same_small = torch.full((4, 200), 0.5, device=DEV).to(dtype)
    r = check(same_small, None, 1.0, 5, 0.3, 1, 0, f"select all equal, short row {dtype}")
    assert (r.kept == 200).all()
    wide = torch.full((2, 40_000), -1.5, device=DEV)
    wide[:, 17] = 2.0
    r = check(wide.to(dtype), None, 1.0, 3, 1.0, 2, 0, f"select plateau under one peak {dtype}")
    assert (r.kept == 40_000).all()
    # a cut level of 150 equal columns under ten larger ones, the rest far below: a short candidate
    # list whose cut level is longer than the 64 columns that are listed apart; the level holds
    # most of the mass, so most rows draw from it
    lvl = torch.full((24, 3000), -20.0, device=DEV) - torch.rand((24, 3000), generator=g, device=DEV)
    for r in range(24):
        perm = torch.randperm(3000, generator=g, device=DEV)
        lvl[r, perm[:150]] = 0.5
        lvl[r, perm[150:160]] = 0.75 + 0.125 * torch.arange(10, device=DEV)
    for k, p in [(20, 1.0), (20, 0.999), (64, 1.0), (11, 0.9)]:
        r = check(lvl.to(dtype), None, 1.0, k, p, 12, 0, f"select long cut level {dtype} k={k} p={p}")
        assert (r.kept == 160).all()
    # rows without a non-negative value, and values down in the subnormals
    neg = (torch.randn((6, 9000), generator=g, device=DEV) * 3 - 40.0).to(dtype)
    check(neg, None, 1.0, 40, 0.9, 6, 0, f"select all negative {dtype}")
    tiny = (torch.randn((4, 3000), generator=g, device=DEV) * 1e-39).to(dtype)
    check(tiny, None, 1.0, 9, 1.0, 6, 0, f"select subnormal {dtype}")


@pytest.mark.gpu
def test_selection_on_sorted_and_blocky_rows():
    # adversarial for the lower bound: the largest values sit next to each other (one chunk holds
    # many kept columns) or are spread so that single threads hold several of them
    V = 151_936
    asc = torch.arange(V, device=DEV, dtype=torch.float32) * 1e-4
    rows = torch.stack([asc, asc.flip(0), torch.roll(asc, 12345), (asc % 7.0) + (asc > 15.0) * 3.0])
    for dtype in (torch.float32, torch.bfloat16):
        for k in (1, 17, 256):
            check(rows.to(dtype), None, 0.5, k, 0.97, 8, 9, f"select sorted {dtype} k={k}")


@pytest.mark.gpu
def test_selection_widest_row():
    V = 1_040_384
    g = torch.Generator(device=DEV).manual_seed(45)
    lg = (torch.randn((2, V), generator=g, device=DEV) * 2.5)
    check(lg, None, 0.9, 50, 0.95, 8, 1, "select widest fp32")
    check(lg.to(torch.bfloat16), None, 0.9, 256, 0.95, 8, 1, "select widest bf16")
    same = torch.full((1, V), -1.5, device=DEV)
    r = check(same, None, 1.0, 3, 0.5, 2, 0, "select widest fp32, all equal")
    assert (r.kept == V).all()


def _random_select_cases(n, seed):
    rng = np.random.default_rng(seed)
    out = []
    for i in range(n):
        V = int(rng.choice([rng.integers(1, 100), rng.integers(100, 9000), rng.integers(9000, 60_000)]))
        rows = int(rng.integers(1, 10))
        k = int(rng.choice([1, 2, rng.integers(3, 257), 256]))
        p = float(rng.choice([1.0, 0.999, 0.9, 0.5, 0.1, 1e-4]))
        out.append((i, V, rows, k, p, float(rng.choice([0.1, 1.0, 4.0, 60.0])), float(rng.choice([0.3, 3.0, 10.0])),
                    float(rng.choice([0.0, 0.0, -8.0, 8.0])), bool(rng.integers(0, 2))))
    return out


@pytest.mark.gpu
@pytest.mark.parametrize("i,V,rows,k,p,tau,sigma,shift,coarse", _random_select_cases(40, 78))
def test_seeded_random_fp32_settings(i, V, rows, k, p, tau, sigma, shift, coarse):
    g = torch.Generator(device=DEV).manual_seed(900 + i)
    pitch = -(-V // 4) * 4 + 4 * (i % 2)
    lg = (torch.randn((rows, pitch), generator=g, device=DEV) * sigma + shift)
    if coarse:                                     # few distinct values: levels with many columns
        lg = torch.round(lg * 4) / 4
    lg = lg[:, :V]
    tau_rows = None if i % 2 else (tau * (0.5 + torch.rand(rows, generator=g, device=DEV))).float()
    check(lg, tau_rows, tau, k, p, seed=i, row_base=i << 21, label=f"fp32 case {i}: {rows}x{V} k={k} p={p} tau={tau}")


@pytest.mark.gpu
def test_fp32_rows_need_a_small_top_k():
    lg = torch.zeros((2, 64), device=DEV)
    for k in (0, 257, 1000):
        with pytest.raises(e3.E3Error) as ei:
            e3.e3_sample_restricted(lg, None, 1.0, k, 0.9, 1, 0)
        assert ei.value.status == -5


# ---------------------------------------------------------------- the near window and what lies outside it
# 32 binades up to [256, 512) (or one above the magnitude of the largest logit of the first vectors) are
# counted directly; nearer to zero than that: at most 62 columns, listed; zeros apart; below it: masked columns.
# A row that this does not hold is counted once more in a window raised or lowered for it; everything else
# takes the wide form.  Bars as for every test of this file.
def _outside_rows(kind, V, rows, g):
    x = torch.randn((rows, V), generator=g, device=DEV) * 3

    def put(n, values):
        for r in range(rows):
            cols = torch.randperm(V, generator=g, device=DEV)[:n]
            x[r, cols] = values(n)

    sign = lambda n: (torch.randint(0, 2, (n,), generator=g, device=DEV) * 2 - 1).float()
    if kind.startswith("small"):                  # the list up to, at and past its capacity; repeated values
        n = int(kind[5:])
        put(n, lambda n: sign(n) * 2.0 ** -torch.randint(24, 60, (n,), generator=g, device=DEV).float())
    elif kind == "zeros":
        put(V // 3, lambda n: sign(n) * 0.0)
    elif kind == "zeros_and_small":
        put(V // 4, lambda n: sign(n) * 0.0)
        put(20, lambda n: sign(n) * 1e-12)
    elif kind == "zeros_and_many_small":
        put(V // 4, lambda n: sign(n) * 0.0)
        put(300, lambda n: sign(n) * 1e-12)
    elif kind == "masked_inf":
        put(V // 2, lambda n: torch.full((n,), -float("inf"), device=DEV))
    elif kind == "masked_lowest":
        put(V // 2, lambda n: torch.full((n,), torch.finfo(torch.bfloat16).min, device=DEV))
    elif kind == "masked_1e4":
        put(V // 2, lambda n: torch.full((n,), -1e4, device=DEV))
    elif kind == "large_first":                   # the window moves up with the first vectors
        x *= 3000.0
    elif kind == "large_late":                    # ... which do not show it
        x[:, V // 2:] *= 3000.0
        x[:, -1] = 9000.0
    elif kind == "all_below":
        x = x * 10 - 2000.0
    elif kind == "subnormal":
        x *= 1e-39
    elif kind == "subnormal_and_zeros":           # a window that reaches down to the zeros
        x *= 1e-39
        put(V // 3, lambda n: sign(n) * 0.0)
    elif kind == "tiny":                          # the window moves down
        x *= 3e-5
    elif kind == "tiny_first":                    # ... and the row's rest lies above it
        x[:, :V * 3 // 4] *= 1e-7
    elif kind == "raised_twice":                  # larger than what the second window was made for
        x[:, V // 2:] *= 3000.0
        x[:, -1] = 1e30
    elif kind == "masked_first":                  # the first vectors show nothing but a mask
        x[:, :V * 3 // 4] = -1e4
    elif kind == "masked_first_lowest":
        x[:, :V * 3 // 4] = torch.finfo(torch.bfloat16).min
    elif kind == "masked_added":                  # several levels below the window
        put(V // 2, lambda n: -1e4 + 100 * torch.randn(n, generator=g, device=DEV))
    elif kind == "masked_few_left":
        x[:, torch.randperm(V, generator=g, device=DEV)[50:]] = -1e4
    elif kind == "below_weighs":                  # columns below the window that still count
        put(V // 2, lambda n: -520.0 - 3 * torch.rand(n, generator=g, device=DEV))
        x -= 300.0
    return x.to(torch.bfloat16)


@pytest.mark.gpu
@pytest.mark.parametrize("kind", ["small1", "small61", "small62", "small63", "small500", "zeros", "zeros_and_small", "zeros_and_many_small",
                                  "masked_inf", "masked_lowest", "masked_1e4", "large_first", "large_late",
                                  "all_below", "subnormal", "subnormal_and_zeros", "tiny", "tiny_first", "raised_twice",
                                  "masked_first", "masked_first_lowest", "masked_added", "masked_few_left",
                                  "below_weighs"])
@pytest.mark.parametrize("V", [3_003, 70_001])
def test_levels_outside_the_near_window(kind, V):
    g = torch.Generator(device=DEV).manual_seed(V + sum(map(ord, kind)))
    pitch = -(-V // 8) * 8
    lg = torch.full((6, pitch), 77.0, device=DEV).to(torch.bfloat16)         # what lies past a row must not count
    lg[:, :V] = _outside_rows(kind, V, 6, g)
    lg = lg[:, :V]
    # high temperatures put the cuts among the small values and the zeros, and the draw with them;
    # a count cut of 90 % of the row lies among the masked columns
    for k, p, tau in [(0, 0.9, 1.0), (0, 0.5, 60.0), (0, 0.55, 900.0), (V // 2, 1.0, 60.0), (V // 2 + 7, 0.99, 500.0),
                      (9 * V // 10, 0.999, 5.0), (9 * V // 10, 1.0, 1.0), (300, 0.7, 2.0), (300, 1.0, 20.0)]:
        if kind == "masked_inf" and p == 1.0 and k > V // 2:
            continue                              # the cut would lie among the infinite columns: no levels here
        check(lg, None, tau, k, p, 6, 40, f"outside {kind} V={V} k={k} p={p} tau={tau}")
    if kind != "masked_inf":                      # without a cut the infinite columns are no level here
        check(lg, None, 60.0, 0, 1.0, 6, 40, f"outside {kind} V={V} no cut")


# Eight waves per row, or sixteen for few rows of 114,688 columns and more; a vector holds 8 columns, a stream step 4096
# or 8192, the first 4 steps choose the window.
@pytest.mark.gpu
@pytest.mark.parametrize("V", [7, 9, 4_095, 4_097, 16_383, 16_390, 114_687, 114_689, 131_075])
def test_edges_of_the_near_window_and_of_the_row(V):
    g = torch.Generator(device=DEV).manual_seed(V)
    rows, pitch = 6, -(-V // 8) * 8 + 8
    tail = V - V // 8 * 8                             # the columns behind the last complete vector
    x = torch.randn((rows, pitch), generator=g, device=DEV) * 3
    edges = torch.tensor([511.9, 510.0, 384.0, 256.0, -511.9, -384.0, 2.0 ** -23, 1.5 * 2.0 ** -23, 1.49 * 2.0 ** -23,
                          -1.5 * 2.0 ** -23, -1.25 * 2.0 ** -23, 0.0, -0.0], device=DEV)
    for r in range(rows):                             # levels at both ends of the window, anywhere in the row
        n = min(V, edges.numel() * 2)
        x[r, torch.randperm(V, generator=g, device=DEV)[:n]] = edges[torch.randint(0, edges.numel(), (n,), generator=g, device=DEV)]
    if tail:                                          # ... and in its last columns
        x[1, V - tail:V] = torch.tensor([512.0, 0.0, -0.0, 1e-12, -1e4, -float("inf"), 3.0], device=DEV)[:tail]
        x[2, V - tail:V] = -1e4
    x[3, :min(V - 1, 20_000)] = -300.0                # nothing but negative values at first
    x[4, :V] -= 3000.0
    x[4, V - 1] = 400.0                               # far above everything that the first vectors show
    lg = x.to(torch.bfloat16)
    lg[:, V:] = 77.0                                  # what lies past a row must not count
    lg = lg[:, :V]
    for k, p, tau in [(0, 0.9, 1.0), (0, 0.999, 0.5), (0, 0.6, 400.0), (0, 0.9, 0.02), (V // 2 + 1, 0.99, 300.0), (300, 0.7, 2.0)]:
        if (k > 256 or k == 0) and k <= V - 3:        # an infinite column is no level: no cut may reach it
            check(lg, None, tau, k, p, 6, 40, f"edges V={V} k={k} p={p} tau={tau}")


def _by_c_call(lg, tau, k, p, seed, ws, ws_bytes):
    rows, V = lg.shape
    out = [torch.empty(rows, dtype=t, device=DEV) for t in (torch.int32, torch.float32, torch.int32)]
    rc = e3.lib().e3_sample_restricted_ws(lg.data_ptr(), e3.E3_BF16, rows, V, lg.stride(0), None, tau, k, p, seed, 9,
                                          out[0].data_ptr(), out[1].data_ptr(), out[2].data_ptr(),
                                          ws, ws_bytes, torch.cuda.current_stream().cuda_stream)
    assert rc == 0
    return out


# Few rows of 65,536 columns and more are cut into eight slices (sixteen from 524,225 columns on) given a workspace:
# slices of equal and unequal length, with and without columns behind the last complete vector.
@pytest.mark.gpu
@pytest.mark.parametrize("rows,V", [(1, 65_536), (16, 65_543), (5, 131_071), (3, 524_224), (2, 524_232), (2, 1_040_384)])
def test_cut_rows_give_what_whole_rows_give(rows, V):
    need = e3.lib().e3_restricted_workspace_bytes(e3.E3_BF16, rows, V, 0)
    assert need == rows * (8 if V <= 524_224 else 16) * (16_384 + 544)
    g = torch.Generator(device=DEV).manual_seed(V)
    pitch = -(-V // 8) * 8
    for kind in ("plain", "late", "small", "masked", "zeros", "wide", "at_most_zero", "tiny_positive", "few_negative", "few_larger"):
        x = torch.randn((rows, pitch), generator=g, device=DEV) * 3
        if kind == "late":
            x[0, V - 1] = 9000.0                      # above the window: counted anew by the second launch
        elif kind == "small":                         # listed by several slices; row 0 more than the list holds
            x[:, 5:V:V // 50] = 2.0 ** -30
            x[0, 3:V:V // 90] = -(2.0 ** -28)
        elif kind == "masked":
            x = torch.where(torch.rand(x.shape, generator=g, device=DEV) < 0.999, -1e4, x)
            x[0, :V // 3] = -float("inf")
        elif kind == "zeros":
            x = torch.relu(x)
            x[:, 1:V:2] *= -1.0
        elif kind == "wide":
            x[0] = 0.5                                # one level longer than a quarter's counters
            x[rows - 1] = -600.0 - x[rows - 1]        # columns below the window that weigh
            x[rows - 1, 7] = -590.0
        elif kind == "at_most_zero":                  # nothing positive: the columns that matter are zeros and negative ones
            x = x.clamp(max=0)
        elif kind == "tiny_positive":
            x = torch.where(x < 0, x, x * 1e-4)
        elif kind == "few_negative":                  # ordinary negative values that a sample hardly meets
            x *= 1e-4
            x[:, 3:V:V // 30] = -20.0
        elif kind == "few_larger":                    # ... and positive ones
            x *= 1e-4
            x[:, 3:V:V // 30] = -300.0
            x[:, 5:V:V // 20] = 6.0
        lg = x.to(torch.bfloat16)
        lg[:, V:] = 77.0                              # what lies past a row must not count
        lg = lg[:, :V]
        ws = torch.randint(0, 256, (need,), generator=g, device=DEV, dtype=torch.uint8)      # its contents do not matter
        for k, p, tau in [(0, 0.9, 1.0), (300, 0.95, 0.7), (V // 2, 0.999, 40.0), (0, 0.7, 500.0)]:
            want = _by_c_call(lg, tau, k, p, 3, None, 0)
            for got in (_by_c_call(lg, tau, k, p, 3, ws.data_ptr(), need), _by_c_call(lg, tau, k, p, 3, ws.data_ptr(), need - 1)):
                assert torch.equal(got[2], want[2]), (kind, k, p, tau)
                assert torch.equal(got[0], want[0]), (kind, k, p, tau)
                assert torch.allclose(got[1], want[1], rtol=1e-6, atol=1e-7, equal_nan=True), (kind, k, p, tau)
    check(lg, None, 1.0, 0, 0.9, 3, 9, f"cut rows {rows}x{V}")


def _held(rows):
    return [torch.empty(rows, dtype=t, device=DEV) for t in (torch.int32, torch.float32, torch.int32)]


def _few_rows(rows=8, V=65_536, seed=1):
    g = torch.Generator(device=DEV).manual_seed(seed)
    return (torch.randn((rows, V), generator=g, device=DEV) * 3).to(torch.bfloat16)


@pytest.mark.gpu
@pytest.mark.parametrize("native", [True, False])
def test_a_call_that_is_given_its_outputs_allocates_nothing(native, monkeypatch):
    e3.lib()
    if not native:
        monkeypatch.setattr(e3.binding, "_native", None)
    lg = _few_rows()
    need = e3.e3_restricted_workspace_bytes(e3.E3_BF16, *lg.shape, 0)
    want = e3.e3_sample_restricted(lg, None, 1.0, 0, 0.9, 3)
    ws = torch.empty(need, dtype=torch.uint8, device=DEV)
    allocations = lambda: torch.cuda.memory_stats()["allocation.all.allocated"]
    for workspace in (None, False, ws):
        out = _held(8)
        before = allocations()
        got = e3.e3_sample_restricted(lg, None, 1.0, 0, 0.9, 3, 0, *out, workspace=workspace)
        assert allocations() == before
        assert all(a is b for a, b in zip(got, out))
        assert torch.equal(got[0], want[0]) and torch.equal(got[2], want[2])
        assert torch.allclose(got[1], want[1], rtol=1e-6, atol=1e-7)
    for bad in (ws.cpu(), ws[::2]):                   # a workspace that the launch could not use
        with pytest.raises(ValueError):
            e3.e3_sample_restricted(lg, None, 1.0, 0, 0.9, 3, workspace=bad)


@pytest.mark.gpu
@pytest.mark.parametrize("native", [True, False])
def test_few_rows_without_memory_for_a_workspace(native, monkeypatch):
    e3.lib()
    if not native:
        monkeypatch.setattr(e3.binding, "_native", None)
    lg = _few_rows(64, 262_144)
    need = e3.e3_restricted_workspace_bytes(e3.E3_BF16, 64, 262_144, 0)
    want = [x.clone() for x in e3.e3_sample_restricted(lg, None, 1.0, 0, 0.9, 3, 0, *_held(64))]
    torch.cuda.empty_cache()
    torch.cuda.set_per_process_memory_fraction(1e-9)          # torch's allocator gets no further memory
    held = []
    try:
        with pytest.raises(torch.OutOfMemoryError):
            for _ in range(1000):                             # what it has left in large pieces
                held.append(torch.empty(need, dtype=torch.uint8, device=DEV))
        got = e3.e3_sample_restricted(lg, None, 1.0, 0, 0.9, 3, 0, *_held(64)[:2])       # allocates one small output
    finally:
        torch.cuda.set_per_process_memory_fraction(1.0)
    for a, b in zip(got, want):
        assert torch.equal(a, b)                              # whole rows either way


@pytest.mark.gpu
def test_cut_rows_on_two_streams():
    # each call with a workspace of its own, from torch: many calls in flight on both streams give what single ones do
    batches = [_few_rows(8, 70_001 // 8 * 8, seed) for seed in range(4)]
    want = [[x.clone() for x in e3.e3_sample_restricted(lg, None, 1.0, 0, 0.9, 3)] for lg in batches]
    streams = [torch.cuda.Stream(), torch.cuda.Stream()]
    torch.cuda.synchronize()
    got = []
    for i in range(40):
        with torch.cuda.stream(streams[i % 2]):
            got.append(e3.e3_sample_restricted(batches[i % 4], None, 1.0, 0, 0.9, 3))
    torch.cuda.synchronize()
    for i, out in enumerate(got):
        for a, b in zip(out, want[i % 4]):
            assert torch.equal(a, b), i


def test_workspace_of_cut_rows_needs_no_gpu():
    need = e3.lib().e3_restricted_workspace_bytes
    assert need(e3.E3_BF16, 8, 151_936, 0) == 8 * 8 * (16_384 + 544)
    assert need(e3.E3_BF16, 8, 151_936, 50) == 0 and need(e3.E3_F32, 8, 151_936, 0) == 0
    assert need(e3.E3_BF16, 8, 65_535, 0) == 0 and need(e3.E3_BF16, 512, 151_936, 0) == 0
    assert need(e3.E3_BF16, 0, 151_936, 0) == 0 and need(e3.E3_BF16, -1, 151_936, 0) == 0 and need(7, 8, 151_936, 0) == 0


@pytest.mark.gpu
def test_draws_among_listed_values_and_zeros():
    # most of the mass on a zero level and on small listed values, so that the draw falls on them
    rows, V = 64, 5_000
    g = torch.Generator(device=DEV).manual_seed(12)
    lg = torch.full((rows, V), -30.0, device=DEV)
    for r in range(rows):
        cols = torch.randperm(V, generator=g, device=DEV)
        lg[r, cols[:40]] = 2.0 ** -torch.randint(24, 28, (40,), generator=g, device=DEV).float()
        lg[r, cols[40:60]] = -2.0 ** -30
        lg[r, cols[60:90]] = 0.0
        lg[r, cols[90:120]] = -0.0
    lg = lg.to(torch.bfloat16)
    for k, p in [(0, 1.0), (0, 0.5), (0, 0.99), (300, 0.4), (60, 1.0), (45, 0.9)]:
        check(lg, None, 1.0, k, p, 31, 7, f"draws among listed values k={k} p={p}")


@pytest.mark.gpu
def test_levels_longer_than_a_quarter_counter():
    # a level of 65,536 columns or more within a quarter of the row wraps its 16-bit counter: 49 steps of 8192
    # columns, 13 to a quarter; quarters 0 and 2 count in the low halves of the words, 1 and 3 in the high ones
    V, quarter = 400_000, 13 * 8192
    g = torch.Generator(device=DEV).manual_seed(46)
    base = torch.randn((8, V), generator=g, device=DEV) * 0.05 - 2.0
    base[0, :65_536] = 0.5
    base[1, quarter:quarter + 65_535] = 0.5         # one short of wrapping, high half
    base[2, :] = torch.where(torch.rand(V, generator=g, device=DEV) < 0.9, 0.5, base[2])
    base[3, 100_000:300_000] = -1.0
    base[4, 2 * quarter:2 * quarter + 65_535] = 0.5  # ... low half
    base[5, quarter:quarter + 65_536] = 0.5         # the high half wraps
    base[6, :65_535] = 0.5                          # both halves of a word one short of wrapping
    base[6, quarter:quarter + 65_535] = 0.5
    base[7, quarter + 1:quarter + 1 + 65_535] = 0.5  # a full counter and one column in the next quarter
    base[7, 2 * quarter] = 0.5
    lg = base.to(torch.bfloat16)
    for k, p in [(0, 0.9), (1000, 1.0), (0, 0.2), (100_000, 0.999)]:
        check(lg, None, 1.0, k, p, 21, 5, f"long quarter levels k={k} p={p}")


# ---------------------------------------------------------------- selection: both workgroup sizes, list overflow
# 1024 threads per row up to one row per compute unit, 512 beyond; the list of vectors holds 2688.
@pytest.mark.gpu
@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float32])
@pytest.mark.parametrize("rows", [9, 260])
@pytest.mark.parametrize("V", [1, 15, 16, 17, 63, 64, 65, 128, 129, 192, 193, 252, 256, 257])
def test_short_candidate_lists(V, rows, dtype):
    # so few vectors that (nearly) every column is a candidate: the sizes at which the ranking of a list changes its split over
    # the waves (64, 128, 256 entries) and reads (16), on both workgroup sizes, with levels that end before, at
    # and behind the 64th entry
    g = torch.Generator(device=DEV).manual_seed(V + rows)
    x = torch.randn((rows, -(-V // 8) * 8), generator=g, device=DEV) * 2.5
    x[1::5] = (x[1::5] * 2).round() / 2                                # few distinct values
    x[2::5] = 0.75                                                     # one level
    x[3::5] = torch.where(x[3::5] > 1.0, x[3::5], torch.full_like(x[3::5], -1.0))     # a cut level that is a plateau
    x[4::5, ::3] = 0.0
    x[4::5, 1::3] = -0.0
    lg = x.to(dtype)[:, :V]
    for k, p in [(64, 1.0), (64, 0.7), (20, 0.9), (1, 0.5)]:
        check(lg, None, 0.8, k, p, V + k, 7, f"V={V} rows={rows} {dtype} k={k} p={p}")


@pytest.mark.gpu
@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float32])
@pytest.mark.parametrize("rows,V", [(256, 33_001), (257, 5), (257, 4_099), (260, 16_387), (260, 33_001), (300, 70_001)])
def test_selection_workgroup_sizes(rows, V, dtype):
    g = torch.Generator(device=DEV).manual_seed(rows + V)
    per = 8 if dtype == torch.bfloat16 else 4
    pitch = -(-V // per) * per
    lg = torch.full((rows, pitch), 77.0, device=DEV).to(dtype)               # what lies past a row must not count
    lg[:, :V] = torch.randn((rows, V), generator=g, device=DEV) * 2.5
    lg[3, :V] = 0.25                                                          # a plateau among ordinary rows
    lg[4, :V] = torch.sort(lg[4, :V].float()).values.to(dtype)
    lg[5, :V:2] = -float("inf")
    lg = lg[:, :V]
    for k, p in ((50, 0.95), (1, 1.0), (64, 1.0), (65, 0.9), (256, 0.9)):
        if V == 5 and k > 1:
            continue                              # infinite columns would reach the cut: no levels here
        check(lg, None, 0.8, k, p, V, 3, f"select {rows}x{V} {dtype} k={k} p={p}")


@pytest.mark.gpu
@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float32])
@pytest.mark.parametrize("rows,threads", [(6, 1024), (258, 512)])
def test_selection_rows_that_mislead_the_first_bound(rows, threads, dtype):
    # the vectors that the first requests take hold small values, all others large ones: the list
    # overflows with the first bound and is made again with the final one
    g = torch.Generator(device=DEV).manual_seed(threads)
    per = 8 if dtype == torch.bfloat16 else 4
    slots = 24
    V = slots * threads * per - 3
    lg = torch.randn((rows, slots * threads * per), generator=g, device=DEV) + 20.0
    nsets = -(-slots // 8)
    for s in range(0, slots, nsets):
        lg[:, s * threads * per:(s + 1) * threads * per] -= 40.0
    lg = lg.to(dtype)[:, :V]
    for k, p in ((50, 0.9), (256, 1.0)):
        check(lg, None, 0.7, k, p, 5, 9, f"misled {threads} {dtype} k={k}")


@pytest.mark.gpu
@pytest.mark.parametrize("rows", [6, 258])
@pytest.mark.parametrize("kind", ["offset", "negative", "few_patterns", "one_ulp", "subnormal", "around_zero"])
def test_selection_of_fp32_values_that_share_their_upper_bits(kind, rows):
    # the bound of the listed vectors comes from all 32 bits: rows whose largest values differ in the lower
    # sixteen only, repeat a few patterns of those, or lie around the two zeros
    V = 40_003
    g = torch.Generator(device=DEV).manual_seed(sum(map(ord, kind)) + rows)
    x = torch.randn((rows, -(-V // 4) * 4), generator=g, device=DEV)
    if kind == "offset":
        x = 100.0 + 0.3 * x
    elif kind == "negative":
        x = -100.0 + 0.02 * x
    elif kind == "few_patterns":
        x = 100.0 + (x * 3).round() * 2.0 ** -14
    elif kind == "one_ulp":
        x = (1.0 + (torch.rand(x.shape, generator=g, device=DEV) < 0.001).float() * 2.0 ** -23) * torch.ones_like(x)
    elif kind == "subnormal":
        x = x * 1e-41
    elif kind == "around_zero":
        x = torch.where(x > 3.5, x * 1e-42, -0.0 * torch.ones_like(x))
    lg = x[:, :V]
    for k, p in ((1, 1.0), (20, 0.9), (50, 0.95), (200, 0.99)):
        check(lg, None, 0.8, k, p, 3, 5, f"shared upper bits {kind} k={k} p={p}")


@pytest.mark.gpu
@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float32])
@pytest.mark.parametrize("rows,V", [(3, 140_003), (258, 70_001)])
@pytest.mark.parametrize("kind", ["relu", "signed_zeros", "masked_1e4", "masked_lowest", "two_levels", "coarse", "climbing",
                                  "falling", "equal"])
def test_selection_of_rows_that_are_mostly_a_plateau(kind, rows, V, dtype):
    # most of a row is one value and the bound starts there: with k below, at and above the number of columns
    # that stand out of it; sorted rows, whose large columns all lie in one wave's vectors
    g = torch.Generator(device=DEV).manual_seed(rows + sum(map(ord, kind)))
    shape = (rows, -(-V // 8) * 8)
    x = torch.randn(shape, generator=g, device=DEV) * 3
    if kind == "relu":
        x = torch.relu(x - 9.0)                       # 0.13 % stand out
    elif kind == "signed_zeros":
        x = torch.where(x > 10.5, x, torch.where(x > 0, 0.0, -0.0))
    elif kind == "masked_1e4":
        x = torch.where(torch.rand(shape, generator=g, device=DEV) < 0.9995, -1e4, x)
    elif kind == "masked_lowest":
        x = torch.where(torch.rand(shape, generator=g, device=DEV) < 0.9995, torch.finfo(dtype).min, x)
    elif kind == "two_levels":
        x = (torch.rand(shape, generator=g, device=DEV) < 0.002).float() * 2
    elif kind == "coarse":
        x = 100.0 + (x * 0.2).round() * 0.5           # the cut level is long, too
    elif kind == "climbing":
        x = torch.sort(x, 1).values
    elif kind == "falling":
        x = torch.sort(x, 1, descending=True).values
    else:
        x = torch.full(shape, 0.5, device=DEV)
    lg = x.to(dtype).contiguous()
    lg[:, V:] = 77.0                                  # what lies past a row must not count
    lg = lg[:, :V]
    for k, p in ((20, 0.9), (50, 0.95), (200, 1.0)):
        check(lg, None, 0.8, k, p, 11, 2, f"plateau {kind} {rows}x{V} {dtype} k={k} p={p}")


@pytest.mark.gpu
@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float32])
@pytest.mark.parametrize("rows,V", [(18, 20_003), (270, 20_003), (18, 140_001)])
def test_selection_where_maxima_are_not_positive(rows, V, dtype):
    # the stream takes bf16 maxima as signed integers, which is wrong for vectors without a non-negative value: rows of which all,
    # most or some lanes or vectors hold none, cuts at zero and below it, and patterns that are no numbers of either sign
    g = torch.Generator(device=DEV).manual_seed(rows + V)
    x = torch.randn((rows, -(-V // 8) * 8), generator=g, device=DEV) * 3
    x[0::9] -= 60.0                                                    # negative throughout
    x[1::9] = torch.where(torch.rand(x[1::9].shape, generator=g, device=DEV) < 2e-4, x[1::9].abs(), -x[1::9].abs() - 1.0)
    x[2::9] = -torch.relu(x[2::9])                                     # zeros on top, half of the columns
    x[3::9] = torch.where(x[3::9] > 11.0, x[3::9], torch.full_like(x[3::9], -0.0))
    x[4::9, 40:] = -x[4::9, 40:].abs()                                 # forty columns that may be positive
    x[5::9, ::7] = float("nan")
    x[5::9, 1::7] = float("-inf")
    x[6::9, 5::1000] = float("inf")
    x[6::9] -= 8.0
    x[7::9] = torch.where(x[7::9] > 6.0, torch.zeros_like(x[7::9]), -x[7::9].abs())        # +0 and -0 at the cut
    x[7::9, 3::50] = -0.0
    x[8::9, 4_000:] = -1.0e4
    full = x.to(dtype)
    lg = full[:, :V]
    bits = lg.view(torch.int16 if dtype == torch.bfloat16 else torch.int32)
    bits[5::9, 2::7] |= -0x8000 if dtype == torch.bfloat16 else -0x80000000    # negative values, and NaN of the negative sign
    numbers = torch.isfinite(lg).all(1)
    assert int((~numbers).sum()) == 2 * rows // 9
    finite = full.clone()[:, :V]                                       # (with its pitch)
    finite[~numbers] = 0.0
    for k, p in [(50, 0.95), (64, 1.0), (3, 1.0), (200, 0.9)]:
        check(finite, None, 0.9, k, p, k, 5, f"not positive {rows}x{V} {dtype} k={k} p={p}")
        # patterns that are no numbers are no levels: the row without these columns
        tok, logp, kept = (t.cpu() for t in e3.e3_sample_restricted(lg, None, 0.9, k, p, k, 5))
        for r in (~numbers).nonzero().squeeze(1).tolist()[:6]:
            cols = torch.isfinite(lg[r]).nonzero().squeeze(1)
            ref = o.sample_restricted(wl.host_bits(lg[r, cols].unsqueeze(0)), None, 0.9, k, p, k, 5 + r)
            assert ref.near_cut[0] or kept[r] == ref.kept[0], (r, k)
            if not (ref.near_cut[0] or ref.near_tie[0]):
                assert int(tok[r]) == int(cols[int(ref.token[0])]), (r, k)
                assert abs(float(logp[r]) - ref.logp[0]) <= 1e-4 * max(abs(ref.logp[0]), 1e-6)

"""What the speed of this library is measured on: its public entry points on the inputs that an
RL loop with large-vocabulary logits brings, from a handful of rows to a whole training batch.

A case is a dict of plain values.  `prepare` makes what a program has in hand before the call
(logits, temperatures, target ids, rewards, preallocated outputs, workspace), `run` is one pass
through the entry points of `paper_2505_18573_amd`, `work` what the pass cannot do without,
`exact` the same results in 64 bits from plain torch.  Logits are N(0, 3^2) with a few columns
per row raised by 8 (a peaked next-token distribution), as in the benchmark's workloads.
"""
import math
import statistics

import torch

import paper_2505_18573_amd as e3

DEV = "cuda"
DTYPES = {"bf16": torch.bfloat16, "f32": torch.float32}


def listed():
    return [
        # the advantages of one step's rollouts: 64 prompts x 8 (the smallest call there is)
        {"name": "advantages_64x8", "kind": "advantages", "groups": 64, "size": 8, "mixed": False},
        # decoding with a few sequences left: launches and latency; buffers held by the loop
        {"name": "sample_4_rows", "kind": "sample", "rows": 4, "V": 151_936, "dtype": "bf16",
         "tau": "rows", "held": True},
        # one decode step of 64 prompts x 8 rollouts
        {"name": "sample_512_rows", "kind": "sample", "rows": 512, "V": 151_936, "dtype": "bf16",
         "tau": "rows", "held": True},
        # fp32 logits, a width that is no multiple of anything, outputs allocated by the call
        {"name": "sample_f32_ragged", "kind": "sample", "rows": 100, "V": 70_005, "dtype": "f32",
         "tau": "scalar", "held": False},
        # training side: every response token of a batch, some of it padding
        {"name": "logprob_32768_rows", "kind": "logprob", "rows": 32_768, "V": 151_936, "dtype": "bf16",
         "tau": "scalar", "masked": 0.1, "gap": False},
        # training side with the measured gap of the temperature update, fp32 logits, small vocabulary
        {"name": "gap_f32", "kind": "logprob", "rows": 1000, "V": 32_000, "dtype": "f32",
         "tau": "rows", "masked": 0.25, "gap": True},
        # a whole step: statistics and advantages of the last rollouts, the temperature update on the
        # host from the two numbers in pinned memory, the next sample at the new temperature
        {"name": "rl_step_512_rows", "kind": "step", "rows": 512, "V": 151_936, "dtype": "bf16", "size": 8},
        # truncated sampling of a decode step: nucleus alone
        {"name": "top_p_512_rows", "kind": "restricted", "rows": 512, "V": 151_936, "dtype": "bf16",
         "tau": "rows", "top_k": 0, "top_p": 0.9},
        # ... a count cut followed by a nucleus
        {"name": "top_k50_p_512_rows", "kind": "restricted", "rows": 512, "V": 151_936, "dtype": "bf16",
         "tau": "rows", "top_k": 50, "top_p": 0.95},
        # ... a nucleus for a few interactive sequences
        {"name": "top_p_8_rows", "kind": "restricted", "rows": 8, "V": 151_936, "dtype": "bf16",
         "tau": "scalar", "top_k": 0, "top_p": 0.95},
        # ... fp32 logits with a small count cut
        {"name": "top_k20_f32_100_rows", "kind": "restricted", "rows": 100, "V": 128_000, "dtype": "f32",
         "tau": "scalar", "top_k": 20, "top_p": 0.8},
        # the objective of one step: 512 rollouts of up to 8192 tokens, very different lengths
        {"name": "objective_512_rollouts", "kind": "objective", "groups": 64, "size": 8, "longest": 8192},
    ]


def _log_int(rng, lo, hi):
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng):
    kind = rng.choice(["advantages", "sample", "sample", "sample", "logprob", "logprob", "step",
                       "restricted", "restricted", "restricted", "objective", "objective"])
    if kind == "advantages":
        return {"kind": kind, "groups": _log_int(rng, 4, 4096), "size": rng.choice([4, 8, 12, 16]),
                "mixed": rng.random() < 0.5}
    if kind == "objective":
        return {"kind": kind, "groups": _log_int(rng, 4, 256), "size": rng.choice([4, 8, 12]),
                "longest": _log_int(rng, 128, 16_384)}
    c = {"kind": kind, "rows": 0, "V": rng.choice([151_936, 32_000, 128_000, _log_int(rng, 1000, 260_000)]),
         "dtype": rng.choice(["bf16", "bf16", "f32"])}
    most_rows = {"sample": 4096, "logprob": 8192, "step": 1024, "restricted": 1024}[kind]
    c["rows"] = _log_int(rng, 1, most_rows)
    if kind == "step":
        c["size"] = rng.choice([4, 8])
        c["rows"] = max(1, c["rows"] // c["size"]) * c["size"]
        return c
    c["tau"] = rng.choice(["rows", "scalar"])
    if kind == "sample":
        c["held"] = rng.random() < 0.5
    elif kind == "logprob":
        c["masked"] = rng.choice([0.0, 0.1, 0.5])
        c["gap"] = rng.random() < 0.4
    else:
        c["top_k"] = rng.choice([20, 50, _log_int(rng, 1, 256)] + ([0, 0, 0] if c["dtype"] == "bf16" else []))
        c["top_p"] = rng.choice([1.0, 0.8, 0.9, 0.95]) if c["top_k"] else rng.choice([0.8, 0.9, 0.95, 0.99])
    return c


# ---------------------------------------------------------------- inputs (from the seed alone)
def _pitch(V, dtype):
    per = 8 if dtype == "bf16" else 4             # rows start on 16 bytes
    return -(-V // per) * per


def _logits(rows, V, dtype, g):
    out = torch.empty((rows, _pitch(V, dtype)), dtype=DTYPES[dtype], device=DEV)
    for r0 in range(0, rows, 2048):
        r1 = min(rows, r0 + 2048)
        x = torch.randn((r1 - r0, out.shape[1]), generator=g, device=DEV).mul_(3.0)
        cols = torch.randint(0, V, (r1 - r0, 20), generator=g, device=DEV)
        x.scatter_(1, cols, torch.gather(x, 1, cols) + 8.0)
        out[r0:r1] = x
    return out[:, :V]


def _tau(case, g):
    if case.get("tau") == "rows":
        return (0.6 + 0.8 * torch.rand(case["rows"], generator=g, device=DEV)).float(), 1.0
    return None, 0.9


def _offsets(sizes):
    out = torch.zeros(sizes.numel() + 1, dtype=torch.int64, device=DEV)
    out[1:] = torch.cumsum(sizes, 0)
    return out.to(torch.int32)


def _lengths(case):
    """Rollout lengths: the quantiles of a log-normal law cut off at the longest; most are far below it."""
    n = case["groups"] * case["size"]
    law = statistics.NormalDist(-1.2, 0.8)
    return [max(1, int(min(1.0, math.exp(law.inv_cdf((i + 0.5) / n))) * case["longest"])) for i in range(n)]


def _inputs(case, seed):
    g = torch.Generator(device=DEV).manual_seed(seed)
    s = {"seed": seed % 1_000_003}
    kind = case["kind"]
    if kind in ("advantages", "objective"):
        sizes = torch.full((case["groups"],), case["size"], device=DEV)
        if case.get("mixed"):                     # budgets that differ per prompt
            sizes = 2 + torch.arange(case["groups"], device=DEV) % (2 * case["size"] - 1)
            sizes = sizes[torch.randperm(case["groups"], generator=g, device=DEV)]
        s["group_offsets"] = _offsets(sizes)
        n = int(s["group_offsets"][-1])
        p = torch.rand(case["groups"], generator=g, device=DEV).repeat_interleave(sizes)
        s["rewards"] = (torch.rand(n, generator=g, device=DEV) < p).float()
    if kind == "objective":
        lens = torch.tensor(_lengths(case), device=DEV)
        s["seq_offsets"] = _offsets(lens[torch.randperm(n, generator=g, device=DEV)])
        T = int(s["seq_offsets"][-1])
        s["logp_old"] = -torch.rand(T, generator=g, device=DEV).pow(4) * 12.0
        s["logp_new"] = s["logp_old"] + 0.15 * torch.randn(T, generator=g, device=DEV)
        s["adv"] = torch.randn(n, generator=g, device=DEV)
    if kind in ("sample", "logprob", "restricted", "step"):
        s["logits"] = _logits(case["rows"], case["V"], case["dtype"], g)
        s["tau_rows"], s["tau"] = _tau(case, g)
    if kind in ("logprob", "step"):
        s["targets"] = torch.randint(0, case["V"], (case["rows"],), generator=g, device=DEV).to(torch.int32)
        # half of the targets are a likely token, as the sampled ones of a rollout are
        rows = torch.arange(0, case["rows"], 2, device=DEV)
        for r in rows.split(2048):
            s["targets"][r] = s["logits"][r].argmax(1).to(torch.int32)
        s["mask"] = None
        if case.get("masked"):
            s["mask"] = (torch.rand(case["rows"], generator=g, device=DEV) >= case["masked"]).to(torch.uint8)
    if kind == "step":
        s["tau"] = 1.0
        s["group_offsets"] = _offsets(torch.full((case["rows"] // case["size"],), case["size"], device=DEV))
        s["rewards"] = (torch.rand(case["rows"], generator=g, device=DEV) < 0.5).float()
    return s


def prepare(case, seed):
    s = _inputs(case, seed)
    s["case"] = case
    kind, rows, V = case["kind"], case.get("rows", 0), case.get("V", 0)
    f32 = lambda n: torch.empty(n, dtype=torch.float32, device=DEV)
    if kind == "advantages":
        s["out"] = f32(s["rewards"].numel())
    if kind == "sample" and case["held"] or kind == "step":
        s["token"] = torch.empty(rows, dtype=torch.int32, device=DEV)
        s["logp"], s["entropy"] = f32(rows), f32(rows)
        s["workspace"] = e3.new_workspace(rows, V, DEV)
    if kind == "step":
        s["train"] = {"logp_out": f32(rows), "entropy_out": f32(rows), "adv_out": f32(rows),
                      "entropy_sum_out": torch.empty(1, dtype=torch.float64, pin_memory=True),
                      "entropy_count_out": torch.empty(1, dtype=torch.int64, pin_memory=True),
                      "workspace": s["workspace"]}
        s["event"] = torch.cuda.Event()
    return s


def run(s):
    c = s["case"]
    kind = c["kind"]
    if kind == "advantages":
        return e3.e3_grpo_advantages(s["rewards"], s["group_offsets"], adv_out=s["out"])
    if kind == "objective":
        J, seq_mean, terms = e3.e3_grpo_objective(s["logp_new"], s["logp_old"], s["seq_offsets"], s["adv"],
                                                  s["group_offsets"], 0.2, want_token_terms=True)
        return {"objective": J, "seq_mean": seq_mean, "terms": terms}
    if kind == "sample":
        if c["held"]:
            tok, logp, ent = e3.e3_sample_entropy(s["logits"], s["tau_rows"], s["tau"], s["seed"], 0, s["token"],
                                                  s["logp"], s["entropy"], workspace=s["workspace"])
        else:
            tok, logp, ent = e3.e3_sample_entropy(s["logits"], s["tau_rows"], s["tau"], s["seed"])
        return {"token": tok, "logp": logp, "entropy": ent}
    if kind == "restricted":
        tok, logp, kept = e3.e3_sample_restricted(s["logits"], s["tau_rows"], s["tau"], c["top_k"], c["top_p"],
                                                  s["seed"])
        return {"token": tok, "logp": logp, "kept": kept}
    if kind == "logprob" and c["gap"]:
        logp, ent, gap, hs, gs, n = e3.e3_logprob_entropy_gap(s["logits"], s["targets"], s["mask"], s["tau_rows"],
                                                              s["tau"])
        return {"logp": logp, "entropy": ent, "gap": gap, "entropy_sum": hs, "gap_sum": gs, "count": n}
    if kind == "logprob":
        logp, ent, hs, n = e3.e3_logprob_entropy(s["logits"], s["targets"], s["mask"], s["tau_rows"], s["tau"])
        return {"logp": logp, "entropy": ent, "entropy_sum": hs, "count": n}
    # a whole step
    t = s["train"]
    e3.e3_logprob_entropy_advantages(s["logits"], s["targets"], None, None, 1.0, s["rewards"], s["group_offsets"], **t)
    s["event"].record()
    s["event"].synchronize()                      # the scheduler needs the two numbers
    H = float(t["entropy_sum_out"]) / float(t["entropy_count_out"])
    tau, _ = e3.e3_temperature_update(1.0, H, 1.02 * H, c["V"])
    e3.e3_sample_entropy(s["logits"], None, tau, s["seed"], 0, s["token"], s["logp"], s["entropy"],
                         workspace=s["workspace"])
    return {"train_logp": t["logp_out"], "train_entropy": t["entropy_out"], "adv": t["adv_out"],
            "entropy_sum": t["entropy_sum_out"], "count": t["entropy_count_out"], "tau": tau,
            "token": s["token"], "logp": s["logp"], "entropy": s["entropy"]}


def work(case):
    """Bytes: every input once, every output once.  Operations: an exponential, two multiply-adds, an
    add and a comparison per logit (seven), about ten per token of the objective."""
    kind = case["kind"]
    if kind == "advantages":
        sizes = [2 + i % (2 * case["size"] - 1) if case["mixed"] else case["size"] for i in range(case["groups"])]
        return {"bytes": 8 * sum(sizes) + 4 * (case["groups"] + 1), "flops": 6 * sum(sizes)}
    if kind == "objective":
        n = case["groups"] * case["size"]
        tokens = sum(_lengths(case))
        return {"bytes": 12 * tokens + 16 * n + 4 * case["groups"], "flops": 10 * tokens}
    esz = 2 if case["dtype"] == "bf16" else 4
    cells = case["rows"] * case["V"]
    passes = 2 if kind == "step" else 1           # the old policy's logits, then the new ones
    return {"bytes": passes * (cells * esz + 20 * case["rows"]), "flops": passes * 7 * cells}


def tolerance(case):
    # fp32 sums in another order; whole numbers (tokens, counts) only where a race or a cut is decided
    # inside fp32 rounding
    if case["kind"] == "advantages":
        return {"rel": 1e-6}
    if case["kind"] == "objective":
        return {"rel": 2e-6, "max": 1e-5}
    return {"rel": 1e-6, "max": 1e-5, "differ": 0.002}


# ---------------------------------------------------------------- the same results in 64 bits, plain torch
def _philox(index, row, stream, seed):
    """Word (index % 4) of Philox4x32-10 with counter (index / 4, row lo, row hi, stream)."""
    M = 0xFFFFFFFF
    c = [(index >> 2) & M, row & M, (row >> 32) & M, torch.full_like(index, stream)]
    c = [x.expand(index.shape) for x in c]
    k0, k1 = seed & M, (seed >> 32) & M
    for _ in range(10):
        pa, pb = c[0] * 0xD2511F53, c[2] * 0xCD9E8D57      # wraps mod 2^64, which keeps all 64 bits
        ha, la, hb, lb = (pa >> 32) & M, pa & M, (pb >> 32) & M, pb & M
        c = [hb ^ c[1] ^ k0, lb, ha ^ c[3] ^ k1, la]
        k0, k1 = (k0 + 0x9E3779B9) & M, (k1 + 0xBB67AE85) & M
    return torch.stack(c, -1).gather(-1, (index & 3).unsqueeze(-1)).squeeze(-1)


def _minus_ln_u(word):
    return -torch.log(((word >> 9).double() + 0.5) * 2.0 ** -23)


def _tau64(case, s, lo, hi):
    if s["tau_rows"] is None:                     # the call takes it in 32 bits
        return torch.full((hi - lo, 1), float(torch.tensor(s["tau"], dtype=torch.float32)), dtype=torch.float64, device=DEV)
    return s["tau_rows"][lo:hi].double().unsqueeze(1)


def _rows64(case, s, tau=None):
    """(lo, hi, logits as fp64, a = logits / tau - max, ln sum exp a, entropy) in bounded chunks."""
    step = max(1, (1 << 27) // case["V"])
    for lo in range(0, case["rows"], step):
        hi = min(case["rows"], lo + step)
        z = s["logits"][lo:hi].double()
        t = _tau64(case, s, lo, hi) if tau is None else tau
        a = z / t
        a -= a.max(1, keepdim=True).values
        e = a.exp()
        S = e.sum(1)
        yield lo, hi, z, a, e, t, S.log(), S.log() - (a * e).sum(1) / S


def _exact_sample(case, s, tau=None):
    tokens, logps, entropies = [], [], []
    V = case["V"]
    nst = -(-V // 4096)
    for lo, hi, z, a, e, t, lnS, H in _rows64(case, s, tau):
        n = hi - lo
        row = torch.arange(lo, hi, device=DEV).unsqueeze(1)
        mass = torch.nn.functional.pad(e, (0, nst * 4096 - V)).view(n, nst, 8, 64, 8).sum((2, 4)).view(n, nst * 64)
        tile_ids = torch.arange(nst * 64, device=DEV).unsqueeze(0).expand(n, -1)
        tile = (mass / _minus_ln_u(_philox(tile_ids, row, 1, s["seed"]))).argmax(1)
        st, lane = tile // 64, tile % 64
        j = torch.arange(64, device=DEV).unsqueeze(0)
        col = st.unsqueeze(1) * 4096 + (j // 8) * 512 + lane.unsqueeze(1) * 8 + j % 8
        ok = col < V
        g = -_minus_ln_u(_philox(col, row, 2, s["seed"])).log()
        score = a.gather(1, col.clamp(max=V - 1)) + g
        tok = col.gather(1, score.masked_fill(~ok, -math.inf).argmax(1, keepdim=True))
        tokens.append(tok.squeeze(1))
        logps.append(a.gather(1, tok).squeeze(1) - lnS)
        entropies.append(H)
    return torch.cat(tokens), torch.cat(logps), torch.cat(entropies)


def _exact_restricted(case, s):
    V, k, p = case["V"], case["top_k"], float(torch.tensor(case["top_p"], dtype=torch.float32))
    bf16 = case["dtype"] == "bf16"
    tokens, logps, kepts = [], [], []
    for r in range(case["rows"]):
        x = s["logits"][r]
        bits = x.view(torch.int16).long() & 0xFFFF if bf16 else x.view(torch.int32).long() & 0xFFFFFFFF
        top = 1 << (15 if bf16 else 31)
        key = torch.where(bits >= top, 2 * top - 1 - bits, bits + top)     # value order, -0 below +0
        if k:
            key = key.masked_fill(key < key.topk(min(k, V)).values[-1], -1)
        levels, counts = torch.unique(key[key >= 0], return_counts=True)
        levels, counts = levels.flip(0), counts.flip(0).double()
        pattern = torch.where(levels >= top, levels - top, 2 * top - 1 - levels)
        z = (pattern << 16 if bf16 else pattern).to(torch.int32).view(torch.float32).double()
        tau = float(_tau64(case, s, r, r + 1))
        w = ((z - z[0]) / tau).exp() * counts
        M = w.cumsum(0)
        if p < 1.0:
            n = int((M < p * M[-1]).sum()) + 1
            pattern, z, w, M, counts, levels = (t[:n] for t in (pattern, z, w, M, counts, levels))
        row = torch.tensor(r, device=DEV)
        j = int((w / _minus_ln_u(_philox(pattern, row, 3, s["seed"]))).argmax())
        k23 = int(_philox(torch.zeros(1, dtype=torch.int64, device=DEV), row, 4, s["seed"])) >> 9
        tokens.append((key == levels[j]).nonzero().squeeze(1)[((2 * k23 + 1) * int(counts[j])) >> 24])
        logps.append((z[j] - z[0]) / tau - M[-1].log())
        kepts.append(counts.sum().long())
    return torch.stack(tokens), torch.stack(logps), torch.stack(kepts)


def _exact_advantages(s):
    sizes = (s["group_offsets"][1:] - s["group_offsets"][:-1]).long()
    group = torch.arange(sizes.numel(), device=DEV).repeat_interleave(sizes)
    mean_of = lambda x: torch.zeros(sizes.numel(), dtype=torch.float64, device=DEV).index_add_(0, group, x) / sizes
    r = s["rewards"].double()
    d = r - mean_of(r)[group]
    var = mean_of(d * d)[group]
    return torch.where(var > 0, d / var.sqrt(), torch.zeros_like(d))


def exact(case, seed):
    s = _inputs(case, seed)
    kind = case["kind"]
    if kind == "advantages":
        return _exact_advantages(s)
    if kind == "objective":
        sizes = (s["seq_offsets"][1:] - s["seq_offsets"][:-1]).long()
        seq = torch.arange(sizes.numel(), device=DEV).repeat_interleave(sizes)
        A = s["adv"].double()[seq]
        r = (s["logp_new"].double() - s["logp_old"].double()).exp()
        terms = torch.minimum(r * A, r.clamp(1 - 0.2, 1 + 0.2) * A)
        seq_mean = torch.zeros(sizes.numel(), dtype=torch.float64, device=DEV).index_add_(0, seq, terms) / sizes
        J = seq_mean.view(case["groups"], case["size"]).mean(1).mean().view(1)
        return {"objective": J, "seq_mean": seq_mean, "terms": terms}
    if kind == "restricted":
        tok, logp, kept = _exact_restricted(case, s)
        return {"token": tok, "logp": logp, "kept": kept}
    if kind == "sample":
        tok, logp, ent = _exact_sample(case, s)
        return {"token": tok, "logp": logp, "entropy": ent}
    logp, ent, gap = [], [], []
    for lo, hi, z, a, e, t, lnS, H in _rows64(case, s, 1.0 if kind == "step" else None):
        logp.append(a.gather(1, s["targets"][lo:hi].long().unsqueeze(1)).squeeze(1) - lnS)
        ent.append(H)
        if case.get("gap"):                       # mean of z_max - z_i over all tokens but one maximum
            rest = e.sum(1) - 1.0
            gap.append(-(a * e).sum(1) * (t.squeeze(1) if torch.is_tensor(t) else t) / rest)
    logp, ent = torch.cat(logp), torch.cat(ent)
    keep = torch.ones(case["rows"], dtype=torch.bool, device=DEV) if s["mask"] is None else s["mask"].bool()
    hs, n = ent[keep].sum().view(1), keep.sum().view(1)
    if kind == "logprob" and case["gap"]:
        gap = torch.cat(gap)
        return {"logp": logp, "entropy": ent, "gap": gap, "entropy_sum": hs, "gap_sum": gap[keep].sum().view(1),
                "count": n}
    if kind == "logprob":
        return {"logp": logp, "entropy": ent, "entropy_sum": hs, "count": n}
    H = float(hs) / case["rows"]
    V = case["V"]
    tau = 1.0 + math.log(1.02 * H / H) / (math.log(V) + math.log(math.log(V)))
    tau32 = float(torch.tensor(tau, dtype=torch.float32))
    tok, lp, en = _exact_sample(case, s, tau32)
    return {"train_logp": logp, "train_entropy": ent, "adv": _exact_advantages(s), "entropy_sum": hs, "count": n,
            "tau": tau, "token": tok, "logp": lp, "entropy": en}

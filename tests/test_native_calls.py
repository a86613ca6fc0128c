"""The binding's native calls against its Python path: the same outputs bit for bit, the same errors, and arguments
that are not plain tensors, ints and floats are left to the Python path."""
import struct

import numpy as np
import pytest
import torch

import paper_2505_18573_amd as e3

DEV = "cuda:0"


class Sub(torch.Tensor):
    pass


def _calls(dev, rows=6, V=40_000, groups=3):
    g = torch.Generator(device=dev).manual_seed(1)
    lg = (torch.randn((rows, V), generator=g, device=dev) * 3).to(torch.bfloat16)
    tau = (0.5 + torch.rand(rows, generator=g, device=dev)).float()
    tgt = torch.randint(0, V, (rows,), generator=g, device=dev).to(torch.int32)
    mask = torch.tensor([1, 0] * (rows // 2), dtype=torch.uint8, device=dev)
    off = torch.arange(0, rows + 1, rows // groups, dtype=torch.int32, device=dev)
    rew = torch.rand(rows, generator=g, device=dev)
    T = 100
    new, old = -torch.rand(T, generator=g, device=dev), -torch.rand(T, generator=g, device=dev)
    soff = torch.tensor([0, 10, 10, 40, 77, 90, T], dtype=torch.int32, device=dev)
    f32 = lambda n: torch.empty(n, dtype=torch.float32, device=dev)
    return {
        "sample": (e3.e3_sample_entropy, dict(logits=lg, tau_rows=tau, tau_scalar=1.0, seed=7, row_base=1 << 40)),
        "sample_into": (e3.e3_sample_entropy, dict(logits=lg, tau_rows=None, tau_scalar=1, seed=-3, logp_out=f32(rows), workspace=False)),
        "restricted": (e3.e3_sample_restricted, dict(logits=lg, tau_rows=tau, tau_scalar=1.0, top_k=0, top_p=0.9, seed=3)),
        "restricted_k": (e3.e3_sample_restricted, dict(logits=lg.float(), tau_rows=None, tau_scalar=0.7, top_k=20, top_p=1, seed=3)),
        "logprob": (e3.e3_logprob_entropy, dict(logits=lg, target_ids=tgt, row_mask=mask, tau_rows=tau, tau_scalar=1.0)),
        "logprob_plain": (e3.e3_logprob_entropy, dict(logits=lg, target_ids=None, row_mask=None, tau_rows=None, tau_scalar=0.8, want_sum=False)),
        "both": (e3.e3_logprob_entropy_advantages, dict(logits=lg, target_ids=tgt, row_mask=None, tau_rows=None, tau_scalar=1.0, rewards=rew,
                                                       group_offsets=off, ddof=1, eps=1e-6)),
        "advantages": (e3.e3_grpo_advantages, dict(rewards=rew, group_offsets=off, eps=0.5)),
        "objective": (e3.e3_grpo_objective, dict(logp_new=new, logp_old=old, seq_offsets=soff, adv=rew, group_offsets=off, clip_eps=0.2,
                                                 want_token_terms=True)),
        "objective_plain": (e3.e3_grpo_objective, dict(logp_new=new, logp_old=old, seq_offsets=soff, adv=rew, group_offsets=off, clip_eps=0)),
        "temperature": (e3.e3_temperature_update, dict(tau_t=1.0, H_t=0.5, H_init=0.6, vocab=1000, t=3, t_anneal=1, t_max=9, eta=0.5)),
    }


def _outcome(f, kw, monkeypatch, native):
    e3.lib()
    with monkeypatch.context() as m:
        if not native:
            m.setattr(e3.binding, "_native", None)
        try:
            out = f(**kw)
        except Exception as e:                        # the error is what is compared
            return type(e), str(e)
    if torch.cuda.is_available():
        torch.cuda.synchronize()
    return out if isinstance(out, tuple) else (out,)


NAMES = list(_calls("cpu", V=64))


@pytest.mark.gpu
@pytest.mark.parametrize("name", NAMES)
def test_same_outputs_as_the_python_path(name, monkeypatch):
    f, kw = _calls(DEV)[name]
    odd = dict(kw)                                    # values of types that the native calls leave alone
    for key, cast in (("seed", np.int64), ("tau_scalar", torch.tensor), ("ddof", np.int32), ("clip_eps", np.float64), ("tau_t", np.float64)):
        if key in odd:
            odd[key] = cast(odd[key])
    want = [x.clone() if torch.is_tensor(x) else x for x in _outcome(f, kw, monkeypatch, native=False)]
    for got in (_outcome(f, kw, monkeypatch, native=True), _outcome(f, odd, monkeypatch, native=True)):
        assert len(got) == len(want)
        for a, b in zip(got, want):
            if torch.is_tensor(b):
                assert a.dtype == b.dtype and a.device == b.device and torch.equal(a.view(torch.uint8), b.view(torch.uint8))
            else:
                assert a == b


def _spoilt(kw):
    """One argument at a time replaced by what the call must refuse."""
    for key, v in kw.items():
        if torch.is_tensor(v):
            yield dict(kw, **{key: v.to(torch.float64)})
            yield dict(kw, **{key: v[:-1]})
            yield dict(kw, **{key: v.repeat_interleave(2, -1)[..., ::2]})
            yield dict(kw, **{key: v.cpu()})
            yield dict(kw, **{key: 5})
            yield dict(kw, **{key: v.as_subclass(Sub)[:-1]})
        elif key in ("tau_scalar", "eps", "clip_eps", "top_p", "H_t", "tau_t"):
            yield dict(kw, **{key: -1.0})
            yield dict(kw, **{key: float("nan")})
            yield dict(kw, **{key: "x"})
        elif key in ("ddof", "top_k", "vocab"):
            yield dict(kw, **{key: -1})


def _same_errors(f, kw, monkeypatch):
    for bad in _spoilt(kw):
        want, got = (_outcome(f, bad, monkeypatch, native=n) for n in (False, True))
        if isinstance(want[0], type):
            assert got == want, bad
        else:                                         # not refused (a short reward list, say): not refused either way
            assert not isinstance(got[0], type), bad


@pytest.mark.parametrize("name", NAMES)
def test_same_errors_without_a_gpu(name, monkeypatch):
    if torch.cuda.is_available():
        pytest.skip("tensors on the CPU, all of them refused")
    f, kw = _calls("cpu", V=64)[name]
    if name != "temperature":
        with pytest.raises(ValueError):
            f(**kw)
    _same_errors(f, kw, monkeypatch)


@pytest.mark.gpu
@pytest.mark.parametrize("name", ["sample", "restricted", "logprob", "temperature"])
def test_same_errors(name, monkeypatch):
    # (calls whose shortened offsets or targets would be read out of bounds are not made here)
    f, kw = _calls(DEV)[name]
    _same_errors(f, kw, monkeypatch)


def test_the_module_brings_no_thread_local_storage():
    # loaded after torch's libraries, it would make their own thread-local variables slower to reach (see build_native)
    elf = open(e3.binding.NATIVE_PATH, "rb").read()
    assert elf[:6] == b"\x7fELF\x02\x01"
    at, = struct.unpack_from("<Q", elf, 32)
    size, n = struct.unpack_from("<HH", elf, 54)
    kinds = [struct.unpack_from("<I", elf, at + i * size)[0] for i in range(n)]
    assert 1 in kinds and 7 not in kinds                  # PT_LOAD, PT_TLS


def test_every_load_raises_while_a_library_is_missing(monkeypatch, tmp_path):
    b = e3.binding
    with monkeypatch.context() as m:
        m.setattr(b, "_lib", None)
        m.setattr(b, "_native", None)
        m.setattr(b, "NATIVE_PATH", str(tmp_path / "_native.so"))
        for _ in range(2):
            with pytest.raises(ImportError):
                e3.lib()
            with pytest.raises(ImportError):
                e3.e3_temperature_update(1.0, 0.5, 0.6, 1000)


# Every output and workspace given by the caller; the names are those of _ENTRY's calls.
HELD = ["sample", "restricted", "logprob", "both", "advantages", "objective"]


def _held_calls(name, dev):
    f, kw = _calls(dev)[name]
    rows, V = kw["logits"].shape if "logits" in kw else (6, 0)
    f32 = lambda: torch.empty(rows, dtype=torch.float32, device=dev)
    i32 = lambda: torch.empty(rows, dtype=torch.int32, device=dev)
    if name == "sample":
        kw.update(token_out=i32(), logp_out=f32(), entropy_out=f32(), workspace=e3.new_workspace(rows, V, dev))
    elif name == "restricted":
        kw.update(logits=torch.cat([kw["logits"], kw["logits"]], 1), token_out=i32(), logp_out=f32(), kept_out=i32())
        need = e3.e3_restricted_workspace_bytes(e3.E3_BF16, rows, 2 * V, kw["top_k"])
        assert need > 0
        kw.update(workspace=torch.empty(need, dtype=torch.uint8, device=dev))
    elif name == "logprob":
        kw.update(logp_out=f32(), entropy_out=f32(), entropy_sum_out=torch.empty(1, dtype=torch.float64, device=dev),
                  entropy_count_out=torch.empty(1, dtype=torch.int64, device=dev), workspace=e3.new_workspace(rows, V, dev))
    elif name == "both":
        kw.update(logp_out=f32(), entropy_out=f32(), adv_out=f32(), row_mask=torch.ones(rows, dtype=torch.uint8, device=dev),
                  tau_rows=f32().fill_(0.8), entropy_sum_out=torch.empty(1, dtype=torch.float64, pin_memory=True),
                  entropy_count_out=torch.empty(1, dtype=torch.int64, pin_memory=True), workspace=e3.new_workspace(rows, V, dev))
    elif name == "advantages":
        kw.update(adv_out=f32())
    return f, kw


def _refused(name, kw):
    """One tensor at a time replaced by one that the checks on the host refuse."""
    for key, v in kw.items():
        if not torch.is_tensor(v):
            continue
        if key == "workspace":
            if name == "restricted":                  # (elsewhere any tensor is taken)
                yield dict(kw, workspace=v.cpu())
                yield dict(kw, workspace=v.repeat_interleave(2)[::2])
            continue
        yield dict(kw, **{key: v.to(torch.float16)})
        if v.numel() > 1:
            yield dict(kw, **{key: v.repeat_interleave(2, -1)[..., ::2]})
        yield dict(kw, **{key: v.cpu()} if v.is_cuda else {key: v.clone()})          # on the host, and not pinned
        yield dict(kw, **{key: 5})
        yield dict(kw, **{key: torch.cat([v, v], -1)} if v.dim() == 1 and key not in ("rewards", "group_offsets") else {key: v[None]})


@pytest.mark.gpu
@pytest.mark.parametrize("name", HELD)
def test_given_outputs_and_what_the_checks_refuse(name, monkeypatch):
    f, kw = _held_calls(name, DEV)
    given = [v for k, v in kw.items() if k.endswith("_out")]
    want = [x if x is None else x.clone() for x in _outcome(f, kw, monkeypatch, native=False)]
    for t in given:
        t.zero_()
    got = _outcome(f, kw, monkeypatch, native=True)
    assert not isinstance(got[0], type) and all(any(t is x for x in got) for t in given)
    for a, b in zip(got, want):
        assert b is None or torch.equal(a.view(torch.uint8), b.view(torch.uint8))
    sub = dict(kw, **{k: v.as_subclass(Sub) for k, v in kw.items() if torch.is_tensor(v) and not k.endswith("_out")})
    for a, b in zip(_outcome(f, sub, monkeypatch, native=True), want):
        assert b is None or torch.equal(a.as_subclass(torch.Tensor).view(torch.uint8), b.view(torch.uint8))
    n = 0
    for bad in _refused(name, kw):
        refused, native = (_outcome(f, bad, monkeypatch, native=x) for x in (False, True))
        assert isinstance(refused[0], type) and native == refused, (bad, refused, native)
        n += 1
    assert n >= 8


# Logits in every layout that the checks let through, and two that they do not.
LAYOUTS = {
    "no rows": lambda x: x[:0],
    "one column": lambda x: x.as_strided((6, 1), (40_000, 8)),
    "one row, short pitch": lambda x: x.as_strided((1, 40_000), (8, 1)),
    "wide pitch": lambda x: x.repeat(1, 2)[:, :39_991],
    "few wide rows": lambda x: x.repeat(1, 4)[:, :159_997],
    "expanded": lambda x: x[:1].expand(6, -1),
    "misaligned pitch": lambda x: x.as_strided((5, 30_001), (30_001, 1)),
}


@pytest.mark.gpu
@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float32])
@pytest.mark.parametrize("layout", list(LAYOUTS))
def test_layouts_of_the_logits(layout, dtype, monkeypatch):
    lg = LAYOUTS[layout](_calls(DEV)["sample"][1]["logits"].to(dtype))
    rows = lg.shape[0]
    tgt, mask = torch.zeros(rows, dtype=torch.int32, device=DEV), torch.ones(rows, dtype=torch.uint8, device=DEV)
    refused = layout in ("expanded", "misaligned pitch")
    for f, kw in [(e3.e3_sample_entropy, dict(tau_rows=None, tau_scalar=0.8, seed=5)),
                  (e3.e3_sample_restricted, dict(tau_rows=None, tau_scalar=0.8, top_k=0, top_p=0.9, seed=5)),
                  (e3.e3_sample_restricted, dict(tau_rows=None, tau_scalar=0.8, top_k=7, top_p=0.9, seed=5)),
                  (e3.e3_logprob_entropy, dict(target_ids=tgt, row_mask=mask, tau_rows=None, tau_scalar=0.8))]:
        want, got = (_outcome(f, dict(kw, logits=lg), monkeypatch, native=n) for n in (False, True))
        if refused or (dtype == torch.float32 and kw.get("top_k") == 0):
            assert isinstance(want[0], type) and got == want
            continue
        for a, b in zip(got, want):
            assert a.shape == b.shape and torch.equal(a.view(torch.uint8), b.view(torch.uint8)), (f, kw)


@pytest.mark.gpu
@pytest.mark.parametrize("V", [1_000, 40_000])
@pytest.mark.parametrize("target,mask,tau,workspace", [(True, True, True, None), (False, False, False, False), (True, False, True, "own")])
def test_gap_call(V, target, mask, tau, workspace, monkeypatch):
    c = _calls(DEV, V=V)["logprob"][1]
    kw = dict(logits=c["logits"], target_ids=c["target_ids"] if target else None, row_mask=c["row_mask"] if mask else None,
              tau_rows=c["tau_rows"] if tau else None, tau_scalar=0.9,
              workspace=e3.new_workspace(6, V, DEV) if workspace == "own" else workspace)
    want = [x.clone() if torch.is_tensor(x) else x for x in _outcome(e3.e3_logprob_entropy_gap, kw, monkeypatch, native=False)]
    native = e3.binding._native.logprob_gap(kw["logits"], kw["target_ids"], kw["row_mask"], kw["tau_rows"], kw["tau_scalar"], kw["workspace"])
    for got in (native, _outcome(e3.e3_logprob_entropy_gap, kw, monkeypatch, native=True)):
        assert len(got) == len(want) == 6
        for a, b in zip(got, want):
            assert a is b is None or (a.dtype == b.dtype and a.shape == b.shape and torch.equal(a.view(torch.uint8), b.view(torch.uint8)))
    for wrong in (dict(tau_scalar=-1.0, tau_rows=None), dict(logits=kw["logits"].half()), dict(target_ids=torch.zeros(5, dtype=torch.int32, device=DEV)),
                  dict(row_mask=torch.ones(6, device=DEV)), dict(logits=kw["logits"].cpu())):
        a, b = (_outcome(e3.e3_logprob_entropy_gap, {**kw, **wrong}, monkeypatch, native=n) for n in (True, False))
        assert a == b and issubclass(a[0], Exception), wrong

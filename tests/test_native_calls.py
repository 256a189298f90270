"""The binding's native calls (csrc/dodo_torch.cpp) against the same calls through ctypes: results, returned objects and
refusals are the same, and what is not in the plain form is declined."""
import threading
import types

import pytest
import torch

import paper_2310_02409_amd.binding as B

NAMES = ("score", "select_topk", "gather_nuggets", "nugget_attention", "nugget_attention_indexed", "nugget_attention_cached",
         "stream_append", "score_mlp")


@pytest.fixture
def without_native(monkeypatch):
    def switch():
        monkeypatch.setattr(B, "_native", types.SimpleNamespace(**{n: (lambda *a: None) for n in NAMES}))
    return switch


class Recording:
    """The extension module, with a note of which calls it did itself."""
    def __init__(self, module):
        self.done = []
        for n in NAMES:
            setattr(self, n, self._noting(n, getattr(module, n)))

    def _noting(self, name, f):
        def call(*a):
            r = f(*a)
            if r is not None:
                self.done.append(name)
            return r
        return call


def _inputs(device, dtype):
    g = torch.Generator().manual_seed(5)
    r = lambda *s, dt=dtype: torch.randn(s, generator=g).to(dt).to(device)
    cu = lambda *v: torch.tensor(v, dtype=torch.int32, device=device)
    t = dict(hidden=r(300, 256), w=r(256), W1=r(256, 256), b1=r(256, dt=torch.float32), K=r(300, 4, 64), V=r(300, 4, 64),
             Q=r(40, 4, 64), Kl=r(60, 4, 64), Vl=r(60, 4, 64), cu_s=cu(0, 100, 300), cu_k=cu(0, 10, 30), cu_q=cu(0, 20, 40), cu_l=cu(0, 25, 60),
             Q1=r(2, 4, 64), cu_q1=cu(0, 1, 2), starts=cu(0, 10), counts=cu(10, 20), cacheK=r(2, 40, 4, 64), cacheV=r(2, 40, 4, 64),
             rows=r(2, 4, 64), lam=torch.tensor([0.0], device=device), s2=torch.tensor([1.0, -1.0], device=device))
    return t


def _calls(t):
    """Every function in the forms that programs use: results allocated or given, optional arguments named or left out."""
    out = {}
    s = out["score"] = B.dodo_score(t["hidden"], t["w"], 0.5)
    mine = torch.empty(300, device=s.device)
    assert B.dodo_score(t["hidden"], t["w"], bias=0.5, scores=mine) is mine
    out["score given"] = mine
    idx = out["select"] = B.dodo_select_topk(s, t["cu_s"], t["cu_k"], 200, 20, 30, B.FORCE_LAST)
    kn, vn = out["gather"] = B.dodo_gather_nuggets(t["K"], t["V"], idx, t["cu_s"], t["cu_k"], 30)
    out["gather head"] = B.dodo_gather_nuggets(t["K"], t["V"], idx, t["cu_s"], t["cu_k"], 30, B.HEAD_MAJOR)
    hk, hv = out["gather head"]
    a = (t["Kl"], t["Vl"], t["cu_q"], t["cu_k"], t["cu_l"], 20, 20, 35)
    out["attention"] = B.dodo_nugget_attention(t["Q"], kn, vn, *a)
    O = torch.empty_like(t["Q"])
    got = out["attention lse"] = B.dodo_nugget_attention(t["Q"], kn, vn, *a, 0.2, O=O, want_lse=True)
    assert got[0] is O and got[1].shape == (40, 4)
    lse = torch.empty(40, 4, device=O.device)
    got = out["attention head"] = B.dodo_nugget_attention(t["Q"], hk, hv, *a, 0.2, B.HEAD_MAJOR, lse=lse)
    assert got[1] is lse
    out["attention indexed"] = B.dodo_nugget_attention_indexed(t["Q"], t["K"], t["V"], idx, t["cu_s"], *a, 200, want_lse=True)
    ck, cv = t["cacheK"].clone(), t["cacheV"].clone()
    counts = t["counts"].clone()
    assert B.dodo_stream_append(t["s2"], t["lam"], t["rows"], t["rows"], counts, ck, cv) is None
    out["append"] = (counts, ck, cv)
    ws = torch.zeros(1 << 20, dtype=torch.uint8, device=O.device)
    out["cached"] = B.dodo_nugget_attention_cached(t["Q1"], ck.view(-1, 4, 64), cv.view(-1, 4, 64), t["Kl"], t["Vl"], t["cu_q1"], t["starts"],
                                                   counts, t["cu_l"], 1, 40, 35, ws=ws)
    out["mlp"] = B.dodo_score_mlp(t["hidden"], t["W1"], t["b1"], t["w"], 0.1, B.GELU)
    out["mlp few"] = B.dodo_score_mlp(t["hidden"][:7], t["W1"], t["b1"], t["w"])
    return out


def _flat(v):
    return [x for y in v for x in _flat(y)] if isinstance(v, (tuple, list)) else [v]


@pytest.mark.gpu
@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
def test_same_results_as_through_ctypes(dtype, monkeypatch, without_native):
    t = _inputs("cuda", dtype)
    noting = Recording(B._native)
    monkeypatch.setattr(B, "_native", noting)
    native = _calls(t)
    assert set(noting.done) == set(NAMES) and len(noting.done) == 13
    without_native()
    plain = _calls(t)
    for name in native:
        for x, y in zip(_flat(native[name]), _flat(plain[name])):
            assert (x is None and y is None) or (x.dtype == y.dtype and torch.equal(x, y)), name


# what the native calls leave to the Python functions: still accepted
@pytest.mark.gpu
def test_other_forms_are_still_accepted():
    t = _inputs("cuda", torch.bfloat16)
    want = B.dodo_score(t["hidden"], t["w"], 1.0)
    wide = torch.zeros(300, 512, dtype=torch.bfloat16, device="cuda")
    wide[:, :256] = t["hidden"]
    assert torch.equal(B.dodo_score(wide[:, :256], t["w"], 1), want)  # rows further apart, a whole number as the bias
    sub = t["hidden"].as_subclass(type("Sub", (torch.Tensor,), {}))
    assert torch.equal(B.dodo_score(sub, t["w"], 1.0).as_subclass(torch.Tensor), want)


def _refused(device):
    t = _inputs(device, torch.bfloat16)
    f32 = t["w"].float()
    i = torch.zeros(30, dtype=torch.int32, device=device)
    s = torch.zeros(300, device=device)
    a = (t["Kl"], t["Vl"], t["cu_q"], t["cu_k"], t["cu_l"], 20, 20, 35)
    return [lambda: B.dodo_score(t["hidden"], f32), lambda: B.dodo_score(t["hidden"].half(), t["w"].half()),
            lambda: B.dodo_score(t["hidden"].t(), t["w"]), lambda: B.dodo_score(t["hidden"], t["w"], 0.0, torch.empty(299, device=device)),
            lambda: B.dodo_select_topk(s.double(), t["cu_s"], t["cu_k"], 200, 20, 30), lambda: B.dodo_select_topk(s, t["cu_s"].long(), t["cu_k"], 200, 20, 30),
            lambda: B.dodo_select_topk(s, t["cu_s"], t["cu_k"], -1, 20, 30), lambda: B.dodo_gather_nuggets(t["K"], t["V"][:200], i, t["cu_s"], t["cu_k"], 30),
            lambda: B.dodo_gather_nuggets(t["K"], t["V"], i, t["cu_s"], t["cu_k"], 30, 0, torch.empty_like(t["K"][:29])),
            lambda: B.dodo_nugget_attention(t["Q"].transpose(0, 1), t["K"], t["V"], *a), lambda: B.dodo_nugget_attention(t["Q"][0], t["K"], t["V"], *a),
            lambda: B.dodo_nugget_attention(t["Q"], t["K"], t["V"], *a, float("nan")), lambda: B.dodo_nugget_attention(t["Q"], t["K"], t["V"], *a, 0.1, 7),
            lambda: B.dodo_nugget_attention_indexed(t["Q"], t["K"], t["V"], i, t["cu_s"], *a, 5),
            lambda: B.dodo_stream_append(t["s2"], t["lam"], t["rows"], t["rows"], t["counts"], t["cacheK"][:1], t["cacheV"]),
            lambda: B.dodo_score_mlp(t["hidden"], t["W1"][:, :128], t["b1"], t["w"]), lambda: B.dodo_score_mlp(t["hidden"], t["W1"], t["b1"], t["w"], 0.0, 9)]


def _errors(calls):
    out = []
    for f in calls:
        with pytest.raises(Exception) as e:
            f()
        out.append((type(e.value), str(e.value)))
    return out


@pytest.mark.gpu
def test_refusals_are_the_same_on_the_gpu(without_native):
    native = _errors(_refused("cuda"))
    without_native()
    assert _errors(_refused("cuda")) == native


def test_host_tensors_are_declined(without_native):
    calls = _refused("cpu")[:1] + [lambda: B.dodo_score(torch.zeros(2, 4), torch.zeros(4)),
                                   lambda: B.dodo_select_topk(torch.zeros(4), torch.zeros(2, dtype=torch.int32), torch.zeros(2, dtype=torch.int32), 4, 1, 1)]
    native = _errors(calls)
    without_native()
    assert _errors(calls) == native
    assert all(kind is ValueError for kind, _ in native)


# Threads with streams of their own, whose calls give up the interpreter lock where they allocate and where they launch
@pytest.mark.gpu
def test_calls_from_several_threads():
    t = _inputs("cuda", torch.bfloat16)
    want = _calls(t)
    torch.cuda.synchronize()
    wrong = []

    def work():
        with torch.cuda.stream(torch.cuda.Stream()):
            for _ in range(20):
                got = _calls(t)
                torch.cuda.current_stream().synchronize()
                wrong.extend(n for n in want for x, y in zip(_flat(got[n]), _flat(want[n])) if x is not None and not torch.equal(x, y))
    threads = [threading.Thread(target=work) for _ in range(4)]
    for th in threads:
        th.start()
    for th in threads:
        th.join()
    assert not wrong


# The calls of the autoregressive objective and of training, in the forms that programs use: the native call does them, with the
# results of the one through ctypes, and what it declines the Python function refuses or takes as before.
@pytest.mark.gpu
@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
def test_training_calls_as_through_ctypes(dtype, monkeypatch):
    t = _inputs("cuda", dtype)
    names = ("threshold_from_sample", "select_threshold", "segment_plan", "nugget_attention_segments", "ste_score_grad")
    real = B._native
    done = []

    def noting(name):
        def call(*a):
            r = getattr(real, name)(*a)
            if r is not None:
                done.append(name)
            return r
        return call

    def calls():
        out = {}
        s = B.dodo_score(t["hidden"], t["w"])
        lam = out["lambda"] = B.dodo_threshold_from_sample(s, 1, 10)
        mine = torch.empty(1, device=s.device)
        assert B.dodo_threshold_from_sample(s, 1, 10, out=mine) is mine and torch.equal(mine, lam)
        counts, cu_k, idx = out["selection"] = B.dodo_select_threshold(s, t["cu_s"], lam)
        total = int(cu_k[-1])
        assert counts.shape == (2,) and cu_k.shape == (3,) and idx.shape == (300,)
        out["selection"] = (counts, cu_k, idx[:total])
        kn, vn = B.dodo_gather_nuggets(t["K"], t["V"], idx, t["cu_s"], cu_k, total)
        plan = out["plan"] = B.dodo_segment_plan(idx, t["cu_s"], cu_k, 32, 7, 11)
        q = t["K"].contiguous()
        O = torch.empty_like(q)
        got = out["segments"] = B.dodo_nugget_attention_segments(q, kn, vn, t["K"], t["V"], *plan[:5], 32, total, 39, 0.2, O=O, want_lse=True)
        assert got[0] is O
        a = (t["Kl"], t["Vl"], t["cu_q"], cu_k, t["cu_l"], 20, total, 35)
        O, lse = B.dodo_nugget_attention(t["Q"], kn, vn, *a, want_lse=True)
        b = (t["Q"], kn, vn, t["Q"], O, lse, t["cu_q"], cu_k, 20, total)
        grad = out["grad"] = B.dodo_ste_score_grad(*b)
        twice = grad.clone()
        assert B.dodo_ste_score_grad(*b, grad=twice, accumulate=True) is twice
        out["grad twice"] = twice
        with pytest.raises((AssertionError, ValueError)):
            B.dodo_ste_score_grad(*b, accumulate=True)
        with pytest.raises((AssertionError, TypeError, ValueError)):
            B.dodo_ste_score_grad(t["Q"], kn, vn, t["Q"], O, lse.double(), t["cu_q"], cu_k, 20, total)
        with pytest.raises((AssertionError, ValueError)):
            B.dodo_select_threshold(s.double(), t["cu_s"], lam)
        with pytest.raises(B.DodoError):
            B.dodo_threshold_from_sample(s, 0, 10)
        return out

    monkeypatch.setattr(B, "_native", types.SimpleNamespace(**{n: getattr(real, n) for n in dir(real) if not n.startswith("_")}))
    for n in names:
        monkeypatch.setattr(B._native, n, noting(n))
    native = calls()
    assert set(done) == set(names) and len(done) == 7
    for n in names:
        monkeypatch.setattr(B._native, n, lambda *a: None)
    plain = calls()
    for name in native:
        for x, y in zip(_flat(native[name]), _flat(plain[name])):
            assert x.dtype == y.dtype and torch.equal(x, y), name

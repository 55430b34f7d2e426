"""The Python binding validates every tensor (dtype, exact shape, contiguity,
device) before anything reaches the C library, whose kernels index each
buffer by the shapes taken from q and k.  Runs on the CPU: a mismatched
tensor must raise ValueError naming it, and the library must not be called."""

import pytest

torch = pytest.importorskip("torch")
cowa = pytest.importorskip("paper_2609_32704_amd")


@pytest.fixture
def no_library(monkeypatch):
    def boom():
        raise AssertionError("the library was called")
    monkeypatch.setattr(cowa._abi, "lib", boom)
    import inspect
    for name in dir(cowa._abi):
        if name.startswith("cowa_") and inspect.isfunction(getattr(cowa._abi, name)):
            monkeypatch.setattr(cowa._abi, name, lambda *a, **k: boom())


B, HQ, HK, N, NK, D = 2, 4, 2, 64, 96, 64


def bf(*shape, dtype=torch.bfloat16):
    return torch.zeros(shape, dtype=dtype)


def fwd_args():
    return dict(q=bf(B, HQ, N, D), k=bf(B, HK, NK, D), v=bf(B, HK, NK, D))


@pytest.mark.parametrize("name,bad", [
    ("v", bf(B, HK, NK + 1, D)), ("v", bf(B, HK + 1, NK, D)), ("k", bf(B + 1, HK, NK, D)),
    ("k", bf(B, HK, NK, D + 8)), ("out", bf(B, HQ, N + 1, D)), ("lse", bf(B, HQ, N, dtype=torch.float32)[:, :, :-1]),
    ("lse", bf(B, HQ, N)), ("v", bf(B, HK, NK, D, dtype=torch.float32)),
])
def test_fwd_rejects_mismatched_tensors(no_library, name, bad):
    a = fwd_args()
    a[name] = bad
    with pytest.raises(ValueError, match=name):
        cowa.fwd(a["q"], a["k"], a["v"], 4, 16, 64, 64, out=a.get("out"), lse=a.get("lse"))


def test_fwd_rejects_host_tensors(no_library):
    a = fwd_args()
    with pytest.raises(ValueError, match="device"):
        cowa.fwd(a["q"], a["k"], a["v"], 4, 16, 64, 64)


def bwd_args():
    return dict(q=bf(B, HQ, N, D), k=bf(B, HK, NK, D), v=bf(B, HK, NK, D), o=bf(B, HQ, N, D),
                lse=bf(B, HQ, N, dtype=torch.float32), do=bf(B, HQ, N, D))


@pytest.mark.parametrize("name,bad", [
    ("v", bf(B, HK, NK - 1, D)), ("o", bf(B, HQ, N, D + 1)), ("do", bf(B, HQ - 1, N, D)),
    ("lse", bf(B, HQ, N + 1, dtype=torch.float32)), ("dq", bf(B, HQ, N - 1, D)), ("dk", bf(B, HK, N, D)),
    ("dv", bf(B, HQ, NK, D)), ("k", bf(B, HK, NK, D + 64)),
])
def test_bwd_rejects_mismatched_tensors(no_library, name, bad):
    a = bwd_args()
    a[name] = bad
    with pytest.raises(ValueError, match=name):
        cowa.bwd(a["q"], a["k"], a["v"], a["o"], a["lse"], a["do"], 4, 16, 64, 64, dq=a.get("dq"), dk=a.get("dk"),
                 dv=a.get("dv"))


def dec_args():
    return dict(q=bf(B, HQ, D), k_cache=bf(B, HK, NK, D), v_cache=bf(B, HK, NK, D),
                seqlens_k=torch.zeros(B, dtype=torch.int32))


@pytest.mark.parametrize("name,bad", [
    ("v_cache", bf(B, HK, NK + 1, D)), ("k_cache", bf(B + 1, HK, NK, D)), ("seqlens_k", torch.zeros(B + 1, dtype=torch.int32)),
    ("seqlens_k", torch.zeros(B, dtype=torch.int64)), ("out", bf(B, HQ, D + 1)), ("lse", bf(B, HQ + 1, dtype=torch.float32)),
])
def test_decode_rejects_mismatched_tensors(no_library, name, bad):
    a = dec_args()
    a[name] = bad
    with pytest.raises(ValueError, match=name):
        cowa.decode(a["q"], a["k_cache"], a["v_cache"], a["seqlens_k"], 4, 16, out=a.get("out"), lse=a.get("lse"))


def test_noncontiguous_rejected(no_library):
    a = fwd_args()
    k = bf(B, HK, D, NK).transpose(2, 3)
    with pytest.raises(ValueError, match="contiguous"):
        cowa.fwd(a["q"], k, a["v"], 4, 16, 64, 64)


class _FakeStream:
    def __init__(self, handle):
        self.cuda_stream = handle


@pytest.fixture
def fake_gpu(monkeypatch):
    """CPU tensors and a stand-in for torch's streams: logs the stream that is current
    at each allocation, the handle of each library call and each record_stream."""
    import contextlib
    log = {"now": 0, "alloc": [], "calls": [], "recorded": []}

    @contextlib.contextmanager
    def stream_ctx(st):
        before, log["now"] = log["now"], st.cuda_stream
        yield
        log["now"] = before

    def logged(fn):
        def make(*a, **kw):
            t = fn(*a, **{k: v for k, v in kw.items() if k != "device"})
            log["alloc"].append((t.data_ptr(), log["now"]))
            return t
        return make
    monkeypatch.setattr(torch.cuda, "current_device", lambda: 0)
    monkeypatch.setattr(torch.cuda, "current_stream", lambda device=None: _FakeStream(log["now"]))
    monkeypatch.setattr(torch.cuda, "ExternalStream", lambda handle, device=None: _FakeStream(handle))
    monkeypatch.setattr(torch.cuda, "stream", stream_ctx)
    monkeypatch.setattr(torch._C, "_cuda_getCurrentRawStream", lambda dev: log["now"], raising=False)
    monkeypatch.setattr(torch, "empty", logged(torch.empty))
    monkeypatch.setattr(torch, "empty_like", logged(torch.empty_like))
    monkeypatch.setattr(torch.Tensor, "record_stream",
                        lambda t, st: log["recorded"].append((t.data_ptr(), st.cuda_stream)))
    monkeypatch.setattr(cowa, "_validate", lambda specs: None)
    for name in ("cowa_schedule", "cowa_fwd", "cowa_bwd", "cowa_decode"):
        monkeypatch.setattr(cowa._abi, name, lambda *a, n=name: log["calls"].append((n, a[-1])))
    return log


def test_temporaries_belong_to_the_callers_stream(fake_gpu):
    """With a stream handle that is not the current one, everything a call allocates
    (tables, workspace, outputs) belongs to that stream, outputs are also kept for the
    current one, and a schedule handed in is kept for that stream."""
    lib_calls = fake_gpu["calls"]
    a, d = bwd_args(), dec_args()
    S = 4096
    sched = cowa.Schedule(cowa.make_params(B, N, NK, HQ, HK, D, 4, 16, 64, 64), "cpu")
    assert [s for _, s in fake_gpu["alloc"]] == [0] and lib_calls == [("cowa_schedule", 0)]
    runs = [lambda **kw: cowa.fwd(a["q"], a["k"], a["v"], 4, 16, 64, 64, **kw),
            lambda **kw: cowa.bwd(a["q"], a["k"], a["v"], a["o"], a["lse"], a["do"], 4, 16, 64, 64, **kw)]
    for run in runs + [lambda **kw: cowa.decode(d["q"], d["k_cache"], d["v_cache"], d["seqlens_k"], 4, 16, **kw)]:
        for kw in [{}] + ([{"schedule": sched}] if run in runs else []):
            for v in ("alloc", "calls", "recorded"):
                fake_gpu[v].clear()
            outs = run(stream=S, **kw)
            assert {s for _, s in fake_gpu["alloc"]} == {S}
            assert lib_calls and {h for _, h in lib_calls} == {S}
            for t in outs:
                assert (t.data_ptr(), 0) in fake_gpu["recorded"]
            assert not kw or (sched.buf.data_ptr(), S) in fake_gpu["recorded"]
            for v in ("alloc", "calls", "recorded"):
                fake_gpu[v].clear()
            run(stream=0, **kw)  # the current stream's own handle
            assert {s for _, s in fake_gpu["alloc"]} == {0} and not fake_gpu["recorded"]
    fake_gpu["alloc"].clear()
    cowa.Schedule(sched.params, "cpu", stream=S)
    assert [s for _, s in fake_gpu["alloc"]] == [S] and lib_calls[-1] == ("cowa_schedule", S)

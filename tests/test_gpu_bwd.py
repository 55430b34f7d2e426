"""Backward parity (cowa_bwd through the C ABI) against the fp64 oracle.

Two paths: the device forward's own O and LSE fed to the backward (the
training path), and the oracle's O and LSE (rounded to the kernel's input
types) fed to it, which isolates the backward.  Full gradients at the 8K
workload and odd shapes (the 32K and 128K workloads are sampled against
stored oracle values in test_gpu_sampled.py).  Outputs are poisoned with NaN
before each call.
"""

import numpy as np
import pytest

import inputs
from oracle import attention as ref
from gpu_util import need_gpu, log, to_dev, to_host, compare, torch

pytestmark = pytest.mark.gpu


def _bf16_of(x, dev):
    return torch.from_numpy(np.ascontiguousarray(x, dtype=np.float32)).to(dev).to(torch.bfloat16)


def _run_bwd(w, t, dev, o=None, lse=None, tile_q=None, tile_k=None):
    import paper_2609_32704_amd as cowa
    tq, tk = tile_q or w.tile, tile_k or w.tile
    q, k, v, do = (to_dev(t[n][0], dev) for n in ("q", "k", "v", "do"))
    p = cowa.make_params(w.batch, w.n_q, w.n_k, w.h_q, w.h_k, w.head_dim, w.w_sink, w.w_near, tq, tk, w.scale,
                         h_k_total=w.kv_total, h_k_offset=w.h_offset)
    sched = cowa.Schedule(p, dev)
    if o is None:
        o, lse = cowa.fwd(q, k, v, w.w_sink, w.w_near, tq, tk, w.scale, h_k_total=w.kv_total,
                          h_k_offset=w.h_offset, schedule=sched)
    dq = torch.full_like(q, float("nan"))
    dk = torch.full_like(k, float("nan"))
    dv = torch.full_like(v, float("nan"))
    cowa.bwd(q, k, v, o, lse, do, w.w_sink, w.w_near, tq, tk, w.scale, h_k_total=w.kv_total,
             h_k_offset=w.h_offset, schedule=sched, dq=dq, dk=dk, dv=dv)
    torch.cuda.synchronize()
    return dq, dk, dv


def _full_check(w, key=None, tile_q=None, tile_k=None, isolated=False):
    dev = need_gpu()
    log(f"bwd {w.name}: B={w.batch} n_q={w.n_q} n_k={w.n_k} h={w.h_q}/{w.h_k} d={w.head_dim} sink={w.w_sink} "
        f"near={w.w_near} tiles={tile_q or w.tile}x{tile_k or w.tile} isolated={isolated}")
    t = inputs.train_tensors(w, key=key)
    dq_r, dk_r, dv_r, o_r, l_r = ref.backward(t["q"][1], t["k"][1], t["v"][1], t["do"][1], w.w_sink, w.w_near,
                                              w.scale, h_total=w.kv_total, h_offset=w.h_offset)
    o = lse = None
    if isolated:
        o = _bf16_of(o_r, dev)
        lse = torch.from_numpy(l_r.astype(np.float32)).to(dev)
    dq, dk, dv = _run_bwd(w, t, dev, o, lse, tile_q, tile_k)
    compare("dQ", to_host(dq), dq_r)
    compare("dK", to_host(dk), dk_r)
    compare("dV", to_host(dv), dv_r)


def test_bwd_bf16_t8k():
    _full_check(inputs.WORKLOADS["bf16_t8k"])


def test_bwd_bf16_t8k_isolated():
    _full_check(inputs.WORKLOADS["bf16_t8k"], isolated=True)


ODD = [
    # name, batch, n_q, n_k, h_q, h_k, d, sink, near, tile_q, tile_k, h_total, h_offset
    ("ragged", 2, 333, 333, 4, 2, 128, 5, 40, 64, 64, 0, 0),
    ("chunked_prefill", 1, 200, 1111, 8, 2, 128, 16, 100, 128, 128, 0, 0),
    ("gqa8_d64", 1, 1000, 1000, 8, 1, 64, 3, 77, 128, 64, 0, 0),
    ("mha", 1, 700, 700, 3, 3, 128, 0, 50, 64, 128, 0, 0),
    ("tp_rank", 1, 2048, 2048, 4, 1, 128, 32, 256, 128, 128, 8, 5),
    ("dense", 1, 777, 777, 4, 2, 128, 0, 777, 128, 128, 0, 0),
    ("wide_windows", 1, 500, 500, 2, 2, 64, 400, 400, 64, 128, 0, 0),
    ("no_near", 1, 300, 300, 2, 2, 64, 0, 0, 64, 64, 0, 0),
    ("tiny", 1, 5, 9, 2, 1, 128, 1, 2, 64, 64, 0, 0),
    # four-wave dQ workgroups of 64-row query blocks (4 QO heads each)
    ("gqa4_tq64", 1, 900, 900, 8, 2, 128, 8, 200, 64, 128, 0, 0),
    ("gqa4_d64_t64", 1, 650, 650, 4, 1, 64, 16, 130, 64, 64, 0, 0),
    # the pipelined dQ pass (128-key blocks) at head dimension 64
    ("gqa2_d64_t128", 1, 600, 600, 4, 2, 64, 8, 150, 128, 128, 0, 0),
    ("gqa4_d64_tq64_t128", 1, 700, 700, 8, 2, 64, 8, 150, 64, 128, 0, 0),
    # a sink of three 128-key blocks, each split into parts in the dK/dV pass
    ("wide_sink", 1, 1500, 1500, 8, 2, 128, 300, 64, 128, 128, 0, 0),
]


@pytest.mark.parametrize("case", ODD, ids=[c[0] for c in ODD])
def test_bwd_odd_shapes(case):
    name, bsz, n_q, n_k, h_q, h_k, d, ws, wn, tq, tk, ht, ho = case
    w = inputs.custom("bwd_" + name, batch=bsz, n_q=n_q, n_k=n_k, h_q=h_q, h_k=h_k, head_dim=d, w_sink=ws,
                      w_near=wn, tile=tq, h_total=ht, h_offset=ho)
    _full_check(w, key=inputs.key_of("bwd", name), tile_q=tq, tile_k=tk)


@pytest.mark.parametrize("h_q,h_k,n_q,near", [(16, 16, 4173, 8300), (32, 16, 2049, 8300), (16, 4, 4100, 8300),
                                              (64, 16, 8200, 4200)])
def test_bwd_dq_long_rows_by_heads_per_workgroup(h_q, h_k, n_q, near):
    """dQ of rows long and many enough for the 64-row waves (128-key blocks from
    8192 visible keys on, 64-key blocks from 4096), with one, two and four QO heads
    per workgroup and a ragged last row tile, against the oracle on the first
    and last 100 rows (dQ of a row depends on that row's dO and O alone)."""
    dev = need_gpu()
    import paper_2609_32704_amd as cowa
    n_k, d, win = max(9001, n_q), 128, [(5, near, 100, 200)] * h_k
    key = inputs.key_of("long_dq", h_q, h_k)
    t = {n: inputs.normal_bf16((1, h, m, d), inputs.seed_sequence(key, n))
         for n, h, m in (("q", h_q, n_q), ("k", h_k, n_k), ("v", h_k, n_k), ("do", h_q, n_q))}
    q, k, v, do = (to_dev(t[n][0], dev) for n in ("q", "k", "v", "do"))
    o, lse = cowa.fwd(q, k, v, 0, 0, 128, 64, d ** -0.5, windows=win)
    dq, dk, dv = (torch.full_like(x, float("nan")) for x in (q, k, v))
    cowa.bwd(q, k, v, o, lse, do, 0, 0, 128, 64, d ** -0.5, dq=dq, dk=dk, dv=dv, windows=win)
    torch.cuda.synchronize()
    assert not any(torch.isnan(x).any().item() for x in (dq, dk, dv))
    for rows, keys in ((slice(0, 100), n_k - n_q + 100), (slice(n_q - 100, n_q), n_k)):
        dq_r = ref.backward(t["q"][1][:, :, rows], t["k"][1][:, :, :keys], t["v"][1][:, :, :keys],
                            t["do"][1][:, :, rows], 0, 0, d ** -0.5, windows=win)[0]
        compare("dQ", to_host(dq[:, :, rows]), dq_r)


def test_autograd_function_and_determinism():
    """cowa.attention (torch.autograd.Function over cowa_fwd / cowa_bwd):
    gradients of sum(O * dO) match the oracle, and a second forward and
    backward on the same inputs give bitwise the same O, LSE and gradients (the
    backward has no atomics)."""
    import paper_2609_32704_amd as cowa
    dev = need_gpu()
    w = inputs.custom("autograd", batch=2, n_q=700, n_k=900, h_q=8, h_k=2, head_dim=128, w_sink=16, w_near=128,
                      tile=128)
    t = inputs.train_tensors(w, key=inputs.key_of("autograd"))
    dq_r, dk_r, dv_r, o_r, _ = ref.backward(t["q"][1], t["k"][1], t["v"][1], t["do"][1], w.w_sink, w.w_near,
                                            w.scale)
    do = to_dev(t["do"][0], dev)
    runs = []
    for _ in range(2):
        q, k, v = (to_dev(t[n][0], dev).requires_grad_(True) for n in ("q", "k", "v"))
        o, lse = cowa.attention(q, k, v, w.w_sink, w.w_near, 128, 128, w.scale, return_lse=True)
        (o.float() * do.float()).sum().backward()
        torch.cuda.synchronize()
        runs.append((o.detach(), lse.detach(), q.grad, k.grad, v.grad))
    compare("O", to_host(runs[0][0]), o_r)
    compare("dQ", to_host(runs[0][2]), dq_r)
    compare("dK", to_host(runs[0][3]), dk_r)
    compare("dV", to_host(runs[0][4]), dv_r)
    for a, b, n in zip(runs[0], runs[1], ("O", "LSE", "dQ", "dK", "dV")):
        assert torch.equal(a, b), f"{n} differs between two identical runs"


def test_bwd_bitwise_deterministic_8k():
    """The backward at the 8K workload, run twice on the same inputs, gives
    bitwise equal dQ, dK and dV."""
    dev = need_gpu()
    w = inputs.WORKLOADS["bf16_t8k"]
    t = inputs.train_tensors(w, values=False)
    first = _run_bwd(w, t, dev)
    second = _run_bwd(w, t, dev)
    for a, b, n in zip(first, second, ("dQ", "dK", "dV")):
        assert torch.equal(a, b), f"{n} differs between two identical runs"


def test_bwd_reads_no_rows_past_the_sequence():
    """Regression: with 128-row QO blocks and n_q % 128 <= 64, the last block's
    second 64-row step lies wholly past n_q.  Its copies of Q and dO must read
    nothing (they once read past the end of the tensors).  Q and dO sit at the
    start of NaN-filled buffers here, so a row read past the last QO head's end
    would turn dK and dV into NaN; the reads stay inside those buffers."""
    import paper_2609_32704_amd as cowa
    dev = need_gpu()
    n, h_q, h_k, d, sink, near, tile = 3000, 4, 2, 128, 16, 256, 128
    assert 0 < n % tile <= 64
    t = {nm: inputs.normal_bf16(s, inputs.seed_sequence(inputs.key_of("past_end", n), nm))
         for nm, s in (("q", (1, h_q, n, d)), ("k", (1, h_k, n, d)), ("v", (1, h_k, n, d)), ("do", (1, h_q, n, d)))}
    k, v = to_dev(t["k"][0], dev), to_dev(t["v"][0], dev)

    def padded(bits):  # the tensor at the start of a buffer with 256 NaN rows behind it
        buf = torch.full(((h_q * n + 256) * d,), float("nan"), dtype=torch.bfloat16, device=dev)
        view = buf[:h_q * n * d].view(1, h_q, n, d)
        view.copy_(to_dev(bits, dev))
        return buf, view

    qbuf, q = padded(t["q"][0])
    dobuf, do = padded(t["do"][0])
    scale = d ** -0.5
    o, lse = cowa.fwd(q, k, v, sink, near, tile, tile, scale)
    dq, dk, dv = (torch.full_like(x, float("nan")) for x in (q, k, v))
    cowa.bwd(q, k, v, o, lse, do, sink, near, tile, tile, scale, dq=dq, dk=dk, dv=dv)
    torch.cuda.synchronize()
    dq_r, dk_r, dv_r, _, _ = ref.backward(t["q"][1], t["k"][1], t["v"][1], t["do"][1], sink, near, scale)
    compare("dQ", to_host(dq), dq_r)
    compare("dK", to_host(dk), dk_r)
    compare("dV", to_host(dv), dv_r)
    del qbuf, dobuf


@pytest.mark.parametrize("case", [
    # name, batch, n, h_q, h_k, d, sink, near, tile: the dK/dV pass with ordinary columns in
    # parts (few columns), its 128-key columns at their edges, and 64-key schedule tiles
    ("one_column", 1, 128, 4, 1, 128, 4, 64, 128), ("column_edge", 2, 129, 2, 2, 128, 0, 50, 64),
    ("parts", 1, 1000, 16, 4, 128, 16, 128, 64), ("parts_d64", 1, 1111, 8, 2, 64, 130, 200, 128),
    ("no_sink", 1, 900, 8, 1, 128, 0, 300, 128), ("no_near", 1, 500, 2, 1, 64, 20, 0, 64),
    ("many_columns", 3, 2300, 6, 6, 64, 3, 64, 128)], ids=lambda c: c[0])
def test_bwd_column_parts(case):
    name, bsz, n, h_q, h_k, d, ws, wn, tile = case
    w = inputs.custom("bwd_parts_" + name, batch=bsz, n_q=n, n_k=n, h_q=h_q, h_k=h_k, head_dim=d, w_sink=ws,
                      w_near=wn, tile=tile)
    _full_check(w, key=inputs.key_of("bwd_parts", name))


@pytest.mark.parametrize("ragged", [False, True])
def test_bwd_columns_past_the_order_table(ragged):
    """More columns than the order table lists (1024): the dK/dV pass takes them
    in clusters.  Values against torch's float64 autograd of the masked softmax on
    the first sequence (the pass has no state across sequences)."""
    dev = need_gpu()
    import paper_2609_32704_amd as cowa
    h, n, d, win = 64, 2113 if not ragged else 700, 64, [(5, 70, 30, 100)] * 64
    seqs = [n] if not ragged else [n, 1500]
    gen = torch.Generator(device=dev)
    gen.manual_seed(3)
    q, k, v, do = (torch.randn((h, sum(seqs), d), generator=gen, device=dev).to(torch.bfloat16) for _ in range(4))
    if ragged:
        cu = [0, n, sum(seqs)]
        o, lse = cowa.fwd_varlen(q, k, v, cu, cu, 0, 0, 64, 64, windows=win)
        dq, dk, dv = cowa.bwd_varlen(q, k, v, o, lse, do, cu, cu, 0, 0, 64, 64, windows=win)
    else:
        a = [x[None] for x in (q, k, v, do)]
        o, lse = cowa.fwd(*a[:3], 0, 0, 64, 64, windows=win)
        dq, dk, dv = (x[0] for x in cowa.bwd(*a[:3], o, lse, a[3], 0, 0, 64, 64, windows=win))
    torch.cuda.synchronize()
    pos = torch.arange(n, device=dev)
    delta = pos[:, None] - pos[None, :]
    seen = (delta >= 0) & ((delta < 70) | (pos[None, :] < 5) | ((delta >= 100) & (delta < 200)))
    for hh in (0, 17, 63):
        qf, kf, vf = (x[hh, :n].double().requires_grad_(True) for x in (q, k, v))
        s = (qf @ kf.t()) * d ** -0.5
        p = torch.softmax(s.masked_fill(~seen, float("-inf")), -1)
        ref_g = torch.autograd.grad(p @ vf, (qf, kf, vf), do[hh, :n].double())
        for name, got, want in zip(("dQ", "dK", "dV"), (dq, dk, dv), ref_g):
            compare(name, to_host(got[hh, :n]), want.cpu().numpy())


def test_autograd_checks_what_saved_tensor_hooks_return():
    """A saved-tensor hook that leaves the tensors on the host is refused before
    anything reaches the GPU."""
    import paper_2609_32704_amd as cowa
    dev = need_gpu()
    q, k, v = (torch.randn((1, 2, 200, 64), device=dev).to(torch.bfloat16).requires_grad_(True) for _ in range(3))
    with torch.autograd.graph.saved_tensors_hooks(lambda x: x.cpu(), lambda x: x):
        o = cowa.attention(q, k, v, 4, 32)
    with pytest.raises(ValueError, match="device tensor"):
        o.sum().backward()


def test_callers_stream_handle():
    """Every entry point on a stream handle other than the current stream's (a side
    stream, or the default stream while a side stream is current) gives the same bits."""
    import paper_2609_32704_amd as cowa
    dev = need_gpu()
    gen = torch.Generator(device=dev)
    gen.manual_seed(23)
    q, k, v, do = (torch.randn((1, h, 700, 128), generator=gen, device=dev).to(torch.bfloat16) for h in (8, 2, 2, 8))
    sl, q1 = torch.tensor([700], dtype=torch.int32, device=dev), q[:, :, -1].contiguous()
    p = cowa.make_params(1, 700, 700, 8, 2, 128, 16, 128, 64, 64)

    def run(stream):
        o, lse = cowa.fwd(q, k, v, 16, 128, 64, 64, stream=stream)
        sched = cowa.Schedule(p, dev, stream=stream)
        o2, _ = cowa.fwd(q, k, v, 16, 128, 64, 64, schedule=sched, stream=stream)
        del sched
        grads = cowa.bwd(q, k, v, o, lse, do, 16, 128, 64, 64, stream=stream)
        return (o, lse, o2) + grads + cowa.decode(q1, k, v, sl, 16, 128, stream=stream)
    want = run(None)
    torch.cuda.synchronize()
    side = torch.cuda.Stream()
    got = run(side.cuda_stream)
    with torch.cuda.stream(side):
        got0 = run(0)
    torch.cuda.synchronize()
    for x in (got, got0):
        assert all(torch.equal(a, b) for a, b in zip(x, want))

"""One rank's share of a KV-head split, and one sequence of a batch, equal the
corresponding slice of the whole, bit for bit.

Sec. 2.3 (global KV-head assignment): rank r of a tensor-parallel group owns KV
head r and the QO heads of its group, builds its windows from the global head
index (Eq. fwa_global_head), and needs nothing from the other ranks.  The
library takes the global index through h_k_offset / h_k_total, so the call
with h_k = 1, h_q = 4, h_k_offset = r, h_k_total = 8 on the slices of the
tensors must reproduce the all-heads call's O, LSE, dQ, dK and dV for those
heads exactly: every row and column is computed by the same steps in the same
order.  In the dK/dV pass that order includes the parts into which a column is
cut, which follow from one KV head of one sequence and the number of all heads,
whoever walks them (a workgroup per part, or per column where a batch has many).
The 131072-token case is the benchmark's full-size launch configuration at every
output element, without an oracle; the shorter ones are the sizes at which
columns are cut, taken one by one and, in a batch, one after the other.
"""

import pytest

from gpu_util import need_gpu, log, torch

pytestmark = pytest.mark.gpu

N, HQ, HK, D, SINK, NEAR, TILE = 131072, 32, 8, 128, 128, 4096, 128


def _run(q, k, v, do, h_k_total, h_k_offset):
    import paper_2609_32704_amd as cowa
    o, lse = cowa.fwd(q, k, v, SINK, NEAR, TILE, TILE, h_k_total=h_k_total, h_k_offset=h_k_offset)
    dq, dk, dv = cowa.bwd(q, k, v, o, lse, do, SINK, NEAR, TILE, TILE, h_k_total=h_k_total, h_k_offset=h_k_offset)
    return o, lse, dq, dk, dv


def test_rank_share_equals_all_heads_slice():
    dev = need_gpu()
    gen = torch.Generator(device=dev)
    gen.manual_seed(2609)

    def randn(shape):
        return torch.randn(shape, generator=gen, device=dev, dtype=torch.float32).to(torch.bfloat16)

    q, k, v, do = randn((1, HQ, N, D)), randn((1, HK, N, D)), randn((1, HK, N, D)), randn((1, HQ, N, D))
    log("all 8 KV heads at 131072 tokens")
    full = _run(q, k, v, do, HK, 0)
    torch.cuda.synchronize()
    g = HQ // HK
    for r in (0, 3, 7):
        log(f"rank {r} of 8: KV head {r}, QO heads {g * r}..{g * r + g - 1}")
        qs, ks, vs, dos = (x[:, a:b].contiguous() for x, a, b in ((q, g * r, g * r + g), (k, r, r + 1),
                                                                  (v, r, r + 1), (do, g * r, g * r + g)))
        part = _run(qs, ks, vs, dos, HK, r)
        torch.cuda.synchronize()
        for name, a, b, sl in (("O", part[0], full[0], slice(g * r, g * r + g)),
                               ("LSE", part[1], full[1], slice(g * r, g * r + g)),
                               ("dQ", part[2], full[2], slice(g * r, g * r + g)),
                               ("dK", part[3], full[3], slice(r, r + 1)),
                               ("dV", part[4], full[4], slice(r, r + 1))):
            ref = b[:, sl]
            same = torch.equal(a, ref)
            if not same:
                diff = (a.float() - ref.float()).abs().max().item()
                log(f"  {name}: max |diff| {diff:.3e}")
            assert same, f"rank {r}: {name} differs from the all-heads run"
        log(f"  rank {r}: O, LSE, dQ, dK, dV bitwise equal")


@pytest.mark.parametrize("n,batch,h_q,h_k,d,near", [
    # columns in parts: by a workgroup each alone, in a batch by a workgroup each (1000) or
    # by one per column (the next two); sink columns only (4096, 65536); d = 64
    (1000, 4, 32, 8, 128, 128), (1000, 10, 32, 8, 128, 128), (2048, 4, 32, 8, 128, 1024), (4096, 4, 32, 8, 128, 1024),
    (8192, 1, 32, 8, 128, 1024), (8192, 3, 8, 2, 128, 1024),
    (16384, 2, 32, 8, 128, 2048), (65536, 2, 32, 8, 128, 4096), (1500, 3, 16, 4, 64, 128), (1500, 104, 8, 2, 64, 128)])
def test_rank_and_batch_entry_equal_the_whole(n, batch, h_q, h_k, d, near):
    import paper_2609_32704_amd as cowa
    dev = need_gpu()
    gen = torch.Generator(device=dev)
    gen.manual_seed(7)
    q, k, v, do = (torch.randn((batch, h, n, d), generator=gen, device=dev).to(torch.bfloat16)
                   for h in (h_q, h_k, h_k, h_q))

    def run(x, h_k_offset):
        o, lse = cowa.fwd(*x[:3], 64, near, 128, 128, h_k_total=h_k, h_k_offset=h_k_offset)
        return (o, lse) + cowa.bwd(*x[:3], o, lse, x[3], 64, near, 128, 128, h_k_total=h_k, h_k_offset=h_k_offset)

    log(f"{batch} x {n} tokens, {h_q}/{h_k} heads, d={d}")
    names, g = ("O", "LSE", "dQ", "dK", "dV"), h_q // h_k
    whole = run((q, k, v, do), 0)
    for b in (0, batch - 1):
        alone = run([x[b:b + 1].contiguous() for x in (q, k, v, do)], 0)
        for name, x, y in zip(names, alone, whole):
            assert torch.equal(x, y[b:b + 1]), f"entry {b} of {batch}: {name} differs from the batch's"
        for r in (0, h_k - 1):
            part = run([x[b:b + 1, m * r:m * r + m].contiguous() for x, m in ((q, g), (k, 1), (v, 1), (do, g))], r)
            for name, x, y in zip(names, part, alone):
                m = 1 if name in ("dK", "dV") else g
                assert torch.equal(x, y[:, m * r:m * r + m]), f"rank {r}: {name} differs from all heads'"


@pytest.mark.parametrize("lens,h_q,h_k,d,near,tile,windows", [
    # sequences and heads that take different shapes of the forward and the dQ pass:
    # d = 128, rows of 8192 visible keys beside short ones; 4096 and many rows; one
    # head dense and the others narrow; d = 64 around 1024 visible keys
    ([(8200, 8200), (900, 900), (1, 70)], 8, 2, 128, 8192, 128, None),
    ([(300, 300), (32800, 32800), (0, 40)], 8, 2, 128, 4000, 64, None),
    ([(8300, 8300), (600, 1000)], 8, 4, 128, 512,
     128, [(16, 512, 0, 40), (16, 9000, 0, 0), (16, 512, 100, 300), (0, 64, 0, 0)]),
    ([(500, 500), (3000, 3000), (77, 2500), (64, 64)], 16, 4, 64, 512, 64, None)])
def test_packed_sequence_and_window_head_equal_alone(lens, h_q, h_k, d, near, tile, windows):
    import paper_2609_32704_amd as cowa
    dev = need_gpu()
    gen = torch.Generator(device=dev)
    gen.manual_seed(11)
    cq = [sum(a for a, _ in lens[:x]) for x in range(len(lens) + 1)]
    ck = [sum(b for _, b in lens[:x]) for x in range(len(lens) + 1)]
    q, k, v, do = (torch.randn((h, n, d), generator=gen, device=dev).to(torch.bfloat16)
                   for h, n in ((h_q, cq[-1]), (h_k, ck[-1]), (h_k, ck[-1]), (h_q, cq[-1])))

    def run(x, cq, ck, wins, h_k_offset):
        kw = dict(h_k_total=h_k, h_k_offset=h_k_offset, windows=wins)
        o, lse = cowa.fwd_varlen(*x[:3], cq, ck, 16, near, tile, tile, **kw)
        return (o, lse) + cowa.bwd_varlen(*x[:3], o, lse, x[3], cq, ck, 16, near, tile, tile, **kw)

    log(f"{lens}, {h_q}/{h_k} heads, d={d}, windows {windows}")
    names, g = ("O", "LSE", "dQ", "dK", "dV"), h_q // h_k
    whole = run((q, k, v, do), cq, ck, windows, 0)
    for b, (n_q, n_k) in enumerate(lens):
        if n_q == 0:
            continue
        sl = [slice(cq[b], cq[b + 1]), slice(ck[b], ck[b + 1])]
        alone = run([x[:, s].contiguous() for x, s in ((q, sl[0]), (k, sl[1]), (v, sl[1]), (do, sl[0]))],
                    [0, n_q], [0, n_k], windows, 0)
        for name, x, y in zip(names, alone, whole):
            assert torch.equal(x, y[:, sl[1 if name in ("dK", "dV") else 0]]), f"sequence {b}: {name} differs from the batch's"
    for r in range(h_k):
        part = run([x[m * r:m * r + m].contiguous() for x, m in ((q, g), (k, 1), (v, 1), (do, g))], cq, ck,
                   None if windows is None else windows[r:r + 1], r)
        for name, x, y in zip(names, part, whole):
            m = 1 if name in ("dK", "dV") else g
            assert torch.equal(x, y[m * r:m * r + m]), f"rank {r}: {name} differs from all heads'"


@pytest.mark.parametrize("lens,h_q,h_k,d,tile", [
    # float32: sequences and ranks on both sides of 256 and of 4096 (d = 128) row tiles
    # of all heads together; a batch of equal lengths
    ([512, 4000, 100, 1025], 4, 2, 64, 32), ([600, 2100, 17], 32, 8, 128, 64), ([500, 500, 500], 4, 2, 64, 32)])
def test_fp32_sequence_and_rank_equal_the_whole(lens, h_q, h_k, d, tile):
    import paper_2609_32704_amd as cowa
    dev = need_gpu()
    gen = torch.Generator(device=dev)
    gen.manual_seed(13)
    cu = [sum(lens[:x]) for x in range(len(lens) + 1)]
    q, k, v = (torch.randn((h, cu[-1], d), generator=gen, device=dev) for h in (h_q, h_k, h_k))
    g = h_q // h_k
    log(f"{lens} tokens, {h_q}/{h_k} heads, d={d}, float32")
    whole = cowa.fwd_varlen(q, k, v, cu, cu, 16, 64, tile, tile)
    for b, n in enumerate(lens):
        x = [t[:, cu[b]:cu[b + 1]].contiguous() for t in (q, k, v)]
        alone = cowa.fwd(*(t[None] for t in x), 16, 64, tile, tile)
        for name, a, w in zip(("O", "LSE"), alone, whole):
            assert torch.equal(a[0], w[:, cu[b]:cu[b + 1]]), f"sequence {b}: {name} differs from the batch's"
    if len(set(lens)) == 1:
        x = [t.reshape(t.shape[0], len(lens), lens[0], d).transpose(0, 1).contiguous() for t in (q, k, v)]
        for name, a, w in zip(("O", "LSE"), cowa.fwd(*x, 16, 64, tile, tile), whole):
            assert torch.equal(a.transpose(0, 1).reshape(w.shape), w), f"{name} of the fixed-length batch differs"
    for r in (0, h_k - 1):
        x = [t[m * r:m * r + m].contiguous() for t, m in ((q, g), (k, 1), (v, 1))]
        part = cowa.fwd_varlen(*x, cu, cu, 16, 64, tile, tile, h_k_total=h_k, h_k_offset=r)
        for name, a, w in zip(("O", "LSE"), part, whole):
            assert torch.equal(a, w[g * r:g * r + g]), f"rank {r}: {name} differs from all heads'"

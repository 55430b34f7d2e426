"""Forward parity (cowa_fwd through the C ABI) against the fp64 oracle.

Full outputs at the fp32 512-token and the bf16 8K workloads and at odd
shapes (the 32K and 128K workloads are sampled against stored oracle values
in test_gpu_sampled.py).  Outputs are poisoned with NaN before each call so unwritten elements
fail.
"""

import numpy as np
import pytest

import inputs
from oracle import attention as ref
from gpu_util import need_gpu, log, to_dev, to_host, compare, torch

pytestmark = pytest.mark.gpu


def _run_fwd(w, t, dev, tile_q=None, tile_k=None):
    import paper_2609_32704_amd as cowa
    q, k, v = (to_dev(t[n][0], dev) for n in ("q", "k", "v"))
    o = torch.full_like(q, float("nan"))
    lse = torch.full((w.batch, w.h_q, w.n_q), float("nan"), dtype=torch.float32, device=dev)
    cowa.fwd(q, k, v, w.w_sink, w.w_near, tile_q or w.tile, tile_k or w.tile, w.scale,
             h_k_total=w.kv_total, h_k_offset=w.h_offset, out=o, lse=lse)
    torch.cuda.synchronize()
    return o, lse


def _full_check(w, key=None, tile_q=None, tile_k=None):
    dev = need_gpu()
    log(f"fwd {w.name}: B={w.batch} n_q={w.n_q} n_k={w.n_k} h={w.h_q}/{w.h_k} d={w.head_dim} "
        f"sink={w.w_sink} near={w.w_near} tiles={tile_q or w.tile}x{tile_k or w.tile} {w.dtype}")
    t = inputs.train_tensors(w, which=("q", "k", "v"), key=key)
    o, lse = _run_fwd(w, t, dev, tile_q, tile_k)
    o_r, l_r = ref.forward(t["q"][1], t["k"][1], t["v"][1], w.w_sink, w.w_near, w.scale,
                           h_total=w.kv_total, h_offset=w.h_offset)
    compare("O", to_host(o), o_r, w.dtype)
    compare("LSE", to_host(lse), l_r, w.dtype)


def test_fwd_fp32_t512():
    _full_check(inputs.WORKLOADS["fwd_fp32_t512"])


def test_fwd_bf16_t8k():
    _full_check(inputs.WORKLOADS["bf16_t8k"])


ODD = [
    # name, batch, n_q, n_k, h_q, h_k, d, sink, near, tile_q, tile_k, dtype, h_total, h_offset
    ("tiny", 1, 1, 1, 1, 1, 64, 0, 1, 64, 64, "bf16", 0, 0),
    ("ragged", 2, 333, 333, 4, 2, 128, 5, 40, 64, 64, "bf16", 0, 0),
    ("chunked_prefill", 1, 200, 1111, 8, 2, 128, 16, 100, 128, 128, "bf16", 0, 0),
    ("gqa8", 1, 1000, 1000, 8, 1, 64, 3, 77, 128, 64, "bf16", 0, 0),
    ("mha", 1, 700, 700, 3, 3, 128, 0, 50, 64, 64, "bf16", 0, 0),
    ("tp_rank", 1, 2048, 2048, 4, 1, 128, 32, 256, 128, 128, "bf16", 8, 5),
    ("dense", 1, 777, 777, 4, 2, 128, 0, 777, 128, 128, "bf16", 0, 0),
    ("wide_windows", 1, 500, 500, 2, 2, 64, 400, 400, 64, 128, "bf16", 0, 0),
    ("no_near", 1, 300, 300, 2, 2, 64, 0, 0, 64, 64, "bf16", 0, 0),
    ("fp32_ragged", 1, 301, 450, 4, 2, 128, 7, 33, 64, 32, "fp32", 0, 0),
    ("fp32_d64", 2, 129, 129, 2, 1, 64, 2, 17, 128, 128, "fp32", 0, 0),
    ("fp32_tp", 1, 512, 512, 4, 2, 64, 16, 64, 32, 32, "fp32", 4, 2),
]


@pytest.mark.parametrize("case", ODD, ids=[c[0] for c in ODD])
def test_fwd_odd_shapes(case):
    name, bsz, n_q, n_k, h_q, h_k, d, ws, wn, tq, tk, dt, ht, ho = case
    w = inputs.custom("fwd_" + name, batch=bsz, n_q=n_q, n_k=n_k, h_q=h_q, h_k=h_k, head_dim=d, w_sink=ws,
                      w_near=wn, tile=tq, dtype=dt, h_total=ht, h_offset=ho)
    _full_check(w, key=inputs.key_of("fwd", name), tile_q=tq, tile_k=tk)


@pytest.mark.parametrize("case", [
    # name, batch, n_q, n_k, h_q, h_k, d, sink, near, tile: the float32 kernel's
    # 16-row tiles and 16-key chunks at their edges, both wave counts (the last two
    # have more than 256 row tiles), rows without keys, one key, every key
    ("one", 1, 1, 1, 1, 1, 64, 0, 1, 32), ("edge16", 1, 16, 16, 2, 1, 128, 1, 3, 32),
    ("edge17", 2, 17, 49, 4, 1, 64, 2, 16, 64), ("tail", 1, 130, 131, 3, 3, 128, 0, 33, 128),
    ("no_near", 1, 100, 100, 2, 2, 64, 0, 0, 32), ("dense", 1, 257, 300, 2, 1, 128, 0, 300, 64),
    ("grid_256", 1, 1024, 1024, 4, 2, 64, 16, 64, 32), ("grid_257", 1, 1025, 1025, 4, 2, 64, 16, 64, 32),
    ("many_tiles", 2, 700, 900, 8, 2, 128, 5, 100, 64), ("rows32", 1, 2100, 2100, 32, 4, 128, 5, 100, 64)], ids=lambda c: c[0])
def test_fwd_fp32_tiles(case):
    name, bsz, n_q, n_k, h_q, h_k, d, ws, wn, tile = case
    w = inputs.custom("fwd32_" + name, batch=bsz, n_q=n_q, n_k=n_k, h_q=h_q, h_k=h_k, head_dim=d, w_sink=ws,
                      w_near=wn, tile=tile, dtype="fp32")
    _full_check(w, key=inputs.key_of("fwd32", name))


@pytest.mark.parametrize("h_q,h_k,n_q", [(16, 16, 4173), (32, 16, 2049), (16, 4, 4100)])
def test_fwd_long_rows_by_heads_per_workgroup(h_q, h_k, n_q):
    """Rows of more than 8192 visible keys in a grid large enough for the 64-row
    waves, with one, two and four QO heads per workgroup (tiles of 256, 128 and 64
    rows, a ragged last one), against the oracle on the first and last 200 rows."""
    dev = need_gpu()
    import paper_2609_32704_amd as cowa
    n_k, d, win = 9001, 128, [(5, 8300, 100, 200)] * h_k
    seq = {n: inputs.seed_sequence(inputs.key_of("long_rows", h_q, h_k), n) for n in ("q", "k", "v")}
    qb, qv = inputs.normal_bf16((1, h_q, n_q, d), seq["q"])
    kb, kv = inputs.normal_bf16((1, h_k, n_k, d), seq["k"])
    vb, vv = inputs.normal_bf16((1, h_k, n_k, d), seq["v"])
    q, k, v = (to_dev(b, dev) for b in (qb, kb, vb))
    o = torch.full_like(q, float("nan"))
    lse = torch.full((1, h_q, n_q), float("nan"), dtype=torch.float32, device=dev)
    cowa.fwd(q, k, v, 0, 0, 64, 128, d ** -0.5, out=o, lse=lse, windows=win)
    torch.cuda.synchronize()
    assert not torch.isnan(o).any().item() and not torch.isnan(lse).any().item()
    for rows, keys in ((slice(0, 200), n_k - n_q + 200), (slice(n_q - 200, n_q), n_k)):
        o_r, l_r = ref.forward(qv[:, :, rows], kv[:, :, :keys], vv[:, :, :keys], 0, 0, d ** -0.5, windows=win)
        compare("O", to_host(o[:, :, rows]), o_r)
        compare("LSE", to_host(lse[:, :, rows]), l_r)


def test_fwd_deterministic():
    dev = need_gpu()
    w = inputs.custom("fwd_det", batch=1, n_q=2000, n_k=2000, h_q=8, h_k=2, head_dim=128, w_sink=16, w_near=256,
                      tile=128)
    t = inputs.train_tensors(w, which=("q", "k", "v"), key=inputs.key_of("det"))
    o1, l1 = _run_fwd(w, t, dev)
    o2, l2 = _run_fwd(w, t, dev)
    assert torch.equal(o1, o2) and torch.equal(l1, l2)


@pytest.mark.parametrize("lift,lse_min,d,tile", [(4.0, 60.0, 64, 128), (9.0, 130.0, 64, 128), (4.0, 60.0, 64, 64),
                                                 (9.0, 130.0, 64, 64), (3.0, 60.0, 128, 64), (3.0, 60.0, 128, 128),
                                                 (6.5, 90.0, 64, 128), (6.5, 90.0, 64, 64)])
def test_fwd_wide_score_range(lift, lse_min, d, tile):
    """Keys of the second 128-key block score far above the rest, so rows whose
    first processed block is another one pass the forward's starting exponent
    offset by a wide margin.  lift 4 (about 90 in log2 units): the offset moves
    at the end of that block and O, l and the pending P are rescaled once.
    lift 9 (about 200): P overflows within the block, and the row runs its
    second pass with the row maximum.  lift 6.5 (about 150): no overflow, but
    the rescale factor 2^(m_old - m) alone would underflow.  With 64-key blocks the pending P^T at a
    block end is the block's first chunk instead of its third.  The fp64 oracle
    has no offset at all."""
    dev = need_gpu()
    import paper_2609_32704_amd as cowa
    n, h_q, h_k = 512, 2, 1
    rng = np.random.default_rng(11)
    qf = (rng.standard_normal((1, h_q, n, d)) * 0.25 + 2.0).astype(np.float32)
    kf = (rng.standard_normal((1, h_k, n, d)) * 0.1).astype(np.float32)
    kf[:, :, 128:256, :] += lift
    vf = rng.standard_normal((1, h_k, n, d)).astype(np.float32)
    bits = [inputs.f32_to_bf16_bits(x) for x in (qf, kf, vf)]
    vals = [inputs.bf16_bits_to_f64(b) for b in bits]
    q, k, v = (to_dev(b, dev) for b in bits)
    scale = d ** -0.5
    o = torch.full_like(q, float("nan"))
    lse = torch.full((1, h_q, n), float("nan"), dtype=torch.float32, device=dev)
    cowa.fwd(q, k, v, 16, 512, tile, tile, scale, out=o, lse=lse)
    torch.cuda.synchronize()
    o_r, l_r = ref.forward(vals[0], vals[1], vals[2], 16, 512, scale)
    assert l_r.max() > lse_min  # the score range of the case
    compare("O", to_host(o), o_r)
    compare("LSE", to_host(lse), l_r)


@pytest.mark.parametrize("window", [(0, 20, 0, 0), (0, 0, 33, 20)])
@pytest.mark.parametrize("level", [-62.0, -67.0, -73.0, 40.0])
@pytest.mark.parametrize("d", [64, 128])
def test_fwd_rows_without_a_starting_offset(level, d, window):
    """Rows that meet no legal key among the first 32 of their tile's first block: a
    near window of 20 keys, whose rows take their offset from their own diagonal,
    and a window of the 20 keys at distance 33 to 52, whose rows see no key there
    either and start at offset 0.  Their scores lie near `level` (base 2), on both
    sides of the sum below which rows without an offset go to the tracked launch
    (2^-60) and, at 40, high enough that the offset moves at once."""
    dev = need_gpu()
    import paper_2609_32704_amd as cowa
    n, h_q, h_k = 400, 4, 1
    rng = np.random.default_rng(5)
    a = (abs(level) * np.log(2.0) * d ** 0.5 / d) ** 0.5  # d a^2 / sqrt(d) = |level| ln 2
    qf = (np.full((1, h_q, n, d), a) + 0.02 * rng.standard_normal((1, h_q, n, d))).astype(np.float32)
    kf = (np.sign(level) * np.full((1, h_k, n, d), a) + 0.02 * rng.standard_normal((1, h_k, n, d))).astype(np.float32)
    vf = rng.standard_normal((1, h_k, n, d)).astype(np.float32)
    bits = [inputs.f32_to_bf16_bits(x) for x in (qf, kf, vf)]
    vals = [inputs.bf16_bits_to_f64(b) for b in bits]
    q, k, v = (to_dev(b, dev) for b in bits)
    o = torch.full_like(q, float("nan"))
    lse = torch.full((1, h_q, n), float("nan"), dtype=torch.float32, device=dev)
    cowa.fwd(q, k, v, 0, 0, 128, 128, d ** -0.5, out=o, lse=lse, windows=[window])
    torch.cuda.synchronize()
    o_r, l_r = ref.forward(vals[0], vals[1], vals[2], 0, 0, d ** -0.5, windows=[window])
    compare("O", to_host(o), o_r)
    compare("LSE", to_host(lse), l_r)


@pytest.mark.parametrize("h_q,h_k,d", [(32, 32, 128), (32, 32, 64), (32, 16, 128)])
def test_fwd_first_rows_keep_an_offset_of_their_own(h_q, h_k, d):
    """The first rows of a sequence, whose tile (128 rows for one QO head per KV
    head, 64 for two) has no full block and starts at its last 64 keys: P is rounded
    to bf16 relative to the maximum over 32 keys that the row sees, among them the
    largest of its few, which so keeps its full weight.  A row without an offset
    of its own rounds that weight as well.  The kernel's error must be the one of
    that rounding, which the reference applies in float64: measured, they agree
    to 0.01 % (1 % allowed); without the offsets the error is 6 % larger for 128-row
    tiles."""
    dev = need_gpu()
    import paper_2609_32704_amd as cowa
    n, near = 256, 256
    key = inputs.key_of("first_rows", h_q, h_k, d)
    t = {x: inputs.normal_bf16((1, h, n, d), inputs.seed_sequence(key, x))
         for x, h in (("q", h_q), ("k", h_k), ("v", h_k))}
    q, k, v = (to_dev(t[x][0], dev) for x in ("q", "k", "v"))
    o, lse = cowa.fwd(q, k, v, 0, near, 128, 128)
    torch.cuda.synchronize()
    g = h_q // h_k
    rows = 128 // g  # of the first tile
    qv, kv, vv = (t[x][1][0].astype(np.float64) for x in ("q", "k", "v"))
    err = err_ref = 0.0
    for h in range(h_q):
        s = qv[h, :rows] @ kv[h // g, :rows].T * d ** -0.5
        seen = np.tri(rows, dtype=bool)
        s[~seen] = -np.inf
        p = np.exp(s - s.max(1, keepdims=True))
        exact = p @ vv[h // g, :rows] / p.sum(1, keepdims=True)
        # the 32 keys of a row's offset: those of the tile's last block where the
        # row sees one of them, else those of its own 32-row tile
        first = rows - 64
        own = np.array([first if r >= first else r // 32 * 32 for r in range(rows)])
        m = np.array([s[r, own[r]:own[r] + 32].max() for r in range(rows)])
        pr = _round_bf16(np.where(seen, np.exp(s - m[:, None]), 0.0))
        ref_o = _round_bf16(pr @ vv[h // g, :rows] / pr.sum(1, keepdims=True))
        got = to_host(o[0, h, :rows])
        err += ((got - exact) ** 2).sum()
        err_ref += ((ref_o - exact) ** 2).sum()
    log(f"first rows {h_q}/{h_k} d={d}: error / error of the rounding {np.sqrt(err / err_ref):.5f}")
    assert np.sqrt(err) <= 1.01 * np.sqrt(err_ref)


def _round_bf16(x):
    return torch.from_numpy(np.ascontiguousarray(x)).to(torch.bfloat16).double().numpy()


@pytest.mark.parametrize("d,n_q,n_k,tile", [(64, 1, 1, 32), (64, 33, 70, 32), (128, 100, 100, 64), (128, 5, 1003, 128)])
def test_fwd_fp32_infinite_last_value(d, n_q, n_k, tile):
    """An infinite V element of the last key makes that element of the last row's O
    infinite and changes nothing else of it: key positions past the end must not
    count it with weight 0.  (Earlier rows may share a chunk with the key.)"""
    import paper_2609_32704_amd as cowa
    dev = need_gpu()
    gen = torch.Generator(device=dev)
    gen.manual_seed(17)
    q, k, v = (torch.randn((1, h, n, d), generator=gen, device=dev) for h, n in ((4, n_q), (2, n_k), (2, n_k)))
    log(f"fp32 d={d} {n_q} x {n_k}")
    o, lse = cowa.fwd(q, k, v, 0, n_k, tile, tile)
    v[:, :, -1, 7] = float("-inf")
    o2, lse2 = cowa.fwd(q, k, v, 0, n_k, tile, tile)
    o[:, :, -1, 7] = float("-inf")
    assert torch.equal(o2[:, :, -1], o[:, :, -1]) and torch.equal(lse2, lse)
    keep = [x for x in range(d) if x != 7]
    assert torch.equal(o2[..., keep], o[..., keep])

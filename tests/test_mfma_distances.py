"""Distances around the matrix products that the forward and the dQ pass write as
assembly (csrc/fwd_bf16.hip, csrc/dq_bf16.hip).  The compiler inserts no wait states
for those, so the kernels' schedule has to keep them; this reads the assembly of the
two files as built here and, over every path of every kernel, checks that

* a result is touched by anything but the next product of its chain (the same
  registers as accumulator input) no earlier than 12 wait states after a product of 8
  passes (32x32x16), 8 after one of 4 (16x16x32), products occupying the matrix pipe
  for their passes;
* no operand of a product was written by a vector instruction less than 2 wait states
  before it.

A wait state is one issue slot (4 cycles).  The second test plants mistakes in a
small listing."""

import os
import re
import subprocess

import pytest

from conftest import ROOT

HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
PASSES = {"v_mfma_f32_32x32x16_bf16": 8, "v_mfma_f32_16x16x32_bf16": 4}
READ_AFTER = 4          # wait states past a product's passes before its result is touched
OPERAND = 2             # wait states from a vector write to the product that reads it
REG = re.compile(r"\b([va])(?:\[(\d+):(\d+)\]|(\d+)\b)")


def _regs(text):
    out = set()
    for kind, lo, hi, one in REG.findall(text):
        out.update((kind, n) for n in (range(int(lo), int(hi) + 1) if lo else (int(one),)))
    return out


def _parse(lines):
    """Blocks [(instructions, successors)] of one kernel; an instruction is
    (line, opcode, [operand texts])."""
    blocks, labels, cur = [], {}, []

    def close(succ):
        nonlocal cur
        blocks.append((cur, succ))
        cur = []
    for no, raw in lines:
        s = raw.split(";")[0].strip()
        if not s:
            continue
        if s.endswith(":"):
            if cur:
                close([len(blocks) + 1])
            labels[s[:-1]] = len(blocks)
            continue
        if s.startswith("."):
            continue
        op, _, rest = s.partition(" ") if " " in s else s.partition("\t")
        op, args = op.strip(), [a.strip() for a in re.split(r",\s*(?![^\[]*\])", rest.strip())] if rest.strip() else []
        cur.append((no, op, args))
        if op == "s_branch":
            close([args[0]])
        elif op.startswith("s_cbranch"):
            close([args[0], len(blocks) + 1])
        elif op == "s_endpgm":
            close([])
    if cur:
        close([])
    return [(ins, [labels[x] if isinstance(x, str) else x for x in succ if x in labels or x < len(blocks)]
             if succ else []) for ins, succ in blocks]


def _run(ins, state, found):
    """state: {reg: (until touched, chain) or ("op", until read by a product)}, pipe."""
    busy, written, pipe = dict(state[0]), dict(state[1]), state[2]
    now = 0
    for no, op, args in ins:
        if op == "s_nop":
            now += int(args[0]) + 1
            continue
        if op in PASSES:
            start = max(now, pipe)
            dst, a, b = _regs(args[0]), _regs(args[1]), _regs(args[2])
            c = _regs(args[3])
            for r in a | b | c:
                if written.get(r, -99) > start:
                    found.append((no, op, "operand written just before", r))
            for r in a | b | ((c | dst) if c != dst else set()):
                if r in busy and busy[r][0] > start:
                    found.append((no, op, "reads or overwrites a product in flight", r))
            if c == dst:  # the chain: the very same registers, written by the same kind of product
                for r in dst:
                    if r in busy and busy[r][0] > start and busy[r][1] != (op, frozenset(dst)):
                        found.append((no, op, "accumulates on another product in flight", r))
            pipe = start + PASSES[op]
            for r in dst:
                busy[r] = (start + PASSES[op] + READ_AFTER + 1, (op, frozenset(dst)))
                written.pop(r, None)
            now = start + 1
            continue
        touched = _regs(" ".join(args))
        for r in touched:
            if r in busy and busy[r][0] > now:
                found.append((no, op, "touches a product in flight", r))
        if op.startswith("v_") and args:
            for r in _regs(args[0]):
                written[r] = now + 1 + OPERAND
        now += 1
    busy = {r: (t - now, c) for r, (t, c) in busy.items() if t > now}
    written = {r: t - now for r, t in written.items() if t > now}
    return busy, written, max(0, pipe - now)


def hazards(lines):
    blocks = _parse(lines)
    entry = [None] * len(blocks)
    entry[0] = ({}, {}, 0)
    work, found = [0], []
    while work:
        x = work.pop()
        out = _run(blocks[x][0], entry[x], found)
        for y in blocks[x][1]:
            old = entry[y]
            if old is None:
                new = out
            else:  # the later of both for hazards; the earlier for the pipe, which only delays
                busy = dict(old[0])
                for r, v in out[0].items():
                    if r not in busy or v[0] > busy[r][0]:
                        busy[r] = v
                written = dict(old[1])
                for r, v in out[1].items():
                    written[r] = max(v, written.get(r, v))
                new = (busy, written, min(old[2], out[2]))
            if new != old:
                entry[y] = new
                work.append(y)
    return sorted(set(found)), sum(op in PASSES for ins, _ in blocks for _, op, _ in ins)


def kernels(text):
    """{name: [(line number, text)]} of the functions of an assembly file."""
    out, name = {}, None
    for no, line in enumerate(text.splitlines(), 1):
        m = re.match(r"^(_Z\w+):", line)
        if m:
            name = m.group(1)
            out[name] = []
        elif line.startswith(".Lfunc_end"):
            name = None
        elif name:
            out[name].append((no, line))
    return out


@pytest.mark.parametrize("source", ["fwd_bf16.hip", "dq_bf16.hip"])
def test_products_keep_their_distances(source, tmp_path):
    if not os.path.exists(HIPCC):
        pytest.skip("hipcc not available")
    from paper_2609_32704_amd import build
    asm = str(tmp_path / "kernels.s")
    subprocess.run([HIPCC, *build.FLAGS, *build.FILE_FLAGS.get(source, []), "--cuda-device-only", "-S",
                    os.path.join(build.CSRC, source), "-o", asm], check=True, capture_output=True)
    with open(asm) as f:
        funcs = kernels(f.read())
    assert len(funcs) >= 5
    for name, lines in funcs.items():
        found, products = hazards(lines)
        assert products > 50, (name, products)
        assert not found, (name, len(found), found[:10])


M = "v_mfma_f32_32x32x16_bf16 v[0:15], v[16:19], a[0:3], "


@pytest.mark.parametrize("listing,bad", [
    ([M + "0", M + "v[0:15]", "s_nop 7", "s_nop 4", "v_mov_b32 v20, v3"], False),
    ([M + "0", "s_nop 7", "s_nop 2", "v_mov_b32 v20, v3"], True),          # 11 wait states
    ([M + "0", "s_nop 7", "s_nop 3", "v_mov_b32 v20, v3"], False),         # 12
    ([M + "0", "v_mfma_f32_32x32x16_bf16 a[16:31], v[20:23], v[24:27], a[16:31]",
      "s_nop 3", "v_exp_f32 v20, v3"], False),                             # one product between: 9 + 4
    ([M + "0", "ds_read_b128 v[12:15], v40", "s_nop 7", "s_nop 7"], True),  # a load over a result
    ([M + "0", "v_mfma_f32_32x32x16_bf16 v[8:23], v[24:27], a[0:3], 0"], True),
    (["v_mov_b32 v16, 0", M + "0"], True), (["v_mov_b32 v16, 0", "s_nop 1", M + "0"], False),
    (["v_accvgpr_write_b32 a2, v60", "s_nop 0", M + "0"], True),
    ([".LBB0_1:", "v_mov_b32 v20, v3", M + "0", "s_cbranch_scc1 .LBB0_1", "s_endpgm"], True)])  # around a loop
def test_planted_mistakes_are_found(listing, bad):
    found, _ = hazards(list(enumerate(listing)))
    assert bool(found) == bad, found

"""Wait states around the inline assembly of the kernels, read off the code that the compiler makes of it (no GPU).

The compiler keeps the wait states that gfx950 leaves to software between instructions of its own, but does not look into an asm
block, neither at what the block reads nor at what it leaves behind.  Whether an operand was written right in front of the block (a scalar
that was spilled to a lane of a vector register comes back by v_readlane) is up to register allocation, so the sources alone
cannot show it: each file whose asm blocks hold instructions is compiled with the build's own flags and every block is followed
backwards and forwards over all paths.

Rules (wait states: instructions in between, s_nop n counting n + 1):
  a scalar register written by a vector instruction: 2 before a vector instruction reads it, 5 before a memory address does
  m0: 1 from a scalar write to a load that goes to LDS
  a vector register written by a vector instruction: 2 before a matrix product reads it, 1 more after exp, log, rcp, sqrt
  the result of a 32 x 32 x 16 product (8 passes): 12 before anything else touches it, except the product that adds to all of it
"""
import os
import re
import subprocess

import pytest

from paper_2604_04215_amd import build

LOOK = 12                  # the longest of the rules above
TRANS = ("v_exp_", "v_log_", "v_rcp_", "v_rsq_", "v_sqrt_", "v_sin_", "v_cos_")
# instructions whose first operand is read, not written
NO_DST = ("ds_write", "global_store", "scratch_store", "buffer_store", "flat_store", "s_cmp", "s_bitcmp", "s_waitcnt", "s_nop", "s_barrier", "s_cbranch",
          "s_branch", "s_endpgm", "s_setprio", "s_sleep", "global_load_lds")


def regs(text):
    """Register names ('v7', 'a7', 's7', 'm0', 'vcc') in an operand list."""
    out = set()
    for m in re.finditer(r"\b([vas])\[(\d+):(\d+)\]|\b([vas])(\d+)\b|\b(m0|vcc)\b|\b(vcc)_(?:lo|hi)\b", text):
        if m[1]:
            out |= {f"{m[1]}{k}" for k in range(int(m[2]), int(m[3]) + 1)}
        elif m[4]:
            out.add(m[4] + m[5])
        else:
            out.add(m[6] or m[7])
    return out


class Ins:
    def __init__(self, text, asm):
        self.text, self.asm = text, asm
        self.op, _, rest = text.partition(" ")
        ops = [x.strip() for x in re.split(r",(?![^\[]*\])", rest)] if rest else []
        self.ops = ops
        n_dst = 0 if self.op.startswith(NO_DST) else 1
        if n_dst and len(ops) > 1 and re.match(r"v_(add|sub|subrev)c?_co_|v_div_scale|v_mad_[iu]64|s_\w*saveexec", self.op):
            n_dst = 1 if self.op.startswith("s_") else 2
        self.dst = set().union(*(regs(x) for x in ops[:n_dst])) if ops else set()
        self.src = set().union(*(regs(x) for x in ops[n_dst:])) if ops else set()
        if self.op == "v_swap_b32":
            self.dst = self.src = regs(rest)
        if self.op.startswith("global_load_lds"):
            self.src.add("m0")
        self.states = int(ops[0], 0) + 1 if self.op == "s_nop" else 1
        self.mfma = self.op.startswith(("v_mfma", "v_smfmac"))
        self.valu = self.op.startswith("v_")
        self.mem = self.op.startswith(("global_", "scratch_", "buffer_", "flat_", "ds_"))


def functions(listing):
    """name -> (instructions, successors, predecessors), in the order of the listing."""
    for f in re.finditer(r"^(_ZN\w+):\s*; @.*?\n(.*?)^\.Lfunc_end", listing, re.S | re.M):
        ins, at, pending, asm = [], {}, [], False
        for line in f[2].split("\n"):
            x = line.strip()
            if x.startswith(";;#ASMSTART") or x.startswith(";;#ASMEND"):
                asm = x.startswith(";;#ASMSTART")
                continue
            x = x.split(";")[0].strip()
            if m := re.match(r"(\.LBB\w+):", x):
                pending.append(m[1])
            elif x and not x.startswith((".", "#")) and not x.endswith(":"):
                for p in pending:
                    at[p] = len(ins)
                pending = []
                ins.append(Ins(re.sub(r"\s+", " ", x), asm))
        succ = [[] for _ in ins]
        for k, i in enumerate(ins):
            if i.op.startswith(("s_branch", "s_cbranch")):
                succ[k].append(at[i.ops[0]])
            if i.op not in ("s_branch", "s_endpgm", "s_setpc_b64") and k + 1 < len(ins):
                succ[k].append(k + 1)
        pred = [[] for _ in ins]
        for k, ss in enumerate(succ):
            for s in ss:
                pred[s].append(k)
        yield f[1], ins, succ, pred


def reach(ins, step, start):
    """(instruction index, wait states in between) of everything within LOOK wait states of start, over all paths."""
    best, todo = {}, [(s, 0) for s in step[start]]
    while todo:
        k, st = todo.pop()
        if st >= LOOK or best.get(k, LOOK) <= st:
            continue
        best[k] = st
        todo += [(s, st + ins[k].states) for s in step[k]]
    return best.items()


def need(a, b):
    """Wait states that instruction b needs behind a, and the register they are for."""
    if (hit := a.dst & b.src) and a.valu and not a.mfma:
        scalar = {r for r in hit if r[0] == "s" or r == "vcc"}
        if scalar and b.mem:
            return 5, scalar
        if scalar and b.valu:
            return 2, scalar
        if b.mfma:
            return 2 + a.op.startswith(TRANS), hit
        if a.op.startswith(TRANS) and b.valu:
            return 1, hit
    if a.op.startswith("s_") and "m0" in a.dst and "m0" in b.src and b.mem:
        return 1, {"m0"}
    if a.mfma and (hit := a.dst & (b.src | b.dst)) and (b.valu or b.mem):
        whole = b.mfma and regs(b.ops[3]) == a.dst == b.dst and not a.dst & (regs(b.ops[1]) | regs(b.ops[2]))
        return (0 if whole else 12), hit
    return 0, set()


def violations(listing):
    out = []
    for name, ins, succ, pred in functions(listing):
        for k, i in enumerate(ins):
            if not i.asm:
                continue
            for pairs in ([(j, k, st) for j, st in reach(ins, pred, k)], [(k, j, st) for j, st in reach(ins, succ, k)]):
                for a, b, st in pairs:
                    n, r = need(ins[a], ins[b])
                    if st < n:
                        out.append(f"{name}: '{ins[a].text}' .. '{ins[b].text}': {sorted(r)[0]}, {st} of {n} wait states")
    return sorted(set(out))


def sources():
    """Files with an asm block that reads or writes a register."""
    for s in build.SOURCES + build.PEAKS_SOURCES:
        text = open(os.path.join(build.CSRC, s)).read()
        if re.search(r'asm volatile\("[a-z][^;]*?"[=+&]*[vas]"\s*\(', text):
            yield s


@pytest.mark.parametrize("source", list(sources()))
def test_wait_states(source, tmp_path):
    listing = tmp_path / "listing.s"
    subprocess.run([os.environ.get("HIPCC", "hipcc"), *build.FLAGS, *build.SOURCE_FLAGS.get(source, []), "--cuda-device-only", "-S", os.path.join(build.CSRC, source), "-o",
                    str(listing)], check=True, stdout=subprocess.DEVNULL, stderr=subprocess.STDOUT)
    text = listing.read_text()
    assert len(list(functions(text))) > 0 and any(i.asm and i.mem for _, ins, _, _ in functions(text) for i in ins)
    # (asm blocks write m0, which the compiler does not take as clobbered: nothing outside them may rely on it)
    assert not any("m0" in i.dst | i.src for _, ins, _, _ in functions(text) for i in ins if not i.asm)
    found = violations(text)
    assert not found, f"{len(found)} places:\n" + "\n".join(found[:20])


LINES = """_ZNtest:                    ; @_ZNtest
; %bb.0:
	{before}
	;;#ASMSTART
	{asm}
	;;#ASMEND
	{after}
	s_endpgm
.Lfunc_end0:
"""


@pytest.mark.parametrize("before,asm,after,n", [
    ("v_readlane_b32 s4, v255, 25", "s_mov_b32 m0, s3\n\tv_add_u32 v1, s4, v230", "", 1),
    ("v_readlane_b32 s4, v255, 25", "s_mov_b32 m0, s4\n\ts_nop 0\n\tv_add_u32 v1, s4, v230", "", 0),
    ("v_readfirstlane_b32 s5, v1", "s_mov_b32 m0, s3\n\ts_nop 2\n\tglobal_load_lds_dwordx4 v1, s[4:5]", "", 1),
    ("v_readfirstlane_b32 s5, v1", "s_mov_b32 m0, s3\n\ts_nop 3\n\tglobal_load_lds_dwordx4 v1, s[4:5]", "", 0),
    ("v_readfirstlane_b32 s5, v1", "s_mov_b32 m0, s3\n\ts_mov_b64 s[8:9], s[4:5]\n\tglobal_load_lds_dwordx4 v1, s[8:9]", "", 0),
    ("", "s_mov_b32 m0, s3\n\tglobal_load_lds_dwordx4 v1, s[4:5]", "", 1),
    ("v_mov_b32_e32 v9, v1\n\ts_nop 0", "v_mfma_f32_32x32x16_bf16 a[0:15], v[4:7], v[8:11], a[0:15]", "", 1),
    ("v_mov_b32_e32 v9, v1\n\ts_nop 1", "v_mfma_f32_32x32x16_bf16 a[0:15], v[4:7], v[8:11], a[0:15]", "", 0),
    ("v_exp_f32_e32 v9, v1\n\ts_nop 1", "v_mfma_f32_32x32x16_bf16 a[0:15], v[4:7], v[8:11], a[0:15]", "", 1),
    ("", "v_mfma_f32_32x32x16_bf16 v[16:31], v[4:7], v[8:11], 0", "s_nop 10\n\tv_mov_b32_e32 v1, v31", 1),
    ("", "v_mfma_f32_32x32x16_bf16 v[16:31], v[4:7], v[8:11], 0", "s_nop 11\n\tv_mov_b32_e32 v1, v31", 0),
    ("", "v_mfma_f32_32x32x16_bf16 v[16:31], v[4:7], v[8:11], 0", "v_mfma_f32_32x32x16_bf16 v[16:31], v[4:7], v[8:11], v[16:31]", 0),
    ("", "v_mfma_f32_32x32x16_bf16 v[16:31], v[4:7], v[8:11], 0", "v_mfma_f32_32x32x16_bf16 v[32:47], v[4:7], v[16:19], v[32:47]", 1),
    ("s_cbranch_scc0 .LBB0_2\n; %bb.1:\n\tv_readlane_b32 s4, v255, 25\n.LBB0_2:", "v_add_u32 v1, s4, v230", "", 1)])
def test_the_check_itself(before, asm, after, n):
    assert len(violations(LINES.format(before=before, asm=asm, after=after))) == n

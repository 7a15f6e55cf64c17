"""Wait states around the matrix instructions and row broadcasts of the built
library.

A matrix instruction written as assembly is not seen by the compiler's hazard
recognizer, so nothing but the source keeps the distances that the hardware
asks for.  This test disassembles the gfx950 code built here and follows every
path through it:

* an operand of a matrix instruction was written by a vector instruction at
  least two wait states before;
* the result of a matrix instruction is read or rewritten by another kind of
  instruction only when it is there: MFMA_RESULT, the distances that the compiler
  keeps for the same products through builtins;
* a register read through DPP was written at least two wait states before.

Every instruction is one wait state, s_nop N is N + 1."""

import os
import re
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
LIB = os.path.join(ROOT, "paper_1502_05366_amd", "librsvd.so")

VALU_TO_MFMA = 2
VALU_TO_DPP = 2
# wait states before the result is read by a vector instruction, read by a memory
# instruction, overwritten
MFMA_RESULT = (("v_mfma_f64_16x16x4", (19, 18, 11)), ("v_mfma_f32_16x16x4_f32", (10, 10, 10)),
               ("v_mfma_f32_16x16x32_bf16", (8, 8, 8)),
               ("v_mfma_f32_16x16x128_f8f6f4", (12, 12, 12)))
HORIZON = 20

REG = re.compile(r"\b([va])(?:\[(\d+):(\d+)\]|(\d+)\b)")
LINE = re.compile(r"^\s+([a-z]\S*)\s*(.*?)\s*// ([0-9A-F]{12}):.*?(?:<\S+\+0x([0-9a-f]+)>)?$")
HEAD = re.compile(r"^([0-9a-f]{16}) <(\S+)>:$")
DPP = re.compile(r"\b(quad_perm|row_\w+|wave_\w+)\b")


def tool(name):
    for d in ("/opt/rocm/llvm/bin", "/opt/rocm/lib/llvm/bin"):
        if os.path.exists(os.path.join(d, name)):
            return os.path.join(d, name)
    return shutil.which(name)


def regs(text):
    out = []
    for kind, lo, hi, one in REG.findall(text):
        a, b = (int(one), int(one)) if one else (int(lo), int(hi))
        out.extend((kind, i) for i in range(a, b + 1))
    return out


def split_operands(text):
    out, depth, cur = [], 0, ""
    for ch in text:
        depth += (ch == "[") - (ch == "]")
        if ch == "," and depth == 0:
            out.append(cur)
            cur = ""
        else:
            cur += ch
    return out + [cur] if cur.strip() else out


class Inst:
    __slots__ = ("op", "text", "addr", "target", "states", "kind", "need", "writes", "reads", "dpp")

    def __init__(self, op, args, addr, target):
        self.op, self.text, self.addr, self.target = op, args, addr, target
        self.states = int(args.split()[0], 0) + 1 if op == "s_nop" else 1
        self.kind = ("mfma" if op.startswith("v_mfma") else
                     "valu" if op.startswith("v_") else "other")
        self.need = 0
        if self.kind == "mfma":
            need = [n for p, n in MFMA_RESULT if op.startswith(p)]
            assert len(need) == 1, "no distance known for " + op
            self.need = need[0]
        ops = split_operands(args)
        nw = 0
        if self.kind != "other":
            nw = 2 if "swap" in op else 1
        self.writes = [r for o in ops[:nw] for r in regs(o)]
        self.reads = [r for o in ops[0 if nw == 2 or self.kind == "other" else 1:] for r in regs(o)]
        if "fmac" in op:                                   # (the addend)
            self.reads = self.reads + self.writes
        self.dpp = regs(ops[1]) if self.kind == "valu" and len(ops) > 1 and DPP.search(args) else []


def functions(asm):
    name, insts, base = None, [], 0
    for line in asm.splitlines():
        h = HEAD.match(line)
        if h:
            if name:
                yield name, insts
            base, name, insts = int(h.group(1), 16), h.group(2), []
            continue
        m = LINE.match(line)
        if m and name:
            t = base + int(m.group(4), 16) if m.group(4) else None
            insts.append(Inst(m.group(1), m.group(2), int(m.group(3), 16), t))
    if name:
        yield name, insts


def scan(insts):
    """Faults of one function: (rule, instruction, register, wait states, needed), the
    rule "operand" or "result"."""
    at = {x.addr: i for i, x in enumerate(insts)}
    leaders = {0} | {at[x.target] for x in insts if x.target in at}
    leaders |= {i + 1 for i, x in enumerate(insts)
                if x.op.startswith(("s_cbranch", "s_branch", "s_endpgm", "s_setpc"))}
    starts = sorted(i for i in leaders if i < len(insts))
    end = dict(zip(starts, starts[1:] + [len(insts)]))
    entry = {s: {} for s in starts}
    faults = {}
    work = [0]
    seen = set()
    while work:
        s = work.pop()
        seen.add(s)
        # (register, 'valu' or 'mfma') -> [wait states since it was written, needed (mfma)]
        state = dict(entry[s])
        last = None
        for i in range(s, end[s]):
            x = last = insts[i]
            wr = set(x.writes)
            for (r, k), (age, need) in state.items():
                if k == "mfma" and x.kind != "mfma" and (r in x.reads or r in wr):
                    n = need[2 if r not in x.reads else 0 if x.kind == "valu" else 1]
                    if age < n:
                        faults[(x.addr, r)] = ("result", x, r, age, n)
                if k == "valu" and x.kind == "mfma" and age < VALU_TO_MFMA and r in x.reads:
                    faults[(x.addr, r)] = ("operand", x, r, age, VALU_TO_MFMA)
                if k == "valu" and age < VALU_TO_DPP and r in x.dpp:
                    faults[(x.addr, r)] = ("operand", x, r, age, VALU_TO_DPP)
            nxt = {}
            for (r, k), (age, need) in state.items():
                if r not in wr and age + x.states < HORIZON:
                    nxt[(r, k)] = (age + x.states, need)
            if x.kind != "other":
                for r in x.writes:
                    nxt[(r, x.kind)] = (0, x.need)
            state = nxt
        succ = []
        if last is not None:
            if last.target in at:
                succ.append(at[last.target])
            if not last.op.startswith(("s_branch", "s_endpgm", "s_setpc")) and end[s] in entry:
                succ.append(end[s])
        for t in succ:
            changed = t not in seen
            for key, v in state.items():
                old = entry[t].get(key)
                if old is None or v[0] < old[0]:
                    entry[t][key] = v
                    changed = True
            if changed and t not in work:
                work.append(t)
    return list(faults.values())


@pytest.fixture(scope="module")
def faults(tmp_path_factory):
    """The faults of every function of the built library, a text for each."""
    objdump = tool("llvm-objdump")
    assert objdump, "llvm-objdump not found"
    if not os.path.exists(LIB):
        import __graft_entry__ as g
        g.build()
    d = tmp_path_factory.mktemp("code")
    so = shutil.copy(LIB, d / "librsvd.so")
    subprocess.run([objdump, "--offloading", str(so)], check=True, cwd=d, capture_output=True)
    objs = sorted(f for f in os.listdir(d) if f.endswith("gfx950"))
    out, nfun, nmfma = [], 0, 0
    for f in objs:
        asm = subprocess.run([objdump, "-d", "--mcpu=gfx950", str(d / f)], check=True,
                             capture_output=True, text=True).stdout
        for name, insts in functions(asm):
            nfun += 1
            nmfma += sum(x.kind == "mfma" for x in insts)
            out += [(rule, name, "%s +%x: %s %s: %s%d after %d of %d wait states"
                     % (name, x.addr, x.op, x.text, r[0], r[1], age, need))
                    for rule, x, r, age, need in scan(insts)]
    assert nfun > 100 and nmfma > 10000                    # (the library was read)
    return out


def test_scan_finds_short_distances():
    def one(*lines):
        asm = "0000000000000100 <f>:\n" + "".join(
            "\t%s // %012X: 00000000\n" % (t, 0x100 + 4 * i) for i, t in enumerate(lines))
        return [f[0] for f in scan(next(functions(asm))[1])]
    mf = "v_mfma_f32_16x16x4_f32 a[0:3], v1, v2, a[0:3]"
    assert one("v_mov_b32_e32 v1, 0", "s_nop 0", mf) == ["operand"]
    assert not one("v_mov_b32_e32 v1, 0", "s_nop 1", mf)
    assert not one("v_mov_b32_e32 v3, 0", mf)
    assert one("v_permlane32_swap_b32_e32 v0, v1", mf) == ["operand"]
    assert one(mf, "s_nop 8", "v_accvgpr_read_b32 v9, a3") == ["result"]
    assert not one(mf, "s_nop 9", "v_accvgpr_read_b32 v9, a3")
    assert one(mf, "v_accvgpr_write_b32 a2, v9") == ["result"]
    assert one(mf, "global_store_dwordx4 v[4:5], a[0:3], off") == ["result"] * 4
    assert not one(mf, mf)
    assert one("v_add_f64 v[2:3], v[2:3], v[2:3]",
               "v_fmac_f64_dpp v[0:1], -v[2:3], v[4:5] row_newbcast:3 row_mask:0xf bank_mask:0xf")


def test_scan_follows_branches():
    asm = """0000000000000100 <f>:
\tv_mfma_f32_16x16x4_f32 a[0:3], v1, v2, a[0:3] // 000000000100: 00000000
\ts_cbranch_scc1 4 // 000000000104: 00000000 <f+0x10>
\ts_nop 9 // 000000000108: 00000000
\ts_nop 0 // 00000000010C: 00000000
\tv_accvgpr_read_b32 v9, a3 // 000000000110: 00000000
\tv_mov_b32_e32 v1, 0 // 000000000114: 00000000
\ts_branch 65530 // 000000000118: 00000000 <f+0x0>
"""
    assert sorted(f[0] for f in scan(next(functions(asm))[1])) == ["operand", "result"]


def check(faults, rule, pick=lambda name: True):
    bad = [text for r, name, text in faults if r == rule and pick(name)]
    assert not bad, "%d short distances, first:\n%s" % (len(bad), "\n".join(bad[:12]))


def test_operands_are_written_in_time(faults):
    check(faults, "operand")


def test_results_are_there_in_time_fp32_fp64_passes(faults):
    check(faults, "result", lambda name: "gemmreg" in name)


def test_results_are_there_in_time(faults):
    check(faults, "result")

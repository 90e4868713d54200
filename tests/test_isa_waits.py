"""Wait states of the built code, on the CPU.  Some instructions may follow others only after a number of wait states
that the hardware does not enforce (the published tables of required no-ops; an instruction is one wait state,
s_nop N is N + 1).  The compiler keeps them between instructions that it knows, not around those that sit in inline
assembly: the LDS-DMA loads, the block-scaled MFMAs, the additions of another lane's value.  So the library as built is disassembled and every pair is
looked at, along every path that leads to the second instruction."""
import functools
import os
import re
import shutil
import subprocess

import pytest

OBJDUMP = next((p for p in ("/opt/rocm/llvm/bin/llvm-objdump", shutil.which("llvm-objdump")) if p and os.path.exists(p)), None)
pytestmark = pytest.mark.skipif(OBJDUMP is None, reason="needs llvm-objdump")

_REG = re.compile(r"^-?\|?([sva])(?:(\d+)|\[(\d+):(\d+)\])\|?$")


def registers(operand):
    m = _REG.match(operand)
    if m:
        lo, hi = (m[2], m[2]) if m[2] else (m[3], m[4])
        return {(m[1], i) for i in range(int(lo), int(hi) + 1)}
    return {(operand, 0)} if operand in ("m0", "vcc") else set()


class Instruction:
    def __init__(self, text):
        self.text = text
        self.op, _, rest = text.partition(" ")
        self.operands = [o.split()[0] if o.split() else "" for o in rest.split(",")]
        self.states = int(self.operands[0], 0) + 1 if self.op == "s_nop" else 1

    def is_mfma(self):
        return self.op.startswith("v_mfma")

    def is_valu(self):
        return self.op.startswith("v_") and not self.is_mfma()

    def is_vmem(self):
        return self.op.startswith(("global_", "buffer_", "flat_", "scratch_"))

    def written(self):
        regs = registers(self.operands[0])
        return regs | registers(self.operands[1]) if "swap" in self.op else regs

    def read(self):
        skip = 0 if self.is_vmem() and ("store" in self.op or "lds" in self.op) or "swap" in self.op else 1
        return set().union(*(registers(o) for o in self.operands[skip:]))


def parse(disassembly):
    """[(kernel, [Instruction], {index: indices that can come right before it})]"""
    kernels, name, start, instr, target = [], None, 0, [], []

    def flush():
        if name is None:
            return
        index = {a: i for i, (a, _, _) in enumerate(instr)}
        before = {}
        for i, (_, ins, jump) in enumerate(instr):
            if ins.op not in ("s_branch", "s_endpgm", "s_setpc_b64"):
                before.setdefault(i + 1, []).append(i)
            if jump is not None and jump in index:
                before.setdefault(index[jump], []).append(i)
        kernels.append((name, [ins for _, ins, _ in instr], before))

    for line in disassembly.splitlines():
        m = re.match(r"^([0-9a-f]+) <(\S+)>:", line)
        if m:
            flush()
            name, start, instr = m[2], int(m[1], 16), []
            continue
        m = re.match(r"^\s+(\S.*?)\s*// ([0-9A-F]+): [0-9A-F ]+(?:<\S+?\+0x([0-9a-f]+)>)?", line)
        if m and name is not None:
            ins = Instruction(re.sub(r"\s+", " ", m[1]))
            jump = start + int(m[3], 16) if m[3] and "branch" in ins.op else None
            instr.append((int(m[2], 16), ins, jump))
    flush()
    return kernels


@functools.lru_cache(maxsize=None)
def built_kernels():
    import tempfile
    import paper_2511_04214_amd as brq
    brq.lib()
    so = os.path.join(os.path.dirname(os.path.abspath(brq.__file__)), "libbrq.so")
    kernels = []
    with tempfile.TemporaryDirectory() as d:
        shutil.copy(so, os.path.join(d, "lib.so"))
        subprocess.check_call([OBJDUMP, "--offloading", "lib.so"], cwd=d, stdout=subprocess.DEVNULL)
        for f in sorted(os.listdir(d)):
            if f.endswith("gfx950") and os.path.getsize(os.path.join(d, f)):
                kernels += parse(subprocess.check_output([OBJDUMP, "-d", f], cwd=d, text=True))
    assert len(kernels) > 20, "the library's kernels were not found in it"
    return kernels


def violations(kernels, first, second, needed, regs=Instruction.read):
    """Pairs (an instruction `first` that writes a register, one `second` that uses it by `regs`) closer than `needed`."""
    found, looked = [], 0
    for name, ins, before in kernels:
        for i, b in enumerate(ins):
            if not second(b):
                continue
            looked += 1
            want = frozenset(regs(b))
            todo, seen = [(j, 0, want) for j in before.get(i, [])], set()
            while todo:
                j, states, left = todo.pop()
                if states >= needed or not left or (j, states, left) in seen:
                    continue
                seen.add((j, states, left))
                a = ins[j]
                wrote = a.written() & left
                if first(a) and wrote:
                    found.append("%s: %s -> %s after %d of %d wait states" % (name, a.text, b.text, states, needed))
                left -= wrote           # what wrote them before that is no longer what is used
                todo += [(p, states + a.states, left) for p in before.get(j, [])]
    return found, looked


def is_lds_dma(i):
    return i.is_vmem() and "load_lds" in i.op


def is_fp4_mfma(i):
    return i.op == "v_mfma_scale_f32_32x32x64_f8f6f4" and "cbsz:4 blgp:4" in i.text


def is_dpp(i):
    return i.is_valu() and re.search(r" (quad_perm:|row_)", i.text) is not None


PAIRS = {
    "M0 written, then an LDS-DMA load": (lambda i: i.op.startswith("s_"), is_lds_dma, 1, lambda i: {("m0", 0)}),
    "scalar register from the vector unit, then an address of a memory access": (Instruction.is_valu, Instruction.is_vmem, 5, lambda i: {r for r in i.read() if r[0] == "s"}),
    "vector register from the vector unit, then an MFMA": (Instruction.is_valu, Instruction.is_mfma, 2, Instruction.read),
    "vector register from the vector unit, then another lane's copy of it": (Instruction.is_valu, is_dpp, 2, lambda i: registers(i.operands[1])),
    # (8 passes: fp4 operands)
    "result of a block-scaled MFMA, then the vector unit": (is_fp4_mfma, Instruction.is_valu, 12, lambda i: i.read() | i.written()),
}


@pytest.mark.parametrize("pair", sorted(PAIRS))
def test_wait_states(pair):
    first, second, needed, regs = PAIRS[pair]
    found, looked = violations(built_kernels(), first, second, needed, regs)
    assert looked > 100, "nothing to look at"
    assert not found, "%d pairs, the first: %s" % (len(found), found[0])


def test_the_check_sees_a_missing_wait():
    listing = """
0000000000001000 <k>:
	s_add_u32 m0, s25, 0                                       // 000000001000: 807C8019
	%s
	global_load_lds_dwordx4 v120, s[22:23]                     // 000000001008: DDF48000 00160078
	v_readfirstlane_b32 s22, v3                                // 000000001010: 7E2C0503
	s_cbranch_scc1 65531                                       // 000000001014: BF85FFFB <k+0x4>
	s_endpgm                                                   // 000000001018: BF810000
"""
    for nop, n in (("s_mov_b32 s1, s2                     // 000000001004: BE810002", 0),
                   ("s_nop 0                              // 000000001004: BF800000", 0), ("", 1)):
        kernels = parse(listing % nop)
        first, second, needed, regs = PAIRS["M0 written, then an LDS-DMA load"]
        assert len(violations(kernels, first, second, needed, regs)[0]) == n
    # along the loop's back edge: the load's base was written 2 wait states before
    first, second, needed, regs = PAIRS["scalar register from the vector unit, then an address of a memory access"]
    kernels = parse(listing % "s_nop 0                              // 000000001004: BF800000")
    assert len(violations(kernels, first, second, needed, regs)[0]) == 1
    assert not violations(kernels, first, second, 2, regs)[0]

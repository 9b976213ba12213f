"""The main loop of the 256x128 GEMM tile, run on the CPU as it is committed (gemm16_asm.hpp): its scalar instructions, load addresses and waits, with every
load arriving as late as the waits allow.  Every MFMA must find the fragments of the stage it is at, and no load may leave the K range or land in a unit
that is still being read.  One wavefront is run for all four, which load a quarter of every unit each: what it waited for is there for the others, and what it has read is free for
their loads, from the next barrier on.  No GPU needed."""
import os
import re

import pytest

from test_gemm16_registers import device_asm  # noqa: F401

HPP = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2507_03220_amd", "csrc", "gemm16_asm.hpp")
MB, NB, UNIT_A, UNIT_B = 8, 4, 32768, 16384
M32, M64 = (1 << 32) - 1, (1 << 64) - 1


def _lines(name):
    body = re.search(r"#define %s \\\n(.*?)\n    \"\"" % name, open(HPP).read(), re.S).group(1)
    return [re.match(r'\s*"(.*)\\n\\t" \\', l).group(1) for l in body.splitlines()]


class Loop:
    def __init__(self, nn, KF, first, stride):
        self.KF, self.stride, self.nn = KF, stride, nn
        self.A0, self.B0 = (1 << 40) + 12345 * 4096, (1 << 41) + 777 * 8192          # addresses of stage 0
        self.op = {20: self.A0 + first * 128 - 4096, 21: self.B0 + first * stride - 4096, 22: stride, 23: KF, 24: 0, 25: 0, 26: first}
        self.order = [(first + n) % KF for n in range(KF)]
        self.s, self.scc, self.m0 = {}, 0, 0
        self.vm, self.lg, self.frag = [], [], {}      # loads and LDS reads on their way (oldest first), fragment halves by register
        self.lds = {}                                 # (operand, unit, load) -> stage, barriers before it was waited for
        self.read_at = {}                             # (operand, unit) -> barriers before its last read was waited for
        self.barriers = 0
        self.mfma = []

    def val(self, x):
        if x.startswith("%"):
            return self.op[int(x[1:])]
        return self.s[int(x[1:])] if x.startswith("s") else int(x) & M32

    def load(self, arg, off):
        v, base = re.match(r"%(\d+), s\[(\d+):", arg).groups()
        v, base = int(v), int(base)
        which, j, sw = ("A", v - 8, UNIT_A // 4) if v < 16 else ("B", v - 16, UNIT_B // 4)
        at = (self.s[base] | self.s[base + 1] << 32) + 4096 - (self.A0 if which == "A" else self.B0)
        step = 128 if which == "A" else self.stride
        assert at % step == 0 and 0 <= at // step < self.KF, (which, at)
        assert off == 1024 * (j % 4)
        addr = self.m0 + off
        unit, where = divmod(addr, UNIT_A) if which == "A" else divmod(addr - 3 * UNIT_A, UNIT_B)
        assert where == 1024 * j < sw and unit < (3 if which == "A" else 4), (which, addr)
        assert not any(r[2:] == (which, unit) for r in self.lg), (which, unit)
        assert self.read_at.get((which, unit), -1) < self.barriers, (which, unit)       # the other wavefronts have read it, too
        self.lds[(which, unit, j)] = None             # from its request on a unit holds neither the old nor the new stage
        self.vm.append((which, unit, j, at // step))

    def read(self, ins):
        dst, addr, off = re.match(r"ds_read_b64\S* v\[(\d+):\d+\], v(\d+) offset:(\d+)", ins).groups()
        dst, addr, off = int(dst), int(addr), int(off)
        base, which, q = self.addr[addr]
        if which == "A":
            unit, rows = base // UNIT_A, off // 2048
            assert base % UNIT_A == 0 and unit < 3 and rows < MB
            need, half = [(which, unit, j) for j in range(MB)], (self.ks[addr], q)
        else:
            unit = (base - 3 * UNIT_A) // UNIT_B
            assert (base - 3 * UNIT_A) % UNIT_B == 0 and unit < 4
            half = (off // 8192, off % 8192 // 4096) if self.nn else (self.ks[addr], q)
            need = [(which, unit, j) for j in range(NB)]
        held = [self.lds.get(k) for k in need]
        assert None not in held and len({h[0] for h in held}) == 1, (ins, held)
        assert all(h[1] < self.barriers for h in held), (ins, held)                     # the other wavefronts' loads are there, too
        self.lg.append((dst, (which, held[0][0], half), which, unit))
        self.frag[dst] = None

    def run(self, lines):
        labels = {l[:-1]: k for k, l in enumerate(lines) if re.fullmatch(r"\d+:", l)}
        self.addr, self.ks, pc = {}, {}, 0
        while pc < len(lines):
            ins = lines[pc]
            pc += 1
            op, _, rest = ins.partition(" ")
            a = [x.strip() for x in rest.split(",")]
            if op == "s_mov_b64":
                lo, v = int(re.match(r"s\[(\d+)", a[0]).group(1)), self.val(a[1])
                self.s[lo], self.s[lo + 1] = v & M32, v >> 32
            elif op == "s_mov_b32":
                self.s[int(a[0][1:])] = self.val(a[1])
            elif op in ("s_add_u32", "s_addc_u32", "s_sub_u32", "s_subb_u32"):
                x, y, c = self.val(a[1]), self.val(a[2]), self.scc if op in ("s_addc_u32", "s_subb_u32") else 0
                r = x + y + c if "add" in op else x - y - c
                self.scc = int(r > M32 or r < 0)
                if a[0] == "m0":
                    self.m0 = r & M32
                else:
                    self.s[int(a[0][1:])] = r & M32
            elif op in ("s_mul_i32", "s_mul_hi_u32"):
                r = self.val(a[1]) * self.val(a[2])
                self.s[int(a[0][1:])] = r >> 32 if "hi" in op else r & M32
            elif op.startswith("s_cmp"):
                x, y = self.val(a[0]), self.val(a[1])
                self.scc = int({"s_cmp_lt_u32": x < y, "s_cmp_eq_u32": x == y, "s_cmp_lg_u32": x != y}[op])
            elif op == "s_cselect_b32":
                self.s[int(a[0][1:])] = self.val(a[1]) if self.scc else self.val(a[2])
            elif op == "s_cbranch_scc1":
                if self.scc:
                    pc = labels[a[0][:-1]]
            elif op == "v_add_u32":
                base, vop = self.val(a[1]), int(a[2][1:])
                which = "A" if vop < 4 else "B"
                self.addr[int(a[0][1:])] = (base, which, vop % 2)
                self.ks[int(a[0][1:])] = vop % 4 // 2
            elif op == "global_load_lds_dwordx4":
                self.load(rest.split(" offset:")[0], int(rest.split(" offset:")[1]))
            elif op.startswith("ds_read"):
                self.read(ins)
            elif op == "s_waitcnt":
                for what, n in re.findall(r"(vmcnt|lgkmcnt)\((\d+)\)", rest):
                    queue = self.vm if what == "vmcnt" else self.lg
                    while len(queue) > int(n):
                        x = queue.pop(0)
                        if what == "vmcnt":
                            self.lds[x[:3]] = (x[3], self.barriers)
                        else:
                            self.frag[x[0]] = x[1]
                            self.read_at[x[2:]] = self.barriers
            elif op == "s_barrier":
                self.barriers += 1
                assert not self.lg                    # everybody has read what this barrier gives away
            elif op.startswith("v_mfma"):
                regs = [int(x) for x in re.findall(r"v\[(\d+):", rest)]
                acc = int(re.match(r"a\[(\d+):", a[0]).group(1)) // 4
                i, j = divmod(acc, NB)
                n = len(self.mfma)
                stage, ks = self.order[n // (2 * MB * NB)], n // (MB * NB) % 2
                got = [self.frag.get(r + 2 * q) for r in regs for q in range(2)]
                assert got == [("B", stage, (ks, 0)), ("B", stage, (ks, 1)), ("A", stage, (ks, 0)), ("A", stage, (ks, 1))], (n, i, j, got)
                self.mfma.append(acc)
            elif not re.fullmatch(r"\d+:|s_nop.*|v_accvgpr_write_b32.*", ins):
                raise AssertionError(ins)
        assert not self.vm and not self.lg
        assert self.mfma == list(range(MB * NB)) * (2 * self.KF)


@pytest.mark.parametrize("nn", [False, True])
@pytest.mark.parametrize("KF", [1, 2, 3, 4, 5, 8, 17])
def test_every_mfma_finds_its_stage(nn, KF):
    lines = _lines("SYMB_GEMM16T_LOOP_" + ("NN" if nn else "NT"))
    for first in sorted({x * KF // 8 for x in range(8)}):
        Loop(nn, KF, first, 128 * 40000 if nn else 128).run(lines)
    Loop(nn, KF, KF - 1, (1 << 32) - 128 if nn else 128).run(lines)           # a stage stride times KF beyond 32 bits


@pytest.mark.parametrize("nn", [False, True])
def test_a_missing_barrier_or_wait_is_seen(nn):
    """The simulation itself: every barrier taken out, and every wait for loads or fragments loosened by one, must fail it."""
    lines = _lines("SYMB_GEMM16T_LOOP_" + ("NN" if nn else "NT"))
    barriers = [k for k, l in enumerate(lines) if l == "s_barrier"]
    waits = [k for k, l in enumerate(lines) if "vmcnt" in l]
    assert len(barriers) == 4 and len(waits) == 5

    def fails(changed):
        for KF in (1, 2, 3, 4, 17):
            try:
                Loop(nn, KF, 0, 128).run(changed)
            except AssertionError:
                return True
        return False
    assert not fails(lines)
    for k in barriers:
        assert fails(lines[:k] + lines[k + 1:]), k
    for k, l in enumerate(lines):
        for what, n in re.findall(r"(vmcnt|lgkmcnt)\((\d+)\)", l):
            if (what, n) != ("lgkmcnt", "15"):           # (the largest there is: may be less than needed)
                looser = l.replace(f"{what}({n})", f"{what}({int(n) + 1})")
                assert fails(lines[:k] + [looser] + lines[k + 1:]), (k, looser)


def test_compiler_code_leaves_the_accumulators_alone(device_asm):  # noqa: F811
    """As test_gemm16_registers.py has it for the square tiles; 128 accumulation registers, one wavefront per SIMD."""
    kernels = re.findall(r"^(_ZN4symb18symb_gemm16_kernelILi4E\w+ELi8EEE\w+):(.*?)^\.Lfunc_end", device_asm, re.S | re.M)
    assert len(kernels) == 4
    for name, body in kernels:
        inside = False
        for raw in body.splitlines():
            if "ASMSTART" in raw or "ASMEND" in raw:
                inside = "ASMSTART" in raw
            elif not inside:
                assert not re.search(r"\ba\d+\b|\ba\[\d+|accvgpr|v_mfma", raw.split(";")[0]), (name, raw)

"""The skinny, gradient, small-batch, narrow-layer and short-inner-dimension kernels read LDS from assembly statements with a wait of their own: nothing between
such a read and the wait that covers it may touch the registers still in flight (see test_gemm16_registers.py; no GPU needed)."""
import re

import pytest

from test_gemm16_registers import _regs, device_asm  # noqa: F401


def _blocks(text):
    """{label: ([(inside an assembly statement?, instruction)], [labels that may follow])} of one kernel's listing."""
    blocks, label, inside, after = {"": ([], [])}, "", False, True
    for n, raw in enumerate(text.splitlines()):
        if "ASMSTART" in raw or "ASMEND" in raw:
            inside = "ASMSTART" in raw
            continue
        s = raw.split(";")[0].strip()
        if s.endswith(":"):
            if after:
                blocks[label][1].append(s[:-1])
            label, after = s[:-1], True
            blocks[label] = ([], [])
        elif s and not s.startswith("."):
            op, _, to = s.partition(" ")
            blocks[label][0].append((inside, s))
            if op.startswith("s_cbranch") or op == "s_branch":
                blocks[label][1].append(to.strip())
                if op == "s_branch":
                    after = False
                else:                                # what follows is a block of its own
                    blocks[label][1].append(f"{label}+{n}")
                    label = f"{label}+{n}"
                    blocks[label] = ([], [])
            elif op == "s_endpgm":
                after = False
    return blocks


def reads_that_are_touched(text):
    """(reads, [(instruction, registers)]): the LDS reads of assembly statements along every path of one kernel's listing, and the instructions between such a read and its wait
    that name its registers.  LDS operations return in order: lgkmcnt(n) retires all but the newest n, another counter none."""
    blocks = _blocks(text)
    reads, touched, seen = set(), [], set()
    work = [("", ())]
    while work:
        label, pending = work.pop()
        if (label, pending) in seen:
            continue
        seen.add((label, pending))
        assert len(seen) < 100000
        pending = list(pending)                      # registers of each LDS operation under way, oldest first
        for at, (inside, s) in enumerate(blocks[label][0]):
            op, _, rest = s.partition(" ")
            named = set().union(*[_regs(t) for t in re.findall(r"v\[\d+:\d+\]|v\d+", rest)] or [set()])
            if op == "s_waitcnt":
                m = re.search(r"lgkmcnt\((\d+)\)", rest)
                if m:
                    pending = pending[len(pending) - min(int(m.group(1)), len(pending)):]
            else:
                if named & set().union(*pending):
                    touched.append((s, sorted(named & set().union(*pending))))
                if inside and op in ("ds_read_b128", "ds_read_b64_tr_b16"):
                    reads.add((label, at))
                    pending.append(frozenset(_regs(rest.split(",")[0].strip())))
                elif op.startswith("ds_"):           # (the compiler waits for these itself)
                    pending.append(frozenset())
        while pending and not pending[0]:
            pending.pop(0)
        work += [(to, tuple(pending)) for to in blocks[label][1]]
    return len(reads), touched


# kernel, the reads that each of its instantiations has at least
KERNELS = [("24symb_small_stream_kernel", 25), ("24symb_small_narrow_kernel", 12), ("20symb_gemm_mid_kernel", 24), ("18symb_skinny_kernel", 8), ("26symb_lora_grad_wave_kernel", 20),
           ("26symb_lora_grad_pair_kernel", 52), ("27symb_lora_grad_short_kernel", 40), ("23symb_gemm_narrow_kernel", 18), ("23symb_gemm_shortk_kernel", 22)]


@pytest.mark.parametrize("name,least", KERNELS)
def test_lds_reads_are_untouched_until_their_wait(device_asm, name, least):  # noqa: F811
    kernels = re.findall(r"^(_ZN4symb%s\w+):(.*?)^\.Lfunc_end" % name, device_asm, re.S | re.M)
    assert kernels
    for kernel, text in kernels:
        reads, touched = reads_that_are_touched(text)
        assert reads >= least, (kernel, reads)
        assert not touched, (kernel, touched[:5])


LISTING = """
\t;;#ASMSTART
\tds_read_b128 v[0:3], v20
\t;;#ASMEND
\t;;#ASMSTART
\tds_read_b128 v[4:7], v20 offset:16
\t;;#ASMEND
\ts_cbranch_scc1 .LBB0_2
\tv_add_u32_e32 v21, 1, v21
.LBB0_2:
\t;;#ASMSTART
\t%s
\t;;#ASMEND
\tv_mfma_f32_16x16x32_bf16 v[8:11], v[0:3], v[12:15], v[8:11]
\t%s
\ts_waitcnt lgkmcnt(0)
\tv_mov_b32_e32 v16, v4
\ts_endpgm
"""


@pytest.mark.parametrize("wait,between,count", [
    ("s_waitcnt lgkmcnt(1)", "v_mov_b32_e32 v17, v21", 0), ("s_waitcnt lgkmcnt(1)", "v_mov_b32_e32 v16, v5", 1), ("s_waitcnt vmcnt(0)", "s_nop 0", 1),
    ("s_waitcnt lgkmcnt(0)", "v_mov_b32_e32 v16, v5", 0), ("s_waitcnt lgkmcnt(2)", "s_nop 0", 1)])
def test_what_the_check_of_lds_reads_sees(wait, between, count):
    reads, touched = reads_that_are_touched(LISTING % (wait, between))
    assert reads == 2 and len({t[0] for t in touched}) == count


def test_short_inner_dimension_kernel_leaves_its_stores_open(device_asm):  # noqa: F811
    """Its loop waits once per chunk of rows, ahead of the barrier, for that chunk's requests: requests and stores are counted together, so that any other
    wait in it (for a vector load, say) would be one for the output just stored."""
    kernels = re.findall(r"^_ZN4symb23symb_gemm_shortk_kernel\w+:(.*?)^\.Lfunc_end", device_asm, re.S | re.M)
    assert len(kernels) == 4
    for text in kernels:
        loop, stores = text[text.rindex("s_barrier"):], text.count("global_store_dwordx4")
        assert stores == loop.count("global_store_dwordx4") == 4
        assert not re.search(r"s_waitcnt[^\n]*vmcnt", loop), loop
        before = text[:text.rindex("s_barrier")]
        req = before.count("global_load_lds_dwordx4", before.rindex("s_barrier"))        # two chunks' requests, with dH
        assert {f"vmcnt({n})" for n in (req // 2 + 8, req // 2 + 4, req // 2 + 7)} <= set(re.findall(r"vmcnt\(\d+\)", before))

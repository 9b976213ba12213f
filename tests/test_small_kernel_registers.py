"""The skinny, gradient and small-batch kernels read LDS from assembly statements with a wait of their own: nothing the compiler generates between
such a read and the wait may touch the registers still in flight (see test_gemm16_registers.py; no GPU needed)."""
import re

import pytest

from test_gemm16_registers import _regs, device_asm  # noqa: F401


def test_lds_reads_are_untouched_until_their_wait(device_asm):  # noqa: F811
    checked = 0
    for m in re.finditer(r"^(_ZN4symb(?:24symb_small_(?:stream|narrow)_kernel|18symb_skinny_kernel|26symb_lora_grad_(?:wave|pair)_kernel)\w+):(.*?)^\.Lfunc_end", device_asm, re.S | re.M):
        pending, inside = set(), False
        for raw in m.group(2).splitlines():
            if "ASMSTART" in raw or "ASMEND" in raw:
                inside = "ASMSTART" in raw
                continue
            s = raw.split(";")[0].strip()
            if not s or s.startswith(".") or s.endswith(":"):
                if s.endswith(":"):
                    pending.clear()              # checked per straight-line stretch
                continue
            op, _, rest = s.partition(" ")
            if inside and op in ("ds_read_b128", "ds_read_b64_tr_b16"):
                pending |= _regs(rest.split(",")[0].strip())
                checked += 1
            elif inside and op == "s_waitcnt":
                pending.clear()
            else:
                touched = set().union(*[_regs(t) for t in re.findall(r"v\[\d+:\d+\]|v\d+", rest)] or [set()])
                assert not (touched & pending), (m.group(1), s)
    assert checked > 200


@pytest.mark.parametrize("name", ["27symb_lora_grad_short_kernel", "23symb_gemm_narrow_kernel", "23symb_gemm_shortk_kernel"])
def test_lds_reads_of_further_kernels(device_asm, name):  # noqa: F811
    only = "\n".join(m.group(0) for m in re.finditer(r"^_ZN4symb%s\w+:.*?^\.Lfunc_end" % name, device_asm, re.S | re.M))
    assert only
    # (under a name that it looks for, and as often as it takes to make up the number of reads that it wants to see)
    test_lds_reads_are_untouched_until_their_wait("\n".join([only.replace("_ZN4symb" + name, "_ZN4symb26symb_lora_grad_wave_kernel")] * 20))


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

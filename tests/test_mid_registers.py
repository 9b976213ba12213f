"""As test_small_kernel_registers.py, for the kernel of small layers: nothing the compiler generates between an LDS read issued from
an assembly statement and its wait touches the registers still in flight (no GPU needed)."""
import re

from test_gemm16_registers import _regs, device_asm  # noqa: F401


def test_lds_reads_are_untouched_until_their_wait(device_asm):  # noqa: F811
    kernels = re.findall(r"^(_ZN4symb20symb_gemm_mid_kernel\w+):(.*?)^\.Lfunc_end", device_asm, re.S | re.M)
    assert len(kernels) == 2
    for name, body in kernels:
        pending, inside, checked = set(), False, 0
        for raw in body.splitlines():
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
                assert not (touched & pending), (name, s)
        assert checked >= 5, name

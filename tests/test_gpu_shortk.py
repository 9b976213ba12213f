"""The input gradient of a layer of 64 to 256 outputs over many rows: every inner dimension it takes, ragged chunks of rows and columns, LoRA segments beside
others, dH of its own and taken over, without adapters, and the calls that are not its."""
import pytest
import torch

import gpu_harness as gh
import synth
from helpers import check_dx
from paper_2507_03220_amd import binding as sb
from test_gpu_parity import I, L, N, make_problem, oracle_ads
import test_gpu_parity as tp

pytestmark = pytest.mark.gpu
tp.gh, tp.sb = gh, sb                    # what its problem maker uses
IN = 3                                   # IA3 on the input


def shortk_launches(call):
    sb.symb_debug_gemm_timing_enable(gh.handle(), 1)
    try:
        call()
        return sb.symb_debug_gemm_timing_read(gh.handle(), 33)[1]
    finally:
        sb.symb_debug_gemm_timing_enable(gh.handle(), 0)


def run(p, d_in, d_out, want, conv1d=False, flags=sb.SYMB_BWD_FULL, tag="", grads_first=False):
    dev = gh.upload_adapters(p["ads"], d_in, d_out, grads=grads_first)
    b = sb.Batch(d_in, d_out, p["off"], dev.descs, int(conv1d))
    W, dY = gh.weight_to_dev(p["W"], conv1d), gh.to_dev(p["dY"])
    ws = torch.empty(max(sb.symb_workspace_bytes(b, op) for op in (sb.SYMB_OP_BWD_INPUT, sb.SYMB_OP_ADAPTER_GRAD)), device="cuda", dtype=torch.uint8)
    if grads_first:
        sb.symb_adapter_grad(gh.handle(), b, gh.to_dev(p["X"]), dY, None, sb.SYMB_GRAD_OVERWRITE, ws)
        flags = sb.SYMB_BWD_REUSE_DH
    dX = torch.full((p["T"], d_in), float("nan"), device="cuda", dtype=torch.bfloat16)
    assert shortk_launches(lambda: sb.symb_base_linear_bwd_input(gh.handle(), b, dY, W, dX, flags, ws)) == want
    ads = oracle_ads([gh.HostAdapter() for _ in p["ads"]] if flags == sb.SYMB_BWD_BASE_ONLY else p["ads"])
    rows = synth.sample_rows(p["off"], 8, f"shortk{tag}", block=64)
    check_dx(gh.bf16_to_f64(dX)[rows], p["off"], ads, p["dY"], p["W"], f"dX {tag}", rows=rows)
    assert not torch.isnan(dX.float()).any()


@pytest.mark.parametrize("d_out,d_in,ranks", [(64, 8200, [16]), (128, 10056, [8, 5]), (192, 8256, [12, 4]), (256, 9160, [16, 7])])
def test_input_gradient(d_out, d_in, ranks):
    lens = [1500, 1, 0, 33, 1000, 31, 32, 1703]
    p = make_problem(d_out + d_in, d_in, d_out, lens, [L, L, L, N, L, N, L, L], ranks)
    run(p, d_in, d_out, 1, tag=f"{d_out}")
    run(p, d_in, d_out, 1, flags=sb.SYMB_BWD_BASE_ONLY, tag=f"{d_out} base only")
    run(p, d_in, d_out, 1, grads_first=True, tag=f"{d_out} dH of the gradient call")


@pytest.mark.parametrize("T,d_out,d_in,kinds,rank,conv1d", [
    (4000, 256, 8200, [L, I], 16, False), (4000, 256, 8200, [L, IN], 16, False), (4000, 256, 8200, [L, N], 17, False), (4000, 256, 8200, [L, N], 16, True),
    (4000, 72, 8200, [L, N], 16, False), (4000, 320, 8200, [L, N], 16, False), (1900, 256, 8192, [L, N], 16, False), (12100, 64, 4104, [L, N], 16, False)])
def test_calls_that_are_not_its(T, d_out, d_in, kinds, rank, conv1d):
    p = make_problem(T + d_out, d_in, d_out, [T - 1000, 1000], kinds, [rank])
    run(p, d_in, d_out, 0, conv1d=conv1d, tag=f"{T} {d_out} {kinds}")


@pytest.mark.parametrize("clients,tokens,d_out,d_in,kind,want", [
    (512, 1, 256, 11008, L, 0), (512, 1, 256, 11008, N, 0), (512, 1, 64, 6144, L, 1), (3000, 1, 64, 6144, N, 1), (500, 4, 256, 4096, L, 0), (512, 4, 64, 1024, L, 1), (128, 4, 128, 4096, L, 1),
    (750, 8, 64, 4096, L, 1)])
def test_which_calls_of_short_segments_take_it(clients, tokens, d_out, d_in, kind, want):
    """A chunk of rows costs as much whatever it holds; without adapters it may cross segments."""
    p = make_problem(clients + d_in, d_in, d_out, [tokens] * clients, [kind], [8])
    dev = gh.upload_adapters(p["ads"], d_in, d_out, grads=False)
    b = sb.Batch(d_in, d_out, p["off"], dev.descs)
    W, dY = gh.to_dev(p["W"]), gh.to_dev(p["dY"])
    dX = torch.full((p["T"], d_in), float("nan"), device="cuda", dtype=torch.bfloat16)
    assert shortk_launches(lambda: sb.symb_base_linear_bwd_input(gh.handle(), b, dY, W, dX, sb.SYMB_BWD_FULL, gh.workspace(b, sb.SYMB_OP_BWD_INPUT))) == want
    rows = synth.sample_rows([0, p["T"]], 100, f"short{clients}", block=64)
    check_dx(gh.bf16_to_f64(dX)[rows], p["off"], oracle_ads(p["ads"]), p["dY"], p["W"], "dX", rows=rows)
    assert not torch.isnan(dX.float()).any()

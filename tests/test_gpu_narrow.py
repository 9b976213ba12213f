"""The forward of a narrow layer over many rows in one launch, LoRA shrink included: ragged chunks of rows, every kind of segment, ranks to 16, one stage of the
inner dimension and more than the rings hold, the H it leaves for a gradient call, and the calls that are not its."""
import numpy as np
import pytest
import torch

import gpu_harness as gh
import oracle
import synth
from helpers import assert_close, check_y
from paper_2507_03220_amd import binding as sb
from test_gpu_parity import I, L, N, make_problem, oracle_ads
import test_gpu_parity as tp

pytestmark = pytest.mark.gpu
tp.gh, tp.sb = gh, sb                    # what its problem maker uses


def narrow_launches(call):
    sb.symb_debug_gemm_timing_enable(gh.handle(), 1)
    try:
        call()
        return sb.symb_debug_gemm_timing_read(gh.handle(), 32)[1]
    finally:
        sb.symb_debug_gemm_timing_enable(gh.handle(), 0)


@pytest.mark.parametrize("d_in,d_out,ranks", [(64, 136, [16]), (192, 256, [8, 5]), (448, 200, [16, 12, 4]), (832, 256, [7, 16])])
def test_forward_and_the_h_it_leaves(d_in, d_out, ranks):
    lens = [4100, 1, 0, 2600, 63, 1500, 65, 64, 1700]
    kinds = [L, L, L, I, L, N, L, L, L]
    p = make_problem(d_in + d_out, d_in, d_out, lens, kinds, ranks)
    off, oads = p["off"], oracle_ads(p["ads"])
    dev = gh.upload_adapters(p["ads"], d_in, d_out, grads=True)
    b = sb.Batch(d_in, d_out, off, dev.descs)
    X, W, bias, dY = gh.to_dev(p["X"]), gh.to_dev(p["W"]), gh.to_dev(p["bias"]), gh.to_dev(p["dY"])
    ws = torch.empty(max(sb.symb_workspace_bytes(b, op) for op in (sb.SYMB_OP_FWD, sb.SYMB_OP_ADAPTER_GRAD)), device="cuda", dtype=torch.uint8)
    rows = synth.sample_rows(off, 12, f"narrow{d_in}", block=64)
    for bv, bd in ((p["bias"], bias), (None, None)):
        Y = torch.full((p["T"], d_out), float("nan"), device="cuda", dtype=torch.bfloat16)
        assert narrow_launches(lambda: sb.symb_base_linear_fwd(gh.handle(), b, X, W, bd, Y, None, ws)) == 1  # noqa: B023
        check_y(gh.bf16_to_f64(Y)[rows], off, oads, p["X"], p["W"], bv, "Y", rows=rows)
        assert not torch.isnan(Y.float()).any()
    Yb = torch.from_numpy(np.zeros((p["T"], d_out), dtype=np.float32)).cuda().to(torch.bfloat16)
    sb.symb_adapter_grad(gh.handle(), b, X, dY, Yb, sb.SYMB_GRAD_OVERWRITE | sb.SYMB_GRAD_REUSE_HS, ws)
    for i, k in enumerate(kinds):
        if k == L and lens[i]:
            dAr, dBr = oracle.lora_grad(off, oads, p["X"], p["dY"], i)
            assert_close(dev.descs[i].dA.cpu().numpy(), dAr, f"dA[{i}]")
            assert_close(dev.descs[i].dB.cpu().numpy(), dBr, f"dB[{i}]")


@pytest.mark.parametrize("T,d_in,d_out,rank,want", [
    (9800, 128, 256, 16, 1), (9700, 128, 256, 16, 0), (16384, 128, 256, 8, 1), (16400, 128, 256, 8, 0),      # 154, 152, 256 and 257 chunks
    (27800, 64, 256, 8, 0), (27904, 64, 256, 8, 1),                                                          # 435 and 436
    (12000, 136, 256, 8, 0), (12000, 128, 128, 8, 0), (12000, 128, 264, 8, 0), (12000, 128, 256, 17, 0)])
def test_which_calls_take_it(T, d_in, d_out, rank, want):
    which_calls_take_it(T, d_in, d_out, rank, want, [T])


def which_calls_take_it(T, d_in, d_out, rank, want, lens):
    p = make_problem(T, d_in, d_out, lens, [L], [rank])
    dev = gh.upload_adapters(p["ads"], d_in, d_out, grads=False)
    X, W = gh.to_dev(p["X"]), gh.to_dev(p["W"])
    rows = synth.sample_rows(p["off"], 20 if len(lens) == 1 else 1, f"takes{T}", block=512)
    for conv1d, base in ((0, False), (0, True), (1, False)):
        b = sb.Batch(d_in, d_out, p["off"], dev.descs, conv1d)
        Wl = W if not conv1d else gh.weight_to_dev(p["W"], True)
        Y = torch.full((T, d_out), float("nan"), device="cuda", dtype=torch.bfloat16)
        Yb = torch.empty_like(Y) if base else None
        ws = gh.workspace(b, sb.SYMB_OP_FWD)
        assert narrow_launches(lambda: sb.symb_base_linear_fwd(gh.handle(), b, X, Wl, None, Y, Yb, ws)) == (want if not conv1d and not base else 0)  # noqa: B023
        check_y(gh.bf16_to_f64(Y)[rows], p["off"], oracle_ads(p["ads"]), p["X"], p["W"], None, "Y", rows=rows)


@pytest.mark.parametrize("clients,tokens,d_in,want", [
    (160, 1, 6144, 0), (200, 1, 6144, 0), (256, 1, 6144, 0), (500, 1, 6144, 0), (200, 16, 2048, 0), (160, 56, 1600, 1), (160, 55, 1600, 0), (250, 40, 1600, 1),
    (200, 1, 1536, 1), (500, 16, 512, 1), (500, 17, 512, 0), (500, 17, 384, 1), (250, 72, 256, 0), (250, 72, 128, 1), (440, 56, 6144, 1), (440, 8, 6144, 0)])
def test_which_calls_of_short_segments_take_it(clients, tokens, d_in, want):
    """A chunk of rows costs the whole weight, so that chunks of a few rows are for short inner dimensions."""
    which_calls_take_it(clients * tokens, d_in, 256, 8, want, [tokens] * clients)

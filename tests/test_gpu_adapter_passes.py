"""The shrink of the backward (dH = s dY B) reads B_i [d_out][r] as it lies: every way it can lie (rows of 8 to 256 bytes, with and
without the swizzle of ranks 64 and 128), slices and remainders of the inner dimension, launches of few and many chunks, and
the packed copy that ranks that are no multiple of 4 still take."""
import pytest
import torch

import gpu_harness as gh
import oracle
import test_gpu_parity as tp
from helpers import assert_close, check_dx
from paper_2507_03220_amd import binding as sb
from test_gpu_parity import L, N, make_problem, oracle_ads

pytestmark = pytest.mark.gpu
tp.gh, tp.sb = gh, sb                    # what its problem maker uses


def _check(p, tag):
    off, oads = p["off"], oracle_ads(p["ads"])
    check_dx(gh.bf16_to_f64(gh.backward_input(off, p["ads"], p["dY"], p["W"])), off, oads, p["dY"], p["W"], f"dX {tag}")
    dev = gh.adapter_grad(off, p["ads"], p["X"], p["dY"])
    for i, d in enumerate(dev.descs):
        dAr, dBr = oracle.lora_grad(off, oads, p["X"], p["dY"], i)
        assert_close(d.dA.cpu().numpy(), dAr, f"dA[{i}] {tag}")
        assert_close(d.dB.cpu().numpy(), dBr, f"dB[{i}] {tag}")


@pytest.mark.parametrize("ranks", [[4], [8, 16, 12], [32, 20], [64, 48, 4], [128, 64, 100, 32, 16, 8], [16, 5]])
@pytest.mark.parametrize("d_out", [40, 136, 1096])
def test_shrink_of_the_backward_for_every_rank(ranks, d_out):
    _check(make_problem(sum(ranks) + d_out, 72, d_out, [33, 64, 1, 100, 31, 70], [L], ranks), f"ranks {ranks} d_out {d_out}")


@pytest.mark.parametrize("rank", [8, 16, 32, 64, 128])
def test_shrink_of_the_backward_over_many_chunks(rank):
    _check(make_problem(rank, 72, 328, [8300], [L], [rank]), f"rank {rank}")          # more than 256 row chunks: the two-buffer build


@pytest.mark.parametrize("rank", [5, 12, 16])
def test_db_and_dh_in_one_pass_over_a_wide_layer(rank):
    _check(make_problem(rank, 72, 16392, [40, 33], [L], [rank]), f"rank {rank}")


@pytest.mark.parametrize("lens,ranks", [([31, 32, 33, 127, 128, 129], [16, 5, 8]), ([1, 160, 257, 1537], [32, 17]), ([300, 95], [64, 40]), ([520, 64], [128, 72, 4])])
@pytest.mark.parametrize("dims", [(8, 136), (120, 64), (264, 392)])
def test_gradients_over_slices_of_tokens(lens, ranks, dims):
    """Edges of the 32-token slices dealt over four wavefronts, of the column blocks and of a segment walked in runs; accumulation."""
    p = make_problem(sum(lens) + dims[0], dims[0], dims[1], lens, [L], ranks)
    off, oads = p["off"], oracle_ads(p["ads"])
    dev = gh.adapter_grad(off, p["ads"], p["X"], p["dY"])
    once = [(d.dA.clone(), d.dB.clone()) for d in dev.descs]
    gh.adapter_grad(off, p["ads"], p["X"], p["dY"], accumulate_into=dev)
    for i, (d, (dA, dB)) in enumerate(zip(dev.descs, once)):
        dAr, dBr = oracle.lora_grad(off, oads, p["X"], p["dY"], i)
        assert_close(dA.cpu().numpy(), dAr, f"dA[{i}]")
        assert_close(dB.cpu().numpy(), dBr, f"dB[{i}]")
        assert_close(d.dA.cpu().numpy(), 2 * dAr, f"accumulated dA[{i}]")
        assert_close(d.dB.cpu().numpy(), 2 * dBr, f"accumulated dB[{i}]")


@pytest.mark.parametrize("ranks", [[8], [32], [64, 48], [8, 16, 32, 64], [5, 100]])
@pytest.mark.parametrize("lens", [[16] * 40, [1, 33, 7] * 8, [400, 390, 16]])
def test_gradients_of_many_short_segments(lens, ranks):
    """Launches of more workgroups than CUs, of few and of short walks: both gradient kernels, dB alone and beside dH."""
    p = make_problem(len(lens) + sum(ranks), 264, 1032, lens, [L], ranks)
    off, oads = p["off"], oracle_ads(p["ads"])
    dev = gh.adapter_grad(off, p["ads"], p["X"], p["dY"])
    for i, d in enumerate(dev.descs):
        dAr, dBr = oracle.lora_grad(off, oads, p["X"], p["dY"], i)
        assert_close(d.dA.cpu().numpy(), dAr, f"dA[{i}]")
        assert_close(d.dB.cpu().numpy(), dBr, f"dB[{i}]")


@pytest.mark.parametrize("T,ranks", [(4096, [16]), (4090, [32, 5]), (3000, [64, 100]), (4100, [8]), (8190, [20]), (5000, [40, 64]), (8200, [16]), (9000, [32, 12]), (12280, [64]), (12300, [48])])
def test_shrink_by_its_number_of_rows(T, ranks):
    """The builds of 16, 32 and 48 rows and the one of 32 rows that more rows take, at their edges; the wavefronts' slices of the inner dimensions: some, one or none whole,
    and a remainder."""
    for d_in, d_out in ((1096, 72), (72, 1608)):
        lens = [T // 3, 1, T - T // 3 - 1]
        p = make_problem(T + sum(ranks) + d_in, d_in, d_out, lens, [L], ranks)
        Y, _ = gh.forward(p["off"], p["ads"], p["X"], p["W"], None, want_base=False)
        _, Yr = oracle.forward(p["off"], oracle_ads(p["ads"]), p["X"], p["W"])
        assert_close(gh.bf16_to_f64(Y), Yr, f"Y {T} rows", out_bf16=True)
        _check(p, f"{T} rows, ranks {ranks}")


@pytest.mark.parametrize("lens", [[1], [16], [17, 2], [32, 33], [64, 63, 0, 5], [65, 8]])                # (65: the launches of longer segments)
@pytest.mark.parametrize("d_in,d_out,ranks", [(72, 136, [16, 4]), (264, 1096, [8, 12]), (136, 4040, [16])])
def test_gradients_of_short_segments_in_one_launch(lens, d_in, d_out, ranks):
    """Gradients, accumulated ones, and the input gradient on the dH that the call leaves behind."""
    p = make_problem(sum(lens) + d_in, d_in, d_out, lens + [3], [L] * len(lens) + [N], ranks)
    off, oads = p["off"], oracle_ads(p["ads"])
    dev = gh.upload_adapters(p["ads"], d_in, d_out, grads=True)
    b = sb.Batch(d_in, d_out, off, dev.descs)
    X, dY, W = gh.to_dev(p["X"]), gh.to_dev(p["dY"]), gh.to_dev(p["W"])
    ws = torch.empty(max(sb.symb_workspace_bytes(b, op) for op in (sb.SYMB_OP_FWD, sb.SYMB_OP_BWD_INPUT, sb.SYMB_OP_ADAPTER_GRAD)), device="cuda", dtype=torch.uint8)
    dX = torch.full((p["T"], d_in), float("nan"), device="cuda", dtype=torch.bfloat16)
    want = [oracle.lora_grad(off, oads, p["X"], p["dY"], i) for i in range(len(lens))]
    for times, flags in ((1, sb.SYMB_GRAD_OVERWRITE), (2, sb.SYMB_GRAD_ACCUMULATE)):
        sb.symb_adapter_grad(gh.handle(), b, X, dY, None, flags, ws)
        for i, (dAr, dBr) in enumerate(want):
            assert_close(dev.descs[i].dA.cpu().numpy(), times * dAr, f"dA[{i}]")
            assert_close(dev.descs[i].dB.cpu().numpy(), times * dBr, f"dB[{i}]")
    sb.symb_base_linear_bwd_input(gh.handle(), b, dY, W, dX, sb.SYMB_BWD_REUSE_DH, ws)
    check_dx(gh.bf16_to_f64(dX), off, oads, p["dY"], p["W"], "dX")
    sb.symb_adapter_grad(gh.handle(), b, X, dY, None, sb.SYMB_GRAD_OVERWRITE, ws)
    once = [(d.dA.clone(), d.dB.clone()) for d in dev.descs[:len(lens)]]
    sb.symb_adapter_grad(gh.handle(), b, X, dY, None, sb.SYMB_GRAD_OVERWRITE | sb.SYMB_GRAD_REUSE_DH | sb.SYMB_GRAD_REUSE_HS, ws)        # the two launches: the same bits
    assert all(torch.equal(x, d.dA) and torch.equal(y, d.dB) for (x, y), d in zip(once, dev.descs))

"""Products that take the 256x128 GEMM tile: whole and split over K, inner dimensions with and without a
remainder of 64, ragged edges, every epilogue, LoRA steps of ranks 5 to 128, in both directions and weight layouts."""
import numpy as np
import pytest
import torch

import gpu_harness as gh
import synth
from helpers import assert_close, check_dx, check_y
from paper_2507_03220_amd import binding as sb
from test_gpu_parity import I, L, N, make_problem, oracle_ads
import test_gpu_parity as tp

pytestmark = pytest.mark.gpu
tp.gh, tp.sb = gh, sb                    # what its problem maker uses


@pytest.mark.parametrize("T,d_in,d_out,tile,parts", [
    (1000, 264, 2056, 2, 1), (250, 2056, 392, 2, 4), (1300, 3144, 4104, 10, 1), (700, 6152, 4104, 10, 2), (1000, 6152, 2056, 10, 3)])
def test_forms_of_calls_in_tiles_of_128_columns(T, d_in, d_out, tile, parts):
    """The 128x128 and 256x128 tiles, whole and in K parts, with terms of short segments, IA3 and the noise effect in the epilogue, IA3 of the input in the input gradient's, and
    the same calls on a buffer per client, in another order in memory."""
    lens = [1] * 80 + [T // 3, 0, 17, T // 4, T - T // 3 - T // 4 - 97]
    rng = np.random.default_rng(T)

    def pieces(M, width):                # a buffer per segment, the last segment's first
        arena = torch.full((T, width), float("nan"), device="cuda", dtype=torch.bfloat16)
        v = [arena[T - off[i + 1]:T - off[i]] if lens[i] else None for i in range(len(lens))]
        for i in range(len(lens)):
            if M is not None and lens[i]:
                v[i].copy_(M[off[i]:off[i + 1]])
        return v

    def joined(v):
        return torch.cat([x for x in v if x is not None])
    plain = sb.Batch(d_in, d_out, [0, T], [sb.Adapter()])
    need = sb.symb_workspace_bytes(plain, sb.SYMB_OP_FWD)
    assert need == (-(-T // (256 if tile & 8 else 128)) * -(-d_out // 128) * parts * (256 if tile & 8 else 128) * 128 * 4 if parts > 1 else 0)
    p = make_problem(T + d_in, d_in, d_out, lens, [L] * 80 + [L, N, I, N, L], [16])
    off, oads = p["off"], oracle_ads(p["ads"])
    rows = synth.sample_rows(off, 2, f"forms{T}", block=128)
    neff = [synth.f32_to_bf16_bits(rng.standard_normal((1 if i % 2 else n, d_out)).astype(np.float32)) if n and i % 3 else None for i, n in enumerate(lens)]
    dev = gh.upload_adapters(p["ads"], d_in, d_out, grads=False)
    X, bias, nd = gh.to_dev(p["X"]), gh.to_dev(p["bias"]), [gh.to_dev(n) for n in neff]
    for conv1d in (0, 1):
        b = sb.Batch(d_in, d_out, off, dev.descs, conv1d)
        W, ws = gh.weight_to_dev(p["W"], bool(conv1d)), gh.workspace(b, sb.SYMB_OP_FWD)
        if not conv1d:
            assert ws.numel() == need + (T * 2 * 16 * 2 + 255) // 256 * 256 + 80 * d_out * 4                   # partial tiles, Hs, the short segments' terms
        Y, Yn = (torch.full((T, d_out), float("nan"), device="cuda", dtype=torch.bfloat16) for _ in range(2))
        xs, ys = pieces(X, d_in), pieces(None, d_out)
        for call in (lambda: sb.symb_base_linear_fwd(gh.handle(), b, X, W, bias, Y, None, ws),
                     lambda: sb.symb_base_linear_fwd_denoise(gh.handle(), b, X, W, bias, nd, Yn, ws),
                     lambda: sb.symb_base_linear_fwd_seg(gh.handle(), b, xs, W, bias, ys, ws)):
            assert gh.gemm_launches(call) == {conv1d + tile + 4: 1}
        _, Yr = check_y(gh.bf16_to_f64(Y)[rows], off, oads, p["X"], p["W"], p["bias"], f"Y conv1d={conv1d}", rows=rows)
        seg = np.searchsorted(off, rows, side="right") - 1
        taken = np.stack([np.zeros(d_out) if neff[i] is None else synth.bf16_bits_to_f32(neff[i][0 if len(neff[i]) == 1 else t - off[i]]) for i, t in zip(seg, rows)])
        assert_close(gh.bf16_to_f64(Yn)[rows], Yr - taken, f"denoised Y conv1d={conv1d}", out_bf16=True)
        assert torch.equal(joined(ys).view(torch.int16), Y.view(torch.int16))
    q = make_problem(T + d_out, d_out, d_in, lens, [L] * 80 + [L, N, 3, N, L], [16])          # its input gradient has the same product
    qd = gh.upload_adapters(q["ads"], d_out, d_in, grads=False)
    dY = gh.to_dev(q["dY"])
    for conv1d in (0, 1):
        b = sb.Batch(d_out, d_in, off, qd.descs, conv1d)
        W, ws = gh.weight_to_dev(q["W"], bool(conv1d)), gh.workspace(b, sb.SYMB_OP_BWD_INPUT)
        dX = torch.full((T, d_out), float("nan"), device="cuda", dtype=torch.bfloat16)
        gs, xs = pieces(dY, d_in), pieces(None, d_out)
        for call in (lambda: sb.symb_base_linear_bwd_input(gh.handle(), b, dY, W, dX, sb.SYMB_BWD_FULL, ws),
                     lambda: sb.symb_base_linear_bwd_input_seg(gh.handle(), b, gs, W, xs, sb.SYMB_BWD_FULL, ws)):
            assert gh.gemm_launches(call) == {1 - conv1d + tile + 4: 1}
        check_dx(gh.bf16_to_f64(dX)[rows], off, oracle_ads(q["ads"]), q["dY"], q["W"], f"dX conv1d={conv1d}", rows=rows)
        assert torch.equal(joined(xs).view(torch.int16), dX.view(torch.int16))


def launches(call, variant):
    """Launches of one instantiation, its tile included (bit 3: 256x128), and what the call returns."""
    sb.symb_debug_gemm_timing_enable(gh.handle(), 1)
    try:
        out = call()
        return sb.symb_debug_gemm_timing_read(gh.handle(), variant)[1], out
    finally:
        sb.symb_debug_gemm_timing_enable(gh.handle(), 0)


@pytest.mark.parametrize("T,d_in,d_out,parts,ranks", [
    (1300, 3144, 4104, 1, [16, 5]), (1500, 3080, 4096, 1, [16, 40, 5]),         # whole: a remainder of 8 beyond the last stage
    (700, 6152, 4104, 2, [16, 128, 5]), (1000, 6152, 2056, 3, [100, 16, 5])])
def test_tall_tile(T, d_in, d_out, parts, ranks):
    plain = sb.Batch(d_in, d_out, [0, T], [sb.Adapter()])
    tiles = -(-T // 256) * -(-d_out // 128)
    need = sb.symb_workspace_bytes(plain, sb.SYMB_OP_FWD)
    assert need == (tiles * parts * 256 * 128 * 4 if parts > 1 else 0)
    lens = [T // 3, 1, T // 4, 0, 17, T - T // 3 - T // 4 - 18]
    p = make_problem(T + d_in, d_in, d_out, lens, [L, I, L, N, L], ranks)
    off, oads = p["off"], oracle_ads(p["ads"])
    rows = synth.sample_rows(off, 6, f"tall{T}", block=128)
    base = [gh.HostAdapter() for _ in lens]
    for conv1d in (False, True):
        n, (Y, _) = launches(lambda: gh.forward(off, base, p["X"], p["W"], None, want_base=False, conv1d=conv1d), 8 + 2 + conv1d)
        assert n == 1
        check_y(gh.bf16_to_f64(Y)[rows], off, oracle_ads(base), p["X"], p["W"], None, "plain Y", rows=rows)
        n, (Y, Yb) = launches(lambda: gh.forward(off, p["ads"], p["X"], p["W"], p["bias"], want_base=parts == 1, conv1d=conv1d), 8 + 4 + 2 + conv1d)
        assert n == 1
        Y0, _ = check_y(gh.bf16_to_f64(Y)[rows], off, oads, p["X"], p["W"], p["bias"], "Y", rows=rows)
        if parts == 1:
            assert_close(gh.bf16_to_f64(Yb)[rows], Y0, "Ybase", out_bf16=True)
    q = make_problem(T + d_out, d_out, d_in, lens, [L, I, L, N, L], ranks)       # its input gradient has the same product
    for conv1d in (False, True):
        n, dX = launches(lambda: gh.backward_input(off, q["ads"], q["dY"], q["W"], conv1d=conv1d), 8 + 2 + (not conv1d))
        assert n == 1
        check_dx(gh.bf16_to_f64(dX)[rows], off, oracle_ads(q["ads"]), q["dY"], q["W"], "dX", rows=rows)
    if parts > 1:                        # one byte too few for the partial tiles, and a call whose tiles cannot be split: the 128x128 tile
        X, W = gh.to_dev(p["X"]), gh.to_dev(p["W"])
        for ws, want_base, variant in ((need - 1, False, 2), (need, True, 4 + 2)):
            Y = torch.full((T, d_out), float("nan"), device="cuda", dtype=torch.bfloat16)
            Yb = torch.empty_like(Y) if want_base else None
            buf = torch.empty(ws, device="cuda", dtype=torch.uint8)
            call = lambda: sb.symb_base_linear_fwd(gh.handle(), plain, X, W, None, Y, Yb, buf)  # noqa: B023,E731
            assert launches(call, variant)[0] == 1 and launches(call, variant + 8)[0] == 0
            check_y(gh.bf16_to_f64(Y[rows]), off, oracle_ads(base), p["X"], p["W"], None, f"Y in {ws} bytes", rows=rows)


def test_tall_tile_with_empty_halves():
    test_tall_tile(600, 3080, 6536, 1, [16, 5])          # 156 tiles, a third of them with 88 rows; 260 of 128x128


@pytest.mark.parametrize("lens,d_in,d_out,room", [
    ([1] * 2000, 4096, 4096, False),                     # no room for the terms: 256 steps in a tile of 256 rows
    ([1] * 276 + [124], 3072, 11008, True)])             # the second tile's 20 steps are too few for memory beside 276 rows of terms
def test_not_with_many_steps_left(lens, d_in, d_out, room):
    """Steps of short segments that do not come from memory count in full: the 128x128 tile."""
    p = make_problem(len(lens), d_in, d_out, lens, [L] * 276 + [N] if room else [L], [16])
    off = p["off"]
    dev = gh.upload_adapters(p["ads"], d_in, d_out, grads=False)
    b = sb.Batch(d_in, d_out, off, dev.descs)
    X, W = gh.to_dev(p["X"]), gh.to_dev(p["W"])
    Y = torch.empty(p["T"], d_out, device="cuda", dtype=torch.bfloat16)
    ws = gh.workspace(b, sb.SYMB_OP_FWD)
    if not room:
        ws = ws[:p["T"] * 2 * 16 * 2]                    # Hs alone
    call = lambda: sb.symb_base_linear_fwd(gh.handle(), b, X, W, None, Y, None, ws)  # noqa: E731
    full = 4 if room else 0
    assert launches(call, 2 + full)[0] == 1 and launches(call, 8 + 2 + full)[0] == 0
    rows = synth.sample_rows(off, 6, f"left{d_in}", block=128)[:64]
    check_y(gh.bf16_to_f64(Y[rows]), off, oracle_ads(p["ads"]), p["X"], p["W"], None, "Y", rows=rows)

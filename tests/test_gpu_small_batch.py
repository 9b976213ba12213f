"""Calls of at most 64 rows (the weight-streaming kernels): row counts around the blocks of 16 and the limit, inner and output
widths around the slices and tiles, ranks that are and are not multiples of 4 and 8, an adapter matrix that is not 16-byte
aligned, and the workspace hand-over to a gradient call."""
import numpy as np
import pytest
import torch

import gpu_harness as gh
import oracle
import synth
import test_gpu_parity as tp
from helpers import assert_close, check_dx, check_y
from paper_2507_03220_amd import binding as sb
from test_gpu_parity import L, I, N, make_problem, oracle_ads

pytestmark = pytest.mark.gpu
tp.gh, tp.sb = gh, sb                    # what its problem maker uses


@pytest.mark.parametrize("dims", [(8, 8), (40, 136), (136, 40), (72, 264), (584, 520), (2056, 128)])
@pytest.mark.parametrize("lens", [[16], [17], [1] * 32, [33], [20, 1, 0, 43], [64], [63, 2]])
def test_edges_of_rows_and_widths(dims, lens):
    d_in, d_out = dims
    p = make_problem(sum(lens) + d_in, d_in, d_out, lens, [L, L, I, L, N, 3], [1, 16, 12, 128, 40, 5, 64, 99])
    off, oads = p["off"], oracle_ads(p["ads"])
    base = [gh.HostAdapter() for _ in lens]
    for conv1d in (False, True):
        for want_base in (False, True):
            Y, _ = gh.forward(off, p["ads"], p["X"], p["W"], p["bias"], want_base=want_base, conv1d=conv1d)
            check_y(gh.bf16_to_f64(Y), off, oads, p["X"], p["W"], p["bias"], f"Y {dims} {lens} conv1d={conv1d}")
        Y, _ = gh.forward(off, base, p["X"], p["W"], p["bias"], want_base=False, conv1d=conv1d)        # no adapters: finished in one kernel
        check_y(gh.bf16_to_f64(Y), off, oracle_ads(base), p["X"], p["W"], p["bias"], f"base Y {dims} {lens} conv1d={conv1d}")
        for base_only in (False, True):
            dX = gh.backward_input(off, p["ads"], p["dY"], p["W"], base_only=base_only, conv1d=conv1d)
            check_dx(gh.bf16_to_f64(dX), off, oads, p["dY"], p["W"], f"dX {dims} {lens} conv1d={conv1d}", base_only=base_only)


@pytest.mark.parametrize("lens", [[1], [5, 0, 12, 15], [40, 0, 24]])
@pytest.mark.parametrize("dims", [(520, 2048), (2000, 648)])
def test_calls_without_lora_in_every_form(dims, lens):
    """Base products finished in the streaming kernel itself (K up to 2048), the same calls in the tiled kernels, and which of them runs:
    matrices, a buffer per client, one buffer for input and output, noise effects taken off."""
    d_in, d_out = dims
    p = make_problem(700 + d_in + sum(lens), d_in, d_out, lens, [I, N], [1])
    off, T, S, oads, h = p["off"], p["T"], len(lens), oracle_ads(p["ads"]), gh.handle()
    _, Yr = oracle.forward(off, oads, p["X"], p["W"], p["bias"])
    dXr = oracle.backward_input(off, oads, p["dY"], p["W"])
    rng = np.random.default_rng(17)
    neff = [None if off[i + 1] == off[i] else synth.f32_to_bf16_bits(rng.standard_normal((1 if i % 2 else lens[i], d_out)).astype(np.float32)) for i in range(S)]
    Ydr = oracle.forward_denoise(off, oads, p["X"], p["W"], p["bias"], neff)
    Xd, Gd, bd = gh.to_dev(p["X"]), gh.to_dev(p["dY"]), gh.to_dev(p["bias"])
    dev = gh.upload_adapters(p["ads"], d_in, d_out, grads=False)

    def pieces(M, width):                # a buffer per segment, in one arena of rows wide enough for both sides
        arena = torch.full((T + S, max(dims)), float("nan"), device="cuda", dtype=torch.bfloat16)
        v = [arena[off[i] + i:off[i + 1] + i].view(-1)[:lens[i] * width].view(lens[i], width) if lens[i] else None for i in range(S)]
        if M is not None:
            for i in range(S):
                if lens[i]:
                    v[i].copy_(M[off[i]:off[i + 1]])
        return v, lambda w: [None if x is None else torch.as_strided(x, (x.shape[0], w), (w, 1)) for x in v]

    def joined(v):
        return gh.bf16_to_f64(torch.cat([x for x in v if x is not None]))
    try:
        for conv1d in (0, 1):
            b = sb.Batch(d_in, d_out, off, dev.descs, conv1d)
            Wd = gh.weight_to_dev(p["W"], bool(conv1d))
            fwd_ws, bwd_ws = gh.workspace(b, sb.SYMB_OP_FWD), gh.workspace(b, sb.SYMB_OP_BWD_INPUT)
            for on in (1, 0):
                sb.symb_debug_set_option(h, sb.SYMB_OPT_SMALL_BATCH_KERNELS, on)
                Y, Yd = (torch.full((T, d_out), float("nan"), device="cuda", dtype=torch.bfloat16) for _ in range(2))
                dX = torch.full((T, d_in), float("nan"), device="cuda", dtype=torch.bfloat16)
                xin, _ = pieces(Xd, d_in)
                yout, _ = pieces(None, d_out)
                xy, xy_as = pieces(Xd, d_in)
                gin, _ = pieces(Gd, d_out)
                gout, _ = pieces(None, d_in)
                gx, gx_as = pieces(Gd, d_out)
                calls = {
                    "Y": lambda: sb.symb_base_linear_fwd(h, b, Xd, Wd, bd, Y, None, fwd_ws),
                    "denoised": lambda: sb.symb_base_linear_fwd_denoise(h, b, Xd, Wd, bd, [gh.to_dev(n) for n in neff], Yd, fwd_ws),
                    "seg Y": lambda: sb.symb_base_linear_fwd_seg(h, b, xin, Wd, bd, yout, fwd_ws),
                    "in-place Y": lambda: sb.symb_base_linear_fwd_seg(h, b, xy, Wd, bd, xy_as(d_out), gh.workspace(b, sb.SYMB_OP_FWD_INPLACE)),
                    "dX": lambda: sb.symb_base_linear_bwd_input(h, b, Gd, Wd, dX, sb.SYMB_BWD_FULL, bwd_ws),
                    "seg dX": lambda: sb.symb_base_linear_bwd_input_seg(h, b, gin, Wd, gout, sb.SYMB_BWD_FULL, bwd_ws),
                    "in-place dX": lambda: sb.symb_base_linear_bwd_input_seg(h, b, gx, Wd, gx_as(d_in), sb.SYMB_BWD_FULL, gh.workspace(b, sb.SYMB_OP_BWD_INPUT_INPLACE))}
                for name, call in calls.items():
                    forward = "Y" in name or name == "denoised"
                    across = forward == bool(conv1d)             # the weight is read across its rows: tiled above 32 rows
                    streams = bool(on) and (T <= 32 or not across)
                    ran = gh.gemm_launches(call)
                    assert (ran == {}) == streams, f"{name} conv1d={conv1d} on={on}: {ran}"
                torch.cuda.synchronize()
                tag = f"conv1d={conv1d} on={on}"
                assert_close(gh.bf16_to_f64(Y), Yr, f"Y {tag}", out_bf16=True)
                assert_close(gh.bf16_to_f64(Yd), Ydr, f"denoised {tag}", out_bf16=True)
                assert_close(joined(yout), Yr, f"seg Y {tag}", out_bf16=True)
                assert_close(joined(xy_as(d_out)), Yr, f"in-place Y {tag}", out_bf16=True)
                for got, what in ((gh.bf16_to_f64(dX), "dX"), (joined(gout), "seg dX"), (joined(gx_as(d_in)), "in-place dX")):
                    assert_close(got, dXr, f"{what} {tag}", out_bf16=True)
    finally:
        sb.symb_debug_set_option(h, sb.SYMB_OPT_SMALL_BATCH_KERNELS, 1)


def test_workspaces_at_their_limits():
    """The exact figure takes the streaming kernels; one byte less the tiled one, down to H alone; less than that is refused."""
    lens, d_in, d_out = [60, 4], 4104, 520
    p = make_problem(77, d_in, d_out, lens, [L, I], [8])
    off, oads, h = p["off"], oracle_ads(p["ads"]), gh.handle()
    dev = gh.upload_adapters(p["ads"], d_in, d_out, grads=False)
    b = sb.Batch(d_in, d_out, off, dev.descs)
    X, W, bias = gh.to_dev(p["X"]), gh.to_dev(p["W"]), gh.to_dev(p["bias"])
    ws = gh.workspace(b, sb.SYMB_OP_FWD)
    hs = p["T"] * 2 * 16 * 2
    for n, streams in ((ws.numel(), True), (ws.numel() - 1, False), (hs, False)):
        Y = torch.full((p["T"], d_out), float("nan"), device="cuda", dtype=torch.bfloat16)
        ran = gh.gemm_launches(lambda: sb.symb_base_linear_fwd(h, b, X, W, bias, Y, None, ws[:n]))
        assert (ran == {}) == streams, f"{n} bytes: {ran}"
        check_y(gh.bf16_to_f64(Y), off, oads, p["X"], p["W"], p["bias"], f"Y with {n} bytes")
    with pytest.raises(sb.SymbError) as e:
        sb.symb_base_linear_fwd(h, b, X, W, bias, Y, None, ws[:hs - 1])
    assert e.value.status == sb.SYMB_ERR_WORKSPACE_TOO_SMALL


@pytest.mark.parametrize("d_in,d_out,lens", [(5000, 10248, [1, 9, 6]),       # 40 tiles in 5 long ranges: one buffer
                                             (33000, 2056, [3, 9]), (33000, 2056, [20, 17])])      # more tiles than CUs
def test_large_n_contiguous_weights(d_in, d_out, lens):
    p = make_problem(d_in + len(lens), d_in, d_out, lens, [L, N, L], [16, 40])
    oads = oracle_ads(p["ads"])
    for base_only in (False, True):
        dX = gh.backward_input(p["off"], p["ads"], p["dY"], p["W"], base_only=base_only)
        check_dx(gh.bf16_to_f64(dX), p["off"], oads, p["dY"], p["W"], f"dX base_only={base_only}", base_only=base_only)


@pytest.mark.parametrize("rank", [4, 12, 20])
def test_adapter_matrix_off_its_16_byte_alignment(rank):
    """B of a rank that is no multiple of 8 need only be 2-byte aligned."""
    p = make_problem(rank, 520, 392, [5, 30], [L], [rank])
    off, oads = p["off"], oracle_ads(p["ads"])
    dev = gh.upload_adapters(p["ads"], 520, 392, grads=False)
    for d, shift in zip(dev.descs, (1, 3)):
        room = torch.zeros(d.B.numel() + 8, device="cuda", dtype=torch.bfloat16)
        room[shift:shift + d.B.numel()] = d.B.reshape(-1)
        d.B = room[shift:shift + d.B.numel()]
    b = sb.Batch(520, 392, off, dev.descs)
    Xd, Gd, Wd = gh.to_dev(p["X"]), gh.to_dev(p["dY"]), gh.to_dev(p["W"])
    Y = torch.empty(35, 392, device="cuda", dtype=torch.bfloat16)
    dX = torch.empty(35, 520, device="cuda", dtype=torch.bfloat16)
    sb.symb_base_linear_fwd(gh.handle(), b, Xd, Wd, None, Y, None, gh.workspace(b, sb.SYMB_OP_FWD))
    sb.symb_base_linear_bwd_input(gh.handle(), b, Gd, Wd, dX, sb.SYMB_BWD_FULL, gh.workspace(b, sb.SYMB_OP_BWD_INPUT))
    torch.cuda.synchronize()
    check_y(gh.bf16_to_f64(Y), off, oads, p["X"], p["W"], None, "Y")
    check_dx(gh.bf16_to_f64(dX), off, oads, p["dY"], p["W"], "dX")


@pytest.mark.parametrize("rank", [8, 12, 20, 40, 100])
@pytest.mark.parametrize("lens", [[5, 30], [1] * 150])              # the streaming kernels; short segments of a tiled call
def test_an_infinity_in_the_last_row_of_a(rank, lens):
    """The rank rows that pad A_i to whole blocks count as zero: an infinity in its last row stays one in dX.  (In a tiled call it meets value
    and residual of dH, which may differ in sign: not finite, in this column of this segment alone.)"""
    p = make_problem(rank, 392, 264, lens, [L], [rank])
    p["ads"][0].A[rank - 1, 3] = 0x7f80
    off, oads = p["off"], oracle_ads(p["ads"])
    got = gh.bf16_to_f64(gh.backward_input(off, p["ads"], p["dY"], p["W"]))
    ref = oracle.backward_input(off, oads, p["dY"], p["W"])
    assert np.isinf(ref[:lens[0], 3]).all() and not np.isfinite(got[:lens[0], 3]).any()
    assert p["T"] > 64 or np.array_equal(got[:lens[0], 3], ref[:lens[0], 3])
    got[:lens[0], 3] = ref[:lens[0], 3] = 0.0
    assert_close(got, ref, f"dX rank {rank}", out_bf16=True)


@pytest.mark.parametrize("lens", [[16], [9, 30, 0, 25]])
def test_gradients_take_hs_and_dh_from_the_streaming_calls(lens):
    p = make_problem(77, 584, 392, lens, [L], [16, 5, 8, 40])
    off, oads = p["off"], oracle_ads(p["ads"])
    dev = gh.upload_adapters(p["ads"], 584, 392, grads=True)
    b = sb.Batch(584, 392, off, dev.descs)
    ws = torch.full((max(sb.symb_workspace_bytes(b, op) for op in range(3)),), 0x7f, device="cuda", dtype=torch.uint8)
    Xd, Gd, Wd = gh.to_dev(p["X"]), gh.to_dev(p["dY"]), gh.to_dev(p["W"])
    Y, dX = torch.empty(p["T"], 392, device="cuda", dtype=torch.bfloat16), torch.empty(p["T"], 584, device="cuda", dtype=torch.bfloat16)
    h = gh.handle()
    sb.symb_base_linear_fwd(h, b, Xd, Wd, None, Y, None, ws)
    sb.symb_base_linear_bwd_input(h, b, Gd, Wd, dX, sb.SYMB_BWD_FULL, ws)
    sb.symb_adapter_grad(h, b, Xd, Gd, None, sb.SYMB_GRAD_REUSE_DH | sb.SYMB_GRAD_REUSE_HS, ws)
    torch.cuda.synchronize()
    for i, n in enumerate(lens):
        dAr, dBr = oracle.lora_grad(off, oads, p["X"], p["dY"], i)
        assert_close(dev.descs[i].dA.cpu().numpy(), dAr, f"dA[{i}]")
        assert_close(dev.descs[i].dB.cpu().numpy(), dBr, f"dB[{i}]")
    # ... and the input gradient the dH a gradient call left
    sb.symb_adapter_grad(h, b, Xd, Gd, None, sb.SYMB_GRAD_OVERWRITE, ws)
    dX.fill_(float("nan"))
    sb.symb_base_linear_bwd_input(h, b, Gd, Wd, dX, sb.SYMB_BWD_REUSE_DH, ws)
    torch.cuda.synchronize()
    check_dx(gh.bf16_to_f64(dX), off, oads, p["dY"], p["W"], "dX from the gradient call's dH")


@pytest.mark.parametrize("T,d_in,d_out,tile,parts", [
    (2048, 264, 4096, 128, 1), (4096, 328, 2000, 128, 1),         # 128 tiles of 256x256, as 512 of 128x128
    (2048, 4680, 4096, 256, 2),                                   # above that rule's inner dimension: every tile in two parts
    (100, 2056, 1032, 128, 4), (397, 8320, 520, 128, 8),
    (397, 8200, 3400, 128, 4), (397, 12296, 2600, 128, 6)])       # parts of 64 stages: twice two and twice three
def test_tile_and_split_rules_of_mid_sized_batches(T, d_in, d_out, tile, parts):
    """The tile and the K parts a product of each rule runs in (by the partial tiles' bytes), and its results."""
    plain = sb.Batch(d_in, d_out, [0, T], [sb.Adapter()])
    partial = -(-T // tile) * -(-d_out // tile) * parts * tile * tile * 4 if parts > 1 else 0
    assert sb.symb_workspace_bytes(plain, sb.SYMB_OP_FWD) == partial
    p = make_problem(T, d_in, d_out, [T // 2, T // 4, T - T // 2 - T // 4], [L, I, N], [16])
    rows = synth.sample_rows(p["off"], 12, f"mid{T}", block=128)
    oads = oracle_ads(p["ads"])
    for conv1d in (False, True):
        res = []
        ran = gh.gemm_launches(lambda: res.append(gh.forward(p["off"], p["ads"], p["X"], p["W"], p["bias"], want_base=False, conv1d=conv1d)[0]))
        assert ran == {conv1d + (2 if tile == 128 else 0) + 4: 1}
        check_y(gh.bf16_to_f64(res[0])[rows], p["off"], oads, p["X"], p["W"], p["bias"], "Y", rows=rows)


@pytest.mark.parametrize("T,d_in,d_out,tile", [       # 0: 256x256, 2: 128x128, 2 + 8: 256x128
    (2048, 4608, 4096, 10), (2048, 3064, 4096, 2), (2048, 4616, 4096, 0), (1800, 512, 4096, 2), (1024, 4096, 8192, 10), (1024, 3064, 8192, 2), (1024, 4104, 8192, 0),
    (512, 3072, 16384, 10), (512, 3064, 16384, 2), (512, 4096, 16384, 0), (3700, 512, 2056, 2), (3840, 512, 2184, 0), (1792, 8192, 4096, 10),
    (8770, 9176, 768, 2), (8770, 9216, 768, 10), (9600, 9176, 768, 10), (2100, 9176, 2816, 10)])          # many rows off the lines: from 220 tiles of 256x128 on, or with more columns
def test_tile_size(T, d_in, d_out, tile):
    """Which tile a product runs in, around 128 tiles of 256x256, 512 of 128x128 and an inner dimension of 3072."""
    X, W, Y = (torch.zeros(s, device="cuda", dtype=torch.bfloat16) for s in ((T, d_in), (d_out, d_in), (T, d_out)))
    for conv1d in (0, 1):
        b = sb.Batch(d_in, d_out, [0, T], [sb.Adapter()], conv1d)
        ws = gh.workspace(b, sb.SYMB_OP_FWD)
        ran = gh.gemm_launches(lambda: sb.symb_base_linear_fwd(gh.handle(), b, X, W, None, Y, None, ws))
        assert ran == {conv1d + tile: 1}


@pytest.mark.parametrize("T,d_in,d_out,tile", [
    (731, 6144, 6144, 10), (731, 3064, 6144, 2), (600, 8192, 6656, 10), (600, 8192, 6528, 2),          # 288 and 260 tiles of 128x128, 255
    (2536, 12544, 1904, 10), (2536, 12528, 1904, 2), (8761, 4864, 472, 2), (5000, 4864, 904, 10)])     # rows off the lines, few columns
def test_tile_size_where_small_tiles_are_more_than_the_cus(T, d_in, d_out, tile):
    test_tile_size(T, d_in, d_out, tile)


@pytest.mark.parametrize("d_in,d_out,tile", [(264, 392, 128), (2056, 264, 128), (200, 9480, 256)])     # whole, split over K, large tiles
def test_short_segments_of_a_larger_batch(d_in, d_out, tile):
    """LoRA terms of short segments are added from memory where a row tile holds many of their steps: scattered over the tiles,
    across a tile's edge, beside long segments, empty ones and other kinds; with the pre-adapter output; in both directions."""
    lens = [1] * 9 + [300, 16, 3, 0, 17] + [1, 2] * 8 + [200, 1, 40] + [1] * 5 + [5, 16, 260]
    kinds = [L, L, L, I, L, N, L]
    p = make_problem(5 + d_out, d_in, d_out, lens, kinds, [16, 128, 5, 40, 8, 33])
    off, oads = p["off"], oracle_ads(p["ads"])
    b = sb.Batch(d_in, d_out, off, gh.upload_adapters(p["ads"], d_in, d_out, grads=False).descs)
    steps_only = p["T"] * 2 * 128 * 2 + sb.symb_workspace_bytes(sb.Batch(d_in, d_out, [0, p["T"]], [sb.Adapter()]), sb.SYMB_OP_FWD)
    assert sb.symb_workspace_bytes(b, sb.SYMB_OP_FWD) > steps_only + 16 * d_out * 4           # room for terms of more than 16 rows
    small = 2 if tile == 128 else 0

    def run(call):
        res = []
        ran = gh.gemm_launches(lambda: res.append(call()))
        assert len(ran) == 1 and next(iter(ran)) & 2 == small
        return res[0]
    for conv1d in (False, True):
        for want_base in (False, True):
            Y, Yb = run(lambda: gh.forward(off, p["ads"], p["X"], p["W"], p["bias"], want_base=want_base, conv1d=conv1d))
            Y0r, _ = check_y(gh.bf16_to_f64(Y), off, oads, p["X"], p["W"], p["bias"], f"Y conv1d={conv1d}")
            if want_base:
                assert_close(gh.bf16_to_f64(Yb), Y0r, "Ybase", out_bf16=True)
    q = make_problem(6 + d_out, d_out, d_in, lens, kinds, [16, 128, 5, 40, 8, 33])
    for conv1d in (False, True):
        dX = run(lambda: gh.backward_input(off, q["ads"], q["dY"], q["W"], conv1d=conv1d))
        check_dx(gh.bf16_to_f64(dX), off, oracle_ads(q["ads"]), q["dY"], q["W"], f"dX conv1d={conv1d}")


def test_timed_work_of_a_gemm_leaves_out_the_terms_from_memory():
    lens = [1] * 40 + [300]
    p = make_problem(8, 264, 392, lens, [L], [16] * 40 + [8])
    dev = gh.upload_adapters(p["ads"], 264, 392, grads=False)
    b = sb.Batch(264, 392, p["off"], dev.descs)
    X, W = gh.to_dev(p["X"]), gh.to_dev(p["W"])
    Y = torch.empty(p["T"], 392, device="cuda", dtype=torch.bfloat16)
    full = gh.workspace(b, sb.SYMB_OP_FWD)
    for ws, rows in ((full, 300 * 8), (full[:p["T"] * 2 * 16 * 2], 40 * 16 + 300 * 8)):          # with the terms' region, and without
        sb.symb_debug_gemm_timing_enable(gh.handle(), 1)
        try:
            sb.symb_base_linear_fwd(gh.handle(), b, X, W, None, Y, None, ws)
            work = sum(sb.symb_debug_gemm_timing_read(gh.handle(), v)[2] for v in range(8))
        finally:
            sb.symb_debug_gemm_timing_enable(gh.handle(), 0)
        assert work == 2.0 * 392 * (p["T"] * 264 + rows)


@pytest.mark.parametrize("d_in,d_out", [(4096, 4096), (6144, 2056)])         # 128x128 tiles in five parts; 256x128 tiles in two
def test_terms_of_a_call_with_pre_adapter_output_fit_the_reported_workspace(d_in, d_out):
    """Such a call does not split: its chains of steps are as long as they are, and it selects more rows for memory than the figure's split call."""
    lens = [1] * 160 + ([1100] if d_in == 6144 else [])
    p = make_problem(d_in, d_in, d_out, lens, [L] * 160 + [N], [16])
    off, oads = p["off"], oracle_ads(p["ads"])
    dev = gh.upload_adapters(p["ads"], d_in, d_out, grads=False)
    b = sb.Batch(d_in, d_out, off, dev.descs)
    X, W, dY = gh.to_dev(p["X"]), gh.to_dev(p["W"]), gh.to_dev(p["dY"])
    rows = synth.sample_rows(off, 12, f"base{d_in}", block=128)
    for base in (False, True):
        for back in (False, True):
            k, n = (d_out, d_in) if back else (d_in, d_out)
            out = torch.empty(p["T"], n, device="cuda", dtype=torch.bfloat16)
            extra = torch.empty_like(out) if base else None
            ws = torch.empty(sb.symb_workspace_bytes(b, sb.SYMB_OP_BWD_INPUT if back else sb.SYMB_OP_FWD), device="cuda", dtype=torch.uint8)
            sb.symb_debug_gemm_timing_enable(gh.handle(), 1)
            try:
                if back:
                    sb.symb_base_linear_bwd_input_ex(gh.handle(), b, dY, W, out, extra, sb.SYMB_BWD_FULL, ws)
                else:
                    sb.symb_base_linear_fwd(gh.handle(), b, X, W, None, out, extra, ws)
                work = sum(sb.symb_debug_gemm_timing_read(gh.handle(), v)[2] for v in range(8))
            finally:
                sb.symb_debug_gemm_timing_enable(gh.handle(), 0)
            left = 32 if not base and d_in == 4096 else 0            # (the second row tile of a call in five parts keeps its 32 steps)
            assert work == 2.0 * n * (p["T"] * k + left * 16), (base, back)
            if back:
                check_dx(gh.bf16_to_f64(out[rows]), off, oads, p["dY"], p["W"], "dX", rows=rows)
            else:
                check_y(gh.bf16_to_f64(out[rows]), off, oads, p["X"], p["W"], None, "Y", rows=rows)


def test_short_segments_beside_more_rows_than_their_masks_have_room_for():
    """The terms of short segments cost 36 bytes of descriptors per row tile: a batch of 3.4 million rows, whose other descriptors fit
    the 2 MiB slot, is accepted and its short segments keep their steps inside the GEMM."""
    lens = [3_400_000] + [1] * 20
    p = make_problem(31, 8, 8, lens, [L], [16])
    off, oads = p["off"], oracle_ads(p["ads"])
    rows = np.concatenate([np.arange(0, 3_400_000, 170_001), np.arange(3_399_990, p["T"])])
    Y, _ = gh.forward(off, p["ads"], p["X"], p["W"], p["bias"], want_base=False)
    check_y(gh.bf16_to_f64(Y[rows]), off, oads, p["X"], p["W"], p["bias"], "Y", rows=rows)
    dX = gh.backward_input(off, p["ads"], p["dY"], p["W"])
    check_dx(gh.bf16_to_f64(dX[rows]), off, oads, p["dY"], p["W"], "dX", rows=rows)


@pytest.mark.parametrize("T,d_in,d_out,short", [(397, 11008, 4096, 0),       # 128 tiles: four parts do not fit beside H, two do
                                                (2560, 4096, 7168, 600)])    # a last round in three parts, which do not fit behind the short segments' terms
def test_k_split_within_the_static_scratch(T, d_in, d_out, short):
    """A workspace of a fixed size too small for all optional regions still splits the inner dimension: the bits show it, as a split sums in
    another order."""
    lens = [T - short] + [1] * short
    p = make_problem(T, d_in, d_out, lens, [L] if not short else [N] + [L] * short, [16])
    dev = gh.upload_adapters(p["ads"], d_in, d_out, grads=False)
    b = sb.Batch(d_in, d_out, p["off"], dev.descs)
    assert sb.symb_workspace_bytes(b, sb.SYMB_OP_FWD) > sb.SYMB_STATIC_SCRATCH_BYTES
    Xd, Wd = gh.to_dev(p["X"]), gh.to_dev(p["W"])
    got = []
    try:
        for split in (1, 0):
            sb.symb_debug_set_option(gh.handle(), sb.SYMB_OPT_K_SPLIT, split)
            Y = torch.empty(T, d_out, device="cuda", dtype=torch.bfloat16)
            sb.symb_base_linear_fwd_static(gh.handle(), b, Xd, Wd, None, Y, None)
            torch.cuda.synchronize()
            got.append(Y)
    finally:
        sb.symb_debug_set_option(gh.handle(), sb.SYMB_OPT_K_SPLIT, 1)
    assert not torch.equal(got[0].view(torch.int16), got[1].view(torch.int16)), "not split"
    rows = synth.sample_rows(p["off"], 1, f"static{T}", block=128)[:48]
    check_y(gh.bf16_to_f64(got[0][rows]), p["off"], oracle_ads(p["ads"]), p["X"], p["W"], None, "Y", rows=rows)

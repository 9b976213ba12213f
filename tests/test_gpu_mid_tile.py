"""Products of small layers in tiles of 32 rows: row counts around the tile, widths around 64 and 128 columns, inner dimensions around the slices (64 and 32 k) and with
a remainder, every epilogue, LoRA ranks of several steps, buffers per client, in both directions and weight layouts."""
import numpy as np
import pytest
import torch

import gpu_harness as gh
from helpers import check_dx, check_y
from paper_2507_03220_amd import binding as sb
from test_gpu_parity import I, L, N, make_problem, oracle_ads
from test_gpu_tall_tile import launches
import test_gpu_parity as tp

pytestmark = pytest.mark.gpu
tp.gh, tp.sb = gh, sb                    # what its problem maker uses


@pytest.mark.parametrize("d_in,d_out", [(8, 136), (72, 64), (264, 200), (776, 768), (1536, 392), (2040, 264)])
@pytest.mark.parametrize("lens,ranks", [([65], [16]), ([30, 0, 34, 17, 16], [8, 5, 40]), ([100, 1, 96], [128, 12]), ([260], [33])])
def test_small_layers(d_in, d_out, lens, ranks):
    p = make_problem(sum(lens) + d_in, d_in, d_out, lens, [L, I, L, N, 3], ranks)
    off, oads, T = p["off"], oracle_ads(p["ads"]), p["T"]
    base = [gh.HostAdapter() for _ in lens]
    for conv1d in (False, True):
        n, (Y, _) = launches(lambda: gh.forward(off, p["ads"], p["X"], p["W"], p["bias"], want_base=False, conv1d=conv1d), 16 + 4 + 2 + conv1d)
        assert n == (not conv1d or d_in < 1536)          # (an N-contiguous weight keeps 128x128 tiles in K parts)
        check_y(gh.bf16_to_f64(Y), off, oads, p["X"], p["W"], p["bias"], f"Y conv1d={conv1d}")
        n, (Y, _) = launches(lambda: gh.forward(off, base, p["X"], p["W"], None, want_base=False, conv1d=conv1d), 16 + 2 + conv1d)
        assert n == (not conv1d or d_in < 1536)          # (an N-contiguous weight keeps 128x128 tiles in K parts)
        check_y(gh.bf16_to_f64(Y), off, oracle_ads(base), p["X"], p["W"], None, f"plain Y conv1d={conv1d}")
        for base_only in (False, True):
            dX = gh.backward_input(off, p["ads"], p["dY"], p["W"], base_only=base_only, conv1d=conv1d)
            check_dx(gh.bf16_to_f64(dX), off, oads, p["dY"], p["W"], f"dX conv1d={conv1d} {base_only}", base_only=base_only)
    # a buffer per client gives the bits of the flat call
    dev = gh.upload_adapters(p["ads"], d_in, d_out, grads=False)
    b = sb.Batch(d_in, d_out, off, dev.descs)
    X, W, bias = gh.to_dev(p["X"]), gh.to_dev(p["W"]), gh.to_dev(p["bias"])
    Y, _ = gh.forward(off, p["ads"], p["X"], p["W"], p["bias"], want_base=False)
    Z = torch.full((T, d_out), float("nan"), device="cuda", dtype=torch.bfloat16)
    cut = [(a, c) if c > a else None for a, c in zip(off, off[1:])]
    seg = lambda t: [t[c[0]:c[1]] if c else None for c in cut]  # noqa: E731
    n, _ = launches(lambda: sb.symb_base_linear_fwd_seg(gh.handle(), b, seg(X), W, bias, seg(Z), gh.workspace(b, sb.SYMB_OP_FWD)), 16 + 4 + 2)
    assert n == 1 and torch.equal(Y.view(torch.int16), Z.view(torch.int16))


def test_an_infinity_stays_out_of_other_blocks_of_rows():
    """A LoRA step meets only the blocks of 16 rows that hold rows of its segment."""
    p = make_problem(3, 264, 200, [16, 60], [L], [8])
    p["ads"][0].B[3] = 0x7f80
    got = gh.bf16_to_f64(gh.forward(p["off"], p["ads"], p["X"], p["W"], p["bias"], want_base=False)[0])
    assert not np.isfinite(got[:16, 3]).any() and np.isfinite(np.delete(got, 3, 1)).all() and np.isfinite(got[16:]).all()


@pytest.mark.parametrize("lens", [[4] * 7 + [44], [1] * 7 + [58, 30], [16] * 5 + [3, 2]])
def test_short_segments_that_share_a_tile(lens):
    """As many as the tiles of 32 rows take: their LoRA steps are dealt out over the wavefronts."""
    p = make_problem(len(lens) + sum(lens), 264, 200, lens, [L], [8, 16, 5])
    for conv1d in (False, True):
        n, (Y, _) = launches(lambda: gh.forward(p["off"], p["ads"], p["X"], p["W"], p["bias"], want_base=False, conv1d=conv1d), 16 + 4 + 2 + conv1d)
        assert n == 1
        check_y(gh.bf16_to_f64(Y), p["off"], oracle_ads(p["ads"]), p["X"], p["W"], p["bias"], f"Y conv1d={conv1d}")
        check_dx(gh.bf16_to_f64(gh.backward_input(p["off"], p["ads"], p["dY"], p["W"], conv1d=conv1d)), p["off"], oracle_ads(p["ads"]), p["dY"], p["W"], "dX")


@pytest.mark.parametrize("lens,kinds,ranks,order", [
    ([4, 7, 9, 12, 16, 5, 11, 40, 3, 24], [L, L, L, N, L, L, I, L, L, L], [8, 16, 5], [8, 2, 5, 0, 9, 3, 7, 1, 6, 4]),
    ([4, 7, 40, 12, 24, 30], [L, L, L, N, L, L], [8, 16, 40, 33, 100], [5, 2, 0, 3, 4, 1])])
def test_a_row_hangs_on_its_own_segment(lens, kinds, ranks, order):
    """Clients that share tiles, in another order: every row has the same bits, in both directions and weight layouts."""
    p = make_problem(31 + len(ranks), 264, 200, lens, kinds, ranks)
    off = p["off"]
    idx = np.concatenate([np.arange(off[i], off[i + 1]) for i in order])
    noff = np.concatenate([[0], np.cumsum([lens[i] for i in order])]).astype(np.int32)
    ads = [p["ads"][i] for i in order]
    X, dY = np.ascontiguousarray(p["X"][idx]), np.ascontiguousarray(p["dY"][idx])
    for conv1d in (False, True):
        n, (Y, _) = launches(lambda: gh.forward(off, p["ads"], p["X"], p["W"], p["bias"], want_base=False, conv1d=conv1d), 16 + 4 + 2 + conv1d)
        assert n == 1
        again, _ = gh.forward(noff, ads, X, p["W"], p["bias"], want_base=False, conv1d=conv1d)
        np.testing.assert_array_equal(gh.bf16_bits(again), gh.bf16_bits(Y)[idx])
        dX = gh.backward_input(off, p["ads"], p["dY"], p["W"], conv1d=conv1d)
        np.testing.assert_array_equal(gh.bf16_bits(gh.backward_input(noff, ads, dY, p["W"], conv1d=conv1d)), gh.bf16_bits(dX)[idx])

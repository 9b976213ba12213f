"""Host-side checks of libsymb.so that need no GPU: every declared symbol is exported,
argument validation, the segment planner and the row->segment map (bit-exact against
the oracle's map).  No compute entry point is called here."""
import ctypes as C
import os
import re

import numpy as np
import pytest

import oracle
from paper_2507_03220_amd import binding as sb

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.fixture(scope="module", autouse=True)
def _built():
    from paper_2507_03220_amd import build
    build.build(force=False)


def _declared_symbols():
    text = ""
    inc = os.path.join(ROOT, "include")
    for f in sorted(os.listdir(inc)):
        if f.endswith(".h"):
            text += open(os.path.join(inc, f)).read()
    text = re.sub(r"/\*.*?\*/", "", text, flags=re.S)
    return sorted(set(re.findall(r"\b(symb_[a-z_0-9]+)\s*\(", text)))


def test_every_declared_symbol_is_exported():
    names = _declared_symbols()
    assert set(names) == set(sb.EXPORTS), names
    l = sb.lib()
    for n in names:
        assert getattr(l, n) is not None


def test_status_strings():
    l = sb.lib()
    assert l.symb_status_string(0) == b"SYMB_OK"
    assert l.symb_status_string(2) == b"SYMB_ERR_BAD_SEGMENTS"


def _batch(off, ads=None, d_in=64, d_out=64):
    ads = ads if ads is not None else [sb.Adapter() for _ in range(len(off) - 1)]
    return sb.Batch(d_in, d_out, off, ads)


def test_validation_rejects_bad_batches():
    assert sb.symb_validate_batch(_batch([0, 4, 9])) == sb.SYMB_OK
    assert sb.symb_validate_batch(_batch([0, 0, 0])) == sb.SYMB_OK          # empty segments are legal
    assert sb.symb_validate_batch(_batch([0])) == sb.SYMB_OK                # no segments at all
    assert sb.symb_validate_batch(_batch([1, 4])) == sb.SYMB_ERR_BAD_SEGMENTS
    assert sb.symb_validate_batch(_batch([0, 5, 3])) == sb.SYMB_ERR_BAD_SEGMENTS
    assert sb.symb_validate_batch(_batch([0, 4], d_in=0)) == sb.SYMB_ERR_INVALID_ARG
    assert sb.symb_validate_batch(_batch([0, 4], d_out=12)) == sb.SYMB_ERR_INVALID_ARG   # not a multiple of 8
    fake = 0x1000  # an aligned, never dereferenced address: validation is host-only
    lora = lambda **kw: sb.Adapter(**{**dict(kind=sb.SYMB_ADAPTER_LORA, rank=8, scale=2.0, A=fake, B=fake), **kw})
    assert sb.symb_validate_batch(_batch([0, 4], [lora()])) == sb.SYMB_OK
    assert sb.symb_validate_batch(_batch([0, 4], [lora(rank=0)])) == sb.SYMB_ERR_INVALID_ARG
    assert sb.symb_validate_batch(_batch([0, 4], [lora(A=None)])) == sb.SYMB_ERR_INVALID_ARG
    assert sb.symb_validate_batch(_batch([0, 4], [lora(B=None)])) == sb.SYMB_ERR_INVALID_ARG
    assert sb.symb_validate_batch(_batch([0, 4], [lora(A=fake + 2)])) == sb.SYMB_ERR_INVALID_ARG
    assert sb.symb_validate_batch(_batch([0, 4], [lora(rank=sb.SYMB_MAX_RANK + 1)])) == sb.SYMB_ERR_UNSUPPORTED
    assert sb.symb_validate_batch(_batch([0, 4], [lora(rank=5, B=fake + 2)])) == sb.SYMB_OK   # odd rank: 2-byte B
    assert sb.symb_validate_batch(_batch([0, 4], [sb.Adapter(kind=7)])) == sb.SYMB_ERR_INVALID_ARG
    assert sb.symb_validate_batch(_batch([0, 4], [sb.Adapter(kind=sb.SYMB_ADAPTER_IA3)])) == sb.SYMB_ERR_INVALID_ARG
    assert sb.symb_validate_batch(_batch([0, 4], [sb.Adapter(kind=sb.SYMB_ADAPTER_IA3, A=fake)])) == sb.SYMB_OK
    assert sb.symb_validate_batch(_batch([0, 4], [sb.Adapter(kind=sb.SYMB_ADAPTER_IA3_IN, A=fake)])) == sb.SYMB_OK
    assert sb.symb_validate_batch(_batch([0, 4], [sb.Adapter(kind=sb.SYMB_ADAPTER_IA3_IN)])) == sb.SYMB_ERR_INVALID_ARG
    assert b"IA3 input scaling" in sb.lib().symb_last_error(None)


@pytest.mark.parametrize("seed", range(6))
def test_row_segment_map_is_bit_exact_vs_oracle(seed):
    rng = np.random.default_rng(seed)
    S = int(rng.integers(1, 70))
    lens = rng.choice([0, 1, 1, 2, 3, 17, 64, 255, 256, 257, 1000], size=S)
    off = np.zeros(S + 1, dtype=np.int32)
    off[1:] = np.cumsum(lens)
    got = sb.symb_debug_row_segment_map(_batch(off))
    np.testing.assert_array_equal(got, oracle.row_segment_map(off))


@pytest.mark.parametrize("seed", range(6))
@pytest.mark.parametrize("tile_m", [16, 128, 256])
def test_row_tile_plan_matches_oracle_map(seed, tile_m):
    rng = np.random.default_rng(100 + seed)
    S = int(rng.integers(1, 70))
    lens = rng.choice([0, 0, 1, 1, 2, 3, 17, 64, 255, 256, 257, 1000], size=S)
    off = np.zeros(S + 1, dtype=np.int32)
    off[1:] = np.cumsum(lens)
    lo, hi = sb.symb_plan_row_tiles(_batch(off), tile_m)
    seg = oracle.row_segment_map(off)
    T = int(off[-1])
    assert len(lo) == (T + tile_m - 1) // tile_m
    for u in range(len(lo)):
        rows = seg[u * tile_m:min(T, (u + 1) * tile_m)]
        assert lo[u] == rows.min() and hi[u] == rows.max()


def test_workspace_bytes_formula():
    fake = 0x1000
    ads = [sb.Adapter(sb.SYMB_ADAPTER_LORA, 5, 1.0, fake, fake, fake, fake), sb.Adapter(),
           sb.Adapter(sb.SYMB_ADAPTER_IA3, 0, 0.0, fake), sb.Adapter(sb.SYMB_ADAPTER_LORA, 40, 1.0, fake, fake)]
    b = sb.Batch(64, 128, [0, 10, 20, 30, 100], ads)
    T, rp = 100, 2 * 48                               # pitch = 2 * (max rank rounded up to 16)
    up = lambda n: (n + 255) // 256 * 256
    packed = (16 + 48) * 128 * 2
    assert sb.symb_workspace_bytes(b, sb.SYMB_OP_FWD) == up(T * rp * 2)
    # Hs (left alone by the input-gradient call), dH, packed B^T, IA3-scaled dY
    assert sb.symb_workspace_bytes(b, sb.SYMB_OP_BWD_INPUT) == 2 * up(T * rp * 2) + up(packed) + up(T * 128 * 2)
    assert sb.symb_workspace_bytes(b, sb.SYMB_OP_ADAPTER_GRAD) == 2 * up(T * rp * 2) + up(packed)   # Hs, dH, packed B^T
    # input-major (Conv1D) weight: forward also packs B^T (at the offset the other operations use), the
    # input gradient also packs A^T (5*64 and 40*64 elements, each rounded up to 8)
    c = sb.Batch(64, 128, [0, 10, 20, 30, 100], ads, sb.SYMB_WEIGHT_CONV1D)
    assert sb.symb_workspace_bytes(c, sb.SYMB_OP_FWD) == 2 * up(T * rp * 2) + up(packed)
    assert sb.symb_workspace_bytes(c, sb.SYMB_OP_BWD_INPUT) == 2 * up(T * rp * 2) + up(packed) + up(T * 128 * 2) + up((5 * 64 + 40 * 64) * 2)
    assert sb.symb_workspace_bytes(c, sb.SYMB_OP_ADAPTER_GRAD) == 2 * up(T * rp * 2) + up(packed)
    none = sb.Batch(64, 128, [0, 100], [sb.Adapter()])
    for op in (sb.SYMB_OP_FWD, sb.SYMB_OP_BWD_INPUT, sb.SYMB_OP_ADAPTER_GRAD):
        assert sb.symb_workspace_bytes(none, op) == 0


def test_workspace_includes_the_runs_of_long_segments_gradients():
    # LoRA gradients of a segment of more than 1536 tokens are summed in runs of 1024 tokens, each run an
    # fp32 array of the gradient's size in the workspace; dB's runs and dA's share the place
    fake = 0x1000
    up = lambda n: (n + 255) // 256 * 256
    ads = [sb.Adapter(sb.SYMB_ADAPTER_LORA, 5, 1.0, fake, fake, fake, fake),      # 2100 tokens: 3 runs
           sb.Adapter(sb.SYMB_ADAPTER_LORA, 40, 1.0, fake, fake, fake, fake),     # 1536 tokens: stays whole
           sb.Adapter(sb.SYMB_ADAPTER_LORA, 8, 1.0, fake, fake)]                  # 1700 tokens, no gradients wanted
    b = sb.Batch(64, 128, [0, 2100, 3636, 5336], ads)
    T, rp = 5336, 2 * 48
    base = 2 * up(T * rp * 2) + up((16 + 48 + 16) * 128 * 2)                     # Hs, dH, packed B^T
    assert sb.symb_workspace_bytes(b, sb.SYMB_OP_ADAPTER_GRAD) == base + up(3 * 5 * 128 * 4)
    assert sb.symb_workspace_bytes(b, sb.SYMB_OP_FWD) == up(T * rp * 2)


def test_workspace_includes_partial_tiles_of_a_k_split():
    # 378 rows on a 4096 x 4096 layer: 3 x 32 = 96 tiles of 128 x 128 for 256 CUs; every tile is computed
    # by 320 // 96 = 3 workgroups, one per K range, each leaving a 64 KiB fp32 partial tile
    none = sb.Batch(4096, 4096, [0, 378], [sb.Adapter()])
    assert sb.symb_workspace_bytes(none, sb.SYMB_OP_FWD) == 96 * 3 * 128 * 128 * 4
    assert sb.symb_workspace_bytes(none, sb.SYMB_OP_BWD_INPUT) == 96 * 3 * 128 * 128 * 4
    assert sb.symb_workspace_bytes(none, sb.SYMB_OP_ADAPTER_GRAD) == 0
    # K = 448 = 7 stages of 64: too short to split; 1500 rows: 12 x 32 = 384 tiles, enough workgroups
    assert sb.symb_workspace_bytes(sb.Batch(448, 4096, [0, 378], [sb.Adapter()]), sb.SYMB_OP_FWD) == 0
    assert sb.symb_workspace_bytes(sb.Batch(4096, 4096, [0, 1500], [sb.Adapter()]), sb.SYMB_OP_FWD) == 0
    # 20480 rows: 80 x 16 tiles of 256 x 256, 160 per XCD = 5 full rounds of its 32 CUs: no split
    assert sb.symb_workspace_bytes(sb.Batch(4096, 4096, [0, 20480], [sb.Adapter()]), sb.SYMB_OP_FWD) == 0
    # 9049 rows: 36 x 16 = 576 tiles, 72 per XCD: the last 8 of them would be a round of their own and are
    # split over 3 K ranges each (24 workgroups on the XCD's 32 CUs; a fourth part would save less than it costs
    # to add up): 8 XCDs x 8 tiles x 3 partial tiles of 256 KiB
    assert sb.symb_workspace_bytes(sb.Batch(4096, 4096, [0, 9049], [sb.Adapter()]), sb.SYMB_OP_FWD) == 8 * 8 * 3 * 256 * 256 * 4
    # 20480 rows on 4608 -> 2048: 640 tiles, 80 per XCD, the last 16 split in two
    assert sb.symb_workspace_bytes(sb.Batch(4608, 2048, [0, 20480], [sb.Adapter()]), sb.SYMB_OP_FWD) == 8 * 16 * 2 * 256 * 256 * 4
    # ... 1440 tiles, 180 per XCD, a last round of 20 tiles: in three parts they are 60 workgroups, two passes of
    # a third of a tile's time each.  Worth it on the long inner dimension (input gradient of 36864 -> 4608:
    # 576 stages per tile); on 4096 stages of work the sum of the partial tiles would eat the gain
    assert sb.symb_workspace_bytes(sb.Batch(36864, 4608, [0, 20480], [sb.Adapter()]), sb.SYMB_OP_FWD) == 8 * 20 * 3 * 256 * 256 * 4
    assert sb.symb_workspace_bytes(sb.Batch(4096, 4608, [0, 20480], [sb.Adapter()]), sb.SYMB_OP_FWD) == 0


def test_parts_of_256x128_tiles_fit_an_xcd():
    """All parts of the tiles that an XCD walks are resident at once: one workgroup on each of its 32 CUs."""
    for rows, d_out, tiles, parts in ((1300, 1720, 84, 2), (2000, 1280, 80, 3), (2999, 888, 84, 2), (700, 3640, 87, 2), (1030, 2040, 80, 3)):
        assert -(-rows // 256) * -(-d_out // 128) == tiles and -(-tiles // 8) * parts <= 32
        assert sb.symb_workspace_bytes(sb.Batch(8192, d_out, [0, rows], [sb.Adapter()]), sb.SYMB_OP_FWD) == tiles * parts * 256 * 128 * 4, rows


def test_short_inner_dimensions_do_not_split_256x128_tiles():
    # 675 rows, 4096 wide: 96 tiles of 256x128 (192 of 128x128, whole); partial tiles pay from K = 6144 on
    for k, parts in ((4096, 0), (6136, 0), (6144, 2), (11008, 2)):
        assert sb.symb_workspace_bytes(sb.Batch(k, 4096, [0, 675], [sb.Adapter()]), sb.SYMB_OP_FWD) == 96 * parts * 256 * 128 * 4, k
    # 5357 rows, 680 wide: 126 tiles, activation rows off the 128-byte lines (K no multiple of 64) from 7168 on
    for k, parts in ((6136, 0), (6144, 2), (7136, 0), (7168, 2), (7176, 2)):
        assert sb.symb_workspace_bytes(sb.Batch(k, 680, [0, 5357], [sb.Adapter()]), sb.SYMB_OP_FWD) == 126 * parts * 256 * 128 * 4, k


def test_one_row_tile_or_three_parts_split_sooner():
    # 250 rows, 11008 wide: 86 tiles of 256x128 in two parts from K = 4096 on, else 172 of 128x128, whole
    for k, parts in ((4088, 0), (4096, 2)):
        assert sb.symb_workspace_bytes(sb.Batch(k, 11008, [0, 250], [sb.Adapter()]), sb.SYMB_OP_FWD) == 86 * parts * 256 * 128 * 4, k
    # 1264 rows, 2048 wide: 80 tiles in three parts from K = 4700 on, else 160 of 128x128 in two
    for k, tiles, parts, rows in ((4696, 160, 2, 128), (4704, 80, 3, 256)):
        assert sb.symb_workspace_bytes(sb.Batch(k, 2048, [0, 1264], [sb.Adapter()]), sb.SYMB_OP_FWD) == tiles * parts * rows * 128 * 4, k


def test_parts_of_a_k_split_on_narrow_layers():
    # 32 stages of 64: four parts of 8 where few tiles leave the chip idle, two for 64 tiles; 16 stages: whole
    part = 128 * 128 * 4
    for rows, parts in ((128, 4), (200, 4), (300, 3), (512, 2)):
        tiles = -(-rows // 128) * 16
        assert sb.symb_workspace_bytes(sb.Batch(2048, 2048, [0, rows], [sb.Adapter()]), sb.SYMB_OP_FWD) == tiles * parts * part, rows
    assert sb.symb_workspace_bytes(sb.Batch(1024, 4096, [0, 200], [sb.Adapter()]), sb.SYMB_OP_FWD) == 0


def test_small_batches_on_which_the_tiled_kernels_are_faster():
    """Their workspace holds the tiled kernel's regions alone (the figure is the larger of the two routes')."""
    fake = 0x1000
    lora = [sb.Adapter(sb.SYMB_ADAPTER_LORA, 16, 1.0, fake, fake)]
    up = lambda n: (n + 255) // 256 * 256
    one = sb.Batch(36864, 4608, [0, 64], [sb.Adapter()])
    # input gradient of 36864 -> 4608: 288 tiles of 128x128, whole; up to 38 rows partial sums over 3 ranges
    assert sb.symb_workspace_bytes(one, sb.SYMB_OP_BWD_INPUT) == 0
    assert sb.symb_workspace_bytes(sb.Batch(36864, 4608, [0, 33], [sb.Adapter()]), sb.SYMB_OP_BWD_INPUT) == up(3 * 33 * 36864 * 4)
    h = 64 * 2 * 16 * 2
    assert sb.symb_workspace_bytes(sb.Batch(36864, 4608, [0, 64], lora), sb.SYMB_OP_BWD_INPUT) == 2 * up(h) + up(16 * 4608 * 2)
    # 4096 -> 16384, input-major: 128 tiles in two parts; with 32 rows two ranges of partial sums, less than those
    for rows in (32, 64):
        assert sb.symb_workspace_bytes(sb.Batch(4096, 16384, [0, rows], [sb.Adapter()], sb.SYMB_WEIGHT_CONV1D), sb.SYMB_OP_FWD) == 128 * 2 * 65536
    # 2048 -> 4608, input-major: 33 rows tiled (36 tiles in four parts), 32 rows 7 ranges
    for rows in (32, 33):
        assert sb.symb_workspace_bytes(sb.Batch(2048, 4608, [0, rows], [sb.Adapter()], sb.SYMB_WEIGHT_CONV1D), sb.SYMB_OP_FWD) == 36 * 4 * 65536


def test_terms_of_short_segments_in_the_workspace():
    """Only where they are faster than the steps inside the GEMM: many steps in a row tile for few rows."""
    fake = 0x1000

    def figure(n, rank, rows, plain, d_in=4096, d_out=11008):
        c = rows // n
        ads = [sb.Adapter(sb.SYMB_ADAPTER_LORA, rank, 1.0, fake, fake)] * c + [sb.Adapter()]
        off = [n * i for i in range(c + 1)] + [n * c + plain]
        b = sb.Batch(d_in, d_out, off, ads)
        rest = sb.symb_workspace_bytes(sb.Batch(d_in, d_out, [0, off[-1]], [sb.Adapter()]), sb.SYMB_OP_FWD)     # what a split takes
        hs = off[-1] * 2 * (-(-rank // 16) * 16) * 2
        return sb.symb_workspace_bytes(b, sb.SYMB_OP_FWD) - rest - (hs + 255) // 256 * 256
    assert figure(1, 64, 48, 9000) == 48 * 11008 * 4           # 192 steps in one row tile of 256
    assert figure(16, 32, 2048, 8) == 0                        # 32 steps per row tile, 90 MB of terms: 246 us from memory, 241 in steps
    assert figure(8, 8, 2048, 8) == 0
    assert figure(1, 8, 128, 2000, 1024, 1024) == 128 * 1024 * 4
    assert figure(16, 128, 96, 0, 4096, 4096) == 96 * 4096 * 4
    assert figure(16, 16, 96, 0, 4096, 4096) == 0              # 6 steps
    assert figure(16, 64, 64, 1984, 4096, 4096) == 64 * 4096 * 4        # 16 steps of a whole tile; of one in five K parts: none
    assert figure(16, 64, 96, 0, 4096, 4096) == 0
    assert figure(1, 128, 3600, 8, 64, 36864) == 0             # more than 160 MiB of terms
    # 256x128 tiles: 16 steps are worth it in a whole tile, of one in three parts 24 are
    assert figure(8, 8, 128, 3766, 9072, 544) == 0
    assert figure(8, 8, 256, 3638, 9072, 544) == 256 * 544 * 4
    assert figure(8, 8, 128, 869, 4096, 6144) == 128 * 6144 * 4


def test_unknown_weight_layout_is_rejected():
    b = sb.Batch(64, 64, [0, 4], [sb.Adapter()], weight_layout=7)
    assert sb.lib().symb_validate_batch(b.ref()) == sb.SYMB_ERR_INVALID_ARG


def test_compute_entry_points_fail_cleanly_without_gpu():
    import torch
    if torch.cuda.is_available():
        pytest.skip("a GPU is present")
    with pytest.raises(sb.SymbError) as e:
        sb.symb_create(0)
    assert e.value.status == sb.SYMB_ERR_DEVICE
    with pytest.raises(sb.SymbError) as e:
        sb.symb_base_linear_fwd(None, _batch([0, 4]), 0x1000, 0x1000, None, 0x1000)
    assert e.value.status == sb.SYMB_ERR_INVALID_ARG      # null handle, nothing launched

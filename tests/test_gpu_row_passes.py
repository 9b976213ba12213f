"""Elementwise passes over the rows of a batch (noise prepass of the privacy flow, IA3 row scale): edges of the 8-row x
1024-column blocks a workgroup takes, and a chunk list longer than one grid."""
import numpy as np
import pytest
import torch

import gpu_harness as gh
import oracle
import synth
from helpers import assert_close, check_dx, check_y
from paper_2507_03220_amd import binding as sb

pytestmark = pytest.mark.gpu


def _bits(rng, shape):
    return synth.f32_to_bf16_bits(rng.standard_normal(shape).astype(np.float32))


@pytest.mark.parametrize("width,lens", [(8, [1]), (1024, [8, 0, 9]), (1032, [7, 33, 1, 64, 40]), (2056, [31, 5]),
                                        (8, [2097200, 3])])        # 65538 row chunks: two launches
def test_noise_add_bit_exact(width, lens):
    rng = np.random.default_rng(width + len(lens))
    off = np.zeros(len(lens) + 1, dtype=np.int32)
    off[1:] = np.cumsum(lens)
    X = _bits(rng, (int(off[-1]), width))
    noise = [[_bits(rng, (n, width)), _bits(rng, (1, width)), None][i % 3] if n else None for i, n in enumerate(lens)]
    b = sb.Batch(width, 8, off, [sb.Adapter() for _ in lens])
    Xn = torch.full((int(off[-1]), width), float("nan"), device="cuda", dtype=torch.bfloat16)
    sb.symb_noise_add(gh.handle(), b, gh.to_dev(X), [gh.to_dev(n) for n in noise], Xn)
    torch.cuda.synchronize()
    assert np.array_equal(gh.bf16_bits(Xn), oracle.noise_add(off, X, noise))


@pytest.mark.parametrize("width,lens", [(8, [1, 2]), (1024, [8, 0, 9, 3]), (1032, [7, 33, 1, 64, 40])])
def test_ia3_scaled_rows(width, lens):
    """Input gradient through output-scaling segments and forward through input-scaling ones, beside segments
    whose rows are copied or left alone: the rows the product contracts are scaled (or copied) by the row pass."""
    rng = np.random.default_rng(100 + width)
    off = np.zeros(len(lens) + 1, dtype=np.int32)
    off[1:] = np.cumsum(lens)
    W, V = _bits(rng, (width, 40)), _bits(rng, (40, width))
    G = _bits(rng, (int(off[-1]), width))
    for kind, weight in ((sb.SYMB_ADAPTER_IA3, W), (sb.SYMB_ADAPTER_IA3_IN, V)):
        ads = [gh.HostAdapter(kind, 0, 0.0, synth.f32_to_bf16_bits(1 + 0.1 * rng.standard_normal(width).astype(np.float32))) if i % 2
               else gh.HostAdapter() for i in range(len(lens))]
        oads = [oracle.Adapter(a.kind, a.rank, a.scale, a.A, a.B) for a in ads]
        if kind == sb.SYMB_ADAPTER_IA3:
            check_dx(gh.bf16_to_f64(gh.backward_input(off, ads, G, weight)), off, oads, G, weight, "dX")
        else:
            check_y(gh.bf16_to_f64(gh.forward(off, ads, G, weight, want_base=False)[0]), off, oads, G, weight, None, "Y")


@pytest.mark.parametrize("width,lens", [(8, [1, 3]), (64, [127, 128, 129]), (72, [384, 385, 16]), (136, [511, 512, 1300, 0])])
def test_ia3_vector_gradient(width, lens):
    """dl of output-scaling segments: edges of the 64 columns and the 128 tokens (four deep) a workgroup walks side by side."""
    rng = np.random.default_rng(200 + width)
    off = np.zeros(len(lens) + 1, dtype=np.int32)
    off[1:] = np.cumsum(lens)
    T = int(off[-1])
    X, G, Y0 = _bits(rng, (T, 16)), _bits(rng, (T, width)), _bits(rng, (T, width))
    ads = [gh.HostAdapter(sb.SYMB_ADAPTER_IA3, 0, 0.0, _bits(rng, (width,))) for _ in lens]
    got = gh.adapter_grad(off, ads, X, G, Y0)
    for i, n in enumerate(lens):
        rows = slice(int(off[i]), int(off[i + 1]))
        ref = (synth.bf16_bits_to_f64(G[rows]) * synth.bf16_bits_to_f64(Y0[rows])).sum(0)
        # fp32 products and sums in any order: at most (n + 1) roundings of 2^-24 of the absolute sum
        bound = (n + 1) * 2.0 ** -24 * np.abs(synth.bf16_bits_to_f64(G[rows]) * synth.bf16_bits_to_f64(Y0[rows])).sum(0)
        assert np.all(np.abs(got.descs[i].dA.cpu().numpy() - ref) <= bound + 1e-300)


@pytest.mark.parametrize("width,lens", [(72, [1, 15, 16, 17, 63, 64, 65]), (264, [191, 192, 193]), (136, [1023, 1024, 1025, 2]), (40, [200] * 3 + [1, 0]),
                                        (2248, [3] * 60 + [1100])])        # both shapes of the kernel, in one launch and (last) in two
def test_ia3_gradient(width, lens):
    rng = np.random.default_rng(width)
    off = np.zeros(len(lens) + 1, dtype=np.int32)
    off[1:] = np.cumsum(lens)
    T = int(off[-1])
    dY, Y0 = _bits(rng, (T, width)), _bits(rng, (T, width))
    l = gh.to_dev(_bits(rng, (width,)))
    dl = [torch.full((width,), float("nan"), device="cuda") for _ in lens]
    b = sb.Batch(8, width, off, [sb.Adapter(sb.SYMB_ADAPTER_IA3, 0, 0.0, l, None, d) for d in dl])
    X = torch.zeros(T, 8, device="cuda", dtype=torch.bfloat16)
    dYd, Yd = gh.to_dev(dY), gh.to_dev(Y0)
    for times, flag in ((1, sb.SYMB_GRAD_OVERWRITE), (2, sb.SYMB_GRAD_ACCUMULATE)):
        sb.symb_adapter_grad(gh.handle(), b, X, dYd, Yd, flag, None)
        torch.cuda.synchronize()
        for i, n in enumerate(lens):
            rows = slice(off[i], off[i + 1])
            ref = times * (synth.bf16_bits_to_f64(dY[rows]) * synth.bf16_bits_to_f64(Y0[rows])).sum(0)
            assert_close(dl[i].cpu().numpy(), ref, f"dl[{i}] x{times}")

"""Layers with a round of wide tiles and more (bcr_conv_wide): the epilogue's forms.  Compared with the conv reference and, where
the same sums are stored in another form, bit for bit."""
from __future__ import annotations

import numpy as np
import pytest

import bcr_inputs as gen
from test_conv import _run_plan


def _layer(dtype, M, Cin, H, W, kh, kw, BR, BC, B, seed):
    import paper_2108_11033_amd as g
    from helpers import pack_workload
    K = Cin * kh * kw
    mask = gen.random_mask(M, K, BR, BC, tuple(sorted({1, BR // 2, BR})), tuple(sorted({1, BC // 4 + 1, BC})), seed=seed)
    Wt = gen.normal_weights(M, K, dtype, seed=seed + 1)
    F = gen.normal_activations(Cin, B * H * W, dtype, seed=seed + 2, relu=True).reshape(Cin, B, H, W).transpose(1, 0, 2, 3).copy()
    A = pack_workload(g, Wt, dtype, mask)
    assert g.conv2d_kernel_name(A, Cin, H, W, kh, kw, B, 1) == "bcr_conv_wide"
    return g, A, Wt, mask, F


@pytest.mark.gpu
@pytest.mark.parametrize("dtype", [gen.F16, gen.BF16])
@pytest.mark.parametrize("M,BR,H,W,B", [(128, 16, 130, 128, 3), (256, 32, 130, 64, 3), (144, 16, 104, 120, 4)])
@pytest.mark.parametrize("pad", [0, 4, 2, 3])
def test_outputs_of_16_bits_are_the_rounded_sums(dtype, M, BR, H, W, B, pad):
    """Rows of the output at every alignment (four outputs at once, or one by one): the fp32 sums of the same layer, with bias and
    rectifier applied in fp32 and rounded once -- the same bits."""
    import torch
    g, A, Wt, mask, F = _layer(dtype, M, 16, H, W, 1, 1, BR, 16, B, 900 + M)
    bias = (0.05 * np.random.default_rng(903).standard_normal(M)).astype(np.float32)
    sums = _run_plan(g, A, F, dtype, M, 1, 1, 1).astype(np.float32)
    want = np.maximum(sums + bias[None, :, None, None], np.float32(0))
    tdt = {gen.F16: torch.float16, gen.BF16: torch.bfloat16}[dtype]
    want = torch.from_numpy(want).to(tdt).float().numpy()
    got = _run_plan(g, A, F, dtype, M, 1, 1, 1, bias=bias, relu=True, out_dtype=dtype, pad=pad).astype(np.float32)
    assert np.array_equal(got, want)

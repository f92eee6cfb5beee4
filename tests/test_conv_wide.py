"""Layers with a round of wide tiles and more (bcr_conv_wide): the ways the rows of the im2col matrix are dealt to the fetching
threads and the epilogue's forms.  Compared with the conv reference and, where the same sums are stored in another form, bit for bit."""
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
@pytest.mark.parametrize("M,BR,BC,Cin,H,W,kh,kw,B", [
    (256, 32, 27, 27, 64, 128, 3, 3, 3),     # 243 rows: a whole chunk of 192, then 51; channels that begin inside a chunk
    (256, 32, 16, 16, 100, 88, 1, 3, 3),     # way after way of a flat kernel
    (256, 32, 21, 11, 88, 96, 7, 3, 3),      # 21 taps: one thread per (tap, piece), the most there is room for
    (256, 32, 23, 10, 88, 96, 23, 1, 3),     # 23 taps: through the tables
    (128, 16, 30, 10, 130, 128, 3, 3, 3),    # 192-column tiles
    (128, 16, 22, 12, 130, 128, 11, 1, 3),   # 192-column tiles, more taps than they have threads for
    (128, 16, 25, 200, 130, 128, 1, 1, 3),   # a row per channel
    (256, 32, 9, 5, 1, 24584, 3, 3, 1),      # windows a row above and below a map of one row
    (256, 32, 9, 5, 8, 5, 3, 3, 700),        # maps smaller than a tile
])
def test_rows_of_every_kernel_shape(M, BR, BC, Cin, H, W, kh, kw, B):
    from helpers import TOL
    from oracle import conv_ref
    from test_conv import _masked
    g, A, Wt, mask, F = _layer(gen.F16, M, Cin, H, W, kh, kw, BR, BC, B, 920 + kh)
    Wm, F64 = _masked(Wt, gen.F16, mask), gen.storage_to_f64(F, gen.F16)
    pad = 4 if B > 1 else 0
    Y = _run_plan(g, A, F, gen.F16, M, kh, kw, 1, pad=pad)
    Yref, S = conv_ref.conv2d(Wm, F64, kh, kw, 1), conv_ref.conv2d(np.abs(Wm), np.abs(F64), kh, kw, 1)
    assert (np.abs(Y - Yref) <= TOL[gen.F16] * S).all()


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

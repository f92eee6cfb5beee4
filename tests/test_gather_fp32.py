"""The fp32 row-gathering kernel and the products of a few columns that run as one padded tile (grim_bcr_spmm,
grim_bcr_spmv): every tile width and form at its edges against the oracle, pieces that end behind the last element of X,
blocks that keep no rows, no columns or counts that are no multiple of four, and infinities and NaNs in X, which must
reach the rows that keep their column and no others."""
import numpy as np
import pytest

import bcr_inputs as gen
from helpers import assert_close, oracle_product, pack_workload, run_spmm, run_spmv

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def g():
    import paper_2108_11033_amd as mod
    mod.load_library()
    return mod


def _case(dtype, M, K, BR, BC, N, seed):
    mask = gen.random_mask(M, K, BR, BC, tuple(sorted({0, 1, BR // 2, BR})), tuple(sorted({0, min(3, BC), min(8, BC), BC})), seed=seed)
    return mask, gen.normal_weights(M, K, dtype, seed=seed + 1), gen.normal_activations(K, N, dtype, seed=seed + 2)


def _keeping_rows(mask, k):
    """Per row of the matrix: does it keep column k?"""
    keep = np.zeros(mask.M, dtype=bool)
    c, j = divmod(k, mask.BC)
    for s in range(mask.nbr):
        b = s * mask.nbc + c
        if j in mask.col_idx[mask.col_ptr[b]:mask.col_ptr[b + 1]]:
            keep[s * mask.BR + mask.row_idx[mask.row_ptr[b]:mask.row_ptr[b + 1]].astype(int)] = True
    return keep


@pytest.mark.parametrize("BR,BC", [(16, 32), (32, 32), (4, 16), (64, 16)])
@pytest.mark.parametrize("N,ldx_pad", [(9, 0), (16, 0), (17, 0), (18, 1), (32, 0), (33, 0), (35, 0), (36, 3), (63, 0), (64, 0), (65, 0),
                                       (130, 1), (1001, 0)])
def test_fp32_tiles(g, BR, BC, N, ldx_pad):
    M, K = 192, 16 * 42
    mask, W, X = _case(gen.F32, M, K, BR, BC, N, 1000 + N)
    Yref, S = oracle_product(W, X, gen.F32, mask)
    Y = run_spmm(g, pack_workload(g, W, gen.F32, mask), X, gen.F32, M, N, ldx=N + ldx_pad, ldy=N + 3)
    assert_close(Y, Yref, S, gen.F32, f"fp32 {BR}x{BC} N={N}")


@pytest.mark.parametrize("M,K,BR,BC,N", [(64, 96, 16, 32, 33333),       # a run per wave, odd N
                                         (16, 2400, 16, 32, 130),       # eight waves per run
                                         (20, 64, 4, 16, 100)])         # a last run of four rows
def test_fp32_forms(g, M, K, BR, BC, N):
    mask, W, X = _case(gen.F32, M, K, BR, BC, N, 1100 + M)
    Yref, S = oracle_product(W, X, gen.F32, mask)
    assert_close(run_spmm(g, pack_workload(g, W, gen.F32, mask), X, gen.F32, M, N), Yref, S, gen.F32, f"fp32 {M}x{K}")


@pytest.mark.parametrize("dtype", [gen.F32, gen.F16, gen.BF16])
@pytest.mark.parametrize("N", [1, 2, 3, 5, 7, 8])
def test_few_columns_of_mixed_blocks(g, dtype, N):
    for M, K, BR, BC, pad in [(96, 96, 32, 32, 0), (128, 2048, 32, 32, 3), (64, 64, 8, 32, 0), (16, 1, 16, 1, 0)]:
        mask, W, X = _case(dtype, M, K, BR, BC, N, 1200 + K)
        Yref, S = oracle_product(W, X, dtype, mask)
        A = pack_workload(g, W, dtype, mask)
        assert_close(run_spmv(g, A, X, dtype, M, N, ldx=N + pad, ldy=N + 1), Yref, S, dtype, f"{dtype} {M}x{K} batch {N}")


@pytest.mark.parametrize("dtype,BR,BC,N", [(gen.F32, 16, 32, 3), (gen.F32, 16, 32, 100), (gen.F32, 32, 32, 9000), (gen.F16, 32, 32, 5),
                                           (gen.BF16, 32, 32, 1), (gen.F16, 4, 16, 101), (gen.BF16, 4, 16, 20001), (gen.F16, 8, 32, 33)])
@pytest.mark.parametrize("value", [np.inf, -np.inf, np.nan])
def test_non_finite_values_reach_the_rows_that_keep_them(g, dtype, BR, BC, N, value):
    M, K = 64, 32 * 9
    mask, W, X = _case(dtype, M, K, BR, BC, N, 1300)
    hit = _keeping_rows(mask, 37)
    k, n = 37, N // 2
    assert hit.any() and not hit.all()
    Yref, S = oracle_product(W, X, dtype, mask)
    bits = {gen.F32: np.float32, gen.F16: np.float16}.get(dtype)
    X = X.copy()
    X[k, n] = value if bits else (np.array([value], np.float32).view(np.uint32) >> 16).astype(np.uint16)[0]
    A = pack_workload(g, W, dtype, mask)
    Y = run_spmv(g, A, X, dtype, M, N) if N <= 8 else run_spmm(g, A, X, dtype, M, N)
    assert not np.isfinite(Y[hit, n]).any()
    Y[hit, n] = Yref[hit, n]
    assert_close(Y, Yref, S, dtype, f"{dtype} {BR}x{BC} N={N} {value}")


@pytest.mark.parametrize("M,K,BR,BC,kr,kc,N", [(32, 16384, 16, 32, 16, 32, 40),      # 1024 steps over eight waves
                                               (64, 4608, 1, 16, 1, 4, 70),
                                               (512, 4608, 16, 32, 8, 8, 200)])
def test_fp32_no_less_exact_than_the_vector_alus(g, M, K, BR, BC, kr, kc, N):
    """The distance from a 64-bit product against that of the vector-ALU kernel with its sixteen partial sums, which took these
    products before; the two differ by a few per cent either way."""
    import torch
    from helpers import to_device
    mask = gen.random_mask(M, K, BR, BC, kr, kc, seed=1400)
    W = gen.normal_weights(M, K, gen.F32, seed=1401)
    X = gen.normal_activations(K, N, gen.F32, seed=1402, relu=True)
    A = pack_workload(g, W, gen.F32, mask)
    ref = torch.from_numpy(A.unpack().astype(np.float64)).cuda() @ torch.from_numpy(X.astype(np.float64)).cuda()
    xd, y = to_device(X, gen.F32), torch.empty((M, N), dtype=torch.float32, device="cuda")
    err = []
    for kernel in (0, 1):
        g.spmm(A, xd, N, N, y, N, kernel=kernel)
        torch.cuda.synchronize()
        err.append(float((y.double() - ref).norm() / ref.norm()))
    assert err[0] <= 1.15 * err[1], err


@pytest.mark.parametrize("M,K,BR,BC,N", [(64, 576, 1, 16, 64), (256, 1152, 2, 32, 33), (1024, 1024, 2, 16, 64), (64, 576, 4, 16, 200),
                                         (4096, 64, 1, 16, 3), (256, 1024, 2, 16, 8), (8192, 2048, 32, 32, 3)])
def test_fp32_small_blocks_on_either_kernel(g, M, K, BR, BC, N):
    """Blocks of a few rows and tall matrices, on both sides of the rules that choose between this kernel and the vector ALUs."""
    mask, W, X = _case(gen.F32, M, K, BR, BC, N, 1500)
    Yref, S = oracle_product(W, X, gen.F32, mask)
    A = pack_workload(g, W, gen.F32, mask)
    Y = run_spmv(g, A, X, gen.F32, M, N) if N <= 8 else run_spmm(g, A, X, gen.F32, M, N)
    assert_close(Y, Yref, S, gen.F32, f"fp32 {M}x{K} {BR}x{BC} N={N}")

"""Products whose rows of X have any alignment, on the row-gathering kernel (grim_bcr_spmm with N or ldx not a multiple of
4): every tile width of products below 64 columns and its edges, tiles that overlap at a ragged end, padded leading
dimensions, the last rows of X (nothing past its last element may be read into a result), mixed and empty blocks."""
import numpy as np
import pytest

import bcr_inputs as gen
from helpers import assert_close, oracle_product, pack_workload, run_spmm

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def g():
    import paper_2108_11033_amd as mod
    mod.load_library()
    return mod


@pytest.mark.parametrize("dtype,BR,BC", [(gen.F16, 16, 32), (gen.BF16, 32, 32), (gen.F16, 4, 16)])
@pytest.mark.parametrize("N,ldx_pad", [(9, 0), (11, 2), (15, 0), (17, 0), (18, 0), (31, 1), (33, 0), (63, 0), (65, 0), (66, 1),
                                       (127, 0), (130, 0), (1001, 0), (64, 1)])
def test_rows_of_any_alignment(g, dtype, BR, BC, N, ldx_pad):
    M, K = 96, 32 * 21
    mask = gen.random_mask(M, K, BR, BC, tuple(sorted({0, 1, BR // 2, BR})), (0, 3, 8, 16), seed=900 + N)
    W = gen.normal_weights(M, K, dtype, seed=901)
    X = gen.normal_activations(K, N, dtype, seed=902)
    A = pack_workload(g, W, dtype, mask)
    Yref, S = oracle_product(W, X, dtype, mask)
    Y = run_spmm(g, A, X, dtype, M, N, ldx=N + ldx_pad, ldy=N + 3)
    assert_close(Y, Yref, S, dtype, f"{dtype} {BR}x{BC} N={N} ldx=N+{ldx_pad}")


def test_rows_of_any_alignment_wave_per_strip(g):
    # thousands of (tile, strip) pairs of a few steps, and a strip that keeps nothing
    dtype, M, K, N = gen.F16, 96, 96, 33333
    mask = gen.random_mask(M, K, 16, 32, (0, 3, 8, 16), (0, 5, 8, 32), seed=910)
    W = gen.normal_weights(M, K, dtype, seed=911)
    X = gen.normal_activations(K, N, dtype, seed=912, relu=True)
    Yref, S = oracle_product(W, X, dtype, mask)
    Y = run_spmm(g, pack_workload(g, W, dtype, mask), X, dtype, M, N)
    assert_close(Y, Yref, S, dtype, "wave per strip, odd N")
    assert np.isfinite(Y).all()


@pytest.mark.parametrize("dtype", [gen.F16, gen.BF16])
@pytest.mark.parametrize("M,BR,BC,N,ldx_pad", [(48, 16, 32, 64, 0), (48, 16, 32, 65, 0), (64, 32, 32, 96, 0), (32, 4, 16, 97, 2),
                                               (32, 8, 16, 200, 8), (16, 16, 32, 8192, 0), (16, 16, 32, 8191, 1)])
def test_long_strips_and_few_tiles(g, dtype, M, BR, BC, N, ldx_pad):
    """32-column tiles with twelve waves to a strip: fewer steps than three to a wave, a few more, and several batches; the
    last workgroup count of the form and the columns around it, aligned and odd."""
    K = 32 * 60
    mask = gen.random_mask(M, K, BR, BC, tuple(sorted({0, BR // 2, BR})), (BC // 4, BC // 2, BC), seed=920 + N)
    W = gen.normal_weights(M, K, dtype, seed=921)
    X = gen.normal_activations(K, N, dtype, seed=922)
    Yref, S = oracle_product(W, X, dtype, mask)
    Y = run_spmm(g, pack_workload(g, W, dtype, mask), X, dtype, M, N, ldx=N + ldx_pad, ldy=N + 1)
    assert_close(Y, Yref, S, dtype, f"{dtype} {M}x{K} {BR}x{BC} N={N}")


@pytest.mark.parametrize("dtype", [gen.F32, gen.F16, gen.BF16])
def test_blocks_of_more_than_64_rows(g, dtype):
    """Only the row-gathering kernels on 8-byte-aligned rows take them: the rest is refused, and leaves the output alone."""
    import torch
    from helpers import to_device
    M, K, BR = 384, 64, 128
    mask = gen.random_mask(M, K, BR, 16, (8, 64, 128), (4, 16), seed=930)
    W = gen.normal_weights(M, K, dtype, seed=931)
    A = pack_workload(g, W, dtype, mask)
    for N, ldx in [(1, 1), (3, 3), (4, 4), (5, 5), (8, 8), (9, 9), (12, 12), (12, 13), (33, 33), (64, 64), (66, 66), (101, 101)]:
        X = gen.normal_activations(K, N, dtype, seed=932)
        if dtype != gen.F32 and N % 4 == 0 and ldx % 4 == 0:
            Yref, S = oracle_product(W, X, dtype, mask)
            assert_close(run_spmm(g, A, X, dtype, M, N), Yref, S, dtype, f"{dtype} BR=128 N={N}")
            continue
        xd = torch.zeros((K, ldx), dtype=torch.float32, device="cuda").to(to_device(X, dtype).dtype)
        y = torch.full((M, N), 7.0, dtype=torch.float32, device="cuda")
        for call in [lambda: g.spmm(A, xd, N, ldx, y, N)] + ([lambda: g.spmv(A, xd, N, ldx, y, N)] if N <= 8 else []):
            with pytest.raises(g.GrimError) as e:
                call()
            assert e.value.name == "GRIM_ERR_UNSUPPORTED", (N, ldx)
        torch.cuda.synchronize()
        assert (y == 7.0).all()


@pytest.mark.parametrize("batch", [5, 12])
def test_recurrent_steps_of_blocks_of_more_than_64_rows(g, batch):
    import torch
    H, I, BR = 128, 64, 128
    mats = []
    for M, K in ((4 * H, I + H), (3 * H, I), (3 * H, H)):
        mask = gen.random_mask(M, K, BR, 16, (8, 64, 128), (4, 16), seed=940 + K)
        mats.append(pack_workload(g, gen.normal_weights(M, K, gen.F16, seed=941), gen.F16, mask))
    half, full = (lambda n: torch.zeros((n, batch), dtype=torch.float16, device="cuda")), (lambda n: torch.zeros((n, batch), device="cuda"))
    calls = [lambda: g.lstm_step(mats[0], half(I + H), batch, batch, full(4 * H), batch, None, full(H), batch, half(H), batch, full(H), batch),
             lambda: g.gru_step(mats[1], mats[2], half(I), batch, half(H), batch, batch, full(3 * H), batch, full(3 * H), batch, None, None,
                                full(H), batch, half(H), batch)]
    for call in calls:
        if batch % 4 == 0:
            call()
            continue
        with pytest.raises(g.GrimError) as e:
            call()
        assert e.value.name == "GRIM_ERR_UNSUPPORTED"
    torch.cuda.synchronize()


@pytest.mark.parametrize("dtype", [gen.F16, gen.BF16])
@pytest.mark.parametrize("M,BR,kernel", [(96, 48, 0), (32, 16, 3), (64, 32, 3), (256, 128, 0), (192, 64, 0)])
def test_products_of_one_row_of_four(g, dtype, M, BR, kernel):
    """K = 1 and four columns: X is shorter than the 16 bytes the kernel loads at a time."""
    mask = gen.random_mask(M, 1, BR, 1, (BR // 2, BR), (1,), seed=950)
    W = gen.normal_weights(M, 1, dtype, seed=951)
    X = gen.normal_activations(1, 4, dtype, seed=952)
    Yref, S = oracle_product(W, X, dtype, mask)
    assert_close(run_spmm(g, pack_workload(g, W, dtype, mask), X, dtype, M, 4, ldy=5, kernel=kernel), Yref, S, dtype, f"BR={BR}")


@pytest.mark.parametrize("M,K,BR,BC,kr,kc,N", [(256, 1152, 1, 16, 1, 4, 9999),      # a wave per run, long chains of multiplies
                                               (256, 1152, 4, 16, 2, 4, 9999),
                                               (512, 4608, 64, 64, 16, 16, 3135),   # four waves to a run
                                               (512, 4608, 4, 16, 2, 4, 1001),
                                               (512, 4096, 32, 32, 32, 32, 1)])     # one column, dense blocks
@pytest.mark.parametrize("dtype", [gen.F16, gen.BF16])
def test_no_less_exact_than_the_vector_alus(g, dtype, M, K, BR, BC, kr, kc, N):
    """These operands used to be multiplied on the vector ALUs in sixteen partial sums (or more).  The distance from a 64-bit
    product is no larger now; the two differ by a few per cent either way."""
    import torch
    from helpers import to_device
    mask = gen.random_mask(M, K, BR, BC, kr, kc, seed=960)
    W = gen.normal_weights(M, K, dtype, seed=961)
    X = gen.normal_activations(K, N, dtype, seed=962, relu=N > 1)
    A = pack_workload(g, W, dtype, mask)
    kept = torch.from_numpy(gen.storage_to_f64(A.unpack(), dtype)).cuda()
    ref = kept @ torch.from_numpy(gen.storage_to_f64(X, dtype)).cuda()
    xd, y = to_device(X, dtype), torch.empty((M, N), dtype=torch.float32, device="cuda")
    err = []
    for kernel in (0, 1):
        g.spmm(A, xd, N, N, y, N, kernel=kernel)
        torch.cuda.synchronize()
        err.append(float((y.double() - ref).norm() / ref.norm()))
    assert err[0] <= 1.15 * err[1], err


@pytest.mark.parametrize("dtype", [gen.F16, gen.BF16])
@pytest.mark.parametrize("steps", [1, 2, 8, 9, 16, 17, 32, 33, 65])
@pytest.mark.parametrize("N", [8, 9, 15, 17, 33])
def test_narrow_tiles_by_length_of_the_strips(g, dtype, steps, N):
    """Dense blocks, a step per 32 columns of the matrix: the steps in flight and the waves of narrow tiles change at 8, 16 and
    32 steps (16-column tiles) and at 16 (wider ones); a matrix with more strips than compute units keeps four waves."""
    for M in (64, 4128) if N == 9 and steps in (17, 33) else (64,):
        K = 32 * steps
        mask = gen.random_mask(M, K, 16, 32, (16,), (32,), seed=970)
        W = gen.normal_weights(M, K, dtype, seed=971)
        X = gen.normal_activations(K, N, dtype, seed=972)
        Yref, S = oracle_product(W, X, dtype, mask)
        assert_close(run_spmm(g, pack_workload(g, W, dtype, mask), X, dtype, M, N), Yref, S, dtype, f"{M}x{K} N={N}")

"""Host-side checks of the layouts the kernels read (no GPU): every derived layout -- the staged matrix-core
SpMM's step records, the row-gathering SpMM's steps per 16-row run, the SpMV's bit masks -- decodes back to
exactly the masked dense matrix, over a seeded sweep of odd shapes: block heights and widths from 1 to 64,
empty blocks, empty strips, a K = 27 dense first layer, matrices of one block, matrices large enough that their
layouts are written in parallel parts.  The fp32 row-gathering layout and a convolution plan's 64-row runs have no
decoder in the library; the build of test_sanitize_host.py has them (tests/sanitize/derived_layouts.cpp)."""
import ctypes

import numpy as np
import pytest

import bcr_inputs as gen
import paper_2108_11033_amd as g
from paper_2108_11033_amd.binding import GrimError
from oracle import bcr_oracle as orc

LAYOUTS = {1: "staged SpMM", 2: "row-gathering SpMM", 3: "SpMV", 4: "wide-tile staged SpMM"}


def _expected_layouts(dtype, BR, BC):
    want = set()
    if dtype != gen.F32 and BR in (16, 32) and BC <= 256:
        want.add(1)
    if dtype != gen.F32 and BR in (16, 32) and BC <= 128:
        want.add(4)
    if dtype != gen.F32 and (16 % BR == 0 or BR % 16 == 0):
        want.add(2)
    if BR <= 32 and BC <= 32:
        want.add(3)
    return want


def _check(M, K, BR, BC, kr, kc, dtype, seed, dense=False):
    mask = gen.full_mask(M, K, BR, BC) if dense else gen.random_mask(M, K, BR, BC, kr, kc, seed=seed)
    W = gen.normal_weights(M, K, dtype, seed=seed + 1)
    for reorder in (True, False):
        A = g.pack(W, dtype, BR, BC, mask.row_ptr, mask.row_idx, mask.col_ptr, mask.col_idx, host_only=2,
                   no_reorder=not reorder)
        ref = A.unpack()
        Wm = orc.masked_dense(gen.storage_to_f64(W, dtype), BR, BC, mask.row_ptr, mask.row_idx, mask.col_ptr, mask.col_idx)
        assert ref.tobytes() == np.where(Wm != 0, W, np.zeros_like(W)).tobytes()
        have = set()
        for lay in LAYOUTS:
            try:
                got = A.unpack_layout(lay)
            except GrimError as e:
                assert e.name == "GRIM_ERR_UNSUPPORTED", (lay, e)
                continue
            have.add(lay)
            assert got.tobytes() == ref.tobytes(), f"{LAYOUTS[lay]} layout of {M}x{K} {BR}x{BC} {dtype} decodes wrongly"
        assert have == _expected_layouts(dtype, BR, BC), (have, dtype, BR, BC)


@pytest.mark.parametrize("dtype", [gen.F16, gen.BF16, gen.F32])
@pytest.mark.parametrize("M,K,BR,BC,kr,kc", [
    (64, 96, 16, 32, (0, 4, 8, 16), (0, 8, 32)),       # empty and full blocks
    (96, 128, 32, 32, (4, 8, 16), (4, 8, 16)),         # the non-uniform workload's law
    (48, 64, 4, 16, (0, 2, 4), (0, 4, 16)),            # the paper's CNN block size
    (128, 128, 64, 64, (8, 32), (8, 24)),
    (30, 28, 5, 7, (0, 1, 5), (0, 2, 7)),              # heights that fit no matrix-core tile
    (12, 10, 1, 1, (0, 1), (0, 1)),                    # non-structured limit
    (16, 24, 16, 24, 5, 9),                            # one block = the whole matrix
    (96, 40, 48, 8, (0, 7, 48), (1, 3, 8)),
    (32, 576, 16, 32, 8, 8),                           # c2's pattern, several chunks of the staged layout
    (64, 512, 32, 32, (0, 32), (0, 1, 32)),
    (40, 66, 8, 33, (1, 8), (1, 17, 33)),              # odd block width
    (34, 64, 2, 64, (0, 1, 2), (3, 9, 64)),
    (272, 544, 16, 32, (4, 8, 16), (8, 16, 32)),       # more than 32 K kept weights: several parts, 17 runs
    (264, 512, 8, 16, (4, 8), (8, 16)),                # the last run is half a run
    (384, 512, 128, 32, (64, 128), (8, 32)),
])
def test_every_layout_decodes_to_the_masked_matrix(dtype, M, K, BR, BC, kr, kc):
    _check(M, K, BR, BC, kr, kc, dtype, seed=500 + M + K)


@pytest.mark.parametrize("dtype", [gen.F16, gen.BF16])
def test_dense_first_layer_layouts(dtype):
    # VGG-16 layer 1: K = 27, one dense 16 x 27 block per strip
    _check(64, 27, 16, 27, 16, 27, dtype, seed=700, dense=True)


def test_seeded_sweep_of_block_shapes():
    rng = np.random.default_rng(20210811)
    for it in range(60):
        BR = int(rng.choice([1, 2, 3, 4, 6, 8, 12, 16, 24, 32, 48, 64]))
        BC = int(rng.choice([1, 2, 5, 8, 9, 16, 27, 32, 40, 64]))
        nbr, nbc = int(rng.integers(1, 5)), int(rng.integers(1, 7))
        kr = tuple(sorted({0, int(rng.integers(0, BR + 1)), int(rng.integers(0, BR + 1)), BR}))
        kc = tuple(sorted({0, int(rng.integers(0, BC + 1)), int(rng.integers(0, BC + 1)), BC}))
        dtype = [gen.F16, gen.BF16, gen.F32][it % 3]
        _check(nbr * BR, nbc * BC, BR, BC, kr, kc, dtype, seed=1000 + it)


def test_unpack_layout_argument_errors():
    mask = gen.random_mask(32, 32, 16, 16, 4, 8, seed=1)
    W = gen.normal_weights(32, 32, gen.F16, seed=2)
    A = g.pack(W, gen.F16, 16, 16, mask.row_ptr, mask.row_idx, mask.col_ptr, mask.col_idx, host_only=2)
    lib = g.load_library()
    out = np.empty((32, 32), dtype=np.float16)
    p = out.ctypes.data
    assert lib.grim_bcr_unpack_layout(None, 1, p, 32) == 1                 # NULL
    assert lib.grim_bcr_unpack_layout(A.handle, 1, None, 32) == 1
    assert lib.grim_bcr_unpack_layout(A.handle, 1, p, 31) == 2             # ldw < K
    assert lib.grim_bcr_unpack_layout(A.handle, 0, p, 32) == 2             # unknown layout
    assert lib.grim_bcr_unpack_layout(A.handle, 5, p, 32) == 2
    B = g.pack(W, gen.F16, 16, 16, mask.row_ptr, mask.row_idx, mask.col_ptr, mask.col_idx, host_only=True)
    assert lib.grim_bcr_unpack_layout(B.handle, 2, p, 32) == 7             # canonical arrays only: no layouts


@pytest.fixture
def decoders():
    lib = g.load_library()
    if not hasattr(lib, "grim_test_decode_gather32"):
        pytest.skip("not the build with these decoders")
    for f in (lib.grim_test_decode_gather32, lib.grim_test_decode_64_row_runs):
        f.argtypes, f.restype = [ctypes.c_void_p, ctypes.c_void_p, ctypes.c_int64], ctypes.c_int
    return lib


@pytest.mark.parametrize("M,K,BR,BC,kr,kc", [
    (64, 96, 16, 32, (0, 4, 8, 16), (0, 8, 32)),
    (16, 64, 4, 16, (0, 2, 4), (0, 4, 16)),            # a quarter of a 64-row run
    (72, 64, 4, 16, (0, 2, 4), (0, 4, 16)),            # a second run of 8 rows
    (80, 66, 16, 33, (0, 8, 16), (1, 17, 33)),         # a second run of 16 rows; odd block width
    (66, 64, 2, 64, (0, 1, 2), (3, 9, 64)),
    (13, 10, 1, 1, (0, 1), (0, 1)),
    (192, 128, 64, 64, (0, 8, 64), (0, 8, 24)),
    (384, 96, 128, 32, (0, 64, 128), (0, 8, 32)),      # blocks of two 64-row runs
    (60, 28, 5, 7, (0, 1, 5), (0, 2, 7)),              # heights that fit no run
    (144, 40, 48, 8, (0, 7, 48), (1, 3, 8)),           # whole 16-row runs, no 64-row ones
    (1000, 256, 8, 16, (4, 8), (8, 16)),               # more than 32 K kept weights and 8 runs of 64 rows: several parts
    (1024, 256, 128, 32, (64, 128), (8, 32)),
])
@pytest.mark.parametrize("dtype", [gen.F16, gen.F32])
@pytest.mark.parametrize("reorder", [True, False])
def test_layouts_without_a_decoder_in_the_library(decoders, dtype, reorder, M, K, BR, BC, kr, kc):
    mask = gen.random_mask(M, K, BR, BC, kr, kc, seed=600 + M + K)
    W = gen.normal_weights(M, K, dtype, seed=601)
    A = g.pack(W, dtype, BR, BC, mask.row_ptr, mask.row_idx, mask.col_ptr, mask.col_idx, host_only=2, no_reorder=not reorder)
    ref = A.unpack()
    got = np.full_like(ref, 1)
    height, decode = (16, decoders.grim_test_decode_gather32) if dtype == gen.F32 else (64, decoders.grim_test_decode_64_row_runs)
    has = height % BR == 0 or BR % height == 0
    if dtype == gen.F32:
        has = has and BR <= 64
    res = decode(A.handle, got.ctypes.data, K)
    assert res == (0 if has else 1)
    if has:
        assert got.tobytes() == ref.tobytes()


def _sizes_of_one_block_groups(mask, M, K, BR, BC, max_rows, g_most, most_bytes):
    """Sizes of a staged layout in which every group of k slots belongs to one block, at the largest chunk that fits."""
    nbr, nbc = M // BR, K // BC
    kr, kc = np.diff(mask.row_ptr).reshape(nbr, nbc), np.diff(mask.col_ptr).reshape(nbr, nbc)
    ng, hdr = (4, 6) if BR == 16 else (2, 3)                    # groups to a step, 16-byte units of a step's header
    groups = np.where(kr > 0, (kc + 7) // 8, 0)
    blocks = max(1, max_rows // BC)
    while True:
        nchunks = -(-nbc // blocks)
        most = {}
        for g in (4, 8, 16, 32):
            most[g] = max(int(sum(-(-int(groups[s, c:c + blocks].sum()) // ng) * hdr + int((groups * kr)[s, c:c + blocks].sum())
                                  for s in range(t, min(nbr, t + g)))) for c in range(0, nbc, blocks) for t in range(0, nbr, g))
        if most[g_most] * 16 <= most_bytes or blocks == 1:
            return blocks * BC, nchunks, most
        blocks = (blocks + 1) // 2


def _wide_forms(BR, K, rows, nchunks, most):
    """(tile, kernel taps; 0: a product) that have room for the records: eight 16-byte units per fetching thread (four beside the rows of
    192 columns), two stages and the tables of a convolution that needs them in 160 KB."""
    forms = set()
    for tn in (96,) if BR == 32 else (128, 192):
        stages = 2 * ((rows + 1) * (2 * tn + 32) + 16 * most[16])
        if most[16] > 256 * (4 if tn == 192 else 8) or stages > 160 * 1024:
            continue
        forms.add((tn, 0))
        for taps in (t for t in range(1, 256, 2) if K % t == 0):                # (kernels are odd both ways)
            ways = 256 // (taps * (tn // 8))
            by_tap = ways > 0 and -(-(-(-rows // taps)) // ways) <= (11 if tn == 96 else 15)
            tables = 0 if by_tap else (taps + 1) * (tn // 8) * 16 + 4 * (192 if BR == 32 else 128) * 8
            if stages + tables <= 160 * 1024:
                forms.add((tn, taps))
    return forms


def _staged_forms(BR, K, rows, nchunks, most):
    """(tile, strips) that have room: 16 KB of records for four strips, 32 for eight, 48 for sixteen, two stages in 160 KB."""
    forms = set()
    for tn in (32, 64, 128):
        for strips in (4, 8, 16):
            if (tn == 128 and strips != 4) or (BR == 32 and strips // min(strips, 8) * (tn // 32) > 4):
                continue
            kb = -(-most[strips] * 16 // 1024)
            if kb <= {4: 16, 8: 32, 16: 48}[strips] and 2 * ((rows + 1) * tn * 2 + (kb + 1) * 1024) + nchunks * (strips + 1) * 8 <= 160 * 1024:
                forms.add((tn, strips))
    return forms


@pytest.mark.parametrize("BR,BC,kr,kc", [
    (16, 16, (6,), (4, 8)),             # groups that blocks share take more room than 192-column tiles have
    (16, 16, (8,), (4, 12)),
    (16, 16, (4, 8, 16), (6, 10)),
    (32, 16, (12,), (4, 8, 16)),        # ... and would need smaller chunks
    (32, 16, (8, 16, 32), (4, 8, 16)),
    (32, 16, (10,), (4, 8)),
    (32, 32, (16,), (12,)),
    (32, 32, (8, 16, 32), (6, 10)),
    (32, 32, (4, 8, 16), (4, 8, 16)),
    (16, 32, (8,), (8,)),
])
def test_staged_layouts_have_room_in_every_form_that_one_block_groups_have(decoders, BR, BC, kr, kc):
    """A launch form that a caller asks for by its tile is refused where a chunk's records have no room: packing columns of several
    blocks into a group must not take one away, nor a row from a chunk."""
    M, K = 16 * BR, 768
    for seed in range(4):
        mask = gen.random_mask(M, K, BR, BC, kr, kc, seed=900 + seed)
        W = gen.normal_weights(M, K, gen.F16, seed=901)
        A = g.pack(W, gen.F16, BR, BC, mask.row_ptr, mask.row_idx, mask.col_ptr, mask.col_idx, host_only=2, no_reorder=True)
        for wide, forms, max_rows, g_most, most_bytes in ((0, _staged_forms, 256, 4, 16 * 1024),
                                                          (1, _wide_forms, 192 if BR == 32 else 128, 16, 32 * 1024)):
            out = np.zeros(6, dtype=np.int64)
            assert decoders.grim_test_staged_sizes(A.handle, wide, out.ctypes.data_as(ctypes.c_void_p)) == 0
            rows, nchunks, most = _sizes_of_one_block_groups(mask, M, K, BR, BC, max_rows, g_most, most_bytes)
            assert out[0] >= rows, (wide, seed, out, rows)
            missing = forms(BR, K, rows, nchunks, most) - forms(BR, K, int(out[0]), int(out[1]), dict(zip((4, 8, 16, 32), out[2:].tolist())))
            assert not missing, (wide, seed, sorted(missing)[:5], out, rows, most)

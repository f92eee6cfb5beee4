"""The host side of the library under the address and undefined-behaviour sanitizers (no GPU).

csrc/bcr_pack.cpp -- validation, compaction into the canonical arrays, the derived kernel layouts and
their decoders, the BCRC export -- is built with g++ -fsanitize=address,undefined, with decoders for the layouts
that the library itself has none for (tests/sanitize/derived_layouts.cpp), against stand-ins for the
kernel launchers (tests/sanitize/device_stubs.cpp), and the host-side test files run against that build in a
child interpreter with the sanitizer runtimes preloaded.  Any out-of-bounds access, use after free or
undefined operation in the index-building code aborts the child and fails this test."""
import ctypes
import os
import subprocess
import sys

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
HOST_TESTS = ["tests/test_host_pack.py", "tests/test_bcrc_export.py", "tests/test_host_layouts.py", "tests/test_host_plan.py"]


def _runtime(name):
    path = subprocess.run(["g++", f"-print-file-name={name}"], capture_output=True, text=True).stdout.strip()
    return path if os.path.isabs(path) and os.path.exists(path) else None


def test_host_code_is_clean_under_asan_and_ubsan(tmp_path):
    asan, ubsan = _runtime("libasan.so"), _runtime("libubsan.so")
    if not asan or not ubsan:
        pytest.skip("g++ sanitizer runtimes not installed")
    lib = str(tmp_path / "libgrim_bcr_sanitized.so")
    build = ["g++", "-std=c++17", "-O1", "-g", "-fno-omit-frame-pointer", "-fsanitize=address,undefined",
             "-fno-sanitize-recover=undefined", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include",
             "-I", os.path.join(ROOT, "include"), "-I", os.path.join(ROOT, "paper_2108_11033_amd", "csrc"),
             "-shared", "-fPIC", "-Wl,-Bsymbolic",
             os.path.join(ROOT, "tests", "sanitize", "derived_layouts.cpp"),
             os.path.join(ROOT, "tests", "sanitize", "device_stubs.cpp"), "-o", lib]
    res = subprocess.run(build, capture_output=True, text=True)
    assert res.returncode == 0, res.stderr[-4000:]
    env = dict(os.environ)
    env["GRIM_BCR_LIB"] = lib
    preload = [asan, ubsan] + ([env["LD_PRELOAD"]] if env.get("LD_PRELOAD") else [])
    env["LD_PRELOAD"] = ":".join(preload)
    # Python itself is not instrumented: no leak report at exit, and the runtime may come after other preloads
    env["ASAN_OPTIONS"] = "detect_leaks=0:verify_asan_link_order=0:abort_on_error=1"
    env["UBSAN_OPTIONS"] = "halt_on_error=1:print_stacktrace=1"
    run = subprocess.run([sys.executable, "-m", "pytest", "-x", "-q", "-p", "no:cacheprovider", "-m", "not gpu"] + HOST_TESTS,
                         cwd=ROOT, env=env, capture_output=True, text=True, timeout=900)
    tail = (run.stdout + run.stderr)[-4000:]
    assert run.returncode == 0, tail
    assert "passed" in run.stdout and "skipped" not in run.stdout and "AddressSanitizer" not in tail and "runtime error" not in tail, tail


def _host_library(tmp_path, name):
    """tests/sanitize/<name>.cpp built for the host with the library's headers."""
    lib = str(tmp_path / (name + ".so"))
    res = subprocess.run(["g++", "-std=c++17", "-O2", "-shared", "-fPIC", "-I", os.path.join(ROOT, "paper_2108_11033_amd", "csrc"),
                          os.path.join(ROOT, "tests", "sanitize", name + ".cpp"), "-o", lib], capture_output=True, text=True)
    assert res.returncode == 0, res.stderr[-4000:]
    return ctypes.CDLL(lib)


def test_convolution_loads_without_range_checks_stay_inside_the_map(tmp_path):
    """Every load of every tile that the convolution kernels fetch without range checks, by their own arithmetic
    (csrc/conv_window.hpp) built for the host: small, flat and odd maps, both strides and both tile widths."""
    outside = _host_library(tmp_path, "conv_windows").conv_loads_outside
    outside.restype = ctypes.c_int64
    sizes = list(range(1, 21)) + list(range(21, 131, 3)) + [33, 47, 48, 63, 64, 65, 79, 95, 111, 112, 113, 128, 129]
    for stride in (1, 2):
        for kh, kw in ((1, 1), (3, 3), (1, 3), (3, 1), (5, 5)):
            for H in (1, 2, 3, 4, 5, 6, 7, 8, 9, 13, 14, 15, 28, 57):
                for W in sizes:
                    for tn in (32, 64):
                        for Cin in (1, 3):
                            n = outside(Cin, H, W, kh, kw, stride, tn)
                            assert n == 0, (n, dict(Cin=Cin, H=H, W=W, kh=kh, kw=kw, stride=stride, tile=tn))


def test_patch_convolution_holds_every_pixel_its_taps_meet(tmp_path):
    """Every tap of every position of every tile of the patch convolution, by its own arithmetic (csrc/conv_patch.hpp): the pixel
    is among those the tile loads, there is room for it, and no load leaves the channel."""
    faults = _host_library(tmp_path, "conv_patches").conv_patch_faults
    faults.restype = ctypes.c_int64
    sizes = list(range(1, 20)) + [27, 28, 31, 33, 47, 48, 63, 64, 65, 66, 95, 112, 113, 131]
    for stride in (1, 2):
        for kh, kw in ((3, 3), (1, 3), (3, 1), (5, 5), (1, 5), (7, 3)):
            for H in (1, 2, 3, 4, 5, 7, 8, 9, 14, 28, 33):
                for W in sizes:
                    if H * W < 8:
                        continue
                    for odd in (0, 1):
                        assert faults(H, W, kh, kw, stride, odd) == 0, dict(H=H, W=W, kh=kh, kw=kw, stride=stride, odd=odd)


def test_patch_convolution_workgroups_of_eight_waves_have_a_compute_unit_each(tmp_path):
    """A workgroup of eight waves fills a compute unit: an XCD has 32, and one workgroup more would run behind the others."""
    lib = _host_library(tmp_path, "conv_patches")
    waves = ctypes.c_int()
    seen = set()
    for runs in range(1, 33):
        for tiles in range(1, 600 // runs + 2):
            each = lib.conv_patch_per_xcd(tiles, runs, ctypes.byref(waves))
            assert waves.value == (8 if each <= 32 else 4), (tiles, runs, each)
            seen.add((waves.value, tiles * runs <= 256))
    assert seen == {(8, True), (4, True), (4, False)}


def test_wide_convolution_rows_dealt_by_tap(tmp_path):
    """Every row and piece of a chunk has one fetching thread, whichever tap the chunk begins with; the narrow tiles of a rest, which
    are slower that way, keep the tables."""
    faults = _host_library(tmp_path, "conv_taps").conv_tap_faults
    for tn in (32, 96, 128, 192):
        for KK in (1, 3, 5, 9, 15, 21, 25, 49):
            for rows in (32, 64, 96, 128, 160, 192):
                n = faults(tn, KK, rows)
                assert n == (-1 if tn == 32 or KK * tn // 8 > 256 else n), (tn, KK, rows)
                assert n <= 0, (n, tn, KK, rows)
    assert faults(96, 9, 192) == faults(192, 9, 128) == faults(128, 1, 192) == 0


def test_groups_of_small_matrices_are_dealt_to_all_xcds(tmp_path):
    """Every unit of every matrix of a group has one workgroup, and no XCD has more of them than its share."""
    excess = _host_library(tmp_path, "group_map").group_map_excess
    for units in list(range(1, 40)) + [63, 64, 65, 128, 234]:
        for count in (1, 2, 3, 7, 8, 100, 211):
            assert excess(units, count) == 0, (units, count)


def test_uniform_groups_run_on_the_matrix_cores_where_they_are_quicker(tmp_path):
    on_cores = _host_library(tmp_path, "group_map").group_on_matrix_cores
    for (count, M, K, BR, BC, kr, kc, kept, batch), quicker in (
            # microseconds wave per strip, on the matrix cores
            ((16, 1824, 1696, 16, 32, 4, 12, 12, 2), False),      # 6.0, 8.5
            ((33, 896, 1632, 16, 32, 4, 12, 12, 2), False),       # 5.9, 8.6
            ((8, 3744, 1376, 8, 32, 4, 8, 14, 3), False),         # 7.3, 10.4
            ((199, 128, 1504, 16, 32, 4, 12, 12, 8), False),      # 7.9, 11.5
            ((226, 128, 1952, 16, 32, 4, 12, 12, 5), False),      # 8.4, 13.4
            ((9, 2880, 1888, 8, 32, 4, 8, 14, 2), False),         # 7.0, 10.1
            ((16, 2048, 1024, 32, 32, 8, 8, 8, 2), True),         # 5.9, 4.4
            ((16, 2048, 1024, 32, 32, 8, 8, 8, 8), True),         # 9.0, 4.9
            ((32, 1024, 512, 8, 32, 4, 8, 14, 2), True),          # 6.0, 4.5
            ((64, 1024, 1024, 32, 32, 8, 8, 8, 2), False)):       # 6.9, 9.2: 4096 pairs
        assert on_cores(count, M, K, BR, BC, kr, kc, kept, batch) == quicker, (count, M, K, BR, BC, kr, kc, batch)


def test_sequence_sets_placed_on_xcds_crowd_none(tmp_path):
    """Workgroups of a sequence call wait for one another: placing its sets on XCDs must not put more of them on any XCD than
    the plain order does, or calls on several streams could each hold a part of one XCD and wait for the rest."""
    excess = _host_library(tmp_path, "seq_placement").seq_placement_excess
    for sets in range(1, 33):
        for wgs in (1, 2, 3, 7, 8, 31, 32, 64):
            assert excess(sets, wgs) == 0, (sets, wgs)


@pytest.mark.parametrize("polls", [0, 1, 4, 64])
def test_claimed_sets_have_every_workgroup_once(tmp_path, polls):
    """Whatever order the workgroups of a call run in, wherever, and whenever one of them calls the claim off: every (set, number) is
    one workgroup's, placed sets are on one XCD each, and the call ends where the chip has room for its sets."""
    outcome = _host_library(tmp_path, "seq_claim").seq_claim_outcome
    modes = {}
    for sets, wgs in [(1, 2), (1, 32), (3, 8), (5, 16), (7, 4), (9, 2), (12, 8), (13, 3), (15, 16), (25, 2), (25, 8), (29, 2), (31, 2), (31, 8)]:
        for xcds in range(4):
            grid = 8 * ((sets + 7) // 8) * wgs
            for room in sorted({sets * wgs, (sets * wgs + grid) // 2, grid}):
                for seed in range(3 if grid > 64 else 20):
                    mode = outcome(sets, wgs, xcds, polls, room, seed)
                    assert mode > 0, (mode, sets, wgs, xcds, room, seed)
                    modes.setdefault(mode, 0)
                    modes[mode] += 1
    assert 2 in modes and (polls < 64 or modes[1] > modes[2]), modes          # called off with few polls, mostly placed with many


def test_sets_are_claimed_where_that_is_quicker(tmp_path):
    claimed = _host_library(tmp_path, "seq_placement").seq_form_is_claimed
    for (sets, wgs, steps), quicker in (
            # microseconds in the plain order, claimed
            ((1, 32, 8), False), ((1, 32, 10), True),             # 21.2, 21.8; 25.2, 24.9
            ((7, 32, 8), False), ((7, 32, 12), True),             # 21.9, 22.9; 30.1, 29.3
            ((1, 8, 8), True), ((7, 8, 8), True),                 # 21.4, 18.7; 21.0, 20.6
            ((12, 8, 8), False), ((12, 8, 10), False), ((12, 8, 16), True),      # 21.0, 22.1; 24.9, 25.3; 36.5, 33.8
            ((25, 8, 12), False), ((25, 8, 16), True),            # 28.7, 29.5; 36.5, 34.9
            ((12, 16, 8), False), ((12, 16, 16), True),           # 21.6, 23.5; 37.6, 35.4
            ((8, 32, 64), False), ((9, 32, 64), False)):          # placed by their numbers; no room for two sets on an XCD
        assert bool(claimed(sets, wgs, steps)) == quicker, (sets, wgs, steps)


def test_a_matrix_has_room_for_the_words_of_every_sequence(tmp_path):
    """Its exchange words are allocated by the first call on it; 12 n rows are an LSTM's gate matrix of 3 n units and the hidden
    side of a GRU of 4 n."""
    missing = _host_library(tmp_path, "seq_placement").seq_words_missing
    missing.restype, missing.argtypes = ctypes.c_int64, [ctypes.c_int64, ctypes.c_int64, ctypes.c_int, ctypes.c_int]
    for n in (1, 2, 5, 8, 10, 24, 32, 85, 96, 256, 341):
        for H in (3 * n, 4 * n):
            for BR in [d for d in (1, 2, 3, 4, 5, 8, 16, 32) if H % d == 0 and H // d <= 256]:
                for cus in (32, 80, 256, 304):
                    assert missing(12 * n, H, BR, cus) <= 0, (n, H, BR, cus)


def test_a_step_of_many_sequences_gives_up_after_one_wait(tmp_path):
    """A wait that is given up is a thread's last of the step, whichever of its workgroup's pairs of sequences it was for."""
    reads = _host_library(tmp_path, "seq_placement").seq_reads_of_a_step
    reads.restype = ctypes.c_int64
    for pairs in range(1, 17):
        waits = (pairs + 1) // 2
        assert reads(pairs, 2, -1, 1000) == waits
        for fails in range(waits):
            assert reads(pairs, 2, fails, 1000) == fails + 1000, (pairs, fails)


def test_division_by_an_inverse_made_beforehand(tmp_path):
    """Quotients around multiples of the divisor, up to the largest numbers a launch can hold, are those of the division."""
    faults = _host_library(tmp_path, "divide").divide_faults
    for d in list(range(1, 70)) + [127, 128, 129, 196, 255, 1000, 3136, 4097, 65535, 65536, 65537, 1 << 24, (1 << 30) + 1, (1 << 31) - 1]:
        for k in [0, 1, 2, 3, 100, 65535, 65536] + [(((1 << 31) - 1) // d) * f // 7 for f in range(8)]:
            assert faults(min(k * d, (1 << 31) - 1), d) == 0, (k, d)

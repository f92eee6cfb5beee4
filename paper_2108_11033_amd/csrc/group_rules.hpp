// Which kernel a group of uniformly pruned matrices runs on, where both apply: the rule of the launcher, on the host, where the tests
// of the dispatch use it too.
#pragma once
#include <cstdint>

namespace grim {

// A wave per (matrix, run) pair and no split of a run over waves, no partial tiles: enough pairs to fill the GPU.  Four waves to a
// run / a wave (16 bytes of a row): 64 of 2048 x 2048 of mixed rates at 8 columns 29.3 / 26.8 us, 43 of 3872 x 1248 at one 34.9 / 30.3, 32 of 1024
// x 512 in 8 x 32 blocks (2048 pairs of 7 steps) at 4 5.4 / 5.1; 39 of 960 x 1632 (2340 of 16 steps) 9.0 / 10.1, 12 of 2048 x
// 512 (1536) 6.3 / 6.4, 8 of 736 x 1440 (368) 5.2 / 7.5.
inline bool group_run_to_a_wave(int64_t pairs, int64_t steps) { return pairs >= 3072 || (pairs >= 2048 && steps <= 12 * pairs); }

// `count` matrices of nbr strips of nbc blocks keeping kr x kc, in `runs` 16-row runs each and `steps` steps of 32 in all, on `batch`
// columns: are they quicker on the matrix cores than on the wave-per-strip kernel for several columns?  Microseconds, by the runs,
// their steps and the rows of x that they fetch (just their bytes up to four columns, three of them slower than two or four) against
// the strips, their sums and their weights.  Fitted to 352 groups of 512 to 2048 (matrix, run) pairs that split a run over four waves,
// 8 and 11 % (rms); the matrix cores have to be estimated 10 % ahead.  307 of them run there, three of which lose 3 % or more, the worst
// 8; in all 1846 us with all of them there, 2755 with none, 1814 with this rule, 1801 with the quicker one each time.  A run to a
// wave was quicker there in all of 43 groups of 2048 to 2400 pairs.  Larger groups have not moved (of 300 with 2049 to 6144 pairs 276
// are quicker there, 24 lose up to 1.57 times; the estimates are not fitted to them).  Wave per strip / matrix cores: 16 of 1824 x 1696
// in 16 x 32 blocks keeping 4 x 12 at 2 columns 6.0 / 8.5 us, 199 of 128 x 1504 at 8 7.9 / 11.5, 9 of 2880 x 1888 in 8 x 32 blocks keeping
// 4 x 8 at 2 7.0 / 10.1; 16 of 2048 x 1024 keeping 8 x 8 in 32 x 32 at 2 / 4 / 8 5.7 / 7.3 / 9.0 against 4.4 / 4.5 / 4.9, 32 of 1024 x 512
// in 8 x 32 blocks 6.0 / 7.6 / 11.3 against 4.5 / 4.6 / 5.1.
inline bool group_quicker_on_matrix_cores(int64_t count, int64_t nbr, int64_t nbc, int32_t kr, int32_t kc, int64_t K, int64_t runs, int64_t steps, int32_t batch) {
    if (count * runs > 2048) return false;
    if (group_run_to_a_wave(count * runs, steps)) return true;
    const double pairs = (double)(count * runs), strips = (double)count * (double)nbr;
    const double step = batch > 4 ? 1.87e-4 : batch == 3 ? 1.73e-4 : 1.35e-4;
    const double cores = 2.6 + 0.53e-3 * pairs + step * (double)steps + 0.21e-6 * (double)count * (double)K * batch;
    const double waves = 4.0 + strips * (2.2e-5 * batch * (kr + kc) + 3.2e-7 * (double)nbc * kr * kc);
    return cores * 1.1 <= waves;
}

}  // namespace grim

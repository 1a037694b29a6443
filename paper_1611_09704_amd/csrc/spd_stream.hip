// spd_stream.hip -- the streaming form of the boxcar pass for the width lists
// 1..n, n <= 16 (Sec. 2.3 / Algorithm 1 with the fused threshold of Sec.
// 2.4).  The arithmetic lives in spd_device.h (boxcar_run_fast,
// boxcar_run_short).
//
// Each row's starts are cut into runs of `steps` steps, one wave per run, four
// runs per work-group.  A run that lies wholly inside its row (every start
// valid, every sample it reads inside the row), with both outputs on vector
// boundaries or none at all, takes boxcar_run_fast; the others (each row's
// first and last run) boxcar_run_short.
#include <algorithm>

#include "spd_device.h"
#include "spd_kernels.h"

namespace spd {

template <int DT, int N, bool OUT>
__global__ __launch_bounds__(256) void boxcar_stream_kernel(PlaneArg pl, const spd_row_stats* stats, BoxcarArgs ba,
                                                            WidthPlan wp)
{
    extern __shared__ float smem[];
    const uint32_t wg = (uint32_t)xcd_remap(blockIdx.x, gridDim.x), per = (uint32_t)ba.tiles_per_row;
    const int64_t r = wg / per;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int64_t run = (int64_t)(wg % per) * (int64_t)(blockDim.x >> 6) + wave;
    const int64_t len = (int64_t)ba.steps * kStreamStep;
    const int64_t t0 = run * len - stream_origin(ba, r);
    if (t0 >= ba.nout) return;
    const spd_row_stats st = stats[ba.scope == SPD_SCOPE_ROW ? r : 0];
    float* buf = smem + (size_t)wave * 2 * kStreamBuf;
    // OUT: both outputs given and their offsets from a vector boundary agree
    if (t0 >= 0 && t0 + len <= ba.nout && t0 + len + 16 <= pl.n_cols && (OUT || (!ba.snr && !ba.widx)))
        boxcar_run_fast<DT, N, OUT>(pl, r, t0, st, ba, wp, buf);
    else
        boxcar_run_short<DT, N>(pl, r, t0, st, ba, wp, buf);
}

template <int DT, int N>
static hipError_t launch_n(const PlaneArg& pl, const spd_row_stats* stats, const BoxcarArgs& ba, const WidthPlan& wp,
                           bool out, int waves, uint64_t grid, size_t lds, hipStream_t s)
{
    if constexpr (N < 16) {
        if (wp.n != N) return launch_n<DT, N + 1>(pl, stats, ba, wp, out, waves, grid, lds, s);
    }
    if (out)
        hipLaunchKernelGGL((boxcar_stream_kernel<DT, N, true>), dim3(grid), dim3(64 * waves), lds, s, pl, stats, ba, wp);
    else
        hipLaunchKernelGGL((boxcar_stream_kernel<DT, N, false>), dim3(grid), dim3(64 * waves), lds, s, pl, stats, ba, wp);
    return hipGetLastError();
}

hipError_t launch_stream(int dtype, const PlaneArg& pl, const spd_row_stats* stats, const BoxcarArgs& ba0,
                         const WidthPlan& wp, int waves, hipStream_t s)
{
    if (wp.n < 1 || wp.n > 16) return hipErrorInvalidValue;
    const size_t lds = (size_t)waves * 2 * kStreamBuf * sizeof(float);
    BoxcarArgs ba = ba0;
    const int64_t steps = (ba.nout + 15 + kStreamStep - 1) / kStreamStep;   // of any row
    // Long runs amortise a wave's start (coefficients, first loads), short ones give small planes enough waves:
    // 8 steps against 4 and 2 take 1582, 1644 and 1756 us on 2,048 x 524,281 U8 (262,000 waves), 38.6,
    // 38.3 and 36.0 on 256 x 65,536 F32, 19.1, 14.7 and 13.1 on 64 x 65,536 F32 (30.2 with 16).
    auto wave_count = [&](int64_t per) { return pl.n_rows * ((steps + per - 1) / per); };
    ba.steps = wave_count(kStreamSteps) >= 32768 ? kStreamSteps : wave_count(kStreamSteps / 2) >= 16384 ? kStreamSteps / 2
                                                                                                       : kStreamSteps / 4;
    auto tiles = [&](int64_t per) { return ((steps + per - 1) / per + waves - 1) / waves; };   // per row
    while ((uint64_t)pl.n_rows * (uint64_t)tiles(ba.steps) * 64u * (uint64_t)waves > kMaxGridItems) ba.steps *= 2;
    ba.tiles_per_row = tiles(ba.steps);
    // 16-byte SNR stores and 4-byte width-index stores on one grid of starts
    const bool out = ba.snr && ba.widx && (((uintptr_t)ba.snr / 4 - (uintptr_t)ba.widx) & 3) == 0;
    const uint64_t grid = (uint64_t)pl.n_rows * (uint64_t)ba.tiles_per_row;
    switch (dtype) {
    case SPD_F32: return launch_n<SPD_F32, 1>(pl, stats, ba, wp, out, waves, grid, lds, s);
    case SPD_F16: return launch_n<SPD_F16, 1>(pl, stats, ba, wp, out, waves, grid, lds, s);
    default: return launch_n<SPD_U8, 1>(pl, stats, ba, wp, out, waves, grid, lds, s);
    }
}

}  // namespace spd

// spd_stream.hip -- the streaming form of the boxcar pass for the width lists
// 1..n, n <= 16 (Sec. 2.3 / Algorithm 1 with the fused threshold of Sec.
// 2.4).  The arithmetic lives in spd_device.h (boxcar_run_fast,
// boxcar_run_short).
//
// Each row's starts are cut into runs of `steps` steps, one wave per run, up to
// four runs per work-group (stream_shape).  A run that lies wholly inside its row (every start
// valid, every sample it reads inside the row), with both outputs on vector
// boundaries or none at all, takes boxcar_run_fast; the others (each row's
// first and last run) boxcar_run_short.
#include "spd_device.h"
#include "spd_kernels.h"

namespace spd {

template <int DT, int N, bool OUT, bool ONCE>
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
        boxcar_run_fast<DT, N, OUT, ONCE>(pl, r, t0, st, ba, wp, buf);
    else
        boxcar_run_short<DT, N>(pl, r, t0, st, ba, wp, buf);
}

template <int DT, int N>
static hipError_t launch_n(const PlaneArg& pl, const spd_row_stats* stats, const BoxcarArgs& ba, const WidthPlan& wp,
                           bool out, bool once, int waves, uint64_t grid, size_t lds, hipStream_t s)
{
    if constexpr (N < 16) {
        if (wp.n != N) return launch_n<DT, N + 1>(pl, stats, ba, wp, out, once, waves, grid, lds, s);
    }
    const dim3 g(grid), b(64 * waves);
    if (out && once)
        hipLaunchKernelGGL((boxcar_stream_kernel<DT, N, true, true>), g, b, lds, s, pl, stats, ba, wp);
    else if (out)
        hipLaunchKernelGGL((boxcar_stream_kernel<DT, N, true, false>), g, b, lds, s, pl, stats, ba, wp);
    else if (once)
        hipLaunchKernelGGL((boxcar_stream_kernel<DT, N, false, true>), g, b, lds, s, pl, stats, ba, wp);
    else
        hipLaunchKernelGGL((boxcar_stream_kernel<DT, N, false, false>), g, b, lds, s, pl, stats, ba, wp);
    return hipGetLastError();
}

hipError_t launch_stream(int dtype, const PlaneArg& pl, const spd_row_stats* stats, const BoxcarArgs& ba0,
                         const WidthPlan& wp, hipStream_t s)
{
    if (wp.n < 1 || wp.n > 16) return hipErrorInvalidValue;
    const StreamShape f = stream_shape(pl.n_rows, ba0.nout, ba0.snr || ba0.widx);
    const int waves = f.waves;
    const size_t lds = (size_t)waves * 2 * kStreamBuf * sizeof(float);
    BoxcarArgs ba = ba0;
    ba.steps = f.steps;
    ba.aligned = f.aligned;
    const bool once = stream_once(pl.n_rows * pl.n_cols * (dtype == SPD_F32 ? 4 : dtype == SPD_F16 ? 2 : 1));
    ba.tiles_per_row = f.tiles_per_row;
    // 16-byte SNR stores and 4-byte width-index stores on one grid of starts
    const bool out = ba.snr && ba.widx && (((uintptr_t)ba.snr / 4 - (uintptr_t)ba.widx) & 3) == 0;
    const uint64_t grid = (uint64_t)pl.n_rows * (uint64_t)ba.tiles_per_row;
    switch (dtype) {
    case SPD_F32: return launch_n<SPD_F32, 1>(pl, stats, ba, wp, out, once, waves, grid, lds, s);
    case SPD_F16: return launch_n<SPD_F16, 1>(pl, stats, ba, wp, out, once, waves, grid, lds, s);
    default: return launch_n<SPD_U8, 1>(pl, stats, ba, wp, out, once, waves, grid, lds, s);
    }
}

}  // namespace spd

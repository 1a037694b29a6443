// spd_kernels.hip -- one-plane launches of the detection path on gfx950.
//
//   msd_x_kernel / msd_xy_kernel   per-block (n, T, S) partials, Sec. 2.1
//   msd_finalize(_lanes)_kernel    FP64 merge across blocks and sigma_N
//                                  coefficients, Sec. 2.1-2.2
//   boxcar_kernel                  boxcars, SNR, highest SNR and its width,
//                                  fused threshold, Sec. 2.3 / Algorithm 1,
//                                  Sec. 2.4 (starts 64 apart per lane)
//   boxcar_win_kernel              the same with 8 consecutive starts per lane
//                                  and each group's reads held in registers
//   boxcar_dit_kernel              boxcars combined with decimation in time
//                                  (widths 2^l*(9..16) on the decimated series)
// (the streaming form of the lists 1..n, n <= 16, is in spd_stream.hip)
//   select_kernel                  threshold over stored outputs, Sec. 2.4
//
// One work-group per (row, column block) or (row, time tile), numbered so that
// each XCD gets a contiguous range (a grid's numbers fit in 32 bits).  The arithmetic lives in spd_device.h.
#include "spd_device.h"
#include "spd_kernels.h"

namespace spd {

template <int DT>
__global__ __launch_bounds__(256) void msd_x_kernel(PlaneArg pl, bool vec, int64_t ncb, int64_t bc,
                                                    int64_t nblk, double* part)
{
    __shared__ MsdScratch sh;
    const uint32_t wg = (uint32_t)xcd_remap(blockIdx.x, gridDim.x);
    const int64_t r = wg / (uint32_t)nblk, b = wg % (uint32_t)nblk;
    msd_block_x<DT>(pl, vec, r, b, ncb, bc, part + (size_t)wg * 6, sh);
}

template <int DT>
__global__ __launch_bounds__(256) void msd_xy_kernel(PlaneArg pl, bool vec, int64_t ncb, int64_t bc,
                                                     int64_t nblk, int32_t nmax, int64_t nout, double* part)
{
    __shared__ MsdScratch sh;
    const uint32_t wg = (uint32_t)xcd_remap(blockIdx.x, gridDim.x);
    const int64_t r = wg / (uint32_t)nblk, b = wg % (uint32_t)nblk;
    msd_block_xy<DT>(pl, vec, r, b, ncb, bc, nmax, nout, part + (size_t)wg * 6, sh);
}

// `zero` (may be NULL): a counter for the launches after this one to add to.
__global__ __launch_bounds__(256) void msd_finalize_kernel(const double* part, int64_t per_unit,
                                                           int32_t need_y, int32_t accumulate,
                                                           spd_msd_state* state, spd_row_stats* stats,
                                                           int32_t nmax, int32_t mode, double kappa, int64_t* zero)
{
    __shared__ FinalizeScratch sh;
    const int64_t u = blockIdx.x;
    finalize_unit(part + (size_t)u * per_unit * 6, per_unit, need_y != 0, accumulate != 0,
                  state ? state + u : nullptr, stats + u, nmax, mode, kappa, sh);
    // last: before the merge it takes a scalar load and 0.2 us of its own (3 rows of 306 partials 5.6 us, 5.4 here)
    if (threadIdx.x == 0 && u == 0 && zero) *zero = 0;
}

// Units of few partials: a wave takes 64 / lanes of them.  All latency (the
// loads, then log2(lanes) dependent FP64 merges), so a work-group per unit only
// adds work-groups to start and tree levels of nothing: 64 units of 4 partials
// 4.6 -> 3.2 us; with the count reset in here as well, detection of 64 x 65,536
// F32 with 1..32 goes from 32.5 to 29.1 us.
__global__ __launch_bounds__(64) void msd_finalize_lanes_kernel(const double* part, int64_t units, int32_t per_unit,
                                                                int32_t lanes, int32_t need_y, int32_t accumulate,
                                                                spd_msd_state* state, spd_row_stats* stats,
                                                                int32_t nmax, int32_t mode, double kappa, int64_t* zero)
{
    if (zero && blockIdx.x == 0 && threadIdx.x == 0) *zero = 0;
    const int64_t u = (int64_t)blockIdx.x * (64 / lanes) + threadIdx.x / lanes;
    const bool on = u < units;
    finalize_unit_lanes(part + (on ? u : 0) * per_unit * 6, per_unit, lanes, on, need_y != 0, accumulate != 0,
                        state ? state + u : nullptr, stats + u, nmax, mode, kappa);
}

template <int DT, int X, bool UNIT, int SMALL>
__global__ __launch_bounds__(256) void boxcar_kernel(PlaneArg pl, bool vec, const spd_row_stats* stats,
                                                     BoxcarArgs ba, WidthPlan wp)
{
    extern __shared__ float smem[];
    const uint32_t tile = (uint32_t)xcd_remap(blockIdx.x, gridDim.x), per = (uint32_t)ba.tiles_per_row;
    const int64_t r = tile / per, tt = tile % per;
    const spd_row_stats st = stats[ba.scope == SPD_SCOPE_ROW ? r : 0];
    boxcar_tile<DT, X, UNIT, SMALL>(pl, vec, r, tt, st, ba, wp, smem, true);
}

// The group form holds each start's running sum, maximum, group and group-start
// sum plus two groups' windows; capping it at 128 VGPRs keeps 4 waves per SIMD
// without spills (uncapped it takes 132 and drops to 3).  The lists that step by
// 1 throughout (1..24, 1..32, ...) have a variant of their own without the
// step's choice: 74 VGPRs, 6 waves per SIMD.  Bound by the vector units (two
// instructions per start and width); with the window's loads in flight before
// the tables are made, at any alignment of the rows: U8 1024 x 262144, 1..64,
// 1,524 -> 1,276 us on contiguous rows; F32 1024 x 262144, 1..32, 1,266 -> 902 us
// and 1..128 2,231 -> 2,017 us; the mixed Sec. 3.3 list 2,690 -> 2,627 us.
template <int DT, int SMALLN, bool UNIT = false>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(SMALLN == 0 ? 4 : 1))) void boxcar_win_kernel(PlaneArg pl, bool vec, const spd_row_stats* stats,
                                                         BoxcarArgs ba, WidthPlan wp)
{
    extern __shared__ float smem[];
    const uint32_t tile = (uint32_t)xcd_remap(blockIdx.x, gridDim.x), per = (uint32_t)ba.tiles_per_row;
    const int64_t r = tile / per, tt = tile % per;
    const spd_row_stats st = stats[ba.scope == SPD_SCOPE_ROW ? r : 0];
    boxcar_tile_win<DT, SMALLN, false, UNIT>(pl, vec, r, tt, st, ba, wp, smem);
}

// Boxcars combined with decimation in time: widths 1..16 at every start, and
// 2^l*(9..16) at starts that are multiples of 2^l, l = 1..levels.  Bound by HBM
// (9 bytes a start) and the vector units together.  The levels share two LDS
// regions (23 KB a work-group instead of 30 at four levels) and a cap of 80 VGPRs,
// which spills 2 or 3 of them to scratch, gives 6 waves per SIMD instead of 5: 2,048 x 524,288 with statistics 4,091 -> 4,050 us.
template <int DT>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(6))) void boxcar_dit_kernel(PlaneArg pl, bool vec, const spd_row_stats* stats,
                                                         BoxcarArgs ba, WidthPlan wp)
{
    extern __shared__ float smem[];
    const uint64_t tile = xcd_remap(blockIdx.x, gridDim.x);
    const int64_t r = (int64_t)(tile / (uint64_t)ba.tiles_per_row);
    const int64_t tt = (int64_t)(tile % (uint64_t)ba.tiles_per_row);
    const spd_row_stats st = stats[ba.scope == SPD_SCOPE_ROW ? r : 0];
    boxcar_tile_win<DT, kDitBase, true>(pl, vec, r, tt, st, ba, wp, smem);
}

// Sec. 2.4 over stored snr / width-index arrays.  A work-group covers kSelCols
// columns of one row, 16 per lane in dword loads 256 columns apart: every load
// instruction reads 256 consecutive bytes per wave, and sixteen loads per lane
// are in flight (measured faster than four 16-byte loads per lane, even on
// aligned rows).  A wave with no SNR at the threshold stops there; the others
// compact with one ballot per value and one atomic per wave.
__global__ __launch_bounds__(256) void select_kernel(const float* snr, const uint8_t* widx,
                                                     int64_t ncols, int64_t stride, int64_t chunks,
                                                     SelectArgs sa)
{
    const int tid = threadIdx.x;
    const uint64_t blk = xcd_remap(blockIdx.x, gridDim.x);
    const int64_t r = (int64_t)(blk / (uint64_t)chunks), ch = (int64_t)(blk % (uint64_t)chunks);
    const float* row = snr + r * stride;
    const int64_t p0 = ch * kSelCols + tid;                         // column of v[i] is p0 + 256i
    float v[16];
#pragma unroll
    for (int i = 0; i < 16; ++i) {
        const int64_t t = p0 + 256 * i;
        v[i] = t < ncols ? row[t] : -INFINITY;                     // never at a finite threshold
    }
    float m = v[0];
#pragma unroll
    for (int i = 1; i < 16; ++i) m = fmaxf(m, v[i]);
    if (!__ballot(m >= sa.threshold)) return;                      // the whole wave leaves
    CandSlots slots;
#pragma unroll
    for (int i = 0; i < 16; ++i) slots.add(i, v[i] >= sa.threshold);
    unsigned long long k = slots.take(sa.cand_count);
#pragma unroll
    for (int i = 0; i < 16; ++i) {
        if (!slots.has(i)) continue;
        if (k < (unsigned long long)sa.cand_capacity) {
            const int64_t t = p0 + 256 * i;
            spd_candidate cd;
            cd.row = (int32_t)r;
            cd.width = sa.width[widx[r * stride + t]];
            cd.t = t + sa.t_offset;
            cd.snr = v[i];
            cd.beam = 0;
            sa.cand[k] = cd;
        }
        ++k;
    }
}

__global__ void fill_i64_kernel(int64_t* p, int64_t n, int64_t v)
{
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) p[i] = v;
}

// ---------------------------------------------------------------------------
// launchers
// ---------------------------------------------------------------------------

template <int DT>
static hipError_t launch_msd_dt(const PlaneArg& pl, bool vec, bool with_y, int64_t ncb, int64_t bc,
                                int64_t nblk, int32_t nmax, int64_t nout, double* part, hipStream_t s)
{
    const uint64_t nwg = (uint64_t)pl.n_rows * (uint64_t)nblk;
    if (!with_y) {
        hipLaunchKernelGGL((msd_x_kernel<DT>), dim3(nwg), dim3(256), 0, s, pl, vec, ncb, bc, nblk, part);
    } else {
        hipLaunchKernelGGL((msd_xy_kernel<DT>), dim3(nwg), dim3(256), 0, s, pl, vec, ncb, bc, nblk, nmax, nout,
                           part);
    }
    return hipGetLastError();
}

hipError_t launch_msd(int dtype, const PlaneArg& pl, bool vec, bool with_y, int64_t ncb, int64_t bc,
                      int64_t nblk, int32_t nmax, int64_t nout, double* part, hipStream_t s)
{
    switch (dtype) {
    case SPD_F32: return launch_msd_dt<SPD_F32>(pl, vec, with_y, ncb, bc, nblk, nmax, nout, part, s);
    case SPD_F16: return launch_msd_dt<SPD_F16>(pl, vec, with_y, ncb, bc, nblk, nmax, nout, part, s);
    default: return launch_msd_dt<SPD_U8>(pl, vec, with_y, ncb, bc, nblk, nmax, nout, part, s);
    }
}

hipError_t launch_finalize(const double* part, int64_t n_units, int64_t per_unit, bool need_y,
                           bool accumulate, spd_msd_state* state, spd_row_stats* stats, int32_t nmax,
                           int32_t mode, double kappa, int64_t* zero, hipStream_t s)
{
    if (per_unit <= kFinalizeLanes) {
        int lanes = 1;
        while (lanes < per_unit) lanes <<= 1;
        const int64_t per_wg = 64 / lanes;
        hipLaunchKernelGGL(msd_finalize_lanes_kernel, dim3((uint32_t)((n_units + per_wg - 1) / per_wg)), dim3(64), 0, s,
                           part, n_units, (int32_t)per_unit, lanes, (int32_t)need_y, (int32_t)accumulate, state, stats,
                           nmax, mode, kappa, zero);
        return hipGetLastError();
    }
    hipLaunchKernelGGL(msd_finalize_kernel, dim3((uint32_t)n_units), dim3(256), 0, s, part, per_unit,
                       (int32_t)need_y, (int32_t)accumulate, state, stats, nmax, mode, kappa, zero);
    return hipGetLastError();
}

size_t boxcar_lds_bytes(int waves, const BoxcarArgs& ba, bool win)
{
    return (size_t)(win ? kWinTableFloats : kTableFloats) * 4 + (size_t)waves * ba.wave_floats * 4;
}

template <int DT>
static hipError_t launch_boxcar_dt(const PlaneArg& pl, bool vec, const spd_row_stats* stats,
                                   const BoxcarArgs& ba, const WidthPlan& wp, int waves, uint64_t ntiles,
                                   hipStream_t s)
{
    const size_t lds = boxcar_lds_bytes(waves, ba, wp.win != 0);   // <= 64 KiB by construction of the plan
    constexpr int X = kOutPerLane;
    if (wp.win == 4)
        return launch_stream(DT, pl, stats, ba, wp, s);
    if (wp.win == 3)
        hipLaunchKernelGGL((boxcar_dit_kernel<DT>), dim3(ntiles), dim3(64 * waves), lds, s, pl, vec, stats, ba, wp);
    else if (wp.win == 1 && wp.win_unit)
        hipLaunchKernelGGL((boxcar_win_kernel<DT, 0, true>), dim3(ntiles), dim3(64 * waves), lds, s, pl, vec, stats, ba,
                           wp);
    else if (wp.win == 1)
        hipLaunchKernelGGL((boxcar_win_kernel<DT, 0>), dim3(ntiles), dim3(64 * waves), lds, s, pl, vec, stats, ba, wp);
    else if (wp.win == 2 && wp.n <= 8)
        hipLaunchKernelGGL((boxcar_win_kernel<DT, 8>), dim3(ntiles), dim3(64 * waves), lds, s, pl, vec, stats, ba, wp);
    else if (wp.win == 2)
        hipLaunchKernelGGL((boxcar_win_kernel<DT, 16>), dim3(ntiles), dim3(64 * waves), lds, s, pl, vec, stats, ba,
                           wp);
    else if (wp.unit_counts && wp.n <= 8)
        hipLaunchKernelGGL((boxcar_kernel<DT, X, true, 8>), dim3(ntiles), dim3(64 * waves), lds, s, pl, vec, stats,
                           ba, wp);
    else if (wp.unit_counts && wp.n <= 16)
        hipLaunchKernelGGL((boxcar_kernel<DT, X, true, 16>), dim3(ntiles), dim3(64 * waves), lds, s, pl, vec, stats,
                           ba, wp);
    else if (wp.unit_counts)
        hipLaunchKernelGGL((boxcar_kernel<DT, X, true, 0>), dim3(ntiles), dim3(64 * waves), lds, s, pl, vec, stats,
                           ba, wp);
    else
        hipLaunchKernelGGL((boxcar_kernel<DT, X, false, 0>), dim3(ntiles), dim3(64 * waves), lds, s, pl, vec, stats,
                           ba, wp);
    return hipGetLastError();
}

hipError_t launch_boxcar(int dtype, const PlaneArg& pl, bool vec, const spd_row_stats* stats,
                         const BoxcarArgs& ba, const WidthPlan& wp, int X, int waves, uint64_t ntiles,
                         hipStream_t s)
{
    (void)X;
    switch (dtype) {
    case SPD_F32: return launch_boxcar_dt<SPD_F32>(pl, vec, stats, ba, wp, waves, ntiles, s);
    case SPD_F16: return launch_boxcar_dt<SPD_F16>(pl, vec, stats, ba, wp, waves, ntiles, s);
    default: return launch_boxcar_dt<SPD_U8>(pl, vec, stats, ba, wp, waves, ntiles, s);
    }
}

hipError_t launch_fill_i64(int64_t* p, int64_t n, int64_t v, hipStream_t s)
{
    hipLaunchKernelGGL(fill_i64_kernel, dim3((uint32_t)((n + 255) / 256)), dim3(256), 0, s, p, n, v);
    return hipGetLastError();
}

hipError_t launch_zero_count(int64_t* count, hipStream_t s) { return launch_fill_i64(count, 1, 0, s); }

hipError_t launch_select(const float* snr, const uint8_t* widx, int64_t nrows, int64_t ncols,
                         int64_t stride, const SelectArgs& sa, hipStream_t s)
{
    const int64_t chunks = (ncols + kSelCols - 1) / kSelCols;
    const uint64_t nb = (uint64_t)nrows * (uint64_t)chunks;
    if (nb == 0) return hipSuccess;
    hipLaunchKernelGGL(select_kernel, dim3(nb), dim3(256), 0, s, snr, widx, ncols, stride, chunks, sa);
    return hipGetLastError();
}

}  // namespace spd

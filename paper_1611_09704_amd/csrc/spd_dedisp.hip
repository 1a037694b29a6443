// spd_dedisp.hip -- brute-force incoherent de-dispersion, the step before the
// detection path (Sec. 1: detection runs on de-dispersed time series).
//
// A filterbank of 8-bit samples x[c][s] (channel 0 the highest frequency)
// becomes one series per trial DM:
//     y[d][t] = sum over c of x[c][t + delay(d, c)],  t < n_samp - max delay,
// with delay(d, c) = floor(dm[d] * k_c + 0.5) and
// k_c = KDM * (1/f_c^2 - 1/f_top^2) / t_samp, the cold-plasma delay law.  The
// sums are of whole 8-bit counts, so they are exact in every form below and
// the output (float) holds them exactly (below 2^24 for the up to 65,536
// channels a plan accepts).
//
// Lists whose neighbouring trials lie within a few samples of delay, the common
// case, go to the matrix cores (dedisp_mfma_kernel below).  The kernels for any
// other list:
//
// Kernel layout (gfx950).  A work-group owns 16 consecutive trials x 512
// consecutive starts; each of its 4 waves owns 4 trials, and lane l the
// starts t0 + l + 64k (k < 8).  Channels come in chunks of up to 16, staged
// in LDS relative to g = (t0 + delay of the group's first trial) & ~3:
//  * wide layout (dedisp_u8_wide_kernel): entry e is 16
//    bytes holding x[g + e + 64k], k < 8, as 16-bit fields, so one 16-byte
//    LDS read gives a lane all 8 of its starts for a trial; the next chunk's
//    bytes are loaded into registers while the current one accumulates;
//  * narrow layout (dedisp_u8_kernel, any span of delays): entry e is 4
//    bytes holding x[g + e] and x[g + e + 64]; staging between barriers.
// Either way one 32-bit integer add accumulates two starts as 16-bit fields,
// flushed into 32-bit totals every 256 channels (256 * 255 < 65536).  Lanes
// read consecutive entries, so the reads are free of bank conflicts.  Each
// 4 bytes read from LDS carry two of the definition's additions, and the LDS
// read bandwidth is the binding resource.
//
// The delays are evaluated where they are used, in FP64, with the product and
// the sum rounded separately (no fused multiply-add), the same way the host
// evaluates them for the plan's maximum delay and span.

#include <hip/hip_runtime.h>
#include <math.h>
#include <stdint.h>
#include <stdlib.h>
#include <string.h>

#include <algorithm>
#include <new>
#include <vector>

#include "spd_abi_internal.h"
#include "spd_device.h"

namespace spd {
namespace {

constexpr double kKdm = 4.148808e3;          // MHz^2 pc^-1 cm^3 s
constexpr int kDdWaves = 4;
constexpr int kDdDmPerWave = 4;
constexpr int kDdDms = kDdWaves * kDdDmPerWave;   // trials per work-group
constexpr int kDdOut = 512;                       // starts per work-group
constexpr int kDdFlush = 256;                     // channels per 16-bit partial sum
constexpr int kDdMaxChunk = 16;                   // channels per LDS chunk (<= 256 / kDdDms)
constexpr size_t kDdLdsMax = 65536;

struct DedispArgs {
    const uint8_t* fb;
    int64_t stride, n_samp;
    const double* dm;
    const double* kc;
    float* out;
    int64_t out_stride, n_out;
    int32_t n_chan, n_dm, n_dm_tiles, entries, chunk;
    int32_t groups;          // wide layout: groups of 4 entries staged per channel
    int32_t max_delay;
};

// floor(dm * k + 0.5) with the product and the sum each rounded to FP64.
__host__ __device__ inline int32_t dd_delay(double dm, double k)
{
#pragma clang fp contract(off)
    const double p = dm * k;
    return (int32_t)floor(p + 0.5);
}

// Four bytes of a channel row from byte g on (g a multiple of 4); bytes at or
// beyond n_samp read as zero.
__device__ inline uint32_t dd_load4(const uint8_t* row, int64_t g, int64_t n_samp)
{
    if (g + 3 < n_samp) return *(const uint32_t*)(row + g);
    uint32_t v = 0;
    for (int i = 0; i < 4; ++i)
        if (g + i < n_samp) v |= (uint32_t)row[g + i] << (8 * i);
    return v;
}

// The chunk's accumulation: for each staged channel, the wave's 4 trials x
// 4 entries per lane, all 16 reads in flight before the adds.  my_off (lane
// cc < ncc) is channel cc's entry offset, my_dl (lane 4cc + j) trial j's
// delay minus the group's first trial's; both are read as scalars.
__device__ inline void dd_accumulate(const uint32_t* P, int ncc, int32_t my_off, int32_t my_dl, int lane,
                                     uint32_t (&part)[kDdDmPerWave][4])
{
    for (int cc = 0; cc < ncc; ++cc) {
        const int32_t off_c = __builtin_amdgcn_readlane(my_off, cc);
        uint32_t v[kDdDmPerWave][4];
#pragma unroll
        for (int j = 0; j < kDdDmPerWave; ++j) {
            const uint32_t* q = P + off_c + __builtin_amdgcn_readlane(my_dl, cc * kDdDmPerWave + j) + lane;
#pragma unroll
            for (int i = 0; i < 4; ++i) v[j][i] = q[128 * i];
        }
#pragma unroll
        for (int j = 0; j < kDdDmPerWave; ++j) {
#pragma unroll
            for (int i = 0; i < 4; ++i) part[j][i] += v[j][i];
        }
    }
}

// The 16-bit partial sums (fields: starts t and t + 64) into the 32-bit totals.
__device__ inline void dd_flush(uint32_t (&part)[kDdDmPerWave][4], uint32_t (&tot)[kDdDmPerWave][8])
{
#pragma unroll
    for (int j = 0; j < kDdDmPerWave; ++j) {
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            tot[j][2 * i] += part[j][i] & 0xffffu;
            tot[j][2 * i + 1] += part[j][i] >> 16;
            part[j][i] = 0;
        }
    }
}

__device__ inline void dd_store(const DedispArgs& a, int d0, int wv, int lane, int64_t t0,
                                const uint32_t (&tot)[kDdDmPerWave][8])
{
#pragma unroll
    for (int j = 0; j < kDdDmPerWave; ++j) {
        const int d = d0 + wv * kDdDmPerWave + j;
        if (d >= a.n_dm) continue;
        float* orow = a.out + (int64_t)d * a.out_stride;
#pragma unroll
        for (int k = 0; k < 8; ++k) {
            const int64_t t = t0 + lane + 64 * k;
            if (t < a.n_out) orow[t] = (float)tot[j][k];
        }
    }
}

// Entries 4q..4q+3 of a channel from the bytes A = x[g..g+3], B = x[g+64..g+67].
__device__ inline uint4 dd_pack(uint32_t A, uint32_t B)
{
    uint4 v;
    v.x = (A & 0xffu) | ((B & 0xffu) << 16);
    v.y = ((A >> 8) & 0xffu) | (((B >> 8) & 0xffu) << 16);
    v.z = ((A >> 16) & 0xffu) | (((B >> 16) & 0xffu) << 16);
    v.w = (A >> 24) | ((B >> 24) << 16);
    return v;
}

// Any chunk size and span: delays through LDS, staging between barriers.
__global__ __launch_bounds__(64 * kDdWaves) void dedisp_u8_kernel(DedispArgs a)
{
    extern __shared__ __align__(16) uint32_t dd_smem[];
    uint32_t* P = dd_smem;                                   // [chunk][entries]
    int32_t* dl = (int32_t*)(P + a.chunk * a.entries);       // [chunk][16] delay - first trial's delay
    int32_t* base = dl + a.chunk * kDdDms;                   // [chunk] first trial's delay
    const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
    const int64_t t0 = (int64_t)(blockIdx.x / (uint32_t)a.n_dm_tiles) * kDdOut;
    const int d0 = (int)(blockIdx.x % (uint32_t)a.n_dm_tiles) * kDdDms;

    uint32_t part[kDdDmPerWave][4] = {};
    uint32_t tot[kDdDmPerWave][8] = {};
    int since = 0;
    const int nq = a.entries / 4;
    for (int c0 = 0; c0 < a.n_chan; c0 += a.chunk) {
        const int ncc = min(a.chunk, a.n_chan - c0);
        __syncthreads();                                     // the previous chunk is consumed
        if (tid < ncc * kDdDms) {
            const int cc = tid / kDdDms, j = tid % kDdDms;
            const double k = a.kc[c0 + cc];
            const int32_t db = dd_delay(a.dm[d0], k);
            dl[tid] = dd_delay(a.dm[min(d0 + j, a.n_dm - 1)], k) - db;
            if (j == 0) base[cc] = db;
        }
        __syncthreads();
        // wave w stages channels w, w + 4, ...; lane l the entries 4q..4q+3, q = l, l + 64, ...
        for (int cc = wv; cc < ncc; cc += kDdWaves) {
            const uint8_t* row = a.fb + (int64_t)(c0 + cc) * a.stride;
            const int64_t g0 = (t0 + base[cc]) & ~(int64_t)3;
            uint32_t* pc = P + cc * a.entries;
            for (int q = lane; q < nq; q += 64)
                *(uint4*)(pc + 4 * q) = dd_pack(dd_load4(row, g0 + 4 * q, a.n_samp),
                                               dd_load4(row, g0 + 4 * q + 64, a.n_samp));
        }
        __syncthreads();
        const int32_t my_dl = (lane >> 2) < ncc ? dl[(lane >> 2) * kDdDms + wv * kDdDmPerWave + (lane & 3)] : 0;
        const int32_t my_off = lane < ncc ? lane * a.entries + (int)((t0 + base[lane]) & 3) : 0;
        dd_accumulate(P, ncc, my_off, my_dl, lane, part);
        since += ncc;
        if (since + a.chunk > kDdFlush || c0 + a.chunk >= a.n_chan) {
            dd_flush(part, tot);
            since = 0;
        }
    }
    dd_store(a, d0, wv, lane, t0, tot);
}

// ---------------------------------------------------------------------------
// Wide layout: entry e of a channel is 16 bytes holding x[g + e + 64k] for
// k < 8 as 16-bit fields (k = 2p, 2p+1 in dword p), so one 16-byte LDS read
// gives a lane all 8 of its starts for a trial, and the 4 dwords add into
// the same partial sums as above.  A channel needs 67 + span entries.
// ---------------------------------------------------------------------------
constexpr int kWideRounds = 2;              // staging items per thread per chunk (prefetching kernel)

// Entries 4m..4m+3 of a channel (dst = entry 4m) from D[k] = x[g + 4m + 64k
// .. +3], k < 8.  Entry 4m + b, dword p, is byte b of D[2p] | byte b of
// D[2p+1] << 16: one v_perm_b32 (selector bytes 0-3 pick from its second
// operand, 4-7 from its first, 0x0c gives zero).  The four 16-byte writes go
// out in the order b = (i + item/4) mod 4, i = 0..3, so that in each write
// instruction 16 consecutive items (lanes) hit 16 different 16-byte bank
// groups instead of four.
__device__ inline void dd_pack_wide(const uint32_t (&D)[8], int item, uint4* dst)
{
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const uint32_t b = (uint32_t)(i + (item >> 2)) & 3u;
        const uint32_t sel = 0x0c040c00u + b * 0x00010001u;
        dst[b] = make_uint4(__builtin_amdgcn_perm(D[1], D[0], sel), __builtin_amdgcn_perm(D[3], D[2], sel),
                            __builtin_amdgcn_perm(D[5], D[4], sel), __builtin_amdgcn_perm(D[7], D[6], sel));
    }
}

__device__ inline void dd_load_group(const uint8_t* row, int64_t g, int64_t n_samp, bool interior, uint32_t (&D)[8])
{
    if (interior) {
#pragma unroll
        for (int k = 0; k < 8; ++k) D[k] = *(const uint32_t*)(row + g + 64 * k);
    } else {
#pragma unroll
        for (int k = 0; k < 8; ++k) D[k] = dd_load4(row, g + 64 * k, n_samp);
    }
}

__device__ inline void dd_accumulate_wide(const uint4* P4, int ncc, int32_t my_off, int32_t my_dl, int lane,
                                          uint32_t (&part)[kDdDmPerWave][4])
{
    for (int cc = 0; cc < ncc; ++cc) {
        const int32_t off_c = __builtin_amdgcn_readlane(my_off, cc);
        uint4 v[kDdDmPerWave];
#pragma unroll
        for (int j = 0; j < kDdDmPerWave; ++j)
            v[j] = P4[off_c + __builtin_amdgcn_readlane(my_dl, cc * kDdDmPerWave + j) + lane];
#pragma unroll
        for (int j = 0; j < kDdDmPerWave; ++j) {
            part[j][0] += v[j].x;
            part[j][1] += v[j].y;
            part[j][2] += v[j].z;
            part[j][3] += v[j].w;
        }
    }
}

// Wide layout, next chunk prefetched into registers (16-channel chunks, at
// most 2 * 256 staging groups per chunk).
__global__ __launch_bounds__(64 * kDdWaves) void dedisp_u8_wide_kernel(DedispArgs a)
{
    extern __shared__ __align__(16) uint32_t dd_smem[];
    uint4* P4 = (uint4*)dd_smem;                             // [16][4 * groups]
    const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
    const int64_t t0 = (int64_t)(blockIdx.x / (uint32_t)a.n_dm_tiles) * kDdOut;
    const int d0 = (int)(blockIdx.x % (uint32_t)a.n_dm_tiles) * kDdDms;
    const int G = a.groups, E4 = 4 * a.groups;
    const double dm0 = a.dm[d0];
    const double dmj = a.dm[min(d0 + wv * kDdDmPerWave + (lane & 3), a.n_dm - 1)];
    // every byte this group stages lies inside the rows (the last tiles take the checked loads)
    const bool interior = t0 + a.max_delay + 4 * G + 64 * 8 <= a.n_samp;

    uint32_t D[kWideRounds][8];
    auto fetch = [&](int c0) {
#pragma unroll
        for (int r = 0; r < kWideRounds; ++r) {
            const int item = min(tid + 64 * kDdWaves * r, kDdMaxChunk * G - 1);
            const int cc = item / G, m = item - cc * G;
            const int c = min(c0 + cc, a.n_chan - 1);
            const int64_t g = ((t0 + dd_delay(dm0, a.kc[c])) & ~(int64_t)3) + 4 * m;
            dd_load_group(a.fb + (int64_t)c * a.stride, g, a.n_samp, interior, D[r]);
        }
    };
    auto store = [&](int ncc) {
#pragma unroll
        for (int r = 0; r < kWideRounds; ++r) {
            const int item = tid + 64 * kDdWaves * r;
            const int cc = item / G, m = item - cc * G;
            if (cc < ncc) dd_pack_wide(D[r], item, P4 + cc * E4 + 4 * m);
        }
    };

    uint32_t part[kDdDmPerWave][4] = {};
    uint32_t tot[kDdDmPerWave][8] = {};
    int since = 0;
    fetch(0);
    store(min(kDdMaxChunk, a.n_chan));
    __syncthreads();
    for (int c0 = 0; c0 < a.n_chan; c0 += kDdMaxChunk) {
        const int ncc = min(kDdMaxChunk, a.n_chan - c0);
        const double kd = a.kc[min(c0 + (lane >> 2), a.n_chan - 1)];
        const double ko = a.kc[min(c0 + lane, a.n_chan - 1)];
        const int32_t my_dl = dd_delay(dmj, kd) - dd_delay(dm0, kd);
        const int32_t my_off = lane * E4 + (int)((t0 + dd_delay(dm0, ko)) & 3);
        const bool more = c0 + kDdMaxChunk < a.n_chan;
        if (more) fetch(c0 + kDdMaxChunk);
        dd_accumulate_wide(P4, ncc, my_off, my_dl, lane, part);
        since += ncc;
        if (since + kDdMaxChunk > kDdFlush || !more) {
            dd_flush(part, tot);
            since = 0;
        }
        if (more) {
            __syncthreads();
            store(min(kDdMaxChunk, a.n_chan - c0 - kDdMaxChunk));
            __syncthreads();
        }
    }
    dd_store(a, d0, wv, lane, t0, tot);
}

// ---------------------------------------------------------------------------
// Matrix form (fine DM grids: 4 consecutive trials differ by at most 4 samples, or 9: FAR)
// ---------------------------------------------------------------------------
//
// The sum over channels is a product with 0/1 matrices, which the matrix cores
// evaluate exactly in 8-bit integers.  One product covers 4 consecutive trials
// x 4 consecutive starts (its 16 rows), 16 columns of starts 16 apart, and 8
// channels x 16 sample shifts (its 128 inner elements):
//   row (trial i, phase j), column n:  y[4q+i][t + 16n + j]
//     += sum over c, r of A[(i,j)][(c,r)] * x[c][w_c + 16n + r],
//   A[(i,j)][(c,r)] = 1 iff r == j + t + D(4q+i, c) - w_c,
// with w_c = t + D(4q, c) rounded down to 4 bytes, so r <= 3 + 3 + 4.  A has one
// 1 in 16 elements, so it goes in as the structured-sparse operand
// (v_smfmac_i32_16x16x128_i8: 2 of every 4 elements, 2 index bits each), which
// doubles the channels per product.  The starts 4 further on are the same
// bytes with A moved by 4 (r <= 14), so 24 bytes of a lane serve the 16
// consecutive starts t + 16n ..: four products.
//   B (samples): lane (n = l%16, g = l/16) holds 16 bytes of channel g, then 16
//   of channel g + 4.  A: lane (row l%16, g = l/16) holds channels 2g and
//   2g + 1, 8 bytes each: byte 2(r/4) is 1, every index field of the channel
//   r%4.  Lane (n, g) ends with starts t + 16n .. of trial 4q + g.
// Samples enter as x - 128 (xor 0x80: signed bytes) and every output gets
// 128 * n_chan back; all sums are exact in 32 bits.
//
// A work-group owns 4*NW trials (a quad per wave) x 256*NS starts and walks the
// channels 8 at a time, the bytes of the next 8 in flight.  In LDS each channel
// has two copies, one dword apart, so that the reads, which start at any dword,
// are aligned 8-byte reads (off their natural alignment they take 64 cycles
// instead of 2.5); a channel sits an odd number of entries after the one
// before, so that the 16-lane groups of a read use different banks.
//
// FAR (4 consecutive trials up to 9 samples apart): r may reach 15, so A is
// never moved; every 4 starts take their own read, in the other copy.
//
// Measured (4,096 channels x 6,000 trials x 2^17 samples): 28.3 ms, 1.1e14 of the
// definition's additions per second, against 97.6 ms for the wide layout, whose
// LDS reads and vector adds cover 8 sums an instruction.  The products take
// about half of it (22.5 cycles each, 1.52e9 of them); the rest is the staging's
// vector work, which the products only partly hide (66 instructions a wave and 8
// channels), and the LDS (53% busy).  Against the steps on the way: dense
// products (4 channels) 33.4 ms; exact byte alignment through 8 copies, with 8
// shifts a channel, 34.1 (the copies' LDS writes); 512 starts x 128 trials 33.0
// dense (twice the matrix-A work a product).
constexpr int kMfCh = 8;                    // channels per product and per LDS buffer
constexpr int kMfSpan4 = 4, kMfSpan4Far = 9;   // most delay between trials 4q and 4q+3 (see FAR below)
constexpr int kMfSpan = 120;                // most delay between the first trials of a work-group's quads

typedef int i32x4 __attribute__((ext_vector_type(4)));
typedef int i32x8 __attribute__((ext_vector_type(8)));
typedef const __attribute__((address_space(3))) uint8_t LdsByte;
typedef const __attribute__((address_space(3))) uint32_t LdsWord;
typedef const volatile __attribute__((address_space(3))) u32x2 LdsPair;

// The 8-byte entries of a copy read when a work-group's trials differ by at most `span`, and the entries a copy has
// room for.
__host__ __device__ constexpr int mf_entries(int ns, int span, bool far)
{
    return ((3 + (far ? 4 : 0) + span) >> 3) + 32 * ns + 1;
}
__host__ __device__ constexpr int mf_copy(int ns) { return (mf_entries(ns, kMfSpan, true) + 15) & ~15; }
// LDS bytes: a channel's two copies; one buffer with its table (4 bytes per trial and channel, quads 144 bytes
// apart so that 16 of them use all banks).
__host__ __device__ constexpr int mf_chan_bytes(int ns) { return 2 * 8 * mf_copy(ns) + 24; }
__host__ __device__ constexpr int mf_buffer_bytes(int nw, int ns) { return kMfCh * mf_chan_bytes(ns) + nw * 144; }
constexpr int kMfRows = 4 * 256 * 4;        // a wave's sums on their way out: 256 starts of its 4 trials

// Three dwords of a row from byte g on (a multiple of 4).  Dwords past the last whole one of the row, which only
// reach starts past the last, repeat it; a row's last, partial dword is read byte by byte.
__device__ inline void mf_load3(const uint8_t* row, int64_t g, int64_t n_samp, uint32_t (&D)[3])
{
    const int64_t whole = n_samp & ~(int64_t)3;
#pragma unroll
    for (int k = 0; k < 3; ++k) D[k] = whole ? *(const uint32_t*)(row + min(g + 4 * k, whole - 4)) : 0u;
#pragma unroll
    for (int k = 0; k < 3; ++k)
        if (g + 4 * k == whole && whole < n_samp) D[k] = dd_load4(row, whole, n_samp);
}

template <int NW, int NS, bool FAR>
__global__ __launch_bounds__(64 * NW) __attribute__((amdgpu_waves_per_eu(4, 4))) void dedisp_mfma_kernel(DedispArgs a)
{
    extern __shared__ __align__(16) uint8_t mf_smem[];
    constexpr int NT = 4 * NW, TPC = 8 * NW;                // trials; threads staging one channel
    constexpr int RND = (mf_copy(NS) + TPC - 1) / TPC;      // staging items per thread
    constexpr int CB = 8 * mf_copy(NS), kTabAt = kMfCh * mf_chan_bytes(NS), kBuf = mf_buffer_bytes(NW, NS);
    constexpr uint32_t kOdd = 0x8000;                       // table: the quad's bytes start in the second copy
    const int tid = threadIdx.x, lane = tid & 63, wv = __builtin_amdgcn_readfirstlane(tid >> 6);
    const uint64_t wg = xcd_remap(blockIdx.x, gridDim.x);
    const int64_t t0 = (int64_t)(wg / (uint32_t)a.n_dm_tiles) * mf_starts(NS);   // a multiple of 4
    const int d0 = (int)(wg % (uint32_t)a.n_dm_tiles) * NT;
    const int E = a.entries;
    // thread (ch, i): entries of channel c0 + ch's copies and, i < NT, trial i's table entry there (the threads
    // without one stage the first entries, so that they also have the last, partial round)
    const int ch = tid / TPC, i0 = tid % TPC, e0 = (i0 + NT) % TPC;
    const int chan_at = ch * mf_chan_bytes(NS);
    const double dm0 = a.dm[d0], dmt = a.dm[min(d0 + i0, a.n_dm - 1)];
    const bool interior = t0 + a.max_delay + 8 * E + 16 <= a.n_samp;
    const int last = a.n_chan - 1;

    // the next chunk: its samples, its first trial's delay and this thread's trial's
    uint32_t D[RND][3];
    int32_t base = 0, dly = 0;
    double kc = a.kc[min(ch, last)];                        // loaded a chunk ahead
    auto fetch = [&](int c0) {
        const int c = min(c0 + ch, last);
        base = dd_delay(dm0, kc);
        if (i0 < NT) dly = dd_delay(dmt, kc);
        const uint8_t* row = a.fb + (int64_t)c * a.stride;
        const int64_t g0 = (t0 + base) & ~(int64_t)3;
#pragma unroll
        for (int r = 0; r < RND; ++r) {
            const int i = e0 + TPC * r;
            if (i >= E) break;
            const int64_t g = g0 + 8 * i;
            if (interior) {
                struct __attribute__((aligned(4))) U3 { uint32_t v[3]; };
                const U3 u = *(const U3*)(row + g);
#pragma unroll
                for (int k = 0; k < 3; ++k) D[r][k] = u.v[k];
            } else {
                mf_load3(row, g, a.n_samp, D[r]);
            }
        }
        kc = a.kc[min(c0 + kMfCh + ch, last)];
    };
    auto store = [&](uint8_t* buf, int c0) {
        if (c0 + kMfCh > a.n_chan) {                        // channels past the last add nothing
            const bool have = c0 + ch < a.n_chan;
#pragma unroll
            for (int r = 0; r < RND; ++r)
#pragma unroll
                for (int k = 0; k < 3; ++k) D[r][k] = have ? D[r][k] : 0x80808080u;
        }
#pragma unroll
        for (int r = 0; r < RND; ++r) {
            const int i = e0 + TPC * r;
            if (i >= E) break;
            const u32x2 v0 = {D[r][0] ^ 0x80808080u, D[r][1] ^ 0x80808080u};
            const u32x2 v1 = {v0.y, D[r][2] ^ 0x80808080u};
            *(u32x2*)(buf + chan_at + 8 * i) = v0;
            *(u32x2*)(buf + chan_at + CB + 8 * i) = v1;
        }
        if (i0 < NT) {
            // per trial: the offset of its quad's bytes, and 4 * (its first phase's shift) in the high half
            int32_t dq = __builtin_amdgcn_mov_dpp(dly, 0x00, 0xf, 0xf, true);      // quad_perm 0,0,0,0
            asm("" : "+v"(dq));                             // keep the move by itself
            const int p = (base & 3) + (dq - base);
            const uint32_t odd = (p >> 2) & 1;
            const uint32_t off = (uint32_t)(chan_at + (p & ~7)) + odd * (CB | kOdd);
            const uint32_t r4 = (uint32_t)(4 * ((p & 3) + (dly - dq)));
            *(uint32_t*)(buf + kTabAt + 144 * (i0 >> 2) + 16 * ch + 4 * (i0 & 3)) = off | (r4 << 16);
        }
    };

    i32x4 acc[4 * NS] = {};
    const int n = lane & 15, kb = lane >> 4;
    auto multiply = [&](const uint8_t* buf) {
        // table entries of this lane's trial (A's row) for channels g, g + 4 (B) and 2g, 2g + 1 (A)
        LdsByte* tab = (LdsByte*)buf + kTabAt + 144 * wv + 4 * (n >> 2);
        const uint32_t e0 = *(LdsWord*)(tab + 16 * kb), e1 = *(LdsWord*)(tab + 16 * kb + 64);
        LdsByte* b0 = (LdsByte*)buf + (e0 & 0x7fff) + 16 * n;
        LdsByte* b1 = (LdsByte*)buf + (e1 & 0x7fff) + 16 * n;
        const uint32_t s0 = (*(LdsWord*)(tab + 32 * kb) >> 16) + 4 * (n & 3);        // 4r
        const uint32_t s1 = (*(LdsWord*)(tab + 32 * kb + 16) >> 16) + 4 * (n & 3);
        // 1 in byte 2(r/4): bit 16(r/4) = (4r & 48); A moved by 4: 16 bits higher
        const uint64_t v0 = 1ull << (s0 & 48), v1 = 1ull << (s1 & 48);
        const uint64_t w0 = v0 << 16, w1 = v1 << 16;
        const i32x4 av = {(int)v0, (int)(v0 >> 32), (int)v1, (int)(v1 >> 32)};
        const i32x4 aw = {(int)w0, (int)(w0 >> 32), (int)w1, (int)(w1 >> 32)};
        const int ix = (int)((s0 >> 2 & 3) * 0x5555u + (s1 >> 2 & 3) * 0x55550000u);
        // FAR: operand m is starts 256 (m/4) + 4 (m%4) + 16n ..; else starts 256 (m/2) + 8 (m%2) + 16n .., for
        // two products.  It is read a step ahead, and the steps are kept apart (the scheduler would fold the
        // reads into one register set and wait for each).
        constexpr int kSteps = FAR ? 4 * NS : 2 * NS;
        LdsByte* c0 = b0;
        LdsByte* c1 = b1;
        if (FAR) {                                          // 4 bytes on: the other copy
            c0 += e0 & kOdd ? 8 - CB : CB;
            c1 += e1 & kOdd ? 8 - CB : CB;
        }
        i32x8 bv[2];
        auto read = [&](int m) {
            // volatile: single 8-byte reads straight into the operand (paired by the compiler they take three
            // times as long)
            const int at = FAR ? 256 * (m >> 2) + 8 * (m >> 1 & 1) : 256 * (m >> 1) + 8 * (m & 1);
            LdsByte* p = (FAR && (m & 1) ? c0 : b0) + at;
            LdsByte* q = (FAR && (m & 1) ? c1 : b1) + at;
            const u32x2 x0 = *(LdsPair*)p, x1 = *(LdsPair*)(p + 8);
            const u32x2 y0 = *(LdsPair*)q, y1 = *(LdsPair*)(q + 8);
            bv[m & 1] = i32x8{(int)x0.x, (int)x0.y, (int)x1.x, (int)x1.y, (int)y0.x, (int)y0.y, (int)y1.x, (int)y1.y};
        };
        read(0);
#pragma unroll
        for (int m = 0; m < kSteps; ++m) {
            if (m + 1 < kSteps) read(m + 1);
            if (FAR) {
                acc[m] = __builtin_amdgcn_smfmac_i32_16x16x128_i8(av, bv[m & 1], acc[m], ix, 0, 0);
            } else {
                acc[2 * m] = __builtin_amdgcn_smfmac_i32_16x16x128_i8(av, bv[m & 1], acc[2 * m], ix, 0, 0);
                acc[2 * m + 1] = __builtin_amdgcn_smfmac_i32_16x16x128_i8(aw, bv[m & 1], acc[2 * m + 1], ix, 0, 0);
            }
            __builtin_amdgcn_sched_barrier(0);
        }
    };

    fetch(0);
    store(mf_smem, 0);
    if (kMfCh < a.n_chan) fetch(kMfCh);
    __syncthreads();
    int cur = 0;
    for (int c0 = 0; c0 < a.n_chan; c0 += kMfCh) {
        const bool more = c0 + kMfCh < a.n_chan;
        if (more) {
            store(mf_smem + (cur ^ 1) * kBuf, c0 + kMfCh);
            if (c0 + 2 * kMfCh < a.n_chan) fetch(c0 + 2 * kMfCh);
        }
        multiply(mf_smem + cur * kBuf);
        __syncthreads();
        cur ^= 1;
    }

    // A lane holds 16 consecutive starts of its trial per 256; through LDS (kMfRows a wave, float4s swizzled so
    // that neither side conflicts) a store instruction covers 256 consecutive bytes of each of the 4 rows.  Stored
    // straight from the accumulators, 16 bytes of each of 64 lines an instruction, the sums of few channels were
    // bound by their stores (128 trials x 262,144 samples, 4 and 16 channels: 62 and 65 us; 30 and 31 like this).
    const int bias = 128 * a.n_chan;
    // the lane anew: kept from the loop, its parts would take the kernel past 120 VGPRs, and then nothing that runs
    // beside it finds a register (two served beams: 2% slower, with the other stream's copies waiting)
    const int me = __builtin_amdgcn_mbcnt_hi(~0u, __builtin_amdgcn_mbcnt_lo(~0u, 0)), en = me & 15, ek = me >> 4;
    const int d = d0 + 4 * wv + ek;
    const bool have = d < a.n_dm, whole = t0 + mf_starts(NS) <= a.n_out;
    float* orow = a.out + (int64_t)d * a.out_stride + t0 + 4 * en;
    float* tr = (float*)(mf_smem + kMfRows * wv) + 256 * ek;
    typedef f32x4 RowAny __attribute__((aligned(4)));
#pragma unroll
    for (int s = 0; s < NS; ++s) {
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const i32x4 v = acc[4 * s + q] + bias;
            *(f32x4*)(tr + 16 * en + 4 * ((q + (en >> 2)) & 3)) = __builtin_convertvector(v, f32x4);
        }
        wave_sync();
        f32x4 w[4];
#pragma unroll
        for (int m = 0; m < 4; ++m) w[m] = *(const f32x4*)(tr + 64 * m + (4 * en & 48) + 4 * ((en + m) & 3));
        wave_sync();
        if (have && whole) {
#pragma unroll
            for (int m = 0; m < 4; ++m) *(RowAny*)(orow + 256 * s + 64 * m) = w[m];
        } else if (have) {
#pragma unroll
            for (int m = 0; m < 4; ++m) {
                const int64_t left = a.n_out - (t0 + 256 * s + 64 * m + 4 * en);
                if (left >= 4) {
                    *(RowAny*)(orow + 256 * s + 64 * m) = w[m];
                } else {
#pragma unroll
                    for (int j = 0; j < 3; ++j)
                        if (j < left) orow[256 * s + 64 * m + j] = w[m][j];
                }
            }
        }
    }
}

}  // namespace
}  // namespace spd

using namespace spd;

struct spd_dedisp_plan {
    spd_band band;
    int32_t n_dm;
    std::vector<double> dm, kc;
    double* d_dm = nullptr;
    double* d_kc = nullptr;
    int32_t max_delay = 0, span = 0, entries = 0, chunk = 0, groups = 0;
    int32_t mf_span[3] = {-1, -1, -1};       // matrix form with 4, 8, 16 waves: the bound on its trials' delays, -1: none
    bool mf_far = false;
    int device = 0, cus = 256;
};

extern "C" {

}  // extern "C"

namespace {

// Validation shared by the plan and the host delay table; fills k_c.
spd_status dd_prepare(const spd_band* band, const double* dm, int32_t n_dm, std::vector<double>& kc,
                      int32_t* max_delay)
{
    if (!band || !dm) return fail(SPD_E_INVALID, "band and dm are required");
    const spd_band b = *band;
    if (b.n_chan < 1 || b.n_chan > SPD_MAX_CHANNELS) return fail(SPD_E_INVALID, "n_chan must lie in [1, %d]", SPD_MAX_CHANNELS);
    if (!(b.f_top_mhz > 0.0) || !(b.chan_bw_mhz > 0.0) || !(b.t_samp_s > 0.0) || !isfinite(b.f_top_mhz) ||
        !isfinite(b.chan_bw_mhz) || !isfinite(b.t_samp_s))
        return fail(SPD_E_INVALID, "f_top_mhz, chan_bw_mhz and t_samp_s must be finite and > 0");
    if (!(b.f_top_mhz - (double)(b.n_chan - 1) * b.chan_bw_mhz > 0.0))
        return fail(SPD_E_INVALID, "the lowest channel frequency must be > 0");
    if (n_dm < 1 || n_dm > SPD_MAX_DM_TRIALS) return fail(SPD_E_INVALID, "n_dm must lie in [1, %d]", SPD_MAX_DM_TRIALS);
    for (int32_t d = 0; d < n_dm; ++d) {
        if (!isfinite(dm[d]) || dm[d] < 0.0) return fail(SPD_E_INVALID, "dm[%d] must be finite and >= 0", d);
        if (d && dm[d] < dm[d - 1]) return fail(SPD_E_INVALID, "dm must be non-decreasing (dm[%d] < dm[%d])", d, d - 1);
    }
    kc.resize(b.n_chan);
    for (int32_t c = 0; c < b.n_chan; ++c) {
        const double f = b.f_top_mhz - (double)c * b.chan_bw_mhz, ft = b.f_top_mhz;
        kc[c] = kKdm * (1.0 / (f * f) - 1.0 / (ft * ft)) / b.t_samp_s;
    }
    // the delays grow with the trial and towards the last channel
    const double p = dm[n_dm - 1] * kc[b.n_chan - 1];
    if (!(p < (double)SPD_MAX_DELAY)) return fail(SPD_E_UNSUPPORTED, "largest delay exceeds %d samples", SPD_MAX_DELAY);
    *max_delay = dd_delay(dm[n_dm - 1], kc[b.n_chan - 1]);
    return SPD_OK;
}

// A bound on the delay difference, at any channel, between two trials of the same group of `n` (the first and
// last of each group differ by at most the floor of their FP64 difference plus one; the products' rounding is
// below 1e-6 samples for delays up to SPD_MAX_DELAY).
int64_t dd_span_bound(const std::vector<double>& dm, int n, double k_last)
{
    double most = 0.0;
    for (size_t d = 0; d < dm.size(); d += (size_t)n)
        most = std::max(most, (dm[std::min(d + (size_t)n, dm.size()) - 1] - dm[d]) * k_last);
    return (int64_t)floor(most + 1e-6) + 1;
}

}  // namespace

extern "C" {

spd_status spd_dedisp_delay_table(const spd_band* band, const double* dm, int32_t n_dm, int32_t* delays,
                                  int32_t* max_delay)
{
    clear_error();
    std::vector<double> kc;
    int32_t md = 0;
    spd_status st = dd_prepare(band, dm, n_dm, kc, &md);
    if (st) return st;
    if (max_delay) *max_delay = md;
    if (delays)
        for (int32_t d = 0; d < n_dm; ++d)
            for (int32_t c = 0; c < band->n_chan; ++c) delays[(int64_t)d * band->n_chan + c] = dd_delay(dm[d], kc[c]);
    return SPD_OK;
}

spd_status spd_dedisp_plan_create(const spd_band* band, const double* dm, int32_t n_dm, spd_dedisp_plan** plan)
{
    clear_error();
    if (!plan) return fail(SPD_E_INVALID, "plan is required");
    *plan = nullptr;
    std::vector<double> kc;
    int32_t md = 0;
    spd_status st = dd_prepare(band, dm, n_dm, kc, &md);
    if (st) return st;
    spd_dedisp_plan* P = new (std::nothrow) spd_dedisp_plan;
    if (!P) return fail(SPD_E_NOMEM, "host allocation");
    const spd_band b = *band;
    P->band = b;
    P->n_dm = n_dm;
    P->dm.assign(dm, dm + n_dm);
    P->kc = kc;
    P->max_delay = md;
    int32_t span = 0;
    for (int32_t d0 = 0; d0 < n_dm; d0 += kDdDms) {
        const int32_t d1 = d0 + kDdDms - 1 < n_dm - 1 ? d0 + kDdDms - 1 : n_dm - 1;
        for (int32_t c = 0; c < b.n_chan; ++c) {
            const int32_t s = dd_delay(P->dm[d1], P->kc[c]) - dd_delay(P->dm[d0], P->kc[c]);
            span = s > span ? s : span;
        }
    }
    P->span = span;
    // entries per channel: the largest index read is 3 + 63 + 384 + span
    P->entries = (451 + span + 3) & ~3;
    const size_t per_chan = (size_t)P->entries * 4 + kDdDms * 4 + 4;
    P->chunk = 0;
    for (int cc = kDdMaxChunk; cc >= 1; cc >>= 1)
        if ((size_t)cc * per_chan <= kDdLdsMax) { P->chunk = cc; break; }
    // wide layout: the largest entry read is 3 + 63 + span
    P->groups = (67 + span + 3) / 4;
    // matrix form: trials 4q .. 4q+3 near enough, and per work-group size the span that its LDS copies hold
    const int64_t span4 = dd_span_bound(P->dm, 4, kc[b.n_chan - 1]);
    P->mf_far = span4 > kMfSpan4;
    for (int k = 0; k < 3; ++k) {
        const int64_t sp = dd_span_bound(P->dm, 16 << k, kc[b.n_chan - 1]);
        P->mf_span[k] = span4 <= kMfSpan4Far && sp <= kMfSpan ? (int32_t)sp : -1;
    }
    if (!P->chunk) {
        delete P;
        return fail(SPD_E_UNSUPPORTED, "trials 16 apart differ by %d samples of delay; at most about %d fit the LDS",
                    span, (int)(kDdLdsMax / 4) - 460);
    }
    hipError_t e = hipGetDevice(&P->device);
    if (e == hipSuccess) e = hipDeviceGetAttribute(&P->cus, hipDeviceAttributeMultiprocessorCount, P->device);
    if (e == hipSuccess) e = hipMalloc((void**)&P->d_dm, sizeof(double) * n_dm);
    if (e == hipSuccess) e = hipMalloc((void**)&P->d_kc, sizeof(double) * b.n_chan);
    if (e == hipSuccess) e = hipMemcpy(P->d_dm, P->dm.data(), sizeof(double) * n_dm, hipMemcpyHostToDevice);
    if (e == hipSuccess) e = hipMemcpy(P->d_kc, P->kc.data(), sizeof(double) * b.n_chan, hipMemcpyHostToDevice);
    if (e != hipSuccess) {
        if (P->d_dm) (void)hipFree(P->d_dm);
        if (P->d_kc) (void)hipFree(P->d_kc);
        delete P;
        return device_status(e, "de-dispersion plan tables");
    }
    *plan = P;
    return SPD_OK;
}

}  // extern "C"

namespace {

template <int NW, int NS>
hipError_t launch_mfma_nw(const DedispArgs& a, bool far, uint32_t grid, hipStream_t s)
{
    const dim3 g(grid), b(64 * NW);
    const size_t lds = std::max(2 * mf_buffer_bytes(NW, NS), NW * kMfRows);
    if (far) hipLaunchKernelGGL((dedisp_mfma_kernel<NW, NS, true>), g, b, lds, s, a);
    else hipLaunchKernelGGL((dedisp_mfma_kernel<NW, NS, false>), g, b, lds, s, a);
    return hipGetLastError();
}

MfShape mf_pick(const spd_dedisp_plan* plan, int64_t n_out)
{
    const bool fits[3] = {plan->mf_span[0] >= 0, plan->mf_span[1] >= 0, plan->mf_span[2] >= 0};
    MfShape f = mf_shape(plan->band.n_chan, plan->n_dm, n_out, fits, plan->cus);
    const int64_t nt = f.k >= 0 ? 16 << f.k : 16;
    const int64_t groups = ((plan->n_dm + nt - 1) / nt) * ((n_out + mf_starts(f.ns) - 1) / mf_starts(f.ns));
    if (f.k >= 0 && (uint64_t)groups * (uint64_t)(256 << f.k) > kMaxGridItems) f.k = -1;
    return f;
}

hipError_t launch_mfma(const spd_dedisp_plan* plan, DedispArgs a, MfShape f, hipStream_t s)
{
    const int nt = 16 << f.k;
    a.n_dm_tiles = (a.n_dm + nt - 1) / nt;
    a.entries = mf_entries(f.ns, plan->mf_span[f.k], plan->mf_far);
    const uint32_t grid = (uint32_t)(a.n_dm_tiles * ((a.n_out + mf_starts(f.ns) - 1) / mf_starts(f.ns)));
    if (f.k == 2) return launch_mfma_nw<16, 4>(a, plan->mf_far, grid, s);
    if (f.k == 0) return launch_mfma_nw<4, 2>(a, plan->mf_far, grid, s);
    return f.ns == 4 ? launch_mfma_nw<8, 4>(a, plan->mf_far, grid, s) : launch_mfma_nw<8, 2>(a, plan->mf_far, grid, s);
}

}  // namespace

namespace spd {

void dedisp_plan_shape(const spd_dedisp_plan* plan, int32_t* n_chan, int32_t* n_dm, int32_t* max_delay, int* device)
{
    *n_chan = plan->band.n_chan;
    *n_dm = plan->n_dm;
    *max_delay = plan->max_delay;
    *device = plan->device;
}

}  // namespace spd

extern "C" {

void spd_dedisp_plan_destroy(spd_dedisp_plan* plan)
{
    if (!plan) return;
    if (plan->d_dm) (void)hipFree(plan->d_dm);
    if (plan->d_kc) (void)hipFree(plan->d_kc);
    delete plan;
}

spd_status spd_dedisp_describe(const spd_dedisp_plan* plan, int32_t* max_delay, int32_t* span16)
{
    clear_error();
    if (!plan) return fail(SPD_E_INVALID, "plan is required");
    if (max_delay) *max_delay = plan->max_delay;
    if (span16) *span16 = plan->span;
    return SPD_OK;
}

spd_status spd_dedisp_delays(const spd_dedisp_plan* plan, int32_t* delays)
{
    clear_error();
    if (!plan || !delays) return fail(SPD_E_INVALID, "plan and delays are required");
    const int32_t C = plan->band.n_chan;
    for (int32_t d = 0; d < plan->n_dm; ++d)
        for (int32_t c = 0; c < C; ++c) delays[(int64_t)d * C + c] = dd_delay(plan->dm[d], plan->kc[c]);
    return SPD_OK;
}

spd_status spd_dedisperse(const spd_dedisp_plan* plan, const spd_plane* fb, float* out, int64_t out_stride,
                          void* stream)
{
    clear_error();
    if (!plan || !fb || !out) return fail(SPD_E_INVALID, "plan, fb and out are required");
    if (!fb->data) return fail(SPD_E_INVALID, "fb->data is NULL");
    if (fb->dtype != SPD_U8) return fail(SPD_E_UNSUPPORTED, "de-dispersion takes 8-bit filterbanks (SPD_U8)");
    if (fb->row_scale || fb->row_zero) return fail(SPD_E_INVALID, "de-dispersion sums raw counts: no scale or zero");
    if (fb->n_rows != plan->band.n_chan) return fail(SPD_E_INVALID, "fb has %lld rows, the plan %d channels",
                                                     (long long)fb->n_rows, plan->band.n_chan);
    if (fb->row_stride < fb->n_cols || fb->row_stride % 4 != 0 || ((uintptr_t)fb->data & 3))
        return fail(SPD_E_INVALID, "fb rows must be 4-byte aligned: data and row_stride (>= n_cols) multiples of 4");
    const int64_t n_out = fb->n_cols - plan->max_delay;
    if (n_out < 1) return fail(SPD_E_INVALID, "n_cols %lld must exceed the largest delay %d", (long long)fb->n_cols,
                               plan->max_delay);
    if (out_stride < n_out) return fail(SPD_E_INVALID, "out_stride < n_out (%lld)", (long long)n_out);
    int dev = 0;
    hipError_t ge = hipGetDevice(&dev);
    if (ge != hipSuccess) return device_status(ge, "hipGetDevice");
    if (dev != plan->device) return fail(SPD_E_INVALID, "the plan was made on device %d, not %d", plan->device, dev);
    const int64_t n_dm_tiles = (plan->n_dm + kDdDms - 1) / kDdDms;
    const int64_t n_t_tiles = (n_out + kDdOut - 1) / kDdOut;
    if ((uint64_t)(n_dm_tiles * n_t_tiles) * 64 * kDdWaves > kMaxGridItems)
        return fail(SPD_E_UNSUPPORTED, "output too large for one launch");
    DedispArgs a;
    memset(&a, 0, sizeof a);
    a.fb = (const uint8_t*)fb->data;
    a.stride = fb->row_stride;
    a.n_samp = fb->n_cols;
    a.dm = plan->d_dm;
    a.kc = plan->d_kc;
    a.out = out;
    a.out_stride = out_stride;
    a.n_out = n_out;
    a.n_chan = plan->band.n_chan;
    a.n_dm = plan->n_dm;
    a.n_dm_tiles = (int32_t)n_dm_tiles;
    a.entries = plan->entries;
    a.chunk = plan->chunk;
    a.groups = plan->groups;
    a.max_delay = plan->max_delay;
    const dim3 grid((uint32_t)(n_dm_tiles * n_t_tiles));
    // SPD_DEDISP_FORM=generic selects the chunk-by-chunk kernel for any plan, "wide" the wide layout wherever it fits
    // (all kernels give identical sums)
    const char* form = getenv("SPD_DEDISP_FORM");
    const bool generic = form && strcmp(form, "generic") == 0, wide = form && strcmp(form, "wide") == 0;
    if (!generic && !wide) {
        const MfShape f = mf_pick(plan, n_out);
        if (f.k >= 0) return device_status(launch_mfma(plan, a, f, (hipStream_t)stream), "de-dispersion launch");
    }
    const size_t wide_lds = (size_t)kDdMaxChunk * plan->groups * 64;
    if (!generic && kDdMaxChunk * plan->groups <= 64 * kDdWaves * kWideRounds && wide_lds <= kDdLdsMax)
        hipLaunchKernelGGL(dedisp_u8_wide_kernel, grid, dim3(64 * kDdWaves), wide_lds, (hipStream_t)stream, a);
    else
        hipLaunchKernelGGL(dedisp_u8_kernel, grid, dim3(64 * kDdWaves),
                           (size_t)plan->chunk * ((size_t)plan->entries * 4 + kDdDms * 4 + 4), (hipStream_t)stream, a);
    return device_status(hipGetLastError(), "de-dispersion launch");
}

}  // extern "C"

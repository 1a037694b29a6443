// spd_sched.h -- host rules of the launches: whether a batched-run schedule
// read from the tuning cache can run a given plan, and how the streaming form
// cuts its rows.  Plain C++ (no HIP types), so the rules are also compiled and
// checked on their own on the host.
#pragma once

#include <stdint.h>

namespace spd {

constexpr uint64_t kMaxGridItems = 0xffffffffull;   // work-items per launch (1-D grid)

// Streaming form of the short lists 1..n (n <= 16): a wave walks a run of a
// few steps of kStreamStep consecutive starts of one row.
constexpr int kStreamStep = 512;

struct StreamShape {
    int steps;              // steps per run (2 or more)
    int waves;              // runs, and waves, per work-group
    int64_t tiles_per_row;  // work-groups per row
    bool aligned;           // the steps lie on 64-byte boundaries of the outputs, so that the first of a row begins
                            // up to 15 starts before it
};

// Long runs amortise a wave's start (coefficients, first loads), short ones give small planes enough waves:
// 8 steps against 4 and 2 take 1582, 1644 and 1756 us on 2,048 x 524,281 U8 (262,000 waves), 38.6,
// 38.3 and 36.0 on 256 x 65,536 F32, 19.1, 14.7 and 13.1 on 64 x 65,536 F32 (30.2 with 16).  Without outputs
// (candidates only) a step is shorter, and 16 steps are better than 8 where they still give 32,768 waves
// (2,048 x 262,144, 1..8, F16 355 and 363 us, 1..16, U8 562 and 576; with U8 outputs, 1..8, 612 and 602).
//
// Rows of fewer than 4 steps are walked from their first start: on the boundaries of the outputs they may take a
// step more (F32, list 1..1, 39,603 x 505: 38.7 us, 29.9 from the first start; 6,664 x 3,001 29.7 and 31.8; U8
// 29.5 and 24.0 on 13,324 x 1,501, 22.6 and 25.0 on 4,900 x 4,081).
//
// A work-group has no more waves than a row has runs: with 4 for rows of one run, three of them ended at once and
// the planes of many short rows were bound by starting them (200,000 x 107 F32, 1..8: 294 us, 157 with one).
inline StreamShape stream_shape(int64_t n_rows, int64_t nout, bool outputs)
{
    StreamShape f;
    f.aligned = nout >= 4 * kStreamStep;
    const int64_t steps = (nout + (f.aligned ? 15 : 0) + kStreamStep - 1) / kStreamStep;   // of any row
    auto runs = [&](int64_t per) { return (steps + per - 1) / per; };
    f.steps = !outputs && n_rows * runs(16) >= 32768 ? 16
              : n_rows * runs(8) >= 32768            ? 8
              : n_rows * runs(4) >= 16384            ? 4
                                                     : 2;
    for (;; f.steps *= 2) {
        f.waves = runs(f.steps) < 4 ? (int)runs(f.steps) : 4;
        f.tiles_per_row = (runs(f.steps) + f.waves - 1) / f.waves;
        // one run per row always fits: the caller's rows are at most kMaxGridItems / 256
        if ((uint64_t)n_rows * (uint64_t)f.tiles_per_row * 64u * (uint64_t)f.waves <= kMaxGridItems || runs(f.steps) == 1)
            break;
    }
    return f;
}

// A cached schedule (outputs per lane X, register-window form `win`,
// persistent work-groups per CU, tiles per queue grab) is usable for a plan
// whose layout for that schedule has `tiles` tiles of `waves` waves when its
// fields are in range, the register-window form exists for the plan
// (has_win) and is asked for as a grid launch, and a grid launch
// (wgs_per_cu == 0, one work-group per tile) holds every tile in one launch of
// at most max_items work-items.  The cache key does not include the beam
// shapes, so the last test is what keeps a grid schedule tuned on small beams
// from being used for beams too large for one launch.
inline bool schedule_usable(int X, int win, int wgs_per_cu, int grab, bool has_win, int64_t tiles, int waves,
                            uint64_t max_items)
{
    if (!(X == 4 || X == 8) || wgs_per_cu < 0 || grab < 1 || waves < 1 || tiles < 0) return false;
    if (win && !(has_win && X == 8 && wgs_per_cu == 0)) return false;
    if (wgs_per_cu == 0 && (uint64_t)tiles * 64u * (uint64_t)waves > max_items) return false;
    return true;
}

// The streaming form loads samples past the caches (nontemporal) where the plane is larger than the 256 MB
// memory-side cache; a smaller one may still be there from the statistics pass or the call before.  F32 with both
// outputs, past the caches and not: 128 MB, 1..1 65 and 46 us; 256 MB, 1..16 120 and 110; 320 MB 137 and 139; 2 GB
// 871 and 891.  F16, candidates only, 1..8: 192 MB 76 and 69, 400 MB 146 and 149.
inline bool stream_once(int64_t plane_bytes) { return plane_bytes > (int64_t)256 << 20; }

// Lists of groups of 8 unit-count widths that step by 1 or 2 (the last group may hold fewer) can take the
// register-window form.  On one plane the strided form keeps a list of up to 16 widths whose last group is short:
// it has variants that hold all its SNRs in registers and evaluate no more than 8 or 16 widths (F32 1,024 x 131,072,
// strided and window: 2,4 315 and 446 us; 2,4..20 390 and 495; 1..8,10,12,14 391 and 539; 64 x 65,536, 2,4,6 15.0
// and 19.8; F16, candidates only, 2,4 213 and 350), and they return NaN where every SNR is NaN, as the window form
// does not.  From 17 widths on, and in batched runs, whose strided form has no such variants, the window form is the
// faster one (1..17 547 and 415, 1..16,18,20 655 and 589; batched 2,4,6 on 256 x 65,536 117 and 69).
inline bool window_pays(int n_widths, bool batched) { return batched || n_widths > 16 || n_widths % 8 == 0; }

// The matrix form of the de-dispersion: work-groups of 4 << k waves, 16 << k trials x 256 * ns starts each; k = -1:
// not this form.  fits[k]: the list's delays allow k.  Sizes are channels x trials x starts.
//
// 64 trials x 1,024 starts amortise the staging best (4,096 x 6,000 x 2^17: 28.3-29.6 ms against 39.4 with 32 x 512
// starts) while they give three quarters of the CUs a work-group (256 x 200 x 50,001, 196 groups: 57 against 68 us);
// below that smaller groups keep more CUs busy (128 x 100 x 10,000: 19 against 29 us; 512 x 64 x 20,000: 68 against
// 97).  Not for 32 trials or fewer, which leave half of their waves without a trial (256 x 32 x 2^20: 152 us with
// 32 x 1,024 starts, 216 with 64), nor for fewer than 16 channels, whose time goes into the stores, during which a
// CU's only group of 16 waves has nothing beside it (4 x 128 x 2^18: 30.3 us, 25.6 with 32 x 1,024, 26.4 in the wide
// layout; 16 x 64 x 2^20: 61, 67 and 80).  Up to 16 trials take groups of 16 where those are 4 a CU or more
// (256 x 16 x 2^20: 117 us, 138 with 32; 2^18 starts, 2 a CU: 51 and 50).  One channel has nothing to sum
// (1 x 64 x 2^20: 44 us, 41 in the wide layout).  The 64-trial groups' span limit also sends coarse lists to the
// smaller ones (512 x 500 x 20,000, 2 samples a trial: 145 us with 32 x 512 starts, 263 in the wide layout).
struct MfShape { int k, ns; };
constexpr int mf_starts(int ns) { return 256 * ns; }

inline MfShape mf_shape(int n_chan, int n_dm, int64_t n_out, const bool (&fits)[3], int cus)
{
    auto groups = [&](int k, int ns) {
        return ((n_dm + (16 << k) - 1) / (16 << k)) * ((n_out + mf_starts(ns) - 1) / mf_starts(ns));
    };
    if (n_chan < 2) return {-1, 2};
    if (fits[2] && n_chan >= 16 && n_dm > 32 && 4 * groups(2, 4) >= 3 * cus) return {2, 4};
    if (fits[0] && n_dm <= 16 && groups(0, 2) >= 4 * cus) return {0, 2};
    if (fits[1]) return {1, 2 * groups(1, 4) >= 3 * cus ? 4 : 2};
    return {fits[0] ? 0 : -1, 2};
}

}  // namespace spd

// Which kernel takes a problem, and in what launch: host-only rules on sizes and formats, shared by the launches
// (atb_skinny.hip, atb_gemm.hip) and by what a plan reports (atb_api.cpp).
#pragma once

#include "atb_internal.h"

namespace atb {

// CUs that the rules are reckoned with where there is no device to ask
constexpr int kDefaultCUs = 256;

// HIP takes fewer than 2^32 threads in a launch: what fits, in workgroups of 256 threads.  A route that needs more has workgroups == 0.
constexpr int64_t kMaxWorkgroups256 = ((int64_t)1 << 24) - 1;

// Quantiser: steps of two rows that a wave takes, and workgroups of 2 steps rows x 512 k (four waves side by side along k).
struct QuantizeRoute {
    int steps;
    int64_t workgroups;
};

// Measured, cold inputs, us, steps = 2 / 4 / 8:
//   512 x 4096 4.1 / 5.0 / 7.4   4096 x 1024 5.2 / 5.8 / 7.7   8192 x 8192 54.0 / 53.4 / 57.9: a wave holds few loads, so waves are
//   what fills the chip; more rows per wave only save workgroups.
//   Up to 256 columns, where half of a workgroup's waves or more have nothing to do, saving workgroups is what counts once there are
//   many: 10^6 x 8 186 / 157 / 149, 200000 x 256 58.9 / 54.5 / 52.5, 65536 x 200 21.1 / 19.4 / 19.0 (32768 x 64 8.2 / 7.4 / 8.0;
//   150000 x 384 53.8 / 51.1 / 51.3).
inline QuantizeRoute quantize_route(int64_t M, int64_t K)
{
    const int64_t panels = (K + kPanelK - 1) / kPanelK, kblocks = (panels + 7) / 8;
    const int64_t small = ((M + 3) / 4) * kblocks;
    int steps = small <= 12 * kDefaultCUs ? 2 : (K <= 256 && small >= 16384) ? 8 : 4;
    if (((M + 7) / 8) * kblocks > kMaxWorkgroups256) steps = 8;          // up to 2^28 rows of at most 512 columns in one launch
    const int64_t n = ((M + 2 * steps - 1) / (2 * steps)) * kblocks;
    return {steps, n <= kMaxWorkgroups256 ? n : 0};
}

// Decoder.  rows == 0: a lane takes a block of 8 in row order (decode_lanes); else a wave takes 8 rows of a panel, `rows` of them
// one after the other (decode_panels), with `past_caches` written non-temporally. 
struct DecodeRoute {
    int rows;
    bool past_caches;
    int64_t workgroups;
};

// Measured, inputs in turns, us, lanes / panels:
//   narrow outputs leave lanes and waves of the panel form without work: 10^6 x 8 14.3 / 24.6, 10^6 x 24 22.1 / 36.1, 300000 x 200
//   40.1 / 43.4; from 512 columns on it is the faster one (4000 x 4104 12.4 / 9.6, 8192 x 3000 19.2 / 14.0),
//   but for outputs of a few MiB, where it has too few loads in flight: 1000 x 1000 2.3 / 2.5, 3891 x 792 3.3 / 3.9; 1124 x 3408
//   4.5 / 3.9, 1024 x 4096 4.5 / 3.7.
//   Above 64 MiB one group of rows per wave instead of two: 4571 x 8040 33.6 -> 28.7, 8192^2 45.2 -> 42.6 (below, 4000 x 4104 9.6 ->
//   10.1).  past_caches: see decode_panels.
inline DecodeRoute decode_route(int64_t M, int64_t K, bool out_on_lines)
{
    const int64_t panels = (K + kPanelK - 1) / kPanelK, bytes = 2 * M * K;
    const bool past_caches = K % kPanelK == 0 && out_on_lines && bytes >= ((int64_t)96 << 20);
    if (past_caches || (K >= 512 && M * K >= ((int64_t)7 << 19))) {
        const int rows = (past_caches || bytes <= ((int64_t)64 << 20)) ? 2 : 1;
        const int64_t n = ((M + 8 * rows - 1) / (8 * rows)) * ((panels + 3) / 4);
        if (n <= kMaxWorkgroups256) return {rows, past_caches, n};       // 2^28 rows of a few panels are more than that
    }
    const int64_t n = (M * (K / 8) + 255) / 256;
    return {0, false, n <= kMaxWorkgroups256 ? n : 0};
}

}  // namespace atb

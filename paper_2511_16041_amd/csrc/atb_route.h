// Which kernel takes a problem, and in what launch: host-only rules on sizes and formats, shared by the launches
// (atb_skinny.hip, atb_gemm.hip) and by what a plan reports (atb_api.cpp).
#pragma once

#include "atb_internal.h"

namespace atb {

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
    const bool past_caches = K % kPanelK == 0 && out_on_lines && bytes > ((int64_t)32 << 20);
    if (past_caches || (K >= 512 && M * K >= ((int64_t)7 << 19))) {
        const int rows = (past_caches || bytes <= ((int64_t)64 << 20)) ? 2 : 1;
        return {rows, past_caches, ((M + 8 * rows - 1) / (8 * rows)) * ((panels + 3) / 4)};
    }
    return {0, false, (M * (K / 8) + 255) / 256};
}

}  // namespace atb

// Which kernel takes a problem, and in what launch: host-only rules on sizes and formats, shared by the launches and
// by what a plan reports.
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

// Reductions up to here stay with the tile pipeline.  Not a line of speed (M 16, N 8192, K 1088: 8.3 us there, 5.7 streamed): up to here
// every plan of a problem gives the same bits, whatever the instance, B or B^T, and whatever M is for a row of C.
constexpr int kStreamMinK = 1024;

// Bytes of LDS that the 64-row forms with B in LDS (atb_rows.hip) ask for at the launch: two panels of B for each wave but the first, whose
// panels lie in the static part, and a panel of A for each; or the partial C tiles of all waves but the first.
constexpr int rows_dynamic_lds(int mb, int nb, int waves)
{
    const int panels = (waves - 1) * 2 * 64 * 32 * nb + waves * (mb * 1024 + (mb + 1) / 2 * 256), partial = (waves - 1) * 16 * mb * (16 * nb + 4) * 4;
    return panels > partial ? panels : partial;
}

// The streaming kernel's variant for a problem: a workgroup takes a tile of 16 mb rows x 16 nb columns with `waves` waves,
// each with `depth` panels of K in flight, in LDS (atb_rows.hip) or in registers.  mb == 0: the problem stays with the tile pipeline.
struct StreamRoute {
    int mb, nb, waves, depth;
    bool in_lds = false;
    bool streams() const { return mb > 0; }
    int threads() const { return 64 * waves; }
    int lds_bytes() const { return waves * 16 * (16 * nb + 4) * 4; }         // static: the partial C tiles
    int dynamic_lds() const { return in_lds ? rows_dynamic_lds(mb, nb, waves) : 0; }
};

inline int64_t tile_count(const GemmParams &p, int rows, int cols)
{
    const int64_t columns = p.n_panels > 0 ? (int64_t)p.n_panels * kPanelK : p.N;      // C in BFP16: the zero tail of its last panel as well
    return (int64_t)((p.M + rows - 1) / rows) * ((columns + cols - 1) / cols);
}

inline int64_t stream_workgroups(const GemmParams &p, const StreamRoute &r) { return (tile_count(p, 16 * r.mb, 16 * r.nb) + 7) / 8 * 8; }

// M <= 64: 16 nb columns per workgroup, the narrowest of 32, 64 and 128 that needs no more workgroups than there are CUs.
// Measured (us, M = 16, bf16 B): N = 14336, K = 4096: 35.4 / 24.4 / 31.9 with 32 / 64 / 128 columns; N = 28672: 59 / 54 / 44.
inline int stream_column_blocks(int N, int cus) { return N <= 32 * cus ? 2 : N <= 64 * cus ? 4 : 8; }

// Panels of K in flight per wave with B in BFP16, 32 or 64 columns and eight waves.  With one panel a wave either waits or decodes; two
// are taken where they come out even (a wave's last round may otherwise be one of zeros; a branch around it costs the overlap).
// Measured, one / two, us: 32 x 14336 x 4096 16.4 / 15.0, 64 x 14336 x 4096 21.2 / 19.8, 128 x 4096 x 4096 16.3 / 14.6, 256 x 2048 x 8192 27.5 /
// 23.9, 64 x 12288 x 2048 13.3 / 13.0; three rounds: 64 x 10000 x 1536 11.3 / 12.9, 65 x 3000 x 1088 7.4 / 8.0; 16 rows are level.
inline int stream_depth_bfp16(int k_panels, int mb) { return mb >= 2 && (k_panels + 7) / 8 % 2 == 0 ? 2 : 1; }

// With B^T in bf16, 64 columns and four waves: two from 33 rows on, whatever the number of rounds, since what a round of zeros costs here is
// little against what the second panel gives.  Two over one, M 33 .. 64, N 8200 .. 16384, five to 25 rounds: 0.89 - 1.01 from memory, the odd
// numbers 0.91 - 1.01; from the cache 0.88 - 1.00 at even and 0.90 - 1.02 at odd numbers (K 1280 and 1792 1.00 - 1.02, K 1088 and 1600 0.97 - 0.99).
// 64 x 14336 x 4096 31.5 / 29.4 us, 48 x 14336 x 4096 29.4 / 28.6; fewer rows lose up to 6 % at K = 2048.
inline int stream_depth_bf16_t(int mb) { return mb >= 3 ? 2 : 1; }

// With row-major bf16 B, 64 columns and four waves: two, through LDS, at 49 to 64 rows.  One panel through registers over that, N 8256 ..
// 16322: M 64 1.08 - 1.28 at K 1032, 1.03 - 1.29 at K 4096, 1.05 at K 8192; N = 16384 (rows 32 KiB apart) 1.07 at K 1032, 1.00 at 4096, 0.99 from 6144 on.  At 33 to 48 rows 1.0 - 1.25 up to N = 14336, but 0.93 - 0.96
// at 16128 and 16384.
inline int stream_depth_bf16(int mb) { return mb == 4 ? 2 : 1; }

// More than 64 rows: tiles of 64 x 32, 64 x 64, 64 x 128 or 128 x 64, the smallest that makes at most one per CU, and
// none where the tile pipeline is as good or better.  Measured in us, the pipeline / this kernel, or as the ratio of the two; "memory":
// 700 MB of operands in turns, so that B comes from memory as a model's weights do; "cache": three sets in turns, which the 256 MiB
// memory-side cache holds:
//   B bf16    64 x 64: M 128, 8192, 8192 54.4 / 47.0, M 256, 4096, 4096 22.3 / 19.5; eight shapes of 130 to 256 tiles, K 1032 to 4096: 1.0 - 1.3
//             x memory, 0.96 - 1.2 x cache (lowest at K 1536, where the pipeline has whole K-steps)
//             64 x 128: M 1024, 2048, 4096 38.2 / 26.7 memory, 26.2 / 21.7 cache, M 512, 4096, 14336 121 / 78; eight shapes, K 4096 to 14336: 1.35 - 1.6 x
//             memory, 1.15 - 1.55 x cache; below K 4096 see stream_route_lds
//             not 64 x 32 (M 256, 2048, 2048 9.9 / 10.4) nor odd N (M 512, 5001, 4096 61 / 70), nor 64 x 64 where the pipeline's 32 x 64
//             tiles fit one to a CU (rows just above a multiple of 64: M 193, 2304, M 129, 3000 and M 96, 5000, K 1032 .. 4096: 0.83 - 0.94 x
//             memory, 0.72 - 0.91 x cache)
//   B^T bf16  K 1032 / 2048 / 4096 / 8192, the pipeline on its 64 x 64 tiles where these are few (bt_small_tiles): 64 x 32 tiles (M 65 .. 200, N 2000 .. 4096)
//             1.6 / 1.9 / 2.3 / 2.4 x memory, 1.3 / 1.4 / 1.5 / 1.6 x cache; 64 x 64 (256 x 4096, 100 x 8000, 300 x 3000) 1.25 / 1.4 / 1.65 / 1.75
//             and 1.05 - 1.1 / 0.97 - 1.0 / 1.06 - 1.1 / 1.05 - 1.8; 128 x 64 (512 x 4096, 1024 x 2048, 129 x 6000) 0.90 - 0.95 / 1.02 - 1.04 / 1.14 - 1.17 /
//             1.2 - 1.3 and 0.79 - 0.82 / 0.85 - 0.89 / 0.91 - 0.96 / 0.97 - 1.2.  (The last line dates from when the pipeline had no tile below 128 x 256 for
//             B^T, 57 / 36 us at 512 x 4096 x 4096; with B from the caches the small tiles have overtaken it.)
//   B^T BFP16 M 128, 4096, 4096: 19.9 / 17.5 (64 x 32)   M 128, 8192, 8192: 47.9 / 38.4 (64 x 64); where 32 x 64 tiles fit one to a CU, K 1032
//             and 1152 0.98 - 1.16 x, from 1296 on 0.88 - 0.97 x memory
inline StreamRoute stream_route_many_rows(const GemmParams &p, int b_format, int cus)
{
    const bool small_tiles = tile_count(p, 32, 64) <= cus;            // the pipeline's 32 x 64 tiles: one per CU or fewer
    if (b_format == ATB_FMT_BF16) {
        if (p.N % 2 != 0 || tile_count(p, 64, 32) <= cus) return {};
        if (tile_count(p, 64, 64) <= cus) return small_tiles ? StreamRoute{} : StreamRoute{4, 4, 8, 1};
        if (tile_count(p, 64, 128) <= cus && p.K >= 4096) return {4, 8, 4, 2, true};
        return {};
    }
    const int depth = b_format == ATB_FMT_BFP16 ? stream_depth_bfp16(p.k_panels, 4) : 1;
    if (tile_count(p, 64, 32) <= cus) return {4, 2, 8, depth};
    if (tile_count(p, 64, 64) <= cus) return b_format == ATB_FMT_BFP16 && small_tiles && p.K > 1152 ? StreamRoute{} : StreamRoute{4, 4, 8, depth};
    if (b_format == ATB_FMT_BF16_T && tile_count(p, 128, 64) <= cus) return {8, 4, 4, 1};
    return {};
}

// At most 64 rows: whether the streaming kernel is at least as fast as the pipeline.  The lines lie where both sides were measured, over
// M 1 .. 64, N 32 .. 151936, K 1032 .. 14336; figures are the pipeline's time over this kernel's, with the operands of three problems in
// turns (B comes from memory where it is larger than 90 MB) and, where that differs, of 700 MB of them ("memory") or of one ("cache").
// What they come down to: one tile per CU is where this kernel is at its best; with fewer tiles than CUs, or a second round of them that
// is nearly empty, CUs idle, and the pipeline, whose requests go straight to LDS, gets more out of the others.
inline bool stream_few_rows(const GemmParams &p, int b_format, int cus)
{
    const int M = p.M, N = p.N, K = p.K;
    if (b_format == ATB_FMT_BFP16) return N <= 64 * cus || M <= 48;        // 1.0 - 1.9; M 64, N 28672, K 8192 0.87: out of registers
    if (b_format == ATB_FMT_BF16_T) {
        // Up to N = 16384 1.13 - 4.2 from memory, 0.98 - 2.9 from the caches.  To 32768 M <= 16 1.0 - 1.3; M 33 .. 48 0.93 - 0.98 at K = 1032, 0.99 - 1.18
        // above (cache 0.83 - 1.17); M 64 0.87 - 0.93, 0.97 - 1.1 (cache 0.77 - 1.1).  Beyond, N 33000 .. 48000 0.70 - 0.99, 57344 and 128256 0.90 - 1.17, but
        // 1.01 - 1.29 for N 66000 .. 90000 and 151936, where 256 columns (the pipeline's tile) come to more rounds than 128
        if (N <= 128 * cus) return true;
        const int64_t rounds128 = ((N + 127) / 128 + cus - 1) / cus, rounds256 = ((N + 255) / 256 + cus - 1) / cus;
        return rounds128 < 2 * rounds256;
    }
    if (N % 2 != 0) {
        // 32 columns per workgroup whatever N is: 1.03 - 2.1 up to N = 24576.  Then the pipeline's 128-column tiles fill more than three
        // quarters of the CUs, until they need a second round: M > 32 0.78 - 1.0 (0.97 - 1.2 at K = 1032), M <= 32 1.01 - 1.4 up to
        // 30720, 0.91 - 1.02 from there at K >= 4096.  Beyond: M <= 48 0.98 - 1.5, M 49 .. 64 at K >= 4096 0.94 - 1.05.
        if (N <= 96 * cus) return true;
        if (N > 128 * cus) return M <= 48 || K < 4096;
        return M > 32 ? K < 1536 : N <= 120 * cus || K < 4096;
    }
    if (N <= 32 * cus) return M <= 48;                                     // 0.97 - 2.2; M 64, N = K = 8192 0.94: every workgroup decodes all of A
    if (N <= 64 * cus) {
        if (M > 32) return true;                                           // 1.0 - 1.3
        // 129 to 256 workgroups of 64 columns.  Rows of B that are not whole lines and one or two rows of A: the pipeline skips the
        // dead rows of its tile, 0.88 - 1.0 from K = 2560 (under 208 workgroups) or above 4096 on.
        const bool ragged = N % 64 != 0 && M <= 2;
        if (N < 36 * cus) return K < 2048;                                 // 0.97 - 1.25 below, 0.71 - 1.09 from 2048 on
        if (N < 52 * cus) return K < (ragged ? 2560 : 4096);               // 0.98 - 1.17 below (memory 0.94 - 1.08), 0.92 - 1.05 from 4096 on
        return !ragged || K <= 4096;                                       // 0.96 - 1.19
    }
    // 1.03 - 1.6; M 49 .. 64: K 1032 .. 2048 0.80 - 0.96, 4096 0.96 - 1.03 (cache 0.85 - 0.95), 8192 0.99 - 1.08
    if (N <= 128 * cus) return M <= 48 || K >= 8192;
    // more than one workgroup of 128 columns per CU: 0.76 - 1.0 (K 1032 .. 1240 1.0 - 1.3, 1536 0.92 - 1.03) until the second
    // round is half full, 0.97 - 1.4 then
    return M <= 48 && (K < 1536 || N >= 192 * cus);
}

// Where the streaming kernel takes over from the tile pipeline, and in what form.
// Waves: four where their requests already fill the CU's share (64 and 128 columns of bf16 B: 24.4 against 28.1 us with
// eight), eight or sixteen where more hands are needed to decode B.
// cus: CUs of the device (a partition of the chip has fewer than 256).
inline StreamRoute stream_route(const GemmParams &p, int b_format, int cus)
{
    if (p.K <= kStreamMinK) return {};
    if (p.M > 64) return stream_route_many_rows(p, b_format, cus);
    if (!stream_few_rows(p, b_format, cus)) return {};
    const int mb = (p.M + 15) / 16, nb = stream_column_blocks(p.N, cus);
    if (b_format == ATB_FMT_BFP16) return {mb, nb, nb == 2 ? 16 : 8, nb == 4 ? stream_depth_bfp16(p.k_panels, mb) : 1};
    if (b_format == ATB_FMT_BF16 && p.N % 2 != 0) return {mb, 2, 8, 1};
    const int depth = nb != 4 ? 1 : b_format == ATB_FMT_BF16_T ? stream_depth_bf16_t(mb) : stream_depth_bf16(mb);
    return {mb, nb, nb == 2 ? 8 : 4, depth, b_format == ATB_FMT_BF16 && depth == 2};
}

// What stream_route leaves to the pipeline and the 64 x 128 tiles with B through LDS (atb_rows.hip) still take: row-major bf16 B of even N that
// makes at most one such tile per CU and more 64 x 64 tiles than CUs, from K = 1536 on.  The pipeline's time over theirs, twelve shapes of 136
// to 250 tiles, K 1032 / 1280 / 1536 / 2048 / 3072: 0.95 - 1.04 / 0.97 - 1.08 / 1.0 - 1.11 / 1.05 - 1.18 / 1.12 - 1.26 (1024 x 2048 x 2048
// 14.8 / 13.5 us, 512 x 4096 x 3072 20.4 / 17.3).
inline StreamRoute stream_route_lds(const GemmParams &p, int b_format, int cus)
{
    const bool takes = b_format == ATB_FMT_BF16 && p.N % 2 == 0 && p.M > 64 && p.K >= 1536 && tile_count(p, 64, 128) <= cus && tile_count(p, 64, 64) > cus;
    return takes ? StreamRoute{4, 8, 4, 2, true} : StreamRoute{};
}

// Odd N, row-major bf16 B, on 128 x 128 tiles: whether the 128 x 256 tiles (128,128,64,256; the same bits) run in their place.  A request for rows at odd
// addresses takes a CU twice as long as an aligned one, the staging waves of the 128 x 128 tiles then wait for A behind B, and two of these tiles on a CU
// ask for B twice.  The wide tiles stage A and B with different waves and have a third B buffer.  What decides is how many tiles one CU gets through,
// a wide one counted as two: narrow N, of which the wide tiles multiply up to twice the padding, and last rounds that are nearly empty come out in it.  64,128,64,128
// over the wide tiles, 110 shapes from 350 to 2000 tiles of 128 x 128, by the wide tiles' count over the small ones', at K 1032 / 2056 / 4104:
//   1            0.99 - 1.10 (0.94 with 1/7 of padding) / 1.06 - 1.17 / 1.11 - 1.26 (1500 x 3001 x 2056 41.0 us / 33.6)
//   up to 8/7    0.89 - 0.98 / 0.97 - 1.06 / 1.02 - 1.12
//   up to 6/5    0.87 - 0.95 / 0.95 - 1.02 / 1.01 - 1.06
//   4/3          0.81 - 0.89 / 0.90 - 0.95 / 0.95 - 1.00;  2, N below 128: 0.62 - 0.70
// (from memory 0.02 less at the best and the same at the line).  Not where one 128 x 128 tile per CU is enough (64 wide tiles take twice as long).
inline bool odd_n_runs_wide(const GemmParams &p, int T_MC, int T_N, int cus)
{
    if (p.N % 2 == 0 || T_MC != 128 || T_N != 128 || p.K < 1024) return false;
    const int64_t per_cu = (tile_count(p, 128, 128) + cus - 1) / cus, wide = 2 * ((tile_count(p, 128, 256) + cus - 1) / cus);
    return per_cu > 1 && 100 * wide <= (p.K < 2048 ? 100 : p.K < 4096 ? 112 : 120) * per_cu;
}

// Odd N, row-major bf16 B, on the tiles that have a kernel with a third B buffer (64,64,128,128 and 128,128,64,128): whether that one runs.  B requests
// at odd addresses are slow, and from memory a K-step is not time enough for them.  Two buffers over three, operands from memory / from the caches,
// fourteen shapes, K 264 / 520 / 776 / 1032 / 2056 / 4104:
//   64,64,128,128   0.97 / 1.00 / 1.04 / 1.06 / 1.1 / 1.14    0.95 - 0.98 / 0.98 - 0.99 / 0.98 - 1.00 / 0.99 - 1.01 / 1.00 - 1.03 / 1.01 - 1.03 (600 x 3001 x 4104 46.5 / 40.6 and 34.1 / 33.9 us)
//   128,128,64,128  1.02 / 1.08 / 1.14 / 1.17 / 1.25 / 1.31   0.97 - 0.98 / 0.98 - 1.00 / 0.98 - 1.01 / 0.97 - 1.02 / 1.00 - 1.04 / 1.00 - 1.05 (300 x 3001 x 4104 59.9 / 45.9 and 44.4 / 43.0)
// The line is where two buffers begin to lose from memory what B through registers had (600 x 5001 x 776 25.2 / 25.5).  Two workgroups of 128 x 128 tiles
// fit a CU with two buffers but not with three: 3000 x 1281 x 776 24.9 / 29.8.
inline bool odd_n_third_buffer(const GemmParams &p, int T_MC, int T_N, int cus)
{
    return p.N % 2 != 0 && p.K >= 768 && (T_MC < 128 || tile_count(p, T_MC, T_N) <= cus);
}

// B^T in bf16 that the pipeline runs: the side of the square tiles (64: 64,64,64,64; 128: 64,128,64,128; the same bits) that take a problem too small
// for the tiles of 128 x 256 and more that a plan can name; 0 where those run.  The latter over 64 / 128, 200 problems, by the number of the
// square tiles: up to 256 64 x 64 ones 1.4 - 1.7 / 1.15 - 1.3 at K 72, 1.65 - 1.8 / 1.25 - 1.35 at 264, 1.7 - 1.9 / 1.3 - 1.4 at 520, 1.7 - 2.1 / 1.3 - 1.45 at 1024;
// 512 of them 1.27 - 1.55 / 1.2 - 1.34, 625 1.18 - 1.38 / 1.27 - 1.38, 1024 0.93 - 0.99 / 1.18 - 1.33 (256 128 x 128 ones); 315 128 x 128 ones 0.9 / 0.96 - 0.99.
// us: 1000 x 1000 x 1024 16.7 / 8.9, 100 x 2000 x 520 10.9 / 5.8, 88 x 1792 x 72 5.7 / 3.6, 1000 x 4000 x 520 12.7 / 9.7.
inline int bt_small_tiles(const GemmParams &p, int cus) { return tile_count(p, 64, 64) <= 2 * cus ? 64 : tile_count(p, 128, 128) <= cus ? 128 : 0; }

}  // namespace atb

// BFP16 quantiser and stand-alone decoder for gfx950.
//
// BFP16 (Sec. 2.4 of arXiv 2511.16041): 8 consecutive values along K share one
// 8-bit exponent, each keeps an 8-bit mantissa.  The reading implemented here:
//   E = max over the block of the fp32 biased exponent field (= 127 + floor(log2|x|)
//       for normal x; fp32 subnormals and zeros contribute 0),
//   m = clamp(round_to_nearest_even(x * 2^(133 - E)), -127, 127),
//   value = m * 2^(E - 133).
// All kernels here are HBM-bound streaming kernels.  The BFP16
// buffer is K-panel-major (see include/atb.h): [panel of 64 k][row][64] mantissas, [panel][row][8] exponents.
#include <mutex>

#include "atb_device.h"
#include "atb_route.h"

namespace atb {
namespace {

// Quantiser.  A wave covers 2 STEPS rows x 128 k (two panels of the K-panel-major output); the 4 waves of a
// workgroup sit side by side along k.  In step v lanes 0-31 take row 2v and lanes 32-63 row 2v + 1, four
// consecutive k each, so a load instruction reads two contiguous runs of 512 B and the mantissa store of the
// same step writes, per panel, the 2 x 64 B of the row pair, which are one 128-byte line of the output.  A
// BFP16 block is the 8 values of two neighbouring lanes, which exchange their exponent maxima.  The
// exponent bytes of the wave, 16 per row, are collected in LDS and leave as two contiguous runs.  Chunks beyond K
// (the tail of the last panel) are written as zero.
// STEPS: quantize_route chooses; 8192 x 8192 53.4 us = 6.4 TB/s.
template <int STEPS>
__global__ void __launch_bounds__(256) quantize_kernel(const float *__restrict__ A, int64_t lda,
                                                       int8_t *__restrict__ Am, uint8_t *__restrict__ Ae,
                                                       int64_t M, int64_t K, int64_t panels, int64_t kblocks)
{
    constexpr int ROWS = 2 * STEPS;
    __shared__ __attribute__((aligned(8))) uint8_t exps[4][2][ROWS][8];
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63, half = lane >> 5, q = lane & 31;
    const int64_t r0 = ((int64_t)blockIdx.x / kblocks) * ROWS;
    const int64_t kg = ((int64_t)blockIdx.x % kblocks) * 4 + wave;       // group of 128 k
    const int64_t k = kg * 128 + 4 * q;
    const int64_t panel = kg * 2 + (q >> 4);
    const int kin = 4 * (q & 15);
#pragma unroll
    for (int v = 0; v < STEPS; ++v) {
        const int64_t row = r0 + 2 * v + half;
        // the input is read once: non-temporal loads (+12 % whether or not the input was in a cache before the
        // launch); the output keeps ordinary stores, its reader comes next
        floatx4 f = {0.0f, 0.0f, 0.0f, 0.0f};
        if (row < M && k < K) f = __builtin_nontemporal_load(reinterpret_cast<const floatx4 *>(A + row * lda + k));     // K % 8 == 0: k < K implies k + 4 <= K
        unsigned e = max(max(exp_field(f.x), exp_field(f.y)), max(exp_field(f.z), exp_field(f.w)));
        e = max(e, (unsigned)__shfl_xor((int)e, 1));
        const int shift = 133 - (int)e;
        const float x[4] = {f.x, f.y, f.z, f.w};
        const unsigned w = bfp16_mantissas4(x, shift);
        if (row < M && panel < panels) *reinterpret_cast<unsigned *>(Am + (panel * M + row) * kPanelK + kin) = w;
        if ((q & 1) == 0) exps[wave][q >> 4][2 * v + half][(q & 15) >> 1] = (uint8_t)e;
    }
    __syncthreads();
    if (lane < 2 * ROWS) {
        const int pl = lane / ROWS, rl = lane % ROWS;
        const int64_t row = r0 + rl, pn = kg * 2 + pl;
        if (row < M && pn < panels)
            *reinterpret_cast<uint2 *>(Ae + (pn * M + row) * (kPanelK / 8)) = *reinterpret_cast<const uint2 *>(&exps[wave][pl][rl][0]);
    }
}

// Decoders.  Bound: HBM, 1.125 B read and 2 B written per element; a small one is its launch (2.1 us).  decode_route says
// which of the two takes a problem.
// A lane takes a block in row order: every store of a wave is contiguous, its requests are pieces of 64 bytes of each panel.
__global__ void __launch_bounds__(256) decode_lanes(const int8_t *__restrict__ Am, const uint8_t *__restrict__ Ae,
                                                    uint16_t *__restrict__ out, int64_t M, int64_t K)
{
    const unsigned blocks_per_row = (unsigned)(K / 8), n = (unsigned)M * blocks_per_row;      // fewer than 2^32: one launch
    const unsigned c = blockIdx.x * 256u + threadIdx.x;
    if (c >= n) return;
    const unsigned row = c / blocks_per_row, kb = c % blocks_per_row;
    const int64_t rec = (int64_t)(kb / 8) * M + row;                                          // (panel, row)
    const int2 w = *reinterpret_cast<const int2 *>(Am + rec * kPanelK + (kb % 8) * 8);
    const int shift = (int)Ae[rec * (kPanelK / 8) + kb % 8] - 133;
    *reinterpret_cast<bf16x8 *>(out + (int64_t)row * K + (int64_t)kb * 8) = bfp16_decode8(w.x, w.y, shift);  // K % 8 == 0: 16-byte aligned as `out` is
}

// A wave takes 8 rows of a panel: a lane one block, eight lanes a row, so that its requests are contiguous (512 + 64 bytes) and
// each of its stores whole 128-byte lines of the output, 8 rows x 64 k.  A wave does R such groups of rows, the workgroup's waves
// neighbouring panels.
// NT: the output is written past the caches.  That pays only for whole lines (K % 64 == 0; with lines shared by two waves it costs
// two partial writes: 8192 x 8104 cold 56.4, hot 34 -> 54), and only for outputs so large that their next reader would not have found
// them in the 256 MiB memory-side cache.  Measured, us, decode / decode and then one pass that reads the output, stores through the
// caches -> past them: 64 MiB 25.3 / 43.0 -> 16.4 / 44.4, 96 MiB - / 66.9 -> - / 64.6, 128 MiB (8192 x 8192) 45.2 / 94.0 -> 31.2 / 85.7
// (6.7 TB/s), 192 MiB - / 134.0 -> - / 130.4: below 96 MiB the reader pays for what the decoder saves.
template <bool NT, int R>
__global__ void __launch_bounds__(256) decode_panels(const int8_t *__restrict__ Am, const uint8_t *__restrict__ Ae,
                                                     uint16_t *__restrict__ out, int64_t M, int64_t K, int64_t panels, unsigned kblocks)
{
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63, q = lane & 7;
    const int64_t row0 = (int64_t)(blockIdx.x / kblocks) * (8 * R) + (lane >> 3);
    const int64_t panel = (int64_t)(blockIdx.x % kblocks) * 4 + wave, k = panel * kPanelK + 8 * q;
    if (panel >= panels || k >= K) return;                   // K % 8 == 0: a block is inside or outside
    int2 w[R] = {};
    int e[R] = {};
#pragma unroll
    for (int g = 0; g < R; ++g) {
        const int64_t row = row0 + 8 * g;
        if (row < M) {
            w[g] = *reinterpret_cast<const int2 *>(Am + (panel * M + row) * kPanelK + 8 * q);
            e[g] = Ae[(panel * M + row) * (kPanelK / 8) + q];
        }
    }
#pragma unroll
    for (int g = 0; g < R; ++g) {
        const int64_t row = row0 + 8 * g;
        const bf16x8 r = bfp16_decode8(w[g].x, w[g].y, e[g] - 133);
        if (row < M) {
            bf16x8 *dst = reinterpret_cast<bf16x8 *>(out + row * K + k);      // 16-byte aligned as `out` is
            if constexpr (NT) __builtin_nontemporal_store(r, dst); else *dst = r;
        }
    }
}

}  // namespace

// Looked up once per device; the table is
// guarded, so concurrent first launches from several threads are fine, and the lookup enqueues nothing
// (a first launch inside a stream capture is as good as any other).
int compute_units()
{
    constexpr int kMaxDevices = 64;
    static std::mutex guard;
    static int cached[kMaxDevices] = {};
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxDevices) return 0;
    std::lock_guard<std::mutex> lock(guard);
    if (cached[dev] == 0) {
        int cus = 0;
        if (hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || cus < 8) return 0;
        cached[dev] = cus;
    }
    return cached[dev];
}

hipError_t launch_quantize(const float *A, int64_t lda, int8_t *Am, uint8_t *Ae, int64_t M, int64_t K,
                           hipStream_t stream)
{
    const int64_t panels = (K + kPanelK - 1) / kPanelK;
    if (M == 0 || panels == 0) return hipSuccess;
    const QuantizeRoute r = quantize_route(M, K);
    if (r.workgroups == 0) return hipErrorInvalidConfiguration;
    auto *kernel = r.steps == 2 ? quantize_kernel<2> : r.steps == 4 ? quantize_kernel<4> : quantize_kernel<8>;
    hipLaunchKernelGGL(kernel, dim3((unsigned)r.workgroups), dim3(256), 0, stream, A, lda, Am, Ae, M, K, panels, (panels + 7) / 8);
    return hipGetLastError();
}

hipError_t launch_decode(const int8_t *Am, const uint8_t *Ae, uint16_t *out, int64_t M, int64_t K,
                         hipStream_t stream)
{
    const int64_t panels = (K + kPanelK - 1) / kPanelK;
    if (M == 0 || panels == 0) return hipSuccess;
    const DecodeRoute r = decode_route(M, K, (reinterpret_cast<uintptr_t>(out) & 127u) == 0);
    if (r.workgroups == 0) return hipErrorInvalidConfiguration;
    const dim3 grid((unsigned)r.workgroups), block(256);
    if (r.rows == 0)
        hipLaunchKernelGGL(decode_lanes, grid, block, 0, stream, Am, Ae, out, M, K);
    else {
        const unsigned kblocks = (unsigned)((panels + 3) / 4);         // a workgroup covers 8 rows (times r.rows) x 4 panels
        auto *kernel = r.past_caches ? decode_panels<true, 2> : r.rows == 2 ? decode_panels<false, 2> : decode_panels<false, 1>;
        hipLaunchKernelGGL(kernel, grid, block, 0, stream, Am, Ae, out, M, K, panels, kblocks);
    }
    return hipGetLastError();
}

}  // namespace atb

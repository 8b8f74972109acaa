// GEMM for few rows and a long reduction (K > 1024): a streaming kernel, bound by the bytes of B.  For M <= 64, and above
// that for problems of at most one 64 x 32 to 128 x 64 tile per CU (stream_route).
//
// With one band of 16 to 64 rows of C there is nothing to share a B tile with, so the tile pipeline of atb_gemm.hip (B
// through LDS, a barrier per K-step, a workgroup per 64 columns) only adds waits.  Here every wave is on its own: the
// W waves of a workgroup share a tile of 16 NB columns and take the 64-wide panels of K in turn, each loads its
// operands straight into registers in MFMA layout, and the W partial C tiles are added once at the end through LDS, in
// wave order (the sums of a result are therefore W shorter chains; the tile pipeline adds in one).
//
// What bounds it: a CU keeps about 200 lines of 128 bytes in flight (measured at M = 16: 27 GB/s per CU from HBM whatever the
// number of waves or of panels in flight per wave, 1 to 4), so all CUs have to take part and every line that is asked for should
// be used whole.  With more rows a wave decodes and multiplies for as long as it waits, and a second panel in flight per wave is
// worth up to 12 % (stream_depth_bfp16, stream_depth_bf16_t).  Hence the tile width (stream_column_blocks): as wide as leaves one workgroup per CU.  With B row-major and N
// <= 8192 that is 32 columns, half a line per row, and the rate stays at 3.9 TB/s against 5.1 with B^T.
// Measured in us, three sets of operands in turns, the tile pipeline before / this kernel now:
//   B bf16    M 16, N 8192, K 8192: 39.6 / 34.5  (64 rows: atb_rows.hip)     M 16, 5001, 4096: 23.7 / 12.9
//   B^T bf16  M 16, N 8192, K 8192: 105 / 29        M 64, 14336, 4096: 57.7 / 29.4
//   B^T BFP16 M 16, N 14336, K 4096: 20.1 / 13.0    M 64, 14336, 4096: 26.0 / 18.7 (decoding A takes as long as B's bytes)
//
// MFMA v_mfma_f32_16x16x32_bf16: lane l supplies index l % 16 of its operand and 8 k values of group l / 16.  Which k
// a group holds is free as long as both operands agree: lane group q takes k = 16 q .. 16 q + 15 of the panel, the
// first half in one MFMA, the second in the next, so that a lane's A operands of a panel are one 16-byte request
// (a wave's requests are then the panel's rows, one contiguous KiB).
//   B row-major bf16   lane c of a group takes the NB neighbouring columns NB c .. of 16 rows; v_perm_b32 pairs the
//                      rows up, which makes MFMA operand p the columns NB c + p.  Odd N: every odd row starts in the
//                      middle of a dword; its lanes fetch the two dwords around their two columns, and the same
//                      v_perm_b32 picks the halves
//   B^T bf16           two 16-byte requests per 16 columns are the operands as they are
//   B^T BFP16          one 16-byte request per 16 columns, decoded in registers like A
#include <type_traits>

#include "atb_device.h"
#include "atb_route.h"

namespace atb {
namespace {

// (a tile's rows of a panel may lie further from the end of B than 2^31 bytes; its offsets do not reach that far)
template <class T>
ATB_DEV __amdgpu_buffer_rsrc_t panel_rsrc(const T *ptr, int64_t bytes)
{
    return uniform_rsrc(ptr, (int)(bytes < 0x7fffffff ? bytes : 0x7fffffff));
}

enum { kBRow = 0, kBT = 1, kBBfp = 2, kBRowOdd = 3 };

// One panel's operands of a lane.
template <int FMT, int MB, int NB>
struct Panel {
    intx4 am[MB];                      // 16 mantissas of a row of A
    unsigned ae[MB];                   // the aligned dword that holds their two exponents
    int b[FMT == kBRow ? 16 * (NB / 2) : FMT == kBRowOdd ? 24 : 1];      // odd N: rows 2 i in b[i], rows 2 i + 1 in b[8 + 2 i], b[9 + 2 i]
    intx4 bt[FMT == kBT ? 2 * NB : FMT == kBBfp ? NB : 1];
    unsigned be[FMT == kBBfp ? NB : 1];
};

template <int FMT, int MB, int NB, int W, int D>
struct Skinny {
    const GemmParams &p;
    int lane, c, q, wave, m0, n0;
    static constexpr bool ROWS = (FMT == kBRow || FMT == kBRowOdd);
    static_assert(NB % 2 == 0 && (FMT != kBRowOdd || NB == 2), "column pairs; odd N is written for one pair per lane");
    int a_off[MB], e_off[MB], b_off[ROWS ? 16 : NB], be_off[NB];
    floatx4 acc[MB][NB];
    Panel<FMT, MB, NB> st[D];          // D panels of this wave in flight

    ATB_DEV Skinny(const GemmParams &p_, int m0_, int n0_) : p(p_), m0(m0_), n0(n0_)
    {
        lane = threadIdx.x & 63;
        c = lane & 15;
        q = lane >> 4;
        wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
        // rows >= M and columns >= N repeat a valid one: they only feed elements of C that are never stored
#pragma unroll
        for (int i = 0; i < MB; ++i) {
            const int row = min(m0 + 16 * i + c, p.M - 1);
            a_off[i] = row * kPanelK + 16 * q;
            e_off[i] = row * (kPanelK / 8) + 4 * (q >> 1);
        }
        if constexpr (ROWS) {
            const int col = min(NB * c, ((p.N - 1) & ~1) - n0);   // even; relative to the tile
#pragma unroll
            for (int j = 0; j < 16; ++j) b_off[j] = (((16 * q + j) * p.N + col) * 2) & ~3;
        } else {
#pragma unroll
            for (int i = 0; i < NB; ++i) {
                const int col = min(16 * i + c, p.N - 1 - n0);
                if constexpr (FMT == kBT) {
                    b_off[i] = (col * p.K + 16 * q) * 2;
                } else {
                    b_off[i] = col * kPanelK + 16 * q;
                    be_off[i] = col * (kPanelK / 8) + 4 * (q >> 1);
                }
            }
        }
#pragma unroll
        for (int i = 0; i < MB; ++i)
#pragma unroll
            for (int j = 0; j < NB; ++j) acc[i][j] = floatx4{0.0f, 0.0f, 0.0f, 0.0f};
    }

    // Panel k of the reduction into st[s]; panels past the last read zeros without touching memory.
    ATB_DEV void load(Panel<FMT, MB, NB> &s, int k)
    {
        const bool live = k < p.k_panels;
        const int64_t kp = live ? k : 0;
        const __amdgpu_buffer_rsrc_t am = panel_rsrc(p.Am + kp * p.M * kPanelK, live ? (int64_t)p.M * kPanelK : 0);
        const __amdgpu_buffer_rsrc_t ae = panel_rsrc(p.Ae + kp * p.M * (kPanelK / 8), live ? (int64_t)p.M * (kPanelK / 8) : 0);
        if constexpr (ROWS) {
            // rows >= K lie past the end of B and read as zero
            const int64_t first = kp * kPanelK * p.N + n0;
            const __amdgpu_buffer_rsrc_t b = panel_rsrc(p.B + first, live ? ((int64_t)p.K * p.N - first) * 2 : 0);
#pragma unroll
            for (int j = 0; j < 16; ++j) {
                if constexpr (FMT == kBRowOdd) {
                    if (j % 2 == 0) {
                        s.b[j / 2] = __builtin_amdgcn_raw_buffer_load_b32(b, b_off[j], 0, 0);
                    } else {
                        const intx2 v = __builtin_amdgcn_raw_buffer_load_b64(b, b_off[j], 0, 0);
                        s.b[7 + j] = v.x;
                        s.b[8 + j] = v.y;
                    }
                } else if constexpr (NB == 8) {
                    const intx4 v = __builtin_amdgcn_raw_buffer_load_b128(b, b_off[j], 0, 0);
#pragma unroll
                    for (int e = 0; e < 4; ++e) s.b[4 * j + e] = v[e];
                } else if constexpr (NB == 4) {
                    const intx2 v = __builtin_amdgcn_raw_buffer_load_b64(b, b_off[j], 0, 0);
                    s.b[2 * j] = v.x;
                    s.b[2 * j + 1] = v.y;
                } else {
                    s.b[j] = __builtin_amdgcn_raw_buffer_load_b32(b, b_off[j], 0, 0);
                }
            }
        } else if constexpr (FMT == kBT) {
            // k >= K runs into the next row of B^T (or past its end, which reads as zero): finite values against the
            // zero tail of A
            const int64_t first = (int64_t)n0 * p.K + kp * kPanelK;
            const __amdgpu_buffer_rsrc_t b = panel_rsrc(p.B + first, live ? ((int64_t)p.N * p.K - first) * 2 : 0);
#pragma unroll
            for (int i = 0; i < NB; ++i) {
                s.bt[2 * i] = __builtin_amdgcn_raw_buffer_load_b128(b, b_off[i], 0, 0);
                s.bt[2 * i + 1] = __builtin_amdgcn_raw_buffer_load_b128(b, b_off[i] + 16, 0, 0);
            }
        } else {
            const int64_t row = kp * p.N + n0;
            const __amdgpu_buffer_rsrc_t bm = panel_rsrc(p.Bm + row * kPanelK, live ? (int64_t)(p.N - n0) * kPanelK : 0);
            const __amdgpu_buffer_rsrc_t be = panel_rsrc(p.Be + row * (kPanelK / 8), live ? (int64_t)(p.N - n0) * (kPanelK / 8) : 0);
#pragma unroll
            for (int i = 0; i < NB; ++i) {
                s.bt[i] = __builtin_amdgcn_raw_buffer_load_b128(bm, b_off[i], 0, 0);
                s.be[i] = __builtin_amdgcn_raw_buffer_load_b32(be, be_off[i], 0, 0);
            }
        }
#pragma unroll
        for (int i = 0; i < MB; ++i) {
            s.am[i] = __builtin_amdgcn_raw_buffer_load_b128(am, a_off[i], 0, 0);
            s.ae[i] = __builtin_amdgcn_raw_buffer_load_b32(ae, e_off[i], 0, 0);
        }
    }

    // With B^T the decode is what the waves wait for, and a multiplication is the shorter instruction: B in BFP16 1.01 - 1.04 x (5 x 5016 x 11328
    // 16.7 / 16.1 us, 256 x 2048 x 8192 23.4 / 22.5), bf16 1.00 - 1.03; row-major B 0.99 - 1.005.
    typedef typename std::conditional<ROWS, int, float>::type Scale;
    ATB_DEV static Scale scale_of(unsigned e, int q, int h)
    {
        const int E = (int)((e >> (16 * (q & 1) + 8 * h)) & 0xFFu);
        if constexpr (ROWS) return E - 133;
        else return ldexpf(0x1p-133f, E);
    }

    ATB_DEV void multiply(const Panel<FMT, MB, NB> &s)
    {
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            bf16x8 bf[NB];
#pragma unroll
            for (int j = 0; j < NB; ++j) {
                if constexpr (FMT == kBRowOdd) {
                    union { unsigned w[4]; bf16x8 v; } u;
#pragma unroll
                    for (int t = 0; t < 4; ++t) {
                        const int i = 4 * h + t;
                        u.w[t] = j == 0 ? __builtin_amdgcn_perm(s.b[8 + 2 * i], s.b[i], 0x07060100u) : __builtin_amdgcn_perm(s.b[9 + 2 * i], s.b[i], 0x05040302u);
                    }
                    bf[j] = u.v;
                } else if constexpr (FMT == kBRow) {
                    union { unsigned w[4]; bf16x8 v; } u;
#pragma unroll
                    for (int t = 0; t < 4; ++t) {
                        const unsigned r0 = s.b[(8 * h + 2 * t) * (NB / 2) + j / 2], r1 = s.b[(8 * h + 2 * t + 1) * (NB / 2) + j / 2];
                        u.w[t] = __builtin_amdgcn_perm(r1, r0, (j & 1) ? 0x07060302u : 0x05040100u);
                    }
                    bf[j] = u.v;
                } else if constexpr (FMT == kBT) {
                    union { intx4 w; bf16x8 v; } u;
                    u.w = s.bt[2 * j + h];
                    bf[j] = u.v;
                } else {
                    bf[j] = bfp16_decode8(s.bt[j][2 * h], s.bt[j][2 * h + 1], scale_of(s.be[j], q, h));
                }
            }
#pragma unroll
            for (int i = 0; i < MB; ++i) {
                const bf16x8 af = bfp16_decode8(s.am[i][2 * h], s.am[i][2 * h + 1], scale_of(s.ae[i], q, h));
#pragma unroll
                for (int j = 0; j < NB; ++j) acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(bf[j], af, acc[i][j], 0, 0, 0);
            }
        }
    }

    // Two panels in flight per wave, the one requested while the other is multiplied.  The fences keep the compiler from sinking the first
    // panel's requests below the second's arithmetic.
    static constexpr bool FENCED = D > 1;

    ATB_DEV void run()
    {
#pragma unroll
        for (int d = 0; d < D; ++d) {
            load(st[d], wave + d * W);
            if constexpr (FENCED) __builtin_amdgcn_sched_barrier(0);
        }
        for (int k = wave; k < p.k_panels; k += D * W) {
#pragma unroll
            for (int d = 0; d < D; ++d) {
                multiply(st[d]);
                if constexpr (FENCED) __builtin_amdgcn_sched_barrier(0);
                load(st[d], k + (D + d) * W);
                if constexpr (FENCED) __builtin_amdgcn_sched_barrier(0);
            }
        }
    }

    // Column of the tile that register t of acc[.][j] holds in this lane (its row is lane % 16 of the row block).
    ATB_DEV int column(int j, int t) const { return ROWS ? NB * (4 * q + t) + j : 16 * j + 4 * q + t; }

    // 128 columns of row-major B: a lane has eight consecutive columns per register index, 16 bytes of C or a whole BFP16 block.
    // This wave's sums of row block i to LDS, [register][half][lane].  (The asm keeps the branches apart: merged, they would index acc at
    // run time.)
    static constexpr bool EIGHTS = (FMT == kBRow && NB == 8);
    template <int a = 0>
    ATB_DEV void put_eights(int i, floatx4 *part) const
    {
        if constexpr (a < MB) {
            if (i == a) {
                asm volatile("" : : "n"(a));
#pragma unroll
                for (int t = 0; t < 4; ++t)
#pragma unroll
                    for (int h = 0; h < 2; ++h)
                        part[(2 * t + h) * 64 + lane] = floatx4{acc[a][4 * h][t], acc[a][4 * h + 1][t], acc[a][4 * h + 2][t], acc[a][4 * h + 3][t]};
                asm volatile("" : : "n"(a));
            } else {
                put_eights<a + 1>(i, part);
            }
        }
    }
};

template <int FMT, int MB, int NB, int W, int D>
__global__ void __launch_bounds__(W * 64) skinny_kernel(const GemmParams p)
{
    constexpr int TN = 16 * NB, PITCH = TN + 4;
    __shared__ __attribute__((aligned(16))) float part[W][16][PITCH];
    // consecutive tiles on one XCD, rows of tiles first: they share B's columns, and neighbouring columns the 128-byte
    // lines of a row of B, in that XCD's L2
    const int per_xcd = ((int)gridDim.x + 7) / 8;
    const int tile = (int)(blockIdx.x % 8) * per_xcd + (int)blockIdx.x / 8;
    const int cols = p.Cm ? p.n_panels * kPanelK : p.N;          // C in BFP16: the zero tail of the last panel as well
    const int rows = (p.M + 16 * MB - 1) / (16 * MB), m0 = tile % rows * (16 * MB), n0 = tile / rows * TN;
    if (n0 >= cols) return;                                       // the whole workgroup
    const bool any = n0 < p.N;                                    // else a tile of that tail: nothing to multiply
    Skinny<FMT, MB, NB, W, D> sk(p, m0, any ? n0 : 0);
    if (any) sk.run();
    // The sums of the waves' partial tiles, row block by row block.  Four row blocks unrolled are 4 KiB of code that runs once, and such
    // code comes into the instruction cache at about two bytes per ns; for tiles of 128 columns, which have up to four and eight
    // accumulator blocks in each, one copy serves them all (26.6 -> 25.5 us for 1024 x 2048 x 4096 when it ran here; the narrower tiles lose 1 %).
    if constexpr (Skinny<FMT, MB, NB, W, D>::EIGHTS) {
        floatx4 *const mem = reinterpret_cast<floatx4 *>(&part[0][0][0]);
        static_assert(W * 8 * 64 * sizeof(floatx4) <= sizeof(part), "a row block's partial sums");
#pragma nounroll
        for (int i = 0; i < MB; ++i) {
            if (i > 0) __syncthreads();
            sk.put_eights(i, mem + sk.wave * (8 * 64));
            __syncthreads();
#pragma nounroll
            for (int t = sk.wave; t < 4; t += W) {
                const floatx4 *const src = mem + t * 128 + sk.lane;
                floatx4 sum[2] = {src[0], src[64]};
#pragma unroll
                for (int w = 1; w < W; ++w) {
                    sum[0] += src[w * (8 * 64)];
                    sum[1] += src[w * (8 * 64) + 64];
                }
                store_eight(p, m0 + 16 * i + sk.c, n0 + 8 * (4 * sk.q + t), sum, cols);
            }
        }
        return;
    }
#pragma unroll
    for (int i = 0; i < MB; ++i) {
        if (i > 0) __syncthreads();
#pragma unroll
        for (int j = 0; j < NB; ++j)
#pragma unroll
            for (int v = 0; v < 4; ++v) part[sk.wave][sk.c][sk.column(j, v)] = sk.acc[i][j][v];
        __syncthreads();
        // item t of 64 NB: row t / (TN / 4) of the row block, four columns from 4 (t % (TN / 4))
        for (int t = threadIdx.x; t < 64 * NB; t += W * 64) {
            const int rr = t / (TN / 4), cc = 4 * (t % (TN / 4));
            floatx4 sum = *reinterpret_cast<const floatx4 *>(&part[0][rr][cc]);
#pragma unroll
            for (int w = 1; w < W; ++w) sum += *reinterpret_cast<const floatx4 *>(&part[w][rr][cc]);
            const int m = m0 + 16 * i + rr, n = n0 + cc;
            if (p.Cm) {
                // BFP16 C, as TileKernel::store_c_bfp: a block is this thread's four columns and its neighbour's
                unsigned e = 0;
                float x[4];
#pragma unroll
                for (int v = 0; v < 4; ++v) {
                    x[v] = n < p.N ? sum[v] : 0.0f;               // whole blocks: N % 8 == 0
                    e = max(e, exp_field(x[v]));
                }
                e = max(e, (unsigned)__shfl_xor((int)e, 1));
                const unsigned w = bfp16_mantissas4(x, 133 - (int)e);
                if (m < p.M && n < cols) {
                    const int64_t rec = (int64_t)(n / kPanelK) * p.M + m;
                    *reinterpret_cast<unsigned *>(p.Cm + rec * kPanelK + n % kPanelK) = w;
                    if ((t & 1) == 0) p.Ce[rec * (kPanelK / 8) + (n % kPanelK) / 8] = (uint8_t)e;
                }
            } else if (m < p.M) {
                union { bf16x4 v; uint16_t h[4]; } u;
#pragma unroll
                for (int v = 0; v < 4; ++v) u.v[v] = (__bf16)sum[v];
                uint16_t *dst = p.C + (int64_t)m * p.N + n;
                if (n + 4 <= p.N) {
                    *reinterpret_cast<bf16x4_u *>(dst) = u.v;
                } else {
#pragma unroll
                    for (int v = 0; v < 4; ++v)
                        if (n + v < p.N) dst[v] = u.h[v];
                }
            }
        }
    }
}

template <int FMT, int MB, int NB, int W, int D = 1>
hipError_t launch(const GemmParams &p, const StreamRoute &r, hipStream_t stream)
{
    hipLaunchKernelGGL((skinny_kernel<FMT, MB, NB, W, D>), dim3((unsigned)stream_workgroups(p, r)), dim3(W * 64), 0, stream, p);
    return hipGetLastError();
}

// One of 1 to MAX blocks of 16 rows.
template <int FMT, int NB, int W, int MAX>
hipError_t launch_rows(const GemmParams &p, const StreamRoute &r, hipStream_t stream)
{
    if (r.mb == 1) return launch<FMT, 1, NB, W>(p, r, stream);
    if (r.mb == 2) return launch<FMT, 2, NB, W>(p, r, stream);
    if constexpr (MAX >= 3)
        if (r.mb == 3) return launch<FMT, 3, NB, W>(p, r, stream);
    if constexpr (MAX == 4)
        if (r.mb == 4) return launch<FMT, 4, NB, W>(p, r, stream);
    return hipErrorInvalidValue;
}

}  // namespace

// The variants that stream_route chooses from; no others are compiled, and a route to another is refused.
hipError_t launch_skinny(const GemmParams &p, int b_format, const StreamRoute &r, hipStream_t stream)
{
    const int form = 1000 * r.depth + 100 * r.nb + r.waves;
    if (b_format == ATB_FMT_BFP16) {
        if (form == 1216) return launch_rows<kBBfp, 2, 16, 4>(p, r, stream);
        if (form == 1408) return launch_rows<kBBfp, 4, 8, 4>(p, r, stream);
        if (form == 1808) return launch_rows<kBBfp, 8, 8, 3>(p, r, stream);
        if (form == 1208 && r.mb == 4) return launch<kBBfp, 4, 2, 8>(p, r, stream);
        if (form == 2408 && r.mb == 2) return launch<kBBfp, 2, 4, 8, 2>(p, r, stream);
        if (form == 2408 && r.mb == 3) return launch<kBBfp, 3, 4, 8, 2>(p, r, stream);
        if (form == 2408 && r.mb == 4) return launch<kBBfp, 4, 4, 8, 2>(p, r, stream);
        if (form == 2208 && r.mb == 4) return launch<kBBfp, 4, 2, 8, 2>(p, r, stream);
    } else if (b_format == ATB_FMT_BF16_T) {
        if (form == 1208) return launch_rows<kBT, 2, 8, 4>(p, r, stream);
        if (form == 1404 && r.mb == 8) return launch<kBT, 8, 4, 4>(p, r, stream);
        if (form == 1404) return launch_rows<kBT, 4, 4, 2>(p, r, stream);
        if (form == 2404 && r.mb == 3) return launch<kBT, 3, 4, 4, 2>(p, r, stream);
        if (form == 2404 && r.mb == 4) return launch<kBT, 4, 4, 4, 2>(p, r, stream);
        if (form == 1804) return launch_rows<kBT, 8, 4, 4>(p, r, stream);
        if (form == 1408 && r.mb == 4) return launch<kBT, 4, 4, 8>(p, r, stream);
    } else if (p.N % 2 != 0) {
        if (form == 1208) return launch_rows<kBRowOdd, 2, 8, 4>(p, r, stream);
    } else {
        if (form == 1208) return launch_rows<kBRow, 2, 8, 3>(p, r, stream);
        if (form == 1404) return launch_rows<kBRow, 4, 4, 3>(p, r, stream);
        if (r.in_lds) return launch_lds_rows(p, r, stream);
        if (form == 1804) return launch_rows<kBRow, 8, 4, 4>(p, r, stream);
        if (form == 1408 && r.mb == 4) return launch<kBRow, 4, 4, 8>(p, r, stream);
    }
    return hipErrorInvalidValue;
}

}  // namespace atb

// The streaming kernel (atb_skinny.hip has its idea: the waves of a workgroup share a C tile and take the 64-wide panels of K in turn) for
// 64 rows, row-major bf16 B of even N and 64 or 128 columns.  Tiles this large keep a wave's MFMAs as busy as its loads, so what bounds
// them is one wave per SIMD, which starts at most one instruction, of whatever kind, in four cycles: a panel of a 64 x 128 tile has 64
// MFMAs of 16 cycles, which leave room for 192 other instructions, and decoding A alone takes 168.  So:
//   * B goes straight into LDS, in rings of two panels that belong to one wave each (no barriers), and comes out as MFMA operands through
//     the transposing read: 16 requests and 32 reads per panel in place of 16 loads, 64 v_perm_b32 and 64 registers;
//   * A comes in through LDS too, so that every request of a wave is issued by hand and its waits are counted by hand;
//   * each MFMA is followed by two or three of the decode's instructions for the next row block, none of which waits for the one before it,
//     and the requests are spread over the panel: bunched, they fill the queue to the caches and the wave stands still;
//   * descriptors, LDS addresses and M0 take three scalar instructions per request and about twenty per panel.
// What is left is bytes into a CU: 84 KB per round of panels at 95 to 100 GB/s, what a loop of such requests alone reaches from the caches.
// us, operands through registers with the compiler's schedule / now: 1024 x 2048 x 4096 25.5 / 21.9 (27.1 / 25.8 from memory), 512 x 4096 x 4096 25.8 / 21.8
// (27.8 / 26.8), 200 x 8000 x 4096 26.1 / 21.8 (28.8 / 27.0); 64 x 8256 x 4096 21.8 / 16.9 (26.3 / 21.3), 64 x 14336 x 4096 29.3 / 28.3 (29.5 / 28.4).
#include "atb_device.h"
#include "atb_route.h"

namespace atb {
namespace {

#define ATB_FENCE() __builtin_amdgcn_sched_barrier(0)

typedef short shortx4 __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(3))) shortx4 lds_shortx4;

// LDS of a workgroup.  The static part is as large as the partial C tile of one wave and holds wave 0's ring, then its partial tile; the
// rest is asked for at the launch.
template <int MB, int NB, int W>
struct RowsLds {
    static constexpr int PANEL = 64 * NB * 32;                       // a panel of B
    static constexpr int RING = 2 * PANEL;                           // a wave's panels
    static constexpr int A_MANT = MB * 1024, A_BYTES = A_MANT + (MB + 1) / 2 * 256;      // a panel of A: mantissas, exponents
    static constexpr int PITCH = 16 * NB + 4;                        // floats in a row of a partial C tile: its 16-byte stores hit every bank once
    static constexpr int PART = 16 * MB * PITCH * 4;
    static constexpr int FIXED = W * 16 * PITCH * 4;
    static constexpr int A_AT = (W - 1) * RING;                      // in the dynamic part: the rings of waves 1 .. W - 1, then A
    static constexpr int DYNAMIC = rows_dynamic_lds(MB, NB, W);
    static_assert(DYNAMIC >= A_AT + W * A_BYTES && DYNAMIC >= (W - 1) * PART, "the other waves, before and after");
    static_assert(RING <= FIXED && PART <= FIXED, "wave 0 lives in the static part");
    static_assert(FIXED + DYNAMIC <= 160 * 1024, "LDS of a CU");
};

template <int MB, int NB, int W>
struct Rows {
    typedef RowsLds<MB, NB, W> L;
    static constexpr int CPR = 2 * NB;                 // 16-byte chunks per row of a panel, requests per panel
    static constexpr int GROUPS = 2 * MB;              // A fragments per panel: row block g % MB, half g / MB
    static constexpr int A_REQ = MB + (MB + 1) / 2;    // requests per panel of A
    const GemmParams &p;
    int lane, c, q, wave, m0, n0;
    int b_off[CPR], a_off[MB], e_off[(MB + 1) / 2];    // byte offsets of this lane's requests in a panel
    const char *b_rd[NB], *a_rd, *e_rd;                // where this lane reads its fragments
    unsigned fill, a_at;                               // LDS addresses of the panel being multiplied, of A
    int step;                                          // from that panel of the ring to the other one
    intx4 b_words, am_words, ae_words;                 // descriptors of the panels that are requested next
    int rows_left;                                     // rows of B from there on
    floatx4 acc[MB][NB];
    bf16x8 bf[2][NB], af[2];                           // B fragments of the two halves of a panel, A fragments of this group and the next
    intx4 am[MB];                                      // 16 mantissas of a row of A, and their two exponents
    unsigned ae[MB];
    float cv[8];
    unsigned dec[4];
    int shift;

    // A panel is two halves; half h has k = 16 q + 8 h + e (q = 0 .. 3, e = 0 .. 7), the k order of the other streaming kernels, and is
    // kept as 32 rows 8 q + e of LDS.  Chunk x of a row is at position x ^ swz(row): the 8 rows that 32 lanes of a transposing read
    // touch (e and e + 8, four of each) then lie in different banks.
    static constexpr int swz(int row) { return NB == 8 ? ((row & 3) << 2) | (((row >> 3) & 1) << 1) : (((row >> 1) & 1) << 1) | (((row >> 3) & 1) << 2); }
    static constexpr int k_of(int row) { return 16 * ((row >> 3) & 3) + 8 * (row >> 5) + (row & 7); }
    static_assert(NB == 8 || NB == 4, "the swizzles are written for rows of 16 and 8 chunks");
    static_assert(MB == 4, "the time line of slots() is checked for four row blocks");

    static ATB_DEV int uni(int x) { return __builtin_amdgcn_readfirstlane(x); }
    static ATB_DEV intx4 words(const void *ptr, int bytes)
    {
        const uint64_t a = reinterpret_cast<uint64_t>(ptr);
        return intx4{uni((int)(uint32_t)a), uni((int)(uint32_t)(a >> 32) & 0xFFFF), uni(bytes), kRsrcFlags};
    }

    ATB_DEV Rows(const GemmParams &p_, char *fixed, char *dynamic, int m0_, int n0_) : p(p_), m0(m0_), n0(n0_)
    {
        lane = threadIdx.x & 63;
        c = lane & 15;
        q = lane >> 4;
        wave = uni((int)threadIdx.x >> 6);
        char *const ring = wave == 0 ? fixed : dynamic + (wave - 1) * L::RING;
        char *const a_lds = dynamic + L::A_AT + wave * L::A_BYTES;
        fill = (unsigned)reinterpret_cast<uintptr_t>(ring);
        a_at = (unsigned)reinterpret_cast<uintptr_t>(a_lds);
        // request j fills the KiB at j of the panel, lane l its 16 bytes at l; columns >= N run into the next row (or past the end of B, which
        // reads as zero) and only feed columns of C that are never stored
#pragma unroll
        for (int j = 0; j < CPR; ++j) {
            const int row = (64 * j + lane) / CPR;
            b_off[j] = k_of(row) * p.N * 2 + ((lane % CPR) ^ swz(row)) * 16;
        }
        // A: the row block's 16 x 64 mantissas, the 16-byte chunks of row r at position x ^ (-(r / 4) mod 4), which keeps the reads of
        // four chunk columns at once out of each other's banks.  Rows >= M repeat the last one: they feed rows of C that are never stored.
#pragma unroll
        for (int i = 0; i < MB; ++i) a_off[i] = min(m0 + 16 * i + lane / 4, p.M - 1) * kPanelK + ((lane % 4) ^ (-(lane / 16) & 3)) * 16;
#pragma unroll
        for (int i = 0; i < (MB + 1) / 2; ++i) e_off[i] = min(m0 + 32 * i + lane / 2, p.M - 1) * (kPanelK / 8) + (lane % 2) * 4;
        // B fragment: within each group of 16 lanes, lane i addresses 4 consecutive columns of row i / 4, and lane j receives column j of
        // those 4 rows; a second read, 4 rows on, completes the lane's 8 k values
        const int r = c >> 2, row = 8 * q + r;
#pragma unroll
        for (int j = 0; j < NB; ++j) b_rd[j] = ring + row * (NB * 32) + (((2 * j + ((c & 3) >> 1)) ^ swz(row)) * 16) + (c & 1) * 8;
        a_rd = a_lds + c * 64 + ((q ^ (-(c >> 2) & 3)) * 16);
        e_rd = a_lds + L::A_MANT + c * (kPanelK / 8) + 2 * q;
        rows_left = max(p.K - wave * kPanelK, 0);
        b_words = words(p.B + (int64_t)wave * kPanelK * p.N + n0, b_bytes());
        const int panels = max(p.k_panels - wave, 0);
        am_words = words(p.Am + (int64_t)wave * p.M * kPanelK, panels * p.M * kPanelK);
        ae_words = words(p.Ae + (int64_t)wave * p.M * (kPanelK / 8), panels * p.M * (kPanelK / 8));
    }

    // ---- requests ---------------------------------------------------------------------------
    // 64 x 16 (or 4) bytes straight into LDS at the wave-uniform address base + at.  By hand, because the compiler would wait for all of a
    // wave's requests ahead of every LDS read.  M0 is not put back: nothing else in this kernel has a use for it (its code is checked for that).
    template <int at>
    static ATB_DEV void dma16(unsigned base, int off, const intx4 &w)
    {
#if defined(__HIP_DEVICE_COMPILE__)
        asm volatile("s_add_u32 m0, %0, %1\n\ts_nop 0\n\tbuffer_load_dwordx4 %2, %3, 0 offen lds" : : "s"(base), "i"(at), "v"(off), "s"(w) : "memory", "scc");
#endif
    }
    template <int at>
    static ATB_DEV void dma4(unsigned base, int off, const intx4 &w)
    {
#if defined(__HIP_DEVICE_COMPILE__)
        asm volatile("s_add_u32 m0, %0, %1\n\ts_nop 0\n\tbuffer_load_dword %2, %3, 0 offen lds" : : "s"(base), "i"(at), "v"(off), "s"(w) : "memory", "scc");
#endif
    }
    template <int j>
    ATB_DEV void request_a()
    {
        if constexpr (j < MB) dma16<j * 1024>(a_at, a_off[j], am_words);
        else dma4<L::A_MANT + (j - MB) * 256>(a_at, e_off[j - MB], ae_words);
    }
    // Requests [j, end) of a panel of A, then (from A_REQ on) of one of B into the ring's place `fill`
    template <int j, int end>
    ATB_DEV void requests()
    {
        if constexpr (j < end) {
            if constexpr (j < A_REQ) request_a<j>();
            else dma16<(j - A_REQ) * 1024>(fill, b_off[j - A_REQ], b_words);
            requests<j + 1, end>();
        }
    }

    // The descriptors of the wave's next panel.  Past the last one nothing is left in them, and requests read zeros without touching memory.
    static ATB_DEV void advance(intx4 &w, int by)
    {
        const uint64_t a = (((uint64_t)(unsigned)w.y << 32) | (unsigned)w.x) + (unsigned)by;
        w.x = uni((int)(uint32_t)a);
        w.y = uni((int)(uint32_t)(a >> 32));
    }
    ATB_DEV void advance_a()
    {
        advance(am_words, W * p.M * kPanelK);
        advance(ae_words, W * p.M * (kPanelK / 8));
        am_words.z = uni(max(am_words.z - W * p.M * kPanelK, 0));
        ae_words.z = uni(max(ae_words.z - W * p.M * (kPanelK / 8), 0));
    }
    // A panel's rows below K, from its column n0 (N < 2^21: K N < 2^31 and K > 1024)
    ATB_DEV int b_bytes() const { return max(min(rows_left, kPanelK) * p.N - n0, 0) * 2; }
    ATB_DEV void advance_b()
    {
        advance(b_words, W * kPanelK * 2 * p.N);
        rows_left = max(rows_left - W * kPanelK, 0);
        b_words.z = uni(b_bytes());
    }

    template <int younger>
    static ATB_DEV void wait_vm()        // for all requests but the `younger` last ones
    {
        __builtin_amdgcn_s_waitcnt((younger & 15) | (7 << 4) | (15 << 8) | ((younger >> 4) << 14));
    }
    static ATB_DEV void wait_lds() { asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory"); }

    // ---- LDS -> registers -------------------------------------------------------------------
    // Read t of 2 NB of half h, `at` bytes from the panel that b_rd is at
    template <int h, int t>
    ATB_DEV void read_b(int at)
    {
        const char *src = b_rd[t / 2] + at + (32 * h + 4 * (t % 2)) * (NB * 32);
        union { shortx4 s[2]; bf16x8 b; } u;
        u.b = bf[h][t / 2];
        u.s[t % 2] = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_shortx4 *)src);
        bf[h][t / 2] = u.b;
    }
    template <int h, int t, int end>
    ATB_DEV void read_bs(int at)
    {
        if constexpr (t < end) { read_b<h, t>(at); read_bs<h, t + 1, end>(at); }
    }
    template <int i>
    ATB_DEV void read_a()
    {
        am[i] = *reinterpret_cast<const intx4 *>(a_rd + i * 1024);
        ae[i] = *reinterpret_cast<const uint16_t *>(e_rd + i * 16 * (kPanelK / 8));
    }
    // Row block i of the next panel: from slot w on, and once this panel's has been decoded for the last time
    template <int m, int w, int i = 0>
    ATB_DEV void read_a_at()
    {
        if constexpr (i < MB) {
            if constexpr (m == (i == 0 || w + i > (MB + i) * NB ? w + i : (MB + i) * NB)) read_a<i>();
            read_a_at<m, w, i + 1>();
        }
    }

    // Instruction n of the decode of group g's A fragment.  order[n] = 0 .. 7: mantissa to float, 8 .. 15: scaled, 16 .. 19: a pair packed, 20: the
    // exponent; none waits for the one before it.
    static constexpr int OPS = 21;
    static constexpr int op_at(int n)
    {
        constexpr int order[OPS] = {20, 0, 1, 2, 8, 3, 9, 4, 10, 16, 11, 5, 12, 17, 6, 13, 7, 18, 14, 15, 19};
        return order[n];
    }
    template <int g, int n, int end>
    ATB_DEV void decode()
    {
        if constexpr (n < end) {
            constexpr int i = g % MB, h = g / MB, op = op_at(n);
            if constexpr (op < 8) {
                cv[op] = (float)(int)(signed char)(am[i][2 * h + op / 4] >> (8 * (op % 4)));
            } else if constexpr (op < 16) {
                cv[op - 8] = ldexpf(cv[op - 8], shift);
            } else if constexpr (op < 20) {
                union { bf16x2 v; unsigned w; } pk;
                pk.v = bf16x2{(__bf16)cv[2 * (op - 16)], (__bf16)cv[2 * (op - 16) + 1]};
                dec[op - 16] = pk.w;
            } else {
                shift = (int)((ae[i] >> (8 * h)) & 0xFFu) - 133;
            }
            if constexpr (n == OPS - 1) {
                union { unsigned w[4]; bf16x8 v; } o;
#pragma unroll
                for (int t = 0; t < 4; ++t) o.w[t] = dec[t];
                af[g % 2] = o.v;
            }
            decode<g, n + 1, end>();
        }
    }

    // One panel: slot m is its m-th MFMA and what is done in that one's shadow.
    //   decode           of the next group's A fragment, over the slots of this group (the last group's: the next panel's first)
    //   requests         of the next panel of A, whose place was read a panel ago, and of the panel of B after the next, into this one's place: its first
    //                    half in slots FROM1 .. TO1 - 1, its second in FROM2 .. TO2 - 1, by when every fragment of that half has been read
    //   B fragments      of this panel's second half during the first, of the next panel's first half at the end
    //   the wait         ahead of those, for the next panel: younger than its requests are those for B since then
    // When to ask is a matter of where B is; us with operands through registers / asked for in slots NB .. SLOTS / 2 - 1 and SLOTS / 2 .. SLOTS - 1 / now.
    // 128 columns: early, and the second half in one go, since from memory it came late: 1024 x 2048 x 8192 48.7 / 48.3 / 45.6, 1000 x 2000 x 8192
    // 49.7 / 51.5 / 49.4, 700 x 2900 x 8192 50.9 / 53.9 / 51.7 (rows of B that begin at multiples of 8 bytes).  From the caches it is level: 1024 x 2048 x 4096
    // 27.1 / 22.6 / 22.6, x 8192 48.1 / 40.0 / 39.9 (earlier still, slots 28 .. 43, 2 % slower).
    // 64 columns: late, since where rows of B are 32 KiB apart all requests of a CU go to one memory channel, and the more in flight the worse: 64 x
    // 16384 x 14336 88.1 / 91.5 / 89.3, 49 x 16384 x 8192 51.6 / 52.7 / 51.5.  It costs 1 to 2 % where half of the CUs have a tile: 64 x 8256 x 4096
    // from memory 26.3 / 21.2 / 21.4, from the caches 21.8 / 16.5 / 16.9.
    static constexpr int SLOTS = GROUPS * NB, WAIT = SLOTS - 2 * NB - 2;
    static constexpr int FROM1 = 8, TO1 = NB == 8 ? 28 : 17, FROM2 = NB == 8 ? 36 : 22, TO2 = NB == 8 ? 48 : 32;
    static constexpr int spread(int m, int from, int to, int n) { return m <= from ? 0 : m < to ? (m - from) * n / (to - from) : n; }       // of n requests, those before slot m
    static constexpr int first_half(int m) { return spread(m, FROM1, TO1, A_REQ + NB); }
    static constexpr int second_half(int m) { return spread(m, FROM2, TO2, NB); }
    template <int m>
    ATB_DEV void slots()
    {
        static_assert(TO1 <= FROM2 && FROM2 > 3 * NB && TO2 <= SLOTS, "requests in the order that wait_vm counts, none for a place that is still to be read");
        static_assert(first_half(WAIT + 1) >= A_REQ, "all of A's requests are older than what may be under way");
        if constexpr (m < SLOTS) {
            constexpr int g = m / NB, j = m % NB, h = g / MB;
            acc[g % MB][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(bf[h][j], af[g % 2], acc[g % MB][j], 0, 0, 0);
            ATB_FENCE();
            decode<(g + 1) % GROUPS, j * OPS / NB, (j + 1) * OPS / NB>();
            if constexpr (m == FROM1) { wait_lds(); advance_a(); advance_b(); }
            if constexpr (m >= FROM1 && m < TO1) requests<first_half(m), first_half(m + 1)>();
            if constexpr (m > NB && m <= 3 * NB) read_b<1, (m - NB - 1) % (2 * NB)>(0);
            if constexpr (m == FROM2) wait_lds();
            if constexpr (m >= FROM2) requests<A_REQ + NB + second_half(m), A_REQ + NB + second_half(m + 1)>();
            if constexpr (m == WAIT) wait_vm<first_half(WAIT + 1) - A_REQ + second_half(WAIT + 1)>();
            read_a_at<m, WAIT>();
            if constexpr (m >= SLOTS - 2 * NB) read_b<0, (m + 2 * NB - SLOTS) % (2 * NB)>(step);
            ATB_FENCE();
            slots<m + 1>();
        }
    }

    // This wave's share of the first `panels` panels of K.
    ATB_DEV void run(int panels)
    {
        step = L::PANEL;
        requests<0, A_REQ + CPR>();
        advance_b();
        fill += step;
        requests<A_REQ, A_REQ + CPR>();
        fill -= step;
#pragma unroll
        for (int i = 0; i < MB; ++i)
#pragma unroll
            for (int j = 0; j < NB; ++j) {
                acc[i][j] = floatx4{0.0f, 0.0f, 0.0f, 0.0f};
#if defined(__HIP_DEVICE_COMPILE__)
                asm volatile("" : "+a"(acc[i][j]));          // here, while the requests are on their way
#endif
            }
        wait_vm<CPR>();
        read_a<0>();
        read_a<1>();
        read_a<2>();
        read_a<3>();
        read_bs<0, 0, 2 * NB>(0);
        decode<0, 0, OPS>();
        ATB_FENCE();
        for (int k = wave; k < panels; k += W) {
            slots<0>();
#pragma unroll
            for (int j = 0; j < NB; ++j) b_rd[j] += step;
            fill += step;
            step = -step;
        }
        wait_vm<0>();        // requests past the last panel: the partial tiles go where they write zeros
    }
};

// FMT and D have one value each; they stand here so that the name of a compiled form says the same of it as skinny_kernel's does.
template <int FMT, int MB, int NB, int W, int D>
__global__ void __launch_bounds__(W * 64) rows_skinny_kernel(const GemmParams p)
{
    static_assert(FMT == 0 && D == 2, "row-major B of even N, two panels in flight");
    typedef RowsLds<MB, NB, W> L;
    constexpr int TN = 16 * NB;
    __shared__ __attribute__((aligned(16))) char fixed[L::FIXED];
    extern __shared__ __attribute__((aligned(16))) char dynamic[];
    // consecutive tiles on one XCD, rows of tiles first: they share B's columns in that XCD's L2
    const int per_xcd = ((int)gridDim.x + 7) / 8;
    const int tile = (int)(blockIdx.x % 8) * per_xcd + (int)blockIdx.x / 8;
    const int cols = p.Cm ? p.n_panels * kPanelK : p.N;           // C in BFP16: the zero tail of the last panel as well
    const int rows = (p.M + 16 * MB - 1) / (16 * MB), m0 = tile % rows * (16 * MB), n0 = tile / rows * TN;
    if (n0 >= cols) return;                                       // the whole workgroup
    const bool any = n0 < p.N;                                    // else a tile of that tail: nothing to multiply
    Rows<MB, NB, W> r(p, fixed, dynamic, m0, any ? n0 : 0);
    r.run(any ? p.k_panels : 0);
    // the waves' partial tiles, added in wave order
    __syncthreads();
    float *const mine = reinterpret_cast<float *>(r.wave == 0 ? fixed : dynamic + (r.wave - 1) * L::PART);
#pragma unroll
    for (int i = 0; i < MB; ++i)
#pragma unroll
        for (int j = 0; j < NB; ++j) *reinterpret_cast<floatx4 *>(mine + (16 * i + r.c) * L::PITCH + 16 * j + 4 * r.q) = r.acc[i][j];
    __syncthreads();
#pragma nounroll
    for (int t = threadIdx.x; t < 16 * MB * (TN / 8); t += W * 64) {
        const int row = t / (TN / 8), col = 8 * (t % (TN / 8)), at = (row * L::PITCH + col) * 4;
        floatx4 sum[2];
#pragma unroll
        for (int f = 0; f < 2; ++f) {
            sum[f] = *reinterpret_cast<const floatx4 *>(fixed + at + 16 * f);
#pragma unroll
            for (int w = 1; w < W; ++w) sum[f] += *reinterpret_cast<const floatx4 *>(dynamic + (w - 1) * L::PART + at + 16 * f);
        }
        store_eight(p, m0 + row, n0 + col, sum, cols);
    }
}

template <int MB, int NB, int W>
hipError_t launch(const GemmParams &p, const StreamRoute &r, hipStream_t stream)
{
    hipLaunchKernelGGL((rows_skinny_kernel<0, MB, NB, W, 2>), dim3((unsigned)stream_workgroups(p, r)), dim3(W * 64), (RowsLds<MB, NB, W>::DYNAMIC), stream, p);
    return hipGetLastError();
}

}  // namespace

hipError_t launch_lds_rows(const GemmParams &p, const StreamRoute &r, hipStream_t stream)
{
    if (r.mb == 4 && r.nb == 8) return launch<4, 8, 4>(p, r, stream);
    if (r.mb == 4 && r.nb == 4) return launch<4, 4, 4>(p, r, stream);
    return hipErrorInvalidValue;
}

}  // namespace atb

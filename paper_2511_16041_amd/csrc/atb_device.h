// Device code that the kernels share: vector types, buffer descriptors and the two directions of the BFP16 format.
#pragma once

#include "atb_internal.h"

namespace atb {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));
typedef bf16x4 bf16x4_u __attribute__((aligned(2)));     // at any element of a row of C
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef float floatx4 __attribute__((ext_vector_type(4)));
typedef int intx4 __attribute__((ext_vector_type(4)));
typedef int intx2 __attribute__((ext_vector_type(2)));

#define ATB_DEV __device__ __forceinline__

constexpr int kRsrcFlags = 0x00020000;           // raw buffer, 32-bit data format

// Descriptor of the `bytes` bytes at ptr.  It is wave-uniform by construction; saying so keeps it in scalar registers.
template <class T>
ATB_DEV __amdgpu_buffer_rsrc_t uniform_rsrc(const T *ptr, int bytes)
{
    const uint64_t a = reinterpret_cast<uint64_t>(ptr);
    const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)a);
    const uint32_t hi = __builtin_amdgcn_readfirstlane((uint32_t)(a >> 32));
    void *u = reinterpret_cast<void *>(((uint64_t)hi << 32) | lo);
    return __builtin_amdgcn_make_buffer_rsrc(u, 0, __builtin_amdgcn_readfirstlane(bytes), kRsrcFlags);
}

// 8 mantissas (two dwords) scaled, as bf16: exact, |m| <= 127 has 7 significant bits.  The scale is the exponent of a power of two, or that
// power (2^(E - 133), from a denormal on): a multiplication takes 2.5 issue cycles beside MFMAs and four bytes of code, v_ldexp_f32 3.6 to 4.1 and
// eight.
ATB_DEV float scaled(float x, int shift) { return ldexpf(x, shift); }
ATB_DEV float scaled(float x, float power) { return x * power; }
template <class Scale>
ATB_DEV bf16x8 bfp16_decode8(int lo, int hi, Scale scale)
{
    bf16x8 r;
#pragma unroll
    for (int t = 0; t < 4; ++t) {
        r[t] = (__bf16)scaled((float)(int)(signed char)(lo >> (8 * t)), scale);
        r[4 + t] = (__bf16)scaled((float)(int)(signed char)(hi >> (8 * t)), scale);
    }
    return r;
}

ATB_DEV unsigned exp_field(float x) { return (__float_as_uint(x) >> 23) & 0xFFu; }

// Four mantissas of a block with exponent E = 133 - shift: clamp(rne(x * 2^(133 - E)), -127, 127), one byte each
ATB_DEV unsigned bfp16_mantissas4(const float x[4], int shift)
{
    unsigned w = 0;
#pragma unroll
    for (int t = 0; t < 4; ++t) {
        float r = rintf(ldexpf(x[t], shift));           // exact power-of-two scaling, then RNE
        r = fminf(fmaxf(r, -127.0f), 127.0f);
        w |= ((unsigned)((int)r) & 0xFFu) << (8 * t);
    }
    return w;
}

// Columns n .. n + 7 of row m of C (whose rows end, in BFP16 with their zero tail, at column cols).
ATB_DEV void store_eight(const GemmParams &p, int m, int n, const floatx4 (&sum)[2], int cols)
{
    if (__builtin_expect(p.Cm != nullptr, 0)) {
        unsigned e = 0;
        float x[8];
#pragma unroll
        for (int f = 0; f < 8; ++f) {
            x[f] = n < p.N ? sum[f / 4][f % 4] : 0.0f;        // whole blocks: N % 8 == 0
            e = max(e, exp_field(x[f]));
        }
        if (m < p.M && n < cols) {
            const int64_t rec = (int64_t)(n / kPanelK) * p.M + m;
            *reinterpret_cast<intx2 *>(p.Cm + rec * kPanelK + n % kPanelK) = intx2{(int)bfp16_mantissas4(x, 133 - (int)e), (int)bfp16_mantissas4(x + 4, 133 - (int)e)};
            p.Ce[rec * (kPanelK / 8) + (n % kPanelK) / 8] = (uint8_t)e;
        }
    } else if (m < p.M) {
        typedef bf16x8 bf16x8_u __attribute__((aligned(2)));      // rows of C start anywhere
        union { bf16x8 v; uint16_t h[8]; } o;
#pragma unroll
        for (int f = 0; f < 8; ++f) o.v[f] = (__bf16)sum[f / 4][f % 4];
        uint16_t *dst = p.C + (int64_t)m * p.N + n;
        if (n + 8 <= p.N) {
            *reinterpret_cast<bf16x8_u *>(dst) = o.v;
        } else {
#pragma unroll
            for (int f = 0; f < 8; ++f)
                if (n + f < p.N) dst[f] = o.h[f];
        }
    }
}

}  // namespace atb

// Float products on the bf16 matrix instructions: every float is taken apart into three bf16 values, x = h + m + l (each the
// rounding of what the ones before leave: 8 + 8 + 8 significant bits, nothing is lost down to 2^-110), and six of the nine
// products are taken, h h, h m, m h, m m, h l, l h.  What is left out, m l, l m and l l, is up to 2^-24 of |x y|; the sums are
// float.  Six bf16 instructions take 3/8 of the time of the float ones for the same contraction.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace gelo {

typedef float f32x4_t __attribute__((ext_vector_type(4)));
typedef double f64x4_t __attribute__((ext_vector_type(4)));
typedef __bf16 bf16x8_t __attribute__((ext_vector_type(8)));
typedef uint32_t u32x4_t __attribute__((ext_vector_type(4)));

constexpr int kFrag = 512;                                // bf16 values one v_mfma_f32_16x16x32_bf16 takes of an operand: 64 lanes x 8

struct Split { bf16x8_t h, m, l; };
// of 2^SHIFT times the values.  With 16 nothing is lost anywhere: the last bit of the smallest float, 2^-149, is a bf16 then (a
// subnormal one, which the instructions take as it is), but values from 2^112 on leave the range.
template <int SHIFT = 0>
__device__ __forceinline__ Split split3(f32x4_t a, f32x4_t b) {
    constexpr float scale = 1 << SHIFT;
    Split s;
#pragma unroll
    for (int e = 0; e < 8; ++e) {
        const float x = e < 4 ? a[e] : b[e - 4];
        s.h[e] = (__bf16)(x * scale);
        const float r = SHIFT == 0 ? x - (float)s.h[e] : fmaf(x, scale, -(float)s.h[e]);       // exact
        s.m[e] = (__bf16)r;
        s.l[e] = (__bf16)(r - (float)s.m[e]);
    }
    return s;
}

__device__ __forceinline__ bf16x8_t frag_of(const uint16_t* p) { return __builtin_bit_cast(bf16x8_t, *reinterpret_cast<const u32x4_t*>(p)); }
// the three planes of a fragment, `plane` values apart; at: this lane's place in the first one
__device__ __forceinline__ void put_split(uint16_t* at, int64_t plane, const Split& s) {
    *reinterpret_cast<u32x4_t*>(at) = __builtin_bit_cast(u32x4_t, s.h);
    *reinterpret_cast<u32x4_t*>(at + plane) = __builtin_bit_cast(u32x4_t, s.m);
    *reinterpret_cast<u32x4_t*>(at + 2 * plane) = __builtin_bit_cast(u32x4_t, s.l);
}

// acc += A B for FA x FB fragments: A's plane p of fragment f is load_a(p, f), B in registers.  Small products first.
template <int FA, int FB, class LoadA>
__device__ __forceinline__ void products(LoadA&& load_a, const Split (&b)[FB], f32x4_t (&acc)[FA][FB]) {
    bf16x8_t a[FA];
    auto load = [&](int plane) {
#pragma unroll
        for (int f = 0; f < FA; ++f) a[f] = load_a(plane, f);
    };
    auto times = [&](bf16x8_t Split::*plane) {
#pragma unroll
        for (int f = 0; f < FA; ++f)
#pragma unroll
            for (int n = 0; n < FB; ++n) acc[f][n] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[f], b[n].*plane, acc[f][n], 0, 0, 0);
    };
    load(2); times(&Split::h);
    load(1); times(&Split::m); times(&Split::h);
    load(0); times(&Split::l); times(&Split::m); times(&Split::h);
}

}  // namespace gelo

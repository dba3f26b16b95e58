// Householder QR of an n x n matrix (n <= 128) with explicit Q^T by ONE workgroup, the matrix in registers.
#pragma once
#include "gelo_internal.h"

namespace gelo {

// value of lane (lane ^ 1) / (lane ^ 2) of the quad, summed over the quad
__device__ __forceinline__ float quad_sum(float v) {
    v += __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), 0xB1, 0xF, 0xF, false));
    v += __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), 0x4E, 0xF, 0xF, false));
    return v;
}

template <int NR>
struct SmallQrShared {
    // pitch of one quad lane's share of the reflector: the four shares fall on distinct banks (not with a multiple of 32: at 25
    // rows per lane 84 rows took 54 us with a pitch of 32, 51 with 36)
    static constexpr int SEG = (NR + 3) / 4 * 4 + ((NR + 3) / 4 * 4 % 32 == 28 ? 8 : 4);
    __attribute__((aligned(16))) float u[2][4][SEG];
    float inv[2];
    float rdiag[4 * NR];
};

// The four lanes of a quad own ONE column of [G | I] (2 n columns, column c = thread / 4): lane q holds rows q, q + 4,
// ..., NR of them.  Step j applies H_j = I - inv u u^T (u = column j from row j down, its top entry moved away from zero
// by the norm) to every later column: the product u^T x is a walk over the lane's own registers and two additions inside
// the quad, so a step needs one barrier and nothing but the reflector from LDS.  The quad of column j + 1 prepares and
// publishes the next reflector behind its own update, while the other columns are still at theirs.  What bounds it is
// the latency of that chain (barrier, LDS read, product, square root and reciprocal, update): a launch of one or 32
// 68 x 68 matrices takes 30 us, 0.4 us per column.  The walks shrink with the column index at compile time (rows above the diagonal are not touched).
// Two things keep A orthogonal: inv is 2 / u^T u of the u in LDS (I - inv u u^T is then a reflection whatever rounding the
// norm carries; with 1 / (norm (norm + |top|)) by the bare hardware reciprocal each step stretched its direction by up to
// three roundings), and the product walks upward, so that u's large top entry is added last instead of lifting every
// partial sum.  A^T A - I, rms over 96 draws: 7 to 8% less than with a thread per column at 36 to 128 rows (4 to 6% at 16 to 33), where
// without the two it was 2 to 7% more; R = A^T G below the diagonal 2% less to 1% more (4 to 9% more without).  Cost: 0.3 of
// 38 us at 68 rows, 2 of 58 at 100.
// On return the columns c >= n hold Q^T (thread (n + i, q): Q[i][q + 4 t] in x[t]) and sh.rdiag the diagonal of R.
template <int NR>
__device__ __forceinline__ void small_householder(float (&x)[NR], int n, SmallQrShared<NR>& sh) {
    typedef float f32x4_t __attribute__((ext_vector_type(4)));
    const int c = threadIdx.x >> 2, q = threadIdx.x & 3;
    // column j = 4 JB + qj becomes reflector j: only its own quad comes here
    auto publish = [&](auto JBc, int qj) {
        constexpr int JB = decltype(JBc)::value;
        const int j = 4 * JB + qj, buf = j & 1;
        const float top = x[JB];
        float s0 = q > qj ? top * top : 0.f, s1 = 0.f;
#pragma unroll
        for (int i = JB + 1; i < NR; ++i) { if (i & 1) s1 = fmaf(x[i], x[i], s1); else s0 = fmaf(x[i], x[i], s0); }
        const float nn = quad_sum(s0 + s1);                              // square of the column below row j
        const float nrm = __builtin_amdgcn_sqrtf(fmaf(top, top, nn));    // hardware root and reciprocal (1 ulp)
        const float ut = q > qj ? top : (q == qj ? top + copysignf(nrm, top) : 0.f);
#pragma unroll
        for (int i = JB / 4 * 4; i < NR; i += 4) {
            f32x4_t v;
#pragma unroll
            for (int t = 0; t < 4; ++t) v[t] = i + t >= NR ? 0.f : (i + t == JB ? ut : x[i + t < NR ? i + t : 0]);
            *reinterpret_cast<f32x4_t*>(&sh.u[buf][q][i]) = v;
        }
        if (q == qj) {
            // a column that is zero below the diagonal needs no reflector; otherwise 2 / u^T u, of the u that was published
            const float uu = fmaf(ut, ut, nn), r = __builtin_amdgcn_rcpf(uu);
            sh.inv[buf] = nn > 0.f ? 2.f * fmaf(fmaf(-uu, r, 1.f), r, r) : 0.f;
            sh.rdiag[j] = nn > 0.f ? -copysignf(nrm, top) : top;
        }
    };
    if (c == 0) publish(std::integral_constant<int, 0>{}, 0);
    static_for<NR>([&](auto JBc) {
        constexpr int JB = decltype(JBc)::value;
#pragma unroll 1
        for (int qj = 0; qj < 4; ++qj) {
            const int j = 4 * JB + qj;
            if (j >= n) break;
            __syncthreads();
            if (c > j && c < 2 * n) {
                const int buf = j & 1;
                constexpr int I0 = JB / 4 * 4;
                float u[SmallQrShared<NR>::SEG - I0];
#pragma unroll
                for (int i = I0; i < NR; i += 4) {
                    const f32x4_t v = *reinterpret_cast<const f32x4_t*>(&sh.u[buf][q][i]);
#pragma unroll
                    for (int t = 0; t < 4; ++t) u[i - I0 + t] = v[t];
                }
                const float inv = sh.inv[buf];
                float d0 = 0.f, d1 = 0.f;
#pragma unroll
                for (int i = NR - 1; i >= JB; --i) { if (i & 1) d1 = fmaf(u[i - I0], x[i], d1); else d0 = fmaf(u[i - I0], x[i], d0); }
                const float f = -inv * quad_sum(d0 + d1);
#pragma unroll
                for (int i = JB; i < NR; ++i) x[i] = fmaf(f, u[i - I0], x[i]);
                if (c == j + 1 && c < n) {
                    if (qj < 3) publish(std::integral_constant<int, JB>{}, qj + 1);
                    else if constexpr (JB + 1 < NR) publish(std::integral_constant<int, JB + 1>{}, 0);
                }
            }
        }
    });
    __syncthreads();
}

}  // namespace gelo

// The explicit inverse and the kappa_2 estimate (Lanczos) behind the non-orthogonal mixing matrices (Section 3.2.1,
// Mitigation 1: a well-conditioned non-orthogonal A, generated and verified; Section 3.2 eq. 3 needs A^-1 explicitly so
// that un-mixing is one GEMM).  Everything is deterministic: reductions run in a fixed order, no atomics.
//
// CONDITIONED beyond 128 rows: Newton's iteration from the orthogonal part's transpose, on bf16 products with float sums, the last residual
// from all 24 bits of A (inverse_near_orthogonal).  Otherwise, and in the condition estimate, everything is float (the refinement of up to 128 rows double):
// A^-1 = R^-1 Q^T from the Householder QR of A (factor.hip): no pivot searches and row interchanges, whose chain - two
// barriers per column, 1.1 us of one workgroup - bounded a row-pivoted LU in this place (512 rows: 1.1 ms of kernels
// without the condition estimate, here 0.48; 4096 rows: 15.5 ms, here 4.9).  Up to 128 rows everything behind the QR is one
// launch (small_inverse_kernel).  Beyond, Q^T is the right-hand side of a block back substitution with R: the inverses of
// R's 128 x 128 diagonal blocks come from one launch, everything else is float GEMMs with K = 128.  The QR needs no pivots
// for its accuracy, whatever A is, except that its panels are built from Gram matrices (gram_panel_body, block_core_kernel): a panel's
// condition number is at most A's, times a panel of Gaussians' for the GAUSSIAN kind.
#include "gelo_internal.h"
#include "wave_tile.h"

namespace gelo {
namespace {

constexpr int NB = kPanel;
constexpr int BW = kInvBlock;
constexpr int TB = BW / NB;                               // tiles across a diagonal block
constexpr int TP = NB + 4;                                // LDS pitch of a row-major tile, floats
typedef float f32x4_t __attribute__((ext_vector_type(4)));
typedef double f64x4_t __attribute__((ext_vector_type(4)));

__device__ __forceinline__ float wave_sum(float v) {
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off, 64);
    return v;
}

// ------------------------------------------------ inverses of R's diagonal blocks --
// One workgroup per 128 x 128 diagonal block of R (upper triangular; tiles above the diagonal in M, diagonal tiles in Rd;
// the identity beyond n).  The 16 x 16 diagonal tiles are inverted by back substitution, one thread per column; then
// twice the size at a time: [A B; 0 C]^-1 = [A^-1, -A^-1 B C^-1; 0, C^-1].  Dinv: row-major, pitch BW, zeros below the diagonal.
constexpr int IP = BW + 4;                                // LDS pitch, floats
constexpr size_t kDiagLds = 2 * (size_t)BW * IP * sizeof(float);

__global__ __launch_bounds__(512)
void diag_inverse_kernel(const float* M, const float* Rd, float* Dinv, int nbr, int n, int* flag) {
    extern __shared__ __attribute__((aligned(16))) float diag_lds[];
    float* U = diag_lds;
    float* I = diag_lds + BW * IP;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int t0 = blockIdx.x * TB;                       // the block's first tile
    for (int t = wave; t < TB * TB; t += 8) {
        const int i = t / TB, j = t % TB;                 // tile (i, j) of the block
        if (j < i) continue;
        const int c = lane & 15, g = lane >> 4;
        if (i < j) {
            f32x4_t v = {0.f, 0.f, 0.f, 0.f};
            if (t0 + j < nbr) v = *reinterpret_cast<const f32x4_t*>(M + ((int64_t)(t0 + j) * nbr + t0 + i) * 256 + c * 16 + 4 * g);
#pragma unroll
            for (int e = 0; e < 4; ++e) U[(i * NB + 4 * g + e) * IP + j * NB + c] = v[e];
        } else {
            const int r = lane >> 2, q = (lane & 3) * 4;
            f32x4_t v = {0.f, 0.f, 0.f, 0.f};
            if (t0 + i < nbr) v = *reinterpret_cast<const f32x4_t*>(Rd + (int64_t)(t0 + i) * 256 + r * NB + q);
#pragma unroll
            for (int e = 0; e < 4; ++e) if ((t0 + i) * NB + r >= n) v[e] = q + e == r ? 1.f : 0.f;
            *reinterpret_cast<f32x4_t*>(&U[(i * NB + r) * IP + j * NB + q]) = v;
        }
    }
    __syncthreads();
    if (tid < BW) {
        const int o = tid & ~15, j = tid & 15;
        float x[NB];
#pragma unroll
        for (int i = NB - 1; i >= 0; --i) {
            float t = i == j ? 1.f : 0.f;
#pragma unroll
            for (int k = i + 1; k < NB; ++k) t = fmaf(-U[(o + i) * IP + o + k], x[k], t);
            const float u = U[(o + i) * IP + o + i];
            if (i == j && !(fabsf(u) > 0.f)) *flag = 1;
            x[i] = t / u;
        }
#pragma unroll
        for (int i = 0; i < NB; ++i) I[(o + i) * IP + o + j] = x[i];
    }
    __syncthreads();
    // a thread owns 8 rows of one column; B C^-1 waits in the unused lower triangle
    for (int s = NB; s < BW; s *= 2) {
        const int outs = BW * s / 16;                     // (BW / 2 s) pairs x s columns x s / 8 row groups
        const int c = tid % s, r0 = tid / s % (s / 8) * 8, o1 = tid / (s * s / 8) * 2 * s, o2 = o1 + s;
        float acc[8];
#pragma unroll
        for (int i = 0; i < 8; ++i) acc[i] = 0.f;
        if (tid < outs) {
            for (int k = 0; k < s; k += 4) {
                float x[4];
#pragma unroll
                for (int e = 0; e < 4; ++e) { const float y = I[(o2 + k + e) * IP + o2 + c]; x[e] = k + e <= c ? y : 0.f; }
#pragma unroll
                for (int i = 0; i < 8; ++i) {
                    const f32x4_t a = *reinterpret_cast<const f32x4_t*>(&U[(o1 + r0 + i) * IP + o2 + k]);
#pragma unroll
                    for (int e = 0; e < 4; ++e) acc[i] = fmaf(a[e], x[e], acc[i]);
                }
            }
#pragma unroll
            for (int i = 0; i < 8; ++i) I[(o2 + r0 + i) * IP + o1 + c] = acc[i];
        }
        __syncthreads();
        if (tid < outs) {
#pragma unroll
            for (int i = 0; i < 8; ++i) acc[i] = 0.f;
            for (int k = 0; k < s; k += 4) {
                float x[4];
#pragma unroll
                for (int e = 0; e < 4; ++e) x[e] = I[(o2 + k + e) * IP + o1 + c];
#pragma unroll
                for (int i = 0; i < 8; ++i) {
                    const f32x4_t a = *reinterpret_cast<const f32x4_t*>(&I[(o1 + r0 + i) * IP + o1 + k]);
#pragma unroll
                    for (int e = 0; e < 4; ++e) acc[i] = fmaf(k + e >= r0 + i ? a[e] : 0.f, x[e], acc[i]);
                }
            }
#pragma unroll
            for (int i = 0; i < 8; ++i) I[(o1 + r0 + i) * IP + o2 + c] = -acc[i];
        }
        __syncthreads();
    }
    for (int id = tid; id < BW * BW; id += 512) {
        const int r = id / BW, c = id % BW;
        if (t0 * NB + r < nbr * NB) Dinv[((int64_t)t0 * NB + r) * BW + c] = c >= r ? I[r * IP + c] : 0.f;
    }
}

// ------------------------------------------------ the inverse of a matrix of at most 128 rows --
// One launch, a workgroup per 16 columns of A^-1: X = R^-1 (Q^T)'s columns by back substitution over 16 x 16 tiles, then one
// step of iterative refinement, X += R^-1 Q^T (I - A X) with the residual in double precision, and the rows go out in both
// types.  Everything a workgroup needs of the other columns is in A, Q and R, so the workgroups are independent.
// The products keep the accumulator layout throughout: what the matrix instructions leave in a lane (column c, rows 4 g ..)
// is what they take as right operand when instruction e contracts the rows 4 g + e.
// Bound by latency: a chain of at most 8 tile rows, twice; the other waves only load and form residuals.  Without the
// refinement R^-1 Q^T is further off than a row-pivoted LU's inverse up to 40 rows (geometric means over 48 matrices: GAUSSIAN 16 rows,
// |A^-1 A - I| 2.2 times, H recovered from A H 1.9 times as far off, CONDITIONED 8 rows 1.7 and 1.5 times), and with R^-1 as a
// GEMM operand it takes seven launches.  With it, against the LU: |A^-1 A - I| 0.19 and 0.23, H recovered 0.57 and 0.59, at
// 128 rows 0.04 and 0.31 (GAUSSIAN).  CONDITIONED draw (LU, seven launches, one): 16 rows 246, 236, 204 us; 64 rows 383, 366, 334;
// 128 rows 545, 466, 458.

__global__ __launch_bounds__(256)
void small_inverse_kernel(const float* M, const float* Rd, const float* Q, const float* A, int nbr, int n, int64_t ldk,
                          float* dst32, uint16_t* dst16, int* flag) {
    __shared__ __attribute__((aligned(16))) float Rt[TB * (TB + 1) / 2][NB * TP];   // R's tiles (t, s), t <= s, at s (s + 1) / 2 + t
    __shared__ __attribute__((aligned(16))) float Di[TB][NB * TP];                  // inverses of the diagonal ones
    __shared__ __attribute__((aligned(16))) float Xs[TB][64][4];                    // X, later the refinement's right-hand side
    __shared__ __attribute__((aligned(16))) float Es[TB][NB * NB];                  // I - A X, column by column
    __shared__ int singular, far;
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int c = lane & 15, g = lane >> 4, cb = blockIdx.x;
    if (tid == 0) { singular = 0; far = 0; }
    for (int s = wave; s < nbr; s += 4)
        for (int t = 0; t <= s; ++t) {
            float* tile = Rt[s * (s + 1) / 2 + t];
            if (t < s) {
                const f32x4_t v = *reinterpret_cast<const f32x4_t*>(M + ((int64_t)s * nbr + t) * 256 + c * 16 + 4 * g);
#pragma unroll
                for (int e = 0; e < 4; ++e) tile[(4 * g + e) * TP + c] = v[e];
            } else {                                      // row-major in Rd; the identity beyond n
                const int r = lane >> 2, q = (lane & 3) * 4;
                f32x4_t v = *reinterpret_cast<const f32x4_t*>(Rd + (int64_t)t * 256 + r * NB + q);
#pragma unroll
                for (int e = 0; e < 4; ++e) if (t * NB + r >= n) v[e] = q + e == r ? 1.f : 0.f;
                *reinterpret_cast<f32x4_t*>(&tile[r * TP + q]) = v;
            }
        }
    __syncthreads();
    if (tid < nbr * NB) {                                 // back substitution in a diagonal tile, a thread per column
        const int o = tid / NB, j = tid % NB;
        const float* U = Rt[o * (o + 1) / 2 + o];
        float x[NB];
#pragma unroll
        for (int i = NB - 1; i >= 0; --i) {
            float t = i == j ? 1.f : 0.f;
#pragma unroll
            for (int k = i + 1; k < NB; ++k) t = fmaf(-U[i * TP + k], x[k], t);
            const float u = U[i * TP + i];
            if (i == j && !(fabsf(u) > 0.f)) singular = 1;
            x[i] = t / u;
        }
#pragma unroll
        for (int i = 0; i < NB; ++i) Di[o][i * TP + j] = x[i];
    }
    __syncthreads();
    if (tid == 0 && cb == 0) *flag = singular;
    // b <- R^-1 b (wave 0)
    auto row_operand = [&](const float* tile) { return *reinterpret_cast<const f32x4_t*>(tile + c * TP + 4 * g); };
    auto solve = [&](f32x4_t (&b)[TB]) {
#pragma unroll
        for (int s = TB - 1; s >= 0; --s) {
            if (s >= nbr) continue;
            const f32x4_t d = row_operand(Di[s]);
            f32x4_t x = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int e = 0; e < 4; ++e) x = __builtin_amdgcn_mfma_f32_16x16x4f32(d[e], b[s][e], x, 0, 0, 0);
            b[s] = x;
#pragma unroll
            for (int t = s - 1; t >= 0; --t) {
                const f32x4_t r = row_operand(Rt[s * (s + 1) / 2 + t]);
#pragma unroll
                for (int e = 0; e < 4; ++e) b[t] = __builtin_amdgcn_mfma_f32_16x16x4f32(-r[e], x[e], b[t], 0, 0, 0);
            }
        }
    };
    f32x4_t X[TB];
    if (wave == 0) {
#pragma unroll
        for (int t = 0; t < TB; ++t) {
            X[t] = f32x4_t{0.f, 0.f, 0.f, 0.f};
            if (t >= nbr) continue;
#pragma unroll
            for (int e = 0; e < 4; ++e) X[t][e] = Q[((int64_t)t * nbr + cb) * 256 + (4 * g + e) * 16 + c];     // Q^T[4 g + e][c]
        }
        solve(X);
#pragma unroll
        for (int t = 0; t < TB; ++t) if (t < nbr) *reinterpret_cast<f32x4_t*>(Xs[t][lane]) = X[t];
    }
    __syncthreads();
    // I - A X in double precision (its instruction leaves row 4 v + g of column c in element v)
    bool big = false;
    for (int t = wave; t < nbr; t += 4) {
        f64x4_t acc;
#pragma unroll
        for (int v = 0; v < 4; ++v) acc[v] = t == cb && 4 * v + g == c && t * NB + c < n ? 1. : 0.;
        const int row = t * NB + c;
        for (int s = 0; s < nbr; ++s) {
            f32x4_t a = {0.f, 0.f, 0.f, 0.f};
            if (row < n) a = *reinterpret_cast<const f32x4_t*>(A + (int64_t)row * ldk + s * NB + 4 * g);
            const f32x4_t x = *reinterpret_cast<const f32x4_t*>(Xs[s][lane]);
#pragma unroll
            for (int e = 0; e < 4; ++e) acc = __builtin_amdgcn_mfma_f64_16x16x4f64(-(double)a[e], (double)x[e], acc, 0, 0, 0);
        }
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            const float e = (float)acc[v];
            big = big || !(fabsf(e) < 0.1f);
            Es[t][c * NB + 4 * v + g] = e;
        }
    }
    if (big) far = 1;
    __syncthreads();
    // A correction is taken from a residual that is small: beyond that X is a first approximation of nothing (condition
    // numbers around 1e6 and more, NaN), and stays as it is
    if (far == 0) {                                       // the same for the whole workgroup
        for (int t = wave; t < nbr; t += 4) {
            f32x4_t y = {0.f, 0.f, 0.f, 0.f};
            for (int s = 0; s < nbr; ++s) {
                const f32x4_t q = *reinterpret_cast<const f32x4_t*>(Q + ((int64_t)t * nbr + s) * 256 + c * 16 + 4 * g);    // Q^T[c][4 g ..]
                const f32x4_t r = *reinterpret_cast<const f32x4_t*>(&Es[s][c * NB + 4 * g]);
#pragma unroll
                for (int e = 0; e < 4; ++e) y = __builtin_amdgcn_mfma_f32_16x16x4f32(q[e], r[e], y, 0, 0, 0);
            }
            *reinterpret_cast<f32x4_t*>(Xs[t][lane]) = y;
        }
        __syncthreads();
        if (wave == 0) {
            f32x4_t y[TB];
#pragma unroll
            for (int t = 0; t < TB; ++t) { y[t] = f32x4_t{0.f, 0.f, 0.f, 0.f}; if (t < nbr) y[t] = *reinterpret_cast<const f32x4_t*>(Xs[t][lane]); }
            solve(y);
#pragma unroll
            for (int t = 0; t < TB; ++t) if (t < nbr) *reinterpret_cast<f32x4_t*>(Xs[t][lane]) = X[t] + y[t];
        }
        __syncthreads();
    }
    // rows of A^-1, zero beyond column n; the last workgroup also writes the columns beyond its own
    const int quads = cb + 1 < nbr ? NB / 4 : (int)(ldk - (int64_t)cb * NB) / 4;
    for (int i = tid; i < n * quads; i += 256) {
        const int r = i / quads, q = (i - r * quads) * 4;
        f32x4_t v = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int e = 0; e < 4; ++e) if (q + e < NB && cb * NB + q + e < n) v[e] = Xs[r / NB][(r % NB) / 4 * 16 + q + e][r % 4];
        const int64_t at = (int64_t)r * ldk + cb * NB + q;
        *reinterpret_cast<f32x4_t*>(dst32 + at) = v;
        if (dst16) {
            typedef __bf16 bf16x4_t __attribute__((ext_vector_type(4)));
            const bf16x4_t h = {(__bf16)v[0], (__bf16)v[1], (__bf16)v[2], (__bf16)v[3]};
            *reinterpret_cast<uint2*>(dst16 + at) = __builtin_bit_cast(uint2, h);
        }
    }
}

// ------------------------------------------------ the inverse of an orthogonal matrix and a perturbation --
// A taken apart into three bf16 matrices h + m + l (split_float.h), pitch ld like A.  ld / 4 quads per row, zero beyond column n as A is.
__global__ __launch_bounds__(256)
void planes_kernel(const float* A, int64_t quads, uint16_t* h, uint16_t* m, uint16_t* l) {
    typedef __bf16 bf16x4_t __attribute__((ext_vector_type(4)));
    const int64_t q = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (q >= quads) return;
    const f32x4_t x = *reinterpret_cast<const f32x4_t*>(A + 4 * q);
    bf16x4_t vh, vm, vl;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        vh[e] = (__bf16)x[e];
        const float r = x[e] - (float)vh[e];
        vm[e] = (__bf16)r;
        vl[e] = (__bf16)(r - (float)vm[e]);
    }
    *reinterpret_cast<uint2*>(h + 4 * q) = __builtin_bit_cast(uint2, vh);
    *reinterpret_cast<uint2*>(m + 4 * q) = __builtin_bit_cast(uint2, vm);
    *reinterpret_cast<uint2*>(l + 4 * q) = __builtin_bit_cast(uint2, vl);
}

// ------------------------------------------------------------------ Lanczos --
// sigma_max of a matrix M from a few steps of the Lanczos recurrence on M^T M (no
// reorthogonalisation: the largest Ritz value converges first and never overshoots).  The two
// operators the condition number needs, A and A^-1, share every launch.
constexpr int kLanczosMax = 32;      // coefficient slots per operator

template <int WAVES>
__device__ __forceinline__ float block_sum(float v, float* red) {       // the same value in every thread, fixed order
    v = wave_sum(v);
    __syncthreads();                                   // red may still be read from the previous call
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = v;
    __syncthreads();
    float s = 0.f;
#pragma unroll
    for (int w = 0; w < WAVES; ++w) s += red[w];
    return s;
}

// Vector `step` of the recurrence, OWN elements per thread (threadIdx.x, + 64 WAVES, ...), by every workgroup of a launch for itself (all the same
// bits): for step 0 a fixed pseudo-random unit vector, else from x = w = M^T (M v) of vector v, step - 1,
//   alpha = w . v, r = w - alpha v - beta_prev v_prev, beta = |r|, x = r / beta; tr[0][step - 1] = alpha, tr[1][step - 1] = beta.
// Vector j lies in slot j % 3, where the caller's first workgroup (`writes`) keeps it: nobody writes what others of the launch still read.
// `before`: the two vectors ahead of it, asked for before x is formed.
template <int OWN, int WAVES>
struct LanczosBefore {
    float v[OWN], v_prev[OWN], beta;
    __device__ __forceinline__ LanczosBefore(const float* slots, int64_t ld, int n, const float* tr, int step) {
        const float* p = slots + (int64_t)((step + 2) % 3) * ld;             // vector step - 1
        const float* q = slots + (int64_t)((step + 1) % 3) * ld;             // vector step - 2
#pragma unroll
        for (int k = 0; k < OWN; ++k) {
            const int i = threadIdx.x + 64 * WAVES * k;
            v[k] = i < n && step > 0 ? p[i] : 0.f;
            v_prev[k] = i < n && step > 1 ? q[i] : 0.f;
        }
        beta = step > 1 ? tr[kLanczosMax + step - 2] : 0.f;
    }
};
template <int OWN, int WAVES>
__device__ __forceinline__ void next_vector(float (&x)[OWN], const LanczosBefore<OWN, WAVES>& before, int n, float* tr, int step, bool writes, float* red) {
    constexpr int THREADS = 64 * WAVES;
    const int tid = threadIdx.x;
    if (step == 0) {
        float ss = 0.f;
#pragma unroll
        for (int k = 0; k < OWN; ++k) {
            const int i = tid + THREADS * k;
            uint32_t h = (uint32_t)i * 2654435761u + 0x9E3779B9u;   // fixed pseudo-random signs and sizes
            h ^= h >> 15; h *= 2246822519u; h ^= h >> 13;
            x[k] = i < n ? ((h & 1u) ? 1.f : -1.f) * (0.5f + (float)((h >> 8) & 0xFFFF) * (1.0f / 65536.0f)) : 0.f;
            ss = fmaf(x[k], x[k], ss);
        }
        const float inv = rsqrtf(block_sum<WAVES>(ss, red));
#pragma unroll
        for (int k = 0; k < OWN; ++k) x[k] *= inv;
        return;
    }
    float dot = 0.f;
#pragma unroll
    for (int k = 0; k < OWN; ++k) dot = fmaf(x[k], before.v[k], dot);
    const float alpha = block_sum<WAVES>(dot, red);
    float ss = 0.f;
#pragma unroll
    for (int k = 0; k < OWN; ++k) {
        x[k] = fmaf(-before.beta, before.v_prev[k], fmaf(-alpha, before.v[k], x[k]));
        ss = fmaf(x[k], x[k], ss);
    }
    const float beta = sqrtf(block_sum<WAVES>(ss, red));
    const float inv = beta > 0.f ? 1.0f / beta : 0.f;
#pragma unroll
    for (int k = 0; k < OWN; ++k) x[k] *= inv;
    if (writes && tid == 0) { tr[step - 1] = alpha; tr[kLanczosMax + step - 1] = beta; }
}

// M^T (M v) for M = A (grid y 0) and A^-1 (1), every row read once: a wave holds a row in registers, takes its product with v and adds
// that many times the row to its sum; the workgroup's sum goes to part[workgroup][ld].  The vector itself is formed first, by every workgroup.  CH: blocks of 256 columns (n <= 256 CH).
// Bound by the last-level cache: 4 n^2 bytes per operator.  With a product by rows of M and one by rows of a transposed copy
// (8 n^2, and more than the 256 MB the cache holds at 4096 rows) a Lanczos step took 62 us at 4096 rows, now 36; the whole
// condition estimate 1.32 ms, then 0.74; with the vector formed here instead of in a launch of its own between the products a draw of 1025 rows
// went from 1120 to 1060 us, of 4096 from 5819 to 5718.
constexpr int kProductGroups = 128;                    // workgroups per operator

template <int CH>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(1, 2)))
void normal_product_kernel(const float* Ma, const float* Mb, float* pa, float* pb, int64_t w_at, float* vec, int64_t lda, int64_t ld, int n, float* tri, int step, int steps) {
    __shared__ __attribute__((aligned(16))) float vs[CH * 256];
    __shared__ float red[4];
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const float* M = blockIdx.y ? Mb : Ma;
    const float* w = (blockIdx.y ? pb : pa) + w_at;
    float* slots = vec + (int64_t)blockIdx.y * 3 * ld;
    float* part = (blockIdx.y ? pb : pa) + (int64_t)blockIdx.x * ld;
    float* tr = tri + blockIdx.y * 2 * kLanczosMax;
    const LanczosBefore<CH, 4> before(slots, ld, n, tr, step);
    float v[CH];
#pragma unroll
    for (int k = 0; k < CH; ++k) v[k] = step > 0 && tid + 256 * k < n ? w[tid + 256 * k] : 0.f;
    next_vector<CH, 4>(v, before, n, tr, step, blockIdx.x == 0, red);
    if (step == steps) return;
#pragma unroll
    for (int k = 0; k < CH; ++k) {
        vs[tid + 256 * k] = v[k];
        if (blockIdx.x == 0 && tid + 256 * k < n) slots[(int64_t)(step % 3) * ld + tid + 256 * k] = v[k];
    }
    __syncthreads();
    f32x4_t sum[CH];
#pragma unroll
    for (int j = 0; j < CH; ++j) sum[j] = f32x4_t{0.f, 0.f, 0.f, 0.f};
    for (int r = blockIdx.x * 4 + wave; r < n; r += gridDim.x * 4) {
        const float* row = M + (int64_t)r * lda;
        f32x4_t x[CH];
#pragma unroll
        for (int j = 0; j < CH; ++j) {
            const int c = j * 256 + lane * 4;          // (beyond its end the row's start again: v is zero there and nobody reads the sums)
            x[j] = *reinterpret_cast<const f32x4_t*>(row + (c < lda ? c : 0));
        }
        float dot = 0.f;
#pragma unroll
        for (int j = 0; j < CH; ++j) {
            const f32x4_t y = *reinterpret_cast<const f32x4_t*>(&vs[j * 256 + lane * 4]);
#pragma unroll
            for (int e = 0; e < 4; ++e) dot = fmaf(x[j][e], y[e], dot);
        }
        dot = wave_sum(dot);
#pragma unroll
        for (int j = 0; j < CH; ++j)
#pragma unroll
            for (int e = 0; e < 4; ++e) sum[j][e] = fmaf(dot, x[j][e], sum[j][e]);
    }
    for (int w = 0; w < 4; ++w) {                      // the waves' sums, one after the other
        __syncthreads();
        if (wave == w) {
#pragma unroll
            for (int j = 0; j < CH; ++j) {
                f32x4_t* at = reinterpret_cast<f32x4_t*>(&vs[j * 256 + lane * 4]);
                *at = w == 0 ? sum[j] : *at + sum[j];
            }
        }
    }
    __syncthreads();
    for (int c = tid; c < n; c += 256) part[c] = vs[c];
}

// w[c] = sum of the workgroups' parts, in a fixed order
__global__ __launch_bounds__(256)
void sum_parts_kernel(const float* pa, float* wa, const float* pb, float* wb, int64_t ld, int n, int parts) {
    __shared__ float red[4][64];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, c = blockIdx.x * 64 + lane;
    const float* p = (blockIdx.y ? pb : pa) + (c < n ? c : n - 1);
    const int per = (parts + 3) / 4, end = (wave + 1) * per < parts ? (wave + 1) * per : parts;
    float s = 0.f;
#pragma unroll 8
    for (int i = wave * per; i < end; ++i) s += p[(int64_t)i * ld];
    red[wave][lane] = s;
    __syncthreads();
    if (wave == 0 && c < n) (blockIdx.y ? wb : wa)[c] = ((red[0][lane] + red[1][lane]) + red[2][lane]) + red[3][lane];
}

// The same steps with one launch each, for small matrices: every workgroup forms the sum of the parts and the next vector itself (all the
// same bits) before its rows of the product.  Launch j < steps leaves the parts of product j, launch `steps` the last coefficients; vector
// j lies in slot j % 3, the parts of even and odd products in either half, so that nobody writes what others of the launch still read.
// Bound by latency, a read of the parts, one of the rows and two sums over the workgroup: 5.3 us per step at 512 rows, where three launches
// took 3.7 + 4.0 + 3.4 and the gaps between them.  Draw, us: CONDITIONED 64 rows 330 -> 258, 129 404 -> 315, 512 714 -> 632, 1024 1068 -> 990;
// GAUSSIAN (one attempt) 512 728 -> 632, 1024 1083 -> 1006.  With 256 threads, the parts summed by one thread per column: 678 and 1098.  The parts that
// every workgroup reads (32 rows) grow with n, the rows of few workgroups with n^2: beyond 1024 rows the launches stay apart.
constexpr int kFusedGroups = 32;                       // workgroups per operator, at most
constexpr int kFusedMaxN = 1024;

constexpr int kFusedWaves = 8, kFusedThreads = 64 * kFusedWaves;

template <int CH>
__global__ __launch_bounds__(kFusedThreads) __attribute__((amdgpu_waves_per_eu(2, 2)))
void lanczos_step_kernel(const float* Ma, const float* Mb, float* pa, float* pb, float* vec, int64_t lda, int64_t ld, int n, float* tri, int step, int steps,
                         int groups) {
    constexpr int COLS = CH * 256, QUADS = COLS / 4;
    constexpr int SETS = kFusedThreads / QUADS;        // of parts: each is added up by QUADS threads
    constexpr int PER = kFusedGroups / SETS;
    constexpr int OWN = (COLS + kFusedThreads - 1) / kFusedThreads;      // elements of the vector per thread
    constexpr int RB = 4;                              // rows whose reads are on their way together
    __shared__ __attribute__((aligned(16))) float vs[COLS];
    __shared__ __attribute__((aligned(16))) float sums[kFusedWaves][COLS];
    __shared__ float red[kFusedWaves];
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6), o = blockIdx.y;
    const float* M = o ? Mb : Ma;
    float* parts = o ? pb : pa;
    float* slots = vec + (int64_t)o * 3 * ld;
    float* tr = tri + o * 2 * kLanczosMax;
    const LanczosBefore<OWN, kFusedWaves> before(slots, ld, n, tr, step);
    float x[OWN];
    if (step > 0) {
        const float* last = parts + (int64_t)((step - 1) & 1) * groups * ld;
        {
            const int q = tid % QUADS, set = tid / QUADS;
            const int at = 4 * q < (int)ld ? 4 * q : 0;
            f32x4_t p[PER], s = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int i = 0; i < PER; ++i) p[i] = *reinterpret_cast<const f32x4_t*>(last + (int64_t)(set * PER + i < groups ? set * PER + i : 0) * ld + at);
#pragma unroll
            for (int i = 0; i < PER; ++i)
#pragma unroll
                for (int e = 0; e < 4; ++e) s[e] += set * PER + i < groups ? p[i][e] : 0.f;
            *reinterpret_cast<f32x4_t*>(&sums[set][4 * q]) = s;
        }
        __syncthreads();
#pragma unroll
        for (int k = 0; k < OWN; ++k) {
            const int i = tid + kFusedThreads * k;
            x[k] = 0.f;
            if (i < n) {
#pragma unroll
                for (int t = 0; t < SETS; ++t) x[k] += sums[t][i];
            }
        }
    }
    next_vector<OWN, kFusedWaves>(x, before, n, tr, step, blockIdx.x == 0, red);
    if (step == steps) return;
#pragma unroll
    for (int k = 0; k < OWN; ++k) {
        const int i = tid + kFusedThreads * k;
        if (i < COLS) vs[i] = x[k];
        if (blockIdx.x == 0 && i < n) slots[(int64_t)(step % 3) * ld + i] = x[k];
    }
    __syncthreads();
    f32x4_t sum[CH];
#pragma unroll
    for (int j = 0; j < CH; ++j) sum[j] = f32x4_t{0.f, 0.f, 0.f, 0.f};
    const int stride = groups * kFusedWaves;
    for (int r0 = blockIdx.x * kFusedWaves + wave; r0 < n; r0 += RB * stride) {
        f32x4_t m[RB][CH];
#pragma unroll
        for (int b = 0; b < RB; ++b) {
            const int r = r0 + b * stride;
            const float* row = M + (int64_t)(r < n ? r : r0) * lda;
#pragma unroll
            for (int j = 0; j < CH; ++j) {
                const int c = j * 256 + lane * 4;      // (beyond its end the row's start again, as in normal_product_kernel)
                m[b][j] = *reinterpret_cast<const f32x4_t*>(row + (c < lda ? c : 0));
            }
        }
#pragma unroll
        for (int b = 0; b < RB; ++b) {
            if (r0 + b * stride >= n) break;           // (the same for the whole wave)
            float dot = 0.f;
#pragma unroll
            for (int j = 0; j < CH; ++j) {
                const f32x4_t y = *reinterpret_cast<const f32x4_t*>(&vs[j * 256 + lane * 4]);
#pragma unroll
                for (int e = 0; e < 4; ++e) dot = fmaf(m[b][j][e], y[e], dot);
            }
            dot = wave_sum(dot);
#pragma unroll
            for (int j = 0; j < CH; ++j)
#pragma unroll
                for (int e = 0; e < 4; ++e) sum[j][e] = fmaf(dot, m[b][j][e], sum[j][e]);
        }
    }
#pragma unroll
    for (int j = 0; j < CH; ++j) *reinterpret_cast<f32x4_t*>(&sums[wave][j * 256 + lane * 4]) = sum[j];
    __syncthreads();
    float* part = parts + ((int64_t)(step & 1) * groups + blockIdx.x) * ld;
    for (int c = tid; c < n; c += kFusedThreads) {
        float s = 0.f;
#pragma unroll
        for (int w = 0; w < kFusedWaves; ++w) s += sums[w][c];
        part[c] = s;
    }
}

// Largest eigenvalue of the symmetric tridiagonal matrix (alpha[0..k), beta[0..k-1)) by sectioning on
// the Sturm count: one wave, lanes 0..31 work on A, lanes 32..63 on A^-1; each round every lane counts
// the eigenvalues below its own trial value (32 trial values per bracket), and the bracket shrinks to
// the interval between the last trial with an eigenvalue at or above it and the first one above all.
// out[0] = sqrt(lambda_A lambda_Ainv) = the kappa_2 estimate, out[1], out[2] its factors.
__device__ __forceinline__ void largest_ritz_values(const float* co, int k, float* out) {      // one wave; co: as tri
    const int lane = threadIdx.x & 63, o = lane >> 5, l = lane & 31;
    const float* al = co + o * 2 * kLanczosMax;
    const float* be = al + kLanczosMax;
    float hi = 0.f;
    for (int i = 0; i < k; ++i) {
        const float gsh = fabsf(al[i]) + (i > 0 ? fabsf(be[i - 1]) : 0.f) + (i + 1 < k ? fabsf(be[i]) : 0.f);
        hi = fmaxf(hi, gsh);
    }
    float lo = 0.f;
    for (int round = 0; round < 6; ++round) {
        const float step = (hi - lo) * (1.0f / 32.0f);
        const float x = lo + step * (float)(l + 1);        // l = 31: the current upper end
        int below = 0;                                     // eigenvalues below x
        float d = 1.f;
        for (int i = 0; i < k; ++i) {
            const float b2 = i > 0 ? be[i - 1] * be[i - 1] : 0.f;
            d = al[i] - x - b2 * __builtin_amdgcn_rcpf(d);
            if (fabsf(d) < 1e-30f) d = -1e-30f;
            below += d < 0.f;
        }
        const unsigned long long all = __ballot(below == k);
        const unsigned half = (unsigned)(all >> (32 * o));  // this operator's lanes
        const int first = half ? __ffs(half) - 1 : 31;      // first trial above every eigenvalue
        hi = lo + step * (float)(first + 1);
        lo = lo + step * (float)first;
    }
    const float sigma = sqrtf(0.5f * (lo + hi));
    const float s0 = __shfl(sigma, 0, 64), s1 = __shfl(sigma, 32, 64);
    if (lane == 0) { out[1] = s0; out[2] = s1; out[0] = s0 * s1; }
}
__global__ __launch_bounds__(64)
void lanczos_finish_kernel(const float* tri, int k, float* out) {
    __shared__ float co[2 * 2 * kLanczosMax];
    co[threadIdx.x] = tri[threadIdx.x]; co[threadIdx.x + 64] = tri[threadIdx.x + 64];
    __syncthreads();
    largest_ritz_values(co, k, out);
}

// The whole estimate of a matrix of at most 128 rows in one workgroup: eight waves for each operator, a wave with every eighth row in
// registers (two columns a lane) and the vectors too, every wave all of them (the same bits); the waves' sums of a product meet in LDS at one
// barrier per step.  Bound by that chain, about 0.9 us per step, where a launch per step takes 5.2.  Draw of a CONDITIONED matrix, us: 16 rows 135 -> 90,
// 64 rows 199 -> 149, 128 rows 289 -> 237; GAUSSIAN, 64 rows 400 -> 246.
__global__ __launch_bounds__(1024)
void small_kappa_kernel(const float* A, const float* Ainv, int64_t lda, int n, int steps, float* out) {
    __shared__ float parts[2][2][8][128];
    __shared__ float co[2 * 2 * kLanczosMax];
    const int lane = threadIdx.x & 63, number = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), o = number >> 3, wave = number & 7;
    const float* M = o ? Ainv : A;
    float* tr = co + o * 2 * kLanczosMax;
    constexpr int ROWS = 16;
    float m[ROWS][2], v[2], v_prev[2] = {0.f, 0.f}, beta = 0.f;
    auto total = [](float x) {                            // over the wave, the same in every lane
        x += dpp_mov<0x128>(x); x += dpp_mov<0x124>(x); x += dpp_mov<0x122>(x); x += dpp_mov<0x121>(x);      // row_ror 8, 4, 2, 1
        return sum_of_rows(x);
    };
#pragma unroll
    for (int i = 0; i < ROWS; ++i)
#pragma unroll
        for (int e = 0; e < 2; ++e) {
            const int r = wave + 8 * i, c = 2 * lane + e;
            m[i][e] = r < n && c < n ? M[(int64_t)r * lda + c] : 0.f;
        }
#pragma unroll
    for (int e = 0; e < 2; ++e) {                         // as next_vector's
        const int i = 2 * lane + e;
        uint32_t h = (uint32_t)i * 2654435761u + 0x9E3779B9u;
        h ^= h >> 15; h *= 2246822519u; h ^= h >> 13;
        v[e] = i < n ? ((h & 1u) ? 1.f : -1.f) * (0.5f + (float)((h >> 8) & 0xFFFF) * (1.0f / 65536.0f)) : 0.f;
    }
    {
        const float inv = rsqrtf(total(fmaf(v[0], v[0], v[1] * v[1])));
        v[0] *= inv; v[1] *= inv;
    }
    for (int step = 0; step < steps; ++step) {
        float t[ROWS];
#pragma unroll
        for (int i = 0; i < ROWS; ++i) t[i] = fmaf(m[i][0], v[0], m[i][1] * v[1]);
        const float dots = wave_reduce16(t, lane);
        float s0 = 0.f, s1 = 0.f;
        static_for<ROWS>([&](auto ic) {
            constexpr int i = decltype(ic)::value;
            const float d = lane_value<(i >> 3 & 1) * 4 + (i >> 2 & 1) * 8 + (i & 3)>(dots);      // reduce16_slot's inverse
            s0 = fmaf(d, m[i][0], s0); s1 = fmaf(d, m[i][1], s1);
        });
        *reinterpret_cast<float2*>(&parts[step & 1][o][wave][2 * lane]) = make_float2(s0, s1);
        __syncthreads();
        float w[2] = {0.f, 0.f};
#pragma unroll
        for (int k = 0; k < 8; ++k) {
            const float2 p = *reinterpret_cast<const float2*>(&parts[step & 1][o][k][2 * lane]);
            w[0] += p.x; w[1] += p.y;
        }
        const float alpha = total(fmaf(w[0], v[0], w[1] * v[1]));
#pragma unroll
        for (int e = 0; e < 2; ++e) {
            w[e] = fmaf(-beta, v_prev[e], fmaf(-alpha, v[e], w[e]));
            v_prev[e] = v[e];
        }
        beta = sqrtf(total(fmaf(w[0], w[0], w[1] * w[1])));
        const float inv = beta > 0.f ? 1.0f / beta : 0.f;
        v[0] = w[0] * inv; v[1] = w[1] * inv;
        if (wave == 0 && lane == 0) { tr[step] = alpha; tr[kLanczosMax + step] = beta; }
    }
    __syncthreads();
    if (number == 0) largest_ritz_values(co, steps, out);
}

#define GELO_TRY(expr) do { hipError_t e_ = (expr); if (e_ != hipSuccess) return e_; } while (0)

hipError_t gemm(const float* A, int64_t lda, const float* B, int64_t ldb, float* C, int64_t ldc, int M, int N, int K,
                bool subtract, hipStream_t s) {
    if (M <= 0 || N <= 0 || K <= 0) return hipSuccess;
    GemmOperands g;
    g.A = A; g.lda = lda;
    g.B0 = B; g.ldb0 = ldb; g.K0 = K;
    g.B1 = B; g.ldb1 = ldb;
    g.C = C; g.ldc = ldc;
    g.M = M; g.N = N; g.K = K;
    g.subtract = subtract;
    return gemm_f32(g, s);
}

}  // namespace

hipError_t inverse_init() {    // brings this file's code onto the device (see factor_init)
    return hipFuncSetAttribute(reinterpret_cast<const void*>(&diag_inverse_kernel), hipFuncAttributeMaxDynamicSharedMemorySize, (int)kDiagLds);
}

hipError_t inverse_from_qr(const FactorWorkspace& ws, int n, const float* A, int64_t ldk, float* Ainv32, uint16_t* Ainv16, hipStream_t s) {
    const int n_pad = ws.n_pad, nbr = n_pad / NB;
    if (n <= BW) {
        hipLaunchKernelGGL(small_inverse_kernel, dim3(nbr), dim3(256), 0, s, ws.M, ws.Rd, ws.X, A, nbr, n, ldk, Ainv32, Ainv16, ws.flag);
        return hipGetLastError();
    }
    const int64_t ld = ws.ld;
    float* R = ws.Vc;                                         // row-major (read above its diagonal blocks only)
    float* X = ws.M;
    GELO_TRY(zero_ints(ws.flag, 1, s));
    hipLaunchKernelGGL(diag_inverse_kernel, dim3((n_pad + BW - 1) / BW), dim3(512), kDiagLds, s, ws.M, ws.Rd, ws.Dinv, nbr, n, ws.flag);
    GELO_TRY(hipGetLastError());
    GELO_TRY(emit_matrix(ws.M, nbr, 1, nullptr, n, ld, R, nullptr, nullptr, nullptr, s));
    GELO_TRY(emit_matrix(ws.X, nbr, 1, nullptr, n, ld, nullptr, nullptr, X, nullptr, s));
    if (n < n_pad) GELO_TRY(pad_matrix(X, ld, n, n_pad, s));
    // a finished block of rows goes straight to its place in A^-1
    for (int c0 = (n_pad - 1) / BW * BW; c0 >= 0; c0 -= BW) {
        const int w = n - c0 < BW ? n - c0 : BW;
        GELO_TRY(gemm(ws.Dinv + (int64_t)c0 * BW, BW, X + (int64_t)c0 * ld, ld, Ainv32 + (int64_t)c0 * ldk, ldk, w, (int)ldk, w, false, s));
        GELO_TRY(gemm(R + c0, ld, Ainv32 + (int64_t)c0 * ldk, ldk, X, ld, c0, n_pad, w, true, s));
    }
    if (Ainv16 == nullptr) return hipSuccess;
    return emit_matrix(Ainv32, ldk, 0, nullptr, n, ldk, nullptr, Ainv16, nullptr, nullptr, s);
}

// Newton's iteration X <- X + X (I - A X) from X = Q^T, whose residual I - A Q^T = -E Q^T has the eigenvalues of a Gaussian of
// spectral radius 0.25: squared by every step, 2^-4, 2^-8, ... (2-norm 0.5, 0.16, 0.014 measured from 129 to 4096 rows; below 0.65 in
// all but 1e-10 of the draws at 129 rows, so that the steps cannot diverge; the residual of X3, whose square is left at the end, would show
// from a radius of 0.45 on, 0.45^16 = 3e-6 in one direction: a real eigenvalue of a Gaussian there has the probability exp(-n (x^2 - 1 - 2 ln x) / 2) with x =
// 0.45 / 0.25, e^-68 at 129 rows).  What a step adds need not be more
// exact than what the next one removes: the first two steps run on bf16 matrices (the second one's residual is the first one's squared),
// X's own rounding included; then two corrections from residuals of 16 bits of A, and of all of A and 16 bits of X, each a bf16 product:
// residuals 5e-3, 2.6e-5, then what the sums of the last one round (Frobenius, of |I|): 1.0e-7 at 129 rows, 1.9e-7 at 1024, 3.8e-7 at 4096,
// where R^-1 Q^T from a second QR left 4.3e-7, 6.1e-7, 8.7e-7; I - X A and X itself against 64 bits likewise, the largest error of an element (of the elements' root
// mean square) 8e-7 at 129 rows and 4.5e-6 at 4096, where it was 3.8e-6 and 4.8e-5.
// Bound by the matrix instructions, thirteen products of n^3: 1.42 ms at 4096 rows (0.4 more with the last residual as a float
// product, whose sums also rounded more: 8.2e-7), where the second QR and the back substitution took 4.9.  A whole draw, us, then and now: 129 rows 500 and 310,
// 512 1071 and 625, 1024 1684 and 985, 2150 3664 and 2207, 4301 10380 and 6965 (the condition estimate's launches are fewer now, too).
hipError_t inverse_near_orthogonal(const FactorWorkspace& ws, int n, const float* A, int64_t ldk, float* Ainv32, uint16_t* Ainv16, hipStream_t s) {
    const int64_t ld = ws.ld, half = (int64_t)ws.n_pad * ld;
    if (n <= BW || ldk != ld) return hipErrorInvalidValue;
    // Al lies where A^-1 will: it is read for the last time by the product before the last
    uint16_t* Ah = (uint16_t*)ws.Vc;
    uint16_t* Am = Ah + half;
    uint16_t* Al = (uint16_t*)Ainv32;
    uint16_t* m0 = (uint16_t*)ws.M;
    uint16_t* m1 = m0 + half;
    uint16_t* m2 = (uint16_t*)ws.X;
    uint16_t* m3 = m2 + half;
    GemmSum g;
    g.ld = ld; g.M = n; g.N = (int)ld; g.K = n;
    auto product = [&](const uint16_t* L, const uint16_t* R, uint16_t* out) { g.count = 1; g.A[0] = L; g.B[0] = R; g.out = out; return gemm_bf16_sum(g, s); };
    GELO_TRY(emit_matrix(ws.X, ws.n_pad / NB, 1, ws.rdiag, n, ld, nullptr, nullptr, nullptr, m0, s));    // X0 = Q^T
    const int64_t quads = (int64_t)n * ld / 4;
    hipLaunchKernelGGL(planes_kernel, dim3((unsigned)((quads + 255) / 256)), dim3(256), 0, s, A, quads, Ah, Am, Al);
    GELO_TRY(hipGetLastError());
    g.identity = g.subtract = true;
    GELO_TRY(product(Ah, m0, m2));                        // R0 = I - A X0
    g.identity = g.subtract = false;
    GELO_TRY(product(m2, m2, m1));                        // R1 = R0^2 = I - A X1
    g.x = m0;
    GELO_TRY(product(m0, m2, m3));                        // X1 = X0 + X0 R0
    g.x = m3;
    GELO_TRY(product(m3, m1, m0));                        // X2 = X1 + X1 R1
    g.x = nullptr; g.identity = g.subtract = true;
    g.A[1] = Ah; g.B[1] = m0;
    g.count = 2; g.A[0] = Am; g.B[0] = m0; g.out = m2;
    GELO_TRY(gemm_bf16_sum(g, s));                        // R2 = I - A X2
    g.x = m0; g.identity = g.subtract = false; g.out_low = m1;
    GELO_TRY(product(m0, m2, m3));                        // X3 = X2 + X2 R2
    const uint16_t* left[kGemmSumMax] = {Al, Am, Am, Ah, Ah};
    const uint16_t* right[kGemmSumMax] = {m3, m1, m3, m1, m3};
    for (int i = 0; i < kGemmSumMax; ++i) { g.A[i] = left[i]; g.B[i] = right[i]; }
    g.x = nullptr; g.identity = g.subtract = true; g.count = kGemmSumMax; g.out = m2; g.out_low = nullptr;
    GELO_TRY(gemm_bf16_sum(g, s));                        // R3 = I - A X3, the small products first
    g.x = m3; g.x_low = m1; g.identity = g.subtract = false; g.out32 = Ainv32;
    return product(m3, m2, Ainv16);                       // A^-1 = X3 + X3 R3
}

hipError_t kappa_estimate(const float* A, const float* Ainv, int64_t lda, int n, const FactorWorkspace& ws,
                          int steps, hipStream_t s) {
    const int64_t ld = ws.ld;
    if (steps < 1 || steps > kLanczosMax) return hipErrorInvalidValue;
    if (steps > n) steps = n;
    if (n <= 128) {
        hipLaunchKernelGGL(small_kappa_kernel, dim3(1), dim3(1024), 0, s, A, Ainv, lda, n, steps, ws.scalars);
        return hipGetLastError();
    }
    if (n <= kFusedMaxN) {
        // (two halves of at most n / 8 + 1 rows of ld each)
        const int few = (n + kFusedWaves - 1) / kFusedWaves < kFusedGroups ? (n + kFusedWaves - 1) / kFusedWaves : kFusedGroups;
        for (int j = 0; j <= steps; ++j) {
            auto step = [&](auto chc) {
                hipLaunchKernelGGL((lanczos_step_kernel<decltype(chc)::value>), dim3(j < steps ? few : 1, 2), dim3(kFusedThreads), 0, s, A, Ainv, ws.M, ws.X, ws.vec, lda, ld, n,
                                   ws.tri, j, steps, few);
                return hipGetLastError();
            };
            if (n <= 256) GELO_TRY(step(std::integral_constant<int, 1>{}));
            else if (n <= 512) GELO_TRY(step(std::integral_constant<int, 2>{}));
            else GELO_TRY(step(std::integral_constant<int, 4>{}));
        }
        hipLaunchKernelGGL(lanczos_finish_kernel, dim3(1), dim3(64), 0, s, ws.tri, steps, ws.scalars);
        return hipGetLastError();
    }
    // the workgroups' sums go to the (now free) factorisation buffers, kProductGroups rows of each, their sum behind them
    const int64_t w_at = (int64_t)kProductGroups * ld;
    for (int j = 0; j <= steps; ++j) {
        // the next vector, w = M^T (M v) for M = A and M = Ainv
        auto product = [&](auto chc) {
            hipLaunchKernelGGL((normal_product_kernel<decltype(chc)::value>), dim3(j < steps ? kProductGroups : 1, 2), dim3(256), 0, s, A, Ainv, ws.M, ws.X, w_at, ws.vec, lda, ld, n,
                               ws.tri, j, steps);
            return hipGetLastError();
        };
        if (n <= 2048) GELO_TRY(product(std::integral_constant<int, 8>{}));
        else if (n <= 3072) GELO_TRY(product(std::integral_constant<int, 12>{}));
        else if (n <= 4096) GELO_TRY(product(std::integral_constant<int, 16>{}));
        else GELO_TRY(product(std::integral_constant<int, 20>{}));
        if (j == steps) break;
        hipLaunchKernelGGL(sum_parts_kernel, dim3((n + 63) / 64, 2), dim3(256), 0, s, ws.M, ws.M + w_at, ws.X, ws.X + w_at, ld, n, kProductGroups);
        GELO_TRY(hipGetLastError());
    }
    hipLaunchKernelGGL(lanczos_finish_kernel, dim3(1), dim3(64), 0, s, ws.tri, steps, ws.scalars);
    return hipGetLastError();
}

}  // namespace gelo

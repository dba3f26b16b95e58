// Decode-shaped batches (n = n_data + k_shield <= 128): the trusted side's two latency-bound steps as
// single launches.
//
//   small_sample   draws the secrets of MANY batches at once (Section 3.2 step 1.2: a fresh A per batch; a
//                  decode step needs one per layer, and A does not depend on the data, so a whole step's
//                  worth is drawn ahead in one launch).  One workgroup per matrix: Philox Gaussian into
//                  LDS, unblocked Householder QR in registers (small_qr.h), A = Q diag(sign r_ii) and its
//                  transpose written out; one more workgroup per shield direction row.
//   small_mix      shield rows (row-norm statistic of H, exact-norm scaling; Section 3.2.1 eqs. 7-8) and
//                  U = A [H ; S] (eq. 1) in one launch.
//
// Both replace chains of 4 - 8 launches of the general kernels, each of which costs more in launch latency
// than in work at this size.
#include "gelo_internal.h"
#include "small_qr.h"

namespace gelo {
namespace {

typedef float f32x4_t __attribute__((ext_vector_type(4)));
typedef float f32x16_t __attribute__((ext_vector_type(16)));
typedef __bf16 bf16x8_t __attribute__((ext_vector_type(8)));
typedef uint32_t u32x4_t __attribute__((ext_vector_type(4)));

// pitch (floats) of a row of the Gaussian in LDS: 16 neighbouring columns of four neighbouring rows (what a wave moves
// between LDS and its registers at a time) fall on distinct banks, and the pitch is odd for the transposing read
__host__ __device__ inline int small_pitch(int n) { return (n + 63) / 64 * 64 + 17; }

struct SmallSampleArgs {
    SmallSampleTargets t;
    uint32_t key0, key1, c1_mix, c1_shield;
    uint64_t first_batch;
    int count, n, k, d;
    int64_t ldk;
};

// Workgroup of role 0: one matrix.  The Gaussian goes through LDS once (its elements are drawn in row order, four per
// Philox block) into the registers of small_householder; Q^T comes back through the same LDS and leaves as rows of A and
// A^T, 16 (float) or 8 (bf16) bytes per lane.  The columns and the identity beside them lived in LDS before, one thread
// walking down its column twice per reflector: 94 us at 68 rows.
template <int NR>
__global__ __launch_bounds__(32 * NR < 256 ? 256 : (32 * NR + 63) / 64 * 64)
void small_sample_kernel(SmallSampleArgs a) {
    extern __shared__ __attribute__((aligned(16))) float W[];
    __shared__ SmallQrShared<NR> sh;
    __shared__ float wave_part[4];
    // the matrices first: their workgroups run longest
    const int item = blockIdx.x < a.count ? blockIdx.x : (blockIdx.x - a.count) / a.k;
    const int role = blockIdx.x < a.count ? 0 : 1 + (blockIdx.x - a.count) % a.k;
    const uint64_t batch = a.first_batch + (uint64_t)item;
    const int tid = threadIdx.x, nthr = blockDim.x;
    PhiloxStream ps;
    ps.key0 = a.key0; ps.key1 = a.key1; ps.c2 = (uint32_t)batch; ps.c3 = (uint32_t)(batch >> 32);
    char* block = (char*)a.t.block[item];
    if (role > 0) {
        if (tid >= 256) return;                                  // a row of shield directions is the work of 256 threads
        ps.c1 = a.c1_shield;
        shield_direction_row((float*)(block + a.t.off_GS), a.d, role - 1, ps, (float*)(block + a.t.off_gsnorm), wave_part);
        return;
    }
    const int n = a.n, pitch = small_pitch(n);
    // G: element e = r n + c is output e % 4 of Philox block e / 4
    const int total = n * n;
    for (int q = tid; q * 4 < total; q += nthr) {
        uint32_t c0 = (uint32_t)q, c1 = a.c1_mix, c2 = ps.c2, c3 = ps.c3;
        philox4x32_10(c0, c1, c2, c3, ps.key0, ps.key1);
        float z[4];
        box_muller(c0, c1, &z[0], &z[1]);
        box_muller(c2, c3, &z[2], &z[3]);
        int e = q * 4;
        int r = e / n, c = e - r * n;
#pragma unroll
        for (int t = 0; t < 4; ++t) {
            if (e + t < total) W[r * pitch + c] = z[t];
            if (++c == n) { c = 0; ++r; }
        }
    }
    __syncthreads();
    const int c = tid >> 2, q = tid & 3;
    float x[NR];
#pragma unroll
    for (int i = 0; i < NR; ++i) {
        const int r = 4 * i + q;
        x[i] = c < n ? (r < n ? W[r * pitch + c] : 0.f) : (r == c - n ? 1.f : 0.f);
    }
    small_householder<NR>(x, n, sh);
    // W[r][i] = A[i][r] = Q[i][r] sign(r_rr)
    if (c >= n && c < 2 * n) {
#pragma unroll
        for (int i = 0; i < NR; ++i) {
            const int r = 4 * i + q;
            if (r < n) W[r * pitch + (c - n)] = sh.rdiag[r] < 0.f ? -x[i] : x[i];
        }
    }
    __syncthreads();
    // A and A^-1 = A^T, zero beyond column n
    float* A32 = (float*)(block + a.t.off_A32);
    float* Ai32 = (float*)(block + a.t.off_Ainv32);
    uint16_t* A16 = a.t.off_A16 >= 0 ? (uint16_t*)(block + a.t.off_A16) : nullptr;
    uint16_t* Ai16 = a.t.off_A16 >= 0 ? (uint16_t*)(block + a.t.off_Ainv16) : nullptr;
    const int ldk = (int)a.ldk, quads = ldk / 4;
    auto pack4 = [](f32x4_t v) {
        typedef __bf16 bf16x4_t __attribute__((ext_vector_type(4)));
        const bf16x4_t h = {(__bf16)v[0], (__bf16)v[1], (__bf16)v[2], (__bf16)v[3]};
        return __builtin_bit_cast(uint2, h);
    };
    for (int e = tid; e < n * quads; e += nthr) {
        const int i = e / quads, cc = (e - i * quads) * 4;
        f32x4_t v, vt;
#pragma unroll
        for (int t = 0; t < 4; ++t) {
            const bool in = cc + t < n;
            v[t] = in ? W[(cc + t) * pitch + i] : 0.f;
            vt[t] = in ? W[i * pitch + cc + t] : 0.f;
        }
        const int64_t at = (int64_t)i * ldk + cc;
        *reinterpret_cast<f32x4_t*>(A32 + at) = v;
        *reinterpret_cast<f32x4_t*>(Ai32 + at) = vt;
        if (A16) {
            *reinterpret_cast<uint2*>(A16 + at) = pack4(v);
            *reinterpret_cast<uint2*>(Ai16 + at) = pack4(vt);
        }
    }
}

// ---------------------------------------------------------------------------------------------- mix --
struct SmallMixArgs {
    const uint16_t* A16; int64_t ldk;
    const uint16_t* H; int64_t ldh;
    const float* GS; const float* gsnorm; const float* rownorm;
    int stat_kind; float shield_scale;
    int n_data, k, d;
    uint16_t* S; uint16_t* U; int64_t ldu;
};

constexpr int MIX_BN = 64;           // columns of U per workgroup

// The median of `count` row norms (count <= kSmallMaxN; norms[count .. rounded up to 4 - 1] all ones in bits) as its two middle elements,
// by 256 threads: two per norm count the (value, index) pairs below it, four at a time.
__device__ __forceinline__ void middle_norms(const float* norms, int count, float* middle) {
    const int e = threadIdx.x >> 1, half = threadIdx.x & 1;
    const float value = norms[e < count ? e : 0];
    const uint32_t mine = __float_as_uint(value);
    int below = 0;
#pragma unroll 2
    for (int i = 4 * half; i < count; i += 8) {
        const u32x4_t o = *reinterpret_cast<const u32x4_t*>(norms + i);
#pragma unroll
        for (int t = 0; t < 4; ++t) below += (o[t] < mine || (o[t] == mine && i + t < e)) ? 1 : 0;
    }
    below += __shfl_xor(below, 1, 64);
    if (half == 0 && e < count) {
        if (below == (count - 1) / 2) middle[0] = value;
        if (below == count / 2) middle[1] = value;
    }
}
__device__ __forceinline__ float norm_or_padding(float norm, int i, int count) { return i < count ? norm : __uint_as_float(0xFFFFFFFFu); }

// The operand tile of a product with at most kSmallMaxN contraction rows: 64 columns of bf16, row after row in LDS, 128 bytes each, in
// chunks of 16; the halves of rows 2, 3, 6, 7, ... are swapped, which puts the four rows of a transposing read on distinct banks.
__device__ __forceinline__ int tile_chunk(int r, int c) { return r * 8 + (c ^ (4 * ((r >> 1) & 1))); }

// One workgroup: 64 columns of U, contraction over 16 KS >= n rows; wave w owns rows 32 w .. 32 w + 31.
//
// A chain of latencies, and most of all of instruction fetches: between the projections of a decode step, each of which sends a whole
// weight through the caches, the code of this kernel is cold, and straight-line code then runs at some 30 ns per 64 bytes (cycle
// stamps).  So the code is kept short: sizes by template and clamped addresses instead of a test per load, loops over shield rows and
// norms, immediate offsets: 3.6 KB of it for 96 rows; one body for all sizes, with a test per load, took 11.7.  64 + 4 rows of 4096
// between such projections 8.7 -> 5.2 us (by themselves 8.4 -> 4.9); ranking the norms by more threads and the transposing reads, in
// the long body, 0.2 of that.
template <int KS>
__global__ __launch_bounds__(256)
void small_mix_kernel(SmallMixArgs a) {
    typedef short s16x4_t __attribute__((ext_vector_type(4)));
    typedef short s16x8_t __attribute__((ext_vector_type(8)));
    typedef __bf16 bf16x4_t __attribute__((ext_vector_type(4)));
    typedef s16x4_t __attribute__((address_space(3))) * lds_ptr_t;
    __shared__ __attribute__((aligned(16))) uint16_t tile[KS * 16 * MIX_BN];
    __shared__ __attribute__((aligned(16))) float norms[kSmallMaxN];
    __shared__ float middle[2];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int n = a.n_data + a.k, c0 = blockIdx.x * MIX_BN;
    const int j = lane & 31, grp = lane >> 5;

    // every load from memory is issued before anything waits; columns from d on repeat others and are not stored
    float my_norm = 0.f, direction = 0.f, length = 1.f;
    const int gc = c0 + lane, gcl = gc < a.d ? gc : a.d - 1;
    if (a.k > 0) {
        my_norm = a.rownorm[tid < a.n_data ? tid : 0];
        const int r = wave < a.k ? wave : 0;                     // wave w: shield rows w, w + 4, ...
        direction = a.GS[(int64_t)r * a.d + gcl];
        length = a.gsnorm[r];
    }
    constexpr int HR = KS / 2;                                   // 16-byte chunks of H per thread
    const int hr = tid >> 3, ch = tid & 7;
    const int hc = c0 + ch * 8 < a.d ? c0 + ch * 8 : a.d - 8;
    u32x4_t hreg[HR];
#pragma unroll
    for (int it = 0; it < HR; ++it) {
        const int r = hr + it * 32;
        hreg[it] = *reinterpret_cast<const u32x4_t*>(a.H + (int64_t)(r < a.n_data ? r : a.n_data - 1) * a.ldh + hc);
    }
    bf16x8_t af[KS];                                             // the wave's rows of A, zero beyond column n up to their pitch
    const int row = wave * 32 + j;
    const uint16_t* ap = a.A16 + (int64_t)(row < n ? row : n - 1) * a.ldk + grp * 8;
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) af[ks] = *reinterpret_cast<const bf16x8_t*>(ap + ks * 16);

    if (tid < kSmallMaxN) norms[tid] = norm_or_padding(my_norm, tid, a.n_data);
#pragma unroll
    for (int it = 0; it < HR; ++it) {                            // rows from n on are cleared, shield rows follow
        const int r = hr + it * 32;
        const u32x4_t zero = {0u, 0u, 0u, 0u};
        if (r < a.n_data || r >= n) *reinterpret_cast<u32x4_t*>(tile + tile_chunk(r, ch) * 8) = r < n ? hreg[it] : zero;
    }
    __syncthreads();
    if (a.k > 0) {
        float m;
        if (a.stat_kind == 0) {
            middle_norms(norms, a.n_data, middle);
            __syncthreads();
            m = 0.5f * (middle[0] + middle[1]);
        } else {
            float s = 0.f;
#pragma unroll 1
            for (int i = 0; i < a.n_data; ++i) s += norms[i];
            m = s / (float)a.n_data;
        }
#pragma unroll 1
        for (int r = wave; r < a.k; r += 4) {
            const __bf16 h = (__bf16)(direction * (a.shield_scale * m / length));
            const uint16_t bits = __builtin_bit_cast(uint16_t, h);
            const int next = r + 4 < a.k ? r + 4 : r;
            direction = a.GS[(int64_t)next * a.d + gcl];
            length = a.gsnorm[next];
            if (gc < a.d) a.S[(int64_t)r * a.d + gc] = bits;
            tile[tile_chunk(a.n_data + r, lane >> 3) * 8 + (lane & 7)] = bits;
        }
        __syncthreads();
    }
    if (wave * 32 >= n) return;
    // v_mfma_f32_32x32x16_bf16 with the tile as first operand: lane l supplies column l % 32 of the tile and row l % 32 of A, contraction
    // values 8 (l / 32) .. + 7; it receives row l % 32, columns 8 (v / 4) + 4 (l / 32) + v % 4: four neighbours are one 8-byte store.
    const int s16 = lane & 15, nh = (lane >> 4) & 1;
    const int rl = grp * 8 + (s16 >> 2);                         // row of the first transposing read; the second is 4 below
#pragma unroll
    for (int t = 0; t < 2; ++t) {
        const uint16_t* at = tile + tile_chunk(rl, t * 4 + nh * 2) * 8 + (s16 & 3) * 4;
        f32x16_t acc;
#pragma unroll
        for (int v = 0; v < 16; ++v) acc[v] = 0.f;
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) {
            const s16x4_t lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_ptr_t)(at + ks * 16 * MIX_BN));
            const s16x4_t hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_ptr_t)(at + (ks * 16 + 4) * MIX_BN));
            const s16x8_t both = {lo[0], lo[1], lo[2], lo[3], hi[0], hi[1], hi[2], hi[3]};
            acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8_t, both), af[ks], acc, 0, 0, 0);
        }
        if (row < n) {
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const int col = c0 + t * 32 + 8 * q + 4 * grp;   // d is a multiple of 8
                const bf16x4_t h = {(__bf16)acc[4 * q], (__bf16)acc[4 * q + 1], (__bf16)acc[4 * q + 2], (__bf16)acc[4 * q + 3]};
                if (col < a.d) *reinterpret_cast<uint2*>(a.U + (int64_t)row * a.ldu + col) = __builtin_bit_cast(uint2, h);
            }
        }
    }
}

struct SmallMixF32Args {
    const float* A; int64_t ldk;
    const float* H; int64_t ldh;
    const float* GS; const float* gsnorm; const float* rownorm;
    int stat_kind; float shield_scale;
    int n_data, k, d;
    float* S; float* U; int64_t ldu;
};

// || row ||_2 of `cols` floats for up to kRowsTogether rows of pitch `ld` by one wave, in every lane; cols a multiple of 8, the rows
// 16-byte aligned, their reads on their way together.  Rows from `rows` on repeat the last one.  The sums run as in row_norms (sampler.hip).
constexpr int kRowsTogether = 8;
__device__ __forceinline__ void row_norms_of_wave(const float* first, int64_t ld, int rows, int cols, int lane, float (&norm)[kRowsTogether]) {
#pragma unroll
    for (int i = 0; i < kRowsTogether; ++i) norm[i] = 0.f;
#pragma unroll 1
    for (int c = lane * 4; c < cols; c += 64 * 4) {
        f32x4_t v[kRowsTogether];
#pragma unroll
        for (int i = 0; i < kRowsTogether; ++i) v[i] = *reinterpret_cast<const f32x4_t*>(first + (int64_t)(i < rows ? i : rows - 1) * ld + c);
#pragma unroll
        for (int i = 0; i < kRowsTogether; ++i)
#pragma unroll
            for (int e = 0; e < 4; ++e) norm[i] = fmaf(v[i][e], v[i][e], norm[i]);
    }
#pragma unroll
    for (int off = 32; off > 0; off >>= 1)
#pragma unroll
        for (int i = 0; i < kRowsTogether; ++i) norm[i] += __shfl_xor(norm[i], off, 64);
#pragma unroll
    for (int i = 0; i < kRowsTogether; ++i) norm[i] = sqrtf(norm[i]);
}

// The factors of the k shield rows from the row norms, 256 threads: thread t brings norm t (t < n_data) and the norm of
// shield direction t (t < k).  NORMS: the norms are taken here, from H.
struct SmallStatistic { __attribute__((aligned(16))) float norms[kSmallMaxN]; float factor[kSmallMaxN], middle[2]; };
template <bool NORMS>
__device__ __forceinline__ void shield_factors(SmallStatistic& sh, const SmallMixF32Args& a, float my_norm, float my_gsnorm) {
    const int tid = threadIdx.x;
    if (tid < kSmallMaxN && (!NORMS || tid >= a.n_data)) sh.norms[tid] = norm_or_padding(my_norm, tid, a.n_data);
    if (NORMS) {
        const int lane = tid & 63, wave = tid >> 6;
        for (int r0 = wave; r0 < a.n_data; r0 += 4 * kRowsTogether) {
            float norm[kRowsTogether];
            row_norms_of_wave(a.H + (int64_t)r0 * a.ldh, 4 * a.ldh, (a.n_data - r0 + 3) / 4, a.d, lane, norm);
#pragma unroll
            for (int i = 0; i < kRowsTogether; ++i) if (lane == 0 && r0 + 4 * i < a.n_data) sh.norms[r0 + 4 * i] = norm[i];
        }
    }
    __syncthreads();
    float m;
    if (a.stat_kind == 0) {
        middle_norms(sh.norms, a.n_data, sh.middle);
        __syncthreads();
        m = 0.5f * (sh.middle[0] + sh.middle[1]);
    } else {                                                     // a tree sum, as mean_kernel's
        if (tid < kSmallMaxN) sh.factor[tid] = tid < a.n_data ? sh.norms[tid] : 0.f;
        __syncthreads();
        for (int half = kSmallMaxN / 2; half > 0; half >>= 1) {
            if (tid < half) sh.factor[tid] += sh.factor[tid + half];
            __syncthreads();
        }
        m = sh.factor[0] / (float)a.n_data;
        __syncthreads();
    }
    if (tid < a.k) sh.factor[tid] = a.shield_scale * m / my_gsnorm;
}

// The same in float, on v_mfma_f32_32x32x2_f32 and in the order of gemm_f32_kernel (the same bits).  The operand tile lies in LDS row by row: a lane's
// values of B are single dwords, contiguous across lanes.  It takes the place of three launches (statistic, shield rows, product), NORMS of
// four, each of which costs the host about 2.5 us and the GPU 2 to 3.  mix, us from the host / in a graph, launches apart -> here: 16 + 2 rows of
// 64 (NORMS) 18.8 / 8.5 -> 11.5 / 5.8, 64 + 4 of 4096 18.8 / 11.9 -> 13.7 / 9.2, 120 + 6 of 4096 18.8 / 13.2 -> 13.6 / 12.7.  Tiny layer (16 + 2 x 64 x 192), the whole step
// 34.6 -> 28.2.  With 64 columns per workgroup 12.7 and 18.2 for the latter two: twice the float products per wave.
constexpr int MIX_FN = 32;           // columns of U per workgroup
constexpr int MIX_FP = MIX_FN + 4;   // pitch (floats) of a row of the operand tile in LDS
template <bool NORMS>
__global__ __launch_bounds__(256)
void small_mix_f32_kernel(SmallMixF32Args a) {
    __shared__ __attribute__((aligned(16))) float B[kSmallMaxN * MIX_FP];
    __shared__ SmallStatistic sh;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int n = a.n_data + a.k, c0 = blockIdx.x * MIX_FN;
    const int kp = (n + 7) & ~7;
    const int j = lane & 31, grp = lane >> 5;
    const float my_norm = (a.k > 0 && !NORMS && tid < a.n_data) ? a.rownorm[tid] : 0.f;
    const float my_gsnorm = tid < a.k ? a.gsnorm[tid] : 1.f;
    constexpr int CPR = MIX_FN / 4, HR = kSmallMaxN * CPR / 256;  // 16-byte chunks per row, of H per thread: at most 4
    f32x4_t hreg[HR];
#pragma unroll
    for (int it = 0; it < HR; ++it) {
        const int i = tid + it * 256;
        const int r = i / CPR, col = c0 + (i % CPR) * 4;
        hreg[it] = f32x4_t{0.f, 0.f, 0.f, 0.f};
        if (r < a.n_data && col < a.d) hreg[it] = *reinterpret_cast<const f32x4_t*>(a.H + (int64_t)r * a.ldh + col);
    }
    f32x4_t af[kSmallMaxN / 8];
    {
        int arow = wave * 32 + j; arow = arow < n ? arow : n - 1;
        const float* ap = a.A + (int64_t)arow * a.ldk + grp * 4;
#pragma unroll
        for (int ks = 0; ks < kSmallMaxN / 8; ++ks)
            if (ks * 8 < kp && wave * 32 < n) af[ks] = *reinterpret_cast<const f32x4_t*>(ap + ks * 8);
    }
    if (a.k > 0) shield_factors<NORMS>(sh, a, my_norm, my_gsnorm);
    __syncthreads();
#pragma unroll
    for (int it = 0; it < HR; ++it) {                            // rows n .. kp - 1 are cleared, shield rows follow
        const int i = tid + it * 256;
        const int r = i / CPR;
        if (r < a.n_data || (r >= n && r < kp)) *reinterpret_cast<f32x4_t*>(&B[r * MIX_FP + (i % CPR) * 4]) = hreg[it];
    }
    for (int i = tid; i < a.k * MIX_FN; i += 256) {
        const int r = i / MIX_FN, cc = i - r * MIX_FN;
        const int col = c0 + cc;
        float x = 0.f;
        if (col < a.d) {
            x = a.GS[(int64_t)r * a.d + col] * sh.factor[r];
            a.S[(int64_t)r * a.d + col] = x;
        }
        B[(a.n_data + r) * MIX_FP + cc] = x;
    }
    __syncthreads();
    if (wave * 32 >= n) return;
    f32x16_t acc;
#pragma unroll
    for (int v = 0; v < 16; ++v) acc[v] = 0.f;
#pragma unroll
    for (int ks = 0; ks < kSmallMaxN / 8; ++ks) {
        if (ks * 8 < kp) {
#pragma unroll
            for (int e = 0; e < 4; ++e) acc = __builtin_amdgcn_mfma_f32_32x32x2f32(af[ks][e], B[(ks * 8 + grp * 4 + e) * MIX_FP + j], acc, 0, 0, 0);
        }
    }
    const int col = c0 + j;
#pragma unroll
    for (int v = 0; v < 16; ++v) {
        const int row = wave * 32 + 8 * (v >> 2) + 4 * grp + (v & 3);
        if (row < n && col < a.d) a.U[(int64_t)row * a.ldu + col] = acc[v];
    }
}

}  // namespace

namespace {
// rows per lane of a quad: 20, 36, 68, 100 and 128 rows (a workgroup of eight threads per row; a step costs what its
// longest walk over the registers costs, so the walk is sized for the matrix: multiples of 32 rows with four more, the data and
// shield rows of a decode batch, and the largest).  Draw: 36 rows 23 us, 37 28, 68 38, 69 46, 100 58, 101 64, 128 73.  Kernels for
// 52, 84 and 116 rows in between took 7%, 9% and 1% less at their sizes.
template <class F>
hipError_t for_small_rows(int n, F&& f) {
    if (n <= 20) return f(std::integral_constant<int, 5>{});
    if (n <= 36) return f(std::integral_constant<int, 9>{});
    if (n <= 68) return f(std::integral_constant<int, 17>{});
    if (n <= 100) return f(std::integral_constant<int, 25>{});
    return f(std::integral_constant<int, 32>{});
}
size_t small_lds_bytes(int n) { return (size_t)n * small_pitch(n) * sizeof(float); }
}  // namespace

hipError_t small_init() {
    for (int n : {20, 36, 68, 100, kSmallMaxN}) {
        if (small_lds_bytes(n) <= 60 * 1024) continue;       // with the static part below 64 KB: no attribute needed
        const hipError_t e = for_small_rows(n, [&](auto R) {
            return hipFuncSetAttribute(reinterpret_cast<const void*>(&small_sample_kernel<decltype(R)::value>),
                                       hipFuncAttributeMaxDynamicSharedMemorySize, (int)small_lds_bytes(n));
        });
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

hipError_t small_sample(const SmallSampleTargets& t, int count, uint64_t first_batch, PhiloxStream ps, uint32_t c1_shield,
                        int n, int k, int d, int64_t ldk, hipStream_t stream) {
    if (count <= 0) return hipSuccess;
    if (count > kSmallMaxBatch || n < 1 || n > kSmallMaxN || k < 0 || ldk < n || ldk % 4 != 0) return hipErrorInvalidValue;
    SmallSampleArgs a;
    a.t = t;
    a.key0 = ps.key0; a.key1 = ps.key1; a.c1_mix = ps.c1; a.c1_shield = c1_shield;
    a.first_batch = first_batch;
    a.count = count; a.n = n; a.k = k; a.d = d; a.ldk = ldk;
    // at least 256 threads: what a row of shield directions takes
    const int threads = 8 * n < 256 ? 256 : (8 * n + 63) / 64 * 64;
    return for_small_rows(n, [&](auto R) {
        hipLaunchKernelGGL(small_sample_kernel<decltype(R)::value>, dim3((unsigned)(count * (1 + k))), dim3(threads), small_lds_bytes(n),
                           stream, a);
        return hipGetLastError();
    });
}

hipError_t small_mix(const uint16_t* A16, int64_t ldk, const uint16_t* H, int64_t ldh, const float* GS, const float* gsnorm,
                     const float* rownorm, int stat_kind, float shield_scale, int n_data, int k, int d,
                     uint16_t* S, uint16_t* U, int64_t ldu, hipStream_t stream) {
    const int n = n_data + k;
    if (n < 1 || n > kSmallMaxN || d < 8 || d % 8 != 0 || ldk < ((n + 31) & ~31)) return hipErrorInvalidValue;
    SmallMixArgs a;
    a.A16 = A16; a.ldk = ldk; a.H = H; a.ldh = ldh; a.GS = GS; a.gsnorm = gsnorm; a.rownorm = rownorm;
    a.stat_kind = stat_kind; a.shield_scale = shield_scale; a.n_data = n_data; a.k = k; a.d = d;
    a.S = S; a.U = U; a.ldu = ldu;
    const dim3 grid((unsigned)((d + MIX_BN - 1) / MIX_BN));
    switch ((n + 31) / 32) {
        case 1: hipLaunchKernelGGL(small_mix_kernel<2>, grid, dim3(256), 0, stream, a); break;
        case 2: hipLaunchKernelGGL(small_mix_kernel<4>, grid, dim3(256), 0, stream, a); break;
        case 3: hipLaunchKernelGGL(small_mix_kernel<6>, grid, dim3(256), 0, stream, a); break;
        default: hipLaunchKernelGGL(small_mix_kernel<8>, grid, dim3(256), 0, stream, a); break;
    }
    return hipGetLastError();
}

hipError_t small_mix_f32(const float* A, int64_t ldk, const float* H, int64_t ldh, const float* GS, const float* gsnorm,
                         const float* rownorm, int stat_kind, float shield_scale, int n_data, int k, int d,
                         float* S, float* U, int64_t ldu, hipStream_t stream) {
    const int n = n_data + k;
    if (n < 1 || n > kSmallMaxN || k < 1 || d < 8 || d % 8 != 0 || ldk < ((n + 7) & ~7)) return hipErrorInvalidValue;
    SmallMixF32Args a;
    a.A = A; a.ldk = ldk; a.H = H; a.ldh = ldh; a.GS = GS; a.gsnorm = gsnorm; a.rownorm = rownorm;
    a.stat_kind = stat_kind; a.shield_scale = shield_scale; a.n_data = n_data; a.k = k; a.d = d;
    a.S = S; a.U = U; a.ldu = ldu;
    const dim3 grid((unsigned)((d + MIX_FN - 1) / MIX_FN));
    if (rownorm == nullptr) hipLaunchKernelGGL(small_mix_f32_kernel<true>, grid, dim3(256), 0, stream, a);
    else hipLaunchKernelGGL(small_mix_f32_kernel<false>, grid, dim3(256), 0, stream, a);
    return hipGetLastError();
}

}  // namespace gelo

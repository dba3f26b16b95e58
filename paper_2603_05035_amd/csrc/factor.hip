// Blocked Householder QR with explicit Q: the orthogonal mixing matrix the trusted side draws
// for every batch (Section 3.2 step 1.2; Table 3's "A-gen (QR)" step), and the workspace shared
// with the inverse of the non-orthogonal kinds, which is built on the same factorisation.  Everything is float and deterministic: reductions run in a fixed order, no
// atomics.
//
// Matrices from 321 rows on are factorised by blocks of 128 columns (block_factor.hip); smaller ones, and what the blocks leave (144 to 272
// rows), by panels of 16 columns, each by ONE workgroup from its 16 x 16 Gram matrix (gram_panel_body); the last 128 rows, or a matrix of no
// more, by one workgroup in registers (square_qr_kernel).  Reflectors are applied on the matrix cores.  From 720 rows on Q is formed by
// blocks of 256 reflectors (block_reflect.hip), below by strips of 16 columns.
#include <type_traits>
#include <utility>

#include "gelo_internal.h"
#include "tile_qr.h"
#include "wave_tile.h"

namespace gelo {
namespace {

constexpr int NB = kPanel;

// ------------------------------------------------------------------ directly drawn panels --
// The reflectors of an m x 16 panel, every one from its column as it stands in memory (the later columns of the panel do not see the
// earlier reflectors: what the product of directly drawn reflectors needs, householder_qr with `direct`), and what the block reflector
// I - V T V^T takes: V with explicit unit diagonal and zeros above, T (16 x 16, dense row-major at Tg) and rdiag[0:16] = the beta_j.
// Reflector j: beta = -sign(alpha) ||x||, tau = (beta - alpha)/beta, v = x / (alpha - beta) below the diagonal; a zero tail gets tau = 0.
//
// One workgroup reduction and one barrier per column: with x the column below the diagonal,
// t[s] = x . P[below, s] for all 16 columns s gives the tail norm (s = j) and, with the broadcast
// pivot row, v . P[:, s] = scale * t[s] + P[j][s], for s < j the Gram entry v_s . v_j that the T factor needs.  After the reduction
// lane s of every wave holds the quantities of column s.  The column loop is unrolled so that all register indices are constants.
// Mp: the panel's first 16 x 16 tile; the tiles of the rows below follow at 256 floats each
// (element (r, c) at Mp[(r / 16) * 256 + c * 16 + r % 16]).  The reflector block is written twice,
// compactly: Vr[r * 16 + c] (row-major, the A operand of C += V W') and Vt in the same tiles as
// the panel (the A operand of W = V^T C), both with explicit unit diagonal and zeros above.
template <int NTHR, int R>
__device__ __forceinline__ void direct_panel_body(float* Mp, float* Vr, float* Vt, float* Tg, float* rdiag, int m) {
    constexpr int NW = NTHR / 64;
    __shared__ float red[2][NW][NB];
    __shared__ float prow[2][NB];
    __shared__ float Z[NB][NB];          // Z[j][s] = v_j . (column s) at step j
    __shared__ float tau_s[NB];

    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int li = lane & 15;
    const int slot = reduce16_slot(lane);
    float P[R][NB];
#pragma unroll
    for (int i = 0; i < R; ++i) {
        const int r = tid + i * NTHR;
        const int64_t at = (int64_t)(r >> 4) * 256 + (r & 15);
#pragma unroll
        for (int c = 0; c < NB; ++c) P[i][c] = r < m ? Mp[at + c * 16] : 0.f;             // 16 consecutive lanes, consecutive addresses
    }

    // Rows at or beyond m hold zeros and stay zero, rows tid + i NTHR with i > 0 lie below every
    // diagonal entry of the panel: only register row 0 needs a test against j, and that test is a
    // select, so the column loop is straight-line code.
    static_for<NB>([&](auto jc) {
        constexpr int j = decltype(jc)::value;
        constexpr int pb = j & 1;                       // LDS buffers alternate between columns
        float t[NB];
        {
            const float x = tid > j ? P[0][j] : 0.f;
#pragma unroll
            for (int s = 0; s < NB; ++s) t[s] = x * P[0][s];
        }
#pragma unroll
        for (int i = 1; i < R; ++i) {
            const float x = P[i][j];
#pragma unroll
            for (int s = 0; s < NB; ++s) t[s] = fmaf(x, P[i][s], t[s]);
        }
        if (tid == j) {                                 // row j is register row 0 of thread j
#pragma unroll
            for (int s = 0; s < NB; ++s) prow[pb][s] = P[0][s];
        }
        const float part = wave_reduce16(t, lane);
        if (lane < NB) red[pb][wave][slot] = part;
        __syncthreads();
        float tot = red[pb][0][li];                     // lane (li) now works on column li
#pragma unroll
        for (int w = 1; w < NW; ++w) tot += red[pb][w][li];
        const float pr = prow[pb][li];
        const float xnorm2 = lane_value<j>(tot);
        const float alpha = lane_value<j>(pr);
        // beta = -sign(alpha) sqrt(alpha^2 + |x|^2), tau = (beta - alpha) / beta, scale = 1 / (alpha - beta); the
        // hardware square root and reciprocals (1 ulp) keep this dependent chain short.  A zero tail: tau = 0.
        const bool tail = xnorm2 > 0.f;
        const float nrm = __builtin_amdgcn_sqrtf(fmaf(alpha, alpha, xnorm2));
        const float beta = tail ? -copysignf(nrm, alpha) : alpha;
        const float tau = tail ? (beta - alpha) * __builtin_amdgcn_rcpf(beta) : 0.f;
        const float scale = tail ? __builtin_amdgcn_rcpf(alpha - beta) : 0.f;
        const float wl = fmaf(scale, tot, pr);          // v_j . (column li)
        if (tid < NB) {
            Z[j][tid] = wl;
            if (tid == 0) { tau_s[j] = tau; rdiag[j] = beta; }
        }
        // register row 0: below the diagonal v = x * scale, on it and above it nothing reads the column again
        P[0][j] = tid > j ? P[0][j] * scale : P[0][j];
#pragma unroll
        for (int i = 1; i < R; ++i) P[i][j] *= scale;
    });
    __syncthreads();

    // T by the forward recurrence T[a][j] = -tau_j sum_{b<j} T[a][b] (v_b . v_j), T[j][j] = tau_j;
    // lane a of the first wave carries row a.
    if (tid < NB) {
        float Trow[NB];
#pragma unroll
        for (int c = 0; c < NB; ++c) Trow[c] = 0.f;
        static_for<NB>([&](auto jc) {
            constexpr int j = decltype(jc)::value;
            float acc = 0.f;
#pragma unroll
            for (int bb = 0; bb < j; ++bb) acc = fmaf(Trow[bb], Z[j][bb], acc);
            const float tj = tau_s[j];
            Trow[j] = tid < j ? -tj * acc : (tid == j ? tj : 0.f);
        });
#pragma unroll
        for (int c4 = 0; c4 < NB / 4; ++c4)
            *reinterpret_cast<float4*>(Tg + tid * NB + c4 * 4) =
                make_float4(Trow[c4 * 4], Trow[c4 * 4 + 1], Trow[c4 * 4 + 2], Trow[c4 * 4 + 3]);
    }

    // write the clean reflector block in its two layouts, in place of the panel (nobody reads these columns again)
#pragma unroll
    for (int i = 0; i < R; ++i) {
        const int r = tid + i * NTHR;
        if (r < m) {
#pragma unroll
            for (int c4 = 0; c4 < NB / 4; ++c4) {
                float v[4];
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const int c = c4 * 4 + e;
                    v[e] = r > c ? P[i][c] : (r == c ? 1.f : 0.f);
                    Vt[(int64_t)(r >> 4) * 256 + c * 16 + (r & 15)] = v[e];
                }
                *reinterpret_cast<float4*>(Vr + (int64_t)r * NB + c4 * 4) = make_float4(v[0], v[1], v[2], v[3]);
            }
        }
    }
}

// All the panels of a matrix at once, every reflector from the raw column (grid x = panel, grid y = matrix): panel p
// is the tile column p from its diagonal tile down, 16 (panels - p) rows; its reflector block goes where
// householder_qr keeps panel p's (Vr side by side in Vc, Vt in place of the panel, T and diag(R) in their arrays).
template <int NTHR, int R>
__global__ __launch_bounds__(NTHR)
void direct_panels_kernel(float* M, float* Vc, float* Tmat, float* rdiag, int nbr, int64_t batch_stride) {
    const int p = blockIdx.x;
    const int64_t off = (int64_t)blockIdx.y * batch_stride;
    float* Mp = M + off + (int64_t)p * nbr * 256 + (int64_t)p * 256;
    direct_panel_body<NTHR, R>(Mp, Vc + off + (int64_t)p * nbr * 16 * NB, Mp, Tmat + off + (int64_t)p * NB * NB, rdiag + off + p * NB, (nbr - p) * NB);
}

// ------------------------------------------------- fused block-reflector update --
// C <- C - V op(T) V^T C for a 16-column strip of C per workgroup, in ONE pass over C: the strip
// (m x 16, m a multiple of 16) lives in registers as 16 x 16 blocks in the accumulator layout of
// v_mfma_f32_16x16x4_f32, so the same registers serve as the B operand of W = V^T C (K = rows)
// and as the accumulator of C -= V W' (K = the 16 reflectors).  Wave w of 8 owns blocks
// w, w+8, ...; the 8 partial W are added in wave order (fixed order, reproducible), then
// W' = -op(T) W is formed once per strip.  V W' is summed by itself and added to C once: with C in the accumulator every
// instruction rounds at its size (|A^T A - I| / sqrt(n) at 129, 256, 400, 700 rows 3.93e-7, 4.92e-7, 5.82e-7, 7.33e-7 that way, 3.12e-7, 3.31e-7, 3.51e-7, 3.74e-7
// now; part of A^T G below the diagonal at 256 rows 2.76e-7, now 1.82e-7; 1% of a draw's time).
// Layouts, chosen so that every global access of a wave is one contiguous kilobyte, 16 bytes per
// lane: the strip is a column of 16 x 16 tiles (256 floats each, [column][row] inside: the four
// rows 4 g .. 4 g + 3 a lane owns are adjacent), the reflectors come in the same tiles (Vt) for the
// first product and as Vr[r * 16 + i] for the second.

// One block reflector I - V op(T) V^T as a strip sees it: V in both layouts, its triangle, and `shift`, the
// number of 16-row blocks by which its first row lies below the strip's first row (a strip behind a block of panels
// starts at the first row of the block's oldest reflector).
struct Reflector { const float* Vr; const float* Vt; const float* T; int shift; };
// op(T): T^T, what the factorisation applies to the columns behind a panel (reflect_strip_body, whose strips start at the
// reflector's first row), or T, the reflector itself: what forming Q applies (reflect_strip_lds_body)
// (the pointers are those of the first matrix of a batch; `off` below is the distance to this workgroup's matrix)

constexpr int kStepBlocks = 4;           // strip blocks per wave of the panels by themselves: less than kBlockTiles tile rows
static_assert(8 * kStepBlocks >= kBlockTiles - 1, "a strip's blocks");
constexpr int kPanelRows256 = 1024;      // panels of directly drawn reflectors: up to this many rows by 256 threads, longer ones by 512
constexpr int kMaxProduct = 8;           // most reflectors a strip pass applies while Q is formed (qr_bulk_kernel: all reflectors exist by then,
                                         // so the passes can be longer: measured 10% less time for the same reflectors than passes of four)

// a tile of zeros: what a strip block reads in place of a reflector block that does not exist for it
__device__ __attribute__((aligned(1024))) float g_zero_tile[256];

// One strip, one reflector.  (Two strips per workgroup, so that every reflector block a wave fetches feeds twice the matrix
// instructions, measured equal to two one-strip workgroups per compute unit, reflect_strip_lds_body.)
// `done` gets the strip's registers behind the reflector: block wave + 8 b in cr[b].
struct StripShared {
    float Wp[8][NB][NB];                                     // the waves' partial W
    float Ts[NB][NB];
};

template <int NBLK, class Done>
__device__ __forceinline__ void reflect_strip_body(StripShared& sh, const Reflector& R, int64_t off, float* Cs, int nblocks, Done&& done) {
    // the wave index as a scalar: block numbers and their offsets then live in scalar registers
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int c = lane & 15, g = lane >> 4;

    float* Cl = Cs + c * 16 + 4 * g;                         // this lane's column, its first row of tile 0
    // Blocks past the end take no part: their strip registers are zero and they are not stored; their loads are
    // clamped to the last block (a valid address, no branch).
    const int last = nblocks - 1;
    f32x4_t cr[NBLK];
#pragma unroll
    for (int b = 0; b < NBLK; ++b) {
        const int blk = wave + 8 * b;
        const f32x4_t v = *reinterpret_cast<const f32x4_t*>(Cl + 256 * (blk < nblocks ? blk : last));
        const bool valid = blk < nblocks;
        cr[b] = f32x4_t{valid ? v[0] : 0.f, valid ? v[1] : 0.f, valid ? v[2] : 0.f, valid ? v[3] : 0.f};
    }
    // The reflector's operands stream through two register groups of GRP blocks: 2 NG groups, first those of the
    // tiled layout (W = V^T C), then those of the row layout (C += V W'); group j uses register group j % 2, and as
    // soon as a group has been consumed the group two places further on is requested into the same registers.  Two
    // groups are always on their way, across the barrier too: a load consumed right behind its issue would expose
    // one memory latency per group.
    constexpr int GRP = NBLK < 5 ? NBLK : 5, NG = NBLK / GRP;
    static_assert(NBLK % GRP == 0, "blocks per wave must be a multiple of the load group");
    f32x4_t va[2][GRP];
    const float* zero_l = g_zero_tile + c * 16 + 4 * g;
    auto request = [&](auto jc) {
        constexpr int j = decltype(jc)::value, phase = j / NG, grp = j % NG;
        if constexpr (j < 2 * NG) {
            // Vt: reflector c, this lane's four rows of the block; Vr: row c of the block, reflectors 4 g ..
            const float* base = (phase == 0 ? R.Vt : R.Vr) + off + c * 16 + 4 * g;
#pragma unroll
            for (int k = 0; k < GRP; ++k) {
                const int blk = wave + 8 * (grp * GRP + k);
                const float* src = blk <= last ? base + 256 * blk : zero_l;
                va[j & 1][k] = *reinterpret_cast<const f32x4_t*>(src);
            }
        }
    };
    // (the triangle is needed behind the barrier only: fetched first, no wait for it ever stands between a request
    // and the products that use older requests)
    const float t_mine = tid < NB * NB ? R.T[off + tid] : 0.f;
    request(std::integral_constant<int, 0>{});
    request(std::integral_constant<int, 1>{});
    // W_partial[i][col] = sum over this wave's rows of V[r][i] C[r][col]; MFMA (b, v) contracts the four
    // rows 16 blk + 4 kk + v (kk = lane / 16): A = V[row][lane % 16], B = the strip register itself.
    f32x4_t w0 = {0.f, 0.f, 0.f, 0.f}, w1 = {0.f, 0.f, 0.f, 0.f};
    static_for<NG>([&](auto gc) {
        constexpr int grp = decltype(gc)::value;
#pragma unroll
        for (int k = 0; k < GRP; ++k) {
            const int b = grp * GRP + k;
            const f32x4_t a = va[grp & 1][k];
            if (wave + 8 * b > last) continue;                // a block past the end (wave-uniform): nothing to add
            w0 = __builtin_amdgcn_mfma_f32_16x16x4f32(a[0], cr[b][0], w0, 0, 0, 0);
            w1 = __builtin_amdgcn_mfma_f32_16x16x4f32(a[1], cr[b][1], w1, 0, 0, 0);
            w0 = __builtin_amdgcn_mfma_f32_16x16x4f32(a[2], cr[b][2], w0, 0, 0, 0);
            w1 = __builtin_amdgcn_mfma_f32_16x16x4f32(a[3], cr[b][3], w1, 0, 0, 0);
        }
        request(std::integral_constant<int, grp + 2>{});
    });
    if (tid < NB * NB) sh.Ts[tid >> 4][tid & 15] = t_mine;
#pragma unroll
    for (int v = 0; v < 4; ++v) sh.Wp[wave][4 * g + v][c] = w0[v] + w1[v];     // accumulator row 4 g + v, column c
    __syncthreads();
    // ONE barrier: every wave adds the eight partial W (in wave order) for the entries it needs as an operand and
    // forms W' = -T^T W itself, on the matrix cores: step s contracts reflectors 4 s + kk,
    // A = T[4 s + kk][lane % 16], B = W[4 s + kk][lane % 16]; the result arrives in the accumulator layout,
    // which is the operand layout of the second product.
    // C_block += V_block W': MFMA k contracts reflectors 4 kk + k; A = V[16 blk + lane % 16][4 kk + k]
    float bq[4];
    {
        f32x4_t wn = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int sx = 0; sx < 4; ++sx) {
            float sum = sh.Wp[0][4 * sx + g][c];
#pragma unroll
            for (int w = 1; w < 8; ++w) sum += sh.Wp[w][4 * sx + g][c];
            wn = __builtin_amdgcn_mfma_f32_16x16x4f32(sh.Ts[4 * sx + g][c], sum, wn, 0, 0, 0);
        }
#pragma unroll
        for (int k = 0; k < 4; ++k) bq[k] = -wn[k];
    }
    static_for<NG>([&](auto gc) {
        constexpr int grp = decltype(gc)::value, j = NG + grp;
#pragma unroll
        for (int k = 0; k < GRP; ++k) {
            const int b = grp * GRP + k;
            const f32x4_t a4 = va[j & 1][k];
            if (wave + 8 * b > last) continue;
            f32x4_t sum = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int kk = 0; kk < 4; ++kk) sum = __builtin_amdgcn_mfma_f32_16x16x4f32(a4[kk], bq[kk], sum, 0, 0, 0);
            cr[b] += sum;
        }
        request(std::integral_constant<int, j + 2>{});
    });
    done(cr);
}

// the same, the strip written back in place
template <int NBLK>
__device__ __forceinline__ void reflect_strip_in_place(StripShared& sh, const Reflector& R, int64_t off, float* Cs, int nblocks) {
    reflect_strip_body<NBLK>(sh, R, off, Cs, nblocks, [&](f32x4_t (&cr)[NBLK]) {
        const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
        float* Cl = Cs + (lane & 15) * 16 + 4 * (lane >> 4);
#pragma unroll
        for (int b = 0; b < NBLK; ++b) {
            const int blk = wave + 8 * b;
            if (blk < nblocks) *reinterpret_cast<f32x4_t*>(Cl + 256 * blk) = cr[b];
        }
    });
}

// The same strip for launches that hold nothing but strips (several factorisations side by side: see
// householder_qr).  There the strips' own phases - read the strip, matrix instructions, write it - must overlap
// BETWEEN workgroups of a compute unit, which takes two workgroups per unit, that is at most 128 registers per
// lane.  So the reflector blocks do not pass through registers: each wave fetches them straight into a small
// ring in LDS (direct-to-LDS loads; a block is one contiguous kilobyte in either layout, and lane l's 16 bytes
// land at 16 l, which is where it reads them back as the instruction's operand).  One 16-column strip per
// workgroup, arithmetic and summation order exactly those of reflect_strip_body.
__device__ __forceinline__ void fetch_block_to_lds(const void* gptr, uint32_t lds_addr) {      // lds_addr wave-uniform (travels in M0)
    asm volatile("s_mov_b32 m0, %1\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, off" :: "v"(gptr), "s"(lds_addr) : "memory", "m0");
}
template <int N> __device__ __forceinline__ void wait_fetches() { asm volatile("s_waitcnt vmcnt(%0)" :: "n"(N) : "memory"); }

template <int NBLK>
__device__ __forceinline__ void reflect_strip_lds_body(const Reflector* refl, int count, int64_t off, float* Cs, int nblocks) {
    constexpr int GRP = NBLK % 3 == 0 ? 3 : NBLK % 2 == 0 ? 2 : 1, NG = NBLK / GRP;      // blocks per fetch group, groups per product
    constexpr int DEPTH = 2;                                         // ring slots per wave: one group in use, one on its way
    __shared__ __attribute__((aligned(1024))) float ring[8][DEPTH][GRP][256];
    __shared__ float Wp[2][8][NB][NB];
    __shared__ float Ts[2][NB][NB];
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int c = lane & 15, g = lane >> 4;
    float* Cl = Cs + c * 16 + 4 * g;
    const int last = nblocks - 1;
    if (count < 1) return;                                           // no reflector: the strip stays as it is (and is not loaded at all)
    // The strip's own blocks arrive group by group behind the first product of the first reflector, each requested
    // two groups ahead of its use, so that a workgroup starts on the matrix cores after two groups instead of
    // after the whole strip.  (Blocks past the end load the last block again - a valid address, a fixed number of
    // loads - and are never used: the products and the stores skip them.)
    f32x4_t cr[NBLK];
    auto load_strip = [&](auto gc) {
        constexpr int grp = decltype(gc)::value;
        if constexpr (grp < NG) {
#pragma unroll
            for (int k = 0; k < GRP; ++k) {
                const int blk = wave + 8 * (grp * GRP + k);
                // the strip passes through once: keep it out of the way of the reflectors, which every strip of the matrix re-reads from L2
                cr[grp * GRP + k] = __builtin_nontemporal_load(reinterpret_cast<const f32x4_t*>(Cl + 256 * (blk < nblocks ? blk : last)));
            }
        }
    };
    const uint32_t ring_addr = __builtin_amdgcn_readfirstlane((uint32_t)(size_t)&ring[wave][0][0][0]);
    const float* mine = &ring[wave][0][0][0] + lane * 4;                 // this lane's operand inside a block
    const float* zero_l = g_zero_tile + c * 16 + 4 * g;
    // Group j of reflector q (first the NG groups of the tiled layout, then the NG of the row layout) is number
    // u = 2 NG q + j of the strip and goes to ring slot u % DEPTH.  Before a wave waits for group u it requests group
    // u + 1 into the slot that group u - 1 has just left: one group is on its way while one is in use, across the
    // barriers and from one reflector to the next.
    auto request = [&](const Reflector& R, auto uc) {
        constexpr int u = decltype(uc)::value, j = u % (2 * NG), phase = j / NG, grp = j % NG;
        const float* base = (phase == 0 ? R.Vt : R.Vr) + off + c * 16 + 4 * g;
#pragma unroll
        for (int k = 0; k < GRP; ++k) {
            const int blk = wave + 8 * (grp * GRP + k), vb = blk - R.shift;
            const float* src = (vb >= 0 && blk <= last) ? base + 256 * vb : zero_l;
            fetch_block_to_lds(src, ring_addr + (uint32_t)(((u % DEPTH) * GRP + k) * 1024));
        }
    };
    float t_next = tid < NB * NB ? refl[0].T[off + tid] : 0.f;
    load_strip(std::integral_constant<int, 0>{});
    load_strip(std::integral_constant<int, 1>{});
    request(refl[0], std::integral_constant<int, 0>{});
    static_for<kMaxProduct>([&](auto qc) {
        constexpr int q = decltype(qc)::value;
        if (q >= count) return;
        const Reflector R = refl[q];
        const bool more = q + 1 < count;
        const Reflector Rn = more ? refl[q + 1] : R;
        // Fetches (and the strip's loads) are counted in issue order, so block k of group j has landed once no more
        // are outstanding than were issued behind it: the rest of its group, the strip group that went out with the
        // request for group j + 1 (first product of the first reflector only), and group j + 1 itself - which does
        // not exist behind the last group of the last reflector.  (Any other load of this wave in between only makes
        // the wait longer.)
        auto landed = [&](auto jc, auto kc) {
            constexpr int j = decltype(jc)::value, k = decltype(kc)::value;
            constexpr int own = GRP - 1 - k, strip = (q == 0 && j + 2 < NG) ? GRP : 0;
            if constexpr (j + 1 < 2 * NG) wait_fetches<own + strip + GRP>();
            else { if (more) wait_fetches<own + GRP>(); else wait_fetches<own>(); }
        };
        auto request_ahead = [&](auto jc) {                   // the next group, into the slot consumed last
            constexpr int j = decltype(jc)::value, nj = j + 1;
            if constexpr (nj < 2 * NG) request(R, std::integral_constant<int, 2 * NG * q + nj>{});
            else if (more) request(Rn, std::integral_constant<int, 2 * NG * q + nj>{});
        };
        const float t_mine = t_next;
        f32x4_t w0 = {0.f, 0.f, 0.f, 0.f}, w1 = {0.f, 0.f, 0.f, 0.f};
        static_for<NG>([&](auto gc) {
            constexpr int grp = decltype(gc)::value;
            if constexpr (q == 0) load_strip(std::integral_constant<int, grp + 2>{});
            request_ahead(gc);
            static_for<GRP>([&](auto kc) {
                constexpr int k = decltype(kc)::value, b = grp * GRP + k;
                if (wave + 8 * b > last) return;              // a block past the end (wave-uniform): its fetch was the zero tile
                landed(gc, kc);
                const f32x4_t a = *reinterpret_cast<const f32x4_t*>(mine + (((2 * NG * q + grp) % DEPTH) * GRP + k) * 256);
                w0 = __builtin_amdgcn_mfma_f32_16x16x4f32(a[0], cr[b][0], w0, 0, 0, 0);
                w1 = __builtin_amdgcn_mfma_f32_16x16x4f32(a[1], cr[b][1], w1, 0, 0, 0);
                w0 = __builtin_amdgcn_mfma_f32_16x16x4f32(a[2], cr[b][2], w0, 0, 0, 0);
                w1 = __builtin_amdgcn_mfma_f32_16x16x4f32(a[3], cr[b][3], w1, 0, 0, 0);
            });
            asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");      // the operands are in registers before their ring slot is refilled
        });
        if (tid < NB * NB) Ts[q & 1][tid & 15][tid >> 4] = t_mine;
        if (more && tid < NB * NB) t_next = Rn.T[off + tid];
#pragma unroll
        for (int v = 0; v < 4; ++v) Wp[q & 1][wave][4 * g + v][c] = w0[v] + w1[v];
        __syncthreads();
        float bq[4];                                          // W' = -T W, formed by every wave (see reflect_strip_body)
        {
            f32x4_t wn = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int sx = 0; sx < 4; ++sx) {
                float sum = Wp[q & 1][0][4 * sx + g][c];
#pragma unroll
                for (int w = 1; w < 8; ++w) sum += Wp[q & 1][w][4 * sx + g][c];
                wn = __builtin_amdgcn_mfma_f32_16x16x4f32(Ts[q & 1][4 * sx + g][c], sum, wn, 0, 0, 0);
            }
#pragma unroll
            for (int k = 0; k < 4; ++k) bq[k] = -wn[k];
        }
        static_for<NG>([&](auto gc) {
            constexpr int grp = decltype(gc)::value, j = NG + grp;
            request_ahead(std::integral_constant<int, j>{});
            static_for<GRP>([&](auto kc) {
                constexpr int k = decltype(kc)::value, b = grp * GRP + k;
                if (wave + 8 * b > last) return;
                landed(std::integral_constant<int, j>{}, kc);
                const f32x4_t a4 = *reinterpret_cast<const f32x4_t*>(mine + (((2 * NG * q + j) % DEPTH) * GRP + k) * 256);
                f32x4_t sum = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
                for (int kk = 0; kk < 4; ++kk) sum = __builtin_amdgcn_mfma_f32_16x16x4f32(a4[kk], bq[kk], sum, 0, 0, 0);
                cr[b] += sum;
            });
            asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
        });
    });
#pragma unroll
    for (int b = 0; b < NBLK; ++b) {
        const int blk = wave + 8 * b;
        if (blk < nblocks) __builtin_nontemporal_store(cr[b], reinterpret_cast<f32x4_t*>(Cl + 256 * blk));
    }
}

// A block of panels' reflectors applied to strips of X (forming Q), for `count` matrices, one strip per workgroup, dealt to the dies
// matrix by matrix (deal_to_dies; a matrix's reflectors of a block of four panels are 1.1 MB).
struct QrBulkArgs {
    Reflector refl[kMaxProduct]; int pending;
    float* X; int strips;
    int64_t strip_stride; int nb_block; int64_t batch_stride; int count;
};
// A strip fits the 128 registers of two workgroups per CU.
template <int NBLK>
__global__ __launch_bounds__(512) __attribute__((amdgpu_waves_per_eu(4, 4)))
void qr_bulk_kernel(QrBulkArgs a) {
    int matrix, b;
    if (!deal_to_dies(blockIdx.x, a.strips, a.count, &matrix, &b)) return;
    const int64_t off = (int64_t)matrix * a.batch_stride;
    reflect_strip_lds_body<NBLK>(a.refl, a.pending, off, a.X + (int64_t)b * a.strip_stride + off, a.nb_block);
}


// ------------------------------------------------------------- panel from its Gram matrix --
// The Householder reflectors of a tall panel without a reduction per column.  Householder's step j needs of the columns
// below its row only their inner products with column j; those of all steps follow from the panel's 16 x 16 Gram matrix,
// because a reflector keeps inner products: with G the Gram matrix of rows j onward, beta = -sign(alpha) sqrt(G[j][j]),
// row j of R is G[j][s] / beta, column s loses f_s = (P[j][s] - G[j][s] / beta) / (alpha - beta) times column j, and the
// Gram matrix of the rows below j is G[i][s] - G[i][j] G[j][s] / G[j][j].  All of it happens on 16 x 16 matrices - G, the
// panel's top tile and the column operations X accumulated so far - which wave 0 keeps in registers, lane (., s) holding
// column s of each: one step is "column s -= coefficient(s) x column j", the broadcast of column j a DPP modifier of the
// multiply-add.  Then V = [L ; P2 X]: one product of the rows below the top tile with X, on the matrix cores, straight
// from the accumulator layout the strip is in.  The triangle T is the inverse of V^T V's upper triangle with half its
// diagonal (what makes I - V T V^T orthogonal for ANY V), V^T V = L^T L + X^T (P2^T P2) X.
// The Gram matrix squares the panel's condition number, which for m x 16 independent Gaussians is about
// (sqrt(m) + 4) / (sqrt(m) - 4): 3 at 64 rows, 1.2 at 2000.  So this is for tall panels of a matrix drawn as independent
// Gaussians (a panel behind its reflectors is such a matrix again); the last panels are square_qr_kernel's.
// Bound by the latency of one workgroup.  With the strip in front, per launch: 9 us (15 with a reduction and a
// barrier per column), of which the launch itself is 4.  Against 64 bits, compared with a reduction per column on the same Gaussians (24 draws at each of 12 sizes from
// 129 to 517 rows, 8 at 1000, 4 at 2150, 2 at 4096): |A^T A - I| 0.95 to 0.99 of it, part of A^T G below the diagonal 0.99 to 1.00,
// distance of A from the exact factor 0.90 to 1.05 (geometric means; the factor itself moves by the Gaussian's condition number).

constexpr int kTilePitch = NB + 4;       // floats per row of a 16 x 16 tile in LDS: row-wise 16-byte reads and column-wise 4-byte
                                         // writes of a wave are then both free of bank conflicts
constexpr int kPanelGroup = 2;           // tiles a wave turns around in LDS at a time
template <int NBLK>
struct GramShared {
    __attribute__((aligned(16))) float part[8][64][4];                      // the waves' partial Gram matrices of the rows below the top tile
    __attribute__((aligned(16))) float top[64][4];                          // the top tile, as it lies in its wave's registers
    __attribute__((aligned(16))) float X[64][4], L[64][4];                  // the column operations and the top of V, lane (g, c): rows 4 g ..
    __attribute__((aligned(16))) float turn[8][kPanelGroup][NB * kTilePitch];
    __attribute__((aligned(16))) float first[NBLK][NB * kTilePitch];        // wave 0's tiles: its registers go to the 16 x 16 matrices
};

// The panel is the strip cr (block wave + 8 b in cr[b], accumulator layout) from block FIRST on (its top tile) to block
// `last`.  Outputs as direct_panel_body's, R's diagonal tile at Rd: block FIRST of the panel goes to tile 0 of Vr and Vt.  512 threads.
// The steps on the 16 x 16 matrices are the work of wave 0 alone (on every wave they took twice as long: two waves share
// a SIMD's issue slots); the others turn their tiles around meanwhile.
template <int NBLK, int FIRST>
__device__ __forceinline__ void gram_panel_body(GramShared<NBLK>& sh, f32x4_t (&cr)[NBLK], int last, float* Vr, float* Vt, float* Tg, float* Rd, float* rdiag) {
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int c = lane & 15, g = lane >> 4;
    // P2^T P2 of this wave's blocks: register e of a block is row 4 g + e of column c, which is what lane (g, c) supplies
    // for either operand of the instruction that contracts rows 4 g + e
    {
        f32x4_t sum[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) sum[e] = f32x4_t{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int b = 0; b < NBLK; ++b) {
            const int blk = wave + 8 * b;
            if (blk > last || blk <= FIRST) continue;         // wave-uniform
#pragma unroll
            for (int e = 0; e < 4; ++e) sum[e] = __builtin_amdgcn_mfma_f32_16x16x4f32(cr[b][e], cr[b][e], sum[e], 0, 0, 0);
        }
        *reinterpret_cast<f32x4_t*>(sh.part[wave][lane]) = (sum[0] + sum[1]) + (sum[2] + sum[3]);
        if (wave == FIRST) *reinterpret_cast<f32x4_t*>(sh.top[lane]) = cr[0];
    }
    __syncthreads();
    float* mine = sh.turn[wave][0];
    // every lane gets the whole column c of a matrix in accumulator layout (symmetric or not)
    auto columns = [&](f32x4_t v, float (&col)[NB]) {
        *reinterpret_cast<f32x4_t*>(mine + c * kTilePitch + 4 * g) = v;
        __builtin_amdgcn_wave_barrier();
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const f32x4_t x = *reinterpret_cast<const f32x4_t*>(mine + c * kTilePitch + 4 * q);
#pragma unroll
            for (int e = 0; e < 4; ++e) col[4 * q + e] = x[e];
        }
        __builtin_amdgcn_wave_barrier();
    };
    // rows instead of columns: block b becomes lane (g, i): row i, columns 4 g .. 4 g + 3 (the A operand of P2 X)
    auto put = [&](float* t, f32x4_t v) {
#pragma unroll
        for (int e = 0; e < 4; ++e) t[(4 * g + e) * kTilePitch + c] = v[e];
    };
    auto get = [&](const float* t) { return *reinterpret_cast<const f32x4_t*>(t + c * kTilePitch + 4 * g); };
    f32x4_t gb = {0.f, 0.f, 0.f, 0.f}, xd, ld, xs, rd;
    float scale_c = 0.f, beta_c = 0.f;                        // of this lane's own column (wave 0)
    if (wave == 0) {
#pragma unroll
        for (int b = 0; b < NBLK; ++b) if (8 * b <= last) put(sh.first[b], cr[b]);
        f32x4_t pw[8];
#pragma unroll
        for (int w = 0; w < 8; ++w) pw[w] = *reinterpret_cast<const f32x4_t*>(sh.part[w][lane]);
        gb = ((pw[0] + pw[1]) + (pw[2] + pw[3])) + ((pw[4] + pw[5]) + (pw[6] + pw[7]));
        const f32x4_t p1 = *reinterpret_cast<const f32x4_t*>(sh.top[lane]);
        f32x4_t gf = gb;
#pragma unroll
        for (int e = 0; e < 4; ++e) gf = __builtin_amdgcn_mfma_f32_16x16x4f32(p1[e], p1[e], gf, 0, 0, 0);
        float Gc[NB], Pc[NB], Xc[NB];
        columns(gf, Gc);
        columns(p1, Pc);
#pragma unroll
        for (int i = 0; i < NB; ++i) Xc[i] = i == c ? 1.f : 0.f;
        static_for<NB>([&](auto jc) {
            constexpr int j = decltype(jc)::value;
            const float gjj = row_bcast<j>(Gc[j]), alpha = row_bcast<j>(Pc[j]);
            const bool some = gjj > 0.f;                      // a column of zeros needs no reflector
            // hardware reciprocals and root (1 ulp) keep this dependent chain short
            const float irn = some ? __builtin_amdgcn_rsqf(gjj) : 0.f;
            const float beta = -copysignf(gjj * irn, alpha), ibeta = -copysignf(irn, alpha);
            const float scale = some ? __builtin_amdgcn_rcpf(alpha - beta) : 0.f;
            const float h = c > j ? -Gc[j] * (irn * irn) : 0.f;
            const float f = c > j ? fmaf(Gc[j], ibeta, -Pc[j]) * scale : 0.f;
            if (c == j) { scale_c = scale; beta_c = beta; }
            Gc[j] = c > j ? Gc[j] * ibeta : (c == j ? beta : 0.f);      // row j of R: nobody reads row j of G again
            add_column<j, j + 1, NB>(Gc, h);
            add_column<j, j + 1, NB>(Pc, f);
            add_column<j, 0, j + 1>(Xc, f);
        });
#pragma unroll
        for (int i = 0; i < NB; ++i) {
            Xc[i] *= scale_c;
            Pc[i] = i > c ? Pc[i] * scale_c : (i == c ? 1.f : 0.f);
        }
        xd = rows_of_group(Xc, g);
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            const float x0 = Xc[4 * v], x1 = Xc[4 * v + 1], x2 = Xc[4 * v + 2], x3 = Xc[4 * v + 3];
            const float lo = g & 1 ? x1 : x0, hi = g & 1 ? x3 : x2;
            xs[v] = g & 2 ? hi : lo;                          // rows 4 v + g
        }
        ld = rows_of_group(Pc, g);
        *reinterpret_cast<f32x4_t*>(sh.X[lane]) = xd;
        *reinterpret_cast<f32x4_t*>(sh.L[lane]) = ld;
        rd = rows_of_group(Gc, g);
    } else {
#pragma unroll
        for (int b0 = 0; b0 < NBLK; b0 += kPanelGroup) {
            if (wave + 8 * b0 > last) continue;
#pragma unroll
            for (int k = 0; k < kPanelGroup; ++k) if (b0 + k < NBLK) put(sh.turn[wave][k], cr[b0 + k < NBLK ? b0 + k : 0]);
            __builtin_amdgcn_wave_barrier();
#pragma unroll
            for (int k = 0; k < kPanelGroup; ++k) if (b0 + k < NBLK) cr[b0 + k < NBLK ? b0 + k : 0] = get(sh.turn[wave][k]);
            __builtin_amdgcn_wave_barrier();
        }
    }
    __syncthreads();
    if (wave == 0) {
        // T, while the other waves form V (this one has a block less than they have).  V^T V in double precision, from the
        // float Gram matrix: its rounding would be what the orthogonality of I - V T V^T is lost to (|A^T A - I| / sqrt(n) at
        // 129, 300 and 1000 rows: 4.8e-7, 5.9e-7, 9.1e-7 with float products, 4.2e-7, 5.3e-7, 8.65e-7 this way, 4.3e-7, 5.5e-7,
        // 8.8e-7 with a reduction per column).  The double instruction leaves row 4 v + g of column c in element v.
        f64x4_t gx = {0., 0., 0., 0.}, m = {0., 0., 0., 0.};
#pragma unroll
        for (int e = 0; e < 4; ++e) gx = __builtin_amdgcn_mfma_f64_16x16x4f64((double)gb[e], (double)xd[e], gx, 0, 0, 0);
#pragma unroll
        for (int e = 0; e < 4; ++e) m = __builtin_amdgcn_mfma_f64_16x16x4f64((double)ld[e], (double)ld[e], m, 0, 0, 0);
#pragma unroll
        for (int v = 0; v < 4; ++v) m = __builtin_amdgcn_mfma_f64_16x16x4f64((double)xs[v], gx[v], m, 0, 0, 0);
        float Mc[NB], Tc[NB];
#pragma unroll
        for (int v = 0; v < 4; ++v) mine[c * kTilePitch + 4 * v + g] = (float)m[v];
        __builtin_amdgcn_wave_barrier();
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const f32x4_t x = *reinterpret_cast<const f32x4_t*>(mine + c * kTilePitch + 4 * q);
#pragma unroll
            for (int e = 0; e < 4; ++e) Mc[4 * q + e] = x[e];
        }
        float tau_c = 0.f;
#pragma unroll
        for (int i = 0; i < NB; ++i) { Tc[i] = i == c ? 1.f : 0.f; tau_c = i == c ? Mc[i] : tau_c; }
        tau_c = scale_c != 0.f ? 2.f / tau_c : 0.f;
        static_for<NB - 1>([&](auto jc) {
            constexpr int j = decltype(jc)::value;
            const float tau = row_bcast<j>(tau_c);            // (outside of the selection: all lanes have to be active)
            add_column<j, 0, j + 1>(Tc, c > j ? -Mc[j] * tau : 0.f);
        });
        const f32x4_t td = rows_of_group(Tc, g);
#pragma unroll
        for (int e = 0; e < 4; ++e) { Tg[(4 * g + e) * NB + c] = td[e] * tau_c; Rd[(4 * g + e) * NB + c] = rd[e]; }
        if (g == 0) rdiag[c] = beta_c;
#pragma unroll
        for (int b = 0; b < NBLK; ++b) if (8 * b <= last) cr[b] = get(sh.first[b]);
    } else {
        xd = *reinterpret_cast<const f32x4_t*>(sh.X[lane]);
    }
    // V = P2 X below the top tile, written in both layouts
#pragma unroll
    for (int b = 0; b < NBLK; ++b) {
        const int blk = wave + 8 * b;
        if (blk > last || blk < FIRST) continue;
        f32x4_t v = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int e = 0; e < 4; ++e) v = __builtin_amdgcn_mfma_f32_16x16x4f32(cr[b][e], xd[e], v, 0, 0, 0);
        if (blk == FIRST) v = *reinterpret_cast<const f32x4_t*>(sh.L[lane]);
        *reinterpret_cast<f32x4_t*>(Vt + 256 * (blk - FIRST) + c * 16 + 4 * g) = v;
#pragma unroll
        for (int e = 0; e < 4; ++e) Vr[256 * (blk - FIRST) + (4 * g + e) * NB + c] = v[e];
    }
}

// panel 0: the strip as it stands, nothing to apply first
template <int NBLK>
__global__ __launch_bounds__(512) __attribute__((amdgpu_waves_per_eu(2, 2)))
void gram_panel_kernel(float* Mp, float* Vr, float* Vt, float* Tg, float* Rd, float* rdiag, int nblocks, int64_t batch_stride) {
    __shared__ GramShared<NBLK> sh;
    const int64_t off = (int64_t)blockIdx.y * batch_stride;
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    f32x4_t cr[NBLK];
#pragma unroll
    for (int b = 0; b < NBLK; ++b) {
        const int blk = wave + 8 * b < nblocks ? wave + 8 * b : nblocks - 1;
        cr[b] = *reinterpret_cast<const f32x4_t*>(Mp + off + 256 * blk + (lane & 15) * 16 + 4 * (lane >> 4));
    }
    gram_panel_body<NBLK, 0>(sh, cr, nblocks - 1, Vr + off, Vt + off, Tg + off, Rd + off, rdiag + off);
}

// One launch per QR step p.  The chain of panel factorisations (one workgroup each) is the critical path, so
// the launch that follows the factorisation of panel p also factorises panel p + 1.
//   workgroup 0          applies reflector p to the 16 columns of panel p + 1, then factorises them (if they are one of these panels);
//   the others           apply reflector p to a tile column each.
// Every strip reads only the reflector and its own columns; panel p + 1 writes its own columns and its own reflector
// buffers: the workgroups of one launch never touch the same data.  Q is formed afterwards (householder_qr).
struct QrStepArgs {
    Reflector reflector;                 // p
    float* C;                            // tile (row block p, column block p + 1)
    int64_t strip_stride;                // floats between the tiles of neighbouring column blocks
    int nblocks;                         // rows / 16 from reflector p's first on
    float* Vr_next; float* Vt_next; float* Tnext; float* Rd_next; float* rdiag_next;   // outputs of panel p + 1 (Vr_next null: it is none)
    int64_t batch_stride;                // floats from one matrix's workspace to the next one's (grid y = matrix)
};

template <int NBLK>
__global__ __launch_bounds__(512) __attribute__((amdgpu_waves_per_eu(4, 4)))
void qr_step_kernel(QrStepArgs a) {
    __shared__ StripShared strip;
    const int b = blockIdx.x;
    const int64_t off = (int64_t)blockIdx.y * a.batch_stride;
    float* C = a.C + off + (int64_t)b * a.strip_stride;
    if (b > 0 || a.Vr_next == nullptr) {
        reflect_strip_in_place<NBLK>(strip, a.reflector, off, C, a.nblocks);
        return;
    }
    __shared__ GramShared<NBLK> gram;
    reflect_strip_body<NBLK>(strip, a.reflector, off, C, a.nblocks, [&](f32x4_t (&cr)[NBLK]) {
        // block 0 is a finished tile of R; the rest becomes the reflectors
        if (threadIdx.x < 64) *reinterpret_cast<f32x4_t*>(C + (threadIdx.x & 15) * 16 + 4 * (threadIdx.x >> 4)) = cr[0];
        gram_panel_body<NBLK, 1>(gram, cr, a.nblocks - 1, a.Vr_next + off, a.Vt_next + off, a.Tnext + off, a.Rd_next + off, a.rdiag_next + off);
    });
}

// ------------------------------------------------------------- the last rows, or a small matrix --
// What is left of every matrix from its tile (t0, t0) on, at most 8 x 8 tiles, by one workgroup (tile_qr.h).
// 128 rows 50 us, 64 rows 18, where a launch per panel took 8.5 each: draw alone of 144 rows 135 -> 104 us, 256 rows 203 -> 170; CONDITIONED,
// 64 rows 257 -> 200.  Bound by the chain of 16 x 8 columns, 340 cycles each (two sums over the rows of lanes, the root, the reciprocal) and
// 30 more for every tile it walks over, by the triangle of each 16 (5 us of the 50), and by 1500 to 5500 cycles per 16 columns for the reflectors of the
// tile column before.  Up to 16 x 16 tiles it was tried:
// at 9 to 16 the matrix instructions of all tile columns on one CU (16 000 cycles a tile column) cost more than the launches they save (256 rows 220 us).
// Against 64 bits, panels to the end / this (16 to 48 draws; of the first figures a part is that strips sum V W' by itself, above): |A^T A - I| / sqrt(n) at
// 129, 160, 256 rows 4.16e-7 / 3.11e-7, 4.37 / 3.14, 5.02 / 3.31; part of A^T G below the diagonal 2.24e-7 / 1.65e-7, 2.39 / 1.71, 2.81 / 1.81; distance of
// A from the exact factor 8.4e-7 / 6.0e-7, 8.8 / 6.8, 11.7 / 7.3.
struct SquareQrArgs {
    float *M, *Vc, *Tmat, *Rd, *rdiag;   // Vc: null where nobody reads the reflectors row by row
    int nbr, t0;
    int64_t batch_stride;                // (grid x = matrix)
};
template <int NT, int WAVES>                                // WAVES: on a SIMD
__global__ __launch_bounds__(64 * NT) __attribute__((amdgpu_waves_per_eu(WAVES, WAVES)))
void square_qr_kernel(SquareQrArgs a) {
    extern __shared__ __attribute__((aligned(16))) float lds[];
    const int lane = threadIdx.x & 63, c = lane & 15, g = lane >> 4;
    const int t0 = a.t0, nbt = a.nbr - t0, w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    if (w >= nbt) return;
    const TileQrShared sh(lds, nbt);
    const int64_t off = (int64_t)blockIdx.x * a.batch_stride;
    float* column = a.M + off + ((int64_t)(t0 + w) * a.nbr + t0) * 256 + c * NB + 4 * g;
    float y[4 * NT];
#pragma unroll
    for (int i = 0; i < NT; ++i) {
        f32x4_t x = {0.f, 0.f, 0.f, 0.f};
        if (i < nbt) x = *reinterpret_cast<const f32x4_t*>(column + i * 256);
#pragma unroll
        for (int e = 0; e < 4; ++e) y[4 * i + e] = x[e];
    }
    if (w == 0) {
#pragma unroll
        for (int e = 0; e < 4; ++e) sh.zero[lane * 4 + e] = 0.f;
    }
    const int panel = t0 + w;
    factorise_tile_column<NT>(sh, y, w, nbt, lane, [&](auto last) {
#pragma unroll
        for (int i = 0; i <= decltype(last)::value; ++i) *reinterpret_cast<f32x4_t*>(column + i * 256) = f32x4_t{y[4 * i], y[4 * i + 1], y[4 * i + 2], y[4 * i + 3]};      // R
    }, [&](const ColumnEnds& ends, f32x4_t diagonal, f32x4_t t, auto tiles) {
        constexpr int TC = decltype(tiles)::value;
        float* v = a.Vc + off + (int64_t)panel * a.nbr * 256 + 64 * g + c;
        float* down = column + w * 256;
#pragma unroll
        for (int b = 0; b < TC; ++b) {
            if (b >= nbt - w) continue;
            *reinterpret_cast<f32x4_t*>(down + b * 256) = f32x4_t{y[4 * b], y[4 * b + 1], y[4 * b + 2], y[4 * b + 3]};
            if (a.Vc != nullptr) {
#pragma unroll
                for (int e = 0; e < 4; ++e) v[b * 256 + e * NB] = y[4 * b + e];
            }
        }
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            a.Tmat[off + panel * 256 + (4 * g + e) * NB + c] = t[e];
            a.Rd[off + panel * 256 + (4 * g + e) * NB + c] = diagonal[e];
        }
        if (g == 0) a.rdiag[off + panel * NB + c] = ends.r;
    });
}

// zeroes what lies beyond n x n of the tiled matrix M (n_pad x n_pad) and sets the tiled X to the identity
__global__ __launch_bounds__(256)
void qr_prepare_kernel(float* M, float* X, int n, int n_pad, int64_t batch_stride) {
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;          // index into the tiled arrays
    if (i >= (int64_t)n_pad * n_pad) return;
    M += (int64_t)blockIdx.y * batch_stride; X += (int64_t)blockIdx.y * batch_stride;
    const int nbr = n_pad >> 4;
    const int tile = (int)(i >> 8), in = (int)(i & 255);
    const int r = (tile % nbr) * 16 + (in & 15), c = (tile / nbr) * 16 + (in >> 4);
    if (r >= n || c >= n) M[i] = 0.f;
    X[i] = r == c ? 1.f : 0.f;
}

__global__ __launch_bounds__(256)
void set_identity_kernel(float* X, int64_t ld, int n_pad) {
    const int c = blockIdx.x * 256 + threadIdx.x;
    const int r = blockIdx.y;
    if (c < ld && r < n_pad) X[(int64_t)r * ld + c] = (r == c) ? 1.f : 0.f;
}

__global__ __launch_bounds__(256)
void pad_matrix_kernel(float* M, int64_t ld, int n, int n_pad) {
    const int c = blockIdx.x * 256 + threadIdx.x;
    const int r = blockIdx.y;
    if (c >= ld || r >= n_pad) return;
    if (r >= n || c >= n) M[(int64_t)r * ld + c] = 0.f;
}

template <int NTHR>
hipError_t launch_direct_panels(int rows_per_thread, const FactorWorkspace& ws, int nbr, int count, int64_t batch_stride, hipStream_t s) {
    switch (rows_per_thread) {
#define GELO_CASE(RR) case RR: hipLaunchKernelGGL((direct_panels_kernel<NTHR, RR>), dim3(nbr, count), dim3(NTHR), 0, s, ws.M, ws.Vc, ws.Tmat, ws.rdiag, nbr, batch_stride); break;
        GELO_CASE(1) GELO_CASE(2) GELO_CASE(3) GELO_CASE(4) GELO_CASE(5)
        GELO_CASE(6) GELO_CASE(7) GELO_CASE(8) GELO_CASE(9) GELO_CASE(10)
#undef GELO_CASE
        default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

#define GELO_TRY(expr) do { hipError_t e_ = (expr); if (e_ != hipSuccess) return e_; } while (0)

}  // namespace

// From here on Q is formed 256 reflectors at a time (block_reflect.hip), below by strips.  One line for every count, since a matrix drawn
// alone and the same one drawn among others agree bit for bit.
bool wide_rows(int n_pad) { return n_pad >= 720; }
// the product of directly drawn reflectors, which has no chain of panels to lose: 256 at a time from here on, again whatever the count.
// One alone, strips / blocks: 640 rows 145 / 157 us, 1024 rows 240 / 199, 2150 rows 713 / 417, 4301 rows 2790 / 1390; 8 side by side 1024
// rows 431 / 473, 1300 rows 692 / 681; 32 of 2150 rows 6870 / 5770.
constexpr int kWideProduct = 1280;

static bool wide_product(int n_pad, bool direct) { return direct ? n_pad >= kWideProduct : wide_rows(n_pad); }

size_t factor_workspace_bytes(int n, bool direct) {
    const int64_t n_pad = round_up(n, NB), ld = round_up(n, 64);
    const int64_t floats = 3 * n_pad * ld + 2 * n_pad * NB + n_pad * kInvBlock + n_pad + 6 * ld + 256 + 64;
    size_t bytes = (size_t)floats * sizeof(float) + 8192;
    if (wide_product((int)n_pad, direct)) {
        const int64_t nbr = n_pad / NB, blocks = (nbr + kWideTiles - 1) / kWideTiles, area = (int64_t)(kWideTiles * 16) * (kWideTiles * 16);
        bytes += (size_t)wide_plane_values((int)n_pad) * 2 + (size_t)(nbr * 16 * kWideTiles * 16) * (3 * 2 + kWideChunks * 4) + (size_t)(blocks * area) * (4 + 8) + 4096;
    }
    if (!direct && n_pad / NB >= kBlockTiles) {
        bytes += (size_t)block_panel_values((int)n_pad) * 2 + (size_t)kCoreFloats * 4 + 1024;
        if (!wide_rows((int)n_pad)) bytes += (size_t)n_pad * 128 * (3 * 2 + kWideChunks * 4) + (size_t)(n_pad / NB) * kYrBlock * 2 + 1024;
    }
    return bytes;
}

void factor_workspace_carve(void* base, int n, FactorWorkspace* ws, bool direct) {
    const int64_t n_pad = round_up(n, NB), ld = round_up(n, 64);
    float* p = (float*)base;
    auto take = [&](int64_t count) { float* q = p; p += round_up(count, 64); return q; };
    ws->M = take(n_pad * ld);
    ws->X = take(n_pad * ld);
    ws->Vc = take(n_pad * ld);
    ws->Tmat = take(n_pad * NB);
    ws->Rd = take(n_pad * NB);
    ws->Dinv = take(n_pad * kInvBlock);
    ws->rdiag = take(n_pad);
    ws->vec = take(6 * ld);
    ws->tri = take(128);
    ws->scalars = take(16);
    ws->flag = (int*)take(16);
    ws->Yp = ws->Yr = ws->Wp = nullptr; ws->panel = nullptr; ws->Wpart = ws->Tbig = ws->core = nullptr; ws->wide_gram = nullptr;
    if (wide_product((int)n_pad, direct)) {
        const int64_t nbr = n_pad / NB, blocks = (nbr + kWideTiles - 1) / kWideTiles, w = nbr * 16 * kWideTiles * 16, area = (int64_t)(kWideTiles * 16) * (kWideTiles * 16);
        p = (float*)(((uintptr_t)p + 1023) & ~(uintptr_t)1023);
        ws->Yp = (uint16_t*)take((wide_plane_values((int)n_pad) + 1) / 2);
        ws->Yr = ws->Yp + wide_yr_offset((int)n_pad);
        ws->Wp = (uint16_t*)take(w * 3 / 2);
        ws->Wpart = take(w * kWideChunks);
        ws->Tbig = take(blocks * area);
        ws->wide_gram = (double*)take(blocks * area * 2);
    }
    if (!direct && n_pad / NB >= kBlockTiles) {
        p = (float*)(((uintptr_t)p + 1023) & ~(uintptr_t)1023);
        ws->panel = (uint16_t*)take((block_panel_values((int)n_pad) + 1) / 2);
        ws->core = take(kCoreFloats);
        if (!wide_rows((int)n_pad)) {
            ws->Wp = (uint16_t*)take(n_pad * 128 * 3 / 2);
            ws->Wpart = take(n_pad * 128 * kWideChunks);
            ws->Yr = (uint16_t*)take(n_pad / NB * kYrBlock / 2);
        }
    }
    ws->n_pad = (int)n_pad;
    ws->ld = ld;
}

__global__ void zero_ints_kernel(int* p, int count) {
    const int i = blockIdx.x * 256 + threadIdx.x;
    if (i < count) p[i] = 0;
}

hipError_t zero_ints(int* p, int count, hipStream_t stream) {
    hipLaunchKernelGGL(zero_ints_kernel, dim3((count + 255) / 256), dim3(256), 0, stream, p, count);
    return hipGetLastError();
}

hipError_t set_identity(float* X, int64_t ld, int n_pad, hipStream_t stream) {
    hipLaunchKernelGGL(set_identity_kernel, dim3((unsigned)((ld + 255) / 256), n_pad), dim3(256), 0, stream, X, ld, n_pad);
    return hipGetLastError();
}

hipError_t pad_matrix(float* M, int64_t ld, int n, int n_pad, hipStream_t stream) {
    hipLaunchKernelGGL(pad_matrix_kernel, dim3((unsigned)((ld + 255) / 256), n_pad), dim3(256), 0, stream,
                       M, ld, n, n_pad);
    return hipGetLastError();
}

namespace {

constexpr int kSquareTiles = 8;           // what one workgroup takes of the end of a matrix, or a whole one
hipError_t launch_square_qr(const SquareQrArgs& a, int count, hipStream_t s) {
    const int tiles = a.nbr - a.t0;
    const dim3 grid(count), block(64 * tiles);
    const size_t lds = tile_qr_floats(tiles) * sizeof(float);
    if (tiles <= 4) hipLaunchKernelGGL((square_qr_kernel<4, 4>), grid, block, lds, s, a);
    // more matrices than CUs: two workgroups on one, for which 30 registers are spilled.  32 draws in 9, 10 and 17 blocks each 887 -> 846 us, 920 -> 880,
    // 1419 -> 1388; one draw, which has them all, 177 -> 180
    else if (count > kWideCus) hipLaunchKernelGGL((square_qr_kernel<kSquareTiles, 4>), grid, block, lds, s, a);
    else hipLaunchKernelGGL((square_qr_kernel<kSquareTiles, 2>), grid, block, lds, s, a);
    return hipGetLastError();
}

template <int NBLK>
hipError_t launch_qr_bulk_t(const QrBulkArgs& b, int count, hipStream_t s) {
    hipLaunchKernelGGL((qr_bulk_kernel<NBLK>), dim3(8 * dies_slots(b.strips, count)), dim3(512), 0, s, b);
    return hipGetLastError();
}

hipError_t launch_qr_bulk(const QrBulkArgs& b, int count, hipStream_t s) {
    // blocks per wave in steps of two, up to 10 (below kWideProduct): a strip kernel sized for 20 blocks spends a third more time
    // on a strip of 11 than one sized for 12 (it still requests and waits for the blocks that do not exist)
    const int per_wave = (b.nb_block + 7) / 8;
    switch ((per_wave + 1) / 2) {
        case 0: case 1: return launch_qr_bulk_t<2>(b, count, s);
        case 2: return launch_qr_bulk_t<4>(b, count, s);
        case 3: return launch_qr_bulk_t<6>(b, count, s);
        case 4: return launch_qr_bulk_t<8>(b, count, s);
        case 5: return launch_qr_bulk_t<10>(b, count, s);
        default: return hipErrorInvalidValue;
    }
}

}  // namespace

hipError_t householder_qr(const FactorWorkspace& ws, int n, int count, int64_t batch_stride, hipStream_t s, bool direct) {
    if (count < 1 || count > 65535) return hipErrorInvalidValue;
    const int64_t elems = (int64_t)ws.n_pad * ws.n_pad;
    hipLaunchKernelGGL(qr_prepare_kernel, dim3((unsigned)((elems + 255) / 256), count), dim3(256), 0, s, ws.M, ws.X, n, ws.n_pad, batch_stride);
    GELO_TRY(hipGetLastError());
    return householder_qr_prepared(ws, count, batch_stride, s, direct);
}

hipError_t householder_qr_prepared(const FactorWorkspace& ws, int count, int64_t batch_stride, hipStream_t s, bool direct) {
    if (count < 1 || count > 65535) return hipErrorInvalidValue;
    const int n_pad = ws.n_pad;
    const int nbr = n_pad / NB;                               // tile rows (= tile columns)
    const int64_t strip_stride = (int64_t)nbr * 256;
    const int panels = nbr;
    // Every panel's reflector block is kept until the end: the row-major copies side by side in ws.Vc (n_pad x 16 each,
    // n_pad x n_pad in all), the tiled copies IN PLACE of the panels they came from (a factored panel is dead: nobody
    // reads those columns of M again, and the panel kernel has all its rows in registers before it writes).
    const int64_t set_floats = (int64_t)n_pad * NB;
    auto Vr_of = [&](int p) { return ws.Vc + (int64_t)p * set_floats; };
    auto Vt_of = [&](int p) { return ws.M + (int64_t)p * strip_stride + (int64_t)p * 256; };
    // Q is formed AFTER the factorisation, last block first: block b then only meets the columns from its own first
    // one on - the rest of H_b+1 ... H_N is still the identity there - which is 4/3 n^3 operations instead of the
    // 2 n^3 of carrying Q^T along with the factorisation.
    const bool wide = wide_product(n_pad, direct);
    if (direct) {
        // every panel's reflectors from the raw columns, in one launch: nothing to factorise, no chain of panels
        const int m = n_pad;
        if (m <= kPanelRows256) GELO_TRY(launch_direct_panels<256>((m + 255) / 256, ws, nbr, count, batch_stride, s));
        else GELO_TRY(launch_direct_panels<512>((m + 511) / 512, ws, nbr, count, batch_stride, s));
    } else {
        // blocks of 128 columns, panels by themselves until one workgroup can take the rest
        int start = 0;
        if (nbr >= kBlockTiles) GELO_TRY(factor_blocks(ws, wide ? nullptr : ws.Vc, count, batch_stride, &start, s));
        const int stop = nbr - start > kSquareTiles ? nbr - kSquareTiles : start;
        if (start < stop) {
            hipLaunchKernelGGL((gram_panel_kernel<kStepBlocks>), dim3(1, count), dim3(512), 0, s, Vt_of(start), Vr_of(start), Vt_of(start),
                               ws.Tmat + (int64_t)start * NB * NB, ws.Rd + (int64_t)start * NB * NB, ws.rdiag + start * NB, nbr - start, batch_stride);
            GELO_TRY(hipGetLastError());
        }
        for (int p = start; p < stop; ++p) {
            QrStepArgs a;
            a.reflector = Reflector{Vr_of(p), Vt_of(p), ws.Tmat + (int64_t)p * NB * NB, 0};
            a.C = ws.M + (int64_t)(p + 1) * strip_stride + (int64_t)p * 256;
            a.strip_stride = strip_stride;
            a.nblocks = nbr - p;
            a.Vr_next = p + 1 < stop ? Vr_of(p + 1) : nullptr; a.Vt_next = Vt_of(p + 1);
            a.Tnext = ws.Tmat + (int64_t)(p + 1) * NB * NB; a.Rd_next = ws.Rd + (int64_t)(p + 1) * NB * NB; a.rdiag_next = ws.rdiag + (p + 1) * NB;
            a.batch_stride = batch_stride;
            hipLaunchKernelGGL((qr_step_kernel<kStepBlocks>), dim3(nbr - p - 1, count), dim3(512), 0, s, a);
            GELO_TRY(hipGetLastError());
        }
        SquareQrArgs a;
        a.M = ws.M; a.Vc = wide ? nullptr : ws.Vc; a.Tmat = ws.Tmat; a.Rd = ws.Rd; a.rdiag = ws.rdiag;
        a.nbr = nbr; a.t0 = stop; a.batch_stride = batch_stride;
        GELO_TRY(launch_square_qr(a, count, s));
    }
    if (wide) return form_product_wide(ws, count, batch_stride, s);
    {
        // X = I so far.  Block by block from the last: X[p0:, p0:] <- H_p0 (H_p0+1 (... X[p0:, p0:])), one 16-column
        // strip per workgroup, the block's reflectors newest first, each as I - V T V^T.
        // (Columns that a pass meets before their own block's turn hold the identity below the pass's first row: the
        // reflectors beyond their block leave them as they are, bit for bit, so the grouping does not show in Q.)
        const int Dq = ws.ld >= 64 * kMaxProduct ? kMaxProduct : ws.ld >= 256 ? 4 : ws.ld >= 128 ? 2 : 1;
        for (int p0 = (panels - 1) / Dq * Dq; p0 >= 0; p0 -= Dq) {
            const int pend = panels - p0 < Dq ? panels - p0 : Dq;
            QrBulkArgs b;
            for (int q = 0; q < kMaxProduct; ++q) {
                const int src = q < pend ? pend - 1 - q : 0;
                b.refl[q].Vr = Vr_of(p0 + src); b.refl[q].Vt = Vt_of(p0 + src);
                b.refl[q].T = ws.Tmat + (int64_t)(p0 + src) * NB * NB; b.refl[q].shift = src;
            }
            b.pending = pend; b.X = ws.X + (int64_t)p0 * strip_stride + (int64_t)p0 * 256;
            b.strips = nbr - p0;
            b.strip_stride = strip_stride; b.nb_block = nbr - p0; b.batch_stride = batch_stride; b.count = count;
            GELO_TRY(launch_qr_bulk(b, count, s));
        }
    }
    return hipSuccess;
}


// Brings this file's code onto the device (the runtime loads a code object on its first use, which allocates
// device memory): contexts do this when they are created, so that no later call does.
hipError_t factor_init() {
    hipFuncAttributes attr;
    return hipFuncGetAttributes(&attr, reinterpret_cast<const void*>(&qr_prepare_kernel));
}

}  // namespace gelo

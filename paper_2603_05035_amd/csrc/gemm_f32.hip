// float GEMM on the gfx950 matrix cores, used by the single-precision GELO chain (Section 3.2, eqs. 1-3) and the inverse:
// C[M x N] = A[M x K] * B[K x N], all row-major, B optionally split into two row segments ([H ; S]); optionally C <- C - A * B.
// Products of at least one 128 x 128 tile per CU go through the bf16 instructions (gemm_f32_split_kernel), smaller ones
// through v_mfma_f32_32x32x2_f32 in 64 x 64 tiles: the sums run in another order there, so a product and its parts need not agree
// to the last bit.
// A 128 x 128 tile of gemm_f32_kernel reads all of its operands before it stores, so the product may overwrite B in place with M <= 128
// (C == B0, K0 == K: a caller's un-mix into its Y) and A where
// one tile spans N.  So does a tile of gemm_f32_split_kernel.  Smaller tiles would read what their neighbours have stored: they are not
// taken where C meets an operand.
//
// gemm_f32_kernel: a workgroup of 4 waves walks K in steps of 32 through double-buffered LDS.  A lane reads four consecutive k of its A
// row with one 16-byte LDS read and spends them on four successive MFMAs; the matching B values are single dwords,
// contiguous across lanes; the fragments of the next 8 k are read while the MFMAs of the current 8 run.
#include <algorithm>

#include "gelo_internal.h"
#include "split_float.h"

namespace gelo {
namespace {

typedef float f32x16_t __attribute__((ext_vector_type(16)));

constexpr int kTileM = 128, BK = 32;   // rows of a tile (64 where the tile is 64 x 64); K step
constexpr int NT = 256;
constexpr int kCus = 256;
constexpr int A_PITCH = BK + 4;    // floats: 144-byte rows, conflict-free 16-byte reads down a column of rows

struct F32Args {
    const float* A;  int64_t lda;
    const float* B0; int64_t ldb0; int K0;
    const float* B1; int64_t ldb1;
    float* C;        int64_t ldc;
    int M, N, K;
    int tiles_m, tiles_n;
    int subtract;              // C <- C - A B (the back substitution's updates)
};

// On the float instructions: 2 x 2 waves, 64 x 64 tiles where there are too few large ones, 128 x 128 where C meets an operand.
template <int TILE>
__global__ __launch_bounds__(NT)
void gemm_f32_kernel(F32Args g) {
    constexpr int BM = TILE, BN = TILE, WAVES_M = 2;
    constexpr int ALD = BM * (BK / 4) / NT;      // A chunks per thread and K step
    constexpr int B_PITCH = BN + 4;
    constexpr int WAVES_N = 4 / WAVES_M;
    constexpr int WROWS = BM / WAVES_M, WCOLS = BN / WAVES_N;
    constexpr int MTM = WROWS / 32;              // 32-row MFMA blocks per wave
    constexpr int NTN = WCOLS / 32;              // 32-column MFMA blocks per wave
    constexpr int BCH = BN / 4;                  // 16-byte chunks per B row
    constexpr int BLD = BK * BCH / NT;           // B chunks per thread and K step
    __shared__ __attribute__((aligned(16))) float As[2][BM * A_PITCH];
    __shared__ __attribute__((aligned(16))) float Bs[2][BK * B_PITCH];

    // XCD-contiguous tile runs, N fastest inside a run (A row panel stays in that XCD's L2)
    const int total = g.tiles_m * g.tiles_n;
    const int bid = blockIdx.x;
    const int xcd = bid & 7, slot = bid >> 3;
    const int base = total >> 3, rem = total & 7;
    const int lid = xcd * base + (xcd < rem ? xcd : rem) + slot;
    const int tm = lid / g.tiles_n, tn = lid % g.tiles_n;
    const int m0 = tm * BM, n0 = tn * BN;

    const int tid = threadIdx.x;
    const int lane = tid & 63, wave = tid >> 6;
    const int wm = wave / WAVES_N, wn = wave % WAVES_N;
    const int j = lane & 31, grp = lane >> 5;
    const int KA = (g.K + 3) & ~3;
    const int k_tiles = (g.K + BK - 1) / BK;

    // the arguments the loads need, by value (scalar registers)
    const float* B0 = g.B0;
    const float* B1 = g.B1;
    const int64_t ldb0 = g.ldb0, ldb1 = g.ldb1;
    const int K0 = g.K0, Kd = g.K, Nd = g.N;

    f32x4_t a_stage[ALD], b_stage[BLD];

    auto load_global = [&](int kt) {
        const int k0 = kt * BK;
#pragma unroll
        for (int i = 0; i < ALD; ++i) {
            const int id = tid + i * NT;
            {   // A: BM rows x 8 chunks
                const int r = id >> 3, c = id & 7;
                int row = m0 + r;
                row = row < g.M ? row : g.M - 1;
                const int gk = k0 + c * 4;
                f32x4_t v = {0.f, 0.f, 0.f, 0.f};
                if (gk < KA) v = *reinterpret_cast<const f32x4_t*>(g.A + (int64_t)row * g.lda + gk);
                a_stage[i] = v;
            }
        }
        // B: 32 rows x BN / 4 chunks.  A K step that lies in one row segment of B (the common case) takes its
        // base pointer from scalar registers; picking B0 or B1 per lane makes the compiler fetch the pointer
        // itself from the argument block with a vector load, one exposed memory latency per chunk.
        const bool seg0 = k0 + BK <= K0, seg1 = k0 >= K0;
        if (seg0 || seg1) {
            const float* base = seg0 ? B0 + (int64_t)k0 * ldb0 : B1 + (int64_t)(k0 - K0) * ldb1;
            const int64_t ldb = seg0 ? ldb0 : ldb1;
#pragma unroll
            for (int i = 0; i < BLD; ++i) {
                const int id = tid + i * NT;
                const int r = id / BCH, c = id - r * BCH;
                const int gn = n0 + c * 4;
                f32x4_t v = {0.f, 0.f, 0.f, 0.f};
                if (k0 + r < Kd && gn < Nd) v = *reinterpret_cast<const f32x4_t*>(base + (int64_t)r * ldb + gn);
                b_stage[i] = v;
            }
        } else {
#pragma unroll
            for (int i = 0; i < BLD; ++i) {
                const int id = tid + i * NT;
                const int r = id / BCH, c = id - r * BCH;
                const int gk = k0 + r, gn = n0 + c * 4;
                const bool first = gk < K0;
                const int64_t off = first ? (int64_t)gk * ldb0 : (int64_t)(gk - K0) * ldb1;
                f32x4_t v = {0.f, 0.f, 0.f, 0.f};
                if (gk < Kd && gn < Nd) {
                    if (first) v = *reinterpret_cast<const f32x4_t*>(B0 + off + gn);
                    else v = *reinterpret_cast<const f32x4_t*>(B1 + off + gn);
                }
                b_stage[i] = v;
            }
        }
    };
    auto store_lds = [&](int buf) {
#pragma unroll
        for (int i = 0; i < ALD; ++i) {
            const int id = tid + i * NT;
            *reinterpret_cast<f32x4_t*>(&As[buf][(id >> 3) * A_PITCH + (id & 7) * 4]) = a_stage[i];
        }
#pragma unroll
        for (int i = 0; i < BLD; ++i) {
            const int id = tid + i * NT;
            const int r = id / BCH, c = id - r * BCH;
            *reinterpret_cast<f32x4_t*>(&Bs[buf][r * B_PITCH + c * 4]) = b_stage[i];
        }
    };

    f32x16_t acc[MTM][NTN];
#pragma unroll
    for (int a = 0; a < MTM; ++a)
#pragma unroll
        for (int b = 0; b < NTN; ++b)
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[a][b][v] = 0.f;

    load_global(0);
    store_lds(0);
    __syncthreads();

    for (int kt = 0; kt < k_tiles; ++kt) {
        const int buf = kt & 1;
        if (kt + 1 < k_tiles) load_global(kt + 1);
        // fragments of sub-step ks + 1 are read while the 16 MFMAs of sub-step ks run
        f32x4_t a4[2][MTM];
        float b1[2][4][NTN];
        auto load_frags = [&](int fb, int ks) {
#pragma unroll
            for (int mt = 0; mt < MTM; ++mt)
                a4[fb][mt] = *reinterpret_cast<const f32x4_t*>(
                    &As[buf][(wm * WROWS + mt * 32 + j) * A_PITCH + ks * 8 + grp * 4]);
#pragma unroll
            for (int e = 0; e < 4; ++e)
#pragma unroll
                for (int nt = 0; nt < NTN; ++nt)
                    b1[fb][e][nt] = Bs[buf][(ks * 8 + grp * 4 + e) * B_PITCH + wn * WCOLS + nt * 32 + j];
        };
        load_frags(0, 0);
#pragma unroll
        for (int ks = 0; ks < BK / 8; ++ks) {
            const int fb = ks & 1;
            if (ks + 1 < BK / 8) load_frags(fb ^ 1, ks + 1);
#pragma unroll
            for (int e = 0; e < 4; ++e)
#pragma unroll
                for (int mt = 0; mt < MTM; ++mt)
#pragma unroll
                    for (int nt = 0; nt < NTN; ++nt)
                        acc[mt][nt] = __builtin_amdgcn_mfma_f32_32x32x2f32(a4[fb][mt][e], b1[fb][e][nt], acc[mt][nt], 0, 0, 0);
        }
        if (kt + 1 < k_tiles) store_lds(buf ^ 1);
        __syncthreads();
    }

#pragma unroll
    for (int mt = 0; mt < MTM; ++mt)
#pragma unroll
        for (int nt = 0; nt < NTN; ++nt) {
            const int col = n0 + wn * WCOLS + nt * 32 + j;
            if (col < g.N) {
#pragma unroll
                for (int v = 0; v < 16; ++v) {
                    const int row = m0 + wm * WROWS + mt * 32 + 8 * (v >> 2) + 4 * grp + (v & 3);
                    if (row < g.M) {
                        float* cp = g.C + (int64_t)row * g.ldc + col;
                        *cp = g.subtract ? *cp - acc[mt][nt][v] : acc[mt][nt][v];
                    }
                }
            }
        }
}

// M <= 128 and K <= 128 (K a multiple of 16) where C meets B (a caller's un-mix into its Y).  One 128 x 128 tile per 128 columns would leave
// most of the chip idle and each tile bound by the float MFMA rate of its one CU, so the tiles here are 128 x 32 (four times as
// many workgroups, a wave owns 32 x 32), and with so few K steps both panels of the tile are
// fetched at once (all loads in flight together) and stored to LDS behind ONE barrier.
constexpr int SN = 32;             // tile width
constexpr int KP = 132;            // LDS pitch of the A panel, floats (conflict-free as A_PITCH is)
constexpr int SP = SN + 4;         // LDS pitch of the B panel
constexpr size_t kShortLds = ((size_t)kTileM * KP + (size_t)kTileM * SP) * sizeof(float);

__global__ __launch_bounds__(NT)
void gemm_f32_short_kernel(F32Args g) {
    extern __shared__ __attribute__((aligned(16))) float panels[];
    float* As = panels;                 // [row][k]
    float* Bs = panels + kTileM * KP;       // [k][col]
    const int n0 = blockIdx.x * SN;
    const int tid = threadIdx.x;
    const int lane = tid & 63, wave = tid >> 6;
    const int j = lane & 31, grp = lane >> 5;
    const int kc = g.K >> 2;            // 16-byte chunks per A row

    f32x4_t a_st[16], b_st[4];
#pragma unroll
    for (int i = 0; i < 16; ++i) {
        const int id = tid + i * NT;
        const int r = id / kc, c = id - r * kc;
        const int row = r < g.M ? r : g.M - 1;
        f32x4_t v = {0.f, 0.f, 0.f, 0.f};
        if (r < kTileM) v = *reinterpret_cast<const f32x4_t*>(g.A + (int64_t)row * g.lda + c * 4);
        a_st[i] = v;
    }
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const int id = tid + i * NT;
        const int r = id >> 3, c = id & 7;
        const int gn = n0 + c * 4;
        f32x4_t v = {0.f, 0.f, 0.f, 0.f};
        if (r < g.K && gn < g.N) v = *reinterpret_cast<const f32x4_t*>(g.B0 + (int64_t)r * g.ldb0 + gn);
        b_st[i] = v;
    }
#pragma unroll
    for (int i = 0; i < 16; ++i) {
        const int id = tid + i * NT;
        const int r = id / kc, c = id - r * kc;
        if (r < kTileM) *reinterpret_cast<f32x4_t*>(&As[r * KP + c * 4]) = a_st[i];
    }
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const int id = tid + i * NT;
        *reinterpret_cast<f32x4_t*>(&Bs[(id >> 3) * SP + (id & 7) * 4]) = b_st[i];
    }
    __syncthreads();

    f32x16_t acc;
#pragma unroll
    for (int v = 0; v < 16; ++v) acc[v] = 0.f;
    const int k_steps = g.K >> 3;
    for (int ks = 0; ks < k_steps; ++ks) {
        const f32x4_t a4 = *reinterpret_cast<const f32x4_t*>(&As[(wave * 32 + j) * KP + ks * 8 + grp * 4]);
#pragma unroll
        for (int e = 0; e < 4; ++e)
            acc = __builtin_amdgcn_mfma_f32_32x32x2f32(a4[e], Bs[(ks * 8 + grp * 4 + e) * SP + j], acc, 0, 0, 0);
    }
    const int col = n0 + j;
    if (col < g.N) {
#pragma unroll
        for (int v = 0; v < 16; ++v) {
            const int row = wave * 32 + 8 * (v >> 2) + 4 * grp + (v & 3);
            if (row < g.M) {
                float* cp = g.C + (int64_t)row * g.ldc + col;
                *cp = g.subtract ? *cp - acc[v] : acc[v];
            }
        }
    }
}

// The same product on the bf16 matrix instructions, every float taken apart into three bf16 values (split_float.h).  A workgroup of four
// waves has a 128 x 128 tile of C (a wave 64 x 64 of it) and walks K in steps of 32.  A thread takes apart eight
// consecutive k of a row of A or a column of B at a time and leaves the three planes in LDS as the instructions take them
// (fragments of 16 rows or columns x 32 k, lane (g, c): row c, k 8 g ..): one 16-byte write and one 16-byte read per plane, no
// conflicts but of the writes for B, which go by column pairs.  One stage in LDS, the next step's floats on their way to
// registers: two workgroups share a CU, one parks while the other multiplies.  The operands are swapped, so that a lane ends
// up with four consecutive columns of a row of C.
// Bound by what stands beside the matrix instructions, which take 45% of a step (1.66 us with a neighbour on the CU): the floats are
// taken apart anew in every tile, and two barriers stand in a step.  Error against 64 bits 0.77 to 0.9 of the float instructions'
// (K = 128 to 11008).
// Both operands are taken apart 2^16 times as large, and the sums scaled back: bf16 then holds every float down to the last bit of the
// smallest one, where it would lose the low bits of operands below 2^-110 (1 to 2% of the time; keeping the smallest magnitude of every
// step and sending small ones to the float instructions took 5 to 12%).
// What meets an infinity or a NaN comes out as NaN here (inf - inf when it is taken apart), and so may what meets operands from
// 2^112 on or sums from 2^96 on.  Such results are computed again on the float instructions, the finite ones of the tile keep their bits:
// first over the K steps that hold anything not finite, which alone decide a result that meets one; if the tile has operands large
// enough for sums to have left the range, over all steps.  Without / with a NaN or an infinity in every tile, on the float instructions
// alone, us: 2048 x 12288 x 4096 1125 / 1340 to 1590, 1720; 512 x 12288 x 4096 327 / 515, 431; 2048 x 2048 x 1000 78 / 110, 87.  All sums past
// 2^96: 3590, 1210, 214.
constexpr int kShift = 16;
constexpr float kUnscale = 0x1p-32f;
constexpr float kLarge = 0x1p32f;      // sums of less than 2^31 products of smaller operands stay below 2^95
__device__ __forceinline__ bool finite(float x) { return fabsf(x) <= 3.402823466e38f; }
constexpr int SF = kTileM / 16;                           // fragments across the tile
constexpr int SFW = SF / 2;                               // across a wave's quarter

// A thread's share of a step: eight consecutive k of two rows of A and of two columns of B
struct SplitFeed {
    static constexpr int ITEMS = kTileM * 4 / NT;
    // A: item i of this thread is row 16 (wave + 4 i) + c, k 8 q ..; B: wave w has k 8 w .., lane l the columns ITEMS l ..
    const float* arow[ITEMS];
    const float* B0;
    const float* B1;
    int64_t ldb0, ldb1;
    int K0, Kd, col0, lane, wave, q;
    f32x4_t ra[ITEMS][2];
    float rb[8][ITEMS];
    __device__ __forceinline__ SplitFeed(const F32Args& g, int m0, int n0, int tid) {
        lane = tid & 63; wave = __builtin_amdgcn_readfirstlane(tid >> 6); q = lane >> 4;
#pragma unroll
        for (int i = 0; i < ITEMS; ++i) {
            const int row = m0 + 16 * (wave + 4 * i) + (lane & 15);
            arow[i] = g.A + (int64_t)(row < g.M ? row : g.M - 1) * g.lda;
        }
        col0 = n0 + ITEMS * lane < g.N ? n0 + ITEMS * lane : g.N - ITEMS;      // (N is a multiple of 8)
        B0 = g.B0; B1 = g.B1; ldb0 = g.ldb0; ldb1 = g.ldb1; K0 = g.K0; Kd = g.K;
    }
    __device__ __forceinline__ void fetch(int t) {
        const int k0 = t * BK, ka = k0 + 8 * q, kb = k0 + 8 * wave;
#pragma unroll
        for (int i = 0; i < ITEMS; ++i) {
            const float* p = arow[i] + (ka < Kd ? ka : 0);
            ra[i][0] = *reinterpret_cast<const f32x4_t*>(p);
            ra[i][1] = *reinterpret_cast<const f32x4_t*>(p + 4);
        }
        static_assert(ITEMS == 2, "a lane's columns are read at once");
        // (the rows, and so which segment they lie in, are the same for the whole wave)
        const bool first = kb + 8 <= K0;
        if (first || (kb >= K0 && kb + 8 <= Kd)) {
            const float* p = (first ? B0 + (int64_t)kb * ldb0 : B1 + (int64_t)(kb - K0) * ldb1) + col0;
            const int64_t ld = first ? ldb0 : ldb1;
#pragma unroll
            for (int e = 0; e < 8; ++e) { const float2 v = *reinterpret_cast<const float2*>(p + e * ld); rb[e][0] = v.x; rb[e][1] = v.y; }
        } else {
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                const int k = kb + e < Kd ? kb + e : Kd - 1;
                const float* b = k < K0 ? B0 : B1;
                const int64_t at = (k < K0 ? k : k - K0) * (k < K0 ? ldb0 : ldb1) + col0;
                const float2 v = *reinterpret_cast<const float2*>(b + at);
                rb[e][0] = v.x; rb[e][1] = v.y;
            }
        }
    }
    // use(k .. k + 3, the next four, their place in the stage), cleared beyond K
    template <class Use>
    __device__ __forceinline__ void items(int t, uint16_t (*stage)[3 * SF * kFrag], Use&& use) {
        const int k0 = t * BK;
        const bool a_in = k0 + 8 * q < Kd;                // (A is zero up to the next multiple of 8)
        f32x4_t x, y;
#pragma unroll
        for (int i = 0; i < ITEMS; ++i) {
            x = ra[i][0]; y = ra[i][1];
            if (k0 + BK > Kd) {
#pragma unroll
                for (int e = 0; e < 4; ++e) { x[e] = a_in ? x[e] : 0.f; y[e] = a_in ? y[e] : 0.f; }
            }
            use(x, y, &stage[0][(wave + 4 * i) * 3 * kFrag + lane * 8]);
        }
#pragma unroll
        for (int i = 0; i < ITEMS; ++i) {
#pragma unroll
            for (int e = 0; e < 4; ++e) { x[e] = rb[e][i]; y[e] = rb[4 + e][i]; }
            if (k0 + BK > Kd) {
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    x[e] = k0 + 8 * wave + e < Kd ? x[e] : 0.f;
                    y[e] = k0 + 8 * wave + 4 + e < Kd ? y[e] : 0.f;
                }
            }
            const int col = ITEMS * lane + i;
            use(x, y, &stage[1][(col >> 4) * 3 * kFrag + (wave * 16 + (col & 15)) * 8]);
        }
    }
};

// The results of a tile that came out not finite, on the float instructions.  The stage takes the floats where the planes h and m would be.
// What it needs is formed anew from the arguments in memory and from numbers the compiler cannot tell from others, and half of a wave's
// columns are taken at a time: kept in registers through the kernel's loop it cost that a tenth of its speed.
constexpr int kTakenBits = 1024;
__device__ __forceinline__ void float_results(uint16_t (*stage)[3 * SF * kFrag], uint32_t (&taken)[kTakenBits / 32], int m0, int n0, f32x4_t (&acc)[SFW][SFW]) {
    typedef const __attribute__((address_space(4))) F32Args* KernelArgs;
    KernelArgs args = (KernelArgs)__builtin_amdgcn_kernarg_segment_ptr();
    int tid = threadIdx.x;
    asm volatile("" : "+s"(args), "+v"(tid), "+s"(m0), "+s"(n0));
    F32Args g;
    g.A = args->A; g.lda = args->lda; g.B0 = args->B0; g.ldb0 = args->ldb0; g.K0 = args->K0; g.B1 = args->B1; g.ldb1 = args->ldb1;
    g.M = args->M; g.N = args->N; g.K = args->K;
    SplitFeed in(g, m0, n0, tid);
    const int steps = (g.K + BK - 1) / BK, per_bit = (steps + kTakenBits - 1) / kTakenBits;
    // which steps hold anything not finite?
    if (tid < kTakenBits / 32) taken[tid] = 0;
    __syncthreads();
    bool large = false;
#pragma unroll 1
    for (int t0 = 0; t0 < steps; t0 += 4) {               // four steps' reads on their way at a time
        SplitFeed ahead[4] = {in, in, in, in};
#pragma unroll
        for (int i = 0; i < 4; ++i) ahead[i].fetch(t0 + i < steps ? t0 + i : steps - 1);
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const int t = t0 + i < steps ? t0 + i : steps - 1;
            uint32_t most = 0;                            // magnitudes as integers, twice
            ahead[i].items(t, stage, [&](f32x4_t x, f32x4_t y, uint16_t*) {
#pragma unroll
                for (int e = 0; e < 4; ++e) most = max(max(most, 2 * __float_as_uint(x[e])), 2 * __float_as_uint(y[e]));
            });
            const bool odd = most >= 2 * 0x7f800000u;
            if (!odd) large = large | (most >= 2 * __float_as_uint(kLarge));
            else ahead[i].items(t, stage, [&](f32x4_t x, f32x4_t y, uint16_t*) {
#pragma unroll 1
                for (int e = 0; e < 4; ++e) large = large | (finite(x[e]) & (fabsf(x[e]) >= kLarge)) | (finite(y[e]) & (fabsf(y[e]) >= kLarge));
            });
            if (odd) atomicOr(&taken[t / per_bit / 32], 1u << (t / per_bit % 32));
        }
    }
    const bool all = __syncthreads_or(large);
    auto next = [&](int t) {                              // the next step that counts from t on (the same in all waves)
        while (!all && t < steps && !(__builtin_amdgcn_readfirstlane(taken[t / per_bit / 32]) >> (t / per_bit % 32) & 1)) ++t;
        return t;
    };
    const uint16_t* fa = &stage[0][(in.wave & 1) * SFW * 3 * kFrag + in.lane * 8];
    const uint16_t* fb = &stage[1][(in.wave >> 1) * SFW * 3 * kFrag + in.lane * 8];
#pragma unroll
    for (int half = 0; half < 2; ++half) {
        f32x4_t sum[SFW / 2][SFW];
#pragma unroll
        for (int f = 0; f < SFW / 2; ++f)
#pragma unroll
            for (int n = 0; n < SFW; ++n) sum[f][n] = f32x4_t{0.f, 0.f, 0.f, 0.f};
        int t = next(0);
        in.fetch(t < steps ? t : 0);
#pragma unroll 1
        while (t < steps) {
            __syncthreads();                              // nobody reads the last stage any more
            in.items(t, stage, [&](f32x4_t x, f32x4_t y, uint16_t* at) { *reinterpret_cast<f32x4_t*>(at) = x; *reinterpret_cast<f32x4_t*>(at + kFrag) = y; });
            __syncthreads();
            t = next(t + 1);
            in.fetch(t < steps ? t : 0);
#pragma unroll 1
            for (int h = 0; h < 2; ++h) {
                f32x4_t rows[SFW];
#pragma unroll
                for (int n = 0; n < SFW; ++n) rows[n] = *reinterpret_cast<const f32x4_t*>(fa + (n * 3 + h) * kFrag);
#pragma unroll
                for (int f = 0; f < SFW / 2; ++f) {
                    const f32x4_t col = *reinterpret_cast<const f32x4_t*>(fb + ((half * SFW / 2 + f) * 3 + h) * kFrag);
#pragma unroll
                    for (int e = 0; e < 4; ++e)
#pragma unroll
                        for (int n = 0; n < SFW; ++n) sum[f][n] = __builtin_amdgcn_mfma_f32_16x16x4f32(col[e], rows[n][e], sum[f][n], 0, 0, 0);
                }
            }
        }
#pragma unroll
        for (int f = 0; f < SFW / 2; ++f)
#pragma unroll
            for (int n = 0; n < SFW; ++n)
#pragma unroll
                for (int v = 0; v < 4; ++v) {
                    const float r = acc[half * SFW / 2 + f][n][v];
                    acc[half * SFW / 2 + f][n][v] = finite(r) ? r : sum[f][n][v];
                }
    }
    __syncthreads();                                      // everybody has read its operands
}

__global__ __launch_bounds__(NT) __attribute__((amdgpu_waves_per_eu(2, 2)))
void gemm_f32_split_kernel(F32Args g) {
    constexpr int FW = SFW;
    __shared__ __attribute__((aligned(1024))) uint16_t stage[2][3 * SF * kFrag];     // A, B: [fragment][plane]
    __shared__ uint32_t taken[kTakenBits / 32];
    const int total = g.tiles_m * g.tiles_n, bid = blockIdx.x;
    const int xcd = bid & 7, slot = bid >> 3, share = total >> 3, rem = total & 7;
    const int lid = xcd * share + (xcd < rem ? xcd : rem) + slot;
    const int m0 = lid / g.tiles_n * kTileM, n0 = lid % g.tiles_n * kTileM;
    SplitFeed in(g, m0, n0, threadIdx.x);
    const int lane = in.lane, c = lane & 15, q = in.q, wm = in.wave & 1, wn = in.wave >> 1;
    const int steps = (g.K + BK - 1) / BK;
    f32x4_t acc[FW][FW];                                  // [columns][rows]
#pragma unroll
    for (int f = 0; f < FW; ++f)
#pragma unroll
        for (int n = 0; n < FW; ++n) acc[f][n] = f32x4_t{0.f, 0.f, 0.f, 0.f};
    in.fetch(0);
    for (int t = 0; t < steps; ++t) {
        if (t > 0) __syncthreads();                       // nobody reads the last stage any more
        in.items(t, stage, [&](f32x4_t x, f32x4_t y, uint16_t* at) { put_split(at, kFrag, split3<kShift>(x, y)); });
        __syncthreads();
        __builtin_amdgcn_sched_barrier(0);
        in.fetch(t + 1 < steps ? t + 1 : t);              // unconditional: a wait then counts what was issued behind what it waits for
        __builtin_amdgcn_sched_barrier(0);
        const uint16_t* fa = &stage[0][wm * FW * 3 * kFrag + lane * 8];
        const uint16_t* fb = &stage[1][wn * FW * 3 * kFrag + lane * 8];
        Split rows[FW];
#pragma unroll
        for (int n = 0; n < FW; ++n) { rows[n].h = frag_of(fa + n * 3 * kFrag); rows[n].m = frag_of(fa + (n * 3 + 1) * kFrag); rows[n].l = frag_of(fa + (n * 3 + 2) * kFrag); }
        products([&](int plane, int f) { return frag_of(fb + (f * 3 + plane) * kFrag); }, rows, acc);
    }
    bool bad = false;
#pragma unroll
    for (int f = 0; f < FW; ++f)
#pragma unroll
        for (int n = 0; n < FW; ++n)
#pragma unroll
            for (int v = 0; v < 4; ++v) { bad = bad | !finite(acc[f][n][v]); acc[f][n][v] *= kUnscale; }
    if (__syncthreads_or(bad)) float_results(stage, taken, m0, n0, acc);       // (nothing is stored before everything has been read, here too)
#pragma unroll
    for (int f = 0; f < FW; ++f) {
        const int col = n0 + (wn * FW + f) * 16 + 4 * q;
        if (col >= g.N) continue;
#pragma unroll
        for (int n = 0; n < FW; ++n) {
            const int row = m0 + (wm * FW + n) * 16 + c;
            if (row >= g.M) continue;
            f32x4_t* cp = reinterpret_cast<f32x4_t*>(g.C + (int64_t)row * g.ldc + col);
            *cp = g.subtract ? *cp - acc[f][n] : acc[f][n];
        }
    }
}

}  // namespace

hipError_t gemm_f32_init() {
    return hipFuncSetAttribute(reinterpret_cast<const void*>(gemm_f32_short_kernel),
                               hipFuncAttributeMaxDynamicSharedMemorySize, (int)kShortLds);
}

hipError_t gemm_f32(const GemmOperands& o, hipStream_t stream) {
    if (o.M <= 0 || o.N <= 0 || o.K <= 0) return hipSuccess;
    F32Args a;
    a.A = (const float*)o.A;   a.lda = o.lda;
    a.B0 = (const float*)o.B0; a.ldb0 = o.ldb0; a.K0 = o.K0;
    a.B1 = (const float*)o.B1; a.ldb1 = o.ldb1;
    a.C = (float*)o.C;         a.ldc = o.ldc;
    a.M = o.M; a.N = o.N; a.K = o.K;
    a.tiles_m = (o.M + kTileM - 1) / kTileM;
    a.subtract = o.subtract ? 1 : 0;
    // Does C share memory with an operand?  Slices of the columns of one buffer, which have the same pitch, do not where their columns
    // are apart; with different pitches the ranges from the first to the last element tell.
    auto meets_c = [&](const void* p, int64_t ld, int64_t rows, int64_t cols) {
        const intptr_t lo = (intptr_t)p, hi = lo + ((rows - 1) * ld + cols) * sizeof(float);
        const intptr_t c_lo = (intptr_t)o.C, c_hi = c_lo + ((o.M - 1) * o.ldc + o.N) * sizeof(float);
        if (rows <= 0 || lo >= c_hi || c_lo >= hi) return false;
        const intptr_t pitch = ld * sizeof(float);
        const intptr_t behind = ((lo - c_lo) % pitch + pitch) % pitch;       // from a row of C to the operand's next one
        return ld != o.ldc || behind < (intptr_t)(o.N * sizeof(float)) || behind + (intptr_t)(cols * sizeof(float)) > pitch;
    };
    const int tiles = a.tiles_m * ((o.N + kTileM - 1) / kTileM);
    const bool over_a = meets_c(o.A, o.lda, o.M, o.K);
    const bool in_place = tiles < kCus && (over_a || meets_c(o.B0, o.ldb0, std::min(o.K0, o.K), o.N) || meets_c(o.B1, o.ldb1, o.K - o.K0, o.N));
    if (in_place && !over_a && o.M <= kTileM && o.K <= 128 && o.K % 16 == 0 && o.K0 >= o.K) {
        // (not over A: every tile reads all of it.)  Against 128 x 128 tiles, us: 16 x 1024 x 16 4.5 and 6.9, 128 x 64 x 128 7.3 and 15.6, 128 x 4096 x 128
        // 8.0 and 16.1, 128 x 12288 x 128 14.4 and 17.0; only beyond does one round of large tiles win, 128 x 22016 x 128 21.1 and 17.5.  Where C meets no
        // operand 64 x 64 tiles are faster at every size: 16 x 192 x 16 3.5 us against 4.4, 128 x 12288 x 128 10.2 and 14.4.
        a.tiles_n = (o.N + SN - 1) / SN;
        hipLaunchKernelGGL(gemm_f32_short_kernel, dim3(a.tiles_n), dim3(NT), kShortLds, stream, a);
    } else if (in_place) {
        a.tiles_n = (o.N + kTileM - 1) / kTileM;
        hipLaunchKernelGGL((gemm_f32_kernel<kTileM>), dim3(a.tiles_m * a.tiles_n), dim3(NT), 0, stream, a);
    } else if (tiles < kCus) {
        // Too few large tiles to give every CU one: 64 x 64 on the float instructions.  This / 128 x 128 taken apart: 543 x 1544 x 776
        // (65 large tiles) 32 / 59 us, 1024 x 2048 x 2048 (128) 110 / 149, 700 x 4096 x 11008 (192) 697 / 764, 1900 x 2048 x 128 (240)
        // 15.9 / 15.5.  (Taken apart in 64 x 64 tiles, where the taking apart weighs twice as much: 33, 111, 849.)
        a.tiles_m = (o.M + 63) / 64; a.tiles_n = (o.N + 63) / 64;
        hipLaunchKernelGGL((gemm_f32_kernel<64>), dim3(a.tiles_m * a.tiles_n), dim3(NT), 0, stream, a);
    } else {
        // Against 128 x 96, 128 x 128 or 128 x 192 tiles on the float instructions, us: 2048 x 2048 x 1000 (256 tiles) 93 / 82, 512 x 12288 x 4096
        // (384) 520 / 410 (126 TFLOP/s), 300 x 11008 x 4096 (258) 440 / 315, 2150 x 12288 x 4096 2100 / 1510 (143), 4096 x 4096 x 4096 1330 /
        // 792 (173), 640 x 8192 x 128 25 / 21.
        a.tiles_n = (o.N + kTileM - 1) / kTileM;
        hipLaunchKernelGGL(gemm_f32_split_kernel, dim3(a.tiles_m * a.tiles_n), dim3(NT), 0, stream, a);
    }
    return hipGetLastError();
}

}  // namespace gelo

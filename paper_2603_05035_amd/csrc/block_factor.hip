// Householder QR of a large matrix in blocks of 128 columns (Section 3.2 step 1.2's orthogonal factor): the columns until
// 144 to 272 rows are left; householder_qr's panels take those.  No panel is walked column by column.  With P the block's
// m x 128 panel, C the columns behind it, C1 and P1 their first 128 rows,
//
//   S  = P^T [P | C]                    launch_panel_products; of C, behind the first block, block_overlap_kernel
//   P^T P = R^T R,  P1 - R = L U        block_core, one workgroup: Cholesky and LU elimination together, the sign of every
//                                       row of R opposite to the pivot it meets; R^-T, L^-1 and U^-1 beside them
//   Y  = [L ; P2 U^-1]                  the Householder vectors: I - Y T Y^T maps P to [R ; 0]
//   R1 = R^-T S,  N = L^-1 (C1 - R1)    block_apply_kernel: R's rows behind the block; T^T Y^T C without T
//   C2 <- C2 - Y2 N                     the next panel's columns by launch_block_update, which also takes the panel apart for the next S;
//                                       the others in block_overlap_kernel, beside the next panel's 128 x 128 part
//
// The LU elimination of the panel's top minus R is how Householder vectors are had from an orthogonal factor (Ballard, Demmel,
// Grigori, Jacquelin, Knight, Nguyen, "Reconstructing Householder vectors from tall-skinny QR", 2015), here with R from the Gram
// matrix: an m x 128 panel of a Gaussian matrix behind its reflectors is Gaussian again, with a condition number of about
// (sqrt(m) + 11.3) / (sqrt(m) - 11.3): 1.6 at 2150 rows, 5.4 at 272, where the blocks end.  CONDITIONED matrices' panels are
// no worse than A (2 to 4).
//
// A draw alone is bound by the chain of four launches per 128 columns, at 2150 rows 5.5 (panel update) + 9 (P^T P) + 34 (the core, with the columns
// further on beside it) + 7.5 us; with those columns in the chain it was 8 to 15 + 31.5 + 7 + 5 to 25.  A whole draw, that way / this, both down to
// 15 tile rows: 1024 rows 584 / 581 us, 2150 rows 1371 / 1342 (down to 17, as it is, 602 and 1361), 4301 rows 4000 / 3622; 8 side by side 2150 rows 3680 /
// 3227; 32, whose columns pass through memory once a block instead of twice, 10 420 / 10 150; up to 720 rows it makes no difference.  Panel by panel 2150
// rows took 2661, 32 side by side 14 730.  Against 64 bits, panels / blocks (four draws): |A^T A - I| / sqrt(n) at 720, 1040, 2150 rows 7.5e-7 / 5.3e-7, 8.8e-7 /
// 5.7e-7, 1.24e-6 / 6.4e-7; part of A^T G below the diagonal, of |G|, 4.34e-7 / 3.77e-7, 5.14e-7 / 3.86e-7, 7.3e-7 / 4.0e-7; distance of A from the exact
// factor at 1300 and 2150 rows 2.6e-6 / 1.9e-6, 3.4e-6 / 1.6e-6.
#include "block_reflect.h"
#include "wave_tile.h"

namespace gelo {
namespace {

constexpr int NB = kPanel;
constexpr int BT = 8;                                     // tile columns of a block
constexpr int kTurn = NB + 4;                             // LDS pitch of a tile that is turned around, floats
constexpr int kCoreTiles = BT * BT;                       // tiles of each of the core's three triangles

struct BlockArgs {
    WideArgs w;                                           // as for launch_panel_products: X at tile (t0, t0)
    float* core;                                          // R^-T, L^-1, (U^-1)^T: 8 x 8 tiles each, row-major inside
    uint16_t* Yr;                                         // of tile row t0 + 8: where Y2 goes taken apart
    float* Rd; float* rdiag;                              // of the block's first panel
};

// ------------------------------------------------------------ the 128 x 128 part --
// In-place elimination on two 8 x 8 arrays of tiles, a tile per step i.  Array S: the Gram matrix's Schur complement at (k, l), l >= k
// > i, R in its finished rows, and below the diagonal the identity that becomes R^-T.  Array A: P1's Schur complement at (k, l),
// k, l > i; the identity that becomes L^-1 at l <= i < k; the one that becomes U^-1 at k <= i < l.  Eight waves hold the tiles
// in registers, wave (k + l) % 8 both tiles of (k, l): every wave has one tile of each row and of each column.  What a step
// multiplies by - the finished row of S (PR), the finished row of A (PU) and column of A (PL) - goes through LDS as the lanes hold
// it.  A float product X Y takes X transposed and Y in that layout, so tiles of A below the diagonal and of U^-1 are kept
// transposed: then every operand is one 16-byte read.  The ninth wave eliminates the diagonal tiles: 16 columns each, column
// operations on registers (as gram_panel_body's).  It is the critical path; the others update beside it.
// Bound by that chain's latency: 8 x 16 dependent columns of about 290 cycles, and by 2000 cycles per tile for the two barriers,
// what is done between them and the tile's way through LDS.  31.5 us; 50 with the four matrices of a diagonal tile in every lane's
// registers one after the other, 45 with a matrix per row of lanes, 40 with a wave to itself and its code in a loop.
__device__ __forceinline__ f32x4_t tile_product(f32x4_t x, f32x4_t y, f32x4_t acc) {
#pragma unroll
    for (int e = 0; e < 4; ++e) acc = __builtin_amdgcn_mfma_f32_16x16x4f32(x[e], y[e], acc, 0, 0, 0);
    return acc;
}

// A tile in LDS, lane (g, c)'s four values at kCoreRow g + 4 c: the rows of 16 lanes are apart by four banks more than all of them, so
// that writing a column's sixteen values one by one into the places of the transpose meets no bank twice, nor does it in
// neighbouring tiles.
constexpr int kCoreRow = 4 * NB + 4, kCoreTile = 4 * kCoreRow;
struct CoreShared {
    __attribute__((aligned(16))) float PR[2][BT][kCoreTile], PU[2][BT][kCoreTile], PL[2][BT][kCoreTile];
    __attribute__((aligned(16))) float DF[kCoreTile], DL[kCoreTile], DX[kCoreTile];        // R_ii^-T, L_ii^-1, U_ii^-T as left operands
    __attribute__((aligned(16))) float DA[2][kCoreTile], DS[2][kCoreTile];                 // the next diagonal tiles
    __attribute__((aligned(16))) float turn[2][kCoreTile];                                 // the ninth wave's own
};

// 16 columns of both eliminations; a, s: the diagonal tiles in accumulator layout.  One wave, lane (g, c) column c of matrix g, each
// in place: S_ii, above whose diagonal the column operations grow that make R_ii^-1 of the identity; A_ii with those that make
// U_ii^-1; A_ii again, below whose diagonal the row operations grow that make L_ii^-1.  A step adds multiples of column j to other
// columns, all matrices in the same 15 instructions.  `published` (the barrier) comes between what the other waves wait for and the
// stores to memory.
template <class Published>
__device__ __forceinline__ void core_diagonal(CoreShared& sh, int q, int i, f32x4_t a, f32x4_t s, float* Vtile, float* Rd, float* rdiag, int lane, Published&& published) {
    const int c = lane & 15, g = lane >> 4;
    const int place = g * kCoreRow + c * 4;
    *reinterpret_cast<f32x4_t*>(sh.turn[0] + place) = s;
    *reinterpret_cast<f32x4_t*>(sh.turn[1] + place) = a;
    __builtin_amdgcn_wave_barrier();
    float col[NB], Rc[NB];
    const float* mine = sh.turn[g == 0 ? 0 : 1] + c * 4;
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        const f32x4_t x = *reinterpret_cast<const f32x4_t*>(mine + k * kCoreRow);
#pragma unroll
        for (int e = 0; e < 4; ++e) col[4 * k + e] = x[e];
    }
    float scale_c = 0.f, beta_c = 0.f, ibeta_c = 0.f;
    float gj, pj, gjj, alpha, irn;                        // row j of S and of A at this lane's column; the pivots
    bool some;
    auto pivot = [&](auto jc) {
        constexpr int j = decltype(jc)::value;
        first_two_rows(col[j], &gj, &pj);
        gjj = row_bcast<j>(gj); alpha = row_bcast<j>(pj);
        // hardware reciprocals and root (1 ulp), as in gram_panel_body.  Nothing left of a column (or less, by
        // rounding): zeros in R, and a reflector that keeps Q orthogonal; no Gaussian panel of 272 rows and more comes near it
        some = gjj > 0.f;
        irn = some ? __builtin_amdgcn_rsqf(gjj) : 0.f;
    };
    pivot(std::integral_constant<int, 0>{});
    static_for<NB>([&](auto jc) {
        constexpr int j = decltype(jc)::value;
        const float beta = -copysignf(gjj * irn, alpha), ibeta = -copysignf(irn, alpha);
        const float scale = some ? __builtin_amdgcn_rcpf(alpha - beta) : 0.f;
        const float later = g == 0 ? -gj * (irn * irn) : fmaf(gj, ibeta, -pj) * scale;
        // (L_ii^-1 grows column by column without its factor -scale_c)
        float down = g == 2 ? -scale * col[j] : 0.f;
        down = c > j ? later : (c == j ? 0.f : down);
        const float row = gj;
        __builtin_amdgcn_sched_barrier(0);
        // the next pivot's row first: its root is on its way while the other rows follow
        if constexpr (j + 1 < NB) {
            add_lane<j>(col[j + 1], down);
            pivot(std::integral_constant<int, j + 1>{});
        }
        __builtin_amdgcn_sched_barrier(0);
        add_column_around<j>(col, g == 2 ? 0.f : down, down);
        Rc[j] = c > j ? row * ibeta : (c == j ? beta : 0.f);
        if (c == j) { scale_c = scale; beta_c = beta; ibeta_c = ibeta; }
        if (g < 2) col[j] = c > j ? later : (c == j ? 1.f : col[j]);
        __builtin_amdgcn_sched_barrier(0);
    });
    // (selections only: the compiler makes branches of nested conditions)
    const bool low = g == 2;
    float m = scale_c;
    m = g == 0 ? ibeta_c : m;
    m = low ? -m : m;
    float* base = reinterpret_cast<float*>(&sh);
    auto place_of = [&](const float* t) { return (int)(t - base); };
    const int plain_0 = place_of(sh.DF), plain_1 = place_of(sh.DX), plain_2 = place_of(sh.PU[q][i]);
    const int turned_0 = place_of(sh.PR[q][i]), turned_1 = place_of(sh.PL[q][i]), turned_2 = place_of(sh.DL);
    int plain = low ? plain_2 : plain_1, turned = low ? turned_2 : turned_1;
    plain = (g == 0 ? plain_0 : plain) + c * 4;
    turned = (g == 0 ? turned_0 : turned) + (c >> 2) * kCoreRow + (c & 3);
    float out[NB];                                        // R_ii^-1, U_ii^-1, L_ii^-1
#pragma unroll
    for (int k = 0; k < NB; ++k) {
        col[k] *= m;
        const bool keep = (k > c) == low;
        const float one = ((k == c) & low) ? 1.f : 0.f;
        out[k] = keep ? col[k] : one;
    }
    if (g < 3) {
#pragma unroll
        for (int k = 0; k < 4; ++k) *reinterpret_cast<f32x4_t*>(base + plain + k * kCoreRow) = f32x4_t{out[4 * k], out[4 * k + 1], out[4 * k + 2], out[4 * k + 3]};
#pragma unroll
        for (int k = 0; k < NB; ++k) base[turned + k * 4] = out[k];
    }
    published();
    if (g == 1) {
#pragma unroll
        for (int k = 0; k < NB; ++k) { const float one = k == c ? 1.f : 0.f; col[k] = k > c ? col[k] : one; }
#pragma unroll
        for (int k = 0; k < 4; ++k) *reinterpret_cast<f32x4_t*>(Vtile + c * NB + 4 * k) = f32x4_t{col[4 * k], col[4 * k + 1], col[4 * k + 2], col[4 * k + 3]};
    }
    if (g == 0) {
#pragma unroll
        for (int k = 0; k < NB; ++k) Rd[i * 256 + k * NB + c] = Rc[k];
        rdiag[i * NB + c] = beta_c;
    }
}

// Waves go to the four SIMDs in turn: wave 3 eliminates, wave 7 leaves, so that it has a SIMD to itself (with two of the others
// beside it its 16 columns took 6700 cycles instead of 4900).
constexpr int kCoreThreads = 640;
template <int RANGES>
__device__ __forceinline__ void block_core(const BlockArgs& a, CoreShared& sh, int matrix) {
    const int tid = threadIdx.x, lane = tid & 63, number = __builtin_amdgcn_readfirstlane(tid >> 6);
    if (number == 7) return;
    const int wave = number == 3 ? BT : number < 3 ? number : number < 7 ? number - 1 : number - 2;
    const int c = lane & 15, g = lane >> 4;
    const int64_t off = (int64_t)matrix * a.w.batch_stride;
    float* X = a.w.X + off;
    float* core = a.core + off;
    auto tile = [&](int k, int l) { return X + ((int64_t)l * a.w.nbr + k) * 256; };
    auto gram = [&](int k, int l) {
        return sum_of_ranges<RANGES>(a.w.Wpart + off + ((int64_t)l * BT + k) * 256 + lane * 4, (int64_t)a.w.mt * BT * 256, a.w);
    };
    auto at = [&](float* p) { return reinterpret_cast<f32x4_t*>(p + g * kCoreRow + c * 4); };
    // scattered store of an accumulator tile, row-major
    auto rows = [&](float* p, f32x4_t v) {
#pragma unroll
        for (int e = 0; e < 4; ++e) p[(4 * g + e) * NB + c] = v[e];
    };
    const f32x4_t zero = {0.f, 0.f, 0.f, 0.f};
    // Both sides take the steps one by one and meet at the same two barriers: the diagonal tile of the step is finished; its row and
    // column are.  The elimination's loop is not unrolled: eight copies of its columns would be fetched from L2 as they run.
    if (wave == BT) {
        f32x4_t da = *reinterpret_cast<const f32x4_t*>(tile(0, 0) + c * NB + 4 * g), ds = gram(0, 0);
#pragma unroll 1
        for (int i = 0; i < BT; ++i) {
            const int q = i & 1, p = q ^ 1;
            if (i > 0) {
                da = tile_product(-*at(sh.PL[p][i]), *at(sh.PU[p][i]), *at(sh.DA[q]));
                ds = tile_product(-*at(sh.PR[p][i]), *at(sh.PR[p][i]), *at(sh.DS[q]));
            }
            int here = lane;
            asm volatile("" : "+v"(here));                // (its comparisons with the column would all be kept across the loop)
            core_diagonal(sh, q, i, da, ds, tile(i, i), a.Rd + off, a.rdiag + off, here, [&] { __syncthreads(); });
            __syncthreads();
        }
        return;
    }
    f32x4_t A[BT], S[BT];                                 // tiles (k, (wave - k) % 8)
#pragma unroll
    for (int k = 0; k < BT; ++k) {
        const int l = (wave - k) & 7;
        A[k] = S[k] = zero;
        if (k > l) {
#pragma unroll
            for (int e = 0; e < 4; ++e) A[k][e] = tile(k, l)[(4 * g + e) * NB + c];
        } else {
            A[k] = *reinterpret_cast<const f32x4_t*>(tile(k, l) + c * NB + 4 * g);
            S[k] = gram(k, l);
        }
        if (k % 2) __builtin_amdgcn_sched_barrier(0);     // (two tiles' requests at a time: more would not fit the registers)
    }
    // The part of a step that everyone waits for is a loop's body, fetched once; the products behind it exist once per step, with the
    // step known to the compiler, so that the tiles stay in registers.  The next step's tiles are picked out of them there.
    f32x4_t row_a = A[0], row_s = S[0], col_a = zero;
#pragma unroll
    for (int k = 0; k < BT; ++k) if (k == wave) col_a = A[k];
    if (((wave - 1) & 7) == 1) { *at(sh.DA[1]) = A[1]; *at(sh.DS[1]) = S[1]; }
#pragma unroll 1
    for (int i = 0; i < BT;) {
        const int q = i & 1, m = (wave - i) & 7;          // this wave's tiles (i, m) and (m, i)
        __syncthreads();                                  // the diagonal tile of step i is finished
        const f32x4_t r = tile_product(*at(sh.DF), row_s, zero);
        const f32x4_t v = tile_product(*at(sh.DX), col_a, zero);
        const f32x4_t u = tile_product(*at(sh.DL), m > i ? row_a - r : row_a, zero);
        const f32x4_t corner = *at(wave == 0 ? sh.DF : wave == 1 ? sh.DL : sh.DX);
        if (m != i) {
            *at(sh.PR[q][m]) = r;
            *at(sh.PL[q][m]) = v;
            *at(sh.PU[q][m]) = u;
        }
        __syncthreads();
        if (wave < 3) *reinterpret_cast<f32x4_t*>(core + (wave * kCoreTiles + i * BT + i) * 256 + c * NB + 4 * g) = corner;      // the diagonal tile's triangles
        if (m > i) {
            *reinterpret_cast<f32x4_t*>(tile(i, m) + c * NB + 4 * g) = r;
            rows(tile(m, i), v);                          // L's tile, column by column
        } else if (m < i) {
            rows(core + (i * BT + m) * 256, r);
            rows(core + (kCoreTiles + i * BT + m) * 256, u);
            rows(core + (2 * kCoreTiles + i * BT + m) * 256, v);
        }
        static_for<BT - 1>([&](auto bc) {
            constexpr int b = decltype(bc)::value, p = b & 1;
            if (i != b) return;
#pragma unroll
            for (int k = 0; k < BT; ++k) {                // step b's products; the next diagonal tile is the ninth wave's
                const int l = (wave - k) & 7;             // wave-uniform, as every condition here
                if (k == b + 1 && l == b + 1) continue;
                if (k > b && (l >= k || l <= b))
                    S[k] = tile_product(-*at(sh.PR[p][k]), *at(sh.PR[p][l]), l == b ? zero : S[k]);
                if (k > b || l > b) {
                    const bool swapped = l > b && (k <= b || k > l);
                    const f32x4_t x = *at(swapped ? sh.PU[p][l] : sh.PL[p][k]), y = *at(swapped ? sh.PL[p][k] : sh.PU[p][l]);
                    A[k] = tile_product(-x, y, (k > b && l == b) || (k == b && l > b) ? zero : A[k]);
                }
            }
            row_a = A[b + 1]; row_s = S[b + 1];
            const int next = (wave - (b + 1)) & 7;
#pragma unroll
            for (int k = 0; k < BT; ++k) if (k == next) col_a = A[k];
            if constexpr (b + 2 < BT) {
                if (((wave - (b + 2)) & 7) == b + 2) { *at(sh.DA[p]) = A[b + 2]; *at(sh.DS[p]) = S[b + 2]; }
            }
        });
        ++i;
        asm volatile("" : "+s"(i));                       // (the compiler would peel the first steps off)
    }
}

template <int RANGES>
__global__ __launch_bounds__(kCoreThreads)
void block_core_kernel(BlockArgs a) {
    extern __shared__ __attribute__((aligned(1024))) uint8_t lds[];
    block_core<RANGES>(a, *reinterpret_cast<CoreShared*>(lds), blockIdx.x);
}

// ------------------------------------------------------------ beside it: the columns further on --
// The columns behind the panel do not hold up its 128 x 128 part: while one workgroup is at that, the others bring them up to date with
// the block before (C <- C - Y2 N) and, with the rows still in registers, take P^T C of them.  A workgroup has eight tile columns,
// a wave each, of one range of rows (one part of ranges, many matrices); what they share, Y2's and P's fragments of 32 rows, goes through
// LDS, fetched by all ten waves a unit ahead.
struct OverlapArgs {
    BlockArgs b;                                          // w: the block's own, ranges of all columns
    const uint16_t* P;                                    // the panel taken apart; w.Yr, w.Wp: still those of the block before
    int core_slots, groups, items, per_item;              // workgroups before the others; groups of columns, ranges or parts, pairs of tile rows in each
};
constexpr int kOverlapWaves = kCoreThreads / 64;
constexpr int kOverlapFrags = 24 + 24;                    // of a unit: two tile rows of Y2, four units of three planes; three planes of eight tile columns of P
constexpr int kOverlapLds = 2 * kOverlapFrags * kFrag * 2;
static_assert(kOverlapLds >= (int)sizeof(CoreShared), "the core's share");

__device__ __forceinline__ void fetch_fragment(const uint16_t* from, uint32_t lds_addr) {      // lds_addr wave-uniform (travels in M0)
    asm volatile("s_mov_b32 m0, %1\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, off" :: "v"(from), "s"(lds_addr) : "memory", "m0");
}

__device__ __forceinline__ void columns_behind(const OverlapArgs& o, uint8_t* lds, int block) {
    const WideArgs& a = o.b.w;
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    int matrix, item;
    if (!deal_to_dies(block, o.groups * o.items, a.count, &matrix, &item)) return;
    const int cg = item / o.items, part = item % o.items;
    const int units = (a.mt + 1) / 2, t_begin = part * o.per_item, t_end = t_begin + o.per_item < units ? t_begin + o.per_item : units;
    const int own = BT + cg * 8 + wave, col = own < a.mt ? own : a.mt - 1;
    const bool works = wave < 8, there = works && own < a.mt;
    const uint32_t base = __builtin_amdgcn_readfirstlane((uint32_t)(size_t)lds);
    const uint16_t* Yr = a.Yr + 2 * (int64_t)matrix * a.batch_stride + lane * 8;
    const uint16_t* P = o.P + 2 * (int64_t)matrix * a.batch_stride + lane * 8;
    float* x_at = a.X + (int64_t)matrix * a.batch_stride + (int64_t)col * a.nbr * 256 + (lane & 15) * NB + 4 * (lane >> 4);
    auto fetch = [&](int t, int buf) {
#pragma unroll
        for (int i = 0; i < (kOverlapFrags + kOverlapWaves - 1) / kOverlapWaves; ++i) {
            const int id = wave + kOverlapWaves * i;
            if (id >= kOverlapFrags) continue;            // wave-uniform
            const int e = id / 12, row = 2 * t + e < a.mt ? 2 * t + e : a.mt - 1;       // the odd last tile row: P is zero there
            const uint16_t* from = id < 24 ? Yr + (int64_t)row * kYrBlock + (id - 12 * e) * kFrag : P + (int64_t)t * kUnitPanel + (id - 24) * kFrag;
            fetch_fragment(from, base + (uint32_t)((buf * kOverlapFrags + id) * kFrag * 2));
        }
    };
    auto load = [&](int t, f32x4_t (&x)[2]) {
#pragma unroll
        for (int e = 0; e < 2; ++e) {
            const int r = 2 * t + e < a.mt ? 2 * t + e : a.mt - 1;
            x[e] = *reinterpret_cast<const f32x4_t*>(x_at + (int64_t)r * 256);
        }
    };
    Split n[BT / 2][1];                                   // -N of this wave's column
    f32x4_t x[2], acc[2][4][1];
    if (works) {
        const uint16_t* w = a.Wp + 2 * (int64_t)matrix * a.batch_stride + (int64_t)col * a.wp_unit + lane * 8;
#pragma unroll
        for (int u = 0; u < BT / 2; ++u) { n[u][0].h = frag_of(w + u * 3 * kFrag); n[u][0].m = frag_of(w + (u * 3 + 1) * kFrag); n[u][0].l = frag_of(w + (u * 3 + 2) * kFrag); }
        load(t_begin, x);
    }
    fetch(t_begin, 0);
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");      // (from here on the fetches are counted by what is issued behind them)
    float* sums = a.Wpart + (int64_t)matrix * a.batch_stride + ((int64_t)part * a.mt + col) * BT * 256 + lane * 4;
    int in_range = 0;                                     // units of the present range that are done
    bool first = true;
    for (int t = t_begin; t < t_end; ++t) {
        const int buf = (t - t_begin) & 1;
        // This unit's fragments have landed (two loads at least were issued behind them), nobody reads the other stage any more
        if (works) asm volatile("s_waitcnt vmcnt(2) lgkmcnt(0)" ::: "memory");
        else asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        __builtin_amdgcn_s_barrier();
        asm volatile("" ::: "memory");
        if (t + 1 < t_end) fetch(t + 1, buf ^ 1);
        if (works) {
            f32x4_t ahead[2];
            load(t + 1 < t_end ? t + 1 : t, ahead);
            const uint16_t* mine = reinterpret_cast<const uint16_t*>(lds) + buf * kOverlapFrags * kFrag + lane * 8;
            f32x4_t change[2][1];
            change[0][0] = change[1][0] = f32x4_t{0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int u = 0; u < BT / 2; ++u) products([&](int plane, int f) { return frag_of(mine + ((f * (BT / 2) + u) * 3 + plane) * kFrag); }, n[u], change);
#pragma unroll
            for (int e = 0; e < 2; ++e) x[e] = x[e] + change[e][0];
            Split xs[1];
            xs[0] = split3(x[0], x[1]);
            if (in_range == 0) {
#pragma unroll
                for (int h = 0; h < 2; ++h)
#pragma unroll
                    for (int f = 0; f < 4; ++f) acc[h][f][0] = f32x4_t{0.f, 0.f, 0.f, 0.f};
            }
#pragma unroll
            for (int h = 0; h < 2; ++h) products([&](int plane, int f) { return frag_of(mine + (24 + plane * 8 + 4 * h + f) * kFrag); }, xs, acc[h]);
            if (there) {
#pragma unroll
                for (int e = 0; e < 2; ++e) if (2 * t + e < a.mt) *reinterpret_cast<f32x4_t*>(x_at + (int64_t)(2 * t + e) * 256) = x[e];
            }
            if (++in_range == a.per_chunk || t + 1 == t_end) {
                if (there) {
#pragma unroll
                    for (int f = 0; f < BT; ++f) {
                        f32x4_t* at = reinterpret_cast<f32x4_t*>(sums + f * 256);
                        *at = first ? acc[f / 4][f % 4][0] : *at + acc[f / 4][f % 4][0];
                    }
                }
                first = false; in_range = 0;
            }
            x[0] = ahead[0]; x[1] = ahead[1];
        }
    }
}

__global__ __launch_bounds__(kCoreThreads)
void block_overlap_kernel(OverlapArgs o) {
    extern __shared__ __attribute__((aligned(1024))) uint8_t lds[];
    if ((int)blockIdx.x >= o.core_slots) { columns_behind(o, lds, blockIdx.x - o.core_slots); return; }
    if ((int)blockIdx.x < o.b.w.count) block_core<kWideChunks>(o.b, *reinterpret_cast<CoreShared*>(lds), blockIdx.x);
}

// ------------------------------------------------------------ the columns behind the block, the rows below it --
// Workgroup b < mt - 8: tile column 8 + b of the rows of the block (R1 in its place, -N taken apart); the next mt - 8: tile row 8 +
// b' of the panel (Y2 in its place, and taken apart).  A wave per tile of the block.
template <int RANGES>
__global__ __launch_bounds__(512)
void block_apply_kernel(BlockArgs a) {
    __shared__ __attribute__((aligned(16))) float part[2][BT][256];
    const int tid = threadIdx.x, lane = tid & 63, i = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int c = lane & 15, g = lane >> 4, behind = a.w.mt - BT;
    const int64_t off = (int64_t)blockIdx.y * a.w.batch_stride;
    const float* core = a.core + off + i * BT * 256 + c * NB + 4 * g;
    f32x4_t t[2][BT];
    f32x4_t acc = {0.f, 0.f, 0.f, 0.f};
    if ((int)blockIdx.x < behind) {
        const int col = BT + blockIdx.x;
        float* x = a.w.X + off + ((int64_t)col * a.w.nbr + i) * 256 + c * NB + 4 * g;
        const f32x4_t c1 = *reinterpret_cast<const f32x4_t*>(x);
        const f32x4_t s = sum_of_ranges<RANGES>(a.w.Wpart + off + ((int64_t)col * BT + i) * 256 + lane * 4, (int64_t)a.w.mt * BT * 256, a.w);
#pragma unroll
        for (int l = 0; l < BT; ++l)
            if (l <= i) { t[0][l] = *reinterpret_cast<const f32x4_t*>(core + l * 256); t[1][l] = *reinterpret_cast<const f32x4_t*>(core + (kCoreTiles + l) * 256); }
        *reinterpret_cast<f32x4_t*>(&part[0][i][lane * 4]) = s;
        __syncthreads();
#pragma unroll
        for (int l = 0; l < BT; ++l) if (l <= i) acc = tile_product(t[0][l], *reinterpret_cast<const f32x4_t*>(&part[0][l][lane * 4]), acc);
        *reinterpret_cast<f32x4_t*>(x) = acc;
        *reinterpret_cast<f32x4_t*>(&part[1][i][lane * 4]) = c1 - acc;
        __syncthreads();
        acc = f32x4_t{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int l = 0; l < BT; ++l) if (l <= i) acc = tile_product(t[1][l], *reinterpret_cast<const f32x4_t*>(&part[1][l][lane * 4]), acc);
        *reinterpret_cast<f32x4_t*>(&part[0][i][lane * 4]) = -acc;
        __syncthreads();
        if (i < BT / 2)
            put_split(a.w.Wp + 2 * off + (int64_t)blockIdx.x * a.w.wp_unit + i * 3 * kFrag + lane * 8, kFrag,
                      split3(*reinterpret_cast<const f32x4_t*>(&part[0][2 * i][lane * 4]), *reinterpret_cast<const f32x4_t*>(&part[0][2 * i + 1][lane * 4])));
    } else {
        const int row = blockIdx.x - behind;              // of those below the block
        float* x = a.w.X + off + (int64_t)(BT + row) * 256 + c;
        // Y2^T = U^-T P2^T: the panel's tiles turned around as they are read
        f32x4_t y[BT];
#pragma unroll
        for (int l = 0; l < BT; ++l)
            if (l <= i) {
                t[0][l] = *reinterpret_cast<const f32x4_t*>(core + (2 * kCoreTiles + l) * 256);
#pragma unroll
                for (int e = 0; e < 4; ++e) y[l][e] = x[(int64_t)l * a.w.nbr * 256 + (4 * g + e) * NB];
            }
#pragma unroll
        for (int l = 0; l < BT; ++l) if (l <= i) acc = tile_product(t[0][l], y[l], acc);
        *reinterpret_cast<f32x4_t*>(&part[0][i][lane * 4]) = acc;
        __syncthreads();                                  // every wave has read what it needs of the panel
#pragma unroll
        for (int e = 0; e < 4; ++e) x[(int64_t)i * a.w.nbr * 256 + (4 * g + e) * NB] = acc[e];
        if (i < BT / 2)
            put_split(a.Yr + 2 * off + (int64_t)row * kYrBlock + i * 3 * kFrag + lane * 8, kFrag,
                      split3(*reinterpret_cast<const f32x4_t*>(&part[0][2 * i][lane * 4]), *reinterpret_cast<const f32x4_t*>(&part[0][2 * i + 1][lane * 4])));
    }
}

// the first panel taken apart (the later ones: launch_block_update)
__global__ __launch_bounds__(512)
void first_panel_kernel(const float* M, uint16_t* out, int nbr, int64_t batch_stride) {
    const int tid = threadIdx.x, lane = tid & 63, f = __builtin_amdgcn_readfirstlane(tid >> 6);
    const float* t = M + (int64_t)blockIdx.y * batch_stride + ((int64_t)f * nbr + 2 * blockIdx.x) * 256 + (lane & 15) * NB + 4 * (lane >> 4);
    const f32x4_t v0 = *reinterpret_cast<const f32x4_t*>(t);
    f32x4_t v1 = {0.f, 0.f, 0.f, 0.f};
    if (2 * (int)blockIdx.x + 1 < nbr) v1 = *reinterpret_cast<const f32x4_t*>(t + 256);
    put_split(out + 2 * (int64_t)blockIdx.y * batch_stride + (int64_t)blockIdx.x * kUnitPanel + f * kFrag + lane * 8, 8 * kFrag, split3(v0, v1));
}

// T of every panel of 16 finished reflectors, from V^T V in double precision (see gram_panel_body), and V row by row (Vc, unless it is
// null): a workgroup per panel
__global__ __launch_bounds__(512)
void panel_triangle_kernel(const float* M, float* Vc, float* Tmat, int nbr, int64_t batch_stride) {
    __shared__ double part[8][256];
    __shared__ __attribute__((aligned(16))) float m[NB * kTurn];
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int c = lane & 15, g = lane >> 4, f = blockIdx.x;
    const float* v = M + (int64_t)blockIdx.y * batch_stride + (int64_t)f * nbr * 256 + c * NB + 4 * g;
    f64x4_t acc = {0., 0., 0., 0.};
    for (int r = f + wave; r < nbr; r += 8) {
        const f32x4_t x = *reinterpret_cast<const f32x4_t*>(v + (int64_t)r * 256);
        if (Vc != nullptr) {
            float* row = Vc + (int64_t)blockIdx.y * batch_stride + ((int64_t)f * nbr + r - f) * 256 + 4 * g * NB + c;
#pragma unroll
            for (int e = 0; e < 4; ++e) row[e * NB] = x[e];
        }
#pragma unroll
        for (int e = 0; e < 4; ++e) acc = __builtin_amdgcn_mfma_f64_16x16x4f64((double)x[e], (double)x[e], acc, 0, 0, 0);
    }
#pragma unroll
    for (int e = 0; e < 4; ++e) part[wave][(4 * e + g) * NB + c] = acc[e];        // the double instruction: element e is row 4 e + g
    __syncthreads();
    if (tid < 256) {
        double s = part[0][tid];
#pragma unroll
        for (int w = 1; w < 8; ++w) s += part[w][tid];
        m[(tid & 15) * kTurn + (tid >> 4)] = (float)s;
    }
    __syncthreads();
    if (wave > 0) return;
    float Mc[NB], Tc[NB], tau_c = 0.f;
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        const f32x4_t x = *reinterpret_cast<const f32x4_t*>(m + c * kTurn + 4 * k);
#pragma unroll
        for (int e = 0; e < 4; ++e) Mc[4 * k + e] = x[e];
    }
#pragma unroll
    for (int k = 0; k < NB; ++k) { Tc[k] = k == c ? 1.f : 0.f; tau_c = k == c ? 2.f / Mc[k] : tau_c; }
    static_for<NB - 1>([&](auto jc) {
        constexpr int j = decltype(jc)::value;
        const float tau = row_bcast<j>(tau_c);
        add_column<j, 0, j + 1>(Tc, c > j ? -Mc[j] * tau : 0.f);
    });
    const f32x4_t t = rows_of_group(Tc, g);
    float* out = Tmat + (int64_t)blockIdx.y * batch_stride + (int64_t)f * 256;
#pragma unroll
    for (int e = 0; e < 4; ++e) out[(4 * g + e) * NB + c] = t[e] * tau_c;
}

#define GELO_TRY(expr) do { hipError_t e_ = (expr); if (e_ != hipSuccess) return e_; } while (0)

}  // namespace

int64_t block_panel_values(int n_pad) { return (int64_t)((n_pad / NB + 1) / 2) * kUnitPanel; }

hipError_t block_factor_init() {    // brings this file's code onto the device (see factor_init)
    return hipFuncSetAttribute(reinterpret_cast<const void*>(&block_overlap_kernel), hipFuncAttributeMaxDynamicSharedMemorySize, kOverlapLds);
}

hipError_t factor_blocks(const FactorWorkspace& ws, float* Vc, int count, int64_t batch_stride, int* panels_done, hipStream_t s) {
    const int nbr = ws.n_pad / NB;
    int done = 0;
    hipLaunchKernelGGL(first_panel_kernel, dim3((nbr + 1) / 2, count), dim3(512), 0, s, ws.M, ws.panel, nbr, batch_stride);
    GELO_TRY(hipGetLastError());
    WideArgs update;                                          // the last block's, where it has not been applied yet
    for (const int last = last_block_tiles(nbr); nbr - done >= last; done += BT) {
        OverlapArgs o;
        BlockArgs& b = o.b;
        WideArgs& a = b.w;
        a.nbr = nbr; a.t0 = done; a.mt = a.cols = nbr - done; a.nt = BT;
        a.Yp = ws.panel; a.T = nullptr;
        a.X = ws.M + ((int64_t)done * nbr + done) * 256;
        a.Wpart = ws.Wpart; a.Wp = ws.Wp; a.wp_unit = a.yr_unit = kYrBlock;
        a.next = nullptr;
        a.batch_stride = batch_stride; a.count = count;
        a.Yr = b.Yr = ws.Yr;
        o.groups = (a.mt - BT + 7) / 8;
        cut_into_ranges(a, 1, done == 0 ? (a.mt + 3) / 4 : o.groups);
        b.core = ws.core; b.Rd = ws.Rd + (int64_t)done * 256; b.rdiag = ws.rdiag + done * NB;
        if (done == 0) {
            GELO_TRY(launch_panel_products(a, s));
            if (a.by_part) hipLaunchKernelGGL((block_core_kernel<kWideParts>), dim3(count), dim3(kCoreThreads), sizeof(CoreShared), s, b);
            else hipLaunchKernelGGL((block_core_kernel<kWideChunks>), dim3(count), dim3(kCoreThreads), sizeof(CoreShared), s, b);
        } else {
            update.cols = BT; update.next = ws.panel;
            GELO_TRY(launch_block_update(update, s));
            WideArgs own = a;
            own.cols = BT; own.groups = 1; own.by_part = false;      // few columns: ranges fill the chip
            GELO_TRY(launch_panel_products(own, s));
            o.P = ws.panel;
            o.core_slots = (count + 7) / 8 * 8;
            o.items = a.by_part ? a.parts : a.chunks;
            o.per_item = a.by_part ? a.per_chunk * a.part_chunks : a.per_chunk;
            const dim3 grid(o.core_slots + 8 * dies_slots(o.groups * o.items, count));
            hipLaunchKernelGGL(block_overlap_kernel, grid, dim3(kCoreThreads), kOverlapLds, s, o);
        }
        GELO_TRY(hipGetLastError());
        if (a.by_part) hipLaunchKernelGGL((block_apply_kernel<kWideParts>), dim3(2 * (a.mt - BT), count), dim3(512), 0, s, b);
        else hipLaunchKernelGGL((block_apply_kernel<kWideChunks>), dim3(2 * (a.mt - BT), count), dim3(512), 0, s, b);
        GELO_TRY(hipGetLastError());
        update = a;
        update.X += (int64_t)BT * nbr * 256 + BT * 256;
        update.mt -= BT; update.cols = update.mt; update.t0 += BT;
    }
    if (done > 0) GELO_TRY(launch_block_update(update, s));
    if (done > 0) {
        hipLaunchKernelGGL(panel_triangle_kernel, dim3(done, count), dim3(512), 0, s, ws.M, Vc, ws.Tmat, nbr, batch_stride);
        GELO_TRY(hipGetLastError());
    }
    *panels_done = done;
    return hipSuccess;
}

}  // namespace gelo

// Householder QR by ONE workgroup, the matrix in registers: a wave per tile column (16 columns), the tiles in the accumulator
// layout of v_mfma_f32_16x16x4_f32, lane (g, c): rows 4 g .. 4 g + 3 of column c.
//
// Wave w factorises its 16 columns without leaving its registers (columns_qr): lane (g, c) walks its rows of column c for the
// inner product with column j, whose elements come by the multiply-add's own row broadcast; four lanes' sums meet, and the same walk
// applies the reflector.  Then the 16 reflectors and their triangle lie in LDS, the workgroup meets at a barrier, and every wave
// behind w applies them to its tiles on the matrix cores (apply_reflectors) while wave w + 1, first in line, goes on to its own columns.
#pragma once

#include "wave_tile.h"

namespace gelo {

// LDS tiles: column c at 16 tile_slot(c), its rows in order: 16-byte reads of a column's rows, and 4-byte reads of four columns of one
// row, meet no bank twice.
__device__ __forceinline__ int tile_slot(int c) { return (c & ~3) | ((c + (c >> 2)) & 3); }
constexpr int kTurnPitch = kPanel + 4;                    // of a tile that is turned around: rows by 16 bytes, columns by 4

// Of `tiles` tile columns: the reflectors of tile column p, tiles p .. of it.
__host__ __device__ inline int tile_qr_before(int tiles, int p) { return p * tiles - p * (p - 1) / 2; }
// U, a tile of zeros, two triangles, a tile to turn around in
__host__ __device__ inline int tile_qr_floats(int tiles) { return (tile_qr_before(tiles, tiles) + 1 + 2) * 256 + kPanel * kTurnPitch; }
struct TileQrShared {
    float *U, *zero, *T, *turn;
    int tiles;
    __device__ __forceinline__ TileQrShared(float* base, int tiles_) : tiles(tiles_) {
        U = base;
        zero = U + tile_qr_before(tiles, tiles) * 256;
        T = zero + 256; turn = T + 512;
    }
    __device__ __forceinline__ float* tile(int p, int i) const { return U + (tile_qr_before(tiles, p) + i - p) * 256; }
};

// ------------------------------------------------------------ 16 columns in registers --
// What a step does to a tile whose rows all lie below the pivot: a0, a1 += x_j x, and x += f x_j (f = 0 in lane j), x_j the
// value of lane J of the row of 16.  A register that a row broadcast reads must not have been written by one of the two instructions in front.
#define GELO_DOT(a, x) "v_fmac_f32_dpp %" #a ", %" #x ", %" #x " row_newbcast:%c18 row_mask:0xf bank_mask:0xf\n\t"
template <int J, int F, int N>
__device__ __forceinline__ void dot_tiles(float& a0, float& a1, const float (&y)[N]) {
    auto at = [&](int k) { return y[4 * F + k < N ? 4 * F + k : N - 1]; };
    if constexpr (4 * F + 15 < N)
        asm("s_nop 1\n\t" GELO_DOT(0, 2) GELO_DOT(1, 3) GELO_DOT(0, 4) GELO_DOT(1, 5) GELO_DOT(0, 6) GELO_DOT(1, 7) GELO_DOT(0, 8) GELO_DOT(1, 9)
            GELO_DOT(0, 10) GELO_DOT(1, 11) GELO_DOT(0, 12) GELO_DOT(1, 13) GELO_DOT(0, 14) GELO_DOT(1, 15) GELO_DOT(0, 16) GELO_DOT(1, 17)
            : "+v"(a0), "+v"(a1)
            : "v"(at(0)), "v"(at(1)), "v"(at(2)), "v"(at(3)), "v"(at(4)), "v"(at(5)), "v"(at(6)), "v"(at(7)), "v"(at(8)), "v"(at(9)), "v"(at(10)),
              "v"(at(11)), "v"(at(12)), "v"(at(13)), "v"(at(14)), "v"(at(15)), "n"(J));
}
#undef GELO_DOT
#define GELO_DOT(a, x) "v_fmac_f32_dpp %" #a ", %" #x ", %" #x " row_newbcast:%c6 row_mask:0xf bank_mask:0xf\n\t"
template <int J>
__device__ __forceinline__ void dot_tile(float& a0, float& a1, float y0, float y1, float y2, float y3) {
    asm("s_nop 1\n\t" GELO_DOT(0, 2) GELO_DOT(1, 3) GELO_DOT(0, 4) GELO_DOT(1, 5) : "+v"(a0), "+v"(a1) : "v"(y0), "v"(y1), "v"(y2), "v"(y3), "n"(J));
}
#undef GELO_DOT
// the pivot's own tile: only the rows below it, which the mask of rows of 16 lanes takes
#define GELO_DOT(a, x, e) ".if %c" #e "\n\tv_fmac_f32_dpp %" #a ", %" #x ", %" #x " row_newbcast:%c6 row_mask:%c" #e " bank_mask:0xf\n.endif\n\t"
template <int J>
__device__ __forceinline__ void dot_first(float& a0, float& a1, float y0, float y1, float y2, float y3) {
    constexpr int q = J / 4, e = J % 4, from = (0xf << q) & 0xf, behind = (0xf << (q + 1)) & 0xf;
    asm("s_nop 1\n\t" GELO_DOT(0, 2, 7) GELO_DOT(1, 3, 8) GELO_DOT(0, 4, 9) GELO_DOT(1, 5, 10)
        : "+v"(a0), "+v"(a1) : "v"(y0), "v"(y1), "v"(y2), "v"(y3), "n"(J), "n"(0 > e ? from : behind), "n"(1 > e ? from : behind), "n"(2 > e ? from : behind),
          "n"(3 > e ? from : behind));
}
#undef GELO_DOT
#define GELO_ADD(x, e) ".if %c" #e "\n\tv_fmac_f32_dpp %" #x ", %" #x ", %4 row_newbcast:%c6 row_mask:%c" #e " bank_mask:0xf\n.endif\n\t"
#define GELO_TOP(x) ".if %c11 == " #x "\n\tv_fmac_f32_dpp %" #x ", %5, %4 quad_perm:[0,1,2,3] row_mask:%c12 bank_mask:0xf\n.endif\n\t"
template <int J>
__device__ __forceinline__ void add_first(float& y0, float& y1, float& y2, float& y3, float f, float ut) {
    constexpr int q = J / 4, e = J % 4, from = (0xf << q) & 0xf, behind = (0xf << (q + 1)) & 0xf;
    asm("s_nop 1\n\t" GELO_ADD(0, 7) GELO_ADD(1, 8) GELO_ADD(2, 9) GELO_ADD(3, 10) GELO_TOP(0) GELO_TOP(1) GELO_TOP(2) GELO_TOP(3) "s_nop 1"
        : "+v"(y0), "+v"(y1), "+v"(y2), "+v"(y3)
        : "v"(f), "v"(ut), "n"(J), "n"(0 > e ? from : behind), "n"(1 > e ? from : behind), "n"(2 > e ? from : behind), "n"(3 > e ? from : behind),
          "n"(e), "n"(1 << q));
}
#undef GELO_ADD
#undef GELO_TOP
#define GELO_ADD(x) "v_fmac_f32_dpp %" #x ", %" #x ", %4 row_newbcast:%c5 row_mask:0xf bank_mask:0xf\n\t"
template <int J>
__device__ __forceinline__ void add_tile(float& y0, float& y1, float& y2, float& y3, float f) {
    asm("s_nop 1\n\t" GELO_ADD(0) GELO_ADD(1) GELO_ADD(2) GELO_ADD(3) : "+v"(y0), "+v"(y1), "+v"(y2), "+v"(y3) : "v"(f), "n"(J));
}
#undef GELO_ADD
#define GELO_ADD(x) "v_fmac_f32_dpp %" #x ", %" #x ", %16 row_newbcast:%c17 row_mask:0xf bank_mask:0xf\n\t"
template <int J, int F, int N>
__device__ __forceinline__ void add_tiles(float (&y)[N], float f) {
    if constexpr (4 * F + 15 < N)
        asm("s_nop 1\n\t" GELO_ADD(0) GELO_ADD(1) GELO_ADD(2) GELO_ADD(3) GELO_ADD(4) GELO_ADD(5) GELO_ADD(6) GELO_ADD(7) GELO_ADD(8) GELO_ADD(9)
            GELO_ADD(10) GELO_ADD(11) GELO_ADD(12) GELO_ADD(13) GELO_ADD(14) GELO_ADD(15)
            : "+v"(y[4 * F]), "+v"(y[4 * F + 1]), "+v"(y[4 * F + 2]), "+v"(y[4 * F + 3]), "+v"(y[4 * F + 4]), "+v"(y[4 * F + 5]), "+v"(y[4 * F + 6]),
              "+v"(y[4 * F + 7]), "+v"(y[4 * F + 8]), "+v"(y[4 * F + 9]), "+v"(y[4 * F + 10]), "+v"(y[4 * F + 11]), "+v"(y[4 * F + 12]), "+v"(y[4 * F + 13]),
              "+v"(y[4 * F + 14]), "+v"(y[4 * F + 15])
            : "v"(f), "n"(J));
}
#undef GELO_ADD

// Householder QR of TC tiles of 16 columns, y[4 b + e] row 16 b + 4 g + e of the lane's column.  On return R above the diagonal, u below
// it; of the lane's column u's entry on the diagonal, R's, and whether there is anything to reflect (the reflector is I - 2 u u^T / u^T u).
struct ColumnEnds { float ut, r; bool some; };
template <int TC, int N>
__device__ __forceinline__ ColumnEnds columns_qr(float (&y)[N], int c) {
    static_assert(4 * TC <= N, "tiles that are not there");
    constexpr int GROUPS = (TC - 1) / 4;                  // of four tiles below the first; what is left over one by one
    float pivot_c = 0.f, below_c = 0.f;
    static_for<kPanel>([&](auto jc) {
        constexpr int j = decltype(jc)::value;
        const float p = row_to_all<j / 4>(y[j % 4]);      // the pivot's row
        float a0 = 0.f, a1 = 0.f;
        // from the bottom up: u's large entry on the diagonal comes last
        static_for<TC - 1 - 4 * GROUPS>([&](auto kc) { constexpr int k = 4 * (TC - 1 - decltype(kc)::value); dot_tile<j>(a0, a1, y[k], y[k + 1], y[k + 2], y[k + 3]); });
        static_for<GROUPS>([&](auto bc) { dot_tiles<j, 1 + 4 * (GROUPS - 1 - decltype(bc)::value)>(a0, a1, y); });
        dot_first<j>(a0, a1, y[0], y[1], y[2], y[3]);
        const float below = sum_of_rows(a0 + a1);         // x_j^T x of the rows below the pivot's
        const float alpha = row_bcast<j>(p), nn = row_bcast<j>(below);
        const float nrm = __builtin_amdgcn_sqrtf(fmaf(alpha, alpha, nn));      // hardware root and reciprocal (1 ulp)
        const float ut = alpha + copysignf(nrm, alpha);
        const float uu = fmaf(ut, ut, nn), r = __builtin_amdgcn_rcpf(uu);
        float inv = 2.f * fmaf(fmaf(-uu, r, 1.f), r, r);
        inv = nn > 0.f ? inv : 0.f;
        const float d = fmaf(ut, p, below);               // u^T x
        const float f = c > j ? -inv * d : 0.f;
        add_first<j>(y[0], y[1], y[2], y[3], f, ut);
        static_for<GROUPS>([&](auto bc) { add_tiles<j, 1 + 4 * decltype(bc)::value>(y, f); });
        static_for<TC - 1 - 4 * GROUPS>([&](auto kc) { constexpr int k = 4 * (1 + 4 * GROUPS + decltype(kc)::value); add_tile<j>(y[k], y[k + 1], y[k + 2], y[k + 3], f); });
        pivot_c = c == j ? p : pivot_c;
        below_c = c == j ? below : below_c;
    });
    ColumnEnds ends;
    const float nrm = __builtin_amdgcn_sqrtf(fmaf(pivot_c, pivot_c, below_c));
    ends.ut = pivot_c + copysignf(nrm, pivot_c);
    ends.some = below_c > 0.f;
    ends.r = ends.some ? -copysignf(nrm, pivot_c) : pivot_c;
    return ends;
}

// The triangle T of I - U T U^T = H_0 H_1 .., from U^T U in double precision: what the orthogonality of I - U T U^T is lost to is
// U^T U's rounding.  The same T takes the columns behind to R and forms Q.  (The inner products that the walks leave anyhow are
// float: 6 us of 103 at 129 rows less with a T from those for R, and 1 to 3% more of A^T G below the diagonal, 44 to 160 rows.)  u: the
// reflectors in accumulator layout, zeros above their diagonal; turn: kPanel x kTurnPitch floats.  Returns T in accumulator layout.
template <int TC, int N>
__device__ __forceinline__ f32x4_t exact_triangle(const float (&u)[N], bool some, float* turn, int lane) {
    const int c = lane & 15, g = lane >> 4;
    f64x4_t m0 = {0., 0., 0., 0.}, m1 = {0., 0., 0., 0.};
#pragma unroll
    for (int k = 0; k < 4 * TC; k += 2) {
        m0 = __builtin_amdgcn_mfma_f64_16x16x4f64((double)u[k], (double)u[k], m0, 0, 0, 0);
        m1 = __builtin_amdgcn_mfma_f64_16x16x4f64((double)u[k + 1], (double)u[k + 1], m1, 0, 0, 0);
    }
#pragma unroll
    for (int v = 0; v < 4; ++v) turn[c * kTurnPitch + 4 * v + g] = (float)(m0[v] + m1[v]);      // element v: row 4 v + g
    __builtin_amdgcn_wave_barrier();
    float Mc[kPanel], Tc[kPanel], tau_c = 0.f;
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        const f32x4_t x = *reinterpret_cast<const f32x4_t*>(turn + c * kTurnPitch + 4 * k);
#pragma unroll
        for (int e = 0; e < 4; ++e) Mc[4 * k + e] = x[e];
    }
    __builtin_amdgcn_wave_barrier();
#pragma unroll
    for (int i = 0; i < kPanel; ++i) { Tc[i] = i == c ? 1.f : 0.f; tau_c = i == c ? Mc[i] : tau_c; }
    tau_c = some ? 2.f / tau_c : 0.f;
    static_for<kPanel - 1>([&](auto jc) {
        constexpr int j = decltype(jc)::value;
        const float tau = row_bcast<j>(tau_c);            // (outside of the selection: all lanes have to be active)
        add_column<j, 0, j + 1>(Tc, c > j ? -Mc[j] * tau : 0.f);
    });
    f32x4_t t = rows_of_group(Tc, g);
#pragma unroll
    for (int e = 0; e < 4; ++e) t[e] *= tau_c;
    return t;
}

// X <- (I - U T U^T)^T X for the reflectors of tile column p and a wave's tiles p .. nbt - 1; x[4 i + e]: row 16 i + 4 g + e of its column;
// T: a tile in LDS, column after column.  U T^T U^T X is summed by itself and subtracted once.
template <int NT>
__device__ __forceinline__ void apply_reflectors(const TileQrShared& sh, float (&x)[4 * NT], const float* T, int p, int nbt, int lane) {
    constexpr int GRP = 2, NG = (NT + GRP - 1) / GRP;
    const int c = lane & 15, g = lane >> 4;
    const int down = 16 * tile_slot(c) + 4 * g;
    int across[4];
#pragma unroll
    for (int e = 0; e < 4; ++e) across[e] = 16 * tile_slot(4 * g + e) + c;
    // everything is on its way at once; tiles that are not there are zeros
    f32x4_t a[NT];
    float b[NT][4];
#pragma unroll
    for (int i = NT - 1; i >= 0; --i) a[i] = *reinterpret_cast<const f32x4_t*>((i >= p && i < nbt ? sh.tile(p, i) : sh.zero) + down);
    const f32x4_t t = *reinterpret_cast<const f32x4_t*>(T + c * 16 + 4 * g);
#pragma unroll
    for (int i = 0; i < NT; ++i)
#pragma unroll
        for (int e = 0; e < 4; ++e) b[i][e] = (i >= p && i < nbt ? sh.tile(p, i) : sh.zero)[across[e]];
    __builtin_amdgcn_sched_barrier(0);
    f32x4_t w[2] = {{0.f, 0.f, 0.f, 0.f}, {0.f, 0.f, 0.f, 0.f}};
    static_for<NG>([&](auto gc) {
        constexpr int i0 = GRP * (NG - 1 - decltype(gc)::value);
        if (i0 + GRP <= p || i0 >= nbt) return;           // wave-uniform
#pragma unroll
        for (int k = GRP - 1; k >= 0; --k)
            if (i0 + k < NT)
#pragma unroll
                for (int e = 0; e < 4; ++e) w[e & 1] = __builtin_amdgcn_mfma_f32_16x16x4f32(a[i0 + k < NT ? i0 + k : 0][e], x[i0 + k < NT ? 4 * (i0 + k) + e : 0], w[e & 1], 0, 0, 0);
    });
    const f32x4_t sum = w[0] + w[1];
    f32x4_t s0 = {0.f, 0.f, 0.f, 0.f}, s1 = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int e = 0; e < 4; e += 2) {
        s0 = __builtin_amdgcn_mfma_f32_16x16x4f32(t[e], sum[e], s0, 0, 0, 0);
        s1 = __builtin_amdgcn_mfma_f32_16x16x4f32(t[e + 1], sum[e + 1], s1, 0, 0, 0);
    }
    const f32x4_t s = -(s0 + s1);
    static_for<NG>([&](auto gc) {
        constexpr int i0 = GRP * decltype(gc)::value;
        if (i0 + GRP <= p || i0 >= nbt) return;
        f32x4_t acc[GRP];
#pragma unroll
        for (int k = 0; k < GRP; ++k) acc[k] = f32x4_t{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int e = 0; e < 4; ++e)
#pragma unroll
            for (int k = 0; k < GRP; ++k) if (i0 + k < NT) acc[k] = __builtin_amdgcn_mfma_f32_16x16x4f32(b[i0 + k < NT ? i0 + k : 0][e], s[e], acc[k], 0, 0, 0);
#pragma unroll
        for (int k = 0; k < GRP; ++k)
            if (i0 + k < NT)
#pragma unroll
                for (int e = 0; e < 4; ++e) x[4 * (i0 + k) + e] += acc[k][e];
    });
}

// tile b <- tile b + by, what is behind the end cleared; above(i): those before tile i + 1 = by are still there
template <int NT, class Above>
__device__ __forceinline__ void shift_tiles(float (&x)[4 * NT], int by, Above&& above) {
    static_for<NT - 1>([&](auto ic) {
        constexpr int i = decltype(ic)::value + 1;
        if (by != i) return;
        asm volatile("");                                 // (selections instead of branches would need all registers twice)
        above(ic);
#pragma unroll
        for (int k = 0; k < 4 * NT; ++k) x[k] = k + 4 * i < 4 * NT ? x[k + 4 * i < 4 * NT ? k + 4 * i : 0] : 0.f;
    });
}

// One wave's tile column `w` of nbt: the reflectors before it, its own, which it publishes at the barrier behind them (number w, one per
// tile column).  y: its tiles.  above(i): tiles 0 .. i, those above the diagonal, are R's.  done(ends, diagonal, triangle, tiles): behind the
// barrier; tile w + b is in y[4 b ..], U's below the diagonal and zeros above, `diagonal` R's, `triangle` T, and no more than `tiles` of
// them are there.  (Two triangles in LDS: the one before is still read while this
// one is written.  One tile to turn around in: the wave before is behind its barrier.)
template <int NT, class Above, class Done>
__device__ __forceinline__ void factorise_tile_column(const TileQrShared& sh, float (&y)[4 * NT], int w, int nbt, int lane, Above&& above, Done&& done) {
    const int c = lane & 15, g = lane >> 4;
#pragma unroll 1
    for (int p = 0; p < w; ++p) {
        __syncthreads();
        apply_reflectors<NT>(sh, y, sh.T + (p & 1) * 256, p, nbt, lane);
    }
    __builtin_amdgcn_s_setprio(2);
    shift_tiles<NT>(y, w, above);
    const int nt = nbt - w;
    constexpr int STEP = NT <= 4 ? 1 : NT <= 8 ? 2 : 4;   // a walk is as long as the tiles that are left, in steps of this
    static_for<NT / STEP>([&](auto sc) {
        constexpr int TC = STEP * (decltype(sc)::value + 1);
        if (nt <= TC - STEP || nt > TC) return;           // wave-uniform
        const ColumnEnds ends = columns_qr<TC>(y, c);
        f32x4_t diagonal;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const int r = 4 * g + e;
            diagonal[e] = r < c ? y[e] : (r == c ? ends.r : 0.f);
            y[e] = r > c ? y[e] : (r == c ? ends.ut : 0.f);
        }
        const f32x4_t triangle = exact_triangle<TC>(y, ends.some, sh.turn, lane);
        *reinterpret_cast<f32x4_t*>(sh.T + (w & 1) * 256 + c * 16 + 4 * g) = triangle;
        float* u = sh.tile(w, w) + 16 * tile_slot(c) + 4 * g;
#pragma unroll
        for (int b = 0; b < TC; ++b)
            if (b < nt) *reinterpret_cast<f32x4_t*>(u + b * 256) = f32x4_t{y[4 * b], y[4 * b + 1], y[4 * b + 2], y[4 * b + 3]};
        __builtin_amdgcn_s_setprio(0);
        __syncthreads();
        done(ends, diagonal, triangle, std::integral_constant<int, TC>{});
    });
}

}  // namespace gelo

// Products of many block reflectors, 256 at a time, as matrix products (the orthogonal factor behind Section 3.2 step 1.2
// once its reflectors exist): X <- H_0 H_1 ... H_last X for block reflectors H = I - Y T Y^T of 256 columns.
//
//   W  = Y^T X               reflect_wt_kernel      256 x c, contraction over all rows below the block's first one
//   W' = -T W                reflect_w_kernel
//   X += Y W'                reflect_update_kernel  contraction over the 256 reflectors
//
// Y W' is summed by itself and added to X once: with X in the accumulator from the start every instruction rounds at its size, and
// |A^T A - I| was 1.4 to 1.8 times what it is (720 to 2150 rows), the part of A^T G below the diagonal 1.3 to 1.7 times.
//
// The two large products run on the bf16 matrix instructions with every float taken apart into three bf16 values (split_float.h).
//
// Everything stays in the 16 x 16 tiles of the factorisation (qr_tile_index): v_mfma_f32_16x16x32_bf16 leaves a tile in the
// same accumulator layout as the float instruction, and a lane's eight values of the contraction are rows 4 g .. 4 g + 3 of
// two neighbouring tiles (g = lane / 16), so X is loaded a contiguous kilobyte at a time and taken apart in registers.
// Y is taken apart once, for either product: a "fragment" is what one instruction takes, 64 lanes x 16 bytes.
//   Yp  [pair of tile rows][plane h, m, l][16 tile columns]   lane (c, g): column c, rows 4 g .. of both tiles
//   Yr  [tile row][pair of tile columns][plane]               lane (c, g): row c, columns 4 g .. of both tiles
//   Wp  [tile column of X][pair of reflector tiles][plane]    lane (c, g): column c, reflectors 4 g .. of both tiles
// T of 256 reflectors: T^-1's upper triangle is Y^T Y's (contracted in double precision: its rounding is what the
// orthogonality of I - Y T Y^T is lost to), its diagonal blocks are the 16 x 16 triangles of the panels.
#include "gelo_internal.h"
#include "block_reflect.h"

namespace gelo {
namespace {

constexpr int WT = kWideTiles;                            // tile columns of a wide block

// ------------------------------------------------------------ Y^T Y and the triangles --
// Tile (i, j), i < j, of every wide block's Y^T Y, in double: a workgroup has two of a column of them, its eight waves share the
// tile rows.  gram: [block][i][j][256], row-major tiles.  (Two by two tiles per workgroup read a third less, but their longest
// workgroup took 26 us at 2150 rows, and the taking apart 8 in a launch of its own: 22 together now, a draw of 2150 rows alone 1438 ->
// 1422 us, 32 of them 10 900 -> 10 720.)
constexpr int kGramPairs = WT * (WT + 2) / 4;             // pairs of tile columns a, tile columns b behind them: b / 2 + 1 for each b

__device__ __forceinline__ void wide_gram(const float* M, double* gram, int nbr, int item) {
    __shared__ double part[8][2][256];
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int c = lane & 15, g = lane >> 4;
    const int q = item / kGramPairs;
    int j = 0, a = item % kGramPairs;
    while (a > j / 2) { a -= j / 2 + 1; ++j; }
    const int t0 = q * WT, mt = nbr - t0;                 // tile rows from the block's first one on
    if (j >= mt) return;
    f64x4_t acc[2];
    acc[0] = acc[1] = f64x4_t{0., 0., 0., 0.};
    for (int r = j + wave; r < mt; r += 8) {              // (column j starts in its tile row j, those before it higher up)
        f32x4_t v[3];
#pragma unroll
        for (int k = 0; k < 3; ++k) {
            const int f = k < 2 ? (2 * a + k < j ? 2 * a + k : j) : j;
            v[k] = *reinterpret_cast<const f32x4_t*>(M + ((int64_t)(t0 + f) * nbr + t0 + r) * 256 + c * 16 + 4 * g);
        }
#pragma unroll
        for (int e = 0; e < 4; ++e)
#pragma unroll
            for (int i = 0; i < 2; ++i) acc[i] = __builtin_amdgcn_mfma_f64_16x16x4f64((double)v[i][e], (double)v[2][e], acc[i], 0, 0, 0);
    }
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int v = 0; v < 4; ++v) part[wave][i][(4 * v + g) * 16 + c] = acc[i][v];      // element v: row 4 v + g
    __syncthreads();
    const int i = 2 * a + (tid >> 8), at = tid & 255;
    double s = part[0][tid >> 8][at];
#pragma unroll
    for (int w = 1; w < 8; ++w) s += part[w][tid >> 8][at];
    if (i < j) gram[((int64_t)q * WT * WT + i * WT + j) * 256 + at] = s;
}

// T of a wide block, row of tiles by row of tiles, a wave each: T[i][j] = -(sum over i <= k < j of T[i][k] G[k][j]) T[j][j].
// The wave carries the transposes (what an instruction leaves is then what the next one takes), in double.
// Tbig: [block][256 x 256] row-major, zeros below the diagonal and beyond the last reflector.
__global__ __launch_bounds__(64)
void wide_triangle_kernel(const double* gram, const float* Tmat, float* Tbig, int nbr, int64_t batch_stride) {
    const int lane = threadIdx.x, c = lane & 15, g = lane >> 4;
    const int q = blockIdx.x / WT, i = blockIdx.x % WT;
    const int nt = nbr - q * WT < WT ? nbr - q * WT : WT;
    gram += (int64_t)blockIdx.y * (batch_stride / 2) + (int64_t)q * WT * WT * 256 + g * 16 + c;
    const float* Tq = Tmat + (int64_t)blockIdx.y * batch_stride + (int64_t)q * WT * 256;
    float* out = Tbig + (int64_t)blockIdx.y * batch_stride + (int64_t)q * (WT * 16) * (WT * 16) + (int64_t)(16 * i + c) * (WT * 16) + g;
    for (int j = 0; j < WT; ++j)
        if (j < i || j >= nt || i >= nt)
#pragma unroll
            for (int v = 0; v < 4; ++v) out[16 * j + 4 * v] = 0.f;
    if (i >= nt) return;
    f64x4_t U[WT];
#pragma unroll
    for (int v = 0; v < 4; ++v) {
        U[0][v] = (double)Tq[i * 256 + c * 16 + 4 * v + g];
        out[16 * i + 4 * v] = (float)U[0][v];
    }
    double next[WT][4];                                   // column i + r of G, requested a column ahead
    f32x4_t t_next;
    auto request = [&](auto rc) {
        constexpr int r = decltype(rc)::value;
        if constexpr (r < WT) {
            const int j = i + r < nt ? i + r : nt - 1;
#pragma unroll
            for (int s = 0; s < r; ++s) {
                const int k = i + s < j ? i + s : (j > 0 ? j - 1 : 0);
#pragma unroll
                for (int v = 0; v < 4; ++v) next[s][v] = j > 0 ? gram[((int64_t)k * WT + j) * 256 + v * 64] : 0.;
            }
#pragma unroll
            for (int v = 0; v < 4; ++v) t_next[v] = Tq[j * 256 + (4 * v + g) * 16 + c];
        }
    };
    request(std::integral_constant<int, 1>{});
    static_for<WT - 1>([&](auto rc) {
        constexpr int r = decltype(rc)::value + 1;
        if (i + r >= nt) return;                          // wave-uniform
        double cur[WT][4];
#pragma unroll
        for (int s = 0; s < r; ++s)
#pragma unroll
            for (int v = 0; v < 4; ++v) cur[s][v] = next[s][v];
        const f32x4_t t = t_next;
        request(std::integral_constant<int, r + 1>{});
        f64x4_t sum = {0., 0., 0., 0.};
#pragma unroll
        for (int s = 0; s < r; ++s)
#pragma unroll
            for (int v = 0; v < 4; ++v) sum = __builtin_amdgcn_mfma_f64_16x16x4f64(cur[s][v], U[s][v], sum, 0, 0, 0);
        f64x4_t u = {0., 0., 0., 0.};
#pragma unroll
        for (int v = 0; v < 4; ++v) u = __builtin_amdgcn_mfma_f64_16x16x4f64(-(double)t[v], sum[v], u, 0, 0, 0);
        U[r] = u;
#pragma unroll
        for (int v = 0; v < 4; ++v) out[16 * (i + r) + 4 * v] = (float)u[v];
    });
}

// ------------------------------------------------------------ Y taken apart --
// one workgroup per pair of tile rows of a wide block
__device__ __forceinline__ void wide_planes(const float* M, uint16_t* Yp, uint16_t* Yr, int nbr, int item) {
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int c = lane & 15, g = lane >> 4;
    int q = 0;
    while ((q + 1) * WT < nbr && pairs_before(nbr, q + 1) <= (int64_t)item) ++q;
    const int pair = item - (int)pairs_before(nbr, q), t0 = q * WT, mt = nbr - t0;
    Yp += (pairs_before(nbr, q) + pair) * kUnitYp + lane * 8;
    Yr += (rows_before(nbr, q) + 2 * pair) * kUnitYr + lane * 8;
    auto tile_of = [&](int r, int f) { return M + ((int64_t)(t0 + f) * nbr + t0 + r) * 256; };
#pragma unroll
    for (int k = 0; k < 2; ++k) {
        const int f = wave + 8 * k;                       // tile column
        f32x4_t v[2];
#pragma unroll
        for (int e = 0; e < 2; ++e) {
            const int r = 2 * pair + e;
            v[e] = f32x4_t{0.f, 0.f, 0.f, 0.f};
            if (f < mt && r < mt && r >= f) v[e] = *reinterpret_cast<const f32x4_t*>(tile_of(r, f) + c * 16 + 4 * g);
        }
        put_split(Yp + f * kFrag, (int64_t)WT * kFrag, split3(v[0], v[1]));
    }
#pragma unroll
    for (int k = 0; k < 2; ++k) {
        const int u = wave, r = 2 * pair + k;             // pair of tile columns, tile row
        if (r >= mt) continue;
        f32x4_t v[2];
#pragma unroll
        for (int e = 0; e < 2; ++e) {
            const int f = 2 * u + e;
            v[e] = f32x4_t{0.f, 0.f, 0.f, 0.f};
            if (f < mt && r >= f) {
#pragma unroll
                for (int x = 0; x < 4; ++x) v[e][x] = tile_of(r, f)[(4 * g + x) * 16 + c];
            }
        }
        put_split(Yr + (int64_t)k * kUnitYr + u * 3 * kFrag, kFrag, split3(v[0], v[1]));
    }
}

// both, in one launch: neither needs the other
__global__ __launch_bounds__(512)
void wide_prepare_kernel(const float* M, double* gram, uint16_t* Yp, uint16_t* Yr, int nbr, int64_t batch_stride) {
    const int blocks = (nbr + WT - 1) / WT, item = blockIdx.x;
    const int64_t off = (int64_t)blockIdx.y * batch_stride;
    if (item < blocks * kGramPairs) wide_gram(M + off, gram + off / 2, nbr, item);
    else wide_planes(M + off, Yp + 2 * off, Yr + 2 * off, nbr, item - blocks * kGramPairs);
}

// ------------------------------------------------------------ the three products --
// W.  The rows are cut into ranges, those into parts of a few ranges; the sums are added range by range, part by part, here or by
// reflect_w_kernel: the bits do not depend on which kernel took the product.
// TC: tile columns of the block (16, or 8 in the factorisation).  Many matrices: a workgroup has 128 reflectors x 128 columns of one part, a wave 128 x 32 (each float is taken apart once in a
// workgroup), Y through LDS.
template <int TC>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(2, 2)))
void reflect_wt_kernel(WideArgs a) {
    constexpr int HALVES = TC / 8;
    __shared__ __attribute__((aligned(1024))) uint16_t stage[2][24 * kFrag];      // [plane][8 tile columns of Y]
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    int matrix, b;
    if (!deal_to_dies(blockIdx.x, HALVES * a.groups * a.parts, a.count, &matrix, &b)) return;
    const int half = b % HALVES, part = b / HALVES % a.parts, cg = b / (HALVES * a.parts);
    const int units = (a.mt + 1) / 2, per_part = a.per_chunk * a.part_chunks;
    const int t_begin = part * per_part, t_end = t_begin + per_part < units ? t_begin + per_part : units;
    const uint16_t* yp = a.Yp + 2 * (int64_t)matrix * a.batch_stride + half * 8 * kFrag + lane * 8;
    const float* xc[2];
    float* w[2];
#pragma unroll
    for (int n = 0; n < 2; ++n) {
        const int col = cg * 8 + wave * 2 + n < a.cols ? cg * 8 + wave * 2 + n : a.cols - 1;
        xc[n] = a.X + (int64_t)matrix * a.batch_stride + (int64_t)col * a.nbr * 256 + (lane & 15) * 16 + 4 * (lane >> 4);
        // as the lanes hold it: only reflect_w_kernel reads it
        w[n] = a.Wpart + (int64_t)matrix * a.batch_stride + (((int64_t)part * a.mt + col) * TC + half * 8) * 256 + lane * 4;
    }
    u32x4_t st[6];
    f32x4_t raw[2][2][2];
    auto fetch_y = [&](int t) {
#pragma unroll
        for (int i = 0; i < 6; ++i) {
            const int id = wave * 6 + i;
            st[i] = *reinterpret_cast<const u32x4_t*>(yp + (int64_t)t * (3 * TC * kFrag) + ((id >> 3) * TC + (id & 7)) * kFrag);
        }
    };
    auto fetch_x = [&](int t, f32x4_t (&x)[2][2]) {
#pragma unroll
        for (int n = 0; n < 2; ++n)
#pragma unroll
            for (int e = 0; e < 2; ++e) {
                const int r = 2 * t + e < a.mt ? 2 * t + e : a.mt - 1;       // the odd last tile row: Y is zero there
                x[n][e] = *reinterpret_cast<const f32x4_t*>(xc[n] + (int64_t)r * 256);
            }
    };
    auto park = [&](int buf) {
#pragma unroll
        for (int i = 0; i < 6; ++i) *reinterpret_cast<u32x4_t*>(&stage[buf][(wave * 6 + i) * kFrag + lane * 8]) = st[i];
    };
    f32x4_t acc[8][2];
#pragma unroll
    for (int f = 0; f < 8; ++f)
#pragma unroll
        for (int n = 0; n < 2; ++n) acc[f][n] = f32x4_t{0.f, 0.f, 0.f, 0.f};
    // Requests are unconditional (the last ones repeat the last unit): a wait then counts exactly what was issued behind what it
    // waits for, instead of everything.
    auto step = [&](int t, int buf, f32x4_t (&mine_x)[2][2]) {
        Split x[2];
#pragma unroll
        for (int n = 0; n < 2; ++n) x[n] = split3(mine_x[n][0], mine_x[n][1]);
        __syncthreads();                                  // this stage is complete, the other one free
        __builtin_amdgcn_sched_barrier(0);                // the compiler would move the requests behind the products
        fetch_y(t + 1 < t_end ? t + 1 : t_end - 1);
        fetch_x(t + 2 < t_end ? t + 2 : t_end - 1, mine_x);
        __builtin_amdgcn_sched_barrier(0);
        const uint16_t* mine = &stage[buf][lane * 8];
        products([&](int plane, int f) { return frag_of(mine + (plane * 8 + f) * kFrag); }, x, acc);
        park(buf ^ 1);
    };
    fetch_x(t_begin, raw[0]);
    fetch_y(t_begin);
    fetch_x(t_begin + 1 < t_end ? t_begin + 1 : t_begin, raw[1]);
    park(0);
    int t = t_begin;
    for (int range = 0; t < t_end; ++range) {
        const int range_end = t + a.per_chunk < t_end ? t + a.per_chunk : t_end;
        for (; t < range_end; t += 2) {                   // (per_chunk is even)
            step(t, 0, raw[0]);
            if (t + 1 < t_end) step(t + 1, 1, raw[1]);
        }
#pragma unroll
        for (int n = 0; n < 2; ++n)
#pragma unroll
            for (int f = 0; f < 8; ++f) {
                if (cg * 8 + wave * 2 + n < a.cols) {     // (a clamped column belongs to another wave)
                    f32x4_t* at = reinterpret_cast<f32x4_t*>(w[n] + f * 256);
                    *at = range == 0 ? acc[f][n] : *at + acc[f][n];
                }
                acc[f][n] = f32x4_t{0.f, 0.f, 0.f, 0.f};
            }
    }
}

// Few matrices: a workgroup has all reflectors x 32 columns (64 of a block of 128) of one range of rows, a wave 64 x 32, everything two units ahead in
// registers: no barrier, and a launch takes little more than its few units.
template <int TC>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(2, 2)))
void reflect_wt_direct_kernel(WideArgs a) {
    constexpr int RG = TC / 4, CP = 4 / RG;               // waves along the reflectors, along the columns
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int pairs = (a.mt + 1) / 2, sets = ((a.cols + 1) / 2 + CP - 1) / CP;      // pairs of tile rows
    int matrix, b;
    if (!deal_to_dies(blockIdx.x, sets * a.chunks, a.count, &matrix, &b)) return;
    const int cp = b % sets * CP + wave / RG, fr = wave % RG * 4, chunk = b / sets;
    const int t_begin = chunk * a.per_chunk, t_end = t_begin + a.per_chunk < pairs ? t_begin + a.per_chunk : pairs;
    const uint16_t* yp = a.Yp + 2 * (int64_t)matrix * a.batch_stride + fr * kFrag + lane * 8;
    const float* xc[2];
#pragma unroll
    for (int n = 0; n < 2; ++n) {
        const int col = 2 * cp + n < a.cols ? 2 * cp + n : a.cols - 1;
        xc[n] = a.X + (int64_t)matrix * a.batch_stride + (int64_t)col * a.nbr * 256 + (lane & 15) * 16 + 4 * (lane >> 4);
    }
    bf16x8_t y[2][3][4];
    f32x4_t raw[2][2][2];
    auto fetch = [&](int t, bf16x8_t (&yd)[3][4], f32x4_t (&xd)[2][2]) {
        const int tt = t < t_end ? t : t_end - 1;
#pragma unroll
        for (int n = 0; n < 2; ++n)
#pragma unroll
            for (int e = 0; e < 2; ++e) {
                const int r = 2 * tt + e < a.mt ? 2 * tt + e : a.mt - 1;     // the odd last tile row: Y is zero there
                xd[n][e] = *reinterpret_cast<const f32x4_t*>(xc[n] + (int64_t)r * 256);
            }
#pragma unroll
        for (int p = 2; p >= 0; --p)
#pragma unroll
            for (int f = 0; f < 4; ++f) yd[p][f] = frag_of(yp + (int64_t)tt * (3 * TC * kFrag) + (p * TC + f) * kFrag);
    };
    f32x4_t acc[4][2];
#pragma unroll
    for (int f = 0; f < 4; ++f)
#pragma unroll
        for (int n = 0; n < 2; ++n) acc[f][n] = f32x4_t{0.f, 0.f, 0.f, 0.f};
    auto step = [&](int t, bf16x8_t (&yd)[3][4], f32x4_t (&xd)[2][2]) {
        Split x[2];
#pragma unroll
        for (int n = 0; n < 2; ++n) x[n] = split3(xd[n][0], xd[n][1]);
        products([&](int plane, int f) { return yd[plane][f]; }, x, acc);
        __builtin_amdgcn_sched_barrier(0);
        fetch(t + 2, yd, xd);
        __builtin_amdgcn_sched_barrier(0);
    };
    fetch(t_begin, y[0], raw[0]);
    fetch(t_begin + 1, y[1], raw[1]);
    for (int t = t_begin; t < t_end; t += 2) {
        step(t, y[0], raw[0]);
        if (t + 1 < t_end) step(t + 1, y[1], raw[1]);
    }
#pragma unroll
    for (int n = 0; n < 2; ++n) {
        if (2 * cp + n >= a.cols) continue;
#pragma unroll
        for (int f = 0; f < 4; ++f)
            *reinterpret_cast<f32x4_t*>(a.Wpart + (int64_t)matrix * a.batch_stride + (((int64_t)chunk * a.mt + 2 * cp + n) * TC + fr + f) * 256 + lane * 4) = acc[f][n];
    }
}

// W' = -T W, taken apart: a workgroup per NC tile columns of X, a wave per pair of reflector tiles.  RANGES: most sums of ranges
// (kWideParts: sums of parts) to be added.
template <int NC, int RANGES>
__global__ __launch_bounds__(512) __attribute__((amdgpu_waves_per_eu(2, 2)))
void reflect_w_kernel(WideArgs a) {
    __shared__ __attribute__((aligned(16))) float W[NC][WT][256];
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int c = lane & 15, g = lane >> 4, col0 = blockIdx.x * NC;
    const float* T = a.T + (int64_t)blockIdx.y * a.batch_stride + (int64_t)(wave * 32 + c) * (WT * 16) + 4 * g;
#pragma unroll
    for (int n = 0; n < NC; ++n) {
        const int col = col0 + n < a.mt ? col0 + n : a.mt - 1;
        const float* wp = a.Wpart + (int64_t)blockIdx.y * a.batch_stride + ((int64_t)col * WT + wave * 2) * 256 + lane * 4;
#pragma unroll
        for (int k = 0; k < 2; ++k)
            *reinterpret_cast<f32x4_t*>(&W[n][wave * 2 + k][lane * 4]) = sum_of_ranges<RANGES>(wp + k * 256, (int64_t)a.mt * WT * 256, a);
    }
    f32x4_t t[2][WT];                                     // its rows of T from the diagonal on, all requested at once
#pragma unroll
    for (int s = 0; s < WT; ++s)
        if (s >= wave * 2)
#pragma unroll
        for (int k = 0; k < 2; ++k) t[k][s] = *reinterpret_cast<const f32x4_t*>(T + k * 16 * (WT * 16) + s * 16);
    __syncthreads();
#pragma unroll
    for (int n = 0; n < NC; ++n) {
        f32x4_t acc[2][2];
#pragma unroll
        for (int k = 0; k < 2; ++k) acc[k][0] = acc[k][1] = f32x4_t{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int s = 0; s < WT; ++s) {
            if (s < wave * 2) continue;                   // below the diagonal
            const f32x4_t w = *reinterpret_cast<const f32x4_t*>(&W[n][s][lane * 4]);
#pragma unroll
            for (int e = 0; e < 4; ++e)
#pragma unroll
                for (int k = 0; k < 2; ++k) acc[k][e & 1] = __builtin_amdgcn_mfma_f32_16x16x4f32(t[k][s][e], w[e], acc[k][e & 1], 0, 0, 0);
        }
        if (col0 + n >= a.mt) break;
        put_split(a.Wp + 2 * (int64_t)blockIdx.y * a.batch_stride + ((int64_t)(col0 + n) * (WT / 2) + wave) * 3 * kFrag + lane * 8, kFrag,
                  split3(-(acc[0][0] + acc[0][1]), -(acc[1][0] + acc[1][1])));
    }
}

// the first eight tile columns behind a block of the factorisation are its next panel: taken apart here, tile rows r and r + 1 of column cc
__device__ __forceinline__ void next_panel(const WideArgs& a, int matrix, int r, int cc, f32x4_t v0, f32x4_t v1, int lane) {
    if (r >= a.mt) return;
    if (r + 1 >= a.mt) v1 = f32x4_t{0.f, 0.f, 0.f, 0.f};
    put_split(a.next + 2 * (int64_t)matrix * a.batch_stride + (int64_t)(r / 2) * kUnitPanel + cc * kFrag + lane * 8, 8 * kFrag, split3(v0, v1));
}

// X += Y W', few matrices: a workgroup has 64 x 64 of X, a wave 32 x 32, two units ahead in registers
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(2, 2)))
void reflect_update_direct_kernel(WideArgs a) {
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int quads = (a.cols + 3) / 4;                   // of tile columns
    int matrix, b;
    if (!deal_to_dies(blockIdx.x, (a.mt + 3) / 4 * quads, a.count, &matrix, &b)) return;
    const int r0 = b / quads * 4 + (wave & 1) * 2, c0 = b % quads * 4 + (wave >> 1) * 2;
    const int units = (a.nt + 1) / 2;
    const uint16_t* ya[2];
    const uint16_t* wb[2];
#pragma unroll
    for (int i = 0; i < 2; ++i) {
        ya[i] = a.Yr + 2 * (int64_t)matrix * a.batch_stride + (int64_t)(r0 + i < a.mt ? r0 + i : a.mt - 1) * a.yr_unit + lane * 8;
        wb[i] = a.Wp + 2 * (int64_t)matrix * a.batch_stride + (int64_t)(c0 + i < a.cols ? c0 + i : a.cols - 1) * a.wp_unit + lane * 8;
    }
    bf16x8_t y[3][3][2];
    Split w[3][2];
    auto fetch = [&](int u, bf16x8_t (&yd)[3][2], Split (&wd)[2]) {
        const int uu = u < units ? u : units - 1;
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            wd[i].h = frag_of(wb[i] + uu * 3 * kFrag);
            wd[i].m = frag_of(wb[i] + (uu * 3 + 1) * kFrag);
            wd[i].l = frag_of(wb[i] + (uu * 3 + 2) * kFrag);
#pragma unroll
            for (int p = 0; p < 3; ++p) yd[p][i] = frag_of(ya[i] + (uu * 3 + p) * kFrag);
        }
    };
    fetch(0, y[0], w[0]);
    fetch(1, y[1], w[1]);
    f32x4_t x[2][2], acc[2][2];
    auto tile = [&](int f, int n) {
        const int r = r0 + f < a.mt ? r0 + f : a.mt - 1, c = c0 + n < a.cols ? c0 + n : a.cols - 1;
        return a.X + (int64_t)matrix * a.batch_stride + ((int64_t)c * a.nbr + r) * 256 + (lane & 15) * 16 + 4 * (lane >> 4);
    };
#pragma unroll
    for (int f = 0; f < 2; ++f)
#pragma unroll
        for (int n = 0; n < 2; ++n) {
            x[f][n] = *reinterpret_cast<const f32x4_t*>(tile(f, n));
            acc[f][n] = f32x4_t{0.f, 0.f, 0.f, 0.f};
        }
    static_for<WT / 2>([&](auto uc) {
        constexpr int u = decltype(uc)::value;
        if (u >= units) return;
        if constexpr (u + 2 < WT / 2) fetch(u + 2, y[(u + 2) % 3], w[(u + 2) % 3]);
        __builtin_amdgcn_sched_barrier(0);
        products([&](int plane, int f) { return y[u % 3][plane][f]; }, w[u % 3], acc);
    });
#pragma unroll
    for (int f = 0; f < 2; ++f)
#pragma unroll
        for (int n = 0; n < 2; ++n) {
            acc[f][n] = x[f][n] + acc[f][n];
            if (r0 + f < a.mt && c0 + n < a.cols) *reinterpret_cast<f32x4_t*>(tile(f, n)) = acc[f][n];
        }
    if (a.next != nullptr && c0 < 8) {                    // wave-uniform
#pragma unroll
        for (int n = 0; n < 2; ++n) next_panel(a, matrix, r0, c0 + n, acc[0][n], acc[1][n], lane);
    }
}

// X += Y W', many matrices: a workgroup has 128 rows x 128 columns of X, a wave 64 x 64.  One stage in LDS, the next one on its way to registers: two
// workgroups share a CU, one waits and parks while the other multiplies.  X is on its way during the last products (read behind them: 32
// draws of 2150 rows 11510 instead of 10570 us).
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(2, 2)))
void reflect_update_kernel(WideArgs a) {
    __shared__ __attribute__((aligned(1024))) uint16_t stage[2][24 * kFrag];      // [8 tile rows of Y][plane], [8 tile columns of W'][plane]
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm = wave & 1, wn = wave >> 1;
    int matrix, b;
    if (!deal_to_dies(blockIdx.x, (a.mt + 7) / 8 * a.groups, a.count, &matrix, &b)) return;
    const int rg = b / a.groups, cg = b % a.groups;
    const int units = (a.nt + 1) / 2;
    const uint16_t* src[4];                               // this wave's two tile rows of Y, two tile columns of W'
#pragma unroll
    for (int i = 0; i < 2; ++i) {
        const int row = rg * 8 + wave * 2 + i, col = cg * 8 + wave * 2 + i;
        src[i] = a.Yr + 2 * (int64_t)matrix * a.batch_stride + (int64_t)(row < a.mt ? row : a.mt - 1) * a.yr_unit + lane * 8;
        src[2 + i] = a.Wp + 2 * (int64_t)matrix * a.batch_stride + (int64_t)(col < a.cols ? col : a.cols - 1) * a.wp_unit + lane * 8;
    }
    u32x4_t st[4][3];
    auto fetch = [&](int u) {
#pragma unroll
        for (int i = 0; i < 4; ++i)
#pragma unroll
            for (int p = 0; p < 3; ++p) st[i][p] = *reinterpret_cast<const u32x4_t*>(src[i] + (u * 3 + p) * kFrag);
    };
    fetch(0);
    f32x4_t acc[4][4];
    auto tile = [&](int f, int n) {
        const int r = rg * 8 + wm * 4 + f, cc = cg * 8 + wn * 4 + n;
        return a.X + (int64_t)matrix * a.batch_stride + ((int64_t)(cc < a.cols ? cc : a.cols - 1) * a.nbr + (r < a.mt ? r : a.mt - 1)) * 256 + (lane & 15) * 16 + 4 * (lane >> 4);
    };
#pragma unroll
    for (int f = 0; f < 4; ++f)
#pragma unroll
        for (int n = 0; n < 4; ++n) acc[f][n] = f32x4_t{0.f, 0.f, 0.f, 0.f};
    auto step = [&](int u, auto&& request) {
        if (u > 0) __syncthreads();                       // nobody reads the last stage any more
#pragma unroll
        for (int i = 0; i < 4; ++i)
#pragma unroll
            for (int p = 0; p < 3; ++p)
                *reinterpret_cast<u32x4_t*>(&stage[i >> 1][((wave * 2 + (i & 1)) * 3 + p) * kFrag + lane * 8]) = st[i][p];
        __syncthreads();
        __builtin_amdgcn_sched_barrier(0);
        request();
        __builtin_amdgcn_sched_barrier(0);
        const uint16_t* ya = &stage[0][wm * 12 * kFrag + lane * 8];
        const uint16_t* wb = &stage[1][wn * 12 * kFrag + lane * 8];
        Split x[4];
#pragma unroll
        for (int n = 0; n < 4; ++n) { x[n].h = frag_of(wb + n * 3 * kFrag); x[n].m = frag_of(wb + (n * 3 + 1) * kFrag); x[n].l = frag_of(wb + (n * 3 + 2) * kFrag); }
        products([&](int plane, int f) { return frag_of(ya + (f * 3 + plane) * kFrag); }, x, acc);
    };
    for (int u = 0; u + 1 < units; ++u) step(u, [&] { fetch(u + 1); });
    f32x4_t before[4][4];
    step(units - 1, [&] {
#pragma unroll
        for (int f = 0; f < 4; ++f)
#pragma unroll
            for (int n = 0; n < 4; ++n) before[f][n] = *reinterpret_cast<const f32x4_t*>(tile(f, n));
    });
#pragma unroll
    for (int f = 0; f < 4; ++f)
#pragma unroll
        for (int n = 0; n < 4; ++n) {
            acc[f][n] = before[f][n] + acc[f][n];
            if (rg * 8 + wm * 4 + f < a.mt && cg * 8 + wn * 4 + n < a.cols) *reinterpret_cast<f32x4_t*>(tile(f, n)) = acc[f][n];
        }
    if (a.next != nullptr && cg == 0) {
#pragma unroll
        for (int f = 0; f < 4; f += 2)
#pragma unroll
            for (int n = 0; n < 4; ++n) next_panel(a, matrix, rg * 8 + wm * 4 + f, wn * 4 + n, acc[f][n], acc[f + 1][n], lane);
    }
}

#define GELO_TRY(expr) do { hipError_t e_ = (expr); if (e_ != hipSuccess) return e_; } while (0)

}  // namespace

int64_t wide_plane_values(int n_pad) {
    const int nbr = n_pad / kPanel, blocks = (nbr + WT - 1) / WT;
    return pairs_before(nbr, blocks) * kUnitYp + rows_before(nbr, blocks) * kUnitYr;
}
int64_t wide_yr_offset(int n_pad) {
    const int nbr = n_pad / kPanel, blocks = (nbr + WT - 1) / WT;
    return pairs_before(nbr, blocks) * kUnitYp;
}

hipError_t block_reflect_init() {    // brings this file's code onto the device (see factor_init)
    hipFuncAttributes attr;
    return hipFuncGetAttributes(&attr, reinterpret_cast<const void*>(&reflect_update_kernel));
}

void cut_into_ranges(WideArgs& a, int halves, int workgroups) {
    // ranges of rows so that one matrix alone fills the chip about once, an even number of pairs of tile rows each
    const int units = (a.mt + 1) / 2, want = kWideCus / workgroups;
    const int chunks = want < 1 ? 1 : want > kWideChunks ? kWideChunks : want;
    a.groups = (a.cols + 7) / 8;
    a.per_chunk = ((units + chunks - 1) / chunks + 1) / 2 * 2;
    a.chunks = (units + a.per_chunk - 1) / a.per_chunk;
    a.part_chunks = (a.chunks + kWideParts - 1) / kWideParts;
    a.parts = (a.chunks + a.part_chunks - 1) / a.part_chunks;
    a.by_part = halves * a.groups * a.count >= kWideCus;
}

template <int TC>
static hipError_t launch_wt(const WideArgs& a, hipStream_t s) {
    const int pairs = (a.cols + 1) / 2;
    constexpr int CP = 16 / TC;
    if (a.by_part) hipLaunchKernelGGL((reflect_wt_kernel<TC>), dim3(8 * dies_slots(TC / 8 * a.groups * a.parts, a.count)), dim3(256), 0, s, a);
    else hipLaunchKernelGGL((reflect_wt_direct_kernel<TC>), dim3(8 * dies_slots((pairs + CP - 1) / CP * a.chunks, a.count)), dim3(256), 0, s, a);
    return hipGetLastError();
}
hipError_t launch_panel_products(const WideArgs& a, hipStream_t s) { return launch_wt<8>(a, s); }

hipError_t launch_block_update(WideArgs a, hipStream_t s) {
    a.groups = (a.cols + 7) / 8;
    const int items = (a.mt + 7) / 8 * a.groups, small = (a.mt + 3) / 4 * ((a.cols + 3) / 4);
    if (items * a.count >= 2 * kWideCus) hipLaunchKernelGGL(reflect_update_kernel, dim3(8 * dies_slots(items, a.count)), dim3(256), 0, s, a);
    else hipLaunchKernelGGL(reflect_update_direct_kernel, dim3(8 * dies_slots(small, a.count)), dim3(256), 0, s, a);
    return hipGetLastError();
}

hipError_t form_product_wide(const FactorWorkspace& ws, int count, int64_t batch_stride, hipStream_t s) {
    const int nbr = ws.n_pad / kPanel, blocks = (nbr + WT - 1) / WT;
    hipLaunchKernelGGL(wide_prepare_kernel, dim3((unsigned)(blocks * kGramPairs + pairs_before(nbr, blocks)), count), dim3(512), 0, s,
                       ws.M, ws.wide_gram, ws.Yp, ws.Yr, nbr, batch_stride);
    GELO_TRY(hipGetLastError());
    hipLaunchKernelGGL(wide_triangle_kernel, dim3(blocks * WT, count), dim3(64), 0, s, ws.wide_gram, ws.Tmat, ws.Tbig, nbr, batch_stride);
    GELO_TRY(hipGetLastError());
    for (int q = blocks - 1; q >= 0; --q) {
        WideArgs a;
        a.nbr = nbr; a.t0 = q * WT; a.mt = a.cols = nbr - a.t0; a.nt = a.mt < WT ? a.mt : WT;
        a.Yp = ws.Yp + pairs_before(nbr, q) * kUnitYp;
        a.Yr = ws.Yr + rows_before(nbr, q) * kUnitYr;
        a.T = ws.Tbig + (int64_t)q * (WT * 16) * (WT * 16);
        a.X = ws.X + ((int64_t)a.t0 * nbr + a.t0) * 256;
        a.Wpart = ws.Wpart; a.Wp = ws.Wp; a.wp_unit = a.yr_unit = kUnitYr; a.next = nullptr;
        a.batch_stride = batch_stride; a.count = count;
        cut_into_ranges(a, 2, 2 * ((a.mt + 7) / 8));
        GELO_TRY(launch_wt<WT>(a, s));
        if (a.by_part) hipLaunchKernelGGL((reflect_w_kernel<4, kWideParts>), dim3((a.mt + 3) / 4, count), dim3(512), 0, s, a);
        else hipLaunchKernelGGL((reflect_w_kernel<1, kWideChunks>), dim3(a.mt, count), dim3(512), 0, s, a);
        GELO_TRY(hipGetLastError());
        GELO_TRY(launch_block_update(a, s));
    }
    return hipSuccess;
}

}  // namespace gelo

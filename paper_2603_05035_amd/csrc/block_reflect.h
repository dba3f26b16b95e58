// Shared by the factorisation and the forming of Q with blocks of reflectors (block_factor.hip, block_reflect.hip).
#pragma once

#include "gelo_internal.h"
#include "split_float.h"

namespace gelo {

constexpr int kUnitYp = 3 * kWideTiles * kFrag;           // bf16 values of a pair of tile rows in Yp
constexpr int kUnitYr = 3 * (kWideTiles / 2) * kFrag;     // of a tile row in a wide block's Yr, and of a tile column in its Wp
static_assert(kYrBlock == 3 * 4 * kFrag, "a tile row of a block of 128 reflectors");
static_assert(kWideChunks <= 2 * kWideParts, "a part has at most two ranges");
constexpr int kUnitPanel = 3 * 8 * kFrag;                 // of a pair of tile rows of a panel of 128 columns

// pairs of tile rows / tile rows in the wide blocks before block q (block q has nbr - 16 q tile rows)
__host__ __device__ inline int64_t pairs_before(int nbr, int q) { return (int64_t)q * ((nbr + 1) / 2) - (int64_t)(kWideTiles / 4) * q * (q - 1); }
__host__ __device__ inline int64_t rows_before(int nbr, int q) { return (int64_t)q * nbr - (int64_t)(kWideTiles / 2) * q * (q - 1); }

struct WideArgs {
    const uint16_t* Yp; const uint16_t* Yr;               // of this block
    const float* T;                                       // of this block, 256 x 256 (forming Q)
    float* X;                                             // the matrix the reflectors meet, from its tile (t0, t0) on
    float* Wpart; uint16_t* Wp; int wp_unit, yr_unit;     // bf16 values of a tile column in Wp, of a tile row in Yr
    uint16_t* next;                                       // where the update leaves the next panel taken apart (the factorisation)
    int nbr, t0, mt;                                      // tile rows of the matrix, the first one taken, those from it on (as many columns)
    int cols;                                             // the tile columns of X this launch takes, the first ones (Wpart's pitch is mt)
    int nt;                                               // tile columns of the block
    int groups;                                           // of eight of them
    int chunks, per_chunk;                                // the rows are cut into so many ranges of pairs of tile rows
    int part_chunks, parts;                               // ranges per part, parts
    int by_part;                                          // Wpart holds sums of parts (many matrices), not of ranges
    int64_t batch_stride; int count;
};

// Sum of one tile of W over the ranges: range by range inside a part, part by part (RANGES: kWideParts where Wpart holds sums of
// parts).  A part has at most two ranges.  Without branches: what does not exist is cleared.
template <int RANGES>
__device__ __forceinline__ f32x4_t sum_of_ranges(const float* p, int64_t stride, const WideArgs& a) {
    constexpr int PER = RANGES / kWideParts;
    static_assert(PER == 1 || PER == 2, "a part has one or two ranges");
    const int have = PER == 2 ? a.chunks : a.parts, step = PER == 2 ? a.part_chunks : 1;
    f32x4_t s[kWideParts][PER];
#pragma unroll
    for (int i = 0; i < kWideParts; ++i)
#pragma unroll
        for (int e = 0; e < PER; ++e) {
            const int range = i * step + e;
            s[i][e] = *reinterpret_cast<const f32x4_t*>(p + (range < have ? range : have - 1) * stride);
        }
    f32x4_t total = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int i = 0; i < kWideParts; ++i) {
        f32x4_t part;
#pragma unroll
        for (int e = 0; e < PER; ++e) {
            const int mask = ((i * step + e < have) & (e < step)) ? -1 : 0;
#pragma unroll
            for (int x = 0; x < 4; ++x) {
                const float w = s[i][e][x];               // (a vector's element itself would be cast as element 0)
                const float v = __builtin_bit_cast(float, __builtin_bit_cast(int, w) & mask);
                part[x] = e == 0 ? v : part[x] + v;
            }
        }
        total = i == 0 ? part : total + part;
    }
    return total;
}

void cut_into_ranges(WideArgs& a, int halves, int workgroups);                  // chunks .. by_part, groups
hipError_t launch_panel_products(const WideArgs& a, hipStream_t s);             // Wpart <- ranges of P^T X, P a panel of 128 columns (a.Yp)
hipError_t launch_block_update(WideArgs a, hipStream_t s);                      // X <- X + Y W'

}  // namespace gelo

// Operations of one wave on 16 x 16 tiles: lane (g, c) = (lane / 16, lane % 16) holds rows of column c.
#pragma once

#include "gelo_internal.h"
#include "split_float.h"

namespace gelo {

// value of lane J of the row of 16 lanes
template <int J>
__device__ __forceinline__ float row_bcast(float v) {                                      // row_newbcast:J
    return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), 0x150 + J, 0xF, 0xF, true));
}

// col[i] += k x (col[i] of lane J of the row of 16), rows FROM <= i < TO: one instruction each, which the compiler does not
// form by itself (it leaves a move with the broadcast and a multiply-add: twice the issue slots of the loop below).  The
// register a broadcast reads must not have been written by one of the two preceding instructions: the leading wait covers
// what the compiler put in front, inside each register is read and written once, the trailing one covers what follows.
#define GELO_ROW(i) ".if (" #i " >= %c18) && (" #i " < %c19)\n\tv_fmac_f32_dpp %" #i ", %" #i ", %16 row_newbcast:%c17 row_mask:0xf bank_mask:0xf\n.endif\n\t"
template <int J, int FROM, int TO>
__device__ __forceinline__ void add_column(float (&col)[kPanel], float k) {
    if constexpr (FROM < TO)
        asm("s_nop 1\n\t"
            GELO_ROW(0) GELO_ROW(1) GELO_ROW(2) GELO_ROW(3) GELO_ROW(4) GELO_ROW(5) GELO_ROW(6) GELO_ROW(7)
            GELO_ROW(8) GELO_ROW(9) GELO_ROW(10) GELO_ROW(11) GELO_ROW(12) GELO_ROW(13) GELO_ROW(14) GELO_ROW(15)
            "s_nop 1"
            : "+v"(col[0]), "+v"(col[1]), "+v"(col[2]), "+v"(col[3]), "+v"(col[4]), "+v"(col[5]), "+v"(col[6]), "+v"(col[7]),
              "+v"(col[8]), "+v"(col[9]), "+v"(col[10]), "+v"(col[11]), "+v"(col[12]), "+v"(col[13]), "+v"(col[14]), "+v"(col[15])
            : "v"(k), "n"(J), "n"(FROM), "n"(TO));
}
#undef GELO_ROW

// the same for every row but J and J + 1: above with coefficient `up`, below with `down`
#define GELO_ROW(i) ".if (" #i " < %c18)\n\tv_fmac_f32_dpp %" #i ", %" #i ", %16 row_newbcast:%c18 row_mask:0xf bank_mask:0xf\n.endif\n\t" \
                    ".if (" #i " > %c18 + 1)\n\tv_fmac_f32_dpp %" #i ", %" #i ", %17 row_newbcast:%c18 row_mask:0xf bank_mask:0xf\n.endif\n\t"
template <int J>
__device__ __forceinline__ void add_column_around(float (&col)[kPanel], float up, float down) {
    asm("s_nop 1\n\t"
        GELO_ROW(0) GELO_ROW(1) GELO_ROW(2) GELO_ROW(3) GELO_ROW(4) GELO_ROW(5) GELO_ROW(6) GELO_ROW(7)
        GELO_ROW(8) GELO_ROW(9) GELO_ROW(10) GELO_ROW(11) GELO_ROW(12) GELO_ROW(13) GELO_ROW(14) GELO_ROW(15)
        "s_nop 1"
        : "+v"(col[0]), "+v"(col[1]), "+v"(col[2]), "+v"(col[3]), "+v"(col[4]), "+v"(col[5]), "+v"(col[6]), "+v"(col[7]),
          "+v"(col[8]), "+v"(col[9]), "+v"(col[10]), "+v"(col[11]), "+v"(col[12]), "+v"(col[13]), "+v"(col[14]), "+v"(col[15])
        : "v"(up), "v"(down), "n"(J));
}
#undef GELO_ROW
// x += k x (x of lane J of the row of 16)
template <int J>
__device__ __forceinline__ void add_lane(float& x, float k) {
    asm("s_nop 1\n\tv_fmac_f32_dpp %0, %0, %1 row_newbcast:%c2 row_mask:0xf bank_mask:0xf\n\ts_nop 1" : "+v"(x) : "v"(k), "n"(J));
}

// the value of the lane's column in the first (second) row of 16 lanes, in every row
__device__ __forceinline__ void first_two_rows(float v, float* first, float* second) {
    const auto r = __builtin_amdgcn_permlane16_swap(__builtin_bit_cast(unsigned, v), __builtin_bit_cast(unsigned, v), false, false);
    *first = __builtin_bit_cast(float, (unsigned)__builtin_amdgcn_permlane32_swap(r[0], r[0], false, false)[0]);
    *second = __builtin_bit_cast(float, (unsigned)__builtin_amdgcn_permlane32_swap(r[1], r[1], false, false)[0]);
}

// lane (g, c) of a wave with all 16 rows of column c (the same in its four groups g) -> rows 4 g .. 4 g + 3
__device__ __forceinline__ f32x4_t rows_of_group(const float (&col)[kPanel], int g) {
    f32x4_t r;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        const float c0 = col[e], c1 = col[4 + e], c2 = col[8 + e], c3 = col[12 + e];
        const float lo = g & 1 ? c1 : c0, hi = g & 1 ? c3 : c2;
        r[e] = g & 2 ? hi : lo;
    }
    return r;
}

// a value summed over the four rows of 16 lanes; that of row Q in all of them
__device__ __forceinline__ float sum_of_rows(float v) {
    const auto a = __builtin_amdgcn_permlane16_swap(__builtin_bit_cast(unsigned, v), __builtin_bit_cast(unsigned, v), false, false);
    v = __builtin_bit_cast(float, (unsigned)a[0]) + __builtin_bit_cast(float, (unsigned)a[1]);
    const auto b = __builtin_amdgcn_permlane32_swap(__builtin_bit_cast(unsigned, v), __builtin_bit_cast(unsigned, v), false, false);
    return __builtin_bit_cast(float, (unsigned)b[0]) + __builtin_bit_cast(float, (unsigned)b[1]);
}
template <int Q>
__device__ __forceinline__ float row_to_all(float v) {
    const unsigned x = __builtin_amdgcn_permlane16_swap(__builtin_bit_cast(unsigned, v), __builtin_bit_cast(unsigned, v), false, false)[Q & 1];
    return __builtin_bit_cast(float, (unsigned)__builtin_amdgcn_permlane32_swap(x, x, false, false)[Q >> 1]);
}

template <int CTRL>
__device__ __forceinline__ float dpp_mov(float v) {
    return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), CTRL, 0xF, 0xF, false));
}
template <int PATTERN>
__device__ __forceinline__ float swizzle(float v) {
    return __builtin_bit_cast(float, __builtin_amdgcn_ds_swizzle(__builtin_bit_cast(int, v), PATTERN));
}

// Index of the value that lane `lane` ends up holding after wave_reduce16.
__device__ __forceinline__ int reduce16_slot(int lane) {
    return ((lane >> 2) & 1) * 8 + ((lane >> 3) & 1) * 4 + ((lane >> 1) & 1) * 2 + (lane & 1);
}

// Sums 16 per-lane values over the 64 lanes of a wave in ~50 instructions: each exchange step
// halves the number of values a lane carries (the lane keeps the half its partner does not),
// so after four steps inside a row of 16 lanes every lane holds ONE value, summed over its row;
// two more exchanges add the four rows.  Returns, in every lane, the wave total of value
// reduce16_slot(lane).  All 64 lanes must be active.  The order of additions is fixed.
__device__ __forceinline__ float wave_reduce16(const float (&t)[16], int lane) {
    const bool b0 = lane & 1, b1 = lane & 2, b2 = lane & 4, b3 = lane & 8;
    float a[8], c[4], e[2];
#pragma unroll
    for (int k = 0; k < 8; ++k) {
        const float keep = b0 ? t[2 * k + 1] : t[2 * k];
        const float give = b0 ? t[2 * k] : t[2 * k + 1];
        a[k] = keep + dpp_mov<0xB1>(give);              // lane ^ 1  (quad_perm [1,0,3,2])
    }
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        const float keep = b1 ? a[2 * k + 1] : a[2 * k];
        const float give = b1 ? a[2 * k] : a[2 * k + 1];
        c[k] = keep + dpp_mov<0x4E>(give);              // lane ^ 2  (quad_perm [2,3,0,1])
    }
#pragma unroll
    for (int k = 0; k < 2; ++k) {
        const float keep = b3 ? c[2 * k + 1] : c[2 * k];
        const float give = b3 ? c[2 * k] : c[2 * k + 1];
        e[k] = keep + dpp_mov<0x128>(give);             // lane ^ 8  (row_ror:8)
    }
    const float keep = b2 ? e[1] : e[0];
    const float give = b2 ? e[0] : e[1];
    float f = keep + swizzle<0x101F>(give);             // lane ^ 4
    f += swizzle<0x401F>(f);                            // lane ^ 16
    f += __builtin_bit_cast(float, __builtin_amdgcn_ds_bpermute((lane ^ 32) << 2, __builtin_bit_cast(int, f)));
    return f;
}

template <int LANE>
__device__ __forceinline__ float lane_value(float v) {
    return __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, v), LANE));
}

}  // namespace gelo

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

}  // namespace gelo

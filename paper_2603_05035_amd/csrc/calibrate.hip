// What the matrix cores deliver when nothing else is in the way: every wave of every compute unit issues
// independent matrix instructions from registers, in the mix of one K step of the projection kernels, two waves
// per SIMD.  No memory, no LDS, no barrier.  The published peaks (Section
// 4.2's "fraction of peak" is quoted against them) assume the top clock; under this load the chip settles lower,
// so this rate is the ceiling a kernel can be held against.  A measurement aid: nothing in the protocol calls it.
#include "gelo_internal.h"

namespace gelo {
namespace {

typedef __bf16 bf16x8_t __attribute__((ext_vector_type(8)));
typedef float f32x4_t __attribute__((ext_vector_type(4)));
typedef float f32x16_t __attribute__((ext_vector_type(16)));
typedef uint32_t u32x4_t __attribute__((ext_vector_type(4)));
typedef int i32x8_t __attribute__((ext_vector_type(8)));

constexpr int kRateWorkgroups = 256, kRateThreads = 512;

// Operands like real data - the power the matrix cores draw, and with it the clock they are given, depends on
// how many operand bits change from one instruction to the next: every element has a random sign and mantissa and a magnitude
// between 2^-3 and 2^4 (bf16), or is a random E4M3 code with the top exponent bit clear (no NaN code).
__device__ __forceinline__ uint32_t hash(uint32_t x) { x ^= x >> 16; x *= 0x7feb352du; x ^= x >> 15; x *= 0x846ca68bu; x ^= x >> 16; return x; }
__device__ __forceinline__ uint32_t random_word(uint32_t seed, int index) {
    return hash(seed + 977u * (uint32_t)(blockIdx.x * kRateThreads + threadIdx.x) + 31u * (uint32_t)index);
}

// v_mfma_f32_16x16x32_bf16 as a K step of 64 of the bf16 projection has them: a wave's tile of 64 x 128, 4 x 8 accumulators, two halves of
// K with four "A" and eight "B" fragments each.
constexpr int kInstructionsBf16 = 64;                                     // per wave and loop pass
__global__ __launch_bounds__(kRateThreads)
void matrix_rate_bf16_kernel(float* out, int iters, uint32_t seed) {
    f32x4_t acc[4][8];
#pragma unroll
    for (int r = 0; r < 4; ++r)
#pragma unroll
        for (int c = 0; c < 8; ++c) acc[r][c] = f32x4_t{0.f, 0.f, 0.f, 0.f};
    bf16x8_t frag[2][12];
#pragma unroll
    for (int f = 0; f < 24; ++f) {
        u32x4_t w;
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            auto half = [](uint32_t b) { return (b & 0x8000u) | ((0x7Cu + ((b >> 8) & 7u)) << 7) | (b & 0x7Fu); };
            const uint32_t h = random_word(seed, f * 4 + v);
            w[v] = half(h) | (half(h >> 16) << 16);
        }
        frag[f / 12][f % 12] = __builtin_bit_cast(bf16x8_t, w);
    }
    for (int it = 0; it < iters; ++it)
#pragma unroll
        for (int k = 0; k < 2; ++k)
#pragma unroll
            for (int c = 0; c < 8; ++c)
#pragma unroll
                for (int r = 0; r < 4; ++r) acc[r][c] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(frag[k][4 + c], frag[k][r], acc[r][c], 0, 0, 0);
    float sum = 0.f;
#pragma unroll
    for (int r = 0; r < 4; ++r)
#pragma unroll
        for (int c = 0; c < 8; ++c) sum += acc[r][c][0] + acc[r][c][3];
    out[blockIdx.x * kRateThreads + threadIdx.x] = sum;
}

// v_mfma_f32_32x32x64_f8f6f4 on E4M3 operands, eight accumulators per wave, four "A" and two "B" fragments
constexpr int kInstructionsFp8 = 32;
__global__ __launch_bounds__(kRateThreads)
void matrix_rate_fp8_kernel(float* out, int iters, uint32_t seed) {
    f32x16_t acc[8];
#pragma unroll
    for (int i = 0; i < 8; ++i)
#pragma unroll
        for (int v = 0; v < 16; ++v) acc[i][v] = 0.f;
    i32x8_t frag[6];
#pragma unroll
    for (int f = 0; f < 6; ++f)
#pragma unroll
        for (int v = 0; v < 8; ++v) frag[f][v] = (int)(random_word(seed, f * 8 + v) & 0xBFBFBFBFu);
    for (int it = 0; it < iters; ++it)
#pragma unroll
        for (int g = 0; g < kInstructionsFp8 / 8; ++g)
#pragma unroll
            for (int i = 0; i < 8; ++i) acc[i] = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(frag[4 + (i & 1)], frag[i >> 1], acc[i], 0, 0, 0, 0, 0, 0);
    float sum = 0.f;
#pragma unroll
    for (int i = 0; i < 8; ++i) sum += acc[i][0] + acc[i][7] + acc[i][15];
    out[blockIdx.x * kRateThreads + threadIdx.x] = sum;
}

}  // namespace

size_t matrix_rate_scratch_bytes() { return (size_t)kRateWorkgroups * kRateThreads * sizeof(float); }

// Enqueues one launch; flop = what it executes.
hipError_t matrix_rate_launch(int fp8, int iters, float* scratch, double* flop, hipStream_t stream) {
    if (fp8) hipLaunchKernelGGL(matrix_rate_fp8_kernel, dim3(kRateWorkgroups), dim3(kRateThreads), 0, stream, scratch, iters, 7u);
    else hipLaunchKernelGGL(matrix_rate_bf16_kernel, dim3(kRateWorkgroups), dim3(kRateThreads), 0, stream, scratch, iters, 7u);
    const double per_pass = fp8 ? 2.0 * 32 * 32 * 64 * kInstructionsFp8 : 2.0 * 16 * 16 * 32 * kInstructionsBf16;
    *flop = per_pass * (double)iters * (kRateThreads / 64) * kRateWorkgroups;
    return hipGetLastError();
}

}  // namespace gelo

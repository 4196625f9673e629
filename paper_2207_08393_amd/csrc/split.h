// Float32 operands as sums of three bfloat16 numbers, and what the kernels that multiply them share (gfx950 device code).
// x = x1 + x2 + x3 exactly, with x1 = bf16(x), x2 = bf16(x - x1), x3 = x - x1 - x2 (8 + 8 + 8 significant bits; the method of
// Henry, Tang and Heinecke, "Leveraging the bfloat16 Artificial Intelligence Datatype For Higher-Precision Computations", 2019).
// Range: 2^-103 <= |x| <= 3.39e38, the largest bfloat16.  Below, parts are subnormal and x is kept to 2^-126; above, and for
// infinity, x - x1 is NaN.  Partial products lose what lies below 2^-126 too: of numbers whose product is below about 2^-94, bits are
// gone.  What is split are sums of two (transformed inputs) or three (weights) float32 numbers: an input is
// good up to 1.69e38.
#pragma once
#include "prox_common.h"

namespace gleam {
namespace {

struct Split {
    bf16x8 p[3];
};
struct SplitWords {   // the same while it is being formed: [part][pair of values]
    unsigned w[3][4];
    __device__ __forceinline__ Split done() const {
        Split s;
#pragma unroll
        for (int k = 0; k < 3; ++k) s.p[k] = __builtin_bit_cast(bf16x8, *reinterpret_cast<const uint4*>(w[k]));
        return s;
    }
};
// One pair of values: 11 vector instructions.  (A dot product with (-1, 0) or (0, -1) would subtract a half of a packed pair in
// one instruction, 7 per pair; measured 10 - 20 % slower in the kernels that use this, the dot product is not a full-rate
// instruction.)
__device__ __forceinline__ void split_pair(float a, float b, int i, SplitWords& s) {
#pragma unroll
    for (int p = 0; p < 3; ++p) {
        s.w[p][i] = pack_bf16x2(a, b);
        a -= __uint_as_float(s.w[p][i] << 16);
        b -= __uint_as_float(s.w[p][i] & 0xffff0000u);
    }
}
__device__ __forceinline__ Split split8(const float* v) {
    SplitWords s;
#pragma unroll
    for (int i = 0; i < 4; ++i) split_pair(v[2 * i], v[2 * i + 1], i, s);
    return s.done();
}

// Keeps the operand's instructions where they are written: without it the compiler sinks them to their first use, behind the
// next barrier.
__device__ __forceinline__ void pin(Split& s) {
#pragma unroll
    for (int k = 0; k < 3; ++k) asm volatile("" : "+v"(s.p[k]));
}

// The six partial products of a product of split numbers that count, small ones first.
constexpr int kProducts = 6;
__device__ constexpr int kPartA[kProducts] = {2, 1, 0, 1, 0, 0}, kPartB[kProducts] = {0, 1, 2, 0, 1, 0};

// 16 bytes per lane from a buffer resource straight into LDS (a plain function: the host pass drops the stub of a kernel
// template whose own body makes this call)
__device__ __forceinline__ void load_lds(__amdgpu_buffer_rsrc_t rs, float* dst, unsigned lane_off, int off) {
    __builtin_amdgcn_raw_ptr_buffer_load_lds(rs, (__attribute__((address_space(3))) void*)dst, 16, lane_off, off, 0, 0);
}

typedef unsigned uint4v __attribute__((ext_vector_type(4)));
__device__ __forceinline__ uint4v load16(__amdgpu_buffer_rsrc_t rs, unsigned lane_off, unsigned off) {
    return __builtin_amdgcn_raw_buffer_load_b128(rs, lane_off, off, 0);
}
// The data registers of a store of 16 bytes are read over several clocks.  With an offset in a scalar register the compiler lets the
// next instruction overwrite them (without one it leaves a clock in between), and on this chip the last four of every sixteen
// lanes then stored the new value of the first register: the value stays in use for one instruction more.  ("memory" keeps the store in
// front of it; it costs nothing: ten calls take 0.997 to 1.008 times as long with it, 1.000 in the mean.)
__device__ __forceinline__ void store16(__amdgpu_buffer_rsrc_t rs, uint4v v, unsigned lane_off, unsigned off) {
    __builtin_amdgcn_raw_buffer_store_b128(v, rs, lane_off, off, 0);
    asm volatile("s_nop 0" : : "v"(v) : "memory");
}

// Instruction order: N times one matrix instruction, D LDS reads and V vector instructions (a matrix instruction occupies its
// unit for 32 clocks, in which the other units take four to six instructions for free).
template <int N, int V, int D = 0>
__device__ __forceinline__ void interleave() {
    if constexpr (N > 0) {
        __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
        if constexpr (D > 0) __builtin_amdgcn_sched_group_barrier(0x100, D, 0);
        __builtin_amdgcn_sched_group_barrier(0x002, V, 0);
        interleave<N - 1, V, D>();
    }
}

}  // namespace
}  // namespace gleam

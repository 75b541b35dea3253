// What the kernels that multiply on the matrix cores share (gemm.hip, stream.hip): loads from memory to LDS, conversions, small loops.
#pragma once
#include <type_traits>
#include <utility>

#include "common.h"
#include "slices.h"

namespace {

typedef float f32x4_t __attribute__((ext_vector_type(4)));
typedef td_i32x4 i32x4_t;

constexpr int kLdsBytes = 160 * 1024;

// The slice of `len` that a block starts with
__device__ __forceinline__ int first_slice(int xcd, int local, int len) {
    const int at = (local & 7) + xcd * len / 8;
    return len < 8 ? 0 : at >= len ? at - len : at;
}

__device__ __forceinline__ i32x4_t buffer_of(const void* p, uint32_t bytes) {
    const uint64_t a = reinterpret_cast<uint64_t>(p);
    i32x4_t r;
    r.x = __builtin_amdgcn_readfirstlane((int)(uint32_t)a);
    r.y = __builtin_amdgcn_readfirstlane((int)((a >> 32) & 0xffffu));
    r.z = __builtin_amdgcn_readfirstlane((int)bytes);
    r.w = 0x00020000;
    return r;
}

// 64 x 16 bytes from rs[voff + soff] to LDS at lds + 16 * lane (past the buffer's end: nothing is fetched).
// (m0 is set and used in the one statement.  It is a reserved register, which the compiler does not take as a clobber; it
// uses it nowhere else in the kernels of gemm.hip and stream.hip, and the tests of their listings hold it to that)
template <bool ONCE = false>
__device__ __forceinline__ void load_to_lds(uint32_t lds, uint32_t voff, i32x4_t rs, uint32_t soff) {
    if constexpr (ONCE)
        asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tbuffer_load_dwordx4 %1, %2, %3 offen nt lds"
                     ::"s"(lds), "v"(voff), "s"(rs), "s"(soff));
    else
        asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tbuffer_load_dwordx4 %1, %2, %3 offen lds"
                     ::"s"(lds), "v"(voff), "s"(rs), "s"(soff));
}

// round to nearest even, two in one instruction
typedef __bf16 bf16x2_t __attribute__((ext_vector_type(2)));
typedef float f32x2_t __attribute__((ext_vector_type(2)));
__device__ __forceinline__ uint32_t to_bf16x2(float a, float b) {
    return __builtin_bit_cast(uint32_t, __builtin_convertvector((f32x2_t{a, b}), bf16x2_t));
}

template <int V> using num = std::integral_constant<int, V>;
// f(num<0>), ..., f(num<N - 1>)
template <typename F, int... I> __device__ __forceinline__ void for_each_constant(F f, std::integer_sequence<int, I...>) { (f(num<I>{}), ...); }
template <int N, typename F> __device__ __forceinline__ void for_constants(F f) { for_each_constant(f, std::make_integer_sequence<int, N>{}); }

// v of lanes l, l^16, l^32 and l^48 or-ed together
__device__ __forceinline__ uint32_t or_halves(uint32_t v) {
    const auto a = __builtin_amdgcn_permlane16_swap(v, v, false, false);
    v = a[0] | a[1];
    const auto b = __builtin_amdgcn_permlane32_swap(v, v, false, false);
    return b[0] | b[1];
}

template <typename F> __device__ __forceinline__ void with_act(int act, F f) {
    if (act == TARDIS_ACT_GELU_ERF) f(num<TARDIS_ACT_GELU_ERF>{});
    else if (act == TARDIS_ACT_GELU_TANH) f(num<TARDIS_ACT_GELU_TANH>{});
    else if (act == TARDIS_ACT_RELU) f(num<TARDIS_ACT_RELU>{});
    else f(num<TARDIS_ACT_IDENTITY>{});
}

struct StreamBlock {
    int64_t n0;                    // first row of the weights
    int s0, nk, rot;               // slices [s0, s0 + nk), from s0 + rot on
};
__device__ __forceinline__ StreamBlock stream_block(const StreamPlan& p, int block) {
    StreamBlock b;
    const int ks = block & (p.splits - 1), all = (int)((p.k + p.k2) / kStreamSlice);
    b.n0 = (int64_t)(block >> __builtin_ctz(p.splits)) * p.tile;
    b.s0 = ks * p.slices;
    b.nk = max(0, min(p.slices, all - b.s0));
    b.rot = first_slice(block & 7, block >> 3, b.nk);
    return b;
}
constexpr int kWarmSlices = 4;
// What number i of tile * 4 * kWarmSlices threads asks for so that the first slices of a block are in the caches: a word of every 64 bytes
// (null: nothing)
__device__ __forceinline__ const uint32_t* stream_warm(const StreamPlan& p, const StreamBlock& b, int i) {
    const int slice = p.tile == 64 ? i >> 8 : i >> 7, row = (i >> 2) & (p.tile - 1), n1 = (int)(p.k / kStreamSlice);
    if (slice >= kWarmSlices || slice >= b.nk || b.n0 + row >= p.N) return nullptr;
    int s = b.rot + slice;
    s = b.s0 + (s >= b.nk ? s - b.nk : s);
    const unsigned char* from = s < n1 ? p.B + (b.n0 + row) * p.k + (size_t)s * kStreamSlice : p.B2 + (b.n0 + row) * p.k2 + (size_t)(s - n1) * kStreamSlice;
    return reinterpret_cast<const uint32_t*>(from + (i & 3) * 64);
}

}  // namespace

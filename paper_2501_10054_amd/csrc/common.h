// Shared declarations of libtardis: the layer handle, status helpers and the
// small device-side numeric helpers every kernel file uses.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include <mutex>

#include "../../include/tardis.h"

typedef uint16_t bf16_t;  // raw bfloat16 bits
typedef unsigned int td_u32x4 __attribute__((ext_vector_type(4)));  // one 16-byte load

#define TD_WAVE 64

constexpr float kRmsEps = 1e-6f;

#define TD_HIP(expr)                                                              \
    do {                                                                          \
        hipError_t e__ = (expr);                                                  \
        if (e__ != hipSuccess)                                                    \
            return (e__ == hipErrorOutOfMemory) ? TARDIS_ERR_OOM : TARDIS_ERR_HIP; \
    } while (0)

#define TD_TRY(expr)                          \
    do {                                      \
        tardis_status_t s__ = (expr);         \
        if (s__ != TARDIS_OK) return s__;     \
    } while (0)

// One-time set-up that may be reached from several host threads (kernel attributes are raised
// when the first layer is folded): `fn` runs under a lock until it has succeeded once.
struct td_once {
    std::mutex lock;
    bool done = false;
    template <typename F> tardis_status_t run(F fn) {
        std::lock_guard<std::mutex> guard(lock);
        if (done) return TARDIS_OK;
        const tardis_status_t st = fn();
        if (st == TARDIS_OK) done = true;
        return st;
    }
};

// What the single-launch stack kernel needs of one layer (a copy lives in device memory, filled when
// the layer is folded).
struct td_stack_layer_dev {
    const bf16_t* Wp;
    const float* bp;
    const int8_t* Q;
    const float* tlo;
    const float* thi;
    const bf16_t* W1;
    const bf16_t* b1;
    const bf16_t* W2T;
    const float* a;
    const float* c;
    uint32_t* mask;
    bf16_t* xnext;
    float* yfix;       // the layer's accumulator copies (zero between launches)
    int32_t* sync;     // the layer's counters (zero between launches)
    int32_t h, npb, act, reserved;
};

// Everything one folded layer owns.  Pointers are device memory.
struct tardis_layer_s {
    int64_t d, h;
    int32_t dtype, act;
    int64_t max_batch;
    int64_t mask_words;  // ceil(h/32)
    // borrowed from the caller
    const void* W1;  // h x d
    const void* b1;  // h or null
    const void* b2;  // d or null
    // owned: `memory` is the one allocation everything below lies in
    void* memory;
    size_t memory_bytes;
    int device;    // where it lies
    void* W2T;     // h x d, neuron-major copy of W2
    void* W2;      // d x h, copy of W2 as given (dense baseline)
    void* Wp;      // d x d folded matrix
    uint8_t* Wp8;      // d x d e4m3 codes of the folded matrix (8-bit storage only, else null): Wp = code * scale
    float* wp8_scale;  // d power-of-two row scales of Wp8
    float* bp;     // d folded bias
    int8_t* Q;     // h x d predictor codes, one byte each (absent when only the packed 4-bit form is kept)
    uint8_t* Q4;   // packed 4-bit sketch, h x d/2 bytes: one 16-byte vector per group of 32 columns (or null)
    uint8_t* M4;   // 4-bit sketch: h x ceil(d/32) group multipliers, one byte each (or null)
    int32_t sketch_bits;   // 8, or 4 / 3 / 2: grouped codes in 4-bit slots
    float margin;          // fraction of a range's width the predictor's test is narrowed by at either end
    float* tlo;    // h
    float* thi;    // h
    float* a;      // h
    float* c;      // h
    float* code_scale;     // h: the 8-bit codes are rint(weight * this) (td_code_scale); null where some row's are not
    // working memory of the online calls (sized by max_batch)
    float* yacc;       // max_batch x d fp32 accumulator
    uint32_t* mask;    // max_batch x mask_words
    int32_t* counts;   // max_batch flagged-neuron counters (zero between calls)
    int32_t* list;     // max_batch x h flagged indices
    float* hidden;     // max_batch x h activations for the dense baseline
    int32_t* sync;     // small block of device counters (zero between calls)
    void* zeros_h;     // h zero elements of the layer dtype (stands in for a missing b1)
    void* xnext;       // max_batch x d, layer dtype: normalised output handed to the next stacked layer
    float* yfix;       // dec_copies x kDecodeMaxTokens x d fp32 repair accumulators of the fused decode kernel (zero between calls)
    const tardis_layer_s* next_layer;   // the layer that runs after this one (hint, may be null; not owned)
    int32_t prefetch_bytes;             // bytes of that layer's predictor rows each finished block requests
    int32_t strict_release;             // the signalling thread of a decode block also executes an agent-scope release fence
    int32_t prefetch_shape;             // next-layer warming by order of arrival: first16 | last16 << 8 (sixteenths of prefetch_bytes; 0 = flat)
    int32_t dec_blocks;   // grid of the fused decode kernel
    int32_t dec_threads;  // block size of the fused decode kernel (512 or 1024)
    int32_t dec_copies;   // number of repair accumulator copies
    int32_t use_fused;    // fused single-launch decode path available for this layer
    void* pf_scratch;              // matrix products: int8 tokens, exponents, aligned tokens, repair factors, fp32 partial sums of y
    int32_t prefill_min_tokens;    // calls with at least this many tokens run as matrix products (if there is scratch)
    int32_t prefill_chunk;         // ... in chunks of at most this many tokens (what the scratch is sized for)
    int32_t fine_max_tokens;       // ... and those with at most this many carry the repair factors as head and remainder
    int32_t* rec_count;            // two-kernel path: flagged neurons per predictor block,
    uint32_t* rec_jb;              //   neuron index and
    uint32_t* rec_tb;              //   token bits of each record (dec_blocks x neurons per block),
    float* rec_delta;              //   and kDecodeMaxTokens deltas per record
    int32_t defer_min_tokens;      // groups of at least this many tokens take the two-kernel path (4, 8; 99 = never)
    int64_t last_n;    // token count of the most recent online call
    int32_t fx;        // decode kernels accumulate the repair in counted fixed-point words (deterministic results)
    int32_t deterministic;   // every online call runs as decode groups on those accumulators
    float* fx_bound;   // K1, K2 of the accumulators' magnitude bound (device, 2 floats)
    td_stack_layer_dev* stack_desc;   // device copy of this layer's entry for the single-launch stack kernel (or null)
    int32_t stack_fused;              // knob: one-token stacks of such layers run in one launch
    int32_t stack_spin_limit;         // knob: polls a block of that launch spends on one layer's counter before it gives up
    int32_t poisoned;  // a launch of an online call failed half way: counters and accumulators may be left armed
};

static inline size_t td_elem_size(int32_t dtype) { return dtype == TARDIS_BF16 ? 2 : 4; }

// ---------------------------------------------------------------- device helpers
__device__ __forceinline__ float td_bf16_to_f32(bf16_t v) {
    return __uint_as_float(((uint32_t)v) << 16);
}

// round-to-nearest-even; NaN stays NaN
__device__ __forceinline__ bf16_t td_f32_to_bf16(float f) {
    uint32_t u = __float_as_uint(f);
    if ((u & 0x7FFFFFFFu) > 0x7F800000u) return (bf16_t)((u >> 16) | 0x0040u);
    u += 0x7FFFu + ((u >> 16) & 1u);
    return (bf16_t)(u >> 16);
}

// 16-byte load of data that is read once (weights streamed from HBM)
__device__ __forceinline__ td_u32x4 td_load_stream16(const void* p) {
    return __builtin_nontemporal_load(static_cast<const td_u32x4*>(p));
}

template <typename T> __device__ __forceinline__ float td_load(const T* p);
template <> __device__ __forceinline__ float td_load<float>(const float* p) { return *p; }
template <> __device__ __forceinline__ float td_load<bf16_t>(const bf16_t* p) { return td_bf16_to_f32(*p); }

template <typename T> __device__ __forceinline__ void td_store(T* p, float v);
template <> __device__ __forceinline__ void td_store<float>(float* p, float v) { *p = v; }
template <> __device__ __forceinline__ void td_store<bf16_t>(bf16_t* p, float v) { *p = td_f32_to_bf16(v); }

__device__ __forceinline__ float td_wave_sum(float v) {
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
    return v;
}
__device__ __forceinline__ int td_wave_sum_i(int v) {
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
    return v;
}
__device__ __forceinline__ float td_wave_max(float v) {
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v = fmaxf(v, __shfl_xor(v, o, 64));
    return v;
}

// sigma(z) for the four supported activations (fp32)
__device__ __forceinline__ float td_act(float z, int act) {
    switch (act) {
        case TARDIS_ACT_GELU_ERF:
            return 0.5f * z * (1.0f + erff(z * 0.70710678118654752440f));
        case TARDIS_ACT_GELU_TANH: {
            float u = 0.79788456080286535588f * (z + 0.044715f * z * z * z);
            return 0.5f * z * (1.0f + tanhf(u));
        }
        case TARDIS_ACT_RELU:
            return z > 0.0f ? z : 0.0f;
        default:
            return z;
    }
}

// fp64 version for the offline fit
__device__ __forceinline__ double td_act_f64(double z, int act) {
    switch (act) {
        case TARDIS_ACT_GELU_ERF:
            return 0.5 * z * (1.0 + erf(z * 0.70710678118654752440));
        case TARDIS_ACT_GELU_TANH: {
            double u = 0.79788456080286535588 * (z + 0.044715 * z * z * z);
            return 0.5 * z * (1.0 + tanh(u));
        }
        case TARDIS_ACT_RELU:
            return z > 0.0 ? z : 0.0;
        default:
            return z;
    }
}

// ---------------------------------------------------------------- internal launchers
// (each validates nothing: the C-ABI layer in api.cpp has already done so)

// api.hip: memory of destroyed layers that is kept for the next one goes back to the device; false: there was none
bool td_give_back_memory();
struct td_dev_buf {  // frees on scope exit
    void* p = nullptr;
    td_dev_buf() = default;
    td_dev_buf(const td_dev_buf&) = delete;
    td_dev_buf& operator=(const td_dev_buf&) = delete;
    ~td_dev_buf() {
        if (p) (void)hipFree(p);
    }
    tardis_status_t alloc(size_t bytes) {
        hipError_t e = hipMalloc(&p, bytes ? bytes : 16);
        if (e == hipErrorOutOfMemory && td_give_back_memory()) e = hipMalloc(&p, bytes ? bytes : 16);
        if (e != hipSuccess) {
            p = nullptr;
            (void)hipGetLastError();
            return e == hipErrorOutOfMemory ? TARDIS_ERR_OOM : TARDIS_ERR_HIP;
        }
        return TARDIS_OK;
    }
};
// working memory of td_fold (two buffers: up to 64 MiB each is what the runtime keeps for the next call)
struct td_fold_work {
    td_dev_buf terms, sums;
    tardis_status_t alloc(const tardis_ffn_desc* desc) {
        TD_TRY(terms.alloc((size_t)desc->h * 8));
        return desc->dtype == TARDIS_BF16 ? sums.alloc((size_t)desc->d * desc->d * 4) : TARDIS_OK;
    }
};
// offline.hip
// dst = src transposed, copy = src
tardis_status_t td_transpose(const void* src, void* dst, void* copy, int64_t rows, int64_t cols, int32_t dtype, hipStream_t s);
// bits = 8: Q (required).  bits = 4, 3, 2 (codes up to 7, 3, 1 in 4-bit slots): M4 (required), Q
// (effective one-byte codes, optional) and Q4 (packed, optional, needs d % 32 == 0).  margin: fraction
// of every range's width taken off at either end for the predictor's test.  code_scale (bits = 8, bf16; or null): td_code_scale of
// every row; no_scale (zero before) becomes 1 if some row has none.
tardis_status_t td_build_sketch(const void* W1, const void* b1, const float* lo, const float* hi, int64_t h,
                                int64_t d, int32_t dtype, int32_t bits, float margin, int8_t* Q, uint8_t* Q4,
                                uint8_t* M4, float* tlo, float* thi, float* code_scale, int32_t* no_scale, hipStream_t s);
// one-byte effective codes (multiplier * 4-bit code) from the packed 4-bit sketch
tardis_status_t td_unpack_sketch4(const uint8_t* Q4, const uint8_t* M4, int64_t h, int64_t d, int8_t* Q,
                                  hipStream_t s);
// Wp8 / wp8_scale non-null (bf16 layers): W' is stored as e4m3 codes with a power-of-two scale per row, and Wp
// receives the same values as bf16
// work1, work2: h x d elements of the layer dtype each, overwritten
tardis_status_t td_fold(const tardis_ffn_desc* desc, const float* a, const float* c, void* Wp, float* bp,
                        uint8_t* Wp8, float* wp8_scale, void* work1, void* work2, const td_fold_work& work, hipStream_t s);
// step > 0: greedy range search with that increment; step <= 0: central quantile ranges
tardis_status_t td_calibrate(const tardis_ffn_desc* desc, const void* X, int64_t n, float coverage,
                             const float* cov_pn, float step, float* lo, float* hi, float* a, float* c,
                             hipStream_t s);
tardis_status_t td_estimate_errors(const tardis_ffn_desc* desc, const void* X, int64_t n, const float* lo,
                                   const float* hi, const float* a, const float* c, float* err, float* err_layer,
                                   hipStream_t s);
tardis_status_t td_assign_thresholds(const float* err, int64_t n, float t, float t_min, float t_max, float* out,
                                     hipStream_t s);
tardis_status_t td_fx_bounds(const tardis_layer_s* L, float* out2, hipStream_t s);
// gemm.hip:  C[m][n] (+)= sum_k A[m][k] * B[n][k] (+ row_bias[m]); C fp32, ldc = N
tardis_status_t td_gemm_nt(const void* A, const void* B, float* C, int64_t M, int64_t N, int64_t K, int32_t dtype,
                           int accumulate, const void* row_bias, hipStream_t s, void* out16 = nullptr);
bool td_gemm_on_matrix_cores(const void* A, const void* B, int64_t M, int64_t N, int64_t K, int32_t dtype);
bool td_gemm_refuses_rows(int64_t M);
// the products of calls with many tokens, each with the step that follows it (see gemm.hip)
tardis_status_t td_gemm_repair(const tardis_layer_s* L, const int8_t* XQ, const int32_t* e, const void* X, const void* b1,
                               uint32_t* mask, void* out, void* rest, int64_t n, hipStream_t s);
tardis_status_t td_gemm_hidden(const tardis_layer_s* L, const void* X, const void* b1, void* out, int64_t n, hipStream_t s);
tardis_status_t td_gemm_output(const void* X, const void* Wp, const void* H, const void* W2, float* part, int* parts,
                               int64_t n, int64_t d, int64_t h, hipStream_t s);
size_t td_gemm_part_floats(int64_t n, int64_t d);
// stream.hip: the same for up to kStreamMaxTokens tokens
constexpr int64_t kStreamMaxTokens = 64;
// The weights of a launch of stream_kernel and how its blocks divide them; tile = 0: not for that kernel.  (The kernel that runs before
// it asks for what its blocks begin with: that waits in the caches when it starts, and HBM has work meanwhile.)
struct StreamPlan {
    const unsigned char *B, *B2;   // weights: rows of k bytes (and of k2: a second matrix whose K follows)
    int64_t N;
    uint32_t k, k2;
    int tile, splits, slices;      // rows of a block; ranges of K (a power of two), slices of 256 bytes in one
};
constexpr int kStreamSlice = 256;
inline int64_t stream_blocks(const StreamPlan& p) { return (p.N + p.tile - 1) / p.tile * p.splits; }
StreamPlan td_stream_up_plan(const tardis_layer_s* L, int64_t n);
StreamPlan td_stream_output_plan(bool folded, const void* Wp, const void* W2, int64_t n, int64_t d, int64_t h);
tardis_status_t td_stream_repair(const tardis_layer_s* L, const StreamPlan& plan, const int8_t* XQ, const int32_t* e, const void* X,
                                 const void* b1, uint32_t* mask, void* out, void* rest, int64_t n, const StreamPlan& next, hipStream_t s);
tardis_status_t td_stream_output(const StreamPlan& plan, const void* X, const void* H, float* part, int* parts, int64_t n, hipStream_t s);
tardis_status_t td_stream_init();
tardis_status_t td_gemm_init();
// prefill.hip
bool td_prefill_supported(const tardis_layer_s* L);
size_t td_prefill_scratch_bytes(const tardis_layer_s* L);   // for calls of any size, in chunks of prefill_chunk
tardis_status_t td_forward_prefill(tardis_layer_s* L, const void* x, int64_t n, void* y, int norm_out, hipStream_t s);
tardis_status_t td_dense_prefill(tardis_layer_s* L, const void* x, int64_t n, void* y, hipStream_t s);
bool td_layer_is_live(const tardis_layer_s* L);
// decode.hip
tardis_status_t td_decode_init();
bool td_decode_fused_supported(const tardis_layer_s* L);
constexpr int kDecodeMaxTokens = 16;  // tokens one weight pass of the decode kernel can be shared between
// n consecutive tokens (bf16 layers the fused kernels support) as groups of 16, 8, 4, 2, 1 with the
// layer's own working memory
tardis_status_t td_decode_fused(tardis_layer_s* L, const void* x, int64_t n, void* y, int norm_out, hipStream_t s);
// looks up the current device's static decode working memory (once per device)
tardis_status_t td_static_scratch_setup();
tardis_status_t td_mask_union(const tardis_layer_s* L, int64_t n, uint32_t* union_mask, int32_t* union_count,
                              hipStream_t s);
tardis_status_t td_mask_to_list(const tardis_layer_s* L, int64_t n, int32_t* counts, int32_t* list, hipStream_t s);
// stack.hip
tardis_status_t td_stack_init();
bool td_stack_decode_supported(const tardis_layer_s* L);
tardis_status_t td_stack_decode(tardis_layer_s* const* layers, int n_layers, const void* x, void* y, hipStream_t s);
// forward.hip
// norm_out != 0: the output is y / sqrt(mean(y^2) + kRmsEps) per token (glue between stacked layers)
tardis_status_t td_forward(tardis_layer_s* L, const void* x, int64_t n, void* y, int norm_out, hipStream_t s);
tardis_status_t td_dense_forward(tardis_layer_s* L, const void* x, int64_t n, void* y, hipStream_t s);

// Many tokens at once (prompt processing), as dense matrix products.
//
// With hundreds of tokens the union of the flagged neurons is the whole layer (Sec. "Inference
// Runtime" notes that the method does not help prompt processing), so gathering rows per token
// gains nothing; the same per-token result is computed here from three matrix products on the
// matrix cores, each with the step that follows it in its epilogue:
//     ACC = Xq Q^T            exact int32 (the predictor's integer sums) -> range test -> mask words
//     Z   = X W1^T            fp32 accumulate (the exact pre-activations) -> D[t][j] = sigma(z) - (a_j z + c_j)
//                             where token t flagged neuron j, else 0, rounded to bf16
//     Y   = [X | D] [W' | W2]^T   one product over d + h columns, in up to 8 ranges whose fp32 sums the
//                             finishing kernel adds: y = Y + b' (then the optional RMS norm and the conversion)
// (The first d columns could be left out, W'x being the sum over the neurons of a_j z_j W2_j, whose factors are all here, and the
// output product then runs over h columns: 333 tokens 153 -> 143 us, 2048 tokens 573 -> 549 at d = 4096, h = 16384.  But every
// factor is then rounded to bf16 before the sum over the neurons, W' once behind it: where the sum is 2^-6 of its terms, y is off by
// 15 % instead of 0.2 %, and a pre-activation beyond 32 bits makes a NaN of a y that is an ordinary number.)
// Calls with few tokens on some layers (fine_max_tokens) keep what the rounding of D left as well and add its product
// with W2^T: the kernels that serve fewer tokens multiply factors of 32 bits.
// Up to 64 tokens the products stream the weights (stream.hip) where they can, and the first two read W1 alone.
// Neither the sums nor the pre-activations (n x h, 4 bytes each) reach memory.  Masks are bit-exact with
// the per-token path (same integer sums, same range test).
#include "common.h"
#include "rowdot.h"
#include "tiles.h"

namespace {

// int8 code and exponent of every token (one block per token; d % 8 == 0).  COPY: x is not 16-byte
// aligned; an aligned copy is left for the products.
// Blocks from `tokens` on (next.tile: the launch behind this one is a stream_kernel) ask for the weights that its blocks begin with.
template <bool COPY>
__global__ void __launch_bounds__(256)
quantize_rows_kernel(const bf16_t* __restrict__ X, int d, int8_t* __restrict__ XQ, int32_t* __restrict__ E,
                     bf16_t* __restrict__ XC, int tokens, StreamPlan next) {
    __shared__ float red[4];
    const int t = blockIdx.x;
    if (t >= tokens) {                               // (from a multiple of 8 on: on the XCD that needs them)
        const int block = t - (tokens + 7) / 8 * 8;
        if (block < 0) return;
        const StreamBlock b = stream_block(next, block);
        uint32_t got[kWarmSlices] = {};
#pragma unroll
        for (int u = 0; u < kWarmSlices; ++u) {
            const uint32_t* from = stream_warm(next, b, (int)threadIdx.x + u * 256);
            if (from) got[u] = *from;
        }
#pragma unroll
        for (int u = 0; u < kWarmSlices; ++u) asm volatile("" ::"v"(got[u]));
        return;
    }
    const bf16_t* x = X + (size_t)t * d;
    auto load8 = [&](int v, bf16_t (&o)[8]) {
        if constexpr (COPY) {
#pragma unroll
            for (int u = 0; u < 8; ++u) o[u] = x[v * 8 + u];
        } else {
            const td_u32x4 w = reinterpret_cast<const td_u32x4*>(x)[v];
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                o[2 * u] = (bf16_t)(w[u] & 0xffffu);
                o[2 * u + 1] = (bf16_t)(w[u] >> 16);
            }
        }
    };
    constexpr int kKeep = 2;                         // vectors a thread keeps between the two passes (d <= 4096: all)
    bf16_t keep[kKeep][8];
    float m = 0.0f;
#pragma unroll
    for (int i = 0; i < kKeep; ++i) {
        const int v = i * 256 + (int)threadIdx.x;
        if (v < d / 8) {
            load8(v, keep[i]);
#pragma unroll
            for (int u = 0; u < 8; ++u) m = fmaxf(m, fabsf(td_bf16_to_f32(keep[i][u])));
        }
    }
    for (int v = kKeep * 256 + (int)threadIdx.x; v < d / 8; v += 256) {
        bf16_t o[8];
        load8(v, o);
#pragma unroll
        for (int u = 0; u < 8; ++u) m = fmaxf(m, fabsf(td_bf16_to_f32(o[u])));
    }
    m = td_wave_max(m);
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = m;
    __syncthreads();
    m = fmaxf(fmaxf(red[0], red[1]), fmaxf(red[2], red[3]));
    const int e = token_exponent(m);
    auto put8 = [&](int v, const bf16_t (&o)[8]) {
        uint32_t q[2] = {0u, 0u};
#pragma unroll
        for (int u = 0; u < 8; ++u)
            q[u >> 2] |= (uint32_t)(uint8_t)quantize_value(td_bf16_to_f32(o[u]), e) << (8 * (u & 3));
        *reinterpret_cast<uint2*>(XQ + (size_t)t * d + v * 8) = make_uint2(q[0], q[1]);
        if constexpr (COPY) {
            td_u32x4 w;
#pragma unroll
            for (int u = 0; u < 4; ++u) w[u] = (uint32_t)o[2 * u] | ((uint32_t)o[2 * u + 1] << 16);
            *reinterpret_cast<td_u32x4*>(XC + (size_t)t * d + v * 8) = w;
        }
    };
#pragma unroll
    for (int i = 0; i < kKeep; ++i) {
        const int v = i * 256 + (int)threadIdx.x;
        if (v < d / 8) put8(v, keep[i]);
    }
    for (int v = kKeep * 256 + (int)threadIdx.x; v < d / 8; v += 256) {
        bf16_t o[8];
        load8(v, o);
        put8(v, o);
    }
    if (threadIdx.x == 0) E[t] = e;
}

// y[t] = sum over the parts of Y[t] + bias (optionally RMS-normalised); d % 4 == 0.  One block per token with the
// norm, which needs whole rows; gridDim.y blocks of 1024 columns each per token without (64 tokens: 7.3 -> 4.6 us).
// bias: fp32 (b') or bf16 (b2), or neither.
__global__ void __launch_bounds__(256)
finish_rows_kernel(const float* __restrict__ Y, int parts, size_t part_stride, const float* __restrict__ bias32,
                   const bf16_t* __restrict__ bias16, int d, bf16_t* __restrict__ y, int vector_store, int norm_out,
                   float eps) {
    __shared__ float red[4];
    const int t = blockIdx.x;
    const float* row = Y + (size_t)t * d;
    auto value = [&](int v) {
        float4 s = reinterpret_cast<const float4*>(row)[v];
        for (int k = 1; k < parts; ++k) {
            const float4 a = reinterpret_cast<const float4*>(row + k * part_stride)[v];
            s.x += a.x;
            s.y += a.y;
            s.z += a.z;
            s.w += a.w;
        }
        if (bias32) {
            const float4 b = reinterpret_cast<const float4*>(bias32)[v];
            s.x += b.x;
            s.y += b.y;
            s.z += b.z;
            s.w += b.w;
        } else if (bias16) {
            s.x += td_bf16_to_f32(bias16[4 * v]);
            s.y += td_bf16_to_f32(bias16[4 * v + 1]);
            s.z += td_bf16_to_f32(bias16[4 * v + 2]);
            s.w += td_bf16_to_f32(bias16[4 * v + 3]);
        }
        return s;
    };
    float scale = 1.0f;
    if (norm_out) {
        float ss = 0.0f;
        for (int v = threadIdx.x; v < d / 4; v += 256) {
            const float4 s = value(v);
            ss += s.x * s.x + s.y * s.y + s.z * s.z + s.w * s.w;
        }
        ss = td_wave_sum(ss);
        if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = ss;
        __syncthreads();
        scale = 1.0f / sqrtf((red[0] + red[1] + red[2] + red[3]) / (float)d + eps);
    }
    for (int v = (int)blockIdx.y * 256 + (int)threadIdx.x; v < d / 4; v += (int)gridDim.y * 256) {
        const float4 s = value(v);
        const bf16_t o[4] = {td_f32_to_bf16(s.x * scale), td_f32_to_bf16(s.y * scale), td_f32_to_bf16(s.z * scale),
                             td_f32_to_bf16(s.w * scale)};
        bf16_t* dst = y + (size_t)t * d + 4 * v;
        if (vector_store)
            *reinterpret_cast<uint2*>(dst) = make_uint2((uint32_t)o[0] | ((uint32_t)o[1] << 16),
                                                        (uint32_t)o[2] | ((uint32_t)o[3] << 16));
        else
#pragma unroll
            for (int u = 0; u < 4; ++u) dst[u] = o[u];
    }
}

// Scratch of one chunk of n tokens
struct PromptScratch {
    int8_t* xq;
    int32_t* e;
    bf16_t* x;          // aligned copy of the tokens (used when the caller's are not 16-byte aligned)
    bf16_t* hid;        // repair factors D, or the dense hidden activations (n x h)
    bf16_t* rest;       // fine: remainders of D (n x h)
    float* part;        // partial sums of the output (fine: of both products)
    size_t bytes;
    PromptScratch(void* base, int64_t n, int64_t d, int64_t h, bool fine) {
        unsigned char* p = static_cast<unsigned char*>(base);
        auto take = [&](size_t b) {
            unsigned char* at = p;
            p += (b + 255) / 256 * 256;
            return at;
        };
        xq = reinterpret_cast<int8_t*>(take((size_t)n * d));
        e = reinterpret_cast<int32_t*>(take((size_t)n * 4));
        x = reinterpret_cast<bf16_t*>(take((size_t)n * d * 2));
        hid = reinterpret_cast<bf16_t*>(take((size_t)n * h * 2));
        rest = reinterpret_cast<bf16_t*>(take(fine ? (size_t)n * h * 2 : 0));
        part = reinterpret_cast<float*>(take((fine ? 2 : 1) * td_gemm_part_floats(n, d) * 4));
        bytes = (size_t)(p - static_cast<unsigned char*>(base));
    }
};

bool aligned(const void* p, uintptr_t to) { return (reinterpret_cast<uintptr_t>(p) & (to - 1)) == 0; }

void finish(const PromptScratch& w, int parts, const float* bias32, const bf16_t* bias16, int64_t n, int64_t d, bf16_t* y,
            int norm_out, hipStream_t s) {
    hipLaunchKernelGGL(finish_rows_kernel, dim3((unsigned)n, norm_out ? 1u : (unsigned)((d + 1023) / 1024)), dim3(256), 0, s, w.part, parts, (size_t)n * d, bias32, bias16,
                       (int)d, y, aligned(y, 8) ? 1 : 0, norm_out, kRmsEps);
}

tardis_status_t output(const StreamPlan& plan, const void* X, const void* Wp, const void* H, const void* W2, float* part, int* parts,
                       int64_t n, int64_t d, int64_t h, hipStream_t s) {
    return plan.tile ? td_stream_output(plan, X, H, part, parts, n, s) : td_gemm_output(X, Wp, H, W2, part, parts, n, d, h, s);
}

// codes and exponents; the tokens as the products can read them.  next: the launch that follows, if it is a stream_kernel
const bf16_t* quantize(const PromptScratch& w, const bf16_t* x, int64_t n, int64_t d, const StreamPlan& next, hipStream_t s) {
    const int64_t blocks = next.tile ? (n + 7) / 8 * 8 + stream_blocks(next) : n;
    hipLaunchKernelGGL(aligned(x, 16) ? quantize_rows_kernel<false> : quantize_rows_kernel<true>, dim3((unsigned)blocks), dim3(256), 0, s, x, (int)d, w.xq, w.e, w.x, (int)n, next);
    return aligned(x, 16) ? x : w.x;
}

}  // namespace

bool td_prefill_supported(const tardis_layer_s* L) {
    return L->dtype == TARDIS_BF16 && L->d % 128 == 0 && L->h >= 128 && L->h % 8 == 0;
}

size_t td_prefill_scratch_bytes(const tardis_layer_s* L) {
    const int64_t chunk = L->prefill_chunk, fine = L->fine_max_tokens < chunk ? L->fine_max_tokens : chunk;
    const size_t all = PromptScratch(nullptr, chunk, L->d, L->h, false).bytes;
    const size_t few = fine > 0 ? PromptScratch(nullptr, fine, L->d, L->h, true).bytes : 0;
    return all > few ? all : few;                    // (either grows with its number of tokens)
}

// one chunk of at most L->prefill_chunk tokens (the scratch is sized for that many)
static tardis_status_t prefill_chunk(tardis_layer_s* L, const bf16_t* x, int64_t n, bf16_t* y, uint32_t* mask,
                                     bool fine, int norm_out, hipStream_t s) {
    const int64_t d = L->d, h = L->h;
    const PromptScratch w(L->pf_scratch, n, d, h, fine);
    const StreamPlan up = td_stream_up_plan(L, n);
    const StreamPlan down = td_stream_output_plan(true, L->Wp, L->W2, n, d, h);
    x = quantize(w, x, n, d, up, s);
    const void* b1 = L->b1 ? L->b1 : L->zeros_h;
    void* rest = fine ? w.rest : nullptr;
    if (up.tile) TD_TRY(td_stream_repair(L, up, w.xq, w.e, x, b1, mask, w.hid, rest, n, down, s));
    else TD_TRY(td_gemm_repair(L, w.xq, w.e, x, b1, mask, w.hid, rest, n, s));
    int parts = 1, more = 0;
    TD_TRY(output(down, x, L->Wp, w.hid, L->W2, w.part, &parts, n, d, h, s));
    if (fine)
        TD_TRY(output(td_stream_output_plan(false, nullptr, L->W2, n, d, h), nullptr, nullptr, w.rest, L->W2, w.part + (size_t)parts * n * d, &more, n, d, h, s));
    parts += more;
    finish(w, parts, L->bp, nullptr, n, d, y, norm_out, s);
    TD_HIP(hipGetLastError());
    return TARDIS_OK;
}

// Long prompts run in chunks of L->prefill_chunk tokens (tokens are independent): the scratch and
// the launch grids stay bounded whatever max_batch is.
tardis_status_t td_forward_prefill(tardis_layer_s* L, const void* xv, int64_t n, void* yv, int norm_out,
                                   hipStream_t s) {
    const bf16_t* x = static_cast<const bf16_t*>(xv);
    bf16_t* y = static_cast<bf16_t*>(yv);
    for (int64_t t0 = 0; t0 < n; t0 += L->prefill_chunk) {
        const int64_t nc = n - t0 < L->prefill_chunk ? n - t0 : L->prefill_chunk;
        TD_TRY(prefill_chunk(L, x + t0 * L->d, nc, y + t0 * L->d, L->mask + t0 * L->mask_words, n <= L->fine_max_tokens, norm_out, s));
    }
    L->last_n = n;
    return TARDIS_OK;
}

// The unmodified FFN on many tokens: two matrix-core products, the activation in the first one's epilogue
// (the hidden activations are rounded to bf16, as the per-token dense kernels round them).
tardis_status_t td_dense_prefill(tardis_layer_s* L, const void* xv, int64_t n, void* yv, hipStream_t s) {
    const int64_t d = L->d, h = L->h;
    for (int64_t t0 = 0; t0 < n; t0 += L->prefill_chunk) {
        const int64_t nc = n - t0 < L->prefill_chunk ? n - t0 : L->prefill_chunk;
        const PromptScratch w(L->pf_scratch, nc, d, h, false);
        const bf16_t* x = static_cast<const bf16_t*>(xv) + t0 * d;
        if (!aligned(x, 16)) x = quantize(w, x, nc, d, StreamPlan{}, s);
        TD_TRY(td_gemm_hidden(L, x, L->b1 ? L->b1 : L->zeros_h, w.hid, nc, s));
        int parts = 1;
        TD_TRY(output(td_stream_output_plan(false, nullptr, L->W2, nc, d, h), nullptr, nullptr, w.hid, L->W2, w.part, &parts, nc, d, h, s));
        finish(w, parts, nullptr, static_cast<const bf16_t*>(L->b2), nc, d, static_cast<bf16_t*>(yv) + t0 * d, 0, s);
    }
    TD_HIP(hipGetLastError());
    return TARDIS_OK;
}

// Online path of the partially-linear FFN (Sec. "Inference Runtime"):
//   speculative result  y = W'x + b'
//   predictor           int8 sketch of W1 against an int8 code of x, range test,
//                       flagged neurons compacted into a list
//   result fixing       for each flagged neuron j: z_j = W1[j].x + b1_j,
//                       y += (sigma(z_j) - (a_j z_j + c_j)) * W2[:, j]
// plus the unmodified FFN on the same row-streaming core (the dense baseline).
//
// One token is bound by HBM bandwidth: each weight row is read once per token (the
// tokens of a call share rows through the caches only) with 16-byte loads per
// lane, one wavefront per row, the token staged in LDS, and the per-row reduction
// done with cross-lane shuffles.
#include "common.h"
#include "rowdot.h"

#include <hip/amd_detail/amd_hip_unsafe_atomics.h>

namespace {

constexpr int kBlock = 256;                 // 4 wavefronts
constexpr int kWaves = kBlock / TD_WAVE;
constexpr int kPredRowsPerWave = 8;         // 4 waves x 8 rows = one 32-bit mask word per block
constexpr int kGemvRowsPerWave = 4;

// ------------------------------------------------------------ token staging
// Copies x (d values) into LDS; returns max|x_k| over the block (all threads).
template <typename T>
__device__ __forceinline__ float stage_token(const T* __restrict__ x, T* xs, int d, float* red) {
    float m = 0.0f;
    for (int k = threadIdx.x; k < d; k += kBlock) {
        const T v = x[k];
        xs[k] = v;
        m = fmaxf(m, fabsf(td_load<T>(&v)));
    }
    m = td_wave_max(m);
    if ((threadIdx.x & (TD_WAVE - 1)) == 0) red[threadIdx.x / TD_WAVE] = m;
    __syncthreads();
    float r = red[0];
#pragma unroll
    for (int w = 1; w < kWaves; ++w) r = fmaxf(r, red[w]);
    return r;
}

// ----------------------------------------------- folded product + predictor
// blockIdx.y = token.  Blocks [0, gemv_blocks) compute rows of W'x + b' into yacc (fp32).
// Blocks [gemv_blocks, gemv_blocks + pred_blocks) each own 32 consecutive
// neurons: they form the block's mask word and append the flagged indices to
// the token's list.
template <typename T>
__global__ void __launch_bounds__(kBlock)
fold_predict_kernel(const T* __restrict__ Wp, const float* __restrict__ bp, const int8_t* __restrict__ Q,
                    const float* __restrict__ tlo, const float* __restrict__ thi, const T* __restrict__ x,
                    float* __restrict__ yacc, uint32_t* __restrict__ mask, int32_t* __restrict__ count,
                    int32_t* __restrict__ list, int d, int h, int gemv_blocks) {
    extern __shared__ __align__(16) unsigned char smem[];
    T* xs = reinterpret_cast<T*>(smem);
    int8_t* xq = reinterpret_cast<int8_t*>(smem + (((size_t)d * sizeof(T) + 15) & ~(size_t)15));
    __shared__ float red[kWaves];
    __shared__ uint32_t word_parts[kWaves];
    __shared__ int list_base;

    const int lane = threadIdx.x & (TD_WAVE - 1);
    const int wave = threadIdx.x / TD_WAVE;
    const size_t tok = blockIdx.y;
    x += tok * d;
    yacc += tok * d;
    mask += tok * ((h + 31) / 32);
    count += tok;
    list += tok * h;
    const float m = stage_token<T>(x, xs, d, red);

    if ((int)blockIdx.x < gemv_blocks) {
        __syncthreads();
        const int r0 = ((int)blockIdx.x * kWaves + wave) * kGemvRowsPerWave;
        const T* rows[kGemvRowsPerWave];
#pragma unroll
        for (int i = 0; i < kGemvRowsPerWave; ++i) rows[i] = (r0 + i < d) ? Wp + (size_t)(r0 + i) * d : nullptr;
        float out[kGemvRowsPerWave];
        rows_dot<T, kGemvRowsPerWave>(rows, xs, d, lane, out);
        if (lane == 0) {
#pragma unroll
            for (int i = 0; i < kGemvRowsPerWave; ++i)
                if (r0 + i < d) yacc[r0 + i] = out[i] + bp[r0 + i];
        }
        return;
    }

    // ---- predictor block
    const int e = token_exponent(m);
    for (int k = threadIdx.x; k < d; k += kBlock) xq[k] = quantize_value(td_load<T>(xs + k), e);
    __syncthreads();

    const int pb = (int)blockIdx.x - gemv_blocks;
    const int j0 = pb * 32 + wave * kPredRowsPerWave;
    const int8_t* rows[kPredRowsPerWave];
#pragma unroll
    for (int i = 0; i < kPredRowsPerWave; ++i) rows[i] = (j0 + i < h) ? Q + (size_t)(j0 + i) * d : nullptr;
    int acc[kPredRowsPerWave];
    rows_dot_i8<kPredRowsPerWave>(rows, xq, d, lane, acc);

    uint32_t bits = 0;
#pragma unroll
    for (int i = 0; i < kPredRowsPerWave; ++i) {
        if (j0 + i < h) {
            const float v = ldexpf((float)acc[i], e);
            const bool inside = (v >= tlo[j0 + i]) && (v < thi[j0 + i]);
            if (!inside) bits |= 1u << i;
        }
    }
    if (lane == 0) word_parts[wave] = bits << (wave * kPredRowsPerWave);
    __syncthreads();
    uint32_t word = 0;
#pragma unroll
    for (int w = 0; w < kWaves; ++w) word |= word_parts[w];
    if (threadIdx.x == 0) {
        mask[pb] = word;
        const int n = __popc(word);
        list_base = n ? atomicAdd(count, n) : 0;
    }
    __syncthreads();
    if (threadIdx.x < 32 && ((word >> threadIdx.x) & 1u)) {
        const int rank = __popc(word & ((1u << threadIdx.x) - 1u));
        if (list_base + rank < h) list[list_base + rank] = pb * 32 + (int)threadIdx.x;
    }
}

// ------------------------------------------------------------ result fixing
// blockIdx.y = token; one wavefront per flagged neuron (grid-stride over the device-side count).
template <typename T>
__global__ void __launch_bounds__(kBlock)
fix_kernel(const T* __restrict__ W1, const T* __restrict__ b1, const T* __restrict__ W2T,
           const float* __restrict__ a, const float* __restrict__ c, const T* __restrict__ x,
           const int32_t* __restrict__ count, const int32_t* __restrict__ list, float* __restrict__ yacc, int d,
           int h, int act) {
    extern __shared__ __align__(16) unsigned char smem[];
    T* xs = reinterpret_cast<T*>(smem);
    const size_t tok = blockIdx.y;
    x += tok * d;
    yacc += tok * d;
    list += tok * h;
    const int n = min(count[tok], h);
    const int lane = threadIdx.x & (TD_WAVE - 1);
    const int gw = (int)blockIdx.x * kWaves + threadIdx.x / TD_WAVE;
    const int total = (int)gridDim.x * kWaves;
    if ((int)blockIdx.x * kWaves >= n) return;  // whole block idle (uniform)
    for (int k = threadIdx.x; k < d; k += kBlock) xs[k] = x[k];
    __syncthreads();

    for (int i = gw; i < n; i += total) {
        const int j = list[i];
        if (j < 0 || j >= h) continue;
        const T* rows[1] = {W1 + (size_t)j * d};
        float z[1];
        rows_dot<T, 1>(rows, xs, d, lane, z);
        float zj = z[0];
        if (b1) zj += td_load<T>(b1 + j);
        const float delta = td_act(zj, act) - fmaf(a[j], zj, c[j]);
        const T* w2 = W2T + (size_t)j * d;
        // (a lane per column: the atomics of a wavefront fall on whole lines; 16-byte loads would spread every one of
        //  them over eight lines: d=256, h=1024, bf16, 27 -> 13 us a token)
#pragma unroll 4
        for (int k = lane; k < d; k += TD_WAVE) unsafeAtomicAdd(yacc + k, delta * td_load<T>(w2 + k));
    }
}

// fp32 accumulator -> output dtype (one block per token; optionally y / sqrt(mean(y^2) + eps))
template <typename T>
__global__ void __launch_bounds__(kBlock)
finish_kernel(const float* __restrict__ yacc, T* __restrict__ y, int32_t* __restrict__ count, int d, int norm_out, float eps) {
    __shared__ float red[kWaves];
    yacc += (size_t)blockIdx.x * d;
    y += (size_t)blockIdx.x * d;
    if (threadIdx.x == 0) count[blockIdx.x] = 0;     // (the counters are zero between calls)
    float scale = 1.0f;
    if (norm_out) {
        float ss = 0.0f;
        for (int k = threadIdx.x; k < d; k += kBlock) ss += yacc[k] * yacc[k];
        ss = td_wave_sum(ss);
        if ((threadIdx.x & (TD_WAVE - 1)) == 0) red[threadIdx.x / TD_WAVE] = ss;
        __syncthreads();
        float tot = 0.0f;
#pragma unroll
        for (int w = 0; w < kWaves; ++w) tot += red[w];
        scale = 1.0f / sqrtf(tot / (float)d + eps);
    }
    for (int k = threadIdx.x; k < d; k += kBlock) td_store<T>(y + k, yacc[k] * scale);
}

// ------------------------------------------------------------- small layers
// The whole step of one token in one block (blockIdx.x = token): for a layer whose W' and predictor rows a single
// compute unit reads in a few microseconds, launches are what the steps above spend their time on.  Rows are shared
// by `lanes` lanes each (a power of two, about one 16-byte vector a lane), so that short rows fill a wavefront.
// Bound: four dependent round trips to L2 (token; W' and Q rows; W1 rows; W2^T rows).
// d=64, h=256, fp32: 1 token 15 -> 7.4 us, 32 tokens 392 -> 8.2 us (four launches for every token before).
constexpr int kSmallBlock = 1024;
constexpr int kSmallWaves = kSmallBlock / TD_WAVE;

// row . x over `lanes` lanes of which this is number `sub`; every lane of the wavefront calls it (row null: 0)
template <typename T>
__device__ __forceinline__ float shared_row_dot(const T* row, const T* xs, int n, int sub, int lanes) {
    constexpr int V = RowVec<T>::N;
    float acc = 0.0f;
    if (row) {
        if (n % V == 0) {
#pragma unroll 4
            for (int v = sub; v < n / V; v += lanes)
                acc = RowVec<T>::dot(reinterpret_cast<const td_u32x4*>(row)[v], reinterpret_cast<const td_u32x4*>(xs)[v], acc);
        } else {
            for (int k = sub; k < n; k += lanes) acc = fmaf(td_load<T>(row + k), td_load<T>(xs + k), acc);
        }
    }
    for (int o = lanes >> 1; o > 0; o >>= 1) acc += __shfl_xor(acc, o, 64);
    return acc;
}

__device__ __forceinline__ int shared_row_dot_i8(const int8_t* row, const int8_t* xq, int n, int sub, int lanes) {
    int acc = 0;
    if (row) {
        if (n % 16 == 0) {
#pragma unroll 4
            for (int v = sub; v < n / 16; v += lanes) {
                const td_u32x4 w = reinterpret_cast<const td_u32x4*>(row)[v], x = reinterpret_cast<const td_u32x4*>(xq)[v];
#pragma unroll
                for (int u = 0; u < 4; ++u) acc = __builtin_amdgcn_sdot4((int)w[u], (int)x[u], acc, false);
            }
        } else {
            for (int k = sub; k < n; k += lanes) acc += (int)row[k] * (int)xq[k];
        }
    }
    for (int o = lanes >> 1; o > 0; o >>= 1) acc += __shfl_xor(acc, o, 64);
    return acc;
}

// LDS: token, its code, y (d floats), partial sums (max(d, 1024) floats), flagged neurons and their factors, mask words
struct SmallLds {
    size_t xq, y, part, list, delta, words, bytes;
    __host__ __device__ SmallLds(int d, int h, size_t es) {
        auto up = [](size_t b) { return (b + 15) & ~(size_t)15; };
        xq = up((size_t)d * es);
        y = xq + up((size_t)d);
        part = y + up((size_t)d * 4);
        list = part + up((size_t)(d > kSmallBlock ? d : kSmallBlock) * 4);
        delta = list + up((size_t)h * 4);
        words = delta + up((size_t)h * 4);
        bytes = words + up((size_t)((h + 31) / 32) * 4);
    }
};

template <typename T>
__global__ void __launch_bounds__(kSmallBlock)
small_layer_kernel(const T* __restrict__ Wp, const float* __restrict__ bp, const int8_t* __restrict__ Q,
                   const float* __restrict__ tlo, const float* __restrict__ thi, const T* __restrict__ W1,
                   const T* __restrict__ b1, const T* __restrict__ W2T, const float* __restrict__ a,
                   const float* __restrict__ c, const T* __restrict__ x, T* __restrict__ y, uint32_t* __restrict__ mask,
                   int d, int h, int act, int norm_out, float eps, int lanes, int lanes_i8) {
    extern __shared__ __align__(16) unsigned char smem[];
    __shared__ float red[kSmallWaves];
    __shared__ int flagged;
    const SmallLds at(d, h, sizeof(T));
    T* xs = reinterpret_cast<T*>(smem);
    int8_t* xq = reinterpret_cast<int8_t*>(smem + at.xq);
    float* ys = reinterpret_cast<float*>(smem + at.y);
    float* part = reinterpret_cast<float*>(smem + at.part);
    int* list = reinterpret_cast<int*>(smem + at.list);
    float* delta = reinterpret_cast<float*>(smem + at.delta);
    uint32_t* words = reinterpret_cast<uint32_t*>(smem + at.words);
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int nwords = (h + 31) / 32;
    x += (size_t)blockIdx.x * d;
    y += (size_t)blockIdx.x * d;
    mask += (size_t)blockIdx.x * nwords;

    float m = 0.0f;
    for (int k = tid; k < d; k += kSmallBlock) {
        const T v = x[k];
        xs[k] = v;
        m = fmaxf(m, fabsf(td_load<T>(&v)));
    }
    for (int w = tid; w < nwords; w += kSmallBlock) words[w] = 0u;
    if (tid == 0) flagged = 0;
    m = td_wave_max(m);
    if (lane == 0) red[wave] = m;
    __syncthreads();
#pragma unroll
    for (int w = 0; w < kSmallWaves; ++w) m = fmaxf(m, red[w]);
    const int e = token_exponent(m);
    for (int k = tid; k < d; k += kSmallBlock) xq[k] = quantize_value(td_load<T>(xs + k), e);
    __syncthreads();

    // speculative rows, then the predictor
    for (int r0 = wave * (64 / lanes); r0 < d; r0 += kSmallWaves * (64 / lanes)) {
        const int r = r0 + lane / lanes, sub = lane % lanes;
        const float v = shared_row_dot<T>(r < d ? Wp + (size_t)r * d : nullptr, xs, d, sub, lanes);
        if (r < d && sub == 0) ys[r] = v + bp[r];
    }
    for (int j0 = wave * (64 / lanes_i8); j0 < h; j0 += kSmallWaves * (64 / lanes_i8)) {
        const int j = j0 + lane / lanes_i8, sub = lane % lanes_i8;
        const int acc = shared_row_dot_i8(j < h ? Q + (size_t)j * d : nullptr, xq, d, sub, lanes_i8);
        if (j < h && sub == 0) {
            const float v = ldexpf((float)acc, e);
            if (!((v >= tlo[j]) && (v < thi[j]))) {
                list[atomicAdd(&flagged, 1)] = j;
                atomicOr(&words[j >> 5], 1u << (j & 31));
            }
        }
    }
    __syncthreads();
    const int n = flagged;
    for (int w = tid; w < nwords; w += kSmallBlock) mask[w] = words[w];

    // repair factors of the flagged neurons, then their rows of W2^T: `groups` groups of threads take every
    // groups-th neuron and the columns k, k + (threads of the group), ...
    for (int i0 = wave * (64 / lanes); i0 < n; i0 += kSmallWaves * (64 / lanes)) {
        const int i = i0 + lane / lanes, sub = lane % lanes;
        const int j = i < n ? list[i] : 0;
        float z = shared_row_dot<T>(i < n ? W1 + (size_t)j * d : nullptr, xs, d, sub, lanes);
        if (i < n && sub == 0) {
            if (b1) z += td_load<T>(b1 + j);
            delta[i] = td_act(z, act) - fmaf(a[j], z, c[j]);
        }
    }
    __syncthreads();
    const int groups = d < kSmallBlock ? kSmallBlock / d : 1;
    const int g = d < kSmallBlock ? tid / d : 0;
    for (int k = d < kSmallBlock ? tid % d : tid; k < d && g < groups; k += kSmallBlock) {
        float s = 0.0f;
#pragma unroll 4
        for (int i = g; i < n; i += groups) s = fmaf(delta[i], td_load<T>(W2T + (size_t)list[i] * d + k), s);
        part[g * d + k] = s;                          // (groups * d <= max(d, 1024))
    }
    __syncthreads();
    float ss = 0.0f;
    for (int k = tid; k < d; k += kSmallBlock) {
        float v = ys[k];
        for (int q = 0; q < groups; ++q) v += part[q * d + k];
        ys[k] = v;
        ss += v * v;
    }
    float scale = 1.0f;
    if (norm_out) {
        ss = td_wave_sum(ss);
        if (lane == 0) red[wave] = ss;
        __syncthreads();
        float tot = 0.0f;
#pragma unroll
        for (int w = 0; w < kSmallWaves; ++w) tot += red[w];
        scale = 1.0f / sqrtf(tot / (float)d + eps);
    }
    for (int k = tid; k < d; k += kSmallBlock) td_store<T>(y + k, ys[k] * scale);
}

// What one compute unit reads per token before the flags are known; up to this much the one-block form is the
// faster one.  One token, one block / three launches, us: 32 KB 7.4 / 15, 128 KB (d=128, h=512, fp32) 12 / 16, 273 KB 39 / 35,
// 288 KB 25 / 15.
constexpr size_t kSmallLayerBytes = 128 * 1024;

bool small_layer(const tardis_layer_s* L) {
    const size_t es = td_elem_size(L->dtype);
    return (size_t)L->d * L->d * es + (size_t)L->d * L->h <= kSmallLayerBytes &&
           SmallLds((int)L->d, (int)L->h, es).bytes <= 60 * 1024;
}

// lanes that share a row of `vectors` 16-byte vectors
int lanes_for(int64_t vectors) {
    int lanes = 1;
    while (lanes < TD_WAVE && lanes < vectors) lanes *= 2;
    return lanes;
}

// -------------------------------------------------------------- dense FFN
// out[r] = post(rows[r] . x + bias[r]) for r < n_rows; x has n_in values.  blockIdx.y = token.
template <typename T, bool kActivate>
__global__ void __launch_bounds__(kBlock)
dense_rows_kernel(const T* __restrict__ W, const T* __restrict__ bias, const T* __restrict__ x,
                  T* __restrict__ out, int n_rows, int n_in, int act, int x_in_lds) {
    extern __shared__ __align__(16) unsigned char smem[];
    x += (size_t)blockIdx.y * n_in;
    out += (size_t)blockIdx.y * n_rows;
    const T* xs = x;
    if (x_in_lds) {
        T* s = reinterpret_cast<T*>(smem);
        for (int k = threadIdx.x; k < n_in; k += kBlock) s[k] = x[k];
        __syncthreads();
        xs = s;
    }
    const int lane = threadIdx.x & (TD_WAVE - 1);
    const int wave = threadIdx.x / TD_WAVE;
    const int r0 = ((int)blockIdx.x * kWaves + wave) * kGemvRowsPerWave;
    const T* rows[kGemvRowsPerWave];
#pragma unroll
    for (int i = 0; i < kGemvRowsPerWave; ++i) rows[i] = (r0 + i < n_rows) ? W + (size_t)(r0 + i) * n_in : nullptr;
    float o[kGemvRowsPerWave];
    rows_dot<T, kGemvRowsPerWave>(rows, xs, n_in, lane, o);
    if (lane == 0) {
#pragma unroll
        for (int i = 0; i < kGemvRowsPerWave; ++i) {
            if (r0 + i < n_rows) {
                float v = o[i];
                if (bias) v += td_load<T>(bias + r0 + i);
                if (kActivate) v = td_act(v, act);
                td_store<T>(out + r0 + i, v);
            }
        }
    }
}

inline int div_up(int64_t a, int64_t b) { return (int)((a + b - 1) / b); }

template <typename T>
tardis_status_t forward_t(tardis_layer_s* L, const void* xv, int64_t n, void* yv, int norm_out, hipStream_t s) {
    const int d = (int)L->d, h = (int)L->h;
    const size_t xs_bytes = (((size_t)d * sizeof(T) + 15) & ~(size_t)15);
    const int gemv_blocks = div_up(d, kWaves * kGemvRowsPerWave);
    const int pred_blocks = div_up(h, 32);
    const int fix_blocks = 256;
    // (a deterministic layer runs every call as decode groups on the counted fixed-point accumulators: one
    //  rounding for every number of tokens)
    if (!L->deterministic && L->pf_scratch && L->Q && n >= L->prefill_min_tokens)
        return td_forward_prefill(L, xv, n, yv, norm_out, s);
    if (L->use_fused) {   // groups of 16, 8, 4, 2, 1 tokens share one pass over the weights
        TD_TRY(td_decode_fused(L, xv, n, yv, norm_out, s));
        L->last_n = n;
        return TARDIS_OK;
    }
    if (small_layer(L)) {
        constexpr int V = RowVec<T>::N;
        hipLaunchKernelGGL(small_layer_kernel<T>, dim3((unsigned)n), dim3(kSmallBlock), SmallLds(d, h, sizeof(T)).bytes, s,
                           static_cast<const T*>(L->Wp), L->bp, L->Q, L->tlo, L->thi, static_cast<const T*>(L->W1),
                           static_cast<const T*>(L->b1), static_cast<const T*>(L->W2T), L->a, L->c,
                           static_cast<const T*>(xv), static_cast<T*>(yv), L->mask, d, h, (int)L->act, norm_out, kRmsEps,
                           lanes_for((d + V - 1) / V), lanes_for((d + 15) / 16));
        TD_HIP(hipGetLastError());
        L->last_n = n;
        return TARDIS_OK;
    }
    // (at most 65535 tokens per launch: max_batch is far below)
    hipLaunchKernelGGL(fold_predict_kernel<T>, dim3(gemv_blocks + pred_blocks, (unsigned)n), dim3(kBlock), xs_bytes + d, s,
                       static_cast<const T*>(L->Wp), L->bp, L->Q, L->tlo, L->thi, static_cast<const T*>(xv), L->yacc,
                       L->mask, L->counts, L->list, d, h, gemv_blocks);
    hipLaunchKernelGGL(fix_kernel<T>, dim3(fix_blocks, (unsigned)n), dim3(kBlock), xs_bytes, s,
                       static_cast<const T*>(L->W1), static_cast<const T*>(L->b1), static_cast<const T*>(L->W2T), L->a, L->c,
                       static_cast<const T*>(xv), L->counts, L->list, L->yacc, d, h, (int)L->act);
    hipLaunchKernelGGL(finish_kernel<T>, dim3((unsigned)n), dim3(kBlock), 0, s, L->yacc, static_cast<T*>(yv), L->counts, d,
                       norm_out, kRmsEps);
    TD_HIP(hipGetLastError());
    L->last_n = n;
    return TARDIS_OK;
}

template <typename T>
tardis_status_t dense_t(tardis_layer_s* L, const void* xv, int64_t n, void* yv, hipStream_t s) {
    const int d = (int)L->d, h = (int)L->h;
    const size_t lds_cap = 60 * 1024;
    const size_t x_bytes = (size_t)d * sizeof(T), hid_bytes = (size_t)h * sizeof(T);
    const T* x = static_cast<const T*>(xv);
    T* hid = reinterpret_cast<T*>(L->hidden);
    const int l1 = x_bytes <= lds_cap, l2 = hid_bytes <= lds_cap;
    hipLaunchKernelGGL((dense_rows_kernel<T, true>), dim3(div_up(h, kWaves * kGemvRowsPerWave), (unsigned)n), dim3(kBlock),
                       l1 ? x_bytes : 0, s, static_cast<const T*>(L->W1), static_cast<const T*>(L->b1), x, hid, h, d,
                       (int)L->act, l1);
    hipLaunchKernelGGL((dense_rows_kernel<T, false>), dim3(div_up(d, kWaves * kGemvRowsPerWave), (unsigned)n), dim3(kBlock),
                       l2 ? hid_bytes : 0, s, static_cast<const T*>(L->W2), static_cast<const T*>(L->b2), hid,
                       static_cast<T*>(yv), d, h, 0, l2);
    TD_HIP(hipGetLastError());
    return TARDIS_OK;
}

}  // namespace

tardis_status_t td_forward(tardis_layer_s* L, const void* x, int64_t n, void* y, int norm_out, hipStream_t s) {
    return L->dtype == TARDIS_BF16 ? forward_t<bf16_t>(L, x, n, y, norm_out, s)
                                   : forward_t<float>(L, x, n, y, norm_out, s);
}

tardis_status_t td_dense_forward(tardis_layer_s* L, const void* x, int64_t n, void* y, hipStream_t s) {
    if (L->pf_scratch && n >= 2) return td_dense_prefill(L, x, n, y, s);
    return L->dtype == TARDIS_BF16 ? dense_t<bf16_t>(L, x, n, y, s) : dense_t<float>(L, x, n, y, s);
}

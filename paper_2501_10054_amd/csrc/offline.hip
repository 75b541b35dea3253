// Offline steps: range selection and line fit (calibrate), constant folding,
// predictor construction, and the layout copies the online path needs.
#include <type_traits>

#include "common.h"
#include "codes.h"
#include "sigma.h"

namespace {

constexpr int kBlock = 256;

// ------------------------------------------------------------------ transpose
// dst[c][r] = src[r][c], element size 2 or 4 bytes.
template <typename E>
__global__ void __launch_bounds__(256)
transpose_kernel(const E* __restrict__ src, E* __restrict__ dst, int64_t rows, int64_t cols) {
    __shared__ E tile[32][33];
    const int tx = threadIdx.x % 32, ty = threadIdx.x / 32;  // 32 x 8
    const int64_t c0 = (int64_t)blockIdx.x * 32, r0 = (int64_t)blockIdx.y * 32;
#pragma unroll
    for (int i = 0; i < 32; i += 8) {
        const int64_t r = r0 + ty + i, c = c0 + tx;
        if (r < rows && c < cols) tile[ty + i][tx] = src[r * cols + c];
    }
    __syncthreads();
#pragma unroll
    for (int i = 0; i < 32; i += 8) {
        const int64_t c = c0 + ty + i, r = r0 + tx;
        if (r < rows && c < cols) dst[c * rows + r] = tile[tx][ty + i];
    }
}

// The same for 2-byte elements with rows and cols multiples of 8 and 16-byte aligned arrays: 64 x 64 tiles, 16 bytes
// a thread on both sides (the 32 x 32 form moves 64 bytes of a row at a time).  Two source rows share a word
// of the LDS tile; a thread collects eight of them for one destination row.
// dst_lo: a straight copy of src (46 us for the transpose alone, 67 with the copy, which would otherwise read src again).
// SPLIT: the fold's operands instead of copies: p = a[row] * src, its bf16 head to dst and the bf16 remainder to
// dst_lo, so that the folded matrix is accumulated from ~16 significant bits instead of 8 (the paper's
// Sec. "Precision Effects on Reordering FFN" finds bf16 intermediates visibly worse than fp32).
// Bound: HBM.  16384 x 4096: copy 127 -> 46 us, split 217 -> 76 us (32 x 32 tiles before).
template <bool SPLIT>
__global__ void __launch_bounds__(256)
transpose16_kernel(const bf16_t* __restrict__ src, bf16_t* __restrict__ dst, bf16_t* __restrict__ dst_lo,
                   const float* __restrict__ a, int64_t rows, int64_t cols) {
    constexpr int PITCH = 65;                                    // words: column c of source rows 2r, 2r+1 at [r][c]
    __shared__ uint32_t hi[32 * PITCH], lo[SPLIT ? 32 * PITCH : 1];
    const int64_t c0 = (int64_t)blockIdx.x * 64, r0 = (int64_t)blockIdx.y * 64;
    {
        const int pr = threadIdx.x >> 3, pc = (threadIdx.x & 7) * 8;   // row pair, first of 8 columns
        const int64_t r = r0 + 2 * pr, c = c0 + pc;
        td_u32x4 v[2] = {{0, 0, 0, 0}, {0, 0, 0, 0}};
        float s[2] = {0.0f, 0.0f};
#pragma unroll
        for (int u = 0; u < 2; ++u)
            if (r + u < rows && c < cols) {
                v[u] = *reinterpret_cast<const td_u32x4*>(src + (r + u) * cols + c);
                if constexpr (SPLIT) s[u] = a[r + u];
                else *reinterpret_cast<td_u32x4*>(dst_lo + (r + u) * cols + c) = v[u];
            }
#pragma unroll
        for (int k = 0; k < 8; ++k) {
            uint32_t e[2], rest[2] = {0u, 0u};
#pragma unroll
            for (int u = 0; u < 2; ++u) {
                e[u] = (v[u][k >> 1] >> (16 * (k & 1))) & 0xffffu;
                if constexpr (SPLIT) {
                    const float p = s[u] * td_bf16_to_f32((bf16_t)e[u]);
                    const bf16_t head = td_f32_to_bf16(p);
                    e[u] = head;
                    rest[u] = td_f32_to_bf16(p - td_bf16_to_f32(head));
                }
            }
            hi[pr * PITCH + pc + k] = e[0] | (e[1] << 16);
            if constexpr (SPLIT) lo[pr * PITCH + pc + k] = rest[0] | (rest[1] << 16);
        }
    }
    __syncthreads();
    // thread -> destination row (source column) and 8 source rows
#pragma unroll
    for (int u = 0; u < 2; ++u) {
        const int cc = u * 32 + (threadIdx.x >> 3), rr = (threadIdx.x & 7) * 4;   // column; first of 4 row pairs
        const int64_t c = c0 + cc, r = r0 + 2 * rr;
        if (c >= cols || r >= rows) continue;                    // rows % 8 == 0: all eight or none
        td_u32x4 o;
#pragma unroll
        for (int k = 0; k < 4; ++k) o[k] = hi[(rr + k) * PITCH + cc];
        *reinterpret_cast<td_u32x4*>(dst + c * rows + r) = o;
        if constexpr (SPLIT) {
#pragma unroll
            for (int k = 0; k < 4; ++k) o[k] = lo[(rr + k) * PITCH + cc];
            *reinterpret_cast<td_u32x4*>(dst_lo + c * rows + r) = o;
        }
    }
}

// ------------------------------------------------------- scaled transpose (fold)
// P = diag(a) W1 (h x d) written transposed (d x h) as head and remainder (see above), any sizes.
__global__ void __launch_bounds__(256)
scale_transpose_bf16_kernel(const bf16_t* __restrict__ W1, const float* __restrict__ a, bf16_t* __restrict__ Phi,
                            bf16_t* __restrict__ Plo, int64_t h, int64_t d) {
    __shared__ float tile[32][33];
    const int tx = threadIdx.x % 32, ty = threadIdx.x / 32;
    const int64_t k0 = (int64_t)blockIdx.x * 32, j0 = (int64_t)blockIdx.y * 32;
#pragma unroll
    for (int i = 0; i < 32; i += 8) {
        const int64_t j = j0 + ty + i, k = k0 + tx;
        if (j < h && k < d) tile[ty + i][tx] = a[j] * td_bf16_to_f32(W1[j * d + k]);
    }
    __syncthreads();
#pragma unroll
    for (int i = 0; i < 32; i += 8) {
        const int64_t k = k0 + ty + i, j = j0 + tx;
        if (j < h && k < d) {
            const float p = tile[tx][ty + i];
            const bf16_t hi = td_f32_to_bf16(p);
            Phi[k * h + j] = hi;
            Plo[k * h + j] = td_f32_to_bf16(p - td_bf16_to_f32(hi));
        }
    }
}

__global__ void __launch_bounds__(256)
scale_transpose_f32_kernel(const float* __restrict__ W1, const float* __restrict__ a, float* __restrict__ P,
                           int64_t h, int64_t d) {
    __shared__ float tile[32][33];
    const int tx = threadIdx.x % 32, ty = threadIdx.x / 32;
    const int64_t k0 = (int64_t)blockIdx.x * 32, j0 = (int64_t)blockIdx.y * 32;
#pragma unroll
    for (int i = 0; i < 32; i += 8) {
        const int64_t j = j0 + ty + i, k = k0 + tx;
        if (j < h && k < d) tile[ty + i][tx] = a[j] * W1[j * d + k];
    }
    __syncthreads();
#pragma unroll
    for (int i = 0; i < 32; i += 8) {
        const int64_t k = k0 + ty + i, j = j0 + tx;
        if (j < h && k < d) P[k * h + j] = tile[tx][ty + i];
    }
}

__global__ void __launch_bounds__(256)
f32_to_bf16_kernel(const float* __restrict__ src, bf16_t* __restrict__ dst, int64_t n) {
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (i < n) dst[i] = td_f32_to_bf16(src[i]);
}

// k_j = c_j + a_j b1_j, the vector that the folded bias multiplies W2 with
template <typename T>
__global__ void __launch_bounds__(kBlock)
fold_bias_terms_kernel(const T* __restrict__ b1, const float* __restrict__ a, const float* __restrict__ c,
                       double* __restrict__ k, int64_t h) {
    const int64_t j = (int64_t)blockIdx.x * kBlock + threadIdx.x;
    if (j < h) k[j] = (double)c[j] + (b1 ? (double)a[j] * (double)td_load<T>(b1 + j) : 0.0);
}

// b'[r] = sum_j W2[r][j] * k_j + b2[r]; one block per kBiasRows output rows, fp64 accumulation.  Bound: HBM (W2 once, 16
// bytes a load where rows are whole vectors).  Several rows, because k (8 bytes where W2 has 2) comes from L2 for
// every block: d=4096, h=16384: 26 us with four rows, 42 with one.
constexpr int kBiasRows = 4;
template <typename T>
__global__ void __launch_bounds__(kBlock)
fold_bias_kernel(const T* __restrict__ W2, const double* __restrict__ k, const T* __restrict__ b2, float* __restrict__ bp,
                 int64_t d, int64_t h) {
    __shared__ double red[kBiasRows][kBlock / TD_WAVE];
    constexpr int V = 16 / (int)sizeof(T);
    const int64_t r0 = (int64_t)blockIdx.x * kBiasRows;
    const T* row[kBiasRows];                         // (past the last row: the last one once more, not stored)
    double acc[kBiasRows];
#pragma unroll
    for (int i = 0; i < kBiasRows; ++i) {
        row[i] = W2 + (r0 + i < d ? r0 + i : d - 1) * h;
        acc[i] = 0.0;
    }
    if (h % V == 0) {
        for (int64_t v = threadIdx.x; v < h / V; v += kBlock) {
            td_u32x4 w[kBiasRows];
#pragma unroll
            for (int i = 0; i < kBiasRows; ++i) w[i] = td_load_stream16(reinterpret_cast<const td_u32x4*>(row[i]) + v);
            double kv[V];
#pragma unroll
            for (int u = 0; u < V; ++u) kv[u] = k[v * V + u];
#pragma unroll
            for (int i = 0; i < kBiasRows; ++i) {
                const T* wt = reinterpret_cast<const T*>(&w[i]);
#pragma unroll
                for (int u = 0; u < V; ++u) acc[i] += (double)td_load<T>(wt + u) * kv[u];
            }
        }
    } else {
        for (int64_t j = threadIdx.x; j < h; j += kBlock)
#pragma unroll
            for (int i = 0; i < kBiasRows; ++i) acc[i] += (double)td_load<T>(row[i] + j) * k[j];
    }
#pragma unroll
    for (int i = 0; i < kBiasRows; ++i) {
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) acc[i] += __shfl_xor(acc[i], o, 64);
        if ((threadIdx.x & 63) == 0) red[i][threadIdx.x / 64] = acc[i];
    }
    __syncthreads();
    const int64_t r = r0 + threadIdx.x;
    if (threadIdx.x < kBiasRows && r < d) {
        double t = 0.0;
        for (int w = 0; w < kBlock / TD_WAVE; ++w) t += red[threadIdx.x][w];
        if (b2) t += (double)td_load<T>(b2 + r);
        bp[r] = (float)t;
    }
}

// ---------------------------------------------------------------- predictor
// One block per neuron row: s = max|w| / 127 (fp64), q = rint(w / s) clamped,
// bounds in code units.  All arithmetic is IEEE fp64 so the codes are a pure
// function of the inputs.
// The range the predictor tests against: the neuron's range with the fraction `margin` of its
// width taken off at either end (margin = 0: the range itself).  A narrower test flags more
// neurons - flagged neurons are repaired exactly, so this trades time for recall of a coarse sketch.
__device__ __forceinline__ void predictor_range(double lo, double hi, double margin, double& rl, double& rh) {
    rl = lo;
    rh = hi;
    const double w = hi - lo;
    if (margin > 0.0 && w > 0.0 && w < INFINITY) {
        rl = lo + margin * w;
        rh = hi - margin * w;
    }
}

// rint(w / s) clamped to [-127, 127], the quotient as IEEE division gives it.  w * (1/s) is within 3 units in the
// last place of it, i.e. (|quotient| <= 127) within 1e-13; only where that could reach another integer - the
// quotient is that close to a half - the division itself is done.
__device__ __forceinline__ int sketch_code(float w, double s, double inv) {
    double q = (double)w * inv;
    const double n = rint(q);
    if (fabs(fabs(q - n) - 0.5) < 1e-9) q = (double)w / s;
    return (int)fmin(fmax(rint(q), -127.0), 127.0);
}

// The codes of N weights in fp32: w * inv32 (inv32: 1 / s, rounded) is within 2^-23 of the quotient, with |quotient| <= 127
// 1.6e-5, so where none of them is that close to a half, rint gives the integers that the exact quotients give; else false.
// For maxima of at least kFlatMin and at most kFlatMax: inv32 is a normal number, and a NaN's code is -top here and there.
constexpr float kFlatMin = 1e-30f, kFlatMax = 1e30f, kNearHalf = 0.5f - 4e-5f;
template <int N> __device__ __forceinline__ bool flat_codes(const float (&w)[N], float inv32, float top, int (&code)[N]) {
    float far = 0.0f;
#pragma unroll
    for (int u = 0; u < N; ++u) {
        const float q = w[u] * inv32, n = rintf(q);
        far = fmaxf(far, fabsf(q - n));
        code[u] = (int)fminf(fmaxf(n, -top), top);
    }
    return far < kNearHalf;
}

// Bound: HBM (W1 once, a byte per weight out) and vector instructions together.  16384 x 4096: with the quotient of
// every weight in fp64 75 us (a few large columns) and 80 (normal weights), now 49 and 68; a 64-bit division per weight and 2-byte
// loads: 140.  (A wavefront per row, all its loads under way at once and no barrier: 67 for normal weights.)
template <typename T>
__global__ void __launch_bounds__(kBlock)
sketch_kernel(const T* __restrict__ W1, const T* __restrict__ b1, const float* __restrict__ lo,
              const float* __restrict__ hi, int64_t d, int8_t* __restrict__ Q, float* __restrict__ tlo,
              float* __restrict__ thi, float margin, float* __restrict__ code_scale, int32_t* __restrict__ no_scale) {
    __shared__ float red[kBlock / TD_WAVE];
    constexpr int V = 16 / (int)sizeof(T);
    constexpr int kKeep = 2;                         // vectors a thread keeps between the two passes
    const int64_t j = blockIdx.x;
    const T* row = W1 + j * d;
    const bool vec = d % V == 0;                     // (W1 is 16-byte aligned: so is every row)
    const int64_t nv = vec ? d / V : 0;
    td_u32x4 keep[kKeep];
    float m = 0.0f;
    bool nan = false;                                // (a NaN's stored code is -127, which no scale gives)
    auto vmax = [&](const td_u32x4& w) {
        const T* wt = reinterpret_cast<const T*>(&w);
#pragma unroll
        for (int u = 0; u < V; ++u) {
            const float f = td_load<T>(wt + u);
            m = fmaxf(m, fabsf(f));
            nan |= f != f;
        }
    };
#pragma unroll
    for (int i = 0; i < kKeep; ++i) {
        const int64_t v = i * kBlock + threadIdx.x;
        if (v < nv) {
            keep[i] = reinterpret_cast<const td_u32x4*>(row)[v];
            vmax(keep[i]);
        }
    }
    for (int64_t v = kKeep * kBlock + threadIdx.x; v < nv; v += kBlock) vmax(reinterpret_cast<const td_u32x4*>(row)[v]);
    for (int64_t k = nv * V + threadIdx.x; k < d; k += kBlock) {
        const float f = td_load<T>(row + k);
        m = fmaxf(m, fabsf(f));
        nan |= f != f;
    }
    if (no_scale && nan) *no_scale = 1;
    m = td_wave_max(m);
    if ((threadIdx.x & 63) == 0) red[threadIdx.x / 64] = m;
    __syncthreads();
    m = red[0];
#pragma unroll
    for (int w = 1; w < kBlock / TD_WAVE; ++w) m = fmaxf(m, red[w]);
    const double s = (double)m / 127.0;
    const double bj = b1 ? (double)td_load<T>(b1 + j) : 0.0;
    double rl, rh;
    predictor_range((double)lo[j], (double)hi[j], (double)margin, rl, rh);
    const bool live = m > 0.0f;
    const double inv = live ? 1.0 / s : 0.0;
    const bool flat = m >= kFlatMin && m <= kFlatMax;
    const float inv32 = (float)inv;
    auto code = [&](float w) { return live ? sketch_code(w, s, inv) : 0; };
    auto put = [&](int64_t v, const td_u32x4& w) {
        const T* wt = reinterpret_cast<const T*>(&w);
        uint32_t o[2] = {0u, 0u};
        float f[V];
        int q[V];
#pragma unroll
        for (int u = 0; u < V; ++u) f[u] = td_load<T>(wt + u);
        if (!(flat && flat_codes(f, inv32, 127.0f, q))) {
#pragma unroll
            for (int u = 0; u < V; ++u) q[u] = code(f[u]);
        }
#pragma unroll
        for (int u = 0; u < V; ++u) o[u >> 2] |= (uint32_t)(uint8_t)(int8_t)q[u] << (8 * (u & 3));
        int8_t* dst = Q + j * d + v * V;             // V-byte aligned: d % V == 0
        if constexpr (V == 8) *reinterpret_cast<uint2*>(dst) = make_uint2(o[0], o[1]);
        else *reinterpret_cast<uint32_t*>(dst) = o[0];
    };
#pragma unroll
    for (int i = 0; i < kKeep; ++i) {
        const int64_t v = i * kBlock + threadIdx.x;
        if (v < nv) put(v, keep[i]);
    }
    for (int64_t v = kKeep * kBlock + threadIdx.x; v < nv; v += kBlock) put(v, reinterpret_cast<const td_u32x4*>(row)[v]);
    for (int64_t k = nv * V + threadIdx.x; k < d; k += kBlock) Q[j * d + k] = (int8_t)code(td_load<T>(row + k));
    if (threadIdx.x == 0) {
        if (live) {
            tlo[j] = (float)((rl - bj) / s);
            thi[j] = (float)((rh - bj) / s);
        } else {
            const bool inside = (rl <= bj) && (bj < rh);
            tlo[j] = inside ? -INFINITY : INFINITY;
            thi[j] = INFINITY;
        }
        if (code_scale) {
            code_scale[j] = flat ? td_code_scale(m, code(0.5f * m)) : 0.0f;
            if (live && !flat) *no_scale = 1;
        }
    }
}

// the predictor's bounds of a neuron with a low-bit sketch, in units of s
__device__ __forceinline__ void low_bit_bounds(float lo, float hi, float margin, double b, bool live, double s, float* tlo, float* thi) {
    double rl, rh;
    predictor_range((double)lo, (double)hi, (double)margin, rl, rh);
    if (live) {
        *tlo = (float)((rl - b) / s);
        *thi = (float)((rh - b) / s);
    } else {
        const bool inside = (rl <= b) && (b < rh);
        *tlo = inside ? -INFINITY : INFINITY;
        *thi = INFINITY;
    }
}

// Grouped low-bit sketch (groups of 32 consecutive columns), codes of 4, 3 or 2 bits with the
// largest code qmax = 7, 3 or 1: group maxima g, row maximum r,
// s = r / (qmax*15), multiplier m = ceil(g / (qmax s)) in [1, 15], code q = rint(w / (m s)) in [-qmax, qmax];
// all in fp64, each step one IEEE operation, so every output is a function of the inputs.
// Outputs: M4 (one byte per group); Q (optional) the effective one-byte code m*q; Q4 (optional,
// d % 32 == 0) the packed form read by the decode kernel: group G is the 16-byte vector G of the
// row, byte b of its dword w holds column 4w+b in the low nibble and column 16+4w+b in the high one.
// (This kernel: rows that are not whole groups, for which there is no packed form.)
template <typename T>
__global__ void __launch_bounds__(kBlock)
sketch4_kernel(const T* __restrict__ W1, const T* __restrict__ b1, const float* __restrict__ lo,
               const float* __restrict__ hi, int64_t d, int ng, int8_t* __restrict__ Q, uint8_t* __restrict__ M4,
               float* __restrict__ tlo, float* __restrict__ thi, int qmax, float margin) {
    extern __shared__ int gval[];                    // group maxima (bit patterns), then multipliers
    __shared__ float red[kBlock / TD_WAVE];
    const int64_t j = blockIdx.x;
    const T* row = W1 + j * d;
    for (int g = threadIdx.x; g < ng; g += kBlock) gval[g] = 0;
    __syncthreads();
    for (int64_t k = threadIdx.x; k < d; k += kBlock)   // non-negative floats order like their bit patterns
        atomicMax(&gval[k >> 5], __float_as_int(fabsf(td_load<T>(row + k))));
    __syncthreads();
    float r = 0.0f;
    for (int g = threadIdx.x; g < ng; g += kBlock) r = fmaxf(r, __int_as_float(gval[g]));
    r = td_wave_max(r);
    if ((threadIdx.x & 63) == 0) red[threadIdx.x / 64] = r;
    __syncthreads();
    r = red[0];
#pragma unroll
    for (int w = 1; w < kBlock / TD_WAVE; ++w) r = fmaxf(r, red[w]);
    const double s = (double)r / (double)(qmax * 15);   // (4 bits: 7 * 15)
    const double bj = b1 ? (double)td_load<T>(b1 + j) : 0.0;
    const bool live = r > 0.0f;
    for (int g = threadIdx.x; g < ng; g += kBlock) {
        int m = 1;
        if (live) {
            const double t = ceil((double)__int_as_float(gval[g]) / ((double)qmax * s));
            m = (int)fmin(fmax(t, 1.0), 15.0);
        }
        gval[g] = m;
        M4[j * ng + g] = (uint8_t)m;
    }
    __syncthreads();
    auto code = [&](int64_t k) -> int {              // 4-bit code of column k
        if (!live) return 0;
        const double q = rint((double)td_load<T>(row + k) / ((double)gval[k >> 5] * s));
        return (int)fmin(fmax(q, -(double)qmax), (double)qmax);
    };
    if (Q)
        for (int64_t k = threadIdx.x; k < d; k += kBlock) Q[j * d + k] = (int8_t)(gval[k >> 5] * code(k));
    if (threadIdx.x == 0) low_bit_bounds(lo[j], hi[j], margin, bj, live, s, tlo + j, thi + j);
}

// The same for rows of whole groups.  Four lanes hold a group, each the eight columns of its word of the packed form, so a
// group's maximum and multiplier stay in registers, and the codes are taken in fp32 where that decides them (flat_codes; the
// unit of a group, m s, has a reciprocal within 2^-22, so quotients up to 105 - a group with a NaN has m = 1 - are within 3.4e-5).
// Bound: HBM (W1 once, half a byte and where kept a byte per weight out).  16384 x 4096: 61 us; 250 with maxima by
// LDS atomics, 2-byte loads and an fp64 division per weight; 66 with a wavefront per row.
template <typename T>
__global__ void __launch_bounds__(kBlock)
sketch4_rows_kernel(const T* __restrict__ W1, const T* __restrict__ b1, const float* __restrict__ lo,
                    const float* __restrict__ hi, int64_t d, int8_t* __restrict__ Q, uint8_t* __restrict__ Q4,
                    uint8_t* __restrict__ M4, float* __restrict__ tlo, float* __restrict__ thi, int qmax, float margin) {
    __shared__ float red[kBlock / TD_WAVE];
    constexpr int kKeep = 2;                         // words a thread keeps between the two passes
    typedef T quad_t __attribute__((ext_vector_type(4)));
    const int64_t j = blockIdx.x;
    const T* row = W1 + j * d;                       // (W1 is 16-byte aligned: so is every group)
    const int64_t words = d / 8;                     // a multiple of four: a group's lanes are all there or none
    auto fetch = [&](int64_t idx, float (&f)[8]) {
        const T* at = row + 32 * (idx >> 2) + 4 * (idx & 3);
        const quad_t a = *reinterpret_cast<const quad_t*>(at), b = *reinterpret_cast<const quad_t*>(at + 16);
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const T x = a[u], y = b[u];
            f[u] = td_load<T>(&x);
            f[4 + u] = td_load<T>(&y);
        }
    };
    auto group_max = [&](const float (&f)[8]) {      // non-negative floats order like their bit patterns, NaNs above all
        int g = 0;
#pragma unroll
        for (int u = 0; u < 8; ++u) g = max(g, __float_as_int(fabsf(f[u])));
        g = max(g, __shfl_xor(g, 1, 64));
        return __int_as_float(max(g, __shfl_xor(g, 2, 64)));
    };
    float keep[kKeep][8], top[kKeep];
    float r = 0.0f;
#pragma unroll
    for (int i = 0; i < kKeep; ++i) {
        const int64_t idx = i * kBlock + threadIdx.x;
        if (idx < words) {
            fetch(idx, keep[i]);
            top[i] = group_max(keep[i]);
            r = fmaxf(r, top[i]);
        }
    }
    for (int64_t idx = kKeep * kBlock + threadIdx.x; idx < words; idx += kBlock) {
        float f[8];
        fetch(idx, f);
        r = fmaxf(r, group_max(f));
    }
    r = td_wave_max(r);
    if ((threadIdx.x & 63) == 0) red[threadIdx.x / 64] = r;
    __syncthreads();
    r = red[0];
#pragma unroll
    for (int w = 1; w < kBlock / TD_WAVE; ++w) r = fmaxf(r, red[w]);
    const double s = (double)r / (double)(qmax * 15);
    const bool live = r > 0.0f, flat = r >= kFlatMin && r <= kFlatMax;
    const float inv32 = flat ? (float)(1.0 / s) : 0.0f;
    auto put = [&](int64_t idx, const float (&f)[8], float g) {
        int m = 1, q[8];
        if (live) m = (int)fmin(fmax(ceil((double)g / ((double)qmax * s)), 1.0), 15.0);
        if (!(flat && flat_codes(f, inv32 * __builtin_amdgcn_rcpf((float)m), (float)qmax, q))) {
            const double unit = (double)m * s;
#pragma unroll
            for (int u = 0; u < 8; ++u)
                q[u] = live ? (int)fmin(fmax(rint((double)f[u] / unit), -(double)qmax), (double)qmax) : 0;
        }
        if ((idx & 3) == 0) M4[j * (d / 32) + (idx >> 2)] = (uint8_t)m;
        if (Q4) {
            uint32_t word = 0;
#pragma unroll
            for (int b = 0; b < 4; ++b) word |= (uint32_t)((q[b] & 0xF) | ((q[4 + b] & 0xF) << 4)) << (8 * b);
            reinterpret_cast<uint32_t*>(Q4 + j * (d / 2))[idx] = word;
        }
        if (Q) {
            uint32_t o[2] = {0u, 0u};
#pragma unroll
            for (int u = 0; u < 8; ++u) o[u >> 2] |= (uint32_t)(uint8_t)(int8_t)(m * q[u]) << (8 * (u & 3));
            uint32_t* dst = reinterpret_cast<uint32_t*>(Q + j * d + 32 * (idx >> 2) + 4 * (idx & 3));
            dst[0] = o[0];
            dst[4] = o[1];
        }
    };
#pragma unroll
    for (int i = 0; i < kKeep; ++i) {
        const int64_t idx = i * kBlock + threadIdx.x;
        if (idx < words) put(idx, keep[i], top[i]);
    }
    for (int64_t idx = kKeep * kBlock + threadIdx.x; idx < words; idx += kBlock) {
        float f[8];
        fetch(idx, f);
        put(idx, f, group_max(f));
    }
    if (threadIdx.x == 0) {
        const double bj = b1 ? (double)td_load<T>(b1 + j) : 0.0;
        low_bit_bounds(lo[j], hi[j], margin, bj, live, s, tlo + j, thi + j);
    }
}

__global__ void __launch_bounds__(kBlock)
unpack_sketch4_kernel(const uint8_t* __restrict__ Q4, const uint8_t* __restrict__ M4, int64_t d,
                      int8_t* __restrict__ Q) {
    const int64_t j = blockIdx.x;
    const uint32_t* in = reinterpret_cast<const uint32_t*>(Q4 + j * (d / 2));
    for (int64_t idx = threadIdx.x; idx < d / 8; idx += kBlock) {
        const int64_t g = idx >> 2, w = idx & 3;
        const int m = M4[j * (d / 32) + g];
        const uint32_t word = in[idx];
#pragma unroll
        for (int b = 0; b < 4; ++b) {
            const int byte = (int)((word >> (8 * b)) & 0xFFu);
            const int qlo = ((byte & 0xF) ^ 8) - 8, qhi = ((byte >> 4) ^ 8) - 8;   // sign-extend 4 bits
            Q[j * d + 32 * g + 4 * w + b] = (int8_t)(m * qlo);
            Q[j * d + 32 * g + 16 + 4 * w + b] = (int8_t)(m * qhi);
        }
    }
}

// -------------------------------------------------------------- calibration
// One block per neuron.  zt: that neuron's n calibration pre-activations.
// Sort in LDS (bitonic, padded with +inf), read the two quantiles by linear
// interpolation at q*(n-1), then fit sigma(z) ~ a z + c over lo <= z < hi.
__device__ __forceinline__ double block_sum(double v, double* red) {
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
    __syncthreads();
    if ((threadIdx.x & 63) == 0) red[threadIdx.x / 64] = v;
    __syncthreads();
    double t = 0.0;
#pragma unroll
    for (int w = 0; w < kBlock / TD_WAVE; ++w) t += red[w];
    return t;
}

// sorts vals[0..npad) ascending (npad a power of two, padded with +inf), by a block of T threads
template <int T>
__device__ __forceinline__ void sort_lds(float* vals, int npad) {
    for (int k = 2; k <= npad; k <<= 1) {
        for (int s = k >> 1; s > 0; s >>= 1) {
            for (int t = threadIdx.x; t < npad / 2; t += T) {
                const int i = 2 * t - (t & (s - 1));  // index with bit `s` clear
                const int p = i + s;
                const bool up = (i & k) == 0;
                const float x0 = vals[i], x1 = vals[p];
                if ((x0 > x1) == up) {
                    vals[i] = x1;
                    vals[p] = x0;
                }
            }
            __syncthreads();
        }
    }
}

// least-squares line of sigma(z) on z over the samples with lo32 <= z < hi32, and the four outputs
__device__ __forceinline__ void fit_and_store(const float* vals, int n, float lo32, float hi32, int act, double* red,
                                              int64_t j, float* lo, float* hi, float* a, float* c) {
    double cnt = 0.0, sz = 0.0, sg = 0.0;
    for (int i = threadIdx.x; i < n; i += kBlock) {
        const float v = vals[i];
        if (v >= lo32 && v < hi32) {
            cnt += 1.0;
            sz += (double)v;
            sg += td_act_f64((double)v, act);
        }
    }
    cnt = block_sum(cnt, red);
    sz = block_sum(sz, red);
    sg = block_sum(sg, red);
    float aj, cj;
    if (cnt < 0.5) {
        aj = 0.0f;
        cj = (float)td_act_f64((double)lo32, act);
    } else {
        const double zbar = sz / cnt, gbar = sg / cnt;
        double var = 0.0, cov = 0.0;
        for (int i = threadIdx.x; i < n; i += kBlock) {
            const float v = vals[i];
            if (v >= lo32 && v < hi32) {
                const double dz = (double)v - zbar;
                var += dz * dz;
                cov += dz * (td_act_f64((double)v, act) - gbar);
            }
        }
        var = block_sum(var, red);
        cov = block_sum(cov, red);
        if (cnt < 1.5 || !(var > 0.0)) {
            aj = 0.0f;
            cj = (float)gbar;
        } else {
            const double slope = cov / var;
            aj = (float)slope;
            cj = (float)(gbar - slope * zbar);
        }
    }
    if (threadIdx.x == 0) {
        lo[j] = lo32;
        hi[j] = hi32;
        a[j] = aj;
        c[j] = cj;
    }
}

// Quantile ranges and line fit, one block of T threads per neuron, NPT samples in each thread's registers
// (n <= T * NPT).  Only four order statistics are needed, so nothing is sorted: a histogram of kSelBins
// equal cells between the smallest and the largest sample finds the cells that hold them, and the few
// samples of those cells are ranked by counting.  (A neuron whose samples crowd into one cell - an outlier
// stretches the histogram, or most samples are equal - or that are not all finite falls back to the sort in LDS.)  The fit takes
// sigma of every sample once, in fp64.
// What bounds it: vector instructions, about half of them for sigma (without it 59 of 107 us).  4096 neurons x 4096 samples:
// 112 us with the library's erf, whose two branches a wavefront both takes, and a fit in two passes; 95 us with the sigma of
// sigma.h and one pass; 81 with its constants in scalar registers, shared by two samples, and registers for five blocks a CU (one of them
// spills; left to the compiler 88, with six or more blocks 92 to 104).  (A full bitonic sort in LDS and sigma taken twice: 375.)
// Samples that all lie below 1, 4096 x 4096 with N(0, 0.23^2): 58 when only the compiler kept sigma's far form apart, 68 with both forms for
// every pair, 52 with the far one behind a branch; 8192 samples 65, 80, 64.  (Blocks of 512 threads are two a CU with 96 registers as
// with 128: with 96 two spill, 8192 samples, N(0, 1.6^2), 85 us either way.)
//
// A sample closer to the end of a range than fp32 can tell (both are fp32 here) would count as inside or
// outside by luck of rounding.  For those (a few of 16384 neurons) the pre-activations of the two samples
// the end lies between are recomputed in fp64, and end and membership follow from them.
constexpr int kSelBins = 1024;
constexpr int kSelList = 256;

template <typename E, int T, int NPT>
__global__ void __launch_bounds__(T, T == 256 ? 5 : 4)
calibrate_neuron_kernel(const float* __restrict__ Zt, const E* __restrict__ W1, const E* __restrict__ b1,
                        const E* __restrict__ X, int n, int npad, int64_t d, float coverage,
                        const float* __restrict__ cov_pn, int act, float* __restrict__ lo, float* __restrict__ hi,
                        float* __restrict__ a, float* __restrict__ c) {
    constexpr int NW = T / TD_WAVE;
    static_assert(NPT % 2 == 0 && T >= 256 && kSelBins % 256 == 0, "four cells a thread in the search for the ranks' cells");
    extern __shared__ float vals[];                  // npad floats, for the sort and the parked samples
    __shared__ int hist[kSelBins];
    __shared__ int wave_tot[4];
    __shared__ float list[2][kSelList];
    __shared__ int list_n[2], cell[4], cell_before[4], found[2];
    __shared__ float stat[4];
    __shared__ float redf[2][NW];
    __shared__ double red[NW][3];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int64_t j = blockIdx.x;
    const float* z = Zt + j * (int64_t)n;
    const double t = cov_pn ? (double)cov_pn[j] : (double)coverage;

    float v[NPT];
    float mn = INFINITY, mx = -INFINITY;
#pragma unroll
    for (int k = 0; k < NPT; ++k) {
        const int i = k * T + tid;
        v[k] = i < n ? z[i] : 0.0f;
        if (i < n) {
            mn = fminf(mn, v[k]);
            mx = fmaxf(mx, v[k]);
        }
    }
    bool nan = false;                                // a NaN has no cell: the histogram is left out as for an infinity
#pragma unroll
    for (int k = 0; k < NPT; k += 2) nan |= __builtin_isunordered(v[k], v[k + 1]);
    if (nan) mx = INFINITY;
    for (int i = tid; i < kSelBins; i += T) hist[i] = 0;
    if (tid < 2) list_n[tid] = 0;
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) {
        mn = fminf(mn, __shfl_xor(mn, o, 64));
        mx = fmaxf(mx, __shfl_xor(mx, o, 64));
    }
    if (lane == 0) {
        redf[0][wave] = mn;
        redf[1][wave] = mx;
    }
    __syncthreads();
#pragma unroll
    for (int w = 0; w < NW; ++w) {
        mn = fminf(mn, redf[0][w]);
        mx = fmaxf(mx, redf[1][w]);
    }

    // the four order statistics: ranks of the lower end, of the upper end, and one above each
    const double pos[2] = {(1.0 - t) / 2.0 * (double)(n - 1), (1.0 + t) / 2.0 * (double)(n - 1)};
    int rank[4];
    double frac[2];
#pragma unroll
    for (int q = 0; q < 2; ++q) {
        const int i = min(max((int)floor(pos[q]), 0), n - 1);
        rank[2 * q] = i;
        rank[2 * q + 1] = min(i + 1, n - 1);
        frac[q] = pos[q] - (double)i;
    }
    const float scale = (float)kSelBins / (mx - mn);
    bool by_cells = mx > mn && scale > 0.0f && scale < INFINITY;      // (uniform)
    auto cell_of = [&](float x) { return min((int)((x - mn) * scale), kSelBins - 1); };   // monotone in x
    if (by_cells) {
#pragma unroll
        for (int k = 0; k < NPT; ++k)
            if (k * T + tid < n) atomicAdd(&hist[cell_of(v[k])], 1);
        __syncthreads();
        int cnt[4], sum = 0;
        if (tid < 256) {
#pragma unroll
            for (int u = 0; u < 4; ++u) sum += cnt[u] = hist[tid * (kSelBins / 256) + u];
        }
        int incl = sum;
#pragma unroll
        for (int o = 1; o < 64; o <<= 1) {
            const int up = __shfl_up(incl, o, 64);
            if (lane >= o) incl += up;
        }
        if (tid < 256 && lane == 63) wave_tot[wave] = incl;
        __syncthreads();
        if (tid < 256) {
            int before = incl - sum;
            for (int w = 0; w < wave; ++w) before += wave_tot[w];
#pragma unroll
            for (int u = 0; u < 4; ++u) {
#pragma unroll
                for (int q = 0; q < 4; ++q)
                    if (rank[q] >= before && rank[q] < before + cnt[u]) {
                        cell[q] = tid * (kSelBins / 256) + u;
                        cell_before[q] = before;
                    }
                before += cnt[u];
            }
        }
        __syncthreads();
#pragma unroll
        for (int k = 0; k < NPT; ++k)
            if (k * T + tid < n) {
                const int ce = cell_of(v[k]);
#pragma unroll
                for (int q = 0; q < 2; ++q)
                    if (ce == cell[2 * q] || ce == cell[2 * q + 1]) {
                        const int at = atomicAdd(&list_n[q], 1);
                        if (at < kSelList) list[q][at] = v[k];
                    }
            }
        __syncthreads();
        by_cells = list_n[0] <= kSelList && list_n[1] <= kSelList;
    }
    if (by_cells) {
        // the cells between a rank's and the next rank's are empty, so a list is one run of the sorted samples
#pragma unroll
        for (int q = 0; q < 2; ++q) {
            const int len = list_n[q], first = cell_before[2 * q];
            for (int i = tid; i < len; i += T) {
                const float x = list[q][i];
                int less = 0;
                for (int k = 0; k < len; ++k) less += (list[q][k] < x || (list[q][k] == x && k < i)) ? 1 : 0;
                if (first + less == rank[2 * q]) stat[2 * q] = x;
                if (first + less == rank[2 * q + 1]) stat[2 * q + 1] = x;
            }
        }
        __syncthreads();
    } else {
        for (int i = tid; i < npad; i += T) vals[i] = INFINITY;
        __syncthreads();
#pragma unroll
        for (int k = 0; k < NPT; ++k)
            if (k * T + tid < n) vals[k * T + tid] = v[k];
        __syncthreads();
        sort_lds<T>(vals, npad);
        if (tid < 4) stat[tid] = vals[rank[tid]];
        __syncthreads();
    }

    auto total3 = [&](double (&s)[3]) {              // block-wide sums, in every thread
#pragma unroll
        for (int q = 0; q < 3; ++q)
#pragma unroll
            for (int o = 32; o > 0; o >>= 1) s[q] += __shfl_xor(s[q], o, 64);
        __syncthreads();
        if (lane == 0) {
#pragma unroll
            for (int q = 0; q < 3; ++q) red[wave][q] = s[q];
        }
        __syncthreads();
#pragma unroll
        for (int q = 0; q < 3; ++q) {
            double r = 0.0;
#pragma unroll
            for (int w = 0; w < NW; ++w) r += red[w][q];
            s[q] = r;
        }
    };

    // (ranges that hold next to nothing have no end of their own to decide: by value)
    const bool wide = rank[1] < rank[2] && stat[2] - stat[1] > 1e-6f * fmaxf(fabsf(stat[1]), fabsf(stat[2]));
    float end[2];
    float cut[2];                                    // the samples inside are those with cut[0] <= v < cut[1]
#pragma unroll
    for (int q = 0; q < 2; ++q) {
        const float v0 = stat[2 * q], v1 = stat[2 * q + 1];
        const bool two = rank[2 * q + 1] != rank[2 * q];
        const float e32 = (float)((double)v0 + frac[q] * ((double)v1 - (double)v0));
        end[q] = cut[q] = e32;
        const float eps = fabsf(e32) * 2.4e-7f;      // two units in the last place
        if (!wide || (!(e32 - v0 <= eps) && !(two && v1 - e32 <= eps))) continue;   // (uniform: shared and uniform values)
        int near = 0;                                // samples in [v0, v1], and the first of either end
        if (tid < 2) found[tid] = n;
        __syncthreads();
#pragma unroll
        for (int k = 0; k < NPT; ++k) {
            const int i = k * T + tid;
            if (i < n && v[k] >= v0 && v[k] <= v1) {
                ++near;
                if (v[k] == v0) atomicMin(&found[0], i);
            }
        }
        double s[3] = {(double)near, 0.0, 0.0};
        total3(s);
        const int i0 = found[0];
        if (two) {
#pragma unroll
            for (int k = 0; k < NPT; ++k) {
                const int i = k * T + tid;
                if (i < n && v[k] == v1 && i != i0) atomicMin(&found[1], i);
            }
        }
        __syncthreads();
        const int i1 = found[1];
        __syncthreads();
        if ((int)s[0] != (two ? 2 : 1) || i0 >= n || (two && i1 >= n)) continue;   // equal samples: by value
        double p[3] = {0.0, 0.0, 0.0};
        for (int64_t k = tid; k < d; k += T) {
            const double w = (double)td_load<E>(W1 + j * d + k);
            p[0] += w * (double)td_load<E>(X + i0 * d + k);
            if (two) p[1] += w * (double)td_load<E>(X + i1 * d + k);
        }
        total3(p);
        const double bj = b1 ? (double)td_load<E>(b1 + j) : 0.0;
        const double x0 = p[0] + bj, x1 = p[1] + bj;
        if (two && x0 == x1) continue;
        const double e0 = two ? fmin(x0, x1) : x0, e1 = two ? fmax(x0, x1) : x0;
        end[q] = (float)(e0 + frac[q] * (e1 - e0));
        // (of the two samples the end lies between; no other has their values.  Are they equal here and only one of them inside, the
        // other one is taken out by its index)
        const int below = (e0 < (double)end[q] ? 1 : 0) + (two && e1 < (double)end[q] ? 1 : 0);
        const bool split = two && below == 1, equal = split && v0 == v1;
        cut[q] = below == 0 || (equal && q == 0) ? v0 : split && !equal ? v1 : nextafterf(two ? v1 : v0, INFINITY);
        if (equal) {
#pragma unroll
            for (int k = 0; k < NPT; ++k)
                if (k * T + tid == i0) v[k] = NAN;
        }
    }
    const float lo32 = end[0], hi32 = end[1];

    // least-squares line of sigma(z) on z over the samples with lo32 <= z < hi32, in one pass: sums of dz = z - pivot, of
    // sigma and of their products.  The pivot is the first sample in the range (unless both next to the end are left out by its
    // rounding), so equal samples have dz = 0 exactly; what the subtractions of the sums lose in fp64 is far below what fp32 resolves of
    // z.  (A sample that is left out is in none of the sums: it may be far away.)
    const float pivot32 = stat[0] >= cut[0] ? stat[0] : stat[1];
    const double pivot = (double)pivot32;
    double s[3] = {0.0, 0.0, 0.0}, sq[3] = {0.0, 0.0, 0.0};          // count, sum dz, sum sigma; sum dz^2, sum dz sigma
    int inside = 0;
    auto sums = [&](auto act_constant) {
        constexpr int ACT = decltype(act_constant)::value;
        // (32 samples a thread beside the coefficients of this sigma are more than 128 registers: they go through LDS, each
        // thread's own.  4096 neurons x 16384, 32768 samples: 1070, 1580 us, so 925, 1380)
        constexpr bool kParked = NPT > 16 && ACT == TARDIS_ACT_GELU_ERF;
        constexpr int kPair = 2, kUnroll = kParked ? 1 : NPT / kPair;    // sigma of two samples at a time, side by side
        if constexpr (kParked) {
#pragma unroll
            for (int k = 0; k < NPT; ++k)
                if (k * T + tid < n) vals[k * T + tid] = v[k];
        }
#pragma unroll kUnroll
        for (int k0 = 0; k0 < NPT; k0 += kPair) {
            double g[kPair], dz[kPair];
#pragma unroll
            for (int u = 0; u < kPair; ++u) {
                const int k = k0 + u;
                const float x = !kParked ? v[k] : k * T + tid < n ? vals[k * T + tid] : 0.0f;
                const bool in = (k * T + tid < n) & (x >= cut[0]) & (x < cut[1]);
                g[u] = (double)(in ? x : 0.0f);                        // (sigma(0) = 0)
                dz[u] = (double)(in ? x : pivot32) - pivot;
                inside += in ? 1 : 0;
            }
            act_flat_f64<ACT>(g);
#pragma unroll
            for (int u = 0; u < kPair; ++u) {
                s[1] += dz[u];
                s[2] += g[u];
                sq[0] = fma(dz[u], dz[u], sq[0]);
                sq[1] = fma(dz[u], g[u], sq[1]);
            }
            // (the sums are taken here: put off, all of these are kept in registers)
            asm volatile("" : "+v"(s[1]), "+v"(s[2]), "+v"(sq[0]), "+v"(sq[1]));
            __builtin_amdgcn_sched_barrier(0);
        }
    };
    if (act == TARDIS_ACT_GELU_ERF) sums(std::integral_constant<int, TARDIS_ACT_GELU_ERF>{});
    else if (act == TARDIS_ACT_GELU_TANH) sums(std::integral_constant<int, TARDIS_ACT_GELU_TANH>{});
    else if (act == TARDIS_ACT_RELU) sums(std::integral_constant<int, TARDIS_ACT_RELU>{});
    else sums(std::integral_constant<int, TARDIS_ACT_IDENTITY>{});
    s[0] = (double)inside;
    total3(s);
    total3(sq);
    float aj, cj;
    if (s[0] < 0.5) {
        aj = 0.0f;
        cj = (float)td_act_f64((double)lo32, act);
    } else {
        const double dbar = s[1] / s[0], gbar = s[2] / s[0];
        const double var = sq[0] - s[1] * dbar, cov = sq[1] - s[1] * gbar;
        if (s[0] < 1.5 || !(var > 0.0)) {
            aj = 0.0f;
            cj = (float)gbar;
        } else {
            const double slope = cov / var;
            aj = (float)slope;
            cj = (float)(gbar - slope * (pivot + dbar));
        }
    }
    if (tid == 0) {
        lo[j] = lo32;
        hi[j] = hi32;
        a[j] = aj;
        c[j] = cj;
    }
}

// n <= 32768 samples per neuron
template <typename E>
tardis_status_t launch_calibrate(const tardis_ffn_desc* desc, const float* zt, const void* X, int n, float coverage,
                                 const float* cov_pn, float* lo, float* hi, float* a, float* c, hipStream_t s) {
    int npad = 2;
    while (npad < n) npad <<= 1;
    const size_t lds = (size_t)npad * sizeof(float);
    auto go = [&](auto kernel, int threads) -> tardis_status_t {
        if (lds > 48 * 1024)
            TD_HIP(hipFuncSetAttribute(reinterpret_cast<const void*>(kernel), hipFuncAttributeMaxDynamicSharedMemorySize,
                                       (int)lds));
        hipLaunchKernelGGL(kernel, dim3((unsigned)desc->h), dim3(threads), lds, s, zt, static_cast<const E*>(desc->W1),
                           static_cast<const E*>(desc->b1), static_cast<const E*>(X), n, npad, desc->d, coverage, cov_pn,
                           (int)desc->act, lo, hi, a, c);
        TD_HIP(hipGetLastError());
        return TARDIS_OK;
    };
    if (n <= 1024) return go(calibrate_neuron_kernel<E, 256, 4>, 256);
    if (n <= 4096) return go(calibrate_neuron_kernel<E, 256, 16>, 256);
    if (n <= 8192) return go(calibrate_neuron_kernel<E, 512, 16>, 512);
    return go(calibrate_neuron_kernel<E, 1024, 32>, 1024);
}

// ------------------------------------------------------------- range search
// Greedy range of Algorithm 1 (inner loop), one block per neuron: centroid = mode of a Gaussian
// kernel density estimate on a grid of 256 points (bandwidth 1.06 std n^-1/5), then the range
// grows by `step` to the left or to the right, whichever candidate's least-squares line leaves
// the smaller sum of |sigma(z) - (a z + c)| over its samples (right on equality), until it holds
// the portion t of the samples.  A side whose end lies beyond every sample is not offered again,
// so the loop ends after at most (max z - min z) / step + 2 steps; kSearchMaxSteps is a guard on
// the run time of one block, and a neuron that hits it makes the whole call fail.
constexpr int kKdeGrid = 256;
constexpr int kSearchMaxSteps = 4096;
static_assert(kKdeGrid == kBlock, "one grid point per thread");

// four block-wide sums at once
__device__ __forceinline__ void block_sum4(double (&v)[4], double (*red4)[4]) {
#pragma unroll
    for (int q = 0; q < 4; ++q)
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) v[q] += __shfl_xor(v[q], o, 64);
    __syncthreads();
    if ((threadIdx.x & 63) == 0) {
#pragma unroll
        for (int q = 0; q < 4; ++q) red4[threadIdx.x / 64][q] = v[q];
    }
    __syncthreads();
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        double t = 0.0;
#pragma unroll
        for (int w = 0; w < kBlock / TD_WAVE; ++w) t += red4[w][q];
        v[q] = t;
    }
}

// first index i in [0, n) with vals[i] >= x (n if none)
__device__ __forceinline__ int lower_bound_lds(const float* vals, int n, double x) {
    int lo = 0, hi = n;
    while (lo < hi) {
        const int mid = (lo + hi) >> 1;
        if ((double)vals[mid] >= x) hi = mid; else lo = mid + 1;
    }
    return lo;
}

__global__ void __launch_bounds__(kBlock)
range_search_kernel(const float* __restrict__ Zt, int n, int npad, float coverage, const float* __restrict__ cov_pn,
                    float step32, int act, float* __restrict__ lo, float* __restrict__ hi, float* __restrict__ a,
                    float* __restrict__ c, int* __restrict__ n_capped) {
    extern __shared__ double gv[];                   // sigma of the sorted samples, then the samples
    float* vals = reinterpret_cast<float*>(gv + ((n + 1) & ~1));
    __shared__ double red[kBlock / TD_WAVE];
    __shared__ double red4[kBlock / TD_WAVE][4];
    __shared__ double dens[kKdeGrid];
    const int64_t j = blockIdx.x;
    const float* z = Zt + j * (int64_t)n;
    for (int i = threadIdx.x; i < npad; i += kBlock) vals[i] = i < n ? z[i] : INFINITY;
    __syncthreads();
    sort_lds<kBlock>(vals, npad);
    for (int i = threadIdx.x; i < n; i += kBlock) gv[i] = td_act_f64((double)vals[i], act);
    const double zmin = (double)vals[0], zmax = (double)vals[n - 1];
    const double t = cov_pn ? (double)cov_pn[j] : (double)coverage;
    const double step = (double)step32;

    // ---- centroid
    double cen = zmin;
    if (n >= 2 && zmax > zmin) {
        double sz = 0.0;
        for (int i = threadIdx.x; i < n; i += kBlock) sz += (double)vals[i];
        const double mean = block_sum(sz, red) / (double)n;
        double sv = 0.0;
        for (int i = threadIdx.x; i < n; i += kBlock) {
            const double dz = (double)vals[i] - mean;
            sv += dz * dz;
        }
        const double sd = sqrt(block_sum(sv, red) / (double)(n - 1));
        const double bw = 1.06 * sd * pow((double)n, -0.2);
        const double delta = (zmax - zmin) / (double)(kKdeGrid - 1);
        const double u = zmin + (double)threadIdx.x * delta;
        double dsum = 0.0;
        for (int k = 0; k < n; ++k) {
            const double q = (u - (double)vals[k]) / bw;
            dsum += exp(-0.5 * q * q);
        }
        dens[threadIdx.x] = dsum;
        __syncthreads();
        int best = 0;
        double best_d = dens[0];
        for (int g = 1; g < kKdeGrid; ++g)           // the leftmost among equal maxima
            if (dens[g] > best_d) {
                best_d = dens[g];
                best = g;
            }
        cen = zmin + (double)best * delta;
    }
    __syncthreads();

    // ---- growth (every thread carries the same scalars)
    double rlo = cen, rhi = cen;
    bool done = false;
    for (int it = 0; it < kSearchMaxSteps && !done; ++it) {
        const int il = lower_bound_lds(vals, n, rlo), ih = lower_bound_lds(vals, n, rhi);
        if ((double)(ih - il) / (double)n >= t) {
            done = true;
            break;
        }
        const bool left_open = rlo > zmin, right_open = !(rhi > zmax);
        if (!left_open && !right_open) {
            done = true;
            break;
        }
        bool go_left = left_open;
        if (left_open && right_open) {
            // candidate 0: [rlo - step, rhi) = samples [cl, ih); candidate 1: [rlo, rhi + step) = samples [il, ch)
            const int cl = lower_bound_lds(vals, n, rlo - step), ch = lower_bound_lds(vals, n, rhi + step);
            const int n0 = ih - cl, n1 = ch - il;
            double sums[4] = {0.0, 0.0, 0.0, 0.0};   // sum z, sum g of both candidates
            for (int i = cl + (int)threadIdx.x; i < ch; i += kBlock) {
                const double zi = (double)vals[i], gi = gv[i];
                if (i < ih) { sums[0] += zi; sums[1] += gi; }
                if (i >= il) { sums[2] += zi; sums[3] += gi; }
            }
            block_sum4(sums, red4);
            const double zb0 = n0 ? sums[0] / n0 : 0.0, gb0 = n0 ? sums[1] / n0 : 0.0;
            const double zb1 = n1 ? sums[2] / n1 : 0.0, gb1 = n1 ? sums[3] / n1 : 0.0;
            double vc[4] = {0.0, 0.0, 0.0, 0.0};     // var, cov of both candidates
            for (int i = cl + (int)threadIdx.x; i < ch; i += kBlock) {
                const double zi = (double)vals[i], gi = gv[i];
                if (i < ih) { vc[0] += (zi - zb0) * (zi - zb0); vc[1] += (zi - zb0) * (gi - gb0); }
                if (i >= il) { vc[2] += (zi - zb1) * (zi - zb1); vc[3] += (zi - zb1) * (gi - gb1); }
            }
            block_sum4(vc, red4);
            double a0 = 0.0, c0 = gb0, a1 = 0.0, c1 = gb1;
            if (n0 >= 2 && vc[0] > 0.0) { a0 = vc[1] / vc[0]; c0 = gb0 - a0 * zb0; }
            if (n1 >= 2 && vc[2] > 0.0) { a1 = vc[3] / vc[2]; c1 = gb1 - a1 * zb1; }
            double er[4] = {0.0, 0.0, 0.0, 0.0};
            for (int i = cl + (int)threadIdx.x; i < ch; i += kBlock) {
                const double zi = (double)vals[i], gi = gv[i];
                if (i < ih) er[0] += fabs(gi - (a0 * zi + c0));
                if (i >= il) er[1] += fabs(gi - (a1 * zi + c1));
            }
            block_sum4(er, red4);
            go_left = er[0] < er[1];
        }
        if (go_left) rlo = rlo - step; else rhi = rhi + step;
    }
    if (!done) {   // the run-time guard on the number of steps was hit (a step far below the samples'
                   // spread): reported to the host, which fails the call; the whole sample range is
                   // stored so that the outputs are at least well defined
        if (threadIdx.x == 0) atomicAdd(n_capped, 1);
        rlo = zmin;
        rhi = nextafter(zmax, INFINITY);
    }
    __syncthreads();
    fit_and_store(vals, n, (float)rlo, (float)rhi, act, red, j, lo, hi, a, c);
}

// ------------------------------------------------- 8-bit floating-point storage of W'
// Nearest e4m3 code (1 sign, 4 exponent bits with bias 7, 3 mantissa bits, no infinities, largest
// value 448) of v, ties to the even mantissa, magnitudes above 448 saturate.
__device__ __forceinline__ uint32_t f32_to_e4m3(float v) {
    const uint32_t sign = (__float_as_uint(v) >> 24) & 0x80u;
    float m = fminf(fabsf(v), 448.0f);
    if (!(m == m)) return sign | 0x7Fu;
    uint32_t code;
    if (m < 0.015625f) {                              // below 2^-6: multiples of 2^-9 (8 is the first normal code)
        code = (uint32_t)rintf(m * 512.0f);
    } else {
        uint32_t u = __float_as_uint(m);
        u += 0x7FFFFu + ((u >> 20) & 1u);            // round the mantissa to 3 bits, ties to even (may carry into the exponent)
        u &= 0xFFF00000u;
        const uint32_t e = (u >> 23) - 127u + 7u;
        code = (e << 3) | ((u >> 20) & 7u);
        if (code > 0x7Eu) code = 0x7Eu;
    }
    return sign | code;
}

__device__ __forceinline__ float e4m3_to_f32(uint32_t code) {
    const uint32_t e = (code >> 3) & 15u, m = code & 7u;
    const float mag = e ? ldexpf(1.0f + (float)m * 0.125f, (int)e - 7) : (float)m * 0.001953125f;
    return (code & 0x80u) ? -mag : mag;
}

// One block per row of the fp32 folded matrix: the smallest power of two 2^e with max|row| / 2^e <= 448,
// the row's e4m3 codes in that scale, and the stored values code * 2^e as bf16 (exactly representable)
__global__ void __launch_bounds__(kBlock)
wp_to_fp8_kernel(const float* __restrict__ acc, int64_t d, uint8_t* __restrict__ codes, float* __restrict__ scale,
                 bf16_t* __restrict__ Wp) {
    __shared__ float red[kBlock / TD_WAVE];
    const int64_t i = blockIdx.x;
    const float* row = acc + i * d;
    float m = 0.0f;
    for (int64_t k = threadIdx.x; k < d; k += kBlock) m = fmaxf(m, fabsf(row[k]));
    m = td_wave_max(m);
    if ((threadIdx.x & 63) == 0) red[threadIdx.x / 64] = m;
    __syncthreads();
    m = red[0];
#pragma unroll
    for (int w = 1; w < kBlock / TD_WAVE; ++w) m = fmaxf(m, red[w]);
    int e = 0;
    if (m > 0.0f && m < INFINITY) {
        int k;
        const float f = frexpf(m, &k);               // m = f 2^k, 0.5 <= f < 1; 448 = 0.875 * 2^9
        e = f <= 0.875f ? k - 9 : k - 8;
    }
    if (threadIdx.x == 0) scale[i] = ldexpf(1.0f, e);
    for (int64_t k = threadIdx.x; k < d; k += kBlock) {
        const uint32_t cde = f32_to_e4m3(ldexpf(row[k], -e));
        codes[i * d + k] = (uint8_t)cde;
        Wp[i * d + k] = td_f32_to_bf16(ldexpf(e4m3_to_f32(cde), e));
    }
}

// ------------------------------------------------- adaptive thresholding (Algorithm 1, outer loops)
// E_n = ||W2[:, n]||_2 * sum over the calibration inputs with lo_n <= z < hi_n of |sigma(z) - (a_n z + c_n)|:
// the section's per-neuron error metric err_n summed over the calibration set (outside the range
// the approximated activation equals the exact one).  One block per neuron, fp64 sums.
__global__ void __launch_bounds__(kBlock)
neuron_error_kernel(const float* __restrict__ Zt, int n, const float* __restrict__ lo, const float* __restrict__ hi,
                    const float* __restrict__ a, const float* __restrict__ c, const float* __restrict__ colnorm, int act,
                    float* __restrict__ err) {
    __shared__ double red[kBlock / TD_WAVE];
    const int64_t j = blockIdx.x;
    const float* z = Zt + j * (int64_t)n;
    const double l = (double)lo[j], r = (double)hi[j], aj = (double)a[j], cj = (double)c[j];
    double sum = 0.0;
    for (int i = threadIdx.x; i < n; i += kBlock) {
        const double zi = (double)z[i];
        if (zi >= l && zi < r) sum += fabs(td_act_f64(zi, act) - (aj * zi + cj));
    }
    sum = block_sum(sum, red);
    if (threadIdx.x == 0) err[j] = (float)(sum * (double)colnorm[j]);
}

// colnorm[j] = ||W2[:, j]||_2 for W2 stored d x h (thread per column, rows walked in order)
template <typename T>
__global__ void __launch_bounds__(kBlock)
col_norm_kernel(const T* __restrict__ W2, int64_t d, int64_t h, float* __restrict__ colnorm) {
    const int64_t j = (int64_t)blockIdx.x * kBlock + threadIdx.x;
    if (j >= h) return;
    double ss = 0.0;
    for (int64_t i = 0; i < d; ++i) {
        const double w = (double)td_load<T>(W2 + i * h + j);
        ss += w * w;
    }
    colnorm[j] = (float)sqrt(ss);
}

// out[0] = sum of v[0..n) in a fixed order (one block)
__global__ void __launch_bounds__(kBlock) sum_fixed_kernel(const float* __restrict__ v, int64_t n, float* __restrict__ out) {
    __shared__ double red[kBlock / TD_WAVE];
    double sum = 0.0;
    for (int64_t i = threadIdx.x; i < n; i += kBlock) sum += (double)v[i];
    sum = block_sum(sum, red);
    if (threadIdx.x == 0) out[0] = (float)sum;
}

// Solution of   minimise sum E_i t_i,  sum t_i = t n,  t_min <= t_i <= t_max :
// the k = floor((n t_max - t n) / (t_max - t_min)) items of largest error (equal errors: lower index
// first) get t_min, the next one t_max minus the rest of the excess, all others t_max.  Thread i
// finds its own rank by counting (tiles of the errors staged in LDS).
__global__ void __launch_bounds__(kBlock)
assign_thresholds_kernel(const float* __restrict__ E, int64_t n, double t, double t_min, double t_max,
                         float* __restrict__ out) {
    __shared__ float tile[kBlock];
    const int64_t i = (int64_t)blockIdx.x * kBlock + threadIdx.x;
    const float mine = i < n ? E[i] : 0.0f;
    int64_t rank = 0;
    for (int64_t j0 = 0; j0 < n; j0 += kBlock) {
        __syncthreads();
        tile[threadIdx.x] = j0 + threadIdx.x < n ? E[j0 + threadIdx.x] : 0.0f;
        __syncthreads();
        const int lim = (int)(n - j0 < kBlock ? n - j0 : kBlock);
        for (int u = 0; u < lim; ++u) {
            const float other = tile[u];
            rank += (other > mine || (other == mine && j0 + u < i)) ? 1 : 0;
        }
    }
    if (i >= n) return;
    double v = t_max;
    if (t_max > t_min) {
        const double width = t_max - t_min;
        const double excess = (double)n * t_max - t * (double)n;
        double k = floor(excess / width);
        if (k > (double)n) k = (double)n;
        if ((double)rank < k) v = t_min;
        else if ((double)rank == k) v = t_max - (excess - k * width);
    }
    out[i] = (float)v;
}

// ------------------------------------------------- bound for the fixed-point repair accumulators
// For a token x and any set F of neurons, every partial sum of the terms that make up output i,
//     W'[i,:] x + b'_i      and      delta_j W2[i,j]  (j in F),
// is bounded in magnitude by  K1 max|x| + K2  with
//     K1 = max_i ( sum_k |W'_ik| + sum_j |W2_ij| (1 + |a_j|) ||W1_j||_1 )
//     K2 = max_i ( |b'_i|        + sum_j |W2_ij| ((1 + |a_j|) |b1_j| + |c_j|) )
// because |delta_j| = |sigma(z_j) - (a_j z_j + c_j)| <= (1 + |a_j|) |z_j| + |c_j| for every supported
// activation (|sigma(z)| <= |z|) and |z_j| <= ||W1_j||_1 max|x| + |b1_j|.
template <typename T>
__global__ void __launch_bounds__(kBlock)
fx_row_terms_kernel(const T* __restrict__ W1, const T* __restrict__ b1, const float* __restrict__ a,
                    const float* __restrict__ c, int64_t d, float* __restrict__ g, float* __restrict__ kk) {
    __shared__ float red[kBlock / TD_WAVE];
    const int64_t j = blockIdx.x;
    float sabs = 0.0f;
    for (int64_t k = threadIdx.x; k < d; k += kBlock) sabs += fabsf(td_load<T>(W1 + j * d + k));
    sabs = td_wave_sum(sabs);
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = sabs;
    __syncthreads();
    if (threadIdx.x == 0) {
        float tot = 0.0f;
        for (int w = 0; w < kBlock / TD_WAVE; ++w) tot += red[w];
        const float aj = 1.0f + fabsf(a[j]);
        g[j] = aj * tot;
        kk[j] = aj * (b1 ? fabsf(td_load<T>(b1 + j)) : 0.0f) + fabsf(c[j]);
    }
}

// P[(chunk * 2 + q) * d + i] = sum over the chunk's neurons j of |W2T[j][i]| * (q == 0 ? g_j : kk_j)
template <typename T>
__global__ void __launch_bounds__(kBlock)
fx_col_terms_kernel(const T* __restrict__ W2T, int64_t h, int64_t d, const float* __restrict__ g,
                    const float* __restrict__ kk, int64_t rows_per_chunk, float* __restrict__ P) {
    const int64_t i = (int64_t)blockIdx.x * kBlock + threadIdx.x;
    const int64_t ch = blockIdx.y;
    if (i >= d) return;
    const int64_t j0 = ch * rows_per_chunk, j1 = j0 + rows_per_chunk < h ? j0 + rows_per_chunk : h;
    float s1 = 0.0f, s2 = 0.0f;
    for (int64_t j = j0; j < j1; ++j) {
        const float w = fabsf(td_load<T>(W2T + j * d + i));
        s1 = fmaf(w, g[j], s1);
        s2 = fmaf(w, kk[j], s2);
    }
    P[(ch * 2 + 0) * d + i] = s1;
    P[(ch * 2 + 1) * d + i] = s2;
}

// out[0] = K1, out[1] = K2 (maxima over the outputs; non-negative floats order like their bit patterns)
template <typename T>
__global__ void __launch_bounds__(kBlock)
fx_bound_kernel(const T* __restrict__ Wp, const float* __restrict__ bp, int64_t d, const float* __restrict__ P,
                int chunks, float* __restrict__ out) {
    __shared__ float red[kBlock / TD_WAVE];
    const int64_t i = blockIdx.x;
    float sabs = 0.0f;
    for (int64_t k = threadIdx.x; k < d; k += kBlock) sabs += fabsf(td_load<T>(Wp + i * d + k));
    sabs = td_wave_sum(sabs);
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = sabs;
    __syncthreads();
    if (threadIdx.x == 0) {
        float k1 = 0.0f, k2 = fabsf(bp[i]);
        for (int w = 0; w < kBlock / TD_WAVE; ++w) k1 += red[w];
        for (int ch = 0; ch < chunks; ++ch) {
            k1 += P[((int64_t)ch * 2 + 0) * d + i];
            k2 += P[((int64_t)ch * 2 + 1) * d + i];
        }
        // a little above the fp32 value of the sums, so that their own rounding cannot undercut the bound
        atomicMax(reinterpret_cast<int*>(out), __float_as_int(k1 * 1.01f));
        atomicMax(reinterpret_cast<int*>(out) + 1, __float_as_int(k2 * 1.01f));
    }
}

dim3 tile_grid(int64_t cols, int64_t rows, int64_t side = 32) {
    return dim3((unsigned)((cols + side - 1) / side), (unsigned)((rows + side - 1) / side));
}

}  // namespace

template <typename T>
static tardis_status_t fx_bounds_t(const tardis_layer_s* L, float* out2, hipStream_t s) {
    const int64_t d = L->d, h = L->h;
    const int chunks = 32;
    const int64_t rpc = (h + chunks - 1) / chunks;
    td_dev_buf g, kk, P;
    TD_TRY(g.alloc((size_t)h * 4));
    TD_TRY(kk.alloc((size_t)h * 4));
    TD_TRY(P.alloc((size_t)chunks * 2 * d * 4));
    TD_HIP(hipMemsetAsync(out2, 0, 8, s));
    hipLaunchKernelGGL(fx_row_terms_kernel<T>, dim3((unsigned)h), dim3(kBlock), 0, s, static_cast<const T*>(L->W1),
                       static_cast<const T*>(L->b1), L->a, L->c, d, static_cast<float*>(g.p), static_cast<float*>(kk.p));
    hipLaunchKernelGGL(fx_col_terms_kernel<T>, dim3((unsigned)((d + kBlock - 1) / kBlock), chunks), dim3(kBlock), 0, s,
                       static_cast<const T*>(L->W2T), h, d, static_cast<const float*>(g.p),
                       static_cast<const float*>(kk.p), rpc, static_cast<float*>(P.p));
    hipLaunchKernelGGL(fx_bound_kernel<T>, dim3((unsigned)d), dim3(kBlock), 0, s, static_cast<const T*>(L->Wp), L->bp, d,
                       static_cast<const float*>(P.p), chunks, out2);
    TD_HIP(hipGetLastError());
    TD_HIP(hipStreamSynchronize(s));   // the temporaries go out of scope
    return TARDIS_OK;
}

tardis_status_t td_estimate_errors(const tardis_ffn_desc* desc, const void* X, int64_t n, const float* lo,
                                   const float* hi, const float* a, const float* c, float* err, float* err_layer,
                                   hipStream_t s) {
    const int64_t d = desc->d, h = desc->h;
    td_dev_buf zt, cn;
    TD_TRY(zt.alloc((size_t)h * n * 4));
    TD_TRY(cn.alloc((size_t)h * 4));
    TD_TRY(td_gemm_nt(desc->W1, X, static_cast<float*>(zt.p), h, n, d, desc->dtype, 0, desc->b1, s));
    const dim3 cgrid((unsigned)((h + kBlock - 1) / kBlock));
    if (desc->dtype == TARDIS_BF16)
        hipLaunchKernelGGL(col_norm_kernel<bf16_t>, cgrid, dim3(kBlock), 0, s, static_cast<const bf16_t*>(desc->W2), d, h,
                           static_cast<float*>(cn.p));
    else
        hipLaunchKernelGGL(col_norm_kernel<float>, cgrid, dim3(kBlock), 0, s, static_cast<const float*>(desc->W2), d, h,
                           static_cast<float*>(cn.p));
    hipLaunchKernelGGL(neuron_error_kernel, dim3((unsigned)h), dim3(kBlock), 0, s, static_cast<const float*>(zt.p), (int)n,
                       lo, hi, a, c, static_cast<const float*>(cn.p), (int)desc->act, err);
    if (err_layer) hipLaunchKernelGGL(sum_fixed_kernel, dim3(1), dim3(kBlock), 0, s, err, h, err_layer);
    TD_HIP(hipGetLastError());
    TD_HIP(hipStreamSynchronize(s));
    return TARDIS_OK;
}

tardis_status_t td_assign_thresholds(const float* err, int64_t n, float t, float t_min, float t_max, float* out,
                                     hipStream_t s) {
    hipLaunchKernelGGL(assign_thresholds_kernel, dim3((unsigned)((n + kBlock - 1) / kBlock)), dim3(kBlock), 0, s, err, n,
                       (double)t, (double)t_min, (double)t_max, out);
    TD_HIP(hipGetLastError());
    return TARDIS_OK;
}

// K1, K2 of the fixed-point accumulators' magnitude bound into out2[0..1] (device); needs W2T, W', b', a, c
tardis_status_t td_fx_bounds(const tardis_layer_s* L, float* out2, hipStream_t s) {
    return L->dtype == TARDIS_BF16 ? fx_bounds_t<bf16_t>(L, out2, s) : fx_bounds_t<float>(L, out2, s);
}

tardis_status_t td_transpose(const void* src, void* dst, void* copy, int64_t rows, int64_t cols, int32_t dtype, hipStream_t s) {
    if ((rows + 31) / 32 > 65535) return TARDIS_ERR_SHAPE;
    const bool whole = rows % 8 == 0 && cols % 8 == 0 && (reinterpret_cast<uintptr_t>(src) & 15) == 0;
    if (dtype == TARDIS_BF16 && whole)
        hipLaunchKernelGGL(transpose16_kernel<false>, tile_grid(cols, rows, 64), dim3(256), 0, s,
                           static_cast<const bf16_t*>(src), static_cast<bf16_t*>(dst), static_cast<bf16_t*>(copy), nullptr, rows, cols);
    else if (dtype == TARDIS_BF16)
        hipLaunchKernelGGL(transpose_kernel<uint16_t>, tile_grid(cols, rows), dim3(256), 0, s,
                           static_cast<const uint16_t*>(src), static_cast<uint16_t*>(dst), rows, cols);
    else
        hipLaunchKernelGGL(transpose_kernel<uint32_t>, tile_grid(cols, rows), dim3(256), 0, s,
                           static_cast<const uint32_t*>(src), static_cast<uint32_t*>(dst), rows, cols);
    if (!(dtype == TARDIS_BF16 && whole))
        TD_HIP(hipMemcpyAsync(copy, src, (size_t)rows * cols * td_elem_size(dtype), hipMemcpyDeviceToDevice, s));
    TD_HIP(hipGetLastError());
    return TARDIS_OK;
}

tardis_status_t td_build_sketch(const void* W1, const void* b1, const float* lo, const float* hi, int64_t h,
                                int64_t d, int32_t dtype, int32_t bits, float margin, int8_t* Q, uint8_t* Q4,
                                uint8_t* M4, float* tlo, float* thi, float* code_scale, int32_t* no_scale, hipStream_t s) {
    if (bits == 4 || bits == 3 || bits == 2) {
        const int qmax = (1 << (bits - 1)) - 1;
        const int64_t ng = (d + 31) / 32;
        if (!M4 || (Q4 && d % 32 != 0) || ng * 4 > 64 * 1024) return TARDIS_ERR_SHAPE;
        auto launch = [&](auto type) {
            typedef decltype(type) T;
            const T *W = static_cast<const T*>(W1), *b = static_cast<const T*>(b1);
            if (d % 32 == 0)
                hipLaunchKernelGGL(sketch4_rows_kernel<T>, dim3((unsigned)h), dim3(kBlock), 0, s, W, b, lo, hi, d, Q, Q4, M4, tlo, thi, qmax,
                                   margin);
            else
                hipLaunchKernelGGL(sketch4_kernel<T>, dim3((unsigned)h), dim3(kBlock), (size_t)ng * 4, s, W, b, lo, hi, d, (int)ng, Q, M4,
                                   tlo, thi, qmax, margin);
        };
        if (dtype == TARDIS_BF16) launch(bf16_t{});
        else launch(float{});
        TD_HIP(hipGetLastError());
        return TARDIS_OK;
    }
    if (bits != 8 || !Q) return TARDIS_ERR_INVALID_ARG;
    if (dtype == TARDIS_BF16)
        hipLaunchKernelGGL(sketch_kernel<bf16_t>, dim3((unsigned)h), dim3(kBlock), 0, s,
                           static_cast<const bf16_t*>(W1), static_cast<const bf16_t*>(b1), lo, hi, d, Q, tlo, thi, margin, code_scale, no_scale);
    else
        hipLaunchKernelGGL(sketch_kernel<float>, dim3((unsigned)h), dim3(kBlock), 0, s,
                           static_cast<const float*>(W1), static_cast<const float*>(b1), lo, hi, d, Q, tlo, thi, margin, nullptr, nullptr);
    TD_HIP(hipGetLastError());
    return TARDIS_OK;
}

tardis_status_t td_unpack_sketch4(const uint8_t* Q4, const uint8_t* M4, int64_t h, int64_t d, int8_t* Q,
                                  hipStream_t s) {
    hipLaunchKernelGGL(unpack_sketch4_kernel, dim3((unsigned)h), dim3(kBlock), 0, s, Q4, M4, d, Q);
    TD_HIP(hipGetLastError());
    return TARDIS_OK;
}

tardis_status_t td_fold(const tardis_ffn_desc* desc, const float* a, const float* c, void* Wp, float* bp,
                        uint8_t* Wp8, float* wp8_scale, void* work1, void* work2, const td_fold_work& work, hipStream_t s) {
    if (Wp8 && desc->dtype != TARDIS_BF16) return TARDIS_ERR_DTYPE;
    const int64_t d = desc->d, h = desc->h;
    if ((h + 31) / 32 > 65535 || (d + 31) / 32 > 65535) return TARDIS_ERR_SHAPE;
    const td_dev_buf &kk = work.terms, &acc = work.sums;
    if (desc->dtype == TARDIS_BF16) {
        if (d % 8 == 0 && h % 8 == 0)
            hipLaunchKernelGGL(transpose16_kernel<true>, tile_grid(d, h, 64), dim3(256), 0, s,
                               static_cast<const bf16_t*>(desc->W1), static_cast<bf16_t*>(work1),
                               static_cast<bf16_t*>(work2), a, h, d);
        else
            hipLaunchKernelGGL(scale_transpose_bf16_kernel, tile_grid(d, h), dim3(256), 0, s,
                               static_cast<const bf16_t*>(desc->W1), a, static_cast<bf16_t*>(work1),
                               static_cast<bf16_t*>(work2), h, d);
        TD_TRY(td_gemm_nt(desc->W2, work1, static_cast<float*>(acc.p), d, d, h, TARDIS_BF16, 0, nullptr, s));
        // (the second product's epilogue rounds the sums; a kernel for that took 27 us and their 64 MB once more each way)
        const bool round = !Wp8 && td_gemm_on_matrix_cores(desc->W2, work2, d, d, h, TARDIS_BF16);
        TD_TRY(td_gemm_nt(desc->W2, work2, static_cast<float*>(acc.p), d, d, h, TARDIS_BF16, 1, nullptr, s, round ? Wp : nullptr));
        const int64_t n = d * d;
        if (Wp8)
            hipLaunchKernelGGL(wp_to_fp8_kernel, dim3((unsigned)d), dim3(kBlock), 0, s, static_cast<const float*>(acc.p),
                               d, Wp8, wp8_scale, static_cast<bf16_t*>(Wp));
        else if (!round)
            hipLaunchKernelGGL(f32_to_bf16_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s,
                               static_cast<const float*>(acc.p), static_cast<bf16_t*>(Wp), n);
        hipLaunchKernelGGL(fold_bias_terms_kernel<bf16_t>, dim3((unsigned)((h + kBlock - 1) / kBlock)), dim3(kBlock), 0, s,
                           static_cast<const bf16_t*>(desc->b1), a, c, static_cast<double*>(kk.p), h);
        hipLaunchKernelGGL(fold_bias_kernel<bf16_t>, dim3((unsigned)((d + kBiasRows - 1) / kBiasRows)), dim3(kBlock), 0, s,
                           static_cast<const bf16_t*>(desc->W2), static_cast<const double*>(kk.p),
                           static_cast<const bf16_t*>(desc->b2), bp, d, h);
        TD_HIP(hipGetLastError());
        TD_HIP(hipStreamSynchronize(s));  // `work` is the caller's to free
    } else {
        hipLaunchKernelGGL(scale_transpose_f32_kernel, tile_grid(d, h), dim3(256), 0, s,
                           static_cast<const float*>(desc->W1), a, static_cast<float*>(work1), h, d);
        TD_TRY(td_gemm_nt(desc->W2, work1, static_cast<float*>(Wp), d, d, h, TARDIS_F32, 0, nullptr, s));
        hipLaunchKernelGGL(fold_bias_terms_kernel<float>, dim3((unsigned)((h + kBlock - 1) / kBlock)), dim3(kBlock), 0, s,
                           static_cast<const float*>(desc->b1), a, c, static_cast<double*>(kk.p), h);
        hipLaunchKernelGGL(fold_bias_kernel<float>, dim3((unsigned)((d + kBiasRows - 1) / kBiasRows)), dim3(kBlock), 0, s,
                           static_cast<const float*>(desc->W2), static_cast<const double*>(kk.p),
                           static_cast<const float*>(desc->b2), bp, d, h);
        TD_HIP(hipGetLastError());
        TD_HIP(hipStreamSynchronize(s));
    }
    return TARDIS_OK;
}

tardis_status_t td_calibrate(const tardis_ffn_desc* desc, const void* X, int64_t n, float coverage,
                             const float* cov_pn, float step, float* lo, float* hi, float* a, float* c,
                             hipStream_t s) {
    const int64_t d = desc->d, h = desc->h;
    if (td_gemm_refuses_rows(h)) return TARDIS_ERR_SHAPE;   // (of all neurons, also where they come in chunks below)
    td_dev_buf zt;
    if (step <= 0.0f) {
        // The pre-activations of a chunk of neurons at a time: 64 MiB of them make one round of 256 x 256 tiles
        // over the 256 CUs, are still in the last-level cache when the fit reads them, and are the largest
        // buffer the runtime keeps for the next call instead of mapping and unmapping it (0.3 ms and more).
        int64_t rows = (int64_t)(64 << 20) / (4 * n) / 256 * 256;
        rows = rows < 256 ? 256 : (rows > h ? h : rows);
        TD_TRY(zt.alloc((size_t)rows * n * 4));
        const size_t es = td_elem_size(desc->dtype);
        for (int64_t j0 = 0; j0 < h; j0 += rows) {
            tardis_ffn_desc part = *desc;                 // the neurons [j0, j0 + part.h)
            part.h = h - j0 < rows ? h - j0 : rows;
            part.W1 = static_cast<const char*>(desc->W1) + (size_t)j0 * d * es;
            part.b1 = desc->b1 ? static_cast<const char*>(desc->b1) + (size_t)j0 * es : nullptr;
            float* z = static_cast<float*>(zt.p);
            TD_TRY(td_gemm_nt(part.W1, X, z, part.h, n, d, desc->dtype, 0, part.b1, s));
            const float* cov = cov_pn ? cov_pn + j0 : nullptr;
            if (desc->dtype == TARDIS_BF16)
                TD_TRY(launch_calibrate<bf16_t>(&part, z, X, (int)n, coverage, cov, lo + j0, hi + j0, a + j0, c + j0, s));
            else
                TD_TRY(launch_calibrate<float>(&part, z, X, (int)n, coverage, cov, lo + j0, hi + j0, a + j0, c + j0, s));
        }
        TD_HIP(hipStreamSynchronize(s));
        return TARDIS_OK;
    }
    TD_TRY(zt.alloc((size_t)h * n * 4));
    TD_TRY(td_gemm_nt(desc->W1, X, static_cast<float*>(zt.p), h, n, d, desc->dtype, 0, desc->b1, s));
    int npad = 2;
    while (npad < n) npad <<= 1;
    const size_t lds = (size_t)((n + 1) & ~(int64_t)1) * sizeof(double) + (size_t)npad * sizeof(float);
    if (lds > 48 * 1024)
        TD_HIP(hipFuncSetAttribute(reinterpret_cast<const void*>(range_search_kernel),
                                   hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds));
    td_dev_buf capped;
    TD_TRY(capped.alloc(sizeof(int)));
    TD_HIP(hipMemsetAsync(capped.p, 0, sizeof(int), s));
    hipLaunchKernelGGL(range_search_kernel, dim3((unsigned)h), dim3(kBlock), lds, s,
                       static_cast<const float*>(zt.p), (int)n, npad, coverage, cov_pn, step, (int)desc->act, lo,
                       hi, a, c, static_cast<int*>(capped.p));
    TD_HIP(hipGetLastError());
    int n_capped = 0;
    TD_HIP(hipMemcpyAsync(&n_capped, capped.p, sizeof(int), hipMemcpyDeviceToHost, s));
    TD_HIP(hipStreamSynchronize(s));
    // Algorithm 1 has no limit on the number of growth steps; the kernel's guard (4096) is only
    // reached when `step` is absurdly small against a neuron's spread of inputs: refuse, do not
    // substitute another range
    return n_capped > 0 ? TARDIS_ERR_INVALID_ARG : TARDIS_OK;
}

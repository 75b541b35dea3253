// Products of up to 64 tokens with a weight matrix, as streams of the weights (bf16 layers, rows that are whole slices):
//  * the up product of the folded path.  One pass over W1 gives the predictor's integer sums and the pre-activations: a code is
//    rint(w s) with a scale s of the row (td_code_scale), so the fragments of W1 that are multiplied by the tokens are also rounded to
//    codes (one fma onto 1.5 * 2^23, whose low byte is the code) and multiplied by the tokens' codes.  Q, a third of the bytes, is not read;
//  * the output product [X | D] [W' | W2]^T, in ranges of K whose sums the finishing kernel adds.
//
// What bounds it: the weights' stream from HBM, once, and what stands before and behind it in a launch.  Hence:
//  * a block has 64 (32) rows of the weights, so that there is one for each of the 256 CUs, and all tokens; K runs in slices of 128
//    columns (256 bytes of a weight row: shorter runs stream slower), loaded straight to LDS;
//  * wavefronts 0-3 load weights, 4-7 tokens.  A wavefront's loads arrive in order, so with both kinds in one wavefront the deeper
//    ring could not be waited for without the other one's newest loads; apart, the weights are up to NW slices ahead (64 KB and more
//    per CU under way, HBM's latency) and the tokens, which come from L2, NX (with 2 for 3: 77 -> 90 us; 5 for 3 where they fit: -2 %);
//  * the 8 wavefronts divide a slice by quarters of its K first, then by row blocks of the weights (two each), then by tokens: a
//    fragment of tokens is multiplied by two of the weights, and every weight is rounded once (32-row tiles: twice).  The quarters' sums
//    meet in LDS at the end;
//  * the fragments of the next slice are read while this one's are multiplied;
//  * the kernel before asks for the first slices (stream_warm: 79.0 -> 77.3 us; twice as many: 83).
// d = 4096, h = 16384, 64 tokens, kernel trace: up product 40.5 (both matrices read, gemm_tile_kernel) -> 34 us, of which the stream of
// 134 MB 24 (5.5 TB/s), its beginning 2.5, the end 4; output product 38.9 -> 34 (168 MB, 27 of the 34 stream: 6.2 TB/s).  The same without
// any multiplication 29 and 30.5.  The whole call: 64 tokens 85.2 -> 77.0 us, 18 tokens 82.6 -> 72.3; d = 2048, h = 8192, 24 tokens
// 33.1 -> 30.4; dense, d = 4096, h = 16384, 20 tokens 67.5 -> 59.3.
#include "common.h"
#include "codes.h"
#include "sigma.h"
#include "tiles.h"

namespace {

typedef __bf16 bf16x8_t __attribute__((ext_vector_type(8)));

struct StreamArgs {
    StreamPlan w;                  // the weights (a second matrix and ranges of K: PART)
    const unsigned char *A, *A2;   // tokens, K-contiguous as the weights
    const unsigned char* XQ;       // REPAIR: token codes
    int64_t M;
    StreamPlan next;               // REPAIR: what the launch behind this one begins with (tile = 0: nothing)
    float* C;                      // PART: [range][M][N]
    const bf16_t* bias;            // REPAIR, per column: b1,
    const float *codes, *lo, *hi;  //   code per weight, bounds of the range test,
    const float *slope, *icept;    //   line
    const int32_t* e;              //   exponent per row (readable to the next multiple of 16 bytes)
    uint32_t* mask;
    int mask_words;
    bf16_t *out, *rest;            //   as td_gemm_repair's
    int act;
};

enum { STREAM_PART, STREAM_REPAIR };

template <int MODE, int TF, int NF>
struct StreamTile {
    static constexpr int SL = 256, TM = 16 * TF, TN = 16 * NF;
    static constexpr int WN = NF / 2, TS = 2 / WN, TW = TF / TS;   // wavefronts along the weights' rows, along the tokens; token blocks of one
    static constexpr int UW = TN * SL, UX = TM * SL, UQ = MODE == STREAM_REPAIR ? TM * SL / 2 : 0;   // bytes of a slice
    static constexpr int kPar = MODE == STREAM_REPAIR ? 6 * 1024 : 0;
    static constexpr int NX = UQ > 0 && TF == 4 ? 3 : 5;     // slices in the rings of the tokens, of the weights
    static constexpr int kRoom = (kLdsBytes - kPar - NX * (UX + UQ)) / UW, NW = kRoom < 12 ? kRoom : 12;
    static constexpr int LW = UW / 4096, LX = UX / 4096, LQ = UQ / 4096;      // loads of a wavefront per slice
    static constexpr int kX = NW * UW, kQ = kX + NX * UX, kParAt = kQ + NX * UQ, kLds = kParAt + kPar;
    static constexpr int FR = 2 * TW, KEEP = FR >= 4 ? FR / 4 : 1;   // sums of a wavefront; how many of them it finishes
    static constexpr int kSum = MODE == STREAM_REPAIR ? 2048 : 1024;
    static constexpr int kStage = 8 * FR * kSum;             // (behind the sums that are exchanged)
    static_assert((NF == 4 || NF == 2) && (TF == 4 || TF == 2), "eight wavefronts");
    static_assert(NW >= 4 && (NW - 1) * LW <= 63 && kStage + TM * TN * 4 <= kParAt, "rings, staging");
};

// The 8 predictor codes of a lane's fragment: the stored ones, see td_code_scale
__device__ __forceinline__ long codes_of(const td_u32x4& w, float s) {
    auto code = [&](uint32_t bits) { return td_code_bits(__uint_as_float(bits), s); };
    auto four = [&](uint32_t a, uint32_t b) {
        const uint32_t lo = __builtin_amdgcn_perm(code(a & 0xffff0000u), code(a << 16), 0x0c0c0400u);
        const uint32_t hi = __builtin_amdgcn_perm(code(b & 0xffff0000u), code(b << 16), 0x04000c0cu);
        return lo | hi;
    };
    return __builtin_bit_cast(long, make_uint2(four(w[0], w[1]), four(w[2], w[3])));
}

template <int MODE, int TF, int NF>
__global__ void __launch_bounds__(512) stream_kernel(StreamArgs p) {
    typedef StreamTile<MODE, TF, NF> G;
    constexpr int SL = G::SL, TM = G::TM, TN = G::TN, TW = G::TW, NW = G::NW, NX = G::NX, FR = G::FR, KEEP = G::KEEP;
    extern __shared__ __align__(1024) unsigned char lds[];
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int quarter = wave >> 1, wn = G::WN == 2 ? wave & 1 : 0, tw = G::TS == 2 ? wave & 1 : 0;   // of K; along the weights' rows, the tokens
    const int frow = lane & 15, fp = lane >> 4;

    const StreamBlock blk = stream_block(p.w, (int)blockIdx.x);
    const int64_t n0 = blk.n0, N = p.w.N;
    const uint32_t k1 = p.w.k, k2 = MODE == STREAM_PART ? p.w.k2 : 0u;
    const int nk1 = (int)(k1 / SL), s0 = blk.s0, nk = blk.nk;
    const uint32_t rows_w = (uint32_t)min((int64_t)TN, N - n0), rows_x = (uint32_t)p.M;

    const uint32_t base = __builtin_amdgcn_readfirstlane((uint32_t)(uintptr_t)(__attribute__((address_space(3))) unsigned char*)lds);
    const int part = wave & 3;                        // wavefronts 0-3: this quarter of the weight rows, 4-7: of the tokens
    const bool weights = wave < 4;
    const i32x4_t r1 = weights ? buffer_of(p.w.B + (size_t)n0 * k1, rows_w * k1) : buffer_of(p.A, rows_x * k1);
    const i32x4_t r2 = MODE == STREAM_PART ? (weights ? buffer_of(p.w.B2 + (size_t)n0 * k2, rows_w * k2) : buffer_of(p.A2, rows_x * k2)) : r1;
    const i32x4_t rq = buffer_of(p.XQ, rows_x * (k1 / 2));
    // a load of weights or tokens: 4 rows of 256 bytes, lane -> row lane / 16, piece (lane % 16) ^ row; of token codes 8 rows of 128
    constexpr int LW = G::LW, LX = G::LX, LQ = G::LQ, LMAX = LW > LX ? LW : LX;
    const uint32_t row0 = (uint32_t)(part * (weights ? TN / 4 : TM / 4)) + ((uint32_t)lane >> 4);
    uint32_t off1[LMAX], off2[LMAX], off_q[LQ > 0 ? LQ : 1];   // offsets of this lane's loads in a slice, of either pair, of the codes
#pragma unroll
    for (int i = 0; i < LMAX; ++i) {
        const uint32_t row = row0 + 4 * i, pc = (((uint32_t)lane ^ row) & 15u) * 16u;
        off1[i] = row * k1 + pc;
        off2[i] = row * k2 + pc;
    }
#pragma unroll
    for (int i = 0; i < LQ; ++i) {
        const uint32_t row = (uint32_t)(part * (TM / 4) + 8 * i) + ((uint32_t)lane >> 3);
        off_q[i] = row * (k1 / 2) + (((uint32_t)lane ^ row) & 7u) * 16u;
    }
    int left = nk, at = s0 + blk.rot;                     // slices to load, the next one
    const uint32_t to_w = base + (uint32_t)part * (G::UW / 4), to_x = base + G::kX + (uint32_t)part * (G::UX / 4), to_q = base + G::kQ + (uint32_t)part * (G::UQ / 4);
    auto load_slice = [&](uint32_t slot) {            // this wavefront's share of the next slice (past the last one: nothing is fetched)
        const bool live = left > 0, second = MODE == STREAM_PART && at >= nk1;
        const uint32_t soff = live ? (uint32_t)(second ? at - nk1 : at) * SL : 0u;
        i32x4_t rs = r1;
        if (second) rs = r2;
        rs.z = live ? rs.z : 0;
        auto fetch = [&](const uint32_t (&off)[LMAX]) {
            if (weights) {
#pragma unroll
                for (int i = 0; i < LW; ++i) load_to_lds<true>(to_w + slot * G::UW + i * 1024u, off[i], rs, soff);
            } else {
#pragma unroll
                for (int i = 0; i < LX; ++i) load_to_lds(to_x + slot * G::UX + i * 1024u, off[i], rs, soff);
            }
        };
        if (second) fetch(off2);
        else fetch(off1);
        if constexpr (MODE == STREAM_REPAIR) {
            if (!weights) {
                i32x4_t r = rq;
                r.z = live ? r.z : 0;
#pragma unroll
                for (int i = 0; i < LQ; ++i) load_to_lds(to_q + slot * G::UQ + i * 1024u, off_q[i], r, soff / 2);
            }
        }
        --left;
        at = at + 1 == s0 + nk ? s0 : at + 1;
    };

    bf16_t bias = 0;
    if constexpr (MODE == STREAM_REPAIR) {
        if (tid < TN && n0 + tid < N) bias = p.bias[n0 + tid];
        const uint32_t at_par = base + G::kParAt;
        if (wave == 4) load_to_lds(at_par, lane * 16, buffer_of(p.codes + n0, rows_w * 4), 0u);
        if (wave == 5) load_to_lds(at_par + 1024, lane * 16, buffer_of(p.lo + n0, rows_w * 4), 0u);
        if (wave == 6) load_to_lds(at_par + 2048, lane * 16, buffer_of(p.hi + n0, rows_w * 4), 0u);
        if (wave == 7) load_to_lds(at_par + 3072, lane * 16, buffer_of(p.slope + n0, rows_w * 4), 0u);
        if (wave == 4) load_to_lds(at_par + 4096, lane * 16, buffer_of(p.icept + n0, rows_w * 4), 0u);
        if (wave == 5) load_to_lds(at_par + 5120, lane * 16, buffer_of(p.e, (rows_x * 4 + 15u) & ~15u), 0u);
    }
    if (weights) {
#pragma unroll 1
        for (int s = 0; s < NW; ++s) load_slice(s);
    } else {
#pragma unroll 1
        for (int s = 0; s < NX; ++s) load_slice(s);
    }

    // (found here: behind the loop the trip for these arguments would be waited for)
    [[maybe_unused]] const uint32_t* warm_at[2] = {nullptr, nullptr};
    if constexpr (MODE == STREAM_REPAIR) {
        if (p.next.tile) {
            const StreamBlock b = stream_block(p.next, (int)blockIdx.x);
#pragma unroll
            for (int u = 0; u < 2; ++u) {
                warm_at[u] = stream_warm(p.next, b, tid + u * 512);
                asm volatile("" : "+v"(warm_at[u]));
            }
        }
    }

    f32x4_t sum[2][TW];                               // [row block of the weights][token block]
    i32x4_t isum[2][TW];
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
        for (int t = 0; t < TW; ++t) {
            sum[j][t] = f32x4_t{0, 0, 0, 0};
            isum[j][t] = i32x4_t{0, 0, 0, 0};
        }
    // fragments: lane holds 16 bytes (of token codes 8) of row lane % 16 at piece 4 quarter + lane / 16
    const uint32_t piece = (uint32_t)(frow * SL + (((4 * quarter + fp) ^ frow) & 15) * 16);
    const uint32_t w_at = (uint32_t)(wn * 2 * 16 * SL) + piece, x_at = (uint32_t)(G::kX + tw * TW * 16 * SL) + piece;
    const uint32_t q_at = (uint32_t)(G::kQ + (tw * TW * 16 + frow) * (SL / 2) + (((2 * quarter + (fp >> 1)) ^ frow) & 7) * 16 + (fp & 1) * 8);
    struct Fragments {
        td_u32x4 w[2], x[TW];
        long q[TW];
    };
    uint32_t slot_w = 0, slot_x = 0;                  // of the slice that is read next
    auto read = [&](Fragments& f) {
#pragma unroll
        for (int j = 0; j < 2; ++j) f.w[j] = *reinterpret_cast<const td_u32x4*>(lds + slot_w * G::UW + w_at + j * (16 * SL));
#pragma unroll
        for (int t = 0; t < TW; ++t) {
            if constexpr (MODE == STREAM_REPAIR) f.q[t] = *reinterpret_cast<const long*>(lds + slot_x * G::UQ + q_at + t * (16 * SL / 2));
            f.x[t] = *reinterpret_cast<const td_u32x4*>(lds + slot_x * G::UX + x_at + t * (16 * SL));
        }
    };
    auto arrived = [&](auto ahead) {                  // this wavefront's share of all but the newest `ahead` slices; the barrier makes it everybody's
        constexpr int n = decltype(ahead)::value;
        __builtin_amdgcn_s_waitcnt(0xc07f);           // lgkmcnt(0): the fragments read before are in registers
        if (weights) asm volatile("s_waitcnt vmcnt(%0)" ::"n"((NW - n) * G::LW) : "memory");
        else asm volatile("s_waitcnt vmcnt(%0)" ::"n"((NX - n) * (G::LX + G::LQ)) : "memory");
        __builtin_amdgcn_s_barrier();
        asm volatile("" ::: "memory");
    };
    float scale[2] = {0.0f, 0.0f};
    Fragments f[2];
    auto step = [&](const Fragments& now, Fragments& next) {
        // slice kt + 1 is here, and slice kt's buffers are free
        arrived(num<2>{});
        const uint32_t free_w = slot_w, free_x = slot_x;
        slot_w = slot_w + 1 == NW ? 0 : slot_w + 1;
        slot_x = slot_x + 1 == NX ? 0 : slot_x + 1;
        if (weights) load_slice(free_w);
        else load_slice(free_x);
        read(next);
        if constexpr (MODE == STREAM_REPAIR) {
#pragma unroll
            for (int j = 0; j < 2; ++j) {
                const long c = codes_of(now.w[j], scale[j]);
#pragma unroll
                for (int t = 0; t < TW; ++t) isum[j][t] = __builtin_amdgcn_mfma_i32_16x16x32_i8(c, now.q[t], isum[j][t], 0, 0, 0);
            }
        }
#pragma unroll
        for (int j = 0; j < 2; ++j)
#pragma unroll
            for (int t = 0; t < TW; ++t)
                sum[j][t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8_t, now.w[j]), __builtin_bit_cast(bf16x8_t, now.x[t]), sum[j][t], 0, 0, 0);
    };
    if (nk > 0) {
        arrived(num<1>{});
        read(f[0]);
        if constexpr (MODE == STREAM_REPAIR) {
#pragma unroll
            for (int j = 0; j < 2; ++j) scale[j] = reinterpret_cast<const float*>(lds + G::kParAt)[(wn * 2 + j) * 16 + frow];
        }
    }
#pragma unroll 1
    for (int kt = 0; kt < nk; kt += 2) {
        step(f[0], f[1]);
        if (kt + 1 < nk) step(f[1], f[0]);
    }
    float* par = reinterpret_cast<float*>(lds + G::kParAt);
    if constexpr (MODE == STREAM_REPAIR) {
        if (tid < TN) par[tid] = td_bf16_to_f32(bias);            // (in the place of the codes' scales)
    }
    asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)" ::: "memory");
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");

    [[maybe_unused]] uint32_t warm[2] = {};
    if constexpr (MODE == STREAM_REPAIR) {
#pragma unroll
        for (int u = 0; u < 2; ++u)
            if (warm_at[u]) warm[u] = *warm_at[u];
    }
    auto lds_barrier = [&]() {                        // (not __syncthreads: what was asked for above need not be here)
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
        __builtin_amdgcn_s_barrier();
        asm volatile("" ::: "memory");
    };
    // The quarters of K meet: number u = j TW + t of a wavefront's sums is finished by the quarter u / KEEP.
    // sum[j][t][q]: token lane % 16 of its block, row 4 (lane / 16) + q of the weights' block
    auto sums_of = [&](int of_wave, int u) { return lds + (of_wave * FR + u) * G::kSum + lane * 16; };
#pragma unroll
    for (int u = 0; u < FR; ++u) {
        *reinterpret_cast<f32x4_t*>(sums_of(wave, u)) = sum[u / TW][u % TW];
        if constexpr (MODE == STREAM_REPAIR) *reinterpret_cast<i32x4_t*>(sums_of(wave, u) + 1024) = isum[u / TW][u % TW];
    }
    lds_barrier();
    float* stage = reinterpret_cast<float*>(lds + G::kStage);
    auto place_of = [&](int row, int piece_of_row) { return row * TN + ((piece_of_row ^ row) & (TN / 4 - 1)) * 4; };
#pragma unroll 1                                      // (a second copy of the code costs more than the loop: it is fetched once)
    for (int k = 0; k < KEEP; ++k) {
        const int u = quarter * KEEP + k;
        if (u >= FR) break;
        f32x4_t v = {0, 0, 0, 0};
#pragma unroll
        for (int r = 0; r < 4; ++r) v += *reinterpret_cast<const f32x4_t*>(sums_of((wave & 1) + 2 * r, u));
        const int nf = wn * 2 + u / TW, nc = nf * 16 + 4 * fp, row = (tw * TW + u % TW) * 16 + frow;   // this lane's first column, row in the tile
        if constexpr (MODE == STREAM_REPAIR) {
            i32x4_t i = {0, 0, 0, 0};
#pragma unroll
            for (int r = 0; r < 4; ++r) i += *reinterpret_cast<const i32x4_t*>(sums_of((wave & 1) + 2 * r, u) + 1024);
            const f32x4_t b1 = *reinterpret_cast<const f32x4_t*>(par + nc), lo = *reinterpret_cast<const f32x4_t*>(par + 256 + nc),
                          hi = *reinterpret_cast<const f32x4_t*>(par + 512 + nc), slope = *reinterpret_cast<const f32x4_t*>(par + 768 + nc),
                          icept = *reinterpret_cast<const f32x4_t*>(par + 1024 + nc);
            const int ex = reinterpret_cast<const int*>(par)[1280 + row];
            uint32_t flags = 0u;
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const float s = ldexpf((float)i[q], ex);
                const bool inside = (s >= lo[q]) & (s < hi[q]);
                flags |= inside ? 0u : 1u << q;
            }
            flags = n0 + nc < N && row < p.M ? flags : 0u;          // (N % 8 == 0: four columns or none)
            const uint32_t word = or_halves(flags << (4 * fp));
            const int64_t n = n0 + nf * 16;
            if (fp == 0 && row < p.M && n < N) {
                uint16_t* halves = reinterpret_cast<uint16_t*>(p.mask + (size_t)row * p.mask_words) + (n >> 4);
                halves[0] = (uint16_t)word;
                if (n + 16 >= N && ((n >> 4) & 1) == 0) halves[1] = 0;     // the rest of a last word
            }
            with_act(p.act, [&](auto act) {
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    const float z = v[q] + b1[q];
                    const float d = act_flat<decltype(act)::value>(z) - fmaf(slope[q], z, icept[q]);
                    v[q] = (flags >> q) & 1u ? d : 0.0f;
                }
            });
        }
        if constexpr (MODE == STREAM_REPAIR) *reinterpret_cast<f32x4_t*>(stage + place_of(row, nc / 4)) = v;
        else if (row < p.M && n0 + nc < N) *reinterpret_cast<f32x4_t*>(p.C + ((int64_t)((int)blockIdx.x & (p.w.splits - 1)) * p.M + row) * N + n0 + nc) = v;
    }
    if constexpr (MODE == STREAM_REPAIR) {
        lds_barrier();
#pragma unroll 1
        for (int v = tid; v < TM * TN / 8; v += 512) {
            const int row = v / (TN / 8), at_row = v % (TN / 8);
            const int64_t n = n0 + at_row * 8;
            if (row >= p.M || n >= N) continue;
            const f32x4_t a[2] = {*reinterpret_cast<const f32x4_t*>(stage + place_of(row, 2 * at_row)),
                                  *reinterpret_cast<const f32x4_t*>(stage + place_of(row, 2 * at_row + 1))};
            td_u32x4 o, r;
#pragma unroll
            for (int q = 0; q < 4; ++q) o[q] = to_bf16x2(a[q >> 1][2 * (q & 1)], a[q >> 1][2 * (q & 1) + 1]);
            *reinterpret_cast<td_u32x4*>(p.out + row * N + n) = o;
            if (p.rest) {
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    float d[2] = {a[q >> 1][2 * (q & 1)] - __uint_as_float(o[q] << 16), a[q >> 1][2 * (q & 1) + 1] - __uint_as_float(o[q] & 0xffff0000u)};
#pragma unroll
                    for (int u = 0; u < 2; ++u) d[u] = fabsf(d[u]) < INFINITY ? d[u] : 0.0f;   // (infinite and NaN factors are all in the head)
                    r[q] = to_bf16x2(d[0], d[1]);
                }
                *reinterpret_cast<td_u32x4*>(p.rest + row * N + n) = r;
            }
        }
        asm volatile("" ::"v"(warm[0]), "v"(warm[1]));
    }
}

// f(token blocks, row blocks) with the constants of a tile (output products of more than 32 tokens have 64 rows a block)
template <int MODE, typename F> void for_stream_tile(bool many, bool wide, F f) {
    if (many && (wide || MODE == STREAM_PART)) f(num<4>{}, num<4>{});
    else if constexpr (MODE == STREAM_REPAIR) {
        if (many) f(num<4>{}, num<2>{});
        else if (wide) f(num<2>{}, num<4>{});
        else f(num<2>{}, num<2>{});
    } else if (wide) f(num<2>{}, num<4>{});
    else f(num<2>{}, num<2>{});
}

template <int MODE> void launch_stream(const StreamArgs& p, hipStream_t s) {
    for_stream_tile<MODE>(p.M > 32, p.w.tile == 64, [&](auto tf, auto nf) {
        typedef StreamTile<MODE, tf, nf> G;
        hipLaunchKernelGGL((stream_kernel<MODE, tf, nf>), dim3((unsigned)stream_blocks(p.w)), dim3(512), G::kLds, s, p);
    });
}

const unsigned char* bytes_of(const void* p) { return static_cast<const unsigned char*>(p); }

}  // namespace

tardis_status_t td_stream_init() {
    static td_once once;
    return once.run([]() -> tardis_status_t {
        bool ok = true;
        auto raise = [&](auto mode, auto tf, auto nf) {
            ok &= hipFuncSetAttribute(reinterpret_cast<const void*>(stream_kernel<decltype(mode)::value, decltype(tf)::value, decltype(nf)::value>),
                                      hipFuncAttributeMaxDynamicSharedMemorySize, StreamTile<decltype(mode)::value, decltype(tf)::value, decltype(nf)::value>::kLds) == hipSuccess;
        };
        for (int many = 0; many < 2; ++many)
            for (int wide = 0; wide < 2; ++wide) {
                for_stream_tile<STREAM_PART>(many, wide, [&](auto tf, auto nf) { raise(num<STREAM_PART>{}, tf, nf); });
                for_stream_tile<STREAM_REPAIR>(many, wide, [&](auto tf, auto nf) { raise(num<STREAM_REPAIR>{}, tf, nf); });
            }
        return ok ? TARDIS_OK : TARDIS_ERR_HIP;
    });
}

// Where one pass over W1 is the faster way to both products of the up product. A block is alone on its CU, so nothing hides its beginning and its
// end: rows of W1 have to be long, and one round of blocks to do. us a call with gemm_tile_kernel and Q / with this, layers in turn so that
// weights come from HBM, 20, 32, 40, 64 tokens: d = 4096, h = 10240 68 / 62, 67 / 61, 68 / 65, 73 / 69; d = 2048, h = 4096 30.5 / 28, 31 / 28.5,
// 31 / 30.5, 32 / 32, h = 8192 35 / 33, 35 / 33, 35 / 35, 37 / 37; d = 1536, h = 12288 37 / 36, 37 / 35.5, 38 / 39, 40 / 41.5; d = 1024, h =
// 12288 30 / 29, 31 / 30, 30 / 32, 32 / 34; d = 512, h = 4096 21 / 21, 21 / 22, 21 / 22, 22 / 22. Two full rounds: d = 4096, h = 32768 137 / 133,
// 132 / 131, 133 / 137, 135 / 143; d = 512, h = 32768 36 / 41, 38 / 43, 38 / 47, 39 / 49; more of them, of 32 rows: d = 4096, h = 20480 98 / 103,
// 96 / 103, 97 / 113, 103 / 120. Blocks of 32 rows that are longer than 12 KB: d = h = 6144 76 / 64, 77 / 62, 74 / 69, 80 / 76; d = h = 8192 111
// / 114, 111 / 111, 108 / 117, 112 / 118.
StreamPlan td_stream_up_plan(const tardis_layer_s* L, int64_t n) {
    StreamPlan w{};
    if (n > kStreamMaxTokens || !L->code_scale || L->d < (n <= 32 ? 1024 : 2048)) return w;
    w.B = w.B2 = bytes_of(L->W1);
    w.N = L->h;
    w.k = (uint32_t)(L->d * 2);
    w.splits = 1;
    w.slices = (int)(w.k / kStreamSlice);
    // 64 rows a block, or 32 where those leave fewer rows to the CU that has most of them
    const int64_t wide = (w.N + 63) / 64, narrow = (w.N + 31) / 32;
    if (narrow <= 256 && L->d <= 6144) w.tile = 32;
    else if (narrow > 256 && (wide <= 256 || (n <= 32 && L->d >= 3072 && wide >= 410 && wide <= 512))) w.tile = 64;
    return w;
}

// Matrices of 60 MB and more (33 tokens and more: 100) and of up to 4096 rows, where a round of blocks fills the CUs. Below that what stands
// around the stream counts for more, and gemm_tile_kernel has less of it. us with gemm_tile_kernel / this, layers in turn so that weights come
// from HBM: dense, 20, 32, 64 tokens: d = 3072, h = 6144 (38 MB) 31 / 30, 30 / 29, 33.5 / 33; d = 4096, h = 8192 (67 MB) 39 / 38, 38 / 37, 41.5 /
// 42; d = 3072, h = 12288 (75 MB) 42 / 38.5, 42 / 40, 49 / 47; d = 4096, h = 14336 (117 MB) 56.5 / 50, 57 / 51, 63 / 58; d = 4096, h = 16384 66 /
// 56.5, 66 / 57, 70 / 63. Folded, 20, 32, 40, 64 tokens: d = 2048, h = 16384 (75 MB) 47.5 / 45, 46 / 44, 47 / 45, 49.5 / 48; d = 4096, h = 10240
// (117 MB) 68 / 61.5, 67 / 59, 68 / 62, 73 / 67; d = 4096, h = 16384 82 / 77, 81 / 75, 82 / 76, 85 / 80. CUs without a block, three quarters
// filled: d = 3072, h = 12288 (94 MB) 56 / 53, 55 / 52, 57 / 54, 62 / 60; h = 24576 87 / 86, 85 / 86, 88 / 86, 96 / 95; h = 31104 134 / 140, 133
// / 145, 137 / 145, 146 / 160; nine sixteenths: d = 2304, h = 13824 66 / 68, 67 / 67, 68 / 71, 73 / 78. More rows: d = 5120, h = 13696 119 / 126,
// 120 / 127, 124 / 135, 137 / 150; d = h = 8192 111 / 124, 111 / 120, 108 / 119, 112 / 126. Fewer, with many tokens: d = 1920, h = 16384, 40, 64
// tokens 65 / 68, 67 / 70. (The loads pass the last cache by. A layer that is called again and again, with nothing between that takes its place
// there, loses by that: d = 4096, h = 8192, dense, 20, 32 tokens 33 / 36, 33.5 / 37; d = 4096, h = 16384, 20, 32, 40, 64 tokens 72.5 / 73, 72 /
// 72, 72 / 76, 74 / 78.)
StreamPlan td_stream_output_plan(bool folded, const void* Wp, const void* W2, int64_t n, int64_t d, int64_t h) {
    StreamPlan w{};
    const int64_t bytes = d * (h + (folded ? d : 0)) * 2;
    if (n > kStreamMaxTokens || d % 128 != 0 || h % 128 != 0 || d > 4096 || bytes < 60000000) return w;
    if (n > 32 && (d < 2048 || bytes < 100000000)) return w;
    w.B = bytes_of(folded ? Wp : W2);
    w.B2 = bytes_of(W2);
    w.N = d;
    w.k = (uint32_t)((folded ? d : h) * 2);
    w.k2 = folded ? (uint32_t)(h * 2) : 0u;
    const int slices = (int)((w.k + w.k2) / kStreamSlice);
    // the tile and the number of ranges with the least time: rounds over 256 CUs x (slices at the rate of HBM per CU + a launch's
    // beginning and end), and the partial sums written and read again
    double best = 1e300;
    int64_t launched = 0;
    for (int tile = 64; tile >= (n > 32 ? 64 : 32); tile /= 2)
        for (int sp = 1; sp <= 8 && (sp == 1 || slices / sp >= 4); sp *= 2) {
            const int64_t blocks = (w.N + tile - 1) / tile * sp;
            const double per = (double)((slices + sp - 1) / sp) * (double)(tile + (n > 32 ? 16 : 8)) * 256.0 / 24e3;
            const double cost = (double)((blocks + 255) / 256) * (per + 3.0) + (double)(sp * n * d) * 8.0 / 4e6;
            if (cost < best) { best = cost; w.tile = tile; w.splits = sp; launched = blocks; }
        }
    const bool few = n <= 32 && bytes <= 160000000;
    if (launched > 256 || launched < (few ? 192 : 205)) w.tile = 0;      // (three quarters, four fifths of the CUs)
    w.slices = (slices + w.splits - 1) / w.splits;
    return w;
}

// as td_gemm_repair; plan: td_stream_up_plan's, next: of the launch that follows
tardis_status_t td_stream_repair(const tardis_layer_s* L, const StreamPlan& plan, const int8_t* XQ, const int32_t* e, const void* X,
                                 const void* b1, uint32_t* mask, void* out, void* rest, int64_t n, const StreamPlan& next, hipStream_t s) {
    StreamArgs p{};
    p.w = plan;
    p.next = next;
    p.A = p.A2 = bytes_of(X);
    p.XQ = bytes_of(XQ);
    p.M = n;
    p.bias = static_cast<const bf16_t*>(b1);
    p.codes = L->code_scale;
    p.lo = L->tlo;
    p.hi = L->thi;
    p.slope = L->a;
    p.icept = L->c;
    p.e = e;
    p.mask = mask;
    p.mask_words = (int)L->mask_words;
    p.out = static_cast<bf16_t*>(out);
    p.rest = static_cast<bf16_t*>(rest);
    p.act = L->act;
    launch_stream<STREAM_REPAIR>(p, s);
    TD_HIP(hipGetLastError());
    return TARDIS_OK;
}

// as td_gemm_output; plan: td_stream_output_plan's
tardis_status_t td_stream_output(const StreamPlan& plan, const void* X, const void* H, float* part, int* parts, int64_t n, hipStream_t s) {
    StreamArgs p{};
    p.w = plan;
    p.A = bytes_of(X ? X : H);
    p.A2 = bytes_of(H);
    p.M = n;
    p.C = part;
    launch_stream<STREAM_PART>(p, s);
    *parts = plan.splits;
    TD_HIP(hipGetLastError());
    return TARDIS_OK;
}

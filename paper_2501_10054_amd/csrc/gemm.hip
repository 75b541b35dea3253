// C[m][n] = sum_k A[m][k] * B[n][k]  -- both operands K-contiguous ("NT"); bf16 or fp32 operands and
// fp32 sums, or int8 operands and exact int32 sums, which only feed the range test and are not stored.
//
// Used offline: the fold  W' = W2 . (diag(a) W1)  (Sec. "Constant Folded Matrix
// Generation") with A = W2 (d x h) and B = (diag(a) W1)^T (d x h), and the
// calibration pre-activations Z^T = W1 . X_cal^T (Sec. "Non-linear Function
// Approximation", step 2) with A = W1 (h x d) and B = X_cal (n x d).  Used online for calls with
// many tokens (prompts), where every step of the method is a product of the token matrix with a
// weight matrix: predictor sums Xq . Q^T (int8) and their range test, pre-activations X . W1^T and the
// repair factors of the flagged ones, and the folded product together with the down projection of the
// masked factors, [X | D] . [W' | W2]^T.
#include <cstdlib>

#include "common.h"
#include "sigma.h"
#include "slices.h"
#include "tiles.h"

namespace {

// ------------------------------------------------------------------ any shape
// 64x64 output tile, 16-deep K slices through LDS, 4x4 outputs per thread.
// Works for any M, N, K and for fp32 or bf16 operands (fp32 arithmetic).
constexpr int GT = 64, GK = 16;

template <typename T>
__global__ void __launch_bounds__(256)
gemm_nt_generic_kernel(const T* __restrict__ A, const T* __restrict__ B, float* __restrict__ C, int64_t M,
                       int64_t N, int64_t K, int accumulate, const T* __restrict__ row_bias) {
    __shared__ float As[GK][GT + 4];
    __shared__ float Bs[GK][GT + 4];
    const int tid = threadIdx.x;
    const int64_t m0 = (int64_t)blockIdx.y * GT, n0 = (int64_t)blockIdx.x * GT;
    const int tx = tid % 16, ty = tid / 16;
    float acc[4][4];
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int j = 0; j < 4; ++j) acc[i][j] = 0.0f;

    // each thread stages 4 consecutive k of one row of A and of B per slice
    const int lr = tid / 4, lk = (tid % 4) * 4;
    for (int64_t k0 = 0; k0 < K; k0 += GK) {
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const int64_t k = k0 + lk + u;
            const int64_t am = m0 + lr, bn = n0 + lr;
            As[lk + u][lr] = (am < M && k < K) ? td_load<T>(A + am * K + k) : 0.0f;
            Bs[lk + u][lr] = (bn < N && k < K) ? td_load<T>(B + bn * K + k) : 0.0f;
        }
        __syncthreads();
#pragma unroll
        for (int kk = 0; kk < GK; ++kk) {
            float av[4], bv[4];
#pragma unroll
            for (int i = 0; i < 4; ++i) av[i] = As[kk][ty * 4 + i];
#pragma unroll
            for (int j = 0; j < 4; ++j) bv[j] = Bs[kk][tx * 4 + j];
#pragma unroll
            for (int i = 0; i < 4; ++i)
#pragma unroll
                for (int j = 0; j < 4; ++j) acc[i][j] = fmaf(av[i], bv[j], acc[i][j]);
        }
        __syncthreads();
    }
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const int64_t m = m0 + ty * 4 + i;
        if (m >= M) continue;
        const float rb = row_bias ? td_load<T>(row_bias + m) : 0.0f;
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const int64_t n = n0 + tx * 4 + j;
            if (n >= N) continue;
            float v = acc[i][j] + rb;
            if (accumulate) v += C[m * N + n];
            C[m * N + n] = v;
        }
    }
}


// ------------------------------------------------------------------ MFMA (bf16 or int8)
// Two kernels for the products on the matrix cores, with the step that follows the product in their
// epilogue (finish_tile): gemm_tile_kernel, 8 wavefronts in a WM x (8/WM) grid, each NA x NB tiles of
// v_mfma_f32_16x16x32_bf16 / v_mfma_i32_16x16x64_i8 (the byte geometry of the two is the same: 16 bytes per lane
// and MFMA), so an output tile of (WM*NA*16) x ((8/WM)*NB*16); and gemm_quad_kernel, 4 wavefronts in a 2 x 2 grid, for
// large tiles.  K runs in slices of 128 bytes per row (256 for few rows).
//
// What bounds it.  With real (not constant) data the chip is power limited: the clock settles where the
// energy per MFMA and per moved byte allows (a loop of nothing but 16x16x32 MFMAs on random data runs at
// 1.95-2.0 PFLOP/s, of 32x32x16 ones at 1.75; with zeros 2.4), and every stall raises the clock it would
// need.  Hence:
//  * 16x16 MFMAs;
//  * slices go from memory straight to LDS (buffer_load ... lds): no staging registers and no LDS writes by
//    the wavefronts.  A load instruction covers 8 rows x 128 bytes; half lines (64 bytes per row) fetch
//    every line twice from L2 (0.94 against 1.13 PFLOP/s);
//  * a lane asks for the 16-byte piece (slot ^ row) of its row, so that the fragment reads below (16 rows,
//    same piece) hit all banks: no padding, no conflicts;
//  * A has SA and B has SB slice buffers, together up to 160 KB.  The loads that refill the buffers of
//    slice kt are issued, between MFMAs, right after the barrier behind which nobody reads them any more,
//    and are waited for SB-1 / SA-1 slices later (never for the newest ones);
//  * fragments of the next half slice are read while the MFMAs of this one run.  The MFMAs are inline
//    assembly because the compiler, given the builtins, moves accumulators between the two register files;
//  * blocks start at different slices (rotated within a window of 8 between the blocks of an XCD, which
//    share lines in its L2, and by an eighth of K from XCD to XCD): with all of them at the same column of
//    K the requests crowd onto few memory channels (zeros: 358 -> 300 us at 4096 x 4096 x 16384).
// 4096 x 4096 x 16384 in bf16 with random data (tile 256 x 256, kernel trace): 404 us with eight wavefronts, 375 with four (360 to
// 390 from card to card), 1.47 PFLOP/s; with staging through registers 605, 0.91.

constexpr int kWavesPerTile = 8;
constexpr int kNoLds = 0xc07f, kNoLoads = 0x0f70;            // s_waitcnt lgkmcnt(0), vmcnt(0)

// Which block computes which tile.  Blocks b, b+8, b+16, ... run on one XCD and share its L2, so
// each XCD gets a rectangle of rm x rn tiles (the 8 XCDs form a gm x gn grid over the tile grid,
// times `splits` ranges of K), and inside the rectangle consecutive blocks walk `group` tile rows
// column by column: the 32 blocks an XCD runs at once then cover a compact patch and re-use each
// other's slices of A and B from L2 instead of fetching them from HBM again.
struct TileMap {
    int tiles_m, tiles_n;      // tile grid of C
    int splits_log2;           // K ranges (1, 2, 4 or 8)
    int gn_log2;               // XCD grid columns (rows = 8 / splits / gn)
    int rm, rn;                // tiles per XCD rectangle
    int group;                 // tile rows walked together (fewer in the last group)
    uint32_t inv_walk, inv_group, inv_last;   // reciprocals (see quotient) of group x rn, of group, of the last group's rows
    int slices;                // K slices per range
};

// n / d, with inv = 2^32 / d rounded down: scalar multiplications (the compiler divides on the vector unit, and a block's
// six divisions one after another are most of a microsecond)
uint32_t reciprocal(uint32_t d) { return d > 1 ? (uint32_t)(0x100000000ull / d) : 0xffffffffu; }
__device__ __forceinline__ uint32_t quotient(uint32_t n, uint32_t d, uint32_t inv, uint32_t& rest) {
    uint32_t q = __umulhi(n, inv);                          // the quotient, or one less
    rest = n - q * d;
    if (rest >= d) {
        ++q;
        rest -= d;
    }
    return q;
}

TileMap make_tile_map(int64_t M, int64_t N, int tile_m, int tile_n, int slices, int splits) {
    TileMap t;
    t.tiles_m = (int)((M + tile_m - 1) / tile_m);
    t.tiles_n = (int)((N + tile_n - 1) / tile_n);
    t.splits_log2 = __builtin_ctz((unsigned)splits);
    const int nx = 8 / splits;
    int best = 1 << 30, gm = nx;
    for (int cand = 1; cand <= nx; cand *= 2) {            // cand = XCD grid rows
        const int rm = (t.tiles_m + cand - 1) / cand, rn = (t.tiles_n + nx / cand - 1) / (nx / cand);
        const int cost = rm * rn * 4096 + rm * tile_m + rn * tile_n;   // fewest blocks, then least operand bytes
        if (cost < best) { best = cost; gm = cand; }
    }
    const int gn = nx / gm;
    t.gn_log2 = __builtin_ctz((unsigned)gn);
    t.rm = (t.tiles_m + gm - 1) / gm;
    t.rn = (t.tiles_n + gn - 1) / gn;
    t.group = t.rm < 8 ? t.rm : 8;
    t.inv_walk = reciprocal((uint32_t)(t.group * t.rn));
    t.inv_group = reciprocal((uint32_t)t.group);
    t.inv_last = reciprocal((uint32_t)(t.rm - (t.rm - 1) / t.group * t.group));
    t.slices = (slices + splits - 1) / splits;
    return t;
}

// This block's tile and K range; false: none
__device__ __forceinline__ bool place(const TileMap& t, int xcd, int local, int& tile_m, int& tile_n, int& range) {
    range = xcd & ((1 << t.splits_log2) - 1);
    const int xg = xcd >> t.splits_log2;
    uint32_t r, row;
    const int first = (int)quotient((uint32_t)local, (uint32_t)(t.group * t.rn), t.inv_walk, r) * t.group;
    const int rows = min(t.group, t.rm - first);
    const int col = (int)quotient(r, (uint32_t)rows, rows == t.group ? t.inv_group : t.inv_last, row);
    tile_m = (xg >> t.gn_log2) * t.rm + first + (int)row;
    tile_n = (xg & ((1 << t.gn_log2) - 1)) * t.rn + col;
    return tile_m < t.tiles_m && tile_n < t.tiles_n;
}

// C = A.B^T (+ A2.B2^T: a second pair of operands whose K follows the first's).  Rows of A are rows of
// C (M of them), rows of B columns of C (N); k, k2: bytes of a row of the first / second pair.
struct GemmArgs {
    const unsigned char *A, *B, *A2, *B2;
    int64_t M, N;
    uint32_t k, k2;
    // epilogues
    float* C;                      // F32: M x N; PART: [split][M][N]
    int accumulate;                // F32: add to C
    const bf16_t* bias;            // F32: per row of C (or null); HIDDEN, REPAIR: per column
    bf16_t* out;                   // HIDDEN, REPAIR: M x N; F32, accumulate: the sum goes here, rounded, and C stays (or null)
    bf16_t* rest;                  // REPAIR: what the rounding of `out` to bf16 left, M x N (or null)
    const float *lo, *hi;          // REPAIR: bounds of the range test per column,
    const float *slope, *icept;    //   line per column,
    const int32_t* e;              //   exponent per row (readable to the next multiple of 16 bytes),
    uint32_t* mask;                //   flags, M x mask_words, written
    int mask_words;
    int act;
};

// F32: C = product (+ bias), or C += product.  PART: one range of K's share of C.  HIDDEN: out = sigma(product + bias).
// REPAIR: the first pair of operands is int8 (token codes and predictor codes), the second bf16 (tokens and
// W1): the sums of the first give the flags, those of the second z, and out = sigma(z) - (slope z + icept) at
// the flagged places, 0 elsewhere (with `rest`: as bf16 head and bf16 remainder, 16 significant bits together).  Neither
// the sums nor z leave the block, and the stream of slices goes on from the one product to the other.
enum { EPI_F32, EPI_PART, EPI_HIDDEN, EPI_REPAIR };

// (the accumulator of the int8 form holds integers)
template <bool I8> __device__ __forceinline__ void mma16(f32x4_t& c, const td_u32x4& a, const td_u32x4& b) {
    if constexpr (I8) asm volatile("v_mfma_i32_16x16x64_i8 %0, %1, %2, %0" : "+v"(c) : "v"(a), "v"(b));
    else asm volatile("v_mfma_f32_16x16x32_bf16 %0, %1, %2, %0" : "+v"(c) : "v"(a), "v"(b));
}

// The compiler does not know how long those take.  Every use of the accumulators from here on (of their new values, for
// the compiler) comes behind the statements before this, a wait among them, and every definition before it: without it
// plain arithmetic on them may be moved in front of the wait.
template <int NA, int NB> __device__ __forceinline__ void fence(f32x4_t (&acc)[NA][NB]) {
#pragma unroll
    for (int i = 0; i < NA; ++i)
#pragma unroll
        for (int j = 0; j < NB; ++j) asm volatile("" : "+v"(acc[i][j])::"memory");
    __builtin_amdgcn_sched_barrier(0);
}

// Row blocks (of 16 rows) that a wavefront stages in LDS at a time: as many as fit (beside REPAIR's three parameters per column)
template <int EPI, int W, int WM, int NA, int NB> struct EpiRows {
    static constexpr int kParams = EPI == EPI_REPAIR ? 3 * (W / WM) * NB * 16 * 4 : 0;
    static constexpr int fit(int n) { return n == 1 || (NA % n == 0 && W * n * 16 * NB * 16 * 4 + kParams <= kLdsBytes) ? n : fit(n - 1); }
    static constexpr int value = fit(NA);
    static constexpr int kWaveBytes = value * 16 * NB * 16 * 4, kBytes = W * kWaveBytes + kParams;
};

// RAGGED: a row is not a whole number of slices; the pieces past its end are loaded from the row's last
// slice start instead (in bounds) and the fragments that hold them are zeroed as they are read.
template <int EPI, bool RAGGED, int SL, int WM, int NA, int NB>
struct GemmTile {
    static constexpr int WN = kWavesPerTile / WM;
    static constexpr int TM = WM * NA * 16, TN = WN * NB * 16;
    static constexpr int UA = TM * SL, UB = TN * SL;      // bytes of one slice
    // one row of tiles: a row of B is read by one block, so its lines are not kept (64 tokens: 40.6 -> 38.8 us; the
    // output product, whose blocks share lines between K ranges, loses by it: 31.7 -> 35.5 us)
    static constexpr bool kOnce = TM == 64 && EPI == EPI_REPAIR;
    static constexpr int LA = UA / 8192, LB = UB / 8192;                        // loads per wavefront and slice
    // REPAIR: bounds and exponents wait in LDS for the range test
    static constexpr int kPar = EPI == EPI_REPAIR ? 3 * 1024 : 0;
    // as many slices as fit; A one ahead of B where the two do not fit equally often
    static constexpr int kRoom = kLdsBytes - kPar;
    static constexpr int SB = kRoom / (UA + UB) > 10 ? 10 : kRoom / (UA + UB);
    static constexpr int SA = SB < 10 && SB * (UA + UB) + UA <= kRoom ? SB + 1 : SB;
    static constexpr int kRing = SA * UA + SB * UB;
    static constexpr int kPer = LA + LB;
    // loads that may still be in flight when slice kt+2 has to be there (see the order in the kernel)
    static constexpr int kWaitB = LA + (SB - 2) * kPer, kWaitA = (SA - 2) * kPer;
    static constexpr int kWait = kWaitB < kWaitA ? kWaitB : kWaitA;
    static constexpr int kEpiLds = EpiRows<EPI, kWavesPerTile, WM, NA, NB>::kBytes;
    static constexpr int kLds = kRing + kPar > kEpiLds ? kRing + kPar : kEpiLds;
    static_assert(SL % 128 == 0 && UA % 8192 == 0 && UB % 8192 == 0, "whole loads of 1 KB for 8 wavefronts");
    static_assert(TM <= 256 && TN <= 256, "a load of 1 KB for each parameter");
    static_assert(SB >= 2 && SA >= 2 && kWait + kPer <= 63 && kLds <= kLdsBytes, "slice buffers");
};

// What follows the products, W wavefronts in a grid of WM rows.  Some row blocks at a time go through LDS, so that a store covers
// whole lines of a row, and so that what is done to the elements is a loop: unrolled over the accumulators, sigma alone is
// 100 to 200 KB of instructions, which every block fetches once (2048 x 16384 x 4096 with GELU, eight wavefronts: sigma as a loop and without branches 251 -> 228 us).
// REPAIR: the flagged pre-activations are staged, zeros elsewhere, and every lane replaces its own by their factors, as many
// times as the lane with the most of them has any (5 %: about 14 times for 128 elements a lane).
template <int EPI, int W, int WM, int NA, int NB>
__device__ __forceinline__ void finish_tile(const GemmArgs& p, f32x4_t (&acc)[NA][NB], const uint32_t (&bits)[NA], unsigned char* lds,
                                            int tid, int64_t m0, int64_t n0, int ks) {
    typedef EpiRows<EPI, W, WM, NA, NB> E;
    constexpr int WN = W / WM, TN = WN * NB * 16, RB = E::value, CW = NB * 16, PC = CW / 4;
    const int lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6), wm = wave / WN, wn = wave % WN;
    const int frow = lane & 15, fp = lane >> 4;
    // acc[i][j][q] = C[row m0 + (wm*NA + i)*16 + lane%16][column n0 + (wn*NB + j)*16 + 4*(lane/16) + q]
    const int64_t mw = m0 + wm * NA * 16, nw = n0 + wn * CW;         // this wavefront's corner, CW columns
    float* chunk = reinterpret_cast<float*>(lds + wave * E::kWaveBytes);
    [[maybe_unused]] float* par = reinterpret_cast<float*>(lds + W * E::kWaveBytes);
    if constexpr (EPI == EPI_REPAIR) {
        for (int c = tid; c < TN; c += W * 64) {
            const int64_t n = n0 + c < p.N ? n0 + c : p.N - 1;
            par[c] = td_bf16_to_f32(p.bias[n]);
            par[TN + c] = p.slope[n];
            par[2 * TN + c] = p.icept[n];
        }
        __syncthreads();
    }
    // (pieces of 16 bytes, rotated by the row, against bank conflicts)
    auto place_of = [&](int row, int piece) { return row * CW + ((piece ^ (row & 15 & (PC - 1))) * 4); };
    auto piece_of = [&](int row, int piece) { return *reinterpret_cast<const f32x4_t*>(chunk + place_of(row, piece)); };
    for_constants<NA / RB>([&](auto batch) {
        constexpr int first = decltype(batch)::value * RB;
        const int64_t m1 = mw + first * 16;
        for_constants<RB>([&](auto row_block) {
            constexpr int u = decltype(row_block)::value, i = first + u;
            if constexpr (EPI == EPI_REPAIR) {
                // mask: the four lanes of a row and (where the tile holds them) two tile columns make a word of 32 bits
                const int64_t m = mw + i * 16 + frow;
#pragma unroll
                for (int w = 0; w < (NB + 1) / 2; ++w) {
                    uint32_t word = ((bits[i] >> (8 * w)) & 15u) << (4 * fp);
                    if constexpr (NB >= 2) word |= ((bits[i] >> (8 * w + 4)) & 15u) << (4 * fp + 16);
                    word = or_halves(word);
                    const int64_t n = nw + w * 32;
                    if (fp == 0 && m < p.M && n < p.N) {
                        uint32_t* row = p.mask + (size_t)m * p.mask_words;
                        if constexpr (NB >= 2) {
                            row[n >> 5] = word;
                        } else {
                            uint16_t* half = reinterpret_cast<uint16_t*>(row) + (n >> 4);
                            half[0] = (uint16_t)word;
                            if (n + 16 >= p.N && ((n >> 4) & 1) == 0) half[1] = 0;   // the rest of a last word
                        }
                    }
                }
            }
            float rb = 0.0f;
            if constexpr (EPI == EPI_F32) {
                const int64_t m = mw + i * 16 + frow;
                if (p.bias && m < p.M) rb = td_bf16_to_f32(p.bias[m]);
            }
#pragma unroll
            for (int j = 0; j < NB; ++j) {
                f32x4_t v;
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    if constexpr (EPI == EPI_REPAIR) v[q] = (bits[i] >> (4 * j + q)) & 1u ? acc[i][j][q] : 0.0f;
                    else v[q] = acc[i][j][q] + rb;
                }
                *reinterpret_cast<f32x4_t*>(chunk + place_of(u * 16 + frow, j * 4 + fp)) = v;
            }
        });
        __builtin_amdgcn_wave_barrier();
        if constexpr (EPI == EPI_REPAIR) {
            // flags of this lane's RB x 4 NB elements, lowest first
            static_assert(RB * 4 * NB <= 128, "two words of flags");
            uint64_t now = 0, later = 0;
            for_constants<RB>([&](auto row_block) {
                constexpr int at = decltype(row_block)::value * 4 * NB;
                if constexpr (at < 64) now |= (uint64_t)bits[first + decltype(row_block)::value] << at;
                else later |= (uint64_t)bits[first + decltype(row_block)::value] << (at - 64);
            });
            with_act(p.act, [&](auto act) {
                int row0 = frow;
                while (__any((now | later) != 0)) {
                    if (now == 0) {
                        now = later;
                        later = 0;
                        row0 = 64 / (4 * NB) * 16 + frow;
                    }
                    if (now != 0) {
                        const int e = __builtin_ctzll(now), piece = (e / 4 % NB) * 4 + fp;
                        now &= now - 1;
                        float* z = chunk + place_of(row0 + e / (4 * NB) * 16, piece) + e % 4;
                        const int c = wn * CW + piece * 4 + e % 4;
                        const float v = *z + par[c];
                        *z = act_flat<decltype(act)::value>(v) - fmaf(par[TN + c], v, par[2 * TN + c]);
                    }
                }
            });
            __builtin_amdgcn_wave_barrier();
        }
        if constexpr (EPI == EPI_HIDDEN || EPI == EPI_REPAIR) {      // N % 8 == 0: whole 16-byte vectors
            constexpr int RPS = 64 / (CW / 8);                       // rows at a time
            const int64_t nn = nw + lane % (CW / 8) * 8;
            auto rows = [&](auto store) {
#pragma unroll 2
                for (int row = lane / (CW / 8); row < RB * 16; row += RPS) {
                    const f32x4_t v[2] = {piece_of(row, lane % (CW / 8) * 2), piece_of(row, lane % (CW / 8) * 2 + 1)};
                    store(v, m1 + row < p.M && nn < p.N, (m1 + row) * p.N + nn);
                }
            };
            if constexpr (EPI == EPI_HIDDEN) {
                float bias[8];
#pragma unroll
                for (int q = 0; q < 8; ++q) bias[q] = nn < p.N ? td_bf16_to_f32(p.bias[nn + q]) : 0.0f;
                with_act(p.act, [&](auto act) {
                    rows([&](const f32x4_t (&v)[2], bool in, int64_t at) {
                        float s[8];
#pragma unroll
                        for (int q = 0; q < 8; ++q) s[q] = act_flat<decltype(act)::value>(v[q >> 2][q & 3] + bias[q]);
                        td_u32x4 o;
#pragma unroll
                        for (int q = 0; q < 4; ++q) o[q] = to_bf16x2(s[2 * q], s[2 * q + 1]);
                        if (in) *reinterpret_cast<td_u32x4*>(p.out + at) = o;
                    });
                });
            } else {
                rows([&](const f32x4_t (&v)[2], bool in, int64_t at) {
                    td_u32x4 o;
#pragma unroll
                    for (int q = 0; q < 4; ++q) o[q] = to_bf16x2(v[q >> 1][2 * (q & 1)], v[q >> 1][2 * (q & 1) + 1]);
                    if (in) *reinterpret_cast<td_u32x4*>(p.out + at) = o;
                    if (p.rest) {
#pragma unroll
                        for (int q = 0; q < 4; ++q) {
                            float rest[2] = {v[q >> 1][2 * (q & 1)] - __uint_as_float(o[q] << 16),
                                             v[q >> 1][2 * (q & 1) + 1] - __uint_as_float(o[q] & 0xffff0000u)};
#pragma unroll
                            for (int u = 0; u < 2; ++u) rest[u] = fabsf(rest[u]) < INFINITY ? rest[u] : 0.0f;   // (infinite and NaN factors are all in the head)
                            o[q] = to_bf16x2(rest[0], rest[1]);
                        }
                        if (in) *reinterpret_cast<td_u32x4*>(p.rest + at) = o;
                    }
                });
            }
        } else {
            float* C = EPI == EPI_PART ? p.C + (size_t)ks * p.M * p.N : p.C;
            const bool add = EPI == EPI_F32 && p.accumulate;
            bf16_t* rounded = add ? p.out : nullptr;
            if (p.N % 4 == 0) {                                  // (C is 16-byte aligned)
                constexpr int RPS = 64 / PC, S = RB * 16 / RPS, U = S % 8 == 0 ? 8 : S % 4 == 0 ? 4 : S % 2 == 0 ? 2 : 1;   // rows at a time; times
                static_assert(RB * 16 % (RPS * U) == 0, "whole steps");
                const int row0 = lane / PC, piece = lane % PC;
                const bool whole = m1 + RB * 16 <= p.M;          // (uniform)
                float* at = C + (m1 + row0) * p.N + nw + piece * 4;
                if (nw + piece * 4 < p.N) {
#pragma unroll 1
                    for (int row = row0; row < RB * 16; row += RPS * U, at += RPS * U * p.N) {
                        f32x4_t v[U];
#pragma unroll
                        for (int u = 0; u < U; ++u) v[u] = piece_of(row + u * RPS, piece);
                        if (add) {
                            f32x4_t old[U];
#pragma unroll
                            for (int u = 0; u < U; ++u)
                                if (whole || m1 + row + u * RPS < p.M) old[u] = *reinterpret_cast<const f32x4_t*>(at + u * RPS * p.N);
#pragma unroll
                            for (int u = 0; u < U; ++u)
#pragma unroll
                                for (int q = 0; q < 4; ++q) v[u][q] = old[u][q] + v[u][q];
                        }
#pragma unroll
                        for (int u = 0; u < U; ++u)
                            if (whole || m1 + row + u * RPS < p.M) {
                                if (rounded) *reinterpret_cast<uint2*>(rounded + (at - C) + u * RPS * p.N) = make_uint2(to_bf16x2(v[u][0], v[u][1]), to_bf16x2(v[u][2], v[u][3]));
                                else *reinterpret_cast<f32x4_t*>(at + u * RPS * p.N) = v[u];
                            }
                    }
                }
            } else {
#pragma unroll 1
                for (int t = lane; t < RB * 16 * CW; t += 64) {
                    const int row = t / CW, col = t % CW;
                    const float v = piece_of(row, col >> 2)[col & 3];
                    const int64_t mm = m1 + row, nn = nw + col;
                    if (mm >= p.M || nn >= p.N) continue;
                    const float sum = add ? C[mm * p.N + nn] + v : v;
                    if (rounded) rounded[mm * p.N + nn] = (bf16_t)to_bf16x2(sum, 0.0f);
                    else C[mm * p.N + nn] = sum;
                }
            }
        }
        __builtin_amdgcn_wave_barrier();
    });
}

template <int EPI, bool RAGGED, int SL, int WM, int NA, int NB>
__global__ void __launch_bounds__(512) gemm_tile_kernel(GemmArgs p, TileMap tm) {
    typedef GemmTile<EPI, RAGGED, SL, WM, NA, NB> G;
    constexpr int WN = G::WN, TM = G::TM, TN = G::TN, SA = G::SA, SB = G::SB, LA = G::LA, LB = G::LB;
    extern __shared__ __align__(1024) unsigned char lds[];
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm = wave / WN, wn = wave % WN;

    const int xcd = (int)blockIdx.x & 7, local = (int)blockIdx.x >> 3;
    int tile_m, tile_n, ks;
    if (!place(tm, xcd, local, tile_m, tile_n, ks)) return;
    const int64_t m0 = (int64_t)tile_m * TM, n0 = (int64_t)tile_n * TN;

    // slices [s0, s0 + nk) of this block's range, from a starting point of its own (REPAIR: of either product)
    const int nk1 = (int)((p.k + SL - 1) / SL), nk2 = (int)((p.k2 + SL - 1) / SL);
    const int s0 = ks * tm.slices;
    const int nk = max(0, min(tm.slices, nk1 + nk2 - s0));
    const int rot = first_slice(xcd, local, EPI == EPI_REPAIR ? nk1 : nk), rot2 = EPI == EPI_REPAIR ? first_slice(xcd, local, nk2) : 0;
    auto slice_of = [&](int kt) {
        if constexpr (EPI == EPI_REPAIR) {
            const bool second = kt >= nk1;
            const int s = second ? kt + rot2 : kt + rot;
            return s - (second ? (s >= nk1 + nk2 ? nk2 : 0) : (s >= nk1 ? nk1 : 0));
        }
        const int s = kt + rot;
        return s0 + (s >= nk ? s - nk : s);
    };

    const uint32_t rows_a = (uint32_t)min((int64_t)TM, p.M - m0), rows_b = (uint32_t)min((int64_t)TN, p.N - n0);
    const i32x4_t ra1 = buffer_of(p.A + (size_t)m0 * p.k, rows_a * p.k), rb1 = buffer_of(p.B + (size_t)n0 * p.k, rows_b * p.k);
    const i32x4_t ra2 = buffer_of(p.A2 + (size_t)m0 * p.k2, rows_a * p.k2), rb2 = buffer_of(p.B2 + (size_t)n0 * p.k2, rows_b * p.k2);

    // a load is 1024 / SL rows, lane -> row lane / (pieces of a row), slot lane % (pieces of a row); wavefront w
    // loads rows [w*TM/8, (w+1)*TM/8) of A, of B alike
    constexpr int PS = SL / 16, RPL = 1024 / SL, SWZ = PS < 16 ? PS - 1 : 15;
    const int lrow = lane / PS, lslot = lane % PS;
    uint32_t lds_a, lds_b;
    {
        const uint32_t base = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) unsigned char*)lds;
        lds_a = __builtin_amdgcn_readfirstlane(base + wave * (G::UA / kWavesPerTile));
        lds_b = __builtin_amdgcn_readfirstlane(base + SA * G::UA + wave * (G::UB / kWavesPerTile));
    }
    const uint32_t row_a = (uint32_t)(wave * (TM / 8) + lrow), row_b = (uint32_t)(wave * (TN / 8) + lrow);
    struct Source {                                   // one operand's slice (uniform)
        i32x4_t rs;
        uint32_t soff, pitch;
    };
    auto source = [&](bool is_a, int kt) {
        const bool live = kt < nk;                                  // past the last slice: an empty buffer
        const int s = live ? slice_of(kt) : 0;
        const bool second = s >= nk1;
        Source o;
        const i32x4_t r1 = is_a ? ra1 : rb1, r2 = is_a ? ra2 : rb2;
        o.rs.x = second ? r2.x : r1.x;
        o.rs.y = second ? r2.y : r1.y;
        o.rs.z = live ? (second ? r2.z : r1.z) : 0;
        o.rs.w = r1.w;
        o.soff = (uint32_t)(second ? s - nk1 : s) * SL;
        o.pitch = second ? p.k2 : p.k;
        return o;
    };
    auto load_one = [&](bool is_a, int i, uint32_t buf, const Source& o) {
        const uint32_t row = (is_a ? row_a : row_b) + (uint32_t)(RPL * i);
        uint32_t pc = ((uint32_t)lslot ^ (row & SWZ)) * 16u;
        if constexpr (RAGGED) pc = o.soff + pc < o.pitch ? pc : 0u;
        const uint32_t voff = row * o.pitch + pc;
        if (is_a) load_to_lds(lds_a + buf * G::UA + i * 1024u, voff, o.rs, o.soff);
        else load_to_lds<G::kOnce>(lds_b + buf * G::UB + i * 1024u, voff, o.rs, o.soff);
    };

    f32x4_t acc[NA][NB];
#pragma unroll
    for (int i = 0; i < NA; ++i)
#pragma unroll
        for (int j = 0; j < NB; ++j)
#pragma unroll
            for (int q = 0; q < 4; ++q) acc[i][j][q] = 0;

    // fragments: lane holds 16 bytes of row lane%16 at piece 4*step + lane/16
    constexpr int KS = SL / 64;                       // steps (MFMA depths) of a slice
    const int frow = lane & 15, fp = lane >> 4;
    uint32_t fsw[KS];
#pragma unroll
    for (int s = 0; s < KS; ++s) fsw[s] = (uint32_t)(frow * SL + (((s * 4 + fp) ^ (frow & SWZ)) * 16));
    td_u32x4 fa[2][NA], fb[2][NB];
    auto read_one = [&](int buf, int t, uint32_t ba, uint32_t bb, int s, int slice) {   // fa[0], all of fb, the rest of fa
        td_u32x4 v;
        if (t == 0 || t > NB)
            v = *reinterpret_cast<const td_u32x4*>(lds + ba * G::UA + (wm * NA + (t == 0 ? 0 : t - NB)) * (16 * SL) + fsw[s]);
        else
            v = *reinterpret_cast<const td_u32x4*>(lds + SA * G::UA + bb * G::UB + (wn * NB + t - 1) * (16 * SL) + fsw[s]);
        if constexpr (RAGGED) {
            const bool second = slice >= nk1;
            const uint32_t at = (uint32_t)(second ? slice - nk1 : slice) * SL + (uint32_t)(s * 4 + fp) * 16u;
            if (at >= (second ? p.k2 : p.k)) v = td_u32x4{0, 0, 0, 0};
        }
        if (t == 0 || t > NB) fa[buf][t == 0 ? 0 : t - NB] = v; else fb[buf][t - 1] = v;
    };
    constexpr int NM = NA * NB, NR = NA + NB;
    constexpr int kReadEvery = NM / NR > 2 ? 2 : (NM / NR > 0 ? NM / NR : 1), kReadsPer = (NR + NM - 1) / NM;
    constexpr int kLoadEvery = NM / G::kPer > 0 ? NM / G::kPer : 1, kLoadsPer = (G::kPer + NM - 1) / NM;

    if constexpr (EPI == EPI_REPAIR) {
        const uint32_t at = __builtin_amdgcn_readfirstlane(
            (uint32_t)(uintptr_t)(__attribute__((address_space(3))) unsigned char*)lds + G::kRing + wave * 1024);
        if (wave == 0) load_to_lds(at, lane * 16, buffer_of(p.lo + n0, rows_b * 4), 0u);
        if (wave == 1) load_to_lds(at, lane * 16, buffer_of(p.hi + n0, rows_b * 4), 0u);
        if (wave == 2) load_to_lds(at, lane * 16, buffer_of(p.e + m0, (rows_a * 4 + 15u) & ~15u), 0u);
    }
    // In period p (the half of slice p behind the barrier, and the first half of slice p+1) the loads of
    // B(p+SB) and then of A(p+SA) are issued; the prologue issues those of periods -SB .. -1.
#pragma unroll
    for (int s = 0; s < SA - SB; ++s) {
        const Source o = source(true, s);
#pragma unroll
        for (int i = 0; i < LA; ++i) load_one(true, i, s, o);
    }
#pragma unroll
    for (int s = 0; s < SB; ++s) {
        const Source ob = source(false, s), oa = source(true, s + SA - SB);
#pragma unroll
        for (int i = 0; i < LB; ++i) load_one(false, i, s, ob);
#pragma unroll
        for (int i = 0; i < LA; ++i) load_one(true, i, s + SA - SB, oa);
    }
    asm volatile("s_waitcnt vmcnt(%0)" ::"n"(G::kWait + G::kPer) : "memory");
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
    uint32_t ba = 0, bb = 0;
    if (nk > 0) {
#pragma unroll
        for (int t = 0; t < NR; ++t) read_one(0, t, 0, 0, 0, slice_of(0));
    }
    fence(acc);
    asm volatile("s_nop 7" ::: "memory");
    __builtin_amdgcn_sched_barrier(0);
    auto multiply = [&](auto i8, int from, int to) {
        // (a wait that the compiler knows of: what it believes to be under way here it waits for in every turn of the loop)
        __builtin_amdgcn_sched_barrier(0);
        __builtin_amdgcn_s_waitcnt(kNoLds);
        __builtin_amdgcn_sched_barrier(0);
        for (int kt = from; kt < to; ++kt) {
            const Source ob = source(false, kt + SB), oa = source(true, kt + SA);
            const uint32_t na = ba + 1 == SA ? 0 : ba + 1, nb = bb + 1 == SB ? 0 : bb + 1;
            const int cur = RAGGED ? slice_of(kt) : 0, nxt = RAGGED ? slice_of(kt + 1 < nk ? kt + 1 : kt) : 0;
#pragma unroll
            for (int st = 0; st < KS - 1; ++st)
#pragma unroll
                for (int q = 0; q < NM; ++q) {
#pragma unroll
                    for (int u = 0; u < kReadsPer; ++u) {
                        const int t = (q / kReadEvery) * kReadsPer + u;
                        if (q % kReadEvery == 0 && t < NR) read_one((st + 1) & 1, t, ba, bb, st + 1, cur);
                    }
                    __builtin_amdgcn_sched_barrier(0);
                    if constexpr (RAGGED) asm volatile("s_nop 1");
                    mma16<decltype(i8)::value>(acc[q / NB][q % NB], fb[st & 1][q % NB], fa[st & 1][q / NB]);
                    __builtin_amdgcn_sched_barrier(0);
                }
            // slice kt+1 has arrived (this wavefront's share; the barrier makes it everybody's) and the last
            // fragments of slice kt are in registers
            asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)" ::"n"(G::kWait) : "memory");
            __builtin_amdgcn_s_barrier();
            asm volatile("" ::: "memory");
#pragma unroll
            for (int q = 0; q < NM; ++q) {
#pragma unroll
                for (int u = 0; u < kReadsPer; ++u) {
                    const int t = (q / kReadEvery) * kReadsPer + u;
                    if (q % kReadEvery == 0 && t < NR) read_one(0, t, na, nb, 0, nxt);
                }
#pragma unroll
                for (int u = 0; u < kLoadsPer; ++u) {
                    const int t = (q / kLoadEvery) * kLoadsPer + u;
                    if (q % kLoadEvery != 0) continue;
                    if (t < LB) load_one(false, t, bb, ob);
                    else if (t < LB + LA) load_one(true, t - LB, ba, oa);
                }
                __builtin_amdgcn_sched_barrier(0);
                if constexpr (RAGGED) asm volatile("s_nop 1");
                mma16<decltype(i8)::value>(acc[q / NB][q % NB], fb[1][q % NB], fa[1][q / NB]);
                __builtin_amdgcn_sched_barrier(0);
            }
            ba = na;
            bb = nb;
        }
    };
    uint32_t bits[NA] = {};                           // REPAIR: bit 4j + q: the element acc[i][j][q] is flagged
    if constexpr (EPI == EPI_REPAIR) {
        multiply(std::true_type{}, 0, nk1);
        asm volatile("s_nop 15\n\ts_nop 15" ::: "memory");   // (the products are in inline assembly: their results are waited for here)
        fence(acc);
        f32x4_t lo[NB], hi[NB];
        int ex[NA];
        const float* par = reinterpret_cast<const float*>(lds + G::kRing);
        const int nc = wn * NB * 16 + 4 * fp, mr = wm * NA * 16 + frow;   // first column, row of this lane in the tile
        uint32_t columns = 0u;                        // flags of existing columns
#pragma unroll
        for (int j = 0; j < NB; ++j) {                // N % 8 == 0: four columns or none
            const bool in = n0 + nc + j * 16 < p.N;
            columns |= in ? 15u << (4 * j) : 0u;
            lo[j] = *reinterpret_cast<const f32x4_t*>(par + nc + j * 16);
            hi[j] = *reinterpret_cast<const f32x4_t*>(par + 256 + nc + j * 16);
        }
#pragma unroll
        for (int i = 0; i < NA; ++i) ex[i] = reinterpret_cast<const int*>(par)[512 + mr + i * 16];
#pragma unroll
        for (int i = 0; i < NA; ++i) {
            bits[i] = 0u;
#pragma unroll
            for (int j = 0; j < NB; ++j)
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    const float v = ldexpf((float)__float_as_int(acc[i][j][q]), ex[i]);
                    const bool inside = (v >= lo[j][q]) & (v < hi[j][q]);             // (no short cuts: as branches, a third more time)
                    bits[i] |= inside ? 0u : 1u << (4 * j + q);
                    acc[i][j][q] = 0.0f;
                }
            if (m0 + mr + i * 16 >= p.M) bits[i] = 0u;
            bits[i] &= columns;
            // (one row block at a time, and its cleared accumulators made here: the compiler otherwise prepares all of the
            // second product's beside the first one's, and the 256 x 128 tile spills: 256 -> 172 registers)
#pragma unroll
            for (int j = 0; j < NB; ++j) asm volatile("" : "+v"(acc[i][j]));
            asm volatile("" : "+v"(bits[i]));
            __builtin_amdgcn_sched_barrier(0);
        }
        fence(acc);
        asm volatile("s_nop 7" ::: "memory");
        __builtin_amdgcn_sched_barrier(0);
        multiply(std::false_type{}, nk1, nk);
#pragma unroll
        for (int i = 0; i < NA; ++i) asm volatile("" : "+v"(bits[i]));   // (nothing derived from them is kept through the loop)
    } else {
        multiply(std::false_type{}, 0, nk);
    }
    // (the products are in inline assembly: their results are waited for here)
    asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)\n\ts_nop 15\n\ts_nop 15" ::: "memory");
    __builtin_amdgcn_s_barrier();
    fence(acc);

    finish_tile<EPI, kWavesPerTile, WM, NA, NB>(p, acc, bits, lds, tid, m0, n0, ks);
}

// The same products with 4 wavefronts, one per SIMD, in a 2 x 2 grid: 32 NA x 32 NB per tile.  For large tiles: a wavefront's
// part is 128 x 128 instead of 128 x 64, so a slice's fragments are read 4 (instead of 6) times the slice's bytes from LDS,
// which the eight wavefronts above keep busy all the time; the accumulators fill the second half of the register file.
// One wavefront per SIMD hides nothing behind another one, so what stands between two MFMAs (16 cycles, four issue slots)
// is placed by hand, one thing to a gap: a fragment read in every second gap of a half slice, and in equal distances
// over the whole slice the loads that refill the ring, m0 in one gap and the load in the next (which is also the wait state
// between them).  The same loads in bursts or with everything in one gap: 392 instead of 376 us, 4096 x 4096 x 16384 on random data
// (eight wavefronts: 404).
template <int EPI, int NA, int NB>
struct QuadTile {
    static constexpr int SL = 128, TM = 32 * NA, TN = 32 * NB, UA = TM * SL, UB = TN * SL;
    static constexpr int SB = kLdsBytes / (UA + UB), SA = SB * (UA + UB) + UA <= kLdsBytes ? SB + 1 : SB;
    static constexpr int kPer = NA + NB;                    // loads of a wavefront per slice, and reads per half slice
    static constexpr int NM = NA * NB, TOT = 2 * NM;        // MFMAs (gaps) of half a slice, of a slice
    static constexpr int kEvery = TOT / kPer;               // gaps from load to load
    static constexpr int kFirst = (NM - 2 + kEvery) / kEvery;   // loads of a period that fall into its first half
    static constexpr int kTurnA = 2 * kPer <= NM - 4 ? NM - 4 : NM - 1, kTurnB = 2 * kPer <= NM - 4 ? NM - 2 : NM - 1;   // behind the reads
    static constexpr int kWaitB = NA + (SB - 2) * kPer, kWaitA = (SA - 2) * kPer, kWait = kWaitB < kWaitA ? kWaitB : kWaitA;
    static constexpr int kStart = (SA > SB ? NA : 0) + (SB - 2) * kPer + kFirst;   // loads behind those of slice 0 in the prologue
    static constexpr int kEpiLds = EpiRows<EPI, 4, 2, NA, NB>::kBytes;
    static constexpr int kLds = SA * UA + SB * UB > kEpiLds ? SA * UA + SB * UB : kEpiLds;
    static_assert(SB >= 2 && kWait <= 63 && kStart <= 63 && kLds <= kLdsBytes, "slice buffers");
    static_assert(2 * kPer <= NM + 1 && kFirst * kEvery >= NM && (kPer - 1) * kEvery + 1 < TOT, "places of reads and loads");
};

template <int EPI, bool RAGGED, int NA, int NB>
__global__ void __launch_bounds__(256, 1) gemm_quad_kernel(GemmArgs p, TileMap tm) {
    typedef QuadTile<EPI, NA, NB> G;
    constexpr int SL = G::SL, TM = G::TM, TN = G::TN, SA = G::SA, SB = G::SB, NM = G::NM, TOT = G::TOT;
    extern __shared__ __align__(1024) unsigned char lds[];
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6), wm = wave >> 1, wn = wave & 1;

    const int xcd = (int)blockIdx.x & 7, local = (int)blockIdx.x >> 3;
    int tile_m, tile_n, ks;
    if (!place(tm, xcd, local, tile_m, tile_n, ks)) return;
    const int64_t m0 = (int64_t)tile_m * TM, n0 = (int64_t)tile_n * TN;

    // whole slices [s0, s0 + nk) of this block's range (RAGGED: the last range has the rest of the row as well), from a
    // starting point of its own (REPAIR: of either product)
    const int nk1 = (int)(p.k / SL), nk2 = (int)(p.k2 / SL);
    const int s0 = ks * tm.slices;
    const int nk = max(0, min(tm.slices, nk1 + nk2 - s0));
    const int rot = first_slice(xcd, local, EPI == EPI_REPAIR ? nk1 : nk), rot2 = EPI == EPI_REPAIR ? first_slice(xcd, local, nk2) : 0;

    const uint32_t rows_a = (uint32_t)min((int64_t)TM, p.M - m0), rows_b = (uint32_t)min((int64_t)TN, p.N - n0);
    const i32x4_t ra1 = buffer_of(p.A + (size_t)m0 * p.k, rows_a * p.k), rb1 = buffer_of(p.B + (size_t)n0 * p.k, rows_b * p.k);
    const i32x4_t ra2 = buffer_of(p.A2 + (size_t)m0 * p.k2, rows_a * p.k2), rb2 = buffer_of(p.B2 + (size_t)n0 * p.k2, rows_b * p.k2);

    // a load is 8 rows of 128 bytes: lane -> row lane / 8, piece (lane % 8) ^ row; wavefront w loads rows [w*TM/4, (w+1)*TM/4) of A,
    // of B alike
    const uint32_t lrow = (uint32_t)lane >> 3, piece = (((uint32_t)lane & 7u) ^ lrow) * 16u;
    const uint32_t row_a = (uint32_t)(wave * (TM / 4)) + lrow, row_b = (uint32_t)(wave * (TN / 4)) + lrow;
    const uint32_t base = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) unsigned char*)lds;
    const uint32_t lds_a = __builtin_amdgcn_readfirstlane(base + wave * (G::UA / 4));
    const uint32_t lds_b = __builtin_amdgcn_readfirstlane(base + SA * G::UA + wave * (G::UB / 4));

    // The slice that the next loads of A (of B) fetch.  It is found in steps, which stand in different gaps.
    const td_slices seq{nk1, nk2, s0, nk, rot, rot2, p.k, p.k2};
    struct Stream : td_slice_source {
        uint32_t voff, to;                    // this lane's offset; ring buffer of this wavefront
    };
    auto find = [&](Stream& o, bool is_a, int step) {
        td_find_slice<EPI == EPI_REPAIR, SL>(o, seq, is_a ? ra1 : rb1, is_a ? ra2 : rb2, step);
        if (step == 2 || step == 4) asm volatile("" : "+s"(o.soff));
        if (step == 5) {
            o.voff = __umul24(is_a ? row_a : row_b, o.pitch) + piece;   // (rows of at most 2^23 bytes)
            asm volatile("" : "+v"(o.voff));                            // here, and not where it is used
        }
    };
    // (m0 and the load are two statements: see the listing's test)
    auto target = [&](uint32_t to, auto n) { asm volatile("s_add_u32 m0, %0, %1" ::"s"(to), "n"(decltype(n)::value * 1024) : "scc"); };
    auto fetch = [&](const Stream& o) { asm volatile("buffer_load_dwordx4 %0, %1, %2 offen lds" ::"v"(o.voff), "s"(o.rs), "s"(o.soff)); };
    auto load = [&](auto n, Stream& o) {
        target(o.to, n);
        asm volatile("s_nop 0");
        fetch(o);
        o.voff += 8 * o.pitch;
    };
    auto at = [&](Stream& o, bool is_a, int t, uint32_t to) {
        o.t = t;
        o.to = to;
#pragma unroll
        for (int step = 0; step < 6; ++step) find(o, is_a, step);
    };
    // In period p (the half of slice p behind the barrier, and the first half of slice p+1) the loads of B(p+SB) and then
    // of A(p+SA) are issued; the prologue issues those of periods -SB .. -2 and the first half of period -1.
    Stream oa, ob;
    oa.rs.w = ob.rs.w = ra1.w;
    asm volatile("s_nop 4");   // (scalars that vector instructions have written are read by the loads below, which the compiler cannot see)
    if constexpr (SA > SB) {
        at(oa, true, 0, lds_a);
        for_constants<NA>([&](auto i) { load(i, oa); });
    }
    for_constants<SB>([&](auto s) {
        constexpr int n = decltype(s)::value, most = n + 1 < SB ? G::kPer : G::kFirst;
        at(ob, false, n, lds_b + n * G::UB);
        at(oa, true, n + SA - SB, lds_a + (n + SA - SB) * G::UA);
        for_constants<NB>([&](auto i) { if constexpr (decltype(i)::value < most) load(i, ob); });
        for_constants<NA>([&](auto i) { if constexpr (NB + decltype(i)::value < most) load(i, oa); });
    });

    f32x4_t acc[NA][NB];
#pragma unroll
    for (int i = 0; i < NA; ++i)
#pragma unroll
        for (int j = 0; j < NB; ++j) acc[i][j] = f32x4_t{0, 0, 0, 0};
    // fragments: lane holds 16 bytes of row lane%16 at piece 4*step + lane/16
    const int frow = lane & 15, fp = lane >> 4;
    uint32_t frag_a[2], frag_b[2];
#pragma unroll
    for (int s = 0; s < 2; ++s) {
        const uint32_t sw = (uint32_t)(frow * SL + (((s * 4 + fp) ^ (frow & 7)) * 16));
        frag_a[s] = (uint32_t)(wm * NA * 16 * SL) + sw;
        frag_b[s] = (uint32_t)(SA * G::UA + wn * NB * 16 * SL) + sw;
    }
    td_u32x4 fa[2][NA], fb[2][NB];
    uint32_t xa = frag_a[0], xb = frag_b[0];          // where the next half slice's fragments lie
    auto read_one = [&](int buf, int t) {             // fa[0], all of fb, the rest of fa
        if (t == 0) fa[buf][0] = *reinterpret_cast<const td_u32x4*>(lds + xa);
        else if (t <= NB) fb[buf][t - 1] = *reinterpret_cast<const td_u32x4*>(lds + xb + (t - 1) * (16 * SL));
        else fa[buf][t - NB] = *reinterpret_cast<const td_u32x4*>(lds + xa + (t - NB) * (16 * SL));
    };
    auto mma = [&](auto i8, f32x4_t& c, const td_u32x4& a, const td_u32x4& b) {
        if constexpr (decltype(i8)::value) asm volatile("v_mfma_i32_16x16x64_i8 %0, %1, %2, %0" : "+a"(c) : "v"(a), "v"(b));
        else asm volatile("v_mfma_f32_16x16x32_bf16 %0, %1, %2, %0" : "+a"(c) : "v"(a), "v"(b));
    };
    auto hold = [&]() {                               // as fence(), for accumulators in the other half of the register file
#pragma unroll
        for (int i = 0; i < NA; ++i)
#pragma unroll
            for (int j = 0; j < NB; ++j) asm volatile("" : "+a"(acc[i][j])::"memory");
        __builtin_amdgcn_sched_barrier(0);
    };
    asm volatile("s_waitcnt vmcnt(%0)" ::"n"(G::kStart) : "memory");
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
#pragma unroll
    for (int t = 0; t < G::kPer; ++t) read_one(0, t);
    xa = frag_a[1];
    xb = frag_b[1];
    uint32_t ra = 0, rb = 0;                          // ring offsets of the slice that is multiplied
    auto turn = [&](uint32_t o, uint32_t unit, uint32_t ring) { return o + unit == ring ? 0u : o + unit; };
    hold();
    asm volatile("s_nop 7" ::: "memory");
    __builtin_amdgcn_sched_barrier(0);
    // One slice: the MFMAs of its first half while the fragments of the second are read, the barrier behind which slice kt+1
    // has arrived and this slice's buffers are free, the MFMAs of the second half while slice kt+1's first are read.
    auto multiply = [&](auto i8, int from, int to) {
        // (waits that the compiler knows of: what it believes to be under way here it waits for in every turn of the loop, for
        // loads from memory with all of the ring's: REPAIR, 128 x 128, 520 -> 450 us)
        __builtin_amdgcn_sched_barrier(0);
        __builtin_amdgcn_s_waitcnt(kNoLds & (EPI == EPI_REPAIR && !decltype(i8)::value ? kNoLoads : 0xffff));
        __builtin_amdgcn_sched_barrier(0);
        for (int kt = from; kt < to; ++kt) {
            for_constants<TOT>([&](auto gap) {
                constexpr int q = decltype(gap)::value, half = q / NM, h = q % NM;
                constexpr int since = (q + NM) % TOT;                                     // gaps since the barrier
                constexpr int until_b = NM - 1 - h, until_a = (G::kEvery * NB < NM ? G::kEvery * NB : NM) - 1 - h;
                if constexpr (q == NM) {
                    __builtin_amdgcn_s_waitcnt(kNoLds);
                    asm volatile("s_waitcnt vmcnt(%0)" ::"n"(G::kWait) : "memory");
                    __builtin_amdgcn_s_barrier();
                    asm volatile("" ::: "memory");
                    oa.to = lds_a + ra;
                    ob.to = lds_b + rb;
                }
                if constexpr (h % 2 == 0 && h / 2 < G::kPer) read_one(1 - half, h / 2);
                // the loads of this period: m0, the load
                constexpr int n = since / G::kEvery, in = since % G::kEvery;
                if constexpr (n < NB) {
                    if constexpr (in == 0) target(ob.to, num<n>{});
                    if constexpr (in == 1) {
                        fetch(ob);
                        ob.voff += 8 * ob.pitch;
                    }
                } else if constexpr (n < G::kPer) {
                    if constexpr (in == 0) target(oa.to, num<n - NB>{});
                    if constexpr (in == 1) {
                        fetch(oa);
                        oa.voff += 8 * oa.pitch;
                    }
                }
                // the slices of the next period's loads: B's before the barrier, A's while B's are issued
                if constexpr (half == 0 && until_b < 12 && until_b % 2 == 0) find(ob, false, 5 - until_b / 2);
                if constexpr (half == 1 && until_a >= 0 && until_a < 12 && until_a % 2 == 0) find(oa, true, 5 - until_a / 2);
                // ring offsets and addresses of the next fragments, once this half's are under way
                if constexpr (half == 0 && h == G::kTurnA) xa = frag_a[0] + turn(ra, G::UA, SA * G::UA);
                if constexpr (half == 0 && h == G::kTurnB) xb = frag_b[0] + turn(rb, G::UB, SB * G::UB);
                if constexpr (half == 1 && h == G::kTurnA) {
                    ra = turn(ra, G::UA, SA * G::UA);
                    xa = frag_a[1] + ra;
                }
                if constexpr (half == 1 && h == G::kTurnB) {
                    rb = turn(rb, G::UB, SB * G::UB);
                    xb = frag_b[1] + rb;
                }
                __builtin_amdgcn_sched_barrier(0);
                mma(i8, acc[h / NB][h % NB], fb[half][h % NB], fa[half][h / NB]);
                __builtin_amdgcn_sched_barrier(0);
            });
        }
    };
    uint32_t bits[NA] = {};                           // REPAIR: bit 4j + q: the element acc[i][j][q] is flagged
    if constexpr (EPI == EPI_REPAIR) {
        multiply(std::true_type{}, 0, nk1);
        asm volatile("s_nop 15\n\ts_nop 15" ::: "memory");   // (the products are in inline assembly: their results are waited for here)
        hold();
        const int nc = wn * NB * 16 + 4 * fp, mr = wm * NA * 16 + frow;   // first column, row of this lane in the tile
        const f32x4_t none = {0, 0, 0, 0};
        int ex[NA];
#pragma unroll
        for (int i = 0; i < NA; ++i) ex[i] = m0 + mr + i * 16 < p.M ? p.e[m0 + mr + i * 16] : 0;
        f32x4_t lo[NB], hi[NB];
#pragma unroll
        for (int j = 0; j < NB; ++j) {                // N % 8 == 0: four columns or none
            const int64_t n = n0 + nc + j * 16 < p.N ? n0 + nc + j * 16 : 0;
            lo[j] = *reinterpret_cast<const f32x4_t*>(p.lo + n);
            hi[j] = *reinterpret_cast<const f32x4_t*>(p.hi + n);
        }
        __builtin_amdgcn_sched_barrier(0);
        // (column block by column block: row by row all bounds stay in registers to the end, and some spill)
        for_constants<NB>([&](auto column_block) {
            constexpr int j = decltype(column_block)::value;
            const bool in = n0 + nc + j * 16 < p.N;
            for_constants<NA>([&](auto row_block) {
                constexpr int i = decltype(row_block)::value;
                uint32_t out = 0u;
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    const float v = ldexpf((float)__float_as_int(acc[i][j][q]), ex[i]);
                    const bool inside = (v >= lo[j][q]) & (v < hi[j][q]);    // (no short cuts: as branches, a third more time)
                    out |= inside ? 0u : 1u << (4 * j + q);
                }
                bits[i] |= in && m0 + mr + i * 16 < p.M ? out : 0u;
                acc[i][j] = none;
                asm volatile("" : "+a"(acc[i][j]));
                asm volatile("" : "+v"(bits[i]));
                __builtin_amdgcn_sched_barrier(0);
            });
        });
        hold();
        asm volatile("s_nop 7" ::: "memory");
        __builtin_amdgcn_sched_barrier(0);
        multiply(std::false_type{}, nk1, nk);
#pragma unroll
        for (int i = 0; i < NA; ++i) asm volatile("" : "+v"(bits[i]));   // (nothing derived from them is kept through the loop)
    } else {
        multiply(std::false_type{}, 0, nk);
    }
    if constexpr (RAGGED) {
        // the rest of the row, alone: pieces past its end are loaded from its start (in bounds) and zeroed as they are read
        const uint32_t k = p.k2 ? p.k2 : p.k, from = k / SL * SL;
        if (ks == (1 << tm.splits_log2) - 1 && from < k) {
            asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)" ::: "memory");
            __builtin_amdgcn_s_barrier();
            const uint32_t pc = from + piece < k ? from + piece : 0u;
            oa.rs = p.k2 ? ra2 : ra1;
            ob.rs = p.k2 ? rb2 : rb1;
            oa.pitch = ob.pitch = k;
            oa.soff = ob.soff = 0u;
            oa.voff = row_a * k + pc;
            ob.voff = row_b * k + pc;
            oa.to = lds_a;
            ob.to = lds_b;
            for_constants<NA>([&](auto i) { load(i, oa); });
            for_constants<NB>([&](auto i) { load(i, ob); });
            asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
            __builtin_amdgcn_s_barrier();
            asm volatile("" ::: "memory");
#pragma unroll
            for (int s = 0; s < 2; ++s) {
                xa = frag_a[s];
                xb = frag_b[s];
                const bool in = from + (uint32_t)(s * 4 + fp) * 16u < k;
                const td_u32x4 zero = {0, 0, 0, 0};
#pragma unroll
                for (int t = 0; t < G::kPer; ++t) read_one(s, t);
#pragma unroll
                for (int i = 0; i < NA; ++i) {
                    fa[s][i] = in ? fa[s][i] : zero;
                    asm volatile("" : "+v"(fa[s][i]));
                }
#pragma unroll
                for (int j = 0; j < NB; ++j) {
                    fb[s][j] = in ? fb[s][j] : zero;
                    asm volatile("" : "+v"(fb[s][j]));
                }
                __builtin_amdgcn_sched_barrier(0);
                asm volatile("s_nop 7" ::: "memory");
                __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                for (int h = 0; h < NM; ++h) mma(std::false_type{}, acc[h / NB][h % NB], fb[s][h % NB], fa[s][h / NB]);
                __builtin_amdgcn_sched_barrier(0);
            }
        }
    }
    // (the products are in inline assembly: their results are waited for here)
    asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)\n\ts_nop 15\n\ts_nop 15" ::: "memory");
    __builtin_amdgcn_s_barrier();
    hold();
    finish_tile<EPI, 4, 2, NA, NB>(p, acc, bits, lds, tid, m0, n0, ks);
}

// The tile for a product of more than 64 rows: the one with the least time by
//     rounds over 256 CUs x (slices x time of a slice + time of the prologue and epilogue) + partial sums,
// with the times below (least squares over 10 tiles, 512 products: d, h from 512, 2048 to 4096, 16384, 70 to 3000 tokens, all
// epilogues).  The slices' times are those of operands of zeros, which draw less power: 2048 x 16384 x 4096 with sigma is 197 us by the
// rule, 193 measured on zero weights and 258 on random ones, and on random data the other large products take 1.3 to 1.4 times the
// rule's time as well (range test 340 for 268, calibration 103 for 73, fold 375 for 275).  So the rule ranks tiles, and takes an
// epilogue for more slices than it costs.
// Four wavefronts (Q) take less per slice, eight finish a tile with a range test or sigma sooner.
// Up to 64 rows the weights stream from memory: the larger of MFMA cycles and of the cycles in which the operands arrive, at 34
// bytes per cycle and CU (a chosen number, which ranks these tiles; the larger one for slices of 256 bytes stands for longer runs from HBM: 64
// tokens, us with 256 / 128 bytes a slice: d = 4096, up projection of h = 16384 38.9 / 46.2, of h = 11008 (40 tokens) 33.9 / 44.1,
// dense 27.4 / 29.0; d = 2048 output product 10.8 / 12.1).
// `splittable`: K may be cut into 2, 4 or 8 ranges (at most kPartRows rows of partial sums are kept).
constexpr int64_t kPartRows = 4096;
struct TileChoice { int shape, splits; };
struct Shape {
    int m, n, slice;
    bool quad;
    float slice_us, repair_us, hidden_us, store_us;      // a slice; prologue and epilogue with the range test, with sigma, with stores alone
};
constexpr Shape kShape[] = {
    {256, 256, 128, true, 1.055f, 32.9f, 30.8f, 5.3f}, {192, 256, 128, true, 0.828f, 26.8f, 24.0f, 4.6f},
    {256, 128, 128, true, 0.611f, 18.0f, 15.9f, 3.6f}, {192, 128, 128, true, 0.494f, 13.5f, 12.0f, 3.2f},
    {128, 128, 128, true, 0.391f, 10.2f, 9.0f, 2.7f}, {192, 256, 128, false, 0.952f, 17.1f, 16.6f, 3.6f},
    {256, 128, 128, false, 0.730f, 9.9f, 9.9f, 3.0f}, {192, 128, 128, false, 0.564f, 9.3f, 8.4f, 2.8f},
    {128, 128, 128, false, 0.418f, 9.0f, 6.8f, 2.6f}, {128, 64, 128, false, 0.368f, 6.1f, 5.2f, 2.5f},
    // at most 64 rows
    {64, 64, 128, false}, {64, 64, 256, false}, {64, 32, 256, false}, {64, 128, 128, false}};
constexpr int kShapes = sizeof(kShape) / sizeof(Shape);
constexpr float kRaggedSlice = 1.35f;                    // eight wavefronts check every fragment of a ragged product (Q: the last slice's)
constexpr float kPartUs = 0.22f / (1024 * 1024);         // a byte of partial sums, written and read again

// whole: K has to be whole slices (of both products); else a ragged K is allowed
TileChoice choose_tile(const GemmArgs& p, int epi, bool whole) {
    TileChoice best{0, 1};
    double best_cost = 1e300;
    const int64_t M = p.M, N = p.N;
    const bool splittable = epi == EPI_PART;
    for (int s = 0; s < kShapes; ++s) {
        const Shape& t = kShape[s];
        const int SL = t.slice;
        const bool ragged = p.k % SL != 0 || p.k2 % SL != 0;
        if ((whole && ragged) || (t.m == 64) != (M <= 64)) continue;
        const int64_t slices = (p.k + SL - 1) / SL + (p.k2 + SL - 1) / SL;
        for (int sp = 1; sp <= (splittable ? 8 : 1); sp *= 2) {
            if (sp > 1 && (slices * SL / sp < 1024 || sp * M > kPartRows)) break;
            const TileMap map = make_tile_map(M, N, t.m, t.n, (int)slices, sp);
            const double rounds = (double)(((int64_t)map.rm * map.rn + 31) / 32);   // blocks of one XCD (of one range): 32 at once
            double cost;
            if (M > 64) {
                const double fixed = epi == EPI_REPAIR ? t.repair_us : epi == EPI_HIDDEN ? t.hidden_us : t.store_us;
                cost = rounds * (map.slices * t.slice_us * (ragged && !t.quad ? kRaggedSlice : 1.0f) + fixed) +
                       (splittable ? sp * (double)M * (double)N * 4.0 * kPartUs : 0.0);
            } else {
                const double mfma = 2100.0 / 128.0 * SL * t.m * t.n / 65536.0;
                const double feed = (M + t.n) * (double)SL / (SL > 128 ? 34.5 : 34.0);
                const double tail = 3000.0 + (epi == EPI_F32 ? 0.12 : 0.06) * t.m * t.n;
                cost = rounds * (map.slices * (mfma > feed ? mfma : feed) + tail) + (splittable ? sp * (double)M * (double)N * 8.0 / 2000.0 : 0.0);
            }
            if (cost < best_cost) { best_cost = cost; best = {s, sp}; }
        }
    }
    return best;
}

// f(slice bytes, wm, na, nb) with the constants of a shape (wm = 0: gemm_quad_kernel)
template <typename F> void for_shape(int shape, F f) {
    switch (shape) {
        case 0: f(num<128>{}, num<0>{}, num<8>{}, num<8>{}); break;
        case 1: f(num<128>{}, num<0>{}, num<6>{}, num<8>{}); break;
        case 2: f(num<128>{}, num<0>{}, num<8>{}, num<4>{}); break;
        case 3: f(num<128>{}, num<0>{}, num<6>{}, num<4>{}); break;
        case 4: f(num<128>{}, num<0>{}, num<4>{}, num<4>{}); break;
        case 5: f(num<128>{}, num<2>{}, num<6>{}, num<4>{}); break;
        case 6: f(num<128>{}, num<2>{}, num<8>{}, num<2>{}); break;
        case 7: f(num<128>{}, num<2>{}, num<6>{}, num<2>{}); break;
        case 8: f(num<128>{}, num<2>{}, num<4>{}, num<2>{}); break;
        case 9: f(num<128>{}, num<2>{}, num<4>{}, num<1>{}); break;
        case 10: f(num<128>{}, num<2>{}, num<2>{}, num<1>{}); break;
        case 11: f(num<256>{}, num<2>{}, num<2>{}, num<1>{}); break;
        case 12: f(num<256>{}, num<4>{}, num<1>{}, num<1>{}); break;
        default: f(num<128>{}, num<2>{}, num<2>{}, num<2>{}); break;
    }
}

template <int EPI, bool RAGGED> void launch_ragged(const GemmArgs& p, const TileChoice& c, hipStream_t s) {
    for_shape(c.shape, [&](auto sl, auto wm, auto na, auto nb) {
        if constexpr (decltype(wm)::value == 0) {
            typedef QuadTile<EPI, na, nb> G;
            const TileMap tm = make_tile_map(p.M, p.N, G::TM, G::TN, (int)(p.k / sl + p.k2 / sl), c.splits);
            hipLaunchKernelGGL((gemm_quad_kernel<EPI, RAGGED, na, nb>), dim3(8 * tm.rm * tm.rn), dim3(256), G::kLds, s, p, tm);
        } else {
            typedef GemmTile<EPI, RAGGED, sl, wm, na, nb> G;
            const int slices = (int)((p.k + sl - 1) / sl + (p.k2 + sl - 1) / sl);
            const TileMap tm = make_tile_map(p.M, p.N, G::TM, G::TN, slices, c.splits);
            hipLaunchKernelGGL((gemm_tile_kernel<EPI, RAGGED, sl, wm, na, nb>), dim3(8 * tm.rm * tm.rn), dim3(512), G::kLds, s, p, tm);
        }
    });
}

// EPI_F32 and EPI_PART take any K that is whole 16-byte pieces
template <int EPI> TileChoice launch_tile(const GemmArgs& p, hipStream_t s) {
    constexpr bool may_be_ragged = EPI == EPI_F32 || EPI == EPI_PART;
    const TileChoice c = choose_tile(p, EPI, !may_be_ragged);
    const int sl = kShape[c.shape].slice;
    if constexpr (may_be_ragged) {
        if (p.k % sl != 0 || p.k2 % sl != 0) {
            launch_ragged<EPI, true>(p, c, s);
            return c;
        }
    }
    launch_ragged<EPI, false>(p, c, s);
    return c;
}

template <typename K> bool raise_lds_of(K kernel, int bytes) {
    return hipFuncSetAttribute(reinterpret_cast<const void*>(kernel), hipFuncAttributeMaxDynamicSharedMemorySize, bytes) == hipSuccess;
}

template <int EPI, bool RAGGED> tardis_status_t raise_lds() {
    bool ok = true;
    for (int shape = 0; shape < kShapes; ++shape)
        for_shape(shape, [&](auto sl, auto wm, auto na, auto nb) {
            if constexpr (decltype(wm)::value == 0) ok &= raise_lds_of(gemm_quad_kernel<EPI, RAGGED, na, nb>, QuadTile<EPI, na, nb>::kLds);
            else ok &= raise_lds_of(gemm_tile_kernel<EPI, RAGGED, sl, wm, na, nb>, GemmTile<EPI, RAGGED, sl, wm, na, nb>::kLds);
        });
    return ok ? TARDIS_OK : TARDIS_ERR_HIP;
}

template <typename T>
void launch_generic(const void* A, const void* B, float* C, int64_t M, int64_t N, int64_t K, int accumulate,
                    const void* row_bias, hipStream_t s) {
    dim3 grid((unsigned)((N + GT - 1) / GT), (unsigned)((M + GT - 1) / GT));
    hipLaunchKernelGGL(gemm_nt_generic_kernel<T>, grid, dim3(256), 0, s, static_cast<const T*>(A),
                       static_cast<const T*>(B), C, M, N, K, accumulate, static_cast<const T*>(row_bias));
}

bool gemm_force_generic() {
    const char* v = std::getenv("TARDIS_GEMM_GENERIC");
    return v && v[0] == '1';
}

const unsigned char* bytes_of(const void* p) { return static_cast<const unsigned char*>(p); }
bool is_aligned16(const void* p) { return (reinterpret_cast<uintptr_t>(p) & 15) == 0; }

}  // namespace

// the matrix-core kernels use more LDS than the default limit; raised once, outside any stream capture
tardis_status_t td_gemm_init() {
    static td_once once;
    return once.run([]() -> tardis_status_t {
        TD_TRY((raise_lds<EPI_F32, false>()));
        TD_TRY((raise_lds<EPI_F32, true>()));
        TD_TRY((raise_lds<EPI_PART, false>()));
        TD_TRY((raise_lds<EPI_PART, true>()));
        TD_TRY((raise_lds<EPI_HIDDEN, false>()));
        TD_TRY((raise_lds<EPI_REPAIR, false>()));
        return TARDIS_OK;
    });
}

// more rows than the grid of the kernel for any shape counts
bool td_gemm_refuses_rows(int64_t M) { return (M + GT - 1) / GT > 65535; }

// (any M, N work on the matrix cores; small products are not worth it)
bool td_gemm_on_matrix_cores(const void* A, const void* B, int64_t M, int64_t N, int64_t K, int32_t dtype) {
    return dtype == TARDIS_BF16 && M >= 32 && N >= 32 && M * N >= 128 * 128 && K >= 64 && is_aligned16(A) && is_aligned16(B) &&
           K % 8 == 0 && !gemm_force_generic();
}

// C = A.B^T (+ row_bias), or C += A.B^T (or that sum rounded to bf16 into out16, C left as it was: matrix cores only).  (A second product is added to the first one's finished sums and not summed
// onto them: partial sums of the first may be far larger than the second.)
tardis_status_t td_gemm_nt(const void* A, const void* B, float* C, int64_t M, int64_t N, int64_t K, int32_t dtype,
                           int accumulate, const void* row_bias, hipStream_t s, void* out16) {
    if (M <= 0 || N <= 0 || K <= 0) return TARDIS_ERR_SHAPE;
    if (td_gemm_refuses_rows(M)) return TARDIS_ERR_SHAPE;
    if (td_gemm_on_matrix_cores(A, B, M, N, K, dtype)) {
        TD_TRY(td_gemm_init());
        GemmArgs p{};
        p.A = p.A2 = bytes_of(A);
        p.B = p.B2 = bytes_of(B);
        p.M = M;
        p.N = N;
        p.k = (uint32_t)(K * 2);
        p.C = C;
        p.accumulate = accumulate;
        p.bias = static_cast<const bf16_t*>(row_bias);
        p.out = static_cast<bf16_t*>(out16);
        launch_tile<EPI_F32>(p, s);
    } else if (dtype == TARDIS_BF16) {
        launch_generic<bf16_t>(A, B, C, M, N, K, accumulate, row_bias, s);
    } else {
        launch_generic<float>(A, B, C, M, N, K, accumulate, row_bias, s);
    }
    TD_HIP(hipGetLastError());
    return TARDIS_OK;
}

// The products of calls with many tokens (bf16 layers, d % 128 == 0, h % 8 == 0, 16-byte aligned operands).
// mask[t] = range test of Xq . Q^T (exact int32 sums), out[t] = sigma(z) - (a z + c) at its bits, else 0, z = X . W1^T + b1;
// rest (or null) = what `out` lost when it was rounded to bf16, in bf16
tardis_status_t td_gemm_repair(const tardis_layer_s* L, const int8_t* XQ, const int32_t* e, const void* X, const void* b1,
                               uint32_t* mask, void* out, void* rest, int64_t n, hipStream_t s) {
    GemmArgs p{};
    p.A = bytes_of(XQ);
    p.B = bytes_of(L->Q);
    p.A2 = bytes_of(X);
    p.B2 = bytes_of(L->W1);
    p.M = n;
    p.N = L->h;
    p.k = (uint32_t)L->d;
    p.k2 = (uint32_t)(L->d * 2);
    p.bias = static_cast<const bf16_t*>(b1);
    p.out = static_cast<bf16_t*>(out);
    p.rest = static_cast<bf16_t*>(rest);
    p.lo = L->tlo;
    p.hi = L->thi;
    p.slope = L->a;
    p.icept = L->c;
    p.e = e;
    p.mask = mask;
    p.mask_words = (int)L->mask_words;
    p.act = L->act;
    launch_tile<EPI_REPAIR>(p, s);
    TD_HIP(hipGetLastError());
    return TARDIS_OK;
}

// out[t] = sigma(X . W1^T + b1), the dense FFN's hidden activations
tardis_status_t td_gemm_hidden(const tardis_layer_s* L, const void* X, const void* b1, void* out, int64_t n, hipStream_t s) {
    GemmArgs p{};
    p.A = p.A2 = bytes_of(X);
    p.B = p.B2 = bytes_of(L->W1);
    p.M = n;
    p.N = L->h;
    p.k = (uint32_t)(L->d * 2);
    p.bias = static_cast<const bf16_t*>(b1);
    p.act = L->act;
    p.out = static_cast<bf16_t*>(out);
    launch_tile<EPI_HIDDEN>(p, s);
    TD_HIP(hipGetLastError());
    return TARDIS_OK;
}

// part[0 .. *parts)[n][d] = partial sums of X . Wp^T + H . W2^T (X, Wp null: the second product alone); the caller
// adds them up.  At most 8 of them.
tardis_status_t td_gemm_output(const void* X, const void* Wp, const void* H, const void* W2, float* part, int* parts,
                               int64_t n, int64_t d, int64_t h, hipStream_t s) {
    GemmArgs p{};
    p.A = bytes_of(X ? X : H);
    p.B = bytes_of(X ? Wp : W2);
    p.A2 = bytes_of(H);
    p.B2 = bytes_of(W2);
    p.M = n;
    p.N = d;
    p.k = (uint32_t)((X ? d : h) * 2);
    p.k2 = X ? (uint32_t)(h * 2) : 0u;
    p.C = part;
    *parts = launch_tile<EPI_PART>(p, s).splits;
    TD_HIP(hipGetLastError());
    return TARDIS_OK;
}

// floats that `part` of td_gemm_output has to hold for calls of up to n tokens (grows with n)
size_t td_gemm_part_floats(int64_t n, int64_t d) {
    const int64_t rows = n > kPartRows ? n : (8 * n < kPartRows ? 8 * n : kPartRows);
    return (size_t)rows * (size_t)d;
}

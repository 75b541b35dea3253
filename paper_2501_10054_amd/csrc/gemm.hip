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
#include <type_traits>

#include "common.h"

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
// One kernel for every product on the matrix cores, with the step that follows the product in its
// epilogue.  Output tile TM x TN = (WM*NA*16) x ((8/WM)*NB*16), 8 wavefronts in a WM x (8/WM) grid, each
// NA x NB tiles of v_mfma_f32_16x16x32_bf16 / v_mfma_i32_16x16x64_i8 (the byte geometry of the two is the
// same: 16 bytes per lane and MFMA).  K runs in slices of 128 bytes per row.
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
// 4096 x 4096 x 16384 in bf16 with random data: 390 us, 1.41 PFLOP/s (one wavefront per SIMD with staging
// through registers, which was here before: 605 us, 0.91).
typedef __bf16 bf16x8_t __attribute__((ext_vector_type(8)));
typedef float f32x4_t __attribute__((ext_vector_type(4)));
typedef int i32x4_t __attribute__((ext_vector_type(4)));

constexpr int kWavesPerTile = 8;
constexpr int kLdsBytes = 160 * 1024;

// Which block computes which tile.  Blocks b, b+8, b+16, ... run on one XCD and share its L2, so
// each XCD gets a rectangle of rm x rn tiles (the 8 XCDs form a gm x gn grid over the tile grid,
// times `splits` ranges of K), and inside the rectangle consecutive blocks walk `group` tile rows
// column by column: the 32 blocks an XCD runs at once then cover a compact patch and re-use each
// other's slices of A and B from L2 instead of fetching them from HBM again.
struct TileMap {
    int tiles_m, tiles_n;      // tile grid of C
    int splits;                // K ranges (1, 2, 4 or 8)
    int gn;                    // XCD grid columns (rows = 8 / splits / gn)
    int rm, rn;                // tiles per XCD rectangle
    int group;                 // tile rows walked together
    int slices;                // K slices per range
};

TileMap make_tile_map(int64_t M, int64_t N, int tile_m, int tile_n, int slices, int splits) {
    TileMap t;
    t.tiles_m = (int)((M + tile_m - 1) / tile_m);
    t.tiles_n = (int)((N + tile_n - 1) / tile_n);
    t.splits = splits;
    const int nx = 8 / splits;
    int best = 1 << 30, gm = nx;
    for (int cand = 1; cand <= nx; cand *= 2) {            // cand = XCD grid rows
        const int rm = (t.tiles_m + cand - 1) / cand, rn = (t.tiles_n + nx / cand - 1) / (nx / cand);
        const int cost = rm * rn * 4096 + rm * tile_m + rn * tile_n;   // fewest blocks, then least operand bytes
        if (cost < best) { best = cost; gm = cand; }
    }
    t.gn = nx / gm;
    t.rm = (t.tiles_m + gm - 1) / gm;
    t.rn = (t.tiles_n + t.gn - 1) / t.gn;
    t.group = t.rm < 8 ? t.rm : 8;
    t.slices = (slices + splits - 1) / splits;
    return t;
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
    bf16_t* out;                   // HIDDEN, REPAIR: M x N
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
// uses it nowhere else in these kernels, and the listing's test holds it to that)
template <bool ONCE = false>
__device__ __forceinline__ void load_to_lds(uint32_t lds, uint32_t voff, i32x4_t rs, uint32_t soff) {
    if constexpr (ONCE)
        asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tbuffer_load_dwordx4 %1, %2, %3 offen nt lds"
                     ::"s"(lds), "v"(voff), "s"(rs), "s"(soff));
    else
        asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tbuffer_load_dwordx4 %1, %2, %3 offen lds"
                     ::"s"(lds), "v"(voff), "s"(rs), "s"(soff));
}

// round to nearest even, in one instruction
__device__ __forceinline__ uint32_t to_bf16(float v) { return __builtin_bit_cast(uint16_t, (__bf16)v); }

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
    // REPAIR: bounds and exponents wait in LDS for the range test (the largest tile has no room and reads them then)
    static constexpr int kPar = EPI == EPI_REPAIR && TM * TN < 256 * 256 ? 3 * 1024 : 0;
    // as many slices as fit; A one ahead of B where the two do not fit equally often
    static constexpr int kRoom = kLdsBytes - kPar;
    static constexpr int SB = kRoom / (UA + UB) > 10 ? 10 : kRoom / (UA + UB);
    static constexpr int SA = SB < 10 && SB * (UA + UB) + UA <= kRoom ? SB + 1 : SB;
    static constexpr int kRing = SA * UA + SB * UB;
    static constexpr int kPer = LA + LB;
    // loads that may still be in flight when slice kt+2 has to be there (see the order in the kernel)
    static constexpr int kWaitB = LA + (SB - 2) * kPer, kWaitA = (SA - 2) * kPer;
    static constexpr int kWait = kWaitB < kWaitA ? kWaitB : kWaitA;
    static constexpr int kEpiWave = 16 * NB * 16 * (EPI == EPI_REPAIR ? 12 : 4);   // LDS of a wavefront in the epilogue
    static constexpr int kEpiLds = kWavesPerTile * kEpiWave + (EPI == EPI_REPAIR ? 3 * TN * 4 : 0);
    static constexpr int kLds = kRing + kPar > kEpiLds ? kRing + kPar : kEpiLds;
    static_assert(SL % 128 == 0 && UA % 8192 == 0 && UB % 8192 == 0, "whole loads of 1 KB for 8 wavefronts");
    static_assert(SB >= 2 && SA >= 2 && kWait + kPer <= 63 && kLds <= kLdsBytes, "slice buffers");
};

template <int EPI, bool RAGGED, int SL, int WM, int NA, int NB>
__global__ void __launch_bounds__(512) gemm_tile_kernel(GemmArgs p, TileMap tm) {
    typedef GemmTile<EPI, RAGGED, SL, WM, NA, NB> G;
    constexpr int WN = G::WN, TM = G::TM, TN = G::TN, SA = G::SA, SB = G::SB, LA = G::LA, LB = G::LB;
    extern __shared__ __align__(1024) unsigned char lds[];
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm = wave / WN, wn = wave % WN;

    const int xcd = (int)blockIdx.x & 7, local = (int)blockIdx.x >> 3;
    const int ks = xcd % tm.splits, xg = xcd / tm.splits;
    const int per_group = tm.group * tm.rn;
    const int grp = local / per_group, r = local % per_group;
    const int gsz = min(tm.group, tm.rm - grp * tm.group);
    const int tile_m = (xg / tm.gn) * tm.rm + grp * tm.group + r % gsz;
    const int tile_n = (xg % tm.gn) * tm.rn + r / gsz;
    if (tile_m >= tm.tiles_m || tile_n >= tm.tiles_n) return;
    const int64_t m0 = (int64_t)tile_m * TM, n0 = (int64_t)tile_n * TN;

    // slices [s0, s0 + nk) of this block's range, from a starting point of its own (REPAIR: of either product)
    const int nk1 = (int)((p.k + SL - 1) / SL), nk2 = (int)((p.k2 + SL - 1) / SL);
    const int s0 = ks * tm.slices;
    const int nk = max(0, min(tm.slices, nk1 + nk2 - s0));
    auto start = [&](int len) { return len > 0 ? ((local & 7) + xcd * len / 8) % len : 0; };
    const int rot = start(EPI == EPI_REPAIR ? nk1 : nk), rot2 = EPI == EPI_REPAIR ? start(nk2) : 0;
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

    if constexpr (G::kPar > 0) {
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
    [[maybe_unused]] uint32_t bits[NA];               // REPAIR: bit 4j + q: the element acc[i][j][q] is flagged
    if constexpr (EPI == EPI_REPAIR) {
        multiply(std::true_type{}, 0, nk1);
        asm volatile("s_nop 15\n\ts_nop 15" ::: "memory");   // (the products are in inline assembly: their results are waited for here)
        fence(acc);
        f32x4_t lo[NB], hi[NB];
        int ex[NA];
        const float* par = reinterpret_cast<const float*>(lds + G::kRing);
        const int nc = wn * NB * 16 + 4 * fp, mr = wm * NA * 16 + frow;   // first column, row of this lane in the tile
        const f32x4_t none = {0, 0, 0, 0};
#pragma unroll
        for (int j = 0; j < NB; ++j) {                // N % 8 == 0: four columns or none
            const bool in = n0 + nc + j * 16 < p.N;
            if constexpr (G::kPar > 0) {
                lo[j] = *reinterpret_cast<const f32x4_t*>(par + nc + j * 16);
                hi[j] = *reinterpret_cast<const f32x4_t*>(par + 256 + nc + j * 16);
            } else {
                lo[j] = in ? *reinterpret_cast<const f32x4_t*>(p.lo + n0 + nc + j * 16) : none;
                hi[j] = in ? *reinterpret_cast<const f32x4_t*>(p.hi + n0 + nc + j * 16) : none;
            }
        }
#pragma unroll
        for (int i = 0; i < NA; ++i) {
            if constexpr (G::kPar > 0) ex[i] = reinterpret_cast<const int*>(par)[512 + mr + i * 16];
            else ex[i] = m0 + mr + i * 16 < p.M ? p.e[m0 + mr + i * 16] : 0;
        }
#pragma unroll
        for (int i = 0; i < NA; ++i) {
            bits[i] = 0u;
#pragma unroll
            for (int j = 0; j < NB; ++j)
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    const float v = ldexpf((float)__float_as_int(acc[i][j][q]), ex[i]);
                    const bool inside = (v >= lo[j][q]) && (v < hi[j][q]);
                    if (!inside && n0 + nc + j * 16 < p.N && m0 + mr + i * 16 < p.M) bits[i] |= 1u << (4 * j + q);
                    acc[i][j][q] = 0.0f;
                }
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

    // acc[i][j][q] = C[row m0 + (wm*NA + i)*16 + lane%16][column n0 + (wn*NB + j)*16 + 4*(lane/16) + q]
    const int64_t mw = m0 + wm * NA * 16, nw = n0 + wn * NB * 16;   // this wavefront's corner
    constexpr int CW = NB * 16;                                      // its columns
    if constexpr (EPI == EPI_F32 || EPI == EPI_PART) {
        // 16 rows at a time through LDS, so that a store covers whole lines of a row
        float* chunk = reinterpret_cast<float*>(lds + wave * G::kEpiWave);
        float* C = EPI == EPI_PART ? p.C + (size_t)ks * p.M * p.N : p.C;
#pragma unroll
        for (int i = 0; i < NA; ++i) {
            const int64_t m = mw + i * 16 + frow;
            float rb = 0.0f;
            if (EPI == EPI_F32 && p.bias && m < p.M) rb = td_bf16_to_f32(p.bias[m]);
#pragma unroll
            for (int j = 0; j < NB; ++j) {
                f32x4_t v;
#pragma unroll
                for (int q = 0; q < 4; ++q) v[q] = acc[i][j][q] + rb;
                // (pieces of 16 bytes rotated by the row, against bank conflicts)
                *reinterpret_cast<f32x4_t*>(chunk + frow * CW + (((j * 4 + fp) ^ (frow & (NB * 4 - 1))) * 4)) = v;
            }
            __builtin_amdgcn_wave_barrier();
            auto store = [&](auto add) {
#pragma unroll
                for (int u = 0; u < 16 * CW / 64; ++u) {
                    const int at = u * 64 + lane, row = at / CW, col = at % CW;
                    const float v = chunk[row * CW + (((col >> 2) ^ (row & (NB * 4 - 1))) * 4) + (col & 3)];
                    const int64_t mm = mw + i * 16 + row, nn = nw + col;
                    if (mm < p.M && nn < p.N) C[mm * p.N + nn] = decltype(add)::value ? C[mm * p.N + nn] + v : v;
                }
            };
            if (EPI == EPI_F32 && p.accumulate) store(std::true_type{});
            else store(std::false_type{});
            __builtin_amdgcn_wave_barrier();
        }
    } else {
        // REPAIR: the flagged elements (few) of 16 rows are listed in LDS first and then evaluated 64 at a time:
        // evaluating all accumulators of a lane would run sigma 128 times per wavefront in the largest tile, the
        // list needs about (share flagged) x 128 runs.
        // HIDDEN: sigma(z + b) of every element.
        bf16_t* chunk = reinterpret_cast<bf16_t*>(lds + wave * G::kEpiWave);
        bf16_t* chunk2 = chunk + 16 * CW;                            // REPAIR: the remainders
        uint2* list = reinterpret_cast<uint2*>(lds + wave * G::kEpiWave + 16 * CW * 4);
        float* par = reinterpret_cast<float*>(lds + kWavesPerTile * G::kEpiWave);
        if constexpr (EPI == EPI_REPAIR) {
            for (int c = tid; c < TN; c += 512) {
                const int64_t n = n0 + c < p.N ? n0 + c : p.N - 1;
                par[c] = td_bf16_to_f32(p.bias[n]);
                par[TN + c] = p.slope[n];
                par[2 * TN + c] = p.icept[n];
            }
            __syncthreads();
        }
#pragma unroll
        for (int i = 0; i < NA; ++i) {
            if constexpr (EPI == EPI_REPAIR) {
                // mask: the four lanes of a row and (where the tile holds them) two tile columns make a word of 32 bits
                const int64_t m = mw + i * 16 + frow;
#pragma unroll
                for (int w = 0; w < (NB + 1) / 2; ++w) {
                    uint32_t word = ((bits[i] >> (8 * w)) & 15u) << (4 * fp);
                    if constexpr (NB >= 2) word |= ((bits[i] >> (8 * w + 4)) & 15u) << (4 * fp + 16);
                    word |= __shfl_xor(word, 16);
                    word |= __shfl_xor(word, 32);
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
                const td_u32x4 zero = {0, 0, 0, 0};
                for (int v = lane; v < (p.rest ? 2 : 1) * 16 * CW / 8; v += 64) reinterpret_cast<td_u32x4*>(chunk)[v] = zero;
                __builtin_amdgcn_wave_barrier();
                int total = 0;
#pragma unroll
                for (int j = 0; j < NB; ++j)
#pragma unroll
                    for (int q = 0; q < 4; ++q) {
                        const bool flagged = (bits[i] >> (4 * j + q)) & 1u;
                        const unsigned long long all = __ballot(flagged);
                        if (flagged) {
                            const int at = total + (int)__builtin_amdgcn_mbcnt_hi((uint32_t)(all >> 32),
                                                                                  __builtin_amdgcn_mbcnt_lo((uint32_t)all, 0u));
                            list[at] = make_uint2(__float_as_uint(acc[i][j][q]), (uint32_t)(frow * CW + j * 16 + 4 * fp + q));
                        }
                        total += __popcll(all);
                    }
                __builtin_amdgcn_wave_barrier();
                for (int t = lane; t < total; t += 64) {
                    const uint2 en = list[t];
                    const int c = wn * CW + (int)(en.y % CW);
                    const float z = __uint_as_float(en.x) + par[c];
                    const float factor = td_act(z, p.act) - fmaf(par[TN + c], z, par[2 * TN + c]);
                    const uint32_t head = to_bf16(factor);
                    chunk[en.y] = (bf16_t)head;
                    if (p.rest) {                                     // (infinite and NaN factors are all in the head)
                        const float rest = factor - td_bf16_to_f32((bf16_t)head);
                        chunk2[en.y] = (bf16_t)(fabsf(rest) < INFINITY ? to_bf16(rest) : 0u);
                    }
                }
            } else {
#pragma unroll
                for (int j = 0; j < NB; ++j) {
                    const int64_t n = nw + j * 16 + 4 * fp;
                    uint2 b = make_uint2(0u, 0u);
                    if (n < p.N) b = *reinterpret_cast<const uint2*>(p.bias + n);
                    const float bv[4] = {__uint_as_float(b.x << 16), __uint_as_float(b.x & 0xffff0000u),
                                         __uint_as_float(b.y << 16), __uint_as_float(b.y & 0xffff0000u)};
                    uint32_t o[4];
#pragma unroll
                    for (int q = 0; q < 4; ++q) o[q] = to_bf16(td_act(acc[i][j][q] + bv[q], p.act));
                    *reinterpret_cast<uint2*>(chunk + frow * CW + j * 16 + 4 * fp) = make_uint2(o[0] | (o[1] << 16), o[2] | (o[3] << 16));
                }
            }
            __builtin_amdgcn_wave_barrier();
            for (int v = lane; v < 16 * CW / 8; v += 64) {           // N % 8 == 0: whole 16-byte vectors
                const int row = v / (CW / 8), col = (v % (CW / 8)) * 8;
                const int64_t mm = mw + i * 16 + row, nn = nw + col;
                if (mm < p.M && nn < p.N) {
                    *reinterpret_cast<td_u32x4*>(p.out + mm * p.N + nn) = reinterpret_cast<const td_u32x4*>(chunk)[v];
                    if (EPI == EPI_REPAIR && p.rest)
                        *reinterpret_cast<td_u32x4*>(p.rest + mm * p.N + nn) = reinterpret_cast<const td_u32x4*>(chunk2)[v];
                }
            }
            __builtin_amdgcn_wave_barrier();
        }
    }
}

// The tile for a product: the one whose rounds over 256 CUs cost least.  A block spends per slice either the
// cycles of its MFMAs or those in which the two operand slices arrive, at 34 bytes per cycle and CU.  That rate is a
// chosen number, not a measured bandwidth, and the rule's cycles only rank tiles: they stand for neither the clock under
// load nor HBM (up / output product at 2.1 GHz by the rule, and measured, us: d = 4096, h = 16384, 2048 tokens 199 / 197,
// 378 / 267; 333 tokens 57 / 57, 94 / 71; 64 tokens 23 / 20, 39 / 31; d = 2048, h = 8192, 23 tokens 6 / 6, 17 / 10).
// The larger rate for slices of 256 bytes stands for what the rule does not model: with one row of tiles the weights
// stream from HBM, which delivers longer runs faster (64 tokens, us with 256 / 128 bytes a slice: d = 4096, up
// projection of h = 16384 38.9 / 46.2, of h = 11008 (40 tokens) 33.9 / 44.1, dense 27.4 / 29.0; d = 2048 output product 10.8 /
// 12.1).  `splittable`: K may be cut into 2, 4 or 8 ranges (each then adds the partial tile's bytes, written and read
// again; at most kPartRows rows of partial sums are kept).
constexpr int64_t kPartRows = 4096;
struct TileChoice { int shape, splits; };
constexpr int kShapes = 10;
constexpr int kShapeM[kShapes] = {256, 192, 256, 192, 128, 128, 64, 64, 64, 64},
              kShapeN[kShapes] = {256, 256, 128, 128, 128, 64, 64, 64, 32, 128},
              kShapeSlice[kShapes] = {128, 128, 128, 128, 128, 128, 128, 256, 256, 128};

// whole: K has to be whole slices (of both products); else a ragged K is allowed
TileChoice choose_tile(const GemmArgs& p, bool splittable, bool store_f32, bool whole) {
    TileChoice best{0, 1};
    double best_cost = 1e300;
    const int64_t M = p.M, N = p.N;
    for (int s = 0; s < kShapes; ++s) {
        const int SL = kShapeSlice[s], TM = kShapeM[s], TN = kShapeN[s];
        if (whole && (p.k % SL != 0 || p.k2 % SL != 0)) continue;
        if (TM == 64 && M > 64) continue;
        const int64_t slices = (p.k + SL - 1) / SL + (p.k2 + SL - 1) / SL;
        for (int sp = 1; sp <= (splittable ? 8 : 1); sp *= 2) {
            if (sp > 1 && (slices * SL / sp < 1024 || sp * M > kPartRows)) break;
            const TileMap t = make_tile_map(M, N, TM, TN, (int)slices, sp);
            const int64_t per_xcd = (int64_t)t.rm * t.rn;              // blocks of one XCD (of one range): 32 at once
            const double mfma = 2100.0 / 128.0 * SL * TM * TN / 65536.0;
            const double feed = ((M < TM ? M : TM) + TN) * (double)SL / (SL > 128 ? 34.5 : 34.0);
            const double tail = 3000.0 + (store_f32 ? 0.12 : 0.06) * TM * TN;
            const double cost = (double)((per_xcd + 31) / 32) * ((double)t.slices * (mfma > feed ? mfma : feed) + tail) +
                                (splittable ? sp * (double)M * (double)N * 8.0 / 2000.0 : 0.0);   // partial sums, about 2 KB a cycle
            if (cost < best_cost) { best_cost = cost; best = {s, sp}; }
        }
    }
    return best;
}

// f(slice bytes, wm, na, nb) with the constants of a shape
template <int V> using num = std::integral_constant<int, V>;
template <typename F> void for_shape(int shape, F f) {
    switch (shape) {
        case 0: f(num<128>{}, num<2>{}, num<8>{}, num<4>{}); break;
        case 1: f(num<128>{}, num<2>{}, num<6>{}, num<4>{}); break;
        case 2: f(num<128>{}, num<2>{}, num<8>{}, num<2>{}); break;
        case 3: f(num<128>{}, num<2>{}, num<6>{}, num<2>{}); break;
        case 4: f(num<128>{}, num<2>{}, num<4>{}, num<2>{}); break;
        case 5: f(num<128>{}, num<2>{}, num<4>{}, num<1>{}); break;
        case 6: f(num<128>{}, num<2>{}, num<2>{}, num<1>{}); break;
        case 7: f(num<256>{}, num<2>{}, num<2>{}, num<1>{}); break;
        case 8: f(num<256>{}, num<4>{}, num<1>{}, num<1>{}); break;
        default: f(num<128>{}, num<2>{}, num<2>{}, num<2>{}); break;
    }
}

template <int EPI, bool RAGGED> void launch_ragged(const GemmArgs& p, const TileChoice& c, hipStream_t s) {
    for_shape(c.shape, [&](auto sl, auto wm, auto na, auto nb) {
        typedef GemmTile<EPI, RAGGED, sl, wm, na, nb> G;
        const int slices = (int)((p.k + sl - 1) / sl + (p.k2 + sl - 1) / sl);
        const TileMap tm = make_tile_map(p.M, p.N, G::TM, G::TN, slices, c.splits);
        hipLaunchKernelGGL((gemm_tile_kernel<EPI, RAGGED, sl, wm, na, nb>), dim3(8 * tm.rm * tm.rn), dim3(512), G::kLds, s, p, tm);
    });
}

// EPI_F32 and EPI_PART take any K that is whole 16-byte pieces
template <int EPI> TileChoice launch_tile(const GemmArgs& p, hipStream_t s) {
    constexpr bool may_be_ragged = EPI == EPI_F32 || EPI == EPI_PART;
    const TileChoice c = choose_tile(p, EPI == EPI_PART, may_be_ragged, !may_be_ragged);
    const int sl = kShapeSlice[c.shape];
    if constexpr (may_be_ragged) {
        if (p.k % sl != 0 || p.k2 % sl != 0) {
            launch_ragged<EPI, true>(p, c, s);
            return c;
        }
    }
    launch_ragged<EPI, false>(p, c, s);
    return c;
}

template <int EPI, bool RAGGED> tardis_status_t raise_lds() {
    tardis_status_t st = TARDIS_OK;
    for (int shape = 0; shape < kShapes; ++shape)
        for_shape(shape, [&](auto sl, auto wm, auto na, auto nb) {
            const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(gemm_tile_kernel<EPI, RAGGED, sl, wm, na, nb>),
                                                     hipFuncAttributeMaxDynamicSharedMemorySize,
                                                     GemmTile<EPI, RAGGED, sl, wm, na, nb>::kLds);
            if (e != hipSuccess) st = TARDIS_ERR_HIP;
        });
    return st;
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

// C = A.B^T (+ row_bias), or C += A.B^T.  (A second product is added to the first one's finished sums and not summed
// onto them: partial sums of the first may be far larger than the second.)
tardis_status_t td_gemm_nt(const void* A, const void* B, float* C, int64_t M, int64_t N, int64_t K, int32_t dtype,
                           int accumulate, const void* row_bias, hipStream_t s) {
    if (M <= 0 || N <= 0 || K <= 0) return TARDIS_ERR_SHAPE;
    if (td_gemm_refuses_rows(M)) return TARDIS_ERR_SHAPE;
    // (any M, N work on the matrix cores; small products are not worth it)
    if (dtype == TARDIS_BF16 && M >= 32 && N >= 32 && M * N >= 128 * 128 && K >= 64 && is_aligned16(A) && is_aligned16(B) &&
        K % 8 == 0 && !gemm_force_generic()) {
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

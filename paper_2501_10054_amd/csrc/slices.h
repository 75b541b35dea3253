// Which slice of K a matrix product loads next (gemm_quad_kernel), and from where.  For host and device, so that the offsets can be
// checked against the operands on a CPU.
#pragma once
#include <cstdint>

#ifdef __HIPCC__
#define TD_HD __host__ __device__ __forceinline__
#else
#define TD_HD inline
#endif

typedef int td_i32x4 __attribute__((ext_vector_type(4)));

// The sequence of a block: nk slices from s0 on of the nk1 of the first pair of operands and the nk2 of the second one, each range
// (REPAIR: each pair) from a starting point of its own; k, k2: bytes of a row.
struct td_slices {
    int nk1, nk2, s0, nk, rot, rot2;
    uint32_t k, k2;
};

struct td_slice_source {
    td_i32x4 rs;                          // buffer descriptor
    uint32_t soff, pitch;                 // K offset; bytes of a row
    int t, s;                             // number in the sequence, slice
    bool second;
};

// Step 0 to 5 of finding slice number o.t; r1, r2: descriptors of the operand in the first and in the second pair.  Past the last
// slice nothing is to be fetched: an empty buffer, and no offset either (the hardware compares with num_records - soff, which for an empty
// buffer and another offset may wrap: rows past the operand's end).
template <bool REPAIR, int SL> TD_HD void td_find_slice(td_slice_source& o, const td_slices& q, const td_i32x4& r1, const td_i32x4& r2, int step) {
    if (step == 0) {
        if constexpr (REPAIR) o.s = o.t + (o.t >= q.nk1 ? q.rot2 : q.rot);
        else o.s = o.t + q.rot;
    } else if (step == 1) {
        if constexpr (REPAIR) o.s -= o.t >= q.nk1 ? (o.s >= q.nk1 + q.nk2 ? q.nk2 : 0) : (o.s >= q.nk1 ? q.nk1 : 0);
        else o.s += q.s0 - (o.s >= q.nk ? q.nk : 0);
    } else if (step == 2) {
        o.second = o.s >= q.nk1;
        o.soff = (uint32_t)(o.second ? o.s - q.nk1 : o.s) * SL;
    } else if (step == 3) {
        o.rs.x = o.second ? r2.x : r1.x;
        o.rs.y = o.second ? r2.y : r1.y;
    } else if (step == 4) {
        const bool live = o.t < q.nk;
        const int bytes = o.second ? r2.z : r1.z;
        o.rs.z = live ? bytes : 0;
        o.soff = live ? o.soff : 0u;
        o.pitch = o.second ? q.k2 : q.k;
    } else {
        ++o.t;
    }
}

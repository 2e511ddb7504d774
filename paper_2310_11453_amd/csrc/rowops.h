// Row-wise reduction helpers shared by the quantiser and the LayerNorm backward (gfx950, wave64).
#pragma once
#include "common.h"

namespace bl {

// ---- wave reductions on the DPP path (no LDS traffic) ---------------------------------
// Butterfly inside each row of 16 lanes (xor 1, xor 2, mirror inside 8, mirror inside 16), then
// across rows with the lane-swap instructions: (row 0 + row 1) + (row 2 + row 3) in every lane, so
// every lane ends with the same bits and the result does not depend on the run.  (Reading the four
// row totals back as scalars instead serialises on the vector-to-scalar trips: the four reductions of
// a quantiser's statistics took 0.28 us of a launch.)
template <int CTRL>
__device__ inline int dpp_mov(int v) {
    return __builtin_amdgcn_mov_dpp(v, CTRL, 0xF, 0xF, true);
}
template <int CTRL>
__device__ inline float dpp_mov(float v) {
    return __int_as_float(dpp_mov<CTRL>(__float_as_int(v)));
}
template <int CTRL>
__device__ inline double dpp_mov(double v) {
    return __hiloint2double(dpp_mov<CTRL>(__double2hiint(v)), dpp_mov<CTRL>(__double2loint(v)));
}
// {even rows, odd rows} of v, or {rows 0 and 1, rows 2 and 3}, spread so that combining the two gives
// every lane its share of the butterfly
template <bool HALVES>
__device__ inline void lane_swap(int v, int& lo, int& hi) {
    typedef unsigned v2u __attribute__((ext_vector_type(2)));
    v2u r;
    if constexpr (HALVES) r = __builtin_amdgcn_permlane32_swap((unsigned)v, (unsigned)v, false, false);
    else r = __builtin_amdgcn_permlane16_swap((unsigned)v, (unsigned)v, false, false);
    lo = (int)r[0];
    hi = (int)r[1];
}
template <bool HALVES>
__device__ inline void lane_swap(float v, float& lo, float& hi) {
    int a, b;
    lane_swap<HALVES>(__float_as_int(v), a, b);
    lo = __int_as_float(a);
    hi = __int_as_float(b);
}
template <bool HALVES>
__device__ inline void lane_swap(double v, double& lo, double& hi) {
    int al, bl, ah, bh;
    lane_swap<HALVES>(__double2loint(v), al, bl);
    lane_swap<HALVES>(__double2hiint(v), ah, bh);
    lo = __hiloint2double(ah, al);
    hi = __hiloint2double(bh, bl);
}
struct OpSum {
    template <class T> __device__ T operator()(T a, T b) const { return a + b; }
};
// (the median with an infinity is the maximum or minimum in one instruction: fmaxf and fminf first
// quieten both operands)
struct OpMax {
    __device__ float operator()(float a, float b) const {
        return __builtin_amdgcn_fmed3f(a, b, __builtin_inff());
    }
};
struct OpMin {
    __device__ float operator()(float a, float b) const {
        return __builtin_amdgcn_fmed3f(a, b, -__builtin_inff());
    }
};
template <class T, class Op>
__device__ inline T wave_reduce(T v, Op op) {
    v = op(v, dpp_mov<0xB1>(v));   // quad_perm [1,0,3,2]
    v = op(v, dpp_mov<0x4E>(v));   // quad_perm [2,3,0,1]
    v = op(v, dpp_mov<0x141>(v));  // row_half_mirror
    v = op(v, dpp_mov<0x140>(v));  // row_mirror
    T lo, hi;
    lane_swap<false>(v, lo, hi);
    v = op(lo, hi);
    lane_swap<true>(v, lo, hi);
    return op(lo, hi);
}

// ---- rounding to codes -------------------------------------------------------------------
// clamp(rne(t), LO, 127) as the low byte of the result.  The bounds are integers, so clamping before
// the rounding is the same thing; 1.5 * 2^23 has an ulp of one and is even, so adding it rounds half to
// even and leaves the integer, in two's complement, in the low bits of the mantissa.
template <int LO>
__device__ inline uint32_t code_bits(float t) {
    return __float_as_uint(__builtin_amdgcn_fmed3f(t, (float)LO, 127.f) + 12582912.f);
}
// four codes, the first in the low byte
template <int LO>
__device__ inline uint32_t code_word(float t0, float t1, float t2, float t3) {
    const uint32_t lo = __builtin_amdgcn_perm(code_bits<LO>(t1), code_bits<LO>(t0), 0x0C0C0400u);
    const uint32_t hi = __builtin_amdgcn_perm(code_bits<LO>(t3), code_bits<LO>(t2), 0x04000C0Cu);
    return lo | hi;
}

// N slots in LDS (a power of two up to 16) folded into every lane: each lane reads one of them and a
// butterfly inside the row of 16 lanes does the rest.  One LDS read a wave; reading all the slots in every
// lane kept LDS busy for 0.8 us with 16 waves.
template <int N, class T, class Op>
__device__ inline T fold_slots(const T* slots, Op op) {
    static_assert(N == 1 || N == 2 || N == 4 || N == 8 || N == 16, "inside a row of lanes");
    T v = slots[threadIdx.x & (N - 1)];
    if constexpr (N > 1) v = op(v, dpp_mov<0xB1>(v));
    if constexpr (N > 2) v = op(v, dpp_mov<0x4E>(v));
    if constexpr (N > 4) v = op(v, dpp_mov<0x141>(v));
    if constexpr (N > 8) v = op(v, dpp_mov<0x140>(v));
    return v;
}

// Reduction over the WPR waves that share a row: wave totals meet in LDS.  Every wave of the
// workgroup takes part (rows past M are computed on a clamped row and never stored).  Each
// slot array serves one reduction per kernel, so no barrier is needed ahead of the write.
template <int WPR, class T, class Op>
__device__ inline T row_reduce(T v, Op op, T* slots /* [rows per workgroup][WPR] */, int rw, int wr) {
    v = wave_reduce(v, op);
    if constexpr (WPR == 1) return v;
    if ((threadIdx.x & (kWave - 1)) == 0) slots[rw * WPR + wr] = v;
    __syncthreads();
    return fold_slots<WPR>(slots + rw * WPR, op);
}

}  // namespace bl

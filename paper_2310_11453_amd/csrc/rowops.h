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

// ---- LayerNorm statistics of a row in one pass ---------------------------------------------
// Sums in fp64 of d = x - c and of d^2 about an element c of the row, so that mean = c + sum / K and var =
// E[d^2] - E[d]^2 lose nothing to a large common offset, and the extremes, for the absmax: x -> x^ is
// monotone.  A launch of a few rows is the length of this chain: a wave issues one instruction in four cycles
// whatever its kind (2.5 ns at the clock of such launches), so what counts here is how many there are.
// Elements past the row hold c and add nothing.  The smallest value is kept negated: both are maxima then.
struct RowStats {
    double s = 0.0, q = 0.0;
    float mx, nmn;
};
// the row's own element, or 0 where that is not finite (inf - inf would lose an infinity elsewhere in the row)
__device__ inline float stats_centre(float first) {
    return (__float_as_uint(first) & 0x7f800000u) == 0x7f800000u ? 0.f : first;
}
// plain instructions: fmaxf quietens both operands first, three more instructions each
__device__ inline float max_raw(float a, float b) {
    float r;
    asm("v_max_f32 %0, %1, %2" : "=v"(r) : "v"(a), "v"(b));
    return r;
}
__device__ inline void stats_add(RowStats& st, const float4& v, double c, double (&d)[4]) {
    d[0] = (double)v.x - c;
    d[1] = (double)v.y - c;
    d[2] = (double)v.z - c;
    d[3] = (double)v.w - c;
    st.s += (d[0] + d[1]) + (d[2] + d[3]);
    st.q = fma(d[0], d[0], st.q);
    st.q = fma(d[1], d[1], st.q);
    st.q = fma(d[2], d[2], st.q);
    st.q = fma(d[3], d[3], st.q);
    asm("v_max3_f32 %0, %0, %1, %2\n\tv_max3_f32 %0, %0, %3, %4" : "+v"(st.mx) : "v"(v.x), "v"(v.y), "v"(v.z), "v"(v.w));
    asm("v_max3_f32 %0, %0, -%1, -%2\n\tv_max3_f32 %0, %0, -%3, -%4"
        : "+v"(st.nmn) : "v"(v.x), "v"(v.y), "v"(v.z), "v"(v.w));
}
// The wave's totals with the even lanes carrying the sum and the maximum, the odd ones the sum of squares and the
// negated minimum: two reductions instead of four.  All even lanes hold the same bits, and all odd ones: each step adds
// two values that the two lanes meet in either order.
struct PairStats {
    double k;
    float f;
};
template <int CTRL>
__device__ inline void pair_step(PairStats& p) {
    p.k += dpp_mov<CTRL>(p.k);
    p.f = max_raw(p.f, dpp_mov<CTRL>(p.f));
}
constexpr int kXor1 = 0xB1, kXor2 = 0x4E, kRor4 = 0x124, kRor8 = 0x128;  // DPP: lane ^ 1, lane ^ 2, rotations of 16
constexpr int kEven = 0xA0, kOdd = 0xF5;                                 // the pair's even, odd lane in both
__device__ inline PairStats stats_wave(const RowStats& st) {
    const bool odd = threadIdx.x & 1;
    PairStats p;
    p.k = (odd ? st.q : st.s) + dpp_mov<kXor1>(odd ? st.s : st.q);
    p.f = max_raw(odd ? st.nmn : st.mx, dpp_mov<kXor1>(odd ? st.mx : st.nmn));
    pair_step<kXor2>(p);
    pair_step<kRor8>(p);  // (quads j and j + 2 hold the same bits now, so that the next sum is commuted, not reordered)
    pair_step<kRor4>(p);
    double lo, hi;
    float flo, fhi;
    lane_swap<false>(p.k, lo, hi);
    lane_swap<false>(p.f, flo, fhi);
    p.k = lo + hi;
    p.f = max_raw(flo, fhi);
    lane_swap<true>(p.k, lo, hi);
    lane_swap<true>(p.f, flo, fhi);
    p.k = lo + hi;
    p.f = max_raw(flo, fhi);
    return p;
}
// `parts` waves share the row (a power of two up to 16, uniform): lanes 0 and 1 of each leave their pair in slots
// 2 * part, 2 * part + 1, and behind a barrier every wave folds them.
__device__ inline void stats_leave(const PairStats& p, double* k, float* f, int part) {
    const int l = threadIdx.x & (kWave - 1);
    if (l < 2) {
        k[2 * part + l] = p.k;
        f[2 * part + l] = p.f;
    }
}
__device__ inline PairStats stats_fold(const double* k, const float* f, int parts) {
    const int i = threadIdx.x & (2 * parts - 1);
    PairStats p{k[i], f[i]};
    pair_step<kXor2>(p);
    if (parts > 4) pair_step<kRor8>(p);
    if (parts > 2) pair_step<kRor4>(p);
    if (parts > 8) {
        double lo, hi;
        float flo, fhi;
        lane_swap<false>(p.k, lo, hi);
        lane_swap<false>(p.f, flo, fhi);
        p.k = lo + hi;
        p.f = max_raw(flo, fhi);
    }
    return p;
}
// x^ = fl32(d * rstd + shift), d = x - c
struct RowNorm {
    double rstd, shift;
};
__device__ inline float normalised(const RowNorm& n, double d) { return (float)fma(d, n.rstd, n.shift); }
// 1 / sqrt(v) for v >= 0: the hardware's estimate (a relative error below 2^-22) and one step of third order.  Off by at
// most 0.99 ulp, 0.33 rms, over 2 * 10^7 values in an emulation with estimates of that error; a square root and a
// division, each rounded, are off by up to 1.49 (0.44 rms), and four times the instructions, one after another.
__device__ inline double rsqrt64(double v) {
    const double y = __builtin_amdgcn_rsq(v);
    const double e = fma(-(v * y), y, 1.0);
    const double r = fma(y * e, fma(e, 0.375, 0.5), y);
    return v > 0.0 ? r : y;
}
// inv_k = 1 / K.  lo and hi: the row's smallest and largest x^.
__device__ inline RowNorm stats_finish(const PairStats& p, double c, double inv_k, double eps, float& lo, float& hi) {
    const double dm = dpp_mov<kEven>(p.k) * inv_k;
    const double var = fmax(fma(-dm, dm, dpp_mov<kOdd>(p.k) * inv_k), 0.0);
    RowNorm n;
    n.rstd = rsqrt64(var + eps);
    n.shift = -(dm * n.rstd);
    lo = normalised(n, -(double)dpp_mov<kOdd>(p.f) - c);
    hi = normalised(n, (double)dpp_mov<kEven>(p.f) - c);
    return n;
}

// ---- rounding to codes -------------------------------------------------------------------
// clamp(rne(t), least, 127) as the low byte of the result (least = -128, or 0 for Eq. 6).  The bounds are integers, so
// clamping before the rounding is the same thing; 1.5 * 2^23 has an ulp of one and is even, so adding it rounds half to
// even and leaves the integer, in two's complement, in the low bits of the mantissa.
__device__ inline uint32_t code_bits(float t, float least) {
    return __float_as_uint(__builtin_amdgcn_fmed3f(t, least, 127.f) + 12582912.f);
}
// four codes, the first in the low byte
__device__ inline uint32_t code_word(float t0, float t1, float t2, float t3, float least = -128.f) {
    const uint32_t lo = __builtin_amdgcn_perm(code_bits(t1, least), code_bits(t0, least), 0x0C0C0400u);
    const uint32_t hi = __builtin_amdgcn_perm(code_bits(t3, least), code_bits(t2, least), 0x04000C0Cu);
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

// Fused LayerNorm + absmax + round/clip activation quantiser
// (arXiv 2310.11453, Eq. 12 for LN, Eq. 4-5 for the 8-bit absmax quantiser).
//
// One to eight waves own one token.  The row is read from HBM once and stays in
// registers through the reductions (sum with min/max, then variance) and the
// rounding pass, so the kernel moves 4 bytes in and 1 byte out per element.
// Mean, variance and the normalisation itself are evaluated in fp64 (the
// kernel is bandwidth-bound, the extra ALU work is free) so that the fp32
// value handed to the rounding step is the correctly rounded normalised
// input; the steps that decide a code are single fp32 operations:
//   scale = 128 / gamma,  t = x^ * scale,  code = clamp(rne(t), -128, 127).
#include "common.h"
#include "kernels.h"
#include "rowops.h"

namespace bl {

enum QuantMode { kFull = 0, kStats = 1, kApply = 2 };

// Order-preserving map of floats (any sign) onto unsigned integers and back, so that the
// minimum and maximum over the whole tensor are integers': exact and order-free.
__device__ inline uint32_t float_key(float v) {
    const uint32_t b = __float_as_uint(v);
    return (b & 0x80000000u) ? ~b : (b | 0x80000000u);
}
__device__ inline float key_float(uint32_t k) {
    return __uint_as_float((k & 0x80000000u) ? (k & 0x7fffffffu) : ~k);
}
// Per tensor: the first pass leaves every row's largest magnitude (Eq. 6: its maximum and minimum), as integers of the
// same order, where the codes will be, which nobody writes before the second pass (a row has 32 bytes there or more);
// a launch between the passes folds them.  As atomic maxima on one address, behind a launch that cleared it, rows that
// end together queue, the longer the faster the pass is.  us of a call, atomic / now: 16 x 4096 6.9 / 6.7, 512 x 4096
// 11.5 / 7.8, 8192 x 1024 30.5 / 13.8, 2000 x 4096 25.7 / 13.8, 2000 x 5120 41.0 / 20.1, 8192 x 4096 57.0 / 49.0.
struct Extremes {
    uint32_t *most, *least;
};
__device__ inline Extremes extremes(const QuantArgs& a) {
    uint32_t* const at = reinterpret_cast<uint32_t*>(a.codes);
    return {at, at + a.M};
}
struct OpMaxBits {
    __device__ int operator()(int a, int b) const { return (uint32_t)a > (uint32_t)b ? a : b; }
};
// Workgroup g: the extremes of K-group g, entries g, g + groups, ... of n.
__global__ __launch_bounds__(1024) void fold_extremes(QuantArgs a, uint32_t n) {
    constexpr int NW = 16;
    __shared__ int sm[2][NW];
    const Extremes e = extremes(a);
    const uint32_t step = (uint32_t)a.groups * 1024u;
    int most = 0, least = 0;  // (the minimum's complement)
#pragma unroll 8
    for (uint64_t i = blockIdx.x + (uint64_t)threadIdx.x * (uint32_t)a.groups; i < n; i += step) {
        most = OpMaxBits{}(most, (int)e.most[i]);
        if (a.nonneg) least = OpMaxBits{}(least, (int)~e.least[i]);
    }
    most = wave_reduce(most, OpMaxBits{});
    least = wave_reduce(least, OpMaxBits{});
    if (threadIdx.x % kWave == 0) {
        sm[0][threadIdx.x / kWave] = most;
        sm[1][threadIdx.x / kWave] = least;
    }
    __syncthreads();
    if (threadIdx.x >= kWave) return;
    most = fold_slots<NW>(sm[0], OpMaxBits{});
    least = fold_slots<NW>(sm[1], OpMaxBits{});
    if (threadIdx.x == 0) {
        a.gmax_bits[blockIdx.x] = (uint32_t)most;
        if (a.nonneg) a.gmin_bits[blockIdx.x] = ~(uint32_t)least;
    }
}

// A batch of a few rows is the length of one row's instruction stream (a wave issues one in four cycles, 2.5 ns in a
// graph of short launches): the row's address is scalar, whole pieces of it go without masks, gain, bias and the shift
// of Eq. 6 stand behind one branch each.  us in a layer's two launches, with these in every element's path and the
// address in 64-bit vector arithmetic / now: 8 x 7168 4.2 / 3.4, 8 x 28672 7.7 / 6.7, 16 x 2048 3.4 / 3.2.
// WPR waves share one token (row); a lane holds NV float4 of it.  Workgroups have at least
// four waves, so short rows are handled four (or two) to a workgroup, one per wave, with no
// barrier at all.
// kFull : per-token gamma, everything in one pass.
// kStats: per-tensor, pass 1: the row's statistics to rowstats, its extremes to where the codes will be.
// kApply: per-tensor, pass 2: re-read the row, normalise with the saved stats,
//         quantise with the tensor-wide gamma.
template <int WPR, int NV, int MODE>
__global__ __launch_bounds__((WPR < 4 ? 4 : WPR) * kWave, 4) void ln_quant_rows(QuantArgs a) {
    constexpr int NW = WPR < 4 ? 4 : WPR;  // waves per workgroup
    constexpr int RPW = NW / WPR;          // rows per workgroup
    constexpr int RT = WPR * kWave;        // lanes per row
    __shared__ double sm_k[2 * NW];
    __shared__ float sm_f[2 * NW], smf[2][NW];
    __shared__ int smi[NW];

    // the wave's index, and with it the row and its address, as scalars
    const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x / kWave);
    const int rw = wave / WPR, wr = wave % WPR;
    const int t = wr * kWave + (threadIdx.x & (kWave - 1));
    int64_t row = (int64_t)blockIdx.x * RPW + rw;
    const bool live = row < a.M;
    if constexpr (WPR == 1 && MODE != kStats) {
        if (!live) return;  // no barriers on this path
    } else {
        if (!live) row = a.M - 1;
    }
    const int K4 = (int)(a.K / 4);
    const float* __restrict__ xrow = a.X + row * a.K;
    const float4* __restrict__ x4 = reinterpret_cast<const float4*>(xrow);

    // The loads are unconditional (clamped index, value masked afterwards) so that all of
    // them are in flight before the first is needed.
    float4 v[NV];
#pragma unroll
    for (int j = 0; j < NV; ++j) {
        const int idx = t + j * RT;
        v[j] = x4[(uint32_t)(idx < K4 ? idx : K4 - 1)];
    }
    const float first = *xrow;
    const int grp = a.groups > 1 ? (int)((uint32_t)row % (uint32_t)a.groups) : 0;  // K-group of this row (Eq. 14-15)
    // Each pass over the row converts its elements to fp64 again: `forget` hides the values
    // from the optimiser between passes, or it would keep all the converted copies alive
    // (two registers per element) and the kernel would run at minimal occupancy.
    auto forget = [&]() {
#pragma unroll
        for (int j = 0; j < NV; ++j)
            asm volatile("" : "+v"(v[j].x), "+v"(v[j].y), "+v"(v[j].z), "+v"(v[j].w));
    };
    const bool affine = a.gain != nullptr || a.bias != nullptr;
    bool have_amax = false;
    float amax = 0.f;
    float lo = 0.f, hi_row = 0.f;  // Eq. 6 only: the row's minimum (eta) and maximum; amax = max - min

    if (!a.skip_ln) {
        const float cf = stats_centre(first);
        const double c = (double)cf;
        RowNorm n;
        if constexpr (MODE == kApply) {
            n.shift = a.rowstats[2 * row];
            n.rstd = a.rowstats[2 * row + 1];
        } else {
            RowStats rs;
            rs.mx = cf;
            rs.nmn = -cf;
#pragma unroll
            for (int j = 0; j < NV; ++j) {
                if (K4 < (j + 1) * RT) {  // uniform: this piece of the row is ragged
                    const bool in = t + j * RT < K4;
                    v[j].x = in ? v[j].x : cf;
                    v[j].y = in ? v[j].y : cf;
                    v[j].z = in ? v[j].z : cf;
                    v[j].w = in ? v[j].w : cf;
                }
                double d[4];
                stats_add(rs, v[j], c, d);
            }
            // one barrier for the four values
            PairStats st = stats_wave(rs);
            if constexpr (WPR > 1) {
                stats_leave(st, sm_k, sm_f, wave);
                __syncthreads();
                st = stats_fold(sm_k + 2 * rw * WPR, sm_f + 2 * rw * WPR, WPR);
            }
            float hi;
            n = stats_finish(st, c, a.inv_k, (double)a.eps, lo, hi);
            if constexpr (MODE == kStats) {
                if (t == 0 && live) {
                    a.rowstats[2 * row] = n.shift;
                    a.rowstats[2 * row + 1] = n.rstd;
                }
            }
            if (!affine) {
                // x -> x^ is monotone, so the largest magnitude of the normalised row is reached at the row's
                // minimum or maximum.
                hi_row = hi;
                amax = a.nonneg ? hi - lo : fmaxf(fabsf(lo), fabsf(hi));
                have_amax = true;
            }
        }
        if (MODE != kStats || affine) {
            if constexpr (NV > 4) forget();
#pragma unroll
            for (int j = 0; j < NV; ++j) {  // (elements past the row too: nothing is stored of them)
                v[j].x = normalised(n, (double)v[j].x - c);
                v[j].y = normalised(n, (double)v[j].y - c);
                v[j].z = normalised(n, (double)v[j].z - c);
                v[j].w = normalised(n, (double)v[j].w - c);
            }
            if (affine) {  // uniform
#pragma unroll
                for (int j = 0; j < NV; ++j) {
                    const int idx = t + j * RT;
                    if (idx < K4) {
                        float4 o = v[j];
                        if (a.gain) {
                            const float4 g = reinterpret_cast<const float4*>(a.gain + grp * a.K)[idx];
                            o.x = o.x * g.x; o.y = o.y * g.y; o.z = o.z * g.z; o.w = o.w * g.w;
                        }
                        if (a.bias) {
                            const float4 b = reinterpret_cast<const float4*>(a.bias + grp * a.K)[idx];
                            o.x = o.x + b.x; o.y = o.y + b.y; o.z = o.z + b.z; o.w = o.w + b.w;
                        }
                        v[j] = o;
                    }
                }
            }
        }
    }

    if constexpr (MODE != kStats) {
        if (a.xhat_dump && live) {
            float4* __restrict__ d4 = reinterpret_cast<float4*>(a.xhat_dump + row * a.K);
#pragma unroll
            for (int j = 0; j < NV; ++j) {
                const int idx = t + j * RT;
                if (idx < K4) d4[idx] = v[j];
            }
        }
    }

    float gamma;
    if constexpr (MODE == kApply) {
        if (a.nonneg) {  // Eq. 6 per tensor: eta and gamma from the tensor's extremes
            lo = key_float(a.gmin_bits[grp]);
            gamma = fmaxf(key_float(a.gmax_bits[grp]) - lo, 1e-5f);
        } else {
            gamma = fmaxf(__uint_as_float(a.gmax_bits[grp]), 1e-5f);
        }
    } else {
        if (!have_amax && !a.nonneg) {  // uniform: no LayerNorm, or a gain/bias after it
            float m = 0.f;
#pragma unroll
            for (int j = 0; j < NV; ++j) {
                if (t + j * RT < K4)
                    m = fmaxf(m, fmaxf(fmaxf(fabsf(v[j].x), fabsf(v[j].y)),
                                       fmaxf(fabsf(v[j].z), fabsf(v[j].w))));
            }
            amax = row_reduce<WPR>(m, OpMax{}, smf[0], rw, wr);
        } else if (!have_amax) {  // Eq. 6 on such a row: minimum and maximum of the values
            float mn = v[0].x, mx = v[0].x;  // lane 0's first element always exists
#pragma unroll
            for (int j = 0; j < NV; ++j) {
                if (t + j * RT < K4) {
                    mn = fminf(fminf(mn, v[j].x), fminf(fminf(v[j].y, v[j].z), v[j].w));
                    mx = fmaxf(fmaxf(mx, v[j].x), fmaxf(fmaxf(v[j].y, v[j].z), v[j].w));
                }
            }
            if (t >= K4) {  // a lane without elements must not contribute the padding it holds
                mn = __builtin_inff();
                mx = -__builtin_inff();
            }
            lo = row_reduce<WPR>(mn, OpMin{}, smf[0], rw, wr);
            hi_row = row_reduce<WPR>(mx, OpMax{}, smf[1], rw, wr);
            amax = hi_row - lo;
        }
        if constexpr (MODE == kStats) {
            const Extremes e = extremes(a);
            // Non-negative floats order like their bit patterns.  With one K-group the rows of a workgroup share an
            // entry (a launch of one workgroup folds them: Eq. 6 on 2^20 x 32 689 us with an entry a row, 468 now).
            __shared__ float wg[2][NW];
            if (RPW > 1 && a.groups <= 1) {  // uniform
                if (t == 0) {
                    wg[0][rw] = a.nonneg ? hi_row : amax;  // (rows past the last one repeat it)
                    wg[1][rw] = lo;
                }
                __syncthreads();
                if (threadIdx.x == 0) {
                    float m = wg[0][0], least = wg[1][0];
#pragma unroll
                    for (int i = 1; i < RPW; ++i) {
                        m = fmaxf(m, wg[0][i]);
                        least = fminf(least, wg[1][i]);
                    }
                    e.most[blockIdx.x] = a.nonneg ? float_key(m) : __float_as_uint(m);
                    if (a.nonneg) e.least[blockIdx.x] = float_key(least);
                }
            } else if (t == 0 && live) {
                e.most[row] = a.nonneg ? float_key(hi_row) : __float_as_uint(amax);
                if (a.nonneg) e.least[row] = float_key(lo);
            }
            return;
        }
        gamma = fmaxf(amax, 1e-5f);
    }

    const float scale = 128.0f / gamma;
    int rs = 0;
    uint32_t* __restrict__ c4 = reinterpret_cast<uint32_t*>(a.codes + row * a.K);
    // code = clamp(rne(x^ * scale), -128, 127) (Eq. 6: shifted by eta and clamped to [0, 127])
    if (a.nonneg) {  // uniform
#pragma unroll
        for (int j = 0; j < NV; ++j) {
            v[j].x = v[j].x - lo;
            v[j].y = v[j].y - lo;
            v[j].z = v[j].z - lo;
            v[j].w = v[j].w - lo;
        }
    }
    const float least = a.nonneg ? 0.f : -128.f;
#pragma unroll
    for (int j = 0; j < NV; ++j) {
        const int idx = t + j * RT;
        const float4 x = v[j];
        const uint32_t wd = code_word(x.x * scale, x.y * scale, x.z * scale, x.w * scale, least);
        if (idx < K4) {
            rs = __builtin_amdgcn_sdot4((int)wd, 0x01010101, rs, false);  // sum of the four codes
            if (live) c4[(uint32_t)idx] = wd;
        }
    }
    if (a.rowsum) {
        rs = row_reduce<WPR>(rs, OpSum{}, smi, rw, wr);
        if (t == 0 && live) a.rowsum[row] = rs;
    }
    if (t == 0 && live && (MODE == kFull || row < a.groups)) {  // rows 0 .. groups-1 cover every group
        a.gamma[row] = gamma;
        if (a.nonneg) a.eta[row] = lo;
    }
}

// Rows too long for registers (K > 32768): one workgroup of eight waves per row walks the row
// from memory in each pass (it stays in L2 between passes): sums with minimum and maximum,
// then - only with a gain / bias or without LayerNorm, where the largest magnitude is not at
// the minimum or maximum of the raw row - the absmax of the normalised values, then the
// rounding pass.  The arithmetic per element and the order of the fp32 / fp64 operations that
// decide a code are those of ln_quant_rows; only the summation order of the statistics
// differs (each K is served by exactly one of the two kernels, so results stay deterministic).
template <int MODE>
__global__ __launch_bounds__(512) void ln_quant_long(QuantArgs a) {
    constexpr int NW = 8, T = NW * kWave;
    __shared__ double smd[2][NW];
    __shared__ float smf[4][NW];
    __shared__ int smi[NW];
    const int wave = threadIdx.x / kWave, t = threadIdx.x;
    const bool lead = (threadIdx.x & (kWave - 1)) == 0;
    const int64_t row = blockIdx.x;
    const int64_t K4 = a.K / 4;
    const float4* __restrict__ x4 = reinterpret_cast<const float4*>(a.X + row * a.K);
    const int grp = a.groups > 1 ? (int)(row % a.groups) : 0;
    const bool affine = a.gain != nullptr || a.bias != nullptr;
    bool have_amax = false;
    float amax = 0.f, lo = 0.f, hi_row = 0.f;
    double mu = 0.0, rstd = 1.0;

    if (!a.skip_ln) {
        if constexpr (MODE == kApply) {
            mu = a.rowstats[2 * row];
            rstd = a.rowstats[2 * row + 1];
        } else {
            const double c = (double)a.X[row * a.K];
            double s = 0.0, q = 0.0;
            float mn = a.X[row * a.K], mx = mn;
            for (int64_t idx = t; idx < K4; idx += T) {
                const float4 v = x4[idx];
                const double dx = (double)v.x, dy = (double)v.y, dz = (double)v.z, dw = (double)v.w;
                s += (dx + dy) + (dz + dw);
                q = fma(dx - c, dx - c, q);
                q = fma(dy - c, dy - c, q);
                q = fma(dz - c, dz - c, q);
                q = fma(dw - c, dw - c, q);
                mn = fminf(fminf(mn, v.x), fminf(fminf(v.y, v.z), v.w));
                mx = fmaxf(fmaxf(mx, v.x), fmaxf(fmaxf(v.y, v.z), v.w));
            }
            s = wave_reduce(s, OpSum{});
            q = wave_reduce(q, OpSum{});
            mn = wave_reduce(mn, OpMin{});
            mx = wave_reduce(mx, OpMax{});
            if (lead) {
                smd[0][wave] = s;
                smd[1][wave] = q;
                smf[0][wave] = mn;
                smf[1][wave] = mx;
            }
            __syncthreads();
            s = smd[0][0];
            q = smd[1][0];
            mn = smf[0][0];
            mx = smf[1][0];
#pragma unroll
            for (int i = 1; i < NW; ++i) {
                s += smd[0][i];
                q += smd[1][i];
                mn = fminf(mn, smf[0][i]);
                mx = fmaxf(mx, smf[1][i]);
            }
            mu = s / (double)a.K;
            const double var = fmax(q / (double)a.K - (mu - c) * (mu - c), 0.0);
            rstd = 1.0 / sqrt(var + (double)a.eps);
            if constexpr (MODE == kStats) {
                if (t == 0) {
                    a.rowstats[2 * row] = mu;
                    a.rowstats[2 * row + 1] = rstd;
                }
            }
            if (!affine) {
                lo = (float)(((double)mn - mu) * rstd);
                const float hi = (float)(((double)mx - mu) * rstd);
                hi_row = hi;
                amax = a.nonneg ? hi - lo : fmaxf(fabsf(lo), fabsf(hi));
                have_amax = true;
            }
        }
    }
    // the normalised (and scaled, shifted) values of four consecutive elements
    auto xhat_at = [&](int64_t idx) {
        float4 v = x4[idx];
        if (!a.skip_ln) {
            v.x = (float)(((double)v.x - mu) * rstd);
            v.y = (float)(((double)v.y - mu) * rstd);
            v.z = (float)(((double)v.z - mu) * rstd);
            v.w = (float)(((double)v.w - mu) * rstd);
            if (a.gain) {
                const float4 g = reinterpret_cast<const float4*>(a.gain + grp * a.K)[idx];
                v.x = v.x * g.x; v.y = v.y * g.y; v.z = v.z * g.z; v.w = v.w * g.w;
            }
            if (a.bias) {
                const float4 b = reinterpret_cast<const float4*>(a.bias + grp * a.K)[idx];
                v.x = v.x + b.x; v.y = v.y + b.y; v.z = v.z + b.z; v.w = v.w + b.w;
            }
        }
        return v;
    };
    float gamma;
    if constexpr (MODE == kApply) {
        if (a.nonneg) {
            lo = key_float(a.gmin_bits[grp]);
            gamma = fmaxf(key_float(a.gmax_bits[grp]) - lo, 1e-5f);
        } else {
            gamma = fmaxf(__uint_as_float(a.gmax_bits[grp]), 1e-5f);
        }
    } else {
        if (!have_amax) {  // uniform: minimum and maximum of the values that get rounded
            float mn = __builtin_inff(), mx = -__builtin_inff();
            for (int64_t idx = t; idx < K4; idx += T) {
                const float4 v = xhat_at(idx);
                mn = fminf(fminf(mn, v.x), fminf(fminf(v.y, v.z), v.w));
                mx = fmaxf(fmaxf(mx, v.x), fmaxf(fmaxf(v.y, v.z), v.w));
            }
            mn = wave_reduce(mn, OpMin{});
            mx = wave_reduce(mx, OpMax{});
            if (lead) {
                smf[2][wave] = mn;
                smf[3][wave] = mx;
            }
            __syncthreads();
            mn = smf[2][0];
            mx = smf[3][0];
#pragma unroll
            for (int i = 1; i < NW; ++i) {
                mn = fminf(mn, smf[2][i]);
                mx = fmaxf(mx, smf[3][i]);
            }
            lo = mn;
            hi_row = mx;
            amax = a.nonneg ? mx - mn : fmaxf(fabsf(mn), fabsf(mx));
        }
        if constexpr (MODE == kStats) {
            if (t == 0) {
                const Extremes e = extremes(a);
                e.most[row] = a.nonneg ? float_key(hi_row) : __float_as_uint(amax);
                if (a.nonneg) e.least[row] = float_key(lo);
            }
            return;
        }
        gamma = fmaxf(amax, 1e-5f);
    }
    const float scale = 128.0f / gamma;
    int rs = 0;
    uint32_t* __restrict__ c4 = reinterpret_cast<uint32_t*>(a.codes + row * a.K);
    float4* __restrict__ d4 = a.xhat_dump ? reinterpret_cast<float4*>(a.xhat_dump + row * a.K) : nullptr;
    for (int64_t idx = t; idx < K4; idx += T) {
        const float4 x = xhat_at(idx);
        if (d4) d4[idx] = x;
        const uint32_t wd = a.nonneg ? code_word((x.x - lo) * scale, (x.y - lo) * scale, (x.z - lo) * scale,
                                                 (x.w - lo) * scale, 0.f)
                                     : code_word(x.x * scale, x.y * scale, x.z * scale, x.w * scale);
        rs = __builtin_amdgcn_sdot4((int)wd, 0x01010101, rs, false);
        c4[idx] = wd;
    }
    if (a.rowsum) {
        rs = wave_reduce(rs, OpSum{});
        if (lead) smi[wave] = rs;
        __syncthreads();
        if (t == 0) {
            int r = smi[0];
#pragma unroll
            for (int i = 1; i < NW; ++i) r += smi[i];
            a.rowsum[row] = r;
        }
    }
    if (t == 0 && (MODE == kFull || row < a.groups)) {
        a.gamma[row] = gamma;
        if (a.nonneg) a.eta[row] = lo;
    }
}

// rows of up to 32768 elements stay in registers (16 float4 per lane, up to 8 waves); longer
// ones take ln_quant_long
bool quant_supported(int64_t K) { return K % 4 == 0; }
static bool quant_in_registers(int64_t K) { return K / 4 <= 8 * kWave * 16; }

template <int WPR, int NV>
static void launch_mode(const QuantArgs& a, hipStream_t s) {
    constexpr int NW = WPR < 4 ? 4 : WPR, RPW = NW / WPR;
    const unsigned grid = (unsigned)((a.M + RPW - 1) / RPW);
    if (!a.per_tensor) {
        ln_quant_rows<WPR, NV, kFull><<<grid, NW * kWave, 0, s>>>(a);
    } else {
        const bool shared = RPW > 1 && a.groups <= 1;  // an entry for a workgroup's rows
        ln_quant_rows<WPR, NV, kStats><<<grid, NW * kWave, 0, s>>>(a);
        fold_extremes<<<a.groups, 1024, 0, s>>>(a, shared ? grid : (uint32_t)a.M);
        ln_quant_rows<WPR, NV, kApply><<<grid, NW * kWave, 0, s>>>(a);
    }
}

// Waves per row (up to 16): enough of them that the chip holds about sixteen waves per CU (short rows
// of a small batch are split over several waves rather than leaving most SIMDs idle), and
// never more than 16 float4 per lane.
QuantShape quant_shape(int64_t M, int64_t K, bool per_tensor) {
    const int64_t K4 = K / 4;
    int wpr = 1;
    while (wpr < 8 && K4 > (int64_t)wpr * kWave * 16) wpr *= 2;             // capacity
    while (wpr < 8 && M * wpr < 4096 && K4 >= (int64_t)wpr * 2 * kWave * 4) wpr *= 2;  // occupancy
    // A small batch is the latency of one row: loads, two passes of fp64 per element of a lane, the
    // reductions.  One more doubling, down to two float4 per lane, and 16 waves beyond K = 16384, pay
    // while the batch stays below 2048 waves (us, before / after: 8 x 2048 4.05 / 3.6, 8 x 4096 4.3 / 4.05,
    // 64 x 7168 5.8 / 4.9, 64 x 28672 9.5 / 8.6; 512 x 4096 would go from 6.4 to 6.5, 8 x 16384 with 16
    // waves from 6.1 to 6.35).  Not for short rows with a gamma per tensor from about 128 rows on: a workgroup
    // sends one candidate for the maximum, and half the rows to a workgroup are twice the candidates on
    // one address (both passes, without / with: 512 x 1024 9.2 / 10.2, 333 x 2048 10.1 / 11.8, but 33 x 2048 8.3 / 7.5
    // and 512 x 3072 12.8 / 11.4).
    if (M * wpr * 2 <= 2048 && !(per_tensor && M > 128 && K4 <= 512)) {
        if (wpr < 8 && K4 >= (int64_t)wpr * 2 * kWave * 2) wpr *= 2;
        else if (K4 > 8 * kWave * 8) wpr = 16;
    }
    if (const int v = tuning().quant_wpr)
        if ((v == 1 || v == 2 || v == 4 || v == 8) && K4 <= (int64_t)v * kWave * 16) wpr = v;
    const int64_t per_lane = (K4 + wpr * kWave - 1) / (wpr * kWave);
    int nv = 1;
    while (nv < per_lane) nv *= 2;
    if (wpr > 1 && nv < 2) nv = 2;
    return {wpr, nv};
}

hipError_t launch_quant(const QuantArgs& a_in, hipStream_t s) {
    QuantArgs a = a_in;
    a.inv_k = 1.0 / (double)a.K;
    if (!quant_in_registers(a.K)) {
        const unsigned grid = (unsigned)a.M;
        if (!a.per_tensor) {
            ln_quant_long<kFull><<<grid, 512, 0, s>>>(a);
        } else {
            ln_quant_long<kStats><<<grid, 512, 0, s>>>(a);
            fold_extremes<<<a.groups, 1024, 0, s>>>(a, grid);
            ln_quant_long<kApply><<<grid, 512, 0, s>>>(a);
        }
        return hipGetLastError();
    }
    const QuantShape q = quant_shape(a.M, a.K, a.per_tensor);
    const int wpr = q.wpr, nv = q.nv;
#define BL_QUANT_CASE(W, V) if (wpr == W && nv == V) launch_mode<W, V>(a, s); else
    BL_QUANT_CASE(1, 1) BL_QUANT_CASE(1, 2) BL_QUANT_CASE(1, 4) BL_QUANT_CASE(1, 8) BL_QUANT_CASE(1, 16)
    BL_QUANT_CASE(2, 2) BL_QUANT_CASE(2, 4) BL_QUANT_CASE(2, 8) BL_QUANT_CASE(2, 16)
    BL_QUANT_CASE(4, 2) BL_QUANT_CASE(4, 4) BL_QUANT_CASE(4, 8) BL_QUANT_CASE(4, 16)
    BL_QUANT_CASE(8, 2) BL_QUANT_CASE(8, 4) BL_QUANT_CASE(8, 8) BL_QUANT_CASE(8, 16)
    BL_QUANT_CASE(16, 8)
    return hipErrorInvalidValue;
#undef BL_QUANT_CASE
    return hipGetLastError();
}

}  // namespace bl

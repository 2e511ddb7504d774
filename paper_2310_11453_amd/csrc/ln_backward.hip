// Backward of the LayerNorm in front of the quantiser (arXiv 2310.11453, Eq. 12; per K-group:
// Eq. 15).  Under the straight-through estimator of Section 2.2 the gradient that
// bitlinear_backward_ste returns is the gradient with respect to the LayerNorm output; this
// file takes it to the layer's input x and to the optional gain and bias:
//   xn = (x - mu) * rstd,  gh = g * gain
//   dx = rstd * (gh - mean(gh) - xn * mean(gh * xn))
//   dgain[k] = sum_m g[m,k] * xn[m,k],   dbias[k] = sum_m g[m,k]
// HBM-bound: 8 bytes read and 4 written per element for dx; the gain/bias gradients are a
// second pass over g and x (column sums) and only run when asked for.
#include "common.h"
#include "kernels.h"
#include "rowops.h"

namespace bl {

// Sum over a wave for these kernels: the four row totals are read back as scalars.  Two sums of doubles are
// too few to hide the lane swaps of wave_reduce: 33 to 128 rows of 2048 take 4.3 us this way, 4.6 with those.
template <int CTRL>
__device__ inline double dpp_row(double v) {
    return __hiloint2double(__builtin_amdgcn_update_dpp(0, __double2hiint(v), CTRL, 0xF, 0xF, false),
                            __builtin_amdgcn_update_dpp(0, __double2loint(v), CTRL, 0xF, 0xF, false));
}
__device__ inline double lane_value(double v, int lane) {
    return __hiloint2double(__builtin_amdgcn_readlane(__double2hiint(v), lane),
                            __builtin_amdgcn_readlane(__double2loint(v), lane));
}
__device__ inline double row_sum(double v) {
    v += dpp_row<0xB1>(v);   // quad_perm [1,0,3,2]
    v += dpp_row<0x4E>(v);   // quad_perm [2,3,0,1]
    v += dpp_row<0x141>(v);  // row_half_mirror
    v += dpp_row<0x140>(v);  // row_mirror
    return (lane_value(v, 0) + lane_value(v, 16)) + (lane_value(v, 32) + lane_value(v, 48));
}

// One to eight waves own one row (a token, or one K-group of a token); x and g of the row
// stay in registers (NV float4 per lane each).  Statistics and the two means are fp64, as in
// the forward kernel.  Rows are the consecutive K-element pieces of X, so a K-group of a
// token is simply a row of its own.  STREAM: streaming stores of dX (launch_ln_backward).
template <int WPR, int NV, bool STREAM>
__global__ __launch_bounds__((WPR < 4 ? 4 : WPR) * kWave, 4) void ln_backward_rows(LnBackwardArgs a) {
    constexpr int NW = WPR < 4 ? 4 : WPR;
    constexpr int RT = WPR * kWave;
    __shared__ double smd[4][NW];

    const int wave = threadIdx.x / kWave;
    const int rw = wave / WPR, wr = wave % WPR;
    const int t = wr * kWave + (threadIdx.x & (kWave - 1));
    int64_t row = (int64_t)blockIdx.x * (NW / WPR) + rw;
    const bool live = row < a.M;
    if constexpr (WPR == 1) {
        if (!live) return;  // no barriers on this path
    } else {
        if (!live) row = a.M - 1;
    }
    const int K4 = (int)(a.K / 4);
    const float4* __restrict__ x4 = reinterpret_cast<const float4*>(a.X + row * a.K);
    const float4* g4 = reinterpret_cast<const float4*>(a.g + row * a.K);  // may alias dX
    const int grp = a.groups > 1 ? (int)(row % a.groups) : 0;

    float4 x[NV], g[NV];
#pragma unroll
    for (int j = 0; j < NV; ++j) {
        const int idx = t + j * RT;
        x[j] = x4[idx < K4 ? idx : K4 - 1];
        g[j] = g4[idx < K4 ? idx : K4 - 1];
    }
    if (a.gain) {
        const float4* __restrict__ w4 = reinterpret_cast<const float4*>(a.gain + grp * a.K);
#pragma unroll
        for (int j = 0; j < NV; ++j) {
            const int idx = t + j * RT;
            const float4 w = w4[idx < K4 ? idx : K4 - 1];
            g[j].x *= w.x; g[j].y *= w.y; g[j].z *= w.z; g[j].w *= w.w;
        }
    }

    // mean and variance of the row, one pass, shifted by an element of the row
    const double c = (double)a.X[row * a.K];
    double s = 0.0, q = 0.0;
#pragma unroll
    for (int j = 0; j < NV; ++j) {
        if (t + j * RT < K4) {
            const double dx = (double)x[j].x, dy = (double)x[j].y, dz = (double)x[j].z, dw = (double)x[j].w;
            s += (dx + dy) + (dz + dw);
            q = fma(dx - c, dx - c, q);
            q = fma(dy - c, dy - c, q);
            q = fma(dz - c, dz - c, q);
            q = fma(dw - c, dw - c, q);
        }
    }
    s = row_sum(s);
    q = row_sum(q);
    if constexpr (WPR > 1) {
        if ((threadIdx.x & (kWave - 1)) == 0) {
            smd[0][wave] = s;
            smd[1][wave] = q;
        }
        __syncthreads();
        s = smd[0][rw * WPR];
        q = smd[1][rw * WPR];
#pragma unroll
        for (int i = 1; i < WPR; ++i) {
            s += smd[0][rw * WPR + i];
            q += smd[1][rw * WPR + i];
        }
    }
    const double mu = s / (double)a.K;
    const double var = fmax(q / (double)a.K - (mu - c) * (mu - c), 0.0);
    const double rstd = 1.0 / sqrt(var + (double)a.eps);
    if (a.rowstats && t == 0 && live) {
        a.rowstats[2 * row] = mu;
        a.rowstats[2 * row + 1] = rstd;
    }
    if (!a.dX) return;  // uniform: only the statistics were wanted

    // hide x from the optimiser so that the fp64 copies of the first pass are not kept alive
#pragma unroll
    for (int j = 0; j < NV; ++j) asm volatile("" : "+v"(x[j].x), "+v"(x[j].y), "+v"(x[j].z), "+v"(x[j].w));
    // xn replaces x; c1 = sum gh, c2 = sum gh * xn
    double c1 = 0.0, c2 = 0.0;
#pragma unroll
    for (int j = 0; j < NV; ++j) {
        x[j].x = (float)(((double)x[j].x - mu) * rstd);
        x[j].y = (float)(((double)x[j].y - mu) * rstd);
        x[j].z = (float)(((double)x[j].z - mu) * rstd);
        x[j].w = (float)(((double)x[j].w - mu) * rstd);
        if (t + j * RT < K4) {
            c1 += ((double)g[j].x + (double)g[j].y) + ((double)g[j].z + (double)g[j].w);
            c2 = fma((double)g[j].x, (double)x[j].x, c2);
            c2 = fma((double)g[j].y, (double)x[j].y, c2);
            c2 = fma((double)g[j].z, (double)x[j].z, c2);
            c2 = fma((double)g[j].w, (double)x[j].w, c2);
        }
    }
    c1 = row_sum(c1);
    c2 = row_sum(c2);
    if constexpr (WPR > 1) {
        if ((threadIdx.x & (kWave - 1)) == 0) {
            smd[2][wave] = c1;
            smd[3][wave] = c2;
        }
        __syncthreads();
        c1 = smd[2][rw * WPR];
        c2 = smd[3][rw * WPR];
#pragma unroll
        for (int i = 1; i < WPR; ++i) {
            c1 += smd[2][rw * WPR + i];
            c2 += smd[3][rw * WPR + i];
        }
    }
    const float m1 = (float)(c1 / (double)a.K), m2 = (float)(c2 / (double)a.K);
    const float r = (float)rstd;
    float4* d4 = reinterpret_cast<float4*>(a.dX + row * a.K);
#pragma unroll
    for (int j = 0; j < NV; ++j) {
        const int idx = t + j * RT;
        float4 o;
        o.x = r * ((g[j].x - m1) - x[j].x * m2);
        o.y = r * ((g[j].y - m1) - x[j].y * m2);
        o.z = r * ((g[j].z - m1) - x[j].z * m2);
        o.w = r * ((g[j].w - m1) - x[j].w * m2);
        if (idx < K4 && live) {
            if constexpr (STREAM)
                __builtin_nontemporal_store((v4f){o.x, o.y, o.z, o.w}, reinterpret_cast<v4f*>(d4 + idx));
            else d4[idx] = o;
        }
    }
}

// Rows too long for registers (K / groups > 16384): one workgroup of eight waves per row walks
// the row from memory in each of the three passes (statistics, the two means, dx), the same
// arithmetic per element; x and g of a row stay in L2 between the passes.
__global__ __launch_bounds__(512) void ln_backward_long(LnBackwardArgs a) {
    constexpr int NW = 8, T = NW * kWave;
    __shared__ double smd[4][NW];
    const int wave = threadIdx.x / kWave, t = threadIdx.x;
    const bool lead = (threadIdx.x & (kWave - 1)) == 0;
    const int64_t row = blockIdx.x;
    const int64_t K4 = a.K / 4;
    const float4* __restrict__ x4 = reinterpret_cast<const float4*>(a.X + row * a.K);
    const float4* g4 = reinterpret_cast<const float4*>(a.g + row * a.K);  // may alias dX
    const int grp = a.groups > 1 ? (int)(row % a.groups) : 0;
    const float4* __restrict__ w4 =
        a.gain ? reinterpret_cast<const float4*>(a.gain + grp * a.K) : nullptr;

    const double c = (double)a.X[row * a.K];
    double s = 0.0, q = 0.0;
    for (int64_t idx = t; idx < K4; idx += T) {
        const float4 v = x4[idx];
        const double dx = (double)v.x, dy = (double)v.y, dz = (double)v.z, dw = (double)v.w;
        s += (dx + dy) + (dz + dw);
        q = fma(dx - c, dx - c, q);
        q = fma(dy - c, dy - c, q);
        q = fma(dz - c, dz - c, q);
        q = fma(dw - c, dw - c, q);
    }
    s = row_sum(s);
    q = row_sum(q);
    if (lead) {
        smd[0][wave] = s;
        smd[1][wave] = q;
    }
    __syncthreads();
    s = smd[0][0];
    q = smd[1][0];
#pragma unroll
    for (int i = 1; i < NW; ++i) {
        s += smd[0][i];
        q += smd[1][i];
    }
    const double mu = s / (double)a.K;
    const double var = fmax(q / (double)a.K - (mu - c) * (mu - c), 0.0);
    const double rstd = 1.0 / sqrt(var + (double)a.eps);
    if (a.rowstats && t == 0) {
        a.rowstats[2 * row] = mu;
        a.rowstats[2 * row + 1] = rstd;
    }
    if (!a.dX) return;

    auto load = [&](int64_t idx, float4& xn, float4& gh) {
        const float4 v = x4[idx];
        gh = g4[idx];
        if (w4) {
            const float4 w = w4[idx];
            gh.x *= w.x; gh.y *= w.y; gh.z *= w.z; gh.w *= w.w;
        }
        xn.x = (float)(((double)v.x - mu) * rstd);
        xn.y = (float)(((double)v.y - mu) * rstd);
        xn.z = (float)(((double)v.z - mu) * rstd);
        xn.w = (float)(((double)v.w - mu) * rstd);
    };
    double c1 = 0.0, c2 = 0.0;
    for (int64_t idx = t; idx < K4; idx += T) {
        float4 xn, gh;
        load(idx, xn, gh);
        c1 += ((double)gh.x + (double)gh.y) + ((double)gh.z + (double)gh.w);
        c2 = fma((double)gh.x, (double)xn.x, c2);
        c2 = fma((double)gh.y, (double)xn.y, c2);
        c2 = fma((double)gh.z, (double)xn.z, c2);
        c2 = fma((double)gh.w, (double)xn.w, c2);
    }
    c1 = row_sum(c1);
    c2 = row_sum(c2);
    if (lead) {
        smd[2][wave] = c1;
        smd[3][wave] = c2;
    }
    __syncthreads();  // also: every read of g in the pass above is done before dX (= g) is written
    c1 = smd[2][0];
    c2 = smd[3][0];
#pragma unroll
    for (int i = 1; i < NW; ++i) {
        c1 += smd[2][i];
        c2 += smd[3][i];
    }
    const float m1 = (float)(c1 / (double)a.K), m2 = (float)(c2 / (double)a.K);
    const float r = (float)rstd;
    float4* d4 = reinterpret_cast<float4*>(a.dX + row * a.K);
    for (int64_t idx = t; idx < K4; idx += T) {
        float4 xn, gh, o;
        load(idx, xn, gh);
        o.x = r * ((gh.x - m1) - xn.x * m2);
        o.y = r * ((gh.y - m1) - xn.y * m2);
        o.z = r * ((gh.z - m1) - xn.z * m2);
        o.w = r * ((gh.w - m1) - xn.w * m2);
        d4[idx] = o;
    }
}

// Column sums for the gain and bias gradients.  A workgroup takes 64 float4 columns of the full
// token width (groups * K) and a chunk of tokens; its four waves take every fourth token of the
// chunk (whole 1 KiB lines each) and meet in LDS: fp64 partials per chunk.  Bound by the latency of
// its loads (8 M K bytes, in cache after the statistics pass): the chunks are short enough that
// some 1024 workgroups are in flight, and two tokens of a wave are loaded at once.  M = 1000, K = 2048: 5.1 us;
// in 8 chunks, a thread walking 125 tokens (16 workgroups in all), it took 44.7 us.
constexpr int kAffineWaves = 4;
__global__ __launch_bounds__(256) void ln_backward_affine_partial(LnBackwardArgs a, int64_t tokens,
                                                                  int64_t width, int rows_per_chunk,
                                                                  double* __restrict__ partials) {
    __shared__ double sums[kAffineWaves - 1][kWave][8];
    const int lane = threadIdx.x & (kWave - 1), wave = threadIdx.x / kWave;
    const int64_t c4 = (int64_t)blockIdx.x * kWave + lane;  // float4 column
    const bool in = c4 * 4 < width;
    const int64_t cc = in ? c4 : 0;
    const int grp = (int)(cc * 4 / a.K);
    const int64_t m0 = (int64_t)blockIdx.y * rows_per_chunk;
    const int64_t m1 = m0 + rows_per_chunk < tokens ? m0 + rows_per_chunk : tokens;
    double dg[4] = {0, 0, 0, 0}, db[4] = {0, 0, 0, 0};
#pragma unroll 2
    for (int64_t m = m0 + wave; m < m1; m += kAffineWaves) {
        const float4 x = reinterpret_cast<const float4*>(a.X + m * width)[cc];
        const float4 g = reinterpret_cast<const float4*>(a.g + m * width)[cc];
        const double mu = a.rowstats[2 * (m * a.groups + grp)];
        const double rstd = a.rowstats[2 * (m * a.groups + grp) + 1];
        dg[0] = fma((double)g.x, ((double)x.x - mu) * rstd, dg[0]);
        dg[1] = fma((double)g.y, ((double)x.y - mu) * rstd, dg[1]);
        dg[2] = fma((double)g.z, ((double)x.z - mu) * rstd, dg[2]);
        dg[3] = fma((double)g.w, ((double)x.w - mu) * rstd, dg[3]);
        db[0] += (double)g.x; db[1] += (double)g.y; db[2] += (double)g.z; db[3] += (double)g.w;
    }
    if (wave > 0) {
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            sums[wave - 1][lane][i] = dg[i];
            sums[wave - 1][lane][4 + i] = db[i];
        }
    }
    __syncthreads();
    if (wave > 0 || !in) return;
#pragma unroll
    for (int w = 0; w < kAffineWaves - 1; ++w)
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            dg[i] += sums[w][lane][i];
            db[i] += sums[w][lane][4 + i];
        }
    double* p = partials + ((int64_t)blockIdx.y * 2) * width + c4 * 4;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        p[i] = dg[i];
        p[width + i] = db[i];
    }
}

// A workgroup folds 32 columns: eight threads share a column's chunks and meet in LDS.
__global__ __launch_bounds__(256) void ln_backward_affine_final(const double* __restrict__ partials,
                                                                int chunks, int64_t width,
                                                                float* __restrict__ dgain,
                                                                float* __restrict__ dbias) {
    __shared__ double sums[2][8][32];
    const int col = threadIdx.x & 31, part = threadIdx.x >> 5;
    const int64_t k = (int64_t)blockIdx.x * 32 + col;  // width is a multiple of 32
    double dg = 0.0, db = 0.0;
#pragma unroll 4
    for (int cidx = part; cidx < chunks; cidx += 8) {
        dg += partials[((int64_t)cidx * 2) * width + k];
        db += partials[((int64_t)cidx * 2 + 1) * width + k];
    }
    sums[0][part][col] = dg;
    sums[1][part][col] = db;
    __syncthreads();
    if (part > 1) return;  // thread rows 0 and 1: gain and bias
    double r = sums[part][0][col];
#pragma unroll
    for (int i = 1; i < 8; ++i) r += sums[part][i][col];
    float* const o = part ? dbias : dgain;
    if (o) o[k] = (float)r;
}

bool ln_backward_supported(int64_t K) { return K % 4 == 0; }
static bool ln_backward_in_registers(int64_t K) { return K / 4 <= 8 * kWave * 8; }

// Chunks of tokens of the column sums.  What the workspace must hold at least: 128 tokens a chunk,
// 64 chunks at most.
int ln_backward_min_chunks(int64_t tokens) {
    int64_t c = (tokens + 127) / 128;
    return (int)(c < 1 ? 1 : c > 64 ? 64 : c);
}
// What it is asked for: enough chunks for about 1024 workgroups (`width` / 256 share a chunk), at
// least 16 tokens (four per wave) in each.
int ln_backward_chunks(int64_t tokens, int64_t width) {
    int64_t c = 1024 / ((width + 255) / 256);
    if (c > (tokens + 15) / 16) c = (tokens + 15) / 16;
    const int64_t lo = ln_backward_min_chunks(tokens);
    return (int)(c > 128 ? 128 : c < lo ? lo : c);
}

template <int WPR, int NV>
static void launch_rows(const LnBackwardArgs& a, hipStream_t s) {
    constexpr int NW = WPR < 4 ? 4 : WPR, RPW = NW / WPR;
    // Streaming stores of dX where they pay with a reader behind them, us with a pass over dX: 1000 x 2048 11.9 /
    // 11.3 with them, 333 x 7168 14.2 / 13.0, 1200 x 4096 19.6 / 19.0; but 64 x 2048 6.2 / 6.6, 3000 x 2048 20.8 /
    // 22.4, 8192 x 4096 124 / 128 (there the call by itself 75 / 61, and the reader pays for it).
    const int64_t out = a.M * a.K;
    const auto kernel = out >= (int64_t)1 << 20 && out <= (int64_t)5 << 20 ? ln_backward_rows<WPR, NV, true>
                                                                          : ln_backward_rows<WPR, NV, false>;
    kernel<<<(unsigned)((a.M + RPW - 1) / RPW), NW * kWave, 0, s>>>(a);
}

// a.M counts rows of a.K elements (tokens * groups); a.rowstats must be given when dgain or
// dbias is wanted; `partials` holds at least ln_backward_min_chunks * 2 * width doubles.
hipError_t launch_ln_backward(const LnBackwardArgs& a, float* dgain, float* dbias, double* partials,
                              size_t partials_bytes, hipStream_t s) {
    const int64_t K4 = a.K / 4;
    int wpr = 1;
    while (wpr < 8 && K4 > (int64_t)wpr * kWave * 8) wpr *= 2;
    const int64_t per_lane = (K4 + wpr * kWave - 1) / (wpr * kWave);
    int nv = 1;
    while (nv < per_lane) nv *= 2;
    if (wpr > 1 && nv < 8) nv = 8;
    auto rows = [&](const LnBackwardArgs& r) {
        if (!ln_backward_in_registers(r.K)) {
            ln_backward_long<<<(unsigned)r.M, 512, 0, s>>>(r);
            return true;
        }
#define BL_LNB_CASE(W, V) if (wpr == W && nv == V) launch_rows<W, V>(r, s); else
        BL_LNB_CASE(1, 1) BL_LNB_CASE(1, 2) BL_LNB_CASE(1, 4) BL_LNB_CASE(1, 8)
        BL_LNB_CASE(2, 8) BL_LNB_CASE(4, 8) BL_LNB_CASE(8, 8)
        return false;
#undef BL_LNB_CASE
        return true;
    };
    // The column sums read the rows' statistics, x and g.  The pass that writes dX leaves the statistics too, so it
    // goes first and they need no launch of their own, unless dX lies on x or g: then statistics, sums, dX. us of the
    // call with dgain and dbias, statistics in a launch of their own / with dX: 256 x 1024 12.5 / 9.9, 1000 x 2048
    // 18.4 / 15.1, 3000 x 4096 60.3 / 44.4, 8192 x 4096 157 / 117.
    auto apart = [&](const float* v) {
        const uintptr_t p = (uintptr_t)v, d = (uintptr_t)a.dX, bytes = (uintptr_t)(a.M * a.K) * sizeof(float);
        return d + bytes <= p || p + bytes <= d;
    };
    const bool affine = dgain || dbias, dx_first = a.dX && (!affine || (apart(a.X) && apart(a.g)));
    if (dx_first && !rows(a)) return hipErrorInvalidValue;
    if (affine) {
        LnBackwardArgs st = a;
        st.dX = nullptr;
        if (!dx_first && !rows(st)) return hipErrorInvalidValue;
        const int64_t tokens = a.M / a.groups, width = a.K * a.groups;
        const int64_t room = (int64_t)(partials_bytes / ((size_t)width * 16));
        int chunks = ln_backward_chunks(tokens, width);
        if (chunks > room) chunks = ln_backward_min_chunks(tokens);
        const int rows_per_chunk = (int)((tokens + chunks - 1) / chunks);
        chunks = (int)((tokens + rows_per_chunk - 1) / rows_per_chunk);  // the ones that hold tokens
        dim3 grid((unsigned)((width / 4 + kWave - 1) / kWave), (unsigned)chunks);
        ln_backward_affine_partial<<<grid, 256, 0, s>>>(a, tokens, width, rows_per_chunk, partials);
        ln_backward_affine_final<<<(unsigned)(width / 32), 256, 0, s>>>(partials, chunks, width, dgain,
                                                                         dbias);
    }
    if (a.dX && !dx_first && !rows(a)) return hipErrorInvalidValue;
    return hipGetLastError();
}

}  // namespace bl

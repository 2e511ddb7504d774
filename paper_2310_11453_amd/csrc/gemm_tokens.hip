// One to eight tokens of a short row in one launch: LayerNorm (Eq. 12), the 8-bit absmax quantiser (Eq. 4-5) and the
// 1-bit x 8-bit product with its dequantisation (Eq. 7, Eq. 11) of arXiv 2310.11453, gamma per token.
//
// What bounds the layer at these sizes is launches and their dependent chains, not bytes: a graph node costs 1.6 us
// when it is empty, the stand-alone quantiser of such a batch 3 us more, and its work (a few thousand elements) can be
// repeated by every workgroup while the workgroup's weight tiles are on their way.  So each workgroup loads all rows
// (M * K * 4 bytes, out of L2), requests its tiles behind them (loads return in order), quantises the rows into LDS
// and multiplies. With one or two waves a SIMD the chain's length is the number of instructions of a wave, each four
// cycles whatever its kind: scalars come from the host in 32 bits, the row is requested before anything else is worked
// out, and the bit planes of a tile meet in four accumulators instead of eight. Two and more rows are split over waves
// exactly as the stand-alone quantiser splits them (quant_shape) and every sum runs in its order, so codes, gamma and
// row sums are the same bits as in two launches. us a launch in a graph of such layers, K -> N, one token (the 1300 to
// 2600 instructions of the small-batch kernel with a quantiser in it / here) and two tokens (two launches / here):
// 2048 -> 2048 3.8 / 3.1 and 6.1 / 3.3, 2048 -> 8192 4.1 / 3.3 and 6.4 / 3.6, 8192 -> 2048 5.7 / 4.3 and 8.9 / 6.4,
// 4096 -> 16384 5.6 / 4.8 and 8.7 / 6.1, 7168 -> 28672 12.0 / 10.8, 28672 -> 7168 16.8 / 15.1; eight tokens of 256 ->
// 512 5.1 / 2.8.
#include "common.h"
#include "kernels.h"
#include "rowops.h"

namespace bl {

constexpr int kTokWaves = 8;      // waves of a workgroup
constexpr int kTokRows = 8;       // most tokens
constexpr int kTokCodes = 20480;  // bytes of codes in LDS: rows padded to whole chunks (32768 with eight chunks a wave)

enum TokFlags : uint32_t { kTokSkipLn = 1, kTokOutAcc = 2, kTokRaggedN = 4 };

struct TokArgs {
    const float* x;
    const uint8_t* packed;
    uint32_t row_bytes, K4, TK, tpb;   // K * 4, K / 4, tiles in a row of tiles, rows of tiles a workgroup
    uint32_t part_shift, slot_shift;   // waves to a row, waves to a set of chunks of K (logarithms)
    uint32_t M, N;
    uint32_t last_tile, flags;
    float eps;
    const float* beta;
    double inv_k;
    float* Y;
    const float *gain, *bias;
    int8_t* codes_out;
    float* gamma_out;
    int32_t* rowsum_out;
    float* xhat_out;
};

// P = (row, part of a row) pairs of a wave, NV = float4 of a pair in a lane; C = chunks of K of a wave, T = its rows of
// weight tiles.  Waves that share a set of chunks (8 >> slot_shift of them) take every so-manieth row of tiles.
// Rows of more than four float4 a lane are converted again for the normalisation: their fp64 copies would not fit; with
// eight chunks a wave the operands of a product are read as they are needed.
template <int P, int NV, int C, int T>
__global__ __launch_bounds__(kTokWaves* kWave) void gemm_tokens_kernel(TokArgs a) {
    constexpr bool kKeep = NV <= 4, kActRegs = C < 8;
    __shared__ __attribute__((aligned(16))) uint8_t codes[C < 8 ? kTokCodes : 32768];
    __shared__ __attribute__((aligned(16))) int red[kTokWaves * T * 256];  // [wave][T][64][4]
    __shared__ double sm_k[2 * P * kTokWaves];
    __shared__ float sm_f[2 * P * kTokWaves], sm_amax[P * kTokWaves];
    __shared__ int sm_rs[kTokRows];
    __shared__ float sm_gamma[kTokRows];
    const int w = __builtin_amdgcn_readfirstlane((int)threadIdx.x / kWave), l = threadIdx.x % kWave;
    const int parts = 1 << a.part_shift, RT = kWave << a.part_shift, K4 = (int)a.K4;

    // this wave's pairs: pair w * P + p is part pair % parts of row pair / parts; pairs past the last row repeat it and
    // leave nothing behind
    int row[P], t[P];
    bool live[P];
    float4 v[P][NV];
    float first[P];
#pragma unroll
    for (int p = 0; p < P; ++p) {
        const int pair = w * P + p, r = pair >> a.part_shift;
        live[p] = r < (int)a.M;
        row[p] = live[p] ? r : (int)a.M - 1;
        t[p] = (pair & (parts - 1)) * kWave + l;
        const char* __restrict__ x = reinterpret_cast<const char*>(a.x) + (uint32_t)row[p] * a.row_bytes;
#pragma unroll
        for (int j = 0; j < NV; ++j) {
            const int idx = t[p] + j * RT;
            v[p][j] = *reinterpret_cast<const float4*>(x + (uint32_t)(idx < K4 ? idx : K4 - 1) * 16u);
        }
        first[p] = *reinterpret_cast<const float*>(x);
    }
    // the tiles behind them, without a branch (behind one, the row's arithmetic would wait for them too): a chunk past
    // the end of K is the last one again, masked below, a tile past the workgroup's last one that one, never stored
    const int slots = 1 << a.slot_shift, slot = w & (slots - 1), set = w >> a.slot_shift, sets = kTokWaves >> a.slot_shift;
    const int tk0 = slot * C, TK = (int)a.TK;
    const int tn0 = (int)(blockIdx.x * a.tpb), tn_end = tn0 + (int)a.tpb - 1;
    const int tn_last = tn_end < (int)a.last_tile ? tn_end : (int)a.last_tile;
    const bool multiplies = tk0 < TK && set < (int)a.tpb;  // uniform
    v4i wt[T][C];
    __builtin_amdgcn_sched_barrier(0);
    const uint8_t* __restrict__ lane_base = a.packed + l * 16;
#pragma unroll
    for (int i = 0; i < T; ++i) {
        int tile = tn0 + set + i * sets;
        tile = tile < tn_last ? tile : tn_last;
#pragma unroll
        for (int c = 0; c < C; ++c) {
            const int chunk = tk0 + c < TK ? tk0 + c : TK - 1;
            wt[i][c] = __builtin_nontemporal_load(
                reinterpret_cast<const v4i*>(lane_base + (uint32_t)(tile * TK + chunk) * 1024u));
        }
    }
    __builtin_amdgcn_sched_barrier(0);
    const float beta = a.beta[0];
    if (parts > 1 && threadIdx.x < kTokRows) sm_rs[threadIdx.x] = 0;  // a barrier ahead of the additions
    if (!multiplies) {
#pragma unroll
        for (int i = 0; i < T; ++i) *reinterpret_cast<v4i*>(&red[((w * T + i) * kWave + l) * 4]) = (v4i){0, 0, 0, 0};
    }

    // ---- LayerNorm
    const bool affine = a.gain != nullptr || a.bias != nullptr, skip_ln = a.flags & kTokSkipLn;
    float amax[P];
    if (!skip_ln) {
        PairStats st[P];
        double d[P][kKeep ? NV : 1][4];
        float cf[P];
#pragma unroll
        for (int p = 0; p < P; ++p) {
            cf[p] = stats_centre(first[p]);
            const double c = (double)cf[p];
            RowStats rs;
            rs.mx = cf[p];
            rs.nmn = -cf[p];
#pragma unroll
            for (int j = 0; j < NV; ++j) {
                if (K4 < (j + 1) * RT) {  // uniform: this piece of the row is ragged
                    const bool in = t[p] + j * RT < K4;
                    v[p][j].x = in ? v[p][j].x : cf[p];
                    v[p][j].y = in ? v[p][j].y : cf[p];
                    v[p][j].z = in ? v[p][j].z : cf[p];
                    v[p][j].w = in ? v[p][j].w : cf[p];
                }
                stats_add(rs, v[p][j], c, d[p][kKeep ? j : 0]);
            }
            if constexpr (!kKeep) {  // hidden from the optimiser, which would keep the copies
#pragma unroll
                for (int j = 0; j < NV; ++j)
                    asm volatile("" : "+v"(v[p][j].x), "+v"(v[p][j].y), "+v"(v[p][j].z), "+v"(v[p][j].w));
            }
            st[p] = stats_wave(rs);
        }
        if (parts > 1) {  // uniform
#pragma unroll
            for (int p = 0; p < P; ++p) stats_leave(st[p], sm_k, sm_f, w * P + p);
            __syncthreads();
#pragma unroll
            for (int p = 0; p < P; ++p) {
                const int base = (w * P + p) >> a.part_shift << a.part_shift;
                st[p] = stats_fold(sm_k + 2 * base, sm_f + 2 * base, parts);
            }
        }
#pragma unroll
        for (int p = 0; p < P; ++p) {
            float lo, hi;
            const RowNorm n = stats_finish(st[p], (double)cf[p], a.inv_k, (double)a.eps, lo, hi);
            amax[p] = max_raw(fabsf(lo), fabsf(hi));
#pragma unroll
            for (int j = 0; j < NV; ++j) {
                const double c = (double)cf[p];
                v[p][j].x = normalised(n, kKeep ? d[p][j][0] : (double)v[p][j].x - c);
                v[p][j].y = normalised(n, kKeep ? d[p][j][1] : (double)v[p][j].y - c);
                v[p][j].z = normalised(n, kKeep ? d[p][j][2] : (double)v[p][j].z - c);
                v[p][j].w = normalised(n, kKeep ? d[p][j][3] : (double)v[p][j].w - c);
            }
        }
    }
    // Gain and bias.  Two pairs: all pieces' at once, past the row the last one's, and one butterfly over the parts (one
    // after another, each behind a branch of its own, they are up to 16 trips to L2 in a row: 3 x 2496 -> 16384 9.0 us,
    // 8.2 now, 6.6 without gain and bias).  One pair: piece by piece, so that those past the row cost nothing (1 x
    // 16416 -> 1024 11.8 us, 12.5 at once).
    if constexpr (P == 2) {
        if (affine && !skip_ln) {  // uniform
            float4 gn[P][NV], bs[P][NV];
#pragma unroll
            for (int i = 0; i < P * NV; ++i) {
                const int p = i / NV, j = i % NV, idx = t[p] + j * RT, at = idx < K4 ? idx : K4 - 1;
                if (a.gain) gn[p][j] = reinterpret_cast<const float4*>(a.gain)[at];
                if (a.bias) bs[p][j] = reinterpret_cast<const float4*>(a.bias)[at];
            }
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int i = 0; i < P * NV; ++i) {
                const int p = i / NV, j = i % NV;
                float4& o = v[p][j];
                const float4 g = gn[p][j], b = bs[p][j];
                if (a.gain) {
                    o.x = o.x * g.x; o.y = o.y * g.y; o.z = o.z * g.z; o.w = o.w * g.w;
                }
                if (a.bias) {
                    o.x = o.x + b.x; o.y = o.y + b.y; o.z = o.z + b.z; o.w = o.w + b.w;
                }
            }
        }
    }
    if (affine || skip_ln) {  // uniform
#pragma unroll
        for (int p = 0; p < P; ++p) {
            float mxa = 0.f;
#pragma unroll
            for (int j = 0; j < NV; ++j) {
                const int idx = t[p] + j * RT;
                if (idx < K4) {
                    float4 o = v[p][j];
                    if (P == 1 && a.gain && !skip_ln) {
                        const float4 gn = reinterpret_cast<const float4*>(a.gain)[idx];
                        o.x = o.x * gn.x; o.y = o.y * gn.y; o.z = o.z * gn.z; o.w = o.w * gn.w;
                    }
                    if (P == 1 && a.bias && !skip_ln) {
                        const float4 b = reinterpret_cast<const float4*>(a.bias)[idx];
                        o.x = o.x + b.x; o.y = o.y + b.y; o.z = o.z + b.z; o.w = o.w + b.w;
                    }
                    v[p][j] = o;
                    mxa = fmaxf(mxa, fmaxf(fmaxf(fabsf(o.x), fabsf(o.y)), fmaxf(fabsf(o.z), fabsf(o.w))));
                }
            }
            amax[p] = wave_reduce(mxa, OpMax{});
            if (l == 0) sm_amax[w * P + p] = amax[p];
        }
        if (parts > 1) {  // uniform
            __syncthreads();
#pragma unroll
            for (int p = 0; p < P; ++p) {
                const int base = (w * P + p) >> a.part_shift << a.part_shift;
                if constexpr (P == 1) {
                    for (int i = 0; i < parts; ++i) amax[p] = fmaxf(amax[p], sm_amax[base + i]);
                } else {  // parts is 2, 4 or 8
                    amax[p] = sm_amax[base + (l & (parts - 1))];
                    amax[p] = OpMax{}(amax[p], dpp_mov<kXor1>(amax[p]));
                    if (parts > 2) amax[p] = OpMax{}(amax[p], dpp_mov<kXor2>(amax[p]));
                    if (parts > 4) amax[p] = OpMax{}(amax[p], dpp_mov<kRor4>(amax[p]));
                }
            }
        }
    }

    // ---- codes to LDS (row r: 16-byte slot s at s ^ r, so that the operand reads of the tokens, whose rows are whole
    // chunks apart, fall on different banks); workgroup 0 leaves them in the workspace too
    const bool keep = blockIdx.x == 0;  // uniform
    const int pitch = TK * kChunkK;
#pragma unroll
    for (int p = 0; p < P; ++p) {
        const float gamma = fmaxf(amax[p], 1e-5f);
        const float scale = 128.0f / gamma;
        int rs = 0;
#pragma unroll
        for (int j = 0; j < NV; ++j) {
            const int idx = t[p] + j * RT;
            const float4 x = v[p][j];
            const uint32_t wd = code_word(x.x * scale, x.y * scale, x.z * scale, x.w * scale);
            if (idx < K4 && live[p]) {
                rs = __builtin_amdgcn_sdot4((int)wd, 0x01010101, rs, false);  // sum of the four codes
                *reinterpret_cast<uint32_t*>(codes + row[p] * pitch + ((idx * 4) ^ (row[p] * 16))) = wd;
                if (keep) {
                    reinterpret_cast<uint32_t*>(a.codes_out + (uint32_t)row[p] * (a.row_bytes / 4))[idx] = wd;
                    if (a.xhat_out) reinterpret_cast<float4*>(a.xhat_out)[idx] = x;
                }
            }
        }
        rs = wave_reduce(rs, OpSum{});
        if (l == 0 && live[p]) {
            if (parts > 1)  // (atomicAdd becomes a loop over the wave's lanes, of which only this one is there)
                asm volatile("ds_add_u32 %0, %1\n\ts_waitcnt lgkmcnt(0)"
                             : : "v"((uint32_t)(uintptr_t)&sm_rs[row[p]]), "v"(rs) : "memory");
            else
                sm_rs[row[p]] = rs;
            if (t[p] == 0) sm_gamma[row[p]] = gamma;
        }
    }
    __syncthreads();
    const int m = l & 15, g = l >> 4;
    const int mr = m < (int)a.M ? m : (int)a.M - 1;

    // ---- the product.  A bit plane of a tile is one AND, {0, 2^i} bytes; planes i and i + 4 of the tile and of the
    // tile shifted by 4 meet in one accumulator: 8 sum_k q b = 8 acc_0 + 4 acc_1 + 2 acc_2 + acc_3
    if (multiplies) {
        v4i act[kActRegs ? C : 1][8];
        auto load_act = [&](int c, v4i(&x)[8], int offset) {
            const int chunk = tk0 + c < TK ? tk0 + c : TK - 1;
            const uint8_t* base = codes + mr * pitch + chunk * kChunkK + offset;
            const uint8_t* even = base + (g ^ mr) * 16;
            const uint8_t* odd = base + ((4 + g) ^ mr) * 16;
#pragma unroll
            for (int i = 0; i < 8; ++i) x[i] = *reinterpret_cast<const v4i*>((i & 1 ? odd : even) + (i >> 1) * 128);
        };
        if constexpr (kActRegs) {
#pragma unroll
            for (int c = 0; c < C; ++c) load_act(c, act[c], 0);
        }
        // (the masks in scalar registers: as literals they double the size of the ANDs, and with eight waves a CU the
        // instruction fetch, which two CUs share, is what such code waits for)
        int plane[4] = {0x01010101, 0x02020202, 0x04040404, 0x08080808};
        asm volatile("" : "+s"(plane[0]), "+s"(plane[1]), "+s"(plane[2]), "+s"(plane[3]));
#pragma unroll
        for (int i = 0; i < T; ++i) {
            v4i acc[4];
#pragma unroll
            for (int c = 0; c < C; ++c) {
                const int livem = C > 1 && c ? -(int)(tk0 + c < TK) : -1;
                if constexpr (!kActRegs) {
                    int again = 0;  // an offset that the compiler cannot see through, or it would keep them all
                    asm volatile("" : "+v"(again));
                    load_act(c, act[0], again);
                }
                const v4i hi = wt[i][c] >> 4;
#pragma unroll
                for (int b = 0; b < 8; ++b) {
                    const int mask = plane[b & 3] & livem;
                    const v4i z = {0, 0, 0, 0};
                    acc[b & 3] = __builtin_amdgcn_mfma_i32_16x16x64_i8((b < 4 ? wt[i][c] : hi) & mask,
                                                                      act[kActRegs ? c : 0][b],
                                                                      c == 0 && b < 4 ? z : acc[b & 3], 0, 0, 0);
                }
            }
            v4i sum = acc[0];
#pragma unroll
            for (int b = 1; b < 4; ++b) sum = (sum << 1) + acc[b];
            *reinterpret_cast<v4i*>(&red[((w * T + i) * kWave + l) * 4]) = sum;
        }
    }
    const int rsum = sm_rs[mr];
    const float gm = sm_gamma[mr];
    if (keep && w == 0 && l < (int)a.M) {  // lane l: token l
        a.gamma_out[l] = gm;
        a.rowsum_out[l] = rsum;
    }
    __syncthreads();
    if (w >= (int)a.tpb) return;  // a wave per row of tiles
    const int tile = tn0 + w;
    const uint32_t n = (uint32_t)tile * kTileN + 4 * g;
    const int* part0 = &red[(((w & (sets - 1)) * slots * T + w / sets) * kWave + l) * 4];
    v4i sum = *reinterpret_cast<const v4i*>(part0);
    auto add = [&](auto n_slots) {
        constexpr int S = decltype(n_slots)::value;
        v4i q[S];
#pragma unroll
        for (int i = 1; i < S; ++i) q[i] = *reinterpret_cast<const v4i*>(part0 + i * T * 256);
#pragma unroll
        for (int i = 1; i < S; ++i) sum += q[i];
    };
    if (slots == 8) add(std::integral_constant<int, 8>{});
    else if (slots == 4) add(std::integral_constant<int, 4>{});
    else if (slots == 2) add(std::integral_constant<int, 2>{});
    if (tile > (int)a.last_tile || m >= (int)a.M || n >= a.N) return;
    const v4i pm = (sum >> 2) - rsum;  // sum_k q s = 2 sum_k q b - sum_k q, exact shift
    const float sc = (beta * gm) / 128.0f;
    v4i o;
#pragma unroll
    for (int r = 0; r < 4; ++r) o[r] = a.flags & kTokOutAcc ? pm[r] : __float_as_int((float)pm[r] * sc);
    int* y = reinterpret_cast<int*>(reinterpret_cast<char*>(a.Y) + ((uint32_t)m * a.N + n) * 4u);
    if (!(a.flags & kTokRaggedN)) *reinterpret_cast<v4i*>(y) = o;
    else
        for (int r = 0; r < 4; ++r)
            if (n + r < a.N) y[r] = o[r];
}

namespace {
struct TokensPlan {
    int P, NV, C, T, tpb, wpr, slot_shift;
};
// false: not a shape of this kernel
bool tokens_plan(int64_t M, int64_t K, int64_t N, TokensPlan& p) {
    if (M < 1 || M > kTokRows || K > 32768 || (M > 1 && tuning().quant_wpr)) return false;
    const int64_t TK = tiles_k(K), tpb = (tiles_n(N) + num_cus() - 1) / num_cus();
    if (tpb > 8) return false;
    const QuantShape q = quant_shape(M, K, false);
    p.wpr = q.wpr;
    p.NV = q.nv;
    if (M == 1) {  // all waves on the one row
        p.wpr = 1;
        while (p.wpr < kTokWaves && K / 4 > p.wpr * kWave) p.wpr *= 2;
        p.NV = 1;
        while (p.NV * p.wpr * kWave < K / 4) p.NV *= 2;
    }
    p.P = 1;
    while (p.P * kTokWaves < M * p.wpr) p.P *= 2;
    p.C = TK <= kTokWaves ? 1 : TK <= 2 * kTokWaves ? 2 : TK <= 4 * kTokWaves ? 4 : 8;
    p.slot_shift = 0;
    while ((p.C << p.slot_shift) < TK) ++p.slot_shift;
    const int sets = kTokWaves >> p.slot_shift;
    p.tpb = (int)tpb;
    p.T = (int)((tpb + sets - 1) / sets);
    // Every workgroup repeats the quantiser, so it pays only while one round of workgroups covers N, and while a
    // wave has one or two pairs: each costs 0.7 to 1 us (8 x 1024 -> 1024 with two 4.3 us, 6.0 in two launches; 8 x
    // 2048 -> 2048 with four 7.0 and 6.4, 4 x 4096 -> 4096 with four 6.95 and 6.9).  Two pairs of four pieces are the
    // line: 0.93 to 0.98 of the time of two launches, 1.01 to 1.06 with gain and bias.
    const int most = p.C == 4 ? 2 : p.C == 8 ? 3 : p.P > 1 || p.NV != 2 * p.C ? 4 : 8;
    return p.wpr <= kTokWaves && p.P <= 2 && p.P * p.NV <= (M == 1 ? 16 : 8) && p.T <= most &&
           M * TK * kChunkK <= (p.C < 8 ? kTokCodes : 32768);
}
}  // namespace

bool gemm_tokens_fuses_quant(int64_t M, int64_t K, int64_t N) {
    TokensPlan p;
    return !tuning().decode_nofuse && tokens_plan(M, K, N, p);
}

hipError_t launch_gemm_tokens(const GemmArgs& a, hipStream_t s) {
    TokensPlan p;
    if (!a.x_row || a.eta || (a.per_tensor && a.M > 1) || a.kgroups > 1 || !tokens_plan(a.M, a.K, a.N, p))
        return hipErrorInvalidValue;
    TokArgs t{};
    t.x = a.x_row;
    t.packed = reinterpret_cast<const uint8_t*>(a.packed);
    t.row_bytes = (uint32_t)a.K * 4;
    t.K4 = (uint32_t)a.K / 4;
    t.TK = (uint32_t)tiles_k(a.K);
    t.tpb = (uint32_t)p.tpb;
    t.part_shift = (uint32_t)__builtin_ctz(p.wpr);
    t.slot_shift = (uint32_t)p.slot_shift;
    t.M = (uint32_t)a.M;
    t.N = (uint32_t)a.N;
    t.last_tile = (uint32_t)tiles_n(a.N) - 1;
    t.flags = (a.skip_ln ? kTokSkipLn : 0) | (a.out_acc ? kTokOutAcc : 0) | (a.N % 4 ? kTokRaggedN : 0);
    t.eps = a.ln_eps;
    t.beta = a.beta;
    t.inv_k = 1.0 / (double)a.K;
    t.Y = a.Y;
    t.gain = a.ln_gain;
    t.bias = a.ln_bias;
    t.codes_out = a.codes_out;
    t.gamma_out = a.gamma_out;
    t.rowsum_out = a.rowsum_out;
    t.xhat_out = a.M == 1 ? a.xhat_out : nullptr;
    const unsigned grid = (unsigned)((tiles_n(a.N) + p.tpb - 1) / p.tpb);
#define BL_TOKENS_CASE(PP, VV, CC, TT)                                               \
    if (p.P == PP && p.NV == VV && p.C == CC && p.T == TT) {                          \
        gemm_tokens_kernel<PP, VV, CC, TT><<<grid, kTokWaves * kWave, 0, s>>>(t);     \
        return hipGetLastError();                                                     \
    }
#define BL_TOKENS_TILES(PP, VV, CC) BL_TOKENS_CASE(PP, VV, CC, 1) BL_TOKENS_CASE(PP, VV, CC, 2) BL_TOKENS_CASE(PP, VV, CC, 3) BL_TOKENS_CASE(PP, VV, CC, 4)
    BL_TOKENS_TILES(1, 1, 1) BL_TOKENS_TILES(1, 2, 1) BL_TOKENS_TILES(1, 4, 1) BL_TOKENS_TILES(2, 2, 1)
    BL_TOKENS_TILES(2, 4, 1) BL_TOKENS_TILES(2, 4, 2) BL_TOKENS_TILES(1, 4, 2)
    BL_TOKENS_CASE(1, 2, 1, 5) BL_TOKENS_CASE(1, 2, 1, 6) BL_TOKENS_CASE(1, 2, 1, 7) BL_TOKENS_CASE(1, 2, 1, 8)
    BL_TOKENS_CASE(1, 4, 2, 5) BL_TOKENS_CASE(1, 4, 2, 6) BL_TOKENS_CASE(1, 4, 2, 7) BL_TOKENS_CASE(1, 4, 2, 8)
    BL_TOKENS_CASE(1, 8, 4, 1) BL_TOKENS_CASE(1, 8, 4, 2) BL_TOKENS_CASE(1, 16, 8, 1) BL_TOKENS_CASE(1, 16, 8, 2)
    BL_TOKENS_CASE(1, 16, 8, 3)
#undef BL_TOKENS_TILES
#undef BL_TOKENS_CASE
    return hipErrorInvalidValue;
}

}  // namespace bl

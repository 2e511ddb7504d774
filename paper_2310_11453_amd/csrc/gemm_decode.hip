// 1-bit x 8-bit GEMM + dequantisation for a handful of tokens (M <= 16):
//   Y[m,n] = (sum_k q[m,k] * s[n,k]) * beta * gamma_m / 128     (Eq. 7, Eq. 11)
// of arXiv 2310.11453, with s in {-1,+1} stored 1 bit per weight.
//
// This shape is bound by streaming the packed weights from HBM, and the only
// ALU work the stream can afford is about two VALU operations per 32 weights.
// The kernel therefore never expands a bit to a +-1 byte.  One AND with 0x01010101 << i turns a packed
// dword into four bytes in {0, 2^i} ("bit plane i"); planes i and i + 4, the latter of the dword shifted right by
// four, feed one of four i8 MFMA accumulators, which are folded once per output tile:
//   8 sum_k q b = 8 acc_0 + 4 acc_1 + 2 acc_2 + acc_3   (exact shifts)
//   sum_k q s = 2 * sum_k q b - sum_k q,        s = 2 b - 1
// with sum_k q taken from the quantiser's row sums.
//
// Four accumulators rather than eight, 32-bit scalars ahead of the first load and the epilogue's operands behind the
// last one (a wave issues one instruction in four cycles, and these launches are short): us a launch, before / now, 8
// tokens 2048 -> 8192 3.6 / 3.3, 4096 -> 16384 4.9 / 4.75, 7168 -> 28672 8.5 / 8.4, 16 tokens 9.65 / 9.15.
//
// Work split: a workgroup owns up to T consecutive 16-row weight tiles and all of K;
// wave w of the group owns the K-chunks {w*C .. w*C+C-1} (+ W*C per round) and
// keeps the matching slice of the activation codes in registers as MFMA
// operands, reusing them for every tile.  Partial sums meet in LDS.
#include "common.h"
#include "kernels.h"
#include "rowops.h"

namespace bl {

// C = K-chunks per wave and round, T = weight tiles per workgroup (compile-time bound; `tpb`
// <= T of them are used), MAXT = launch bound.  ONE_ROUND: the waves of the group cover K in a
// single round, so a tile's partial sum goes straight to LDS and no per-tile registers are
// kept - this is what lets a wave keep eight 1 KiB weight loads in flight.
// KGRP (one round, codes from memory): the a.kgroups K-groups of a grouped layer (Eq. 13-15) inside
// one workgroup.  a.K is one group's K; the waves are dealt to the groups (W / kgroups consecutive
// waves each, C chunks of the group's K per wave), every group reads its own columns of the codes
// and its own blob of tiles, and a tile's sums are added per group and written to the group's slice
// of split_ws (2 * sum_k q b, as a K split does), for groups_reduce to dequantise group by group.
// PARKS: the codes may go through LDS (below), eight rows of a KiB a wave where T is less.
template <int C, int T, int MAXT, bool ONE_ROUND, bool KGRP = false, bool PARKS = ONE_ROUND>
__global__ __launch_bounds__(MAXT) void gemm_decode_kernel(GemmArgs a, int tpb) {
    static_assert(!KGRP || ONE_ROUND, "K-groups inside the workgroup: one round");
    constexpr int kStageRows = 8, kRegion = PARKS && T < kStageRows ? kStageRows : T;  // KiB of a wave's part
    __shared__ __attribute__((aligned(16))) int red[(MAXT / kWave) * kRegion * 256];  // [W][T][64][4]
    constexpr int MAXW = MAXT / kWave;
    const int W = blockDim.x / kWave;
    // the wave's index as a scalar: which chunks and tiles it owns is then scalar arithmetic and
    // the tile loads take a scalar base, instead of 64-bit compares and selects in every lane
    const int w = __builtin_amdgcn_readfirstlane((int)threadIdx.x / kWave), l = threadIdx.x % kWave;
    const int m = l & 15, g = l >> 4;
    const bool to_slices = a.split_k || a.kgroups > 1;  // partial sums go to split_ws
    int K = (int)a.K;  // at most 65536 (kMaxGemmK)
    const uint32_t TKp = a.tk_pitch ? (uint32_t)a.tk_pitch : (uint32_t)tiles_k(K);  // tiles per tile row in memory
    // KGRP: waves per K-group, this wave's group and its index inside the group
    const int wpg = KGRP ? W / a.kgroups : W;
    const int gw = KGRP ? w / wpg : 0, wg = KGRP ? w % wpg : w;
    if constexpr (KGRP) {  // this wave's K-group (wave-uniform)
        a.codes += (int64_t)gw * a.K;
        a.packed += (int64_t)gw * a.group_packed;
    } else if (a.kgroups > 1) {  // this workgroup's K-group (uniform)
        a.codes += (int64_t)blockIdx.y * a.K;
        a.packed += (int64_t)blockIdx.y * a.group_packed;
    } else if (a.split_k) {  // this workgroup's slice of K (uniform)
        const int k0 = (int)blockIdx.y * (int)a.split_k;
        a.codes += k0;
        a.packed += (k0 / kChunkK) * 256;
        K = K - k0 < (int)a.split_k ? K - k0 : (int)a.split_k;
    }
    const uint32_t N = (uint32_t)a.N, TN = (uint32_t)tiles_n(a.N), tn0 = blockIdx.x * (uint32_t)tpb;  // N <= 2^30
    const int TK = (int)tiles_k(K);
    const int M = (int)a.M;
    const int mc = m < M ? m : M - 1;
    // beta belongs to the group of output rows that holds a tile (Eq. 13; one group: beta[0])
    auto beta_of = [&](uint32_t tn) {
        if (a.beta_rows >= a.N) return a.beta[0];
        if (tn > TN - 1) tn = TN - 1;
        return a.beta[(int64_t)(tn * kTileN / (uint32_t)a.beta_rows) * a.beta_stride];
    };

    int part[ONE_ROUND ? 1 : T][4];
    if (!ONE_ROUND) {
#pragma unroll
        for (int t = 0; t < T; ++t)
#pragma unroll
            for (int r = 0; r < 4; ++r) part[t][r] = 0;
    }
    // the masks of four bit planes in scalar registers: as literals they double the size of the ANDs
    int plane_mask[4] = {0x01010101, 0x02020202, 0x04040404, 0x08080808};
    asm volatile("" : "+s"(plane_mask[0]), "+s"(plane_mask[1]), "+s"(plane_mask[2]), "+s"(plane_mask[3]));

    const int rounds = ONE_ROUND ? 1 : (TK + W * C - 1) / (W * C);
    for (int rd = 0; rd < rounds; ++rd) {
        const int tk0 = (rd * W + wg) * C;

        // Every load below is unconditional (addresses are clamped instead of guarded): with
        // no branches around them the loads complete in issue order and the MFMAs of tile t
        // wait for tile t only, not for the whole weight stream behind it.
        //
        // activation operand: lane (m, g) holds codes[m][512*tk + 64*i + 16*g .. +15].  Rows
        // m >= M read row M-1 (their outputs are never stored); columns k >= K read the last 16
        // valid bytes (the packed bits there are zero, so they contribute nothing).
        v4i act[C][8];
        auto load_act = [&]() {
            const int8_t* __restrict__ base = a.codes + (uint32_t)mc * (uint32_t)a.ldq;  // at most 16 rows of 4 MiB
            if ((tk0 + C) * kChunkK <= K) {  // uniform: whole chunks, one address
                base += tk0 * kChunkK + 16 * g;
#pragma unroll
                for (int c = 0; c < C; ++c)
#pragma unroll
                    for (int i = 0; i < 8; ++i)
                        act[c][i] = *reinterpret_cast<const v4i*>(base + c * kChunkK + 64 * i);
            } else {
#pragma unroll
                for (int c = 0; c < C; ++c)
#pragma unroll
                    for (int i = 0; i < 8; ++i) {
                        const int k = (tk0 + c) * kChunkK + 64 * i + 16 * g;
                        act[c][i] = *reinterpret_cast<const v4i*>(base + (uint32_t)(k > K - 16 ? K - 16 : k));
                    }
            }
        };
        // One round: the wave's slice of the codes is M rows of C * 512 bytes.  In operand layout a load touches
        // half a line of each row, so L2 serves every line twice, and there are C * 8 of them whatever M is.
        // Instead each row is fetched with one instruction, 16 consecutive bytes a lane (rows past M, up to a whole
        // set of four: row M-1 again), and (below, once the first weight tiles have been requested behind it) parked
        // in the wave's own part of `red`, which holds nothing before the wave's first tile is done, eight rows at a
        // time, and read from there in operand layout.  A row is 1 KiB, so the same 16 bytes of every row would share
        // their banks: the 16-byte slots of row r are stored at slot ^ r.  us a launch, from memory in operand layout
        // (unless the part of `red` that the sums need held the rows) / now: 8 tokens 4096 -> 4096 3.95 / 3.2, 7168 ->
        // 7168 5.4 / 4.5, 8192 -> 2048 5.0 / 3.8, 16 tokens 8192 -> 2048 6.3 / 4.55, 7168 -> 7168 6.4 / 5.3, 16384 ->
        // 4096 10.2 / 6.85.  With 16 waves rows 0 and 1 are sets of their own: one token's launch of several rounds
        // was 14.95 us with four rows loaded for it (9312 -> 28672), 14.2 now; launches of K-groups, shorter, lose by
        // it (4 x 7168 -> 736 in 2 x 2 groups 9.15 us the layer, 9.45).
        // In place where parking is the longer chain: a single chunk of K (16 x 256 -> 512 2.8, 2.45 in place), and
        // with a chunk a wave, few tiles and a second pass of eight rows (parked / in place: 9 x 544 -> 2048 2.99 /
        // 2.61, 16 x 2496 -> 2048 3.69 / 3.34, 9 x 3584 -> 2048 3.77 / 3.55; four tiles, 16 x 2048 -> 16384, 4.03 /
        // 4.17), but for 12 rows and more of four whole chunks or more (12 x 3584 -> 2048 3.78 / 3.94)
        // and for K-groups over 9 to 16 waves (12 x 4736 -> 224 in 2 x 4 groups, the layer, 10.4 / 10.9).
        const bool stage_lane = l < C * 32;
        // one past the last row of the set that starts with row r
        auto rows_end = [](int r) { return MAXT == 1024 && !KGRP && r < 2 ? r + 1 : (r + 4) & ~3; };
        constexpr int kHeld = MAXT == 512 ? 16 : kStageRows;  // rows in registers; 16 waves have room for eight
        v4i rowv[kHeld];
        auto load_rows = [&](int first, int count) {  // rows first, first + 1, ... into rowv[0], ...
            int kl = tk0 * kChunkK + 16 * l;  // this lane's 16 bytes of a row slice
            kl = kl > K - 16 ? K - 16 : kl;
            const int8_t* __restrict__ src = a.codes + kl;
#pragma unroll
            for (int r0 = 0; r0 < kHeld; r0 = rows_end(r0))
                if (r0 < count && first + r0 < M) {  // uniform
#pragma unroll
                    for (int r = r0; r < rows_end(r0); ++r)
                        rowv[r] =
                            *reinterpret_cast<const v4i*>(src + (int64_t)(first + r < M ? first + r : M - 1) * a.ldq);
                }
        };
        const bool long_whole = M >= 12 && K >= 4 * kChunkK && K % kChunkK == 0;
        const bool staged =
            PARKS && (C > 1 || (TK > 1 && (T >= 4 || M <= 8 || long_whole || (KGRP && MAXT == 1024))));  // uniform
        if (staged) load_rows(0, kHeld);
        else load_act();

        // Weight tiles: a software pipeline of depth kDepth per wave.  Asking for everything at
        // once looks attractive for a 4-microsecond stream, but the memory system then returns
        // the requests in no particular order, every wave gets its first tile late and all the
        // MFMA work piles up behind the stream.  With three tiles in flight per wave (~42 KiB per
        // CU, enough to cover the latency) tiles arrive in order and compute overlaps the stream.
        // Tiles past the end re-read the last tile (never stored); chunks past the end are
        // masked to zero arithmetically (no branch around a load).
        constexpr int kDepth = T < 3 ? T : 3;
        v4i wt[T][C];
        // chunk c of this wave: all-ones / all-zeros mask
        int livem[C];
        // tile t of the group lies t*TK KiB after tile 0; tiles past the last valid one
        // (ragged N, or tpb < T) re-read the last valid tile
        const uint32_t tn_end = tn0 + (uint32_t)tpb - 1;
        const uint32_t t_last = (tn_end < TN - 1 ? tn_end : TN - 1) - tn0;
        const uint32_t* wbase[C];
#pragma unroll
        for (int c = 0; c < C; ++c) {
            livem[c] = -(int)(tk0 + c < TK);
            wbase[c] = a.packed + ((uint64_t)tn0 * TKp + (uint32_t)(tk0 + c < TK ? tk0 + c : TK - 1)) * 256 + l * 4;
        }
        const uint32_t tile_stride = TKp * 256;  // dwords
        auto load_tile = [&](int t) {
            const uint32_t off = ((uint32_t)t < t_last ? (uint32_t)t : t_last) * tile_stride;
#pragma unroll
            for (int c = 0; c < C; ++c)  // read once: streaming loads leave L2 to the codes (3-6 %)
                wt[t][c] = __builtin_nontemporal_load(reinterpret_cast<const v4i*>(wbase[c] + off));
        };
#pragma unroll
        for (int t = 0; t < kDepth; ++t) load_tile(t);
        if (staged) {
            uint8_t* stage = reinterpret_cast<uint8_t*>(&red[w * kRegion * 256]);
#pragma unroll
            for (int p = 0; p < 16 / kStageRows; ++p) {
                if (p * kStageRows < M) {  // uniform
                    if (stage_lane) {
#pragma unroll
                        for (int r0 = 0; r0 < kStageRows; r0 = rows_end(r0))
                            if (p * kStageRows + r0 < M) {  // uniform
#pragma unroll
                                for (int r = r0; r < rows_end(r0); ++r)
                                    *reinterpret_cast<v4i*>(stage + r * 1024 + (l ^ r) * 16) =
                                        rowv[kHeld == 16 ? p * kStageRows + r : r];
                            }
                    }
                    if (kHeld == kStageRows && p == 0 && M > kStageRows) load_rows(kStageRows, kStageRows);
                    if (mc / kStageRows == p) {
                        const int rr = mc % kStageRows;
                        // slot 32 c + 4 i + g of row rr: the row number flips bit 2 of it for odd i or for even
                        const uint8_t* even = stage + rr * 1024 + (g ^ rr) * 16;
                        const uint8_t* odd = stage + rr * 1024 + ((4 + g) ^ rr) * 16;
#pragma unroll
                        for (int c = 0; c < C; ++c)
#pragma unroll
                            for (int i = 0; i < 8; ++i)
                                act[c][i] = *reinterpret_cast<const v4i*>((i & 1 ? odd : even) + c * 512 + (i >> 1) * 128);
                    }
                }
            }
        }

#pragma unroll
        for (int t = 0; t < T; ++t) {
            if (t + kDepth < T) load_tile(t + kDepth);
            __builtin_amdgcn_sched_barrier(0);  // keep the request ahead of this tile's MFMAs
            // planes i and i + 4 of the tile and of the tile shifted by 4 meet in one accumulator:
            //   8 sum_k q b = 8 acc_0 + 4 acc_1 + 2 acc_2 + acc_3
            // chunks past the end of K are masked here, at the point of use (masking at the load
            // would tie a wait for the whole stream to the first tile), and inside the plane mask,
            // a scalar: it costs no instruction of its own
            v4i acc[4];
#pragma unroll
            for (int c = 0; c < C; ++c) {
                const v4i high = wt[t][c] >> 4;
#pragma unroll
                for (int i = 0; i < 8; ++i) {
                    const v4i zero = {0, 0, 0, 0};
                    // rows of the MFMA = weights (n), columns = tokens (m)
                    acc[i & 3] = __builtin_amdgcn_mfma_i32_16x16x64_i8(
                        (i < 4 ? wt[t][c] : high) & (plane_mask[i & 3] & livem[c]), act[c][i],
                        c == 0 && i < 4 ? zero : acc[i & 3], 0, 0, 0);
                }
            }
            v4i sum = acc[0];
#pragma unroll
            for (int i = 1; i < 4; ++i) sum = (sum << 1) + acc[i];
            if (ONE_ROUND) {
                *reinterpret_cast<v4i*>(&red[((w * kRegion + t) * kWave + l) * 4]) = sum;
            } else {
#pragma unroll
                for (int r = 0; r < 4; ++r) part[t][r] += sum[r];
            }
            __builtin_amdgcn_sched_barrier(0);
        }
    }
    // the epilogue's operands, on their way while the waves meet
    const float beta_first = beta_of(tn0 + w);
    int rs = 0;
    float gm = 0.f, eta = 0.f;
    if constexpr (!KGRP) {
        rs = a.rowsum[mc * a.gstride];
        gm = a.per_tensor ? a.gamma[0] : a.gamma[mc * a.gstride];
        if (a.eta) eta = a.eta[a.per_tensor ? 0 : mc * a.gstride];
    }

    // cross-wave reduction over K, then the dequantisation epilogue
    if (!ONE_ROUND) {
#pragma unroll
        for (int t = 0; t < T; ++t)
            *reinterpret_cast<v4i*>(&red[((w * kRegion + t) * kWave + l) * 4]) =
                (v4i){part[t][0], part[t][1], part[t][2], part[t][3]};
    }
    __syncthreads();
    if constexpr (KGRP) {
        // (tile, group) pairs are dealt to the waves; a pair's sum runs over the group's waves
        for (int item = w; item < tpb * a.kgroups; item += W) {
            const int t = item % tpb, grp = item / tpb;
            v4i sum = (v4i){0, 0, 0, 0};
            for (int ww = grp * wpg; ww < (grp + 1) * wpg; ++ww)
                sum += *reinterpret_cast<const v4i*>(&red[((ww * kRegion + t) * kWave + l) * 4]);
            const uint32_t tn = tn0 + t, n = tn * kTileN + 4 * g;
            if (tn >= TN || m >= M || n >= N) continue;
            int* p = a.split_ws + (uint64_t)(uint32_t)(grp * M + m) * N + n;
            const v4i h = sum >> 2;
            if ((N & 3) == 0) *reinterpret_cast<v4i*>(p) = h;
            else
                for (int r = 0; r < 4; ++r)
                    if (n + r < N) p[r] = h[r];
        }
        return;
    }
    for (int t = w; t < tpb; t += W) {
        v4i sum = (v4i){0, 0, 0, 0};
        if (MAXW == 8 && W >= 3) {  // uniform
            // four waves' sums at a time, read independently of one another (the regions of absent waves are
            // not read: another wave's is, masked)
#pragma unroll
            for (int w0 = 0; w0 < MAXW; w0 += 4) {
                if (w0 && w0 >= W) break;  // uniform
                v4i p[4];
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    const int ww = w0 + i < W ? w0 + i : W - 1;
                    p[i] = *reinterpret_cast<const v4i*>(&red[((ww * kRegion + t) * kWave + l) * 4]);
                }
#pragma unroll
                for (int i = 0; i < 4; ++i) sum += p[i] & -(int)(w0 + i < W);
            }
        } else {
            // with one or two waves, or with 16, the plain loop is the faster one (from codes 1 x 256 -> 512 2.47 us
            // for 2.56, 1 x 16384 -> 4096 4.4 for 4.7)
            for (int ww = 0; ww < W; ++ww)
                sum += *reinterpret_cast<const v4i*>(&red[((ww * kRegion + t) * kWave + l) * 4]);
        }
        const uint32_t tn = tn0 + t, n = tn * kTileN + 4 * g;
        if (tn >= TN || m >= M || n >= N) continue;
        if (to_slices) {  // partial sum of this K-slice: 2 * sum_k q b, folded by splitk_reduce
            int* p = a.split_ws + (uint64_t)(blockIdx.y * (uint32_t)M + (uint32_t)m) * N + n;
            const v4i h = sum >> 2;
            if ((N & 3) == 0) *reinterpret_cast<v4i*>(p) = h;
            else
                for (int r = 0; r < 4; ++r)
                    if (n + r < N) p[r] = h[r];
            continue;
        }
        const v4i pm = (sum >> 2) - rs;  // sum_k q s = 2 sum_k q b - sum_k q, exact shift
        float* y = a.Y + (uint64_t)(uint32_t)m * N + n;
        if (a.out_acc) {
            int* yi = reinterpret_cast<int*>(y);
            if ((N & 3) == 0) *reinterpret_cast<v4i*>(yi) = pm;
            else
                for (int r = 0; r < 4; ++r)
                    if (n + r < N) yi[r] = pm[r];
        } else {
            const float beta = t == w ? beta_first : beta_of(tn);
            const float sc = (beta * gm) / 128.0f;
            v4f o = {(float)pm[0] * sc, (float)pm[1] * sc, (float)pm[2] * sc, (float)pm[3] * sc};
            if (a.eta) {  // Eq. 6: the shift eta of the activations adds (beta * eta) * sum_k s[n,k]
                const float be = beta * eta;
                for (int r = 0; r < 4; ++r)
                    o[r] = o[r] + be * (float)a.wsum[n + r < N ? n + r : N - 1];
            }
            if ((N & 3) == 0) {
                // not a streaming store: what reads Y next pays more than it gains (2048 -> 2048 and a pass over Y 5.9
                // us, 6.3 streaming; a step of 24 layers of width 1408 at 16 tokens with an addition to every Y 992,
                // 1019 streaming, though 809 and 768 with nothing that reads Y); rows that are no whole lines lose by
                // themselves (8 x 6144 -> 21860 11.3 us, 11.7 streaming)
                *reinterpret_cast<v4f*>(y) = o;
            } else {
                for (int r = 0; r < 4; ++r)
                    if (n + r < N) y[r] = o[r];
            }
        }
    }
}

// Second step of a K split: Y[m,n] = epilogue(sum_s partial[s][m][n] - rowsum[m]).  V consecutive columns a
// thread (V = 4: N % 4 == 0, split_ws and Y 16-byte aligned), rows m = blockIdx.y, + gridDim.y, ...
// With the slices of a small batch this launch is latency: four slices and the row's scales are requested at once, and
// nothing that can be a scalar (the row, and beta while the matrix has one) costs a vector instruction; read one
// after another behind a 64-bit division the launch took 4.0 us at 8 x 7168 and 4.8 at 333 x 2048.
struct FoldArgs {
    const int32_t* sums;
    uint32_t M, N, splits, gstride;
    const int32_t* rowsum;
    const float *gamma, *beta, *eta;
    const int32_t* wsum;
    float* Y;
    int64_t ldy, beta_stride;
    uint32_t beta_rows;
    bool per_tensor, out_acc;
};
template <int V>
__global__ __launch_bounds__(256) void splitk_reduce(FoldArgs a) {
    typedef int vi __attribute__((ext_vector_type(V)));
    typedef float vf __attribute__((ext_vector_type(V)));
    const uint32_t n = (blockIdx.x * blockDim.x + threadIdx.x) * V;
    if (n >= a.N) return;
    const int splits = (int)a.splits;
    const uint64_t stride = (uint64_t)a.M * a.N;
    uint32_t m = blockIdx.y;
    // the first row's slices are on their way before anything else is asked for
    auto slices = [&](int sp, vi(&q)[4]) {
        const int32_t* p = a.sums + ((uint64_t)m * a.N + n);
#pragma unroll
        for (int i = 0; i < 4; ++i)
            q[i] = *reinterpret_cast<const vi*>(p + (uint32_t)(sp + i < splits ? sp + i : splits - 1) * stride);
    };
    vi q[4];
    slices(0, q);
    float beta[V], wsum[V];
#pragma unroll
    for (int c = 0; c < V; ++c) {
        beta[c] = a.beta_rows >= a.N ? a.beta[0] : a.beta[(int64_t)((n + c) / a.beta_rows) * a.beta_stride];
        wsum[c] = a.eta ? (float)a.wsum[n + c] : 0.f;
    }
    while (true) {
        const uint64_t mg = (uint64_t)m * a.gstride;
        const int rs = a.rowsum[mg];
        const float gm = a.gamma[a.per_tensor ? 0 : mg];
        const float eta = *(a.eta ? a.eta + (a.per_tensor ? 0 : mg) : a.gamma);  // (always a valid address)
        __builtin_amdgcn_sched_barrier(0);
        vi sum = {};
        for (int sp = 0;;) {
#pragma unroll
            for (int i = 0; i < 4; ++i) sum += q[i] & -(int)(sp + i < splits);
            sp += 4;
            if (sp >= splits) break;
            slices(sp, q);
        }
        const vi pm = sum - rs;
        if (a.out_acc) {
            *reinterpret_cast<vi*>(reinterpret_cast<int*>(a.Y) + (uint64_t)m * a.ldy + n) = pm;
        } else {
            vf y;
#pragma unroll
            for (int c = 0; c < V; ++c) {
                y[c] = (float)pm[c] * ((beta[c] * gm) / 128.0f);
                if (a.eta) y[c] = y[c] + (beta[c] * eta) * wsum[c];
            }
            *reinterpret_cast<vf*>(a.Y + (uint64_t)m * a.ldy + n) = y;
        }
        m += gridDim.y;
        if (m >= a.M) return;
        slices(0, q);
    }
}

// The same where the slices are the K-groups of a layer (Eq. 13-15): each is dequantised with its own
// beta_g gamma_g / 128 (and shifted by its own eta_g, Eq. 14) and the groups are added in the order 0, 1, ...
// A thread per V columns over the whole output, not a grid row per token: a row's scales are then vector loads
// in flight with the sums; as scalars, group after group, the launch waited for each (16 x 50257 with four
// groups 6.3 us / 8.5, 333 x 2048 5.7 / 7.6, 1254 x 1664 10.3 / 14.3).
template <int V>
__global__ __launch_bounds__(256) void groups_reduce(GemmArgs a) {
    typedef int vi __attribute__((ext_vector_type(V)));
    typedef float vf __attribute__((ext_vector_type(V)));
    const int64_t per_row = a.N / V, idx = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (idx >= a.M * per_row) return;
    const int64_t m = a.M * per_row < (int64_t)1 << 32 ? (uint32_t)idx / (uint32_t)per_row : idx / per_row;
    const int64_t n = (idx - m * per_row) * V;
    const int G = a.kgroups;
    uint32_t bg[V];
#pragma unroll
    for (int c = 0; c < V; ++c)
        bg[c] = ((uint32_t)(n + c) / (uint32_t)a.beta_rows) * (uint32_t)a.beta_stride;
    vf y = {};
    for (int g = 0; g < G; ++g) {
        const vi part = *reinterpret_cast<const vi*>(a.split_ws + ((int64_t)g * a.M + m) * a.N + n);
        const int rs = a.rowsum[m * a.gstride + g];
        const float gm = a.gamma[a.per_tensor ? g : m * a.gstride + g];
        const float eta = a.eta ? a.eta[a.per_tensor ? g : m * a.gstride + g] : 0.f;
#pragma unroll
        for (int c = 0; c < V; ++c) {
            const float beta = a.beta[bg[c] + g];
            float yg = (float)(part[c] - rs) * ((beta * gm) / 128.0f);
            if (a.eta) yg = yg + (beta * eta) * (float)a.wsum[(int64_t)g * a.N + n + c];
            y[c] = g ? yg + y[c] : yg;
        }
    }
    *reinterpret_cast<vf*>(a.Y + m * a.N + n) = y;
}

int num_cus() {
    static int n = 0;
    if (n == 0) {
        int dev = 0;
        hipDeviceProp_t prop;
        if (hipGetDevice(&dev) == hipSuccess && hipGetDeviceProperties(&prop, dev) == hipSuccess)
            n = prop.multiProcessorCount;
        if (n <= 0) n = 256;
    }
    return n;
}

template <int C, int T, int MAXT, bool ONE_ROUND, bool KGRP = false, bool PARKS = ONE_ROUND>
static void launch_one(const GemmArgs& a, int W, int tpb, hipStream_t s) {
    const int64_t TN = tiles_n(a.N);
    const unsigned splits = KGRP ? 1u : a.kgroups > 1 ? (unsigned)a.kgroups
                            : a.split_k ? (unsigned)((a.K + a.split_k - 1) / a.split_k) : 1u;
    const dim3 grid((unsigned)((TN + tpb - 1) / tpb), splits);
    gemm_decode_kernel<C, T, MAXT, ONE_ROUND, KGRP, PARKS><<<grid, W * kWave, 0, s>>>(a, tpb);
}

// one round, up to 8 waves, exactly tpb = 1..8 tiles per group
template <int C, bool KGRP = false>
static void launch_tiles(const GemmArgs& a, int W, int tpb, hipStream_t s) {
    switch (tpb) {
        case 1: launch_one<C, 1, 512, true, KGRP>(a, W, 1, s); break;
        case 2: launch_one<C, 2, 512, true, KGRP>(a, W, 2, s); break;
        case 3: launch_one<C, 3, 512, true, KGRP>(a, W, 3, s); break;
        case 4: launch_one<C, 4, 512, true, KGRP>(a, W, 4, s); break;
        case 5: launch_one<C, 5, 512, true, KGRP>(a, W, 5, s); break;
        case 6: launch_one<C, 6, 512, true, KGRP>(a, W, 6, s); break;
        case 7: launch_one<C, 7, 512, true, KGRP>(a, W, 7, s); break;
        default: launch_one<C, 8, 512, true, KGRP>(a, W, 8, s); break;
    }
}

// K > 16384 with a workspace: split K over workgroups so that every slice takes the one-round
// path with two chunks per wave (at most 16 chunks a slice), and fold the slices afterwards.
size_t gemm_split_ws_bytes(int64_t M, int64_t N, int64_t K) {
    const int64_t TK = tiles_k(K);
    int64_t splits = 0;
    if (M <= 16) {
        if (TK > 32) splits = (TK + 15) / 16;
    } else {  // enough for whichever of the two mid-batch kernels takes the shape
        if (const int64_t per = prefill_split_tiles(M, N, K)) splits = (TK + per - 1) / per;
        if (const int64_t per = stream_split_tiles(M, K)) {
            const int64_t s2 = (TK + per - 1) / per;
            splits = s2 > splits ? s2 : splits;
        }
    }
    return (size_t)splits * (size_t)M * (size_t)N * 4;
}

// Measurement aid: reads `bytes` of device memory the way the small-batch kernel streams its
// weight tiles (16-byte nontemporal loads, a wave takes 1 KiB at a time, the workgroups share the
// range evenly, kDepth loads in flight per lane) and does nothing else.  What such a launch takes
// is the floor for any kernel that has to bring the same bytes in from HBM.
__global__ __launch_bounds__(1024) void read_probe_kernel(const v4i* __restrict__ src, int64_t n16,
                                                          uint32_t* sink) {
    constexpr int kDepth = 4;
    const int64_t per = (n16 + gridDim.x - 1) / gridDim.x;  // 16-byte pieces per workgroup
    const int64_t lo = per * blockIdx.x, hi = lo + per < n16 ? lo + per : n16;
    v4i x = {0, 0, 0, 0};
    for (int64_t i = lo + threadIdx.x; i < hi; i += (int64_t)blockDim.x * kDepth) {
        v4i v[kDepth];
#pragma unroll
        for (int d = 0; d < kDepth; ++d) {
            const int64_t j = i + (int64_t)d * blockDim.x;
            v[d] = __builtin_nontemporal_load(src + (j < hi ? j : hi - 1));
        }
#pragma unroll
        for (int d = 0; d < kDepth; ++d) x ^= v[d];
    }
    // never true for the all-ones pattern no weight blob holds in every lane; keeps the loads alive
    if ((x[0] & x[1] & x[2] & x[3]) == -1 && sink) sink[blockIdx.x] = 1u;
}
hipError_t launch_read_probe(const void* src, size_t bytes, int workgroups, int threads,
                             uint32_t* sink, hipStream_t s) {
    read_probe_kernel<<<(unsigned)workgroups, (unsigned)threads, 0, s>>>(
        reinterpret_cast<const v4i*>(src), (int64_t)(bytes / 16), sink);
    return hipGetLastError();
}

// Four columns a thread from 2^18 outputs on, below that one, which reaches more CUs (us of the layer, one
// column / four: 8 x 28672 -> 7168 19.1 / 19.3, 24 x 16384 -> 4096 19.05 / 19.2, 64 x 7168 -> 7168 22.9 / 22.8,
// 333 x 8192 -> 2048 29.9 / 28.8).
void launch_splitk_reduce(const GemmArgs& a, int splits, hipStream_t s) {
    const bool vec = a.M * a.N >= (1 << 18) && ((a.N | a.ldy) & 3) == 0 &&
                     (((uintptr_t)a.Y | (uintptr_t)a.split_ws) & 15) == 0;
    const int64_t cols = vec ? a.N / 4 : a.N;
    const int threads = vec && a.M * a.N < (1 << 20) ? 64 : 256;
    const dim3 grid((unsigned)((cols + threads - 1) / threads), (unsigned)(a.M < 65535 ? a.M : 65535));
    if (a.kgroups > 1) {
        const unsigned blocks = (unsigned)((a.M * cols + 255) / 256);
        if (vec) groups_reduce<4><<<blocks, 256, 0, s>>>(a);
        else groups_reduce<1><<<blocks, 256, 0, s>>>(a);
        return;
    }
    const FoldArgs f{a.split_ws, (uint32_t)a.M, (uint32_t)a.N, (uint32_t)splits, (uint32_t)a.gstride, a.rowsum, a.gamma,
                     a.beta, a.eta, a.wsum, a.Y, a.ldy ? a.ldy : a.N, a.beta_stride, (uint32_t)a.beta_rows,
                     a.per_tensor, a.out_acc};
    if (vec) splitk_reduce<4><<<grid, threads, 0, s>>>(f);
    else splitk_reduce<1><<<grid, threads, 0, s>>>(f);
}

hipError_t launch_gemm_decode(const GemmArgs& a_in, hipStream_t s) {
    GemmArgs a = a_in;
    const int64_t TN = tiles_n(a.N);
    int64_t TK = tiles_k(a.K);
    int splits = 1;
    const size_t need = gemm_split_ws_bytes(a.M, a.N, a.K);
    if (a.kgroups > 1) {  // one slice per K-group; the caller sized split_ws for it
        if (!a.split_ws || a.split_ws_bytes < (size_t)a.kgroups * a.M * a.N * 4)
            return hipErrorInvalidValue;
        a.split_k = 0;
        // All groups inside a workgroup when their chunks fit the waves of one (up to 8 waves of
        // one or two chunks, or 16 waves with at most two tiles a group); a wave's chunks must
        // lie in one group.  One round of workgroups then covers N as in the plain layer.
        const int64_t V = TK * a.kgroups;  // chunks of all groups
        auto tiles_for = [&](int cap) {
            int tpb = (int)((TN + num_cus() - 1) / num_cus());
            tpb = tpb > cap ? cap : tpb < 1 ? 1 : tpb;
            const int t = tuning().decode_tiles;
            return t >= 1 && t <= cap ? t : tpb;
        };
        bool done = true;
        if (tuning().group_slices) done = false;  // (tests: the K-groups as slices of the grid)
        else if (TK % 2 == 0 && V / 2 <= 8) launch_tiles<2, true>(a, (int)(V / 2), tiles_for(8), s);
        else if (V <= 8) launch_tiles<1, true>(a, (int)V, tiles_for(8), s);
        else if (TK % 2 == 0 && V / 2 <= 16) {
            if (tiles_for(2) <= 1) launch_one<2, 1, 1024, true, true>(a, (int)(V / 2), 1, s);
            else launch_one<2, 2, 1024, true, true>(a, (int)(V / 2), 2, s);
        } else if (V <= 16) {
            // In more than one round of workgroups the codes are read in place: without LDS for eight rows a wave a
            // CU holds two workgroups (the layer, us, parked / in place: 5 x 5504 -> 23296 in 8 x 4 groups 17.1 /
            // 15.2, 14 x 4736 -> 22784 24.0 / 21.0, 16 x 4608 -> 8208 in 1 x 3 13.8 / 13.0; in one round 16 x 4608 ->
            // 8192 11.7 / 11.9, 4 x 7168 -> 736 in 2 x 2 9.2 / 9.7).
            if (tiles_for(2) <= 1) launch_one<1, 1, 1024, true, true>(a, (int)V, 1, s);
            else if (TN <= 2 * num_cus()) launch_one<1, 2, 1024, true, true>(a, (int)V, 2, s);
            else launch_one<1, 2, 1024, true, true, false>(a, (int)V, 2, s);
        } else {
            done = false;
        }
        if (done) {
            launch_splitk_reduce(a, a.kgroups, s);
            return hipGetLastError();
        }
        splits = a.kgroups;  // else: the K-groups as slices of the grid
    } else if (need && a.split_ws && a.split_ws_bytes >= need && !tuning().decode_nosplit) {
        splits = (int)((TK + 15) / 16);
        const int64_t per = (TK + splits - 1) / splits;  // tiles per slice, evenly
        splits = (int)((TK + per - 1) / per);            // slices that actually hold tiles
        a.tk_pitch = a.tk_pitch ? a.tk_pitch : TK;
        a.split_k = per * kChunkK;
        TK = per;
    } else {
        a.split_k = 0;
    }
    // The whole matrix is a few microseconds of HBM time, so the kernel is built to have every
    // byte requested at once: one round of workgroups (about one per CU), each wave asking for
    // all of its weight tiles before the first MFMA.
    auto tiles_per_group = [&](int cap) {
        int tpb = (int)((TN * splits + num_cus() - 1) / num_cus());
        tpb = tpb > cap ? cap : tpb < 1 ? 1 : tpb;
        const int t = tuning().decode_tiles;
        return t >= 1 && t <= cap ? t : tpb;
    };
    if (TK < 8) {
        // K < 4096: one K-chunk per wave, W = TK waves cover K in one round
        const int W = (int)TK;
        const int tpb = tiles_per_group(8);
        launch_tiles<1>(a, W, tpb, s);
    } else if (TK <= 16) {
        // 4096 <= K <= 8192: two chunks per wave (the fold of the bit planes, once per tile and
        // wave, is then shared by two chunks), W = ceil(TK/2) <= 8 waves, one round
        const int W = (int)((TK + 1) / 2);
        const int tpb = tiles_per_group(8);
        launch_tiles<2>(a, W, tpb, s);
    } else if (TK <= 32) {
        // K <= 16384: up to 16 waves of two chunks, one round; 128 registers per lane
        const int W = (int)((TK + 1) / 2);
        const int tpb = tiles_per_group(2);
        if (tpb <= 1) launch_one<2, 1, 1024, true>(a, W, 1, s);
        else launch_one<2, 2, 1024, true>(a, W, 2, s);
    } else {
        // longer K: two chunks per wave and round, up to 16 waves, several rounds
        const int64_t slots = (TK + 1) / 2;
        const int64_t rounds = (slots + 15) / 16;
        const int W = (int)((slots + rounds - 1) / rounds);
        launch_one<2, 1, 1024, false>(a, W, 1, s);
    }
    if (splits > 1) launch_splitk_reduce(a, splits, s);
    return hipGetLastError();
}

}  // namespace bl

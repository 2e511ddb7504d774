// 1-bit x 8-bit GEMM + dequantisation for 17 to 32 tokens, Eq. 7 and Eq. 11 of arXiv 2310.11453,
// built like the small-batch kernel: the packed weights stream from HBM through registers exactly
// once, and the activation codes of all tokens wait for them in registers as MFMA operands.
//
//  * v_mfma_i32_32x32x32_i8 with the WEIGHTS as its row operand (two 16-row packed tiles make
//    32 rows) and the TOKENS as its 32 columns.  A lane's 16-byte load of a packed tile covers 16
//    consecutive k in each of the 8 bit planes; (w >> i) & 0x01010101 turns plane i into {0,1}
//    operand bytes.  The epilogue restores sum_k q s = 2 sum_k q b - sum_k q with the
//    quantiser's row sums.
//  * Wave w of a workgroup owns the 512-chunks w, w + W, ... of K.  Per chunk it reads the codes
//    of all tokens as whole 512-byte rows, turns them into the MFMA's column operands through a
//    staging area of its own in LDS (no other wave touches it, so no barrier), and walks the
//    workgroup's pairs of weight tiles.  The next chunk's codes and tiles are fetched during the
//    MFMAs of this one.
//  * The waves' partial sums meet in LDS by integer atomic adds (order-free), then all threads
//    dequantise and store 16 bytes each.
// Every workgroup reads all M x K codes (from L2), which is why the token count is bounded: at
// more tokens that traffic, not the weight stream, sets the time, and the LDS-tiled mid-batch
// kernel is as fast.  Long K is split over workgroups (second kernel: splitk_reduce) where these are few and the
// caller brought the workspace.

#include "common.h"
#include "kernels.h"
#include "ring.h"

namespace bl {

namespace stream {
constexpr int kTokens = 32;    // columns of the MFMA
constexpr int kMaxPairs = 4;   // pairs of weight tiles per workgroup (the switch below names each count)
constexpr int kPitch = 33;     // ints per weight row in LDS: 32 tokens + 1 (column reads hit every bank)
constexpr int kMaxWaves = 8;
constexpr int kStageRow = 528; // bytes per token in a wave's staging area: 512 + 16, so that the 16-byte
                               // operand reads of 16 tokens at one k fall on different banks
constexpr int kStageBytes = kTokens * kStageRow;
}  // namespace stream

// What the kernel wants to know, in 32 bits (M <= 32, N <= 2^30): 150 instructions stood ahead of a wave's first
// request, most of them 64-bit arithmetic and the scales' addresses, and four waits for arguments.  us a launch,
// before / now, 24 tokens: 2048 -> 8192 4.4 / 4.05, 4096 -> 12288 7.2 / 6.45, 16384 -> 4096 10.6 / 10.15, 7168 -> 28672
// 15.2 / 14.8.
namespace stream {
struct Args {
    const int8_t* codes;
    const uint32_t* packed;
    uint32_t M, N, ldq, TKp, K, split_k, pairs_wg, extra;  // pairs of tile rows: pairs_wg a workgroup, one more in the
                                                           // first `extra`
    uint32_t gstride, beta_rows;
    const float *gamma, *beta, *eta;
    const int32_t *rowsum, *wsum;
    int64_t beta_stride;
    bool per_tensor, out_acc;
    float* Y;
    int32_t* split_ws;
};
}  // namespace stream

// grid.x workgroups share the pairs of tile rows, grid.y = K-slices (a.split_k elements each,
// 0 = one slice).  M <= 32.
__global__ __launch_bounds__(stream::kMaxWaves* kWave) void gemm_stream_kernel(stream::Args a) {
    using namespace stream;
    __shared__ int red[kMaxPairs * 32 * kPitch];
    // per wave: one chunk of the codes of 32 tokens on its way from row-major memory (read as
    // whole 512-byte rows) to the MFMA's operand layout (16-byte pieces of 32 tokens at one k)
    __shared__ __attribute__((aligned(16))) uint8_t stage[kMaxWaves * kStageBytes];
    __shared__ int tok_sum[kWave];
    __shared__ float tok_gamma[kWave], tok_eta[kWave];

    // all of the arguments that the first requests need at once, not as the branches come to them
    asm volatile(""
                 : "+s"(a.M), "+s"(a.N), "+s"(a.ldq), "+s"(a.TKp), "+s"(a.K),
                   "+s"(a.split_k), "+s"(a.pairs_wg), "+s"(a.extra));
    const int W = (int)blockDim.x / kWave;
    const int w = __builtin_amdgcn_readfirstlane((int)threadIdx.x / kWave), l = threadIdx.x % kWave;
    const int tok = l & 31, half = l >> 5;
    const int M = (int)a.M, N = (int)a.N;
    const int sp = (int)blockIdx.y;
    int k0 = 0, K = (int)a.K;  // ldq < 2^22, M <= 32: offsets into the codes fit 32 bits
    if (a.split_k) {
        k0 = sp * (int)a.split_k;
        K = K - k0 < (int)a.split_k ? K - k0 : (int)a.split_k;
    }
    const int TK = (int)((uint32_t)(K + kChunkK - 1) / kChunkK);

    // this workgroup's pairs of tile rows
    const uint32_t wg = blockIdx.x;
    const int p0 = (int)(wg * a.pairs_wg + (wg < a.extra ? wg : a.extra));
    const int np = (int)(a.pairs_wg + (wg < a.extra ? 1 : 0));  // 1 .. kMaxPairs (the launcher sees to it)

    const bool one_beta = a.beta_rows >= a.N;
    auto clear_sums = [&]() {  // every thread, once: it synchronises
        for (int i = threadIdx.x; i < np * 32 * kPitch; i += blockDim.x) red[i] = 0;
        // Factors of the epilogue, straight into LDS, so that nothing waits on a load of theirs: a token's by wave 0.
        // Neither they nor the clearing of the sums stand ahead of the first chunk's requests: 64-bit divisions,
        // products and a barrier behind the factors' loads were 1.5 us of a launch.
        if (w == 0 && !a.split_k) {
            const uint32_t m = (uint32_t)(l < M ? l : M - 1) * a.gstride, mg = a.per_tensor ? 0 : m;
            auto to_lds = [](const void* src, void* dst) {
                __builtin_amdgcn_global_load_lds(src, (__attribute__((address_space(3))) void*)dst, 4, 0, 0);
            };
            to_lds(a.rowsum + m, tok_sum);
            to_lds(a.gamma + mg, tok_gamma);
            if (a.eta) to_lds(a.eta + mg, tok_eta);
        }
        // a bare barrier behind the LDS writes: a fence would also wait for the chunk's loads
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
        block_barrier();
    };

    // lane -> weight row (tok is also the row index of the A operand) and its 16-byte slot:
    // tile 2p + row/16, slot (2 mf + half) * 16 + row % 16
    const int wrow = tok;
    const uint32_t slot_dw = (uint32_t)((half * 16 + (wrow & 15)) * 4);  // + 128 dwords for mf = 1
    // uniform bases, 32-bit offsets (a tile row is at most 128 KiB here, a row of codes less than 4 MiB)
    const uint32_t* const wbase = a.packed + ((uint64_t)(uint32_t)(2 * p0) * a.TKp + (uint32_t)k0 / kChunkK) * 256;
    const int8_t* const cbase = a.codes + (uint32_t)k0;
    const int last_row = (int)((a.N + kTileN - 1) / kTileN - 1) - 2 * p0;  // rows behind it are never stored
    auto pair_off = [&](int p) {
        const int row = 2 * p + (wrow >> 4);
        return __umul24((uint32_t)(row < last_row ? row : last_row), a.TKp * 256) + slot_dw;
    };

    // NP = pairs of this workgroup, a compile-time count so that the tiles sit in registers
    auto wave_chunks = [&](auto np_c) {
        constexpr int NP = decltype(np_c)::value;
        uint8_t* const mine = stage + w * kStageBytes;
        v4i q[NP][2], qn[NP][2], raw[16];
        auto load_q = [&](v4i (&dst)[NP][2], int c) {
#pragma unroll
            for (int p = 0; p < NP; ++p) {
                const uint32_t* s = wbase + (int64_t)c * 256;
                const uint32_t off = pair_off(p);
                dst[p][0] = __builtin_nontemporal_load(reinterpret_cast<const v4i*>(s + off));
                dst[p][1] = __builtin_nontemporal_load(reinterpret_cast<const v4i*>(s + off + 128));
            }
        };
        // wave-load jj brings tokens 2 jj and 2 jj + 1: lane -> (token, 16-byte piece), whole rows
        auto load_raw = [&](int c) {
            uint32_t k = (uint32_t)c * kChunkK + 16 * tok;
            if (k > (uint32_t)K - 16) k = (uint32_t)K - 16;  // the packed bits there are zero
            // tokens 0 .. 15 exist; a token's offset adds up from the one before, the last token's is the largest
            const uint32_t last = __umul24((uint32_t)M - 1, a.ldq) + k;
            uint32_t at = __umul24((uint32_t)half, a.ldq) + k;
#pragma unroll
            for (int jj = 0; jj < 16; ++jj) {
                raw[jj] = *reinterpret_cast<const v4i*>(cbase + (jj < 8 || at < last ? at : last));
                at += 2 * a.ldq;
            }
        };
        load_q(q, w);
        load_raw(w);
        __builtin_amdgcn_sched_barrier(0);
        int ones = 0x01010101;  // in a scalar register: as a literal it doubles the size of the ANDs
        asm volatile("" : "+s"(ones));
        clear_sums();
        // the first tiles are waited for here, once: inside the loop a wait for them would have to
        // count the conditional fetches behind them as absent, and so wait for those as well
#pragma unroll
        for (int p = 0; p < NP; ++p) asm volatile("" : "+v"(q[p][0]), "+v"(q[p][1]));
#pragma unroll 1
        for (int chunk = w; chunk < TK; chunk += W) {
            // ---- the fetched codes become the B operands of plane i, k-half mf -------------------
            v4i act[8][2];
#pragma unroll
            for (int jj = 0; jj < 16; ++jj)
                *reinterpret_cast<v4i*>(mine + (2 * jj + half) * kStageRow + 16 * tok) = raw[jj];
            __builtin_amdgcn_wave_barrier();  // same wave, other lanes: LDS keeps a wave's accesses in order
#pragma unroll
            for (int i = 0; i < 8; ++i)
#pragma unroll
                for (int mf = 0; mf < 2; ++mf)
                    act[i][mf] =
                        *reinterpret_cast<const v4i*>(mine + tok * kStageRow + 64 * i + 32 * mf + 16 * half);
            __builtin_amdgcn_wave_barrier();
            __builtin_amdgcn_sched_barrier(0);
            // ---- the next chunk's fetches (wave-uniform branch) ------------------------------------
            const bool more = chunk + W < TK;
            if (more) {
                load_raw(chunk + W);
                load_q(qn, chunk + W);
            }
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int p = 0; p < NP; ++p) {
                v16i acc;
#pragma unroll
                for (int r = 0; r < 16; ++r) acc[r] = 0;
#pragma unroll
                for (int i = 0; i < 8; ++i)
#pragma unroll
                    for (int mf = 0; mf < 2; ++mf) {
                        const v4i wv = q[p][mf];
                        v4i b;
#pragma unroll
                        for (int d = 0; d < 4; ++d) b[d] = (int)(((uint32_t)wv[d] >> i) & (uint32_t)ones);
                        acc = __builtin_amdgcn_mfma_i32_32x32x32_i8(b, act[i][mf], acc, 0, 0, 0);
                    }
                // lane (tok, half) holds token tok, weight rows 8 (r/4) + 4 half + r%4
#pragma unroll
                for (int r = 0; r < 16; ++r)
                    atomicAdd(&red[(p * 32 + 8 * (r >> 2) + 4 * half + (r & 3)) * kPitch + tok], acc[r]);
                // the scheduler stays inside one pair: across pairs it would expand every plane of
                // every pair ahead of the MFMAs, and the registers run out
                __builtin_amdgcn_sched_barrier(0);
            }
            if (more) {
#pragma unroll
                for (int p = 0; p < NP; ++p) {
                    q[p][0] = qn[p][0];
                    q[p][1] = qn[p][1];
                }
            }
        }
    };

    if (w >= TK) {  // uniform per wave
        clear_sums();
    } else {
        switch (np) {  // np >= 1: there are no more workgroups than pairs
            case 1: wave_chunks(std::integral_constant<int, 1>{}); break;
            case 2: wave_chunks(std::integral_constant<int, 2>{}); break;
            case 3: wave_chunks(std::integral_constant<int, 3>{}); break;
            case 4: wave_chunks(std::integral_constant<int, 4>{}); break;
            default: clear_sums(); break;
        }
    }
    wait_vmcnt<0>();  // the tokens' factors
    __syncthreads();
    const float beta0 = a.beta[0];

    // ---- epilogue (Eq. 11): sum_k q s = 2 sum_k q b - sum_k q ; y = that * (beta gamma / 128) ----
    // item -> four consecutive weight rows of a pair and a token, eight items to a line of the output.
    // kind 0: one beta and none of the options; 1: sums (a slice, or int32 output); 2: the rest; 3: 0 with streaming
    // stores, for outputs of whole lines from 768 KB on.  There they pay with a pass over Y behind them as well (us of
    // the layer with that pass, ordinary / streaming: 24 x 4096 -> 12288 14.45 / 14.34, 32 x 2048 -> 6144 10.76 /
    // 10.56, 32 x 4096 -> 16384 15.27 / 15.21; without it 11.71 / 11.54, 7.93 / 7.86, 12.10 / 11.84); below, the
    // reader pays more than they gain (24 x 2048 -> 2048 9.17 / 9.79, 20 x 1408 -> 5632 10.34 / 10.64).
    const bool vec = (N & 3) == 0;  // then n + 3 < N and the row starts 16-byte aligned
    auto finish = [&](auto kind) {
        constexpr int KIND = decltype(kind)::value;
        uint32_t* const out = KIND == 1 && a.split_k
                                  ? reinterpret_cast<uint32_t*>(a.split_ws) + (int64_t)(sp * M) * N
                                  : reinterpret_cast<uint32_t*>(a.Y);
        for (int i = threadIdx.x; i < np * 8 * kTokens; i += blockDim.x) {
            const int nl = (i >> 8) * 32 + (i & 7) * 4, m = (i >> 3) & (kTokens - 1);
            const int n = p0 * 32 + nl;
            if (m >= M || n >= N) continue;
            int sum[4];
#pragma unroll
            for (int j = 0; j < 4; ++j) sum[j] = 2 * red[(nl + j) * kPitch + m];
            uint32_t* const dst = out + (int64_t)m * N + n;
            uint32_t o[4];
            if constexpr (KIND == 1) {
                const int rs = a.split_k ? 0 : tok_sum[m];
#pragma unroll
                for (int j = 0; j < 4; ++j) o[j] = (uint32_t)(sum[j] - rs);
            } else {
                const float sc = tok_gamma[m] * 0.0078125f;  // gamma / 128, exact
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    const int nj = n + j < N ? n + j : N - 1;
                    const float beta =
                        KIND != 2 || one_beta ? beta0 : a.beta[(int64_t)((uint32_t)nj / a.beta_rows) * a.beta_stride];
                    // beta * (gamma / 128) has the bits of (beta * gamma) / 128
                    float y = (float)(sum[j] - tok_sum[m]) * (beta * sc);
                    if (KIND == 2 && a.eta) y = y + (beta * tok_eta[m]) * (float)a.wsum[nj];       // Eq. 6
                    o[j] = __float_as_uint(y);
                }
            }
            if constexpr (KIND == 3) {
                const v4i v = {(int)o[0], (int)o[1], (int)o[2], (int)o[3]};
                __builtin_nontemporal_store(v, reinterpret_cast<v4i*>(dst));
            } else if (vec) {
                *reinterpret_cast<uint4*>(dst) = make_uint4(o[0], o[1], o[2], o[3]);
            } else {
#pragma unroll
                for (int j = 0; j < 4; ++j)
                    if (n + j < N) dst[j] = o[j];
            }
        }
    };
    if (a.split_k || a.out_acc) finish(std::integral_constant<int, 1>{});
    else if (!one_beta || a.eta) finish(std::integral_constant<int, 2>{});
    else if ((int64_t)M * N >= (int64_t)3 << 16 && (N & 31) == 0) finish(std::integral_constant<int, 3>{});
    else finish(std::integral_constant<int, 0>{});
}

// K-slices for 16 < M <= 32 that a call brings room for: longer K than 16 chunks (two per wave) in slices of at most
// 16 chunks; the launch takes as many of them as pay.  0 = no split.
int64_t stream_split_tiles(int64_t M, int64_t K) {
    if (M <= 16 || M > stream::kTokens) return 0;
    const int64_t TK = tiles_k(K);
    if (TK <= 16) return 0;
    const int64_t splits = (TK + 15) / 16;
    return (TK + splits - 1) / splits;
}

// false: the shape is not for this kernel (the mid-batch MFMA-tile kernel takes it)
bool launch_gemm_stream(const GemmArgs& a_in, hipStream_t s) {
    using namespace stream;
    GemmArgs a = a_in;
    a.split_k = 0;
    if (a.M <= 16 || a.M > kTokens || a.K >= ((int64_t)1 << 22)) return false;
    const int64_t TP = (tiles_n(a.N) + 1) / 2;
    int grid = num_cus();
    if (grid > TP) grid = (int)TP;
    if ((TP + grid - 1) / grid > kMaxPairs) return false;
    // every workgroup reads the codes of 32 tokens over all of K from L2 (K-slices share the
    // workgroups' pairs, so the split does not change the sum): past about 256 MB of that the
    // LDS-tiled kernel, whose workgroups share codes across more weight rows, takes over (24 x 28672 -> 7168, 205 MB,
    // 25.5 us here, 27.9 there; 24 x 24576 -> 10240, 201 MB in rounds of two pairs, 28.6 and 28.4)
    if ((int64_t)grid * kTokens * a.K > ((int64_t)1 << 28)) return false;
    // K-slices, of those the workspace has room for: the number that costs least, in us: a round of workgroups (one a
    // CU) 4.4 + 1.75 for every chunk and pair that a wave walks, the fold of the slices 3 and its sums at 5 TB/s.  The
    // layer at 24 tokens, in one slice / as many as give a wave two chunks: 16384 -> 4096 16.7 / 15.8, 12800 -> 3200
    // 14.6 / 14.3; but 22528 -> 5632 21.1 / 27.3, whose 528 workgroups are three rounds.
    int splits = 1;
    const int64_t TK = tiles_k(a.K), most = stream_split_tiles(a.M, a.K);
    if (most && a.split_ws && !tuning().mid_nosplit) {
        const int64_t n_max = (TK + most - 1) / most, pairs = (TP + grid - 1) / grid;
        double best_us = 1e30;
        for (int64_t want = 1; want <= n_max; ++want) {
            const int64_t per = (TK + want - 1) / want, n = (TK + per - 1) / per, cus = num_cus();
            const double bytes = (double)n * (double)a.M * (double)a.N * 4.0;
            if (n > 1 && bytes > (double)a.split_ws_bytes) break;
            const double us = (double)((grid * n + cus - 1) / cus) *
                                  (4.4 + 1.75 * (double)((per + kMaxWaves - 1) / kMaxWaves * pairs)) +
                              (n > 1 ? 3.0 + bytes * 2.0 / 5e6 : 0.0);
            if (us < best_us) {
                best_us = us;
                splits = (int)n;
                a.split_k = n > 1 ? per * kChunkK : 0;
            }
        }
        if (splits > 1) a.tk_pitch = a.tk_pitch ? a.tk_pitch : TK;
    }
    // as many waves as give every wave the same number of chunks (14 chunks: 7 waves, not 8)
    const int64_t TKs = splits > 1 ? a.split_k / kChunkK : TK;
    const int64_t rounds = (TKs + kMaxWaves - 1) / kMaxWaves;
    const int W = (int)((TKs + rounds - 1) / rounds);
    const dim3 g((unsigned)grid, (unsigned)splits);
    Args t{};
    t.codes = a.codes;
    t.packed = a.packed;
    t.M = (uint32_t)a.M;
    t.N = (uint32_t)a.N;
    t.ldq = (uint32_t)a.ldq;
    t.TKp = (uint32_t)(a.tk_pitch ? a.tk_pitch : tiles_k(a.K));
    t.K = (uint32_t)a.K;
    t.split_k = (uint32_t)a.split_k;
    t.pairs_wg = (uint32_t)(TP / grid);
    t.extra = (uint32_t)(TP % grid);
    t.gstride = (uint32_t)a.gstride;
    t.beta_rows = (uint32_t)a.beta_rows;
    t.gamma = a.gamma;
    t.beta = a.beta;
    t.eta = a.eta;
    t.rowsum = a.rowsum;
    t.wsum = a.wsum;
    t.beta_stride = a.beta_stride;
    t.per_tensor = a.per_tensor;
    t.out_acc = a.out_acc;
    t.Y = a.Y;
    t.split_ws = a.split_ws;
    gemm_stream_kernel<<<g, W * kWave, 0, s>>>(t);
    if (splits > 1) launch_splitk_reduce(a, splits, s);
    return true;
}

}  // namespace bl

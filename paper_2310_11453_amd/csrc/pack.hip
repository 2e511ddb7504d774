// Weight preparation for BitLinear (arXiv 2310.11453, Eq. 1-3 and Eq. 12):
// alpha = mean(W), beta = mean|W|, bit = (W > alpha), packed 1 bit per weight
// into 16x512 tiles (layout described in common.h).  HBM-bound: 4 bytes read
// per weight per pass, 1/8 byte written.
//
// alpha needs all of W before the first comparison with it, but it is the mean of a matrix and the
// weights it separates from zero are few: pack_scan reads W once, packs the bits of W > 0, and keeps
// the smallest |w| of every row of a tile (512 weights); a row's bits are those of W > alpha whenever
// |alpha| is below that, and pack_fix reads again only the rows where it is not (about one in 20 of a
// zero-mean 16384 x 4096 matrix; all of them if the mean is large, which costs what a second pass does).
#include "common.h"
#include "kernels.h"
#include "rowops.h"

namespace bl {

// One row of a tile: this lane's eight weights (columns 4 l .. and 256 + 4 l ..) against a threshold, as
// the dword that the tile's lane (g, c) = (q >> 2, row), dword q & 3 holds, q = l % 16: a comparison lands
// in bit 8 j + i, and the four lanes of a q meet in two steps.
__device__ inline uint32_t row_dword(const float4 (&w)[2], const bool (&valid)[2], float thr, int l) {
    uint32_t part = 0;
#pragma unroll
    for (int it = 0; it < 2; ++it) {
        const uint32_t nib = (uint32_t)(w[it].x > thr) | (uint32_t)(w[it].y > thr) << 8 |
                             (uint32_t)(w[it].z > thr) << 16 | (uint32_t)(w[it].w > thr) << 24;
        part |= valid[it] ? nib << (4 * it + (l >> 4)) : 0u;
    }
    int lo, hi;
    lane_swap<false>((int)part, lo, hi);
    lane_swap<true>(lo | hi, lo, hi);
    return (uint32_t)(lo | hi);
}

// ---- one reading of W: sums for alpha and beta, bits of W > 0, smallest |w| of a tile's rows ------
// One wave per tile, tiles dealt over a fixed grid; kRows rows of a tile are in flight at a time and the
// two halves of a tile are kept apart (together they take 193 registers and half the waves).
// partials[2*b] = sum of W, partials[2*b+1] = sum of |W| over workgroup b's tiles.
// The whole call, us, against two readings of W with the fold of the sums as a launch between them:
// 16384 x 4096 92 -> 62, 8192 x 2048 33 -> 22, 28672 x 7168 321 -> 183, 512 x 256 15 -> 12.5; with a mean of
// half the standard deviation, where pack_fix reads everything again, 94 -> 99 and 33 -> 30.
__global__ __launch_bounds__(256, 4) void pack_scan(const float* __restrict__ W, int64_t N, int64_t K,
                                                 int64_t ldw, uint32_t* __restrict__ packed,
                                                 float* __restrict__ rowmin,
                                                 double* __restrict__ partials) {
    constexpr int kRows = 8;
    __shared__ __attribute__((aligned(16))) uint32_t sm[4][256];
    __shared__ double smd[4];
    const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x / kWave), l = threadIdx.x % kWave;
    const int64_t TN = tiles_n(N), TK = tiles_k(K);
    double s = 0.0, a = 0.0;
    for (int64_t task = (int64_t)blockIdx.x * 4 + wave; task < TN * TK; task += (int64_t)gridDim.x * 4) {
        const int64_t tn = task / TK, tk = task % TK;
        float keep = 0.f;  // lane c keeps row c's smallest |w|
        const int64_t k0 = tk * kChunkK + 4 * l;
#pragma unroll 1
        for (int cb = 0; cb < kTileN; cb += kRows) {
            float4 w[kRows][2];
#pragma unroll
            for (int r = 0; r < kRows; ++r) {
                const int64_t n = tn * kTileN + cb + r < N ? tn * kTileN + cb + r : N - 1;
#pragma unroll
                for (int it = 0; it < 2; ++it) {
                    const int64_t k = k0 + 256 * it < K ? k0 + 256 * it : K - 4;
                    w[r][it] = *reinterpret_cast<const float4*>(W + n * ldw + k);
                }
            }
#pragma unroll
            for (int r = 0; r < kRows; ++r) {
                const bool row = tn * kTileN + cb + r < N;
                const bool valid[2] = {row && k0 < K, row && k0 + 256 < K};
                float mn = __builtin_inff();
#pragma unroll
                for (int it = 0; it < 2; ++it) {
                    float4 v = w[r][it];
                    const float m4 = fminf(fminf(fabsf(v.x), fabsf(v.y)), fminf(fabsf(v.z), fabsf(v.w)));
                    if (!valid[it]) v = make_float4(0.f, 0.f, 0.f, 0.f);
                    else mn = fminf(mn, m4);
                    const double x = (double)v.x, y = (double)v.y, z = (double)v.z, u = (double)v.w;
                    s += (x + y) + (z + u);
                    a += (fabs(x) + fabs(y)) + (fabs(z) + fabs(u));
                }
                mn = wave_reduce(mn, OpMin{});
                if (l == cb + r) keep = mn;
                const uint32_t dw = row_dword(w[r], valid, 0.f, l);
                if (l < 16) sm[wave][((l >> 2) * 16 + cb + r) * 4 + (l & 3)] = dw;
            }
        }
        // a wave's own part of sm: LDS serves a wave in order, so the compiler keeping the order of the lanes'
        // writes, this read and the next tile's writes is all it takes
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        __builtin_amdgcn_wave_barrier();
        const uint4 v = *reinterpret_cast<const uint4*>(&sm[wave][l * 4]);
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        __builtin_amdgcn_wave_barrier();
        *reinterpret_cast<uint4*>(packed + tile_dword_offset(tn, tk, TK) + l * 4) = v;
        if (l < kTileN) rowmin[task * kTileN + l] = keep;
    }
    s = block_sum<4>(s, smd);
    a = block_sum<4>(a, smd);
    if (threadIdx.x == 0) {
        partials[2 * blockIdx.x] = s;
        partials[2 * blockIdx.x + 1] = a;
    }
}

// ---- alpha, beta, and the rows of tiles whose bits depend on alpha --------------------------------
// Every workgroup folds the partials for itself (the same sums in the same order, out of L2); workgroup 0
// writes the two scalars.  A wave looks at the 16 rows of a tile at once and repacks the ones with a
// weight within |alpha| of zero, four at a time.
__global__ __launch_bounds__(256) void pack_fix(const float* __restrict__ W, int64_t N, int64_t K,
                                                int64_t ldw, const double* __restrict__ partials,
                                                int nparts, double count,
                                                const float* __restrict__ rowmin,
                                                uint32_t* __restrict__ packed,
                                                float* __restrict__ alpha_out,
                                                float* __restrict__ beta_out) {
    __shared__ double sm[4];
    const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x / kWave), l = threadIdx.x % kWave;
    double s = 0.0, a = 0.0;
    for (int i = threadIdx.x; i < nparts; i += 256) {
        s += partials[2 * i];
        a += partials[2 * i + 1];
    }
    s = block_sum<4>(s, sm);
    const float alpha = (float)(s / count);
    if (blockIdx.x == 0) {
        a = block_sum<4>(a, sm);
        if (threadIdx.x == 0) {
            *alpha_out = alpha;
            *beta_out = (float)(a / count);
        }
    }
    const int64_t TN = tiles_n(N), TK = tiles_k(K);
    for (int64_t task = (int64_t)blockIdx.x * 4 + wave; task < TN * TK; task += (int64_t)gridDim.x * 4) {
        const float mn = l < kTileN ? rowmin[task * kTileN + l] : __builtin_inff();
        const int64_t tn = task / TK, tk = task % TK, k0 = tk * kChunkK + 4 * l;
        const int64_t rows = N - tn * kTileN < kTileN ? N - tn * kTileN : kTileN;
        uint32_t redo = (uint32_t)__ballot(!(mn > fabsf(alpha))) & ((1u << rows) - 1u);
        while (redo) {  // uniform for the wave
            int c[4];
            float4 w[4][2];
            const bool valid[2] = {k0 < K, k0 + 256 < K};
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                c[r] = redo ? __builtin_ctz(redo) : c[r ? r - 1 : 0];
                redo &= redo - 1;
#pragma unroll
                for (int it = 0; it < 2; ++it) {
                    const int64_t k = k0 + 256 * it < K ? k0 + 256 * it : K - 4;
                    w[r][it] = *reinterpret_cast<const float4*>(W + (tn * kTileN + c[r]) * ldw + k);
                }
            }
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const uint32_t dw = row_dword(w[r], valid, alpha, l);
                if (l < 16)
                    packed[tile_dword_offset(tn, tk, TK) + ((l >> 2) * 16 + c[r]) * 4 + (l & 3)] = dw;
            }
        }
    }
}

// ---- pass 1: per-block partial sums of W and |W - centre| in fp64 ----------
// partials[2*b] = sum of W, partials[2*b+1] = sum of |W - centre| over the
// block's grid-stride share.  centre_ptr == nullptr means centre = 0.
// The block's rows are cols4 float4 long and ld4 float4 apart (ld4 == cols4: contiguous, the
// index is used as it is).
__global__ __launch_bounds__(256) void weight_partial_sums(const float4* __restrict__ W4,
                                                           int64_t count4, int64_t cols4,
                                                           int64_t ld4,
                                                           const float* __restrict__ centre_ptr,
                                                           double* __restrict__ partials) {
    __shared__ double sm[4];
    const double centre = centre_ptr ? (double)*centre_ptr : 0.0;
    double s = 0.0, a = 0.0;
    const int64_t stride = (int64_t)gridDim.x * 256;
    const bool strided = ld4 != cols4;
    auto at = [&](int64_t i) { return W4[strided ? (i / cols4) * ld4 + i % cols4 : i]; };
    auto add = [&](const float4& w) {
        const double x = (double)w.x, y = (double)w.y, z = (double)w.z, u = (double)w.w;
        s += (x + y) + (z + u);
        a += (fabs(x - centre) + fabs(y - centre)) + (fabs(z - centre) + fabs(u - centre));
    };
    // four loads in flight per thread (one at a time, the pass is bound by their latency); the
    // order of the sums stays that of the plain loop
    int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    for (; i + 3 * stride < count4; i += 4 * stride) {
        const float4 w0 = at(i), w1 = at(i + stride), w2 = at(i + 2 * stride), w3 = at(i + 3 * stride);
        add(w0);
        add(w1);
        add(w2);
        add(w3);
    }
    for (; i < count4; i += stride) add(at(i));
    s = block_sum<4>(s, sm);
    a = block_sum<4>(a, sm);
    if (threadIdx.x == 0) {
        partials[2 * blockIdx.x] = s;
        partials[2 * blockIdx.x + 1] = a;
    }
}

// ---- pass 2: one block folds the partials in a fixed order -----------------
// write_alpha / write_beta select which scalars this call produces.
__global__ __launch_bounds__(256) void weight_finalize(const double* __restrict__ partials,
                                                       int nblocks, double count, int write_alpha,
                                                       int write_beta, float* __restrict__ alpha,
                                                       float* __restrict__ beta) {
    __shared__ double sm[4];
    double s = 0.0, a = 0.0;
    for (int i = threadIdx.x; i < nblocks; i += 256) {
        s += partials[2 * i];
        a += partials[2 * i + 1];
    }
    s = block_sum<4>(s, sm);
    a = block_sum<4>(a, sm);
    if (threadIdx.x == 0) {
        if (write_alpha) *alpha = (float)(s / count);
        if (write_beta) *beta = (float)(a / count);
    }
}

// ---- pass 3: compare with alpha and pack ----------------------------------
// One wave builds one 16x512 tile.  For each of the 16 rows the wave reads the
// row's 512 floats with two coalesced float4 loads per lane; a lane's four
// comparisons land in bit positions 8*j + i of the dword owned by lanes with
// the same (lane % 16), which two xor-shuffles OR together.  The tile is
// staged in LDS so the final store is one 16-byte write per lane.
__global__ __launch_bounds__(256) void pack_tiles(const float* __restrict__ W, int64_t N,
                                                  int64_t K, int64_t ldw,
                                                  const float* __restrict__ alpha_ptr,
                                                  uint32_t* __restrict__ packed) {
    __shared__ uint32_t sm[4][256];
    const int wave = threadIdx.x / kWave, l = threadIdx.x % kWave;
    const int64_t TN = tiles_n(N), TK = tiles_k(K);
    const int64_t task = (int64_t)blockIdx.x * 4 + wave;
    const bool live = task < TN * TK;
    const int64_t tn = live ? task / TK : 0, tk = live ? task % TK : 0;
    const float alpha = *alpha_ptr;

#pragma unroll 4
    for (int c = 0; c < kTileN; ++c) {
        const int64_t n = tn * kTileN + c;
        uint32_t part = 0;
#pragma unroll
        for (int it = 0; it < 2; ++it) {
            const int64_t k = tk * kChunkK + 256 * it + 4 * l;
            if (live && n < N && k < K) {
                const float4 w = *reinterpret_cast<const float4*>(W + n * ldw + k);
                const int i = 4 * it + (l >> 4);
                part |= (uint32_t)(w.x > alpha) << i;
                part |= (uint32_t)(w.y > alpha) << (8 + i);
                part |= (uint32_t)(w.z > alpha) << (16 + i);
                part |= (uint32_t)(w.w > alpha) << (24 + i);
            }
        }
        part |= (uint32_t)__shfl_xor((int)part, 16, kWave);
        part |= (uint32_t)__shfl_xor((int)part, 32, kWave);
        if (l < 16) sm[wave][((l >> 2) * 16 + c) * 4 + (l & 3)] = part;
    }
    __syncthreads();
    if (live) {
        const uint4 v = *reinterpret_cast<const uint4*>(&sm[wave][l * 4]);
        *reinterpret_cast<uint4*>(packed + tile_dword_offset(tn, tk, TK) + l * 4) = v;
    }
}

// ---- inspection: tiles -> canonical words ---------------------------------
// canonical[n][kw] bit b  <->  sign bit of (n, k = 32*kw + b).
__global__ __launch_bounds__(256) void tiles_to_canonical(const uint32_t* __restrict__ packed,
                                                          int64_t N, int64_t K,
                                                          uint32_t* __restrict__ canonical,
                                                          int64_t ldc) {
    const int64_t KW = K / 32;
    const int64_t idx = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (idx >= N * KW) return;
    const int64_t n = idx / KW, kw = idx % KW;
    const int64_t TK = tiles_k(K);
    const int64_t tn = n / kTileN, c = n % kTileN;
    const int64_t k0 = kw * 32;
    const int64_t tk = k0 / kChunkK;
    const int r0 = (int)(k0 % kChunkK);
    const int i = r0 / 64;
    const uint32_t* tile = packed + tile_dword_offset(tn, tk, TK);
    uint32_t word = 0;
    for (int b = 0; b < 32; ++b) {
        const int r = r0 + b;
        const int g = (r % 64) / 16, d = (r % 16) / 4, j = r % 4;
        const uint32_t dw = tile[(g * 16 + c) * 4 + d];
        word |= ((dw >> (8 * j + i)) & 1u) << b;
    }
    canonical[n * ldc + kw] = word;
}

// ---- wsum[n] = sum_k s[n,k] = 2 * popcount(row n) - K, from the packed tiles ----------
// One wave per tile row: it walks the row's tiles (1 KiB, coalesced), every lane counts the set
// bits of its 4 dwords (16 columns of weight row lane%16), the four lanes of a row add up.
// Padding bits are zero, so only real columns are counted.
__global__ __launch_bounds__(256) void weight_rowsums(const uint32_t* __restrict__ packed,
                                                      int64_t N, int64_t K,
                                                      int32_t* __restrict__ wsum) {
    const int wave = threadIdx.x / kWave, l = threadIdx.x % kWave;
    const int64_t TN = tiles_n(N), TK = tiles_k(K);
    const int64_t tn = (int64_t)blockIdx.x * 4 + wave;
    if (tn >= TN) return;
    int pop = 0;
    for (int64_t tk = 0; tk < TK; ++tk) {
        const uint4 v = *reinterpret_cast<const uint4*>(packed + tile_dword_offset(tn, tk, TK) + l * 4);
        pop += __popc(v.x) + __popc(v.y) + __popc(v.z) + __popc(v.w);
    }
    pop += __shfl_xor(pop, 16, kWave);
    pop += __shfl_xor(pop, 32, kWave);
    const int64_t n = tn * kTileN + l;
    if (l < kTileN && n < N) wsum[n] = 2 * pop - (int)K;
}

// ---------------------------------------------------------------------------
int reduce_grid(int64_t count4) {
    int64_t g = (count4 + 256 * 8 - 1) / (256 * 8);
    if (g < 1) g = 1;
    if (g > 1024) g = 1024;
    return (int)g;
}

static int scan_grid(int64_t tiles) { return (int)((tiles + 3) / 4 < 1024 ? (tiles + 3) / 4 : 1024); }
// workspace with which W is read once: the scan's partial sums, then the tiles' smallest |w|
size_t pack_scan_bytes(int64_t N, int64_t K) {
    const int64_t tiles = tiles_n(N) * tiles_k(K);
    return (size_t)scan_grid(tiles) * 16 + (size_t)tiles * kTileN * 4;
}

hipError_t launch_pack(const float* W, int64_t N, int64_t K, int64_t ldw, bool beta_centered,
                       uint32_t* packed, float* alpha, float* beta, double* partials,
                       size_t partials_bytes, hipStream_t s) {
    const int64_t count4 = N * K / 4;
    // beta about alpha needs a second reading of every weight in any case
    if (!beta_centered && partials_bytes >= pack_scan_bytes(N, K)) {
        const int64_t tiles = tiles_n(N) * tiles_k(K);
        const int G = scan_grid(tiles);
        float* rowmin = reinterpret_cast<float*>(partials + 2 * G);
        pack_scan<<<G, 256, 0, s>>>(W, N, K, ldw, packed, rowmin, partials);
        pack_fix<<<(unsigned)((tiles + 3) / 4 < 2048 ? (tiles + 3) / 4 : 2048), 256, 0, s>>>(W, N, K, ldw, partials, G, (double)N * (double)K, rowmin, packed,
                                   alpha, beta);
        return hipGetLastError();
    }
    const int G = reduce_grid(count4);
    const double cnt = (double)N * (double)K;
    const float4* W4 = (const float4*)W;
    weight_partial_sums<<<G, 256, 0, s>>>(W4, count4, K / 4, ldw / 4, nullptr, partials);
    weight_finalize<<<1, 256, 0, s>>>(partials, G, cnt, 1, beta_centered ? 0 : 1, alpha, beta);
    if (beta_centered) {
        weight_partial_sums<<<G, 256, 0, s>>>(W4, count4, K / 4, ldw / 4, alpha, partials);
        weight_finalize<<<1, 256, 0, s>>>(partials, G, cnt, 0, 1, alpha, beta);
    }
    const int64_t tasks = tiles_n(N) * tiles_k(K);
    pack_tiles<<<(unsigned)((tasks + 3) / 4), 256, 0, s>>>(W, N, K, ldw, alpha, packed);
    return hipGetLastError();
}

hipError_t launch_weight_rowsums(const uint32_t* packed, int64_t N, int64_t K, int32_t* wsum,
                                 hipStream_t s) {
    weight_rowsums<<<(unsigned)((tiles_n(N) + 3) / 4), 256, 0, s>>>(packed, N, K, wsum);
    return hipGetLastError();
}

hipError_t launch_to_canonical(const uint32_t* packed, int64_t N, int64_t K, uint32_t* canonical,
                               int64_t ldc, hipStream_t s) {
    const int64_t words = N * (K / 32);
    tiles_to_canonical<<<(unsigned)((words + 255) / 256), 256, 0, s>>>(packed, N, K, canonical, ldc);
    return hipGetLastError();
}

}  // namespace bl

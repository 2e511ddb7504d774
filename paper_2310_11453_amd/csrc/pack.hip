// Weight preparation for BitLinear (arXiv 2310.11453, Eq. 1-3 and Eq. 12):
// alpha = mean(W), beta = mean|W|, bit = (W > alpha), packed 1 bit per weight
// into 16x512 tiles (layout described in common.h).  HBM-bound: 4 bytes read
// per weight per pass, 1/8 byte written.
//
// alpha needs all of W before the first comparison with it, but it is the mean of a matrix and the
// weights it separates from zero are few: pack_scan reads W once, packs the bits of W > 0, and keeps
// the smallest |w| of every row of a tile (512 weights); a row's bits are those of W > alpha whenever
// |alpha| is below that, and pack_fix reads again only the rows where it is not (about one in 20 of a
// zero-mean 16384 x 4096 matrix; all of them if the mean is a fiftieth of the deviation or more, which costs what
// a second pass does).
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

// Stores the dwords of four rows of a tile: every lane has all four rows' for q = l % 16 and stores row l / 16's.
// By value: a choice between array elements would put the arrays into LDS and make the kernel read its
// workgroup size out of the dispatch packet, in host memory (13 us a launch).
__device__ inline void store_rows(uint32_t* tile, int l, uint32_t dw0, uint32_t dw1, uint32_t dw2, uint32_t dw3,
                                  int c0, int c1, int c2, int c3) {
    const bool odd = l & 16, high = l & 32;
    const uint32_t dw = high ? (odd ? dw3 : dw2) : (odd ? dw1 : dw0);
    const int c = high ? (odd ? c3 : c2) : (odd ? c1 : c0);
    tile[(((l & 15) >> 2) * 16 + c) * 4 + (l & 3)] = dw;
}

// ---- one reading of W: sums for alpha and beta, bits of W > 0, smallest |w| of a tile's rows ------
// One wave per half tile (8 rows, all in flight at once), dealt over a fixed grid.
// partials[2*b] = sum of W, partials[2*b+1] = sum of |W| over workgroup b's rows.
// The whole call, us: two readings of W with the fold of the sums as a launch between them / this with a zero mean /
// this with a mean of half the deviation, where pack_fix reads everything again: 64 x 32 10.6 / 8.6 / 8.7,
// 512 x 256 12.0 / 9.0 / 9.0, 2048 x 2048 20.5 / 10.5 / 11.4, 8192 x 2048 31 / 19.6 / 27.8, 16384 x 4096 88 / 54 / 87,
// 28672 x 7168 314 / 179 / 311; up to 3 % slower than two readings only where W is 100 to 200 MB and all of it is
// repacked (8192 x 4096 46.4 / 30.8 / 48, 50257 x 1024 69 / 42.5 / 70.5).
__global__ __launch_bounds__(256, 4) void pack_scan(const float* __restrict__ W, int64_t N, int64_t K,
                                                 int64_t ldw, uint32_t* __restrict__ packed,
                                                 float* __restrict__ rowmin,
                                                 double* __restrict__ partials) {
    constexpr int kRows = 8;
    __shared__ double smd[4];
    const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x / kWave), l = threadIdx.x % kWave;
    const uint32_t TK = (uint32_t)tiles_k(K), items = (uint32_t)tiles_n(N) * TK * (kTileN / kRows);  // < 2^31
    double s = 0.0, a = 0.0;
    for (uint32_t item = blockIdx.x * 4 + wave; item < items; item += gridDim.x * 4) {
        const uint32_t tile = item >> 1, tn = tile / TK, tk = tile - tn * TK;
        const int cb = (int)(item & 1) * kRows;
        const int64_t n0 = (int64_t)tn * kTileN + cb, k0 = (int64_t)tk * kChunkK + 4 * l;
        float keep = 0.f;  // lane r keeps row cb + r's smallest |w|
        float4 w[kRows][2];
#pragma unroll
        for (int r = 0; r < kRows; ++r) {
            const int64_t n = n0 + r < N ? n0 + r : N - 1;
#pragma unroll
            for (int it = 0; it < 2; ++it) {
                const int64_t k = k0 + 256 * it < K ? k0 + 256 * it : K - 4;
                w[r][it] = *reinterpret_cast<const float4*>(W + n * ldw + k);
            }
        }
        uint32_t dw[kRows];
#pragma unroll
        for (int r = 0; r < kRows; ++r) {
            const bool row = n0 + r < N;
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
            if (l == r) keep = mn;
            dw[r] = row_dword(w[r], valid, 0.f, l);
        }
        uint32_t* const at = packed + tile_dword_offset(tn, tk, TK);
#pragma unroll
        for (int r = 0; r < kRows; r += 4)
            store_rows(at, l, dw[r], dw[r + 1], dw[r + 2], dw[r + 3], cb + r, cb + r + 1, cb + r + 2, cb + r + 3);
        if (l < kRows) rowmin[(int64_t)item * kRows + l] = keep;
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
// writes the two scalars.  A wave looks at `nrows` rows of a tile at once (4, 8 or 16) and repacks the ones with
// a weight within |alpha| of zero, four at a time and two such fours in flight.
__global__ __launch_bounds__(256) void pack_fix(const float* __restrict__ W, int64_t N, int64_t K,
                                                int64_t ldw, const double* __restrict__ partials,
                                                int nparts, double count, int nrows, bool backwards,
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
    const uint32_t TK = (uint32_t)tiles_k(K), per = kTileN / nrows;  // items of a tile
    const uint32_t items = (uint32_t)tiles_n(N) * TK * per;           // < 2^31
    for (uint32_t i = blockIdx.x * 4 + wave; i < items; i += gridDim.x * 4) {
        const uint32_t item = backwards ? items - 1 - i : i, tile = item / per, tk = tile % TK;
        const int64_t tn = tile / TK, k0 = (int64_t)tk * kChunkK + 4 * l;
        const int c0 = (int)(item % per) * nrows;
        const int64_t left = N - tn * kTileN - c0;
        const int rows = (int)(left < nrows ? left : nrows);  // may be negative: nothing
        const float mn = l < rows ? rowmin[(int64_t)tile * kTileN + c0 + l] : __builtin_inff();
        // a NaN or infinite alpha repacks every row
        uint32_t redo = (uint32_t)__ballot(l < rows && !(mn > fabsf(alpha)));
        const bool valid[2] = {k0 < K, k0 + 256 < K};
        // the next (up to) four rows to repack; a missing one repeats the one before it
        auto take4 = [&](float4 (&w)[4][2], int (&c)[4]) {
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                c[r] = redo ? c0 + __builtin_ctz(redo) : c[r ? r - 1 : 0];
                redo &= redo - 1;
#pragma unroll
                for (int it = 0; it < 2; ++it) {
                    const int64_t k = k0 + 256 * it < K ? k0 + 256 * it : K - 4;
                    w[r][it] = *reinterpret_cast<const float4*>(W + (tn * kTileN + c[r]) * ldw + k);
                }
            }
        };
        auto store4 = [&](const float4 (&w)[4][2], const int (&c)[4]) {
            uint32_t dw[4];
#pragma unroll
            for (int r = 0; r < 4; ++r) dw[r] = row_dword(w[r], valid, alpha, l);
            store_rows(packed + tile_dword_offset(tn, tk, TK), l, dw[0], dw[1], dw[2], dw[3], c[0], c[1], c[2], c[3]);
        };
        while (redo) {  // uniform for the wave
            float4 w0[4][2], w1[4][2];
            int r0[4], r1[4] = {};
            take4(w0, r0);
            const bool more = redo != 0;
            if (more) take4(w1, r1);
            store4(w0, r0);
            if (more) store4(w1, r1);
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

static int scan_grid(int64_t tiles) {
    const int64_t blocks = (tiles + 1) / 2;  // of four waves with one half tile each
    return (int)(blocks < 512 ? blocks : 512);  // 2 a CU: with 4, 64 MB matrices took 0.6 us more (20.2 / 19.6)
}
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
        // Few tiles: more, shorter items (8 rows / 16, repacked as a whole: 4500 x 2048, 1128 tiles, 17.7 us / 20.7;
        // 3840 x 3840, 1920 tiles, 26.6 / 26.1).  W beyond the Infinity Cache: last tiles first, they are still in it
        // (28672 x 7168 all repacked 333 us -> 317); else in the scan's order, which finds them in the XCD's
        // own L2 (4096 x 2048 16.0 / 18.9 -> 13.3 / 13.8).
        const int nrows = tiles <= 512 ? 4 : tiles <= 1600 ? 8 : kTileN;
        const bool backwards = N * K * 4 > (int64_t)256 << 20;
        const int64_t blocks = (tiles * (kTileN / nrows) + 3) / 4;
        pack_fix<<<(unsigned)(blocks < 1280 ? blocks : 1280), 256, 0, s>>>(
            W, N, K, ldw, partials, G, (double)N * (double)K, nrows, backwards, rowmin, packed, alpha, beta);
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

// Straight-through-estimator backward of BitLinear (arXiv 2310.11453, Section 2.2):
// Sign, Clip and rounding are treated as identity and alpha, beta, gamma as constants, so
//   y = x^ (beta S)^T  with  x^ ~ q gamma/128,  S = sign matrix in {-1,+1}
//   dX^[M,K] = beta * g[M,N] S[N,K]                 g  = bf16(dY)
//   dW [N,K] = gw^T[N,M] q[M,K] * (gamma/128)       gw = bf16(dY) per tensor,
//                                                    bf16(dY * gamma_m/128) per token
// Both are bf16 MFMA contractions with fp32 accumulation (+-1 and int8 codes are exact in
// bf16; only dY is rounded).
//
// Structure.  Each operand is first written once in the layout the product kernels read (in blocks
// of 32 reduction indices, padded with zeros; see block_offset):
//   g   [M][Np]    rows of dY, cast                (A operand of dX, reduction over N)
//   Sw  [Np/32][K] the signs of 32 weight rows of a column in one word (B operand of dX: the
//                  kernel builds +-1 bf16 from it in registers)
//   gwT [N][Mp]    dY transposed, scaled, cast     (A operand of dW, reduction over M)
//   qT  [K][Mp]    codes transposed, cast          (B operand of dW)
// (one pass over dY writes g and gwT) and one product, C[I][J] = scale * sum_r A[I][r] B[J][r],
// serves both: persistent 256 x 256 kernels fed by DMA, cut along r where the tiles are few.  The
// preparation passes are HBM-bound and small next to the 2*M*N*K flops of each product.

#include "common.h"
#include "kernels.h"
#include "ring.h"

namespace bl {

typedef __bf16 v8bf __attribute__((ext_vector_type(8)));

// round-to-nearest-even fp32 -> bf16 bits (inputs are finite)
__device__ inline uint32_t bf16_bits(float v) {
    uint32_t u = __float_as_uint(v);
    u += 0x7fffu + ((u >> 16) & 1u);
    return u >> 16;
}

// Layout of the bf16 copies: blocks of 32 reduction indices, inside a block row by row, i.e. element
// (row, r) of a copy with R rows lies at ((r / 32) * R + row) * 32 + r % 32.  A stage of the product
// kernels (32 r of 256 rows) is then 16 KiB in one piece: whole 128-byte lines, each requested once.
// (Row-major copies gave it 64 bytes of each of 256 rows, half a line per request, and a pitch that
// had to be kept off multiples of 4 KiB.)  M = 8192, 4096 -> 16384: dW 963 -> 946 us, the pass over dY 205 ->
// 188 us, whose stores fall on contiguous 256-byte pieces now.
__host__ __device__ inline int64_t block_offset(int64_t row, int64_t r, int64_t R) {
    return ((r >> 5) * R + row) * 32 + (r & 31);
}
//
// ---- in[R][C] (fp32 or int8) -> bf16 copies, one read of the input ----------------------------
//   rows[R][Cp]  = bf16(in)                      (reduction over C; columns C..Cp-1 zero)
//   tr  [C][Rp]  = bf16(scale_r * in)^T          (reduction over R; columns R..Rp-1 zero)
// scale_r = row_gamma[r] / 128 or 1.  Either output may be null.  A workgroup takes a 64 x 64
// tile: each thread reads 4 x 4 consecutive elements, writes its 8-byte pieces of `rows`, and
// the transpose goes through LDS (row pitch 66 halfwords: the 4-row steps of the 16 lanes that
// build one output row fall on distinct banks) and leaves as 8-byte pieces too.
// VEC: C % 4 == 0 and `in` 16-byte aligned, so that a thread's 4 elements are one load.
typedef uint16_t CastTile[64][66];
template <typename IN, bool VEC>
__device__ inline void cast_transpose_tile(const IN* __restrict__ in, int64_t R, int64_t C, int64_t Cp, int64_t Rp,
                                           const float* __restrict__ row_gamma, uint16_t* __restrict__ rows,
                                           uint16_t* __restrict__ tr, int64_t r0, int64_t c0, CastTile& tile) {
    // Rows that are no whole float4: everything is requested first, without a branch, past the input's end the last row
    // or column again, zeroed below.  Behind branches, load and use by turns, they pay four trips to memory a tile (M x K
    // x N, us of the call, behind branches / now: dX of 4154 x 192 x 20971 190 / 169, dW of 8192 x 256 x 16382 281 /
    // 252).  A float4 a row at once takes registers that more waves use better: the launch for 1000 x 2048 x 8192 16.9 us,
    // 15.9 one by one.
    const int cl = ((int)threadIdx.x & 15) * 4;
    const int64_t c = c0 + cl;
    float all[VEC ? 1 : 4][4], gamma[VEC ? 1 : 4];
    if constexpr (!VEC) {
#pragma unroll
        for (int it = 0; it < 4; ++it) {
            if (r0 + it * 16 >= R) break;  // uniform (2 x 256 x 774, dW, 7.1 us, 7.7 with all four)
            const int64_t r = r0 + it * 16 + (threadIdx.x >> 4), at = r < R ? r : R - 1;
#pragma unroll
            for (int e = 0; e < 4; ++e) all[it][e] = (float)in[at * C + (c + e < C ? c + e : C - 1)];
            if (row_gamma) gamma[it] = row_gamma[at];  // uniform
        }
    }
#pragma unroll
    for (int it = 0; it < 4; ++it) {
        const int rl = it * 16 + (threadIdx.x >> 4);
        const int64_t r = r0 + rl;
        float v[4] = {0.f, 0.f, 0.f, 0.f};
        if constexpr (!VEC) {
#pragma unroll
            for (int e = 0; e < 4; ++e) v[e] = r < R && c + e < C ? all[it][e] : 0.f;
        } else if (r < R && c < C) {
            if constexpr (sizeof(IN) == 4) {
                const float4 t = *reinterpret_cast<const float4*>(in + r * C + c);
                v[0] = t.x, v[1] = t.y, v[2] = t.z, v[3] = t.w;
            } else {
                const char4 t = *reinterpret_cast<const char4*>(in + r * C + c);
                v[0] = (float)t.x, v[1] = (float)t.y, v[2] = (float)t.z, v[3] = (float)t.w;
            }
        }
        if (rows && r < R && c < Cp)
            *reinterpret_cast<uint2*>(rows + block_offset(r, c, R)) =
                make_uint2(bf16_bits(v[0]) | (bf16_bits(v[1]) << 16),
                           bf16_bits(v[2]) | (bf16_bits(v[3]) << 16));
        if (row_gamma && r < R) {
            const float sc = (VEC ? row_gamma[r] : gamma[VEC ? 0 : it]) / 128.0f;
#pragma unroll
            for (int e = 0; e < 4; ++e) v[e] = v[e] * sc;
        }
        uint32_t* t32 = reinterpret_cast<uint32_t*>(&tile[rl][cl]);
        t32[0] = bf16_bits(v[0]) | (bf16_bits(v[1]) << 16);
        t32[1] = bf16_bits(v[2]) | (bf16_bits(v[3]) << 16);
    }
    if (!tr) return;
    __syncthreads();
#pragma unroll
    for (int it = 0; it < 4; ++it) {
        const int idx = it * 256 + threadIdx.x;
        const int cl = idx >> 4, rl = (idx & 15) * 4;
        const int64_t c = c0 + cl, r = r0 + rl;
        if (c < C && r < Rp)
            *reinterpret_cast<uint2*>(tr + block_offset(c, r, C)) =
                make_uint2((uint32_t)tile[rl][cl] | ((uint32_t)tile[rl + 1][cl] << 16),
                           (uint32_t)tile[rl + 2][cl] | ((uint32_t)tile[rl + 3][cl] << 16));
    }
}

// ---- Sw[Np/32][K]: the signs of 32 consecutive weight rows of one column k in one word -------
// What the ring kernel below reads as the B operand of dX (reduction over n): a stage of 32 n is
// one word per column, 1 KiB for a 256-column tile instead of 16 KiB of bf16.  Bit layout of a
// word, chosen so that a lane builds an MFMA operand dword with one shift and one and-or: row
// n = 32 sw + r sits at bit 8 (r/16) + 4 ((r%16)/8) + (r%8)/2 + 16 (r%2), and holds 1 for -1
// (the bf16 sign bit), 0 for +1.  Rows past N: their columns of g are zero, any bit does.
// One workgroup transposes two tiles (32 rows) x 512 columns.
__device__ inline void bits_transpose_tile(const uint32_t* __restrict__ packed, int64_t N, int64_t K,
                                           uint32_t* __restrict__ Sw, int64_t sw, int64_t tk, uint32_t (&sm)[2][256]) {
    const int64_t TN = tiles_n(N), TK = tiles_k(K);
    for (int t = 0; t < 2; ++t) {
        uint32_t v = 0;
        if (2 * sw + t < TN) v = packed[tile_dword_offset(2 * sw + t, tk, TK) + threadIdx.x];
        sm[t][threadIdx.x] = v;
    }
    __syncthreads();
    for (int it = 0; it < 2; ++it) {
        const int kl = it * 256 + threadIdx.x;
        const int64_t k = tk * kChunkK + kl;
        if (k >= K) continue;
        const int i = kl >> 6, g = (kl & 63) >> 4, d = (kl & 15) >> 2, j = kl & 3;
        uint32_t word = 0;
#pragma unroll
        for (int r = 0; r < 32; ++r) {
            const uint32_t dw = sm[r >> 4][(g * 16 + (r & 15)) * 4 + d];
            const uint32_t minus = ((dw >> (8 * j + i)) & 1u) ^ 1u;
            word |= minus << (8 * (r >> 4) + 4 * ((r & 15) >> 3) + ((r & 7) >> 1) + 16 * (r & 1));
        }
        Sw[sw * K + k] = word;
    }
}

// All of it in one launch: 64 x 64 tiles of dY, of the codes, and 32 x 512 pieces of the sign matrix are the items of
// one grid.  Each part alone is HBM-bound when large, but at a thousand tokens the two small ones are launches of
// latency (whole call, us, three launches / one, M x N x K: 256 x 1024 x 1024 32.0 / 26.5, 333 x 2048 x 2048 40.5 /
// 36.0, 1000 x 8192 x 2048 108.9 / 104.2; 8192 x 16384 x 4096 1752 / 1752).  The small parts come first: behind dY
// they would be the tail.
struct PrepareArgs {
    const float* dY;
    const int8_t* codes;
    const uint32_t* packed;
    const float* row_gamma;  // null: per tensor
    uint16_t *g, *gwT, *qT;  // what is not wanted is null
    uint32_t* Sw;
    int64_t M, N, K, Np, Mp;
    uint32_t bits_items, code_items, items;  // items: of all three parts
    uint32_t bits_x, code_x, dy_x;           // items in a row of each part
};
template <bool VECY, bool VECQ>
__global__ __launch_bounds__(256) void prepare_operands(PrepareArgs a) {
    __shared__ __attribute__((aligned(8))) union {
        CastTile tile;
        uint32_t words[2][256];
    } sm;
    for (uint32_t it = blockIdx.x; it < a.items; it += gridDim.x) {
        if (it != blockIdx.x) __syncthreads();  // the item before has been read
        uint32_t i = it;
        if (i < a.bits_items) {
            bits_transpose_tile(a.packed, a.N, a.K, a.Sw, i % a.bits_x, i / a.bits_x, sm.words);
            continue;
        }
        i -= a.bits_items;
        if (i < a.code_items) {
            cast_transpose_tile<int8_t, VECQ>(a.codes, a.M, a.K, a.K, a.Mp, nullptr, nullptr, a.qT,
                                              (int64_t)(i / a.code_x) * 64, (int64_t)(i % a.code_x) * 64, sm.tile);
            continue;
        }
        i -= a.code_items;
        cast_transpose_tile<float, VECY>(a.dY, a.M, a.N, a.Np, a.Mp, a.row_gamma, a.g, a.gwT,
                                         (int64_t)(i / a.dy_x) * 64, (int64_t)(i % a.dy_x) * 64, sm.tile);
    }
}

static void launch_prepare(const BackwardArgs& b, uint16_t* g, uint32_t* Sw, uint16_t* gwT, uint16_t* qT, int64_t Np,
                           int64_t Mp, hipStream_t s) {
    PrepareArgs a{b.dY, b.codes, b.packed, b.per_tensor ? nullptr : b.gamma, g, gwT, qT, Sw, b.M, b.N, b.K, Np, Mp,
                  0, 0, 0, 1, 1, 1};
    auto tiles = [](int64_t v) { return (v + 63) / 64; };
    int64_t items = 0;
    if (Sw) {
        a.bits_x = (uint32_t)(Np / 32);
        items = (Np / 32) * tiles_k(b.K);
        a.bits_items = (uint32_t)items;
    }
    if (qT) {
        a.code_x = (uint32_t)tiles(b.K);
        a.code_items = (uint32_t)(tiles(b.K) * tiles(Mp));
        items += tiles(b.K) * tiles(Mp);
    }
    // the items cover the padded extents of whichever copies are written
    a.dy_x = (uint32_t)tiles(g ? Np : b.N);
    items += tiles(g ? Np : b.N) * tiles(gwT ? Mp : b.M);
    a.items = (uint32_t)items;
    const unsigned grid = (unsigned)(items < (1 << 23) ? items : (1 << 23));
    const bool vy = b.N % 4 == 0 && ((uintptr_t)b.dY & 15) == 0, vq = b.K % 4 == 0 && ((uintptr_t)b.codes & 15) == 0;
    if (vy && vq) prepare_operands<true, true><<<grid, 256, 0, s>>>(a);
    else if (vy) prepare_operands<true, false><<<grid, 256, 0, s>>>(a);
    else if (vq) prepare_operands<false, true><<<grid, 256, 0, s>>>(a);
    else prepare_operands<false, false><<<grid, 256, 0, s>>>(a);
}

// Tile order of the persistent bf16 kernels.  Workgroups are dealt round-robin to the 8 XCDs (one
// L2 each).  An XCD gets grid_i / 8 whole rows of tiles, and the G / 8 tiles it runs together
// form a blk_i x blk_j block of them: both operands are equally wide here, so what the XCD
// streams from memory per step of the contraction is blk_i + blk_j operand blocks, least for a
// square.  blk_i = 0 (the host found no such blocks for this grid): one contiguous range of tiles
// per XCD, J fastest.  i0 = -1: no tile (the XCD's range ended before the last round did).
__device__ inline void ring_tile_origin(int t, int G, int grid_i, int grid_j, int blk_i, int blk_j,
                                        int BM, int BN, int64_t& i0, int64_t& j0) {
    const int ntiles = grid_i * grid_j;
    int logical = t;
    if ((ntiles & 7) == 0 && (G & 7) == 0) {
        const int q = ((t % G) >> 3) + (t / G) * (G >> 3);
        const int per = ntiles >> 3;
        if (q >= per) {
            logical = -1;
        } else if (blk_i > 0) {
            const int cpx = G >> 3, b = q / cpx, within = q % cpx, bpr = grid_j / blk_j;
            const int row = (t & 7) * (grid_i >> 3) + (b / bpr) * blk_i + within / blk_j;
            const int col = (b % bpr) * blk_j + within % blk_j;
            logical = row * grid_j + col;
        } else {
            logical = (t & 7) * per + q;
        }
    }
    i0 = logical < 0 ? -1 : (int64_t)(logical / grid_j) * BM;
    j0 = logical < 0 ? -1 : (int64_t)(logical % grid_j) * BN;
}

// Slices of the reduction (SPLIT).  A product whose tiles cannot fill the CUs (dX^ of 1000 tokens x
// 2048 columns: 32 tiles) is cut along r as well: work item t is tile t / splits, slice t % splits
// of `per` stages, and C is then the base of the slices' fp32 sums [splits][I][J], which
// fold_slices adds in the order 0, 1, ... and scales.  Workgroups go round-robin to the XCDs, so
// the items of one slice share an L2 when splits divides 8 and the XCD streams only its r range.
struct RingSlices {
    int splits, per;  // per: stages of 32 r in a slice
};

// ---- C[I][J] = scale * sum_r A[I][r] B[J][r], bf16 operands, fp32 accumulation -----------------
// Workgroup tile T x T, four waves of T/2 x T/2, persistent over the tiles.  T = 256: 4 x 4 MFMA tiles a
// wave, one workgroup per CU; T = 128 (few stages or few tiles, dw_plan): 2 x 2, two workgroups per CU.
// A stage is 32 reduction elements: 64-byte rows of A and of B, streamed global -> LDS by
// global_load_lds_dwordx4 into a ring of NS stages; the 16-byte
// segments of a row are XOR-swizzled with (row/4)%4, so the operand reads of 16 consecutive rows
// touch every bank once.  Between the half-steps of stage st every wave waits for its own DMA of
// stage st+1 (s_waitcnt vmcnt(n), n counted by hand), meets the others at a bare s_barrier, and
// the DMA of stage st+NS-1 goes to the buffer stage st-1 has left.
//
// Why four waves (T = 256).  With eight waves of 128 x 64 LDS sets the pace: every operand row is read by the
// waves that share it, 96 KiB of reads and 32 KiB of DMA writes a stage, at 128 bytes a cycle as
// long as the MFMAs of the stage take (1024 cycles).  128 x 128 waves read 64 KiB.  There is one wave
// per SIMD then: 256 accumulator registers (the compiler keeps them in the AGPR half of the file, and the
// other 256 are full: the epilogue's column indices, 8 registers sliced and 2 unsliced, are spilled ahead of the
// tiles and read back behind the last stage, outside the counted waits), and only the wave's own
// instruction stream hides latency.  A half-step (16 r) is 16 MFMAs, 512
// cycles; the reads of the next one's operands go out behind its first four, the DMA of a stage (its
// addresses and issue would idle the pipe) behind each row of four.  M = 8192, 4096 -> 16384: dW
// 900 us, 946 us with eight waves; without any DMA in the loop (timing only) it takes 740 us.
__device__ inline void wide_issue(v4i (&a)[4], v4i (&b)[4], uint32_t ad_a, uint32_t ad_b) {
    asm volatile(
        "ds_read_b128 %0, %8\n\t"
        "ds_read_b128 %1, %8 offset:2048\n\t"
        "ds_read_b128 %2, %8 offset:4096\n\t"
        "ds_read_b128 %3, %8 offset:6144\n\t"
        "ds_read_b128 %4, %9\n\t"
        "ds_read_b128 %5, %9 offset:2048\n\t"
        "ds_read_b128 %6, %9 offset:4096\n\t"
        "ds_read_b128 %7, %9 offset:6144"
        : "=&v"(a[0]), "=&v"(a[1]), "=&v"(a[2]), "=&v"(a[3]), "=&v"(b[0]), "=&v"(b[1]), "=&v"(b[2]),
          "=&v"(b[3])
        : "v"(ad_a), "v"(ad_b));
}
__device__ inline void wide_wait(v4i (&a)[4], v4i (&b)[4]) {
    asm volatile("s_waitcnt lgkmcnt(0)"
                 : "+v"(a[0]), "+v"(a[1]), "+v"(a[2]), "+v"(a[3]), "+v"(b[0]), "+v"(b[1]), "+v"(b[2]),
                   "+v"(b[3]));
}

// the same for 64 x 64 waves
__device__ inline void wide_issue(v4i (&a)[2], v4i (&b)[2], uint32_t ad_a, uint32_t ad_b) {
    asm volatile(
        "ds_read_b128 %0, %4\n\t"
        "ds_read_b128 %1, %4 offset:2048\n\t"
        "ds_read_b128 %2, %5\n\t"
        "ds_read_b128 %3, %5 offset:2048"
        : "=&v"(a[0]), "=&v"(a[1]), "=&v"(b[0]), "=&v"(b[1])
        : "v"(ad_a), "v"(ad_b));
}
__device__ inline void wide_wait(v4i (&a)[2], v4i (&b)[2]) {
    asm volatile("s_waitcnt lgkmcnt(0)" : "+v"(a[0]), "+v"(a[1]), "+v"(b[0]), "+v"(b[1]));
}

template <int T, int NS, bool SPLIT>
__global__ __launch_bounds__(256, T == 256 ? 1 : 2) void gemm_tn_bf16_wide(const uint16_t* __restrict__ A,
                                                            const uint16_t* __restrict__ B,
                                                            int64_t I, int64_t J, int64_t Rp,
                                                            const float* __restrict__ scale_ptr,
                                                            float scale_mul, float* __restrict__ C,
                                                            int grid_i, int grid_j, int blk_i,
                                                            int blk_j, RingSlices sl) {
    constexpr int BM = T, BN = T, WN = 2, THREADS = 256, WTM = T / 2, WTN = T / 2, MI = T / 64, NI = T / 64;
    constexpr int PA = BM * 4 / THREADS, PB = BN * 4 / THREADS, P = PA + PB;
    constexpr int A_BYTES = BM * 64, STAGE_BYTES = (BM + BN) * 64;
    static_assert((NS - 1) * P < 64, "vmcnt range");
    __shared__ __attribute__((aligned(1024))) uint8_t sm[NS * STAGE_BYTES];

    const int w = __builtin_amdgcn_readfirstlane((int)threadIdx.x / kWave), l = threadIdx.x % kWave;
    const int wm = w / WN, wn = w % WN;
    const int j = l & 31, g2 = l >> 5;
    const int nst_all = (int)(Rp / 32);
    const int nitems = grid_i * grid_j * (SPLIT ? sl.splits : 1);
    int nst = nst_all;  // stages of the current work item, the first one st0 (SPLIT)
    int st0 = 0;
    // groups of NS stages whose look-ahead stage st+NS-1 exists for every stage of the group
    int main_groups = nst >= 2 * NS - 1 ? (nst - (2 * NS - 1)) / NS + 1 : 0;

    auto tile_origin = [&](int t, int64_t& i0, int64_t& j0) {
        if constexpr (SPLIT) {
            const int tile = t / sl.splits;
            i0 = (int64_t)(tile / grid_j) * BM;
            j0 = (int64_t)(tile % grid_j) * BN;
        } else {
            ring_tile_origin(t, (int)gridDim.x, grid_i, grid_j, blk_i, blk_j, BM, BN, i0, j0);
        }
    };
    auto set_slice = [&](int t) {
        if constexpr (SPLIT) {
            st0 = (t % sl.splits) * sl.per;
            nst = nst_all - st0 < sl.per ? nst_all - st0 : sl.per;
            main_groups = nst >= 2 * NS - 1 ? (nst - (2 * NS - 1)) / NS + 1 : 0;
        }
    };

    // DMA: thread -> PA + PB pieces of 16 bytes per stage; piece = (row, swizzled segment).
    // Rows past the matrix re-read its last row (their results are never stored).
    uint32_t goffA[PA], goffB[PB];
    const uint8_t *baseA = nullptr, *baseB = nullptr;
    auto setup_dma = [&](int64_t i0, int64_t j0) {
#pragma unroll
        for (int q = 0; q < PA; ++q) {
            const int slot = q * THREADS + threadIdx.x;
            int row = slot >> 2;
            const int seg = ((slot & 3) ^ ((row >> 2) & 3)) * 16;
            if (i0 + row > I - 1) row = (int)(I - 1 - i0);
            goffA[q] = (uint32_t)row * 64 + seg;
        }
#pragma unroll
        for (int q = 0; q < PB; ++q) {
            const int slot = q * THREADS + threadIdx.x;
            int row = slot >> 2;
            const int seg = ((slot & 3) ^ ((row >> 2) & 3)) * 16;
            if (j0 + row > J - 1) row = (int)(J - 1 - j0);
            goffB[q] = (uint32_t)row * 64 + seg;
        }
        baseA = reinterpret_cast<const uint8_t*>(A) + (st0 * I + i0) * 64;
        baseB = reinterpret_cast<const uint8_t*>(B) + (st0 * J + j0) * 64;
    };
    const uint32_t lds_wave = (uint32_t)(w * kWave * 16);
    // stage `st` into ring slot st % NS; `src_st` is the stage whose bytes are read (== st, or
    // the last stage when st does not exist: the slot is filled with bytes nobody uses)
    // (piece q of A and of B)
    static_assert(PA == PB && PA == MI, "one piece of each per row of MFMAs");
    auto issue_piece = [&](int st, int src_st, int q) {
        uint8_t* dst = sm + (st % NS) * STAGE_BYTES + lds_wave;
        __builtin_amdgcn_global_load_lds(
            (const void*)(baseA + src_st * I * 64 + goffA[q]),
            (__attribute__((address_space(3))) void*)(dst + q * THREADS * 16), 16, 0, 0);
        __builtin_amdgcn_global_load_lds(
            (const void*)(baseB + src_st * J * 64 + goffB[q]),
            (__attribute__((address_space(3))) void*)(dst + A_BYTES + q * THREADS * 16), 16, 0, 0);
    };
    auto issue = [&](int st, int src_st) {
#pragma unroll
        for (int q = 0; q < PA; ++q) issue_piece(st, src_st, q);
    };
    auto issue_tile_start = [&]() {
#pragma unroll
        for (int s = 0; s < NS - 1; ++s) issue(s, s < nst ? s : nst - 1);
    };

    // lane's operand addresses inside a stage: row, segment (2h + g2) ^ swizzle
    const int sw = (j >> 2) & 3;
    const uint32_t smb = (uint32_t)(uintptr_t)sm;
    const uint32_t a_lane[2] = {smb + (wm * WTM + j) * 64 + ((g2) ^ sw) * 16,
                                smb + (wm * WTM + j) * 64 + ((2 + g2) ^ sw) * 16};
    const uint32_t b_lane[2] = {smb + A_BYTES + (wn * WTN + j) * 64 + ((g2) ^ sw) * 16,
                                smb + A_BYTES + (wn * WTN + j) * 64 + ((2 + g2) ^ sw) * 16};
    auto ring = [&](int st) { return (uint32_t)((st % NS) * STAGE_BYTES); };

    v16f acc[MI][NI];
    v4i ax[MI], ay[MI], bx[NI], by[NI];
    // acc += ac x bc; an, bn = operands at ad_a, ad_b, valid on return; between(mi) is placed behind the
    // MFMAs of row mi: the DMA of a stage, whose addresses and issue would otherwise idle the pipe
    auto half_step = [&](const v4i(&ac)[MI], const v4i(&bc)[NI], v4i(&an)[MI], v4i(&bn)[NI], uint32_t ad_a,
                         uint32_t ad_b, auto between) {
#pragma unroll
        for (int mi = 0; mi < MI; ++mi) {
#pragma unroll
            for (int s = 0; s < NI; ++s)
                acc[mi][s] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(v8bf, ac[mi]),
                                                                     __builtin_bit_cast(v8bf, bc[s]),
                                                                     acc[mi][s], 0, 0, 0);
            __builtin_amdgcn_sched_barrier(0);
            if (mi == 0) wide_issue(an, bn, ad_a, ad_b);
            between(mi);
            __builtin_amdgcn_sched_barrier(0);
        }
        wide_wait(an, bn);
    };
    // In: ax/bx = operands of (st, half 0).  Out: operands of (st+1, half 0); for the last stage
    // these are stale ring bytes that nobody uses.
    auto stage = [&](int st, bool ahead) {
        half_step(ax, bx, ay, by, a_lane[1] + ring(st), b_lane[1] + ring(st), [](int) {});
        // younger than stage st+1: stages st+2 .. st+NS-2
        if (ahead) wait_vmcnt<(NS - 3) * P>();
        else wait_vmcnt<0>();
        block_barrier();
        half_step(ay, by, ax, bx, a_lane[0] + ring(st + 1), b_lane[0] + ring(st + 1), [&](int mi) {
            if (ahead) issue_piece(st + NS - 1, st + NS - 1, mi);
        });
    };

    const float scale = (scale_ptr ? *scale_ptr : 1.0f) * scale_mul;
    int t = (int)blockIdx.x;
    int64_t i0, j0;
    tile_origin(t, i0, j0);
    if (i0 < 0) return;  // uniform for the whole workgroup
    set_slice(t);
    setup_dma(i0, j0);
    issue_tile_start();

    while (true) {
#pragma unroll
        for (int mi = 0; mi < MI; ++mi)
#pragma unroll
            for (int s = 0; s < NI; ++s)
#pragma unroll
                for (int r = 0; r < 16; ++r) acc[mi][s][r] = 0.f;

        wait_vmcnt<(NS - 2) * P>();  // younger than stage 0: stages 1 .. NS-2
        block_barrier();
        wide_issue(ax, bx, a_lane[0], b_lane[0]);
        wide_wait(ax, bx);

        for (int gidx = 0; gidx < main_groups; ++gidx)
            static_for<0, NS>([&](auto ic) { stage(gidx * NS + decltype(ic)::value, true); });
        for (int st = main_groups * NS; st < nst; ++st) stage(st, st + NS - 1 < nst);

        // every wave is done with the ring: start the next tile's stream, then store
        block_barrier();
        const int t_next = t + (int)gridDim.x;
        int64_t i0n = -1, j0n = -1;
        if (t_next < nitems) tile_origin(t_next, i0n, j0n);
        float* const Cs = SPLIT ? C + (int64_t)(t % sl.splits) * I * J : C;
        if (i0n >= 0) {
            set_slice(t_next);
            setup_dma(i0n, j0n);
            issue_tile_start();
        }

        {
            const int64_t ib = i0 + __builtin_amdgcn_readfirstlane(wm * WTM);
            const int64_t jb = j0 + __builtin_amdgcn_readfirstlane(wn * WTN);
            if constexpr (T < 256) {
                store_tile<MI, NI, true>(Cs + ib * J + jb, J, I - ib, J - jb, j, g2, [](int, int) {},
                                         [&](int mi, int r, int s) { return scale * acc[mi][s][r]; });
            } else  // with 256 accumulators the walk of store_tile spills 29 registers and gains nothing
#pragma unroll
                for (int mi = 0; mi < MI; ++mi)
#pragma unroll
                    for (int r = 0; r < 16; ++r) {
                        const int64_t i = i0 + wm * WTM + 32 * mi + 8 * (r >> 2) + 4 * g2 + (r & 3);
                        if (i >= I) continue;
#pragma unroll
                        for (int s = 0; s < NI; ++s) {
                            const int64_t jj = j0 + wn * WTN + 32 * s + j;
                            if (jj < J) __builtin_nontemporal_store(scale * acc[mi][s][r], &Cs[i * J + jj]);
                        }
                    }
        }
        if (i0n < 0) break;
        t = t_next;
        i0 = i0n;
        j0 = j0n;
    }
}

// ---- dX^: the same persistent kernel with the +-1 operand built from sign words ----------------
// C[I][J] = scale * sum_r A[I][r] S[r][J], A = g (bf16 rows, as above), S given as Sw[r / 32][J]
// (bits_transpose_tile).  Only A goes through the big ring (16 KiB a stage, half the bytes the
// bf16 copy of S would add); a stage of S is one word per column, which each wave fetches for
// its own 64 columns (one 4-byte DMA per lane) into a ring of its own, one stage ahead of A, so
// that the words of stage st+1 can be read while stage st is being multiplied.  A lane turns its
// word into the four dwords of an MFMA operand (eight +-1 bf16 values) with a shift and an
// and-or each, placed between the MFMAs of the half-step before (the same scheduling as in the
// forward GEMM).  BM = 256: waves of 128 x 64, one workgroup per CU; BM = 128 (few tiles, dx_plan): waves of 64 x 64,
// two workgroups per CU.  Group of DMA operations of stage s: the words of stage s+1, then A of stage s; they complete
// in this order, so the hand-counted waits are those of the kernel above with one more operation per stage.
__device__ inline void a_issue(v4i (&a)[4], uint32_t ad) {
    asm volatile(
        "ds_read_b128 %0, %4\n\t"
        "ds_read_b128 %1, %4 offset:2048\n\t"
        "ds_read_b128 %2, %4 offset:4096\n\t"
        "ds_read_b128 %3, %4 offset:6144"
        : "=&v"(a[0]), "=&v"(a[1]), "=&v"(a[2]), "=&v"(a[3])
        : "v"(ad));
}
__device__ inline void a_issue(v4i (&a)[2], uint32_t ad) {
    asm volatile(
        "ds_read_b128 %0, %2\n\t"
        "ds_read_b128 %1, %2 offset:2048"
        : "=&v"(a[0]), "=&v"(a[1])
        : "v"(ad));
}
__device__ inline void words_issue(uint32_t (&wd)[2], uint32_t ad) {
    asm volatile(
        "ds_read_b32 %0, %2\n\t"
        "ds_read_b32 %1, %2 offset:128"
        : "=&v"(wd[0]), "=&v"(wd[1])
        : "v"(ad));
}
__device__ inline void a_wait(v4i (&a)[4]) {
    asm volatile("s_waitcnt lgkmcnt(0)" : "+v"(a[0]), "+v"(a[1]), "+v"(a[2]), "+v"(a[3]));
}
__device__ inline void a_words_wait(v4i (&a)[4], uint32_t (&wd)[2]) {
    asm volatile("s_waitcnt lgkmcnt(0)"
                 : "+v"(a[0]), "+v"(a[1]), "+v"(a[2]), "+v"(a[3]), "+v"(wd[0]), "+v"(wd[1]));
}

__device__ inline void a_wait(v4i (&a)[2]) { asm volatile("s_waitcnt lgkmcnt(0)" : "+v"(a[0]), "+v"(a[1])); }
__device__ inline void a_words_wait(v4i (&a)[2], uint32_t (&wd)[2]) {
    asm volatile("s_waitcnt lgkmcnt(0)" : "+v"(a[0]), "+v"(a[1]), "+v"(wd[0]), "+v"(wd[1]));
}

template <int BM, int NS, bool SPLIT>
__global__ __launch_bounds__(512, BM == 256 ? 2 : 4) void gemm_tn_signs_ring(const uint16_t* __restrict__ A,
                                                             const uint32_t* __restrict__ Sw,
                                                             int64_t I, int64_t J, int64_t Rp,
                                                             const float* __restrict__ scale_ptr,
                                                             float scale_mul, float* __restrict__ C,
                                                             int grid_i, int grid_j, int blk_i,
                                                             int blk_j, RingSlices sl) {
    constexpr int BN = 256, WN = 4, THREADS = 512, WTM = BM / 2, WTN = 64, MI = WTM / 32, NI = 2;
    constexpr int PA = BM * 4 / THREADS, P = PA + 1;  // DMA operations per thread and stage
    constexpr int STAGE_BYTES = BM * 64;
    static_assert((NS - 1) * P + 1 < 64, "vmcnt range");
    __shared__ __attribute__((aligned(1024))) uint8_t sm[NS * STAGE_BYTES];
    __shared__ __attribute__((aligned(256))) uint32_t smW[8][NS][64];  // [wave][slot][column]

    const int w = threadIdx.x / kWave, l = threadIdx.x % kWave;
    const int wm = w / WN, wn = w % WN;
    const int j = l & 31, g2 = l >> 5;
    const int nst_all = (int)(Rp / 32);
    const int nitems = grid_i * grid_j * (SPLIT ? sl.splits : 1);
    int nst = nst_all;  // stages of the current work item, the first one st0 (SPLIT)
    int st0 = 0;
    int main_groups = nst >= 2 * NS - 1 ? (nst - (2 * NS - 1)) / NS + 1 : 0;

    auto tile_origin = [&](int t, int64_t& i0, int64_t& j0) {
        if constexpr (SPLIT) {
            const int tile = t / sl.splits;
            i0 = (int64_t)(tile / grid_j) * BM;
            j0 = (int64_t)(tile % grid_j) * BN;
        } else {
            ring_tile_origin(t, (int)gridDim.x, grid_i, grid_j, blk_i, blk_j, BM, BN, i0, j0);
        }
    };
    auto set_slice = [&](int t) {
        if constexpr (SPLIT) {
            st0 = (t % sl.splits) * sl.per;
            nst = nst_all - st0 < sl.per ? nst_all - st0 : sl.per;
            main_groups = nst >= 2 * NS - 1 ? (nst - (2 * NS - 1)) / NS + 1 : 0;
        }
    };

    uint32_t goffA[PA];
    const uint8_t* baseA = nullptr;
    const uint32_t* wsrc = Sw;  // this lane's column of the sign words, stage 0
    auto setup_dma = [&](int64_t i0, int64_t j0) {
#pragma unroll
        for (int q = 0; q < PA; ++q) {
            const int slot = q * THREADS + threadIdx.x;
            int row = slot >> 2;
            const int seg = ((slot & 3) ^ ((row >> 2) & 3)) * 16;
            if (i0 + row > I - 1) row = (int)(I - 1 - i0);
            goffA[q] = (uint32_t)row * 64 + seg;
        }
        baseA = reinterpret_cast<const uint8_t*>(A) + (st0 * I + i0) * 64;
        int64_t col = j0 + wn * WTN + l;  // columns past J re-read the last one (never stored)
        if (col > J - 1) col = J - 1;
        wsrc = Sw + (int64_t)st0 * J + col;
    };
    const uint32_t lds_wave = (uint32_t)(w * kWave * 16);
    // sign words of stage sb (the last stage's again when sb does not exist) into slot sb % NS
    auto issue_words = [&](int sb) {
        const int src = sb < nst ? sb : nst - 1;
        __builtin_amdgcn_global_load_lds(
            (const void*)(wsrc + (int64_t)src * J),
            (__attribute__((address_space(3))) void*)(&smW[w][sb % NS][0]), 4, 0, 0);
    };
    // the group of stage st: words of stage st+1, then A of stage st
    auto issue = [&](int st, int src_st) {
        issue_words(st + 1);
        uint8_t* dst = sm + (st % NS) * STAGE_BYTES + lds_wave;
#pragma unroll
        for (int q = 0; q < PA; ++q)
            __builtin_amdgcn_global_load_lds(
                (const void*)(baseA + src_st * I * 64 + goffA[q]),
                (__attribute__((address_space(3))) void*)(dst + q * THREADS * 16), 16, 0, 0);
    };
    auto issue_tile_start = [&]() {
        issue_words(0);
#pragma unroll
        for (int s = 0; s < NS - 1; ++s) issue(s, s < nst ? s : nst - 1);
    };

    const int sw = (j >> 2) & 3;
    const uint32_t smb = (uint32_t)(uintptr_t)sm;
    const uint32_t a_lane[2] = {smb + (wm * WTM + j) * 64 + ((g2) ^ sw) * 16,
                                smb + (wm * WTM + j) * 64 + ((2 + g2) ^ sw) * 16};
    auto ring = [&](int st) { return (uint32_t)((st % NS) * STAGE_BYTES); };
    // word of column 32 s + j of this wave (s = 0, 1: +128 bytes) for stage st
    const uint32_t w_lane = (uint32_t)(uintptr_t)&smW[w][0][j];
    auto w_addr = [&](int st) { return w_lane + (uint32_t)((st % NS) * 256); };

    v16f acc[MI][NI];
    v4i ax[MI], ay[MI], bx[NI], by[NI];
    uint32_t wcur[NI], wnext[NI];  // sign words of the current / next stage, shifted by 4 g2
    // bf16 +-1 pair number d of half h from a shifted word: bit 8h + d -> 15, bit 8h + d + 16 -> 31
    // (the two constants live in registers the compiler cannot see through: as literals they
    // would split the and-or into two instructions)
    uint32_t k_signs = 0x80008000u, k_ones = 0x3f803f80u;
    asm volatile("" : "+s"(k_signs), "+v"(k_ones));
    auto pm_one = [&](uint32_t wq, int h, int d) {
        return (int)(((wq << (15 - 8 * h - d)) & k_signs) | k_ones);
    };
    // One half-step: acc += ac x b (MI * NI MFMAs) with the next half-step's +-1 operand bn (half h
    // of the words ws) built between them; the A operand at `ad` is read into an meanwhile, and
    // with WORDS the sign words at `adw` into wr (both valid on return).
    auto half_step = [&](const v4i(&ac)[MI], const v4i(&b)[NI], v4i(&bn)[NI], uint32_t(&ws)[NI],
                         int h, v4i(&an)[MI], uint32_t ad, auto words, uint32_t(&wr)[NI],
                         uint32_t adw, auto between) {
        constexpr bool WORDS = decltype(words)::value;
        a_issue(an, ad);
        if constexpr (WORDS) words_issue(wr, adw);
        asm volatile("" : "+v"(ws[0]), "+v"(ws[1]));
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int mi = 0; mi < MI; ++mi)
#pragma unroll
            for (int s = 0; s < NI; ++s) {
                acc[mi][s] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(
                    __builtin_bit_cast(v8bf, ac[mi]), __builtin_bit_cast(v8bf, b[s]), acc[mi][s], 0, 0, 0);
                constexpr int DW = NI * 4 / (MI * NI);  // dwords of the new operand per MFMA: 1 or 2
                const int q = mi * NI + s;
#pragma unroll
                for (int e = 0; e < DW; ++e) {
                    const int idx = q * DW + e;  // 0 .. 7: dword idx % 4 of sub-tile idx / 4
                    bn[idx >> 2][idx & 3] = pm_one(ws[idx >> 2], h, idx & 3);
                }
                __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
                __builtin_amdgcn_sched_group_barrier(0x002, 2 * DW, 0);
                if (q == 1) {  // the DMA of a stage: behind two MFMAs, not ahead of them
                    __builtin_amdgcn_sched_barrier(0);
                    between();
                    __builtin_amdgcn_sched_barrier(0);
                }
            }
        asm volatile("" : "+v"(bn[0]), "+v"(bn[1]));
        __builtin_amdgcn_sched_barrier(0);
        if constexpr (WORDS) a_words_wait(an, wr);
        else a_wait(an);
    };
    uint32_t wraw[NI];
    auto stage = [&](int st, bool ahead) {
        // MFMAs of (st, half 0); operand of (st, half 1) from this stage's words; the words of stage
        // st+1 (their group landed before the barrier that released stage st) are read meanwhile
        half_step(ax, bx, by, wcur, 1, ay, a_lane[1] + ring(st), std::true_type{}, wraw, w_addr(st + 1),
                  []() {});
        if (ahead) wait_vmcnt<(NS - 3) * P>();  // younger than stage st+1: stages st+2 .. st+NS-2
        else wait_vmcnt<0>();
        block_barrier();
#pragma unroll
        for (int s = 0; s < NI; ++s) wnext[s] = wraw[s] >> (4 * g2);
        half_step(ay, by, bx, wnext, 0, ax, a_lane[0] + ring(st + 1), std::false_type{}, wraw, 0u,
                  [&]() {
                      if (ahead) issue(st + NS - 1, st + NS - 1);
                  });
#pragma unroll
        for (int s = 0; s < NI; ++s) wcur[s] = wnext[s];
    };

    const float scale = (scale_ptr ? *scale_ptr : 1.0f) * scale_mul;
    int t = (int)blockIdx.x;
    int64_t i0, j0;
    tile_origin(t, i0, j0);
    if (i0 < 0) return;  // uniform for the whole workgroup
    set_slice(t);
    setup_dma(i0, j0);
    issue_tile_start();

    while (true) {
#pragma unroll
        for (int mi = 0; mi < MI; ++mi)
#pragma unroll
            for (int s = 0; s < NI; ++s)
#pragma unroll
                for (int r = 0; r < 16; ++r) acc[mi][s][r] = 0.f;

        wait_vmcnt<(NS - 2) * P>();  // younger than stage 0's group: those of stages 1 .. NS-2
        block_barrier();
        a_issue(ax, a_lane[0]);
        words_issue(wraw, w_addr(0));
        a_words_wait(ax, wraw);
#pragma unroll
        for (int s = 0; s < NI; ++s) {
            wcur[s] = wraw[s] >> (4 * g2);
#pragma unroll
            for (int d = 0; d < 4; ++d) bx[s][d] = pm_one(wcur[s], 0, d);
        }

        for (int gidx = 0; gidx < main_groups; ++gidx)
            static_for<0, NS>([&](auto ic) { stage(gidx * NS + decltype(ic)::value, true); });
        for (int st = main_groups * NS; st < nst; ++st) stage(st, st + NS - 1 < nst);

        // every wave is done with the rings: start the next tile's stream, then store
        block_barrier();
        const int t_next = t + (int)gridDim.x;
        int64_t i0n = -1, j0n = -1;
        if (t_next < nitems) tile_origin(t_next, i0n, j0n);
        float* const Cs = SPLIT ? C + (int64_t)(t % sl.splits) * I * J : C;
        if (i0n >= 0) {
            set_slice(t_next);
            setup_dma(i0n, j0n);
            issue_tile_start();
        }

        {
            const int64_t ib = i0 + __builtin_amdgcn_readfirstlane(wm * WTM);
            const int64_t jb = j0 + __builtin_amdgcn_readfirstlane(wn * WTN);
            store_tile<MI, NI, true>(Cs + ib * J + jb, J, I - ib, J - jb, j, g2, [](int, int) {},
                               [&](int mi, int r, int s) { return scale * acc[mi][s][r]; });
        }
        if (i0n < 0) break;
        t = t_next;
        i0 = i0n;
        j0 = j0n;
    }
}

// out = scale * (slice 0 + slice 1 + ...), the sums a split product left.  HBM- (mostly cache-) bound.
// VEC: 16 bytes per lane; the slices always allow it (their rows are a multiple of 32 wide), `out`
// when it is 16-byte aligned.
template <bool VEC>
__global__ __launch_bounds__(256) void fold_slices(const float* __restrict__ part, int splits,
                                                   int64_t count, const float* __restrict__ scale_ptr,
                                                   float scale_mul, float* __restrict__ out) {
    constexpr int E = VEC ? 4 : 1;
    const int64_t i = ((int64_t)blockIdx.x * 256 + threadIdx.x) * E;
    if (i >= count) return;
    const float scale = (scale_ptr ? *scale_ptr : 1.0f) * scale_mul;
    if constexpr (VEC) {
        v4f v = *reinterpret_cast<const v4f*>(part + i);
#pragma unroll 4
        for (int s = 1; s < splits; ++s) v += *reinterpret_cast<const v4f*>(part + s * count + i);
        *reinterpret_cast<v4f*>(out + i) = v * scale;
    } else {
        float v = part[i];
        for (int s = 1; s < splits; ++s) v += part[s * count + i];
        out[i] = v * scale;
    }
}

// The plan of a product: the grid, the block of tiles an XCD runs together (ring_tile_origin):
// blk_i x blk_j = grid / 8 tiles out of its grid_i / 8 rows, as square as the divisors allow; 0 =
// no such tiling; and the slices of the reduction.
struct RingPlan {
    int tile, grid, gi, gj, blk_i, blk_j;  // tile: rows of a tile
    RingSlices sl;
};

// Cost in us of a product in slices of `per` of its nst stages on `cus` CUs: a stage of a tile takes `stage` us on a
// CU, an item `item` us besides (two workgroups of a CU take the time of both), and the fp32 sums of a slice
// (`bytes`) are written and read at `rate` MB/us by a second launch of `fold` us.  These choose the slices (with 0.345,
// 4.5, 4 and 5 for the smaller tile dX over 78 shapes of 256 to 5000 tokens was 1 % slower).
struct RingCost {
    double stage, item, fold, rate;
};
constexpr RingCost kWideCost{0.6, 7.0, 4.0, 5.0};   // 256 x 256
constexpr RingCost kRowsCost{0.33, 4.5, 3.0, 8.0};  // 128 x 256 (dX)
static double ring_cost(RingCost c, int64_t tiles, int64_t nst, int64_t per, double bytes, int64_t cus) {
    const int64_t n = (nst + per - 1) / per, rounds = (tiles * n + cus - 1) / cus;
    return (double)rounds * (c.stage * (double)per + c.item) +
           (n > 1 ? c.fold + (double)n * bytes * 2e-6 / c.rate : 0.0);
}
// The slices that cost least.  dX^ of M = 1000, N = 8192, K = 2048 (64 tiles of 128 x 256 and 256 stages): whole call
// 98.9 us in one slice, 66.9 in two, 53.0 in four, 66.6 in eight (62.8 in six slices of 32 tiles of 256 x 256).
static RingSlices ring_slices(RingCost c, int64_t tiles, int64_t nst, double bytes, int64_t cus) {
    RingSlices best{1, (int)nst};
    double best_cost = 1e30;
    for (int64_t want = 1; want <= 16; ++want) {
        const int64_t per = (nst + want - 1) / want, n = (nst + per - 1) / per;
        if (want > 1 && per < 8) break;
        const double cost = ring_cost(c, tiles, nst, per, bytes, cus);
        if (cost < best_cost * 0.97) {
            best_cost = cost;
            best = RingSlices{(int)n, (int)per};
        }
    }
    return best;
}

static int ring_cus() { return tuning().bwd_grid > 0 ? tuning().bwd_grid : num_cus(); }

// Tiles of bm x bn: 256 x 256; 128 x 256 (dX); 128 x 128 (dW, not sliced).  Of the smaller ones a CU holds two.
static RingPlan ring_plan(int64_t I, int64_t J, int64_t Rp, int bm, int bn) {
    RingPlan p{};
    const int64_t gi = (I + bm - 1) / bm, gj = (J + bn - 1) / bn;
    p.tile = bm;
    p.gi = (int)gi;
    p.gj = (int)gj;
    const int64_t ntiles = gi * gj, nst = Rp / 32;
    p.sl = RingSlices{1, (int)nst};
    if (ntiles == 0 || nst == 0) return p;  // no tokens: nothing to launch (a size query asks)
    if (bn == 256)
        p.sl = ring_slices(bm == 256 ? kWideCost : kRowsCost, ntiles, nst, (double)I * (double)J * 4.0, ring_cus());
    if (const int n = tuning().bwd_splits; n > 0 && bn == 256) {
        const int64_t per = (nst + n - 1) / n;
        p.sl = RingSlices{(int)((nst + per - 1) / per), (int)per};
    }
    const int64_t items = ntiles * p.sl.splits, cap = (int64_t)ring_cus() * (bm == 256 ? 1 : 2);
    const int grid = (int)(cap > items ? items : cap);
    p.grid = grid;
    if (p.sl.splits == 1 && ntiles % 8 == 0 && grid % 8 == 0 && gi % 8 == 0 &&
        (ntiles / 8) % (grid / 8) == 0 && !tuning().bwd_rowmajor) {
        const int cpx = grid / 8;
        const int64_t rx = gi / 8;
        for (int br = 1; br <= cpx; ++br) {
            if (cpx % br) continue;
            const int bc = cpx / br;
            if (br <= rx && bc <= gj && rx % br == 0 && gj % bc == 0 &&
                (p.blk_i == 0 || br + bc < p.blk_i + p.blk_j)) {
                p.blk_i = br;
                p.blk_j = bc;
            }
        }
    }
    return p;
}
// the plan when no room for slices is there
static RingPlan unsliced(RingPlan p, int64_t Rp) {
    const int64_t ntiles = (int64_t)p.gi * p.gj;
    p.sl = RingSlices{1, (int)(Rp / 32)};
    if (p.grid > ntiles) p.grid = (int)ntiles;
    return p;
}
static size_t slices_bytes(const RingPlan& p, int64_t I, int64_t J) {
    return p.sl.splits > 1 ? (size_t)p.sl.splits * I * J * 4 : 0;
}

static void launch_fold(const float* part, const RingPlan& p, int64_t count, const float* scale_ptr,
                        float scale_mul, float* C, hipStream_t s) {
    if (((uintptr_t)C & 15) == 0 && (count & 3) == 0)
        fold_slices<true><<<(unsigned)((count / 4 + 255) / 256), 256, 0, s>>>(
            part, p.sl.splits, count, scale_ptr, scale_mul, C);
    else
        fold_slices<false><<<(unsigned)((count + 255) / 256), 256, 0, s>>>(
            part, p.sl.splits, count, scale_ptr, scale_mul, C);
}

// dX's plan: 256 x 256 tiles, or 128 x 256 where they cost less.  A stage of the smaller tile takes more than half of
// the larger one's time (its waves read and expand the same signs for half the rows), and more still in a single
// round, where a CU has one workgroup, but with few tokens the larger ones are too few for the CUs, or in so many
// slices that their sums cost what the product does.  The constants compare the two, each in the slices chosen above,
// and are fitted to whole calls under either tile, 487 shapes of 100 to 8192 tokens, K and N of 1024 to 28672, half of
// them near the line: 0.25 % slower than the better tile on average, 2.6 % at most where the smaller one is taken, 4.9
// % where the larger one is (with the constants that choose the slices 0.54 %, and 8.4 % at most).  M x K x N, us, 256
// / 128 rows: 1 x 4096 x 16384 47.0 / 36.5, 500 x 4096 x 4096 45.1 / 37.6, 1000 x 2048 x 8192 63.8 / 54.7, 2048 x 4096
// x 4096 91.3 / 76.7, 4000 x 2048 x 8192 166 / 153, 8192 x 1024 x 4096 118 / 97; but 1700 x 2560 x 7680 92.4 / 94.7,
// 677 x 6048 x 6048 72.3 / 78.4, 1000 x 4096 x 16384 136 / 143, 8192 x 4096 x 16384 873 / 908; 4232 x 3456 x 1760,
// 63.3 / 60.3, goes the wrong way.
static RingPlan dx_plan(int64_t I, int64_t J, int64_t Rp) {
    constexpr RingCost kWide{0.615, 12.0, 5.0, 6.0}, kRows{0.33, 5.0, 5.0, 6.0}, kRowsAlone{0.39, 2.0, 5.0, 6.0};
    const RingPlan wide = ring_plan(I, J, Rp, 256, 256), rows = ring_plan(I, J, Rp, 128, 256);
    if (const int force = tuning().bwd_dx) return force == 2 ? rows : wide;
    const int64_t nst = Rp / 32, cus = ring_cus(), tiles = (int64_t)rows.gi * rows.gj;
    const double bytes = (double)I * (double)J * 4.0;
    if (wide.grid == 0) return wide;
    return ring_cost(tiles * rows.sl.splits > cus ? kRows : kRowsAlone, tiles, nst, rows.sl.per, bytes, cus) <
                   ring_cost(kWide, (int64_t)wide.gi * wide.gj, nst, wide.sl.per, bytes, cus)
               ? rows
               : wide;
}

// dW's plan: 256 x 256 tiles, or 128 x 128 where they cost less.  The fixed cost of a 256 x 256 tile (13 us: its
// first DMA, its 64 K outputs stored by four waves) is what a product of a few stages consists of; the
// 128 x 128 tile has a quarter of it and two workgroups per CU, but reads every operand twice as often:
//   a round of 256 x 256, one workgroup per CU   12.8 + 0.68 us per stage
//   of 128 x 128, up to one workgroup per CU      3.6 + 0.23
//   of 128 x 128, two per CU                      4.9 + 0.39
// (a sliced product of 256 x 256 tiles is cheaper, kWideCost).  From two full rounds on the second reading of the
// operands decides: beyond so many stages, or with a B operand well beyond an XCD's 4 MB of L2, the large tile it is.
// Where the small tiles' number is no multiple of 8 they go round the XCDs one by one (ring_tile_origin), and with an
// odd number of columns every XCD then reads all columns of B: 22 % more a stage in products of a round and more, from
// 16 stages on (27 columns, 5115 x 3360 x 3360 161 / 187; 26 columns, 6631 x 3328 x 3328 198 / 189).  Between one and
// two full rounds a stage of the small tile costs more the longer the reduction (with constants as below from 140 to
// 210 stages on): 4779 x 2560 x 4096 149 / 157, 6661 x 2048 x 5120 199 / 212, 6987 x 2560 x 4096 207 / 224, but 5016 x
// 4262 x 2816 172 / 161.  With operands of more than some 140 MB, which with dY before them do not stay in the 256 MB
// cache, a stage of it takes half as long again (7819 x 10120 x 256 167 / 193, 4124 x 18061 x 224 176 / 185; with 120
// MB, 3931 x 16384 x 512, 155 / 135).  From two full rounds on the small tile is taken where it costs up to 2 % more:
// without that 1000 x 16384 x 4096, 184 / 166, goes the wrong way; with it for fewer 1090 x 11456 x 1280, 56 / 62,
// does.  Over 549 shapes of 100 to 8192 tokens, most of them near the line, this was 0.6 % slower than the better tile
// on average without the rules for long reductions and large operands, and 13 of them 10 to 33 % (1700 x 7680 x 2560,
// 117 / 88, beyond `most`).  Up to 32 small tiles count 1.5 us less: the slices' fold is dearer than its bytes there
// (2059 x 512 x 256 28.1 / 24.2; 38 of 5400 drawn shapes, 3 % faster on average).  The whole call (M x N x K, with the
// operand copies), 256 against 128, us: 64 x 2048 x 2048 18.6 / 10.0, 1000 x 2048 x 2048 42.0 / 22.6, 8192 x 6144 x
// 2048 268 / 257, 512 x 8192 x 2048 37.6 / 32.8, 1300 x 8192 x 2048 62.8 / 61.0, 2000 x 8192 x 2048 86.0 / 87.5, 1000
// x 9216 x 3072 89.7 / 78.5, 512 x 16384 x 4096 120.9 / 108.5, 1600 x 16384 x 4096 242.7 / 249.2, 700 x 7168 x 7168
// 133 / 123, 700 x 21504 x 7168 321 / 331, 2000 x 21504 x 7168 647 / 811; in slices 3300 x 4224 x 1056 73.9 / 72.1,
// 6000 x 4224 x 1056 106 / 126.
static RingPlan dw_plan(int64_t I, int64_t J, int64_t Rp) {
    const int force = tuning().bwd_ring;
    if (force == 2) return ring_plan(I, J, Rp, 128, 128);
    const RingPlan p = ring_plan(I, J, Rp, 256, 256);
    if (force == 1 || tuning().bwd_splits > 0 || p.grid == 0) return p;
    const int64_t cus = ring_cus(), nst = Rp / 32, ntiles = (I + 127) / 128 * ((J + 127) / 128);
    const int64_t full = ntiles / (2 * cus), rest = ntiles % (2 * cus);
    const int64_t most = full < 4 ? 44 : full < 9 ? 32 : 16;  // stages
    if (full == 1 && rest && nst > 136) return p;
    if (full >= 2 && (nst > most || J * Rp * 2 > 12000000)) return p;
    const RingCost uncut{0.68, 12.8, 4.0, 5.0};
    const double wide = ring_cost(p.sl.splits > 1 ? kWideCost : uncut, (int64_t)p.gi * p.gj, nst, p.sl.per,
                                  (double)I * (double)J * 4.0, cus);
    const bool scattered = full > 0 && nst >= 16 && ntiles % 8 != 0 && (J + 127) / 128 % 2 != 0;
    const bool cold = (I + J) * Rp * 2 > 140000000;
    const double st = (double)nst * (scattered ? 1.22 : 1.0) * (cold ? 1.5 : 1.0);
    const double two = 4.9 + 0.39 * st, one = 3.6 + 0.226 * st;
    const double small = (double)full * two + (rest > cus ? two : rest ? one : 0.0) - (ntiles <= 32 ? 1.5 : 0.0);
    return small < (full < 2 ? 1.0 : 1.02) * wide ? ring_plan(I, J, Rp, 128, 128) : p;
}

// C[I][J] = scale * A[I][:] . B[J][:], in slices of r where the plan has them and `part` has room
static void launch_gemm_tn(const uint16_t* A, const uint16_t* B, int64_t I, int64_t J, int64_t Rp,
                           const float* scale_ptr, float scale_mul, float* C, float* part,
                           size_t part_bytes, hipStream_t s) {
    RingPlan p = dw_plan(I, J, Rp);
    if (slices_bytes(p, I, J) > part_bytes) p = unsliced(p, Rp);
    if (p.sl.splits > 1) {
        gemm_tn_bf16_wide<256, 4, true><<<(unsigned)p.grid, 256, 0, s>>>(
            A, B, I, J, Rp, nullptr, 1.0f, part, p.gi, p.gj, 0, 0, p.sl);
        launch_fold(part, p, I * J, scale_ptr, scale_mul, C, s);
    } else if (p.tile == 256) {
        gemm_tn_bf16_wide<256, 4, false><<<(unsigned)p.grid, 256, 0, s>>>(
            A, B, I, J, Rp, scale_ptr, scale_mul, C, p.gi, p.gj, p.blk_i, p.blk_j, p.sl);
    } else {
        gemm_tn_bf16_wide<128, 4, false><<<(unsigned)p.grid, 256, 0, s>>>(
            A, B, I, J, Rp, scale_ptr, scale_mul, C, p.gi, p.gj, p.blk_i, p.blk_j, p.sl);
    }
}

// ---------------------------------------------------------------------------------------------
static inline int64_t pad32(int64_t v) { return (v + 31) / 32 * 32; }

// What the copies need: g[M][Np], the sign words [Np / 32][K], gwT[N][Mp], qT[K][Mp] (bf16), each
// region 256-byte aligned.
struct BackwardWs {
    size_t words, gwT, qT, total;
};
static BackwardWs backward_ws(int64_t M, int64_t N, int64_t K) {
    const int64_t Np = pad32(N), Mp = pad32(M);
    auto al = [](size_t v) { return (v + 255) & ~(size_t)255; };
    BackwardWs w{};
    w.words = al((size_t)M * Np * 2);
    w.gwT = w.words + al((size_t)(Np / 32) * K * 4);
    w.qT = w.gwT + al((size_t)N * Mp * 2);
    w.total = w.qT + al((size_t)K * Mp * 2);
    return w;
}
size_t backward_workspace_min_bytes(int64_t M, int64_t N, int64_t K) { return backward_ws(M, N, K).total; }
// The same and room for the slices of whichever product is cut (one after the other): optional.
size_t backward_workspace_bytes(int64_t M, int64_t N, int64_t K) {
    const size_t dx = slices_bytes(dx_plan(M, K, pad32(N)), M, K);
    const size_t dw = slices_bytes(dw_plan(N, K, pad32(M)), N, K);
    const size_t need = backward_ws(M, N, K).total + (dx > dw ? dx : dw);
    // never less than four bf16 copies of a small product's operands, which callers may have budgeted
    const size_t copies = 2 * ((size_t)M * pad32(N) * 2 + (size_t)K * pad32(N) + (size_t)K * pad32(M));
    const bool small = ((M + 255) / 256) * ((K + 255) / 256) < 128;
    return small && need < copies ? copies : need;
}

hipError_t launch_backward(const BackwardArgs& a, hipStream_t s) {
    const int64_t M = a.M, N = a.N, K = a.K, Np = pad32(N), Mp = pad32(M);
    const BackwardWs ws = backward_ws(M, N, K);
    char* base = (char*)a.workspace;
    uint16_t* g = (uint16_t*)base;
    uint32_t* Sw = (uint32_t*)(base + ws.words);
    uint16_t* gwT = (uint16_t*)(base + ws.gwT);
    uint16_t* qT = (uint16_t*)(base + ws.qT);
    float* part = (float*)(base + ws.total);
    const size_t part_bytes = a.workspace_bytes > ws.total ? a.workspace_bytes - ws.total : 0;

    // dY is read once: g for dX and gwT for dW come out of the same pass when both are wanted
    launch_prepare(a, a.dX ? g : nullptr, a.dX ? Sw : nullptr, a.dW ? gwT : nullptr, a.dW ? qT : nullptr, Np, Mp, s);
    if (a.dX) {  // +-1 from sign words inside the kernel: no bf16 copy of the weights
        RingPlan p = dx_plan(M, K, Np);
        if (slices_bytes(p, M, K) > part_bytes) p = unsliced(p, Np);
        if (p.sl.splits > 1) {
            const auto kernel = p.tile == 256 ? gemm_tn_signs_ring<256, 4, true> : gemm_tn_signs_ring<128, 4, true>;
            kernel<<<(unsigned)p.grid, 512, 0, s>>>(g, Sw, M, K, Np, nullptr, 1.0f, part, p.gi, p.gj, 0, 0, p.sl);
            launch_fold(part, p, M * K, a.beta, 1.0f, a.dX, s);
        } else {
            const auto kernel = p.tile == 256 ? gemm_tn_signs_ring<256, 4, false> : gemm_tn_signs_ring<128, 4, false>;
            kernel<<<(unsigned)p.grid, 512, 0, s>>>(g, Sw, M, K, Np, a.beta, 1.0f, a.dX, p.gi, p.gj, p.blk_i, p.blk_j,
                                                    p.sl);
        }
    }
    if (a.dW) {
        launch_gemm_tn(gwT, qT, N, K, Mp, a.per_tensor ? a.gamma : nullptr,
                       a.per_tensor ? 1.0f / 128.0f : 1.0f, a.dW, part, part_bytes, s);
    }
    return hipGetLastError();
}

}  // namespace bl

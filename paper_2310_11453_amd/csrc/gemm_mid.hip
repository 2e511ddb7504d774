// 1-bit x 8-bit GEMM + dequantisation for a few dozen tokens (16 < M <= 64), Eq. 7 and Eq. 11
// of arXiv 2310.11453: the batch between the weight-streaming kernel (M <= 16) and the large
// MFMA tiles; and, walking row tiles of 64 or 128 tokens, for larger batches where the large
// tiles leave CUs idle (gemm_prefill.hip chooses).  One 64 x 128 output tile per workgroup gives
// at most a few hundred workgroups, each with a long serial walk over K, so the walk is split
// INSIDE the workgroup: eight waves, four K-groups of two waves (64 x 64 each; with 128 rows two
// K-groups of four waves), each group streaming its own part of K through its own LDS ring (codes
// and packed bits by global_load_lds, bits expanded in registers, hand-counted vmcnt), all groups
// meeting at the same barriers.  The integer accumulators of the groups are added through LDS at
// the end, each group finishing its share of the tile: the same integers as any other split of K, so the
// result does not depend on it.
//
// What bounds this shape is the stream of activation codes from L2 into LDS: every workgroup
// reads all M x K of them (64 bytes per k against 16 bytes of packed weights), 100 MB per launch
// at the 30B shapes.  L2 serves whole 128-byte lines, so a stage holds 128 k: a row of a stage
// is one line, and the eight lanes that fetch it sit in one DMA instruction.  (With 64-k stages
// every line was requested twice, half of it each time, and the kernel ran at the L2's request
// rate: 1.79 M requests of 128 bytes per launch for 128 MB of operands.)
//
// The walk is two thirds matrix time, at 1.9 GHz (the clock falls from 2.4 within it); the rest of a launch
// of one or two chunks is what stands before and after, and is kept short: integer indices, one row or one
// column of scales a thread, the groups' sums added from their registers' layout, rows stored by adding the
// pitch.  us of the layer before / after that: 200 x 4096 x 16384 27.4 / 25.4, 333 x 2048 x 2048 15.4 / 14.0,
// 333 x 2048 x 6144 19.9 / 17.8, 64 x 7168 x 28672 26.2 / 24.8, 64 x 7168 x 7168 22.5 / 21.7.
//
// A wave expands its weight bits to {0,1} operand bytes with two vector ALU operations per dword,
// for an operand that only two MFMAs use.  That work sits between the MFMAs of the half-step
// before (the compiler's scheduler is told so with sched_group_barrier), two half-steps ahead of
// its use, so a wave keeps the matrix pipe fed without help from the other wave of its SIMD.
#include "common.h"
#include "kernels.h"
#include "ring.h"

namespace bl {

namespace mid {
constexpr int BN = 128, WN = 2;
constexpr int THREADS = 512;
constexpr int STAGE_K = 128;                  // k per stage: a row of a stage is one 128-byte line
constexpr int SPC = kChunkK / STAGE_K;        // stages per 512-chunk: 4
constexpr int P = 4;                          // 16-byte DMA pieces per thread and stage
static_assert(SPC == 4, "tile shape");

// operands of one half-step (rows j and 32 + j of the wave's 64), complete on exit
__device__ inline void read_a(v4i (&a)[2], uint32_t ad) {
    asm volatile(
        "ds_read_b128 %0, %2\n\t"
        "ds_read_b128 %1, %2 offset:4096\n\t"
        "s_waitcnt lgkmcnt(0)"
        : "=&v"(a[0]), "=&v"(a[1])
        : "v"(ad));
}
// packed bits of the lane's two columns (sub-tile s at +2048), two halves of a chunk (+512)
__device__ inline void read_bits(v4i (&bw)[2][2], uint32_t ad) {
    asm volatile(
        "ds_read_b128 %0, %4\n\t"
        "ds_read_b128 %1, %4 offset:512\n\t"
        "ds_read_b128 %2, %4 offset:2048\n\t"
        "ds_read_b128 %3, %4 offset:2560\n\t"
        "s_waitcnt lgkmcnt(0)"
        : "=&v"(bw[0][0]), "=&v"(bw[0][1]), "=&v"(bw[1][0]), "=&v"(bw[1][1])
        : "v"(ad));
}
// The LDS reads stay in asm (a read the compiler can see makes it wait for every DMA in flight).
// lds_issue starts the reads of the next half-step's operands; they become valid at lds_wait,
// which ties the registers so that nothing the compiler schedules can use them earlier.
__device__ inline void lds_issue(v4i (&a)[2], uint32_t ad) {
    asm volatile(
        "ds_read_b128 %0, %2\n\t"
        "ds_read_b128 %1, %2 offset:4096"
        : "=&v"(a[0]), "=&v"(a[1])
        : "v"(ad));
}
__device__ inline void lds_wait(v4i (&a)[2]) {
    asm volatile("s_waitcnt lgkmcnt(0)" : "+v"(a[0]), "+v"(a[1]));
}


// What the kernel wants to know, in 32 bits and with what a division needs worked out by the host: ahead of a launch's
// first request stood 330 instructions, 64-bit products and divisions most of them, and five waits for arguments.
// us a launch, before / now: 64 x 2048 -> 2048 7.7 / 7.3, 64 x 4096 -> 16384 11.5 / 10.9, 64 x 7168 -> 7168 15.5 /
// 15.1, 333 x 2048 -> 2048 8.1 / 7.6, 333 x 8192 -> 2048 16.0 / 15.4.
struct Args {
    const int8_t* codes;
    const uint32_t* packed;
    uint32_t M, N, ldq, last_row, TKp, K, split_k, gmode;  // last_row: of tiles
    uint32_t items, grid_m, div_m, splits, grid_n, div_n, kgroups;
    int64_t group_packed;
    const float *gamma, *beta, *eta;
    const int32_t *rowsum, *wsum;
    uint32_t gstride, beta_rows;
    int64_t beta_stride, ldy;
    bool per_tensor, out_acc, to_slices;
    float* Y;
    int32_t* split_ws;
};
// n / d by a multiplication where the host found it exact (m = 2^32 / d, rounded up; n d < 2^32)
__device__ inline uint32_t divided(uint32_t n, uint32_t d, uint32_t m) {
    return d == 1 ? n : m ? __umulhi(n, m) : n / d;
}
static uint32_t divisor(int64_t d, int64_t n_max) {
    return d > 1 && n_max * d < (int64_t)1 << 32 ? (uint32_t)(((int64_t)1 << 32) / d + 1) : 0;
}
}  // namespace mid

// Tile BM x 128 (64 x 64 per wave): BM = 64 has four K-groups of two waves, BM = 128 two K-groups of
// four.  Work item = (K-slice, column tile, row tile), row tiles fastest; with several row tiles
// (M > 64) each XCD gets one contiguous range of the items, so that the row tiles of a column
// tile, which read the same packed bits, share an L2.  With a.split_k the
// slice's partial sums 2 * sum_k q b go to a.split_ws and splitk_reduce finishes; otherwise the
// workgroup owns all of K and writes Y.
// gmode 2 (a grouped layer, Eq. 13-15): a work item is (column tile, four K-groups of the layer), one
// per K-group of the workgroup: each walks its own layer group's K (its own columns of the codes,
// its own blob) and its sums go, without being added, to that group's slice of a.split_ws.
// gmode 1: a work item is (column tile, one K-group of the layer), split over the workgroup's four.
// NS = stages in each group's ring.
// ROWS = false: one row tile (M <= BM).  STREAM: streaming stores (streaming_stores below).
template <int BM, int NS, bool ROWS, bool STREAM>
__global__ __launch_bounds__(mid::THREADS) void gemm_mid_kernel(mid::Args a) {
    using namespace mid;
    constexpr int WM = BM / 64, GW = WM * WN;   // waves of a K-group
    constexpr int KG = THREADS / kWave / GW;    // K-groups
    constexpr int GT = GW * kWave;              // threads of a K-group
    constexpr int STAGE_BYTES = BM * STAGE_K;   // 8 or 16 KiB
    constexpr int NBW = (BN / 16) / GW;         // packed tiles per wave and chunk
    static_assert(P == BM * (STAGE_K / 16) / GT && NBW * GW * 16 == BN, "tile shape");
    // rings of the K-groups; after the walk the groups' sums meet in the same bytes
    __shared__ __attribute__((aligned(1024))) uint8_t smA[KG * NS * STAGE_BYTES];
    __shared__ __attribute__((aligned(1024))) uint8_t smB[KG * (BN / 16) * 1024];
    static_assert(NS >= 4, "the wait bookkeeping below: a stage's codes are requested NS-1 >= 3 stages ahead");

    // all of the arguments that the first requests need at once, not as the branches come to them
    asm volatile(""
                 : "+s"(a.codes), "+s"(a.packed), "+s"(a.M), "+s"(a.N), "+s"(a.ldq), "+s"(a.last_row), "+s"(a.TKp),
                   "+s"(a.K), "+s"(a.split_k), "+s"(a.gmode));
    if constexpr (ROWS)
        asm volatile("" : "+s"(a.items), "+s"(a.grid_m), "+s"(a.div_m), "+s"(a.splits), "+s"(a.grid_n), "+s"(a.div_n));
    // wave-uniform values in scalar registers: the loop below branches on them
    const int w = __builtin_amdgcn_readfirstlane((int)threadIdx.x / kWave), l = threadIdx.x % kWave;
    const int kg = w / GW, wi = w % GW, wm = wi / WN, wn = wi % WN;
    const int tg = threadIdx.x % GT;  // thread inside the K-group
    const int j = l & 31, g2 = l >> 5;
    const int M = (int)a.M, N = (int)a.N;  // at most 2^30
    int tm = 0, tcol = (int)blockIdx.x, sp = (int)blockIdx.y;
    if constexpr (ROWS) {  // the host rounds the grid up to a multiple of 8
        const uint32_t item = (blockIdx.x & 7) * (gridDim.x >> 3) + (blockIdx.x >> 3);
        if (item >= a.items) return;  // uniform for the workgroup
        const uint32_t rest = divided(item, a.grid_m, a.div_m);
        tm = (int)(item - rest * a.grid_m);
        sp = a.splits > 1 ? (int)divided(rest, a.grid_n, a.div_n) : 0;
        tcol = (int)(rest - (uint32_t)sp * a.grid_n);
    }
    const int m0 = ROWS ? tm * BM : 0;
    const int n0 = tcol * BN;

    // ---- this item's slice of K, then this group's chunks of it ----------------------------
    int ki0 = 0, Ki = (int)a.K;
    const bool to_slices = a.to_slices;  // partial sums go to split_ws
    const int gmode = (int)a.gmode;
    const int lgrp = gmode == 2 ? sp * KG + kg : sp;  // gmode 1, 2: the layer's K-group walked here
    if (gmode) {  // a K-group of a grouped layer: its own codes columns and blob
        const int gi = lgrp < (int)a.kgroups ? lgrp : (int)a.kgroups - 1;
        a.codes += (int64_t)gi * a.K;
        a.packed += (int64_t)gi * a.group_packed;
    } else if (a.split_k) {
        ki0 = sp * (int)a.split_k;
        Ki = Ki - ki0 < (int)a.split_k ? Ki - ki0 : (int)a.split_k;
    }
    const int TKi = (int)((uint32_t)(Ki + kChunkK - 1) / kChunkK);  // K < 2^22
    // gmode 2: the whole group (nothing for a group past the layer's last)
    const int c0 = gmode == 2 ? 0 : TKi * kg / KG;
    const int c1 = gmode == 2 ? (lgrp < (int)a.kgroups ? TKi : 0) : TKi * (kg + 1) / KG;
    const int TK = c1 - c0;
    const int k0 = ki0 + c0 * kChunkK;
    int K = Ki - c0 * kChunkK;  // this group's K
    if (K > TK * kChunkK) K = TK * kChunkK;
    // Every group walks the same number of stages, whole chunks of the longest group; what lies
    // past a group's own K meets zero bits (padding of its last chunk, or a zero mask past its
    // last chunk), so it adds nothing.
    const int TKmax = gmode == 2 ? TKi : (TKi + KG - 1) / KG;
    const int nrun = TKmax * SPC;

    // ---- DMA of this group.  A stage is BM rows of 128 bytes; thread -> four 16-byte pieces of
    // it, piece = (row, physical segment).  The eight lanes of a row sit in one instruction, so
    // the row's line is requested once.  Segments are XOR-swizzled with (row / 2) % 8: the
    // 16-byte operand reads of 16 consecutive rows then touch every LDS bank exactly once.
    uint8_t* const ringA = smA + kg * (NS * STAGE_BYTES);
    uint8_t* const ringB = smB + kg * ((BN / 16) * 1024);
    // (row offsets fit 32 bits: at most 128 rows of less than 2^22 bytes)
    const int8_t* const gbase = a.codes + ((uint64_t)(uint32_t)m0 * a.ldq + (uint32_t)k0);
    static_assert((GT / 8) % 16 == 0, "the pieces of a thread lie in the same segment of their rows");
    const uint32_t gseg = (uint32_t)(((tg & 7) ^ ((tg >> 4) & 7)) * 16);
    uint32_t grow[P];
#pragma unroll
    for (int q = 0; q < P; ++q) {
        const int row = q * (GT / 8) + (tg >> 3);
        grow[q] = __umul24((uint32_t)(row < M - 1 - m0 ? row : M - 1 - m0), a.ldq);
    }
    const uint32_t klast = K >= 16 ? (uint32_t)K - 16 : 0;
    // uniform base, 32-bit offsets: eight rows of tiles of at most 128 KiB
    const uint32_t* const bbase =
        a.packed + ((uint64_t)(uint32_t)(n0 >> 4) * a.TKp + (uint32_t)k0 / kChunkK) * 256;
    uint32_t brow[NBW];
#pragma unroll
    for (int q = 0; q < NBW; ++q) {
        const uint32_t row = (uint32_t)(wi + q * GW), last = a.last_row - (uint32_t)(n0 >> 4);
        brow[q] = (row < last ? row : last) * a.TKp * 256;
    }
    const uint32_t lds_wave = (uint32_t)(wi * kWave * 16);
    // Past the group's K the last 16 valid bytes of the row are read again (the packed bits there are
    // zero, or masked); a min per piece instead of a branch.
    auto issue_piece = [&](int st, int q) {
        const uint32_t k = (uint32_t)(st * STAGE_K) + gseg;
        __builtin_amdgcn_global_load_lds(
            (const void*)(gbase + (grow[q] + (k < klast ? k : klast))),
            (__attribute__((address_space(3))) void*)(ringA + (st % NS) * STAGE_BYTES + q * GT * 16 +
                                                      lds_wave),
            16, 0, 0);
    };
    auto issue = [&](int st) {
#pragma unroll
        for (int q = 0; q < P; ++q) issue_piece(st, q);
    };
    auto issue_bits = [&](int tk) {
#pragma unroll
        for (int q = 0; q < NBW; ++q)
            __builtin_amdgcn_global_load_lds(
                (const void*)(bbase + (brow[q] + (uint32_t)tk * 256 + (uint32_t)l * 4)),
                (__attribute__((address_space(3))) void*)(ringB + (wi + q * GW) * 1024), 16, 0, 0);
    };
    const bool has_k = TK > 0;  // a group without chunks requests nothing and multiplies by zero
    if (has_k) {
        issue_bits(0);
#pragma unroll
        for (int s = 0; s < NS - 1; ++s) issue(s);
    }

    // ---- epilogue operands, behind the first stages' requests (the waits below count those and may so wait for
    // these as well): thread -> one row, or one column, of the tile (waves 0 .. BM/64 - 1 the rows, waves 4 and
    // 5 the columns; nothing for sums that go to slices)
    int e0 = 0, e1 = 0, e2 = 0;
    if (!to_slices) {
        if (w < BM / kWave) {
            const int r = m0 + (int)threadIdx.x;
            const int64_t m = (int64_t)(r < M ? r : M - 1) * a.gstride, mg = a.per_tensor ? 0 : m;
            e0 = __float_as_int(a.gamma[mg]);
            e1 = a.rowsum[m];
            if (a.eta) e2 = __float_as_int(a.eta[mg]);
        } else if (w == 4 || w == 5) {
            const int c = n0 + (int)threadIdx.x - 4 * kWave, n = c < N ? c : N - 1;
            int64_t at = 0;
            if ((int)a.beta_rows < N) at = (int64_t)((uint32_t)n / a.beta_rows) * a.beta_stride;
            e0 = __float_as_int(a.beta[at]);
            if (a.eta) e1 = a.wsum[n];
        }
    }

    const uint32_t b_lane = (uint32_t)(uintptr_t)ringB + ((wn * 64 + j) >> 4) * 1024 +
                            (g2 * 16 + (j & 15)) * 16;
    // lane (j, g2) reads logical segment 2 hs + g2 of row j in half-step hs of a stage
    const int sw = (j >> 1) & 7;
    uint32_t a_lane[4];
#pragma unroll
    for (int hs = 0; hs < 4; ++hs)
        a_lane[hs] = (uint32_t)(uintptr_t)ringA + (wm * 64 + j) * STAGE_K + ((2 * hs + g2) ^ sw) * 16;
    auto a_addr = [&](int st, int hs) { return a_lane[hs] + (uint32_t)((st % NS) * STAGE_BYTES); };

    v16i acc[2][2];
#pragma unroll
    for (int mi = 0; mi < 2; ++mi)
#pragma unroll
        for (int s2 = 0; s2 < 2; ++s2)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[mi][s2][r] = 0;
    // Packed bits of the current chunk and of the next one; plane i of half h of a chunk as {0,1}
    // bytes, nothing past the group's last chunk.  Half-step u of a chunk (plane u / 2, half u % 2)
    // multiplies A[u % 2] by B[u % 4], starts the LDS reads of A[(u + 1) % 2] and builds B[(u + 2) % 4].
    v4i bw[2][2], bwn[2][2];
    v4i A[2][2], B[4][2];
    wait_vmcnt<(NS - 2) * P>();  // younger than stage 0: stages 1 .. NS-2
    block_barrier();
    read_bits(bw, b_lane);
    read_a(A[0], a_addr(0, 0));
    {
        const uint32_t m01 = 0 < TK ? 0x01010101u : 0u;
#pragma unroll
        for (int h = 0; h < 2; ++h)
#pragma unroll
            for (int s2 = 0; s2 < 2; ++s2)
#pragma unroll
                for (int d = 0; d < 4; ++d) B[h][s2][d] = (int)((uint32_t)bw[s2][h][d] & m01);
    }

    // DMA bookkeeping: at the wait of stage st the operations younger than stage st+1 are those of
    // stages st+2 .. st+NS-2 and the bits of the next chunk while they may still be on their way:
    // they are requested in stage 0 of a chunk BEHIND that stage's codes (the buffer is free once
    // every wave has read the current chunk's bits, one barrier earlier), so they are younger than
    // what the waits of stages 1 and 2 are for, and the wait of stage 3, which is for a group
    // requested after them, covers them: three stages for a trip to HBM, then they are read.
    for (int c = 0; c < TKmax; ++c) {
        const bool bits_next = c + 1 < TK;
        static_for<0, 16>([&](auto uc) {
            constexpr int u = decltype(uc)::value;
            constexpr int s = u >> 2, hs = u & 3;
            const int st = c * SPC + s;
            if constexpr (hs == 2) {  // mid-stage: stage st+1 becomes readable, stage st-1's buffer free
                const bool ahead = st + NS - 1 < nrun;
                if (!ahead) wait_vmcnt<0>();
                else if (bits_next && (s == 1 || s == 2)) wait_vmcnt<(NS - 3) * P + NBW>();
                else wait_vmcnt<(NS - 3) * P>();
                block_barrier();
                if (s == 3) read_bits(bwn, b_lane);
            }
            // stage st + NS - 1 goes out behind the MFMAs of this half-step (two pieces) and of the next
            // (two more, then in stage 0 the bits): in one piece behind the barrier, with a branch per
            // piece for the end of K, it idled the matrix pipe of all waves at once (7168 -> 28672 at
            // M = 64: 22.8 us, now 21.2)
            const bool more = hs >= 2 && has_k && st + NS - 1 < nrun;
            constexpr int u2 = u + 2;  // the operand built in this half-step
            constexpr int i2 = (u2 >> 1) & 7, h2 = u2 & 1;
            v4i(&src)[2][2] = u2 >= 16 ? bwn : bw;
            const uint32_t m01 = (u2 >= 16 ? c + 1 : c) < TK ? 0x01010101u : 0u;
            v4i(&an)[2] = A[(u + 1) & 1];
            v4i(&bn)[2] = B[u2 & 3];
            lds_issue(an, a_addr(hs == 3 ? st + 1 : st, (hs + 1) & 3));
            // the bits pass through an (empty) asm placed after the reads, and the new operand
            // through one at the end: the expansion can neither be moved ahead of this half-step
            // nor be left for a later one before the scheduler sees the groups below
            asm volatile("" : "+v"(src[0][h2]), "+v"(src[1][h2]));
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int mi = 0; mi < 2; ++mi)
#pragma unroll
                for (int s2 = 0; s2 < 2; ++s2) {
                    acc[mi][s2] = __builtin_amdgcn_mfma_i32_32x32x32_i8(A[u & 1][mi], B[u & 3][s2],
                                                                        acc[mi][s2], 0, 0, 0);
                    const int q = mi * 2 + s2;  // two of the eight dwords of the new operand per MFMA
#pragma unroll
                    for (int e = 0; e < 2; ++e) {
                        const int d = (q & 1) * 2 + e, sn = q >> 1;
                        bn[sn][d] = (int)(((uint32_t)src[sn][h2][d] >> i2) & m01);
                    }
                    __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
                    __builtin_amdgcn_sched_group_barrier(0x002, 4, 0);
                    if constexpr (hs >= 2) {
                        if (s2 == 1) {
                            __builtin_amdgcn_sched_barrier(0);
                            if (more) issue_piece(st + NS - 1, (hs - 2) * 2 + mi);
                            __builtin_amdgcn_sched_barrier(0);
                        }
                    }
                }
            asm volatile("" : "+v"(bn[0]), "+v"(bn[1]));
            __builtin_amdgcn_sched_barrier(0);
            if constexpr (u == 3) {
                if (bits_next) issue_bits(c + 1);
            }
            lds_wait(an);
        });
#pragma unroll
        for (int s2 = 0; s2 < 2; ++s2)
#pragma unroll
            for (int h = 0; h < 2; ++h) bw[s2][h] = bwn[s2][h];
    }
    wait_vmcnt<0>();
    __syncthreads();  // every group is done with its ring

    // ---- add the groups.  Lane (j, g2) of wave (wm, wn) holds columns 64 wn + 32 s + j, rows 64 wm +
    // 32 mi + 8 q + 4 g2 + 0..3 as pieces (mi, s, q) of four; the waves (wm, wn) of the KG groups hold sums
    // of the same 64 x 64 outputs.  Group g finishes 16 / KG of the pieces: every wave leaves the
    // others' in LDS as they lie in its registers (16 bytes a lane, no conflicts), and after one
    // barrier reads its own from the other groups.  (Adding in the tile's layout, half of the waves after the
    // other and then all of them reading it back, took 1.1 us of a 20 us launch and a barrier more.)
    constexpr int OWN = 16 / KG;
    v4i own[OWN];
    int* const red = reinterpret_cast<int*>(smA);
    // where group `from` of waves wi leaves piece i of group `to`
    auto slot = [&](int from, int to, int i) {
        const int rank = to < from ? to : to - 1;  // of the KG - 1 groups it writes to
        return red + ((((wi * KG + from) * (KG - 1) + rank) * OWN + i) * kWave + l) * 4;
    };
    static_assert(GW * KG * (KG - 1) * OWN * kWave * 16 + 4096 <= KG * NS * STAGE_BYTES, "room beside the scales");
    auto piece = [&](int q) {
        const v16i& t = acc[q >> 3][(q >> 2) & 1];
        const int r = (q & 3) * 4;
        return (v4i){t[r], t[r + 1], t[r + 2], t[r + 3]};
    };
    int* const scales = red + GW * KG * (KG - 1) * OWN * kWave * 4;  // gamma, row sums, eta; beta, column sums
    const bool add_groups = gmode != 2;
    if (add_groups) {
        static_for<0, KG>([&](auto gc) {
            constexpr int g = decltype(gc)::value;
            if (kg == g) {  // uniform for the wave
                static_for<0, 16>([&](auto qc) {
                    constexpr int q = decltype(qc)::value;
                    if constexpr (q / OWN == g) own[q % OWN] = piece(q);
                    else *reinterpret_cast<v4i*>(slot(g, q / OWN, q % OWN)) = piece(q);
                });
            }
        });
        if (!to_slices) {
            if (w < BM / kWave) {
                scales[threadIdx.x] = e0;
                scales[BM + threadIdx.x] = e1;
                scales[2 * BM + threadIdx.x] = e2;
            } else if (w == 4 || w == 5) {
                scales[3 * BM + threadIdx.x - 4 * kWave] = e0;
                scales[3 * BM + BN + threadIdx.x - 4 * kWave] = e1;
            }
        }
        __syncthreads();
#pragma unroll
        for (int d = 1; d < KG; ++d) {
            const int from = (kg + d) % KG;
#pragma unroll
            for (int i = 0; i < OWN; ++i) own[i] += *reinterpret_cast<const v4i*>(slot(from, kg, i));
        }
    }

    // ---- store: sum_k q s = 2 sum_k q b - sum_k q ; y = that * (beta gamma / 128) (Eq. 11) --------
    // 32 consecutive columns of two rows an instruction, whole lines.  What a store costs here is the
    // instructions around it (3 us a tile with a row's bounds, branches and 64-bit product at each): the rows
    // are walked by adding the pitch, with a count of the valid ones where the tile is ragged.
    const bool inside = m0 + BM <= M && n0 + BN <= N;  // uniform
    const int prow = wm * 64 + 4 * g2, pcol = wn * 64 + j;  // of piece q: + 32 (q / 8) + 8 (q % 4), + 32 (q / 4 % 2)
    auto put = [](auto v, auto* at) {
        if constexpr (STREAM) __builtin_nontemporal_store(v, at);
        else *at = v;
    };
    auto store_sums = [&](const v4i& p, int q, int64_t grp) {
        const int m = m0 + prow + 32 * (q >> 3) + 8 * (q & 3), n = n0 + pcol + 32 * ((q >> 2) & 1);
        int32_t* o = a.split_ws + (grp * M + m) * N + n;
        const int rows = n < N ? (M - m < 4 ? M - m : 4) : 0;
#pragma unroll
        for (int rr = 0; rr < 4; ++rr, o += N)
            if (inside || rr < rows) put(2 * p[rr], o);
    };
    if (!add_groups) {  // each group's sums to its layer group's slice
        if (lgrp < (int)a.kgroups)
            static_for<0, 16>([&](auto qc) {
                store_sums(piece(decltype(qc)::value), decltype(qc)::value, lgrp);
            });
        return;
    }
    if (to_slices) {
#pragma unroll
        for (int i = 0; i < OWN; ++i) store_sums(own[i], kg * OWN + i, sp);
        return;
    }
    // kind 0: a tile inside the output; 1: a ragged one; 2: either, int32 output
    auto store = [&](auto with_eta, auto kind) {
        constexpr bool ETA = decltype(with_eta)::value;
        constexpr int KIND = decltype(kind)::value;
#pragma unroll
        for (int i = 0; i < OWN; ++i) {
            const int q = kg * OWN + i;
            const int row = prow + 32 * (q >> 3) + 8 * (q & 3), col = pcol + 32 * ((q >> 2) & 1);
            const v4f gm = *reinterpret_cast<const v4f*>(scales + row);
            const v4i rs = *reinterpret_cast<const v4i*>(scales + BM + row);
            v4f eta = {};
            if constexpr (ETA) eta = *reinterpret_cast<const v4f*>(scales + 2 * BM + row);
            const float beta = __int_as_float(scales[3 * BM + col]);
            const float ws = ETA ? (float)scales[3 * BM + BN + col] : 0.f;
            float* o = a.Y + (int64_t)(m0 + row) * a.ldy + (n0 + col);
            const int left = M - m0 - row;
            const int rows = n0 + col < N ? (left < 4 ? left : 4) : 0;
#pragma unroll
            for (int rr = 0; rr < 4; ++rr, o += a.ldy) {
                const int pm = 2 * own[i][rr] - rs[rr];
                if constexpr (KIND == 2) {
                    if (rr < rows) *reinterpret_cast<int*>(o) = pm;
                    continue;
                }
                // beta * (gamma / 128) has the bits of (beta * gamma) / 128 (gamma / 128 is exact)
                float y = (float)pm * (beta * (gm[rr] * 0.0078125f));
                if constexpr (ETA) y = y + (beta * eta[rr]) * ws;  // Eq. 6
                if (KIND == 0 || rr < rows) put(y, o);
            }
        }
    };
    auto store_kind = [&](auto with_eta) {
        if (inside) store(with_eta, std::integral_constant<int, 0>{});
        else store(with_eta, std::integral_constant<int, 1>{});
    };
    if (a.out_acc) store(std::false_type{}, std::integral_constant<int, 2>{});
    else if (a.eta) store_kind(std::true_type{});
    else store_kind(std::false_type{});
}

// Small batches (16 < M <= 64) leave most of the chip idle when N supplies few 64 x 128 tiles: K is
// then split over workgroups too, and splitk_reduce folds the slices.

// 512-chunks of K per slice of the workspace that a call must bring (0 = no slices): about one work
// item per CU, sums no larger than the packed weights.  256 CUs are assumed.  This is only the size that
// calls have always been required to bring; the launch decides by mid_slice_tiles what it makes of it.
int64_t prefill_split_tiles(int64_t M, int64_t N, int64_t K) {
    if (M <= 16 || M > 64) return 0;
    if (const int64_t per = tuning().mid_split_tiles) return per > 0 && per < tiles_k(K) ? per : 0;
    const int64_t tiles = ((M + 63) / 64) * ((N + 127) / 128), TK = tiles_k(K);
    if (tiles > 128) return 0;
    int64_t smax = 256 / tiles;
    if (smax > K / (32 * M)) smax = K / (32 * M);
    if (smax > 16) smax = 16;
    if (smax < 2) return 0;
    int64_t per = (TK + smax - 1) / smax;
    if (per < 2) per = 2;
    return (TK + per - 1) / per >= 2 ? per : 0;
}

// What the launch takes of ws_bytes: the slices of least cost, in us: a round of items 3.5 + 4.1 c (c
// 512-chunks per K-group of the workgroup), the slices 6.5 and their sums written and read at 5 TB/s.
// The layer, us, M x K x N: 64 x 7168 x 7168 18.8 in 4 slices, 19.7 in 2, 19.9 without; 48 x 4096 x 12288
// 14.5 without, 17.0 in 2; 48 x 16384 x 4096 20.1 in the 8 taken, 20.7 in 4, 31.4 without; 48 x 8192 x
// 2048 15.6 in the 4 taken, 17.8 in 2, 20.1 without.  Over 54 shapes (18 K x N, 33 to 64 tokens) the slices taken
// are at most 1.2 % slower than the best number of them.  Returns 512-chunks per slice, 0 = no slices.
static int64_t mid_slice_tiles(int64_t M, int64_t N, int64_t K, size_t ws_bytes) {
    const int64_t TK = tiles_k(K), tiles = (N + mid::BN - 1) / mid::BN;
    if (const int64_t per = tuning().mid_split_tiles)
        return per > 0 && per < TK && (size_t)((TK + per - 1) / per) * M * N * 4 <= ws_bytes ? per : 0;
    int64_t best = 0;
    double best_us = 1e30;
    for (int64_t want = 1; want <= 16; ++want) {
        const int64_t per = (TK + want - 1) / want, n = (TK + per - 1) / per;
        const double bytes = (double)n * (double)M * (double)N * 4.0;
        if (n > 1 && bytes > (double)ws_bytes) continue;
        const double us = (double)((tiles * n + 255) / 256) * (3.5 + 4.1 * (double)((per + 3) / 4)) +
                          (n > 1 ? 6.5 + bytes * 2.0 / 5e6 : 0.0);
        if (us < best_us) {
            best_us = us;
            best = n > 1 ? per : 0;
        }
    }
    return best;
}
// Room for them (32 < M <= 64), where it is more than the required slices take: optional.
size_t mid_split_bytes(int64_t M, int64_t N, int64_t K) {
    if (M <= 32 || M > 64) return 0;
    const int64_t per = mid_slice_tiles(M, N, K, (size_t)1 << 40);
    const size_t bytes = per ? (size_t)((tiles_k(K) + per - 1) / per) * M * N * 4 : 0;
    return bytes > gemm_split_ws_bytes(M, N, K) ? bytes : 0;
}

// Whether a launch's stores are streaming: whole lines only (others 1 % slower), the slices of a K split (64 x 7168 ->
// 7168 21.3 us / 20.6), and outputs from 4 MiB on (200 x 4096 -> 16384 22.5 / 21.15; of layers at 65 to 4096
// tokens 1.3 % by themselves and still 0.7 % with a pass over Y behind; smaller outputs lose 0.5 % with that pass).
// Slices of K-groups are not: their fold gets slower by more (64 x 6144 -> 21860 in four groups 36 / 31).
static bool streaming_stores(const GemmArgs& a, int splits, bool grouped) {
    if (grouped || (a.N | a.ldy) & 31) return false;
    return splits > 1 || a.M * a.ldy >= (int64_t)1 << 20;
}

static mid::Args mid_args(const GemmArgs& a, int grid_m, int grid_n, int splits, int gmode) {
    const int64_t items = (int64_t)grid_m * grid_n * splits;
    mid::Args m{};
    m.codes = a.codes;
    m.packed = a.packed;
    m.M = (uint32_t)a.M;
    m.N = (uint32_t)a.N;
    m.ldq = (uint32_t)a.ldq;
    m.last_row = (uint32_t)tiles_n(a.N) - 1;
    m.TKp = (uint32_t)(a.tk_pitch ? a.tk_pitch : tiles_k(a.K));
    m.K = (uint32_t)a.K;
    m.split_k = (uint32_t)a.split_k;
    m.grid_m = (uint32_t)grid_m;
    m.grid_n = (uint32_t)grid_n;
    m.splits = (uint32_t)splits;
    m.items = (uint32_t)items;
    m.div_m = mid::divisor(grid_m, items);
    m.div_n = mid::divisor(grid_n, (int64_t)grid_n * splits);
    m.gmode = (uint32_t)gmode;
    m.kgroups = (uint32_t)a.kgroups;
    m.group_packed = a.group_packed;
    m.gamma = a.gamma;
    m.beta = a.beta;
    m.eta = a.eta;
    m.rowsum = a.rowsum;
    m.wsum = a.wsum;
    m.gstride = (uint32_t)a.gstride;
    m.beta_rows = (uint32_t)a.beta_rows;
    m.beta_stride = a.beta_stride;
    m.ldy = a.ldy;
    m.per_tensor = a.per_tensor;
    m.out_acc = a.out_acc;
    m.to_slices = a.split_k || a.kgroups > 1;
    m.Y = a.Y;
    m.split_ws = a.split_ws;
    return m;
}

// 16 < M <= 64.  K is also split over workgroups (second kernel: splitk_reduce) when N gives
// few tiles and the caller brought the workspace for it, as mid_slice_tiles decides.
hipError_t launch_gemm_mid(const GemmArgs& a_in, hipStream_t s) {
    GemmArgs a = a_in;
    a.split_k = 0;
    if (!a.ldy) a.ldy = a.N;
    if (a.M > 64 || a.K >= ((int64_t)1 << 22) || a.ldq >= ((int64_t)1 << 22))
        return hipErrorInvalidValue;
    const int grid_n = (int)((a.N + mid::BN - 1) / mid::BN);
    int splits = 1;
    const int64_t per = a.split_ws && a.kgroups <= 1 && !tuning().mid_nosplit
                            ? mid_slice_tiles(a.M, a.N, a.K, a.split_ws_bytes) : 0;
    int gmode = 0;
    if (a.kgroups > 1) {  // the caller sized split_ws for one slice per K-group
        if (!a.split_ws || a.split_ws_bytes < (size_t)a.kgroups * a.M * a.N * 4)
            return hipErrorInvalidValue;
        // four K-groups per work item, one per K-group of the workgroup, unless the layer's groups
        // are long enough to be worth splitting over the workgroup's four themselves
        gmode = tuning().group_slices || tiles_k(a.K) >= 8 ? 1 : 2;
        splits = gmode == 2 ? (a.kgroups + 3) / 4 : a.kgroups;
    } else if (per) {
        splits = (int)((tiles_k(a.K) + per - 1) / per);
        a.tk_pitch = a.tk_pitch ? a.tk_pitch : tiles_k(a.K);
        a.split_k = per * kChunkK;
    }
    const dim3 grid((unsigned)grid_n, (unsigned)splits);
    const mid::Args args = mid_args(a, 1, grid_n, splits, gmode);
    if (streaming_stores(a, splits, gmode != 0)) gemm_mid_kernel<64, 4, false, true><<<grid, mid::THREADS, 0, s>>>(args);
    else gemm_mid_kernel<64, 4, false, false><<<grid, mid::THREADS, 0, s>>>(args);
    if (splits > 1 || gmode) launch_splitk_reduce(a, gmode ? a.kgroups : splits, s);
    return hipGetLastError();
}

// M > 64: bm x 128 tiles (bm = 64 or 128), K in slices of `per` 512-chunks (per >= the chunks of K: no
// slices; else a.split_ws must hold slices * M * N * 4 bytes).  A grouped layer: a slice per K-group.
hipError_t launch_gemm_mid_tiles(const GemmArgs& a_in, int bm, int64_t per, hipStream_t s) {
    GemmArgs a = a_in;
    const int64_t TK = tiles_k(a.K);
    const int grid_m = (int)((a.M + bm - 1) / bm), grid_n = (int)((a.N + mid::BN - 1) / mid::BN);
    const bool grouped = a.kgroups > 1;
    const int splits = grouped ? a.kgroups : (int)((TK + per - 1) / per);
    a.split_k = 0;
    if (splits > 1) {
        if (!a.split_ws || a.split_ws_bytes < (size_t)splits * a.M * a.N * 4) return hipErrorInvalidValue;
        a.tk_pitch = a.tk_pitch ? a.tk_pitch : TK;
        if (!grouped) a.split_k = per * kChunkK;
    }
    int64_t items = (int64_t)grid_m * grid_n * splits;
    if (items > ((int64_t)1 << 30)) return hipErrorInvalidValue;
    items = (items + 7) / 8 * 8;
    auto launch = [&](auto kernel) {
        kernel<<<(unsigned)items, mid::THREADS, 0, s>>>(mid_args(a, grid_m, grid_n, splits, grouped));
    };
    const bool streaming = streaming_stores(a, splits, grouped);
    if (bm == 64) launch(streaming ? gemm_mid_kernel<64, 4, true, true> : gemm_mid_kernel<64, 4, true, false>);
    else launch(streaming ? gemm_mid_kernel<128, 4, true, true> : gemm_mid_kernel<128, 4, true, false>);
    if (splits > 1) launch_splitk_reduce(a, splits, s);
    return hipGetLastError();
}

}  // namespace bl

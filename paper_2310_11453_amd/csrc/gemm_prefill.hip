// 1-bit x 8-bit GEMM + dequantisation for many tokens (prefill / training):
//   Y[m,n] = (sum_k q[m,k] * s[n,k]) * beta * gamma_m / 128     (Eq. 7, Eq. 11)
// of arXiv 2310.11453.  Compute-bound: the contraction runs on the i8 MFMA
// (v_mfma_i32_32x32x32_i8, int32 accumulators).
//
// Tiling.  A workgroup computes a BM x BN block of Y; a wave a WTM x WTN part of it.
//  * Activation codes (int8) are streamed global -> LDS with the direct
//    global_load_lds_dwordx4 path, no registers in between, through a ring of NS
//    stages of BM rows x 64 k.  The 16-byte segments of a row are XOR-swizzled with
//    (row/4)%4 so that the 16-byte operand reads of 16 consecutive rows hit every LDS
//    bank exactly once.
//  * The 1-bit weights of the block's BN columns for one 512-chunk (BN/16 packed tiles of
//    1 KiB) take the same DMA path into a small LDS buffer, one chunk ahead.  Once per
//    chunk each lane copies the 16-byte groups of its own columns to registers (16 bytes
//    cover 16 k in each of the eight 64-wide sub-blocks of the chunk) and expands them
//    right before use, never as bytes in LDS:
//        b = (w << (7 - i)) & 0x80808080     four {0,-128} bytes, two VALU operations
//    amortised over the WTM/32 MFMAs that reuse the operand.  The MFMA accumulates
//    -128 sum_k q b (K <= kMaxGemmK: at most 2^30); the epilogue restores sum_k q s = 2 sum_k q b - sum_k q
//    with the row sums of the codes that the quantiser already produced.
//  * Which operand is which, and the value a set bit has, cost power, and at large batches power is
//    what the clock is made of: a register-resident loop over these operands reaches 4.65 POP/s with the
//    codes as the first operand and {0,-128} weights, 4.4 with {0,1}, 3.8 with +-1 or with the
//    weights as the first operand.
//  * A 128 x 64 wave tile keeps LDS traffic (one 1 KiB operand read per two MFMAs) and
//    expansion cost (16 VALU per 8 MFMAs) well below the MFMA time.
//  * Eight waves share a 256 x 256 (or 128 x 256) block, one block per CU.  The L2 -> LDS
//    stream of codes is BM*K bytes per block, i.e. 2*BN operations per byte: with BN = 256
//    the whole chip needs ~5 TB/s of it at half the MFMA peak, and with a latency of about
//    2 us that is ~40 KiB in flight per CU, hence the deep ring (NS = 8 stages of 16 KiB).
//
// Schedule.  The unit of work is a half-step: 32 k of a stage, MI*NI MFMAs.  It starts the LDS
// reads of the NEXT half-step's activation operand (asm), issues the MFMAs of the current one
// with the expansion of the next weight operand scheduled between them, then waits for the
// reads (asm): LDS latency and expansion both hide under the MFMAs.  (An LDS read the compiler
// can see makes it drain the whole DMA queue first, because it cannot tell the read from the
// DMA's target; the registers of a read in flight are tied to the asm that waits for it, so
// nothing can use them earlier.)
// Between the two half-steps of stage st every wave waits for its own DMA of stage st+1
// (s_waitcnt vmcnt(n), n counted by hand) and meets the others at a bare s_barrier (no
// fence: a fence would drain every DMA in flight).  After that barrier stage st+1 is
// readable and the buffer of stage st-1 is free, so the DMA of stage st+NS-1 goes there.
#include "common.h"
#include "kernels.h"
#include "ring.h"

namespace bl {

constexpr int kStageK = 64;  // k per LDS stage (= bytes per staged row)

// ---- asm blocks ----------------------------------------------------------------------
// Operand reads of one half-step (sub-tile mi at +2048*mi), complete on exit.
__device__ inline void lds_read_a(v4i (&a)[4], uint32_t ad) {
    asm volatile(
        "ds_read_b128 %0, %4\n\t"
        "ds_read_b128 %1, %4 offset:2048\n\t"
        "ds_read_b128 %2, %4 offset:4096\n\t"
        "ds_read_b128 %3, %4 offset:6144\n\t"
        "s_waitcnt lgkmcnt(0)"
        : "=&v"(a[0]), "=&v"(a[1]), "=&v"(a[2]), "=&v"(a[3])
        : "v"(ad));
}
__device__ inline void lds_read_a(v4i (&a)[2], uint32_t ad) {
    asm volatile(
        "ds_read_b128 %0, %2\n\t"
        "ds_read_b128 %1, %2 offset:2048\n\t"
        "s_waitcnt lgkmcnt(0)"
        : "=&v"(a[0]), "=&v"(a[1])
        : "v"(ad));
}
// packed weight bits of a lane: [NI][h]; sub-tile s at +2048, half h at +512
__device__ inline void lds_read_bits(v4i (&bw)[2][2], uint32_t ad) {
    asm volatile(
        "ds_read_b128 %0, %4\n\t"
        "ds_read_b128 %1, %4 offset:512\n\t"
        "ds_read_b128 %2, %4 offset:2048\n\t"
        "ds_read_b128 %3, %4 offset:2560\n\t"
        "s_waitcnt lgkmcnt(0)"
        : "=&v"(bw[0][0]), "=&v"(bw[0][1]), "=&v"(bw[1][0]), "=&v"(bw[1][1])
        : "v"(ad));
}

// The LDS reads of the next half-step's operands, started here and valid at lds_wait, which ties
// the registers so that nothing the compiler schedules in between can use them earlier.
__device__ inline void lds_issue(v4i (&a)[4], uint32_t ad) {
    asm volatile(
        "ds_read_b128 %0, %4\n\t"
        "ds_read_b128 %1, %4 offset:2048\n\t"
        "ds_read_b128 %2, %4 offset:4096\n\t"
        "ds_read_b128 %3, %4 offset:6144"
        : "=&v"(a[0]), "=&v"(a[1]), "=&v"(a[2]), "=&v"(a[3])
        : "v"(ad));
}
__device__ inline void lds_issue(v4i (&a)[2], uint32_t ad) {
    asm volatile(
        "ds_read_b128 %0, %2\n\t"
        "ds_read_b128 %1, %2 offset:2048"
        : "=&v"(a[0]), "=&v"(a[1])
        : "v"(ad));
}
__device__ inline void lds_wait(v4i (&a)[4]) {
    asm volatile("s_waitcnt lgkmcnt(0)" : "+v"(a[0]), "+v"(a[1]), "+v"(a[2]), "+v"(a[3]));
}
__device__ inline void lds_wait(v4i (&a)[2]) {
    asm volatile("s_waitcnt lgkmcnt(0)" : "+v"(a[0]), "+v"(a[1]));
}
// Row scale and row sum of four consecutive rows (epilogue), complete on exit.
__device__ inline void lds_read_rows(v4f& sc, v4i& rs, uint32_t ad_sc, uint32_t ad_rs) {
    asm volatile(
        "ds_read_b128 %0, %2\n\t"
        "ds_read_b128 %1, %3\n\t"
        "s_waitcnt lgkmcnt(0)"
        : "=&v"(sc), "=&v"(rs)
        : "v"(ad_sc), "v"(ad_rs));
}
// four times four consecutive rows, 8 rows apart
__device__ inline void lds_read_quads(v4i (&q)[4], uint32_t ad) {
    asm volatile(
        "ds_read_b128 %0, %4\n\t"
        "ds_read_b128 %1, %4 offset:32\n\t"
        "ds_read_b128 %2, %4 offset:64\n\t"
        "ds_read_b128 %3, %4 offset:96\n\t"
        "s_waitcnt lgkmcnt(0)"
        : "=&v"(q[0]), "=&v"(q[1]), "=&v"(q[2]), "=&v"(q[3])
        : "v"(ad));
}
__device__ inline float lds_read_f32(uint32_t ad) {
    float v;
    asm volatile("ds_read_b32 %0, %1\n\ts_waitcnt lgkmcnt(0)" : "=&v"(v) : "v"(ad));
    return v;
}
__device__ inline void lds_write_b32(uint32_t ad, uint32_t v) {
    asm volatile("ds_write_b32 %0, %1" : : "v"(ad), "v"(v) : "memory");
}

// NS = stages in the LDS ring (4 or 8: it must divide the 8 stages of a chunk).
// Persistent: gridDim.x workgroups (one per CU) walk the tiles t = blockIdx.x, + gridDim.x, ...
// GEN = false: the plain layer (one beta, Y = result): nothing of what follows costs anything.
// GEN = true adds beta per column group (Eq. 13) and the shift term of Eq. 6.
template <int BM, int BN, int WM, int WN, int NS, bool GEN>
__global__ __launch_bounds__(WM * WN * 64, 2) void gemm_prefill_kernel(GemmArgs a, int grid_m,
                                                                        int grid_n, int xbm) {
    constexpr int THREADS = WM * WN * kWave;
    constexpr int WTM = BM / WM, WTN = BN / WN;
    constexpr int MI = WTM / 32, NI = WTN / 32;
    constexpr int P = BM * 4 / THREADS;  // 16-byte DMA pieces per thread per stage
    constexpr int NWAVES = WM * WN;
    constexpr int NBW = (BN / 16) / NWAVES;  // packed-weight tiles (DMA pieces) per wave per chunk
    constexpr int STAGE_BYTES = BM * kStageK;
    static_assert(BM * 4 % THREADS == 0, "tile shape");
    static_assert((MI == 4 && NI == 2) || (MI == 2 && NI == 2), "wave tiles with LDS-read asm blocks");
    static_assert(NS == 4 || NS == 8, "ring size");
    static_assert((BN / 16) % NWAVES == 0 && (NS - 2) * P + NBW < 64, "tile shape");

    __shared__ __attribute__((aligned(1024))) uint8_t smA[NS * STAGE_BYTES];
    __shared__ __attribute__((aligned(1024))) uint8_t smB[(BN / 16) * 1024];
    __shared__ __attribute__((aligned(16))) float smScale[2][BM];  // gamma_m / 128, per tile parity
    __shared__ __attribute__((aligned(16))) float smBeta[2][GEN ? BN : 4];  // beta of each column's group
    __shared__ __attribute__((aligned(16))) float smEta[2][GEN ? BM : 4];   // Eq. 6 only: eta_m
    __shared__ __attribute__((aligned(16))) int smWsum[2][GEN ? BN : 4];    // Eq. 6 only: sum_k s[n,k]
    __shared__ __attribute__((aligned(16))) int smRowsum[2][BM];   // -sum_k q[m,k]

    const int w = threadIdx.x / kWave, l = threadIdx.x % kWave;
    const int wm = w / WN, wn = w % WN;
    const int j = l & 31, g2 = l >> 5;
    const int64_t TN = tiles_n(a.N);
    const int64_t M = a.M;
    const int64_t K = a.K, TK = tiles_k(K);
    const int nst = (int)((K + kStageK - 1) / kStageK);
    const int64_t kfull = K / kStageK;
    // chunks whose look-ahead stays inside K and that have a successor chunk
    const int64_t main_chunks = kfull >= NS + 7 ? (kfull - NS - 7) / 8 + 1 : 0;
    const int64_t TKp = a.tk_pitch ? a.tk_pitch : tiles_k(a.K);  // tiles per tile row in memory
    const int ntiles = grid_m * grid_n;

    // Tile order.  Workgroups are dealt round-robin to the 8 XCDs, each with its own L2; give
    // each XCD one contiguous range of the tile sequence, so that the tiles running together on
    // an XCD share operands in its L2.  The sequence walks bands of xbm rows of tiles, inside a
    // band the rows fastest: an XCD's range is then a block of xbm x (range / xbm) tiles and it
    // fetches xbm row blocks of codes (BM x K bytes each) and range / xbm column blocks of packed
    // weights (BN x K / 8 bytes each).  xbm = 1 unless the host asks otherwise (see launch_tile).
    auto tile_origin = [&](int t, int64_t& m0, int64_t& n0) {
        int logical = t;
        const int G = (int)gridDim.x;
        if ((ntiles & 7) == 0 && (G & 7) == 0) {
            const int q = ((t % G) >> 3) + (t / G) * (G >> 3);  // index inside the XCD's range
            logical = (t & 7) * (ntiles >> 3) + q;
            // the XCD's range may end before the last round does
            if (q >= (ntiles >> 3)) logical = -1;
        }
        int tm = logical / grid_n, tn = logical % grid_n;
        if (xbm > 1 && logical >= 0) {
            const int band = logical / (xbm * grid_n), rem = logical - band * xbm * grid_n;
            const int rows = min(xbm, grid_m - band * xbm);  // the last band may be lower
            tm = band * xbm + rem % rows;
            tn = rem / rows;
        }
        m0 = logical < 0 ? -1 : (int64_t)tm * BM;
        n0 = logical < 0 ? -1 : (int64_t)tn * BN;
    };

    // ---- DMA of one stage: thread -> P pieces; piece = (row, swizzled 16-byte segment) ----
    // Global address = uniform base (tile row 0, stage k) + a 32-bit per-lane offset.  Rows
    // past M re-read row M-1 (never stored).  clamp: stages that may reach past K re-read the
    // last 16 valid bytes of the row (nobody reads those buffer bytes).
    uint32_t goff[P];
    int gseg[P];
    const int8_t* gbase = a.codes;
    const uint32_t* bsrc[NBW];
    auto setup_dma = [&](int64_t m0, int64_t n0) {
#pragma unroll
        for (int q = 0; q < P; ++q) {
            const int slot = q * THREADS + threadIdx.x;
            int row = slot >> 2;
            gseg[q] = ((slot & 3) ^ ((row >> 2) & 3)) * 16;
            if (m0 + row > M - 1) row = (int)(M - 1 - m0);
            goff[q] = (uint32_t)row * (uint32_t)a.ldq + gseg[q];
        }
        gbase = a.codes + m0 * a.ldq;
        // packed weights: tile t of the block goes to smB + t KiB, lane for lane as it lies in
        // memory; wave w moves tiles w, w + NWAVES, ...  Columns past N read a valid tile.
#pragma unroll
        for (int q = 0; q < NBW; ++q) {
            int64_t tn = (n0 >> 4) + w + q * NWAVES;
            if (tn > TN - 1) tn = TN - 1;
            bsrc[q] = a.packed + tile_dword_offset(tn, 0, TKp) + l * 4;
        }
    };
    const uint32_t lds_wave = (uint32_t)(w * kWave * 16);
    auto issue = [&](int st, bool clamp) {
#pragma unroll
        for (int q = 0; q < P; ++q) {
            const int8_t* src = gbase + (int64_t)st * kStageK + goff[q];
            if (clamp) {
                const int64_t k = (int64_t)st * kStageK + gseg[q];
                if (k > K - 16) src -= k - (K - 16);
            }
            __builtin_amdgcn_global_load_lds(
                (const void*)src,
                (__attribute__((address_space(3))) void*)(smA + (st % NS) * STAGE_BYTES +
                                                          q * THREADS * 16 + lds_wave),
                16, 0, 0);
        }
    };
    auto issue_bits = [&](int64_t tk) {
#pragma unroll
        for (int q = 0; q < NBW; ++q)
            __builtin_amdgcn_global_load_lds(
                (const void*)(bsrc[q] + tk * 256),
                (__attribute__((address_space(3))) void*)(smB + (w + q * NWAVES) * 1024), 16, 0, 0);
    };
    // what a tile starts with: weight bits of chunk 0 and stages 0 .. NS-2 (clamped: K may be short)
    auto issue_tile_start = [&]() {
        issue_bits(0);
#pragma unroll
        for (int s = 0; s < NS - 1; ++s) issue(s, true);
    };

    // lane (j, g2) of sub-tile s, half h reads lane slot (2h+g2)*16 + j%16 of tile (..+j/16)
    const uint32_t b_lane = (uint32_t)(uintptr_t)smB + ((wn * WTN + j) >> 4) * 1024 +
                            (g2 * 16 + (j & 15)) * 16;
    // lane's operand address inside a stage: row (wm*WTM + j), segment (2h+g2) ^ swizzle
    const int sw = (j >> 2) & 3;
    const uint32_t a_lane[2] = {
        (uint32_t)(uintptr_t)smA + (wm * WTM + j) * kStageK + ((g2) ^ sw) * 16,
        (uint32_t)(uintptr_t)smA + (wm * WTM + j) * kStageK + ((2 + g2) ^ sw) * 16};
    auto a_addr = [&](int st, int h) { return a_lane[h] + (uint32_t)((st % NS) * STAGE_BYTES); };

    v16i acc[MI][NI];
    v4i bw[NI][2];  // packed bits of the current chunk
    // bit plane i of half h as {0,-128} bytes; the epilogue turns -128 sum_k q b into sum_k q (2b - 1)
    auto expand = [&](v4i (&b)[NI], int h, int i) {
#pragma unroll
        for (int s = 0; s < NI; ++s)
#pragma unroll
            for (int d = 0; d < 4; ++d) b[s][d] = (int)(((uint32_t)bw[s][h][d] << (7 - i)) & 0x80808080u);
    };
    v4i ax[MI], ay[MI], bx[NI], by[NI];
    // One half-step (32 k of a stage): acc += ac x b, MI * NI MFMAs, with the next half-step's
    // weight operand bn = plane i of half h expanded BETWEEN them (the compiler's scheduler is told
    // so with sched_group_barrier: one MFMA, then the two vector ALU operations of a dword, ...), so
    // that a wave expands under its own MFMAs instead of ahead of them; the operands at `ad` are
    // read into an meanwhile (valid on return).  Against an asm block of the MFMAs with the
    // expansion ahead of it: 117 against 129 us on 2048 x 4096 x 16384, 1-2 % on the longer K.
    auto half_step = [&](const v4i(&ac)[MI], const v4i(&b)[NI], v4i(&bn)[NI], int h, int i,
                          v4i(&an)[MI], uint32_t ad, auto between) {
        lds_issue(an, ad);
        // the bits pass through an (empty) asm placed after the reads, and the new operand through
        // one at the end: the expansion can neither be moved ahead of this half-step nor be left
        // for a later one before the scheduler sees the groups below
        asm volatile("" : "+v"(bw[0][h]), "+v"(bw[1][h]));
        __builtin_amdgcn_sched_barrier(0);
        constexpr int DW = NI * 4 / (MI * NI);  // dwords of the new operand per MFMA: 1 or 2
#pragma unroll
        for (int mi = 0; mi < MI; ++mi)
#pragma unroll
            for (int s = 0; s < NI; ++s) {
                acc[mi][s] = __builtin_amdgcn_mfma_i32_32x32x32_i8(ac[mi], b[s], acc[mi][s], 0, 0, 0);
                const int q = mi * NI + s;
#pragma unroll
                for (int e = 0; e < DW; ++e) {
                    const int idx = q * DW + e;  // 0 .. NI*4-1
                    bn[idx >> 2][idx & 3] = (int)(((uint32_t)bw[idx >> 2][h][idx & 3] << (7 - i)) & 0x80808080u);
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
        lds_wait(an);
    };

    // Stage st, bit plane i = st % 8.  In: ax/bx = operands of (st, h=0).  Out: ax/bx =
    // operands of (st+1, h=0).  DMA bookkeeping at the mid-stage point, while the look-ahead
    // stage st+NS-1 exists (`ahead`): the groups younger than stage st+1 are stages st+2 ..
    // st+NS-2 ((NS-3)*P operations), plus the NBW weight tiles while they are among them: the
    // tiles are issued at i == 2 ahead of stage st+NS-1's group, so they are younger than stage
    // st+1 at i = 3 .. NS-1.  At i == 7 they are never allowed to be outstanding: smB is read
    // right after that barrier.  Near the end of K nothing more is issued and the wait is for
    // everything outstanding (all of it is needed within the next NS-2 stages).
    auto stage = [&](int st, int i, bool clamp, bool half, bool ahead, bool bits_in_flight) {
        half_step(ax, bx, by, 1, i, ay, a_addr(st, 1), []() {});
        if (!ahead) wait_vmcnt<0>();
        else if (bits_in_flight && i >= 3 && i <= NS - 1 && i <= 6) wait_vmcnt<(NS - 3) * P + NBW>();
        else wait_vmcnt<(NS - 3) * P>();
        block_barrier();
        if (i == 7) lds_read_bits(bw, b_lane);  // bits of the next chunk (landed long ago)
        auto dma = [&]() {
            if (i == 2 && (st >> 3) + 1 < TK) issue_bits((st >> 3) + 1);
            if (ahead) issue(st + NS - 1, clamp);
        };
        if (!half) half_step(ay, by, bx, 0, (i + 1) & 7, ax, a_addr(st + 1, 0), dma);
        else dma();
    };

    int t = (int)blockIdx.x, parity = 0;
    int64_t m0, n0;
    tile_origin(t, m0, n0);
    if (m0 < 0) return;  // uniform for the whole workgroup
    setup_dma(m0, n0);
    issue_tile_start();

    while (true) {
        if constexpr (GEN) {
            // Per-row gamma and row sum of the codes, per-column beta (Eq. 11, Eq. 13), for the
            // epilogue.  Thread i serves row i and column i (BM, BN <= THREADS); every load is
            // issued before the first value is needed, so the tile pays one memory latency here.
            {
                static_assert(BM <= THREADS && BN <= THREADS, "one row and one column per thread");
                const int i = threadIdx.x;
                const int64_t m = m0 + i < M ? m0 + i : M - 1;
                int64_t n = n0 + i;
                if (n > a.N - 1) n = a.N - 1;
                // branch-free (a branch here makes the compiler drain the loads issued so far):
                // with one beta for the matrix the quotient is 0 by itself; the Eq. 6 operands are
                // read from a valid stand-in address when they are not in use
                const uint32_t bg = (uint32_t)n / (uint32_t)a.beta_rows;
                const float gm = a.gamma[a.per_tensor ? 0 : m * a.gstride];
                const int rs = a.rowsum[m * a.gstride];
                const float b = a.beta[bg * a.beta_stride];
                const float e = *(a.eta ? a.eta + (a.per_tensor ? 0 : m * a.gstride) : a.gamma);
                const int ws = *(a.eta ? a.wsum + n : a.rowsum);
                if (i < BM) {
                    // gamma / 128 is exact, so beta * (gamma / 128) has the bits of (beta * gamma) / 128
                    lds_write_b32((uint32_t)(uintptr_t)&smScale[parity][i], __float_as_uint(gm * 0.0078125f));
                    lds_write_b32((uint32_t)(uintptr_t)&smRowsum[parity][i], (uint32_t)-rs);
                    lds_write_b32((uint32_t)(uintptr_t)&smEta[parity][i], __float_as_uint(e));
                }
                if (i < BN) {
                    lds_write_b32((uint32_t)(uintptr_t)&smBeta[parity][i], __float_as_uint(b));
                    lds_write_b32((uint32_t)(uintptr_t)&smWsum[parity][i], (uint32_t)ws);
                }
            }
        } else {
            // per-row dequantisation scale (Eq. 11) and row sum of the codes, for the epilogue
            const float beta = *a.beta;
            for (int r = threadIdx.x; r < BM; r += THREADS) {
                const int64_t m = m0 + r;
                float sc = 0.f;
                int rs = 0;
                if (m < M) {
                    sc = (beta * (a.per_tensor ? a.gamma[0] : a.gamma[m])) / 128.0f;
                    rs = a.rowsum[m];
                }
                lds_write_b32((uint32_t)(uintptr_t)&smScale[parity][r], __float_as_uint(sc));
                lds_write_b32((uint32_t)(uintptr_t)&smRowsum[parity][r], (uint32_t)-rs);
            }
        }
#pragma unroll
        for (int mi = 0; mi < MI; ++mi)
#pragma unroll
            for (int s = 0; s < NI; ++s)
#pragma unroll
                for (int r = 0; r < 16; ++r) acc[mi][s][r] = 0;

        // stage 0 and the bits of chunk 0 have landed; operands of half-step 0
        wait_vmcnt<(NS - 2) * P>();  // younger than stage 0: stages 1 .. NS-2
        block_barrier();
        lds_read_bits(bw, b_lane);
        lds_read_a(ax, a_addr(0, 0));
        expand(bx, 0, 0);

        // Main loop: no clamps, i folds to a constant.  Then the remaining stages.
        for (int64_t tk = 0; tk < main_chunks; ++tk) {
            static_for<0, 8>([&](auto ic) {
                constexpr int i = decltype(ic)::value;
                stage((int)tk * 8 + i, i, false, false, true, true);
            });
        }
        for (int st = (int)main_chunks * 8; st < nst; ++st)
            stage(st, st & 7, true, (int64_t)st * kStageK + 32 >= K, st + NS - 1 < nst,
                  (st >> 3) + 1 < TK);

        // Every wave is done with the LDS ring: start the next tile's stream, then store.
        block_barrier();
        const int t_next = t + (int)gridDim.x;
        int64_t m0n = -1, n0n = -1;
        if (t_next < ntiles) tile_origin(t_next, m0n, n0n);
        if (m0n >= 0) {
            setup_dma(m0n, n0n);
            issue_tile_start();
        }

        // ---- epilogue (Eq. 11): lane (j, g2) holds column n, rows 8*(r/4) + 4*g2 + r%4 ----
        //   sum_k q s = 2 sum_k q b - sum_k q, the accumulators holding -128 sum_k q b ;
        //   y = that * (beta_n * gamma_m / 128)
        float bcol[NI];
#pragma unroll
        for (int s = 0; s < NI; ++s)
            bcol[s] = GEN ? lds_read_f32((uint32_t)(uintptr_t)&smBeta[parity][wn * WTN + 32 * s + j])
                          : 1.f;
        const uint32_t sc_base = (uint32_t)(uintptr_t)&smScale[parity][wm * WTM + 4 * g2];
        const uint32_t rs_base = (uint32_t)(uintptr_t)&smRowsum[parity][wm * WTM + 4 * g2];
        const bool special = a.out_acc || (GEN && a.eta != nullptr);
        float wcol[NI];  // Eq. 6 only
#pragma unroll
        for (int s = 0; s < NI; ++s)
            wcol[s] = (GEN && a.eta) ? (float)__float_as_int(lds_read_f32(
                                  (uint32_t)(uintptr_t)&smWsum[parity][wn * WTN + 32 * s + j]))
                            : 0.f;
        const int wrow = __builtin_amdgcn_readfirstlane(wm * WTM), wcolumn = __builtin_amdgcn_readfirstlane(wn * WTN);
        auto store_plain = [&](auto with_eta) {
            constexpr bool ETA = decltype(with_eta)::value;
            v4f sc4;
            v4i rs4;
            float e = 0.f;
            store_tile<MI, NI, (BM < 256)>(
                a.Y + (m0 + wrow) * a.ldy + n0 + wcolumn, a.ldy, M - m0 - wrow, a.N - n0 - wcolumn, j, g2,
                [&](int mi, int rq) {
                    lds_read_rows(sc4, rs4, sc_base + (32 * mi + 8 * rq) * 4, rs_base + (32 * mi + 8 * rq) * 4);
                },
                [&](int mi, int r, int s) {
                    const int pm = rs4[r & 3] - (acc[mi][s][r] >> 6);  // exact: a multiple of 128
                    float y = GEN ? (float)pm * (bcol[s] * sc4[r & 3]) : (float)pm * sc4[r & 3];
                    if constexpr (ETA) {  // Eq. 6: + (beta * eta_m) * sum_k s[n,k]
                        if (s == 0)
                            e = lds_read_f32((uint32_t)(uintptr_t)&smEta[parity][wm * WTM + 32 * mi + 8 * (r >> 2) +
                                                                                 4 * g2 + (r & 3)]);
                        y = y + (bcol[s] * e) * wcol[s];
                    }
                    return y;
                });
        };
        if (!a.out_acc &&  // uniform
            (BM < 256 || (m0 + BM <= M && n0 + BN <= a.N && a.ldy < (1 << 24)))) {
            if (GEN && a.eta) store_plain(std::integral_constant<bool, GEN>{});
            else store_plain(std::false_type{});
        } else {
            // a 256-row tile at an edge, or int32 output.  Register allocation here is at the limit of 256 and
            // sensitive to the form of these loops: hoisting the uniform branches into a second copy of the
            // loops, or naming the row index as a 32-bit temporary, makes the compiler precompute the
            // store addresses and spill over a hundred registers.
#pragma unroll
            for (int mi = 0; mi < MI; ++mi)
#pragma unroll
                for (int rq = 0; rq < 4; ++rq) {
                    v4f sc4;
                    v4i rs4;
                    lds_read_rows(sc4, rs4, sc_base + (32 * mi + 8 * rq) * 4, rs_base + (32 * mi + 8 * rq) * 4);
#pragma unroll
                    for (int rr = 0; rr < 4; ++rr) {
                        const int r = rq * 4 + rr;
                        const int64_t m = m0 + wm * WTM + 32 * mi + 8 * rq + 4 * g2 + rr;
                        if (m >= M) continue;
#pragma unroll
                        for (int s = 0; s < NI; ++s) {
                            const int64_t n = n0 + wn * WTN + 32 * s + j;
                            if (n >= a.N) continue;
                            const int pm = rs4[rr] - (acc[mi][s][r] >> 6);
                            float y = GEN ? (float)pm * (bcol[s] * sc4[rr]) : (float)pm * sc4[rr];
                            if (special) {  // uniform
                                if (a.out_acc) {
                                    reinterpret_cast<int*>(a.Y)[m * a.ldy + n] = pm;
                                    continue;
                                }
                                if (GEN && a.eta) {
                                    const float e = lds_read_f32(
                                        (uint32_t)(uintptr_t)&smEta[parity][wm * WTM + 32 * mi + 8 * rq + 4 * g2 + rr]);
                                    y = y + (bcol[s] * e) * wcol[s];
                                }
                            }
                            __builtin_nontemporal_store(y, &a.Y[m * a.ldy + n]);
                        }
                    }
                }
        }
        if (m0n < 0) break;
        t = t_next;
        m0 = m0n;
        n0 = n0n;
        parity ^= 1;
    }
}

// ---- grouped layers (Eq. 13-15): all K-groups of a 128 x 256 tile in one workgroup --------------
// Y[m,n] = sum_g (beta_g[n] * (gamma_g[m] / 128)) * (2 sum_{k in g} q b - sum_{k in g} q)  (+ Eq. 6's
// (beta_g eta_g) wsum_g): a work item is (tile, K-group), the groups of a tile following each other;
// each item's int32 sums are dequantised into an fp32 register copy of the tile in the order 0, 1,
// ..., which is stored once, after the last group.
//
// Bound by the matrix pipe and, at short groups, by whatever happens between items: K = 7168 in 8
// groups is 14 stages an item.  So the stream of operands does not stop there.  Codes, packed bits
// and the items' scales have cursors of their own that run ahead of the multiplication (7 stages, two
// 512-chunks, two items) straight across the ends of groups and tiles; every mid-stage point issues
// the same operations, so the waits are the same constants everywhere.  The bits have two LDS buffers
// (a chunk's bits are requested when the chunk before the last starts), the scales four.
// A group's K may end inside a stage or a chunk: what follows meets zero bits (tiles are padded with
// them), and the at most 32 bytes behind the codes of the last row lie in the workspace.  A cursor
// at the end of the workgroup's work re-reads its last piece into a buffer nobody reads.
//
// The waits.  Mid-point of stage s (between its half-steps), per wave and in this order: wait,
// barrier, [last stage of a chunk: read the next chunk's bits], [first stage of an item: request the scales of
// the item after the next], [first stage of a chunk: request the bits of the chunk after the next],
// request codes of stage s + 7.  Needed there: codes of stage s + 1, with the codes of stages s + 2
// .. s + 6 (five operations) younger; the bits read there; and behind the last stage of an item the scales of
// the next one, whose row sums its products start from.  Younger than these are the codes of at least 2 nst - 1
// stages and the bits of two chunks, five or more when an item has two stages or more (nst).  One wait for
// all but the last five covers all three; items of one stage wait for everything.
//
// The fold is vector instructions that all waves issue at once while the matrix pipe stands still, two waves a SIMD
// and four cycles each, beside 112 MFMAs of 32 cycles in an item of 14 stages.  So what can be is in the MFMAs: a set
// bit is a byte of 2 and an item's first half-step adds to the negated row sums instead of to zeros, and the
// accumulators are sum_k q s as they are; left are conversion, product of the scales, product and addition, 320
// instructions of 450 a wave.  us of the layer, before / after: 1000 x 7168 x 28672 in 8 x 8 groups 238.6 / 224.5,
// 4096 x 7168 x 7168 in 2 x 8 265 / 249, 3000 x 2048 x 8192 in 8 x 8 106.7 / 92.0, 4096 x 1024 x 4096 in 1 x 8 71.8 /
// 58.2.  (The scales' products from a 32 x 32 x 2 f32 MFMA, 64 vector instructions fewer, are 1 to 6 % slower; bytes
// of {0, -128} are no faster; with the ring drained and filled for every item and the scales loaded behind it the
// first of these took 445 us.)
template <bool ETA>
__global__ __launch_bounds__(512, 2) void gemm_group_kernel(GemmArgs a, int grid_m, int grid_n) {
    constexpr int BM = 128, BN = 256, WN = 4, NS = 8, THREADS = 512, NWAVES = 8;
    constexpr int WTM = 64, WTN = 64, MI = 2, NI = 2;
    constexpr int STAGE_BYTES = BM * kStageK;  // 8 KiB: one 16-byte DMA piece per thread
    constexpr int BITS_BYTES = (BN / 16) * 1024;
    constexpr int NBW = BN / 16 / NWAVES;
    __shared__ __attribute__((aligned(1024))) uint8_t smA[NS * STAGE_BYTES];
    __shared__ __attribute__((aligned(1024))) uint8_t smB[2 * BITS_BYTES];
    // per item, in a ring: gamma [128], row sums [128], beta [256]; Eq. 6: eta [128], unused [128], wsum [256]
    __shared__ __attribute__((aligned(1024))) uint32_t smS[4][THREADS];
    __shared__ __attribute__((aligned(1024))) uint32_t smE[4][ETA ? THREADS : 4];

    const int w = __builtin_amdgcn_readfirstlane((int)threadIdx.x / kWave), l = threadIdx.x % kWave;
    const int wm = w / WN, wn = w % WN;
    const int j = l & 31, g2 = l >> 5;
    const int M = (int)a.M, N = (int)a.N;
    const int TN = (int)tiles_n(a.N);
    const int64_t TK = tiles_k(a.K);
    const int nst = (int)((a.K + kStageK - 1) / kStageK), nch = (int)TK;
    const int ntiles = grid_m * grid_n, G = (int)gridDim.x, ngroups = a.kgroups;

    // a workgroup's tiles t = blockIdx.x, + G, ...: one contiguous range of the row-major sequence of
    // tiles per XCD (as in gemm_prefill_kernel); false: no such tile
    auto tile_origin = [&](int t, int& m0, int& n0) {
        if (t >= ntiles) return false;
        int logical = t;
        if ((ntiles & 7) == 0 && (G & 7) == 0) {
            const int q = ((t % G) >> 3) + (t / G) * (G >> 3);
            if (q >= (ntiles >> 3)) return false;
            logical = (t & 7) * (ntiles >> 3) + q;
        }
        m0 = logical / grid_n * BM;
        n0 = logical % grid_n * BN;
        return true;
    };
    // a position in the workgroup's sequence of items
    struct Item {
        int t, grp, m0, n0;
    };
    // false (and unchanged) at the last item
    auto next_item = [&](Item& it) {
        if (it.grp + 1 < ngroups) {
            ++it.grp;
            return true;
        }
        int m0, n0;
        if (!tile_origin(it.t + G, m0, n0)) return false;
        it = Item{it.t + G, 0, m0, n0};
        return true;
    };
    Item cur{(int)blockIdx.x, 0, 0, 0};
    if (!tile_origin(cur.t, cur.m0, cur.n0)) return;  // uniform for the whole workgroup
    Item ca = cur, cb = cur, cs = cur;                // codes, bits, scales

    // ---- codes: thread -> one piece (row, swizzled segment) of a stage ------------------------
    const int arow = (int)threadIdx.x >> 2;
    const int aseg = (((int)threadIdx.x & 3) ^ ((arow >> 2) & 3)) * 16;
    uint32_t goff = 0;
    const int8_t* abase = nullptr;
    int ast = 0, aslot = 0;
    auto set_codes = [&]() {
        const int last = M - 1 - ca.m0;
        goff = (uint32_t)(arow < last ? arow : last) * (uint32_t)a.ldq + aseg;
        abase = a.codes + (int64_t)ca.m0 * a.ldq + (int64_t)ca.grp * a.K;
    };
    auto issue_codes = [&]() {
        __builtin_amdgcn_global_load_lds(
            (const void*)(abase + (int64_t)ast * kStageK + goff),
            (__attribute__((address_space(3))) void*)(smA + aslot * STAGE_BYTES + w * (kWave * 16)), 16, 0, 0);
        aslot = (aslot + 1) & (NS - 1);
        if (ast + 1 < nst) ++ast;
        else if (next_item(ca)) {
            ast = 0;
            set_codes();
        }
    };
    // ---- packed bits: wave w moves tiles w and w + 8 of the block; columns past N read a valid tile
    int bch = 0, bbuf = 0;
    auto issue_bits = [&]() {
#pragma unroll
        for (int q = 0; q < NBW; ++q) {
            int tn = (cb.n0 >> 4) + w + q * NWAVES;
            if (tn > TN - 1) tn = TN - 1;
            __builtin_amdgcn_global_load_lds(
                (const void*)(a.packed + (int64_t)cb.grp * a.group_packed +
                              tile_dword_offset(tn, bch, TK) + l * 4),
                (__attribute__((address_space(3))) void*)(smB + bbuf * BITS_BYTES + (w + q * NWAVES) * 1024),
                16, 0, 0);
        }
        bbuf ^= 1;
        if (bch + 1 < nch) ++bch;
        else if (next_item(cb)) bch = 0;
    };
    // ---- scales of an item: a dword per thread (two with Eq. 6) -----------------------------------
    int sbuf = 0;
    auto issue_scales = [&]() {
        const int i = (int)threadIdx.x;
        const int r = cs.m0 + (i & (BM - 1)), c = cs.n0 + (i & (BN - 1));
        const int64_t m = r < M ? r : M - 1;
        const int n = c < N ? c : N - 1;
        const int64_t gi = (a.per_tensor ? 0 : m * a.gstride) + cs.grp;
        const void* src;
        if (w < 2) src = a.gamma + gi;  // uniform branches
        else if (w < 4) src = a.rowsum + m * a.gstride + cs.grp;
        else src = a.beta + (int64_t)((uint32_t)n / (uint32_t)a.beta_rows) * a.beta_stride + cs.grp;
        __builtin_amdgcn_global_load_lds(
            src, (__attribute__((address_space(3))) void*)(&smS[sbuf][w * kWave]), 4, 0, 0);
        if constexpr (ETA) {
            if (w < 4) src = a.eta + gi;
            else src = a.wsum + (int64_t)cs.grp * a.N + n;
            __builtin_amdgcn_global_load_lds(
                src, (__attribute__((address_space(3))) void*)(&smE[sbuf][w * kWave]), 4, 0, 0);
        }
        sbuf = (sbuf + 1) & 3;
        next_item(cs);
    };

    // operand addresses, as in gemm_prefill_kernel
    const uint32_t b_lane = (uint32_t)(uintptr_t)smB + ((wn * WTN + j) >> 4) * 1024 +
                            (g2 * 16 + (j & 15)) * 16;
    const int sw = (j >> 2) & 3;
    const uint32_t a_lane[2] = {
        (uint32_t)(uintptr_t)smA + (wm * WTM + j) * kStageK + ((g2) ^ sw) * 16,
        (uint32_t)(uintptr_t)smA + (wm * WTM + j) * kStageK + ((2 + g2) ^ sw) * 16};

    v16i acc[MI][NI];
    v4i bw[NI][2];
    v4i ax[MI], ay[MI], bx[NI], by[NI];
    // the tile's sum over the groups so far: from -0, which leaves the first term as it is (0 + -0 is 0)
    float side[MI][NI][16];
    auto clear_side = [&]() {
#pragma unroll
        for (int mi = 0; mi < MI; ++mi)
#pragma unroll
            for (int s = 0; s < NI; ++s)
#pragma unroll
                for (int r = 0; r < 16; ++r) side[mi][s][r] = -0.f;
    };
    clear_side();
    // bit plane i as {0, 2} bytes
    auto plane = [](int bits, int i) {
        return (int)(__builtin_amdgcn_alignbit((uint32_t)bits, (uint32_t)bits, (uint32_t)(i + 31) & 31) & 0x02020202u);
    };
    // acc += ac x b; meanwhile an = operands at `ad`, bn = plane i of half h (see gemm_prefill_kernel);
    // between() goes behind the first two MFMAs: the cursors' scalar work would idle the matrix pipe of
    // all waves at once if it stood right behind the barrier
    // `first`: the item's first, on top of the rows' -sum_k q
    v16i base[MI];
    auto half_step = [&](auto first, const v4i(&ac)[MI], const v4i(&b)[NI], v4i(&bn)[NI], int h, int i, v4i(&an)[MI],
                         uint32_t ad, auto between) {
        lds_issue(an, ad);
        asm volatile("" : "+v"(bw[0][h]), "+v"(bw[1][h]));
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int mi = 0; mi < MI; ++mi)
#pragma unroll
            for (int s = 0; s < NI; ++s) {
                acc[mi][s] = __builtin_amdgcn_mfma_i32_32x32x32_i8(ac[mi], b[s], first ? base[mi] : acc[mi][s], 0, 0, 0);
                const int q = mi * NI + s;
#pragma unroll
                for (int e = 0; e < 2; ++e) {
                    const int idx = q * 2 + e;
                    bn[idx >> 2][idx & 3] = plane(bw[idx >> 2][h][idx & 3], i);
                }
                __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
                __builtin_amdgcn_sched_group_barrier(0x002, 4, 0);
                if (q == 1) {
                    __builtin_amdgcn_sched_barrier(0);
                    between();
                    __builtin_amdgcn_sched_barrier(0);
                }
            }
        asm volatile("" : "+v"(bn[0]), "+v"(bn[1]));
        __builtin_amdgcn_sched_barrier(0);
        lds_wait(an);
    };

    const bool one_stage = nst == 1;
    int slot = 0, rbuf = 0;  // the stage's ring slot; the buffer the current chunk's bits came from
    auto stage = [&](auto ic, bool last, bool first_chunk) {
        constexpr int i = decltype(ic)::value;
        const uint32_t second = a_lane[1] + (uint32_t)(slot * STAGE_BYTES);
        if (i == 0 && first_chunk) half_step(std::true_type{}, ax, bx, by, 1, i, ay, second, []() {});
        else half_step(std::false_type{}, ax, bx, by, 1, i, ay, second, []() {});
        if (one_stage) wait_vmcnt<0>();
        else wait_vmcnt<5>();
        block_barrier();
        if (last) {
            rbuf ^= 1;
            lds_read_bits(bw, b_lane + (uint32_t)(rbuf * BITS_BYTES));
        }
        slot = (slot + 1) & (NS - 1);
        half_step(std::false_type{}, ay, by, bx, 0, last ? 0 : i + 1, ax, a_lane[0] + (uint32_t)(slot * STAGE_BYTES), [&]() {
            if constexpr (i == 0) {
                if (first_chunk) issue_scales();
                issue_bits();
            }
            issue_codes();
        });
    };
    // the row sums of an item, negated, from its scales' buffer
    auto load_base = [&](int buf) {
        const uint32_t ad = (uint32_t)(uintptr_t)&smS[buf][BM + wm * WTM + 4 * g2];
#pragma unroll
        for (int mi = 0; mi < MI; ++mi) {
            v4i q[4];
            lds_read_quads(q, ad + 128 * mi);
#pragma unroll
            for (int r = 0; r < 16; ++r) base[mi][r] = -q[r >> 2][r & 3];
        }
    };

    set_codes();
    issue_scales();
    issue_scales();
    issue_bits();
    issue_bits();
#pragma unroll
    for (int s = 0; s < NS - 1; ++s) issue_codes();
    wait_vmcnt<NS - 2>();  // younger than stage 0: stages 1 .. 6
    block_barrier();
    lds_read_bits(bw, b_lane);
    lds_read_a(ax, a_lane[0]);
#pragma unroll
    for (int s = 0; s < NI; ++s)
#pragma unroll
        for (int d = 0; d < 4; ++d) bx[s][d] = plane(bw[s][0][d], 0);
    load_base(0);

    int fbuf = 0;  // the scales of the item being folded
    while (true) {
        for (int c = 0; c < nch; ++c) {
            const int len = nst - 8 * c;  // stages of this chunk: min(len, 8)
            static_for<0, 8>([&](auto ic) {
                constexpr int i = decltype(ic)::value;
                if (i < len) stage(ic, i == 7 || i + 1 == len, c == 0);
            });
        }
        // ---- fold: lane (j, g2) holds column n, rows 8 (r / 4) + 4 g2 + r % 4 of each sub-tile ----
        float bcol[NI], wcol[NI];
#pragma unroll
        for (int s = 0; s < NI; ++s) {
            const int col = wn * WTN + 32 * s + j;
            bcol[s] = lds_read_f32((uint32_t)(uintptr_t)&smS[fbuf][2 * BM + col]);
            wcol[s] = ETA ? (float)__float_as_int(lds_read_f32((uint32_t)(uintptr_t)&smE[fbuf][2 * BM + col]))
                            : 0.f;
        }
        const uint32_t row_base = (uint32_t)(uintptr_t)&smS[fbuf][wm * WTM + 4 * g2];
        const uint32_t eta_base = (uint32_t)(uintptr_t)&smE[fbuf][wm * WTM + 4 * g2];
#pragma unroll
        for (int mi = 0; mi < MI; ++mi) {
            v4i q[4];
            lds_read_quads(q, row_base + 128 * mi);
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                const float sc = __int_as_float(q[r >> 2][r & 3]) * 0.0078125f;  // gamma / 128, exact
                const float e = ETA ? lds_read_f32(eta_base + (32 * mi + 8 * (r >> 2) + (r & 3)) * 4) : 0.f;
#pragma unroll
                for (int s = 0; s < NI; ++s) {
                    float y = (float)acc[mi][s][r] * (bcol[s] * sc);
                    if constexpr (ETA) y = y + (bcol[s] * e) * wcol[s];
                    side[mi][s][r] = y + side[mi][s][r];
                }
            }
        }
        if (cur.grp + 1 == ngroups) {
            const int row = cur.m0 + wm * WTM, col = cur.n0 + wn * WTN;
            store_tile<MI, NI, true>(a.Y + (int64_t)row * N + col, N, M - row, N - col, j, g2, [](int, int) {},
                               [&](int mi, int r, int s) { return side[mi][s][r]; });
            clear_side();
        }
        if (!next_item(cur)) break;
        fbuf = (fbuf + 1) & 3;
        load_base(fbuf);
    }
    wait_vmcnt<0>();
}

template <int BM, int BN, int WM, int WN, int NS>
static void launch_tile(const GemmArgs& a, hipStream_t s) {
    const bool plain = a.beta_rows >= a.N && a.gstride == 1 && !a.eta;
    const int grid_m = (int)((a.M + BM - 1) / BM), grid_n = (int)((a.N + BN - 1) / BN);
    const int ntiles = grid_m * grid_n;
    int grid = num_cus();  // one workgroup per CU
    if (tuning().prefill_grid > 0) grid = tuning().prefill_grid;
    if (grid > ntiles) grid = ntiles;
    // Rows of tiles in an XCD's block.  One row (the XCD's tiles share their codes and stream all
    // the packed weights) is the fastest on every shape measured, although two or four rows fetch
    // fewer bytes: 2048 x 4096 x 16384 takes 115.2 us with 1 (84 MB fetched per launch), 117.5 us
    // with 2 (55 MB), 124.1 us with 4 (medians of 12 alternating runs); the kernel is not bound by
    // HBM.  prefill_xbm overrides.
    int xbm = 1;
    if ((ntiles & 7) == 0 && (grid & 7) == 0 && tuning().prefill_xbm > 0)
        xbm = tuning().prefill_xbm < grid_m ? tuning().prefill_xbm : grid_m;
    if (plain)
        gemm_prefill_kernel<BM, BN, WM, WN, NS, false>
            <<<(unsigned)grid, WM * WN * kWave, 0, s>>>(a, grid_m, grid_n, xbm);
    else
        gemm_prefill_kernel<BM, BN, WM, WN, NS, true>
            <<<(unsigned)grid, WM * WN * kWave, 0, s>>>(a, grid_m, grid_n, xbm);
}

// Kernel and K-slices for M > 64: the cheapest of all by these costs in us, fitted to medians of graph
// replays (n stages of 64 k, c 512-chunks per K-group of the workgroup):
//   a round of 128 x 256 tiles    8 + 0.35 n     (n = 32: 19, 64: 30, 112: 45)
//   a round of 256 x 256 tiles   14 + 0.62 n     (n = 32: 33, 64: 51 to 58, 112: 82, 256: 158)
//   a round of 128 x 128 tiles    5 + 3.0 c      (c = 1: 8, 2: 11, 4: 17, 7: 26, 16: 53)
//   a round of 64 x 128 tiles   4.5 + 3.1 c      (c = 1: 8, 2: 11, 4: 17, 7: 26, 14: 46)
//   the last two in three rounds and more 5 % more (the large tiles read the operands less often), and from 20 to 28
//   rows of tiles up to 0.8 c more: items run down a column of tiles, so that an XCD's 32 workgroups then hold hardly
//   more than one column and share no codes (in all, c costs 3.0 up to 20 rows, 3.3 at 24, 3.8 to 4.0 from 28 on)
//   slices of K                   4 + the int32 sums written and read at 5 TB/s
// The large tiles do the most work per byte and expanded bit; where they leave CUs idle the small
// ones win; the layer, us, M x K x N: 333 x 2048 x 2048 12.8 (64 x 128) against 19.4 (128 x 256), 700 x 4096 x 16384
// 60.5 (128 x 128) against 64.0 (128 x 256 and 256 x 256), 700 x 28672 x 7168 161.5 (64 x 128) against 186.1; the
// product, 2176 x 16384 x 2586 96 (128 x 256) against 113 (64 x 128).  Over 185 shapes of 440 to 5000 tokens, K and N of
// 1024 to 28672, the tile is 0.3 % slower than the best of the four on average, 11 % at most (1320 x 20288 x 882 39.9,
// 36.0 as 128 x 128); with 1.2 c more from 40 MB of codes on in place of what the rows cost it was 1.1 and 32 %.
struct TilePlan {
    int tile;     // 1: 128 x 256, 2: 256 x 256 (this file); 3: 128 x 128, 4: 64 x 128 (gemm_mid.hip)
    int64_t per;  // 512-chunks of K per slice (3 and 4)
    double us;
};
static double large_round_us(int tile, int64_t nst) { return tile == 1 ? 8.0 + 0.35 * nst : 14.0 + 0.62 * nst; }
static TilePlan tile_plan(int64_t M, int64_t N, int64_t K, size_t ws_bytes) {
    const int64_t cus = num_cus(), TK = tiles_k(K), nst = (K + kStageK - 1) / kStageK;
    const int force = tuning().prefill_tile;
    const int64_t force_n = tuning().prefill_split > 0 ? tuning().prefill_split : 0;
    // a forced tile stays that tile, unsliced, where its slices have no room; forced slices are
    // as many as the chunks of K give in equal parts
    TilePlan best{force >= 1 && force <= 4 ? force : 2, TK, 1e30};
    auto offer = [&](int tile, int64_t per, double us) {
        if (us < best.us) best = TilePlan{tile, per, us};
    };
    for (int tile = 1; tile <= 4; ++tile) {
        if (force && tile != force) continue;
        const int64_t bm = tile == 4 ? 64 : tile == 2 ? 256 : 128, bn = tile <= 2 ? 256 : 128;
        const int64_t tiles = ((M + bm - 1) / bm) * ((N + bn - 1) / bn);
        if (tile <= 2) {
            const int64_t rounds = (tiles + cus - 1) / cus;
            offer(tile, TK, (double)rounds * large_round_us(tile, nst));
            continue;
        }
        const int kg = tile == 3 ? 2 : 4;
        for (int64_t want = force_n ? force_n : 1; want <= (force_n ? force_n : 8); ++want) {
            const int64_t per = (TK + want - 1) / want, n = (TK + per - 1) / per;
            const double bytes = (double)n * (double)M * (double)N * 4.0;
            if (n > 1 && ((n != want && !force_n) || bytes > (double)ws_bytes)) continue;
            const int64_t rounds = (tiles * n + cus - 1) / cus;
            const double c = (double)((per + kg - 1) / kg);
            const double more = 0.1 * (double)((M + bm - 1) / bm - 20);
            const double chunk = (tile == 3 ? 3.0 : 3.1) + (more < 0.0 ? 0.0 : more < 0.8 ? more : 0.8);
            offer(tile, per, (double)rounds * ((tile == 3 ? 5.0 : 4.5) + chunk * c) * (rounds > 2 ? 1.05 : 1.0) +
                                 (n > 1 ? 4.0 + bytes * 2.0 / 5e6 : 0.0));
        }
    }
    return best;
}

// The last round of large tiles may be nearly empty (4096 x 7168 x 21504: 1344 tiles are 5.25 rounds of 256
// CUs, run as 6).  Then the columns that fill the rounds before it keep the large tiles, and the rest
// is a launch of its own with whatever costs least there, 3 us between the two.  us of the layer, one launch /
// two: 4096 x 7168 x 21504 553 / 528 (a quarter-filled round runs at a higher clock, or it would be more),
// 300 x 4096 x 24000 57.9 / 52.3, 2048 x 3072 x 12288 88.6 / 85.7, 4096 x 2048 x 6144 70.7 / 69.6.  Where one
// launch is of large tiles too, two have to cost 4 % less: of 23 shapes nearer the line, of 1500 drawn, 17 are faster in
// one (the product, 4008 x 7168 x 3072 78 to 85 / 87 to 89, 1218 x 960 x 17006 45.5 / 57.4, 4086 x 19328 x 2959 189 /
// 212; but 4806 x 512 x 28672 136 / 126).
struct PrefillPlan {
    TilePlan first, rest;
    int64_t cut;  // columns of the first launch, a multiple of 256; 0: one launch
};
// (one_beta: columns in groups with a beta of their own are not cut)
static PrefillPlan prefill_plan(int64_t M, int64_t N, int64_t K, size_t ws_bytes, bool one_beta) {
    PrefillPlan best{tile_plan(M, N, K, ws_bytes), {}, 0};
    if (!one_beta || tuning().prefill_tile || tuning().prefill_split || tuning().prefill_grid) return best;
    const int64_t cus = num_cus(), nst = (K + kStageK - 1) / kStageK;
    double best_us = (best.first.tile <= 2 ? 0.96 : 1.0) * best.first.us;
    for (int tile = 1; tile <= 2; ++tile) {
        const int64_t bm = tile == 1 ? 128 : 256;
        const int64_t grid_m = (M + bm - 1) / bm, grid_n = (N + 255) / 256;
        const int64_t rounds = grid_m * grid_n / cus;
        const int64_t cols = rounds * cus / grid_m;  // columns of tiles that the full rounds hold
        if (cols < 1 || cols >= grid_n) continue;
        const TilePlan rest = tile_plan(M, N - cols * 256, K, ws_bytes);
        const double first_us = (double)rounds * large_round_us(tile, nst), us = first_us + 3.0 + rest.us;
        if (us < best_us) {
            best_us = us;
            best = PrefillPlan{{tile, tiles_k(K), first_us}, rest, cols * 256};
        }
    }
    return best;
}
static int64_t plan_slices(const TilePlan& p, int64_t K) { return (tiles_k(K) + p.per - 1) / p.per; }
// Room for the K-slices of the plan: optional, without it K is not split (or in fewer slices).
size_t prefill_split_bytes(int64_t M, int64_t N, int64_t K, bool one_beta) {
    if (M <= 64) return mid_split_bytes(M, N, K);
    const PrefillPlan p = prefill_plan(M, N, K, (size_t)1 << 40, one_beta);
    const int64_t n = plan_slices(p.cut ? p.rest : p.first, K);
    return n > 1 ? (size_t)n * M * (N - p.cut) * 4 : 0;
}

// The same choice for a grouped layer (K = a group's): 0 = the stream kernel, 3 or 4 = the tiles of
// gemm_mid.hip with every K-group an item of its own, its int32 sums in a slice that the fold
// dequantises (same fp32 operations in the same order, same bits).  The stream kernel's round of
// tiles is taken to cost 6 + groups (1 + 0.42 n) us (1000 x 7168 x 28672, 8 groups: 244 us in 4 rounds, measured 212;
// with constants that fit this one, layers of 66 to 641 tokens at the line, 2 % of all, got up to 15 % slower).
// Whole layers, stream / 128 x 128 slices / 64 x 128 slices: 172 x 1024 x 2560 in 4 groups 19.1 / 18.0 / 17.9, 306 x
// 4352 x 4352 in 4 groups 40.8 / 39.4 / 38.5, 300 x 4096 x 7168 in 4 groups 37.6 / 42.8 / 51.1, 500 x 2048 x 2048 in 4
// groups 25.8 / 24.1 / 28.7; 1000 x 4096 x 4096 in 8 groups 46 / 87 / 126.
static int group_plan(int64_t M, int64_t N, int64_t K, int groups, size_t ws_bytes) {
    const int64_t cus = num_cus(), TK = tiles_k(K), nst = (K + kStageK - 1) / kStageK;
    const int force = tuning().prefill_tile;
    const double bytes = (double)groups * (double)M * (double)N * 4.0;
    const int64_t rounds = ((M + 127) / 128 * ((N + 255) / 256) + cus - 1) / cus;
    double best_us = (double)rounds * (6.0 + groups * (1.0 + 0.42 * (double)nst));
    int best = 0;
    for (int tile = 3; tile <= 4; ++tile) {
        if ((force && tile != force) || bytes > (double)ws_bytes) continue;
        const int64_t bm = tile == 4 ? 64 : 128, kg = tile == 3 ? 2 : 4;
        const int64_t items = ((M + bm - 1) / bm) * ((N + 127) / 128) * groups;
        const double us = (double)((items + cus - 1) / cus) * (3.5 + 4.2 * (double)((TK + kg - 1) / kg)) +
                          5.0 + bytes * 2.0 / 5e6;
        if (us < best_us || force) {
            best_us = us;
            best = tile;
        }
    }
    return best;
}
// Room for the slices of the plan (M > 64): optional.
size_t group_split_bytes(int64_t M, int64_t N, int64_t K, int groups) {
    if (M <= 64 || groups <= 1 || !group_plan(M, N, K, groups, (size_t)1 << 40)) return 0;
    return (size_t)groups * M * N * 4;
}

// K <= kMaxGemmK (a group's K: the large tiles sum up to 2^14 per element of it in int32) and rows of codes below
// 2^22 bytes (the per-lane offset into a block of 256 of them is kept in 32 bits).
hipError_t launch_gemm_prefill(const GemmArgs& a_in, hipStream_t s) {
    GemmArgs a = a_in;
    a.split_k = 0;  // set here only
    if (!a.ldy) a.ldy = a.N;
    if (a.K > kMaxGemmK || a.ldq >= ((int64_t)1 << 22)) return hipErrorInvalidValue;
    if (a.M <= 64) {  // up to 32 tokens: gemm_stream.hip where it takes the shape; else gemm_mid.hip
        if (!tuning().mid_only && a_in.kgroups <= 1 && launch_gemm_stream(a_in, s)) return hipGetLastError();
        return launch_gemm_mid(a_in, s);
    }
    if (a.kgroups > 1) {
        const int tile = group_plan(a.M, a.N, a.K, a.kgroups, a.split_ws ? a.split_ws_bytes : 0);
        if (tile) return launch_gemm_mid_tiles(a, tile == 3 ? 128 : 64, tiles_k(a.K), s);
        const int grid_m = (int)((a.M + 127) / 128), grid_n = (int)((a.N + 255) / 256);
        int grid = num_cus();  // one workgroup per CU
        if (tuning().prefill_grid > 0) grid = tuning().prefill_grid;
        if (grid > grid_m * grid_n) grid = grid_m * grid_n;
        if (a.eta) gemm_group_kernel<true><<<(unsigned)grid, 512, 0, s>>>(a, grid_m, grid_n);
        else gemm_group_kernel<false><<<(unsigned)grid, 512, 0, s>>>(a, grid_m, grid_n);
        return hipGetLastError();
    }
    const PrefillPlan p = prefill_plan(a.M, a.N, a.K, a.split_ws ? a.split_ws_bytes : 0, a.beta_rows >= a.N);
    auto launch = [&](const GemmArgs& b, const TilePlan& t) {
        if (t.tile >= 3) return launch_gemm_mid_tiles(b, t.tile == 3 ? 128 : 64, t.per, s);
        if (t.tile == 1) launch_tile<128, 256, 2, 4, 8>(b, s);
        else launch_tile<256, 256, 2, 4, 8>(b, s);
        return hipGetLastError();
    };
    if (!p.cut) return launch(a, p.first);
    GemmArgs b = a;
    a.N = a.beta_rows = p.cut;
    b.N = b.beta_rows = b.N - p.cut;
    b.Y += p.cut;
    b.packed += tile_dword_offset(p.cut / kTileN, 0, b.tk_pitch ? b.tk_pitch : tiles_k(b.K));
    if (b.wsum) b.wsum += p.cut;
    if (const hipError_t e = launch(a, p.first); e != hipSuccess) return e;
    return launch(b, p.rest);
}

}  // namespace bl

// Pieces shared by the MFMA kernels that stream their operands global -> LDS by DMA
// (global_load_lds) and keep count of the outstanding operations by hand.
#pragma once
#include <type_traits>

#include "common.h"

namespace bl {

// compile-time loop: f(integral_constant<int, B>), ..., f(integral_constant<int, E-1>)
template <int B, int E, class F>
__device__ inline void static_for(F&& f) {
    if constexpr (B < E) {
        f(std::integral_constant<int, B>{});
        static_for<B + 1, E>(f);
    }
}

template <int N>
__device__ inline void wait_vmcnt() {
    static_assert(N >= 0 && N < 64, "vmcnt range");
    // gfx9 encoding: vmcnt = {[15:14],[3:0]}, expcnt [6:4] = 7 and lgkmcnt [11:8] = 15 (no wait).
    // The compiler barrier keeps ordinary memory operations on their side of the wait.
    asm volatile("" ::: "memory");
    __builtin_amdgcn_s_waitcnt((N & 15) | ((N >> 4) << 14) | (7 << 4) | (15 << 8));
}

__device__ inline void block_barrier() {
    asm volatile("" ::: "memory");
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
}

// Stores a wave's tile of MI x NI MFMA blocks of 32 x 32: lane (j, g2) holds columns 32 s + j, rows 32 mi + 8 rq +
// 4 g2 + rr of it.  `base` (uniform: the tile's first element) walks the rows by the pitch, as a scalar
// that is hidden from the optimiser, which would compute all the addresses ahead and spill; a lane's place in
// a row is one register.  With the rows' bounds, a 64-bit product per row and their branches at every store,
// the instructions around the stores were 10 us of a 256 x 256 tile.  rows, cols: how many of the tile exist;
// pre(mi, rq) runs ahead of four rows, val(mi, r, s) is the value of block (mi, s), register r = 4 rq + rr.
// EDGES = false (kernels without a register to spare): the caller vouches that all of the tile exists
// and pitch < 2^24.
template <int MI, int NI, bool EDGES, class PRE, class VAL>
__device__ inline void store_tile(float* base, int64_t pitch, int64_t rows, int64_t cols, int j, int g2,
                                  PRE&& pre, VAL&& val) {
    typedef __attribute__((address_space(1))) float* gptr;
    const uint64_t at = (uint64_t)(uintptr_t)base;
    const gptr first = (gptr)((uint64_t)(uint32_t)__builtin_amdgcn_readfirstlane((int)at) |
                              (uint64_t)(uint32_t)__builtin_amdgcn_readfirstlane((int)(at >> 32)) << 32);
    using offset = std::conditional_t<EDGES, int64_t, uint32_t>;
    const offset lane = (offset)(4 * g2) * (offset)pitch + (offset)j;
    auto walk = [&](auto ragged) {
        constexpr bool RAGGED = decltype(ragged)::value;
        gptr rowp = first;
        const int mine = (int)(rows < 32 * MI ? rows : 32 * MI) - 4 * g2;  // this lane's rows end here
        const int last = (int)(cols < 32 * NI ? cols : 32 * NI) - j;       // and its columns
#pragma unroll
        for (int mi = 0; mi < MI; ++mi)
#pragma unroll
            for (int rq = 0; rq < 4; ++rq) {
                pre(mi, rq);
#pragma unroll
                for (int rr = 0; rr < 4; ++rr) {
                    asm volatile("" : "+s"(rowp));
                    if (!RAGGED || 32 * mi + 8 * rq + rr < mine) {
#pragma unroll
                        for (int s = 0; s < NI; ++s)
                            // streaming: keeping the output out of L2 leaves the operands there
                            if (!RAGGED || 32 * s < last)
                                __builtin_nontemporal_store(val(mi, 4 * rq + rr, s), rowp + (lane + 32 * s));
                    }
                    rowp += rr == 3 ? 5 * pitch : pitch;
                }
            }
    };
    if (!EDGES || (rows >= 32 * MI && cols >= 32 * NI)) walk(std::false_type{});  // uniform
    else walk(std::integral_constant<bool, EDGES>{});
}

}  // namespace bl

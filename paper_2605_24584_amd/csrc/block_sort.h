// Stable sort of the (key, value) pairs of one workgroup, by merging in LDS (used by run_sort_kernels.hip).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace laplex {

// Thread t holds the ITEMS consecutive pairs t * ITEMS .. of a tile of THREADS * ITEMS; afterwards the same slots of the
// sorted tile.  Each thread sorts its own pairs by exchanges of neighbours (stable), then runs of doubling width are merged:
// a thread finds where its ITEMS outputs start in the two runs (binary search along the diagonal) and merges them serially;
// the values follow by index.  Merges of runs that lie inside one wavefront need no barrier (LDS operations of a wavefront
// take effect in program order).  The chain of dependent LDS reads is what bounds it, so few items per thread and many
// threads win: 1024 pairs take 4.3 us as 512 x 2 and 5.1 us as 256 x 4, 2048 pairs 6.7 us as 1024 x 2 (ranking by ballots,
// digit by digit, costs 0.7 us per 512 keys and pass, four passes of it).
// sk, sv: THREADS * ITEMS + 2 words of LDS each.
template <int THREADS, int ITEMS>
__device__ __forceinline__ void block_sort(uint32_t (&key)[ITEMS], uint32_t (&val)[ITEMS], uint32_t* sk, uint32_t* sv)
{
    const int tid = threadIdx.x;
#pragma unroll
    for (int r = 0; r < ITEMS; ++r) {
#pragma unroll
        for (int i = r & 1; i + 1 < ITEMS; i += 2) {
            const bool swap = key[i + 1] < key[i];
            const uint32_t k0 = swap ? key[i + 1] : key[i], k1 = swap ? key[i] : key[i + 1];
            const uint32_t v0 = swap ? val[i + 1] : val[i], v1 = swap ? val[i] : val[i + 1];
            key[i] = k0; key[i + 1] = k1; val[i] = v0; val[i + 1] = v1;
        }
    }
    for (int width = ITEMS; width < THREADS * ITEMS; width *= 2) {
        const bool in_wave = 2 * width <= 64 * ITEMS;          // uniform
        auto meet = [&]() {
            if (in_wave) {
                __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
                __builtin_amdgcn_wave_barrier();
            } else {
                __syncthreads();
            }
        };
        meet();
#pragma unroll
        for (int i = 0; i < ITEMS; ++i) { sk[tid * ITEMS + i] = key[i]; sv[tid * ITEMS + i] = val[i]; }
        meet();
        const int base = (tid * ITEMS) & ~(2 * width - 1);
        const int diag = tid * ITEMS - base;
        const int second = base + width;
        int lo = diag > width ? diag - width : 0, hi = diag < width ? diag : width;
        while (lo < hi) {
            const int mid = (lo + hi) >> 1;
            if (sk[base + mid] <= sk[second + diag - 1 - mid]) lo = mid + 1; else hi = mid;
        }
        int i = base + lo, j = second + diag - lo;
        const int i_end = second, j_end = second + width;
        uint32_t ka = sk[i], kb = sk[j];                       // (one past the tile at most: the two spare words)
        int from[ITEMS];
#pragma unroll
        for (int e = 0; e < ITEMS; ++e) {
            const bool take_a = i < i_end && (j >= j_end || ka <= kb);
            key[e] = take_a ? ka : kb;
            from[e] = take_a ? i : j;
            if (take_a) ++i; else ++j;
            const uint32_t next = sk[take_a ? i : j];
            ka = take_a ? next : ka;
            kb = take_a ? kb : next;
        }
#pragma unroll
        for (int e = 0; e < ITEMS; ++e) val[e] = sv[from[e]];
    }
}

}  // namespace laplex

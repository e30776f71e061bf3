// Sorting the merged anchors in two launches (Sec. 3 "Complexity": the O(n log n) term), for sequences that are too long to be
// ranked by counting and too short for a radix sort to be bound by anything but the latency of its launches and of the hops
// from tile to tile: up to kRunSortMax merged positions.
//
//   k_run_sort     every workgroup sorts a tile of consecutive positions in LDS (block_sort.h) and writes it as a run of
//                  (key, id) pairs, with every STEP-th key once more in an array of samples
//   k_bucket_sort  workgroup g owns the g-th stretch of the sorted sequence.  It finds the samples that bound the stretch
//                  (radix selection over all samples, in LDS), the place of either bound in every run (search among the run's
//                  samples, then among the STEP - 1 keys between two of them), gathers what lies between from all runs,
//                  sorts it in LDS and writes the plan: ids, sorted anchors and, since it holds neighbours, the decays.
//
// Nothing is counted, cleared or waited for across workgroups, and the order is that of the radix sort bit for bit: pairs
// are compared as (key, run, position in the run), and runs are stretches of positions in ascending order.
// A bound is a sample, so a stretch holds the average number of pairs up to what lies between samples: for R runs a
// boundary scatters by about STEP * sqrt(R / 12) pairs, and the configurations below leave more than three times the scatter of
// a stretch to the capacity of a workgroup.  In the worst case it holds (samples per stretch + R) * STEP pairs, 2.7 times the
// capacity; a stretch beyond the capacity is sorted in parts, whose pairs are then searched in each other.
//
// Measured (MI355X, us, this sort / radix sort and decay pass; keys uniform): 9000 positions 22 / 35, 2^15: 23 / 41, 2^17: 28 / 48,
// 2^18: 36 / 57, 2^19: 57 / 71; at 2^20 positions, with 257 runs, 107 / 83: hence kRunSortMax = 2^19.  Of the second kernel's 18 us at
// 2^17 positions the sort in LDS is 5.6, the selection 5.3, cutting and gathering 4.7.  Keys that arrive ascending: 39 / 49 at 2^17,
// 62 / 69 at 2^19; all equal, where the radix sort skips every pass: 31 / 28 and 56 / 40; all stretches' keys between two samples of
// every run (the most that a stretch can hold): 56 / 49 and 148 / 73.
#include "laplex_internal.h"
#include "block_sort.h"

namespace laplex {

namespace {

__device__ __forceinline__ uint32_t run_key(float f)
{
    const uint32_t u = __float_as_uint(f + 0.0f);       // -0.0 sorts as +0.0
    return u ^ ((uint32_t)((int32_t)u >> 31) | 0x80000000u);
}
__device__ __forceinline__ float run_key_to_float(uint32_t key)
{
    return __uint_as_float(key ^ ((key >> 31) ? 0x80000000u : 0xFFFFFFFFu));
}

struct RunArgs {
    const float* a; const float* b; int64_t k; float tau; int N;
    uint32_t* run_keys; uint32_t* run_ids; uint32_t* samples;      // the runs; their samples, 2^kRunSampleBits per run
    uint32_t* ids; float* dh; float* pk; float2* pk8; uint32_t* counters;     // the plan
    int runs, buckets, total_samples;
    int64_t op_a, op_b, op_ws;                            // strides from one operator to the next (elements; bytes of workspace)
};

// Position of a run's first sample; the others follow STEP pairs apart.  Staggered from run to run: with the same place in every run
// the stretches at the ends of the sequence, and on inputs that repeat themselves any stretch, would hold what lies between two samples
// of all runs at once (R * STEP / 2 pairs more or less than the average).  The samples of a last run that is shorter repeat its largest
// key.
__device__ __forceinline__ int first_sample(int run, int step) { return (run * 11) & (step - 1); }

template <typename T>
__device__ __forceinline__ T* op_shift(T* p, int64_t bytes) { return reinterpret_cast<T*>(reinterpret_cast<char*>(p) + bytes); }

template <int THREADS, int ITEMS>
__global__ void __launch_bounds__(THREADS)
k_run_sort(const RunArgs A)
{
    constexpr int TILE = THREADS * ITEMS, STEP = TILE >> kRunSampleBits;
    __shared__ uint32_t sk[TILE + 2], sv[TILE + 2];
    const int64_t op = blockIdx.y;
    const float* a = A.a + op * A.op_a;
    const float* b = A.b + op * A.op_b;
    uint32_t* run_keys = op_shift(A.run_keys, op * A.op_ws);
    uint32_t* run_ids = op_shift(A.run_ids, op * A.op_ws);
    uint32_t* samples = op_shift(A.samples, op * A.op_ws);
    const int run = blockIdx.x, base = run * TILE, q0 = threadIdx.x * ITEMS;
    const int len = A.N - base < TILE ? A.N - base : TILE;
    uint32_t key[ITEMS], id[ITEMS];
#pragma unroll
    for (int i = 0; i < ITEMS; ++i) {
        const int q = q0 + i;
        const int64_t pos = base + (q < len ? q : len - 1);
        const uint32_t kk = run_key(A.tau * (pos < A.k ? a[pos] : b[pos - A.k]));
        key[i] = q < len ? kk : 0xFFFFFFFFu;              // padding comes last: it is behind every key that is equal to it
        id[i] = (uint32_t)pos;
    }
    block_sort<THREADS, ITEMS>(key, id, sk, sv);
#pragma unroll
    for (int i = 0; i < ITEMS; ++i) {
        const int q = q0 + i;
        if (q < len) {
            run_keys[base + q] = key[i];
            run_ids[base + q] = id[i];
            if ((q & (STEP - 1)) == first_sample(run, STEP)) samples[(run << kRunSampleBits) + q / STEP] = key[i];
        }
        if (q == len - 1)
            for (int m = (q - first_sample(run, STEP) + STEP) / STEP; m < 1 << kRunSampleBits; ++m) samples[(run << kRunSampleBits) + m] = key[i];
    }
}

typedef uint32_t u4 __attribute__((ext_vector_type(4), aligned(4)));

// Where a bound cuts a run: p0 + the number of keys in [p0, p1), fewer than STEP of them, that are below `key` (or equal, with
// or_equal).  Up to 32 keys are all loaded at once; 64 in two rounds of eight (a binary search would be six dependent loads).
// (Loads may reach past the end of the run, up to STEP words: into the next run or the ids behind the last one.)
template <int STEP>
__device__ __forceinline__ int cut_between(const uint32_t* __restrict__ run, int p0, int p1, uint32_t key, bool or_equal)
{
    const uint32_t limit = or_equal ? key : key - 1u;           // left of the bound: v <= limit (none if key is 0 and equal keys stay)
    const bool none = !or_equal && key == 0u;
    auto count8 = [&](const uint32_t* at, int stop) {
        const u4 v0 = *reinterpret_cast<const u4*>(at), v1 = *reinterpret_cast<const u4*>(at + 4);
        int c = 0;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            c += (i < stop && v0[i] <= limit) ? 1 : 0;
            c += (i + 4 < stop && v1[i] <= limit) ? 1 : 0;
        }
        return c;
    };
    if (p1 <= p0 || none) return p0 < p1 ? p0 : p1;
    if constexpr (STEP <= 32) {
        int c = 0;
#pragma unroll
        for (int q = 0; q < STEP; q += 8) c += count8(run + p0 + q, p1 - p0 - q);
        return p0 + c;
    } else {
        static_assert(STEP == 64, "eight stretches of eight");
        uint32_t v[8];
#pragma unroll
        for (int i = 0; i < 8; ++i) v[i] = run[p0 + 8 * i + 7 < p1 ? p0 + 8 * i + 7 : p1 - 1];
        int c = 0;
#pragma unroll
        for (int i = 0; i < 8; ++i) c += (p0 + 8 * i + 7 < p1 && v[i] <= limit) ? 1 : 0;
        p0 += 8 * c;
        return p0 < p1 ? p0 + count8(run + p0, p1 - p0) : p0;
    }
}

// Exclusive scan of one word per thread over the workgroup; *total gets the sum.  part: THREADS / 64 words of LDS.
template <int THREADS>
__device__ __forceinline__ uint32_t block_exclusive_scan(uint32_t v, uint32_t* part, uint32_t* total)
{
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    uint32_t inc = v;
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) {
        const uint32_t o = __shfl_up(inc, d);
        if (lane >= d) inc += o;
    }
    if (lane == 63) part[wave] = inc;
    __syncthreads();
    uint32_t before = 0u, all = 0u;
#pragma unroll
    for (int w = 0; w < THREADS / 64; ++w) {
        const uint32_t t = part[w];
        if (w < wave) before += t;
        all += t;
    }
    *total = all;
    __syncthreads();
    return before + inc - v;
}

constexpr int kBucketBins = 2048, kBucketList = 256;

template <int THREADS, int ITEMS>
__global__ void __launch_bounds__(THREADS, THREADS / 128)
k_bucket_sort(const RunArgs A)
{
    constexpr int CAP = THREADS * ITEMS, TILE = CAP, STEP = TILE >> kRunSampleBits;
    constexpr int HALF = THREADS / 2, MAX_RUNS = kRunSortMaxRuns < HALF ? kRunSortMaxRuns : HALF;
    constexpr int BINS_PER = kBucketBins / THREADS;
    extern __shared__ __align__(16) uint32_t buf[];           // the samples; then keys and ids of the stretch (sized by the launcher)
    __shared__ uint32_t hist[kBucketBins];                    // two 16-bit counts per word: for the lower bound, for the upper bound
    __shared__ uint32_t part[THREADS / 64], part2[THREADS / 64];
    __shared__ uint32_t list[2][kBucketList], list_len[2];
    __shared__ uint32_t key_min, key_max, prev_key;
    __shared__ uint32_t sel_bin[2], sel_rank[2], sel_count[2], sel_key[2];
    __shared__ int cut[2][MAX_RUNS];
    __shared__ int offset[MAX_RUNS + 1];
    const int tid = threadIdx.x, lane = tid & 63;
    const int64_t op = blockIdx.y;
    const uint32_t* __restrict__ run_keys = op_shift(A.run_keys, op * A.op_ws);
    const uint32_t* __restrict__ run_ids = op_shift(A.run_ids, op * A.op_ws);
    const uint32_t* __restrict__ samples = op_shift(A.samples, op * A.op_ws);
    uint32_t* ids = op_shift(A.ids, op * A.op_ws);
    float* dh = op_shift(A.dh, op * A.op_ws);
    float* pk = op_shift(A.pk, op * A.op_ws);
    float2* pk8 = A.pk8 ? op_shift(A.pk8, op * A.op_ws) : nullptr;
    const int g = blockIdx.x, runs = A.runs, total = A.total_samples, N = A.N;

    if (g == 0 && tid < 64) op_shift(A.counters, op * A.op_ws)[tid] = 0u;        // list lengths of the scans; the plan is valid
    if (tid == 0) { key_min = 0xFFFFFFFFu; key_max = 0u; prev_key = 0u; }
    if (tid < 2) {
        const long long r = (long long)(g + tid) * total / A.buckets;
        sel_rank[tid] = (uint32_t)(r < total ? r : total - 1);
        list_len[tid] = 0u;
    }
    for (int i = tid; i < kBucketBins; i += THREADS) hist[i] = 0u;
    __syncthreads();
    // 1. the two samples of the given ranks, by histograms of 2048 bins over the range of the samples, then of the bin a rank
    //    falls into, until the bin holds few samples (one round, as a rule) or a single value.  A thread keeps its share of the
    //    samples in registers for this; step 2 reads them by run from LDS.
    constexpr int QUADS = (MAX_RUNS << kRunSampleBits) / 4 / THREADS;
    static_assert((MAX_RUNS << kRunSampleBits) % (4 * THREADS) == 0, "whole quads per thread");
    uint4 quad[QUADS];
    auto each_sample = [&](auto use) {
#pragma unroll
        for (int q = 0; q < QUADS; ++q) {
            if (4 * (q * THREADS + tid) < total) { use(quad[q].x); use(quad[q].y); use(quad[q].z); use(quad[q].w); }
        }
    };
#pragma unroll
    for (int q = 0; q < QUADS; ++q) {
        const int i = 4 * (q * THREADS + tid);
        quad[q] = make_uint4(0u, 0u, 0u, 0u);
        if (i < total) quad[q] = *reinterpret_cast<const uint4*>(samples + i);
    }
    {
        uint32_t lo = 0xFFFFFFFFu, hi = 0u;
        each_sample([&](uint32_t v) { lo = v < lo ? v : lo; hi = v > hi ? v : hi; });
#pragma unroll
        for (int q = 0; q < QUADS; ++q) {
            const int i = 4 * (q * THREADS + tid);
            if (i < total) *reinterpret_cast<uint4*>(buf + i) = quad[q];
        }
#pragma unroll
        for (int m = 32; m >= 1; m >>= 1) {
            const uint32_t l2 = __shfl_xor(lo, m), h2 = __shfl_xor(hi, m);
            lo = l2 < lo ? l2 : lo; hi = h2 > hi ? h2 : hi;
        }
        if (lane == 0) { atomicMin(&key_min, lo); atomicMax(&key_max, hi); }
    }
    __syncthreads();
    uint32_t low[2], shift[2];                      // uniform, like everything that is read from sel_*
    {
        const uint32_t span = key_max - key_min;
        const int bits = span ? 32 - __clz((int)span) : 0;
        low[0] = low[1] = key_min;
        shift[0] = shift[1] = (uint32_t)(bits > 11 ? bits - 11 : 0);
    }
    bool done[2] = {false, false}, first_round = true;
#pragma unroll 1
    for (;;) {
        if (first_round) {                          // the same range for both bounds
            each_sample([&](uint32_t v) { atomicAdd(&hist[(v - low[0]) >> shift[0]], 0x10001u); });
        } else {
            each_sample([&](uint32_t v) {
                const uint32_t d0 = (v - low[0]) >> shift[0], d1 = (v - low[1]) >> shift[1];
                if (!done[0] && v >= low[0] && d0 < (uint32_t)kBucketBins) atomicAdd(&hist[d0], 1u);
                if (!done[1] && v >= low[1] && d1 < (uint32_t)kBucketBins) atomicAdd(&hist[d1], 0x10000u);
            });
        }
        __syncthreads();
        uint32_t mine = 0u, c[BINS_PER], all;
#pragma unroll
        for (int q = 0; q < BINS_PER; ++q) { c[q] = hist[tid * BINS_PER + q]; hist[tid * BINS_PER + q] = 0u; mine += c[q]; }
        uint32_t sum = block_exclusive_scan<THREADS>(mine, part, &all);
        const uint32_t want[2] = {sel_rank[0], sel_rank[1]};
        __syncthreads();
#pragma unroll
        for (int q = 0; q < BINS_PER; ++q) {
#pragma unroll
            for (int w = 0; w < 2; ++w) {
                const uint32_t below = (sum >> (16 * w)) & 0xFFFFu, here = (c[q] >> (16 * w)) & 0xFFFFu;
                if (want[w] >= below && want[w] < below + here) {
                    sel_bin[w] = (uint32_t)(tid * BINS_PER + q);
                    sel_rank[w] = want[w] - below;
                    sel_count[w] = here;
                }
            }
            sum += c[q];
        }
        __syncthreads();
#pragma unroll
        for (int w = 0; w < 2; ++w) {
            if (done[w]) continue;
            low[w] += sel_bin[w] << shift[w];
            done[w] = sel_count[w] <= (uint32_t)kBucketList || shift[w] == 0u;
            if (!done[w]) shift[w] = shift[w] > 11u ? shift[w] - 11u : 0u;
        }
        if (done[0] && done[1]) break;
        first_round = false;
        __syncthreads();
    }
    if ((shift[0] | shift[1]) == 0u) {              // bins of a single value
        if (tid < 2) sel_key[tid] = low[tid];
    } else {
        // the samples of the two bins by brute force: each against all of its own bin
        const uint32_t width[2] = {(1u << shift[0]) - 1u, (1u << shift[1]) - 1u};
        each_sample([&](uint32_t v) {
            const bool in0 = v - low[0] <= width[0], in1 = v - low[1] <= width[1];
            if (in0 || in1) {
                if (in0) list[0][atomicAdd(&list_len[0], 1u) & (kBucketList - 1)] = v;
                if (in1) list[1][atomicAdd(&list_len[1], 1u) & (kBucketList - 1)] = v;
            }
        });
        __syncthreads();
        const int w = tid / HALF, me_at = tid % HALF;
        const uint32_t rank = sel_rank[w];
        const int len = (int)(list_len[w] < (uint32_t)kBucketList ? list_len[w] : (uint32_t)kBucketList);
        __syncthreads();
        if ((w ? shift[1] : shift[0]) == 0u) {
            if (me_at == 0) sel_key[w] = w ? low[1] : low[0];
        } else if ((me_at & ~63) < len) {           // uniform per wavefront
            const uint32_t me = me_at < len ? list[w][me_at] : 0u;
            uint32_t less = 0u, equal = 0u;
#pragma unroll 4
            for (int i = 0; i < len; ++i) { const uint32_t v = list[w][i]; less += v < me ? 1u : 0u; equal += v == me ? 1u : 0u; }
            if (me_at < len && rank >= less && rank < less + equal) { sel_key[w] = me; sel_rank[w] = rank - less; }      // (equal keys write the same)
        }
    }
    __syncthreads();
    // 2. where the bounds cut the runs: half of the threads per bound, one run each
    {
        const int w = tid / HALF, r = tid % HALF;
        const uint32_t key = sel_key[w];
        const bool live = r < runs;
        const int len = !live ? 0 : (N - r * TILE < TILE ? N - r * TILE : TILE);
        const int first = first_sample(r, STEP), count = live ? 1 << kRunSampleBits : 0;
        auto at_sample = [&](int q) { const int p = q * STEP + first; return p < len ? p : len; };
        const uint32_t* sm = buf + (r << kRunSampleBits);
        int lo = 0, hi = count;
        while (lo < hi) { const int mid = (lo + hi) >> 1; if (sm[mid] < key) lo = mid + 1; else hi = mid; }
        const int lb = lo;
        hi = count;
        if (lo < count && sm[lo] == key)
            while (lo < hi) { const int mid = (lo + hi) >> 1; if (sm[mid] <= key) lo = mid + 1; else hi = mid; }
        const int ub = lo;
        // among equal samples the runs come in order: those before the run that holds the bound take the equal keys with them
        uint32_t all;
        const uint32_t eq = (uint32_t)(ub - lb);
        const uint32_t ex = block_exclusive_scan<THREADS>(w ? eq << 16 : eq, part, &all);
        const uint32_t before = w ? ex >> 16 : ex & 0xFFFFu, rank = sel_rank[w];
        int at = 0;
        if (live) {
            if (w == 0 && g == 0) {
                at = 0;
            } else if (w == 1 && g == A.buckets - 1) {
                at = len;
            } else if (rank >= before && rank < before + eq) {
                at = at_sample(lb + (int)(rank - before));
            } else {
                const bool or_equal = before + eq <= rank;
                const int q = or_equal ? ub : lb;
                const int p0 = q == 0 ? 0 : at_sample(q - 1) + 1;
                const int p1 = q < count ? at_sample(q) : len;
                at = cut_between<STEP>(run_keys + r * TILE, p0, p1, key, or_equal);
            }
            cut[w][r] = at;
        }
    }
    __syncthreads();
    // 3. the stretch: its place in the sorted sequence, its length, and the largest key before it
    int cnt, base;
    {
        const int lo = tid < runs ? cut[0][tid] : 0, n = tid < runs ? cut[1][tid] - lo : 0;
        uint32_t last = lo > 0 ? run_keys[tid * TILE + lo - 1] : 0u;
        uint32_t all_n, all_lo;
        const uint32_t ex = block_exclusive_scan<THREADS>((uint32_t)n, part, &all_n);
        if (tid < runs) offset[tid] = (int)ex;
        if (tid == 0) offset[runs] = (int)all_n;
        uint32_t sum_lo = (uint32_t)lo;
#pragma unroll
        for (int m = 32; m >= 1; m >>= 1) {
            sum_lo += __shfl_xor(sum_lo, m);
            const uint32_t l2 = __shfl_xor(last, m);
            last = l2 > last ? l2 : last;
        }
        if (lane == 0) { part[tid >> 6] = sum_lo; part2[tid >> 6] = last; }
        __syncthreads();
        all_lo = 0u;
        uint32_t top = 0u;
#pragma unroll
        for (int w = 0; w < THREADS / 64; ++w) { all_lo += part[w]; top = part2[w] > top ? part2[w] : top; }
        if (tid == 0) prev_key = top;
        cnt = (int)all_n;
        base = (int)all_lo;
    }
    auto place = [&](int e) -> int {                // where pair e of the stretch lies
        int lo = 0, hi = runs;                      // the last run whose offset is at most e
        while (hi - lo > 1) { const int mid = (lo + hi) >> 1; if (offset[mid] <= e) lo = mid; else hi = mid; }
        return lo * TILE + cut[0][lo] + (e - offset[lo]);
    };
    auto write = [&](int j, uint32_t key, uint32_t before, uint32_t id) {
        const float p = run_key_to_float(key);
        ids[j] = id;
        pk[j + 1] = p;
        dh[j] = j == 0 ? 0.0f : key == before ? -1.0f : expf(-(p - run_key_to_float(before)));
        if (pk8) {                                  // pk8[m] = (pk[8m], pk[8m + 1])
            if ((j & 7) == 7) pk8[(j + 1) >> 3].x = p;
            if ((j & 7) == 0) pk8[j >> 3].y = p;
        }
    };
    if (cnt <= CAP) {                               // uniform
        uint32_t key[ITEMS], id[ITEMS];
        uint32_t* const sk = buf;
        uint32_t* const sv = buf + CAP + 2;
        const int e0 = tid * ITEMS;
#pragma unroll
        for (int i = 0; i < ITEMS; ++i) {
            const bool ok = e0 + i < cnt;
            const int at = cnt > 0 ? place(ok ? e0 + i : 0) : 0;
            const uint32_t kk = run_keys[at];
            key[i] = ok ? kk : 0xFFFFFFFFu;
            id[i] = run_ids[at];
        }
        __syncthreads();                            // (the samples are done with)
        block_sort<THREADS, ITEMS>(key, id, sk, sv);
        __syncthreads();
        sk[tid] = key[ITEMS - 1];
        __syncthreads();
        uint32_t before = tid == 0 ? prev_key : sk[tid - 1];
#pragma unroll
        for (int i = 0; i < ITEMS; ++i) {
            if (e0 + i < cnt) write(base + e0 + i, key[i], before, id[i]);
            before = key[i];
        }
    } else {
        // Beyond the capacity: CAP pairs at a time are sorted in LDS, and every pair of the stretch is searched in each such part (in its
        // own with its place in the stretch as the second key; equal keys of earlier parts come before it).  At most three parts.
        constexpr int MINE = 3 * ITEMS;
        uint32_t* const sk = buf;
        uint32_t* const sv = buf + CAP + 2;
        for (int e0 = 0; e0 < cnt; e0 += MINE * THREADS) {
            uint32_t me[MINE];
            int rank[MINE];
#pragma unroll
            for (int i = 0; i < MINE; ++i) {
                const int e = e0 + i * THREADS + tid;
                me[i] = e < cnt ? run_keys[place(e)] : 0u;
                rank[i] = 0;
            }
            for (int c0 = 0; c0 < cnt; c0 += CAP) {
                const int len = cnt - c0 < CAP ? cnt - c0 : CAP;
                uint32_t key[ITEMS], val[ITEMS];
#pragma unroll
                for (int i = 0; i < ITEMS; ++i) {
                    const int q = tid * ITEMS + i;
                    key[i] = q < len ? run_keys[place(c0 + q)] : 0xFFFFFFFFu;
                    val[i] = (uint32_t)q;
                }
                __syncthreads();
                block_sort<THREADS, ITEMS>(key, val, sk, sv);
                __syncthreads();
#pragma unroll
                for (int i = 0; i < ITEMS; ++i) { sk[tid * ITEMS + i] = key[i]; sv[tid * ITEMS + i] = val[i]; }
                __syncthreads();
#pragma unroll
                for (int i = 0; i < MINE; ++i) {
                    const int e = e0 + i * THREADS + tid;
                    if (e >= cnt) continue;
                    const uint32_t own = e < c0 ? 0u : e - c0 < CAP ? (uint32_t)(e - c0) : 0xFFFFFFFFu;      // equal keys below this place count
                    int lo = 0, hi = len;
                    while (lo < hi) {
                        const int mid = (lo + hi) >> 1;
                        const uint32_t v = sk[mid];
                        if (v < me[i] || (v == me[i] && sv[mid] < own)) lo = mid + 1; else hi = mid;
                    }
                    rank[i] += lo;
                }
            }
#pragma unroll
            for (int i = 0; i < MINE; ++i) {
                const int e = e0 + i * THREADS + tid;
                if (e < cnt) { ids[base + rank[i]] = run_ids[place(e)]; pk[base + rank[i] + 1] = run_key_to_float(me[i]); }
            }
            __syncthreads();
        }
        __threadfence_block();
        __syncthreads();
        for (int e = tid; e < cnt; e += THREADS) {
            const int j = base + e;
            const uint32_t key = run_key(pk[j + 1]), before = e == 0 ? prev_key : run_key(pk[j]);
            write(j, key, before, ids[j]);
        }
    }
    if (g == 0 && tid == 0) {
        pk[0] = __uint_as_float(0xFF800000u);
        if (pk8) pk8[0].x = __uint_as_float(0xFF800000u);
    }
    if (g == A.buckets - 1 && tid == 0) {
        const float inf = __uint_as_float(0x7F800000u);
        dh[N] = 0.0f;
        pk[N + 1] = inf;
        if (pk8) {
            if ((N & 7) == 7) pk8[(N + 1) >> 3] = make_float2(inf, inf);
            if ((N & 7) == 0) pk8[N >> 3].y = inf;
        }
    }
}

template <int THREADS, int ITEMS>
hipError_t launch(RunArgs A, int64_t average, int64_t operators, hipStream_t st)
{
    constexpr int TILE = THREADS * ITEMS;
    A.runs = (A.N + TILE - 1) / TILE;
    A.buckets = (int)((A.N + average - 1) / average);
    A.total_samples = A.runs << kRunSampleBits;
    LAPLEX_TIMED("run_sort", st, hipLaunchKernelGGL((k_run_sort<THREADS, ITEMS>), dim3((unsigned)A.runs, (unsigned)operators), dim3(THREADS), 0, st, A));
    const int sample_words = A.total_samples, sort_words = 2 * (TILE + 2);
    const size_t lds = sizeof(uint32_t) * (size_t)(sample_words > sort_words ? sample_words : sort_words);
    LAPLEX_TIMED("bucket_sort", st, hipLaunchKernelGGL((k_bucket_sort<THREADS, ITEMS>), dim3((unsigned)A.buckets, (unsigned)operators), dim3(THREADS), lds, st, A));
    return hipGetLastError();
}

}  // namespace

hipError_t launch_run_sort(const float* a, int64_t k, const float* b, int64_t n, float tau, uint32_t* runs, uint32_t* samples,
                           uint32_t* ids, float* dh, float* pk, float2* pk8, uint32_t* counters,
                           int64_t operators, int64_t op_a, int64_t op_b, int64_t op_ws, hipStream_t st)
{
    RunArgs A{};
    A.a = a; A.b = b; A.k = k; A.tau = tau; A.N = (int)(k + n);
    A.run_keys = runs; A.run_ids = runs + (k + n); A.samples = samples; A.ids = ids; A.dh = dh; A.pk = pk; A.pk8 = pk8; A.counters = counters;
    A.op_a = op_a; A.op_b = op_b; A.op_ws = op_ws;
    // (tile and capacity, average stretch): up to 128 runs, so the scatter of a stretch's length is at most a 14th of the
    // capacity; the average leaves five times that, and 870 / 1940 / 3330 pairs were the most seen on random keys
    if (A.N <= (1 << 17)) return launch<512, 2>(A, 640, operators, st);
    if (A.N <= (1 << 18)) return launch<1024, 2>(A, 1280, operators, st);
    return launch<1024, 4>(A, 2560, operators, st);
}

}  // namespace laplex

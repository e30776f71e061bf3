// Sorting the merged anchors by samples (Sec. 3 "Complexity": the O(n log n) term): bounds, one distribution, one sort in LDS per
// stretch of the sorted sequence.
//
//   k_split_sample, k_split_pick   samples of the anchors are ranked by counting, every sample against all others; every per_bound-th is
//                  the lower bound of a stretch
//   k_split_tiles  every workgroup takes a tile of consecutive positions and lays it out stretch by stretch (search among the bounds,
//                  counts in LDS), in the tile's own place, with a table of where each stretch starts in it
//   k_split_sort   workgroup g gathers stretch g from all tiles, sorts it in LDS and writes the plan: ids, sorted anchors and, since it
//                  holds neighbours, the decays
//
// Pairs are compared as (key, id) throughout, bounds included, so equal keys are spread over stretches like any others, the order is
// that of a stable sort bit for bit in whatever order the counts in LDS land, and how long a stretch can get depends on the places of
// the samples alone, not on the values.  Nothing is waited for across workgroups and no place in memory is reserved: a stretch starts
// where the tiles' counts add up to.  What bounds it is the chain of dependent steps of each launch, and in the tiles the counts: an LDS
// atomic that returns a value serves about one lane a clock.
//
// The sort in LDS is one count, not a merge or a radix pass (split_sort.h): a pair's place in the range of its stretch gives its bin (four times as many
// bins as pairs, their counts one byte each), the bins' counts its group, and the few pairs of a group are compared with each other.  Only where a group
// is beyond 16 pairs (keys far from evenly spread inside the stretch, many equal ones) is everything counted again.
//
// Measured (MI355X, us, this sort / runs merged in LDS up to 2^19 and radix passes with a decay pass beyond, which it replaced; uniform
// keys): 9000 positions 20 / 22, 2^17: 25 / 27, 4 10^5: 32 / 50, 2^19 + 1: 33 / 65, 2^20 + 1024: 40 / 81, 2^21: 56 / 105, 3 2^20: 79 / 131,
// 4 10^6: 105 / 145.  Bins four to a word, the anchor itself as the place where the range is wide, no bank conflicts in the search among the bounds (before: two bins to a
// pair, a 64-bit place of key and id): the last kernel 38 -> 32 us at 2^21 positions, the tiles 16 -> 13; 2^19 x 2^19 with normal anchors, batch 8, forward +
// backward 215 -> 209, the weighted Gram matrix of 1024 over 2^20 69.1 -> 67.6.  Near zero the stretches of a grid are counted by the multiple and the id instead of once
// more (a product with batch 1, 32 equal anchors to a value: 20000 positions 42.0 -> 40.0, 65537: 45.0 -> 40.2, 200000: 53.5 -> 46.4, 2^21: 124 -> 116).
#include "split_sort.h"

namespace laplex {

namespace {

struct SplitArgs {
    const float* a; const float* b; int64_t k; float tau; int N;
    uint2* pairs;                   // N (key, id) pairs, tile by tile
    uint2* spare;                   // N more, for stretches beyond a workgroup's capacity
    unsigned long long* bounds;     // [buckets] (key, id) of the first pair of a stretch; the first stretch has none
    unsigned long long* edges;      // [2][buckets + 1] the keys on either side of a bound, once they are known
    uint16_t* starts;               // [tiles][buckets + 1]
    uint32_t* sampled;              // [samples] keys
    uint32_t* ids; float* dh; float* pk; float2* pk8; uint32_t* counters;     // the plan
    int tiles, buckets, samples, per_bound, id_bits;
    int64_t op_a, op_b, op_ws;      // strides from one operator to the next (elements; bytes of workspace)
};

template <typename T>
__device__ __forceinline__ T* op_shift(T* p, int64_t bytes) { return reinterpret_cast<T*>(reinterpret_cast<char*>(p) + bytes); }

__device__ __forceinline__ uint32_t split_anchor(const SplitArgs& A, int64_t op, int64_t pos)
{
    return split_key(A.tau * (pos < A.k ? A.a[op * A.op_a + pos] : A.b[op * A.op_b + pos - A.k]));
}

// One sample per stretch of N / samples positions, at a place inside it that a hash picks: no period of the input coincides with them.
// (Its multipliers are Knuth's, The Art of Computer Programming 6.4, and one of the 32-bit mixers that C. Wellons' hash prospector lists.)
__device__ __forceinline__ int sample_position(int i, int N, int samples)
{
    const int width = N / samples;
    uint32_t h = (uint32_t)i * 2654435761u + 40503u;
    h ^= h >> 15; h *= 0x2C1B3C6Du; h ^= h >> 13;
    return i * width + (int)__umulhi(h, (uint32_t)width);
}

__global__ void __launch_bounds__(256)
k_split_sample(const SplitArgs A)
{
    const int64_t op = blockIdx.y;
    const int i = blockIdx.x * 256 + threadIdx.x;
    if (i < A.samples) op_shift(A.sampled, op * A.op_ws)[i] = split_anchor(A, op, sample_position(i, A.N, A.samples));
}

constexpr int kPickThreads = 1024, kPickQueries = 16;

// Rank of a sample = samples with a smaller key + those with an equal key and a smaller index (indexes ascend with positions).
// Every workgroup holds all samples in registers, 64 to a word, and ranks 16 of them: words before the queries' own count with <=,
// words behind with <; one comparison and one population count of the lane mask per query and word.
// GATHERED: the samples are in memory already, side by side; otherwise every workgroup fetches them from among the anchors.
template <int PER, bool GATHERED>      // PER: words per wavefront, at most
__global__ void __launch_bounds__(kPickThreads)
k_split_pick(const SplitArgs A)
{
    constexpr int WAVES = kPickThreads / 64;
    __shared__ uint32_t counts[kPickQueries], query_keys[kPickQueries];
    const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
    const int64_t op = blockIdx.y;
    unsigned long long* const bounds = op_shift(A.bounds, op * A.op_ws);
    if (blockIdx.x == 0)
        for (int i = tid; i < 2 * (A.buckets + 1); i += kPickThreads) op_shift(A.edges, op * A.op_ws)[i] = 0ull;
    const int q0 = (int)blockIdx.x * kPickQueries, own = q0 >> 6, own_lane = q0 & 63;
    uint32_t key[PER];
#pragma unroll
    for (int r = 0; r < PER; ++r) {
        const int i = r * kPickThreads + tid;
        key[r] = 0xFFFFFFFFu;                       // behind every sample: never counted
        if (i < A.samples) {
            if (GATHERED) key[r] = op_shift(A.sampled, op * A.op_ws)[i];
            else key[r] = split_anchor(A, op, sample_position(i, A.N, A.samples));
        }
    }
    if (tid < kPickQueries) counts[tid] = 0u;
#pragma unroll
    for (int r = 0; r < PER; ++r)
        if (r * WAVES + wave == own && lane >= own_lane && lane < own_lane + kPickQueries) query_keys[lane - own_lane] = key[r];
    __syncthreads();
    const uint32_t queries = query_keys[lane & (kPickQueries - 1)];
    uint32_t query[kPickQueries], count[kPickQueries];
#pragma unroll
    for (int q = 0; q < kPickQueries; ++q) { query[q] = (uint32_t)__builtin_amdgcn_readlane((int)queries, q); count[q] = 0u; }
#pragma unroll
    for (int r = 0; r < PER; ++r) {
        const int word = r * WAVES + wave;          // uniform
        if (word < own) {
#pragma unroll
            for (int q = 0; q < kPickQueries; ++q) count[q] += (uint32_t)__popcll(__ballot(key[r] <= query[q]));
        } else if (word > own) {
            if (word * 64 < A.samples) {
#pragma unroll
                for (int q = 0; q < kPickQueries; ++q) count[q] += (uint32_t)__popcll(__ballot(key[r] < query[q]));
            }
        } else {
#pragma unroll
            for (int q = 0; q < kPickQueries; ++q)
                count[q] += (uint32_t)__popcll(__ballot(key[r] < query[q] || (key[r] == query[q] && lane < own_lane + q)));
        }
    }
    uint32_t sum = 0u;
#pragma unroll
    for (int q = 0; q < kPickQueries; ++q) sum = lane == q ? count[q] : sum;
    if (lane < kPickQueries) atomicAdd(&counts[lane], sum);
    __syncthreads();
    if (tid < kPickQueries && q0 + tid < A.samples) {
        const uint32_t rank = counts[tid];
        if (rank % (uint32_t)A.per_bound == 0u)
            bounds[rank / (uint32_t)A.per_bound] = ((unsigned long long)queries << 32) | (uint32_t)sample_position(q0 + tid, A.N, A.samples);
    }
}

constexpr int64_t kSplitWholeMax = kSmallMax;      // positions that one workgroup sorts in one launch


template <int THREADS, int PER>
__global__ void __launch_bounds__(THREADS)
k_split_tiles(const SplitArgs A)
{
    constexpr int TILE = THREADS * PER, BUCKETS_PER = kSplitMaxBuckets / THREADS > 0 ? kSplitMaxBuckets / THREADS : 1;
    __shared__ uint32_t bound_key[kBoundWords], bound_id[kSplitMaxBuckets];
    __shared__ uint32_t hist[kSplitMaxBuckets];
    __shared__ uint16_t same[kSplitMaxBuckets];             // bounds with this one's key, from it on
    __shared__ uint2 laid[TILE];
    __shared__ uint32_t part[THREADS / 64];
    const int tid = threadIdx.x, buckets = A.buckets;
    const int64_t op = blockIdx.y, base = (int64_t)blockIdx.x * TILE;
    const int len = A.N - base < TILE ? (int)(A.N - base) : TILE;
    uint32_t key[PER];
#pragma unroll
    for (int i = 0; i < PER; ++i) {
        const int q = i * THREADS + tid;
        key[i] = split_anchor(A, op, base + (q < len ? q : len - 1));
    }
    for (int i = tid; i < kSplitMaxBuckets; i += THREADS) hist[i] = 0u;
    const StretchBounds<THREADS> bound(op_shift(A.bounds, op * A.op_ws), buckets, 1, bound_key, bound_id, same);
    uint32_t at[PER];               // stretch in the upper half, place among the tile's pairs of the stretch in the lower half
    bound.find(key, at, [&](int i) { return (uint32_t)(base + i * THREADS + tid); });
#pragma unroll
    for (int i = 0; i < PER; ++i)
        if (i * THREADS + tid < len) at[i] = (at[i] << 16) | atomicAdd(&hist[at[i]], 1u);
    __syncthreads();
    uint32_t c[BUCKETS_PER], mine = 0u, total;
#pragma unroll
    for (int q = 0; q < BUCKETS_PER; ++q) { c[q] = tid * BUCKETS_PER + q < kSplitMaxBuckets ? hist[tid * BUCKETS_PER + q] : 0u; mine += c[q]; }
    uint32_t sum = block_scan<THREADS>(mine, part, &total);
    uint16_t* const starts = op_shift(A.starts, op * A.op_ws) + (int64_t)blockIdx.x * (buckets + 1);
#pragma unroll
    for (int q = 0; q < BUCKETS_PER; ++q) {
        const int g = tid * BUCKETS_PER + q;
        if (g < kSplitMaxBuckets) hist[g] = sum;
        if (g < buckets) starts[g] = (uint16_t)sum;
        sum += c[q];
    }
    if (tid == 0) starts[buckets] = (uint16_t)len;
    __syncthreads();
#pragma unroll
    for (int i = 0; i < PER; ++i)
        if (i * THREADS + tid < len) laid[hist[at[i] >> 16] + (at[i] & 0xFFFFu)] = make_uint2(key[i], (uint32_t)(base + i * THREADS + tid));
    __syncthreads();
    uint2* const out = op_shift(A.pairs, op * A.op_ws) + base;
#pragma unroll
    for (int i = 0; i < PER; ++i)
        if (i * THREADS + tid < len) out[i * THREADS + tid] = laid[i * THREADS + tid];
}

// WHOLE: the anchors are one stretch, and are read where they are (buckets = 1, no tiles).
template <int THREADS, int ITEMS, bool WHOLE>
__global__ void __launch_bounds__(THREADS, 4)
k_split_sort(const SplitArgs A, int tile_size, int group_bits)
{
    constexpr int CAP = THREADS * ITEMS, WAVES = THREADS / 64, MAX_TILES = THREADS < 512 ? THREADS : 512;
    __shared__ __align__(16) uint32_t buf[2 * CAP];        // counts of bins, then the pairs
    __shared__ uint32_t offset[MAX_TILES + 2];             // pairs of the stretch in the tiles before
    __shared__ uint32_t place[MAX_TILES + 1];                  // pair e of the stretch lies at place[tile] + e
    __shared__ uint32_t part[WAVES], s_long;
    __shared__ StretchShared<THREADS> S;
    const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
    const int64_t op = blockIdx.y;
    const uint2* const pairs = op_shift(A.pairs, op * A.op_ws);
    const uint16_t* const starts = op_shift(A.starts, op * A.op_ws);
    uint32_t* const ids = op_shift(A.ids, op * A.op_ws);
    float* const dh = op_shift(A.dh, op * A.op_ws);
    float* const pk = op_shift(A.pk, op * A.op_ws);
    float2* const pk8 = A.pk8 ? op_shift(A.pk8, op * A.op_ws) : nullptr;
    const int g = blockIdx.x, tiles = A.tiles, N = A.N;

    if (g == 0 && tid < 64) op_shift(A.counters, op * A.op_ws)[tid] = 0u;        // list lengths of the scans; the plan is valid
    if (tid == 0) { S.init(); s_long = 0u; }
    // where the stretch lies in every tile, and where in the sorted sequence
    constexpr int LOADS = 4;
    int cnt = A.N, base = 0;
    if (!WHOLE) {
        uint32_t lo = 0u, n = 0u;
        if (tid < tiles) {
            const uint16_t* const row = starts + (int64_t)tid * (A.buckets + 1) + g;
            lo = row[0];
            n = row[1] - lo;
        }
        const uint32_t inc_n = wave_scan(n), inc_lo = wave_scan(lo);
        if (lane == 63) { part[wave] = inc_n; S.sums[wave] = inc_lo; }
        __syncthreads();
        uint32_t before = 0u, all_n = 0u, all_lo = 0u;
#pragma unroll
        for (int w = 0; w < WAVES; ++w) { before += w < wave ? part[w] : 0u; all_n += part[w]; all_lo += S.sums[w]; }
        const uint32_t ex = before + inc_n - n;
        if (tid < tiles) { offset[tid] = ex; place[tid] = (uint32_t)(tid * tile_size) + lo - ex; }
        if (tid == 0) { offset[tiles] = offset[tiles + 1] = all_n; place[tiles] = 0u; }
        cnt = (int)all_n;
        base = (int)all_lo;
        if (__any(n > (uint32_t)(2 * LOADS << group_bits)) && lane == 0) s_long = 1u;
    }
    __syncthreads();
    auto tile_of = [&](int e) {             // of pair e of the stretch
        int t = 0;
        for (int step = MAX_TILES / 2; step > 0; step >>= 1) t += (t + step < tiles && offset[t + step] <= (uint32_t)e) ? step : 0;
        return t;
    };
    auto write = [&](int j, uint32_t key, uint32_t before, uint32_t id, bool has_before) {
        const float p = split_key_to_float(key);
        ids[j] = id;
        pk[j + 1] = p;
        if (has_before) dh[j] = key == before ? -1.0f : expf(-(p - split_key_to_float(before)));
        if (pk8) {                                  // pk8[m] = (pk[8m], pk[8m + 1])
            if ((j & 7) == 7) pk8[(j + 1) >> 3].x = p;
            if ((j & 7) == 0) pk8[j >> 3].y = p;
        }
    };
    // The decay across a bound needs the keys on both sides of it: either side leaves its own and looks for the other's at the end, and
    // whoever comes second (both, if they meet) writes it.  Every stretch holds a pair: its bound, or for the first one the smallest sample.
    unsigned long long* const left_of = op_shift(A.edges, op * A.op_ws);            // [g]: the last key before stretch g
    unsigned long long* const right_of = left_of + A.buckets + 1;                   // [g]: the first key of stretch g
    constexpr unsigned long long known = 1ull << 32;
    uint32_t first_key = 0u, last_key = 0u;         // these four: thread 0
    unsigned long long seen_left = 0ull, seen_right = 0ull;
    auto publish = [&](uint32_t first, uint32_t last) {
        first_key = first; last_key = last;
        if (g > 0) seen_left = __hip_atomic_exchange(right_of + g, known | first, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        if (g + 1 < A.buckets) seen_right = __hip_atomic_exchange(left_of + g + 1, known | last, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    };
    unsigned long long key_left = 0ull, key_right = 0ull;
    auto look = [&]() {
        asm volatile("" :: "v"(seen_left), "v"(seen_right) : "memory");       // the exchanges have been performed
        if (g > 0) key_left = __hip_atomic_load(left_of + g, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        if (g + 1 < A.buckets) key_right = __hip_atomic_load(right_of + g + 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    };
    if (WHOLE || cnt <= CAP) {                      // uniform
        // 2^group_bits lanes take the run of a tile, up to four pairs each at once and three runs at a time, into LDS; then every thread its
        // own pairs
        unsigned long long* const slot = reinterpret_cast<unsigned long long*>(buf);
        if (!WHOLE) {
            constexpr int RUNS = 3;
            const int lanes = 1 << group_bits, sub = tid & (lanes - 1), per = THREADS >> group_bits;
            for (int t0 = tid >> group_bits; t0 < tiles; t0 += RUNS * per) {
                uint32_t first[RUNS], end[RUNS], at[RUNS];
                unsigned long long v[RUNS][LOADS];
#pragma unroll
                for (int u = 0; u < RUNS; ++u) {
                    const int t = t0 + u * per < tiles ? t0 + u * per : tiles;
                    first[u] = offset[t] + sub; end[u] = offset[t + 1]; at[u] = place[t];
                }
#pragma unroll
                for (int u = 0; u < RUNS; ++u)
#pragma unroll
                    for (int q = 0; q < LOADS; ++q) {
                        const uint32_t e = first[u] + q * lanes;
                        v[u][q] = *reinterpret_cast<const unsigned long long*>(pairs + (e < end[u] ? at[u] + e : 0u));
                    }
#pragma unroll
                for (int u = 0; u < RUNS; ++u) {
#pragma unroll
                    for (int q = 0; q < LOADS; ++q)
                        if (first[u] + q * lanes < end[u]) slot[first[u] + q * lanes] = v[u][q] << 32 | v[u][q] >> 32;       // key above id
                    const uint32_t stop = first[u] + 2 * LOADS * lanes < end[u] ? first[u] + 2 * LOADS * lanes : end[u];
                    for (uint32_t e = first[u] + LOADS * lanes; e < stop; e += lanes) {
                        const uint2 w = pairs[at[u] + e];
                        slot[e] = ((unsigned long long)w.x << 32) | w.y;
                    }
                }
            }
            if (s_long) {       // uniform.  Input that is in order in places: what goes beyond that in long runs, spread over all threads
                for (int e = tid; e < cnt; e += THREADS) {
                    const int t = tile_of(e);
                    if (e - offset[t] < (uint32_t)(2 * LOADS * lanes)) continue;
                    const uint2 w = pairs[place[t] + (uint32_t)e];
                    slot[e] = ((unsigned long long)w.x << 32) | w.y;
                }
            }
        }
        __syncthreads();
        uint32_t key[ITEMS], id[ITEMS];
        uint32_t rank[ITEMS];
        stretch_ranks<THREADS, ITEMS>(key, id, cnt, WHOLE ? split_anchor(A, op, 0) : (uint32_t)(slot[0] >> 32), A.id_bits, buf, S, rank, [&](int e, uint32_t& key_e, uint32_t& id_e) {
            if (WHOLE) {
                key_e = split_anchor(A, op, e); id_e = (uint32_t)e;
            } else {
                const unsigned long long v = slot[e];
                key_e = (uint32_t)(v >> 32); id_e = (uint32_t)v;
            }
        }, publish);
        __syncthreads();
#pragma unroll
        for (int i = 0; i < ITEMS; ++i)
            if (i * THREADS + tid < cnt) slot[rank[i]] = ((unsigned long long)key[i] << 32) | id[i];
        if (tid == 0) look();
        __syncthreads();
#pragma unroll
        for (int i = 0; i < ITEMS; ++i) {
            const int e = i * THREADS + tid;
            if (e < cnt) {
                const unsigned long long v = slot[e];
                write(base + e, (uint32_t)(v >> 32), e > 0 ? (uint32_t)(slot[e - 1] >> 32) : 0u, (uint32_t)v, e > 0);
            }
        }
    } else {
        uint2* const spare = op_shift(A.spare, op * A.op_ws) + base;
        uint32_t k_and = 0xFFFFFFFFu, k_or = 0u, k_min = 0xFFFFFFFFu, k_max = 0u, i_min = 0xFFFFFFFFu, i_max = 0u;
        for (int e = tid; e < cnt; e += THREADS) {
            const int t = tile_of(e);
            const uint2 v = pairs[place[t] + (uint32_t)e];
            spare[e] = v;
            k_and &= v.x; k_or |= v.x;
            k_min = v.x < k_min ? v.x : k_min; k_max = v.x > k_max ? v.x : k_max;
            i_min = v.y < i_min ? v.y : i_min; i_max = v.y > i_max ? v.y : i_max;
        }
        atomicAnd(&S.key_and, k_and); atomicOr(&S.key_or, k_or); atomicMin(&S.key_min, k_min); atomicMax(&S.key_max, k_max);
        atomicMin(&S.id_min, i_min); atomicMax(&S.id_max, i_max);
        __threadfence_block();
        __syncthreads();
        const uint32_t vary = S.key_or & ~S.key_and;
        if (!count_in_memory<THREADS, CAP>(spare, ids + base, pk + base + 1, cnt, StretchRange(S.key_min, S.key_max, S.id_min, S.id_max, vary), buf, part)) {
            const uint32_t id_span = S.id_max - S.id_min;      // the low digits of the ids up to where the smallest and the largest differ
            sort_in_memory<THREADS>(spare, ids + base, pk + base + 1, cnt, vary, id_span ? 0xFFFFFFFFu >> __clz((int)(S.id_min ^ S.id_max)) : 0u, buf);
        }
        for (int e = tid; e < cnt; e += THREADS) {
            const uint2 v = spare[e];
            write(base + e, v.x, e > 0 ? spare[e - 1].x : 0u, v.y, e > 0);
        }
        if (tid == 0) { publish(spare[0].x, spare[cnt - 1].x); look(); }
    }
    if (tid == 0) {
        auto decay = [&](int j, uint32_t before, uint32_t key) {
            dh[j] = key == before ? -1.0f : expf(-(split_key_to_float(key) - split_key_to_float(before)));
        };
        if (key_left & known) decay(base, (uint32_t)key_left, first_key);
        if (key_right & known) decay(base + cnt, last_key, (uint32_t)key_right);
        if (g == 0) {
            dh[0] = 0.0f;
            pk[0] = __uint_as_float(0xFF800000u);
            if (pk8) pk8[0].x = __uint_as_float(0xFF800000u);
        }
        if (g == A.buckets - 1) {
            const float inf = __uint_as_float(0x7F800000u);
            dh[N] = 0.0f;
            pk[N + 1] = inf;
            if (pk8) {
                if ((N & 7) == 7) pk8[(N + 1) >> 3] = make_float2(inf, inf);
                if ((N & 7) == 0) pk8[N >> 3].y = inf;
            }
        }
    }
}

}  // namespace

namespace {
// Tiles and stretches by the number of positions.  A stretch takes one workgroup a fixed 8 us of dependent steps and little more with its
// length, so from 2^19 positions on there are as few of them as the capacity (1024 x 16 pairs) allows, in whole rounds of the 256
// compute units (us for the whole sort; 2^20 + 1024 positions: 256 stretches 41, 512 of half the length, two to a compute unit, 49;
// 2^21: 256 of 8192 pairs 59, 512 of 4096 67).  The samples keep a stretch inside the capacity: with s samples per stretch, of which it
// would have to hold fewer than s where its length calls for s * capacity / average, the chance of one beyond it is, for a whole sort, 2e-4
// at 256 * 6144 positions, 9e-4 at 2^21, 5e-4 at 512 * 6144, 8e-4 at 2^22, and falls to below 1e-5 at five sixths of these sizes (18 or 19
// pairs a thread, a longer LDS buffer, would bring it to 1e-5, and cost 5 to 10 % in spilled registers).  Such a set of anchors is sorted
// in memory there (count_in_memory: 58 us more at 2^21).  Tiles: the fewest keys that still make at most 512 of them.
// Up to 2^17 positions, where stretches are far fewer than the device has room for, they are short and taken by more threads than they need, and
// half the samples do, since the capacity is four and more times the average (us for the whole sort, 1024 pairs by 256 threads, 16 samples
// each / now: 20000 21.0 / 19.7; 65536 22.2 / 20.8; 131072 24.3 / 22.7).  Beyond, half the samples leave
// longer longest stretches, which is what the sort waits for (2^19: 33 / 39; 2^20: 39 / 44).
struct SplitGeom { int per, threads, group_bits; int64_t tile, tiles, buckets, samples; };
constexpr int kTileThreads = 1024;
SplitGeom split_geom(int64_t N, bool many = false)      // many: several operators in one launch, which fill the device between them
{
    SplitGeom G;
    int64_t per_bound = 16;
    if (many && N <= int64_t(1) << 17) {
        G.per = 1; G.threads = 256; G.buckets = (N + 1023) / 1024;
    } else if (N <= int64_t(1) << 16) {
        G.per = 1; G.threads = 256; G.buckets = (N + 511) / 512; per_bound = 8;
    } else if (N <= int64_t(1) << 17) {
        G.per = 1; G.threads = 512; G.buckets = (N + 1023) / 1024; per_bound = 8;
    } else if (N <= int64_t(1) << 19) {
        G.per = 2; G.threads = 512; G.buckets = (N + 2047) / 2048;
    } else {
        G.per = N <= int64_t(1) << 20 ? 2 : N <= int64_t(1) << 21 ? 4 : 8;
        G.threads = 1024;
        G.buckets = N <= int64_t(1) << 21 ? 256 : N <= 512 * 6144 ? 512 : 768;
        per_bound = N <= 256 * 6144 ? 16 : N <= int64_t(1) << 21 ? 32 : N <= 512 * 6144 ? 16 : 12;
    }
    G.tile = (int64_t)kTileThreads * G.per;
    G.tiles = (N + G.tile - 1) / G.tile;
    G.samples = G.buckets * per_bound;
    G.group_bits = 0;
    while (G.group_bits < 6 && (G.tile >> G.group_bits) > 2 * G.buckets) ++G.group_bits;      // (four times as many pairs as lanes: twice the average run)
    return G;
}
size_t split_words(const SplitGeom& G) { return (size_t)(2 * G.buckets + 4 * (G.buckets + 1) + G.samples + (G.tiles * (G.buckets + 1) + 1) / 2); }
}  // namespace

size_t split_sort_words(int64_t N)          // (for one operator or for each of many, whichever takes more: from 2^16 to 2^17 positions many take twice the samples)
{
    const size_t one = split_words(split_geom(N)), many = split_words(split_geom(N, true));
    return one > many ? one : many;
}

hipError_t launch_split_sort(const float* a, int64_t k, const float* b, int64_t n, float tau, uint2* pair0, uint2* pair1, uint32_t* scratch,
                             uint32_t* ids, float* dh, float* pk, float2* pk8, uint32_t* counters,
                             int64_t operators, int64_t op_a, int64_t op_b, int64_t op_ws, hipStream_t st)
{
    const SplitGeom G = split_geom(k + n, operators > 1);
    if (split_words(G) > split_sort_words(k + n)) return hipErrorInvalidValue;      // (what `scratch` holds)
    SplitArgs A{};
    A.a = a; A.b = b; A.k = k; A.tau = tau; A.N = (int)(k + n);
    A.pairs = pair0; A.spare = pair1;
    A.bounds = reinterpret_cast<unsigned long long*>(scratch);
    A.edges = A.bounds + G.buckets;
    A.sampled = reinterpret_cast<uint32_t*>(A.edges + 2 * (G.buckets + 1));
    A.starts = reinterpret_cast<uint16_t*>(A.sampled + G.samples);
    A.ids = ids; A.dh = dh; A.pk = pk; A.pk8 = pk8; A.counters = counters;
    A.tiles = (int)G.tiles; A.buckets = (int)G.buckets; A.samples = (int)G.samples; A.per_bound = (int)(G.samples / G.buckets);
    A.id_bits = 1; while ((int64_t(1) << A.id_bits) < k + n) ++A.id_bits;
    A.op_a = op_a; A.op_b = op_b; A.op_ws = op_ws;
    const unsigned ops = (unsigned)operators;
    if (k + n <= kSplitWholeMax) {
        A.tiles = 0; A.buckets = 1;
        LAPLEX_TIMED("split_sort", st, hipLaunchKernelGGL((k_split_sort<1024, 8, true>), dim3(1, ops), dim3(1024), 0, st, A, 0, 0));
        return hipGetLastError();
    }
    const dim3 pick((unsigned)((G.samples + kPickQueries - 1) / kPickQueries), ops);
    auto go = [&](auto kernel) { LAPLEX_TIMED("split_pick", st, hipLaunchKernelGGL(kernel, pick, dim3(kPickThreads), 0, st, A)); };
    // up to 2048 samples every workgroup fetches them for itself (2^18 positions: 28 us, 30 with a launch of their own); beyond, the
    // workgroups' fetches from all over the anchors would take longer than the launch (2^20: 18 us for the ranks alone, 6)
    if (G.samples <= 2 * kPickThreads) {
        go(k_split_pick<2, false>);
    } else {
        LAPLEX_TIMED("split_sample", st, hipLaunchKernelGGL(k_split_sample, dim3((unsigned)((G.samples + 255) / 256), ops), dim3(256), 0, st, A));
        if (G.samples <= 4 * kPickThreads) go(k_split_pick<4, true>);
        else if (G.samples <= 8 * kPickThreads) go(k_split_pick<8, true>);
        else go(k_split_pick<9, true>);
    }
    const dim3 tiles((unsigned)G.tiles, ops), buckets((unsigned)G.buckets, ops);
    auto distribute = [&](auto kernel) { LAPLEX_TIMED("split_tiles", st, hipLaunchKernelGGL(kernel, tiles, dim3(kTileThreads), 0, st, A)); };
    if (G.per == 1) distribute(k_split_tiles<kTileThreads, 1>);
    else if (G.per == 2) distribute(k_split_tiles<kTileThreads, 2>);
    else if (G.per == 4) distribute(k_split_tiles<kTileThreads, 4>);
    else distribute(k_split_tiles<kTileThreads, 8>);
    auto sort = [&](auto kernel) { LAPLEX_TIMED("split_sort", st, hipLaunchKernelGGL(kernel, buckets, dim3(G.threads), 0, st, A, (int)G.tile, G.group_bits)); };
    if (G.threads == 256) sort(k_split_sort<256, 16, false>);
    else if (G.threads == 512) sort(k_split_sort<512, 16, false>);
    else sort(k_split_sort<1024, 16, false>);
    return hipGetLastError();
}

}  // namespace laplex

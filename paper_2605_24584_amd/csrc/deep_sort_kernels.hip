// Sorting many anchors for batch 1 (Sec. 3 "Complexity": the O(n log n) term) by samples, in two distributions and one sort in LDS, and
// moving values of the caller's order into the sorted order along the very same way (the gather of S4).
//
//   samples         one anchor per 128 (fewer beyond 2^29 positions), sorted by launch_split_sort; every samples_per-th is the first pair of a
//                   stretch of the sorted sequence, and the first of per_bucket stretches the first of a bucket
//   k_deep_tiles    (k_deep_distribute<false>) a tile of 16384 (8192, see deep_geom) consecutive positions is laid out bucket by bucket, in the tile's own place
//   k_deep_col_*, k_deep_bases    where every tile's run of a bucket lies in that bucket (prefix sums over the tiles)
//   k_deep_pieces   (k_deep_distribute<true>) a piece of as many consecutive pairs of a bucket is gathered from the tiles' runs and laid out
//                   stretch by stretch, in the piece's own place
//   k_deep_units    consecutive stretches that fit a workgroup's LDS together
//   k_deep_sort     a unit is gathered from its bucket's pieces, sorted in LDS and written to the plan: ids, anchors, decays
//   k_deep_edges    the decays across the units' ends, the sentinels, the plan's counter words
//
// Every pass reads runs and writes whole stretches of memory, nothing is reserved and nothing is waited for across workgroups.  Each pass
// also leaves 2 bytes per position of how it laid its pairs out: from1 (tile layout: index inside the tile in the caller's order), slot2 (place
// inside the piece's layout, by place in the bucket) and slot3 (place inside the unit, by place among the pairs as gathered).  With these a value
// per position follows the pairs without keys, ids or destinations (launch_deep_move), and the inverse permutation is never formed.  Pairs
// are compared as (key, id), bounds included, so the order is the stable sort's bit for bit and the length of a stretch depends on the
// samples' places alone.
//
// Why two distributions: runs of 64 and more pairs on either side, buckets and stretches that LDS holds (at most 1024 bounds), and units of 4096
// pairs.  The numbers of buckets and stretches make the tiles' runs and the units' about equally long.  Stretches are cut fine (768 pairs on
// average, six samples each) and put together again by their counts: a workgroup's LDS is filled to nine tenths, where stretches of samples alone
// would have to leave most of it free.
//
// What bounds it: memory traffic in the tiles (10 bytes a pair, 3.8 TB/s), latency elsewhere: a workgroup passes eight to twelve barriers with
// loads and LDS atomics in between, two or three workgroups a compute unit (16 bytes a pair in the pieces, 3.6 TB/s, 23 in the sort, 3.2).
//
// Measured (MI355X, us, before / now; before: four radix passes with chained look-back, histogram, a decay pass, the inverse permutation by
// partition passes of (id, position), and values in as (rank, value) records): the plan of 2^28 positions 7720 / 4080, a move of 2^27 values into their
// order 1350 / 1050; forward + backward at 2^27 x 2^27 17115 / 12776, 2^24 x 2^24 with 32 equal anchors a value 2451 / 1829, 2^22 x 2^22 574 /
// 515.  Anchors that are promised to arrive in order are merged, not sorted (move_in_order, below).  The workspace is 26 % smaller.  What was tried and did not pay: units of stretches with three times the
// pairs (LDS for the longest, a third filled): 5090 us for the sort of 2^28 pairs in place of 1893; 1024 threads of 4 pairs 2254, 256 of 16 2092.
#include "split_sort.h"

#include <string>

namespace laplex {

namespace {

constexpr int kDeepThreads = 1024;        // of a tile or piece: 8 or 16 positions each (PER)
constexpr int kDeepChunk = 64;            // tiles whose runs are added up together
constexpr int kDeepManyPieces = 8191;     // (what a unit's record has room for)

struct DeepArgs {
    const float* a; const float* b; int64_t k; float tau; int64_t N;
    DeepPlan P;
    int buckets, per_bucket, samples_per; int64_t tiles, chunks, samples, stretches; uint64_t sample_step; int id_bits;
    // scratch
    float* sampled; const uint32_t* sample_ids; const float* sample_pk;
    unsigned long long* bounds;      // [stretches] (key, id) of the first pair of a stretch
    uint32_t* keys1;                 // [N] tile layout
    uint16_t* starts1;               // [tiles][buckets + 1]
    uint32_t* chunk_sums;            // [chunks][buckets]
    uint2* pairs2;                   // [N] (key, id), piece layout
    uint2* spare;                    // [N] for stretches beyond a workgroup's capacity
    // the plan
    uint32_t* ids; float* dh; float* pk; float2* pk8; uint32_t* counters;
};

__device__ __forceinline__ float deep_anchor(const DeepArgs& A, int64_t pos) { return A.tau * (pos < A.k ? A.a[pos] : A.b[pos - A.k]); }

// One sample per 1 / samples of the positions, at a place inside it that a hash picks (split_sort_kernels.hip; step: the positions per
// sample in units of 2^-20, so that the samples cover the positions to the last).
__device__ __forceinline__ int64_t deep_sample_position(int64_t i, uint64_t step)
{
    const int64_t from = (int64_t)(((uint64_t)i * step) >> 20), to = (int64_t)((((uint64_t)i + 1u) * step) >> 20);
    uint32_t h = (uint32_t)i * 2654435761u + 40503u;
    h ^= h >> 15; h *= 0x2C1B3C6Du; h ^= h >> 13;
    return from + (int64_t)__umulhi(h, (uint32_t)(to - from));
}

__global__ void __launch_bounds__(256)
k_deep_sample(const DeepArgs A)
{
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (i < A.samples) A.sampled[i] = deep_anchor(A, deep_sample_position(i, A.sample_step));
}

__global__ void __launch_bounds__(256)
k_deep_bounds(const DeepArgs A)
{
    const int64_t s = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (s >= A.stretches) return;
    const int64_t i = s * A.samples_per;
    A.bounds[s] = ((unsigned long long)split_key(A.sample_pk[i + 1]) << 32) | (uint32_t)deep_sample_position(A.sample_ids[i], A.sample_step);
}

// Which of `runs` a place belongs to when each begins at the place of a set bit: mask words, bits set in the words before.
__device__ __forceinline__ uint32_t run_of(const uint32_t* mask, const uint32_t* before, uint32_t e)
{
    return before[e >> 5] + (uint32_t)__popc(mask[e >> 5] & (0xFFFFFFFFu >> (31u - (e & 31u)))) - 1u;
}

// LDS of a distribution.  lay: the layout buffer; before the pairs are laid out it holds the runs of a gathered piece.
template <int PER>
struct DeepShared {
    __align__(16) uint32_t lay[kDeepThreads * PER];
    uint32_t bound_key[kBoundWords], bound_id[kSplitMaxBuckets];
    uint32_t hist[kSplitMaxBuckets + 1];       // (before the counts: mask and words of the runs)
    uint16_t same[kSplitMaxBuckets];
    uint32_t part[kDeepThreads / 64];
};
static_assert(sizeof(DeepShared<16>) <= 80 * 1024, "two workgroups to a compute unit");
static_assert(2 * (kDeepThreads * 16 / 32) <= kSplitMaxBuckets, "mask and words fit where the counts go later");

// The piece a workgroup of k_deep_pieces or k_move_pieces takes, and its runs: place e of the piece lies at delta[run] + e of the tile layout.
struct DeepPiece { int bucket; uint32_t seq0; int len; uint32_t tile; };
__device__ __forceinline__ bool find_piece(const DeepPlan& P, int buckets, uint32_t piece, DeepPiece& out)
{
    const uint4 v = P.pieces[piece];            // (uniform, all three; beyond the last piece, or without tables, whatever lies there)
    const uint32_t all = P.piece_base[buckets];
    if (*P.unit_count == kDeepMerged || piece >= all) return false;
    out.tile = v.x; out.bucket = (int)v.y; out.seq0 = v.z; out.len = (int)v.w;
    return true;
}
// delta: a word for every pair of a piece, mask and before: a word for every 32, part: kDeepThreads / 64.  Ends with a barrier.
template <int PER>
__device__ __forceinline__ void piece_runs(const DeepPlan& P, int64_t tiles, const DeepPiece& p, uint32_t* delta, uint32_t* mask, uint32_t* before, uint32_t* part)
{
    constexpr int TILE = kDeepThreads * PER;
    const int tid = threadIdx.x;
    const uint32_t* const col = P.before + (int64_t)p.bucket * tiles;
    const uint16_t* const start = P.start1 + (int64_t)p.bucket * tiles;
    const uint32_t cnt = P.bucket_base[p.bucket + 1] - P.bucket_base[p.bucket], end = p.seq0 + (uint32_t)p.len;
    if (tid < TILE / 32) mask[tid] = 0u;
    __syncthreads();
    uint32_t runs = 0u;
    for (int64_t t0 = p.tile; t0 < tiles; t0 += kDeepThreads) {
        const int64_t t = t0 + tid;
        uint32_t ex = 0u, nx = 0u, st = 0u;
        if (t < tiles) { ex = col[t]; nx = t + 1 < tiles ? col[t + 1] : cnt; st = start[t]; }
        const uint32_t lo = ex > p.seq0 ? ex : p.seq0, hi = nx < end ? nx : end;
        const bool some = t < tiles && lo < hi;
        uint32_t total;
        const uint32_t at = runs + block_scan<kDeepThreads>(some ? 1u : 0u, part, &total);
        if (some) {
            delta[at] = (uint32_t)t * (uint32_t)TILE + st + p.seq0 - ex;
            atomicOr(&mask[(lo - p.seq0) >> 5], 1u << ((lo - p.seq0) & 31u));
        }
        runs += total;
        if (__syncthreads_or(t < tiles && nx >= end)) break;
    }
    const uint32_t bits = tid < TILE / 32 ? (uint32_t)__popc(mask[tid]) : 0u;
    uint32_t total;
    const uint32_t ex = block_scan<kDeepThreads>(bits, part, &total);
    if (tid < TILE / 32) before[tid] = ex;
    __syncthreads();
}

// A distribution: of the anchors of a tile to the buckets (PIECES = false), or of a piece of a bucket to the bucket's stretches.
template <bool PIECES, int PER>
__global__ void __launch_bounds__(kDeepThreads, 8)
k_deep_distribute(const DeepArgs A)
{
    constexpr int TILE = kDeepThreads * PER;
    __shared__ DeepShared<PER> S;
    const int tid = threadIdx.x;
    const int targets = PIECES ? A.per_bucket : A.buckets;
    DeepPiece p{0, 0u, TILE, 0u};
    int64_t out = (int64_t)blockIdx.x * TILE;           // first place of the layout
    uint32_t key[PER];
    if (PIECES) {
        if (!find_piece(A.P, A.buckets, blockIdx.x, p)) return;
        out = (int64_t)A.P.bucket_base[p.bucket] + p.seq0;
        piece_runs<PER>(A.P, A.tiles, p, S.lay, S.hist, S.hist + TILE / 32, S.part);
        // the ids wait in the layout buffer, each in a word that its own thread alone reads
        uint32_t id[PER];
#pragma unroll
        for (int i = 0; i < PER; ++i) {
            const uint32_t e = (uint32_t)(i * kDeepThreads + tid) < (uint32_t)p.len ? (uint32_t)(i * kDeepThreads + tid) : (uint32_t)p.len - 1u;
            const uint32_t src = S.lay[run_of(S.hist, S.hist + TILE / 32, e)] + e;
            key[i] = A.keys1[src];
            id[i] = (src & ~(uint32_t)(TILE - 1)) + A.P.from1[src];
            if (i % 4 == 3) __builtin_amdgcn_sched_barrier(0);        // (no more than four addresses at once: two workgroups to a compute unit leave 64 registers)
        }
        __syncthreads();
#pragma unroll
        for (int i = 0; i < PER; ++i) S.lay[i * kDeepThreads + tid] = id[i];
    } else {
        const int64_t left = A.N - out;
        p.len = left < TILE ? (int)left : TILE;
        const int last = p.len - 1;
        const int64_t of_a = A.k > out ? A.k - out : 0;         // the tile's first anchors are outputs'
        const float* const a = A.a + (of_a ? out : 0);
        const float* const b = A.b + (out - A.k);
#pragma unroll
        for (int i = 0; i < PER; ++i) {
            const int q = i * kDeepThreads + tid, c = q < last ? q : last;
            key[i] = split_key(A.tau * (c < of_a ? a : b)[c]);
        }
    }
    const int len = p.len;
    for (int i = tid; i < kSplitMaxBuckets + 1; i += kDeepThreads) S.hist[i] = 0u;
    uint32_t at[PER];          // target in the upper half, place among the tile's pairs of the target in the lower half; then the place in the layout
    {
        // (the bounds of the buckets lie per_bucket apart: the first of every bucket's stretches)
        const StretchBounds<kDeepThreads> bound(PIECES ? A.bounds + (int64_t)p.bucket * A.per_bucket : A.bounds, targets, PIECES ? 1 : A.per_bucket,
                                                S.bound_key, S.bound_id, S.same);
        if (PIECES) bound.find(key, at, [&](int i) { return S.lay[i * kDeepThreads + tid]; });
        else bound.find(key, at, [&](int i) { return (uint32_t)(out + i * kDeepThreads + tid); });
    }
    // (places beyond the last pair go behind all targets)
#pragma unroll
    for (int i = 0; i < PER; ++i) {
        at[i] = i * kDeepThreads + tid < len ? at[i] : (uint32_t)kSplitMaxBuckets;
        at[i] = (at[i] << 16) | atomicAdd(&S.hist[at[i]], 1u);
        asm volatile("" : "+v"(at[i]));         // (one register, not two)
    }
    __syncthreads();
    {
        const uint32_t c = tid < kSplitMaxBuckets ? S.hist[tid] : 0u;
        uint32_t total;
        const uint32_t ex = block_scan<kDeepThreads>(c, S.part, &total);
        uint16_t* const starts = (PIECES ? A.P.starts2 : A.starts1) + (int64_t)blockIdx.x * (targets + 1);
        S.hist[tid] = ex;
        if (tid < targets) starts[tid] = (uint16_t)ex;
        if (tid == 0) { starts[targets] = (uint16_t)len; S.hist[kSplitMaxBuckets] = (uint32_t)len; }
    }
    // (one uniform address per array and 32-bit offsets from it; the places are formed again rather than kept in registers)
    uint32_t me = (uint32_t)tid;
    asm volatile("" : "+v"(me));
    uint16_t* const slot2 = A.P.slot2 + out;
    uint2* const pairs2 = A.pairs2 + out;
    uint32_t* const keys1 = A.keys1 + out;
    uint16_t* const from1 = A.P.from1 + out;
    uint32_t other[PER];       // the other half of a pair: its id, or for a tile the index it came from
#pragma unroll
    for (int i = 0; i < PER; ++i) other[i] = PIECES ? S.lay[(uint32_t)(i * kDeepThreads) + me] : (uint32_t)(i * kDeepThreads) + me;
    __syncthreads();
#pragma unroll
    for (int i = 0; i < PER; ++i) {
        const uint32_t q = (uint32_t)(i * kDeepThreads) + me;
        at[i] = S.hist[at[i] >> 16] + (at[i] & 0xFFFFu);
        S.lay[at[i]] = key[i];
        if (PIECES && q < (uint32_t)len) slot2[q] = (uint16_t)at[i];
        if (PIECES && i % 4 == 3) __builtin_amdgcn_sched_barrier(0);
    }
    // (a piece's ids are there as well: two places to a register while the keys come back, and places formed again; with one each six registers went
    // to scratch, 24 bytes of memory traffic a lane: 2^28 pairs 1370 -> 1227 us, 2^25 183 -> 172)
#pragma unroll
    for (int i = 0; PIECES && i < PER; i += 2) {
        at[i] |= at[i + 1] << 16;
        asm volatile("" : "+v"(at[i]));
    }
    __syncthreads();
    if (PIECES) asm volatile("" : "+v"(me));
#pragma unroll
    for (int i = 0; i < PER; ++i) {
        const uint32_t q = (uint32_t)(i * kDeepThreads) + me;
        key[i] = S.lay[q];
        if (!PIECES && q < (uint32_t)len) keys1[q] = key[i];
    }
    __syncthreads();
#pragma unroll
    for (int i = 0; i < PER; ++i) S.lay[!PIECES ? at[i] : i % 2 ? at[i - 1] >> 16 : at[i] & 0xFFFFu] = other[i];
    __syncthreads();
    if (PIECES) asm volatile("" : "+v"(me));
#pragma unroll
    for (int i = 0; i < PER; ++i) {
        const uint32_t q = (uint32_t)(i * kDeepThreads) + me;
        if (q < (uint32_t)len) {
            if (PIECES) pairs2[q] = make_uint2(key[i], S.lay[q]);
            else from1[q] = (uint16_t)S.lay[q];
        }
    }
}

// Pairs of every bucket in a chunk of tiles.
__global__ void __launch_bounds__(kSplitMaxBuckets)
k_deep_col_sums(const DeepArgs A)
{
    const int b = threadIdx.x;
    if (b >= A.buckets) return;
    const int64_t t0 = (int64_t)blockIdx.x * kDeepChunk, t1 = t0 + kDeepChunk < A.tiles ? t0 + kDeepChunk : A.tiles;
    const uint16_t* row = A.starts1 + t0 * (A.buckets + 1) + b;
    uint32_t sum = 0u;
#pragma unroll 8
    for (int64_t t = t0; t < t1; ++t, row += A.buckets + 1) sum += (uint32_t)row[1] - row[0];
    A.chunk_sums[(int64_t)blockIdx.x * A.buckets + b] = sum;
}

// ... turned into the pairs of the bucket in earlier chunks; 64 buckets per workgroup, a 16th of the chunks per wavefront.  The buckets' sizes go
// to bucket_base[b + 1].
__global__ void __launch_bounds__(1024)
k_deep_col_chunks(const DeepArgs A)
{
    __shared__ uint32_t sums[16][64];
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    const int b = blockIdx.x * 64 + lane;
    const bool ok = b < A.buckets;
    const int64_t per = (A.chunks + 15) / 16, c0 = wave * per < A.chunks ? wave * per : A.chunks, c1 = c0 + per < A.chunks ? c0 + per : A.chunks;
    uint32_t* const col = A.chunk_sums + (ok ? b : 0);
    uint32_t sum = 0u;
#pragma unroll 8
    for (int64_t c = c0; c < c1; ++c) sum += col[c * A.buckets];
    sums[wave][lane] = sum;
    __syncthreads();
    uint32_t run = 0u;
    for (int w = 0; w < wave; ++w) run += sums[w][lane];
    if (!ok) return;
#pragma unroll 8
    for (int64_t c = c0; c < c1; ++c) { const uint32_t v = col[c * A.buckets]; col[c * A.buckets] = run; run += v; }
    if (wave == 15) A.P.bucket_base[b + 1] = run;
}

// First sorted position and first piece of every bucket.  CHUNKS: the chunks are few, and their sums are turned into prefixes here.
constexpr int64_t kDeepFewChunks = 64;
template <bool CHUNKS>
__global__ void __launch_bounds__(kSplitMaxBuckets)
k_deep_bases(const DeepArgs A)
{
    __shared__ uint32_t part[kSplitMaxBuckets / 64];
    const int b = threadIdx.x;
    uint32_t cnt = 0u;
    if (b < A.buckets) {
        if (CHUNKS) {
            uint32_t* const col = A.chunk_sums + b;
#pragma unroll 16
            for (int64_t c = 0; c < A.chunks; ++c) { const uint32_t v = col[c * A.buckets]; col[c * A.buckets] = cnt; cnt += v; }
        } else {
            cnt = A.P.bucket_base[b + 1];
        }
    }
    uint32_t total, pieces;
    const uint32_t ex = block_scan<kSplitMaxBuckets>(cnt, part, &total);
    const uint32_t pex = block_scan<kSplitMaxBuckets>((uint32_t)(((uint64_t)cnt + (1u << A.P.tile_bits) - 1u) >> A.P.tile_bits), part, &pieces);
    __syncthreads();
    if (b < A.buckets) { A.P.bucket_base[b] = ex; A.P.piece_base[b] = pex; }
    if (b == A.buckets - 1) { A.P.bucket_base[b + 1] = total; A.P.piece_base[b + 1] = pieces; }
    if (b == 0) *A.P.unit_count = 0u;
}

// The runs of 64 buckets in a chunk of tiles, bucket by bucket: pairs in the tiles before, place in the tile; and which tile a piece begins in.
__global__ void __launch_bounds__(1024)
k_deep_col_runs(const DeepArgs A)
{
    __shared__ uint16_t st[kDeepChunk][66];
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    const int64_t t0 = (int64_t)blockIdx.x * kDeepChunk;
    const int b0 = blockIdx.y * 64;
    for (int i = threadIdx.x; i < kDeepChunk * 65; i += 1024) {
        const int r = i / 65, c = i % 65;
        const int64_t t = t0 + r;
        uint16_t v = 0;
        if (t < A.tiles && b0 + c <= A.buckets) v = A.starts1[t * (A.buckets + 1) + b0 + c];
        st[r][c] = v;
    }
    __syncthreads();
    const int64_t t = t0 + lane;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const int c = wave * 4 + i, b = b0 + c;
        if (b >= A.buckets) break;
        const uint32_t from = st[lane][c], n = t < A.tiles ? st[lane][c + 1] - from : 0u;
        const uint32_t ex = A.chunk_sums[(int64_t)blockIdx.x * A.buckets + b] + wave_scan(n) - n;
        if (t < A.tiles) {
            A.P.before[(int64_t)b * A.tiles + t] = ex;
            A.P.start1[(int64_t)b * A.tiles + t] = (uint16_t)from;
            const uint32_t tile = 1u << A.P.tile_bits, piece = (uint32_t)(((uint64_t)ex + tile - 1u) >> A.P.tile_bits);
            if (((uint64_t)piece << A.P.tile_bits) < (uint64_t)ex + n) {
                const uint32_t seq0 = piece << A.P.tile_bits, left = A.P.bucket_base[b + 1] - A.P.bucket_base[b] - seq0;
                A.P.pieces[A.P.piece_base[b] + piece] = make_uint4((uint32_t)t, (uint32_t)b, seq0, left < tile ? left : tile);
            }
        }
    }
}

// Consecutive stretches of a bucket that a workgroup's LDS holds together are a unit (a stretch beyond that is one of its own), taken from the
// first on while they fit.  One workgroup per bucket; the units of a bucket lie side by side in the list.
__global__ void __launch_bounds__(kSplitMaxBuckets)
k_deep_units(const DeepArgs A, uint32_t capacity)
{
    __shared__ uint32_t from[kSplitMaxBuckets + 1], part[kSplitMaxBuckets / 64], at;
    __shared__ uint16_t next[kSplitMaxBuckets], cut[kSplitMaxBuckets + 1];
    __shared__ int units;
    const int g = threadIdx.x, b = blockIdx.x, G = A.per_bucket;
    const uint32_t piece0 = A.P.piece_base[b];
    const int pieces = (int)(A.P.piece_base[b + 1] - piece0);
    uint32_t n = 0u;
    if (g < G) {
        const uint16_t* row = A.P.starts2 + (int64_t)piece0 * (G + 1) + g;
#pragma unroll 8
        for (int p = 0; p < pieces; ++p, row += G + 1) n += (uint32_t)row[1] - row[0];
    }
    uint32_t total;
    const uint32_t ex = block_scan<kSplitMaxBuckets>(n, part, &total);
    if (g <= G) from[g] = ex;
    if (g == G - 1) from[G] = total;
    __syncthreads();
    if (g < G) {
        int h = g;                      // the last stretch that still fits beside g
        for (int step = kSplitMaxBuckets / 2; step > 0; step >>= 1) h += (h + step < G && from[h + step + 1] - ex <= capacity) ? step : 0;
        next[g] = (uint16_t)(h + 1);
    }
    __syncthreads();
    if (g == 0) {
        int u = 0, h = 0;
        while (h < G && from[h] < total) {
            cut[u++] = (uint16_t)h;
            h = next[h];
        }
        cut[u] = (uint16_t)G;
        units = u;
        at = atomicAdd(A.P.unit_count, (uint32_t)u);
    }
    __syncthreads();
    if (g < units) {
        const uint32_t g0 = cut[g], g1 = cut[g + 1];
        A.P.units[at + g] = make_uint4((uint32_t)b << 20 | g0 << 10 | (g1 - 1u), A.P.bucket_base[b] + from[g0], from[g1] - from[g0], piece0 | (uint32_t)(pieces < kDeepManyPieces ? pieces : kDeepManyPieces) << 19);
    }
}

// A unit, read by its workgroup.  Workgroups go to the chiplets in turn; neighbouring units, which share the cache lines at their runs' ends,
// to the same one.  LDS: where the unit's runs lie in the pieces of its bucket; place e of the unit lies at delta[run] + e of the bucket's
// pieces.  A unit of more pairs than the capacity, or in a bucket of more pieces than threads, is handled in memory, piece after piece.
struct DeepUnit {
    int b, g0, g1, pieces;
    int64_t base, cnt;
    uint32_t piece0, first;           // first: sorted position of the bucket's first pair
    __device__ __forceinline__ bool find(const DeepPlan& P, uint32_t total)
    {
        const uint32_t per = (total + 7u) / 8u, u = (blockIdx.x & 7u) * per + (blockIdx.x >> 3);
        if ((blockIdx.x >> 3) >= per || u >= total) return false;
        const uint4 v = P.units[u];
        b = (int)(v.x >> 20); g0 = (int)(v.x >> 10 & 1023u); g1 = (int)(v.x & 1023u) + 1;
        base = v.y; cnt = v.z;
        piece0 = v.w & 0x7FFFFu; pieces = (int)(v.w >> 19);
        if (pieces == kDeepManyPieces) pieces = (int)(P.piece_base[b + 1] - P.piece_base[b]);      // uniform
        first = P.bucket_base[b];
        return true;
    }
};
template <int THREADS, int ITEMS>
struct UnitRuns {
    uint32_t delta[THREADS];
    uint32_t mask[THREADS * ITEMS / 32], before[THREADS * ITEMS / 32];
    uint32_t part[THREADS / 64], some[THREADS / 64];
};
template <int THREADS, int ITEMS>
__device__ __forceinline__ void unit_runs(const DeepPlan& P, int per_bucket, const DeepUnit& U, UnitRuns<THREADS, ITEMS>& R)
{
    constexpr int WORDS = THREADS * ITEMS / 32, WAVES = THREADS / 64;
    static_assert(WORDS <= THREADS, "one thread per word");
    const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
    uint32_t lo = 0u, n = 0u;
    if (tid < U.pieces) {
        const uint16_t* const row = P.starts2 + (int64_t)(U.piece0 + tid) * (per_bucket + 1);
        lo = row[U.g0];
        n = row[U.g1] - lo;
    }
    if (tid < WORDS) R.mask[tid] = 0u;
    const uint32_t inc = wave_scan(n);
    const uint64_t some = __ballot(n != 0u);
    if (lane == 63) { R.part[wave] = inc; R.some[wave] = (uint32_t)__popcll(some); }
    __syncthreads();
    uint32_t ex = inc - n, at = (uint32_t)__popcll(some & ((1ull << lane) - 1ull));
#pragma unroll
    for (int w = 0; w < WAVES; ++w) {
        ex += w < wave ? R.part[w] : 0u;
        at += w < wave ? R.some[w] : 0u;
    }
    if (n) {
        R.delta[at] = ((uint32_t)tid << P.tile_bits) + lo - ex;
        if (ex < (uint32_t)(THREADS * ITEMS)) atomicOr(&R.mask[ex >> 5], 1u << (ex & 31u));
    }
    __syncthreads();
    uint32_t total;
    const uint32_t bits = block_scan<THREADS>(tid < WORDS ? (uint32_t)__popc(R.mask[tid]) : 0u, R.part, &total);
    if (tid < WORDS) R.before[tid] = bits;
    __syncthreads();
}

// The pairs of a unit piece by piece, where it does not fit: use(place among the pairs as gathered, place in the piece layout, piece).
template <int THREADS, typename USE>
__device__ __forceinline__ void each_of_unit(const DeepPlan& P, int per_bucket, const DeepUnit& U, USE use)
{
    int64_t e0 = 0;
    for (int p = 0; p < U.pieces; ++p) {
        const uint16_t* const row = P.starts2 + (int64_t)(U.piece0 + p) * (per_bucket + 1);
        const int lo = row[U.g0], n = row[U.g1] - lo;
        const int64_t from = (int64_t)U.first + ((int64_t)p << P.tile_bits) + lo;
        for (int i = threadIdx.x; i < n; i += THREADS) use(e0 + i, from + i, p);
        e0 += n;
    }
}

// (The larger units as 16 pairs a thread: as 8 of 1024 threads, whose registers spill, 2^31 positions take 112.4 ms a step in place of 110.0.)
template <int THREADS, int ITEMS>
__global__ void __launch_bounds__(THREADS, ITEMS == 16 ? 4 : 6)
k_deep_sort(const DeepArgs A)
{
    constexpr int CAP = THREADS * ITEMS;
    __shared__ __align__(16) uint32_t buf[2 * CAP];         // counts of bins, then the pairs
    __shared__ UnitRuns<THREADS, ITEMS> R;
    __shared__ StretchShared<THREADS> S;
    const int tid = threadIdx.x;
    DeepUnit U;
    if (!U.find(A.P, *A.P.unit_count)) return;
    if (tid == 0) S.init();
    const int64_t cnt = U.cnt, base = U.base;
    if (cnt == 0) return;               // uniform
    // (the decay of the first pair, and what pk8 holds of it, are k_deep_edges')
    uint32_t* const ids = A.ids + base;
    float* const pk = A.pk + base + 1;
    float* const dh = A.dh + base;
    float2* const pk8 = A.pk8 + (base >> 3);
    auto write = [&](uint32_t e, uint32_t key, uint32_t before, uint32_t id) {
        const float p = split_key_to_float(key), q = split_key_to_float(before);
        ids[e] = id;
        pk[e] = p;
        if (e > 0u) {
            dh[e] = key == before ? -1.0f : expf(-(p - q));
            const uint32_t at = e + ((uint32_t)base & 7u);
            if ((at & 7u) == 0u) pk8[at >> 3] = make_float2(q, p);          // pk8[m] = (pk[8m], pk[8m + 1])
        }
    };
    if (cnt <= CAP && U.pieces <= THREADS) {      // uniform
        unit_runs<THREADS, ITEMS>(A.P, A.per_bucket, U, R);
        uint32_t key[ITEMS], id[ITEMS], rank[ITEMS];
        const int n = (int)cnt;
        // (within 2^23 pairs of the bucket's first)
        const uint2* const pairs = A.pairs2 + U.first;
        stretch_ranks<THREADS, ITEMS>(key, id, n, pairs[R.delta[0]].x, A.id_bits, buf, S, rank, [&](int e, uint32_t& key_e, uint32_t& id_e) {
            const uint2 v = pairs[R.delta[run_of(R.mask, R.before, (uint32_t)e)] + (uint32_t)e];
            key_e = v.x; id_e = v.y;
        }, [](uint32_t, uint32_t) {});
        __syncthreads();
        unsigned long long* const slot = reinterpret_cast<unsigned long long*>(buf);
        uint16_t* const slot3 = A.P.slot3 + base;
#pragma unroll
        for (int i = 0; i < ITEMS; ++i)
            if (i * THREADS + tid < n) {
                slot[rank[i]] = ((unsigned long long)key[i] << 32) | id[i];
                slot3[(uint32_t)(i * THREADS + tid)] = (uint16_t)rank[i];
            }
        __syncthreads();
#pragma unroll
        for (int i = 0; i < ITEMS; ++i) {
            const int e = i * THREADS + tid;
            if (e < n) {
                const unsigned long long v = slot[e];
                write((uint32_t)e, (uint32_t)(v >> 32), e > 0 ? (uint32_t)(slot[e - 1] >> 32) : 0u, (uint32_t)v);
            }
        }
        return;
    }
    __syncthreads();
    uint2* const spare = A.spare + base;
    uint32_t k_and = 0xFFFFFFFFu, k_or = 0u, k_min = 0xFFFFFFFFu, k_max = 0u, i_min = 0xFFFFFFFFu, i_max = 0u;
    each_of_unit<THREADS>(A.P, A.per_bucket, U, [&](int64_t e, int64_t src, int) {
        const uint2 v = A.pairs2[src];
        spare[e] = v;
        k_and &= v.x; k_or |= v.x;
        k_min = v.x < k_min ? v.x : k_min; k_max = v.x > k_max ? v.x : k_max;
        i_min = v.y < i_min ? v.y : i_min; i_max = v.y > i_max ? v.y : i_max;
    });
    atomicAnd(&S.key_and, k_and); atomicOr(&S.key_or, k_or); atomicMin(&S.key_min, k_min); atomicMax(&S.key_max, k_max);
    atomicMin(&S.id_min, i_min); atomicMax(&S.id_max, i_max);
    __threadfence_block();
    __syncthreads();
    const uint32_t vary = S.key_or & ~S.key_and;
    if (!count_in_memory<THREADS, CAP>(spare, A.ids + base, A.pk + base + 1, cnt, StretchRange(S.key_min, S.key_max, S.id_min, S.id_max, vary), buf, R.part)) {
        const uint32_t id_span = S.id_max - S.id_min;      // the low digits of the ids up to where the smallest and the largest differ
        sort_in_memory<THREADS>(spare, A.ids + base, A.pk + base + 1, cnt, vary, id_span ? 0xFFFFFFFFu >> __clz((int)(S.id_min ^ S.id_max)) : 0u, buf);
    }
    // where every gathered pair went: its place among the sorted ones
    each_of_unit<THREADS>(A.P, A.per_bucket, U, [&](int64_t e, int64_t src, int) {
        const uint2 v = A.pairs2[src];
        int64_t lo = 0, hi = cnt;
        while (lo < hi) {
            const int64_t m = (lo + hi) >> 1;
            const uint2 o = spare[m];
            if (o.x < v.x || (o.x == v.x && o.y < v.y)) lo = m + 1; else hi = m;
        }
        A.P.slot3[base + e] = (uint16_t)lo;
        A.P.slot3_high[base + e] = (uint16_t)(lo >> 16);
    });
    for (int64_t e = tid; e < cnt; e += THREADS) {
        const uint2 v = spare[e];
        write((uint32_t)e, v.x, e > 0 ? spare[e - 1].x : 0u, v.y);
    }
}

__global__ void __launch_bounds__(256)
k_deep_edges(const DeepArgs A)
{
    const int64_t u = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (u < (int64_t)*A.P.unit_count) {
        const int64_t j = A.P.units[u].y;
        if (A.pk8 && (j & 7) == 0) A.pk8[j >> 3] = make_float2(j > 0 ? A.pk[j] : -__uint_as_float(0x7F800000u), A.pk[j + 1]);
        if (j > 0) {
            const float before = A.pk[j], p = A.pk[j + 1];
            A.dh[j] = p == before ? -1.0f : expf(-(p - before));
        }
    }
    if (blockIdx.x == 0 && threadIdx.x < 64) A.counters[threadIdx.x] = 0u;        // list lengths of the scans; the plan is valid
    if (blockIdx.x == 0 && threadIdx.x == 0) {
        const float inf = __uint_as_float(0x7F800000u);
        A.dh[0] = 0.0f; A.dh[A.N] = 0.0f;
        A.pk[0] = -inf; A.pk[A.N + 1] = inf;
        if (A.pk8) {
                if ((A.N & 7) == 7) A.pk8[(A.N + 1) >> 3] = make_float2(inf, inf);
            if ((A.N & 7) == 0) A.pk8[A.N >> 3] = make_float2(A.pk[A.N], inf);
        }
    }
}

// ---------------------------------------------------------------------------------------------------------------------
// Values along the same way.  The values of ids lo .. hi - 1 take part; every other position of the sorted order reads as zero.  What the
// other ids' tiles, and pieces without any of these ids, would leave is neither written nor read.
// ---------------------------------------------------------------------------------------------------------------------
struct MoveArgs {
    DeepPlan P;
    const uint32_t* ids;
    int buckets, per_bucket; int64_t N, tiles;
    const float* src; int64_t ld; int64_t lo, hi;
    int64_t tile0, tile1;            // tiles that hold ids of the range
    float* by_tile; float* by_piece; float* dst;
};

// Anchors that came in order: the ids of either side ascend along the sorted sequence, and rows are fetched one after the other.  Bound by memory: 4 bytes
// of id, 4 of result and a value for every row of the side (us, sort and moves along its passes / merge and this: forward 1380000 x 3220000 276 / 116, 2^23 x 2^23
// 660 / 362, Gram form of 2^23 412 / 172; forward + backward 2516583 x 5872025 557 / 338; radix sort and records of (rank, value): 194, 685, 289; 475).
__device__ __forceinline__ void move_in_order(int64_t N, const uint32_t* ids, const float* src, int64_t ld, int64_t lo, int64_t hi, float* dst, int64_t quad)
{
    auto value = [&](uint32_t id) { return (int64_t)id >= lo && (int64_t)id < hi ? src[((int64_t)id - lo) * ld] : 0.0f; };
    const int64_t j = 4 * quad;
    if (j + 4 <= N) {
        const uint4 v = reinterpret_cast<const uint4*>(ids)[quad];
        reinterpret_cast<float4*>(dst)[quad] = make_float4(value(v.x), value(v.y), value(v.z), value(v.w));
    } else {
        for (int64_t i = j; i < N; ++i) dst[i] = value(ids[i]);
    }
}
__global__ void __launch_bounds__(256)
k_move_in_order(int64_t N, const uint32_t* __restrict__ ids, const float* __restrict__ src, int64_t ld, int64_t lo, int64_t hi, float* __restrict__ dst)
{
    move_in_order(N, ids, src, ld, lo, hi, dst, (int64_t)blockIdx.x * 256 + threadIdx.x);
}

// A tile's values in its layout.
template <int PER>
__global__ void __launch_bounds__(kDeepThreads, 8)
k_move_tiles(const MoveArgs A)
{
    constexpr int TILE = kDeepThreads * PER;
    __shared__ __align__(16) float v[TILE];
    const int tid = threadIdx.x;
    const int64_t base = (A.tile0 + blockIdx.x) * TILE;
    const int len = A.N - base < TILE ? (int)(A.N - base) : TILE;
    float* const by_tile = A.by_tile + base;
    const uint16_t* const from1 = A.P.from1 + base;
    const bool tables = *A.P.unit_count != kDeepMerged;
    float x[PER];
    uint16_t from[PER];
#pragma unroll
    for (int i = 0; i < PER; ++i) {
        const int64_t id = base + i * kDeepThreads + tid;
        x[i] = id >= A.lo && id < A.hi ? A.src[(id - A.lo) * A.ld] : 0.0f;
    }
#pragma unroll
    for (int i = 0; i < PER; ++i) {
        const int q = i * kDeepThreads + tid;
        from[i] = from1[(uint32_t)(q < len ? q : 0)];
    }
    if (!tables) return;                // uniform (asked for above: nothing waits for it)
#pragma unroll
    for (int i = 0; i < PER; ++i) v[i * kDeepThreads + tid] = x[i];
    __syncthreads();
#pragma unroll
    for (int i = 0; i < PER; ++i) {
        const int q = i * kDeepThreads + tid;
        if (q < len) by_tile[(uint32_t)q] = v[from[i]];
    }
}

// Places of a bucket (its pairs in the order of their tiles) that ids of the range can have.
__device__ __forceinline__ void seq_range(const MoveArgs& A, int b, uint32_t& from, uint32_t& to)
{
    const uint32_t* const col = A.P.before + (int64_t)b * A.tiles;
    from = col[A.tile0];
    to = A.tile1 < A.tiles ? col[A.tile1] : A.P.bucket_base[b + 1] - A.P.bucket_base[b];
}

// A piece's values in its layout.
template <int PER>
__global__ void __launch_bounds__(kDeepThreads, 8)
k_move_pieces(const MoveArgs A)
{
    constexpr int TILE = kDeepThreads * PER;
    __shared__ __align__(16) float v[TILE];
    __shared__ uint32_t mask[TILE / 32], before[TILE / 32], part[kDeepThreads / 64];
    const int tid = threadIdx.x;
    DeepPiece p;
    if (!find_piece(A.P, A.buckets, blockIdx.x, p)) return;
    uint32_t from, to;
    seq_range(A, p.bucket, from, to);
    if (p.seq0 >= to || p.seq0 + (uint32_t)p.len <= from) return;       // uniform: nothing of the range
    const int64_t out = (int64_t)A.P.bucket_base[p.bucket] + p.seq0;
    piece_runs<PER>(A.P, A.tiles, p, reinterpret_cast<uint32_t*>(v), mask, before, part);
    float* const by_piece = A.by_piece + out;
    const uint16_t* const slot2 = A.P.slot2 + out;
    float x[PER];
    uint16_t slot[PER];
#pragma unroll
    for (int i = 0; i < PER; ++i) {
        const uint32_t q = (uint32_t)(i * kDeepThreads + tid), e = q < (uint32_t)p.len ? q : (uint32_t)p.len - 1u;
        const uint32_t src = reinterpret_cast<const uint32_t*>(v)[run_of(mask, before, e)] + e;
        x[i] = p.seq0 + e >= from && p.seq0 + e < to ? A.by_tile[src] : 0.0f;
        slot[i] = slot2[e];
    }
    __syncthreads();
#pragma unroll
    for (int i = 0; i < PER; ++i)
        if (i * kDeepThreads + tid < p.len) v[slot[i]] = x[i];
    __syncthreads();
#pragma unroll
    for (int i = 0; i < PER; ++i) {
        const int q = i * kDeepThreads + tid;
        if (q < p.len) by_piece[(uint32_t)q] = v[q];
    }
}

// A unit's values in sorted order.  (256 threads of 16 pairs: the units of 2^22 to 2^23 positions are a few more than as many workgroups of 512 threads as fit; us, forward on
// a kept plan, 512 of 8 / this: 2^22 x 2^22 115.4 / 113.1, 2^23 x 2^23 211 / 206.)  What slot3 says does not depend on how the sort went about the unit, in LDS or in
// memory: places among the pairs as gathered count piece by piece either way, so that this may go the other way.
template <int THREADS, int ITEMS>
__global__ void __launch_bounds__(THREADS, 8)
k_move_units(const MoveArgs A)
{
    constexpr int CAP = THREADS * ITEMS;
    __shared__ float v[CAP];
    __shared__ UnitRuns<THREADS, ITEMS> R;
    const int tid = threadIdx.x;
    const uint32_t units = *A.P.unit_count;
    if (units == kDeepMerged) {         // uniform
        for (int64_t q = (int64_t)blockIdx.x * THREADS + tid; 4 * q < A.N; q += (int64_t)gridDim.x * THREADS) move_in_order(A.N, A.ids, A.src, A.ld, A.lo, A.hi, A.dst, q);
        return;
    }
    DeepUnit U;
    if (!U.find(A.P, units)) return;
    const int64_t cnt = U.cnt, base = U.base;
    uint32_t from, to;
    seq_range(A, U.b, from, to);
    // pieces that were written: those with a place of the range
    const uint32_t first = from >> A.P.tile_bits, last = to > from ? (to - 1u) >> A.P.tile_bits : 0u;
    const bool any = to > from;
    if (cnt <= CAP && U.pieces <= THREADS) {      // uniform
        unit_runs<THREADS, ITEMS>(A.P, A.per_bucket, U, R);
        const int n = (int)cnt;
        const float* const by_piece = A.by_piece + U.first;
        const uint16_t* const slot3 = A.P.slot3 + base;
        float* const dst = A.dst + base;
        const uint32_t lo = first << A.P.tile_bits, span = any ? (last - first + 1u) << A.P.tile_bits : 0u;
        float x[ITEMS];
        uint16_t slot[ITEMS];
#pragma unroll
        for (int i = 0; i < ITEMS; ++i) {
            if (i * THREADS < n) {                // uniform
                const uint32_t e = (uint32_t)(i * THREADS + tid < n ? i * THREADS + tid : n - 1);
                const uint32_t src = R.delta[run_of(R.mask, R.before, e)] + e;
                x[i] = src - lo < span ? by_piece[src] : 0.0f;
                slot[i] = slot3[e];
            }
        }
#pragma unroll
        for (int i = 0; i < ITEMS; ++i)
            if (i * THREADS + tid < n) v[slot[i]] = x[i];
        __syncthreads();
#pragma unroll
        for (int i = 0; i < ITEMS; ++i)
            if (i * THREADS + tid < n) dst[(uint32_t)(i * THREADS + tid)] = v[i * THREADS + tid];
        return;
    }
    each_of_unit<THREADS>(A.P, A.per_bucket, U, [&](int64_t e, int64_t src, int piece) {
        const bool in = any && (uint32_t)piece >= first && (uint32_t)piece <= last;
        int64_t to_place = A.P.slot3[base + e];
        to_place |= (int64_t)A.P.slot3_high[base + e] << 16;
        A.dst[base + to_place] = in ? A.by_piece[src] : 0.0f;
    });
}

DeepArgs deep_args(const DeepGeom& G, const DeepPlan& P)
{
    DeepArgs A{};
    A.P = P; A.N = G.N;
    A.buckets = G.buckets; A.per_bucket = G.per_bucket; A.samples_per = G.samples_per;
    A.tiles = G.tiles; A.chunks = (G.tiles + kDeepChunk - 1) / kDeepChunk; A.samples = G.samples; A.stretches = G.stretches;
    A.id_bits = 1; while (A.id_bits < 32 && ((int64_t)1 << A.id_bits) < G.N) ++A.id_bits;
    A.sample_step = ((uint64_t)G.N << 20) / (uint64_t)G.samples;
    return A;
}

// The sort's scratch, in bytes from its start.
struct DeepScratch {
    size_t bounds, keys1, starts1, chunk_sums, pairs2, spare, sampled, sample_ids, sample_dh, sample_pk, sample_pair0, sample_pair1, sample_words, sample_counters, total;
    explicit DeepScratch(const DeepGeom& G)
    {
        const int64_t chunks = (G.tiles + kDeepChunk - 1) / kDeepChunk;
        const size_t S = (size_t)G.samples, N = (size_t)G.N;
        size_t o = 0;
        auto take = [&](size_t bytes) { const size_t at = o; o = align_up(o + bytes); return at; };
        bounds = take(8 * (size_t)G.stretches);
        starts1 = take(2 * (size_t)G.tiles * (size_t)(G.buckets + 1));
        chunk_sums = take(4 * (size_t)chunks * (size_t)G.buckets);
        pairs2 = take(8 * N);
        keys1 = spare = take(8 * N);      // the keys in tile layout are dead when a stretch may need the spare pairs
        const size_t end = o;
        o = pairs2;                       // the samples are dead when the pieces are laid out
        sampled = take(4 * S); sample_ids = take(4 * S); sample_dh = take(4 * (S + 1)); sample_pk = take(4 * (S + 2));
        sample_pair0 = take(8 * S); sample_pair1 = take(8 * S);
        sample_words = take(4 * split_sort_words(G.samples)); sample_counters = take(4 * 64);
        total = o > end ? o : end;
    }
};

}  // namespace

// Tiles and pieces of 8192 positions where those of 16384 would leave most of the compute units one workgroup, or none (us, 16384 / 8192, forward on a kept plan, forward,
// forward + backward: 1258292 x 2936012 77.9 / 72.5, 220 / 206, 323 / 306; 2^22 x 2^22 116 / 114, 351 / 328, 536 / 514; Gram form of 10^7 252 / 246, 497 / 474, 907 / 886;
// 2^23 x 2^23 211 / 211, 573 / 563, 914 / 910), but not where runs get short (2^24 x 2^24 forward + backward 1842 / 1857; 2^25 x 2^25 forward 2001 / 2057).
constexpr int64_t kDeepSmallTilesMax = int64_t(1) << 24;
// Stretches longer than a workgroup sorts in LDS, expected per sort of anchors without ties (a stretch's length is a sum of samples_per gaps between samples, so a Gamma variable): 1e-3
// at 2^28 positions, 0.05 at 2^29 (five samples a stretch), 1e-4 at 2^30, 98 at 2^31 (four samples, 2048 pairs on average), 3700 at 3e9 and 44000, 4.2 %, at 2^32.  A workgroup sorts such a
// stretch in memory.  At 2^31 they hide among the other units; the largest problems wait for them: forward + backward 106 ms for 2^30 x 2^30 (the sort of the units 19), 162 for
// 1.5e9 x 1.5e9 (39) and 417 for 2147483647 x 2147483647 (199, and 27 instead of 7 a move).
DeepGeom deep_geom(int64_t N)
{
    DeepGeom G;
    G.N = N;
    G.capacity = N > (int64_t(1) << 29) ? 8192 : 4096;
    int64_t stretches = (N + 767) / 768;
    if (stretches > (int64_t(1) << 20)) stretches = int64_t(1) << 20;
    int64_t buckets = 1;
    while (buckets * buckets < N / 3600) ++buckets;
    while (buckets * kSplitMaxBuckets < stretches) ++buckets;
    if (buckets > kSplitMaxBuckets) buckets = kSplitMaxBuckets;
    G.buckets = (int)buckets;
    G.per_bucket = (int)((stretches + buckets - 1) / buckets);
    if (G.per_bucket > kSplitMaxBuckets) G.per_bucket = kSplitMaxBuckets;
    G.stretches = (int64_t)G.buckets * G.per_bucket;
    const int64_t per = kSplitSortMax / G.stretches;
    G.samples_per = per < 6 ? (int)per : 6;
    G.samples = G.stretches * G.samples_per;
    G.max_units = 2 * (N / G.capacity) + 2 * G.buckets;
    G.tile_bits = N <= kDeepSmallTilesMax ? 13 : 14;
    G.tiles = (N + ((int64_t)1 << G.tile_bits) - 1) >> G.tile_bits;
    G.max_pieces = G.tiles + G.buckets;
    return G;
}

size_t deep_scratch_bytes(const DeepGeom& G) { return DeepScratch(G).total; }

hipError_t launch_deep_sort(const float* a, int64_t k, const float* b, int64_t n, float tau, const DeepGeom& G, const DeepPlan& P, char* scratch,
                            uint32_t* ids, float* dh, float* pk, float2* pk8, uint32_t* counters, hipStream_t st)
{
    const DeepScratch D(G);
    DeepArgs A = deep_args(G, P);
    A.a = a; A.b = b; A.k = k; A.tau = tau;
    A.sampled = reinterpret_cast<float*>(scratch + D.sampled);
    A.sample_ids = reinterpret_cast<const uint32_t*>(scratch + D.sample_ids); A.sample_pk = reinterpret_cast<const float*>(scratch + D.sample_pk);
    A.bounds = reinterpret_cast<unsigned long long*>(scratch + D.bounds);
    A.keys1 = reinterpret_cast<uint32_t*>(scratch + D.keys1); A.starts1 = reinterpret_cast<uint16_t*>(scratch + D.starts1);
    A.chunk_sums = reinterpret_cast<uint32_t*>(scratch + D.chunk_sums);
    A.pairs2 = reinterpret_cast<uint2*>(scratch + D.pairs2); A.spare = reinterpret_cast<uint2*>(scratch + D.spare);
    A.ids = ids; A.dh = dh; A.pk = pk; A.pk8 = pk8; A.counters = counters;
    auto of = [](int64_t items, int per) { return dim3((unsigned)((items + per - 1) / per)); };
    LAPLEX_TIMED("deep_sample", st, hipLaunchKernelGGL(k_deep_sample, of(A.samples, 256), dim3(256), 0, st, A));
    const hipError_t e = launch_split_sort(A.sampled, A.samples, nullptr, 0, 1.0f, reinterpret_cast<uint2*>(scratch + D.sample_pair0),
                                           reinterpret_cast<uint2*>(scratch + D.sample_pair1), reinterpret_cast<uint32_t*>(scratch + D.sample_words),
                                           reinterpret_cast<uint32_t*>(scratch + D.sample_ids), reinterpret_cast<float*>(scratch + D.sample_dh),
                                           reinterpret_cast<float*>(scratch + D.sample_pk), nullptr,
                                           reinterpret_cast<uint32_t*>(scratch + D.sample_counters), 1, 0, 0, 0, st);
    if (e != hipSuccess) return e;
    LAPLEX_TIMED("deep_bounds", st, hipLaunchKernelGGL(k_deep_bounds, of(A.stretches, 256), dim3(256), 0, st, A));
    auto distribute = [&](const char* family, auto kernel, int64_t groups) { LAPLEX_TIMED(family, st, hipLaunchKernelGGL(kernel, dim3((unsigned)groups), dim3(kDeepThreads), 0, st, A)); };
    if (G.tile_bits == 13) distribute("deep_tiles", k_deep_distribute<false, 8>, A.tiles); else distribute("deep_tiles", k_deep_distribute<false, 16>, A.tiles);
    LAPLEX_TIMED("deep_columns", st, hipLaunchKernelGGL(k_deep_col_sums, dim3((unsigned)A.chunks), dim3(kSplitMaxBuckets), 0, st, A));
    if (A.chunks <= kDeepFewChunks) {
        LAPLEX_TIMED("deep_columns", st, hipLaunchKernelGGL((k_deep_bases<true>), dim3(1), dim3(kSplitMaxBuckets), 0, st, A));
    } else {
        LAPLEX_TIMED("deep_columns", st, hipLaunchKernelGGL(k_deep_col_chunks, of(A.buckets, 64), dim3(1024), 0, st, A));
        LAPLEX_TIMED("deep_columns", st, hipLaunchKernelGGL((k_deep_bases<false>), dim3(1), dim3(kSplitMaxBuckets), 0, st, A));
    }
    LAPLEX_TIMED("deep_columns", st, hipLaunchKernelGGL(k_deep_col_runs, dim3((unsigned)A.chunks, (unsigned)((A.buckets + 63) / 64)), dim3(1024), 0, st, A));
    if (G.tile_bits == 13) distribute("deep_pieces", k_deep_distribute<true, 8>, G.max_pieces); else distribute("deep_pieces", k_deep_distribute<true, 16>, G.max_pieces);
    LAPLEX_TIMED("deep_units", st, hipLaunchKernelGGL(k_deep_units, dim3((unsigned)A.buckets), dim3(kSplitMaxBuckets), 0, st, A, (uint32_t)G.capacity));
    const dim3 units((unsigned)((G.max_units + 7) / 8 * 8));
    if (G.capacity == 8192) LAPLEX_TIMED("deep_sort", st, hipLaunchKernelGGL((k_deep_sort<512, 16>), units, dim3(512), 0, st, A));
    else LAPLEX_TIMED("deep_sort", st, hipLaunchKernelGGL((k_deep_sort<512, 8>), units, dim3(512), 0, st, A));
    LAPLEX_TIMED("deep_edges", st, hipLaunchKernelGGL(k_deep_edges, of(G.max_units, 256), dim3(256), 0, st, A));
    return hipGetLastError();
}

hipError_t launch_move_in_order(int64_t N, const uint32_t* ids, const float* src, int64_t ld, int64_t lo, int64_t hi, float* dst, const char* tag, hipStream_t st)
{
    const std::string f = std::string("move_in_order.") + tag;
    LAPLEX_TIMED(f.c_str(), st, hipLaunchKernelGGL(k_move_in_order, dim3((unsigned)((N + 1023) / 1024)), dim3(256), 0, st, N, ids, src, ld, lo, hi, dst));
    return hipGetLastError();
}

hipError_t launch_deep_move(const DeepGeom& G, const DeepPlan& P, const uint32_t* ids, const float* src, int64_t ld, int64_t lo, int64_t hi,
                            float* by_tile, float* by_piece, float* dst, const char* tag, hipStream_t st)
{
    MoveArgs A{};
    A.P = P; A.ids = ids; A.buckets = G.buckets; A.per_bucket = G.per_bucket; A.N = G.N; A.tiles = G.tiles;
    A.src = src; A.ld = ld; A.lo = lo; A.hi = hi;
    A.tile0 = lo >> G.tile_bits; A.tile1 = (hi + ((int64_t)1 << G.tile_bits) - 1) >> G.tile_bits;
    A.by_tile = by_tile; A.by_piece = by_piece; A.dst = dst;
    const std::string ft = std::string("move_tiles.") + tag, fp = std::string("move_pieces.") + tag, fs = std::string("move_units.") + tag;
    auto move = [&](const std::string& family, auto kernel, int64_t groups) { LAPLEX_TIMED(family.c_str(), st, hipLaunchKernelGGL(kernel, dim3((unsigned)groups), dim3(kDeepThreads), 0, st, A)); };
    if (G.tile_bits == 13) { move(ft, k_move_tiles<8>, A.tile1 - A.tile0); move(fp, k_move_pieces<8>, G.max_pieces); }
    else { move(ft, k_move_tiles<16>, A.tile1 - A.tile0); move(fp, k_move_pieces<16>, G.max_pieces); }
    const dim3 units((unsigned)((G.max_units + 7) / 8 * 8));
    if (G.capacity == 8192) LAPLEX_TIMED(fs.c_str(), st, hipLaunchKernelGGL((k_move_units<1024, 8>), units, dim3(1024), 0, st, A));
    else LAPLEX_TIMED(fs.c_str(), st, hipLaunchKernelGGL((k_move_units<256, 16>), units, dim3(256), 0, st, A));
    return hipGetLastError();
}

}  // namespace laplex

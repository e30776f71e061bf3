// Device code of the sort by samples (split_sort_kernels.hip): keys, scans, the search among the bounds, and the sort of one stretch.
#pragma once

#include "laplex_internal.h"

namespace laplex {

namespace {

__device__ __forceinline__ uint32_t split_key(float f)
{
    const uint32_t u = __float_as_uint(f + 0.0f);       // -0.0 sorts as +0.0
    return u ^ ((uint32_t)((int32_t)u >> 31) | 0x80000000u);
}
__device__ __forceinline__ float split_key_to_float(uint32_t key)
{
    return __uint_as_float(key ^ ((key >> 31) ? 0x80000000u : 0xFFFFFFFFu));
}

// Inclusive scan of one word per lane.
__device__ __forceinline__ uint32_t wave_scan(uint32_t v)
{
    v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x111, 0xF, 0xF, false);      // row_shr:1, 2, 4, 8
    v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x112, 0xF, 0xF, false);
    v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x114, 0xF, 0xF, false);
    v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x118, 0xF, 0xF, false);
    v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x142, 0xA, 0xF, false);      // the row before's last lane into rows 1 and 3
    v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x143, 0xC, 0xF, false);      // lane 31 into rows 2 and 3
    return v;
}

// Reduction over the wavefront, the result in lane 63 only.
template <typename OP>
__device__ __forceinline__ uint32_t wave_fold(uint32_t v, uint32_t none, OP op)
{
    auto step = [&](uint32_t o) { v = op(v, o); };
    step((uint32_t)__builtin_amdgcn_update_dpp((int)none, (int)v, 0x111, 0xF, 0xF, false));
    step((uint32_t)__builtin_amdgcn_update_dpp((int)none, (int)v, 0x112, 0xF, 0xF, false));
    step((uint32_t)__builtin_amdgcn_update_dpp((int)none, (int)v, 0x114, 0xF, 0xF, false));
    step((uint32_t)__builtin_amdgcn_update_dpp((int)none, (int)v, 0x118, 0xF, 0xF, false));
    step((uint32_t)__builtin_amdgcn_update_dpp((int)none, (int)v, 0x142, 0xA, 0xF, false));
    step((uint32_t)__builtin_amdgcn_update_dpp((int)none, (int)v, 0x143, 0xC, 0xF, false));
    return v;
}

// Exclusive scan of one word per thread; *total gets the sum.  part: THREADS / 64 words of LDS, free again when this returns.
template <int THREADS>
__device__ __forceinline__ uint32_t block_scan(uint32_t v, uint32_t* part, uint32_t* total)
{
    const int wave = threadIdx.x >> 6;
    const uint32_t inc = wave_scan(v);
    if ((threadIdx.x & 63) == 63) part[wave] = inc;
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

// The bounds of the stretches in LDS, (key, id) of the first pair of each (the first stretch has none; `stride` apart), and the search among them.
// id: kSplitMaxBuckets words, same: as many half-words, key: kBoundWords, a word of padding behind every 32 (the steps of the search are powers of two: without it
// the words that the lanes of a wavefront compare with share a bank; one of 1024 bounds for 2^27 pairs, cycles of the LDS, without / with: 455 / 251 million of
// a whole distribution).  To be made by all threads of the workgroup, before a barrier of theirs frees what lies in these arrays.
constexpr int kSplitMaxBuckets = 1024;
constexpr int kBoundWords = kSplitMaxBuckets + kSplitMaxBuckets / 32;
template <int THREADS>
struct StretchBounds {
    const uint32_t* key; const uint32_t* id; const uint16_t* same;      // same: bounds with this one's key, from it on
    static __device__ __forceinline__ uint32_t padded(uint32_t i) { return i + (i >> 5); }
    int top = 1;                    // half the power of two that holds all stretches
    int tied = 0;
    __device__ __forceinline__ StretchBounds(const unsigned long long* bounds, int buckets, int stride, uint32_t* key_, uint32_t* id_, uint16_t* same_)
        : key(key_), id(id_), same(same_)
    {
        while (2 * top < buckets) top *= 2;
        for (int i = threadIdx.x; i < 2 * top; i += THREADS) {
            const unsigned long long v = i > 0 && i < buckets ? bounds[(int64_t)i * stride] : ~0ull;      // (never reached: ids are below 2^32 - 1)
            key_[padded(i)] = (uint32_t)(v >> 32); id_[i] = (uint32_t)v;
            tied |= i > 0 && i + 1 < buckets && bounds[(int64_t)(i + 1) * stride] >> 32 == v >> 32;
        }
        tied = __syncthreads_or(tied);
        if (tied) {                     // uniform: many equal anchors.  How many bounds share a key
            for (int i = threadIdx.x; i < 2 * top; i += THREADS) {
                const uint32_t v = key_[padded(i)];
                int last = i;
                for (int step = top; step > 0; step >>= 1) last += (last + step < buckets && key_[padded(last + step)] <= v) ? step : 0;
                same_[i] = (uint16_t)(i > 0 ? last - i + 1 : 1);
            }
            __syncthreads();
        }
    }
    // at[i]: the stretch of (keys[i], id_of(i))
    template <int PER, typename ID>
    __device__ __forceinline__ void find(const uint32_t (&keys)[PER], uint32_t (&at)[PER], ID id_of) const
    {
        // bytes from the start of the padded array: the place of a sum of distinct powers of two is the sum of theirs
#pragma unroll
        for (int i = 0; i < PER; ++i) at[i] = 0u;
#pragma unroll 1
        for (int step = top; step > 0; step >>= 1) {
            const uint32_t by = 4u * padded((uint32_t)step);
#pragma unroll
            for (int i = 0; i < PER; ++i) {
                const uint32_t t = at[i] + by;
                at[i] = *reinterpret_cast<const uint32_t*>(reinterpret_cast<const char*>(key) + t) < keys[i] ? t : at[i];
            }
        }
        // the bounds of an equal key, if there are any, by their ids: a search among those that share it (in place of a second search among all of
        // them, keys and ids; 2^22 anchors, us: 31 values 59 / 40, narrow clusters 53 / 36, 32 of a value 39 / 33, none equal 33 / 32)
#pragma unroll
        for (int i = 0; i < PER; ++i) {
            at[i] >>= 2;
            at[i] -= (at[i] * 1986u) >> 16;      // at / 33, up to 1087
            const uint32_t next = at[i] + 1 < (uint32_t)(2 * top) ? at[i] + 1 : at[i];
            if (next != at[i] && key[padded(next)] == keys[i] && id[next] <= id_of(i)) {
                uint32_t g = next;
                if (tied) {
                    const uint32_t end = next + same[next], me = id_of(i);
                    uint32_t step = 1u;
                    while (next + step < end) step *= 2u;
                    for (; step > 0u; step >>= 1) g += (g + step < end && id[g + step] <= me) ? step : 0u;
                }
                at[i] = g;
            }
        }
    }
};

// Where (key, id) lies in the range of a stretch, as 64 bits from the top: (key - smallest key, id - smallest id) without the low bits that
// no key differs in.
struct StretchRange {
    uint32_t kmin, imin;
    int low_zeros, id_bits, up;
    __device__ __forceinline__ StretchRange(uint32_t kmin_, uint32_t kmax, uint32_t imin_, uint32_t imax, uint32_t vary)
        : kmin(kmin_), imin(imin_), low_zeros(vary ? __ffs((int)vary) - 1 : 0)
    {
        const uint32_t span = (kmax - kmin_) >> low_zeros, ispan = imax - imin_;
        id_bits = ispan ? 32 - __clz((int)ispan) : 0;
        const int bits = (span ? 32 - __clz((int)span) : 0) + id_bits;
        up = bits > 0 ? 64 - bits : 0;
    }
    // The fraction times bins: the bin in the upper word, the fraction inside the bin below.
    __device__ __forceinline__ unsigned long long place(uint32_t key, uint32_t id, uint32_t bins) const
    {
        const unsigned long long f = ((((unsigned long long)((key - kmin) >> low_zeros)) << id_bits) | (id - imin)) << up;
        return (f >> 32) * bins + ((f & 0xFFFFFFFFull) * bins >> 32);
    }
};

// A stretch beyond the capacity (split_geom's samples leave a chance of up to 1e-3 per sort that there is one; for the many more stretches of
// a sort in two distributions see deep_geom): the workgroup sorts it in memory.  from: cnt pairs; to_id, to_pk: the stretch's place in the plan.  Leaves the pairs in from.
//
// First by the count that sorts a stretch in LDS: bins of the pairs' places in the range, the pairs laid out bin by bin, and every pair
// ranked among its bin's; false, and the pairs as they were, where a bin holds too many for that.  lds: 2 * CAP words, part: THREADS / 64.
constexpr uint32_t kMemoryBin = 32;
template <int THREADS, int CAP>
__device__ bool count_in_memory(uint2* from, uint32_t* to_id, float* to_pk, int64_t cnt, const StretchRange& R, uint32_t* lds, uint32_t* part)
{
    constexpr int BINS = 2 * CAP, ROWS = BINS / THREADS, SIDE = 4;
    const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
    for (int i = tid; i < BINS; i += THREADS) lds[i] = 0u;
    __syncthreads();
    auto each = [&](auto load, auto use) {          // pairs of a thread side by side
        for (int64_t e0 = tid; e0 < cnt; e0 += SIDE * THREADS) {
            uint2 v[SIDE];
#pragma unroll
            for (int u = 0; u < SIDE; ++u) v[u] = load(e0 + u * THREADS < cnt ? e0 + u * THREADS : cnt - 1);
#pragma unroll
            for (int u = 0; u < SIDE; ++u)
                if (e0 + u * THREADS < cnt) use(v[u]);
        }
    };
    auto unordered = [&](int64_t e) { return from[e]; };
    auto binned = [&](int64_t e) { return make_uint2(__float_as_uint(to_pk[e]), to_id[e]); };
    auto bin_of = [&](uint2 v) { return (uint32_t)(R.place(v.x, v.y, BINS) >> 32); };
    each(unordered, [&](uint2 v) { atomicAdd(&lds[bin_of(v)], 1u); });
    __syncthreads();
    uint32_t* const row = lds + wave * (ROWS * 64) + lane;
    uint32_t run = 0u, big = 0u;
    for (int i = 0; i < ROWS; ++i) { const uint32_t c = row[i * 64]; run += c; big = c > big ? c : big; }
    run = wave_scan(run);
    if (lane == 63) part[wave] = run;
    if (__syncthreads_or(big > kMemoryBin)) return false;
    run = 0u;
    for (int w = 0; w < wave; ++w) run += part[w];
    for (int i = 0; i < ROWS; ++i) {
        const uint32_t c = row[i * 64], inc = wave_scan(c);
        row[i * 64] = run + inc - c;
        run += (uint32_t)__builtin_amdgcn_readlane((int)inc, 63);
    }
    __syncthreads();
    each(unordered, [&](uint2 v) {
        const uint32_t at = atomicAdd(&lds[bin_of(v)], 1u);
        to_pk[at] = __uint_as_float(v.x); to_id[at] = v.y;
    });
    __threadfence_block();
    __syncthreads();
    each(binned, [&](uint2 v) {                     // a bin's counter stands at its end now, the one before at its start
        const uint32_t b = bin_of(v), first = b ? lds[b - 1] : 0u, end = lds[b];
        uint32_t at = first;
        for (uint32_t q = first; q < end; ++q) {
            const uint2 o = binned(q);
            at += o.x < v.x || (o.x == v.x && o.y < v.y) ? 1u : 0u;
        }
        from[at] = v;
    });
    __threadfence_block();
    __syncthreads();
    return true;
}

// Otherwise by the 8-bit digits of (key, id) from the lowest up, stably; digits that do not vary are passed over.
template <int THREADS>
__device__ void sort_in_memory(uint2* from, uint32_t* to_id, float* to_pk, int64_t cnt, uint32_t vary_key, uint32_t vary_id, uint32_t* lds)
{
    constexpr int WAVES = THREADS / 64;
    uint32_t (*wcount)[256] = reinterpret_cast<uint32_t (*)[256]>(lds);     // [WAVES][256]
    uint32_t* const next = lds + WAVES * 256;                                // [256]
    uint32_t* const part = next + 256;
    const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
    bool in_plan = false;
    for (int pass = 0; pass < 8; ++pass) {
        const bool of_key = pass >= 4;
        const int shift = (pass & 3) * 8;
        if ((((of_key ? vary_key : vary_id) >> shift) & 255u) == 0u) continue;      // uniform
        auto load = [&](int64_t i) { return in_plan ? make_uint2(__float_as_uint(to_pk[i]), to_id[i]) : from[i]; };
        auto digit = [&](uint2 v) { return ((of_key ? v.x : v.y) >> shift) & 255u; };
        __syncthreads();
        if (tid < 256) next[tid] = 0u;
        __syncthreads();
        for (int64_t i = tid; i < cnt; i += THREADS) atomicAdd(&next[digit(load(i))], 1u);
        __syncthreads();
        uint32_t total;
        const uint32_t c = tid < 256 ? next[tid] : 0u;
        const uint32_t ex = block_scan<THREADS>(c, part, &total);
        if (tid < 256) next[tid] = ex;
        for (int64_t i0 = 0; i0 < cnt; i0 += THREADS) {
            for (int i = tid; i < WAVES * 256; i += THREADS) wcount[0][i] = 0u;
            __syncthreads();
            const bool ok = i0 + tid < cnt;
            const uint2 v = load(ok ? i0 + tid : cnt - 1);
            const uint32_t d = digit(v);
            uint64_t peers = __ballot(ok);
#pragma unroll
            for (int bit = 0; bit < 8; ++bit) {
                const bool set = (d >> bit) & 1u;
                const uint64_t m = __ballot(set);
                peers &= set ? m : ~m;
            }
            const uint32_t below = (uint32_t)__popcll(peers & ((1ull << lane) - 1ull));
            if (ok && below == 0u) wcount[wave][d] = (uint32_t)__popcll(peers);
            __syncthreads();
            if (tid < 256) {
                uint32_t run = next[tid];
                for (int w = 0; w < WAVES; ++w) { const uint32_t t = wcount[w][tid]; wcount[w][tid] = run; run += t; }
                next[tid] = run;
            }
            __syncthreads();
            if (ok) {
                const uint32_t dst = wcount[wave][d] + below;
                if (in_plan) from[dst] = v; else { to_pk[dst] = __uint_as_float(v.x); to_id[dst] = v.y; }
            }
            __syncthreads();
        }
        __threadfence_block();
        __syncthreads();
        in_plan = !in_plan;
    }
    if (in_plan)
        for (int64_t i = tid; i < cnt; i += THREADS) from[i] = make_uint2(__float_as_uint(to_pk[i]), to_id[i]);
    __threadfence_block();
    __syncthreads();
}

constexpr uint32_t kSplitRounds = 7;
constexpr uint32_t kSplitSmallGroup = 16;     // pairs that a bin may hold and still be put in order by comparing them

template <int THREADS>
struct StretchShared {
    uint32_t sums[THREADS / 64];
    uint32_t key_and, key_or, key_min, key_max, id_min, id_max, big, quantum;
    __device__ __forceinline__ void init() { key_and = 0xFFFFFFFFu; key_or = 0u; key_min = 0xFFFFFFFFu; key_max = 0u; id_min = 0xFFFFFFFFu; id_max = 0u; big = 0u; quantum = 0xFFFFFFFFu; }
};

// A pair's bin.  Where the range has far more keys than pairs, by the anchor itself, as evenly spread inside a stretch as any function of the key
// (near zero the key is not), and by the id behind it where the anchors are on a grid and near zero; else by 32 bits of its place in the range: those of (key - smallest key) without the low bits that no key differs in, and
// behind them the upper bits of the id, as far as there is room, scaled so that the range fills the bins.  Never decreasing in (key, id), also
// where the range ends in an anchor that is not finite: no number goes into the last bin.
struct StretchBins {
    uint32_t kmin, mult, last, id_mask;
    float pmin, scale, per_quantum, per_id;
    int low_zeros, key_up, id_down, id_up;
    bool by_value, by_quantum;
    __device__ __forceinline__ StretchBins(uint32_t kmin_, uint32_t kmax, uint32_t vary, int id_bits, int cnt, int bins)
        : kmin(kmin_), last((uint32_t)bins - 1u), low_zeros(vary ? __ffs((int)vary) - 1 : 0)
    {
        const uint32_t span = (kmax - kmin_) >> low_zeros;
        by_value = span >> 4 >= (uint32_t)cnt;
        by_quantum = false; per_quantum = per_id = 0.0f;
        pmin = split_key_to_float(kmin_);
        scale = (float)bins / (split_key_to_float(kmax) - pmin);
        const int room = span ? __clz((int)span) : 32;
        key_up = room & 31;                         // (no span: the key's part is zero)
        id_mask = room ? 0xFFFFFFFFu : 0u;
        id_down = room && id_bits > room ? id_bits - room : 0;
        id_up = id_bits < room ? room - id_bits : 0;
        const float top = (float)(span << key_up | (room ? 0xFFFFFFFFu >> (32 - room) : 0u)) + 1.0f;        // at most 2^32, at least 2^31
        mult = (uint32_t)((float)bins * (4294967296.0f / top) * 0.999999f);
    }
    // Equal anchors of a grid near zero, where one step of it is many times as many keys as elsewhere in the range: by the anchor, and by the id up to the next multiple
    // of 2^(quantum - 150).
    __device__ __forceinline__ bool may_have_quantum(uint32_t kmax) const
    {
        const int from = (int)(__float_as_uint(pmin) >> 23), to = (int)(__float_as_uint(split_key_to_float(kmax)) >> 23);      // (signs: 256 apart)
        return low_zeros >= 8 && (from - to > 1 || to - from > 1);
    }
    __device__ __forceinline__ static uint32_t quantum_of(uint32_t key)
    {
        const uint32_t u = __float_as_uint(split_key_to_float(key)), e = (u >> 23) & 255u, m = (u & 0x7FFFFFu) | (e ? 0x800000u : 0u);
        return m ? (e ? e : 1u) + (uint32_t)__ffs((int)m) - 1u : 0xFFFFFFFFu;
    }
    __device__ __forceinline__ void set_quantum(uint32_t quantum, uint32_t kmax, int id_bits, int bins)
    {
        per_quantum = ldexpf(1.0f, quantum < 277u ? 150 - (int)quantum : -127);
        const float quanta = (split_key_to_float(kmax) - pmin) * per_quantum;
        by_quantum = quanta < 4194304.0f;               // (else, or not a number: the ids would be lost behind so many)
        per_id = ldexpf(1.0f, -id_bits);
        if (by_quantum) scale = (float)bins / (quanta + 1.0f);
    }
    __device__ __forceinline__ uint32_t of(uint32_t key, uint32_t id) const
    {
        uint32_t b;
        if (by_quantum) b = (uint32_t)fminf(__builtin_fmaf(split_key_to_float(key) - pmin, per_quantum, (float)id * per_id) * scale, 65535.0f);      // uniform
        else if (by_value) b = (uint32_t)fminf((split_key_to_float(key) - pmin) * scale, 65535.0f);      // uniform
        else b = __umulhi((((key - kmin) >> low_zeros) << key_up) | (((id >> id_down) << id_up) & id_mask), mult);
        return b < last ? b : last;
    }
};

// The sort of one stretch in LDS: load(e, key, id) brings pair e of cnt <= THREADS * ITEMS, thread by thread e = i * THREADS + tid into key[i]
// and id[i], and rank[i] is its place in the order of (key, id).  ref: the key of any of the pairs; ids are below 2^id_bits.  buf: 2 * THREADS * ITEMS words,
// 16-byte aligned, which load may read and which are in use until the next barrier; S: initialised before a barrier; known(smallest key,
// largest key): called by thread 0.
// A bin's pairs are its group.  Where one is beyond kSplitSmallGroup (keys far from evenly spread, many equal ones) the pairs are counted once
// more by their exact places, the range of the ids included, and groups that are still too large are split into as many bins as they have
// pairs, again and again.
template <int THREADS, int ITEMS, typename LOAD, typename KNOWN>
__device__ __forceinline__ void stretch_ranks(uint32_t (&key)[ITEMS], uint32_t (&id)[ITEMS], int cnt, uint32_t ref, int id_bits, uint32_t* buf,
                                              StretchShared<THREADS>& S, uint32_t (&rank)[ITEMS], LOAD load, KNOWN known)
{
    constexpr int CAP = THREADS * ITEMS, WAVES = THREADS / 64;
    static_assert(ITEMS % 4 == 0, "the bins are scanned in quads");
    const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
    unsigned long long* const slot = reinterpret_cast<unsigned long long*>(buf);
    const auto lesser = [](uint32_t p, uint32_t q) { return p < q ? p : q; };
    const auto greater = [](uint32_t p, uint32_t q) { return p > q ? p : q; };
    uint32_t vary = 0u, k_min = 0xFFFFFFFFu, k_max = 0u;
#pragma unroll
    for (int i = 0; i < ITEMS; ++i) {
        key[i] = id[i] = 0u;
        if (i * THREADS < cnt) {                    // uniform
            load(i * THREADS + tid < cnt ? i * THREADS + tid : cnt - 1, key[i], id[i]);      // (the last pair once more: it changes none of these)
            vary |= key[i] ^ ref;
            k_min = lesser(k_min, key[i]); k_max = greater(k_max, key[i]);
        }
    }
    vary = wave_fold(vary, 0u, [](uint32_t p, uint32_t q) { return p | q; });
    k_min = wave_fold(k_min, 0xFFFFFFFFu, lesser); k_max = wave_fold(k_max, 0u, greater);
    if (lane == 63) { atomicOr(&S.key_or, vary); atomicMin(&S.key_min, k_min); atomicMax(&S.key_max, k_max); }
    auto clear = [&](int count) {               // whole rows of quads of the scan below
        const int quads = (count + 4 * THREADS - 1) / (4 * THREADS) * THREADS;
        for (int i = tid; i < quads; i += THREADS) reinterpret_cast<uint4*>(buf)[i] = make_uint4(0u, 0u, 0u, 0u);
    };
    __syncthreads();
    // First in four bins per pair, whose counts are bytes: a pair that is not among the first kSplitSmallGroup of its bin sees it, before a
    // byte overflows.
    const int words = cnt < CAP ? cnt : CAP;
    clear(words);
    __syncthreads();
    if (tid == 0) known(S.key_min, S.key_max);
    uint32_t seg[ITEMS];                        // first slot and size (upper half) of the group the pair belongs to (rank: its place there)
    {
        StretchBins B(S.key_min, S.key_max, S.key_or, id_bits, cnt, 4 * words);
        if (B.may_have_quantum(S.key_max)) {             // uniform
            uint32_t q = 0xFFFFFFFFu;
#pragma unroll
            for (int i = 0; i < ITEMS; ++i)
                if (i * THREADS < cnt) q = lesser(q, StretchBins::quantum_of(key[i]));
            q = wave_fold(q, 0xFFFFFFFFu, lesser);
            if (lane == 63) atomicMin(&S.quantum, q);
            __syncthreads();
            B.set_quantum(S.quantum, S.key_max, id_bits, 4 * words);
        }
        bool over = false;
#pragma unroll
        for (int i = 0; i < ITEMS; ++i) {
            seg[i] = 0u;
            if (i * THREADS < cnt) {                // uniform
                seg[i] = B.of(key[i], id[i]);
                const uint32_t shift = (seg[i] & 3u) * 8u;
                if (i * THREADS + tid < cnt) {
                    rank[i] = (atomicAdd(&buf[seg[i] >> 2], 1u << shift) >> shift) & 255u;
                    over |= rank[i] >= kSplitSmallGroup;
                }
            }
        }
        if (__any(over) && lane == 0) S.big = 1u;
    }
    __syncthreads();
    const bool many = S.big != 0u;              // uniform
    if (!many) {
        // the words' first slots behind the counts; a wavefront owns a stretch of whole rows of 64 quads of words
        const uint4* const quad = reinterpret_cast<const uint4*>(buf) + lane;
        uint4* const first = reinterpret_cast<uint4*>(buf + CAP) + lane;
        const int rows = (words + 4 * THREADS - 1) / (4 * THREADS);
        auto sums_of = [](const uint4& v) {
            uint4 r;
            r.x = __builtin_amdgcn_sad_u8(v.x, 0u, 0u); r.y = __builtin_amdgcn_sad_u8(v.y, 0u, r.x);
            r.z = __builtin_amdgcn_sad_u8(v.z, 0u, r.y); r.w = __builtin_amdgcn_sad_u8(v.w, 0u, r.z);
            return r;
        };
        uint32_t run = 0u;
        for (int i = 0; i < rows; ++i) run += sums_of(quad[(wave * rows + i) * 64]).w;
        run = wave_scan(run);
        if (lane == 63) S.sums[wave] = run;
        __syncthreads();
        run = 0u;
#pragma unroll
        for (int w = 0; w < WAVES; ++w) run += w < wave ? S.sums[w] : 0u;
        for (int i = 0; i < rows; ++i) {
            const uint4 sum = sums_of(quad[(wave * rows + i) * 64]);
            const uint32_t in = wave_scan(sum.w), ex = run + in - sum.w;
            first[(wave * rows + i) * 64] = make_uint4(ex, ex + sum.x, ex + sum.y, ex + sum.z);
            run += (uint32_t)__builtin_amdgcn_readlane((int)in, 63);
        }
        __syncthreads();
#pragma unroll
        for (int i = 0; i < ITEMS; ++i) {
            if (i * THREADS < cnt) {                // uniform
                const uint32_t counts = buf[seg[i] >> 2], shift = (seg[i] & 3u) * 8u;
                seg[i] = __builtin_amdgcn_sad_u8(counts & ((1u << shift) - 1u), 0u, buf[CAP + (seg[i] >> 2)]) | ((counts >> shift) & 255u) << 16;
            }
        }
        __syncthreads();
    }
    if (many) {
        uint32_t i_min = 0xFFFFFFFFu, i_max = 0u;
#pragma unroll
        for (int i = 0; i < ITEMS; ++i)
            if (i * THREADS < cnt) { i_min = lesser(i_min, id[i]); i_max = greater(i_max, id[i]); }
        i_min = wave_fold(i_min, 0xFFFFFFFFu, lesser); i_max = wave_fold(i_max, 0u, greater);
        if (lane == 63) { atomicMin(&S.id_min, i_min); atomicMax(&S.id_max, i_max); }
        int bins = 2 * cnt < CAP ? 2 * cnt : CAP;
        clear(bins);
        __syncthreads();
        uint32_t* const left = buf + CAP + tid; // behind the bins: the fraction inside the bin, its first 32 bits, of pair i at [i * THREADS]
        {
            const StretchRange R(S.key_min, S.key_max, S.id_min, S.id_max, S.key_or);
#pragma unroll
            for (int i = 0; i < ITEMS; ++i) {
                if (i * THREADS + tid < cnt) {
                    const unsigned long long place = R.place(key[i], id[i], (uint32_t)bins);
                    seg[i] = (uint32_t)(place >> 32);
                    left[i * THREADS] = (uint32_t)place;
                    rank[i] = atomicAdd(&buf[seg[i]], 1u);
                }
                __builtin_amdgcn_sched_barrier(0);      // (one at a time: seldom needed, and side by side they cost the registers of all that follows)
            }
        }
#pragma unroll 1
        for (uint32_t round = 1u; ; ++round) {
            // the bins' counts become their groups, for every pair: exclusive scan of the counts, in quads; a wavefront owns a stretch of whole
            // rows of 64 quads.  Start in the lower half of a word, count in the upper.
            __syncthreads();
            uint4* const quad = reinterpret_cast<uint4*>(buf) + lane;
            const int rows = (bins + 4 * THREADS - 1) / (4 * THREADS);
            uint32_t big = 0u, run = 0u;
            for (int i = 0; i < rows; ++i) {
                const uint4 v = quad[(wave * rows + i) * 64];
                big = greater(big, greater(greater(v.x, v.y), greater(v.z, v.w)));
                run += v.x + v.y + v.z + v.w;
            }
            run = wave_scan(run);
            if (lane == 63) S.sums[wave] = run;
            if (__any(big > kSplitSmallGroup) && lane == 0) S.big = round + 1u;
            __syncthreads();
            run = 0u;
#pragma unroll
            for (int w = 0; w < WAVES; ++w) run += w < wave ? S.sums[w] : 0u;
            for (int i = 0; i < rows; ++i) {
                const uint4 v = quad[(wave * rows + i) * 64];
                const uint32_t sum = v.x + v.y + v.z + v.w, in = wave_scan(sum), ex = run + in - sum;
                quad[(wave * rows + i) * 64] = make_uint4(ex | (v.x << 16), (ex + v.x) | (v.y << 16), (ex + v.x + v.y) | (v.z << 16), (ex + v.x + v.y + v.z) | (v.w << 16));
                run += (uint32_t)__builtin_amdgcn_readlane((int)in, 63);
            }
            const bool again = S.big == round + 1u;      // uniform
            __syncthreads();
#pragma unroll
            for (int i = 0; i < ITEMS; ++i)
                if (i * THREADS + tid < cnt) seg[i] = buf[seg[i]];
            __syncthreads();
            if (!again || round == kSplitRounds) break;
            // groups that are still large are split into as many bins as they have pairs: from here on a bin is a slot
            bins = cnt;
            clear(bins);
            __syncthreads();
#pragma unroll
            for (int i = 0; i < ITEMS; ++i) {
                if (i * THREADS + tid < cnt) {
                    const uint32_t n = seg[i] >> 16;
                    uint32_t bin = seg[i] & 0xFFFFu;
                    if (n > kSplitSmallGroup) {
                        const unsigned long long v = (unsigned long long)left[i * THREADS] * n;
                        bin += (uint32_t)(v >> 32);
                        left[i * THREADS] = (uint32_t)v;
                    }
                    rank[i] = atomicAdd(&buf[bin], 1u);
                    seg[i] = bin;
                }
                __builtin_amdgcn_sched_barrier(0);
            }
        }
    }
    // group by group into LDS; then a pair's place in its group by comparing, four pairs of a thread side by side
#pragma unroll
    for (int i = 0; i < ITEMS; ++i) {
        if (i * THREADS + tid < cnt) slot[(seg[i] & 0xFFFFu) + rank[i]] = ((unsigned long long)key[i] << 32) | id[i];
        else seg[i] = 0u;
    }
    __syncthreads();
#pragma unroll
    for (int i0 = 0; i0 < ITEMS; i0 += 4) {
        if (i0 * THREADS < cnt) {               // uniform
            uint32_t most = 0u;
#pragma unroll
            for (int i = i0; i < i0 + 4; ++i) { rank[i] = seg[i] & 0xFFFFu; most = seg[i] > most ? seg[i] : most; }
            most >>= 16;
            if (most < 2u) most = 0u;
            for (uint32_t q = 0; q < most; ++q) {
                unsigned long long o[4];
#pragma unroll
                for (int u = 0; u < 4; ++u) o[u] = slot[q < seg[i0 + u] >> 16 ? (seg[i0 + u] & 0xFFFFu) + q : (uint32_t)lane];
#pragma unroll
                for (int u = 0; u < 4; ++u) {
                    const unsigned long long me = ((unsigned long long)key[i0 + u] << 32) | id[i0 + u];
                    rank[i0 + u] += (q < seg[i0 + u] >> 16 && o[u] < me) ? 1u : 0u;
                }
            }
        }
    }
}

}  // namespace

}  // namespace laplex

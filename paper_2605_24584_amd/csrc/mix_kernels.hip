// LAPLEX^(r), y = sum_q w_q L(a_q, b_q) x, with all operators in the same launches (Sec. 7, "Learned anchor geometry in neural
// heads"), for operators whose merged sequence the two-launch sort takes.
//
// One side of an operator is shorter (a head over a vocabulary: few inputs, many outputs).  Nothing per operator is ever as
// large as the long side times the batch:
//   short -> long   the rows of the short side are scanned in sorted order into, per row s, the inclusive decayed sums
//                   F_s (rows at or before s) and R_s (rows at or after s); a row of the long side at anchor p is then
//                   exp(-(p - p_lo)) F_lo + exp(-(p_hi - p)) R_hi of its two neighbours (Thm "Dual reduction", App. B.3), and
//                   one kernel adds that up over the operators, in registers (k_mix_scan_reduce, k_mix_scan_down, k_mix_gather)
//   long -> short   the other way round: the long rows between two short anchors are folded into two sums, decayed to the one
//                   above and to the one below (k_mix_fold), these are scanned like rows of the short side, and the same
//                   kernel in its other form adds the operators up
// Anchor gradients are row products of the caller's matrices with the strict sums, formed where the sums are in registers.
//
// The batch is cut into slabs of up to 32 columns, workgroup % slabs = slab: with eight slabs a slab's rows F, R of the
// operator at hand (2 x 128 bytes x 4096 short rows = 1 MB) stay in the L2 of one chiplet while its workgroups walk through
// the operators together.
//
// Measured (MI355X, forward + backward): 16 operators of 32000 x 4096, batch 256: 2.97 ms one operator after the other on four
// streams (320 launches, 4 GB of per-operator products and strict sums of the long side written and read) -> 0.55 ms in 17
// launches; 16 of 1000 x 2048: 0.31 ms (k_small) -> 0.149.  Of the former 0.18 ms are k_mix_gather, which reads 2 x 16 rows per
// output at 10 to 13 TB/s, most of it from the L2, 0.09 k_mix_fold (5.6 TB/s of the long rows), 0.12 the scans of what it
// leaves, 0.09 the sort and the plan.
#include "laplex_internal.h"

namespace laplex {

namespace {

constexpr int kMixThreads = 256;
constexpr int kMixWaves = kMixThreads / 64;
constexpr int kMixItems = 8;                             // rows per row-lane of the scan kernels
constexpr int kMixTileMax = kMixWaves * 64 * kMixItems;  // rows of a workgroup with one lane across the batch
constexpr int kIndexThreads = 512;
constexpr int kIndexTile = kIndexThreads * 4;

template <typename T>
__device__ __forceinline__ T* shift_bytes(T* p, int64_t bytes)
{
    return reinterpret_cast<T*>(reinterpret_cast<uintptr_t>(p) + (uintptr_t)bytes);
}

// dst[0 .. VEC) <- ok ? src : 0 (not read if !ok)
template <int VEC>
__device__ __forceinline__ void load_cols(float* dst, const float* src, bool ok)
{
    if (VEC == 4) {
        const float4 t = ok ? *reinterpret_cast<const float4*>(src) : make_float4(0.0f, 0.0f, 0.0f, 0.0f);
        dst[0] = t.x; dst[1] = t.y; dst[2] = t.z; dst[3] = t.w;
    } else {
        dst[0] = ok ? src[0] : 0.0f;
    }
}

template <int VEC>
__device__ __forceinline__ void store_cols(float* dst, const float* src)
{
    if (VEC == 4) *reinterpret_cast<float4*>(dst) = make_float4(src[0], src[1], src[2], src[3]);
    else dst[0] = src[0];
}

// Row j of the sorted short list, clamped to it.
__device__ __forceinline__ int clamp_row(int j, int m) { return j < 0 ? 0 : (j < m ? j : m - 1); }

// The sort's order of the anchors, not-a-numbers included: what is counted and searched by it is consistent whatever they hold.
__device__ __forceinline__ uint32_t order_of(float f)
{
    const uint32_t u = __float_as_uint(f);
    return u ^ ((uint32_t)((int32_t)u >> 31) | 0x80000000u);
}

// ---------------------------------------------------------------------------
// From the merged order of an operator: its short side as a list in sorted order, the intervals' bounds, and for every row of the
// long side how many short anchors lie strictly below it, how many at or below it, and its place among the long rows.  A
// workgroup takes 2048 merged positions and has to know the short ones before them: up to kIndexRecount such tiles it counts them
// itself (a few dozen KB of ids from the L2), beyond that a launch before it leaves every tile's count (the plan after the sort, us,
// without / with it: 16 x 36096 positions 47 / 52, 2 x 501000 105 / 88).
// ---------------------------------------------------------------------------
constexpr int kIndexRecount = 32;

__global__ void __launch_bounds__(kIndexThreads)
k_mix_count(const MixPath A)
{
    __shared__ int total[kIndexThreads / 64];
    const int64_t op = blockIdx.y;
    const uint32_t* ids = shift_bytes(A.ids, op * A.op_ws);
    int count = 0;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const int j = blockIdx.x * kIndexTile + i * kIndexThreads + threadIdx.x;
        if (j < A.N && (ids[j] >= (uint32_t)A.k) == (A.short_b != 0)) ++count;
    }
#pragma unroll
    for (int m = 32; m >= 1; m >>= 1) count += __shfl_xor(count, m);
    if ((threadIdx.x & 63) == 0) total[threadIdx.x >> 6] = count;
    __syncthreads();
    if (threadIdx.x == 0) {
        for (int w = 1; w < kIndexThreads / 64; ++w) count += total[w];
        A.counts[op * gridDim.x + blockIdx.x] = (uint32_t)count;
    }
}

// One tile, by a workgroup of kIndexThreads; `before`: the threads' parts of the number of short positions before it.  Returns those in it.
__device__ __forceinline__ int index_tile(const MixPath& A, int64_t op, int tile, int before_part)
{
    __shared__ int before[kIndexThreads / 64], total[kIndexThreads / 64];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const uint32_t* ids = shift_bytes(A.ids, op * A.op_ws);
    const float* pk = shift_bytes(A.pk, op * A.op_ws);
    const uint32_t k = (uint32_t)A.k;
    const bool short_b = A.short_b != 0;
    auto is_short = [&](uint32_t id) { return (id >= k) == short_b; };
    const int base = tile * kIndexTile;
    int count = before_part;
#pragma unroll
    for (int m = 32; m >= 1; m >>= 1) count += __shfl_xor(count, m);

    const int j0 = base + tid * 4;
    uint32_t id[4];
    int mine = 0;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        id[i] = j0 + i < A.N ? ids[j0 + i] : 0xFFFFFFFFu;
        mine += j0 + i < A.N && is_short(id[i]) ? 1 : 0;
    }
    int incl = mine;
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) { const int o = __shfl_up(incl, d); if (lane >= d) incl += o; }
    if (lane == 63) total[wave] = incl;
    if (lane == 0) before[wave] = count;
    __syncthreads();
    int s = incl - mine;
#pragma unroll
    for (int w = 0; w < kIndexThreads / 64; ++w) s += before[w] + (w < wave ? total[w] : 0);

    uint32_t* srow = A.srow + op * A.m;
    float* sp = A.sp + op * A.m;
    uint32_t* tied = A.tied + op * A.m;
    uint32_t* equals = A.equals + op * A.m;
    uint32_t* bound = A.bound + op * (A.m + 2);
    uint4* recs = A.recs + op * A.l;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const int j = j0 + i;
        if (j >= A.N) break;
        const float p = pk[j + 1];
        const uint32_t key = order_of(p);
        // Equal keys, in the stable order: outputs first, then inputs.  [a0, b0): the run; f0: its first input.
        int a0 = j, b0 = j + 1, f0 = 0;
        const bool run = order_of(pk[j]) == key || order_of(pk[j + 2]) == key;
        if (run) {
            a0 = 0;
            for (int hi = j; a0 < hi;) { const int mid = (a0 + hi) >> 1; if (order_of(pk[mid + 1]) < key) a0 = mid + 1; else hi = mid; }
            for (int hi = A.N; b0 < hi;) { const int mid = (b0 + hi) >> 1; if (order_of(pk[mid + 1]) <= key) b0 = mid + 1; else hi = mid; }
            f0 = a0;
            for (int hi = b0; f0 < hi;) { const int mid = (f0 + hi) >> 1; if (ids[mid] < k) f0 = mid + 1; else hi = mid; }
        }
        if (is_short(id[i])) {
            int not_above = j - s, first = 0, equal = 0;  // long rows at or below this anchor; 1 + first short row of the run; long rows in it
            if (run) {
                const int head = short_b ? s - (j - f0) : s - (j - a0);
                if (!short_b) not_above = b0 - head - (f0 - a0);
                equal = short_b ? f0 - a0 : b0 - f0;
                first = equal > 0 ? 1 + head : 0;
            }
            srow[s] = short_b ? id[i] - k : id[i];
            sp[s] = p;
            tied[s] = (uint32_t)first;
            equals[s] = (uint32_t)equal;
            bound[s + 1] = (uint32_t)not_above;
            ++s;
        } else {
            int lo = s, hi = s;
            if (run) {
                if (short_b) hi = s + (b0 - f0);
                else lo = s - (f0 - a0);
            }
            recs[short_b ? id[i] : id[i] - k] = make_uint4((uint32_t)lo, (uint32_t)hi, (uint32_t)(j - s), 0u);
        }
    }
    if (tile == 0 && tid == 0) { bound[0] = 0u; bound[A.m + 1] = (uint32_t)A.l; }
    int here = 0;
#pragma unroll
    for (int w = 0; w < kIndexThreads / 64; ++w) here += total[w];
    return here;
}

__global__ void __launch_bounds__(kIndexThreads)
k_mix_index(const MixPath A)
{
    const int tid = threadIdx.x;
    const int64_t op = blockIdx.y;
    const uint32_t* ids = shift_bytes(A.ids, op * A.op_ws);
    auto is_short = [&](uint32_t id) { return (id >= (uint32_t)A.k) == (A.short_b != 0); };
    const int base = blockIdx.x * kIndexTile;
    int count = 0;
    if (A.counted) {
        for (int q = tid; q < (int)blockIdx.x; q += kIndexThreads) count += (int)A.counts[op * gridDim.x + q];
    } else {                                              // (base is a multiple of 2048 and the ids start on 256 bytes)
        for (int j1 = tid * 4; j1 < base; j1 += 8 * kIndexTile) {
            uint4 v[8];
#pragma unroll
            for (int q = 0; q < 8; ++q) v[q] = *reinterpret_cast<const uint4*>(ids + (j1 + q * kIndexTile < base ? j1 + q * kIndexTile : 0));
#pragma unroll
            for (int q = 0; q < 8; ++q) {
                const int here = (is_short(v[q].x) ? 1 : 0) + (is_short(v[q].y) ? 1 : 0) + (is_short(v[q].z) ? 1 : 0) + (is_short(v[q].w) ? 1 : 0);
                count += j1 + q * kIndexTile < base ? here : 0;
            }
        }
    }
    index_tile(A, op, blockIdx.x, count);
}


// Second launch of the plan: the long rows' decays to their short neighbours (rows in the caller's order for the gather, in sorted
// order for the fold), and the fold's tasks.
__device__ __forceinline__ void make_record(const MixPath& A, int64_t op, int i)
{
    const int m = A.m;
    const float* sp = A.sp + op * m;
    const uint32_t* bound = A.bound + op * (m + 2);
    uint2* tasks = A.tasks + op * A.task_count;
    // the tasks of interval c, which holds the sorted rows first .. end, start at this one
    auto first_task = [&](int c, int first) { return c + first / kMixTaskRows; };
    if (i < A.l) {
        const uint4 r = A.recs[op * A.l + i];
        const int lo = (int)r.x;
        const float p = A.long_anchor[op * A.l + i];
        const float el = lo > 0 ? expf(-(p - sp[lo - 1])) : 0.0f;
        const float er = lo < m ? expf(-(sp[lo] - p)) : 0.0f;
        A.recs[op * A.l + i] = make_uint4(r.x, r.y, __float_as_uint(el), __float_as_uint(er));
        const bool equal = r.x != r.y;
        A.sorted[op * A.l + r.z] = make_uint4((uint32_t)i, __float_as_uint(el), equal ? 0u : __float_as_uint(er), equal ? 1u : 0u);
        const int first = (int)bound[lo], end = (int)bound[lo + 1], at = (int)r.z;      // every 32nd row of an interval writes a task
        if ((at - first) % kMixTaskRows == 0)
            tasks[first_task(lo, first) + (at - first) / kMixTaskRows] = make_uint2((uint32_t)at, (uint32_t)(end - at < kMixTaskRows ? end - at : kMixTaskRows));
    }
    if (i <= m) {
        const int first = (int)bound[i], end = (int)bound[i + 1], t0 = first_task(i, first);
        A.slots[op * (m + 1) + i] = make_uint2((uint32_t)t0, (uint32_t)(end - first));
        // the room behind them, at most one task, and behind the last interval's
        const int t1 = i < m ? first_task(i + 1, end) : A.task_count;
        for (int t = t0 + (end - first + kMixTaskRows - 1) / kMixTaskRows; t < t1; ++t) tasks[t] = make_uint2(0u, 0u);
    }
}

__device__ __forceinline__ uint32_t* index_word(const MixPath& A, int64_t op) { return shift_bytes(A.counters, op * A.op_ws) + kPlanIndexWord; }

__global__ void __launch_bounds__(kMixThreads)
k_mix_records(const MixPath A)
{
    make_record(A, blockIdx.y, blockIdx.x * kMixThreads + threadIdx.x);
    if (blockIdx.x == 0 && threadIdx.x == 0) *index_word(A, blockIdx.y) = kMixIndexed + (uint32_t)A.operators;
}

// All of it for one operator, by one workgroup, if it is not there: a kept plan of this sum costs the look at the word (16 x (9000 x
// 1000), batch 8, a product on a kept plan: 21 us without, 22 with), one that was built by other calls a walk over its tiles.
__global__ void __launch_bounds__(kIndexThreads)
k_mix_replan(const MixPath A)
{
    const int64_t op = blockIdx.x;
    if (*index_word(A, op) == kMixIndexed + (uint32_t)A.operators) return;      // uniform
    int before = 0;
    for (int tile = 0; tile * kIndexTile < A.N; ++tile) {
        before += index_tile(A, op, tile, threadIdx.x == 0 ? before : 0);
        __syncthreads();
    }
    const int items = A.l > A.m + 1 ? A.l : A.m + 1;
    for (int i = threadIdx.x; i < items; i += kIndexThreads) make_record(A, op, i);
    __syncthreads();
    if (threadIdx.x == 0) *index_word(A, op) = kMixIndexed + (uint32_t)A.operators;
}

// ---------------------------------------------------------------------------
// Fold: a row-lane takes one task, a few consecutive long rows of an interval in sorted order, and adds them up with the two
// decays of their records.  Every row is read once per operator; what leaves is two rows per interval.  With 64 lanes across the
// batch (UNI) a task is a wavefront's: its records are scalars, and no row-lane waits for a longer neighbour (16 operators of
// 32000 x 4096, batch 256: 140 us with eight tasks of 32 columns a wavefront, busy with the longest of the eight).
// ---------------------------------------------------------------------------
template <int VEC, bool UNI>
__global__ void __launch_bounds__(kMixThreads)
k_mix_fold(const MixPath A, const float* __restrict__ v, int64_t ldv, int lanes, int spans)
{
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int64_t op = blockIdx.y;
    const int span = (int)blockIdx.x % spans, chunk = (int)blockIdx.x / spans;
    const int c = UNI ? lane : lane & (lanes - 1);
    const int t = UNI ? chunk * kMixWaves + wave : (chunk * kMixWaves + wave) * (64 / lanes) + lane / lanes;
    if (t >= A.task_count) return;
    const int64_t col = ((int64_t)span * lanes + c) * VEC;
    const bool col_ok = col < A.batch;
    const uint2 task = A.tasks[op * A.task_count + t];
    const int n = (int)task.y;
    if (n == 0) return;                                   // (nobody reads the sums of an empty task)
    const uint4* recs = A.sorted + op * A.l + task.x;
    float up[VEC], down[VEC], eq[VEC];
    uint32_t any = 0u;
#pragma unroll
    for (int e = 0; e < VEC; ++e) up[e] = down[e] = eq[e] = 0.0f;
    constexpr int AHEAD = 8;
    for (int i0 = 0; i0 < n; i0 += AHEAD) {
        uint4 rec[AHEAD];
        float x[AHEAD][VEC];
#pragma unroll
        for (int i = 0; i < AHEAD; ++i) rec[i] = recs[i0 + i < n ? i0 + i : n - 1];
#pragma unroll
        for (int i = 0; i < AHEAD; ++i) load_cols<VEC>(x[i], v + (int64_t)rec[i].x * ldv + col, col_ok && i0 + i < n);
#pragma unroll
        for (int i = 0; i < AHEAD; ++i) {
            if (UNI && i0 + i >= n) break;
            const float el = __uint_as_float(rec[i].y), er = __uint_as_float(rec[i].z);
#pragma unroll
            for (int e = 0; e < VEC; ++e) down[e] += el * x[i][e];
            if (rec[i].w != 0u) {                         // equal to the short anchor above: kept apart (no 0 * x: x may be infinite)
                any = 1u;
#pragma unroll
                for (int e = 0; e < VEC; ++e) eq[e] += x[i][e];
            } else {
#pragma unroll
                for (int e = 0; e < VEC; ++e) up[e] += er * x[i][e];
            }
        }
    }
    if (col >= (int64_t)A.slabs * A.width) return;        // (columns that fill up the last slab are written, as zeros)
    const int64_t slot = (op * A.slabs + (int64_t)(col / A.width)) * A.task_count + t;
    const int in = (int)(col % A.width);
    store_cols<VEC>(A.folds + slot * (2 * A.width) + in, up);
    store_cols<VEC>(A.folds + slot * (2 * A.width) + A.width + in, down);
    if (any) store_cols<VEC>(A.equal + slot * A.width + in, eq);
}

// ---------------------------------------------------------------------------
// Join: the sums of an interval's tasks, added up in the place of its first task's, so that the scans read one of them.  Most
// intervals have a single task: a workgroup looks through some of them, shares its row-lanes among those that have more, and sets all
// of them to work on one with very many (few short rows between many long ones, or all of them between two).  With the scans adding up
// the tasks themselves, interval after interval, 100 x 100000, batch 8, a product on a kept plan took 289 us, now 36.
// ---------------------------------------------------------------------------
constexpr int kJoinIntervals = 256, kJoinAlone = 32;

template <int VEC, int THREADS>
__global__ void __launch_bounds__(THREADS)
k_mix_join(const MixPath A, int per)
{
    static_assert(THREADS >= kJoinIntervals, "an interval per thread");
    __shared__ int list[kJoinIntervals], count;
    __shared__ __align__(16) float part[THREADS * VEC];
    const int tid = threadIdx.x;
    const int64_t op = blockIdx.y;
    const int slab = (int)blockIdx.x % A.slabs, i0 = (int)blockIdx.x / A.slabs * per;
    const uint2* slots = A.slots + op * (A.m + 1);
    if (tid == 0) count = 0;
    __syncthreads();
    if (tid < per && i0 + tid <= A.m && slots[i0 + tid].y > (uint32_t)kMixTaskRows) list[atomicAdd(&count, 1)] = i0 + tid;
    __syncthreads();
    const int found = count;
    if (found == 0) return;                               // uniform
    // columns: those of the folds (2 * width), then those of the equal rows (width)
    const int row = 3 * A.width, lanes = row / VEC, side = THREADS / lanes;
    const int c = tid % lanes * VEC, rl = tid / lanes;    // (rl >= side: lanes that make no whole row)
    const bool folds = c < 2 * A.width;
    const int stride = folds ? 2 * A.width : A.width;
    float* const at = folds ? A.folds + (op * A.slabs + slab) * (int64_t)A.task_count * (2 * A.width) + c
                            : A.equal + (op * A.slabs + slab) * (int64_t)A.task_count * A.width + (c - 2 * A.width);
    const int group = found < side ? side / found : 1;    // row-lanes of an interval
    struct Range { int first, end; bool many; };
    auto range = [&](int q) {
        const int i = list[q];
        const uint2 slot = slots[i];
        Range r;
        r.first = (int)slot.x;
        r.end = r.first + ((int)slot.y + kMixTaskRows - 1) / kMixTaskRows;
        r.many = r.end - r.first > kJoinAlone * group;
        if (!folds) {                                     // (they come last in the interval; tasks without any have not written theirs)
            const bool tied = i < A.m && A.tied[op * A.m + i] == (uint32_t)i + 1u;
            r.first = tied ? r.first + (int)(slot.y - A.equals[op * A.m + i]) / kMixTaskRows : r.end;
        }
        return r;
    };
    auto add_up = [&](float* s, int first, int end, int step) {
        constexpr int AHEAD = 4;
#pragma unroll
        for (int e = 0; e < VEC; ++e) s[e] = 0.0f;
        for (int t = first; t < end; t += AHEAD * step) {
            float v[AHEAD][VEC];
#pragma unroll
            for (int i = 0; i < AHEAD; ++i) load_cols<VEC>(v[i], at + (int64_t)(t + i * step) * stride, t + i * step < end);
#pragma unroll
            for (int i = 0; i < AHEAD; ++i)
#pragma unroll
                for (int e = 0; e < VEC; ++e) s[e] += v[i][e];
        }
    };
    // the row-lanes at first .. first + lanes hold parts of a sum: the first of them adds them up
    auto finish = [&](const Range& r, int first, int lanes_of_it) {
        float s[VEC];
#pragma unroll
        for (int e = 0; e < VEC; ++e) s[e] = 0.0f;
        for (int u = first; u < first + lanes_of_it; ++u) {
#pragma unroll
            for (int e = 0; e < VEC; ++e) s[e] += part[u * row + c + e];
        }
        store_cols<VEC>(at + (int64_t)r.first * stride, s);
    };
    for (int q0 = 0; q0 < found; q0 += side / group) {
        const int q = q0 + rl / group;
        const bool mine = rl < side / group * group && q < found;
        const Range r = range(mine ? q : 0);
        const bool work = mine && !r.many && r.end - r.first > 1;
        float s[VEC];
        if (work) add_up(s, r.first + rl % group, r.end, group);
        if (group == 1) {                                 // uniform
            if (work) store_cols<VEC>(at + (int64_t)r.first * stride, s);
            continue;
        }
        if (work) store_cols<VEC>(part + rl * row + c, s);
        __syncthreads();
        if (work && rl % group == 0) finish(r, rl, group);
        __syncthreads();
    }
    for (int q = 0; q < found; ++q) {
        const Range r = range(q);
        if (!r.many) continue;                            // uniform
        if (rl < side) {
            float s[VEC];
            add_up(s, r.first + rl, r.end, side);
            store_cols<VEC>(part + rl * row + c, s);
        }
        __syncthreads();
        if (rl == 0 && r.first < r.end) finish(r, 0, side);
        __syncthreads();
    }
}

// What the scans add at the kMixItems rows from j0 on of the short side: forward and backward the row itself; or (FOLDED) forward
// the folded rows of the interval below it, backward those of the interval above it.
template <int VEC, bool FOLDED>
__device__ __forceinline__ void load_rows(const MixPath& A, int64_t op, int slab, int c, int j0, const float* __restrict__ v, int64_t ldv,
                                          float (*f)[VEC], float (*b)[VEC])
{
    if constexpr (!FOLDED) {
        const int64_t col = (int64_t)slab * A.width + c * VEC;
        const uint32_t* srow = A.srow + op * A.m;
#pragma unroll
        for (int i = 0; i < kMixItems; ++i) {
            const int j = j0 + i;
            load_cols<VEC>(f[i], v + (int64_t)srow[j < A.m ? j : A.m - 1] * ldv + col, col < A.batch && j < A.m);
        }
    } else {
        const float* folds = A.folds + (op * A.slabs + slab) * (int64_t)A.task_count * (2 * A.width) + c * VEC;
        const uint2* slots = A.slots + op * (A.m + 1);
        uint2 slot[kMixItems + 1];
#pragma unroll
        for (int i = 0; i <= kMixItems; ++i) {
            slot[i] = slots[j0 + i <= A.m ? j0 + i : A.m];
            if (j0 + i > A.m) slot[i].y = 0u;
        }
#pragma unroll
        for (int i = 0; i < kMixItems; ++i) load_cols<VEC>(f[i], folds + (int64_t)slot[i].x * (2 * A.width), j0 + i < A.m && slot[i].y > 0u);
#pragma unroll
        for (int i = 0; i < kMixItems; ++i) load_cols<VEC>(b[i], folds + (int64_t)slot[i + 1].x * (2 * A.width) + A.width, slot[i + 1].y > 0u);
    }
}
// The long rows equal to short anchor j, to be added to the forward value (they are in the interval of the first such anchor).
template <int VEC>
__device__ __forceinline__ void load_equal(const MixPath& A, int64_t op, int slab, int c, int j, float* t)
{
    const float* equal = A.equal + (op * A.slabs + slab) * (int64_t)A.task_count * A.width + c * VEC;
    const uint2 slot = A.slots[op * (A.m + 1) + j];
    load_cols<VEC>(t, equal + (int64_t)(slot.x + (slot.y - A.equals[op * A.m + j]) / kMixTaskRows) * A.width, true);
}

// ---------------------------------------------------------------------------
// Scan of the short side, first launch: per tile and slab the sum of its rows decayed to the tile's last row and to its first
// one, as weighted sums (a row's two weights are one exponential of an anchor difference each, taken once per workgroup).
// ---------------------------------------------------------------------------
template <int VEC, bool FOLDED>
__global__ void __launch_bounds__(kMixThreads)
k_mix_scan_reduce(const MixPath A, const float* __restrict__ v, int64_t ldv)
{
    constexpr int SUMS = FOLDED ? kMixSums : 2;
    __shared__ float wf[kMixTileMax], wb[kMixTileMax];
    __shared__ float part[SUMS][kMixWaves][kMixWidth];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int64_t op = blockIdx.y;
    const float* sp = A.sp + op * A.m;
    const int m = A.m;
    const int slab = (int)blockIdx.x % A.slabs, tile = (int)blockIdx.x / A.slabs;
    const int bv = A.width / VEC, rv = 64 / bv;
    const int c = lane & (bv - 1), rl = wave * rv + lane / bv;
    const int rows = kMixWaves * rv * kMixItems;
    const int base = tile * rows, last = clamp_row(base + rows - 1, m);
    float vf[kMixItems][VEC], vb[FOLDED ? kMixItems : 1][VEC];
    load_rows<VEC, FOLDED>(A, op, slab, c, base + rl * kMixItems, v, ldv, vf, vb);
    float eq[VEC];                                        // rows equal to the tile's last anchor: not part of its strict sum
#pragma unroll
    for (int e = 0; e < VEC; ++e) eq[e] = 0.0f;
    if (FOLDED) {
        const uint32_t last_run = A.tied[op * m + last];
#pragma unroll
        for (int i = 0; i < kMixItems; ++i) {
            const int j = base + rl * kMixItems + i;
            if (j < m && A.tied[op * m + j] == (uint32_t)j + 1u) {
                float t[VEC];
                load_equal<VEC>(A, op, slab, c, j, t);
#pragma unroll
                for (int e = 0; e < VEC; ++e) { if (last_run == (uint32_t)j + 1u) eq[e] = t[e]; else vf[i][e] += t[e]; }
            }
        }
    }
    const float p_first = sp[base], p_last = sp[last];
    for (int q = tid; q < rows; q += kMixThreads) {
        const float p = sp[clamp_row(base + q, m)];
        wf[q] = expf(-(p_last - p));
        wb[q] = expf(-(p - p_first));
    }
    __syncthreads();
    float f[VEC], b[VEC];
#pragma unroll
    for (int e = 0; e < VEC; ++e) f[e] = b[e] = 0.0f;
#pragma unroll
    for (int i = 0; i < kMixItems; ++i) {
        const float x = wf[rl * kMixItems + i], y = wb[rl * kMixItems + i];
#pragma unroll
        for (int e = 0; e < VEC; ++e) { f[e] += x * vf[i][e]; b[e] += y * (FOLDED ? vb[FOLDED ? i : 0][e] : vf[i][e]); }
    }
    for (int d = bv; d < 64; d <<= 1) {
#pragma unroll
        for (int e = 0; e < VEC; ++e) {
            f[e] += __shfl_xor(f[e], d); b[e] += __shfl_xor(b[e], d);
            if (FOLDED) eq[e] += __shfl_xor(eq[e], d);
        }
    }
    if (lane < bv) {
#pragma unroll
        for (int e = 0; e < VEC; ++e) {
            part[0][wave][c * VEC + e] = f[e]; part[1][wave][c * VEC + e] = b[e];
            if (FOLDED) part[SUMS - 1][wave][c * VEC + e] = eq[e];
        }
    }
    __syncthreads();
    if (tid < 2 * A.width) {
        const int dir = tid / A.width, w = tid % A.width;
        float* at = A.sums + (((op * A.slabs + slab) * kMixSums + dir) * A.tiles + tile) * A.width + w;
        float s = 0.0f;
#pragma unroll
        for (int u = 0; u < kMixWaves; ++u) s += part[dir][u][w];
        if (FOLDED && dir == 0) {                         // without, then with the rows equal to the last anchor (of weight 1)
            at[(int64_t)2 * A.tiles * A.width] = s;
            float t = 0.0f;
#pragma unroll
            for (int u = 0; u < kMixWaves; ++u) t += part[SUMS - 1][u][w];
            s += t;
        }
        *at = s;
    }
}

// ---------------------------------------------------------------------------
// Second launch: a tile adds up the other tiles' sums itself, each brought to the tile by one exponential of an anchor
// difference, scans its row-lanes, and walks its rows in both directions.
// Rows of the short side: fr[op][slab][row] = (F_row | R_row), 2 x width floats.  FOLDED: F_j holds the long rows not above short
// anchor j, R_j those above it, E_j those strictly below; products F + R and strict sums R - E leave row by row, or as dots with
// the rows of u.  E is never F with the equal rows taken out again, which would keep no digit of a strict sum that is 2^-24 of
// them: it is the forward sum at the first row of a run of equal short anchors before they are added, and stays over the run.  A
// row-lane that starts inside a run takes it from the row-lane with the run's first row or, where the run reaches back over the
// tile's edge, from the tile sums, with the strict one for the tile with that row (the tiles in between hold rows of the run alone).
// ---------------------------------------------------------------------------
template <int VEC, bool FOLDED>
__global__ void __launch_bounds__(kMixThreads)
k_mix_scan_down(const MixPath A, const float* __restrict__ v, int64_t ldv, const MixFolded O)
{
    __shared__ float dec[kMixTileMax + 1];                // dec[q]: decay between rows base + q - 1 and base + q
    __shared__ float part[FOLDED ? 5 : 4][kMixWaves][32]; // wavefront totals and carries, forward and backward; strict carries
    __shared__ __align__(16) float run_e[FOLDED ? kMixThreads * VEC : 1];      // per row-lane: E of the run at its last row
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int64_t op = blockIdx.y;
    const int m = A.m;
    const float* sp = A.sp + op * m;
    const int slab = (int)blockIdx.x % A.slabs, tile = (int)blockIdx.x / A.slabs;
    const int bv = A.width / VEC, rv = 64 / bv;
    const int c = lane & (bv - 1), r = lane / bv, rl = wave * rv + r;
    const int rows = kMixWaves * rv * kMixItems;
    const int base = tile * rows;
    const int j0 = base + rl * kMixItems;
    float vf[kMixItems][VEC], vr[FOLDED ? kMixItems : 1][VEC];
    load_rows<VEC, FOLDED>(A, op, slab, c, j0, v, ldv, vf, vr);
    // rows of the long side equal to a short anchor: 1 + the first short row with it, or 0
    uint32_t tie[FOLDED ? kMixItems : 1];
    if (FOLDED) {
#pragma unroll
        for (int i = 0; i < kMixItems; ++i) tie[FOLDED ? i : 0] = j0 + i < m ? A.tied[op * m + j0 + i] : 0u;
    }
    auto is_first = [&](int i) { return FOLDED && tie[FOLDED ? i : 0] == (uint32_t)(j0 + i) + 1u; };
    auto pos = [&](int j) { return sp[clamp_row(j, m)]; };
    for (int q = tid; q <= rows; q += kMixThreads) dec[q] = expf(-(pos(base + q) - pos(base + q - 1)));

    // the tiles before and after, spread over the row-lanes
    float Fc[VEC], Rc[VEC], Ec[VEC];
#pragma unroll
    for (int e = 0; e < VEC; ++e) Fc[e] = Rc[e] = Ec[e] = 0.0f;
    // the tile that holds the first row of the run that this tile starts inside of, or -1
    const uint32_t open_run = FOLDED ? A.tied[op * m + base] : 0u;
    const int run_tile = open_run != 0u && (int)open_run - 1 < base ? ((int)open_run - 1) / rows : -1;
    {
        const float p_before = pos(base - 1), p_after = pos(base + rows);
        const float* sf = A.sums + ((op * A.slabs + slab) * kMixSums) * (int64_t)A.tiles * A.width + c * VEC;
        const float* sb = sf + (int64_t)A.tiles * A.width;
        for (int u = rl; u < A.tiles; u += kMixWaves * rv) {
            if (u == tile) continue;
            const float w = u < tile ? expf(-(p_before - pos((u + 1) * rows - 1))) : expf(-(pos(u * rows) - p_after));
            float t[VEC];                                 // (read whatever the decay: 0 * NaN and 0 * inf are NaN, as in the dense product)
            load_cols<VEC>(t, (u < tile ? sf : sb) + (int64_t)u * A.width, true);
#pragma unroll
            for (int e = 0; e < VEC; ++e) { if (u < tile) Fc[e] += w * t[e]; else Rc[e] += w * t[e]; }
            if (FOLDED && u <= run_tile) {
                if (u == run_tile) load_cols<VEC>(t, sb + ((int64_t)A.tiles + u) * A.width, true);
#pragma unroll
                for (int e = 0; e < VEC; ++e) Ec[e] += w * t[e];
            }
        }
        for (int d = bv; d < 64; d <<= 1) {
#pragma unroll
            for (int e = 0; e < VEC; ++e) {
                Fc[e] += __shfl_xor(Fc[e], d); Rc[e] += __shfl_xor(Rc[e], d);
                if (FOLDED) Ec[e] += __shfl_xor(Ec[e], d);
            }
        }
        if (r == 0) {
#pragma unroll
            for (int e = 0; e < VEC; ++e) {
                part[2][wave][c * VEC + e] = Fc[e]; part[3][wave][c * VEC + e] = Rc[e];
                if (FOLDED) part[FOLDED ? 4 : 0][wave][c * VEC + e] = Ec[e];
            }
        }
    }
    __syncthreads();
    // own rows from zero, then an inclusive scan over the wavefront's row-lanes with decays from the anchors
    float S[VEC], U[VEC];
#pragma unroll
    for (int e = 0; e < VEC; ++e) S[e] = U[e] = 0.0f;
#pragma unroll
    for (int i = 0; i < kMixItems; ++i) {
        const float d = dec[rl * kMixItems + i];
#pragma unroll
        for (int e = 0; e < VEC; ++e) S[e] = d * S[e] + vf[i][e];
        if (is_first(i)) {
            float t[VEC];
            load_equal<VEC>(A, op, slab, c, j0 + i, t);
#pragma unroll
            for (int e = 0; e < VEC; ++e) S[e] += t[e];
        }
    }
#pragma unroll
    for (int i = kMixItems - 1; i >= 0; --i) {
        const float d = dec[rl * kMixItems + i + 1];
#pragma unroll
        for (int e = 0; e < VEC; ++e) U[e] = d * U[e] + (FOLDED ? vr[FOLDED ? i : 0][e] : vf[i][e]);
    }
    for (int d = 1; d < rv; d <<= 1) {
        const float Df = expf(-(pos(j0 + kMixItems - 1) - pos(j0 - d * kMixItems + kMixItems - 1)));
        const float Db = expf(-(pos(j0 + d * kMixItems) - pos(j0)));
#pragma unroll
        for (int e = 0; e < VEC; ++e) {
            const float So = __shfl_up(S[e], (unsigned)(d * bv)), Uo = __shfl_down(U[e], (unsigned)(d * bv));
            if (r >= d) S[e] += Df * So;
            if (r + d < rv) U[e] += Db * Uo;
        }
    }
    if (r == rv - 1) {
#pragma unroll
        for (int e = 0; e < VEC; ++e) part[0][wave][c * VEC + e] = S[e];
    }
    if (r == 0) {
#pragma unroll
        for (int e = 0; e < VEC; ++e) part[1][wave][c * VEC + e] = U[e];
    }
    __syncthreads();
    // state at the row before this row-lane (after it): what precedes the wavefront, then the row-lanes before this one
    float F[VEC], R[VEC];
    {
        const int w0 = base + wave * rv * kMixItems, w1 = w0 + rv * kMixItems;      // this wavefront's rows
        const float pw = pos(w0 - 1), pe = pos(w1);
        float Fw[VEC], Rw[VEC];
#pragma unroll
        for (int e = 0; e < VEC; ++e) Fw[e] = Rw[e] = 0.0f;
        const float cf = expf(-(pw - pos(base - 1))), cb = expf(-(pos(base + rows) - pe));
#pragma unroll
        for (int u = 0; u < kMixWaves; ++u) {
            const float gf = u < wave ? expf(-(pw - pos(base + (u + 1) * rv * kMixItems - 1))) : 0.0f;
            const float gb = u > wave ? expf(-(pos(base + u * rv * kMixItems) - pe)) : 0.0f;
#pragma unroll
            for (int e = 0; e < VEC; ++e) {
                // (the sums on the other side are left out, not multiplied by zero: they may be infinite)
                Fw[e] += (u < wave ? gf * part[0][u][c * VEC + e] : 0.0f) + cf * part[2][u][c * VEC + e];
                Rw[e] += (u > wave ? gb * part[1][u][c * VEC + e] : 0.0f) + cb * part[3][u][c * VEC + e];
            }
        }
        const float df = expf(-(pos(j0 - 1) - pw)), db = expf(-(pe - pos(j0 + kMixItems)));
#pragma unroll
        for (int e = 0; e < VEC; ++e) {
            const float Sb = __shfl_up(S[e], (unsigned)bv), Ua = __shfl_down(U[e], (unsigned)bv);
            F[e] = df * Fw[e] + (r > 0 ? Sb : 0.0f);
            R[e] = db * Rw[e] + (r < rv - 1 ? Ua : 0.0f);
        }
    }
    const uint32_t poison = A.status && *shift_bytes(A.status, op * A.op_ws) ? 0x7FC00000u : 0u;
    auto mark = [&](float x) { return __uint_as_float(__float_as_uint(x) | poison); };
    if constexpr (!FOLDED) {
        float* out = A.fr + ((op * A.slabs + slab) * (int64_t)m) * (2 * A.width) + c * VEC;
#pragma unroll
        for (int i = 0; i < kMixItems; ++i) {
            const float d = dec[rl * kMixItems + i];
            float t[VEC];
#pragma unroll
            for (int e = 0; e < VEC; ++e) { F[e] = d * F[e] + vf[i][e]; t[e] = mark(F[e]); }
            if (j0 + i < m) store_cols<VEC>(out + (int64_t)(j0 + i) * (2 * A.width), t);
        }
#pragma unroll
        for (int i = kMixItems - 1; i >= 0; --i) {
            const float d = dec[rl * kMixItems + i + 1];
            float t[VEC];
#pragma unroll
            for (int e = 0; e < VEC; ++e) { R[e] = d * R[e] + vf[i][e]; t[e] = mark(R[e]); }
            if (j0 + i < m) store_cols<VEC>(out + (int64_t)(j0 + i) * (2 * A.width) + A.width, t);
        }
    } else {
        const int64_t col = (int64_t)slab * A.width + c * VEC;
        const bool col_ok = col < A.batch;
        // backward first: R of every row takes the place of what was added there
#pragma unroll
        for (int i = kMixItems - 1; i >= 0; --i) {
            const float d = dec[rl * kMixItems + i + 1];
#pragma unroll
            for (int e = 0; e < VEC; ++e) { R[e] = d * R[e] + vr[i][e]; vr[i][e] = R[e]; }
        }
        // forward: the row's product takes the place of its F, its strict sum that of its R; E is unknown at the rows of a run that
        // the row-lane starts inside of
        float run[VEC];
#pragma unroll
        for (int e = 0; e < VEC; ++e) run[e] = 0.0f;
        auto unknown = [&](int i) { return tie[i] != 0u && (int)tie[i] - 1 < j0; };
#pragma unroll
        for (int i = 0; i < kMixItems; ++i) {
            const float d = dec[rl * kMixItems + i];
            float t[VEC], E[VEC];
#pragma unroll
            for (int e = 0; e < VEC; ++e) { F[e] = d * F[e] + vf[i][e]; E[e] = F[e]; t[e] = 0.0f; }
            if (is_first(i)) load_equal<VEC>(A, op, slab, c, j0 + i, t);
#pragma unroll
            for (int e = 0; e < VEC; ++e) {
                if (is_first(i)) run[e] = E[e];
                if (tie[i] != 0u) E[e] = run[e];          // (unknown: nothing taken off yet)
                F[e] += t[e];
                vf[i][e] = F[e] + vr[i][e];
                vr[i][e] -= unknown(i) ? 0.0f : E[e];
            }
        }
        store_cols<VEC>(run_e + rl * A.width + c * VEC, run);
        __syncthreads();
        if (unknown(0)) {
            const int at = (int)tie[0] - 1 - base;
#pragma unroll
            for (int e = 0; e < VEC; ++e) run[e] = 0.0f;
            if (at >= 0) {
                load_cols<VEC>(run, run_e + (at / kMixItems) * A.width + c * VEC, true);
            } else {
#pragma unroll
                for (int u = 0; u < kMixWaves; ++u)
#pragma unroll
                    for (int e = 0; e < VEC; ++e) run[e] += part[4][u][c * VEC + e];
            }
#pragma unroll
            for (int i = 0; i < kMixItems; ++i)
#pragma unroll
                for (int e = 0; e < VEC; ++e) vr[i][e] -= unknown(i) ? run[e] : 0.0f;
        }
#pragma unroll
        for (int i = 0; i < kMixItems; ++i) {
            const int j = j0 + i;
            float P[VEC], Z[VEC];
#pragma unroll
            for (int e = 0; e < VEC; ++e) { P[e] = mark(vf[i][e]); Z[e] = mark(vr[i][e]); }
            if (j >= m) continue;
            const int64_t row = A.srow[op * m + j], at = (op * m + row) * A.batch + col;
            if (O.p && col_ok) store_cols<VEC>(O.p + at, P);
            if (O.z && col_ok) store_cols<VEC>(O.z + at, Z);
            if (O.u) {                                   // uniform
                float u[VEC], dz = 0.0f, dp = 0.0f;
                load_cols<VEC>(u, O.u + row * O.ldu + col, col_ok);
#pragma unroll
                for (int e = 0; e < VEC; ++e) { dz += u[e] * Z[e]; dp += u[e] * P[e]; }
                for (int q = 1; q < bv; q <<= 1) { dz += __shfl_xor(dz, q); dp += __shfl_xor(dp, q); }
                const int64_t slot = ((int64_t)slab * A.operators + op) * m + row;
                if (c == 0 && O.dot_z) O.dot_z[slot] = A.slabs == 1 ? O.w[op] * dz : dz;
                if (c == 0 && O.dot_p) O.dot_p[slot] = dp;
            }
        }
    }
}

// ---------------------------------------------------------------------------
// The operators added up, and the anchor gradients' row products.  T target rows and VEC columns a lane.
//   ROWS = false   targets: the long side, from the scanned short side:
//                  out_i = sum_q w_q (el F_lo + er R_lo'),   dot1[q][i] = sum_t u_it (strict R - strict F)
//   ROWS = true    targets: the short side, whose products P_q and strict sums Z_q (either may be null) lie in memory:
//                  out_j = sum_q w_q P_q[j],   dot1[q][j] = sum_t u_jt Z_q[j][t],   dot2[q][j] = sum_t u_jt P_q[j][t]
// Dots are left per slab (dot[slab][q][row]) for k_mix_ends to add; a single slab writes w_q dot1, the gradient, itself.
// ---------------------------------------------------------------------------
template <int VEC, int T, bool ROWS>
__global__ void __launch_bounds__(kMixThreads)
k_mix_gather(const MixPath A, const MixGather S)
{
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int slab = (int)blockIdx.x % A.slabs, chunk = (int)blockIdx.x / A.slabs;
    const int width = A.width, bv = width / VEC, rv = 64 / bv;
    const int c = lane & (bv - 1);
    const int count = ROWS ? A.m : A.l, m = A.m;
    const int64_t col = (int64_t)slab * width + c * VEC;
    const bool col_ok = col < A.batch;
    int row[T];
    bool live[T];
    float acc[T][VEC], u[T][VEC];
#pragma unroll
    for (int t = 0; t < T; ++t) {
        row[t] = ((chunk * kMixWaves + wave) * T + t) * rv + lane / bv;
        live[t] = row[t] < count;
        row[t] = live[t] ? row[t] : count - 1;
#pragma unroll
        for (int e = 0; e < VEC; ++e) acc[t][e] = u[t][e] = 0.0f;
        if (S.u) load_cols<VEC>(u[t], S.u + (int64_t)row[t] * S.ldu + col, col_ok);
    }
    const bool first = !ROWS || S.p != nullptr, second = ROWS && S.z != nullptr;
    uint4 rec[T];
    if (!ROWS) {
#pragma unroll
        for (int t = 0; t < T; ++t) rec[t] = A.recs[row[t]];
    }
    for (int q = 0; q < A.operators; ++q) {
        const float wq = S.w[q];
        float f[T][VEC], g[T][VEC];
        uint4 now[T];
        if (!ROWS) {
            const float* fr = A.fr + ((int64_t)q * A.slabs + slab) * m * (2 * width) + c * VEC;
#pragma unroll
            for (int t = 0; t < T; ++t) {
                now[t] = rec[t];
                const int lo = (int)now[t].x;
                load_cols<VEC>(f[t], fr + (int64_t)(lo - 1) * (2 * width), lo > 0);
                load_cols<VEC>(g[t], fr + (int64_t)lo * (2 * width) + width, lo < m);
            }
            if (q + 1 < A.operators) {
#pragma unroll
                for (int t = 0; t < T; ++t) rec[t] = A.recs[(int64_t)(q + 1) * A.l + row[t]];
            }
        } else {
#pragma unroll
            for (int t = 0; t < T; ++t) {
                const int64_t at = ((int64_t)q * m + row[t]) * A.batch + col;
                load_cols<VEC>(f[t], S.p + at, first && col_ok);
                load_cols<VEC>(g[t], S.z + at, second && col_ok);
            }
        }
#pragma unroll
        for (int t = 0; t < T; ++t) {
            const float el = ROWS ? 1.0f : __uint_as_float(now[t].z), er = ROWS ? 0.0f : __uint_as_float(now[t].w);
            float d1 = 0.0f, d2 = 0.0f;
#pragma unroll
            for (int e = 0; e < VEC; ++e) {
                if (ROWS) {
                    acc[t][e] += wq * f[t][e];
                    d1 += u[t][e] * g[t][e];
                    d2 += u[t][e] * f[t][e];
                } else {
                    acc[t][e] += wq * (el * f[t][e] + er * g[t][e]);
                }
            }
            if (!ROWS && S.dot1) {
                float es = er;
                if (now[t].x != now[t].y) {               // short anchors equal to this one: the strict sum starts behind them
                    const int hi = (int)now[t].y;
                    const bool any = hi < m;
                    es = any ? expf(-(A.sp[(int64_t)q * m + (any ? hi : 0)] - A.long_anchor[(int64_t)q * A.l + row[t]])) : 0.0f;
                    load_cols<VEC>(g[t], A.fr + (((int64_t)q * A.slabs + slab) * m + hi) * (2 * width) + width + c * VEC, any);
                }
#pragma unroll
                for (int e = 0; e < VEC; ++e) d1 += u[t][e] * (es * g[t][e] - el * f[t][e]);
            }
            if (S.dot1) {
                for (int d = 1; d < bv; d <<= 1) d1 += __shfl_xor(d1, d);
                if (c == 0 && live[t]) S.dot1[((int64_t)slab * A.operators + q) * count + row[t]] = A.slabs == 1 ? wq * d1 : d1;
            }
            if (ROWS && S.dot2) {
                for (int d = 1; d < bv; d <<= 1) d2 += __shfl_xor(d2, d);
                if (c == 0 && live[t]) S.dot2[((int64_t)slab * A.operators + q) * count + row[t]] = d2;
            }
        }
    }
    if (S.out && col_ok) {
#pragma unroll
        for (int t = 0; t < T; ++t)
            if (live[t]) store_cols<VEC>(S.out + (int64_t)row[t] * S.ldo + col, acc[t]);
    }
}

// What a call's dots come to, in one launch at its end (three took 13 us of the 139 of 16 operators 1000 x 2048, batch 256, forward + backward):
// the first workgroups of an operator (blockIdx.y) take out[q][i] = w_q sum_slab dot[slab][q][i], the next ones the same of the
// other side, and the last one total[q] = sum over slabs and rows of dot_total[slab][q][row], in a fixed order.
constexpr int kTotalThreads = 1024;

__device__ __forceinline__ void mix_finish(const float* __restrict__ dot, const float* __restrict__ w, int slabs, int operators, int count, float* __restrict__ out,
                                           int64_t q, int block)
{
    const int i = block * kTotalThreads + (int)threadIdx.x;
    if (i >= count) return;
    float s = 0.0f;
    for (int b = 0; b < slabs; ++b) s += dot[((int64_t)b * operators + q) * count + i];
    out[q * count + i] = w[q] * s;
}

__global__ void __launch_bounds__(kTotalThreads)
k_mix_ends(const MixEnds E, int slabs, int operators, int blocks0, int blocks1)
{
    __shared__ float red[kTotalThreads];
    const int64_t q = blockIdx.y;
    const int block = (int)blockIdx.x;
    if (block < blocks0) { mix_finish(E.dot[0], E.w, slabs, operators, E.count[0], E.out[0], q, block); return; }
    if (block < blocks0 + blocks1) { mix_finish(E.dot[1], E.w, slabs, operators, E.count[1], E.out[1], q, block - blocks0); return; }
    const float* const dot = E.dot_total;
    const int count = E.total_rows;
    float* const out = E.total;
    float s = 0.0f;
    for (int b = 0; b < slabs; ++b) {
        const float* at = dot + ((int64_t)b * operators + q) * count;
#pragma unroll 4
        for (int i = threadIdx.x; i < count; i += kTotalThreads) s += at[i];
    }
    red[threadIdx.x] = s;
    __syncthreads();
    for (int d = kTotalThreads / 2; d >= 1; d >>= 1) {
        if ((int)threadIdx.x < d) red[threadIdx.x] += red[threadIdx.x + d];
        __syncthreads();
    }
    if (threadIdx.x == 0) out[q] = red[0];
}

bool aligned_rows(const float* p, int64_t ld) { return !p || ((reinterpret_cast<uintptr_t>(p) & 15u) == 0 && ld % 4 == 0); }

template <int VEC, bool ROWS>
void go_gather(const MixPath& A, const MixGather& S, hipStream_t st)
{
    const int64_t count = ROWS ? A.m : A.l, per = (int64_t)kMixWaves * (64 / (A.width / VEC));
    const char* family = ROWS ? "mix_rows" : "mix_gather";
    // four rows a lane once that still leaves every compute unit four workgroups, else one
    if ((count + 4 * per - 1) / (4 * per) * A.slabs >= 1024) {
        LAPLEX_TIMED(family, st, hipLaunchKernelGGL((k_mix_gather<VEC, 4, ROWS>), dim3((unsigned)((count + 4 * per - 1) / (4 * per) * A.slabs)),
                                                    dim3(kMixThreads), 0, st, A, S));
    } else {
        LAPLEX_TIMED(family, st, hipLaunchKernelGGL((k_mix_gather<VEC, 1, ROWS>), dim3((unsigned)((count + per - 1) / per * A.slabs)),
                                                    dim3(kMixThreads), 0, st, A, S));
    }
}

}  // namespace

hipError_t launch_mix_plan(const MixPath& path, hipStream_t st)
{
    MixPath A = path;
    const int tiles = (A.N + kIndexTile - 1) / kIndexTile;
    const dim3 grid((unsigned)tiles, (unsigned)A.operators);
    A.counted = tiles > kIndexRecount;
    if (A.counted) LAPLEX_TIMED("mix_plan", st, hipLaunchKernelGGL(k_mix_count, grid, dim3(kIndexThreads), 0, st, A));
    LAPLEX_TIMED("mix_plan", st, hipLaunchKernelGGL(k_mix_index, grid, dim3(kIndexThreads), 0, st, A));
    const int64_t items = A.l > A.m + 1 ? A.l : A.m + 1;
    LAPLEX_TIMED("mix_plan", st, hipLaunchKernelGGL(k_mix_records, dim3((unsigned)((items + kMixThreads - 1) / kMixThreads), (unsigned)A.operators),
                                                    dim3(kMixThreads), 0, st, A));
    return hipGetLastError();
}

hipError_t launch_mix_replan(const MixPath& A, hipStream_t st)
{
    LAPLEX_TIMED("mix_plan", st, hipLaunchKernelGGL(k_mix_replan, dim3((unsigned)A.operators), dim3(kIndexThreads), 0, st, A));
    return hipGetLastError();
}

namespace {

template <int VEC, bool FOLDED>
void go_scan(MixPath A, const float* v, int64_t ldv, const MixFolded& S, hipStream_t st)
{
    const int rows = kMixWaves * (64 / (A.width / VEC)) * kMixItems;
    A.tiles = (A.m + rows - 1) / rows;
    const dim3 grid((unsigned)(A.tiles * A.slabs), (unsigned)A.operators), block(kMixThreads);
    if (A.tiles > 1)      // (a single tile has no others to add up)
        LAPLEX_TIMED("mix_scan", st, hipLaunchKernelGGL((k_mix_scan_reduce<VEC, FOLDED>), grid, block, 0, st, A, v, ldv));
    LAPLEX_TIMED("mix_scan", st, hipLaunchKernelGGL((k_mix_scan_down<VEC, FOLDED>), grid, block, 0, st, A, v, ldv, S));
}

template <int VEC>
void go_fold(const MixPath& A, const float* v, int64_t ldv, hipStream_t st)
{
    const int64_t groups = (A.batch + VEC - 1) / VEC;
    const int lanes = groups >= 64 ? 64 : pow2_at_least(groups), spans = (int)((groups + lanes - 1) / lanes);
    const int per = kMixWaves * (64 / lanes);
    const dim3 grid((unsigned)((A.task_count + per - 1) / per * spans), (unsigned)A.operators), block(kMixThreads);
    if (lanes == 64) LAPLEX_TIMED("mix_fold", st, hipLaunchKernelGGL((k_mix_fold<VEC, true>), grid, block, 0, st, A, v, ldv, lanes, spans));
    else LAPLEX_TIMED("mix_fold", st, hipLaunchKernelGGL((k_mix_fold<VEC, false>), grid, block, 0, st, A, v, ldv, lanes, spans));
}

// Many threads for a few intervals where they have several tasks each (row-lanes to share a long sum among); else few threads, and as
// many intervals as leave enough workgroups (11 x (422 x 7059), batch 256, half a task an interval: many threads 31 us, few 11).
template <int VEC>
void go_join(const MixPath& A, hipStream_t st)
{
    auto groups = [&](int per) { return (unsigned)((A.m + 1 + per - 1) / per * A.slabs); };
    int per = kJoinIntervals;
    while (per > 16 && (int64_t)groups(per) * A.operators < 1024) per /= 4;
    if (A.l / 128 >= A.m) LAPLEX_TIMED("mix_join", st, hipLaunchKernelGGL((k_mix_join<VEC, 1024>), dim3(groups(16), (unsigned)A.operators), dim3(1024), 0, st, A, 16));
    else LAPLEX_TIMED("mix_join", st, hipLaunchKernelGGL((k_mix_join<VEC, kJoinIntervals>), dim3(groups(per), (unsigned)A.operators), dim3(kJoinIntervals), 0, st, A, per));
}

}  // namespace

hipError_t launch_mix_scan(const MixPath& A, const float* v, int64_t ldv, hipStream_t st)
{
    if (A.batch % 4 == 0 && aligned_rows(v, ldv)) go_scan<4, false>(A, v, ldv, MixFolded{}, st);
    else go_scan<1, false>(A, v, ldv, MixFolded{}, st);
    return hipGetLastError();
}

hipError_t launch_mix_fold(const MixPath& A, const float* v, int64_t ldv, const MixFolded& S, hipStream_t st)
{
    if (A.batch % 4 == 0 && aligned_rows(v, ldv)) go_fold<4>(A, v, ldv, st);
    else go_fold<1>(A, v, ldv, st);
    if (A.l > kMixTaskRows) {      // (else no interval has two tasks)
        if (A.batch % 4 == 0) go_join<4>(A, st);
        else go_join<1>(A, st);
    }
    if (A.batch % 4 == 0 && aligned_rows(S.u, S.ldu)) go_scan<4, true>(A, nullptr, 0, S, st);
    else go_scan<1, true>(A, nullptr, 0, S, st);
    return hipGetLastError();
}

hipError_t launch_mix_gather(const MixPath& A, const MixGather& S, bool rows, hipStream_t st)
{
    const bool v4 = A.batch % 4 == 0 && aligned_rows(S.u, S.ldu) && aligned_rows(S.out, S.ldo);
    if (v4) { if (rows) go_gather<4, true>(A, S, st); else go_gather<4, false>(A, S, st); }
    else    { if (rows) go_gather<1, true>(A, S, st); else go_gather<1, false>(A, S, st); }
    return hipGetLastError();
}

hipError_t launch_mix_ends(const MixPath& A, const MixEnds& E, hipStream_t st)
{
    int blocks[2];
    for (int i = 0; i < 2; ++i) blocks[i] = E.out[i] ? (E.count[i] + kTotalThreads - 1) / kTotalThreads : 0;
    const int all = blocks[0] + blocks[1] + (E.total ? 1 : 0);
    if (all == 0) return hipSuccess;
    LAPLEX_TIMED("mix_finish", st, hipLaunchKernelGGL(k_mix_ends, dim3((unsigned)all, (unsigned)A.operators), dim3(kTotalThreads), 0, st,
                                                      E, A.slabs, A.operators, blocks[0], blocks[1]));
    return hipGetLastError();
}

}  // namespace laplex

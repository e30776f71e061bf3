// Small problems in one launch or two.  With few pairs of an output and an input the products are formed from the definition, beside the sort
// (k_small_pairs).  Else, when the merged sequence a ++ b has at most kSmallMax positions, the
// whole path of one call (Sec. 3: sort, then the prefix recurrence and its mirror image) is one launch
// that sorts (k_small_rank: ranks by counting, over the whole device) and one that runs the decayed scans in both directions
// and scatters the results (k_small),
// where the large path needs about ten launches of a few microseconds each.  (App. "GPU runtime": below
// n = 2^17 the paper's curves are flat at the cost of the launches.)  Where a wide batch makes the second launch read too much the scans
// are the large path's (small_reads_too_much).  Several operators (the r anchor
// pairs of a sum of operators) and several slabs of batch columns are separate workgroups of a launch.
//
// The numbers carried are those of the large path: F (inclusive decayed sum) and E (the sum over
// strictly smaller keys), summarised per segment as (D, S, H, Q):
//     F_out = D F_in + S,    E_out = H ? D F_in + Q : E_in.
#include "laplex_internal.h"

#include <type_traits>

namespace laplex {

namespace {

constexpr int kSmallThreads = 1024;
constexpr int kSmallWaves = kSmallThreads / 64;
constexpr int kSmallItems = 8;

__device__ __forceinline__ uint32_t small_float_to_key(float f)
{
    uint32_t u = __float_as_uint(f);
    if (u == 0x80000000u) u = 0u;                       // -0.0 sorts as +0.0
    return u ^ ((u >> 31) ? 0xFFFFFFFFu : 0x80000000u);
}

__device__ __forceinline__ float small_key_to_float(uint32_t key)
{
    return __uint_as_float(key ^ ((key >> 31) ? 0x80000000u : 0xFFFFFFFFu));
}

// The sort of a small problem, spread over the whole device: the stable rank of an anchor is the number
// of pairs (key, position) below its own, and counting that by brute force costs N^2 comparisons, which
// 256 compute units do in about a microsecond for N = 8192 when the count is taken 64 comparisons at a
// time (one compare instruction, one population count of the resulting lane mask).  A workgroup takes
// a block of queries; each of its 16 wavefronts keeps 512 of the candidates in registers (8 per lane),
// counts for every query how many of them lie below it, and the 16 partial counts are added per query.
// Output: the plan's ids and sorted anchors (pk, between its two sentinels).
constexpr int kRankQueriesMax = 256;      // queries per workgroup: 32 .. 256, chosen by the launcher

struct RankShared {
    uint32_t query[kRankQueriesMax];
    uint32_t partial[kSmallWaves][kRankQueriesMax];
};
// Positions need not be compared: the 64 candidates of a word lie before, behind or in the queries' own word, so a candidate counts
// where its key is not above, below, or, in the queries' own, by key and position.  One full-rate comparison of 32 bits a word instead of one of 64 (us: forward
// + backward, 4096 x 4096, batch 1 33.3 -> 31.6, 2048 x 2048, batch 8 33.6 -> 32.3; forward, 4096 x 4096, batch 8 22.9 -> 21.4; the weighted Gram matrix of 1024 over 6000
// 28.5 -> 27.1; four queries at a time instead of two take 106 scalar registers, and with them one of two workgroups off a compute unit).
__device__ __forceinline__ void small_rank(const SmallArgs& A, int queries, int block, RankShared& L)
{
    constexpr int kAtOnce = 32;                                     // queries whose own word is the same (they begin at a multiple of 32)
    auto& query = L.query;
    auto& partial = L.partial;
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int64_t op = blockIdx.y;
    const int N = (int)(A.k + A.n);
    const float* a = A.a + op * A.op_a;
    const float* b = A.b + op * A.op_b;
    uint32_t* g_ids = reinterpret_cast<uint32_t*>(reinterpret_cast<char*>(A.ids) + op * A.op_ws);
    float* g_pk = reinterpret_cast<float*>(reinterpret_cast<char*>(A.pk) + op * A.op_ws);
    auto key_of = [&](int e) { return small_float_to_key(A.tau * (e < A.k ? a[e] : b[e - A.k])); };
    // candidates of this wavefront: positions (wave * kSmallItems + r) * 64 + lane; one past the end is above every query or behind it
    uint32_t cand[kSmallItems];
#pragma unroll
    for (int r = 0; r < kSmallItems; ++r) {
        const int e = (wave * kSmallItems + r) * 64 + lane;
        cand[r] = e < N ? key_of(e) : 0xFFFFFFFFu;
    }
    const int q0 = block * queries;
    if (tid < queries) query[tid] = q0 + tid < N ? key_of(q0 + tid) : 0u;
    __syncthreads();
    for (int c = 0; c < queries; c += kAtOnce) {
        const uint32_t mine = query[c + (lane & (kAtOnce - 1))];
        const int own = ((q0 + c) >> 6) - wave * kSmallItems;       // the queries' word, counted from this wavefront's first
        uint32_t counts = 0u;                                       // lane q: of query c + q
        auto count_all = [&](auto below) {                          // below(r, key, query): the mask of the candidates that count
#pragma unroll 2
            for (int q = 0; q < kAtOnce; ++q) {
                const uint32_t key = (uint32_t)__builtin_amdgcn_readlane((int)mine, q);
                uint32_t n = 0u;
#pragma unroll
                for (int r = 0; r < kSmallItems; ++r) n += (uint32_t)__popcll(below(r, key, q));
                counts = lane == q ? n : counts;
            }
        };
        if (wave * 64 * kSmallItems >= N) {                         // (uniform: no candidates here)
        } else if (own >= kSmallItems) {
            count_all([&](int r, uint32_t key, int) { return __ballot(cand[r] <= key); });
        } else if (own < 0) {
            count_all([&](int r, uint32_t key, int) { return __ballot(cand[r] < key); });
        } else {
            count_all([&](int r, uint32_t key, int q) {             // (one wavefront of sixteen; masks for the words' own sides would be more instructions)
                const unsigned long long it = (unsigned long long)cand[r] << 32 | (uint32_t)((wave * kSmallItems + r) * 64 + lane);
                return __ballot(it < ((unsigned long long)key << 32 | (uint32_t)(q0 + c + q)));
            });
        }
        if (lane < kAtOnce) partial[wave][c + lane] = counts;
    }
    __syncthreads();
    if (tid < queries && q0 + tid < N) {
        uint32_t rank = 0u;
#pragma unroll
        for (int w = 0; w < kSmallWaves; ++w) rank += partial[w][tid];
        g_ids[rank] = (uint32_t)(q0 + tid);
        g_pk[rank + 1] = small_key_to_float(query[tid]);
    }
    if (block == 0 && tid == 0) {
        g_pk[0] = __uint_as_float(0xFF800000u);
        g_pk[N + 1] = __uint_as_float(0x7F800000u);
        reinterpret_cast<uint32_t*>(reinterpret_cast<char*>(A.counters) + op * A.op_ws)[kPlanIndexWord] = 0u;      // a new plan
    }
}

__global__ void __launch_bounds__(kSmallThreads)
k_small_rank(SmallArgs A, int queries)
{
    __shared__ RankShared L;
    small_rank(A, queries, (int)blockIdx.x, L);
}

// ---------------------------------------------------------------------------
// Few pairs: the products by the definition (Sec. 1), y_i = sum_j exp(-|a_i - b_j|) x_j and, for the anchor gradients, the same sum with the sign
// of b_j - a_i and without the pairs that are tied, straight from the anchors.  They need no sorted order, so the plan is ranked by other workgroups of the same launch, and a
// call is one launch where ranks and scans are two in a row (measured: see small_pairwise).  Bound by the launch and one chain of loads,
// then by the vector units: an exponential of eight instructions and one or two multiply-adds a column for every pair.
// A wavefront takes ROWS result rows and every fourth 64 of the injected rows, a lane one injected row at a time; lanes and the four quarters are added up
// as a butterfly and in order, so the sums are trees over chains of m / 256 terms.
// ---------------------------------------------------------------------------
constexpr int kPairSplits = 4;                                             // wavefronts that share result rows
constexpr int kPairGroups = kSmallWaves / kPairSplits;
template <int C> constexpr int kPairKeptGroups = C == 1 ? 1 : kPairGroups;      // (rows of several columns are staged once for as many result rows as there are)
template <int C> constexpr int kPairRows = C <= 2 ? 4 : 2;                 // result rows of a wavefront

// exp(-x) for x >= 0 within 0.82 units in the last place (measured over [0, 104]), subnormal results included: x log2(e) is split into a whole
// number, which goes straight into the exponent, and a fraction for the hardware's 2^f, which returns no subnormal numbers itself (2^t of the whole
// product lost every weight below 2^-126, and with it outputs whose nearest input is 88 to 104 away).  The exponent is kept 64 too high
// until the last multiplication, the one place where a subnormal result is rounded; from 130 on the result is zero, as it is from 104 on.
// (n = k = 4096, batch 1: 14.6 us; v_ldexp in place of the last two steps 14.8, with v_rndne and v_cvt before it 15.2; 2^t at once 14.7.)
__device__ __forceinline__ float exp_minus(float x)
{
    constexpr float log2e = 1.44269504088896340736f, log2e_low = 1.92596299112661746887e-8f, down = 5.42101086242752217004e-20f;      // down: 2^-64
    constexpr float round = 12582912.0f + 64.0f;          // 3 * 2^22: adding it rounds to a whole number, which is then in the lower bits
    x = fminf(x, 130.0f);
    const float sum = __builtin_fmaf(x, -log2e, round);
    const float f = __builtin_fmaf(x, -log2e_low, __builtin_fmaf(x, -log2e, round - sum));
    return __uint_as_float(__float_as_uint(__builtin_amdgcn_exp2f(f)) + (__float_as_uint(sum) << 23)) * down;
}

// The sum over the wavefront, in lane 63 only.  The last LATE of its six steps are in fp64, like the sum of the quarters after them: a tree's error is that
// of its upper levels.  Relative l2 errors against fp64 (y, gx, ga, gb; mean over 32 combinations of sizes, anchors and columns) are 0.73, 0.70, 0.79 and 0.76 of those of the
// scans in place of which these sums are taken (fp32 throughout: 1.03, 0.99, 1.04, 0.99; n = k = 4096, uniform anchors: y 9.6e-8 -> 6.9e-8).
template <int LATE>
__device__ __forceinline__ double wave_sum(float v)
{
    double d = 0.0;
    auto step = [&](auto index, auto ctrl, auto rows) {
        constexpr int I = decltype(index)::value, CTRL = decltype(ctrl)::value, ROWS = decltype(rows)::value;
        if constexpr (I < 6 - LATE) {
            v += __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), CTRL, ROWS, 0xF, false));
        } else {
            if constexpr (I == 6 - LATE) d = (double)v;
            const int low = __builtin_amdgcn_update_dpp(0, __double2loint(d), CTRL, ROWS, 0xF, false);
            const int high = __builtin_amdgcn_update_dpp(0, __double2hiint(d), CTRL, ROWS, 0xF, false);
            d += __hiloint2double(high, low);
        }
    };
    using std::integral_constant;
    using All = integral_constant<int, 0xF>;
    step(integral_constant<int, 0>{}, integral_constant<int, 0x111>{}, All{});                          // row_shr:1, 2, 4, 8
    step(integral_constant<int, 1>{}, integral_constant<int, 0x112>{}, All{});
    step(integral_constant<int, 2>{}, integral_constant<int, 0x114>{}, All{});
    step(integral_constant<int, 3>{}, integral_constant<int, 0x118>{}, All{});
    step(integral_constant<int, 4>{}, integral_constant<int, 0x142>{}, integral_constant<int, 0xA>{});  // the row before's last lane into rows 1 and 3
    step(integral_constant<int, 5>{}, integral_constant<int, 0x143>{}, integral_constant<int, 0xC>{});  // lane 31 into rows 2 and 3
    return d;
}

// LDS: injected rows of more than one column, kPairStage at a time (their anchors, and the columns in planes of up to four, so that a lane's read is as wide
// and conflict-free as it can be; a lane that read its row's columns one by one from memory touched every line of them once per column: 4096 x 4096, batch 8, 126 us), and at the
// end the sums of the wavefronts.
constexpr int kPairStage = 1024;
template <int C, int GROUPS>
struct PairShared {
    static constexpr int W = C < 4 ? C : 4;
    union {
        struct { __align__(16) float v[C > 1 ? C / W : 1][C > 1 ? kPairStage : 1][W]; float at[C > 1 ? kPairStage : 1]; } stage;
        double part[kPairSplits][GROUPS * kPairRows<C>][C][2];
    };
};

template <int C, bool STRICT, int GROUPS>
__device__ __forceinline__ void small_pairs(const SmallArgs& A, const SmallProblem& P, const SmallDot& D, int64_t op, int block, int slabs, PairShared<C, GROUPS>& L)
{
    constexpr int ROWS = kPairRows<C>, BLOCK = GROUPS * ROWS, THREADS = GROUPS * kPairSplits * 64, LATE = C <= 2 ? 6 : 3;
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int split = wave % kPairSplits, group = wave / kPairSplits;
    const int slab = block % slabs, block0 = (block / slabs) * BLOCK, row0 = block0 + group * ROWS;
    const int64_t col0 = (int64_t)slab * C;
    const float* const a = A.a + op * A.op_a;
    const float* const b = A.b + op * A.op_b;
    auto anchor = [&](uint32_t id) {
        float v = A.tau * (id < A.k ? a[id] : b[id - A.k]);
        asm("" : "+v"(v));          // (the product rounded, as the plan has it: fused into the difference below a tie would not be zero)
        return v;
    };
    const int m = (int)(P.inj_hi - P.inj_lo), res = (int)(P.res_hi - P.res_lo);
    const float* const inj = P.inj + op * P.op_inj + col0;
    float at[ROWS], p[ROWS][C], z[ROWS][C];
#pragma unroll
    for (int r = 0; r < ROWS; ++r) {
        at[r] = anchor(P.res_lo + (uint32_t)(row0 + r < res ? row0 + r : res - 1));
#pragma unroll
        for (int c = 0; c < C; ++c) p[r][c] = z[r][c] = 0.0f;
    }
    auto pair = [&](float from, const float (&v)[C]) {
#pragma unroll
        for (int r = 0; r < ROWS; ++r) {
            const float d = from - at[r];
            const float e = exp_minus(fabsf(d)), s = __builtin_copysignf(e, d);
            const bool tie = d == 0.0f;
#pragma unroll
            for (int c = 0; c < C; ++c) p[r][c] = __builtin_fmaf(e, v[c], p[r][c]);
            if (STRICT) {
                if (__any(tie)) {
#pragma unroll
                    for (int c = 0; c < C; ++c) z[r][c] = tie ? z[r][c] : __builtin_fmaf(s, v[c], z[r][c]);
                } else {
#pragma unroll
                    for (int c = 0; c < C; ++c) z[r][c] = __builtin_fmaf(s, v[c], z[r][c]);
                }
            }
        }
    };
    if constexpr (C == 1) {
        constexpr int U = 4;
        for (int j0 = split * 64 + lane; j0 < m; j0 += U * kPairSplits * 64) {
            float from[U], v[U][1];
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const int j = j0 + u * kPairSplits * 64, jc = j < m ? j : j0;
                from[u] = anchor(P.inj_lo + (uint32_t)jc);
                v[u][0] = j < m ? inj[(int64_t)jc * P.ld_inj] : 0.0f;
            }
#pragma unroll
            for (int u = 0; u < U; ++u) pair(from[u], v[u]);
        }
    } else {
        constexpr int W = PairShared<C, GROUPS>::W, LOADS = C * kPairStage / THREADS, ANCHORS = kPairStage / THREADS;
        float next[LOADS], next_at[ANCHORS];
        auto fetch = [&](int base) {
#pragma unroll
            for (int i = 0; i < LOADS; ++i) {
                if (base + i * THREADS / C >= m) break;          // uniform
                const int q = i * THREADS + tid, j = base + q / C, c = q % C;
                next[i] = j < m && col0 + c < A.batch ? inj[(int64_t)j * P.ld_inj + c] : 0.0f;
            }
#pragma unroll
            for (int i = 0; i < ANCHORS; ++i) {
                const int j = base + i * THREADS + tid;
                next_at[i] = anchor(P.inj_lo + (uint32_t)(j < m ? j : m - 1));
            }
        };
        fetch(0);
        for (int base = 0; base < m; base += kPairStage) {
#pragma unroll
            for (int i = 0; i < LOADS; ++i) {
                if (base + i * THREADS / C >= m) break;
                const int q = i * THREADS + tid, j = q / C, c = q % C;
                L.stage.v[c / W][j][c % W] = next[i];
            }
#pragma unroll
            for (int i = 0; i < ANCHORS; ++i) L.stage.at[i * THREADS + tid] = next_at[i];
            __syncthreads();
            if (base + kPairStage < m) fetch(base + kPairStage);
            const int end = m - base < kPairStage ? m - base : kPairStage;
#pragma unroll 1
            for (int j = split * 64 + lane; j < end; j += kPairSplits * 64) {
                float v[C];
#pragma unroll
                for (int c = 0; c < C; ++c) v[c] = L.stage.v[c / W][j][c % W];
                pair(L.stage.at[j], v);
            }
            __syncthreads();
        }
    }
    // (a wavefront that held no injected row has nothing to add up)
    const int splits = m >= kPairSplits * 64 ? kPairSplits : (m + 63) / 64;
#pragma unroll
    for (int r = 0; r < ROWS && split < splits; ++r) {
#pragma unroll
        for (int c = 0; c < C; ++c) {
            const double ps = wave_sum<LATE>(p[r][c]), zs = STRICT ? wave_sum<LATE>(z[r][c]) : 0.0;
            if (lane == 63) { L.part[split][group * ROWS + r][c][0] = ps; L.part[split][group * ROWS + r][c][1] = zs; }
        }
    }
    __syncthreads();
    static_assert(BLOCK * C <= 64, "the results of a workgroup are one wavefront's");
    if (tid >= BLOCK * C) return;
    const int row = tid / C, c = tid % C, rr = block0 + row;
    const int64_t col = col0 + c;
    const bool ok = rr < res && col < A.batch;
    double ps = 0.0, zs = 0.0;
#pragma unroll
    for (int q = 0; q < kPairSplits; ++q) {          // (all are read at once, also what no wavefront wrote)
        const double pq = L.part[q][row][c][0], zq = L.part[q][row][c][1];
        ps += q < splits ? pq : 0.0; zs += q < splits ? zq : 0.0;
    }
    const float pv = (float)ps, zv = (float)zs;
    if (ok && P.out_p) (P.out_p + op * P.op_p)[(int64_t)rr * P.ld_p + col] = pv;
    if (STRICT && ok && P.out_z) (P.out_z + op * P.op_z)[(int64_t)rr * A.batch + col] = zv;
    if (STRICT && D.out) {              // one slab: all columns of a row are here
        float dot = ok ? D.w[(int64_t)rr * D.ld_w + col] * zv : 0.0f;
        if (ok && D.u) dot += D.u[(int64_t)rr * D.ld_u + col] * D.v[(int64_t)rr * A.batch + col];
#pragma unroll
        for (int d = 1; d < C; d <<= 1) dot += __shfl_xor(dot, d);
        if (ok && c == 0) D.out[rr] = dot;
    }
}

// Workgroups [0, pairs0): the first problem's, [pairs0, pairs0 + pairs1): the second's, then those of the ranks (GROUPS = kPairGroups only),
// then the row products'.  On a kept plan the workgroups are smaller: nothing ranks beside them, and a row's sums are the same.
template <int C, bool STRICT, int GROUPS>
__global__ void __launch_bounds__(GROUPS * kPairSplits * 64)
k_small_pairs(const SmallArgs A, const SmallDots D, int slabs, int pairs0, int pairs1, int rank_blocks, int queries)
{
    constexpr bool RANKS = GROUPS == kPairGroups;
    struct Nothing {};
    __shared__ union { PairShared<C, GROUPS> pairs; std::conditional_t<RANKS, RankShared, Nothing> rank; } L;
    const int64_t op = blockIdx.y;
    int block = (int)blockIdx.x;
    if (block < pairs0) { small_pairs<C, STRICT, GROUPS>(A, A.prob[0], D.prob[0], op, block, slabs, L.pairs); return; }
    block -= pairs0;
    if (block < pairs1) { small_pairs<C, STRICT, GROUPS>(A, A.prob[1], D.prob[1], op, block, slabs, L.pairs); return; }
    block -= pairs1;
    if constexpr (RANKS) {
        if (block < rank_blocks) { small_rank(A, queries, block, L.rank); return; }
        block -= rank_blocks;
    }
    // (a row's columns side by side and added up as above: the same bits whoever forms the strict sums)
    const int64_t row = (int64_t)block * (GROUPS * kPairSplits * 64 / C) + threadIdx.x / C;
    const int64_t col = threadIdx.x % C;
    const bool ok = row < D.rows && col < A.batch;
    float dot = ok ? D.row_u[row * D.ld_row + col] * D.row_v[row * A.batch + col] : 0.0f;
#pragma unroll
    for (int d = 1; d < C; d <<= 1) dot += __shfl_xor(dot, d);
    if (ok && col == 0) D.row_out[row] = dot;
}

// ---------------------------------------------------------------------------
// One scan problem.  A workgroup owns a chunk of consecutive rows of the merged sequence and C batch columns, and needs nothing
// from other workgroups: the state before its chunk is a weighted sum of all rows before it, sum_j exp(-(p_before - p_j)) v_j
// (the recurrence of Sec. 3 unrolled), the state after it likewise.  Each workgroup forms those two sums itself -- reading every
// injected row once more per chunk costs less than one workgroup walking all of them, because a small problem leaves the device
// idle --, then scans its own rows in both directions.  Lane l works on column l % C (adjacent lanes read adjacent columns of a
// row); a row-lane holds ITEMS consecutive rows.  Only those are chained by products of decays; everything else is combined with
// decays taken from the anchors.
// Measured (MI355X, us, this kernel / one workgroup per up to 16 columns that walked all rows; plan reused): n = k = 4096, batch 1:
// 11.8 / 21.2, batch 64: 18 / 30, batch 256: 44 / 53; 1024: 9.8 / 13.3, batch 256: 10.5 / 18.6; 16 operators of 100 x 768, batch 64:
// 17 / 20.  Bound by one chain: ids and anchors, injected rows, the reduction over the workgroup, the scan, the stores.
// Rows beyond the reach of an fp32 decay are read like the others: 0 * NaN and 0 * inf are NaN, as in the dense product.
// Strict channel: rows with the key at which a sum is taken are kept apart (weight -1 stands for "equal": the strict sum leaves
// them out, the inclusive sum is strict + equal).
// ---------------------------------------------------------------------------
constexpr int kChunkThreads = 512;
constexpr int kChunkWaves = kChunkThreads / 64;

template <int ITEMS, bool STRICT>
__global__ void __launch_bounds__(kChunkThreads)
k_small(const SmallArgs A, int slabs)
{
    extern __shared__ __align__(8) uint2 others[];            // [N] weight and row of the injected matrix (none: not an injected row)
    __shared__ float red[4][kChunkWaves][16];                 // sums outside the chunk; then the wavefronts' summaries
    __shared__ float wave_s[2][3][kChunkWaves][16];
    __shared__ float wave_p[2][kChunkWaves];
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int N = (int)(A.k + A.n), C = A.cols, RPW = 64 / C, RL = kChunkThreads / C;
    const int64_t op = blockIdx.y / A.nprob;
    const SmallProblem P = A.prob[blockIdx.y % A.nprob];
    const uint32_t* ids = reinterpret_cast<const uint32_t*>(reinterpret_cast<const char*>(A.ids) + op * A.op_ws);
    const float* pk = reinterpret_cast<const float*>(reinterpret_cast<const char*>(A.pk) + op * A.op_ws);
    const float* inj = P.inj + op * P.op_inj;
    const int slab = (int)blockIdx.x % slabs, chunk = (int)blockIdx.x / slabs;
    const int rows = RL * ITEMS, row0 = chunk * rows, row1 = row0 + rows < N ? row0 + rows : N;
    const int c = lane % C, r = lane / C, rl = wave * RPW + r;
    const int64_t col = (int64_t)slab * C + c;
    const bool col_ok = col < A.batch;
    constexpr uint32_t none = 0xFFFFFFFFu;
    auto pos = [&](int j) { return pk[1 + (j < 0 ? 0 : (j < N ? j : N - 1))]; };
    const float pf = pos(row0 - 1), pb = pos(row1);          // (clamped: at the ends of the sequence there is nothing to carry)

    // own rows
    const int q0 = row0 + rl * ITEMS;
    uint32_t id[ITEMS];
    float p[ITEMS], v[ITEMS];
#pragma unroll
    for (int i = 0; i < ITEMS; ++i) {
        const int q = q0 + i;
        id[i] = q < N ? ids[q] : 0xFFFFFFFFu;
        p[i] = pos(q);
        v[i] = q < N && col_ok && id[i] >= P.inj_lo && id[i] < P.inj_hi ? inj[(int64_t)(id[i] - P.inj_lo) * P.ld_inj + col] : 0.0f;
    }
    const float p_left = pos(q0 - 1), p_right = pos(q0 + ITEMS);

    // the other rows' weights, once per workgroup
    for (int j = row0 > 0 || row1 < N ? tid : N; j < N; j += kChunkThreads) {
        const uint32_t e = ids[j];
        const float pj = pk[j + 1];
        const bool in = e >= P.inj_lo && e < P.inj_hi && !(j >= row0 && j < row1);
        const float at = j < row0 ? pf : pb;
        const float w = pj == at ? -1.0f : expf(j < row0 ? pj - pf : pb - pj);
        others[j] = make_uint2(in ? __float_as_uint(w) : 0u, in ? e - P.inj_lo : none);
    }
    __syncthreads();
    float sum[2], same[2];                                    // strictly beyond the key at the chunk's edge, and at it
    sum[0] = sum[1] = same[0] = same[1] = 0.0f;
    constexpr int AHEAD = 8;
#pragma unroll
    for (int dir = 0; dir < 2; ++dir) {
        const int lo = dir == 0 ? rl : row1 + rl, hi = dir == 0 ? row0 : N;
        for (int j0 = lo; j0 < hi; j0 += AHEAD * RL) {
            float w[AHEAD], x[AHEAD];
#pragma unroll
            for (int i = 0; i < AHEAD; ++i) {
                const int j = j0 + i * RL;
                const uint2 o = j < hi ? others[j] : make_uint2(0u, none);
                w[i] = __uint_as_float(o.x);
                x[i] = o.y != none && col_ok ? inj[(int64_t)o.y * P.ld_inj + col] : 0.0f;
            }
#pragma unroll
            for (int i = 0; i < AHEAD; ++i) {
                if (STRICT) {
                    sum[dir] += w[i] >= 0.0f ? w[i] * x[i] : 0.0f;
                    same[dir] += w[i] < 0.0f ? x[i] : 0.0f;
                } else {
                    sum[dir] += fabsf(w[i]) * x[i];
                }
            }
        }
    }
#pragma unroll
    for (int dir = 0; dir < 2; ++dir) {
        for (int m = C; m < 64; m <<= 1) {
            sum[dir] += __shfl_xor(sum[dir], m);
            if (STRICT) same[dir] += __shfl_xor(same[dir], m);
        }
        if (r == 0) { red[2 * dir][wave][c] = sum[dir]; if (STRICT) red[2 * dir + 1][wave][c] = same[dir]; }
    }

    // the row-lane's rows from zero, in both directions (cf, cb: decays from the row-lane's edges, at most ITEMS factors)
    float F0[ITEMS], E0[ITEMS], cf[ITEMS], R0[ITEMS], G0[ITEMS], cb[ITEMS];
    int seen_f = 0, seen_b = 0;                               // bit i: the key has changed between the edge and row i
    {
        float F = 0.0f, E = 0.0f, prod = 1.0f;
        int sn = 0;
#pragma unroll
        for (int i = 0; i < ITEMS; ++i) {
            const float before = i == 0 ? p_left : p[i > 0 ? i - 1 : 0];
            const bool first = q0 + i == 0, h = first || p[i] != before;      // (rows past the end repeat the last anchor)
            const float d = first ? 0.0f : expf(-(p[i] - before));
            E = h ? d * F : E;
            F = (h ? E : F) + v[i];
            prod *= d;
            sn |= h ? 1 : 0;
            F0[i] = F; E0[i] = E; cf[i] = prod; seen_f |= sn << i;
        }
        F = E = 0.0f; prod = 1.0f; sn = 0;
#pragma unroll
        for (int i = ITEMS - 1; i >= 0; --i) {
            const float after = i == ITEMS - 1 ? p_right : p[i < ITEMS - 1 ? i + 1 : 0];
            const bool h = p[i] != after;
            const float d = expf(-(after - p[i]));
            E = h ? d * F : E;
            F = (h ? E : F) + v[i];
            prod *= d;
            sn |= h ? 1 : 0;
            R0[i] = F; G0[i] = E; cb[i] = prod; seen_b |= sn << i;
        }
    }
    // inclusive scans over the wavefront's row-lanes, decays from the anchors at their ends
    const float pe = p[ITEMS - 1], ps = p[0];
    float S = F0[ITEMS - 1], Q = E0[ITEMS - 1], U = R0[0], V = G0[0];
    int H = (seen_f >> (ITEMS - 1)) & 1, J = seen_b & 1;
    for (int d = 1; d < RPW; d <<= 1) {
        const float So = __shfl_up(S, d * C), Qo = __shfl_up(Q, d * C), peo = __shfl_up(pe, d * C);
        const float Uo = __shfl_down(U, d * C), Vo = __shfl_down(V, d * C), pso = __shfl_down(ps, d * C);
        const int Ho = __shfl_up(H, d * C), Jo = __shfl_down(J, d * C);
        if (r >= d) {
            const float D = expf(-(pe - peo));
            Q = H ? D * So + Q : Qo;
            S = D * So + S;
            H |= Ho;
        }
        if (r + d < RPW) {
            const float D = expf(-(pso - ps));
            V = J ? D * Uo + V : Vo;
            U = D * Uo + U;
            J |= Jo;
        }
    }
    if (r == RPW - 1) {
        wave_s[0][0][wave][c] = S; wave_s[0][1][wave][c] = Q; wave_s[0][2][wave][c] = __int_as_float(H);
        if (c == 0) wave_p[0][wave] = pe;
    }
    if (r == 0) {
        wave_s[1][0][wave][c] = U; wave_s[1][1][wave][c] = V; wave_s[1][2][wave][c] = __int_as_float(J);
        if (c == 0) wave_p[1][wave] = ps;
    }
    // the row-lanes before (after) this one in the wavefront
    float Sb = __shfl_up(S, C), Qb = __shfl_up(Q, C), Ua = __shfl_down(U, C), Va = __shfl_down(V, C);
    int Hb = __shfl_up(H, C), Ja = __shfl_down(J, C);
    if (r == 0) { Sb = Qb = 0.0f; Hb = 0; }
    if (r == RPW - 1) { Ua = Va = 0.0f; Ja = 0; }
    __syncthreads();
    // state entering the wavefront: the chunk's, and the wavefronts in between, each decayed to the wavefront's edge directly
    const float pw = wave == 0 ? pf : wave_p[0][wave - 1], pv = wave == kChunkWaves - 1 ? pb : wave_p[1][wave + 1];
    float ef = 0.0f, eb = 0.0f;                               // factors of wavefront `lane`; lane kChunkWaves: of the chunk's edge
    if (lane <= kChunkWaves) {
        const float from_f = lane < kChunkWaves ? wave_p[0][lane] : pf, from_b = lane < kChunkWaves ? wave_p[1][lane] : pb;
        if (lane < wave || lane == kChunkWaves) ef = expf(-(pw - from_f));
        if (lane > wave) eb = expf(-(from_b - pv));
    }
    auto lane_value = [](float x, int l) -> float { return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(x), l)); };
    float Fin = 0.0f, Ein = 0.0f, Rin = 0.0f, Gin = 0.0f;
#pragma unroll
    for (int u = 0; u < kChunkWaves; ++u) {
        Ein += red[0][u][c]; Gin += red[2][u][c];
        if (STRICT) { Fin += red[1][u][c]; Rin += red[3][u][c]; }
    }
    Fin = lane_value(ef, kChunkWaves) * (Ein + Fin);
    Rin = lane_value(eb, kChunkWaves) * (Gin + Rin);
#pragma unroll
    for (int u = 0; u < kChunkWaves; ++u) {
        if (u < wave) {
            if (STRICT && __float_as_int(wave_s[0][2][u][c])) Ein = Fin + wave_s[0][1][u][c];
            Fin += lane_value(ef, u) * wave_s[0][0][u][c];
        }
    }
#pragma unroll
    for (int u = kChunkWaves - 1; u >= 0; --u) {
        if (u > wave) {
            if (STRICT && __float_as_int(wave_s[1][2][u][c])) Gin = Rin + wave_s[1][1][u][c];
            Rin += lane_value(eb, u) * wave_s[1][0][u][c];
        }
    }
    // ... and the row-lane
    {
        const float f = (r == 0 ? 1.0f : expf(-(p_left - pw))) * Fin, b = (r == RPW - 1 ? 1.0f : expf(-(pv - p_right))) * Rin;
        Ein = Hb ? f + Qb : Ein;
        Fin = f + Sb;
        Gin = Ja ? b + Va : Gin;
        Rin = b + Ua;
    }
    float* const out_p = P.out_p ? P.out_p + op * P.op_p : nullptr;
    float* const out_z = P.out_z ? P.out_z + op * P.op_z : nullptr;
#pragma unroll
    for (int i = 0; i < ITEMS; ++i) {
        if (id[i] < P.res_lo || id[i] >= P.res_hi || !col_ok) continue;
        const int64_t rr = (int64_t)(id[i] - P.res_lo);
        const float f = cf[i] * Fin, b = cb[i] * Rin;
        if (out_p) out_p[rr * P.ld_p + col] = f + F0[i] + (b + R0[i]) - v[i];
        if (STRICT && out_z) out_z[rr * A.batch + col] = (((seen_b >> i) & 1) ? b + G0[i] : Gin) - (((seen_f >> i) & 1) ? f + E0[i] : Ein);
    }
}

}  // namespace

// Measured at the line (us, forward + backward; forward: chunks / tiled scans / one workgroup per 16 columns that walks all rows):
// n = k = 4096, batch 128 (3.4e7 values): 68 / 68 / 130; 33 / 33 / 50, batch 160: 98 / 88 / 129, batch 1024 (2.7e8): 407 / 130 / 327;
// 181 / 43 / 119; 4000 x 2000, batch 192 (2.8e7): 88 / 85 / 112, batch 384 (5.5e7): 138 / 96 / 210; 2000 x 2000, batch 512 (3.3e7):
// 78 / 91 / 141, batch 768 (4.9e7): 114 / 99 / 210; 500 x 500, batch 8192 (3.3e7): 192 / 175 / 227.
constexpr double kSmallReads = 3.5e7;
bool small_reads_too_much(int64_t N, int64_t batch)
{
    const int64_t rows = kChunkThreads / 16 * 8;               // a chunk of the widest form below
    const int64_t chunks = (N + rows - 1) / rows;
    return chunks > 1 && (double)chunks * (double)N * (double)batch > kSmallReads;
}

static int pair_columns(int64_t batch) { return batch >= 5 ? 8 : batch >= 3 ? 4 : (int)batch; }

// Where forming every pair's exponential is faster than ranking first and scanning then, in a forward product.  The line is the same whatever a call wants of
// it and whether its plan is kept, since the form shows in the last bits; it lies where a product on a kept plan, which saves no launch, takes no
// longer.  What is counted:
//   pairs       about the cycles of a lane (PairLimits::cost)
//   workgroups  One of up to 8 (16) result rows takes its 3 to 5 us of launch, loads, barriers and sums over lanes however few injected rows there are.
//               A compute unit holds one of 1024 threads at a time (8 columns with strict sums, 85 registers) or two: more than 256 in one launch queue up.
//   stages      of injected rows of several columns: each waits for its loads
//   ranks       of many operators, which share the compute units with the pairs (so many that they are sorted in a launch before: one column is no worse off then, seven of
//               15 x 4361 25.1 / 21.5)
// A backward pass has its plan: its transposed product is formed pair by pair only where the forward product, of the opposite shape, is as well and
// has saved the time; the Gram form's, which goes with its forward, like the transposed one (beside scans in the forward, 1089 x 9, batch 9, forward + backward 31.2 / 33.6 us; 794 x 2405, batch 8 33.6 / 40.3).
// Measured (us, ranks, then scans / pair by pair; forward, forward on a kept plan, forward + backward): n = k = 4096, batch 1 24.2 / 14.6, 11.2 / 9.9, 41.9 / 29.8; 1986 x 121, batch 1
// 17.5 / 10.4, 10.1 / 10.1, 32.0 / 21.2; 2981 x 1035, batch 3 18.9 / 11.6, 10.2 / 10.2, 34.5 / 27.2; Gram form of 1348, batch 4 17.0 / 10.2, 9.6 / 9.7, 29.8 / 21.0, of 1645, batch 8
// 17.4 / 11.8, 9.8 / 10.1, 30.5 / 29.0; 640 x 1979, batch 8 17.4 / 10.2, 10.0 / 10.1, 32.9 / 24.0; 575 x 648, batch 9 16.1 / 10.2, 10.2 / 10.2, 31.0 / 27.7; 118 x 118, batch 128 (240
// workgroups), Gram form 13.5 / 9.8, 9.6 / 9.7, 26.9 / 24.0; sixteen operators of 100 x 39, batch 1 19.7 / 14.1, 13.5 / 13.8, 45.6 / 43.8; six of 143 x 87, batch 9 18.1 / 14.3, 13.7 / 13.9,
// 46.4 / 44.6; forward alone: 2 x 1969, batch 31 (4 workgroups; its transpose has 988) 17.0 / 9.4, 2248 x 190, batch 5 17.9 / 11.0.
// Beyond: Gram form of 2115, batch 4 17.5 / 12.2, 9.8 / 11.1, 31.3 / 36.6; 490 x 3539, batch 5 18.6 / 12.5, 10.0 / 12.3; 3765 x 36, batch 8 (471 workgroups) 17.8 / 13.9, 9.3 / 9.3, keeping its scans
// 19.6 / 21.4; 243 x 243, batch 100 (403), Gram form 14.2 / 10.0, 9.8 / 9.9, 26.4 / 34.3; 3000 x 10, batch 256 (12000) 22.3 / 138, 13.3 / 134, 49.7 / 336; two operators of 2453 x 1295,
// batch 1 21.4 / 18.4, 13.5 / 13.8, keeping scans 23.2 / 24.9; twelve of 15 x 1640, batch 9 21.6 / 22.0, 14.0 / 14.4, 21.7 / 24.6; sixteen of 100 x 900, batch 8 23.3 / 24.0, 14.3 / 15.9, 53.8 / 101.
struct PairLimits { double cost, cost_operators; int64_t injected, workgroups; };
constexpr PairLimits kPairLimits[4] = {      // one slab of 1, 2, 4, 8 columns
    {2.4e8, 1.2e8, kSmallMax, kSmallMax}, {9e7, 5e7, 3 * kPairStage, 416}, {6.5e7, 5e7, 3 * kPairStage, 416}, {8e7, 3e7, 2 * kPairStage, 352}};
constexpr PairLimits kPairLimitsSlabs = {7e7, 2.5e7, 2 * kPairStage, 352};
constexpr int64_t kPairAtOnce = 256;                    // workgroups of 8 columns
constexpr double kPairCostQueued = 1.5e7;               // ... and what more of them may cost
constexpr double kPairCostSlabsBackward = 2.5e7, kPairCostOperatorsBackward = 4e7;
constexpr int64_t kPairWorkgroupsOperators = 300, kPairRankedOperators = 12000;
constexpr double kPairCostBeside = 3e8, kPairCostRanked = 1.5e7;      // one column, ranks beside it: shared by the operators; beside more ranks than that
static double pair_cost(int64_t k, int64_t n, int cols, int64_t slabs, int64_t operators)
{
    return (double)k * (double)n * (double)(slabs * operators) * (12.0 + 2.0 * cols);
}
static int64_t pair_workgroups(int64_t results, int cols, int64_t slabs, int64_t operators)
{
    const int rows = kPairGroups * (cols <= 2 ? kPairRows<1> : kPairRows<8>);
    return (results + rows - 1) / rows * slabs * operators;
}
static bool pairs_pay(int64_t results, int64_t injected, int cols, int64_t slabs, int64_t operators)
{
    const PairLimits& M = slabs > 1 ? kPairLimitsSlabs : kPairLimits[cols == 1 ? 0 : cols == 2 ? 1 : cols == 4 ? 2 : 3];
    const double cost = pair_cost(results, injected, cols, slabs, operators);
    const int64_t workgroups = pair_workgroups(results, cols, slabs, operators);
    if (injected > M.injected || workgroups > M.workgroups || cost > M.cost) return false;
    if (cols == 8 && workgroups > kPairAtOnce && cost > kPairCostQueued) return false;
    if (operators == 1) return true;
    if (cols < 8 && workgroups > kPairWorkgroupsOperators) return false;
    const bool beside = mix_ranked(operators, results + injected), many = operators * (results + injected) > kPairRankedOperators;
    if (cols > 1) return !many && cost <= M.cost_operators;
    return cost <= (!beside ? M.cost_operators : many ? kPairCostRanked : kPairCostBeside / (double)operators);
}
int small_pairwise(int64_t k, int64_t n, int64_t batch, int64_t operators, bool transposed)
{
    const int cols = pair_columns(batch);
    const int64_t slabs = (batch + cols - 1) / cols;
    if (!pairs_pay(k, n, cols, slabs, operators)) return 0;
    if (transposed) {
        if (!pairs_pay(n, k, cols, slabs, operators)) return 0;
        if (cols == 8 && pair_workgroups(k > n ? k : n, cols, slabs, operators) > kPairAtOnce) return 0;
        const double cost = pair_cost(k, n, cols, slabs, operators);
        if ((slabs > 1 && cost > kPairCostSlabsBackward) || (operators > 1 && cost > kPairCostOperatorsBackward)) return 0;
    }
    return (int)slabs;
}

hipError_t launch_small(const SmallArgs& all, int64_t operators, hipStream_t st, const SmallDots* dots)
{
    SmallArgs pairs = all, A = all;           // the problems formed pair by pair; those that are scanned
    SmallDots D = dots ? *dots : SmallDots{};
    pairs.nprob = A.nprob = 0;
    int pair_slabs = 1;
    for (int i = 0; i < all.nprob; ++i) {
        const SmallProblem& p = all.prob[i];
        const int slabs = small_pairwise(all.k, all.n ? all.n : all.k, all.batch, operators, p.res_lo > 0 || all.n == 0);
        if (slabs) {
            pair_slabs = slabs;
            D.prob[pairs.nprob] = dots ? dots->prob[i] : SmallDot{};
            pairs.prob[pairs.nprob++] = p;
        } else {
            A.prob[A.nprob++] = p;
        }
    }
    const int64_t N = A.k + A.n;
    int queries = 32;          // of the ranks, per workgroup (more per workgroup measured slower until the grid gets very large)
    while (queries < kRankQueriesMax && ((N + queries - 1) / queries) * operators > 8192) queries <<= 1;
    if (pairs.nprob > 0 || D.row_out) {
        const int cols = pair_columns(pairs.batch);
        bool strict = pairs.nprob == 0;       // (row products alone: either form)
        const int groups = pairs.reuse_plan && cols == 1 ? kPairKeptGroups<1> : kPairGroups, threads = groups * kPairSplits * 64;
        int blocks[2] = {0, 0};
        for (int i = 0; i < pairs.nprob; ++i) {
            strict = strict || pairs.prob[i].out_z != nullptr || D.prob[i].out != nullptr;
            const int rows = groups * (cols <= 2 ? kPairRows<1> : kPairRows<8>);
            blocks[i] = (int)((pairs.prob[i].res_hi - pairs.prob[i].res_lo + rows - 1) / rows) * pair_slabs;
        }
        const int rank_blocks = pairs.reuse_plan ? 0 : (int)((N + queries - 1) / queries);
        const int row_blocks = D.row_out ? (int)((D.rows * cols + threads - 1) / threads) : 0;
        const dim3 grid((unsigned)(blocks[0] + blocks[1] + rank_blocks + row_blocks), (unsigned)operators);
        auto go = [&](auto kernel) { LAPLEX_TIMED("small_pairs", st, hipLaunchKernelGGL(kernel, grid, dim3((unsigned)threads), 0, st, pairs, D, pair_slabs, blocks[0], blocks[1], rank_blocks, queries)); };
        auto with = [&](auto columns) {
            constexpr int C = decltype(columns)::value;
            if (pairs.reuse_plan) { if (strict) go(k_small_pairs<C, true, kPairKeptGroups<C>>); else go(k_small_pairs<C, false, kPairKeptGroups<C>>); }
            else { if (strict) go(k_small_pairs<C, true, kPairGroups>); else go(k_small_pairs<C, false, kPairGroups>); }
        };
        if (cols == 1) with(std::integral_constant<int, 1>{});
        else if (cols == 2) with(std::integral_constant<int, 2>{});
        else if (cols == 4) with(std::integral_constant<int, 4>{});
        else with(std::integral_constant<int, 8>{});
        if (A.nprob == 0) return hipGetLastError();
        A.reuse_plan = 1;                     // (ranked there, or kept)
    }
    if (!A.reuse_plan) {
        LAPLEX_TIMED("small_sort", st, hipLaunchKernelGGL(k_small_rank, dim3((unsigned)((N + queries - 1) / queries), (unsigned)operators),
                                                          dim3(kSmallThreads), 0, st, A, queries));
    }
    if (A.nprob > 0) {
        // Columns and rows per lane: as few as still leave a compute unit no more than one workgroup (short chains, nothing
        // chained twice), since every chunk reads the rows of all others; then wider.  With four chunks or more four columns with four
        // rows are worth two workgroups a compute unit (100 x 5000, batch 128, forward: 27 us, sixteen with eight 34; 4000 x 2000, batch
        // 128, forward + backward: 58 / 75), not more (100 x 5000, batch 256: 44 / 37; two chunks, 512 x 512, batch 1024: 51 / 46).  Measured (us, forward + backward; the four forms): n = k =
        // 4096, batch 8: 43 / 44 / 56 / 72, batch 32: 60 / 51 / 56 / 104, batch 64: 94 / 67 / 61 / 104; 16 operators of 500 x 500, batch
        // 64: 102 / 82 / 68 / 70, batch 256: 231 / 150 / 118 / 105.
        const int forms[4][2] = {{1, 1}, {1, 2}, {4, 4}, {16, 8}};      // columns, rows
        int cols = 1, items = 1;
        int64_t slabs = 0, chunks = 0;
        for (const auto& f : forms) {
            cols = 1; items = f[1];
            while (cols < A.batch && cols < f[0]) cols <<= 1;
            const int64_t rows = (int64_t)kChunkThreads / cols * items;
            slabs = (A.batch + cols - 1) / cols; chunks = (N + rows - 1) / rows;
            if (slabs * chunks * operators <= (f[0] == 4 && chunks >= 4 ? 512 : 256)) break;      // (whatever the problems of the launch: the form shows in the last bits)
        }
        A.cols = cols;
        const dim3 grid((unsigned)(chunks * slabs), (unsigned)(operators * A.nprob));
        const size_t lds = sizeof(uint2) * (size_t)N;
        bool strict = false;
        for (int i = 0; i < A.nprob; ++i) strict = strict || A.prob[i].out_z != nullptr;
        auto go = [&](auto kernel) { LAPLEX_TIMED("small", st, hipLaunchKernelGGL(kernel, grid, dim3(kChunkThreads), lds, st, A, (int)slabs)); };
        if (strict) { if (items == 1) go(k_small<1, true>); else if (items == 2) go(k_small<2, true>); else if (items == 4) go(k_small<4, true>); else go(k_small<8, true>); }
        else        { if (items == 1) go(k_small<1, false>); else if (items == 2) go(k_small<2, false>); else if (items == 4) go(k_small<4, false>); else go(k_small<8, false>); }
    }
    return hipGetLastError();
}

}  // namespace laplex

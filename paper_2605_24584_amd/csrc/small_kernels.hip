// Small problems in two launches.  When the merged sequence a ++ b has at most kSmallMax positions the
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

__global__ void __launch_bounds__(kSmallThreads)
k_small_rank(SmallArgs A, int queries)
{
    __shared__ unsigned long long query[kRankQueriesMax];
    __shared__ uint32_t partial[kRankQueriesMax][kSmallWaves];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int64_t op = blockIdx.y;
    const int N = (int)(A.k + A.n);
    const float* a = A.a + op * A.op_a;
    const float* b = A.b + op * A.op_b;
    uint32_t* g_ids = reinterpret_cast<uint32_t*>(reinterpret_cast<char*>(A.ids) + op * A.op_ws);
    float* g_pk = reinterpret_cast<float*>(reinterpret_cast<char*>(A.pk) + op * A.op_ws);
    auto composite = [&](int e) -> unsigned long long {
        const float f = A.tau * (e < A.k ? a[e] : b[e - A.k]);
        return ((unsigned long long)small_float_to_key(f) << 32) | (unsigned long long)(uint32_t)e;
    };
    // candidates of this wavefront: positions wave * 512 + r * 64 + lane; a position past the end never counts
    // (one 64-bit compare per 64 candidates; splitting it into key and position compares with lane masks
    //  was four times slower)
    unsigned long long cand[kSmallItems];
#pragma unroll
    for (int r = 0; r < kSmallItems; ++r) {
        const int e = wave * 64 * kSmallItems + r * 64 + lane;
        cand[r] = e < N ? composite(e) : ~0ull;
    }
    const int q0 = blockIdx.x * queries;
    if (tid < queries) query[tid] = q0 + tid < N ? composite(q0 + tid) : 0ull;
    __syncthreads();
    const bool any = wave * 64 * kSmallItems < N;                   // uniform: does this wavefront hold candidates at all
    for (int q = 0; q < queries; ++q) {
        const unsigned long long me = query[q];                     // the same for every lane
        uint32_t below = 0u;
        if (any) {
#pragma unroll
            for (int r = 0; r < kSmallItems; ++r) below += (uint32_t)__popcll(__ballot(cand[r] < me));
        }
        if (lane == 0) partial[q][wave] = below;
    }
    __syncthreads();
    if (tid < queries && q0 + tid < N) {
        uint32_t rank = 0u;
#pragma unroll
        for (int w = 0; w < kSmallWaves; ++w) rank += partial[tid][w];
        const unsigned long long me = query[tid];
        g_ids[rank] = (uint32_t)me;
        g_pk[rank + 1] = small_key_to_float((uint32_t)(me >> 32));
    }
    if (blockIdx.x == 0 && tid == 0) {
        g_pk[0] = __uint_as_float(0xFF800000u);
        g_pk[N + 1] = __uint_as_float(0x7F800000u);
        reinterpret_cast<uint32_t*>(reinterpret_cast<char*>(A.counters) + op * A.op_ws)[kPlanIndexWord] = 0u;      // a new plan
    }
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

hipError_t launch_small(const SmallArgs& A0, int64_t operators, hipStream_t st)
{
    SmallArgs A = A0;
    const int64_t N = A.k + A.n;
    if (!A.reuse_plan) {
        int queries = 32;          // per workgroup (more per workgroup measured slower until the grid gets very large)
        while (queries < kRankQueriesMax && ((N + queries - 1) / queries) * operators > 8192) queries <<= 1;
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

// Weighted Gram matrix  M = A diag(d) A^T,  A = L(a, b)  (Sec. 3 "Computation of Gram matrix";
// App. "Fast weighted Gram matrix", Thm "Exact Gram decomposition"):
//
//   M_ij = sum_t d_t exp(-|a_i - b_t|) exp(-|a_j - b_t|)
//        = exp(-(a_hi - a_lo)) * ( U_lo + (W_hi - W_lo) + V_hi ),      lo / hi: the pair in sorted order,
//
// with, for a Gram anchor at sorted position p of the merged sequence a ++ b,
//   U = sum over middle anchors before p of  d_t exp(-2 (a - b_t))   (forward scan, doubled decay),
//   V = sum over middle anchors after  p of  d_t exp(-2 (b_t - a))   (backward scan, doubled decay),
//   W = sum over middle anchors before p of  d_t                     (plain prefix sum).
// W enters only through differences W_hi - W_lo, and two Gram anchors with no middle anchor between them must get
// the SAME number (their entry can be as small as exp(-2 gap) of the nearest middle anchor, next to which a
// rounding difference of two prefix sums associated differently is enormous).  So every stretch between two
// neighbouring middle anchors has ONE value of W, whichever thread or workgroup evaluates it: see k_g64_down.
// The regions are taken by POSITION in the stable merged order, so a middle anchor equal to a Gram
// anchor lies in exactly one of them, and each region's closed form holds at a tie by continuity.
// Only non-positive numbers are ever exponentiated (the theorem's interval statistic e^{2(a_i - b_t)}
// overflows on wide intervals; the merged scan never forms it).
//
// U, V and W come from a scan of their own (tile summaries, downsweep; a spine between them when there are many tiles) over the
// plan of the doubled anchors; a segment is summarised by (D, S) with F_out = D F_in + S in each direction.
// Everything between the fp32 anchors and the result is fp64, for the fp32 entry point too: the fill
// subtracts two prefix sums of the weights, and with weights of one sign an fp32 prefix of a million terms
// has lost the digits of a short interval; and the device's fp64 rate makes the wider type free here (the
// kernels wait for memory and for each other).  The fp64 entry point (App. "Density model", training: the
// Gram matrices run in fp64 through the same scan) differs only in the types of the weights and the result.
#include "laplex_internal.h"

namespace laplex {

namespace {

constexpr int kWThreads = 256;
constexpr int kWItems = 8;
constexpr int kWTile = kWThreads * kWItems;      // merged positions per workgroup
constexpr int kWSpineThreads = 1024;
// Up to this many tiles the downsweep adds up the summaries of all other tiles itself (each decayed by one exponential of an
// anchor difference); beyond it the summaries go through a spine kernel first.
constexpr int64_t kWDirectTiles = 2048;

__device__ __forceinline__ double wave_inclusive_scan_f64(double v)
{
    const int lane = threadIdx.x & 63;
#pragma unroll
    for (int s = 1; s < 64; s <<= 1) {
        const double o = __shfl_up(v, s);
        if (lane >= s) v += o;
    }
    return v;
}

// Sums of NV doubles per thread over the workgroup, in a fixed order; every thread gets them.
template <int THREADS, int NV>
__device__ __forceinline__ void block_sum_f64(double (&v)[NV])
{
    __shared__ double part[THREADS / 64][NV];
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
#pragma unroll
    for (int m = 32; m >= 1; m >>= 1)
#pragma unroll
        for (int q = 0; q < NV; ++q) v[q] += __shfl_xor(v[q], m);
    if (lane == 0)
#pragma unroll
        for (int q = 0; q < NV; ++q) part[wave][q] = v[q];
    __syncthreads();
#pragma unroll
    for (int q = 0; q < NV; ++q) {
        v[q] = 0.0;
#pragma unroll
        for (int w = 0; w < THREADS / 64; ++w) v[q] += part[w][q];
    }
    __syncthreads();
}

struct Pair64 { double D, S; };

__device__ __forceinline__ Pair64 pair_then(const Pair64& first, const Pair64& second)
{
    return Pair64{first.D * second.D, second.D * first.S + second.S};
}

// Exclusive scan of one pair per thread over the workgroup, in thread order (FWD) or against it; *total = all of them.
template <int THREADS, bool FWD>
__device__ __forceinline__ Pair64 block_exclusive_scan_pair(Pair64 v, Pair64* total)
{
    constexpr int WAVES = THREADS / 64;
    __shared__ double wD[WAVES], wS[WAVES];
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    Pair64 inc = v;
#pragma unroll
    for (int s = 1; s < 64; s <<= 1) {
        const Pair64 o = FWD ? Pair64{__shfl_up(inc.D, s), __shfl_up(inc.S, s)} : Pair64{__shfl_down(inc.D, s), __shfl_down(inc.S, s)};
        if (FWD ? lane >= s : lane + s < 64) inc = pair_then(o, inc);
    }
    if (lane == (FWD ? 63 : 0)) { wD[wave] = inc.D; wS[wave] = inc.S; }
    Pair64 before = FWD ? Pair64{__shfl_up(inc.D, 1), __shfl_up(inc.S, 1)} : Pair64{__shfl_down(inc.D, 1), __shfl_down(inc.S, 1)};
    if (lane == (FWD ? 0 : 63)) before = Pair64{1.0, 0.0};
    __syncthreads();
    Pair64 head{1.0, 0.0}, all{1.0, 0.0};
#pragma unroll
    for (int q = 0; q < WAVES; ++q) {
        const int w = FWD ? q : WAVES - 1 - q;
        const Pair64 t{wD[w], wS[w]};
        if (FWD ? w < wave : w > wave) head = pair_then(head, t);
        all = pair_then(all, t);
    }
    *total = all;
    __syncthreads();
    return pair_then(head, before);
}

// Tile summaries, and the weights in sorted order (zero at Gram anchors) for the downsweep: the gather of d by sorted id is what
// this kernel waits for, and it is done once.  A tile's state from zero is a plain weighted sum with the weights from the anchors,
//   S_f = sum_i w_i exp(-(p_last - p_i)),   S_b = sum_i w_i exp(-(p_i - p_first)),
// so the positions are read in coalesced order and nothing is scanned.  (Serial walks over positions staged in LDS, sixteen
// consecutive doubles per thread, queued 64 lanes on one LDS bank and took 28 us at 2^20 positions; the downsweep in the same
// manner 38 us, with a spine and a pick-up of W of 11 us between and behind them.  Now 12.8 and 11.1 us.)
// summ: [6][tiles] = forward (D, S), backward (D, S), sum of the weights, number of middle anchors
template <typename TW>
__global__ void __launch_bounds__(kWThreads)
k_g64_tiles(const uint32_t* __restrict__ ids, const float* __restrict__ pk, const TW* __restrict__ d,
            uint32_t k, int64_t N, int64_t tiles, double* __restrict__ summ, TW* __restrict__ sorted)
{
    const int64_t base = (int64_t)blockIdx.x * kWTile;
    const int64_t end = base + kWTile < N ? base + kWTile : N;
    const double p_first = (double)pk[base + 1], p_last = (double)pk[end];       // pk is shifted by one
    uint32_t id[kWItems];
    float p[kWItems];
    TW w[kWItems];
#pragma unroll
    for (int i = 0; i < kWItems; ++i) {
        const int64_t j = base + i * kWThreads + threadIdx.x;
        const int64_t jc = j < N ? j : N - 1;
        id[i] = ids[jc];
        if (j >= N) id[i] = 0u;            // (a Gram anchor's id: no weight)
        p[i] = pk[jc + 1];
    }
#pragma unroll
    for (int i = 0; i < kWItems; ++i) w[i] = d[id[i] >= k ? id[i] - k : 0u];
    double v[4] = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
    for (int i = 0; i < kWItems; ++i) {
        const int64_t j = base + i * kWThreads + threadIdx.x;
        const bool middle = id[i] >= k;
        if (!middle) w[i] = TW(0);
        if (j < N) sorted[j] = w[i];
        if (middle) {
            const double wd = (double)w[i];
            v[0] += wd * exp(-(p_last - (double)p[i]));
            v[1] += wd * exp(-((double)p[i] - p_first));
            v[2] += wd;
            v[3] += 1.0;                   // counts stay exact in fp64
        }
    }
    block_sum_f64<kWThreads, 4>(v);
    if (threadIdx.x == 0) {
        summ[0 * tiles + blockIdx.x] = exp(-(p_last - (double)pk[base])); summ[1 * tiles + blockIdx.x] = v[0];
        summ[2 * tiles + blockIdx.x] = exp(-((double)pk[end + 1] - p_first)); summ[3 * tiles + blockIdx.x] = v[1];
        summ[4 * tiles + blockIdx.x] = v[2];
        summ[5 * tiles + blockIdx.x] = v[3];
    }
}

// Many tiles: in place, summ[1][t] <- forward state entering tile t, summ[3][t] <- backward state entering it (from the right),
// summ[4][t] <- weights before it: the inclusive sum through the last tile before t that holds a middle anchor, so that tiles
// without one pass the same bits on.  One workgroup, kWSpineThreads tiles at a time.
__global__ void __launch_bounds__(kWSpineThreads)
k_g64_spine(double* __restrict__ summ, int64_t tiles)
{
    __shared__ double incl[kWSpineThreads];
    __shared__ double wtot[kWSpineThreads / 64];
    __shared__ int wlast[kWSpineThreads / 64];
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    double cF = 0.0, cW = 0.0;
    for (int64_t c0 = 0; c0 < tiles; c0 += kWSpineThreads) {
        const int64_t t = c0 + threadIdx.x;
        const bool ok = t < tiles;
        Pair64 v{ok ? summ[0 * tiles + t] : 1.0, ok ? summ[1 * tiles + t] : 0.0}, tot;
        const Pair64 ex = block_exclusive_scan_pair<kWSpineThreads, true>(v, &tot);
        const double inc = wave_inclusive_scan_f64(ok ? summ[4 * tiles + t] : 0.0);
        const uint64_t has = __ballot(ok && summ[5 * tiles + t] > 0.0);
        if (lane == 63) wtot[wave] = inc;
        if (lane == 0) wlast[wave] = has ? (wave << 6) + 63 - __clzll((long long)has) : -1;
        __syncthreads();
        double head = 0.0;
        int last = -1, last_all = -1;
        for (int w = 0; w < kWSpineThreads / 64; ++w) {
            if (w < wave) { head += wtot[w]; if (wlast[w] >= 0) last = wlast[w]; }
            if (wlast[w] >= 0) last_all = wlast[w];
        }
        incl[threadIdx.x] = cW + (head + inc);
        const uint64_t below = has & ((1ull << lane) - 1ull);
        if (below) last = (wave << 6) + 63 - __clzll((long long)below);
        __syncthreads();
        const double enter = last >= 0 ? incl[last] : cW;
        if (ok) { summ[1 * tiles + t] = ex.D * cF + ex.S; summ[4 * tiles + t] = enter; }
        cF = tot.D * cF + tot.S;
        if (last_all >= 0) cW = incl[last_all];
        __syncthreads();
    }
    double cB = 0.0;
    const int64_t chunks = (tiles + kWSpineThreads - 1) / kWSpineThreads;
    for (int64_t c = chunks - 1; c >= 0; --c) {
        const int64_t t = c * kWSpineThreads + threadIdx.x;
        const bool ok = t < tiles;
        Pair64 v{ok ? summ[2 * tiles + t] : 1.0, ok ? summ[3 * tiles + t] : 0.0}, tot;
        const Pair64 ex = block_exclusive_scan_pair<kWSpineThreads, false>(v, &tot);
        if (ok) summ[3 * tiles + t] = ex.D * cB + ex.S;
        cB = tot.D * cB + tot.S;
    }
}

// dst[0..8) = src[row0 .. row0 + 8), zero past the end
template <typename T>
__device__ __forceinline__ void load_eight(const T* __restrict__ src, int64_t row0, int64_t N, T (&dst)[kWItems])
{
    if (row0 + kWItems <= N) {
        typedef T vec __attribute__((ext_vector_type(16 / sizeof(T))));
        constexpr int per = 16 / (int)sizeof(T);
#pragma unroll
        for (int q = 0; q < kWItems / per; ++q) {
            const vec t = reinterpret_cast<const vec*>(src + row0)[q];
#pragma unroll
            for (int e = 0; e < per; ++e) dst[q * per + e] = t[e];
        }
    } else {
#pragma unroll
        for (int i = 0; i < kWItems; ++i) dst[i] = row0 + i < N ? src[row0 + i] : T(0);
    }
}

// One workgroup per tile, eight consecutive positions per thread, everything in registers; a tile without Gram anchors has
// nothing to do.  SPINE: the states entering the tile come from k_g64_spine; otherwise each thread adds up its share of the
// other tiles' summaries, each decayed by one exponential of an anchor difference.
//
// The value of W between two neighbouring middle anchors m, m' is
//   the thread's own running sum           if m' lies in the same thread's eight positions as m,
//   the inclusive sum through m's thread   if m' lies in a later thread of the tile,
//   the sum entering the next tile         if m is the last middle anchor of its tile (and there is a next tile),
// and the next tile takes the very same number for the Gram anchors before its first middle anchor.
// status: the plan's status word, or null for plans that are always valid; an invalid plan (the radix sort gave up a wait)
// turns W, and with it every entry of the matrix, into a NaN.
template <typename TW, bool SPINE>
__global__ void __launch_bounds__(kWThreads)
k_g64_down(const uint32_t* __restrict__ ids, const float* __restrict__ pk, const TW* __restrict__ sorted,
           uint32_t k, int64_t N, int64_t tiles, const double* __restrict__ summ,
           double* __restrict__ U, double* __restrict__ V, double* __restrict__ W, const uint32_t* __restrict__ status)
{
    constexpr int WAVES = kWThreads / 64;
    __shared__ double wtot[WAVES], wlast[WAVES];
    __shared__ int whas[WAVES];
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    const int64_t tile = blockIdx.x, base = tile * kWTile;
    const int64_t end = base + kWTile < N ? base + kWTile : N;
    if (summ[5 * tiles + tile] == (double)(end - base)) return;        // uniform: no Gram anchor here

    const int64_t row0 = base + (int64_t)threadIdx.x * kWItems;
    uint32_t id[kWItems];
    TW wv[kWItems];
    float p[kWItems + 2];                  // anchors of positions row0 - 1 .. row0 + 8
    load_eight(ids, row0, N, id);
    load_eight(sorted, row0, N, wv);
    {
        float t[kWItems];
        load_eight(pk, row0, N + 2, t);
#pragma unroll
        for (int i = 0; i < kWItems; ++i) p[i] = t[i];
        p[kWItems] = row0 + kWItems <= N + 1 ? pk[row0 + kWItems] : 0.0f;
        p[kWItems + 1] = row0 + kWItems + 1 <= N + 1 ? pk[row0 + kWItems + 1] : 0.0f;
    }
    // states entering the tile
    double F, R, cW, nW;
    if (SPINE) {
        F = summ[1 * tiles + tile]; R = summ[3 * tiles + tile]; cW = summ[4 * tiles + tile];
        nW = tile + 1 < tiles ? summ[4 * tiles + tile + 1] : 0.0;
    } else {
        double v[4] = {0.0, 0.0, 0.0, 0.0};
        const double p_before = (double)pk[base], p_after = (double)pk[end + 1];
        for (int64_t s = threadIdx.x; s < tiles; s += kWThreads) {
            const double ws = summ[4 * tiles + s];
            if (s < tile) {
                v[0] += summ[1 * tiles + s] * exp(-(p_before - (double)pk[(s + 1) * kWTile]));      // from the last position of tile s
                v[2] += ws;
            } else if (s > tile) {
                v[1] += summ[3 * tiles + s] * exp(-((double)pk[s * kWTile + 1] - p_after));         // from the first position of tile s
            }
            if (s <= tile) v[3] += ws;
        }
        block_sum_f64<kWThreads, 4>(v);
        F = v[0]; R = v[1]; cW = v[2]; nW = v[3];
    }

    // decay into position i from its left neighbour (i = 8: into the first position of the next thread); 1 past the end
    double dec[kWItems + 1];
#pragma unroll
    for (int i = 0; i <= kWItems; ++i)
        dec[i] = row0 + i <= N && row0 < N ? exp(-((double)p[i + 1] - (double)p[i])) : 1.0;
    Pair64 f{1.0, 0.0}, b{1.0, 0.0};
    double wsum = 0.0;
    uint32_t mid = 0u;                     // bit i: position i is a middle anchor
#pragma unroll
    for (int i = 0; i < kWItems; ++i) {
        const int r = kWItems - 1 - i;
        const double wi = (double)wv[i], wr = (double)wv[r];
        const bool live = row0 + i < N, live_r = row0 + r < N;
        const double df = live ? dec[i] : 1.0, db = live_r ? dec[r + 1] : 1.0;
        f = Pair64{f.D * df, df * f.S + wi};
        b = Pair64{b.D * db, db * b.S + wr};
        wsum += wi;
        mid |= (live && id[i] >= k) ? 1u << i : 0u;
    }
    Pair64 tot;
    const Pair64 ef = block_exclusive_scan_pair<kWThreads, true>(f, &tot);
    const Pair64 eb = block_exclusive_scan_pair<kWThreads, false>(b, &tot);
    F = ef.D * F + ef.S;
    R = eb.D * R + eb.S;

    const double inc = wave_inclusive_scan_f64(wsum);
    double exc = __shfl_up(inc, 1);
    if (lane == 0) exc = 0.0;
    const uint64_t has = __ballot(mid != 0u);
    const double at_last = __shfl(inc, has ? 63 - __clzll((long long)has) : 0);
    if (lane == 63) { wtot[wave] = inc; wlast[wave] = at_last; whas[wave] = has != 0ull; }
    __syncthreads();
    double head = 0.0, before = cW;        // before: W up to the first middle anchor of this thread, as far as this tile knows
    bool any_before = false, any_after = false;
#pragma unroll
    for (int w = 0; w < WAVES; ++w) {
        if (w < wave) {
            if (whas[w]) { before = cW + (head + wlast[w]); any_before = true; }
            head += wtot[w];
        } else if (w > wave && whas[w]) {
            any_after = true;
        }
    }
    const uint64_t below = has & ((1ull << lane) - 1ull);
    const double in_wave = __shfl(inc, below ? 63 - __clzll((long long)below) : 0);
    if (below) { before = cW + (head + in_wave); any_before = true; }
    any_after = any_after || ((has >> lane) >> 1) != 0ull;
    const bool next_tile = tile + 1 < tiles;
    if (any_before && mid == 0u && !any_after && next_tile) before = nW;       // the last middle anchor of the tile is behind
    const double after = (!any_after && next_tile) ? nW : cW + (head + inc);   // W after the thread's last middle anchor
    const double start = cW + (head + exc);
    const bool invalid = status != nullptr && *status != 0u;
    const double poison = invalid ? __longlong_as_double(0x7FF8000000000000LL) : 0.0;

    double run = 0.0;
#pragma unroll
    for (int i = 0; i < kWItems; ++i) {
        const int r = kWItems - 1 - i;
        const bool live = row0 + i < N, live_r = row0 + r < N;
        F = (live ? dec[i] : 1.0) * F + (double)wv[i];
        R = (live_r ? dec[r + 1] : 1.0) * R + (double)wv[r];
        run += (double)wv[i];
        // a Gram anchor carries no weight: F, R are the sums strictly beside it
        if (live && id[i] < k) {
            const bool seen = (mid & ((1u << i) - 1u)) != 0u, more = (mid >> i) != 0u;
            U[id[i]] = F;
            W[id[i]] = (!seen ? before : more ? start + run : after) + poison;
        }
        if (live_r && id[r] < k) V[id[r]] = R;
    }
}

// The fill: one thread per four consecutive columns of one row; lo / hi of a pair by (anchor, index), the
// stable merged order.
template <typename TM>
__global__ void __launch_bounds__(256)
k_wgram_fill(const float* __restrict__ a, const double* __restrict__ U, const double* __restrict__ V,
             const double* __restrict__ W, int64_t k, TM* __restrict__ M, int64_t ldm, int vec4)
{
    const int64_t i = blockIdx.x;
    const int64_t j0 = ((int64_t)blockIdx.y * blockDim.x + threadIdx.x) * 4;
    if (j0 >= k) return;
    const float ai = a[i];
    const double Ui = U[i], Vi = V[i], Wi = W[i];
    TM out[4];
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        const int64_t j = j0 + e < k ? j0 + e : k - 1;
        const float aj = a[j];
        const bool i_first = ai < aj || (ai == aj && i <= j);
        const double inner = i_first ? Ui + (W[j] - Wi) + V[j] : U[j] + (Wi - W[j]) + Vi;
        out[e] = (TM)(exp(-fabs((double)ai - (double)aj)) * inner);
    }
    TM* row = M + i * ldm;
    if (sizeof(TM) == 4 && vec4 && j0 + 4 <= k) {
        typedef float v4f __attribute__((ext_vector_type(4)));
        __builtin_nontemporal_store((v4f){(float)out[0], (float)out[1], (float)out[2], (float)out[3]}, reinterpret_cast<v4f*>(row + j0));
    } else {
#pragma unroll
        for (int e = 0; e < 4; ++e)
            if (j0 + e < k) row[j0 + e] = out[e];
    }
}

}  // namespace

int64_t wgram_tiles(int64_t N);

template <typename TW, typename TM>
hipError_t launch_wgram_t(const uint32_t* ids, const float* pk, const float* a, const TW* d, int64_t k, int64_t N,
                          double* summ, double* U, double* V, double* W, void* sorted, TM* M, int64_t ldm,
                          const uint32_t* status, hipStream_t st)
{
    const int64_t tiles = wgram_tiles(N);
    const dim3 grid_t((unsigned)tiles), block(kWThreads);
    TW* const ws = static_cast<TW*>(sorted);
    LAPLEX_TIMED("wgram_scan", st, hipLaunchKernelGGL((k_g64_tiles<TW>), grid_t, block, 0, st, ids, pk, d, (uint32_t)k, N, tiles, summ, ws));
    if (tiles > kWDirectTiles) {
        LAPLEX_TIMED("wgram_scan", st, hipLaunchKernelGGL(k_g64_spine, dim3(1), dim3(kWSpineThreads), 0, st, summ, tiles));
        LAPLEX_TIMED("wgram_scan", st, hipLaunchKernelGGL((k_g64_down<TW, true>), grid_t, block, 0, st, ids, pk, (const TW*)ws, (uint32_t)k, N, tiles,
                                                          (const double*)summ, U, V, W, status));
    } else {
        LAPLEX_TIMED("wgram_scan", st, hipLaunchKernelGGL((k_g64_down<TW, false>), grid_t, block, 0, st, ids, pk, (const TW*)ws, (uint32_t)k, N, tiles,
                                                          (const double*)summ, U, V, W, status));
    }
    const int vec4 = (reinterpret_cast<uintptr_t>(M) & 15u) == 0 && ldm % 4 == 0;
    const dim3 grid((unsigned)k, (unsigned)((k + 1023) / 1024));     // rows on x (up to 2^31 - 1), column chunks on y
    LAPLEX_TIMED("wgram_fill", st, hipLaunchKernelGGL((k_wgram_fill<TM>), grid, dim3(256), 0, st,
                                                      a, (const double*)U, (const double*)V, (const double*)W, k, M, ldm, vec4));
    return hipGetLastError();
}

int64_t wgram_tiles(int64_t N) { return (N + kWTile - 1) / kWTile; }

hipError_t launch_wgram_f32(const uint32_t* ids, const float* pk, const float* a, const float* d, int64_t k, int64_t N,
                            double* summ, double* U, double* V, double* W, void* sorted, float* M, int64_t ldm,
                            const uint32_t* status, hipStream_t st)
{
    return launch_wgram_t<float, float>(ids, pk, a, d, k, N, summ, U, V, W, sorted, M, ldm, status, st);
}

hipError_t launch_wgram_f64(const uint32_t* ids, const float* pk, const float* a, const double* d, int64_t k, int64_t N,
                            double* summ, double* U, double* V, double* W, void* sorted, double* M, int64_t ldm,
                            const uint32_t* status, hipStream_t st)
{
    return launch_wgram_t<double, double>(ids, pk, a, d, k, N, summ, U, V, W, sorted, M, ldm, status, st);
}

}  // namespace laplex

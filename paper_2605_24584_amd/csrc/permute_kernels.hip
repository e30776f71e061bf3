// Results of batch 1 back to the caller's order without random accesses (the scatter of S7; Sec. 3 "Complexity": the permutation is the
// price of sorting arbitrary anchors).
//
// At batch 1 a row is one float.  Storing a result at y[id] costs a partial line and is bound by the number of memory
// transactions, not by bytes.  Here every result travels as a record (destination, value[, value]) through at most two partition
// levels, each of which reads its records once and writes them once in runs, and a last pass that places the records of one window of
// 16384 (8192, see permute_window_bits) consecutive destinations inside LDS and writes the window out whole:
//
//   level 1   the batch-1 downsweep places its results itself, into up to 512 buckets by the top bits of the destination (or, with
//             at most 512 windows, into the windows)
//   level 2   the records of one bucket -> its (up to 512) windows
//   final     one workgroup per window: scatter inside LDS, coalesced store (destinations that no record
//             names read as zero)
//
// Destinations are positions of a permutation, so a bucket that covers C destinations receives at most C
// records: its region in the record arrays is simply the stretch [first destination, first + C).  No
// histogram pass is needed, nothing has to be stable and no tile waits for another: a tile ranks its records
// with returning LDS atomics and reserves the stretch for each of its runs with ONE returning atomic on the
// bucket's cursor (device scope).  Measured on this device: 512 such atomics per tile of 64 KB, all tiles on
// the same 512 words, cost 15 % on top of a plain copy of the tile.  The order of the records inside a bucket
// depends on the order in which the atomics land; the result does not (every destination is written once).
// (The way in, x and gy into the sorted order, follows the sort's own passes: deep_sort_kernels.hip.)
#include "permute_tile.h"

#include <string>

namespace laplex {

namespace {

constexpr int kPtThreads = 1024;
constexpr int kPtPer = 16;                               // records per thread
constexpr int kPtTile = kPtThreads * kPtPer;             // 16384 records per tile: a run is 32 records on average with 512 buckets
static_assert(kPtTile == (1 << kPermuteWindowBits), "a tile of level 2 is one window's worth of records");

struct PartArgs {
    const uint2* in_dv; const float* in_v1;             // records of the level before: (destination, first value), second value ...
    const uint32_t* in_len;                             // ... and how many each of its buckets holds (its cursors)
    int chain_bits;                // a bucket of the level before is read by 2^chain_bits consecutive tiles
    PartEmit emit;                 // this level
};

// The second partition level.  NV: values per record (1 or 2).
template <int NV>
__global__ void __launch_bounds__(kPtThreads)
k_part(const PartArgs A)
{
    __shared__ PartShared<kPtThreads> S;
    __shared__ uint2 sdv[kPtTile];                  // the tile's records, bucket by bucket: (destination, first value); then the second values
    const int tid = threadIdx.x;
    const int64_t tile = blockIdx.x;
    const int64_t chain = tile >> A.chain_bits;
    const int64_t chunk = tile & (((int64_t)1 << A.chain_bits) - 1);

    // the tile's source records
    uint32_t bucket_len = A.in_len[chain];                  // records of this bucket of the level before
    const uint32_t cap = 1u << (A.chain_bits + kPermuteWindowBits);
    bucket_len = bucket_len < cap ? bucket_len : cap;       // (a valid plan never fills a region beyond its size)
    const int64_t base = chain << A.chain_bits << kPermuteWindowBits;     // 2^chain_bits tiles cover the bucket's region
    const int64_t src0 = base + chunk * kPtTile, src1 = base + bucket_len < src0 + kPtTile ? base + bucket_len : src0 + kPtTile;
    if (src0 >= src1) return;

    uint32_t dest[kPtPer];
    float v0[kPtPer], v1[NV == 2 ? kPtPer : 1];
    uint32_t okmask = 0u;
#pragma unroll
    for (int i = 0; i < kPtPer; ++i) {
        const int64_t j = src0 + i * kPtThreads + tid;
        const bool in = j < src1;
        const int64_t jc = in ? j : src0;
        const uint2 dv = A.in_dv[jc];
        dest[i] = dv.x; v0[i] = __uint_as_float(dv.y);
        if (NV == 2) v1[i] = A.in_v1[jc];
        okmask |= in && (int64_t)dest[i] < A.emit.dest_count ? 1u << i : 0u;      // (the latter always, for a valid plan)
    }
    PartTicket<kPtPer> K;
    partition_reserve<kPtThreads, kPtPer>(A.emit, chain, dest, okmask, S, K);
    partition_place<kPtThreads, kPtPer, NV>(A.emit, chain, dest, okmask, v0, v1, S, sdv, K);
}

struct FinalArgs {
    const uint2* in_dv; const float* in_v1;
    const uint32_t* in_len;                        // records of each window (the cursors of the level that filled them)
    float* out0; int64_t ld0; float* out1; int64_t ld1;
    int64_t dest_count;
    const uint32_t* poison;                        // the plan's status word, or null (never for the plan's own arrays)
};

// The last pass: one workgroup per window of 2^BITS consecutive destinations.  The windows are taken from the last one down: the level
// before it fills them in ascending order, so the records it wrote last are still in the 256 MB memory-side cache (us, ascending /
// descending, 2^25 positions, two values: 82 -> 73).
template <int NV, int BITS>
__global__ void __launch_bounds__(kPtThreads)
k_part_final(const FinalArgs A)
{
    constexpr int W = 1 << BITS;
    __shared__ float s0[W];
    __shared__ float s1[NV == 2 ? W : 1];
    const int tid = threadIdx.x;
    const int64_t w = (int64_t)(gridDim.x - 1u - blockIdx.x);
    uint32_t count = A.in_len[w];
    if (count > (uint32_t)W) count = (uint32_t)W;
    for (int i = tid; i < W; i += kPtThreads) { s0[i] = 0.0f; if (NV == 2) s1[i] = 0.0f; }
    __syncthreads();
    const int64_t base = w << BITS;
    for (uint32_t i = tid; i < count; i += kPtThreads) {
        const uint2 dv = A.in_dv[base + i];
        const uint32_t d = dv.x & (uint32_t)(W - 1);
        s0[d] = __uint_as_float(dv.y);
        if (NV == 2) s1[d] = A.in_v1[base + i];
    }
    __syncthreads();
    const uint32_t poison = (A.poison != nullptr && *A.poison != 0u) ? 0x7FC00000u : 0u;
    for (int i = tid; i < W; i += kPtThreads) {
        const int64_t d = base + i;
        if (d < A.dest_count) {
            A.out0[d * A.ld0] = __uint_as_float(__float_as_uint(s0[i]) | poison);
            if (NV == 2) A.out1[d * A.ld1] = __uint_as_float(__float_as_uint(s1[i]) | poison);
        }
    }
}

int ceil_log2(int64_t v) { int l = 0; while (((int64_t)1 << l) < v) ++l; return l; }

}  // namespace

bool permute_supported(int64_t dest_count)
{
    if (dest_count <= 0) return false;
    const int bits = permute_window_bits(dest_count);
    const int64_t windows = (dest_count + (1 << bits) - 1) >> bits;
    return ceil_log2(windows) <= 2 * kPermuteMaxBucketBits;
}

size_t permute_cursor_words(int64_t dest_count)
{
    // level 1: at most 2^9 buckets; level 2 (or the only level): one cursor per window, padded to a power of two
    const int bits = permute_window_bits(dest_count);
    const int64_t windows = (dest_count + (1 << bits) - 1) >> bits;
    return (size_t)(((int64_t)1 << kPermuteMaxBucketBits) + ((int64_t)1 << ceil_log2(windows)));
}

namespace {
struct Geom { int bits, lw, p1, p2; int64_t windows, tiles2; };
Geom geom_of(int64_t dest_count)
{
    Geom g;
    g.bits = permute_window_bits(dest_count);
    g.windows = (dest_count + (1 << g.bits) - 1) >> g.bits;
    g.lw = ceil_log2(g.windows);
    g.p2 = g.lw < kPermuteMaxBucketBits ? g.lw : kPermuteMaxBucketBits;
    g.p1 = g.lw - g.p2;
    g.tiles2 = (int64_t)1 << (g.p1 + g.p2);
    return g;
}
}  // namespace

void permute_begin(const PermuteJob& J, PartEmit* first_level)
{
    const Geom g = geom_of(J.dest_count);
    uint32_t* const cursor1 = J.cursors;                                          // level 1's buckets
    uint32_t* const cursor2 = J.cursors + ((int64_t)1 << kPermuteMaxBucketBits);  // the windows
    PartEmit E;
    E.clear = J.cursors; E.clear_words = ((int64_t)1 << kPermuteMaxBucketBits) + ((int64_t)1 << g.lw);
    E.out_dv = J.rec_dv[0]; E.out_v1 = J.rec_v1[0]; E.dest_count = J.dest_count;
    if (g.p1 > 0) {      // two levels: the first one fills 2^p1 buckets of 2^p2 windows each
        E.bucket_bits = g.p1; E.shift = kPermuteWindowBits + g.p2; E.region_shift = kPermuteWindowBits + g.p2; E.cursor = cursor1;
    } else {             // one level: straight into the windows
        E.bucket_bits = g.p2; E.shift = g.bits; E.region_shift = g.bits; E.cursor = cursor2;
    }
    *first_level = E;
}

hipError_t permute_finish(const PermuteJob& J, hipStream_t st)
{
    const Geom g = geom_of(J.dest_count);
    uint32_t* const cursor1 = J.cursors;
    uint32_t* const cursor2 = J.cursors + ((int64_t)1 << kPermuteMaxBucketBits);
    const std::string f1 = std::string("permute_part.") + J.tag, f2 = std::string("permute_final.") + J.tag;
    FinalArgs F{};
    F.dest_count = J.dest_count; F.out0 = J.out0; F.ld0 = J.ld0; F.out1 = J.out1; F.ld1 = J.ld1; F.poison = J.poison;
    F.in_len = cursor2;
    F.in_dv = J.rec_dv[0]; F.in_v1 = J.rec_v1[0];
    if (g.p1 > 0) {      // level 2: each bucket of level 1 -> its windows, records into the second buffer
        PartArgs A{};
        A.in_dv = J.rec_dv[0]; A.in_v1 = J.rec_v1[0]; A.in_len = cursor1;
        A.chain_bits = g.p2;
        A.emit.bucket_bits = g.p2; A.emit.shift = kPermuteWindowBits; A.emit.region_shift = kPermuteWindowBits;
        A.emit.out_dv = J.rec_dv[1]; A.emit.out_v1 = J.rec_v1[1]; A.emit.cursor = cursor2; A.emit.dest_count = J.dest_count;
        if (J.values == 2) LAPLEX_TIMED(f1.c_str(), st, hipLaunchKernelGGL((k_part<2>), dim3((unsigned)g.tiles2), dim3(kPtThreads), 0, st, A));
        else LAPLEX_TIMED(f1.c_str(), st, hipLaunchKernelGGL((k_part<1>), dim3((unsigned)g.tiles2), dim3(kPtThreads), 0, st, A));
        F.in_dv = J.rec_dv[1]; F.in_v1 = J.rec_v1[1];
    }
    auto last = [&](auto kernel) { LAPLEX_TIMED(f2.c_str(), st, hipLaunchKernelGGL(kernel, dim3((unsigned)g.windows), dim3(kPtThreads), 0, st, F)); };
    constexpr int B = kPermuteWindowBits;
    if (g.bits == B) { if (J.values == 2) last(k_part_final<2, B>); else last(k_part_final<1, B>); }
    else { if (J.values == 2) last(k_part_final<2, B - 1>); else last(k_part_final<1, B - 1>); }
    return hipGetLastError();
}

}  // namespace laplex

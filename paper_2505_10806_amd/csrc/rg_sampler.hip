// Epoch schedule and multi-hop neighbour sampling (Alg. 1 line 1; SAMPLE(eta(v), k) of Section II-B).
//
// Data layout in HBM: CSR (row_ptr int32/int64, col_idx int32) is read-only; the batch's cumulative
// frontier `nodes` grows tier by tier; `visited` is the N-bit bitmap of its members.  A hop's new tier is found in one of
// five ways (TierMode below); a member's position comes from the tier's rank blocks or from `pos[v]`.  All sizes that
// depend on the data (frontier and edge counts) stay on the device: launches are sized by static upper bounds and
// kernels read the actual counts.
#include <string.h>

#include <type_traits>

#include "rg_internal.h"

namespace {

constexpr int kChunk = 1024;         // frontier nodes per workgroup in the count kernel: the unit of hop_sum

// How the ids a hop has sampled become its new tier.
//  kTierSliced    (ascending order) no marking during the draw.  A workgroup owns an id range of slice_words * 32 ids as a bitmap
//                 in LDS and reads the hop's whole edge list (or one split of it) for the ids of its range.  Measured on hop 2
//                 of 8 batches of 4096 seeds at N = 10 M (15.9 M edges): reading col_idx and writing nbr took 207 us, with
//                 one global atomicOr per edge behind a probe 717 us (37 G atomics/s, the same for every scope), with a
//                 byte store per edge 341 us; the LDS pass adds 44 us.  (Since batches share lines of col_idx the reading takes 163.)
//  kTierAtomic    (ascending order) one probe and at most one atomicOr per edge on the bitmap `marked`.
//  kTierBytes     (ascending order) a byte store per edge by the draw, then one or two launches per hop where slices take three.
//  kTierFirstSeen (first-seen order) the first edge of the hop that names a node is kept per node (atomicMax).
//  kTierRankedSeen (first-seen order) the tier is found as in kTierSliced, which gives its nodes their ascending positions; the
//                 first edges are kept by those (N / 6 bytes of rank blocks and 4 bytes per new node instead of 4 N scattered
//                 bytes), edges that open a node are counted and emitted in edge order, and `place` maps one position to the
//                 other.  See rg_use_ranked_seen for the line between the two.
// The sliced way moves about N bytes per hop whatever the edges, and every slice reads every edge; the atomic way costs 27 ps
// per edge.  Whole call, sliced against atomic: 8 batches of 4096 seeds (15,10,5) at N = 10 M 586 / 1700 us, at 40 M 733 / 1026 (before
// rows were shared and ranks packed, which made it 715 at 10 M), at 100 M (80 slices) 1312 / 841; 8 batches of 64 seeds (10,5) at N = 10 M 102 / 92 us, at 40 M 239 / 160; on smaller graphs
// both are bound by their launches, of which the sliced way has fewer.
// The edges of this line, and of the other lines between kernels, are those of nodes of average degree (rg_expected_edges), not the
// static bound, which for RG_FANOUT_ALL is every edge of the graph: one batch of 16 seeds, all neighbours of one / two / three hops,
// N = 10 M with 20 edges per node 39 / 67 / 116 us by the atomic way, 50 / 106 / 172 by slices.
// by_threads: every hop is drawn by threads or lanes.  Such calls of less than N / 16 edges take the atomic way from 512 Ki nodes on, where they
// don't take bytes and name 256 Ki edges at most in all: eight batches of 19 k edges on 1.2 M nodes 50 / 58 us, on 2 M 52 / 61, of 9 k in three hops on
// 1.2 M 61 / 78, one of 144 k on 4.1 M 55 / 67.  Of more edges the hubs' words queue up: eight of 33 k on 0.7 M nodes of 105 neighbours 67 / 58, three
// of 170 k on 3 M 104 / 98, eight of 157 k on 3.7 M 144 / 97.
inline bool rg_use_slices(int slices, int64_t num_nodes, int64_t edges, int group, bool by_threads) {
    if (slices <= 0) return false;
    const bool few = by_threads && edges * group <= 256ll << 10;
    return num_nodes <= (few ? 512ll << 10 : 4ll << 20) || edges >= num_nodes / 16;
}
// Edges per hop of a batch of `seeds` nodes whose degrees are the graph's average, eub[] at most; returns their sum.
inline int64_t rg_expected_edges(int64_t num_nodes, int64_t num_edges, int64_t seeds, const int32_t* fanouts, int num_hops,
                                 const int64_t* eub, int64_t* expected) {
    const double degree = num_nodes > 0 ? (double)num_edges / (double)num_nodes : 0.0;
    double frontier = (double)seeds;
    int64_t sum = 0;
    for (int h = 0; h < num_hops; ++h) {
        const double per_node = fanouts[h] < 0 || (double)fanouts[h] > degree ? degree : (double)fanouts[h];
        expected[h] = rg_min64(eub[h], (int64_t)(frontier * per_node) + 1);
        frontier += (double)expected[h];
        if (frontier > (double)num_nodes) frontier = (double)num_nodes;
        sum += expected[h];
    }
    return sum;
}
enum TierMode { kTierSliced = 0, kTierAtomic = 1, kTierFirstSeen = 2, kTierRankedSeen = 3, kTierBytes = 4 };
// First-seen order through rank blocks: four more launches per hop and a pass over the hop's edges for every kSeenSlice new nodes,
// but cheaper edges where the first-edge keys of all batches (4 N bytes each) are far from fitting the L2s.  Whole call, ranked
// against kTierFirstSeen, on graphs of 49-50 edges per node unless said otherwise:
//   one batch    slower on all of 0.1 M to 10 M nodes: 1.12 (4.3 M edges, N = 10 M) to 1.67 times
//   2 batches    N = 10 M 0.83-0.98 from 1.1 M edges each, N = 2.4 M 0.98-1.11, N = 1 M 1.12-1.22
//   3            N = 10 M 0.79-0.86, N = 2.4 M 0.81-0.90, N = 1 M 0.89-0.99, N = 233 k 1.02-1.22
//   4            N = 10 M 0.62-0.72, N = 2.4 M 0.73-0.84, N = 1 M 0.85-0.96, N = 233 k 0.93-1.10, N = 100 k 1.00-1.17
//   8            N = 300 k, 20 edges per node, 0.52-0.73 for N edges per batch, 0.88 for 13 N
// so by N and the square of the batches; 2.1 M edges in all are too few (1.08-1.12 at 4 batches of 64 and 3 neighbours).  The passes
// bound it above: 2 batches, N = 10 M, 8 M edges each 0.80-0.82, 16 M 0.85-1.12; N = 40 M 0.87 and 0.94-1.10.
constexpr int64_t kRankedSeenMin = 2200 * 1000;
inline bool rg_use_ranked_seen(int slices, int64_t num_nodes, int64_t edges, int group) {
    return rg_use_slices(slices, num_nodes, edges, group, false) && group >= 2 && num_nodes * group * group >= 9000 * 1000 &&
           edges * group >= kRankedSeenMin && edges <= 2 * group * num_nodes;
}
constexpr int64_t kRankedSeenEdges = 8ll << 20;      // per hop and batch at most
constexpr int kSliceWords = 40000;   // bitmap words of a slice: 160,000 of the 163,840 bytes of LDS a compute unit has
constexpr int kMaxSlices = 32;
constexpr int kSliceGroups = 256;    // workgroups the marking pass is split into at most (slices x splits x batches): one per
                                     // compute unit, which is what a full slice's LDS admits
constexpr int kSplitEdges = 8192;    // edges per split at least, and two per bitmap word (a split writes its slice out once)
constexpr int kTierWords = 768;      // bitmap words per workgroup in the tier kernels of kTierSliced
constexpr int kTierWordsSmall = 192; // the same where few workgroups come of that, which then are larger than their words: the rows
constexpr int kEmitThreadsSmall = 384;       // of up to 6144 new ids wait to be read (192 threads 119 us a call, 384 116; 768 are up to 12 % slower in groups)
constexpr unsigned kTierSelfScan = 4096;     // workgroups up to which k_tier_emit adds up the counts in front of its own itself
// kTierBytes saves launches (two hops 6 instead of 10, or 8 where the tiers are counted by launches of their own), which are what bounds calls
// of few edges, on the host as on the device; its stores cost 9 ps each, more where the bytes of all batches, which every hop clears and reads,
// outgrow an XCD's L2 (two maps of 2 MB).  So the line is by the product of the batches' edges and nodes, and lower from 2 M nodes in all on, below
// the calls that lose; whole call, bytes against slices:
//   below it   one batch of 356 k edges on 186 k nodes 59 / 77 us, 459 k on 40 k 58 / 83, 299 k on 254 k 61 / 78, 1.4 M on 673 k 88 / 110, 30 k on
//              865 k 43 / 55, 80 k on 2 M 48 / 61; two of 527 k on 236 k 73 / 88, of 486 k on 972 k 86 / 96; four of 285 k on 59 k 66 / 85;
//              eight of 61 k on 209 k 50 / 56, of 246 k on 119 k 81 / 90, of 25 k on 583 k 48 / 55
//   above it   two of 670 k on 1.8 M 87 / 82, one of 3.1 M on 2.8 M 165 / 148, two of 1 M on 3.1 M 150 / 133, four of 419 k on 1.6 M 103 / 89, eight of
//              178 k on 2.2 M 103 / 89, two of 1 M on 1.1 M 121 / 126
//   from 2 M nodes in all on, between 1.1e12 and 4e12, either: one of 390 k on 4.1 M 62 / 74, of 397 k on 2.8 M 82 / 100, of 344 k on 3.8 M 85 / 101, two of
//              127 k on 3.3 M 60 / 68, four of 118 k on 1.0 M 62 / 72, eight of 78 k on 263 k 53 / 59; two of 623 k on 1.4 M 103 / 100, and where few edges
//              would take the atomic way (rg_use_slices) four of 25 k on 2.7 M 55 / 49, of 21 k on 3.8 M 80 / 68, three of 58 k on 4.0 M 81 / 77
// An atomic on a bitmap in place of the byte makes words that many edges name queue up (dense-social batch 95 / 57); above 4 Mi nodes, where few
// edges take it, it reads an eighth (one batch on 5-11 M nodes 46-52 us, with bytes 52-61).
constexpr double kBytesEdgesNodes[2] = {4e12, 1.1e12};
constexpr int64_t kBytesFit = 2 * 1000 * 1000;
constexpr int64_t kBytesNodes = 4 << 20;
// A byte map for all batches fits where slices' bitmaps do (sliced_bytes: up to kSliceWords words in all there is room for 32 maps, above for
// kSliceGroups * kSliceWords words); the second one that kBytesSelfWords takes, below.
inline bool rg_use_bytes(int64_t num_nodes, int64_t words, int64_t edges, int group) {
    return num_nodes <= kBytesNodes &&
           (double)edges * group * ((double)num_nodes * group) <= kBytesEdgesNodes[num_nodes * group >= kBytesFit] &&
           group * words * 32 <= (int64_t)kSliceGroups * kSliceWords * 4;
}
// Bitmap words up to which a tier workgroup counts the bytes in front of its own itself, and the bytes all of them read for that: one batch on
// 133 k nodes 37.4 us a call, 38.3 with a launch that counts, 177 k 60.1 / 58.7, 254 k 63.5 / 60.7, 486 k 75 / 62; eight on 119 k 82 / 86; four on
// 59 k 66 / 71.
constexpr int64_t kBytesSelfWords = 5000, kBytesSelfRead = 12 * 1000 * 1000;
static_assert(2 * 32 * RG_MAX_GROUP * kBytesSelfWords <= (int64_t)kSliceGroups * kSliceWords * 4 && 2 * 32 <= kSliceGroups * 4,
              "two byte maps of so many words fit");
constexpr int kRankIds = 48;         // ids to a rank block, two to three bitmap words (see rg_rank_blocks)
constexpr int kBaseIds = kRankIds * 1024;      // ids to a base: the members among them are counted in 16 bits
static_assert(kBaseIds % (32 * kTierWords) == 0 && kBaseIds % (32 * kTierWordsSmall) == 0 && kTierWords % 3 == 0 && kTierWordsSmall % 3 == 0,
              "whole rank blocks and bases");
constexpr int kRankHops = 4;         // hops whose rank blocks share a buffer
static_assert(RG_MAX_HOPS <= 2 * kRankHops && kRankHops == 4, "rank blocks of all hops");

template <typename RP>
__device__ __forceinline__ void rg_row_extent(const RP* __restrict__ row_ptr, int v, int64_t& start, int64_t& deg) {
    const RP a = row_ptr[v];
    const RP b = row_ptr[v + 1];
    start = (int64_t)a;
    deg = (int64_t)(b - a);
}

struct RowPtr {                      // a row_ptr array of either width
    const void* p;
    int wide;
};
__device__ __forceinline__ void rg_row_extent(const RowPtr& row_ptr, int v, int64_t& start, int64_t& deg) {
    if (row_ptr.wide) rg_row_extent((const int64_t*)row_ptr.p, v, start, deg);
    else rg_row_extent((const int32_t*)row_ptr.p, v, start, deg);
}

// ---------------------------------------------------------------------------- schedule
// The keys are Philox words, spread evenly whatever the ids, so their top bits are a perfect first radix digit: the pairs (32 more
// bits of the key, id) go to one of 2^log2_buckets buckets, each of which has room for kSchedRoom of them where half of kSchedAvg to
// all of it come, and every bucket is finished by one workgroup in LDS (a second digit of kSubBits bits leaves about one pair per sub-bucket;
// pairs alike in the bits at hand have their keys worked out again).  Ids that find their bucket full, which only ids picked for
// their keys do, wait in a list.  Nothing is counted beforehand: the keys are worked out once, and a call is two launches.
// Bound by launches, the Philox blocks (3.3 us for 1 M ids on the whole device) and the scattered 8-byte writes.
// Few ids get small buckets, whose sort is a shorter chain of LDS passes (100 k ids 9.5 us, in buckets of 2048 12.0; 10 k 7.2 / 9.3; 400 k 14.8 / 15.9),
// many get large ones, to whose counters the workgroups add less often (700 k 24.7 / 19.3).  Up to 4096 ids one workgroup does it all (1000 5.0 us, in
// buckets 7.1; 3072 7.5 either way), of 1024 threads (4096 ids 9.4 us, with 512 threads 12.4; in buckets 8.4, but so a call needs no scratch, which
// a graph that records a context's first call cannot allocate), with room for 3072 where that does (1000 ids 5.1 us, with room for 4096 5.6).
constexpr int kSchedLds[2] = {3072, 4096};         // pairs one workgroup sorts in LDS
constexpr int kSchedAvg[2] = {512, 2048};          // pairs per bucket on average, at most
constexpr int kSchedRoom = 2560;                   // eleven standard deviations more than the large ones' average; in small ones for ids picked for their
                                                   // keys (20 k ids, 1500 in one bucket: 10.0 us, with room for 1024 36)
constexpr int64_t kSchedFew = 400 * 1000;          // ids that get the small ones
constexpr int64_t kSchedFewBuckets = 1024;         // of the most of these
static_assert(kSchedFew <= kSchedFewBuckets * kSchedAvg[0], "buckets for them");
constexpr int kSchedLdsBuckets = 4096;   // buckets whose counters a workgroup keeps in LDS; with more (n > 8 Mi) every id
                                         // adds to the counter in HBM, and the counters are scanned by a launch of their own

__device__ __forceinline__ uint64_t rg_sched_key(int32_t v, uint32_t epoch, uint32_t k0, uint32_t k1) {
    uint32_t w[4];
    rg_philox4x32_10((uint32_t)v, 0xFFFFFFFFu, 0u, epoch, k0, k1, w);
    return ((uint64_t)w[0] << 32) | (uint64_t)w[1];
}

__global__ void __launch_bounds__(256) k_sched_clear(int32_t* __restrict__ p, int64_t n) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) p[i] = 0;
}

// start[b] = pairs in the buckets in front of b, start[buckets] = n.  One workgroup.
__global__ void __launch_bounds__(1024) k_sched_scan(const int32_t* __restrict__ count, int buckets, int32_t* __restrict__ start) {
    __shared__ int smem[1024 / RG_WAVE + 1];
    int carry = 0;
    for (int base = 0; base < buckets; base += 1024) {
        const int b = base + threadIdx.x;
        const int x = b < buckets ? count[b] : 0;
        int total;
        const int excl = rg_block_excl_scan<1024 / RG_WAVE>(x, smem, &total);
        if (b < buckets) start[b] = carry + excl;
        carry += total;
    }
    if (threadIdx.x == 0) start[buckets] = carry;
}

// Pairs go to their bucket; the order inside is left to k_sched_sort.  count[b] = pairs of bucket b, those without room among them;
// count[buckets] = ids in the list `late`.  PER ids per thread.
template <bool LDS, int PER>
__global__ void __launch_bounds__(1024) k_sched_scatter(const int32_t* __restrict__ train_ids, int64_t n, int log2_buckets, uint32_t k0,
                                                        uint32_t k1, uint32_t epoch, int32_t* __restrict__ count,
                                                        uint2* __restrict__ pairs, int32_t* __restrict__ late) {
    __shared__ int32_t h[LDS ? kSchedLdsBuckets : 1];
    const int buckets = 1 << log2_buckets;
    const int64_t i0 = (int64_t)blockIdx.x * (1024 * PER);
    int32_t v[PER];
    uint64_t key[PER];
#pragma unroll
    for (int j = 0; j < PER; ++j) {
        const int64_t i = i0 + j * 1024 + threadIdx.x;
        v[j] = i < n ? train_ids[i] : 0;
    }
    if (LDS) {
        for (int b = threadIdx.x; b < buckets; b += 1024) h[b] = 0;
        __syncthreads();
    }
#pragma unroll
    for (int j = 0; j < PER; ++j) key[j] = rg_sched_key(v[j], epoch, k0, k1);
    int32_t rank[PER];
#pragma unroll
    for (int j = 0; j < PER; ++j)
        if (i0 + j * 1024 + threadIdx.x < n) rank[j] = atomicAdd(&(LDS ? h : count)[key[j] >> (64 - log2_buckets)], 1);
    if (LDS) {
        __syncthreads();
        for (int b = threadIdx.x; b < buckets; b += 1024)                // a place for this workgroup's pairs of the bucket
            if (h[b]) h[b] = atomicAdd(&count[b], h[b]);
        __syncthreads();
    }
#pragma unroll
    for (int j = 0; j < PER; ++j) {
        if (i0 + j * 1024 + threadIdx.x >= n) continue;
        const int64_t b = (int64_t)(key[j] >> (64 - log2_buckets));
        const int32_t at = (LDS ? h[b] : 0) + rank[j];
        if (at < kSchedRoom) pairs[b * kSchedRoom + at] = make_uint2((uint32_t)(key[j] >> (32 - log2_buckets)), (uint32_t)v[j]);
        else late[atomicAdd(&count[buckets], 1)] = v[j];
    }
}

// The m ids of a bucket (SINGLE: of the call) to their places, in PER rounds of T.
template <int PER, bool SINGLE, int T, int SUB_BITS>
__device__ __forceinline__ void rg_sched_finish(const int32_t* __restrict__ train_ids, const uint2* __restrict__ pairs, int64_t m, uint32_t epoch, uint32_t k0,
                                                uint32_t k1, uint32_t* sk, int32_t* si, int32_t* sub, int* smem, int32_t* out) {
    constexpr int SUB = 1 << SUB_BITS;
    const auto full_key = [&](int32_t v) { return rg_sched_key(v, epoch, k0, k1); };
    uint32_t key[PER];
    int32_t id[PER], rank[PER];
    for (int b = threadIdx.x; b <= SUB; b += T) sub[b] = 0;
#pragma unroll
    for (int j = 0; j < PER; ++j) {
        const int i = j * T + threadIdx.x;
        if (i < m) {
            if (SINGLE) {
                id[j] = train_ids[i];
                key[j] = (uint32_t)(full_key(id[j]) >> 32);
            } else {
                const uint2 x = pairs[i];
                key[j] = x.x;
                id[j] = (int32_t)x.y;
            }
        }
    }
    __syncthreads();
#pragma unroll
    for (int j = 0; j < PER; ++j)
        if (j * T + (int)threadIdx.x < m) rank[j] = atomicAdd(&sub[key[j] >> (32 - SUB_BITS)], 1);
    __syncthreads();
    int mine[SUB / T], sum = 0;                                          // counts -> starts, SUB / T consecutive ones per thread
#pragma unroll
    for (int q = 0; q < SUB / T; ++q) { mine[q] = sub[threadIdx.x * (SUB / T) + q]; sum += mine[q]; }
    int total;
    int at = rg_block_excl_scan<T / RG_WAVE>(sum, smem, &total);         // its barriers separate the reads from the writes
#pragma unroll
    for (int q = 0; q < SUB / T; ++q) { sub[threadIdx.x * (SUB / T) + q] = at; at += mine[q]; }
    if (threadIdx.x == T - 1) sub[SUB] = at;
    __syncthreads();
#pragma unroll
    for (int j = 0; j < PER; ++j)
        if (j * T + (int)threadIdx.x < m) {
            const int p = sub[key[j] >> (32 - SUB_BITS)] + rank[j];
            sk[p] = key[j];
            si[p] = id[j];
        }
    __syncthreads();
#pragma unroll
    for (int j = 0; j < PER; ++j)
        if (j * T + (int)threadIdx.x < m) {
            const int b = (int)(key[j] >> (32 - SUB_BITS));
            const int lo = sub[b], hi = sub[b + 1], me = lo + rank[j];
            int place = lo;
            for (int q = lo; q < hi; ++q) {
                if (sk[q] != key[j]) {
                    place += sk[q] < key[j];
                } else if (q != me) {
                    if (si[q] == id[j]) {                                // (equal pairs, which distinct ids do not give, keep their places)
                        place += q < me;
                    } else {
                        const uint64_t mine_ = full_key(id[j]), other = full_key(si[q]);
                        place += other != mine_ ? other < mine_ : si[q] < id[j];
                    }
                }
            }
            out[place] = id[j];
        }
}

// One workgroup per bucket: its pairs in order, the ids to their final places.  CAP: pairs it has room for in LDS; up to FEW of them take fewer
// rounds (100 k ids 10.0 us, with those for 2560 10.1 to 10.5).
// SINGLE: one bucket, the n train ids themselves.  start == NULL: the workgroup adds up the counts in front of its own.
// `clear` (or NULL): n_clear counters that the next call will use.
template <int CAP, bool SINGLE, int T, int FEW = CAP>
__global__ void __launch_bounds__(T) k_sched_sort(const int32_t* __restrict__ train_ids, int64_t n, int log2_buckets, uint32_t k0,
                                                    uint32_t k1, uint32_t epoch, const int32_t* __restrict__ count,
                                                    const int32_t* __restrict__ start, const uint2* __restrict__ pairs,
                                                    const int32_t* __restrict__ late, int32_t* order_out,
                                                    int32_t* __restrict__ clear, int n_clear) {
    constexpr int kTile = SINGLE ? 0 : 2048;            // of an overfull bucket
    constexpr int kSubBits = FEW > 1024 ? 11 : 10, SUB = 1 << kSubBits;
    static_assert(CAP % T == 0 && FEW % T == 0 && SUB % T == 0, "whole rounds");
    __shared__ uint32_t sk[CAP > kTile ? CAP : kTile];
    __shared__ int32_t si[CAP > kTile ? CAP : kTile];
    __shared__ int32_t sub[SUB + 1];
    __shared__ int smem[T / RG_WAVE + 1];
    const int64_t bucket = blockIdx.x;
    if (clear) for (int64_t i = bucket * T + threadIdx.x; i < n_clear; i += (int64_t)gridDim.x * T) clear[i] = 0;
    int64_t s0 = 0, m = n;
    if (!SINGLE) {
        m = count[bucket];
        if (start) {
            s0 = start[bucket];
        } else {
            int before = 0, total;
            for (int b = threadIdx.x; b < (int)bucket; b += T) before += count[b];
            (void)rg_block_excl_scan<T / RG_WAVE>(before, smem, &total);
            s0 = total;
        }
    }
    if (m == 0) return;                                                  // uniform
    int32_t* out = order_out + s0;
    const auto full_key = [&](int32_t v) { return rg_sched_key(v, epoch, k0, k1); };
    if (!SINGLE && m > CAP) {
        // Only ids picked for their keys get here: the bucket's and those of the list that belong to it, sorted where they will be,
        // by a network whose every comparison is ascending, so that the places behind its end count as larger than everything and are
        // never touched.  Steps within kTile ids are made in LDS, tile by tile; of the others there are few, which work the keys out
        // from the ids.  A call of 100,000 ids of which 4000 belong to one bucket 89 us, 6000 of them 150, 12,000 334 (10 where every bucket
        // has room), one of 1 M ids with 4000 in a bucket 103 (24).
        int32_t* fill = sub;
        if (threadIdx.x == 0) *fill = CAP;
        for (int i = threadIdx.x; i < CAP; i += T) out[i] = (int32_t)pairs[bucket * CAP + i].y;
        __syncthreads();
        const int n_late = count[1ll << log2_buckets];
        for (int i = threadIdx.x; i < n_late; i += T) {
            const int32_t v = late[i];
            if ((int64_t)(full_key(v) >> (64 - log2_buckets)) == bucket) out[atomicAdd(fill, 1)] = v;
        }
        for (int64_t width = kTile; width < 2 * m; width <<= 1) {       // runs of `width` ids from the halves of each; the first ones from single ids
            for (int64_t d = width - 1; d >= kTile; d = d == width - 1 ? width >> 2 : d >> 1) {
                __syncthreads();
                for (int64_t i = threadIdx.x; i < m; i += T) {
                    const int64_t l = i ^ d;
                    if (l <= i || l >= m) continue;
                    const int32_t a = out[i], b = out[l];
                    const uint64_t ka = full_key(a), kb = full_key(b);
                    if (kb < ka || (kb == ka && b < a)) { out[i] = b; out[l] = a; }
                }
            }
            const bool first = width == kTile;
            for (int64_t t0 = 0; t0 < m; t0 += kTile) {
                const int here = (int)(m - t0 < kTile ? m - t0 : kTile);
                __syncthreads();
                for (int i = threadIdx.x; i < here; i += T) {
                    si[i] = out[t0 + i];
                    sk[i] = (uint32_t)(full_key(si[i]) >> (32 - log2_buckets));
                }
                for (int w = first ? 2 : 2 * kTile; w <= (first ? kTile : 2 * kTile); w <<= 1)
                    for (int d = first ? w - 1 : kTile / 2; d > 0; d = d == w - 1 ? w >> 2 : d >> 1) {
                        constexpr int P = kTile / 2 / T + SINGLE;                 // pairs per thread
                        const int top = d == w - 1 ? w >> 1 : d;         // the bit of i that l has and i has not
                        uint32_t ka[P], kb[P];
                        int32_t a[P], b[P];
                        __syncthreads();
#pragma unroll
                        for (int q = 0; q < P; ++q) {
                            const int x = q * T + (int)threadIdx.x, i = x + (x & -top), l = i ^ d;
                            ka[q] = kb[q] = 0u;
                            a[q] = b[q] = 0;
                            if (l < here) { ka[q] = sk[i]; kb[q] = sk[l]; a[q] = si[i]; b[q] = si[l]; }
                        }
#pragma unroll
                        for (int q = 0; q < P; ++q) {
                            const int x = q * T + (int)threadIdx.x, i = x + (x & -top), l = i ^ d;
                            bool swap = kb[q] < ka[q];
                            if (ka[q] == kb[q] && a[q] != b[q]) {
                                const uint64_t fa = full_key(a[q]), fb = full_key(b[q]);
                                swap = fb < fa || (fb == fa && b[q] < a[q]);
                            }
                            if (swap) { sk[i] = kb[q]; sk[l] = ka[q]; si[i] = b[q]; si[l] = a[q]; }
                        }
                    }
                __syncthreads();
                for (int i = threadIdx.x; i < here; i += T) out[t0 + i] = si[i];
            }
        }
        return;
    }
    if (FEW < CAP && m <= FEW) rg_sched_finish<FEW / T, SINGLE, T, kSubBits>(train_ids, pairs + bucket * CAP, m, epoch, k0, k1, sk, si, sub, smem, out);
    else rg_sched_finish<CAP / T, SINGLE, T, kSubBits>(train_ids, pairs + bucket * CAP, m, epoch, k0, k1, sk, si, sub, smem, out);
}

// ---------------------------------------------------------------------------- batches of a group
// Several batches are sampled by the same launches: every workgroup belongs to one (rg_batch), which brings its own outputs
// (BatchTable) and its own slice of the scratch (SampleScratch).  Most kernels of one batch are
// far smaller than the device (hop 0 of a 4096-seed batch is 16 workgroups), so a group fills it better and pays
// every launch once.
constexpr int kMaxGroup = RG_MAX_GROUP;
constexpr unsigned kXcds = 8;
// Frontier nodes in a row to an XCD at most, for the kernels that draw and count, and no more than a 64th of a batch's, or the XCDs would be
// unequal (fewer than 64 workgroups are not shared; the emit's go one by one): batches' tiers are not cut alike, so
// short runs miss each other (hop 2 of 8 batches, 256 nodes 700 us a call, 1024 to 8192 679, 16,384 689, not shared 717).
constexpr int kSharedNodes = 4096;

// The batches' buffers: a table of 8-byte entries, [field][batch].  It goes to the first kernel as an argument, which leaves a copy in the
// scratch for the others: arguments are read over the host link, and every kilobyte of them costs a launch 1.4 us of
// the host's time and 0.7 of the device's.
enum BatchField { kSeeds, kNumSeeds, kNodes, kTierOff, kEdgesOut, kHopFields };      // then kIndptr, kNbr, kNbrLocal of every hop
enum HopField { kIndptr, kNbr, kNbrLocal, kHopFieldCount };
constexpr int kTableFew = 32, kTableSome = 128, kTableMost = 480;       // sizes of the argument: one batch of three hops takes 14 entries
static_assert(kMaxGroup * (kHopFields + kHopFieldCount * RG_MAX_HOPS) <= kTableMost, "a table of the largest group");
template <int N>
struct BatchTable {
    uint64_t v[N];
};

struct SampleScratch {
    const uint64_t* table;
    uint32_t* visited;                // [group][words]
    uint32_t* marked;                 // kTierAtomic: [group][words], every id met
    uint32_t* slice_marks;            // kTierSliced: [group][splits][words], ids of a hop; kTierBytes: rg_bytes
    uint4* rank[2];                   // kTierSliced: rank blocks and bases of four hops each (rg_rank_blocks)
    int32_t* pos;                     // [group][num_nodes] (kTierSliced: of the seeds only)
    int32_t* chunk_sum;               // [group][chunk_stride]: new ids per workgroup of the tier kernels
    int32_t* hop_sum[2];              // the same: edges of the even and the odd hops per kChunk frontier nodes
    int64_t* row_start;               // [group][frontier_stride]
    int32_t* row_deg;                 // [group][frontier_stride]
    int32_t* first_edge;              // kTierRankedSeen: [group][frontier_stride], by ascending position (k_seen_min)
    int32_t* place;                   // the same: ascending position -> position
    int32_t* first_key;               // [group][num_nodes], kTierFirstSeen only: 0x7FFFFFFF - (index of the first edge of
                                      // the current hop that names the node), 0 = not named (kept all-zero between hops)
    int64_t words, rank_blocks, rank_bases, num_nodes, chunk_stride, frontier_stride;
    int hops;
    int slices, splits;               // of the marking pass: id ranges of slice_words bitmap words, parts of the edge list
    int slice_words;
    int group;                        // batches in this call
    int table_entries;
    int xcd_map;                      // 1: consecutive workgroups belong to consecutive batches (see rg_batch)
    uint32_t group_inv;               // 2^32 / group, rounded up; 0 for a group of one (rg_over_group)
};

// Entries of the table: read through the constant address space, so that a pointer is uniform, and used as an address of global memory
// (a flat access is slower: 53 us against 44 in k_slice_mark).
__device__ __forceinline__ int32_t* rg_global(uint64_t address) { return (int32_t*)(__attribute__((address_space(1))) int32_t*)address; }
__device__ __forceinline__ uint64_t rg_entry(const SampleScratch& S, int field, int g) {
    return ((const __attribute__((address_space(4))) uint64_t*)(uintptr_t)S.table)[field * S.group + g];
}
__device__ __forceinline__ int32_t* rg_nodes(const SampleScratch& S, int g) { return rg_global(rg_entry(S, kNodes, g)); }
__device__ __forceinline__ int32_t* rg_tier_off(const SampleScratch& S, int g) { return rg_global(rg_entry(S, kTierOff, g)); }
__device__ __forceinline__ int32_t* rg_hop_list(const SampleScratch& S, int g, int hop, HopField f) {
    return rg_global(rg_entry(S, kHopFields + kHopFieldCount * hop + f, g));
}
// kTierBytes: a byte per id, 1 for those the hop has sampled.
__device__ __forceinline__ uint8_t* rg_bytes(const SampleScratch& S, int g) { return (uint8_t*)S.slice_marks + g * S.words * 32; }
__device__ __forceinline__ void rg_put_edges(const SampleScratch& S, int g, int hop, int edges) {
    int32_t* out = rg_global(rg_entry(S, kEdgesOut, g));               // may be NULL
    if (out) out[hop] = edges;
}
template <int N>
__device__ __forceinline__ void rg_copy_table(const SampleScratch& S, const BatchTable<N>& B) {
    for (int i = threadIdx.x; i < S.table_entries; i += blockDim.x) ((uint64_t*)S.table)[i] = B.v[i];
}

// Workgroup -> (batch, block within the batch) for the per-batch kernels, launched as one 1-D grid of blocks x group
// workgroups.  The device hands consecutive workgroup ids to its 8 XCDs in turn, and every XCD has an L2 of its own.
// With xcd_map, workgroup id w works on batch w % group: with a group of 8 all workgroups of one batch run on one XCD,
// whose L2 then holds that batch's membership bitmaps (2 x N/8 bytes, probed at random by every sampled edge) instead
// of every XCD holding a share of all eight.
// Every kernel begins with these, and most are short: a division takes 25 instructions, which every compute unit fetches anew for each
// launch (a batch of 1024 seeds, (25,10), in eight launches 45.5 us with divisions, 45.0 without; 48 calls of 10 k to 4 M nodes 1.5 % less).
__device__ __forceinline__ unsigned rg_over_group(const SampleScratch& S, unsigned x) {        // x / group, x < 2^28
    return S.group_inv ? __umulhi(x, S.group_inv) : x;
}
__device__ __forceinline__ unsigned rg_blocks_per_batch(const SampleScratch& S) { return rg_over_group(S, gridDim.x); }
__device__ __forceinline__ int rg_batch(const SampleScratch& S) {
    if (S.xcd_map) return (int)(blockIdx.x - rg_over_group(S, blockIdx.x) * (unsigned)S.group);
    int g = 0;
    for (unsigned x = blockIdx.x, per = rg_blocks_per_batch(S); x >= per; x -= per) ++g;
    return g;
}
__device__ __forceinline__ unsigned rg_block(const SampleScratch& S) {
    return S.xcd_map ? rg_over_group(S, blockIdx.x) : blockIdx.x - (unsigned)rg_batch(S) * rg_blocks_per_batch(S);
}
// The same for the kernels that read the graph at the ids of an ascending frontier: workgroups 8 apart, on one XCD, take 2^(run - 1)
// consecutive blocks of every batch in turn.
__device__ __forceinline__ void rg_shared_rows(const SampleScratch& S, int run, int& g, unsigned& blk) {
    if (run == 0) { g = rg_batch(S); blk = rg_block(S); return; }
    const unsigned seq = blockIdx.x / kXcds, turn = rg_over_group(S, seq), r = (unsigned)run - 1u;
    g = (int)(seq - turn * (unsigned)S.group);
    blk = (((turn >> r) * kXcds + blockIdx.x % kXcds) << r) + (turn & ((1u << r) - 1u));
}
// Rank blocks: which of kRankIds ids are in a tier (the low 48 bits), and the position of the first of them as what it is above
// the base of its kBaseIds ids (the upper 16).  The blocks of the last hop's tier and of the one before it lie side by side, and so
// on backwards, so that one 16-byte read asks two tiers; an odd first tier has its blocks to itself.
// A random read costs the same for 4 to 16 bytes (258 G/s from L2 on the whole device, 197 from a table of 5 MB per XCD), so what
// counts is the number of reads, and that the tables of a batch fit its XCD's 4 MB: N / 3 bytes per pair.
// [pair][group][rank_blocks], kRankHops / 2 pairs to a buffer, then the bases, [hop][group][rank_bases].
struct RankBlocks {
    uint2* at;
    int stride;
};
__device__ __forceinline__ uint4* rg_rank_pair(const SampleScratch& S, int g, int pair) {
    return S.rank[pair >> 1] + ((pair & 1) * S.group + g) * S.rank_blocks;
}
__device__ __forceinline__ RankBlocks rg_rank_blocks(const SampleScratch& S, int g, int hop) {
    const int d = S.hops - 1 - hop;
    uint2* p = (uint2*)rg_rank_pair(S, g, d >> 1);
    return hop == 0 && (d & 1) == 0 ? RankBlocks{p, 1} : RankBlocks{p + (d & 1), 2};
}
__device__ __forceinline__ int32_t* rg_rank_bases(const SampleScratch& S, int g, int hop) {
    const int d = S.hops - 1 - hop;
    return (int32_t*)(S.rank[d >> 2] + 2 * S.group * S.rank_blocks) + ((d & 3) * S.group + g) * S.rank_bases;
}
// Bytes of one buffer for batches of `members` bitmap words in all.
inline int64_t rg_rank_bytes(int64_t members) {
    const int64_t blocks = 2 * (members / 3 + kMaxGroup), bases = members / (kBaseIds / 32) + kMaxGroup;
    return kRankHops * (blocks * (int64_t)sizeof(uint2) + bases * 4);
}

// ---------------------------------------------------------------------------- batch start
__global__ void __launch_bounds__(256) k_clear_words(uint32_t* __restrict__ w, int64_t n) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) w[i] = 0u;
}

template <int N>
__device__ __forceinline__ void rg_mark_seeds(const BatchTable<N>& B, const SampleScratch& S) {
    const int g = rg_batch(S);
    const unsigned blk = rg_block(S);
    if (blockIdx.x == 0) rg_copy_table(S, B);
    const int num_seeds = (int)B.v[kNumSeeds * S.group + g];
    const int i = blk * blockDim.x + threadIdx.x;
    int32_t* __restrict__ tier_off = rg_global(B.v[kTierOff * S.group + g]);
    if (i == 0) { tier_off[0] = 0; tier_off[1] = num_seeds; }
    if (i >= num_seeds) return;
    const int32_t v = rg_global(B.v[kSeeds * S.group + g])[i];
    rg_global(B.v[kNodes * S.group + g])[i] = v;
    S.pos[g * S.num_nodes + v] = i;
    atomicOr(&S.visited[g * S.words + ((uint32_t)v >> 5)], 1u << (v & 31));
    atomicOr(&S.marked[g * S.words + ((uint32_t)v >> 5)], 1u << (v & 31));
}

__global__ void __launch_bounds__(256) k_mark_seeds(const BatchTable<kTableSome> B, const SampleScratch S) { rg_mark_seeds(B, S); }
__global__ void __launch_bounds__(256) k_mark_seeds_most(const BatchTable<kTableMost> B, const SampleScratch S) { rg_mark_seeds(B, S); }

// The same in one launch for graphs of up to kMaxSlices slices: a workgroup owns one slice of a batch's ids, collects the
// seeds of its range in LDS and writes its part of `visited`.
// `marked` starts as `visited` (kTierAtomic), the bytes as zeros (kTierBytes).
// Every slice's workgroup reads all seeds, 1024 at a time: for more than 8192 of them clearing and marking take less in launches
// of their own, unless several batches make many workgroups of them.  One hop after it, one launch against two or three: one
// batch of 4096 seeds, N = 1 M 38 / 39 us, of 8192 43 / 39, of 16 k 52 / 41, of 65 k 126 / 64, of 200 k 305 / 117, at N = 10 M 38 / 43,
// 45 / 45, 57 / 53, 97 / 76, 192 / 130; 8 batches of 16 k, N = 1 M 104 / 97, N = 4 M 106 / 111, N = 10 M 127 / 134.
inline bool rg_use_init(int slices, int group, int64_t seeds) {
    return slices > 0 && (seeds <= 8192 || (group >= 4 && slices * group >= 32));
}
// The workgroups behind the slices do for the seeds what k_hop_count does.
template <int N>
__device__ __forceinline__ void rg_sample_init(const RowPtr& row_ptr, const BatchTable<N>& B, const SampleScratch& S, int fanout, int mode) {
    extern __shared__ uint32_t slice_bits[];
    const int g = rg_batch(S);
    const unsigned slice = rg_block(S);
    if (blockIdx.x == 0) rg_copy_table(S, B);
    const int num_seeds = (int)B.v[kNumSeeds * S.group + g];
    const int32_t* __restrict__ seeds = rg_global(B.v[kSeeds * S.group + g]);
    if (mode == kTierBytes) {                            // (words * 32 of them: whole 16-byte chunks)
        uint4* __restrict__ bytes = (uint4*)rg_bytes(S, g);
        for (int64_t i = (int64_t)slice * 1024 + threadIdx.x; i < S.words * 2; i += (int64_t)rg_blocks_per_batch(S) * 1024) bytes[i] = make_uint4(0u, 0u, 0u, 0u);
    }
    if (slice >= (unsigned)S.slices) {
        const unsigned chunk = slice - (unsigned)S.slices;
        const int i = (int)(chunk * kChunk + threadIdx.x);
        int m = 0;
        if (i < num_seeds) {
            int64_t start, deg;
            rg_row_extent(row_ptr, seeds[i], start, deg);
            S.row_start[g * S.frontier_stride + i] = start;
            S.row_deg[g * S.frontier_stride + i] = (int32_t)deg;
            m = deg <= fanout ? (int)deg : fanout;
        }
        m = rg_wave_sum(m);
        if (rg_lane() == 0) slice_bits[threadIdx.x >> 6] = (uint32_t)m;
        __syncthreads();
        if (threadIdx.x < RG_WAVE) {
            m = rg_wave_sum(threadIdx.x < 1024 / RG_WAVE ? (int)slice_bits[threadIdx.x] : 0);
            if (threadIdx.x == 0) S.hop_sum[0][g * S.chunk_stride + chunk] = m;
        }
        return;
    }
    const int64_t w0 = (int64_t)slice * S.slice_words;
    const int n_words = (int)(S.words - w0 < S.slice_words ? S.words - w0 : S.slice_words);
    for (int w = threadIdx.x; w < n_words; w += 1024) slice_bits[w] = 0u;
    int32_t* __restrict__ tier_off = rg_global(B.v[kTierOff * S.group + g]);
    int32_t* __restrict__ nodes = rg_global(B.v[kNodes * S.group + g]);
    if (slice == 0 && threadIdx.x == 0) { tier_off[0] = 0; tier_off[1] = num_seeds; }
    __syncthreads();
    const uint32_t id0 = (uint32_t)(w0 << 5), n_ids = (uint32_t)n_words << 5;
    for (int i = threadIdx.x; i < num_seeds; i += 1024) {
        const int32_t v = seeds[i];
        const uint32_t d = (uint32_t)v - id0;
        if (d >= n_ids) continue;
        nodes[i] = v;
        S.pos[g * S.num_nodes + v] = i;
        atomicOr(&slice_bits[d >> 5], 1u << (d & 31u));
    }
    __syncthreads();
    uint32_t* __restrict__ visited = S.visited + g * S.words + w0;
    uint32_t* __restrict__ marked = S.marked + g * S.words + w0;
    for (int w = threadIdx.x; w < n_words; w += 1024) {
        visited[w] = slice_bits[w];
        if (mode == kTierAtomic) marked[w] = slice_bits[w];
    }
}

__global__ void __launch_bounds__(1024) k_sample_init(const RowPtr row_ptr, const BatchTable<kTableSome> B, const SampleScratch S, int fanout, int mode) {
    rg_sample_init(row_ptr, B, S, fanout, mode);
}
__global__ void __launch_bounds__(1024) k_sample_init_most(const RowPtr row_ptr, const BatchTable<kTableMost> B, const SampleScratch S, int fanout, int mode) {
    rg_sample_init(row_ptr, B, S, fanout, mode);
}

// ---------------------------------------------------------------------------- per hop: sizes
// hop_sum[b] = edges of the kChunk nodes from b * kChunk on; row_start[i], row_deg[i] = the node's adjacency row; indptr[i] (where
// `offsets` asks for it) = exclusive prefix of m within the node's chunk.  Bound by the random row_ptr lines, so every thread has
// kCountNodes of them in flight.
constexpr int kCountNodes = 4;

template <typename RP>
__global__ void __launch_bounds__(kChunk / kCountNodes) k_hop_count(const RP* __restrict__ row_ptr, const SampleScratch S,
                                                                    int hop, int fanout, int run, int offsets) {
    constexpr int T = kChunk / kCountNodes, NW = T / RG_WAVE;
    __shared__ int smem[NW + 1];
    int g;
    unsigned blk;
    rg_shared_rows(S, run, g, blk);
    const int n_h = rg_tier_off(S, g)[hop + 1];
    const int64_t first = (int64_t)blk * kChunk;
    if (first >= n_h) return;                       // uniform per workgroup
    const int n_here = (int)(n_h - first < kChunk ? n_h - first : kChunk);
    const int32_t* __restrict__ nodes = rg_nodes(S, g) + first;
    int32_t* __restrict__ indptr = rg_hop_list(S, g, (int)hop, kIndptr) + first;
    int64_t* __restrict__ row_start = S.row_start + g * S.frontier_stride + first;
    int32_t* __restrict__ row_deg = S.row_deg + g * S.frontier_stride + first;
    int32_t v[kCountNodes];
    RP a[kCountNodes], b[kCountNodes];
    int m[kCountNodes], before[kCountNodes];
    const int wave = threadIdx.x >> 6, i0 = wave * RG_WAVE * kCountNodes + rg_lane();      // a wavefront takes consecutive nodes
#pragma unroll
    for (int q = 0; q < kCountNodes; ++q) v[q] = i0 + q * RG_WAVE < n_here ? nodes[i0 + q * RG_WAVE] : -1;
#pragma unroll
    for (int q = 0; q < kCountNodes; ++q) {
        a[q] = b[q] = 0;
        if (v[q] >= 0) { a[q] = row_ptr[v[q]]; b[q] = row_ptr[v[q] + 1]; }
    }
    int sum = 0;
#pragma unroll
    for (int q = 0; q < kCountNodes; ++q) {
        const int64_t deg = (int64_t)(b[q] - a[q]);
        m[q] = (fanout < 0 || deg <= fanout) ? (int)deg : fanout;
        const int incl = rg_wave_incl_scan(m[q]);
        before[q] = sum + incl - m[q];
        sum += __shfl(incl, RG_WAVE - 1, RG_WAVE);
        if (v[q] >= 0) {
            row_start[i0 + q * RG_WAVE] = (int64_t)a[q];   // kept for the draw kernel: one coalesced read there instead
            row_deg[i0 + q * RG_WAVE] = (int32_t)deg;      // of a second random lookup of row_ptr
        }
    }
    if (rg_lane() == 0) smem[wave] = sum;
    __syncthreads();
    int base = 0, total = 0;
#pragma unroll
    for (int w = 0; w < NW; ++w) {
        if (w < wave) base += smem[w];
        total += smem[w];
    }
#pragma unroll
    for (int q = 0; q < kCountNodes; ++q)
        if (offsets && v[q] >= 0) indptr[i0 + q * RG_WAVE] = base + before[q];
    if (threadIdx.x == 0) S.hop_sum[hop & 1][g * S.chunk_stride + blk] = total;
}

// In-place exclusive scan of data[0..n) by one workgroup; returns (to thread 0) the grand total.
__device__ __forceinline__ int rg_scan_in_place(int32_t* __restrict__ data, int64_t n) {
    __shared__ int smem[1024 / RG_WAVE + 1];
    __shared__ int carry_s;
    if (threadIdx.x == 0) carry_s = 0;
    __syncthreads();
    for (int64_t base = 0; base < n; base += 1024) {
        const int64_t i = base + threadIdx.x;
        const int x = i < n ? data[i] : 0;
        int total;
        const int excl = rg_block_excl_scan<1024 / RG_WAVE>(x, smem, &total);
        const int carry = carry_s;
        if (i < n) data[i] = carry + excl;
        __syncthreads();
        if (threadIdx.x == 0) carry_s = carry + total;
        __syncthreads();
    }
    return carry_s;
}

// Chunk totals of a hop -> exclusive offsets; the hop's edge total goes behind the last indptr entry.  In front of the
// wavefront-per-node draw, and of the thread-per-node draw on frontiers of over kDrawSelfScan chunks.
__global__ void __launch_bounds__(1024) k_scan_hop(const SampleScratch S, int hop) {
    const int g = rg_batch(S);
    const int n_h = rg_tier_off(S, g)[hop + 1];
    const int total = rg_scan_in_place(S.hop_sum[hop & 1] + g * S.chunk_stride, ((int64_t)n_h + kChunk - 1) / kChunk);
    if (threadIdx.x == 0) {
        rg_hop_list(S, g, hop, kIndptr)[n_h] = total;
        rg_put_edges(S, g, hop, total);
    }
}

// Per-block counts of fresh ids -> exclusive offsets; the end of the new tier goes to tier_off[hop + 2].  block_edges: a block is
// that many of the hop's edges, of which there may be more or fewer than were launched for; 0: there are tier_blocks of them.
__global__ void __launch_bounds__(1024) k_scan_tier(const SampleScratch S, int hop, int tier_blocks, int block_edges) {
    const int g = rg_batch(S);
    if (block_edges) {
        const int n = rg_hop_list(S, g, hop, kIndptr)[rg_tier_off(S, g)[hop + 1]];
        tier_blocks = n / block_edges + (n % block_edges != 0);
    }
    const int total = rg_scan_in_place(S.chunk_sum + g * S.chunk_stride, tier_blocks);
    if (threadIdx.x == 0) rg_tier_off(S, g)[hop + 2] = rg_tier_off(S, g)[hop + 1] + total;
}

// ---------------------------------------------------------------------------- per hop: draw + read
// `marked` holds every id a batch has met so far: the frontier members (`visited`) plus the ids the current hop has
// sampled.  One probe per sampled edge; the hop's new tier is marked & ~visited.  A stale probe only costs a redundant atomic.
// The probes of a thread's U ids (those whose bit of `live` is set) are on their way together: one behind the other a draw of 8 ids a thread
// waited for them twice as long as for its columns.
template <int U>
__device__ __forceinline__ void rg_mark(const int32_t (&u)[U], uint32_t live, uint32_t* __restrict__ marked) {
    uint32_t old[U];
#pragma unroll
    for (int q = 0; q < U; ++q) old[q] = (live >> q) & 1u ? marked[(uint32_t)u[q] >> 5] : ~0u;
#pragma unroll
    for (int q = 0; q < U; ++q)
        if (!((old[q] >> (u[q] & 31)) & 1u) && ((live >> q) & 1u)) atomicOr(&marked[(uint32_t)u[q] >> 5], 1u << (u[q] & 31));
}

// kTierBytes: a byte store, which waits for nothing, where an atomic on a word that many edges name waits for all of theirs.
__device__ __forceinline__ void rg_mark_byte(const SampleScratch& S, int g, int32_t u) { rg_bytes(S, g)[u] = 1; }

// First-seen order: instead of a bit, remember the first edge of the hop that names a node outside the frontier.  Edge of u[q]: e + q * step.
template <int U>
__device__ __forceinline__ void rg_note_first_edges(const int32_t (&u)[U], uint32_t live, int64_t e, int step, const uint32_t* __restrict__ visited,
                                                    int32_t* __restrict__ first_key) {
    uint32_t members[U];
    int32_t old[U];
#pragma unroll
    for (int q = 0; q < U; ++q) {
        members[q] = ~0u;
        old[q] = 0;
        if ((live >> q) & 1u) { members[q] = visited[(uint32_t)u[q] >> 5]; old[q] = first_key[u[q]]; }
    }
#pragma unroll
    for (int q = 0; q < U; ++q) {
        const int32_t key = 0x7FFFFFFF - (int32_t)(e + q * step);
        if (!((members[q] >> (u[q] & 31)) & 1u) && old[q] < key && ((live >> q) & 1u)) atomicMax(&first_key[u[q]], key);
    }
}
template <int MODE, int U>
__device__ __forceinline__ void rg_note(const SampleScratch& S, int g, const int32_t (&u)[U], uint32_t live, int64_t e, int step) {
    if (MODE == kTierFirstSeen) rg_note_first_edges<U>(u, live, e, step, S.visited + g * S.words, S.first_key + g * S.num_nodes);
    if (MODE == kTierAtomic) rg_mark<U>(u, live, S.marked + g * S.words);
    if (MODE == kTierBytes) {
#pragma unroll
        for (int q = 0; q < U; ++q)
            if ((live >> q) & 1u) rg_mark_byte(S, g, u[q]);
    }
}

// The tiers' emits add to the next hop's sums, which the draw in front of them clears (with slices k_slice_mark does).
__device__ __forceinline__ void rg_clear_next_sum(const SampleScratch& S, int g, uint32_t hop, int64_t thread, int64_t threads) {
    int32_t* __restrict__ next_sum = S.hop_sum[(hop + 1) & 1] + g * S.chunk_stride;
    for (int64_t c = thread; c <= S.frontier_stride / kChunk; c += threads) next_sum[c] = 0;
}

// General sampler (fan-outs above 64, all neighbours, more than kWideNodes): one wavefront (= one 64-thread workgroup) per frontier node, any
// fan-out up to RG_MAX_FANOUT.  The Floyd set lives in LDS; step i tests membership of t with all lanes.
template <int MODE>
__global__ void __launch_bounds__(RG_WAVE) k_hop_sample_wave(const int32_t* __restrict__ col_idx, const SampleScratch S, int fanout, uint32_t hop, uint32_t k0,
                                                            uint32_t k1, uint32_t epoch) {
    __shared__ uint32_t draws[RG_MAX_FANOUT];
    __shared__ uint32_t chosen[RG_MAX_FANOUT];
    const int g = rg_batch(S);
    const unsigned blk = rg_block(S);
    const int n_h = rg_tier_off(S, g)[hop + 1];
    const int32_t* __restrict__ nodes = rg_nodes(S, g);
    int32_t* __restrict__ indptr = rg_hop_list(S, g, (int)hop, kIndptr);
    int32_t* __restrict__ nbr = rg_hop_list(S, g, (int)hop, kNbr);
    const int32_t* __restrict__ hop_sum = S.hop_sum[hop & 1] + g * S.chunk_stride;
    const int64_t* __restrict__ row_start = S.row_start + g * S.frontier_stride;
    const int32_t* __restrict__ row_deg = S.row_deg + g * S.frontier_stride;
    const int lane = threadIdx.x;
    if (MODE != kTierSliced) rg_clear_next_sum(S, g, hop, (int64_t)blk * RG_WAVE + lane, (int64_t)rg_blocks_per_batch(S) * RG_WAVE);
    for (int64_t i = blk; i < n_h; i += rg_blocks_per_batch(S)) {
        const int32_t v = nodes[i];
        const int64_t start = row_start[i], deg = row_deg[i];
        const int base = indptr[i] + hop_sum[i / kChunk];
        __syncthreads();                               // every lane has read indptr[i] before it is rewritten
        if (lane == 0) indptr[i] = base;
        if (fanout < 0 || deg <= fanout) {             // whole row, CSR order
            for (int64_t t = lane; t < deg; t += RG_WAVE) {
                const int32_t u[1] = {col_idx[start + t]};
                nbr[base + t] = u[0];
                rg_note<MODE, 1>(S, g, u, 1u, base + t, 0);
            }
            continue;
        }
        const int k = fanout;
        for (int blk = lane; blk * 4 < k; blk += RG_WAVE) {
            uint32_t w[4];
            rg_philox4x32_10((uint32_t)v, hop, (uint32_t)blk, epoch, k0, k1, w);
#pragma unroll
            for (int q = 0; q < 4; ++q)
                if (blk * 4 + q < k) draws[blk * 4 + q] = w[q];
        }
        __syncthreads();
        for (int s = 0; s < k; ++s) {                  // Floyd: j = d-k+s, t uniform in [0, j]
            const uint32_t j = (uint32_t)(deg - k + s);
            const uint32_t t = __umulhi(draws[s], j + 1u);
            int found = 0;
            for (int l = lane; l < s; l += RG_WAVE) found |= (chosen[l] == t);
            found = __any(found);
            __syncthreads();
            if (lane == 0) chosen[s] = found ? j : t;
            __syncthreads();
        }
        for (int t = lane; t < k; t += RG_WAVE) {
            const int32_t u[1] = {col_idx[start + (int64_t)chosen[t]]};
            nbr[base + t] = u[0];
            rg_note<MODE, 1>(S, g, u, 1u, base + t, 0);
        }
    }
}

// Fast sampler for fan-outs up to 32 on graphs with fewer than 2^32 edges: NODES frontier nodes per workgroup of 256
// threads, one thread per node draws (Philox + Floyd entirely in registers) and stages the col_idx offsets of its picks in
// LDS in output order, then the whole workgroup reads col_idx and writes nbr with consecutive lanes on consecutive output
// slots.  Bound by the random col_idx lines, so every thread keeps kDrawLoads of them in flight (one at a time: hop 0 of
// 8 batches of 4096 seeds 35 us, hop 1 235 us with its marking atomics; now 15 and 66).
// NODES = 64 spreads the reads of a frontier that fills less than two workgroups of 256 nodes per compute unit.
constexpr int kDrawLoads = 8;
constexpr int kDrawSelfScan = 16384;    // count chunks up to which a workgroup adds up those in front of its own itself

// A thread's part (of a workgroup of 256) of the edges in front of frontier node `first`: the chunks in front of its own, then the
// nodes in front of it within the chunk.
__device__ __forceinline__ int rg_edges_before(const SampleScratch& S, int g, int hop, int64_t first, int fanout, int scanned) {
    const int32_t* __restrict__ hop_sum = S.hop_sum[hop & 1] + g * S.chunk_stride;
    const int32_t* __restrict__ row_deg = S.row_deg + g * S.frontier_stride;
    const int chunk = (int)(first / kChunk);
    int before = 0;
    for (int64_t i = (int64_t)chunk * kChunk + threadIdx.x; i < first; i += 256) {
        const int deg = row_deg[i];
        before += deg <= fanout ? deg : fanout;
    }
    if (scanned) {
        if (threadIdx.x == 0) before += hop_sum[chunk];
    } else {
        for (int c = threadIdx.x; c < chunk; c += 256) before += hop_sum[c];
    }
    return rg_wave_sum(before);
}

template <int KMAX, int NODES, int MODE>
__global__ void __launch_bounds__(256) k_hop_sample_thread(const int32_t* __restrict__ col_idx, const SampleScratch S, int fanout, uint32_t hop, uint32_t k0,
                                                           uint32_t k1, uint32_t epoch, int scanned, int run) {
    extern __shared__ uint32_t staged[];                 // NODES * fanout col_idx offsets
    __shared__ int part[4];
    __shared__ int smem[5];
    int g;
    unsigned blk;
    rg_shared_rows(S, run, g, blk);
    const int n_h = rg_tier_off(S, g)[hop + 1];
    int32_t* __restrict__ indptr = rg_hop_list(S, g, (int)hop, kIndptr);
    const int64_t first = (int64_t)blk * NODES;
    if (MODE != kTierSliced) rg_clear_next_sum(S, g, hop, (int64_t)blk * 256 + threadIdx.x, (int64_t)rg_blocks_per_batch(S) * 256);
    if (first >= n_h) {                                  // uniform per workgroup
        if (n_h == 0 && blk == 0 && threadIdx.x == 0) {
            indptr[0] = 0;
            rg_put_edges(S, g, (int)hop, 0);
        }
        return;
    }
    int32_t* __restrict__ nbr = rg_hop_list(S, g, (int)hop, kNbr);
    const int64_t i = first + threadIdx.x;
    const int k = fanout;
    const int n_here = (int)(n_h - first < NODES ? n_h - first : NODES);
    int32_t v = 0;
    int64_t start = 0, deg = 0;
    if ((int)threadIdx.x < n_here) {
        v = rg_nodes(S, g)[i];
        start = S.row_start[g * S.frontier_stride + i];
        deg = S.row_deg[g * S.frontier_stride + i];
    }
    const int before = rg_edges_before(S, g, (int)hop, first, k, scanned);
    if (rg_lane() == 0) part[threadIdx.x >> 6] = before;
    int n_edges;
    const int off = rg_block_excl_scan<4>((int)(deg <= k ? deg : k), smem, &n_edges);       // its barriers publish part[]
    if ((int)threadIdx.x < n_here) {
        if (deg <= k) {                                  // whole row, CSR order
            for (int t = 0; t < (int)deg; ++t) staged[off + t] = (uint32_t)(start + t);
        } else {
            uint32_t c[KMAX];
#pragma unroll
            for (int blk = 0; blk < KMAX / 4; ++blk) {
                if (blk * 4 < k) {
                    uint32_t w[4];
                    rg_philox4x32_10((uint32_t)v, hop, (uint32_t)blk, epoch, k0, k1, w);
#pragma unroll
                    for (int q = 0; q < 4; ++q) {
                        const int s = blk * 4 + q;
                        if (s < k) {                     // Floyd: j = d-k+s, t uniform in [0, j]
                            const uint32_t j = (uint32_t)(deg - k + s);
                            const uint32_t t = __umulhi(w[q], j + 1u);
                            bool found = false;
#pragma unroll
                            for (int l = 0; l < s; ++l) found |= (c[l] == t);
                            c[s] = found ? j : t;
                        }
                    }
                }
            }
#pragma unroll
            for (int s = 0; s < KMAX; ++s)
                if (s < k) staged[off + s] = (uint32_t)(start + (int64_t)c[s]);
        }
    }
    __syncthreads();
    const int base = part[0] + part[1] + part[2] + part[3];
    if ((int)threadIdx.x < n_here) indptr[i] = base + off;
    if (threadIdx.x == 0 && first + NODES >= n_h) {
        indptr[n_h] = base + n_edges;
        rg_put_edges(S, g, (int)hop, base + n_edges);
    }
    for (int e0 = threadIdx.x; e0 < n_edges; e0 += 256 * kDrawLoads) {
        int32_t u[kDrawLoads];
#pragma unroll
        for (int q = 0; q < kDrawLoads; ++q)
            if (e0 + 256 * q < n_edges) u[q] = col_idx[staged[e0 + 256 * q]];
        uint32_t live = 0u;
#pragma unroll
        for (int q = 0; q < kDrawLoads; ++q) {
            const int e = e0 + 256 * q;
            if (e >= n_edges) break;
            nbr[base + e] = u[q];
            live |= 1u << q;
        }
        rg_note<MODE, kDrawLoads>(S, g, u, live, base + e0, 256);
    }
}

// Draws (lanes) of a hop for which k_hop_sample_lanes is faster: 1024 nodes of 25 neighbours 11.2 -> 7.2 us, three batches' 78 k nodes of 10
// (1.25 M lanes) make the call 66 us against 63.  With fan-outs up to 16 a thread per node takes less (10: 5.4 against 7.4 us, 5: 4.7 / 6.6).
constexpr int64_t kLaneDraws = 1 << 18;
// Frontier nodes up to which it draws for fan-outs of 33 to 64, where the other way is a wavefront per node with its set in LDS behind two launches for
// the offsets: 64 of 0.5 M nodes 680 us a call against 1014, 40 of 2.4 M 1436 / 1773, 64 of eight batches of 91 nodes 33 / 60.  (Beyond, every
// workgroup of four nodes adding up the chunks in front of it would be what takes time.)
constexpr int64_t kWideNodes = 1 << 22, kWideNodesAll = 1 << 24;

// The same for few frontier nodes of large fan-outs, and all of 33 to 64: KMAX lanes per node, one draw each, no staging.  Floyd's set by itself: draw s is taken already if an
// earlier draw has its value, or if its value is the last position j_l of an earlier step l that found its own draw taken.
template <int KMAX, int MODE>
__global__ void __launch_bounds__(256) k_hop_sample_lanes(const int32_t* __restrict__ col_idx, const SampleScratch S, int fanout, uint32_t hop, uint32_t k0,
                                                          uint32_t k1, uint32_t epoch) {
    constexpr int NODES = 256 / KMAX;
    static_assert(RG_WAVE % KMAX == 0 && kChunk % NODES == 0, "a node's lanes share a wavefront, a workgroup's nodes a chunk");
    __shared__ int part[4];
    __shared__ int smem[5];
    const int g = rg_batch(S);
    const unsigned blk = rg_block(S);
    const int n_h = rg_tier_off(S, g)[hop + 1];
    int32_t* __restrict__ indptr = rg_hop_list(S, g, (int)hop, kIndptr);
    const int64_t first = (int64_t)blk * NODES;
    if (MODE != kTierSliced) rg_clear_next_sum(S, g, hop, (int64_t)blk * 256 + threadIdx.x, (int64_t)rg_blocks_per_batch(S) * 256);
    if (first >= n_h) {                                  // uniform per workgroup
        if (n_h == 0 && blk == 0 && threadIdx.x == 0) {
            indptr[0] = 0;
            rg_put_edges(S, g, (int)hop, 0);
        }
        return;
    }
    const int lane = (int)threadIdx.x & (KMAX - 1), k = fanout;
    const int64_t i = first + threadIdx.x / KMAX;
    const bool live = i < n_h;
    int32_t v = 0;
    int64_t start = 0, deg = 0;
    if (live) {
        v = rg_nodes(S, g)[i];
        start = S.row_start[g * S.frontier_stride + i];
        deg = S.row_deg[g * S.frontier_stride + i];
    }
    const int m = (int)(deg <= k ? deg : k);
    const int before = rg_edges_before(S, g, (int)hop, first, k, 0);
    if (rg_lane() == 0) part[threadIdx.x >> 6] = before;
    uint32_t at = (uint32_t)lane;                        // whole row, CSR order
    if (__any(live && deg > k)) {
        uint32_t w[4];
        rg_philox4x32_10((uint32_t)v, hop, (uint32_t)lane >> 2, epoch, k0, k1, w);
        const uint32_t word = lane & 2 ? (lane & 1 ? w[3] : w[2]) : (lane & 1 ? w[1] : w[0]);
        const uint32_t j0 = (uint32_t)(deg - k), j = j0 + (uint32_t)lane;      // Floyd: j = d-k+s, t uniform in [0, j]
        const uint32_t t = __umulhi(word, j + 1u);
        bool taken = false;
        for (int l = 0; l + 1 < k; ++l) {
            if constexpr (KMAX == RG_WAVE) taken |= (uint32_t)__builtin_amdgcn_readlane((int)t, l) == t && l < lane;
            else taken |= (uint32_t)__shfl((int)t, l, KMAX) == t && l < lane;
        }
        const int node0 = rg_lane() & ~(KMAX - 1);
        const int l = (int)(t - j0);                     // the step whose last position t is
        const bool late = deg > k && t >= j0 && l < lane;
        for (;;) {                                       // a step is added to the taken ones at most once: k rounds at most
            const unsigned long long all = __ballot(taken);
            const bool more = late && !taken && ((all >> (node0 + l)) & 1ull);
            if (!__any(more)) break;
            taken |= more;
        }
        if (deg > k) at = taken ? j : t;
    }
    int total;
    int off = rg_block_excl_scan<4>(lane == 0 ? m : 0, smem, &total);          // its barriers publish part[]
    off = __shfl(off, 0, KMAX) + part[0] + part[1] + part[2] + part[3];
    if (!live) return;
    if (lane == 0) {
        indptr[i] = off;
        if (i == n_h - 1) {
            indptr[n_h] = off + m;
            rg_put_edges(S, g, (int)hop, off + m);
        }
    }
    if (lane >= m) return;
    const int32_t u[1] = {col_idx[start + at]};
    rg_hop_list(S, g, (int)hop, kNbr)[off + lane] = u[0];
    rg_note<MODE, 1>(S, g, u, 1u, off + lane, 0);
}

// ---------------------------------------------------------------------------- per hop: new tier, sliced
// slice_marks[split][w] = the ids of the hop's edges of that split, one workgroup per (batch, slice of ids, split of the edges).
// The workgroups of a batch read the same list side by side, so all but the first read of a line hits L2.
__device__ __forceinline__ void rg_slice_or(uint32_t* bits, int32_t u, uint32_t id0, uint32_t n_ids) {
    const uint32_t d = (uint32_t)u - id0;
    if (d < n_ids) atomicOr(&bits[d >> 5], 1u << (d & 31u));
}

__global__ void __launch_bounds__(1024) k_slice_mark(const SampleScratch S, int hop) {
    extern __shared__ uint32_t slice_bits[];
    constexpr int U = 4;                                 // 16-byte loads in flight per thread
    const int g = rg_batch(S);
    const unsigned blk = rg_block(S);
    int32_t* __restrict__ next_sum = S.hop_sum[(hop + 1) & 1] + g * S.chunk_stride;        // k_slice_emit adds to it
    for (int64_t c = (int64_t)blk * 1024 + threadIdx.x; c < S.chunk_stride; c += (int64_t)rg_blocks_per_batch(S) * 1024) next_sum[c] = 0;
    const int split = S.slices == 1 ? (int)blk : (int)(blk / (unsigned)S.slices), slice = (int)blk - split * S.slices;
    const int64_t w0 = (int64_t)slice * S.slice_words;
    const int n_words = (int)(S.words - w0 < S.slice_words ? S.words - w0 : S.slice_words);
    for (int w = threadIdx.x; w < n_words; w += 1024) slice_bits[w] = 0u;
    const int n_edges = rg_hop_list(S, g, (int)hop, kIndptr)[rg_tier_off(S, g)[hop + 1]];
    const int each = S.splits == 1 ? n_edges : (int)((uint32_t)n_edges / (uint32_t)S.splits), rest = n_edges - each * S.splits;
    const int64_t e0 = (int64_t)split * each + (split < rest ? split : rest);
    const int n = each + (split < rest ? 1 : 0);
    const int32_t* __restrict__ nbr = rg_hop_list(S, g, (int)hop, kNbr) + e0;
    const uint32_t id0 = (uint32_t)(w0 << 5), n_ids = (uint32_t)n_words << 5;
    __syncthreads();
    // the list may start at any 4-byte address: single ids up to the first 16-byte boundary and behind the last one
    const int to_line = (int)((16u - ((uint32_t)(uintptr_t)nbr & 15u)) & 15u) / 4;
    const int head = to_line < n ? to_line : n;
    const int n4 = (n - head) / 4;
    const int4* __restrict__ body = (const int4*)(nbr + head);
    int i = threadIdx.x;
    for (; i + (U - 1) * 1024 < n4; i += U * 1024) {
        int4 x[U];
#pragma unroll
        for (int q = 0; q < U; ++q) x[q] = body[i + q * 1024];
#pragma unroll
        for (int q = 0; q < U; ++q) {
            rg_slice_or(slice_bits, x[q].x, id0, n_ids);
            rg_slice_or(slice_bits, x[q].y, id0, n_ids);
            rg_slice_or(slice_bits, x[q].z, id0, n_ids);
            rg_slice_or(slice_bits, x[q].w, id0, n_ids);
        }
    }
    for (; i < n4; i += 1024) {
        const int4 x = body[i];
        rg_slice_or(slice_bits, x.x, id0, n_ids);
        rg_slice_or(slice_bits, x.y, id0, n_ids);
        rg_slice_or(slice_bits, x.z, id0, n_ids);
        rg_slice_or(slice_bits, x.w, id0, n_ids);
    }
    if ((int)threadIdx.x < head) rg_slice_or(slice_bits, nbr[threadIdx.x], id0, n_ids);
    const int tail = head + 4 * n4;
    if ((int)threadIdx.x < n - tail) rg_slice_or(slice_bits, nbr[tail + threadIdx.x], id0, n_ids);
    __syncthreads();
    uint32_t* __restrict__ out = S.slice_marks + ((int64_t)g * S.splits + split) * S.words + w0;
    for (int w = threadIdx.x; w < n_words; w += 1024) out[w] = slice_bits[w];
}

// W consecutive words from w on; words behind the end read as 0 (`whole`, uniform: none are).
template <int W>
__device__ __forceinline__ void rg_load_words(const uint32_t* __restrict__ p, int64_t w, int64_t words, bool whole, uint32_t (&x)[W]) {
    if (whole) {
#pragma unroll
        for (int q = 0; q < W; ++q) x[q] = p[w + q];
    } else {
#pragma unroll
        for (int q = 0; q < W; ++q) x[q] = w + q < words ? p[w + q] : 0u;
    }
}

// The splits' bitmaps -> the new tier's bits (into split 0) and the number of them per workgroup of T threads, W words each.
template <int T, int W>
__global__ void __launch_bounds__(T) k_slice_count(const SampleScratch S) {
    constexpr int NW = T / RG_WAVE;
    __shared__ int part[NW];
    const int g = rg_batch(S);
    const unsigned blk = rg_block(S);
    const int64_t w = ((int64_t)blk * T + threadIdx.x) * W;
    uint32_t* __restrict__ marks = S.slice_marks + (int64_t)g * S.splits * S.words;
    const bool whole = ((int64_t)blk + 1) * T * W <= S.words;
    uint32_t bits[W], members[W];
    rg_load_words<W>(S.visited + g * S.words, w, S.words, whole, members);
    rg_load_words<W>(marks, w, S.words, whole, bits);
    const auto join = [&](bool all) {
#pragma unroll 8
        for (int s = 1; s < S.splits; ++s) {
            uint32_t more[W];
            rg_load_words<W>(marks + s * S.words, w, S.words, all, more);
#pragma unroll
            for (int q = 0; q < W; ++q) bits[q] |= more[q];
        }
    };
    if (whole) join(true); else join(false);
    int c = 0;
#pragma unroll
    for (int q = 0; q < W; ++q) {
        bits[q] &= ~members[q];
        if (w + q < S.words) marks[w + q] = bits[q];
        c += __popc(bits[q]);
    }
    c = rg_wave_sum(c);
    if (rg_lane() == 0) part[threadIdx.x >> 6] = c;
    __syncthreads();
    if (threadIdx.x < RG_WAVE) {
        const int total = rg_wave_sum(threadIdx.x < NW ? part[threadIdx.x] : 0);
        if (threadIdx.x == 0) S.chunk_sum[g * S.chunk_stride + blk] = total;
    }
}

// Where a workgroup keeps its new ids until consecutive lanes store them: as distances from its first id where its LDS decides how many workgroups
// a compute unit takes (three words to a thread: 33 KB, four workgroups; 17 KB, eight: the emits of three hops of 8 stress batches 24 + 48 + 25 us,
// now 21.5 + 46 + 23), else as they are (a distance more to add: 1 % of calls of 50 us).
template <int W> using EmitId = typename std::conditional<W == 1, int32_t, uint16_t>::type;

// The ids of the bits of word `w` of a workgroup's words, from place j on, which moves on behind them: into LDS, or to nodes[].
template <class Id>
__device__ __forceinline__ void rg_put_ids(uint32_t bits, int w, bool in_lds, Id* ids, int32_t* __restrict__ nodes, int32_t first_id, int& j) {
    if constexpr (sizeof(Id) == 4) {
        int32_t* dst = in_lds ? ids : nodes;
        for (uint32_t b = bits; b; b &= b - 1u) dst[j++] = first_id + (w << 5) + __ffs(b) - 1;
    } else if (in_lds) {
        for (uint32_t b = bits; b; b &= b - 1u) ids[j++] = (Id)((w << 5) + __ffs(b) - 1);
    } else {
        for (uint32_t b = bits; b; b &= b - 1u) nodes[j++] = first_id + (w << 5) + __ffs(b) - 1;
    }
}

// What k_hop_count does for the next hop, by the kernels that emit a tier of ascending ids: the rows of its `total` nodes from position
// `out` on, and their edges per chunk; the edges of the nodes in front of them, a chunk to a workgroup.
// in_lds: the new ids are in LDS (EmitId) and go to nodes[] here; else they are there already.  POS: their positions go to pos[] too.
template <int T, bool POS, class Id>
__device__ __forceinline__ void rg_new_rows(const RowPtr& row_ptr, const SampleScratch& S, int g, int hop, int out, int total,
                                            int32_t* __restrict__ nodes, const Id* ids, int32_t first_id, bool in_lds, int* edges, int num_chunks,
                                            int next_fanout) {
    constexpr int U = 4;                                 // rows in flight per thread
    int32_t* __restrict__ pos = S.pos + g * S.num_nodes;
    int64_t* __restrict__ row_start = S.row_start + g * S.frontier_stride + out;
    int32_t* __restrict__ row_deg = S.row_deg + g * S.frontier_stride + out;
    for (int i0 = threadIdx.x; i0 < total; i0 += T * U) {
        int32_t v[U];
        int64_t start[U], deg[U];
#pragma unroll
        for (int q = 0; q < U; ++q) {
            v[q] = -1;
            if (i0 + T * q >= total) continue;
            if constexpr (sizeof(Id) == 4) v[q] = in_lds ? ids[i0 + T * q] : nodes[i0 + T * q];
            else if (in_lds) v[q] = first_id + ids[i0 + T * q];
            else v[q] = nodes[i0 + T * q];
        }
        if (in_lds) {
#pragma unroll
            for (int q = 0; q < U; ++q)
                if (v[q] >= 0) nodes[i0 + T * q] = v[q];
        }
        if (POS) {
#pragma unroll
            for (int q = 0; q < U; ++q)
                if (v[q] >= 0) pos[v[q]] = out + i0 + T * q;
        }
        if (next_fanout < 0) continue;
        const auto rows = [&](auto* p) {
#pragma unroll
            for (int q = 0; q < U; ++q)
                if (v[q] >= 0) rg_row_extent(p, v[q], start[q], deg[q]);
        };
        if (row_ptr.wide) rows((const int64_t*)row_ptr.p); else rows((const int32_t*)row_ptr.p);
#pragma unroll
        for (int q = 0; q < U; ++q)
            if (v[q] >= 0) {
                row_start[i0 + T * q] = start[q];
                row_deg[i0 + T * q] = (int32_t)deg[q];
                atomicAdd(&edges[(out + i0 + T * q) / kChunk - out / kChunk], (int)(deg[q] <= next_fanout ? deg[q] : next_fanout));
            }
    }
    if (next_fanout < 0) return;
    __syncthreads();
    int32_t* __restrict__ next_sum = S.hop_sum[(hop + 1) & 1] + g * S.chunk_stride;
    for (int i = threadIdx.x; i < num_chunks; i += T)
        if (edges[i]) atomicAdd(&next_sum[out / kChunk + i], edges[i]);
}

template <int T>
__device__ __forceinline__ void rg_old_edges(const SampleScratch& S, int g, int hop, int chunk, int next_fanout) {
    const int n_h = rg_tier_off(S, g)[hop + 1];
    if (chunk * kChunk >= n_h) return;                                   // uniform
    const int32_t* __restrict__ row_deg = S.row_deg + g * S.frontier_stride;
    int m = 0;
    for (int i = chunk * kChunk + threadIdx.x; i < n_h && i < (chunk + 1) * kChunk; i += T) {
        const int deg = row_deg[i];
        m += deg <= next_fanout ? deg : next_fanout;
    }
    m = rg_wave_sum(m);
    if (rg_lane() == 0 && m) atomicAdd(&S.hop_sum[(hop + 1) & 1][g * S.chunk_stride + chunk], m);
}

// Emits the new tier behind the current frontier, ascending, with its rank blocks, and makes its ids frontier members.  The
// ids go through LDS so that they are stored by consecutive lanes (thread by thread: 135 us at hop 2 of 8 batches, 7.5 M ids;
// now 23); a workgroup with more new ids than fit there (over a third of its range) stores them directly.
// A thread takes W words: three, which are two rank blocks, or one where few workgroups leave the serial walk over the bits of a
// word as what takes time; the words then meet in LDS.
// RANKED_SEEN: the positions are ascending ones only, the nodes come later.
// next_fanout >= 0: also what k_hop_count does for the next hop, the new nodes' rows here, where their ids are at hand and ascending, and
// their edges per chunk; those of the nodes in front of them by the workgroups behind the tier_blocks.  (Hop 1 of the same batches,
// 3.3 M rows: 46 us with the next hop's sizes, 20 + 44 apart; on XCDs of their own, without sharing lines of row_ptr, 65.)
template <bool RANKED_SEEN, int T, int W, int WORDS = T * W>
__device__ __forceinline__ void rg_slice_emit(const RowPtr& row_ptr, const SampleScratch& S, int hop,
                                              unsigned tier_blocks, int next_fanout, int run) {
    constexpr int NW = T / RG_WAVE, kEmitIds = W == 1 ? WORDS * 32 : WORDS * 32 / 3;
    constexpr int TW = WORDS / W;                        // threads that take words
    constexpr unsigned per_base = kBaseIds / (32 * WORDS);               // workgroups to a base
    __shared__ int smem[NW + 1];
    __shared__ int part[NW], part_above[NW];
    __shared__ EmitId<W> ids[RANKED_SEEN ? 1 : kEmitIds];
    static_assert(WORDS * 32 <= 1 << 16, "ids are kept as 16-bit distances");
    __shared__ uint32_t word_bits[W == 1 ? TW : 1];
    __shared__ int word_rank[W == 1 ? TW : 1];
    __shared__ int edges[WORDS * 32 / kChunk + 2];
    int g;
    unsigned blk;
    rg_shared_rows(S, run, g, blk);
    if (!RANKED_SEEN && blk >= tier_blocks) {
        rg_old_edges<T>(S, g, hop, (int)(blk - tier_blocks), next_fanout);
        return;
    }
    if (!RANKED_SEEN) for (int i = threadIdx.x; i < (int)(sizeof(edges) / sizeof(int)); i += T) edges[i] = 0;
    const int64_t w = TW == T || (int)threadIdx.x < TW ? ((int64_t)blk * TW + threadIdx.x) * W : S.words;
    const int32_t* __restrict__ chunk_sum = S.chunk_sum + g * S.chunk_stride;
    uint32_t* __restrict__ visited = S.visited + g * S.words;
    uint32_t bits[W], members[W];
    const bool whole = TW == T && ((int64_t)blk + 1) * WORDS <= S.words;
    rg_load_words<W>(S.slice_marks + (int64_t)g * S.splits * S.words, w, S.words, whole, bits);
    rg_load_words<W>(visited, w, S.words, whole, members);
    int before = 0, above = 0;                           // new ids in front of this workgroup's words, those behind the last base
    const unsigned base_blk = blk / per_base * per_base;
    for (unsigned c = threadIdx.x; c < blk; c += T) {
        const int n = chunk_sum[c];
        before += n;
        if (c >= base_blk) above += n;
    }
    before = rg_wave_sum(before);
    above = rg_wave_sum(above);
    if (rg_lane() == 0) { part[threadIdx.x >> 6] = before; part_above[threadIdx.x >> 6] = above; }
    int mine = 0;
#pragma unroll
    for (int q = 0; q < W; ++q) mine += __popc(bits[q]);
    int total;
    int j = rg_block_excl_scan<NW>(mine, smem, &total);                        // its barriers publish part[]
    int out = rg_tier_off(S, g)[hop + 1];
#pragma unroll
    for (int q = 0; q < NW; ++q) out += part[q];
    if (threadIdx.x == 0 && blk + 1 == tier_blocks) rg_tier_off(S, g)[hop + 2] = out + total;
    int base = out;
#pragma unroll
    for (int q = 0; q < NW; ++q) base -= part_above[q];
    if (threadIdx.x == 0 && blk == base_blk) rg_rank_bases(S, g, hop)[blk / per_base] = base;
    int32_t* __restrict__ nodes = rg_nodes(S, g) + out;
    const bool in_lds = total <= kEmitIds;
    const int32_t first_id = (int32_t)((int64_t)blk * WORDS * 32);
    const RankBlocks rank = rg_rank_blocks(S, g, hop);
    const auto store_rank = [&](int64_t r, uint32_t b0, uint32_t b1, uint32_t b2, uint32_t above) {      // three words: two rank blocks
        rank.at[2 * r * rank.stride] = make_uint2(b0, (b1 & 0xFFFFu) | above << 16);
        above += (uint32_t)(__popc(b0) + __popc(b1 & 0xFFFFu));
        rank.at[(2 * r + 1) * rank.stride] = make_uint2(b1 >> 16 | b2 << 16, b2 >> 16 | above << 16);
    };
    if (W == 3) {
        if (w < S.words) store_rank(w / 3, bits[0], bits[W / 3], bits[W - 1], (uint32_t)(out + j - base));
    } else {
        if (TW == T || (int)threadIdx.x < TW) {
            word_bits[threadIdx.x] = bits[0];
            word_rank[threadIdx.x] = out + j - base;
        }
    }
#pragma unroll
    for (int q = 0; q < W; ++q) {
        if (bits[q]) visited[w + q] = members[q] | bits[q];
        if (!RANKED_SEEN) rg_put_ids<EmitId<W>>(bits[q], (int)threadIdx.x * W + q, in_lds, ids, nodes, first_id, j);
    }
    if (RANKED_SEEN && W == 3) return;
    __syncthreads();                                     // ids, nodes, words and edges are there
    if (W == 1 && threadIdx.x < TW / 3) {
        const int q = 3 * threadIdx.x;
        const int64_t r = (int64_t)blk * (TW / 3) + threadIdx.x;
        if (3 * r < S.words) store_rank(r, word_bits[q], word_bits[q + 1], word_bits[q + 2], (uint32_t)word_rank[q]);
    }
    if (RANKED_SEEN) return;
    rg_new_rows<T, false, EmitId<W>>(row_ptr, S, g, hop, out, total, nodes, ids, first_id, in_lds, edges, (int)(sizeof(edges) / sizeof(int)), next_fanout);
}

template <bool RANKED_SEEN>
__global__ void __launch_bounds__(kTierWords / 3) k_slice_emit(const RowPtr row_ptr, const SampleScratch S, int hop,
                                                               unsigned tier_blocks, int next_fanout, int run) {
    rg_slice_emit<RANKED_SEEN, kTierWords / 3, 3>(row_ptr, S, hop, tier_blocks, next_fanout, run);
}

template <bool RANKED_SEEN>
__global__ void __launch_bounds__(kEmitThreadsSmall) k_slice_emit_small(const RowPtr row_ptr, const SampleScratch S, int hop,
                                                                      unsigned tier_blocks, int next_fanout, int run) {
    rg_slice_emit<RANKED_SEEN, kEmitThreadsSmall, 1, kTierWordsSmall>(row_ptr, S, hop, tier_blocks, next_fanout, run);
}

// ---------------------------------------------------------------------------- per hop: new tier, from `marked`
// chunk_sum[b] = new ids (marked, not yet visited) of the words_per words of workgroup b.
__global__ void __launch_bounds__(256) k_tier_count(const SampleScratch S, int words_per) {
    __shared__ int part[4];
    const int g = rg_batch(S);
    const unsigned blk = rg_block(S);
    const uint32_t* __restrict__ marked = S.marked + g * S.words;
    const uint32_t* __restrict__ visited = S.visited + g * S.words;
    const int64_t w0 = (int64_t)blk * words_per, w1 = w0 + words_per < S.words ? w0 + words_per : S.words;
    int c = 0;
    for (int64_t w = w0 + threadIdx.x; w < w1; w += 256) c += __popc(marked[w] & ~visited[w]);
    c = rg_wave_sum(c);
    if (rg_lane() == 0) part[threadIdx.x >> 6] = c;
    __syncthreads();
    if (threadIdx.x == 0) S.chunk_sum[g * S.chunk_stride + blk] = part[0] + part[1] + part[2] + part[3];
}

// The 32 bytes of word w as bits.
__device__ __forceinline__ uint32_t rg_byte_word(const uint8_t* __restrict__ bytes, int64_t w) {
    const uint4* p = (const uint4*)bytes + 2 * w;
    const uint4 lo = p[0], hi = p[1];
    const auto four = [](uint32_t x) { return (x * 0x01020408u) >> 24 & 0xFu; };       // (sums of single bits, none of which meet)
    return four(lo.x) | four(lo.y) << 4 | four(lo.z) << 8 | four(lo.w) << 12 | four(hi.x) << 16 | four(hi.y) << 20 | four(hi.z) << 24 | four(hi.w) << 28;
}

// kTierBytes on larger graphs: the same as k_tier_count, and the bytes as bits.
__global__ void __launch_bounds__(256) k_bytes_count(const SampleScratch S, int words_per, int clear) {
    __shared__ int part[4];
    const int g = rg_batch(S);
    const unsigned blk = rg_block(S);
    uint32_t* __restrict__ marked = S.marked + g * S.words;
    uint8_t* __restrict__ bytes = rg_bytes(S, g);
    const uint32_t* __restrict__ visited = S.visited + g * S.words;
    const int64_t w0 = (int64_t)blk * words_per, w1 = w0 + words_per < S.words ? w0 + words_per : S.words;
    int c = 0;
    for (int64_t w = w0 + threadIdx.x; w < w1; w += 256) {
        const uint32_t members = visited[w], bits = rg_byte_word(bytes, w) | members;
        marked[w] = bits;
        if (clear) ((uint4*)bytes)[2 * w] = ((uint4*)bytes)[2 * w + 1] = make_uint4(0u, 0u, 0u, 0u);
        c += __popc(bits & ~members);
    }
    c = rg_wave_sum(c);
    if (rg_lane() == 0) part[threadIdx.x >> 6] = c;
    __syncthreads();
    if (threadIdx.x == 0) S.chunk_sum[g * S.chunk_stride + blk] = part[0] + part[1] + part[2] + part[3];
}

// Emits the new tier behind the current frontier, ascending, makes its ids frontier members and does for the next hop what rg_slice_emit
// does; the positions go to pos[].  A workgroup takes WORDS words, a thread one or three of them.
// What is in front of a workgroup's words: it counts them in the bytes itself (BYTES; `before` is then read by all of them and `after`
// written, two bitmaps that take turns, as do the bytes, of which those of the next hop are cleared here), it adds up what k_tier_count
// found, or k_scan_tier did (scanned).
template <int T, int WORDS, bool BYTES>
__device__ __forceinline__ void rg_tier_emit(const RowPtr& row_ptr, const SampleScratch& S, int hop, unsigned tier_blocks, int next_fanout, int run,
                                             int scanned, const uint32_t* before_all, uint32_t* after_all, uint8_t* next_bytes) {
    constexpr int NW = T / RG_WAVE, W = WORDS > T ? WORDS / T : 1, TW = WORDS / W, kEmitIds = W == 1 ? WORDS * 32 : WORDS * 32 / 3;
    __shared__ int smem[NW + 1];
    __shared__ int part[NW];
    __shared__ EmitId<W> ids[kEmitIds];
    static_assert(WORDS * 32 <= 1 << 16, "ids are kept as 16-bit distances");
    __shared__ int edges[WORDS * 32 / kChunk + 2];
    int g;
    unsigned blk;
    rg_shared_rows(S, run, g, blk);
    if (blk >= tier_blocks) {
        rg_old_edges<T>(S, g, hop, (int)(blk - tier_blocks), next_fanout);
        return;
    }
    const int num_chunks = (int)(sizeof(edges) / sizeof(int));
    for (int i = threadIdx.x; i < num_chunks; i += T) edges[i] = 0;
    const uint32_t* __restrict__ marked = S.marked + g * S.words;
    const uint8_t* __restrict__ bytes = rg_bytes(S, g);
    const uint32_t* before = before_all + g * S.words;
    uint32_t* after = after_all + g * S.words;
    const int n_h = rg_tier_off(S, g)[hop + 1];
    const int64_t w = TW == T || (int)threadIdx.x < TW ? ((int64_t)blk * TW + threadIdx.x) * W : S.words;
    uint32_t bits[W], members[W];
    const bool whole = TW == T && ((int64_t)blk + 1) * WORDS <= S.words;
    rg_load_words<W>(before, w, S.words, whole, members);
    if (BYTES) {
#pragma unroll
        for (int q = 0; q < W; ++q) {
            bits[q] = 0u;
            if (w + q < S.words) {
                bits[q] = rg_byte_word(bytes, w + q) | members[q];
                if (next_bytes) {
                    uint4* clear = (uint4*)(next_bytes + g * S.words * 32) + 2 * (w + q);
                    clear[0] = clear[1] = make_uint4(0u, 0u, 0u, 0u);
                }
            }
        }
    } else {
        rg_load_words<W>(marked, w, S.words, whole, bits);
    }
    int c = 0;
    if (BYTES) {
        const int w_end = (int)blk * WORDS;
#pragma unroll 8
        for (int i = threadIdx.x; i < w_end; i += T) c += __popc(rg_byte_word(bytes, i) & ~before[i]);
    } else if (!scanned) {
        for (unsigned b = threadIdx.x; b < blk; b += T) c += S.chunk_sum[g * S.chunk_stride + b];
    } else if (threadIdx.x == 0) {
        c = S.chunk_sum[g * S.chunk_stride + blk];
    }
    c = rg_wave_sum(c);
    if (rg_lane() == 0) part[threadIdx.x >> 6] = c;
    int mine = 0;
#pragma unroll
    for (int q = 0; q < W; ++q) {
        if (w + q < S.words && (BYTES || bits[q] != members[q])) after[w + q] = bits[q];
        bits[q] &= ~members[q];
        mine += __popc(bits[q]);
    }
    int total;
    int j = rg_block_excl_scan<NW>(mine, smem, &total);                        // its barriers publish part[]
    int out = n_h;
#pragma unroll
    for (int q = 0; q < NW; ++q) out += part[q];
    if (threadIdx.x == 0 && blk + 1 == tier_blocks) rg_tier_off(S, g)[hop + 2] = out + total;
    if (total == 0) return;                              // uniform
    int32_t* __restrict__ nodes = rg_nodes(S, g) + out;
    const bool in_lds = total <= kEmitIds;
    const int32_t first_id = (int32_t)((int64_t)blk * WORDS * 32);
#pragma unroll
    for (int q = 0; q < W; ++q) rg_put_ids<EmitId<W>>(bits[q], (int)threadIdx.x * W + q, in_lds, ids, nodes, first_id, j);
    __syncthreads();                                     // ids, nodes and edges are there
    rg_new_rows<T, true, EmitId<W>>(row_ptr, S, g, hop, out, total, nodes, ids, first_id, in_lds, edges, num_chunks, next_fanout);
}

__global__ void __launch_bounds__(kTierWords / 3) k_tier_emit(const RowPtr row_ptr, const SampleScratch S, int hop, unsigned tier_blocks,
                                                              int next_fanout, int run, int scanned) {
    rg_tier_emit<kTierWords / 3, kTierWords, false>(row_ptr, S, hop, tier_blocks, next_fanout, run, scanned, S.visited, S.visited, nullptr);
}
__global__ void __launch_bounds__(kEmitThreadsSmall) k_tier_emit_small(const RowPtr row_ptr, const SampleScratch S, int hop, unsigned tier_blocks,
                                                                       int next_fanout, int run, int scanned) {
    rg_tier_emit<kEmitThreadsSmall, kTierWordsSmall, false>(row_ptr, S, hop, tier_blocks, next_fanout, run, scanned, S.visited, S.visited, nullptr);
}
__global__ void __launch_bounds__(kEmitThreadsSmall) k_bytes_emit_small(const RowPtr row_ptr, const SampleScratch S, int hop, unsigned tier_blocks,
                                                                        int next_fanout, int run, const uint32_t* before, uint32_t* after, uint8_t* next_bytes) {
    rg_tier_emit<kEmitThreadsSmall, kTierWordsSmall, true>(row_ptr, S, hop, tier_blocks, next_fanout, run, 0, before, after, next_bytes);
}

// ---------------------------------------------------------------------------- per hop: new tier in first-seen order
// Edge e opens a new node when it is the first edge of the hop naming a node outside the frontier.  Ordered
// compaction over the hop's edge list: counts per kEdgesPerBlock edges, the scan of k_scan_tier, then the emit below.
constexpr int kEdgesPerBlock = 1024;   // 256 threads x 4 consecutive edges

// Which of a thread's 4 edges from e0 on open a node; their ids.
__device__ __forceinline__ uint32_t rg_opens_nodes(const int32_t* __restrict__ nbr, const int32_t* __restrict__ first_key, int64_t e0, int64_t n_edges,
                                                   int32_t (&u)[4]) {
    int32_t key[4];
    uint32_t opens = 0u;
#pragma unroll
    for (int q = 0; q < 4; ++q) u[q] = e0 + q < n_edges ? nbr[e0 + q] : -1;
#pragma unroll
    for (int q = 0; q < 4; ++q) key[q] = u[q] >= 0 ? first_key[u[q]] : 0;                // (no edge has the key 0)
#pragma unroll
    for (int q = 0; q < 4; ++q) opens |= (uint32_t)(key[q] == 0x7FFFFFFF - (int32_t)(e0 + q)) << q;
    return opens;
}

__global__ void __launch_bounds__(256) k_first_seen_count(const SampleScratch S, int hop) {
    const int g = rg_batch(S);
    const unsigned blk = rg_block(S);
    const int32_t* __restrict__ nbr = rg_hop_list(S, g, (int)hop, kNbr);
    const int32_t* __restrict__ first_key = S.first_key + g * S.num_nodes;
    const int64_t n_edges = rg_hop_list(S, g, (int)hop, kIndptr)[rg_tier_off(S, g)[hop + 1]];
    __shared__ int part[4];
    int64_t chunk = blk;
    do {                                                           // (a workgroup without an edge writes a zero)
        int32_t u[4];
        int c = __popc(rg_opens_nodes(nbr, first_key, chunk * kEdgesPerBlock + threadIdx.x * 4, n_edges, u));
        c = rg_wave_sum(c);
        __syncthreads();                                           // part[] of the chunk before has been read
        if (rg_lane() == 0) part[threadIdx.x >> 6] = c;
        __syncthreads();
        if (threadIdx.x == 0) S.chunk_sum[g * S.chunk_stride + chunk] = part[0] + part[1] + part[2] + part[3];
        chunk += rg_blocks_per_batch(S);
    } while (chunk * kEdgesPerBlock < n_edges);
}

// The row of a new node for the next hop, read while the workgroup's other new nodes' are, and its edges, which the caller adds up.
__device__ __forceinline__ int rg_put_row(const SampleScratch& S, int g, int at, int64_t start, int64_t deg, int next_fanout) {
    S.row_start[g * S.frontier_stride + at] = start;
    S.row_deg[g * S.frontier_stride + at] = (int32_t)deg;
    return (int)(deg <= next_fanout ? deg : next_fanout);
}

// Appends the opened nodes behind the current frontier in edge order, records their positions, marks them visited
// and clears their first-edge keys (the array is all-zero again when the hop is done).  next_fanout >= 0: also the next hop's sizes, as in
// rg_new_rows.  scanned: chunk_sum holds exclusive offsets, and the
// tier's end is known; else every workgroup adds up the counts in front of its own.
__global__ void __launch_bounds__(256) k_first_seen_emit(const RowPtr row_ptr, const SampleScratch S, int hop, int next_fanout, int scanned) {
    constexpr int NW = 256 / RG_WAVE;
    __shared__ int smem[NW + 1];
    __shared__ int part[NW];
    __shared__ int edges[2];
    const int g = rg_batch(S);
    const unsigned blk = rg_block(S);
    const unsigned edge_blocks = rg_blocks_per_batch(S);
    const int32_t* __restrict__ nbr = rg_hop_list(S, g, (int)hop, kNbr);
    int32_t* __restrict__ first_key = S.first_key + g * S.num_nodes;
    uint32_t* __restrict__ visited = S.visited + g * S.words;
    int32_t* __restrict__ nodes = rg_nodes(S, g);
    int32_t* __restrict__ pos = S.pos + g * S.num_nodes;
    const int32_t* __restrict__ chunk_sum = S.chunk_sum + g * S.chunk_stride;
    int32_t* __restrict__ next_sum = S.hop_sum[(hop + 1) & 1] + g * S.chunk_stride;
    const int n_h = rg_tier_off(S, g)[hop + 1];
    const int64_t n_edges = rg_hop_list(S, g, (int)hop, kIndptr)[n_h];
    if (!scanned && n_edges == 0 && blk == 0 && threadIdx.x == 0) rg_tier_off(S, g)[hop + 2] = n_h;
    if (next_fanout >= 0)                                          // (the last workgroups are the ones that may have no edges)
        for (int64_t chunk = edge_blocks - 1 - blk; chunk * kChunk < n_h; chunk += edge_blocks) rg_old_edges<256>(S, g, hop, (int)chunk, next_fanout);
    int64_t added = 0;                                             // chunks whose counts are in `before`
    int before = n_h;
    for (int64_t chunk = blk; chunk * kEdgesPerBlock < n_edges; chunk += edge_blocks) {
        int c = 0;
        if (!scanned) {
            for (int64_t b = added + threadIdx.x; b < chunk; b += 256) c += chunk_sum[b];
            added = chunk;
        } else {
            if (threadIdx.x == 0) c = chunk_sum[chunk];
            before = n_h;                                          // (by every thread: the rounds before have added theirs)
        }
        c = rg_wave_sum(c);
        __syncthreads();                                           // part[] and edges[] of the chunk before have been read
        if (rg_lane() == 0) part[threadIdx.x >> 6] = c;
        if (threadIdx.x < 2) edges[threadIdx.x] = 0;
        const int64_t e0 = chunk * kEdgesPerBlock + threadIdx.x * 4;
        int32_t u[4];
        const uint32_t opens = rg_opens_nodes(nbr, first_key, e0, n_edges, u);
        int total;
        const int excl = rg_block_excl_scan<NW>(__popc(opens), smem, &total);      // its barriers publish part[] and edges[]
#pragma unroll
        for (int q = 0; q < NW; ++q) before += part[q];
        if (!scanned && threadIdx.x == 0 && (chunk + 1) * kEdgesPerBlock >= n_edges) rg_tier_off(S, g)[hop + 2] = before + total;
        if (total == 0) continue;                                         // uniform
        int out = before + excl;
        int64_t start[4], deg[4];
        if (next_fanout >= 0) {
            const auto rows = [&](auto* p) {
#pragma unroll
                for (int q = 0; q < 4; ++q)
                    if ((opens >> q) & 1u) rg_row_extent(p, u[q], start[q], deg[q]);
            };
            if (row_ptr.wide) rows((const int64_t*)row_ptr.p); else rows((const int32_t*)row_ptr.p);
        }
#pragma unroll
        for (int q = 0; q < 4; ++q)
            if ((opens >> q) & 1u) {
                nodes[out] = u[q];
                pos[u[q]] = out;
                atomicOr(&visited[(uint32_t)u[q] >> 5], 1u << (u[q] & 31));
                first_key[u[q]] = 0;                  // only the opening edge's thread touches this entry now
                if (next_fanout >= 0) atomicAdd(&edges[out / kChunk - before / kChunk], rg_put_row(S, g, out, start[q], deg[q], next_fanout));
                ++out;
            }
        if (next_fanout < 0) continue;
        __syncthreads();
        if (threadIdx.x < 2 && edges[threadIdx.x]) atomicAdd(&next_sum[before / kChunk + threadIdx.x], edges[threadIdx.x]);
    }
}

// ---------------------------------------------------------------------------- per hop: first-seen order by rank blocks
// The bases of a batch's tiers, [hop][rank_bases], into LDS.
__device__ __forceinline__ void rg_load_bases(const SampleScratch& S, int g, int hops, int32_t* bases) {
    const int n = (int)S.rank_bases;
    for (int hop = 0; hop < hops; ++hop) {
        const int32_t* __restrict__ from = rg_rank_bases(S, g, hop);
        for (int i = threadIdx.x; i < n; i += blockDim.x) bases[hop * n + i] = from[i];
    }
    __syncthreads();
}

// Positions of U ids (-1: none) from the rank blocks of the hops' tiers, latest first, and from pos[] for the seeds; the U reads of
// a step are in flight together.
template <int U>
__device__ __forceinline__ void rg_ranked_positions(const int32_t (&u)[U], const SampleScratch& S, int g, int hop,
                                                    const int32_t* __restrict__ pos, const int32_t* bases, int32_t (&r)[U]) {
    uint32_t at[U], bit[U][2], below[U][2];              // the id's rank block, its bit there and the bits below it
    const int nb = (int)S.rank_bases;
#pragma unroll
    for (int q = 0; q < U; ++q) {
        r[q] = u[q] >= 0 ? -1 : 0;
        at[q] = (uint32_t)u[q] / (uint32_t)kRankIds;
        const uint32_t in = (uint32_t)u[q] - at[q] * (uint32_t)kRankIds, b = 1u << (in & 31u);
        bit[q][0] = in < 32u ? b : 0u;
        bit[q][1] = in < 32u ? 0u : b;
        below[q][0] = bit[q][0] - 1u;                    // (all ones where the bit is in the upper word)
        below[q][1] = in < 32u ? 0u : b - 1u;
    }
    for (int t = hop; t >= 0;) {                         // tiers t and below are left
        const int d = S.hops - 1 - t;
        const char* __restrict__ rank = (const char*)rg_rank_pair(S, g, d >> 1);
        bool open = false;
        if (t == 0 && (d & 1) == 0) {
            uint2 x[U];
#pragma unroll
            for (int q = 0; q < U; ++q) x[q] = r[q] < 0 ? *(const uint2*)(rank + at[q] * 8u) : make_uint2(0u, 0u);
#pragma unroll
            for (int q = 0; q < U; ++q) {
                if ((x[q].x & bit[q][0]) | (x[q].y & bit[q][1]))
                    r[q] = bases[at[q] >> 10] + (int)(x[q].y >> 16) + __popc(x[q].x & below[q][0]) + __popc(x[q].y & below[q][1]);
                open = open || r[q] < 0;
            }
            t = -1;
        } else {
            const uint32_t ask = d & 1 ? 0u : ~0u;       // the later tier of the pair is not there yet in front of its hop
            const int earlier = d & 1 ? t : t - 1;
            uint4 x[U];
#pragma unroll
            for (int q = 0; q < U; ++q) x[q] = r[q] < 0 ? *(const uint4*)(rank + at[q] * 16u) : make_uint4(0u, 0u, 0u, 0u);
#pragma unroll
            for (int q = 0; q < U; ++q) {
                const bool late = (((x[q].x & bit[q][0]) | (x[q].y & bit[q][1])) & ask) != 0u;
                const uint32_t lo = late ? x[q].x : x[q].z, hi = late ? x[q].y : x[q].w;
                if ((lo & bit[q][0]) | (hi & bit[q][1]))
                    r[q] = bases[(late ? earlier + 1 : earlier) * nb + (int)(at[q] >> 10)] + (int)(hi >> 16) + __popc(lo & below[q][0]) +
                           __popc(hi & below[q][1]);
                open = open || r[q] < 0;
            }
            t = earlier - 1;
        }
        if (!__any(open)) return;
    }
#pragma unroll
    for (int q = 0; q < U; ++q)
        if (r[q] < 0) r[q] = pos[u[q]];
}

// nbr_local[e] = ascending position of nbr[e].
__global__ void __launch_bounds__(256) k_seen_rank(const SampleScratch S, int hop) {
    extern __shared__ int32_t bases[];
    constexpr int U = 2;
    const int g = rg_batch(S);
    rg_load_bases(S, g, hop + 1, bases);
    const int64_t stride = (int64_t)rg_blocks_per_batch(S) * 256;
    const int64_t n = rg_hop_list(S, g, (int)hop, kIndptr)[rg_tier_off(S, g)[hop + 1]];
    const int32_t* __restrict__ nbr = rg_hop_list(S, g, (int)hop, kNbr);
    const int32_t* __restrict__ pos = S.pos + g * S.num_nodes;
    int32_t* __restrict__ nbr_local = rg_hop_list(S, g, (int)hop, kNbrLocal);
    for (int64_t e0 = (int64_t)rg_block(S) * 256 + threadIdx.x; e0 < n; e0 += stride * U) {
        int32_t u[U], r[U];
#pragma unroll
        for (int q = 0; q < U; ++q) u[q] = e0 + stride * q < n ? nbr[e0 + stride * q] : -1;
        rg_ranked_positions<U>(u, S, g, hop, pos, bases, r);
#pragma unroll
        for (int q = 0; q < U; ++q)
            if (u[q] >= 0) nbr_local[e0 + stride * q] = r[q];
    }
}

// first_edge[position] = the first edge of the hop that names the new node.  A workgroup owns kSeenSlice of the new positions in
// LDS and reads every edge's position.  With one global atomicMin per edge behind a read (the positions in 1.1 MB per batch) hop 2
// of 8 batches of 1024 seeds, 4.6 M edges, took 180 us.  Cutting the edges into parts as well, with a bitmap of the positions that each part names,
// is no faster (4 to 16 parts 40 + 7 us against 34): clearing and reading out the slices then take the time.
constexpr int kSeenSlice = 40000;
__device__ __forceinline__ void rg_seen_min(int32_t* first, int32_t a, int64_t e, uint32_t a0, uint32_t n) {
    const uint32_t d = (uint32_t)a - a0;
    if (d < n) atomicMin(&first[d], (int32_t)e);
}

__global__ void __launch_bounds__(1024) k_seen_min(const SampleScratch S, int hop) {
    extern __shared__ int32_t slice_first[];
    constexpr int U = 4;                                 // 16-byte loads in flight per thread
    const int g = rg_batch(S);
    const int n_h = rg_tier_off(S, g)[hop + 1];
    const int64_t a0 = n_h + (int64_t)rg_block(S) * kSeenSlice, left = rg_tier_off(S, g)[hop + 2] - a0;
    if (left <= 0) return;                               // uniform per workgroup
    const int n_here = (int)(left < kSeenSlice ? left : kSeenSlice);
    for (int i = threadIdx.x; i < n_here; i += 1024) slice_first[i] = 0x7FFFFFFF;
    const int n = rg_hop_list(S, g, (int)hop, kIndptr)[n_h];
    const int32_t* __restrict__ at = rg_hop_list(S, g, (int)hop, kNbrLocal);
    __syncthreads();
    const int to_line = (int)((16u - ((uint32_t)(uintptr_t)at & 15u)) & 15u) / 4;      // at[] may start at any 4-byte address
    const int head = to_line < n ? to_line : n;
    const int n4 = (n - head) / 4;
    const int4* __restrict__ body = (const int4*)(at + head);
    for (int i = threadIdx.x; i < n4; i += U * 1024) {
        int4 x[U];
#pragma unroll
        for (int q = 0; q < U; ++q) x[q] = body[i + q * 1024 < n4 ? i + q * 1024 : i];
#pragma unroll
        for (int q = 0; q < U; ++q) {
            if (i + q * 1024 >= n4) break;
            const int e = head + 4 * (i + q * 1024);
            rg_seen_min(slice_first, x[q].x, e, (uint32_t)a0, (uint32_t)n_here);
            rg_seen_min(slice_first, x[q].y, e + 1, (uint32_t)a0, (uint32_t)n_here);
            rg_seen_min(slice_first, x[q].z, e + 2, (uint32_t)a0, (uint32_t)n_here);
            rg_seen_min(slice_first, x[q].w, e + 3, (uint32_t)a0, (uint32_t)n_here);
        }
    }
    const int tail = head + 4 * n4;
    if ((int)threadIdx.x < head) rg_seen_min(slice_first, at[threadIdx.x], threadIdx.x, (uint32_t)a0, (uint32_t)n_here);
    if ((int)threadIdx.x < n - tail) rg_seen_min(slice_first, at[tail + threadIdx.x], tail + threadIdx.x, (uint32_t)a0, (uint32_t)n_here);
    __syncthreads();
    int32_t* __restrict__ out = S.first_edge + g * S.frontier_stride + a0;
    for (int i = threadIdx.x; i < n_here; i += 1024) out[i] = slice_first[i];
}

constexpr int kSeenEdges = 4096;       // edges per workgroup of the count and the emit: 1024 threads x 4
constexpr uint32_t kOpens = 0x80000000u;         // in nbr_local, from the count to the relabelling: the edge opens a node

// The edges that open a node, marked in nbr_local, where the emit meets them (looking their first edges up again it took 32 us at that hop,
// now 25), and their number per workgroup.

__global__ void __launch_bounds__(1024) k_seen_count(const SampleScratch S, int hop) {
    __shared__ int part[1024 / RG_WAVE];
    const int g = rg_batch(S);
    const unsigned blk = rg_block(S);
    const int n_h = rg_tier_off(S, g)[hop + 1];
    const int64_t n = rg_hop_list(S, g, (int)hop, kIndptr)[n_h], first = (int64_t)blk * kSeenEdges;
    if (first >= n) return;                              // uniform per workgroup
    int32_t* __restrict__ at = rg_hop_list(S, g, (int)hop, kNbrLocal) + first;
    const int32_t* __restrict__ first_edge = S.first_edge + g * S.frontier_stride;
    int c = 0;
    int32_t a[4], f[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) a[q] = first + q * 1024 + threadIdx.x < n ? at[q * 1024 + threadIdx.x] : -1;
#pragma unroll
    for (int q = 0; q < 4; ++q) f[q] = a[q] >= n_h ? first_edge[a[q]] : -1;
#pragma unroll
    for (int q = 0; q < 4; ++q)
        if (f[q] == (int32_t)(first + q * 1024 + threadIdx.x)) {
            ++c;
            at[q * 1024 + threadIdx.x] = (int32_t)((uint32_t)a[q] | kOpens);
        }
    c = rg_wave_sum(c);
    if (rg_lane() == 0) part[threadIdx.x >> 6] = c;
    __syncthreads();
    if (threadIdx.x < RG_WAVE) {
        c = rg_wave_sum(threadIdx.x < 1024 / RG_WAVE ? part[threadIdx.x] : 0);
        if (threadIdx.x == 0) S.chunk_sum[g * S.chunk_stride + blk] = c;
    }
}

// The nodes that edges open, in edge order, and where each ascending position ended up; edge_blocks workgroups per batch.  next_fanout >= 0:
// also the next hop's sizes, as in rg_new_rows, those of the nodes in front of the tier by the workgroups behind.
__global__ void __launch_bounds__(1024) k_seen_emit(const RowPtr row_ptr, const SampleScratch S, int hop, unsigned edge_blocks, int next_fanout) {
    constexpr int NW = 1024 / RG_WAVE;
    __shared__ int smem[NW + 1];
    __shared__ int part[NW];
    __shared__ int edges[kSeenEdges / kChunk + 2];
    const int g = rg_batch(S);
    const unsigned blk = rg_block(S);
    if (blk >= edge_blocks) {
        rg_old_edges<1024>(S, g, hop, (int)(blk - edge_blocks), next_fanout);
        return;
    }
    const int n_h = rg_tier_off(S, g)[hop + 1];
    const int64_t n = rg_hop_list(S, g, (int)hop, kIndptr)[n_h], first = (int64_t)blk * kSeenEdges;
    if (first >= n) return;                              // uniform per workgroup
    const int32_t* __restrict__ at = rg_hop_list(S, g, (int)hop, kNbrLocal);
    const int32_t* __restrict__ nbr = rg_hop_list(S, g, (int)hop, kNbr);
    const int32_t* __restrict__ chunk_sum = S.chunk_sum + g * S.chunk_stride;
    int before = 0;                                      // nodes opened by the edges in front of this workgroup's
    for (unsigned c = threadIdx.x; c < blk; c += 1024) before += chunk_sum[c];
    before = rg_wave_sum(before);
    if (rg_lane() == 0) part[threadIdx.x >> 6] = before;
    if (threadIdx.x < sizeof(edges) / sizeof(int)) edges[threadIdx.x] = 0;
    const int64_t e0 = first + threadIdx.x * 4;
    int32_t a[4], u[4];
    uint32_t opens = 0u;
#pragma unroll
    for (int q = 0; q < 4; ++q) a[q] = e0 + q < n ? at[e0 + q] : 0;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        u[q] = -1;
        if (a[q] < 0) { u[q] = nbr[e0 + q]; opens |= 1u << q; }
    }
    int total;
    int out = n_h + rg_block_excl_scan<NW>(__popc(opens), smem, &total);   // its barriers publish part[] and edges[]
    before = n_h;
#pragma unroll
    for (int q = 0; q < NW; ++q) { out += part[q]; before += part[q]; }
    int64_t start[4], deg[4];
    if (next_fanout >= 0) {
        const auto rows = [&](auto* p) {
#pragma unroll
            for (int q = 0; q < 4; ++q)
                if ((opens >> q) & 1u) rg_row_extent(p, u[q], start[q], deg[q]);
        };
        if (row_ptr.wide) rows((const int64_t*)row_ptr.p); else rows((const int32_t*)row_ptr.p);
    }
    int32_t* __restrict__ nodes = rg_nodes(S, g);
    int32_t* __restrict__ place = S.place + g * S.frontier_stride;
    const int chunk0 = out / kChunk - before / kChunk;
    int in_first = 0, in_next = 0;                       // edges of this thread's nodes in the chunk of the first of them, and in the one behind
#pragma unroll
    for (int q = 0; q < 4; ++q)
        if ((opens >> q) & 1u) {
            nodes[out] = u[q];
            place[(uint32_t)a[q] & ~kOpens] = out;
            if (next_fanout >= 0) {
                const int m = rg_put_row(S, g, out, start[q], deg[q], next_fanout);
                if (out / kChunk - before / kChunk == chunk0) in_first += m; else in_next += m;
            }
            ++out;
        }
    if (next_fanout < 0) return;
    // one addition for a wavefront whose nodes share a chunk: lanes that add to one address queue up
    const int lead = __builtin_amdgcn_readfirstlane(chunk0);
    if (__all(chunk0 == lead && in_next == 0)) {
        in_first = rg_wave_sum(in_first);
        if (rg_lane() == 0 && in_first) atomicAdd(&edges[lead], in_first);
    } else {
        if (in_first) atomicAdd(&edges[chunk0], in_first);
        if (in_next) atomicAdd(&edges[chunk0 + 1], in_next);
    }
    __syncthreads();
    if (threadIdx.x < sizeof(edges) / sizeof(int) && edges[threadIdx.x])
        atomicAdd(&S.hop_sum[(hop + 1) & 1][g * S.chunk_stride + before / kChunk + threadIdx.x], edges[threadIdx.x]);
}

// ---------------------------------------------------------------------------- relabelling, all hops in one launch
// A member's position never changes, so nbr_local of every hop can be written after the last one, if every hop's lists are still
// there by then (rg_hops_share_buffers).
// nbr_local[e] = position of nbr[e] in the extended frontier; the hop's edge count is indptr[n_h].
// RANKED: the rank blocks of the tiers, latest first, pos[] for the seeds.  N / 3 bytes for two tiers (3.3 MB at N = 10 M) where pos[]
// is 4 N.  Three hops of 8 batches of 4096 seeds, 20.6 M edges: 148 us, bound by random reads of L2, 25.6 M of them (a quarter of the edges
// name the first tier, whose blocks are a second read; 3.6 M miss).  With 8 bytes per 32 ids and tier, 32 M reads of which 9.2 M
// missed, 200; with 16 bytes per 96 ids and tier, 32 M and 3.4 M, 186.  Two edges in flight per thread: four take 85 registers and 6 us more.
template <bool RANKED>
__global__ void __launch_bounds__(256) k_relabel(const SampleScratch S, int first_hop, int last_hop) {
    extern __shared__ int32_t bases[];
    constexpr int U = RANKED ? 2 : 4;                    // edges in flight per thread
    const int g = rg_batch(S);
    const int64_t stride = (int64_t)rg_blocks_per_batch(S) * 256;
    const int32_t* __restrict__ pos = S.pos + g * S.num_nodes;
    if (RANKED) rg_load_bases(S, g, last_hop + 1, bases);
    for (int hop = last_hop; hop >= first_hop; --hop) {
        int32_t* __restrict__ nbr_local = rg_hop_list(S, g, hop, kNbrLocal);
        if (!nbr_local) continue;
        const int32_t* __restrict__ nbr = rg_hop_list(S, g, hop, kNbr);
        const int64_t n = rg_hop_list(S, g, hop, kIndptr)[rg_tier_off(S, g)[hop + 1]];
        for (int64_t e0 = (int64_t)rg_block(S) * 256 + threadIdx.x; e0 < n; e0 += stride * U) {
            int32_t u[U], r[U];
#pragma unroll
            for (int q = 0; q < U; ++q) u[q] = e0 + stride * q < n ? nbr[e0 + stride * q] : -1;
            if (RANKED) {
                rg_ranked_positions<U>(u, S, g, hop, pos, bases, r);
            } else {
#pragma unroll
                for (int q = 0; q < U; ++q) r[q] = u[q] >= 0 ? pos[u[q]] : 0;
            }
#pragma unroll
            for (int q = 0; q < U; ++q)
                if (u[q] >= 0) __builtin_nontemporal_store(r[q], &nbr_local[e0 + stride * q]);
        }
    }
}

// ---------------------------------------------------------------------------- small batches, one launch
// All hops of a small batch by one workgroup: the membership bits and the hop's marks are in LDS, the phases are separated by
// barriers instead of launches (12 launches for two hops, each bound by its own latency).  A thread draws for one frontier
// node and has all its picks' col_idx reads in flight.  One launch against one per phase, by nodes and the bound on a batch's
// edges, (10,5) on graphs of 20 / 50 / 400 neighbours per node on average, of power-law degrees: 100 k nodes 8 k edges 23 / 28 / 30 us
// against 45, 16 k 34 / 43 / 53 against 46, 20 k 40 / 51 / 68 against 46, of 16 batches 28 / 31 / 38 against 46, 40 / 59 / 71 against 49 and
// 49 / 73 / 85 against 49 (of eight as of one, on as many compute units); 500 k nodes 8 k 30 / 35 / 37 against 48, of 16 batches 37 / 47 / 52
// against 50.  A hop more is 17 us for the launches, and little here: (10,10,10) 20 k 39 / 56 / 70 against 63.  So the lines suit graphs many of
// whose nodes have fewer neighbours than are drawn; where nearly all have more, and the bound's edges come, calls just below them lose.
// The frontiers' nodes count like edges: there may be more of them where a fan-out is 0 or the graph has few edges (500 k seeds 1320-1370 /
// 73-124 us).  Larger fan-outs take longer above 65,536 nodes: (25,10) on 100 k nodes 12 k 29 / 38 / 49 against 45, 20 k 34 / 53 / 72 against 46.
// On graphs of 70 neighbours per node or more, whose batches bring nearly the bound's edges, and where the lists don't fit LDS, the launches of the
// byte tiers are faster from 10,500 edges (two hops) on: eight batches of 18.5 k edges on 77 k nodes of 377 neighbours 62 / 34 us, two of 16.9 k on 86 k
// 54 / 36, one of 13.7 k on 125 k 46 / 37, of 10.1 k on 67 k 40 / 35, of 8 k on 88 k 27 / 35; three hops 17.7 k 59 / 49, 12.4 k 48 / 46, 9.4 k 38 / 46.
constexpr int64_t kSmallNodes = 512 * 1024;     // two bitmaps of 64 KB
constexpr int64_t kSmallDense = 70;
inline bool rg_is_small(int64_t num_nodes, int64_t num_edges, int hops, bool in_lds, int64_t edges_bound, int64_t frontiers_bound) {
    const bool few = !in_lds && num_edges >= kSmallDense * num_nodes;
    return num_nodes > 0 && num_nodes <= kSmallNodes &&
           rg_max64(edges_bound, frontiers_bound) <= (num_nodes > 128 * 1024 ? 8 * 1024 : few ? 8500 + 1000 * hops : 20 * 1024);
}

struct Fanouts {
    int32_t v[RG_MAX_HOPS];
};

// Picks whose columns a thread has on their way: all of them, but with KMAX = 32 eight.  1024 threads have 128 registers each, and with 32 on
// their way, and the first Philox round in vector registers, 42 to 47 did not fit and went to scratch memory: (25,10) on 366 k nodes 47 us, on
// 30,000 31, now (5 to 10 registers) 41 and 24; (32,16) on 30,000 36 and 27.
constexpr int rg_small_reads(int kmax) { return kmax > 16 ? 8 : kmax; }

// Floyd's picks for one node, all in registers (whole row: its places in order).
template <int KMAX>
__device__ __forceinline__ void rg_draw(int32_t v, int64_t deg, int k, uint32_t hop, uint32_t k0, uint32_t k1, uint32_t epoch, uint32_t (&c)[KMAX]) {
    if (deg <= k) {
#pragma unroll
        for (int s = 0; s < KMAX; ++s) c[s] = (uint32_t)s;             // whole row, CSR order
        return;
    }
#pragma unroll
    for (int blk = 0; blk < KMAX / 4; ++blk) {
        if (blk * 4 < k) {
            uint32_t w[4];
            rg_philox4x32_10<(KMAX > 16)>((uint32_t)v, hop, (uint32_t)blk, epoch, k0, k1, w);
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const int s = blk * 4 + q;
                if (s < k) {                                           // Floyd: j = d-k+s, t uniform in [0, j]
                    const uint32_t j = (uint32_t)(deg - k + s);
                    const uint32_t t = __umulhi(w[q], j + 1u);
                    bool found = false;
#pragma unroll
                    for (int l = 0; l < s; ++l) found |= (c[l] == t);
                    c[s] = found ? j : t;
                }
            }
        }
    }
}

template <typename RP, int KMAX, int N>
__global__ void __launch_bounds__(1024) k_sample_small(const RP* __restrict__ row_ptr, const int32_t* __restrict__ col_idx, const BatchTable<N> B, int group, const Fanouts fanouts,
                                                       uint32_t* __restrict__ visited_out, int64_t words64, int32_t* pos_all, int64_t num_nodes,
                                                       int hops, uint32_t k0, uint32_t k1, uint32_t epoch) {
    extern __shared__ uint32_t small_bits[];
    __shared__ int smem[1024 / RG_WAVE + 1];
    const int g = blockIdx.x, words = (int)words64;
    uint32_t* visited = small_bits;
    uint32_t* marked = small_bits + words;                             // members and the ids the hop has sampled
    const auto entry = [&](int field) { return rg_global(B.v[field * group + g]); };
    const int32_t* seeds = entry(kSeeds);
    int32_t* nodes = entry(kNodes);
    int32_t* tier_off = entry(kTierOff);
    int32_t* edges_out = entry(kEdgesOut);
    int32_t* pos = pos_all + g * num_nodes;
    for (int w = threadIdx.x; w < 2 * words; w += 1024) small_bits[w] = 0u;
    int n_h = (int)B.v[kNumSeeds * group + g];
    __syncthreads();
    for (int i = threadIdx.x; i < n_h; i += 1024) {
        const int32_t v = seeds[i];
        nodes[i] = v;
        pos[v] = i;
        atomicOr(&visited[(uint32_t)v >> 5], 1u << (v & 31));
        atomicOr(&marked[(uint32_t)v >> 5], 1u << (v & 31));
    }
    if (threadIdx.x == 0) { tier_off[0] = 0; tier_off[1] = n_h; }
    const int per = (words + 1023) / 1024 | 1;                         // consecutive bitmap words per thread, odd: no two lanes on a bank
    const int w0 = (int)threadIdx.x * per, w1 = w0 + per < words ? w0 + per : words;
    for (int hop = 0; hop < hops; ++hop) {
        const int k = fanouts.v[hop];
        int32_t* indptr = entry(kHopFields + kHopFieldCount * hop + kIndptr);
        int32_t* nbr = entry(kHopFields + kHopFieldCount * hop + kNbr);
        int edges = 0;
        __syncthreads();                                               // nodes[] and the bits are complete
        for (int i0 = 0; i0 < n_h; i0 += 1024) {
            const int i = i0 + (int)threadIdx.x;
            int32_t v = 0;
            int64_t start = 0, deg = 0;
            int m = 0;
            if (i < n_h) {
                v = nodes[i];
                rg_row_extent(row_ptr, v, start, deg);
                m = deg <= k ? (int)deg : k;
            }
            int total;
            const int at = edges + rg_block_excl_scan<1024 / RG_WAVE>(m, smem, &total);
            edges += total;
            if (i >= n_h) continue;
            indptr[i] = at;
            uint32_t c[KMAX];
            rg_draw<KMAX>(v, deg, k, (uint32_t)hop, k0, k1, epoch, c);
            constexpr int U = rg_small_reads(KMAX);
#pragma unroll
            for (int s0 = 0; s0 < KMAX; s0 += U) {
                int32_t u[U];
                if (s0) __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                for (int s = 0; s < U; ++s)
                    if (s0 + s < m) u[s] = col_idx[start + (int64_t)c[s0 + s]];
#pragma unroll
                for (int s = 0; s < U; ++s)
                    if (s0 + s < m) {
                        nbr[at + s0 + s] = u[s];
                        atomicOr(&marked[(uint32_t)u[s] >> 5], 1u << (u[s] & 31));
                    }
            }
        }
        if (threadIdx.x == 0) {
            indptr[n_h] = edges;
            if (edges_out) edges_out[hop] = edges;
        }
        __syncthreads();                                               // the marks and nbr[] are complete
        int fresh = 0;
        for (int w = w0; w < w1; ++w) fresh += __popc(marked[w] & ~visited[w]);
        int total;
        int out = n_h + rg_block_excl_scan<1024 / RG_WAVE>(fresh, smem, &total);
        for (int w = w0; w < w1; ++w) {
            uint32_t b = marked[w] & ~visited[w];
            if (b == 0u) continue;
            visited[w] |= b;
            for (; b; b &= b - 1u) {
                const int32_t id = (w << 5) + __ffs(b) - 1;
                nodes[out] = id;
                pos[id] = out++;
            }
        }
        n_h += total;
        if (threadIdx.x == 0) tier_off[hop + 2] = n_h;
        int32_t* nbr_local = entry(kHopFields + kHopFieldCount * hop + kNbrLocal);
        if (nbr_local) {                                               // uniform
            __syncthreads();                                           // pos[] is complete
            for (int e0 = threadIdx.x; e0 < edges; e0 += 4096) {
                int32_t u[4];
#pragma unroll
                for (int q = 0; q < 4; ++q) u[q] = e0 + 1024 * q < edges ? nbr[e0 + 1024 * q] : -1;
#pragma unroll
                for (int q = 0; q < 4; ++q)
                    if (u[q] >= 0) u[q] = pos[u[q]];
#pragma unroll
                for (int q = 0; q < 4; ++q)
                    if (e0 + 1024 * q < edges) nbr_local[e0 + 1024 * q] = u[q];
            }
        }
    }
    __syncthreads();
    for (int w = threadIdx.x; w < words; w += 1024) visited_out[g * words64 + w] = visited[w];
}

// A barrier for what is in LDS: global stores and loads stay in flight across it.
__device__ __forceinline__ void rg_lds_barrier() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}
// rg_block_excl_scan over 16 wavefronts with such barriers.
__device__ __forceinline__ int rg_lds_excl_scan(int x, int* smem, int* total) {
    const int wave = threadIdx.x >> 6, incl = rg_wave_incl_scan(x);
    rg_lds_barrier();
    if (rg_lane() == RG_WAVE - 1) smem[wave] = incl;
    rg_lds_barrier();
    int base = 0, tot = 0;
#pragma unroll
    for (int w = 0; w < 1024 / RG_WAVE; ++w) {
        if (w < wave) base += smem[w];
        tot += smem[w];
    }
    *total = tot;
    return base + incl - x;
}

// Graphs and batches whose lists fit LDS as 16-bit numbers: positions, a hop's edges and the frontier, of which keep_hops tiers are kept:
// the last one, which is not drawn for, only where there is room.  Nothing is then read back
// from memory, the lists are written by consecutive lanes, and the only waits are for the rows and columns; the rows of a
// round's nodes are on their way while the round before is drawn for.  The barriers order what is in LDS only, but for the one that a hop
// begins with: hops may share their lists, and the offset behind the last node is stored by thread 0 in its hop and by another one in the
// next (any other entry by the same thread in every hop).  It takes no wait for the stores: those of one workgroup reach the
// cache of its compute unit in order.  nbr and nbr_local of a hop may be one list: the second store is the later one.
// 256 seeds (10,5) on 10,000 nodes 25.6 -> 17.8 us, 8 x 300 on 30,000 37.6 -> 24.6.
inline int64_t rg_small_lists_bytes(int64_t num_nodes, int64_t frontier, int64_t edges) {
    return 2 * rg_div_up(num_nodes, 32) * 4 + 2 * (num_nodes + frontier + edges) + 8;
}
constexpr int64_t kSmallLds = 160 * 1024 - 512;
// Whose lists fit: by edges up to which one launch is the faster way.  Its time grows with the edges, that of a launch per phase with
// the hops.  Just below the line, on graphs of 20 / 50 / 400 neighbours as above: (10,5) on 10,000 nodes 22 / 24 / 33 us against 46, on 30,000
// 24 / 28 / 45 against 46, (16,8) on 40,000 24 / 32 / 47 against 47, (10,10,10) on 30,000 29 / 39 / 67 against 64.
// The number of batches is left out: of 16 the same take 24 / 27 / 46, 27 / 32 / 53, 28 / 37 / 58 and 36 / 46 / 78 against 50, 50, 50
// and 66-75, so a lower line for them would win up to a tenth where all nodes have more neighbours than are drawn and lose up to half elsewhere.
// Fan-outs above 16 keep to rg_is_small, which was their line when they left registers in scratch memory (40-60 us at 26 k edges); since then
// (25,10) 26 k on 30,000 nodes takes 28 / 33 / 50 against 46, of 16 batches 31 / 37 / 62 against 46-52.
constexpr int64_t kSmallEdgesPerHop = 13500;
inline bool rg_small_lists_fit(int64_t num_nodes, int64_t frontier, int64_t hop_edges) {
    return num_nodes > 0 && num_nodes <= 65536 && rg_small_lists_bytes(num_nodes, frontier, hop_edges) <= kSmallLds;
}

template <typename RP, int KMAX, int N>
__global__ void __launch_bounds__(1024) k_sample_small_lists(const RP* __restrict__ row_ptr, const int32_t* __restrict__ col_idx,
                                                             const BatchTable<N> B, int group, const Fanouts fanouts,
                                                             uint32_t* __restrict__ visited_out, int64_t words64, int64_t num_nodes,
                                                             int frontier_most, int keep_hops, int hops, uint32_t k0, uint32_t k1,
                                                             uint32_t epoch) {
    extern __shared__ uint32_t small_bits[];
    __shared__ int smem[1024 / RG_WAVE + 1];
    const int g = blockIdx.x, words = (int)words64;
    uint32_t* visited = small_bits;
    uint32_t* marked = small_bits + words;                             // members and the ids the hop has sampled
    uint16_t* pos = (uint16_t*)(small_bits + 2 * words);
    uint16_t* front = pos + num_nodes;
    uint16_t* list = front + frontier_most;
    const auto entry = [&](int field) { return rg_global(B.v[field * group + g]); };
    const int32_t* __restrict__ seeds = entry(kSeeds);
    int32_t* __restrict__ nodes = entry(kNodes);
    int32_t* __restrict__ tier_off = entry(kTierOff);
    int32_t* __restrict__ edges_out = entry(kEdgesOut);
    for (int w = threadIdx.x; w < 2 * words; w += 1024) small_bits[w] = 0u;
    int n_h = (int)B.v[kNumSeeds * group + g];
    rg_lds_barrier();
    for (int i = threadIdx.x; i < n_h; i += 1024) {
        const int32_t v = seeds[i];
        nodes[i] = v;
        front[i] = (uint16_t)v;
        pos[v] = (uint16_t)i;
        atomicOr(&visited[(uint32_t)v >> 5], 1u << (v & 31));
        atomicOr(&marked[(uint32_t)v >> 5], 1u << (v & 31));
    }
    if (threadIdx.x == 0) { tier_off[0] = 0; tier_off[1] = n_h; }
    const int per = (words + 1023) / 1024 | 1;                         // consecutive bitmap words per thread, odd: no two lanes on a bank
    const int w0 = (int)threadIdx.x * per, w1 = w0 + per < words ? w0 + per : words;
    for (int hop = 0; hop < hops; ++hop) {
        const int k = fanouts.v[hop];
        int32_t* __restrict__ indptr = entry(kHopFields + kHopFieldCount * hop + kIndptr);
        int32_t* nbr = entry(kHopFields + kHopFieldCount * hop + kNbr);
        int32_t* nbr_local = entry(kHopFields + kHopFieldCount * hop + kNbrLocal);
        int edges = 0;
        __syncthreads();                                               // the frontier and the bits are complete, and the last hop's stores made
        int32_t v_next = 0;
        RP a_next = 0, b_next = 0;
        const auto rows_of = [&](int i) {
            if (i < n_h) {
                v_next = front[i];
                a_next = row_ptr[v_next];
                b_next = row_ptr[v_next + 1];
            }
        };
        rows_of((int)threadIdx.x);
        for (int i0 = 0; i0 < n_h; i0 += 1024) {
            const int i = i0 + (int)threadIdx.x;
            const int32_t v = v_next;
            const int64_t start = (int64_t)a_next, deg = i < n_h ? (int64_t)(b_next - a_next) : 0;
            rows_of(i + 1024);
            const int m = deg <= k ? (int)deg : k;
            int total;
            const int at = edges + rg_lds_excl_scan(m, smem, &total);
            edges += total;
            if (i >= n_h) continue;
            indptr[i] = at;
            uint32_t c[KMAX];
            rg_draw<KMAX>(v, deg, k, (uint32_t)hop, k0, k1, epoch, c);
            constexpr int U = rg_small_reads(KMAX);
#pragma unroll
            for (int s0 = 0; s0 < KMAX; s0 += U) {
                int32_t u[U];
                if (s0) __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                for (int s = 0; s < U; ++s)
                    if (s0 + s < m) u[s] = col_idx[start + (int64_t)c[s0 + s]];
#pragma unroll
                for (int s = 0; s < U; ++s)
                    if (s0 + s < m) {
                        list[at + s0 + s] = (uint16_t)u[s];
                        atomicOr(&marked[(uint32_t)u[s] >> 5], 1u << (u[s] & 31));
                    }
            }
        }
        if (threadIdx.x == 0) {
            indptr[n_h] = edges;
            if (edges_out) edges_out[hop] = edges;
        }
        rg_lds_barrier();                                              // the marks and the list are complete
        int fresh = 0;
        for (int w = w0; w < w1; ++w) fresh += __popc(marked[w] & ~visited[w]);
        int total;
        int out = n_h + rg_lds_excl_scan(fresh, smem, &total);
        for (int w = w0; w < w1; ++w) {
            uint32_t b = marked[w] & ~visited[w];
            if (b == 0u) continue;
            visited[w] |= b;
            for (; b; b &= b - 1u) {
                const int id = (w << 5) + __ffs(b) - 1;
                if (hop < keep_hops) front[out] = (uint16_t)id; else nodes[out] = id;
                pos[id] = (uint16_t)out++;
            }
        }
        rg_lds_barrier();                                              // the new tier is there
        if (hop < keep_hops)
            for (int i = n_h + (int)threadIdx.x; i < n_h + total; i += 1024) nodes[i] = front[i];
        n_h += total;
        if (threadIdx.x == 0) tier_off[hop + 2] = n_h;
        for (int e = threadIdx.x; e < edges; e += 1024) {
            const int id = list[e];
            nbr[e] = id;
            if (nbr_local) nbr_local[e] = pos[id];
        }
    }
    rg_lds_barrier();
    for (int w = threadIdx.x; w < words; w += 1024) visited_out[g * words64 + w] = visited[w];
}

// kTierRankedSeen: nbr_local holds ascending positions; the seeds' are their own.
__global__ void __launch_bounds__(256) k_seen_relabel(const SampleScratch S, int first_hop, int last_hop) {
    constexpr int U = 4;
    const int g = rg_batch(S);
    const int64_t stride = (int64_t)rg_blocks_per_batch(S) * 256;
    const int32_t* __restrict__ place = S.place + g * S.frontier_stride;
    const int seeds = rg_tier_off(S, g)[1];
    for (int hop = last_hop; hop >= first_hop; --hop) {
        int32_t* __restrict__ nbr_local = rg_hop_list(S, g, hop, kNbrLocal);
        if (!nbr_local) continue;
        const int64_t n = rg_hop_list(S, g, hop, kIndptr)[rg_tier_off(S, g)[hop + 1]];
        for (int64_t e0 = (int64_t)rg_block(S) * 256 + threadIdx.x; e0 < n; e0 += stride * U) {
            int32_t a[U];
#pragma unroll
            for (int q = 0; q < U; ++q) a[q] = e0 + stride * q < n ? nbr_local[e0 + stride * q] & (int32_t)~kOpens : -1;
#pragma unroll
            for (int q = 0; q < U; ++q)
                if (a[q] >= seeds) a[q] = place[a[q]];
#pragma unroll
            for (int q = 0; q < U; ++q)
                if (e0 + stride * q < n) nbr_local[e0 + stride * q] = a[q];
        }
    }
}

// Per-batch strides of the scratch slices for a graph of N nodes and frontiers of up to `frontier` nodes.
// max_edges: the largest per-hop edge bound when tiers are built from the edge list (first-seen order), else 0.
void sampler_scratch_shape(int64_t N, int64_t frontier, int64_t max_edges, SampleScratch& S) {
    S.words = rg_div_up(N, 32);
    S.rank_blocks = 2 * rg_div_up(S.words, 3);
    S.rank_bases = rg_div_up(N, kBaseIds);
    S.num_nodes = N;
    S.frontier_stride = rg_max64(frontier, 1);
    // (a quarter of a count chunk per entry leaves room for the first-seen blocks of up to four edges per frontier node)
    S.chunk_stride = rg_max64(rg_max64(rg_div_up(S.frontier_stride, kChunk / 4), rg_div_up(max_edges, kEdgesPerBlock)),
                              rg_max64(1, rg_div_up(S.words, kTierWordsSmall))) + 2;
    const int64_t slices = rg_max64(1, rg_div_up(S.words, kSliceWords));
    S.slices = slices <= kMaxSlices ? (int)slices : 0;       // 0: too large for the sliced marking
    S.slice_words = S.slices ? (int)rg_max64(1, rg_div_up(S.words, slices)) : 0;
    S.splits = 1;
    S.hops = 1;
    S.slice_marks = nullptr;
    S.rank[0] = S.rank[1] = nullptr;
    S.first_edge = S.place = S.first_key = nullptr;
    S.group = 1;
    S.group_inv = 0u;
    S.xcd_map = 1;
}

// ---------------------------------------------------------------------------- access counts straight from the bitmaps
// After the last hop a batch's `visited` bitmap is exactly its input-node set.  A wavefront takes 64 words of every batch of the group,
// a word per lane, and counts all 32 ids of a word at once in bit planes; then the lanes take the ids of two words at a time and
// add to counts[] (and lower first_batch[]), 64 consecutive counters to an instruction.  No id list is read.
// Other contexts may add to the same counts, so they are atomics, and bound by the lines they touch: with a thread per word, whose atomics
// went to 64 lines at a time, 8 batches of 2.4 M nodes took 45 us.
struct BatchIndices {
    uint32_t v[kMaxGroup];            // ascending
    uint8_t batch[kMaxGroup];         // of the group, in that order
};

// PARTS wavefronts share the counting of 64 words.  With first batches every two words are a read that is waited for, behind the additions
// in front of it, so on graphs of up to 4 Mi nodes eight do: 8 batches of 1024 seeds (15,10) on 1 M nodes 19.5 -> 8.2 us, on 2.4 M 20.0 -> 9.7,
// on 5 M 21.5 -> 15.6, but there 4 of 64 (10,5) 9.2 -> 10.3.  Without them nothing is waited for.
template <bool FIRST, int PARTS>
__global__ void __launch_bounds__(256) k_histogram_bitmaps(const uint32_t* __restrict__ visited, int64_t words, int group,
                                                           const BatchIndices order, uint32_t* __restrict__ counts,
                                                           uint32_t* __restrict__ first_batch, int64_t num_nodes) {
    constexpr int C = 5, F = 4;                       // planes: up to 16 batches, the ordinal of the first of them
    static_assert(kMaxGroup <= 16, "planes");
    const int lane = rg_lane();
    const int wave = blockIdx.x * 4 + (threadIdx.x >> 6);
    const int64_t w0 = (int64_t)(wave / PARTS) * RG_WAVE;
    const bool in = w0 + lane < words;
    uint32_t bits[kMaxGroup];
#pragma unroll
    for (int j = 0; j < kMaxGroup; ++j) bits[j] = j < group && in ? visited[(FIRST ? order.batch[j] : j) * words + w0 + lane] : 0u;
    uint32_t count[C] = {0u}, first[F] = {0u}, any = 0u;
#pragma unroll
    for (int j = 0; j < kMaxGroup; ++j) {
        uint32_t carry = bits[j];
        any |= carry;
#pragma unroll
        for (int k = 0; k < C; ++k) {
            const uint32_t x = count[k] & carry;
            count[k] ^= carry;
            carry = x;
        }
    }
    if (FIRST) {
#pragma unroll
        for (int j = kMaxGroup - 1; j >= 0; --j)
#pragma unroll
            for (int k = 0; k < F; ++k) first[k] = (j >> k) & 1 ? first[k] | bits[j] : first[k] & ~bits[j];
    }
    const unsigned long long named = __ballot(any != 0u);
    const int bit = lane & 31;
    for (int pair = 0; pair < RG_WAVE / 2 / PARTS; ++pair) {
        const int w = 2 * (PARTS == 1 ? pair : pair * PARTS + __builtin_amdgcn_readfirstlane(wave % PARTS));
        if (((named >> w) & 3ull) == 0ull) continue;                      // uniform
        const int from = w + (lane >> 5);
        uint32_t c = 0u, f = 0u;
#pragma unroll
        for (int k = 0; k < C; ++k) c |= (((uint32_t)__shfl((int)count[k], from, RG_WAVE) >> bit) & 1u) << k;
        if (FIRST) {
#pragma unroll
            for (int k = 0; k < F; ++k) f |= (((uint32_t)__shfl((int)first[k], from, RG_WAVE) >> bit) & 1u) << k;
        }
        const int64_t v = ((w0 + from) << 5) + bit;
        if (c == 0u || v >= num_nodes) continue;      // (bits beyond the last node are never set; the check costs nothing)
        atomicAdd(&counts[v], c);
        if (FIRST && order.v[f] < first_batch[v]) atomicMin(&first_batch[v], order.v[f]);
    }
}

// True if a later hop writes into a list of an earlier one (a caller that keeps nothing but nbr_local may pass one nbr or indptr
// buffer for all hops): every hop has to be relabelled before the next one is drawn.
bool rg_hops_share_buffers(const rg_blocks& o, int num_hops, const int64_t* fub, const int64_t* eub) {
    if (!o.nbr_local) return false;
    struct Range { uintptr_t lo, hi; } r[RG_MAX_HOPS][3];
    for (int h = 0; h < num_hops; ++h) {
        const int32_t* p[3] = {o.indptr[h], o.nbr[h], o.nbr_local[h]};
        const int64_t n[3] = {fub[h] + 1, eub[h], eub[h]};
        for (int j = 0; j < 3; ++j) r[h][j] = {(uintptr_t)p[j], (uintptr_t)p[j] + (uintptr_t)(p[j] ? 4 * n[j] : 0)};
        for (int e = 0; e < h; ++e)
            for (int j = 0; j < 3; ++j)
                for (int q = 0; q < 3; ++q)
                    if (r[e][j].lo < r[h][q].hi && r[h][q].lo < r[e][j].hi) return true;
    }
    return false;
}

int grid_for(int64_t work_items, int per_block, int64_t cap) {
    int64_t g = rg_div_up(work_items, per_block);
    if (g < 1) g = 1;
    if (g > cap) g = cap;
    return (int)g;
}

}  // namespace

// Scratch of the tier kernels that mark in slices, more than the others use, for `members` words of `visited` (all batches) and
// `frontier` entries of row_start; rank: per buffer of four hops.  It is allocated for as much as those two hold, so that only a
// call they have to grow for replaces any of it: were its size to follow the kind of call, its hops or its slices, a smaller
// call would leave a captured graph with freed memory.  All splits of all batches are at most kSliceGroups slices, or one bitmap each.
struct SlicedBytes { size_t marks, rank, seen; };
static SlicedBytes sliced_bytes(int64_t members, int64_t frontier, bool first_seen) {
    const int64_t marks = rg_max64(members, kSliceGroups * rg_min64(members, kSliceWords));
    const int64_t rank = rg_max64(kRankHops * members * 8, rg_rank_bytes(members));      // (more than enough for any but small graphs)
    return {(size_t)marks * 4, (size_t)rank, first_seen ? (size_t)frontier * 8 : 0};
}
// Hops beyond kRankHops have a buffer of their own unless the first one holds them too.
static bool rank_in_one(const rg_ctx* ctx, const SlicedBytes& need) { return ctx->rank[0].bytes >= 2 * need.rank; }
static bool has_slices(const rg_ctx* ctx, const SlicedBytes& need, int hops) {
    return ctx->slice_marks.bytes >= need.marks && ctx->seen.bytes >= need.seen && ctx->rank[0].bytes >= need.rank &&
           (hops <= kRankHops || rank_in_one(ctx, need) || ctx->rank[1].bytes >= need.rank);
}

rg_status rg_sampler_reserve(rg_ctx* ctx, int64_t num_nodes, int64_t max_frontier, int group, int64_t max_edges, bool first_seen) {
    SampleScratch S;
    sampler_scratch_shape(num_nodes, max_frontier, max_edges, S);
    const size_t g = (size_t)group;
    rg_status st;
    if ((st = rg_ensure(ctx, ctx->visited, g * S.words * 4)) != RG_OK) return st;
    if ((st = rg_ensure(ctx, ctx->marked, g * S.words * 4)) != RG_OK) return st;
    if ((st = rg_ensure(ctx, ctx->pos, g * (size_t)num_nodes * 4)) != RG_OK) return st;
    if ((st = rg_ensure(ctx, ctx->chunk_sum, kTableMost * 8 + 3 * g * S.chunk_stride * 4)) != RG_OK) return st;
    if ((st = rg_ensure(ctx, ctx->row_start, g * S.frontier_stride * 8)) != RG_OK) return st;
    if ((st = rg_ensure(ctx, ctx->row_deg, g * S.frontier_stride * 4)) != RG_OK) return st;
    // first-seen order: the first-edge keys must be all-zero between hops (every hop leaves them zeroed)
    if (first_seen && (st = rg_ensure(ctx, ctx->first_key, g * (size_t)num_nodes * 4, true)) != RG_OK) return st;
    return RG_OK;
}

rg_status rg_sampler_reserve_slices(rg_ctx* ctx, int64_t num_nodes, int hops, bool first_seen) {
    SampleScratch S;
    sampler_scratch_shape(num_nodes, 0, 0, S);
    if (!S.slices) return RG_OK;
    if (ctx->visited.bytes >= ctx->slices_denied) return rg_set_error(ctx, RG_ERR_OOM, "no memory for the sampler's slices at the last try");
    const SlicedBytes need = sliced_bytes((int64_t)(ctx->visited.bytes / 4), (int64_t)(ctx->row_start.bytes / 8), first_seen);
    const bool more_hops = hops > kRankHops;
    RgBuf* bufs[4] = {&ctx->slice_marks, &ctx->rank[0], &ctx->rank[1], &ctx->seen};
    void* had[4];
    for (int j = 0; j < 4; ++j) had[j] = bufs[j]->p;
    for (int j = 0; j < 4; ++j) {
        const size_t bytes = j == 0 ? need.marks : j == 1 ? need.rank * (more_hops && !ctx->rank[0].p ? 2 : 1)
                             : j == 2 ? (more_hops && !rank_in_one(ctx, need) ? need.rank : 0) : need.seen;
        const rg_status st = rg_ensure(ctx, *bufs[j], bytes);
        if (st == RG_OK) continue;
        // what was to be had is of no use without the rest: it is given back, and calls of that size do not try again
        if (st == RG_ERR_OOM) ctx->slices_denied = ctx->visited.bytes;
        for (int k = 0; k < j; ++k)
            if (bufs[k]->p != had[k]) {
                (void)hipFree(bufs[k]->p);
                *bufs[k] = RgBuf();
            }
        return st;
    }
    return RG_OK;
}

// Slices use more LDS than a kernel may by default.
rg_status rg_sampler_init(rg_ctx* ctx) {
    RG_HIP(ctx, hipFuncSetAttribute((const void*)k_sample_init, hipFuncAttributeMaxDynamicSharedMemorySize, kSliceWords * 4));
    RG_HIP(ctx, hipFuncSetAttribute((const void*)k_sample_init_most, hipFuncAttributeMaxDynamicSharedMemorySize, kSliceWords * 4));
    RG_HIP(ctx, hipFuncSetAttribute((const void*)k_slice_mark, hipFuncAttributeMaxDynamicSharedMemorySize, kSliceWords * 4));
    RG_HIP(ctx, hipFuncSetAttribute((const void*)k_seen_min, hipFuncAttributeMaxDynamicSharedMemorySize, kSeenSlice * 4));
#define RG_SMALL(RP, N) (const void*)k_sample_small<RP, 8, N>, (const void*)k_sample_small<RP, 16, N>, (const void*)k_sample_small<RP, 32, N>
    const void* small[] = {RG_SMALL(int32_t, kTableFew), RG_SMALL(int32_t, kTableMost), RG_SMALL(int64_t, kTableFew), RG_SMALL(int64_t, kTableMost)};
#undef RG_SMALL
    for (const void* f : small) RG_HIP(ctx, hipFuncSetAttribute(f, hipFuncAttributeMaxDynamicSharedMemorySize, (int)(kSmallNodes / 4)));
#define RG_SMALL(RP, N) (const void*)k_sample_small_lists<RP, 8, N>, (const void*)k_sample_small_lists<RP, 16, N>, (const void*)k_sample_small_lists<RP, 32, N>
    const void* lists[] = {RG_SMALL(int32_t, kTableFew), RG_SMALL(int32_t, kTableMost), RG_SMALL(int64_t, kTableFew), RG_SMALL(int64_t, kTableMost)};
#undef RG_SMALL
    for (const void* f : lists) RG_HIP(ctx, hipFuncSetAttribute(f, hipFuncAttributeMaxDynamicSharedMemorySize, (int)kSmallLds));
    return RG_OK;
}

extern "C" {

rg_status rg_epoch_schedule(rg_ctx* ctx, const int32_t* train_ids, int64_t n, uint64_t seed, uint32_t epoch,
                            int32_t* order_out, void* stream) {
    if (!ctx) return RG_ERR_INVALID_ARG;
    RG_REQUIRE(ctx, n >= 0, "rg_epoch_schedule: n = %lld is negative", (long long)n);
    RG_REQUIRE(ctx, n <= (1ll << 30), "rg_epoch_schedule: n = %lld exceeds 2^30", (long long)n);
    if (n == 0) return RG_OK;
    RG_REQUIRE(ctx, train_ids && order_out, "rg_epoch_schedule: null pointer");
    RG_HIP(ctx, hipSetDevice(ctx->device));
    hipStream_t s = (hipStream_t)stream;
    const uint32_t k0 = (uint32_t)(seed & 0xffffffffu), k1 = (uint32_t)(seed >> 32);
    if (n <= kSchedLds[1]) {
#define RG_SORT(MORE) k_sched_sort<kSchedLds[MORE], true, 1024><<<1, 1024, 0, s>>>(train_ids, n, 0, k0, k1, epoch, nullptr, nullptr, nullptr, nullptr, order_out, nullptr, 0)
        if (n <= kSchedLds[0]) RG_SORT(0); else RG_SORT(1);
#undef RG_SORT
        RG_LAUNCH_CHECK(ctx, "k_sched_sort");
        return RG_OK;
    }
    const int many = n > kSchedFew;
    int lb = 1;
    while (((int64_t)kSchedAvg[many] << lb) < n) ++lb;
    const int64_t buckets = 1ll << lb;
    rg_status st;
    // sized for the largest n of as many buckets, so that a call of another such n, captured perhaps, allocates nothing, and where there are
    // many ids for few as well, who have more buckets
    const int64_t most_buckets = many ? rg_max64(buckets, kSchedFewBuckets) : buckets;
    const int64_t most_pairs = kSchedRoom * most_buckets;
    if ((st = rg_ensure(ctx, ctx->sched_pairs, (size_t)most_pairs * 8)) != RG_OK) return st;
    if ((st = rg_ensure(ctx, ctx->sched_late, (size_t)rg_max64(kSchedAvg[many] * buckets, many ? kSchedAvg[0] * kSchedFewBuckets : 0) * 4)) != RG_OK) return st;
    const void* counters = ctx->sched_buckets.p;
    if ((st = rg_ensure(ctx, ctx->sched_buckets, (size_t)(4 * (most_buckets + 1)) * 4, true)) != RG_OK) return st;
    if (ctx->sched_buckets.p != counters) ctx->sched_dirty[0] = ctx->sched_dirty[1] = 0;
    uint2* pairs = (uint2*)ctx->sched_pairs.p;
    int32_t* late = (int32_t*)ctx->sched_late.p;
    // Three sets of counters, and the starts.  Calls take the first two in turn, each clearing the other one's for the next; a call that
    // is recorded into a graph keeps to the third, which its replays clear themselves.
    const int64_t set = (int64_t)(ctx->sched_buckets.bytes / 16);
    const bool captured = rg_capturing(s);
    const int turn = captured ? 2 : ctx->sched_turn, other = 1 - ctx->sched_turn;
    int32_t* count = (int32_t*)ctx->sched_buckets.p + turn * set;
    int32_t* start = buckets > kSchedLdsBuckets ? (int32_t*)ctx->sched_buckets.p + 3 * set : nullptr;
    if (captured || ctx->sched_dirty[turn]) {            // (dirty: the call before this one ended with an error)
        const int64_t to_clear = captured ? buckets + 1 : ctx->sched_dirty[turn];
        k_sched_clear<<<(int)rg_div_up(to_clear, 256), 256, 0, s>>>(count, to_clear);
        RG_LAUNCH_CHECK(ctx, "k_sched_clear");
    }
    if (!captured) ctx->sched_dirty[turn] = buckets + 1;
    const bool lds = buckets <= kSchedLdsBuckets;
    // 1024 ids to a workgroup while that leaves compute units without one
    const bool few = n <= 1024ll * ctx->num_cus;
    const int g = (int)rg_div_up(n, few ? 1024 : 4096);
#define RG_SCATTER(LDS, PER) k_sched_scatter<LDS, PER><<<g, 1024, 0, s>>>(train_ids, n, lb, k0, k1, epoch, count, pairs, late)
    if (few) RG_SCATTER(true, 1);
    else if (lds) RG_SCATTER(true, 4);
    else RG_SCATTER(false, 4);
#undef RG_SCATTER
    RG_LAUNCH_CHECK(ctx, "k_sched_scatter");
    if (start) {
        k_sched_scan<<<1, 1024, 0, s>>>(count, (int)buckets, start);
        RG_LAUNCH_CHECK(ctx, "k_sched_scan");
    }
    int32_t* clear = captured || !ctx->sched_dirty[other] ? nullptr : (int32_t*)ctx->sched_buckets.p + other * set;
#define RG_SORT(MANY)                                                                                                 \
    k_sched_sort<kSchedRoom, false, 512, MANY ? kSchedRoom : 1024><<<(unsigned)buckets, 512, 0, s>>>(nullptr, n, lb, k0, k1, epoch, count, start, pairs, late, order_out, \
                                                                                clear, clear ? (int)ctx->sched_dirty[other] : 0)
    if (many) RG_SORT(1); else RG_SORT(0);
#undef RG_SORT
    RG_LAUNCH_CHECK(ctx, "k_sched_sort");
    if (!captured) {
        ctx->sched_dirty[other] = 0;
        ctx->sched_turn = other;
    }
    return RG_OK;
}

rg_status rg_sample_blocks_group(rg_ctx* ctx, const rg_csr* csr, int32_t group, const int32_t* const* seeds,
                                 const int32_t* num_seeds, const int32_t* fanouts, int32_t num_hops, uint64_t seed,
                                 uint32_t epoch, int32_t node_order, rg_blocks* out, void* stream) {
    if (!ctx) return RG_ERR_INVALID_ARG;
    RG_REQUIRE(ctx, node_order == RG_ORDER_ASCENDING || node_order == RG_ORDER_FIRST_SEEN,
               "rg_sample_blocks: node_order = %d is neither RG_ORDER_ASCENDING nor RG_ORDER_FIRST_SEEN", node_order);
    const bool first_seen = node_order == RG_ORDER_FIRST_SEEN;
    RG_REQUIRE(ctx, group >= 1 && group <= RG_MAX_GROUP, "rg_sample_blocks: group = %d not in [1,%d]", group, RG_MAX_GROUP);
    RG_REQUIRE(ctx, csr && out && fanouts && seeds && num_seeds, "rg_sample_blocks: null argument");
    RG_REQUIRE(ctx, num_hops >= 1 && num_hops <= RG_MAX_HOPS, "rg_sample_blocks: num_hops = %d not in [1,%d]", num_hops, RG_MAX_HOPS);
    RG_REQUIRE(ctx, csr->num_nodes >= 0 && csr->num_nodes <= (int64_t)RG_ROW_MASK + 1, "rg_sample_blocks: num_nodes out of range");
    RG_REQUIRE(ctx, csr->num_edges >= 0, "rg_sample_blocks: num_edges is negative");
    RG_REQUIRE(ctx, csr->row_ptr_bits == 32 || csr->row_ptr_bits == 64, "rg_sample_blocks: row_ptr_bits must be 32 or 64");
    RG_REQUIRE(ctx, csr->row_ptr_bits == 64 || csr->num_edges < (1ll << 31), "rg_sample_blocks: 32-bit row_ptr with >= 2^31 edges");
    RG_REQUIRE(ctx, csr->row_ptr && (csr->col_idx || csr->num_edges == 0), "rg_sample_blocks: null CSR array");
    for (int h = 0; h < num_hops; ++h)
        RG_REQUIRE(ctx, fanouts[h] == RG_FANOUT_ALL || (fanouts[h] >= 0 && fanouts[h] <= RG_MAX_FANOUT),
                   "rg_sample_blocks: fanouts[%d] = %d not in [0,%d] and not RG_FANOUT_ALL", h, fanouts[h], RG_MAX_FANOUT);
    // static bounds: per batch for the capacity checks, their maximum for the launch shapes
    int64_t fub_max[RG_MAX_HOPS + 1] = {0}, eub_max[RG_MAX_HOPS] = {0};
    int32_t seeds_max = 0;
    bool capacity_error = false, shared = false;
    for (int g = 0; g < group; ++g) {
        rg_blocks* o = out + g;
        RG_REQUIRE(ctx, num_seeds[g] >= 0, "rg_sample_blocks: num_seeds is negative (batch %d)", g);
        RG_REQUIRE(ctx, num_seeds[g] <= csr->num_nodes, "rg_sample_blocks: more seeds than nodes (seeds must be distinct; batch %d)", g);
        RG_REQUIRE(ctx, seeds[g] || num_seeds[g] == 0, "rg_sample_blocks: seeds is NULL (batch %d)", g);
        RG_REQUIRE(ctx, o->nodes && o->tier_off && o->indptr && o->indptr_cap && o->nbr && o->nbr_cap,
                   "rg_sample_blocks: null output pointer (batch %d)", g);
        int64_t fub[RG_MAX_HOPS + 1], eub[RG_MAX_HOPS];
        rg_blocks_bounds(csr->num_nodes, csr->num_edges, num_seeds[g], fanouts, num_hops, fub, eub);
        bool too_small = o->nodes_cap < fub[num_hops];
        for (int h = 0; h < num_hops; ++h) {
            RG_REQUIRE(ctx, eub[h] < (1ll << 31), "rg_sample_blocks: hop %d may produce >= 2^31 edges", h);
            RG_REQUIRE(ctx, o->indptr[h] && (o->nbr[h] || eub[h] == 0), "rg_sample_blocks: null buffer for hop %d (batch %d)", h, g);
            RG_REQUIRE(ctx, !o->nbr_local || o->nbr_local[h] || eub[h] == 0, "rg_sample_blocks: nbr_local[%d] is NULL (batch %d)", h, g);
            too_small = too_small || o->indptr_cap[h] < fub[h] + 1 || o->nbr_cap[h] < eub[h];
            eub_max[h] = rg_max64(eub_max[h], eub[h]);
        }
        if (too_small) {
            // the required sizes go back to the caller in place of the capacities that were passed in
            rg_set_error(ctx, RG_ERR_CAPACITY, "rg_sample_blocks: output buffers of batch %d are below the static bounds "
                         "(nodes_cap %lld < %lld, or a hop's indptr_cap / nbr_cap); the required sizes were written back",
                         g, (long long)o->nodes_cap, (long long)fub[num_hops]);
            o->nodes_cap = fub[num_hops];
            for (int h = 0; h < num_hops; ++h) { o->indptr_cap[h] = fub[h] + 1; o->nbr_cap[h] = eub[h]; }
            capacity_error = true;
        }
        shared = shared || rg_hops_share_buffers(*o, num_hops, fub, eub);
        for (int h = 0; h <= num_hops; ++h) fub_max[h] = rg_max64(fub_max[h], fub[h]);
        seeds_max = num_seeds[g] > seeds_max ? num_seeds[g] : seeds_max;
    }
    if (capacity_error) return RG_ERR_CAPACITY;

    RG_HIP(ctx, hipSetDevice(ctx->device));
    hipStream_t s = (hipStream_t)stream;
    const int64_t N = csr->num_nodes;
    int64_t max_edges = 0;
    if (first_seen)
        for (int h = 0; h < num_hops; ++h) max_edges = rg_max64(max_edges, eub_max[h]);
    SampleScratch S;
    sampler_scratch_shape(N, fub_max[num_hops], max_edges, S);
    const int64_t words = S.words;
    ctx->last_sample_group = 0;                       // no membership bitmaps to add until this call has been queued
    int64_t edges_bound = 0, frontiers_bound = 0;
    for (int h = 0; h < num_hops; ++h) { edges_bound += eub_max[h]; frontiers_bound += fub_max[h]; }
    int64_t expected[RG_MAX_HOPS];
    const int64_t edges = rg_expected_edges(N, csr->num_edges, seeds_max, fanouts, num_hops, eub_max, expected);
    // Hops that a thread or a few lanes per node draw for; these need no offsets per node.
    const auto drawn_by_threads = [&](int h) {
        return fanouts[h] >= 1 && (fanouts[h] <= 32 || (fanouts[h] <= RG_WAVE && fub_max[h] <= kWideNodes && fub_max[h] * group <= kWideNodesAll)) && csr->num_edges < (1ll << 32);
    };
    bool by_threads = true;
    for (int h = 0; h < num_hops; ++h) by_threads = by_threads && drawn_by_threads(h);
    // in first-seen order the edges' ascending positions are kept where their final ones go
    bool ranked_seen = first_seen && rg_use_ranked_seen(S.slices, N, edges, group);
    for (int g = 0; g < group && ranked_seen; ++g)
        for (int h = 0; h < num_hops; ++h)
            ranked_seen = ranked_seen && eub_max[h] <= kRankedSeenEdges && out[g].nbr_local && out[g].nbr_local[h] && out[g].nbr_local[h] != out[g].nbr[h];
    TierMode mode = ranked_seen ? kTierRankedSeen : first_seen ? kTierFirstSeen : (rg_use_slices(S.slices, N, edges, group, by_threads) ? kTierSliced : kTierAtomic);
    if (!first_seen && by_threads && rg_use_bytes(N, words, edges, group)) mode = kTierBytes;
    rg_status st = rg_sampler_reserve(ctx, N, fub_max[num_hops], group, max_edges, first_seen);
    if (st != RG_OK) return st;
    int max_fanout = 0;
    for (int h = 0; h < num_hops; ++h) max_fanout = fanouts[h] < 0 ? RG_MAX_FANOUT : (fanouts[h] > max_fanout ? fanouts[h] : max_fanout);
    int64_t hop_edges = 0;
    for (int h = 0; h < num_hops; ++h) hop_edges = rg_max64(hop_edges, eub_max[h]);
    const bool in_lds = rg_small_lists_fit(N, fub_max[num_hops - 1], hop_edges);
    const bool small = !first_seen && max_fanout <= 32 && csr->num_edges < (1ll << 32) &&
                       (rg_is_small(N, csr->num_edges, num_hops, in_lds, edges_bound, frontiers_bound) ||
                        (in_lds && max_fanout <= 16 && rg_max64(edges_bound, frontiers_bound) <= kSmallEdgesPerHop * num_hops));
    // Slices whose scratch is not there and cannot be allocated (a captured call, no memory): the atomic kernels, same results.
    if (!small && (mode == kTierSliced || mode == kTierRankedSeen || mode == kTierBytes)) {
        const SlicedBytes need = sliced_bytes(group * words, group * S.frontier_stride, first_seen);
        bool there = has_slices(ctx, need, num_hops);
        if (!there && !rg_capturing(s)) {
            st = rg_sampler_reserve_slices(ctx, N, num_hops, first_seen);
            if (st != RG_OK && st != RG_ERR_OOM) return st;
            there = st == RG_OK;
        }
        if (!there) mode = first_seen ? kTierFirstSeen : kTierAtomic;
        S.rank[0] = (uint4*)ctx->rank[0].p;
        S.rank[1] = rank_in_one(ctx, need) ? S.rank[0] + need.rank / sizeof(uint4) : (uint4*)ctx->rank[1].p;
    }
    S.hops = num_hops;
    S.slice_marks = (uint32_t*)ctx->slice_marks.p;
    S.first_key = mode == kTierFirstSeen ? (int32_t*)ctx->first_key.p : nullptr;
    S.first_edge = (int32_t*)ctx->seen.p;
    S.place = S.first_edge + group * S.frontier_stride;
    S.group = group;
    S.group_inv = group > 1 ? 0xFFFFFFFFu / (uint32_t)group + 1u : 0u;
    S.xcd_map = ctx->knobs.xcd_map;
    S.visited = (uint32_t*)ctx->visited.p;
    S.marked = (uint32_t*)ctx->marked.p;
    S.pos = (int32_t*)ctx->pos.p;
    S.chunk_sum = (int32_t*)((uint64_t*)ctx->chunk_sum.p + kTableMost);
    S.hop_sum[0] = S.chunk_sum + group * S.chunk_stride;
    S.hop_sum[1] = S.hop_sum[0] + group * S.chunk_stride;
    S.row_start = (int64_t*)ctx->row_start.p;
    S.row_deg = (int32_t*)ctx->row_deg.p;
    const uint32_t k0 = (uint32_t)(seed & 0xffffffffu), k1 = (uint32_t)(seed >> 32);
    const bool rp64 = csr->row_ptr_bits == 64;

    BatchTable<kTableMost> table;
    S.table = (const uint64_t*)ctx->chunk_sum.p;
    S.table_entries = (kHopFields + kHopFieldCount * num_hops) * group;
    for (int g = 0; g < group; ++g) {
        const auto put = [&](int field, const void* p) { table.v[field * group + g] = (uint64_t)(uintptr_t)p; };
        put(kSeeds, seeds[g]);
        table.v[kNumSeeds * group + g] = (uint64_t)num_seeds[g];
        put(kNodes, out[g].nodes);
        put(kTierOff, out[g].tier_off);
        put(kEdgesOut, out[g].num_edges);
        for (int h = 0; h < num_hops; ++h) {
            put(kHopFields + kHopFieldCount * h + kIndptr, out[g].indptr[h]);
            put(kHopFields + kHopFieldCount * h + kNbr, out[g].nbr[h]);
            put(kHopFields + kHopFieldCount * h + kNbrLocal, out[g].nbr_local && eub_max[h] > 0 ? out[g].nbr_local[h] : nullptr);
        }
    }
    BatchTable<kTableSome> some;
    const bool most = S.table_entries > kTableSome;
    if (!most) memcpy(some.v, table.v, (size_t)S.table_entries * 8);
    const unsigned ug = (unsigned)group;

    if (small) {
        Fanouts fan = {};
        for (int h = 0; h < num_hops; ++h) fan.v[h] = fanouts[h];
        BatchTable<kTableFew> few;
        const bool is_few = S.table_entries <= kTableFew;
        if (is_few) memcpy(few.v, table.v, (size_t)S.table_entries * 8);
        const int tok = rg_prof_begin(ctx, RG_K_SAMPLE, s);
        const int keep_hops = rg_small_lists_fit(N, fub_max[num_hops], hop_edges) ? num_hops : num_hops - 1;
        const int64_t lists = rg_small_lists_bytes(N, fub_max[keep_hops], hop_edges);
#define RG_LAUNCH_SMALL_N(RP, KM, N, TABLE)                                                                           \
    do {                                                                                                              \
        if (in_lds) k_sample_small_lists<RP, KM, N><<<ug, 1024, (size_t)lists, s>>>((const RP*)csr->row_ptr, csr->col_idx, TABLE, group, fan, \
                                                S.visited, words, N_nodes, (int)fub_max[keep_hops], keep_hops, num_hops, k0, k1, epoch); \
        else k_sample_small<RP, KM, N><<<ug, 1024, (size_t)words * 8, s>>>((const RP*)csr->row_ptr, csr->col_idx, TABLE, group, fan, S.visited, \
                                                                           words, S.pos, N_nodes, num_hops, k0, k1, epoch); \
    } while (0)
#define RG_LAUNCH_SMALL(RP, KM) do { if (is_few) RG_LAUNCH_SMALL_N(RP, KM, kTableFew, few); else RG_LAUNCH_SMALL_N(RP, KM, kTableMost, table); } while (0)
        const int64_t N_nodes = N;
        if (rp64) { if (max_fanout <= 8) RG_LAUNCH_SMALL(int64_t, 8); else if (max_fanout <= 16) RG_LAUNCH_SMALL(int64_t, 16); else RG_LAUNCH_SMALL(int64_t, 32); }
        else { if (max_fanout <= 8) RG_LAUNCH_SMALL(int32_t, 8); else if (max_fanout <= 16) RG_LAUNCH_SMALL(int32_t, 16); else RG_LAUNCH_SMALL(int32_t, 32); }
#undef RG_LAUNCH_SMALL
#undef RG_LAUNCH_SMALL_N
        rg_prof_end(ctx, tok, s);
        RG_LAUNCH_CHECK(ctx, "k_sample_small");
        ctx->last_sample_group = group;
        ctx->last_sample_nodes = N;
        return RG_OK;
    }
    if (words > 0) {
        if (ctx->sampler_dirty && ctx->first_key.bytes) {   // an earlier first-seen call stopped between a draw kernel and its emit
            const int64_t key_words = (int64_t)(ctx->first_key.bytes / 4);
            k_clear_words<<<(int)rg_div_up(key_words, 256), 256, 0, s>>>((uint32_t*)ctx->first_key.p, key_words);
            RG_LAUNCH_CHECK(ctx, "k_clear_words");
        }
        ctx->sampler_dirty = true;       // cleared again when every launch of this call has been queued
    }
    const RowPtr row_ptr = {csr->row_ptr, rp64};
    int counted = -1;                                  // the hop whose sizes are there already
    // Small workgroups for the tiers while large ones would leave compute units without work: one batch on 233 k nodes 69 us a call with large, 56 with
    // small ones, on 380 k 150 / 117; 369 large ones (3 batches, 3 M nodes) 147 / 158, 648 (8 batches, 2 M) 120 / 140.
    const bool small_tier = mode != kTierAtomic && rg_div_up(words, kTierWords) * group < ctx->num_cus;
    const unsigned tier_blocks = (unsigned)rg_max64(1, rg_div_up(words, small_tier ? kTierWordsSmall : kTierWords));
    const bool self_count = mode == kTierBytes && small_tier && words <= kBytesSelfWords && (int64_t)tier_blocks * group * words * 16 <= kBytesSelfRead;
    uint32_t* const bytes_at[2] = {S.slice_marks, S.slice_marks + (self_count ? group * words * 8 : 0)};
    // Counted so, the members after the last hop are to be in `visited`.
    const auto members = [&](int h) { return self_count && ((num_hops - h) & 1) ? S.marked : S.visited; };
    uint32_t* const seeds_at = members(0);
    if (rg_use_init(S.slices, group, seeds_max)) {
        const unsigned count_blocks = drawn_by_threads(0) ? (unsigned)rg_div_up(seeds_max, kChunk) : 0u;
        const size_t lds = (size_t)rg_max64(S.slice_words, 1024 / RG_WAVE) * 4;
        const unsigned init_blocks = ((unsigned)S.slices + count_blocks) * ug;
        SampleScratch S0 = S;
        S0.visited = seeds_at;
        if (most) k_sample_init_most<<<init_blocks, 1024, lds, s>>>(row_ptr, table, S0, fanouts[0], mode);
        else k_sample_init<<<init_blocks, 1024, lds, s>>>(row_ptr, some, S0, fanouts[0], mode);
        if (count_blocks) counted = 0;
        RG_LAUNCH_CHECK(ctx, "k_sample_init");
    } else {
        const int64_t group_words = (int64_t)group * words;
        k_clear_words<<<(int)rg_div_up(group_words, 256), 256, 0, s>>>(seeds_at, group_words);
        RG_LAUNCH_CHECK(ctx, "k_clear_words");
        if (mode == kTierBytes) {
            k_clear_words<<<(int)rg_div_up(group_words * 8, 256), 256, 0, s>>>(S.slice_marks, group_words * 8);
            RG_LAUNCH_CHECK(ctx, "k_clear_words");
        }
        if (mode == kTierAtomic) {
            k_clear_words<<<(int)rg_div_up(group_words, 256), 256, 0, s>>>(S.marked, group_words);
            RG_LAUNCH_CHECK(ctx, "k_clear_words");
        }
        const unsigned mark_blocks = (unsigned)(grid_for(seeds_max, 256, 1 << 30)) * ug;
        SampleScratch S0 = S;
        S0.visited = seeds_at;
        if (most) k_mark_seeds_most<<<mark_blocks, 256, 0, s>>>(table, S0); else k_mark_seeds<<<mark_blocks, 256, 0, s>>>(some, S0);
        RG_LAUNCH_CHECK(ctx, "k_mark_seeds");
    }

    // Edges of a hop that the kernels which walk its list are launched for; more of them take further rounds.  The static bound may be far
    // from what comes (RG_FANOUT_ALL: the whole graph), and a workgroup without an edge takes its time all the same.  Launched for the
    // bound and for these: two batches of 6 seeds, all neighbours, then five, on 190 k nodes of 186 edges in first-seen order 168 / 67 us;
    // four of 92 seeds on 22 k nodes of 103, ascending, 72 / 62.
    const auto launch_edges = [&](int h) {
        return rg_min64(eub_max[h], rg_max64(8 * expected[h], rg_div_up(4ll * ctx->num_cus, group) * 1024));
    };
    const auto relabel = [&](int first_hop, int last_hop) -> rg_status {
        int64_t edges_most = 0;
        for (int h = first_hop; h <= last_hop; ++h)
            for (int g = 0; g < group; ++g)
                if (out[g].nbr_local) edges_most = rg_max64(edges_most, launch_edges(h));
        if (edges_most == 0) return RG_OK;
        const unsigned blocks = (unsigned)grid_for(edges_most, 1024, rg_div_up((int64_t)ctx->num_cus * 32, group));
        if (mode == kTierSliced) k_relabel<true><<<blocks * ug, 256, (size_t)((last_hop + 1) * S.rank_bases) * 4, s>>>(S, first_hop, last_hop);
        else if (mode == kTierRankedSeen) k_seen_relabel<<<blocks * ug, 256, 0, s>>>(S, first_hop, last_hop);
        else k_relabel<false><<<blocks * ug, 256, 0, s>>>(S, first_hop, last_hop);
        RG_LAUNCH_CHECK(ctx, "k_relabel");
        return RG_OK;
    };
    // How `blocks` workgroups per batch are dealt out (rg_shared_rows), a power of two of consecutive ones, `longest` at most.
    const auto shared_run = [&](int64_t blocks, int64_t longest, unsigned& grid) -> int {
        grid = (unsigned)blocks * ug;
        const int64_t most = rg_min64(longest, blocks / (8 * kXcds));
        if (group == 1 || first_seen || !S.xcd_map || most < 1) return 0;
        int log2_run = 0;
        while ((2ll << log2_run) <= most) ++log2_run;
        const int64_t run = 1ll << log2_run;
        grid = (unsigned)(rg_div_up(blocks, kXcds * run) * kXcds * run) * ug;
        return log2_run + 1;
    };
    for (int h = 0; h < num_hops; ++h) {
        if (counted != h) {
            unsigned count_grid;
            const int count_run = shared_run(grid_for(fub_max[h], kChunk, 1ll << 30), kSharedNodes / kChunk, count_grid);
            const int offsets = drawn_by_threads(h) ? 0 : 1;
            if (rp64)
                k_hop_count<int64_t><<<count_grid, kChunk / kCountNodes, 0, s>>>((const int64_t*)csr->row_ptr, S, h, fanouts[h], count_run, offsets);
            else
                k_hop_count<int32_t><<<count_grid, kChunk / kCountNodes, 0, s>>>((const int32_t*)csr->row_ptr, S, h, fanouts[h], count_run, offsets);
            RG_LAUNCH_CHECK(ctx, "k_hop_count");
        }

        const int F = fanouts[h];
        if (mode == kTierBytes) S.slice_marks = bytes_at[h & 1];
        if (drawn_by_threads(h)) {
            const int tok = rg_prof_begin(ctx, RG_K_SAMPLE, s);
            // 64 nodes per workgroup while 256 would leave compute units without two workgroups (see the kernel)
            const bool few = rg_div_up(fub_max[h], 256) * group < 2ll * ctx->num_cus;
            const int nodes_per = few ? 64 : 256;
            unsigned draw_grid;
            const int draw_run = shared_run(grid_for(fub_max[h], nodes_per, 1ll << 30), kSharedNodes / nodes_per, draw_grid);
            const size_t lds = (size_t)nodes_per * F * sizeof(uint32_t);
            const bool lanes = F > 16 && fub_max[h] * group * 32 <= kLaneDraws;
            // Adding up grows with the square of the frontier, a scan costs 3 us for a small one: of 1 M nodes 172 / 175 us, of 8 M
            // 1206 / 1196, of 16 M 2555 / 2498, of 40 M 7213 / 6750.
            const int scanned = rg_div_up(fub_max[h], kChunk) > kDrawSelfScan;
            if (scanned) {
                k_scan_hop<<<ug, 1024, 0, s>>>(S, h);
                RG_LAUNCH_CHECK(ctx, "k_scan_hop");
            }
#define RG_LAUNCH_DRAW(KM, NP, MODE)                                                                                  \
    k_hop_sample_thread<KM, NP, MODE><<<draw_grid, 256, lds, s>>>(csr->col_idx, S, F, (uint32_t)h, k0, k1, epoch, scanned, draw_run)
#define RG_LAUNCH_LANES(KM, MODE)                                                                                     \
    k_hop_sample_lanes<KM, MODE><<<(unsigned)grid_for(fub_max[h], 256 / KM, 1ll << 30) * ug, 256, 0, s>>>(csr->col_idx, S, F, (uint32_t)h, k0, k1, epoch)
#define RG_LAUNCH_DRAW_K(NP, MODE)                                                                                    \
    do { if (F <= 8) RG_LAUNCH_DRAW(8, NP, MODE); else if (F <= 16) RG_LAUNCH_DRAW(16, NP, MODE); else RG_LAUNCH_DRAW(32, NP, MODE); } while (0)
#define RG_LAUNCH_DRAW_N(MODE) do { if (F > 32) RG_LAUNCH_LANES(64, MODE); else if (lanes) RG_LAUNCH_LANES(32, MODE); else if (few) RG_LAUNCH_DRAW_K(64, MODE); else RG_LAUNCH_DRAW_K(256, MODE); } while (0)
            if (mode == kTierSliced || mode == kTierRankedSeen) RG_LAUNCH_DRAW_N(kTierSliced);
            else if (mode == kTierAtomic) RG_LAUNCH_DRAW_N(kTierAtomic);
            else if (mode == kTierBytes) RG_LAUNCH_DRAW_N(kTierBytes);
            else RG_LAUNCH_DRAW_N(kTierFirstSeen);
#undef RG_LAUNCH_DRAW_N
#undef RG_LAUNCH_LANES
#undef RG_LAUNCH_DRAW_K
#undef RG_LAUNCH_DRAW
            rg_prof_end(ctx, tok, s);
        } else {
            // chunk sums -> exclusive offsets; total edge count -> indptr[n_h]
            k_scan_hop<<<ug, 1024, 0, s>>>(S, h);
            RG_LAUNCH_CHECK(ctx, "k_scan_hop");
            const int tok = rg_prof_begin(ctx, RG_K_SAMPLE, s);
            const unsigned sample_blocks = (unsigned)grid_for(fub_max[h], 1, (int64_t)ctx->num_cus * 64);
#define RG_LAUNCH_WAVE(MODE)                                                                                          \
    k_hop_sample_wave<MODE><<<sample_blocks * ug, RG_WAVE, 0, s>>>(csr->col_idx, S, F, (uint32_t)h, k0, k1, epoch)
            if (mode == kTierSliced || mode == kTierRankedSeen) RG_LAUNCH_WAVE(kTierSliced);
            else if (mode == kTierAtomic) RG_LAUNCH_WAVE(kTierAtomic);
            else RG_LAUNCH_WAVE(kTierFirstSeen);
#undef RG_LAUNCH_WAVE
            rg_prof_end(ctx, tok, s);
        }
        RG_LAUNCH_CHECK(ctx, "k_hop_sample");

        if (mode == kTierSliced || mode == kTierRankedSeen) {
            const int64_t split_edges = rg_max64(kSplitEdges, 2 * (int64_t)S.slice_words);
            // (hubs among the frontier: up to eight times the edges of average nodes)
            S.splits = (int)rg_max64(1, rg_min64(rg_min64(eub_max[h], 8 * expected[h]) / split_edges, kSliceGroups / (S.slices * group)));
            k_slice_mark<<<(unsigned)(S.slices * S.splits) * ug, 1024, (size_t)S.slice_words * 4, s>>>(S, h);
            RG_LAUNCH_CHECK(ctx, "k_slice_mark");
            const bool count_next = mode == kTierSliced && h + 1 < num_hops && drawn_by_threads(h + 1);
            const int next_fanout = count_next ? fanouts[h + 1] : -1;
            unsigned emit_grid = tier_blocks * ug;
            const int emit_run = count_next ? shared_run((int64_t)tier_blocks + rg_div_up(fub_max[h], kChunk), 1, emit_grid) : 0;
            if (count_next) counted = h + 1;
#define RG_LAUNCH_TIER(EMIT, TE, T, W)                                                                                    \
    do {                                                                                                              \
        k_slice_count<T, W><<<tier_blocks * ug, T, 0, s>>>(S);                                                        \
        RG_LAUNCH_CHECK(ctx, "k_slice_count");                                                                        \
        if (mode == kTierSliced) EMIT<false><<<emit_grid, TE, 0, s>>>(row_ptr, S, h, tier_blocks, next_fanout, emit_run);             \
        else EMIT<true><<<tier_blocks * ug, TE, 0, s>>>(row_ptr, S, h, tier_blocks, -1, 0);                                   \
        RG_LAUNCH_CHECK(ctx, "k_slice_emit");                                                                         \
    } while (0)
            if (small_tier) RG_LAUNCH_TIER(k_slice_emit_small, kEmitThreadsSmall, kTierWordsSmall, 1); else RG_LAUNCH_TIER(k_slice_emit, kTierWords / 3, kTierWords / 3, 3);
#undef RG_LAUNCH_TIER
            if (mode == kTierRankedSeen) {
                // the edges that open a node, counted per block of the edge list, emitted in edge order
                k_seen_rank<<<(unsigned)grid_for(eub_max[h], 1024, (int64_t)ctx->num_cus * 16) * ug, 256, (size_t)((h + 1) * S.rank_bases) * 4, s>>>(S, h);
                RG_LAUNCH_CHECK(ctx, "k_seen_rank");
                const int64_t most_new = rg_min64(N, eub_max[h]);
                k_seen_min<<<(unsigned)grid_for(most_new, kSeenSlice, 1 << 30) * ug, 1024, (size_t)rg_min64(most_new, kSeenSlice) * 4, s>>>(S, h);
                RG_LAUNCH_CHECK(ctx, "k_seen_min");
                const unsigned seen_blocks = (unsigned)grid_for(eub_max[h], kSeenEdges, 1 << 30);
                k_seen_count<<<seen_blocks * ug, 1024, 0, s>>>(S, h);
                RG_LAUNCH_CHECK(ctx, "k_seen_count");
                const bool sizes = h + 1 < num_hops && drawn_by_threads(h + 1);
                if (sizes) counted = h + 1;
                k_seen_emit<<<(seen_blocks + (sizes ? (unsigned)rg_div_up(fub_max[h], kChunk) : 0u)) * ug, 1024, 0, s>>>(row_ptr, S, h, seen_blocks,
                                                                                                                        sizes ? fanouts[h + 1] : -1);
                RG_LAUNCH_CHECK(ctx, "k_seen_emit");
            }
        } else if (mode == kTierFirstSeen) {
            // new tier: edges that open a node, counted per block of the edge list, scanned, emitted in edge order
            const int fs_blocks = (int)rg_max64(1, rg_div_up(launch_edges(h), kEdgesPerBlock));
            k_first_seen_count<<<(unsigned)(fs_blocks) * ug, 256, 0, s>>>(S, h);
            RG_LAUNCH_CHECK(ctx, "k_first_seen_count");
            // Adding up grows with the square of the chunks, a scan takes a launch.  (The edges there are make one chunk per workgroup where it was
            // launched for the bound; asking for them takes 1 us a hop.)
            const int scanned = rg_div_up(eub_max[h], kEdgesPerBlock) > kTierSelfScan;
            if (scanned) {
                k_scan_tier<<<ug, 1024, 0, s>>>(S, h, fs_blocks, launch_edges(h) < eub_max[h] ? kEdgesPerBlock : 0);
                RG_LAUNCH_CHECK(ctx, "k_scan_tier");
            }
            const bool count_next = h + 1 < num_hops && drawn_by_threads(h + 1);
            if (count_next) counted = h + 1;
            k_first_seen_emit<<<(unsigned)(fs_blocks) * ug, 256, 0, s>>>(row_ptr, S, h, count_next ? fanouts[h + 1] : -1, scanned);
            RG_LAUNCH_CHECK(ctx, "k_first_seen_emit");
        } else {
            const int words_per = small_tier ? kTierWordsSmall : kTierWords, scanned = tier_blocks > kTierSelfScan;
            if (mode == kTierBytes && !self_count) {
                k_bytes_count<<<tier_blocks * ug, 256, 0, s>>>(S, words_per, h + 1 < num_hops);
                RG_LAUNCH_CHECK(ctx, "k_bytes_count");
            } else if (!self_count) {
                k_tier_count<<<tier_blocks * ug, 256, 0, s>>>(S, words_per);
                RG_LAUNCH_CHECK(ctx, "k_tier_count");
                if (scanned) {
                    k_scan_tier<<<ug, 1024, 0, s>>>(S, h, (int)tier_blocks, 0);
                    RG_LAUNCH_CHECK(ctx, "k_scan_tier");
                }
            }
            const bool count_next = h + 1 < num_hops && drawn_by_threads(h + 1);
            const int next_fanout = count_next ? fanouts[h + 1] : -1;
            unsigned emit_grid = tier_blocks * ug;
            const int emit_run = count_next ? shared_run((int64_t)tier_blocks + rg_div_up(fub_max[h], kChunk), 1, emit_grid) : 0;
            if (count_next) counted = h + 1;
            if (self_count) {
                uint8_t* next = h + 1 < num_hops ? (uint8_t*) bytes_at[(h + 1) & 1] : nullptr;
                k_bytes_emit_small<<<emit_grid, kEmitThreadsSmall, 0, s>>>(row_ptr, S, h, tier_blocks, next_fanout, emit_run, members(h), members(h + 1), next);
            } else {
                if (small_tier) k_tier_emit_small<<<emit_grid, kEmitThreadsSmall, 0, s>>>(row_ptr, S, h, tier_blocks, next_fanout, emit_run, scanned);
                else k_tier_emit<<<emit_grid, kTierWords / 3, 0, s>>>(row_ptr, S, h, tier_blocks, next_fanout, emit_run, scanned);
            }
            RG_LAUNCH_CHECK(ctx, "k_tier_emit");
        }
        if (shared && (st = relabel(h, h)) != RG_OK) return st;
    }
    if (!shared && (st = relabel(0, num_hops - 1)) != RG_OK) return st;
    ctx->sampler_dirty = false;
    ctx->last_sample_group = group;
    ctx->last_sample_nodes = N;
    return RG_OK;
}

rg_status rg_access_histogram_sampled(rg_ctx* ctx, int32_t group, const int32_t* batch_index, uint32_t* counts,
                                      uint32_t* first_batch, int64_t num_nodes, void* stream) {
    if (!ctx) return RG_ERR_INVALID_ARG;
    RG_REQUIRE(ctx, group >= 1 && group <= RG_MAX_GROUP, "rg_access_histogram_sampled: group = %d not in [1,%d]", group, RG_MAX_GROUP);
    RG_REQUIRE(ctx, counts && (batch_index || !first_batch), "rg_access_histogram_sampled: null counts, or first_batch without batch_index");
    if (ctx->last_sample_group != group || ctx->last_sample_nodes != num_nodes)
        return rg_set_error(ctx, RG_ERR_STATE, "rg_access_histogram_sampled: the last sampling call of this context covered %d "
                            "batches on %lld nodes, not %d on %lld", ctx->last_sample_group, (long long)ctx->last_sample_nodes,
                            group, (long long)num_nodes);
    BatchIndices order = {};
    for (int g = 0; g < group; ++g) {
        RG_REQUIRE(ctx, !batch_index || batch_index[g] >= 0, "rg_access_histogram_sampled: negative batch index");
        const uint32_t v = batch_index ? (uint32_t)batch_index[g] : 0u;
        int at = g;
        for (; at > 0 && order.v[at - 1] > v; --at) { order.v[at] = order.v[at - 1]; order.batch[at] = order.batch[at - 1]; }
        order.v[at] = v;
        order.batch[at] = (uint8_t)g;
    }
    if (num_nodes == 0) return RG_OK;
    RG_HIP(ctx, hipSetDevice(ctx->device));
    hipStream_t s = (hipStream_t)stream;
    const int64_t words = rg_div_up(num_nodes, 32);
    const int64_t waves = rg_div_up(words, RG_WAVE);
    const int parts = first_batch && waves <= 8ll * ctx->num_cus ? 8 : 1;
    const unsigned blocks = (unsigned)rg_div_up(waves * parts, 4);
    const int tok = rg_prof_begin(ctx, RG_K_HISTOGRAM, s);
#define RG_LAUNCH_BITMAPS(FIRST, PARTS)                                                                                   \
    k_histogram_bitmaps<FIRST, PARTS><<<blocks, 256, 0, s>>>((const uint32_t*)ctx->visited.p, words, group, order, counts, first_batch, num_nodes)
    if (!first_batch) RG_LAUNCH_BITMAPS(false, 1); else if (parts == 1) RG_LAUNCH_BITMAPS(true, 1); else RG_LAUNCH_BITMAPS(true, 8);
#undef RG_LAUNCH_BITMAPS
    rg_prof_end(ctx, tok, s);
    RG_LAUNCH_CHECK(ctx, "k_histogram_bitmaps");
    return RG_OK;
}

rg_status rg_sample_blocks(rg_ctx* ctx, const rg_csr* csr, const int32_t* seeds, int32_t num_seeds,
                           const int32_t* fanouts, int32_t num_hops, uint64_t seed, uint32_t epoch,
                           rg_blocks* out, void* stream) {
    return rg_sample_blocks_group(ctx, csr, 1, &seeds, &num_seeds, fanouts, num_hops, seed, epoch, RG_ORDER_ASCENDING, out, stream);
}

}  // extern "C"

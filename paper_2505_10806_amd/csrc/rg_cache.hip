// Access-frequency histogram (Section IV, offline stage), TopHot selection (Alg. 1 line 3), the hit curve
// against cache size (Section V), and VectorPull (Alg. 1 line 4) in its two forms: one bulk pull, or pulls by
// first use ahead of the gathers (the prefetcher of Section III: with a per-batch claim pass or from a
// per-epoch plan).
#include <math.h>
#include <stddef.h>

#include "rg_rowcopy.h"

namespace {

// ---------------------------------------------------------------------------- histogram
__global__ void __launch_bounds__(256) k_histogram(const int32_t* __restrict__ nodes, int64_t n, const int32_t* __restrict__ n_dev,
                                                   uint32_t* __restrict__ counts) {
    int64_t n_act = n;
    if (n_dev) { const int64_t d = *n_dev; n_act = d < n ? d : n; }
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n_act; i += (int64_t)gridDim.x * blockDim.x)
        atomicAdd(&counts[nodes[i]], 1u);
}

// Epoch-level histogram over many sampled batches.  Every tier after the seeds is ascending by id, so a
// workgroup that owns the id range [j * range, (j + 1) * range) accumulates its entries of each (batch, tier) run in
// an LDS-private copy of its counters with LDS atomics and adds the range to `counts` once with plain coalesced
// read-modify-writes: no global atomics, every id read once.
// Where the ranges begin in every run is found first, by k_hist_bounds: searched for by every workgroup itself (two bisections
// per run of 18 steps, whose lines no other lane shares) the 10 M random lines took 180 of 184 us for 72 M entries on 2.4 M
// nodes with first batches.  The range is chosen so that the workgroups, two per compute unit, make whole rounds of the
// device (598 on 512 places: 273 us).  The counting is bound by latency, LDS atomics and VALU alike (a third of the time each for
// the last two): with a step's loads waited for before the next one's began it took 95 us, now 66, and the bounds 19.
constexpr int kHistRangeMax = 8192;    // ids per workgroup at most (32 KB of LDS, 64 KB when first batches are tracked as well)
constexpr int kHistRangeMin = 512;
constexpr int kHistRunTile = 1024;     // runs whose bounds are in LDS at a time
// Entries of a run per range (by the lists' room, about twice what is in them) from which on reading ahead is never slower.  Without and with it,
// clearing included: 62 33 / 37 us, 114 31 / 33, 173 57 / 62, 206 56 / 57 and 80 / 78, 255 66 / 61, 29 / 26 and 43 / 35, but 260 63 / 66, 275 61 / 60
// and 54 / 52, 344 65 / 65 and 65 / 63; 412 57 / 53, 481 111 / 95, 584 125 / 102, 651 56 / 54 to 74 / 67, 704 141 / 113, 1100 63 / 57.
constexpr int kHistAhead = 384;

// Seeds of batch b, by blocks of 256 threads, `block` of `blocks`.  They are in caller order (not sorted): one global atomic each.
__device__ __forceinline__ void rg_count_seeds(const int32_t* __restrict__ nodes, int64_t batch_stride, const int32_t* __restrict__ tier_off,
                                               int num_hops, int b, int block, int blocks, uint32_t* __restrict__ counts,
                                               uint32_t* __restrict__ first_batch) {
    const int n_seeds = tier_off[(int64_t)b * (num_hops + 2) + 1];
    const int32_t* base = nodes + (int64_t)b * batch_stride;
    for (int i = block * 256 + threadIdx.x; i < n_seeds; i += blocks * 256) {
        atomicAdd(&counts[base[i]], 1u);
        if (first_batch) atomicMin(&first_batch[base[i]], (uint32_t)b);
    }
}

__global__ void __launch_bounds__(256) k_histogram_seeds(const int32_t* __restrict__ nodes, int64_t batch_stride,
                                                         const int32_t* __restrict__ tier_off, int num_hops,
                                                         uint32_t* __restrict__ counts, uint32_t* __restrict__ first_batch) {
    rg_count_seeds(nodes, batch_stride, tier_off, num_hops, blockIdx.y, blockIdx.x, gridDim.x, counts, first_batch);
}

constexpr int kSeedsBeside = 256;      // seeds per batch from which on k_hist_bounds counts them
// Few batches get workgroups for kSeedRounds rounds of 256 seeds each, as far as all of them make kSeedBlocks workgroups to a compute unit (with one row
// of the grid to a batch, two or three workgroups, 16 k seeds of 8 batches on 1 M nodes took 38 us a call, now 18, in a launch of their own 21, 65 k
// 111 / 51 / 54); of many batches one row is enough (192 of 16 k on 10 M nodes 308, with four rounds each 327).
constexpr int kSeedRounds = 4, kSeedBlocks = 4;

// bounds[r * (ranges + 1) + j] = first entry of run r with an id >= j * range, as an index into the batch's list.  Consecutive
// threads search one run for consecutive keys.  Bound by the lines the probes touch: ids sampled at random lie within a few
// sqrt(len) / 2 entries of their proportional place and a correction from there ends a few entries away, so about four lines
// per bound instead of the ten or more a bisection reads (any other run of ids only takes more steps): 295 k bounds in runs
// of up to 283 k entries 19 us, with a bisection of the 4 sqrt(len) entries around the proportional place 41.
// seed_batches: the first workgroups, seed_rows rows of them to a batch, count the seeds of so many batches meanwhile, whose atomics wait for
// memory where the searches wait for their probes: 192 batches of 1024 seeds, 393 k atomics, beside the 295 k bounds 29.6 us, in launches of their own 17.5 + 19.
__global__ void __launch_bounds__(256) k_hist_bounds(const int32_t* __restrict__ nodes, int64_t batch_stride,
                                                     const int32_t* __restrict__ tier_off, int num_hops, int64_t num_nodes, int range,
                                                     int ranges, int32_t* __restrict__ bounds, int seed_batches, int seed_rows,
                                                     uint32_t* __restrict__ counts, uint32_t* __restrict__ first_batch) {
    const int r = (int)blockIdx.y - seed_batches * seed_rows;
    if (r < 0) {
        int b = blockIdx.y, row = 0;
        for (; b >= seed_batches; b -= seed_batches) ++row;
        rg_count_seeds(nodes, batch_stride, tier_off, num_hops, b, row * gridDim.x + blockIdx.x, seed_rows * gridDim.x, counts, first_batch);
        return;
    }
    const int j = blockIdx.x * 256 + threadIdx.x;
    if (j > ranges) return;
    const int b = r / num_hops, t = r % num_hops + 1;                  // tier t of batch b
    const int32_t* to = tier_off + (int64_t)b * (num_hops + 2);
    const int begin = to[t], len = to[t + 1] - to[t];
    const int32_t* __restrict__ run = nodes + (int64_t)b * batch_stride + begin;
    const int64_t key = (int64_t)j * range;
    int lo = 0, hi = len;
    if (j == 0) hi = 0;
    if (j == ranges) lo = len;
    const double per_id = (double)len / (double)num_nodes;
    int at = (int)(per_id * (double)key);
    bool below = false;                                                // run[at] < key
    for (int step = 0; step < 3 && lo < hi; ++step) {                  // proportional place, then corrected by what is found there
        at = at < lo ? lo : (at >= hi ? hi - 1 : at);
        const int x = run[at];
        below = x < key;
        if (below) lo = at + 1; else hi = at;
        at += (int)(per_id * (double)(key - x));
    }
    for (int64_t g = 8; lo < hi; g *= 2) {                             // doubling steps away from there
        const int64_t p = below ? lo + g : hi - g;
        if (p < lo || p >= hi) break;
        const bool b2 = run[p] < key;
        if (b2) lo = (int)p + 1; else hi = (int)p;
        if (b2 != below) break;
    }
    while (lo < hi) {
        const int mid = (lo + hi) >> 1;
        if (run[mid] < key) lo = mid + 1; else hi = mid;
    }
    bounds[(int64_t)r * (ranges + 1) + j] = begin + lo;
}

// Batches and hops that a workgroup's 16 wavefronts, or a tile of runs, take it further, so that no wavefront divides for them.
struct RunStep {
    int wave_b, wave_t, tile_b, tile_t;
};

// FIRST: also record, per id, the smallest batch index whose list contains it (first_batch[v] = min(old, b)); b0 = index of the
// first of these batches.  bounds == NULL: the workgroup bisects every run for its range itself.
// AHEAD: a wavefront reads the next step's entries while it counts (see kHistAhead).
template <bool FIRST, bool AHEAD>
__global__ void __launch_bounds__(1024) k_histogram_runs(const int32_t* __restrict__ nodes, int64_t batch_stride,
                                                         const int32_t* __restrict__ tier_off, const int32_t* __restrict__ bounds,
                                                         int num_batches, int num_hops, int b0,
                                                         uint32_t* __restrict__ counts, uint32_t* __restrict__ first_batch,
                                                         int64_t num_nodes, int range, const RunStep by) {
    constexpr int U = 4;                                  // entries in flight per lane
    __shared__ uint32_t priv[kHistRangeMax];
    __shared__ uint32_t firstb[FIRST ? kHistRangeMax : 1];
    __shared__ int seg_lo[kHistRunTile];
    __shared__ int seg_hi[kHistRunTile];
    const int64_t v0 = (int64_t)blockIdx.x * range;
    const int64_t v1 = v0 + range < num_nodes ? v0 + range : num_nodes;
    for (int j = threadIdx.x; j < range; j += blockDim.x) {
        priv[j] = 0u;
        if (FIRST) firstb[j] = 0xFFFFFFFFu;
    }
    const int num_runs = num_batches * num_hops;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = rg_lane(), nwaves = blockDim.x >> 6;
    int tile_b = 0, tile_t = 0;                           // of run `tile`
    for (int tile = 0; tile < num_runs; tile += kHistRunTile) {
        __syncthreads();                                  // priv zeroed / previous tile's segments consumed
        const int r = tile + threadIdx.x;
        if (!bounds && threadIdx.x < kHistRunTile && r < num_runs) {
            const int b = r / num_hops, t = r % num_hops + 1;
            const int32_t* to = tier_off + (int64_t)b * (num_hops + 2);
            const int32_t* list = nodes + (int64_t)b * batch_stride;
            for (int side = 0; side < 2; ++side) {
                const int64_t key = v0 + (int64_t)side * range;
                int lo = to[t], hi = to[t + 1];
                while (lo < hi) {
                    const int mid = lo + (hi - lo) / 2;
                    if (list[mid] < key) lo = mid + 1; else hi = mid;
                }
                (side ? seg_hi : seg_lo)[threadIdx.x] = lo;
            }
        }
        if (bounds && threadIdx.x < kHistRunTile && r < num_runs) {
            const int32_t* at = bounds + (int64_t)r * (gridDim.x + 1) + blockIdx.x;
            seg_lo[threadIdx.x] = at[0];
            seg_hi[threadIdx.x] = at[1];
        }
        __syncthreads();
        const int in_tile = num_runs - tile < kHistRunTile ? num_runs - tile : kHistRunTile;
        if (!AHEAD) {
            for (int q = wave; q < in_tile; q += nwaves) {                  // one wavefront per run segment
                const int lo = __builtin_amdgcn_readfirstlane(seg_lo[q]), hi = __builtin_amdgcn_readfirstlane(seg_hi[q]);
                if (lo >= hi) continue;
                const int b = (tile + q) / num_hops;
                const int32_t* base = nodes + (int64_t)b * batch_stride;
                int e0 = lo + lane;
                if (hi - lo <= RG_WAVE) {                                   // short segments, of which a call may have mostly
                    const uint32_t off = e0 < hi ? (uint32_t)(base[e0] - (int)v0) : 0xFFFFFFFFu;
                    if (off < (uint32_t)range) {                            // always true inside an ascending segment
                        atomicAdd(&priv[off], 1u);
                        if (FIRST) atomicMin(&firstb[off], (uint32_t)(b0 + b));
                    }
                    continue;
                }
                for (; e0 < hi; e0 += RG_WAVE * U) {
                    uint32_t off[U];
#pragma unroll
                    for (int u = 0; u < U; ++u) off[u] = e0 + RG_WAVE * u < hi ? (uint32_t)(base[e0 + RG_WAVE * u] - (int)v0) : 0xFFFFFFFFu;
#pragma unroll
                    for (int u = 0; u < U; ++u)
                        if (off[u] < (uint32_t)range) {
                            atomicAdd(&priv[off[u]], 1u);
                            if (FIRST) atomicMin(&firstb[off[u]], (uint32_t)(b0 + b));
                        }
                }
            }
            continue;
        }
        // One wavefront per run segment, 64 * U entries a step.  The entries of its next step are on their way while it counts: lanes
        // behind the segment's end read its last entry again, and behind the last segment something else that is there, so that
        // every step has the same loads in flight and the wait for one does not take in the other's.
        int q = wave - nwaves, e = 0, hi = 0;
        int b = tile_b, t = tile_t + wave;                                // batch and hop of run tile + q + nwaves, without dividing for them
        while (t >= num_hops) { t -= num_hops; ++b; }
        int at = 0;                                                       // batch of the segment
        const int32_t* base = tier_off;
        const auto advance = [&](int& left, int& batch) {
            while (e >= hi && q < in_tile) {
                q += nwaves;
                if (q < in_tile) {
                    e = __builtin_amdgcn_readfirstlane(seg_lo[q]);
                    hi = __builtin_amdgcn_readfirstlane(seg_hi[q]);
                    at = b;
                    base = nodes + (int64_t)at * batch_stride;
                    b += by.wave_b;
                    t += by.wave_t;
                    if (t >= num_hops) { t -= num_hops; ++b; }
                } else {
                    base = tier_off;
                    e = hi = 0;
                }
            }
            left = hi - e;
            batch = b0 + at;
        };
        const auto fetch = [&](uint32_t (&id)[U], int left) {
            const int last = left > 0 ? left - 1 : 0;
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const int i = RG_WAVE * u + lane;
                id[u] = (uint32_t)base[e + (i < last ? i : last)];
            }
            e = e + RG_WAVE * U < hi ? e + RG_WAVE * U : hi;
        };
        const auto count = [&](const uint32_t (&id)[U], int left, int batch) {
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const uint32_t off = id[u] - (uint32_t)v0;
                if (RG_WAVE * u + lane < left && off < (uint32_t)range) {            // (always in the range inside an ascending segment)
                    atomicAdd(&priv[off], 1u);
                    if (FIRST) atomicMin(&firstb[off], (uint32_t)batch);
                }
            }
        };
        uint32_t x[U], y[U];
        int bx, bz, nx, ny;
        advance(nx, bx);
        if (nx > 0) fetch(x, nx);                                         // (most wavefronts of many short runs have nothing to read)
        while (nx > 0) {
            advance(ny, bz);
            fetch(y, ny);
            count(x, nx, bx);
            if (ny <= 0) break;
            advance(nx, bx);
            fetch(x, nx);
            count(y, ny, bz);
        }
        tile_b += by.tile_b;
        tile_t += by.tile_t;
        if (tile_t >= num_hops) { tile_t -= num_hops; ++tile_b; }
    }
    __syncthreads();
    for (int64_t j = threadIdx.x; v0 + j < v1; j += blockDim.x) {
        const uint32_t c = priv[j];
        if (c) {
            counts[v0 + j] += c;
            if (FIRST) { const uint32_t f = firstb[j], g = first_batch[v0 + j]; if (f < g) first_batch[v0 + j] = f; }
        }
    }
}

// ---------------------------------------------------------------------------- threshold select
// Finds the count threshold T of the K_eff-th best candidate.  Access counts are bounded by the number of batches of
// the period (a few hundred), so one streaming pass with a histogram of the counts clamped to kLowBins - 1 resolves T
// whenever T < kLowBins - 1, and its last workgroup says so.  Only when the K_eff-th best candidate sits in the clamped last bin do
// the passes of a most-significant-digit-first radix select (11 + 11 + 10 bits, the first of them by the streaming pass) run; otherwise their kernels return at once.
// What they find stays in TopkCtl and is read off there by the kernels up to the count (rg_topk_state).
// Bound by launches: with four passes of 8 bits, every kernel working out the state from the bins for itself and the bins cleared by a
// launch in front, selection at 2.4 M nodes took 60 us, now 37 (at 10 M nodes 107, now 70; at 40 M 362, now 239).  The emit clears them for the next call.
constexpr int kLowBins = 2048;
constexpr int kBallotBins = 4;       // counts 1..kBallotBins are tallied with wave ballots instead of LDS atomics

struct TopkState {
    uint32_t T;          // the threshold (while radix passes are open: its resolved high bytes)
    uint32_t need;       // how many of the candidates tied with T are to be taken
    uint32_t k_eff;
    uint32_t resolved;   // 1: T and need are final without radix passes
};

constexpr int kRadixPasses = 3;
constexpr int kRadixBins = 2048;
struct TopkCtl {                     // everything up to `low_state` is zero in front of a selection
    uint32_t hist[kRadixPasses][kRadixBins];
    uint32_t low[kLowBins];          // candidates per clamped count
    unsigned long long ovf_sum;      // sum of the counts of the candidates in the last (clamped) bin
    uint32_t done, pad;              // workgroups of k_topk_hist_low that have added theirs
    TopkState low_state;             // from `low` alone, by the last of them
    TopkState state;                 // as k_topk_count found it
};
constexpr int kCtlClear = offsetof(TopkCtl, low_state) / 4;

// Digit `pass` of a count, and the bits in front of it.
__device__ __forceinline__ int rg_radix_shift(int pass) { return pass == 0 ? 21 : (pass == 1 ? 10 : 0); }
__device__ __forceinline__ uint32_t rg_radix_digit(uint32_t c, int pass) { return (c >> rg_radix_shift(pass)) & (pass == 2 ? 1023u : 2047u); }
__device__ __forceinline__ uint32_t rg_radix_front(uint32_t c, int pass) { return pass == 0 ? 0u : c >> (pass == 1 ? 21 : 10); }

__device__ __forceinline__ bool rg_is_candidate(uint32_t home_word, uint32_t count) {
    return (home_word >> RG_TAG_SHIFT) == RG_TAG_REMOTE && count >= 1u;
}

__global__ void __launch_bounds__(256) k_topk_init(TopkCtl* __restrict__ ctl, int hist_only) {
    uint32_t* w = (uint32_t*)ctl;
    const int n = hist_only ? (int)(sizeof(ctl->hist) / 4) : kCtlClear;              // hist_only: a later selection of the hit curve, the same first digits
    for (int i = (hist_only ? kRadixBins : 0) + blockIdx.x * 256 + threadIdx.x; i < n; i += gridDim.x * 256) w[i] = 0u;
}

// The bin of one of 2048 that holds the need-th best, bins in descending order, `n` of them in bin h[j] of this thread
// (bins 2047 - PER * t downwards): its index, and through `need` how many of it are wanted.  Every thread of the workgroup calls it.
template <int NT>
__device__ __forceinline__ void rg_pick_bin(const uint32_t (&h)[kRadixBins / NT], uint32_t need, int* smem, uint32_t* bin_s, uint32_t* need_s) {
    constexpr int PER = kRadixBins / NT;
    int mine = 0;
#pragma unroll
    for (int j = 0; j < PER; ++j) mine += (int)h[j];
    int total;
    uint32_t above = (uint32_t)rg_block_excl_scan<NT / RG_WAVE>(mine, smem, &total);
#pragma unroll
    for (int j = 0; j < PER; ++j) {
        if (above < need && need <= above + h[j]) {                       // exactly one bin satisfies this
            *bin_s = (uint32_t)(kRadixBins - 1 - (PER * (int)threadIdx.x + j));
            *need_s = need - above;
        }
        above += h[j];
    }
    __syncthreads();
}

// K_eff = min(capacity, #candidates) and its threshold as far as the low histogram knows it.
template <int NT>
__device__ __forceinline__ TopkState rg_low_state(const TopkCtl* ctl, int64_t capacity) {
    static_assert(kLowBins == kRadixBins, "one way to look a bin up");
    __shared__ int smem[NT / RG_WAVE + 1];
    __shared__ uint32_t bin, need;
    constexpr int PER = kLowBins / NT;
    uint32_t h[PER];
    int mine = 0, total;
#pragma unroll
    for (int j = 0; j < PER; ++j) {      // (the last workgroup of k_topk_hist_low reads what others have just added)
        h[j] = __hip_atomic_load(&ctl->low[kLowBins - 1 - (PER * (int)threadIdx.x + j)], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        mine += (int)h[j];
    }
    (void)rg_block_excl_scan<NT / RG_WAVE>(mine, smem, &total);
    const uint64_t k = (uint64_t)capacity < (uint64_t)total ? (uint64_t)capacity : (uint64_t)total;
    if (k == 0) return TopkState{0xFFFFFFFFu, 0u, 0u, 1u};                // uniform; a threshold no count reaches
    rg_pick_bin<NT>(h, (uint32_t)k, smem, &bin, &need);
    return bin < (uint32_t)(kLowBins - 1) ? TopkState{bin, need, (uint32_t)k, 1u}
                                          : TopkState{0u, (uint32_t)k, (uint32_t)k, 0u};      // the clamped bin: radix passes decide
}

// The same with what the first `passes` radix histograms say where the low one leaves it open.
template <int NT>
__device__ __forceinline__ TopkState rg_topk_state(const TopkCtl* ctl, TopkState st, int passes) {
    __shared__ int smem[NT / RG_WAVE + 1];
    __shared__ uint32_t bin, need;
    constexpr int PER = kRadixBins / NT;
    if (st.resolved) return st;                                           // uniform
    for (int pass = 0; pass < passes; ++pass) {
        uint32_t h[PER];
#pragma unroll
        for (int j = 0; j < PER; ++j) h[j] = ctl->hist[pass][kRadixBins - 1 - (PER * (int)threadIdx.x + j)];
        rg_pick_bin<NT>(h, st.need, smem, &bin, &need);
        st.T |= bin << rg_radix_shift(pass);
        st.need = need;
        __syncthreads();
    }
    return st;
}

// Four consecutive words from i on, 0 behind the end: one 16-byte access where the array and all four allow it.
__device__ __forceinline__ void rg_load4(const void* __restrict__ p, int64_t i, int64_t n, uint32_t (&x)[4]) {
    const uint32_t* w = (const uint32_t*)p;
    if (((uintptr_t)w & 15u) == 0u && i + 3 < n) {
        const uint4 v = *(const uint4*)(w + i);
        x[0] = v.x; x[1] = v.y; x[2] = v.z; x[3] = v.w;
    } else {
#pragma unroll
        for (int q = 0; q < 4; ++q) x[q] = i + q < n ? w[i + q] : 0u;
    }
}

// low[min(count, kLowBins - 1)] += 1 for every candidate; ovf_sum += count for those in the last bin, and the histogram of their first
// digits, with which the radix select begins where the threshold is one of them.  One workgroup per
// compute unit: with more of them their additions to the same few bins queue up (1196 workgroups 38 us at 2.4 M nodes).  Above
// 8 Mi nodes two, which read faster: the selection at 10 M nodes 110 -> 104 us, at 40 M 412 -> 364, at 100 M 972 -> 858.
__global__ void __launch_bounds__(1024) k_topk_hist_low(const uint32_t* __restrict__ counts, const int32_t* __restrict__ home, int64_t n,
                                                        TopkCtl* ctl, int64_t capacity) {
    constexpr int U = 4;
    __shared__ uint32_t h[kLowBins], top[kRadixBins];
    __shared__ int last_s;
    __shared__ unsigned long long ovf_s;
    for (int i = threadIdx.x; i < kLowBins; i += 1024) h[i] = top[i] = 0u;
    if (threadIdx.x == 0) ovf_s = 0ull;
    __syncthreads();
    unsigned long long ovf = 0ull;
    const int lane = rg_lane();
    for (int64_t v0 = (int64_t)blockIdx.x * (1024 * U); v0 < n; v0 += (int64_t)gridDim.x * (1024 * U)) {   // uniform per workgroup
        uint32_t c[U], hw[U];
        rg_load4(counts, v0 + 4 * threadIdx.x, n, c);
        rg_load4(home, v0 + 4 * threadIdx.x, n, hw);
#pragma unroll
        for (int u = 0; u < U; ++u) {
            uint32_t bin = 0u;                               // bin 0: not a candidate
            if (rg_is_candidate(hw[u], c[u])) {
                bin = c[u] < (uint32_t)(kLowBins - 1) ? c[u] : (uint32_t)(kLowBins - 1);
                if (c[u] >= (uint32_t)(kLowBins - 1)) {
                    ovf += c[u];
                    atomicAdd(&top[rg_radix_digit(c[u], 0)], 1u);
                }
            }
            // most candidates of a long-tailed distribution have a count of 1..4: one LDS atomic per wavefront for each
#pragma unroll
            for (uint32_t q = 1; q <= (uint32_t)kBallotBins; ++q) {
                const unsigned long long m = __ballot(bin == q);
                if (lane == 0 && m) atomicAdd(&h[q], (uint32_t)__popcll(m));
            }
            if (bin > (uint32_t)kBallotBins) atomicAdd(&h[bin], 1u);
        }
    }
    if (ovf) atomicAdd(&ovf_s, ovf);
    __syncthreads();
    for (int i = threadIdx.x; i < kLowBins; i += 1024) {
        const uint32_t mine = h[i];
        // The last workgroup reads what the others have added without a fence, which writes back the L2 and took 65 us.  That holds
        // because low[] is touched in this kernel by additions and loads of agent scope alone, which are made where every XCD sees
        // them, and because an addition whose old value has arrived has been made: `done` is raised behind the wait for those values
        // (and the barrier below).  A plain store, or one of a smaller scope, to something the last workgroup reads would need the fence.
        if (mine) { const uint32_t old = atomicAdd(&ctl->low[i], mine); asm volatile("" :: "v"(old) : "memory"); }
    }
    if (threadIdx.x == 0 && ovf_s) atomicAdd(&ctl->ovf_sum, ovf_s);
    if (ovf_s)                                               // uniform; read by launches behind this one
        for (int i = threadIdx.x; i < kRadixBins; i += 1024)
            if (top[i]) atomicAdd(&ctl->hist[0][i], top[i]);
    if (capacity < 0) return;                                             // the hit curve looks its capacities up itself
    __syncthreads();                                                      // every addition of this workgroup is made
    if (threadIdx.x == 0) last_s = atomicAdd(&ctl->done, 1u) == gridDim.x - 1;
    __syncthreads();
    if (!last_s) return;                                                  // uniform
    const TopkState st = rg_low_state<1024>(ctl, capacity);
    if (threadIdx.x == 0) ctl->low_state = st;
}

// Histogram of digit `pass` (1 or 2; 0, the most significant, is k_topk_hist_low's) of the counts of candidates that match the digits in front.  skip: of the hit curve, a
// flag that, when set, says that nobody asks for it; NULL: the low state is there.
__global__ void __launch_bounds__(1024) k_topk_hist(const uint32_t* __restrict__ counts, const int32_t* __restrict__ home, int64_t n,
                                                   int pass, int64_t capacity, TopkCtl* ctl, const uint32_t* __restrict__ skip) {
    __shared__ uint32_t h[kRadixBins];
    if (skip ? *skip : ctl->low_state.resolved) return;      // uniform
    const TopkState st = rg_topk_state<1024>(ctl, skip ? rg_low_state<1024>(ctl, capacity) : ctl->low_state, pass);
    if (st.resolved) return;                                 // uniform
    for (int i = threadIdx.x; i < kRadixBins; i += 1024) h[i] = 0u;
    __syncthreads();
    const uint32_t front = rg_radix_front(st.T, pass);
    for (int64_t v = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; v < n; v += (int64_t)gridDim.x * blockDim.x) {
        const uint32_t c = counts[v];
        if (!rg_is_candidate((uint32_t)home[v], c) || rg_radix_front(c, pass) != front) continue;
        atomicAdd(&h[rg_radix_digit(c, pass)], 1u);
    }
    __syncthreads();
    for (int i = threadIdx.x; i < kRadixBins; i += 1024)
        if (h[i]) atomicAdd(&ctl->hist[pass][i], h[i]);
}

constexpr int kCapChunk = 64;
struct CapChunk { int64_t v[kCapChunk]; };

__global__ void k_store_caps(int64_t* __restrict__ dst, const CapChunk chunk, int count) {
    if ((int)threadIdx.x < count) dst[threadIdx.x] = chunk.v[threadIdx.x];
}

// One workgroup, after k_topk_hist_low: requests served by a cache of each capacity, read off the histogram.
// hits[j] = sum of the counts above the threshold of capacity j + (ties taken) x threshold.  A capacity whose
// threshold lies inside the clamped last bin is left to the radix passes: radix_flag[j] = 0 ("not resolved").
// Bound by latency: all bins are read at once and joined by two scans (read in turn by one thread the kernel took 60-80 us; now the whole
// call without capacities takes 26 us at 1 M nodes, of which 25 are the host's).
__global__ void __launch_bounds__(256) k_hit_curve_low(const TopkCtl* __restrict__ ctl, const int64_t* __restrict__ capacities,
                                                       int num_capacities, unsigned long long* __restrict__ hits,
                                                       unsigned long long* __restrict__ total_out, uint32_t* __restrict__ resolved_flag) {
    constexpr int PER = kLowBins / 256;                      // thread t owns bins kLowBins-1-PER*t downwards
    __shared__ uint32_t cnt_above[kLowBins];                 // candidates with a larger clamped count
    __shared__ unsigned long long sum_above[kLowBins];       // and the sum of their counts
    __shared__ unsigned long long part[256];
    __shared__ int smem[256 / RG_WAVE + 1];
    const int top = kLowBins - 1 - PER * (int)threadIdx.x;
    uint32_t h[PER];
    unsigned long long w[PER], sum = 0ull;
    int cnt = 0, total;
#pragma unroll
    for (int j = 0; j < PER; ++j) {
        const int bin = top - j;                             // bin 0 is empty
        h[j] = ctl->low[bin];
        w[j] = bin == kLowBins - 1 ? ctl->ovf_sum : (unsigned long long)h[j] * (unsigned long long)bin;
        cnt += (int)h[j];
        sum += w[j];
    }
    uint32_t above = (uint32_t)rg_block_excl_scan<256 / RG_WAVE>(cnt, smem, &total);
    part[threadIdx.x] = sum;
    for (int off = 1; off < 256; off <<= 1) {
        __syncthreads();
        const unsigned long long x = (int)threadIdx.x >= off ? part[threadIdx.x - off] : 0ull;
        __syncthreads();
        part[threadIdx.x] += x;
    }
    __syncthreads();
    const unsigned long long grand = part[255];
    sum = part[threadIdx.x] - sum;
#pragma unroll
    for (int j = 0; j < PER; ++j) {
        cnt_above[top - j] = above;
        sum_above[top - j] = sum;
        above += h[j];
        sum += w[j];
    }
    if (threadIdx.x == 0 && total_out) *total_out = grand;
    __syncthreads();
    const uint32_t n_cand = (uint32_t)total;
    for (int j = threadIdx.x; j < num_capacities; j += 256) {
        const uint64_t cap = (uint64_t)capacities[j];
        const uint32_t k = cap < (uint64_t)n_cand ? (uint32_t)cap : n_cand;
        if (k == 0u) { hits[j] = 0ull; resolved_flag[j] = 1u; continue; }
        if (k == n_cand) { hits[j] = grand; resolved_flag[j] = 1u; continue; }
        // the threshold bin T holds the k-th best candidate: cnt_above[T] < k <= cnt_above[T - 1].  cnt_above falls as
        // the bin index rises and cnt_above[kLowBins - 1] = 0 < k, so T is the smallest bin with cnt_above[T] < k.
        int lo = 1, hi = kLowBins - 1;
        while (lo < hi) {
            const int mid = (lo + hi) >> 1;
            if (cnt_above[mid] < k) hi = mid; else lo = mid + 1;
        }
        if (lo == kLowBins - 1) { hits[j] = 0ull; resolved_flag[j] = 0u; continue; }
        hits[j] = sum_above[lo] + (unsigned long long)(k - cnt_above[lo]) * (unsigned long long)lo;
        resolved_flag[j] = 1u;
    }
}

constexpr int kNodesPerBlock = 4096;   // 1024 threads x 4 consecutive nodes
constexpr int kTopkSelfScan = 4096;    // blocks up to which the emit kernel adds up the totals in front of it itself (N <= 16 Mi)

// Per block: number of candidates above the threshold and number tied with it; the number of rows selected.
__global__ void __launch_bounds__(1024) k_topk_count(const uint32_t* __restrict__ counts, const int32_t* __restrict__ home, int64_t n,
                                                     TopkCtl* ctl, int32_t* __restrict__ blk_gt,
                                                     int32_t* __restrict__ blk_eq, int64_t* __restrict__ num_cached) {
    __shared__ int part[1024 / RG_WAVE];
    const int64_t v0 = (int64_t)blockIdx.x * kNodesPerBlock + threadIdx.x * 4;
    uint32_t c[4], hw[4];
    bool cand[4];
    rg_load4(counts, v0, n, c);
    rg_load4(home, v0, n, hw);
#pragma unroll
    for (int q = 0; q < 4; ++q) cand[q] = v0 + q < n && rg_is_candidate(hw[q], c[q]);
    const TopkState st = rg_topk_state<1024>(ctl, ctl->low_state, kRadixPasses);
    int both = 0;                                            // above the threshold << 16 | tied with it: at most 4096 of either
#pragma unroll
    for (int q = 0; q < 4; ++q) both += cand[q] ? (c[q] > st.T ? 1 << 16 : c[q] == st.T) : 0;
    both = rg_wave_sum(both);
    if (rg_lane() == 0) part[threadIdx.x >> 6] = both;
    __syncthreads();
    if (threadIdx.x == 0) {
        both = 0;
#pragma unroll
        for (int w = 0; w < 1024 / RG_WAVE; ++w) both += part[w];
        blk_gt[blockIdx.x] = both >> 16;
        blk_eq[blockIdx.x] = both & 0xFFFF;
        if (blockIdx.x == 0) { *num_cached = (int64_t)st.k_eff; ctl->state = st; }
    }
}

// One workgroup: exclusive scans of both per-block arrays, in place.
__global__ void __launch_bounds__(1024) k_topk_scan(int32_t* __restrict__ blk_gt, int32_t* __restrict__ blk_eq, int64_t nblocks) {
    __shared__ int smem[1024 / RG_WAVE + 1];
    int carry_g = 0, carry_e = 0;
    for (int64_t base = 0; base < nblocks; base += 1024) {
        const int64_t i = base + threadIdx.x;
        const int g = i < nblocks ? blk_gt[i] : 0;
        const int e = i < nblocks ? blk_eq[i] : 0;
        int tg, te;
        const int xg = rg_block_excl_scan<1024 / RG_WAVE>(g, smem, &tg);
        const int xe = rg_block_excl_scan<1024 / RG_WAVE>(e, smem, &te);
        if (i < nblocks) { blk_gt[i] = carry_g + xg; blk_eq[i] = carry_e + xe; }
        carry_g += tg;
        carry_e += te;
    }
}

// Selected = above the threshold, or tied with it and among the first `need` ties in id order.
// Slots are handed out in ascending id, so cache_ids comes out sorted.  scanned: the per-block counts are exclusive prefixes
// already.  filled (NULL: left alone): bit s = `resident` for every selected slot, 0 behind them.
__global__ void __launch_bounds__(1024) k_topk_emit(const uint32_t* __restrict__ counts, const int32_t* __restrict__ home, int64_t n,
                                                    TopkCtl* ctl, const int32_t* __restrict__ blk_gt,
                                                    const int32_t* __restrict__ blk_eq, int scanned, int32_t* __restrict__ cache_ids,
                                                    int32_t* __restrict__ loc, uint32_t* __restrict__ filled, int64_t filled_words,
                                                    int resident) {
    constexpr int NW = 1024 / RG_WAVE;
    __shared__ int smem[NW + 1];
    __shared__ int pg[NW], pe[NW];
    const int64_t v0 = (int64_t)blockIdx.x * kNodesPerBlock + threadIdx.x * 4;
    uint32_t hw[4], c[4];
    rg_load4(counts, v0, n, c);
    rg_load4(home, v0, n, hw);
    int gt_before = 0, eq_before = 0;
    if (scanned) {
        gt_before = blk_gt[blockIdx.x];
        eq_before = blk_eq[blockIdx.x];
    } else {
        for (unsigned b = threadIdx.x; b < blockIdx.x; b += 1024) { gt_before += blk_gt[b]; eq_before += blk_eq[b]; }
        gt_before = rg_wave_sum(gt_before);
        eq_before = rg_wave_sum(eq_before);
        if (rg_lane() == 0) { pg[threadIdx.x >> 6] = gt_before; pe[threadIdx.x >> 6] = eq_before; }
        __syncthreads();
        gt_before = eq_before = 0;
#pragma unroll
        for (int w = 0; w < NW; ++w) { gt_before += pg[w]; eq_before += pe[w]; }
    }
    const TopkState st = ctl->state;
    for (int i = blockIdx.x * 1024 + threadIdx.x; i < kCtlClear; i += gridDim.x * 1024) ((uint32_t*)ctl)[i] = 0u;      // for the next call
    const int need = (int)st.need;
    if (filled) {
        for (int64_t w = (int64_t)blockIdx.x * 1024 + threadIdx.x; w < filled_words; w += (int64_t)gridDim.x * 1024) {
            uint32_t bits = 0u;
            const int64_t lo = w * 32, k = st.k_eff;
            if (resident) bits = k >= lo + 32 ? 0xFFFFFFFFu : (k > lo ? (1u << (uint32_t)(k - lo)) - 1u : 0u);
            filled[w] = bits;
        }
    }
    bool is_gt[4], is_eq[4];
    int both = 0;                                            // above the threshold << 16 | tied with it: at most 4096 of either
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        const bool cand = v0 + q < n && rg_is_candidate(hw[q], c[q]);
        is_gt[q] = cand && c[q] > st.T;
        is_eq[q] = cand && c[q] == st.T;
        both += is_gt[q] ? 1 << 16 : is_eq[q];
    }
    int tot;
    both = rg_block_excl_scan<NW>(both, smem, &tot);
    int eq_rank = eq_before + (both & 0xFFFF);
    int slot = gt_before + (both >> 16) + (eq_rank < need ? eq_rank : need);       // every tie in front of this node that was taken
    bool sel[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        sel[q] = is_gt[q] || (is_eq[q] && eq_rank < need);
        eq_rank += is_eq[q];
    }
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        const int64_t v = v0 + q;
        if (sel[q]) {
            cache_ids[slot] = (int32_t)v;
            hw[q] = (RG_TAG_CACHE << RG_TAG_SHIFT) | (uint32_t)slot;
            ++slot;
        }
    }
    if (((uintptr_t)loc & 15u) == 0u && v0 + 3 < n) {
        *(uint4*)(loc + v0) = make_uint4(hw[0], hw[1], hw[2], hw[3]);
    } else {
#pragma unroll
        for (int q = 0; q < 4; ++q)
            if (v0 + q < n) loc[v0 + q] = (int32_t)hw[q];
    }
}

// Radix path of the hit curve: hits += sum of the counts above the threshold plus (ties taken) x threshold.
// `resolved` = 1 when the histogram pass already produced this capacity's value.
__global__ void __launch_bounds__(256) k_hit_sum(const uint32_t* __restrict__ counts, const int32_t* __restrict__ home, int64_t n,
                                                 const TopkCtl* ctl, int64_t capacity, const uint32_t* __restrict__ resolved,
                                                 unsigned long long* __restrict__ hits) {
    if (*resolved) return;                                   // uniform
    const TopkState st = rg_topk_state<256>(ctl, rg_low_state<256>(ctl, capacity), kRadixPasses);
    const uint32_t T = st.T;
    unsigned long long above = 0ull;
    for (int64_t v = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; v < n; v += (int64_t)gridDim.x * blockDim.x) {
        const uint32_t c = counts[v];
        if (rg_is_candidate((uint32_t)home[v], c) && c > T) above += c;
    }
#pragma unroll
    for (int off = RG_WAVE / 2; off > 0; off >>= 1) above += __shfl_xor(above, off, RG_WAVE);
    __shared__ unsigned long long pa[4];
    if (rg_lane() == 0) pa[threadIdx.x >> 6] = above;
    __syncthreads();
    if (threadIdx.x == 0) {
        unsigned long long a = pa[0] + pa[1] + pa[2] + pa[3];
        if (blockIdx.x == 0) a += (unsigned long long)st.need * (unsigned long long)T;   // need == 0 when nothing is selected
        if (a) atomicAdd(hits, a);
    }
}

// ---------------------------------------------------------------------------- VectorPull
// cache_rows[slot] = remote_store[row(home[cache_ids[slot]])] for slot < *num_cached.
template <int VEC>
__global__ void __launch_bounds__(256) k_cache_fill(const int32_t* __restrict__ cache_ids, const int32_t* __restrict__ home,
                                                    const int64_t* __restrict__ num_cached, const float* __restrict__ remote_store,
                                                    int64_t remote_stride, float* __restrict__ cache_rows, int64_t cache_stride,
                                                    int cpr, int log2L, int tail) {
    typedef typename RgVec<VEC>::type V;
    constexpr int U = 4;
    const int64_t n = *num_cached;
    const int lane = rg_lane();
    const int L = 1 << log2L;
    const int R = RG_WAVE >> log2L;            // rows per wave step
    const int sub = lane >> log2L;
    const int c0 = lane & (L - 1);
    const int64_t wave = ((int64_t)blockIdx.x * blockDim.x + threadIdx.x) >> 6;
    const int64_t nwaves = ((int64_t)gridDim.x * blockDim.x) >> 6;
    for (int64_t row0 = wave * (R * U); row0 < n; row0 += nwaves * (R * U)) {
        const V* src[U];
        V* dst[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int64_t slot = row0 + u * R + sub;
            src[u] = nullptr;
            dst[u] = nullptr;
            if (slot < n) {
                const uint32_t hw = (uint32_t)home[cache_ids[slot]];
                src[u] = (const V*)(remote_store + (int64_t)(hw & RG_ROW_MASK) * remote_stride);
                dst[u] = (V*)(cache_rows + slot * cache_stride);
            }
        }
        for (int c = c0; c < cpr; c += L) {
            V val[U];
#pragma unroll
            for (int u = 0; u < U; ++u)
                if (src[u]) val[u] = src[u][c];
            const bool head_only = tail < VEC && c == cpr - 1;      // only the row's own floats of its last chunk are stored
#pragma unroll
            for (int u = 0; u < U; ++u)
                if (dst[u]) {
                    if (head_only) rg_store_head(&dst[u][c], val[u], tail);
                    else dst[u][c] = val[u];
                }
        }
    }
}

__global__ void k_prefetch_reset(uint32_t* __restrict__ pctl) {
    if (threadIdx.x == 0) pctl[0] = 0u;
}

// For every listed node whose location word names a cache slot that is not yet resident: claim the slot
// (atomic test-and-set of its bit) and append (slot, remote row) to the pull list.
__global__ void __launch_bounds__(256) k_prefetch_select(const int32_t* __restrict__ nodes, int64_t n, const int32_t* __restrict__ n_dev,
                                                         const int32_t* __restrict__ loc, const int32_t* __restrict__ home,
                                                         uint32_t* __restrict__ filled, int32_t* __restrict__ list,
                                                         uint32_t* __restrict__ pctl, int mirror) {
    __shared__ int smem[256 / RG_WAVE + 1];
    __shared__ uint32_t base_s;
    int64_t n_act = n;
    if (n_dev) { const int64_t d = *n_dev; n_act = d < n ? d : n; }
    if ((int64_t)blockIdx.x * blockDim.x >= n_act) return;        // uniform per workgroup
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    int take = 0;
    uint32_t slot = 0u, rrow = 0u;
    if (i < n_act) {
        const int32_t v = nodes[i];
        bool wanted;
        if (mirror) {       // every remote row a batch names will be cached, at the row it has in the remote store
            const uint32_t hw = (uint32_t)home[v];
            wanted = (hw >> RG_TAG_SHIFT) == RG_TAG_REMOTE;
            slot = rrow = hw & RG_ROW_MASK;
        } else {
            const uint32_t w = (uint32_t)loc[v];
            wanted = (w >> RG_TAG_SHIFT) == RG_TAG_CACHE;
            slot = w & RG_ROW_MASK;
        }
        if (wanted) {
            const uint32_t bit = 1u << (slot & 31u);
            if (!(filled[slot >> 5] & bit)) {
                const uint32_t old = atomicOr(&filled[slot >> 5], bit);
                if (!(old & bit)) { take = 1; rrow = (uint32_t)home[v] & RG_ROW_MASK; }
            }
        }
    }
    int total;
    const int excl = rg_block_excl_scan<256 / RG_WAVE>(take, smem, &total);
    if (total == 0) return;                                        // uniform
    if (threadIdx.x == 0) base_s = atomicAdd(&pctl[0], (uint32_t)total);
    __syncthreads();
    if (take) {
        const int64_t j = (int64_t)base_s + excl;
        list[2 * j] = (int32_t)slot;
        list[2 * j + 1] = (int32_t)rrow;
    }
}

// dst_rows[list[2j]] = src_rows[list[2j+1]] for every pair of the list (host link or HBM source alike); with `mark` the
// destination rows' resident bits are set by the same kernel.
// The pairs are list[0..pctl[0]) or, when seg_off is given, list[seg_off[0]..seg_off[1]).
template <int VEC, int U>
__global__ void __launch_bounds__(1024) k_prefetch_pull(const int32_t* __restrict__ list, const uint32_t* __restrict__ pctl,
                                                       const int32_t* __restrict__ seg_off,
                                                       const float* __restrict__ remote_store, int64_t remote_stride,
                                                       float* __restrict__ cache_rows, int64_t cache_stride, int64_t dst_rows,
                                                       int cpr, int log2L, int tail, uint32_t* __restrict__ mark) {
    typedef typename RgVec<VEC>::type V;
    int64_t n;
    if (seg_off) { list += 2 * (int64_t)seg_off[0]; n = seg_off[1] - seg_off[0]; } else { n = pctl[0]; }
    const int lane = rg_lane();
    const int L = 1 << log2L;
    const int R = RG_WAVE >> log2L;
    const int sub = lane >> log2L;
    const int c0 = lane & (L - 1);
    const int64_t wave = ((int64_t)blockIdx.x * blockDim.x + threadIdx.x) >> 6;
    const int64_t nwaves = ((int64_t)gridDim.x * blockDim.x) >> 6;
    for (int64_t j0 = wave * (R * U); j0 < n; j0 += nwaves * (R * U)) {
        // Few wavefronts feed the link, so each must keep all U row loads in flight: the loads are unconditional
        // (a lane group without a row reads destination row 0, which is in HBM and costs no link traffic; the value
        // is discarded) and only the stores are predicated.
        const V* src[U];
        V* dst[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int64_t j = j0 + u * R + sub;
            src[u] = (const V*)cache_rows;
            dst[u] = nullptr;
            if (j < n) {
                const int64_t slot = list[2 * j], rrow = list[2 * j + 1];
                if (slot >= 0 && slot < dst_rows) {      // a list built for another destination must not write outside this one
                    src[u] = (const V*)(remote_store + rrow * remote_stride);
                    dst[u] = (V*)(cache_rows + slot * cache_stride);
                    // the row's resident bit, by the first lane of its group (whoever reads the bits waits for this kernel)
                    if (mark && c0 == 0) atomicOr(&mark[slot >> 5], 1u << (slot & 31));
                }
            }
        }
        for (int c = c0; c < cpr; c += L) {
            V val[U];
#pragma unroll
            for (int u = 0; u < U; ++u) val[u] = src[u][c];
            const bool head_only = tail < VEC && c == cpr - 1;
#pragma unroll
            for (int u = 0; u < U; ++u)
                if (dst[u]) {
                    if (head_only) rg_store_head(&dst[u][c], val[u], tail);
                    else dst[u][c] = val[u];
                }
        }
    }
}

// ---------------------------------------------------------------------------- prefetch plan
// counters[b + 1] += 1 for every selected slot whose node is first used by batch b (b = num_batches: by none).
__global__ void __launch_bounds__(256) k_plan_count(const int32_t* __restrict__ cache_ids, const int64_t* __restrict__ num_cached,
                                                    const uint32_t* __restrict__ first_batch, int num_batches,
                                                    int32_t* __restrict__ counters) {
    const int64_t k = *num_cached;
    for (int64_t s = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; s < k; s += (int64_t)gridDim.x * blockDim.x) {
        const uint32_t f = first_batch[cache_ids[s]];
        atomicAdd(&counters[(f < (uint32_t)num_batches ? (int)f : num_batches) + 1], 1);
    }
}

// One workgroup: offsets[0] = 0, offsets[b + 1] = inclusive prefix of the counters; cursor[b] = offsets[b].
__global__ void __launch_bounds__(1024) k_plan_scan(int32_t* __restrict__ offsets, int32_t* __restrict__ cursor, int n_seg) {
    __shared__ int smem[1024 / RG_WAVE + 1];
    __shared__ int carry_s;
    if (threadIdx.x == 0) { carry_s = 0; offsets[0] = 0; }
    __syncthreads();
    for (int base = 0; base < n_seg; base += 1024) {
        const int i = base + threadIdx.x;
        const int x = i < n_seg ? offsets[i + 1] : 0;
        int total;
        const int excl = rg_block_excl_scan<1024 / RG_WAVE>(x, smem, &total);
        const int carry = carry_s;
        if (i < n_seg) { offsets[i + 1] = carry + excl + x; cursor[i] = carry + excl; }
        __syncthreads();
        if (threadIdx.x == 0) carry_s = carry + total;
        __syncthreads();
    }
}

// list[cursor[b]++] = (slot, remote row).  The order inside a segment is unspecified; the rows pulled are not.
__global__ void __launch_bounds__(256) k_plan_scatter(const int32_t* __restrict__ cache_ids, const int64_t* __restrict__ num_cached,
                                                      const uint32_t* __restrict__ first_batch, const int32_t* __restrict__ home,
                                                      int num_batches, int32_t* __restrict__ cursor, int32_t* __restrict__ list) {
    const int64_t k = *num_cached;
    for (int64_t s = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; s < k; s += (int64_t)gridDim.x * blockDim.x) {
        const int32_t v = cache_ids[s];
        const uint32_t f = first_batch[v];
        const int64_t j = atomicAdd(&cursor[f < (uint32_t)num_batches ? (int)f : num_batches], 1);
        list[2 * j] = (int32_t)s;
        list[2 * j + 1] = (int32_t)((uint32_t)home[v] & RG_ROW_MASK);
    }
}

// Ordered plan (num_batches + 1 <= 1024): a stable counting sort of the slots by first batch, so that every segment
// lists its slots in ascending order, i.e. ascending remote rows: the link serves ascending host addresses
// measurably faster than scattered ones (52 against 46 GB/s on 1 KiB rows).
constexpr int kPlanChunk = 1024;     // slots per workgroup, one per thread
constexpr int kPlanKeyBits = 10;

// Chunks in use, one at least: a cache may hold far fewer rows than its capacity.
__device__ __forceinline__ int rg_plan_chunks(int64_t num_cached, int nblocks) {
    const int64_t used = (num_cached + kPlanChunk - 1) / kPlanChunk;
    return used < 1 ? 1 : used < nblocks ? (int)used : nblocks;
}

__device__ __forceinline__ int rg_plan_key(const uint32_t* __restrict__ first_batch, int32_t v, int num_batches) {
    const uint32_t f = first_batch[v];
    return f < (uint32_t)num_batches ? (int)f : num_batches;
}

// hist[key * nblocks + blk] = number of slots of chunk blk first used by batch `key`, for the chunks in use.
// by_chunk: hist[blk * keys + key] instead, which k_plan_block_scatter adds up itself: with few chunks that takes less than a launch that
// scans them (5 k to 49 k slots, 20 to 400 batches: a call 11.6 us instead of 14.6; the reads of 48 chunks take as long as that launch).
constexpr int kPlanFewChunks = 48;
__global__ void __launch_bounds__(1024) k_plan_block_hist(const int32_t* __restrict__ cache_ids, const int64_t* __restrict__ num_cached,
                                                          const uint32_t* __restrict__ first_batch, int num_batches, int nblocks, int by_chunk,
                                                          int32_t* __restrict__ hist) {
    __shared__ int h[1024];
    const int64_t k = *num_cached;
    if ((int)blockIdx.x >= rg_plan_chunks(k, nblocks)) return;          // uniform
    const int n_seg = num_batches + 1;
    if ((int)threadIdx.x < n_seg) h[threadIdx.x] = 0;
    __syncthreads();
    const int64_t s = (int64_t)blockIdx.x * kPlanChunk + threadIdx.x;
    if (s < k) atomicAdd(&h[rg_plan_key(first_batch, cache_ids[s], num_batches)], 1);
    __syncthreads();
    if ((int)threadIdx.x < n_seg) hist[by_chunk ? (int64_t)blockIdx.x * n_seg + threadIdx.x : (int64_t)threadIdx.x * nblocks + blockIdx.x] = h[threadIdx.x];
}

// One workgroup per key: in-place exclusive scan of the key's chunks, its total to total[key].  (One workgroup for all keys
// took 39 us for 193 keys x 180 chunks.)
__global__ void __launch_bounds__(256) k_plan_row_scan(const int64_t* __restrict__ num_cached, int32_t* __restrict__ hist, int nblocks,
                                                       int32_t* __restrict__ total) {
    __shared__ int smem[256 / RG_WAVE + 1];
    int32_t* __restrict__ row = hist + (int64_t)blockIdx.x * nblocks;
    const int used = rg_plan_chunks(*num_cached, nblocks);
    int carry = 0;
    for (int base = 0; base < used; base += 256) {
        const int i = base + threadIdx.x;
        const int x = i < used ? row[i] : 0;
        int sum;
        const int excl = rg_block_excl_scan<256 / RG_WAVE>(x, smem, &sum);
        if (i < used) row[i] = carry + excl;
        carry += sum;
    }
    if (threadIdx.x == 0) total[blockIdx.x] = carry;
}

// Every slot to its place: the keys in front of its own, its key's slots in earlier chunks, in earlier wavefronts of this
// chunk, in lower lanes.  Lanes of the same key find each other with one ballot per key bit; the wavefronts' counts per key
// meet in LDS.  (One thread per key walking the chunk's keys took 169 us for 367 k slots, 193 keys; now 13.)
__global__ void __launch_bounds__(kPlanChunk) k_plan_block_scatter(const int32_t* __restrict__ cache_ids, const int64_t* __restrict__ num_cached,
                                                                   const uint32_t* __restrict__ first_batch, const int32_t* __restrict__ home,
                                                                   int num_batches, int nblocks, int by_chunk, const int32_t* __restrict__ hist,
                                                                   const int32_t* __restrict__ total, int32_t* __restrict__ offsets,
                                                                   int32_t* __restrict__ list) {
    constexpr int NW = kPlanChunk / RG_WAVE;
    __shared__ uint16_t cnt[NW][1024];   // slots of a key in the wavefront, then in the earlier wavefronts
    __shared__ int key_base[1024];
    __shared__ int smem[NW + 1];
    const int64_t k = *num_cached;
    if ((int)blockIdx.x >= rg_plan_chunks(k, nblocks)) return;          // uniform
    const int n_seg = num_batches + 1;
    const int wave = threadIdx.x >> 6, lane = rg_lane();
    for (int i = threadIdx.x; i < NW * 1024 / 2; i += kPlanChunk) ((uint32_t*)cnt)[i] = 0u;
    const int64_t s = (int64_t)blockIdx.x * kPlanChunk + threadIdx.x;
    const int32_t v = s < k ? cache_ids[s] : 0;
    const int key = s < k ? rg_plan_key(first_batch, v, num_batches) : 1 << kPlanKeyBits;   // no key: matches only its like
    const int32_t row = s < k ? (int32_t)((uint32_t)home[v] & RG_ROW_MASK) : 0;
    int sum, mine = 0, earlier = 0;                                   // of this thread's key: all slots, those of earlier chunks
    if ((int)threadIdx.x < n_seg) {
        if (by_chunk) {
            const int used = rg_plan_chunks(k, nblocks);
#pragma unroll 8
            for (int b = 0; b < used; ++b) {
                const int x = hist[b * n_seg + threadIdx.x];
                mine += x;
                earlier += b < (int)blockIdx.x ? x : 0;
            }
        } else {
            mine = total[threadIdx.x];
        }
    }
    const int before = rg_block_excl_scan<NW>(mine, smem, &sum);      // its barriers also end the clearing of cnt
    if ((int)threadIdx.x < n_seg) {
        key_base[threadIdx.x] = before + (by_chunk ? earlier : hist[(int64_t)threadIdx.x * nblocks + blockIdx.x]);
        if (blockIdx.x == 0) offsets[threadIdx.x] = before;
    }
    if (blockIdx.x == 0 && threadIdx.x == 0) offsets[n_seg] = sum;
    unsigned long long same = ~0ull;
#pragma unroll
    for (int q = 0; q <= kPlanKeyBits; ++q) {
        const unsigned long long ones = __ballot((key >> q) & 1);
        same &= (key >> q) & 1 ? ones : ~ones;
    }
    const int rank = __popcll(same & ((1ull << lane) - 1ull));
    if (s < k && rank == 0) cnt[wave][key] = (uint16_t)__popcll(same);
    __syncthreads();
    if ((int)threadIdx.x < n_seg) {
        int run = 0;
#pragma unroll
        for (int w = 0; w < NW; ++w) { const int c = cnt[w][threadIdx.x]; cnt[w][threadIdx.x] = (uint16_t)run; run += c; }
    }
    __syncthreads();
    if (s < k) {
        const int64_t j = (int64_t)key_base[key] + cnt[wave][key] + rank;
        list[2 * j] = (int32_t)s;
        list[2 * j + 1] = row;
    }
}

// ---------------------------------------------------------------------------- plan segments straight from the sampler's bitmaps
// After the last hop the `visited` bitmaps of a sampler group are its batches' input-node sets.  The remote rows the
// group is the first to name are the new bits of their union against `claimed` (all nodes any earlier group named)
// whose home is the remote store: two streaming passes over N/32 words and one home[] lookup per new node, instead of
// one lookup and one probe per input node of every batch.  The pairs come out ascending by node id, i.e. by remote row.
// A workgroup takes kClaimWords words, a lane one of them, whose ids' home words it asks for kClaimIds at a time: few instructions where there are few
// ids to a word, and every lane has lines on their way.  Calls with nothing claimed before, (15,10), clearing `claimed` included; four words to a lane and
// one id at a time / a lane per id, 64 of them together / now: 8 batches of 4096 seeds on 1 M nodes 56 / 20 / 15 us, on 10 M 53 / 39 / 25, 2 of them on
// 10 M 28 / 33 / 15, one of 1024 on 4 M 17.6 / 18.6 / 12.0; with 8 ids at a time the same or 3 % more.
constexpr int kClaimWords = 256, kClaimIds = 4;
static_assert(kClaimWords == 256, "a lane per word");
constexpr int kClaimSelfScan = 4096;        // workgroups up to which the emit adds up the counts in front of its own itself

// f(number, id, its home word) for the ids of a lane's word.
template <typename F>
__device__ __forceinline__ void rg_claim_ids(uint32_t bits, int64_t word, const int32_t* __restrict__ home, F f) {
    for (int k = 0; bits != 0u; k += kClaimIds) {
        int id[kClaimIds];
        uint32_t hw[kClaimIds];
#pragma unroll
        for (int q = 0; q < kClaimIds; ++q) {
            id[q] = __ffs(bits) - 1;
            bits &= bits - 1u;
        }
#pragma unroll
        for (int q = 0; q < kClaimIds; ++q) hw[q] = id[q] >= 0 ? (uint32_t)home[(word << 5) + id[q]] : 0u;
#pragma unroll
        for (int q = 0; q < kClaimIds; ++q)
            if (id[q] >= 0) f(k + q, id[q], hw[q]);
    }
}

// newbits = the ids that this group is the first to name and whose home is the remote store; their number per workgroup.
__global__ void __launch_bounds__(256) k_claim_count(const uint32_t* __restrict__ visited, int64_t words, int group,
                                                     uint32_t* __restrict__ claimed, uint32_t* __restrict__ newbits,
                                                     const int32_t* __restrict__ home, int32_t* __restrict__ blk_count) {
    __shared__ int part[4];
    const int64_t w = (int64_t)blockIdx.x * kClaimWords + threadIdx.x;
    uint32_t nw = 0u;
    if (w < words) {
        uint32_t u = 0u;
        for (int g = 0; g < group; ++g) u |= visited[g * words + w];
        const uint32_t old = claimed[w];
        nw = u & ~old;
        if (nw) claimed[w] = old | nw;
    }
    uint32_t remote = 0u;
    rg_claim_ids(nw, w, home, [&](int, int id, uint32_t hw) { remote |= (uint32_t)((hw >> RG_TAG_SHIFT) == RG_TAG_REMOTE) << id; });
    if (w < words) newbits[w] = remote;
    const int c = rg_wave_sum(__popc(remote));
    if (rg_lane() == 0) part[threadIdx.x >> 6] = c;
    __syncthreads();
    if (threadIdx.x == 0) blk_count[blockIdx.x] = part[0] + part[1] + part[2] + part[3];
}

// One workgroup: block counts -> exclusive offsets, their sum behind them.
__global__ void __launch_bounds__(1024) k_claim_scan(int32_t* __restrict__ blk_count, int nblocks) {
    __shared__ int smem[1024 / RG_WAVE + 1];
    __shared__ int carry_s;
    if (threadIdx.x == 0) carry_s = 0;
    __syncthreads();
    for (int base = 0; base < nblocks; base += 1024) {
        const int i = base + threadIdx.x;
        const int x = i < nblocks ? blk_count[i] : 0;
        int total;
        const int excl = rg_block_excl_scan<1024 / RG_WAVE>(x, smem, &total);
        const int carry = carry_s;
        if (i < nblocks) blk_count[i] = carry + excl;
        __syncthreads();
        if (threadIdx.x == 0) carry_s = carry + total;
        __syncthreads();
    }
    if (threadIdx.x == 0) blk_count[nblocks] = carry_s;
}

// The pairs, ascending; the segment's end goes behind its start in the plan's offsets.  scanned: blk_count is k_claim_scan's.
__global__ void __launch_bounds__(256) k_claim_emit(const uint32_t* __restrict__ newbits, int64_t words, const int32_t* __restrict__ home,
                                                    const int32_t* __restrict__ blk_count, int scanned, int32_t* __restrict__ seg_off,
                                                    int64_t list_capacity, int32_t* __restrict__ list) {
    __shared__ int smem[256 / RG_WAVE + 1];
    __shared__ int part[2][4];
    int before = 0, all = 0;
    if (scanned) {
        if (threadIdx.x == 0) { before = blk_count[blockIdx.x]; all = blk_count[gridDim.x]; }
    } else {
        for (unsigned b = threadIdx.x; b < gridDim.x; b += 256) {
            const int x = blk_count[b];
            all += x;
            before += b < blockIdx.x ? x : 0;
        }
    }
    before = rg_wave_sum(before);
    all = rg_wave_sum(all);
    if (rg_lane() == 0) { part[0][threadIdx.x >> 6] = before; part[1][threadIdx.x >> 6] = all; }
    const int64_t w = (int64_t)blockIdx.x * kClaimWords + threadIdx.x;
    const uint32_t nw = w < words ? newbits[w] : 0u;
    int total;
    const int first = rg_block_excl_scan<256 / RG_WAVE>(__popc(nw), smem, &total);          // its barriers publish part[]
    all = part[1][0] + part[1][1] + part[1][2] + part[1][3];
    // a list that cannot take the segment (it holds one pair per remote row, so this means a caller error) gets an
    // empty segment instead of an overrun
    const int64_t begin = seg_off[0];
    const bool fits = begin + all <= list_capacity;
    if (blockIdx.x == 0 && threadIdx.x == 0) seg_off[1] = (int32_t)(fits ? begin + all : begin);
    if (!fits || total == 0) return;                                  // uniform
    list += 2 * (begin + part[0][0] + part[0][1] + part[0][2] + part[0][3] + first);
    rg_claim_ids(nw, w, home, [&](int k, int, uint32_t hw) {
        list[2 * k] = list[2 * k + 1] = (int32_t)(hw & RG_ROW_MASK);  // mirrored cache: the row's place is its remote-store row
    });
}

__global__ void __launch_bounds__(256) k_zero_i32(int32_t* __restrict__ p, int n) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) p[i] = 0;
}

int low_grid_of(const rg_ctx* ctx, int64_t num_nodes) {
    return (int)rg_max64(1, rg_min64(rg_div_up(num_nodes, 4096), ctx->num_cus * (num_nodes > (8ll << 20) ? 2 : 1)));
}

// Launches the list-driven row copy.  `blocks` and `threads` bound the wavefronts in flight.
rg_status launch_list_copy(rg_ctx* ctx, const int32_t* list, const uint32_t* pctl, const float* src, int64_t src_stride,
                           float* dst, int64_t dst_stride, int64_t dst_rows, int32_t dim, int64_t n_upper, int64_t blocks,
                           int threads, hipStream_t s, const int32_t* seg_off = nullptr, uint32_t* mark = nullptr) {
    const void* ptrs[2] = {src, dst};
    const int64_t strides[2] = {src_stride, dst_stride};
    const int vec = rg_pick_vec(dim, ptrs, 2, strides, 2);
    const RgRowShape shp = rg_row_shape(dim, vec);
    const int U = ctx->knobs.pull_rows == 8 ? 8 : 4;        // rows in flight per lane group
    const int rows_per_block = (threads / RG_WAVE) * (RG_WAVE >> shp.log2L) * U;
    const int grid = (int)rg_max64(1, rg_min64(rg_div_up(n_upper, rows_per_block), blocks));
    const int tok = rg_prof_begin(ctx, RG_K_CACHE_FILL, s);
#define RG_LAUNCH_PULL(V, UU)                                                                                          \
    k_prefetch_pull<V, UU><<<grid, threads, 0, s>>>(list, pctl, seg_off, src, src_stride, dst, dst_stride, dst_rows, shp.cpr, \
                                                    shp.log2L, shp.tail, mark)
    if (vec == 4) { if (U == 8) RG_LAUNCH_PULL(4, 8); else RG_LAUNCH_PULL(4, 4); }
    else if (vec == 2) RG_LAUNCH_PULL(2, 4);
    else RG_LAUNCH_PULL(1, 4);
#undef RG_LAUNCH_PULL
    rg_prof_end(ctx, tok, s);
    RG_LAUNCH_CHECK(ctx, "k_prefetch_pull");
    return RG_OK;
}

// Id ranges of the epoch histogram: whole rounds of two workgroups per compute unit, but no more ranges than runs of up to run_len
// entries pay for.  A range costs every run a search and a segment (50 ns per thousand), and saves its share of the LDS atomics: least
// in sum near sqrt(4.4 run_len) ranges.  Up to 136 they are on compute units that would idle (750 runs, 64 entries a step: 334 k nodes, 30
// entries each, 41 ranges 21 us, 64 18, 128 16; 20 k nodes, 3 each, 3 ranges 18 us, 40 11).
int hist_range(const rg_ctx* ctx, int64_t num_nodes, int64_t run_len) {
    const int64_t places = 2ll * ctx->num_cus;
    const int64_t rounds = rg_max64(1, rg_div_up(num_nodes, places * kHistRangeMax));
    const int64_t even = rg_max64(kHistRangeMin, rg_div_up(num_nodes, places * rounds));
    const int64_t worth = rg_max64(136, (int64_t)sqrt(4.4 * (double)run_len));
    return (int)rg_min64(kHistRangeMax, rg_max64(even, rg_div_up(num_nodes, worth)));
}

// Most entries of the bounds' scratch (8 MB; one batch of 8 hops on 2^30 nodes needs half of that): a call of more batches takes
// several launches.
constexpr int64_t kHistBoundsMax = 2ll << 20;

}  // namespace

// Room for `entries` bounds.  An outgrown buffer stays allocated: a histogram needed no scratch once, and a graph that holds this
// one must survive any later call.  A buffer has at least twice its predecessor's size, up to the 8 MB: less than 16 MB in all.
static rg_status hist_bounds_grow(rg_ctx* ctx, int64_t entries) {
    RgBuf& buf = ctx->hist_bounds;
    if (buf.bytes >= (size_t)entries * 4 || ctx->bounds_denied) return RG_OK;
    RgBuf larger;
    const rg_status st = rg_ensure(ctx, larger, (size_t)rg_max64(entries * 4, rg_min64((int64_t)buf.bytes * 2, kHistBoundsMax * 4)));
    ctx->bounds_denied = st == RG_ERR_OOM;
    if (st != RG_OK) return st;
    if (buf.p) ctx->outgrown.push_back(buf.p);
    buf = larger;
    return RG_OK;
}

rg_status rg_histogram_reserve(rg_ctx* ctx, int64_t num_nodes) {
    if (num_nodes <= 0) return RG_OK;
    ctx->hist_reserved = true;
    const int64_t per_batch = RG_MAX_HOPS * (rg_div_up(num_nodes, hist_range(ctx, num_nodes, kHistBoundsMax)) + 1);
    return hist_bounds_grow(ctx, per_batch * rg_max64(1, rg_min64(128, kHistBoundsMax / per_batch)));
}

extern "C" {

rg_status rg_access_histogram(rg_ctx* ctx, const int32_t* nodes, int64_t n, const int32_t* n_dev, uint32_t* counts,
                              int64_t num_nodes, void* stream) {
    if (!ctx) return RG_ERR_INVALID_ARG;
    RG_REQUIRE(ctx, n >= 0 && num_nodes >= 0, "rg_access_histogram: negative size");
    if (n == 0) return RG_OK;
    RG_REQUIRE(ctx, nodes && counts, "rg_access_histogram: null pointer");
    RG_REQUIRE(ctx, num_nodes > 0, "rg_access_histogram: entries given but num_nodes is 0");
    RG_HIP(ctx, hipSetDevice(ctx->device));
    hipStream_t s = (hipStream_t)stream;
    const int grid = (int)rg_min64(rg_div_up(n, 256), (int64_t)ctx->num_cus * 32);
    const int tok = rg_prof_begin(ctx, RG_K_HISTOGRAM, s);
    k_histogram<<<grid, 256, 0, s>>>(nodes, n, n_dev, counts);
    rg_prof_end(ctx, tok, s);
    RG_LAUNCH_CHECK(ctx, "k_histogram");
    return RG_OK;
}

rg_status rg_access_histogram_epoch(rg_ctx* ctx, const int32_t* nodes, int64_t batch_stride, const int32_t* tier_off,
                                    int32_t num_batches, int32_t num_hops, int32_t max_seeds, uint32_t* counts,
                                    uint32_t* first_batch, int64_t num_nodes, void* stream) {
    if (!ctx) return RG_ERR_INVALID_ARG;
    RG_REQUIRE(ctx, num_batches >= 0 && num_batches <= 65535, "rg_access_histogram_epoch: num_batches = %d not in [0, 65535]", num_batches);
    RG_REQUIRE(ctx, num_hops >= 1 && num_hops <= RG_MAX_HOPS, "rg_access_histogram_epoch: num_hops = %d not in [1,%d]", num_hops, RG_MAX_HOPS);
    RG_REQUIRE(ctx, batch_stride >= 0 && max_seeds >= 0 && num_nodes >= 0, "rg_access_histogram_epoch: negative size");
    RG_REQUIRE(ctx, num_nodes <= (int64_t)RG_ROW_MASK + 1, "rg_access_histogram_epoch: num_nodes exceeds 2^30");
    if (num_batches == 0 || num_nodes == 0) return RG_OK;
    RG_REQUIRE(ctx, nodes && tier_off && counts, "rg_access_histogram_epoch: null pointer");
    RG_HIP(ctx, hipSetDevice(ctx->device));
    hipStream_t s = (hipStream_t)stream;
    const int64_t run_len = batch_stride / num_hops;
    const int range = hist_range(ctx, num_nodes, run_len);
    const int ranges = (int)rg_div_up(num_nodes, range);
    // batches per launch: the bounds of their runs fit the scratch, and a grid's second dimension.  (After rg_reserve, which leaves
    // room for 128 batches or more, a call takes more launches rather than more scratch.)  Without scratch, in a captured call or for
    // want of memory, the counting kernel searches for itself.
    const int64_t per_batch = (int64_t)num_hops * (ranges + 1);
    const int64_t most = rg_min64(num_batches, rg_max64(1, kHistBoundsMax / per_batch));
    // The counting kernel also searches where that is faster, for two reasons.  The launch of its own that the bounds take costs 3 us, more
    // than few or short runs are worth: the chains of probes weigh runs x ranges x log2(entries)^4 (1 M nodes, 25 runs of 30,000
    // entries, 4.45e8: 11.4-11.8 us against 14-15, 60 of them 15.8 / 15.5; 750 of 300, 4.3e8, 29 / 26; 2.4 M nodes, 60 of 3000, 3.1e8:
    // 12.5 / 14.7, 8 of 300,000, 4.5e8, 19 / 15).  Above a round of the device the probes of every round add up, so only very short runs are
    // searched (10 M nodes, 180 runs of 30, 1.4e8: 15 / 18, 360 of them 25 / 23; 24 of 300: 16 / 15, one of 30,000: 20 / 14).
    const double steps = log2((double)run_len + 2.0);
    const double weight = (double)num_batches * (double)per_batch * steps * steps * steps * steps;
    const bool few = num_nodes <= (1 << 22) ? weight <= 4.46e8 : run_len <= 64 && weight <= 2e8;
    // And a launch of few batches does little besides clearing and adding its ranges: 245 batches on 200 M nodes, 28 to a
    // launch, 2.2-3.5 ms in one launch that searches against 2.7-5.0 ms (64 batches 0.7-1.2 / 0.75-1.6, but 32 batches in two launches
    // 0.52-0.56 / 0.42-0.47); on 100 M nodes, 56 to a launch, 1.2-2.0 ms either way.
    const int64_t wanted = per_batch * (ctx->hist_reserved ? rg_min64(most, 128) : most);
    if (!few && (int64_t)(ctx->hist_bounds.bytes / 4) < wanted && !rg_capturing(s)) (void)hist_bounds_grow(ctx, wanted);
    const int fit = (int)rg_min64((int64_t)(ctx->hist_bounds.bytes / 4) / per_batch, 65535 / (num_hops + 1));
    const bool search = few || fit == 0 || (fit < 48 && num_batches > 2 * fit);
    const int step = search ? num_batches : fit;
    int32_t* bounds = search ? nullptr : (int32_t*)ctx->hist_bounds.p;
    const RunStep by = {16 / num_hops, 16 % num_hops, kHistRunTile / num_hops, kHistRunTile % num_hops};
    const bool ahead = run_len >= (int64_t)kHistAhead * ranges;
    const int tok = rg_prof_begin(ctx, RG_K_HISTOGRAM, s);
    // Batches of a workgroup's seeds or more are counted beside the bounds, by some 64 workgroups each at most.
    const int bound_blocks = (int)rg_div_up(ranges + 1, 256);
    const int64_t seed_blocks = rg_min64(rg_min64(rg_div_up(max_seeds, 256 * kSeedRounds), 64), rg_div_up((int64_t)kSeedBlocks * ctx->num_cus, num_batches));
    const int seed_rows = (int)rg_max64(1, (seed_blocks + bound_blocks / 2) / bound_blocks);
    const bool beside = bounds && max_seeds >= kSeedsBeside && num_batches <= fit && (int64_t)num_batches * (num_hops + seed_rows) <= 65535;
    if (max_seeds > 0 && !beside) {
        dim3 seed_grid((unsigned)rg_min64(rg_div_up(max_seeds, 256), 64), (unsigned)num_batches);
        k_histogram_seeds<<<seed_grid, 256, 0, s>>>(nodes, batch_stride, tier_off, num_hops, counts, first_batch);
    }
    for (int b0 = 0; b0 < num_batches; b0 += step) {
        const int nb = num_batches - b0 < step ? num_batches - b0 : step;
        const int32_t* list = nodes + (int64_t)b0 * batch_stride;
        const int32_t* tiers = tier_off + (int64_t)b0 * (num_hops + 2);
        if (bounds)
            k_hist_bounds<<<dim3((unsigned)bound_blocks, (unsigned)(nb * (num_hops + (beside ? seed_rows : 0)))), 256, 0, s>>>(
                list, batch_stride, tiers, num_hops, num_nodes, range, ranges, bounds, beside ? nb : 0, seed_rows, counts, first_batch);
#define RG_LAUNCH_RUNS(FIRST, AHEAD)                                                                                      \
    k_histogram_runs<FIRST, AHEAD><<<ranges, 1024, 0, s>>>(list, batch_stride, tiers, bounds, nb, num_hops, b0, counts, first_batch, num_nodes, range, by)
        if (first_batch) { if (ahead) RG_LAUNCH_RUNS(true, true); else RG_LAUNCH_RUNS(true, false); }
        else { if (ahead) RG_LAUNCH_RUNS(false, true); else RG_LAUNCH_RUNS(false, false); }
#undef RG_LAUNCH_RUNS
    }
    rg_prof_end(ctx, tok, s);
    RG_LAUNCH_CHECK(ctx, "k_histogram_runs");
    return RG_OK;
}

rg_status rg_build_cache(rg_ctx* ctx, const uint32_t* counts, const int32_t* home, int64_t num_nodes,
                         const float* remote_store, int64_t remote_stride, int32_t dim, const rg_cache* cache,
                         void* stream) {
    if (!ctx) return RG_ERR_INVALID_ARG;
    RG_REQUIRE(ctx, cache, "rg_build_cache: cache is NULL");
    RG_REQUIRE(ctx, num_nodes >= 0 && num_nodes <= (int64_t)RG_ROW_MASK + 1, "rg_build_cache: num_nodes out of range");
    RG_REQUIRE(ctx, cache->capacity_rows >= 0 && cache->capacity_rows <= (int64_t)RG_ROW_MASK + 1,
               "rg_build_cache: capacity_rows = %lld out of range", (long long)cache->capacity_rows);
    RG_REQUIRE(ctx, dim >= 1, "rg_build_cache: dim = %d must be positive", dim);
    RG_REQUIRE(ctx, cache->row_stride >= dim && (!remote_store || remote_stride >= dim), "rg_build_cache: row stride smaller than dim");
    RG_REQUIRE(ctx, remote_store || cache->filled || cache->capacity_rows == 0 || num_nodes == 0,
               "rg_build_cache: select-only mode (remote_store == NULL) needs cache->filled");
    RG_REQUIRE(ctx, cache->num_cached, "rg_build_cache: num_cached is NULL");
    RG_REQUIRE(ctx, cache->mirror_rows >= 0 && cache->mirror_rows <= cache->capacity_rows,
               "rg_build_cache: mirror_rows = %lld exceeds capacity_rows = %lld", (long long)cache->mirror_rows, (long long)cache->capacity_rows);
    RG_REQUIRE(ctx, cache->mirror_rows == 0 || (!remote_store && cache->home),
               "rg_build_cache: a mirrored cache is filled by rg_prefetch_cache_rows (remote_store must be NULL) and needs cache->home");
    RG_REQUIRE(ctx, num_nodes == 0 || (counts && home && cache->loc), "rg_build_cache: null node array");
    const bool may_select = cache->capacity_rows > 0 && num_nodes > 0;
    RG_REQUIRE(ctx, !may_select || (cache->cache_ids && cache->cache_rows), "rg_build_cache: null cache buffer");
    RG_HIP(ctx, hipSetDevice(ctx->device));
    if (may_select && remote_store) {
        const rg_status chk = rg_check_device_readable(ctx, remote_store, "rg_build_cache: remote_store");
        if (chk != RG_OK) return chk;
    }
    hipStream_t s = (hipStream_t)stream;

    const int64_t nblocks = rg_max64(1, rg_div_up(num_nodes, kNodesPerBlock));
    rg_status st;
    if ((st = rg_ensure(ctx, ctx->topk_ctl, sizeof(TopkCtl))) != RG_OK) return st;
    if ((st = rg_ensure(ctx, ctx->topk_blk, (size_t)nblocks * 8)) != RG_OK) return st;
    TopkCtl* ctl = (TopkCtl*)ctx->topk_ctl.p;
    int32_t* blk_gt = (int32_t*)ctx->topk_blk.p;
    int32_t* blk_eq = blk_gt + nblocks;

    // the emit of the call before this one has left the histograms zero; a recorded call does not count on it
    const bool captured = rg_capturing(s);
    if (captured || !ctx->topk_clean) {
        k_topk_init<<<4, 256, 0, s>>>(ctl, 0);
        RG_LAUNCH_CHECK(ctx, "k_topk_init");
    }
    if (!captured) ctx->topk_clean = false;                  // until the emit has been queued
    const int low_grid = low_grid_of(ctx, num_nodes);
    k_topk_hist_low<<<low_grid, 1024, 0, s>>>(counts, home, num_nodes, ctl, cache->capacity_rows);
    RG_LAUNCH_CHECK(ctx, "k_topk_hist_low");
    const int hist_grid = (int)rg_max64(1, rg_min64(rg_div_up(num_nodes, 1024 * 8), (int64_t)ctx->num_cus * 2));
    for (int pass = 1; pass < kRadixPasses; ++pass) {        // return at once unless the threshold is in the clamped bin
        k_topk_hist<<<hist_grid, 1024, 0, s>>>(counts, home, num_nodes, pass, cache->capacity_rows, ctl, nullptr);
        RG_LAUNCH_CHECK(ctx, "k_topk_hist");
    }
    k_topk_count<<<(int)nblocks, 1024, 0, s>>>(counts, home, num_nodes, ctl, blk_gt, blk_eq, cache->num_cached);
    RG_LAUNCH_CHECK(ctx, "k_topk_count");
    const int scanned = nblocks > kTopkSelfScan;
    if (scanned) {
        k_topk_scan<<<1, 1024, 0, s>>>(blk_gt, blk_eq, nblocks);
        RG_LAUNCH_CHECK(ctx, "k_topk_scan");
    }
    const int64_t filled_words = cache->mirror_rows == 0 ? rg_div_up(rg_min64(cache->capacity_rows, num_nodes), 32) : 0;
    k_topk_emit<<<(int)nblocks, 1024, 0, s>>>(counts, home, num_nodes, ctl, blk_gt, blk_eq, scanned, cache->cache_ids,
                                              cache->loc, filled_words > 0 ? cache->filled : nullptr, filled_words, remote_store ? 1 : 0);
    RG_LAUNCH_CHECK(ctx, "k_topk_emit");
    if (!captured) ctx->topk_clean = true;

    if (may_select && remote_store) {
        const void* ptrs[2] = {remote_store, cache->cache_rows};
        const int64_t strides[2] = {remote_stride, cache->row_stride};
        const int vec = rg_pick_vec(dim, ptrs, 2, strides, 2);
        const RgRowShape shp = rg_row_shape(dim, vec);
        const int64_t rows_ub = rg_min64(cache->capacity_rows, num_nodes);
        const int rows_per_block = 4 * (RG_WAVE >> shp.log2L) * 4;
        const int grid = (int)rg_max64(1, rg_min64(rg_div_up(rows_ub, rows_per_block), (int64_t)ctx->num_cus * 16));
        const int tok = rg_prof_begin(ctx, RG_K_CACHE_FILL, s);
        if (vec == 4)
            k_cache_fill<4><<<grid, 256, 0, s>>>(cache->cache_ids, home, cache->num_cached, remote_store, remote_stride, cache->cache_rows, cache->row_stride, shp.cpr, shp.log2L, shp.tail);
        else if (vec == 2)
            k_cache_fill<2><<<grid, 256, 0, s>>>(cache->cache_ids, home, cache->num_cached, remote_store, remote_stride, cache->cache_rows, cache->row_stride, shp.cpr, shp.log2L, shp.tail);
        else
            k_cache_fill<1><<<grid, 256, 0, s>>>(cache->cache_ids, home, cache->num_cached, remote_store, remote_stride, cache->cache_rows, cache->row_stride, shp.cpr, shp.log2L, shp.tail);
        rg_prof_end(ctx, tok, s);
        RG_LAUNCH_CHECK(ctx, "k_cache_fill");
    }
    return RG_OK;
}

rg_status rg_cache_hit_curve(rg_ctx* ctx, const uint32_t* counts, const int32_t* home, int64_t num_nodes,
                             const int64_t* capacities, int32_t num_capacities, uint64_t* hits, uint64_t* remote_total,
                             void* stream) {
    if (!ctx) return RG_ERR_INVALID_ARG;
    RG_REQUIRE(ctx, num_nodes >= 0 && num_nodes <= (int64_t)RG_ROW_MASK + 1, "rg_cache_hit_curve: num_nodes out of range");
    RG_REQUIRE(ctx, num_capacities >= 0 && num_capacities <= 4096, "rg_cache_hit_curve: num_capacities not in [0, 4096]");
    RG_REQUIRE(ctx, num_capacities == 0 || (capacities && hits), "rg_cache_hit_curve: null capacities / hits");
    RG_REQUIRE(ctx, num_nodes == 0 || (counts && home), "rg_cache_hit_curve: null node array");
    for (int j = 0; j < num_capacities; ++j)
        RG_REQUIRE(ctx, capacities[j] >= 0 && capacities[j] <= (int64_t)RG_ROW_MASK + 1, "rg_cache_hit_curve: capacities[%d] out of range", j);
    RG_HIP(ctx, hipSetDevice(ctx->device));
    hipStream_t s = (hipStream_t)stream;
    rg_status st;
    if ((st = rg_ensure(ctx, ctx->topk_ctl, sizeof(TopkCtl))) != RG_OK) return st;
    TopkCtl* ctl = (TopkCtl*)ctx->topk_ctl.p;
    // device copy of the capacities and one "resolved" flag per capacity
    const size_t caps_bytes = (size_t)rg_max64(num_capacities, 1) * 8;
    if ((st = rg_ensure(ctx, ctx->topk_caps, caps_bytes + (size_t)rg_max64(num_capacities, 1) * 4)) != RG_OK) return st;
    int64_t* caps_dev = (int64_t*)ctx->topk_caps.p;
    uint32_t* resolved = (uint32_t*)((char*)ctx->topk_caps.p + caps_bytes);
    for (int j0 = 0; j0 < num_capacities; j0 += kCapChunk) {             // by value: the host array is not read after the call
        CapChunk chunk;
        const int cnt = num_capacities - j0 < kCapChunk ? num_capacities - j0 : kCapChunk;
        for (int j = 0; j < kCapChunk; ++j) chunk.v[j] = j < cnt ? capacities[j0 + j] : 0;
        k_store_caps<<<1, kCapChunk, 0, s>>>(caps_dev + j0, chunk, cnt);
        RG_LAUNCH_CHECK(ctx, "k_store_caps");
    }
    const int grid = (int)rg_max64(1, rg_min64(rg_div_up(num_nodes, 256 * 8), (int64_t)ctx->num_cus * 8));
    const int hist_grid = (int)rg_max64(1, rg_min64(rg_div_up(num_nodes, 1024 * 8), (int64_t)ctx->num_cus * 2));
    const int low_grid = low_grid_of(ctx, num_nodes);
    // one pass over the nodes gives the histogram of the counts; every capacity is read off it
    const bool captured = rg_capturing(s);
    if (captured || !ctx->topk_clean) {
        k_topk_init<<<4, 256, 0, s>>>(ctl, 0);
        RG_LAUNCH_CHECK(ctx, "k_topk_init");
    }
    if (!captured) ctx->topk_clean = false;                  // until it has been cleared again
    k_topk_hist_low<<<low_grid, 1024, 0, s>>>(counts, home, num_nodes, ctl, -1);
    RG_LAUNCH_CHECK(ctx, "k_topk_hist_low");
    k_hit_curve_low<<<1, 256, 0, s>>>(ctl, caps_dev, num_capacities, (unsigned long long*)hits, (unsigned long long*)remote_total, resolved);
    RG_LAUNCH_CHECK(ctx, "k_hit_curve_low");
    // capacities whose threshold lies among counts >= kLowBins - 1 (never the case when the counts are bounded by a few
    // hundred batches) go through the radix select one by one; for all others, capacities of all candidates among them, these kernels return at once
    for (int j = 0; j < num_capacities; ++j) {
        if (j > 0) {
            k_topk_init<<<4, 256, 0, s>>>(ctl, 1);
            RG_LAUNCH_CHECK(ctx, "k_topk_init");
        }
        for (int pass = 1; pass < kRadixPasses; ++pass) {
            k_topk_hist<<<hist_grid, 1024, 0, s>>>(counts, home, num_nodes, pass, capacities[j], ctl, resolved + j);
            RG_LAUNCH_CHECK(ctx, "k_topk_hist");
        }
        k_hit_sum<<<grid, 256, 0, s>>>(counts, home, num_nodes, ctl, capacities[j], resolved + j, (unsigned long long*)hits + j);
        RG_LAUNCH_CHECK(ctx, "k_hit_sum");
    }
    k_topk_init<<<4, 256, 0, s>>>(ctl, 0);
    RG_LAUNCH_CHECK(ctx, "k_topk_init");
    if (!captured) ctx->topk_clean = true;
    return RG_OK;
}

rg_status rg_prefetch_cache_rows(rg_ctx* ctx, const int32_t* input_nodes, int64_t n, const int32_t* n_dev,
                                 const rg_cache* cache, const int32_t* home, const float* remote_store,
                                 int64_t remote_stride, int32_t dim, void* stream) {
    if (!ctx) return RG_ERR_INVALID_ARG;
    RG_REQUIRE(ctx, n >= 0 && n <= (1ll << 31) - 1, "rg_prefetch_cache_rows: n = %lld out of range", (long long)n);
    if (n == 0) return RG_OK;
    RG_REQUIRE(ctx, cache && cache->filled && cache->cache_rows && (cache->loc || cache->mirror_rows > 0),
               "rg_prefetch_cache_rows: cache needs filled, cache_rows and (unless mirrored) loc");
    RG_REQUIRE(ctx, cache->mirror_rows >= 0 && cache->mirror_rows <= cache->capacity_rows,
               "rg_prefetch_cache_rows: mirror_rows = %lld exceeds capacity_rows = %lld", (long long)cache->mirror_rows, (long long)cache->capacity_rows);
    RG_REQUIRE(ctx, input_nodes && home && remote_store, "rg_prefetch_cache_rows: null pointer");
    RG_REQUIRE(ctx, dim >= 1 && cache->row_stride >= dim && remote_stride >= dim, "rg_prefetch_cache_rows: bad dim / stride");
    RG_HIP(ctx, hipSetDevice(ctx->device));
    { const rg_status chk = rg_check_device_readable(ctx, remote_store, "rg_prefetch_cache_rows: remote_store"); if (chk != RG_OK) return chk; }
    hipStream_t s = (hipStream_t)stream;
    rg_status st;
    if ((st = rg_ensure(ctx, ctx->pf_ctl, 64)) != RG_OK) return st;
    if ((st = rg_ensure(ctx, ctx->pf_list, (size_t)n * 8)) != RG_OK) return st;
    uint32_t* pctl = (uint32_t*)ctx->pf_ctl.p;
    int32_t* list = (int32_t*)ctx->pf_list.p;
    k_prefetch_reset<<<1, 64, 0, s>>>(pctl);
    RG_LAUNCH_CHECK(ctx, "k_prefetch_reset");
    const bool mirror = cache->mirror_rows > 0;
    k_prefetch_select<<<(int)rg_div_up(n, 256), 256, 0, s>>>(input_nodes, n, n_dev, cache->loc, home, cache->filled, list, pctl, mirror ? 1 : 0);
    RG_LAUNCH_CHECK(ctx, "k_prefetch_select");
    return launch_list_copy(ctx, list, pctl, remote_store, remote_stride, cache->cache_rows, cache->row_stride,
                            mirror ? cache->mirror_rows : cache->capacity_rows, dim, n, ctx->knobs.pull_blocks, ctx->knobs.pull_threads, s);
}

rg_status rg_plan_prefetch(rg_ctx* ctx, const rg_cache* cache, const int32_t* home, const uint32_t* first_batch,
                           int64_t num_nodes, const rg_prefetch_plan* plan, void* stream) {
    if (!ctx) return RG_ERR_INVALID_ARG;
    RG_REQUIRE(ctx, cache && cache->num_cached && plan && plan->offsets, "rg_plan_prefetch: null cache / plan");
    RG_REQUIRE(ctx, cache->mirror_rows == 0, "rg_plan_prefetch: a mirrored cache is filled by rg_prefetch_cache_rows");
    RG_REQUIRE(ctx, plan->num_batches >= 0 && plan->num_batches <= 65535, "rg_plan_prefetch: num_batches not in [0, 65535]");
    RG_REQUIRE(ctx, num_nodes >= 0 && cache->capacity_rows >= 0, "rg_plan_prefetch: negative size");
    const int64_t rows_ub = rg_min64(cache->capacity_rows, num_nodes);
    RG_REQUIRE(ctx, rows_ub == 0 || (cache->cache_ids && home && first_batch && plan->list), "rg_plan_prefetch: null array");
    RG_REQUIRE(ctx, plan->list_capacity >= rows_ub, "rg_plan_prefetch: plan list holds %lld pairs, %lld required",
               (long long)plan->list_capacity, (long long)rows_ub);
    RG_HIP(ctx, hipSetDevice(ctx->device));
    hipStream_t s = (hipStream_t)stream;
    const int n_seg = plan->num_batches + 1;
    rg_status st;
    if (n_seg <= 1024) {
        // ordered plan: stable counting sort by first batch
        const int nblocks = (int)rg_max64(1, rg_div_up(rows_ub, kPlanChunk));
        const int64_t n_hist = (int64_t)n_seg * nblocks;
        if ((st = rg_ensure(ctx, ctx->plan_cursor, (size_t)(n_hist + n_seg) * 4)) != RG_OK) return st;
        int32_t* hist = (int32_t*)ctx->plan_cursor.p;
        int32_t* total = hist + n_hist;
        const int by_chunk = nblocks <= kPlanFewChunks;
        if (rows_ub == 0) {
            k_zero_i32<<<(n_seg + 1 + 255) / 256, 256, 0, s>>>(plan->offsets, n_seg + 1);
            RG_LAUNCH_CHECK(ctx, "k_zero_i32");
            return RG_OK;
        }
        k_plan_block_hist<<<nblocks, 1024, 0, s>>>(cache->cache_ids, cache->num_cached, first_batch, plan->num_batches, nblocks, by_chunk, hist);
        RG_LAUNCH_CHECK(ctx, "k_plan_block_hist");
        if (!by_chunk) {
            k_plan_row_scan<<<n_seg, 256, 0, s>>>(cache->num_cached, hist, nblocks, total);
            RG_LAUNCH_CHECK(ctx, "k_plan_row_scan");
        }
        k_plan_block_scatter<<<nblocks, kPlanChunk, 0, s>>>(cache->cache_ids, cache->num_cached, first_batch, home, plan->num_batches,
                                                            nblocks, by_chunk, hist, total, plan->offsets, plan->list);
        RG_LAUNCH_CHECK(ctx, "k_plan_block_scatter");
        return RG_OK;
    }
    // more than 1023 batches: unordered scatter with atomics (segments hold the right slots in arbitrary order)
    if ((st = rg_ensure(ctx, ctx->plan_cursor, (size_t)n_seg * 4)) != RG_OK) return st;
    int32_t* cursor = (int32_t*)ctx->plan_cursor.p;
    k_zero_i32<<<(n_seg + 1 + 255) / 256, 256, 0, s>>>(plan->offsets, n_seg + 1);
    RG_LAUNCH_CHECK(ctx, "k_zero_i32");
    const int grid = (int)rg_max64(1, rg_min64(rg_div_up(rows_ub, 256), (int64_t)ctx->num_cus * 8));
    if (rows_ub > 0) {
        k_plan_count<<<grid, 256, 0, s>>>(cache->cache_ids, cache->num_cached, first_batch, plan->num_batches, plan->offsets);
        RG_LAUNCH_CHECK(ctx, "k_plan_count");
    }
    k_plan_scan<<<1, 1024, 0, s>>>(plan->offsets, cursor, n_seg);
    RG_LAUNCH_CHECK(ctx, "k_plan_scan");
    if (rows_ub > 0) {
        k_plan_scatter<<<grid, 256, 0, s>>>(cache->cache_ids, cache->num_cached, first_batch, home, plan->num_batches, cursor, plan->list);
        RG_LAUNCH_CHECK(ctx, "k_plan_scatter");
    }
    return RG_OK;
}

rg_status rg_prefetch_planned(rg_ctx* ctx, const rg_prefetch_plan* plan, int32_t batch, const rg_cache* cache,
                              const float* remote_store, int64_t remote_stride, int32_t dim, void* stream) {
    if (!ctx) return RG_ERR_INVALID_ARG;
    RG_REQUIRE(ctx, plan && plan->offsets && plan->list, "rg_prefetch_planned: incomplete plan");
    RG_REQUIRE(ctx, batch >= 0 && batch <= plan->num_batches, "rg_prefetch_planned: batch = %d not in [0, %d]", batch, plan->num_batches);
    RG_REQUIRE(ctx, cache && cache->cache_rows && cache->filled && remote_store, "rg_prefetch_planned: null cache rows / filled / store");
    RG_REQUIRE(ctx, cache->mirror_rows >= 0 && cache->mirror_rows <= cache->capacity_rows, "rg_prefetch_planned: mirror_rows out of range");
    RG_REQUIRE(ctx, dim >= 1 && cache->row_stride >= dim && remote_stride >= dim, "rg_prefetch_planned: bad dim / stride");
    RG_HIP(ctx, hipSetDevice(ctx->device));
    { const rg_status chk = rg_check_device_readable(ctx, remote_store, "rg_prefetch_planned: remote_store"); if (chk != RG_OK) return chk; }
    hipStream_t s = (hipStream_t)stream;
    const int64_t dst_rows = cache->mirror_rows > 0 ? cache->mirror_rows : cache->capacity_rows;
    rg_status st = launch_list_copy(ctx, plan->list, nullptr, remote_store, remote_stride, cache->cache_rows, cache->row_stride,
                                    dst_rows, dim, rg_max64(plan->list_capacity, 1), ctx->knobs.pull_blocks,
                                    ctx->knobs.pull_threads, s, plan->offsets + batch, cache->filled);   // marks the slots resident too
    return st;
}

rg_status rg_plan_sampled(rg_ctx* ctx, int32_t group, const rg_cache* cache, uint32_t* claimed, const rg_prefetch_plan* plan,
                          int32_t segment, int64_t num_nodes, void* stream) {
    if (!ctx) return RG_ERR_INVALID_ARG;
    RG_REQUIRE(ctx, group >= 1 && group <= RG_MAX_GROUP, "rg_plan_sampled: group = %d not in [1,%d]", group, RG_MAX_GROUP);
    RG_REQUIRE(ctx, cache && cache->mirror_rows > 0 && cache->home, "rg_plan_sampled: needs a mirrored cache with its home words");
    RG_REQUIRE(ctx, claimed && plan && plan->list && plan->offsets, "rg_plan_sampled: null claimed bitmap / plan");
    RG_REQUIRE(ctx, segment >= 0 && segment < plan->num_batches, "rg_plan_sampled: segment = %d not in [0, %d)", segment, plan->num_batches);
    RG_REQUIRE(ctx, plan->list_capacity >= cache->mirror_rows, "rg_plan_sampled: plan list holds %lld pairs, %lld required",
               (long long)plan->list_capacity, (long long)cache->mirror_rows);
    if (ctx->last_sample_group != group || ctx->last_sample_nodes != num_nodes)
        return rg_set_error(ctx, RG_ERR_STATE, "rg_plan_sampled: the last sampling call of this context covered %d batches on %lld "
                            "nodes, not %d on %lld", ctx->last_sample_group, (long long)ctx->last_sample_nodes, group, (long long)num_nodes);
    RG_HIP(ctx, hipSetDevice(ctx->device));
    hipStream_t s = (hipStream_t)stream;
    const int64_t words = rg_div_up(num_nodes, 32);
    const int nblocks = (int)rg_max64(1, rg_div_up(words, kClaimWords));
    rg_status st;
    if ((st = rg_ensure(ctx, ctx->claim_bits, (size_t)rg_max64(words, 1) * 4)) != RG_OK) return st;
    if ((st = rg_ensure(ctx, ctx->claim_blk, (size_t)(nblocks + 1) * 4)) != RG_OK) return st;
    uint32_t* newbits = (uint32_t*)ctx->claim_bits.p;
    int32_t* blk = (int32_t*)ctx->claim_blk.p;
    k_claim_count<<<nblocks, 256, 0, s>>>((const uint32_t*)ctx->visited.p, words, group, claimed, newbits, cache->home, blk);
    RG_LAUNCH_CHECK(ctx, "k_claim_count");
    const int scanned = nblocks > kClaimSelfScan;
    if (scanned) {
        k_claim_scan<<<1, 1024, 0, s>>>(blk, nblocks);
        RG_LAUNCH_CHECK(ctx, "k_claim_scan");
    }
    k_claim_emit<<<nblocks, 256, 0, s>>>(newbits, words, cache->home, blk, scanned, plan->offsets + segment, plan->list_capacity, plan->list);
    RG_LAUNCH_CHECK(ctx, "k_claim_emit");
    return RG_OK;
}

}  // extern "C"

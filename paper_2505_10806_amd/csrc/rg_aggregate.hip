// Consumer of the gathered features: mean aggregation over a sampled block (Eq. 1 with AGG = mean, the
// GraphSAGE aggregator of Section II-A).  Bandwidth-bound: every sampled edge reads one feature row.
#include "rg_rowcopy.h"

namespace {

// agg[i] = (1/m_i) * sum over the block's edges e of row i, in edge order, of feat[nbr_local[e]].
// A wavefront is split into groups of L lanes per destination row; each lane owns chunk c0 (+ L, + 2L, ...) of the
// row and accumulates it in registers, E edges at a time so that E independent row loads are in flight.  Up to few_rows rows: L = 64, up to twice
// as many at least 32.
// Bound by the source rows' traffic behind L2 (270 k destinations of 5 edges on a power-law block, 256 floats: 1.31 GB of rows
// asked for, 27 % of the reads hit L2, so 0.96 GB from behind it, and 0.28 written in 196 us; 373 k distinct rows would be 0.38 GB).  E = 8 takes fan-outs of 5 in one step (E = 4: 206).
// Cutting the columns into one part per XCD, so that every L2 holds its part of more rows, was slower (8 parts 228, 4 parts 205).
template <int VEC, int E>
__global__ void __launch_bounds__(256) k_mean_aggregate(const int32_t* __restrict__ indptr, const int32_t* __restrict__ nbr_local,
                                                        int64_t n_dst, const int32_t* __restrict__ n_dst_dev,
                                                        const float* __restrict__ feat, int64_t feat_stride,
                                                        float* __restrict__ agg, int64_t agg_stride, int cpr, int log2L, int tail,
                                                        int64_t few_rows) {
    typedef typename RgVec<VEC>::type V;
    int64_t n_act = n_dst;
    if (n_dst_dev) { const int64_t d = *n_dst_dev; n_act = d < n_dst ? d : n_dst; }
    if (n_act <= few_rows) log2L = 6;
    else if (n_act < 2 * few_rows && log2L == 4) log2L = 5;
    const int lane = rg_lane();
    const int L = 1 << log2L;
    const int R = RG_WAVE >> log2L;
    const int sub = lane >> log2L;
    const int c0 = lane & (L - 1);
    const int64_t wave = ((int64_t)blockIdx.x * blockDim.x + threadIdx.x) >> 6;
    const int64_t nwaves = ((int64_t)gridDim.x * blockDim.x) >> 6;
    for (int64_t row0 = wave * R; row0 < n_act; row0 += nwaves * R) {
        const int64_t i = row0 + sub;
        if (i >= n_act) continue;
        const int e0 = indptr[i], e1 = indptr[i + 1];
        const float m = (float)(e1 - e0);
        V* dst = (V*)(agg + i * agg_stride);
        for (int c = c0; c < cpr; c += L) {
            V acc;
#pragma unroll
            for (int q = 0; q < VEC; ++q) ((float*)&acc)[q] = 0.0f;
            for (int e = e0; e < e1; e += E) {
                V val[E];
#pragma unroll
                for (int u = 0; u < E; ++u)
                    if (e + u < e1) val[u] = ((const V*)(feat + (int64_t)nbr_local[e + u] * feat_stride))[c];
#pragma unroll
                for (int u = 0; u < E; ++u)
                    if (e + u < e1) {
#pragma unroll
                        for (int q = 0; q < VEC; ++q) ((float*)&acc)[q] += ((const float*)&val[u])[q];
                    }
            }
            if (e1 > e0) {
#pragma unroll
                for (int q = 0; q < VEC; ++q) ((float*)&acc)[q] = ((float*)&acc)[q] / m;
            }
            // a 16-byte chunk may reach into the sources' row padding: only the row's own floats are stored
            if (tail < VEC && c == cpr - 1) rg_store_head(&dst[c], acc, tail);
            else __builtin_nontemporal_store(acc, &dst[c]);
        }
    }
}

constexpr int64_t kFewRows = 8192;     // rows up to which a wavefront has one to itself (see rg_mean_aggregate)

}  // namespace

extern "C" {

rg_status rg_mean_aggregate(rg_ctx* ctx, const int32_t* indptr, const int32_t* nbr_local, int64_t n_dst,
                            const int32_t* n_dst_dev, const float* feat, int64_t feat_stride, int32_t dim,
                            float* agg, int64_t agg_stride, void* stream) {
    if (!ctx) return RG_ERR_INVALID_ARG;
    RG_REQUIRE(ctx, n_dst >= 0 && n_dst <= (1ll << 31) - 1, "rg_mean_aggregate: n_dst = %lld out of range", (long long)n_dst);
    RG_REQUIRE(ctx, dim >= 1 && feat_stride >= dim && agg_stride >= dim, "rg_mean_aggregate: bad dim / stride");
    if (n_dst == 0) return RG_OK;
    RG_REQUIRE(ctx, indptr && nbr_local && feat && agg, "rg_mean_aggregate: null pointer");
    RG_HIP(ctx, hipSetDevice(ctx->device));
    hipStream_t s = (hipStream_t)stream;
    const void* ptrs[2] = {feat, agg};
    const int64_t strides[2] = {feat_stride, agg_stride};
    const int vec = rg_pick_vec(dim, ptrs, 2, strides, 2);
    RgRowShape shp = rg_row_shape(dim, vec);
    // Rows longer than a wavefront whose last step would idle most lanes: groups of 32 lanes instead if that takes a quarter fewer
    // lane steps and three lanes in four work, of 16 if none of theirs is idle (15 edges; 33 k rows of 80 chunks: 64 lanes 98 us, 32 lanes
    // 90, 16 lanes 82, of 76 chunks 101 / 97 / 98; 100 k rows of 65 chunks 298 / 311 / 354; 151 chunks, 160 / 192 steps: all 74; 301 chunks
    // of 8 bytes, 304 / 320: 97 with 16 lanes, 84 with 64).  A row then takes its group two to five passes over its edges one after the
    // other, so up to kFewRows rows, which leave wavefronts idle, keep whole ones (80 chunks, 15 edges: 256 rows 10 / 11 / 15 us, 2048 14 / 17 /
    // 28, 8192 26 / 26 / 34, 10,000 38 / 29 / 36, 16,384 51 / 44 / 43; of 2 edges 144 chunks, 8193 rows 12 / 12 / 15), and up to twice as many
    // take 32 lanes rather than 16.
    int64_t few_rows = 0;
    if (shp.cpr > RG_WAVE && n_dst > kFewRows) {
        const int64_t whole = rg_div_up(shp.cpr, RG_WAVE) * RG_WAVE, half = rg_div_up(shp.cpr, 32) * 32;
        if (half * 5 <= whole * 4 && shp.cpr * 4 >= half * 3) shp.log2L = 5;
        if (shp.cpr * 5 <= whole * 4 && shp.cpr % 16 == 0 && shp.cpr < half) shp.log2L = 4;
        if (shp.log2L < 6) few_rows = kFewRows;
    }
    const int rows_per_block = 4 * (RG_WAVE >> shp.log2L);
    // 32 workgroups per compute unit; with 16 / 32 / 64 of them the 270 k destinations above take 195 / 195 / 197 us, 100 k of 10 edges
    // and 256 floats 118 / 117 / 115, 200 k of 5 and 128 84 / 82 / 80, 200 k of 1 and 256 60 / 56 / 55.
    const int grid = (int)rg_max64(few_rows / 4, rg_max64(1, rg_min64(rg_div_up(n_dst, rows_per_block), (int64_t)ctx->num_cus * 32)));
    const int tok = rg_prof_begin(ctx, RG_K_AGGREGATE, s);
    if (vec == 4)
        k_mean_aggregate<4, 8><<<grid, 256, 0, s>>>(indptr, nbr_local, n_dst, n_dst_dev, feat, feat_stride, agg, agg_stride, shp.cpr, shp.log2L, shp.tail, few_rows);
    else if (vec == 2)
        k_mean_aggregate<2, 8><<<grid, 256, 0, s>>>(indptr, nbr_local, n_dst, n_dst_dev, feat, feat_stride, agg, agg_stride, shp.cpr, shp.log2L, shp.tail, few_rows);
    else
        k_mean_aggregate<1, 8><<<grid, 256, 0, s>>>(indptr, nbr_local, n_dst, n_dst_dev, feat, feat_stride, agg, agg_stride, shp.cpr, shp.log2L, shp.tail, few_rows);
    rg_prof_end(ctx, tok, s);
    RG_LAUNCH_CHECK(ctx, "k_mean_aggregate");
    return RG_OK;
}

}  // extern "C"

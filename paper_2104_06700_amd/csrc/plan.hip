// Degree-binning plan: the GPU-side replacement for dynamic scheduling over
// destination rows of very different length (Section 4.2, "Multithreading").
//
// Rows are grouped by row-length bin with a stable multi-way split (ascending
// row id inside a bin), rows of the last bin are cut into fixed-size pieces, and
// the per-vertex column counts (needed for MEAN backward and GCN_SYM scaling)
// are histogrammed.  Everything is integer work and fully deterministic.
#include <new>

#include "common.h"

namespace {

constexpr int kSplitThreads = 1024;  // rows per workgroup in the split kernels
constexpr int kSplitWaves = kSplitThreads / 64;

struct Thresholds {
    int32_t k;
    int64_t t[GNN_MAX_THRESHOLDS];
};

__device__ __forceinline__ int64_t load_ip(const void *indptr, int ip64, int64_t i) {
    return ip64 ? static_cast<const int64_t *>(indptr)[i]
                : static_cast<int64_t>(static_cast<const int32_t *>(indptr)[i]);
}

__device__ __forceinline__ int bin_of(int64_t deg, const Thresholds &thr) {
    int b = 0;
    for (int i = 0; i < thr.k; ++i) b += (thr.t[i] <= deg) ? 1 : 0;
    return b;
}

__global__ void __launch_bounds__(256) count_cols_kernel(const int32_t *__restrict__ indices, int64_t E,
                                                         int32_t *__restrict__ col_counts) {
    int64_t stride = int64_t(gridDim.x) * blockDim.x;
    for (int64_t e = int64_t(blockIdx.x) * blockDim.x + threadIdx.x; e < E; e += stride)
        atomicAdd(&col_counts[indices[e]], 1);
}

// 256 buckets over the count axis: counts below 16 one bucket each, then 8 buckets per octave.
__device__ __forceinline__ int count_bucket(int c) {
    if (c < 16) return c;
    const int o = 31 - __clz(c);
    return 16 + (o - 4) * 8 + ((c >> (o - 3)) & 7);
}

// What one pass over the rows of a graph produces, in device memory until plan_place_kernel hands it to the host.
struct RowTotals {
    unsigned long long bucket_vertices[256], bucket_edges[256];  // histogram of the column counts (gnn_plan_top_share)
    unsigned long long bin_edges[GNN_MAX_BINS];                  // edges of the rows of each bin
    unsigned long long n_chunks;                                 // pieces of the hub rows
    long long bin_begin[GNN_MAX_BINS];                           // first row of each bin
    int unordered;                                               // of kSplitThreads rows: sources in descending order (plan_order_kernel)
};
static_assert(sizeof(RowTotals) <= size_t(GNN_HOST_BLOCK_BYTES), "fits a host block");

// One graph orientation of a pair that is set up side by side (blockIdx.y).
struct PlanJob {
    const void *indptr;
    const void *other_indptr;  // of the transposed graph, whose row lengths are the column counts; null: col_counts is filled
    int32_t *col_counts;
    int64_t *block_counts;
    RowTotals *totals;         // zeroed
    RowTotals *host;
    int32_t *row_perm;
    int4 *row_info;            // or null
    int64_t *hub_offsets;
    int64_t *chunks;
    uint32_t *hub_done;
};
struct PlanJobs {
    PlanJob job[2];
    int64_t N, n_blocks, hub_chunk;
    int32_t ip64, nb;
    Thresholds thr;
};

// Whether the rows list their sources in ascending order, as a sorted graph has them: two edges of each of kSplitThreads rows, a
// third and two thirds into the row, compared.  One workgroup; the result goes to the host.
__global__ void __launch_bounds__(kSplitThreads) plan_order_kernel(const void *indptr, int ip64, const int32_t *__restrict__ indices,
                                                                   int64_t N, int64_t E, RowTotals *host) {
    const int64_t v = int64_t(threadIdx.x) * N / kSplitThreads;
    const int64_t e0 = load_ip(indptr, ip64, v), len = load_ip(indptr, ip64, v + 1) - e0;
    bool descending = false;
    if (e0 >= 0 && len > 1 && e0 + len <= E) descending = indices[e0 + len / 3] > indices[e0 + len * 2 / 3];
    const int n = __syncthreads_count(descending);
    if (threadIdx.x == 0) host->unordered = n;
}

// Per 1024 rows: block_counts[b * n_blocks + blk] = rows of bin b among them; and the totals over all rows, integer sums, so
// that the order of the additions does not matter.
__global__ void __launch_bounds__(kSplitThreads) plan_rows_kernel(PlanJobs jobs) {
    __shared__ unsigned long long sv[256], se[256], bin_edges[GNN_MAX_BINS], pieces;
    __shared__ int counts[GNN_MAX_BINS];
    const PlanJob &job = jobs.job[blockIdx.y];
    const int t = threadIdx.x;
    if (t < 256) sv[t] = se[t] = 0;
    if (t < GNN_MAX_BINS) bin_edges[t] = 0;
    if (t == 0) pieces = 0;
    for (int64_t blk = blockIdx.x; blk < jobs.n_blocks; blk += gridDim.x) {
        if (t < GNN_MAX_BINS) counts[t] = 0;
        __syncthreads();
        const int64_t v = blk * kSplitThreads + t;
        if (v < jobs.N) {
            const int64_t deg = load_ip(job.indptr, jobs.ip64, v + 1) - load_ip(job.indptr, jobs.ip64, v);
            const int bin = bin_of(deg, jobs.thr);
            atomicAdd(&counts[bin], 1);
            if (deg > 0) atomicAdd(&bin_edges[bin], static_cast<unsigned long long>(deg));
            if (jobs.hub_chunk > 0 && bin == jobs.nb - 1 && deg > 0)
                atomicAdd(&pieces, static_cast<unsigned long long>((deg + jobs.hub_chunk - 1) / jobs.hub_chunk));
            int c;
            if (job.other_indptr) {
                c = static_cast<int>(load_ip(job.other_indptr, jobs.ip64, v + 1) - load_ip(job.other_indptr, jobs.ip64, v));
                job.col_counts[v] = c;
            } else {
                c = job.col_counts[v];
            }
            const int b = count_bucket(c);
            atomicAdd(&sv[b], 1ull);
            atomicAdd(&se[b], static_cast<unsigned long long>(c));
        }
        __syncthreads();
        if (t < jobs.nb) job.block_counts[int64_t(t) * jobs.n_blocks + blk] = counts[t];
        __syncthreads();
    }
    if (t < 256) {
        if (sv[t]) atomicAdd(&job.totals->bucket_vertices[t], sv[t]);
        if (se[t]) atomicAdd(&job.totals->bucket_edges[t], se[t]);
    }
    if (t < GNN_MAX_BINS && bin_edges[t]) atomicAdd(&job.totals->bin_edges[t], bin_edges[t]);
    if (t == 0 && pieces) atomicAdd(&job.totals->n_chunks, pieces);
}

// Stable placement: row v goes to block_counts[bin][blk] (prefix sums by now) + (#rows of the same bin before it in the block).
// The first workgroup hands the totals to the host.
__global__ void __launch_bounds__(kSplitThreads) plan_place_kernel(PlanJobs jobs) {
    __shared__ int wave_tot[kSplitWaves][GNN_MAX_BINS];
    const PlanJob &job = jobs.job[blockIdx.y];
    const int lane = threadIdx.x & 63;
    const int wave = threadIdx.x >> 6;
    if (blockIdx.x == 0) {
        const int t = threadIdx.x;
        if (t < 256) {
            job.host->bucket_vertices[t] = job.totals->bucket_vertices[t];
            job.host->bucket_edges[t] = job.totals->bucket_edges[t];
        }
        if (t < jobs.nb) {
            job.host->bin_edges[t] = job.totals->bin_edges[t];
            job.host->bin_begin[t] = job.block_counts[int64_t(t) * jobs.n_blocks];
        }
        if (t == 0) job.host->n_chunks = job.totals->n_chunks;
    }
    int64_t v = int64_t(blockIdx.x) * kSplitThreads + threadIdx.x;
    int bin = -1;
    int64_t begin = 0, deg = 0;
    if (v < jobs.N) {
        begin = load_ip(job.indptr, jobs.ip64, v);
        deg = load_ip(job.indptr, jobs.ip64, v + 1) - begin;
        bin = bin_of(deg, jobs.thr);
    }
    int rank_in_wave = 0;
    for (int b = 0; b < jobs.nb; ++b) {
        unsigned long long m = __ballot(bin == b);
        if (bin == b) rank_in_wave = __popcll(m & ((1ull << lane) - 1ull));
        if (lane == 0) wave_tot[wave][b] = __popcll(m);
    }
    __syncthreads();
    if (bin >= 0) {
        int before = 0;
        for (int w = 0; w < wave; ++w) before += wave_tot[w][bin];
        int64_t pos = job.block_counts[int64_t(bin) * jobs.n_blocks + blockIdx.x] + before + rank_in_wave;
        job.row_perm[pos] = static_cast<int32_t>(v);
        if (job.row_info) job.row_info[pos] = make_int4(static_cast<int32_t>(v), static_cast<int32_t>(begin), static_cast<int32_t>(deg), 0);
    }
}

// pieces of the hub rows, zero behind the last of them: the arrays are sized before the host knows how many there are
__global__ void __launch_bounds__(256) hub_count_kernel(PlanJobs jobs, int64_t n_bound) {
    const PlanJob &job = jobs.job[blockIdx.y];
    const int64_t hub_begin = job.block_counts[int64_t(jobs.nb - 1) * jobs.n_blocks];
    const int64_t stride = int64_t(gridDim.x) * blockDim.x;
    for (int64_t i = int64_t(blockIdx.x) * blockDim.x + threadIdx.x; i < n_bound; i += stride) {
        int64_t pieces = 0;
        if (hub_begin + i < jobs.N) {
            const int64_t v = job.row_perm[hub_begin + i];
            const int64_t deg = load_ip(job.indptr, jobs.ip64, v + 1) - load_ip(job.indptr, jobs.ip64, v);
            pieces = (deg + jobs.hub_chunk - 1) / jobs.hub_chunk;
        }
        job.hub_offsets[i] = pieces;
    }
}

__global__ void __launch_bounds__(256) hub_fill_kernel(PlanJobs jobs, int64_t n_bound, int64_t chunk_bound) {
    const PlanJob &job = jobs.job[blockIdx.y];
    const int64_t hub_begin = job.block_counts[int64_t(jobs.nb - 1) * jobs.n_blocks];
    const int64_t stride = int64_t(gridDim.x) * blockDim.x;
    for (int64_t i = int64_t(blockIdx.x) * blockDim.x + threadIdx.x; i < n_bound && hub_begin + i < jobs.N; i += stride) {
        const int64_t v = job.row_perm[hub_begin + i];
        int64_t b = load_ip(job.indptr, jobs.ip64, v);
        const int64_t end = load_ip(job.indptr, jobs.ip64, v + 1);
        int64_t c = job.hub_offsets[i];
        if (c < chunk_bound)
            for (int s = 0; s < 8; ++s) job.hub_done[8 * c + s] = 0;
        for (; b < end && c < chunk_bound; b += jobs.hub_chunk, ++c) {
            job.chunks[3 * c + 0] = v;
            job.chunks[3 * c + 1] = b;
            job.chunks[3 * c + 2] = b + jobs.hub_chunk < end ? b + jobs.hub_chunk : end;
        }
    }
}

__global__ void __launch_bounds__(256) edge_scale_kernel(const int32_t *__restrict__ indices, int64_t E,
                                                         const int32_t *__restrict__ col_counts, int mode,
                                                         float *__restrict__ out) {
    int64_t stride = int64_t(gridDim.x) * blockDim.x;
    for (int64_t e = int64_t(blockIdx.x) * blockDim.x + threadIdx.x; e < E; e += stride) {
        int c = col_counts[indices[e]];
        float d = static_cast<float>(c > 1 ? c : 1);
        out[e] = mode == 3 ? 1.0f / static_cast<float>(c + 1) : (mode == 1 ? 1.0f / d : 1.0f / sqrtf(d));
    }
}

int grid_for(int64_t n, int block, int64_t cap = (int64_t(1) << 20)) {
    int64_t g = (n + block - 1) / block;
    if (g < 1) g = 1;
    if (g > cap) g = cap;
    return static_cast<int>(g);
}

}  // namespace

extern "C" GNN_API void gnn_plan_default_params(gnn_plan_params *p) {
    if (!p) return;
    *p = gnn_plan_params{};
    const int64_t t[] = {1, 2, 4, 8, 16, 32, 64, 128, 256, 512, 1024, 2048, 4096};
    p->n_thresholds = static_cast<int32_t>(sizeof(t) / sizeof(t[0]));
    for (int i = 0; i < p->n_thresholds; ++i) p->thresholds[i] = t[i];
    p->hub_chunk = 1024;
}

int gnn_plan_edge_scale(gnn_plan *plan, const int32_t *indices, int mode, hipStream_t stream, const float **out) {
    if (!plan || !out || mode < 1 || mode > 3) return GNN_ERR_INVALID_ARG;
    float *&arr = plan->edge_scale[mode - 1];
    if (!arr && plan->n_edges > 0) {
        if (!indices) return GNN_ERR_INVALID_ARG;
        (void)hipGetLastError();
        if (!gnn_dev_alloc(&arr, plan->n_edges, stream)) return GNN_ERR_ALLOC;
        edge_scale_kernel<<<grid_for(plan->n_edges, 256, 1 << 16), 256, 0, stream>>>(indices, plan->n_edges, plan->col_counts, mode, arr);
        if (hipGetLastError() != hipSuccess) {  // an unfilled array must not serve a later call
            gnn_dev_free(arr);
            arr = nullptr;
            return GNN_ERR_LAUNCH;
        }
    }
    *out = arr;
    return GNN_OK;
}

__global__ void __launch_bounds__(256) edge_operand_kernel(const float *__restrict__ fE, int64_t lde,
                                                           const int64_t *__restrict__ edge_ids, int64_t E,
                                                           float *__restrict__ out) {
    const int64_t stride = int64_t(gridDim.x) * blockDim.x;
    for (int64_t e = int64_t(blockIdx.x) * blockDim.x + threadIdx.x; e < E; e += stride) {
        const int64_t id = edge_ids ? edge_ids[e] : e;
        __builtin_nontemporal_store(fE[id * lde], out + e);
    }
}

typedef int64_t i64x2_any __attribute__((ext_vector_type(2), aligned(8)));
typedef float f32x2_any __attribute__((ext_vector_type(2), aligned(4)));
constexpr int64_t kOperandEdges = 48000000;
constexpr int kOperandRows = 2;                // rows of a wavefront at a time ...
// ... and 16 wavefronts per compute unit where an eighth of a row has most of a wavefront's 128 loads, because more rows in flight touch more lines than
// an L2 holds, else 32 (a vertex gradient of 4 columns, us, 16 / 24 / 32, mild skew: 600 edges a row, 133 K rows 1416 / 1481 / 1508, 100 K 1045 / 1013 /
// 1047; 395, 200 K 1576 / 1475 / 1467; 316, 250 K 1683 / 1521 / 1476; 226, 350 K 1993 / 1709 / 1616; 208, 240 K 1295 / 1107 / 1007).
constexpr int64_t kOperandLong = 500;

// The same with the k-th eighth of every row on XCD k, rows in ascending order.  Where the operand is that of a transposed graph an
// id is a place in the row of the edge's other end, so an eighth leads to an eighth of those rows, and a line of 32 scalars is met
// again by the next few hundred rows: it waits for them in the L2 (133 K rows: 17,000 lines) where the plain kernel misses on every
// one (62 G loads/s, the rate behind the L2s; 268 G from an L2).  What remains is latency: ids, scalars and the turn between rows.
// Any ids give the right result.  133 K rows, 79 M edges, mild skew 1.27 -> 0.93 ms, strong skew 1.03 -> 1.07 (see below).
__global__ void __launch_bounds__(256) edge_operand_rows_kernel(const float *__restrict__ fE, int64_t lde, const int64_t *__restrict__ edge_ids,
                                                                const void *indptr, int ip64, int64_t N, float *__restrict__ out) {
    constexpr int ROWS = kOperandRows;
    const int lane = threadIdx.x & 63;
    const int part = int(blockIdx.x & 7);
    const int64_t step = int64_t(gridDim.x >> 3) * 4 * ROWS;
    auto pointer = [&](int64_t row) {
        row = row < N ? row : N;
        return ip64 ? static_cast<const int64_t *>(indptr)[row] : int64_t(static_cast<const int32_t *>(indptr)[row]);
    };
    int64_t first = (int64_t(blockIdx.x >> 3) * 4 + (threadIdx.x >> 6)) * ROWS;
    const int at = lane < ROWS ? lane : ROWS;
    // 128 edges of the parts of ROWS rows at a time; the rows' pointers arrive a group of rows ahead, the ids a turn ahead
    struct Ids { int64_t begin[ROWS], id[ROWS][2]; int n[ROWS]; };
    int64_t begin[ROWS];
    int left[ROWS], longest = 0;
    auto start_rows = [&](int64_t mine) {
        longest = 0;
#pragma unroll
        for (int r = 0; r < ROWS; ++r) {
            const int64_t e0 = __shfl(mine, r), len = __shfl(mine, r + 1) - e0;
            const int64_t b = len * part >> 3;
            begin[r] = e0 + b;
            left[r] = int((len * (part + 1) >> 3) - b);
            longest = left[r] > longest ? left[r] : longest;
        }
        longest = __builtin_amdgcn_readfirstlane(longest);
    };
    auto fetch = [&](Ids &x) {
#pragma unroll
        for (int r = 0; r < ROWS; ++r) {
            x.begin[r] = begin[r];
            x.n[r] = left[r];
            const int i = 2 * lane;
            x.id[r][0] = x.id[r][1] = 0;
            const int64_t *q = edge_ids + begin[r] + i;
            if (i + 1 < left[r]) {
                const i64x2_any two = __builtin_nontemporal_load(reinterpret_cast<const i64x2_any *>(q));  // not in the place of scalars that wait: 1.44 -> 1.42 ms
                x.id[r][0] = two.x;
                x.id[r][1] = two.y;
            } else if (i < left[r]) {
                x.id[r][0] = *q;
            }
            begin[r] += 128;
            left[r] -= 128;
        }
        longest -= 128;
    };
    if (first >= N) return;
    Ids nxt;
    start_rows(pointer(first + at));
    int64_t p_nxt = pointer(first + step + at);
    fetch(nxt);
    for (;;) {
        const Ids cur = nxt;
        float v[ROWS][2];
#pragma unroll
        for (int r = 0; r < ROWS; ++r)
#pragma unroll
            for (int j = 0; j < 2; ++j)
                if (2 * lane + j < cur.n[r]) v[r][j] = fE[cur.id[r][j] * lde];
        bool more = true;
        if (longest <= 0) {
            first += step;
            more = first < N;
            if (more) {
                start_rows(p_nxt);
                p_nxt = pointer(first + step + at);
            }
        }
        if (more) fetch(nxt);
#pragma unroll
        for (int r = 0; r < ROWS; ++r) {
            float *q = out + cur.begin[r] + 2 * lane;
            if (2 * lane + 1 < cur.n[r]) *reinterpret_cast<f32x2_any *>(q) = f32x2_any{v[r][0], v[r][1]};
            else if (2 * lane < cur.n[r]) *q = v[r][0];
        }
        if (!more) break;
    }
}

int gnn_plan_edge_operand(gnn_plan *plan, const float *fE, int64_t lde, const int64_t *edge_ids, const void *indptr, int ip64, hipStream_t stream,
                          const float **out) {
    if (!plan || !out || !fE || lde < 1) return GNN_ERR_INVALID_ARG;
    *out = nullptr;
    if (plan->n_edges == 0) return GNN_OK;
    (void)hipGetLastError();
    if (!plan->edge_operand && !gnn_dev_alloc(&plan->edge_operand, plan->n_edges, stream)) return GNN_ERR_ALLOC;
    // Long rows, and more scalars than the caches behind the L2s hold well (a vertex gradient of 4 columns, plain -> by rows, ms: 100 K rows,
    // 60 M edges 1.25 -> 1.05, 200 K, 79 M 1.88 -> 1.56, 250 K, 79 M 1.96 -> 1.68 / strong skew 1.68 -> 1.65, 350 K 2.06 -> 1.97;
    // below, 100 K, 40 M 0.80 -> 0.77, 133 K, 40 M 0.83 -> 0.85, 60 K, 20 M 0.34 -> 0.41).  Not where few vertices have most of the edges: the lines of
    // their rows stay in the L2s either way, and an eighth of a very long row is one wavefront's work (share of the most-gathered twentieth, ms:
    // 0.39 133 K, 79 M 1.85 -> 1.45; 0.42 100 K, 50 M 0.99 -> 0.93, 350 K, 79 M 2.14 -> 2.02; 0.46 133 K, 79 M 1.74 -> 1.50; 0.50 250 K, 79 M 1.93 -> 1.70; 0.52 350 K,
    // 79 M 2.02 -> 1.98; 0.53 100 K, 60 M 1.10 -> 1.14; 0.58 133 K, 79 M 1.57 -> 1.60; 0.60 133 K, 60 M 1.14 -> 1.21; 0.61 133 K, 50 M 0.91 -> 1.01; 0.65 250 K, 79 M
    // 1.70 -> 1.68, by seed 1.63 to 1.74; 0.66 250 K, 60 M 1.25 -> 1.42).
    if (edge_ids && plan->n_edges >= kOperandEdges && plan->n_edges >= 200 * plan->n_rows &&
        gnn_plan_top_share(plan, plan->n_rows / 20) < kStrongSkew)
        edge_operand_rows_kernel<<<8 * 32 * (plan->n_edges >= kOperandLong * plan->n_rows ? 4 : 8), 256, 0, stream>>>(fE, lde, edge_ids, indptr, ip64, plan->n_rows, plan->edge_operand);
    else
        edge_operand_kernel<<<grid_for(plan->n_edges, 256, 1 << 16), 256, 0, stream>>>(fE, lde, edge_ids, plan->n_edges, plan->edge_operand);
    if (hipGetLastError() != hipSuccess) return GNN_ERR_LAUNCH;
    *out = plan->edge_operand;
    return GNN_OK;
}

__global__ void __launch_bounds__(256) flag_cold_kernel(const int32_t *__restrict__ indices, int64_t E,
                                                        const int32_t *__restrict__ counts, int threshold,
                                                        int32_t *__restrict__ out) {
    const int64_t stride = int64_t(gridDim.x) * blockDim.x;
    for (int64_t e = int64_t(blockIdx.x) * blockDim.x + threadIdx.x; e < E; e += stride) {
        const int32_t u = indices[e];
        out[e] = counts[u] < threshold ? int32_t(uint32_t(u) | 0x80000000u) : u;
    }
}

// smallest count that falls into bucket b of count_bucket()
static int64_t bucket_lower_bound(int b) {
    if (b < 16) return b;
    const int o = 4 + (b - 16) / 8, m = (b - 16) % 8;
    return int64_t(8 + m) << (o - 3);
}

// Cold hints.  With column slices an XCD's L2 holds one line each of 32,768 rows; rows that are
// gathered rarely pass through it without ever being hit again and only displace warmer rows.
// Measured on the 2.45 M-vertex power-law graph: fetching the sources outside the ~160 K
// most-gathered vertices (13-19 % of the gathers) with non-temporal loads takes 4-6 % off a call
// (F=256: 13.45 -> 12.8 ms, F=100: 6.82 -> 6.4 ms), while marking warmer sources, or any sources
// of a graph whose vertices nearly all fit that set (the 233 K- and 133 K-vertex graphs), costs
// time: the non-temporal path is slower per byte and forfeits hits.  Hence the gate: the graph has
// at least 8 x 163,840 vertices and the cold sources receive 5-30 % of the gathers.
int gnn_plan_cold_indices(gnn_plan *plan, const int32_t *indices, bool force, hipStream_t stream, const int32_t **out) {
    *out = nullptr;
    if (!plan || plan->n_edges <= 0) return GNN_OK;
    if (plan->cold_decided && plan->cold_forced != (force ? 1 : 0)) {  // built under the other rule: build again
        gnn_plan_drop(plan, plan->cold_indices, plan->cold_recorded);
        plan->cold_indices = nullptr;
        plan->cold_decided = 0;
        plan->cold_recorded = false;
    }
    if (!plan->cold_decided) {
        const int64_t warm = force ? (plan->n_rows + 3) / 4 : int64_t(5) * 32768;
        bool enable = force;
        if (!force && plan->n_rows >= 8 * warm) {
            const double cold_share = 1.0 - gnn_plan_top_share(plan, warm);
            enable = cold_share >= 0.05 && cold_share <= 0.30;
        }
        if (enable) {
            // count threshold: lower bound of the bucket in which the `warm` most-gathered vertices end
            int64_t seen = 0, thr = 1;
            for (int b = 255; b >= 0; --b) {
                seen += plan->bucket_vertices[b];
                if (seen >= warm) { thr = bucket_lower_bound(b); break; }
            }
            if (thr < 1) thr = 1;
            if (!indices) return GNN_ERR_INVALID_ARG;
            (void)hipGetLastError();
            if (!gnn_dev_alloc(&plan->cold_indices, plan->n_edges, stream)) return GNN_ERR_ALLOC;
            plan->cold_threshold = int32_t(thr > INT32_MAX ? INT32_MAX : thr);
            flag_cold_kernel<<<grid_for(plan->n_edges, 256, 1 << 16), 256, 0, stream>>>(indices, plan->n_edges, plan->col_counts,
                                                                                       plan->cold_threshold, plan->cold_indices);
            if (hipGetLastError() != hipSuccess) {
                gnn_dev_free(plan->cold_indices);
                plan->cold_indices = nullptr;
                return GNN_ERR_LAUNCH;
            }
        }
        plan->cold_decided = 1;
        plan->cold_forced = force ? 1 : 0;
    }
    *out = plan->cold_indices;
    if (*out && !plan->cold_recorded) plan->cold_recorded = gnn_capturing(stream);
    return GNN_OK;
}

// lens[i] = length of the row at position i of row_perm
__global__ void __launch_bounds__(256) plan_order_lens_kernel(const int32_t *__restrict__ row_perm, int64_t N,
                                                              const void *__restrict__ indptr, int ip64,
                                                              int64_t *__restrict__ lens) {
    const int64_t stride = int64_t(gridDim.x) * blockDim.x;
    for (int64_t i = int64_t(blockIdx.x) * blockDim.x + threadIdx.x; i < N; i += stride) {
        const int64_t v = row_perm[i];
        lens[i] = load_ip(indptr, ip64, v + 1) - load_ip(indptr, ip64, v);
    }
}

// Copies the rows' edge lists to their plan-order positions, mapping every source id to its rank and flagging the cold ones
// (rank >= warm) in bit 31.  A workgroup writes kFillEdges consecutive positions whatever rows they belong to: it looks up
// the row of the first, marks where the further rows begin, and spreads the marks with a running maximum.  (One wavefront
// per row was bound by the longest rows' chains of loads: 3.1 M edges, 61,226 rows 94 us.)
constexpr int kFillEdges = 2048;

__global__ void __launch_bounds__(256) plan_order_fill_kernel(const int32_t *__restrict__ row_perm, int64_t N, int64_t E,
                                                              const void *__restrict__ indptr, int ip64,
                                                              const int64_t *__restrict__ p_indptr,
                                                              const int32_t *__restrict__ indices,
                                                              const int32_t *__restrict__ rank, int64_t warm,
                                                              int32_t *__restrict__ out) {
    constexpr int PER = kFillEdges / 256;
    __shared__ int32_t owner[kFillEdges];
    __shared__ int32_t wave_max[4];
    const int t = threadIdx.x, lane = t & 63, wave = t >> 6;
    const int64_t first = int64_t(blockIdx.x) * kFillEdges;
    const int64_t end = first + kFillEdges < E ? first + kFillEdges : E;
    int64_t lo = 0, hi = N;  // the last row that begins at `first` or before
    while (hi - lo > 1) {
        const int64_t mid = (lo + hi) >> 1;
        if (p_indptr[mid] <= first) lo = mid; else hi = mid;
    }
    const int32_t row0 = int32_t(lo);
#pragma unroll
    for (int k = 0; k < PER; ++k) owner[k * 256 + t] = row0;
    __syncthreads();
    for (int64_t i0 = int64_t(row0) + 1; i0 < N; i0 += 256) {
        const int64_t i = i0 + t;
        const int64_t begin = i < N ? p_indptr[i] : E;
        if (begin < end) atomicMax(&owner[begin - first], int32_t(i));  // of rows that begin together, the last has the edges
        if (__syncthreads_or(begin >= end)) break;
    }
    __syncthreads();
    int32_t mine[PER], top = 0;
#pragma unroll
    for (int k = 0; k < PER; ++k) {
        const int32_t x = owner[t * PER + k];
        top = x > top ? x : top;
        mine[k] = top;
    }
    int32_t upto = top;
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) {
        const int32_t y = __shfl_up(upto, off);
        if (lane >= off && y > upto) upto = y;
    }
    if (lane == 63) wave_max[wave] = upto;
    int32_t before = __shfl_up(upto, 1);
    if (lane == 0) before = 0;
    __syncthreads();
    for (int w = 0; w < wave; ++w) before = wave_max[w] > before ? wave_max[w] : before;
#pragma unroll
    for (int k = 0; k < PER; ++k) owner[t * PER + k] = mine[k] > before ? mine[k] : before;
    __syncthreads();
#pragma unroll
    for (int k = 0; k < PER; ++k) {
        const int64_t at = first + k * 256 + t;
        if (at >= end) continue;
        const int32_t i = owner[k * 256 + t];
        const int64_t from = load_ip(indptr, ip64, row_perm[i]) + (at - p_indptr[i]);
        const int32_t r = rank[indices[from]];
        out[at] = r >= warm ? int32_t(uint32_t(r) | 0x80000000u) : r;
    }
}

// The hub pieces in plan-order coordinates: (row, begin, end, original minus plan-order position).
__global__ void __launch_bounds__(256) plan_order_chunks_kernel(int64_t n_hub, int64_t hub_begin,
                                                                const void *__restrict__ indptr, int ip64,
                                                                const int64_t *__restrict__ p_indptr,
                                                                const int64_t *__restrict__ offsets,
                                                                const int64_t *__restrict__ chunks,
                                                                int64_t *__restrict__ p_chunks) {
    const int64_t i = int64_t(blockIdx.x) * blockDim.x + threadIdx.x;
    if (i >= n_hub) return;
    for (int64_t c = offsets[i]; c < offsets[i + 1]; ++c) {
        const int64_t v = chunks[3 * c];
        const int64_t delta = load_ip(indptr, ip64, v) - p_indptr[hub_begin + i];
        p_chunks[4 * c + 0] = v;
        p_chunks[4 * c + 1] = chunks[3 * c + 1] - delta;
        p_chunks[4 * c + 2] = chunks[3 * c + 2] - delta;
        p_chunks[4 * c + 3] = delta;
    }
}

// Rank layout.  The padded copy of the gathered matrix is plan-owned, so its row order is free:
// rows are stored by descending column count.  The dense tail table then holds the tails of the
// most-gathered vertices in its first lines (8 rows per line at F = 100), the warm part of the
// main table is one contiguous range, and the cold rule is exact (rank >= warm).  The index copy
// that maps sources to ranks is laid out in plan order at the same time, because the rows that a
// workgroup processes side by side are neighbours in row_perm, not in the CSR: read from the
// caller's CSR, their edge lists are scattered ~200-byte pieces whose 128-byte lines are fetched
// more than once.  Measured on the 2.45 M-vertex graph: rank order F=100 6.21 -> 6.05 ms, F=256
// 12.6 -> 12.26 ms; plan order on top of it: see the kernel profile.  The cold gate is that of
// gnn_plan_cold_indices.
int gnn_plan_rank_indices(gnn_plan *plan, const void *indptr, const int32_t *indices, bool force_cold, hipStream_t stream,
                          gnn_rank_layout *out) {
    *out = gnn_rank_layout{};
    if (!plan || plan->n_edges <= 0 || plan->n_rows <= 0) return GNN_OK;
    if (plan->rank_indices && plan->rank_forced != (force_cold ? 1 : 0)) {  // flagged under the other rule: build again
        gnn_plan_drop(plan, plan->rank_indices, plan->rank_recorded);
        gnn_plan_drop(plan, plan->p_indptr, plan->rank_recorded);
        gnn_plan_drop(plan, plan->p_chunks, plan->rank_recorded);
        plan->rank_indices = nullptr;
        plan->p_indptr = nullptr;
        plan->p_chunks = nullptr;
        plan->rank_recorded = false;
    }
    if (!plan->rank_indices) {
        if (!indices || !indptr) return GNN_ERR_INVALID_ARG;
        const int64_t N = plan->n_rows;
        (void)hipGetLastError();
        if (!plan->rank) {
            if (!gnn_dev_alloc(&plan->rank, N, stream)) return GNN_ERR_ALLOC;
            int top = 255;  // the counts lie below the bound of the next bucket
            while (top > 0 && plan->bucket_vertices[top] == 0) --top;
            const int64_t max_count = top < 255 ? bucket_lower_bound(top + 1) - 1 : INT32_MAX;
            int rc = gnn_rank_by_count(plan->col_counts, N, max_count, plan->rank, stream);
            if (rc != GNN_OK) { gnn_dev_free(plan->rank); plan->rank = nullptr; return rc; }
        }
        // The indices of this copy are ranks, so the kernel finds the cold sources by comparing with
        // the warm-set size of the call; bit 31 is only set when the tests force it.
        const int64_t warm = force_cold ? (N + 3) / 4 : N;
        int64_t *p_indptr = nullptr, *p_chunks = nullptr;
        int32_t *idx = nullptr;
        auto fail = [&](int s) { gnn_dev_free(p_indptr); gnn_dev_free(p_chunks); gnn_dev_free(idx); return s; };
        gnn_dev_ptr<int64_t> sums;
        if (!gnn_dev_alloc(&p_indptr, N + 1, stream) || !gnn_dev_alloc(&idx, plan->n_edges, stream)) return fail(GNN_ERR_ALLOC);
        if (plan->n_chunks > 0 && !gnn_dev_alloc(&p_chunks, 4 * plan->n_chunks, stream)) return fail(GNN_ERR_ALLOC);
        if (!sums.alloc_on(gnn_scan_sums_elems(N), stream)) return fail(GNN_ERR_ALLOC);
        plan_order_lens_kernel<<<grid_for(N, 256), 256, 0, stream>>>(plan->row_perm, N, indptr, plan->indptr_is_64, p_indptr);
        const int scan_rc = gnn_scan_exclusive_i64(p_indptr, N, 1, 0, sums.p, stream);
        if (scan_rc != GNN_OK) return fail(scan_rc);
        plan_order_fill_kernel<<<static_cast<unsigned>((plan->n_edges + kFillEdges - 1) / kFillEdges), 256, 0, stream>>>(
            plan->row_perm, N, plan->n_edges, indptr, plan->indptr_is_64, p_indptr, indices, plan->rank, warm, idx);
        if (plan->n_chunks > 0) {
            const int64_t hub_begin = plan->bin_offsets[plan->n_bins - 1];
            plan_order_chunks_kernel<<<grid_for(plan->n_hub_rows, 256), 256, 0, stream>>>(
                plan->n_hub_rows, hub_begin, indptr, plan->indptr_is_64, p_indptr, plan->hub_chunk_offsets, plan->chunks, p_chunks);
        }
        if (hipGetLastError() != hipSuccess) return fail(GNN_ERR_LAUNCH);
        plan->p_indptr = p_indptr;
        plan->p_chunks = p_chunks;
        plan->rank_indices = idx;
        plan->rank_forced = force_cold ? 1 : 0;
    }
    if (!plan->rank_recorded) plan->rank_recorded = gnn_capturing(stream);
    out->rank = plan->rank;
    out->indices = plan->rank_indices;
    out->cold_pays = false;
    if (plan->n_rows >= 8 * int64_t(5) * 32768) {  // the gate of gnn_plan_cold_indices
        const double cold_share = 1.0 - gnn_plan_top_share(plan, int64_t(5) * 32768);
        out->cold_pays = cold_share >= 0.05 && cold_share <= 0.30;
    }
    out->p_indptr = plan->p_indptr;
    out->p_chunks = plan->p_chunks;
    return GNN_OK;
}

double gnn_plan_top_share(const gnn_plan *plan, int64_t K) {
    if (!plan || plan->n_edges <= 0 || K <= 0) return 0.0;
    double edges = 0.0;
    int64_t left = K;
    for (int b = 255; b >= 0 && left > 0; --b) {
        const int64_t nv = plan->bucket_vertices[b];
        if (nv <= 0) continue;
        if (nv <= left) {
            edges += static_cast<double>(plan->bucket_edges[b]);
            left -= nv;
        } else {
            edges += static_cast<double>(plan->bucket_edges[b]) * static_cast<double>(left) / static_cast<double>(nv);
            left = 0;
        }
    }
    return edges / static_cast<double>(plan->n_edges);
}

extern "C" GNN_API double gnn_plan_gather_share(const gnn_plan *plan, int64_t K) { return gnn_plan_top_share(plan, K); }

void gnn_plan_drop(gnn_plan *plan, void *p, bool recorded) {
    if (p && recorded) {
        try {
            plan->retired.push_back(p);
        } catch (const std::bad_alloc &) {  // stays allocated
        }
    } else {
        gnn_dev_free(p);
    }
}

int gnn_plan_room(gnn_plan *plan, gnn_grown &b, int64_t bytes, hipStream_t stream) {
    if (bytes > b.bytes) {
        (void)hipGetLastError();
        gnn_plan_drop(plan, b.p, b.recorded);
        b = gnn_grown{};
        if (gnn_dev_alloc_bytes(&b.p, size_t(bytes)) != GNN_OK) return GNN_ERR_ALLOC;
        b.bytes = bytes;
    }
    if (!b.recorded) b.recorded = gnn_capturing(stream);
    return GNN_OK;
}

int gnn_plan_padded(gnn_plan *plan, int64_t bytes, hipStream_t stream) {
    if (!plan || bytes < 0) return GNN_ERR_INVALID_ARG;
    const bool grows = bytes > plan->padded.bytes;
    const int rc = gnn_plan_room(plan, plan->padded, bytes, stream);
    if (rc != GNN_OK || !grows) return rc;
    // padding columns are never written again; clear them once so that they hold finite values
    if (hipMemset(plan->padded.p, 0, bytes) != hipSuccess) {
        plan->padded.bytes = 0;  // not cleared
        return GNN_ERR_LAUNCH;
    }
    return GNN_OK;
}

namespace {

// What an attempt to build hot tables goes back to where there is no room: what it has built, and nothing that was there before, is freed.
struct BeforeHot {
    bool rank_indices, rank, blocks, vertices, padded, blk_partial, tile_partial;
    explicit BeforeHot(const gnn_plan *p)
        : rank_indices(p->rank_indices), rank(p->rank), blocks(p->blk_decided), vertices(p->blk_hot_vertices), padded(p->padded.p),
          blk_partial(p->blk_partial.p), tile_partial(p->tile_partial.p) {}
    void restore(gnn_plan *p) const {
        auto drop = [](auto *&q) { gnn_dev_free(q); q = nullptr; };
        auto drop_room = [](gnn_grown &g, bool had) {
            if (had) return;
            gnn_dev_free(g.p);
            g = gnn_grown{};
        };
        if (!vertices) { drop(p->blk_hot_vertices); drop(p->blk_cold_vertices); }
        if (!blocks) {
            drop(p->blk_indices); drop(p->blk_epos); drop(p->blk_idx16); drop(p->blk_piece_block); drop(p->blk_cell_off); drop(p->blk_pieces);
            drop(p->blk_rowbase); drop(p->blk_bound_w);
            for (float *&q : p->blk_edge_scale) drop(q);
            for (gnn_tiles &t : p->tiles) gnn_tiles_free(t);
            p->blk_n_edges = p->blk_n_pieces = p->blk_n_hot = 0;
            p->blk_decided = 0;
            p->blk_last_in_place = false;
        }
        if (!rank_indices) { drop(p->rank_indices); drop(p->p_indptr); drop(p->p_chunks); }
        if (!rank) drop(p->rank);
        drop_room(p->padded, padded);
        drop_room(p->blk_partial, blk_partial);
        drop_room(p->tile_partial, tile_partial);
    }
};

}  // namespace

bool gnn_plan_hot_ready(gnn_plan *plan, const void *indptr, const int32_t *indices, int mode, gnn_weight_kind weights, int64_t F, int esz, hipStream_t stream,
                        bool build, gnn_hot_layout *out) {
    const int line_elems = 128 / esz;
    const int64_t lines = (F + line_elems - 1) / line_elems;
    uint64_t &word = plan->hot_ready[esz == 2][weights == GNN_WEIGHTS_NONE ? mode : 4][lines >> 6];
    const uint64_t bit = uint64_t(1) << (lines & 63);
    if (weights == GNN_WEIGHTS_FREE || (mode && weights != GNN_WEIGHTS_NONE) || (plan->blk_decided && plan->blk_n_pieces <= 0)) return false;
    if (!(word & bit) && (!build || gnn_capturing(stream))) return false;
    const BeforeHot before(plan);
    int slices = 1;
    while (slices < 8 && slices * 2 <= lines) slices *= 2;
    const gnn_tiles *tl = nullptr;
    const float *unused = nullptr;
    int rc = gnn_plan_hot(plan, indptr, indices, stream, out);
    if (rc == GNN_OK && !out->blocks.active) {
        before.restore(plan);
        return false;
    }
    if (rc == GNN_OK) rc = gnn_plan_padded(plan, out->rows * lines * 128, stream);
    if (rc == GNN_OK) rc = gnn_plan_blocked_partial(plan, slices, line_elems, stream);
    if (rc == GNN_OK) rc = gnn_plan_tiles_with_room(plan, 8, esz == 2, !mode && weights == GNN_WEIGHTS_NONE, int(lines), line_elems, stream, &tl);
    if (rc == GNN_OK && mode) {
        rc = gnn_plan_edge_scale(plan, indices, mode, stream, &unused);
        if (rc == GNN_OK) rc = gnn_plan_blocked_edge_scale(plan, mode, stream, &unused);
        if (rc == GNN_OK && tl) rc = gnn_plan_tile_coefs(plan, tl, nullptr, plan->edge_scale[mode - 1], mode, false, stream, &unused);
    }
    if (rc == GNN_OK && weights == GNN_WEIGHTS_BOUND) {
        rc = gnn_plan_blocked_bound_weights(plan, stream, &unused);
        if (rc == GNN_OK && tl) rc = gnn_plan_tile_coefs(plan, tl, plan->bound_w, nullptr, 0, true, stream, &unused);
    }
    if (rc != GNN_OK) {
        (void)hipGetLastError();
        before.restore(plan);
        plan->hot_lacks_room |= rc == GNN_ERR_ALLOC;
        return false;
    }
    word |= bit;
    return true;
}

// What a hot call with edge weights of this kind takes (run_aggregate of aggregate.hip, on a dense matrix at a line boundary:
// ld = F), except for the per-edge factors `mode` (0: none).
static int prepare_layout(gnn_plan *plan, const int32_t *indices, int mode, int64_t F, int esz, gnn_weight_kind weights, hipStream_t stream) {
    const bool blocks = gnn_call_blocks_expected(plan, esz, F, weights);
    const gnn_layout layout = gnn_choose_layout(plan, plan->n_rows, F, esz, F, true, 0, 0, /*allow_tail=*/true, /*scaled_source=*/mode != 0,
                                                blocks, weights != GNN_WEIGHTS_NONE);
    if (!layout.padded_copy) {
        gnn_hot_layout unused_hot{};
        if (layout.hot_tables) (void)gnn_plan_hot_ready(plan, plan->indptr_seen, indices, mode, weights, F, esz, stream, /*build=*/true, &unused_hot);  // else in place
        if (!layout.slices_wanted) return GNN_OK;
        const int32_t *unused_idx = nullptr;  // the flagged index copy of the cold hints, where they pay
        return gnn_plan_cold_indices(plan, indices, false, stream, &unused_idx);
    }
    int rc = gnn_plan_padded(plan, layout.bytes, stream);
    if (rc != GNN_OK) return rc;
    gnn_rank_layout unused_rank{};  // built from the row pointers the plan was created from
    rc = gnn_plan_rank_indices(plan, plan->indptr_seen, indices, false, stream, &unused_rank);
    if (rc != GNN_OK || layout.line_lanes == 0) return rc;
    // the long rows as source-blocked pieces, their partial sums, and the part of them that is staged in LDS
    gnn_blocked_layout bl{};
    rc = gnn_plan_blocked(plan, plan->indptr_seen, stream, &bl);
    if (rc != GNN_OK || !blocks) return rc;
    if (!bl.active) return prepare_layout(plan, indices, mode, F, esz, weights, stream);  // decided now: the calls expect none
    const int line_floats = layout.line_lanes * (16 / esz);
    int slices = 1;
    while (slices < 8 && slices * 2 <= layout.main_lines) slices *= 2;
    rc = gnn_plan_blocked_partial(plan, slices, line_floats, stream);
    if (rc != GNN_OK) return rc;
    const gnn_tiles *tl = nullptr;
    rc = gnn_plan_tiles_with_room(plan, layout.line_lanes, esz == 2, weights == GNN_WEIGHTS_NONE, int(layout.main_lines), line_floats, stream, &tl);
    const float *unused = nullptr;
    if (rc == GNN_OK && weights == GNN_WEIGHTS_BOUND) rc = gnn_plan_blocked_bound_weights(plan, stream, &unused);
    if (rc != GNN_OK || !tl || weights == GNN_WEIGHTS_NONE) return rc;
    // bound weights have a copy in stream order, unless they are multiplied by a factor that the table does not hold (bf16)
    if (weights == GNN_WEIGHTS_BOUND && (mode == 0 || esz == 4)) return gnn_plan_tile_coefs(plan, tl, plan->bound_w, nullptr, 0, true, stream, &unused);
    return gnn_plan_tile_coef_room(plan, tl, stream);
}

extern "C" GNN_API int gnn_plan_lacks_room(const gnn_plan *plan) { return plan && plan->hot_lacks_room ? 1 : 0; }

extern "C" GNN_API int gnn_plan_prepare(gnn_plan *plan, const int32_t *indices, int op, int backward, int64_t F,
                                        int dtype, void *stream_v) {
    if (!plan || F < 0 || op < GNN_SUM || op > GNN_SAGE_GCN) return GNN_ERR_INVALID_ARG;
    if (dtype != GNN_F32 && dtype != GNN_BF16) return GNN_ERR_INVALID_ARG;
    hipStream_t stream = static_cast<hipStream_t>(stream_v);
    plan->hot_lacks_room = false;
    int rc = gnn_plan_reserve(plan, F);
    const int esz = dtype == GNN_BF16 ? 2 : 4;
    const int mode = (op == GNN_MEAN && backward) ? 1 : (op == GNN_GCN_SYM ? 2 : ((op == GNN_SAGE_GCN && backward) ? 3 : 0));
    // Calls may come without weights, with the bound ones or with others, and what these choose differs.  Under GCN_SYM the
    // weights take the place of the factors.
    const int weighted_mode = op == GNN_GCN_SYM ? 0 : mode;
    if (rc == GNN_OK) rc = prepare_layout(plan, indices, mode, F, esz, GNN_WEIGHTS_NONE, stream);
    if (rc == GNN_OK && plan->bound_w) rc = prepare_layout(plan, indices, weighted_mode, F, esz, GNN_WEIGHTS_BOUND, stream);
    if (rc == GNN_OK) rc = prepare_layout(plan, indices, weighted_mode, F, esz, GNN_WEIGHTS_FREE, stream);
    if (rc != GNN_OK) return rc;
    const float *unused = nullptr;
    if (mode) {
        rc = gnn_plan_edge_scale(plan, indices, mode, stream, &unused);
        // ... and in the order of the source-blocked pieces, for the calls that read it there
        if (rc == GNN_OK && plan->blk_decided && plan->blk_n_pieces > 0 && plan->n_edges > 0)
            rc = gnn_plan_blocked_edge_scale(plan, mode, stream, &unused);
        for (const gnn_tiles &t : plan->tiles)
            if (rc == GNN_OK && t.active && !t.dense_groups && plan->n_edges > 0)
                rc = gnn_plan_tile_coefs(plan, &t, nullptr, plan->edge_scale[mode - 1], mode, false, stream, &unused);
    }
    return rc;
}

extern "C" GNN_API void gnn_plan_destroy(gnn_plan *plan) {
    if (!plan) return;
    gnn_dev_free(plan->edge_scale[0]);
    gnn_dev_free(plan->edge_scale[1]);
    gnn_dev_free(plan->edge_scale[2]);
    gnn_dev_free(plan->padded.p);
    gnn_dev_free(plan->cold_indices);
    gnn_dev_free(plan->rank);
    gnn_dev_free(plan->rank_indices);
    gnn_dev_free(plan->p_indptr);
    gnn_dev_free(plan->p_chunks);
    gnn_dev_free(plan->edge_operand);
    gnn_dev_free(plan->blk_indices);
    gnn_dev_free(plan->blk_epos);
    gnn_dev_free(plan->blk_idx16);
    gnn_dev_free(plan->blk_piece_block);
    gnn_dev_free(plan->blk_pieces);
    gnn_dev_free(plan->blk_rowbase);
    gnn_dev_free(plan->blk_partial.p);
    gnn_dev_free(plan->blk_cell_off);
    gnn_dev_free(plan->blk_hot_vertices);
    gnn_dev_free(plan->blk_cold_vertices);
    for (gnn_tiles &t : plan->tiles) gnn_tiles_free(t);
    gnn_dev_free(plan->tile_partial.p);
    for (int i = 0; i < 3; ++i) gnn_dev_free(plan->blk_edge_scale[i]);
    gnn_dev_free(plan->blk_bound_w);
    if (plan->row_info) gnn_dev_free(plan->row_info);  // with row_perm behind it
    else gnn_dev_free(plan->row_perm);
    gnn_dev_free(plan->col_counts);
    gnn_dev_free(plan->chunks);
    gnn_dev_free(plan->hub_chunk_offsets);
    gnn_dev_free(plan->scratch.p);
    for (void *p : plan->retired) gnn_dev_free(p);
    delete plan;
}

namespace {

int check_params(const gnn_plan_params *params, gnn_plan_params *prm) {
    if (params) *prm = *params; else gnn_plan_default_params(prm);
    if (prm->n_thresholds < 0 || prm->n_thresholds > GNN_MAX_THRESHOLDS || prm->hub_chunk < 0) return GNN_ERR_INVALID_ARG;
    for (int i = 0; i < prm->n_thresholds; ++i) {
        if (prm->thresholds[i] <= 0) return GNN_ERR_INVALID_ARG;
        if (i > 0 && prm->thresholds[i] <= prm->thresholds[i - 1]) return GNN_ERR_INVALID_ARG;
    }
    return GNN_OK;
}

gnn_plan *new_plan(const void *indptr, int64_t N, int64_t E, int indptr_is_64, const gnn_plan_params &prm) {
    gnn_plan *plan = new (std::nothrow) gnn_plan();
    if (!plan) return nullptr;
    plan->n_rows = N;
    plan->n_edges = E;
    plan->n_bins = prm.n_thresholds + 1;
    plan->indptr_is_64 = indptr_is_64 ? 1 : 0;
    plan->params = prm;
    plan->indptr_seen = indptr;
    return plan;
}

// Fills one plan, or the two of a graph and its transpose (whose column counts are each other's row lengths) with the same
// launches.  Everything is launched before the host waits, once: the arrays whose size depends on the graph are allocated
// for the most that E edges can need.  indices: of the first; those of a transposed graph are in ascending order.
int fill_plans(gnn_plan *const *plans, int n_plans, const void *const *indptrs, const int32_t *indices, hipStream_t stream) {
    const int64_t N = plans[0]->n_rows, E = plans[0]->n_edges;
    const gnn_plan_params &prm = plans[0]->params;
    const int nb = plans[0]->n_bins;
    PlanJobs jobs{};
    jobs.N = N;
    jobs.n_blocks = (N + kSplitThreads - 1) / kSplitThreads;
    jobs.hub_chunk = prm.hub_chunk;
    jobs.ip64 = plans[0]->indptr_is_64;
    jobs.nb = nb;
    jobs.thr.k = prm.n_thresholds;
    for (int i = 0; i < jobs.thr.k; ++i) jobs.thr.t[i] = prm.thresholds[i];
    const int64_t n_counts = jobs.n_blocks * nb, count_stride = n_counts + 1;
    // rows of the last bin have at least this many edges
    const int64_t hub_degree = prm.n_thresholds > 0 ? prm.thresholds[prm.n_thresholds - 1] : 0;
    int64_t hub_bound = prm.hub_chunk > 0 ? (hub_degree > 0 && E / hub_degree < N ? E / hub_degree : N) : 0;
    const int64_t chunk_bound = hub_bound > 0 ? E / prm.hub_chunk + hub_bound : 0;

    auto hub_done_of = [](int64_t *chunks, int64_t n) { return reinterpret_cast<uint32_t *>(chunks + 3 * n); };
    // [totals of both][block counts of both][scan scratch]
    const int64_t n_scan = n_counts > hub_bound ? n_counts : hub_bound;
    const int64_t totals_words = (int64_t(sizeof(RowTotals)) + 7) / 8;
    gnn_dev_ptr<int64_t> arena;
    if (!arena.alloc_on(n_plans * (totals_words + count_stride + gnn_scan_sums_elems(n_scan)), stream)) return GNN_ERR_ALLOC;
    int64_t *totals = arena.p, *counts = totals + n_plans * totals_words, *sums = counts + n_plans * count_stride;
    struct HostBlocks {
        void *p[2] = {nullptr, nullptr};
        hipStream_t stream = nullptr;
        bool in_use = false;  // a launched kernel may still write to them
        ~HostBlocks() {
            if (in_use) (void)hipStreamSynchronize(stream);
            gnn_host_block_free(p[0]);
            gnn_host_block_free(p[1]);
        }
    } host;
    host.stream = stream;
    for (int i = 0; i < n_plans; ++i) {
        gnn_plan *p = plans[i];
        if (E <= INT32_MAX) {  // one block for both: a plan of a mini-batch is made in every step
            if (!gnn_dev_alloc(&p->row_info, N + (N + 3) / 4, stream)) return GNN_ERR_ALLOC;
            p->row_perm = reinterpret_cast<int32_t *>(p->row_info + N);
        } else if (!gnn_dev_alloc(&p->row_perm, N, stream)) {
            return GNN_ERR_ALLOC;
        }
        if (!gnn_dev_alloc(&p->col_counts, N, stream)) return GNN_ERR_ALLOC;
        if (hub_bound > 0 && (!gnn_dev_alloc(&p->hub_chunk_offsets, hub_bound + 1, stream) ||
                              !gnn_dev_alloc(&p->chunks, 7 * chunk_bound, stream))) return GNN_ERR_ALLOC;
        // without thresholds a hub row may have no edges, so no piece, and is written by the kernels that finish hub rows
        if (hub_bound > 0 && prm.n_thresholds > 0 && prm.hub_chunk <= INT32_MAX) p->hub_done = hub_done_of(p->chunks, chunk_bound);
        if (!(host.p[i] = gnn_host_block())) return GNN_ERR_ALLOC;
        PlanJob &j = jobs.job[i];
        j.indptr = indptrs[i];
        j.other_indptr = n_plans == 2 ? indptrs[1 - i] : nullptr;
        j.col_counts = p->col_counts;
        j.block_counts = counts + i * count_stride;
        j.totals = reinterpret_cast<RowTotals *>(totals + i * totals_words);
        j.host = static_cast<RowTotals *>(host.p[i]);
        j.row_perm = p->row_perm;
        j.row_info = p->row_info;
        j.hub_offsets = p->hub_chunk_offsets;
        j.chunks = p->chunks;
        j.hub_done = hub_done_of(p->chunks, chunk_bound);
    }
    GNN_HIP_TRY(hipMemsetAsync(totals, 0, size_t(n_plans * totals_words) * 8, stream));  // not in a capture: the pool has refused those
    if (n_plans == 1) {
        GNN_HIP_TRY(hipMemsetAsync(plans[0]->col_counts, 0, sizeof(int32_t) * N, stream));
        if (E > 0) count_cols_kernel<<<grid_for(E, 256, 1 << 16), 256, 0, stream>>>(indices, E, plans[0]->col_counts);
    }
    const unsigned y = static_cast<unsigned>(n_plans);
    plan_rows_kernel<<<dim3(grid_for(jobs.n_blocks, 1, 2048), y), kSplitThreads, 0, stream>>>(jobs);
    int rc = gnn_scan_exclusive_i64(counts, n_counts, n_plans, count_stride, sums, stream);
    if (rc != GNN_OK) return rc;
    host.in_use = true;
    plan_place_kernel<<<dim3(static_cast<unsigned>(jobs.n_blocks), y), kSplitThreads, 0, stream>>>(jobs);
    if (hub_bound > 0) {
        const dim3 grid(grid_for(hub_bound, 256, 1 << 16), y);
        hub_count_kernel<<<grid, 256, 0, stream>>>(jobs, hub_bound);
        for (int i = 0; i < n_plans; ++i)
            if ((rc = gnn_scan_exclusive_i64(plans[i]->hub_chunk_offsets, hub_bound, 1, 0, sums, stream)) != GNN_OK) return rc;
        hub_fill_kernel<<<grid, 256, 0, stream>>>(jobs, hub_bound, chunk_bound);
    }
    const bool look_at_order = E > 0 && gnn_long_rows(E, N);
    if (look_at_order) plan_order_kernel<<<1, kSplitThreads, 0, stream>>>(indptrs[0], jobs.ip64, indices, N, E, jobs.job[0].host);
    GNN_HIP_TRY(hipGetLastError());
    GNN_HIP_TRY(hipStreamSynchronize(stream));
    host.in_use = false;
    plans[0]->rows_unordered = look_at_order && jobs.job[0].host->unordered > kSplitThreads / 8;  // half of them where there is no order
    for (int i = 0; i < n_plans; ++i) {
        gnn_plan *p = plans[i];
        const RowTotals &r = *jobs.job[i].host;
        for (int b = 0; b < 256; ++b) {
            p->bucket_vertices[b] = static_cast<int64_t>(r.bucket_vertices[b]);
            p->bucket_edges[b] = static_cast<int64_t>(r.bucket_edges[b]);
        }
        for (int b = 0; b < nb; ++b) {
            p->bin_edges[b] = static_cast<int64_t>(r.bin_edges[b]);
            p->bin_offsets[b] = r.bin_begin[b];
        }
        p->bin_offsets[nb] = N;
        if (prm.hub_chunk > 0) {
            p->n_hub_rows = N - p->bin_offsets[nb - 1];
            p->n_chunks = static_cast<int64_t>(r.n_chunks);
            if (p->n_hub_rows > hub_bound || p->n_chunks > chunk_bound) return GNN_ERR_INVALID_GRAPH;  // row pointers that decrease
        }
    }
    return GNN_OK;
}

}  // namespace

extern "C" GNN_API int gnn_plan_create(const void *indptr, const int32_t *indices, int64_t N, int indptr_is_64,
                               const gnn_plan_params *params, void *stream_v, gnn_plan **out) {
    if (!out) return GNN_ERR_INVALID_ARG;
    *out = nullptr;
    if (N < 0 || N > INT32_MAX || (N > 0 && !indptr)) return GNN_ERR_INVALID_ARG;
    gnn_plan_params prm;
    int rc = check_params(params, &prm);
    if (rc != GNN_OK) return rc;
    hipStream_t stream = static_cast<hipStream_t>(stream_v);
    (void)hipGetLastError();  // a stale error of an earlier, failed call must not be blamed on this one
    int64_t E = 0;
    if (N > 0) {
        rc = gnn_read_edge_count(indptr, N, indptr_is_64, stream, &E);
        if (rc != GNN_OK) return rc;
        if (E < 0 || (E > 0 && !indices)) return GNN_ERR_INVALID_ARG;
    }
    gnn_plan *plan = new_plan(indptr, N, E, indptr_is_64, prm);
    if (!plan) return GNN_ERR_ALLOC;
    if (N > 0 && (rc = fill_plans(&plan, 1, &indptr, indices, stream)) != GNN_OK) {
        (void)hipStreamSynchronize(stream);
        gnn_plan_destroy(plan);
        return rc;
    }
    *out = plan;
    return GNN_OK;
}

int gnn_plan_create_pair(const void *indptr, const void *indptr_t, const int32_t *indices, int64_t E, int64_t N, int indptr_is_64,
                         const gnn_plan_params *params, hipStream_t stream, gnn_plan **fwd, gnn_plan **bwd) {
    gnn_plan_params prm;
    int rc = check_params(params, &prm);
    if (rc != GNN_OK) return rc;
    const void *indptrs[2] = {indptr, indptr_t};
    gnn_plan *plans[2] = {new_plan(indptr, N, E, indptr_is_64, prm), new_plan(indptr_t, N, E, indptr_is_64, prm)};
    if (!plans[0] || !plans[1]) rc = GNN_ERR_ALLOC;
    if (rc == GNN_OK && N > 0) rc = fill_plans(plans, 2, indptrs, indices, stream);
    if (rc != GNN_OK) {
        (void)hipStreamSynchronize(stream);
        gnn_plan_destroy(plans[0]);
        gnn_plan_destroy(plans[1]);
        return rc;
    }
    *fwd = plans[0];
    *bwd = plans[1];
    return GNN_OK;
}

extern "C" GNN_API int gnn_plan_sizes(const gnn_plan *plan, int64_t *n_rows, int32_t *n_bins, int64_t *n_chunks) {
    if (!plan) return GNN_ERR_INVALID_ARG;
    if (n_rows) *n_rows = plan->n_rows;
    if (n_bins) *n_bins = plan->n_bins;
    if (n_chunks) *n_chunks = plan->n_chunks;
    return GNN_OK;
}

extern "C" GNN_API int gnn_plan_export(const gnn_plan *plan, int64_t *bin_offsets, int32_t *row_perm, int64_t *chunks,
                               int32_t *col_counts) {
    if (!plan) return GNN_ERR_INVALID_ARG;
    if (bin_offsets) for (int b = 0; b <= plan->n_bins; ++b) bin_offsets[b] = plan->bin_offsets[b];
    if (row_perm && plan->n_rows > 0)
        GNN_HIP_TRY(hipMemcpy(row_perm, plan->row_perm, sizeof(int32_t) * plan->n_rows, hipMemcpyDeviceToHost));
    if (col_counts && plan->n_rows > 0)
        GNN_HIP_TRY(hipMemcpy(col_counts, plan->col_counts, sizeof(int32_t) * plan->n_rows, hipMemcpyDeviceToHost));
    if (chunks && plan->n_chunks > 0)
        GNN_HIP_TRY(hipMemcpy(chunks, plan->chunks, sizeof(int64_t) * 3 * plan->n_chunks, hipMemcpyDeviceToHost));
    return GNN_OK;
}

extern "C" GNN_API int64_t gnn_plan_workspace_bytes(const gnn_plan *plan, int64_t F) {
    if (!plan || F < 0) return 0;
    return plan->n_chunks * gnn_partial_ld(F) * int64_t(sizeof(float));
}

extern "C" GNN_API int gnn_plan_reserve(gnn_plan *plan, int64_t F) {
    if (!plan || F < 0) return GNN_ERR_INVALID_ARG;
    return gnn_plan_room(plan, plan->scratch, gnn_plan_workspace_bytes(plan, F), nullptr);
}

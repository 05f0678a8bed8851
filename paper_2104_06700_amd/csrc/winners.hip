// Vertex gradient of max / min pooling on large outputs: dfV[u(arg[v, j]), j] += dO[v, j] * d(binop)/dx.
//
// One global atomic addition per (v, j) touches a line of its own: 2.4 M vertices, 100 columns, 245 M additions into
// 980 MB ran at the rate at which lines move behind the L2s (48 G/s, 5.05 ms).  Here the additions are brought to where
// their sums are kept.  Columns are taken four at a time (a quad), so that the sums of 4096 vertices fit the LDS of a
// compute unit, and the pairs (vertex, value) of a quad are sorted by such ranges of vertices first:
//   1 resolve    winner positions -> source vertices, quad by quad ([quad][v][4]), beside the values; large rounds (kWideTiles) leave rows
//                without winners out
//   2 count      pairs per (quad, range, part of the rows), scanned into write positions
//   3 partition  tiles of 16384 pairs, 8192 in small rounds, are ordered by range in LDS and leave as runs of consecutive pairs, 6 bytes each
//   4 add        a workgroup adds the pairs of a range in LDS and writes its rows; a range with many pairs (the vertices
//                that win often) is cut into pieces, which add their sums to rows filled with zeros
// All of it streams, about 44 bytes per pair, 20 of them before rows without winners (43 % there) are left out, at 2.4 to 3.4 TB/s: a run of the
// partition is 27 pairs, 54 and 108 bytes, and a row of the sums 16 bytes, which leave the L2s as lines only where they meet there (counters: 1.6
// GB written for 0.94 of pairs in runs half as long, 2.3 for 0.98 of sums).  Per round of 13 quads, 122 M pairs, with all rows and tiles of 8192 pairs ->
// now: resolve 0.74 -> 0.54 ms, count 0.16 -> 0.09, partition 0.62 -> 0.43 (of 8192 0.50), add 0.55.  Ranges of 8192 vertices (one workgroup per compute unit)
// add slower, 0.61, for runs twice as long, 0.53.
#include "common.h"

namespace {

constexpr int kPairsPerThread = 16;
constexpr int kPartThreads = 512, kWideThreads = 1024;  // of a partition: a tile is 4 rows of a quad for every thread
constexpr int kTileRows = kPartThreads * kPairsPerThread / 4, kWideRows = kWideThreads * kPairsPerThread / 4;
// Large rounds have the wide one, which fills a compute unit, and leave rows without winners out, for an atomic and a wait per 64 rows (rows, columns, us with
// 2048-row tiles and all rows -> so: 150 K, 64 189 -> 214, 300 K, 100 557 -> 583, 400 K, 16 165 -> 190, 64 428 -> 412, without such rows 451 -> 475; 1 M,
// 128 1705 -> 1480, without such rows 2076 -> 2087; 2.4 M, 100 without such rows 4337 -> 4264).
constexpr int64_t kWideTiles = 2048;
constexpr int kMaxRanges = 1024;
constexpr int kMaxRangeLog2 = 13, kMinRangeLog2 = 9;
constexpr int kAddThreads = 1024;
constexpr uint32_t kPiecePairs = 1u << 17;
constexpr int kMaxQuads = 16;                  // quads per round; every round reads the indices again
// Bytes per vertex and quad of the largest arrays of a round.  A round takes as many quads as keep them within a block of the
// pool (2,449,029 vertices, 112 columns, arrays of 523 MiB from the driver: 5.6 ms, in which the host waits; of 374 MiB: 4.8).
constexpr int64_t kQuadBytes = 4 * sizeof(float);
// three such arrays and one of half the size, beside tables of a few MB, are all kept for the next call
static_assert(7 * GNN_POOL_MAX_BLOCK / 2 + (int64_t(64) << 20) <= GNN_CACHED_MEMORY_BYTES, "scratch of a call");

struct Round {
    int64_t N, n_out;
    int32_t d, col0, n_quads;                  // columns col0 .. col0 + 4 * n_quads
    int32_t range_log2, n_ranges, n_parts;
    int64_t part_rows;
    uint32_t *live;                            // [n_parts] rows of the part that have winners, the first so many below; or nullptr: all rows are there
    uint32_t *u;                               // [n_quads][N][4], a part's rows from its first on; ~0: no winner
    float *val;                                // likewise
    uint32_t *table;                           // [n_quads][n_ranges][n_parts] + 1
    uint4 *pieces;                             // (range, quad * 2 + 1 if the range is split, begin, end)
    uint32_t *n_pieces;
    uint16_t *key;                             // ordered pairs: (vertex in the range) * 4 + column of the quad
    float *key_val;
};

// PACK: rows without a winner (no edges: 43 % of the vertices of the 2.45 M-vertex graph) are left out, so that no later pass reads them.
template <bool PACK>
__global__ void __launch_bounds__(PACK ? 512 : 256) resolve_kernel(const Round r, const int32_t *__restrict__ indices, const int64_t *__restrict__ eid,
                                                                   const int32_t *__restrict__ arg, const float *__restrict__ dO, int64_t ldo,
                                                                   const float *__restrict__ fE, int64_t lde, int ewide, int binop) {
    // Lanes run along the rows, so that one load instruction looks up winners of a few rows (their edges lie side by side);
    // the results turn in LDS and leave as runs of 512 bytes and more per quad.
    constexpr int ROWS = PACK ? 64 : 32, THREADS = PACK ? 512 : 256;
    static_assert(kTileRows % ROWS == 0, "the rows of a workgroup lie in one part");
    __shared__ uint4 out_u[kMaxQuads][ROWS + 1];
    __shared__ float4 out_g[kMaxQuads][ROWS + 1];
    __shared__ uint32_t has_winner[PACK ? ROWS : 1], n_packed, first_out;
    __shared__ uint8_t rows_out[PACK ? ROWS : 1];
    if constexpr (PACK) {
        if (threadIdx.x < ROWS) has_winner[threadIdx.x] = 0;
        __syncthreads();
    }
    const int64_t v0 = int64_t(blockIdx.x) * ROWS;
    const int n_rows = r.N - v0 < ROWS ? int(r.N - v0) : ROWS;
    for (int item = threadIdx.x; item < n_rows * r.n_quads; item += THREADS) {
        const int row = item / r.n_quads, q = item - row * r.n_quads, col = r.col0 + q * 4;
        const int64_t v = v0 + row;
        uint32_t u[4];
        float g[4];
        int32_t e[4];
        const bool whole = col + 4 <= r.d;
        if (whole) {
            typedef int32_t i32x4 __attribute__((ext_vector_type(4), aligned(4)));
            typedef float f32x4 __attribute__((ext_vector_type(4), aligned(4)));
            const i32x4 a = __builtin_nontemporal_load(reinterpret_cast<const i32x4 *>(arg + v * r.d + col));
            f32x4 x = {0.0f, 0.0f, 0.0f, 0.0f};
            if (!PACK || (a[0] & a[1] & a[2] & a[3]) >= 0) x = __builtin_nontemporal_load(reinterpret_cast<const f32x4 *>(dO + v * ldo + col));
#pragma unroll
            for (int i = 0; i < 4; ++i) { e[i] = a[i]; g[i] = x[i]; }
        } else {
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                e[i] = col + i < r.d ? arg[v * r.d + col + i] : -1;
                g[i] = col + i < r.d ? dO[v * ldo + col + i] : 0.0f;
            }
        }
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            u[i] = e[i] >= 0 ? uint32_t(indices[e[i]]) : ~0u;
            if (u[i] >= r.n_out) u[i] = ~0u;
        }
        if (binop == GNN_BIN_MUL || binop == GNN_BIN_DIV) {
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                if (e[i] < 0) continue;
                const float y = fE[(eid ? eid[e[i]] : int64_t(e[i])) * lde + (ewide ? col + i : 0)];
                g[i] = binop == GNN_BIN_MUL ? g[i] * y : g[i] / y;
            }
        }
        if (PACK && (u[0] & u[1] & u[2] & u[3]) != ~0u) has_winner[row] = 1;
        out_u[q][row] = make_uint4(u[0], u[1], u[2], u[3]);
        out_g[q][row] = make_float4(g[0], g[1], g[2], g[3]);
    }
    __syncthreads();
    int n_out = n_rows;
    int64_t out0 = v0;
    if constexpr (PACK) {
        const int64_t part = v0 / r.part_rows;
        if (threadIdx.x < 64) {
            const unsigned long long m = __ballot(has_winner[threadIdx.x] != 0);
            if (m >> threadIdx.x & 1ull) rows_out[__popcll(m & ((1ull << threadIdx.x) - 1ull))] = uint8_t(threadIdx.x);
            if (threadIdx.x == 0) {
                n_packed = uint32_t(__popcll(m));
                first_out = m ? atomicAdd(&r.live[part], uint32_t(__popcll(m))) : 0u;
            }
        }
        __syncthreads();
        n_out = int(n_packed);
        out0 = part * r.part_rows + first_out;
    }
    for (int item = threadIdx.x; item < ROWS * r.n_quads; item += THREADS) {
        const int q = item / ROWS, k = item % ROWS;
        if (k >= n_out) continue;
        const int row = PACK ? rows_out[k] : k;
        const int64_t at = int64_t(q) * r.N + out0 + k;
        reinterpret_cast<uint4 *>(r.u)[at] = out_u[q][row];
        reinterpret_cast<float4 *>(r.val)[at] = out_g[q][row];
    }
}

// one past the last of a part's rows that are there
__device__ __forceinline__ int64_t part_end(const Round &r, int p) {
    const int64_t begin = p * r.part_rows, rows = r.live ? int64_t(r.live[p]) : r.part_rows;
    return begin + rows < r.N ? begin + rows : r.N;
}

__global__ void __launch_bounds__(kPartThreads) clear_live_kernel(const Round r) {  // one workgroup
    for (int p = threadIdx.x; p < r.n_parts; p += kPartThreads) r.live[p] = 0;
}

__global__ void __launch_bounds__(kPartThreads) count_kernel(const Round r) {
    __shared__ uint32_t hist[kMaxRanges];
    const int q = int(blockIdx.x) / r.n_parts, p = int(blockIdx.x) % r.n_parts;
    for (int b = threadIdx.x; b < r.n_ranges; b += kPartThreads) hist[b] = 0;
    __syncthreads();
    const int64_t begin = p * r.part_rows, end = part_end(r, p);
    const uint4 *u = reinterpret_cast<const uint4 *>(r.u) + int64_t(q) * r.N;
    for (int64_t v = begin + threadIdx.x; v < end; v += kPartThreads) {
        const uint4 x = u[v];
        if (x.x != ~0u) atomicAdd(&hist[x.x >> r.range_log2], 1u);
        if (x.y != ~0u) atomicAdd(&hist[x.y >> r.range_log2], 1u);
        if (x.z != ~0u) atomicAdd(&hist[x.z >> r.range_log2], 1u);
        if (x.w != ~0u) atomicAdd(&hist[x.w >> r.range_log2], 1u);
    }
    __syncthreads();
    for (int b = threadIdx.x; b < r.n_ranges; b += kPartThreads) r.table[(int64_t(q) * r.n_ranges + b) * r.n_parts + p] = hist[b];
    if (blockIdx.x == 0 && threadIdx.x == 0) r.table[int64_t(r.n_quads) * r.n_ranges * r.n_parts] = 0;
}

template <int THREADS>
__global__ void __launch_bounds__(THREADS) partition_kernel(const Round r) {
    constexpr int kTile = THREADS * kPairsPerThread;
    __shared__ uint32_t hist[kMaxRanges], start[kMaxRanges], next[kMaxRanges];  // next: where the range's next pair goes
    __shared__ uint32_t wave_sum[THREADS / 64];
    __shared__ uint32_t pair_key[kTile];
    __shared__ float pair_val[kTile];
    const int q = int(blockIdx.x) / r.n_parts, p = int(blockIdx.x) % r.n_parts;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int64_t begin = p * r.part_rows, end = part_end(r, p);
    for (int b = threadIdx.x; b < r.n_ranges; b += THREADS) next[b] = r.table[(int64_t(q) * r.n_ranges + b) * r.n_parts + p];
    const uint4 *us = reinterpret_cast<const uint4 *>(r.u) + int64_t(q) * r.N;
    const float4 *vals = reinterpret_cast<const float4 *>(r.val) + int64_t(q) * r.N;
    const uint32_t low = (4u << r.range_log2) - 1;
    for (int64_t tile = begin; tile < end; tile += kTile / 4) {
        uint4 u[kPairsPerThread / 4];
        float4 g[kPairsPerThread / 4];
#pragma unroll
        for (int k = 0; k < kPairsPerThread / 4; ++k) {
            const int64_t v = tile + k * THREADS + threadIdx.x;
            u[k] = make_uint4(~0u, ~0u, ~0u, ~0u);
            if (v < end) { u[k] = us[v]; g[k] = vals[v]; }
        }
        for (int b = threadIdx.x; b < r.n_ranges; b += THREADS) hist[b] = 0;
        __syncthreads();
        uint32_t rank[kPairsPerThread];
#pragma unroll
        for (int k = 0; k < kPairsPerThread / 4; ++k) {
            const uint32_t w[4] = {u[k].x, u[k].y, u[k].z, u[k].w};
#pragma unroll
            for (int i = 0; i < 4; ++i) rank[k * 4 + i] = w[i] != ~0u ? atomicAdd(&hist[w[i] >> r.range_log2], 1u) : 0u;
        }
        __syncthreads();
        // exclusive sums of the counts: two ranges per thread, then over lanes, then over wavefronts
        const int b0 = 2 * threadIdx.x;
        const uint32_t h0 = b0 < r.n_ranges ? hist[b0] : 0, h1 = b0 + 1 < r.n_ranges ? hist[b0 + 1] : 0;
        uint32_t incl = h0 + h1;
        for (int off = 1; off < 64; off <<= 1) {
            const uint32_t o = __shfl_up(incl, off);
            if (lane >= off) incl += o;
        }
        if (lane == 63) wave_sum[wave] = incl;
        __syncthreads();
        uint32_t before = incl - (h0 + h1), total = 0;
#pragma unroll
        for (int w = 0; w < THREADS / 64; ++w) {
            if (w < wave) before += wave_sum[w];
            total += wave_sum[w];
        }
        if (b0 < r.n_ranges) { start[b0] = before; hist[b0] = next[b0] - before; next[b0] += h0; }
        if (b0 + 1 < r.n_ranges) { start[b0 + 1] = before + h0; hist[b0 + 1] = next[b0 + 1] - (before + h0); next[b0 + 1] += h1; }
        __syncthreads();
#pragma unroll
        for (int k = 0; k < kPairsPerThread / 4; ++k) {
            const uint32_t w[4] = {u[k].x, u[k].y, u[k].z, u[k].w};
            const float x[4] = {g[k].x, g[k].y, g[k].z, g[k].w};
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                if (w[i] == ~0u) continue;
                const uint32_t at = start[w[i] >> r.range_log2] + rank[k * 4 + i];
                pair_key[at] = w[i] * 4 + i;
                pair_val[at] = x[i];
            }
        }
        __syncthreads();
        for (uint32_t i = threadIdx.x; i < total; i += THREADS) {
            const uint32_t key = pair_key[i];
            const uint32_t to = hist[key >> (r.range_log2 + 2)] + i;  // hist: write position minus position in the tile
            r.key[to] = uint16_t(key & low);
            r.key_val[to] = pair_val[i];
        }
        __syncthreads();
    }
}

// Task t: eight ranges side by side, their quads one after the other.  Workgroup t runs on XCD t % 8, so the quads of a range,
// which write parts of the same lines, are written from the same L2 at about the same time.
__device__ __forceinline__ void task_of(const Round &r, int t, int *range, int *quad) {
    const int per = 8 * r.n_quads;
    *range = t / per * 8 + (t & 7);
    *quad = t % per >> 3;
}
__device__ __forceinline__ void pairs_of(const Round &r, int range, int quad, uint32_t *begin, uint32_t *end) {
    const int64_t i = (int64_t(quad) * r.n_ranges + range) * r.n_parts;
    *begin = r.table[i];
    *end = r.table[i + r.n_parts];
}
__device__ __forceinline__ uint32_t piece_count(uint32_t pairs) { return pairs > kPiecePairs ? (pairs + kPiecePairs - 1) / kPiecePairs : 1; }

__global__ void __launch_bounds__(1024) pieces_kernel(const Round r, int n_tasks) {  // one workgroup
    __shared__ uint32_t wave_sum[16];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    uint32_t done = 0;
    for (int t0 = 0; t0 < n_tasks; t0 += 1024) {
        const int t = t0 + int(threadIdx.x);
        uint32_t n = 0, begin = 0, end = 0;
        int range = 0, quad = 0;
        if (t < n_tasks) task_of(r, t, &range, &quad);
        if (t < n_tasks && range < r.n_ranges) {
            pairs_of(r, range, quad, &begin, &end);
            n = piece_count(end - begin);
        }
        uint32_t incl = n;
        for (int off = 1; off < 64; off <<= 1) {
            const uint32_t o = __shfl_up(incl, off);
            if (lane >= off) incl += o;
        }
        if (lane == 63) wave_sum[wave] = incl;
        __syncthreads();
        uint32_t before = done + incl - n;
        for (int w = 0; w < 16; ++w) {
            if (w < wave) before += wave_sum[w];
            done += wave_sum[w];
        }
        for (uint32_t i = 0; i < n; ++i) {
            const uint32_t at = begin + i * kPiecePairs, left = end - at;
            r.pieces[before + i] = make_uint4(uint32_t(range), uint32_t(quad) * 2 + (n > 1), at, at + (left < kPiecePairs ? left : kPiecePairs));
        }
        __syncthreads();
    }
    if (threadIdx.x == 0) *r.n_pieces = done;
}

__global__ void __launch_bounds__(256) clear_split_kernel(const Round r, float *__restrict__ out, int64_t ldv) {
    int range, quad;
    task_of(r, blockIdx.x, &range, &quad);
    if (range >= r.n_ranges) return;
    uint32_t begin, end;
    pairs_of(r, range, quad, &begin, &end);
    if (piece_count(end - begin) <= 1) return;
    const int64_t v0 = int64_t(range) << r.range_log2;
    const int col = r.col0 + quad * 4;
    for (int t = threadIdx.x; t < (4 << r.range_log2); t += 256) {
        const int64_t v = v0 + t / 4;
        if (v < r.n_out && col + t % 4 < r.d) out[v * ldv + col + t % 4] = 0.0f;
    }
}

template <int RANGE_LOG2>
__global__ void __launch_bounds__(kAddThreads) add_kernel(const Round r, float *__restrict__ out, int64_t ldv) {
    constexpr int n_rows = 1 << RANGE_LOG2;
    __shared__ __attribute__((aligned(16))) float sums[n_rows * 4];
    if (blockIdx.x >= *r.n_pieces) return;
    const uint4 piece = r.pieces[blockIdx.x];
    const int range = int(piece.x), quad = int(piece.y >> 1);
    const bool split = piece.y & 1;
    const uint32_t end = piece.w;
    // the next 8 K pairs are on their way while the ones before are added
    constexpr int U = 8;
    uint16_t k[U];
    float x[U];
    auto fetch = [&](uint32_t first) {
#pragma unroll
        for (int j = 0; j < U; ++j) {
            const uint32_t i = first + j * kAddThreads + threadIdx.x;
            if (i < end) { k[j] = __builtin_nontemporal_load(r.key + i); x[j] = __builtin_nontemporal_load(r.key_val + i); }
        }
    };
    fetch(piece.z);
    for (int t = threadIdx.x; t < n_rows; t += kAddThreads) reinterpret_cast<float4 *>(sums)[t] = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
    __syncthreads();
    for (uint32_t first = piece.z; first < end; first += U * kAddThreads) {
        uint16_t k0[U];
        float x0[U];
#pragma unroll
        for (int j = 0; j < U; ++j) { k0[j] = k[j]; x0[j] = x[j]; }
        fetch(first + U * kAddThreads);
#pragma unroll
        for (int j = 0; j < U; ++j)
            if (first + j * kAddThreads + threadIdx.x < end) unsafeAtomicAdd(&sums[k0[j]], x0[j]);
    }
    __syncthreads();
    const int64_t v0 = int64_t(range) << RANGE_LOG2;
    const int col = r.col0 + quad * 4;
    const int left = r.d - col;
    for (int t = threadIdx.x; t < n_rows; t += kAddThreads) {
        if (v0 + t >= r.n_out) break;
        float *p = out + (v0 + t) * ldv + col;
        const float4 s = reinterpret_cast<float4 *>(sums)[t];
        const float x[4] = {s.x, s.y, s.z, s.w};
        if (split) {
            for (int j = 0; j < 4 && j < left; ++j)
                if (x[j] != 0.0f) unsafeAtomicAdd(p + j, x[j]);
        } else if (left >= 4) {
            typedef float f32x4 __attribute__((ext_vector_type(4), aligned(4)));
            *reinterpret_cast<f32x4 *>(p) = f32x4{x[0], x[1], x[2], x[3]};
        } else {
            for (int j = 0; j < left; ++j) p[j] = x[j];
        }
    }
}

}  // namespace

// Sorting pays where the atomics of a row go to many lines: with few edges per row its winners share them (2.4 M vertices, 5
// edges each, 128 columns: 2.2 ms against 4.2), and small outputs stay in the caches (150 K vertices, 13 edges each, 32
// columns: 0.100 ms against 0.121).  Otherwise, atomics -> sorted: 150 K, 13 edges, 64 columns 0.19 -> 0.16 ms; 400 K, 50
// edges, 16 columns 0.27 -> 0.17, 64 columns 0.65 -> 0.41; 1 M, 20 edges, 128 columns 2.67 -> 1.96; 2.4 M, 50 edges, 100
// columns 4.95 -> 4.15.  Never where the arrays of one quad would not fit a block of the pool.
bool gnn_winners_apply(int64_t n_edges, int64_t n_out, int64_t N, int64_t d) {
    if (n_out <= 0 || n_out > int64_t(kMaxRanges) << kMaxRangeLog2 || N > GNN_POOL_MAX_BLOCK / kQuadBytes) return false;
    return (N * d >= (int64_t(1) << 23) && n_edges >= 12 * N) || (N * d >= (int64_t(1) << 22) && n_edges >= 16 * N);
}

int gnn_scatter_winners(const int32_t *indices, const int64_t *eid, const int32_t *arg, const float *dO, int64_t ldo, const float *fE,
                        int64_t lde, bool ewide, float *out, int64_t ldv, int64_t n_out, int64_t N, int64_t d, int binop,
                        hipStream_t stream) {
    const int64_t all_quads = (d + 3) / 4;
    Round r{};
    r.N = N;
    r.n_out = n_out;
    r.d = int32_t(d);
    // at least 64 ranges where there are vertices enough, so that the pieces of a round fill the chip
    r.range_log2 = n_out > int64_t(kMaxRanges) << 12 ? 13 : 12;
    while (r.range_log2 > kMinRangeLog2 && (n_out >> r.range_log2) < 64) --r.range_log2;
    r.n_ranges = int32_t((n_out + (int64_t(1) << r.range_log2) - 1) >> r.range_log2);
    int64_t quads = GNN_POOL_MAX_BLOCK / (N * kQuadBytes);
    if (quads > kMaxQuads) quads = kMaxQuads;
    const int64_t n_rounds = (all_quads + quads - 1) / quads;
    quads = (all_quads + n_rounds - 1) / n_rounds;
    const bool wide = (N + kWideRows - 1) / kWideRows * quads >= kWideTiles;
    const int64_t tile_rows = wide ? kWideRows : kTileRows, tiles = (N + tile_rows - 1) / tile_rows;
    int64_t parts = (wide ? 256 : 512) / quads;
    if (parts > tiles) parts = tiles;
    r.part_rows = (tiles + parts - 1) / parts * tile_rows;
    r.n_parts = int32_t((N + r.part_rows - 1) / r.part_rows);
    const int64_t pairs = N * quads * 4, entries = quads * r.n_ranges * r.n_parts + 1;
    // every range has a piece, and no more than this are added for the pairs beyond its first
    const int64_t max_pieces = quads * r.n_ranges + pairs / kPiecePairs;
    gnn_dev_ptr<uint32_t> u, table, sums, count, live;
    gnn_dev_ptr<uint4> pieces;
    gnn_dev_ptr<float> val, key_val;
    gnn_dev_ptr<uint16_t> key;
    if (!u.alloc_on(pairs, stream) || !val.alloc_on(pairs, stream) || !key.alloc_on(pairs, stream) || !key_val.alloc_on(pairs, stream) ||
        !table.alloc_on(entries, stream) || !sums.alloc_on(gnn_scan_sums_elems(entries), stream) || !pieces.alloc_on(max_pieces, stream) ||
        !count.alloc_on(1, stream) || (wide && !live.alloc_on(r.n_parts, stream)))
        return GNN_ERR_ALLOC;
    r.u = u.p; r.val = val.p; r.key = key.p; r.key_val = key_val.p; r.table = table.p; r.pieces = pieces.p; r.n_pieces = count.p; r.live = live.p;
    for (int64_t q0 = 0; q0 < all_quads; q0 += quads) {
        r.col0 = int32_t(q0 * 4);
        r.n_quads = int32_t(all_quads - q0 < quads ? all_quads - q0 : quads);
        if (wide) {
            clear_live_kernel<<<1, kPartThreads, 0, stream>>>(r);
            resolve_kernel<true><<<unsigned((N + 63) / 64), 512, 0, stream>>>(r, indices, eid, arg, dO, ldo, fE, lde, ewide ? 1 : 0, binop);
        } else {
            resolve_kernel<false><<<unsigned((N + 31) / 32), 256, 0, stream>>>(r, indices, eid, arg, dO, ldo, fE, lde, ewide ? 1 : 0, binop);
        }
        count_kernel<<<unsigned(r.n_quads * r.n_parts), kPartThreads, 0, stream>>>(r);
        if (hipGetLastError() != hipSuccess) return GNN_ERR_LAUNCH;
        const int rc = gnn_scan_exclusive_u32(r.table, int64_t(r.n_quads) * r.n_ranges * r.n_parts + 1, sums.p, stream);
        if (rc != GNN_OK) return rc;
        const int n_tasks = (r.n_ranges + 7) / 8 * 8 * r.n_quads;
        pieces_kernel<<<1, 1024, 0, stream>>>(r, n_tasks);
        if (wide) partition_kernel<kWideThreads><<<unsigned(r.n_quads * r.n_parts), kWideThreads, 0, stream>>>(r);
        else partition_kernel<kPartThreads><<<unsigned(r.n_quads * r.n_parts), kPartThreads, 0, stream>>>(r);
        clear_split_kernel<<<unsigned(n_tasks), 256, 0, stream>>>(r, out, ldv);
        switch (r.range_log2) {
            case 13: add_kernel<13><<<unsigned(max_pieces), kAddThreads, 0, stream>>>(r, out, ldv); break;
            case 12: add_kernel<12><<<unsigned(max_pieces), kAddThreads, 0, stream>>>(r, out, ldv); break;
            case 11: add_kernel<11><<<unsigned(max_pieces), kAddThreads, 0, stream>>>(r, out, ldv); break;
            case 10: add_kernel<10><<<unsigned(max_pieces), kAddThreads, 0, stream>>>(r, out, ldv); break;
            default: add_kernel<9><<<unsigned(max_pieces), kAddThreads, 0, stream>>>(r, out, ldv); break;
        }
        if (hipGetLastError() != hipSuccess) return GNN_ERR_LAUNCH;
    }
    return GNN_OK;
}

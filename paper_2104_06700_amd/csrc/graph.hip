// Once-per-graph structure kernels: CSR row pointers from a sorted destination
// array, the transposed graph (CSR by source) the backward pass runs over, and a
// precondition checker.  Integer work only; every result is deterministic.
//
// The paper takes the CSR as given (Section 4.1) and builds extra CSRs as
// preprocessing (Section 4.2); the transposed graph is what the implied
// backward pass needs.
#include "common.h"

namespace {

template <typename IP>
__global__ void __launch_bounds__(256) indptr_from_sorted_kernel(const int32_t *__restrict__ keys, int64_t E,
                                                                 int64_t N, IP *__restrict__ indptr) {
    // Thread e (0..E) owns the boundary between keys[e-1] and keys[e]; it writes
    // indptr[v] = e for every v in (keys[e-1], keys[e]].  Each indptr entry has one writer.
    int64_t stride = int64_t(gridDim.x) * blockDim.x;
    for (int64_t e = int64_t(blockIdx.x) * blockDim.x + threadIdx.x; e <= E; e += stride) {
        int64_t prev = e == 0 ? -1 : keys[e - 1];
        int64_t cur = e == E ? N : keys[e];
        for (int64_t v = prev + 1; v <= cur; ++v) indptr[v] = static_cast<IP>(e);
    }
}

// row_of[e] = v for e in [indptr[v], indptr[v+1]) -- one wavefront per row.
template <typename IP>
__global__ void __launch_bounds__(256) expand_rows_kernel(const IP *__restrict__ indptr, int64_t N,
                                                          int32_t *__restrict__ row_of) {
    const int lane = threadIdx.x & 63;
    int64_t wave = (int64_t(blockIdx.x) * blockDim.x + threadIdx.x) >> 6;
    int64_t n_waves = (int64_t(gridDim.x) * blockDim.x) >> 6;
    for (int64_t v = wave; v < N; v += n_waves) {
        int64_t b = indptr[v], e = indptr[v + 1];
        for (int64_t i = b + lane; i < e; i += 64) row_of[i] = static_cast<int32_t>(v);
    }
}

__global__ void __launch_bounds__(256) gather_transposed_kernel(const uint32_t *__restrict__ pos_sorted, int64_t E,
                                                                const int32_t *__restrict__ row_of,
                                                                const float *__restrict__ w,
                                                                int32_t *__restrict__ indices_t,
                                                                int64_t *__restrict__ perm, float *__restrict__ wt) {
    int64_t stride = int64_t(gridDim.x) * blockDim.x;
    for (int64_t i = int64_t(blockIdx.x) * blockDim.x + threadIdx.x; i < E; i += stride) {
        uint32_t p = pos_sorted[i];
        indices_t[i] = row_of[p];
        if (perm) perm[i] = static_cast<int64_t>(p);
        if (wt) wt[i] = w[p];
    }
}

template <typename IP>
__global__ void __launch_bounds__(256) validate_kernel(const IP *__restrict__ indptr, const int32_t *__restrict__ indices,
                                                       int64_t N, int64_t E, int *__restrict__ bad) {
    int64_t stride = int64_t(gridDim.x) * blockDim.x;
    int64_t t0 = int64_t(blockIdx.x) * blockDim.x + threadIdx.x;
    int err = 0;
    for (int64_t v = t0; v < N; v += stride)
        if (indptr[v] > indptr[v + 1]) err = 1;
    if (t0 == 0 && (indptr[0] != 0 || static_cast<int64_t>(indptr[N]) != E)) err = 1;
    for (int64_t e = t0; e < E; e += stride)
        if (indices[e] < 0 || indices[e] >= N) err = 1;
    if (err) atomicOr(bad, 1);
}

// ---------------------------------------------------------------- prefix sums
// Exclusive prefix sums in place: workgroup b sums its 4096 elements, then every workgroup adds up the sums before its own
// and scans its elements.  Up to 4096 elements that is one launch.  blockIdx.y: arrays `stride` elements apart.
// data[n] receives the total when want_total is set.
constexpr int kScanItems = 16;
constexpr int kScanChunk = 256 * kScanItems;

template <typename T>
__device__ __forceinline__ T wave_scan_inclusive(T x) {
    const int lane = threadIdx.x & 63;
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) {
        const T y = __shfl_up(x, off);
        if (lane >= off) x += y;
    }
    return x;
}

// Sum over the 256 threads of a workgroup, in every thread.
template <typename T>
__device__ __forceinline__ T block_sum(T x, T *lds4) {
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) x += __shfl_xor(x, off);
    __syncthreads();
    if ((threadIdx.x & 63) == 0) lds4[threadIdx.x >> 6] = x;
    __syncthreads();
    return lds4[0] + lds4[1] + lds4[2] + lds4[3];
}

template <typename T>
__global__ void __launch_bounds__(256) scan_block_sums_kernel(const T *__restrict__ data, int64_t n, int64_t stride, int64_t n_sums,
                                                              T *__restrict__ sums) {
    __shared__ T red[4];
    data += blockIdx.y * stride;
    const int64_t lo = int64_t(blockIdx.x) * kScanChunk;
    T s = 0;
#pragma unroll
    for (int k = 0; k < kScanItems; ++k) {
        const int64_t i = lo + k * 256 + threadIdx.x;
        if (i < n) s += data[i];
    }
    s = block_sum(s, red);
    if (threadIdx.x == 0) sums[blockIdx.y * n_sums + blockIdx.x] = s;
}

template <typename T>
__global__ void __launch_bounds__(256) scan_local_kernel(T *__restrict__ data, int64_t n, int64_t stride, int64_t n_sums,
                                                         const T *__restrict__ sums, bool want_total) {
    __shared__ T red[4], wave_total[4];
    data += blockIdx.y * stride;
    T before = 0;
    if (n_sums > 1) {
        sums += blockIdx.y * n_sums;
        for (int64_t i = threadIdx.x; i < int64_t(blockIdx.x); i += 256) before += sums[i];
        before = block_sum(before, red);
    }
    const int64_t lo = int64_t(blockIdx.x) * kScanChunk + int64_t(threadIdx.x) * kScanItems;
    T v[kScanItems], s = 0;
#pragma unroll
    for (int k = 0; k < kScanItems; ++k) {
        v[k] = lo + k < n ? data[lo + k] : T(0);
        s += v[k];
    }
    const T upto = wave_scan_inclusive(s);
    const int wave = threadIdx.x >> 6;
    if ((threadIdx.x & 63) == 63) wave_total[wave] = upto;
    __syncthreads();
    for (int w = 0; w < wave; ++w) before += wave_total[w];
    T run = before + upto - s;
#pragma unroll
    for (int k = 0; k < kScanItems; ++k) {
        if (lo + k < n) data[lo + k] = run;
        run += v[k];
        if (want_total && lo + k == n - 1) data[n] = run;
    }
}

template <typename T>
int scan_exclusive(T *data, int64_t n, int n_arrays, int64_t stride, bool want_total, T *sums, hipStream_t stream) {
    if (n <= 0) return GNN_OK;
    const int64_t n_sums = (n + kScanChunk - 1) / kScanChunk;
    if (n_sums > INT32_MAX) return GNN_ERR_UNSUPPORTED;
    const dim3 grid(static_cast<unsigned>(n_sums), static_cast<unsigned>(n_arrays));
    if (n_sums > 1) scan_block_sums_kernel<T><<<grid, 256, 0, stream>>>(data, n, stride, n_sums, sums);
    scan_local_kernel<T><<<grid, 256, 0, stream>>>(data, n, stride, n_sums, sums, want_total);
    return hipGetLastError() == hipSuccess ? GNN_OK : GNN_ERR_LAUNCH;
}

// ---------------------------------------------------------------- stable radix sort
// LSD radix sort of (key, value) pairs of 32-bit words, 8 bits per pass, stable.  A workgroup of 8 wavefronts owns a tile
// of 4096 consecutive pairs, a wavefront 512 of them.  Per pass: (1) every tile counts its digits, (2) the [digit][tile]
// table is prefix-summed (digit-major, so equal digits of earlier tiles come first), (3) every tile orders its pairs by
// digit in LDS and writes each digit's run in one piece.  Lanes with the same digit are found with eight ballots, so the
// counters of a wavefront have one writer per digit and round.
// Bound by the latency of the 8 dependent rounds of a wavefront, not by the 16 bytes per pair and pass: one wavefront per
// tile took 64 rounds and wrote single pairs (3.1 M pairs, 16 bits: 2 x (36 + 15 + 58) us).
constexpr int kSortWaves = 8;
constexpr int kSortRounds = 8;
constexpr int kSortThreads = 64 * kSortWaves;
constexpr int kSortTile = kSortThreads * kSortRounds;

__device__ __forceinline__ unsigned long long same_digit_lanes(unsigned digit, bool valid) {
    unsigned long long peers = __ballot(valid);
#pragma unroll
    for (int bit = 0; bit < 8; ++bit) {
        const bool one = (digit >> bit) & 1u;
        const unsigned long long b = __ballot(one);
        peers &= one ? b : ~b;
    }
    return peers;
}

// from_top: the first pass of a descending order reads key k as from_top - k
__global__ void __launch_bounds__(kSortThreads) sort_count_kernel(const uint32_t *__restrict__ keys, int64_t n, int shift,
                                                                  uint32_t from_top, int64_t n_tiles, uint32_t *__restrict__ table) {
    __shared__ uint32_t hist[kSortWaves][256];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    for (int d = threadIdx.x; d < kSortWaves * 256; d += kSortThreads) (&hist[0][0])[d] = 0;
    const int64_t i0 = int64_t(blockIdx.x) * kSortTile + wave * (64 * kSortRounds) + lane;
    uint32_t key[kSortRounds];
#pragma unroll
    for (int r = 0; r < kSortRounds; ++r) {
        key[r] = i0 + r * 64 < n ? keys[i0 + r * 64] : 0u;
        if (from_top) key[r] = from_top - key[r];
    }
    __syncthreads();
#pragma unroll
    for (int r = 0; r < kSortRounds; ++r) {
        const bool valid = i0 + r * 64 < n;
        const unsigned digit = (key[r] >> shift) & 255u;
        const unsigned long long peers = same_digit_lanes(digit, valid);
        if (valid && (peers & ((1ull << lane) - 1ull)) == 0) hist[wave][digit] += __popcll(peers);  // one leader per digit
        __builtin_amdgcn_wave_barrier();
    }
    __syncthreads();
    if (threadIdx.x < 256) {
        uint32_t s = 0;
#pragma unroll
        for (int w = 0; w < kSortWaves; ++w) s += hist[w][threadIdx.x];
        table[int64_t(threadIdx.x) * n_tiles + blockIdx.x] = s;
    }
}

// vals_in null: the value of pair i is i.  inverse: vals_out[value] = place of the pair, and no keys are written
template <bool INVERSE>
__global__ void __launch_bounds__(kSortThreads) sort_scatter_kernel(const uint32_t *__restrict__ keys_in,
                                                                    const uint32_t *__restrict__ vals_in, int64_t n, int shift,
                                                                    uint32_t from_top, int64_t n_tiles,
                                                                    const uint32_t *__restrict__ table,
                                                                    uint32_t *__restrict__ keys_out, uint32_t *__restrict__ vals_out) {
    __shared__ uint32_t hist[kSortWaves][256];  // pairs per wavefront and digit, then those of the wavefronts before
    __shared__ uint32_t digit_begin[256];       // first place of a digit in the tile
    __shared__ uint32_t digit_out[256];         // its first place in the output, minus that
    __shared__ uint32_t wave_total[4];
    __shared__ uint32_t sorted_key[kSortTile], sorted_val[kSortTile];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    for (int d = threadIdx.x; d < kSortWaves * 256; d += kSortThreads) (&hist[0][0])[d] = 0;
    const int64_t tile0 = int64_t(blockIdx.x) * kSortTile;
    const int64_t i0 = tile0 + wave * (64 * kSortRounds) + lane;
    uint32_t key[kSortRounds], val[kSortRounds], place[kSortRounds];
#pragma unroll
    for (int r = 0; r < kSortRounds; ++r) {
        const int64_t i = i0 + r * 64;
        key[r] = i < n ? keys_in[i] : 0u;
        if (from_top) key[r] = from_top - key[r];
        val[r] = vals_in ? (i < n ? vals_in[i] : 0u) : uint32_t(i);
    }
    __syncthreads();
#pragma unroll
    for (int r = 0; r < kSortRounds; ++r) {
        const bool valid = i0 + r * 64 < n;
        const unsigned digit = (key[r] >> shift) & 255u;
        const unsigned long long peers = same_digit_lanes(digit, valid);
        const unsigned long long before = peers & ((1ull << lane) - 1ull);
        const uint32_t seen = hist[wave][digit];
        place[r] = seen + __popcll(before);
        __builtin_amdgcn_wave_barrier();
        if (valid && before == 0) hist[wave][digit] = seen + __popcll(peers);
        __builtin_amdgcn_wave_barrier();
    }
    __syncthreads();
    if (threadIdx.x < 256) {
        const int d = threadIdx.x;
        uint32_t total = 0;
#pragma unroll
        for (int w = 0; w < kSortWaves; ++w) {
            const uint32_t c = hist[w][d];
            hist[w][d] = total;
            total += c;
        }
        const uint32_t upto = wave_scan_inclusive(total);
        if (lane == 63) wave_total[wave] = upto;
        digit_begin[d] = upto - total;
    }
    __syncthreads();
    if (threadIdx.x < 256) {
        const int d = threadIdx.x;
        uint32_t begin = digit_begin[d];
        for (int w = 0; w < wave; ++w) begin += wave_total[w];
        digit_begin[d] = begin;
        digit_out[d] = table[int64_t(d) * n_tiles + blockIdx.x] - begin;
    }
    __syncthreads();
#pragma unroll
    for (int r = 0; r < kSortRounds; ++r) {
        if (i0 + r * 64 >= n) continue;
        const unsigned digit = (key[r] >> shift) & 255u;
        const uint32_t at = digit_begin[digit] + hist[wave][digit] + place[r];
        sorted_key[at] = key[r];
        sorted_val[at] = val[r];
    }
    __syncthreads();
    const int count = n - tile0 < kSortTile ? int(n - tile0) : kSortTile;
    for (int j = threadIdx.x; j < count; j += kSortThreads) {
        const uint32_t k = sorted_key[j], v = sorted_val[j];
        const uint32_t out = digit_out[(k >> shift) & 255u] + uint32_t(j);
        if (INVERSE) {
            vals_out[v] = out;
        } else {
            keys_out[out] = k;
            vals_out[out] = v;
        }
    }
}

// Sorts n pairs by the low `bits` bits of the key.
struct SortJob {
    const uint32_t *first_keys = nullptr;  // input of the first pass (read only)
    const uint32_t *first_vals = nullptr;  // null: 0, 1, 2, ...
    uint32_t from_top = 0;                 // the first pass reads key k as from_top - k
    uint32_t *buf_k[2] = {nullptr, nullptr}, *buf_v[2] = {nullptr, nullptr};  // written alternately, [1] first; [0] may hold the input
    uint32_t *last_keys = nullptr, *last_vals = nullptr;  // where the last pass writes (null: the buffer whose turn it is)
    bool inverse_last = false;             // the last pass writes last_vals[value] = place, and no keys
};

int radix_sort(const SortJob &job, int64_t n, int bits, uint32_t *table, uint32_t *sums, hipStream_t stream, uint32_t **keys_out,
               uint32_t **vals_out) {
    const int64_t n_tiles = (n + kSortTile - 1) / kSortTile;
    if (n_tiles > INT32_MAX) return GNN_ERR_UNSUPPORTED;
    const unsigned grid = static_cast<unsigned>(n_tiles);
    const uint32_t *kin = job.first_keys, *vin = job.first_vals;
    uint32_t from_top = job.from_top;
    int cur = 0;
    for (int shift = 0; shift < bits; shift += 8) {
        const bool last = shift + 8 >= bits;
        uint32_t *kout = last && job.last_keys ? job.last_keys : job.buf_k[cur ^ 1];
        uint32_t *vout = last && job.last_vals ? job.last_vals : job.buf_v[cur ^ 1];
        sort_count_kernel<<<grid, kSortThreads, 0, stream>>>(kin, n, shift, from_top, n_tiles, table);
        const int rc = scan_exclusive<uint32_t>(table, n_tiles * 256, 1, 0, false, sums, stream);
        if (rc != GNN_OK) return rc;
        if (last && job.inverse_last)
            sort_scatter_kernel<true><<<grid, kSortThreads, 0, stream>>>(kin, vin, n, shift, from_top, n_tiles, table, kout, vout);
        else
            sort_scatter_kernel<false><<<grid, kSortThreads, 0, stream>>>(kin, vin, n, shift, from_top, n_tiles, table, kout, vout);
        if (hipGetLastError() != hipSuccess) return GNN_ERR_LAUNCH;
        kin = kout;
        vin = vout;
        from_top = 0;
        cur ^= 1;
    }
    if (keys_out) *keys_out = const_cast<uint32_t *>(kin);
    if (vals_out) *vals_out = const_cast<uint32_t *>(vin);
    return GNN_OK;
}

int grid_for(int64_t n, int block, int64_t cap = (int64_t(1) << 16)) {
    int64_t g = (n + block - 1) / block;
    if (g < 1) g = 1;
    if (g > cap) g = cap;
    return static_cast<int>(g);
}

// The transposed graph, by a stable sort of the edges on the bits a source id can occupy; asynchronous.  row_of: the row of
// every edge (null: expanded from indptr here).  Where neither the permutation nor weights are asked for, the rows themselves
// are sorted and the last pass writes indices_t; otherwise the edges' positions are.
int transpose(const int32_t *row_of, const void *indptr, const int32_t *indices, const float *edge_w, int64_t E, int64_t N,
              int indptr_is_64, void *indptr_t, int32_t *indices_t, int64_t *perm, float *edge_w_t, hipStream_t stream) {
    const bool by_position = perm || edge_w;
    const int bits = gnn_ilog2_ceil(N > 1 ? N : 2);
    const bool one_pass = bits <= 8;
    const int64_t n_table = gnn_sort_table_elems(E), n_sums = gnn_sort_sums_elems(E);
    // [row_of][keys x 2][values x 2][table][sums]; a single pass writes one buffer of each
    const int64_t n_words = (row_of ? 0 : E) + (one_pass ? 2 : 4) * E + n_table + n_sums;
    gnn_dev_ptr<uint32_t> arena;
    if (!arena.alloc_on(n_words, stream)) return GNN_ERR_ALLOC;
    uint32_t *next = arena.p;
    if (!row_of) {
        int32_t *rows = reinterpret_cast<int32_t *>(next);
        next += E;
        if (indptr_is_64)
            expand_rows_kernel<int64_t><<<grid_for(N * 64, 256), 256, 0, stream>>>(static_cast<const int64_t *>(indptr), N, rows);
        else
            expand_rows_kernel<int32_t><<<grid_for(N * 64, 256), 256, 0, stream>>>(static_cast<const int32_t *>(indptr), N, rows);
        if (hipGetLastError() != hipSuccess) return GNN_ERR_LAUNCH;
        row_of = rows;
    }
    SortJob job;
    job.first_keys = reinterpret_cast<const uint32_t *>(indices);
    job.first_vals = by_position ? nullptr : reinterpret_cast<const uint32_t *>(row_of);
    for (int i = 1; i >= (one_pass ? 1 : 0); --i) {
        job.buf_k[i] = next; next += E;
        job.buf_v[i] = next; next += E;
    }
    if (!by_position) job.last_vals = reinterpret_cast<uint32_t *>(indices_t);
    uint32_t *keys = nullptr, *vals = nullptr;
    int rc = radix_sort(job, E, bits, next, next + n_table, stream, &keys, &vals);
    if (rc != GNN_OK) return rc;
    rc = gnn_csr_from_sorted_coo(reinterpret_cast<const int32_t *>(keys), E, N, indptr_t, indptr_is_64, stream);
    if (rc != GNN_OK) return rc;
    if (by_position)
        gather_transposed_kernel<<<grid_for(E, 256), 256, 0, stream>>>(vals, E, row_of, edge_w, indices_t, perm, edge_w ? edge_w_t : nullptr);
    return hipGetLastError() == hipSuccess ? GNN_OK : GNN_ERR_LAUNCH;
}

}  // namespace

int gnn_read_edge_count(const void *indptr, int64_t N, int indptr_is_64, hipStream_t stream, int64_t *E) {
    union Count { int64_t e64; int32_t e32; };
    Count *host = static_cast<Count *>(gnn_host_block());
    if (!host) return GNN_ERR_ALLOC;
    const size_t bytes = indptr_is_64 ? 8 : 4;
    const hipError_t err = hipMemcpyAsync(host, static_cast<const char *>(indptr) + size_t(N) * bytes, bytes, hipMemcpyDeviceToHost, stream);
    const hipError_t end = hipStreamSynchronize(stream);
    *E = indptr_is_64 ? host->e64 : int64_t(host->e32);
    gnn_host_block_free(host);
    return err == hipSuccess && end == hipSuccess ? GNN_OK : GNN_ERR_LAUNCH;
}

int gnn_radix_sort_pairs(uint32_t *buf_k[2], uint32_t *buf_v[2], int64_t n, int bits, uint32_t *table, uint32_t *sums,
                         hipStream_t stream, int *out) {
    SortJob job;
    job.first_keys = buf_k[0];
    job.first_vals = buf_v[0];
    for (int i = 0; i < 2; ++i) { job.buf_k[i] = buf_k[i]; job.buf_v[i] = buf_v[i]; }
    *out = (bits + 7) / 8 % 2;
    return radix_sort(job, n, bits, table, sums, stream, nullptr, nullptr);
}
int64_t gnn_sort_table_elems(int64_t n) { return (n + kSortTile - 1) / kSortTile * 256; }
int64_t gnn_sort_sums_elems(int64_t n) { return gnn_scan_sums_elems(gnn_sort_table_elems(n)); }
int64_t gnn_scan_sums_elems(int64_t n) { return (n + kScanChunk - 1) / kScanChunk + 1; }
int gnn_scan_exclusive_u32(uint32_t *data, int64_t n, uint32_t *sums, hipStream_t stream) {
    return scan_exclusive<uint32_t>(data, n, 1, 0, false, sums, stream);
}
int gnn_scan_exclusive_i64(int64_t *data, int64_t n, int n_arrays, int64_t stride, int64_t *sums, hipStream_t stream) {
    return scan_exclusive<int64_t>(data, n, n_arrays, stride, true, sums, stream);
}

extern "C" GNN_API int gnn_csr_from_sorted_coo(const int32_t *dst_sorted, int64_t E, int64_t N, void *indptr_out,
                                       int indptr_is_64, void *stream_v) {
    if (N < 0 || E < 0 || !indptr_out || (E > 0 && !dst_sorted)) return GNN_ERR_INVALID_ARG;
    if (!indptr_is_64 && E > INT32_MAX) return GNN_ERR_INVALID_ARG;
    hipStream_t stream = static_cast<hipStream_t>(stream_v);
    (void)hipGetLastError();  // a stale error of an earlier, failed call must not be blamed on this one
    if (indptr_is_64)
        indptr_from_sorted_kernel<int64_t><<<grid_for(E + 1, 256), 256, 0, stream>>>(dst_sorted, E, N, static_cast<int64_t *>(indptr_out));
    else
        indptr_from_sorted_kernel<int32_t><<<grid_for(E + 1, 256), 256, 0, stream>>>(dst_sorted, E, N, static_cast<int32_t *>(indptr_out));
    GNN_HIP_TRY(hipGetLastError());
    return GNN_OK;
}

extern "C" GNN_API int gnn_transpose_csr(const void *indptr, const int32_t *indices, const float *edge_w, int64_t N,
                                 int indptr_is_64, void *indptr_t, int32_t *indices_t, int64_t *perm,
                                 float *edge_w_t, void *stream_v) {
    if (N < 0 || N > INT32_MAX || !indptr || !indptr_t) return GNN_ERR_INVALID_ARG;
    if (edge_w && !edge_w_t) return GNN_ERR_INVALID_ARG;
    hipStream_t stream = static_cast<hipStream_t>(stream_v);
    (void)hipGetLastError();
    int64_t E = 0;
    int rc = gnn_read_edge_count(indptr, N, indptr_is_64, stream, &E);
    if (rc != GNN_OK) return rc;
    if (E < 0 || E > int64_t(UINT32_MAX)) return GNN_ERR_INVALID_ARG;
    if (E > 0 && (!indices || !indices_t)) return GNN_ERR_INVALID_ARG;
    if (E == 0) {
        GNN_HIP_TRY(hipMemsetAsync(indptr_t, 0, (indptr_is_64 ? 8 : 4) * (N + 1), stream));
        GNN_HIP_TRY(hipStreamSynchronize(stream));
        return GNN_OK;
    }

    rc = transpose(static_cast<const int32_t *>(nullptr), indptr, indices, edge_w, E, N, indptr_is_64, indptr_t, indices_t, perm, edge_w_t, stream);
    // synchronous: whatever was launched has ended when the caller sees the outputs, on success and on failure
    if (hipStreamSynchronize(stream) != hipSuccess && rc == GNN_OK) rc = GNN_ERR_LAUNCH;
    return rc;
}

extern "C" GNN_API int gnn_graph_build(const int32_t *dst_sorted, const int32_t *src, const float *edge_w, int64_t E, int64_t N,
                                       int indptr_is_64, void *indptr, void *indptr_t, int32_t *indices_t, int64_t *perm,
                                       float *edge_w_t, const gnn_plan_params *params, void *stream_v, gnn_plan **plan_fwd,
                                       gnn_plan **plan_bwd) {
    if (plan_fwd) *plan_fwd = nullptr;
    if (plan_bwd) *plan_bwd = nullptr;
    if (!plan_fwd != !plan_bwd) return GNN_ERR_INVALID_ARG;
    if (N < 0 || N > INT32_MAX || E < 0 || E > int64_t(UINT32_MAX) || !indptr || !indptr_t) return GNN_ERR_INVALID_ARG;
    if (E > 0 && (!dst_sorted || !src || !indices_t)) return GNN_ERR_INVALID_ARG;
    if (edge_w && !edge_w_t) return GNN_ERR_INVALID_ARG;
    hipStream_t stream = static_cast<hipStream_t>(stream_v);
    int rc = gnn_csr_from_sorted_coo(dst_sorted, E, N, indptr, indptr_is_64, stream_v);
    if (rc != GNN_OK) return rc;
    if (E == 0)
        rc = gnn_csr_from_sorted_coo(nullptr, 0, N, indptr_t, indptr_is_64, stream_v);
    else
        rc = transpose(dst_sorted, indptr, src, edge_w, E, N, indptr_is_64, indptr_t, indices_t, perm, edge_w_t, stream);
    if (rc == GNN_OK && plan_fwd)
        rc = gnn_plan_create_pair(indptr, indptr_t, src, E, N, indptr_is_64, params, stream, plan_fwd, plan_bwd);
    if (hipStreamSynchronize(stream) != hipSuccess && rc == GNN_OK) rc = GNN_ERR_LAUNCH;
    return rc;
}

extern "C" GNN_API int gnn_validate_csr(const void *indptr, const int32_t *indices, int64_t N, int64_t E, int indptr_is_64,
                                void *stream_v) {
    if (N < 0 || E < 0 || !indptr || (E > 0 && !indices)) return GNN_ERR_INVALID_ARG;
    hipStream_t stream = static_cast<hipStream_t>(stream_v);
    (void)hipGetLastError();
    gnn_dev_ptr<int> flag;
    if (!flag.alloc_on(1, stream)) return GNN_ERR_ALLOC;
    int *bad = flag.p;
    int host_bad = 0;
    int rc = GNN_OK;
    if (hipMemsetAsync(bad, 0, sizeof(int), stream) != hipSuccess) rc = GNN_ERR_LAUNCH;
    if (rc == GNN_OK) {
        int64_t work = (N > E ? N : E) + 1;
        if (indptr_is_64)
            validate_kernel<int64_t><<<grid_for(work, 256), 256, 0, stream>>>(static_cast<const int64_t *>(indptr), indices, N, E, bad);
        else
            validate_kernel<int32_t><<<grid_for(work, 256), 256, 0, stream>>>(static_cast<const int32_t *>(indptr), indices, N, E, bad);
        if (hipGetLastError() != hipSuccess) rc = GNN_ERR_LAUNCH;
    }
    if (rc == GNN_OK && hipMemcpyAsync(&host_bad, bad, sizeof(int), hipMemcpyDeviceToHost, stream) != hipSuccess) rc = GNN_ERR_LAUNCH;
    if (rc == GNN_OK && hipStreamSynchronize(stream) != hipSuccess) rc = GNN_ERR_LAUNCH;
    if (rc != GNN_OK) return rc;
    return host_bad ? GNN_ERR_INVALID_GRAPH : GNN_OK;
}

// rank[v] = position of vertex v when the vertices are ordered by descending count (equal counts by ascending id: the sort
// is stable).  max_count: no count is larger; it says how many bits the sort looks at.  Asynchronous.
int gnn_rank_by_count(const int32_t *counts, int64_t N, int64_t max_count, int32_t *rank, hipStream_t stream) {
    if (N <= 0) return GNN_OK;
    if (!counts || !rank || N > INT32_MAX || max_count < 0) return GNN_ERR_INVALID_ARG;
    (void)hipGetLastError();
    const uint32_t top = max_count < 1 ? 1u : (max_count > INT32_MAX ? uint32_t(INT32_MAX) : uint32_t(max_count));
    const int64_t n_table = gnn_sort_table_elems(N), n_sums = gnn_sort_sums_elems(N);
    gnn_dev_ptr<uint32_t> arena;
    if (!arena.alloc_on(4 * N + n_table + n_sums, stream)) return GNN_ERR_ALLOC;
    SortJob job;
    job.first_keys = reinterpret_cast<const uint32_t *>(counts);
    job.from_top = top;  // ascending keys = descending counts
    for (int i = 0; i < 2; ++i) {
        job.buf_k[i] = arena.p + i * N;
        job.buf_v[i] = arena.p + (2 + i) * N;
    }
    job.last_vals = reinterpret_cast<uint32_t *>(rank);
    job.inverse_last = true;
    return radix_sort(job, N, gnn_ilog2_ceil(int64_t(top) + 1), arena.p + 4 * N, arena.p + 4 * N + n_table, stream, nullptr, nullptr);
}

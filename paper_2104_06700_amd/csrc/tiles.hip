// Gather of the long rows from source tiles staged in LDS.
//
// The pieces of blocked.hip gather a block of sources from an L2, one 128-byte request per edge, and the
// request rate of the L2s (about 160 G lines/s over the chip, 20 TB/s) bounds them.  Where the long rows have
// many edges into a block, a second level of blocking pays: a workgroup copies a tile of the block's sources
// (124 KB: 991 lines of 128 bytes, or more shorter ones) into LDS once, and all the rows it owns gather their
// edges into that tile from there; then the next tile.  The sums stay in registers from the first tile to the
// last, so a row writes one partial line per launch and not one per piece.
//
// A workgroup is 16 wavefronts; L lanes (16 bytes each: L = 8, 4 or 2 for lines of 128, 64 or 32 bytes) own a
// row, so a wavefront works on a bundle of 64 / L rows at a time, and it owns up to ten bundles.  The lists are
// stored the way they are read, one stream per wavefront: for every tile, for every bundle of the wavefront, units
// of four edges per row as 16-bit offsets into the tile, in an order that spreads a read over the banks (BankOrder); the
// shorter rows of a bundle are filled up with the offsets of lines of zeros behind the tile.  Rows are bundled by similar number of edges, a row much longer
// than the mean is cut into parts (else it alone would set the time of its workgroup: worst workgroup 4.1 x the
// mean without, 1.02 x with), and the bundles are dealt to the wavefronts like cards.
//
// What bounds it: vector instructions (four additions per lane and line, one multiply-add for the line's address, half a
// move), which fill 88 % of the cycles in which a compute unit has a wavefront of the launch; the LDS is active in 70 %, one
// hundredth of that in bank conflicts (a third before the streams were ordered by banks).  Measured on the 233 K-vertex graph: F=602,
// 19 lines, 3.8 ms alone, where the same edges as pieces took over 9.5 ms; the call 11.45 -> 8.0 (tiles) -> 7.0 (order) ->
// 6.85 ms (half of the next tile fetched ahead).  The 2.45 M-vertex graph: F=256 1.23 ms alone; the call, half of which the
// short rows take, 9.15 -> 8.35 -> 7.50 ms.
#include <algorithm>
#include <new>
#include <type_traits>
#include <utility>
#include <vector>

#include "common.h"

namespace {

constexpr int kTileThreads = 1024;
constexpr int kTileWaves = kTileThreads / 64;
constexpr int kCounts = 16;        // bytes of counts per wavefront and tile (bundles it owns at most)
// Bundles of rows a wavefront owns at most: as many sums as four wavefronts per SIMD leave registers for.
constexpr int kBundlesF32 = 10, kBundlesBf16 = 8;
constexpr int kUnit = 4;          // edges per row in a unit of the streams
constexpr uint32_t kMaxSegment = 255 * kUnit;  // edges of a row part into one tile at most: a byte of units

constexpr int64_t kFewBundles = 5;      // bundles per wavefront before rows are dealt to more workgroups
constexpr int64_t kRowBlocks = 64;     // workgroups the rows are dealt to at least (per column slice)
constexpr int64_t kComputeUnits = 256;
// A row is staged in a block where it has this many edges per tile: a staged line costs a fifth of a gathered one, but a row's list is
// filled up to whole units and to the longest of its bundle (5 -> 3 -> 2, with 3,000 below: 2.45 M vertices F=256 8.20 -> 7.94 ->
// 7.93 ms, 233 K vertices 2.77 -> 2.72 -> 2.67) ...
constexpr int64_t kMinRowEdges = 2;
// ... and a block where those rows have this many edges per tile and workgroup of rows: what copying the tile costs
// (2.45 M vertices F=256 8.45 ms with 1,000, 7.72-7.76 from 2,000 to 4,000; the others within 1 %).
constexpr int64_t kMinTileEdges = 3000;
constexpr int kStreamAhead = 64;  // units of padding behind a stream (the loads run up to 2 KB ahead)

int grid_for(int64_t n, int block, int64_t cap = (int64_t(1) << 16)) {
    int64_t g = (n + block - 1) / block;
    if (g < 1) g = 1;
    if (g > cap) g = cap;
    return static_cast<int>(g);
}

struct TileDesc { int32_t begin, size, block, pad; };

// Number of bundle r of wavefront w in a list sorted by size, or -1: dealt from the largest down, forwards, then
// backwards, so that wavefronts get equal loads; neighbours in the list go to different workgroups.
__host__ __device__ __forceinline__ int64_t dealt_bundle(int64_t w, int r, int64_t n_waves, int64_t n_bundles) {
    const int64_t at = (w % kTileWaves) * (n_waves / kTileWaves) + w / kTileWaves;
    const int64_t k = int64_t(r) * n_waves + ((r & 1) ? n_waves - 1 - at : at);
    return n_bundles - 1 - k;
}

// The cells (block, row) that are worth staging: block_min[k] = edges a row needs in block k for that (0: none).
struct DenseRule {
    const uint32_t *cell_off;
    const uint32_t *block_min;
    int64_t n_hot;
    __device__ __forceinline__ uint32_t edges(int k, int64_t h) const {
        const int64_t c = int64_t(k) * n_hot + h;
        const uint32_t n = cell_off[c + 1] - cell_off[c];
        const uint32_t least = block_min[k];
        return least && n >= least ? n : 0u;
    }
};

// sums[k] += edges of the dense cells of block k (blockIdx.y)
__global__ void __launch_bounds__(256) tile_block_edges_kernel(DenseRule rule, unsigned long long *__restrict__ sums) {
    __shared__ unsigned long long part[256];
    const int k = blockIdx.y;
    unsigned long long s = 0;
    for (int64_t h = int64_t(blockIdx.x) * blockDim.x + threadIdx.x; h < rule.n_hot; h += int64_t(gridDim.x) * blockDim.x) s += rule.edges(k, h);
    part[threadIdx.x] = s;
    __syncthreads();
    for (int off = 128; off > 0; off >>= 1) {
        if (int(threadIdx.x) < off) part[threadIdx.x] += part[threadIdx.x + off];
        __syncthreads();
    }
    if (threadIdx.x == 0 && part[0]) atomicAdd(&sums[k], part[0]);
}

// staged[h] = edges of hot row h in its dense cells; n_staged += rows that have any
__global__ void __launch_bounds__(256) tile_row_edges_kernel(DenseRule rule, int n_blocks, uint32_t *__restrict__ staged,
                                                             uint32_t *__restrict__ n_staged) {
    const int64_t h = int64_t(blockIdx.x) * blockDim.x + threadIdx.x;
    uint32_t s = 0;
    if (h < rule.n_hot) {
        for (int k = 0; k < n_blocks; ++k) s += rule.edges(k, h);
        staged[h] = s;
    }
    const unsigned long long m = __ballot(s != 0);
    if ((threadIdx.x & 63) == 0 && m) atomicAdd(n_staged, uint32_t(__popcll(m)));
}

// parts[h] = parts that row h is cut into: of `cap` edges at most (a row much longer than the others would keep its
// workgroup waiting), and of no more edges into one tile than the counts of a stream can say
__global__ void __launch_bounds__(256) tile_row_parts_kernel(const uint32_t *__restrict__ staged, const uint32_t *__restrict__ longest,
                                                             int64_t n_hot, uint32_t cap, uint32_t *__restrict__ parts) {
    const int64_t h = int64_t(blockIdx.x) * blockDim.x + threadIdx.x;
    if (h >= n_hot) return;
    const uint32_t n = (staged[h] + cap - 1) / cap, m = (longest[h] + kMaxSegment - 1) / kMaxSegment;
    parts[h] = n > m ? n : m;
}

// The parts of every row: row, number within the row, parts of the row; and what they are sorted by.
struct RowPart { uint32_t row, part, parts; };
__global__ void __launch_bounds__(256) tile_parts_kernel(const uint32_t *__restrict__ staged, const uint32_t *__restrict__ part_base,
                                                         int64_t n_hot, RowPart *__restrict__ out,
                                                         uint32_t *__restrict__ keys, uint32_t *__restrict__ ids) {
    const int64_t h = int64_t(blockIdx.x) * blockDim.x + threadIdx.x;
    if (h >= n_hot) return;
    const uint32_t n = part_base[h + 1] - part_base[h];
    for (uint32_t j = 0; j < n; ++j) {
        const uint32_t v = part_base[h] + j;
        out[v] = RowPart{uint32_t(h), j, n};
        keys[v] = staged[h] / n;
        ids[v] = v;
    }
}

// Piece counts of the cells that stay pieces (0 where a cell is staged), and the edge counts they are cut from.
__global__ void __launch_bounds__(256) tile_left_cells_kernel(DenseRule rule, int n_blocks, uint32_t max_piece,
                                                              uint32_t *__restrict__ cell_count, uint32_t *__restrict__ cell_pieces) {
    const int64_t n_cells = int64_t(n_blocks) * rule.n_hot;
    const int64_t stride = int64_t(gridDim.x) * blockDim.x;
    for (int64_t c = int64_t(blockIdx.x) * blockDim.x + threadIdx.x; c < n_cells; c += stride) {
        const int k = int(c / rule.n_hot);
        const uint32_t n = rule.edges(k, c - int64_t(k) * rule.n_hot) ? 0u : rule.cell_off[c + 1] - rule.cell_off[c];
        cell_count[c] = n;
        cell_pieces[c] = (n + max_piece - 1) / max_piece;
    }
}

// first position in [lo, hi) of the ascending list r whose rank is >= bound
__device__ __forceinline__ uint32_t lower_bound_in(const int32_t *__restrict__ r, uint32_t lo, uint32_t hi, int32_t bound) {
    while (lo < hi) {
        const uint32_t mid = lo + ((hi - lo) >> 1);
        if (r[mid] < bound) lo = mid + 1; else hi = mid;
    }
    return lo;
}

// longest[h] = most edges of row h into one tile (zeroed before)
__global__ void __launch_bounds__(256) tile_longest_kernel(const TileDesc *__restrict__ tiles, int n_tiles, DenseRule rule,
                                                           const int32_t *__restrict__ blk_indices, const uint32_t *__restrict__ depth,
                                                           uint32_t *__restrict__ longest) {
    const int64_t total = int64_t(n_tiles) * rule.n_hot;
    const int64_t stride = int64_t(gridDim.x) * blockDim.x;
    for (int64_t x = int64_t(blockIdx.x) * blockDim.x + threadIdx.x; x < total; x += stride) {
        const TileDesc d = tiles[x / rule.n_hot];
        const int64_t h = x % rule.n_hot;
        if (rule.edges(d.block, h) <= kMaxSegment) continue;  // short enough wherever its tiles begin
        if (depth && uint32_t(x / rule.n_hot) < depth[h]) continue;
        const int64_t c = int64_t(d.block) * rule.n_hot + h;
        const uint32_t hi = rule.cell_off[c + 1], b = lower_bound_in(blk_indices, rule.cell_off[c], hi, d.begin);
        atomicMax(&longest[h], lower_bound_in(blk_indices, b, hi, d.begin + d.size) - b);
    }
}

// seg[t * n_parts + i] = (begin, end) in the block-major edge list of the edges of row part order[i] into tile t; none of a row's first
// depth[row] tiles (null: 0), which the bit matrix has
__global__ void __launch_bounds__(256) tile_segments_kernel(const TileDesc *__restrict__ tiles, int n_tiles, DenseRule rule,
                                                            const uint32_t *__restrict__ order, const RowPart *__restrict__ parts,
                                                            int64_t n_parts, const int32_t *__restrict__ blk_indices,
                                                            const uint32_t *__restrict__ depth, uint2 *__restrict__ seg) {
    const int64_t total = int64_t(n_tiles) * n_parts;
    const int64_t stride = int64_t(gridDim.x) * blockDim.x;
    for (int64_t x = int64_t(blockIdx.x) * blockDim.x + threadIdx.x; x < total; x += stride) {
        const int t = int(x / n_parts);
        const RowPart p = parts[order[x - int64_t(t) * n_parts]];
        const TileDesc d = tiles[t];
        uint2 s = make_uint2(0u, 0u);
        if (rule.edges(d.block, p.row) && !(depth && uint32_t(t) < depth[p.row])) {
            const int64_t c = int64_t(d.block) * rule.n_hot + p.row;
            const uint32_t lo = rule.cell_off[c], hi = rule.cell_off[c + 1];
            const uint32_t b = lower_bound_in(blk_indices, lo, hi, d.begin);
            const uint64_t len = lower_bound_in(blk_indices, b, hi, d.begin + d.size) - b;
            s.x = b + uint32_t(len * p.part / p.parts);
            s.y = b + uint32_t(len * (p.part + 1) / p.parts);
        }
        seg[x] = s;
    }
}

// One thread per (wavefront, tile): iterations of each of its bundles there, and their sum.
__global__ void __launch_bounds__(256) tile_counts_kernel(const uint2 *__restrict__ seg, int64_t n_parts, int n_tiles, int64_t n_waves,
                                                          int rr, int rows_per_bundle, uint8_t *__restrict__ counts,
                                                          uint32_t *__restrict__ wave_tile_iters) {
    const int64_t n_bundles = (n_parts + rows_per_bundle - 1) / rows_per_bundle;
    const int64_t total = n_waves * n_tiles;
    const int64_t stride = int64_t(gridDim.x) * blockDim.x;
    for (int64_t x = int64_t(blockIdx.x) * blockDim.x + threadIdx.x; x < total; x += stride) {
        const int64_t w = x / n_tiles;
        const int t = int(x - w * n_tiles);
        uint32_t sum = 0;
        for (int r = 0; r < rr; ++r) {
            const int64_t i0 = dealt_bundle(w, r, n_waves, n_bundles) * rows_per_bundle;
            uint32_t most = 0;
            for (int g = 0; g < rows_per_bundle; ++g) {
                if (i0 < 0 || i0 + g >= n_parts) break;
                const uint2 s = seg[int64_t(t) * n_parts + i0 + g];
                const uint32_t n = (s.y - s.x + kUnit - 1) / kUnit;
                most = n > most ? n : most;
            }
            counts[x * kCounts + r] = uint8_t(most);
            sum += most;
        }
        wave_tile_iters[x] = sum;
    }
}

// Order of a row's edges into a tile.  The LDS serves a 16-byte read of 64 lanes four times 16 lanes at a time, 64 banks of 4
// bytes each: of every 32 lanes first the quads 0, 3, 5, 6, then 1, 2, 4, 7.  L lanes read a line of 16 * L bytes, so a line
// lies in one of C = 16 / L classes of banks (line % C), and C rows of a bundle are served together: where two of their lines
// are of one class, one waits.  (Measured: 4.5 clocks per read of a compute unit without conflicts, 8.1 with.)  So the slots of
// the C rows are cut into C sections, and row i of them puts its lines of class (i + t) % C into section t; what does not
// fit goes where other classes left room, and lines of zeros of the fitting class fill the rest.
template <int L>
struct BankOrder {
    static constexpr int C = 16 / L;
    int pos;              // of the row among the C rows
    int begin[C], size[C];  // sections
    int n[C];             // edges of the row that belong in each

    // position of row g of a bundle among the rows it is served with; those are the g that lay_out() takes the maximum over
    static __device__ __forceinline__ int position(int g) {
        return L == 2 ? ((g & 15) >> 2) * 2 + (g & 1) : (g & (C * 2 - 1)) >> 1;
    }
    __device__ __forceinline__ int section(int line) const { return (line - pos) & (C - 1); }
    __device__ __forceinline__ int line_class(int t) const { return (pos + t) & (C - 1); }

    // n is set; n_slots = slots of every row of the bundle.  All lanes of the wavefront call it.
    __device__ __forceinline__ void lay_out(int n_slots) {
        int need[C], total = 0;
#pragma unroll
        for (int t = 0; t < C; ++t) {
            int m = n[t];
            if (L == 2) m = max(m, __shfl_xor(m, 1 * L));
            m = max(m, __shfl_xor(m, (L == 2 ? 6 : 3) * L));
            if (L < 8) m = max(m, __shfl_xor(m, (L == 2 ? 10 : 5) * L));
            need[t] = m;
            total += m;
        }
        int run = 0, sum = 0;
#pragma unroll
        for (int t = 0; t < C; ++t) {
            begin[t] = run;
            sum += need[t];
            run = t == C - 1 ? n_slots : (total <= n_slots ? run + need[t] : n_slots * sum / total);
            size[t] = run - begin[t];
        }
    }
    // slot number `k` of those that the sections' own edges leave free
    __device__ __forceinline__ int free_slot(int k) const {
        int at = 0;
        bool found = false;
#pragma unroll
        for (int t = 0; t < C; ++t) {
            const int room = size[t] > n[t] ? size[t] - n[t] : 0;
            if (!found && k < room) { at = begin[t] + n[t] + k; found = true; }
            k -= room;
        }
        return at;
    }
    // slot of edge number j of section t
    __device__ __forceinline__ int slot(int t, int j) const {
        int at = 0, before = 0;  // edges of the sections before that do not fit
        bool fits = false;
#pragma unroll
        for (int q = 0; q < C; ++q) {
            if (q == t) { fits = j < size[q]; at = fits ? begin[q] + j : j - size[q]; }
            if (q < t && n[q] > size[q]) before += n[q] - size[q];
        }
        return fits ? at : free_slot(before + at);
    }
    __device__ __forceinline__ int overflow() const {
        int x = 0;
#pragma unroll
        for (int t = 0; t < C; ++t) x += n[t] > size[t] ? n[t] - size[t] : 0;
        return x;
    }
};

// What tile_fill_kernel writes for every slot of the stream.
enum TileFill {
    kFillIndices,    // line of the tile; a line of zeros where a row is filled up
    kFillCoefs,      // w[epos] * scale[epos]; 0 where a row is filled up
    kFillPositions,  // epos; kNoEdge where a row is filled up
};
constexpr uint32_t kNoEdge = 0xFFFFFFFFu;

__device__ __forceinline__ float coefficient(const float *__restrict__ w, const float *__restrict__ scale, uint32_t p) {
    if (p == kNoEdge) return 0.0f;
    const float cf = w ? w[p] : 1.0f;
    return scale ? cf * scale[p] : cf;
}

// One wavefront per (wavefront of the gather, tile): its stretch of the stream.  L lanes own a row.
template <int L, TileFill WHAT>
__global__ void __launch_bounds__(256) tile_fill_kernel(const TileDesc *__restrict__ tiles, int n_tiles, int64_t n_waves, int rr,
                                                        const uint2 *__restrict__ seg, int64_t n_parts,
                                                        const uint8_t *__restrict__ counts, const uint32_t *__restrict__ wave_off,
                                                        const int32_t *__restrict__ blk_indices, const uint32_t *__restrict__ blk_epos,
                                                        const float *__restrict__ w, const float *__restrict__ scale,
                                                        int zero_line, uint16_t *__restrict__ stream, float *__restrict__ wstream,
                                                        uint32_t *__restrict__ positions) {
    constexpr int ROWS = 64 / L, SLOTS = ROWS * kUnit, C = BankOrder<L>::C;
    const int lane = threadIdx.x & 63, g = lane / L, c = lane & (L - 1);
    const unsigned long long row_lanes = ((1ull << L) - 1ull) << (lane & ~(L - 1));
    const unsigned long long before_me = row_lanes & ((1ull << lane) - 1ull);
    const int64_t n_bundles = (n_parts + ROWS - 1) / ROWS;
    const int64_t total = n_waves * n_tiles;
    const int64_t n_workers = int64_t(gridDim.x) * (blockDim.x >> 6);
    for (int64_t x = int64_t(blockIdx.x) * (blockDim.x >> 6) + (threadIdx.x >> 6); x < total; x += n_workers) {
        const int64_t wv = x / n_tiles;
        const int t = int(x - wv * n_tiles);
        const int32_t tile_begin = tiles[t].begin;
        int64_t out = int64_t(wave_off[x]) * SLOTS;
        for (int r = 0; r < rr; ++r) {
            const int n_it = counts[x * kCounts + r];
            const int64_t i = dealt_bundle(wv, r, n_waves, n_bundles) * ROWS + g;
            uint2 sg = make_uint2(0u, 0u);
            if (n_it > 0 && i >= 0 && i < n_parts) sg = seg[int64_t(t) * n_parts + i];
            BankOrder<L> order;
            order.pos = BankOrder<L>::position(g);
            // number of the lane's edge within its section, counted on; every lane of a row holds the row's counts
            auto count = [&](int sec, bool valid, int &mine) {
                mine = 0;
#pragma unroll
                for (int q = 0; q < C; ++q) {
                    const unsigned long long m = __ballot(valid && sec == q);
                    if (sec == q) mine = order.n[q] + __popcll(m & before_me);
                    order.n[q] += __popcll(m & row_lanes);
                }
            };
            auto section_of = [&](uint32_t e) { return order.section(blk_indices[e] - tile_begin); };
#pragma unroll
            for (int q = 0; q < C; ++q) order.n[q] = 0;
            for (uint32_t e0 = sg.x; __any(e0 < sg.y); e0 += L) {
                int unused;
                const bool valid = e0 + c < sg.y;
                count(valid ? section_of(e0 + c) : 0, valid, unused);
            }
            const int n_slots = n_it * kUnit;
            order.lay_out(n_slots);
            auto put = [&](int slot, int idx, uint32_t p) {
                const int64_t at = out + int64_t(slot / kUnit) * SLOTS + g * kUnit + slot % kUnit;
                if constexpr (WHAT == kFillIndices) stream[at] = uint16_t(idx);
                else if constexpr (WHAT == kFillPositions) positions[at] = p;
                else wstream[at] = coefficient(w, scale, p);
            };
            const int spare = n_slots - int(sg.y - sg.x), over = order.overflow();
            for (int k = c; k < spare; k += L) {  // the lines of zeros
                const int slot = order.free_slot(over + k);
                int sec = 0;
#pragma unroll
                for (int q = 1; q < C; ++q) sec = slot >= order.begin[q] ? q : sec;
                put(slot, zero_line + order.line_class(sec), kNoEdge);
            }
            const BankOrder<L> whole = order;
#pragma unroll
            for (int q = 0; q < C; ++q) order.n[q] = 0;
            for (uint32_t e0 = sg.x; __any(e0 < sg.y); e0 += L) {
                const uint32_t e = e0 + c;
                const bool valid = e < sg.y;
                const int sec = valid ? section_of(e) : 0;
                int j;
                count(sec, valid, j);
                if (valid) put(whole.slot(sec, j), blk_indices[e] - tile_begin, WHAT == kFillIndices ? 0u : blk_epos[e]);
            }
            out += int64_t(n_it) * SLOTS;
        }
    }
}

// The same coefficients from the positions of a kFillPositions: four slots per thread, no order to work out again.
__global__ void __launch_bounds__(256) tile_refill_kernel(const uint4 *__restrict__ positions, int64_t n, const float *__restrict__ w,
                                                          const float *__restrict__ scale, float4 *__restrict__ wstream) {
    const int64_t stride = int64_t(gridDim.x) * blockDim.x;
    for (int64_t i = int64_t(blockIdx.x) * blockDim.x + threadIdx.x; i < n; i += stride) {
        const uint4 p = positions[i];
        wstream[i] = make_float4(coefficient(w, scale, p.x), coefficient(w, scale, p.y), coefficient(w, scale, p.z), coefficient(w, scale, p.w));
    }
}

// ---------------------------------------------------------------- the gather
struct TileArgs {
    const TileDesc *tiles;
    int32_t n_tiles, n_slices, n_groups;
    int32_t group_begin[GNN_TILE_MAX_GROUPS + 1];  // tiles of the workgroups' groups
    int64_t n_waves, n_parts;
    const uint16_t *stream;
    const float *wstream;
    const uint32_t *wave_off;   // [n_waves * n_tiles] in iterations
    const uint8_t *counts;      // [n_waves * n_tiles * kCounts]
    const uint32_t *order;
    const void *X;              // first slice table, rows of 16 * L bytes
    int64_t slice_stride;       // bytes
    float *partial;             // [n_groups][n_slices][n_parts][floats per line]
};

typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

template <bool BF16>
__device__ __forceinline__ void add_line(const u32x4 v, float (&acc)[BF16 ? 8 : 4]) {
    if constexpr (BF16) {
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            acc[2 * i] += __uint_as_float(v[i] << 16);
            acc[2 * i + 1] += __uint_as_float(v[i] & 0xFFFF0000u);
        }
    } else {
#pragma unroll
        for (int i = 0; i < 4; ++i) acc[i] += __uint_as_float(v[i]);
    }
}
template <bool BF16>
__device__ __forceinline__ void fma_line(const u32x4 v, float cf, float (&acc)[BF16 ? 8 : 4]) {
    if constexpr (BF16) {
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            acc[2 * i] = fmaf(cf, __uint_as_float(v[i] << 16), acc[2 * i]);
            acc[2 * i + 1] = fmaf(cf, __uint_as_float(v[i] & 0xFFFF0000u), acc[2 * i + 1]);
        }
    } else {
#pragma unroll
        for (int i = 0; i < 4; ++i) acc[i] = fmaf(cf, __uint_as_float(v[i]), acc[i]);
    }
}

// 16 bytes at lds0 + LINE_BYTES * (high or low half of `two`): one multiply-add forms the address.
template <int LINE_BYTES, bool HIGH>
__device__ __forceinline__ u32x4 lds_line(uint32_t two, uint32_t lds0) {
    uint32_t addr;
    if constexpr (HIGH) asm("v_mad_u32_u16 %0, %1, %2, %3 op_sel:[1,0,0,0]" : "=v"(addr) : "v"(two), "s"(LINE_BYTES), "v"(lds0));
    else asm("v_mad_u32_u16 %0, %1, %2, %3" : "=v"(addr) : "v"(two), "s"(LINE_BYTES), "v"(lds0));
    return *reinterpret_cast<__attribute__((address_space(3))) const u32x4 *>(static_cast<uintptr_t>(addr));
}

// Bytes of LDS the tile of lines of L * 16 bytes takes, the line of zeros included: what the streams leave of 160 KB.
// Of them the last are zeros, one per class of banks (BankOrder).
__host__ __device__ constexpr int zero_lines(int L) { return 16 / L; }
__host__ __device__ constexpr int tile_bytes(int L) { return (L == 8 ? 124 : (L == 4 ? 120 : 112)) << 10; }

// Value of lane J of each quad (PAIR: lane J of each pair of lanes) in all of its lanes.
template <int J, bool PAIR>
__device__ __forceinline__ uint32_t spread(uint32_t v) {
    constexpr int ctrl = PAIR ? (J == 0 ? 0xA0 : 0xF5) : J * 0x55;
    return uint32_t(__builtin_amdgcn_mov_dpp(int(v), ctrl, 0xF, 0xF, true));
}

template <bool BF16, int L, bool COEF, int RR>
__global__ void __launch_bounds__(kTileThreads) tile_kernel(const TileArgs a) {
    constexpr int VEC = BF16 ? 8 : 4;             // elements per lane
    constexpr int LOG2L = L == 8 ? 3 : (L == 4 ? 2 : 1);
    constexpr int ROWS = 64 / L;                  // rows of a bundle
    constexpr int TS = tile_bytes(L) / (16 * L);  // lines of the tile, the last zero_lines(L) of them zeros
    constexpr int CHUNKS = (TS * L + kTileThreads - 1) / kTileThreads;
    constexpr int AHEAD = 128 / ROWS;             // units that 1 KB of the offsets lasts
    constexpr int W_AHEAD = AHEAD / 2;            // ... and of the coefficients
    // The streams pass through LDS, 1 KB per wavefront at a time; the next KB waits in registers meanwhile, so
    // that a load has a KB's time to arrive.  Slot 0 takes the last unit of a KB that a step of two units did not fit.
    __shared__ uint2 ring[kTileWaves][(AHEAD + 1) * ROWS];
    __shared__ f32x4 w_ring[COEF ? kTileWaves : 1][(W_AHEAD + 1) * ROWS];
    __shared__ u32x4 tile[TS * L];
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(int(threadIdx.x >> 6));
    const int g = lane >> LOG2L, c = lane & (L - 1);
    const int slice = int(blockIdx.x % uint32_t(a.n_slices));
    const int rest = int(blockIdx.x / uint32_t(a.n_slices));
    const int group = rest % a.n_groups;
    const int64_t wv = int64_t(rest / a.n_groups) * kTileWaves + wave;
    const int t0 = a.group_begin[group], t1 = a.group_begin[group + 1];

    float acc[RR][VEC];
#pragma unroll
    for (int r = 0; r < RR; ++r)
#pragma unroll
        for (int i = 0; i < VEC; ++i) acc[r][i] = 0.0f;

    const int64_t first = int64_t(a.wave_off[wv * a.n_tiles + t0]) * ROWS;  // in units of one row
    const u32x4 *sp = reinterpret_cast<const u32x4 *>(reinterpret_cast<const uint2 *>(a.stream) + first) + lane;
    const f32x4 *wp = COEF ? reinterpret_cast<const f32x4 *>(a.wstream) + first + lane : nullptr;
    u32x4 nxt = sp[0];
    f32x4 w_nxt;
    if (COEF) w_nxt = wp[0];
    int pos = AHEAD + 1, w_pos = W_AHEAD + 1;  // next unit in the rings
    static_assert(RR <= kCounts, "the counts of a tile are one 16-byte load");
    const u32x4 *cnt = reinterpret_cast<const u32x4 *>(a.counts) + wv * a.n_tiles + t0;
    const char *Xs = static_cast<const char *>(a.X) + int64_t(slice) * a.slice_stride;
    // byte address of this lane's part of line 0; the lines of the tile follow each other
    const uint32_t lds0 = uint32_t(uintptr_t((__attribute__((address_space(3))) const u32x4 *)tile)) + 16u * uint32_t(c);
    // A unit of a row is two words of offsets; the four lanes of a quad (the two of a pair) read one (two) words of two
    // units each and spread them.
    constexpr bool PAIR = L == 2;
    const uint32_t *ring_lane = reinterpret_cast<const uint32_t *>(ring[wave]) +
                                (PAIR ? (c * ROWS + g) * 2 : (((lane >> 1) & 1) * ROWS + g) * 2 + (lane & 1));
    const float *w_lane = reinterpret_cast<const float *>(w_ring[COEF ? wave : 0]) + g * 4 + (PAIR ? 2 * c : lane & 3);
    constexpr int BATCH = BF16 ? 4 : 8;  // lines in flight per row: the registers beside 8 sums allow no more

    // one or two units (four edges of every row of the bundle each)
    auto step = [&](auto units, float (&sum)[VEC]) {
        constexpr int EDGES = decltype(units)::value * kUnit;
        if (pos >= AHEAD) {
            if (pos == AHEAD && lane < ROWS) ring[wave][lane] = ring[wave][AHEAD * ROWS + lane];
            *reinterpret_cast<u32x4 *>(&ring[wave][ROWS + 2 * lane]) = nxt;
            sp += 64;
            nxt = *sp;
            pos -= AHEAD;
        }
        uint32_t q[PAIR ? 2 : 1];
        q[0] = ring_lane[pos * (2 * ROWS)];
        if constexpr (PAIR) q[1] = ring_lane[pos * (2 * ROWS) + 1];
        pos += decltype(units)::value;
        float w[2][2];
        if (COEF) {
            if (w_pos >= W_AHEAD) {
                if (w_pos == W_AHEAD && lane < ROWS) w_ring[wave][lane] = w_ring[wave][W_AHEAD * ROWS + lane];
                w_ring[wave][ROWS + lane] = w_nxt;
                wp += 64;
                w_nxt = *wp;
                w_pos -= W_AHEAD;
            }
#pragma unroll
            for (int i = 0; i < EDGES / 4; ++i) {
                w[i][0] = w_lane[(w_pos + i) * (4 * ROWS)];
                if constexpr (PAIR) w[i][1] = w_lane[(w_pos + i) * (4 * ROWS) + 1];
            }
            w_pos += decltype(units)::value;
        }
        uint32_t two[4] = {0u, 0u, 0u, 0u};
        if constexpr (PAIR) {
            two[0] = spread<0, true>(q[0]); two[1] = spread<0, true>(q[1]);
            if (EDGES > 4) { two[2] = spread<1, true>(q[0]); two[3] = spread<1, true>(q[1]); }
        } else {
            two[0] = spread<0, false>(q[0]); two[1] = spread<1, false>(q[0]);
            if (EDGES > 4) { two[2] = spread<2, false>(q[0]); two[3] = spread<3, false>(q[0]); }
        }
        constexpr int B = EDGES < BATCH ? EDGES : BATCH;
#pragma unroll
        for (int h = 0; h < EDGES / B; ++h) {
            u32x4 x[B];
#pragma unroll
            for (int k = 0; k < B; ++k) {
                const uint32_t t = two[(h * B + k) >> 1];
                x[k] = (k & 1) ? lds_line<16 * L, true>(t, lds0) : lds_line<16 * L, false>(t, lds0);
            }
#pragma unroll
            for (int k = 0; k < B; ++k) {
                if constexpr (COEF) {
                    const int e = h * B + k;
                    const uint32_t wv0 = __float_as_uint(w[e >> 2][PAIR ? e & 1 : 0]);
                    const uint32_t cf = PAIR ? ((e & 2) ? spread<1, true>(wv0) : spread<0, true>(wv0))
                                             : ((e & 3) == 0 ? spread<0, false>(wv0) : (e & 3) == 1 ? spread<1, false>(wv0)
                                                : (e & 3) == 2 ? spread<2, false>(wv0) : spread<3, false>(wv0));
                    fma_line<BF16>(x[k], __uint_as_float(cf), sum);
                } else {
                    add_line<BF16>(x[k], sum);
                }
            }
        }
    };

    // Copying a tile takes its latency and 124 KB at a compute unit's share of the memory, with nothing else running there.  So
    // the first AHEAD_CHUNKS of a thread's chunks of the next tile are fetched while this one is gathered from, as many as the
    // registers beside the sums hold, and the others before the wavefronts wait for each other.
    constexpr int AHEAD_CHUNKS = BF16 ? 0 : (COEF ? 2 : 4);
    u32x4 first_chunks[AHEAD_CHUNKS ? AHEAD_CHUNKS : 1];
    auto chunk = [&](const TileDesc &t, int h) {
        const int x = int(threadIdx.x) + h * kTileThreads, n = t.size * L;
        return (reinterpret_cast<const u32x4 *>(Xs) + int64_t(t.begin) * L)[x < n ? x : n - 1];
    };
    auto put = [&](const TileDesc &t, int h, const u32x4 &v) {
        const int x = int(threadIdx.x) + h * kTileThreads;
        // the last zero_lines(L) lines, and what is behind a shorter tile, are zeros
        if (x < TS * L) tile[x] = x < t.size * L ? v : u32x4{0u, 0u, 0u, 0u};
    };
    TileDesc d = a.tiles[t0];
#pragma unroll
    for (int h = 0; h < AHEAD_CHUNKS; ++h) first_chunks[h] = chunk(d, h);
    for (int t = t0; t < t1; ++t) {
        const u32x4 n_units = *cnt++;
        u32x4 v[CHUNKS - AHEAD_CHUNKS < 4 ? CHUNKS - AHEAD_CHUNKS : 4];
        constexpr int BEFORE = int(sizeof(v) / sizeof(v[0]));
#pragma unroll
        for (int i = 0; i < BEFORE; ++i) v[i] = chunk(d, AHEAD_CHUNKS + i);
        __syncthreads();  // everyone is done with the tile before
#pragma unroll
        for (int h = 0; h < AHEAD_CHUNKS; ++h) put(d, h, first_chunks[h]);
#pragma unroll
        for (int i = 0; i < BEFORE; ++i) put(d, AHEAD_CHUNKS + i, v[i]);
#pragma unroll
        for (int h = AHEAD_CHUNKS + BEFORE; h < CHUNKS; h += 4) {
#pragma unroll
            for (int i = 0; i < 4; ++i)
                if (h + i < CHUNKS) v[i] = chunk(d, h + i);
#pragma unroll
            for (int i = 0; i < 4; ++i)
                if (h + i < CHUNKS) put(d, h + i, v[i]);
        }
        if (t + 1 < t1) d = a.tiles[t + 1];
        __syncthreads();
#pragma unroll
        for (int h = 0; h < AHEAD_CHUNKS; ++h) first_chunks[h] = chunk(d, h);  // behind the last tile: that one again
#pragma unroll
        for (int r = 0; r < RR; ++r) {
            int n = int((__builtin_amdgcn_readfirstlane(n_units[r >> 2]) >> (8 * (r & 3))) & 0xFFu);
            for (; n >= 2; n -= 2) step(std::integral_constant<int, 2>(), acc[r]);
            if (n) step(std::integral_constant<int, 1>(), acc[r]);
        }
    }

    float *out = a.partial + (int64_t(group) * a.n_slices + slice) * a.n_parts * (L * VEC) + c * VEC;
#pragma unroll
    for (int r = 0; r < RR; ++r) {
        const int64_t i = dealt_bundle(wv, r, a.n_waves, (a.n_parts + ROWS - 1) / ROWS) * ROWS + g;
        if (i >= 0 && i < a.n_parts) {
            float *q = out + int64_t(a.order[i]) * (L * VEC);
#pragma unroll
            for (int k = 0; k < VEC; k += 4)
                *reinterpret_cast<f32x4 *>(q + k) = f32x4{acc[r][k], acc[r][k + 1], acc[r][k + 2], acc[r][k + 3]};
        }
    }
}

// ---------------------------------------------------------------- dense cells as a bit matrix
// Where the rows with the most edges meet the sources gathered most, a tenth of all cells and more are edges, and a sum over sources is
// cheaper as a product of the matrix cores with the 0/1 matrix of the edges, a bit per cell, than as a read of LDS and an addition per edge: 32
// rows x 16 sources x 32 columns take three bf16 instructions of 32 clocks on one of four units, 24 / 512 clocks per cell, an edge 0.8
// in tile_kernel.  The columns of X are split into three bf16 numbers each, exactly, as in gemm.hip; a product with 0 or 1 is exact.
//
// 233 K vertices, 115 M edges, 57 % of them in 220 groups of 256 rows: F=602 0.9 ms at 0.95 PFLOP/s, the clock's limit under such load; tile_kernel
// 5.2 -> 3.4 ms, where copying the tiles counts for most now; the call 6.83 -> 6.1, F=256 2.66 -> 2.50.  Error of the sums against 64 bits, 2-norm, normal
// operands 8.1e-7 -> 3.2e-7, positive 4.2e-7 -> 1.2e-7, over 40 binary orders of magnitude 6.0e-7 -> 2.5e-7.
constexpr int kDenseWaves = 4;                // of 64 rows each
constexpr int kDenseRows = GNN_BIT_ROWS;      // of a group
static_assert(kDenseRows == 64 * kDenseWaves, "two tiles of 32 rows per wavefront");
constexpr int kChunkSteps = 8, kChunk = 16 * kChunkSteps;  // sources that a workgroup has in LDS at a time
// A row takes the tiles of which it has one line in so many (10 and 16: 233 K vertices, 115 M edges F=602 6.26 and 6.08 ms; 300 K, 120 M F=256
// 2.82 and 2.85; 233 K directed, 80 M 2.00 and 2.12).
constexpr int kDenseParts = 12;
// Groups are made where they take this share of the plan's edges, because every tile is still copied for the others (MEAN forward F=256, ms,
// without -> with: 233 K vertices, 115 M edges, 57 % 2.66 -> 2.50, 133 K, 79 M, 67 % 1.76 -> 1.58, 300 K, 120 M, 50 % 2.92 -> 2.82, 233 K directed,
// 80 M, 45 % 2.10 -> 2.00; below, 505 K, 60 M, 27 % 2.37 -> 2.42, 133 K mild skew, 25 % 2.10 -> 2.17).
constexpr double kDenseShare = 0.4;
constexpr int kMaxChunks = 256;
constexpr int kStepVecs = 3 * 64;             // 16-byte words of a step's split operand: three numbers, 64 lanes
constexpr int kUnitChunks = 64;               // chunks that one workgroup takes (32, 64, 128: F=41 0.70, 0.72, 0.79 ms, F=602 the same)
// Chunks of a group, where its bits begin, and the units it is cut into: the first adds to the partial lines, the others leave theirs at
// slots extra ... extra + units - 2.
struct DenseGroup { int64_t bits; int32_t chunks, units, extra, pad; };
struct DenseUnit { int32_t group, begin, end, slot; };  // slot: -1, or where the sums are left

// depth[h] = tiles from the first on of which row h has a kDenseParts-th of the lines; 0 where a source occurs twice.  A wavefront per row.
__global__ void __launch_bounds__(256) dense_depth_kernel(const TileDesc *__restrict__ tiles, int n_tiles, DenseRule rule,
                                                          const int32_t *__restrict__ blk_indices, uint32_t *__restrict__ depth_key,
                                                          uint32_t *__restrict__ ids, uint32_t *__restrict__ histogram) {
    const int lane = threadIdx.x & 63;
    const int64_t h = (int64_t(blockIdx.x) * blockDim.x + threadIdx.x) >> 6;
    if (h >= rule.n_hot) return;
    uint32_t depth = 0;
    if (rule.edges(0, h)) {
        const uint32_t lo = rule.cell_off[h], hi = rule.cell_off[h + 1];
        uint32_t b = lo;
        while (int(depth) < n_tiles) {
            const TileDesc d = tiles[depth];
            const uint32_t e = lower_bound_in(blk_indices, b, hi, d.begin + d.size);
            if (int64_t(e - b) * kDenseParts < d.size) break;
            b = e;
            ++depth;
        }
        bool twice = false;
        for (uint32_t i = lo + lane; i + 1 < b; i += 64) twice |= blk_indices[i] == blk_indices[i + 1];
        if (__any(twice)) depth = 0;
    }
    if (lane == 0) {
        depth_key[h] = uint32_t(n_tiles) - depth;
        ids[h] = uint32_t(h);
        atomicAdd(&histogram[depth], 1u);
    }
}

__device__ __forceinline__ uint32_t dense_prefix(const DenseRule &rule, const int32_t *blk_indices, uint32_t h, int32_t end) {
    return lower_bound_in(blk_indices, rule.cell_off[h], rule.cell_off[h + 1], end) - rule.cell_off[h];
}

// The rows of the groups: depth[row] = tiles of its group; what is left of its staged edges (one at least: it needs a part).
__global__ void __launch_bounds__(256) dense_assign_kernel(const TileDesc *__restrict__ tiles, DenseRule rule, const uint32_t *__restrict__ rows,
                                                           int64_t n_rows, const uint32_t *__restrict__ group_depth,
                                                           const int32_t *__restrict__ blk_indices, uint32_t *__restrict__ depth,
                                                           uint32_t *__restrict__ staged, unsigned long long *__restrict__ n_edges) {
    const int64_t i = int64_t(blockIdx.x) * blockDim.x + threadIdx.x;
    if (i >= n_rows) return;
    const uint32_t h = rows[i], t = group_depth[i / kDenseRows];
    const uint32_t n = dense_prefix(rule, blk_indices, h, tiles[t - 1].begin + tiles[t - 1].size);
    depth[h] = t;
    staged[h] = staged[h] > n ? staged[h] - n : 1u;
    atomicAdd(n_edges, static_cast<unsigned long long>(n));
}

// The bits.  Chunk c of 32 rows: 64 lanes of 8 bytes, lane = 32 * half + row; byte s of a lane's word of four steps (0 ... 3, then 4 ... 7) has the sources
// 16 * s + 8 * half + 0 ... 7 of the chunk, the even ones in bits 4 * s ... of its low half, the odd ones in the high half: where the
// pairs of bf16 numbers of an operand want them.  A wavefront per row.
__global__ void __launch_bounds__(64) dense_bits_kernel(const TileDesc *__restrict__ tiles, DenseRule rule, const uint32_t *__restrict__ rows,
                                                        const uint32_t *__restrict__ group_depth, const DenseGroup *__restrict__ groups,
                                                        const int32_t *__restrict__ blk_indices, uint32_t *__restrict__ bits) {
    __shared__ uint32_t words[kMaxChunks * 4];  // [chunk][half][steps 0 ... 3, 4 ... 7]
    const int64_t i = blockIdx.x;
    const int group = int(i / kDenseRows), in_group = int(i % kDenseRows);
    const uint32_t h = rows[i], t = group_depth[group];
    const DenseGroup g = groups[group];
    for (int w = threadIdx.x; w < g.chunks * 4; w += 64) words[w] = 0u;
    __syncthreads();
    const uint32_t lo = rule.cell_off[h], n = dense_prefix(rule, blk_indices, h, tiles[t - 1].begin + tiles[t - 1].size);
    for (uint32_t e = threadIdx.x; e < n; e += 64) {
        const int k = blk_indices[lo + e];
        const int step = (k >> 4) & 7, j = k & 7;
        atomicOr(&words[(k >> 7) * 4 + ((k >> 3) & 1) * 2 + (step >> 2)], 1u << (4 * (step & 3) + (j >> 1) + 16 * (j & 1)));
    }
    __syncthreads();
    const int64_t first = g.bits + int64_t(in_group >> 5) * g.chunks * 64;  // in 8-byte words
    for (int w = threadIdx.x; w < g.chunks * 4; w += 64) {
        const int64_t at = first + int64_t(w >> 2) * 64 + ((w >> 1) & 1) * 32 + (in_group & 31);
        bits[at * 2 + (w & 1)] = words[w];
    }
}

typedef float float16v __attribute__((ext_vector_type(16)));
typedef float float2v __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));

// The next bf16 number of each of eight values, which keep what is left.
__device__ __forceinline__ u32x4 split_off(float (&v)[8]) {
    u32x4 q;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const float2v pair = {v[2 * i], v[2 * i + 1]};
        q[i] = __builtin_bit_cast(uint32_t, __builtin_convertvector(pair, bf16x2));
        v[2 * i] -= __uint_as_float(q[i] << 16);
        v[2 * i + 1] -= __uint_as_float(q[i] & 0xFFFF0000u);
    }
    return q;
}

// A step's bits of a row (the low ones of each half of the word) as numbers +1 or -1, whose patterns c holds shifted by 0 ... 3.
__device__ __forceinline__ bf16x8 dense_ones(uint32_t word, const uint32_t (&c)[4]) {
    u32x4 m;
#pragma unroll
    for (int p = 0; p < 4; ++p) m[p] = __umul24(word & (0x00010001u << p), c[p]);
    return __builtin_bit_cast(bf16x8, m);
}

// Beyond this, values take the way of dense_kernel's last loop: split (times 2^16, so that no part of any is cut off below) they and
// their sums would overflow, and infinities and NaN would reach rows that do not gather them.
__device__ __forceinline__ bool dense_exception(float x) { return !(fabsf(x) < 0x1p90f); }

// A wavefront splits 16 sources x 32 columns of one slice; flags: the sources that have a value of the other kind.  Columns from n_cols on, and
// the rows of sources that nobody gathers, are zeros here: in the table they are whatever its memory held.
__global__ void __launch_bounds__(256) dense_split_kernel(const char *__restrict__ X, int64_t slice_stride, int64_t n_cols, int64_t n_sources,
                                                          int64_t n_steps, int n_slices, u32x4 *__restrict__ split, uint16_t *__restrict__ flags) {
    const int lane = threadIdx.x & 63;
    const int64_t w = (int64_t(blockIdx.x) * blockDim.x + threadIdx.x) >> 6;
    if (w >= n_steps * n_slices) return;
    const int64_t slice = w / n_steps, step = w - slice * n_steps;
    const float *x = reinterpret_cast<const float *>(X + slice * slice_stride) + (lane & 31);
    const int64_t k0 = step * 16 + (lane >> 5) * 8, k_end = slice * 32 + (lane & 31) < n_cols ? n_sources : 0;
    float v[8];
    uint32_t mask = 0;
#pragma unroll
    for (int j = 0; j < 8; ++j) {
        v[j] = k0 + j < k_end ? x[(k0 + j) * 32] : 0.0f;
        const bool other = dense_exception(v[j]);
        const unsigned long long m = __ballot(other);
        if (uint32_t(m)) mask |= 1u << j;
        if (uint32_t(m >> 32)) mask |= 256u << j;
        v[j] = other ? 0.0f : v[j] * 0x1p16f;
    }
#pragma unroll
    for (int s = 0; s < 3; ++s) split[w * kStepVecs + s * 64 + lane] = split_off(v);
    if (lane == 0) flags[w] = uint16_t(mask);
}

struct DenseArgs {
    const DenseGroup *groups;
    const DenseUnit *units;
    const uint32_t *rows, *part_base;
    const uint2 *bits;
    const u32x4 *split;
    const uint16_t *flags;
    const char *X;
    int64_t slice_stride, n_steps, n_parts, n_sources;
    int32_t n_slices;
    float *partial;  // of the first group of tiles
    float *extra;    // [slot][slice][row of the group][32]
};

// A workgroup takes the rows of a group and one slice of 32 columns: adds their sums to the partial lines of the rows' first parts.  A
// wavefront has 64 rows, so that an operand read from LDS serves two products.
//
// The matrix cores cut off what lies below the sum's last bit, towards minus infinity: 64 sources at a time are summed from zero,
// and every other such sum is one of negated operands (and of the other rows of a pair), subtracted.
__global__ void __launch_bounds__(64 * kDenseWaves) dense_kernel(const DenseArgs a) {
    constexpr int THREADS = 64 * kDenseWaves, COPIES = kChunkSteps * kStepVecs / THREADS;
    static_assert(kChunkSteps * kStepVecs % THREADS == 0, "whole copies");
    __shared__ u32x4 operand[2][kChunkSteps * kStepVecs];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int slice = int(blockIdx.x) % a.n_slices;
    const DenseUnit unit = a.units[blockIdx.x / uint32_t(a.n_slices)];
    const DenseGroup g = a.groups[unit.group];
    const u32x4 *src = a.split + int64_t(slice) * a.n_steps * kStepVecs + threadIdx.x;
    const uint2 *bits = a.bits + g.bits + int64_t(wave) * 2 * g.chunks * 64 + lane;
    const int64_t second = int64_t(g.chunks) * 64;  // the other 32 rows
    // +1 or -1 as a pair's first number, by the parity of row and sum
    const uint32_t one = (lane & 1) ? 0xBF80u : 0x3F80u;
    uint32_t c_even[4], c_odd[4];
#pragma unroll
    for (int p = 0; p < 4; ++p) { c_even[p] = one >> p; c_odd[p] = (one ^ 0x8000u) >> p; }

    float16v acc[2];
#pragma unroll
    for (int r = 0; r < 2; ++r)
#pragma unroll
        for (int v = 0; v < 16; ++v) acc[r][v] = 0.0f;

    u32x4 nxt[COPIES];
    uint2 b_nxt[2];
    auto fetch = [&](int c) {
#pragma unroll
        for (int i = 0; i < COPIES; ++i) nxt[i] = src[int64_t(c) * (kChunkSteps * kStepVecs) + i * THREADS];
#pragma unroll
        for (int r = 0; r < 2; ++r) b_nxt[r] = bits[r * second + int64_t(c) * 64];
    };
    auto keep = [&](int buf) {
#pragma unroll
        for (int i = 0; i < COPIES; ++i) operand[buf][i * THREADS + threadIdx.x] = nxt[i];
    };
    fetch(unit.begin);
    keep(unit.begin & 1);
    __syncthreads();
    for (int c = unit.begin; c < unit.end; ++c) {
        const uint2 b[2] = {b_nxt[0], b_nxt[1]};
        fetch(c + 1 < unit.end ? c + 1 : c);
        auto half = [&](auto odd) {
            constexpr bool ODD = decltype(odd)::value;
            float16v sum[2] = {};
#pragma unroll
            for (int s = 0; s < 4; ++s) {
                const u32x4 *q = &operand[c & 1][((ODD ? 4 : 0) + s) * kStepVecs + lane];
                bf16x8 x[3];
#pragma unroll
                for (int i = 0; i < 3; ++i) x[i] = __builtin_bit_cast(bf16x8, q[(2 - i) * 64]);  // the smallest first
#pragma unroll
                for (int r = 0; r < 2; ++r) {
                    const bf16x8 ones = dense_ones((ODD ? b[r].y : b[r].x) >> (4 * s), ODD ? c_odd : c_even);
#pragma unroll
                    for (int i = 0; i < 3; ++i) sum[r] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ones, x[i], sum[r], 0, 0, 0);
                }
            }
#pragma unroll
            for (int r = 0; r < 2; ++r)
#pragma unroll
                for (int v = 0; v < 16; ++v) acc[r][v] += ((v & 1) != int(ODD)) ? -sum[r][v] : sum[r][v];
        };
        half(std::false_type());
        half(std::true_type());
        keep((c + 1) & 1);
        __syncthreads();
    }
#pragma unroll
    for (int r = 0; r < 2; ++r)
#pragma unroll
        for (int v = 0; v < 16; ++v) acc[r][v] *= 0x1p-16f;

    // The values that were left out (see dense_exception), 64 sources at a time where they have any, as products again: the finite ones times
    // 2^-64, and one number per source that is an infinity or NaN, so that a sum counts how many of each kind a row gathers.  32 loads in
    // flight bound it (233 K vertices, 115 M edges F=602, no such value 6.07 ms, one column of infinities or of 1e30 6.22, all columns 7.9 and 7.7;
    // one source and one load after the other 6.06, 11.7, 32).
    const uint16_t *flags = a.flags + int64_t(slice) * a.n_steps;
    const float *X = reinterpret_cast<const float *>(a.X + int64_t(slice) * a.slice_stride) + (lane & 31);
    const int n_steps = unit.end * kChunkSteps;
    for (int s0 = unit.begin * kChunkSteps; s0 < n_steps; s0 += 64) {
        const uint32_t mine = s0 + lane < n_steps ? flags[s0 + lane] : 0u;
        unsigned long long steps = __ballot(mine != 0u);
        while (steps) {
            const int first = __builtin_ctzll(steps) & ~3;
            steps &= ~(0xFull << first);
            const int64_t k0 = int64_t(s0 + first) * 16 + (lane >> 5) * 8;
            float v[4][8];
#pragma unroll
            for (int s = 0; s < 4; ++s)
#pragma unroll
                for (int j = 0; j < 8; ++j) v[s][j] = k0 + s * 16 + j < a.n_sources ? X[(k0 + s * 16 + j) * 32] : 0.0f;
            const bool odd = (s0 + first) & 4;
            uint32_t word[2], c[4];
#pragma unroll
            for (int r = 0; r < 2; ++r) {
                const uint2 w = bits[r * second + int64_t((s0 + first) / kChunkSteps) * 64];
                word[r] = odd ? w.y : w.x;
            }
#pragma unroll
            for (int p = 0; p < 4; ++p) c[p] = odd ? c_odd[p] : c_even[p];
            bool any_large = false, any_special = false;
#pragma unroll
            for (int s = 0; s < 4; ++s)
#pragma unroll
                for (int j = 0; j < 8; ++j) {
                    const bool finite = fabsf(v[s][j]) <= 0x1.fffffep127f;
                    any_large |= finite && dense_exception(v[s][j]);
                    any_special |= !finite;
                }
            auto products = [&](auto parts, auto number, float16v (&sum)[2]) {
                constexpr int PARTS = decltype(parts)::value;
#pragma unroll
                for (int s = 0; s < 4; ++s) {
                    float q[8];
#pragma unroll
                    for (int j = 0; j < 8; ++j) q[j] = number(v[s][j]);
                    bf16x8 x[PARTS];
#pragma unroll
                    for (int i = PARTS - 1; i >= 0; --i) x[i] = __builtin_bit_cast(bf16x8, split_off(q));
#pragma unroll
                    for (int r = 0; r < 2; ++r) {
                        const bf16x8 ones = dense_ones(word[r] >> (4 * s), c);
#pragma unroll
                        for (int i = 0; i < PARTS; ++i) sum[r] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ones, x[i], sum[r], 0, 0, 0);
                    }
                }
            };
            if (__any(any_large)) {
                float16v sum[2] = {};
                products(std::integral_constant<int, 3>(),
                         [](float x) { return dense_exception(x) && fabsf(x) <= 0x1.fffffep127f ? x * 0x1p-64f : 0.0f; }, sum);
#pragma unroll
                for (int r = 0; r < 2; ++r)
#pragma unroll
                    for (int i = 0; i < 16; ++i) acc[r][i] += (((i & 1) != int(odd)) ? -sum[r][i] : sum[r][i]) * 0x1p64f;
            }
            if (__any(any_special)) {
                float16v sum[2] = {};  // at most 64 of each kind
                products(std::integral_constant<int, 1>(),
                         [](float x) { return x != x ? 0x1p16f : (x == INFINITY ? 1.0f : (x == -INFINITY ? 0x1p8f : 0.0f)); }, sum);
#pragma unroll
                for (int r = 0; r < 2; ++r)
#pragma unroll
                    for (int i = 0; i < 16; ++i) {
                        const uint32_t n = uint32_t(fabsf(sum[r][i]));
                        if (n & 0xFFu) acc[r][i] += INFINITY;
                        if (n >> 8 & 0xFFu) acc[r][i] -= INFINITY;
                        if (n >> 16) acc[r][i] = NAN;
                    }
            }
        }
    }

    float *out = a.partial + int64_t(slice) * a.n_parts * 32 + (lane & 31);
    const uint32_t *rows = a.rows + int64_t(unit.group) * kDenseRows + wave * 64;
    float *extra = a.extra + (int64_t(unit.slot) * a.n_slices + slice) * (kDenseRows * 32) + wave * 64 * 32 + (lane & 31);
#pragma unroll
    for (int r = 0; r < 2; ++r)
#pragma unroll
        for (int v = 0; v < 16; ++v) {
            if (unit.slot >= 0) {
                extra[(r * 32 + 8 * (v >> 2) + 4 * (lane >> 5) + (v & 3)) * 32] = acc[r][v];
                continue;
            }
            float *q = out + int64_t(a.part_base[rows[r * 32 + 8 * (v >> 2) + 4 * (lane >> 5) + (v & 3)]]) * 32;
            *q += acc[r][v];
        }
}

// Adds the other units' sums of the groups that have any, in order.
__global__ void __launch_bounds__(256) dense_add_kernel(const DenseArgs a) {
    const int slice = int(blockIdx.y), group = int(blockIdx.x) / (kDenseRows / 8);
    const DenseGroup g = a.groups[group];
    const int row = int(blockIdx.x) % (kDenseRows / 8) * 8 + int(threadIdx.x >> 5), col = threadIdx.x & 31;
    float *q = a.partial + (int64_t(slice) * a.n_parts + a.part_base[a.rows[int64_t(group) * kDenseRows + row]]) * 32 + col;
    float s = *q;
    for (int u = 0; u < g.units - 1; ++u) s += a.extra[((int64_t(g.extra + u) * a.n_slices + slice) * kDenseRows + row) * 32 + col];
    *q = s;
}

int64_t dense_steps(const gnn_tiles *t) { return int64_t(t->dense_chunks) * kChunkSteps; }
// Of a launch: sums of the groups' other units, split operand and its flags.
int64_t dense_bytes(const gnn_tiles *t, int n_slices) {
    return t->dense_groups ? n_slices * (int64_t(t->dense_extra) * kDenseRows * 128 + dense_steps(t) * (kStepVecs * 16 + 2)) : 0;
}

// What dense_bytes counts lies behind the partial lines.
hipError_t launch_dense(const gnn_tiles *t, const void *X, int64_t slice_stride, int n_slices, int64_t n_cols, int n_groups, float *partial,
                        hipStream_t stream) {
    DenseArgs a{};
    a.groups = static_cast<const DenseGroup *>(t->dense);
    a.units = reinterpret_cast<const DenseUnit *>(a.groups + t->dense_groups);
    a.rows = t->dense_rows;
    a.part_base = t->part_base;
    a.bits = t->dense_bits;
    a.extra = partial + int64_t(n_groups) * n_slices * t->n_parts * 32;
    u32x4 *split = reinterpret_cast<u32x4 *>(a.extra + int64_t(t->dense_extra) * n_slices * kDenseRows * 32);
    a.n_steps = dense_steps(t);
    uint16_t *flags = reinterpret_cast<uint16_t *>(split + a.n_steps * n_slices * kStepVecs);
    a.split = split;
    a.flags = flags;
    a.X = static_cast<const char *>(X);
    a.slice_stride = slice_stride;
    a.n_parts = t->n_parts;
    a.n_sources = t->dense_sources;
    a.n_slices = n_slices;
    a.partial = partial;
    dense_split_kernel<<<static_cast<unsigned>((a.n_steps * n_slices + 3) / 4), 256, 0, stream>>>(a.X, slice_stride, n_cols, t->dense_sources, a.n_steps,
                                                                                            n_slices, split, flags);
    dense_kernel<<<static_cast<unsigned>(t->dense_units * n_slices), 64 * kDenseWaves, 0, stream>>>(a);
    if (t->dense_cut > 0)
        dense_add_kernel<<<dim3(static_cast<unsigned>(t->dense_cut * (kDenseRows / 8)), static_cast<unsigned>(n_slices)), 256, 0, stream>>>(a);
    return hipGetLastError();
}

// number of the layout for L lanes per row
int level_of(int lanes, bool bf16) { return (lanes == 8 ? 0 : (lanes == 4 ? 1 : 2)) + (bf16 ? 3 : 0); }

}  // namespace

void gnn_tiles_free(gnn_tiles &t) {
    gnn_dev_free(t.part_base); gnn_dev_free(t.order); gnn_dev_free(t.tiles); gnn_dev_free(t.seg); gnn_dev_free(t.stream);
    gnn_dev_free(t.counts); gnn_dev_free(t.wave_off); gnn_dev_free(t.left.pieces); gnn_dev_free(t.left.piece_block);
    gnn_dev_free(t.left.rowbase); gnn_dev_free(t.bound_w); gnn_dev_free(t.tmp_w); gnn_dev_free(t.positions);
    gnn_dev_free(t.dense); gnn_dev_free(t.dense_rows); gnn_dev_free(t.dense_bits);
    for (int i = 0; i < 3; ++i) gnn_dev_free(t.scale[i]);
    t = gnn_tiles{};
}

namespace {

// Device memory that lives as long as this object.
struct Scratch {
    std::vector<void *> all;
    hipStream_t stream;
    explicit Scratch(hipStream_t s) : stream(s) {}
    ~Scratch() {
        if (!all.empty()) (void)hipStreamSynchronize(stream);
        for (void *p : all) gnn_dev_free_on(p, stream);
    }
    template <typename T>
    bool get(T **p, int64_t n) {
        if (!gnn_dev_alloc(p, n, stream)) return false;
        all.push_back(*p);
        return true;
    }
};

// Workgroups (per column slice and group of tiles) that so many bundles are dealt to: up to kRowBlocks with kFewBundles or
// more per wavefront, so that copying a tile is shared by many rows; beyond that as many as the registers ask for.
int64_t row_blocks_for(int64_t n_bundles, int rr) {
    int64_t few = n_bundles / (kTileWaves * kFewBundles);
    if (few > kRowBlocks) few = kRowBlocks;
    const int64_t least = (n_bundles + kTileWaves * rr - 1) / (kTileWaves * rr);
    return few > least ? few : (least > 0 ? least : 1);
}

// The bit matrix: rows by the number of tiles they are dense in, in groups that share it.  Takes the edges away from `staged` and
// *staged_edges; *depth: tiles that a row's lists leave out.
int build_dense(const gnn_plan *plan, const DenseRule &rule, const std::vector<TileDesc> &tiles, int n_tiles, const TileDesc *d_tiles, uint32_t *staged,
                Scratch &tmp, hipStream_t stream, gnn_tiles &B, uint32_t **depth_out, int64_t *staged_edges) {
    const int64_t n_hot = rule.n_hot;
    while (n_tiles > 0 && int64_t(tiles[size_t(n_tiles - 1)].begin) + tiles[size_t(n_tiles - 1)].size > int64_t(kMaxChunks) * kChunk) --n_tiles;
    if (n_tiles == 0 || n_hot < kDenseRows) return GNN_OK;
    uint32_t *keys[2], *ids[2], *table = nullptr, *sums = nullptr, *histogram = nullptr, *depth = nullptr;
    if (!(tmp.get(&keys[0], n_hot) && tmp.get(&keys[1], n_hot) && tmp.get(&ids[0], n_hot) && tmp.get(&ids[1], n_hot) &&
          tmp.get(&table, gnn_sort_table_elems(n_hot)) && tmp.get(&sums, gnn_sort_sums_elems(n_hot)) && tmp.get(&histogram, n_tiles + 1)))
        return GNN_ERR_ALLOC;
    GNN_HIP_TRY(hipMemsetAsync(histogram, 0, sizeof(uint32_t) * size_t(n_tiles + 1), stream));
    dense_depth_kernel<<<grid_for(n_hot * 64, 256, INT32_MAX), 256, 0, stream>>>(d_tiles, n_tiles, rule, plan->blk_indices, keys[0], ids[0], histogram);
    GNN_HIP_TRY(hipGetLastError());
    std::vector<uint32_t> rows_of_depth(size_t(n_tiles) + 1);
    GNN_HIP_TRY(hipMemcpyAsync(rows_of_depth.data(), histogram, sizeof(uint32_t) * rows_of_depth.size(), hipMemcpyDeviceToHost, stream));
    GNN_HIP_TRY(hipStreamSynchronize(stream));
    // a group is as deep as its last row
    std::vector<uint32_t> group_depth;
    std::vector<DenseGroup> groups;
    std::vector<DenseUnit> units;
    int64_t rows = 0, bits = 0;
    int extra = 0, cut = 0;
    for (int t = n_tiles; t > 0; --t) {
        rows += rows_of_depth[size_t(t)];
        const int64_t chunks = (int64_t(tiles[size_t(t - 1)].begin) + tiles[size_t(t - 1)].size + kChunk - 1) / kChunk;
        while (int64_t(groups.size() + 1) * kDenseRows <= rows) {
            const int n = int((chunks + kUnitChunks - 1) / kUnitChunks), group = int(groups.size());
            groups.push_back(DenseGroup{bits, int32_t(chunks), n, extra, 0});
            group_depth.push_back(uint32_t(t));
            bits += chunks * (kDenseRows * 2);
            for (int u = 0; u < n; ++u) units.push_back(DenseUnit{group, int32_t(chunks * u / n), int32_t(chunks * (u + 1) / n), u == 0 ? -1 : extra++});
            cut += n > 1;
        }
    }
    if (groups.empty()) return GNN_OK;
    int where = 0;
    const int rc = gnn_radix_sort_pairs(keys, ids, n_hot, gnn_ilog2_ceil(int64_t(n_tiles) + 1), table, sums, stream, &where);
    if (rc != GNN_OK) return rc;
    const int64_t n_rows = int64_t(groups.size()) * kDenseRows;
    uint32_t *d_depth = nullptr;
    unsigned long long *n_edges = nullptr, host_edges = 0;
    DenseGroup *d_groups = nullptr;
    if (!(tmp.get(&depth, n_hot) && tmp.get(&d_depth, int64_t(groups.size())) && tmp.get(&n_edges, 1))) return GNN_ERR_ALLOC;
    static_assert(sizeof(DenseGroup) % alignof(DenseUnit) == 0 && 2 * sizeof(DenseUnit) >= sizeof(DenseGroup), "units behind the groups");
    if (!gnn_dev_alloc(&d_groups, int64_t(groups.size() + units.size()), stream)) return GNN_ERR_ALLOC;
    B.dense = d_groups;
    std::stable_sort(units.begin(), units.end(), [](const DenseUnit &x, const DenseUnit &y) { return x.end - x.begin > y.end - y.begin; });  // the longest first
    GNN_HIP_TRY(hipMemcpyAsync(d_groups + groups.size(), units.data(), sizeof(DenseUnit) * units.size(), hipMemcpyHostToDevice, stream));
    if (!(gnn_dev_alloc(&B.dense_rows, n_rows, stream) && gnn_dev_alloc(&B.dense_bits, bits, stream))) return GNN_ERR_ALLOC;
    GNN_HIP_TRY(hipMemcpyAsync(d_groups, groups.data(), sizeof(DenseGroup) * groups.size(), hipMemcpyHostToDevice, stream));
    GNN_HIP_TRY(hipMemcpyAsync(d_depth, group_depth.data(), sizeof(uint32_t) * group_depth.size(), hipMemcpyHostToDevice, stream));
    GNN_HIP_TRY(hipMemcpyAsync(B.dense_rows, ids[where], sizeof(uint32_t) * size_t(n_rows), hipMemcpyDeviceToDevice, stream));
    GNN_HIP_TRY(hipMemsetAsync(depth, 0, sizeof(uint32_t) * size_t(n_hot), stream));
    GNN_HIP_TRY(hipMemsetAsync(n_edges, 0, sizeof(*n_edges), stream));
    dense_assign_kernel<<<grid_for(n_rows, 256, INT32_MAX), 256, 0, stream>>>(d_tiles, rule, B.dense_rows, n_rows, d_depth, plan->blk_indices, depth,
                                                                            staged, n_edges);
    dense_bits_kernel<<<static_cast<unsigned>(n_rows), 64, 0, stream>>>(d_tiles, rule, B.dense_rows, d_depth, d_groups, plan->blk_indices,
                                                                     reinterpret_cast<uint32_t *>(B.dense_bits));
    GNN_HIP_TRY(hipGetLastError());
    GNN_HIP_TRY(hipMemcpyAsync(&host_edges, n_edges, sizeof(host_edges), hipMemcpyDeviceToHost, stream));
    GNN_HIP_TRY(hipStreamSynchronize(stream));  // the host arrays end here
    if (double(host_edges) < kDenseShare * double(plan->n_edges)) return GNN_OK;
    B.dense_groups = int32_t(groups.size());
    B.dense_units = int32_t(units.size());
    B.dense_extra = extra;
    B.dense_cut = cut;
    B.dense_chunks = groups[0].chunks;
    // they are in order of their gathers; the last chunk may begin within a table that ends with the tiles
    const TileDesc &last = tiles[size_t(group_depth[0] - 1)];
    B.dense_sources = std::min(plan->n_rows - plan->bucket_vertices[0], int64_t(last.begin) + last.size);
    *staged_edges -= int64_t(host_edges);
    if (*staged_edges < 1) *staged_edges = 1;
    *depth_out = depth;
    return GNN_OK;
}

// Builds B (the caller frees what it holds when this fails).  B.active stays false where nothing is dense enough.
int build_tiles(const gnn_plan *plan, int lanes, int rr, bool dense, hipStream_t stream, gnn_tiles &B) {
    const int64_t n_hot = plan->blk_n_hot;
    const int n_blocks = plan->blk_n_blocks;
    const int tile_lines = tile_bytes(lanes) / (16 * lanes) - zero_lines(lanes);
    const int rows = 64 / lanes;
    (void)hipGetLastError();
    Scratch tmp(stream);

    // Which cells, and which blocks: a row is staged in a block where it has at least kMinRowEdges edges per tile, the
    // block where those rows have enough edges to pay for copying its tiles into LDS.
    auto block_range = [&](int k, int64_t *lo, int64_t *hi) {
        *lo = k == 0 ? 0 : (k == n_blocks - 1 ? int64_t(plan->blk_rest_begin) : int64_t(plan->blk_hot_lines) + int64_t(k - 1) * plan->blk_block_lines);
        *hi = k == n_blocks - 1 ? plan->n_rows : (k == 0 ? int64_t(plan->blk_hot_lines) : *lo + plan->blk_block_lines);
        if (k < n_blocks - 1 && *hi > plan->blk_rest_begin) *hi = plan->blk_rest_begin;
    };
    std::vector<int64_t> n_block_tiles(size_t(n_blocks), 0);
    std::vector<uint32_t> block_min(size_t(n_blocks), 0);
    for (int k = 0; k < n_blocks; ++k) {
        int64_t lo, hi;
        block_range(k, &lo, &hi);
        if (k == n_blocks - 1 && plan->blk_last_in_place) hi = lo;
        n_block_tiles[size_t(k)] = hi > lo ? (hi - lo + tile_lines - 1) / tile_lines : 0;
        block_min[size_t(k)] = uint32_t(n_block_tiles[size_t(k)] * kMinRowEdges);
    }
    uint32_t *d_min = nullptr;
    unsigned long long *d_sums = nullptr;
    std::vector<unsigned long long> sums_of_block(size_t(n_blocks), 0);
    if (!tmp.get(&d_min, n_blocks) || !tmp.get(&d_sums, n_blocks + 1)) return GNN_ERR_ALLOC;
    const DenseRule rule{plan->blk_cell_off, d_min, n_hot};
    GNN_HIP_TRY(hipMemcpyAsync(d_min, block_min.data(), sizeof(uint32_t) * size_t(n_blocks), hipMemcpyHostToDevice, stream));
    GNN_HIP_TRY(hipMemsetAsync(d_sums, 0, sizeof(unsigned long long) * size_t(n_blocks + 1), stream));
    tile_block_edges_kernel<<<dim3(static_cast<unsigned>(grid_for(n_hot, 256, 64)), static_cast<unsigned>(n_blocks)), 256, 0, stream>>>(rule, d_sums);
    GNN_HIP_TRY(hipGetLastError());
    GNN_HIP_TRY(hipMemcpyAsync(sums_of_block.data(), d_sums, sizeof(unsigned long long) * size_t(n_blocks), hipMemcpyDeviceToHost, stream));
    GNN_HIP_TRY(hipStreamSynchronize(stream));
    std::vector<TileDesc> tiles;
    int64_t staged_edges = 0;
    const int64_t est_row_blocks = row_blocks_for((n_hot + rows - 1) / rows, rr);
    for (int k = 0; k < n_blocks; ++k) {
        const int64_t nt = n_block_tiles[size_t(k)];
        if (nt == 0 || int64_t(sums_of_block[size_t(k)]) < kMinTileEdges * est_row_blocks * nt || int64_t(tiles.size()) + nt > 4096) { block_min[size_t(k)] = 0; continue; }
        int64_t lo, hi;
        block_range(k, &lo, &hi);
        for (int64_t i = 0; i < nt; ++i) {  // tiles of equal size
            const int64_t b = lo + (hi - lo) * i / nt, e = lo + (hi - lo) * (i + 1) / nt;
            tiles.push_back(TileDesc{int32_t(b), int32_t(e - b), k, 0});
        }
        staged_edges += int64_t(sums_of_block[size_t(k)]);
    }
    const int n_tiles = int(tiles.size());
    if (n_tiles == 0) return GNN_OK;

    // the rows' staged edges, and their parts
    uint32_t *staged = nullptr, *part_base = nullptr, *scan = nullptr, *n_staged = reinterpret_cast<uint32_t *>(d_sums + n_blocks);
    const int64_t n_cells = int64_t(n_blocks) * n_hot;
    if (!tmp.get(&staged, n_hot) || !tmp.get(&scan, gnn_scan_sums_elems(n_cells > n_hot + 1 ? n_cells : n_hot + 1))) return GNN_ERR_ALLOC;
    if (!gnn_dev_alloc(&B.part_base, n_hot + 1, stream)) return GNN_ERR_ALLOC;
    part_base = B.part_base;
    GNN_HIP_TRY(hipMemcpyAsync(d_min, block_min.data(), sizeof(uint32_t) * size_t(n_blocks), hipMemcpyHostToDevice, stream));
    const int row_grid = grid_for(n_hot, 256, INT32_MAX);
    tile_row_edges_kernel<<<row_grid, 256, 0, stream>>>(rule, n_blocks, staged, n_staged);
    uint32_t host_staged = 0, parts_last = 0, base_last = 0;
    GNN_HIP_TRY(hipGetLastError());
    GNN_HIP_TRY(hipMemcpyAsync(&host_staged, n_staged, 4, hipMemcpyDeviceToHost, stream));
    GNN_HIP_TRY(hipStreamSynchronize(stream));
    if (host_staged == 0) return GNN_OK;
    uint32_t *longest = nullptr, *depth = nullptr;
    TileDesc *d_tiles = nullptr;
    if (!tmp.get(&longest, n_hot) || !gnn_dev_alloc(&d_tiles, n_tiles, stream)) return GNN_ERR_ALLOC;
    B.tiles = d_tiles;
    GNN_HIP_TRY(hipMemcpyAsync(d_tiles, tiles.data(), sizeof(TileDesc) * size_t(n_tiles), hipMemcpyHostToDevice, stream));
    if (dense) {
        if (tiles[0].block == 0) {
            const int rc_dense = build_dense(plan, rule, tiles, int(n_block_tiles[0]), d_tiles, staged, tmp, stream, B, &depth, &staged_edges);
            if (rc_dense != GNN_OK) return rc_dense;
        }
        if (!B.dense_groups) return GNN_OK;  // the layout for all calls serves these too
    }
    const uint32_t cap = uint32_t((2 * staged_edges + host_staged - 1) / host_staged);  // twice the mean row
    GNN_HIP_TRY(hipMemsetAsync(longest, 0, sizeof(uint32_t) * size_t(n_hot), stream));
    tile_longest_kernel<<<grid_for(int64_t(n_tiles) * n_hot, 256), 256, 0, stream>>>(d_tiles, n_tiles, rule, plan->blk_indices, depth, longest);
    tile_row_parts_kernel<<<row_grid, 256, 0, stream>>>(staged, longest, n_hot, cap, part_base);
    GNN_HIP_TRY(hipGetLastError());
    GNN_HIP_TRY(hipMemcpyAsync(&parts_last, part_base + n_hot - 1, 4, hipMemcpyDeviceToHost, stream));
    int rc = gnn_scan_exclusive_u32(part_base, n_hot, scan, stream);
    if (rc != GNN_OK) return rc;
    GNN_HIP_TRY(hipMemcpyAsync(&base_last, part_base + n_hot - 1, 4, hipMemcpyDeviceToHost, stream));
    GNN_HIP_TRY(hipStreamSynchronize(stream));
    const uint32_t n_parts32 = base_last + parts_last;
    const int64_t n_parts = n_parts32;
    GNN_HIP_TRY(hipMemcpyAsync(part_base + n_hot, &n_parts32, 4, hipMemcpyHostToDevice, stream));

    // bundles of parts of similar size, dealt to the wavefronts
    const int64_t n_bundles = (n_parts + rows - 1) / rows;
    int64_t n_row_blocks = row_blocks_for(n_bundles, rr);
    // Few rows: down to a bundle per wavefront where that fills compute units that would be idle (a launch has as many
    // groups of tiles as that asks for, and several slices of whole lines), while a tile is worth copying that often.
    // No more groups than the fullest tile, that of the most-gathered sources, leaves something to do for.
    double fullest = 0.0, all = 0.0;
    for (const TileDesc &t : tiles) {
        const double share = gnn_plan_top_share(plan, int64_t(t.begin) + t.size) - gnn_plan_top_share(plan, t.begin);
        all += share;
        if (share > fullest) fullest = share;
    }
    int64_t groups = fullest > 0.0 ? int64_t(all / fullest) : 1;
    if (groups > n_tiles) groups = n_tiles;
    if (groups > GNN_TILE_MAX_GROUPS) groups = GNN_TILE_MAX_GROUPS;
    if (groups < 1) groups = 1;
    int64_t fill = kComputeUnits / (groups * (lanes == 8 ? 4 : 1));
    if (fill > n_bundles / kTileWaves) fill = n_bundles / kTileWaves;
    if (fill > staged_edges / (n_tiles * kMinTileEdges)) fill = staged_edges / (n_tiles * kMinTileEdges);
    if (n_row_blocks < fill) n_row_blocks = fill;
    const int64_t n_waves = n_row_blocks * kTileWaves, n_wt = n_waves * n_tiles;
    uint32_t *keys[2], *ids[2], *table = nullptr, *sums = nullptr;
    RowPart *parts = nullptr;
    const int64_t sums_n = gnn_sort_sums_elems(n_parts) > gnn_scan_sums_elems(n_wt) ? gnn_sort_sums_elems(n_parts) : gnn_scan_sums_elems(n_wt);
    uint2 *seg = nullptr;
    if (!(tmp.get(&keys[0], n_parts) && tmp.get(&keys[1], n_parts) && tmp.get(&ids[0], n_parts) && tmp.get(&ids[1], n_parts) &&
          tmp.get(&table, gnn_sort_table_elems(n_parts)) && tmp.get(&sums, sums_n) && tmp.get(&parts, n_parts)))
        return GNN_ERR_ALLOC;
    if (!gnn_dev_alloc(&seg, int64_t(n_tiles) * n_parts, stream)) return GNN_ERR_ALLOC;
    B.seg = seg;
    if (!(gnn_dev_alloc(&B.order, n_parts, stream) && gnn_dev_alloc(&B.counts, n_wt * kCounts, stream) && gnn_dev_alloc(&B.wave_off, n_wt, stream))) return GNN_ERR_ALLOC;
    tile_parts_kernel<<<row_grid, 256, 0, stream>>>(staged, part_base, n_hot, parts, keys[0], ids[0]);
    GNN_HIP_TRY(hipGetLastError());
    int where = 0;
    rc = gnn_radix_sort_pairs(keys, ids, n_parts, gnn_ilog2_ceil(int64_t(cap) + 1), table, sums, stream, &where);
    if (rc != GNN_OK) return rc;
    GNN_HIP_TRY(hipMemcpyAsync(B.order, ids[where], sizeof(uint32_t) * size_t(n_parts), hipMemcpyDeviceToDevice, stream));
    tile_segments_kernel<<<grid_for(int64_t(n_tiles) * n_parts, 256), 256, 0, stream>>>(d_tiles, n_tiles, rule, B.order, parts, n_parts,
                                                                                    plan->blk_indices, depth, seg);
    tile_counts_kernel<<<grid_for(n_wt, 256), 256, 0, stream>>>(seg, n_parts, n_tiles, n_waves, rr, rows, B.counts, B.wave_off);
    GNN_HIP_TRY(hipGetLastError());
    std::vector<uint32_t> iters(static_cast<size_t>(n_wt));
    GNN_HIP_TRY(hipMemcpyAsync(iters.data(), B.wave_off, sizeof(uint32_t) * size_t(n_wt), hipMemcpyDeviceToHost, stream));
    GNN_HIP_TRY(hipStreamSynchronize(stream));
    int64_t total = 0;
    B.tile_work.assign(size_t(n_tiles), 0);
    for (int64_t x = 0; x < n_wt; ++x) {
        total += iters[size_t(x)];
        B.tile_work[size_t(x % n_tiles)] += iters[size_t(x)];
    }
    if (total >= int64_t(UINT32_MAX)) return GNN_OK;  // keep the pieces
    int64_t most_work = 1;
    for (int64_t x : B.tile_work) most_work = x > most_work ? x : most_work;
    B.max_groups = int32_t(2 * total / most_work);  // groups are whole tiles: of twice as many none is much longer than that tile
    if ((rc = gnn_scan_exclusive_u32(B.wave_off, n_wt, sums, stream)) != GNN_OK) return rc;
    if (!gnn_dev_alloc(&B.stream, (total + kStreamAhead) * rows * kUnit, stream)) return GNN_ERR_ALLOC;
    auto fill_stream = [&](auto lanes_of_a_row) {
        tile_fill_kernel<decltype(lanes_of_a_row)::value, kFillIndices><<<grid_for(n_wt * 64, 256), 256, 0, stream>>>(
            d_tiles, n_tiles, n_waves, rr, seg, n_parts, B.counts, B.wave_off, plan->blk_indices, nullptr, nullptr, nullptr, tile_lines, B.stream, nullptr,
            nullptr);
    };
    if (lanes == 8) fill_stream(std::integral_constant<int, 8>());
    else if (lanes == 4) fill_stream(std::integral_constant<int, 4>());
    else fill_stream(std::integral_constant<int, 2>());
    GNN_HIP_TRY(hipGetLastError());

    // the cells that are not staged stay pieces
    uint32_t *cell_count = nullptr, *cell_pieces = nullptr;
    if (!tmp.get(&cell_count, n_cells) || !tmp.get(&cell_pieces, n_cells)) return GNN_ERR_ALLOC;
    tile_left_cells_kernel<<<grid_for(n_cells, 256), 256, 0, stream>>>(rule, n_blocks, uint32_t(plan->blk_max_piece), cell_count, cell_pieces);
    GNN_HIP_TRY(hipGetLastError());
    rc = gnn_build_pieces(n_hot, n_blocks, plan->blk_max_piece, cell_count, plan->blk_cell_off, cell_pieces, scan,
                          plan->blk_piece_block != nullptr, stream, &B.left);
    if (rc != GNN_OK) return rc;
    B.lanes = lanes;
    B.rr = rr;
    B.n_tiles = n_tiles;
    B.n_row_blocks = n_row_blocks;
    B.n_waves = n_waves;
    B.n_iters = total;
    B.n_parts = n_parts;
    B.active = true;
    return GNN_OK;
}

// There was no room for the bit matrix: it is asked for again by the calls 1, 2, 4, 8, ... later, because asking costs the sort and two waits.
bool worth_another_try(gnn_tiles &L) {
    const bool now = (L.refused & (L.refused - 1)) == 0;
    if (!now) ++L.refused;
    return now;
}

}  // namespace

// Builds the tile layout for rows of `lanes` x 16 bytes on first use; needs the source-blocked layout.
int gnn_plan_tiles(gnn_plan *plan, int lanes, bool bf16, bool plain, int64_t n_slices, hipStream_t stream, const gnn_tiles **out) {
    *out = nullptr;
    if (!plan || (lanes != 8 && lanes != 4 && lanes != 2)) return GNN_ERR_INVALID_ARG;
    const bool either = plain && lanes == 8 && !bf16, dense = either && gnn_bits_pay(n_slices);
    gnn_tiles &L = plan->tiles[dense ? GNN_TILES_PLAIN : level_of(lanes, bf16)];
    auto lists = [&] { return gnn_plan_tiles(plan, lanes, bf16, false, n_slices, stream, out); };  // they serve these calls as well
    if (dense && !gnn_capturing(stream) && !worth_another_try(L)) return lists();
    if (!L.decided) {
        if (!plan->blk_decided) return GNN_ERR_INVALID_ARG;
        if (either && gnn_capturing(stream)) {
            const gnn_tiles &other = plan->tiles[dense ? level_of(lanes, bf16) : GNN_TILES_PLAIN];
            if (other.active) {
                *out = &other;
                return GNN_OK;
            }
            if (dense) return lists();
        }
        gnn_tiles B{};
        if (plan->blk_n_pieces > 0 && plan->blk_cell_off) {
            int rc;
            try {
                rc = build_tiles(plan, lanes, bf16 ? kBundlesBf16 : kBundlesF32, dense, stream, B);
            } catch (const std::bad_alloc &) {  // of its host arrays: no exception leaves the library
                rc = GNN_ERR_ALLOC;
            }
            if (rc != GNN_OK || !B.active) gnn_tiles_free(B);
            if (dense && rc == GNN_ERR_ALLOC) {
                ++L.refused;
                return lists();
            }
            if (rc != GNN_OK) return rc;
        }
        L = std::move(B);
        L.decided = true;
    }
    if (dense && !L.active) return lists();
    if (L.active) *out = &L;
    return GNN_OK;
}

namespace {

int64_t stream_slots(const gnn_tiles &L) { return L.n_iters * (64 / L.lanes) * kUnit; }

int coef_room(const gnn_tiles &L, float **slot, hipStream_t stream) {
    if (*slot) return GNN_OK;
    (void)hipGetLastError();
    return gnn_dev_alloc(slot, stream_slots(L) + int64_t(kStreamAhead) * (64 / L.lanes) * kUnit, stream) ? GNN_OK : GNN_ERR_ALLOC;
}

hipError_t fill(const gnn_plan *plan, const gnn_tiles &L, const float *w, const float *scale, float *wstream, uint32_t *positions,
                hipStream_t stream) {
    auto launch = [&](auto lanes_of_a_row, auto what) {
        tile_fill_kernel<decltype(lanes_of_a_row)::value, decltype(what)::value><<<grid_for(L.n_waves * L.n_tiles * 64, 256), 256, 0, stream>>>(
            static_cast<const TileDesc *>(L.tiles), L.n_tiles, L.n_waves, L.rr, static_cast<const uint2 *>(L.seg), L.n_parts, L.counts, L.wave_off,
            plan->blk_indices, plan->blk_epos, w, scale, 0, nullptr, wstream, positions);
    };
    auto launch_for = [&](auto what) {
        if (L.lanes == 8) launch(std::integral_constant<int, 8>(), what);
        else if (L.lanes == 4) launch(std::integral_constant<int, 4>(), what);
        else launch(std::integral_constant<int, 2>(), what);
    };
    if (positions) launch_for(std::integral_constant<TileFill, kFillPositions>());
    else launch_for(std::integral_constant<TileFill, kFillCoefs>());
    return hipGetLastError();
}

// The edge of every slot, for coefficients that are filled in again and again, because working out the order of the slots takes
// longer than reading the weights (233 K vertices, F=64: weights of every call's own 3.7 -> 1.9 ms a call, bound anew before
// each call, for two widths 11.2 -> 3.1).  4 bytes a slot, as much as the coefficients.  Under capture, and where there is no
// room for it (asked for once: the driver waits for the device to find out), they are filled in as the first time.
void want_positions(const gnn_plan *plan, gnn_tiles &L, hipStream_t stream) {
    hipStreamCaptureStatus capture = hipStreamCaptureStatusNone;
    if (L.positions || L.no_positions) return;
    if (hipStreamIsCapturing(stream, &capture) != hipSuccess || capture != hipStreamCaptureStatusNone) {
        (void)hipGetLastError();
        return;
    }
    (void)hipGetLastError();
    if (!gnn_dev_alloc(&L.positions, stream_slots(L), stream)) {
        (void)hipGetLastError();
        L.positions = nullptr;
        L.no_positions = true;
    } else if (fill(plan, L, nullptr, nullptr, nullptr, L.positions, stream) != hipSuccess) {
        gnn_dev_free(L.positions);
        L.positions = nullptr;
    }
}

}  // namespace

int gnn_plan_tile_coef_room(gnn_plan *plan, const gnn_tiles *tiles, hipStream_t stream) {
    gnn_tiles &L = plan->tiles[tiles - plan->tiles];
    const int rc = coef_room(L, &L.tmp_w, stream);
    if (rc == GNN_OK) want_positions(plan, L, stream);
    return rc;
}

// Coefficients of the edges in stream order.  Kept: the plan's own factors, and weights bound to the plan; anything
// else is gathered anew by every call.
int gnn_plan_tile_coefs(gnn_plan *plan, const gnn_tiles *tiles_in, const float *w, const float *scale, int scale_mode, bool bound,
                        hipStream_t stream, const float **out) {
    gnn_tiles &L = plan->tiles[tiles_in - plan->tiles];
    float **slot = &L.tmp_w;
    bool need = true;
    if (!w && scale) {
        slot = &L.scale[scale_mode - 1];
        need = !*slot;
    } else if (w && !scale && bound) {
        slot = &L.bound_w;
        need = !*slot || L.bound_version != plan->bound_w_version;
    }
    const bool again = slot == &L.tmp_w || (slot == &L.bound_w && *slot);
    const int rc = coef_room(L, slot, stream);
    if (rc != GNN_OK) return rc;
    if (need) {
        if (again) want_positions(plan, L, stream);
        hipError_t e;
        if (again && L.positions) {
            const int64_t n = stream_slots(L) / 4;
            tile_refill_kernel<<<grid_for(n, 256), 256, 0, stream>>>(reinterpret_cast<const uint4 *>(L.positions), n, w, scale,
                                                                     reinterpret_cast<float4 *>(*slot));
            e = hipGetLastError();
        } else {
            e = fill(plan, L, w, scale, *slot, nullptr, stream);
        }
        if (e != hipSuccess) {
            if (slot != &L.tmp_w && slot != &L.bound_w) {  // an unfilled array must not serve a later call
                gnn_dev_free(*slot);
                *slot = nullptr;
            }
            return GNN_ERR_LAUNCH;
        }
        if (slot == &L.bound_w) L.bound_version = plan->bound_w_version;
    }
    *out = *slot;
    return GNN_OK;
}

// How many groups the tiles are split into: as many as make one round of the compute units (a workgroup takes a whole
// one).  A second, mostly empty round costs more than idle compute units, which the short rows' launch uses meanwhile
// (505 K vertices, 14 M edges, F=99: 0.75 ms with 184 workgroups, 0.83 with 276, 0.78 as pieces).  Nor more than the
// tile with the most work, which no group is shorter than, leaves work for.
int gnn_tile_groups(const gnn_tiles *t, int n_slices) {
    int64_t g = kComputeUnits / (t->n_row_blocks * n_slices);
    if (g > GNN_TILE_MAX_GROUPS) g = GNN_TILE_MAX_GROUPS;
    if (g > t->max_groups) g = t->max_groups;
    if (g > t->n_tiles) g = t->n_tiles;
    return g < 1 ? 1 : int(g);
}

static int64_t tile_partial_bytes(const gnn_tiles *t, int n_slices, int line_floats) {
    return int64_t(gnn_tile_groups(t, n_slices)) * n_slices * t->n_parts * line_floats * int64_t(sizeof(float)) + dense_bytes(t, n_slices);
}

int gnn_plan_tiles_with_room(gnn_plan *plan, int lanes, bool bf16, bool plain, int n_slices, int line_floats, hipStream_t stream, const gnn_tiles **out) {
    int rc = gnn_plan_tiles(plan, lanes, bf16, plain, n_slices, stream, out);
    if (rc != GNN_OK || !*out) return rc;
    const int64_t need = tile_partial_bytes(*out, n_slices, line_floats);
    if (!(*out)->dense_groups) return gnn_plan_room(plan, plan->tile_partial, need, stream);
    // The split operand and the sums of the bit matrix take many times what the lists take.  Where that is refused, or would have to be
    // asked for in a capture while the lists have theirs, the lists serve the call.
    gnn_tiles &bits = plan->tiles[GNN_TILES_PLAIN];
    const gnn_tiles &lists = plan->tiles[level_of(lanes, bf16)];
    if (need > plan->tile_partial.bytes && lists.active && tile_partial_bytes(&lists, n_slices, line_floats) <= plan->tile_partial.bytes &&
        gnn_capturing(stream)) {
        *out = &lists;
        return gnn_plan_room(plan, plan->tile_partial, 0, stream);
    }
    rc = gnn_plan_room(plan, plan->tile_partial, need, stream);
    if (rc != GNN_ERR_ALLOC) {
        bits.refused = 0;
        return rc;
    }
    ++bits.refused;
    (void)hipGetLastError();
    rc = gnn_plan_tiles(plan, lanes, bf16, false, n_slices, stream, out);
    if (rc != GNN_OK || !*out) return rc;
    return gnn_plan_room(plan, plan->tile_partial, tile_partial_bytes(*out, n_slices, line_floats), stream);
}

int gnn_launch_tiles(const gnn_tiles *t, bool bf16, const void *X, int64_t slice_stride_bytes, int n_slices, int64_t n_cols,
                     const float *coefs, float *partial, hipStream_t stream) {
    TileArgs a{};
    a.tiles = static_cast<const TileDesc *>(t->tiles);
    a.n_tiles = t->n_tiles;
    a.n_slices = n_slices;
    a.n_groups = gnn_tile_groups(t, n_slices);
    // group boundaries: equal shares of the iterations
    double total = 0.0;
    for (int64_t x : t->tile_work) total += double(x);
    double run = 0.0;
    int next = 1;
    a.group_begin[0] = 0;
    for (int i = 0; i < t->n_tiles && next < a.n_groups; ++i) {
        run += double(t->tile_work[size_t(i)]);
        // every group gets at least one tile
        if (run >= total * next / a.n_groups || t->n_tiles - (i + 1) <= a.n_groups - next) a.group_begin[next++] = i + 1;
    }
    a.group_begin[a.n_groups] = t->n_tiles;
    a.n_waves = t->n_waves;
    a.n_parts = t->n_parts;
    a.stream = t->stream;
    a.wstream = coefs;
    a.wave_off = t->wave_off;
    a.counts = t->counts;
    a.order = t->order;
    a.X = X;
    a.slice_stride = slice_stride_bytes;
    a.partial = partial;
    const int64_t blocks = t->n_row_blocks * n_slices * a.n_groups;
    if (blocks > INT32_MAX) return GNN_ERR_UNSUPPORTED;
    const dim3 grid(static_cast<unsigned>(blocks));
#define GNN_TILE_LAUNCH(BF, LANES)                                                                              \
    do {                                                                                                        \
        if (coefs) tile_kernel<BF, LANES, true, BF ? kBundlesBf16 : kBundlesF32><<<grid, kTileThreads, 0, stream>>>(a);             \
        else tile_kernel<BF, LANES, false, BF ? kBundlesBf16 : kBundlesF32><<<grid, kTileThreads, 0, stream>>>(a);                  \
    } while (0)
    if (bf16) {
        if (t->lanes == 8) GNN_TILE_LAUNCH(true, 8);
        else if (t->lanes == 4) GNN_TILE_LAUNCH(true, 4);
        else GNN_TILE_LAUNCH(true, 2);
    } else {
        if (t->lanes == 8) GNN_TILE_LAUNCH(false, 8);
        else if (t->lanes == 4) GNN_TILE_LAUNCH(false, 4);
        else GNN_TILE_LAUNCH(false, 2);
    }
#undef GNN_TILE_LAUNCH
    if (t->dense_groups && launch_dense(t, X, slice_stride_bytes, n_slices, n_cols, a.n_groups, partial, stream) != hipSuccess) return GNN_ERR_LAUNCH;
    return hipGetLastError() == hipSuccess ? GNN_OK : GNN_ERR_LAUNCH;
}

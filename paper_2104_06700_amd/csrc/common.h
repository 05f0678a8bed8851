// Internal declarations shared by the translation units of libgnnagg.so.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include <vector>

#include "gnnagg.h"

#define GNN_HIP_TRY(expr)                                  \
    do {                                                   \
        hipError_t gnn_err_ = (expr);                      \
        if (gnn_err_ != hipSuccess) return GNN_ERR_LAUNCH; \
    } while (0)

#define GNN_MAX_BINS (GNN_MAX_THRESHOLDS + 1)

// Source tiles in LDS (tiles.hip): the edges of the long rows into the source blocks where they are dense, as one
// stream per wavefront of the gather, and the piece list of the rest.  One layout per line width (lanes of 16 bytes
// per row); built on first use.
constexpr int GNN_TILE_MAX_GROUPS = 32;
struct gnn_piece_list {
    int32_t *pieces = nullptr;        // [n_pieces * 4] (begin, length, partial slot, row)
    uint16_t *piece_block = nullptr;  // [n_pieces]
    uint32_t *rowbase = nullptr;      // [n_hot + 1] first partial slot of every row
    int64_t n_pieces = 0;
};
struct gnn_tiles {
    bool decided = false, active = false;
    int32_t lanes = 0, rr = 0, n_tiles = 0;  // rr: bundles of rows a wavefront owns at most
    int64_t n_row_blocks = 0, n_waves = 0, n_iters = 0;
    int64_t n_parts = 0;                 // rows, long ones cut into parts: each has a partial line per launch and group
    uint32_t *part_base = nullptr;       // [n_hot + 1] first part of every row
    uint32_t *order = nullptr;           // [n_parts] parts by size
    void *tiles = nullptr;               // [n_tiles] (first rank, ranks, block)
    void *seg = nullptr;                 // [n_tiles][n_parts] edge range of the part at a position of `order`
    uint16_t *stream = nullptr;
    uint8_t *counts = nullptr;           // [n_waves][n_tiles][16]
    uint32_t *wave_off = nullptr;        // [n_waves][n_tiles]
    std::vector<int64_t> tile_work;      // iterations per tile (host)
    int32_t max_groups = 1;              // groups of tiles that can share the work evenly
    gnn_piece_list left;                 // the cells that are not staged
    float *scale[3] = {nullptr, nullptr, nullptr};  // the plan's per-edge factors in stream order
    float *bound_w = nullptr;            // bound edge weights in stream order, as of binding number bound_version
    int64_t bound_version = -1;
    float *tmp_w = nullptr;              // other coefficients, refilled by every call
    uint32_t *positions = nullptr;       // CSR position of the edge in every slot of the stream; made for coefficients that are refilled
    bool no_positions = false;           // there was no room for them
    // Rows whose edges to the first sources are a bit matrix (dense_kernel); their lists leave those edges out.
    int32_t dense_groups = 0, dense_chunks = 0;  // groups of rows; chunks of sources of the longest one
    int32_t dense_units = 0, dense_extra = 0, dense_cut = 0;  // what the groups are cut into, units beyond their first; groups that have some
    int64_t dense_sources = 0;                   // rows of the gathered table that are gathered
    void *dense = nullptr;                       // the groups and their units
    uint32_t *dense_rows = nullptr;              // hot row of every row of the groups
    uint2 *dense_bits = nullptr;
    uint32_t refused = 0;                        // calls since there was no room for it, with that one; 0: there was
};
constexpr int GNN_TILES_PLAIN = 6;  // number in gnn_plan::tiles of the layout with a bit matrix
constexpr int GNN_BIT_ROWS = 256;   // rows of a group of it

// Device memory of a plan that grows with what calls ask of it (gnn_plan_room).  recorded: a captured call has used it, so a graph may hold
// its address.
struct gnn_grown {
    void *p = nullptr;
    int64_t bytes = 0;
    bool recorded = false;
};

// One plan = one graph orientation.  All pointers are device memory owned by
// the plan unless marked host.
struct gnn_plan {
    int64_t n_rows = 0;
    int64_t n_edges = 0;
    int32_t n_bins = 0;
    int32_t indptr_is_64 = 0;
    gnn_plan_params params{};
    int64_t bin_offsets[GNN_MAX_BINS + 1] = {0};  // host copy
    int64_t bin_edges[GNN_MAX_BINS] = {0};        // edges of the rows of each bin (host)
    int32_t *row_perm = nullptr;      // [n_rows]
    // The row at every position of row_perm, the first of its edges, their number (and nothing): one load in the place of two
    // that wait for each other.  E <= INT32_MAX, else nullptr; row_perm lies behind it in the same block.
    int4 *row_info = nullptr;
    int32_t *col_counts = nullptr;    // [n_rows] occurrences of each vertex in indices
    bool rows_unordered = false;      // of a graph of long rows (gnn_long_rows): the sources of its rows are in no order
    // hub rows = rows of the last bin when params.hub_chunk > 0
    int64_t n_hub_rows = 0;
    int64_t n_chunks = 0;
    int64_t *chunks = nullptr;        // [n_chunks * 3] (row, e_begin, e_end)
    int64_t *hub_chunk_offsets = nullptr;  // [n_hub_rows + 1] first piece of each hub row
    uint32_t *hub_done = nullptr;          // behind the pieces: [8 * first piece of a hub row + column slice] pieces that are done (gnn_hub_done)
    gnn_grown scratch;                // hub partial sums
    std::vector<void *> retired;      // outgrown memory that a graph may still use, until the plan goes
    const void *indptr_seen = nullptr;  // the indptr the plan was built from (sanity check only)
    // per-edge factor of the gathered vertex, streamed by the hot kernels:
    // [0] 1/max(c,1)   [1] 1/sqrt(max(c,1))   [2] 1/(c+1), c = col_counts[indices[e]]; built on first use
    float *edge_scale[3] = {nullptr, nullptr, nullptr};
    // Histogram of the column counts in 256 roughly logarithmic buckets (host copies): how many
    // vertices fall in each bucket and how many edges they are gathered by.  It answers "which
    // share of the gathers goes to the K most-gathered vertices", the quantity that decides
    // whether XCD column slices can keep more useful rows in L2.
    int64_t bucket_vertices[256] = {0};
    int64_t bucket_edges[256] = {0};
    gnn_grown padded;                 // copy of the gathered matrix with rows padded to whole 128-byte lines
    // copy of `indices` in which bit 31 marks the rarely gathered ("cold") sources; built on first
    // use when the plan's graph is in the regime where non-temporal loads of cold rows pay
    int32_t *cold_indices = nullptr;
    int32_t cold_decided = 0;    // 0: not yet; 1: decided (cold_indices is null when it does not pay)
    int32_t cold_threshold = 0;  // sources gathered fewer times than this are cold
    int32_t cold_forced = 0;     // the copy was built under GNN_FLAG_FORCE_COLD_HINTS (a call without it rebuilds)
    int32_t rank_forced = 0;     // likewise for rank_indices
    bool cold_recorded = false, rank_recorded = false;  // as in gnn_grown
    // Rank layout of the padded copy: rank[v] = position of v by descending column count; the copy
    // stores row v at row rank[v] and the kernels gather through rank_indices[e] =
    // rank[indices[e]] (bit 31: cold).  Built on first use.
    int32_t *rank = nullptr;
    int32_t *rank_indices = nullptr;
    // ... and in PLAN ORDER: the edge list of the row at position i of row_perm occupies
    // rank_indices[p_indptr[i] .. p_indptr[i+1]), so the rows a workgroup processes side by side read
    // one contiguous stretch of the index stream.  p_chunks: the hub pieces in those coordinates,
    // (row, begin, end, original position minus plan-order position) each.
    int64_t *p_indptr = nullptr;
    int64_t *p_chunks = nullptr;
    // a caller's scalar edge operand brought into CSR order (gnn_plan_edge_operand); refilled per call
    float *edge_operand = nullptr;
    // Source-blocked layout of the long rows (see gnn_plan_blocked); built on first use.
    gnn_blocking_params blocking{};   // requested parameters (zeros: automatic)
    int32_t blk_decided = 0;          // 0: not yet; 1: decided (blk_n_pieces == 0 when it does not apply)
    bool blk_last_in_place = false;   // blocks for hot tables: the last one is of rows that have no table, so nothing of it goes into tiles
    int32_t blk_first_bin = 0;        // rows of bins >= this are processed as pieces
    int64_t blk_hot_begin = 0;        // their range in row_perm is [blk_hot_begin, n_rows)
    int64_t blk_n_hot = 0;
    int64_t blk_n_edges = 0;          // edges of those rows
    int64_t blk_n_pieces = 0;
    int32_t blk_n_blocks = 0;
    int32_t *blk_indices = nullptr;   // [blk_n_edges] source ranks, block-major piece order
    uint32_t *blk_epos = nullptr;     // [blk_n_edges] CSR position of each (the caller's per-edge streams are read there)
    // blk_indices again as 16-bit offsets from the first rank of each edge's block, for the kernel to
    // read in place of the 32-bit ranks in all blocks but the last (whose range is not bounded); null
    // when a block spans more than 65,536 ranks.  blk_piece_block[p] = block of piece p.
    uint16_t *blk_idx16 = nullptr;
    uint16_t *blk_piece_block = nullptr;
    int32_t blk_hot_lines = 0, blk_block_lines = 0, blk_rest_begin = 0, blk_max_piece = 0;
    uint32_t *blk_cell_off = nullptr; // [blk_n_blocks * blk_n_hot + 1] first edge of every (block, hot row)
    int32_t *blk_pieces = nullptr;    // [blk_n_pieces * 4] (begin, length, partial slot, row index in the hot range)
    uint32_t *blk_rowbase = nullptr;  // [blk_n_hot + 1] first partial slot of each hot row
    float *blk_edge_scale[3] = {nullptr, nullptr, nullptr};  // edge_scale[m] at blk_epos, i.e. in the order of blk_indices
    // Edge weights the caller declared static (gnn_plan_bind_edge_weights): the pointer they were bound
    // under and their copy in the order of blk_indices, which the pieces of calls that pass that pointer
    // stream instead of reading the caller's array at blk_epos.
    const float *bound_w = nullptr;
    float *blk_bound_w = nullptr;
    bool bound_w_stale = false;       // the copy is older than the last binding
    int64_t bound_w_version = 0;      // number of the last binding
    // Hot tables (gnn_plan_hot): the vertices of the ranks below blk_rest_begin, and the vertices (not ranks) of the last block's
    // edges, whose first is edge blk_cold_begin of blk_indices.
    int32_t *blk_hot_vertices = nullptr;
    int32_t *blk_cold_vertices = nullptr;
    int64_t blk_cold_begin = 0;
    bool hot_lacks_room = false;      // gnn_plan_lacks_room
    uint64_t hot_ready[2][5][5] = {}; // what calls can use: [type][factor 0 ... 3 or weights], bit `lines`
    gnn_grown blk_partial;            // fp32 partial sums of one launch: [slices][blk_n_pieces][floats per line]
    gnn_tiles tiles[7];               // for lines of 128, 64 and 32 bytes of fp32, then of bf16; [GNN_TILES_PLAIN]: see gnn_plan_tiles
    gnn_grown tile_partial;           // their partial lines: [groups][slices][hot rows][floats per line]
};

// Makes `b` at least `bytes` large, for a call on `stream` (allocation on growth; the old contents are lost).  What a graph may hold the
// address of is kept beside it and freed with the plan: a replay writes there whatever other calls have asked for meanwhile.
int gnn_plan_room(gnn_plan *plan, gnn_grown &b, int64_t bytes, hipStream_t stream);
void gnn_plan_drop(gnn_plan *plan, void *p, bool recorded);  // frees p, or keeps it so

// Source blocking (the GPU reading of Section 4.2's blocks of source vertices, applied to the long
// rows only).  Rows of at least `min_degree` edges are cut into pieces along blocks of source RANK
// (block 0 = the `hot_lines` most-gathered sources, then blocks of `block_lines`, then one block for
// the sources gathered fewer than `rest_min_count` times), and the pieces are processed block by
// block: all rows that gather from a block do so within a short time, so a source row is fetched
// into an L2 once per block instead of once per gather.  Pieces write fp32 partial rows that a
// second kernel adds in a fixed order.
struct gnn_blocked_layout {
    bool active;
    bool automatic;          // the plan chose to block by itself (no gnn_plan_set_blocking with a degree)
    int32_t first_bin;       // bins >= this are served by pieces
    int64_t hot_begin, n_hot, n_pieces;
    const int32_t *indices;  // block-major
    const uint32_t *epos;
    // 16-bit form of `indices` (null: none): piece p lies in block k = piece_block[p], which begins at
    // rank 0 (k = 0) or hot_lines + (k - 1) * block_lines; the last block keeps the 32-bit ranks
    const uint16_t *idx16;
    const uint16_t *piece_block;
    int32_t n_blocks, hot_lines, block_lines;
    const int32_t *pieces;
    const uint32_t *rowbase;
};
// Builds the layout on first use (allocation; needs the rank layout) and reports it.  Inactive when
// the graph or the plan's thresholds do not suit it.
// for_hot_tables: where it is built now, it is for those (gnn_plan::blk_last_in_place), else for tables of all rows.
int gnn_plan_blocked(gnn_plan *plan, const void *indptr, hipStream_t stream, gnn_blocked_layout *out, bool for_hot_tables = false);
// Hot tables, for graphs of few edges per vertex: the copy has the sources of the blocks only, the most-gathered ones, and everything else is
// gathered where it lies: the pieces of the last block by vertex, the short rows by the kernels that serve rows in place.
struct gnn_hot_layout {
    gnn_blocked_layout blocks;
    int64_t rows;                  // of a table: sources of the blocks
    const int32_t *vertices;       // [rows] the vertex of every rank
    const int32_t *cold_vertices;  // of the edges from cold_begin on
    int64_t cold_begin;
};
int gnn_plan_hot(gnn_plan *plan, const void *indptr, const int32_t *indices, hipStream_t stream, gnn_hot_layout *out);
// Makes plan->blk_partial large enough, for a call on `stream`, for `slices` column slices of `line_floats` floats per piece.
int gnn_plan_blocked_partial(gnn_plan *plan, int slices, int line_floats, hipStream_t stream);
// The plan's per-edge factor stream `mode` (gnn_plan_edge_scale, which must have been built) in the order
// of the block-major index array; built on first use (allocation).
int gnn_plan_blocked_edge_scale(gnn_plan *plan, int mode, hipStream_t stream, const float **out);
// The bound edge weights in piece order: refreshed on `stream` when a binding is newer than the copy
// (allocates on first use).  Needs the layout and a binding.
int gnn_plan_blocked_bound_weights(gnn_plan *plan, hipStream_t stream, const float **out);

// The tile layout for lines of lanes * 16 bytes (null: the graph has no block dense enough); needs the blocked layout.
// plain: for sums without coefficients; those of gnn_bits_pay(slices) take the densest cells as a bit matrix where there are enough of them.
// Under three slices a launch of that is too small for the chip (233 K vertices, 115 M edges F=32 0.41 -> 0.44 ms, 133 K, 79 M F=64 0.47 -> 0.50;
// above, F=100 1.31 -> 1.26, 300 K, 120 M F=128 1.46 -> 1.42).
static inline bool gnn_bits_pay(int64_t n_slices) { return n_slices >= 3; }
// Nothing is built in a capture: a sum without coefficients takes the other layout there, if that one is at hand and its own is not.  Where there is no room for
// the bit matrix it takes the lists.
int gnn_plan_tiles(gnn_plan *plan, int lanes, bool bf16, bool plain, int64_t n_slices, hipStream_t stream, const gnn_tiles **out);
void gnn_tiles_free(gnn_tiles &t);
// Coefficients w[e] * scale[e] (either may be null; CSR order) in stream order.
int gnn_plan_tile_coefs(gnn_plan *plan, const gnn_tiles *tiles, const float *w, const float *scale, int scale_mode, bool bound,
                        hipStream_t stream, const float **out);
// Room for coefficients that every call fills anew: those of FREE weights, and products of weights and factors.
int gnn_plan_tile_coef_room(gnn_plan *plan, const gnn_tiles *tiles, hipStream_t stream);
// Groups a launch over n_slices column slices splits the tiles into, each with a partial line of its own per row.
int gnn_tile_groups(const gnn_tiles *t, int n_slices);
// gnn_plan_tiles, and plan->tile_partial large enough for such a launch.
int gnn_plan_tiles_with_room(gnn_plan *plan, int lanes, bool bf16, bool plain, int n_slices, int line_floats, hipStream_t stream, const gnn_tiles **out);
int gnn_build_pieces(int64_t n_hot, int n_blocks, int64_t max_piece, const uint32_t *cell_count, const uint32_t *edge_off,
                     uint32_t *cell_pieces, uint32_t *sums, bool want_block, hipStream_t stream, gnn_piece_list *out);
// n_cols: columns of all slices that hold data.
int gnn_launch_tiles(const gnn_tiles *t, bool bf16, const void *X, int64_t slice_stride_bytes, int n_slices, int64_t n_cols,
                     const float *coefs, float *partial, hipStream_t stream);

// Device memory that is kept for the next plan (pool.hip).  With a stream: for memory that is first used there; fails on a
// stream that is being captured.  gnn_dev_free: any stream may still use the block (as with hipFree, but without waiting);
// gnn_dev_free_on: its last use is ordered on that stream.
// Blocks of more than GNN_POOL_MAX_BLOCK bytes are not kept: they come from the driver and go back to it, which waits for the
// device, so the scratch of an asynchronous call is cut into blocks that are no larger.
constexpr int64_t GNN_POOL_MAX_BLOCK = int64_t(512) << 20;
bool gnn_capturing(hipStream_t stream);
int gnn_dev_alloc_bytes(void **p, size_t bytes, hipStream_t stream);
int gnn_dev_alloc_bytes(void **p, size_t bytes);
void gnn_dev_free(void *p);
void gnn_dev_free_on(void *p, hipStream_t stream);
void gnn_pool_release();
template <typename T>
static inline bool gnn_dev_alloc(T **p, int64_t n, hipStream_t stream) {
    void *q = nullptr;
    const bool ok = gnn_dev_alloc_bytes(&q, sizeof(T) * size_t(n > 0 ? n : 1), stream) == GNN_OK;
    *p = static_cast<T *>(q);
    return ok;
}
template <typename T>
static inline bool gnn_dev_alloc(T **p, int64_t n) {
    void *q = nullptr;
    const bool ok = gnn_dev_alloc_bytes(&q, sizeof(T) * size_t(n > 0 ? n : 1)) == GNN_OK;
    *p = static_cast<T *>(q);
    return ok;
}
// Scratch of one call: given back when it goes out of scope, for use after what the call launched on its stream.
template <typename T>
struct gnn_dev_ptr {
    T *p = nullptr;
    hipStream_t stream = nullptr;
    bool alloc_on(int64_t n, hipStream_t s) { stream = s; return gnn_dev_alloc(&p, n, s); }
    gnn_dev_ptr() = default;
    gnn_dev_ptr(const gnn_dev_ptr &) = delete;
    gnn_dev_ptr &operator=(const gnn_dev_ptr &) = delete;
    ~gnn_dev_ptr() { if (p) gnn_dev_free_on(p, stream); }
};
// Pinned host memory that kernels write small results to.
constexpr int GNN_HOST_BLOCK_BYTES = 8192;
void *gnn_host_block();
void gnn_host_block_free(void *p);

// Stable LSD radix sort of 32-bit (key, value) pairs on the low `bits` bits (graph.hip).  buf_k[0] / buf_v[0] hold the
// input; the result is in buf_k[*out] / buf_v[*out].  table / sums: scratch of gnn_sort_table_elems(n) and
// gnn_sort_sums_elems(n) words.
int gnn_radix_sort_pairs(uint32_t *buf_k[2], uint32_t *buf_v[2], int64_t n, int bits, uint32_t *table, uint32_t *sums,
                         hipStream_t stream, int *out);
int64_t gnn_sort_table_elems(int64_t n);
int64_t gnn_sort_sums_elems(int64_t n);
// Vertex gradient of max / min by sorting instead of global atomics (winners.hip): does it apply, and the call.  Writes all of
// `out`; GNN_ERR_ALLOC (nothing launched): no workspace, or the stream is being captured.
bool gnn_winners_apply(int64_t n_edges, int64_t n_out, int64_t N, int64_t d);
int gnn_scatter_winners(const int32_t *indices, const int64_t *eid, const int32_t *arg, const float *dO, int64_t ldo, const float *fE,
                        int64_t lde, bool ewide, float *out, int64_t ldv, int64_t n_out, int64_t N, int64_t d, int binop,
                        hipStream_t stream);
// In-place exclusive prefix sums; sums: scratch of gnn_scan_sums_elems(n) elements per array.  The 64-bit form scans n_arrays
// arrays `stride` elements apart and writes each one's total behind it.
int gnn_scan_exclusive_u32(uint32_t *data, int64_t n, uint32_t *sums, hipStream_t stream);
int gnn_scan_exclusive_i64(int64_t *data, int64_t n, int n_arrays, int64_t stride, int64_t *sums, hipStream_t stream);
int64_t gnn_scan_sums_elems(int64_t n);

// The 256 buckets over the count axis that a plan's histogram uses (plan.hip: count_bucket): counts below 16 one
// bucket each, then 8 buckets per octave.  Host-side twins for code that turns a count threshold into a rank.
static inline int gnn_count_bucket_of(int64_t c) {
    if (c < 16) return c < 0 ? 0 : int(c);
    int o = 0;
    while ((c >> (o + 1)) > 0) ++o;
    const int b = 16 + (o - 4) * 8 + int((c >> (o - 3)) & 7);
    return b > 255 ? 255 : b;
}
static inline int64_t gnn_count_bucket_lower_bound(int b) {
    if (b < 16) return b;
    const int o = 4 + (b - 16) / 8, m = (b - 16) % 8;
    return int64_t(8 + m) << (o - 3);
}

// Row stride (floats) of the hub partial-sum scratch for width F: whole 32-byte groups, so that
// vector stores of a last, partial strip stay inside the row.
static inline int64_t gnn_partial_ld(int64_t F) { return (F + 7) / 8 * 8; }

// Share of all gathers that goes to the K most-gathered vertices (from the bucket histogram;
// the boundary bucket is taken pro rata).
double gnn_plan_top_share(const gnn_plan *plan, int64_t K);

// Layout decisions shared by the hot calls and gnn_plan_prepare (which must reserve exactly what
// a later call will use).
struct gnn_layout {
    bool slices_wanted;   // spread column slices over the XCDs
    bool padded_copy;     // gather from a plan-owned copy with rows of an odd number of lines
    int64_t ld_pad;       // row stride of that copy in elements
    // Dense tail: when the last line of a row would hold at most 64 bytes, those columns go into a
    // table of their own with rows of 16-byte groups, packed back to back, so that an L2 line holds
    // the tail of several rows (F = 100 fp32: 3 whole lines per row + a 16-byte tail, 8 rows per
    // line) and the copy's rows are whole lines with nothing wasted.
    int64_t tail_elems;   // columns of the tail table (0: none); the main part has F - tail_elems
    int64_t tail_ld;      // its row stride in elements
    // Slice-major: the main part is stored as one table per 128-byte column slice (line k of every
    // row, rows back to back), because a launch's slice k is only ever read by the XCDs that serve
    // it: their page and DRAM-row footprint shrinks to that table, and no row padding is needed to
    // spread the L2 channels.
    bool slice_major;
    int64_t table_stride; // elements between two slice tables (N * elements per line)
    int64_t main_lines;   // number of slice tables
    // Lanes of 16 bytes per line of the tables that the long rows can be gathered from as source-blocked pieces: 8 of a
    // slice-major copy, 8, 4 or 2 of a copy whose rows are one line of 128, 64 or 32 bytes (one table), else 0.
    int32_t line_lanes;
    int64_t bytes;        // size of the whole copy for N rows
    // No copy of the whole matrix: rows are gathered in place, except by the long rows from the most-gathered sources, of which there are
    // slice tables (gnn_plan_hot_ready; lines, line_lanes).
    bool hot_tables;
    int64_t lines;        // of 128 bytes that hold a row
};

// Will calls with this plan serve their long rows as source-blocked pieces (gnn_plan_blocked)?  Known
// once the layout is built; before that, the gate of the automatic choice evaluated on the plan's host
// figures (an explicit gnn_plan_set_blocking counts as yes).
// Does a plan block by itself?  The long rows must hold a good part of the edges (else there is little to win).  The gathered table must
// dwarf an L2, or there are enough edges to pay for the launches that pieces and tiles take: it is the L2s' line rate that bounds a gather
// that hits, too (MEAN forward, ms, without -> with: 100 K vertices, 60 M edges F=602 6.50 -> 2.80, 256 2.67 -> 1.24, 64 0.78 -> 0.36, 16 0.35 -> 0.18;
// 100 K, 20 M 2.31 -> 1.61, 0.95 -> 0.63, 0.26 -> 0.18, 0.10 the same; 60 K, 24 M F=256 1.04 -> 0.57, F=32 0.13 the same; below, 60 K, 9 M F=256 0.41 ->
// 0.36, but F=100 0.20 -> 0.27; 40 K, 10 M F=256 0.47 -> 0.35, F=100 0.21 -> 0.24).
static inline bool gnn_blocks_by_itself(const gnn_plan *plan, int64_t long_edges) {
    return (plan->n_rows >= 4 * int64_t(32768) || (plan->n_rows >= 32768 && plan->n_edges >= 16000000)) && long_edges * 4 >= plan->n_edges;
}
static inline int64_t gnn_edges_from_bin(const gnn_plan *plan, int first_bin) {
    int64_t edges = 0;
    for (int b = first_bin; b < plan->n_bins; ++b) edges += plan->bin_edges[b];
    return edges;
}
// Graphs of fewer edges per vertex than a copy of the whole matrix pays for.  Blocked by themselves they have hot tables (gnn_plan_hot), unless a call
// over a copy that the caller keeps or asks for has made the plan's blocks.
static inline bool gnn_few_edges(const gnn_plan *plan) { return plan->blocking.min_degree == 0 && plan->n_edges < 16 * plan->n_rows; }
// Blocks whose edges have 16-bit indices, all but the last: by them the kernel over hot tables tells the last block's pieces, which gather by vertex.
constexpr int64_t GNN_NARROW_BLOCK = 65536;
static inline bool gnn_narrow_blocks(const gnn_plan *plan) { return plan->blocking.hot_lines <= GNN_NARROW_BLOCK && plan->blocking.block_lines <= GNN_NARROW_BLOCK; }
static inline bool gnn_plan_blocks_expected(const gnn_plan *plan, int esz, int64_t row_bytes, bool weights) {
    if (!plan || plan->n_edges <= 0 || plan->n_edges >= int64_t(INT32_MAX)) return false;
    const bool automatic = plan->blocking.min_degree == 0;
    // bf16 pieces write partial lines twice as large as the lines they gather: on graphs of a few L2s' worth of vertices
    // that eats the gain (233 K vertices, F=256 backward 3.95 -> 4.07 ms; 133 K vertices, F=128 1.16 -> 1.25), on the
    // 2.45 M-vertex graph it does not (F=512 12.9 -> 11.6).  Short rows and many edges pay there, too: a gather from tiles in LDS is not bound by lines
    // (MEAN forward and backward, ms a call: 233 K vertices, 115 M edges F=64 0.91 -> 0.82, 32 0.82 -> 0.44, 16 0.76 -> 0.42; 100 K, 60 M 0.45 ->
    // 0.42, 0.41 -> 0.29, 0.38 -> 0.30; 133 K, 40 M F=64 0.330 -> 0.342, 32 0.30 -> 0.27, 16 0.28 -> 0.19; 80 K, 30 M F=32 0.22 -> 0.18; 133 K, 28 M 0.202 ->
    // 0.220).  Not with weights, whose products with a factor every call makes anew.
    if (esz == 2 && automatic && plan->n_rows < 8 * int64_t(32768) &&
        (weights || row_bytes > 128 || plan->n_edges < (row_bytes <= 64 ? 30000000 : 60000000)))
        return false;
    if (plan->blk_decided) return plan->blk_n_pieces > 0;
    if (plan->blocking.min_degree < 0) return false;
    const int64_t min_degree = automatic ? 256 : plan->blocking.min_degree;
    int first_bin = -1;
    for (int i = 0; i < plan->params.n_thresholds; ++i)
        if (plan->params.thresholds[i] == min_degree) first_bin = i + 1;
    if (first_bin < 0 || plan->n_rows - plan->bin_offsets[first_bin] <= 0) return false;
    const int64_t long_edges = gnn_edges_from_bin(plan, first_bin);
    if (long_edges <= 0) return false;
    return !automatic || gnn_blocks_by_itself(plan, long_edges);
}
// Are there gathers enough for hot tables?  They save lines that come from behind the L2s, and cost the launches of pieces and tiles, so the edges in
// rows of 256 and more count, and the bytes these gather.  Rows off line boundaries are aligned in the tables; bf16 rows have partial lines of
// twice their size.  MEAN, in place -> hot tables, us, power-law graphs by those edges: fp32 19.5 M F=32 461 -> 417, 64 895 -> 777, 100 2316 -> 1760, 256 4506 ->
// 3506; 13.1 M F=32 332 -> 330, 36 718 -> 663, 64 633 -> 597; 6.5 M F=32 160 -> 169, 64 315 -> 316, 100 824 -> 724, 256 1628 -> 1397; 3.1 M F=100 360 -> 338, 200 738
// -> 677, 256 674 -> 648; 2.3 M F=200 (1.9 GB) 1.06 times as long, 252 and 300 (2.3 and 2.8 GB) 0.96 and 0.92 times; 2.4 M F=384 (3.7 GB) 1.07 times, 512 (5.0)
// 0.95; 2.1 M F=200 1.07 times, 500 1.13, 512 1.18; 1.9 M F=200 322 -> 362, 604 914 -> 1074; 0.9 M F=604 441 -> 569; bf16 19.5 M F=48 801 -> 720, 64 449 -> 456, 128
// 1029 -> 880; 13.1 M F=128 702 -> 674; 6.5 M F=128 363 -> 371, 200 814 -> 751; 4.5 M F=400 (3.6 GB) the same; 3.7 M F=264 and 400 (2.0 and 3.0 GB) 1.04 and 1.06
// times, 520 (3.9) 0.92; 3.3 M F=400 (2.6) 1.21 times, 520 (3.4) 0.93; 2.4 M F=400 1.31 times, 520 (2.5) 1.00, 1024 (5.0) 0.88; 243 M (27.8 M vertices) F=128 15.1 ->
// 12.8 ms forward, 15.1 -> 13.5 backward.
static inline bool gnn_hot_tables_pay(const gnn_plan *plan, int64_t row_bytes, int esz, bool lines_ok) {
    int first_bin = -1;
    for (int i = 0; i < plan->params.n_thresholds; ++i)
        if (plan->params.thresholds[i] == 256) first_bin = i + 1;
    if (first_bin < 0) return false;
    const int64_t edges = gnn_edges_from_bin(plan, first_bin);
    if (edges < 2300000) return false;
    double least;
    if (!lines_ok) least = esz == 4 ? (edges < 3000000 ? 2.3e9 : 1.2e9) : (edges < 4400000 ? 3.3e9 : 1.8e9);
    else least = esz == 4 && row_bytes <= 128 ? 2.0e9 : (edges < 3000000 ? 4.5e9 : 3.2e9);
    return double(edges) * double(row_bytes) >= least;
}

// The edge weights of a call.  BOUND: the array of gnn_plan_bind_edge_weights; FREE: any other.
enum gnn_weight_kind { GNN_WEIGHTS_NONE = 0, GNN_WEIGHTS_BOUND = 1, GNN_WEIGHTS_FREE = 2 };
static inline gnn_weight_kind gnn_weight_kind_of(const gnn_plan *plan, const float *w) {
    return !w ? GNN_WEIGHTS_NONE : (plan && w == plan->bound_w ? GNN_WEIGHTS_BOUND : GNN_WEIGHTS_FREE);
}
// Will a call with such weights serve its long rows as pieces?  FREE weights sit in CSR order, the pieces in rank order, so
// every edge would cost a random 4-byte read (1.44 -> 3.67 ms on the weighted workload at F=64): such calls keep the path
// without pieces unless the plan's blocking was asked for explicitly.
static inline bool gnn_call_blocks_expected(const gnn_plan *plan, int esz, int64_t F, gnn_weight_kind weights) {
    return plan && gnn_plan_blocks_expected(plan, esz, F * esz, weights != GNN_WEIGHTS_NONE) && (weights != GNN_WEIGHTS_FREE || plan->blocking.min_degree > 0);
}

static inline gnn_layout gnn_choose_layout(const gnn_plan *plan, int64_t N, int64_t F, int esz, int64_t ldx,
                                           bool base_line_aligned, int flags, int max_slices, bool allow_tail = false,
                                           bool scaled_source = false, bool blocks_expected = false, bool weights = false) {
    gnn_layout L{};
    const int64_t line_elems = 128 / esz;
    const int64_t lines = (F + line_elems - 1) / line_elems;
    const int64_t row_bytes = F * esz;
    // Do column slices pay?  Unsliced, an XCD's 4 MB L2 holds whole rows (32768 / lines of them);
    // sliced, one line each of 32768 rows.  Slicing is used when that wins at least 8 points of
    // the gathers (a power-law graph of a few million vertices: +20..30 points; a 111 M-vertex
    // graph with 2-line rows: ~+2 points, where the extra index reads and the loss of burst
    // locality cost more than the hits bring: 76.2 ms sliced, 74.1 ms without slices).  Matrices that fit the
    // L2s together are sliced for the sake of more, shorter wavefronts (24,490 vertices, 1.2 M edges, F=100:
    // 0.095 ms in one launch of whole rows, 0.045 in four slices).
    L.slices_wanted = !(flags & GNN_FLAG_NO_COLUMN_SLICES);
    if (L.slices_wanted && plan && plan->n_edges > 0 && max_slices == 0) {
        const double gain = gnn_plan_top_share(plan, 32768) - gnn_plan_top_share(plan, 32768 / (lines > 0 ? lines : 1));
        L.slices_wanted = gain >= 0.08 || N * row_bytes < (int64_t(32) << 20);
    }
    // The plan-owned copy: slice tables in rank order (see slice_major below), fp32 factors of the gathered rows
    // multiplied in, the long rows as source-blocked pieces where the graph has them.  It costs a pass over N rows
    // and the gather of whole lines (F = 100: 512 bytes per edge for 400), and it buys hits in the L2s: it pays once
    // the gather is large against that, at 16 edges per vertex and so many gathered bytes (measured on power-law
    // graphs of 2,500 to 1,000,000 vertices, 6 to 200 edges each, against in_place_slices() of aggregate.hip):
    //   rows off line boundaries  2 GB with pieces, 5 GB without (400 K vertices, 30 edges each, F=50 283 us in place, 257
    //                             copied; 140 K, 57, F=50 131 / 145; without pieces 100 K vertices, F=250: 25 edges
    //                             199 / 225, 50 349 / 337)
    //   line-aligned rows         8 GB, 4 GB from 48 edges per vertex on (300 K vertices, 25 edges, F=256 547 / 595; 400 K,
    //                             60, F=64 422 / 347), without pieces 16 GB
    //   rows of one line          1.28 GB of lines (245 K vertices, F=20: 25 edges 77 / 81, 50 124 / 118)
    // Coefficients make the call in place dearer (every slice reads them): about half of that, if there are some.
    const bool lines_ok = (ldx % line_elems == 0) && base_line_aligned;
    const bool even_stride = lines_ok && (ldx / line_elems) % 2 == 0;
    const bool big = N * row_bytes >= (int64_t(32) << 20);  // well beyond the L2s: the layout decides the hit rate
    const bool folds_factor = scaled_source && esz == 4;
    const bool coef = scaled_source || weights;
    const bool dense = plan && plan->n_edges >= 48 * N;
    double least_gb = lines_ok ? (blocks_expected ? (dense ? (coef ? 3.0 : 4.0) : (coef ? 5.0 : 8.0)) : (coef ? 8.0 : 16.0))
                               : (blocks_expected ? (coef ? 1.7 : 2.0) : (coef ? 1.7 : 5.0));
    if (lines == 1) least_gb = coef ? 0.7 : 1.28;
    const bool pays = plan && plan->n_edges >= 16 * N && double(plan->n_edges) * double(lines == 1 ? 128 : row_bytes) >= least_gb * 1e9;
    // An even number of lines per row crowds the L2 channels when slices are gathered in place (F=256, 8 slices: 15.4 ms
    // with 8-line rows, 12.5 ms with 9-line rows), so such rows are copied where slices are wanted: >= 16 edges per vertex
    // for rows of >= 512 bytes, >= 128 for shorter ones.
    bool worth_it = row_bytes > 128 && pays &&
                    (!lines_ok || folds_factor ||
                     (L.slices_wanted && ((even_stride && plan->n_edges >= (row_bytes >= 512 ? 16 : 128) * N) ||
                                          (blocks_expected && allow_tail && lines <= 256))));
    // pieces that were asked for need the slice tables
    if (blocks_expected && plan && plan->blocking.min_degree > 0 && row_bytes > 128 && big && L.slices_wanted && allow_tail && lines <= 256)
        worth_it = true;
    // Rows of at most one line are copied into rows of the next power of two bytes (16 ... 128), in
    // rank order: no row straddles two lines, the most-gathered rows share lines (up to 8 per
    // line).  Worth it when rows would straddle in place (F = 24: 96-byte rows) or carry a factor that the
    // copy folds in, for large matrices when they are at most 64 bytes (rank order packs the hot rows), and where the
    // long rows are served as pieces, which needs it (233 K vertices, 490 edges each, F=16 730 -> 320 us).  A plan that blocks
    // by itself does so for 24 M edges and rows of 32 bytes, 28 M and 64, 32 M and 128 (200 K vertices, F=7: 20 M edges 115
    // us without pieces, 129 with, 40 M 196 / 155; 400 K vertices, F=16: 24 M 154 / 163, 45 M 267 / 218; F=32: 24 M 180 /
    // 195, 45 M 319 / 290): below, the launches that pieces and tiles take weigh more than what they save.
    int64_t narrow_bytes = 16;
    while (narrow_bytes < row_bytes) narrow_bytes *= 2;
    bool narrow_pieces = false;
    if (lines == 1) {
        const int64_t stride_bytes = ldx * esz;
        const bool in_place_ok = base_line_aligned && stride_bytes <= 128 && (stride_bytes & (stride_bytes - 1)) == 0;
        narrow_pieces = blocks_expected && row_bytes > 16 &&
                        (plan->blocking.min_degree > 0 || plan->n_edges >= (narrow_bytes == 32 ? 24000000 : (narrow_bytes == 64 ? 28000000 : 32000000)));
        worth_it = pays && (!in_place_ok || folds_factor || (row_bytes <= 64 && big) || narrow_pieces);
    }
    L.padded_copy = plan && !(flags & GNN_FLAG_NO_PADDED_COPY) && (worth_it || (flags & GNN_FLAG_FORCE_PADDED_COPY));
    L.ld_pad = lines == 1 ? narrow_bytes / esz : (lines | 1) * line_elems;
    L.tail_elems = 0;
    L.tail_ld = 0;
    const int64_t rest = F % line_elems;
    // A dense table for a short last line saves its padding and packs eight rows' tails into a line, but it
    // is a launch of its own over all rows; where the long rows are source-blocked pieces the last line
    // does better as one more slice of whole lines, which the pieces serve like the others (2.45 M
    // vertices: F=100 4.84 -> 4.74 ms, F=112 5.08 -> 4.55; 233 K vertices F=100 2.63 -> 2.44).  Packed
    // copies kept by a caller never have the tail table (GNN_FLAG_NO_DENSE_TAIL): their size must not depend
    // on the plan.
    // ... nor do small matrices: a launch more costs them more than the padding.
    const bool dense_tail = allow_tail && !blocks_expected && !(flags & GNN_FLAG_NO_DENSE_TAIL) && (big || (flags & GNN_FLAG_FORCE_PADDED_COPY));
    if (dense_tail && L.padded_copy && L.slices_wanted && lines >= 2 && lines <= 256 && rest > 0 && rest * esz <= 64) {
        const int64_t group = 16 / esz;
        L.tail_elems = rest;
        L.tail_ld = (rest + group - 1) / group * group;
        L.ld_pad = ((lines - 1) | 1) * line_elems;
    }
    L.main_lines = L.tail_elems > 0 ? lines - 1 : lines;
    L.lines = lines;
    L.slice_major = allow_tail && L.padded_copy && L.slices_wanted && lines >= 2 && lines <= 256 &&
                    !(flags & GNN_FLAG_NO_SLICE_TABLES);
    L.table_stride = 0;
    if (L.slice_major) {
        L.ld_pad = line_elems;
        L.table_stride = N * line_elems;
        L.bytes = N * (L.main_lines * line_elems + L.tail_ld) * esz;
    } else {
        L.bytes = N * (L.ld_pad + L.tail_ld) * esz;
    }
    L.line_lanes = L.slice_major ? 8 : 0;
    if (allow_tail && L.padded_copy && narrow_pieces && !(flags & GNN_FLAG_NO_SLICE_TABLES)) L.line_lanes = int32_t(narrow_bytes / 16);
    // Rows of whole strips of 16 bytes, because those that are gathered in place end with the row; factors or weights, not the products of both,
    // which every call would make anew.
    constexpr int kStay = GNN_FLAG_NO_PADDED_COPY | GNN_FLAG_FORCE_PADDED_COPY | GNN_FLAG_NO_COLUMN_SLICES | GNN_FLAG_NO_SLICE_TABLES |
                          GNN_FLAG_NO_RANK_ORDER | GNN_FLAG_FORCE_COLD_HINTS;
    L.hot_tables = plan && blocks_expected && gnn_few_edges(plan) && gnn_narrow_blocks(plan) && !L.padded_copy && allow_tail && max_slices == 0 && !(flags & kStay) &&
                   row_bytes > 64 && row_bytes % 16 == 0 && lines <= 256 && !(scaled_source && weights) && gnn_hot_tables_pay(plan, row_bytes, esz, lines_ok);
    if (L.hot_tables) L.line_lanes = 8;
    return L;
}

// Makes plan->padded at least `bytes` large (allocation on growth).
int gnn_plan_padded(gnn_plan *plan, int64_t bytes, hipStream_t stream);

// The plan's index copy with cold sources flagged in bit 31, or nullptr when cold hints do not pay
// for this graph (see plan.hip).  force: build it whatever the graph (tests).  Builds on first use
// (allocation).
int gnn_plan_cold_indices(gnn_plan *plan, const int32_t *indices, bool force, hipStream_t stream, const int32_t **out);

// Rank layout (see gnn_plan): the vertex ranks and the rank-mapped, cold-flagged index copy.
// force_cold: flag the sources outside the warmest quarter whatever the graph (tests).
struct gnn_rank_layout {
    const int32_t *rank;       // [N]
    const int32_t *indices;    // [E] rank-mapped, cold-flagged, in plan order
    const int64_t *p_indptr;   // [N+1]
    const int64_t *p_chunks;   // [n_chunks * 4]
    bool cold_pays;            // the graph is in the regime where non-temporal loads of cold rows pay
};
int gnn_plan_rank_indices(gnn_plan *plan, const void *indptr, const int32_t *indices, bool force_cold, hipStream_t stream,
                          gnn_rank_layout *out);

// E = indptr[N]; synchronous.
int gnn_read_edge_count(const void *indptr, int64_t N, int indptr_is_64, hipStream_t stream, int64_t *E);
// rank[v] = position of vertex v by descending count, ties by ascending id; no count exceeds max_count (graph.hip).
int gnn_rank_by_count(const int32_t *counts, int64_t N, int64_t max_count, int32_t *rank, hipStream_t stream);
// Graphs whose edge dot products may be split over the XCDs (gnn_ap_bwd_edge); their plans look at the order of the sources, which is a launch of a
// few microseconds, so smaller graphs, whose plans may serve a call or two, are left out (plans and transposed graph of 4,000 vertices, 0.8 M
// edges: with the launch 165 us, without 156 to 160).
static inline bool gnn_long_rows(int64_t E, int64_t N) { return E >= 400 * N || (E >= 24000000 && E >= 150 * N); }
// Share of the gathers that go to the most-gathered twentieth of the vertices, from which on few of them have most of the edges.
constexpr double kStrongSkew = 0.525;
// The plans of a graph and of its transpose, E edges each; the host fields are valid on return.
int gnn_plan_create_pair(const void *indptr, const void *indptr_t, const int32_t *indices, int64_t E, int64_t N, int indptr_is_64,
                         const gnn_plan_params *params, hipStream_t stream, gnn_plan **fwd, gnn_plan **bwd);

// mode: 1 = reciprocal, 2 = reciprocal square root, 3 = reciprocal of (count + 1).
// Builds the array on first use (allocation).
// out[e] = fE[(edge_ids ? edge_ids[e] : e) * lde] for the plan's n_edges edges, into a plan-owned
// array (allocated on first use, refilled by every call).
int gnn_plan_edge_operand(gnn_plan *plan, const float *fE, int64_t lde, const int64_t *edge_ids, const void *indptr, int ip64, hipStream_t stream,
                          const float **out);
int gnn_plan_edge_scale(gnn_plan *plan, const int32_t *indices, int mode, hipStream_t stream, const float **out);

// gnn_plan_hot and everything else that a call over hot tables takes, but for the tables' contents: their memory (plan->padded), partial sums, tiles,
// coefficients in their order.  mode: the factor of the gathered rows.  Only gnn_plan_prepare builds it (build), because it takes 4 to 25 calls to pay:
// 1.0 M vertices, 15 M edges F=100 a first call of 2.9 ms with and 0.8 without, then 0.73 and 0.81 each; 1.8 M, 26 M F=100 4.7 and 1.6, 1.25 and
// 1.60; 27.8 M, 404 M bf16 F=128 52 and 15, 12.6 and 15.1; a step on a subgraph that is new makes one call with each plan.  False: it is not there, and the
// call stays in place; where there is no room nothing of it is left, and the next gnn_plan_prepare asks again.
bool gnn_plan_hot_ready(gnn_plan *plan, const void *indptr, const int32_t *indices, int mode, gnn_weight_kind weights, int64_t F, int esz, hipStream_t stream,
                        bool build, gnn_hot_layout *out);

// ---- producer-side layout ----
// Where a kernel that PRODUCES a matrix (the dense product of a layer, the masked output gradient)
// writes it when the next step is an aggregation that would otherwise copy it into the plan's layout
// first: directly into that layout -- one table per 128-byte column slice, rows by descending gather
// count, a dense table for a short last line, the factor the rows carry as gathered rows multiplied
// in.  fp32 only.  Element (v, j) of the matrix goes to
//     j <  main_cols:  base[(j / 32) * table_stride + rank[v] * 32 + j % 32]
//     j >= main_cols:  tail[rank[v] * tail_ld + (j - main_cols)]
// times gnn_row_factor(scale_mode, counts[v]).
struct gnn_packed_target {
    bool active;            // false: the aggregation of this plan / width gathers rows where they lie (write them plainly)
    float *base;
    int64_t table_stride;
    int32_t main_cols;
    float *tail;
    int64_t tail_ld;
    const int32_t *rank;
    const int32_t *counts;
    int32_t scale_mode;     // 0 none, 1 reciprocal, 2 reciprocal square root, 3 reciprocal of (count + 1)
};
__host__ __device__ static inline float gnn_row_factor(int mode, int64_t count) {
    if (mode == 3) return 1.0f / static_cast<float>(count + 1);
    const float d = static_cast<float>(count > 1 ? count : 1);
    if (mode == 1) return 1.0f / d;
    if (mode == 2) return 1.0f / sqrtf(d);
    return 1.0f;
}
// The target for the matrix that gnn_aggregate_fwd / _bwd (`backward`) with this plan, op and width F would
// gather next (a dense fp32 [N, F] matrix).  Grows the plan's buffers on first use (allocation).
// force: take the layout whatever the size of the graph (tests).
int gnn_packed_target_for(gnn_plan *plan, const void *indptr, const int32_t *indices, int64_t N, int64_t F, int op, bool backward,
                          bool force, hipStream_t stream, gnn_packed_target *out);
// The aggregation over a matrix that a producer has written into that target (no copy; `force` as above).
int gnn_aggregate_prepacked(const void *indptr, const int32_t *indices, void *out, int64_t N, int64_t F, int op,
                            const gnn_opts *opts, bool backward, bool force, const float *bias, int relu);

// gnn_aggregate_fwd with a fused epilogue: Y = act(aggregate(X) + bias), act = rectifier if relu.
int gnn_aggregate_fwd_epilogue(const void *indptr, const int32_t *indices, const void *X, void *Y, int64_t N, int64_t F,
                               int op, const gnn_opts *opts, const float *bias, int relu);

// A pointer to device memory that an asm statement has passed through is generic to the compiler unless its type says where it
// points, and generic loads count as LDS accesses too: every wait for a shuffle then waits for the gathers before it.
template <typename T>
using gnn_global_ptr = const T __attribute__((address_space(1))) *;

// ---- work distribution shared by the aggregation kernels (aggregate.hip, ap.hip) ----
// A launch serves all degree bins of a plan at once: the workgroup index is looked up in a small
// table of bins (heaviest work first).  A bin holds rows (64 >> log2_g rows per wavefront, each row
// group being 2^(log2_g - log2_sr) column lanes x 2^log2_sr edge slots) or hub pieces (one per
// wavefront).
// GNN_BIN_COOP: the four wavefronts of a workgroup share one row (one piece) at a time.
enum gnn_bin_kind : int32_t { GNN_BIN_ROWS = 0, GNN_BIN_HUB_PIECES = 1, GNN_BIN_COOP = 2 };

struct gnn_bin_desc {
    int64_t first_block;  // first workgroup index of this bin (before any slice interleaving)
    int64_t item_begin;   // offset into row_perm (rows) or into the piece list (hub pieces)
    int64_t n_items;      // rows or pieces
    int32_t log2_g;       // lanes per row group
    int32_t log2_sr;      // edge slots per group
    int32_t kind;
    int32_t pad;
};

constexpr int GNN_WAVES_PER_BLOCK = 4;  // 256-thread workgroups

#if defined(__HIP_DEVICE_COMPILE__) || defined(__HIPCC__)
// The pieces of a hub row are added by the wavefront that is done with its piece last, which finds that out by a counter per row and column
// slice: a kernel of its own took 4.8 us behind every call (24,490 vertices, 1.2 M edges, widths 100, 256, 256, 47, five such calls 481 -> 473 us;
// 63 K, 4.9 M, 40, 32, 10 275 -> 259; 174 K, 6.2 M bf16 weighted F=10 140 -> 131; 12.4 M edge vectors of 33 columns 1873 -> 1846).
// The pieces may be on different XCDs, whose L2s do not see each other's lines: what they leave is written through and read past
// the L2s, at the scope of the device, and has arrived there before its piece counts as done.  The last one sets the counter back.
__device__ __forceinline__ void gnn_store_for_device(float *p, float v) { __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }
__device__ __forceinline__ void gnn_store_for_device(int32_t *p, int32_t v) { __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }
__device__ __forceinline__ float gnn_load_for_device(const float *p) { return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }
__device__ __forceinline__ int32_t gnn_load_for_device(const int32_t *p) { return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }
__device__ __forceinline__ int64_t gnn_uniform(int64_t v) {  // of a value that is the same in all lanes
    return int64_t(uint64_t(uint32_t(__builtin_amdgcn_readfirstlane(int(v >> 32)))) << 32 | uint32_t(__builtin_amdgcn_readfirstlane(int(v))));
}
// Called by the lanes of one wavefront that have stored a piece of a row of n_pieces; true in all of them for the row's last piece.
__device__ __forceinline__ bool gnn_hub_done(uint32_t *counter, int n_pieces) {
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");  // the stores of all lanes have arrived
    uint32_t before = 0;
    const unsigned long long lanes = __ballot(true);
    if (int(threadIdx.x & 63) == __builtin_ctzll(lanes)) {
        before = __hip_atomic_fetch_add(counter, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        if (int(before) == n_pieces - 1) __hip_atomic_store(counter, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    before = uint32_t(__builtin_amdgcn_readfirstlane(int(before)));
    asm volatile("" ::: "memory");  // what follows is read afterwards
    return int(before) == n_pieces - 1;
}
#endif

// The bin of a workgroup.  The first workgroups of the bins (INT32_MAX behind the last) arrive in one scalar load; walking
// the descriptors instead is a load and a wait per bin, a good part of what a workgroup of short rows takes (F=29 on
// power-law graphs of 4,600 vertices 11.9 -> 10.7 us a call, 27.8 M vertices bf16 17.5 -> 17.0 ms).
constexpr int GNN_FLAT_BINS = 16;
__device__ static inline int gnn_bin_of_block(const int32_t (&first_block)[GNN_FLAT_BINS], int64_t block) {
    int b = 0;
#pragma unroll
    for (int i = 1; i < GNN_FLAT_BINS; ++i) b = int32_t(block) >= first_block[i] ? i : b;
    return b;
}
static_assert(GNN_MAX_BINS <= GNN_FLAT_BINS, "a launch has at most one bin per bin of the plan");

// Fills `bins` for a launch whose row groups have 2^log2_c column lanes; returns the number of
// workgroups.  plan == nullptr: all N rows in one bin, whole wavefronts per row.
// first_excluded_bin: rows of bins >= it (and the hub pieces) are left out (they are served as source-blocked pieces).
// slices: column slices the launch multiplies the workgroups by.  left_out: bit b = bin b is served by another launch.
//
// A launch that leaves most of the chip idle is bound by latency: the time of a row is the number of its steps (one
// batch of loads each, about a microsecond), one after the other.  So where there are too few wavefronts, rows get more
// edge slots than throughput asks for, and where the steps of a long row or of a hub piece outlast the launch's
// share per wavefront, the four wavefronts of a workgroup share it (24,490 vertices, 1.2 M edges, F=100: 0.33 -> 0.06 ms).
static inline int64_t gnn_fill_bins(gnn_bin_desc *bins, int32_t *n_bins, int32_t (&first_block)[GNN_FLAT_BINS], const gnn_plan *plan, int64_t N, int log2_c,
                                    int first_excluded_bin = INT32_MAX, int slices = 1, uint32_t left_out = 0) {
    constexpr int64_t kWaveSlots = 256 * 4 * 8;  // wavefronts the chip holds of a kernel with 64 registers
    constexpr int kStepLog2 = 3;                 // loads of a slot in flight: edges per step
    const int max_log2_sr = 6 - log2_c;
    int64_t next_block = 0;
    int nb = 0;
    auto add_bin = [&](int kind, int64_t begin, int64_t n_items, int log2_sr) {
        if (n_items <= 0) return;
        gnn_bin_desc &d = bins[nb++];
        d.first_block = next_block;
        d.item_begin = begin;
        d.n_items = n_items;
        d.kind = kind;
        d.log2_sr = log2_sr;
        d.log2_g = (kind & (GNN_BIN_HUB_PIECES | GNN_BIN_COOP)) ? 6 : log2_c + log2_sr;
        d.pad = 0;
        const int64_t items_per_block = (kind & GNN_BIN_COOP) ? 1 : int64_t(GNN_WAVES_PER_BLOCK) * (64 >> d.log2_g);
        next_block += (n_items + items_per_block - 1) / items_per_block;
    };
    if (plan) {
        const int last = plan->n_bins - 1;
        const bool has_hub = plan->n_chunks > 0;
        // Edge slots per row: enough that the shortest row of the bin still takes ~16 steps of one edge (several
        // batches of loads per group), so short rows share a wavefront (64/G rows each) and only long rows
        // get a whole wavefront.
        auto slots_of_bin = [&](int bi) {
            const int64_t lo = bi == 0 ? 0 : plan->params.thresholds[bi - 1];
            int lsr = 0;
            while (lo > 1 && (int64_t(2) << lsr) <= lo) ++lsr;  // floor(log2(lo))
            lsr -= 4;
            return lsr < 0 ? 0 : (lsr > max_log2_sr ? max_log2_sr : lsr);
        };
        int64_t waves = has_hub && first_excluded_bin > last ? plan->n_chunks : 0, steps = 0;
        for (int bi = last; bi >= 0; --bi) {
            if (bi >= first_excluded_bin) continue;
            const int lsr = bi == last && has_hub ? max_log2_sr : slots_of_bin(bi);
            if (!(bi == last && has_hub)) waves += ((plan->bin_offsets[bi + 1] - plan->bin_offsets[bi]) << (log2_c + lsr)) >> 6;
            steps += plan->bin_edges[bi] >> (6 - log2_c + kStepLog2);  // of whole wavefronts
        }
        waves *= slices;
        int boost = 0;
        while (boost < 3 && (waves << (boost + 1)) <= kWaveSlots) ++boost;
        const int64_t steps_per_slot = steps * slices / kWaveSlots;
        auto coop = [&](int64_t longest) { return (longest >> (max_log2_sr + kStepLog2)) > 4 + 2 * steps_per_slot ? int(GNN_BIN_COOP) : 0; };
        // heaviest work first: hub pieces, then bins from long rows to short rows
        if (has_hub && first_excluded_bin > last)
            add_bin(GNN_BIN_HUB_PIECES | coop(plan->params.hub_chunk), 0, plan->n_chunks, max_log2_sr);
        for (int bi = last; bi >= 0; --bi) {
            if (bi >= first_excluded_bin) continue;
            if (bi == last && has_hub) continue;  // handled as pieces (+ finalize)
            if (left_out >> bi & 1u) continue;
            // the longest row of the bin (of the last one, without pieces: unknown)
            const int64_t hi = bi < plan->params.n_thresholds ? plan->params.thresholds[bi] : plan->n_edges;
            int lsr = slots_of_bin(bi);
            // more slots while a slot keeps two edges of the bin's longest rows
            for (int b = 0; b < boost && lsr < max_log2_sr && (int64_t(4) << lsr) <= hi; ++b) ++lsr;
            const int c = coop(hi);
            add_bin(GNN_BIN_ROWS | c, plan->bin_offsets[bi], plan->bin_offsets[bi + 1] - plan->bin_offsets[bi], c ? max_log2_sr : lsr);
        }
    } else {
        add_bin(GNN_BIN_ROWS, 0, N, max_log2_sr);
    }
    *n_bins = nb;
    for (int i = 0; i < GNN_FLAT_BINS; ++i)
        first_block[i] = i < nb && bins[i].first_block < INT32_MAX ? int32_t(bins[i].first_block) : INT32_MAX;
    return next_block;
}

// Copies an fp32 [N, F] matrix with row stride ld_src into rows of stride ld_dst (elements).
// counts: gathers of each row (a plan's col_counts); rows without any are left out.  nullptr: all rows.
int gnn_pad_rows_f32(const float *src, int64_t ld_src, float *dst, int64_t ld_dst, int64_t N, int64_t F, const int32_t *counts,
                     hipStream_t stream);

// gnn_matmul on a typed stream (shared by the C entry point and the layer calls).
// packed: write the result into a producer-side layout instead of C (C may then be nullptr; M = the plan's rows).
// Rectifier gate of a layer's backward pass folded into the product's operand loads: an element of the
// operand counts as 0 where the gate matrix (same shape and strides) is not positive.  a_gate needs
// trans_a == 0 (dZ = G W^T, with W^T given either way), b_gate and colsum need trans_a != 0 and trans_b == 0
// (dW = Z^T G).  colsum: room for colsum_planes planes of N floats; the call writes n_planes of them
// (the column sums of the gated B over each part of the split reduction, to be added in plane order).
struct gnn_gemm_fold {
    const float *a_gate;
    const float *b_gate;
    float *colsum;
    int64_t colsum_planes;
    int64_t n_planes;  // out
    // row_sum [N]: the sum of those column sums, or where there are none of n_rows rows of `rows`, beside the sum of the partial products
    // where that has a kernel (summed, out; at most GNN_ADD_ROWS rows).
    const float *rows;
    int64_t n_rows;
    float *row_sum;
    bool summed;
};
constexpr int64_t GNN_ADD_ROWS = 512;

#if defined(__HIPCC__)
// out[j] = sum of rows b0 ... b1 - 1 of `rows` (F columns), for the 1 << log2_cols columns of column block `block`: all threads of a workgroup of 256.
// In 64 bits, in a fixed order; the loads take longer than the additions.
__device__ __forceinline__ void gnn_add_rows(const float *__restrict__ rows, int64_t b0, int64_t b1, int F, int log2_cols, int block, float *__restrict__ out) {
    __shared__ double red[256];
    const int cols = 1 << log2_cols, row_lanes = 256 >> log2_cols;
    const int jl = threadIdx.x & (cols - 1), rl = threadIdx.x >> log2_cols;
    const int j = block * cols + jl;
    double s = 0.0;
    if (j < F) {
#pragma unroll 8
        for (int64_t b = b0 + rl; b < b1; b += row_lanes) s += double(rows[b * F + j]);
    }
    red[threadIdx.x] = s;
    __syncthreads();
    if (rl == 0 && j < F) {
        for (int k = 1; k < row_lanes; ++k) s += red[(k << log2_cols) + jl];
        out[j] = float(s);
    }
}
#endif
static inline int gnn_add_rows_log2_cols(int64_t F) {
    int l = 0;
    while ((int64_t(1) << l) < F && l < 4) ++l;
    return l;
}

// k-steps of a part of a split product at least
constexpr int64_t GNN_SPLIT_MIN_K = 128;

int gnn_matmul_impl(const float *A, int64_t lda, int trans_a, const float *B, int64_t ldb, int trans_b, float *C, int64_t ldc,
                    int64_t M, int64_t N, int64_t K, const float *bias, int relu, void *workspace, int64_t workspace_bytes,
                    hipStream_t stream, const gnn_packed_target *packed = nullptr, gnn_gemm_fold *fold = nullptr);

static inline int gnn_ilog2_ceil(int64_t x) {
    int l = 0;
    while ((int64_t(1) << l) < x) ++l;
    return l;
}

// ---- short rows, many per wavefront (run_kernel of aggregate.hip, ap_run_kernel of ap.hip) ----
constexpr int GNN_RUN_EDGES = 8;      // edges of such a row at most
constexpr int GNN_RUN_BINS = 8;       // bins of a launch at most
constexpr int64_t GNN_RUN_ROWS = 1 << 18, GNN_RUN_WAVES = 1 << 14;  // see gnn_run_bins_of, gnn_fill_run_bins
constexpr int64_t GNN_MORE_RUN_ROWS = 390000;  // for fp32 rows of one line, and for max and min

struct gnn_run_bin {
    int64_t first_block, item_begin, n_items;
    int32_t longest;        // edges of a row of the bin at most
    int32_t rows_per_wave;  // 64 at most
};
struct gnn_run_bins {
    int64_t n_blocks;
    int32_t n_bins;
    int32_t log2_c;         // lanes per row
    gnn_run_bin bins[GNN_RUN_BINS];
};
__device__ static inline gnn_run_bin gnn_run_bin_of_block(const gnn_run_bins &r, int64_t block) {
    int b = 0;
#pragma unroll
    for (int i = 1; i < GNN_RUN_BINS; ++i) b = i < r.n_bins && block >= r.bins[i].first_block ? i : b;
    return r.bins[b];
}

// Bit b: the rows of bin b are short.  A wavefront takes many of them, so there have to be enough (MEAN, us, rows of
// aggregate_kernel -> run_kernel, directed power-law graphs of 10 edges per vertex: 200 K vertices F=32 27.4 -> 28.9, 100 K F=100 43 -> 45;
// 500 K F=32 59.0 -> 59.2, 100 282 -> 268, 256 506 -> 464; 1 M F=100 624 -> 578, 256 1258 -> 1110, bf16 128 296 -> 254; 320 K, 271,000 short rows, F=33 78
// -> 75, 64 78 -> 75, 256 290 -> 269, bf16 64 52 -> 51, 128 89 -> 80, but F=32 43 -> 46; 600 K, 516,000 F=32 79 -> 77).
static inline uint32_t gnn_run_bins_of(const gnn_plan *plan, int first_excluded_bin, int64_t least_rows = GNN_RUN_ROWS) {
    uint32_t bins = 0;
    int64_t rows = 0;
    if (!plan) return 0;
    for (int b = 0; b < plan->params.n_thresholds && b < GNN_RUN_BINS && b < first_excluded_bin && plan->params.thresholds[b] - 1 <= GNN_RUN_EDGES; ++b) {
        bins |= 1u << b;
        rows += plan->bin_offsets[b + 1] - plan->bin_offsets[b];
    }
    return rows >= least_rows ? bins : 0u;
}

// strips: of 16 bytes per row
static inline void gnn_fill_run_bins(gnn_run_bins &r, const gnn_plan *plan, uint32_t bins, int64_t strips) {
    int64_t rows = 0, next = 0;
    for (int b = 0; b < GNN_RUN_BINS; ++b)
        if (bins >> b & 1u) rows += plan->bin_offsets[b + 1] - plan->bin_offsets[b];
    // as many rows per wavefront as leave the chip a few rounds of wavefronts (500 K vertices F=301: 64 rows 944 us, 32 890, 16 857; 2.45 M
    // F=100 3.62 ms, 3.67, 3.69)
    int32_t per_wave = 64;
    while (per_wave > 16 && rows < per_wave * GNN_RUN_WAVES) per_wave /= 2;
    r = gnn_run_bins{};
    r.log2_c = strips >= 64 ? 6 : gnn_ilog2_ceil(strips);
    for (int b = GNN_RUN_BINS - 1; b >= 0; --b) {
        if (!(bins >> b & 1u)) continue;
        gnn_run_bin &d = r.bins[r.n_bins++];
        d.first_block = next;
        d.item_begin = plan->bin_offsets[b];
        d.n_items = plan->bin_offsets[b + 1] - d.item_begin;
        d.longest = int32_t(plan->params.thresholds[b] - 1);
        d.rows_per_wave = per_wave;
        next += (d.n_items + GNN_WAVES_PER_BLOCK * per_wave - 1) / (GNN_WAVES_PER_BLOCK * per_wave);  // N / 64 at most, so a grid holds it
    }
    r.n_blocks = next;
}

// Neighbour aggregation kernels (Section 4.1, Algorithm 1) for gfx950.
//
//   Y[v, :] = dst_scale(v) * sum_{e in row v} coef(e) * X[indices[e], :]
//
// The same kernel serves the forward pass (CSR by destination) and the
// backward pass (the transposed graph): only the arrays and the scale modes
// differ.  This is HBM/cache-bandwidth-bound gather work, not a dense
// contraction, so there is no MFMA here; the design points are
//   * a 64-lane wavefront is cut into row groups of G lanes; a group owns one
//     output row (one owner per row, as in the paper, so no atomics).  Inside a
//     group, C lanes span the feature row with 16/8/4-byte loads and SR = G/C
//     "edge slots" walk the neighbour list SR edges at a time; the slots are
//     combined with wavefront shuffles at the end of the row.  G, SR come from
//     the degree bin of the row (light rows: many rows per wavefront; heavy
//     rows: the whole wavefront on one row).
//   * neighbour ids (and per-edge coefficients) are fetched as one coalesced
//     tile per group and handed to the slots by cross-lane shuffles, so the
//     index stream is read once, fully coalesced;
//   * accumulation stays in registers for the whole neighbour loop and the
//     output row is written once (the loop order of Algorithm 3);
//   * rows of the hub bin are cut into pieces reduced by different wavefronts
//     into an fp32 scratch; a second kernel adds the pieces in fixed order;
//   * workgroup b of a launch gathers only the 128-byte column slice b % S of
//     the rows, so that the private L2 of the XCD it runs on holds one line of
//     many rows instead of whole rows of few; for a large graph the gathered
//     matrix is first copied into a plan-owned layout made for that: one table
//     per slice, rows by descending gather count, a dense table for a short last
//     line (run_aggregate below).
#include <mutex>
#include <type_traits>

#include "common.h"

// Hub partial sums of gnn_aggregate_fwd_noalloc, the entry point that allocates nothing: one array
// per GPU, part of the loaded code object, held until the process ends.  In host code this name
// only stands for the symbol; the device address is looked up once per device and kept
// (static_scratch_of_current_device), and only that address is ever handed to a kernel.
static __device__ __align__(256) float scratch[GNN_NOALLOC_SCRATCH_BYTES / sizeof(float)];

namespace {

constexpr int kMaxDevices = 64;
std::mutex g_scratch_mutex;
float *g_scratch_ptr[kMaxDevices] = {nullptr};

// Device address of `scratch` on the current device (looked up on the first call there).
int static_scratch_of_current_device(float **out) {
    int dev = -1;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxDevices) return GNN_ERR_LAUNCH;
    std::lock_guard<std::mutex> lock(g_scratch_mutex);
    if (!g_scratch_ptr[dev]) {
        void *p = nullptr;
        if (hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)) != hipSuccess || !p) return GNN_ERR_LAUNCH;
        g_scratch_ptr[dev] = static_cast<float *>(p);
    }
    *out = g_scratch_ptr[dev];
    return GNN_OK;
}

constexpr int kBlockThreads = 256;
constexpr int kWavesPerBlock = kBlockThreads / 64;

enum ScaleMode : int { kScaleNone = 0, kScaleInv = 1, kScaleRsqrt = 2, kScaleInvPlus1 = 3 };
enum SelfMode : int { kSelfNone = 0, kSelfPlain = 1, kSelfInvPlus1 = 2 };  // own row added to the sum
constexpr int kKindHubPieces = GNN_BIN_HUB_PIECES;
using BinDesc = gnn_bin_desc;

struct AggArgs {
    const void *indptr;
    const int32_t *indices;
    const float *w;
    const void *X;
    void *Y;
    int64_t ldx, ldy;
    int32_t F;
    int32_t ip64;
    const int32_t *row_perm;    // nullptr: identity
    const int4 *row_info;       // see gnn_plan; or nullptr
    const float *edge_scale;    // per-edge factor 1/deg or 1/sqrt(deg) of the gathered vertex, or nullptr
    int32_t dst_mode;
    int32_t self_mode;          // SelfMode: add the row's own gathered vector (GraphSAGE-GCN aggregator)
    const int32_t *col_counts;  // per-vertex column counts of the plan (self term of the backward pass)
    const int64_t *chunks;      // hub pieces (row, e_begin, e_end)
    float *partial;             // [n_chunks, ldp] fp32
    int64_t ldp;
    int32_t n_bins;
    int32_t first_block[GNN_FLAT_BINS];  // see gnn_bin_of_block
    int32_t log2_slices;  // column slices; workgroup b serves slice b % n_slices (see run_aggregate)
    int32_t slice_cols;   // columns per slice (the last slice of a launch may hold fewer)
    int32_t store_vec;    // widest non-temporal store the output rows allow (elements, <= VEC)
    int32_t overlap;      // the last strip of a row begins early enough to end with the row (its first columns are computed twice)
    const int32_t *row_map;  // row of the gathered table that holds vertex v (rank layout), or nullptr: v
    const int64_t *p_indptr;  // rank layout: edge range of the row at position i of row_perm within `indices`
    const int64_t *p_chunks;  // rank layout: hub pieces (row, begin, end, original - plan-order position)
    const void *own_X;    // the caller's matrix, where the gathered copy lacks rows that are read as own rows only; or nullptr
    int64_t own_ld;
    int32_t cold_on;      // honour the cold flag (bit 31) of the indices
    int32_t warm_rank;    // rank layout: sources of rank >= this are cold too (INT32_MAX: none)
    int64_t slice_stride;  // > 0: slice-major copy, slice s of the launch reads the table at X + s * slice_stride elements
    const void *X_tail;   // dense tail table (see gnn_layout), read by slice `tail_slice` of the launch
    int64_t ld_tail;
    int32_t tail_slice;   // -1: none
    const float *bias;    // fused layer epilogue: per-column bias added to the scaled row, or nullptr
    int32_t relu;         // fused layer epilogue: rectifier after the bias
    BinDesc bins[GNN_MAX_BINS + 1];
    // (behind what the way to the first gather reads)
    uint32_t *hub_done; // pieces of each hub row that are done, for the last one to add them (gnn_hub_done); nullptr: hub_finalize_kernel does
    int32_t hub_chunk;  // edges of a piece
};

// ------------------------------------------------------------ element access
struct bf16_t { uint16_t bits; };

__device__ __forceinline__ float bf16_to_f32(uint16_t b) { return __uint_as_float(uint32_t(b) << 16); }

// Round to nearest even; NaN stays NaN (quiet).
__device__ __forceinline__ uint16_t f32_to_bf16(float f) {
    uint32_t u = __float_as_uint(f);
    if ((u & 0x7FFFFFFFu) > 0x7F800000u) return uint16_t((u >> 16) | 0x0040u);
    u += 0x7FFFu + ((u >> 16) & 1u);
    return uint16_t(u >> 16);
}

template <typename T, int VEC> struct VecIO;

typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef float f32x2 __attribute__((ext_vector_type(2)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
// The same at the alignment of one element: global loads and stores of 16 bytes need no more, so rows of any width and
// stride are gathered with the widest loads (the machine code for an aligned address is the same).
typedef float f32x4_any __attribute__((ext_vector_type(4), aligned(4)));
typedef float f32x2_any __attribute__((ext_vector_type(2), aligned(4)));
typedef uint32_t u32x4_any __attribute__((ext_vector_type(4), aligned(2)));
typedef uint32_t u32x2_any __attribute__((ext_vector_type(2), aligned(2)));
typedef uint32_t u32_any __attribute__((aligned(2)));

template <> struct VecIO<float, 4> {
    static __device__ __forceinline__ void load(const float *p, float (&v)[4]) {
        const f32x4_any t = *reinterpret_cast<const f32x4_any *>(p); v[0] = t.x; v[1] = t.y; v[2] = t.z; v[3] = t.w;
    }
    static __device__ __forceinline__ void load_nt(const float *p, float (&v)[4]) {
        const f32x4_any t = __builtin_nontemporal_load(reinterpret_cast<const f32x4_any *>(p)); v[0] = t.x; v[1] = t.y; v[2] = t.z; v[3] = t.w;
    }
    // Output rows are written once and not read again by this kernel: non-temporal stores keep
    // them from displacing gathered rows in the L2 (measured: +0.5..1 %).
    static __device__ __forceinline__ void store(float *p, const float (&v)[4]) {
        f32x4 t = {v[0], v[1], v[2], v[3]};
        __builtin_nontemporal_store(t, reinterpret_cast<f32x4 *>(p));
    }
    static __device__ __forceinline__ void store_any(float *p, const float (&v)[4]) {
        *reinterpret_cast<f32x4_any *>(p) = f32x4_any{v[0], v[1], v[2], v[3]};
    }
};
template <> struct VecIO<float, 2> {
    static __device__ __forceinline__ void load(const float *p, float (&v)[2]) {
        const f32x2_any t = *reinterpret_cast<const f32x2_any *>(p); v[0] = t.x; v[1] = t.y;
    }
    static __device__ __forceinline__ void load_nt(const float *p, float (&v)[2]) {
        const f32x2_any t = __builtin_nontemporal_load(reinterpret_cast<const f32x2_any *>(p)); v[0] = t.x; v[1] = t.y;
    }
    static __device__ __forceinline__ void store(float *p, const float (&v)[2]) {
        f32x2 t = {v[0], v[1]};
        __builtin_nontemporal_store(t, reinterpret_cast<f32x2 *>(p));
    }
    static __device__ __forceinline__ void store_any(float *p, const float (&v)[2]) { *reinterpret_cast<f32x2_any *>(p) = f32x2_any{v[0], v[1]}; }
};
template <> struct VecIO<float, 1> {
    static __device__ __forceinline__ void load(const float *p, float (&v)[1]) { v[0] = *p; }
    static __device__ __forceinline__ void load_nt(const float *p, float (&v)[1]) { v[0] = __builtin_nontemporal_load(p); }
    static __device__ __forceinline__ void store(float *p, const float (&v)[1]) { __builtin_nontemporal_store(v[0], p); }
    static __device__ __forceinline__ void store_any(float *p, const float (&v)[1]) { *p = v[0]; }
};
// bf16: the packed words of a strip
template <int VEC> struct Bf16Words;
template <> struct Bf16Words<8> { typedef u32x4 type; typedef u32x4_any any; };
template <> struct Bf16Words<4> { typedef u32x2 type; typedef u32x2_any any; };
template <> struct Bf16Words<2> { typedef uint32_t type; typedef u32_any any; };
template <int VEC> struct VecIO<bf16_t, VEC> {
    typedef typename Bf16Words<VEC>::type words;
    typedef typename Bf16Words<VEC>::any words_any;
    static __device__ __forceinline__ uint32_t word(const words &t, int i) {
        if constexpr (VEC > 2) return t[i]; else return t;
    }
    static __device__ __forceinline__ void unpack(const words &t, float (&v)[VEC]) {
#pragma unroll
        for (int i = 0; i < VEC / 2; ++i) {
            const uint32_t w = word(t, i);
            v[2 * i] = __uint_as_float(w << 16);
            v[2 * i + 1] = __uint_as_float(w & 0xFFFF0000u);
        }
    }
    static __device__ __forceinline__ words pack(const float (&v)[VEC]) {
        words t;
#pragma unroll
        for (int i = 0; i < VEC / 2; ++i) {
            const uint32_t w = uint32_t(f32_to_bf16(v[2 * i])) | (uint32_t(f32_to_bf16(v[2 * i + 1])) << 16);
            if constexpr (VEC > 2) t[i] = w; else t = w;
        }
        return t;
    }
    static __device__ __forceinline__ void load(const bf16_t *p, float (&v)[VEC]) { unpack(words(*reinterpret_cast<const words_any *>(p)), v); }
    static __device__ __forceinline__ void load_nt(const bf16_t *p, float (&v)[VEC]) {
        unpack(words(__builtin_nontemporal_load(reinterpret_cast<const words_any *>(p))), v);
    }
    static __device__ __forceinline__ void store(bf16_t *p, const float (&v)[VEC]) { __builtin_nontemporal_store(pack(v), reinterpret_cast<words *>(p)); }
    static __device__ __forceinline__ void store_any(bf16_t *p, const float (&v)[VEC]) { *reinterpret_cast<words_any *>(p) = pack(v); }
};
template <> struct VecIO<bf16_t, 1> {
    static __device__ __forceinline__ void load(const bf16_t *p, float (&v)[1]) { v[0] = bf16_to_f32(p->bits); }
    static __device__ __forceinline__ void load_nt(const bf16_t *p, float (&v)[1]) {
        v[0] = bf16_to_f32(__builtin_nontemporal_load(&p->bits));
    }
    static __device__ __forceinline__ void store(bf16_t *p, const float (&v)[1]) { __builtin_nontemporal_store(f32_to_bf16(v[0]), &p->bits); }
    static __device__ __forceinline__ void store_any(bf16_t *p, const float (&v)[1]) { p->bits = f32_to_bf16(v[0]); }
};

// A gathered strip stays in the registers the load filled (the packed bits: 16 bytes are four
// registers whether they hold 4 floats or 8 bf16) until it is added; unpacking at the load would
// keep U * VEC floats alive per lane and halve the occupancy of the bf16 kernels.
template <int BYTES> struct RawBits;
template <> struct RawBits<16> { typedef u32x4 type; typedef u32x4_any any; };
template <> struct RawBits<8> { typedef u32x2 type; typedef u32x2_any any; };
template <> struct RawBits<4> { typedef uint32_t type; typedef u32_any any; };
template <> struct RawBits<2> { typedef uint16_t type; typedef uint16_t any; };

template <typename T, int VEC>
struct Strip {
    static constexpr int BYTES = int(sizeof(T)) * VEC;
    static constexpr int WORDS = BYTES >= 4 ? BYTES / 4 : 1;
    using raw_t = typename RawBits<BYTES>::type;
    using any_t = typename RawBits<BYTES>::any;  // at the alignment of one element
    static __device__ __forceinline__ raw_t load(const T *p) { return *reinterpret_cast<const any_t *>(p); }
    static __device__ __forceinline__ raw_t load_nt(const T *p) {
        return __builtin_nontemporal_load(reinterpret_cast<const any_t *>(p));
    }
    static __device__ __forceinline__ raw_t zero() {
        if constexpr (BYTES >= 8) { raw_t z; for (int i = 0; i < WORDS; ++i) z[i] = 0u; return z; }
        else return raw_t(0);
    }
    static __device__ __forceinline__ uint32_t word(const raw_t &r, int i) {
        if constexpr (BYTES >= 8) return r[i];
        else return uint32_t(r);
    }
    static __device__ __forceinline__ void unpack(const raw_t &r, float (&v)[VEC]) {
        if constexpr (sizeof(T) == 4) {
#pragma unroll
            for (int i = 0; i < VEC; ++i) v[i] = __uint_as_float(word(r, i));
        } else if constexpr (VEC == 1) {
            v[0] = __uint_as_float(word(r, 0) << 16);
        } else {
#pragma unroll
            for (int i = 0; i < VEC / 2; ++i) {
                const uint32_t w = word(r, i);
                v[2 * i] = __uint_as_float(w << 16);
                v[2 * i + 1] = __uint_as_float(w & 0xFFFF0000u);
            }
        }
    }
};

// fp32 store of VEC consecutive values (hub partial sums are fp32 whatever T is)
template <int VEC>
__device__ __forceinline__ void store_f32(float *p, const float (&v)[VEC]) {
    if constexpr (VEC % 4 == 0) {
#pragma unroll
        for (int i = 0; i < VEC; i += 4) *reinterpret_cast<f32x4_any *>(p + i) = f32x4_any{v[i], v[i + 1], v[i + 2], v[i + 3]};
    } else if constexpr (VEC == 2) {
        *reinterpret_cast<f32x2_any *>(p) = f32x2_any{v[0], v[1]};
    } else {
        *p = v[0];
    }
}

// Output strip: one non-temporal vector store where the output rows are aligned for it (store_vec == VEC), else one
// plain store at the alignment of an element, which the L2 merges into lines before they are written back
// (non-temporal pieces reach memory as partial lines); a partial last strip (padded gather source) writes only its
// valid columns.
template <typename T, int VEC>
__device__ __forceinline__ void store_strip(T *y, const float (&o)[VEC], int ncols, int store_vec) {
    if (ncols == VEC) {
        if (store_vec == VEC) VecIO<T, VEC>::store(y, o);
        else VecIO<T, VEC>::store_any(y, o);
        return;
    }
#pragma unroll
    for (int i = 0; i < VEC; ++i) {
        if (i < ncols) {
            const float one[1] = {o[i]};
            VecIO<T, 1>::store_any(y + i, one);
        }
    }
}

__device__ __forceinline__ int64_t load_ip(const void *indptr, int ip64, int64_t i) {
    return ip64 ? static_cast<const int64_t *>(indptr)[i]
                : static_cast<int64_t>(static_cast<const int32_t *>(indptr)[i]);
}

__device__ __forceinline__ float scale_of(int mode, int64_t deg) { return gnn_row_factor(mode, deg); }

// The own-row term of a finalisation kernel reads the caller's matrix G, or -- when a producer wrote the
// gathered matrix straight into the plan's layout and no row-major copy exists -- that layout.
struct OwnRowSrc {
    const void *G;        // row-major [N, ldg], already offset to the first column of the launch; nullptr: use the layout
    int64_t ldg;
    const void *tbl;      // slice tables
    int64_t table_stride;
    int32_t main_cols;
    const void *tail;
    int64_t tail_ld;
    const int32_t *rank;
    int32_t col_off;      // first column of the launch within the matrix
};
template <typename T>
__device__ __forceinline__ float own_row_value(const OwnRowSrc &o, int64_t row, int colx) {
    constexpr int LINE = 128 / int(sizeof(T));
    float xs[1];
    if (o.G) {
        VecIO<T, 1>::load(static_cast<const T *>(o.G) + row * o.ldg + colx, xs);
    } else {
        const int col = o.col_off + colx;
        const int64_t r = o.rank[row];
        const T *q = col < o.main_cols ? static_cast<const T *>(o.tbl) + (col / LINE) * o.table_stride + r * LINE + col % LINE
                                       : static_cast<const T *>(o.tail) + r * o.tail_ld + (col - o.main_cols);
        VecIO<T, 1>::load(q, xs);
    }
    return xs[0];
}

// Epilogue of a row's strip: own vector (in `own` where self_mode asks for it), scale, bias, rectifier, store.
template <typename T, int VEC>
__device__ __forceinline__ void write_strip(const AggArgs &a, int64_t row, int64_t row_len, int col, int ncols, const float (&own)[VEC], float (&acc)[VEC]) {
    const float ds = scale_of(a.dst_mode, row_len);
    if (a.self_mode != kSelfNone) {  // Section 6.1: the vertex's own vector joins the sum
        const float self_cf = a.self_mode == kSelfInvPlus1 ? scale_of(kScaleInvPlus1, a.col_counts[row]) : 1.0f;
#pragma unroll
        for (int i = 0; i < VEC; ++i) acc[i] = fmaf(self_cf, own[i], acc[i]);
    }
    float o[VEC];
#pragma unroll
    for (int i = 0; i < VEC; ++i) o[i] = acc[i] * ds;
    if (a.bias) {
#pragma unroll
        for (int i = 0; i < VEC; ++i)
            if (i < ncols) o[i] += a.bias[col + i];
    }
    if (a.relu) {
#pragma unroll
        for (int i = 0; i < VEC; ++i) o[i] = o[i] > 0.0f ? o[i] : 0.0f;
    }
    store_strip<T, VEC>(static_cast<T *>(a.Y) + row * a.ldy + col, o, ncols, a.store_vec);
}

// The row (or hub piece) a group of lanes owns: e0 .. e1 index the launch's `indices`; the per-edge streams of the caller (weights,
// factors) live at e + wdelta.
struct RowOfGroup {
    int64_t e0, e1, row, row_len, wdelta;
};
template <bool COEF>
__device__ __forceinline__ RowOfGroup find_row(const AggArgs &a, const BinDesc &bin, const int4 *row_info, const int64_t *p_indptr,
                                               int64_t wave_in_bin, int lane, bool coop, int wave_in_block) {
    RowOfGroup r{0, 0, -1, 0, 0};
    if (bin.kind & kKindHubPieces) {
        const int64_t piece = wave_in_bin;  // G == 64: one piece per wavefront (per workgroup when shared)
        if (piece < bin.n_items) {
            if (a.p_chunks) {
                const int64_t *p = a.p_chunks + 4 * (bin.item_begin + piece);
                r.row = p[0]; r.e0 = p[1]; r.e1 = p[2]; r.wdelta = p[3];
            } else {
                const int64_t *p = a.chunks + 3 * (bin.item_begin + piece);
                r.row = p[0]; r.e0 = p[1]; r.e1 = p[2];
            }
        }
    } else {
        const int64_t item = wave_in_bin * (64 >> bin.log2_g) + (lane >> bin.log2_g);
        if (item < bin.n_items) {
            int64_t begin;
            if (row_info) {
                const int4 info = row_info[bin.item_begin + item];
                r.row = info.x;
                begin = uint32_t(info.y);
                r.row_len = info.z;
            } else {
                r.row = a.row_perm ? int64_t(a.row_perm[bin.item_begin + item]) : bin.item_begin + item;
                begin = load_ip(a.indptr, a.ip64, r.row);
                r.row_len = load_ip(a.indptr, a.ip64, r.row + 1) - begin;
            }
            r.e0 = p_indptr ? p_indptr[bin.item_begin + item] : begin;
            r.e1 = r.e0 + r.row_len;
            if (COEF) r.wdelta = begin - r.e0;
        }
    }
    if (coop) {  // this wavefront's quarter of the list
        const int64_t quarter = (r.e1 - r.e0 + kWavesPerBlock - 1) / kWavesPerBlock;
        r.e0 += wave_in_block * quarter;
        if (r.e0 + quarter < r.e1) r.e1 = r.e0 + quarter;
    }
    return r;
}

// Adds the sums of a workgroup's wavefronts in order; true on the first one, which has the total.
template <int NPASS, int VEC>
__device__ __forceinline__ bool add_quarters(float *sums, float (&acc)[NPASS][VEC], int wave_in_block, int lane) {
    if (wave_in_block > 0) {
#pragma unroll
        for (int p = 0; p < NPASS; ++p)
#pragma unroll
            for (int i = 0; i < VEC; ++i) sums[(((wave_in_block - 1) * NPASS + p) * VEC + i) * 64 + lane] = acc[p][i];
    }
    __syncthreads();
    if (wave_in_block > 0) return false;
#pragma unroll
    for (int w = 0; w < kWavesPerBlock - 1; ++w)
#pragma unroll
        for (int p = 0; p < NPASS; ++p)
#pragma unroll
            for (int i = 0; i < VEC; ++i) acc[p][i] += sums[((w * NPASS + p) * VEC + i) * 64 + lane];
    return true;
}

// Leaves the sums of a hub piece; on the row's last piece to be done (true), acc and row_len are those of the row.
template <bool COOP, int NPASS, int VEC>
__device__ __forceinline__ bool end_piece(const AggArgs &a, int64_t piece, int64_t row, int slice, const int (&col)[NPASS], const bool (&col_ok)[NPASS],
                                          float (&acc)[NPASS][VEC], int64_t &row_len) {
    float *sums = a.partial + piece * a.ldp;
    if (!COOP || !a.hub_done) {
#pragma unroll
        for (int p = 0; p < NPASS; ++p)
            if (col_ok[p]) store_f32<VEC>(sums + col[p], acc[p]);
        return false;
    }
#pragma unroll
    for (int p = 0; p < NPASS; ++p)
        if (col_ok[p])
#pragma unroll
            for (int i = 0; i < VEC; ++i) gnn_store_for_device(sums + col[p] + i, acc[p][i]);
    // (looked up again: kept from the beginning of the piece it would take registers from its gathers)
    const int64_t begin = load_ip(a.indptr, a.ip64, row);
    row_len = load_ip(a.indptr, a.ip64, row + 1) - begin;
    const int number = int((a.chunks[3 * piece + 1] - begin) / a.hub_chunk), n = int((row_len + a.hub_chunk - 1) / a.hub_chunk);
    if (!gnn_hub_done(a.hub_done + 8 * (piece - number) + slice, n)) return false;
    constexpr int U = VEC >= 8 ? 2 : 4;  // pieces on their way at a time, added in order
    const float *first = sums - number * a.ldp;
#pragma unroll
    for (int p = 0; p < NPASS; ++p) {
        if (!col_ok[p]) continue;
#pragma unroll
        for (int i = 0; i < VEC; ++i) acc[p][i] = 0.0f;
        for (int q = 0; q < n; q += U) {
            float v[U][VEC];
#pragma unroll
            for (int k = 0; k < U; ++k)
#pragma unroll
                for (int i = 0; i < VEC; ++i) v[k][i] = gnn_load_for_device(first + (q + k < n ? q + k : n - 1) * a.ldp + col[p] + i);
#pragma unroll
            for (int k = 0; k < U; ++k)
#pragma unroll
                for (int i = 0; i < VEC; ++i) acc[p][i] = q + k < n ? acc[p][i] + v[k][i] : acc[p][i];
        }
    }
    return true;
}

// ---------------------------------------------------------------- main kernel
// T: storage type of X and Y.  VEC: elements per lane per load.  NPASS: feature
// passes (a lane owns NPASS strips of VEC columns, C*VEC apart).  COEF: edges
// carry a coefficient (explicit weight and/or a scale of the gathered vertex).  COOP: some bins are
// shared by the wavefronts of a workgroup (a variant of its own: it costs the others a wavefront per SIMD).
template <typename T, int VEC, int NPASS, bool COEF, bool COOP = false>
__global__ void __launch_bounds__(kBlockThreads) aggregate_kernel(const AggArgs a) {
    constexpr int U = NPASS >= 2 ? 4 : 8;  // edges in flight per slot
    __shared__ float coop_sums[COOP ? (kWavesPerBlock - 1) * NPASS * VEC * 64 : 1];  // of wavefronts 1 .. 3, by column and lane
    const int lane = threadIdx.x & 63;
    const int wave_in_block = threadIdx.x >> 6;

    // which bin does this workgroup serve (wave-uniform)
    const int slice = int(blockIdx.x) & ((1 << a.log2_slices) - 1);
    const int64_t vblock = int64_t(blockIdx.x) >> a.log2_slices;
    const int col_base = slice * a.slice_cols;
    const int Fk = a.F - col_base < a.slice_cols ? a.F - col_base : a.slice_cols;  // columns of this slice
    // What the way to the first gather needs arrives with the bins: one wait, where the compiler would load each at its use.
    auto info_g = (gnn_global_ptr<int4>)a.row_info;
    auto p_indptr_g = (gnn_global_ptr<int64_t>)a.p_indptr;
    auto indices_g = (gnn_global_ptr<int32_t>)a.indices;
    auto table_g = (gnn_global_ptr<char>)a.X;
    int64_t table_ld = a.ldx, slice_stride = a.slice_stride;
    asm volatile("" : "+s"(info_g), "+s"(p_indptr_g), "+s"(indices_g), "+s"(table_g), "+s"(table_ld), "+s"(slice_stride));
    const int4 *row_info = (const int4 *)info_g;
    const int64_t *p_indptr = (const int64_t *)p_indptr_g;
    const int32_t *indices = (const int32_t *)indices_g;
    const void *table = (const void *)table_g;
    const int b = gnn_bin_of_block(a.first_block, vblock);
    const BinDesc bin = a.bins[b];
    if (Fk <= 0) return;
    const bool coop = COOP && (bin.kind & GNN_BIN_COOP);
    const int64_t wave_in_bin = coop ? vblock - bin.first_block : (vblock - bin.first_block) * kWavesPerBlock + wave_in_block;

    const int G = 1 << bin.log2_g;
    const int SR = 1 << bin.log2_sr;
    const int log2_c = bin.log2_g - bin.log2_sr;
    const int C = 1 << log2_c;
    const int lane_in_g = lane & (G - 1);
    const int gbase = lane - lane_in_g;
    const int s = lane_in_g >> log2_c;  // edge slot of this lane
    const int c = lane_in_g & (C - 1);  // feature strip of this lane

    const RowOfGroup r = find_row<COEF>(a, bin, row_info, p_indptr, wave_in_bin, lane, coop, wave_in_block);
    const int64_t e0 = r.e0, e1 = r.e1, wdelta = r.wdelta;
    const int32_t row = int32_t(r.row);
    int64_t row_len = r.row_len;

    float acc[NPASS][VEC];
#pragma unroll
    for (int p = 0; p < NPASS; ++p)
#pragma unroll
        for (int i = 0; i < VEC; ++i) acc[p][i] = 0.0f;

    // the slice that holds the last, short line of the rows gathers it from the dense tail table
    const bool is_tail = slice == a.tail_slice;
    const bool own_table = is_tail || slice_stride > 0;  // columns are addressed within the slice
    const T *__restrict__ X = is_tail ? static_cast<const T *>(a.X_tail)
                                      : static_cast<const T *>(table) + int64_t(slice) * slice_stride;
    const int64_t ldx = is_tail ? a.ld_tail : (slice_stride > 0 ? int64_t(a.slice_cols) : table_ld);
    int col[NPASS];    // column in the output (and in a caller's matrix)
    int lcol[NPASS];   // column in the table this slice gathers from
    int ncols[NPASS];  // valid columns of the strip (< VEC only for the last strip of a padded matrix)
    bool col_ok[NPASS];
#pragma unroll
    for (int p = 0; p < NPASS; ++p) {
        int lc = (p * C + c) * VEC;
        col_ok[p] = lc < Fk;
        if (a.overlap && lc > Fk - VEC) lc = Fk - VEC;  // may begin in the slice before: those columns get the same values there
        col[p] = col_base + lc;
        lcol[p] = own_table ? lc : col[p];
        ncols[p] = Fk - lc < VEC ? Fk - lc : VEC;
    }

    // Neighbour ids (and coefficients) travel in coalesced tiles of G edges per group; the next tiles
    // are requested before the current ones are consumed, so only the first index loads of a row are
    // exposed latency.  The one-strip fp32 kernel (the sliced launches) asks for two tiles at a time: the
    // lines of the index stream that a row spans are then touched once instead of once per tile, with
    // some thousand gathers of the compute unit in between (worth 1 %; the other variants would pay for
    // the registers with a wavefront of occupancy).
    constexpr int Q = (sizeof(T) == 4 && NPASS == 1) ? 2 : 1;
    auto fetch_tiles = [&](int64_t e_first, int (&u_out)[Q], float (&cf_out)[Q]) {
#pragma unroll
        for (int q = 0; q < Q; ++q) {
            const int64_t e = e_first + q * G;
            u_out[q] = 0;
            cf_out[q] = 0.0f;
            if (e < e1) {
                u_out[q] = indices[e];
                if (COEF) {
                    cf_out[q] = a.w ? a.w[e + wdelta] : 1.0f;
                    if (a.edge_scale) cf_out[q] *= a.edge_scale[e + wdelta];
                }
            }
        }
    };
    int nxt_u[Q];
    float nxt_cf[Q];
    fetch_tiles(e0 + lane_in_g, nxt_u, nxt_cf);
    for (int64_t first = e0; __any(first < e1); first += Q * G) {
    int cur_u[Q];
    float cur_cf[Q];
#pragma unroll
    for (int q = 0; q < Q; ++q) { cur_u[q] = nxt_u[q]; cur_cf[q] = nxt_cf[q]; }
    fetch_tiles(first + Q * G + lane_in_g, nxt_u, nxt_cf);
#pragma unroll 1
    for (int q = 0; q < Q; ++q) {
        const int64_t tile = first + q * G;
        if (Q > 1 && !__any(tile < e1)) break;
        const int my_u = cur_u[0];
        const float my_cf = cur_cf[0];
#pragma unroll
        for (int i = 0; i + 1 < Q; ++i) { cur_u[i] = cur_u[i + 1]; cur_cf[i] = cur_cf[i + 1]; }
        const int64_t left = e1 - tile;
        const int n_tile = left < G ? (left > 0 ? int(left) : 0) : G;

        for (int j0 = 0; __any(j0 < n_tile); j0 += SR * U) {
            int u[U];
            float cf[U];
            bool ok[U];
#pragma unroll
            for (int k = 0; k < U; ++k) {
                const int j = j0 + k * SR + s;
                const int src_lane = gbase + (j & (G - 1));
                u[k] = __shfl(my_u, src_lane);
                if (COEF) cf[k] = __shfl(my_cf, src_lane);
                ok[k] = j < n_tile;
            }
            // bf16 strips stay packed until they are added (see Strip); fp32 strips are floats already,
            // and the plain arrays schedule slightly better (F=256: 12.04 against 12.26 ms)
            constexpr bool PACKED = sizeof(T) == 2;
            typename Strip<T, VEC>::raw_t xr_[PACKED ? U : 1][NPASS];
            float x[PACKED ? 1 : U][NPASS][VEC];
#pragma unroll
            for (int k = 0; k < U; ++k) {
                // Bit 31 of an index marks a rarely gathered ("cold") source (plan-owned index copy):
                // its row is fetched with a non-temporal load (which the present compiler merges with the other
                // one into a plain load; kept apart they measure the same), so that it does not displace the
                // warm rows of the L2.
                const int32_t src = u[k] & 0x7FFFFFFF;
                const bool cold = a.cold_on && (u[k] < 0 || src >= a.warm_rank);
                const T *xr = X + int64_t(src) * ldx;
#pragma unroll
                for (int p = 0; p < NPASS; ++p) {
                    if (ok[k] && col_ok[p]) {
                        if constexpr (PACKED) {
                            if (cold) xr_[k][p] = Strip<T, VEC>::load_nt(xr + lcol[p]);
                            else xr_[k][p] = Strip<T, VEC>::load(xr + lcol[p]);
                        } else {
                            if (cold) VecIO<T, VEC>::load_nt(xr + lcol[p], x[k][p]);
                            else VecIO<T, VEC>::load(xr + lcol[p], x[k][p]);
                        }
                    } else {
                        if constexpr (PACKED) {
                            xr_[k][p] = Strip<T, VEC>::zero();
                        } else {
#pragma unroll
                            for (int i = 0; i < VEC; ++i) x[k][p][i] = 0.0f;
                        }
                    }
                }
            }
#pragma unroll
            for (int k = 0; k < U; ++k)
#pragma unroll
                for (int p = 0; p < NPASS; ++p) {
                    float xv[VEC];
                    if constexpr (PACKED) {
                        Strip<T, VEC>::unpack(xr_[k][p], xv);
                    } else {
#pragma unroll
                        for (int i = 0; i < VEC; ++i) xv[i] = x[k][p][i];
                    }
#pragma unroll
                    for (int i = 0; i < VEC; ++i) {
                        if (COEF) acc[p][i] = fmaf(ok[k] ? cf[k] : 0.0f, xv[i], acc[p][i]);
                        else acc[p][i] += xv[i];
                    }
                }
        }
    }
    }

    // combine the edge slots of the group
    for (int off = C; off < G; off <<= 1) {
#pragma unroll
        for (int p = 0; p < NPASS; ++p)
#pragma unroll
            for (int i = 0; i < VEC; ++i) acc[p][i] += __shfl_xor(acc[p][i], off);
    }

    if constexpr (COOP) {
        if (coop && !add_quarters<NPASS, VEC>(coop_sums, acc, wave_in_block, lane)) return;
    }
    if (row < 0 || s != 0) return;
    if ((bin.kind & kKindHubPieces) && !end_piece<COOP>(a, bin.item_begin + gnn_uniform(wave_in_bin), row, slice, col, col_ok, acc, row_len)) return;
    const int64_t self_row = (a.self_mode != kSelfNone && a.row_map) ? int64_t(a.row_map[row]) : row;
#pragma unroll
    for (int p = 0; p < NPASS; ++p) {
        if (!col_ok[p]) continue;
        float own[VEC];
        if (a.self_mode != kSelfNone)
            VecIO<T, VEC>::load(a.own_X ? static_cast<const T *>(a.own_X) + row * a.own_ld + col[p] : X + self_row * ldx + lcol[p], own);
        write_strip<T, VEC>(a, row, row_len, col[p], ncols[p], own, acc[p]);
    }
}

// The same for one strip per lane, 16-byte loads and tables below 4 GB, with a third of the vector instructions: where a launch is a
// chain of loads rather than a stream of them, each batch of gathers leaves earlier.  A lane multiplies its own index by the row
// stride as it fetches it, so that a shuffle brings an offset; a slot without an edge carries kNoRow, which lies behind the end of
// the buffer, where a buffer load returns zeros and touches no memory (aggregate_kernel: a compare, four zeros and a 64-bit
// multiply-add per line).  Rows of 4, 2, 1 lanes (CLANES; 8 stands for eight or more) gather from two or four tiles of indices at a
// time, so that they too have eight (four) lines in flight.
//
// 24,490 vertices, 1.2 M edges, us: F=4 27.0 -> 14.9, 16 18.6 -> 14.5, 100 45.5 -> 42.1, 256 78 -> 68; bf16 F=64 on 245 K vertices 107 -> 96,
// F=100 on 2.45 M 2.61 -> 2.55 ms.  fp32 launches that fill the chip are bound by lines and lose 1 to 3 % (133 K vertices, 79 M edges F=64
// 1.235 -> 1.244 ms, 2.45 M F=16 787 -> 810 us): they stay with aggregate_kernel (see use_gather_kernel).
constexpr uint32_t kNoRow = 0xFFFF0000u;         // offset of no row, end of the buffer; columns add less than 64 KB
constexpr int64_t kMaxTableBytes = 0xFFFF0000;

template <typename T, bool COEF, bool COOP, int CLANES>
__global__ void __launch_bounds__(kBlockThreads) gather_kernel(const AggArgs a) {
    constexpr int VEC = 16 / int(sizeof(T));
    __shared__ float coop_sums[COOP ? (kWavesPerBlock - 1) * VEC * 64 : 1];  // of wavefronts 1 .. 3, by column and lane
    const int lane = threadIdx.x & 63;
    const int wave_in_block = threadIdx.x >> 6;
    const int slice = int(blockIdx.x) & ((1 << a.log2_slices) - 1);
    const int64_t vblock = int64_t(blockIdx.x) >> a.log2_slices;
    const int col_base = slice * a.slice_cols;
    const int Fk = a.F - col_base < a.slice_cols ? a.F - col_base : a.slice_cols;  // columns of this slice
    // What the way to the first gather needs arrives with the bins: one wait, where the compiler would load each at its use.
    auto info_g = (gnn_global_ptr<int4>)a.row_info;
    auto p_indptr_g = (gnn_global_ptr<int64_t>)a.p_indptr;
    auto indices_g = (gnn_global_ptr<int32_t>)a.indices;
    auto table_g = (gnn_global_ptr<char>)a.X;
    int64_t table_ld = a.ldx, slice_stride = a.slice_stride;
    asm volatile("" : "+s"(info_g), "+s"(p_indptr_g), "+s"(indices_g), "+s"(table_g), "+s"(table_ld), "+s"(slice_stride));
    const int4 *row_info = (const int4 *)info_g;
    const int64_t *p_indptr = (const int64_t *)p_indptr_g;
    const int32_t *indices = (const int32_t *)indices_g;
    const void *table = (const void *)table_g;
    const int b = gnn_bin_of_block(a.first_block, vblock);
    const BinDesc bin = a.bins[b];
    if (Fk <= 0) return;
    const bool coop = COOP && (bin.kind & GNN_BIN_COOP);
    const int64_t wave_in_bin = coop ? vblock - bin.first_block : (vblock - bin.first_block) * kWavesPerBlock + wave_in_block;

    const int G = 1 << bin.log2_g;
    const int SR = 1 << bin.log2_sr;
    const int log2_c = bin.log2_g - bin.log2_sr;
    const int C = 1 << log2_c;
    const int lane_in_g = lane & (G - 1);
    const int gbase = lane - lane_in_g;
    const int s = lane_in_g >> log2_c;  // edge slot of this lane
    const int c = lane_in_g & (C - 1);  // feature strip of this lane

    const RowOfGroup r = find_row<COEF>(a, bin, row_info, p_indptr, wave_in_bin, lane, coop, wave_in_block);
    const int n_edges = int(r.e1 - r.e0);
    const int32_t row = int32_t(r.row), edges_of_row = int32_t(r.row_len);
    const int32_t *idx = indices + r.e0;
    const float *w = COEF && a.w ? a.w + r.e0 + r.wdelta : nullptr;
    const float *scale = COEF && a.edge_scale ? a.edge_scale + r.e0 + r.wdelta : nullptr;

    // the slice that holds the last, short line of the rows gathers it from the dense tail table
    const bool is_tail = slice == a.tail_slice;
    const bool own_table = is_tail || slice_stride > 0;  // columns are addressed within the slice
    const T *X = is_tail ? static_cast<const T *>(a.X_tail) : static_cast<const T *>(table) + int64_t(slice) * slice_stride;
    const int64_t ldx = is_tail ? a.ld_tail : (slice_stride > 0 ? int64_t(a.slice_cols) : table_ld);
    int lc = c * VEC;
    const bool col_ok = lc < Fk;
    if (a.overlap && lc > Fk - VEC) lc = Fk - VEC;  // may begin in the slice before: those columns get the same values there
    const int col = col_base + lc;                  // column in the output (and in a caller's matrix)
    const int lcol = own_table ? lc : col;          // column in the table this slice gathers from
    const int ncols = Fk - lc < VEC ? Fk - lc : VEC;  // valid columns of the strip (< VEC only for the last strip of a padded matrix)
    const uint32_t row_bytes = uint32_t(ldx) * uint32_t(sizeof(T));
    const uint32_t col_bytes = uint32_t(lcol) * uint32_t(sizeof(T));
    __amdgpu_buffer_rsrc_t rsrc = __builtin_amdgcn_make_buffer_rsrc(const_cast<T *>(X), 0, int(kNoRow), 0x00020000);  // raw, bytes

    float acc[1][VEC];
#pragma unroll
    for (int i = 0; i < VEC; ++i) acc[0][i] = 0.0f;

    auto fetch = [&](int e, uint32_t &off, float &cf) {
        off = kNoRow;
        cf = 0.0f;
        if (e < n_edges) {
            off = uint32_t(idx[e] & 0x7FFFFFFF) * row_bytes;
            if (COEF) {
                cf = a.w ? w[e] : 1.0f;
                if (a.edge_scale) cf *= scale[e];
            }
        }
    };
    const int shfl0 = 4 * (gbase + s), shfl_step = 4 * SR;
    // U edges per slot of a tile (G edges) at a time, of TILES tiles: eight loads in flight.  Q tiles are fetched while the Q before
    // them are gathered.
    auto walk = [&](auto u_const, auto tiles_const, auto q_const) {
        constexpr int U = decltype(u_const)::value, TILES = decltype(tiles_const)::value, Q = decltype(q_const)::value;
        uint32_t nxt[Q];
        float nxt_cf[Q];
#pragma unroll
        for (int q = 0; q < Q; ++q) fetch(lane_in_g + q * G, nxt[q], nxt_cf[q]);
        for (int first = 0; __any(first < n_edges); first += Q * G) {
            uint32_t cur[Q];
            float cur_cf[Q];
#pragma unroll
            for (int q = 0; q < Q; ++q) { cur[q] = nxt[q]; cur_cf[q] = nxt_cf[q]; }
#pragma unroll
            for (int q = 0; q < Q; ++q) fetch(first + (Q + q) * G + lane_in_g, nxt[q], nxt_cf[q]);
#pragma unroll 1
            for (int q0 = 0; q0 < Q; q0 += TILES) {
                const int left = n_edges - (first + q0 * G), n = left < G ? left : G;
                if (q0 > 0 && !__any(left > 0)) break;
                int at = shfl0;
                for (int j0 = 0; __any(j0 < n); j0 += SR * U, at += U * shfl_step) {
                    u32x4 x[TILES][U];
                    float cf[TILES][U];
#pragma unroll
                    for (int q = 0; q < TILES; ++q)
#pragma unroll
                        for (int k = 0; k < U; ++k) {
                            const uint32_t off = uint32_t(__builtin_amdgcn_ds_bpermute(at + k * shfl_step, int(cur[q])));
                            if (COEF) cf[q][k] = __int_as_float(__builtin_amdgcn_ds_bpermute(at + k * shfl_step, __float_as_int(cur_cf[q])));
                            x[q][k] = __builtin_amdgcn_raw_buffer_load_b128(rsrc, col_ok ? off + col_bytes : kNoRow, 0, 0);
                        }
#pragma unroll
                    for (int q = 0; q < TILES; ++q)
#pragma unroll
                        for (int k = 0; k < U; ++k) {
                            float v[VEC];
                            Strip<T, VEC>::unpack(x[q][k], v);
#pragma unroll
                            for (int i = 0; i < VEC; ++i) {
                                if (COEF) acc[0][i] = fmaf(cf[q][k], v[i], acc[0][i]);
                                else acc[0][i] += v[i];
                            }
                        }
                    if (U < 8) break;  // a tile of narrow rows is one step
                }
#pragma unroll
                for (int q = 0; q + TILES < Q; ++q) { cur[q] = cur[q + TILES]; cur_cf[q] = cur_cf[q + TILES]; }
            }
        }
    };
    using std::integral_constant;
    if constexpr (CLANES == 8) walk(integral_constant<int, 8>(), integral_constant<int, 1>(), integral_constant<int, sizeof(T) == 4 ? 2 : 1>());
    else walk(integral_constant<int, CLANES>(), integral_constant<int, CLANES == 1 ? 4 : 8 / CLANES>(), integral_constant<int, CLANES == 1 ? 4 : 8 / CLANES>());

    // combine the edge slots of the group
    for (int off = C; off < G; off <<= 1)
#pragma unroll
        for (int i = 0; i < VEC; ++i) acc[0][i] += __shfl_xor(acc[0][i], off);
    if constexpr (COOP) {
        if (coop && !add_quarters<1, VEC>(coop_sums, acc, wave_in_block, lane)) return;
    }
    if (row < 0 || s != 0 || !col_ok) return;
    int64_t row_len = edges_of_row;
    if (bin.kind & kKindHubPieces) {
        const int cols[1] = {col};
        const bool cols_ok[1] = {true};
        if (!end_piece<COOP>(a, bin.item_begin + gnn_uniform(wave_in_bin), row, slice, cols, cols_ok, acc, row_len)) return;
    }
    float own[VEC];
    if (a.self_mode != kSelfNone) {
        const int64_t self_row = a.row_map ? int64_t(a.row_map[row]) : row;
        VecIO<T, VEC>::load(a.own_X ? static_cast<const T *>(a.own_X) + row * a.own_ld + col : X + self_row * ldx + lcol, own);
    }
    write_strip<T, VEC>(a, row, row_len, col, ncols, own, acc[0]);
}

struct RunArgs {
    AggArgs a;              // X: first slice table, or the matrix of whole rows; F: all columns
    gnn_run_bins bins;
};

// Rows of at most GNN_RUN_EDGES edges, all columns.  A wavefront takes up to 64 of them: lane l reads what describes row l, then sets of
// 64 / C rows follow each other, C lanes per row, the indices of the next set on their way while this one is gathered.
//
// As rows of aggregate_kernel they were bound by the rate at which workgroups start (570 per us over the chip: 32 rows of one line
// each, 16 of two, gone after a few loads that wait for each other) and, off line boundaries, by partial lines of the output that
// the slices write from different XCDs.  Half of the 2.45 M rows of a power-law graph have less than four edges: F=256, rows without
// edges 387 -> 186 us (4.8 TB/s written), of one to seven 600 -> 550, the call 7.44 -> 7.13 ms; F=100 3.85 -> 3.62; 27.8 M vertices,
// bf16 F=128, 16.4 -> 14.8.  Whole rows, because writing counts for more here than what slices keep in an L2 (in slices F=100 3.95 ms,
// 256 7.20).  Up to 15 edges the slices win again: such rows are bound by what they gather.
template <typename T, int VEC, bool COEF>
__global__ void __launch_bounds__(kBlockThreads) run_kernel(const RunArgs r) {
    constexpr int LINE = 128 / int(sizeof(T));
    const AggArgs &a = r.a;
    const int lane = threadIdx.x & 63;
    const gnn_run_bin bin = gnn_run_bin_of_block(r.bins, blockIdx.x);
    const int64_t item0 = ((int64_t(blockIdx.x) - bin.first_block) * kWavesPerBlock + (threadIdx.x >> 6)) * bin.rows_per_wave;
    const int n_rows = bin.n_items - item0 < bin.rows_per_wave ? int(bin.n_items - item0) : bin.rows_per_wave;
    if (n_rows <= 0) return;
    const int log2_c = r.bins.log2_c, C = 1 << log2_c;
    const int c = lane & (C - 1), gbase = lane & ~(C - 1);
    const int per_set = 64 >> log2_c, in_set = lane >> log2_c;

    int my_row = -1, my_len = 0, my_own = 0;
    int64_t my_e0 = 0, my_wdelta = 0;
    if (lane < n_rows) {
        const int64_t at = bin.item_begin + item0 + lane;
        int64_t begin;
        if (a.row_info) {
            const int4 info = a.row_info[at];
            my_row = info.x;
            begin = uint32_t(info.y);
            my_len = info.z;
        } else {
            my_row = a.row_perm[at];
            begin = load_ip(a.indptr, a.ip64, my_row);
            my_len = int(load_ip(a.indptr, a.ip64, int64_t(my_row) + 1) - begin);
        }
        my_e0 = a.p_indptr ? a.p_indptr[at] : begin;
        if (COEF) my_wdelta = begin - my_e0;
        if (a.self_mode != kSelfNone) my_own = a.row_map && !a.own_X ? a.row_map[my_row] : my_row;
    }
    auto of_row = [&](int64_t v, int src) {
        return int64_t((uint64_t(uint32_t(__shfl(int(uint64_t(v) >> 32), src))) << 32) | uint32_t(__shfl(int(uint32_t(v)), src)));
    };
    auto run = [&](auto edges) {
        constexpr int E = decltype(edges)::value;  // edges of a row at most
        for (int strip0 = 0; strip0 * VEC < a.F; strip0 += C) {
            int col = (strip0 + c) * VEC;
            const bool col_ok = col < a.F;
            if (a.overlap && col > a.F - VEC) col = a.F - VEC;
            const int ncols = a.F - col < VEC ? a.F - col : VEC;
            // this lane's columns in the table that has them
            const T *X = static_cast<const T *>(a.X) + col;
            int64_t ldx = a.ldx;
            if (a.slice_stride > 0) {
                X = static_cast<const T *>(a.X) + int64_t(col / LINE) * a.slice_stride + col % LINE;
                ldx = LINE;
            }
            if (a.tail_slice >= 0 && col >= a.tail_slice * LINE) {
                X = static_cast<const T *>(a.X_tail) + (col - a.tail_slice * LINE);
                ldx = a.ld_tail;
            }
            auto fetch = [&](int src, int &u, float &cf) {
                const int len = __shfl(my_len, src);
                const int64_t first = of_row(my_e0, src);
                int64_t first_w = 0;
                if (COEF) first_w = first + of_row(my_wdelta, src);
                u = 0;
                cf = 0.0f;
                if (c < len) {
                    u = a.indices[first + c];
                    if (COEF) {
                        cf = a.w ? a.w[first_w + c] : 1.0f;
                        if (a.edge_scale) cf *= a.edge_scale[first_w + c];
                    }
                }
            };
            int nxt_u = 0;
            float nxt_cf = 0.0f;
            if (E > 0) fetch(in_set, nxt_u, nxt_cf);
            for (int set = 0; set < n_rows; set += per_set) {
                const int src = set + in_set;
                const int row = __shfl(my_row, src), len = E > 0 ? __shfl(my_len, src) : 0;
                const int cur_u = nxt_u;
                const float cur_cf = nxt_cf;
                if (E > 0) fetch((src + per_set) & 63, nxt_u, nxt_cf);  // behind the last set: the first one again
                float own[VEC];
                if (a.self_mode != kSelfNone) {
                    const int64_t own_row = __shfl(my_own, src);
                    if (row >= 0 && col_ok) VecIO<T, VEC>::load(a.own_X ? static_cast<const T *>(a.own_X) + own_row * a.own_ld + col : X + own_row * ldx, own);
                }
                typename Strip<T, VEC>::raw_t x[E > 0 ? E : 1];
                float cf[E > 0 ? E : 1];
#pragma unroll
                for (int k = 0; k < E; ++k) {
                    const int u = __shfl(cur_u, gbase + k);
                    if (COEF) cf[k] = __shfl(cur_cf, gbase + k);
                    const int32_t src_row = u & 0x7FFFFFFF;
                    const T *xr = X + int64_t(src_row) * ldx;
                    if (k < len && col_ok) {
                        if (a.cold_on && (u < 0 || src_row >= a.warm_rank)) x[k] = Strip<T, VEC>::load_nt(xr);
                        else x[k] = Strip<T, VEC>::load(xr);
                    } else {
                        x[k] = Strip<T, VEC>::zero();
                    }
                }
                float sum[VEC];
#pragma unroll
                for (int i = 0; i < VEC; ++i) sum[i] = 0.0f;
#pragma unroll
                for (int k = 0; k < E; ++k) {
                    float xv[VEC];
                    Strip<T, VEC>::unpack(x[k], xv);
#pragma unroll
                    for (int i = 0; i < VEC; ++i) {
                        if (COEF) sum[i] = fmaf(k < len ? cf[k] : 0.0f, xv[i], sum[i]);
                        else sum[i] += xv[i];
                    }
                }
                if (row >= 0 && col_ok) write_strip<T, VEC>(a, row, len, col, ncols, own, sum);
            }
        }
    };
    if (bin.longest <= 0) run(std::integral_constant<int, 0>());
    else if (bin.longest <= 1) run(std::integral_constant<int, 1>());
    else if (bin.longest <= 4) run(std::integral_constant<int, 4>());
    else run(std::integral_constant<int, GNN_RUN_EDGES>());
}

// Adds the pieces of each hub row in their fixed order and writes the row: of launches that fill the chip, beside which it is nothing (in their
// kernels the last piece would take registers from the gathers, 4,096 vertices F=64 10.58 -> 10.66 us), and of calls with scratch of the caller's.
template <typename T>
__global__ void __launch_bounds__(256) hub_finalize_kernel(const int32_t *__restrict__ hub_rows, int64_t n_hub,
                                                           const int64_t *__restrict__ piece_offsets,
                                                           const float *__restrict__ partial, const void *indptr,
                                                           int ip64, int dst_mode, T *__restrict__ Y, int64_t ldy,
                                                           int F, int64_t ldp, int self_mode, const OwnRowSrc own,
                                                           const int32_t *__restrict__ col_counts,
                                                           const float *__restrict__ bias, int relu, int col_begin) {
    const int64_t i = blockIdx.x;
    if (i >= n_hub) return;
    const int64_t row = hub_rows[i];
    const int64_t p0 = piece_offsets[i], p1 = piece_offsets[i + 1];
    const float ds = scale_of(dst_mode, load_ip(indptr, ip64, row + 1) - load_ip(indptr, ip64, row));
    for (int colx = col_begin + threadIdx.x; colx < F; colx += blockDim.x) {
        float sum = 0.0f;
        for (int64_t p = p0; p < p1; p += 8) {  // eight pieces on their way at a time, added in order
            float v[8];
#pragma unroll
            for (int k = 0; k < 8; ++k) v[k] = partial[(p + k < p1 ? p + k : p1 - 1) * ldp + colx];
#pragma unroll
            for (int k = 0; k < 8; ++k) sum = p + k < p1 ? sum + v[k] : sum;
        }
        if (self_mode != kSelfNone)
            sum = fmaf(self_mode == kSelfInvPlus1 ? scale_of(kScaleInvPlus1, col_counts[row]) : 1.0f,
                       own_row_value<T>(own, row, colx), sum);
        float o[1] = {sum * ds};
        if (bias) o[0] += bias[colx];
        if (relu) o[0] = o[0] > 0.0f ? o[0] : 0.0f;
        VecIO<T, 1>::store(Y + row * ldy + colx, o);
    }
}

// ---- source-blocked pieces of the long rows (see blocked.hip) ----
// Four consecutive elements of a per-edge stream, loaded at the alignment of one element.
template <typename E>
struct __attribute__((packed, aligned(alignof(E)))) Packed { E e[4]; };

struct PieceArgs {
    const int32_t *pieces;   // [n_pieces * 4] (begin, length, partial slot, row index)
    int64_t n_pieces;
    const int32_t *idx;      // source ranks, block-major piece order
    const uint16_t *idx16;   // the same as offsets from the block's first rank (null: none); not for the last block
    const uint16_t *piece_block;  // [n_pieces] block of each piece
    int32_t n_blocks, hot_lines, block_lines;
    const uint32_t *epos;    // CSR position of each edge (for the caller's per-edge streams)
    const float *w;          // the caller's weights, read at epos (a random 4-byte read per edge) ...
    const float *w_blk;      // ... or their plan-owned copy in the order of idx (weights bound to the plan)
    const float *scale_blk;  // plan-owned factor of the gathered vertex per edge, in the order of idx
    const void *X;           // first slice table of the launch
    int64_t slice_stride;    // elements between two slice tables
    float *partial;          // [slices][n_pieces][floats per line]
    int32_t log2_slices;
    // Hot tables: the last block's pieces gather the caller's rows (of `cols` columns of the launch from X_cold on) by vertex.  idx16 is there, and tells them.
    const int32_t *cold_vertices;  // of the edges from cold_begin on
    uint32_t cold_begin;
    const void *X_cold;
    int64_t ld_cold;
    int32_t cols;
};

// L lanes own one piece and one line of every gathered row (16 bytes each: L = 8 for lines of 128 bytes, 4 and 2 for
// shorter rows); a wavefront works on 64 / L consecutive pieces, with 8 lines of each in flight.  The pieces of a
// launch follow the block order of the layout, so the workgroups that run side by side gather from the same block of
// source rows.  Every piece writes one fp32 partial line; blk_finalize_kernel adds them.
template <typename T, bool COEF, int L, bool HOT = false>
__global__ void __launch_bounds__(kBlockThreads) piece_kernel(const PieceArgs a) {
    constexpr int VEC = 16 / int(sizeof(T));   // elements per lane
    constexpr int LINE = L * VEC;              // elements per line = floats per partial line
    constexpr int U = 8;
    constexpr int WINDOW = 4 * L;              // edges whose streams a group holds in registers
    const int lane = threadIdx.x & 63;
    const int slice = int(blockIdx.x) & ((1 << a.log2_slices) - 1);
    const int64_t vblock = int64_t(blockIdx.x) >> a.log2_slices;
    const int c = lane & (L - 1), gbase = lane & ~(L - 1);
    const int64_t piece = (vblock * kWavesPerBlock + (threadIdx.x >> 6)) * (64 / L) + lane / L;
    uint32_t begin = 0;
    int len = 0;
    int64_t slot = 0;
    if (piece < a.n_pieces) {
        const int4 d = *reinterpret_cast<const int4 *>(a.pieces + 4 * piece);
        begin = uint32_t(d.x); len = d.y; slot = d.z;
    }
    // the piece's block and its first rank, for the 16-bit indices
    bool narrow = false;
    int base = 0;
    if (a.idx16 && len > 0) {
        const int k = a.piece_block[piece];
        narrow = k < a.n_blocks - 1;
        base = k == 0 ? 0 : a.hot_lines + (k - 1) * a.block_lines;
    }
    const T *__restrict__ X = static_cast<const T *>(a.X) + int64_t(slice) * a.slice_stride + c * VEC;
    int64_t ld = LINE;
    bool lane_ok = true;
    if constexpr (HOT) {
        if (!narrow) {
            X = static_cast<const T *>(a.X_cold) + slice * LINE + c * VEC;
            ld = a.ld_cold;
            lane_ok = slice * LINE + c * VEC < a.cols;  // whole strips: the caller's rows end with one
        }
    }
    float acc[VEC];
#pragma unroll
    for (int i = 0; i < VEC; ++i) acc[i] = 0.0f;

    // The per-edge streams are read a window of 4 L edges at a time: lane c of the group holds edges
    // [t + 4c, t + 4c + 4) of the piece, one 8- or 16-byte load per stream (at the 2- or 4-byte
    // alignment of the element: a piece begins anywhere), so a group touches each line of a stream once
    // instead of once per eight edges.  The loads of a lane may run up to three elements past the piece's
    // end (into the next piece, or into the padding behind the arrays); those elements are never used.
    auto fetch = [&](int t, int (&u_out)[4], float (&cf_out)[4]) {
#pragma unroll
        for (int i = 0; i < 4; ++i) { u_out[i] = 0; cf_out[i] = 0.0f; }
        const int j = t + 4 * c;
        if (j < len) {
            const uint32_t pos = begin + uint32_t(j);
            if (narrow) {
                Packed<uint16_t> v;
                __builtin_memcpy(&v, a.idx16 + pos, sizeof(v));
#pragma unroll
                for (int i = 0; i < 4; ++i) u_out[i] = base + int(v.e[i]);
            } else {
                Packed<int32_t> v;
                __builtin_memcpy(&v, HOT ? a.cold_vertices + (pos - a.cold_begin) : a.idx + pos, sizeof(v));
#pragma unroll
                for (int i = 0; i < 4; ++i) u_out[i] = v.e[i];
            }
            if (COEF) {
#pragma unroll
                for (int i = 0; i < 4; ++i) cf_out[i] = 1.0f;
                if (a.w_blk) {
                    Packed<float> v;
                    __builtin_memcpy(&v, a.w_blk + pos, sizeof(v));
#pragma unroll
                    for (int i = 0; i < 4; ++i) cf_out[i] = v.e[i];
                } else if (a.w) {
                    Packed<uint32_t> v;
                    __builtin_memcpy(&v, a.epos + pos, sizeof(v));
#pragma unroll
                    for (int i = 0; i < 4; ++i) cf_out[i] = j + i < len ? a.w[v.e[i]] : 0.0f;
                }
                if (a.scale_blk) {
                    Packed<float> v;
                    __builtin_memcpy(&v, a.scale_blk + pos, sizeof(v));
#pragma unroll
                    for (int i = 0; i < 4; ++i) cf_out[i] *= v.e[i];
                }
            }
        }
    };
    int nxt_u[4];
    float nxt_cf[4];
    fetch(0, nxt_u, nxt_cf);
    for (int t0 = 0; __any(t0 < len); t0 += WINDOW) {
        int my_u[4];
        float my_cf[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) { my_u[i] = nxt_u[i]; my_cf[i] = nxt_cf[i]; }
        fetch(t0 + WINDOW, nxt_u, nxt_cf);
        for (int m = 0; m < WINDOW / U; ++m) {
            const int t = t0 + U * m;
            if (!__any(t < len)) break;
            typename Strip<T, VEC>::raw_t x[U];
            float cf[U];
#pragma unroll
            for (int k = 0; k < U; ++k) {
                const int src = gbase + 2 * m + (k >> 2);
                const int u = __shfl(my_u[k & 3], src);
                if (COEF) cf[k] = __shfl(my_cf[k & 3], src);
                if (t + k < len && (!HOT || lane_ok)) x[k] = Strip<T, VEC>::load(X + int64_t(u) * (HOT ? ld : int64_t(LINE)));
                else x[k] = Strip<T, VEC>::zero();
            }
#pragma unroll
            for (int k = 0; k < U; ++k) {
                float xv[VEC];
                Strip<T, VEC>::unpack(x[k], xv);
#pragma unroll
                for (int i = 0; i < VEC; ++i) {
                    if (COEF) acc[i] = fmaf(t + k < len ? cf[k] : 0.0f, xv[i], acc[i]);
                    else acc[i] += xv[i];
                }
            }
        }
    }
    if (piece < a.n_pieces) {
        float *out = a.partial + (int64_t(slice) * a.n_pieces + slot) * LINE + c * VEC;
#pragma unroll
        for (int i = 0; i < VEC; i += 4) {
            const f32x4 v = {acc[i], acc[i + 1], acc[i + 2], acc[i + 3]};
            __builtin_nontemporal_store(v, reinterpret_cast<f32x4 *>(out + i));
        }
    }
}

// Adds the partial lines of every long row in a fixed order and writes the columns [0, fw) of the
// launch.  L lanes own one (row, slice) pair, 16 bytes of the output row each, so a wavefront
// finishes 64 / L rows of a slice (eight of 128-byte lines).  The sums themselves are formed by eight lane groups together,
// one of their eight pairs after the other: group g of the eight adds the partial lines g, g + 8, g + 16, ... of the pair (a
// load covers eight consecutive lines), and the eight group sums are added pairwise
// (groups 0+1, 2+3, ... then 0..1 + 2..3, ...).  A hub row has thousands of partial lines: added by its
// own lanes alone, one such row set the duration of the launch.
template <typename T, int L>
__global__ void __launch_bounds__(256) blk_finalize_kernel(const int32_t *__restrict__ rows, int64_t n_rows,
                                                           const uint32_t *__restrict__ rowbase,
                                                           const float *__restrict__ partial, int64_t n_pieces, int n_slices,
                                                           const uint32_t *__restrict__ part_base, int64_t n_parts,
                                                           const float *__restrict__ tile_partial, int n_groups, uint32_t inv_groups,
                                                           int64_t tile_group_stride,
                                                           const void *indptr, int ip64, int dst_mode, T *__restrict__ Y,
                                                           int64_t ldy, int fw, int store_vec, int self_mode,
                                                           const OwnRowSrc own,
                                                           const int32_t *__restrict__ col_counts,
                                                           const float *__restrict__ bias, int relu) {
    constexpr int VEC = 16 / int(sizeof(T));  // output columns per lane
    constexpr int LINE = L * VEC;             // columns per slice = floats per partial line
    constexpr int G = 64 / L;                 // lane groups, and pairs, of a wavefront
    const int lane = threadIdx.x & 63;
    const int own_pair = lane / L, c = lane & (L - 1);
    const int g = own_pair & 7;               // of the eight that work together
    const int64_t n_items = n_rows * n_slices;
    const int64_t first_item = ((int64_t(blockIdx.x) * blockDim.x + threadIdx.x) >> 6) * G;  // wave-uniform
    if (first_item >= n_items) return;
    float mine[VEC];  // the sum of this group's own pair
#pragma unroll
    for (int k = 0; k < VEC; ++k) mine[k] = 0.0f;
    for (int j = 0; j < 8; ++j) {
        const int64_t item = first_item + (own_pair & ~7) + j;
        if (item >= n_items) continue;  // the same for the eight groups
        const int64_t i = item % n_rows;
        const int slice = int(item / n_rows);
        const int64_t p0 = rowbase[i], p1 = rowbase[i + 1];
        const float *__restrict__ src = partial + int64_t(slice) * n_pieces * LINE + c * VEC;
        float sum[VEC];
#pragma unroll
        for (int k = 0; k < VEC; ++k) sum[k] = 0.0f;
        auto load_line = [&](int64_t p, f32x4 (&v)[VEC / 4]) {
#pragma unroll
            for (int q = 0; q < VEC / 4; ++q) {
                v[q] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
                if (p < p1) v[q] = __builtin_nontemporal_load(reinterpret_cast<const f32x4 *>(src + p * LINE) + q);
            }
        };
        auto add_line = [&](const f32x4 (&v)[VEC / 4]) {
#pragma unroll
            for (int q = 0; q < VEC / 4; ++q) {
                sum[4 * q] += v[q].x; sum[4 * q + 1] += v[q].y; sum[4 * q + 2] += v[q].z; sum[4 * q + 3] += v[q].w;
            }
        };
        if (tile_partial) {  // first the partial lines of the row's parts gathered from staged tiles, one per group of tiles
            const uint32_t v0 = part_base[i], n_lines = (part_base[i + 1] - v0) * uint32_t(n_groups);
            const float *__restrict__ ts = tile_partial + (int64_t(slice) * n_parts + v0) * LINE + c * VEC;
            auto load_tile_line = [&](uint32_t p, f32x4 (&v)[VEC / 4]) {
                const uint32_t part = n_groups > 1 ? __umulhi(p, inv_groups) : p;  // p / n_groups
                const float *__restrict__ q = ts + int64_t(p - part * uint32_t(n_groups)) * tile_group_stride + int64_t(part) * LINE;
#pragma unroll
                for (int k = 0; k < VEC / 4; ++k) {
                    v[k] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
                    if (p < n_lines) v[k] = *(reinterpret_cast<const f32x4 *>(q) + k);
                }
            };
            for (uint32_t p = uint32_t(g); p < n_lines; p += 32) {
                f32x4 t0[VEC / 4], t1[VEC / 4], t2[VEC / 4], t3[VEC / 4];
                load_tile_line(p, t0); load_tile_line(p + 8, t1); load_tile_line(p + 16, t2); load_tile_line(p + 24, t3);
                add_line(t0); add_line(t1); add_line(t2); add_line(t3);
            }
        }
        for (int64_t p = p0 + g; p < p1; p += 32) {  // four lines per group in flight
            f32x4 v0[VEC / 4], v1[VEC / 4], v2[VEC / 4], v3[VEC / 4];
            load_line(p, v0); load_line(p + 8, v1); load_line(p + 16, v2); load_line(p + 24, v3);
            add_line(v0); add_line(v1); add_line(v2); add_line(v3);
        }
#pragma unroll
        for (int off = L; off < 8 * L; off <<= 1)
#pragma unroll
            for (int k = 0; k < VEC; ++k) sum[k] += __shfl_xor(sum[k], off);
        if (g == j) {
#pragma unroll
            for (int k = 0; k < VEC; ++k) mine[k] = sum[k];
        }
    }
    const int64_t item = first_item + own_pair;
    if (item >= n_items) return;
    const int64_t i = item % n_rows;
    const int slice = int(item / n_rows);
    const int col0 = slice * LINE + c * VEC;
    if (col0 >= fw) return;
    const int64_t row = rows[i];
    const int ncols = fw - col0 < VEC ? fw - col0 : VEC;
    const float ds = scale_of(dst_mode, load_ip(indptr, ip64, row + 1) - load_ip(indptr, ip64, row));
    const float self_cf = self_mode == kSelfInvPlus1 ? scale_of(kScaleInvPlus1, col_counts[row]) : 1.0f;
    float o[VEC];
#pragma unroll
    for (int k = 0; k < VEC; ++k) {
        float v = mine[k];
        if (k < ncols) {
            if (self_mode != kSelfNone) v = fmaf(self_cf, own_row_value<T>(own, row, col0 + k), v);
            v *= ds;
            if (bias) v += bias[col0 + k];
            if (relu) v = v > 0.0f ? v : 0.0f;
        }
        o[k] = v;
    }
    store_strip<T, VEC>(Y + row * ldy + col0, o, ncols, store_vec);
}

// Copies the gathered matrix into rows of whole 16-byte chunks (plan-owned buffer: lines of 128 bytes, power-of-two rows,
// or the groups of a dense tail), so that aligned loads and XCD column slices apply to widths like 100 or 602.  One
// thread per chunk, loaded at the alignment of an element; a row's last, partial chunk is filled up with zeros.
// SCALE (fp32): row v is multiplied by the factor its vertex carries as a gathered row (1/din, 1/sqrt(deg) or
// 1/(din+1)): folding the factor into the copy that happens anyway saves the per-edge factor stream and the
// per-edge multiply of MEAN / SAGE_GCN backward and GCN.
// gathered_only: rows that nobody gathers (counts 0: 43 % of the vertices of the 2.45 M-vertex graph) are left out; the
// launch is bound by the bytes it moves (2.45 M vertices, F=256: 0.95 -> 0.60 ms).
// src_rows: row v of the copy is row src_rows[v] of the matrix (hot tables).
template <typename T, bool SCALE>
__global__ void __launch_bounds__(256) pad_rows_kernel(const T *__restrict__ src, int64_t ld_src, T *__restrict__ dst, int64_t ld_dst,
                                                       int64_t N, int F, int mode, const int32_t *__restrict__ counts,
                                                       const int32_t *__restrict__ row_map, int log2_chunks_per_line,
                                                       int64_t table_stride, int log2_tpr, int gathered_only,
                                                       const int32_t *__restrict__ src_rows) {
    constexpr int W = 16 / int(sizeof(T));
    const int chunks_per_row = (F + W - 1) / W;
    // 2^log2_tpr consecutive threads walk the chunks of one row (no division per chunk)
    const int tpr = 1 << log2_tpr;
    const int64_t rows_per_block = blockDim.x >> log2_tpr;
    const int c0 = threadIdx.x & (tpr - 1);
    for (int64_t row = int64_t(blockIdx.x) * rows_per_block + (threadIdx.x >> log2_tpr); row < N;
         row += int64_t(gridDim.x) * rows_per_block) {
        const int32_t count = (SCALE || gathered_only) ? counts[row] : 0;
        if (gathered_only && count == 0 && row != 0) continue;  // masked lanes may load row 0
        const int64_t drow = row_map ? int64_t(row_map[row]) : row;
        const float f = SCALE ? scale_of(mode, count) : 1.0f;
        const T *in = src + (src_rows ? int64_t(src_rows[row]) : row) * ld_src;
        for (int c = c0; c < chunks_per_row; c += tpr) {
            // row-major: log2_chunks_per_line is 31 (one table); slice-major: one table per line
            const int line = c >> log2_chunks_per_line, within = c - (line << log2_chunks_per_line);
            u32x4 v = {0u, 0u, 0u, 0u};
            const T *p = in + c * W;
            if (c * W + W <= F) {
                v = *reinterpret_cast<const u32x4_any *>(p);
            } else {
#pragma unroll
                for (int i = 0; i < W; ++i) {
                    if (c * W + i < F) {
                        if constexpr (sizeof(T) == 4) v[i] = __float_as_uint(p[i]);
                        else v[i >> 1] |= uint32_t(p[i].bits) << (16 * (i & 1));
                    }
                }
            }
            if constexpr (SCALE && sizeof(T) == 4) {
#pragma unroll
                for (int i = 0; i < 4; ++i) v[i] = __float_as_uint(__uint_as_float(v[i]) * f);
            }
            __builtin_nontemporal_store(v, reinterpret_cast<u32x4 *>(dst + line * table_stride + drow * ld_dst + int64_t(within) * W));
        }
    }
}

// mode: the factor of the rows (kScaleNone: none).  dst is aligned to 16 bytes, ld_dst and table_stride are whole chunks.
template <typename T>
hipError_t launch_pad(const void *src, int64_t ld_src, void *dst, int64_t ld_dst, int64_t N, int64_t F, int mode, const int32_t *counts,
                      hipStream_t stream, const int32_t *row_map = nullptr, int64_t table_stride = 0, bool gathered_only = false,
                      const int32_t *src_rows = nullptr) {
    const int cpr = int((F * int64_t(sizeof(T)) + 15) / 16);
    // threads per row: the power of two (>= 8 threads: one 128-byte line) that leaves the fewest idle slots in the last
    // round over the row's chunks; the widest among equals
    int l = 0;
    int64_t best_waste = INT64_MAX;
    for (int cand = 8; cand >= 3; --cand) {
        const int64_t tpr = int64_t(1) << cand;
        const int64_t waste = (cpr + tpr - 1) / tpr * tpr - cpr;
        if (waste < best_waste) { best_waste = waste; l = cand; }
    }
    if (cpr < 8) l = gnn_ilog2_ceil(cpr);
    const int64_t rows_per_block = 256 >> l;
    int64_t b = (N + rows_per_block - 1) / rows_per_block;
    if (b > (int64_t(1) << 17)) b = int64_t(1) << 17;
    const dim3 grid(static_cast<unsigned>(b > 0 ? b : 1));
    const int chunks_per_line = table_stride > 0 ? 3 : 31;
    if (sizeof(T) == 4 && mode != kScaleNone)
        pad_rows_kernel<T, true><<<grid, 256, 0, stream>>>(static_cast<const T *>(src), ld_src, static_cast<T *>(dst), ld_dst, N, int(F), mode, counts,
                                                           row_map, chunks_per_line, table_stride, l, gathered_only ? 1 : 0, src_rows);
    else
        pad_rows_kernel<T, false><<<grid, 256, 0, stream>>>(static_cast<const T *>(src), ld_src, static_cast<T *>(dst), ld_dst, N, int(F), mode, counts,
                                                            row_map, chunks_per_line, table_stride, l, gathered_only ? 1 : 0, src_rows);
    return hipGetLastError();
}

// ---------------------------------------------------------------- host side
bool has_coop_bin(const AggArgs &a) {
    bool coop = false;
    for (int i = 0; i < a.n_bins; ++i) coop |= (a.bins[i].kind & GNN_BIN_COOP) != 0;
    return coop;
}

// Shared rows on few edges: the launch is too small for the chip (61 K vertices, 3.1 M edges F=8 25.6 -> 22.5 us, F=100 the same; 245 K,
// 12.4 M F=64 weighted 194 -> 200, 1 M, 10 M F=8 95 -> 98).  bf16 also without them, up to 16 lanes per row and four slices a launch (aggregate_kernel -> this, us:
// 100 K, 5 M F=64 57 -> 50, 128 87 -> 79; 200 K, 8 M F=64 84 -> 76, 100 the same; 400 K, 20 M F=100 435 -> 422, 350 1178 -> 1162; 2.45 M, 124 M F=64 1338 ->
// 1265, 128 2446 -> 2375; at worst 2.45 M, 60 M F=250 3060 -> 3105, 1.4 M, 33 M F=400 2598 -> 2636).  32 lanes lose, 100 K, 5 M F=400 304 -> 314, 200 K, 8 M F=250 378
// -> 390, and so do eight slices, 400 K, 20 M F=512 1418 -> 1448, 602 1815 -> 1887, 2.45 M F=500 10.68 -> 10.90 ms.
bool use_gather_kernel(const AggArgs &a, int64_t n_edges, bool bf16, int log2_c) {
    return (has_coop_bin(a) && n_edges <= (int64_t(1) << 22)) || (bf16 && (log2_c == 3 || log2_c == 4) && a.log2_slices < 3);
}

template <typename T>
hipError_t launch_gather(int log2_c, bool coef, dim3 grid, hipStream_t stream, const AggArgs &a) {
    auto launch = [&](auto coop, auto lanes) {
        constexpr bool COOP = decltype(coop)::value;
        constexpr int L = decltype(lanes)::value;
        if (coef) gather_kernel<T, true, COOP, L><<<grid, kBlockThreads, 0, stream>>>(a);
        else gather_kernel<T, false, COOP, L><<<grid, kBlockThreads, 0, stream>>>(a);
    };
    using std::integral_constant;
    if (!has_coop_bin(a)) {
        if constexpr (sizeof(T) == 2) launch(integral_constant<bool, false>(), integral_constant<int, 8>());
        else return hipErrorInvalidValue;
    } else if (log2_c >= 3) launch(integral_constant<bool, true>(), integral_constant<int, 8>());
    else if (log2_c == 2) launch(integral_constant<bool, true>(), integral_constant<int, 4>());
    else if (log2_c == 1) launch(integral_constant<bool, true>(), integral_constant<int, 2>());
    else launch(integral_constant<bool, true>(), integral_constant<int, 1>());
    return hipGetLastError();
}

template <typename T, int VEC, bool COEF>
hipError_t launch_npass(int npass, dim3 grid, hipStream_t stream, const AggArgs &a) {
    const bool coop = has_coop_bin(a);
    if (npass == 1) {
        if (coop) aggregate_kernel<T, VEC, 1, COEF, true><<<grid, kBlockThreads, 0, stream>>>(a);
        else aggregate_kernel<T, VEC, 1, COEF><<<grid, kBlockThreads, 0, stream>>>(a);
    } else {
        if (coop) aggregate_kernel<T, VEC, 2, COEF, true><<<grid, kBlockThreads, 0, stream>>>(a);
        else aggregate_kernel<T, VEC, 2, COEF><<<grid, kBlockThreads, 0, stream>>>(a);
    }
    return hipGetLastError();
}

template <typename T, int VEC>
hipError_t launch_coef(bool coef, int npass, dim3 grid, hipStream_t stream, const AggArgs &a) {
    return coef ? launch_npass<T, VEC, true>(npass, grid, stream, a) : launch_npass<T, VEC, false>(npass, grid, stream, a);
}

hipError_t launch_runs(bool coef, bool bf16, hipStream_t stream, const RunArgs &r) {
    const dim3 grid(static_cast<unsigned>(r.bins.n_blocks));
    if (bf16 && coef) run_kernel<bf16_t, 8, true><<<grid, kBlockThreads, 0, stream>>>(r);
    else if (bf16) run_kernel<bf16_t, 8, false><<<grid, kBlockThreads, 0, stream>>>(r);
    else if (coef) run_kernel<float, 4, true><<<grid, kBlockThreads, 0, stream>>>(r);
    else run_kernel<float, 4, false><<<grid, kBlockThreads, 0, stream>>>(r);
    return hipGetLastError();
}

// Column slices for rows gathered where they lie (no plan-owned copy), counted in 16-byte strips of a row.
//
// Many strips of fp32 on more vertices than the L2s hold rows of: slices of up to 16 strips, for hits in the L2s (100 K
// vertices, 25 edges each: F=250 223 us whole, 199 sliced; 300 K vertices, 50 edges: F=128 574 / 454, F=256 1380 / 979), and
// two slices from 256 bytes on where the hot rows fit only as single lines (1 M vertices, 12 edges, F=64 348 / 307).
//
// Else slices are a matter of latency.  A slice costs a read of the index stream and, off line boundaries, about half a line
// more per edge; with fewer lanes per row a wavefront has more edges of a long row in flight, and on a small graph the chain
// of loads of the longest rows is what a call lasts.  Both are estimated, the lines at the 130 per ns that hits in the
// L2s come in (a row costs as much as 8 edges) and the chain at 0.8 us per step of 8 edges and slot of a quarter row (a
// workgroup shares it), half of it hidden behind the rest, and the number of slices is raised while that wins a tenth.  Measured against the estimate: 10 K
// vertices, 24 edges each, F=100 24 us whole, 15 in four slices; 30 K vertices, 50 edges, F=100 74 us whole, 52 in two slices,
// 62 in four; bf16 F=250 87 / 66 / 74; 60 K vertices, 8 edges, F=64 35 / 22; 100 K vertices, 25 edges, F=100 89 / 97.
int64_t in_place_slices(const gnn_plan *plan, int64_t N, int64_t row_bytes, int64_t strips, int esz, bool lines_ok) {
    if (strips > 512) return (strips + 63) / 64;
    if (!plan || plan->n_edges <= 0) return lines_ok && strips >= 16 ? (strips + 15) / 16 : 1;
    if (N > 49152 && esz == 4) {
        if (strips >= 28) return (strips + 15) / 16;
        if (lines_ok && row_bytes >= 256 && N * row_bytes >= (int64_t(128) << 20)) return 2;
    }
    int64_t longest = plan->n_chunks > 0 ? plan->params.hub_chunk : 0;
    for (int b = plan->n_bins - (plan->n_chunks > 0 ? 2 : 1); b >= 0; --b)
        if (plan->bin_offsets[b + 1] > plan->bin_offsets[b]) {
            const int64_t bound = b < plan->params.n_thresholds ? plan->params.thresholds[b] : plan->bin_edges[b];
            if (bound > longest) longest = bound;
            break;
        }
    int64_t best = 0;
    double best_us = 0.0;
    for (int64_t n = 1; n <= 8; n *= 2) {
        const int64_t per_slice = (strips + n - 1) / n;
        if (n > 1 && per_slice < 5) break;
        const double slice_lines = double(per_slice) * 16.0 / 128.0;
        const double lines = double(n) * (lines_ok ? (slice_lines > 1.0 ? slice_lines : 1.0) : slice_lines + 0.5);
        const double gather_us = double(plan->n_edges + 8 * N) * lines / 130e3;
        const int64_t lanes = int64_t(1) << gnn_ilog2_ceil(per_slice < 64 ? per_slice : 64);
        const double chain_us = 0.8 * double(longest) / 4.0 / (8.0 * double(64 / lanes)) * double((per_slice + 63) / 64);
        const double us = gather_us + (chain_us > 0.5 * gather_us ? chain_us - 0.5 * gather_us : 0.0);
        if (best == 0 || us < 0.9 * best_us) {
            best = n;
            best_us = us;
        }
    }
    return best;
}

// Strips per lane at most.  Rows of three and more fell off: fewer edges in flight per wavefront, and no sharing of long rows
// (100 K vertices, 6 edges each: F=500, two strips per lane, 170 us; F=600, three, 455 us; as two slabs 215).
constexpr int kMaxPass = 2;

// A library-owned second stream per device (default priority, created on first use, kept until the process
// ends): the launches over the short rows run there while the caller's stream sweeps the source blocks of the
// long rows.
hipStream_t overlap_stream() {
    static std::mutex mu;
    static hipStream_t streams[64] = {};
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) return nullptr;
    std::lock_guard<std::mutex> lock(mu);
    if (!streams[dev] && hipStreamCreateWithFlags(&streams[dev], hipStreamNonBlocking) != hipSuccess) streams[dev] = nullptr;
    return streams[dev];
}

// One direction of the aggregation.  `gathered` is X (forward) or dY (backward).  bias / relu:
// the epilogue of a fused layer (out = act(aggregate + bias)), or nullptr / 0.
// no_alloc: the hub partial sums go into the library's fixed device array and the call allocates
// nothing (gnn_aggregate_fwd_noalloc); else into the plan's or the caller's workspace.
int run_aggregate(const void *indptr, const int32_t *indices, const float *w, const void *gathered, void *out,
                  int64_t N, int64_t F, int op, const gnn_opts *opts_in, bool backward, const float *bias = nullptr,
                  int relu = 0, bool no_alloc = false, bool prepacked = false, void *ext_tables = nullptr,
                  int64_t ext_bytes = 0, bool pack_only = false) {
    // prepacked: the gathered matrix already lies in the plan's layout (written there by a producer, see
    // gnn_packed_target_for, or by an earlier pack_only call); `gathered` is not read, no copy is made.
    // ext_tables: that layout lives in the caller's buffer of ext_bytes instead of the plan's.
    // pack_only: write the layout from `gathered` and return.
    gnn_opts o{};
    if (opts_in) o = *opts_in;
    if (no_alloc) {
        // nothing that a plan would have to grow: rows are gathered where they lie, from the caller's index array
        o.flags = (o.flags | GNN_FLAG_NO_PADDED_COPY | GNN_FLAG_NO_COLD_HINTS) &
                  ~(GNN_FLAG_FORCE_PADDED_COPY | GNN_FLAG_FORCE_COLD_HINTS);
        o.workspace = nullptr;
        o.workspace_bytes = 0;
    }
    if (N < 0 || F < 0) return GNN_ERR_INVALID_ARG;
    if (op != GNN_SUM && op != GNN_MEAN && op != GNN_GCN_SYM && op != GNN_SAGE_GCN) return GNN_ERR_INVALID_ARG;
    if (o.dtype != GNN_F32 && o.dtype != GNN_BF16) return GNN_ERR_INVALID_ARG;
    if (o.max_slices != 0 && o.max_slices != 1 && o.max_slices != 2 && o.max_slices != 4 && o.max_slices != 8)
        return GNN_ERR_INVALID_ARG;
    if (N == 0 || F == 0) return GNN_OK;
    if (!indptr || (!gathered && !prepacked) || !out) return GNN_ERR_INVALID_ARG;
    if (N > INT32_MAX || F > INT32_MAX) return GNN_ERR_INVALID_ARG;
    if ((prepacked || pack_only) && !o.plan) return GNN_ERR_UNSUPPORTED;
    if (prepacked && !ext_tables && (o.dtype != GNN_F32 || w)) return GNN_ERR_INVALID_ARG;
    if (prepacked && pack_only) return GNN_ERR_INVALID_ARG;
    if (prepacked) { gathered = nullptr; o.ldx = 0; }
    const int64_t ldx = o.ldx ? o.ldx : F, ldy = o.ldy ? o.ldy : F;
    if (ldx < F || ldy < F) return GNN_ERR_INVALID_ARG;
    gnn_plan *plan = o.plan;
    if (plan && (plan->n_rows != N || plan->indptr_is_64 != (o.indptr_is_64 ? 1 : 0))) return GNN_ERR_INVALID_ARG;
    if (plan && plan->n_edges > 0 && !indices) return GNN_ERR_INVALID_ARG;

    // scaling of the edge terms and of the output row
    int src_mode = kScaleNone, dst_mode = kScaleNone;
    if (op == GNN_MEAN) {
        if (backward) src_mode = kScaleInv; else dst_mode = kScaleInv;
    } else if (op == GNN_GCN_SYM && !w) {
        src_mode = kScaleRsqrt;
        dst_mode = kScaleRsqrt;
    }
    int self_mode = kSelfNone;
    if (op == GNN_SAGE_GCN) {  // (sum + own vector) / (din + 1) and its adjoint
        if (backward) { src_mode = kScaleInvPlus1; self_mode = kSelfInvPlus1; }
        else { dst_mode = kScaleInvPlus1; self_mode = kSelfPlain; }
    }
    if ((src_mode != kScaleNone || self_mode == kSelfInvPlus1) && !plan) return GNN_ERR_UNSUPPORTED;  // needs the column counts a plan holds
    const float *edge_scale = nullptr;

    const int esz = o.dtype == GNN_BF16 ? 2 : 4;
    if (reinterpret_cast<uintptr_t>(gathered) % esz || reinterpret_cast<uintptr_t>(out) % esz) return GNN_ERR_INVALID_ARG;
    const int max_vec = 16 / esz;
    const int64_t line_elems = 128 / esz;

    hipStream_t stream = static_cast<hipStream_t>(o.stream);
    (void)hipGetLastError();  // a stale error of an earlier, failed call must not be blamed on this one

    // Gathered rows that are not whole 128-byte lines (F = 100, 602, or a misaligned base) are
    // first copied into a plan-owned matrix of padded rows: one streaming pass over N*F elements,
    // small next to the E*F gather, buys 16-byte loads and the XCD column slices below.
    int64_t ldg = ldx;  // row stride of the matrix the kernel gathers from
    bool padded = false;
    const gnn_weight_kind weights = gnn_weight_kind_of(plan, w);
    const bool blocks_expected = !(o.flags & GNN_FLAG_NO_SOURCE_BLOCKS) && gnn_call_blocks_expected(plan, esz, F, weights);
    const gnn_layout layout = gnn_choose_layout(plan, N, F, esz, ldx, reinterpret_cast<uintptr_t>(gathered) % 128 == 0,
                                                o.flags, o.max_slices, /*allow_tail=*/o.max_slices != 1,
                                                /*scaled_source=*/src_mode != kScaleNone, blocks_expected, /*weights=*/w != nullptr);
    // what a producer can write into: the slice tables in rank order (the layout gnn_packed_target_for describes)
    if ((prepacked || pack_only) &&
        !(layout.padded_copy && layout.slice_major && !(o.flags & GNN_FLAG_NO_RANK_ORDER) && plan->n_edges > 0))
        return ext_tables ? GNN_ERR_UNSUPPORTED : GNN_ERR_INVALID_ARG;
    const bool slices_wanted = layout.slices_wanted;
    // the caller's matrix stays the source of the own-row term of the hub rows (hub_finalize_kernel)
    const void *orig = gathered;
    const int orig_self_mode = self_mode;
    const char *tail_table = nullptr;
    bool slice_major = false;  // the copy holds one table per 128-byte column slice
    gnn_rank_layout rl{};  // rank layout of the copy (see gnn_plan)
    const int32_t *rank = nullptr, *rank_indices = nullptr;
    void *tables = nullptr;  // the copy: the plan's buffer or the caller's
    bool factor_in_tables = false;
    bool gathered_only = false;  // the copy holds gathered rows only
    if (layout.padded_copy) {
        int rc = GNN_OK;
        if (ext_tables) {
            if (ext_bytes < layout.bytes || reinterpret_cast<uintptr_t>(ext_tables) % 128) return GNN_ERR_INVALID_ARG;
            tables = ext_tables;
        } else {
            rc = gnn_plan_padded(plan, layout.bytes, stream);
            if (rc != GNN_OK) return rc;
            tables = plan->padded.p;
        }
        if (!(o.flags & GNN_FLAG_NO_RANK_ORDER) && plan->n_edges > 0) {
            rc = gnn_plan_rank_indices(plan, indptr, indices, (o.flags & GNN_FLAG_FORCE_COLD_HINTS) != 0, stream, &rl);
            if (rc != GNN_OK) return rc;
            rank = rl.rank;
            rank_indices = rl.indices;
        }
        const bool scale_in_copy = esz == 4 && src_mode != kScaleNone;  // fp32: the factor of the gathered rows goes into the copy
        factor_in_tables = scale_in_copy;
        if ((prepacked || pack_only) && !rank) return GNN_ERR_UNSUPPORTED;
        const int copy_mode = scale_in_copy ? src_mode : int(kScaleNone);
        // copies `ncols` columns starting at `src` into rows of stride dst_ld
        // Rows that nobody gathers are read as own rows only, and those of the forward pass are read where the caller has them, in
        // whole strips (the backward's carry their factor, with the rounding that a caller-kept packed copy has).
        gathered_only = rank && !pack_only && !prepacked && (self_mode == kSelfNone || (self_mode == kSelfPlain && F % max_vec == 0));
        auto copy_part = [&](const char *src, int64_t ncols, char *dst, int64_t dst_ld, int64_t tstride) -> hipError_t {
            if (esz == 4) return launch_pad<float>(src, ldx, dst, dst_ld, N, ncols, copy_mode, plan->col_counts, stream, rank, tstride, gathered_only);
            return launch_pad<bf16_t>(src, ldx, dst, dst_ld, N, ncols, kScaleNone, plan->col_counts, stream, rank, tstride, gathered_only);
        };
        const int64_t main_cols = F - layout.tail_elems;
        char *dst = static_cast<char *>(tables);
        if (!prepacked &&
            copy_part(static_cast<const char *>(gathered), main_cols, dst, layout.ld_pad, layout.table_stride) != hipSuccess)
            return GNN_ERR_LAUNCH;
        if (layout.tail_elems > 0) {
            // behind the main part, a multiple of 128 bytes into the buffer
            char *tail_dst = dst + (layout.slice_major ? layout.main_lines * layout.table_stride : N * layout.ld_pad) * esz;
            if (!prepacked &&
                copy_part(static_cast<const char *>(gathered) + main_cols * esz, layout.tail_elems, tail_dst, layout.tail_ld, 0) != hipSuccess)
                return GNN_ERR_LAUNCH;
            tail_table = tail_dst;
        }
        if (scale_in_copy) {
            src_mode = kScaleNone;
            if (self_mode == kSelfInvPlus1) self_mode = kSelfPlain;  // the own row is already scaled
        }
        if (pack_only) return GNN_OK;
        gathered = tables;
        ldg = layout.ld_pad;
        padded = true;
        slice_major = layout.slice_major;
    }

    if (src_mode != kScaleNone && plan->n_edges > 0) {
        // streamed per-edge factors (built once per plan and mode) instead of a random 4-byte
        // lookup per edge, which would cost a 128-byte line each
        if (no_alloc && !plan->edge_scale[src_mode - 1]) return GNN_ERR_UNSUPPORTED;  // gnn_plan_prepare builds it
        int rc = gnn_plan_edge_scale(plan, indices, src_mode, stream, &edge_scale);
        if (rc != GNN_OK) return rc;
    }
    const bool coef = (w != nullptr) || src_mode != kScaleNone;

    // Loads of 16 bytes whatever the alignment.  Rows that end in padding (the plan's copies, or where the caller vouches
    // for it with GNN_FLAG_PADDED_ROWS) are read past column F; elsewhere the last strip of a row begins early enough
    // to end with it.
    int vec = max_vec;
    const bool rows_padded = padded || ((o.flags & GNN_FLAG_PADDED_ROWS) && ldg % max_vec == 0);
    while (vec > 1 && !rows_padded && vec > F) vec >>= 1;
    const int overlap = !rows_padded && F % vec != 0 ? 1 : 0;
    // Widest non-temporal store the output rows allow.
    int store_vec = overlap ? 1 : vec;
    while (store_vec > 1 && !(ldy % store_vec == 0 && reinterpret_cast<uintptr_t>(out) % (uintptr_t(store_vec) * esz) == 0))
        store_vec >>= 1;

    // hub scratch
    float *partial = nullptr;
    uint32_t *hub_done = nullptr;  // calls that share a plan do not overlap, calls with scratch of their own might
    const bool has_hub = plan && plan->n_chunks > 0;
    if (has_hub) {
        const int64_t need = gnn_plan_workspace_bytes(plan, F);
        if (no_alloc) {
            if (need > int64_t(GNN_NOALLOC_SCRATCH_BYTES)) return GNN_ERR_SCRATCH_CAPACITY;
            const int rc = static_scratch_of_current_device(&partial);
            if (rc != GNN_OK) return rc;
        } else if (o.workspace && o.workspace_bytes >= need) {
            partial = static_cast<float *>(o.workspace);
        } else if (o.workspace) {
            return GNN_ERR_INVALID_ARG;
        } else {
            int rc = gnn_plan_room(plan, plan->scratch, need, stream);
            if (rc != GNN_OK) return rc;
            partial = static_cast<float *>(plan->scratch.p);
            hub_done = plan->hub_done;
        }
        if (reinterpret_cast<uintptr_t>(partial) % 16) return GNN_ERR_INVALID_ARG;
    }

    // Column slices over the XCDs.  Workgroups are handed to the 8 XCDs round-robin by
    // workgroup id, and every XCD has a private L2.  When the gathered rows are whole 128-byte
    // lines, workgroup b of a launch gathers only column slice (b % S): an XCD's L2 then sees one
    // slice of every gathered row instead of whole rows of an eighth of the destinations, so many
    // more hot source rows stay resident.  Slices of the plan's copy are one line wide, those of rows gathered in place
    // as in_place_slices() says, and a row of more than 8 slices is covered by several launches of 8, 4, 2 or 1 slices
    // (column slabs in time),
    // so that every launch keeps all 8 XCDs equally busy.  The price is one read of the index
    // stream per slice.
    struct Segment { int64_t f0, fw; int log2_s; int64_t slice_cols; int tail_slice; };
    // Sliced: at most 256 slices, two or more per launch (one in the last ones), plus the tail; unsliced: slabs.
    constexpr int kMaxSegs = 260;
    Segment segs[kMaxSegs];
    int n_segs = 0;
    {
        const bool lines_ok = (ldg % line_elems == 0) && reinterpret_cast<uintptr_t>(gathered) % 128 == 0;
        const int64_t lines = (F + line_elems - 1) / line_elems;
        const int64_t s_max = o.max_slices > 0 ? o.max_slices : 8;
        // `units` column slices of `unit` columns each, as launches of 8, 4, 2 and 1 of them
        auto add_slices = [&](int64_t units, int64_t unit) {
            for (int64_t u0 = 0; u0 < units;) {
                int ls = 3;
                while (ls > 0 && ((int64_t(1) << ls) > units - u0 || (int64_t(1) << ls) > s_max)) --ls;
                if (n_segs >= kMaxSegs - 1) return false;  // rows this wide take the unsliced route (max_slices = 1)
                Segment &g = segs[n_segs++];
                g.f0 = u0 * unit;
                g.slice_cols = unit;
                g.log2_s = ls;
                const int64_t end = g.f0 + (unit << ls);
                g.fw = (end < F ? end : F) - g.f0;
                g.tail_slice = -1;
                u0 += int64_t(1) << ls;
            }
            return true;
        };
        const int64_t strips = (F + vec - 1) / vec;
        if (padded && lines_ok && lines >= 2 && lines <= 256 && s_max >= 2 && slices_wanted) {
            // The plan's copy: one-line slices.
            // The last one is the dense tail, when there is one.  It gets a launch of its own over all
            // XCDs: gathering 16 bytes costs a cache request per edge like a whole line does, and as one
            // slice among others it kept its share of the XCDs busy nearly as long as a full line
            // (F = 100 as 3 + tail in one launch: 5.77 ms; F = 96: 4.52 ms).
            const int64_t main_lines = tail_table ? lines - 1 : lines;
            if (!add_slices(main_lines, line_elems)) return GNN_ERR_UNSUPPORTED;
            if (tail_table) {
                Segment &g = segs[n_segs++];
                g.f0 = main_lines * line_elems;
                g.slice_cols = layout.tail_ld;  // few column lanes per row group: the lanes go to more edges instead
                g.log2_s = 0;
                g.fw = F - g.f0;
                g.tail_slice = 0;
            }
        } else {
            if (tail_table || slice_major) return GNN_ERR_UNSUPPORTED;  // those layouts are only made for sliced launches
            const int64_t n = padded || !slices_wanted || s_max < 2 ? 1 : in_place_slices(plan, N, F * esz, strips, esz, lines_ok);
            if (n > 1 && n <= 256) {
                // up to 8 in one launch, the last ones of which may be left without columns
                const int64_t per_slice = (strips + n - 1) / n;
                const bool one_launch = n <= s_max && (n & (n - 1)) == 0;
                if (!add_slices(one_launch ? n : (strips + per_slice - 1) / per_slice, per_slice * vec)) return GNN_ERR_UNSUPPORTED;
            } else {
                // whole rows: slabs of at most kMaxPass strips per lane
                const int64_t n_slabs = (strips + 64 * kMaxPass - 1) / (64 * kMaxPass);
                if (n_slabs > kMaxSegs) return GNN_ERR_UNSUPPORTED;
                const int64_t slab = (strips + n_slabs - 1) / n_slabs * vec;
                for (int64_t f0 = 0; f0 < F; f0 += slab) {
                    Segment &g = segs[n_segs++];
                    g.f0 = f0;
                    g.fw = F - f0 < slab ? F - f0 : slab;
                    g.log2_s = 0;
                    g.slice_cols = g.fw;
                    g.tail_slice = -1;
                }
            }
        }
    }

    // Sliced launches of a large power-law graph gather their rarely used sources with
    // non-temporal loads: the plan keeps a copy of the index array with those sources flagged.
    const int32_t *gather_indices = indices;
    if (rank_indices) {
        gather_indices = rank_indices;  // the copy is in rank order; cold sources are flagged there too
    } else if (plan && ((n_segs > 0 && segs[0].log2_s > 0 && !(o.flags & GNN_FLAG_NO_COLD_HINTS)) ||
                        (o.flags & GNN_FLAG_FORCE_COLD_HINTS))) {
        const int32_t *flagged = nullptr;
        int rc = gnn_plan_cold_indices(plan, indices, (o.flags & GNN_FLAG_FORCE_COLD_HINTS) != 0, stream, &flagged);
        if (rc != GNN_OK) return rc;
        if (flagged) gather_indices = flagged;
    }

    // The long rows of a large power-law graph are served as source-blocked pieces (blocked.hip) in
    // every launch that gathers from slice tables, or from the one table of rows of at most a line; the dense tail
    // keeps the plain path.
    gnn_blocked_layout bl{};
    const float *scale_blk = nullptr, *w_blk = nullptr;
    const int lanes = layout.line_lanes;  // of a line of the tables
    gnn_hot_layout hot{};
    const bool hot_tables = layout.hot_tables && gnn_plan_hot_ready(plan, indptr, indices, src_mode, weights, F, esz, stream, /*build=*/false, &hot);
    if (hot_tables) bl = hot.blocks;
    const int64_t table_stride = hot_tables ? hot.rows * line_elems : layout.table_stride;  // of those that the pieces gather from
    const int64_t n_table_lines = hot_tables ? layout.lines : layout.main_lines;
    if (hot_tables) {
        // 27.8 M vertices, 404 M edges, bf16 F=128, a call: 14.9 -> 12.9 ms.  43 % of the gathers, of 203 K rows from 524 K sources, come from LDS
        // and the L2s; copying all rows that are gathered instead, 13.8 ms, 1.85 of them the copy.
        auto copy = [&](auto elem) {
            return launch_pad<decltype(elem)>(gathered, ldx, plan->padded.p, line_elems, hot.rows, F, kScaleNone, nullptr, stream, nullptr, table_stride,
                                              /*gathered_only=*/false, hot.vertices);
        };
        if ((esz == 4 ? copy(float()) : copy(bf16_t())) != hipSuccess) return GNN_ERR_LAUNCH;
        tables = plan->padded.p;
    }
    if (hot_tables || (padded && lanes > 0 && rank_indices && !(o.flags & GNN_FLAG_NO_SOURCE_BLOCKS))) {
        int rc = hot_tables ? GNN_OK : gnn_plan_blocked(plan, indptr, stream, &bl);
        if (rc != GNN_OK) return rc;
        bl.active = bl.active && blocks_expected;
        if (bl.active && edge_scale) {
            rc = gnn_plan_blocked_edge_scale(plan, src_mode, stream, &scale_blk);
            if (rc != GNN_OK) return rc;
        }
        if (bl.active && weights == GNN_WEIGHTS_BOUND) {
            rc = gnn_plan_blocked_bound_weights(plan, stream, &w_blk);
            if (rc != GNN_OK) return rc;
        }
    }
    // The densest source blocks are gathered from tiles staged in LDS (tiles.hip), all column slices in one
    // launch; the pieces of the other blocks follow.
    const gnn_tiles *tl = nullptr;
    const float *tile_coefs = nullptr;
    if (bl.active) {
        int rc = gnn_plan_tiles_with_room(plan, lanes, esz == 2, !coef, int(n_table_lines), lanes * max_vec, stream, &tl);
        if (rc != GNN_OK) return rc;
        if (tl && coef) {
            rc = gnn_plan_tile_coefs(plan, tl, w, edge_scale, src_mode, weights == GNN_WEIGHTS_BOUND, stream, &tile_coefs);
            if (rc != GNN_OK) return rc;
        }
    }
    // Own-row term of the finalisation kernels: from the caller's matrix, or from the plan's layout when a
    // producer wrote the matrix there (then already multiplied by the factor the rows carry).
    const int fin_self_mode = (prepacked && factor_in_tables && orig_self_mode == kSelfInvPlus1) ? int(kSelfPlain) : orig_self_mode;
    auto own_row_src = [&](int64_t f0) {
        OwnRowSrc s{};
        if (orig) {
            s.G = static_cast<const char *>(orig) + f0 * esz;
            s.ldg = ldx;
        } else {
            s.tbl = tables;
            s.table_stride = layout.table_stride;
            s.main_cols = int32_t(F - layout.tail_elems);
            s.tail = tail_table;
            s.tail_ld = layout.tail_ld;
            s.rank = rank;
            s.col_off = int32_t(f0);
        }
        return s;
    };
    bool plain_hub_columns = false;   // some launch left its hub rows to hub_finalize_kernel
    int64_t plain_hub_col_begin = F;  // ... from this column on

    // The short rows of the blocked launches run on a second stream beside the tiles and pieces: they write other rows and
    // read the same tables.  It paid everywhere when pieces and short rows were bound by different things (2.45 M vertices F=100
    // 5.57 -> 5.32 ms); since the tiles took the gathers that hit in the L2s it gains and loses a little.  MEAN forward, ms, on one
    // stream (GNN_FLAG_NO_SHORT_ROW_OVERLAP) -> two: 505 K vertices, 14 M edges F=100 0.566 -> 0.554, 256 1.039 -> 1.000; 2.45 M F=47
    // 2.09 -> 2.11, 100 3.87 -> 3.82, 256 7.47 -> 7.51; 233 K F=64 0.721 -> 0.699, 256 2.60 -> 2.65, 602 6.64 -> 6.93; 133 K, 600 K
    // and 1 M vertices, and bf16 on all of them, within 1 %.
    hipStream_t side = nullptr;
    hipEvent_t fork = nullptr, join = nullptr;
    if (bl.active && !(o.flags & GNN_FLAG_NO_SHORT_ROW_OVERLAP)) {
        side = overlap_stream();
        if (side && (hipEventCreateWithFlags(&fork, hipEventDisableTiming) != hipSuccess ||
                     hipEventCreateWithFlags(&join, hipEventDisableTiming) != hipSuccess)) {
            if (fork) (void)hipEventDestroy(fork);
            fork = join = nullptr;
            side = nullptr;
            (void)hipGetLastError();
        }
        if (side && (hipEventRecord(fork, stream) != hipSuccess || hipStreamWaitEvent(side, fork, 0) != hipSuccess)) {
            (void)hipEventDestroy(fork);
            (void)hipEventDestroy(join);
            return GNN_ERR_LAUNCH;
        }
    }
    auto finish_overlap = [&]() -> bool {  // the caller's stream waits for the second one; true = fine
        if (!side) return true;
        const bool ok = hipEventRecord(join, side) == hipSuccess && hipStreamWaitEvent(stream, join, 0) == hipSuccess;
        (void)hipEventDestroy(fork);  // released by the runtime once the recorded work has completed
        (void)hipEventDestroy(join);
        side = nullptr;
        return ok;
    };

    const int tile_groups = tl ? gnn_tile_groups(tl, int(n_table_lines)) : 0;
    if (tl) {
        const int rc = gnn_launch_tiles(tl, o.dtype == GNN_BF16, hot_tables ? tables : gathered, table_stride * esz, int(n_table_lines),
                                        F - layout.tail_elems, tile_coefs, static_cast<float *>(plan->tile_partial.p), stream);
        if (rc != GNN_OK) { finish_overlap(); return rc; }
    }

    // The pieces of 1 << log2_s column slices from column f0 on, from the slice tables at X_tables, and the sums of the long rows.
    auto launch_pieces = [&](int64_t f0, int64_t fw, int log2_s, const void *X_tables) -> int {
        const int line_floats = lanes * max_vec;
        int rc = gnn_plan_blocked_partial(plan, 1 << log2_s, line_floats, stream);
        if (rc != GNN_OK) return rc;
        PieceArgs pa{};
        pa.pieces = tl ? tl->left.pieces : bl.pieces;
        pa.n_pieces = tl ? tl->left.n_pieces : bl.n_pieces;
        pa.idx = bl.indices;
        pa.epos = bl.epos;
        pa.idx16 = bl.idx16;
        pa.piece_block = tl ? tl->left.piece_block : bl.piece_block;
        pa.n_blocks = bl.n_blocks;
        pa.hot_lines = bl.hot_lines;
        pa.block_lines = bl.block_lines;
        pa.w = w;
        pa.w_blk = w_blk;
        pa.scale_blk = scale_blk;
        pa.X = X_tables;
        pa.slice_stride = table_stride;
        pa.partial = static_cast<float *>(plan->blk_partial.p);
        pa.log2_slices = log2_s;
        if (hot_tables) {
            pa.cold_vertices = hot.cold_vertices;
            pa.cold_begin = uint32_t(hot.cold_begin);
            pa.X_cold = static_cast<const char *>(gathered) + f0 * esz;
            pa.ld_cold = ldg;
            pa.cols = int32_t(fw);
        }
        const int64_t per_block = int64_t(64 / lanes) * kWavesPerBlock;
        const int64_t pblocks = ((pa.n_pieces + per_block - 1) / per_block) << log2_s;
        if (pblocks > INT32_MAX) return GNN_ERR_UNSUPPORTED;
        const int n_sl = 1 << log2_s;
        const dim3 pgrid(static_cast<unsigned>(pblocks)), fgrid(static_cast<unsigned>((bl.n_hot * n_sl * lanes + 255) / 256));
        const int32_t *hot_rows = plan->row_perm + bl.hot_begin;
        const OwnRowSrc own = own_row_src(f0);
        const float *tile_partial = tl ? static_cast<const float *>(plan->tile_partial.p) + f0 / line_elems * tl->n_parts * line_floats : nullptr;
        const int64_t tile_group_stride = tl ? n_table_lines * tl->n_parts * line_floats : 0;
        const uint32_t *rowbase = tl ? tl->left.rowbase : bl.rowbase, *part_base = tl ? tl->part_base : nullptr;
        auto launch = [&](auto elem, auto n_lanes) {
            using T = decltype(elem);
            constexpr int L = decltype(n_lanes)::value;
            if (pa.n_pieces == 0) {}
            else if (L == 8 && hot_tables && coef) piece_kernel<T, true, 8, true><<<pgrid, kBlockThreads, 0, stream>>>(pa);
            else if (L == 8 && hot_tables) piece_kernel<T, false, 8, true><<<pgrid, kBlockThreads, 0, stream>>>(pa);
            else if (coef) piece_kernel<T, true, L><<<pgrid, kBlockThreads, 0, stream>>>(pa);
            else piece_kernel<T, false, L><<<pgrid, kBlockThreads, 0, stream>>>(pa);
            blk_finalize_kernel<T, L><<<fgrid, 256, 0, stream>>>(
                hot_rows, bl.n_hot, rowbase, pa.partial, pa.n_pieces, n_sl, part_base, tl ? tl->n_parts : 0, tile_partial, tile_groups,
                tile_groups > 1 ? uint32_t(((uint64_t(1) << 32) + tile_groups - 1) / tile_groups) : 0u, tile_group_stride, indptr, o.indptr_is_64 ? 1 : 0, dst_mode,
                static_cast<T *>(out) + f0, ldy, int(fw), store_vec, fin_self_mode, own,
                plan->col_counts, bias ? bias + f0 : nullptr, relu);
        };
        auto launch_lanes = [&](auto elem) {
            if (lanes == 8) launch(elem, std::integral_constant<int, 8>());
            else if (lanes == 4) launch(elem, std::integral_constant<int, 4>());
            else launch(elem, std::integral_constant<int, 2>());
        };
        if (o.dtype == GNN_F32) launch_lanes(float());
        else launch_lanes(bf16_t());
        return hipGetLastError() == hipSuccess ? GNN_OK : GNN_ERR_LAUNCH;
    };

    if (hot_tables) {  // in launches of 8, 4, 2 and 1 lines, as below
        for (int64_t l0 = 0; l0 < n_table_lines;) {
            int ls = 3;
            while ((int64_t(1) << ls) > n_table_lines - l0) --ls;
            const int64_t f0 = l0 * line_elems, left = F - f0, fw = line_elems << ls;
            const int rc = launch_pieces(f0, fw < left ? fw : left, ls, static_cast<const char *>(tables) + l0 * table_stride * esz);
            if (rc != GNN_OK) { finish_overlap(); return rc; }
            l0 += int64_t(1) << ls;
        }
    }

    // gather_kernel: 16-byte strips at the alignment of a word, tables whose offsets are 32 bits
    const bool words = esz == 4 || (reinterpret_cast<uintptr_t>(gathered) % 4 == 0 && ldg % 2 == 0 && (!overlap || F % 2 == 0));
    const bool few_bytes = plan && plan->n_edges < (int64_t(1) << 31) && vec == max_vec && words && ldg < (int64_t(1) << 32) && N * (slice_major ? line_elems : ldg) <= kMaxTableBytes / esz;

    // Bins whose rows run_kernel serves: all columns in one launch, beside the tiles and pieces where there are some (2.45 M vertices
    // F=100, 256: 3.62, 7.13 ms in front of the other short rows, 3.93, 7.19 behind them), else behind the other rows (27.8 M bf16
    // 14.8 ms, 15.4 in front).
    const uint32_t run_bins = vec == max_vec && (F + vec - 1) / vec >= GNN_RUN_EDGES
                                  ? gnn_run_bins_of(plan, bl.active ? bl.first_bin : INT32_MAX, esz == 4 && F <= line_elems ? GNN_MORE_RUN_ROWS : GNN_RUN_ROWS)
                                  : 0u;
    RunArgs runs{};
    bool runs_beside = false;

    for (int gi = 0; gi < n_segs; ++gi) {
        const int64_t f0 = segs[gi].f0, fw = segs[gi].fw;
        const int log2_s = segs[gi].log2_s;
        const int64_t slice_cols = segs[gi].slice_cols;
        const int64_t strips = (slice_cols + vec - 1) / vec;
        const int log2_c = strips >= 64 ? 6 : gnn_ilog2_ceil(strips);
        const int C = 1 << log2_c;
        const int npass = int((strips + C - 1) / C);

        AggArgs a{};
        a.indptr = indptr;
        a.indices = gather_indices;
        a.w = w;
        // row-major: the segment starts f0 columns into every row; slice-major: at its first slice table
        a.X = static_cast<const char *>(gathered) + (slice_major ? (f0 / line_elems) * layout.table_stride : f0) * esz;
        a.slice_stride = slice_major ? layout.table_stride : 0;
        a.Y = static_cast<char *>(out) + f0 * esz;
        a.ldx = ldg;
        a.ldy = ldy;
        a.F = int32_t(fw);
        a.ip64 = o.indptr_is_64 ? 1 : 0;
        a.edge_scale = edge_scale;
        a.dst_mode = dst_mode;
        a.self_mode = self_mode;
        a.col_counts = plan ? plan->col_counts : nullptr;
        a.log2_slices = log2_s;
        a.slice_cols = int32_t(slice_cols);
        a.store_vec = store_vec;
        a.overlap = overlap;
        a.row_map = rank_indices ? rank : nullptr;
        a.own_X = gathered_only && self_mode == kSelfPlain ? static_cast<const char *>(orig) + f0 * esz : nullptr;
        a.own_ld = ldx;
        a.p_indptr = rank_indices ? rl.p_indptr : nullptr;
        a.p_chunks = rank_indices ? rl.p_chunks : nullptr;
        a.cold_on = (o.flags & GNN_FLAG_NO_COLD_HINTS) ? 0 : 1;
        // Warm-set size, measured on the 2.45 M-vertex graph: with <= 4 slices per launch (two or more
        // XCDs share a slice) 8 x 32,768 rows is best (F=100: 5.81 ms against 6.03 at 5 x), with 8
        // slices 5-6 x (F=256: 12.18 ms against 12.28 at 8 x and 12.64 at 3 x).
        // Launches of one slice get none: no measurable effect on a whole line, and the dense tail loses
        // with it (8 rows share a line there: F=100 5.70 -> 5.88 ms).
        a.warm_rank = INT32_MAX;
        // With the long rows taken out as source-blocked pieces the hints stopped paying for the short rows that are
        // left (2.45 M vertices: F=100 5.32 -> 5.28 ms without them, F=256 the same either way, as with any warm set
        // from 12 x 32,768 rows up): they are kept for the launches that serve all rows.
        if (rank_indices && rl.cold_pays && log2_s > 0 && !bl.active) a.warm_rank = int32_t(32768) * (log2_s <= 2 ? 8 : 6);
        a.X_tail = tail_table;
        a.ld_tail = layout.tail_ld;
        a.tail_slice = segs[gi].tail_slice;
        a.bias = bias ? bias + f0 : nullptr;
        a.relu = relu;
        if (plan) {
            a.row_perm = plan->row_perm;
            a.row_info = plan->row_info;
            a.chunks = plan->chunks;
            // The scratch rows are F wide for every slab; point at this slab's columns.
            a.partial = partial ? partial + f0 : nullptr;
            a.ldp = gnn_partial_ld(F);
            a.hub_chunk = int32_t(plan->params.hub_chunk);
        }
        const bool blocked = bl.active && segs[gi].tail_slice < 0;
        if (blocked && !hot_tables) {
            const int rc = launch_pieces(f0, fw, log2_s, a.X);
            if (rc != GNN_OK) { finish_overlap(); return rc; }
        }
        hipStream_t rows_stream = (blocked && side) ? side : stream;  // the short rows of a blocked launch may overlap the pieces
        if (gi == 0 && run_bins) {
            runs.a = a;
            runs.a.X = gathered;
            runs.a.Y = out;
            runs.a.F = int32_t(F);
            runs.a.own_X = gathered_only && self_mode == kSelfPlain ? orig : nullptr;
            runs.a.bias = bias;
            runs.a.tail_slice = tail_table ? int32_t(layout.main_lines) : -1;
            gnn_fill_run_bins(runs.bins, plan, run_bins, (F + vec - 1) / vec);
            runs_beside = rows_stream != stream;
            if (runs_beside && launch_runs(coef, o.dtype == GNN_BF16, rows_stream, runs) != hipSuccess) { finish_overlap(); return GNN_ERR_LAUNCH; }
        }
        int32_t nb = 0;
        int64_t next_block = gnn_fill_bins(a.bins, &nb, a.first_block, plan, N, log2_c, blocked ? bl.first_bin : INT32_MAX, 1 << log2_s, run_bins);
        a.n_bins = nb;
        a.hub_done = has_coop_bin(a) ? hub_done : nullptr;  // large launches, whose kernels have no room for it: see hub_finalize_kernel
        if (!blocked && has_hub && !a.hub_done) {
            plain_hub_columns = true;
            if (f0 < plain_hub_col_begin) plain_hub_col_begin = f0;
        }
        if (nb == 0 || next_block == 0) continue;
        next_block <<= log2_s;
        if (next_block > INT32_MAX) { finish_overlap(); return GNN_ERR_UNSUPPORTED; }
        dim3 grid(static_cast<unsigned>(next_block));
        hipError_t err = hipSuccess;
        // (a last segment narrower than a strip begins before its own first column, which an unsigned offset cannot say; the kernel knows no cold sources)
        if (few_bytes && npass == 1 && !(o.flags & GNN_FLAG_FORCE_COLD_HINTS) && (fw >= vec || !overlap) && use_gather_kernel(a, plan->n_edges, o.dtype == GNN_BF16, log2_c)) {
            err = o.dtype == GNN_F32 ? launch_gather<float>(log2_c, coef, grid, rows_stream, a) : launch_gather<bf16_t>(log2_c, coef, grid, rows_stream, a);
        } else if (o.dtype == GNN_F32) {
            if (vec == 4) err = launch_coef<float, 4>(coef, npass, grid, rows_stream, a);
            else if (vec == 2) err = launch_coef<float, 2>(coef, npass, grid, rows_stream, a);
            else err = launch_coef<float, 1>(coef, npass, grid, rows_stream, a);
        } else {
            if (vec == 8) err = launch_coef<bf16_t, 8>(coef, npass, grid, rows_stream, a);
            else if (vec == 4) err = launch_coef<bf16_t, 4>(coef, npass, grid, rows_stream, a);
            else if (vec == 2) err = launch_coef<bf16_t, 2>(coef, npass, grid, rows_stream, a);
            else err = launch_coef<bf16_t, 1>(coef, npass, grid, rows_stream, a);
        }
        if (err != hipSuccess) { finish_overlap(); return GNN_ERR_LAUNCH; }
    }

    if (run_bins && !runs_beside && launch_runs(coef, o.dtype == GNN_BF16, stream, runs) != hipSuccess) { finish_overlap(); return GNN_ERR_LAUNCH; }
    if (!finish_overlap()) return GNN_ERR_LAUNCH;
    if (has_hub && plain_hub_columns) {
        const int64_t hub_begin = plan->bin_offsets[plan->n_bins - 1];
        dim3 grid(static_cast<unsigned>(plan->n_hub_rows));
        if (o.dtype == GNN_F32)
            hub_finalize_kernel<float><<<grid, 256, 0, stream>>>(plan->row_perm + hub_begin, plan->n_hub_rows, plan->hub_chunk_offsets,
                                                                 partial, indptr, o.indptr_is_64 ? 1 : 0, dst_mode,
                                                                 static_cast<float *>(out), ldy, int(F), gnn_partial_ld(F), fin_self_mode,
                                                                 own_row_src(0), plan->col_counts, bias, relu, int(plain_hub_col_begin));
        else
            hub_finalize_kernel<bf16_t><<<grid, 256, 0, stream>>>(plan->row_perm + hub_begin, plan->n_hub_rows, plan->hub_chunk_offsets,
                                                                  partial, indptr, o.indptr_is_64 ? 1 : 0, dst_mode,
                                                                  static_cast<bf16_t *>(out), ldy, int(F), gnn_partial_ld(F), fin_self_mode,
                                                                  own_row_src(0), plan->col_counts, bias, relu, int(plain_hub_col_begin));
        if (hipGetLastError() != hipSuccess) return GNN_ERR_LAUNCH;
    }
    return GNN_OK;
}

}  // namespace

// Copy of an fp32 matrix into rows of another stride (the plan-owned padded matrix; used by ap.hip).
int gnn_pad_rows_f32(const float *src, int64_t ld_src, float *dst, int64_t ld_dst, int64_t N, int64_t F, const int32_t *counts, hipStream_t stream) {
    return launch_pad<float>(src, ld_src, dst, ld_dst, N, F, kScaleNone, counts, stream, nullptr, 0, counts != nullptr) == hipSuccess ? GNN_OK : GNN_ERR_LAUNCH;
}

int gnn_packed_target_for(gnn_plan *plan, const void *indptr, const int32_t *indices, int64_t N, int64_t F, int op, bool backward,
                          bool force, hipStream_t stream, gnn_packed_target *out) {
    *out = gnn_packed_target{};
    if (!plan || !indptr || N <= 0 || F <= 0 || plan->n_rows != N || plan->n_edges <= 0) return GNN_OK;
    int src_mode = kScaleNone;
    if (op == GNN_MEAN && backward) src_mode = kScaleInv;
    else if (op == GNN_GCN_SYM) src_mode = kScaleRsqrt;
    else if (op == GNN_SAGE_GCN && backward) src_mode = kScaleInvPlus1;
    const gnn_layout layout = gnn_choose_layout(plan, N, F, 4, F, true, force ? GNN_FLAG_FORCE_PADDED_COPY : 0, force ? 8 : 0,
                                                /*allow_tail=*/true, /*scaled_source=*/src_mode != kScaleNone,
                                                gnn_plan_blocks_expected(plan, 4, F * 4, false));
    if (!(layout.padded_copy && layout.slice_major)) return GNN_OK;  // that call gathers rows where they lie
    const int64_t lines = (F + 31) / 32;
    if (lines < 2 || lines > 256) return GNN_OK;
    int rc = gnn_plan_padded(plan, layout.bytes, stream);
    if (rc != GNN_OK) return rc;
    gnn_rank_layout rl{};
    rc = gnn_plan_rank_indices(plan, indptr, indices, false, stream, &rl);
    if (rc != GNN_OK) return rc;
    if (!rl.rank) return GNN_OK;
    out->active = true;
    out->base = static_cast<float *>(plan->padded.p);
    out->table_stride = layout.table_stride;
    out->main_cols = int32_t(F - layout.tail_elems);
    out->tail = layout.tail_elems > 0 ? out->base + layout.main_lines * layout.table_stride : nullptr;
    out->tail_ld = layout.tail_ld;
    out->rank = rl.rank;
    out->counts = plan->col_counts;
    out->scale_mode = src_mode;
    return GNN_OK;
}

int gnn_aggregate_prepacked(const void *indptr, const int32_t *indices, void *out, int64_t N, int64_t F, int op,
                            const gnn_opts *opts, bool backward, bool force, const float *bias, int relu) {
    gnn_opts o{};
    if (opts) o = *opts;
    if (force) {
        o.flags |= GNN_FLAG_FORCE_PADDED_COPY;
        o.max_slices = 8;
    }
    return run_aggregate(indptr, indices, nullptr, nullptr, out, N, F, op, &o, backward, bias, relu, /*no_alloc=*/false,
                         /*prepacked=*/true);
}

// Caller-owned packed copies: the layout every packed call uses is the forced one (slice tables in rank
// order whatever the size of the graph), so that the size depends on N, F and the element size only.
static void packed_opts(const gnn_opts *opts, gnn_opts &o) {
    o = gnn_opts{};
    if (opts) o = *opts;
    o.flags = (o.flags | GNN_FLAG_FORCE_PADDED_COPY | GNN_FLAG_NO_DENSE_TAIL) &
              ~(GNN_FLAG_NO_PADDED_COPY | GNN_FLAG_NO_RANK_ORDER | GNN_FLAG_NO_COLUMN_SLICES | GNN_FLAG_NO_SLICE_TABLES);
    o.max_slices = 8;
}

extern "C" GNN_API int64_t gnn_packed_bytes(int64_t N, int64_t F, int dtype) {
    if (N <= 0 || F <= 0 || (dtype != GNN_F32 && dtype != GNN_BF16)) return 0;
    const int64_t esz = dtype == GNN_BF16 ? 2 : 4, line_elems = 128 / esz;
    const int64_t lines = (F + line_elems - 1) / line_elems;
    if (lines < 2 || lines > 256) return 0;  // rows of one line are not laid out as slice tables
    return N * lines * 128;
}

extern "C" GNN_API int gnn_pack_rows(const void *indptr, const int32_t *indices, const void *X, void *packed,
                                     int64_t packed_bytes, int64_t N, int64_t F, int op, int backward, const gnn_opts *opts) {
    gnn_opts o;
    packed_opts(opts, o);
    if (!packed || !X) return (N == 0 || F == 0) ? GNN_OK : GNN_ERR_INVALID_ARG;
    // `packed` stands in for the output argument, which a pack-only call never writes
    return run_aggregate(indptr, indices, nullptr, X, packed, N, F, op, &o, backward != 0, nullptr, 0, /*no_alloc=*/false,
                         /*prepacked=*/false, packed, packed_bytes, /*pack_only=*/true);
}

extern "C" GNN_API int gnn_aggregate_packed(const void *indptr, const int32_t *indices, const float *edge_w, const void *packed,
                                            int64_t packed_bytes, void *Y, int64_t N, int64_t F, int op, int backward,
                                            const gnn_opts *opts) {
    gnn_opts o;
    packed_opts(opts, o);
    if (!packed) return (N == 0 || F == 0) ? GNN_OK : GNN_ERR_INVALID_ARG;
    return run_aggregate(indptr, indices, edge_w, nullptr, Y, N, F, op, &o, backward != 0, nullptr, 0, /*no_alloc=*/false,
                         /*prepacked=*/true, const_cast<void *>(packed), packed_bytes, /*pack_only=*/false);
}

// Forward aggregation with the epilogue of a fused layer (used by layer.hip).
int gnn_aggregate_fwd_epilogue(const void *indptr, const int32_t *indices, const void *X, void *Y, int64_t N, int64_t F,
                               int op, const gnn_opts *opts, const float *bias, int relu) {
    return run_aggregate(indptr, indices, nullptr, X, Y, N, F, op, opts, /*backward=*/false, bias, relu);
}

extern "C" GNN_API int gnn_aggregate_fwd(const void *indptr, const int32_t *indices, const float *edge_w, const void *X,
                                 void *Y, int64_t N, int64_t F, int op, const gnn_opts *opts) {
    return run_aggregate(indptr, indices, edge_w, X, Y, N, F, op, opts, /*backward=*/false);
}

extern "C" GNN_API int gnn_aggregate_fwd_noalloc(const void *indptr, const int32_t *indices, const float *edge_w,
                                                 const void *X, void *Y, int64_t N, int64_t F, int op, const gnn_opts *opts) {
    return run_aggregate(indptr, indices, edge_w, X, Y, N, F, op, opts, /*backward=*/false, nullptr, 0, /*no_alloc=*/true);
}

extern "C" GNN_API int gnn_aggregate_bwd(const void *indptr_t, const int32_t *indices_t, const float *edge_w_t,
                                 const void *dY, void *dX, int64_t N, int64_t F, int op, const gnn_opts *opts) {
    return run_aggregate(indptr_t, indices_t, edge_w_t, dY, dX, N, F, op, opts, /*backward=*/true);
}

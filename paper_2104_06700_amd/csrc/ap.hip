// General aggregation primitive (Section 4.1, Algorithm 1) with the operator table of Table 1:
//
//   f_O[v, j] = reduce_{e = (u -> v) in row v}  binop(f_V[u, j], f_E[e, j])
//
// and its gradients.  Same execution scheme as the sum-only kernels of aggregate.hip -- row
// groups of G lanes (C column lanes x SR edge slots) chosen per degree bin, coalesced index tiles
// handed out by cross-lane shuffles, register accumulation, one owner per output row, hub rows cut
// into pieces that a second kernel combines in order -- with the message and the reduction as
// template parameters.  max / min carry the winning edge position beside the value and combine
// (value, position) pairs lexicographically, so the winner is the lowest position among equals
// whatever the slot layout.  fp32 only; 16-byte accesses at the alignment of a float (the last strip of a row
// begins early enough to end with it: its first columns are computed twice, with equal results), 4-byte ones
// for fewer than four columns.
#include "common.h"

#include <math.h>

#include <type_traits>

namespace {

constexpr int kBlockThreads = 256;
constexpr int kWavesPerBlock = kBlockThreads / 64;

constexpr int kKindHubPieces = GNN_BIN_HUB_PIECES;
using ApBin = gnn_bin_desc;

struct ApArgs {
    const void *indptr;
    const int32_t *indices;
    const int64_t *eid;
    const float *fV;   // gathered vertex operand (forward: f_V; edge gradient: f_V)
    const float *fE;   // edge operand
    const float *dO;   // edge gradient only: gradient of the output rows
    float *out;        // forward: f_O; edge gradient: dfE
    int32_t *arg_out;  // forward, max / min: winning positions (or nullptr)
    int64_t ld_arg;    // row stride of arg_out
    const int32_t *arg_in;  // edge gradient, max / min
    int64_t ldv, lde, ldo;
    int32_t d;
    int32_t ip64;
    const int32_t *row_perm;
    const int4 *row_info;  // see gnn_plan; or nullptr
    const int64_t *chunks;
    float *pval;       // hub pieces: partial values   [n_chunks, ldp]
    int32_t *parg;     // hub pieces: partial winners  [n_chunks, ldp]
    int64_t ldp;
    int32_t n_bins;
    int32_t first_block[GNN_FLAT_BINS];  // see gnn_bin_of_block
    int32_t slab_cols;    // columns one workgroup covers (a multiple of four, or all of them)
    int32_t col0;         // first column of this launch
    int32_t source_split;  // edge dot products: workgroup b takes the (b % 8)-th eighth of its rows
    int32_t col_end;      // one past its last column
    int32_t log2_slices;  // > 0: workgroup b serves column slab (b % n_slices) of the launch, so that an
                          // XCD (workgroups go to the 8 XCDs round-robin) keeps gathering the same lines
                          // of every row; 0: the slab is blockIdx.y
    ApBin bins[GNN_MAX_BINS + 1];
    uint32_t *hub_done;  // see gnn_hub_done; nullptr: ap_hub_finalize_kernel adds the pieces
    int32_t hub_chunk;
    int32_t staged_wave;  // edge gradient by way of LDS: floats of a wavefront's rows
    int32_t stream_edges;  // sums: f_E is beyond all caches
};

// Floats of LDS for `rows` rows of d floats that begin anywhere within 64 bytes.
__host__ __device__ constexpr int staged_floats(int rows, int d) { return (rows * d + 15 + 3) / 4 * 4; }

__device__ __forceinline__ int64_t load_ip(const void *indptr, int ip64, int64_t i) {
    return ip64 ? static_cast<const int64_t *>(indptr)[i]
                : static_cast<int64_t>(static_cast<const int32_t *>(indptr)[i]);
}

typedef float f32x4_any __attribute__((ext_vector_type(4), aligned(4)));
typedef float f32x4_lds __attribute__((ext_vector_type(4)));
typedef int32_t i32x4_any __attribute__((ext_vector_type(4), aligned(4)));
template <int VEC> __device__ __forceinline__ void load_f(const float *p, float (&v)[VEC]) {
    if constexpr (VEC == 4) {
        const f32x4_any t = *reinterpret_cast<const f32x4_any *>(p);
        v[0] = t.x; v[1] = t.y; v[2] = t.z; v[3] = t.w;
    } else {
        v[0] = *p;
    }
}
// non-temporal variant for rows of rarely gathered ("cold") sources
template <int VEC> __device__ __forceinline__ void load_f_nt(const float *p, float (&v)[VEC]) {
    if constexpr (VEC == 4) {
        const f32x4_any t = __builtin_nontemporal_load(reinterpret_cast<const f32x4_any *>(p));
        v[0] = t.x; v[1] = t.y; v[2] = t.z; v[3] = t.w;
    } else {
        v[0] = __builtin_nontemporal_load(p);
    }
}
template <int VEC> __device__ __forceinline__ void store_f(float *p, const float (&v)[VEC]) {
    if constexpr (VEC == 4) *reinterpret_cast<f32x4_any *>(p) = f32x4_any{v[0], v[1], v[2], v[3]};
    else *p = v[0];
}
template <int VEC> __device__ __forceinline__ void load_i(const int32_t *p, int32_t (&v)[VEC]) {
    if constexpr (VEC == 4) {
        const i32x4_any t = *reinterpret_cast<const i32x4_any *>(p);
        v[0] = t.x; v[1] = t.y; v[2] = t.z; v[3] = t.w;
    } else {
        v[0] = *p;
    }
}
template <int VEC> __device__ __forceinline__ void store_i(int32_t *p, const int32_t (&v)[VEC]) {
    if constexpr (VEC == 4) *reinterpret_cast<i32x4_any *>(p) = i32x4_any{v[0], v[1], v[2], v[3]};
    else *p = v[0];
}

// Sum of v over groups of 2^log2_c adjacent lanes, in all of their lanes.  Within 16 lanes the partner's value comes
// through the operand path of the addition (quad swaps, then mirrored halves); a shuffle through the LDS unit costs a
// memory instruction each.
template <int CTRL> __device__ __forceinline__ float add_partner(float v) {
    return v + __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), CTRL, 0xF, 0xF, true));
}
__device__ __forceinline__ float group_sum(float v, int log2_c) {
    if (log2_c > 0) v = add_partner<0xB1>(v);   // quad_perm [1, 0, 3, 2]
    if (log2_c > 1) v = add_partner<0x4E>(v);   // quad_perm [2, 3, 0, 1]
    if (log2_c > 2) v = add_partner<0x141>(v);  // row_half_mirror: lane i of 8 and lane 7 - i
    if (log2_c > 3) v = add_partner<0x140>(v);  // row_mirror: lane i of 16 and lane 15 - i
    if (log2_c > 4) v += __shfl_xor(v, 16);
    if (log2_c > 5) v += __shfl_xor(v, 32);
    return v;
}

__device__ __forceinline__ int64_t shfl_i64(int64_t v, int src_lane) {
    const int lo = __shfl(int(uint32_t(uint64_t(v))), src_lane);
    const int hi = __shfl(int(uint32_t(uint64_t(v) >> 32)), src_lane);
    return int64_t((uint64_t(uint32_t(hi)) << 32) | uint64_t(uint32_t(lo)));
}

// One correctly rounded fp32 operation per message (max / min compare these values with the
// oracle's bit for bit, so nothing may be fused into them).
template <int BIN> __device__ __forceinline__ float message(float x, float y) {
    if constexpr (BIN == GNN_BIN_ADD) return __fadd_rn(x, y);
    else if constexpr (BIN == GNN_BIN_SUB) return __fsub_rn(x, y);
    else if constexpr (BIN == GNN_BIN_MUL) return __fmul_rn(x, y);
    else if constexpr (BIN == GNN_BIN_DIV) return __fdiv_rn(x, y);
    else if constexpr (BIN == GNN_BIN_COPY_LHS) return x;
    else return y;
}

template <int RED> __device__ __forceinline__ bool better(float cand, float best) {
    return RED == GNN_RED_MAX ? cand > best : cand < best;
}

// Which bin a workgroup serves, and the row (or hub piece) and edge range its group owns.
struct Group {
    int G, SR, C, log2_c, lane_in_g, gbase, s, c;
    int64_t row, e0, e1, piece;
    bool is_piece;
    bool coop;  // shared by the wavefronts of the workgroup: e0 .. e1 is this wavefront's quarter
};

// What the way to the first gather needs, loaded together and before the group is looked up: one wait, where the compiler would load
// each at its use (4,096 vertices, F=64: 0.3 us of a sum's 5.6).
struct Near {
    const int4 *row_info;
    const int32_t *indices;
    const float *fV, *fE;
    int64_t ldv, lde;
    __device__ __forceinline__ explicit Near(const ApArgs &a) : ldv(a.ldv), lde(a.lde) {
        auto info = (gnn_global_ptr<int4>)a.row_info;
        auto idx = (gnn_global_ptr<int32_t>)a.indices;
        auto v = (gnn_global_ptr<float>)a.fV, e = (gnn_global_ptr<float>)a.fE;
        asm volatile("" : "+s"(info), "+s"(idx), "+s"(v), "+s"(e), "+s"(ldv), "+s"(lde));
        row_info = (const int4 *)info;
        indices = (const int32_t *)idx;
        fV = (const float *)v;
        fE = (const float *)e;
    }
};

__device__ __forceinline__ Group locate_group(const ApArgs &a, const Near &near, int64_t vblock) {
    Group g;
    const int lane = threadIdx.x & 63;
    const int wave_in_block = threadIdx.x >> 6;
    const int b = gnn_bin_of_block(a.first_block, vblock);
    const ApBin bin = a.bins[b];
    g.coop = (bin.kind & GNN_BIN_COOP) != 0;
    const int64_t wave_in_bin = g.coop ? vblock - bin.first_block : (vblock - bin.first_block) * kWavesPerBlock + wave_in_block;
    g.G = 1 << bin.log2_g;
    g.SR = 1 << bin.log2_sr;
    g.log2_c = bin.log2_g - bin.log2_sr;
    g.C = 1 << g.log2_c;
    g.lane_in_g = lane & (g.G - 1);
    g.gbase = lane - g.lane_in_g;
    g.s = g.lane_in_g >> g.log2_c;
    g.c = g.lane_in_g & (g.C - 1);
    g.row = -1;
    g.e0 = g.e1 = 0;
    g.piece = -1;
    g.is_piece = (bin.kind & kKindHubPieces) != 0;
    if (g.is_piece) {
        if (wave_in_bin < bin.n_items) {
            const int64_t *p = a.chunks + 3 * (bin.item_begin + wave_in_bin);
            g.row = p[0]; g.e0 = p[1]; g.e1 = p[2];
            g.piece = bin.item_begin + wave_in_bin;
        }
    } else {
        const int64_t item = wave_in_bin * (64 >> bin.log2_g) + (lane >> bin.log2_g);
        if (item < bin.n_items) {
            if (near.row_info) {
                const int4 info = near.row_info[bin.item_begin + item];
                g.row = info.x;
                g.e0 = uint32_t(info.y);
                g.e1 = g.e0 + info.z;
            } else {
                g.row = a.row_perm ? int64_t(a.row_perm[bin.item_begin + item]) : bin.item_begin + item;
                g.e0 = load_ip(a.indptr, a.ip64, g.row);
                g.e1 = load_ip(a.indptr, a.ip64, g.row + 1);
            }
        }
    }
    if (g.coop) {
        const int64_t quarter = (g.e1 - g.e0 + kWavesPerBlock - 1) / kWavesPerBlock;
        g.e0 += wave_in_block * quarter;
        if (g.e0 + quarter < g.e1) g.e1 = g.e0 + quarter;
    }
    return g;
}

// ------------------------------------------------------------------ forward
// EWIDE: f_E has one column per feature column (else one scalar per edge).  STREAM: rows of f_E are loaded non-temporally, see kStreamBytes.
template <int BIN, int RED, int VEC, bool EWIDE, bool STREAM = false>
__global__ void __launch_bounds__(kBlockThreads) ap_fwd_kernel(const ApArgs a) {
    const Near near(a);
    constexpr bool USE_V = BIN != GNN_BIN_COPY_RHS;
    constexpr bool USE_E = BIN != GNN_BIN_COPY_LHS;
    constexpr bool WIDE = USE_E && EWIDE;
    constexpr int U = (VEC == 4 && (WIDE || RED != GNN_RED_SUM)) ? 4 : 8;  // edges in flight per slot (fewer where values and winners fill the registers)
    const int slab = a.log2_slices > 0 ? int(blockIdx.x) & ((1 << a.log2_slices) - 1) : int(blockIdx.y);
    const Group g = locate_group(a, near, int64_t(blockIdx.x) >> a.log2_slices);
    const int G = g.G, SR = g.SR;
    int col = a.col0 + slab * a.slab_cols + g.c * VEC;
    const bool col_ok = col < a.col_end && g.c * VEC < a.slab_cols;
    if (VEC > 1 && col > a.col_end - VEC) col = a.col_end - VEC;
    __shared__ float coop_val[kWavesPerBlock - 1][VEC][64];
    __shared__ int32_t coop_win[RED == GNN_RED_SUM ? 1 : kWavesPerBlock - 1][VEC][64];
    const int64_t e0 = g.e0, e1 = g.e1;

    float acc[VEC];
    int32_t win[VEC];
#pragma unroll
    for (int i = 0; i < VEC; ++i) {
        acc[i] = RED == GNN_RED_SUM ? 0.0f : (RED == GNN_RED_MAX ? -INFINITY : INFINITY);
        win[i] = -1;
    }

    auto fetch_tile = [&](int64_t e, int &u_out, float &y_out, int64_t &r_out) {
        u_out = 0; y_out = 1.0f; r_out = 0;
        if (e < e1) {
            u_out = near.indices[e];
            if (USE_E) {
                r_out = a.eid ? a.eid[e] : e;
                if (!EWIDE) y_out = near.fE[r_out * near.lde];
            }
        }
    };
    int nxt_u; float nxt_y; int64_t nxt_r;
    fetch_tile(e0 + g.lane_in_g, nxt_u, nxt_y, nxt_r);
    for (int64_t tile = e0; __any(tile < e1); tile += G) {
        const int my_u = nxt_u;
        const float my_y = nxt_y;
        const int64_t my_r = nxt_r;
        fetch_tile(tile + G + g.lane_in_g, nxt_u, nxt_y, nxt_r);
        const int64_t left = e1 - tile;
        const int n_tile = left < G ? (left > 0 ? int(left) : 0) : G;
        for (int j0 = 0; __any(j0 < n_tile); j0 += SR * U) {
            int u[U];
            float ys[U];
            int64_t r[U];
            bool ok[U];
#pragma unroll
            for (int k = 0; k < U; ++k) {
                const int j = j0 + k * SR + g.s;
                const int src_lane = g.gbase + (j & (G - 1));
                u[k] = __shfl(my_u, src_lane);
                ys[k] = (USE_E && !EWIDE) ? __shfl(my_y, src_lane) : 1.0f;
                r[k] = 0;
                if (WIDE) r[k] = a.eid ? shfl_i64(my_r, src_lane) : tile + j;
                ok[k] = j < n_tile && col_ok;
            }
            float x[U][VEC], y[U][VEC];
#pragma unroll
            for (int k = 0; k < U; ++k) {
#pragma unroll
                for (int i = 0; i < VEC; ++i) { x[k][i] = 0.0f; y[k][i] = ys[k]; }
                if (ok[k]) {
                    if (USE_V) {  // bit 31 of an index flags a cold source (plan-owned index copy, see aggregate.hip)
                        const float *xr = near.fV + int64_t(u[k] & 0x7FFFFFFF) * near.ldv + col;
                        if (u[k] < 0) load_f_nt<VEC>(xr, x[k]);
                        else load_f<VEC>(xr, x[k]);
                    }
                    if (WIDE && STREAM) load_f_nt<VEC>(near.fE + r[k] * near.lde + col, y[k]);
                    else if (WIDE) load_f<VEC>(near.fE + r[k] * near.lde + col, y[k]);
                } else {
#pragma unroll
                    for (int i = 0; i < VEC; ++i) y[k][i] = 1.0f;
                }
            }
#pragma unroll
            for (int k = 0; k < U; ++k) {
                const int32_t pos = int32_t(tile + j0 + k * SR + g.s);
#pragma unroll
                for (int i = 0; i < VEC; ++i) {
                    if constexpr (RED == GNN_RED_SUM) {
                        float m;
                        if constexpr (BIN == GNN_BIN_ADD) m = x[k][i] + y[k][i];
                        else if constexpr (BIN == GNN_BIN_SUB) m = x[k][i] - y[k][i];
                        else if constexpr (BIN == GNN_BIN_MUL) m = x[k][i] * y[k][i];
                        else m = message<BIN>(x[k][i], y[k][i]);
                        acc[i] += ok[k] ? m : 0.0f;
                    } else {
                        const float m = message<BIN>(x[k][i], y[k][i]);
                        if (ok[k] && (win[i] < 0 || better<RED>(m, acc[i]))) { acc[i] = m; win[i] = pos; }
                    }
                }
            }
        }
    }

    // combine the edge slots of the group
    for (int off = g.C; off < G; off <<= 1) {
#pragma unroll
        for (int i = 0; i < VEC; ++i) {
            const float om = __shfl_xor(acc[i], off);
            if constexpr (RED == GNN_RED_SUM) {
                acc[i] += om;
            } else {
                const int32_t ow = __shfl_xor(win[i], off);
                const bool take = ow >= 0 && (win[i] < 0 || better<RED>(om, acc[i]) || (om == acc[i] && ow < win[i]));
                if (take) { acc[i] = om; win[i] = ow; }
            }
        }
    }

    if (g.coop) {  // the wavefronts' quarters in order
        const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
        if (wave > 0) {
#pragma unroll
            for (int i = 0; i < VEC; ++i) {
                coop_val[wave - 1][i][lane] = acc[i];
                if constexpr (RED != GNN_RED_SUM) coop_win[wave - 1][i][lane] = win[i];
            }
        }
        __syncthreads();
        if (wave > 0) return;
        for (int w = 0; w < kWavesPerBlock - 1; ++w) {
#pragma unroll
            for (int i = 0; i < VEC; ++i) {
                const float om = coop_val[w][i][lane];
                if constexpr (RED == GNN_RED_SUM) {
                    acc[i] += om;
                } else {  // later quarters hold later positions: they win only when better
                    const int32_t ow = coop_win[w][i][lane];
                    if (ow >= 0 && (win[i] < 0 || better<RED>(om, acc[i]))) { acc[i] = om; win[i] = ow; }
                }
            }
        }
    }
    if (g.row < 0 || g.s != 0 || !col_ok) return;
    if (g.is_piece) {
        float *val = a.pval + g.piece * a.ldp + col;
        int32_t *arg = a.parg + g.piece * a.ldp + col;
        if (!a.hub_done) {
            store_f<VEC>(val, acc);
            if (RED != GNN_RED_SUM) store_i<VEC>(arg, win);
            return;
        }
#pragma unroll
        for (int i = 0; i < VEC; ++i) {
            gnn_store_for_device(val + i, acc[i]);
            if (RED != GNN_RED_SUM) gnn_store_for_device(arg + i, win[i]);
        }
        const int64_t begin = load_ip(a.indptr, a.ip64, g.row), len = load_ip(a.indptr, a.ip64, g.row + 1) - begin;
        const int number = int((a.chunks[3 * g.piece + 1] - begin) / a.hub_chunk), n = int((len + a.hub_chunk - 1) / a.hub_chunk);
        if (!gnn_hub_done(a.hub_done + 8 * (g.piece - number) + slab, n)) return;
        val -= number * a.ldp;
        arg -= number * a.ldp;
#pragma unroll
        for (int i = 0; i < VEC; ++i) {
            acc[i] = 0.0f;
            win[i] = -1;
        }
        constexpr int P = RED == GNN_RED_SUM ? 4 : 2;  // pieces on their way at a time, in ascending edge order
        for (int q = 0; q < n; q += P) {
            float v[P][VEC];
            int32_t w[P][VEC];
#pragma unroll
            for (int k = 0; k < P; ++k)
#pragma unroll
                for (int i = 0; i < VEC; ++i) {
                    const int64_t at = (q + k < n ? q + k : n - 1) * a.ldp + i;
                    v[k][i] = gnn_load_for_device(val + at);
                    w[k][i] = RED == GNN_RED_SUM ? 0 : gnn_load_for_device(arg + at);
                }
#pragma unroll
            for (int k = 0; k < P; ++k)
#pragma unroll
                for (int i = 0; i < VEC; ++i) {
                    if constexpr (RED == GNN_RED_SUM) acc[i] = q + k < n ? acc[i] + v[k][i] : acc[i];
                    else if (q + k < n && w[k][i] >= 0 && (win[i] < 0 || better<RED>(v[k][i], acc[i]))) { acc[i] = v[k][i]; win[i] = w[k][i]; }
                }
        }
    }
    if (RED != GNN_RED_SUM) {
#pragma unroll
        for (int i = 0; i < VEC; ++i)
            if (win[i] < 0) acc[i] = 0.0f;  // row without edges
        if (a.arg_out) store_i<VEC>(a.arg_out + g.row * a.ld_arg + col, win);
    }
    store_f<VEC>(a.out + g.row * a.ldo + col, acc);
}

struct ApRunArgs {
    const void *indptr;
    const int32_t *indices, *row_perm;
    const int4 *row_info;
    const float *fV;
    float *out;
    int32_t *arg_out;
    int64_t ldv, ldo, ld_arg;
    int32_t d, ip64;
    gnn_run_bins bins;
    const float *tail;  // columns from tail_col on, in rows of ld_tail
    int64_t ld_tail;
    int32_t tail_col;
};

// max / min of the neighbours' vectors for rows of at most GNN_RUN_EDGES edges, all columns, up to 64 rows per wavefront; see run_kernel
// of aggregate.hip.  Two arrays are written here, so writing whole rows counts twice: 2.45 M vertices, three quarters of them such rows,
// d = 100 7.19 -> 6.78 ms; 1 M, 20 M edges 1.23 -> 1.13.
// TAIL: there is a table of the last columns (a lane's table and stride take three registers more, and with them an eighth of the wavefronts).
template <int RED, bool TAIL>
__global__ void __launch_bounds__(kBlockThreads) ap_run_kernel(const ApRunArgs a) {
    const int lane = threadIdx.x & 63;
    const gnn_run_bin bin = gnn_run_bin_of_block(a.bins, blockIdx.x);
    const int64_t item0 = ((int64_t(blockIdx.x) - bin.first_block) * kWavesPerBlock + (threadIdx.x >> 6)) * bin.rows_per_wave;
    const int n_rows = bin.n_items - item0 < bin.rows_per_wave ? int(bin.n_items - item0) : bin.rows_per_wave;
    if (n_rows <= 0) return;
    const int log2_c = a.bins.log2_c, C = 1 << log2_c;
    const int c = lane & (C - 1), gbase = lane & ~(C - 1);
    const int per_set = 64 >> log2_c, in_set = lane >> log2_c;
    int my_row = -1, my_len = 0;
    int64_t my_e0 = 0;
    if (lane < n_rows) {
        const int64_t at = bin.item_begin + item0 + lane;
        if (a.row_info) {
            const int4 info = a.row_info[at];
            my_row = info.x;
            my_e0 = uint32_t(info.y);
            my_len = info.z;
        } else {
            my_row = a.row_perm[at];
            my_e0 = load_ip(a.indptr, a.ip64, my_row);
            my_len = int(load_ip(a.indptr, a.ip64, int64_t(my_row) + 1) - my_e0);
        }
    }
    auto run = [&](auto edges) {
        constexpr int E = decltype(edges)::value;  // edges of a row at most
        for (int strip0 = 0; strip0 * 4 < a.d; strip0 += C) {
            int col = (strip0 + c) * 4;
            const bool col_ok = col < a.d;
            if (col > a.d - 4) col = a.d - 4;
            const bool in_tail = TAIL && col >= a.tail_col;
            const float *table = in_tail ? a.tail + (col - a.tail_col) : a.fV + col;
            const int64_t ld = in_tail ? a.ld_tail : a.ldv;
            auto fetch = [&](int src) {
                const int len = __shfl(my_len, src);
                const int64_t first = shfl_i64(my_e0, src);
                return c < len ? a.indices[first + c] : 0;
            };
            int nxt = E > 0 ? fetch(in_set) : 0;
            for (int set = 0; set < n_rows; set += per_set) {
                const int src = set + in_set;
                const int row = __shfl(my_row, src), len = E > 0 ? __shfl(my_len, src) : 0;
                const int32_t e0 = E > 0 ? int32_t(shfl_i64(my_e0, src)) : 0;
                const int cur = nxt;
                if (E > 0) nxt = fetch((src + per_set) & 63);  // behind the last set: the first one again
                float x[E > 0 ? E : 1][4];
#pragma unroll
                for (int k = 0; k < E; ++k) {
                    const int u = __shfl(cur, gbase + k) & 0x7FFFFFFF;
#pragma unroll
                    for (int i = 0; i < 4; ++i) x[k][i] = 0.0f;
                    if (k < len && col_ok) load_f<4>(table + int64_t(u) * ld, x[k]);
                }
                float best[4] = {0.0f, 0.0f, 0.0f, 0.0f};
                int32_t win[4] = {-1, -1, -1, -1};
#pragma unroll
                for (int k = 0; k < E; ++k)
#pragma unroll
                    for (int i = 0; i < 4; ++i)
                        if (k < len && (k == 0 || better<RED>(x[k][i], best[i]))) { best[i] = x[k][i]; win[i] = e0 + k; }
                if (row >= 0 && col_ok) {
                    store_f<4>(a.out + int64_t(row) * a.ldo + col, best);
                    if (a.arg_out) store_i<4>(a.arg_out + int64_t(row) * a.ld_arg + col, win);
                }
            }
        }
    };
    using std::integral_constant;
    if (bin.longest <= 0) run(integral_constant<int, 0>());
    else if (bin.longest <= 1) run(integral_constant<int, 1>());
    else if (bin.longest <= 4) run(integral_constant<int, 4>());
    else run(integral_constant<int, GNN_RUN_EDGES>());
}

// Combines the pieces of each hub row in ascending edge order and writes the row.
template <int RED>
__global__ void __launch_bounds__(256) ap_hub_finalize_kernel(const int32_t *__restrict__ hub_rows, int64_t n_hub,
                                                              const int64_t *__restrict__ piece_offsets,
                                                              const float *__restrict__ pval, const int32_t *__restrict__ parg,
                                                              int64_t ldp, float *__restrict__ out, int64_t ldo,
                                                              int32_t *__restrict__ arg_out, int64_t ld_arg, int d) {
    const int64_t i = blockIdx.x;
    if (i >= n_hub) return;
    const int64_t row = hub_rows[i];
    const int64_t p0 = piece_offsets[i], p1 = piece_offsets[i + 1];
    for (int col = threadIdx.x; col < d; col += blockDim.x) {
        float best = 0.0f;
        int32_t won = -1;
        for (int64_t p = p0; p < p1; ++p) {
            const float v = pval[p * ldp + col];
            if (RED == GNN_RED_SUM) {
                best += v;
            } else {
                const int32_t w = parg[p * ldp + col];
                if (w >= 0 && (won < 0 || better<RED>(v, best))) { best = v; won = w; }
            }
        }
        out[row * ldo + col] = best;
        if (RED != GNN_RED_SUM && arg_out) arg_out[row * ld_arg + col] = won;
    }
}

// ------------------------------------------------------------ edge gradient
// dfE[r(e), j] = dO[v, j] * d binop / dy, per edge of the forward graph; summed over j when the
// edge operand is a scalar.  MASKED: only where arg_in[v, j] == e (max / min).
// KEEP: when a lane's first strip of dO, the same for all edges, is loaded.
enum KeepGo { kEveryStep, kBeforeFirst, kInFirst };
// STAGED: rows of f_E that follow each other without gaps (no edge ids, stride d <= 4 C).  A group's rows of a step are put together in LDS, at their place
// within a line of 64 bytes, and what fills such a line is stored non-temporally: from the lanes' strips such stores would reach memory as pieces of
// lines (33 columns, add, 12.4 M edges 395 -> 532 us), and plain ones pass through the L2s, where they replace the rows that are gathered.
template <int BIN, int VEC, bool EWIDE, bool MASKED, KeepGo KEEP, int U, bool STAGED = false>  // U: edges in flight per slot
__global__ void __launch_bounds__(kBlockThreads) ap_bwd_edge_kernel(const ApArgs a) {
    static_assert(!STAGED || (VEC == 4 && EWIDE && !MASKED), "whole rows of f_E");
    extern __shared__ __attribute__((aligned(16))) float staged_rows[];
    const Near near(a);
    constexpr bool NEED_X = BIN == GNN_BIN_MUL || BIN == GNN_BIN_DIV;
    constexpr bool NEED_Y = BIN == GNN_BIN_DIV;
    // Four edges in flight per slot where rows are written (us, 2 / 4 / 8: 245 K vertices, 50 edges each 33 columns 694 / 694 / 717, 60 K vertices, 50 each 174 /
    // 162 / 153, 8 columns 36 / 37 / 47).  Their loads come before the first use, else each waited for the one before it and for its store (60 K vertices
    // 33 columns 172 -> 162, 64 239 -> 211; 245 K 61 1107 from 1149; 100 K, 10 each 33 96 -> 80; all before dO was kept from the first step on).
    const Group g = locate_group(a, near, blockIdx.x);
    const int G = g.G, SR = g.SR, C = g.C;
    const int64_t e0 = g.e0, e1 = g.e1;
    const int64_t row = g.row < 0 ? 0 : g.row;

    auto fetch_tile = [&](int64_t e, int &u_out, float &y_out, int64_t &r_out) {
        u_out = 0; y_out = 1.0f; r_out = 0;
        if (e < e1) {
            u_out = near.indices[e];
            r_out = a.eid ? a.eid[e] : e;
            if (NEED_Y && !EWIDE) y_out = near.fE[r_out * near.lde];
        }
    };
    int nxt_u; float nxt_y; int64_t nxt_r;
    fetch_tile(e0 + g.lane_in_g, nxt_u, nxt_y, nxt_r);
    // Beside the rows of the first step is best where rows are written (20,000 vertices, 30 edges each, us, before the indices have arrived, in every step, in
    // the first: 13 columns 19.0, 18.2, 15.6; 33 49.2, 48.2, 38.4; 64 56.4, 56.4, 45.9; 100 K, 10 each 33 80, 81, 64; 5,000, 20 each 29.3, 27.4, 22.3),
    // before them for scalars (245 K, 50 each 33 columns, add, first step 10 % slower).
    float go_first[VEC];
#pragma unroll
    for (int i = 0; i < VEC; ++i) go_first[i] = 0.0f;
    if (KEEP == kBeforeFirst && e0 < e1 && g.c * VEC < a.d)
        load_f<VEC>(a.dO + row * a.ldo + (VEC > 1 && g.c * VEC > a.d - VEC ? a.d - VEC : g.c * VEC), go_first);
    bool load_first = true;
    for (int64_t tile = e0; __any(tile < e1); tile += G) {
        const int my_u = nxt_u;
        const float my_y = nxt_y;
        const int64_t my_r = nxt_r;
        fetch_tile(tile + G + g.lane_in_g, nxt_u, nxt_y, nxt_r);
        const int64_t left = e1 - tile;
        const int n_tile = left < G ? (left > 0 ? int(left) : 0) : G;
        for (int j0 = 0; __any(j0 < n_tile); j0 += SR * U) {
            int u[U];
            float ys[U];
            int64_t r[U];
            bool ok[U];
            float part[U];
#pragma unroll
            for (int k = 0; k < U; ++k) {
                const int j = j0 + k * SR + g.s;
                const int src_lane = g.gbase + (j & (G - 1));
                u[k] = __shfl(my_u, src_lane);
                ys[k] = (NEED_Y && !EWIDE) ? __shfl(my_y, src_lane) : 1.0f;
                r[k] = a.eid ? shfl_i64(my_r, src_lane) : tile + j;
                ok[k] = j < n_tile;
                part[k] = 0.0f;
            }
            // STAGED: this group's rows of the step, at the place within 64 bytes that they have in memory
            const int shift = STAGED ? int((reinterpret_cast<uintptr_t>(a.out) / 4 + uint64_t(tile + j0) * a.d) & 15) : 0;
            float *rows = STAGED ? staged_rows + (threadIdx.x >> 6) * a.staged_wave + g.gbase / G * staged_floats(SR * U, a.d) + shift : nullptr;
            for (int col0 = g.c * VEC; col0 < a.d; col0 += C * VEC) {
                const int col = VEC > 1 && col0 > a.d - VEC ? a.d - VEC : col0;  // columns before col0 belong to the strip before
                float go[VEC], x[U][VEC], y[U][VEC];
                int32_t aw[VEC];
                const bool first_strip = col0 == g.c * VEC;
                if constexpr (KEEP == kInFirst) {
                    if (load_first || !first_strip) load_f<VEC>(a.dO + row * a.ldo + col, go);
#pragma unroll
                    for (int i = 0; i < VEC; ++i) {  // chosen, not branched to: 20,000 vertices, 30 edges each 33 columns 38.4 us, with a branch 50.3
                        if (!load_first && first_strip) go[i] = go_first[i];
                        else if (first_strip) go_first[i] = go[i];
                    }
                } else {
                    if (KEEP == kEveryStep || !first_strip) load_f<VEC>(a.dO + row * a.ldo + col, go);
                    else
#pragma unroll
                        for (int i = 0; i < VEC; ++i) go[i] = go_first[i];
                }
                if (MASKED) load_i<VEC>(a.arg_in + row * int64_t(a.d) + col, aw);
#pragma unroll
                for (int k = 0; k < U; ++k) {  // all loads before the first use
#pragma unroll
                    for (int i = 0; i < VEC; ++i) { x[k][i] = 0.0f; y[k][i] = ys[k]; }
                    if (!ok[k]) continue;
                    if (NEED_X) load_f<VEC>(near.fV + int64_t(u[k]) * near.ldv + col, x[k]);
                    if (NEED_Y && EWIDE) load_f<VEC>(near.fE + r[k] * near.lde + col, y[k]);
                }
#pragma unroll
                for (int k = 0; k < U; ++k) {
                    if (!ok[k]) continue;
                    float gy[VEC];
                    const int32_t pos = int32_t(tile + j0 + k * SR + g.s);
#pragma unroll
                    for (int i = 0; i < VEC; ++i) {
                        float t;
                        if constexpr (BIN == GNN_BIN_ADD || BIN == GNN_BIN_COPY_RHS) t = go[i];
                        else if constexpr (BIN == GNN_BIN_SUB) t = -go[i];
                        else if constexpr (BIN == GNN_BIN_MUL) t = go[i] * x[k][i];
                        else t = -go[i] * x[k][i] / (y[k][i] * y[k][i]);
                        if (MASKED && aw[i] != pos) t = 0.0f;
                        gy[i] = t;
                    }
                    if constexpr (STAGED) {
#pragma unroll
                        for (int i = 0; i < VEC; ++i) rows[(k * SR + g.s) * a.d + col + i] = gy[i];
                    } else if (EWIDE) {
                        store_f<VEC>(a.out + r[k] * near.lde + col, gy);
                    } else {
#pragma unroll
                        for (int i = 0; i < VEC; ++i) part[k] += VEC > 1 && col + i < col0 ? 0.0f : gy[i];
                    }
                }
            }
            if (KEEP == kInFirst) load_first = false;
            if constexpr (STAGED) {
                __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");  // rows of the wavefront's own: its LDS accesses keep their order
                const int n = (n_tile - j0 < SR * U ? n_tile - j0 : SR * U) * a.d;  // floats, from `shift` on
                float *out = a.out + (tile + j0) * a.d - shift;
                for (int b = 4 * g.lane_in_g; n > 0 && b < shift + n; b += 4 * G) {
                    const f32x4_lds v = *reinterpret_cast<const f32x4_lds *>(rows - shift + b);
                    const int line = b & ~15;
                    if (line >= shift && line + 16 <= shift + n) {
                        __builtin_nontemporal_store(f32x4_any(v), reinterpret_cast<f32x4_any *>(out + b));
                        asm volatile("" ::: "memory");  // else the two stores become one, a plain one
                    } else if (b >= shift && b + 4 <= shift + n) {
                        *reinterpret_cast<f32x4_any *>(out + b) = v;
                    } else {
#pragma unroll
                        for (int i = 0; i < 4; ++i)
                            if (b + i >= shift && b + i < shift + n) out[b + i] = v[i];
                    }
                }
                __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
            }
            if (!EWIDE) {
#pragma unroll
                for (int k = 0; k < U; ++k) {
                    const float t = group_sum(part[k], g.log2_c);
                    if (ok[k] && g.c == 0) a.out[r[k] * near.lde] = t;
                }
            }
        }
    }
}

// Dot products: the gradient of a scalar edge operand under multiplication, dfE[r(e)] = sum_j dO[v, j] f_V[u, j], for
// rows of up to 128 columns.  The row of dO stays in registers; C = 2^LC lanes own an edge at a time, S strips of 16 bytes
// each, and C edges go side by side, so that every lane ends with the sum of one edge (halves are exchanged, then quarters,
// then eighths: 7 additions for 8 sums where a reduction of each would take 24) and a wavefront stores 64 consecutive ones.
// Bound by the lines that the L2s deliver, or those behind them.  With a lane per strip the general kernel was bound by
// its instructions: 16 lanes per edge, four reductions and a reload of dO per four edges.  64 columns: 60 K vertices, 2 M
// edges 332 -> 34 us (120 G lines/s), 200 K, 20 M 525 -> 287; 133 K, 79 M 2.09 -> 1.68 ms.  Slabs of 32 columns, added to
// the sums of the slab before, were 9% faster on the last and slower elsewhere.
constexpr int kDotColumns = 128;

template <int CTRL> __device__ __forceinline__ float exchange(bool upper, float lo, float hi) {  // keep one, add the partner's
    return (upper ? hi : lo) + __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(upper ? lo : hi), CTRL, 0xF, 0xF, true));
}

template <int LC, int S, bool RAGGED>  // RAGGED: fewer than 4 * C * S columns
__global__ void __launch_bounds__(kBlockThreads) ap_edge_dot_kernel(const ApArgs a) {
    const Near near(a);
    constexpr int C = 1 << LC;
    // Edges whose loads are in flight, all before the first use: left to itself the compiler kept as few as three (us, 100 K vertices, 1 M edges 33, 64, 100 columns
    // 24.5 -> 22.0, 22.7 -> 22.1, 52.7 -> 41.8; 130 K, 8 M 117 -> 101, 104 -> 103, 277 -> 247; 40 K, 2 M 80 columns 52 -> 48; 245 K, 12.4 M 128 474 -> 481).
    constexpr int H = S <= 2 ? C : C / 2;
    Group g = locate_group(a, near, a.source_split ? blockIdx.x >> 3 : blockIdx.x);
    if (a.source_split) {  // XCD k takes the k-th eighth of a row's edges, in whole steps of the group
        const int64_t k = blockIdx.x & 7u, len = g.e1 - g.e0, first = g.e0;
        auto cut = [&](int64_t i) { return first + (i >= 8 ? len : min(len, ((len * i >> 3) + (g.G >> 1)) & ~int64_t(g.G - 1))); };
        g.e0 = cut(k);
        g.e1 = cut(k + 1);
        if (!__any(g.e0 < g.e1)) return;
    }
    const int lane = threadIdx.x & 63;
    const int slot0 = lane & ~(C - 1);  // first lane of this edge slot
    const int64_t row = g.row < 0 ? 0 : g.row;
    float go[S][4];
    uint32_t col_bytes[S];
    bool own[4];  // columns of the last strip that are not the strip's before it (their products would be counted twice)
#pragma unroll
    for (int s = 0; s < S; ++s) {
        const int col0 = (s * C + g.c) * 4;
        const int col = col0 > a.col_end - 4 ? a.col_end - 4 : col0;  // columns before col0 belong to the strip before, or there are none left
        load_f<4>(a.dO + row * a.ldo + col, go[s]);
#pragma unroll
        for (int i = 0; i < 4; ++i) own[i] = col + i >= col0;
        col_bytes[s] = uint32_t(col) * 4u;
    }
    const char *fV = reinterpret_cast<const char *>(near.fV);
    const uint32_t row_bytes = uint32_t(near.ldv) * 4u;
    // byte offset of the row an edge gathers; edges behind the last one gather row 0, for nothing
    auto fetch = [&](int64_t e) { return e < g.e1 ? uint32_t(near.indices[e]) * row_bytes : 0u; };
    uint32_t nxt = fetch(g.e0 + g.lane_in_g);
    for (int64_t tile = g.e0; __any(tile < g.e1); tile += g.G) {
        const uint32_t mine = nxt;
        const int64_t e = tile + g.lane_in_g;
        float *out = a.out + (a.eid && e < g.e1 ? a.eid[e] : e) * near.lde;
        nxt = fetch(tile + g.G + g.lane_in_g);
        float p[C];
#pragma unroll
        for (int k0 = 0; k0 < C; k0 += H) {
            float x[H][S][4];
#pragma unroll
            for (int k = 0; k < H; ++k) {
                const uint32_t off = uint32_t(__shfl(int(mine), slot0 + k0 + k));
#pragma unroll
                for (int s = 0; s < S; ++s) load_f<4>(reinterpret_cast<const float *>(fV + (off + col_bytes[s])), x[k][s]);
            }
            if constexpr (S > 1) __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int k = 0; k < H; ++k) {
                float t = 0.0f;
#pragma unroll
                for (int s = 0; s < S; ++s)
#pragma unroll
                    for (int i = 0; i < 4; ++i) {
                        const float next = fmaf(go[s][i], x[k][s][i], t);
                        t = !RAGGED || s < S - 1 || own[i] ? next : t;
                    }
                p[k0 + k] = t;
            }
        }
        if constexpr (C == 8) {
#pragma unroll
            for (int i = 0; i < 4; ++i) p[i] = exchange<0x141>(lane & 4, p[i], p[4 + i]);  // lane i of 8 and lane 7 - i
        }
        if constexpr (C >= 4) {
#pragma unroll
            for (int i = 0; i < 2; ++i) p[i] = exchange<0x4E>(lane & 2, p[i], p[2 + i]);
        }
        if constexpr (C >= 2) p[0] = exchange<0xB1>(lane & 1, p[0], p[1]);
        if (e < g.e1) __builtin_nontemporal_store(p[0], out);
    }
}

// ------------------------------------------- vertex gradient of max / min
template <int BIN>
__global__ void __launch_bounds__(256) ap_scatter_arg_kernel(const int32_t *__restrict__ indices, const int64_t *__restrict__ eid,
                                                             const int32_t *__restrict__ arg, const float *__restrict__ dO,
                                                             int64_t ldo, const float *__restrict__ fE, int64_t lde, int ewide,
                                                             float *__restrict__ dfV, int64_t ldv, int64_t N, int d) {
    const int64_t total = N * d;
    const int64_t stride = int64_t(gridDim.x) * blockDim.x;
    for (int64_t t = int64_t(blockIdx.x) * blockDim.x + threadIdx.x; t < total; t += stride) {
        const int64_t v = t / d;
        const int j = int(t - v * d);
        const int32_t e = arg[t];
        if (e < 0) continue;
        float gx = dO[v * ldo + j];
        if (BIN == GNN_BIN_MUL || BIN == GNN_BIN_DIV) {
            const int64_t r = eid ? eid[e] : int64_t(e);
            const float y = fE[r * lde + (ewide ? j : 0)];
            gx = BIN == GNN_BIN_MUL ? gx * y : gx / y;
        }
        unsafeAtomicAdd(dfV + int64_t(indices[e]) * ldv + j, gx);
    }
}

__global__ void __launch_bounds__(256) fill_rows_kernel(float *__restrict__ p, int64_t ld, int64_t n_rows, int d, float value) {
    const int64_t total = n_rows * d;
    const int64_t stride = int64_t(gridDim.x) * blockDim.x;
    for (int64_t t = int64_t(blockIdx.x) * blockDim.x + threadIdx.x; t < total; t += stride) {
        const int64_t v = t / d;
        p[v * ld + (t - v * d)] = value;
    }
}

// ---------------------------------------------------------------- host side
bool aligned4(const void *p) { return reinterpret_cast<uintptr_t>(p) % 4 == 0; }

unsigned grid_1d(int64_t work, int64_t cap = int64_t(1) << 17) {
    int64_t b = (work + 255) / 256;
    if (b < 1) b = 1;
    if (b > cap) b = cap;
    return static_cast<unsigned>(b);
}

// Fills the bin table (heaviest work first) and returns the number of workgroups along x.
int64_t make_bins(ApArgs &a, const gnn_plan *plan, int64_t N, int log2_c, int slices = 1, uint32_t left_out = 0) {
    if (plan) {
        a.row_perm = plan->row_perm;
        a.row_info = plan->row_info;
        a.chunks = plan->chunks;
    }
    return gnn_fill_bins(a.bins, &a.n_bins, a.first_block, plan, N, log2_c, INT32_MAX, slices, left_out);
}

// Calls with a full vector per edge gather one row of f_V per edge too; where rows lie across line boundaries that is a line more than it
// needs.  The copy has rows of the next power of two floats (up to 32 columns) or of whole lines (where the last one holds more than
// 16 columns); it is made on matrices beyond the L2s with enough edges to pay for the pass over them, in a block that the pool keeps.
// The three calls of a message step together, 245 K vertices, 50 edges each, us: 13 columns 1043 -> 990, 20 1273 -> 1208, 31 1805 -> 1597,
// 61 3037 -> 2848; 28 edges each 13 columns 618 -> 600, 61 1779 -> 1720; 16 edges each 341 -> 347, 1093 -> 1105; 60 K vertices, 50 edges
// each, 20 columns 260 -> 264.  A last line of few columns, kept apart in a table of its own, gained nothing (33 columns 1871 -> 1926).
// Where the pool has no block (none to take, or the stream is being captured) the rows are gathered where they lie.
struct AlignedRows {
    float *copy = nullptr;
    hipStream_t stream;
    explicit AlignedRows(hipStream_t s) : stream(s) {}
    AlignedRows(const AlignedRows &) = delete;
    ~AlignedRows() { if (copy) gnn_dev_free_on(copy, stream); }
    int make(ApArgs &a, const gnn_plan *plan, int64_t N, int64_t d, int flags) {
        const bool in_lines = reinterpret_cast<uintptr_t>(a.fV) % 128 == 0 && (a.ldv % 32 == 0 || (a.ldv < 32 && (a.ldv & (a.ldv - 1)) == 0));
        int64_t ld = 16;
        while (ld < d && ld < 32) ld *= 2;
        if (d > 32) ld = (d + 31) / 32 * 32;
        if (!plan || (flags & GNN_FLAG_NO_PADDED_COPY) || in_lines || d < 12 || (d > 32 && d % 32 > 0 && d % 32 <= 16)) return GNN_OK;
        if (N * d * 4 < 12000000 || N * ld * 4 > (int64_t(256) << 20) || plan->n_edges < 24 * N) return GNN_OK;
        if (!gnn_dev_alloc(&copy, N * ld, stream)) { (void)hipGetLastError(); copy = nullptr; return GNN_OK; }
        const int rc = gnn_pad_rows_f32(a.fV, a.ldv, copy, ld, N, d, plan->col_counts, stream);
        if (rc != GNN_OK) return rc;
        a.fV = copy;
        a.ldv = ld;
        return GNN_OK;
    }
};

// Edge gradients whose rows go through LDS and leave as whole lines of 64 bytes, non-temporally (see ap_bwd_edge_kernel): they are more than the caches
// behind the L2s hold, where plain stores would be absorbed, and for products they push the gathered rows out of the L2s.  us, stored from
// the lanes -> so, mul / add, one call after the other (behind a call that has read another such array, whose rows it finds in the caches instead of the
// gathered ones, mul of 33 columns 651 -> 614, 48 812 -> 744, and the forward call behind it 502 -> 467): 245 K vertices, 12.4 M edges 13 columns 327 -> 220 / 180 -> 159, 19 422 -> 332 / 243 -> 223, 32 481 -> 307 / 317 -> 309, 33 689 ->
// 435 / 395 -> 378, 64 957 -> 630 / 620 -> 604; 60 K, 3 M 24 columns (288 MB) 105 -> 72 / 58 -> 69, 33 (396) 154 -> 109 / 97 -> 98; 100 K, 2 M 33 columns (264 MB) 94 -> 73 /
// 55 -> 67, 24 (192) 53 -> 50 / 35 -> 49; 500 K, 6 M 33 383 -> 268 / 225 -> 210.  Not: 25 K, 0.8 M 100 columns (320 MB, a gathered matrix of 10 MB) 143 -> 161 / 87 ->
// 119, 128 152 -> 158 / 103 -> 112; 10 K, 1.5 M 256 357 -> 376 / 300 -> 311; 800 K, 4 M (rows of 5 edges) 64 columns 364 -> 379 / 244 -> 222, 128 685 -> 765, but
// 33 306 -> 291; quotients, bound by their divisions (245 K, 6 M 33 449 -> 477).
bool staged_pays(int binop, int64_t N, int64_t n_edges, int64_t d) {
    if (d < 13 || d > 256 || n_edges > INT64_MAX / 2048) return false;
    const int64_t bytes = n_edges * d * 4;
    if (binop == GNN_BIN_MUL)
        return bytes >= 264000000 && (d <= 64 || (d <= 100 && bytes >= 384000000) || N * d * 4 >= 28000000) && (d <= 48 || n_edges >= 8 * N);
    return binop != GNN_BIN_DIV && bytes >= 384000000 && N >= 50000;
}

// Sums read an f_E of so many bytes non-temporally, so that it does not push the gathered rows out of the L2s (245 K vertices, 12.4 M edges, us, forward and
// vertex gradient through the edge permutation, alone: 33 columns 460 -> 444 and 689 -> 636, 64 692 -> 626 and 716 -> 650; the three calls of a step
// 1764 -> 1728).  Up to there part of it may still be found in the caches behind the L2s by the next call: 19 columns (940 MB) 279 -> 269 alone, a
// step of differences 614 -> 617; 60 K, 3 M 33 columns (396 MB) 112 -> 113, 100 K, 2 M 19 (152 MB) 44 -> 60.
constexpr int64_t kStreamBytes = 1200000000;

struct Common {
    gnn_ap_opts o;
    int64_t ldv, lde, ldo;
    bool ewide;
    hipStream_t stream;
};

int check_common(const gnn_ap_opts *opts_in, int64_t N, int64_t d, int binop, Common &c) {
    c.o = gnn_ap_opts{};
    if (opts_in) c.o = *opts_in;
    if (N < 0 || d < 0 || N > INT32_MAX || d > INT32_MAX) return GNN_ERR_INVALID_ARG;
    if (binop < GNN_BIN_ADD || binop > GNN_BIN_COPY_RHS) return GNN_ERR_INVALID_ARG;
    if (c.o.edge_width != 0 && c.o.edge_width != 1 && c.o.edge_width != d) return GNN_ERR_INVALID_ARG;
    c.ewide = c.o.edge_width != 1 || d == 1;
    const int64_t ew = c.o.edge_width == 1 ? 1 : d;
    c.ldv = c.o.ldv ? c.o.ldv : d;
    c.lde = c.o.lde ? c.o.lde : ew;
    c.ldo = c.o.ldo ? c.o.ldo : d;
    if (c.ldv < d || c.lde < ew || c.ldo < d) return GNN_ERR_INVALID_ARG;
    if (c.o.plan && (c.o.plan->n_rows != N || c.o.plan->indptr_is_64 != (c.o.indptr_is_64 ? 1 : 0))) return GNN_ERR_INVALID_ARG;
    c.stream = static_cast<hipStream_t>(c.o.stream);
    return GNN_OK;
}

template <int BIN, int RED, int VEC>
void launch_fwd_ew(bool ewide, dim3 grid, hipStream_t stream, const ApArgs &a) {
    if constexpr (RED == GNN_RED_SUM && VEC == 4 && BIN != GNN_BIN_COPY_LHS) {
        if (ewide && a.stream_edges) {
            ap_fwd_kernel<BIN, RED, VEC, true, true><<<grid, kBlockThreads, 0, stream>>>(a);
            return;
        }
    }
    if (BIN == GNN_BIN_COPY_LHS || ewide) ap_fwd_kernel<BIN, RED, VEC, true><<<grid, kBlockThreads, 0, stream>>>(a);
    else ap_fwd_kernel<BIN, RED, VEC, false><<<grid, kBlockThreads, 0, stream>>>(a);
}
template <int BIN, int RED>
void launch_fwd_vec(int vec, bool ewide, dim3 grid, hipStream_t stream, const ApArgs &a) {
    if (vec == 4) launch_fwd_ew<BIN, RED, 4>(ewide, grid, stream, a);
    else launch_fwd_ew<BIN, RED, 1>(ewide, grid, stream, a);
}
template <int BIN>
void launch_fwd_red(int red, int vec, bool ewide, dim3 grid, hipStream_t stream, const ApArgs &a) {
    if (red == GNN_RED_SUM) launch_fwd_vec<BIN, GNN_RED_SUM>(vec, ewide, grid, stream, a);
    else if (red == GNN_RED_MAX) launch_fwd_vec<BIN, GNN_RED_MAX>(vec, ewide, grid, stream, a);
    else launch_fwd_vec<BIN, GNN_RED_MIN>(vec, ewide, grid, stream, a);
}
void launch_fwd(int bin, int red, int vec, bool ewide, dim3 grid, hipStream_t stream, const ApArgs &a) {
    switch (bin) {
        case GNN_BIN_ADD: launch_fwd_red<GNN_BIN_ADD>(red, vec, ewide, grid, stream, a); break;
        case GNN_BIN_SUB: launch_fwd_red<GNN_BIN_SUB>(red, vec, ewide, grid, stream, a); break;
        case GNN_BIN_MUL: launch_fwd_red<GNN_BIN_MUL>(red, vec, ewide, grid, stream, a); break;
        case GNN_BIN_DIV: launch_fwd_red<GNN_BIN_DIV>(red, vec, ewide, grid, stream, a); break;
        case GNN_BIN_COPY_LHS: launch_fwd_red<GNN_BIN_COPY_LHS>(red, vec, ewide, grid, stream, a); break;
        default: launch_fwd_red<GNN_BIN_COPY_RHS>(red, vec, ewide, grid, stream, a); break;
    }
}

int run_ap_fwd(const void *indptr, const int32_t *indices, const float *fV, const float *fE, float *fO, int32_t *arg_e,
               int64_t N, int64_t d, int binop, int reduce, const gnn_ap_opts *opts_in) {
    Common c;
    int rc = check_common(opts_in, N, d, binop, c);
    if (rc != GNN_OK) return rc;
    if (reduce < GNN_RED_SUM || reduce > GNN_RED_MIN) return GNN_ERR_INVALID_ARG;
    if (reduce == GNN_RED_SUM && arg_e) return GNN_ERR_INVALID_ARG;
    if (N == 0 || d == 0) return GNN_OK;
    const bool use_v = binop != GNN_BIN_COPY_RHS, use_e = binop != GNN_BIN_COPY_LHS;
    if (!indptr || !fO || (use_v && !fV) || (use_e && !fE)) return GNN_ERR_INVALID_ARG;
    if (!aligned4(fO) || (use_v && !aligned4(fV)) || (use_e && !aligned4(fE)) || (arg_e && !aligned4(arg_e))) return GNN_ERR_INVALID_ARG;
    gnn_plan *plan = c.o.plan;
    if (plan && plan->n_edges > 0 && !indices) return GNN_ERR_INVALID_ARG;
    if (reduce != GNN_RED_SUM && plan && plan->n_edges > INT32_MAX) return GNN_ERR_UNSUPPORTED;
    (void)hipGetLastError();

    const bool wide = use_e && c.ewide;

    // The sum of the neighbours' vectors, plain or weighted by a scalar per edge in CSR order, is
    // the operation of the sum-only path (Alg. 1): that path has the layouts tuned for it.
    // A scalar operand that is strided or reached through an edge-id map (the backward pass over the
    // transposed graph) is first brought into CSR order, one pass over E values into a plan-owned
    // array: the sliced launches then stream it instead of repeating random 4-byte reads per slice.
    if (reduce == GNN_RED_SUM && (binop == GNN_BIN_COPY_LHS || (binop == GNN_BIN_MUL && !wide))) {
        const float *w = nullptr;
        if (binop == GNN_BIN_MUL) {
            w = fE;
            if (c.o.edge_ids || c.lde != 1) {
                w = nullptr;
                if (plan && plan->n_edges > 0) {
                    rc = gnn_plan_edge_operand(plan, fE, c.lde, c.o.edge_ids, indptr, c.o.indptr_is_64 ? 1 : 0, c.stream, &w);
                    if (rc != GNN_OK) return rc;
                }
            }
        }
        if (binop == GNN_BIN_COPY_LHS || w) rc = GNN_OK; else rc = GNN_ERR_UNSUPPORTED;
        gnn_opts g{};
        g.dtype = GNN_F32;
        g.indptr_is_64 = c.o.indptr_is_64;
        g.ldx = c.ldv;
        g.ldy = c.ldo;
        g.stream = c.o.stream;
        g.plan = plan;
        g.flags = c.o.flags;
        g.max_slices = c.o.max_slices;
        if (rc == GNN_OK) rc = gnn_aggregate_fwd(indptr, indices, w, fV, fO, N, d, GNN_SUM, &g);
        if (rc != GNN_ERR_UNSUPPORTED) return rc;  // shapes that path does not take go through the kernel below
    }

    const int vec = d >= 4 ? 4 : 1;

    ApArgs a{};
    a.indptr = indptr;
    a.indices = indices;
    a.eid = c.o.edge_ids;
    a.fV = fV;
    a.fE = fE;
    a.out = fO;
    a.arg_out = arg_e;
    a.ld_arg = d;
    a.ldv = c.ldv;
    a.stream_edges = plan && wide && plan->n_edges >= kStreamBytes / 4 / c.lde ? 1 : 0;
    a.lde = c.lde;
    a.ldo = c.ldo;
    a.d = int32_t(d);
    a.ip64 = c.o.indptr_is_64 ? 1 : 0;
    const bool has_hub = plan && plan->n_chunks > 0;
    if (has_hub) {
        a.ldp = gnn_partial_ld(d);
        rc = gnn_plan_room(plan, plan->scratch, gnn_plan_workspace_bytes(plan, 2 * a.ldp), c.stream);  // values and winners
        if (rc != GNN_OK) return rc;
        a.pval = static_cast<float *>(plan->scratch.p);
        a.parg = reinterpret_cast<int32_t *>(a.pval + plan->n_chunks * a.ldp);
        a.hub_done = plan->hub_done;
        a.hub_chunk = int32_t(plan->params.hub_chunk);
    }

    AlignedRows aligned(c.stream);
    if (use_v && wide) {
        rc = aligned.make(a, plan, N, d, c.o.flags);
        if (rc != GNN_OK) return rc;
    }

    // Gather-bound calls (no full-width edge operand) get the layout of the sum-only hot path:
    // rows copied to an odd number of 128-byte lines when the plan says column slices pay, and
    // one-line column slices spread over the XCD L2s, 8 / 4 / 2 / 1 slices per launch.
    // Not with an edge-id map on a scalar edge operand (every slice would repeat the random 4-byte
    // reads: measured 10.5 -> 16.6 ms at d = 100), nor for max / min with a scalar operand (the
    // repeated weight stream and winner bookkeeping cost more than the hits bring: 8.4 -> 9.0 ms).
    // Rows that ap_run_kernel serves, of more than a line (d = 32: 500 K vertices, 5 M edges 69 -> 75 us, 2.45 M 1666 -> 1642), and enough of them
    // (d = 33, 64, 100, 128, us, rows of ap_fwd_kernel -> ap_run_kernel; short rows of directed power-law graphs of 10 edges per vertex: 338 K 103 -> 113,
    // 128 -> 127, 255 -> 278, 262 -> 256; 423 K 125 -> 130, 164 -> 156, 340 -> 328, 326 -> 326; 861 K 330 -> 294, 351 -> 339, 735 -> 697, 731 -> 668;
    // of symmetric ones: 393 K 295 -> 293, 305 -> 307, 653 -> 637, 633 -> 608; 517 K 480 -> 470, 490 -> 487, 1127 -> 1073, 999 -> 953).
    const uint32_t run_bins = binop == GNN_BIN_COPY_LHS && reduce != GNN_RED_SUM && d > 32 ? gnn_run_bins_of(plan, INT32_MAX, GNN_MORE_RUN_ROWS) : 0u;
    bool sliced = false;
    const float *tail = nullptr;
    int64_t ld_tail = 0, tail_col = INT32_MAX;
    const bool slice_ok = !use_e || (!wide && !c.o.edge_ids && reduce == GNN_RED_SUM) || c.o.max_slices > 1;
    if (use_v && !wide && vec == 4 && plan && plan->n_edges > 0 && slice_ok) {
        const gnn_layout L = gnn_choose_layout(plan, N, d, 4, c.ldv, reinterpret_cast<uintptr_t>(fV) % 128 == 0, c.o.flags,
                                         c.o.max_slices);
        if (L.padded_copy && d * 4 > 128) {  // rows of one line gain nothing from a copy in their own order
            // A last line of few columns in a table of its own, of 16, 32 or 64 bytes a row: as one slab among others it takes as many lines as they do, in
            // a launch over all XCDs the lanes go to more edges, and up to eight rows share a line (us, 2.45 M vertices, 124 M edges 68 columns 5037 -> 4840, 77 5139 ->
            // 5053, 100 6793 -> 6538, 112 6712 -> 6496; 500 K, 40 M 68 1688 -> 1552, 80 1661 -> 1600, 100 2263 -> 2119; 250 K, 20 M 100 944 -> 850; 1.5 M, 28 M 100 1708 ->
            // 1631; rows of 48 bytes, which lie across lines, 1.2 M, 85 M 75 columns 4398 -> 4593).
            const int64_t rest = d % 32;
            bool apart = !use_e && L.slices_wanted && c.o.max_slices == 0 && d > 64 && d <= 256 * 32 && rest >= 4 && rest <= 16 && (rest <= 8 || rest > 12);
            const int64_t ld_apart = ((d - rest) / 32 | 1) * 32, ld_rest = rest <= 4 ? 4 : rest <= 8 ? 8 : 16;
            // The two tables take more than the one where that has an odd number of lines (68 columns: 400 bytes a row, 384): without room, or in a capture of a
            // plan that has room for the one only, it is the one.
            const int64_t apart_bytes = N * (ld_apart + ld_rest) * 4;
            if (apart && apart_bytes > plan->padded.bytes && gnn_capturing(c.stream)) apart = false;
            if (apart) {
                rc = gnn_plan_padded(plan, apart_bytes, c.stream);
                if (rc == GNN_ERR_ALLOC) apart = false;
                else if (rc != GNN_OK) return rc;
            }
            if (!apart && (rc = gnn_plan_padded(plan, N * L.ld_pad * 4, c.stream)) != GNN_OK) return rc;
            const int64_t main_cols = apart ? d - rest : d, ld_main = apart ? ld_apart : L.ld_pad;
            if (apart) ld_tail = ld_rest;
            float *copy = static_cast<float *>(plan->padded.p);
            rc = gnn_pad_rows_f32(fV, c.ldv, copy, ld_main, N, main_cols, plan->col_counts, c.stream);
            if (rc == GNN_OK && apart) {
                tail = copy + N * ld_main;
                tail_col = main_cols;
                rc = gnn_pad_rows_f32(fV + main_cols, c.ldv, copy + N * ld_main, ld_tail, N, rest, plan->col_counts, c.stream);
            }
            if (rc != GNN_OK) return rc;
            a.fV = copy;
            a.ldv = ld_main;
        }
        const int64_t line = 32;  // floats per 128-byte line
        const bool lines_ok = a.ldv % line == 0 && reinterpret_cast<uintptr_t>(a.fV) % 128 == 0;
        const int64_t cols = tail ? tail_col : d, lines = (cols + line - 1) / line;
        int64_t g16 = 1;
        while (g16 < 16 && (a.ldv / line) % (g16 * 2) == 0) g16 *= 2;
        const int64_t unit_lines = g16 >= 8 ? g16 / 4 : 1;  // even strides: wider slices (see aggregate.hip)
        const int64_t units = (lines + unit_lines - 1) / unit_lines;
        if (L.slices_wanted && lines_ok && units >= 2 && units <= 256 && c.o.max_slices != 1) {
            sliced = true;
            if (!(c.o.flags & GNN_FLAG_NO_COLD_HINTS)) {
                const int32_t *flagged = nullptr;
                rc = gnn_plan_cold_indices(plan, indices, (c.o.flags & GNN_FLAG_FORCE_COLD_HINTS) != 0, c.stream, &flagged);
                if (rc != GNN_OK) return rc;
                if (flagged) a.indices = flagged;
            }
            a.slab_cols = int32_t(unit_lines * line);
            const int log2_c = gnn_ilog2_ceil(a.slab_cols / vec);
            int64_t u0 = 0;
            while (u0 < units) {
                const int64_t s_max = c.o.max_slices > 0 ? c.o.max_slices : 8;
                int ls = 3;
                while (ls > 0 && ((int64_t(1) << ls) > units - u0 || (int64_t(1) << ls) > s_max)) --ls;
                a.col0 = int32_t(u0 * a.slab_cols);
                const int64_t end = int64_t(a.col0) + (int64_t(a.slab_cols) << ls);
                a.col_end = int32_t(end < cols ? end : cols);
                a.log2_slices = ls;
                const int64_t blocks = make_bins(a, plan, N, log2_c, 1 << ls, run_bins) << ls;
                if (blocks > INT32_MAX) return GNN_ERR_UNSUPPORTED;
                if (blocks > 0) {
                    launch_fwd(binop, reduce, vec, c.ewide, dim3(static_cast<unsigned>(blocks)), c.stream, a);
                    if (hipGetLastError() != hipSuccess) return GNN_ERR_LAUNCH;
                }
                u0 += int64_t(1) << ls;
            }
            if (tail) {
                ApArgs t = a;
                t.fV = tail - tail_col;
                t.ldv = ld_tail;
                t.slab_cols = int32_t(ld_tail);
                t.col0 = int32_t(tail_col);
                t.col_end = int32_t(d);
                t.log2_slices = 0;
                const int64_t blocks = make_bins(t, plan, N, gnn_ilog2_ceil(ld_tail / vec), 1, run_bins);
                if (blocks > INT32_MAX) return GNN_ERR_UNSUPPORTED;
                if (blocks > 0) {
                    launch_fwd(binop, reduce, vec, c.ewide, dim3(static_cast<unsigned>(blocks)), c.stream, t);
                    if (hipGetLastError() != hipSuccess) return GNN_ERR_LAUNCH;
                }
            }
        }
    }
    if (!sliced) {
        const int64_t strips = (d + vec - 1) / vec;
        const int log2_c = strips >= 64 ? 6 : gnn_ilog2_ceil(strips);
        const int64_t slab_cols = (int64_t(1) << log2_c) * vec;
        const int64_t n_slabs = (d + slab_cols - 1) / slab_cols;
        if (n_slabs > 65535) return GNN_ERR_UNSUPPORTED;
        if (n_slabs > 8) a.hub_done = nullptr;  // a counter per column slice, eight at most
        a.slab_cols = int32_t(slab_cols);
        a.col0 = 0;
        a.col_end = int32_t(d);
        a.log2_slices = 0;
        const int64_t blocks = make_bins(a, plan, N, log2_c, int(n_slabs < 64 ? n_slabs : 64), run_bins);
        if (blocks > INT32_MAX) return GNN_ERR_UNSUPPORTED;
        if (blocks > 0) {
            dim3 grid(static_cast<unsigned>(blocks), static_cast<unsigned>(n_slabs));
            launch_fwd(binop, reduce, vec, c.ewide, grid, c.stream, a);
            if (hipGetLastError() != hipSuccess) return GNN_ERR_LAUNCH;
        }
    }
    if (run_bins) {
        ApRunArgs r{a.indptr, a.indices, a.row_perm, a.row_info, a.fV, a.out, a.arg_out, a.ldv, a.ldo, a.ld_arg, a.d, a.ip64, {}, tail, ld_tail, int32_t(tail_col)};
        gnn_fill_run_bins(r.bins, plan, run_bins, (d + 3) / 4);
        const dim3 grid(static_cast<unsigned>(r.bins.n_blocks));
        auto launch = [&](auto with_tail) {
            constexpr bool TAIL = decltype(with_tail)::value;
            if (reduce == GNN_RED_MAX) ap_run_kernel<GNN_RED_MAX, TAIL><<<grid, kBlockThreads, 0, c.stream>>>(r);
            else ap_run_kernel<GNN_RED_MIN, TAIL><<<grid, kBlockThreads, 0, c.stream>>>(r);
        };
        if (tail) launch(std::true_type());
        else launch(std::false_type());
        if (hipGetLastError() != hipSuccess) return GNN_ERR_LAUNCH;
    }
    if (has_hub && !a.hub_done) {
        const int64_t hub_begin = plan->bin_offsets[plan->n_bins - 1];
        dim3 grid(static_cast<unsigned>(plan->n_hub_rows));
        const int32_t *hub_rows = plan->row_perm + hub_begin;
        if (reduce == GNN_RED_SUM)
            ap_hub_finalize_kernel<GNN_RED_SUM><<<grid, 256, 0, c.stream>>>(hub_rows, plan->n_hub_rows, plan->hub_chunk_offsets, a.pval, a.parg, a.ldp, a.out, a.ldo, a.arg_out, a.ld_arg, int(d));
        else if (reduce == GNN_RED_MAX)
            ap_hub_finalize_kernel<GNN_RED_MAX><<<grid, 256, 0, c.stream>>>(hub_rows, plan->n_hub_rows, plan->hub_chunk_offsets, a.pval, a.parg, a.ldp, a.out, a.ldo, a.arg_out, a.ld_arg, int(d));
        else
            ap_hub_finalize_kernel<GNN_RED_MIN><<<grid, 256, 0, c.stream>>>(hub_rows, plan->n_hub_rows, plan->hub_chunk_offsets, a.pval, a.parg, a.ldp, a.out, a.ldo, a.arg_out, a.ld_arg, int(d));
        if (hipGetLastError() != hipSuccess) return GNN_ERR_LAUNCH;
    }
    return GNN_OK;
}

template <int BIN, int VEC, bool EWIDE>
void launch_edge_masked(bool masked, KeepGo keep, int in_flight, dim3 grid, hipStream_t stream, const ApArgs &a) {
#define GNN_EDGE(MASKED, KEEP, U) ap_bwd_edge_kernel<BIN, VEC, EWIDE, MASKED, KEEP, U><<<grid, kBlockThreads, 0, stream>>>(a)
    if constexpr (EWIDE) {
        if (masked && in_flight == 2) GNN_EDGE(true, kBeforeFirst, 2);
        else if (masked) GNN_EDGE(true, kBeforeFirst, 4);
        else if (keep == kBeforeFirst) GNN_EDGE(false, kBeforeFirst, 4);
        else if (keep == kInFirst) GNN_EDGE(false, kInFirst, 4);
        else GNN_EDGE(false, kEveryStep, 4);
    } else {
        if (masked && in_flight == 2) GNN_EDGE(true, kBeforeFirst, 2);
        else if (masked && keep == kBeforeFirst) GNN_EDGE(true, kBeforeFirst, 4);
        else if (masked) GNN_EDGE(true, kEveryStep, 4);
        else if (in_flight == 2) GNN_EDGE(false, kBeforeFirst, 2);
        else if (keep == kBeforeFirst) GNN_EDGE(false, kBeforeFirst, 4);
        else GNN_EDGE(false, kEveryStep, 4);
    }
#undef GNN_EDGE
}
template <int BIN>
void launch_edge_bin(int vec, bool ewide, bool masked, KeepGo keep, int in_flight, dim3 grid, hipStream_t stream, const ApArgs &a) {
    if (vec == 4) {
        if (ewide) launch_edge_masked<BIN, 4, true>(masked, keep, in_flight, grid, stream, a);
        else launch_edge_masked<BIN, 4, false>(masked, keep, in_flight, grid, stream, a);
    } else {
        if (ewide) launch_edge_masked<BIN, 1, true>(masked, keep, in_flight, grid, stream, a);
        else launch_edge_masked<BIN, 1, false>(masked, keep, in_flight, grid, stream, a);
    }
}

}  // namespace

extern "C" GNN_API int gnn_ap_fwd(const void *indptr, const int32_t *indices, const float *fV, const float *fE, float *fO,
                                  int32_t *arg_e, int64_t N, int64_t d, int binop, int reduce, const gnn_ap_opts *opts) {
    return run_ap_fwd(indptr, indices, fV, fE, fO, arg_e, N, d, binop, reduce, opts);
}

extern "C" GNN_API int gnn_ap_bwd_vertex(const void *indptr_t, const int32_t *indices_t, const float *dO, const float *fE,
                                         float *dfV, int64_t N, int64_t d, int binop, const gnn_ap_opts *opts) {
    Common c;
    int rc = check_common(opts, N, d, binop, c);
    if (rc != GNN_OK) return rc;
    if (N == 0 || d == 0) return GNN_OK;
    if (!dfV || !aligned4(dfV)) return GNN_ERR_INVALID_ARG;
    // the gathered operand is dO (stride ldo), the output dfV (stride ldv): swap the two strides
    gnn_ap_opts t = c.o;
    t.ldv = c.ldo;
    t.ldo = c.ldv;
    switch (binop) {
        case GNN_BIN_COPY_RHS:
            (void)hipGetLastError();
            fill_rows_kernel<<<grid_1d(N * d), 256, 0, c.stream>>>(dfV, c.ldv, N, int(d), 0.0f);
            return hipGetLastError() == hipSuccess ? GNN_OK : GNN_ERR_LAUNCH;
        case GNN_BIN_MUL:
        case GNN_BIN_DIV:
            return run_ap_fwd(indptr_t, indices_t, dO, fE, dfV, nullptr, N, d, binop, GNN_RED_SUM, &t);
        default:  // add, sub, copylhs: d/dx = 1
            return run_ap_fwd(indptr_t, indices_t, dO, nullptr, dfV, nullptr, N, d, GNN_BIN_COPY_LHS, GNN_RED_SUM, &t);
    }
}

extern "C" GNN_API int gnn_ap_bwd_vertex_arg(const int32_t *indices, const int32_t *arg_e, const float *dO, const float *fE,
                                             float *dfV, int64_t n_vertex_rows, int64_t N, int64_t d, int binop,
                                             const gnn_ap_opts *opts) {
    return gnn_ap_bwd_vertex_arg_edges(indices, arg_e, dO, fE, dfV, n_vertex_rows, N, d, binop, 0, opts);
}

extern "C" GNN_API int gnn_ap_bwd_vertex_arg_edges(const int32_t *indices, const int32_t *arg_e, const float *dO, const float *fE,
                                                   float *dfV, int64_t n_vertex_rows, int64_t N, int64_t d, int binop,
                                                   int64_t n_edges, const gnn_ap_opts *opts) {
    Common c;
    gnn_ap_opts o{};
    if (opts) o = *opts;
    o.plan = nullptr;  // not used here
    int rc = check_common(&o, N, d, binop, c);
    if (rc != GNN_OK) return rc;
    if (n_vertex_rows < 0) return GNN_ERR_INVALID_ARG;
    if (d == 0) return GNN_OK;
    if (!dfV || !aligned4(dfV)) return GNN_ERR_INVALID_ARG;
    (void)hipGetLastError();
    const bool need_y = binop == GNN_BIN_MUL || binop == GNN_BIN_DIV;
    if (binop != GNN_BIN_COPY_RHS && indices && arg_e && dO && (fE || !need_y) && gnn_winners_apply(n_edges, n_vertex_rows, N, d)) {
        rc = gnn_scatter_winners(indices, c.o.edge_ids, arg_e, dO, c.ldo, fE, c.lde, c.ewide, dfV, c.ldv, n_vertex_rows, N, d, binop, c.stream);
        if (rc != GNN_ERR_ALLOC) return rc;
    }
    if (n_vertex_rows > 0) fill_rows_kernel<<<grid_1d(n_vertex_rows * d), 256, 0, c.stream>>>(dfV, c.ldv, n_vertex_rows, int(d), 0.0f);
    if (hipGetLastError() != hipSuccess) return GNN_ERR_LAUNCH;
    if (N == 0 || binop == GNN_BIN_COPY_RHS) return GNN_OK;
    if (!indices || !arg_e || !dO || (need_y && !fE)) return GNN_ERR_INVALID_ARG;
    const unsigned grid = grid_1d(N * d);
    const int ew = c.ewide ? 1 : 0;
    if (binop == GNN_BIN_MUL)
        ap_scatter_arg_kernel<GNN_BIN_MUL><<<grid, 256, 0, c.stream>>>(indices, c.o.edge_ids, arg_e, dO, c.ldo, fE, c.lde, ew, dfV, c.ldv, N, int(d));
    else if (binop == GNN_BIN_DIV)
        ap_scatter_arg_kernel<GNN_BIN_DIV><<<grid, 256, 0, c.stream>>>(indices, c.o.edge_ids, arg_e, dO, c.ldo, fE, c.lde, ew, dfV, c.ldv, N, int(d));
    else
        ap_scatter_arg_kernel<GNN_BIN_COPY_LHS><<<grid, 256, 0, c.stream>>>(indices, c.o.edge_ids, arg_e, dO, c.ldo, fE, c.lde, ew, dfV, c.ldv, N, int(d));
    return hipGetLastError() == hipSuccess ? GNN_OK : GNN_ERR_LAUNCH;
}

extern "C" GNN_API int gnn_ap_bwd_edge(const void *indptr, const int32_t *indices, const int32_t *arg_e, const float *fV,
                                       const float *fE, const float *dO, float *dfE, int64_t N, int64_t d, int binop,
                                       const gnn_ap_opts *opts) {
    Common c;
    int rc = check_common(opts, N, d, binop, c);
    if (rc != GNN_OK) return rc;
    if (binop == GNN_BIN_COPY_LHS) return GNN_ERR_INVALID_ARG;
    if (N == 0 || d == 0) return GNN_OK;
    const bool need_x = binop == GNN_BIN_MUL || binop == GNN_BIN_DIV, need_y = binop == GNN_BIN_DIV;
    if (!indptr || !dO || !dfE || (need_x && !fV) || (need_y && !fE)) return GNN_ERR_INVALID_ARG;
    if (!aligned4(dO) || !aligned4(dfE) || (need_x && !aligned4(fV)) || (need_y && !aligned4(fE)) || (arg_e && !aligned4(arg_e)))
        return GNN_ERR_INVALID_ARG;
    gnn_plan *plan = c.o.plan;
    if (plan && plan->n_edges > 0 && !indices) return GNN_ERR_INVALID_ARG;
    if (arg_e && plan && plan->n_edges > INT32_MAX) return GNN_ERR_UNSUPPORTED;
    (void)hipGetLastError();

    const bool masked = arg_e != nullptr;
    const bool dots = binop == GNN_BIN_MUL && !c.ewide && !masked && d >= 4 && d <= kDotColumns && N * c.ldv * 4 < (int64_t(1) << 32);  // 32-bit offsets
    const int vec = d >= 4 ? 4 : 1;
    const int64_t strips = (d + vec - 1) / vec;
    int log2_c = strips >= 64 ? 6 : gnn_ilog2_ceil(strips);
    if (dots && log2_c > 3) log2_c = 3;

    ApArgs a{};
    a.indptr = indptr;
    a.indices = indices;
    a.eid = c.o.edge_ids;
    a.fV = fV;
    a.fE = fE;
    a.dO = dO;
    a.out = dfE;
    a.arg_in = arg_e;
    a.ldv = c.ldv;
    a.lde = c.lde;
    a.ldo = c.ldo;
    a.d = int32_t(d);
    a.ip64 = c.o.indptr_is_64 ? 1 : 0;
    AlignedRows aligned(c.stream);
    if (need_x && c.ewide) {
        rc = aligned.make(a, plan, N, d, c.o.flags);
        if (rc != GNN_OK) return rc;
    }
    const int64_t blocks = make_bins(a, plan, N, log2_c);
    if (blocks > INT32_MAX) return GNN_ERR_UNSUPPORTED;
    if (blocks == 0) return GNN_OK;
    dim3 grid(static_cast<unsigned>(blocks));
    if (dots) {
        using std::integral_constant;
        a.col_end = int32_t(d);
        // The k-th eighths of rows in ascending order of their sources lead to about an eighth of the gathered matrix each, so that
        // an XCD reads fewer different lines through its L2 (4 MB; the eighth need not fit, the more of it does the better).  ms,
        // off -> on, 600 edges a vertex unless said:
        //   132,534 vertices, mild skew     64 columns 1.61 -> 1.19, 96 2.71 -> 1.78, 128 4.10 -> 2.50; strong skew 1.27 -> 1.18,
        //                                   2.14 -> 1.76, 3.33 -> 2.51
        //   66,000, mild / strong skew      96 columns 1.03 -> 0.74 / 0.79 -> 0.69, 128 1.59 -> 0.99 / 1.17 -> 0.92
        //   250,000, 500 edges a vertex     33 columns 2.95 -> 2.14 / 2.22 -> 2.00, 64 3.34 -> 2.22 / 2.25 -> 2.05
        //   250,000, 316 edges a vertex     33 columns 1.84 -> 1.36 / 1.32 -> 1.23, 64 2.02 -> 1.46 / 1.44 -> 1.29, 128 4.60 -> 3.36 / 3.42 -> 2.69
        //   500,000, 158 edges a vertex     33 columns 2.41 -> 1.95 / 1.59 -> 1.50, 64 2.47 -> 2.14 / 1.66 -> 1.56, 96 3.69 -> 3.59 / 2.72 -> 2.38, 128 (244
        //                                   MB) 5.04 -> 5.08 / 4.00 -> 3.24
        // Below the range the matrix is mostly in the L2s anyway: 66,000 vertices, 33 columns 0.50 -> 0.51 / 0.45 -> 0.47, 64 0.55 ->
        // 0.50 / 0.47 -> 0.47; 40,000, 64 columns 0.27 -> 0.29.  Rows of one line have too few steps (32 columns of 132,534
        // 0.67 -> 0.73), and so have short rows (250,000, 100 edges a vertex 64 columns 0.643 -> 0.645 / 0.39 -> 0.45; 900,000, 88 edges 2.70 -> 2.81).  From
        // 150 to 400 edges a vertex it takes 48 M edges (400,000, 62 M, strong skew 33 columns 1.14 -> 1.13, 64 1.23 -> 1.18; 200,000, 34 M 0.45 -> 0.52 and 0.49 -> 0.53),
        // or 24 M without strong skew (132,534, 26 M 48 columns 0.49 -> 0.44, 64 0.54 -> 0.45, strong skew 0.32 -> 0.38 and 0.33 -> 0.38; 100,000, 20 M 48
        // columns, 18 MB, 0.31 -> 0.32; 200,000, 34 M 33 columns 0.71 -> 0.60): where few vertices have most of the edges their lines are in the L2s either way.
        // Rows in no order gain nothing and have their steps cut: 132,534 vertices, 64 columns 1.75 -> 1.91, 128 4.40 -> 4.82.
        const int64_t bytes = N * d * 4;
        auto split_pays = [&] {
            if (!gnn_long_rows(plan->n_edges, N) || plan->rows_unordered || d <= 32 || bytes < (int64_t(18) << 20) || bytes > (int64_t(200) << 20)) return false;
            if (plan->n_edges >= 400 * N || plan->n_edges >= 48000000) return true;
            return bytes >= (int64_t(24) << 20) && gnn_plan_top_share(plan, N / 20) < kStrongSkew;
        };
        a.source_split = plan && blocks <= INT32_MAX / 8 && split_pays() ? 1 : 0;
        if (a.source_split) grid.x *= 8;
        auto launch = [&](auto lc, auto s) {
            constexpr int LC = decltype(lc)::value, S = decltype(s)::value;
            if (d == 4 * S << LC) ap_edge_dot_kernel<LC, S, false><<<grid, kBlockThreads, 0, c.stream>>>(a);
            else ap_edge_dot_kernel<LC, S, true><<<grid, kBlockThreads, 0, c.stream>>>(a);
        };
        if (log2_c == 0) launch(integral_constant<int, 0>(), integral_constant<int, 1>());
        else if (log2_c == 1) launch(integral_constant<int, 1>(), integral_constant<int, 1>());
        else if (log2_c == 2) launch(integral_constant<int, 2>(), integral_constant<int, 1>());
        else if (strips <= 8) launch(integral_constant<int, 3>(), integral_constant<int, 1>());
        else if (strips <= 16) launch(integral_constant<int, 3>(), integral_constant<int, 2>());
        else if (strips <= 24) launch(integral_constant<int, 3>(), integral_constant<int, 3>());
        else launch(integral_constant<int, 3>(), integral_constant<int, 4>());
        return hipGetLastError() == hipSuccess ? GNN_OK : GNN_ERR_LAUNCH;
    }
    // Rows of dO of one or two strips, where a step does little else: for short launches of mul and div loaded in every step, because keeping them costs
    // instructions (us, 1, 2, 4 columns, every step, before the first: 100 K vertices, 1 M edges 16.8 and 17.2, 19.0 and 19.3, 24.9 and 25.7; 130 K, 8 M 4 columns 84
    // and 91, 2 59 and 57; 245 K, 12.4 M 2, 4 columns 99 and 91, 163 and 150; 5, 8 columns, every step, in the first: 5,000, 100,000 edges 14.0 and 14.5, 14.2
    // and 14.6; 20 K, 600 K 17.8 and 17.6, 19.5 and 19.0; 40 K, 2 M 30 and 29, 31.5 and 29.5), without a gathered operand before the first (add, 4 columns,
    // 130 K, 8 M every step 39, before 35).
    const int64_t n_edges = plan ? plan->n_edges : INT64_MAX;
    if (c.ewide && !masked && !a.eid && c.lde == d && plan && staged_pays(binop, N, n_edges, d)) {
        const int C = 1 << log2_c;
        for (int G = C; G <= 64; G *= 2) {
            const int floats = 64 / G * staged_floats(G / C * 4, int(d));
            if (a.staged_wave < floats) a.staged_wave = floats;
        }
        const size_t lds = size_t(a.staged_wave) * kWavesPerBlock * 4;
        switch (binop) {
            case GNN_BIN_ADD: ap_bwd_edge_kernel<GNN_BIN_ADD, 4, true, false, kInFirst, 4, true><<<grid, kBlockThreads, lds, c.stream>>>(a); break;
            case GNN_BIN_SUB: ap_bwd_edge_kernel<GNN_BIN_SUB, 4, true, false, kInFirst, 4, true><<<grid, kBlockThreads, lds, c.stream>>>(a); break;
            case GNN_BIN_MUL: ap_bwd_edge_kernel<GNN_BIN_MUL, 4, true, false, kInFirst, 4, true><<<grid, kBlockThreads, lds, c.stream>>>(a); break;
            default: ap_bwd_edge_kernel<GNN_BIN_COPY_RHS, 4, true, false, kInFirst, 4, true><<<grid, kBlockThreads, lds, c.stream>>>(a); break;
        }
        return hipGetLastError() == hipSuccess ? GNN_OK : GNN_ERR_LAUNCH;
    }
    const bool large = n_edges >= (d > 4 ? 500000 : (d == 4 ? 10000000 : 4000000));
    KeepGo keep = d > 8 || (d > 4 && large) ? kInFirst : (large || !need_x ? kBeforeFirst : kEveryStep);
    // Scalars, and rows of max and min.  Up to two lanes own an edge of 1, 2 and 4 to 8 columns, so a row has slots for most of its edges and two in flight
    // are enough (us, four and two: 20 K vertices, 600 K edges add, 4 columns 28.7 and 19.8; 2.45 M, 60 M max of mul, 8 columns 952 and 972, add 237 and
    // 215; rows written, 8 columns, 1 M, 5 M 136 and 138, 130 K, 8 M 137 and 146; 3 columns, 19 K to 12 M edges, 2 to 18 % slower with two).  Wider scalars
    // with a gathered operand hold too many registers with a row of dO besides (33 columns, before the first and every step: 245 K, 12.4 M max of mul 386
    // and 340, div 483 and 450; 40 K, 2 M equal), from 8 M edges on also with four in flight (every step, two: 245 K 340 and 324, 2.45 M 2050 and 1920; 80
    // K, 4 M 134 and 158); up to 16 columns it is the other way (10 columns, before and every step: 500 K, 2.5 M 72 and 89, 300 K, 1.5 M 40 and 44; 60 K, 6
    // M 67 and 64; 20 K, 600 K 16.1 and 15.6).  Without one dO is all there is to load (add, 33 columns, 245 K 155 and 162; 130 columns, two strips a lane,
    // 753 and 722); max and min of that, 10 columns, 2.45 M 354 and 381, 33 columns 1052 and 1046, 3,217, 19 K edges 7.3 and 7.1.
    int in_flight = 4;
    if (!c.ewide || masked) {
        if ((d <= 8 && d != 3 && !(c.ewide && d > 4 && n_edges >= 5000000)) || (!c.ewide && need_x && d > 32 && n_edges >= 8000000)) in_flight = 2;
        const bool before = c.ewide || d <= 8 || (need_x ? d <= 16 && n_edges >= 1500000 : masked ? d <= 32 && n_edges >= 2000000 : d <= 128);
        keep = before ? kBeforeFirst : kEveryStep;
    }
    switch (binop) {
        case GNN_BIN_ADD: launch_edge_bin<GNN_BIN_ADD>(vec, c.ewide, masked, keep, in_flight, grid, c.stream, a); break;
        case GNN_BIN_SUB: launch_edge_bin<GNN_BIN_SUB>(vec, c.ewide, masked, keep, in_flight, grid, c.stream, a); break;
        case GNN_BIN_MUL: launch_edge_bin<GNN_BIN_MUL>(vec, c.ewide, masked, keep, in_flight, grid, c.stream, a); break;
        case GNN_BIN_DIV: launch_edge_bin<GNN_BIN_DIV>(vec, c.ewide, masked, keep, in_flight, grid, c.stream, a); break;
        default: launch_edge_bin<GNN_BIN_COPY_RHS>(vec, c.ewide, masked, keep, in_flight, grid, c.stream, a); break;
    }
    return hipGetLastError() == hipSuccess ? GNN_OK : GNN_ERR_LAUNCH;
}

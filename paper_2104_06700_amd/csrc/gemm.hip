// Dense update of a GNN layer (the MLP step that follows the aggregation, Section 6.3 "Memory"):
//
//   C[m, n] = act( sum_k opA(A)[m, k] * opB(B)[k, n] + bias[n] )
//
// fp32 in, fp32 out, fp32 accumulation, on the bf16 matrix cores: every operand element is split into
// three bf16 numbers whose sum it is, exactly (split8), and of the nine products of a pair the six that matter are
// formed (sum_of_products).  The bf16 instruction does 16 times the work of the fp32 one in the same time, so six of them
// are 2.7 times as fast, and the products meet the memory instead of the matrix cores (256 -> 256 excepted).
// Relative error against 64 bits, 2-norm, normal operands, before (fp32 instruction, one chain) -> now: 4096 x 256 with
// k = 256 2.9e-7 -> 0.8e-7, k = 602 4.4e-7 -> 1.2e-7, a weight gradient of 60,000 rows 3.2e-7 -> 1.8e-7, of 2.45 M rows
// 1.2e-6 -> 0.5e-6; positive operands are closer for every k too (k = 3 3.3e-8 -> 3.0e-8, 32 8.6e-8 -> 3.6e-8).  Operands spread evenly over
// 40 binary orders of magnitude, where a sum is one or two products, are closer from k = 32 on (5.2e-8 -> 4.9e-8) and a third of a
// rounding further off below (k = 3 2.8e-8 -> 3.7e-8, 8 3.3e-8 -> 4.1e-8, 16 4.0e-8 -> 4.3e-8): see sum_of_products for what is cut off.
//
// Times, 2,449,029 rows, before -> now: 100 -> 256 1.75 -> 1.30 ms, 256 -> 256 2.95 -> 2.03 (0.95 PFLOP/s of bf16 products; the
// chip's own limit with such operands is 1.8, its clock falls to 1.7 GHz), 256 -> 47 1.01 -> 0.75; weight gradients
// 100 x 256 1.45 -> 1.12, 256 x 256 2.75 -> 2.03, 256 x 47 0.90 -> 0.78; 24,490 rows 256 -> 256 46 -> 31 us.
#include "common.h"

namespace {

constexpr int BK = 16;  // k of one v_mfma_f32_32x32x16_bf16

typedef float float16v __attribute__((ext_vector_type(16)));
typedef float float2v __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4_any __attribute__((ext_vector_type(4), aligned(4)));  // 16-byte access at the alignment of a float

struct GemmArgs {
    const float *A;
    const float *B;
    float *C;           // or the partial buffer when n_split > 1
    const float *bias;  // [N] or nullptr
    int64_t sam, sak;   // element strides of opA(A)[m, k]
    int64_t sbk, sbn;   // element strides of opB(B)[k, n]
    int64_t ldc;
    int64_t M, N, K;
    int64_t k_per_split;
    int32_t relu;
    int32_t n_split;
    gnn_packed_target packed;  // active: the result goes into a producer-side layout instead of C
    // Rectifier gate folded into the operand loads (the backward pass of a layer multiplies by
    // G = dH where H > 0): an element of A (of B) counts as 0 where the gate matrix, which has the
    // operand's shape and strides, is not positive.  colsum: [n_split][N] column sums of opB(B) after
    // its gate (the bias gradient), written by the workgroups of the first tile row.
    const float *a_gate, *b_gate;
    float *colsum;
    // Tile order.  The launch is one-dimensional and workgroup b runs on XCD b % 8, each with an L2 of its own.
    // The tiles that read the same rows of an operand (the column tiles of one row tile of a tall product; all
    // tiles of one part of a split reduction) get ids 8 apart: the same XCD, one after the other, so the second
    // read of those rows hits that XCD's L2.  inner = number of such tiles (0: plain order, x fastest).
    int32_t gx, gy, gz, inner;
};

// Tile of this workgroup (see GemmArgs::inner); false: none, the last group of 8 may be incomplete.
__device__ __forceinline__ bool tile_of_block(const GemmArgs &g, int64_t &bx, int64_t &by, int64_t &bz) {
    const int64_t b = blockIdx.x;
    if (g.inner > 0) {
        const int64_t per = int64_t(8) * g.inner, r = b % per;
        const int64_t outer = b / per * 8 + (r & 7), in = r >> 3;
        if (g.gz > 1) { bz = outer; bx = in % g.gx; by = in / g.gx; }
        else { bx = outer; by = in; bz = 0; }
        return bx < g.gx && bz < g.gz;
    }
    bx = b % g.gx;
    by = b / g.gx % g.gy;
    bz = b / (int64_t(g.gx) * g.gy);
    return true;
}

// Two floats -> two bf16 (round to nearest even), low half first.
__device__ __forceinline__ uint32_t bf16_pair(float x, float y) {
    const float2v v = {x, y};
    return __builtin_bit_cast(uint32_t, __builtin_convertvector(v, bf16x2));
}

// Operands are multiplied by 2^16 before they are split, and the sums of their products by 2^-32 (add_tile), both exact: a float is a
// multiple of 2^-149, so what is split is one of 2^-133, bf16's smallest number, and no part of any operand is cut off there;
// and sums of products lose nothing to underflow that the result could show.
constexpr float kOperandScale = 0x1p16f, kSumScale = 0x1p-32f;

// x = p[0] + p[1] + p[2] exactly: 24 significant bits are three times the eight of a bf16, and x is a multiple of 2^-133.  Each
// difference below is exact (the rounded part shares the leading bits), |p[1]| <= 2^-9 |x|, |p[2]| <= 2^-18 |x|.  What is not
// finite, or rounds up to infinity, leaves infinities and NaNs that reach every result it takes part in (recompute_if_needed).
__device__ __forceinline__ void split8(const float (&x)[8], uint4 (&p)[3]) {
    uint32_t w[3][4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        float a = x[2 * i], b = x[2 * i + 1];
#pragma unroll
        for (int s = 0; s < 3; ++s) {
            const uint32_t q = bf16_pair(a, b);
            w[s][i] = q;
            if (s < 2) {
                a -= __uint_as_float(q << 16);
                b -= __uint_as_float(q & 0xffff0000u);
            }
        }
    }
#pragma unroll
    for (int s = 0; s < 3; ++s) p[s] = make_uint4(w[s][0], w[s][1], w[s][2], w[s][3]);
}

// The products of 16 k: a b = sum over the parts of a_p b_q, |a_p b_q| <= 2^(-9 (p + q)) |a b|.  The three products with
// p + q > 2 are left out: 2^-26 of |a b| at most each and of either sign, where the rounding of one fp32 addition is 2^-25 of the
// sum.  They are summed from zero, the smallest first, and added to the result with one rounding (add_tile): the
// matrix cores cut off what lies below the sum's last bit, so a long chain through them would be the worse sum.
__device__ __forceinline__ void sum_of_products(float16v &sum, const bf16x8 (&a)[3], const bf16x8 (&b)[3]) {
#pragma unroll
    for (int v = 0; v < 16; ++v) sum[v] = 0.0f;
#pragma unroll
    for (int s = 2; s >= 0; --s)
#pragma unroll
        for (int p = 0; p <= s; ++p) sum = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[p], b[s - p], sum, 0, 0, 0);
}

// What is cut off is cut off towards minus infinity, which would add up over the steps of a long k and over the rows of a later
// sum (a bias gradient).  So in step t the rows of A whose number plus t is odd are negated (row_scale), and their sums subtracted.
__device__ __forceinline__ float row_scale(int row, int t) {
    return __uint_as_float(__float_as_uint(kOperandScale) ^ (uint32_t(row + t) << 31));
}
__device__ __forceinline__ void add_tile(float16v &acc, const float16v &sum, int t) {
    const float s = (t & 1) ? -kSumScale : kSumScale;
#pragma unroll
    for (int v = 0; v < 16; ++v) acc[v] = fmaf(sum[v], (v & 1) ? -s : s, acc[v]);
}

// A [ROWS x BK] tile of an operand in LDS, in the order in which the matrix cores take it: per plane of the split and per 32
// rows the 16 bytes (8 k) of every lane, lane = 32 * (k / 8) + row.  The upper half's rows are rotated by four so that the
// writes of K_CONTIG threads, which alternate between the halves, fall into different banks.
template <int ROWS>
struct SplitTile {
    uint4 v[3][ROWS / 32][64];
    static __device__ __forceinline__ int slot(int half, int r32) { return half * 32 + (r32 ^ (half * 4)); }
};

// One tile of an operand on its way from global memory to LDS.  X(r, k) = base[r * sr + k * sk].  K_CONTIG: sk == 1, else
// sr == 1.  A thread takes units of 8 k of a row: two 16-byte loads, or eight loads of 4 bytes with the rows along the
// lanes.  Rows past the end repeat the last one (their results are never stored).  load() and store() are separate so that the
// loads of a later tile are in flight while the matrix cores work.
template <bool K_CONTIG, int ROWS, int THREADS, bool GATED = false, int SETS = 1>
struct Stager {
    static constexpr int UNITS = ROWS * 2;
    static constexpr int PER_THREAD = (UNITS + THREADS - 1) / THREADS;
    float v[SETS][PER_THREAD][8];  // SETS tiles on their way
    float gate[SETS][GATED ? PER_THREAD : 1][8];  // the gate's elements travel beside the operand's and are applied in store()
    // Rows along the lanes, 64 and more: a wavefront's 64 units have one k, so the address is a scalar plus 4 * row.  Otherwise
    // a lane keeps the address of its unit in the tile at k_begin.
    static constexpr bool SCALAR_K = !K_CONTIG && ROWS % 64 == 0;
    const float *p[PER_THREAD];
    uint32_t row_bytes[SCALAR_K ? PER_THREAD : 1];
    int64_t sk, gate_off;

    static __device__ __forceinline__ bool has(int h) { return UNITS % THREADS == 0 || int(threadIdx.x) + h * THREADS < UNITS; }
    static __device__ __forceinline__ int row_of(int h) {
        const int u = int(threadIdx.x) + h * THREADS;
        return K_CONTIG ? u >> 1 : u % ROWS;
    }
    static __device__ __forceinline__ int half_of(int h) {
        const int u = int(threadIdx.x) + h * THREADS;
        return K_CONTIG ? u & 1 : u / ROWS;
    }

    __device__ __forceinline__ void init(const float *__restrict__ base, const float *__restrict__ gate_base, int64_t sr, int64_t sk_,
                                         int64_t r0, int64_t r_end, int64_t k_begin) {
        sk = K_CONTIG ? 1 : sk_;
        gate_off = (GATED && gate_base) ? gate_base - base : 0;
#pragma unroll
        for (int h = 0; h < PER_THREAD; ++h) {
            const int64_t r = r0 + row_of(h), row = r < r_end ? r : r_end - 1;
            if constexpr (SCALAR_K) {
                p[h] = base + r0 + (k_begin + __builtin_amdgcn_readfirstlane(half_of(h)) * 8) * sk;
                row_bytes[h] = uint32_t(row - r0) * 4;
            } else {
                p[h] = base + row * (K_CONTIG ? sr : 1) + (k_begin + half_of(h) * 8) * sk;
            }
        }
    }

    // k_off = first k of the tile - k_begin (uniform; may be negative)
    __device__ __forceinline__ void load(int64_t k_off, bool gated, int set = 0) {
#pragma unroll
        for (int h = 0; h < PER_THREAD; ++h) {
            if (!has(h)) continue;
            fetch(h, p[h] + k_off * sk, v[set][h]);
            if constexpr (GATED) {
                if (gated) fetch(h, p[h] + k_off * sk + gate_off, gate[set][h]);
            }
        }
    }
    __device__ __forceinline__ float at(int h, const float *q, int i) const {
        if constexpr (SCALAR_K) return *reinterpret_cast<const float *>(reinterpret_cast<const char *>(q + i * sk) + row_bytes[h]);
        else return q[i * sk];
    }
    __device__ __forceinline__ void fetch(int h, const float *q, float (&x)[8]) const {
        if constexpr (K_CONTIG) {
            const f32x4_any lo = *reinterpret_cast<const f32x4_any *>(q), hi = *reinterpret_cast<const f32x4_any *>(q + 4);
#pragma unroll
            for (int i = 0; i < 4; ++i) { x[i] = lo[i]; x[4 + i] = hi[i]; }
        } else {
#pragma unroll
            for (int i = 0; i < 8; ++i) x[i] = at(h, q, i);
        }
    }

    // the first tile of an operand with n < 16 k
    __device__ __forceinline__ void load_few(int n, int set = 0) {
#pragma unroll
        for (int h = 0; h < PER_THREAD; ++h) {
            if (!has(h)) continue;
#pragma unroll
            for (int i = 0; i < 8; ++i) v[set][h][i] = half_of(h) * 8 + i < n ? at(h, p[h], i) : 0.0f;
        }
    }
    // the first `n` k of the tile count as 0 (a tile moved back to end with k_end repeats them)
    __device__ __forceinline__ void drop_first(int n, int set = 0) {
#pragma unroll
        for (int h = 0; h < PER_THREAD; ++h)
#pragma unroll
            for (int i = 0; i < 8; ++i) v[set][h][i] = half_of(h) * 8 + i >= n ? v[set][h][i] : 0.0f;
    }

    // flip: the rows are negated as in step `t` (row_scale)
    __device__ __forceinline__ void store(SplitTile<ROWS> &tile, bool gated, bool with_sums, float (&sums)[PER_THREAD][2], bool flip, int t, int set = 0) {
#pragma unroll
        for (int h = 0; h < PER_THREAD; ++h) {
            if (!has(h)) continue;
            if constexpr (GATED) {
                if (gated) {
#pragma unroll
                    for (int i = 0; i < 8; ++i) v[set][h][i] = gate[set][h][i] > 0.0f ? v[set][h][i] : 0.0f;
                }
                if (with_sums) {  // of even and of odd tiles: shorter chains, less rounding
                    const float x = ((v[set][h][0] + v[set][h][1]) + (v[set][h][2] + v[set][h][3])) + ((v[set][h][4] + v[set][h][5]) + (v[set][h][6] + v[set][h][7]));
                    sums[h][0] = (t & 1) ? sums[h][0] : sums[h][0] + x;
                    sums[h][1] = (t & 1) ? sums[h][1] + x : sums[h][1];
                }
            }
            const float scale = flip ? row_scale(row_of(h), t) : kOperandScale;
#pragma unroll
            for (int i = 0; i < 8; ++i) v[set][h][i] *= scale;
            uint4 q[3];
            split8(v[set][h], q);
            const int r = row_of(h), s = SplitTile<ROWS>::slot(half_of(h), r & 31);
#pragma unroll
            for (int pl = 0; pl < 3; ++pl) tile.v[pl][r >> 5][s] = q[pl];
        }
    }
};

// Four k of a row on their way to the fp32 instruction, with their gate.
template <bool K_CONTIG, bool GATED>
struct Four {
    float x[4], gate[GATED ? 4 : 1];
    static __device__ __forceinline__ void fetch(float (&v)[4], const float *p, int64_t sk) {
        if constexpr (K_CONTIG) {
            const f32x4_any q = *reinterpret_cast<const f32x4_any *>(p);
#pragma unroll
            for (int i = 0; i < 4; ++i) v[i] = q[i];
        } else {
#pragma unroll
            for (int i = 0; i < 4; ++i) v[i] = p[i * sk];
        }
    }
    __device__ __forceinline__ void load(const float *p, int64_t sk, bool gated, int64_t gate_off) {
        fetch(x, p, sk);
        if constexpr (GATED) {
            if (gated) fetch(gate, p + gate_off, sk);
        }
    }
    __device__ __forceinline__ float at(int i, bool gated) const {
        if constexpr (GATED) return !gated || gate[i] > 0.0f ? x[i] : 0.0f;
        else return x[i];
    }
};

// An operand that is not finite, or 2^112 and more, splits into infinities and NaNs, and so do the sums of 16 products that reach
// 2^96: none of the results they take part in is finite.  A wavefront with such a result computes its tiles again from the
// operands as they are, by the fp32 matrix instruction.  FEW_K: less than 16 products, 2 = in any case.
// What that costs, 2,449,029 rows, with single elements loaded as they are used -> now, beside finite operands: a row of A that is
// not finite nothing measurable; one element of B, which every wavefront meets, 256 -> 256 7.4 -> 6.1 ms beside 2.0, 256 -> 47
// 2.4 -> 1.6 beside 0.74; an element in the weight gradient 256 x 256 4.9 -> 2.6 beside 2.0, nothing finite 9.2 -> 5.9.
template <bool A_K_CONTIG, bool B_K_CONTIG, bool A_GATED, bool B_GATED, int FEW_K, int TI, int TJ>
__device__ __forceinline__ void recompute_if_needed(const GemmArgs &g, float16v (&acc)[TI][TJ], int64_t m0, int64_t n0, int64_t k_begin,
                                                    int64_t k_end) {
    float most = 0.0f;  // of the absolute values; a NaN stays
#pragma unroll
    for (int i = 0; i < TI; ++i)
#pragma unroll
        for (int j = 0; j < TJ; ++j)
#pragma unroll
            for (int v = 0; v < 16; v += 2)
                asm("v_maximum3_f32 %0, |%1|, |%2|, %0" : "+v"(most) : "v"(acc[i][j][v]), "v"(acc[i][j][v + 1]));
    const bool again = FEW_K == 2 || !(most <= 0x1.fffffep127f);
    if (!__any(again)) return;
    const int l32 = threadIdx.x & 31, lk = (threadIdx.x >> 5) & 1;
#pragma unroll
    for (int i = 0; i < TI; ++i)
#pragma unroll
        for (int j = 0; j < TJ; ++j)
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[i][j][v] = 0.0f;
    // Operand layout of the 32x32x2 instruction: lane l holds A[l % 32][l / 32] and B[l / 32][l % 32].  Rows past the end repeat
    // the last one.  Steps of 8 k: the lower lanes' instructions take the first four, the upper lanes' the others.
    const float *pa[TI], *pb[TJ];
#pragma unroll
    for (int i = 0; i < TI; ++i) {
        const int64_t m = m0 + i * 32 + l32;
        pa[i] = g.A + (m < g.M ? m : g.M - 1) * g.sam + k_begin * g.sak;
    }
#pragma unroll
    for (int j = 0; j < TJ; ++j) {
        const int64_t n = n0 + j * 32 + l32;
        pb[j] = g.B + (n < g.N ? n : g.N - 1) * g.sbn + k_begin * g.sbk;
    }
    const bool a_gated = A_GATED && g.a_gate, b_gated = B_GATED && g.b_gate;
    const int64_t a_gate_off = a_gated ? g.a_gate - g.A : 0, b_gate_off = b_gated ? g.b_gate - g.B : 0;
    const int64_t len = k_begin < k_end ? k_end - k_begin : 0, whole = FEW_K ? 0 : len / 8 * 8;
    if (!FEW_K && whole > 0) {
        Four<A_K_CONTIG, A_GATED> a[2][TI];
        Four<B_K_CONTIG, B_GATED> b[2][TJ];
        auto load = [&](int64_t k, int set) {  // behind the last step: that one again
            const int64_t at = (k < whole ? k : whole - 8) + 4 * lk;
#pragma unroll
            for (int i = 0; i < TI; ++i) a[set][i].load(pa[i] + at * g.sak, g.sak, a_gated, a_gate_off);
#pragma unroll
            for (int j = 0; j < TJ; ++j) b[set][j].load(pb[j] + at * g.sbk, g.sbk, b_gated, b_gate_off);
        };
        auto multiply = [&](int set) {
#pragma unroll
            for (int q = 0; q < 4; ++q)
#pragma unroll
                for (int i = 0; i < TI; ++i)
#pragma unroll
                    for (int j = 0; j < TJ; ++j)
                        acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x2f32(a[set][i].at(q, a_gated), b[set][j].at(q, b_gated), acc[i][j], 0, 0, 0);
        };
        load(0, 0);
#pragma unroll 1
        for (int64_t k = 0; k < whole; k += 16) {
            load(k + 8, 1);
            if (TI > 1) __builtin_amdgcn_sched_barrier(0);  // all ahead of the products that hide them; one row tile has too many to issue at once
            multiply(0);
            if (k + 8 >= whole) break;
            load(k + 16, 0);
            if (TI > 1) __builtin_amdgcn_sched_barrier(0);
            multiply(1);
        }
    }
#pragma unroll 1
    for (int64_t k = whole; k < len; k += 2) {
        const bool in = k + lk < len;
        const int64_t at = in ? k + lk : 0;
        float a[TI], b[TJ];
#pragma unroll
        for (int i = 0; i < TI; ++i) {
            const float *p = pa[i] + at * g.sak;
            a[i] = in && (!a_gated || p[a_gate_off] > 0.0f) ? *p : 0.0f;
        }
#pragma unroll
        for (int j = 0; j < TJ; ++j) {
            const float *p = pb[j] + at * g.sbk;
            b[j] = in && (!b_gated || p[b_gate_off] > 0.0f) ? *p : 0.0f;
        }
#pragma unroll
        for (int i = 0; i < TI; ++i)
#pragma unroll
            for (int j = 0; j < TJ; ++j) acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x2f32(a[i], b[j], acc[i][j], 0, 0, 0);
    }
}

// Writes a wavefront's TI x TJ result tiles, whose first element is C[m0][n0] (of partial plane bz).  EDGE: rows may lie past
// the end.  Register v of lane l holds C[8 * (v / 4) + 4 * (l / 32) + v % 4][l % 32].
template <int TI, int TJ, bool EDGE>
__device__ __forceinline__ void write_rows(const GemmArgs &g, float16v (&acc)[TI][TJ], int64_t m0, int64_t n0, int64_t bz) {
    const int l32 = threadIdx.x & 31, lk = (threadIdx.x >> 5) & 1;
    const gnn_packed_target &pk = g.packed;
    if (pk.active) {
        // producer-side layout: the 32 lanes of a row write one 128-byte line of a slice table (or a piece of the
        // tail) at the row's rank; rank and factor of a row are looked up once for all its column tiles
#pragma unroll
        for (int i = 0; i < TI; ++i)
#pragma unroll
            for (int v = 0; v < 16; ++v) {
                const int64_t m = m0 + i * 32 + 8 * (v / 4) + 4 * lk + (v % 4);
                if (EDGE && m >= g.M) continue;
                const int64_t row = pk.rank[m];
                const float fac = gnn_row_factor(pk.scale_mode, pk.scale_mode ? pk.counts[m] : 0);
#pragma unroll
                for (int j = 0; j < TJ; ++j) {
                    const int64_t n = n0 + j * 32 + l32;
                    if (n >= g.N) continue;
                    float *q = n < pk.main_cols ? pk.base + (n >> 5) * pk.table_stride + row * 32 + (n & 31)
                                                : pk.tail + row * pk.tail_ld + (n - pk.main_cols);
                    *q = acc[i][j][v] * fac;
                }
            }
        return;
    }
    const bool whole = g.n_split == 1;  // else partial planes of M x ldc
    const bool relu = g.relu && whole;
    float *out = g.C + (whole ? 0 : bz * g.M * g.ldc) + (m0 + 4 * lk) * g.ldc + n0 + l32;
#pragma unroll
    for (int j = 0; j < TJ; ++j) {
        const int64_t n = n0 + j * 32 + l32;
        if (n >= g.N) continue;
        const float bv = (g.bias && whole) ? g.bias[n] : 0.0f;
#pragma unroll
        for (int i = 0; i < TI; ++i)
#pragma unroll
            for (int v = 0; v < 16; ++v) {
                const int r = i * 32 + 8 * (v / 4) + (v % 4);
                if (EDGE && m0 + r + 4 * lk >= g.M) continue;
                float x = acc[i][j][v] + bv;
                if (relu) x = x > 0.0f ? x : 0.0f;
                out[r * g.ldc + j * 32] = x;
            }
    }
}

template <int TI, int TJ>
__device__ __forceinline__ void write_tiles(const GemmArgs &g, float16v (&acc)[TI][TJ], int64_t m0, int64_t n0, int64_t bz) {
    if (m0 + TI * 32 <= g.M) write_rows<TI, TJ, false>(g, acc, m0, n0, bz);
    else write_rows<TI, TJ, true>(g, acc, m0, n0, bz);
}

// Workgroup tile (WM * TI * 32) x (WN * TJ * 32): WM x WN wavefronts, each TI x TJ MFMA tiles.
// FOLD: 0 = plain operands; 2 = B may carry a gate and its column sums may be asked for.
template <bool A_K_CONTIG, bool B_K_CONTIG, int WM, int WN, int TI, int TJ, int FOLD = 0>
__global__ void __launch_bounds__(WM * WN * 64) __attribute__((amdgpu_waves_per_eu(2, 8))) gemm_kernel(const GemmArgs g) {
    constexpr int BM = WM * TI * 32, BN = WN * TJ * 32, THREADS = WM * WN * 64;
    struct Tiles { SplitTile<BM> a; SplitTile<BN> b; };
    __shared__ __attribute__((aligned(16))) Tiles tiles[2];
    const int lane = threadIdx.x & 63;
    const int wave = threadIdx.x >> 6;
    const int wm = (wave / WN) * TI * 32, wn = (wave % WN) * TJ * 32;  // this wavefront's part of the tile
    int64_t bx, by, bz;
    if (!tile_of_block(g, bx, by, bz)) return;  // whole workgroup
    const int64_t m0 = bx * BM, n0 = by * BN;
    const int64_t k_begin = bz * g.k_per_split;
    const int64_t k_end = k_begin + g.k_per_split < g.K ? k_begin + g.k_per_split : g.K;

    float16v acc[TI][TJ];
    auto clear = [&]() {
#pragma unroll
        for (int i = 0; i < TI; ++i)
#pragma unroll
            for (int j = 0; j < TJ; ++j)
#pragma unroll
                for (int v = 0; v < 16; ++v) acc[i][j][v] = 0.0f;
    };
    clear();

    // Tiles on their way.  Two where the registers leave two wavefronts per SIMD anyway (2,449,029 rows into 256 x 256 2.04 ->
    // 1.99 ms, 109,316 into 128 x 128 44 -> 40 us); narrow tiles do better with more workgroups (602 x 16: 114 us, 139 with two).
    constexpr int SETS = BN >= 128 ? 2 : 1;
    using StagerA = Stager<A_K_CONTIG, BM, THREADS, false, SETS>;
    using StagerB = Stager<B_K_CONTIG, BN, THREADS, FOLD == 2, SETS>;
    StagerA sa;
    StagerB sb;
    const bool b_gated = FOLD == 2 && g.b_gate;
    const bool sums = FOLD == 2 && g.colsum && bx == 0;  // the first tile row also adds up the columns of B (uniform)
    float no_sum[StagerA::PER_THREAD][2] = {}, col_sum[StagerB::PER_THREAD][2] = {};
    const int l32 = lane & 31, lk = lane >> 5;
    const int my_slot = SplitTile<BM>::slot(lk, l32);
    auto stage = [&](int p) {  // registers -> LDS; p = number of the tile % 2
        sa.store(tiles[p].a, false, false, no_sum, true, p, p % SETS);
        sb.store(tiles[p].b, b_gated, sums, col_sum, false, p, p % SETS);
    };
    auto multiply = [&](int step) {
        const Tiles &t = tiles[step & 1];
        bf16x8 a[TI][3];
#pragma unroll
        for (int i = 0; i < TI; ++i)
#pragma unroll
            for (int p = 0; p < 3; ++p) a[i][p] = __builtin_bit_cast(bf16x8, t.a.v[p][wm / 32 + i][my_slot]);
#pragma unroll
        for (int j = 0; j < TJ; ++j) {
            bf16x8 b[3];
#pragma unroll
            for (int p = 0; p < 3; ++p) b[p] = __builtin_bit_cast(bf16x8, t.b.v[p][wn / 32 + j][my_slot]);
            float16v sum[TI];
#pragma unroll
            for (int i = 0; i < TI; ++i) sum_of_products(sum[i], a[i], b);
#pragma unroll
            for (int i = 0; i < TI; ++i) add_tile(acc[i][j], sum[i], step);
            __builtin_amdgcn_sched_barrier(0);  // what the compiler fetches further ahead does not fit the registers
        }
    };
    // While tile t is multiplied, tile t + 1 is split into the other half of the LDS and the SETS tiles behind it are on their way.
    // A last tile of less than 16 k is moved back to end with the part (K >= 16); what it repeats counts as 0.  Loads past the
    // last tile repeat it, so that the loop has no branches around them.
    const int64_t len = k_begin < k_end ? k_end - k_begin : 0;
    const int64_t n_tiles = (len + BK - 1) / BK;
    const int repeated = int(n_tiles * BK - len);
    auto load = [&](int64_t t, int p) {
        const int64_t k = t * BK < len - BK ? t * BK : len - BK;
        sa.load(k, false, p % SETS);
        sb.load(k, b_gated, p % SETS);
    };
    auto next = [&](int64_t t, int p) {  // p = t % 2
        if (t + 1 == n_tiles && repeated) {
            sa.drop_first(repeated, p % SETS);
            if constexpr (FOLD == 2) sb.drop_first(repeated, p % SETS);  // for its column sums
        }
        stage(p);
        load(t + SETS, p);
        __syncthreads();
    };
    if (n_tiles > 0) {
        sa.init(g.A, g.a_gate, g.sam, g.sak, m0, g.M, k_begin);
        sb.init(g.B, g.b_gate, g.sbn, g.sbk, n0, g.N, k_begin);
        load(0, 0);
        __builtin_amdgcn_sched_barrier(0);  // in this order, as in the loop: what is waited for is counted
        if (SETS == 2) load(1, 1);
        next(0, 0);
#pragma unroll 1
        for (int64_t t = 0;; t += 2) {
            multiply(0);
            if (t + 1 == n_tiles) break;
            next(t + 1, 1);
            multiply(1);
            if (t + 2 == n_tiles) break;
            next(t + 2, 0);
        }
    }

    recompute_if_needed<A_K_CONTIG, B_K_CONTIG, false, FOLD == 2, 0>(g, acc, m0 + wm, n0 + wn, k_begin, k_end);

    if constexpr (FOLD == 2) {
        if (sums) {
            // units that hold the same columns (the two halves of k) are added in order through LDS
            static_assert(!B_K_CONTIG, "column sums are kept for row-contiguous operands only");
            float *scr = reinterpret_cast<float *>(&tiles[0]);
            __syncthreads();  // the operand tiles are no longer needed
#pragma unroll
            for (int h = 0; h < StagerB::PER_THREAD; ++h)
                if (StagerB::has(h)) scr[StagerB::half_of(h) * BN + StagerB::row_of(h)] = col_sum[h][0] + col_sum[h][1];
            __syncthreads();
            for (int n = int(threadIdx.x); n < BN && n0 + n < g.N; n += THREADS) g.colsum[bz * g.N + n0 + n] = scr[n] + scr[BN + n];
        }
    }

    write_tiles<TI, TJ>(g, acc, m0 + wm, n0 + wn, bz);
}

// Of up to this many products fp32 instructions make the better sum: they round where the split sum is cut off.  2-norm error, normal
// operands, split and fp32: k = 1 3.5e-8 and 2.5e-8, 2 3.3e-8 and 3.1e-8, 3 3.3e-8 and 3.6e-8, 15 3.4e-8 and 7.2e-8.  What bounds
// such a product is its stores, and those of rows that are not whole lines get in each other's way if more than five wavefronts per
// SIMD are at it: 2.45 M rows, k = 1, 47 columns 122 us, 193 with eight (split: 144); 256 columns 437 and 462 (split: 509).
constexpr int kFewProducts = 2;

// Tall products: A row-major with k along its rows (a layer's forward product, and the products with W^T of its backward
// pass).  A wavefront owns 32 rows of C and TJ * 32 columns: its elements of A go from global memory straight into the
// lanes that need them, two steps of 16 k ahead of their use, and are split there, once; only B passes through LDS.  FEW_K: 1 =
// less than 16 k, one step of single elements; 2 = at most kFewProducts.
template <int WAVES, int TJ, bool B_K_CONTIG, bool GATED, int FEW_K = 0>
__global__ void __launch_bounds__(WAVES * 64) __attribute__((amdgpu_waves_per_eu(FEW_K == 2 ? 4 : TJ >= 4 ? 2 : TJ == 2 && GATED ? 3 : 4, FEW_K == 2 || (FEW_K == 1 && !B_K_CONTIG) ? 5 : 8))) tall_kernel(const GemmArgs g) {
    constexpr int BM = WAVES * 32, BN = TJ * 32;
    __shared__ __attribute__((aligned(16))) SplitTile<BN> tiles[2];
    const int lane = threadIdx.x & 63;
    const int wave = threadIdx.x >> 6;
    const int l32 = lane & 31, lk = lane >> 5;
    int64_t bx, by, bz;
    if (!tile_of_block(g, bx, by, bz)) return;  // whole workgroup
    const int64_t m0 = bx * BM + wave * 32, n0 = by * BN;
    const int my_slot = SplitTile<BN>::slot(lk, l32);

    float16v acc[1][TJ];
#pragma unroll
    for (int j = 0; j < TJ; ++j)
#pragma unroll
        for (int v = 0; v < 16; ++v) acc[0][j][v] = 0.0f;

    // A: a lane's eight elements of a step, two steps in registers (rows past the end repeat the last one)
    const int64_t my_row = m0 + l32 < g.M ? m0 + l32 : g.M - 1;
    const float *pa = g.A + my_row * g.sam + lk * 8;
    const int64_t gate_off = GATED ? g.a_gate - g.A : 0;
    float va[2][8], ga[GATED ? 2 : 1][8];
    auto fetch = [&](float (&x)[8], const float *q) {
        if constexpr (FEW_K) {
#pragma unroll
            for (int i = 0; i < 8; ++i) x[i] = i < int(g.K) - lk * 8 ? q[i] : 0.0f;
            return;
        }
        const f32x4_any lo = *reinterpret_cast<const f32x4_any *>(q), hi = *reinterpret_cast<const f32x4_any *>(q + 4);
#pragma unroll
        for (int i = 0; i < 4; ++i) { x[i] = lo[i]; x[4 + i] = hi[i]; }
    };
    // A last step of less than 16 k is moved back to end with K (K >= 16); the elements of A that belong to the step before
    // count as 0 there (should one of B be infinite, the result is NaN and computed again).  Loads past the last step repeat it.
    const int64_t n_tiles = (g.K + BK - 1) / BK;
    const int64_t k_last = g.K - BK;
    const int repeated = FEW_K ? 0 : int(n_tiles * BK - g.K);
    auto k_of = [&](int64_t t) { return FEW_K ? 0 : t * BK < k_last ? t * BK : k_last; };
    auto load_a = [&](int64_t t, int p) {
        fetch(va[p], pa + k_of(t));
        if constexpr (GATED) fetch(ga[p], pa + k_of(t) + gate_off);
    };
    Stager<B_K_CONTIG, BN, WAVES * 64> sb;
    float no_sum[decltype(sb)::PER_THREAD][2] = {};
    // Step t (p = t % 2).  The products of a step are summed from zero, smallest first, and added to the result with one
    // rounding: fewer and better roundings than a chain of single products has.
    auto step = [&](int64_t t, int p) {
        if constexpr (!FEW_K) sb.load(k_of(t + 1), false);
        if constexpr (GATED) {
#pragma unroll
            for (int i = 0; i < 8; ++i) va[p][i] = ga[p][i] > 0.0f ? va[p][i] : 0.0f;
        }
        if (t + 1 == n_tiles && repeated) {
#pragma unroll
            for (int i = 0; i < 8; ++i) va[p][i] = i + lk * 8 >= repeated ? va[p][i] : 0.0f;
        }
#pragma unroll
        for (int i = 0; i < 8; ++i) va[p][i] *= row_scale(lane, p);
        uint4 q[3];
        split8(va[p], q);
        if constexpr (!FEW_K) load_a(t + 2, p);
        bf16x8 a[3];
#pragma unroll
        for (int s = 0; s < 3; ++s) a[s] = __builtin_bit_cast(bf16x8, q[s]);
        // The parts of B for the next 32 columns are on their way while these are multiplied; the barriers keep the compiler from
        // fetching them all ahead, which takes more registers than there are.
        if (TJ == 8 || t < n_tiles) {
            bf16x8 b[2][3];
            float16v sum[2];
#pragma unroll
            for (int s = 0; s < 3; ++s) b[0][s] = __builtin_bit_cast(bf16x8, tiles[p].v[s][0][my_slot]);
#pragma unroll
            for (int j = 0; j < TJ; ++j) {
                if (j + 1 < TJ) {
#pragma unroll
                    for (int s = 0; s < 3; ++s) b[(j + 1) & 1][s] = __builtin_bit_cast(bf16x8, tiles[p].v[s][j + 1][my_slot]);
                }
                sum_of_products(sum[j & 1], a, b[j & 1]);
                if (j > 0) add_tile(acc[0][j - 1], sum[(j - 1) & 1], p);
                __builtin_amdgcn_sched_barrier(0);
            }
            add_tile(acc[0][TJ - 1], sum[(TJ - 1) & 1], p);
        }
        if constexpr (!FEW_K) {
            sb.store(tiles[1 - p], false, false, no_sum, false, 0);
            __syncthreads();
        }
    };
    sb.init(g.B, nullptr, g.sbn, g.sbk, n0, g.N, 0);
    if constexpr (FEW_K) {
        if constexpr (FEW_K != 2) {
            sb.load_few(int(g.K));
            load_a(0, 0);
            sb.store(tiles[0], false, false, no_sum, false, 0);
            __syncthreads();
            step(0, 0);
        }
        recompute_if_needed<true, B_K_CONTIG, GATED, false, FEW_K>(g, acc, m0, n0, 0, g.K);
        write_tiles<1, TJ>(g, acc, m0, n0, 0);
        return;
    }
    sb.load(0, false);
    load_a(0, 0);
    __builtin_amdgcn_sched_barrier(0);  // in this order, as in the loop: what is waited for is counted
    load_a(1, 1);
    sb.store(tiles[0], false, false, no_sum, false, 0);
    __builtin_amdgcn_s_waitcnt(GATED ? 0x0f74 : 0x0f72);  // vmcnt: all but the second step's
    __syncthreads();
#pragma unroll 1
    for (int64_t t = 0; t < n_tiles; t += 2) {
        step(t, 0);
        if (TJ == 8 && t + 1 == n_tiles) break;
        step(t + 1, 1);
    }
    recompute_if_needed<true, B_K_CONTIG, GATED, false, 0>(g, acc, m0, n0, 0, g.K);
    write_tiles<1, TJ>(g, acc, m0, n0, 0);
}

template <int WAVES, int TJ>
void launch_tall(bool b_k, dim3 grid, hipStream_t stream, const GemmArgs &g) {
    if (g.a_gate && b_k) tall_kernel<WAVES, TJ, true, true><<<grid, WAVES * 64, 0, stream>>>(g);
    else if (g.a_gate) tall_kernel<WAVES, TJ, false, true><<<grid, WAVES * 64, 0, stream>>>(g);
    else if (b_k) tall_kernel<WAVES, TJ, true, false><<<grid, WAVES * 64, 0, stream>>>(g);
    else tall_kernel<WAVES, TJ, false, false><<<grid, WAVES * 64, 0, stream>>>(g);
}

template <int FEW_K>
void launch_tall_few_k(bool b_k, dim3 grid, hipStream_t stream, const GemmArgs &g) {
    if (g.a_gate && b_k) tall_kernel<4, 2, true, true, FEW_K><<<grid, 256, 0, stream>>>(g);
    else if (g.a_gate) tall_kernel<4, 2, false, true, FEW_K><<<grid, 256, 0, stream>>>(g);
    else if (b_k) tall_kernel<4, 2, true, false, FEW_K><<<grid, 256, 0, stream>>>(g);
    else tall_kernel<4, 2, false, false, FEW_K><<<grid, 256, 0, stream>>>(g);
}

template <int WM, int WN, int TI, int TJ>
void launch_gemm(bool b_k, dim3 grid, hipStream_t stream, const GemmArgs &g) {
    constexpr int T = WM * WN * 64;
    // the product of a layer's backward pass that takes G = (dH where H > 0) as its second operand
    if (g.b_gate || g.colsum) gemm_kernel<false, false, WM, WN, TI, TJ, 2><<<grid, T, 0, stream>>>(g);
    else if (!b_k) gemm_kernel<false, false, WM, WN, TI, TJ><<<grid, T, 0, stream>>>(g);
    else gemm_kernel<false, true, WM, WN, TI, TJ><<<grid, T, 0, stream>>>(g);
}

// k along the rows of A, few tiles and a long k
void launch_rows(bool b_k, dim3 grid, hipStream_t stream, const GemmArgs &g) {
    if (b_k) gemm_kernel<true, true, 2, 2, 2, 2><<<grid, 256, 0, stream>>>(g);
    else gemm_kernel<true, false, 2, 2, 2, 2><<<grid, 256, 0, stream>>>(g);
}

// Less than 16 k where the tall kernel does not apply (a weight gradient over a few rows): one result per thread.
__global__ void __launch_bounds__(256) few_k_kernel(const GemmArgs g) {
    const int64_t t = int64_t(blockIdx.x) * 256 + threadIdx.x;
    if (t >= g.M * g.N) return;
    const int64_t m = t / g.N, n = t - m * g.N;
    float x = 0.0f, col = 0.0f;
    for (int64_t k = 0; k < g.K; ++k) {
        const int64_t ib = k * g.sbk + n * g.sbn;
        const float b = (g.b_gate && !(g.b_gate[ib] > 0.0f)) ? 0.0f : g.B[ib];
        x = fmaf(g.A[m * g.sam + k * g.sak], b, x);
        col += b;
    }
    if (g.colsum && m == 0) g.colsum[n] = col;
    if (g.bias) x += g.bias[n];
    if (g.relu) x = x > 0.0f ? x : 0.0f;
    g.C[m * g.ldc + n] = x;
}

// C = act(sum over the partial planes + bias).  A workgroup owns 64 consecutive outputs; its wavefronts take every
// kReduceWaves-th plane, eight loads in flight each, and their sums are added in order.  (One thread per output walking
// all planes took 0.23 ms for 256 planes of 256 x 256, 67 MB.)  In 64 bits: adding the planes was most
// of the error of many short parts (24,490 rows, 256 x 256, 2-norm 1.5e-7 -> 0.8e-7), and the loads take longer than the additions.
// The workgroups from n_blocks on add up `rows` (a bias gradient), which as a kernel of its own took 4.5 us behind this one.
constexpr int kReduceWaves = 4;
__global__ void __launch_bounds__(kReduceWaves * 64) gemm_reduce_kernel(const float *__restrict__ part, int n_split, float *__restrict__ C,
                                                                       int64_t ldc, int64_t M, int64_t N,
                                                                       const float *__restrict__ bias, int relu, unsigned n_blocks,
                                                                       const float *__restrict__ rows, int64_t n_rows, int log2_cols, float *__restrict__ row_sum) {
    if (blockIdx.x >= n_blocks) {
        gnn_add_rows(rows, 0, n_rows, int(N), log2_cols, int(blockIdx.x - n_blocks), row_sum);
        return;
    }
    constexpr int U = 8;
    __shared__ double sums[kReduceWaves][64];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int64_t total = M * N;
    const int64_t t = int64_t(blockIdx.x) * 64 + lane;
    double s = 0.0;
    if (t < total) {
        int p = wave;
        for (; p + (U - 1) * kReduceWaves < n_split; p += U * kReduceWaves) {
            float v[U];
#pragma unroll
            for (int k = 0; k < U; ++k) v[k] = part[int64_t(p + k * kReduceWaves) * total + t];
#pragma unroll
            for (int k = 0; k < U; ++k) s += double(v[k]);
        }
        for (; p < n_split; p += kReduceWaves) s += double(part[int64_t(p) * total + t]);
    }
    sums[wave][lane] = s;
    __syncthreads();
    if (wave > 0 || t >= total) return;
    for (int w = 1; w < kReduceWaves; ++w) s += sums[w][lane];
    const int64_t m = t / N, n = t - m * N;
    if (bias) s += double(bias[n]);
    if (relu) s = s > 0.0 ? s : 0.0;
    C[m * ldc + n] = float(s);
}

}  // namespace

// Tile of a workgroup, for the weight gradients: a long k, read once where N fits the tile's width.  resident: parts of k that a
// compute unit gets in a round: a second, partly empty one costs a whole round (256 x 256 over 24,490 rows, 256 workgroups 30.6 us,
// 382 43.5; 60,000 56.7 and 512 64.4; 232,965 200 and 210; 100 x 256 over 60,000 37.6 and 52.5, over 2.45 M 1049 and 1065).  Tiles of 256
// columns take the registers of a compute unit by themselves.  Narrow tiles are small so that several workgroups, each waiting for
// memory, share one (602 x 16 over 232,965 rows: 306 us with tiles of 256 rows, two to a unit; 114 with 128 and five;
// 256 x 47 over 60,000 25.9 with three, 29.9 with four, over 232,965 71.6 and 73.0, over 600,000 178 and 173).
struct TileShape { int64_t bm, bn; int resident; };

static TileShape choose_tile(int64_t N, int64_t K) {
    if (N <= 32) return {128, 32, 5};
    if (N <= 64) return {128, 64, K > 400000 ? 4 : 3};
    if (N <= 128) return {128, 128, 2};
    return {128, 256, 1};
}

// Tile of a tall product: wavefronts of 32 rows, tiles of 32 columns.  As wide as the result, so that A is read and split once
// (2.45 M rows, 256 -> 47: 0.70 ms with two column tiles, 0.98 with one; 256 -> 256 2.0 with eight, 2.2 with four, 2.4 with
// two), unless that leaves compute units without a workgroup.  256 -> 256, us with tiles of 256 x 256 (one to a compute unit) and
// 128 x 64: 24,490 rows 44 and 28, 40,000 44 and 47, 49,152 (192 tiles, where the line is) 46 and 54, 100,000 93 and 105.
// 100 -> 128 with tiles of 128 x 128 and 128 x 64: 40,000 rows 17 and 15, 60,000 18 and 20, 65,536 (512 tiles, two to a compute unit)
// 19 and 20, 300,000 80 and 90.  Eight wavefronts instead of four share the split of B: nothing up to 65,536 rows, where the line
// is (602 -> 16, 20,000 rows 33 and 31 us), 1 to 4 % from there on (256 -> 47, 130,000 rows 35 and 37, 2.45 M 753 and 771).
struct TallShape { int waves, tj; };

static TallShape choose_tall(int64_t M, int64_t N) {
    // Fewer than six wavefronts of 32 x 64 per compute unit: twice as many of 32 x 32 (us: 6,000 rows 256 -> 256 17.2 and 15.7, 12,000 21.2 and
    // 19.7; 24,490 256 -> 47 18.3 and 16.4, 256 -> 100 19.5 and 18.1; above, 24,490 256 -> 256 27.8 and 38.2, 40,000 256 -> 100 24.3 and 32.7).
    if ((M + 31) / 32 * ((N + 63) / 64) < 1536) return {4, 1};
    const int waves = M >= 65536 ? 8 : 4;
    if (N <= 32) return {waves, 1};
    if (N <= 64) return {waves, 2};
    if (N <= 128) return {4, (M + 127) / 128 >= 512 ? 4 : 2};
    if ((M + 255) / 256 * ((N + 255) / 256) < 192) return {4, 2};
    return {8, 8};
}

// How many partial planes the reduction over k is split into.  Of the sizes alone, with the tiles of a weight gradient: a caller that
// asks for the workspace does not say which way A lies (launch_rows has tiles of its own).
static int64_t choose_split(int64_t M, int64_t N, int64_t K) {
    const TileShape s = choose_tile(N, K);
    const int64_t tiles = ((M + s.bm - 1) / s.bm) * ((N + s.bn - 1) / s.bn);
    if (tiles >= 512 || K < 1024) return 1;
    const int64_t max_split = K / GNN_SPLIT_MIN_K;
    // Rounds of workgroups: as few as leave the result as close as `enough` planes added in 32 bits did, two workgroups per compute unit (N <= 32:
    // five, N <= 64: four).  Error of normal operands, square of the 2-norm in 1e-14: 0.3 + 0.0021 K / parts, and 0.1 + 0.0095 planes for
    // that many of them in 32 bits.  So fewer, longer parts pass where there were many planes (256 x 256 over 30,000 rows 234 parts 1.6e-7, 60 us,
    // 128 0.9e-7, 48) and not where there were few (2000 x 2560 over 10,000, 4 parts 2.3e-7, 697 us, 2 3.2e-7, 868).  Two to sixteen tiles
    // of a part share an XCD (`inner` in gnn_matmul_impl), so a round has whole parts on each: 602 x 256, 5 tiles, over 100,000 rows 51 parts, a few workgroups
    // too many on some XCDs, 367 us, 103 304, 96 241; over 2.45 M 102 6.85 ms, 152 5.22; 602 x 128 over 100,000 102 196 us, 96 133.
    int64_t enough = (256 * (s.bn <= 32 ? 5 : s.bn <= 64 ? 4 : 2) + tiles - 1) / tiles;
    if (enough > max_split) enough = max_split;
    int64_t split = 0;
    for (int64_t rounds = 1; split < enough; ++rounds) {
        const int64_t slots = 32 * s.resident * rounds;  // per XCD
        split = tiles >= 2 && tiles <= 16 ? 8 * (slots / tiles) : 8 * slots / tiles;
        if (split > max_split) split = max_split;
        if (K <= 2048 * split && 2 * K * (enough - split) <= split * enough * (9 * enough + 96)) break;
    }
    // At least GNN_SPLIT_MIN_K rows per part: a part is bound by the latency of its tiles of 16, one after the other, while the chip is not
    // full; the partial planes cost little beside that.  Parts of 96 would be faster on few rows (24,490 rows, us with parts of 128 and of
    // 96: 128 x 128 22.3 and 18.5, 256 x 47 18.2 and 17.4, 16 x 41 16.0 and 15.2), but callers size their workspaces by 128.
    if (split > 4096) split = 4096;
    return split < 1 ? 1 : split;
}

extern "C" GNN_API int64_t gnn_matmul_workspace_bytes(int64_t M, int64_t N, int64_t K) {
    if (M <= 0 || N <= 0 || K <= 0) return 0;
    const int64_t split = choose_split(M, N, K);
    return split > 1 ? split * M * N * int64_t(sizeof(float)) : 0;
}

extern "C" GNN_API int gnn_matmul(const float *A, int64_t lda, int trans_a, const float *B, int64_t ldb, int trans_b,
                                  float *C, int64_t ldc, int64_t M, int64_t N, int64_t K, const float *bias, int relu,
                                  void *workspace, int64_t workspace_bytes, void *stream) {
    return gnn_matmul_impl(A, lda, trans_a, B, ldb, trans_b, C, ldc, M, N, K, bias, relu, workspace, workspace_bytes,
                           static_cast<hipStream_t>(stream));
}

int gnn_matmul_impl(const float *A, int64_t lda, int trans_a, const float *B, int64_t ldb, int trans_b, float *C, int64_t ldc,
                    int64_t M, int64_t N, int64_t K, const float *bias, int relu, void *workspace, int64_t workspace_bytes,
                    hipStream_t stream, const gnn_packed_target *packed, gnn_gemm_fold *fold) {
    if (M < 0 || N < 0 || K < 0) return GNN_ERR_INVALID_ARG;
    if (fold) { fold->n_planes = 0; fold->summed = false; }
    if (M == 0 || N == 0) return GNN_OK;
    const bool to_packed = packed && packed->active;
    if (!to_packed && (!C || ldc < N)) return GNN_ERR_INVALID_ARG;
    if (K > 0 && (!A || !B)) return GNN_ERR_INVALID_ARG;
    // stored shapes: A is [M, K] (or [K, M] when trans_a), B is [K, N] (or [N, K] when trans_b)
    if (K > 0 && (lda < (trans_a ? M : K) || ldb < (trans_b ? K : N))) return GNN_ERR_INVALID_ARG;
    if (reinterpret_cast<uintptr_t>(C) % 4 || reinterpret_cast<uintptr_t>(A) % 4 || reinterpret_cast<uintptr_t>(B) % 4)
        return GNN_ERR_INVALID_ARG;
    if (to_packed && (bias || relu)) return GNN_ERR_UNSUPPORTED;  // the aggregation that follows applies them
    if (to_packed && (!packed->base || !packed->rank || (packed->scale_mode && !packed->counts) ||
                      (packed->main_cols < N && !packed->tail)))
        return GNN_ERR_INVALID_ARG;
    // gates and column sums exist for the operand layouts of the layer's backward products only
    if (fold && fold->a_gate && (trans_a || fold->b_gate || fold->colsum)) return GNN_ERR_UNSUPPORTED;
    if (fold && (fold->b_gate || fold->colsum) && (!trans_a || trans_b)) return GNN_ERR_UNSUPPORTED;
    (void)hipGetLastError();

    GemmArgs g{};
    g.A = A; g.B = B; g.C = C; g.bias = bias;
    if (fold) { g.a_gate = fold->a_gate; g.b_gate = fold->b_gate; g.colsum = fold->colsum; }
    g.sam = trans_a ? 1 : lda;  g.sak = trans_a ? lda : 1;
    g.sbk = trans_b ? 1 : ldb;  g.sbn = trans_b ? ldb : 1;
    g.ldc = ldc; g.M = M; g.N = N; g.K = K;
    g.relu = relu ? 1 : 0;
    int64_t split = choose_split(M, N, K);
    if (split > 1 && (!workspace || workspace_bytes < split * M * N * int64_t(sizeof(float)))) split = 1;
    if (to_packed) {  // tall results only: no split reduction on this route
        split = 1;
        g.packed = *packed;
    }
    if (g.a_gate) split = 1;
    if (fold && fold->colsum) {
        if (fold->colsum_planes < split) return GNN_ERR_INVALID_ARG;
        fold->n_planes = split;
    }
    g.n_split = int32_t(split);
    g.k_per_split = split > 1 ? ((K + split - 1) / split + BK - 1) / BK * BK : (K > 0 ? K : 1);
    if (split > 1) {
        g.C = static_cast<float *>(workspace);
        g.ldc = N;
    }
    // the tall kernel takes every product with k along the rows of A whose reduction is not split
    const bool tall = !trans_a && split == 1;
    const TallShape ts = K < BK ? TallShape{4, 2} : choose_tall(M, N);
    const TileShape s = tall ? TileShape{ts.waves * 32, ts.tj * 32, 1} : trans_a ? choose_tile(N, K) : TileShape{128, 128, 2};
    const int64_t BM = s.bm, BN = s.bn;
    const int64_t gx = (M + BM - 1) / BM, gy = (N + BN - 1) / BN;
    if (gx > INT32_MAX || gy > INT32_MAX || split > 65535) return GNN_ERR_UNSUPPORTED;
    g.gx = int32_t(gx); g.gy = int32_t(gy); g.gz = int32_t(split);
    int64_t n_groups = gx * gy * split;
    const int64_t inner = split > 1 ? gx * gy : gy, outer = split > 1 ? split : gx;
    if (inner >= 2 && inner <= 16 && outer >= 16) {
        g.inner = int32_t(inner);
        n_groups = (outer + 7) / 8 * 8 * inner;
    }
    if (n_groups > INT32_MAX) return GNN_ERR_UNSUPPORTED;
    dim3 grid(static_cast<unsigned>(n_groups));
    const bool b_k = trans_b != 0;  // is k the contiguous direction of the operand?
    if (tall && K < BK) {
        if (K <= kFewProducts) launch_tall_few_k<2>(b_k, grid, stream, g);
        else launch_tall_few_k<1>(b_k, grid, stream, g);
    } else if (K < BK) {
        const int64_t blocks = (M * N + 255) / 256;
        if (blocks > INT32_MAX) return GNN_ERR_UNSUPPORTED;
        few_k_kernel<<<static_cast<unsigned>(blocks), 256, 0, stream>>>(g);
    } else if (tall) {
        if (ts.tj == 8) launch_tall<8, 8>(b_k, grid, stream, g);
        else if (ts.tj == 4) launch_tall<4, 4>(b_k, grid, stream, g);
        else if (ts.tj == 2 && ts.waves == 8) launch_tall<8, 2>(b_k, grid, stream, g);
        else if (ts.tj == 2) launch_tall<4, 2>(b_k, grid, stream, g);
        else if (ts.waves == 8) launch_tall<8, 1>(b_k, grid, stream, g);
        else launch_tall<4, 1>(b_k, grid, stream, g);
    } else if (!trans_a) launch_rows(b_k, grid, stream, g);
    else if (BN == 256) launch_gemm<2, 4, 2, 2>(b_k, grid, stream, g);
    else if (BN == 128) launch_gemm<2, 2, 2, 2>(b_k, grid, stream, g);
    else if (BN == 64) launch_gemm<4, 1, 1, 2>(b_k, grid, stream, g);
    else launch_gemm<4, 1, 1, 1>(b_k, grid, stream, g);
    if (hipGetLastError() != hipSuccess) return GNN_ERR_LAUNCH;
    if (split > 1) {
        const int64_t blocks = (M * N + 63) / 64;
        const float *rows = fold && fold->row_sum ? (fold->colsum ? fold->colsum : fold->rows) : nullptr;
        const int64_t n_rows = fold && fold->colsum ? split : fold ? fold->n_rows : 0;
        const bool add_rows = rows && n_rows <= GNN_ADD_ROWS;
        const int log2_cols = gnn_add_rows_log2_cols(N);
        const int64_t row_blocks = add_rows ? ((N - 1) >> log2_cols) + 1 : 0;
        if (blocks + row_blocks > INT32_MAX) return GNN_ERR_UNSUPPORTED;
        static_assert(kReduceWaves * 64 == 256, "the workgroups of gnn_add_rows");
        gemm_reduce_kernel<<<static_cast<unsigned>(blocks + row_blocks), kReduceWaves * 64, 0, stream>>>(
            static_cast<const float *>(workspace), int(split), C, ldc, M, N, bias, relu ? 1 : 0, static_cast<unsigned>(blocks), rows, n_rows, log2_cols,
            add_rows ? fold->row_sum : nullptr);
        if (hipGetLastError() != hipSuccess) return GNN_ERR_LAUNCH;
        if (fold) fold->summed = add_rows;
    }
    return GNN_OK;
}

// Internal layouts shared by the host packer and the HIP kernels.
// Not part of the public ABI.
#ifndef MGK_INTERNAL_H
#define MGK_INTERNAL_H

#include <stdint.h>

#if defined(__HIPCC__)
#define MGK_HD __host__ __device__
#else
#define MGK_HD
#endif

// One graph of a batch, as the device sees it.  All offsets index
// the batch-wide arrays of MgkBatchDev.
struct MgkGraphDesc {
    int32_t n;            // vertices
    int32_t nnz;          // stored nonzeros of the symmetric A (2 per edge)
    int32_t n_tiles;      // non-empty octiles
    int32_t n_tile_rows;  // ceil(n / 8)
    int32_t voff;         // first vertex in the per-vertex arrays
    int32_t zoff;         // first packed nonzero in w[] / e[]
    int32_t toff;         // first tile in tiles[]
    int32_t roff;         // first entry in trow_ptr[] (n_tile_rows + 1 entries)
    int32_t max_deg;      // largest number of nonzeros in a row
    int32_t lane_len;     // lane slots of the graph as inner operand (multiple of 64)
    int32_t loff;         // first lane slot of the graph in batch-wide expanded inner lists
    int32_t regs_runs;    // longest run of outer nonzeros of one wavefront under regs_split:
                          // 4 wavefronts in bits 0-15, 8 wavefronts in bits 16-31
    int32_t n_red;        // vertices that stay in the reduced system (see MgkReducedPlan)
    int32_t soff;         // first of the graph's 3 nnz entries in list_sched, if it has a schedule
    uint8_t red_need[8];  // most nonzeros of a wavefront in black and in red rows, with 2, with 4 and with 8
                          // wavefronts; 255 where there is no schedule
};

// Lane layout of a graph used as the inner operand of the on-chip XMV: the
// nonzeros of a row occupy adjacent lanes, and the sum over a row is a DPP
// shift-and-add inside one 16-lane row of a wavefront.  In a graph whose rows
// all have at most 16 nonzeros no row crosses a group of 16 lanes (a row that
// does not fit the rest of a group starts the next one), so every y_ii' has one
// writer.  A graph with longer rows needs atomic adds anyway (a long row is cut
// into several runs); there the rows are packed without gaps and every row that
// crosses a group boundary is cut at it.
#define MGK_LANE_GROUP 16

// Where nonzero `rank` of a row of `deg` nonzeros sits when the row starts at lane
// slot `first`: its position in its run (the part of the row inside one lane group),
// whether it is the last of the run, whether the row has more than one run.
struct MgkRunPos {
    uint32_t rank, last, cut;
};
static inline MGK_HD MgkRunPos mgk_run_pos(int first, int rank, int deg) {
    const int pos = first + rank;
    const int group = pos & ~(MGK_LANE_GROUP - 1);
    MgkRunPos r;
    r.rank = (uint32_t)(pos - (first > group ? first : group));
    r.last = (rank + 1 == deg || pos - group == MGK_LANE_GROUP - 1) ? 1u : 0u;
    r.cut = (first & (MGK_LANE_GROUP - 1)) + deg > MGK_LANE_GROUP ? 1u : 0u;
    return r;
}

// One non-empty octile (Section IV-A/B): tile coordinates, occupancy bitmap
// (bit 8*r + c <-> element (r, c) of the tile) and where its packed nonzeros
// start, relative to the graph's zoff.  Tiles of a graph are sorted by
// (tile_row, tile_col); nonzeros inside a tile are packed in bit order.
struct MgkTile {
    uint16_t tr, tc;
    uint32_t nzoff;
    uint64_t bitmap;
};

struct MgkBatchDev {
    const MgkGraphDesc* graphs;
    const MgkTile* tiles;
    const float* w;          // packed edge weights A_ij
    const float* e;          // packed edge labels E_ij
    const int32_t* vlabel;   // vertex labels (stored order)
    const float* rowsum;     // sum_j A_ij per vertex; d_i = rowsum + q (Eq. 1)
    const float* start;      // starting probability p_i
    const int32_t* rowptr;   // per vertex: nonzeros of the graph in rows before it
    const int32_t* lanepos;  // per vertex: first lane slot of its row (inner operand layout)
    const int32_t* trow_ptr; // per graph: tile-row pointers into its tile list
    const int32_t* tile_graph; // per tile: the graph it belongs to
    const int32_t* iperm;    // per vertex: original id of the stored vertex
    const struct MgkEntry* list_outer;  // per nonzero (CSR order, index zoff + k), see MgkEntry
    const struct MgkEntry* list_inner;  // per lane slot (index loff + slot)
    const int32_t* regs_split;  // per graph MGK_REGS_SPLIT_STRIDE row boundaries, see below
    const uint32_t* list_sched;  // nonzeros in the order of the wavefronts of the reduced solver, see below
    const uint16_t* red_split;  // per graph MGK_RED_SPLIT_STRIDE numbers, see below
    const uint16_t* red_order;  // the vertices of a graph (index 3 voff) in the order of the reduced solver, red ones
                                // first, for 2, 4 and 8 wavefronts
    const float* attr_outer;  // label attribute a of nonzero k (CSR order): attr_outer[a * nnz_total + zoff + k]
    const float* attr_inner;  // the same in lane order: attr_inner[a * lanes_total + loff + slot], 0 on idle slots
    const struct MgkSellDesc* sell_desc;    // per graph, see MgkSellDesc
    const struct MgkSellVertex* sell_vtx;   // records of the owner-computes solver
    const struct MgkSellNbr* sell_nbr;
    int32_t n_graphs, n_tiles_total, nnz_total, lanes_total;
    int32_t label_dim;        // attributes per edge label (1 for plain scalar labels)
    int32_t uniform_start;    // 1: no starting probabilities were given, p_i = 1/n on every graph
};

// One unit of work: solve the pair (outer graph g1 of batch X, inner graph g2
// of batch Y) and write the value to out0 (and to out1 if >= 0).  out1 == -2
// marks a job whose outer graph is the *second* graph of the requested pair
// (the orientation was exchanged); only the nodal output cares.
struct MgkJob {
    int32_t g1, g2;
    int32_t out0, out1;
};
#define MGK_OUT1_NONE (-1)
#define MGK_OUT1_SWAPPED (-2)

// Device pointers the solvers write to.  iters, flags, nodal may be null.
// nodal: solution x of pair k (original vertex numbering of the requested pair,
// row-major n x n') starts at nodal + nodal_off[out0].
struct MgkOutputs {
    float* K;
    int32_t* iters;
    int32_t* flags;
    float* nodal;
    const int64_t* nodal_off;
};

// Edge base kernels (Appendix B).  SE, POLY and CONST take one label per edge;
// KRON_SE and RCONV_SE take label_dim attributes (parts) per edge.
enum { MGK_EK_CONST = 0, MGK_EK_SE = 1, MGK_EK_POLY = 2, MGK_EK_KRON_SE = 3, MGK_EK_RCONV_SE = 4 };
#define MGK_MAX_LABEL_DIM 4
#define MGK_POLY_MAX_COEF 9

struct MgkParams {
    float q;          // stopping probability
    float h;          // vertex kernel off-diagonal value
    float e_scale;    // SE: sqrt(alpha * log2(e)), kappa_e = exp2(-((e-e')*e_scale)^2); POLY: 1 / rho
    float e_shift;    // common shift applied to labels before scaling
    float ke_const;   // constant edge kernel value
    float rtol2;      // rtol^2
    int32_t max_iter; // <= 0: automatic
    int32_t edge_kernel;
    int32_t label_dim;                     // attributes per edge label the kernel reads
    float attr_scale[MGK_MAX_LABEL_DIM];   // KRON_SE: sqrt(alpha_a log2(e)) per attribute; RCONV_SE: [0] for all parts
    float poly_c[MGK_POLY_MAX_COEF];       // POLY: sum_i poly_c[i] r^i on r = |e-e'| / rho < 1, zero-padded
};

#if defined(__HIPCC__)
// Compact polynomial radial basis kernel on the prescaled difference d = (e - e') / rho:
// Horner over all MGK_POLY_MAX_COEF coefficients (the unused high ones are 0), and
// 0 from |d| = 1 on.
__device__ __forceinline__ float mgk_poly_kernel(float d, const float* c) {
    const float r = __builtin_fabsf(d);
    const float rc = __builtin_fminf(r, 1.0f);
    float v = c[MGK_POLY_MAX_COEF - 1];
#pragma unroll
    for (int i = MGK_POLY_MAX_COEF - 2; i >= 0; --i) v = __builtin_fmaf(v, rc, c[i]);
    return r < 1.0f ? v : 0.0f;
}
#endif

// ---- LDS plan of the on-chip solver (one workgroup per pair) ---------------
// All offsets in 4-byte words from the start of dynamic LDS.  Computed the same
// way on the host (to size the launch) and in the kernel.
struct MgkSmallPlan {
    int32_t p, y;            // vectors, padded to waves * 64 * ept words each
    int32_t ent1, ent2;      // expanded nonzeros, 4 words each
    int32_t attr1;           // label attributes of the outer nonzeros, attr_dim arrays of z1pad words
    int32_t rowend;          // bit k set: outer entry k is the last of its row
    int32_t tiles1, tiles2;  // staged octile headers, 4 words each
    int32_t vtx1, vtx2;      // per vertex: d_i, start probability, label
    int32_t red;             // reduction scratch, 64 words
    int32_t total;           // words
    int32_t z1pad;           // outer entries padded (multiple of 4, + 4 spare)
    int32_t share;           // nominal outer entries per wave
    int32_t rowend_words;
};

// attr_dim: attributes per edge label for the kernels over label attributes, else 0
static inline MGK_HD MgkSmallPlan mgk_small_plan(int32_t n1, int32_t n2, int32_t z1,
                                                 int32_t lane_len2, int32_t t1, int32_t t2,
                                                 int32_t waves, int32_t ept, int32_t attr_dim) {
    MgkSmallPlan L;
    const int32_t np = waves * 64 * ept;   // >= n1 * n2: every thread owns ept elements
    (void)n1;
    L.z1pad = ((z1 + 3) & ~3) + 4;
    L.share = (z1 + waves - 1) / waves;
    if (L.share < 1) L.share = 1;
    L.rowend_words = L.z1pad / 32 + 2;
    L.p = 0;
    L.y = np;
    L.ent1 = 2 * np;
    L.attr1 = L.ent1 + 4 * L.z1pad;
    L.ent2 = L.attr1 + attr_dim * L.z1pad;
    L.rowend = L.ent2 + 4 * lane_len2;
    L.tiles1 = L.rowend + ((L.rowend_words + 3) & ~3);
    L.tiles2 = L.tiles1 + 4 * t1;
    L.vtx1 = L.tiles2 + 4 * t2;
    L.vtx2 = L.vtx1 + 3 * n1;
    L.red = L.vtx2 + 3 * n2;
    L.total = L.red + 64;
    return L;
}

// Largest product size N = n n' the on-chip solver takes: 16 waves x 16
// elements per thread.
#define MGK_SMALL_MAX_N (16 * 64 * 16)

#define MGK_LDS_LIMIT_BYTES (160 * 1024)

// ---- register-resident on-chip solver ----------------------------------------
// Four or eight wavefronts per pair.  Each wavefront owns a run of whole outer
// rows of at most SMAX nonzeros and keeps the off-diagonal matrix entries
// A_ij A'_i'j' kappa_e(E_ij, E'_i'j') of (its outer nonzeros) x (all inner lane
// slots) in registers for the whole solve; the inner graph takes `chunks`
// 64-lane chunks and has rows of at most 4 nonzeros.  LDS holds p, y, x and a
// dump area (each padded to the register blocks), the per-vertex data of both graphs and the
// reduction scratch.
#define MGK_REGS_SMAX_W4 24      // longest run of outer nonzeros per wavefront, 4 wavefronts
#define MGK_REGS_SMAX_W8 20      // the same with 8 wavefronts
#define MGK_REGS_MAX_CHUNKS 2
#define MGK_REGS_MAX_EPT 8
#define MGK_REGS_MAX_DEG 4       // inner rows: two shift-and-add steps

struct MgkRegsPlan {
    int32_t p, y, x, dump, vtx1, vtx2, red, total;  // words
};

static inline MGK_HD MgkRegsPlan mgk_regs_plan(int32_t n1, int32_t n2, int32_t waves, int32_t ept) {
    MgkRegsPlan L;
    const int32_t np = waves * 64 * ept;
    L.p = 0;
    L.y = np;
    L.x = 2 * np;
    L.dump = 3 * np;   // same shape as y, 2 np behind it: where lanes that hold no row sum store
    L.vtx1 = 4 * np;
    L.vtx2 = L.vtx1 + 3 * n1;
    L.red = (L.vtx2 + 3 * n2 + 3) & ~3;
    L.total = L.red + 64;
    return L;
}

// ---- register-resident solver of the reduced system -------------------------------
// The vertices of the outer graph are divided into "black" ones, no two of them adjacent, and "red" ones.
// Elements (i, i') of black i are not coupled to each other, so they are eliminated exactly and Alg. 1
// runs on the others,
//     (M_r - W_rr - W_rb M_b^-1 W_br) x_r = b_r + W_rb M_b^-1 b_b,   x_b = M_b^-1 (b_b + W_br x_r).
// One product of this matrix reads every entry of W once, as one of the full system does: first the black
// rows, whose sums (entries scaled by M_b^-1) go to the black part of p, then the red ones.  The stop test is the
// one of the full system: the eliminated elements have no residual.  Two, four or eight wavefronts per pair;
// each owns whole outer rows of both colours, at most MGK_RED_BLACK and MGK_RED_RED nonzeros, and
// keeps their entries in registers as the solver of the full system does.  LDS holds p (the red part padded to
// the register blocks), y of the red rows, 64 words that lanes without a row sum store to, the
// per-vertex data of both graphs and the reduction scratch.
#define MGK_RED_BLACK(waves) ((waves) == 2 ? 16 : (waves) == 4 ? 12 : 8)   // multiples of 4: the fill takes four nonzeros a step
#define MGK_RED_RED(waves) ((waves) == 2 ? 20 : (waves) == 4 ? 16 : 12)
#define MGK_RED_MAX_NNZ 160      // of the outer graph: 8 x (8 + 12)
#define MGK_RED_MAX_P 16384      // words of p: byte offsets of its rows are kept in 16 bits

struct MgkReducedPlan {
    int32_t p, black, y, dump, vtx1, vtx2, red, total;  // words
};

static inline MGK_HD MgkReducedPlan mgk_reduced_plan(int32_t n1, int32_t n_red, int32_t n2, int32_t waves, int32_t ept) {
    MgkReducedPlan L;
    const int32_t np = waves * 64 * ept;   // >= n_red n2
    L.p = 0;
    L.black = np;
    L.y = L.black + (n1 - n_red) * n2;
    L.dump = L.y + np;
    L.vtx1 = L.dump + 64;
    L.vtx2 = L.vtx1 + 3 * n1;
    L.red = (L.vtx2 + 3 * n2 + 3) & ~3;
    L.total = L.red + 64;
    return L;
}

// ---- owner-computes on-chip solver (graphs of at most 64 vertices, degree <= 4) ----
// Every element (i, i') of the product vectors has one owning lane, which keeps the
// off-diagonal entries of its row of the system -- deg(i) deg(i') of them, about four on
// molecule-like graphs -- in registers together with the LDS address of the element of p
// each one multiplies.  Lanes that work side by side must own rows of equal length, so
// the vertices of a graph are sorted by degree (descending) at load and grouped: groups
// of 4 when the graph is the outer operand, groups of 8 when it is the inner one.  A
// "tile" is (outer group U) x (inner group V): 32 elements = one half of a wavefront,
// all of whose rows have at most maxdeg(U) * maxdeg(V) entries.  Tiles are enumerated by
// (maxdeg(U) descending, maxdeg(V) descending); tile number h is held by lanes
// 32 (h & 1) .. + 31 of a wavefront (mgk_sell_wave_of) in its vector slot (h / 2) / W, lane
// 8 u + v owning (vertex u of U, vertex v of V).  An element's p value lives in LDS at
// a word that is 8 u + v modulo 32, so its bank is 8 (k & 3) + (k' & 7) for sorted positions k, k':
// a gather by the 32 lanes of a tile is free of bank conflicts when the a-th neighbours
// of the 4 outer vertices sit at positions distinct mod 4 and the b-th neighbours of the
// 8 inner vertices at positions distinct mod 8 (the loader orders the vertices inside a
// degree class, and each vertex's neighbour list, toward that).
#define MGK_SELL_MAX_N 64        // vertices per graph
#define MGK_SELL_MAX_DEG 4
#define MGK_SELL_OUTER_GROUP 4
#define MGK_SELL_INNER_GROUP 8

// Per graph: where its records start (8 ceil(n / 8) vertex records, 4 neighbour records
// each) and how many outer / inner groups have each maximum degree 0..4.  ok == 0: the
// graph does not qualify (too many vertices or a vertex of higher degree).
struct MgkSellDesc {
    int32_t voff;
    uint32_t ga03;   // groups of 4 whose maximum degree is 0..3, one byte each
    uint32_t gb03;   // groups of 8 whose maximum degree is 0..3
    uint32_t hi;     // groups of 4 with maximum degree 4 | groups of 8 with maximum degree 4 << 8 | ok << 16
};
static inline MGK_HD int mgk_sell_ga(const MgkSellDesc& d, int deg) {
    return (int)((deg < 4 ? d.ga03 >> (8 * deg) : d.hi) & 0xffu);
}
static inline MGK_HD int mgk_sell_gb(const MgkSellDesc& d, int deg) {
    return (int)((deg < 4 ? d.gb03 >> (8 * deg) : d.hi >> 8) & 0xffu);
}
static inline MGK_HD bool mgk_sell_ok(const MgkSellDesc& d) { return ((d.hi >> 16) & 1u) != 0u; }
// Vertex at sorted position k: row sum of A, starting probability, label, and
// (vertex id in stored order) | degree << 16.  Positions >= n are padding (degree 0, id 0xffff).
struct alignas(16) MgkSellVertex {
    float rowsum, start;
    int32_t label;
    uint32_t id_deg;
};
// a-th neighbour of the vertex at sorted position k (record 4 k + a): the neighbour's
// sorted position, A_ij, E_ij.  a >= degree: weight 0, position k itself.
struct alignas(16) MgkSellNbr {
    uint32_t pos;
    float w, e;
    uint32_t pad;
};

// Tiles 2 s and 2 s + 1 share vector slot s / W of wavefront s % W, counted back and forth
// (W - 1 - s % W in odd rounds): rows get shorter with s, and this way no wavefront takes
// the longest rows of every round.
static inline MGK_HD int mgk_sell_wave_of(int s, int waves) {
    const int m = s / waves, j = s - m * waves;
    return (m & 1) ? waves - 1 - j : j;
}

// LDS plan of the owner-computes solver, in words.
struct MgkSellPlan {
    int32_t p, y, x;          // slot layout, waves * 64 * ept words each
    int32_t vtx1, nbr1, vtx2, nbr2;
    int32_t table, rankof;    // tile number -> (U, V, A, B); U * G2 + V -> byte address of the tile's 32 words of p
    int32_t sched;            // per wavefront and slot: entries | (entries per outer neighbour) << 8
    int32_t misfit;           // per wavefront: 1 when its rows do not fit the launch shape
    int32_t red, total;
};
static inline MGK_HD MgkSellPlan mgk_sell_plan(int32_t n1, int32_t n2, int32_t waves, int32_t ept) {
    MgkSellPlan L;
    const int32_t np = waves * 64 * ept;
    const int32_t r1 = (n1 + 7) & ~7, r2 = (n2 + 7) & ~7;   // staged records per graph
    const int32_t tiles = ((n1 + 3) / 4) * ((n2 + 7) / 8);
    L.p = 0;
    L.y = np;
    L.x = 2 * np;
    L.vtx1 = 3 * np;
    L.nbr1 = L.vtx1 + 4 * r1;
    L.vtx2 = L.nbr1 + 16 * r1;
    L.nbr2 = L.vtx2 + 4 * r2;
    L.table = L.nbr2 + 16 * r2;
    L.rankof = L.table + ((tiles + 3) & ~3);
    L.sched = L.rankof + ((tiles + 3) & ~3);
    L.misfit = L.sched + waves * ept;
    L.red = (L.misfit + waves + 3) & ~3;
    L.total = L.red + 64;
    return L;
}

// Order of the tile classes (A, B) = (largest degree of the outer group, of the inner
// group): classes with entries first, by A descending then B descending, then the classes
// without entries (A or B zero: isolated vertices) in the same order.  True when class
// (a, b) comes before class (A, B).
static inline MGK_HD bool mgk_sell_class_before(int a, int b, int A, int B) {
    const bool z = a * b == 0, Z = A * B == 0;
    if (z != Z) return Z;
    return a > A || (a == A && b > B);
}

// Walk of the tiles of a pair in the order the kernel numbers them, for the host planner
// (does the pair fit a launch shape?): returns the largest number of entry registers any
// wavefront needs with `waves` wavefronts, the number of vector slots per lane in *slots
// and the entries all wavefronts execute together in *executed.
static inline int32_t mgk_sell_need(const MgkSellDesc& o, const MgkSellDesc& i, int32_t waves, int32_t* slots,
                                    int32_t* executed) {
    int32_t per_wave[16] = {0};
    int32_t h = 0, prevA = 0, prevB = 0;
    for (int pass = 0; pass < 2; ++pass)   // classes with entries, then those without
        for (int A = MGK_SELL_MAX_DEG; A >= 0; --A)
            for (int B = MGK_SELL_MAX_DEG; B >= 0; --B) {
                if ((A * B == 0) != (pass == 1)) continue;
                const int32_t cnt = mgk_sell_ga(o, A) * mgk_sell_gb(i, B);
                for (int32_t k = 0; k < cnt; ++k, ++h) {
                    if (h & 1) {
                        const int32_t a = A > prevA ? A : prevA, b = B > prevB ? B : prevB;
                        per_wave[mgk_sell_wave_of(h >> 1, waves)] += a * b;
                    } else {
                        prevA = A;
                        prevB = B;
                    }
                }
            }
    if (h & 1) per_wave[mgk_sell_wave_of(h >> 1, waves)] += prevA * prevB;
    int32_t need = 0, sum = 0;
    for (int w = 0; w < waves; ++w) { need = per_wave[w] > need ? per_wave[w] : need; sum += per_wave[w]; }
    *slots = ((h + 1) / 2 + waves - 1) / waves;
    if (executed) *executed = sum;
    return need;
}

// ---- separable edge kernel (mgk_sep.hip) --------------------------------------
// kappa_e(e, e') = sum_{k < rank} phi_k(e) phi_k(e') on the label range of the batches, with
//   phi_k(e) = s^(k mod 2) sum_{m < terms} coef[m][k] s^(2 m),   s = (e - center) / R in [-1, 1].
// exp(-(e - e')^2 / 2 l^2) is the product of two Gaussians and exp(u u' / l^2), u = e - center,
// whose Chebyshev coefficients on [-R, R]^2 form a positive definite matrix that falls off faster
// than geometrically.  The first `rank` columns of its Cholesky factor, all their rows, times the
// Gaussian are the phi_k; each is even or odd.  The constant kernel is rank 1.  The host takes
// the smallest rank whose truncation error is at most MGK_SEP_TOLERANCE, half a unit in the last place of
// the largest value of kappa_e, on a grid over the range in double (6.0e-8 at most between its points).
// The features are then rounded to fp32, which adds up to 2^-23: 0.9e-7 in all at length scales of 0.7 to
// 1.7 times the range, 1.0e-7 the most found.  It is an absolute error: a value far below 1 (labels far
// apart) has lost that much of itself, the kernel values of pairs have not moved by more than 1e-8.
#define MGK_SEP_MAX_RANK 16
#define MGK_SEP_MAX_TERMS 16
#define MGK_SEP_TOLERANCE 5.9e-8
struct MgkSepBasis {
    int32_t rank, terms;
    double center, inv_r;
    double coef[MGK_SEP_MAX_TERMS * MGK_SEP_MAX_RANK];   // [m][k]
};
// How the rank is divided for the sparse product: `passes` passes of `rk` (1, 4, 5, 6 or 7)
// features each, per_packet nonzeros to a packet of 16 words (rk coefficients and one offset
// per nonzero).  slab_bytes: LDS bytes of one column of T.
// numbers: packets (of at most 14 words) also hold the numbers of the columns, from word MGK_SEP_NUMBER_SLOT on.
struct MgkSepLayout {
    int32_t rk, passes, per_packet, slab_bytes, numbers;
};
#define MGK_SEP_NUMBER_SLOT 14
#define MGK_SEP_ROWS 16       // outer rows per workgroup: one row of 16 lanes
#define MGK_SEP_THREADS 1024
#define MGK_SEP_DENSE_ROWS 32 // the same of the dense form: one tile
#define MGK_SEP_DENSE_THREADS 256
#define MGK_SEP_SLAB(rk) ((rk) == 1 ? 17 : 64 * (((rk) + 3) / 4) + 4)   // words per column of T
#define MGK_SEP_DENSE_MAX_N 1024
#define MGK_SEP_PARTS_MAX_N 256   // of the dense form with operands in three 16-bit parts: eight wavefronts of 32 rows
#define MGK_SEP_PARTS_THREADS 512
#define MGK_SEP_PARTS_LDS 101376
static inline MGK_HD bool mgk_sep_in_parts(int32_t max_n1, int32_t max_n2) { return max_n1 <= MGK_SEP_PARTS_MAX_N && max_n2 <= MGK_SEP_PARTS_MAX_N; }
static inline MGK_HD int32_t mgk_sep_per_packet(int32_t rk) { return rk == 1 ? 8 : 2; }
static inline MGK_HD int64_t mgk_sep_lds_bytes(int32_t rk, int32_t n2) {
    return 4 * ((int64_t)MGK_SEP_SLAB(rk) * n2 + (int64_t)MGK_SEP_ROWS * (n2 | 1));
}
// Workgroups of a launch: pairs in eights (one per XCD) by blocks of rows of the largest outer graph.
static inline MGK_HD int64_t mgk_sep_grid(int64_t n_pairs, int32_t max_n1, int32_t rows) {
    return (n_pairs + 7) / 8 * 8 * ((max_n1 + rows - 1) / rows);
}
// Tiles of 64 columns per wavefront of the dense form, 4 wavefronts: 1, 2 or 4.
static inline MGK_HD int32_t mgk_sep_dense_tiles(int32_t max_n2) { return max_n2 <= 256 ? 1 : max_n2 <= 512 ? 2 : 4; }
// What the separable product reads beside MgkBatchDev.  Packets come in steps of 64 words (four
// rows of adjacent rank in deg_order, one packet each): pass q at packets + q total 64; group t of graph g
// has steps at + gptr[qoff[g] + t] .. at + gptr[qoff[g] + t + 1], gptr counting over the whole batch and
// `at` the graph's MgkSepGraph::at.  One step more than all passes have is allocated: stage 2 loads the
// first packet of a group before it looks whether it has one.
struct MgkSepGraph;
struct MgkSepList {
    const int32_t* qoff;        // per graph: first entry in gptr
    const int32_t* gptr;        // per four vertices of a graph, and one more per graph
    const MgkSepGraph* whole;   // all graphs in order, `at` as for dense F_k (0 for packets)
    const int32_t* deg_order;   // per graph (index voff): its vertices by descending number of nonzeros
    const float* packets;
    const float* dense;         // dense F_k
    int32_t total;
};
// A graph whose features a call forms, and where they are: dense F_k from float `at` times the rank on,
// packets see above.
struct MgkSepGraph {
    int64_t at;
    int32_t graph, unused;
};
// Where the features of the two graphs of a pair are (float of F_0, or `at` of the packets); beside the pair's record, which the direct product's kernels
// read in every workgroup (16 bytes more there: 59.8 -> 60.6 us a product of 64 pairs, n = 256, density 0.01)
struct MgkSepAt {
    int64_t f1, f2;
};

// ---- the same for graphs of many vertices (mgk_sep_wide.hip) ---------------------
// kappa_e(e, e') = g(e') sum_{l < rank} psi_l(e) s'^l: psi_l is function l of `outer`, g(e') = exp(-half_t s'^2), s' = (e' - center) / R.
// kappa_e / g has a Chebyshev sum in s' of `rank` terms, whose powers of s' have the psi_l as coefficients.  Tolerance as above.
struct MgkWideBasis {
    MgkSepBasis outer;
    double half_t;
};
// Pass 0 takes the `hi` highest functions, every other one the next `lo`; 4 and 4, 4 and 5 or 5 and 5, or all (4 to 6, 8 to 10) in one
// pass.  rows: outer rows of a workgroup, 4 or 8.
struct MgkWideLayout {
    int32_t rows, hi, lo, passes;
};
#define MGK_WIDE_THREADS 1024
#define MGK_WIDE_MAX_N 2048
#define MGK_WIDE_MAX_ELEMENTS 8192   // rows by columns of a workgroup: eight results to a thread, or four where two workgroups share a CU
static inline MGK_HD int32_t mgk_wide_first(const MgkWideLayout& L, int32_t q) { return (L.passes - 1 - q) * L.lo; }
static inline MGK_HD int64_t mgk_wide_lds_bytes(const MgkWideLayout& L, int32_t n2) {
    const int64_t t = (int64_t)n2 * L.rows * 4 * (L.passes > 1 && L.lo > L.hi ? L.lo : L.hi), y = 4 * ((int64_t)L.rows * (n2 | 1) + MGK_WIDE_THREADS / 64);
    return t > y ? t : y;
}
static inline MGK_HD constexpr int32_t mgk_wide_record(int32_t hi) { return hi > 6 ? 12 : 8; }   // words of a nonzero of an outer graph, per pass
// Byte offset of the four first values of column j of T, row 0; row r's are at that ^ 16 r.
static inline MGK_HD uint32_t mgk_wide_column(int32_t rows, uint32_t j) {
    return rows == 4 ? j * 64u + ((j >> 2) & 3u) * 16u : j * 128u + ((j >> 1) & 7u) * 16u;
}
// Words in front of the steps of an inner graph, and the most steps it can have (groups of 16 vertices by descending
// degree, four nonzeros to a step: the largest of a group is at most the mean of the group before).
static inline MGK_HD int32_t mgk_wide_head(int32_t n) { return ((n + 15) / 16 + 1 + 63) & ~63; }
static inline MGK_HD int32_t mgk_wide_steps(const MgkGraphDesc& g) { return (g.n + 15) / 16 + (g.max_deg + 3) / 4 + g.nnz / 64 + 1; }
static inline MGK_HD int64_t mgk_wide_inner_words(const MgkGraphDesc& g, int32_t passes) {
    return mgk_wide_head(g.n) + (int64_t)passes * mgk_wide_steps(g) * 192;
}
static inline MGK_HD int64_t mgk_wide_grid(int64_t n_pairs, int32_t max_n1, int32_t rows) {
    return n_pairs * ((((max_n1 + rows - 1) / rows + 7) >> 3) << 3);
}
// Two workgroups of this layout share a compute unit (the kernel for that has fewer registers).
static inline MGK_HD bool mgk_wide_two(const MgkWideLayout& L, int32_t n2) {
    return 2 * L.rows * n2 <= MGK_WIDE_MAX_ELEMENTS && 2 * mgk_wide_lds_bytes(L, n2) <= MGK_LDS_LIMIT_BYTES;
}
// What a workgroup needs to know of its pair, in one place: every further record to look up is one more trip to memory
// before the work begins.
struct alignas(64) MgkWidePair {
    int64_t vec, f1, f2;   // vectors; first record of the outer graph; first word of the inner one
    int32_t n1, n2, npad, nnz1, voff1, voff2, cap2, unused[3];
};
// Features of the graphs of a call: records of the outer graphs' nonzeros (mgk_wide_record words each, pass after pass of outer_total
// records, a graph's from MgkWidePair::f1 on) and steps of the inner ones (from word MgkWidePair::f2 on).
struct MgkWideFeatures {
    const float* outer;
    const float* inner;
    const int32_t* deg_order2;
    int64_t outer_total;
};

// ---- whole solve on chip with the separable product (mgk_pcg_sep.hip) ----------
// Columns are the vertices of the smaller graph (n2 <= n1).  p and y with rows of n2 | 1 words, T of rb blocks of 16 rows, per-vertex data, first packet steps and reduction scratch.
#define MGK_PCG_SEP_SLAB(rk) ((rk) == 1 ? 17 : 16 * (rk) + 4)   // words of one column of T for 16 rows
static inline MGK_HD bool mgk_pcg_sep_numbers(int32_t rk) { return rk >= 4 && rk <= 6; }   // see MgkSepLayout
#define MGK_PCG_SEP_MAX_N (16 * 64 * 14)
#define MGK_ONCHIP_PACKET_BYTES ((int64_t)256 << 20)   // of packets of both batches of a call; beyond, the streaming solver
struct MgkPcgSepPlan {
    int32_t y, t, vtx1, vtx2, gptr, red, total;  // words; p at 0
};
static inline MGK_HD MgkPcgSepPlan mgk_pcg_sep_plan(int32_t n1, int32_t n2, int32_t rk, int32_t rb) {
    MgkPcgSepPlan L;
    L.y = n1 * (n2 | 1);
    L.t = (2 * L.y + 3) & ~3;
    L.vtx1 = L.t + MGK_PCG_SEP_SLAB(rk) * n2 * rb;
    L.vtx2 = L.vtx1 + 3 * n1;
    L.gptr = L.vtx2 + 3 * n2;
    L.red = L.gptr + (n1 + 3) / 4 + (n2 + 3) / 4 + 2;
    L.total = L.red + 64;
    return L;
}

// ---- solver with vectors in global memory (pairs too large for LDS) ---------
// Expanded nonzero lists of a whole batch, rebuilt per call because the label
// scaling depends on the edge-kernel parameters:
//   outer list (CSR order, index zoff + position): {col, scaled label or
//     weight, log2 weight, row}
//   inner list (lane layout, index loff + slot): {row, col | rank in run << 24
//     | row longer than a lane group << 30 | last of run << 31, scaled label or
//     weight, log2 weight (the weight itself for the kernels that multiply by it)}
struct alignas(16) MgkEntry {
    uint32_t x, y, z, w;
};

// Parameter-free nonzero lists written once at load (list_outer / list_inner of
// MgkBatchDev) for the register-resident on-chip solver, which reads a graph's
// nonzeros straight into lanes:
//   list_outer[zoff + k], CSR order: {row, col, label bits, weight bits | bit 31
//     set when k is the last nonzero of its row (weights are > 0)}
//   list_inner[loff + slot], lane layout: {row | rank in run << 20 | row longer
//     than a lane group << 30 | last of run << 31, col, label bits, weight bits
//     (0.0f for an idle slot)}

// Outer rows of a graph divided among the wavefronts of the register-resident solver
// (whole rows, contiguous, the most loaded wavefront as light as possible; written at
// load): regs_split[g * MGK_REGS_SPLIT_STRIDE + k], k = 0..4: wavefront w of 4 owns
// rows [b[w], b[w+1]); k = 5..13: the same for 8 wavefronts.
#define MGK_REGS_SPLIT_STRIDE 14
#define MGK_REGS_SPLIT_W8 5

//   list_sched, for graphs that can be outer operand of the reduced solver: for 2, for 4 and for 8
//     wavefronts the graph's nnz nonzeros, wavefront after wavefront, its black rows, then its red rows;
//     k of list_outer | position of the column in red_order << 16
//
// red_split[g * MGK_RED_SPLIT_STRIDE + MGK_RED_SPLIT(waves) + ..]: waves + 1 numbers where the wavefronts' parts of
// list_sched begin, then for every wavefront the number of its nonzeros in black rows, and the positions in
// red_order of its first black row and its first red row (its rows follow there in the order of the list).
#define MGK_RED_SPLIT_STRIDE 59
#define MGK_RED_SPLIT(waves) ((waves) == 2 ? 0 : (waves) == 4 ? 9 : 26)
#define MGK_RED_LIST(waves) ((waves) == 2 ? 0 : (waves) == 4 ? 1 : 2)   // which of the three lists and orders

struct MgkExpanded {
    const MgkEntry* outer;
    const MgkEntry* inner;
};

// Octiles of a batch expanded to dense 8x8 blocks (64 floats per tile each).
struct MgkDenseTiles {
    const float* w;    // A_ij, 0 where absent
    const float* e;    // scaled label, 0 where absent
    const float* lw;   // log2 A_ij, -inf where absent
};

// One pair solved with global-memory vectors.  Vector v of the pair starts at
// vec + v * npad floats: 0 x, 1 r, 2 p, 3 M, 4 y (also holds z).  With the separable product 3 is
// not used and 4 is a = M p - y.
struct MgkLargePair {
    int32_t g1, g2;        // outer graph (batch X), inner graph (batch Y)
    int32_t n1, n2;
    int64_t vec;           // offset of the pair's vectors in the scratch array (floats)
    int32_t npad;          // n1 * n2 rounded up to 64
    int32_t out0, out1;
    int32_t max_iter;
    union {
        struct {
            int32_t nsteps;        // direct product: DPP steps for the inner row sums
            int32_t atomic_rows;   // inner graph has rows longer than a lane group
        };
        struct {
            int32_t voff1, voff2;  // separable product: first vertices of the two graphs
        };
    };
};

// What the vector kernels of the separable product read beside the pairs: it follows the two counters of a call
// (MGK_COUNTERS_BYTES from them), so that M is formed from the vertex data where it is used.
struct MgkVectorEnv {
    const float *rowsum1, *rowsum2;
    const int32_t *vlabel1, *vlabel2;
    float q, h;
};
#define MGK_LEAN_THREADS 512       // of their workgroups,
#define MGK_LEAN_ELEMENTS 2048     // which take as many elements at a time, four to a thread
// body(first element) for every four of the elements of thread `thread` of workgroup `block`; two at a time where there are as many, so
// that their loads are in flight together.  `end` may be close to 2^31: a step past it stays positive.
template <class F>
MGK_HD inline void mgk_each_quad(uint32_t block, uint32_t blocks, uint32_t thread, int32_t end, const F& body) {
    static_assert(MGK_LEAN_ELEMENTS == 4 * MGK_LEAN_THREADS, "four elements to a thread");
    const uint32_t step = blocks * MGK_LEAN_ELEMENTS, last = (uint32_t)end;
    for (uint32_t at = block * MGK_LEAN_ELEMENTS + 4 * thread; at < last; at += 2 * step) {
        body((int32_t)at);
        if (at + step < last) body((int32_t)(at + step));
    }
}
static inline MGK_HD int32_t mgk_lean_blocks(int64_t n_pairs, int32_t max_npad) {   // at most about a thousand in all: each adds to the sums of its pair
    const int64_t most = n_pairs < 64 ? 1024 / n_pairs : 16, all = ((int64_t)max_npad + MGK_LEAN_ELEMENTS - 1) / MGK_LEAN_ELEMENTS;
    return (int32_t)(all < 1 ? 1 : all < most ? all : most);
}
#define MGK_COUNTERS_BYTES 64

// Scalars of one pair in the global-memory solver.  The three sums of iteration `it` go
// to slot it & 1 of their pair of accumulators; the other slot is cleared meanwhile, by a
// kernel that runs when nobody reads it (no separate scalar kernels, no host round trip):
//   rz[it & 1]        r^T z after the update of iteration it; rz[(it + 1) & 1] is the one
//                     of the iteration before (rho of Alg. 1; the set-up puts it in rz[1])
//   pa[it & 1]        p^T a of iteration it
//   rr[it & 1]        r^T r after the update of iteration it
// done: 0 while the pair iterates, else 1 + its last iteration (the separable product's solver; 1 in the other).
struct MgkPairState {
    float rz[2], pa[2], rr[2];
    float bb;       // b^T b
    float kval;
    int32_t iters, done, flag;
    int32_t check;  // a stopped pair whose true residual is being formed
    int32_t growth; // bits of max_i x_i / (M^{-1} b)_i >= 1: how far the solution exceeds the Jacobi guess
};

// A pair whose solution exceeds M^{-1} b by more than this factor somewhere is checked
// after the solve: one more product gives the true residual b - S x in fp32, and if
// (true relative residual) x (that factor) exceeds MGK_VERIFY_ACCURACY the pair's flag
// becomes 3.  Below the threshold even a residual at fp32 rounding level cannot move the
// value by that much, so nothing is checked.
#define MGK_VERIFY_GROWTH 32.0f
#define MGK_VERIFY_ACCURACY 1e-4f

#define MGK_LARGE_ROWS_PER_BLOCK 8    // outer rows per workgroup of the large XMV
#define MGK_LARGE_CHUNKS_PER_WAVE 2   // 64-lane chunks of the inner layout per wave
#define MGK_LARGE_WAVES 4
#define MGK_ROWS_MAX_BATCH 64         // rows of p (= outer nonzeros) staged at a time by the row-staged XMV

#endif

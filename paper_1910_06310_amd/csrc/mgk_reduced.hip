// Register-resident solver of the reduced system: one workgroup of two, four or eight
// wavefronts runs the whole preconditioned CG iteration (Alg. 1) for one graph pair whose
// off-diagonal matrix fits in the register file, on the red elements only (MgkReducedPlan).
//
// Entries, lanes and products are those of mgk_regs.hip: each lane owns one nonzero (i', j') of the
// inner graph per 64-lane chunk, each wavefront whole rows of the outer graph, register kap[c][k] of a lane
// holds the entry for the wavefront's k-th outer nonzero and the lane's inner nonzero of chunk c, and
// the sum over the lanes of an inner row at the end of an outer row is a DPP shift-and-add.
//
// Molecule-like graphs have 55 % black vertices, and the reduced system takes about 7 iterations to the same
// residual where the full one takes 11: the products of an iteration cost the same (every entry once),
// the vector part 45 %.  Gram matrix of 2000 graphs of 20 to 60 vertices (2 001 000 pairs): 62.7 ms with the full
// system, 39.4 ms with this; of 100 graphs of 10 to 40: 133 and 80 us.  Bound by the vector instructions (2.0e10 per
// Gram of the first, 2.96e10 with the full system; 86 % of their slots at four wavefronts per SIMD, LDS 55 %) and by what
// waits at five barriers an iteration.  What holds fewer registers counts twice, for the fourth wavefront: offsets of two
// rows of p in one scalar register, conditions and addresses formed in the iteration and not before it, rows of a
// wavefront that follow each other in y so that their address is a scalar sum (together 56 -> 43 ms).  <8, 8, 2> spills
// one vector register to keep four wavefronts, the other shapes none.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "mgk_internal.h"
#include "mgk_launch.h"
#include "mgk_regs_dev.h"
#include "mgk_wave.h"

namespace {

// Entries of the black rows (outer nonzeros below KEND) times 1 / M_ii' of their row (i, i'): d1 = 1 / d_i and lab1 the
// label of i in the lanes of the outer nonzeros, d2 = 1 / d_i' (d2h: h times that) and lab2 of this lane's i'.
template <int K0, int KEND, int SMAX, int C>
__device__ __forceinline__ void scale_black(float (&kap)[C][SMAX], int stop, const float (&d2)[C], const float (&d2h)[C],
                                            const int (&lab2)[C], float d1, int lab1) {
    if constexpr (K0 < KEND) {
        if (K0 < stop) {
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const float s1 = lane_value(d1, K0 + u);
                const int l1 = (int)lane_value((uint32_t)lab1, K0 + u);
#pragma unroll
                for (int c = 0; c < C; ++c) kap[c][K0 + u] *= s1 * (l1 == lab2[c] ? d2[c] : d2h[c]);
            }
            scale_black<K0 + 4, KEND, SMAX, C>(kap, stop, d2, d2h, lab2, d1, lab1);
        }
    }
}

// per-lane constants of the inner nonzeros, one set per chunk
template <int C>
struct InnerLanes {
    uint32_t jp[C];                   // byte offset of column j' in a row of p
    uint32_t holds[C], ip[C];         // a lane that is the last of its run holds the sum of row i': 1 and the byte offset of i' in
                                      // a row; others 0 and a byte address in the dump area
    float m1[C], m2[C];               // 1 if the lane is at least that far into its run, else 0
};

// Sums of u and v over the wavefront: lane 31 holds u's, lane 63 v's.  The halves of the two registers are
// exchanged first, so that the rest of the tree serves both.
__device__ __forceinline__ float wave_sum_pair(float u, float v) {
    const auto w = __builtin_amdgcn_permlane32_swap(__float_as_uint(u), __float_as_uint(v), false, false);
    float t = __uint_as_float(w[0]) + __uint_as_float(w[1]);   // low halves of u and v, and their high halves
    t = dpp_add<0xB1>(t);   // quad_perm [1,0,3,2]
    t = dpp_add<0x4E>(t);   // quad_perm [2,3,0,1]
    t = dpp_add<0x141>(t);  // row_half_mirror
    t = dpp_add<0x140>(t);  // row_mirror
    asm("s_nop 1\n\tv_add_f32_dpp %0, %0, %0 row_bcast:15 row_mask:0xa bank_mask:0xf\n\ts_nop 0" : "+v"(t));
    return t;
}

// Sum of the W values in lanes W q .. W q + W - 1, in lane W q.
template <int W>
__device__ __forceinline__ float partial_sum(float t, int q) {
    t = dpp_add<0xB1>(t);                         // quad_perm [1,0,3,2]
    if constexpr (W >= 4) t = dpp_add<0x4E>(t);   // quad_perm [2,3,0,1]
    if constexpr (W >= 8) t = dpp_add<0x141>(t);  // row_half_mirror
    return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(t), W * q));
}
// Sums over the workgroup through W (2 W) words of scratch each; every wavefront gets the same bits.
template <int W>
__device__ __forceinline__ float group_total(float v, float* red, int wave, int lane) {
    v = wave_sum(v);
    if (lane == 0) red[wave] = v;
    __syncthreads();
    return partial_sum<W>(red[lane & (W - 1)], 0);
}
template <int W>
__device__ __forceinline__ void group_total2(float& u, float& v, float* red, int wave, int lane) {
    const float t = wave_sum_pair(u, v);
    if ((lane & 31) == 31) red[(lane >> 5) * W + wave] = t;
    __syncthreads();
    const float s = red[lane & (2 * W - 1)];
    u = partial_sum<W>(s, 0);
    v = partial_sum<W>(s, 1);
}

constexpr int STEP = 2;   // outer nonzeros per step of a product

// Gathered reads of p for outer nonzeros K0 .. K0+STEP-1 (lanes past the wave's run hold
// offset 0, so the reads stay inside p).
template <int K0, int C, int SMAX>
__device__ __forceinline__ void gather_step(float (&pv)[STEP][C], const InnerLanes<C>& in,
                                        const uint32_t (&s_poff)[SMAX / 2]) {
#pragma unroll
    for (int u = 0; u < STEP; ++u) {
        const uint32_t two = s_poff[(K0 + u) / 2], po = u & 1 ? two >> 16 : two & 0xffffu;
#pragma unroll
        for (int c = 0; c < C; ++c)
            pv[u][c] = *(const __attribute__((address_space(3))) float*)(uintptr_t)(po + in.jp[c]);   // p is at address 0 of LDS
    }
}

// Multiply-add of outer nonzeros K0 .. K0+STEP-1 (p values already read into pv); at the
// end of an outer row (wave-uniform test) each inner row is summed over its lanes
// (rows of at most 4 nonzeros: two shift-and-add steps) and the sum stored from the
// last lane of the row.  row_at: byte address the row's sums go to; the rows of a wavefront follow each other.
template <int K0, int KBEG, int SMAX, int C>
__device__ __forceinline__ void use_step(const float (&kap)[C][SMAX], const InnerLanes<C>& in,
                                     float (&acc)[C], const float (&pv)[STEP][C], uint32_t rowmask,
                                     uint32_t& row_at, uint32_t row_bytes) {
#pragma unroll
    for (int u = 0; u < STEP; ++u) {
#pragma unroll
        for (int c = 0; c < C; ++c) acc[c] = __builtin_fmaf(kap[c][K0 + u], pv[u][c], acc[c]);
        if ((rowmask >> (K0 - KBEG + u)) & 1u) {
            row_sums<C>(acc, in.m1, in.m2);
#pragma unroll
            for (int c = 0; c < C; ++c) {
                // every lane stores: those without a sum to the dump area (no divergent region)
                uint32_t at;
                asm("v_mad_u32_u24 %0, %1, %2, %3" : "=v"(at) : "s"(row_at), "v"(in.holds[c]), "v"(in.ip[c]));
                *(__attribute__((address_space(3))) float*)(uintptr_t)at = acc[c];
                acc[c] = 0.f;
            }
            row_at += row_bytes;
        }
    }
}

// Steps of a product from outer nonzero K0 (K0 < stop on entry): the reads of p for the next STEP
// outer nonzeros are issued before those already read are used, so that the LDS
// latency overlaps the arithmetic.  They are issued in the last step too (where there are registers for them): with a
// condition around them the compiler made two copies of every step and did the first multiply-adds of both.
template <int K0, int KBEG, int KEND, int SMAX, int C>
__device__ __forceinline__ void xmv_steps(const float (&kap)[C][SMAX], const InnerLanes<C>& in,
                                          float (&acc)[C], const float (&pv)[STEP][C], int stop,
                                          uint32_t rowmask, const uint32_t (&s_poff)[SMAX / 2],
                                          uint32_t row_at, uint32_t row_bytes) {
    float nx[STEP][C];
    if constexpr (K0 + STEP < KEND) gather_step<K0 + STEP, C, SMAX>(nx, in, s_poff);
    use_step<K0, KBEG, SMAX, C>(kap, in, acc, pv, rowmask, row_at, row_bytes);
    if constexpr (K0 + STEP < KEND)
        if (K0 + STEP < stop)   // wave-uniform
            xmv_steps<K0 + STEP, KBEG, KEND, SMAX, C>(kap, in, acc, nx, stop, rowmask, s_poff, row_at, row_bytes);
}

// The rows of one colour: outer nonzeros KBEG .. stop-1; bit k of rowmask: nonzero KBEG + k is the last of its row.
template <int KBEG, int KEND, int SMAX, int C>
__device__ __forceinline__ void xmv_rows(const float (&kap)[C][SMAX], const InnerLanes<C>& in, int stop, uint32_t rowmask,
                                         const uint32_t (&s_poff)[SMAX / 2], uint32_t row_at, uint32_t row_bytes) {
    if (KBEG >= stop) return;   // wave-uniform
    float acc[C], pv[STEP][C];
#pragma unroll
    for (int c = 0; c < C; ++c) acc[c] = 0.f;
    gather_step<KBEG, C, SMAX>(pv, in, s_poff);
    xmv_steps<KBEG, KBEG, KEND, SMAX, C>(kap, in, acc, pv, stop, rowmask, s_poff, row_at, row_bytes);
}

template <int W, int EPT, int C>
__global__ __launch_bounds__(W * 64, C == 1 ? (EPT <= 5 ? 5 : 3) : W * EPT <= 20 || W == 8 ? 4 : 3) void mgk_pcg_reduced(MgkBatchDev first, MgkBatchDev second,
                                                   const MgkJob* __restrict__ jobs, MgkParams prm,
                                                   MgkOutputs out, int weighted) {
    extern __shared__ __align__(16) uint32_t lds[];
    constexpr int NT = W * 64;
    constexpr int NP = NT * EPT;   // the red parts of p and y are padded to the register blocks
    constexpr int WL = MGK_RED_LIST(W), SB = MGK_RED_BLACK(W), SMAX = SB + MGK_RED_RED(W);   // kap[c][0 .. SB-1]: black rows
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);

    const MgkJob job = jobs[blockIdx.x];
    // jobs of both orientations are in one launch: of a swapped one the outer graph is of the second batch
    const bool from_second = job.out1 == MGK_OUT1_SWAPPED;
    const MgkBatchDev& X = from_second ? second : first;
    const MgkBatchDev& Y = from_second ? first : second;
    const MgkGraphDesc g1 = X.graphs[job.g1];
    const MgkGraphDesc g2 = Y.graphs[job.g2];
    const int n1 = g1.n, n2 = g2.n, nr = g1.n_red, len2 = g2.lane_len;
    const int NR = nr * n2, NB = (n1 - nr) * n2;   // elements of the reduced system, and the others
    const MgkReducedPlan L = mgk_reduced_plan(n1, nr, n2, W, EPT);

    float* p = reinterpret_cast<float*>(lds);          // L.p == 0: red part, NP words
    float* pb = reinterpret_cast<float*>(lds) + NP;    // L.black == NP
    float* y = reinterpret_cast<float*>(lds + L.y);
    // per-vertex data of the outer graph in the order of red_order
    float* dq1 = reinterpret_cast<float*>(lds + L.vtx1);   // d_i = rowsum + q
    float* st1 = dq1 + n1;                                 // start probability
    int* lb1 = reinterpret_cast<int*>(st1 + n1);           // vertex label
    float* dq2 = reinterpret_cast<float*>(lds + L.vtx2);
    float* st2 = dq2 + n2;
    int* lb2 = reinterpret_cast<int*>(st2 + n2);
    float* red = reinterpret_cast<float*>(lds + L.red);

    const uint16_t* order1 = X.red_order + 3 * (int64_t)g1.voff + WL * n1;
    // ---- stage per-vertex data; clear y (entries no row pair reaches stay 0) ----
    for (int v = tid; v < n1; v += NT) {
        const int at = g1.voff + order1[v];
        dq1[v] = X.rowsum[at] + prm.q;
        st1[v] = X.start[at];
        lb1[v] = X.vlabel[at];
    }
    for (int v = tid; v < n2; v += NT) {
        dq2[v] = Y.rowsum[g2.voff + v] + prm.q;
        st2[v] = Y.start[g2.voff + v];
        lb2[v] = Y.vlabel[g2.voff + v];
    }
#pragma unroll
    for (int m = 0; m < EPT; ++m) {
        p[tid + m * NT] = 0.f;
        y[tid + m * NT] = 0.f;
    }
    if (tid == 0) red[63] = 0.f;

    // ---- this wave's outer rows: whole rows of both colours, divided at load so that the most loaded
    //      wavefront is as light as possible
    const uint16_t* split = X.red_split + (int64_t)job.g1 * MGK_RED_SPLIT_STRIDE + MGK_RED_SPLIT(W);
    const int kbeg = __builtin_amdgcn_readfirstlane(split[wave]);
    const int kend = __builtin_amdgcn_readfirstlane(split[wave + 1]);
    const int blacks = __builtin_amdgcn_readfirstlane(split[W + 1 + wave]);
    const int brow = __builtin_amdgcn_readfirstlane(split[2 * W + 1 + wave]);
    const int rrow = __builtin_amdgcn_readfirstlane(split[3 * W + 1 + wave]);
    // byte addresses the sums of the first black and the first red row go to: the black part of p, and y
    const uint32_t row_bytes = 4u * (uint32_t)n2;
    const uint32_t brow_at = 4u * (uint32_t)(NP + (brow - nr) * n2), rrow_at = 4u * (uint32_t)(L.y + rrow * n2);
    // The host only sends pairs whose runs fit the unrolled loops.  Should one not fit, the
    // solve goes on with the part that does (so that every loop stays in bounds) and the
    // pair's outputs are replaced at the end: value NaN, flag 2, never a value computed
    // with part of the matrix.  red[63] is cleared before the staging barrier below.
    const bool misfit = blacks > SB || kend - kbeg - blacks > SMAX - SB || NR > NP || NP + NB > MGK_RED_MAX_P;
    const int bstop = min(blacks, SB), rstop = SB + min(kend - kbeg - blacks, SMAX - SB);

    // lane l < bstop holds the wave's l-th nonzero of black rows, lane SB + l its l-th one of red rows
    const bool live1 = lane < SB ? lane < bstop : lane < rstop;
    const uint32_t at1 = live1 ? X.list_sched[g1.soff + WL * g1.nnz + kbeg + (lane < SB ? lane : blacks + lane - SB)] : 0u;
    const MgkEntry o = live1 ? X.list_outer[g1.zoff + (at1 & 0xffffu)] : MgkEntry{0u, 0u, 0u, 0u};
    const int col1 = (int)(at1 >> 16);   // position in red_order
    const uint32_t v_poff = 4u * (uint32_t)(col1 < nr ? col1 * n2 : NP + (col1 - nr) * n2);   // byte offset of row j of p
    const uint64_t rowmask = __ballot(live1 && (o.w >> 31) != 0u);
    const float w1 = live1 ? __uint_as_float(o.w & 0x7fffffffu) : 0.f;
    // lanes past the run: a label so far away that kappa_e underflows to exactly 0
    const float e1s = live1 ? (__uint_as_float(o.z) - prm.e_shift) * prm.e_scale : 1e18f;
    const float l1 = weighted ? __log2f(live1 ? w1 : 1.f) : 0.f;

    // ---- inner nonzeros of this lane, one per chunk; matrix entries into registers --
    InnerLanes<C> in;
    int row2[C];
    float kap[C][SMAX];
    {
        float e2s[C], l2[C], w2c[C], w2r[C];
#pragma unroll
        for (int c = 0; c < C; ++c) {
            const int slot = c * 64 + lane;
            const MgkEntry e = slot < len2 ? Y.list_inner[g2.loff + slot] : MgkEntry{0u, 0u, 0u, 0u};
            row2[c] = (int)(e.x & 0xfffffu);
            in.holds[c] = e.x >> 31;
            in.ip[c] = in.holds[c] != 0u ? (uint32_t)row2[c] * 4u : (uint32_t)(L.dump + lane) * 4u;
            in.jp[c] = e.y * 4u;
            const uint32_t rank = (e.x >> 20) & 0xffu;
            in.m1[c] = rank >= 1 ? 1.f : 0.f;
            in.m2[c] = rank >= 2 ? 1.f : 0.f;
            const float w2 = __uint_as_float(e.w);   // 0 on idle slots
            e2s[c] = (__uint_as_float(e.z) - prm.e_shift) * prm.e_scale;
            l2[c] = w2 > 0.f ? (weighted ? __log2f(w2) : 0.f) : -__builtin_inff();
            w2c[c] = w2 * prm.ke_const;
            w2r[c] = w2;
        }
        if (prm.edge_kernel == MGK_EK_SE) {
            if (weighted) {
                fill_se<0, SB, SMAX, C, true>(kap, bstop, e2s, l2, e1s, l1);
                fill_se<SB, SMAX, SMAX, C, true>(kap, rstop, e2s, l2, e1s, l1);
            } else {
                fill_se<0, SB, SMAX, C, false>(kap, bstop, e2s, l2, e1s, l1);
                fill_se<SB, SMAX, SMAX, C, false>(kap, rstop, e2s, l2, e1s, l1);
            }
        } else if (prm.edge_kernel == MGK_EK_CONST) {
            fill_const<0, SB, SMAX, C>(kap, bstop, w2c, w1);
            fill_const<SB, SMAX, SMAX, C>(kap, rstop, w2c, w1);
        } else if (prm.edge_kernel == MGK_EK_POLY) {
            fill_poly<0, SB, SMAX, C>(kap, bstop, e2s, w2r, e1s, w1, prm.poly_c);
            fill_poly<SB, SMAX, SMAX, C>(kap, rstop, e2s, w2r, e1s, w1, prm.poly_c);
        } else {
            // labels with D attributes, from the attribute planes of the two lists
            const int D = prm.label_dim;
            const bool rconv = prm.edge_kernel == MGK_EK_RCONV_SE;
            auto outer = [&](int a) {
                // past the run: kappa_e underflows to exactly 0 (the R-convolution's weight is 0 there)
                return live1 ? X.attr_outer[(int64_t)a * X.nnz_total + g1.zoff + (at1 & 0xffffu)] * prm.attr_scale[a] : a == 0 && !rconv ? 1e18f : 0.f;
            };
            auto inner = [&](int a, int c) {
                const int slot = c * 64 + lane;
                return slot < len2 ? Y.attr_inner[(int64_t)a * Y.lanes_total + g2.loff + slot] * prm.attr_scale[a] : 0.f;
            };
            if (rconv) {
                const float inv = 1.0f / (float)(D * D);
                float f2[C];
#pragma unroll
                for (int c = 0; c < C; ++c) f2[c] = w2r[c] * inv;   // 0 on idle slots
                fill_attr<SB, SMAX, C, true>(kap, bstop, rstop, D, f2, w1, outer, inner);   // w1 is 0 past the run
            } else {
                const float la = weighted ? __log2f(live1 ? w1 : 1.f) : 0.f;
                fill_attr<SB, SMAX, C, false>(kap, bstop, rstop, D, l2, la, outer, inner);
            }
        }
    }
    __syncthreads();   // per-vertex data staged
    if (misfit && lane == 0) red[63] = 1.f;   // wave-uniform, after the barrier that follows the clearing
    {
        // position of the row of this lane's nonzero: the row ends below the lane tell
        const int row1 = live1 && lane < SB ? brow + __popcll(rowmask & ((1ull << lane) - 1ull)) : 0;
        float d2[C], d2h[C];
        int lab2[C];
#pragma unroll
        for (int c = 0; c < C; ++c) {
            d2[c] = __builtin_amdgcn_rcpf(dq2[row2[c]]);
            d2h[c] = prm.h * d2[c];
            lab2[c] = lb2[row2[c]];
        }
        scale_black<0, SB, SMAX, C>(kap, bstop, d2, d2h, lab2, __builtin_amdgcn_rcpf(dq1[row1]), lb1[row1]);
    }

    // ---- Alg. 1 set-up: M = D_x V_x^{-1}, x = 0, b = D_x q_x; the right side of the reduced system is
    //      b_r + W_rb z0_b with z0 = M^{-1} b = kappa_v q q'
    float rr_[EPT], Mr[EPT], pr[EPT], zr[EPT], xr[EPT];
    const float qq = prm.q * prm.q;
    const float inv_n2 = 1.0f / (float)n2;
    const float inv_h = 1.0f / prm.h;
    float s_bb = 0.f;
#pragma unroll
    for (int m = 0; m < EPT; ++m) {
        const int idx = tid + m * NT;
        const bool ok = idx < NR;
        const int ic = ok ? idx : 0;
        const int i = (int)(((float)ic + 0.5f) * inv_n2);
        const int i2 = ic - i * n2;
        const bool same = lb1[i] == lb2[i2];
        const float dd = dq1[i] * dq2[i2];
        const float b = ok ? dd * qq : 0.f;
        Mr[m] = ok ? (same ? dd : dd * inv_h) : 1.f;           // d d' / kappa_v
        rr_[m] = b;
        pr[m] = 0.f;
        xr[m] = 0.f;
        s_bb = __builtin_fmaf(b, b, s_bb);
    }
    for (int idx = tid; idx < NB; idx += NT) {
        const int i = nr + (int)(((float)idx + 0.5f) * inv_n2);
        const int i2 = idx - (i - nr) * n2;
        const float b = dq1[i] * dq2[i2] * qq;
        pb[idx] = lb1[i] == lb2[i2] ? qq : prm.h * qq;
        s_bb = __builtin_fmaf(b, b, s_bb);
    }
    int max_iter = prm.max_iter;
    if (max_iter <= 0) max_iter = min(2 * n1 * n2, 1000);

    uint32_t black_ends = (uint32_t)rowmask, red_ends = (uint32_t)(rowmask >> SB);   // ends of rows of either colour
    static_assert(SB <= 32 && SMAX - SB <= 32, "a word each");
    // byte offset of row j of p for each of the wave's outer nonzeros (entries past the run read row 0), in
    // scalar registers for the whole solve, two to a register
    uint32_t s_poff[SMAX / 2];
#pragma unroll
    for (int k = 0; k < SMAX; k += 2) s_poff[k / 2] = lane_value(v_poff, k) | lane_value(v_poff, k + 1) << 16;

    float rho = 0.f, thresh = 0.f;
    int it = -1;         // -1: the product that forms the right side
    bool over = false;   // the last pass forms x_b
    int flag = 1;
    while (true) {
        // what is derived from these (lane addresses of the first reads, one condition per nonzero) stays out of
        // registers between the iterations
        asm volatile("" : "+s"(black_ends), "+s"(red_ends));
#pragma unroll
        for (int k = 0; k < SMAX / 2; ++k) asm volatile("" : "+s"(s_poff[k]));
        __syncthreads();   // the red part of p is complete (at first: all of it, and the cleared y)
        // ---- p_b = M_b^{-1} W_br p_r, entries from registers
        if (it >= 0) xmv_rows<0, SB, SMAX, C>(kap, in, bstop, black_ends, s_poff, brow_at, row_bytes);
        __syncthreads();
        if (over) break;
        // ---- y = W_rr p_r + W_rb p_b
        xmv_rows<SB, SMAX, SMAX, C>(kap, in, rstop, red_ends, s_poff, rrow_at, row_bytes);
        __syncthreads();
        float alpha = 0.f;
        if (it < 0) {
#pragma unroll
            for (int m = 0; m < EPT; ++m) {
                rr_[m] += y[tid + m * NT];
                zr[m] = 0.f;
            }
            for (int idx = tid; idx < NB; idx += NT) pb[idx] = 0.f;   // elements no row pair reaches stay 0
        } else {
            // ---- a = M p - y ; alpha = rho / p^T a
            float s_pa = 0.f;
#pragma unroll
            for (int m = 0; m < EPT; ++m) {
                zr[m] = __builtin_fmaf(Mr[m], pr[m], -y[tid + m * NT]);
                s_pa = __builtin_fmaf(pr[m], zr[m], s_pa);
            }
            const float pa = group_total<W>(s_pa, red + 32, wave, lane);
            alpha = rho * __builtin_amdgcn_rcpf(pa);
        }

        // ---- x += alpha p; r -= alpha a; z = M^{-1} r; rho' = r^T z
        float s_rz2 = 0.f, s_rr = 0.f;
#pragma unroll
        for (int m = 0; m < EPT; ++m) {
            // written as instructions with the register of x (r, p) as destination: the compiler's own choice
            // puts the new vectors into other registers and copies them back
            asm("v_fmac_f32 %0, %1, %2" : "+v"(xr[m]) : "v"(alpha), "v"(pr[m]));
            asm("v_fma_f32 %0, -%1, %2, %0" : "+v"(rr_[m]) : "v"(alpha), "v"(zr[m]));
            const float rv = rr_[m];
            const float zv = rv * __builtin_amdgcn_rcpf(Mr[m]);   // 1/M is hoisted by the compiler
            zr[m] = zv;
            s_rz2 = __builtin_fmaf(rv, zv, s_rz2);
            s_rr = __builtin_fmaf(rv, rv, s_rr);
        }
        if (it < 0) {
            s_rr = s_bb;   // the stop test is relative to b of the full system
            group_total2<W>(s_rz2, s_rr, red, wave, lane);
            thresh = prm.rtol2 * s_rr;
            rho = 1.f;
        } else {
            group_total2<W>(s_rz2, s_rr, red, wave, lane);
            over = s_rr <= thresh;
            if (over) flag = 0;
        }
        ++it;
        over = over || it >= max_iter;

        // ---- p = z + beta p (also after the last iteration, where it is not used: the
        //      loop then has a single exit and the register blocks stay in place)
        const float beta = s_rz2 * __builtin_amdgcn_rcpf(rho);
        rho = s_rz2;
        float beta_v = beta;
#pragma unroll
        for (int m = 0; m < EPT; ++m) {
            asm("v_fma_f32 %0, %1, %0, %2" : "+v"(pr[m]) : "v"(beta_v), "v"(zr[m]));
            p[tid + m * NT] = over ? xr[m] : pr[m];
        }
    }

    // ---- K = p_x^T x (Eq. 1), x_b = z0_b + M_b^{-1} W_br x_r
    // rows and columns of the elements are found anew: kept from the set-up they would hold two registers an element
    // through the iterations
    int m2 = n2;
    asm volatile("" : "+s"(m2));
    const float inv_m2 = 1.0f / (float)m2;
    float s_k = 0.f;
    if (X.uniform_start && Y.uniform_start) {   // p_x = 1 / (n n') everywhere
#pragma unroll
        for (int m = 0; m < EPT; ++m) s_k += xr[m];   // x is 0 beyond NR
    } else {
#pragma unroll
        for (int m = 0; m < EPT; ++m) {
            const int idx = tid + m * NT;
            const int ic = idx < NR ? idx : 0;
            const int i = (int)(((float)ic + 0.5f) * inv_m2);
            const int i2 = ic - i * m2;
            s_k = __builtin_fmaf(st1[i] * st2[i2], xr[m], s_k);  // x is 0 beyond NR
        }
    }
    const bool uniform = X.uniform_start && Y.uniform_start;
    for (int idx = tid; idx < NB; idx += NT) {
        const int i = nr + (int)(((float)idx + 0.5f) * inv_m2);
        const int i2 = idx - (i - nr) * m2;
        const float xb = pb[idx] + (lb1[i] == lb2[i2] ? qq : prm.h * qq);
        if (out.nodal) pb[idx] = xb;
        s_k = __builtin_fmaf(uniform ? 1.f : st1[i] * st2[i2], xb, s_k);
    }
    if (uniform) s_k *= inv_m2 * (1.0f / (float)n1);
    float Kval = group_total<W>(s_k, red + 48, wave, lane);
    if (tid == 0) {
        if (red[63] != 0.f) {   // some wavefront's run did not fit
            Kval = __builtin_nanf("");
            flag = 2;
        }
        out.K[job.out0] = Kval;
        if (job.out1 >= 0) out.K[job.out1] = Kval;
        if (out.iters) {
            out.iters[job.out0] = it;
            if (job.out1 >= 0) out.iters[job.out1] = it;
        }
        if (out.flags) {
            out.flags[job.out0] = flag;
            if (job.out1 >= 0) out.flags[job.out1] = flag;
        }
    }
    // ---- nodal similarity: x itself, in the original numbering of the requested pair
    if (out.nodal) {
        float* dst = out.nodal + out.nodal_off[job.out0];
        const bool swapped = job.out1 == MGK_OUT1_SWAPPED;
        auto put = [&](int i, int i2, float v) {
            const int oi = X.iperm[g1.voff + order1[i]], oi2 = Y.iperm[g2.voff + i2];
            dst[swapped ? oi2 * n1 + oi : oi * n2 + oi2] = v;
        };
#pragma unroll
        for (int m = 0; m < EPT; ++m) {
            const int idx = tid + m * NT;
            const int i = (int)(((float)idx + 0.5f) * inv_m2);
            if (idx < NR) put(i, idx - i * m2, xr[m]);
        }
        for (int idx = tid; idx < NB; idx += NT) {   // every thread reads back what it wrote
            const int i = (int)(((float)idx + 0.5f) * inv_m2);
            put(nr + i, idx - i * m2, pb[idx]);
        }
    }
}

template <int W, int EPT, int C>
hipError_t launch_one(const MgkBatchDev& X, const MgkBatchDev& Y, const MgkJob* jobs, int n_jobs,
                      const MgkParams& prm, bool weighted, size_t lds_bytes, const MgkOutputs& out,
                      hipStream_t stream) {
    auto kern = mgk_pcg_reduced<W, EPT, C>;
    static bool configured = false;  // per instantiation
    if (!configured) {
        hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(kern),
                                           hipFuncAttributeMaxDynamicSharedMemorySize,
                                           MGK_LDS_LIMIT_BYTES);
        if (e != hipSuccess) return e;
        configured = true;
    }
    hipLaunchKernelGGL(kern, dim3(n_jobs), dim3(W * 64), lds_bytes, stream, X, Y, jobs, prm, out,
                       weighted ? 1 : 0);
    return hipGetLastError();
}

}  // namespace

#if !defined(MGK_REDUCED_CHUNKS) || !defined(MGK_REDUCED_WAVES)
#error "compile with -DMGK_REDUCED_WAVES=<2|4|8> -DMGK_REDUCED_CHUNKS=<1|2>"
#endif

#define MGK_CAT2(a, b, c, d) a##b##c##d
#define MGK_CAT(a, b, c, d) MGK_CAT2(a, b, c, d)

// One translation unit per (wavefronts, chunk count) keeps the build parallel.
hipError_t MGK_CAT(mgk_launch_reduced_w, MGK_REDUCED_WAVES, _c, MGK_REDUCED_CHUNKS)(
    int ept, bool weighted, const MgkBatchDev& X, const MgkBatchDev& Y, const MgkJob* jobs_dev,
    int n_jobs, const MgkParams& prm, size_t lds_bytes, const MgkOutputs& out, hipStream_t stream) {
    if (n_jobs <= 0) return hipSuccess;
    constexpr int C = MGK_REDUCED_CHUNKS;
    constexpr int W = MGK_REDUCED_WAVES;
    switch (ept) {
#define MGK_CASE(E) \
    case E: return launch_one<W, E, C>(X, Y, jobs_dev, n_jobs, prm, weighted, lds_bytes, out, stream);
        MGK_CASE(1) MGK_CASE(2) MGK_CASE(3) MGK_CASE(4) MGK_CASE(5) MGK_CASE(6) MGK_CASE(7) MGK_CASE(8)
#undef MGK_CASE
        default: return hipErrorInvalidValue;
    }
}

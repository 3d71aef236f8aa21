// Whole PCG on chip (Alg. 1) for pairs whose entries do not fit in registers, with the
// off-diagonal product through a separable edge kernel (mgk_sep_dev.h): y = sum_k F_k P F'_k^T.
//
// One workgroup per pair; p and y in LDS, x, r and M in registers.  The graph with fewer vertices gives the columns.
// For `rb` blocks of 16 rows at a time: stage 1 forms T_k[i, j'] = sum_j F_k[i, j] P[j, j'] (16 columns of 4 rows per
// wavefront step), stage 2 y[i, i'] = sum_j' sum_k F'_k[i', j'] T_k[i, j'] (16 rows of 4 columns).  Rows and columns are
// taken by descending degree, so that the four of a step have packets of similar length; the packets are read
// from L2 one task ahead.
//
// Per nonzero and 64 results a stage does RK multiply-adds and 2 address additions, stage 2 also reads 4 RK bytes x 64 of
// T.  Gram matrix of 160 scale-free graphs of 96 vertices (12 880 pairs, rank 5): 28.4 ms with the streaming solver (one
// exponential per pair of nonzeros), 9.9 ms with this.  Bound by the vector ALUs (67 % of their slots, 47 % of the
// instructions are multiply-adds, the others addresses, the vector part and the ends of tasks) and LDS (52 %, 38 % of it
// bank conflicts) in turn: stage 1 by the first, stage 2 by both.  Tried without gain: long tasks divided among wavefronts
// (11.0 ms; the wavefronts of a SIMD even out by themselves), T with 64 words to a column so that 16-byte reads never
// conflict (10.1 ms; the writes then do).
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "mgk_internal.h"
#include "mgk_launch.h"
#include "mgk_sep_dev.h"
#include "mgk_wave.h"

namespace {

// Packets of 4, 5 or 6 features have room for a nonzero's column in both forms, as the offset of its column of T and as
// the number; the others hold the number.
template <int RK>
constexpr bool kOffsets = RK >= 4 && RK <= 6;

// One column of T for a block of 16 rows: features 0..3 of each row side by side, then the others.  quad: where the
// first four of the row are, rest: the others (16 and 4 or 8 bytes a row).
template <int RK>
__device__ __forceinline__ void tcol_read(float (&t)[RK], const char* quad, const char* rest) {
    if constexpr (RK == 1) {
        t[0] = *reinterpret_cast<const float*>(quad);
    } else {
        const float4 a = *reinterpret_cast<const float4*>(quad);
        t[0] = a.x; t[1] = a.y; t[2] = a.z; t[3] = a.w;
        if constexpr (RK == 5) t[4] = *reinterpret_cast<const float*>(rest + 256);
        if constexpr (RK == 6) {
            const float2 b = *reinterpret_cast<const float2*>(rest + 256);
            t[4] = b.x; t[5] = b.y;
        }
        if constexpr (RK == 7) {   // 12 bytes a row
            const float* b = reinterpret_cast<const float*>(rest + 256);
            t[4] = b[0]; t[5] = b[1]; t[6] = b[2];
        }
    }
}
template <int RK>
__device__ __forceinline__ void tcol_write(char* col, uint32_t row, const float (&t)[RK]) {
    if constexpr (RK == 1) {
        *reinterpret_cast<float*>(col + 4u * row) = t[0];
    } else {
        *reinterpret_cast<float4*>(col + 16u * row) = make_float4(t[0], t[1], t[2], t[3]);
        if constexpr (RK == 5) *reinterpret_cast<float*>(col + 256 + 4u * row) = t[4];
        if constexpr (RK == 6) *reinterpret_cast<float2*>(col + 256 + 8u * row) = make_float2(t[4], t[5]);
        if constexpr (RK == 7) {
            float* b = reinterpret_cast<float*>(col + 256 + 12u * row);
            b[0] = t[4]; b[1] = t[5]; b[2] = t[6];
        }
    }
}

// Where a stage reads: p (T false), from + j stride; T, the two parts of column j of it.
struct Source {
    const char *from, *rest;
    uint32_t stride;
};

// acc += the products of D packets of a lane.
template <bool T, int RK, int G, int D>
__device__ __forceinline__ void packets_once(float (&acc)[RK], const float* c, const Source& src) {
    float tv[T ? D * G : 1][RK], pv[D * G];
#pragma unroll
    for (int d = 0; d < D; ++d) {
        uint32_t j[G];
        if constexpr (T || !kOffsets<RK>) {
            packet_slabs<RK, G>(j, c[d]);
        } else {
            j[0] = bcast16<MGK_SEP_NUMBER_SLOT>(c[d]);
            j[1] = bcast16<MGK_SEP_NUMBER_SLOT + 1>(c[d]);
        }
#pragma unroll
        for (int u = 0; u < G; ++u) {
            if constexpr (T) {
                const uint32_t off = kOffsets<RK> ? j[u] : __umul24(j[u], src.stride);
                tcol_read<RK>(tv[d * G + u], src.from + off, src.rest + off);
            } else {
                pv[d * G + u] = *reinterpret_cast<const float*>(src.from + __umul24(j[u], src.stride));
            }
        }
    }
#pragma unroll
    for (int d = 0; d < D; ++d) {
        if constexpr (T) packet_each<RK, G>(acc, c[d], reinterpret_cast<const float(&)[G][RK]>(tv[d * G]));
        else packet_same<RK, G>(acc, c[d], pv + d * G);
    }
}

// A lane's word of eight packets; those past the last one of a row are of other rows, or the space behind the list.
__device__ __forceinline__ void packets_load(float (&c)[8], const float* list, int first, uint32_t lane4) {
    uint64_t at = (uint64_t)list + (int64_t)first * 256;
    asm("" : "+s"(at));   // a scalar base, so that the loads differ in their immediate offsets only
    // global, not flat: flat loads count as LDS reads too, which would then wait for them
    const auto* base = (const __attribute__((address_space(1))) char*)at;
#pragma unroll
    for (int a = 0; a < 8; ++a) c[a] = *(const __attribute__((address_space(1))) float*)(base + 256 * a + lane4);
}

// acc = the products of a lane's packets: `steps` of them from `first`, eight of which are in c.
template <bool T, int RK, int G>
__device__ __forceinline__ void packets_times(float (&acc)[RK], float (&c)[8], const float* list, int first, int steps, uint32_t lane4,
                                              const Source& src) {
    constexpr int D = G >= 8 ? 1 : 2;   // packets per step
#pragma unroll
    for (int k = 0; k < RK; ++k) acc[k] = 0.f;
    for (int b = 0; b < steps; b += 8) {
        if (b > 0) packets_load(c, list, first + b, lane4);
#pragma unroll
        for (int a = 0; a < 8; a += D) {
            if (b + a < steps) {   // wave-uniform
                if (D > 1 && b + a + 1 >= steps) c[a + D - 1] = 0.f;   // a path of its own would copy the sums
                packets_once<T, RK, G, D>(acc, c + a, src);
            }
        }
    }
}

// Barrier for data in LDS: loads from global memory stay in flight, which __syncthreads() would wait for.
__device__ __forceinline__ void lds_barrier() { asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory"); }

template <int RK, int G, int EPT, int W>
__global__ __launch_bounds__(W * 64) void mgk_pcg_sep(MgkBatchDev X, MgkBatchDev Y, MgkSepList SX, MgkSepList SY, int passes,
                                                      const MgkJob* __restrict__ jobs, MgkParams prm, MgkOutputs out, int rb,
                                                      int lds_words) {
    extern __shared__ __align__(16) float lds[];
    constexpr int NT = W * 64, NP = NT * EPT, SLAB = MGK_PCG_SEP_SLAB(RK) * 4;   // bytes of a column of T
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const MgkJob job = jobs[blockIdx.x];
    const bool turned = X.graphs[job.g1].n < Y.graphs[job.g2].n;   // fewer columns than rows
    const MgkBatchDev &A = turned ? Y : X, &B = turned ? X : Y;
    const MgkSepList &SA = turned ? SY : SX, &SB = turned ? SX : SY;
    const int ga = turned ? job.g2 : job.g1, gb = turned ? job.g1 : job.g2;
    const MgkGraphDesc g1 = A.graphs[ga], g2 = B.graphs[gb];
    const int n1 = g1.n, n2 = g2.n, N = n1 * n2;
    const MgkPcgSepPlan L = mgk_pcg_sep_plan(n1, n2, RK, rb);
    if (N > NP || L.total > lds_words) {   // the host sends none; never a value of part of the pair
        if (tid == 0) {
            out.K[job.out0] = __builtin_nanf("");
            if (job.out1 >= 0) out.K[job.out1] = __builtin_nanf("");
            if (out.flags) out.flags[job.out0] = 2;
            if (out.flags && job.out1 >= 0) out.flags[job.out1] = 2;
        }
        return;
    }
    float* p = lds;
    float* y = lds + L.y;   // as p: rows of n2 | 1 words
    char* tcols = reinterpret_cast<char*>(lds + L.t);
    float* dq1 = lds + L.vtx1;                         // d_i = rowsum + q
    int* lb1 = reinterpret_cast<int*>(dq1 + n1);       // vertex label
    int* order1 = lb1 + n1;                            // vertices by descending degree
    float* dq2 = lds + L.vtx2;
    int* lb2 = reinterpret_cast<int*>(dq2 + n2);
    int* order2 = lb2 + n2;
    int* gp1 = reinterpret_cast<int*>(lds + L.gptr);   // first packet step of each four rows
    const int ng1 = (n1 + 3) >> 2, ng2 = (n2 + 3) >> 2;
    int* gp2 = gp1 + ng1 + 1;
    float* red = lds + L.red;

    for (int v = tid; v < n1; v += NT) {
        dq1[v] = A.rowsum[g1.voff + v] + prm.q;
        lb1[v] = A.vlabel[g1.voff + v];
        order1[v] = SA.deg_order[g1.voff + v];
    }
    for (int v = tid; v < n2; v += NT) {
        dq2[v] = B.rowsum[g2.voff + v] + prm.q;
        lb2[v] = B.vlabel[g2.voff + v];
        order2[v] = SB.deg_order[g2.voff + v];
    }
    for (int v = tid; v <= ng1; v += NT) gp1[v] = SA.gptr[SA.qoff[ga] + v];
    for (int v = tid; v <= ng2; v += NT) gp2[v] = SB.gptr[SB.qoff[gb] + v];
    __syncthreads();

    // ---- set-up: M = D_x V_x^{-1}, x = 0, r = b = D_x q_x, z = M^{-1} r, p = z, rho = r^T z
    float xr[EPT], rr_[EPT], Mr[EPT], zr[EPT];
    const float qq = prm.q * prm.q;
    const float inv_n2 = 1.0f / (float)n2;
    const float inv_h = 1.0f / prm.h;
    float s_rz = 0.f, s_bb = 0.f;
#pragma unroll
    for (int m = 0; m < EPT; ++m) {
        const int idx = tid + m * NT;
        const bool ok = idx < N;
        const int ic = ok ? idx : 0;
        const int i = (int)(((float)ic + 0.5f) * inv_n2);
        const int i2 = ic - i * n2;
        const bool same = lb1[i] == lb2[i2];
        const float dd = dq1[i] * dq2[i2];
        const float b = ok ? dd * qq : 0.f;
        const float z0 = ok ? (same ? qq : prm.h * qq) : 0.f;
        Mr[m] = ok ? (same ? dd : dd * inv_h) : 1.f;
        xr[m] = 0.f;
        rr_[m] = b;
        if (ok) p[i * (n2 | 1) + i2] = z0;
        s_rz = __builtin_fmaf(b, z0, s_rz);
        s_bb = __builtin_fmaf(b, b, s_bb);
    }
    block_sum2<W>(s_rz, s_bb, red, wave, lane);
    float rho = s_rz;
    const float thresh = prm.rtol2 * s_bb;
    int max_iter = prm.max_iter;
    if (max_iter <= 0) max_iter = min(2 * N, 1000);
    __syncthreads();   // p is complete

    const int blocks = (n1 + 15) >> 4, strips = (n2 + 15) >> 4;   // of 16 rows, of 16 columns
    const int stride = n2 | 1;   // odd: rows at different banks
    const uint32_t lane4 = 4u * (uint32_t)lane, l16 = (uint32_t)lane & 15u;
    const uint32_t strips_magic = 65536u / (uint32_t)strips + 1u;   // exact for t strips < 65536
    const char* pbytes = reinterpret_cast<const char*>(p);
    // tasks of a round in alternating direction: tasks come by descending length
    auto task = [&](int m) { return m * W + (m & 1 ? W - 1 - wave : wave); };
    // the next task: its packets are on their way during the one before and the barrier between two stages
    float cn[8];
    int first = 0, steps = 0, grp = 0, sub = 0;
    // task t of stage 1: four rows (from group grp0 on) by 16 columns
    auto next1 = [&](int t, int q, int grp0, int ngrp) {
        if (t >= ngrp * strips) return;
        grp = (int)((uint32_t)t * strips_magic >> 16);
        sub = t - grp * strips;
        first = __builtin_amdgcn_readfirstlane(gp1[grp0 + grp]);
        steps = __builtin_amdgcn_readfirstlane(gp1[grp0 + grp + 1]) - first;
        packets_load(cn, SA.packets + (int64_t)q * SA.total * 64, first, lane4);
    };
    // task t of stage 2: 16 rows (of nb blocks of them) by four columns
    auto next2 = [&](int t, int q, int nb, uint32_t nb_magic) {
        if (t >= nb * ng2) return;
        grp = (int)((uint32_t)t * nb_magic >> 16);
        sub = t - grp * nb;
        first = __builtin_amdgcn_readfirstlane(gp2[grp]);
        steps = __builtin_amdgcn_readfirstlane(gp2[grp + 1]) - first;
        packets_load(cn, SB.packets + (int64_t)q * SB.total * 64, first, lane4);
    };
    auto groups = [&](int blk) { return min(min(rb, blocks - blk) * 4, ng1 - blk * 4); };

    int it = 0, flag = 1;
    next1(task(0), 0, 0, groups(0));
    while (it < max_iter) {
        for (int blk = 0; blk < blocks; blk += rb) {
            const int nb = min(rb, blocks - blk);
            const int grp0 = blk * 4, ngrp = groups(blk);
            const uint32_t nb_magic = 65536u / (uint32_t)nb + 1u;
            for (int q = 0; q < passes; ++q) {
                {
                    const float* list = SA.packets + (int64_t)q * SA.total * 64;
                    const int tasks = ngrp * strips;
                    int m = 0, t = task(0);
                    while (t < tasks) {
                        float c[8], acc[RK];
#pragma unroll
                        for (int a = 0; a < 8; ++a) c[a] = cn[a];
                        const int from = first, now = steps, row = grp * 4 + (lane >> 4), col = sub * 16 + (int)l16;
                        next1(t = task(++m), q, grp0, ngrp);
                        const Source src{pbytes + 4 * min(col, n2 - 1), nullptr, 4u * (uint32_t)stride};
                        packets_times<false, RK, G>(acc, c, list, from, now, lane4, src);
                        if (col < n2) tcol_write<RK>(tcols + __umul24(__umul24(row >> 4, n2) + col, SLAB), (uint32_t)row & 15u, acc);
                    }
                }
                next2(task(0), q, nb, nb_magic);
                lds_barrier();
                {
                    const float* list = SB.packets + (int64_t)q * SB.total * 64;
                    const int tasks = nb * ng2;
                    int m = 0, t = task(0);
                    while (t < tasks) {
                        float c[8], acc[RK];
#pragma unroll
                        for (int a = 0; a < 8; ++a) c[a] = cn[a];
                        const int from = first, now = steps, row = (blk + sub) * 16 + (int)l16, at = grp * 4 + (lane >> 4);
                        const char* cols = tcols + sub * n2 * SLAB;
                        const Source src{cols + (RK == 1 ? 4u : 16u) * l16, cols + (RK == 7 ? 12u : RK == 6 ? 8u : 4u) * l16, SLAB};
                        next2(t = task(++m), q, nb, nb_magic);
                        packets_times<true, RK, G>(acc, c, list, from, now, lane4, src);
                        float s = acc[0];
#pragma unroll
                        for (int k = 1; k < RK; ++k) s += acc[k];
                        if (row < n1 && at < n2) {
                            float* dst = y + order1[row] * stride + order2[at];
                            *dst = q == 0 ? s : *dst + s;   // the same lane in every pass
                        }
                    }
                }
                const bool more = q + 1 < passes;
                const int blk1 = more ? blk : blk + rb < blocks ? blk + rb : 0;
                next1(task(0), more ? q + 1 : 0, blk1 * 4, groups(blk1));
                lds_barrier();
            }
        }

        // ---- a = M p - y ; alpha = rho / p^T a
        // what is derived from these (1 / M, an address per element) stays out of registers between the iterations
        int m2 = n2, at0 = tid;
        asm volatile("" : "+s"(m2), "+v"(at0));
#pragma unroll
        for (int m = 0; m < EPT; ++m) asm volatile("" : "+v"(Mr[m]));
        const float inv_m2 = 1.0f / (float)m2;
        float s_pa = 0.f;
        int at[EPT];   // of the thread's elements in p and y
#pragma unroll
        for (int m = 0; m < EPT; ++m) {
            const int idx = at0 + m * NT;
            const int ic = min(idx, N - 1);   // those past the last one read it, times 0
            const int i = (int)(((float)ic + 0.5f) * inv_m2);
            at[m] = ic + i * (stride - m2);
            const float on = idx < N ? 1.f : 0.f, pv = p[at[m]];
            zr[m] = on * __builtin_fmaf(Mr[m], pv, -y[at[m]]);
            s_pa = __builtin_fmaf(pv, zr[m], s_pa);
        }
        const float pa = block_sum<W>(s_pa, red + 32, wave, lane);
        const float alpha = rho * __builtin_amdgcn_rcpf(pa);

        // ---- x += alpha p; r -= alpha a; z = M^{-1} r; rho' = r^T z
        float s_rz2 = 0.f, s_rr = 0.f;
#pragma unroll
        for (int m = 0; m < EPT; ++m) {
            xr[m] = __builtin_fmaf(alpha, p[at[m]], xr[m]);
            const float rv = __builtin_fmaf(-alpha, zr[m], rr_[m]);
            rr_[m] = rv;
            const float zv = rv * __builtin_amdgcn_rcpf(Mr[m]);
            zr[m] = zv;
            s_rz2 = __builtin_fmaf(rv, zv, s_rz2);
            s_rr = __builtin_fmaf(rv, rv, s_rr);
        }
        block_sum2<W>(s_rz2, s_rr, red, wave, lane);
        ++it;

        const float beta = s_rz2 * __builtin_amdgcn_rcpf(rho);
        rho = s_rz2;
#pragma unroll
        for (int m = 0; m < EPT; ++m)
            if (at0 + m * NT < N) p[at[m]] = __builtin_fmaf(beta, p[at[m]], zr[m]);
        __syncthreads();
        if (s_rr <= thresh) { flag = 0; break; }
    }

    // ---- K = p_x^T x (Eq. 1)
    float s_k = 0.f;
    int m2 = n2, at0 = tid;
    asm volatile("" : "+s"(m2), "+v"(at0));
    const float inv_m2 = 1.0f / (float)m2;
#pragma unroll
    for (int m = 0; m < EPT; ++m) {
        const int idx = at0 + m * NT;
        const int ic = idx < N ? idx : 0;
        const int i = (int)(((float)ic + 0.5f) * inv_m2);
        s_k = __builtin_fmaf(A.start[g1.voff + i] * B.start[g2.voff + ic - i * m2], idx < N ? xr[m] : 0.f, s_k);
    }
    const float Kval = block_sum<W>(s_k, red + 48, wave, lane);
    if (tid == 0) {
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
    if (out.nodal) {   // x itself, in the original numbering of the requested pair
        float* dst = out.nodal + out.nodal_off[job.out0];
        const bool swapped = (job.out1 == MGK_OUT1_SWAPPED) != turned;
#pragma unroll
        for (int m = 0; m < EPT; ++m) {
            const int idx = at0 + m * NT;
            if (idx < N) {
                const int i = (int)(((float)idx + 0.5f) * inv_m2);
                const int i2 = idx - i * m2;
                const int oi = A.iperm[g1.voff + i], oi2 = B.iperm[g2.voff + i2];
                dst[swapped ? oi2 * n1 + oi : oi * n2 + oi2] = xr[m];
            }
        }
    }
}

template <int RK, int G, int EPT, int W>
hipError_t launch_one(const MgkBatchDev& X, const MgkBatchDev& Y, const MgkSepList& SX, const MgkSepList& SY, int passes,
                      const MgkJob* jobs, int n_jobs, const MgkParams& prm, int rb, size_t lds_bytes, const MgkOutputs& out,
                      hipStream_t stream) {
    auto kern = mgk_pcg_sep<RK, G, EPT, W>;
    static bool configured = false;  // per instantiation
    if (!configured) {
        hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(kern), hipFuncAttributeMaxDynamicSharedMemorySize,
                                           MGK_LDS_LIMIT_BYTES);
        if (e != hipSuccess) return e;
        configured = true;
    }
    hipLaunchKernelGGL(kern, dim3(n_jobs), dim3(W * 64), lds_bytes, stream, X, Y, SX, SY, passes, jobs, prm, out, rb, (int)(lds_bytes / 4));
    return hipGetLastError();
}

}  // namespace

#ifndef MGK_PCG_SEP_RK
#error "compile with -DMGK_PCG_SEP_RK=<1|4|5|6|7>"
#endif
#define MGK_CAT2(a, b) a##b
#define MGK_CAT(a, b) MGK_CAT2(a, b)

// One translation unit per number of features keeps the build parallel.
hipError_t MGK_CAT(mgk_launch_pcg_sep_rk, MGK_PCG_SEP_RK)(int waves, int ept, int passes, const MgkBatchDev& X, const MgkBatchDev& Y,
                                                          const MgkSepList& SX, const MgkSepList& SY, const MgkJob* jobs_dev, int n_jobs,
                                                          const MgkParams& prm, int rb, size_t lds_bytes, const MgkOutputs& out,
                                                          hipStream_t stream) {
    if (n_jobs <= 0) return hipSuccess;
    if (lds_bytes > MGK_LDS_LIMIT_BYTES || rb < 1) return hipErrorInvalidValue;
    constexpr int RK = MGK_PCG_SEP_RK, G = RK == 1 ? 8 : 2;
    switch (waves * 100 + ept) {
#define MGK_CASE(W, E) \
    case W * 100 + E: return launch_one<RK, G, E, W>(X, Y, SX, SY, passes, jobs_dev, n_jobs, prm, rb, lds_bytes, out, stream);
        MGK_CASE(8, 4) MGK_CASE(8, 8)
        MGK_CASE(16, 6) MGK_CASE(16, 8) MGK_CASE(16, 10) MGK_CASE(16, 12) MGK_CASE(16, 14)
#undef MGK_CASE
        default: return hipErrorInvalidValue;
    }
}

// Off-diagonal product of the global-memory solver through a separable edge kernel
// (mgk_sep_dev.h): y = sum_k F_k P F'_k^T instead of one kappa_e evaluation per pair of
// nonzeros.  Two forms:
//
//  * mgk_sep_xmv_kernel: sparse.  One workgroup takes 16 outer rows.  Stage 1,
//    T_k[i, j'] = sum_j F_k[i, j] P[j, j']: lanes are columns j', the nonzeros of row i are
//    uniform operands.  Stage 2, y[i, i'] = sum_j' sum_k F'_k[i', j'] T_k[i, j']: lanes are
//    16 rows x 4 columns, T comes from LDS as 16-byte reads and the coefficients of a
//    column's nonzeros are shared by its 16 lanes.  Both stages take their coefficients
//    from packets of 16 words that hold whole nonzeros.
//  * mgk_sep_dense_kernel: well-filled graphs.  F_k and F'_k as dense matrices, both
//    stages on the matrix cores (v_mfma_f32_32x32x2_f32), T_k of 32 outer rows in LDS.
//
// Both store a = M p - y and form the workgroup's share of p^T a.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "mgk_internal.h"
#include "mgk_launch.h"
#include "mgk_sep_dev.h"
#include "mgk_wave.h"

namespace {

// phi_k(e) for the label e (see MgkSepBasis), in double so that the features are correctly
// rounded: they are made once per call and used in every iteration.  coef: S.coef, in LDS.
__device__ __forceinline__ float sep_feature(const MgkSepBasis& S, const double* coef, float label, int k) {
    const double s = ((double)label - S.center) * S.inv_r, s2 = s * s;
    double v = 0.0;
    for (int m = S.terms - 1; m >= 0; --m) v = fma(v, s2, coef[m * MGK_SEP_MAX_RANK + k]);
    return (float)(k & 1 ? v * s : v);
}

// Packets of the graphs a call uses: the vertices of a graph in order of descending degree, in
// groups of four; step t of a group holds packet t of its four rows, 16 words each.  A
// packet holds per_packet nonzeros of its row: rk coefficients A_ij phi_k and the byte offset of
// the slab of column j each; absent nonzeros have coefficients 0 and offset 0.  One wavefront
// per group.
__global__ __launch_bounds__(256) void mgk_sep_pack_kernel(MgkBatchDev B, MgkSepBasis S, MgkSepLayout L,
                                                           MgkSepList list, const MgkSepGraph* used, int packed, float* out) {
    __shared__ double coef[MGK_SEP_MAX_TERMS * MGK_SEP_MAX_RANK];
    for (int k = threadIdx.x; k < S.terms * MGK_SEP_MAX_RANK; k += blockDim.x) coef[k] = S.coef[k];
    __syncthreads();
    const MgkSepGraph sg = used[blockIdx.y];
    const int64_t at = packed ? sg.at : 0;   // packets of the whole batch are in order
    const MgkGraphDesc g = B.graphs[sg.graph];
    const int32_t* gptr = list.gptr + list.qoff[sg.graph];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int slot = lane & 15, number = L.numbers ? slot - MGK_SEP_NUMBER_SLOT : -1;   // >= 0: word of a column's number
    const int u = number >= 0 ? number : slot / (L.rk + 1), kk = number >= 0 ? L.rk : slot - u * (L.rk + 1);
    for (int grp = blockIdx.x * 4 + wave; grp * 4 < g.n; grp += gridDim.x * 4) {
        const int p0 = gptr[grp], p1 = gptr[grp + 1];
        const int pos = grp * 4 + (lane >> 4);
        const int row = list.deg_order[g.voff + min(pos, g.n - 1)];
        const int z0 = B.rowptr[g.voff + row];
        const int z1 = pos >= g.n ? z0 : row + 1 < g.n ? B.rowptr[g.voff + row + 1] : g.nnz;
        for (int p = p0; p < p1; ++p) {
            const int z = z0 + (p - p0) * L.per_packet + u;
            const bool on = u < L.per_packet && z < z1;
            const MgkEntry e = B.list_outer[g.zoff + (on ? z : 0)];
            const float w = __uint_as_float(e.w & 0x7fffffffu);
            for (int q = 0; q < L.passes; ++q) {
                const int k = q * L.rk + kk;
                float v = 0.f;
                if (on && kk < L.rk && k < S.rank) v = w * sep_feature(S, coef, __uint_as_float(e.z), k);
                if (on && kk == L.rk) v = __uint_as_float(e.y * (uint32_t)L.slab_bytes);
                if (number >= 0) v = __uint_as_float(on ? e.y : 0u);
                out[((int64_t)q * list.total + at + p) * 64 + lane] = v;
            }
        }
    }
}

// Dense F_k of the graphs a call uses: F[at + (k np + i) np + j], np = n rounded up to 64,
// zero where there is no edge.  One wavefront per (row, graph): the rows of as many features as there is room for, up to 1024 columns of them,
// are put together in LDS and written once (128 graphs of 256 vertices, density 0.2: 46 us, 80 cleared in memory and then filled; complete
// ones 123 and 112).
__global__ __launch_bounds__(256) void mgk_sep_dense_pack_kernel(MgkBatchDev B, MgkSepBasis S, const MgkSepGraph* used, float* out) {
    constexpr int kRoom = 2048, kWindow = 1024;   // words of a wavefront, columns at a time
    __shared__ double coef[MGK_SEP_MAX_TERMS * MGK_SEP_MAX_RANK];
    __shared__ __align__(16) float room[4][kRoom];
    for (int k = threadIdx.x; k < S.terms * MGK_SEP_MAX_RANK; k += blockDim.x) coef[k] = S.coef[k];
    __syncthreads();
    const MgkSepGraph sg = used[blockIdx.y];
    const MgkGraphDesc g = B.graphs[sg.graph];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int np = (g.n + 63) & ~63;
    float* F = out + sg.at * S.rank;
    float* mine = room[wave];
    for (int row = blockIdx.x * 4 + wave; row < np; row += gridDim.x * 4) {
        const int z0 = row < g.n ? B.rowptr[g.voff + row] : 0;
        const int z1 = row >= g.n ? 0 : row + 1 < g.n ? B.rowptr[g.voff + row + 1] : g.nnz;
        for (int c0 = 0; c0 < np; c0 += kWindow) {
            const int width = min(kWindow, np - c0), features = kRoom / width;
            for (int k0 = 0; k0 < S.rank; k0 += features) {
                const int k1 = min(S.rank, k0 + features);
                for (int c = lane * 4; c < (k1 - k0) * width; c += 256) *reinterpret_cast<float4*>(mine + c) = make_float4(0.f, 0.f, 0.f, 0.f);
                for (int z = z0 + lane; z < z1; z += 64) {
                    const MgkEntry e = B.list_outer[g.zoff + z];
                    const int c = (int)e.y - c0;
                    if (c < 0 || c >= width) continue;
                    const float w = __uint_as_float(e.w & 0x7fffffffu);
                    for (int k = k0; k < k1; ++k) mine[(k - k0) * width + c] = w * sep_feature(S, coef, __uint_as_float(e.z), k);
                }
                __threadfence_block();   // read by other lanes
                __builtin_amdgcn_wave_barrier();
                for (int k = k0; k < k1; ++k)
                    for (int c = lane * 4; c < width; c += 256)
                        *reinterpret_cast<float4*>(F + ((int64_t)k * np + row) * np + c0 + c) = *reinterpret_cast<const float4*>(mine + (k - k0) * width + c);
                __threadfence_block();   // and written again
                __builtin_amdgcn_wave_barrier();
            }
        }
    }
}

// Workgroup b of a 1-D grid -> (pair, block of the pair).  Consecutive workgroups go to the
// eight XCDs in turn: all blocks of a pair get the same b mod 8, so that its vectors and its
// graphs' coefficients are fetched into one XCD's L2 only.
__device__ __forceinline__ void sep_block(int b, int blocks, int* pair, int* blk) {
    const int slot = b >> 3;
    const int q = slot / blocks;
    *pair = q * 8 + (b & 7);
    *blk = slot - q * blocks;
}

// The workgroup's sum into *dst; red: a word of LDS per wavefront.  One addition per workgroup: those of a pair
// to its sum come one after the other, about 70 ns each (64 pairs of n = 256 at density 0.01, 256 wavefronts a pair:
// 51 us a product with one addition per wavefront, 34 with this).
template <int NW>
__device__ __forceinline__ void block_accumulate(float v, float* dst, float* red, int wave, int lane) {
    v = wave_sum(v);
    if (lane == 0) red[wave] = v;
    __syncthreads();
    if (wave == 0) {
        const float s = wave_sum(lane < NW ? red[lane] : 0.f);
        if (lane == 0) atomicAdd(dst, s);
    }
}

// Clears the accumulators of r^T z and r^T r that the update of this iteration adds to (their
// values, from two iterations ago, were last read by the kernel before this one).
__device__ __forceinline__ void clear_sums(MgkPairState& st, int it) {
    st.rz[it & 1] = 0.f;
    st.rr[it & 1] = 0.f;
}

// Per nonzero and 64 results RK multiply-adds (1.15 RK clk per CU) against 4 RK bytes x 64 from LDS in
// stage 2.  Counters at density 0.2, n = 256: vector ALUs 49 % of their issue slots, LDS 61 %, half of that
// bank conflicts, wavefronts waiting 78 % of their cycles: with one workgroup per CU the stages follow each
// other behind barriers.  About 20 multiply-adds per clk and CU.  64 such pairs: 13.5 ms per call with one
// evaluation per pair of nonzeros, 1.31 ms with this.  16 rows per workgroup so that T of one pass
// (RK <= 7) fits in LDS up to 276 columns and the coefficients of a column serve a whole row of 16 lanes.
template <int RK, int G>
__global__ __launch_bounds__(MGK_SEP_THREADS) void mgk_sep_xmv_kernel(MgkBatchDev X, MgkBatchDev Y, MgkSepList SX, MgkSepList SY,
                                                           MgkSepLayout L, const MgkLargePair* pairs, const MgkSepAt* feat,
                                                           MgkPairState* state, float* vec, MgkParams prm,
                                                           int n_pairs, int blocks, int it, int check_only) {
    extern __shared__ __align__(16) float lds[];
    constexpr int SLAB = MGK_SEP_SLAB(RK);            // words
    int pair, blk;
    sep_block(blockIdx.x, blocks, &pair, &blk);
    if (pair >= n_pairs) return;
    MgkPairState& st = state[pair];
    if (check_only ? !st.check : st.done) return;
    const MgkLargePair P = pairs[pair];
    const MgkSepAt F = feat[pair];
    const float* packets1 = SX.packets + F.f1 * 64;
    const float* packets2 = SY.packets + F.f2 * 64;
    const int i0 = blk * MGK_SEP_ROWS;
    if (i0 >= P.n1) return;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    constexpr int NW = MGK_SEP_THREADS / 64;
    if (blk == 0 && tid == 0 && !check_only) clear_sums(st, it);
    const MgkGraphDesc g1 = X.graphs[P.g1], g2 = Y.graphs[P.g2];
    const int n1 = P.n1, n2 = P.n2, rows = min(MGK_SEP_ROWS, n1 - i0);
    const float* p = vec + P.vec + 2 * (int64_t)P.npad;
    float* a = vec + P.vec + 4 * (int64_t)P.npad;
    const int32_t* order1 = SX.deg_order + g1.voff;
    const int32_t* order2 = SY.deg_order + g2.voff;
    float* tile = lds + SLAB * n2;                    // y of the 16 rows, row stride n2 | 1
    const int tp = n2 | 1;
    char* slabs = reinterpret_cast<char*>(lds);
    const int groups2 = (n2 + 3) >> 2;
    const int32_t* gp1 = SX.gptr + SX.qoff[P.g1];
    const int32_t* gp2 = SY.gptr + SY.qoff[P.g2];
    for (int q = 0; q < L.passes; ++q) {
        // ---- stage 1: one row per wavefront (rows of a workgroup have similar degrees)
        for (int ii = wave; ii < rows; ii += NW) {
            const int grp = (i0 + ii) >> 2;
            const int gb = gp1[grp];
            const float* pk = packets1 + ((int64_t)q * SX.total + gb) * 64 + ((i0 + ii) & 3) * 16 + (lane & 15);
            stage1_row<RK, G>(pk, gp1[grp + 1] - gb, PGlobal{reinterpret_cast<const char*>(p), (uint32_t)n2 * 4u}, n2, lane,
                              slabs, (RK == 1 ? 4u : 16u) * (uint32_t)ii);
        }
        __syncthreads();
        // ---- stage 2: 16 rows x 4 columns per task; the packets of the next task are in
        //      flight during this one
        const float* pk2 = packets2 + (int64_t)q * SY.total * 64 + lane;
        const uint32_t lbase = (RK == 1 ? 4u : 16u) * (uint32_t)(lane & 15);
        float cn[8];
        int gb = gp2[min(wave, groups2 - 1)], steps = gp2[min(wave, groups2 - 1) + 1] - gb;
#pragma unroll
        for (int a = 0; a < 8; ++a) cn[a] = pk2[(int64_t)(gb + max(min(a, steps - 1), 0)) * 64];
        for (int t = wave; t < groups2; t += NW) {
            float c[8];
#pragma unroll
            for (int a = 0; a < 8; ++a) c[a] = cn[a];
            const float* pk = pk2 + (int64_t)gb * 64;
            const int now = steps;
            if (t + NW < groups2) {
                gb = gp2[t + NW];
                steps = gp2[t + NW + 1] - gb;
#pragma unroll
                for (int a = 0; a < 8; ++a) cn[a] = pk2[(int64_t)(gb + max(min(a, steps - 1), 0)) * 64];
            }
            const float s = stage2_group<RK, G>(c, pk, now, slabs, lbase);
            const int cidx = t * 4 + (lane >> 4);
            if (cidx < n2) {
                float* dst = tile + (lane & 15) * tp + order2[cidx];
                *dst = q == 0 ? s : *dst + s;         // the same lane in every pass
            }
        }
        __syncthreads();
    }
    // ---- a = M p - y and this workgroup's share of p^T a
    float s_pa = 0.f;
    for (int ii = wave; ii < rows; ii += NW) {
        const int i = __builtin_amdgcn_readfirstlane(order1[i0 + ii]);
        const float d1 = X.rowsum[g1.voff + i] + prm.q, d1h = d1 / prm.h;
        const int lab1 = X.vlabel[g1.voff + i];
        for (int col = lane; col < n2; col += 64) {
            const float yv = tile[ii * tp + col];
            const int64_t at = (int64_t)i * n2 + col;
            const float pv = p[at];
            const float m = (lab1 == Y.vlabel[g2.voff + col] ? d1 : d1h) * (Y.rowsum[g2.voff + col] + prm.q);
            const float av = __builtin_fmaf(m, pv, -yv);
            s_pa = __builtin_fmaf(pv, av, s_pa);
            a[at] = av;
        }
    }
    if (!check_only) block_accumulate<NW>(s_pa, &st.pa[it & 1], lds, wave, lane);   // T is no longer read
}

typedef float f32x16 __attribute__((ext_vector_type(16)));

// One workgroup (4 wavefronts) takes 32 outer rows and all columns, NT tiles of 64 columns per
// wavefront.  Per k: T_k[32 x n'] = F_k P on the matrix cores, to LDS; y += T_k F'_k^T.  F_k and F'_k
// are symmetric, so every operand is read along rows (32 lanes = 128 adjacent bytes).
// Sums are kept in levels of 64 terms to bound the fp32 rounding bias of long running sums.
// Bound by the matrix cores (128 multiply-adds per clk and CU in fp32; 43 % busy) and, with two wavefronts
// per SIMD, by the latency of the operand loads: about 51 per clk measured on 64 pairs of complete
// 256-vertex graphs, 132 ms per call with the tile-pair kernel, 1.68 ms with this.
template <int NT>
__global__ __launch_bounds__(MGK_SEP_DENSE_THREADS) void mgk_sep_dense_kernel(MgkBatchDev X, MgkBatchDev Y, MgkSepList SX,
                                                            MgkSepList SY, int rank, const MgkLargePair* pairs, const MgkSepAt* feat,
                                                            MgkPairState* state, float* vec, MgkParams prm,
                                                            int n_pairs, int blocks, int it, int check_only) {
    extern __shared__ __align__(16) float lds[];   // T_k, 32 rows of stride tp
    int pair, blk;
    sep_block(blockIdx.x, blocks, &pair, &blk);
    if (pair >= n_pairs) return;
    MgkPairState& st = state[pair];
    if (check_only ? !st.check : st.done) return;
    const MgkLargePair P = pairs[pair];
    const MgkSepAt F = feat[pair];
    const int i0 = blk * MGK_SEP_DENSE_ROWS;
    if (i0 >= P.n1) return;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    if (blk == 0 && tid == 0 && !check_only) clear_sums(st, it);
    const MgkGraphDesc g1 = X.graphs[P.g1], g2 = Y.graphs[P.g2];
    const int n1 = P.n1, n2 = P.n2, np1 = (n1 + 63) & ~63, np2 = (n2 + 63) & ~63;
    const float* F1 = SX.dense + F.f1 + i0;
    const float* F2 = SY.dense + F.f2;
    const float* p = vec + P.vec + 2 * (int64_t)P.npad;
    float* a = vec + P.vec + 4 * (int64_t)P.npad;
    const int tp = np2 + 1;
    const int r = lane & 31, half = lane >> 5;
    f32x16 yacc[NT][2];
#pragma unroll
    for (int t = 0; t < NT; ++t)
#pragma unroll
        for (int b = 0; b < 2; ++b)
#pragma unroll
            for (int v = 0; v < 16; ++v) yacc[t][b][v] = 0.f;
    for (int k = 0; k < rank; ++k) {
        const float* A = F1 + (int64_t)k * np1 * np1;
        // ---- T_k = F_k P; rows of F_k beyond n1 are zero, columns of p beyond n2 are
        //      harmless (the rows of F'_k they meet are zero)
#pragma unroll
        for (int t = 0; t < NT; ++t) {
            const int c0 = (t * 4 + wave) * 64;
            if (c0 < np2) {
                f32x16 acc[2], tot[2];
#pragma unroll
                for (int b = 0; b < 2; ++b)
#pragma unroll
                    for (int v = 0; v < 16; ++v) tot[b][v] = 0.f;
                const int cA = min(c0 + r, n2 - 1), cB = min(c0 + 32 + r, n2 - 1);
                for (int j0 = 0; j0 < n1; j0 += 64) {
#pragma unroll
                    for (int b = 0; b < 2; ++b)
#pragma unroll
                        for (int v = 0; v < 16; ++v) acc[b][v] = 0.f;
                    const int j1 = min(j0 + 64, (n1 + 15) & ~15);
                    for (int j = j0; j < j1; j += 16) {
                        float av[8], b0[8], b1[8];
#pragma unroll
                        for (int s = 0; s < 8; ++s) {
                            const int jj = j + 2 * s + half;
                            const float* prow = p + (int64_t)min(jj, n1 - 1) * n2;
                            av[s] = A[(int64_t)jj * np1 + r];
                            b0[s] = prow[cA];
                            b1[s] = prow[cB];
                        }
#pragma unroll
                        for (int s = 0; s < 8; ++s) {
                            acc[0] = __builtin_amdgcn_mfma_f32_32x32x2f32(av[s], b0[s], acc[0], 0, 0, 0);
                            acc[1] = __builtin_amdgcn_mfma_f32_32x32x2f32(av[s], b1[s], acc[1], 0, 0, 0);
                        }
                    }
#pragma unroll
                    for (int b = 0; b < 2; ++b)
#pragma unroll
                        for (int v = 0; v < 16; ++v) tot[b][v] += acc[b][v];
                }
#pragma unroll
                for (int b = 0; b < 2; ++b)
#pragma unroll
                    for (int v = 0; v < 16; ++v)
                        lds[(8 * (v >> 2) + 4 * half + (v & 3)) * tp + c0 + 32 * b + r] = tot[b][v];
            }
        }
        __syncthreads();
        // ---- y += T_k F'_k^T
        const float* Bm = F2 + (int64_t)k * np2 * np2;
#pragma unroll
        for (int t = 0; t < NT; ++t) {
            const int c0 = (t * 4 + wave) * 64;
            if (c0 < np2) {
                f32x16 acc[2];
                for (int j0 = 0; j0 < n2; j0 += 64) {
#pragma unroll
                    for (int b = 0; b < 2; ++b)
#pragma unroll
                        for (int v = 0; v < 16; ++v) acc[b][v] = 0.f;
                    const int j1 = min(j0 + 64, (n2 + 15) & ~15);
                    for (int j = j0; j < j1; j += 16) {
                        float av[8], b0[8], b1[8];
#pragma unroll
                        for (int s = 0; s < 8; ++s) {
                            const int jj = j + 2 * s + half;
                            const float* brow = Bm + (int64_t)jj * np2 + c0 + r;
                            av[s] = lds[r * tp + jj];
                            b0[s] = brow[0];
                            b1[s] = brow[32];
                        }
#pragma unroll
                        for (int s = 0; s < 8; ++s) {
                            acc[0] = __builtin_amdgcn_mfma_f32_32x32x2f32(av[s], b0[s], acc[0], 0, 0, 0);
                            acc[1] = __builtin_amdgcn_mfma_f32_32x32x2f32(av[s], b1[s], acc[1], 0, 0, 0);
                        }
                    }
#pragma unroll
                    for (int b = 0; b < 2; ++b)
#pragma unroll
                        for (int v = 0; v < 16; ++v) yacc[t][b][v] += acc[b][v];
                }
            }
        }
        __syncthreads();
    }
    // ---- a = M p - y and this workgroup's share of p^T a
    float s_pa = 0.f;
#pragma unroll
    for (int t = 0; t < NT; ++t)
#pragma unroll
        for (int b = 0; b < 2; ++b) {
            const int col = (t * 4 + wave) * 64 + 32 * b + r;
            if (col >= n2) continue;
            const float d2 = Y.rowsum[g2.voff + col] + prm.q;
            const int lab2 = Y.vlabel[g2.voff + col];
#pragma unroll
            for (int v = 0; v < 16; ++v) {
                const int i = i0 + 8 * (v >> 2) + 4 * half + (v & 3);
                if (i < n1) {
                    const int64_t at = (int64_t)i * n2 + col;
                    const float yv = yacc[t][b][v], pv = p[at];
                    const float d1 = X.rowsum[g1.voff + i] + prm.q;
                    const float m = (lab2 == X.vlabel[g1.voff + i] ? d1 : d1 / prm.h) * d2;
                    const float av = __builtin_fmaf(m, pv, -yv);
                    s_pa = __builtin_fmaf(pv, av, s_pa);
                    a[at] = av;
                }
            }
        }
    if (!check_only) block_accumulate<MGK_SEP_DENSE_THREADS / 64>(s_pa, &st.pa[it & 1], lds, wave, lane);   // T is no longer read
}

// ---- the same for pairs of at most 256 by 256 vertices, with every operand as three bfloat16 parts -----------------
// x = hi + mid + lo exactly (8 bits each), and the six products of parts above 2^-24 of a b on the 16-bit matrix cores, which do
// 16 times as many multiply-adds a clk as the fp32 ones; sums are in fp32, those of hi hi apart from the rest, whose roundings
// then are 2^-8 as large: error against fp64 as with the fp32 instructions or less (values 0.8e-7 and 0.7e-7 rms).
// 64 pairs of complete 256-vertex graphs: 101 us a product, 236 with the fp32 matrix instructions; per call 1668 -> 819 us.  Bound by what the
// matrix cores (half of their time) and the vector ALUs that take operands apart leave each other with two wavefronts to a SIMD.
// One workgroup of eight wavefronts takes 64 inner columns.  Per k: F'_k of its columns to LDS, T_k = P F'_k
// (a wavefront 32 rows), T_k to LDS in its place, y += F_k T_k.  P and F_k are read from L2 as they are and taken apart
// in registers; every wavefront reads its rows only, what all share comes from LDS.
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef float f32x2 __attribute__((ext_vector_type(2)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
typedef float f32x4_dword __attribute__((ext_vector_type(4), aligned(4)));   // rows of p begin anywhere

constexpr int kPartsThreads = MGK_SEP_PARTS_THREADS, kPartsStride = MGK_SEP_PARTS_MAX_N + 8;   // 16-bit words of a column's part in LDS: columns 4 banks apart
constexpr int kPartsLds = 3 * 64 * kPartsStride * 2;
static_assert(kPartsLds == MGK_SEP_PARTS_LDS && kPartsThreads / 64 * 32 == MGK_SEP_PARTS_MAX_N, "a wavefront per 32 rows");

// Two numbers into three parts each.
__device__ __forceinline__ void split2(float x, float y, uint32_t (&part)[3]) {
#pragma unroll
    for (int k = 0; k < 3; ++k) {
        const uint32_t w = __builtin_bit_cast(uint32_t, __builtin_convertvector(f32x2{x, y}, bf16x2));
        part[k] = w;
        x -= __uint_as_float(w << 16);
        y -= __uint_as_float(w & 0xffff0000u);
    }
}
struct Parts {   // eight numbers
    u32x4 w[3];
    __device__ __forceinline__ void set(const float (&x)[8]) {
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            uint32_t part[3];
            split2(x[2 * q], x[2 * q + 1], part);
#pragma unroll
            for (int k = 0; k < 3; ++k) w[k][q] = part[k];
        }
    }
};
__device__ __forceinline__ f32x16 mfma_parts(u32x4 a, u32x4 b, f32x16 c) {
    return __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, a), __builtin_bit_cast(bf16x8, b), c, 0, 0, 0);
}
__device__ __forceinline__ void load8(float (&x)[8], const float* from) {
    const f32x4_dword a = *reinterpret_cast<const f32x4_dword*>(from), b = *reinterpret_cast<const f32x4_dword*>(from + 4);
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        x[q] = a[q];
        x[4 + q] = b[q];
    }
}

// 32 rows by 64 columns: hi[t] + rest[t] = rows (row: this lane's, of K numbers) times what is in LDS, K in steps of 16.  The
// numbers of the last step that a row does not have are its last one.  Loads one step ahead (two: 107
// instead of 101 us a product of 64 pairs of 256 by 256).
__device__ __forceinline__ void product_parts(f32x16 (&hi)[2], f32x16 (&rest)[2], const float* row, int K, const uint16_t* lds, int r, int half) {
#pragma unroll
    for (int t = 0; t < 2; ++t)
#pragma unroll
        for (int v = 0; v < 16; ++v) hi[t][v] = rest[t][v] = 0.f;
    auto step = [&](const float (&x)[8], int k0) {
        Parts a;
        a.set(x);
        const uint16_t* from = lds + r * kPartsStride + k0 + 8 * half;
#pragma unroll
        for (int t = 0; t < 2; ++t) {
            u32x4 b[3];
#pragma unroll
            for (int k = 0; k < 3; ++k) b[k] = *reinterpret_cast<const u32x4*>(from + (k * 64 + 32 * t) * kPartsStride);
            hi[t] = mfma_parts(a.w[0], b[0], hi[t]);
            rest[t] = mfma_parts(a.w[0], b[1], rest[t]);
            rest[t] = mfma_parts(a.w[1], b[0], rest[t]);
            rest[t] = mfma_parts(a.w[1], b[1], rest[t]);
            rest[t] = mfma_parts(a.w[0], b[2], rest[t]);
            rest[t] = mfma_parts(a.w[2], b[0], rest[t]);
        }
    };
    const int full = K & ~15;
    if (full > 0) {
        float next[8];
        load8(next, row + 8 * half);
        for (int k0 = 0; k0 < full; k0 += 16) {
            float now[8];
#pragma unroll
            for (int q = 0; q < 8; ++q) now[q] = next[q];
            load8(next, row + min(k0 + 16, full - 16) + 8 * half);
            step(now, k0);
        }
    }
    if (full < K) {
        float x[8];
#pragma unroll
        for (int q = 0; q < 8; ++q) x[q] = row[min(full + 8 * half + q, K - 1)];
        step(x, full);
    }
}

__global__ __launch_bounds__(kPartsThreads, 2) void mgk_sep_dense_parts_kernel(MgkBatchDev X, MgkBatchDev Y, MgkSepList SX, MgkSepList SY, int rank,
                                                                               const MgkLargePair* pairs, const MgkSepAt* feat,
                                                                               MgkPairState* state, float* vec, MgkParams prm, int n_pairs,
                                                                               int blocks, int it, int check_only) {
    extern __shared__ __align__(16) float lds[];
    uint16_t* const part = reinterpret_cast<uint16_t*>(lds);
    int pair, blk;
    sep_block(blockIdx.x, blocks, &pair, &blk);
    if (pair >= n_pairs) return;
    MgkPairState& st = state[pair];
    if (check_only ? !st.check : st.done) return;
    const MgkLargePair P = pairs[pair];
    const MgkSepAt F = feat[pair];
    const int c0 = blk * 64;
    if (c0 >= P.n2) return;
    const int tid = threadIdx.x, lane = tid & 63, r = lane & 31, half = lane >> 5;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    if (blk == 0 && tid == 0 && !check_only) clear_sums(st, it);
    const int n1 = P.n1, n2 = P.n2, np1 = (n1 + 63) & ~63, np2 = (n2 + 63) & ~63;
    const int voff1 = P.voff1, voff2 = P.voff2;
    const float* F1 = SX.dense + F.f1;
    const float* F2 = SY.dense + F.f2;
    const float* p = vec + P.vec + 2 * (int64_t)P.npad;
    float* a = vec + P.vec + 4 * (int64_t)P.npad;
    const int i0 = wave * 32, K1 = (n1 + 15) & ~15, K2 = (n2 + 15) & ~15;
    const bool on = i0 < n1;   // wave-uniform
    f32x16 y[2];
#pragma unroll
    for (int t = 0; t < 2; ++t)
#pragma unroll
        for (int v = 0; v < 16; ++v) y[t][v] = 0.f;
    for (int k = 0; k < rank; ++k) {
        // ---- F'_k of the columns (symmetric: its rows), zero beyond n2
        const float* B = F2 + ((int64_t)k * np2 + c0) * np2;
        for (int e = tid; e < 64 * (K2 / 8); e += kPartsThreads) {
            const int c = e / (K2 / 8), j = (e - c * (K2 / 8)) * 8;
            float x[8];
            load8(x, B + (int64_t)c * np2 + j);
            Parts s;
            s.set(x);
#pragma unroll
            for (int q = 0; q < 3; ++q) *reinterpret_cast<u32x4*>(part + (q * 64 + c) * kPartsStride + j) = s.w[q];
        }
        __syncthreads();
        f32x16 hi[2], rest[2];
        if (on) product_parts(hi, rest, p + (int64_t)min(i0 + r, n1 - 1) * n2, n2, part, r, half);
        __syncthreads();
        // ---- T_k: this lane has rows i0 + 8 (v / 4) + 4 half + v % 4 of a column
        if (on) {
#pragma unroll
            for (int t = 0; t < 2; ++t)
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    uint32_t s0[3], s1[3];
                    split2(hi[t][4 * q] + rest[t][4 * q], hi[t][4 * q + 1] + rest[t][4 * q + 1], s0);
                    split2(hi[t][4 * q + 2] + rest[t][4 * q + 2], hi[t][4 * q + 3] + rest[t][4 * q + 3], s1);
#pragma unroll
                    for (int m = 0; m < 3; ++m)
                        *reinterpret_cast<u32x2*>(part + (m * 64 + 32 * t + r) * kPartsStride + i0 + 8 * q + 4 * half) = u32x2{s0[m], s1[m]};
                }
        }
        __syncthreads();
        if (on) {   // columns of F_k beyond n1 are zero, rows of T_k there finite
            product_parts(hi, rest, F1 + ((int64_t)k * np1 + min(i0 + r, np1 - 1)) * np1, K1, part, r, half);
#pragma unroll
            for (int t = 0; t < 2; ++t)
#pragma unroll
                for (int v = 0; v < 16; ++v) y[t][v] += hi[t][v] + rest[t][v];
        }
        __syncthreads();
    }
    // ---- a = M p - y and this workgroup's share of p^T a
    float s_pa = 0.f;
#pragma unroll
    for (int t = 0; t < 2; ++t) {
        const int col = c0 + 32 * t + r;
        if (col >= n2) continue;
        const float d2 = Y.rowsum[voff2 + col] + prm.q;
        const int lab2 = Y.vlabel[voff2 + col];
#pragma unroll
        for (int v = 0; v < 16; ++v) {
            const int i = i0 + 8 * (v >> 2) + 4 * half + (v & 3);
            if (i < n1) {
                const int64_t at = (int64_t)i * n2 + col;
                const float pv = p[at], d1 = X.rowsum[voff1 + i] + prm.q;
                const float m = (lab2 == X.vlabel[voff1 + i] ? d1 : d1 / prm.h) * d2;
                const float av = __builtin_fmaf(m, pv, -y[t][v]);
                s_pa = __builtin_fmaf(pv, av, s_pa);
                a[at] = av;
            }
        }
    }
    if (!check_only) block_accumulate<kPartsThreads / 64>(s_pa, &st.pa[it & 1], lds, wave, lane);   // T is no longer read
}

hipError_t set_lds(const void* kern, bool* configured) {
    if (*configured) return hipSuccess;
    hipError_t e = hipFuncSetAttribute(kern, hipFuncAttributeMaxDynamicSharedMemorySize, MGK_LDS_LIMIT_BYTES);
    if (e == hipSuccess) *configured = true;
    return e;
}

}  // namespace

// the graph index is a grid dimension of at most 65535: more graphs go in parts
hipError_t mgk_launch_sep_pack(const MgkBatchDev& B, const MgkSepBasis& S, const MgkSepLayout& L, const MgkSepList& list,
                               const MgkSepGraph* used, int n_used, int max_n, float* packets, hipStream_t stream) {
    const int gx = (max_n + 15) / 16;
    for (int g0 = 0; g0 < n_used; g0 += 65535)
        hipLaunchKernelGGL(mgk_sep_pack_kernel, dim3(gx, n_used - g0 < 65535 ? n_used - g0 : 65535), dim3(256), 0,
                           stream, B, S, L, list, used + g0, used == list.whole ? 0 : 1, packets);
    return hipGetLastError();
}

hipError_t mgk_launch_sep_dense_pack(const MgkBatchDev& B, const MgkSepBasis& S, const MgkSepGraph* used, int n_used, int max_n,
                                     float* F, hipStream_t stream) {
    const int gx = (max_n + 63) / 64 * 16;   // a row to a wavefront
    for (int g0 = 0; g0 < n_used; g0 += 65535)
        hipLaunchKernelGGL(mgk_sep_dense_pack_kernel, dim3(gx, n_used - g0 < 65535 ? n_used - g0 : 65535), dim3(256), 0,
                           stream, B, S, used + g0, F);
    return hipGetLastError();
}

hipError_t mgk_launch_sep_xmv(const MgkBatchDev& X, const MgkBatchDev& Y, const MgkSepList& SX, const MgkSepList& SY,
                              const MgkSepLayout& L, const MgkLargePair* pairs, const MgkSepAt* feat, MgkPairState* state, float* vec,
                              const MgkParams& prm, int n_pairs, int max_n1, int max_n2, int it, bool check_only, hipStream_t stream) {
    const int blocks = (max_n1 + MGK_SEP_ROWS - 1) / MGK_SEP_ROWS;
    const dim3 grid((unsigned)mgk_sep_grid(n_pairs, max_n1, MGK_SEP_ROWS));
    const size_t bytes = mgk_sep_lds_bytes(L.rk, max_n2);
    if (bytes > MGK_LDS_LIMIT_BYTES) return hipErrorInvalidValue;
#define MGK_SEP_GO(RK, G) \
    case RK: { \
        auto kern = mgk_sep_xmv_kernel<RK, G>; \
        static bool configured = false; \
        hipError_t e = set_lds(reinterpret_cast<const void*>(kern), &configured); \
        if (e != hipSuccess) return e; \
        hipLaunchKernelGGL(kern, grid, dim3(MGK_SEP_THREADS), bytes, stream, X, Y, SX, SY, L, pairs, feat, state, vec, prm, n_pairs, blocks, it, check_only ? 1 : 0); \
        break; \
    }
    switch (L.rk) {
        MGK_SEP_GO(1, 8) MGK_SEP_GO(4, 2) MGK_SEP_GO(5, 2) MGK_SEP_GO(6, 2) MGK_SEP_GO(7, 2)
        default: return hipErrorInvalidValue;
    }
#undef MGK_SEP_GO
    return hipGetLastError();
}

hipError_t mgk_launch_sep_dense(const MgkBatchDev& X, const MgkBatchDev& Y, const MgkSepList& SX, const MgkSepList& SY, int rank,
                                bool parts, const MgkLargePair* pairs, const MgkSepAt* feat, MgkPairState* state, float* vec, const MgkParams& prm,
                                int n_pairs, int max_n1, int max_n2, int it, bool check_only, hipStream_t stream) {
    if (parts) {
        if (!mgk_sep_in_parts(max_n1, max_n2)) return hipErrorInvalidValue;
        static bool configured = false;
        const hipError_t e = set_lds(reinterpret_cast<const void*>(mgk_sep_dense_parts_kernel), &configured);
        if (e != hipSuccess) return e;
        hipLaunchKernelGGL(mgk_sep_dense_parts_kernel, dim3((unsigned)mgk_sep_grid(n_pairs, max_n2, 64)), dim3(kPartsThreads), kPartsLds, stream, X, Y, SX,
                           SY, rank, pairs, feat, state, vec, prm, n_pairs, (max_n2 + 63) / 64, it, check_only ? 1 : 0);
        return hipGetLastError();
    }
    const int blocks = (max_n1 + MGK_SEP_DENSE_ROWS - 1) / MGK_SEP_DENSE_ROWS;
    const dim3 grid((unsigned)mgk_sep_grid(n_pairs, max_n1, MGK_SEP_DENSE_ROWS));
    const int np2 = (max_n2 + 63) & ~63;
    const size_t bytes = (size_t)32 * (np2 + 1) * sizeof(float);
    if (np2 > MGK_SEP_DENSE_MAX_N) return hipErrorInvalidValue;
#define MGK_SEP_DENSE_GO(NT) \
    { \
        auto kern = mgk_sep_dense_kernel<NT>; \
        static bool configured = false; \
        hipError_t e = set_lds(reinterpret_cast<const void*>(kern), &configured); \
        if (e != hipSuccess) return e; \
        hipLaunchKernelGGL(kern, grid, dim3(MGK_SEP_DENSE_THREADS), bytes, stream, X, Y, SX, SY, rank, pairs, feat, state, vec, prm, n_pairs, blocks, it, check_only ? 1 : 0); \
    }
    switch (mgk_sep_dense_tiles(max_n2)) {
        case 1: MGK_SEP_DENSE_GO(1) break;
        case 2: MGK_SEP_DENSE_GO(2) break;
        default: MGK_SEP_DENSE_GO(4)
    }
#undef MGK_SEP_DENSE_GO
    return hipGetLastError();
}

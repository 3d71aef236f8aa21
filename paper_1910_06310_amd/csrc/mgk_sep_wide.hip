// Off-diagonal product of the global-memory solver through a separable edge kernel, for sparse graphs of too many
// vertices for T of 16 outer rows to fit in LDS (mgk_sep.hip): 4 or 8 outer rows to a workgroup.
//
// With fewer rows to share them, the coefficients of the second stage would be read from L2 as often as the LDS reads T.
// So the kernel is separated into powers on the inner side (MgkWideBasis): kappa_e(e, e') = g(e') sum_l psi_l(e) s'^l,
//   T_l[i, j'] = sum_j A_ij psi_l(E_ij) P[j, j'],   y[i, i'] = sum_j' A'_i'j' g(E'_i'j') (T_0 + s' (T_1 + s' (T_2 + ...))),
// and a nonzero of the inner graph is three words whatever the rank: where T of its column is, s', A' g.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "mgk_internal.h"
#include "mgk_launch.h"
#include "mgk_wave.h"

namespace {

constexpr int kThreads = MGK_WIDE_THREADS, kWaves = kThreads / 64;
#define MGK_CONSTANT __attribute__((address_space(4)))   // read with scalar loads, also beside stores

// ---- features of the graphs a call uses -----------------------------------------------------------------
// Outer side, per nonzero and pass 8 or 12 words: its coefficients A_ij psi_l of the pass, and in the last word its column.
__global__ __launch_bounds__(256) void mgk_wide_outer_kernel(MgkBatchDev B, MgkWideBasis S, MgkWideLayout L, const MgkSepGraph* used,
                                                             int64_t total, float* out) {
    __shared__ double coef[MGK_SEP_MAX_TERMS * MGK_SEP_MAX_RANK];
    for (int k = threadIdx.x; k < S.outer.terms * MGK_SEP_MAX_RANK; k += blockDim.x) coef[k] = S.outer.coef[k];
    __syncthreads();
    const MgkSepGraph sg = used[blockIdx.y];
    const MgkGraphDesc g = B.graphs[sg.graph];
    for (int z = blockIdx.x * blockDim.x + threadIdx.x; z < g.nnz; z += gridDim.x * blockDim.x) {
        const MgkEntry e = B.list_outer[g.zoff + z];
        const float w = __uint_as_float(e.w & 0x7fffffffu);
        const double s = ((double)__uint_as_float(e.z) - S.outer.center) * S.outer.inv_r, s2 = s * s;
        for (int q = 0; q < L.passes; ++q) {
            const int first = mgk_wide_first(L, q), count = q == 0 ? L.hi : L.lo;
            const int words = mgk_wide_record(L.hi);
            float* rec = out + ((int64_t)q * total + sg.at + z) * words;
            for (int k = 0; k < words - 1; ++k) rec[k] = 0.f;
            rec[words - 1] = __uint_as_float(e.y);
            for (int k = 0; k < count && first + k < S.outer.rank; ++k) {
                double v = 0.0;
                for (int m = S.outer.terms - 1; m >= 0; --m) v = fma(v, s2, coef[m * MGK_SEP_MAX_RANK + first + k]);
                rec[k] = w * (float)((first + k) & 1 ? v * s : v);
            }
        }
    }
}

// Which of the four 64-byte parts of all LDS banks the quadruples of column j lie in that lanes of one cycle read with a 16-byte
// read, with 4 rows: a cycle takes 16 lanes, of the columns at places {0, 3, 5, 6}, {1, 2, 4, 7}, {8, 11, 13, 14} or {9, 10, 12, 15} of a group of 16.
__device__ __forceinline__ int wide_part(uint32_t j) { return (int)(j & 3u); }   // column j < 4 lies in part j

// Inner side: the columns by descending degree in groups of 16; step p of a group holds nonzeros 4p .. 4p + 3 of every
// column, column after column: 64 words with the byte offset of the column's T, 64 with s', 64 with A' g s'^first.
// In front of a graph's steps the first step of every group.  Absent nonzeros are zeros.
// With 4 rows the nonzeros of a column (of up to 64) come in an order in which the four columns read
// together rarely meet in a bank: the part with the most left that the others do not take.  2048 columns of degree 12: conflicts are 28 % of the
// product's LDS cycles, 45 % in the order of the rows (1074 -> 1039 us a product); this kernel takes 58 us for 16 such graphs, most of them for the order.
__global__ __launch_bounds__(256) void mgk_wide_inner_kernel(MgkBatchDev B, MgkWideBasis S, MgkWideLayout L, const int32_t* deg_order,
                                                             const MgkSepGraph* used, float* out) {
    constexpr int kMost = 64;   // nonzeros of a row that is ordered
    __shared__ int32_t first[MGK_WIDE_MAX_N / 16 + 1];
    __shared__ uint8_t by_part[4][16][kMost], turn[4][16][kMost], parts[4][16][4];
    const MgkSepGraph sg = used[blockIdx.y];
    const MgkGraphDesc g = B.graphs[sg.graph];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, groups = (g.n + 15) >> 4;
    const int32_t* rowptr = B.rowptr + g.voff;
    const int32_t* order = deg_order + g.voff;
    const MgkEntry* list = B.list_outer + g.zoff;
    float* to = out + sg.at;
    auto row_end = [&](int row) { return row + 1 < g.n ? rowptr[row + 1] : g.nnz; };
    for (int t = threadIdx.x; t < groups; t += blockDim.x) {
        const int row = order[t * 16];
        first[t] = (row_end(row) - rowptr[row] + 3) >> 2;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        int sum = 0;
        for (int t = 0; t <= groups; ++t) {
            const int steps = t < groups ? first[t] : 0;
            first[t] = sum;
            sum += steps;
        }
    }
    __syncthreads();
    if (blockIdx.x == 0)
        for (int t = threadIdx.x; t <= groups; t += blockDim.x) to[t] = __int_as_float(first[t]);
    const int head = mgk_wide_head(g.n), cap = mgk_wide_steps(g);
    const int c = lane >> 2, u = lane & 3;
    for (int t = blockIdx.x * 4 + wave; t < groups; t += gridDim.x * 4) {
        const int pos = t * 16 + c, row = order[min(pos, g.n - 1)];
        const int z0 = rowptr[row], z1 = pos < g.n ? row_end(row) : z0;
        const int steps = first[t + 1] - first[t];
        const bool ordered = L.rows == 4 && steps * 4 <= kMost;   // the same for all lanes
        if (ordered) {
            // a column's nonzeros by part: lane u of the column collects part u
            int n = 0;
            for (int z = z0; z < z1; ++z) n += wide_part(list[z].y) == u;
            parts[wave][c][u] = (uint8_t)n;
            int at = 0;
            for (int v = 0; v < 3; ++v) {
                const int m = __shfl(n, (lane & ~3) + v);
                at += v < u ? m : 0;
            }
            for (int z = z0; z < z1; ++z)
                if (wide_part(list[z].y) == u) by_part[wave][c][at++] = (uint8_t)(z - z0);
            __threadfence_block();
            __builtin_amdgcn_wave_barrier();
            if (lane < 4) {   // one lane for the four columns of a cycle
                int col[4], left[4][4], next[4][4];
#pragma unroll
                for (int k = 0; k < 4; ++k) {
                    const int places = lane & 1 ? 0x7421 : 0x6530;
                    col[k] = (lane & 2) * 4 + ((places >> (4 * k)) & 15);
                    int sum = 0;
#pragma unroll
                    for (int v = 0; v < 4; ++v) {
                        left[k][v] = parts[wave][col[k]][v];
                        next[k][v] = sum;
                        sum += left[k][v];
                    }
                }
                for (int slot = 0; slot < steps * 4; ++slot) {
                    int taken = 0;
#pragma unroll
                    for (int kk = 0; kk < 4; ++kk) {
                        int best = -1, most = 0, k = (kk + slot) & 3, from = 0;
#pragma unroll
                        for (int m = 0; m < 4; ++m)   // static indexes: column k in turn
                            if (m == k) {
#pragma unroll
                                for (int v = 0; v < 4; ++v) {
                                    const int score = left[m][v] == 0 ? 0 : left[m][v] + (taken >> v & 1 ? 0 : 256);
                                    if (score > most) { most = score; best = v; }
                                }
#pragma unroll
                                for (int v = 0; v < 4; ++v)
                                    if (v == best) { from = next[m][v]++; --left[m][v]; }
                                if (best >= 0) {
                                    taken |= 1 << best;
                                    turn[wave][col[m]][slot] = by_part[wave][col[m]][from];
                                } else {   // none left: a part that no one reads
                                    const int free = __ffs(~taken & 15) - 1;
                                    taken |= 1 << free;
                                    turn[wave][col[m]][slot] = (uint8_t)(0x80 | free);
                                }
                            }
                    }
                }
            }
            __threadfence_block();
            __builtin_amdgcn_wave_barrier();
        }
        for (int p = 0; p < steps; ++p) {
            const int i = ordered ? turn[wave][c][p * 4 + u] : p * 4 + u, z = z0 + i;
            const bool on = ordered ? i < 0x80 : z < z1;
            const MgkEntry e = list[on ? z : 0];
            const double s = ((double)__uint_as_float(e.z) - S.outer.center) * S.outer.inv_r;
            const double w = (double)__uint_as_float(e.w & 0x7fffffffu) * exp(-S.half_t * s * s);
            const uint32_t at = mgk_wide_column(L.rows, on ? e.y : ordered ? (uint32_t)(i & 3) : 0u);
            for (int q = 0; q < L.passes; ++q) {
                double power = 1.0;
                for (int k = mgk_wide_first(L, q); k > 0; --k) power *= s;
                float* step = to + head + ((int64_t)q * cap + first[t] + p) * 192 + lane;
                step[0] = __uint_as_float(at);
                step[64] = on ? (float)s : 0.f;
                step[128] = on ? (float)(w * power) : 0.f;
            }
        }
        __builtin_amdgcn_wave_barrier();
    }
}

// ---- product --------------------------------------------------------------------------------------------
// Value of lane U of every four lanes, in all of them: the compiler makes it the DPP control of the instruction that uses it.
template <int U>
__device__ __forceinline__ uint32_t quad_bcast(uint32_t c) {
    return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)c, U * 0x55, 0xf, 0xf, true);
}
template <int U>
__device__ __forceinline__ float quad_bcast(float c) {
    return __uint_as_float(quad_bcast<U>(__float_as_uint(c)));
}

// T of R rows in LDS: per column R quadruples, row r's at position r ^ (column / (16 / R) mod R), so that lanes that
// are 64 adjacent columns write to all banks; with eight features or more a second array of quadruples behind it, and what
// is left of RK by four as an array of single values or of twos behind those, all in the same order.
// LDS by its address: the kernel has no other than the dynamic one, which begins at 0.
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef float f32x2 __attribute__((ext_vector_type(2)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
#define MGK_SHARED __attribute__((address_space(3)))
template <class V>
__device__ __forceinline__ MGK_SHARED V* shared(uint32_t at) {
    return (MGK_SHARED V*)(uintptr_t)at;
}
// at: of the column and row in the first array; part: bytes of one array of quadruples
template <int RK>
__device__ __forceinline__ void t_write(uint32_t part, uint32_t at, const float (&v)[RK]) {
    *shared<f32x4>(at) = f32x4{v[0], v[1], v[2], v[3]};
    if constexpr (RK >= 8) *shared<f32x4>(at + part) = f32x4{v[4], v[5], v[6], v[7]};
    if constexpr (RK % 4 == 1) *shared<float>((at >> 2) + RK / 4 * part) = v[RK - 1];
    if constexpr (RK % 4 == 2) *shared<f32x2>((at >> 1) + RK / 4 * part) = f32x2{v[RK - 2], v[RK - 1]};
}

// Stage 1, NB nonzeros of a row: their records (in scalar registers) times p at this lane's C columns.
template <int RK>
struct Record {
    u32x4 a, b, c;
    __device__ __forceinline__ void load(const MGK_CONSTANT u32x4* r) {
        a = r[0];
        b = r[1];
        if constexpr (RK > 6) c = r[2];
    }
    __device__ __forceinline__ uint32_t column() const { return RK > 6 ? c[3] : b[3]; }
    __device__ __forceinline__ float coef(int k) const { return __uint_as_float(k < 4 ? a[k] : k < 8 ? b[k - 4] : c[k - 8]); }
};
template <int RK, int C, int NB>
__device__ __forceinline__ void wide_products(float (&acc)[C][RK], const MGK_CONSTANT u32x4* rec, const char* p, uint32_t row_bytes,
                                              const uint32_t (&col4)[C]) {
    Record<RK> e[NB];
    float v[NB][C];
#pragma unroll
    for (int u = 0; u < NB; ++u) e[u].load(rec + u * mgk_wide_record(RK) / 4);
#pragma unroll
    for (int u = 0; u < NB; ++u) {
        const char* row = p + (uint64_t)e[u].column() * row_bytes;
        asm("" : "+s"(row));   // stays a scalar base: the load then adds a 32-bit lane offset by itself
#pragma unroll
        for (int b = 0; b < C; ++b) v[u][b] = *reinterpret_cast<const float*>(row + col4[b]);
    }
#pragma unroll
    for (int u = 0; u < NB; ++u)
#pragma unroll
        for (int b = 0; b < C; ++b)
#pragma unroll
            for (int k = 0; k < RK; ++k) acc[b][k] = __builtin_fmaf(e[u].coef(k), v[u][b], acc[b][k]);
}

// Stage 1 of one row and C chunks of 64 columns from `chunk` on, four nonzeros at a time so that their loads of p are
// in flight together.
template <int RK, int R, int C>
__device__ __forceinline__ void wide_stage1(const MGK_CONSTANT u32x4* rec, int count, const float* p, int n2, int chunk, int lane, int r,
                                            uint32_t part) {
    float acc[C][RK];
#pragma unroll
    for (int b = 0; b < C; ++b)
#pragma unroll
        for (int k = 0; k < RK; ++k) acc[b][k] = 0.f;
    uint32_t col4[C];
#pragma unroll
    for (int b = 0; b < C; ++b) col4[b] = 4u * (uint32_t)min((chunk + b) * 64 + lane, n2 - 1);
    const char* base = reinterpret_cast<const char*>(p);
    const uint32_t row_bytes = 4u * (uint32_t)n2;
    for (; count >= 4; count -= 4, rec += mgk_wide_record(RK)) wide_products<RK, C, 4>(acc, rec, base, row_bytes, col4);
    if (count == 3) wide_products<RK, C, 3>(acc, rec, base, row_bytes, col4);
    else if (count == 2) wide_products<RK, C, 2>(acc, rec, base, row_bytes, col4);
    else if (count == 1) wide_products<RK, C, 1>(acc, rec, base, row_bytes, col4);
#pragma unroll
    for (int b = 0; b < C; ++b)
        if ((chunk + b) * 64 + lane < n2)
            t_write<RK>(part, mgk_wide_column(R, (uint32_t)((chunk + b) * 64 + lane)) ^ (uint32_t)(r * 16), acc[b]);
}

// Stage 2, one step of a group of 64 / R columns (lanes are columns by R rows): y += w (t0 + s (t1 + ...)) for the four
// nonzeros that the lanes of a quadruple hold between them; o, o2, o3: where their columns are in the arrays.
template <int RK, int U>
__device__ __forceinline__ void wide_read(float (&t)[RK], uint32_t o, uint32_t o2, uint32_t o3, uint32_t row16) {
    const f32x4 q = *shared<const f32x4>(quad_bcast<U>(o) ^ row16);
    t[0] = q.x; t[1] = q.y; t[2] = q.z; t[3] = q.w;
    if constexpr (RK >= 8) {
        const f32x4 v = *shared<const f32x4>(quad_bcast<U>(o2) ^ row16);
        t[4] = v.x; t[5] = v.y; t[6] = v.z; t[7] = v.w;
    }
    if constexpr (RK % 4 == 1) t[RK - 1] = *shared<const float>(quad_bcast<U>(o3) ^ (row16 >> 2));
    if constexpr (RK % 4 == 2) {
        const f32x2 v = *shared<const f32x2>(quad_bcast<U>(o3) ^ (row16 >> 1));
        t[RK - 2] = v.x; t[RK - 1] = v.y;
    }
}
template <int RK, int U>
__device__ __forceinline__ float wide_horner(float y, const float (&t)[RK], float s, float w) {
    float v = t[RK - 1];
#pragma unroll
    for (int k = RK - 2; k >= 0; --k) v = __builtin_fmaf(quad_bcast<U>(s), v, t[k]);
    // written out: the compiler spends a move on the broadcast.  The wait states a DPP read needs after a vector write are explicit.
    asm("s_nop 1\n\tv_fmac_f32_dpp %0, %1, %2 quad_perm:[%3,%3,%3,%3] row_mask:0xf bank_mask:0xf" : "+v"(y) : "v"(w), "v"(v), "n"(U));
    return y;
}
template <int RK>
__device__ __forceinline__ float wide_step(float y, uint32_t o, float s, float w, uint32_t part, uint32_t row16) {
    float t0[RK], t1[RK], t2[RK], t3[RK];
    const uint32_t o2 = o + part, o3 = (RK % 4 == 2 ? o >> 1 : o >> 2) + RK / 4 * part;
    wide_read<RK, 0>(t0, o, o2, o3, row16);
    wide_read<RK, 1>(t1, o, o2, o3, row16);
    if constexpr (RK < 8) {   // all four reads in flight; with more features two at a time, or more registers are spilled
        wide_read<RK, 2>(t2, o, o2, o3, row16);
        wide_read<RK, 3>(t3, o, o2, o3, row16);
    }
    y = wide_horner<RK, 0>(y, t0, s, w);
    y = wide_horner<RK, 1>(y, t1, s, w);
    if constexpr (RK >= 8) {
        wide_read<RK, 2>(t2, o, o2, o3, row16);
        wide_read<RK, 3>(t3, o, o2, o3, row16);
    }
    y = wide_horner<RK, 2>(y, t2, s, w);
    return wide_horner<RK, 3>(y, t3, s, w);
}
// All steps of a group; the words of the next step are in flight during this one (two sets in turn, no copies).  a: those
// of the first step.
struct Words {
    uint32_t o;
    float s, w;
    __device__ __forceinline__ void load(const float* step) {
        o = __float_as_uint(step[0]);
        s = step[64];
        w = step[128];
    }
};
template <int RK>
__device__ __forceinline__ float wide_stage2(float y, Words a, const float* step, int steps, uint32_t part, uint32_t row16) {
    Words b;
    for (; steps > 1; steps -= 2) {
        b.load(step + 192);
        y = wide_step<RK>(y, a.o, a.s, a.w, part, row16);
        step += 384;
        if (steps > 2) a.load(step);
        y = wide_step<RK>(y, b.o, b.s, b.w, part, row16);
    }
    if (steps == 1) y = wide_step<RK>(y, a.o, a.s, a.w, part, row16);
    return y;
}

// Workgroup b of a 1-D grid -> (pair, block of R rows).  Consecutive workgroups go to the eight XCDs in turn: each XCD
// takes an eighth of every pair's rows, adjacent ones, whose neighbours are few rows of p where the vertex order is a good one.
__device__ __forceinline__ void wide_block(int b, int blocks, int* pair, int* blk) {
    const int part = (blocks + 7) >> 3, slot = b >> 3;
    *pair = slot / part;
    *blk = (b & 7) * part + (slot - *pair * part);
}

template <int RK>
struct Features {
    static constexpr int value = RK;
};

// Sixteen wavefronts.  TWO: two workgroups share a CU and overlap each other's barriers and trips to memory, half as many results and
// registers (64) to a thread, which spills 1 to 10 of them with up to six features and 15, 24 and 35 with eight, nine and ten (still the shorter
// call than two passes, at the sizes that wide_layout takes them for); else T takes more than half of LDS (2048 columns, 4 rows and 5 features: all of it).  A wavefront of stage
// 1 takes C chunks of 64 columns of a row, so that rows of unlike degrees are divided evenly.  What the stages
// and the end read first is loaded ahead of the barrier in front of them.
template <int R, int HI, int LO, bool TWO>
__global__ __launch_bounds__(kThreads, TWO ? 8 : 4) void mgk_wide_xmv_kernel(MgkBatchDev X, MgkBatchDev Y, MgkWideFeatures F, MgkWideLayout L,
                                                                             const MgkWidePair* pairs, MgkPairState* state, float* vec, MgkParams prm,
                                                                             int n_pairs, int blocks, int it, int check_only) {
    extern __shared__ __align__(16) float lds[];
    constexpr int C = TWO ? 2 : 4, COLS = 64 / R, GROUPS = MGK_WIDE_MAX_ELEMENTS / kThreads / (TWO ? 2 : 1), AHEAD = 2;
    int pair, blk;
    wide_block(blockIdx.x, blocks, &pair, &blk);
    if (pair >= n_pairs) return;
    MgkPairState& st = state[pair];
    const int idle = check_only ? !st.check : st.done;
    const MGK_CONSTANT MgkWidePair* wp = (const MGK_CONSTANT MgkWidePair*)pairs + pair;
    const int n1 = wp->n1, n2 = wp->n2, nnz1 = wp->nnz1, cap = wp->cap2, voff1 = wp->voff1, voff2 = wp->voff2;
    const int64_t npad = wp->npad, f1 = wp->f1;
    const float* p = vec + wp->vec + 2 * npad;
    float* a = vec + wp->vec + 4 * npad;
    const float* inner = F.inner + wp->f2;
    const int i0 = blk * R;
    if (idle || i0 >= n1) return;
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    if (blk == 0 && tid == 0 && !check_only) {   // sums that the update of this iteration adds to
        st.rz[it & 1] = 0.f;
        st.rr[it & 1] = 0.f;
    }
    const int rows = min(R, n1 - i0);
    const MGK_CONSTANT int32_t* rowptr1 = (const MGK_CONSTANT int32_t*)(X.rowptr + voff1) + i0;
    const MGK_CONSTANT int32_t* first = (const MGK_CONSTANT int32_t*)inner;
    const int chunks = (n2 + 63) >> 6;
    const uint32_t part = (uint32_t)(R * 16 * n2), row16 = (uint32_t)(lane & (R - 1)) * 16u;
    // groups of columns come by descending degree: dealt back and forth
    auto place = [&](int c) { return (c * kWaves + (c & 1 ? kWaves - 1 - wave : wave)) * COLS; };
    const float* steps0 = inner + mgk_wide_head(n2) + 4 * (lane / R) + (lane & 3);
    float y[GROUPS];
    int col[GROUPS];   // of this lane's results
#pragma unroll
    for (int c = 0; c < GROUPS; ++c) {
        y[c] = 0.f;
        col[c] = 0;
    }
    auto pass = [&](auto rk, int q, bool last) {
        constexpr int RK = decltype(rk)::value, WORDS = mgk_wide_record(HI);
        const float* steps = steps0 + (int64_t)q * cap * 192;
        Words next;
        int f0 = 0, n = 0;
        const float* at = steps;
        auto start = [&](int c) {   // where a group's steps are, and the first of them
            const int pos = place(c);
            if (pos >= n2) return;
            f0 = first[pos >> 4];
            n = first[(pos >> 4) + 1] - f0;
            at = steps + (int64_t)f0 * 192 + 4 * (pos & 15);
            if (n > 0) next.load(at);
        };
        start(0);
        if (q > 0) __syncthreads();
        const MGK_CONSTANT u32x4* rec = (const MGK_CONSTANT u32x4*)(F.outer + ((int64_t)q * F.outer_total + f1) * WORDS);
        const int tasks = (chunks + C - 1) / C * R;
        for (int t = wave; t < tasks; t += kWaves) {
            const int r = (t + t / kWaves) % R;   // a wavefront meets all rows in turn
            if (r >= rows) continue;
            const int z0 = rowptr1[r], z1 = i0 + r + 1 < n1 ? rowptr1[r + 1] : nnz1;
            wide_stage1<RK, R, C>(rec + (int64_t)z0 * (WORDS / 4), z1 - z0, p, n2, t / R * C, lane, r, part);
        }
        __syncthreads();
#pragma unroll
        for (int c = 0; c < GROUPS; ++c) {
            if (place(c) >= n2) continue;
            const Words now = next;
            const int count = n;
            const float* step = at;
            if (c + 1 < GROUPS) start(c + 1);
            if (last) col[c] = F.deg_order2[voff2 + min(place(c) + lane / R, n2 - 1)];
            y[c] = wide_stage2<RK>(y[c], now, step, count, part, row16);
        }
    };
    pass(Features<HI>{}, 0, L.passes == 1);
    for (int q = 1; q < L.passes; ++q) pass(Features<LO>{}, q, q + 1 == L.passes);
    // ---- y in the order of the columns; a = M p - y and this workgroup's share of p^T a
    float pv[AHEAD], d2[AHEAD];
    int lab2[AHEAD];
    auto ahead = [&](int t, int k) {
        const int e = t / R * 64 + lane, r = t & (R - 1);
        if (r >= rows || e >= n2) return;
        pv[k] = p[(int64_t)(i0 + r) * n2 + e];
        d2[k] = Y.rowsum[voff2 + e];
        lab2[k] = Y.vlabel[voff2 + e];
    };
#pragma unroll
    for (int k = 0; k < AHEAD; ++k) ahead(wave + k * kWaves, k);
    __syncthreads();
    const int tp = n2 | 1;
#pragma unroll
    for (int c = 0; c < GROUPS; ++c)
        if (place(c) + lane / R < n2) lds[(lane & (R - 1)) * tp + col[c]] = y[c];
    __syncthreads();
    float s_pa = 0.f;
    for (int t0 = wave; t0 < chunks * R; t0 += kWaves * AHEAD) {
#pragma unroll
        for (int k = 0; k < AHEAD; ++k) {
            const int t = t0 + k * kWaves, r = t & (R - 1), e = t / R * 64 + lane;
            if (r < rows && e < n2) {
                const float d1 = ((const MGK_CONSTANT float*)X.rowsum)[voff1 + i0 + r] + prm.q;
                const float m = (((const MGK_CONSTANT int32_t*)X.vlabel)[voff1 + i0 + r] == lab2[k] ? d1 : d1 / prm.h) * (d2[k] + prm.q);
                const float av = __builtin_fmaf(m, pv[k], -lds[r * tp + e]);
                s_pa = __builtin_fmaf(pv[k], av, s_pa);
                a[(int64_t)(i0 + r) * n2 + e] = av;
            }
            ahead(t + kWaves * AHEAD, k);
        }
    }
    if (check_only) return;
    float* red = lds + R * tp;
    s_pa = wave_sum(s_pa);
    if (lane == 0) red[wave] = s_pa;
    __syncthreads();
    if (wave == 0) {
        s_pa = wave_sum(lane < kWaves ? red[lane] : 0.f);
        if (lane == 0) atomicAdd(&st.pa[it & 1], s_pa);
    }
}

template <int R, int HI, int LO, bool TWO>
hipError_t launch(const MgkBatchDev& X, const MgkBatchDev& Y, const MgkWideFeatures& F, const MgkWideLayout& L, const MgkWidePair* pairs,
                  MgkPairState* state, float* vec, const MgkParams& prm, int n_pairs, int max_n1, int max_n2, int it, bool check_only,
                  hipStream_t stream) {
    auto kern = mgk_wide_xmv_kernel<R, HI, LO, TWO>;
    static bool configured = false;
    if (!configured) {
        hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, MGK_LDS_LIMIT_BYTES);
        if (e != hipSuccess) return e;
        configured = true;
    }
    const int blocks = (max_n1 + R - 1) / R;
    hipLaunchKernelGGL(kern, dim3((unsigned)mgk_wide_grid(n_pairs, max_n1, R)), dim3(kThreads), (size_t)mgk_wide_lds_bytes(L, max_n2), stream, X, Y, F,
                       L, pairs, state, vec, prm, n_pairs, blocks, it, check_only ? 1 : 0);
    return hipGetLastError();
}

}  // namespace

// the graph index is a grid dimension of at most 65535: more graphs go in parts
hipError_t mgk_launch_wide_pack(const MgkBatchDev& B, const MgkWideBasis& S, const MgkWideLayout& L, const int32_t* deg_order,
                                const MgkSepGraph* outer_used, int n_outer, const MgkSepGraph* inner_used, int n_inner, int max_n, int64_t outer_total,
                                float* outer, float* inner, hipStream_t stream) {
    for (int g0 = 0; g0 < n_outer; g0 += 65535)
        hipLaunchKernelGGL(mgk_wide_outer_kernel, dim3((max_n + 63) / 64, n_outer - g0 < 65535 ? n_outer - g0 : 65535), dim3(256), 0, stream, B, S, L,
                           outer_used + g0, outer_total, outer);
    for (int g0 = 0; g0 < n_inner; g0 += 65535)
        hipLaunchKernelGGL(mgk_wide_inner_kernel, dim3((max_n + 63) / 64, n_inner - g0 < 65535 ? n_inner - g0 : 65535), dim3(256), 0, stream, B, S, L,
                           deg_order, inner_used + g0, inner);
    return hipGetLastError();
}

hipError_t mgk_launch_wide_xmv(const MgkBatchDev& X, const MgkBatchDev& Y, const MgkWideFeatures& F, const MgkWideLayout& L, const MgkWidePair* pairs,
                               MgkPairState* state, float* vec, const MgkParams& prm, int n_pairs, int max_n1, int max_n2, int it, bool check_only,
                               hipStream_t stream) {
    if (L.rows <= 0 || max_n2 > MGK_WIDE_MAX_ELEMENTS / L.rows || mgk_wide_lds_bytes(L, max_n2) > MGK_LDS_LIMIT_BYTES) return hipErrorInvalidValue;
    const bool two = mgk_wide_two(L, max_n2);
#define MGK_WIDE_GO(R, H, O, T) \
    if (L.rows == R && L.hi == H && L.lo == O && two == T) \
        return launch<R, H, O, T>(X, Y, F, L, pairs, state, vec, prm, n_pairs, max_n1, max_n2, it, check_only, stream);
    MGK_WIDE_GO(4, 4, 4, false) MGK_WIDE_GO(4, 4, 5, false) MGK_WIDE_GO(4, 5, 5, false) MGK_WIDE_GO(4, 6, 6, false)
    MGK_WIDE_GO(4, 4, 4, true) MGK_WIDE_GO(4, 4, 5, true) MGK_WIDE_GO(4, 5, 5, true) MGK_WIDE_GO(4, 6, 6, true)
    MGK_WIDE_GO(8, 4, 4, true) MGK_WIDE_GO(8, 4, 5, true) MGK_WIDE_GO(8, 5, 5, true) MGK_WIDE_GO(8, 6, 6, true)
    MGK_WIDE_GO(8, 8, 8, true) MGK_WIDE_GO(8, 9, 9, true) MGK_WIDE_GO(8, 10, 10, true)
#undef MGK_WIDE_GO
    return hipErrorInvalidValue;
}

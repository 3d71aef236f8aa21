// Host-callable launchers of the HIP kernels (defined in the .hip files).
#ifndef MGK_LAUNCH_H
#define MGK_LAUNCH_H

#include <hip/hip_runtime_api.h>
#include <stddef.h>
#include <stdint.h>

#include "mgk_internal.h"

// On-chip solver: one workgroup of `waves` wavefronts per job, each thread
// owning up to `ept` vector elements (waves * 64 * ept >= n n' of every job),
// `lds_bytes` of dynamic LDS (the largest MgkSmallPlan::total of the jobs).
// atomic_rows: some inner graph of the jobs has a row of more than 16 nonzeros.
// One definition per workgroup size, each in its own translation unit.
#define MGK_DECL_SMALL(W)                                                                         \
    hipError_t mgk_launch_small_w##W(int ept, bool weighted, bool atomic_rows, const MgkBatchDev& X, \
                                     const MgkBatchDev& Y, const MgkJob* jobs_dev, int n_jobs,    \
                                     const MgkParams& prm, size_t lds_bytes,                      \
                                     const MgkOutputs& out, hipStream_t stream);
MGK_DECL_SMALL(1)
MGK_DECL_SMALL(2)
MGK_DECL_SMALL(4)
MGK_DECL_SMALL(8)
MGK_DECL_SMALL(16)
#undef MGK_DECL_SMALL
// four wavefronts with 6, 10 or 14 elements per thread (a translation unit of its own)
hipError_t mgk_launch_small_w4_fine(int ept, bool weighted, bool atomic_rows, const MgkBatchDev& X,
                                    const MgkBatchDev& Y, const MgkJob* jobs_dev, int n_jobs,
                                    const MgkParams& prm, size_t lds_bytes, const MgkOutputs& out,
                                    hipStream_t stream);

static inline hipError_t mgk_launch_small(int waves, int ept, bool weighted, bool atomic_rows, const MgkBatchDev& X,
                                          const MgkBatchDev& Y, const MgkJob* jobs_dev, int n_jobs,
                                          const MgkParams& prm, size_t lds_bytes,
                                          const MgkOutputs& out, hipStream_t stream) {
    switch (waves) {
        case 1: return mgk_launch_small_w1(ept, weighted, atomic_rows, X, Y, jobs_dev, n_jobs, prm, lds_bytes, out, stream);
        case 2: return mgk_launch_small_w2(ept, weighted, atomic_rows, X, Y, jobs_dev, n_jobs, prm, lds_bytes, out, stream);
        case 4:
            if (ept == 6 || ept == 10 || ept == 14)
                return mgk_launch_small_w4_fine(ept, weighted, atomic_rows, X, Y, jobs_dev, n_jobs, prm, lds_bytes, out, stream);
            return mgk_launch_small_w4(ept, weighted, atomic_rows, X, Y, jobs_dev, n_jobs, prm, lds_bytes, out, stream);
        case 8: return mgk_launch_small_w8(ept, weighted, atomic_rows, X, Y, jobs_dev, n_jobs, prm, lds_bytes, out, stream);
        case 16: return mgk_launch_small_w16(ept, weighted, atomic_rows, X, Y, jobs_dev, n_jobs, prm, lds_bytes, out, stream);
        default: return hipErrorInvalidValue;
    }
}

// Register-resident on-chip solver (mgk_regs.hip): `waves` (4 or 8) wavefronts
// per job, `chunks` 64-lane chunks of the inner graph, ept * waves * 64 >= n n'
// of every job, `lds_bytes` the largest MgkRegsPlan::total of the jobs.  One
// definition per (waves, chunks), each in its own translation unit.
#define MGK_DECL_REGS(W, C)                                                                       \
    hipError_t mgk_launch_regs_w##W##_c##C(int ept, bool weighted, const MgkBatchDev& X,          \
                                           const MgkBatchDev& Y, const MgkJob* jobs_dev,          \
                                           int n_jobs, const MgkParams& prm, size_t lds_bytes,    \
                                           const MgkOutputs& out, hipStream_t stream);
MGK_DECL_REGS(4, 1)
MGK_DECL_REGS(4, 2)
MGK_DECL_REGS(8, 1)
MGK_DECL_REGS(8, 2)
#undef MGK_DECL_REGS

static inline hipError_t mgk_launch_regs(int waves, int chunks, int ept, bool weighted,
                                         const MgkBatchDev& X, const MgkBatchDev& Y,
                                         const MgkJob* jobs_dev, int n_jobs, const MgkParams& prm,
                                         size_t lds_bytes, const MgkOutputs& out, hipStream_t stream) {
    switch (waves * 10 + chunks) {
        case 41: return mgk_launch_regs_w4_c1(ept, weighted, X, Y, jobs_dev, n_jobs, prm, lds_bytes, out, stream);
        case 42: return mgk_launch_regs_w4_c2(ept, weighted, X, Y, jobs_dev, n_jobs, prm, lds_bytes, out, stream);
        case 81: return mgk_launch_regs_w8_c1(ept, weighted, X, Y, jobs_dev, n_jobs, prm, lds_bytes, out, stream);
        case 82: return mgk_launch_regs_w8_c2(ept, weighted, X, Y, jobs_dev, n_jobs, prm, lds_bytes, out, stream);
        default: return hipErrorInvalidValue;
    }
}

// Register-resident solver of the reduced system (mgk_reduced.hip): 2 (one chunk only), 4 or 8 wavefronts
// per job, ept * waves * 64 >= n_red n' of every job; jobs of both orientations (MGK_OUT1_SWAPPED: outer
// graph from Y).  Weak: without these kernels the full system is solved.
#define MGK_DECL_REDUCED(W, C)                                                                       \
    __attribute__((weak)) hipError_t mgk_launch_reduced_w##W##_c##C(int ept, bool weighted, const MgkBatchDev& X, \
                                           const MgkBatchDev& Y, const MgkJob* jobs_dev,          \
                                           int n_jobs, const MgkParams& prm, size_t lds_bytes,    \
                                           const MgkOutputs& out, hipStream_t stream);
MGK_DECL_REDUCED(2, 1)
MGK_DECL_REDUCED(4, 1)
MGK_DECL_REDUCED(4, 2)
MGK_DECL_REDUCED(8, 1)
MGK_DECL_REDUCED(8, 2)
#undef MGK_DECL_REDUCED

static inline hipError_t mgk_launch_reduced(int waves, int chunks, int ept, bool weighted,
                                            const MgkBatchDev& X, const MgkBatchDev& Y,
                                            const MgkJob* jobs_dev, int n_jobs, const MgkParams& prm,
                                            size_t lds_bytes, const MgkOutputs& out, hipStream_t stream) {
    switch (waves * 10 + chunks) {
        case 21: return mgk_launch_reduced_w2_c1(ept, weighted, X, Y, jobs_dev, n_jobs, prm, lds_bytes, out, stream);
        case 41: return mgk_launch_reduced_w4_c1(ept, weighted, X, Y, jobs_dev, n_jobs, prm, lds_bytes, out, stream);
        case 42: return mgk_launch_reduced_w4_c2(ept, weighted, X, Y, jobs_dev, n_jobs, prm, lds_bytes, out, stream);
        case 81: return mgk_launch_reduced_w8_c1(ept, weighted, X, Y, jobs_dev, n_jobs, prm, lds_bytes, out, stream);
        case 82: return mgk_launch_reduced_w8_c2(ept, weighted, X, Y, jobs_dev, n_jobs, prm, lds_bytes, out, stream);
        default: return hipErrorInvalidValue;
    }
}

// Owner-computes on-chip solver (mgk_sell.hip): `waves` (4, 8 or 16) wavefronts per job,
// `ept` vector slots per lane (2 waves ept >= tiles of every job), `regs` entry registers
// per lane (>= what mgk_sell_need returns for every job), `lds_bytes` the largest
// MgkSellPlan::total of the jobs.  Launch shapes (waves, ept, regs); one translation unit
// per workgroup size.
#define MGK_SELL_SHAPES_W4(F) F(4, 4, 32) F(4, 6, 40) F(4, 8, 48)
#define MGK_SELL_SHAPES_W8(F) F(8, 2, 16) F(8, 3, 24) F(8, 4, 32) F(8, 5, 36)
#define MGK_SELL_SHAPES_W16(F) F(16, 3, 24) F(16, 4, 28)
struct MgkSellShape { int waves, ept, regs; };
static const MgkSellShape kMgkSellShapes[] = {
#define MGK_SELL_ROW(W, E, R) {W, E, R},
    MGK_SELL_SHAPES_W4(MGK_SELL_ROW) MGK_SELL_SHAPES_W8(MGK_SELL_ROW) MGK_SELL_SHAPES_W16(MGK_SELL_ROW)
#undef MGK_SELL_ROW
};
#define MGK_DECL_SELL(W)                                                                             \
    hipError_t mgk_launch_sell_w##W(int ept, int regs, const MgkBatchDev& X, const MgkBatchDev& Y,    \
                                    const MgkJob* jobs_dev, int n_jobs, const MgkParams& prm,         \
                                    size_t lds_bytes, const MgkOutputs& out, hipStream_t stream);
MGK_DECL_SELL(4)
MGK_DECL_SELL(8)
MGK_DECL_SELL(16)
#undef MGK_DECL_SELL
static inline hipError_t mgk_launch_sell(int waves, int ept, int regs, const MgkBatchDev& X, const MgkBatchDev& Y,
                                         const MgkJob* jobs_dev, int n_jobs, const MgkParams& prm,
                                         size_t lds_bytes, const MgkOutputs& out, hipStream_t stream) {
    switch (waves) {
        case 4: return mgk_launch_sell_w4(ept, regs, X, Y, jobs_dev, n_jobs, prm, lds_bytes, out, stream);
        case 8: return mgk_launch_sell_w8(ept, regs, X, Y, jobs_dev, n_jobs, prm, lds_bytes, out, stream);
        case 16: return mgk_launch_sell_w16(ept, regs, X, Y, jobs_dev, n_jobs, prm, lds_bytes, out, stream);
        default: return hipErrorInvalidValue;
    }
}

// Fixed job-list array in device memory for the entry point that allocates nothing
// (mgk_noalloc.hip): its device address on `device` and how many jobs it holds.
#define MGK_NOALLOC_MAX_PAIRS 65536
hipError_t mgk_noalloc_job_storage(int device, MgkJob** jobs, int64_t* capacity);

// ---- solver with vectors in global memory (mgk_large.hip) --------------------
// Expand every octile of batch B into the outer (CSR order) and inner (lane
// layout) entry lists; `outer` holds B.nnz_total entries, `inner` B.lanes_total.
hipError_t mgk_launch_expand(const MgkBatchDev& B, const MgkParams& prm, MgkEntry* outer, MgkEntry* inner,
                             hipStream_t stream);
// Expand every octile of B to dense 8x8 blocks (64 * B.n_tiles_total floats per array).
hipError_t mgk_launch_expand_dense(const MgkBatchDev& B, const MgkParams& prm, float* dw, float* de,
                                   float* dlw, hipStream_t stream);
// Set-up of Alg. 1 for n_pairs pairs (state must be zero-filled before).  lean: for the separable product, M is not kept.
hipError_t mgk_launch_large_init(const MgkBatchDev& X, const MgkBatchDev& Y, const MgkLargePair* pairs,
                                 MgkPairState* state, float* vec, const MgkParams& prm, bool lean, int n_pairs,
                                 int vec_blocks, hipStream_t stream);
// Iteration `it` (0, 1, ...) of Alg. 1 for all pairs that have not stopped: the product, then
// three kernels over the vectors that also do the scalar steps and the stop test.  n_active[0]
// is decremented for every pair that stops, n_active[1] raised to the number of iterations
// it took.  DX/DY non-null: dense tile-pair XMV
// (xmv_blocks = workgroups of 4 output blocks); else the sparse XMV on the
// expanded lists: with rows_threads > 0 the one that stages rows of p in
// rows_lds_bytes of LDS (xmv_blocks = outer rows, one workgroup of rows_threads
// each; every row of p must fit; rows_chunks = 1, 2 or 4 chunks of the inner layout
// per pass of a wavefront), with rows_threads == 0 the one that gathers p from global
// memory.
hipError_t mgk_launch_large_iteration(const MgkBatchDev& X, const MgkBatchDev& Y, const MgkExpanded& EX,
                                      const MgkExpanded& EY, const MgkLargePair* pairs,
                                      MgkPairState* state, float* vec, const MgkParams& prm,
                                      bool weighted, int n_pairs, int xmv_blocks, int vec_blocks,
                                      int* n_active, int it, const MgkDenseTiles* DX,
                                      const MgkDenseTiles* DY, int rows_threads, int rows_lds_bytes,
                                      int rows_chunks, hipStream_t stream);
// K = p_x^T x, the nodal solution, a check of the true residual for pairs whose solution grew
// far beyond the Jacobi guess (one more product, arguments as for an iteration), and the
// per-pair outputs.
hipError_t mgk_launch_large_final(const MgkBatchDev& X, const MgkBatchDev& Y, const MgkExpanded& EX,
                                  const MgkExpanded& EY, const MgkLargePair* pairs, MgkPairState* state,
                                  float* vec, const MgkParams& prm, bool weighted, int n_pairs, int xmv_blocks,
                                  int vec_blocks, const MgkDenseTiles* DX, const MgkDenseTiles* DY,
                                  int rows_threads, int rows_lds_bytes, int rows_chunks, const MgkOutputs& out,
                                  hipStream_t stream);
// ---- separable product (mgk_sep.hip) ------------------------------------------
// Weak, so that the host code links without the kernels (host-only contexts never get here; elsewhere the
// call fails).
#define MGK_KERNELS_OPTIONAL __attribute__((weak))
// Packets (layout L; gptr and total of that packet size) and dense F_k of the n_used graphs of B listed
// at `used` (memory the device can read; list.whole for all of them), the largest of max_n vertices.
MGK_KERNELS_OPTIONAL hipError_t mgk_launch_sep_pack(const MgkBatchDev& B, const MgkSepBasis& S, const MgkSepLayout& L,
                                                    const MgkSepList& list, const MgkSepGraph* used, int n_used, int max_n,
                                                    float* packets, hipStream_t stream);
MGK_KERNELS_OPTIONAL hipError_t mgk_launch_sep_dense_pack(const MgkBatchDev& B, const MgkSepBasis& S, const MgkSepGraph* used,
                                                          int n_used, int max_n, float* F, hipStream_t stream);
// y = XMV(p) and p^T a of iteration `it` for every pair that still iterates (check_only: y alone, for
// the pairs marked by mgk_launch_large_outputs).  max_n1, max_n2: largest outer and inner graph.
MGK_KERNELS_OPTIONAL hipError_t mgk_launch_sep_xmv(const MgkBatchDev& X, const MgkBatchDev& Y, const MgkSepList& SX, const MgkSepList& SY,
                                                   const MgkSepLayout& L, const MgkLargePair* pairs, const MgkSepAt* feat, MgkPairState* state,
                                                   float* vec, const MgkParams& prm, int n_pairs, int max_n1, int max_n2, int it,
                                                   bool check_only, hipStream_t stream);
// parts: operands in three 16-bit parts, for graphs that mgk_sep_in_parts allows
MGK_KERNELS_OPTIONAL hipError_t mgk_launch_sep_dense(const MgkBatchDev& X, const MgkBatchDev& Y, const MgkSepList& SX, const MgkSepList& SY,
                                                     int rank, bool parts, const MgkLargePair* pairs, const MgkSepAt* feat, MgkPairState* state,
                                                     float* vec, const MgkParams& prm, int n_pairs, int max_n1, int max_n2, int it,
                                                     bool check_only, hipStream_t stream);
// The same for sparse graphs of many vertices (mgk_sep_wide.hip): features of the graphs listed (memory the device can read;
// MgkSepGraph::at a record or a word) as outer and as inner ones, and the product.
MGK_KERNELS_OPTIONAL hipError_t mgk_launch_wide_pack(const MgkBatchDev& B, const MgkWideBasis& S, const MgkWideLayout& L, const int32_t* deg_order,
                                                     const MgkSepGraph* outer_used, int n_outer, const MgkSepGraph* inner_used, int n_inner,
                                                     int max_n, int64_t outer_total, float* outer, float* inner, hipStream_t stream);
MGK_KERNELS_OPTIONAL hipError_t mgk_launch_wide_xmv(const MgkBatchDev& X, const MgkBatchDev& Y, const MgkWideFeatures& F, const MgkWideLayout& L,
                                                    const MgkWidePair* pairs, MgkPairState* state, float* vec, const MgkParams& prm, int n_pairs,
                                                    int max_n1, int max_n2, int it, bool check_only, hipStream_t stream);
// Whole solves on chip with that product (mgk_pcg_sep.hip) by `waves` wavefronts of ept elements a thread, T of rb
// blocks of 16 rows at a time; packets (layout with slab_bytes 1) of all graphs of the two batches.
#define MGK_DECL_PCG_SEP(RK)                                                                                                       \
    MGK_KERNELS_OPTIONAL hipError_t mgk_launch_pcg_sep_rk##RK(int waves, int ept, int passes, const MgkBatchDev& X, const MgkBatchDev& Y, \
                                                              const MgkSepList& SX, const MgkSepList& SY, const MgkJob* jobs_dev,   \
                                                              int n_jobs, const MgkParams& prm, int rb, size_t lds_bytes,           \
                                                              const MgkOutputs& out, hipStream_t stream);
MGK_DECL_PCG_SEP(1)
MGK_DECL_PCG_SEP(4)
MGK_DECL_PCG_SEP(5)
MGK_DECL_PCG_SEP(6)
MGK_DECL_PCG_SEP(7)
#undef MGK_DECL_PCG_SEP
static inline hipError_t mgk_launch_pcg_sep(int rk, int waves, int ept, int passes, const MgkBatchDev& X, const MgkBatchDev& Y,
                                            const MgkSepList& SX, const MgkSepList& SY, const MgkJob* jobs_dev, int n_jobs,
                                            const MgkParams& prm, int rb, size_t lds_bytes, const MgkOutputs& out, hipStream_t stream) {
    switch (rk) {
        case 1: return mgk_launch_pcg_sep_rk1(waves, ept, passes, X, Y, SX, SY, jobs_dev, n_jobs, prm, rb, lds_bytes, out, stream);
        case 4: return mgk_launch_pcg_sep_rk4(waves, ept, passes, X, Y, SX, SY, jobs_dev, n_jobs, prm, rb, lds_bytes, out, stream);
        case 5: return mgk_launch_pcg_sep_rk5(waves, ept, passes, X, Y, SX, SY, jobs_dev, n_jobs, prm, rb, lds_bytes, out, stream);
        case 6: return mgk_launch_pcg_sep_rk6(waves, ept, passes, X, Y, SX, SY, jobs_dev, n_jobs, prm, rb, lds_bytes, out, stream);
        case 7: return mgk_launch_pcg_sep_rk7(waves, ept, passes, X, Y, SX, SY, jobs_dev, n_jobs, prm, rb, lds_bytes, out, stream);
        default: return hipErrorInvalidValue;
    }
}
// The two kernels over the vectors that follow a product which has already formed p^T a and
// overwrites y.
MGK_KERNELS_OPTIONAL hipError_t mgk_launch_large_vectors(const MgkLargePair* pairs, MgkPairState* state, float* vec, int n_pairs,
                                                         int vec_blocks, int it, float rtol2, int* n_active, hipStream_t stream);
// part 0: K, nodal solution and growth of every pair as it stands; pairs that have stopped and
// grew far beyond the Jacobi guess are marked for a check (p = x) -- then a product with
// check_only -- part 1: their true residual, and the per-pair outputs.  Pairs still iterating are
// left as they are.
MGK_KERNELS_OPTIONAL hipError_t mgk_launch_large_outputs(const MgkBatchDev& X, const MgkBatchDev& Y, const MgkLargePair* pairs,
                                                         MgkPairState* state, float* vec, const MgkParams& prm, int n_pairs,
                                                         int vec_blocks, const MgkOutputs& out, int part, hipStream_t stream);
// In-place normalisation K[i][j] /= sqrt(K[i][i] K[j][j]) of an n x n matrix; diag holds n floats.
hipError_t mgk_launch_normalize(float* K, float* diag, int n, hipStream_t stream);

#endif

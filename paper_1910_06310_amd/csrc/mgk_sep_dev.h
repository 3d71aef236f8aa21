// Device code of the kernel that applies the off-diagonal product through a separable edge
// kernel in its sparse form (mgk_sep.hip).
//
// On the labels of a batch the square-exponential (and the constant) edge kernel is a short
// sum of products, kappa_e(e, e') = sum_k phi_k(e) phi_k(e') to fp32 rounding (the host builds
// phi and checks the error), so the off-diagonal operator of a pair is
//     y = sum_k F_k P F'_k^T,   F_k = A (.) phi_k(E),
// two one-sided sparse products per k: nnz n' + n nnz' multiply-adds per k instead of nnz nnz'
// evaluations of kappa_e.
#ifndef MGK_SEP_DEV_H
#define MGK_SEP_DEV_H

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "mgk_internal.h"

namespace {

// Value SLOT of the 16 that lanes 0..15 of every row of 16 lanes hold, in all lanes of the row.
template <int SLOT>
__device__ __forceinline__ uint32_t bcast16(float c) {
    return (uint32_t)__builtin_amdgcn_update_dpp(0, __float_as_int(c), 0x150 + SLOT, 0xf, 0xf, true);
}

// acc[k] += c[SLOT + k] * t[k] for k < RK, c broadcast inside rows of 16 lanes: the coefficient
// is selected by the DPP control of the multiply-add itself, so a product costs one
// instruction and no separate broadcast.  The wait states a DPP read needs after a vector
// write of its operand are spelled out (c normally comes straight from a load).
template <int RK, int SLOT>
__device__ __forceinline__ void fmac_each(float (&acc)[RK], float c, const float (&t)[RK]) {
#define MGK_F(K) "v_fmac_f32_dpp %" #K ", %[c], %[t" #K "] row_newbcast:%[s" #K "] row_mask:0xf bank_mask:0xf\n\t"
    if constexpr (RK == 1)
        asm("s_nop 1\n\t" MGK_F(0) : "+v"(acc[0]) : [c] "v"(c), [t0] "v"(t[0]), [s0] "n"(SLOT));
    if constexpr (RK == 4)
        asm("s_nop 1\n\t" MGK_F(0) MGK_F(1) MGK_F(2) MGK_F(3)
            : "+v"(acc[0]), "+v"(acc[1]), "+v"(acc[2]), "+v"(acc[3])
            : [c] "v"(c), [t0] "v"(t[0]), [t1] "v"(t[1]), [t2] "v"(t[2]), [t3] "v"(t[3]),
              [s0] "n"(SLOT), [s1] "n"(SLOT + 1), [s2] "n"(SLOT + 2), [s3] "n"(SLOT + 3));
    if constexpr (RK == 5)
        asm("s_nop 1\n\t" MGK_F(0) MGK_F(1) MGK_F(2) MGK_F(3) MGK_F(4)
            : "+v"(acc[0]), "+v"(acc[1]), "+v"(acc[2]), "+v"(acc[3]), "+v"(acc[4])
            : [c] "v"(c), [t0] "v"(t[0]), [t1] "v"(t[1]), [t2] "v"(t[2]), [t3] "v"(t[3]), [t4] "v"(t[4]),
              [s0] "n"(SLOT), [s1] "n"(SLOT + 1), [s2] "n"(SLOT + 2), [s3] "n"(SLOT + 3), [s4] "n"(SLOT + 4));
    if constexpr (RK == 6)
        asm("s_nop 1\n\t" MGK_F(0) MGK_F(1) MGK_F(2) MGK_F(3) MGK_F(4) MGK_F(5)
            : "+v"(acc[0]), "+v"(acc[1]), "+v"(acc[2]), "+v"(acc[3]), "+v"(acc[4]), "+v"(acc[5])
            : [c] "v"(c), [t0] "v"(t[0]), [t1] "v"(t[1]), [t2] "v"(t[2]), [t3] "v"(t[3]), [t4] "v"(t[4]), [t5] "v"(t[5]),
              [s0] "n"(SLOT), [s1] "n"(SLOT + 1), [s2] "n"(SLOT + 2), [s3] "n"(SLOT + 3), [s4] "n"(SLOT + 4), [s5] "n"(SLOT + 5));
    if constexpr (RK == 7)
        asm("s_nop 1\n\t" MGK_F(0) MGK_F(1) MGK_F(2) MGK_F(3) MGK_F(4) MGK_F(5) MGK_F(6)
            : "+v"(acc[0]), "+v"(acc[1]), "+v"(acc[2]), "+v"(acc[3]), "+v"(acc[4]), "+v"(acc[5]), "+v"(acc[6])
            : [c] "v"(c), [t0] "v"(t[0]), [t1] "v"(t[1]), [t2] "v"(t[2]), [t3] "v"(t[3]), [t4] "v"(t[4]), [t5] "v"(t[5]), [t6] "v"(t[6]),
              [s0] "n"(SLOT), [s1] "n"(SLOT + 1), [s2] "n"(SLOT + 2), [s3] "n"(SLOT + 3), [s4] "n"(SLOT + 4), [s5] "n"(SLOT + 5), [s6] "n"(SLOT + 6));
#undef MGK_F
}

// One outer (or inner) nonzero against one value of p per lane: acc[k] += c[SLOT + k] * p.
template <int RK, int SLOT>
__device__ __forceinline__ void fmac_same(float (&acc)[RK], float c, float p) {
    float t[RK];
#pragma unroll
    for (int k = 0; k < RK; ++k) t[k] = p;
    fmac_each<RK, SLOT>(acc, c, t);
}

// ---- T of 16 outer rows in LDS: [column j'][quad of k][row][4 values of k], slabs of
// MGK_SEP_SLAB words per column.  Reads of stage 2 are 16 lanes side by side; the 4 words of
// padding per slab spread the writes of stage 1, whose lanes are columns, over all banks.
template <int RK>
__device__ __forceinline__ void slab_read(float (&t)[RK], const char* lds, uint32_t addr) {
    if constexpr (RK == 1) {
        t[0] = *reinterpret_cast<const float*>(lds + addr);
    } else {
        const float4 a = *reinterpret_cast<const float4*>(lds + addr);
        t[0] = a.x; t[1] = a.y; t[2] = a.z; t[3] = a.w;
        if constexpr (RK == 5) t[4] = *reinterpret_cast<const float*>(lds + addr + 256);
        if constexpr (RK == 6) {
            const float2 b = *reinterpret_cast<const float2*>(lds + addr + 256);
            t[4] = b.x; t[5] = b.y;
        }
        if constexpr (RK == 7) {
            const float4 b = *reinterpret_cast<const float4*>(lds + addr + 256);
            t[4] = b.x; t[5] = b.y; t[6] = b.z;
        }
    }
}
template <int RK>
__device__ __forceinline__ void slab_write(char* lds, uint32_t addr, const float (&t)[RK]) {
    if constexpr (RK == 1) {
        *reinterpret_cast<float*>(lds + addr) = t[0];
    } else {
        *reinterpret_cast<float4*>(lds + addr) = make_float4(t[0], t[1], t[2], t[3]);
        if constexpr (RK == 5) *reinterpret_cast<float*>(lds + addr + 256) = t[4];
        if constexpr (RK == 6) *reinterpret_cast<float2*>(lds + addr + 256) = make_float2(t[4], t[5]);
        if constexpr (RK == 7) *reinterpret_cast<float4*>(lds + addr + 256) = make_float4(t[4], t[5], t[6], 0.f);
    }
}

// Multiply-adds of the G nonzeros of a packet in stage 1: pv[u] is this lane's value of p for
// nonzero u.
template <int RK, int G, int U = 0>
__device__ __forceinline__ void packet_same(float (&acc)[RK], float c, const float* pv) {
    if constexpr (U < G) {
        fmac_same<RK, U * (RK + 1)>(acc, c, pv[U]);
        packet_same<RK, G, U + 1>(acc, c, pv);
    }
}
// Byte offsets (slab of the column the nonzero points at) carried by a packet.
template <int RK, int G, int U = 0>
__device__ __forceinline__ void packet_slabs(uint32_t (&a)[G], float c) {
    if constexpr (U < G) {
        a[U] = bcast16<U * (RK + 1) + RK>(c);
        packet_slabs<RK, G, U + 1>(a, c);
    }
}
template <int RK, int G, int U = 0>
__device__ __forceinline__ void packet_lane(uint32_t* a, float c) {   // the same, wave-uniform
    if constexpr (U < G) {
        a[U] = (uint32_t)__builtin_amdgcn_readlane(__float_as_int(c), U * (RK + 1) + RK);
        packet_lane<RK, G, U + 1>(a, c);
    }
}
template <int RK, int G, int U = 0>
__device__ __forceinline__ void packet_each(float (&acc)[RK], float c, const float (&t)[G][RK]) {
    if constexpr (U < G) {
        fmac_each<RK, U * (RK + 1)>(acc, c, t[U]);
        packet_each<RK, G, U + 1>(acc, c, t);
    }
}

// ---- where stage 1 reads p: rows of n' floats in global memory --------------------------------
// row(j): start of row j, wave-uniform; at(row, col4): the element 4-byte offset col4 into it.
struct PGlobal {
    typedef const char* Row;
    const char* base;
    uint32_t row_bytes;
    __device__ __forceinline__ Row row(uint32_t j) const {
        Row r = base + (uint64_t)j * row_bytes;
        asm("" : "+s"(r));   // stays a scalar base: the load then adds a 32-bit lane offset by itself
        return r;
    }
    static __device__ __forceinline__ float at(Row r, uint32_t col4) { return *reinterpret_cast<const float*>(r + col4); }
};

// One chunk of 64 columns of stage 1: the multiply-adds of NB packets with the values pv.
template <int RK, int G, int NB>
__device__ __forceinline__ void stage1_chunk(const float (&c)[NB], const float (&pv)[NB * G], int col, int n2, char* slabs,
                                             uint32_t row_slot, bool first) {
    float acc[RK];
    const uint32_t at = (uint32_t)col * (MGK_SEP_SLAB(RK) * 4) + row_slot;
#pragma unroll
    for (int k = 0; k < RK; ++k) acc[k] = 0.f;
    if (!first && col < n2) slab_read<RK>(acc, slabs, at);
#pragma unroll
    for (int a = 0; a < NB; ++a) packet_same<RK, G>(acc, c[a], pv + a * G);
    if (col < n2) slab_write<RK>(slabs, at, acc);
}

// Stage 1 for NB packets of one outer row (all its columns, 64 at a time): T[row] (+)= the
// products.  c[] and the row addresses stay in registers over the columns; the values of p of
// the next 64 columns are in flight during the multiply-adds of these.  `first`: T is
// written, else added to (rows of more than 16 nonzeros come in several batches).
template <int RK, int G, int NB, class P>
__device__ __forceinline__ void stage1_batch(const float* pk, int left, const P& p, int n2, int lane, char* slabs,
                                             uint32_t row_slot, bool first) {
    constexpr int SLAB = MGK_SEP_SLAB(RK), Z = NB * G;
    constexpr uint32_t MAGIC = (uint32_t)(((1ull << 32) + SLAB * 4 - 1) / (SLAB * 4));   // x / (4 SLAB) for its multiples
    float c[NB];
    typename P::Row row[Z];
#pragma unroll
    for (int a = 0; a < NB; ++a) c[a] = pk[(a < left ? a : 0) * 64];
#pragma unroll
    for (int a = 0; a < NB; ++a) {
        uint32_t sl[G];
        packet_lane<RK, G>(sl, c[a]);
#pragma unroll
        for (int u = 0; u < G; ++u) row[a * G + u] = p.row(__umulhi(sl[u], MAGIC));
        if (a >= left) c[a] = 0.f;   // wave-uniform; only the last one of an odd count
    }
    float pa[Z], pb[Z];
    const uint32_t last4 = (uint32_t)(n2 - 1) * 4u;
    auto load = [&](float (&v)[Z], int ch) {
        const uint32_t col4 = min((uint32_t)(ch + lane) * 4u, last4);
#pragma unroll
        for (int z = 0; z < Z; ++z) v[z] = P::at(row[z], col4);
    };
    load(pa, 0);
    for (int ch = 0; ch < n2; ch += 128) {   // two buffers in turn, no copies
        if (ch + 64 < n2) load(pb, ch + 64);
        stage1_chunk<RK, G, NB>(c, pa, ch + lane, n2, slabs, row_slot, first);
        if (ch + 64 < n2) {
            if (ch + 128 < n2) load(pa, ch + 128);
            stage1_chunk<RK, G, NB>(c, pb, ch + 64 + lane, n2, slabs, row_slot, first);
        }
    }
}

// Stage 1 of one outer row: its packets are at pk, one per 64 words.
template <int RK, int G, class P>
__device__ __forceinline__ void stage1_row(const float* pk, int steps, const P& p, int n2, int lane,
                                           char* slabs, uint32_t row_slot) {
    constexpr int NB = G >= 8 ? 2 : 8;
    bool first = true;
    int b = 0;
    for (; b + NB <= steps; b += NB) {
        stage1_batch<RK, G, NB, P>(pk + b * 64, NB, p, n2, lane, slabs, row_slot, first);
        first = false;
    }
    const int left = steps - b;
    pk += b * 64;
    if constexpr (G < 8) {
        if (left > 6) stage1_batch<RK, G, 8, P>(pk, left, p, n2, lane, slabs, row_slot, first);
        else if (left > 4) stage1_batch<RK, G, 6, P>(pk, left, p, n2, lane, slabs, row_slot, first);
        else if (left > 2) stage1_batch<RK, G, 4, P>(pk, left, p, n2, lane, slabs, row_slot, first);
        else if (left > 0) stage1_batch<RK, G, 2, P>(pk, left, p, n2, lane, slabs, row_slot, first);
    } else {
        if (left > 0) stage1_batch<RK, G, 1, P>(pk, left, p, n2, lane, slabs, row_slot, first);
    }
    if (steps == 0) {   // no nonzeros: T is zero
        float acc[RK];
#pragma unroll
        for (int k = 0; k < RK; ++k) acc[k] = 0.f;
        for (int col = lane; col < n2; col += 64) slab_write<RK>(slabs, (uint32_t)col * (MGK_SEP_SLAB(RK) * 4) + row_slot, acc);
    }
}

// Stage 2 of one group of four columns (16 rows x 4 columns, one result per lane): c[] are the
// first eight packets of this lane's column, pk where the others are.
template <int RK, int G>
__device__ __forceinline__ float stage2_group(float (&c)[8], const float* pk, int steps, const char* slabs, uint32_t lbase) {
    float acc[RK];
#pragma unroll
    for (int k = 0; k < RK; ++k) acc[k] = 0.f;
    for (int b = 0; b < steps; b += 8) {
        if (b > 0) {
#pragma unroll
            for (int a = 0; a < 8; ++a) c[a] = pk[(int64_t)min(b + a, steps - 1) * 64];
        }
        constexpr int D = G >= 8 ? 1 : 2;   // packets per step
#pragma unroll
        for (int a = 0; a < 8; a += D) {
            if (b + a < steps) {   // wave-uniform
                float tv[D][G][RK];
#pragma unroll
                for (int d = 0; d < D; ++d) {
                    uint32_t sl[G];
                    if (D > 1 && d > 0 && b + a + d >= steps) c[a + d] = 0.f;
                    packet_slabs<RK, G>(sl, c[a + d]);
#pragma unroll
                    for (int u = 0; u < G; ++u) slab_read<RK>(tv[d][u], slabs, sl[u] + lbase);
                }
#pragma unroll
                for (int d = 0; d < D; ++d) packet_each<RK, G>(acc, c[a + d], tv[d]);
            }
        }
    }
    float s = acc[0];
#pragma unroll
    for (int k = 1; k < RK; ++k) s += acc[k];
    return s;
}

}  // namespace

#endif

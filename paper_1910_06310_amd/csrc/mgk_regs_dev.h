// Device code shared by the two solvers that keep the matrix entries of a pair in registers
// (mgk_regs.hip: the full system, mgk_reduced.hip: the reduced one): the fill of the registers and the
// sum over the lanes of an inner row.
#ifndef MGK_REGS_DEV_H
#define MGK_REGS_DEV_H

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "mgk_internal.h"

namespace {

// value of v in lane k (k a compile-time constant after unrolling)
__device__ __forceinline__ uint32_t lane_value(uint32_t v, int k) {
    return (uint32_t)__builtin_amdgcn_readlane((int)v, k);
}
__device__ __forceinline__ float lane_value(float v, int k) {
    return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), k));
}

// The loops over the wave's outer nonzeros are unrolled by template recursion, so that every index into the register array kap is a
// compile-time constant.

// Matrix entries of outer nonzeros K0 .. KEND-1 (lanes K0.. of e1s / l1; those below K0 + live are the
// wave's) against this lane's inner nonzeros: square-exponential kernel on prescaled labels,
// exp2(log2 A + log2 A' - (e - e')^2).  Lanes of e1s past the wave's run hold a huge
// label and idle inner slots hold l2 = -inf, so both give exactly 0.
template <int K0, int KEND, int SMAX, int C, bool WEIGHTED>
__device__ __forceinline__ void fill_se(float (&kap)[C][SMAX], int stop, const float (&e2s)[C],
                                        const float (&l2)[C], float e1s, float l1) {
    if constexpr (K0 < KEND) {
        if (K0 < stop) {
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const float e1 = lane_value(e1s, K0 + u);
                const float la = WEIGHTED ? lane_value(l1, K0 + u) : 0.f;
#pragma unroll
                for (int c = 0; c < C; ++c) {
                    const float d = e2s[c] - e1;
                    kap[c][K0 + u] = __builtin_amdgcn_exp2f(__builtin_fmaf(-d, d, WEIGHTED ? l2[c] + la : l2[c]));
                }
            }
        } else {
#pragma unroll
            for (int u = 0; u < 4; ++u)
#pragma unroll
                for (int c = 0; c < C; ++c) kap[c][K0 + u] = 0.f;
        }
        fill_se<K0 + 4, KEND, SMAX, C, WEIGHTED>(kap, stop, e2s, l2, e1s, l1);
    }
}

// the same for the constant edge kernel: A_ij * (A'_i'j' kappa_e); w1 is 0 past the run
template <int K0, int KEND, int SMAX, int C>
__device__ __forceinline__ void fill_const(float (&kap)[C][SMAX], int stop, const float (&w2c)[C], float w1) {
    if constexpr (K0 < KEND) {
        if (K0 < stop) {
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const float wa = lane_value(w1, K0 + u);
#pragma unroll
                for (int c = 0; c < C; ++c) kap[c][K0 + u] = w2c[c] * wa;
            }
        } else {
#pragma unroll
            for (int u = 0; u < 4; ++u)
#pragma unroll
                for (int c = 0; c < C; ++c) kap[c][K0 + u] = 0.f;
        }
        fill_const<K0 + 4, KEND, SMAX, C>(kap, stop, w2c, w1);
    }
}

// compact polynomial kernel on labels prescaled by 1 / rho; wprod = A_ij A'_i'j' per lane
// pair (0 on idle slots and past the run)
template <int K0, int KEND, int SMAX, int C>
__device__ __forceinline__ void fill_poly(float (&kap)[C][SMAX], int stop, const float (&e2s)[C],
                                          const float (&w2)[C], float e1s, float w1, const float* pc) {
    if constexpr (K0 < KEND) {
        if (K0 < stop) {
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const float e1 = lane_value(e1s, K0 + u);
                const float wa = lane_value(w1, K0 + u);
#pragma unroll
                for (int c = 0; c < C; ++c)
                    kap[c][K0 + u] = mgk_poly_kernel(e2s[c] - e1, pc) * (w2[c] * wa);
            }
        } else {
#pragma unroll
            for (int u = 0; u < 4; ++u)
#pragma unroll
                for (int c = 0; c < C; ++c) kap[c][K0 + u] = 0.f;
        }
        fill_poly<K0 + 4, KEND, SMAX, C>(kap, stop, e2s, w2, e1s, w1, pc);
    }
}

// Kernels over labels with D attributes, each prescaled by sqrt(log2(e) / (2 l_a^2)).
// RCONV false: Kronecker product of square exponentials, exp2(log2 A + log2 A' -
// sum_a (e_a - e'_a)^2), with l1 / l2 the log2 weights (-inf on idle slots; lanes past
// the run carry a huge attribute 0).  RCONV true: (A A' / D^2) sum_a sum_b
// exp2(-(e_a - e'_b)^2), with l1 / l2 the weights themselves (0 where there is no entry).
// One pass over the registers for every attribute (pair of attributes), in a loop: with the attributes of an entry side by side, a
// condition for each that D has not, it was 13 instructions and five branches an entry where this is 7 at D = 3 (Gram matrix
// of 350 molecules with three: 1219 -> 1161 us).
enum { kAttrBegin = 0, kAttrAdd = 1, kAttrEnd = 2 };
template <int P>
struct AttrPass {
    static constexpr int value = P;
};
template <int PASS, int K0, int KEND, int SMAX, int C, bool RCONV>
__device__ __forceinline__ void attr_pass(float (&kap)[C][SMAX], int stop, const float (&v2)[C], float v1) {
    if constexpr (K0 < KEND) {
        if (K0 < stop) {
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const float v = (PASS == kAttrBegin && RCONV) || (PASS == kAttrEnd && !RCONV) ? 0.f : lane_value(v1, K0 + u);
#pragma unroll
                for (int c = 0; c < C; ++c) {
                    float& k = kap[c][K0 + u];
                    const float d = v2[c] - v;
                    if (PASS == kAttrBegin) k = RCONV ? 0.f : v2[c] + v;
                    else if (PASS == kAttrAdd) k = RCONV ? k + __builtin_amdgcn_exp2f(-d * d) : __builtin_fmaf(-d, d, k);
                    else k = RCONV ? k * (v2[c] * v) : __builtin_amdgcn_exp2f(k);
                }
            }
        } else if (PASS == kAttrBegin) {
#pragma unroll
            for (int u = 0; u < 4; ++u)
#pragma unroll
                for (int c = 0; c < C; ++c) kap[c][K0 + u] = 0.f;
        }
        attr_pass<PASS, K0 + 4, KEND, SMAX, C, RCONV>(kap, stop, v2, v1);
    }
}
// All entries, in two parts of the registers (0 .. SB-1 and SB .. SMAX-1, up to stop0 and stop1).  outer(a): attribute a of this lane's
// outer nonzero; inner(a, c): of its inner nonzero of chunk c.
template <int SB, int SMAX, int C, bool RCONV, class Outer, class Inner>
__device__ __forceinline__ void fill_attr(float (&kap)[C][SMAX], int stop0, int stop1, int D, const float (&l2)[C], float l1, const Outer& outer,
                                          const Inner& inner) {
    auto pass = [&](auto which, const float (&v2)[C], float v1) {
        constexpr int PASS = decltype(which)::value;
        attr_pass<PASS, 0, SB, SMAX, C, RCONV>(kap, stop0, v2, v1);
        attr_pass<PASS, SB, SMAX, SMAX, C, RCONV>(kap, stop1, v2, v1);
    };
    pass(AttrPass<kAttrBegin>{}, l2, l1);
    const int last = RCONV ? D * D - 1 : D - 1;   // the attributes of the next pass are on their way during this one
    auto inner_of = [&](int t) { return RCONV ? t / D : t; };
    auto outer_of = [&](int t) { return RCONV ? t - t / D * D : t; };
    float e1 = outer(outer_of(0)), e2[C];
#pragma unroll
    for (int c = 0; c < C; ++c) e2[c] = inner(inner_of(0), c);
#pragma unroll 1
    for (int t = 0; t <= last; ++t) {
        const int next = min(t + 1, last);
        const float n1 = outer(outer_of(next));
        float n2[C];
#pragma unroll
        for (int c = 0; c < C; ++c) n2[c] = inner(inner_of(next), c);
        pass(AttrPass<kAttrAdd>{}, e2, e1);
        e1 = n1;
#pragma unroll
        for (int c = 0; c < C; ++c) e2[c] = n2[c];
    }
    pass(AttrPass<kAttrEnd>{}, l2, l1);
}

// acc[c] += m1 * (acc[c] one lane down) and then += m2 * (two lanes down), inside rows of
// 16 lanes: the sum over an inner row of at most 4 nonzeros arrives in its last lane.
// The DPP reads need two wait states after the write of the register they read; with two
// chunks the steps of one chunk fill part of the other's.
template <int C>
__device__ __forceinline__ void row_sums(float (&acc)[C], const float (&m1)[C], const float (&m2)[C]) {
    static_assert(C == 1 || C == 2, "one or two chunks");
    if constexpr (C == 1) {
        asm volatile(
            "s_nop 1\n\tv_fmac_f32_dpp %0, %0, %1 row_shr:1 row_mask:0xf bank_mask:0xf bound_ctrl:1\n\t"
            "s_nop 1\n\tv_fmac_f32_dpp %0, %0, %2 row_shr:2 row_mask:0xf bank_mask:0xf bound_ctrl:1"
            : "+v"(acc[0])
            : "v"(m1[0]), "v"(m2[0]));
    } else {
        asm volatile(
            "s_nop 1\n\tv_fmac_f32_dpp %0, %0, %2 row_shr:1 row_mask:0xf bank_mask:0xf bound_ctrl:1\n\t"
            "v_fmac_f32_dpp %1, %1, %3 row_shr:1 row_mask:0xf bank_mask:0xf bound_ctrl:1\n\t"
            "s_nop 0\n\tv_fmac_f32_dpp %0, %0, %4 row_shr:2 row_mask:0xf bank_mask:0xf bound_ctrl:1\n\t"
            "v_fmac_f32_dpp %1, %1, %5 row_shr:2 row_mask:0xf bank_mask:0xf bound_ctrl:1"
            : "+v"(acc[0]), "+v"(acc[1])
            : "v"(m1[0]), "v"(m1[1]), "v"(m2[0]), "v"(m2[1]));
    }
}

}  // namespace

#endif

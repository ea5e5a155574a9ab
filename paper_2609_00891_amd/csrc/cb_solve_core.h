// cb_solve_core.h -- pieces of the fp64 blocked Cholesky shared by the narrow
// (cb_solve.hip) and the wide (cb_solve_blocked.hip) ridge solves: the fp64
// matrix-core product, and the factorization of one 16 x 16 diagonal block
// with its inverse, in the registers of one wave.
#pragma once
#include <cfloat>
#include <type_traits>

#include "cb_internal.h"

namespace cb {
namespace {

constexpr int kWaves = 8;
constexpr int kThreads = 64 * kWaves;
constexpr int kBR = 17;                          // padded row of a 16 x 16 block (doubles)
constexpr int kBS = 16 * kBR;                    // one block

typedef __attribute__((ext_vector_type(4))) double f64x4_t;

// D += A B of a 16 x 4 by 4 x 16 block: lane l supplies A[l % 16][l / 16] and
// B[l / 16][l % 16] and holds D[l / 16 + 4 e][l % 16] in element e.
__device__ __forceinline__ f64x4_t mfma_f64(double a, double b, f64x4_t c) {
    return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
}

// DPP reads.  A register written by a vector instruction may be read through
// DPP two wait states later at the earliest, and the compiler does not see that
// an inline statement reads through DPP: each of them opens with the wait itself.

// t[i] += (lane R + i of this row of 16 lanes' a) * nt and v[i] += (the same) * nv, i < ROWS.
template <int R, int ROWS>
__device__ __forceinline__ void fmac_rows_bcast(double *t, double *v, double a, double nt, double nv) {
#define CB_FMAC(d, x, i) "v_fmac_f64_dpp %[" #d #i "], %[a], %[" #x "] row_newbcast:%[r" #i "] row_mask:0xf bank_mask:0xf\n\t"
#define CB_ROW(i) CB_FMAC(t, nt, i) CB_FMAC(v, nv, i)
#define CB_OUT(i) [t##i] "+&v"(t[i]), [v##i] "+&v"(v[i])
#define CB_IN [a] "v"(a), [nt] "v"(nt), [nv] "v"(nv)
#define CB_LANE(i) [r##i] "n"(R + i)
    static_assert(ROWS >= 1 && ROWS <= 4 && R + ROWS <= 16, "one to four rows");
    if constexpr (ROWS == 1)
        asm("s_nop 1\n\t" CB_ROW(0) : CB_OUT(0) : CB_IN, CB_LANE(0));
    else if constexpr (ROWS == 2)
        asm("s_nop 1\n\t" CB_ROW(0) CB_ROW(1) : CB_OUT(0), CB_OUT(1) : CB_IN, CB_LANE(0), CB_LANE(1));
    else if constexpr (ROWS == 3)
        asm("s_nop 1\n\t" CB_ROW(0) CB_ROW(1) CB_ROW(2)
            : CB_OUT(0), CB_OUT(1), CB_OUT(2) : CB_IN, CB_LANE(0), CB_LANE(1), CB_LANE(2));
    else
        asm("s_nop 1\n\t" CB_ROW(0) CB_ROW(1) CB_ROW(2) CB_ROW(3)
            : CB_OUT(0), CB_OUT(1), CB_OUT(2), CB_OUT(3) : CB_IN, CB_LANE(0), CB_LANE(1), CB_LANE(2), CB_LANE(3));
#undef CB_FMAC
#undef CB_ROW
#undef CB_OUT
#undef CB_IN
#undef CB_LANE
}

// Lane R of this row of 16 lanes' v.
template <int R>
__device__ __forceinline__ double row_bcast(double v) {
    double o;
    asm("s_nop 1\n\tv_mov_b64_dpp %0, %1 row_newbcast:%2 row_mask:0xf bank_mask:0xf" : "=&v"(o) : "v"(v), "n"(R));
    return o;
}

// 1 / d: the hardware estimate y and 1 / (1 - r) = 1 + r + r^2 with r = 1 - d y.
__device__ __forceinline__ double rcp_f64(double d) {
    const double y = __builtin_amdgcn_rcp(d);
    const double r = __builtin_fma(-d, y, 1.0);
    return __builtin_fma(y, __builtin_fma(r, r, r), y);
}

// Rows R .. 15, up to a multiple of four, then four at a time.
template <int K, int R>
__device__ __forceinline__ void pivot_rows(double (&t)[16], double (&v)[16], double nt, double nv) {
    if constexpr (R < 16) {
        constexpr int ROWS = 4 - R % 4;
        fmac_rows_bcast<R, ROWS>(t + R, v + R, t[K], nt, nv);
        pivot_rows<K, R + ROWS>(t, v, nt, nv);
    }
}

// Steps K .. 15 of T = L D L^T: row k, divided by its pivot, times t_k[lane r] = d_k L[r][k] leaves row r.  dk: the
// pivot of lane q's column.
template <int K>
__device__ __forceinline__ void pivot_steps(double (&t)[16], double (&v)[16], double &dk, int q) {
    if constexpr (K < 16) {
        dk = q == K ? t[K] : dk;
        const double rd = -rcp_f64(row_bcast<K>(t[K]));
        pivot_rows<K, K + 1>(t, v, t[K] * rd, v[K] * rd);
        pivot_steps<K + 1>(t, v, dk, q);
    }
}

// 1 / sqrt(d), d positive and finite: the hardware estimate y and one step of
// the series (1 - r)^(-1/2) = 1 + r/2 + 3 r^2 / 8 with r = 1 - d y^2.
__device__ __forceinline__ double rsqrt_f64(double d) {
    const double y = __builtin_amdgcn_rsq(d);
    const double r = __builtin_fma(-(d * y), y, 1.0);
    return __builtin_fma(y * r, __builtin_fma(0.375, r, 0.5), y);
}

__device__ __forceinline__ void wave_sync_lds() {
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    __builtin_amdgcn_wave_barrier();
}

__device__ __forceinline__ constexpr int block_of(int k, int i) { return i * (i + 1) / 2 + k; }   // k <= i

// Factor the 16 x 16 block T at D (LDS, row stride kBR; symmetric, both halves
// present) as L D L^T: on return D holds L^-1, dk the pivot of lane q's column
// and the return value the ballot of lanes 0-15 whose pivot is not positive
// and finite.  BIAS: bias16[0..15] is replaced by L^-1 times it.  One wave; its
// own writes to D before the call are waited for here.
template <bool BIAS>
__device__ __forceinline__ uint64_t factor_block(double *D, double *bias16, int lane, double &dk) {
    const int q = lane & 15, g = lane >> 4;
    wave_sync_lds();
    double t[16], v[16];
    dk = 1.0;
#pragma unroll
    for (int r = 0; r < 16; ++r) {
        t[r] = D[r * kBR + q];
        v[r] = r == q ? 1.0 : 0.0;
        if (BIAS && g == 1) v[r] = bias16[r];
    }
    pivot_steps<0>(t, v, dk, q);
    if (g == 0) {
#pragma unroll
        for (int r = 0; r < 16; ++r) D[r * kBR + q] = v[r];
    }
    if (BIAS && lane == 16) {
#pragma unroll
        for (int r = 0; r < 16; ++r) bias16[r] = v[r];
    }
    return __ballot(lane < 16 && !(dk > 0.0 && dk <= DBL_MAX));
}

}  // namespace
}  // namespace cb

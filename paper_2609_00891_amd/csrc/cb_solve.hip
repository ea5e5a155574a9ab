// cb_solve.hip -- batched ridge solve, one workgroup per system (gfx950).
//
// CacheBridge Sec. 3.1 (Eq. closedform) and Sec. 3.4: the maps are the ridge
// solutions W~ = (G + lambda D)^{-1} C of the augmented moments, one system of
// P = d_s + 1 unknowns per map, all in fp64.
//   lambda_m = lambda, or lambda * tr(G) / P with CB_LAMBDA_RELATIVE; with
//   CB_RIDGE_BIAS_UNPENALIZED the last (bias) diagonal entry gets no lambda.
//
// Method: blocked Cholesky M = U^T U over the first d_s unknowns in 16 x 16
// blocks, the right-hand sides eliminated along with it, then back
// substitution; the bias unknown (the last row and column of the augmented
// system) is one more elimination step at the end.  Row j of blocks:
//     T_ji = M_ji - sum_{k<j} U_kj^T U_ki      (i >= j; for a right-hand side
//     T_j  = C_j  - sum_{k<j} U_kj^T Z_k        the same with Z in place of U)
//     U_jj^T U_jj = T_jj, V_j = U_jj^{-T}, U_ji = V_j T_ji, Z_j = V_j T_j
// and backwards W_i = V_i^T (Z_i - sum_{k>i} U_ik W_k).
//
// What bounds it: the fp64 rate (2.5 M multiply-adds per system at d_s = d_t =
// 128) and, for few systems, the serial chain of pivots.  So:
//   * the products are v_mfma_f64_16x16x4: its result layout (lane l: rows
//     l / 16 + 4 e, column l mod 16) is the layout of its right operand's four
//     K steps, so a wave keeps one 16-column tile of right-hand sides (32 fp64
//     per lane) in registers through both substitutions and uses it as it is;
//     only the U blocks pass through LDS;
//   * eight waves.  Wave 0 factors the diagonal blocks; waves 1-7 make one
//     block of U's row each (wave 7 the next diagonal block's products) and
//     eliminate their right-hand sides beside it.  Wave 0's own right-hand
//     sides wait until the factor is complete: they are not on its way;
//   * the factorization of a diagonal block (as L D L^T) and its inverse are
//     one sweep in registers: lane q of every 16 lanes holds the block's
//     column q and a column of the identity (lane 16: the bias column), and a
//     pivot step is one v_fmac with a row broadcast (DPP) per row and column;
//   * 36 upper blocks of 16 x 17 doubles are 78 KB of LDS at d_s = 128 and a
//     lane has 128 registers, so two systems share a compute unit and one's
//     pivots overlap the other's products.  (At d_t = 128 two to four values
//     spill, elsewhere none: the bias coefficient is taken out of a row of
//     right-hand sides where the back substitution reaches it.  Out of all rows
//     in a pass before, 30 spilled at d_s = d_t = 128 and 250 at d_t = 64 and 96:
//     1,024 systems 150 -> 146, 154 -> 121 and 120 -> 100 us.)
// Measured, before (Gauss-Jordan in registers, one barrier per pivot) and now,
// us: 1,024 systems of d_s = d_t = 128 942 -> 146 (MFMA floor 70); 320 centered
// ones of 96 and 128 307 -> 45; 10,240 centered ones of 128 and 128 8,960 ->
// 1,400; 4 systems of 64 and 64 97 -> 15.  With a fifth wave factoring beside
// four that own two tiles (168 registers, one system per compute unit) 245; the
// same with broadcasts by v_readlane 250.
//
// A pivot that is not positive and finite gives info = its 1-based index and
// zero maps, the report of an unblocked Cholesky factorization.
//
// Centered form (Sec. 3.1, Eq. closedform as written): the system is
// (A + lambda_m I) W = B of size d_s with the centered moments A, B, and the
// bias row is b = mu_y - W^T mu_x, formed in fp64 from the unrounded W.  The
// relative lambda uses the trace of the augmented matrix the same data would
// give, tr(A) + S |mu_x|^2 + S (S = sum w), so that both forms solve the same
// problem.
#include "cb_solve_core.h"

namespace cb {
namespace {

// NB: 16-row blocks of d_s.  Plain: G [P][P], C [P][d_t] -> maps [P][d_t], P =
// d_s + 1.  Centered: G = A [d_s][d_s], C = B [d_s][d_t], sums [1 + d_s + d_t]
// -> maps [d_s + 1][d_t].  NCT: 16-column tiles of d_t, owned by the last NCT waves.
template <int NB, int NCT, bool CENTERED>
__global__ __launch_bounds__(kThreads, 4) void ridge_solve_kernel(const float *__restrict__ G,
                                                                  const float *__restrict__ C,
                                                                  const double *__restrict__ sums, float lambda,
                                                                  uint32_t flags, float *__restrict__ maps,
                                                                  int32_t *__restrict__ info) {
    constexpr int N = 16 * NB, d_t = 16 * NCT;
    constexpr int P = CENTERED ? N : N + 1;               // size of the system
    static_assert(NB <= kWaves && NCT <= kWaves, "one block of a row of U, and one tile, per wave");
    __shared__ double U[NB * (NB + 1) / 2 * kBS];         // upper blocks (M, then U); L_jj^-1 in the diagonal ones
    __shared__ double rsv[N];                             // D^(-1/2): V_j = rsv_j L_jj^-1
    __shared__ double zg[N];                              // plain: bias column, then its eliminated values; centered: mu_x
    __shared__ double s_h;                                // plain: 1 / last pivot
    __shared__ int s_bad;

    const int m = blockIdx.x;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int q = lane & 15, g = lane >> 4;
    const float *Gm = G + (int64_t)m * P * P;
    const float *Cm = C + (int64_t)m * P * d_t;
    float *Wm = maps + (int64_t)m * (N + 1) * d_t;
    const double *sm = CENTERED ? sums + (int64_t)m * (1 + N + d_t) : nullptr;
    const int tile = wave - (kWaves - NCT);
    const bool owner = tile >= 0;
    const int col = 16 * (owner ? tile : 0) + q;

    // ---- this wave's right-hand-side columns; block row j + 1 is requested while row j is worked on, so a row
    // takes registers only from its own step on
    f64x4_t Z[NB];
    float cn[4];
    auto load_row = [&](int j, int g) __attribute__((always_inline)) {
#pragma unroll
        for (int e = 0; e < 4; ++e) cn[e] = Cm[(16 * j + 4 * e + g) * d_t + col];
    };
    auto take_row = [&](int j) __attribute__((always_inline)) {
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            asm volatile("" : "+v"(cn[e]));               // waited for here, not where it was requested
            Z[j][e] = (double)cn[e];
        }
    };
    if (owner) load_row(0, g);
    double diag[(P + 63) / 64];                           // wave 0: its share of the trace
#pragma unroll
    for (int n = 0; n < (P + 63) / 64; ++n) {
        const int i = 64 * n + lane;
        diag[n] = wave == 0 && i < P ? (double)Gm[i * P + i] : 0.0;
    }
    // ---- upper blocks of G into LDS: block row j is 16 rows from column 16 j on.  All loads are requested before
    // the first is stored (the indices past a block row's end repeat its last element, so no branch separates them)
    {
        constexpr int MAXQ = (16 * N + kThreads - 1) / kThreads;
        float v[NB][MAXQ];
#pragma unroll
        for (int pass = 0; pass < 2; ++pass)
#pragma unroll
            for (int j = 0; j < NB; ++j) {
                const int w = N - 16 * j;
#pragma unroll
                for (int n = 0; n * kThreads < 16 * w; ++n) {
                    const int e = min(n * kThreads + tid, 16 * w - 1);
                    const int r = e / w, c = e - r * w;
                    if (pass == 0) v[j][n] = Gm[(16 * j + r) * P + 16 * j + c];
                    else U[block_of(j, j + c / 16) * kBS + r * kBR + c % 16] = (double)v[j][n];
                }
            }
    }
    if (tid < N) zg[tid] = !CENTERED ? (double)Gm[N * P + tid] : sm[0] != 0.0 ? sm[1 + tid] / sm[0] : 0.0;
    __syncthreads();

    // the A operand of V_j (lane: V[q][4 s + g]) and of V_j^T (V[4 s + g][q])
    auto load_v = [&](double (&v)[4], int j, int q, int g) __attribute__((always_inline)) {
        const double *V = U + block_of(j, j) * kBS + q * kBR + g;
        const double rs = rsv[16 * j + q];
#pragma unroll
        for (int s = 0; s < 4; ++s) v[s] = V[4 * s] * rs;
    };
    // Z_j = V_j (C_j - sum_{k<j} U_kj^T Z_k)
    auto eliminate = [&](int j, const f64x4_t &acc, const double (&v)[4]) __attribute__((always_inline)) {
        const f64x4_t y = Z[j] - acc;
        f64x4_t x = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
        for (int s = 0; s < 4; ++s) x = mfma_f64(v[s], y[s], x);
        Z[j] = x;
    };

    if (wave == 0) {
        // ================= the factoring wave
        double tr = 0.0;
#pragma unroll
        for (int n = 0; n < (P + 63) / 64; ++n) tr += diag[n];
        if (CENTERED)
            for (int i = lane; i < P; i += 64) tr += sm[1 + i] * zg[i];       // S mu_i^2
        for (int o = 32; o > 0; o >>= 1) tr += __shfl_xor(tr, o);
        if (CENTERED) tr += sm[0];
        const double lam = (flags & CB_LAMBDA_RELATIVE) ? (double)lambda * tr / (double)(N + 1) : (double)lambda;
        int bad = 0;
#pragma unroll 1
        for (int j = 0; j < NB; ++j) {
            double *D = U + block_of(j, j) * kBS;
            // T_jj and the bias column's t_j: wave 7 took out the products over the rows before the last one
            f64x4_t acc0 = {0.0, 0.0, 0.0, 0.0}, acc1 = {0.0, 0.0, 0.0, 0.0};
            double tg = 0.0, dv[4];
#pragma unroll
            for (int e = 0; e < 4; ++e) dv[e] = D[(g + 4 * e) * kBR + q] + (g + 4 * e == q ? lam : 0.0);
            if (j > 0) {
                const double *B = U + block_of(j - 1, j) * kBS + g * kBR + q;
                double a[4];
#pragma unroll
                for (int s = 0; s < 4; ++s) a[s] = B[4 * s * kBR];
                acc0 = mfma_f64(a[0], a[0], acc0);
                acc1 = mfma_f64(a[1], a[1], acc1);
                acc0 = mfma_f64(a[2], a[2], acc0);
                acc1 = mfma_f64(a[3], a[3], acc1);
                if (!CENTERED) {
#pragma unroll
                    for (int s = 0; s < 4; ++s) tg = __builtin_fma(a[s], zg[16 * (j - 1) + 4 * s + g], tg);
                    tg += __shfl_xor(tg, 16);
                    tg += __shfl_xor(tg, 32);
                }
            }
#pragma unroll
            for (int e = 0; e < 4; ++e) D[(g + 4 * e) * kBR + q] = dv[e] - (acc0[e] + acc1[e]);
            if (!CENTERED && g == 0) zg[16 * j + q] -= tg;
            double dk;
            const uint64_t wrong = factor_block<!CENTERED>(D, zg + 16 * j, lane, dk);
            if (wrong && bad == 0) bad = 16 * j + __ffsll((unsigned long long)wrong);
            const double rs = rsqrt_f64(dk);
            if (g == 0) rsv[16 * j + q] = rs;
            __syncthreads();                              // V_j is published
            if (!CENTERED && g == 0) zg[16 * j + q] *= rs;
            if (j + 1 < NB) __syncthreads();              // row j of U is published
        }
        if (!CENTERED) {
            // the bias unknown's pivot
            wave_sync_lds();
            double s = 0.0;
            for (int i = lane; i < N; i += 64) s = __builtin_fma(zg[i], zg[i], s);
            for (int o = 32; o > 0; o >>= 1) s += __shfl_xor(s, o);
            const double h = (double)Gm[N * P + N] + ((flags & CB_RIDGE_BIAS_UNPENALIZED) ? 0.0 : lam) - s;
            bad = bad == 0 && !(h > 0.0 && h <= DBL_MAX) ? N + 1 : bad;
            if (lane == 0) s_h = 1.0 / h;
        }
        if (lane == 0) {
            s_bad = bad;
            info[m] = bad;
        }
        __syncthreads();
        if (owner) {
            // its right-hand sides, now that the whole factor is there
#pragma unroll
            for (int j = 0; j < NB; ++j) {
                int q = tid & 15, g = (tid >> 4) & 3;
                asm volatile("" : "+v"(q), "+v"(g));
                take_row(j);
                if (j + 1 < NB) load_row(j + 1, g);
                double v[4];
                load_v(v, j, q, g);
                f64x4_t acc = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
                for (int k = 0; k < j; ++k)
#pragma unroll
                    for (int s = 0; s < 4; ++s)
                        acc = mfma_f64(U[block_of(k, j) * kBS + (4 * s + g) * kBR + q], Z[k][s], acc);
                eliminate(j, acc, v);
            }
        }
    } else {
        // ================= the other waves: rows of U and right-hand sides
#pragma unroll
        for (int j = 0; j < NB; ++j) {
            // (addresses are formed in the row that uses them instead of being held across the kernel)
            int q = tid & 15, g = (tid >> 4) & 3, i = j + wave;
            asm volatile("" : "+v"(q), "+v"(g), "+s"(i));
            if (owner) take_row(j);
            if (owner && j + 1 < NB) load_row(j + 1, g);
            // this wave's block (j, i) of U, i = j + wave; wave 7, from row 1 on, block (j + 1, j + 1)'s products
            f64x4_t am = {0.0, 0.0, 0.0, 0.0}, acc = {0.0, 0.0, 0.0, 0.0};
            if (j > 0 && j + 1 < NB && wave == kWaves - 1) {
                double tg = 0.0;
                f64x4_t a2 = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
                for (int k = 0; k < j; ++k)
#pragma unroll
                    for (int s = 0; s < 4; ++s) {
                        const double b = U[block_of(k, j + 1) * kBS + (4 * s + g) * kBR + q];
                        if (s & 1) a2 = mfma_f64(b, b, a2);
                        else am = mfma_f64(b, b, am);
                        if (!CENTERED) tg = __builtin_fma(b, zg[16 * k + 4 * s + g], tg);
                    }
                double *D = U + block_of(j + 1, j + 1) * kBS + g * kBR + q;
#pragma unroll
                for (int e = 0; e < 4; ++e) D[4 * e * kBR] -= am[e] + a2[e];
                if (!CENTERED) {
                    tg += __shfl_xor(tg, 16);
                    tg += __shfl_xor(tg, 32);
                    if (g == 0) zg[16 * (j + 1) + q] -= tg;
                }
            } else if (j + 1 < NB && i < NB) {
#pragma unroll
                for (int k = 0; k < j; ++k)
#pragma unroll
                    for (int s = 0; s < 4; ++s)
                        am = mfma_f64(U[block_of(k, j) * kBS + (4 * s + g) * kBR + q],
                                      U[block_of(k, i) * kBS + (4 * s + g) * kBR + q], am);
                const double *T = U + block_of(j, i) * kBS + g * kBR + q;
#pragma unroll
                for (int e = 0; e < 4; ++e) am[e] = T[4 * e * kBR] - am[e];
            }
            if (owner) {
#pragma unroll
                for (int k = 0; k < j; ++k)
#pragma unroll
                    for (int s = 0; s < 4; ++s)
                        acc = mfma_f64(U[block_of(k, j) * kBS + (4 * s + g) * kBR + q], Z[k][s], acc);
            }
            __syncthreads();                              // V_j is published
            double v[4];
            load_v(v, j, q, g);
            if (j + 1 < NB && i < NB) {
                f64x4_t x = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
                for (int s = 0; s < 4; ++s) x = mfma_f64(v[s], am[s], x);
                double *T = U + block_of(j, i) * kBS + g * kBR + q;
#pragma unroll
                for (int e = 0; e < 4; ++e) T[4 * e * kBR] = x[e];
            }
            if (j + 1 < NB) __syncthreads();              // row j of U is published
            if (owner) eliminate(j, acc, v);
        }
        __syncthreads();                                  // the last pivot and the verdict
    }
    if (s_bad) {
        for (int e = tid; e < (N + 1) * d_t; e += kThreads) Wm[e] = 0.f;
        return;
    }
    if (!owner) return;
    // plain: the bias unknown, W_N = (C_N - z_g . Z) / h, taken out of the right-hand sides as each row is solved
    double wb = 0.0;
    if constexpr (!CENTERED) {
        f64x4_t s4 = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
        for (int j = 0; j < NB; ++j) {
            int g = (tid >> 4) & 3;
            asm volatile("" : "+v"(g)::"memory");         // z_g is read where it is used, not held in registers
#pragma unroll
            for (int e = 0; e < 4; ++e) s4[e] = __builtin_fma(zg[16 * j + 4 * e + g], Z[j][e], s4[e]);
        }
        double s = (s4[0] + s4[1]) + (s4[2] + s4[3]);
        s += __shfl_xor(s, 16);
        s += __shfl_xor(s, 32);
        wb = ((double)Cm[N * d_t + col] - s) * s_h;
        if (g == 0) Wm[N * d_t + col] = (float)wb;
    }
    // back substitution: every wave for its own columns, no barrier
#pragma unroll
    for (int i = NB - 1; i >= 0; --i) {
        int q = tid & 15, g = (tid >> 4) & 3;
        asm volatile("" : "+v"(q), "+v"(g));
        double v[4];
#pragma unroll
        for (int s = 0; s < 4; ++s) v[s] = U[block_of(i, i) * kBS + (4 * s + g) * kBR + q] * rsv[16 * i + 4 * s + g];
        f64x4_t acc = {0.0, 0.0, 0.0, 0.0}, x = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
        for (int k = i + 1; k < NB; ++k)
#pragma unroll
            for (int s = 0; s < 4; ++s) acc = mfma_f64(U[block_of(i, k) * kBS + q * kBR + 4 * s + g], Z[k][s], acc);
        f64x4_t y = Z[i] - acc;
        if constexpr (!CENTERED) {
#pragma unroll
            for (int e = 0; e < 4; ++e) y[e] = __builtin_fma(-zg[16 * i + 4 * e + g], wb, y[e]);
        }
#pragma unroll
        for (int s = 0; s < 4; ++s) x = mfma_f64(v[s], y[s], x);
        Z[i] = x;
#pragma unroll
        for (int e = 0; e < 4; ++e) Wm[(16 * i + 4 * e + g) * d_t + col] = (float)x[e];
    }
    if constexpr (CENTERED) {
        // b_j = mu_y,j - sum_i mu_x,i W_ij
        const double S = sm[0];
        f64x4_t s4 = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
        for (int j = 0; j < NB; ++j) {
            asm volatile("" ::: "memory");
#pragma unroll
            for (int e = 0; e < 4; ++e) s4[e] = __builtin_fma(zg[16 * j + 4 * e + g], Z[j][e], s4[e]);
        }
        double s = (s4[0] + s4[1]) + (s4[2] + s4[3]);
        s += __shfl_xor(s, 16);
        s += __shfl_xor(s, 32);
        if (g == 0) Wm[N * d_t + col] = (float)((S != 0.0 ? sm[1 + N + col] / S : 0.0) - s);
    }
}

template <int NB, bool CENTERED>
hipError_t launch_nb(int32_t n_maps, int32_t d_t, const float *G, const float *C, const double *sums, float lambda,
                     uint32_t flags, float *maps, int32_t *info, hipStream_t s) {
    const dim3 grid(n_maps), block(kThreads);
    switch (d_t) {
        case 64: hipLaunchKernelGGL((ridge_solve_kernel<NB, 4, CENTERED>), grid, block, 0, s, G, C, sums, lambda, flags, maps, info); break;
        case 96: hipLaunchKernelGGL((ridge_solve_kernel<NB, 6, CENTERED>), grid, block, 0, s, G, C, sums, lambda, flags, maps, info); break;
        case 128: hipLaunchKernelGGL((ridge_solve_kernel<NB, 8, CENTERED>), grid, block, 0, s, G, C, sums, lambda, flags, maps, info); break;
        default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

template <bool CENTERED>
hipError_t launch(int32_t n_maps, int32_t d_s, int32_t d_t, const float *G, const float *C, const double *sums,
                  float lambda, uint32_t flags, float *maps, int32_t *info, hipStream_t s) {
    if (n_maps == 0) return hipSuccess;
    switch (d_s) {
        case 64: return launch_nb<4, CENTERED>(n_maps, d_t, G, C, sums, lambda, flags, maps, info, s);
        case 96: return launch_nb<6, CENTERED>(n_maps, d_t, G, C, sums, lambda, flags, maps, info, s);
        case 128: return launch_nb<8, CENTERED>(n_maps, d_t, G, C, sums, lambda, flags, maps, info, s);
        default: return hipErrorInvalidValue;
    }
}

}  // namespace

hipError_t launch_solve(int32_t n_maps, int32_t P, int32_t d_t, const float *G, const float *C,
                        float lambda, uint32_t flags, float *maps, int32_t *info, hipStream_t s) {
    return launch<false>(n_maps, P - 1, d_t, G, C, nullptr, lambda, flags, maps, info, s);
}

hipError_t launch_solve_centered(int32_t n_maps, int32_t d_s, int32_t d_t, const double *sums, const float *A,
                                 const float *B, float lambda, uint32_t flags, float *maps, int32_t *info,
                                 hipStream_t s) {
    return launch<true>(n_maps, d_s, d_t, A, B, sums, lambda, flags, maps, info, s);
}

}  // namespace cb

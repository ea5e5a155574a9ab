// cb_probe.hip -- held-in R^2 of layer-selection probes on gfx950.
//
// CacheBridge Sec. 3.1 ranks the source layers of every target layer by the
// held-in R^2 of centered single-source-layer probes, averaged over KV heads
// and K/V.  The probes are ordinary maps of a plan whose head map pairs every
// target head with every candidate source layer; their statistics and solve
// are the centered ones.  With the probe's centered moments A, B, its fitted
// map [W ; b] (b = mu_y - W^T mu_x, so the residual has weighted mean zero),
// the weighted sums and the per-channel sums of squares,
//     TSS = sum_j (sum w y_j^2 - (sum w y_j)^2 / S),
//     RSS = TSS - 2 tr(W^T B) + tr(W^T A W),      R^2 = 1 - RSS / TSS,
// which needs no further pass over the tokens.
//
// probe_r2_kernel: one workgroup per map, one wave per 32 rows of A W, formed
// in fp32 by v_mfma_f32_32x32x2_f32.  A is symmetric, so the left operand's
// column k is row k of A: both operands are rows, 32 consecutive floats per half
// wave.  W is staged in LDS (every wave reads all of it); each element of A and B
// is read once, from global memory, A a group of K steps ahead.  The traces and
// TSS are summed in fp64 over the workgroup in a fixed order.
// Bound: HBM, 196 KB per map at d_s = d_t = 128, and near it the fp32 products, 7
// us of a compute unit per map: with 270 registers a lane a SIMD holds one wave at
// d_t = 128 (two at 96, three at 64), that is one map per compute unit, whose loads
// overlap with its own products only.  Measured, 10,240 maps of 128 and 128: 6.70
// ms with FMAs from LDS, a thread per half row, and one thread summing TSS; now
// 0.60 ms.
#include "cb_internal.h"

namespace cb {
namespace {

typedef __attribute__((ext_vector_type(16))) float f32x16_t;

template <int DS, int DT>
__global__ __launch_bounds__(2 * DS) void probe_r2_kernel(const double *__restrict__ sums,
                                                          const double *__restrict__ sq, const float *__restrict__ A,
                                                          const float *__restrict__ B, const float *__restrict__ maps,
                                                          double *__restrict__ r2) {
    constexpr int RB = DS / 32, CB = DT / 32, NT = 64 * RB;   // row blocks (waves), column blocks
    constexpr int GK = 16;                                    // K steps (two rows of A) per group
    static_assert(DS / 2 % GK == 0, "whole groups");
    __shared__ __attribute__((aligned(16))) float Ws[DS * DT];   // W [d_s][d_t]
    __shared__ double red[3][RB];
    const int m = blockIdx.x, tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int n = lane & 31, h = lane >> 5;
    const float *Am = A + (int64_t)m * DS * DS;
    const float *Bm = B + (int64_t)m * DS * DT;
    const float *Wm = maps + (int64_t)m * (DS + 1) * DT;      // rows 0..d_s-1 = W
    const double *sm = sums + (int64_t)m * (1 + DS + DT);
    const double *qm = sq + (int64_t)m * (DS + DT);

    const float *Ap = Am + h * DS + 32 * wave + n;            // A[k][32 wave + n], k = 2 step + h
    float a[2][GK];
#pragma unroll
    for (int s = 0; s < GK; ++s) a[0][s] = Ap[2 * s * DS];
#pragma unroll
    for (int e = 0; e < DS * DT / NT; ++e) Ws[e * NT + tid] = Wm[e * NT + tid];
    __syncthreads();

    f32x16_t acc[CB];
#pragma unroll
    for (int c = 0; c < CB; ++c)
#pragma unroll
        for (int v = 0; v < 16; ++v) acc[c][v] = 0.f;
#pragma unroll
    for (int gk = 0; gk < DS / 2 / GK; ++gk) {
        if (gk + 1 < DS / 2 / GK) {
#pragma unroll
            for (int s = 0; s < GK; ++s) a[(gk + 1) & 1][s] = Ap[2 * ((gk + 1) * GK + s) * DS];
        }
#pragma unroll
        for (int s = 0; s < GK; ++s) {
            const int k = 2 * (gk * GK + s) + h;
#pragma unroll
            for (int c = 0; c < CB; ++c)
                acc[c] = __builtin_amdgcn_mfma_f32_32x32x2f32(a[gk & 1][s], Ws[k * DT + 32 * c + n], acc[c], 0, 0, 0);
        }
    }
    // shares of tr(W^T B) and tr(W^T A W); row of acc[c][v]: 8 (v / 4) + 4 h + v mod 4, column 32 c + n
    double t1 = 0.0, t2 = 0.0, ts = 0.0;
#pragma unroll
    for (int c = 0; c < CB; ++c)
#pragma unroll
        for (int v = 0; v < 16; ++v) {
            const int e = (32 * wave + 8 * (v >> 2) + 4 * h + (v & 3)) * DT + 32 * c + n;
            const double w = (double)Ws[e];
            t1 = __builtin_fma(w, (double)Bm[e], t1);
            t2 = __builtin_fma(w, (double)acc[c][v], t2);
        }
    const double S = sm[0];
    for (int j = tid; j < DT; j += NT)
        if (S != 0.0) ts += qm[DS + j] - sm[1 + DS + j] * (sm[1 + DS + j] / S);
    // fixed-order block sums (wave shuffles, then one value per wave)
    for (int o = 32; o > 0; o >>= 1) {
        t1 += __shfl_xor(t1, o);
        t2 += __shfl_xor(t2, o);
        ts += __shfl_xor(ts, o);
    }
    if (lane == 0) {
        red[0][wave] = t1;
        red[1][wave] = t2;
        red[2][wave] = ts;
    }
    __syncthreads();
    if (tid == 0) {
        double tr1 = 0.0, tr2 = 0.0, tss = 0.0;
        for (int w = 0; w < RB; ++w) {
            tr1 += red[0][w];
            tr2 += red[1][w];
            tss += red[2][w];
        }
        r2[m] = tss > 0.0 ? 1.0 - (tss - 2.0 * tr1 + tr2) / tss : 0.0;
    }
}

template <int DS, int DT>
hipError_t launch_probe_r2_t(int32_t n_maps, const double *sums, const double *sq, const float *A, const float *B,
                             const float *maps, double *r2, hipStream_t s) {
    hipLaunchKernelGGL((probe_r2_kernel<DS, DT>), dim3(n_maps), dim3(2 * DS), 0, s, sums, sq, A, B, maps, r2);
    return hipGetLastError();
}

}  // namespace

hipError_t launch_probe_r2(int32_t n_maps, int32_t d_s, int32_t d_t, const double *sums, const double *sq,
                           const float *A, const float *B, const float *maps, double *r2, hipStream_t s) {
    if (n_maps == 0) return hipSuccess;
    CB_DISPATCH(launch_probe_r2_t, d_s, d_t, n_maps, sums, sq, A, B, maps, r2, s);
}

}  // namespace cb

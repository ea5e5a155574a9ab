// cb_solve_blocked.hip -- batched ridge solve for wide features (P > 129).
//
// CacheBridge Sec. 3.1 (Eq. closedform) with the multi-layer feature of
// Sec. 3.2 (P = k d_s + 1, 1025 at k = 8): the systems no longer fit in one
// workgroup's registers or LDS, so each one is factored in the caller's
// workspace, all arithmetic fp64:
//
//   M = G + lambda_m D  (lambda_m = lambda, or lambda tr(G) / P; D = I, or
//                        diag(1, .., 1, 0) with CB_RIDGE_BIAS_UNPENALIZED)
//
// Right-looking blocked Cholesky M = U^T U of the augmented matrix [M | C] in
// panels of 128 rows, the right-hand sides being columns like any others:
//   first   one workgroup per system: lambda_m, then the factor of the first
//           diagonal block;
//   solve p one workgroup per 128 columns right of panel p: the panel's rows
//           of them, U_p,c = U_pp^-T T_p,c (16 x 16 blocks as in cb_solve.hip,
//           a wave's 16 columns in its registers, no barrier);
//   update p one workgroup per 128 x 128 tile of the rows below: T -= U_p^T U_p.
//           The workgroup of the next diagonal tile goes on to factor it, so
//           that the next panel's solve can start with the next launch;
//   back    the substitution from the last panel up, then the maps: one
//           workgroup per 16 right-hand sides, or per system (see the launch).
// One row and column past a multiple of 128 (P = 128 k + 1, the bias) is no
// panel of its own: it stays a column like the right-hand sides, and "back"
// starts with its pivot.
//
// What bounds it.  Many systems: the fp64 rate (P^3 / 3 + 2 P^2 d_t operations
// each) and, near it, the trailing matrix through HBM.  Few systems: the chain
// of panels.  A workgroup per system (the form before) left most of the chip
// idle below about 500 systems and took the latency of one whole system, 7.8
// ms at P = 1025, however few there were; tiles spread a system over up to 36
// workgroups and the chain is 2 launches per panel.
// Measured at P = 1025, d_t = 128, a workgroup per system -> now, ms: 16 systems
// 7.6 -> 0.77, 128 8.6 -> 3.25, 256 9.2 -> 6.3, 512 13.7 -> 12.4, 1,024 27.1 ->
// 24.4 (26 TFLOP/s; the trailing matrix moves about 33 MB per system); 64 in
// the fixed scratch 39.6 -> 2.6 (batches of 22 instead of 14).  Hundreds of
// narrower ones, us: P = 161 x 512 457 -> 301, 257 x 512 934 -> 627, 300 x 512
// 1,171 -> 876, 385 x 1,024 3,570 -> 2,851, 769 x 1,024 14,222 -> 12,551.  In "back", a
// panel column's operands requested one pair of blocks ahead instead of a whole
// column: 340 against 195 us for 22 systems.
//
// A pivot that is not positive and finite stops the system: info = its
// 1-based column, maps zero-filled (the report of the register solver).
//
// Workspace per system: block row i of U (128 rows from column 128 i on, the
// right-hand sides last) in strips of 16 columns, [strip][row][16], and
// lambda_m.  A strip's rows follow each other, so the operands of the products
// (4 rows of 16 columns, or 16 rows of 4) are 512 consecutive bytes: with rows
// of U after one another (9 KB apart at P = 1025) 16 rows fell on 4 of the 16 L2
// channels.  Systems are solved in batches that fit the workspace.
#include <algorithm>
#include <mutex>

#include "cb_solve_core.h"

namespace cb {
namespace {

constexpr int NB = 8;             // 16-row blocks of a panel
constexpr int NP = 16 * NB;       // panel rows
constexpr int DTMAX = 128;
constexpr int kComputeUnits = 256;

// Geometry of a system and its workspace.  Columns are numbered 0 .. N - 1
// (the factored part of M), then the d_t right-hand sides, then the bias
// column if it is kept apart (border).
struct WideArgs {
    const float *G, *C;
    const double *csums;          // centered form: (sum w, sum w x, sum w y), else null
    float *maps;
    int32_t *info;
    double *ws;
    int64_t ws_stride;            // doubles per system; the last one holds lambda_m
    float lambda;
    uint32_t flags;
    int32_t P, N, d_t, border, W; // W = N + d_t + border columns
    int32_t n, m0;                // systems of this batch, the first one
};

__host__ __device__ __forceinline__ int64_t row_base(const WideArgs &a, int i) {
    return (int64_t)NP * ((int64_t)a.W * i - (int64_t)NP * (i * (int64_t)(i - 1) / 2));
}
__host__ __device__ __forceinline__ int panel_rows(const WideArgs &a, int i) { return min(NP, a.N - NP * i); }

// Column `col` of block row i: row r of it is p[r * rs] (rs = 16 but in a last, narrower strip).
struct Column {
    double *p;
    int rs;
};
__device__ __forceinline__ Column column_of(const WideArgs &a, double *wm, int i, int col) {
    const int cc = col - NP * i, w = a.W - NP * i, s0 = cc & ~15;
    Column c;
    c.p = wm + row_base(a, i) + (int64_t)s0 * panel_rows(a, i) + (cc - s0);
    c.rs = min(16, w - s0);
    return c;
}

// The system of this workgroup and its work item: the items of a system run on
// one XCD (workgroups go round-robin over the eight), so what they share stays
// in its L2.  False past the end.
__device__ __forceinline__ bool item_of(const WideArgs &a, int items, int &m, int &item) {
    const int b = blockIdx.x, r = b >> 3;
    m = (r / items) * 8 + (b & 7);
    item = r % items;
    return m < a.n;
}

// Column `col` of [M | C | bias column] (lambda_m not included): row r of it is p[r * ld].
struct MomentColumn {
    const float *p;
    int64_t ld;
};
__device__ __forceinline__ MomentColumn moment_column(const WideArgs &a, int m, int col) {
    const bool rhs = col >= a.N && col < a.N + a.d_t;
    MomentColumn c;
    c.p = rhs ? a.C + (int64_t)(a.m0 + m) * a.P * a.d_t + (col - a.N)
              : a.G + (int64_t)(a.m0 + m) * a.P * a.P + (col < a.N ? col : a.P - 1);
    c.ld = rhs ? a.d_t : a.P;
    return c;
}

// The 128 x 128 block whose upper 16 x 16 blocks are in U (LDS) is factored in
// place (its first nblk block rows): U's blocks above the diagonal, L^-1 of the
// diagonal ones, D^(-1/2) in rsv.  Eight waves; returns (wave 0) the 1-based first failing pivot or 0.
__device__ __forceinline__ int factor_lds(double *U, double *rsv, int wave, int lane, int nblk) {
    const int q = lane & 15, g = lane >> 4;
    int bad = 0;
#pragma unroll 1
    for (int j = 0; j < nblk; ++j) {
        const int i = j + wave;
        f64x4_t am = {0.0, 0.0, 0.0, 0.0};
        if (wave == 0) {
            double *D = U + block_of(j, j) * kBS;
            if (j > 0) {
                // the last row's product; wave 7 took out those of the rows before
                const double *B = U + block_of(j - 1, j) * kBS + g * kBR + q;
                f64x4_t a0 = {0.0, 0.0, 0.0, 0.0}, a1 = {0.0, 0.0, 0.0, 0.0};
                double b[4], dv[4];
#pragma unroll
                for (int s = 0; s < 4; ++s) b[s] = B[4 * s * kBR];
#pragma unroll
                for (int e = 0; e < 4; ++e) dv[e] = D[(g + 4 * e) * kBR + q];
                a0 = mfma_f64(b[0], b[0], a0);
                a1 = mfma_f64(b[1], b[1], a1);
                a0 = mfma_f64(b[2], b[2], a0);
                a1 = mfma_f64(b[3], b[3], a1);
#pragma unroll
                for (int e = 0; e < 4; ++e) D[(g + 4 * e) * kBR + q] = dv[e] - (a0[e] + a1[e]);
            }
            double dk;
            const uint64_t wrong = factor_block<false>(D, nullptr, lane, dk);
            if (wrong && bad == 0) bad = 16 * j + __ffsll((unsigned long long)wrong);
            const double rs = rsqrt_f64(dk);
            if (g == 0) rsv[16 * j + q] = rs;
        } else if (wave == kWaves - 1 && j > 0) {
            if (j + 1 < nblk) {
                double *D = U + block_of(j + 1, j + 1) * kBS + g * kBR + q;
                for (int k = 0; k < j; ++k) {
                    const double *B = U + block_of(k, j + 1) * kBS + g * kBR + q;
#pragma unroll
                    for (int s = 0; s < 4; ++s) am = mfma_f64(B[4 * s * kBR], B[4 * s * kBR], am);
                }
#pragma unroll
                for (int e = 0; e < 4; ++e) D[4 * e * kBR] -= am[e];
            }
        } else if (i < nblk) {
            for (int k = 0; k < j; ++k) {
                const double *A = U + block_of(k, j) * kBS + g * kBR + q;
                const double *B = U + block_of(k, i) * kBS + g * kBR + q;
#pragma unroll
                for (int s = 0; s < 4; ++s) am = mfma_f64(A[4 * s * kBR], B[4 * s * kBR], am);
            }
            const double *T = U + block_of(j, i) * kBS + g * kBR + q;
#pragma unroll
            for (int e = 0; e < 4; ++e) am[e] = T[4 * e * kBR] - am[e];
        }
        __syncthreads();                                  // L_jj^-1 is published
        if (wave > 0 && i < nblk) {
            const double *V = U + block_of(j, j) * kBS + q * kBR + g;
            const double rs = rsv[16 * j + q];
            f64x4_t x = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
            for (int s = 0; s < 4; ++s) x = mfma_f64(V[4 * s] * rs, am[s], x);
            double *T = U + block_of(j, i) * kBS + g * kBR + q;
#pragma unroll
            for (int e = 0; e < 4; ++e) T[4 * e * kBR] = x[e];
        }
        __syncthreads();                                  // row j of U is published
    }
    return bad;
}

// Factor the diagonal block of panel p (its upper blocks in LDS, rows and
// columns past nb as in the identity) and write it to the workspace, the
// diagonal 16 x 16 blocks as V = D^(-1/2) L^-1.
__device__ __forceinline__ void finish_diagonal(const WideArgs &a, double *U, double *rsv, double *wm, int m, int p,
                                                int nb, int tid, bool first) {
    const int lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int bad = factor_lds(U, rsv, wave, lane, (nb + 15) / 16);
    if (tid == 0 && (bad || first)) a.info[a.m0 + m] = bad ? NP * p + bad : 0;
    for (int e = tid; e < NP * NP; e += kThreads) {
        const int c = 16 * (e / (16 * NP)) + e % 16, r = e / 16 % NP;   // a strip at a time
        if (c / 16 < r / 16 || r >= nb || c >= nb) continue;
        double v = U[block_of(r / 16, c / 16) * kBS + (r % 16) * kBR + c % 16];
        if (r / 16 == c / 16) v *= rsv[r];
        const Column x = column_of(a, wm, p, NP * p + c);
        x.p[r * x.rs] = v;
    }
}

__global__ __launch_bounds__(kThreads, 4) void wide_first_kernel(WideArgs a) {
    __shared__ double U[NB * (NB + 1) / 2 * kBS];
    __shared__ double rsv[NP];
    __shared__ double red[kWaves];
    const int m = blockIdx.x, tid = threadIdx.x;
    const float *Gm = a.G + (int64_t)(a.m0 + m) * a.P * a.P;
    const double *sm = a.csums ? a.csums + (int64_t)(a.m0 + m) * (1 + a.P + a.d_t) : nullptr;
    const double sw = sm ? sm[0] : 0.0;
    double tr = 0.0;
    for (int i = tid; i < a.P; i += kThreads) {
        tr += (double)Gm[(int64_t)i * a.P + i];
        if (sm && sw != 0.0) tr += sm[1 + i] * (sm[1 + i] / sw);             // S mu_i^2
    }
    for (int o = 32; o > 0; o >>= 1) tr += __shfl_xor(tr, o);
    if ((tid & 63) == 0) red[tid >> 6] = tr;
    // the first diagonal block, the identity past the matrix
    constexpr int QN = NP * NP / kThreads;
    const int nb = min(NP, a.N);
#pragma unroll 8
    for (int n = 0; n < QN; ++n) {
        const int e = n * kThreads + tid, r = e / NP, c = e % NP;
        const float v = Gm[(int64_t)min(r, nb - 1) * a.P + min(c, nb - 1)];
        if (c / 16 >= r / 16)
            U[block_of(r / 16, c / 16) * kBS + (r % 16) * kBR + c % 16] =
                r < nb && c < nb ? (double)v : (r == c ? 1.0 : 0.0);
    }
    __syncthreads();
    double trace = sw;
#pragma unroll
    for (int w = 0; w < kWaves; ++w) trace += red[w];
    const double lam = (a.flags & CB_LAMBDA_RELATIVE) ? (double)a.lambda * trace / (double)(sm ? a.P + 1 : a.P)
                                                      : (double)a.lambda;
    double *wm = a.ws + (int64_t)m * a.ws_stride;
    if (tid == 0) wm[a.ws_stride - 1] = lam;
    const int pen = (!sm && (a.flags & CB_RIDGE_BIAS_UNPENALIZED)) ? a.P - 1 : a.P;   // entries < pen get lambda
    if (tid < nb && tid < pen) U[block_of(tid / 16, tid / 16) * kBS + (tid % 16) * (kBR + 1)] += lam;
    __syncthreads();
    finish_diagonal(a, U, rsv, wm, m, 0, nb, tid, true);
}

// Columns right of panel p in groups of 128: the rest of M, then the
// right-hand sides and the bias column.
__host__ __device__ __forceinline__ int groups_right_of(const WideArgs &a, int p) {
    const int c1 = min(NP * (p + 1), a.N);
    return (a.N - c1 + NP - 1) / NP + (a.d_t + a.border + NP - 1) / NP;
}
__device__ __forceinline__ void group_columns(const WideArgs &a, int p, int grp, int &col0, int &ncol) {
    const int c1 = min(NP * (p + 1), a.N), gm = (a.N - c1 + NP - 1) / NP;
    if (grp < gm) {
        col0 = c1 + NP * grp;
        ncol = min(NP, a.N - col0);
    } else {
        col0 = a.N + NP * (grp - gm);
        ncol = min(NP, a.W - col0);
    }
}

// The upper blocks of panel p's diagonal tile into LDS (the identity past its nb rows).
__device__ __forceinline__ void load_diagonal(const WideArgs &a, double *U, double *wm, int p, int tid) {
    const int nb = panel_rows(a, p);
#pragma unroll
    for (int n = 0; n < NB * (NB + 1) / 2 * 256 / kThreads; ++n) {
        const int e = n * kThreads + tid, b = e >> 8, r = (e >> 4) & 15, c = e & 15;
        int i = 0;
#pragma unroll
        for (int x = 1; x < NB; ++x) i += b >= x * (x + 1) / 2;
        const int k = b - i * (i + 1) / 2, R = 16 * k + r, Cc = 16 * i + c;
        const Column x = column_of(a, wm, p, NP * p + min(Cc, nb - 1));
        const double v = x.p[min(R, nb - 1) * x.rs];
        U[b * kBS + r * kBR + c] = R < nb && Cc < nb ? v : (R == Cc ? 1.0 : 0.0);
    }
}

// U_p,c = U_pp^-T T_p,c for one group of columns; wave w has tile w.
__global__ __launch_bounds__(kThreads, 4) void wide_solve_kernel(WideArgs a, int p) {
    __shared__ double U[NB * (NB + 1) / 2 * kBS];
    int m, grp, col0, ncol;
    if (!item_of(a, groups_right_of(a, p), m, grp)) return;
    if (a.info[a.m0 + m] != 0) return;
    group_columns(a, p, grp, col0, ncol);
    const int tid = threadIdx.x, lane = tid & 63, q = lane & 15, g = lane >> 4;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    double *wm = a.ws + (int64_t)m * a.ws_stride;
    const int nb = panel_rows(a, p);
    const bool own = 16 * wave < ncol;
    const int col = min(col0 + 16 * wave + q, col0 + ncol - 1);
    const Column T = column_of(a, wm, p, col);

    f64x4_t Z[NB];
    if (own) {
        if (p == 0) {
            const MomentColumn mc = moment_column(a, m, col);
#pragma unroll
            for (int j = 0; j < NB; ++j)
#pragma unroll
                for (int e = 0; e < 4; ++e) Z[j][e] = (double)mc.p[min(16 * j + 4 * e + g, nb - 1) * mc.ld];
        } else {
#pragma unroll
            for (int j = 0; j < NB; ++j)
#pragma unroll
                for (int e = 0; e < 4; ++e) Z[j][e] = T.p[min(16 * j + 4 * e + g, nb - 1) * T.rs];
        }
    }
    load_diagonal(a, U, wm, p, tid);
    __syncthreads();
    if (!own) return;
#pragma unroll
    for (int j = 0; j < NB; ++j) {
        if (16 * j >= nb) return;                         // a partial last panel
        int q = tid & 15, g = (tid >> 4) & 3;
        asm volatile("" : "+v"(q), "+v"(g));              // addresses are formed in the row that uses them
        f64x4_t acc = {0.0, 0.0, 0.0, 0.0}, x = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
        for (int k = 0; k < j; ++k)
#pragma unroll
            for (int s = 0; s < 4; ++s) acc = mfma_f64(U[block_of(k, j) * kBS + (4 * s + g) * kBR + q], Z[k][s], acc);
        f64x4_t y = Z[j] - acc;
#pragma unroll
        for (int e = 0; e < 4; ++e) y[e] = 16 * j + 4 * e + g < nb ? y[e] : 0.0;
#pragma unroll
        for (int s = 0; s < 4; ++s) x = mfma_f64(U[block_of(j, j) * kBS + q * kBR + 4 * s + g], y[s], x);
        Z[j] = x;
        if (col0 + 16 * wave + q < col0 + ncol) {
#pragma unroll
            for (int e = 0; e < 4; ++e)
                if (16 * j + 4 * e + g < nb) T.p[(16 * j + 4 * e + g) * T.rs] = x[e];
        }
    }
}

// Work items of the update after panel p: block rows i > p, for each the
// groups of columns from its own diagonal on.  Item 0 is the next diagonal tile.
__host__ __device__ __forceinline__ int update_items(const WideArgs &a, int p) {
    int t = 0;
    for (int i = p + 1; i < (a.N + NP - 1) / NP; ++i) t += groups_right_of(a, i) + 1;
    return t;
}

// T_i,c -= U_p,i^T U_p,c for one 128 x 128 tile; wave w has its 32 rows 32 (w / 2) and its 64 columns 64 (w mod 2).
__global__ __launch_bounds__(kThreads, 4) void wide_update_kernel(WideArgs a, int p, int items) {
    __shared__ double U[NB * (NB + 1) / 2 * kBS];
    __shared__ double rsv[NP];
    int m, item;
    if (!item_of(a, items, m, item)) return;
    if (a.info[a.m0 + m] != 0) return;
    int i = p + 1, grp = item;
    while (grp > groups_right_of(a, i)) {
        grp -= groups_right_of(a, i) + 1;
        ++i;
    }
    int col0 = NP * i, ncol = min(NP, a.N - NP * i);
    const int nr = ncol;                                  // rows of block row i
    if (grp > 0) group_columns(a, i, grp - 1, col0, ncol);
    const bool diagonal = grp == 0, factor = diagonal && i == p + 1;
    const int tid = threadIdx.x, lane = tid & 63, q = lane & 15, g = lane >> 4;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int r0 = 32 * (wave >> 1), x0 = 64 * (wave & 1);   // rows and columns within the tile
    double *wm = a.ws + (int64_t)m * a.ws_stride;
    const bool live = r0 < nr && x0 < ncol && !(diagonal && x0 + 64 <= r0);
    f64x4_t acc[2][4];
    if (live) {
#pragma unroll
        for (int x = 0; x < 2; ++x)
#pragma unroll
            for (int y = 0; y < 4; ++y) acc[x][y] = f64x4_t{0.0, 0.0, 0.0, 0.0};
        // operands straight from the workspace (L2): row k of U_p, 16 consecutive columns per 16 lanes, requested
        // one pair of K steps ahead
        Column ca[2], cx[4];
#pragma unroll
        for (int x = 0; x < 2; ++x) ca[x] = column_of(a, wm, p, NP * i + min(r0 + 16 * x + q, nr - 1));
#pragma unroll
        for (int y = 0; y < 4; ++y) cx[y] = column_of(a, wm, p, col0 + min(x0 + 16 * y + q, ncol - 1));
        double av[2][2][2], bv[2][2][4];
        auto fetch = [&](int buf, int s) __attribute__((always_inline)) {
#pragma unroll
            for (int h = 0; h < 2; ++h) {
#pragma unroll
                for (int x = 0; x < 2; ++x) av[buf][h][x] = ca[x].p[(4 * (s + h) + g) * ca[x].rs];
#pragma unroll
                for (int y = 0; y < 4; ++y) bv[buf][h][y] = cx[y].p[(4 * (s + h) + g) * cx[y].rs];
            }
        };
        fetch(0, 0);
#pragma unroll 2
        for (int s = 0; s < NP / 4; s += 2) {
            const int buf = (s >> 1) & 1;
            fetch(buf ^ 1, s + 2 < NP / 4 ? s + 2 : 0);   // (past the end: the first pair again, unused)
#pragma unroll
            for (int h = 0; h < 2; ++h)
#pragma unroll
                for (int x = 0; x < 2; ++x)
#pragma unroll
                    for (int y = 0; y < 4; ++y) acc[x][y] = mfma_f64(av[buf][h][x], bv[buf][h][y], acc[x][y]);
        }
        // T - acc, from the moments after the first panel and from the workspace after the others; eight elements at
        // a time are requested together (rows and columns past the tile's repeat its last)
        const double lam = wm[a.ws_stride - 1];
        const int pen = (!a.csums && (a.flags & CB_RIDGE_BIAS_UNPENALIZED)) ? a.P - 1 : a.P;
#pragma unroll
        for (int y = 0; y < 4; ++y) {
            const int c = x0 + 16 * y + q, cl = col0 + min(c, ncol - 1);
            const Column T = column_of(a, wm, i, cl);
            double t[2][4];
            if (p == 0) {
                const MomentColumn mc = moment_column(a, m, cl);
                float f[2][4];
#pragma unroll
                for (int x = 0; x < 2; ++x)
#pragma unroll
                    for (int e = 0; e < 4; ++e)
                        f[x][e] = mc.p[(int64_t)(NP * i + min(r0 + 16 * x + 4 * e + g, nr - 1)) * mc.ld];
#pragma unroll
                for (int x = 0; x < 2; ++x)
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        const int row = NP * i + r0 + 16 * x + 4 * e + g;
                        t[x][e] = (double)f[x][e] + (row == cl && row < pen ? lam : 0.0);
                    }
            } else {
#pragma unroll
                for (int x = 0; x < 2; ++x)
#pragma unroll
                    for (int e = 0; e < 4; ++e)
                        t[x][e] = T.p[min(r0 + 16 * x + 4 * e + g, nr - 1) * T.rs];
            }
#pragma unroll
            for (int x = 0; x < 2; ++x)
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const int r = r0 + 16 * x + 4 * e + g;
                    const double v = t[x][e] - acc[x][y][e];
                    if (diagonal && c / 16 < r / 16) continue;
                    if (factor)
                        U[block_of(r / 16, c / 16) * kBS + (r % 16) * kBR + c % 16] =
                            r < nr && c < nr ? v : (r == c ? 1.0 : 0.0);
                    else if (r < nr && c < ncol)
                        T.p[r * T.rs] = v;
                }
        }
    }
    if (!factor) return;
    // (a partial last block: waves past its rows or columns fill in the identity)
    if (!live && !(x0 + 64 <= r0)) {
        for (int x = 0; x < 2; ++x)
            for (int y = 0; y < 4; ++y)
                for (int e = 0; e < 4; ++e) {
                    const int r = r0 + 16 * x + 4 * e + g, c = x0 + 16 * y + q;
                    if (c / 16 >= r / 16)
                        U[block_of(r / 16, c / 16) * kBS + (r % 16) * kBR + c % 16] = r == c ? 1.0 : 0.0;
                }
    }
    __syncthreads();
    finish_diagonal(a, U, rsv, wm, m, p + 1, nr, tid, false);
}

// This wave's LDS accesses have completed, then the workgroup barrier; loads
// from global memory stay in flight across it.
__device__ __forceinline__ void lds_sync() {
    asm volatile("" ::: "memory");
    __builtin_amdgcn_s_waitcnt(0xC07F);   // lgkmcnt(0); vmcnt, expcnt untouched
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
}

// Back substitution of 16 right-hand sides from the last panel up; wave w has
// rows 16 w .. + 15 of a panel.
__global__ __launch_bounds__(kThreads, 2) void wide_back_kernel(WideArgs a) {
    __shared__ double Wl[2][16 * 17], Wk[2][NP * 17];
    __shared__ double red[kWaves][16];
    __shared__ double redh[kWaves];
    __shared__ int s_info;
    int m, tile;
    if (!item_of(a, a.d_t / 16, m, tile)) return;
    const int tid = threadIdx.x, lane = tid & 63, q = lane & 15, g = lane >> 4;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int c = 16 * tile + q, out_rows = a.csums ? a.P + 1 : a.P;
    double *wm = a.ws + (int64_t)m * a.ws_stride;
    const float *Gm = a.G + (int64_t)(a.m0 + m) * a.P * a.P, *Cm = a.C + (int64_t)(a.m0 + m) * a.P * a.d_t;
    float *Wm = a.maps + (int64_t)(a.m0 + m) * out_rows * a.d_t;
    // info is read once per workgroup: another workgroup of the system may store the bias pivot's failure while this
    // one starts, and its waves have to agree (this workgroup finds the same pivot, so either reading serves)
    if (tid == 0) s_info = __hip_atomic_load(a.info + a.m0 + m, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    __syncthreads();
    bool bad = s_info != 0;
    double wb = 0.0;                                      // border: this column's bias coefficient
    if (a.border && !bad) {
        // h = M_NN - z . z and (C_N - z . Z) / h with z the bias column's eliminated values
        double zz = 0.0, zc = 0.0;
        for (int r = 4 * wave + g; r < a.N; r += 4 * kWaves) {
            const int i = r / NP;
            const Column b = column_of(a, wm, i, a.W - 1), x = column_of(a, wm, i, a.N + c);
            const double z = b.p[(r - NP * i) * b.rs];
            zz = __builtin_fma(z, z, zz);
            zc = __builtin_fma(z, x.p[(r - NP * i) * x.rs], zc);
        }
        for (int o = 16; o < 64; o <<= 1) {
            zz += __shfl_xor(zz, o);
            zc += __shfl_xor(zc, o);
        }
        if (g == 0) red[wave][q] = zc;
        if (lane == 0) redh[wave] = zz;
        __syncthreads();
        double h = 0.0, s = 0.0;
#pragma unroll
        for (int w = 0; w < kWaves; ++w) {
            h += redh[w];
            s += red[w][q];
        }
        const bool pen = a.csums || !(a.flags & CB_RIDGE_BIAS_UNPENALIZED);
        h = (double)Gm[(int64_t)a.N * a.P + a.N] + (pen ? wm[a.ws_stride - 1] : 0.0) - h;
        bad = !(h > 0.0 && h <= DBL_MAX);                 // the same in every workgroup of the system
        if (bad) {
            if (tid == 0) __hip_atomic_store(a.info + a.m0 + m, a.N + 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        } else {
            wb = ((double)Cm[(int64_t)a.N * a.d_t + c] - s) / h;
        }
    }
    if (bad) {
        for (int r = 4 * wave + g; r < out_rows; r += 4 * kWaves) Wm[(int64_t)r * a.d_t + c] = 0.f;
        return;
    }
    double mu_sum = 0.0;                                  // centered: sum of mu_x,i W_ic over this lane's rows
    const double *sm = a.csums ? a.csums + (int64_t)(a.m0 + m) * (1 + a.P + a.d_t) : nullptr;
    const double sw = sm ? sm[0] : 0.0;
    // One workgroup streams the whole factor past 16 columns, so its speed is that of the requests in flight (they
    // come from beyond L2): a wave's U blocks of a panel column are requested a whole panel of 128 columns ahead, the
    // panel's own blocks before the products of the columns right of it.
    const int panels = (a.N + NP - 1) / NP;
    double av[4][8], uv[NB][4], vv[4], wn[4];
    // two blocks of 16 columns from column k0 on of this wave's rows of panel i; K step s of a block takes its
    // columns 4 g + s (32 consecutive bytes a lane).  (Strips that hold columns of M are 16 wide: d_t >= 64 columns
    // follow them.  Columns past N are read as some of those and masked where they are used.)
    auto fetch = [&](double (&x)[8], int i, int k0) __attribute__((always_inline)) {
        const int nb = panel_rows(a, i), last = (a.N - 1 - NP * i) >> 4;
        const double *A = wm + row_base(a, i) + 16 * min(16 * wave + q, nb - 1) + 4 * g;
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            const double *S = A + (int64_t)16 * nb * min(((k0 - NP * i) >> 4) + h, last);
#pragma unroll
            for (int s = 0; s < 4; ++s) x[4 * h + s] = S[s];
        }
    };
    for (int i = panels - 1; i >= 0; --i) {
        const int nb = panel_rows(a, i), top = (nb - 1) >> 4;
        const Column X = column_of(a, wm, i, a.N + c);    // this lane's right-hand side
        const bool live = 16 * wave < nb;
        auto rows_of = [&](int ik) __attribute__((always_inline)) {
            const int r = min(tid >> 2, panel_rows(a, ik) - 1);
#pragma unroll
            for (int s = 0; s < 4; ++s) {
                const Column w = column_of(a, wm, ik, a.N + 16 * tile + 4 * (tid & 3) + s);
                wn[s] = w.p[r * w.rs];
            }
        };
        rows_of(min(i + 1, panels - 1));                  // first: the loop's wait for it must not cover the rest
        __builtin_amdgcn_sched_barrier(0);
        // the panel's own blocks right of this wave's rows, V of its rows, Z and the bias column's z
        const double *own = wm + row_base(a, i);
#pragma unroll
        for (int l = 1; l < NB; ++l)
#pragma unroll
            for (int s = 0; s < 4; ++s)
                uv[l][s] = own[(int64_t)16 * nb * min(l, top) + 16 * min(16 * wave + q, nb - 1) + 4 * g + s];
#pragma unroll
        for (int s = 0; s < 4; ++s)
            vv[s] = own[(int64_t)16 * nb * min(wave, top) + 16 * min(16 * wave + 4 * s + g, nb - 1) + q];
        f64x4_t R, acc[2];
        acc[0] = acc[1] = f64x4_t{0.0, 0.0, 0.0, 0.0};
#pragma unroll
        for (int e = 0; e < 4; ++e) R[e] = X.p[min(16 * wave + 4 * e + g, nb - 1) * X.rs];
        const Column bias = column_of(a, wm, i, a.W - 1);  // (without a bias column: a right-hand side, not used)
        double zb[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) zb[e] = bias.p[min(16 * wave + 4 * e + g, nb - 1) * bias.rs];
        // minus the sum over the columns right of the panel: the 128 solved rows of one panel at a time, shared by
        // the waves through LDS (rows past N as zero)
        for (int ik = i + 1; ik < panels; ++ik) {
            double *B = Wk[ik & 1];
            const bool more = ik + 1 < panels;
            const int fi = more ? i : max(i - 1, 0), fk = more ? NP * (ik + 1) : NP * max(i, 1);
            const bool in = (tid >> 2) < panel_rows(a, ik);
#pragma unroll
            for (int s = 0; s < 4; ++s) B[(tid >> 2) * 17 + 4 * (tid & 3) + s] = in ? wn[s] : 0.0;
            lds_sync();                                   // (two buffers: everyone is past the last but one)
            rows_of(min(ik + 1, panels - 1));
#pragma unroll
            for (int h = 0; h < 4; ++h) {
                __builtin_amdgcn_sched_barrier(0);        // (reads of one pair of blocks at a time: registers)
#pragma unroll
                for (int s = 0; s < 8; ++s) {
                    const int k = 32 * h + 16 * (s >> 2) + 4 * g + (s & 3);
                    acc[s & 1] = mfma_f64(NP * ik + k < a.N ? av[h][s] : 0.0, B[k * 17 + q], acc[s & 1]);
                }
                // the same columns of the next panel column; after the last, the first ones of the panel above (of
                // panel 0 again at the end, unused).  No branch: its loads would be waited for at the join.
                fetch(av[h], fi, fk + 32 * h);
            }
        }
        if (i + 1 == panels) {
#pragma unroll
            for (int h = 0; h < 4; ++h) fetch(av[h], max(i - 1, 0), NP * max(i, 1) + 32 * h);
        }
        R -= acc[0] + acc[1];
        if (a.border) {
#pragma unroll
            for (int e = 0; e < 4; ++e) R[e] = __builtin_fma(-zb[e], wb, R[e]);
        }
        // within the panel, 16 rows at a time from the bottom: W_l = V_l^T R_l, published to the waves above
#pragma unroll
        for (int l = NB - 1; l >= 0; --l) {
            if (l > top) continue;                        // the same in every wave
            __builtin_amdgcn_sched_barrier(0);
            double *pub = Wl[l & 1];
            if (wave == l) {
                f64x4_t x = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
                for (int s = 0; s < 4; ++s) {
                    const bool in = 16 * l + 4 * s + g < nb && 16 * l + q < nb;
                    x = mfma_f64(in ? vv[s] : 0.0, R[s], x);
                }
#pragma unroll
                for (int e = 0; e < 4; ++e) pub[(4 * e + g) * 17 + q] = x[e];
                R = x;
            }
            if (l == 0) continue;
            lds_sync();
            if (wave < l) {
                f64x4_t x = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
                for (int s = 0; s < 4; ++s)
                    x = mfma_f64(16 * l + 4 * g + s < nb ? uv[l][s] : 0.0, pub[(4 * g + s) * 17 + q], x);
                R -= x;
            }
        }
        if (live) {
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const int r = 16 * wave + 4 * e + g;
                if (r >= nb) continue;
                X.p[r * X.rs] = R[e];                     // read by the panels above
                Wm[(int64_t)(NP * i + r) * a.d_t + c] = (float)R[e];
                if (sm && sw != 0.0) mu_sum = __builtin_fma(sm[1 + NP * i + r] / sw, R[e], mu_sum);
            }
        }
        __syncthreads();
    }
    // (after the barriers above: the caller may solve in place, maps = C, and every wave reads C's last row)
    if (a.border && wave == 0 && g == 0) Wm[(int64_t)a.N * a.d_t + c] = (float)wb;
    if (sm) {
        // b = mu_y - W^T mu_x (the bias unknown of a border system is a feature like the others here)
        if (a.border && sw != 0.0 && wave == 0 && g == 0) mu_sum = __builtin_fma(sm[1 + a.N] / sw, wb, mu_sum);
        mu_sum += __shfl_xor(mu_sum, 16);
        mu_sum += __shfl_xor(mu_sum, 32);
        if (g == 0) red[wave][q] = mu_sum;
        __syncthreads();
        if (wave == 0 && g == 0) {
            double b = sw != 0.0 ? sm[1 + a.P + c] / sw : 0.0;
#pragma unroll
            for (int w = 0; w < kWaves; ++w) b -= red[w][q];
            Wm[(int64_t)a.P * a.d_t + c] = (float)b;
        }
    }
}

// The same back substitution with a system per workgroup: wave w has the 16 right-hand sides 16 w .. + 15 of every
// panel in its registers, as in wide_solve_kernel, so within a panel there is no barrier, the factor comes past once
// for all right-hand sides and two workgroups share a compute unit.
__global__ __launch_bounds__(kThreads, 4) void wide_back_system_kernel(WideArgs a) {
    __shared__ double U[NB * (NB + 1) / 2 * kBS];
    __shared__ int s_info;
    const int m = blockIdx.x, tid = threadIdx.x, lane = tid & 63, q = lane & 15, g = lane >> 4;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const bool own = 16 * wave < a.d_t;
    const int c = 16 * (own ? wave : 0) + q, out_rows = a.csums ? a.P + 1 : a.P, panels = (a.N + NP - 1) / NP;
    double *wm = a.ws + (int64_t)m * a.ws_stride;
    float *Wm = a.maps + (int64_t)(a.m0 + m) * out_rows * a.d_t;
    if (tid == 0) s_info = a.info[a.m0 + m];
    __syncthreads();
    bool bad = s_info != 0;
    double wb = 0.0;                                      // border: this column's bias coefficient
    if (a.border && !bad) {
        // h = M_NN - z . z and (C_N - z . Z) / h with z the bias column's eliminated values (N = 128 panels here)
        double zz = 0.0, zc = 0.0;
        for (int i = 0; i < panels; ++i) {
            const Column b = column_of(a, wm, i, a.W - 1), x = column_of(a, wm, i, a.N + c);
#pragma unroll 8
            for (int r = g; r < NP; r += 4) {
                const double z = b.p[r * b.rs];
                zz = __builtin_fma(z, z, zz);
                zc = __builtin_fma(z, x.p[r * x.rs], zc);
            }
        }
        for (int o = 16; o < 64; o <<= 1) {
            zz += __shfl_xor(zz, o);
            zc += __shfl_xor(zc, o);
        }
        const bool pen = a.csums || !(a.flags & CB_RIDGE_BIAS_UNPENALIZED);
        const double gnn = (double)a.G[((int64_t)(a.m0 + m) * a.P + a.N) * a.P + a.N];
        const double h = gnn + (pen ? wm[a.ws_stride - 1] : 0.0) - zz;
        bad = !(h > 0.0 && h <= DBL_MAX);                 // the same in every wave
        wb = ((double)a.C[((int64_t)(a.m0 + m) * a.P + a.N) * a.d_t + c] - zc) / h;
        if (bad && tid == 0) a.info[a.m0 + m] = a.N + 1;
    }
    if (bad) {
        for (int e = tid; e < out_rows * a.d_t; e += kThreads) Wm[e] = 0.f;
        return;
    }
    double mu_sum = 0.0;                                  // centered: sum of mu_x,i W_ic over this lane's rows
    const double *sm = a.csums ? a.csums + (int64_t)(a.m0 + m) * (1 + a.P + a.d_t) : nullptr;
    const double sw = sm ? sm[0] : 0.0;
    for (int i = panels - 1; i >= 0; --i) {
        const int nb = panel_rows(a, i);
        if (i + 1 < panels) __syncthreads();              // everyone is done with the last panel's U
        int t = tid;
        asm volatile("" : "+v"(t));                       // nothing of the panel's addresses is held across the loop
        load_diagonal(a, U, wm, i, t);
        asm volatile("" : "+v"(t)::"memory");
        const Column X = column_of(a, wm, i, a.N + 16 * (own ? wave : 0) + (t & 15));
        f64x4_t Z[NB];
#pragma unroll
        for (int j = 0; j < NB; ++j) Z[j] = f64x4_t{0.0, 0.0, 0.0, 0.0};
        if (own) {
            // the columns right of the panel (only panels of 128 rows have any), 16 at a time; K step s of a block takes
            // its columns 4 g + s: 32 consecutive bytes a lane of U, row 4 g + s of this wave's solved right-hand sides
#pragma unroll 1
            for (int k0 = NP * (i + 1); k0 < a.N; k0 += 16) {
                int q = tid & 15, g = (tid >> 4) & 3;
                asm volatile("" : "+v"(q), "+v"(g));      // addresses are formed here, not held across the loop
                const int ik = k0 / NP, last = panel_rows(a, ik) - 1;
                const Column B = column_of(a, wm, ik, a.N + c);
                const double *S = wm + row_base(a, i) + (int64_t)NP * (k0 - NP * i) + 16 * q + 4 * g;
                double b[4];
#pragma unroll
                for (int s = 0; s < 4; ++s) b[s] = B.p[min(k0 - NP * ik + 4 * g + s, last) * B.rs];
#pragma unroll
                for (int s = 0; s < 4; ++s) b[s] = k0 + 4 * g + s < a.N ? b[s] : 0.0;
#pragma unroll
                for (int j0 = 0; j0 < NB; j0 += 4) {
                    double u[4][4];
#pragma unroll
                    for (int j = 0; j < 4; ++j)
#pragma unroll
                        for (int s = 0; s < 4; ++s) u[j][s] = S[256 * (j0 + j) + s];
#pragma unroll
                    for (int s = 0; s < 4; ++s)
#pragma unroll
                        for (int j = 0; j < 4; ++j)
                            Z[j0 + j] = mfma_f64(k0 + 4 * g + s < a.N ? u[j][s] : 0.0, b[s], Z[j0 + j]);
                }
            }
            const Column bias = column_of(a, wm, i, a.W - 1);
#pragma unroll
            for (int j = 0; j < NB; ++j) {
                int g = (tid >> 4) & 3;
                asm volatile("" : "+v"(g)::"memory");     // four rows' loads at a time: registers
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const int r = 16 * j + 4 * e + g;
                    double y = X.p[min(r, nb - 1) * X.rs] - Z[j][e];
                    if (a.border) y = __builtin_fma(-bias.p[min(r, nb - 1) * bias.rs], wb, y);
                    Z[j][e] = r < nb ? y : 0.0;
                }
            }
        }
        __syncthreads();
        if (!own) continue;
#pragma unroll
        for (int j = NB - 1; j >= 0; --j) {
            if (16 * j >= nb) continue;
            int q = tid & 15, g = (tid >> 4) & 3;
            asm volatile("" : "+v"(q), "+v"(g));
            f64x4_t acc = {0.0, 0.0, 0.0, 0.0}, x = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
            for (int k = j + 1; k < NB; ++k)
#pragma unroll
                for (int s = 0; s < 4; ++s) acc = mfma_f64(U[block_of(j, k) * kBS + q * kBR + 4 * s + g], Z[k][s], acc);
            const f64x4_t y = Z[j] - acc;
#pragma unroll
            for (int s = 0; s < 4; ++s) x = mfma_f64(U[block_of(j, j) * kBS + (4 * s + g) * kBR + q], y[s], x);
            Z[j] = x;
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const int r = 16 * j + 4 * e + g;
                if (r >= nb) continue;
                X.p[r * X.rs] = x[e];                     // read by the panels above
                Wm[(int64_t)(NP * i + r) * a.d_t + c] = (float)x[e];
                if (sm && sw != 0.0) mu_sum = __builtin_fma(sm[1 + NP * i + r] / sw, x[e], mu_sum);
            }
        }
    }
    if (!own) return;
    if (a.border && g == 0) Wm[(int64_t)a.N * a.d_t + c] = (float)wb;
    if (sm) {
        // b = mu_y - W^T mu_x (the bias unknown of a border system is a feature like the others here)
        if (a.border && sw != 0.0 && g == 0) mu_sum = __builtin_fma(sm[1 + a.N] / sw, wb, mu_sum);
        mu_sum += __shfl_xor(mu_sum, 16);
        mu_sum += __shfl_xor(mu_sum, 32);
        if (g == 0) Wm[(int64_t)a.P * a.d_t + c] = (float)((sw != 0.0 ? sm[1 + a.P + c] / sw : 0.0) - mu_sum);
    }
}

WideArgs geometry(int32_t P, int32_t d_t) {
    WideArgs a = {};
    a.P = P;
    a.d_t = d_t;
    a.border = P % NP == 1;
    a.N = P - a.border;
    a.W = a.N + d_t + a.border;
    return a;
}

// Doubles of one system's workspace: the block rows of U and lambda_m.  Never more than solve_blocked_bytes_per_system
// (each block row drops the columns left of its diagonal block, 128 of them from the second on; P > 129).
int64_t system_doubles(const WideArgs &a) {
    const int last = (a.N + NP - 1) / NP - 1;
    return row_base(a, last) + (int64_t)(a.N - NP * last) * (a.W - NP * last) + 1;
}

}  // namespace

int64_t solve_blocked_bytes_per_system(int32_t P, int32_t d_t) {
    return ((int64_t)P * P + (int64_t)P * d_t) * (int64_t)sizeof(double);
}

hipError_t launch_solve_blocked(int32_t n_maps, int32_t P, int32_t d_t, const float *G, const float *C, float lambda,
                                uint32_t flags, void *ws, int64_t ws_bytes, float *maps, int32_t *info,
                                hipStream_t s, const double *csums) {
    if (n_maps == 0) return hipSuccess;
    if (d_t > DTMAX || d_t % 16 != 0 || P <= NP) return hipErrorInvalidValue;
    WideArgs a = geometry(P, d_t);
    const int64_t told = solve_blocked_bytes_per_system(P, d_t) / (int64_t)sizeof(double);
    a.ws_stride = (system_doubles(a) + 15) / 16 * 16;     // strips on 128-byte lines
    if (a.ws_stride > told) a.ws_stride = system_doubles(a);
    a.G = G;
    a.C = C;
    a.csums = csums;
    a.maps = maps;
    a.info = info;
    a.ws = (double *)ws;
    a.lambda = lambda;
    a.flags = flags;
    const int64_t batch = std::min<int64_t>(ws_bytes / (8 * a.ws_stride), 1 << 16);
    if (batch < 1) return hipErrorInvalidValue;
    const int panels = (a.N + NP - 1) / NP;
    for (int32_t m0 = 0; m0 < n_maps; m0 += a.n) {
        a.m0 = m0;
        a.n = (int32_t)std::min<int64_t>(batch, n_maps - m0);
        const int64_t n8 = (a.n + 7) / 8 * 8;
        hipLaunchKernelGGL(wide_first_kernel, dim3(a.n), dim3(kThreads), 0, s, a);
        for (int p = 0; p < panels; ++p) {
            hipLaunchKernelGGL(wide_solve_kernel, dim3((unsigned)(n8 * groups_right_of(a, p))), dim3(kThreads), 0, s,
                               a, p);
            const int items = update_items(a, p);
            if (items > 0)
                hipLaunchKernelGGL(wide_update_kernel, dim3((unsigned)(n8 * items)), dim3(kThreads), 0, s, a, p, items);
        }
        // A system per workgroup where they fill the chip, up to six panels.  Measured, whole solve at d_t = 128,
        // workgroup per 16 right-hand sides -> per system, us: P = 161 x 512 553 -> 301, 257 x 256 483 -> 360, 300 x
        // 512 1,243 -> 876, 513 x 256 1,565 -> 1,417, 769 x 256 3,440 -> 3,357; with more panels or fewer systems it
        // is the chain of one workgroup: 1,025 x 256 6,344 -> 6,400, 257 x 64 179 -> 231, 513 x 64 483 -> 756.
        if (a.n >= kComputeUnits && panels <= 6)
            hipLaunchKernelGGL(wide_back_system_kernel, dim3(a.n), dim3(kThreads), 0, s, a);
        else
            hipLaunchKernelGGL(wide_back_kernel, dim3((unsigned)(n8 * (d_t / 16))), dim3(kThreads), 0, s, a);
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

// Allocation-free variant: the factors live in `scratch`, a fixed device array
// that the code object carries (every GPU the library runs on holds its own
// copy until the process ends).  Its device address is looked up once per
// device, with that device current, on the first call there; host code never
// passes the array's name itself to a kernel (on the host it only names the
// variable).  Calls that overlap on one GPU share the array and race.
static __device__ __align__(256) double scratch[kStaticSolveScratchBytes / sizeof(double)];

namespace {
constexpr int kMaxDevices = 64;
std::mutex g_scratch_mu;
void *g_scratch_ptr[kMaxDevices] = {};
}  // namespace

hipError_t static_solve_scratch(void **out) {
    int dev = -1;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    if (dev < 0 || dev >= kMaxDevices) return hipErrorInvalidDevice;
    std::lock_guard<std::mutex> lock(g_scratch_mu);
    if (!g_scratch_ptr[dev]) {
        void *p = nullptr;
        e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
        if (e != hipSuccess) return e;
        if (!p) return hipErrorInvalidSymbol;
        g_scratch_ptr[dev] = p;
    }
    *out = g_scratch_ptr[dev];
    return hipSuccess;
}

hipError_t launch_solve_blocked_static(int32_t n_maps, int32_t P, int32_t d_t, const float *G, const float *C,
                                       float lambda, uint32_t flags, float *maps, int32_t *info, hipStream_t s) {
    void *ws = nullptr;
    const hipError_t e = static_solve_scratch(&ws);
    if (e != hipSuccess) return e;
    return launch_solve_blocked(n_maps, P, d_t, G, C, lambda, flags, ws, kStaticSolveScratchBytes, maps, info, s);
}

}  // namespace cb

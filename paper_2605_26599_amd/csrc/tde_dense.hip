// Dense front end: reduction of a real symmetric matrix to tridiagonal form
// on the MI355X, then the boundary-row solve of the tridiagonal.
//
// Dense symmetric EVD first reduces A to T = Q^T A Q by orthogonal
// transformations (the eigenvalues of T are those of A) and then solves the
// tridiagonal problem (Section 2.1); for eigenvalues only the transformations
// are not kept.  The reduction here is the blocked Householder scheme of
// LAPACK's symmetric tridiagonal reduction (lower triangle, panel width kNb):
// inside a panel, column c is brought up to date with the panel's earlier
// reflectors, its reflector v (v_0 = 1) and tau are formed, and
// w = tau (A22 v - V (W^T v) - W (V^T v)) + alpha v with
// alpha = -tau/2 (w^T v) is taken against the trailing matrix as it stood at
// the start of the panel; after the panel the trailing matrix receives the
// rank-2b update A22 <- A22 - V W^T - W V^T as one matrix product on the FP64
// matrix cores.  Only the T x T tiles of the lower triangle are read and kept up
// to date (the diagonal ones in full); what lies above them goes stale.
//
// Per column two launches, each spread over the whole chip:
//   k_trd_sym: tau and scale of the column's reflector (every wave sums the
//     norm's partials itself), and A22 v from the lower triangle alone: one
//     workgroup per T x T tile, whose entries serve y_R += A v_C and
//     y_C += A^T v_R; the tiles' results stay apart (ypart) until the next
//     launch adds them up in tile order, so nothing is atomic and a repeat
//     gives the same bits.  One more workgroup adds up W^T v and V^T v.
//   k_trd_row: completes w (v^T w from the tiles' own v^T A22 v), brings the
//     next column up to date, and leaves its norm and its products with V and
//     W as partial sums, one workgroup per 64 rows.
// Per panel k_trd_row for its first column and after its last one, and
// k_trd_syr2k on the lower triangle's tiles.
// The traffic is the lower triangle read once per column, 4 n^3 / 3 bytes in
// all, plus one partial per tile side (at most 64 up to n = 65536), row and
// column.
#include <hip/hip_runtime.h>

#include "tde_dense.h"

namespace tde {

namespace {

constexpr int kRows = 64;  // rows per workgroup of k_trd_row, side of a subtile of k_trd_sym

__device__ __forceinline__ double join(unsigned lo, unsigned hi) {
    return __longlong_as_double((long long)(((unsigned long long)hi << 32) | lo));
}
__device__ __forceinline__ unsigned lo_of(double x) { return (unsigned)(unsigned long long)__double_as_longlong(x); }
__device__ __forceinline__ unsigned hi_of(double x) {
    return (unsigned)((unsigned long long)__double_as_longlong(x) >> 32);
}

// Value of lane `src` (wave-uniform) in every lane, as a scalar.
__device__ __forceinline__ double lane_value(double x, int src) {
    return join((unsigned)__builtin_amdgcn_readlane((int)lo_of(x), src),
                (unsigned)__builtin_amdgcn_readlane((int)hi_of(x), src));
}

// Lane moves within 16 lanes (no LDS crossbar).
template <int CTRL>
__device__ __forceinline__ double dpp(double x) {
    return join((unsigned)__builtin_amdgcn_update_dpp(0, (int)lo_of(x), CTRL, 0xF, 0xF, false),
                (unsigned)__builtin_amdgcn_update_dpp(0, (int)hi_of(x), CTRL, 0xF, 0xF, false));
}
constexpr int kSwap1 = 0xB1, kSwap2 = 0x4E;            // quad_perm: lane ^ 1, lane ^ 2
constexpr int kHalfMirror = 0x141, kMirror = 0x140;     // lane ^ 7, lane ^ 15

// Sum over the wave, the same bits in every lane: pairs of lanes add each
// other within 16 lanes, then the four rows of 16 in order.
__device__ __forceinline__ double wave_sum(double v) {
    v += dpp<kSwap1>(v);
    v += dpp<kSwap2>(v);
    v += dpp<kHalfMirror>(v);
    v += dpp<kMirror>(v);
    return (lane_value(v, 0) + lane_value(v, 16)) + (lane_value(v, 32) + lane_value(v, 48));
}

// a of the lower 32 lanes (even rows of 16) plus a of the upper ones (odd
// rows) lands in the lower (even) half, the same of b in the other: half a
// step of a transposing sum in two register swaps.
__device__ __forceinline__ double swap_add32(double a, double b) {
    const auto l = __builtin_amdgcn_permlane32_swap(lo_of(a), lo_of(b), false, false);
    const auto h = __builtin_amdgcn_permlane32_swap(hi_of(a), hi_of(b), false, false);
    return join(l[0], h[0]) + join(l[1], h[1]);
}
__device__ __forceinline__ double swap_add16(double a, double b) {
    const auto l = __builtin_amdgcn_permlane16_swap(lo_of(a), lo_of(b), false, false);
    const auto h = __builtin_amdgcn_permlane16_swap(hi_of(a), hi_of(b), false, false);
    return join(l[0], h[0]) + join(l[1], h[1]);
}

// Wave totals of 16 values per lane: lane l returns the total of value l / 4.
__device__ __forceinline__ double fold16(const double (&m)[16]) {
    const int lane = threadIdx.x & 63;
    double a[8], b[4], c[2];
#pragma unroll
    for (int i = 0; i < 8; ++i) a[i] = swap_add32(m[i], m[i + 8]);
#pragma unroll
    for (int i = 0; i < 4; ++i) b[i] = swap_add16(a[i], a[i + 4]);
    const bool u8 = (lane & 8) != 0, u4 = (lane & 4) != 0;
#pragma unroll
    for (int i = 0; i < 2; ++i) c[i] = (u8 ? b[i + 2] : b[i]) + dpp<kMirror>(u8 ? b[i] : b[i + 2]);
    double x = (u4 ? c[1] : c[0]) + dpp<kHalfMirror>(u4 ? c[0] : c[1]);
    x += dpp<kSwap2>(x);
    x += dpp<kSwap1>(x);
    return x;
}

// The reflector of column c from the column itself (unscaled in ua, rows
// c+1..n-1) and the partial sums of its norm below row c+1 (row blocks
// [rb0, rb1)): H = I - tau v v^T, v = ua scale with v_(c+1) = 1.  The whole
// wave; every wave of the launch gets the same bits.
struct Reflector {
    double tau, scale, beta;
};
__device__ __forceinline__ Reflector reflector(const double* __restrict__ ua, int c, const double* __restrict__ partN,
                                               int rb0, int rb1) {
    double x = 0.0;
    for (int b = rb0 + (int)(threadIdx.x & 63); b < rb1; b += 64) x += partN[b];
    const double ah = ua[c + 1];
    const double xn2 = wave_sum(x);
    Reflector f{0.0, 0.0, ah};
    if (xn2 > 0.0) {
        const double nrm = sqrt(fma(ah, ah, xn2));
        f.beta = (ah >= 0.0) ? -nrm : nrm;
        f.tau = (f.beta - ah) / f.beta;
        f.scale = 1.0 / (ah - f.beta);
    }
    return f;
}

// y = A22 v for column c (column i of the panel) from the lower triangle.
// Workgroup idx takes the T x T tile (I, J), I >= J, T = 64 sub, as sub x sub
// subtiles of 64 x 64: a lane holds a row, a wave 16 columns, all 16 loads in
// flight together.  Tiles are numbered from the matrix's lower right corner,
// so a tile keeps its number (and with it the XCD whose L2 holds it) while
// the trailing matrix shrinks.  ypart[J][rows of I] and, off the diagonal,
// ypart[I][columns of J] receive the tile's products, ydot[idx] its share of
// v^T A22 v.  Diagonal tiles also store v as column i of V.  The last
// workgroup forms sdot = (W_q . v, V_q . v) from k_trd_row's partials.
// Bound by the reads: n = 4096 (67 MB of lower triangle, held by the last
// cache) 41 -> 15 us at the first columns, 13.6 -> 7.8 us on average, against
// one wave per column over both triangles with two loads in flight; below
// about 2700 rows the tiles stay in the XCDs' own L2 (11 -> 8 us there), and
// the last thousand columns are a chain of latencies of 4.5 us.
__global__ __launch_bounds__(256) void k_trd_sym(const double* __restrict__ A, long long lda, int n, int c, int i,
                                                int sub, int NT, double* __restrict__ V,
                                                const double* __restrict__ W, const double* __restrict__ ua,
                                                double* __restrict__ tau, double* __restrict__ e,
                                                const double* __restrict__ partN, const double* __restrict__ partD,
                                                double* __restrict__ ypart, double* __restrict__ ydot,
                                                double* __restrict__ sdot) {
    extern __shared__ double lds[];  // yR [4][T], yC [T], the waves' shares of v^T A22 v [4]
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    const long long ln = n;
    const int rb0 = c / kRows, rb1 = (n + kRows - 1) / kRows;
    const int idx = (int)blockIdx.x;
    if (idx == (int)gridDim.x - 1) {
        // the panel's dot products: 64 sums over the row blocks, four threads each
        double x = 0.0;
        for (int b = rb0 + wv; b < rb1; b += 4) x += partD[b * 64 + lane];
        lds[wv * 64 + lane] = x;
        const Reflector f = reflector(ua, c, partN, rb0, rb1);
        if (threadIdx.x == 0) {
            tau[i] = f.tau;
            e[c] = f.beta;
        }
        __syncthreads();
        if (wv == 0) {
            const int q = lane & 31;
            const double t = (lds[lane] + lds[64 + lane]) + (lds[128 + lane] + lds[192 + lane]);
            if (q < i) sdot[lane] = fma(t, f.scale, (lane < 32 ? W : V)[q * ln + c + 1]);
        }
        return;
    }
    const int T = kRows * sub;
    int L = (int)((sqrtf(8.0f * (float)idx + 1.0f) - 1.0f) * 0.5f);
    while (L * (L + 1) / 2 > idx) --L;
    while ((L + 1) * (L + 2) / 2 <= idx) ++L;
    const int J = NT - 1 - L, I = NT - 1 - (idx - L * (L + 1) / 2);
    const bool diag = I == J;
    // live subtiles: columns ci0.. and rows ri0.. up to the matrix's end
    const int ci0 = max(0, (c + 1 - J * T) / kRows), ri0 = max(0, (c + 1 - I * T) / kRows);
    const int nci = min(sub, (n - J * T + kRows - 1) / kRows) - ci0;
    const int nri = min(sub, (n - I * T + kRows - 1) / kRows) - ri0;
    // loads past the matrix's end read its last row or column instead (their
    // entry of v is zero), so none of them waits on a branch
    double a[16], ur, uc;
    auto load = [&](int ci, int ri) {
        const int c0 = J * T + ci * kRows + wv * 16, r = min(I * T + ri * kRows + lane, n - 1);
#pragma unroll
        for (int q = 0; q < 16; ++q) a[q] = A[(long long)min(c0 + q, n - 1) * lda + r];
        ur = ua[r];
        if (ri == ri0) uc = ua[min(c0 + (lane & 15), n - 1)];
    };
    load(ci0, ri0);  // on its way while the reflector's scalars are formed
    const Reflector f = reflector(ua, c, partN, rb0, rb1);
    auto v_of = [&](int r, double u) { return (r > c + 1 && r < n) ? u * f.scale : ((r == c + 1) ? 1.0 : 0.0); };
    double* yR = lds + wv * T;
    double* yC = lds + 4 * T;
    double yv = 0.0, vr = 0.0;
    for (int ci = ci0; ci < ci0 + nci; ++ci) {
        double vc = 0.0;
        for (int ri = ri0; ri < ri0 + nri; ++ri) {
            if (ci > ci0 || ri > ri0) load(ci, ri);
            if (ri == ri0) vc = v_of(J * T + ci * kRows + wv * 16 + (lane & 15), uc);
            vr = v_of(I * T + ri * kRows + lane, ur);
            double y = 0.0;
#pragma unroll
            for (int q = 0; q < 16; ++q) {
                y = fma(a[q], lane_value(vc, q), y);
                a[q] *= vr;
            }
            yv = fma(y, vr, yv);
            double& yr = yR[ri * kRows + lane];
            yr = (ci > ci0) ? yr + y : y;
            if (!diag) {
                const double t = fold16(a);
                double& yc = yC[ci * kRows + wv * 16 + (lane >> 2)];
                if ((lane & 3) == 0) yc = (ri > ri0) ? yc + t : t;
            }
        }
    }
    yv = wave_sum(yv);
    if (lane == 0) lds[5 * T + wv] = yv;
    __syncthreads();
    // (rows and columns up to c get no product and are never read)
    for (int q = threadIdx.x; q < T; q += 256) {
        const int r = I * T + q, s = J * T + q;
        if (r > c && r < n) {
            ypart[J * ln + r] = (lds[q] + lds[T + q]) + (lds[2 * T + q] + lds[3 * T + q]);
            if (diag) V[i * ln + r] = v_of(r, ua[r]);
        }
        if (!diag && s > c && s < n) ypart[I * ln + s] = yC[q];
    }
    if (threadIdx.x == 0) {
        const double t = (lds[5 * T] + lds[5 * T + 1]) + (lds[5 * T + 2] + lds[5 * T + 3]);
        ydot[idx] = diag ? t : 2.0 * t;
    }
}

// After the i-th reflector of a panel (v = column i-1 of V, made at column
// c-1): w = tau (y - V (W^T v) - W (V^T v)) + alpha v with alpha =
// -tau/2 (w'^T v), w' the part before alpha, and w'^T v = tau (v^T y -
// 2 (W^T v).(V^T v)), stored as column i-1 of W.  With `next`, column c is then
// brought up to date (a = A[:, c] - V W[c, :]^T - W V[c, :]^T), its diagonal
// entry recorded, the entries below kept in ua, and this row block's share
// of its norm (rows >= c+2) and of its products with every column of W and V
// left in partN and partD.  One workgroup per 64 rows: a lane holds a row,
// the four waves share the panel's columns (j = wave, wave + 4, ...), so a
// thread's loads are all in flight at once.  i = 0: only the column.
// Bound by latency (a chain of loads, a barrier, a few sums, a barrier):
// n = 4096: 14.2 us for the two launches this replaces, each of which ended in
// an atomic ticket and a last workgroup's sum, 5.8 us now; the partial sums
// cost less in the next launch than a ticket at the end of this one.
__global__ __launch_bounds__(256) void k_trd_row(const double* __restrict__ A, long long lda, int n, int c, int i,
                                                int next, int p0, int NT, int nyd, const double* __restrict__ V,
                                                double* __restrict__ W, double* __restrict__ ua,
                                                const double* __restrict__ tau, double* __restrict__ d,
                                                const double* __restrict__ ypart, const double* __restrict__ ydot,
                                                const double* __restrict__ sdot, double* __restrict__ partN,
                                                double* __restrict__ partD) {
    __shared__ double sS[64], sV[32], sW[32];  // dot products, row c of V and W
    __shared__ double sy[4], sc[3], red[3][4][64];
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    const long long ln = n;
    const int rb = c / kRows + (int)blockIdx.x;
    const int r = rb * kRows + lane;
    const bool live = r >= c && r < n;
    const int jl = i - 1;  // the reflector just made; jl < 0: none
    // (loads a thread has no use for read a valid entry instead, so that none
    // of them waits on a branch)
    const int rl = min(r, n - 1);
    double vj[8], wj[8];
#pragma unroll
    for (int q = 0; q < 8; ++q) {
        const int j = wv + 4 * q;
        const bool on = live && j < jl;
        const double x = V[j * ln + rl], y = W[j * ln + rl];
        vj[q] = on ? x : 0.0;
        wj[q] = on ? y : 0.0;
    }
    const double vx = V[max(jl, 0) * ln + rl], ax = A[(long long)min(c, n - 1) * lda + rl];
    const double vl = (jl >= 0 && live) ? vx : 0.0;
    double accA = (next && wv == 0 && live) ? -ax : 0.0;
    double wr = 0.0, wc = 0.0;
    if (i > 0) {  // uniform
        double ys = 0.0, yd = 0.0;
        // fixed batches of guarded loads, so that they are in flight together
        for (int pb = p0 + wv; pb < NT; pb += 64) {
            double x[16];
#pragma unroll
            for (int q = 0; q < 16; ++q) x[q] = ypart[min(pb + 4 * q, NT - 1) * ln + rl];
#pragma unroll
            for (int q = 0; q < 16; ++q) ys += (live && pb + 4 * q < NT) ? x[q] : 0.0;
        }
        for (int qb = threadIdx.x; qb < nyd; qb += 256 * 9) {
            double x[9];
#pragma unroll
            for (int q = 0; q < 9; ++q) x[q] = ydot[min(qb + 256 * q, nyd - 1)];
#pragma unroll
            for (int q = 0; q < 9; ++q) yd += (qb + 256 * q < nyd) ? x[q] : 0.0;
        }
        // the scalars' sums over the panel's columns (or row c's over the
        // tiles), one per wave: V, W and their dot products in lanes j < jl
        const double t = tau[jl];
        const bool on = lane < jl;
        double x = 0.0;
        if (wv == 3) {
            for (int p = p0 + lane; p < NT; p += 64) x += ypart[p * ln + c];
        } else if (wv > 0) {
            const double dW = on ? sdot[lane] : 0.0, dV = on ? sdot[32 + lane] : 0.0;
            const double Vc = on ? V[lane * ln + c] : 0.0, Wc = on ? W[lane * ln + c] : 0.0;
            x = (wv == 1) ? dW * dV : Vc * dW + Wc * dV;
            if (wv == 1 && lane < 32) {
                sS[lane] = dW;
                sS[32 + lane] = dV;
                sV[lane] = Vc;
                sW[lane] = Wc;
            }
        }
        x = wave_sum(x);
        yd = wave_sum(yd);
        if (lane == 0) {
            sy[wv] = yd;
            if (wv > 0) sc[wv - 1] = x;
        }
        __syncthreads();
        const double yv = (sy[0] + sy[1]) + (sy[2] + sy[3]);
        const double alpha = -0.5 * t * (t * (yv - 2.0 * sc[0]));
        wc = fma(t, sc[2] - sc[1], alpha);  // row c of w (v_c = 1)
        double accW = 0.0;
#pragma unroll
        for (int q = 0; q < 8; ++q) {
            const int j = wv + 4 * q;  // (zeros from jl on)
            accW += vj[q] * sS[j] + wj[q] * sS[32 + j];
            accA += vj[q] * sW[j] + wj[q] * sV[j];
        }
        red[0][wv][lane] = ys;
        red[1][wv][lane] = accW;
        red[2][wv][lane] = accA;
        __syncthreads();
        auto sum4 = [&](int k) { return (red[k][0][lane] + red[k][1][lane]) + (red[k][2][lane] + red[k][3][lane]); };
        wr = fma(alpha, vl, t * (sum4(0) - sum4(1)));
        accA = sum4(2) + (vl * wc + wr);
        if (wv == 0 && live) W[jl * ln + r] = wr;
    }
    if (!next) return;
    if (i == 0) {
        red[2][wv][lane] = accA;
        __syncthreads();
        accA = red[2][0][lane];
    }
    const double a = -accA;
    if (wv == 0 && live) {
        if (r == c) d[c] = a;
        else ua[r] = a;
    }
    const double av = (r >= c + 2 && r < n) ? a : 0.0;
    if (wv == 0) {
        const double s = wave_sum(av * av);
        if (lane == 0) partN[rb] = s;
    }
    if (i > 0) {
        double m[16];
#pragma unroll
        for (int q = 0; q < 8; ++q) {
            const bool last = wv + 4 * q == jl;
            m[q] = (last ? wr : wj[q]) * av;
            m[8 + q] = (last ? vl : vj[q]) * av;
        }
        const double s = fold16(m);
        // value x < 8: W column wv + 4 x, else V column wv + 4 (x - 8)
        const int x = lane >> 2;
        if ((lane & 3) == 0) partD[rb * 64 + (x < 8 ? wv + 4 * x : 32 + wv + 4 * (x - 8))] = s;
    }
}

// Trailing update A[q:, q:] -= V W^T + W V^T (rows and columns q..n-1, the
// T x T tiles of the lower triangle, T = 64 sub, that k_trd_sym reads) on the
// FP64 matrix cores.  With U = [V | W] and Z = [W | V]
// (n x 2b) the update is U Z^T.  One wave per 32 x 32 tile of A, as 2 x 2
// blocks of V_MFMA_F64_16X16X4F64 (D = A_op B_op + C, A_op 16 x 4, B_op
// 4 x 16): A_op[i][k] = Z[s0 + i][k], B_op[k][j] = U[r0 + j][k], so
// D[i][j] is the update of A[r0 + j][s0 + i]; lane l supplies A_op[l % 16][l / 16]
// and B_op[l / 16][l % 16] and holds D[4 t + l / 16][l % 16] in its register
// t = 0..3, i.e. row r0 + l % 16 of column s0 + 4 t + l / 16: sixteen lanes
// touch sixteen consecutive rows of one column.  The tile's entries are loaded
// before the products are formed (n = 4096: 37 us per panel over both
// triangles, 29 over the lower one, 21 with the early loads).
typedef double v4d __attribute__((ext_vector_type(4)));

__global__ __launch_bounds__(256) void k_trd_syr2k(double* __restrict__ A, long long lda, int n, int q, int b,
                                                  const double* __restrict__ V, const double* __restrict__ W,
                                                  int tiles, int T) {
    const int wave = (int)((blockIdx.x * 256 + threadIdx.x) >> 6);
    const int lane = threadIdx.x & 63;
    const int tr = wave % tiles, tc = wave / tiles;
    if (tc >= tiles) return;  // wave-uniform
    const int r0 = q + 32 * tr, s0 = q + 32 * tc;
    if ((r0 + 31) / T < s0 / T) return;  // wave-uniform: above the diagonal tiles
    const long long ln = n;
    const int li = lane & 15, lk = lane >> 4;
    // rows past the end read the last one (their results are not stored)
    const int sr0 = min(s0 + li, n - 1), sr1 = min(s0 + 16 + li, n - 1);  // Z rows (A operand), blocks ib = 0, 1
    const int ur0 = min(r0 + li, n - 1), ur1 = min(r0 + 16 + li, n - 1);  // U rows (B operand), blocks jb = 0, 1
    double old[2][2][4];  // this lane's entries of A, on their way while the products are formed
#pragma unroll
    for (int ib = 0; ib < 2; ++ib)
#pragma unroll
        for (int jb = 0; jb < 2; ++jb)
#pragma unroll
            for (int t = 0; t < 4; ++t)
                old[ib][jb][t] = A[(long long)min(s0 + 16 * ib + 4 * t + lk, n - 1) * lda + (jb ? ur1 : ur0)];
    v4d acc[2][2];
    for (int a = 0; a < 2; ++a)
        for (int bb = 0; bb < 2; ++bb) acc[a][bb] = v4d{0.0, 0.0, 0.0, 0.0};
    // Z = [W | V], U = [V | W]: the panel columns k of both halves per step
    _Pragma("unroll 2") for (int k0 = 0; k0 < b; k0 += 4) {
        const int k = min(k0 + lk, b - 1);
        const bool on = k0 + lk < b;
        const double* __restrict__ v = V + (long long)k * ln;
        const double* __restrict__ x = W + (long long)k * ln;
        double zw0 = x[sr0], zw1 = x[sr1], uv0 = v[ur0], uv1 = v[ur1];
        double zv0 = v[sr0], zv1 = v[sr1], uw0 = x[ur0], uw1 = x[ur1];
        if (!on) zw0 = zw1 = zv0 = zv1 = uv0 = uv1 = uw0 = uw1 = 0.0;
        acc[0][0] = __builtin_amdgcn_mfma_f64_16x16x4f64(zw0, uv0, acc[0][0], 0, 0, 0);
        acc[0][1] = __builtin_amdgcn_mfma_f64_16x16x4f64(zw0, uv1, acc[0][1], 0, 0, 0);
        acc[1][0] = __builtin_amdgcn_mfma_f64_16x16x4f64(zw1, uv0, acc[1][0], 0, 0, 0);
        acc[1][1] = __builtin_amdgcn_mfma_f64_16x16x4f64(zw1, uv1, acc[1][1], 0, 0, 0);
        acc[0][0] = __builtin_amdgcn_mfma_f64_16x16x4f64(zv0, uw0, acc[0][0], 0, 0, 0);
        acc[0][1] = __builtin_amdgcn_mfma_f64_16x16x4f64(zv0, uw1, acc[0][1], 0, 0, 0);
        acc[1][0] = __builtin_amdgcn_mfma_f64_16x16x4f64(zv1, uw0, acc[1][0], 0, 0, 0);
        acc[1][1] = __builtin_amdgcn_mfma_f64_16x16x4f64(zv1, uw1, acc[1][1], 0, 0, 0);
    }
#pragma unroll
    for (int ib = 0; ib < 2; ++ib)
#pragma unroll
        for (int jb = 0; jb < 2; ++jb) {
            const int r = r0 + 16 * jb + li;
            if (r >= n) continue;
#pragma unroll
            for (int t = 0; t < 4; ++t) {
                const int s = s0 + 16 * ib + 4 * t + lk;
                if (s < n) A[(long long)s * lda + r] = old[ib][jb][t] - acc[ib][jb][t];
            }
        }
}

// The last 2 x 2 (or 1 x 1) block after every update.
__global__ void k_trd_tail(const double* __restrict__ A, long long lda, int n, double* __restrict__ d,
                           double* __restrict__ e) {
    if (threadIdx.x != 0 || n < 1) return;
    if (n == 1) {
        d[0] = A[0];
        return;
    }
    d[n - 2] = A[(long long)(n - 2) * lda + (n - 2)];
    d[n - 1] = A[(long long)(n - 1) * lda + (n - 1)];
    e[n - 2] = A[(long long)(n - 2) * lda + (n - 1)];
}

// Side of the tiles of k_trd_sym in subtiles: at most 64 tiles a side (so at
// most 64 partials per row) up to 65536 rows; beyond, tiles of 1024 (their LDS
// is 40 KB then), n / 1024 a side.
int dense_sub(long long n) {
    const long long s = (n + 64 * kRows - 1) / (64 * kRows);
    return (int)(s < 1 ? 1 : (s > 16 ? 16 : s));
}
long long dense_tiles(long long n) {
    const long long T = (long long)kRows * dense_sub(n);
    return (n + T - 1) / T;
}

}  // namespace

size_t dense_layout(long long n, char* base, DenseWork* dw) {
    size_t off = 0;
    auto take = [&](size_t bytes) -> char* {
        char* p = base ? base + off : nullptr;
        off += (bytes + 255) & ~(size_t)255;
        return p;
    };
    const long long nn = n > 0 ? n : 1;
    DenseWork t{};
    t.V = (double*)take(8 * nn * kNb);
    t.W = (double*)take(8 * nn * kNb);
    const long long NT = dense_tiles(nn);
    const long long rb = (nn + kRows - 1) / kRows;
    t.ypart = (double*)take(8 * nn * NT);
    t.ydot = (double*)take(8 * (NT * (NT + 1) / 2));
    t.tau = (double*)take(8 * kNb);
    t.sdot = (double*)take(8 * 2 * kNb);
    t.ua = (double*)take(8 * nn);
    t.partN = (double*)take(8 * rb);
    t.partD = (double*)take(8 * 64 * rb);
    t.d = (double*)take(8 * nn);
    t.e = (double*)take(8 * nn);
    if (dw) *dw = t;
    return off;
}

int enqueue_dense_reduce(double* A, long long lda, int n, const DenseWork& dw, void* stream) {
    hipStream_t s = (hipStream_t)stream;
    if (n <= 0) return 0;
    const int sub = dense_sub(n), T = kRows * sub, NT = (int)dense_tiles(n);
    static_assert(kNb == 32, "k_trd_row shares 32 panel columns over four waves, eight each");
    auto row_step = [&](int c, int i, int next) {
        // the tiles k_trd_sym used for column c-1: tile columns from c / T on
        const int p0 = c / T, nt = NT - p0;
        hipLaunchKernelGGL(k_trd_row, dim3((unsigned)((n + kRows - 1) / kRows - c / kRows)), dim3(256), 0, s, A, lda,
                           n, c, i, next, p0, NT, nt * (nt + 1) / 2, dw.V, dw.W, dw.ua, dw.tau, dw.d, dw.ypart,
                           dw.ydot, dw.sdot, dw.partN, dw.partD);
    };
    for (int p = 0; p < n - 2; p += kNb) {
        const int b = (n - 2 - p < kNb) ? n - 2 - p : kNb;
        row_step(p, 0, 1);
        for (int i = 0; i < b; ++i) {
            const int c = p + i;
            const int nt = NT - (c + 1) / T;
            hipLaunchKernelGGL(k_trd_sym, dim3((unsigned)(nt * (nt + 1) / 2 + 1)), dim3(256),
                               (unsigned)((5 * T + 4) * sizeof(double)), s, A, lda, n, c, i, sub, NT, dw.V, dw.W, dw.ua,
                               dw.tau, dw.e, dw.partN, dw.partD, dw.ypart, dw.ydot, dw.sdot);
            row_step(c + 1, i + 1, i + 1 < b ? 1 : 0);
        }
        const int q = p + b;
        const int M = n - q;
        const int tiles = (M + 31) / 32;
        const long long waves = (long long)tiles * tiles;
        hipLaunchKernelGGL(k_trd_syr2k, dim3((unsigned)((waves + 3) / 4)), dim3(256), 0, s, A, lda, n, q, b, dw.V,
                           dw.W, tiles, T);
    }
    hipLaunchKernelGGL(k_trd_tail, dim3(1), dim3(64), 0, s, A, lda, n, dw.d, dw.e);
    return (int)hipGetLastError();
}

}  // namespace tde

// sbf.hip -- the slender-body formulation (Sec. 3 of the paper) on gfx950:
// moments of the free-space Green's function between every pair of fibers
// (Eq. Gnonper, integrals of the form of Eq. theta_def), the dense Legendre
// system of Eqs. sev_fils and extra_cond with the expansion of Eq.
// force_exp, solved by restarted GMRES, the velocities of Eqs. xadot and
// padot, and Adams-Bashforth-2 time stepping.  C ABI in include/sbf.h.
//
// Layout.  The moments form one dense symmetric FP64 matrix W of order
// D = 3 M (N + 1): row (m, n, a), column (m', k, b) holds
//   Theta^{n,k}_{mm'}[a][b] = int int G(R(s, s'))_ab P_k(s'/l) P_n(s/l) ds' ds,
//   R = x_m + s p_m - x_m' - s' p_m',
// n, k = 0..N, zero for m = m' (a fiber does not see itself through G).
// Every vector (Krylov basis, solution, right-hand side) uses the same
// (m, k, b) layout, its k = 0 entries zero except where the known force
// part F/(2l) is put in.  Then every product with W is one GEMV, the
// system operator is that GEMV followed by 3x3 block operations per (m, n),
// and the velocities come from the n = 0 and n = 1 rows of W [F/(2l); a].
//
// G(R) and G(-R) are equal and symmetric, so Theta^{k,n}_{m'm} is the
// transpose of Theta^{n,k}_{mm'} and W = W^T.  Only its upper triangle is
// stored, as 64 x 64 tiles (i, j), i <= j, packed row after row, each tile
// row-major; the diagonal tiles are stored whole, padding rows and columns
// beyond D are zero.  A product y = W x reads every stored tile once and
// uses it twice, W_ij x_j for the rows of block i and W_ij^T x_i for the
// rows of block j (i < j), writing each into its own slot of a partial-sum
// array part[slot][row] (row sums per chunk of tiles of a tile row, column
// sums per tile); a second pass adds the slots of each row in a fixed order.
//
// Bound: the moments are FP64 ALU work (M^2/2 pairs x (3 nq)^2 Green's
// function evaluations, each pair giving both of its blocks of W); each
// GMRES iteration streams the stored half of W once (about D^2/2 x 8
// bytes, HBM bound).
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstring>
#include <new>
#include <string>
#include <vector>

#include "../../include/sbf.h"

namespace sbfk {

constexpr int MAXN = 8;        // Legendre modes supported (N <= 8)
constexpr int MAXR = 64;       // Krylov dimension
constexpr int TS = 64;         // tile edge of the packed moment matrix

struct Consts {
    int M, N, Q, D;            // fibers, modes, quadrature points per fiber, order of W
    int nt;                    // tiles per side, ceil(D / TS)
    double l, L, r, d, mu;
};

// first element of tile (i, j), i <= j, in the packed upper triangle
__host__ __device__ __forceinline__ size_t tile_base(int i, int j, int nt)
{
    // rows r < i hold nt - r tiles each: i nt - i (i - 1)/2 = i (2 nt - i + 1)/2
    return (size_t(i) * (2 * size_t(nt) - size_t(i) + 1) / 2 + size_t(j - i)) * (TS * TS);
}

// packed tiles of the upper triangle for nt tiles per side
__host__ __device__ __forceinline__ size_t packed_tiles(int nt) { return size_t(nt) * size_t(nt + 1) / 2; }

// ------------------------------------------------------------------ moments
// 1/sqrt(x) for x > 0: the hardware estimate y (relative error e/2 below
// 2^-22) refined by the third-order step y (1 + e/2 + 3 e^2/8), e = 1 - x y^2,
// whose error is of the order of e^3.
__device__ __forceinline__ double rsqrt_nr(double x)
{
    const double y = __builtin_amdgcn_rsq(x);
    const double e = fma(-x * y, y, 1.0);
    return fma(y * e, fma(0.375, e, 0.5), y);
}

// Moments: workgroup b takes the pairs b PB .. b PB + PB - 1 of the list of
// pairs m < m' (row by row; the pair gives both blocks of W, the diagonal
// blocks stay at the zero the packed matrix was cleared to).
//
// With R = D + s p_m - s' p_m', D = x_m - x_m', the tensor part of
// G = alpha I + beta R R^T is a polynomial in s and s' with scalar weights
// beta, and s P_n is a combination of P_{n+1} and P_{n-1}.  So the block of a
// pair follows from the scalar moments of alpha with P_n P_k, n, k <= N, and
// of beta with n, k <= N + 2; the six tensor components need no sums of
// their own.  Thread t serves pair slot t / Q and the outer point s_i, i =
// t % Q, sums over s'_j into N + 1 and N + 3 accumulators (moment_point: 16
// FP64 instructions for the Green's function and 2 N + 4 multiply-adds,
// instead of 7 (N + 1)), the outer sums with P_n(s_i) follow from LDS, and one
// thread per (pair, n, k) then forms the 3 x 3 block.  The split into
// powers of s cancels where fibers are closer than their length, by a
// factor of about (L/R)^2 on a sum exact to 1e-16.
//
// Bound: FP64 ALU.  1024 fibers, N = 5, Q = 48: 4.27 ms with a sum per tensor
// component, 2.06 ms with scalar moments.
// Tables: wl[k][j] = w_j P_k(s_j), k <= N + 2, and the same by points, wj[j] =
// (s_j, w_j P_0(s_j), ...): an inner point's row is one scalar load.  Three
// points are taken at a time (Q is a multiple of three), so that their
// scalar loads are waited for once.
template <int NP1>
__device__ __forceinline__ void moment_term(const double (&b)[3], const double (&pn)[3], double h, const double *w,
                                            double (&acc)[2 * NP1 + 2])
{
    const double R0 = b[0] - w[0] * pn[0], R1 = b[1] - w[0] * pn[1], R2 = b[2] - w[0] * pn[2];
    const double r2 = R0 * R0 + R1 * R1 + R2 * R2;
    const double inv = rsqrt_nr(r2);
    const double inv2 = inv * inv, inv3 = inv * inv2;
    const double alpha = fma(h, inv3, inv);
    const double beta = inv3 * fma(-3.0 * h, inv2, 1.0);
#pragma unroll
    for (int k = 0; k < NP1 + 2; ++k) {
        if (k < NP1) acc[k] = fma(w[1 + k], alpha, acc[k]);
        acc[NP1 + k] = fma(w[1 + k], beta, acc[NP1 + k]);
    }
}
// sums of the inner points j0, j0 + dj, ... for the outer point s_i
template <int NP1>
__device__ __forceinline__ void moment_point(double si, const double (&xm)[3], const double (&pm)[3],
                                             const double (&xn)[3], const double (&pn)[3], double h, int Q,
                                             const double *wj, int j0, int dj, double (&acc)[2 * NP1 + 2])
{
#pragma unroll
    for (int k = 0; k < 2 * NP1 + 2; ++k) acc[k] = 0.0;
    const double b[3] = {xm[0] + si * pm[0] - xn[0], xm[1] + si * pm[1] - xn[1], xm[2] + si * pm[2] - xn[2]};
    for (int j = j0; j < Q; j += dj) moment_term<NP1>(b, pn, h, wj + j * (NP1 + 3), acc);
}

// pair p of the list m < m', start(m) = m (2M - m - 1)/2 pairs precede row m
// (fewer than 2^30 pairs: sbf_create bounds the order of W)
__device__ __forceinline__ void pair_of(int p, int M, int &m, int &mp)
{
    const double b = 2.0 * M - 1.0;
    int r = int((float(b) - sqrtf(float(b * b - 8.0 * double(p)))) * 0.5f);   // off by one at most, then exact
    r = min(max(r, 0), M - 2);
    while (r > 0 && r * (2 * M - r - 1) / 2 > p) --r;
    while (r + 1 <= M - 2 && (r + 1) * (2 * M - r - 2) / 2 <= p) ++r;
    m = r;
    mp = r + 1 + (p - r * (2 * M - r - 1) / 2);
}

// index of (a, b) among the six components xx xy xz yy yz zz
__device__ __forceinline__ int sym_index(int a, int b) { return a == b ? (a == 0 ? 0 : (a == 1 ? 3 : 5)) : (a + b == 1 ? 1 : (a + b == 2 ? 2 : 4)); }

// The 3 x 3 block (n, k) of a pair as its components xx xy xz yy yz zz in o[6],
// from the moments A of alpha [NP1][NP1] and B of beta [NP1 + 2][NP1 + 2], d =
// (D, p_m, p_m') and s P_n = up[n] P_{n+1} + dn[n] P_{n-1}.
template <int NP1>
__device__ __forceinline__ void pair_block(int n, int k, const double *A, const double *B, const double *d,
                                           const double *up, const double *dn, double *o)
{
    constexpr int NB = NP1 + 2;
    const int n1 = max(n - 1, 0), k1 = max(k - 1, 0), n2 = max(n - 2, 0), k2 = max(k - 2, 0);
    const double un = up[n], dnn = dn[n], uk = up[k], dk = dn[k];
    const double b00 = B[n * NB + k];
    const double b10 = un * B[(n + 1) * NB + k] + dnn * B[n1 * NB + k];
    const double b01 = uk * B[n * NB + k + 1] + dk * B[n * NB + k1];
    const double b20 = un * (up[n + 1] * B[(n + 2) * NB + k] + dn[n + 1] * b00) +
                       dnn * (up[n1] * b00 + dn[n1] * B[n2 * NB + k]);
    const double b02 = uk * (up[k + 1] * B[n * NB + k + 2] + dn[k + 1] * b00) +
                       dk * (up[k1] * b00 + dn[k1] * B[n * NB + k2]);
    const double b11 = un * (uk * B[(n + 1) * NB + k + 1] + dk * B[(n + 1) * NB + k1]) +
                       dnn * (uk * B[n1 * NB + k + 1] + dk * B[n1 * NB + k1]);
#pragma unroll
    for (int a = 0; a < 3; ++a)
#pragma unroll
        for (int b = a; b < 3; ++b) {
            double v = b00 * (d[a] * d[b]) + b10 * (d[a] * d[3 + b] + d[3 + a] * d[b]) -
                       b01 * (d[a] * d[6 + b] + d[6 + a] * d[b]) + b20 * (d[3 + a] * d[3 + b]) -
                       b11 * (d[3 + a] * d[6 + b] + d[6 + a] * d[3 + b]) + b02 * (d[6 + a] * d[6 + b]);
            if (a == b) v += A[n * NP1 + k];
            o[sym_index(a, b)] = v;
        }
}

// LDS of k_theta in doubles per pair slot: the point sums [Q][theta_cols] (later
// the blocks' six components), the moments of alpha and beta, and D, p_m, p_m'
__host__ __device__ constexpr int theta_cols(int np1) { return (2 * np1 + 2) | 1; }   // odd: spreads the banks
__host__ __device__ constexpr int theta_points(int np1, int q)
{
    return q * theta_cols(np1) > 6 * np1 * np1 ? q * theta_cols(np1) : 6 * np1 * np1;
}
__host__ __device__ constexpr int theta_lds(int np1, int q)
{
    return theta_points(np1, q) + np1 * np1 + (np1 + 2) * (np1 + 2) + 9;
}

template <int NP1>
__global__ __launch_bounds__(256) void k_theta(const double *__restrict__ X, const double *__restrict__ p, Consts c,
                                               const double *__restrict__ wj, const double *__restrict__ wl,
                                               double *__restrict__ W, int PB, int P)
{
    constexpr int NB = NP1 + 2, NC = NP1 + NB, NCP = theta_cols(NP1), st = 3 * NP1;
    extern __shared__ double sh[];
    __shared__ double up[NB], dn[NB];   // s P_n = up P_{n+1} + dn P_{n-1}
    // where a pair's block lies in W: first element of the tile holding its
    // first row and column, steps to the next tile right and down
    struct Place {
        size_t at, right, down;
        int r0, c0, diag;
    };
    __shared__ Place place[85];               // PB Q <= 256, Q >= 3
    __shared__ uint32_t entry[st * st];       // row, column and component of each entry of a block
    const int per = theta_lds(NP1, c.Q), pts = theta_points(NP1, c.Q);
    const int t = int(threadIdx.x), nt = int(blockDim.x), slot = t / c.Q, i = t % c.Q;
    // neighbouring workgroups write neighbouring columns of W: keep them on one XCD
    const uint32_t nb8 = gridDim.x >> 3, rem = gridDim.x & 7u, xcd = blockIdx.x & 7u;
    const int p0 = int(xcd * nb8 + (xcd < rem ? xcd : rem) + (blockIdx.x >> 3)) * PB;
    if (t < NB) {
        up[t] = c.l * (t + 1) / (2 * t + 1);
        dn[t] = c.l * t / (2 * t + 1);
    }
    for (int e = t; e < st * st; e += nt) {
        const int row = e / st, col = e - row * st, n = row / 3, k = col / 3;
        entry[e] = uint32_t(row) | uint32_t(col) << 8 | uint32_t((n * NP1 + k) * 6 + sym_index(row - 3 * n, col - 3 * k)) << 16;
    }
    if (slot < PB && p0 + slot < P) {
        int m, mp;
        pair_of(p0 + slot, c.M, m, mp);
        const double xm[3] = {X[3 * m], X[3 * m + 1], X[3 * m + 2]};
        const double pm[3] = {p[3 * m], p[3 * m + 1], p[3 * m + 2]};
        const double xn[3] = {X[3 * mp], X[3 * mp + 1], X[3 * mp + 2]};
        const double pn[3] = {p[3 * mp], p[3 * mp + 1], p[3 * mp + 2]};
        if (i == 0) {
            // (m st, mp st), m < mp: on or above the diagonal tile
            const int bi = m * st / TS, bj = mp * st / TS;
            Place q;
            q.at = tile_base(bi, bj, c.nt);
            q.right = TS * TS;
            q.down = tile_base(bi + 1, max(bj, bi + 1), c.nt) - tile_base(bi, max(bj, bi + 1), c.nt);
            q.r0 = m * st % TS;
            q.c0 = mp * st % TS;
            q.diag = bj - bi;
            place[slot] = q;
            double *d = sh + size_t(slot) * per + per - 9;
            for (int a = 0; a < 3; ++a) {
                d[a] = xm[a] - xn[a];
                d[3 + a] = pm[a];
                d[6 + a] = pn[a];
            }
        }
        double acc[NC];
#pragma unroll
        for (int k = 0; k < NC; ++k) acc[k] = 0.0;
        const double si = wj[i * (NB + 1)], h = 0.5 * c.r * c.r;
        const double b[3] = {xm[0] + si * pm[0] - xn[0], xm[1] + si * pm[1] - xn[1], xm[2] + si * pm[2] - xn[2]};
        for (int j = 0; j < c.Q; j += 3) {
            double w[3][NB + 1];
#pragma unroll
            for (int e = 0; e < 3 * (NB + 1); ++e) w[e / (NB + 1)][e % (NB + 1)] = wj[j * (NB + 1) + e];
#pragma unroll
            for (int k = 0; k < 3; ++k) moment_term<NP1>(b, pn, h, w[k], acc);
        }
        double *o = sh + size_t(slot) * per + i * NCP;
#pragma unroll
        for (int k = 0; k < NC; ++k) o[k] = acc[k];
    }
    __syncthreads();
    // outer sums: wave w takes three modes n at a time (weights in scalar
    // registers), the lanes the columns of all pairs
    const int wv = __builtin_amdgcn_readfirstlane(t >> 6), nw = (nt + 63) >> 6;
    for (int n = 3 * wv; n < NB; n += 3 * nw) {
        const double *w0 = wl + n * c.Q, *w1 = wl + min(n + 1, NB - 1) * c.Q, *w2 = wl + min(n + 2, NB - 1) * c.Q;
        for (int e = t & 63; e < PB * NC; e += 64) {
            const int s2 = e / NC, col = e - s2 * NC;
            const double *b = sh + size_t(s2) * per + col;
            double a0 = 0.0, a1 = 0.0, a2 = 0.0;
#pragma unroll 6
            for (int q = 0; q < c.Q; ++q) {
                const double v = b[q * NCP];
                a0 = fma(w0[q], v, a0);
                a1 = fma(w1[q], v, a1);
                a2 = fma(w2[q], v, a2);
            }
            const double s3[3] = {a0, a1, a2};
            double *mo = sh + size_t(s2) * per + pts;
#pragma unroll
            for (int k = 0; k < 3; ++k) {
                if (col < NP1) {
                    if (n + k < NP1) mo[(n + k) * NP1 + col] = s3[k];
                } else if (n + k < NB) {
                    mo[NP1 * NP1 + (n + k) * NB + col - NP1] = s3[k];
                }
            }
        }
    }
    __syncthreads();
    // the six components of each (n, k) block
    for (int e = t; e < PB * NP1 * NP1; e += nt) {
        const int s2 = e / (NP1 * NP1), nk = e - s2 * (NP1 * NP1), n = nk / NP1, k = nk - n * NP1;
        double *base = sh + size_t(s2) * per;
        const double *A = base + pts;
        pair_block<NP1>(n, k, A, A + NP1 * NP1, base + per - 9, up, dn, base + nk * 6);
    }
    __syncthreads();
    // Theta^{n,k}_{m,mp} at (m st + row, mp st + col); its transpose,
    // Theta^{k,n}_{mp,m}, is the mirror entry of the symmetric matrix (a
    // diagonal tile is stored whole: the mirror too)
    for (int s3 = 0; s3 < PB && p0 + s3 < P; ++s3) {
        const Place q = place[s3];
        const double *o = sh + size_t(s3) * per;
        for (int e = t; e < st * st; e += nt) {
            const uint32_t en = entry[e];
            const int r = q.r0 + int(en & 255u), cc = q.c0 + int((en >> 8) & 255u);
            const double v = o[en >> 16];
            const int ri = r & (TS - 1), ci = cc & (TS - 1), br = r >= TS, bc = cc >= TS;
            double *tile = W + q.at + (bc ? q.right : 0) + (br ? q.down : 0);
            tile[ri * TS + ci] = v;
            if (q.diag + bc - br == 0) tile[ci * TS + ri] = v;
        }
    }
}

// Partial products of the packed symmetric matrix.  Workgroup w takes a
// chunk of up to SG consecutive stored tiles of one tile row i, (i, j0) ..
// (i, j0 + ng - 1) (ch[w] = (i, j0, ng, slot)); lane l owns column l of a
// tile, wave v its rows 16 v .. 16 v + 15.  Row sums W_ij x_j build up in
// registers over the chunk and go to part[slot][rows of block i], slot =
// i + (j0 - i)/SG; column sums W_ij^T x_i of each off-diagonal tile go to
// part[i][rows of block j].  For the rows of block b the slots 0 .. b - 1
// hold column sums and b .. b + ceil((nt - b)/SG) - 1 row-sum chunks, each
// written exactly once.  x entries beyond D read as zero.
constexpr int SG = 8;          // tiles per workgroup

// the vectors of a product and their partial sums (two vectors share one pass over W)
template <int NV>
struct SymvArgs {
    const double *x[NV];
    double *part[NV];
};

template <int NV>
__global__ __launch_bounds__(256) void k_symv(const double *__restrict__ W, SymvArgs<NV> a,
                                              const int4 *__restrict__ ch, int D, int nt)
{
    const int4 cw = ch[blockIdx.x];
    const int i = cw.x, j0 = cw.y, ng = cw.z, slot = cw.w;
    const int lane = threadIdx.x & 63;
    const int wv = __builtin_amdgcn_readfirstlane(int(threadIdx.x >> 6));
    const size_t ntT = size_t(nt) * TS;
    const double *tile = W + tile_base(i, j0, nt) + size_t(wv * 16) * TS + lane;
    double xr[NV][16], rp[NV][16];
#pragma unroll
    for (int s = 0; s < NV; ++s)
#pragma unroll
        for (int k = 0; k < 16; ++k) {
            const int ri = i * TS + wv * 16 + k;
            xr[s][k] = ri < D ? a.x[s][ri] : 0.0;
            rp[s][k] = 0.0;
        }
    __shared__ double cs[NV][SG][4][TS];
    double v[16];
#pragma unroll
    for (int k = 0; k < 16; ++k) v[k] = tile[k * TS];
    for (int g = 0; g < ng; ++g) {
        const int cj = (j0 + g) * TS + lane;
#pragma unroll
        for (int s = 0; s < NV; ++s) {
            const double xc = cj < D ? a.x[s][cj] : 0.0;
            double col = 0.0;
#pragma unroll
            for (int k = 0; k < 16; ++k) {
                col = fma(v[k], xr[s][k], col);
                rp[s][k] = fma(v[k], xc, rp[s][k]);
            }
            cs[s][g][wv][lane] = col;
        }
        if (g + 1 < ng) {
            tile += TS * TS;
#pragma unroll
            for (int k = 0; k < 16; ++k) v[k] = tile[k * TS];
        }
    }
    // row sums over the lanes: halve the values held per lane while pairing
    // lanes 32, 16, 8, 4 apart, then add over the last two lane bits; lane l
    // ends with the sum of row 16 v + 8 b5 + 4 b4 + 2 b3 + b2 (b: bits of l)
    const int b5 = (lane >> 5) & 1, b4 = (lane >> 4) & 1, b3 = (lane >> 3) & 1, b2 = (lane >> 2) & 1;
#pragma unroll
    for (int s = 0; s < NV; ++s) {
#pragma unroll
        for (int k = 0; k < 8; ++k) {
            const double send = b5 ? rp[s][k] : rp[s][k + 8], keep = b5 ? rp[s][k + 8] : rp[s][k];
            rp[s][k] = keep + __shfl_xor(send, 32, 64);
        }
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const double send = b4 ? rp[s][k] : rp[s][k + 4], keep = b4 ? rp[s][k + 4] : rp[s][k];
            rp[s][k] = keep + __shfl_xor(send, 16, 64);
        }
#pragma unroll
        for (int k = 0; k < 2; ++k) {
            const double send = b3 ? rp[s][k] : rp[s][k + 2], keep = b3 ? rp[s][k + 2] : rp[s][k];
            rp[s][k] = keep + __shfl_xor(send, 8, 64);
        }
        const double send = b2 ? rp[s][0] : rp[s][1], keep = b2 ? rp[s][1] : rp[s][0];
        double rs = keep + __shfl_xor(send, 4, 64);
        rs += __shfl_xor(rs, 2, 64);
        rs += __shfl_xor(rs, 1, 64);
        if ((lane & 3) == 0) {
            const int r = wv * 16 + 8 * b5 + 4 * b4 + 2 * b3 + b2;
            a.part[s][size_t(slot) * ntT + size_t(i) * TS + r] = rs;
        }
    }
    __syncthreads();
    // column sums of the off-diagonal tiles, the four waves' parts in order
#pragma unroll
    for (int s = 0; s < NV; ++s)
        for (int g = wv; g < ng; g += 4) {
            const int j = j0 + g;
            if (j == i) continue;
            a.part[s][size_t(i) * ntT + size_t(j) * TS + lane] =
                (cs[s][g][0][lane] + cs[s][g][1][lane]) + (cs[s][g][2][lane] + cs[s][g][3][lane]);
        }
}

// Rows GR g .. GR g + GR - 1 of a product from its partial sums: the slots
// 0 .. ns - 1 of a row's block b = R / TS, ns = b + ceil((nt - b)/SG), added by
// four threads per row (slots q, q + 4, ..., four accumulators each), then in
// order.  Called by 4 GR threads; out[GR] in LDS, zero beyond D; ends with a
// barrier.
constexpr int GT = TS;          // (m, n) rows of three per group
constexpr int GR = 3 * GT;      // rows per group: 64 (m, n) triples, three tiles

__device__ __forceinline__ void row_sums(const double *__restrict__ part, int g, int D, int nt, double (&ws)[4][GR],
                                         double (&out)[GR])
{
    const int lr = int(threadIdx.x) % GR, q = int(threadIdx.x) / GR;
    const int r = g * GR + lr, b = r / TS;
    const size_t ntT = size_t(nt) * TS;
    double a0 = 0.0, a1 = 0.0, a2 = 0.0, a3 = 0.0;
    if (r < D) {
        const int ns = b + (nt - b + SG - 1) / SG;
        const double *pc = part + r;
        int t = q;
        for (; t + 12 < ns; t += 16) {
            a0 += pc[size_t(t) * ntT];
            a1 += pc[size_t(t + 4) * ntT];
            a2 += pc[size_t(t + 8) * ntT];
            a3 += pc[size_t(t + 12) * ntT];
        }
        for (; t < ns; t += 4) a0 += pc[size_t(t) * ntT];
    }
    ws[q][lr] = (a0 + a1) + (a2 + a3);
    __syncthreads();
    if (q == 0) out[lr] = (ws[0][lr] + ws[1][lr]) + (ws[2][lr] + ws[3][lr]);
    __syncthreads();
}

// the chunks of k_symv for nt tiles per side: (i, j0, ng, slot) per workgroup
static std::vector<int4> symv_chunks(int nt)
{
    std::vector<int4> out;
    for (int i = 0; i < nt; ++i)
        for (int j0 = i, c = 0; j0 < nt; j0 += SG, ++c) out.push_back(make_int4(i, j0, std::min(SG, nt - j0), i + c));
    return out;
}

static size_t symv_chunk_count(int nt)
{
    size_t n = 0;
    for (int i = 0; i < nt; ++i) n += size_t((nt - i + SG - 1) / SG);
    return n;
}

// per-fiber 3x3 blocks: Lambda = d (I + p p^T) + 2 (I - p p^T), K = I + p p^T
__device__ __forceinline__ void blocks(const double *p, double d, double lam[3][3], double K[3][3], double pp[3][3])
{
    for (int a = 0; a < 3; ++a)
        for (int b = 0; b < 3; ++b) {
            const double ab = p[a] * p[b], id = a == b ? 1.0 : 0.0;
            pp[a][b] = ab;
            K[a][b] = id + ab;
            lam[a][b] = d * (id + ab) + 2.0 * (id - ab);
        }
}

// L_n = -2 sum_{i<=n} 1/i: eigenvalue of the finite-part operator on P_n
__device__ __forceinline__ double kbar_eig(int n)
{
    double s = 0.0;
    for (int i = 1; i <= n; ++i) s += 1.0 / double(i);
    return -2.0 * s;
}

// Rows (m, n) of the system operator from x and z = W x:
//   n >= 2: (Lambda + L_n K) x_n + c_n z_n
//   n  = 1: (I - p p^T) x_1 + p p^T [(Lambda + L_1 K) x_1 + c_1 z_1]
// c_n = (2n + 1)/(2l); rows n = 0 are zero.
__device__ __forceinline__ void apply_row(int n, const double *xi, const double *zi, const double *pm, const Consts &c,
                                          double *yo)
{
    if (n == 0) {
        yo[0] = yo[1] = yo[2] = 0.0;
        return;
    }
    double lam[3][3], K[3][3], pp[3][3];
    blocks(pm, c.d, lam, K, pp);
    const double Ln = kbar_eig(n), cn = (2.0 * n + 1.0) / (2.0 * c.l);
    double v[3];
    for (int a = 0; a < 3; ++a) {
        double s = 0.0;
        for (int b = 0; b < 3; ++b) s += (lam[a][b] + Ln * K[a][b]) * xi[b];
        v[a] = s + cn * zi[a];
    }
    if (n >= 2) {
        for (int a = 0; a < 3; ++a) yo[a] = v[a];
    } else {
        const double pv = pm[0] * v[0] + pm[1] * v[1] + pm[2] * v[2];
        const double px = pm[0] * xi[0] + pm[1] * xi[1] + pm[2] * xi[2];
        for (int a = 0; a < 3; ++a) yo[a] = (xi[a] - pm[a] * px) + pm[a] * pv;
    }
}

// Block-Jacobi preconditioner: out_{m,n} = B_{m,n}^{-1} in_{m,n} with the
// self blocks of the operator, all of the form alpha I + beta p p^T:
//   n >= 2: Lambda + L_n K = (d + 2 + L_n) I + (d - 2 + L_n) p p^T,
//   n  = 1: (I - p p^T) + p p^T (Lambda + L_1 K) = I + (2 d + 2 L_1 - 1) p p^T,
// inverted in closed form, (alpha I + beta p p^T)^-1 =
// (I - beta/(alpha + beta) p p^T)/alpha.  GMRES runs on the right-
// preconditioned operator A B^-1; the self part then is the identity and
// the iteration count reflects the interactions only.
__device__ __forceinline__ void precond_row(int n, const double *xi, const double *pm, const Consts &c, double *yo)
{
    if (n == 0) {
        yo[0] = yo[1] = yo[2] = 0.0;
        return;
    }
    const double Ln = kbar_eig(n);
    const double alpha = n == 1 ? 1.0 : c.d + 2.0 + Ln;
    const double beta = n == 1 ? 2.0 * c.d + 2.0 * Ln - 1.0 : c.d - 2.0 + Ln;
    const double px = pm[0] * xi[0] + pm[1] * xi[1] + pm[2] * xi[2];
    const double f = beta / (alpha + beta);
    for (int a = 0; a < 3; ++a) yo[a] = (xi[a] - f * px * pm[a]) / alpha;
}

// right-hand side from z0 = W [F/(2l); 0]:
//   n = 1: 3/(2 l^2) M x p - c_1 p p^T z0_1;  n >= 2: -c_n z0_n;  n = 0: 0
__device__ __forceinline__ void rhs_row(int n, const double *zi, const double *pm, const double *mm, const Consts &c,
                                        double *bo)
{
    if (n == 0) {
        bo[0] = bo[1] = bo[2] = 0.0;
        return;
    }
    const double cn = (2.0 * n + 1.0) / (2.0 * c.l);
    if (n >= 2) {
        for (int a = 0; a < 3; ++a) bo[a] = -cn * zi[a];
        return;
    }
    const double mxp[3] = {mm[1] * pm[2] - mm[2] * pm[1], mm[2] * pm[0] - mm[0] * pm[2], mm[0] * pm[1] - mm[1] * pm[0]};
    const double pz = pm[0] * zi[0] + pm[1] * zi[1] + pm[2] * zi[2];
    const double tq = 3.0 / (2.0 * c.l * c.l);
    for (int a = 0; a < 3; ++a) bo[a] = tq * mxp[a] - cn * pm[a] * pz;
}

// the known part of the force as a vector of the (m, k, b) layout:
// F_m/(2l) in the k = 0 entries, zero elsewhere
__device__ __forceinline__ double known_entry(int e, const double *F, const Consts &c)
{
    const int b = e % 3, k = (e / 3) % (c.N + 1), m = e / (3 * (c.N + 1));
    return k == 0 ? F[3 * m + b] / (2.0 * c.l) : 0.0;
}
__global__ __launch_bounds__(256) void k_known(double *__restrict__ v, const double *__restrict__ F, Consts c)
{
    const int e = int(blockIdx.x * blockDim.x + threadIdx.x);
    if (e < c.D) v[e] = known_entry(e, F, c);
}

// velocities of fiber m from z = W [F/(2l); a] (rows n = 0: int U ds, n = 1:
// int U P_1 ds):
//   dx/dt = (Lambda F + z_0) / (8 pi mu L)
//   dp/dt = 3/(2 pi mu L^3) [d M x p + (I - p p^T) l z_1]
__device__ __forceinline__ void velocity_of(const double z0[3], const double z1[3], const double *pm, const double *f,
                                            const double *mm, const Consts &c, double *V, double *Pd)
{
    double lam[3][3], K[3][3], pp[3][3];
    blocks(pm, c.d, lam, K, pp);
    const double kv = 1.0 / (8.0 * M_PI * c.mu * c.L);
    const double kw = 3.0 / (2.0 * M_PI * c.mu * c.L * c.L * c.L);
    const double mxp[3] = {mm[1] * pm[2] - mm[2] * pm[1], mm[2] * pm[0] - mm[0] * pm[2], mm[0] * pm[1] - mm[1] * pm[0]};
    const double pz = pm[0] * z1[0] + pm[1] * z1[1] + pm[2] * z1[2];
    for (int a = 0; a < 3; ++a) {
        double s = 0.0;
        for (int b = 0; b < 3; ++b) s += lam[a][b] * f[b];
        V[a] = kv * (s + z0[a]);
        Pd[a] = kw * (c.d * mxp[a] + c.l * (z1[a] - pm[a] * pz));
    }
}

// z = zk + zx: the products with the known and the unknown part
__global__ __launch_bounds__(256) void k_velocity(const double *__restrict__ zk, const double *__restrict__ zx,
                                                  const double *__restrict__ p, const double *__restrict__ F,
                                                  const double *__restrict__ Mt, double *__restrict__ V,
                                                  double *__restrict__ Pd, Consts c)
{
    const int m = int(blockIdx.x * blockDim.x + threadIdx.x);
    if (m >= c.M) return;
    const size_t o = size_t(3) * m * (c.N + 1);
    double z[6];
    for (int a = 0; a < 6; ++a) z[a] = zk[o + a] + zx[o + a];
    velocity_of(z, z + 3, p + 3 * m, F + 3 * m, Mt + 3 * m, c, V + 3 * m, Pd + 3 * m);
}

// ------------------------------------------------------------------ GMRES pieces
// An iteration is five launches: the product's partial sums (k_symv), the rows
// of A B^-1 v_i with the first dot products (k_apply_dots), the two Gram-
// Schmidt passes (k_orth), and the new basis vector with the rotation of its
// column (k_next).  Every dot product is summed per group of GR rows into
// part[j][group], and each workgroup of the next launch adds the groups'
// sums itself (a few thousand doubles from L2), so no launch is spent on a
// reduction.  All orders of summation are fixed.

__device__ __forceinline__ double wave_sum(double s)
{
    for (int o = 32; o > 0; o >>= 1) s += __shfl_xor(s, o, 64);
    return s;
}

// <V_j, w> over the group's rows w[GR] (LDS) for j < nj, one wave per j
__device__ __forceinline__ void group_dots(const double *__restrict__ Vb, const double (&w)[GR], double *__restrict__ part,
                                           int nj, int g, int G, int D)
{
    const int lane = threadIdx.x & 63;
    for (int j = int(threadIdx.x >> 6); j < nj; j += int(blockDim.x >> 6)) {
        const double *v = Vb + size_t(j) * D + size_t(g) * GR;
        double s = 0.0;
#pragma unroll
        for (int k = 0; k < 3; ++k)
            if (g * GR + lane + 64 * k < D) s += v[lane + 64 * k] * w[lane + 64 * k];
        s = wave_sum(s);
        if (lane == 0) part[size_t(j) * G + g] = s;
    }
}

// h[j] = sum over the G groups of part[j], j < nj, in LDS; ends with a barrier
__device__ __forceinline__ void group_totals(const double *__restrict__ part, double *h, int nj, int G)
{
    const int lane = threadIdx.x & 63;
    for (int j = int(threadIdx.x >> 6); j < nj; j += int(blockDim.x >> 6)) {
        double s = 0.0;
        for (int g = lane; g < G; g += 64) s += part[size_t(j) * G + g];
        s = wave_sum(s);
        if (lane == 0) h[j] = s;
    }
    __syncthreads();
}

// rows of z = W x from the partial sums (a plain product)
__global__ __launch_bounds__(4 * GR) void k_rows(const double *__restrict__ part, double *__restrict__ z, int D, int nt)
{
    __shared__ double ws[4][GR], zs[GR];
    row_sums(part, int(blockIdx.x), D, nt, ws, zs);
    const int lr = int(threadIdx.x), r = int(blockIdx.x) * GR + lr;
    if (lr < GR && r < D) z[r] = zs[lr];
}

// z = W t from the partial sums, w = A t, and the group's <V_j, w>, j < nj
__global__ __launch_bounds__(4 * GR) void k_apply_dots(const double *__restrict__ part, const double *__restrict__ t,
                                                       const double *__restrict__ p, const double *__restrict__ Vb,
                                                       double *__restrict__ z, double *__restrict__ w,
                                                       double *__restrict__ dp, int nj, int G, Consts c)
{
    __shared__ double ws[4][GR], zs[GR], wr[GR];
    const int g = int(blockIdx.x), lr = int(threadIdx.x);
    row_sums(part, g, c.D, c.nt, ws, zs);
    if (lr < GT) {
        const int e = g * GT + lr, NP1 = c.N + 1;
        double y[3] = {0.0, 0.0, 0.0};
        if (e < c.M * NP1) apply_row(e % NP1, t + size_t(3) * e, zs + 3 * lr, p + 3 * (e / NP1), c, y);
        for (int a = 0; a < 3; ++a) wr[3 * lr + a] = y[a];
    }
    __syncthreads();
    const int r = g * GR + lr;
    if (lr < GR && r < c.D) {
        z[r] = zs[lr];
        w[r] = wr[lr];
    }
    group_dots(Vb, wr, dp, nj, g, G, c.D);
}

// One Gram-Schmidt pass: h[j] = sum of part_in[j], w -= sum_j h[j] V_j, then
// the group's <V_j, w> (first pass) or <w, w> (second) into part_out.
__global__ __launch_bounds__(256) void k_orth(const double *__restrict__ Vb, double *__restrict__ w,
                                              const double *__restrict__ part_in, double *__restrict__ part_out,
                                              double *__restrict__ h_out, int nj, int G, int D, int second)
{
    __shared__ double h[MAXR + 1], wr[GR];
    const int g = int(blockIdx.x), lr = int(threadIdx.x), r = g * GR + lr;
    group_totals(part_in, h, nj, G);
    if (g == 0 && lr < nj) h_out[lr] = h[lr];
    if (lr < GR) {
        double s = 0.0;
        if (r < D) {
            s = w[r];
            for (int j = 0; j < nj; ++j) s -= h[j] * Vb[size_t(j) * D + r];
            w[r] = s;
        }
        wr[lr] = s;
    }
    __syncthreads();
    if (!second) {
        group_dots(Vb, wr, part_out, nj, g, G, D);
    } else if (lr < 64) {
        const double s = wave_sum(wr[lr] * wr[lr] + wr[lr + 64] * wr[lr + 64] + wr[lr + 128] * wr[lr + 128]);
        if (lr == 0) part_out[g] = s;
    }
}

// Column i of H from the two passes' sums and the norm of w: Givens rotations
// of the column, the residual |g[i+1]| returned.  One thread.
__device__ __forceinline__ double rotate_column(double *H, int ld, const double *h1, const double *h2, double norm,
                                                double *cs, double *sn, double *g, int i)
{
    double cur = h1[0] + h2[0];
    for (int j = 0; j < i; ++j) {
        const double nxt = h1[j + 1] + h2[j + 1];
        H[j * ld + i] = cs[j] * cur + sn[j] * nxt;
        cur = -sn[j] * cur + cs[j] * nxt;
    }
    const double rr = sqrt(cur * cur + norm * norm);
    const double c = rr > 0.0 ? cur / rr : 1.0, s = rr > 0.0 ? norm / rr : 0.0;
    cs[i] = c;
    sn[i] = s;
    H[i * ld + i] = rr;
    g[i + 1] = -s * g[i];
    g[i] = c * g[i];
    return fabs(g[i + 1]);
}

// V_{i+1} = w/|w| (zero when the Krylov space is exhausted) and t = B^-1 V_{i+1};
// workgroup 0 also rotates column i and leaves the residual in host memory.
__global__ __launch_bounds__(256) void k_next(const double *__restrict__ w, double *__restrict__ vn,
                                              double *__restrict__ t, const double *__restrict__ p,
                                              const double *__restrict__ part, double *__restrict__ H,
                                              const double *__restrict__ h1, const double *__restrict__ h2,
                                              double *__restrict__ cs, double *__restrict__ sn, double *__restrict__ g,
                                              double *__restrict__ res, int i, int G, Consts c)
{
    __shared__ double nn[1];
    group_totals(part, nn, 1, G);
    const double n = sqrt(nn[0]);
    const int e = int(blockIdx.x * blockDim.x + threadIdx.x), NP1 = c.N + 1;
    if (e < c.M * NP1) {
        double v[3], y[3];
        for (int a = 0; a < 3; ++a) {
            v[a] = n > 0.0 ? w[size_t(3) * e + a] / n : 0.0;
            vn[size_t(3) * e + a] = v[a];
        }
        precond_row(e % NP1, v, p + 3 * (e / NP1), c, y);
        for (int a = 0; a < 3; ++a) t[size_t(3) * e + a] = y[a];
    }
    if (blockIdx.x == 0 && threadIdx.x == 0) res[i] = rotate_column(H, MAXR, h1, h2, n, cs, sn, g, i);
}

// b from z0 = W [F/(2l); 0], r = b - A x from zx = W x, and the groups' <b, b>
// and <r, r> into part[0][], part[1][]
__global__ __launch_bounds__(GT) void k_start(const double *__restrict__ z0, const double *__restrict__ x,
                                              const double *__restrict__ zx, const double *__restrict__ p,
                                              const double *__restrict__ Mt, double *__restrict__ r,
                                              double *__restrict__ part, int G, Consts c)
{
    const int g = int(blockIdx.x), e = g * GT + int(threadIdx.x), NP1 = c.N + 1;
    double bb = 0.0, rr = 0.0;
    if (e < c.M * NP1) {
        const int n = e % NP1, m = e / NP1;
        double b[3], y[3];
        rhs_row(n, z0 + size_t(3) * e, p + 3 * m, Mt + 3 * m, c, b);
        apply_row(n, x + size_t(3) * e, zx + size_t(3) * e, p + 3 * m, c, y);
        for (int a = 0; a < 3; ++a) {
            const double v = b[a] - y[a];
            r[size_t(3) * e + a] = v;
            bb += b[a] * b[a];
            rr += v * v;
        }
    }
    bb = wave_sum(bb);
    rr = wave_sum(rr);
    if (threadIdx.x == 0) {
        part[g] = bb;
        part[G + g] = rr;
    }
}

// V_0 = r/|r|, t = B^-1 V_0, g[0] = |r|; |b| and |r| to host memory
__global__ __launch_bounds__(256) void k_first(const double *__restrict__ r, double *__restrict__ v0,
                                               double *__restrict__ t, const double *__restrict__ p,
                                               const double *__restrict__ part, double *__restrict__ g,
                                               double *__restrict__ norms, int G, Consts c)
{
    __shared__ double nn[2];
    group_totals(part, nn, 2, G);
    const double n = sqrt(nn[1]);
    const int e = int(blockIdx.x * blockDim.x + threadIdx.x), NP1 = c.N + 1;
    if (e < c.M * NP1) {
        double v[3], y[3];
        for (int a = 0; a < 3; ++a) {
            v[a] = n > 0.0 ? r[size_t(3) * e + a] / n : 0.0;
            v0[size_t(3) * e + a] = v[a];
        }
        precond_row(e % NP1, v, p + 3 * (e / NP1), c, y);
        for (int a = 0; a < 3; ++a) t[size_t(3) * e + a] = y[a];
    }
    if (blockIdx.x == 0 && threadIdx.x == 0) {
        g[0] = n;
        norms[0] = sqrt(nn[0]);
        norms[1] = n;
    }
}

// back substitution H y = g over k <= 64 columns by one wave: lane j holds g_j
__global__ __launch_bounds__(64) void k_backsolve(const double *__restrict__ H, const double *__restrict__ g,
                                                  double *__restrict__ y, int k)
{
    const int j = int(threadIdx.x);
    double s = j < k ? g[j] : 0.0;
    for (int i = k - 1; i >= 0; --i) {
        const double d = H[i * MAXR + i], yi = d != 0.0 ? __shfl(s, i, 64) / d : 0.0;
        if (j == i) y[i] = yi;
        if (j < i) s -= H[j * MAXR + i] * yi;
    }
}

// x += B^-1 sum_j y_j V_j and zx += sum_j y_j Z_j, Z_j = W B^-1 V_j kept from the
// iterations: zx stays W x without another product
__global__ __launch_bounds__(256) void k_update(double *__restrict__ x, double *__restrict__ zx,
                                                const double *__restrict__ Vb, const double *__restrict__ Zb,
                                                const double *__restrict__ y, const double *__restrict__ p, int k,
                                                Consts c)
{
    const int e = int(blockIdx.x * blockDim.x + threadIdx.x), NP1 = c.N + 1;
    if (e >= c.M * NP1) return;
    double v[3] = {0.0, 0.0, 0.0}, z[3] = {0.0, 0.0, 0.0}, u[3];
    for (int j = 0; j < k; ++j) {
        const double yj = y[j];
        for (int a = 0; a < 3; ++a) {
            v[a] += yj * Vb[size_t(j) * c.D + size_t(3) * e + a];
            z[a] += yj * Zb[size_t(j) * c.D + size_t(3) * e + a];
        }
    }
    precond_row(e % NP1, v, p + 3 * (e / NP1), c, u);
    for (int a = 0; a < 3; ++a) {
        x[size_t(3) * e + a] += u[a];
        zx[size_t(3) * e + a] += z[a];
    }
}

// GMRES start of a time step: the linear extrapolation 2 a_n - a_{n-1} of
// the last two solutions (x holds a_n, xh a_{n-1}); xh takes a_n
__global__ __launch_bounds__(256) void k_extrap(double *__restrict__ x, double *__restrict__ xh, int D)
{
    const int e = int(blockIdx.x * blockDim.x + threadIdx.x);
    if (e >= D) return;
    const double a = x[e];
    x[e] = 2.0 * a - xh[e];
    xh[e] = a;
}

// Adams-Bashforth 2 of fiber m (Euler when first), p renormalised
__device__ __forceinline__ void advance_fiber(double *X, double *p, const double *V, const double *Pd, double *Vp,
                                              double *Pp, double dt, bool first)
{
    double q[3];
    for (int a = 0; a < 3; ++a) {
        const double v = V[a], w = Pd[a];
        const double dv = first ? v : 1.5 * v - 0.5 * Vp[a];
        const double dw = first ? w : 1.5 * w - 0.5 * Pp[a];
        X[a] += dt * dv;
        q[a] = p[a] + dt * dw;
        Vp[a] = v;
        Pp[a] = w;
    }
    const double n = sqrt(q[0] * q[0] + q[1] * q[1] + q[2] * q[2]);
    for (int a = 0; a < 3; ++a) p[a] = q[a] / n;
}
__global__ __launch_bounds__(256) void k_advance(double *__restrict__ X, double *__restrict__ p,
                                                 const double *__restrict__ V, const double *__restrict__ Pd,
                                                 double *__restrict__ Vp, double *__restrict__ Pp, int M, double dt,
                                                 int first)
{
    const int m = int(blockIdx.x * blockDim.x + threadIdx.x);
    if (m < M) advance_fiber(X + 3 * m, p + 3 * m, V + 3 * m, Pd + 3 * m, Vp + 3 * m, Pp + 3 * m, dt, first != 0);
}

#include "sbf_small.h"

}  // namespace sbfk

using namespace sbfk;

struct sbf_ctx {
    sbf_params p{};
    std::string err;
    hipStream_t st = nullptr;
    bool own_stream = false;
    Consts c{};
    int M = 0, Dmax = 0;
    // device
    double *X = nullptr, *pd = nullptr, *F = nullptr, *Mt = nullptr;
    double *wl = nullptr, *wj = nullptr;   // weights times P_k at the nodes, by k; nodes and the same by node
    double *W = nullptr;                   // packed upper triangle of the moment matrix
    double *part = nullptr, *part2 = nullptr;   // [nt][nt TS] partial sums of a product with W (of two vectors)
    int4 *chunks = nullptr;                // work list of the product kernel
    double *dpart = nullptr;               // [3][MAXR + 1][groups] dot products per group of rows
    int gmax = 0;                          // groups of Dmax rows
    unsigned nchunks = 0;
    double *x = nullptr, *r = nullptr, *w = nullptr, *kn = nullptr;
    double *z0 = nullptr, *zx = nullptr;   // products of W with the known part and with x
    double *t = nullptr;                   // preconditioned basis vector
    double *Zb = nullptr;                  // [restart][D] W B^-1 V_j
    double *xh = nullptr;                   // the solution of the previous time step
    int nsol = 0;                           // solutions of time steps since the fibers were set
    double *Vb = nullptr;                   // [restart + 1][D]
    double *H = nullptr, *cs = nullptr, *sn = nullptr, *g = nullptr, *h1 = nullptr, *h2 = nullptr, *ys = nullptr;
    double *resh = nullptr;                 // pinned host memory: the residual of each iteration, then |b|, |r|
    SmallResult *small = nullptr;           // pinned host memory: what a one-workgroup solve reports
    hipEvent_t rev[MAXR] = {};              // recorded after each iteration
    double *V = nullptr, *Pd = nullptr, *Vp = nullptr, *Pp = nullptr;
    bool first = true, solved = false;
    // event timing: pairs recorded around the moment kernel and each GEMV
    bool timing = false;
    std::vector<hipEvent_t> ev;
    size_t ev_used = 0;
    std::vector<int> ev_kind;    // 0 moments, 1 GEMV
    double t_theta = 0.0, t_gemv = 0.0;
    int64_t n_theta = 0, n_gemv = 0;
    int iters = 0;
    double relres = 0.0;
    int64_t steps = 0;
};

static lbm_status sfail(sbf_ctx *c, lbm_status s, const std::string &m)
{
    if (c) c->err = m;
    return s;
}

#define SCHK(c, call)                                                                                  \
    do {                                                                                               \
        hipError_t e_ = (call);                                                                        \
        if (e_ != hipSuccess)                                                                          \
            return sfail((c), e_ == hipErrorOutOfMemory ? LBM_E_NOMEM : LBM_E_HIP,                     \
                         std::string(#call) + ": " + hipGetErrorString(e_));                           \
    } while (0)

static inline unsigned nblk(size_t n) { return unsigned((n + 255) / 256); }

// launch of the moment kernel for the compile-time number of modes
template <int NP1>
static hipError_t theta_t(sbf_ctx *c)
{
    const int Q = c->c.Q;
    if (c->M < 2) return hipSuccess;
    // pairs per workgroup: the most lanes busy (PB Q over whole waves), then
    // the most pairs, within 64 KiB of LDS (Q > 128: one pair)
    const size_t per = size_t(theta_lds(NP1, Q)) * sizeof(double), most = 65536 - 7168;   // and the static part
    int pb = 1;
    double best = 0.0;
    for (int k = 1; k * Q <= 256 && size_t(k) * per <= most; ++k) {
        const double use = double(k * Q) / double(((k * Q + 63) / 64) * 64);
        if (use >= best) {
            best = use;
            pb = k;
        }
    }
    const unsigned threads = unsigned(((pb * Q + 63) / 64) * 64);
    const int P = int((long long)c->M * (c->M - 1) / 2);
    hipLaunchKernelGGL((k_theta<NP1>), dim3(unsigned((P + pb - 1) / pb)), dim3(threads), size_t(pb) * per, c->st, c->X,
                       c->pd, c->c, c->wj, c->wl, c->W, pb, P);
    return hipGetLastError();
}

static hipError_t launch_theta(sbf_ctx *c)
{
    switch (c->c.N + 1) {
    case 2: return theta_t<2>(c);
    case 3: return theta_t<3>(c);
    case 4: return theta_t<4>(c);
    case 5: return theta_t<5>(c);
    case 6: return theta_t<6>(c);
    case 7: return theta_t<7>(c);
    case 8: return theta_t<8>(c);
    default: return theta_t<9>(c);
    }
}

// an event pair around the next launch when timing (kind 0: moments, 1: GEMV)
static hipError_t mark(sbf_ctx *c, int kind, bool begin)
{
    if (!c->timing) return hipSuccess;
    if (begin) {
        while (c->ev.size() < c->ev_used + 2) {
            hipEvent_t e;
            hipError_t r = hipEventCreate(&e);
            if (r != hipSuccess) return r;
            c->ev.push_back(e);
        }
        c->ev_kind.resize(c->ev.size() / 2 + 1);
        c->ev_kind[c->ev_used / 2] = kind;
    }
    return hipEventRecord(c->ev[c->ev_used++], c->st);
}

// after a synchronisation: add the recorded pairs to the totals
static hipError_t collect(sbf_ctx *c)
{
    for (size_t i = 0; i + 1 < c->ev_used; i += 2) {
        float ms = 0.0f;
        hipError_t r = hipEventElapsedTime(&ms, c->ev[i], c->ev[i + 1]);
        if (r != hipSuccess) return r;
        if (c->ev_kind[i / 2] == 0) {
            c->t_theta += ms;
            c->n_theta += 1;
        } else {
            c->t_gemv += ms;
            c->n_gemv += 1;
        }
    }
    c->ev_used = 0;
    return hipSuccess;
}

// partial sums of W xin into c->part
static hipError_t product(sbf_ctx *c, const double *xin)
{
    SymvArgs<1> a{{xin}, {c->part}};
    hipLaunchKernelGGL(k_symv<1>, dim3(c->nchunks), dim3(256), 0, c->st, c->W, a, c->chunks, c->c.D, c->c.nt);
    return hipGetLastError();
}

// moments, right-hand side, GMRES (right block-Jacobi preconditioning, from
// the previous solution), velocities
static lbm_status do_solve(sbf_ctx *c)
{
    const int D = c->c.D, G = (D + GR - 1) / GR;
    const dim3 gg{unsigned(G)}, ge{nblk(size_t(c->M) * (c->c.N + 1))}, b256{256}, b4{4 * GR};
    double *dp[3] = {c->dpart, c->dpart + size_t(MAXR + 1) * c->gmax, c->dpart + 2 * size_t(MAXR + 1) * c->gmax};
    double *norms = c->resh + MAXR;
    SCHK(c, mark(c, 0, true));
    SCHK(c, launch_theta(c));
    SCHK(c, mark(c, 0, false));
    // one pass over W for the known part and the start vector
    SCHK(c, mark(c, 1, true));
    SymvArgs<2> two{{c->kn, c->x}, {c->part, c->part2}};
    hipLaunchKernelGGL(k_symv<2>, dim3(c->nchunks), b256, 0, c->st, c->W, two, c->chunks, D, c->c.nt);
    hipLaunchKernelGGL(k_rows, gg, b4, 0, c->st, c->part, c->z0, D, c->c.nt);
    hipLaunchKernelGGL(k_rows, gg, b4, 0, c->st, c->part2, c->zx, D, c->c.nt);
    SCHK(c, hipGetLastError());
    SCHK(c, mark(c, 1, false));
    const int R = c->p.gmres_restart;
    int it = 0;
    double rel = 0.0;
    bool conv = false, restart = false;
    while (!conv && it < c->p.gmres_maxit) {
        if (restart) {
            SCHK(c, mark(c, 1, true));
            SCHK(c, product(c, c->x));
            hipLaunchKernelGGL(k_rows, gg, b4, 0, c->st, c->part, c->zx, D, c->c.nt);
            SCHK(c, hipGetLastError());
            SCHK(c, mark(c, 1, false));
        }
        restart = true;
        // r = b - A x, V_0 = r/|r|, g = (|r|, 0, ...)
        hipLaunchKernelGGL(k_start, gg, dim3(GT), 0, c->st, c->z0, c->x, c->zx, c->pd, c->Mt, c->r, dp[0], G, c->c);
        hipLaunchKernelGGL(k_first, ge, b256, 0, c->st, c->r, c->Vb, c->t, c->pd, dp[0], c->g, norms, G, c->c);
        SCHK(c, hipGetLastError());
        SCHK(c, hipStreamSynchronize(c->st));
        SCHK(c, collect(c));
        const double bnorm = norms[0];
        if (bnorm == 0.0) {
            SCHK(c, hipMemsetAsync(c->x, 0, size_t(D) * sizeof(double), c->st));
            SCHK(c, hipMemsetAsync(c->zx, 0, size_t(D) * sizeof(double), c->st));
            rel = 0.0;
            conv = true;
            break;
        }
        rel = norms[1] / bnorm;
        if (rel <= c->p.gmres_tol) {
            conv = true;
            break;
        }
        int k = 0;
        for (int i = 0; i < R && it < c->p.gmres_maxit; ++i) {
            SCHK(c, mark(c, 1, true));
            SCHK(c, product(c, c->t));
            hipLaunchKernelGGL(k_apply_dots, gg, b4, 0, c->st, c->part, c->t, c->pd, c->Vb, c->Zb + size_t(i) * D, c->w,
                               dp[0], i + 1, G, c->c);
            SCHK(c, hipGetLastError());
            SCHK(c, mark(c, 1, false));
            // classical Gram-Schmidt, twice
            hipLaunchKernelGGL(k_orth, gg, b256, 0, c->st, c->Vb, c->w, dp[0], dp[1], c->h1, i + 1, G, D, 0);
            hipLaunchKernelGGL(k_orth, gg, b256, 0, c->st, c->Vb, c->w, dp[1], dp[2], c->h2, i + 1, G, D, 1);
            hipLaunchKernelGGL(k_next, ge, b256, 0, c->st, c->w, c->Vb + size_t(i + 1) * D, c->t, c->pd, dp[2], c->H,
                               c->h1, c->h2, c->cs, c->sn, c->g, c->resh, i, G, c->c);
            SCHK(c, hipGetLastError());
            // the host tests the previous iteration's residual while this
            // one runs, so the stream never drains for the test (at most one
            // iteration more than needed, which only lowers the residual)
            SCHK(c, hipEventRecord(c->rev[i], c->st));
            ++it;
            k = i + 1;
            if (i >= 1) {
                SCHK(c, hipEventSynchronize(c->rev[i - 1]));
                rel = c->resh[i - 1] / bnorm;
                if (rel <= c->p.gmres_tol) {
                    conv = true;
                    break;
                }
            }
        }
        if (!conv && k > 0) {
            SCHK(c, hipEventSynchronize(c->rev[k - 1]));
            rel = c->resh[k - 1] / bnorm;
            conv = rel <= c->p.gmres_tol;
        }
        hipLaunchKernelGGL(k_backsolve, dim3(1), dim3(64), 0, c->st, c->H, c->g, c->ys, k);
        hipLaunchKernelGGL(k_update, ge, b256, 0, c->st, c->x, c->zx, c->Vb, c->Zb, c->ys, c->pd, k, c->c);
        SCHK(c, hipGetLastError());
    }
    hipLaunchKernelGGL(k_velocity, dim3(nblk(size_t(c->M))), b256, 0, c->st, c->z0, c->zx, c->pd, c->F, c->Mt, c->V,
                       c->Pd, c->c);
    SCHK(c, hipGetLastError());
    c->iters = it;
    c->relres = rel;
    c->solved = true;
    return conv ? LBM_OK : sfail(c, LBM_E_UNSTABLE, "GMRES did not reach the tolerance");
}

// Whether the one-workgroup form takes this system: matrix, basis and
// vectors fit the LDS of one CU (with the event timing off, which brackets
// single kernels).  M = 2, N = 5, seven iterations: 0.276 ms per step with a launch
// for each kernel, 0.046 ms in one.
static bool small_form(const sbf_ctx *c)
{
    return !c->timing && small_lds(c->M, c->c.N + 1, c->c.Q, c->p.gmres_restart) <= SMALL_LDS;
}

template <int NP1>
static hipError_t small_t(sbf_ctx *c, const SmallArgs &a)
{
    const size_t lds = small_lds(c->M, NP1, c->c.Q, c->p.gmres_restart);
    hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void *>(&k_small<NP1>),
                                       hipFuncAttributeMaxDynamicSharedMemorySize, int(lds));
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL((k_small<NP1>), dim3(1), dim3(SMALL_T), lds, c->st, a);
    return hipGetLastError();
}

// n time steps (n = 0: one solve without moving the fibers) in one launch
static lbm_status do_small(sbf_ctx *c, int n, double dt)
{
    SmallArgs a{};
    a.c = c->c;
    a.X = c->X;
    a.p = c->pd;
    a.F = c->F;
    a.Mt = c->Mt;
    a.x = c->x;
    a.xh = c->xh;
    a.V = c->V;
    a.Pd = c->Pd;
    a.Vp = c->Vp;
    a.Pp = c->Pp;
    a.wj = c->wj;
    a.out = c->small;
    a.tol = c->p.gmres_tol;
    a.dt = dt;
    a.restart = c->p.gmres_restart;
    a.maxit = c->p.gmres_maxit;
    a.nsteps = n;
    a.nsol = c->nsol;
    a.first = c->first ? 1 : 0;
    hipError_t e = hipSuccess;
    switch (c->c.N + 1) {
    case 2: e = small_t<2>(c, a); break;
    case 3: e = small_t<3>(c, a); break;
    case 4: e = small_t<4>(c, a); break;
    case 5: e = small_t<5>(c, a); break;
    case 6: e = small_t<6>(c, a); break;
    case 7: e = small_t<7>(c, a); break;
    case 8: e = small_t<8>(c, a); break;
    default: e = small_t<9>(c, a); break;
    }
    SCHK(c, e);
    SCHK(c, hipStreamSynchronize(c->st));
    const SmallResult r = *c->small;
    c->iters = r.iters;
    c->relres = r.relres;
    c->solved = true;
    if (r.steps > 0) {
        c->first = false;
        c->steps += r.steps;
        c->nsol += r.steps;
    }
    return r.converged ? LBM_OK : sfail(c, LBM_E_UNSTABLE, "GMRES did not reach the tolerance");
}

// ====================================================================== ABI
template <typename T>
static hipError_t salloc(T **ptr, size_t n)
{
    *ptr = nullptr;
    return hipMalloc((void **)ptr, std::max<size_t>(n, 1) * sizeof(T));
}

static void release(sbf_ctx *c)
{
    for (hipEvent_t e : c->ev) (void)hipEventDestroy(e);
    c->ev.clear();
    double **bufs[] = {&c->X, &c->pd, &c->F, &c->Mt, &c->wl, &c->wj, &c->W, &c->part, &c->part2, &c->dpart, &c->x,
                       &c->xh, &c->r, &c->w, &c->kn, &c->z0, &c->zx, &c->t, &c->Vb, &c->Zb, &c->H, &c->cs, &c->sn,
                       &c->g, &c->h1, &c->h2, &c->ys, &c->V, &c->Pd, &c->Vp, &c->Pp};
    for (double **b : bufs)
        if (*b) {
            (void)hipFree(*b);
            *b = nullptr;
        }
    if (c->chunks) {
        (void)hipFree(c->chunks);
        c->chunks = nullptr;
    }
    if (c->resh) {
        (void)hipHostFree(c->resh);
        c->resh = nullptr;
    }
    if (c->small) {
        (void)hipHostFree(c->small);
        c->small = nullptr;
    }
    for (hipEvent_t &e : c->rev)
        if (e) {
            (void)hipEventDestroy(e);
            e = nullptr;
        }
}

extern "C" {

lbm_status sbf_params_default(sbf_params *p)
{
    if (!p) return LBM_E_ARG;
    std::memset(p, 0, sizeof *p);
    p->max_fibers = 64;
    p->nmodes = 5;
    p->nq = 16;
    p->gmres_restart = 30;
    p->gmres_maxit = 200;
    p->length = 1.0;
    p->eps = 0.1;
    p->mu = 1.0;
    p->gmres_tol = 1e-12;
    return LBM_OK;
}

lbm_status sbf_create(const sbf_params *p, sbf_ctx **out)
{
    if (!p || !out) return LBM_E_ARG;
    *out = nullptr;
    if (p->max_fibers < 1 || p->nmodes < 1 || p->nmodes > MAXN || p->nq < 1 || p->nq > 64 ||
        p->gmres_restart < 1 || p->gmres_restart > MAXR - 1 || p->gmres_maxit < 1)
        return LBM_E_ARG;
    if (!(p->length > 0.0) || !(p->eps > 0.0 && p->eps < 0.5) || !(p->mu > 0.0) || !(p->gmres_tol > 0.0))
        return LBM_E_ARG;
    // the documented range of nq and N (the moment kernel itself needs at most
    // 34 KB of LDS)
    if (size_t(p->nmodes + 1) * 7 * (3 * size_t(p->nq) + size_t(p->nmodes + 1)) * sizeof(double) > 65536) return LBM_E_ARG;
    const double dmax = 3.0 * p->max_fibers * (p->nmodes + 1);
    if (dmax * dmax > 6.0e10) return LBM_E_ARG;   // the packed moment matrix would exceed 240 GB
    sbf_ctx *c = new (std::nothrow) sbf_ctx;
    if (!c) return LBM_E_NOMEM;
    c->p = *p;
    c->st = (hipStream_t)p->stream;
    if (!c->st) {
        if (hipStreamCreateWithFlags(&c->st, hipStreamNonBlocking) != hipSuccess) {
            delete c;
            return LBM_E_HIP;
        }
        c->own_stream = true;
    }
    const int N = p->nmodes, Q = 3 * p->nq, Mx = p->max_fibers, R = p->gmres_restart;
    c->Dmax = 3 * Mx * (N + 1);
    const size_t Dm = size_t(c->Dmax);
    const int ntm = (c->Dmax + TS - 1) / TS;
    c->c.N = N;
    c->c.Q = Q;
    c->c.L = p->length;
    c->c.l = 0.5 * p->length;
    c->c.r = p->eps * p->length;
    c->c.d = -std::log(p->eps * p->eps * std::exp(1.0));
    c->c.mu = p->mu;
    hipError_t e = hipSuccess;
    auto A = [&](double **ptr, size_t n) {
        if (e == hipSuccess) e = salloc(ptr, n);
    };
    A(&c->X, 3 * size_t(Mx));
    A(&c->pd, 3 * size_t(Mx));
    A(&c->F, 3 * size_t(Mx));
    A(&c->Mt, 3 * size_t(Mx));
    A(&c->V, 3 * size_t(Mx));
    A(&c->Pd, 3 * size_t(Mx));
    A(&c->Vp, 3 * size_t(Mx));
    A(&c->Pp, 3 * size_t(Mx));
    A(&c->wl, size_t(Q) * (N + 3));
    A(&c->wj, size_t(Q) * (N + 4));
    A(&c->W, packed_tiles(ntm) * TS * TS);
    A(&c->part, size_t(ntm) * size_t(ntm) * TS);
    A(&c->part2, size_t(ntm) * size_t(ntm) * TS);
    c->gmax = (c->Dmax + GR - 1) / GR;
    A(&c->dpart, 3 * size_t(MAXR + 1) * size_t(c->gmax));
    if (e == hipSuccess) e = hipMalloc((void **)&c->chunks, std::max<size_t>(symv_chunk_count(ntm), 1) * sizeof(int4));
    if (e == hipSuccess) e = hipHostMalloc((void **)&c->resh, (MAXR + 2) * sizeof(double), hipHostMallocDefault);
    if (e == hipSuccess) e = hipHostMalloc((void **)&c->small, sizeof(SmallResult), hipHostMallocDefault);
    for (int i = 0; i < MAXR && e == hipSuccess; ++i) e = hipEventCreateWithFlags(&c->rev[i], hipEventDisableTiming);
    for (double **v : {&c->x, &c->xh, &c->r, &c->w, &c->kn, &c->z0, &c->zx, &c->t}) A(v, Dm);
    A(&c->Vb, Dm * size_t(R + 1));
    A(&c->Zb, Dm * size_t(R));
    A(&c->H, size_t(MAXR) * MAXR);
    for (double **v : {&c->cs, &c->sn, &c->g, &c->h1, &c->h2, &c->ys}) A(v, size_t(MAXR + 1));
    if (e != hipSuccess) {
        release(c);
        if (c->own_stream) (void)hipStreamDestroy(c->st);
        delete c;
        return e == hipErrorOutOfMemory ? LBM_E_NOMEM : LBM_E_HIP;
    }
    // composite three-point Gauss rule on [-l, l] (nodes +-sqrt(3/5), 0;
    // weights 5/9, 8/9, 5/9 on each sub-interval) and P_0..P_N at its nodes
    std::vector<double> sq(Q), wq(Q), leg(size_t(Q) * (N + 3));
    const double gn[3] = {-std::sqrt(0.6), 0.0, std::sqrt(0.6)}, gw[3] = {5.0 / 9.0, 8.0 / 9.0, 5.0 / 9.0};
    const double hstep = 2.0 / p->nq;
    for (int i = 0; i < p->nq; ++i)
        for (int k = 0; k < 3; ++k) {
            const double t = -1.0 + hstep * (i + 0.5) + 0.5 * hstep * gn[k];
            const int j = 3 * i + k;
            sq[j] = c->c.l * t;
            wq[j] = c->c.l * 0.5 * hstep * gw[k];
            double p0 = 1.0, p1 = t;
            leg[j] = 1.0;
            if (N >= 1) leg[size_t(Q) + j] = t;
            for (int n = 1; n < N + 2; ++n) {
                const double p2 = ((2 * n + 1) * t * p1 - n * p0) / (n + 1);
                leg[size_t(n + 1) * Q + j] = p2;
                p0 = p1;
                p1 = p2;
            }
        }
    std::vector<double> wl(leg.size());
    for (int k = 0; k <= N + 2; ++k)
        for (int j = 0; j < Q; ++j) wl[size_t(k) * Q + j] = wq[j] * leg[size_t(k) * Q + j];
    std::vector<double> wj(size_t(Q) * (N + 4));
    for (int j = 0; j < Q; ++j) {
        wj[size_t(j) * (N + 4)] = sq[j];
        for (int k = 0; k <= N + 2; ++k) wj[size_t(j) * (N + 4) + 1 + k] = wl[size_t(k) * Q + j];
    }
    if (hipMemcpyAsync(c->wj, wj.data(), wj.size() * sizeof(double), hipMemcpyHostToDevice, c->st) != hipSuccess ||
        hipMemcpyAsync(c->wl, wl.data(), wl.size() * sizeof(double), hipMemcpyHostToDevice, c->st) != hipSuccess ||
        hipStreamSynchronize(c->st) != hipSuccess) {
        release(c);
        if (c->own_stream) (void)hipStreamDestroy(c->st);
        delete c;
        return LBM_E_HIP;
    }
    *out = c;
    return LBM_OK;
}

lbm_status sbf_destroy(sbf_ctx *c)
{
    if (!c) return LBM_E_ARG;
    (void)hipStreamSynchronize(c->st);
    release(c);
    if (c->own_stream) (void)hipStreamDestroy(c->st);
    delete c;
    return LBM_OK;
}

const char *sbf_last_error(const sbf_ctx *c) { return c ? c->err.c_str() : ""; }

lbm_status sbf_set_fibers(sbf_ctx *c, int32_t m, const double *X, const double *p, const double *F,
                          const double *M)
{
    if (!c) return LBM_E_ARG;
    if (m < 1 || m > c->p.max_fibers || !X || !p) return sfail(c, LBM_E_ARG, "sbf_set_fibers: bad arguments");
    std::vector<double> pn(3 * size_t(m)), zero(3 * size_t(m), 0.0);
    for (int i = 0; i < m; ++i) {
        const double n = std::sqrt(p[3 * i] * p[3 * i] + p[3 * i + 1] * p[3 * i + 1] + p[3 * i + 2] * p[3 * i + 2]);
        if (!(n > 0.0) || !std::isfinite(n)) return sfail(c, LBM_E_ARG, "sbf_set_fibers: zero direction");
        for (int k = 0; k < 3; ++k) pn[3 * i + k] = p[3 * i + k] / n;
    }
    c->M = m;
    c->c.M = m;
    c->c.D = 3 * m * (c->c.N + 1);
    c->c.nt = (c->c.D + TS - 1) / TS;
    const size_t b3 = 3 * size_t(m) * sizeof(double);
    SCHK(c, hipMemcpyAsync(c->X, X, b3, hipMemcpyHostToDevice, c->st));
    SCHK(c, hipMemcpyAsync(c->pd, pn.data(), b3, hipMemcpyHostToDevice, c->st));
    SCHK(c, hipMemcpyAsync(c->F, F ? F : zero.data(), b3, hipMemcpyHostToDevice, c->st));
    SCHK(c, hipMemcpyAsync(c->Mt, M ? M : zero.data(), b3, hipMemcpyHostToDevice, c->st));
    SCHK(c, hipMemsetAsync(c->x, 0, size_t(c->c.D) * sizeof(double), c->st));
    // the diagonal blocks and the padding of the packed matrix stay zero
    SCHK(c, hipMemsetAsync(c->W, 0, packed_tiles(c->c.nt) * TS * TS * sizeof(double), c->st));
    const std::vector<int4> chunks = symv_chunks(c->c.nt);
    c->nchunks = unsigned(chunks.size());
    SCHK(c, hipMemcpyAsync(c->chunks, chunks.data(), chunks.size() * sizeof(int4), hipMemcpyHostToDevice, c->st));
    hipLaunchKernelGGL(k_known, dim3(nblk(size_t(c->c.D))), dim3(256), 0, c->st, c->kn, c->F, c->c);
    SCHK(c, hipGetLastError());
    SCHK(c, hipStreamSynchronize(c->st));
    c->first = true;
    c->solved = false;
    c->steps = 0;
    c->nsol = 0;
    return LBM_OK;
}

lbm_status sbf_solve(sbf_ctx *c)
{
    if (!c) return LBM_E_ARG;
    if (c->M < 1) return sfail(c, LBM_E_STATE, "sbf_solve: no fibers set");
    return small_form(c) ? do_small(c, 0, 0.0) : do_solve(c);
}

lbm_status sbf_get_velocities(sbf_ctx *c, double *V, double *pdot)
{
    if (!c) return LBM_E_ARG;
    if (!c->solved) return sfail(c, LBM_E_STATE, "no solve since the fibers were set");
    const size_t b3 = 3 * size_t(c->M) * sizeof(double);
    if (V) SCHK(c, hipMemcpyAsync(V, c->V, b3, hipMemcpyDeviceToHost, c->st));
    if (pdot) SCHK(c, hipMemcpyAsync(pdot, c->Pd, b3, hipMemcpyDeviceToHost, c->st));
    SCHK(c, hipStreamSynchronize(c->st));
    return LBM_OK;
}

lbm_status sbf_get_coefficients(sbf_ctx *c, double *a)
{
    if (!c || !a) return LBM_E_ARG;
    if (!c->solved) return sfail(c, LBM_E_STATE, "no solve since the fibers were set");
    std::vector<double> h(size_t(c->c.D));
    SCHK(c, hipMemcpyAsync(h.data(), c->x, h.size() * sizeof(double), hipMemcpyDeviceToHost, c->st));
    SCHK(c, hipStreamSynchronize(c->st));
    const int N = c->c.N;
    for (int m = 0; m < c->M; ++m)
        for (int n = 1; n <= N; ++n)
            for (int b = 0; b < 3; ++b) a[(size_t(m) * N + (n - 1)) * 3 + b] = h[(size_t(m) * (N + 1) + n) * 3 + b];
    return LBM_OK;
}

lbm_status sbf_step(sbf_ctx *c, int64_t n, double dt)
{
    if (!c) return LBM_E_ARG;
    if (n < 0 || !(dt > 0.0)) return sfail(c, LBM_E_ARG, "sbf_step: n >= 0 and dt > 0 required");
    if (c->M < 1) return sfail(c, LBM_E_STATE, "sbf_step: no fibers set");
    if (small_form(c)) {
        for (int64_t left = n; left > 0;) {
            const int k = int(std::min<int64_t>(left, SMALL_STEPS));
            const lbm_status st = do_small(c, k, dt);
            if (st != LBM_OK) return st;
            left -= k;
        }
    } else for (int64_t s = 0; s < n; ++s) {
        // GMRES starts from the extrapolation of the last two solutions
        // (from the last one after the first step)
        const unsigned gd = nblk(size_t(c->c.D));
        if (c->nsol >= 2) {
            hipLaunchKernelGGL(k_extrap, dim3(gd), dim3(256), 0, c->st, c->x, c->xh, c->c.D);
            SCHK(c, hipGetLastError());
        } else if (c->nsol == 1) {
            SCHK(c, hipMemcpyAsync(c->xh, c->x, size_t(c->c.D) * sizeof(double), hipMemcpyDeviceToDevice, c->st));
        }
        lbm_status st = do_solve(c);
        if (st != LBM_OK) return st;
        c->nsol += 1;
        hipLaunchKernelGGL(k_advance, dim3(nblk(size_t(c->M))), dim3(256), 0, c->st, c->X, c->pd, c->V, c->Pd,
                           c->Vp, c->Pp, c->M, dt, c->first ? 1 : 0);
        SCHK(c, hipGetLastError());
        c->first = false;
        c->steps += 1;
    }
    SCHK(c, hipStreamSynchronize(c->st));
    return LBM_OK;
}

lbm_status sbf_get_state(sbf_ctx *c, double *X, double *p)
{
    if (!c) return LBM_E_ARG;
    const size_t b3 = 3 * size_t(c->M) * sizeof(double);
    if (X) SCHK(c, hipMemcpyAsync(X, c->X, b3, hipMemcpyDeviceToHost, c->st));
    if (p) SCHK(c, hipMemcpyAsync(p, c->pd, b3, hipMemcpyDeviceToHost, c->st));
    SCHK(c, hipStreamSynchronize(c->st));
    return LBM_OK;
}

lbm_status sbf_get_stats(sbf_ctx *c, int32_t *iterations, double *residual, int64_t *steps)
{
    if (!c) return LBM_E_ARG;
    if (iterations) *iterations = c->iters;
    if (residual) *residual = c->relres;
    if (steps) *steps = c->steps;
    return LBM_OK;
}

lbm_status sbf_enable_timing(sbf_ctx *c, int32_t on)
{
    if (!c) return LBM_E_ARG;
    SCHK(c, hipStreamSynchronize(c->st));
    SCHK(c, collect(c));
    c->timing = on != 0;
    if (c->timing) {
        c->t_theta = c->t_gemv = 0.0;
        c->n_theta = c->n_gemv = 0;
    }
    return LBM_OK;
}

lbm_status sbf_get_timing(sbf_ctx *c, double *moments_ms, int64_t *moments_launches, double *gemv_ms,
                          int64_t *gemv_launches)
{
    if (!c) return LBM_E_ARG;
    SCHK(c, hipStreamSynchronize(c->st));
    SCHK(c, collect(c));
    if (moments_ms) *moments_ms = c->t_theta;
    if (moments_launches) *moments_launches = c->n_theta;
    if (gemv_ms) *gemv_ms = c->t_gemv;
    if (gemv_launches) *gemv_launches = c->n_gemv;
    return LBM_OK;
}

}  // extern "C"

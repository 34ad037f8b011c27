// sbf_small.h -- the slender-body model for a few fibers: whole time steps in
// one workgroup.  Included by sbf.hip inside its namespace.
//
// A pair of fibers has a system of order 36; its solve is some ten products
// of 10 KB each, so in launches of their own the kernels of a step cost only
// their launch latencies (five launches per GMRES iteration).  Here the
// moment matrix, the Krylov basis and every vector stay in the LDS of one CU
// and the phases are separated by workgroup barriers; the moments, the solve,
// the velocities and the Adams-Bashforth update of all requested steps run in
// one launch.  The method and its stopping rule are those of the many-launch
// form (do_solve); sums are taken in other orders, and the velocities from a
// product of their own.  Bound: the serial chain of about ten barriers and one
// product per iteration.

constexpr int SMALL_T = 512;                  // threads
constexpr size_t SMALL_LDS = 150 * 1024;      // of the CU's 160 KiB
constexpr int SMALL_SCRATCH = 5120;           // doubles for the moments of a chunk of pairs
constexpr int SMALL_STEPS = 1024;             // time steps per launch

struct SmallResult {
    int32_t converged, iters, steps, reserved;
    double relres;
};

struct SmallArgs {
    Consts c;
    double *X, *p, *F, *Mt, *x, *xh, *V, *Pd, *Vp, *Pp;
    const double *wj;
    SmallResult *out;                         // pinned host memory
    double tol, dt;
    int restart, maxit, nsteps, nsol, first;
};

// pairs whose moments are formed at a time
__host__ __device__ inline int small_chunk(int M, int np1, int Q)
{
    const int P = M * (M - 1) / 2, fit = SMALL_SCRATCH / theta_lds(np1, Q);
    int ch = SMALL_T / Q;
    ch = ch < P ? ch : P;
    ch = ch < fit ? ch : fit;
    return ch < 1 ? 1 : ch;
}

// doubles shared by the Krylov basis and the moments' scratch
__host__ __device__ inline size_t small_union(int M, int np1, int Q, int R)
{
    const size_t a = size_t(R + 1) * 3 * M * np1, b = size_t(small_chunk(M, np1, Q)) * theta_lds(np1, Q);
    return a > b ? a : b;
}

__host__ __device__ inline size_t small_lds(int M, int np1, int Q, int R)
{
    const size_t D = 3 * size_t(M) * np1;
    if (D > 192) return ~size_t(0);
    return 8 * (D * D + small_union(M, np1, Q, R) + 7 * D + SMALL_T + size_t(R) * R + 7 * size_t(R + 1) + 24 * size_t(M) +
                size_t(Q) * (np1 + 3) + 2 * size_t(np1 + 2) + 8);
}

template <int NP1>
__global__ __launch_bounds__(SMALL_T) void k_small(SmallArgs a)
{
    constexpr int NB = NP1 + 2, NC = NP1 + NB, NCP = theta_cols(NP1), st = 3 * NP1;
    extern __shared__ double sh[];
    const Consts c = a.c;
    const int M = c.M, D = c.D, Q = c.Q, R = a.restart, tid = int(threadIdx.x), lane = tid & 63, wv = tid >> 6;
    const int P = M * (M - 1) / 2, CH = small_chunk(M, NP1, Q), per = theta_lds(NP1, Q), pts = theta_points(NP1, Q);
    int JS = 1;                               // threads that share the inner points of an outer point
    while (JS < 8 && CH * Q * JS * 2 <= SMALL_T) JS *= 2;
    double *W = sh, *Vb = W + D * D, *x = Vb + small_union(M, NP1, Q, R), *xh = x + D, *w = xh + D, *t = w + D;
    double *kn = t + D, *b = kn + D, *z = b + D, *red = z + D, *H = red + SMALL_T, *cs = H + R * R, *sn = cs + R + 1;
    double *g = sn + R + 1, *h1 = g + R + 1, *h2 = h1 + R + 1, *ys = h2 + R + 1, *res = ys + R + 1, *X = res + R + 1;
    double *p = X + 3 * M, *F = p + 3 * M, *Mt = F + 3 * M, *V = Mt + 3 * M, *Pd = V + 3 * M, *Vp = Pd + 3 * M;
    double *Pp = Vp + 3 * M, *wj = Pp + 3 * M, *up = wj + Q * (NB + 1), *dn = up + NB, *sc = dn + NB;
    double *scr = Vb;

    for (int e = tid; e < D * D; e += SMALL_T) W[e] = 0.0;
    for (int e = tid; e < 3 * M; e += SMALL_T) {
        X[e] = a.X[e];
        p[e] = a.p[e];
        F[e] = a.F[e];
        Mt[e] = a.Mt[e];
        if (!a.first) {
            Vp[e] = a.Vp[e];
            Pp[e] = a.Pp[e];
        }
    }
    for (int e = tid; e < D; e += SMALL_T) {
        x[e] = a.x[e];
        xh[e] = a.nsol >= 2 ? a.xh[e] : 0.0;
    }
    for (int e = tid; e < Q * (NB + 1); e += SMALL_T) wj[e] = a.wj[e];
    if (tid < NB) {
        up[tid] = c.l * (tid + 1) / (2 * tid + 1);
        dn[tid] = c.l * tid / (2 * tid + 1);
    }
    __syncthreads();
    for (int e = tid; e < D; e += SMALL_T) kn[e] = known_entry(e, F, c);

    // out = W in; ends with a barrier
    const int rows = (D + 63) / 64 * 64, parts = SMALL_T / rows, pr = tid % rows, pq = tid / rows;
    auto product = [&](const double *in, double *out) {
        double s = 0.0;
        if (pq < parts && pr < D)
            for (int k = pq; k < D; k += parts) s = fma(W[k * D + pr], in[k], s);
        if (pq < parts) red[pq * rows + pr] = s;
        __syncthreads();
        if (tid < D) {
            double v = red[tid];
            for (int k = 1; k < parts; ++k) v += red[k * rows + tid];
            out[tid] = v;
        }
        __syncthreads();
    };
    // out[j] = <v_j, u>, j < nj; ends with a barrier
    auto dots = [&](const double *v, const double *u, double *out, int nj) {
        for (int j = wv; j < nj; j += SMALL_T / 64) {
            double s = 0.0;
            for (int e = lane; e < D; e += 64) s += v[j * D + e] * u[e];
            s = wave_sum(s);
            if (lane == 0) out[j] = s;
        }
        __syncthreads();
    };
    const int np3 = M * NP1;                  // (m, n) rows of three
    int it = 0, done = 0, nsol = a.nsol;
    double rel = 0.0;
    bool conv = false, first = a.first != 0;
    const int solves = a.nsteps > 0 ? a.nsteps : 1;
    for (int step = 0; step < solves; ++step) {
        if (a.nsteps > 0 && tid < D) {
            // start from the extrapolation of the last two solutions
            const double v = x[tid];
            if (nsol >= 2) x[tid] = 2.0 * v - xh[tid];
            if (nsol >= 1) xh[tid] = v;
        }
        // moments, CH pairs at a time
        for (int p0 = 0; p0 < P; p0 += CH) {
            const int grp = tid / JS, js = tid % JS, slot = grp / Q, i = grp % Q;
            const bool act = slot < CH && p0 + slot < P;
            int m = 0, mp = 0;
            double acc[NC];
#pragma unroll
            for (int k = 0; k < NC; ++k) acc[k] = 0.0;
            if (act) {
                pair_of(p0 + slot, M, m, mp);
                const double xm[3] = {X[3 * m], X[3 * m + 1], X[3 * m + 2]}, pm[3] = {p[3 * m], p[3 * m + 1], p[3 * m + 2]};
                const double xn[3] = {X[3 * mp], X[3 * mp + 1], X[3 * mp + 2]};
                const double pn[3] = {p[3 * mp], p[3 * mp + 1], p[3 * mp + 2]};
                if (i == 0 && js == 0) {
                    double *d = scr + slot * per + per - 9;
                    for (int k = 0; k < 3; ++k) {
                        d[k] = xm[k] - xn[k];
                        d[3 + k] = pm[k];
                        d[6 + k] = pn[k];
                    }
                }
                moment_point<NP1>(wj[i * (NB + 1)], xm, pm, xn, pn, 0.5 * c.r * c.r, Q, wj, js, JS, acc);
            }
            for (int o = 1; o < JS; o <<= 1)
#pragma unroll
                for (int k = 0; k < NC; ++k) acc[k] += __shfl_xor(acc[k], o, 64);
            if (act && js == 0)
#pragma unroll
                for (int k = 0; k < NC; ++k) scr[slot * per + i * NCP + k] = acc[k];
            __syncthreads();
            for (int e = tid; e < CH * NC * NB; e += SMALL_T) {
                const int s2 = e / (NC * NB), r = e % (NC * NB), col = r / NB, n = r % NB;
                if (col < NP1 && n >= NP1) continue;
                const double *v = scr + s2 * per + col;
                double s = 0.0;
                for (int q = 0; q < Q; ++q) s = fma(wj[q * (NB + 1) + 1 + n], v[q * NCP], s);
                scr[s2 * per + pts + (col < NP1 ? n * NP1 + col : NP1 * NP1 + n * NB + col - NP1)] = s;
            }
            __syncthreads();
            for (int e = tid; e < CH * NP1 * NP1; e += SMALL_T) {
                const int s2 = e / (NP1 * NP1), nk = e % (NP1 * NP1);
                double *base = scr + s2 * per;
                const double *A = base + pts;
                pair_block<NP1>(nk / NP1, nk % NP1, A, A + NP1 * NP1, base + per - 9, up, dn, base + nk * 6);
            }
            __syncthreads();
            for (int e = tid; e < CH * st * st; e += SMALL_T) {
                const int s3 = e / (st * st), r = e % (st * st), row = r / st, col = r % st;
                if (p0 + s3 >= P) continue;
                int m3, mp3;
                pair_of(p0 + s3, M, m3, mp3);
                const double v = scr[s3 * per + ((row / 3) * NP1 + col / 3) * 6 + sym_index(row % 3, col % 3)];
                W[(m3 * st + row) * D + mp3 * st + col] = v;
                W[(mp3 * st + col) * D + m3 * st + row] = v;
            }
            __syncthreads();
        }
        __syncthreads();
        // right-hand side
        product(kn, z);
        if (tid < np3) rhs_row(tid % NP1, z + 3 * tid, p + 3 * (tid / NP1), Mt + 3 * (tid / NP1), c, b + 3 * tid);
        __syncthreads();
        dots(b, b, sc, 1);
        const double bnorm = sqrt(sc[0]);
        __syncthreads();
        it = 0;
        rel = 0.0;
        conv = false;
        if (bnorm == 0.0) {
            if (tid < D) x[tid] = 0.0;
            conv = true;
        }
        __syncthreads();
        while (!conv && it < a.maxit) {
            product(x, z);
            if (tid < np3) {
                double y[3];
                apply_row(tid % NP1, x + 3 * tid, z + 3 * tid, p + 3 * (tid / NP1), c, y);
                for (int k = 0; k < 3; ++k) w[3 * tid + k] = b[3 * tid + k] - y[k];
            }
            __syncthreads();
            dots(w, w, sc, 1);
            const double rn = sqrt(sc[0]);
            rel = rn / bnorm;
            if (rel <= a.tol) {
                conv = true;
                break;
            }
            if (tid == 0) g[0] = rn;
            int k = 0;
            double norm = rn;
            double *vi = Vb;
            for (int i = 0; i < R && it < a.maxit; ++i) {
                // v_i = w/norm and t = B^-1 v_i
                if (tid < np3) {
                    double v[3];
                    for (int e = 0; e < 3; ++e) {
                        v[e] = norm > 0.0 ? w[3 * tid + e] / norm : 0.0;
                        vi[3 * tid + e] = v[e];
                    }
                    precond_row(tid % NP1, v, p + 3 * (tid / NP1), c, t + 3 * tid);
                }
                __syncthreads();
                product(t, z);
                if (tid < np3) apply_row(tid % NP1, t + 3 * tid, z + 3 * tid, p + 3 * (tid / NP1), c, w + 3 * tid);
                __syncthreads();
                // classical Gram-Schmidt, twice
                for (int pass = 0; pass < 2; ++pass) {
                    double *h = pass ? h2 : h1;
                    dots(Vb, w, h, i + 1);
                    if (tid < D) {
                        double s = w[tid];
                        for (int j = 0; j <= i; ++j) s -= h[j] * Vb[j * D + tid];
                        w[tid] = s;
                    }
                    __syncthreads();
                }
                dots(w, w, sc, 1);
                norm = sqrt(sc[0]);
                if (tid == 0) res[i] = rotate_column(H, R, h1, h2, norm, cs, sn, g, i);
                __syncthreads();
                vi += D;
                ++it;
                k = i + 1;
                if (i >= 1) {
                    rel = res[i - 1] / bnorm;
                    if (rel <= a.tol) {
                        conv = true;
                        break;
                    }
                }
            }
            if (!conv && k > 0) {
                rel = res[k - 1] / bnorm;
                conv = rel <= a.tol;
            }
            // back substitution by wave 0, then x += B^-1 sum_j y_j V_j
            if (wv == 0) {
                double s = lane < k ? g[lane] : 0.0;
                for (int i = k - 1; i >= 0; --i) {
                    const double d = H[i * R + i], si = __shfl(s, i, 64), yi = d != 0.0 ? si / d : 0.0;
                    if (lane == i) ys[i] = yi;
                    if (lane < i) s -= H[lane * R + i] * yi;
                }
            }
            __syncthreads();
            if (tid < np3) {
                double v[3] = {0.0, 0.0, 0.0}, u[3];
                for (int j = 0; j < k; ++j)
                    for (int e = 0; e < 3; ++e) v[e] += ys[j] * Vb[j * D + 3 * tid + e];
                precond_row(tid % NP1, v, p + 3 * (tid / NP1), c, u);
                for (int e = 0; e < 3; ++e) x[3 * tid + e] += u[e];
            }
            __syncthreads();
        }
        // velocities from W [F/(2l); a]
        if (tid < D) t[tid] = x[tid] + kn[tid];
        __syncthreads();
        product(t, z);
        if (tid < M) {
            const double *zm = z + tid * st;
            velocity_of(zm, zm + 3, p + 3 * tid, F + 3 * tid, Mt + 3 * tid, c, V + 3 * tid, Pd + 3 * tid);
        }
        if (!conv || a.nsteps == 0) break;
        ++nsol;
        if (tid < M) advance_fiber(X + 3 * tid, p + 3 * tid, V + 3 * tid, Pd + 3 * tid, Vp + 3 * tid, Pp + 3 * tid, a.dt, first);
        first = false;
        ++done;
        __syncthreads();
    }
    __syncthreads();
    for (int e = tid; e < 3 * M; e += SMALL_T) {
        a.V[e] = V[e];
        a.Pd[e] = Pd[e];
        if (done > 0) {
            a.X[e] = X[e];
            a.p[e] = p[e];
            a.Vp[e] = Vp[e];
            a.Pp[e] = Pp[e];
        }
    }
    if (tid < D) {
        a.x[tid] = x[tid];
        if (a.nsteps > 0) a.xh[tid] = xh[tid];
    }
    if (tid == 0) {
        a.out->converged = conv ? 1 : 0;
        a.out->iters = it;
        a.out->steps = done;
        a.out->relres = rel;
    }
}

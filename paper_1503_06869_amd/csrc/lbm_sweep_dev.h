// lbm_sweep_dev.h -- device functions of the stream-collide update shared by
// the single-lattice kernels (sweep.hip) and the batched kernel (batched.hip):
// storage conversions, the TRT collision, the AA update of one cell with
// wall and fiber bounce-back, and the momentum-exchange terms of a link.
#pragma once
#include "lbm_dev.h"
#include <type_traits>

namespace lbm {

// ------------------------------------------------------------------ storage
// collision type R, and the load and store of a stored value
template <typename S>
struct St;
template <>
struct St<float> {
    using R = float;
    static __device__ __forceinline__ float ld(const float *p, uint64_t i, float) { return p[i]; }
    static __device__ __forceinline__ void st(float *p, uint64_t i, float v, float)
    {
        __builtin_nontemporal_store(v, p + i);
    }
};
template <>
struct St<double> {
    using R = double;
    static __device__ __forceinline__ double ld(const double *p, uint64_t i, double) { return p[i]; }
    static __device__ __forceinline__ void st(double *p, uint64_t i, double v, double)
    {
        __builtin_nontemporal_store(v, p + i);
    }
};
template <>
struct St<_Float16> {
    using R = float;
    static __device__ __forceinline__ float ld(const _Float16 *p, uint64_t i, float inv)
    {
        return float(p[i]) * inv;
    }
    static __device__ __forceinline__ void st(_Float16 *p, uint64_t i, float v, float scale)
    {
        __builtin_nontemporal_store(_Float16(v * scale), p + i);   // v_cvt_f16_f32: RNE
    }
};
struct bf16s {
    uint16_t b;
};
template <>
struct St<bf16s> {
    using R = float;
    static __device__ __forceinline__ float ld(const bf16s *p, uint64_t i, float)
    {
        const uint16_t *u = reinterpret_cast<const uint16_t *>(p);
        return __uint_as_float(uint32_t(u[i]) << 16);
    }
    static __device__ __forceinline__ void st(bf16s *p, uint64_t i, float v, float)
    {
        uint32_t u = __float_as_uint(v);
        u += 0x7FFFu + ((u >> 16) & 1u);   // round to nearest even
        __builtin_nontemporal_store(uint16_t(u >> 16), reinterpret_cast<uint16_t *>(p) + i);
    }
};

// A value that every lane loads from the same address: keep it in scalar
// registers (the compiler cannot prove that memory written by the kernel is
// uniform when read back).
template <typename T>
__device__ __forceinline__ T uniform(const T &v)
{
    static_assert(sizeof(T) % 4 == 0, "32-bit words");
    T r;
    const int *s = reinterpret_cast<const int *>(&v);
    int *d = reinterpret_cast<int *>(&r);
#pragma unroll
    for (int k = 0; k < int(sizeof(T) / 4); ++k) d[k] = __builtin_amdgcn_readfirstlane(s[k]);
    return r;
}

// Each XCD receives every 8th block; renumber so that each XCD works on a
// contiguous range of cells (neighbouring blocks share partial cache lines).
__device__ __forceinline__ uint32_t xcd_block(uint32_t b, uint32_t nb)
{
    const uint32_t per = nb >> 3, rem = nb & 7u;
    const uint32_t xcd = b & 7u, k = b >> 3;
    return xcd * per + (xcd < rem ? xcd : rem) + k;
}

// the physical parameters in the collision type R (host side, for launches)
template <typename R>
inline Phys<R> cast_phys(const Phys<double> &p)
{
    Phys<R> o;
    o.rho0 = R(p.rho0);
    o.omega_e = R(p.omega_e);
    o.omega_o = R(p.omega_o);
    o.wall_u = R(p.wall_u);
    for (int k = 0; k < 3; ++k) o.g[k] = R(p.g[k]);
    o.has_g = p.has_g;
    o.scale = R(p.scale);
    o.inv_scale = R(p.inv_scale);
    return o;
}

// Where population q of cell (x, y, z) sits in the swapped layout (between
// the even and the odd sweep of a pair), i.e. where the odd sweep gathers
// it: slot opp(q) of x - c_q; through a no-slip x or y wall (and not a
// no-slip z wall), the cell's own slot q; through free-slip walls only,
// slot opp(refl(q)) of x - t, refl(q) the direction it had before the
// reflection and t the components of c_q along the walls it did not cross.
// Returns the plane-shifted cell index, the slot's direction in qq.
__device__ __forceinline__ uint32_t swapped_src(const Geo &g, uint32_t x, uint32_t y, uint32_t z, int q, int &qq)
{
    bool ix = g.xw && ((CX[q] > 0 && x == 0) || (CX[q] < 0 && x + 1 == g.nx));
    bool iy = g.yw && ((CY[q] > 0 && y == 0) || (CY[q] < 0 && y + 1 == g.ny));
    bool iz = !g.zper && ((CZ[q] > 0 && z == 0) || (CZ[q] < 0 && z + 1 == g.nz));
    if (iz && !g.zs) {
        ix = iy = iz = false;      // the z wall's ghost-plane mailbox
    } else if ((ix && g.xw == 1) || (iy && g.yw == 1)) {
        qq = q;
        return (z + 1) * g.nxy + y * g.nx + x;
    }
    const int m = (ix ? 1 : 0) | (iy ? 2 : 0) | (iz ? 4 : 0);
    qq = opp(refl_sel(q, m));
    const int tx = ix ? 0 : CX[q], ty = iy ? 0 : CY[q], tz = iz ? 0 : CZ[q];
    const uint32_t sx = (x + g.nx - tx) % g.nx, sy = (y + g.ny - ty) % g.ny;
    const int32_t szi = int32_t(z) - tz;
    const uint32_t szs = g.zper ? uint32_t((szi + int32_t(g.nz)) % int32_t(g.nz)) + 1 : uint32_t(szi + 1);
    return szs * g.nxy + sy * g.nx + sx;
}

// ------------------------------------------------------------------ stabilization
// Momentum stabilization (Sec. 4.1): the collisions of a step take their
// equilibrium at u - ub, ub the mean fluid velocity of the state they read.
// Each thread also sums, over the cells it updates, the momentum j before
// collision, the momentum change of its bounce-back links and the cell count;
// the per-workgroup totals give the next step's mean without a further pass
// over the lattice (the collision changes each cell's momentum by the uniform
// rho0 (g - omega_o ub), streaming in the interior conserves it).
template <typename R>
struct StabAcc {
    R ub[3];
    R j[3];
    R n;
};

template <typename R>
__device__ __forceinline__ void stab_begin(StabAcc<R> &sa, const double *stab)
{
#pragma unroll
    for (int k = 0; k < 3; ++k) {
        sa.ub[k] = R(stab[k]);
        sa.j[k] = R(0);
    }
    sa.n = R(0);
}

// Workgroup total (256 threads, every thread calls) of 4 doubles, written to
// out by thread 0..3: wave sums by shuffles, then the 4 waves in order.
__device__ __forceinline__ void block_sum4(const double (&v)[4], double *out)
{
    __shared__ double red[4][4];
    const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        double x = v[k];
        for (int o = 32; o > 0; o >>= 1) x += __shfl_xor(x, o, 64);
        if (lane == 0) red[wid][k] = x;
    }
    __syncthreads();
    if (threadIdx.x < 4) {
        const int k = threadIdx.x;
        out[k] = ((red[0][k] + red[1][k]) + red[2][k]) + red[3][k];
    }
}

// j and n of a thread's cells into the workgroup's slot
template <typename R>
__device__ __forceinline__ void stab_flush(const StabAcc<R> &sa, double *out)
{
    const double v[4] = {double(sa.j[0]), double(sa.j[1]), double(sa.j[2]), double(sa.n)};
    block_sum4(v, out);
}

// ------------------------------------------------------------------ collision
// TRT in deviation form: f' = f - w rho0, drho = sum f', j = sum c f'.
// Even/odd equilibrium parts of Eq. EqPDF_TRT minus w rho0:
//   feq_e' = w (drho - 3/2 rho0 u.u + 9/2 rho0 (c.u)^2),  feq_o = 3 w rho0 c.u
// lambda_e = -omega_e, lambda_o = -omega_o (Eq. LBMCollide).  With a body
// force the velocity carries +g/2 and the odd part gains (1 - omega_o/2) 3 w rho0 c.g.
// STAB: the equilibrium velocity is u - sa.ub, and j and the cell are counted.
// The fused multiply-adds are written out, so that an instance of the update has
// the same bits in every kernel that it is compiled into.  SPLIT rounds omega_e
// e of the second value of a pair by itself; nothing in the method asks for
// it: the instances that take it (update_cell) were once compiled so, and keep
// their bits, so that a run goes on from an older checkpoint as it would have.
template <typename R, bool SPLIT, bool STAB>
__device__ __forceinline__ void collide(R (&f)[Q], const Phys<R> &ph, R inv_rho0, StabAcc<R> *sa = nullptr)
{
#pragma clang fp contract(off)
    R drho = R(0), jx = R(0), jy = R(0), jz = R(0);
#pragma unroll
    for (int q = 0; q < Q; ++q) {
        drho += f[q];
        if (CX[q]) jx += CX[q] > 0 ? f[q] : -f[q];
        if (CY[q]) jy += CY[q] > 0 ? f[q] : -f[q];
        if (CZ[q]) jz += CZ[q] > 0 ? f[q] : -f[q];
    }
    const R half = R(0.5), r0 = ph.rho0, we = ph.omega_e, wo = ph.omega_o;
    const bool hg = ph.has_g != 0;
    R ux = hg ? fma(jx, inv_rho0, half * ph.g[0]) : jx * inv_rho0;
    R uy = hg ? fma(jy, inv_rho0, half * ph.g[1]) : jy * inv_rho0;
    R uz = hg ? fma(jz, inv_rho0, half * ph.g[2]) : jz * inv_rho0;
    if constexpr (STAB) {
        sa->j[0] += jx;
        sa->j[1] += jy;
        sa->j[2] += jz;
        sa->n += R(1);
        ux -= sa->ub[0];
        uy -= sa->ub[1];
        uz -= sa->ub[2];
    }
    const R uu = fma(uz, uz, fma(ux, ux, uy * uy));
    const R base = fma(-(R(1.5) * r0), uu, drho);
    f[0] = fma(-we, fma(-R(wq(0)), base, f[0]), f[0]);
#pragma unroll
    for (int q = 1; q <= 9; ++q) {
        const R w = R(wq(q));
        const R cu = R(CX[q]) * ux + R(CY[q]) * uy + R(CZ[q]) * uz;
        const R eeq = w * fma(R(4.5) * r0 * cu, cu, base);
        const R oeq = R(3) * w * r0 * cu;
        const R e = fma(half, f[q] + f[q + 9], -eeq);
        const R o = fma(half, f[q] - f[q + 9], -oeq);
        const R T = (R(1) - half * wo) * R(3) * w * r0 *
                    (R(CX[q]) * ph.g[0] + R(CY[q]) * ph.g[1] + R(CZ[q]) * ph.g[2]);
        const R dd = hg ? fma(wo, o, -T) : wo * o;
        f[q] = fma(-we, e, f[q]) - dd;
        f[q + 9] = (SPLIT ? f[q + 9] - we * e : fma(-we, e, f[q + 9])) + dd;
    }
}

// rigid-body velocity of fiber p at the centre of cell (cx, cy, cz):
// u_s = V + W x d with d the minimum-image vector from the centre of mass.
__device__ __forceinline__ double mi(double d, uint32_t n, bool per)
{
    if (!per) return d;
    const double h = 0.5 * double(n);
    return d > h ? d - double(n) : (d < -h ? d + double(n) : d);
}
__device__ __forceinline__ void surf_vel(const PState &s, double cx, double cy, double cz,
                                         const Geo &g, double us[3])
{
    const double dx = mi(cx - s.X[0], g.nx, true), dy = mi(cy - s.X[1], g.ny, true),
                 dz = mi(cz - s.X[2], g.nz, g.zper != 0);
    us[0] = s.V[0] + (s.W[1] * dz - s.W[2] * dy);
    us[1] = s.V[1] + (s.W[2] * dx - s.W[0] * dz);
    us[2] = s.V[2] + (s.W[0] * dy - s.W[1] * dx);
}

// ------------------------------------------------------------------ one cell
// compile-time loop: f(std::integral_constant<int, I>) for I in [B, E)
template <int I>
struct IntC {
    static constexpr int value = I;
};
template <int B, int E, typename F>
__device__ __forceinline__ void static_for(F &&fn)
{
    if constexpr (B < E) {
        fn(IntC<B>{});
        static_for<B + 1, E>(fn);
    }
}

// fixed-point term of the momentum-exchange sums (see fx_shift)
__device__ __forceinline__ long long fx(double v, int k) { return __double2ll_rn(ldexp(v, fx_shift(k))); }

// Momentum exchange of one link x -> y = x + c_q into fiber-local sums
// (Eq. LBMhydrodynForce and the torque after it): with r = y - X,
//   dF = 2 (f~_q + w_q rho0) c_q - 6 w_q rho0 (c_q.u_s) c_q,  dM = r x dF,
// split into the velocity-free part F0, M0 and the matrices of the part
// linear in u_s = V + W x r: A = k c c^T, B = k c (r x c)^T, C = k (r x c)(r x c)^T,
// k = 6 w_q rho0, so that F = F0 - A V - B W and M = M0 - B^T V - C W.
// This adds the link's F0, M0 terms to acc[0 .. 5]; A, B, C do not depend
// on the populations and are summed as integers, with the links of a step
// (link_sums in boundary.hip) or, in the batched form, when the list is built
// (link_int_terms).
__device__ __forceinline__ void link_terms(long long *acc, double ft, double w, const double c[3],
                                           const double r[3], double r0)
{
    const double m2 = 2.0 * (ft + w * r0);
    const double rc0 = r[1] * c[2] - r[2] * c[1], rc1 = r[2] * c[0] - r[0] * c[2], rc2 = r[0] * c[1] - r[1] * c[0];
    const double t[6] = {m2 * c[0], m2 * c[1], m2 * c[2], m2 * rc0, m2 * rc1, m2 * rc2};
#pragma unroll
    for (int k = 0; k < 6; ++k) acc[k] += fx(t[k], k);
}

// First element of a wall cell's slot: gathering (IN), slot q where the
// population returns from a no-slip wall, else opp(refl(q, m)), m the
// free-slip walls crossed; scattering, slot opp(q) where it bounces, else
// refl(q, m).  m has only bits of nonzero components of c_q.
template <int q, bool IN>
__device__ __forceinline__ uint64_t slot_sel(int m, bool back, uint64_t qs)
{
    constexpr int M = (CX[q] ? 1 : 0) | (CY[q] ? 2 : 0) | (CZ[q] ? 4 : 0);
    uint64_t s = uint64_t(IN ? opp(q) : q) * qs;
    static_for<1, 8>([&](auto mc) {
        constexpr int k = decltype(mc)::value;
        if constexpr ((k & ~M) == 0) s = m == k ? uint64_t(IN ? opp(refl(q, k)) : refl(q, k)) * qs : s;
    });
    return back ? uint64_t(IN ? q : opp(q)) * qs : s;
}

// sink of the cells without fiber links
struct NoLinks {
    template <int q, typename R>
    __device__ __forceinline__ void link(bool, R, uint32_t, uint32_t, uint32_t, uint32_t, uint32_t)
    {
    }
};

// BND: a boundary cell of the list; each of its fiber links (bits of mask) is
// handed to sink.link<q>(is_link, post-collision value, ...), called by every
// lane for every q, which does the bounce-back store and the momentum
// exchange.
// STAB: momentum stabilization with the accumulator sa (see StabAcc).
// XYW: walls on the x and/or y faces (g.xw, g.yw) or free-slip z walls
// (g.zs).  A link leaving the lattice through a resting no-slip x or y wall
// bounces back (Eq. BBBC) into the cell's own slot opp(q) in both sweeps
// (the image cell across the periodic seam is live, so its slots cannot
// serve as a mailbox), and the odd sweep reads a population that arrives
// through such a wall from the cell's own slot; a link crossing a no-slip z
// wall as well keeps the z wall's ghost-plane mailbox.  A link that crosses
// free-slip walls only is reflected (Eq. FreeSlipBC): the components normal
// to the crossed walls reverse and the population lands on the neighbour
// along the other components, x + t.  The even sweep stores it in its own
// slot opp(q) like a streaming population; the odd sweep gathers it there
// from x + t and scatters its own reflected populations into the slot
// refl(q) of x + t, which no other cell touches in that sweep (the slot it
// gathered from for the reverse link), so both sweeps stay in place.  A
// link that crosses walls of both kinds bounces back.
struct CellPos {
    uint32_t x, y, z;
    uint32_t xo[3], yo[3], zo[3];   // offsets of the neighbours' coordinates (wrapped; planes shifted by one)
    uint32_t own;
};
__device__ __forceinline__ CellPos cell_pos(const Geo &g, uint32_t cell)
{
    CellPos c;
    c.z = fdiv(cell, g.dnxy);
    const uint32_t rr = cell - c.z * g.nxy;
    c.y = fdiv(rr, g.dnx);
    c.x = rr - c.y * g.nx;
    c.xo[0] = c.x == 0 ? g.nx - 1 : c.x - 1;
    c.xo[1] = c.x;
    c.xo[2] = c.x + 1 == g.nx ? 0 : c.x + 1;
    c.yo[0] = (c.y == 0 ? g.ny - 1 : c.y - 1) * g.nx;
    c.yo[1] = c.y * g.nx;
    c.yo[2] = (c.y + 1 == g.ny ? 0 : c.y + 1) * g.nx;
    c.zo[0] = (g.zper && c.z == 0 ? g.nz : c.z) * g.nxy;
    c.zo[1] = (c.z + 1) * g.nxy;
    c.zo[2] = (g.zper && c.z + 1 == g.nz ? 1 : c.z + 2) * g.nxy;
    c.own = c.zo[1] + c.yo[1] + c.xo[1];
    return c;
}

// the walls a cell lies at (x and y only with XYW)
struct CellWalls {
    bool lo, hi, x0, x1, y0, y1, zs;
    bool any;   // a cell of the wave lies at a wall that changes slots
};
template <bool XYW>
__device__ __forceinline__ CellWalls cell_walls(const Geo &g, const CellPos &c)
{
    CellWalls w{!g.zper && c.z == 0, !g.zper && c.z + 1 == g.nz, false, false, false, false, false, false};
    if constexpr (XYW) {
        w.x0 = g.xw && c.x == 0;
        w.x1 = g.xw && c.x + 1 == g.nx;
        w.y0 = g.yw && c.y == 0;
        w.y1 = g.yw && c.y + 1 == g.ny;
        w.zs = g.zs != 0;
        // (of the z walls only free-slip ones change the slots)
        w.any = __any(w.x0 || w.x1 || w.y0 || w.y1 || (w.zs && (w.lo || w.hi)));
    }
    return w;
}

// Odd sweeps with walls: selecting every slot costs a wave some 200 more
// instructions, so a wave with no cell at a wall (of the z walls only
// free-slip ones change the slots) takes the update without them.  Odd sweep
// against even, FP32, 768 workgroups, when each population tests for itself
// whether the wave lies at a wall, and as here (x, y free-slip, z free-slip): 160 x
// 160 x 1200 1.12, 1.05; 320^3 1.07, 1.03.  The second copy takes registers (FP32 95
// to 107, FP64 141 to 163): in FP64, with stabilization and for the boundary
// cells they are what a CU needs to hold the two kernels side by side (160 x 160
// x 1200 FP64 with fibers 1960 us a step without the copy, 2197 with), so there
// each population tests for itself.
template <typename S, bool ODD, bool BND, bool STAB, bool XYW>
constexpr bool WALL_WAVES = ODD && XYW && !BND && !STAB && sizeof(typename St<S>::R) == 4;

// The update of the cell at c.  Without XYW the walls w are those of the z
// axis, no-slip: slots then differ by lane only in the scatter.
template <typename S, bool ODD, bool BND, bool STAB, bool XYW, bool SPLIT, typename Sink>
__device__ __forceinline__ void update_at(S *__restrict__ f, const Geo &g, const Phys<typename St<S>::R> &ph,
                                          const CellPos &c, const CellWalls &w, uint32_t mask, Sink &sink,
                                          StabAcc<typename St<S>::R> *sa)
{
    using R = typename St<S>::R;
    const uint64_t qs = g.qstride;
    const R inv = ph.inv_scale, sc = ph.scale;
    R fv[Q];
    static_for<0, Q>([&](auto qc) {
        constexpr int q = decltype(qc)::value;
        if (!ODD) {
            fv[q] = St<S>::ld(f, uint64_t(q) * qs + c.own, inv);
        } else {
            if constexpr (XYW) {
                if (WALL_WAVES<S, ODD, BND, STAB, XYW> || w.any) {
                    // walls crossed on the way in (a no-slip z wall: its
                    // mailbox, a normal read); the source is selected, not
                    // branched to, so that all loads are in flight together
                    bool ix = (CX[q] > 0 && w.x0) || (CX[q] < 0 && w.x1);
                    bool iy = (CY[q] > 0 && w.y0) || (CY[q] < 0 && w.y1);
                    const bool oz = (CZ[q] > 0 && w.lo) || (CZ[q] < 0 && w.hi), iz = w.zs && oz;
                    if (oz && !w.zs) ix = iy = false;
                    const bool side_in = (ix && g.xw == 1) || (iy && g.yw == 1);
                    const int m = (ix ? 1 : 0) | (iy ? 2 : 0) | (iz ? 4 : 0);
                    uint32_t src = (iz ? c.zo[1] : c.zo[1 - CZ[q]]) + (iy ? c.yo[1] : c.yo[1 - CY[q]]) +
                                   (ix ? c.xo[1] : c.xo[1 - CX[q]]);
                    src = side_in ? c.own : src;
                    fv[q] = St<S>::ld(f, slot_sel<q, true>(m, side_in, qs) + src, inv);
                    return;
                }
            }
            const uint32_t src = c.zo[1 - CZ[q]] + c.yo[1 - CY[q]] + c.xo[1 - CX[q]];
            fv[q] = St<S>::ld(f, uint64_t(opp(q)) * qs + src, inv);
        }
    });
    collide<R, SPLIT, STAB>(fv, ph, R(1) / ph.rho0, sa);
    const R six_r0 = R(6) * ph.rho0;
    static_for<0, Q>([&](auto qc) {
        constexpr int q = decltype(qc)::value;
        const uint32_t nb = c.zo[1 + CZ[q]] + c.yo[1 + CY[q]] + c.xo[1 + CX[q]];
        const bool oz = (CZ[q] < 0 && w.lo) || (CZ[q] > 0 && w.hi);
        const bool to_wall = oz && !w.zs;
        bool to_side = false, to_slip = false;
        int slip_m = 0;
        if constexpr (XYW) {
            const bool ox = (CX[q] < 0 && w.x0) || (CX[q] > 0 && w.x1);
            const bool oy = (CY[q] < 0 && w.y0) || (CY[q] > 0 && w.y1);
            to_side = !to_wall && ((ox && g.xw == 1) || (oy && g.yw == 1));
            to_slip = !to_wall && !to_side && (ox || oy || oz);
            slip_m = (ox ? 1 : 0) | (oy ? 2 : 0) | (oz ? 4 : 0);
        }
        if constexpr (BND && q > 0) {
            const bool lk = ((mask >> q) & 1u) && !to_slip && !to_side;
            sink.template link<q>(lk, fv[q], c.own, nb, c.x, c.y, c.z);
            if (lk) return;
        }
        R out = fv[q];
        if (CX[q] != 0 && to_wall) {
#pragma clang fp contract(off)
            const R uw = CZ[q] < 0 ? -ph.wall_u : ph.wall_u;
            out -= six_r0 * R(wq(q)) * R(CX[q]) * uw;
        }
        const bool bounce = to_wall || to_side;
        if constexpr (STAB) {
            // a bounced link returns out in direction -c_q instead of
            // streaming fv[q] along c_q; a reflected one reverses the
            // components normal to the crossed walls
            if (bounce) {
                const R m = fv[q] + out;
                if (CX[q]) sa->j[0] -= CX[q] > 0 ? m : -m;
                if (CY[q]) sa->j[1] -= CY[q] > 0 ? m : -m;
                if (CZ[q]) sa->j[2] -= CZ[q] > 0 ? m : -m;
            } else if (to_slip) {
                const R m = fv[q] + fv[q];
                if (slip_m & 1) sa->j[0] -= CX[q] > 0 ? m : -m;
                if (slip_m & 2) sa->j[1] -= CY[q] > 0 ? m : -m;
                if (slip_m & 4) sa->j[2] -= CZ[q] > 0 ? m : -m;
            }
        }
        if (!ODD) {
            // mailbox for z walls; normal streaming, side walls and
            // reflections: own slot
            if (to_wall) St<S>::st(f, uint64_t(q) * qs + nb, out, sc);
            else St<S>::st(f, uint64_t(opp(q)) * qs + c.own, out, sc);
        } else {
            if constexpr (XYW) {
                if (WALL_WAVES<S, ODD, BND, STAB, XYW> || w.any) {
                    uint32_t dst = ((slip_m & 4) ? c.zo[1] : c.zo[1 + CZ[q]]) + ((slip_m & 2) ? c.yo[1] : c.yo[1 + CY[q]]) +
                                   ((slip_m & 1) ? c.xo[1] : c.xo[1 + CX[q]]);
                    dst = bounce ? c.own : dst;
                    St<S>::st(f, slot_sel<q, false>(slip_m, bounce, qs) + dst, out, sc);
                    return;
                }
            }
            if (bounce) St<S>::st(f, uint64_t(opp(q)) * qs + c.own, out, sc);
            else St<S>::st(f, uint64_t(q) * qs + nb, out, sc);
        }
    });
    (void)six_r0;
    (void)sink;
}

template <typename S, bool ODD, bool BND, bool STAB, bool XYW, typename Sink>
__device__ __forceinline__ void update_cell(S *__restrict__ f, const Geo &g, const Phys<typename St<S>::R> &ph,
                                            uint32_t cell, uint32_t mask, Sink &sink,
                                            StabAcc<typename St<S>::R> *sa = nullptr)
{
    // the forms that round a pair's second value in two steps (collide)
    constexpr bool split = BND || STAB || (ODD && (XYW || std::is_same_v<S, bf16s>));
    const CellPos c = cell_pos(g, cell);
    const CellWalls w = cell_walls<XYW>(g, c);
    if constexpr (WALL_WAVES<S, ODD, BND, STAB, XYW>) {
        if (!w.any) {
            update_at<S, ODD, BND, STAB, false, split>(f, g, ph, c, w, mask, sink, sa);
            return;
        }
    }
    update_at<S, ODD, BND, STAB, XYW, split>(f, g, ph, c, w, mask, sink, sa);
}

// The moving-obstacle bounce-back (Eq. LBMMovWall) of one fiber link from
// cell (x, y, z) in direction c to the solid cell y = x + c of the fiber in
// state X, V, W: the returned value of the post-collision value v; the lever
// arm y - X in r.
template <typename R>
__device__ __forceinline__ R link_bounce(R v, double w6r0, const double c[3], const uint32_t yc[3], const double *X,
                                         const double *V, const double *W, const Geo &g, double r[3])
{
    r[0] = mi(double(yc[0]) - X[0], g.nx, true);
    r[1] = mi(double(yc[1]) - X[1], g.ny, true);
    r[2] = mi(double(yc[2]) - X[2], g.nz, g.zper != 0);
    const double us0 = V[0] + (W[1] * r[2] - W[2] * r[1]);
    const double us1 = V[1] + (W[2] * r[0] - W[0] * r[2]);
    const double us2 = V[2] + (W[0] * r[1] - W[1] * r[0]);
    const double cu = c[0] * us0 + c[1] * us1 + c[2] * us2;
    return v - R(w6r0 * cu);
}

}  // namespace lbm

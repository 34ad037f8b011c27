// boundary.hip -- the boundary-list work of one time step, in one launch: the
// update of the cells next to fibers (the fused stream-collide of the bulk
// sweep), the moving-obstacle bounce-back of their fiber links (Eq.
// LBMMovWall), and the links' momentum exchange (Eq. LBMhydrodynForce and
// the torque after it): the velocity-free sums F0, M0 and the integer sums
// of the part linear in the surface velocity (A, B, C; see abc_restore).
//
// One wave per workgroup takes 64 entries of a fiber's list segment, in two
// halves.  First each lane updates its cell; the post-collision values of
// fiber links go to a queue in LDS.  Then the lanes share the queue, one
// link per lane: a boundary cell has about five fiber links among its 18
// directions, so a wave works through 5-6 full rounds of links instead of 18
// rounds in which a third of the lanes take part, and each round's code
// exists once.  The kernel is bound by the latency of this FP64 and 64-bit
// integer chain, not by memory (57,000 cells move 9 MB).  A list entry whose
// fiber cells all belong to the segment's own fiber (LIST_HOME, set where the
// list is built; all entries unless two fibers are within a cell of each
// other) takes that fiber's state from scalar registers and needs no
// owner look-ups.
#include "lbm_sweep_dev.h"

namespace lbm {

// links of one wave's 64 cells: capacity for every direction of every cell
constexpr uint32_t QCAP = 64u * (Q - 1);

template <typename R>
struct LinkQueue {
    uint32_t *code;   // bits 0-5 the cell's lane, 6-10 q, 11-16 c + 1 (2 bits a component), 17 tag
    R *val;           // post-collision value
    uint32_t n;       // wave-uniform among the lanes that take part
    uint32_t tag;     // the lane, bit 17: owners to be looked up
    template <int q>
    __device__ __forceinline__ void link(bool lk, R v, uint32_t, uint32_t, uint32_t, uint32_t, uint32_t)
    {
        const unsigned long long m = __ballot(lk);
        if (lk) {
            const uint32_t at = n + __builtin_amdgcn_mbcnt_hi(uint32_t(m >> 32), __builtin_amdgcn_mbcnt_lo(uint32_t(m), 0u));
            code[at] = tag | uint32_t(q << 6 | (CX[q] + 1) << 11 | (CY[q] + 1) << 13 | (CZ[q] + 1) << 15);
            val[at] = v;
        }
        n += uint32_t(__popcll(m));
    }
};

}  // namespace lbm

// integer index arithmetic of the particle side (shared with the list rebuild)
#include "lbm_particle_dev.h"

namespace lbm {

// The product of s with c = -1, 0 or 1.
__device__ __forceinline__ int32_t times_c(int32_t s, int32_t c) { return c == 0 ? 0 : (c < 0 ? -s : s); }

// integer terms of a link in direction c to the solid cell at offset s from
// its fiber's reference point (see abc_restore): a[0..5] = SA, then SB, SC
__device__ __forceinline__ void link_sums(const int32_t c[3], const int32_t s[3], int32_t kap, int32_t (&sa)[6],
                                          long long (&sb)[9], long long (&sc)[6])
{
    const int32_t r[3] = {times_c(s[1], c[2]) - times_c(s[2], c[1]), times_c(s[2], c[0]) - times_c(s[0], c[2]),
                          times_c(s[0], c[1]) - times_c(s[1], c[0])};
    const int32_t kr[3] = {kap * r[0], kap * r[1], kap * r[2]};
    const int32_t kc[3] = {kap * c[0], kap * c[1], kap * c[2]};
    int k = 0, k2 = 0;
#pragma unroll
    for (int i = 0; i < 3; ++i)
#pragma unroll
        for (int j = i; j < 3; ++j) sa[k++] += times_c(kc[i], c[j]);
    k = 0;
#pragma unroll
    for (int i = 0; i < 3; ++i)
#pragma unroll
        for (int j = 0; j < 3; ++j) {
            sb[k++] += times_c(kr[j], c[i]);
            if (j >= i) sc[k2++] += (long long)(kr[i]) * r[j];
        }
}

// Sum over the wave of 32 values per lane: each step halves the values held
// and pairs lanes 32, 16, 8, 4, 2 apart, the last adds the remaining pairs;
// lane l ends with the total of value l >> 1.
template <int H>
__device__ __forceinline__ void halve(long long (&v)[32])
{
    const bool up = (threadIdx.x & (2 * H)) != 0;
#pragma unroll
    for (int k = 0; k < H; ++k) {
        const long long send = up ? v[k] : v[k + H], keep = up ? v[k + H] : v[k];
        v[k] = keep + __shfl_xor(send, 2 * H, 64);
    }
}
__device__ __forceinline__ long long wave_totals(long long (&v)[32])
{
    halve<16>(v);
    halve<8>(v);
    halve<4>(v);
    halve<2>(v);
    halve<1>(v);
    return v[0] + __shfl_xor(v[0], 1, 64);
}

// 4 sums over the wave to out
__device__ __forceinline__ void wave_sum4(const double (&v)[4], double *out)
{
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        double x = v[k];
        for (int o = 32; o > 0; o >>= 1) x += __shfl_xor(x, o, 64);
        if (threadIdx.x == 0) out[k] = x;
    }
}

// Beside the FP32 bulk sweep, whose two waves a SIMD stay resident for its
// whole grid-stride run, this kernel must leave them room: of its own waves
// (158 to 186 VGPRs) three fill a SIMD, and bulk workgroups that come after them
// then sit unevenly on the card and the sweep stretches by half.  The launch
// reserves LDS (BND_LDS) so that a CU holds four.
// Grid: np * bpf waves; wave (fiber p, part j) takes entries 64 j, 64 (j +
// bpf), ... of the fiber's list segment.
// nbulk further waves take the cells of the bulk sweep, 64 each (STAB: 64 at a
// time, strided).  STAB: momentum stabilization (mean velocity stab[0..2]; every
// wave writes its sums to a slot of part, the bulk waves first).  XYW: walls on
// the x and/or y faces.
// LEAN (FP64): 168 VGPRs, for 140 to 196 bytes of spills.  At its own 217 and 208
// no wave fits beside the two of the FP64 sweep (148 and 164 of 512 each), and
// behind a sweep that starts first the whole launch waits for its end (256^3 with
// 16 fibers 1201 us a step, 1118 so).
template <typename S, bool ODD, bool STAB, bool XYW, bool LEAN = false>
__global__ __launch_bounds__(64, LEAN ? 3 : 2) void k_boundary(S *__restrict__ f, Geo g, Phys<typename St<S>::R> ph, BndData b,
                                                    const double *stab, double *part,
                                                    const uint8_t *__restrict__ flags, uint32_t nbulk)
{
    using R = typename St<S>::R;
    __shared__ uint32_t s_code[QCAP];
    __shared__ R s_val[QCAP];
    __shared__ uint32_t s_cell[64];
    const uint32_t lane = threadIdx.x, nb = uint32_t(b.np * b.bpf);
    StabAcc<R> st;
    if constexpr (STAB) stab_begin(st, stab);
    if (blockIdx.x >= nb) {   // wave-uniform
        const uint32_t k = xcd_block(blockIdx.x - nb, nbulk);
        NoLinks none;
        if constexpr (STAB) {
            // strided: every wave leaves a slot that one workgroup adds up at
            // the end of the step, so there are few of them (STAB_WAVES)
            double t[4] = {0.0, 0.0, 0.0, 0.0};
            for (uint32_t cell = k * 64u + lane; cell < g.ncell; cell += nbulk * 64u) {
                if (flags[cell]) continue;
                update_cell<S, ODD, false, STAB, XYW>(f, g, ph, cell, 0u, none, &st);
                for (int e = 0; e < 3; ++e) {
                    t[e] += double(st.j[e]);
                    st.j[e] = R(0);
                }
                t[3] += 1.0;
            }
            wave_sum4(t, part + 4 * size_t(k));
        } else {
            const uint32_t cell = k * 64u + lane;
            if (cell < g.ncell && !flags[cell]) update_cell<S, ODD, false, STAB, XYW>(f, g, ph, cell, 0u, none, &st);
        }
        return;
    }
    const int blk = int(xcd_block(blockIdx.x, nb));   // a fiber's waves share one XCD's L2
    const int p = blk / b.bpf, j = blk % b.bpf;       // wave-uniform
    const uint32_t cap = b.seg_cap[p], off = b.seg_off[p];
    // the fiber's state (home links) and the reference point of its sums
    double X[3], V[3], W[3];
    for (int k = 0; k < 3; ++k) {
        X[k] = uniform(b.ps[p].X[k]);
        V[k] = uniform(b.ps[p].V[k]);
        W[k] = uniform(b.ps[p].W[k]);
    }
    int32_t hr[3];
    fiber_ref(X, hr);
    const uint32_t n = min(b.seg_cnt[p], cap);
    const double r0 = double(ph.rho0);
    long long fm[6] = {0, 0, 0, 0, 0, 0}, sb[9] = {0, 0, 0, 0, 0, 0, 0, 0, 0}, sc[6] = {0, 0, 0, 0, 0, 0};
    int32_t sa[6] = {0, 0, 0, 0, 0, 0};
    double lj[3] = {0.0, 0.0, 0.0};   // momentum change of the links (stabilization)
    for (uint32_t e0 = uint32_t(j) * 64u; e0 < n; e0 += uint32_t(b.bpf) * 64u) {
        LinkQueue<R> queue{s_code, s_val, 0u, lane};
        if (e0 + lane < n) {
            const uint32_t cell = b.cell[off + e0 + lane], mask = b.mask[off + e0 + lane];
            s_cell[lane] = cell;
            if (!(mask & LIST_HOME)) queue.tag |= 1u << 17;
            update_cell<S, ODD, true, STAB, XYW>(f, g, ph, cell, mask, queue, &st);
        }
        const uint32_t nl = __builtin_amdgcn_readfirstlane(queue.n);   // lane 0 has an entry
        __syncthreads();
        for (uint32_t l = lane; l < nl; l += 64u) {
            const uint32_t code = s_code[l], q = (code >> 6) & 31u;
            const R v = s_val[l];
            const int32_t c[3] = {int32_t((code >> 11) & 3u) - 1, int32_t((code >> 13) & 3u) - 1,
                                  int32_t((code >> 15) & 3u) - 1};
            const double cd[3] = {double(c[0]), double(c[1]), double(c[2])};
            const bool axis = (c[0] != 0) + (c[1] != 0) + (c[2] != 0) == 1;
            const uint32_t cell = s_cell[code & 63u];
            const uint32_t z = fdiv(cell, g.dnxy), rem = cell - z * g.nxy;
            const uint32_t y = fdiv(rem, g.dnx), x = rem - y * g.nx;
            const int32_t nx = int32_t(g.nx), ny = int32_t(g.ny), nz = int32_t(g.nz);
            const int32_t yx = wrapc(int32_t(x) + c[0], nx), yy = wrapc(int32_t(y) + c[1], ny);
            const int32_t yz = g.zper ? wrapc(int32_t(z) + c[2], nz) : int32_t(z) + c[2];
            const uint32_t yc[3] = {uint32_t(yx), uint32_t(yy), uint32_t(yz)};
            const uint32_t ycell = (yc[2] * g.ny + yc[1]) * g.nx + yc[0];
            const int o = (code >> 17) & 1u ? b.pid[ycell] : p;
            const double w = axis ? wq(1) : wq(4), w6r0 = (axis ? 6.0 * wq(1) : 6.0 * wq(4)) * r0;
            const int32_t kap = axis ? 2 : 1;
            double r[3];
            R out;
            if (!isfinite(double(v))) atomicOr(&b.ctr->err_unstable, 1u);
            if (o == p) {
                out = link_bounce<R>(v, w6r0, cd, yc, X, V, W, g, r);
                link_terms(fm, double(v), w, cd, r, r0);
                const int32_t s[3] = {mi_i(yx - hr[0], nx, true), mi_i(yy - hr[1], ny, true),
                                      mi_i(yz - hr[2], nz, g.zper != 0)};
                link_sums(c, s, kap, sa, sb, sc);
            } else {
                // link to another fiber (fibers closer than the region margin)
                const PState &so = b.ps[o];
                out = link_bounce<R>(v, w6r0, cd, yc, so.X, so.V, so.W, g, r);
                long long tf[6] = {0, 0, 0, 0, 0, 0}, tb[9] = {0, 0, 0, 0, 0, 0, 0, 0, 0}, tc[6] = {0, 0, 0, 0, 0, 0};
                int32_t ta[6] = {0, 0, 0, 0, 0, 0}, rf[3];
                link_terms(tf, double(v), w, cd, r, r0);
                fiber_ref(so.X, rf);
                const int32_t s[3] = {mi_i(yx - rf[0], nx, true), mi_i(yy - rf[1], ny, true),
                                      mi_i(yz - rf[2], nz, g.zper != 0)};
                link_sums(c, s, kap, ta, tb, tc);
                unsigned long long *m = reinterpret_cast<unsigned long long *>(b.mea + size_t(o) * NACC);
#pragma unroll
                for (int k = 0; k < 9; ++k) {
                    if (k < 6) {
                        atomicAdd(m + k, (unsigned long long)tf[k]);
                        if (ta[k]) atomicAdd(m + 6 + k, (unsigned long long)(long long)ta[k]);
                        if (tc[k]) atomicAdd(m + 21 + k, (unsigned long long)tc[k]);
                    }
                    if (tb[k]) atomicAdd(m + 12 + k, (unsigned long long)tb[k]);
                }
            }
            if constexpr (STAB) {
                // the link returns out in direction -c instead of streaming v along c
                const double m = double(v + out);
                for (int k = 0; k < 3; ++k) lj[k] -= cd[k] * m;
            }
            // even sweep: the mailbox, slot q of the solid cell; odd: own slot opp(q)
            const uint64_t slot = ODD ? uint64_t(q <= 9u ? q + 9u : q - 9u) * g.qstride + g.nxy + cell
                                      : uint64_t(q) * g.qstride + g.nxy + ycell;
            St<S>::st(f, slot, out, ph.scale);
        }
        __syncthreads();
    }
    // integer sums: exact, so the reduction order does not matter
    long long v[32] = {fm[0], fm[1], fm[2], fm[3], fm[4], fm[5], sa[0], sa[1], sa[2], sa[3], sa[4], sa[5],
                       sb[0], sb[1], sb[2], sb[3], sb[4], sb[5], sb[6], sb[7], sb[8],
                       sc[0], sc[1], sc[2], sc[3], sc[4], sc[5], 0, 0, 0, 0, 0};
    const long long tot = wave_totals(v);
    if ((lane & 1u) == 0u && lane < 2u * NACC && tot)
        atomicAdd(reinterpret_cast<unsigned long long *>(b.mea + size_t(p) * NACC + (lane >> 1)), (unsigned long long)tot);
    if constexpr (STAB) {
        const double t[4] = {double(st.j[0]) + lj[0], double(st.j[1]) + lj[1], double(st.j[2]) + lj[2], double(st.n)};
        wave_sum4(t, part + 4 * size_t(nbulk + uint32_t(blk)));
    }
}

template <typename S>
static hipError_t boundary_t(bool odd, void *f, const Geo &g, const Phys<double> &ph, const BndData &b,
                             hipStream_t st, const double *stab, double *part, const uint8_t *flags, uint32_t nbulk,
                             uint32_t lds, bool lean)
{
    using R = typename St<S>::R;
    const Phys<R> p = cast_phys<R>(ph);
    const dim3 grid(uint32_t(b.np * b.bpf) + nbulk), bl(64);
    const int mode = (odd ? 1 : 0) | (stab ? 2 : 0) | ((g.xw || g.yw || g.zs) ? 4 : 0);
    if constexpr (std::is_same_v<S, double>) {
        if (lean && !stab) {
            switch (mode) {
            case 0: hipLaunchKernelGGL((k_boundary<S, false, false, false, true>), grid, bl, lds, st, (S *)f, g, p, b, stab, part, flags, nbulk); break;
            case 1: hipLaunchKernelGGL((k_boundary<S, true, false, false, true>), grid, bl, lds, st, (S *)f, g, p, b, stab, part, flags, nbulk); break;
            case 4: hipLaunchKernelGGL((k_boundary<S, false, false, true, true>), grid, bl, lds, st, (S *)f, g, p, b, stab, part, flags, nbulk); break;
            default: hipLaunchKernelGGL((k_boundary<S, true, false, true, true>), grid, bl, lds, st, (S *)f, g, p, b, stab, part, flags, nbulk); break;
            }
            return hipGetLastError();
        }
    }
    switch (mode) {
    case 0: hipLaunchKernelGGL((k_boundary<S, false, false, false>), grid, bl, lds, st, (S *)f, g, p, b, stab, part, flags, nbulk); break;
    case 1: hipLaunchKernelGGL((k_boundary<S, true, false, false>), grid, bl, lds, st, (S *)f, g, p, b, stab, part, flags, nbulk); break;
    case 2: hipLaunchKernelGGL((k_boundary<S, false, true, false>), grid, bl, lds, st, (S *)f, g, p, b, stab, part, flags, nbulk); break;
    case 3: hipLaunchKernelGGL((k_boundary<S, true, true, false>), grid, bl, lds, st, (S *)f, g, p, b, stab, part, flags, nbulk); break;
    case 4: hipLaunchKernelGGL((k_boundary<S, false, false, true>), grid, bl, lds, st, (S *)f, g, p, b, stab, part, flags, nbulk); break;
    case 5: hipLaunchKernelGGL((k_boundary<S, true, false, true>), grid, bl, lds, st, (S *)f, g, p, b, stab, part, flags, nbulk); break;
    case 6: hipLaunchKernelGGL((k_boundary<S, false, true, true>), grid, bl, lds, st, (S *)f, g, p, b, stab, part, flags, nbulk); break;
    default: hipLaunchKernelGGL((k_boundary<S, true, true, true>), grid, bl, lds, st, (S *)f, g, p, b, stab, part, flags, nbulk); break;
    }
    return hipGetLastError();
}

hipError_t launch_boundary(int sk, bool odd, void *f, const Geo &g, const Phys<double> &ph, const BndData &b,
                           hipStream_t st, const double *stab, double *part, const uint8_t *flags, uint32_t nbulk,
                           uint32_t lds, bool lean)
{
    if (b.np <= 0 || b.bpf <= 0) return hipSuccess;
    switch (sk) {
    case S_F32: return boundary_t<float>(odd, f, g, ph, b, st, stab, part, flags, nbulk, lds, lean);
    case S_F16: return boundary_t<_Float16>(odd, f, g, ph, b, st, stab, part, flags, nbulk, lds, lean);
    case S_BF16: return boundary_t<bf16s>(odd, f, g, ph, b, st, stab, part, flags, nbulk, lds, lean);
    default: return boundary_t<double>(odd, f, g, ph, b, st, stab, part, flags, nbulk, lds, lean);
    }
}

}  // namespace lbm

// particles.hip -- per-fiber work of one time step on the device:
//   k_rigid      the momentum-exchange sums of each fiber (Eq.
//                LBMhydrodynForce and the torque after it, Sec. 4.2),
//                accumulated by the boundary sweep, back to FP64; the
//                rigid-body update (Sec. 4.3); the cell boxes of the remap;
//   k_map        cell mapping with the new poses (Sec. 4.2: a cell is an
//                obstacle cell when its centre lies inside a particle),
//                refill of uncovered cells with f_eq(rho0, u_s) of the
//                previous step's motion, flags of fluid cells next to fibers
//                in the flag buffer of the next step, and the boundary-cell
//                list consumed by the next step's boundary launch.
#include "lbm_sweep_dev.h"
#include "lbm_particle_dev.h"

namespace lbm {

#pragma clang fp contract(off)

// Plane rectangle of fiber o's region: the cells it can own or border at the
// new, the current and the previous pose (the flags of the next step are
// written into the buffer that held those of the previous step, so the
// rebuild covers every cell flagged then).
__device__ __forceinline__ Rect remap_rect(const PartData &pd, int o, int32_t z, const Geo &g)
{
    const Box b = pd.box_remap[o];
    const PConst c = pd.pc[o];
    const Rect r = rect_union(plane_rect(pd.ps_cur[o], c, z, b, g, NEAR_MARGIN),
                              plane_rect(pd.ps_next[o], c, z, b, g, NEAR_MARGIN), g);
    return rect_union(r, plane_rect(pd.ps_prev[o], c, z, b, g, NEAR_MARGIN), g);
}

// ------------------------------------------------------------------ boxes of the remap
// Union of the boxes of the previous (box_prev), current (box_cur) and new
// pose s of fiber p, the new box, and the reset of the fiber's boundary-list
// segment.
__device__ __forceinline__ void fiber_remap_boxes(const PartData &pd, int p, const PState &s, const Geo &g)
{
    Box ub, nb;
    const Box bc = pd.box_cur[p];
    remap_boxes(s, pd.pc[p], bc, pd.box_prev[p], g, ub, nb);
    pd.box_remap[p] = ub;
    pd.box_prev[p] = bc;
    pd.box_cur[p] = nb;
    pd.seg_cnt[p] = 0u;
}

// Set-up of the mapping from ps_cur (old poses, or the current ones) to
// ps_next: the previous pose is taken equal to the old one.
__global__ __launch_bounds__(256) void k_setup_boxes(PartData pd, Geo g)
{
    for (int p = blockIdx.x * blockDim.x + threadIdx.x; p < pd.np; p += gridDim.x * blockDim.x) {
        pd.ps_prev[p] = pd.ps_cur[p];
        pd.box_prev[p] = pd.box_cur[p];
        fiber_remap_boxes(pd, p, pd.ps_next[p], g);
    }
}

// ------------------------------------------------------------------ rigid update kernel
// One wave per fiber: its momentum-exchange sums (accumulated in fixed point
// by the boundary launch) back to FP64, the contact loads (when on), the
// rigid-body update, outputs, the boxes of the remap and the list reset.
// Bound by the latency of one serial FP64 chain (a 6x6 Cholesky, sine and
// cosine, three square roots); nine lanes form the B and C matrices, and the
// state and the records move as whole rows.
__global__ __launch_bounds__(64) void k_rigid(PartData pd, Geo g)
{
    constexpr int NPS = int(sizeof(PState) / sizeof(double));
    static_assert(sizeof(PState) % sizeof(double) == 0 && NPS <= 64, "one lane per word of a state");
    __shared__ double ac[NACC], s_out[NPS + 6], s_cl[64][6];
    const int p = int(blockIdx.x), np = pd.np, lane = int(threadIdx.x);
    const int64_t step = int64_t(pd.ctr->step);
    if (lane < NACC) {
        ac[lane] = ldexp(double(pd.mea[size_t(p) * NACC + lane]), -fx_shift(lane));
        pd.mea[size_t(p) * NACC + lane] = 0;   // cleared for the next step's boundary launch
    }
    // the pose of the previous step, about to be overwritten
    double *nxt = reinterpret_cast<double *>(pd.ps_next + p);
    if (lane < NPS) reinterpret_cast<double *>(pd.ps_prev + p)[lane] = nxt[lane];
    const PConst c = pd.pc[p];
    const PState s = pd.ps_cur[p];
    const double *row = nullptr;
    if (c.traj_off >= 0) {
        const int64_t at = pd.traj_pos[p];
        if (at < c.traj_n) row = pd.traj + (c.traj_off + at) * 13;
        __syncthreads();
        if (lane == 0 && row) pd.traj_pos[p] = at + 1;
    }
    // contact loads at the current poses, each pair in the orientation (lower
    // id, higher id) and summed over partners in ascending order
    double cl[6] = {0.0, 0.0, 0.0, 0.0, 0.0, 0.0};
    if (pd.contact_k > 0.0)
        for (int q0 = 0; q0 < np; q0 += 64) {
            const int q = q0 + lane;
            double l[6] = {0.0, 0.0, 0.0, 0.0, 0.0, 0.0};
            if (q < np && q != p) {
                if (p < q) contact_load(s, c, pd.ps_cur[q], pd.pc[q], true, pd.contact_k, pd.contact_range, g, l);
                else contact_load(pd.ps_cur[q], pd.pc[q], s, c, false, pd.contact_k, pd.contact_range, g, l);
            }
#pragma unroll
            for (int k = 0; k < 6; ++k) s_cl[lane][k] = l[k];
            __syncthreads();
            for (int e = 0; e < 64 && q0 + e < np; ++e)
#pragma unroll
                for (int k = 0; k < 6; ++k) cl[k] += s_cl[e][k];
            __syncthreads();
        }
    __syncthreads();
    abc_restore(ac, s.X, pd.rho0_link, lane);
    PState o;
    double F[3], M[3];
    rigid_update(s, c, ac, pd.coupling, row, g, o, F, M, pd.corr ? pd.corr + size_t(p) * 6 : nullptr,
                 pd.contact_k > 0.0 ? cl : nullptr);
    if (lane == 0) {
        bool bad = false;
        for (int k = 0; k < 3; ++k) bad |= !isfinite(F[k]) || !isfinite(M[k]);
        if (bad) atomicOr(&pd.ctr->err_unstable, 1u);
        if (g.xw || g.yw || g.zs) {
            // fibers keep more than one cell from x and y walls (the mapping
            // and momentum exchange take x and y as periodic) and from
            // free-slip z walls (a reflected population lands on a cell of
            // the wall layer, which must be fluid)
#pragma unroll
            for (int k = 0; k < 3; ++k) {
                if (!(k == 0 ? g.xw : (k == 1 ? g.yw : g.zs))) continue;
                const double ext = c.shape == 1 ? (0.5 * c.length - c.radius) * fabs(o.t[k]) + c.radius
                                                : 0.5 * c.length * fabs(o.t[k]) +
                                                      c.radius * sqrt(fmax(0.0, 1.0 - o.t[k] * o.t[k]));
                const double nk = k == 0 ? double(g.nx) : (k == 1 ? double(g.ny) : double(g.nz));
                if (o.X[k] - ext < 1.0 || o.X[k] + ext > nk - 2.0) atomicOr(&pd.ctr->err_wall, 1u);
            }
        }
        fiber_remap_boxes(pd, p, o, g);
        *reinterpret_cast<PState *>(s_out) = o;
#pragma unroll
        for (int k = 0; k < 3; ++k) {
            s_out[NPS + k] = F[k];
            s_out[NPS + 3 + k] = M[k];
        }
    }
    __syncthreads();
    if (lane < NPS) nxt[lane] = s_out[lane];
    if (lane < 6) pd.ft_out[size_t(p) * 6 + lane] = s_out[NPS + lane];
    // record F M X q V W (X q V W lead the state)
    if (lane < 19) pd.hist[((step % pd.hist_cap) * np + p) * 19 + lane] = lane < 6 ? s_out[NPS + lane] : s_out[lane - 6];
}

// ------------------------------------------------------------------ remap and boundary list
// Grid: np * nslab blocks; block (p, s) takes the z-planes s, s + nslab, ...
// of fiber p's remap box.  A cell inside the plane rectangle of a
// lower-indexed fiber is left to that fiber's blocks, so every cell is
// handled once.  The ids and boxes of the neighbouring fibers are staged in
// LDS.
struct NbrStage {
    int32_t id[NBR_CAP];
    Box box[NBR_CAP];
    int32_t n, nlow;
};

// Rectangles of a chunk of the block's planes, for one flattened pass over
// all their cells: rect[k * ne + 0] is the own fiber's rectangle in plane k
// of the chunk, rect[k * ne + j] that of the j-th lower-indexed neighbour
// (empty where the plane is outside the neighbour's box); pref holds the
// prefix of the own rectangles' cell counts.
constexpr int RT_MAXE = 512, RT_MAXP = 32;
struct RegionTable {
    Rect rect[RT_MAXE];
    int32_t z[RT_MAXP];
    int32_t pref[RT_MAXP + 1];
    int32_t npl, ne;
};

__device__ __forceinline__ void stage_nbrs(const PartData &pd, int p, NbrStage &sh, const Geo &g)
{
    __shared__ uint32_t s_wc[4], s_low;
    const Box a = pd.box_remap[p];
    if (threadIdx.x == 0) {
        sh.n = 0;
        s_low = 0u;
    }
    const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
    for (int o0 = 0; o0 < pd.np; o0 += blockDim.x) {   // block-uniform
        const int o = o0 + int(threadIdx.x);
        Box bo{};
        bool hit = false;
        if (o < pd.np && o != p) {
            bo = pd.box_remap[o];
            hit = boxes_meet(a, bo, g);
        }
        const unsigned long long bal = __ballot(hit);
        if (lane == 0) s_wc[wid] = uint32_t(__popcll(bal));
        __syncthreads();
        uint32_t k = uint32_t(sh.n) + uint32_t(__popcll(bal & ((1ull << lane) - 1ull)));
        for (int w = 0; w < wid; ++w) k += s_wc[w];
        const uint32_t pass = s_wc[0] + s_wc[1] + s_wc[2] + s_wc[3];   // read before the next pass writes
        if (hit) {
            if (k < uint32_t(NBR_CAP)) {
                sh.id[k] = o;
                sh.box[k] = bo;
            }
            if (o < p) atomicAdd(&s_low, 1u);
        }
        __syncthreads();
        if (threadIdx.x == 0) sh.n += int32_t(pass);
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        if (sh.n > NBR_CAP) {
            atomicOr(&pd.ctr->err_capacity, 1u);
            sh.n = NBR_CAP;
        }
        sh.nlow = min(int32_t(s_low), sh.n);
    }
    __syncthreads();
}

// Table of the planes iz0, iz0 + ns, ... of box b (as many as fit); returns
// the number of planes taken (block-uniform call).
__device__ int build_table(const PartData &pd, const NbrStage &sh, int p, const Box &b, int iz0, int ns,
                           const Geo &g, RegionTable &t)
{
    const int ne = sh.nlow + 1;
    const int left = iz0 < b.len[2] ? (b.len[2] - iz0 + ns - 1) / ns : 0;
    const int npl = min(left, min(RT_MAXP, RT_MAXE / ne));
    __syncthreads();   // the previous chunk's pass is done with the table
    for (int e = threadIdx.x; e < npl * ne; e += blockDim.x) {
        const int k = e / ne, j = e - k * ne;
        int32_t z = b.lo[2] + iz0 + k * ns;
        bool valid = true;
        if (g.zper) z = wrapc(z, int32_t(g.nz));
        else valid = z >= 0 && z < int32_t(g.nz);
        Rect r{1, 0, 1, 0};
        if (valid) {
            if (j == 0) r = remap_rect(pd, p, z, g);
            else if (in_zrange(sh.box[j - 1], z, g)) r = remap_rect(pd, sh.id[j - 1], z, g);
        }
        t.rect[e] = r;
        if (j == 0) t.z[k] = z;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        int32_t acc = 0;
        for (int k = 0; k < npl; ++k) {
            t.pref[k] = acc;
            const Rect r = t.rect[k * ne];
            if (r.x0 <= r.x1 && r.y0 <= r.y1) acc += (r.x1 - r.x0 + 1) * (r.y1 - r.y0 + 1);
        }
        t.pref[npl] = acc;
        t.npl = npl;
        t.ne = ne;
    }
    __syncthreads();
    return npl;
}

// cell idx of the chunk's flattened index space: plane k, position (x, y)
__device__ __forceinline__ void table_cell(const RegionTable &t, int idx, const Geo &g, int &k, int32_t &x,
                                           int32_t &y)
{
    k = 0;
    while (k + 1 < t.npl && t.pref[k + 1] <= idx) ++k;
    const Rect r = t.rect[k * t.ne];
    const int wx = r.x1 - r.x0 + 1, i = idx - t.pref[k];
    const int iy = i / wx, ix = i - iy * wx;
    x = wrapi(r.x0 + ix, int32_t(g.nx));
    y = wrapi(r.y0 + iy, int32_t(g.ny));
}

// a cell is handled by the lowest-indexed fiber whose region holds it
__device__ __forceinline__ bool owned_here(const RegionTable &t, int k, int32_t x, int32_t y, const Geo &g)
{
    for (int j = 1; j < t.ne; ++j)
        if (in_rect(t.rect[k * t.ne + j], x, y, g)) return false;
    return true;
}

// New owner of each cell of the regions, refill of uncovered cells, flags and
// the boundary-cell list.  The neighbours' owners are not read back but
// tested (claims), so mapping and list are one pass with no wait between
// them; 18 further tests cost 8 FP64 instructions each, on fluid cells within
// 1.5 of a surface only.  These are about a third of a region's cells: with
// QUEUE a wave collects them and tests 64 at a time, one to a lane, instead
// of sitting through the tests for the few of each 64 cells that need them.
// The detour costs 0.8 of 9.3 us where a fiber's blocks have a round of cells or
// two (the rule is where the fibers are set up).  Step in us without and with
// the queue: 64^3 six fibers 45.0, 44.3; 93^3 BF16 ten 65.0, 64.0; 128^3 with 200
// 152, 140, FP16 with 300 182, 165; 256^3 FP16 with 300 482, 459.
// The list is cut into one segment per fiber; a block
// stages the boundary cells it finds in all its planes in LDS and reserves a
// range of its fiber's segment with a single atomic (cells beyond the stage
// are appended one by one).  advance: end of a time step (the step counter).
constexpr int LSTAGE = 1024;

template <typename S, bool QUEUE>
__global__ __launch_bounds__(256) void k_map(S *__restrict__ f, int32_t *__restrict__ pid,
                                             uint8_t *__restrict__ flags, uint32_t *__restrict__ list_cell,
                                             uint32_t *__restrict__ list_mask, PartData pd, Geo g, int next_odd,
                                             double rho0, double scale, int advance)
{
    const int ns = pd.nslab;
    const int blk = int(xcd_block(blockIdx.x, gridDim.x));   // a fiber's blocks share one XCD's L2
    const int p = blk / ns, sl = blk % ns;
    __shared__ NbrStage sh;
    __shared__ uint32_t s_cell[LSTAGE], s_mask[LSTAGE];
    __shared__ uint32_t s_n, s_base;
    __shared__ uint32_t s_queue[QUEUE ? 4 : 1][QUEUE ? 128 : 1];   // cells of each wave to be tested
    if (advance && blockIdx.x == 0 && threadIdx.x == 0) pd.ctr->step += 1ull;
    if (threadIdx.x == 0) s_n = 0u;
    stage_nbrs(pd, p, sh, g);
    const Box b = pd.box_remap[p];
    const PState sp = QUEUE ? uniform(pd.ps_next[p]) : pd.ps_next[p];
    const PConst cp = QUEUE ? uniform(pd.pc[p]) : pd.pc[p];
    const uint32_t off = pd.seg_off[p], cap = pd.seg_cap[p];
    const bool quick = quick_claims(cp, g);
    const int lane = int(threadIdx.x & 63u);
    uint32_t *queue = s_queue[QUEUE ? threadIdx.x >> 6 : 0], nq = 0u;
    // a fluid cell with the bits of the own fiber and of all: flag and list entry
    auto list_fluid = [&](uint32_t cell, uint32_t mine, uint32_t mask) {
        if (!mask) {
            flags[cell] = 0;
            return;
        }
        if (!(mask & ~mine)) mask |= LIST_HOME;
        const uint32_t kk = atomicAdd(&s_n, 1u);
        if (kk < LSTAGE) {
            s_cell[kk] = cell;
            s_mask[kk] = mask;
        } else {
            // stage full: append directly
            const uint32_t r = atomicAdd(&pd.seg_cnt[p], 1u);
            if (r < cap) {
                const uint32_t e = off + r;
                list_cell[e] = cell;
                list_mask[e] = mask;
                flags[cell] = F_NEAR;
            } else {
                flags[cell] = 0;
                atomicOr(&pd.ctr->err_capacity, 2u);
            }
        }
    };
    // tests of the last n <= 64 cells of the queue (fluid: bit 0 stays clear)
    auto drain = [&](uint32_t n) {
        nq -= n;
        if (uint32_t(lane) >= n) return;
        const uint32_t cell = queue[nq + uint32_t(lane)];
        const uint32_t uz = fdiv(cell, g.dnxy), rem = cell - uz * g.nxy, uy = fdiv(rem, g.dnx);
        const int32_t x = int32_t(rem - uy * g.nx), y = int32_t(uy), z = int32_t(uz);
        const uint32_t mine = claims(sp, cp, x, y, z, g, quick);
        uint32_t any = mine;
        for (int j = sh.nlow; j < sh.n; ++j) {
            const int o = sh.id[j];
            if (in_box(sh.box[j], x, y, z, g)) any |= claims(pd.ps_next[o], pd.pc[o], x, y, z, g, quick_claims(pd.pc[o], g));
        }
        list_fluid(cell, mine, any);
    };
    __shared__ RegionTable t;
    for (int iz0 = sl; iz0 < b.len[2];) {   // block-uniform: chunks of planes
        iz0 += ns * build_table(pd, sh, p, b, iz0, ns, g, t);
        const int total = t.pref[t.npl];
        for (int i0 = int(threadIdx.x) - lane; i0 < total; i0 += int(blockDim.x)) {   // wave-uniform
            bool test = false;   // to the queue
            uint32_t cell = 0u;
            int k;
            int32_t x, y;
            if (i0 + lane < total) table_cell(t, i0 + lane, g, k, x, y);
            if (i0 + lane < total && owned_here(t, k, x, y, g)) {
                const int32_t z = t.z[k];
                cell = (uint32_t(z) * g.ny + uint32_t(y)) * g.nx + uint32_t(x);
                const int old = pid[cell];
                // bits of the own fiber, and of all: a lower-indexed fiber
                // cannot own or border this cell (it would handle it)
                auto bits = [&](const PState &s, const PConst &c, bool qk) {
                    return QUEUE ? claim_or_near(s, c, x, y, z, g, qk) : claims(s, c, x, y, z, g, qk);
                };
                const uint32_t mine = bits(sp, cp, quick);
                uint32_t any = mine;
                int owner = (mine & 1u) ? p : -1, nclaim = int(mine & 1u);
                for (int j = sh.nlow; j < sh.n; ++j) {
                    const int o = sh.id[j];
                    if (!in_box(sh.box[j], x, y, z, g)) continue;
                    const uint32_t m = bits(pd.ps_next[o], pd.pc[o], quick_claims(pd.pc[o], g));
                    any |= m;
                    if (m & 1u) {
                        if (owner < 0) owner = o;
                        ++nclaim;
                    }
                }
                if (nclaim > 1) atomicAdd(&pd.ctr->overlaps, (unsigned long long)(nclaim - 1));
                if (old >= 0 && owner < 0)   // uncovered
                    refill_cell<S>(f, g, x, y, z, pd.ps_cur[old], rho0, scale, next_odd);
                if (pd.cov && (old < 0) != (owner < 0)) {
                    // fluid cell count and momentum change for the stabilization
                    const uint32_t kc = atomicAdd(pd.cov, 1u);
                    if (kc < pd.cov_cap) pd.cov[1 + kc] = cell | (owner < 0 ? COV_UNCOVERED : 0u);
                    else atomicOr(&pd.ctr->err_capacity, 4u);
                }
                if (owner != old) pid[cell] = owner;
                test = QUEUE && owner < 0 && any;
                if (owner >= 0) flags[cell] = F_SOLID;
                else if (!test) list_fluid(cell, mine, QUEUE ? 0u : any);
            }
            if constexpr (QUEUE) {
                const unsigned long long hit = __ballot(test);
                if (test)
                    queue[nq + __builtin_amdgcn_mbcnt_hi(uint32_t(hit >> 32), __builtin_amdgcn_mbcnt_lo(uint32_t(hit), 0u))] =
                        cell;
                nq += uint32_t(__popcll(hit));
                __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
                __builtin_amdgcn_wave_barrier();
                if (nq >= 64u) drain(64u);
            }
        }
    }
    if constexpr (QUEUE) drain(nq);
    // one reservation for all planes of the block
    __syncthreads();
    const uint32_t n = min(s_n, uint32_t(LSTAGE));
    if (threadIdx.x == 0 && n) s_base = atomicAdd(&pd.seg_cnt[p], n);
    __syncthreads();
    for (uint32_t k = threadIdx.x; k < n; k += blockDim.x) {
        const uint32_t r = s_base + k, cell = s_cell[k];
        if (r < cap) {
            const uint32_t e = off + r;
            list_cell[e] = cell;
            list_mask[e] = s_mask[k];
            flags[cell] = F_NEAR;
        } else {
            flags[cell] = 0;
            atomicOr(&pd.ctr->err_capacity, 2u);
        }
    }
}

// ------------------------------------------------------------------ launchers
hipError_t launch_rigid(const PartData &pd, const Geo &g, hipStream_t st)
{
    hipLaunchKernelGGL(k_rigid, dim3(uint32_t(pd.np)), dim3(64), 0, st, pd, g);
    return hipGetLastError();
}

hipError_t launch_setup_boxes(const PartData &pd, const Geo &g, hipStream_t st)
{
    hipLaunchKernelGGL(k_setup_boxes, dim3((pd.np + 255) / 256), dim3(256), 0, st, pd, g);
    return hipGetLastError();
}

hipError_t launch_map(int sk, bool next_odd, void *f, int32_t *pid, uint8_t *flags, uint32_t *list_cell,
                      uint32_t *list_mask, const PartData &pd, const Geo &g, double rho0, double scale, bool advance,
                      hipStream_t st)
{
    const int no = next_odd ? 1 : 0, ad = advance ? 1 : 0;
    const dim3 gr(pd.np * pd.nslab), bl(256);
    auto go = [&](auto *fp) {
        using S = std::remove_pointer_t<decltype(fp)>;
        if (pd.queue)
            hipLaunchKernelGGL((k_map<S, true>), gr, bl, 0, st, fp, pid, flags, list_cell, list_mask, pd, g, no, rho0, scale, ad);
        else
            hipLaunchKernelGGL((k_map<S, false>), gr, bl, 0, st, fp, pid, flags, list_cell, list_mask, pd, g, no, rho0, scale, ad);
    };
    switch (sk) {
    case S_F32: go((float *)f); break;
    case S_F16: go((_Float16 *)f); break;
    case S_BF16: go((uint16_t *)f); break;
    default: go((double *)f); break;
    }
    return hipGetLastError();
}

}  // namespace lbm

// mlp.hip -- the closure network (247 -> 64 -> 64 -> 6, GELU, BF16 weights,
// FP32 activations and accumulation): forward, loss and gradient, Adam and
// the training loop.  The per-step closure (features, one-sample forward,
// correction in one launch) is in features.hip.
//
// Work layout.  One wave takes a sample through the network and back: lane j
// owns unit j of a hidden layer, the BF16 weights sit in the workgroup's LDS,
// and the activations stay in registers (a layer reads them lane by lane as
// scalar operands), so samples need no barrier.  A gradient is three launches: the waves leave every
// sample's activations and deltas in a work buffer (2 KiB a sample); the
// products delta x activation, one tile of 32 samples a workgroup and a few
// rows of a weight matrix each, go to a partial buffer; a reduction adds the
// partials in order.  Partial b holds the tiles b, b + 64, ... in that order,
// so the gradient is the same on every run.  The products are tiny (about 20k
// multiply-adds a sample, in FP32): what bounds a training batch is the chain
// of short dependent kernels, not the matrix units.  Measured, batch of 256:
// gradient and update 20 us (105 with one workgroup per tile of 32 samples
// doing all of it, eight workgroups on the card).
#include <algorithm>
#include <cmath>
#include <cstring>
#include <new>
#include <string>
#include <type_traits>
#include <vector>

#include "lbm_mlp_dev.h"

namespace lbm {

constexpr int TILE = 32, MB = 256, GRAD_BLOCKS = 64;
constexpr int ROWS_MAX = 4 * GRAD_BLOCKS * TILE;   // samples of one pass through the work buffer (16 MiB)
constexpr int ROW_GRID = 768;                      // resident workgroups of k_mlp_rows: three a CU
// a sample in the work buffer: normalised inputs and a one (the bias column),
// both hidden activations, dL/dz of both layers, dL/dy
constexpr int RX = 0, RH1 = 248, RH2 = RH1 + NH, RD1 = RH2 + NH, RD2 = RD1 + NH, RDY = RD2 + NH, ROW = 512;
static_assert(RDY + NO <= ROW && RX + NI < RH1, "work row");

__host__ __device__ inline uint16_t to_bf16(float v)
{
    uint32_t u = __builtin_bit_cast(uint32_t, v);
    if ((u & 0x7F800000u) == 0x7F800000u && (u & 0x007FFFFFu)) return uint16_t((u >> 16) | 0x40u);   // NaN stays NaN
    u += 0x7FFFu + ((u >> 16) & 1u);   // round to nearest even
    return uint16_t(u >> 16);
}

// derivative of the exact GELU: g'(z) = Phi(z) + z phi(z)
__device__ __forceinline__ float gelu_d(float z)
{
    return 0.5f * (1.0f + erff(z * 0.70710678118654752f)) + z * 0.39894228040143268f * expf(-0.5f * z * z);
}

// v of lane i, as a scalar operand
__device__ __forceinline__ float lane_val(float v, int i)
{
    return __uint_as_float(__builtin_amdgcn_readlane(__float_as_uint(v), i));
}

// acc + sum over i < NH of w[i] v(lane i) in order; w: 64 BF16 values
__device__ __forceinline__ float dot64(const uint4 (&w)[NH / 8], float v, float acc)
{
#pragma unroll
    for (int k = 0; k < NH / 8; ++k) {
        const uint32_t u[4] = {w[k].x, w[k].y, w[k].z, w[k].w};
#pragma unroll
        for (int l = 0; l < 4; ++l) {
            acc = fmaf(__uint_as_float(u[l] << 16), lane_val(v, 8 * k + 2 * l), acc);
            acc = fmaf(__uint_as_float(u[l] & 0xFFFF0000u), lane_val(v, 8 * k + 2 * l + 1), acc);
        }
    }
    return acc;
}

// Samples first + r (through idx if given), r < n.  !GRAD: y = the outputs
// times out_scale.  GRAD: the work rows r < nrow (zero rows from n on) and the
// workgroup's sum of squared errors, added to lpart[b] if add.
// Bound by a sample's serial chain (247 + 64 + 64 multiply-adds forward, 64
// back, each with its lane-to-scalar read) and the copy of the weights to LDS
// when there are few: 13 us for 256 samples; 37 us for 8192 forward (93 and
// 70 us with a layer's activations in LDS and 32 samples to a workgroup).
template <bool GRAD>
__global__ __launch_bounds__(MB, 3) void k_mlp_rows(const uint16_t *__restrict__ wb, const float *__restrict__ x,
                                                 const float *__restrict__ t, const int32_t *__restrict__ idx,
                                                 int first, int n, int nrow, const float *__restrict__ mean,
                                                 const float *__restrict__ inv_std,
                                                 const float *__restrict__ out_scale, float gscale,
                                                 float *__restrict__ y, float *__restrict__ work,
                                                 double *__restrict__ lpart, int add)
{
    __shared__ alignas(16) uint16_t w[(NP + 7) / 8 * 8];
    __shared__ double sl[MB / 64];
    static_assert(OW2 % 8 == 0 && OW3 % 8 == 0, "16-byte rows of w2 and w3");
    const int lane = threadIdx.x & 63, wid = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    for (int i = threadIdx.x; i < NP / 8; i += MB)
        reinterpret_cast<uint4 *>(w)[i] = reinterpret_cast<const uint4 *>(wb)[i];
    if (threadIdx.x < NP % 8) w[NP / 8 * 8 + threadIdx.x] = wb[NP / 8 * 8 + threadIdx.x];
    __syncthreads();
    const int o = lane < NO ? lane : 0;
    uint4 w2[NH / 8];   // row `lane` of w2
#pragma unroll
    for (int k = 0; k < NH / 8; ++k) w2[k] = *reinterpret_cast<const uint4 *>(&w[OW2 + lane * NH + 8 * k]);
    const float b1 = bf(w[OB1 + lane]), b2 = bf(w[OB2 + lane]), b3 = bf(w[OB3 + o]);
    double lsum = 0.0;
    for (int r = blockIdx.x * (MB / 64) + wid; r < nrow; r += gridDim.x * (MB / 64)) {   // wave-uniform
        float *row = GRAD ? work + size_t(r) * ROW : nullptr;
        if (GRAD && r >= n) {
            const float4 z = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
            reinterpret_cast<float4 *>(row)[lane] = z;
            reinterpret_cast<float4 *>(row)[64 + lane] = z;
            continue;
        }
        const int src = idx ? idx[first + r] : first + r;
        constexpr int NX = (NI + 63) / 64;
        float xv[NX];   // input lane + 64 k; a one in column NI
#pragma unroll
        for (int k = 0; k < NX; ++k) {
            const int i = lane + 64 * k;
            xv[k] = i < NI ? (x[size_t(src) * NI + i] - mean[i]) * inv_std[i] : 1.0f;
        }
        float z1 = b1;
#pragma unroll
        for (int k = 0; k < NX; ++k) {
            constexpr int last = NI - 64 * (NX - 1);
            asm volatile("" ::: "memory");   // the weights of 64 columns at a time in registers
            const uint16_t *wr = &w[OW1 + lane * NI + 64 * k];
#pragma unroll
            for (int i = 0; i < 64; ++i)
                if (k < NX - 1 || i < last) z1 = fmaf(bf(wr[i]), lane_val(xv[k], i), z1);
        }
        const float h1 = gelu(z1);
        const float z2 = dot64(w2, h1, b2), h2 = gelu(z2);
        asm volatile("" ::: "memory");
        uint4 w3[NH / 8];
#pragma unroll
        for (int k = 0; k < NH / 8; ++k) w3[k] = *reinterpret_cast<const uint4 *>(&w[OW3 + o * NH + 8 * k]);
        const float out = dot64(w3, h2, b3);
        if constexpr (!GRAD) {
            if (lane < NO) y[size_t(r) * NO + lane] = out * out_scale[lane];
        } else {
            const float d = lane < NO ? out - t[size_t(src) * NO + lane] : 0.0f, dy = gscale * d;
            lsum += double(d) * double(d);
            float a = 0.0f;
#pragma unroll
            for (int k = 0; k < NO; ++k) a = fmaf(bf(w[OW3 + k * NH + lane]), lane_val(dy, k), a);
            const float d2 = a * gelu_d(z2);
            a = 0.0f;
            asm volatile("" ::: "memory");
#pragma unroll
            for (int j = 0; j < NH; ++j) a = fmaf(bf(w[OW2 + j * NH + lane]), lane_val(d2, j), a);
#pragma unroll
            for (int k = 0; k < NX; ++k)
                if (lane + 64 * k < RH1) row[RX + lane + 64 * k] = xv[k];
            row[RH1 + lane] = h1;
            row[RH2 + lane] = h2;
            row[RD1 + lane] = a * gelu_d(z1);
            row[RD2 + lane] = d2;
            if (lane < ROW - RDY) row[RDY + lane] = dy;
        }
    }
    if constexpr (GRAD) {
        for (int d = 32; d > 0; d >>= 1) lsum += __shfl_xor(lsum, d, 64);
        if (lane == 0) sl[wid] = lsum;
        __syncthreads();
        if (threadIdx.x == 0) {
            double v = add ? lpart[blockIdx.x] : 0.0;
            for (int k = 0; k < MB / 64; ++k) v += sl[k];
            lpart[blockIdx.x] = v;
        }
    }
}

// Workgroups of k_mlp_prod along x: four rows of dW1 each, sixteen of dW2,
// and one for dW3 and the biases of the layers after the first.
constexpr int PROD_W1 = NH / 4, PROD_W2 = NH / 16, PROD_GRID = PROD_W1 + PROD_W2 + 1;

// The gradient's products over the tiles b, b + GRAD_BLOCKS, ... of the work
// rows (b = blockIdx.y), each tile's sum from zero, into part[b] (added to
// what is there if add).  A lane owns a column: its activations are coalesced
// loads, all 32 of a tile in flight, and the deltas of the rows are scalar.
// Bound by one trip to memory and the launch: 4 us for 8 tiles.
__global__ __launch_bounds__(MB) void k_mlp_prod(const float *__restrict__ work, int ntile, float *__restrict__ part,
                                                 int add)
{
    float *gp = part + size_t(blockIdx.y) * NP;
    const int lane = threadIdx.x & 63, wid = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    auto put = [&](int p, float v) { gp[p] = (add ? gp[p] : 0.0f) + v; };
    // NR rows of deltas from offset d against the column at offset c
    auto prod = [&](auto nr, int d, int c, float *g) {
        constexpr int NR = decltype(nr)::value;
#pragma unroll
        for (int k = 0; k < NR; ++k) g[k] = 0.0f;
        for (int tl = blockIdx.y; tl < ntile; tl += GRAD_BLOCKS) {
            const float *w = work + size_t(tl) * TILE * ROW;
            float a[NR], v[TILE];
#pragma unroll
            for (int k = 0; k < NR; ++k) a[k] = 0.0f;
#pragma unroll
            for (int r = 0; r < TILE; ++r) v[r] = w[r * ROW + c];
#pragma unroll
            for (int r = 0; r < TILE; ++r)
#pragma unroll
                for (int k = 0; k < NR; ++k) a[k] = fmaf(w[r * ROW + d + k], v[r], a[k]);
#pragma unroll
            for (int k = 0; k < NR; ++k) g[k] += a[k];
        }
    };
    const int bx = blockIdx.x;
    if (bx < PROD_W1) {
        const int j = bx * 4, i = threadIdx.x;
        if (i > NI) return;   // column NI: the bias
        float g[4];
        prod(std::integral_constant<int, 4>{}, RD1 + j, RX + i, g);
        for (int k = 0; k < 4; ++k) put(i < NI ? OW1 + (j + k) * NI + i : OB1 + j + k, g[k]);
    } else if (bx < PROD_W1 + PROD_W2) {
        const int j = (bx - PROD_W1) * 16 + wid * 4;
        float g[4];
        prod(std::integral_constant<int, 4>{}, RD2 + j, RH1 + lane, g);
        for (int k = 0; k < 4; ++k) put(OW2 + (j + k) * NH + lane, g[k]);
    } else if (wid == 0) {
        float g[NO];
        prod(std::integral_constant<int, NO>{}, RDY, RH2 + lane, g);
        for (int k = 0; k < NO; ++k) put(OW3 + k * NH + lane, g[k]);
    } else if (wid == 1 || (wid == 2 && lane < NO)) {   // a bias: the deltas against the ones
        float g = 0.0f;
        for (int tl = blockIdx.y; tl < ntile; tl += GRAD_BLOCKS) {
            const float *w = work + size_t(tl) * TILE * ROW + (wid == 1 ? RD2 : RDY) + lane;
            float a = 0.0f;
#pragma unroll
            for (int r = 0; r < TILE; ++r) a += w[r * ROW];
            g += a;
        }
        put((wid == 1 ? OB2 : OB3) + lane, g);
    }
}

struct AdamArgs {
    float *w, *m, *v;
    uint16_t *wb;
    float lr, b1, b2, eps, c1, c2;   // c1, c2: the bias corrections 1 - b^t
};

// Adam on the FP32 master: parameter p with gradient gg
__device__ __forceinline__ void adam_one(const AdamArgs &a, int p, float gg)
{
    const float mm = a.b1 * a.m[p] + (1.0f - a.b1) * gg;
    const float vv = a.b2 * a.v[p] + (1.0f - a.b2) * gg * gg;
    a.m[p] = mm;
    a.v[p] = vv;
    const float mh = mm / a.c1, vh = vv / a.c2;
    const float nw = a.w[p] - a.lr * mh / (sqrtf(vh) + a.eps);
    a.w[p] = nw;
    a.wb[p] = to_bf16(nw);
}

// grad[p] = sum over b of part[b][p] in order b, and with ADAM the update by
// it; loss = lscale times the sum of lpart
template <bool ADAM>
__global__ void k_mlp_reduce(const float *__restrict__ part, int nb, float *__restrict__ grad,
                             const double *__restrict__ lpart, int nl, double *__restrict__ loss, double lscale,
                             double *__restrict__ loss_acc, AdamArgs adam)
{
    for (int p = blockIdx.x * blockDim.x + threadIdx.x; p < NP; p += gridDim.x * blockDim.x) {
        float a = 0.0f;
#pragma unroll 8
        for (int b = 0; b < nb; ++b) a += part[size_t(b) * NP + p];
        grad[p] = a;
        if constexpr (ADAM) adam_one(adam, p, a);
    }
    if (blockIdx.x == 0 && threadIdx.x < 64) {
        double l = 0.0;
        for (int b = threadIdx.x; b < nl; b += 64) l += lpart[b];
        for (int d = 32; d > 0; d >>= 1) l += __shfl_xor(l, d, 64);
        if (threadIdx.x == 0) {
            *loss = l * lscale;
            if (loss_acc) *loss_acc += l * lscale;
        }
    }
}

__global__ void k_adam(AdamArgs a, const float *__restrict__ g)
{
    for (int p = blockIdx.x * blockDim.x + threadIdx.x; p < NP; p += gridDim.x * blockDim.x) adam_one(a, p, g[p]);
}

__global__ void k_bf16_copy(const float *__restrict__ w, uint16_t *__restrict__ wb)
{
    for (int p = blockIdx.x * blockDim.x + threadIdx.x; p < NP; p += gridDim.x * blockDim.x) wb[p] = to_bf16(w[p]);
}

__global__ void k_zero_d(double *p, int n)
{
    for (int i = blockIdx.x * blockDim.x + threadIdx.x; i < n; i += gridDim.x * blockDim.x) p[i] = 0.0;
}

}  // namespace lbm

using namespace lbm;

struct lbm_mlp {
    std::string err;
    hipStream_t st = nullptr;
    float *w = nullptr, *m = nullptr, *v = nullptr, *g = nullptr;
    uint16_t *wb = nullptr;
    float *in_mean = nullptr, *in_inv_std = nullptr, *out_scale = nullptr, *env_min = nullptr,
          *env_max = nullptr;
    float *work = nullptr, *part = nullptr;
    double *lpart = nullptr, *loss = nullptr, *loss_acc = nullptr;
    int64_t t = 0;   // Adam steps taken
};

namespace lbm {
MlpDev mlp_device_view(const lbm_mlp *m)
{
    MlpDev d{};
    d.wb = m->wb;
    d.in_mean = m->in_mean;
    d.in_inv_std = m->in_inv_std;
    d.out_scale = m->out_scale;
    d.env_min = m->env_min;
    d.env_max = m->env_max;
    return d;
}

hipError_t launch_mlp_forward(const MlpDev &m, const float *x, int n, float *y, hipStream_t st)
{
    if (n <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_mlp_rows<false>, dim3(std::min((n - 1) / (MB / 64) + 1, ROW_GRID)), dim3(MB), 0, st, m.wb, x,
                       nullptr, nullptr, 0, n, n, m.in_mean, m.in_inv_std, m.out_scale, 0.0f, y, nullptr, nullptr, 0);
    return hipGetLastError();
}

}  // namespace lbm

static lbm_status mfail(lbm_mlp *m, lbm_status s, const std::string &e)
{
    if (m) m->err = e;
    return s;
}

#define MHIP(m, call)                                                                        \
    do {                                                                                     \
        hipError_t e_ = (call);                                                              \
        if (e_ != hipSuccess)                                                                \
            return mfail((m), e_ == hipErrorOutOfMemory ? LBM_E_NOMEM : LBM_E_HIP,            \
                         std::string(#call) + ": " + hipGetErrorString(e_));                 \
    } while (0)

// splitmix64 (Steele, Lea and Flood; the constants of Vigna's reference code)
static uint64_t splitmix64(uint64_t &s)
{
    uint64_t z = (s += 0x9E3779B97F4A7C15ull);
    z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ull;
    z = (z ^ (z >> 27)) * 0x94D049BB133111EBull;
    return z ^ (z >> 31);
}
static double unit(uint64_t &s) { return double(splitmix64(s) >> 11) * (1.0 / 9007199254740992.0); }

static lbm_status upload_master(lbm_mlp *m, const float *w)
{
    MHIP(m, hipMemcpyAsync(m->w, w, NP * sizeof(float), hipMemcpyHostToDevice, m->st));
    hipLaunchKernelGGL(k_bf16_copy, dim3(80), dim3(256), 0, m->st, m->w, m->wb);
    MHIP(m, hipGetLastError());
    MHIP(m, hipMemsetAsync(m->m, 0, NP * sizeof(float), m->st));
    MHIP(m, hipMemsetAsync(m->v, 0, NP * sizeof(float), m->st));
    MHIP(m, hipStreamSynchronize(m->st));
    m->t = 0;
    return LBM_OK;
}

extern "C" {

lbm_status lbm_mlp_create(uint64_t seed, void *stream, lbm_mlp **out)
{
    if (!out) return LBM_E_ARG;
    *out = nullptr;
    lbm_mlp *m = new (std::nothrow) lbm_mlp;
    if (!m) return LBM_E_NOMEM;
    m->st = (hipStream_t)stream;
    auto bail = [&](lbm_status s) {
        lbm_mlp_destroy(m);
        return s;
    };
    if (hipMalloc(&m->w, NP * 4) != hipSuccess || hipMalloc(&m->m, NP * 4) != hipSuccess ||
        hipMalloc(&m->v, NP * 4) != hipSuccess || hipMalloc(&m->g, NP * 4) != hipSuccess ||
        hipMalloc(&m->wb, NP * 2) != hipSuccess || hipMalloc(&m->in_mean, NI * 4) != hipSuccess ||
        hipMalloc(&m->in_inv_std, NI * 4) != hipSuccess || hipMalloc(&m->out_scale, NO * 4) != hipSuccess ||
        hipMalloc(&m->env_min, NI * 4) != hipSuccess || hipMalloc(&m->env_max, NI * 4) != hipSuccess ||
        hipMalloc(&m->work, size_t(ROWS_MAX) * ROW * 4) != hipSuccess ||
        hipMalloc(&m->part, size_t(GRAD_BLOCKS) * NP * 4) != hipSuccess ||
        hipMalloc(&m->lpart, ROW_GRID * 8) != hipSuccess || hipMalloc(&m->loss, 8) != hipSuccess ||
        hipMalloc(&m->loss_acc, 8) != hipSuccess)
        return bail(LBM_E_NOMEM);
    std::vector<float> w(NP, 0.0f);
    uint64_t s = seed;
    auto fill = [&](int off, int rows, int cols, double gain) {
        const double a = gain * std::sqrt(6.0 / cols);
        for (int i = 0; i < rows * cols; ++i) w[off + i] = float((2.0 * unit(s) - 1.0) * a);
    };
    fill(OW1, NH, NI, 1.0);
    fill(OW2, NH, NH, 1.0);
    fill(OW3, NO, NH, 0.1);
    std::vector<float> zero(NI, 0.0f), one(NI, 1.0f), lo(NI, -3.0e38f), hi(NI, 3.0e38f);
    if (upload_master(m, w.data()) != LBM_OK) return bail(LBM_E_HIP);
    if (lbm_mlp_set_norm(m, zero.data(), one.data(), one.data(), lo.data(), hi.data()) != LBM_OK)
        return bail(LBM_E_HIP);
    *out = m;
    return LBM_OK;
}

lbm_status lbm_mlp_destroy(lbm_mlp *m)
{
    if (!m) return LBM_E_ARG;
    if (m->st) hipStreamSynchronize(m->st);
    else hipDeviceSynchronize();
    for (void *p : {(void *)m->w, (void *)m->m, (void *)m->v, (void *)m->g, (void *)m->wb, (void *)m->in_mean,
                    (void *)m->in_inv_std, (void *)m->out_scale, (void *)m->env_min, (void *)m->env_max,
                    (void *)m->work, (void *)m->part, (void *)m->lpart, (void *)m->loss, (void *)m->loss_acc})
        if (p) hipFree(p);
    delete m;
    return LBM_OK;
}

const char *lbm_mlp_last_error(const lbm_mlp *m) { return m ? m->err.c_str() : "null network"; }

lbm_status lbm_mlp_set_params(lbm_mlp *m, const float *w)
{
    if (!m || !w) return mfail(m, LBM_E_ARG, "null argument");
    return upload_master(m, w);
}

lbm_status lbm_mlp_get_params(lbm_mlp *m, float *w, uint16_t *wb)
{
    if (!m) return LBM_E_ARG;
    MHIP(m, hipStreamSynchronize(m->st));
    if (w) MHIP(m, hipMemcpy(w, m->w, NP * sizeof(float), hipMemcpyDeviceToHost));
    if (wb) MHIP(m, hipMemcpy(wb, m->wb, NP * sizeof(uint16_t), hipMemcpyDeviceToHost));
    return LBM_OK;
}

lbm_status lbm_mlp_set_norm(lbm_mlp *m, const float *in_mean, const float *in_inv_std, const float *out_scale,
                            const float *env_min, const float *env_max)
{
    if (!m) return LBM_E_ARG;
    if (in_mean) MHIP(m, hipMemcpyAsync(m->in_mean, in_mean, NI * 4, hipMemcpyHostToDevice, m->st));
    if (in_inv_std) MHIP(m, hipMemcpyAsync(m->in_inv_std, in_inv_std, NI * 4, hipMemcpyHostToDevice, m->st));
    if (out_scale) MHIP(m, hipMemcpyAsync(m->out_scale, out_scale, NO * 4, hipMemcpyHostToDevice, m->st));
    if (env_min) MHIP(m, hipMemcpyAsync(m->env_min, env_min, NI * 4, hipMemcpyHostToDevice, m->st));
    if (env_max) MHIP(m, hipMemcpyAsync(m->env_max, env_max, NI * 4, hipMemcpyHostToDevice, m->st));
    MHIP(m, hipStreamSynchronize(m->st));
    return LBM_OK;
}

lbm_status lbm_mlp_forward(lbm_mlp *m, const float *x, int32_t n, float *y)
{
    if (!m || n < 0 || (n > 0 && (!x || !y))) return mfail(m, LBM_E_ARG, "bad argument");
    MHIP(m, launch_mlp_forward(mlp_device_view(m), x, n, y, m->st));
    MHIP(m, hipStreamSynchronize(m->st));
    return LBM_OK;
}

static AdamArgs adam_args(lbm_mlp *m, float lr, float b1, float b2, float eps)
{
    m->t += 1;
    return {m->w, m->m, m->v, m->wb, lr, b1, b2, eps, float(1.0 - std::pow(double(b1), double(m->t))),
            float(1.0 - std::pow(double(b2), double(m->t)))};
}

// gradient of the mean squared error over samples first .. first+n-1 of
// the order idx (or natural order), into m->g; loss into m->loss (and added
// to m->loss_acc if accumulate); adam: the update by the gradient
static hipError_t grad_pass(lbm_mlp *m, const float *x, const float *t, const int32_t *idx, int first, int n,
                            bool accumulate, const AdamArgs *adam)
{
    const float gscale = 2.0f / float(n * NO);
    const int nb = std::min(GRAD_BLOCKS, (n - 1) / TILE + 1);
    int nl = 0;
    for (int at = 0; at < n; at += std::min(ROWS_MAX, n - at)) {
        const int k = std::min(ROWS_MAX, n - at), ntile = (k + TILE - 1) / TILE;
        const int grid = std::min(ntile * TILE / (MB / 64), ROW_GRID);
        nl = std::max(nl, grid);
        hipLaunchKernelGGL(k_mlp_rows<true>, dim3(grid), dim3(MB), 0, m->st, m->wb, x, t, idx, first + at, k,
                           ntile * TILE, m->in_mean, m->in_inv_std, nullptr, gscale, nullptr, m->work, m->lpart, at > 0);
        hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
        hipLaunchKernelGGL(k_mlp_prod, dim3(PROD_GRID, std::min(nb, ntile)), dim3(MB), 0, m->st, m->work, ntile, m->part,
                           at > 0);
        e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    const double lscale = 1.0 / double(n * NO);
    double *acc = accumulate ? m->loss_acc : nullptr;
    if (adam)
        hipLaunchKernelGGL(k_mlp_reduce<true>, dim3(80), dim3(256), 0, m->st, m->part, nb, m->g, m->lpart, nl, m->loss,
                           lscale, acc, *adam);
    else
        hipLaunchKernelGGL(k_mlp_reduce<false>, dim3(80), dim3(256), 0, m->st, m->part, nb, m->g, m->lpart, nl, m->loss,
                           lscale, acc, AdamArgs{});
    return hipGetLastError();
}

lbm_status lbm_mlp_loss_grad(lbm_mlp *m, const float *x, const float *t, int32_t n, double *loss, float *grad)
{
    if (!m || !x || !t || n < 1) return mfail(m, LBM_E_ARG, "bad argument");
    MHIP(m, grad_pass(m, x, t, nullptr, 0, n, false, nullptr));
    if (loss) MHIP(m, hipMemcpyAsync(loss, m->loss, 8, hipMemcpyDeviceToHost, m->st));
    if (grad) MHIP(m, hipMemcpyAsync(grad, m->g, NP * 4, hipMemcpyDeviceToHost, m->st));
    MHIP(m, hipStreamSynchronize(m->st));
    return LBM_OK;
}

lbm_status lbm_mlp_adam(lbm_mlp *m, float lr, float beta1, float beta2, float eps)
{
    if (!m || !(lr > 0.0f) || !(beta1 >= 0.0f && beta1 < 1.0f) || !(beta2 >= 0.0f && beta2 < 1.0f))
        return mfail(m, LBM_E_ARG, "bad Adam parameters");
    hipLaunchKernelGGL(k_adam, dim3(80), dim3(256), 0, m->st, adam_args(m, lr, beta1, beta2, eps), m->g);
    MHIP(m, hipGetLastError());
    MHIP(m, hipStreamSynchronize(m->st));
    return LBM_OK;
}

lbm_status lbm_mlp_train(lbm_mlp *m, const float *x, const float *t, int32_t n, int32_t epochs, int32_t batch,
                         float lr, uint64_t shuffle_seed, double *loss_per_epoch)
{
    if (!m || !x || !t || n < 1 || epochs < 1 || batch < 1 || !(lr > 0.0f))
        return mfail(m, LBM_E_ARG, "bad argument");
    int32_t *didx = nullptr;
    MHIP(m, hipMalloc(&didx, size_t(n) * sizeof(int32_t)));
    std::vector<int32_t> idx(n);
    uint64_t s = shuffle_seed;
    const int nbatch = (n + batch - 1) / batch;
    lbm_status st = LBM_OK;
    for (int ep = 0; ep < epochs && st == LBM_OK; ++ep) {
        for (int i = 0; i < n; ++i) idx[i] = i;
        for (int i = n - 1; i > 0; --i) {   // Fisher-Yates
            const int j = int(splitmix64(s) % uint64_t(i + 1));
            std::swap(idx[i], idx[j]);
        }
        hipError_t e = hipMemcpyAsync(didx, idx.data(), size_t(n) * 4, hipMemcpyHostToDevice, m->st);
        if (e == hipSuccess) {
            hipLaunchKernelGGL(k_zero_d, dim3(1), dim3(64), 0, m->st, m->loss_acc, 1);
            e = hipGetLastError();
        }
        for (int b = 0; b < nbatch && e == hipSuccess; ++b) {
            const int first = b * batch, cnt = std::min(batch, n - first);
            const AdamArgs adam = adam_args(m, lr, 0.9f, 0.999f, 1e-8f);
            e = grad_pass(m, x, t, didx, first, cnt, true, &adam);
        }
        double acc = 0.0;
        if (e == hipSuccess) e = hipMemcpyAsync(&acc, m->loss_acc, 8, hipMemcpyDeviceToHost, m->st);
        if (e == hipSuccess) e = hipStreamSynchronize(m->st);
        if (e != hipSuccess) st = mfail(m, LBM_E_HIP, std::string("train: ") + hipGetErrorString(e));
        else if (loss_per_epoch) loss_per_epoch[ep] = acc / nbatch;
    }
    hipStreamSynchronize(m->st);
    hipFree(didx);
    return st;
}

}  // extern "C"

// readback.h -- the error counters and one small device buffer to the host in
// one launch and one wait.
//
// A copy to pageable memory waits by itself, so a getter that copied the
// counters, synchronised and copied its data waited three times (about 40 us
// for the history of a case); a kernel that writes both to pinned host memory
// and one synchronisation take about 13.
#pragma once
#include <algorithm>
#include <cstring>

#include "lbm_dev.h"

namespace lbm {

// dst = the na words of a, then the nb words of b
static __global__ void k_pack(const uint64_t *__restrict__ a, uint32_t na, const uint64_t *__restrict__ b, uint32_t nb,
                              uint64_t *__restrict__ dst)
{
    for (uint32_t i = blockIdx.x * blockDim.x + threadIdx.x; i < na + nb; i += gridDim.x * blockDim.x)
        dst[i] = i < na ? a[i] : b[i - na];
}

struct Readback {
    static constexpr size_t CAP = 256 << 10;   // larger reads are copies of their own
    uint64_t *pin = nullptr;

    hipError_t create() { return hipHostMalloc((void **)&pin, sizeof(DevCounters) + CAP, hipHostMallocDefault); }
    void destroy()
    {
        if (pin) hipHostFree(pin);
        pin = nullptr;
    }
    // waits for st; h: the counters ctr; the bytes of src (a multiple of 8, at
    // most CAP of them) are left for take
    hipError_t read(hipStream_t st, const DevCounters *ctr, DevCounters &h, const void *src, size_t bytes)
    {
        constexpr uint32_t nc = sizeof(DevCounters) / 8;
        static_assert(sizeof(DevCounters) % 8 == 0, "whole words");
        const uint32_t nb = uint32_t(bytes / 8);
        hipLaunchKernelGGL(k_pack, dim3(std::min((nc + nb + 255u) / 256u, 64u)), dim3(256), 0, st,
                           reinterpret_cast<const uint64_t *>(ctr), nc, reinterpret_cast<const uint64_t *>(src), nb, pin);
        hipError_t e = hipGetLastError();
        if (e == hipSuccess) e = hipStreamSynchronize(st);
        if (e != hipSuccess) return e;
        std::memcpy(&h, pin, sizeof h);
        return e;
    }
    void take(void *out, size_t bytes) const { std::memcpy(out, pin + sizeof(DevCounters) / 8, bytes); }
};

}  // namespace lbm

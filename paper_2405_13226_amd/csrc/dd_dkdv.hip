// dd_dkdv.hip -- key-resident dK, dV of the attention backward for D = 128.
//
// This kernel is its own translation unit so that it can be built with its
// own machine-instruction scheduling strategy: scheduling for instruction-
// level parallelism measures ~6% faster on it at long sequences, while the
// same strategy slows the other backward and forward kernels.
#include "dd_bwd.hpp"
#include "dd_dkdv.hpp"
#include "dd_launch.hpp"
#include "dd_tile.hpp"

#include <algorithm>
#include <atomic>

namespace dd {

template <int D, bool PERSIST>
__global__ void __launch_bounds__(512, 1)
dkdv_kernel(const uint16_t *__restrict__ Q, const uint16_t *__restrict__ K,
            const uint16_t *__restrict__ V, const uint16_t *__restrict__ dO,
            const float *__restrict__ lse2g, const float *__restrict__ ndeltag,
            uint16_t *__restrict__ dK, uint16_t *__restrict__ dV, int B, int L, int H,
            int causal_i, const int32_t *__restrict__ cu, int n_docs, float scale_log2,
            float scale, int nkb, RopeEpi rt, int rope)
{
    using T = KvTile<D>;
    __shared__ __attribute__((aligned(1024))) uint16_t lds[2 * T::STAGE];
    __shared__ __attribute__((aligned(16))) float pbuf[T::PBUF_FLOATS];
    dkdv_body<D, PERSIST>(lds, pbuf, blockIdx.x, gridDim.x, Q, K, V, dO, lse2g, ndeltag, dK, dV, B, L, H,
                          causal_i, cu, n_docs, scale_log2, scale, nkb, rt, rope);
}

#define DD_KV_ARGS                                                                               \
    const uint16_t *__restrict__, const uint16_t *__restrict__, const uint16_t *__restrict__,   \
        const uint16_t *__restrict__, const float *__restrict__, const float *__restrict__,      \
        uint16_t *__restrict__, uint16_t *__restrict__, int, int, int, int,                      \
        const int32_t *__restrict__, int, float, float, int, RopeEpi, int
template __global__ void dkdv_kernel<128, false>(DD_KV_ARGS);
template __global__ void dkdv_kernel<128, true>(DD_KV_ARGS);
#undef DD_KV_ARGS

int device_cu_count()
{
    constexpr int kMaxDevices = 64;
    static std::atomic<int> cache[kMaxDevices];
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0)
        return 0;
    if (dev < kMaxDevices) {
        const int v = cache[dev].load(std::memory_order_relaxed);
        if (v > 0)
            return v;
    }
    int n = 0;
    if (hipDeviceGetAttribute(&n, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess)
        return 0;
    if (dev < kMaxDevices)
        cache[dev].store(n, std::memory_order_relaxed);
    return n;
}

hipError_t launch_dkdv_paired(const BwdArgs &a, const BwdScalars &s)
{
    using T = KvTile<128>;
    const int nkb = (a.L + T::BN - 1) / T::BN;
    const long long n_items = static_cast<long long>(nkb) * a.B * a.H;
    const long long all = (n_items + kXcds - 1) / kXcds * kXcds;
    hipStream_t st = static_cast<hipStream_t>(a.stream);
    // Persistent for short rows, as many workgroups as are resident at once
    // (one per CU); one item per workgroup otherwise, or when that many
    // workgroups already cover every item.
    const long long pgrid =
        a.L <= kPersistMaxSpan ? persistent_grid<dkdv_kernel<128, true>>(64 * T::NW) : 0;
    const bool persist = pgrid > 0 && pgrid < all;
    return launch_kernel(persist ? dkdv_kernel<128, true> : dkdv_kernel<128, false>,
                         dim3(static_cast<unsigned>(persist ? pgrid : all)), dim3(64 * T::NW), st,
                         a.Q, a.K, a.V, a.dO, s.lse2, s.ndelta, a.dK, a.dV, a.B, a.L, a.H,
                         a.causal ? 1 : 0, a.cu, a.n_docs, s.scale_log2, s.scale, nkb, s.rt,
                         s.rope);
}

}  // namespace dd

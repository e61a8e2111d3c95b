// Un-permute + weighted combine: y[t,:] = sum_i w[t,i] * y_perm[row_of[t*k+i], :].
// Paper: Eq. 3, Sec. 3.5 (fp32 accumulation).  Written as a gather per output row instead
// of the paper's scatter: no atomics, fixed slot order, bit-reproducible.
#include "moe_internal.hpp"

namespace moe {

namespace {

constexpr int kThreads = 256;

// KB: rows requested before the first is used (2, 4 or 8, by k): one row after the other a piece costs k
// memory latencies.  The sum runs in slot order whatever KB is.  Bound by HBM (k d * 2 bytes read, d * 2
// written per token) from a few thousand tokens on; below by latency: k = 8, stage by events, 100 tokens x 3584 9.8 -> 7.0 us,
// 512 x 7168 17.3 -> 15.0, 4096 x 7168 111 -> 111 (4.8 TB/s).
template <int KB>
__global__ __launch_bounds__(kThreads) void combine_kernel(const uint16_t* __restrict__ y_perm,
                                                          const int32_t* __restrict__ row_of,
                                                          const float* __restrict__ topk_w, int k, int d,
                                                          uint16_t* __restrict__ y) {
    const int t = blockIdx.x;
    const int32_t* rows = row_of + (size_t)t * k;
    const float* w = topk_w + (size_t)t * k;
    for (int c = threadIdx.x * 8; c < d; c += kThreads * 8) {
        float acc[8];
#pragma unroll
        for (int q = 0; q < 8; ++q) acc[q] = 0.0f;
        for (int i0 = 0; i0 < k; i0 += KB) {
            uint4 v[KB];
            float wi[KB];
#pragma unroll
            for (int b = 0; b < KB; ++b) {
                const int i = i0 + b < k ? i0 + b : k - 1;   // past the last slot: the last row again, not used
                v[b] = *reinterpret_cast<const uint4*>(y_perm + (size_t)rows[i] * d + c);
                wi[b] = w[i];
            }
#pragma unroll
            for (int b = 0; b < KB; ++b) {
                if (i0 + b < k) {
                    const uint32_t u[4] = {v[b].x, v[b].y, v[b].z, v[b].w};
#pragma unroll
                    for (int q = 0; q < 4; ++q) {
                        acc[2 * q] = fmaf(wi[b], __uint_as_float(u[q] << 16), acc[2 * q]);
                        acc[2 * q + 1] = fmaf(wi[b], __uint_as_float(u[q] & 0xffff0000u), acc[2 * q + 1]);
                    }
                }
            }
        }
        uint4 o;
        o.x = pack2_bf16(acc[0], acc[1]);
        o.y = pack2_bf16(acc[2], acc[3]);
        o.z = pack2_bf16(acc[4], acc[5]);
        o.w = pack2_bf16(acc[6], acc[7]);
        *reinterpret_cast<uint4*>(y + (size_t)t * d + c) = o;
    }
}

}  // namespace

hipError_t launch_combine(const moe_config& c, const uint16_t* y_perm, const int32_t* row_of,
                          const float* topk_w, uint16_t* y, hipStream_t s) {
    auto go = [&](auto kern) {
        hipLaunchKernelGGL(kern, dim3(c.T), dim3(kThreads), 0, s, y_perm, row_of, topk_w, c.k, c.d, y);
    };
    if (c.k <= 2) go(combine_kernel<2>);
    else if (c.k <= 4) go(combine_kernel<4>);
    else go(combine_kernel<8>);
    return hipGetLastError();
}

}  // namespace moe

// Un-permute + weighted combine: y[t,:] = sum_i w[t,i] * y_perm[row_of[t*k+i], :].
// Paper: Eq. 3, Sec. 3.5 (fp32 accumulation).  Written as a gather per output row instead
// of the paper's scatter: no atomics, fixed slot order, bit-reproducible.
#include <type_traits>

#include "moe_internal.hpp"

namespace moe {

namespace {

constexpr int kThreads = 256;
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

// N rows, of slots i .. i + N - 1: requested before the first is used (one row after the other a piece costs a memory
// latency per row), added in slot order.
template <int N, bool STREAM>
__device__ __forceinline__ void add_rows(const uint16_t* __restrict__ y_perm, const int32_t* __restrict__ rows,
                                         const float* __restrict__ w, int i, int d, int c, float (&acc)[8]) {
    u32x4 v[N];
    float wi[N];
#pragma unroll
    for (int b = 0; b < N; ++b) {
        const u32x4* p = reinterpret_cast<const u32x4*>(y_perm + (size_t)rows[i + b] * d + c);
        v[b] = STREAM ? __builtin_nontemporal_load(p) : *p;
        wi[b] = w[i + b];
    }
#pragma unroll
    for (int b = 0; b < N; ++b) {
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            acc[2 * q] = fmaf(wi[b], __uint_as_float(v[b][q] << 16), acc[2 * q]);
            acc[2 * q + 1] = fmaf(wi[b], __uint_as_float(v[b][q] & 0xffff0000u), acc[2 * q + 1]);
        }
    }
}

// K: experts per token where that is up to 8, else 0: batches of eight rows, then of 4, 2 and 1.  No row is requested that is not
// used: batches of 2, 4 or 8 that repeated the last row cost 3-7 % at 3, 5, 6 and 7 experts per token.
// Bound by HBM and the Infinity Cache (k d * 2 bytes read, d * 2 written per token) from about a thousand tokens on; below by
// latency.  Stage inside a layer by events, us, row by row / repeating batches / now: 6 experts, 900 tokens x 2048 8.0 / 8.6 /
// 7.9, 1200 x 3584 12.5 / 12.8 / 12.4, 4096 x 4096 39.6 / 40.4 / 40.2; 8 experts, 100 tokens x 3584 9.8 / 7.1 / 6.1, 512 x 7168
// 17.4 / 15.0 / 13.4, 4096 x 7168 110 / 109 / 105 (5.0 TB/s), 1024 x 4096 (64 MiB of rows) 15.3 / 17.8 / 17.6.
// STREAM: the rows pass the caches by (launch_combine).
template <int K, bool STREAM>
__global__ __launch_bounds__(kThreads) void combine_kernel(const uint16_t* __restrict__ y_perm,
                                                          const int32_t* __restrict__ row_of,
                                                          const float* __restrict__ topk_w, int k, int d,
                                                          uint16_t* __restrict__ y) {
    const int t = blockIdx.x;
    const int32_t* rows = row_of + (size_t)t * (K ? K : k);
    const float* w = topk_w + (size_t)t * (K ? K : k);
    for (int c = threadIdx.x * 8; c < d; c += kThreads * 8) {
        float acc[8];
#pragma unroll
        for (int q = 0; q < 8; ++q) acc[q] = 0.0f;
        if constexpr (K > 0) {
            add_rows<K, STREAM>(y_perm, rows, w, 0, d, c, acc);
        } else {
            int i = 0;
            for (; i + 8 <= k; i += 8) add_rows<8, STREAM>(y_perm, rows, w, i, d, c, acc);
            if (k & 4) add_rows<4, STREAM>(y_perm, rows, w, i, d, c, acc), i += 4;
            if (k & 2) add_rows<2, STREAM>(y_perm, rows, w, i, d, c, acc), i += 2;
            if (k & 1) add_rows<1, STREAM>(y_perm, rows, w, i, d, c, acc);
        }
        const u32x4 o = {pack2_bf16(acc[0], acc[1]), pack2_bf16(acc[2], acc[3]), pack2_bf16(acc[4], acc[5]), pack2_bf16(acc[6], acc[7])};
        *reinterpret_cast<u32x4*>(y + (size_t)t * d + c) = o;
    }
}

}  // namespace

hipError_t launch_combine(const moe_config& c, const uint16_t* y_perm, const int32_t* row_of,
                          const float* topk_w, uint16_t* y, hipStream_t s) {
    // From 128 MiB of rows on, half of the Infinity Cache, little of them is there and none is read again: non-temporal loads.  The result is
    // stored as usual: what comes next reads it.  Stage by events and a pass over the result after it, us, all cached / rows non-temporal / result
    // too: 8 experts, 4096 tokens x 3584 48.8 + 12.7 / 43.6 + 12.4 / 42.2 + 13.5, x 7168 104 + 21.2 / 93.6 + 20.3 (5.6 TB/s) / 90.5 + 21.9; 3 experts, 4096 x 7168
    // 42.0 + 20.3 / 41.6 + 20.2 / 41.6 + 22.3; below the line even or slower (6 experts, 4000 x 2048 21.1 / 22.4).
    const bool stream = (long long)c.T * c.k * c.d >= (1ll << 26);
    auto go = [&](auto k) {
        constexpr int K = decltype(k)::value;
        hipLaunchKernelGGL((stream ? combine_kernel<K, true> : combine_kernel<K, false>), dim3(c.T), dim3(kThreads), 0, s, y_perm, row_of,
                           topk_w, c.k, c.d, y);
    };
    using std::integral_constant;
    switch (c.k) {
        case 1: go(integral_constant<int, 1>{}); break;
        case 2: go(integral_constant<int, 2>{}); break;
        case 3: go(integral_constant<int, 3>{}); break;
        case 4: go(integral_constant<int, 4>{}); break;
        case 5: go(integral_constant<int, 5>{}); break;
        case 6: go(integral_constant<int, 6>{}); break;
        case 7: go(integral_constant<int, 7>{}); break;
        case 8: go(integral_constant<int, 8>{}); break;
        default: go(integral_constant<int, 0>{});
    }
    return hipGetLastError();
}

}  // namespace moe

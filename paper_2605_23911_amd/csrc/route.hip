// Router: logits z = W_r x (+ bias) in fp64 on the fp64 matrix cores, then softmax / sigmoid
// gate and a wavefront top-k.
// Paper: Eq. 1 and Eq. 2 (Sec. 2.1); Sec. 3.4 (max-subtracted softmax, iterative arg-max with
// the winner masked, softmax and sigmoid gating).  Unlike the paper the projection is part of
// this stage (no library GEMM), and the arg-max runs on the logits with an explicit
// "already chosen" mask instead of overwriting scores with -1.
//
// Why fp64: the expert indices must equal those of an exact evaluation.  With hundreds of
// experts and thousands of tokens the smallest gap between neighbouring top-(k+1) logits is of
// the order of 1e-6, below what an fp32-accumulated dot product of length d resolves.  bf16
// operands convert exactly to fp64 and their products are exact there, so the fp64 MFMA
// (v_mfma_f64_16x16x4) gives logits good to ~1e-15 at the fp64 matrix rate.
//
// From half a million logits on (and more than 8 experts) the fp64 work is cut down to the experts that can
// be among the k largest: a first pass computes every logit on the bf16 matrix cores with a
// proven error bound, the top-k pass takes the experts within twice that bound of the k-th
// largest value as candidates (k of them plus, rarely, one or two) and recomputes their logits
// exactly in fp64 before it selects.  Same indices, same order, same weights to ~1e-7 as the
// all-fp64 path at a third of its time (DeepSeek-V3 shape, T=4096); see fast_logits_kernel.
//
// Kernel 1 (logits): one wavefront per work unit (16 tokens x 16 experts x one slice of d).
//   The reduction is cut into enough slices to put >= ~2000 wavefronts on the chip even for
//   one token and eight experts; each unit writes its 16x16 fp64 partial tile.
// Kernel 2 (gate + top-k): one wavefront per token sums the slices, applies the gate and
//   selects k experts.
// Models with at most 8 experts take a single kernel instead (route_direct_kernel).
#include "lds_dma.hpp"
#include "moe_internal.hpp"

namespace moe {

namespace {

typedef double f64x4 __attribute__((ext_vector_type(4)));

constexpr int kThreads = 256;
constexpr int kWavesPerBlock = kThreads / kWave;
constexpr int kChunk = 32;   // reduction elements per chunk: 4 lane groups x 8 consecutive k

__device__ __forceinline__ double wave_sum(double v) {
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off, kWave);
    return v;
}

__device__ __forceinline__ double wave_max(double v) {
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) v = fmax(v, __shfl_xor(v, off, kWave));
    return v;
}

__device__ __forceinline__ void unpack8(const uint4& v, double* out) {
    const uint32_t w[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        out[2 * i] = (double)__uint_as_float(w[i] << 16);
        out[2 * i + 1] = (double)__uint_as_float(w[i] & 0xffff0000u);
    }
}

// ---- kernel 1: partial logit tiles ----------------------------------------------------------
// part[ks][t][e], t < T16*16, e < E16*16 (padded to whole tiles).
// MFMA operand layout (v_mfma_f64_16x16x4): lane l supplies A[i = l%16][k = l/16] and
// B[k = l/16][j = l%16]; it receives D[i = l/16 + 4v][j = l%16], v = 0..3.  The MFMA sums over
// k, so which k a slot carries is free as long as A and B agree: lane group g = l/16 loads 8
// consecutive k (one 16-byte load) and the q-th MFMA of a chunk takes element q of every lane.
// NT: 16-expert tiles per wavefront (1 or 4).  With 4 the token fragment is loaded and
// converted once per chunk for 64 experts (used when there are enough tiles to fill the chip
// without cutting the reduction).
template <int NT>
__global__ __launch_bounds__(kThreads) void logits_kernel(const uint16_t* __restrict__ x,
                                                         const uint16_t* __restrict__ wr,
                                                         double* __restrict__ part, int T, int d, int E, int T16,
                                                         int E16, int KS, int units) {
    const int lane = threadIdx.x % kWave;
    const int unit = blockIdx.x * kWavesPerBlock + threadIdx.x / kWave;
    if (unit >= units) return;
    const int EG = (E16 + NT - 1) / NT;   // expert-tile groups
    const int ks = unit % KS;
    const int eg = (unit / KS) % EG;
    const int tt = unit / (KS * EG);
    const int i = lane & 15, g = lane >> 4;

    const int nchunk = d / kChunk;
    const int per = (nchunk + KS - 1) / KS;
    const int c0 = ks * per;
    const int c1 = (c0 + per) < nchunk ? (c0 + per) : nchunk;

    const int trow = (tt * 16 + i) < T ? (tt * 16 + i) : (T - 1);
    const uint16_t* xp = x + (size_t)trow * d + g * 8;
    const uint16_t* wp[NT];
#pragma unroll
    for (int n = 0; n < NT; ++n) {
        const int erow = ((eg * NT + n) * 16 + i) < E ? ((eg * NT + n) * 16 + i) : (E - 1);
        wp[n] = wr + (size_t)erow * d + g * 8;
    }

    f64x4 acc[NT];
#pragma unroll
    for (int n = 0; n < NT; ++n) acc[n] = f64x4{0.0, 0.0, 0.0, 0.0};
    if (c0 < c1) {
        uint4 xr = *reinterpret_cast<const uint4*>(xp + (size_t)c0 * kChunk);
        uint4 wv[NT];
#pragma unroll
        for (int n = 0; n < NT; ++n) wv[n] = *reinterpret_cast<const uint4*>(wp[n] + (size_t)c0 * kChunk);
        for (int c = c0; c < c1; ++c) {
            const int cn = (c + 1 < c1) ? c + 1 : c;   // prefetch (the last chunk re-reads itself)
            const uint4 xn = *reinterpret_cast<const uint4*>(xp + (size_t)cn * kChunk);
            uint4 wn[NT];
#pragma unroll
            for (int n = 0; n < NT; ++n) wn[n] = *reinterpret_cast<const uint4*>(wp[n] + (size_t)cn * kChunk);
            double a8[8];
            unpack8(xr, a8);
#pragma unroll
            for (int n = 0; n < NT; ++n) {
                double b8[8];
                unpack8(wv[n], b8);
#pragma unroll
                for (int q = 0; q < 8; ++q)
                    acc[n] = __builtin_amdgcn_mfma_f64_16x16x4f64(a8[q], b8[q], acc[n], 0, 0, 0);
            }
            xr = xn;
#pragma unroll
            for (int n = 0; n < NT; ++n) wv[n] = wn[n];
        }
    }
    const size_t EP = (size_t)E16 * 16;
#pragma unroll
    for (int n = 0; n < NT; ++n) {
        const int et = eg * NT + n;
        if (et < E16) {
            double* out = part + ((size_t)ks * T16 * 16 + (size_t)tt * 16) * EP + (size_t)et * 16 + i;
#pragma unroll
            for (int v = 0; v < 4; ++v) out[(size_t)(g + 4 * v) * EP] = acc[n][v];
        }
    }
}

// ---- kernel 1, fast form: all logits on the bf16 matrix cores, with an error bound ----------
// One workgroup per 64 tokens x 128 experts x one slice of d, v_mfma_f32_32x32x16_bf16 with the token
// rows as the first operand.  Per step of 64 elements the workgroup brings its 64 token rows and
// each wavefront its own 32 expert rows global -> LDS (whole 128-byte pieces, swizzled source chunks:
// no bank conflicts), one step ahead into a ring of two buffers; the token rows are shared by the four
// wavefronts.  A lane supplies 8 reduction elements of one row per MFMA (chunk 2 s + lane / 32 of the
// step for MFMA s, in both operands) and receives D[token 8(v/4) + 4(lane/32) + v%4][expert lane%32].
// The four MFMAs of a step accumulate in fp32; the step's sum is added to fp64 accumulators.
// Bound by the loads (24 KiB per step and workgroup from L2).  256 experts, d = 7168, 4096 tokens: 90 us with
// each wavefront loading its own 160 rows to registers, now 31 (the router 167 -> 129; 2048 tokens 97 -> 77); as part of
// a layer, whose other kernels leave nothing of x in L2, 94 -> 41.
//
// Error bound.  bf16 products are exact in fp32.  Taking each MFMA's result (16 products plus
// the accumulator) to be off by at most 2^-19 of the sum of the magnitudes involved (32 units in
// the last place of the largest term: room for truncation and for a multi-stage adder), a group of
// four is off by at most 2^-17 * S_g, S_g = sum over the group of |x_k w_k|; the conversions and
// the fp64 additions add ~1e-16.  So
//     |z_fast - z| <= 2^-17 * sum_k |x_k w_k| <= 2^-17 * |x_t|_2 * |w_e|_2.
// The workgroups of the first token tile also leave sum_k w_ek^2 per expert and slice (fp32) for that.
// part[ks][t][e], t < TP (tokens padded to 64), e < EP (experts padded to 32), fp64; wsq[ks][e], fp32.
constexpr int kFastTokens = 64, kFastExperts = 128;
constexpr int kFastBuffers = 2;   // 48 KiB: three workgroups per CU (three buffers, two workgroups: 129 -> 136 us at T=3333)
constexpr int kFastBuf = (kFastTokens + kFastExperts) * 128;
__global__ __launch_bounds__(kThreads) void fast_logits_kernel(const uint16_t* __restrict__ x,
                                                              const uint16_t* __restrict__ wr,
                                                              double* __restrict__ part, float* __restrict__ wsq,
                                                              int T, int d, int E, int TP, int EP, int KS) {
    __shared__ __attribute__((aligned(1024))) char ring[kFastBuffers * kFastBuf];
    const int tid = threadIdx.x, lane = tid % kWave;
    const int wave = __builtin_amdgcn_readfirstlane(tid / kWave);
    const int li = lane & 31, half = lane >> 5;
    const int EG = (EP + kFastExperts - 1) / kFastExperts;
    const int ks = blockIdx.x % KS, eg = (blockIdx.x / KS) % EG, tt = blockIdx.x / (KS * EG);
    const int nstep = d / 64, per = (nstep + KS - 1) / KS;
    const int g0 = ks * per, g1 = g0 + per < nstep ? g0 + per : nstep;

    uint32_t xo[2], wo[4];   // byte offsets of this lane's source pieces (rows clamped into the tensors)
#pragma unroll
    for (int q = 0; q < 2; ++q) {
        const int rg = q * 4 + wave, t = tt * kFastTokens + rg * 8 + (lane >> 3);
        xo[q] = (uint32_t)((lane & 7) ^ (((lane >> 3) ^ rg) & 7)) * 16u + (uint32_t)(t < T ? t : T - 1) * (uint32_t)d * 2u;
    }
#pragma unroll
    for (int g = 0; g < 4; ++g) {
        const int e = eg * kFastExperts + wave * 32 + g * 8 + (lane >> 3);
        wo[g] = (uint32_t)((lane & 7) ^ (((lane >> 3) ^ g) & 7)) * 16u + (uint32_t)(e < E ? e : E - 1) * (uint32_t)d * 2u;
    }
    const uint32_t lds0 = (uint32_t)(uintptr_t)ring;
    const uint32_t x_dst = lds0 + wave * 1024, w_dst = lds0 + kFastTokens * 128 + wave * 4096;
    auto load = [&](int g, int buf) {
        const int gc = g < g1 ? g : g1 - 1;   // steps past the last re-read it (harmless)
        const char* xb = reinterpret_cast<const char*>(x) + (size_t)gc * 128;
        const char* wb = reinterpret_cast<const char*>(wr) + (size_t)gc * 128;
#pragma unroll
        for (int q = 0; q < 2; ++q) lds_dma16_at<false>(xb, xo[q], x_dst + buf * kFastBuf + q * 4096);
#pragma unroll
        for (int i = 0; i < 4; ++i) lds_dma16_at<false>(wb, wo[i], w_dst + buf * kFastBuf + i * 1024);
    };
    constexpr int LPS = 6;   // loads per wavefront and step
    const int sw0 = (li ^ (li >> 3)) & 7;
    const char* xs_b = ring + li * 128;
    const char* ws_b = ring + kFastTokens * 128 + wave * 4096 + li * 128;

    double acc[2][16];
#pragma unroll
    for (int b = 0; b < 2; ++b)
#pragma unroll
        for (int v = 0; v < 16; ++v) acc[b][v] = 0.0;
    float sq = 0.0f;
    if (g0 < g1) {
        constexpr int XD = kFastBuffers - 1;   // steps the loads run ahead
#pragma unroll
        for (int q = 0; q < XD; ++q) load(g0 + q, q);
        wait_vmcnt<(XD - 1) * LPS>();
        __syncthreads();
        for (int g = g0; g < g1; ++g) {
            const int buf = (g - g0) % kFastBuffers;
            load(g + XD, (g - g0 + XD) % kFastBuffers);   // the buffer read in the step before: free since its barrier
            f32x16 c[2];
#pragma unroll
            for (int b = 0; b < 2; ++b)
#pragma unroll
                for (int v = 0; v < 16; ++v) c[b][v] = 0.0f;
#pragma unroll
            for (int s = 0; s < 4; ++s) {
                const int at = (2 * s + half) ^ sw0;
                const uint4 w4 = *reinterpret_cast<const uint4*>(ws_b + buf * kFastBuf + (at & 7) * 16);
                const bf16x8 x0 = *reinterpret_cast<const bf16x8*>(xs_b + buf * kFastBuf + (at & 7) * 16);
                const bf16x8 x1 = *reinterpret_cast<const bf16x8*>(xs_b + buf * kFastBuf + 4096 + ((at ^ 4) & 7) * 16);
                c[0] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(x0, __builtin_bit_cast(bf16x8, w4), c[0], 0, 0, 0);
                c[1] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(x1, __builtin_bit_cast(bf16x8, w4), c[1], 0, 0, 0);
                if (tt == 0) {
                    const uint32_t u[4] = {w4.x, w4.y, w4.z, w4.w};
#pragma unroll
                    for (int i = 0; i < 4; ++i) {
                        const float lo = __uint_as_float(u[i] << 16), hi = __uint_as_float(u[i] & 0xffff0000u);
                        sq = fmaf(lo, lo, fmaf(hi, hi, sq));
                    }
                }
            }
#pragma unroll
            for (int b = 0; b < 2; ++b)
#pragma unroll
                for (int v = 0; v < 16; ++v) acc[b][v] += (double)c[b][v];
            wait_vmcnt<(XD - 1) * LPS>();   // everything of step g + 1 has landed
            __syncthreads();
        }
        wait_vmcnt<0>();         // nothing of this workgroup may still be writing LDS when it retires
    }
    const int e = eg * kFastExperts + wave * 32 + li;
    if (e >= EP) return;   // a whole wavefront beyond the padded experts
    double* out = part + ((size_t)ks * TP + (size_t)tt * kFastTokens) * EP + e;
#pragma unroll
    for (int b = 0; b < 2; ++b)
#pragma unroll
        for (int v = 0; v < 16; ++v) out[(size_t)(b * 32 + 8 * (v / 4) + 4 * half + v % 4) * EP] = acc[b][v];
    if (tt == 0) {
        const float both = sq + __shfl_xor(sq, 32, kWave);
        if (half == 0) wsq[(size_t)ks * EP + e] = both;
    }
}

// ---- gate + top-k of one token by one wavefront ---------------------------------------------
// Lane l holds the logits of experts l, l+64, ... in z[] (ok[] = expert exists).  Eq. 1-2,
// Sec. 3.4: max-subtracted softmax (or sigmoid), k rounds of arg-max over the logits with the
// winners masked, ties to the lower index.
constexpr int kLogitsPerLane = kMaxExperts / kWave;
// moe_forward's down projection counts, per (token, 128-feature group), how many of the token's
// k expert rows have been written (see ffn_kernels.hpp, fused_combine).  The counters of token t
// are cleared here by the wavefront that routes t, so the layer needs no clearing launch.
__device__ __forceinline__ void zero_token_counters(int32_t* __restrict__ zero, int zero_n, int t, int lane) {
    if (zero == nullptr) return;
    for (int i = lane; i < zero_n; i += kWave) zero[(size_t)t * zero_n + i] = 0;
}

// Q: logits per lane that can exist (E <= 64 Q): the exponentials and compares of the others are left out.
template <int Q>
__device__ __forceinline__ void gate_and_select(double (&z)[Q], const bool (&ok)[Q],
                                                int lane, int wave, int t, int k, int gating,
                                                double (*wsel)[kMaxExperts], int32_t (*sel_idx)[kMaxExperts],
                                                int32_t* __restrict__ topk_idx, float* __restrict__ topk_w) {
    const double ninf = -__builtin_huge_val();
    double p[Q];
#pragma unroll
    for (int q = 0; q < Q; ++q) z[q] = (z[q] != z[q]) ? ninf : z[q];   // a NaN logit can never win and never breaks the index range
    double m = ninf;
#pragma unroll
    for (int q = 0; q < Q; ++q) m = fmax(m, z[q]);
    m = wave_max(m);
    double psum = 0.0;
#pragma unroll
    for (int q = 0; q < Q; ++q) {
        if (gating == MOE_GATE_SIGMOID_NORM)
            p[q] = ok[q] ? 1.0 / (1.0 + exp(-z[q])) : 0.0;
        else
            p[q] = ok[q] ? exp(z[q] - m) : 0.0;
        psum += p[q];
    }
    psum = wave_sum(psum);
    if (gating != MOE_GATE_SIGMOID_NORM) {
        const double inv = 1.0 / psum;
#pragma unroll
        for (int q = 0; q < Q; ++q) p[q] = ok[q] ? p[q] * inv : 0.0;   // softmax scores, Eq. 1
    }

    unsigned taken = 0;   // bit q set: this lane's q-th expert already selected
    double wsum = 0.0;
    for (int r = 0; r < k; ++r) {
        double bv = ninf;
        int be = -1;
#pragma unroll
        for (int q = 0; q < Q; ++q) {
            if (ok[q] && !((taken >> q) & 1u) && (be < 0 || z[q] > bv)) {
                bv = z[q];
                be = lane + kWave * q;
            }
        }
#pragma unroll
        for (int off = 32; off > 0; off >>= 1) {
            const double ov = __shfl_xor(bv, off, kWave);
            const int oe = __shfl_xor(be, off, kWave);
            if (oe >= 0 && (be < 0 || ov > bv || (ov == bv && oe < be))) {
                bv = ov;
                be = oe;
            }
        }
        // every lane now holds the same winner `be` (ties resolved to the lower index)
        const int oq = be / kWave, ol = be % kWave;
        double mine = 0.0;
#pragma unroll
        for (int q = 0; q < Q; ++q) mine = (q == oq) ? p[q] : mine;
        const double wv = __shfl(mine, ol, kWave);
        if (lane == ol) taken |= 1u << oq;
        wsum += wv;
        if (lane == 0) {
            sel_idx[wave][r] = be;
            wsel[wave][r] = wv;
        }
    }
    const double scale = (gating == MOE_GATE_SOFTMAX) ? 1.0 : 1.0 / wsum;
    __builtin_amdgcn_wave_barrier();
    for (int i = lane; i < k; i += kWave) {
        topk_idx[(size_t)t * k + i] = *(volatile int32_t*)&sel_idx[wave][i];
        topk_w[(size_t)t * k + i] = (float)(*(volatile double*)&wsel[wave][i] * scale);
    }
}

// The logits of the experts that can be among the k largest, recomputed exactly (see
// fast_logits_kernel for the bound).  z holds the fast logits (bias included); on return the
// candidates' entries are exact: dot product in fp64 (bf16 operands and their products are
// exact there; the order of the additions moves the sum by ~1e-15), plus the bias.
// Why this is enough: let b = 2^-17 |x_t| max_e |w_e| >= every |z_fast - z|, and v_k the k-th
// largest fast value.  The k experts with the largest fast values have true logits >= v_k - b, so
// the true k-th largest logit is >= v_k - b, every expert of the true top-k has z >= v_k - b and
// therefore z_fast >= v_k - 2b: it is a candidate.  Every non-candidate has z <= z_fast + b <
// v_k - b, i.e. lies below k candidates' exact values, also when it keeps its fast value: the
// selection over the mixed array picks the same experts in the same order as over exact logits.
// The softmax denominator takes the non-candidates' fast values (relative error of a weight
// ~1e-7 at most: their scores weigh in with the error bound times their share).
// cand_list: LDS, kMaxExperts ints per wavefront.
__device__ __forceinline__ void refine_candidates(double (&z)[kLogitsPerLane], const bool (&ok)[kLogitsPerLane],
                                                  int lane, int t, int k, int E, int d, int KS, size_t EP,
                                                  const uint16_t* __restrict__ x, const uint16_t* __restrict__ wr,
                                                  const float* __restrict__ bias, const float* __restrict__ wsq,
                                                  int32_t* cand_list) {
    constexpr int Q = kLogitsPerLane;
    constexpr int CB = 12;  // candidates recomputed per pass over the token row (k = 8 gives 8, 9, rarely 10)
    const double ninf = -__builtin_huge_val();
    const uint16_t* xr = x + (size_t)t * d;
    // |x_t|^2 (fp32: squares of bf16 are exact, the sum is good to 1e-6 relative) and max_e |w_e|^2
    float xs = 0.0f;
    for (int p = lane; p < d / 8; p += kWave) {
        const uint4 v = *reinterpret_cast<const uint4*>(xr + (size_t)p * 8);
        const uint32_t w4[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const float lo = __uint_as_float(w4[i] << 16), hi = __uint_as_float(w4[i] & 0xffff0000u);
            xs = fmaf(lo, lo, fmaf(hi, hi, xs));
        }
    }
    float wm = 0.0f;
#pragma unroll
    for (int q = 0; q < Q; ++q) {
        const int e = lane + kWave * q;
        if (ok[q]) {
            float sum = 0.0f;
            for (int s0 = 0; s0 < KS; ++s0) sum += wsq[(size_t)s0 * EP + e];
            wm = fmaxf(wm, sum);
        }
    }
    const double x2 = wave_sum((double)xs), w2 = wave_max((double)wm);
    // twice the bound, with 1 % for the rounding of the two norms; NaN or inf makes every expert a candidate
    const double margin = 2.02 * 0x1p-17 * sqrt(x2 * w2);
    // k-th largest fast value
    unsigned taken = 0;
    double vk = ninf;
    for (int r = 0; r < k; ++r) {
        double bv = ninf;
        int bq = -1;
#pragma unroll
        for (int q = 0; q < Q; ++q) {
            if (ok[q] && !((taken >> q) & 1u) && (bq < 0 || z[q] > bv)) {
                bv = z[q];
                bq = q;
            }
        }
        int be = bq < 0 ? -1 : lane + kWave * bq;
#pragma unroll
        for (int off = 32; off > 0; off >>= 1) {
            const double ov = __shfl_xor(bv, off, kWave);
            const int oe = __shfl_xor(be, off, kWave);
            if (oe >= 0 && (be < 0 || ov > bv || (ov == bv && oe < be))) {
                bv = ov;
                be = oe;
            }
        }
        if (be >= 0 && lane == be % kWave) taken |= 1u << (be / kWave);
        vk = bv;
    }
    // candidate list (ascending expert index inside each q; the order does not matter)
    int n_cand = 0;
#pragma unroll
    for (int q = 0; q < Q; ++q) {
        const bool c = ok[q] && !(z[q] < vk - margin);   // written so that a NaN anywhere keeps the expert in
        const unsigned long long bal = __ballot(c);
        if (c) cand_list[n_cand + __popcll(bal & ((1ull << lane) - 1ull))] = lane + kWave * q;
        n_cand += __popcll(bal);
    }
    __builtin_amdgcn_wave_barrier();
    for (int c0 = 0; c0 < n_cand; c0 += CB) {
        int ce[CB];
#pragma unroll
        for (int b = 0; b < CB; ++b) ce[b] = *(volatile int32_t*)&cand_list[(c0 + b < n_cand) ? c0 + b : c0];
        double acc[CB];
#pragma unroll
        for (int b = 0; b < CB; ++b) acc[b] = 0.0;
        for (int p = lane; p < d / 8; p += kWave) {
            double xv[8];
            unpack8(*reinterpret_cast<const uint4*>(xr + (size_t)p * 8), xv);
            uint4 wv[CB];
#pragma unroll
            for (int b = 0; b < CB; ++b)   // the condition is uniform over the wavefront: unused slots cost nothing
                if (c0 + b < n_cand) wv[b] = *reinterpret_cast<const uint4*>(wr + (size_t)ce[b] * d + (size_t)p * 8);
#pragma unroll
            for (int b = 0; b < CB; ++b) {
                if (c0 + b < n_cand) {
                    double w8[8];
                    unpack8(wv[b], w8);
#pragma unroll
                    for (int j = 0; j < 8; ++j) acc[b] = fma(xv[j], w8[j], acc[b]);
                }
            }
        }
#pragma unroll
        for (int b = 0; b < CB; ++b) {
            if (c0 + b < n_cand) {   // uniform over the wavefront
                const double tot = wave_sum(acc[b]) + (bias ? (double)bias[ce[b]] : 0.0);
                if (lane == ce[b] % kWave) {
#pragma unroll
                    for (int q = 0; q < Q; ++q) z[q] = (q == ce[b] / kWave) ? tot : z[q];
                }
            }
        }
    }
}

// ---- kernel 2: gate + top-k, one wavefront per token ------------------------------------------
// FAST: `part` holds the fast logits' slices (see fast_logits_kernel), refined here.
// T16, E16: padded tokens and experts in units of 16 (FAST pads tokens to 64 and experts to 32, else both to 16).
template <bool FAST, int Q>
__global__ __launch_bounds__(kThreads) void topk_kernel(const double* __restrict__ part,
                                                       const float* __restrict__ bias,
                                                       int32_t* __restrict__ topk_idx, float* __restrict__ topk_w,
                                                       int T, int E, int k, int gating, int T16, int E16, int KS,
                                                       int32_t* __restrict__ zero, int zero_n,
                                                       const uint16_t* __restrict__ x, const uint16_t* __restrict__ wr,
                                                       int d, const float* __restrict__ wsq) {
    __shared__ double wsel[kWavesPerBlock][kMaxExperts];
    __shared__ int32_t sel_idx[kWavesPerBlock][kMaxExperts];
    const int wave = threadIdx.x / kWave, lane = threadIdx.x % kWave;
    const int t = blockIdx.x * kWavesPerBlock + wave;
    if (t >= T) return;
    zero_token_counters(zero, zero_n, t, lane);

    const double ninf = -__builtin_huge_val();
    const size_t EP = (size_t)E16 * 16;
    double z[Q];
    bool ok[Q];
#pragma unroll
    for (int q = 0; q < Q; ++q) {
        const int e = lane + kWave * q;
        ok[q] = e < E;
        double v = ninf;
        if (ok[q]) {
            v = bias ? (double)bias[e] : 0.0;
            for (int s0 = 0; s0 < KS; s0 += 8) {   // slices in fixed order; 8 independent loads at a time
                double tmp[8];
#pragma unroll
                for (int u = 0; u < 8; ++u)
                    tmp[u] = (s0 + u < KS) ? part[((size_t)(s0 + u) * T16 * 16 + t) * EP + e] : 0.0;
#pragma unroll
                for (int u = 0; u < 8; ++u) v += tmp[u];
            }
        }
        z[q] = v;
    }
    if constexpr (FAST) refine_candidates(z, ok, lane, t, k, E, d, KS, EP, x, wr, bias, wsq, sel_idx[wave]);
    gate_and_select(z, ok, lane, wave, t, k, gating, wsel, sel_idx, topk_idx, topk_w);
}

// ---- few experts (E <= 8): the whole router in one kernel, one workgroup per token ----------
// With 8 experts a 16x16 MFMA tile would be half padding and the two-kernel path costs
// two launches for a few microseconds of work.  Here thread i takes 8 consecutive k of every
// 2048, multiplies them with the same k of all E router rows in fp64 (bf16 -> fp64 is exact, so
// are the products); butterfly sums and one LDS exchange leave the logits in wavefront 0, which
// applies the gate and selects.  All loads of a thread are issued before the first use.
template <int EB>
__global__ __launch_bounds__(kThreads) void route_direct_kernel(const uint16_t* __restrict__ x,
                                                               const uint16_t* __restrict__ wr,
                                                               const float* __restrict__ bias,
                                                               int32_t* __restrict__ topk_idx,
                                                               float* __restrict__ topk_w, int d, int E, int k,
                                                               int gating, int32_t* __restrict__ zero, int zero_n) {
    __shared__ double wsel[1][kMaxExperts];
    __shared__ int32_t sel_idx[1][kMaxExperts];
    __shared__ double partial[kWavesPerBlock][EB];
    const int wave = threadIdx.x / kWave, lane = threadIdx.x % kWave;
    const int t = blockIdx.x;
    double acc[EB];
#pragma unroll
    for (int e = 0; e < EB; ++e) acc[e] = 0.0;
    const uint16_t* xr = x + (size_t)t * d;
    for (int k0 = threadIdx.x * 8; k0 < d; k0 += 2 * kThreads * 8) {
        // two chunks per trip (the second clamped to the first when it falls beyond d)
        const int k1 = k0 + kThreads * 8;
        const bool two = k1 < d;
        const int k1c = two ? k1 : k0;
        uint4 xa = *reinterpret_cast<const uint4*>(xr + k0), xb = *reinterpret_cast<const uint4*>(xr + k1c);
        uint4 wa[EB], wb[EB];
#pragma unroll
        for (int e = 0; e < EB; ++e) {   // rows beyond E re-read the last row; their sums are never used
            const uint16_t* row = wr + (size_t)(e < E ? e : E - 1) * d;
            wa[e] = *reinterpret_cast<const uint4*>(row + k0);
            wb[e] = *reinterpret_cast<const uint4*>(row + k1c);
        }
        double xv[8], yv[8];
        unpack8(xa, xv);
        unpack8(xb, yv);
#pragma unroll
        for (int e = 0; e < EB; ++e) {
            double w8[8];
            unpack8(wa[e], w8);
#pragma unroll
            for (int j = 0; j < 8; ++j) acc[e] = fma(xv[j], w8[j], acc[e]);
            unpack8(wb[e], w8);
            double a2 = 0.0;
#pragma unroll
            for (int j = 0; j < 8; ++j) a2 = fma(yv[j], w8[j], a2);
            acc[e] += two ? a2 : 0.0;
        }
    }
    // Sums over the wavefront: three halving exchanges leave each lane the sum of expert lane % 8 over its
    // eight lane groups' first three levels, three butterflies finish it: 10 exchanges instead of 6 per expert.
    static_assert(EB == 8, "halving exchanges over 8 sums");
    {
        double s4[4], s2[2], s1;
        const bool b0 = lane & 1, b1 = lane & 2, b2 = lane & 4;
#pragma unroll
        for (int i = 0; i < 4; ++i) {   // lanes with bit 0 set keep the odd experts
            const double keep = b0 ? acc[2 * i + 1] : acc[2 * i], give = b0 ? acc[2 * i] : acc[2 * i + 1];
            s4[i] = keep + __shfl_xor(give, 1, kWave);
        }
#pragma unroll
        for (int i = 0; i < 2; ++i) {   // s4[i] belongs to expert 2 i + bit 0; bit 1 keeps the odd i
            const double keep = b1 ? s4[2 * i + 1] : s4[2 * i], give = b1 ? s4[2 * i] : s4[2 * i + 1];
            s2[i] = keep + __shfl_xor(give, 2, kWave);
        }
        {
            const double keep = b2 ? s2[1] : s2[0], give = b2 ? s2[0] : s2[1];
            s1 = keep + __shfl_xor(give, 4, kWave);
        }
#pragma unroll
        for (int off = 8; off < kWave; off <<= 1) s1 += __shfl_xor(s1, off, kWave);
        if (lane < EB) partial[wave][lane] = s1;   // expert = lane % 8
    }
    __syncthreads();
    if (wave != 0) return;
    zero_token_counters(zero, zero_n, t, lane);
    double z[1] = {-__builtin_huge_val()};
    const bool ok[1] = {lane < E};
    if (ok[0]) {
        double v = bias ? (double)bias[lane] : 0.0;
#pragma unroll
        for (int w = 0; w < kWavesPerBlock; ++w) v += partial[w][lane];
        z[0] = v;
    }
    gate_and_select(z, ok, lane, 0, t, k, gating, wsel, sel_idx, topk_idx, topk_w);
}

struct RoutePlan {
    int T16, E16, KS, NT;
    bool fast;          // bf16 logits + exact candidates
    int TP, EP;         // fast: tokens padded to 64, experts padded to 32
};

// mode: the test knob's value.  -1 the rule, 1 every logit in fp64, 0 the bf16 first pass from 256 tokens on.
RoutePlan plan(const moe_config& c, int mode) {
    RoutePlan p{};
    // From half a million logits on (256 experts: 2048 tokens).  Measured, us, all in fp64 / first pass and candidates:
    // 256 experts (d 7168) 512 tokens 57 / 63, 1024 86 / 67, 2048 152 / 77, 4096 289 / 129; 160 experts (d 5120) 1024 tokens
    // 55 / 48, 2048 92 / 55, 4096 208 / 93; 128 experts (d 4096) 2048 tokens 53 / 41, 4096 92 / 69; 64 experts (d 3584) 4096
    // tokens 53 / 78, 8192 93 / 139.  By time alone the line would be at about 2^18 for more than 64 experts and nowhere up to
    // 64 (the candidates, ~k + 1 rows per token, are then too large a part of all).  It lies higher because below it the softmax
    // weights keep the last 0.5-1.4 % of precision that the non-candidates' share of the denominator takes (relative error
    // 2.51e-8 / 2.53e-8 at 256 experts, 1024 tokens; with the other two gates the two forms agree).
    // Its 32-bit byte offsets hold: every entry point refuses T d 2 >= 2^32 bytes, and here E <= 256 <= T.
    p.fast = mode != 1 && c.E > 8 && (mode == 0 ? c.T >= 256 : (long long)c.T * c.E >= (1ll << 19));
    if (p.fast) {
        p.TP = (c.T + kFastTokens - 1) / kFastTokens * kFastTokens;
        p.EP = (c.E + 31) / 32 * 32;
        const long long tiles = (long long)(p.TP / kFastTokens) * ((p.EP + kFastExperts - 1) / kFastExperts);
        const int nstep = c.d / 64;
        long long ks = (512 + tiles - 1) / tiles;           // two workgroups per CU
        if (ks > 8) ks = 8;                                 // the refining kernel sums the slices
        if (ks > nstep / 2) ks = nstep / 2;
        if (ks < 1) ks = 1;
        p.KS = (int)ks;
        return p;
    }
    p.T16 = (c.T + 15) / 16;
    p.E16 = (c.E + 15) / 16;
    // four expert tiles per wavefront (the converted token fragment is then shared by 64 experts)
    // from 64 such units on; the reduction is cut further to keep ~2000 wavefronts (measured:
    // Qwen2-MoE shape T=4096 85 -> 67 us, DeepSeek-V3 shape T=512 66 -> 57 us)
    p.NT = (p.E16 >= 4 && (long long)p.T16 * ((p.E16 + 3) / 4) >= 64) ? 4 : 1;
    const long long tiles = (long long)p.T16 * ((p.E16 + p.NT - 1) / p.NT);
    const int nchunk = c.d / kChunk;
    long long ks = (2048 + tiles - 1) / tiles;          // aim for >= ~2048 wavefronts
    if (ks > 16) ks = 16;                               // the top-k kernel sums the slices serially
    if (ks > nchunk / 2) ks = nchunk / 2;               // at least two chunks per slice
    if (ks < 1) ks = 1;
    if (p.NT == 4 && tiles * ks > 2048) {
        // More wavefronts than two per SIMD: a third round for the few left over.  The slice count
        // whose rounds are shortest: ceil(wavefronts / SIMDs) * chunks per slice.  (256 experts, 1000
        // tokens: 9 slices of 252 tiles 105 us, 8 slices 85; 160 experts, 1024 tokens 68 -> 55.)
        long long best = 1ll << 60;
        for (long long n = 1, most = ks; n <= most; ++n) {
            const long long cost = ((tiles * n + 1023) / 1024) * ((nchunk + n - 1) / n);
            if (cost <= best) {
                best = cost;
                ks = n;
            }
        }
    }
    p.KS = (int)ks;
    return p;
}

}  // namespace

size_t route_workspace_bytes(const moe_config& c) {
    if (c.T == 0) return 0;
    // sized for whichever form a test knob may switch to
    size_t need = 0;
    for (int mode = -1; mode <= 1; ++mode) {
        const RoutePlan p = plan(c, mode);
        const size_t bytes = p.fast ? (size_t)p.KS * p.EP * ((size_t)p.TP * sizeof(double) + sizeof(float))
                                    : (size_t)p.KS * p.T16 * 16 * p.E16 * 16 * sizeof(double);
        need = bytes > need ? bytes : need;
    }
    return need;
}

hipError_t launch_route(const moe_config& c, const uint16_t* x, const uint16_t* wr, const float* bias,
                        int32_t* topk_idx, float* topk_w, void* workspace, int32_t* zero, int zero_per_token, hipStream_t s) {
    if (c.E <= 8 && c.T <= 2048) {   // measured: with 16 experts or more tokens the MFMA path is faster
        const dim3 g(c.T);
        hipLaunchKernelGGL(route_direct_kernel<8>, g, dim3(kThreads), 0, s, x, wr, bias, topk_idx, topk_w, c.d, c.E,
                           c.k, c.gating, zero, zero_per_token);
        return hipGetLastError();
    }
    const RoutePlan p = plan(c, knob(kKnobRouteExact));
    if (p.fast) {
        double* part = (double*)workspace;
        float* wsq = (float*)(part + (size_t)p.KS * p.TP * p.EP);
        hipLaunchKernelGGL(fast_logits_kernel, dim3((p.TP / kFastTokens) * ((p.EP + kFastExperts - 1) / kFastExperts) * p.KS), dim3(kThreads), 0, s, x,
                           wr, part, wsq, c.T, c.d, c.E, p.TP, p.EP, p.KS);
        hipLaunchKernelGGL((topk_kernel<true, kLogitsPerLane>), dim3((c.T + kWavesPerBlock - 1) / kWavesPerBlock), dim3(kThreads), 0, s,
                           part, bias, topk_idx, topk_w, c.T, c.E, c.k, c.gating, p.TP / 16, p.EP / 16, p.KS, zero, zero_per_token,
                           x, wr, c.d, wsq);
        return hipGetLastError();
    }
    const int units = p.T16 * ((p.E16 + p.NT - 1) / p.NT) * p.KS;
    double* part = (double*)workspace;
    const dim3 grid((units + kWavesPerBlock - 1) / kWavesPerBlock);
    if (p.NT == 4)
        hipLaunchKernelGGL(logits_kernel<4>, grid, dim3(kThreads), 0, s, x, wr, part, c.T, c.d, c.E, p.T16, p.E16,
                           p.KS, units);
    else
        hipLaunchKernelGGL(logits_kernel<1>, grid, dim3(kThreads), 0, s, x, wr, part, c.T, c.d, c.E, p.T16, p.E16,
                           p.KS, units);
    auto select = [&](auto kern) {
        hipLaunchKernelGGL(kern, dim3((c.T + kWavesPerBlock - 1) / kWavesPerBlock), dim3(kThreads), 0, s, part, bias, topk_idx,
                           topk_w, c.T, c.E, c.k, c.gating, p.T16, p.E16, p.KS, zero, zero_per_token, nullptr, nullptr, 0, nullptr);
    };
    if (c.E <= 64) select(topk_kernel<false, 1>);
    else if (c.E <= 128) select(topk_kernel<false, 2>);
    else select(topk_kernel<false, 4>);
    return hipGetLastError();
}

}  // namespace moe

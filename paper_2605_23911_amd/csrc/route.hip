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
// Larger calls take the logits from the int8 matrix cores instead (64 times the fp64 rate): rows are cut
// into four 8-bit digits, the digits' products are summed exactly in integers, and what the digits leave out is bounded.
// Tiles where the bound says too little for a softmax over all experts are formed in fp64 as above; tokens whose k + 1 largest
// logits stand closer together than the bound, or whose selected experts' bound is too loose, get the logits in question again in
// fp64.  Same indices, same order, same weights to the last bit but one as the all-fp64 form (digit_logits_kernel, kCertain with
// the exception from 2^19 logits on, digits_pay).  After the splitting of operands into digits with exact products of K. Ozaki, T. Ogita,
// S. Oishi and S. M. Rump, "Error-free transformations of matrix multiplication by using fast routines of matrix
// multiplication and its applications", Numer. Algorithms 59 (2012), and its use on integer matrix units by H. Ootomo, K. Ozaki and
// R. Yokota, "DGEMM on integer matrix multiplication unit" (2023).
//
// Kernel 1 (logits): one wavefront per work unit (16 tokens x 16 experts x one slice of d).
//   The reduction is cut into enough slices to put >= ~2000 wavefronts on the chip even for
//   one token and eight experts; each unit writes its 16x16 fp64 partial tile.
// Kernel 2 (gate + top-k): one wavefront per token sums the slices, applies the gate and
//   selects k experts.
// Models with at most 8 experts take a single kernel instead (route_direct_kernel).
#include <type_traits>

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
// MT, NT: 16-token and 16-expert tiles per wavefront.  xp, wp: this lane's rows.  Chunks c0 .. c1 - 1 of kChunk elements.
template <int MT, int NT>
__device__ __forceinline__ void fp64_tiles(const uint16_t* const (&xp)[MT], const uint16_t* const (&wp)[NT], int c0, int c1, f64x4 (&acc)[MT][NT]) {
#pragma unroll
    for (int m = 0; m < MT; ++m)
#pragma unroll
        for (int n = 0; n < NT; ++n) acc[m][n] = f64x4{0.0, 0.0, 0.0, 0.0};
    if (c0 >= c1) return;
    uint4 xr[MT], wv[NT];
#pragma unroll
    for (int m = 0; m < MT; ++m) xr[m] = *reinterpret_cast<const uint4*>(xp[m] + (size_t)c0 * kChunk);
#pragma unroll
    for (int n = 0; n < NT; ++n) wv[n] = *reinterpret_cast<const uint4*>(wp[n] + (size_t)c0 * kChunk);
    for (int c = c0; c < c1; ++c) {
        const int cn = (c + 1 < c1) ? c + 1 : c;   // prefetch (the last chunk re-reads itself)
        uint4 xn[MT], wn[NT];
#pragma unroll
        for (int m = 0; m < MT; ++m) xn[m] = *reinterpret_cast<const uint4*>(xp[m] + (size_t)cn * kChunk);
#pragma unroll
        for (int n = 0; n < NT; ++n) wn[n] = *reinterpret_cast<const uint4*>(wp[n] + (size_t)cn * kChunk);
        double a8[MT][8];
#pragma unroll
        for (int m = 0; m < MT; ++m) unpack8(xr[m], a8[m]);
#pragma unroll
        for (int n = 0; n < NT; ++n) {
            double b8[8];
            unpack8(wv[n], b8);
#pragma unroll
            for (int q = 0; q < 8; ++q)
#pragma unroll
                for (int m = 0; m < MT; ++m) acc[m][n] = __builtin_amdgcn_mfma_f64_16x16x4f64(a8[m][q], b8[q], acc[m][n], 0, 0, 0);
        }
#pragma unroll
        for (int m = 0; m < MT; ++m) xr[m] = xn[m];
#pragma unroll
        for (int n = 0; n < NT; ++n) wv[n] = wn[n];
    }
}

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
    const uint16_t* xp[1] = {x + (size_t)trow * d + g * 8};
    const uint16_t* wp[NT];
#pragma unroll
    for (int n = 0; n < NT; ++n) {
        const int erow = ((eg * NT + n) * 16 + i) < E ? ((eg * NT + n) * 16 + i) : (E - 1);
        wp[n] = wr + (size_t)erow * d + g * 8;
    }
    f64x4 acc[1][NT];
    fp64_tiles(xp, wp, c0, c1, acc);
    const size_t EP = (size_t)E16 * 16;
#pragma unroll
    for (int n = 0; n < NT; ++n) {
        const int et = eg * NT + n;
        if (et < E16) {
            double* out = part + ((size_t)ks * T16 * 16 + (size_t)tt * 16) * EP + (size_t)et * 16 + i;
#pragma unroll
            for (int v = 0; v < 4; ++v) out[(size_t)(g + 4 * v) * EP] = acc[0][n][v];
        }
    }
}

// ---- kernel 1 on the int8 matrix cores: every logit from exact integer sums ------------------
// A row v (a token or an expert) with 2^E <= max|v_k| < 2^(E+1) is written in fixed point as
//     v_k = 2^(E-29) (q0 2^24 + q1 2^16 + q2 2^8 + q3) + residual,   q0 in [-65, 65], q1..q3 in [-128, 127].
// bf16 has 8 significant bits, so the residual is zero unless |v_k| < 2^(E-22).  The products q_i q_j are summed over k
// by v_mfma_i32_32x32x32_i8, which is exact, one int32 accumulator per order i + j = 0..4; orders 5 and 6 (2^-40 and less of
// the largest possible term) are left out.  The five sums meet in fp64.
//
// Error bound.  Let A be the largest magnitude in a row, N2 and N3 the 2-norms of its parts q2, q3 and q3 alone, R the sum of
// the residuals' magnitudes, as bounded by digits_kernel from how many elements have such a part.  The pairs left out are
// (2,3), (3,2), (3,3) (Cauchy-Schwarz) and whatever a residual meets:
//     |z_digits - z| <= N2(x) N3(w) + N3(x) N2(w) + R(x) A(w) + A(x) R(w)
// plus the fp64 roundings.  For normally distributed rows of 7168 that is about 1e-9, the error itself 1e-11: an exact
// evaluation for the purpose of the weights, and topk_kernel recomputes in fp64 what stands closer together than the bound.
// Where the bound over a tile of 128 tokens x 64 experts says too little (elements hundreds of times the others', infinities,
// NaN), the workgroups of that tile take their logits from the fp64 matrix cores instead: tile_limit.
//
// What bounds it: the int8 matrix rate, 13 products (256 experts, 1024 tokens, d = 7168: 49 GOP, 10 us at 5 POP/s).
// A wavefront takes 64 experts (two 32-expert operands) and 32 tokens, the experts' digits straight from memory in operand
// order (digits_kernel lays them out), one 32-element step ahead in registers; the tokens come as bf16 by DMA
// through LDS and are cut into digits in registers between the matrix
// instructions (7 vector instructions per element, about half of the issue slots that 13 products of 64 experts leave).
constexpr int kShortRows = 2200;     // rows up to which digits_kernel gives each a workgroup
constexpr int kMinExp = -90;         // smallest E: keeps every scale a normal fp32 number
constexpr int kMaxDigitSlice = 32768;                // 4 pairs x 2^14 x this many elements fill an int32
constexpr int kMaxDigitSlices = 16;                  // topk_kernel sums the slices
constexpr int kMaxDigitDim = kMaxDigitSlice * kMaxDigitSlices;

typedef int i32x4 __attribute__((ext_vector_type(4)));
typedef int i32x16 __attribute__((ext_vector_type(16)));

__device__ __forceinline__ float exp2i(int e) { return __uint_as_float((uint32_t)(e + 127) << 23); }   // -126 <= e <= 127

// Digits of four bf16 values (two words, low half first): out[p] holds digit p of all four, one byte each.
__device__ __forceinline__ void four_digits(uint32_t w0, uint32_t w1, float scale, uint32_t (&out)[4]) {
    // v + 0x808080 has the bytes q0, q1 + 128, q2 + 128, q3 + 128
    const uint32_t u0 = (uint32_t)(int)(__uint_as_float(w0 << 16) * scale) + 0x808080u;
    const uint32_t u1 = (uint32_t)(int)(__uint_as_float(w0 & 0xffff0000u) * scale) + 0x808080u;
    const uint32_t u2 = (uint32_t)(int)(__uint_as_float(w1 << 16) * scale) + 0x808080u;
    const uint32_t u3 = (uint32_t)(int)(__uint_as_float(w1 & 0xffff0000u) * scale) + 0x808080u;
    const uint32_t a = __builtin_amdgcn_perm(u1, u0, 0x05010400u), b = __builtin_amdgcn_perm(u1, u0, 0x07030602u);
    const uint32_t c = __builtin_amdgcn_perm(u3, u2, 0x05010400u), e = __builtin_amdgcn_perm(u3, u2, 0x07030602u);
    out[0] = __builtin_amdgcn_perm(e, b, 0x07060302u);
    out[1] = __builtin_amdgcn_perm(e, b, 0x05040100u) ^ 0x80808080u;
    out[2] = __builtin_amdgcn_perm(c, a, 0x07060302u) ^ 0x80808080u;
    out[3] = __builtin_amdgcn_perm(c, a, 0x05040100u) ^ 0x80808080u;
}

// WPR wavefronts per row: rows 0 .. EP-1 are the experts' (their digits are written, in the order in which
// digit_logits_kernel loads them: [32-expert block][32-element step][digit][lane] x 16 bytes), then the tokens'.
// exps[row] = E, parts[row] = A, N2, N3, R (all infinite for a row that holds an infinity or a NaN).
// Rows past the last expert or token repeat it.
// Four wavefronts per row up to kShortRows: bound by the latency of one row's chain (256 experts, d = 7168, one / four per row: 512
// tokens 13.4 / 10.5 us, 1024 13.4 / 10.7; 128 experts, d = 4096, 2048 tokens 11.5 / 10.4).  Beyond, one: bound by reading x and
// the counting, about ten vector instructions per element (256 experts, 4096 tokens 21 / 24 us).
template <int WPR>
__global__ __launch_bounds__(kThreads) void digits_kernel(const uint16_t* __restrict__ x, const uint16_t* __restrict__ wr,
                                                         uint8_t* __restrict__ wdig, int32_t* __restrict__ exps,
                                                         float4* __restrict__ parts, int T, int d, int E, int EP) {
    static_assert(WPR == 1 || WPR == kWavesPerBlock, "a row is one wavefront's or the workgroup's");
    __shared__ uint32_t tops[kWavesPerBlock];
    __shared__ int cnts[kWavesPerBlock][3];
    const int lane = threadIdx.x % kWave, wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x / kWave));
    const int row = WPR == 1 ? (int)blockIdx.x * kWavesPerBlock + wave : (int)blockIdx.x;
    const int sub = WPR == 1 ? 0 : wave;
    const int t = row - EP;
    const bool expert = row < EP;
    const uint16_t* v = expert ? wr + (size_t)(row < E ? row : E - 1) * d : x + (size_t)(t < T ? t : T - 1) * d;
    // A unit is 16 elements: one lane's 16 bytes of every digit.  A lane holds 8 / WPR at a time (all loads in flight at
    // once); rows of up to 8192 elements are read once, longer ones twice.
    constexpr int kHeld = 8 / WPR, kSpan = kWave * WPR;
    const int units = d / 16, chunks = (units + kHeld * kSpan - 1) / (kHeld * kSpan);
    uint32_t held[kHeld][8];
    auto load = [&](int c) {
#pragma unroll
        for (int i = 0; i < kHeld; ++i) {
            const int p0 = (c * kHeld + i) * kSpan + sub * kWave, p = p0 + lane;
            uint4 a = make_uint4(0, 0, 0, 0), b = a;
            if (p0 < units) {                 // uniform; past the end: the first unit again
                const uint4* src = reinterpret_cast<const uint4*>(v + (size_t)(p < units ? p : 0) * 16);
                a = src[0], b = src[1];
            }
            held[i][0] = a.x, held[i][1] = a.y, held[i][2] = a.z, held[i][3] = a.w;
            held[i][4] = b.x, held[i][5] = b.y, held[i][6] = b.z, held[i][7] = b.w;
        }
    };
    uint32_t top = 0;
    for (int c = 0; c < chunks; ++c) {
        load(c);
#pragma unroll
        for (int i = 0; i < kHeld; ++i)
#pragma unroll
            for (int q = 0; q < 8; ++q) {
                const uint32_t lo = held[i][q] & 0x7fffu, hi = (held[i][q] >> 16) & 0x7fffu;
                const uint32_t m = lo > hi ? lo : hi;
                top = m > top ? m : top;
            }
    }
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) {
        const uint32_t o = (uint32_t)__shfl_xor((int)top, off, kWave);
        top = o > top ? o : top;
    }
    if constexpr (WPR > 1) {
        if (lane == 0) tops[wave] = top;
        __syncthreads();
#pragma unroll
        for (int w = 0; w < WPR; ++w) top = tops[w] > top ? tops[w] : top;
    }
    const bool finite = top < 0x7f80u;
    int ex = finite ? (int)(top >> 7) - 127 : 0;
    ex = ex < kMinExp ? kMinExp : ex;
    const float scale = exp2i(29 - ex);
    int n2 = 0, n3 = 0, nr = 0;
    uint8_t* dst = wdig + ((size_t)(row >> 5) * (d / 32) * 4) * 1024 + (row & 31) * 16;
    for (int c = 0; c < chunks; ++c) {
        if (chunks > 1) load(c);
#pragma unroll
        for (int i = 0; i < kHeld; ++i) {
            const int p0 = (c * kHeld + i) * kSpan + sub * kWave, p = p0 + lane;
            if (p0 >= units) continue;        // uniform
            const bool live = p < units;
#pragma unroll
            for (int q = 0; q < 16; ++q) {
                const uint32_t w = live ? held[i][q / 2] : 0u;
                const float f = __uint_as_float(q & 1 ? w & 0xffff0000u : w << 16) * scale;
                const int n = (int)f;
                n2 += __popcll(__ballot((n & 0xffff) != 0));      // wavefront totals, in scalar registers
                n3 += __popcll(__ballot((n & 0xff) != 0));
                nr += __popcll(__ballot((float)n != f));
            }
            if (expert && live) {
                uint32_t g[4][4];
#pragma unroll
                for (int q = 0; q < 4; ++q) four_digits(held[i][2 * q], held[i][2 * q + 1], scale, g[q]);
                uint8_t* out = dst + (size_t)(p >> 1) * 4096 + (p & 1) * 512;
#pragma unroll
                for (int j = 0; j < 4; ++j) *reinterpret_cast<uint4*>(out + j * 1024) = make_uint4(g[0][j], g[1][j], g[2][j], g[3][j]);
            }
        }
    }
    if constexpr (WPR > 1) {
        if (lane == 0) cnts[wave][0] = n2, cnts[wave][1] = n3, cnts[wave][2] = nr;
        __syncthreads();
        n2 = n3 = nr = 0;
#pragma unroll
        for (int w = 0; w < WPR; ++w) n2 += cnts[w][0], n3 += cnts[w][1], nr += cnts[w][2];
    }
    if (lane == 0 && sub == 0) {
        const float unit = exp2i(ex - 29), inf = __builtin_huge_valf();
        exps[row] = ex;
        // parts q2, q3 and q3 alone are at most 2^15 + 2^7 and 2^7 units, a residual is less than one
        parts[row] = finite ? make_float4(__uint_as_float(top << 16), 33000.0f * unit * sqrtf((float)n2), 128.2f * unit * sqrtf((float)n3), unit * (float)nr)
                            : make_float4(inf, inf, inf, inf);
    }
}

// The bound above for a token's and an expert's parts, or for the largest parts of several.
template <class F>
__device__ __forceinline__ F digit_bound(const float4& x, const float4& w) {
    return (F)x.y * (F)w.z + (F)x.z * (F)w.y + (F)x.w * (F)w.x + (F)x.x * (F)w.w;
}

// part[ks][t][e], t < TP, e < EP, fp64.  A workgroup takes 128 tokens x 64 experts, 32 tokens a wavefront: the four read the
// same digits of the experts, three of them from L1 (256 experts side by side on 32 tokens: every wavefront's from L2).
// A lane supplies 16 consecutive k of one row per operand (row lane % 32, half lane / 32 of the 32-element step) and
// receives D[token 8(v/4) + 4(lane/32) + v%4][expert lane%32].  Workgroup b takes slice b % KS of d: with 8 slices (or 4, 16)
// the experts' digits of a slice are read by one XCD (two, two) only and stay in its L2.
// One wavefront per SIMD, software-pipelined by hand: while the 26 matrix instructions of a 32-element step run, the next
// step's tokens are cut into digits (four vector instructions behind each) and the experts' digits of the step after that
// are on their way.
constexpr int kDigitTokens = 128, kDigitExperts = 64;
// A bound up to which a logit is as good as exact for the weights.  Beyond, the selected experts' logits are recomputed in fp64
// token by token, which serves the two gates whose weights hang on them alone.  The softmax over all experts hangs on every logit:
// there a tile beyond the bound is formed in fp64, but only below 2^19 logits, the calls that are all in fp64 without the int8
// form.  Above, the experts that are not selected may carry the digits' error (less than 2^-19 |x| |w|) into the denominator.
// 2^-25: a weight is then off by at most one rounding to fp32 more (2^-24); normal rows stay below 2^-29.
// Router alone, 256 experts, d = 7168, us, normal rows / one channel 1000 times the others / lognormal magnitudes (sigma 1.5): 1024 tokens
// softmax 50 / 95 / 95 (all in fp64 84), renormalised 50 / 72 / 71; 4096 tokens 118 / 160 / 161 (all in fp64 288).  One token of such an
// element among 1024, a router row with a large element, an infinity or a NaN 91 to 95 (4096 tokens: 134, 169 and 295).
constexpr double kCertain = 0x1p-25;
float tile_limit(const moe_config& c) {
    return c.gating == MOE_GATE_SOFTMAX && (long long)c.T * c.E < (1 << 19) ? (float)kCertain : 3e38f;
}
__global__ __launch_bounds__(kThreads) void digit_logits_kernel(const uint16_t* __restrict__ x, const uint8_t* __restrict__ wdig,
                                                               const int32_t* __restrict__ exps, double* __restrict__ part,
                                                               int T, int d, int TP, int EP, int KS, const uint16_t* __restrict__ wr, int E,
                                                               const float4* __restrict__ parts, float4* __restrict__ wmax,
                                                               int32_t* __restrict__ in_fp64, float limit) {
    constexpr int RT = kDigitTokens, TW = RT / 32, BUF = RT * 128, NB = 3;
    __shared__ __attribute__((aligned(1024))) char ring[NB * BUF];
    __shared__ float4 tops[kWavesPerBlock];
    const int tid = threadIdx.x, lane = tid % kWave;
    const int wave = __builtin_amdgcn_readfirstlane(tid / kWave);
    const int li = lane & 31, half = lane >> 5;
    const int EG = EP / kDigitExperts;
    const int ks = blockIdx.x % KS, eg = blockIdx.x / KS % EG, t0 = blockIdx.x / (KS * EG) * RT;
    const int nstep = d / 64, per = (nstep + KS - 1) / KS;
    const int g0 = ks * per, g1 = g0 + per < nstep ? g0 + per : nstep;

    // The largest parts of the tile's tokens (wavefronts 0 and 1) and experts (wavefront 2) decide how its logits are formed.
    static_assert(RT == 2 * kWave && kDigitExperts == kWave, "rows of the tile per wavefront");
    float4 most = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
    if (wave < 3) most = parts[wave < 2 ? EP + t0 + tid : eg * kDigitExperts + lane];
#pragma unroll
    for (int off = 32; off > 0; off >>= 1)
        most = make_float4(fmaxf(most.x, __shfl_xor(most.x, off, kWave)), fmaxf(most.y, __shfl_xor(most.y, off, kWave)),
                           fmaxf(most.z, __shfl_xor(most.z, off, kWave)), fmaxf(most.w, __shfl_xor(most.w, off, kWave)));
    if (lane == 0) tops[wave] = most;
    __syncthreads();
    const float4 a = tops[0], c = tops[1], w = tops[2];
    const float4 xm = make_float4(fmaxf(a.x, c.x), fmaxf(a.y, c.y), fmaxf(a.z, c.z), fmaxf(a.w, c.w));
    const bool fp64 = !(digit_bound<float>(xm, w) <= limit);     // written so that a NaN (infinity times zero) counts
    if (ks == 0 && tid == 0) {
        in_fp64[t0 / RT * EG + eg] = fp64;
        if (t0 == 0) wmax[eg] = w;
    }
    if (fp64) {
        const int i = lane & 15, g = lane >> 4, tw = t0 + wave * 32;
        const uint16_t *xp[2], *ep[4];
#pragma unroll
        for (int m = 0; m < 2; ++m) xp[m] = x + (size_t)(tw + m * 16 + i < T ? tw + m * 16 + i : T - 1) * d + g * 8;
#pragma unroll
        for (int n = 0; n < 4; ++n) ep[n] = wr + (size_t)((eg * 4 + n) * 16 + i < E ? (eg * 4 + n) * 16 + i : E - 1) * d + g * 8;
        f64x4 z[2][4];
        fp64_tiles(xp, ep, g0 * (64 / kChunk), g1 * (64 / kChunk), z);
#pragma unroll
        for (int m = 0; m < 2; ++m)
#pragma unroll
            for (int n = 0; n < 4; ++n)
#pragma unroll
                for (int v = 0; v < 4; ++v) part[((size_t)ks * TP + tw + m * 16 + g + 4 * v) * EP + (eg * 4 + n) * 16 + i] = z[m][n][v];
        return;
    }

    uint32_t xo[TW];   // byte offsets of this lane's pieces: 8 rows x 128 bytes per load, source chunk swizzled
#pragma unroll
    for (int q = 0; q < TW; ++q) {
        const int rg = q * 4 + wave, t = t0 + rg * 8 + (lane >> 3);
        xo[q] = (uint32_t)((lane & 7) ^ (((lane >> 3) ^ rg) & 7)) * 16u + (uint32_t)(t < T ? t : T - 1) * (uint32_t)d * 2u;
    }
    const uint32_t x_dst = (uint32_t)(uintptr_t)ring + wave * 1024;
    auto load_x = [&](int g) {   // steps past the last re-read it (harmless)
        const char* xb = reinterpret_cast<const char*>(x) + (size_t)(g < g1 ? g : g1 - 1) * 128;
        const uint32_t buf = (uint32_t)((g - g0) % NB) * BUF;
#pragma unroll
        for (int q = 0; q < TW; ++q) lds_dma16_at<false>(xb, xo[q], x_dst + buf + q * 4096);
    };
    const uint32_t eb_bytes = (uint32_t)(d / 32) * 4096u;
    const uint8_t* wp = wdig + (size_t)eg * 2 * eb_bytes;        // uniform
    const uint32_t wl[2] = {(uint32_t)lane * 16u, eb_bytes + (uint32_t)lane * 16u};
    const int r = wave * 32 + li, xsw = (r ^ (r >> 3)) & 7;
    const char* xrow = ring + r * 128;
    const float xscale = exp2i(29 - exps[EP + t0 + r]);

    i32x16 acc[5][2];
#pragma unroll
    for (int o = 0; o < 5; ++o)
#pragma unroll
        for (int b = 0; b < 2; ++b)
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[o][b][v] = 0;
    if (g0 < g1) {
        i32x4 wq[2][2][4], xq[2][4];   // [parity of the 32-element step][expert block][digit]
        uint32_t raw[8], u[4];
        auto load_w = [&](int step, int par, int i) {
            const uint8_t* base = wp + (size_t)(step < 2 * g1 ? step : 2 * g1 - 1) * 4096;
            wq[par][i / 4][i % 4] = *reinterpret_cast<const i32x4*>(base + wl[i / 4] + i % 4 * 1024);
        };
        auto read_x = [&](int g, int s, int i) {   // half s of step g: 32 bytes of this lane's row, in two pieces
            const uint4 v = *reinterpret_cast<const uint4*>(xrow + (g - g0) % NB * BUF + ((4 * s + 2 * half + i) ^ xsw) * 16);
            raw[4 * i] = v.x, raw[4 * i + 1] = v.y, raw[4 * i + 2] = v.z, raw[4 * i + 3] = v.w;
        };
        // Sixteenth n of cutting `raw` into digits (four_digits, in pieces that fit behind one matrix instruction).
        auto cut = [&](int n, int par) {
            const int i = n / 4;
            if (n % 4 < 2) {
                const uint32_t w = raw[2 * i + n % 4];
                u[2 * (n % 4)] = (uint32_t)(int)(__uint_as_float(w << 16) * xscale) + 0x808080u;
                u[2 * (n % 4) + 1] = (uint32_t)(int)(__uint_as_float(w & 0xffff0000u) * xscale) + 0x808080u;
            } else if (n % 4 == 2) {
                const uint32_t b = __builtin_amdgcn_perm(u[1], u[0], 0x07030602u), e = __builtin_amdgcn_perm(u[3], u[2], 0x07030602u);
                xq[par][0][i] = (int)__builtin_amdgcn_perm(e, b, 0x07060302u);
                xq[par][1][i] = (int)(__builtin_amdgcn_perm(e, b, 0x05040100u) ^ 0x80808080u);
            } else {
                const uint32_t a = __builtin_amdgcn_perm(u[1], u[0], 0x05010400u), c = __builtin_amdgcn_perm(u[3], u[2], 0x05010400u);
                xq[par][2][i] = (int)(__builtin_amdgcn_perm(c, a, 0x07060302u) ^ 0x80808080u);
                xq[par][3][i] = (int)(__builtin_amdgcn_perm(c, a, 0x05040100u) ^ 0x80808080u);
            }
        };
        // The 26 matrix instructions of half s of step g; behind each its share of what the next half needs.
        auto half_step = [&](int g, int s) {
            constexpr int P[13] = {0, 1, 0, 1, 2, 0, 1, 2, 3, 0, 1, 2, 3}, O[13] = {3, 3, 2, 2, 2, 1, 1, 1, 1, 0, 0, 0, 0};
#pragma unroll
            for (int i = 0; i < 26; ++i) {
                const int p = P[i / 2], q = O[i / 2], b = i % 2;
                acc[p + q][b] = __builtin_amdgcn_mfma_i32_32x32x32_i8(xq[s][p], wq[s][b][q], acc[p + q][b], 0, 0, 0);
                // an expert digit's registers take the digit of two halves on as soon as their last product is issued
                if (b == 1 && (i == 25 || O[i / 2 + 1 < 13 ? i / 2 + 1 : 12] != q)) {
                    load_w(2 * g + s + 2, s, q);
                    load_w(2 * g + s + 2, s, 4 + q);
                }
                if (i < 2) read_x(g + s, s ^ 1, i);      // (the step past the last: a copy of the last, its digits are not used)
                if (i >= 5 && i < 21) cut(i - 5, s ^ 1);
                __builtin_amdgcn_sched_barrier(0);
            }
        };
        load_x(g0);
        load_x(g0 + 1);
#pragma unroll
        for (int i = 0; i < 8; ++i) load_w(2 * g0, 0, i), load_w(2 * g0 + 1, 1, i);
        wait_vmcnt<0>();
        __syncthreads();
#pragma unroll
        for (int i = 0; i < 2; ++i) read_x(g0, 0, i);
#pragma unroll
        for (int n = 0; n < 16; ++n) cut(n, 0);
        for (int g = g0; g < g1; ++g) {
            __builtin_amdgcn_sched_barrier(0);
            half_step(g, 0);
            // The next half reads step g + 1's tokens, which all four wavefronts brought in: each waits for its own (requested a whole
            // step ago, newer are the eight digit loads of each of two halves), then for the others.
            wait_vmcnt<16>();
            __syncthreads();
            load_x(g + 2);           // its buffer was last read in the first half of step g - 1, a barrier ago
            __builtin_amdgcn_sched_barrier(0);
            half_step(g, 1);
        }
        wait_vmcnt<0>();             // nothing of this workgroup may still be writing LDS when it retires
    }
#pragma unroll
    for (int b = 0; b < 2; ++b) {
        const int e = (eg * 2 + b) * 32 + li;
        const int ew = exps[e];
        const int tr = t0 + wave * 32 + 4 * half;
        double* out = part + ((size_t)ks * TP + tr) * EP + e;
#pragma unroll
        for (int v = 0; v < 16; ++v) {
            const int row = 8 * (v / 4) + v % 4;
            const long long e2 = 1023 + exps[EP + tr + row] + ew - 42;     // 2^(Ex-29) 2^(Ew-29) 2^16
            double z = (double)acc[0][b][v];
#pragma unroll
            for (int o = 1; o < 5; ++o) z = fma(z, 256.0, (double)acc[o][b][v]);
            out[(size_t)row * EP] = z * __longlong_as_double(e2 << 52);
        }
    }
}

// ---- gate + top-k of one token by one wavefront ---------------------------------------------
// Lane l holds the logits of experts l, l+64, ... in z[] (ok[] = expert exists).  Eq. 1-2,
// Sec. 3.4: max-subtracted softmax (or sigmoid), k rounds of arg-max over the logits with the
// winners masked, ties to the lower index.
// moe_forward's down projection counts, per (token, 128-feature group), how many of the token's
// k expert rows have been written (see ffn_kernels.hpp, fused_combine).  The counters of token t
// are cleared here by the wavefront that routes t, so the layer needs no clearing launch.
__device__ __forceinline__ void zero_token_counters(int32_t* __restrict__ zero, int zero_n, int t, int lane) {
    if (zero == nullptr) return;
    for (int i = lane; i < zero_n; i += kWave) zero[(size_t)t * zero_n + i] = 0;
}

// Largest value over the wavefront, the same in every lane: four exchanges inside rows of 16 lanes (DPP, no LDS
// crossbar), then the four rows' values through scalar registers.
__device__ __forceinline__ double wave_max_uniform(double v) {
    auto exchanged = [](double a, auto ctrl) {
        const uint64_t u = (uint64_t)__double_as_longlong(a);
        const uint32_t lo = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)(uint32_t)u, decltype(ctrl)::value, 0xf, 0xf, true);
        const uint32_t hi = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)(uint32_t)(u >> 32), decltype(ctrl)::value, 0xf, 0xf, true);
        return __longlong_as_double((long long)((uint64_t)hi << 32 | lo));
    };
    v = fmax(v, exchanged(v, std::integral_constant<int, 0xB1>{}));     // quad_perm 1,0,3,2
    v = fmax(v, exchanged(v, std::integral_constant<int, 0x4E>{}));     // quad_perm 2,3,0,1
    v = fmax(v, exchanged(v, std::integral_constant<int, 0x141>{}));    // row_half_mirror
    v = fmax(v, exchanged(v, std::integral_constant<int, 0x140>{}));    // row_mirror
    auto lane_value = [&](int l) {
        const uint64_t u = (uint64_t)__double_as_longlong(v);
        return __longlong_as_double((long long)((uint64_t)(uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(u >> 32), l) << 32 |
                                                (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)u, l)));
    };
    return fmax(fmax(lane_value(0), lane_value(16)), fmax(lane_value(32), lane_value(48)));
}

// The largest logit of those not taken and its expert (ties to the lower index); expert -1 if every expert is taken.
// Uniform over the wavefront.
template <int Q>
__device__ __forceinline__ double next_best(const double (&z)[Q], const bool (&ok)[Q], unsigned taken, int lane, int& expert) {
    double bv = -__builtin_huge_val();
    int be = -1;
#pragma unroll
    for (int q = 0; q < Q; ++q) {
        if (ok[q] && !((taken >> q) & 1u) && (be < 0 || z[q] > bv)) {
            bv = z[q];
            be = lane + kWave * q;
        }
    }
    const double m = wave_max_uniform(bv);
    const unsigned long long tied = __ballot(be >= 0 && bv == m);
    expert = tied != 0 ? __builtin_amdgcn_readlane(be, __builtin_ctzll(tied)) : -1;
    if ((tied & (tied - 1)) != 0) {      // equal logits: a lane holds the first of its own, the lowest row of 64 goes first
        expert = -1;
#pragma unroll
        for (int q = 0; q < Q; ++q) {
            const unsigned long long row = __ballot(be >= 0 && bv == m && be / kWave == q);
            if (expert < 0 && row != 0) expert = kWave * q + __builtin_ctzll(row);
        }
    }
    return m;
}

// Gate and selection of one token.  Q: logits per lane that can exist (E <= 64 Q): the exponentials and compares of the others
// are left out.  `suspect` is called with (k-th largest logit, smallest distance between two neighbours among the k + 1
// largest); if it returns true it has replaced logits in z and the selection starts over (once).
template <int Q, class Suspect>
__device__ __forceinline__ void gate_and_select(double (&z)[Q], const bool (&ok)[Q],
                                                int lane, int wave, int t, int k, int E, int gating,
                                                double (*wsel)[kMaxExperts], int32_t (*sel_idx)[kMaxExperts],
                                                int32_t* __restrict__ topk_idx, float* __restrict__ topk_w, Suspect&& suspect) {
    const double ninf = -__builtin_huge_val();
    for (bool again = true; again;) {
#pragma unroll
        for (int q = 0; q < Q; ++q) z[q] = (z[q] != z[q]) ? ninf : z[q];   // a NaN logit can never win and never breaks the index range
        unsigned taken = 0;   // bit q set: this lane's q-th expert already selected
        double last = __builtin_huge_val(), gap = __builtin_huge_val();
        for (int r = 0; r < k; ++r) {
            int be;
            const double m = next_best(z, ok, taken, lane, be);
            const double step = last - m;
            if (r > 0 && step < gap) gap = step;      // not for two infinities (a NaN): only a bias makes them, they are equal
            last = m;
            if (lane == be % kWave) taken |= 1u << (be / kWave);
            if (lane == 0) sel_idx[wave][r] = be;
        }
        again = suspect(last, gap, taken);
    }
    double m = ninf;
#pragma unroll
    for (int q = 0; q < Q; ++q) m = fmax(m, z[q]);
    m = wave_max_uniform(m);
    double p[Q], psum = 0.0;
#pragma unroll
    for (int q = 0; q < Q; ++q) {
        if (gating == MOE_GATE_SIGMOID_NORM)
            p[q] = ok[q] ? 1.0 / (1.0 + exp(-z[q])) : 0.0;
        else
            p[q] = ok[q] ? exp(z[q] - m) : 0.0;
        psum += p[q];
    }
    if (gating != MOE_GATE_SIGMOID_NORM) {
        const double inv = 1.0 / wave_sum(psum);
#pragma unroll
        for (int q = 0; q < Q; ++q) p[q] = ok[q] ? p[q] * inv : 0.0;   // softmax scores, Eq. 1
    }
    __builtin_amdgcn_wave_barrier();
    double wsum = 0.0;
    for (int r = 0; r < k; ++r) {
        const int be = __builtin_amdgcn_readfirstlane(*(volatile int32_t*)&sel_idx[wave][r]);
        const int oq = be / kWave, ol = be % kWave;
        double mine = 0.0;
#pragma unroll
        for (int q = 0; q < Q; ++q) mine = (q == oq) ? p[q] : mine;
        const uint64_t u = (uint64_t)__double_as_longlong(mine);
        const double wv = __longlong_as_double((long long)((uint64_t)(uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(u >> 32), ol) << 32 |
                                                           (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)u, ol)));
        wsum += wv;
        if (lane == 0) wsel[wave][r] = wv;
    }
    const double scale = (gating == MOE_GATE_SOFTMAX) ? 1.0 : 1.0 / wsum;
    __builtin_amdgcn_wave_barrier();
    for (int i = lane; i < k; i += kWave) {
        topk_idx[(size_t)t * k + i] = *(volatile int32_t*)&sel_idx[wave][i];
        topk_w[(size_t)t * k + i] = (float)(*(volatile double*)&wsel[wave][i] * scale);
    }
}

// The logits of the experts that can be among the k largest, recomputed in fp64 (bf16 operands and their products are
// exact there; the order of the additions moves the sum by ~1e-15), plus the bias: for tokens whose k + 1 largest logits
// hold neighbours closer than the error of digit_logits_kernel can rule on.  vk: the k-th largest value in z; margin[q]: the
// largest error bound b of z plus the bound b_q of the lane's q-th logit, or less than zero if that one is not off at all.
// Why this is enough: the k experts with the largest z have true logits >= vk - b, so the true k-th largest logit is
// >= vk - b, every expert of the true top-k has z >= vk - b - b_q: it is a candidate, or z is its true logit.  Every other
// expert's value is < vk - b, i.e. lies below those k, also when it keeps its place in z: the selection over the mixed
// array picks the same experts in the same order as over exact logits.
// cand_list: LDS, kMaxExperts ints per wavefront.
template <int Q>
__device__ __forceinline__ void refine_candidates(double (&z)[Q], const bool (&ok)[Q],
                                                  int lane, int t, double vk, const double (&margin)[Q], int d,
                                                  const uint16_t* __restrict__ x, const uint16_t* __restrict__ wr,
                                                  const float* __restrict__ bias, int32_t* cand_list) {
    // Candidates recomputed per pass over the token row.  8 or 12 where there are more than four save passes, but take 160 or 200
    // registers instead of 126 (256 experts, d = 7168, 4096 tokens, rows of heavy tails 161 / 166 / 172 us, normal rows 118 / 122 / 122).
    constexpr int CB = 4;
    const uint16_t* xr = x + (size_t)t * d;
    // candidate list (ascending expert index inside each q; the order does not matter)
    int n_cand = 0;
#pragma unroll
    for (int q = 0; q < Q; ++q) {
        // -infinity is a bias's, it stays
        const bool c = ok[q] && margin[q] >= 0.0 && z[q] >= vk - margin[q] && z[q] != -__builtin_huge_val();
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
// DIGITS: `part` holds the slices of digit_logits_kernel; parts, wmax and in_fp64 say how far off they can be.
// T16, E16: padded tokens and experts in units of 16.
template <bool DIGITS, int Q>
__global__ __launch_bounds__(kThreads) void topk_kernel(const double* __restrict__ part,
                                                       const float* __restrict__ bias,
                                                       int32_t* __restrict__ topk_idx, float* __restrict__ topk_w,
                                                       int T, int E, int k, int gating, int T16, int E16, int KS,
                                                       int32_t* __restrict__ zero, int zero_n,
                                                       const uint16_t* __restrict__ x, const uint16_t* __restrict__ wr,
                                                       int d, const float4* __restrict__ parts, const float4* __restrict__ wmax,
                                                       const int32_t* __restrict__ in_fp64) {
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
        z[q] = (ok[q] && bias) ? (double)bias[e] : 0.0;
    }
    for (int s0 = 0; s0 < KS; s0 += 8) {   // slices in fixed order; 8 Q independent loads at a time
        double tmp[Q][8];
#pragma unroll
        for (int q = 0; q < Q; ++q)
#pragma unroll
            for (int u = 0; u < 8; ++u)
                tmp[q][u] = (ok[q] && s0 + u < KS) ? part[((size_t)(s0 + u) * T16 * 16 + t) * EP + lane + kWave * q] : 0.0;
#pragma unroll
        for (int q = 0; q < Q; ++q)
#pragma unroll
            for (int u = 0; u < 8; ++u) z[q] += tmp[q][u];
    }
#pragma unroll
    for (int q = 0; q < Q; ++q) z[q] = ok[q] ? z[q] : ninf;
    bool refined = !DIGITS;
    gate_and_select(z, ok, lane, wave, t, k, E, gating, wsel, sel_idx, topk_idx, topk_w, [&](double vk, double gap, unsigned taken) {
        if (refined) return false;
        refined = true;
        const float4 n = parts[EP + t];
        const int EG = (int)(EP / kDigitExperts);
        static_assert(kDigitExperts == kWave, "a lane's q-th logit is of the q-th group of experts");
        double b = 0.0, margin[Q], round = 0.0;
#pragma unroll
        for (int q = 0; q < Q; ++q) {
            margin[q] = -1.0;
            if (q < EG && !in_fp64[t / kDigitTokens * EG + q]) {
                const float4 w = wmax[q];
                margin[q] = digit_bound<double>(n, w);
                b = fmax(b, margin[q]);
                round = fmax(round, (double)n.x * w.x);
            }
        }
        if (b == 0.0) return false;    // nothing was left out (a row of zeros, of few bits): equal logits are equal
        round *= 0x1p-53 * d * (d / 64 + 32);        // of the fp64 sums on either side
#pragma unroll
        for (int q = 0; q < Q; ++q) margin[q] = margin[q] > 0.0 ? 1.01 * (b + margin[q]) + 2.0 * round : -1.0;
        if (k < E) {
            int be;
            const double step = vk - next_best(z, ok, taken, lane, be);
            if (step < gap) gap = step;
        }
        if (b <= kCertain && gap > 2.02 * b + 2.0 * round) return false;
        refine_candidates(z, ok, lane, t, vk, margin, d, x, wr, bias, sel_idx[wave]);
        return true;
    });
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
    gate_and_select(z, ok, lane, 0, t, k, E, gating, wsel, sel_idx, topk_idx, topk_w, [](double, double, unsigned) { return false; });
}

// Where the int8 form pays: from about 6e8 multiply-adds on, for at least 32 experts (it pads them to a multiple of 64).  Router
// alone, us, fp64 / int8: 256 experts (d 7168) 256 tokens (4.7e8) 35 / 38, 512 51 / 43, 1024 83 / 48, 2048 149 / 68, 4096
// 286 / 117; 160 (5120) 1024 tokens 52 / 40; 128 (4096) 1024 tokens (5.4e8) 34 / 35, 1500 44 / 34, 4096 89 / 50; 64 (3584)
// 2048 tokens (4.7e8) 33 / 34, 3000 44 / 37, 4096 49 / 42; 32 (4096) 4096 tokens (5.4e8) 38 / 40, 8192 69 / 61; 16 (4096)
// 8192 tokens 40 / 62.  The line is a mean: the fp64 form's time goes in steps, with the rounds of its wavefronts and its groups of 64
// experts, and where one is just begun the int8 form is ahead earlier (160 experts (5120) 384 tokens, 3.1e8, 38 / 31; 65 (2048) 4096
// tokens, 5.5e8, 50 / 37; 48 (4096) 2048 tokens, 4.0e8, 33 / 30).
// And from 36000 logits on, which tells from d = 16384 up: on longer rows the experts' digits, written at 6 bytes an element, are the
// larger part.  d = 32768, fp64 / int8: 256 experts 128 tokens (32768) 69 / 84, 192 118 / 88; 160 129 tokens 64 / 75, 256 100 / 77; 128
// 256 tokens 66 / 68, 384 115 / 71; 64 512 tokens 67 / 68, 800 115 / 76; 32 1000 tokens 67 / 81, 2000 137 / 105.
// Error of the weights against float64 in every one of these: the same four digits (2.5e-8) in both forms.
// The three launches of the int8 form take about 10 us (digits), 14 + 1 a step (products) and 11 (selection), of which 5 each
// are a launch's own.
bool digits_pay(const moe_config& c) {
    const double logits = (double)c.T * c.E;
    return c.E >= 32 && logits * c.d > 6e8 && logits > 36000.0;
}

struct RoutePlan {
    int T16, E16, KS, NT;
    bool digits;        // logits on the int8 matrix cores
    int TP, EP;         // digits: padded tokens and experts
};

size_t digit_bytes(const RoutePlan& p, int d) {
    const size_t groups = p.EP / kDigitExperts;
    return (size_t)p.KS * p.TP * p.EP * sizeof(double) + (size_t)p.EP * d * 4 + (size_t)(p.EP + p.TP) * (sizeof(float4) + sizeof(int32_t)) +
           groups * (sizeof(float4) + p.TP / kDigitTokens * sizeof(int32_t));
}

// mode: the test knob's value.  -1 the rule, 1 every logit in fp64, 0 the int8 form from 256 tokens on.
RoutePlan plan(const moe_config& c, int mode) {
    RoutePlan p{};
    // 32-bit byte offsets hold: every entry point refuses T d 2 >= 2^32 bytes.
    p.digits = mode != 1 && c.E > 8 && c.d <= kMaxDigitDim && (mode == 0 ? c.T >= 256 : digits_pay(c));
    if (p.digits) {
        p.EP = (c.E + kDigitExperts - 1) / kDigitExperts * kDigitExperts;
        p.TP = (c.T + kDigitTokens - 1) / kDigitTokens * kDigitTokens;
        const int nstep = c.d / 64;
        const long long tiles = (long long)(p.TP / kDigitTokens) * (p.EP / kDigitExperts);
        // Slices: rounds of workgroups x steps of each (a quarter more where a slice of the experts' digits fills an XCD's L2),
        // a workgroup's start and end worth eight steps, and the slices' sum.
        double best = 1e30;
        for (int ks = 1; ks <= kMaxDigitSlices && ks <= nstep; ks *= 2) {
            const int steps = (nstep + ks - 1) / ks;
            if (steps > kMaxDigitSlice / 64) continue;
            const double slow = (double)p.EP * 256 * steps > 2e6 ? 1.25 : 1.0;
            const double cost = (double)((tiles * ks + 255) / 256) * (slow * steps + 8.0) + 0.3 * ks;
            if (cost < best) {
                best = cost;
                p.KS = ks;
            }
        }
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
    // for the rule's form and, if the test knob forces one, for that
    size_t need = 0;
    for (const int mode : {-1, knob(kKnobRouteExact)}) {
        const RoutePlan p = plan(c, mode);
        const size_t bytes = p.digits ? digit_bytes(p, c.d)
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
    const dim3 topk_grid((c.T + kWavesPerBlock - 1) / kWavesPerBlock);
    if (p.digits) {
        double* part = (double*)workspace;
        float4* parts = (float4*)(part + (size_t)p.KS * p.TP * p.EP);
        float4* wmax = parts + p.EP + p.TP;
        int32_t* exps = (int32_t*)(wmax + p.EP / kDigitExperts);
        uint8_t* wdig = (uint8_t*)(exps + p.EP + p.TP);      // 16-byte aligned: EP and TP are multiples of 32
        int32_t* in_fp64 = (int32_t*)(wdig + (size_t)p.EP * c.d * 4);
        const int rows = p.EP + p.TP;
        if (rows <= kShortRows)
            hipLaunchKernelGGL(digits_kernel<kWavesPerBlock>, dim3(rows), dim3(kThreads), 0, s, x, wr, wdig, exps, parts, c.T, c.d, c.E, p.EP);
        else
            hipLaunchKernelGGL(digits_kernel<1>, dim3(rows / kWavesPerBlock), dim3(kThreads), 0, s, x, wr, wdig, exps, parts, c.T, c.d, c.E, p.EP);
        hipLaunchKernelGGL(digit_logits_kernel, dim3(p.TP / kDigitTokens * (p.EP / kDigitExperts) * p.KS), dim3(kThreads), 0, s, x, wdig, exps,
                           part, c.T, c.d, p.TP, p.EP, p.KS, wr, c.E, parts, wmax, in_fp64, tile_limit(c));
        auto select = [&](auto kern) {
            hipLaunchKernelGGL(kern, topk_grid, dim3(kThreads), 0, s, part, bias, topk_idx, topk_w, c.T, c.E, c.k, c.gating, p.TP / 16,
                               p.EP / 16, p.KS, zero, zero_per_token, x, wr, c.d, parts, wmax, in_fp64);
        };
        if (c.E <= 64) select(topk_kernel<true, 1>);
        else if (c.E <= 128) select(topk_kernel<true, 2>);
        else select(topk_kernel<true, 4>);
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
        hipLaunchKernelGGL(kern, topk_grid, dim3(kThreads), 0, s, part, bias, topk_idx,
                           topk_w, c.T, c.E, c.k, c.gating, p.T16, p.E16, p.KS, zero, zero_per_token, nullptr, nullptr, 0, nullptr, nullptr, nullptr);
    };
    if (c.E <= 64) select(topk_kernel<false, 1>);
    else if (c.E <= 128) select(topk_kernel<false, 2>);
    else select(topk_kernel<false, 4>);
    return hipGetLastError();
}

}  // namespace moe

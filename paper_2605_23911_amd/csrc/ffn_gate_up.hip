// Fused gate+up grouped GEMM launcher: h = SiLU(x W_gate^T) (.) (x W_up^T)  (Sec. 3.3, Eq. 4).
#include "ffn_kernels.hpp"

namespace moe {

namespace {

// {tallest block, packed?, launcher, kernel template instance as rocprofv3 prints it}.
// tile_kernel<IB, gateup>: row-major weights,
// tile_kernel_mixed<IB, gateup, packed, NT weights for single-block experts, two workgroups per CU>.
const Variant kGateUp[] = {
    /*0*/ {256, false, launch_rows<1, true>, "tile_kernel<1, true>"},
    /*1*/ {256, true, launch_tile_mixed<1, true, true, true>, "tile_kernel_mixed<1, true, true, true, false>"},
    /*2*/ {128, true, launch_tile_mixed<1, true, true, true, true>, "tile_kernel_mixed<1, true, true, true, true>"},
};
constexpr int kNumGateUp = sizeof(kGateUp) / sizeof(kGateUp[0]);
// The same with the permutation inside (routed_tile_kernel_mixed); none for row-major weights.
const launch_fn kRouted[kNumGateUp] = {nullptr, launch_routed_mixed, launch_routed_mixed_half};

// Packed weights: one kernel for every schedule and every routing distribution (built a second
// time for two workgroups per CU, see two_workgroups_per_cu).  It picks the
// body per block from the rows the block holds and the regime per block from the rows its expert
// holds (tile_kernel_mixed).  Row-major weights: the same choices, weights through LDS (rows_body).
int pick(int M, bool packed, const moe_config& c) {
    if (!packed) return 0;
    return (M <= 128 && two_workgroups_per_cu(c)) ? 2 : 1;
}

}  // namespace

// Every workgroup pays for the sort (about a microsecond, more with more slots), the launch that it saves is paid for once: up to
// 512 rows, and up to 1024 where a second workgroup on the CU works meanwhile or there is one round of workgroups only.
// Layer, us, in a launch of its own / inside: 8 experts of 256 x 512, 64 tokens (128 rows) 26.3 / 22.2, 512 tokens 34.5 / 30.3;
// Mixtral shape 1 token 119.5 / 116.3, 47 tokens 438.3 / 436.6, 256 (512 rows) 484.6 / 482.2, 400 514.0 / 516.7, 512 541.7 / 546.2;
// two workgroups per CU: Qwen2-MoE shape 1 token 94.8 / 91.5, 100 (800 rows) 550.8 / 548.4, 128 558.5 / 555.5, 256 experts
// (DeepSeek-V3 widths) 128 (1024) 3240 / 3236; 32 experts of 2880 x 2880 128 (512 rows) 273.7 / 273.7, 256 314.0 / 316.4.
// Not for row-major weights (Mixtral shape 128 tokens 465 / 472, Qwen2-MoE shape 32 tokens 556 / 567).
bool permutes_inside(const moe_config& c, bool packed) {
    const long long R = (long long)c.T * c.k;
    if (!packed || R > kSmallRows || knob(kKnobSmallPermute) == 0) return false;
    const long long groups = (long long)((c.F + 127) / 128) * (R < c.E ? R : c.E);
    return R <= 512 || two_workgroups_per_cu(c) || groups <= 256 || knob(kKnobSmallPermute) == 1;
}

const char* gate_up_variant_name(const moe_config& c, int32_t M, bool packed) {
    int id = forced_variant(kKnobGateUpVariant, kNumGateUp, M, packed, kGateUp);
    if (id < 0) id = pick(M, packed, c);
    return kGateUp[id].name;
}

namespace {

hipError_t launch(GemmArgs& a, const moe_config& c, int32_t M, const uint16_t* x_rows, int32_t ldx, const int32_t* src_of, int32_t ldh,
                  const int32_t* offsets, const int32_t* blocks, const int32_t* num_blocks, const int32_t* num_heavy, const uint16_t* wg, const uint16_t* wu,
                  const uint16_t* packed_gu, uint16_t* h, hipStream_t s) {
    a.X = x_rows;
    a.src = src_of;
    a.src_k = c.k;
    a.x_rows = src_of ? c.T : c.T * c.k;
    a.ldx = ldx;
    a.ldo = ldh;
    a.rot_mul = rot_steps(false);
    a.rot_mul_multi = rot_steps(true);
    a.W0 = wg;
    a.W1 = wu;
    a.P = packed_gu;
    a.Out = h;
    a.offsets = offsets;
    a.blocks = blocks;
    a.num_blocks = num_blocks;
    a.num_multi = num_heavy;
    a.R = c.T * c.k;
    a.N = c.F;
    a.K = c.d;
    a.E = c.E;
    a.M = M;
    // token rows are addressed with 32-bit byte offsets from the buffer's base
    if ((unsigned long long)a.x_rows * (unsigned long long)ldx * 2ull >= (1ull << 32)) return hipErrorInvalidValue;
    const bool packed = packed_gu != nullptr;
    int id = forced_variant(kKnobGateUpVariant, kNumGateUp, M, packed, kGateUp);
    if (id < 0) id = pick(M, packed, c);
    if (kGateUp[id].M < M) return hipErrorInvalidValue;
    return (a.topk_idx ? kRouted[id] : kGateUp[id].fn)(a, moe_max_blocks(&c, M), s);
}

}  // namespace

hipError_t launch_gate_up(const moe_config& c, int32_t M, const uint16_t* x_rows, int32_t ldx, const int32_t* src_of,
                          int32_t ldh, const int32_t* offsets,
                          const int32_t* blocks, const int32_t* num_blocks, const int32_t* num_heavy, const uint16_t* wg,
                          const uint16_t* wu, const uint16_t* packed_gu, uint16_t* h, hipStream_t s) {
    GemmArgs a{};
    return launch(a, c, M, x_rows, ldx, src_of, ldh, offsets, blocks, num_blocks, num_heavy, wg, wu, packed_gu, h, s);
}

hipError_t launch_routed_gate_up(const moe_config& c, int32_t M, const uint16_t* x, const int32_t* topk_idx, const PermuteOut& out,
                                 const uint16_t* wg, const uint16_t* wu, const uint16_t* packed_gu, uint16_t* h, hipStream_t s) {
    if (c.T * c.k > kSmallRows || M < 32 || packed_gu == nullptr) return hipErrorInvalidValue;
    GemmArgs a{};
    a.topk_idx = topk_idx;
    a.perm = out;
    return launch(a, c, M, x, c.d, out.src_of, c.F, out.offsets, out.blocks, out.num_blocks, out.num_heavy, wg, wu, packed_gu, h, s);
}

}  // namespace moe

// Down-projection grouped GEMM launcher: y_perm = h W_down^T  (Sec. 3.2, Eq. 4).
#include "ffn_kernels.hpp"

namespace moe {

namespace {

// See the gate+up table for the template parameters; skinny_kernel<JB, gateup, STAGES, SPLITK, packed>.
const Variant kDown[] = {
    /*0*/ {256, false, launch_rows<1, false>, "tile_kernel<1, false>"},
    /*1*/ {32, false, launch_skinny<1, false, 4, 4, false>, "skinny_kernel<1, false, 4, 4, false>"},
    /*2*/ {64, false, launch_skinny<2, false, 4, 4, false>, "skinny_kernel<2, false, 4, 4, false>"},
    /*3*/ {32, true, launch_skinny<1, false, 4, 4, true>, "skinny_kernel<1, false, 4, 4, true>"},
    /*4*/ {64, true, launch_skinny<2, false, 4, 4, true>, "skinny_kernel<2, false, 4, 4, true>"},
    /*5*/ {256, true, launch_tile_mixed<1, false, true, true>, "tile_kernel_mixed<1, false, true, true, false>"},
    /*6*/ {256, true, launch_down_mixed_wide_nt, "tile_kernel_mixed<2, false, true, true, false>"},
    /*7*/ {256, true, launch_down_mixed_wide, "tile_kernel_mixed<2, false, true, false, false>"},
    /*8*/ {128, true, launch_tile_mixed<1, false, true, true, true>, "tile_kernel_mixed<1, false, true, true, true>"},
    /*9*/ {256, false, launch_down_rows_wide, "tile_kernel<2, false>"},    // as 10; only tests force it
    /*10*/ {256, false, launch_down_rows_wide, "tile_kernel<2, false>"},
};
constexpr int kNumDown = sizeof(kDown) / sizeof(kDown[0]);

// few_rows: the projection has too few output rows to give every CU a workgroup (T = 1 on an
// 8-expert model: 2 experts x 4096 output rows = 64 workgroups of 128 rows), so the skinny
// kernel splits K over its four wavefronts.  wide: two 32-row weight blocks per wavefront when
// that still leaves >= 512 workgroups: every token fragment read from LDS then feeds twice as
// many MFMAs and the token tile is re-read from L2 half as often per weight byte (DeepSeek-V3
// shape: 2048-long rows, 256 experts; any shape once experts hold several 256-row blocks).
int pick(int M, bool packed, const moe_config& c) {
    const long long R = (long long)c.T * c.k;
    const long long active = c.E < R ? c.E : R;
    const bool few_rows = (long long)(c.d / 128) * active < 256;
    const bool wide = (long long)(c.d / 256) * (active + R / 256) >= 512;
    if (few_rows && M <= 32) return packed ? 3 : 1;
    if (few_rows && M <= 64) return packed ? 4 : 2;
    if (packed && M <= 128 && two_workgroups_per_cu(c)) return 8;
    // Per-block regime selection (tile_kernel_mixed, tile_kernel).  The line between one weight block and two for row-major weights:
    const bool once = (double)R / c.E <= 192.0 && (double)R * c.d * 2.0 <= 128e6;
    // Row-major, up to the line: one block and, where that leaves 512 workgroups, two: 256 experts, 512 tokens 1330 against 1240 us.  Beyond the line, one weight block
    // (0, three ring buffers or more at any height) against two (10): from 256 rows per expert on 10 is ahead (Mixtral shape 256
    // rows 432 / 396 us, 320 450 / 370, 512 694 / 545; Qwen2-MoE shape 256 rows 440 / 426).  At 200-248 rows with near-uniform
    // routing 0 is 3-15 % ahead on some shapes (Mixtral 246 / 263, 32 experts of 2880 x 2880 154 / 181) and 0-18 % behind on
    // others (16 experts of 6144 x 4096 247 / 230, 4 of 2048 x 8192 94 / 80), but under routing skew, which the host cannot
    // see, it is up to 1.58x behind (8 experts of 6144 x 16384, 200-240 rows: 611-755 / 455-505), so the line stays.
    if (!packed) return once && !wide ? 0 : 10;
    // Packed.  Two weight blocks also where one block each would make between one and two rounds of workgroups and two make a single
    // one: us, one / two: Mixtral-8x22B shape (24 tiles of 256 x 8 experts) 64 tokens 266 / 240, 512 tokens 373 / 320, at skew 1 416 / 366; 7
    // experts, 8192 -> 5120, 300 tokens 155 / 139; 16 experts, 6400 -> 4096, 1000 tokens 174 / 152.  Not where one block each is a
    // single round (Mixtral-8x7B shape, 700 tokens 212 / 221) or two make a second (24 experts, 4096 -> 3072, 800 tokens 125 / 133).
    // A last tile of 128 features counts as a whole one of 256: 24 experts at d = 2688 are 504 tiles of 128, but 264 of 256 (800 tokens 90 / 110),
    // 102 at d = 640 510 and 306 (89 / 102).  256 CUs, not the device's count: kernels can be named without a device.
    // From 16 tiles of 256 on: below, the second blocks that routing skew makes, which the host cannot see, cost more than a single round gains.
    // us, one / two, near-uniform and at skew 0.8 (mean of three routings): 9 experts, 4096 -> 3712 67 / 62, 75 / 87; 16 experts, 4096 -> 2176
    // 67 / 60, 75 / 84; 60 of 1024 x 1024, 1000 tokens 33 / 31, 40 / 44; 85 of 2048 -> 640 46 / 44, 48 / 54; 128 of 3584 -> 512 85 / 86, 88 / 97.
    const bool one_round = c.d >= 4096 && (c.d + 127) / 128 * active > 256 && (c.d + 255) / 256 * active <= 256;
    // Beyond 192 rows many experts have a second block (Mixtral-8x7B shape, 900 tokens, skew 0.3, one / two weight blocks 353 / 312), unless the
    // launch is still a single round with those (16 experts, 4096 -> 1024, 1600 tokens 59 / 66, 1800 tokens at skew 0.5 58 / 73).
    const bool second_blocks = (double)R / c.E > 192.0 && (c.d + 127) / 128 * (active + R / 256) > 256;
    // Streamed weights up to 240 rows per expert and 256 MB of rows.  us, cached / streamed: Qwen2-MoE shape 1900 tokens (237 rows) 332 / 305, at
    // skew 1 391 / 359; Mixtral-8x22B shape 900 tokens at skew 1 473 / 440; Mixtral-8x7B shape 900 tokens (225 rows) 270 / 260; 128
    // experts, 2048 tokens (134 MB) 332 / 323; 256 experts, 2048 tokens (235 MB) 1420 / 1409; 60 experts, 1408 -> 2048, 3300 tokens (220 rows) 117 / 101.
    // Beyond: 60 experts, 1408 -> 2048, 2400 tokens of 6 (240
    // rows) 138 / 145; 256 experts, 4096 tokens (470 MB) at skew 1, where the cached kernel deals, 1513 / 1561.
    if ((double)R / c.E < 240.0 && (double)R * c.d * 2.0 <= 256e6) return wide || one_round || second_blocks ? 6 : 5;
    return 7;
}

}  // namespace

bool down_deals(const moe_config& c, int32_t M, bool packed) {
    int id = forced_variant(kKnobDownVariant, kNumDown, M, packed, kDown);
    if (id < 0) id = pick(M, packed, c);
    return id == 7;
}

bool down_fuses_combine(const moe_config& c, int32_t M, bool packed) {
    int id = forced_variant(kKnobDownVariant, kNumDown, M, packed, kDown);
    if (id < 0) id = pick(M, packed, c);
    // the per-block-regime kernels (LDS-DMA body) carry the fused epilogue; token * groups + group is an int
    return kDown[id].packed && id >= 5 && (long long)c.T * combine_groups(c) < (1ll << 31);
}

const char* down_variant_name(const moe_config& c, int32_t M, bool packed) {
    int id = forced_variant(kKnobDownVariant, kNumDown, M, packed, kDown);
    if (id < 0) id = pick(M, packed, c);
    return kDown[id].name;
}

hipError_t launch_down(const moe_config& c, int32_t M, const uint16_t* h, int32_t ldh, const int32_t* offsets,
                       const int32_t* blocks, const int32_t* num_blocks, const int32_t* blocks_mix,
                       const int32_t* num_heavy, const uint16_t* wd,
                       const uint16_t* packed_dn, uint16_t* y_perm, const CombineFusion* fuse, hipStream_t s) {
    GemmArgs a{};
    a.X = h;
    a.src = nullptr;
    a.src_k = 1;
    a.x_rows = c.T * c.k;
    a.ldx = ldh;
    a.ldo = c.d;
    a.rot_mul = rot_steps(false);
    a.rot_mul_multi = rot_steps(true);
    a.W0 = wd;
    a.P = packed_dn;
    a.Out = y_perm;
    a.offsets = offsets;
    a.blocks = blocks;
    a.num_blocks = num_blocks;
    a.num_multi = num_heavy;
    a.R = c.T * c.k;
    a.N = c.d;
    a.K = c.F;
    a.E = c.E;
    a.M = M;
    // token rows are addressed with 32-bit byte offsets from the buffer's base
    if ((unsigned long long)a.x_rows * (unsigned long long)ldh * 2ull >= (1ull << 32)) return hipErrorInvalidValue;
    const bool packed = packed_dn != nullptr;
    int id = forced_variant(kKnobDownVariant, kNumDown, M, packed, kDown);
    if (id < 0) id = pick(M, packed, c);
    if (kDown[id].M < M) return hipErrorInvalidValue;
    // The two-weight-block kernel with cached loads (the choice once experts hold many rows, i.e.
    // whenever routing skew has produced multi-block experts in a large batch) is also given the
    // list that holds the heavy blocks first: it deals the two classes evenly over its launch when
    // the light class is a large enough share of it, and keeps Algorithm 1's order otherwise.
    if (id == 7 && blocks_mix != nullptr && num_heavy != nullptr && knob(kKnobInterleave) != 0) {
        a.blocks_mix = blocks_mix;
        a.num_heavy = num_heavy;
        a.deal_always = knob(kKnobInterleave) > 0;
    }
    if (fuse != nullptr) {
        if (id < 5 || !kDown[id].packed) return hipErrorInvalidValue;   // only the per-block-regime kernels have the fused epilogue
        a.comb_src = fuse->src_of;
        a.comb_row_of = fuse->row_of;
        a.comb_w = fuse->topk_w;
        a.comb_arrive = fuse->arrive;
        a.comb_y = fuse->y;
        a.comb_k = c.k;
        a.comb_groups = combine_groups(c);
    }
    return kDown[id].fn(a, moe_max_blocks(&c, M), s);
}

}  // namespace moe

// Test hook (exported, not declared in include/moe.h): enumerate on the HOST what every workgroup
// of a per-block-regime GEMM launch would work on, with the launch-order switches and the grid the
// launcher itself would use.  All array arguments are host memory; E experts hold offsets[E] rows of K elements, `packed` says how
// the weights are laid out, `half` names the build for two workgroups per CU.  out[w] = {has work, expert,
// first row, rows, feature tile, feature-tile width in units of 128, in runs of positions per XCD, results stored
// non-temporally}; returns the grid size, or -1
// if it exceeds `capacity` or (gateup, ib) names no kernel.  blocks_mix may be null (no dealing).
extern "C" __attribute__((visibility("default"))) int32_t moe_test_map_launch(
    int32_t gateup, int32_t ib, int32_t wnt, int32_t half, int32_t packed, int32_t N, int32_t K, int32_t E, int32_t M, const int32_t* offsets,
    const int32_t* blocks, int32_t num_blocks, const int32_t* blocks_mix, int32_t num_heavy, int32_t cus, int32_t max_blocks, int32_t capacity,
    int32_t* out) {
    using namespace moe;
    GemmArgs a{};
    a.N = N;
    a.M = M;
    a.K = K;
    a.E = E;
    a.R = offsets[E];
    const uint16_t weights = 0;
    a.P = packed ? &weights : nullptr;   // only whether there is a packed copy is asked
    a.offsets = offsets;
    a.blocks = blocks;
    a.num_blocks = &num_blocks;
    int32_t multi = 0;
    for (int i = 0; i < num_blocks; ++i) multi += blocks[2 * i + 1] > 0 || (i + 1 < num_blocks && blocks[2 * i + 3] > 0);
    a.num_multi = &multi;
    if (blocks_mix != nullptr && knob(kKnobInterleave) != 0) {
        a.blocks_mix = blocks_mix;
        a.num_heavy = &num_heavy;
        a.deal_always = knob(kKnobInterleave) > 0;
    }
    auto run = [&](auto ibc, auto guc, auto wntc, auto halfc) -> int32_t {
        constexpr int IB = decltype(ibc)::value;
        constexpr bool GU = decltype(guc)::value, WNT = decltype(wntc)::value, HALF = decltype(halfc)::value;
        const long long grid = mixed_launch_shape<IB, GU, WNT, HALF>(a, max_blocks, cus);
        if (grid > capacity) return -1;
        for (int w = 0; w < (int)grid; ++w) {
            MixedWork m{};
            const bool has = mixed_assign<IB, GU>(a, w, m);
            int32_t* o = out + 8 * (size_t)w;
            o[0] = has;
            o[1] = m.e; o[2] = m.row0; o[3] = m.rows; o[4] = m.nt;
            o[5] = m.halves ? 1 : IB;
            o[6] = m.chunked;
            o[7] = m.stream;
        }
        return (int32_t)grid;
    };
    using T_ = std::true_type;
    using F_ = std::false_type;
    const std::integral_constant<int, 1> one;
    const std::integral_constant<int, 2> two;
    if (ib == 1 && half) return gateup ? run(one, T_{}, T_{}, T_{}) : run(one, F_{}, T_{}, T_{});
    if (gateup && ib == 1) return wnt ? run(one, T_{}, T_{}, F_{}) : run(one, T_{}, F_{}, F_{});
    if (!gateup && ib == 1) return wnt ? run(one, F_{}, T_{}, F_{}) : run(one, F_{}, F_{}, F_{});
    if (!gateup && ib == 2) return wnt ? run(two, F_{}, T_{}, F_{}) : run(two, F_{}, F_{}, F_{});
    return -1;
}

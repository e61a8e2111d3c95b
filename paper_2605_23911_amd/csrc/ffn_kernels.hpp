// Block-scheduled grouped GEMMs of the expert FFN on bf16 MFMA (gfx950).
// Paper: Sec. 3.2 (one launch, workgroup -> (expert, row offset) through the block schedule,
// partial tiles masked), Sec. 3.3 (gate and up projections from one shared input tile, two
// accumulators, SiLU(gate)*up in fp32 registers, a single 2-byte intermediate), Eq. 4.
//
// What differs from the paper's A100 design: the MFMA computes the TRANSPOSED tile
//     C^T[f, row] = sum_k W[f, k] * X[row, k]
// with the weight rows as the first MFMA operand.  The stored weight layout ([out, in], the
// reduction dim contiguous) is then exactly the per-lane operand layout: a weight fragment is 16
// bytes per lane, loaded straight to registers or, in rows_body, brought to LDS by DMA and read back
// by the wavefront it belongs to.  The MFMA sums over k, so which k a
// fragment slot carries is free as long as both operands agree: MFMA s of a 64-wide step takes
// k = 16 s + 8 (lane / 32) + 0..7, which makes the two lanes of a weight row read 32 contiguous
// bytes per load instruction (one 64-byte L1 access instead of two).  Each wavefront owns its own weight rows
// and all token rows of the tile, so every weight byte is fetched once per workgroup.  In C^T
// a lane holds four consecutive output features of one token row (8-byte packed bf16 stores).
//
// PACKED weights: lanes of one load instruction read 32 different weight rows, 16 bytes each,
// which costs one L1 access per lane.  moe_pack_weights re-orders the weights once (weights are
// static at inference) into the order the loads consume them, [expert][32-row block][64-k step]
// [matrix][s][lane] x 16 bytes, so that one load instruction reads 1 KiB contiguous and a
// wavefront streams one contiguous region.  Row-major weights have kernels of their own (tile_kernel,
// skinny_kernel<.., false>).
//
// Kernels that share that mapping:
//   tile_kernel_mixed  token tile (up to 256 rows) brought global -> LDS by DMA into a ring of
//                      buffers and shared by the four wavefronts; body chosen per block from
//                      the rows it holds, regime per block from its expert's rows: weights streamed
//                      once (non-temporal, k rotated) for experts that fit one block, shared
//                      through L2 (cached, k in step, row tiles side by side) for experts that
//                      span several (packed weights).
//   tile_kernel        the same for row-major weights, which go through LDS too (rows_body).
//   skinny_kernel      <= 64 token rows, token fragments loaded straight from L2 by each
//                      wavefront: no LDS, no barrier in the reduction loop; the four wavefronts
//                      split K (down projection of few-expert models at a handful of tokens,
//                      where there are too few output rows to fill 256 CUs otherwise).
#pragma once

#include <climits>
#include <type_traits>
#include <utility>

#include "lds_dma.hpp"
#include "moe_internal.hpp"

namespace moe {

struct GemmArgs {
    const uint16_t* X;          // [R, K] expert-contiguous rows, or the un-permuted [T, K] rows if src != nullptr
    const int32_t* src;         // [R] flat (token, slot) index of every expert-contiguous row, or nullptr
    int src_k;                  // slots per token: row r then lives at X[src[r] / src_k]
    int x_rows;                 // rows of X (T with a source map, else R); x_rows * ldx * 2 bytes < 4 GiB
    int ldx, ldo;               // row strides of X and Out in elements (>= K and >= N)
    int rot_mul;                // k-loop rotation between workgroups of one XCD, in steps (see tile_body_dma)
    int rot_mul_multi;          // the same for blocks of experts that span several row tiles (tile_kernel_mixed)
    int slots;                  // workgroups the chip runs at once (one per CU); 0 = do not split the last round
    int cus;                    // CUs of the device (0: not known)
    const uint16_t* W0;         // [E, N, K]  gate (or down)
    const uint16_t* W1;         // [E, N, K]  up   (unused for down)
    const uint16_t* P;          // packed weights of this projection (PACKED kernels), else unused
    uint16_t* Out;              // [R, N]
    const int32_t* offsets;     // [E+1]
    const int32_t* blocks;      // [*, 2] (expert, row offset inside the expert)
    const int32_t* num_blocks;  // device scalar
    const int32_t* num_heavy;   // device scalar or null: the first *num_heavy blocks belong to multi-block experts (tile_kernel_mixed)
    const int32_t* num_multi;   // device scalar: the blocks of experts that have more than one
    int R, N, K, n_tiles_n;
    int M;                      // tile height of the block schedule (rows per block <= M)
    int sib;                    // tile_kernel_mixed: launch the row tiles of one expert side by side (see there)
    int chunk;                  // tile_kernel_mixed: runs of `unit` positions per XCD: 0 never, 1 always, 2 by the rule (see there)
    int unit;                   // length of a run: half of the workgroups that an XCD runs at once
    int multi_from, few_from;   // chunk 2: workgroups from which on a launch with (few) blocks of multi-block experts goes in runs
    int light;                  // ... if the single-block experts number at most light / 5 of those blocks
    int eighths;                // without multi-block experts: one run per XCD
    int stream;                 // results of single-block experts may be stored non-temporally (store_tile)
    int rot_mul_chunk;          // the k-loop rotation of blocks whose feature tiles run on one XCD
    const int32_t* blocks_mix;  // with num_heavy: the same blocks, those of multi-block experts first (the list the dealt order reads)
    int deal_always;            // tile_kernel_mixed with num_heavy: deal the two classes whatever their proportion (tests)
    int even;                   // tile_kernel_mixed: rows of a multi-tile expert dealt evenly over its schedule entries
    int no_nt;                  // tile_kernel_mixed: cached weight loads for every block (test knob)
    int short_nt;               // tile_kernel_mixed: tiles of at most this many rows stream their weights non-temporally
    // Weighted combine folded into the down projection (all null / 0 when it is a separate launch):
    const int32_t* comb_src;    // [R] flat (token, slot) index of every expert-contiguous row
    const int32_t* comb_row_of; // [T, k] expert-contiguous row of every (token, slot)
    const float* comb_w;        // [T, k] gate weights
    int32_t* comb_arrive;       // [T, comb_groups] rows of the token written so far per 128-feature group (zero at launch)
    uint16_t* comb_y;           // [T, N] layer output
    int comb_k, comb_groups;    // experts per token; ceil(N / 128)
    // Permutation done by the gate+up launch itself (permute_inside; all null / 0 when it is a launch of its own):
    const int32_t* topk_idx;    // [R] the router's choice
    PermuteOut perm;            // what the later stages read, written by workgroup 0
    int E;                      // experts
    int tables_in_lds;          // src, offsets and blocks are in the LDS that the token ring will use
};

typedef hipError_t (*launch_fn)(const GemmArgs&, int, hipStream_t);

// The down projection's per-block-regime kernels with two weight blocks per wavefront are
// compiled in a translation unit of their own (ffn_down_wide.hip) to shorten the build.
// (So are, in ffn_gate_up_routed.hip, the gate+up kernels with the permutation inside.)
hipError_t launch_routed_mixed(const GemmArgs& a, int max_blocks, hipStream_t s);
hipError_t launch_routed_mixed_half(const GemmArgs& a, int max_blocks, hipStream_t s);
hipError_t launch_down_mixed_wide_nt(const GemmArgs& a, int max_blocks, hipStream_t s);
hipError_t launch_down_mixed_wide(const GemmArgs& a, int max_blocks, hipStream_t s);
hipError_t launch_down_rows_wide(const GemmArgs& a, int max_blocks, hipStream_t s);

namespace {

constexpr int kThreads = 256;
constexpr int kBK = 64;            // reduction elements per pipeline step


template <int... Is, class F>
__device__ __forceinline__ void static_for_impl(std::integer_sequence<int, Is...>, F&& f) {
    (f(std::integral_constant<int, Is>{}), ...);
}
// Calls f(integral_constant<0>) ... f(integral_constant<N-1>): indices are compile-time
// constants in the source, so register arrays never need a loop-unrolling pass to be promoted.
template <int N, class F>
__device__ __forceinline__ void static_for(F&& f) {
    static_for_impl(std::make_integer_sequence<int, N>{}, f);
}

// Weight loads.  NT: when an expert is a single block each PACKED weight byte is used exactly
// once per launch (one load instruction consumes whole 128-byte lines), and loading it with the
// non-temporal hint keeps the streamed weights from evicting the re-used token tiles from L2
// (+5..10 % at T <= 512).  When an expert spans several row blocks they share the weight panel
// through L2 and the hint would defeat that; so it would for row-major weights loaded to registers,
// where a line is consumed by four load instructions (skinny_kernel).  By DMA (rows_body) a
// row-major load takes whole lines too.
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
template <bool NT>
__device__ __forceinline__ uint4 load_w16(const uint16_t* p) {
    if constexpr (NT) {
        const u32x4 v = __builtin_nontemporal_load(reinterpret_cast<const u32x4*>(p));
        return make_uint4(v[0], v[1], v[2], v[3]);
    } else {
        return *reinterpret_cast<const uint4*>(p);
    }
}

__device__ __forceinline__ float silu_mul(float g, float u) {
    // SiLU(g) * u with SiLU(g) = g / (1 + exp(-g)); exp(-g) = inf for very negative g gives -0.
    // v_rcp_f32 (1 ulp) on purpose: the correctly rounded reciprocal expands to a ten-instruction
    // division, which made up 40 % of the epilogue; the result is rounded to bf16 right after.
    return g * __builtin_amdgcn_rcpf(1.0f + __expf(-g)) * u;
}

// Buffer descriptor: base and range in bytes.  Offsets beyond the range read as zero and are not written.
typedef __amdgpu_buffer_rsrc_t rsrc_t;
__device__ __forceinline__ rsrc_t make_rsrc(const void* base, uint32_t bytes) {
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(base), 0, bytes, 0x00020000);   // raw, 32-bit data format
}
// Weight fragment addressing.  Unpacked: row-major rows, element (row, k).  Packed: 16-byte
// units ordered [expert][row block][k step][matrix][s][lane].
template <bool PACKED, int NM>
struct WAddr {
    static constexpr int kStep = PACKED ? NM * 4 * 512 : kBK;   // elements per 64-wide k step
    static constexpr int sStep = PACKED ? 512 : 16;              // elements per MFMA slot s
    // A fragment address is block() + lane_bytes(): block() is the same for the whole wavefront
    // (it lives in scalar registers and the per-step advance is scalar arithmetic), lane_bytes()
    // is a 32-bit per-lane offset that never changes, so a load needs no per-step vector
    // address arithmetic and no 64-bit address registers.
    __device__ static __forceinline__ int clamp_block(const GemmArgs& a, int row_block) {
        const int last = PACKED ? a.N / 32 - 1 : (a.N - 1) / 32;   // ragged last feature tile: stores are masked
        return row_block < last ? row_block : last;
    }
    __device__ static __forceinline__ const uint16_t* block(const GemmArgs& a, int e, int row_block, int m) {
        const int rb = clamp_block(a, row_block);
        if constexpr (PACKED)
            return a.P + ((size_t)e * (a.N / 32) + rb) * (size_t)(a.K / kBK) * kStep + m * 4 * 512;
        else
            return (m == 0 ? a.W0 : a.W1) + ((size_t)e * a.N + rb * 32) * a.K;
    }
    __device__ static __forceinline__ uint32_t lane_bytes(const GemmArgs& a, int row_block, int lane) {
        if constexpr (PACKED) {
            return (uint32_t)lane * 16u;
        } else {
            const int li = lane & 31, half = lane >> 5;
            const int rb = clamp_block(a, row_block);
            int row = rb * 32 + li;
            row = (row < a.N ? row : a.N - 1) - rb * 32;
            return (uint32_t)(row * a.K + half * 8) * 2u;
        }
    }
    __device__ static __forceinline__ const uint16_t* base(const GemmArgs& a, int e, int row_block, int m, int lane) {
        return block(a, e, row_block, m) + lane_bytes(a, row_block, lane) / 2;
    }
};

// Address of expert-contiguous token row `row` (clamped to the last row).  With a source map the
// permutation of Sec. 3.1 is applied here, in the load address, and the permuted copy of the
// activations is never written.
__device__ __forceinline__ int token_row_index(const GemmArgs& a, int row) {
    row = row < a.R ? row : a.R - 1;
    if (a.src != nullptr) row = a.src[row] / a.src_k;
    return row;
}
__device__ __forceinline__ const uint16_t* token_row(const GemmArgs& a, int row) {
    return a.X + (size_t)token_row_index(a, row) * a.ldx;
}
// Byte offset of a token row from a.X as 32 bits (the launchers refuse buffers of 4 GiB or more).
__device__ __forceinline__ uint32_t token_row_bytes(const GemmArgs& a, int row) {
    return (uint32_t)token_row_index(a, row) * (uint32_t)a.ldx * 2u;
}

// The thread's number at the start of a body, of which a kernel holds up to sixteen.  Opaque to the compiler: it would work out what the bodies derive
// from it (places in LDS, rows of the tile) once, in front of them all, and hold it in registers that the tallest body does not have.
// Scratch, bytes per lane, without / with: tile_kernel_mixed<2, false, true, true, false> 40 / 8, <.., false, false> 12 / 8, tile_kernel<1, true>
// 8 / 0, routed_tile_kernel_mixed<true> 16 / 0; times the same or up to 1 % shorter.
__device__ __forceinline__ int body_thread() {
    int tid = threadIdx.x;
    asm volatile("" : "+v"(tid));
    return tid;
}

// Block schedule entry -> tile geometry (Alg. 1: block = (expert, row offset)).
struct Tile {
    int e, row0, rows;
    int n_e;       // rows of the whole expert
    int rot_mul;   // k-loop rotation between workgroups of one XCD, in steps (tile bodies)
    bool stream;   // the results are stored non-temporally (store_tile)
};
__device__ __forceinline__ bool load_tile(const GemmArgs& a, int tile, int BM, Tile& t) {
    BM = a.M < BM ? a.M : BM;   // a kernel may serve a schedule with shorter blocks than it can hold
    if (tile >= *a.num_blocks) return false;
    t.e = a.blocks[2 * tile];
    const int r_in = a.blocks[2 * tile + 1];
    const int seg0 = a.offsets[t.e];
    const int n_e = a.offsets[t.e + 1] - seg0;
    t.row0 = seg0 + r_in;
    t.rows = (n_e - r_in) < BM ? (n_e - r_in) : BM;
    t.n_e = n_e;
    return true;
}

// Workgroup -> (tile, feature tile): tile-major, feature tiles of one block-schedule entry
// adjacent.  The hardware deals workgroups to the 8 XCDs round-robin; with a feature-tile count
// that is a multiple of 8 the row tiles of one expert that share a weight panel land on the
// same XCD (and run at about the same time), so the panel is fetched into one L2 only.
// (Measured: cutting the work into 8 contiguous per-XCD chunks instead is slower at large T
// because it separates exactly those row tiles in time.)
__device__ __forceinline__ bool map_workgroup(const GemmArgs& a, int& tile, int& nt) {
    tile = blockIdx.x / a.n_tiles_n;
    nt = blockIdx.x - tile * a.n_tiles_n;
    return true;
}

// Epilogue for one 32x32 MFMA block: the lane holds, for token row (j*32 + lane%32), the
// features q*8 + 4*(lane/32) + 0..3 (q = 0..3) of the block that starts at feature f0.  The two
// lanes of a row (lane and lane^32) swap halves so that each writes two 16-byte pieces (lane/32
// = 0: features 0..7 and 16..23, lane/32 = 1: 8..15 and 24..31) instead of four 8-byte ones:
// half as many store instructions and write requests.  For few rows, and for results that other workgroups of the launch read
// (fused_combine); else store_tile.  Every lane of the wavefront must call
// this (the swap is a cross-lane operation); `live` masks the stores of rows beyond the tile.
// DEVICE_SCOPE: the 16-byte pieces are written with device-scope (sc1) stores, which go through
// to the level all XCDs share, so that a workgroup on another XCD can read them after this
// wavefront has waited for its stores and bumped a counter (fused combine), without an L2
// write-back.
template <bool GATEUP, bool DEVICE_SCOPE = false>
__device__ __forceinline__ void store_block(const f32x16& g, const f32x16& u, uint16_t* out_row, int f0, int half,
                                            int N, bool live) {
    uint2 pk[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        float o[4];
#pragma unroll
        for (int v = 0; v < 4; ++v) o[v] = GATEUP ? silu_mul(g[q * 4 + v], u[q * 4 + v]) : g[q * 4 + v];
        pk[q].x = pack2_bf16(o[0], o[1]);
        pk[q].y = pack2_bf16(o[2], o[3]);
    }
#pragma unroll
    for (int p = 0; p < 2; ++p) {   // pair p: groups q = 2p (kept by half 0) and q = 2p + 1 (kept by half 1)
        const uint2 give = half ? pk[2 * p] : pk[2 * p + 1];
        uint2 got;
        got.x = __shfl_xor(give.x, 32, kWave);
        got.y = __shfl_xor(give.y, 32, kWave);
        const int f = f0 + (2 * p + half) * 8;
        const uint4 v = half ? make_uint4(got.x, got.y, pk[2 * p + 1].x, pk[2 * p + 1].y)
                             : make_uint4(pk[2 * p].x, pk[2 * p].y, got.x, got.y);
        if (live && f < N) {
            if constexpr (DEVICE_SCOPE) {
                // one-row descriptor: base = the row, range = N elements
                const u32x4 d4 = {v.x, v.y, v.z, v.w};
                __builtin_amdgcn_raw_buffer_store_b128(d4, make_rsrc(out_row, (uint32_t)N * 2u), (uint32_t)f * 2u, 0, 16);
            } else {
                *reinterpret_cast<uint4*>(out_row + f) = v;
            }
        }
    }
}

// Epilogue of a whole tile (JBE * 32 rows x 128 * IB features): the bf16 results are staged in LDS, which the reduction loop no
// longer needs, and every row is stored in one piece of 256 * IB bytes.  store_block writes the same row in pieces of 32 bytes,
// IB * 8 of them; the write path takes the pieces one by one, and while they wait the workgroup holds its CU.
// Non-temporally (Tile::stream) where the launch writes 2 MiB or more and its weights do not fit the Infinity Cache beside the results (more than 128 MiB per
// matrix), and the expert is one block: whole lines that go straight through L2 leave it
// to the weights and token rows; cached stores of whole rows gain less, non-temporal pieces lose.  Projection alone,
// us, store_block / staged and cached / staged and non-temporal: down, 64 experts of 128 rows, 2048 -> 7168, 371 / 366 / 332,
// 144 rows 384 / 376 / 342, 16 rows 317 / 317 / 310; gate+up, 8 experts of 144 rows, 4096 -> 14336, 350 / 348 / 336.  What is streamed is read back from HBM.
// Cached below those sizes, where the next kernel still finds the results near (us, layer, cached / non-temporal: 24 experts of 512 x 1024, 1000 tokens
// 56.0 / 57.6; 8 of 1024 x 1024, 1000 tokens 63.9 / 67.5; 16 of 512 x 2048, 600 tokens 65.1 / 68.3; above them 32 of 1408 x 1536, 2045 tokens 114.5 / 109.5), and
// for experts of several blocks (32 experts of 2880 x 2880, 1001 tokens at skew 1, down projection 134 / 139).
// The rows of h also under routing skew, where the tall experts are what the down projection ends with and read their rows from HBM then: if an expert has several blocks,
// or this one more than twice the mean (us, layer, cached / non-temporal: 8 experts of 2048 x 8192, 500 tokens at skew 1 233 / 243; Mixtral shape,
// 300 tokens at skew 1 549 / 560, 200 tokens at skew 1.6 520 / 526).
// A single 32-row block with cached stores takes store_block: nothing there pays for two barriers (8 experts of 256 x 512, 64 tokens,
// layer 20.5 / 20.7; 60 of 2048 x 1408, 64 tokens, 186.4 / 187.2).
// Every wavefront must call this, with none of its loads into LDS outstanding.
template <bool GATEUP, int IB, int JBE, int NI>
__device__ __forceinline__ void store_tile(const f32x16 (&acc)[NI][JBE], const GemmArgs& a, const Tile& t, int nt, uint16_t* xs) {
    constexpr int BN = 128 * IB;
    constexpr int LD = BN * 2 + 16;              // bytes of a staged row: 16 more, so that the 32 rows a wavefront writes spread over the banks
    const int tid = threadIdx.x, wave = tid / kWave, lane = tid % kWave;
    const int li = lane & 31, half = lane >> 5;
    char* lds = reinterpret_cast<char*>(xs);
    if constexpr (JBE == 1) {
        if (!t.stream) {
            const bool live = li < t.rows;
            static_for<IB>([&](auto ib) {
                store_block<GATEUP>(acc[ib][0], acc[GATEUP ? IB + ib : ib][0], a.Out + (size_t)(t.row0 + (live ? li : 0)) * a.ldo,
                                    nt * BN + (wave * IB + ib) * 32, half, a.N, live);
            });
            return;
        }
    }
    __syncthreads();                             // nobody reads the ring any more, nothing is landing in it
    static_for<IB>([&](auto ib) {
        static_for<JBE>([&](auto j) {
            char* row = lds + (j * 32 + li) * LD + (wave * IB + ib) * 64 + half * 8;   // the lane's features: q * 8 + 4 * half + 0..3
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                float o[4];
#pragma unroll
                for (int v = 0; v < 4; ++v) {
                    const float g = acc[ib][j][q * 4 + v];
                    o[v] = GATEUP ? silu_mul(g, acc[GATEUP ? IB + ib : ib][j][q * 4 + v]) : g;
                }
                *reinterpret_cast<uint2*>(row + q * 16) = make_uint2(pack2_bf16(o[0], o[1]), pack2_bf16(o[2], o[3]));
            }
        });
    });
    __syncthreads();
    constexpr int LANES = BN / 8, ROWS = kThreads / LANES;   // lanes per row, rows per pass of the workgroup
    const int r0 = tid / LANES, c = tid % LANES, f = nt * BN + c * 8;
    if (f >= a.N) return;
    uint16_t* out = a.Out + (size_t)t.row0 * a.ldo + f;
    auto rows = [&](auto stream) {
#pragma unroll
        for (int p = 0; p < JBE * 32 / ROWS; ++p) {
            const int r = p * ROWS + r0;
            const u32x4 v = *reinterpret_cast<const u32x4*>(lds + r * LD + c * 16);
            u32x4* dst = reinterpret_cast<u32x4*>(out + (size_t)r * a.ldo);
            if (r < t.rows) {
                if constexpr (decltype(stream)::value) __builtin_nontemporal_store(v, dst);
                else *dst = v;
            }
        }
    };
    if (t.stream) rows(std::true_type{});
    else rows(std::false_type{});
}
// LDS that store_tile needs
constexpr int store_lds(int jbe, int ib) { return jbe * 32 * (256 * ib + 16); }

// Up to 1024 rows (permutes_inside): every workgroup of the gate+up launch sorts the router's choice by itself, up to four
// slots per thread, and reads its own place in the schedule from LDS: same counting sort, same tables as permute.hip's.
// It takes the place of a launch (5-8 us) and, in each workgroup, of the chain of loads from the tables that the launch
// wrote.  Workgroup 0 leaves the tables in memory for the later stages.  Costs and gains: permutes_inside.
constexpr int kSmallGroups = kSmallRows / kThreads;
constexpr int kSmallBlocks = kSmallRows / 32 + kMaxExperts;   // schedule entries: R / M + min(R, E), M >= 32
__device__ __forceinline__ void permute_inside(const GemmArgs& a, GemmArgs& b, int32_t* lds) {
    int32_t* off = lds;                            // [E + 1]
    int32_t* blk = off + kMaxExperts + 4;          // [kSmallBlocks, 2]
    int32_t* src = blk + 2 * kSmallBlocks;         // [R]
    int32_t* nblk = src + kSmallRows;              // the number of entries, and the wavefronts' sums
    int32_t(*wc)[kMaxExperts] = reinterpret_cast<int32_t(*)[kMaxExperts]>(nblk + 16);
    const int tid = threadIdx.x, lane = tid % kWave, wave = tid / kWave;
    constexpr int W = kThreads / kWave;
    static_assert(kThreads == kMaxExperts, "one expert per thread");
    const int G = (a.R + kThreads - 1) / kThreads; // 64-slot groups per wavefront, in slot order
#pragma unroll
    for (int w = 0; w < W; ++w) wc[w][tid] = 0;
    if (tid == 0) nblk[1] = 0;
    int e_of[kSmallGroups];
#pragma unroll
    for (int g = 0; g < kSmallGroups; ++g) {
        const int j = (wave * G + g) * kWave + lane;
        e_of[g] = -1;
        if (g < G && j < a.R) {
            const int e = a.topk_idx[j];
            e_of[g] = e < 0 ? 0 : (e >= a.E ? a.E - 1 : e);   // as in permute.hip: an id outside the experts never leaves the buffers
        }
    }
    __syncthreads();
#pragma unroll
    for (int g = 0; g < kSmallGroups; ++g)
        if (e_of[g] >= 0) atomicAdd(&wc[wave][e_of[g]], 1);
    __syncthreads();
    int n = 0;                                     // rows of expert tid
#pragma unroll
    for (int w = 0; w < W; ++w) n += wc[w][tid];
    const int nb = (n + a.M - 1) / a.M;
    const int v = n | nb << 16;                    // both at most 1024 in all: one scan for the two
    int inc = v;
#pragma unroll
    for (int o = 1; o < kWave; o <<= 1) {
        const int up = __shfl_up(inc, o, kWave);
        if (lane >= o) inc += up;
    }
    if (lane == kWave - 1) nblk[4 + wave] = inc;
    __syncthreads();
    int base = inc - v;
#pragma unroll
    for (int w = 0; w < W; ++w) base += w < wave ? nblk[4 + w] : 0;
    const int row0 = base & 0xffff, block0 = base >> 16;
    if (tid < a.E) {
        off[tid] = row0;
        if (tid == a.E - 1) off[a.E] = row0 + n, nblk[0] = block0 + nb;
        int run = row0;                            // counts per wavefront -> first row per wavefront
#pragma unroll
        for (int w = 0; w < W; ++w) {
            const int c = wc[w][tid];
            wc[w][tid] = run;
            run += c;
        }
    }
    for (int q = 0; q < nb; ++q) {
        blk[2 * (block0 + q)] = tid;
        blk[2 * (block0 + q) + 1] = q * a.M;
    }
    if (nb > 1) atomicAdd(&nblk[1], nb);           // cleared before the first barrier
    __syncthreads();
    volatile int32_t* next = wc[wave];
#pragma unroll
    for (int g = 0; g < kSmallGroups; ++g) {
        if (g < G) {                               // uniform over the workgroup
            const int e = e_of[g];
            // lanes holding the same expert: AND over the 8 id bits of agreeing ballots
            unsigned long long same = __ballot(e >= 0);
#pragma unroll
            for (int i = 0; i < 8; ++i) {
                const unsigned long long bal = __ballot((e >> i) & 1);
                same &= ((e >> i) & 1) ? bal : ~bal;
            }
            if (e >= 0) {
                const unsigned long long below = same & ((1ull << lane) - 1ull);
                const int first = next[e], pos = first + __popcll(below), j = (wave * G + g) * kWave + lane;
                src[pos] = j;
                if (below == 0) next[e] = first + __popcll(same);   // lowest lane of the set advances it
                if (blockIdx.x == 0) {
                    a.perm.row_of[j] = pos;
                    a.perm.src_of[pos] = j;
                }
            }
            __builtin_amdgcn_wave_barrier();
        }
    }
    __syncthreads();
    if (blockIdx.x == 0) {
        if (tid < a.E) {
            a.perm.counts[tid] = n;
            a.perm.offsets[tid] = row0;
            if (tid == a.E - 1) a.perm.offsets[a.E] = row0 + n;
        }
        for (int i = tid; i < 2 * nblk[0]; i += kThreads) a.perm.blocks[i] = blk[i];
        if (tid == 0) a.perm.num_blocks[0] = nblk[0], a.perm.num_heavy[0] = nblk[1];
    }
    b.offsets = off;
    b.blocks = blk;
    b.num_blocks = nblk;
    b.num_multi = nblk + 1;
    b.src = src;
    b.tables_in_lds = 1;
}

// ---------------------------------------------------------------------------------------------
// tile_body_dma: same tile, but the token tile goes global -> LDS with the gfx950 LDS-DMA load
// (global_load_lds_dwordx4: each lane supplies its own global address, the 64 x 16 bytes land
// contiguously at M0 + 16*lane), so it needs no staging registers, no ds_write, and can be
// prefetched XD steps ahead into a ring of XD+1 LDS buffers.  LDS rows are 128 bytes, unpadded
// (the DMA fixes the destination order); bank conflicts are avoided by permuting the SOURCE:
// position p of row r holds chunk p ^ swz(r), swz(r) = (r ^ (r >> 3)) & 7, and the fragment
// reads apply the same XOR.  The DMA is issued from inline assembly so that the compiler does
// not serialise every later LDS read behind it; completion is awaited with an explicit
// s_waitcnt vmcnt(N) before the step's barrier (loads complete in issue order; N = the number
// of vector-memory loads this wavefront issues after the batch it waits for).  Memory operations
// the compiler adds on its own (a spill) cannot break the wait: while the awaited DMA is
// outstanding the N later loads are outstanding too, so the counter is above N; extra operations
// only lengthen the wait.
// ---------------------------------------------------------------------------------------------
// Weighted combine (Eq. 3) folded into the down projection: the paper's limitation 1, second
// half.  The k rows of a token come from k different experts, i.e. from workgroups that run at
// different times on different XCDs, each with an L2 of its own.  A device-scope fence pair
// (write back and invalidate the whole L2 around every tile) measured 1.4-2.7x on the down
// projection; instead the tile of y_perm is written with device-scope stores, the wavefronts wait
// for their acknowledgement, and the rows are read back with device-scope loads.  Each workgroup,
// once its tile is written, adds 1 to a counter per (token, 128-feature group) for every row it
// holds (device-scope atomics); whoever brings a counter to k knows that all k rows of that token and group are in
// memory, reads them back and forms
//     y[t, c] = sum_i w[t, i] * y_perm[row_of[t, i], c]
// in fp32 in slot order i = 0..k-1 from the bf16 values in memory, its own row included: the
// same arithmetic on the same operands as the stand-alone combine kernel, whichever workgroup
// arrives last, so y is bit-reproducible and bit-equal to moe_combine's.  No workgroup ever waits
// for another.  The counters are cleared by the router (the wavefront that routes token t clears
// token t's counters), so no extra launch and no host-side reset is involved.
// `nt` is the index of the workgroup's feature tile of width 128 * IB; xs is LDS that the
// reduction loop no longer uses.
template <int IB>
__device__ __forceinline__ void fused_combine(const GemmArgs& a, const Tile& t, int nt, uint16_t* xs) {
    int* list_n = reinterpret_cast<int*>(xs);
    int* list = list_n + 4;            // up to rows * IB entries: token * groups + group
    const int tid = threadIdx.x;
    const int groups = a.comb_groups, k = a.comb_k;
    wait_vmcnt<0>();                   // this wavefront's device-scope y_perm stores have been acknowledged
    __syncthreads();                   // ... and so have the other wavefronts'; LDS is free (all LDS-DMAs have landed too)
    if (tid == 0) *list_n = 0;
    __syncthreads();
    for (int r = tid; r < t.rows; r += kThreads) {
        const int token = a.comb_src[t.row0 + r] / k;
#pragma unroll
        for (int ib = 0; ib < IB; ++ib) {
            const int g = nt * IB + ib;
            if (g < groups) {
                const int old = atomicAdd(&a.comb_arrive[(size_t)token * groups + g], 1);
                if (old == k - 1) list[atomicAdd(list_n, 1)] = token * groups + g;
            }
        }
    }
    __syncthreads();
    const int n = *list_n;
    if (n == 0) return;
    const int sub = tid & 15;          // 16 lanes x 16 bytes = one 128-feature group of one row
    const uint32_t row_bytes = (uint32_t)a.ldo * 2u;
    const rsrc_t out_rows = make_rsrc(a.Out, (uint32_t)a.R * row_bytes);   // < 4 GiB: checked by the launcher
    for (int q = tid >> 4; q < n; q += kThreads / 16) {
        const int tg = list[q];
        const int token = tg / groups, g = tg - token * groups;
        const int c = g * 128 + sub * 8;
        if (c >= a.N) continue;
        const int32_t* rows = a.comb_row_of + (size_t)token * k;
        const float* w = a.comb_w + (size_t)token * k;
        float acc[8];
#pragma unroll
        for (int v = 0; v < 8; ++v) acc[v] = 0.0f;
        // Eight rows are requested before the first is used (the workgroup has its CU to itself:
        // nothing else hides the latency of these loads); the sum still runs in slot order.
        for (int i0 = 0; i0 < k; i0 += 8) {
            u32x4 v[8];
            float wi[8];
#pragma unroll
            for (int b = 0; b < 8; ++b) {
                const int i = i0 + b < k ? i0 + b : k - 1;
                // device-scope (sc1) load: served from the level all XCDs share, never from a line this XCD cached earlier
                v[b] = __builtin_amdgcn_raw_buffer_load_b128(out_rows, (uint32_t)rows[i] * row_bytes + (uint32_t)c * 2u, 0, 16);
                wi[b] = w[i];
            }
#pragma unroll
            for (int b = 0; b < 8; ++b) {
                if (i0 + b < k) {
#pragma unroll
                    for (int p = 0; p < 4; ++p) {
                        acc[2 * p] = fmaf(wi[b], __uint_as_float(v[b][p] << 16), acc[2 * p]);
                        acc[2 * p + 1] = fmaf(wi[b], __uint_as_float(v[b][p] & 0xffff0000u), acc[2 * p + 1]);
                    }
                }
            }
        }
        uint4 o;
        o.x = pack2_bf16(acc[0], acc[1]);
        o.y = pack2_bf16(acc[2], acc[3]);
        o.z = pack2_bf16(acc[4], acc[5]);
        o.w = pack2_bf16(acc[6], acc[7]);
        *reinterpret_cast<uint4*>(a.comb_y + (size_t)token * a.N + c) = o;
    }
}

template <int JBE, int IB, bool GATEUP, int STAGES, int XD, bool WNT>
__device__ __forceinline__ void tile_body_dma(const GemmArgs& a, const Tile& t, int nt, uint16_t* xs) {
    constexpr int NM = GATEUP ? 2 : 1;
    constexpr int NI = IB * NM;
    constexpr int BN = 4 * IB * 32;
    constexpr int NBUF = XD + 1;
    constexpr int BUF_BYTES = JBE * 32 * 128;
    const int tid = body_thread(), wave = tid / kWave, lane = tid % kWave;
    const int li = lane & 31, half = lane >> 5;
    const int K = a.K, N = a.N;
    const int KT = K / kBK;
    const int n0w = nt * BN + wave * (IB * 32);

    typedef WAddr<true, NM> WA;
    const uint16_t* wp[NI];
    static_for<NM>([&](auto m) {
        static_for<IB>([&](auto ib) { wp[m * IB + ib] = WA::base(a, t.e, n0w / 32 + ib, m, lane); });
    });
    // DMA q of this wavefront covers the 8 rows rg*8.., rg = 4q + wave: lane -> row rg*8 + lane/8,
    // LDS position lane%8, source chunk position ^ swz(row) with swz = ((lane>>3) ^ rg) & 7.
    const uint16_t* xp[JBE];
    static_for<JBE>([&](auto q) {
        const int rg = q * 4 + wave;
        const int chunk = (lane & 7) ^ (((lane >> 3) ^ rg) & 7);
        xp[q] = token_row(a, t.row0 + rg * 8 + (lane >> 3)) + chunk * 8;
    });
    const uint32_t lds0 = (uint32_t)(uintptr_t)xs;            // LDS byte address of the ring
    const uint32_t dma_dst = lds0 + wave * 1024;              // + q*4096 + buffer*BUF_BYTES
    // fragment reads: row j*32 + li, logical chunk 2s + half, swizzle (li ^ li>>3 ^ 4(j&1)) & 7
    const int sw0 = (li ^ (li >> 3)) & 7;
    int rd_off[2][4];   // [j parity][slot] byte offset inside a row
    static_for<2>([&](auto pj) {
        static_for<4>([&](auto s) { rd_off[pj][s] = (((2 * s + half) ^ (sw0 ^ (pj * 4))) & 7) * 16; });
    });
    const char* xs_b = reinterpret_cast<const char*>(xs) + li * 128;
    if (GATEUP && a.tables_in_lds) __syncthreads();   // the last look at tables that the ring is about to overwrite

    f32x16 acc[NI][JBE];
    static_for<NI>([&](auto i) {
        static_for<JBE>([&](auto j) {
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[i][j][v] = 0.0f;
        });
    });
    uint4 wreg[STAGES][NI][4];

    // The k loop is rotated per workgroup: logical step i reads physical step (i + rot) mod KT.  All
    // rows of a token tile at one k step are a whole multiple of 4 KiB apart when the row length is
    // (d = 4096, F = 14336, ...), so they sit in the same L2 channel; workgroups that run together on
    // an XCD (ids 8 apart) start two steps apart and so spread over the channels.  The sum over k
    // does not care about the order.  Steps past the last are re-reads of it (harmless).
    const int rot = __builtin_amdgcn_readfirstlane((int)(((blockIdx.x >> 3) * (unsigned)t.rot_mul) % (unsigned)KT));
    auto phys = [&](int i) {
        int p = (i < KT ? i : KT - 1) + rot;
        return p >= KT ? p - KT : p;
    };
    auto load_w = [&](int kt, auto st) {
        const int kc = phys(kt);
        static_for<NI>([&](auto i) {
            static_for<4>([&](auto s) {
                wreg[st][i][s] = load_w16<WNT>(wp[i] + (size_t)kc * WA::kStep + s * WA::sStep);
            });
        });
    };
    auto dma_x = [&](int kt, int buf) {
        const int kc = phys(kt);
        static_for<JBE>([&](auto q) { lds_dma16(xp[q] + (size_t)kc * kBK, dma_dst + buf * BUF_BYTES + q * 4096); });
    };
    auto frag = [&](int buf, auto j, auto s) {
        return *reinterpret_cast<const bf16x8*>(xs_b + buf * BUF_BYTES + j * 4096 + rd_off[j & 1][s]);
    };
    // The token tile of step kt+2 (not kt+1) is awaited at the end of step kt, so a tile is
    // visible to every wavefront one whole step before it is used; the first fragments of step
    // kt+1 can then be read during the last slot of step kt and the MFMAs of the next step
    // start right behind the barrier instead of behind an LDS round trip.
    // The DMA instructions of a step are dealt over its MFMA groups (group g takes q = g, g+NG,
    // ...) behind that group's weight load: the CU's one address unit needs 16 cycles per
    // 64-lane 16-byte access, and a burst of JBE of them from all four wavefronts at once would
    // hold every instruction stream (and so the MFMAs) for several hundred cycles per step.
    // Loads this wavefront issues after its last DMA of step kt+2-XD and before the end of step
    // kt: the weight loads of the groups behind that DMA, then (XD-2) whole steps.
    static_assert(XD >= 2, "needs the tile of step kt+2 in flight during step kt");
    constexpr int NG = 4 * NI;                                   // MFMA groups = weight loads per step
    constexpr int G_LAST = (JBE < NG ? JBE : NG) - 1;            // last group that issues a DMA
    constexpr int VM_AFTER = (NG - 1 - G_LAST) + (XD - 2) * (NG + JBE);

    bf16x8 xnext[JBE];   // slot-0 fragments of the next step
    // One wavefront per SIMD: while it issues a run of memory instructions nothing feeds the
    // matrix pipe, which holds one MFMA (32 cycles) ahead at most.  So the memory instructions
    // of a slot (per group one weight load and the group's share of the token-tile DMAs, JBE
    // fragment reads for the next slot) are dealt singly between its NI*JBE MFMAs: fragment jj of the next slot
    // behind MFMA jj*NI + NI-1, i.e. still NI*JBE - jj*(NI-1) - NI + 1 >= JBE MFMAs before its
    // use.  (Issuing them as one run at the head of each group measured 5 % slower.)
    auto step = [&](int kt, auto u) {
        const int buf = kt % NBUF;
        constexpr int wst = (u + STAGES - 1) % STAGES;
        const int kw = phys(kt + STAGES - 1);
        const int kx = phys(kt + XD);
        const uint32_t dst = dma_dst + ((kt + XD) % NBUF) * BUF_BYTES;   // the buffer read in step kt-1: free since that step's barrier
        bf16x8 xf[2][JBE];
        static_for<JBE>([&](auto j) { xf[0][j] = xnext[j]; });
        __builtin_amdgcn_sched_barrier(0);
        static_for<4>([&](auto s) {
            static_for<NI>([&](auto i) {
                const bf16x8 wf = __builtin_bit_cast(bf16x8, wreg[u % STAGES][i][s]);
                static_for<JBE>([&](auto j) {
                    acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(wf, xf[s & 1][j], acc[i][j], 0, 0, 0);
                    constexpr int p = i * JBE + j;               // position of this MFMA in the slot
                    constexpr int jd = JBE > 2 ? 2 : JBE - 1;    // the group's DMA goes behind this MFMA
                    if constexpr (j == 0)
                        wreg[wst][i][s] = load_w16<WNT>(wp[i] + (size_t)kw * WA::kStep + s * WA::sStep);
                    if constexpr (j == jd) {
                        static_for<JBE>([&](auto q) {
                            if constexpr (q % NG == s * NI + i) lds_dma16(xp[q] + (size_t)kx * kBK, dst + q * 4096);
                        });
                    }
                    if constexpr (p % NI == NI - 1) {
                        constexpr int jj = p / NI;
                        if constexpr (s < 3)
                            xf[(s + 1) & 1][jj] = frag(buf, std::integral_constant<int, jj>{}, std::integral_constant<int, (s + 1) % 4>{});
                        else   // last slot: slot-0 fragments of the next step (its tile is visible since the previous barrier)
                            xnext[jj] = frag((kt + 1) % NBUF, std::integral_constant<int, jj>{}, std::integral_constant<int, 0>{});
                    }
                    __builtin_amdgcn_sched_barrier(0);
                });
            });
        });
        wait_vmcnt<VM_AFTER>();   // this wavefront's share of the token tile of step kt+2 has landed
        __syncthreads();
    };

    // prologue: token tiles of steps 0..XD-1, weights of steps 0..STAGES-2; tiles 0 and 1 complete
    static_for<XD>([&](auto q) { dma_x(q, q % NBUF); });
    static_for<STAGES - 1>([&](auto st) { load_w(st, st); });
    wait_vmcnt<(XD - 2) * JBE + (STAGES - 1) * NI * 4>();
    __syncthreads();
    static_for<JBE>([&](auto j) { xnext[j] = frag(0, j, std::integral_constant<int, 0>{}); });

    constexpr int UNR = STAGES;
    int kt = 0;
    for (; kt + UNR <= KT; kt += UNR) static_for<UNR>([&](auto u) { step(kt + u, u); });
    static_for<UNR>([&](auto u) {
        if (kt + u < KT) step(kt + u, u);
    });
    wait_vmcnt<0>();   // nothing of this workgroup may still be writing LDS when it retires

    if constexpr (!GATEUP) {
        if (a.comb_arrive != nullptr) {
            static_for<IB>([&](auto ib) {
                static_for<JBE>([&](auto j) {
                    const int tr = j * 32 + li;
                    const bool live = tr < t.rows;
                    store_block<GATEUP, true>(acc[ib][j], acc[ib][j], a.Out + (size_t)(t.row0 + (live ? tr : 0)) * a.ldo,
                                              n0w + ib * 32, half, N, live);
                });
            });
            return fused_combine<IB>(a, t, nt, xs);
        }
    }
    store_tile<GATEUP, IB, JBE, NI>(acc, a, t, nt, xs);
}

// =============================================================================================
// rows_body: the weights go through LDS as well.  Every tile of row-major weights and the single-block
// tiles of packed ones.
// Row-major: a fragment read straight into registers touches 32 rows, 16 bytes each, i.e. 64 L1
// accesses per instruction, which is what bounded that form (5.0 TB/s at the Mixtral shape, 512
// tokens).  A DMA instruction takes 8 rows x 128 bytes instead, whole lines, and the wavefront
// reads its fragments back from LDS (its own rows only: no other wavefront waits for them).
// Packed: the load instructions are the same 1 KiB each, but no register is held by a load in flight
// and no MFMA waits for one: weights and tokens are awaited together, once a step.  Bound by HBM; us,
// tile_body_dma / rows_body: Mixtral shape 512 tokens gate+up 346 / 337, Qwen2-MoE shape 512 tokens 401 / 391
// and down 244 / 229, 256 experts (DeepSeek-V3 widths) down 1340 / 1286 at 512 tokens (5.8 TB/s), 1632 / 1602
// at 4096.
// Ring of NB buffers, each one k step: JBE * 4 KiB of tokens and, per wavefront, NI * 4 KiB of
// weights; the loads of step kt + 2 are issued in step kt and awaited at the end of step kt + 1, with
// two buffers those of step kt + 1 (taller than 160 rows with two weight blocks in all, where a step's
// MFMAs are long enough to cover one step of latency).  LDS traffic per step at
// 256 rows: 224 KiB = 1792 of the step's 2048 MFMA cycles.
// `deep`: three steps ahead where 160 KiB hold four buffers (up to 192 rows with one weight block, 64 with two).
// Two steps of one weight block are 32 KiB of weights in flight per CU.  That is enough while every CU streams; where the
// last round of a launch leaves CUs idle the rest could take more from HBM, and it is not: down projection, us, weights to
// registers (48 KiB ahead) / two steps / three: Mixtral shape 4 tokens 101 / 119 / 100, 7 tokens under skew 1.6 98 / 120 / 97;
// 8 experts of 6144 x 16384, 8 tokens 243 / 265 / 242, 200 tokens 311 / 320 / 310; DeepSeek-V3 widths 2 tokens 83 / 87 / 82;
// Qwen2-MoE shape 2 tokens 50 / 54 / 49.  At whole rounds three steps are 0-2 % behind two (Mixtral shape, 16 tokens,
// 141 / 144 with three throughout), and with two weight blocks too (Qwen2-MoE shape, 150 tokens, down 210 / 212; 60 experts
// of 2048 x 1408, 40 tokens, gate+up 116 / 117), except where half of the CUs or fewer have work (8 experts of 4096 x 1024,
// 8 tokens, gate+up: registers 45.6, two steps 47.0, three 45.9).
// Row-major, weights straight to registers and now, us, gate+up / down projection: Mixtral shape 47
// tokens 401 / 230 -> 307 / 151, 512 tokens 470 / 270 -> 343 / 212 (5.5 TB/s of weights), 4096 tokens
// 1955 / 1305 -> 1690 / 940; 256 experts of DeepSeek-V3's widths, 512 tokens 3390 / 1790 -> 2188 / 1233 (6.9 TB/s).
// Against the packed layout: 0.99-1.08x its time up to 128 rows per expert on the Mixtral shape, most behind where a tile
// has two buffers here and registers there: gate+up 1.12x at 192 rows per expert, down projection 1.25x at 256, 1.13x at 1024.
// =============================================================================================
constexpr int kLdsBytes = 160 * 1024;
constexpr int rows_buffer_bytes(int jbe, int ni) { return jbe * 4096 + ni * 16384; }
constexpr int rows_buffers(int jbe, int ni) {
    const int n = kLdsBytes / rows_buffer_bytes(jbe, ni);
    return n > 4 ? 4 : n;
}
// Tallest single-block tile of packed weights (32-row blocks) that takes rows_body: three buffers fit.
// With two (gate and up, or two weight blocks, beyond 160 rows) the register path of tile_body_dma is
// the better one (us, rows_body / tile_body_dma: Mixtral shape 1024 tokens, down projection 391 / 316).
constexpr int rows_max(int ni) { return ni >= 2 ? 5 : 8; }
// LDS that tiles of up to max_jbe 32-row blocks need
constexpr int rows_lds(int max_jbe, int ni) {
    int most = 0;
    for (int j = 1; j <= max_jbe; ++j) {
        const int b = rows_buffer_bytes(j, ni) * rows_buffers(j, ni);
        most = b > most ? b : most;
    }
    return most;
}
template <int JBE, int IB, bool GATEUP, bool PACKED, bool WNT>
__device__ __forceinline__ void rows_body(const GemmArgs& a, const Tile& t, int nt, bool deep, uint16_t* xs) {
    constexpr int NM = GATEUP ? 2 : 1;
    constexpr int NI = IB * NM;
    constexpr int BN = 4 * IB * 32;
    constexpr int NB = rows_buffers(JBE, NI);
    constexpr int XM = NB - 1;                          // steps the loads can run ahead
    constexpr int XD = XM > 2 ? 2 : XM;                 // steps they do, unless `deep`
    const int ahead = deep ? XM : XD;
    constexpr int X_BYTES = JBE * 4096;                 // token tile of a step
    constexpr int BUF = X_BYTES + 4 * NI * 4096;
    constexpr int LPS = JBE + 4 * NI;                   // loads per wavefront and step
    const int tid = body_thread(), lane = tid % kWave;
    const int wave = __builtin_amdgcn_readfirstlane(tid / kWave);
    const int li = lane & 31, half = lane >> 5;
    const int K = a.K, N = a.N;
    const int KT = K / kBK;
    const int n0w = nt * BN + wave * (IB * 32);

    // Packed weights: DMA g of a 32-row block is slot g of the step, 1 KiB in a row, in fragment order.
    // Row-major weights: DMA g of a 32-row block covers rows 8 g .. 8 g + 7: lane -> row 8 g + lane / 8, position
    // lane % 8 of the LDS row, source chunk position ^ swizzle(row) (the swizzle of the token rows).
    typedef WAddr<PACKED, NM> WA;
    const uint16_t* wp[NI];                             // wave-uniform
    static_for<NM>([&](auto m) {
        static_for<IB>([&](auto ib) { wp[m * IB + ib] = WA::block(a, t.e, n0w / 32 + ib, m); });
    });
    uint32_t wo[4];
    static_for<4>([&](auto g) {
        const int chunk = (lane & 7) ^ (((lane >> 3) ^ g) & 7);
        wo[g] = PACKED ? (uint32_t)(g * 1024 + lane * 16)
                       : (uint32_t)(g * 8 + (lane >> 3)) * (uint32_t)K * 2u + (uint32_t)chunk * 16u;
    });
    // Tokens: DMA q covers the rows rg * 8 .., rg = 4 q + wave, as in tile_body_dma.
    uint32_t xo[JBE];
    static_for<JBE>([&](auto q) {
        const int rg = q * 4 + wave;
        const int chunk = (lane & 7) ^ (((lane >> 3) ^ rg) & 7);
        xo[q] = token_row_bytes(a, t.row0 + rg * 8 + (lane >> 3)) + (uint32_t)chunk * 16u;
    });
    const uint32_t lds0 = (uint32_t)(uintptr_t)xs;
    const uint32_t x_dst = lds0 + wave * 1024;                       // + q * 4096 + buffer * BUF
    const uint32_t w_dst = lds0 + X_BYTES + wave * (NI * 4096);      // + i * 4096 + g * 1024 + buffer * BUF
    const int sw0 = (li ^ (li >> 3)) & 7;
    int rd_off[2][4];   // [j parity][slot] byte offset inside a row; weight rows use parity 0
    static_for<2>([&](auto pj) {
        static_for<4>([&](auto s) { rd_off[pj][s] = (((2 * s + half) ^ (sw0 ^ (pj * 4))) & 7) * 16; });
    });
    const char* xs_b = reinterpret_cast<const char*>(xs) + li * 128;
    const char* ws_b = reinterpret_cast<const char*>(xs) + X_BYTES + wave * (NI * 4096) + (PACKED ? lane * 16 : li * 128);
    if (GATEUP && PACKED && a.tables_in_lds) __syncthreads();   // the last look at tables that the ring is about to overwrite

    f32x16 acc[NI][JBE];
    static_for<NI>([&](auto i) {
        static_for<JBE>([&](auto j) {
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[i][j][v] = 0.0f;
        });
    });
    const int rot = __builtin_amdgcn_readfirstlane((int)(((blockIdx.x >> 3) * (unsigned)t.rot_mul) % (unsigned)KT));   // see tile_body_dma
    auto phys = [&](int i) {
        int p = (i < KT ? i : KT - 1) + rot;
        return p >= KT ? p - KT : p;
    };
    // load l of a step: the weight rows first (they come from farthest away), then the token rows
    auto load = [&](auto l, int kc, uint32_t buf) {
        const uint32_t kb = (uint32_t)kc * (kBK * 2);
        if constexpr (l < 4 * NI) {
            constexpr int i = l / 4, g = l % 4;
            lds_dma16_at<WNT>(reinterpret_cast<const char*>(wp[i]) + (PACKED ? (uint32_t)kc * (WA::kStep * 2) : kb), wo[g], w_dst + buf + i * 4096 + g * 1024);
        } else {
            constexpr int q = l - 4 * NI;
            lds_dma16_at<false>(reinterpret_cast<const char*>(a.X) + kb, xo[q], x_dst + buf + q * 4096);
        }
    };
    auto xfrag = [&](int buf, auto j, auto s) {
        return *reinterpret_cast<const bf16x8*>(xs_b + buf + j * 4096 + rd_off[j & 1][s]);
    };
    auto wfrag = [&](int buf, auto i, auto s) {
        return *reinterpret_cast<const bf16x8*>(ws_b + buf + i * 4096 + (PACKED ? s * 1024 : rd_off[0][s]));
    };
    // The step's loads are dealt singly between its MFMAs (one wavefront per SIMD: a run of memory
    // instructions would idle the matrix pipe): over the whole step when they have a step to spare,
    // over its first half when they are awaited at its end.
    constexpr int MF = 4 * NI * JBE;
    constexpr int SPREAD = XD > 1 ? MF : (MF + 1) / 2;
    // All but the last `ahead` - 1 steps' loads have landed (they return in issue order).
    auto landed = [&] {
        if (XM > XD && deep)
            wait_vmcnt<(XM - 1) * LPS>();
        else
            wait_vmcnt<(XD - 1) * LPS>();
    };
    auto step = [&](int kt) {
        const int buf = (kt % NB) * BUF;
        const uint32_t nbuf = (uint32_t)((kt + ahead) % NB) * BUF;    // read in step kt - 1 or before: free since that step's barrier
        const int kc = phys(kt + ahead);
        bf16x8 xf[2][JBE], wf[2][NI];
        static_for<NI>([&](auto i) { wf[0][i] = wfrag(buf, i, std::integral_constant<int, 0>{}); });
        static_for<JBE>([&](auto j) { xf[0][j] = xfrag(buf, j, std::integral_constant<int, 0>{}); });
        __builtin_amdgcn_sched_barrier(0);
        static_for<4>([&](auto s) {
            static_for<NI>([&](auto i) {
                static_for<JBE>([&](auto j) {
                    acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(wf[s & 1][i], xf[s & 1][j], acc[i][j], 0, 0, 0);
                    constexpr int p = i * JBE + j, at = s * NI * JBE + p;
                    static_for<LPS>([&](auto l) {
                        if constexpr (l * SPREAD / LPS == at) load(l, kc, nbuf);
                    });
                    if constexpr (s < 3) {     // next slot's fragments: the weights behind the first MFMA, the tokens spread
                        if constexpr (p == 0)
                            static_for<NI>([&](auto n) { wf[(s + 1) & 1][n] = wfrag(buf, n, std::integral_constant<int, (s + 1) % 4>{}); });
                        if constexpr (p % NI == NI - 1) {
                            constexpr int jj = p / NI;
                            xf[(s + 1) & 1][jj] = xfrag(buf, std::integral_constant<int, jj>{}, std::integral_constant<int, (s + 1) % 4>{});
                        }
                    }
                    __builtin_amdgcn_sched_barrier(0);
                });
            });
        });
        landed();      // everything of step kt + 1
        __syncthreads();
    };
    // Nothing is outstanding here.  The wait tells the compiler so: where it lays this code out behind another body's, it
    // takes that body's last loads for outstanding and waits for them in the loop, which empties the ring at every
    // step (down projection, two weight blocks, 160 rows: Qwen2-MoE shape, 1000 tokens 245 -> 267 us).
    wait_vmcnt<0>();
    static_for<XM>([&](auto q) {
        if (q < XD || deep) {
            const int kc = phys(q);
            static_for<LPS>([&](auto l) { load(l, kc, (uint32_t)(q % NB) * BUF); });
        }
    });
    landed();
    __syncthreads();
    for (int kt = 0; kt < KT; ++kt) step(kt);
    wait_vmcnt<0>();   // nothing of this workgroup may still be writing LDS when it retires

    if constexpr (!GATEUP && PACKED) {
        if (a.comb_arrive != nullptr) {
            static_for<IB>([&](auto ib) {
                static_for<JBE>([&](auto j) {
                    const int tr = j * 32 + li;
                    const bool live = tr < t.rows;
                    store_block<GATEUP, true>(acc[ib][j], acc[ib][j], a.Out + (size_t)(t.row0 + (live ? tr : 0)) * a.ldo,
                                              n0w + ib * 32, half, N, live);
                });
            });
            return fused_combine<IB>(a, t, nt, xs);
        }
    }
    store_tile<GATEUP, IB, JBE, NI>(acc, a, t, nt, xs);
}

// MAXJ: tallest tile handed in, in 32-row blocks.
template <int IB, bool GATEUP, bool PACKED, bool WNT, int MAXJ>
__device__ __forceinline__ void rows_dispatch(const GemmArgs& a, const Tile& t, int nt, bool deep, uint16_t* xs) {
    switch ((t.rows + 31) / 32) {
        case 1: return rows_body<1, IB, GATEUP, PACKED, WNT>(a, t, nt, deep, xs);
        case 2: if constexpr (MAXJ >= 2) return rows_body<2, IB, GATEUP, PACKED, WNT>(a, t, nt, deep, xs); break;
        case 3: if constexpr (MAXJ >= 3) return rows_body<3, IB, GATEUP, PACKED, WNT>(a, t, nt, deep, xs); break;
        case 4: if constexpr (MAXJ >= 4) return rows_body<4, IB, GATEUP, PACKED, WNT>(a, t, nt, deep, xs); break;
        case 5: if constexpr (MAXJ >= 5) return rows_body<5, IB, GATEUP, PACKED, WNT>(a, t, nt, deep, xs); break;
        case 6: if constexpr (MAXJ >= 6) return rows_body<6, IB, GATEUP, PACKED, WNT>(a, t, nt, deep, xs); break;
        case 7: if constexpr (MAXJ >= 7) return rows_body<7, IB, GATEUP, PACKED, WNT>(a, t, nt, deep, xs); break;
        default: if constexpr (MAXJ >= 8) return rows_body<8, IB, GATEUP, PACKED, WNT>(a, t, nt, deep, xs);
    }
}

// The dynamic-height kernel with the LDS-DMA token tile (packed weights).  LDS: (XD+1) buffers of up to 32 KiB.
// MINJ: shortest tile handed in, in 32-row blocks (no body is compiled for shorter ones).
template <int IB, bool GATEUP, bool WNT, bool HALF, int MINJ = 1>
__device__ __forceinline__ void dma_dispatch(const GemmArgs& a, const Tile& t, int nt, uint16_t* xs) {
    constexpr int NI = IB * (GATEUP ? 2 : 1);
    constexpr int SD = NI >= 4 ? 3 : 4;
    if constexpr (HALF) {   // blocks of at most 128 rows, two workgroups per CU: register budget 256 per wavefront
        switch ((t.rows + 31) / 32) {
            case 1: return tile_body_dma<1, IB, GATEUP, 3, 3, WNT>(a, t, nt, xs);
            case 2: return tile_body_dma<2, IB, GATEUP, 3, 3, WNT>(a, t, nt, xs);
            case 3: return tile_body_dma<3, IB, GATEUP, 2, 3, WNT>(a, t, nt, xs);
            default: return tile_body_dma<4, IB, GATEUP, 2, 3, WNT>(a, t, nt, xs);
        }
    }
    switch ((t.rows + 31) / 32) {
        case 1: if constexpr (MINJ <= 1) return tile_body_dma<1, IB, GATEUP, SD, 3, WNT>(a, t, nt, xs); break;
        case 2: if constexpr (MINJ <= 2) return tile_body_dma<2, IB, GATEUP, SD, 3, WNT>(a, t, nt, xs); break;
        case 3: if constexpr (MINJ <= 3) return tile_body_dma<3, IB, GATEUP, SD, 3, WNT>(a, t, nt, xs); break;
        case 4: if constexpr (MINJ <= 4) return tile_body_dma<4, IB, GATEUP, SD, 3, WNT>(a, t, nt, xs); break;
        case 5: if constexpr (MINJ <= 5) return tile_body_dma<5, IB, GATEUP, NI >= 4 ? 2 : SD, 3, WNT>(a, t, nt, xs); break;
        case 6: if constexpr (MINJ <= 6) return tile_body_dma<6, IB, GATEUP, NI >= 4 ? 2 : SD, 3, WNT>(a, t, nt, xs); break;
        case 7: return tile_body_dma<7, IB, GATEUP, 3, 3, WNT>(a, t, nt, xs);
        default: return tile_body_dma<8, IB, GATEUP, 3, 3, WNT>(a, t, nt, xs);
    }
}

// The regime is a property of the EXPERT, not of the launch: under routing skew a few experts
// hold thousands of rows while most hold a handful.  This kernel decides per block; both regimes
// run the LDS-DMA body.  An expert that fits one block streams its weights once: non-temporal
// weight loads if WNT, k loop rotated against its XCD neighbours.  An expert that spans several
// row tiles shares its weight panels through L2: cached weight loads, k walked in step, its row
// tiles launched side by side.
//
// Last round (IB = 2 only).  The grid runs in rounds of `slots` workgroups, one per CU.  With
// two weight blocks per wavefront a projection has few, heavy workgroups (Mixtral shape, down
// projection at T=2048: 320 = 1.25 rounds); when the last round is at most half full, each of
// its workgroups is replaced by two that take one 128-feature half each with the IB = 1 body,
// so the round lasts about half as long and uses twice the CUs.  Only when at most one full
// round precedes it: with many rounds the workgroups do not end together, there is no common
// "last round" to shorten, and the less efficient halves cost more than they gain (measured:
// -10 % at T=2048, +3..5 % at T=4096 and T=8192 without this condition).
//
// mixed_assign: what workgroup w of a tile_kernel_mixed launch works on.  Integer arithmetic on the launch
// arguments and the schedule arrays only, callable on the host as well: the CPU tests enumerate
// whole launches with it (host copies of the arrays) and check that every (row, feature tile) of
// every expert is covered exactly once in each launch order.
struct MixedWork {
    int e, row0, rows, n_e;   // expert, first expert-contiguous row, rows of this workgroup, rows of the expert
    int nt;                   // feature tile: of IB * 128 features, or of 128 when `halves`
    bool halves;              // IB == 2 down projection: one 128-feature half of a tile of the split last round (IB = 1 body)
    bool chunked;             // the launch is dealt to the XCDs in runs of consecutive positions
    bool stream;              // results stored non-temporally (store_tile)
    bool deep;                // loads run three steps ahead where the LDS ring holds four (rows_body)
};
template <int IB, bool GATEUP>
__host__ __device__ inline bool mixed_assign(const GemmArgs& a, const int wg, MixedWork& m) {
    int tile, nt;
    bool halves = false, dealt = false, units = false;
    const int32_t* blist = a.blocks;   // Algorithm 1's order unless the two classes are dealt (below)
    const int blocks = *a.num_blocks, multi = *a.num_multi;
    if (blocks == 0) return false;     // no expert has rows: below, a run of the whole launch would have length 0
    const int total = blocks * a.n_tiles_n;
    int split_from = total;            // first position (in two-block tiles) of a split last round
    {
        int w = wg, sub = 0;
        bool split_round = false;
        if constexpr (IB == 2 && !GATEUP) {
            if (a.slots > 0) {
                const int full = total / a.slots * a.slots, rem = total - full;
                split_round = rem > 0 && 2 * rem <= a.slots && full <= a.slots;
                if (split_round) split_from = full;
                if (split_round && w >= full) {
                    const int h = w - full;
                    w = full + (h >> 1);
                    sub = h & 1;
                    halves = true;
                }
            }
        }
        // Heavy and light blocks dealt evenly over the launch.  With a.num_heavy the block list
        // holds the blocks of multi-block experts first (their workgroups are bound by the matrix
        // cores and leave HBM mostly alone), then the single-block experts (bound by the weight
        // stream).  Launched in that order, or in expert order under routing skew, the chip runs
        // stretches of one kind only: all CUs compute while HBM idles, then all CUs stream and
        // share the bandwidth.  Position p of the launch therefore takes the next unit of the
        // class that a proportional (Bresenham) merge puts there, so that at any time the resident
        // workgroups are a mix in the launch's own proportion: the streaming ones then have the
        // memory system to themselves.  The unit is 8 consecutive ids where the feature-tile count
        // is a multiple of 8 (id % 8, the XCD, and the side-by-side order below are kept), else
        // one block.  Both classes keep their ascending expert order, so the light experts' weights
        // are still read in address order.  Uniform routing has one class only: nothing moves.
        // Dealing costs the heavy class: row tiles that share a weight panel no longer start
        // together (a few percent of their time, whatever the light class holds), and what it
        // gains grows with the light class's share of the launch.  It is therefore done only
        // when the single-block experts number at least 2/5 of the multi-block experts' blocks
        // (measured at T=4096: DeepSeek-V3 shape, 173 / 65 / 31 light against ~130 heavy blocks:
        // -9.6 %, -5.6 %, -1.8 %; Qwen2-MoE shape, 40 / 45 / 32 against ~130: +2.6 %, +2.8 %, +5.5 %).
        bool deal = false;
        int dealU = 1, hu = 0, tu = 0;
        if (a.num_heavy != nullptr && !split_round) {
            const int hb = *a.num_heavy, lb = blocks - hb;
            dealU = (a.n_tiles_n & 7) == 0 ? 8 : a.n_tiles_n;
            hu = hb * a.n_tiles_n / dealU;
            tu = total / dealU;
            deal = hu > 0 && tu > hu && (a.deal_always || 5 * lb >= 2 * hb);
        }
        // Runs of consecutive positions per XCD.  The hardware deals workgroup id to XCD id % 8, so the q-th workgroup of an XCD takes
        // position q % unit of that XCD's next run, and the XCDs take the runs in turn: at any time the chip works on about the same
        // stretch of the launch as without them, but what runs on an XCD at once belongs together.  The feature tiles of a
        // single-block expert then fetch its token tile into one L2 instead of eight (down projection: the h tile of an expert is read
        // by d/128 workgroups and makes up half of what a CU loads), and the row tiles and panels of a multi-block expert meet
        // there whatever the feature-tile count (the order further down needs a multiple of 8).  The positions after the last eight
        // whole runs are cut into eight others.
        //   By the rule: if no expert has more than one block; with blocks of multi-block experts from few_from (they are a sixteenth of all) or
        // multi_from workgroups on, the latter unless there are too many light blocks beside them (mixed_launch_shape).
        // Not when heavy and light blocks are dealt (below).  us, without / with: gate+up 60 experts of 2048 x 1408, 4000 tokens
        // (11 tiles) 334 / 296, 128 of 4096 x 1536, 4096 tokens (12) 867 / 823, Qwen2-MoE shape 4096 tokens (20) 1066 / 1023; down
        // projection of the first (8) 193 / 157, 32 experts of 2880 x 2880, 4000 tokens (12) 310 / 286, Qwen2-MoE shape at skew 1 (14) 620 / 596.
        // A run is half of what an XCD runs at once.  Whole ones share no more (Qwen2-MoE shape, 1024 tokens, down projection 240 / 238 with half;
        // 256 experts, 4096 tokens 1452 / 1415), and under skew tall tiles of one expert crowd an XCD for longer (Qwen2-MoE shape, skew 2,
        // 200 tokens, down projection without runs 122 / whole 132 / half 122; 4096 tokens at skew 1, gate+up 1145 / 1155 / 1114).  One contiguous
        // eighth of the launch per XCD: the same for single-block experts, 6-17 % behind no runs at all where one XCD gets the heavy ones.
        bool runs = !split_round && !deal && a.chunk != 0;
        if (runs && a.chunk == 2)
            runs = multi == 0 || (16 * multi <= blocks ? total >= a.few_from : total >= a.multi_from && 5 * (blocks - multi) <= a.light * multi);
        if (runs) {
            const int U = a.eighths && multi == 0 ? total : a.unit, q = w >> 3, x = w & 7, group = q / U;
            const int groups = total <= 16 * U ? 0 : total / (8 * U);   // one round: an eighth each
            if (group < groups) {
                w = (group * 8 + x) * U + (q - group * U);
            } else {
                const int done = groups * 8 * U, rest = total - done, per = (rest + 7) >> 3, r = q - groups * U;
                if (r >= per || x * per + r >= rest) return false;
                w = done + x * per + r;
            }
            units = true;
        }
        if (w >= total) return false;
        if (deal) {
            blist = a.blocks_mix;
            const int p = w / dealU, r = w - p * dealU;
            // heavy units among positions [0, p): floor(p * hu / tu); position p is heavy iff that count steps at p
            const long long before = (long long)p * hu / tu, upto = (long long)(p + 1) * hu / tu;
            const int unit = upto > before ? (int)before : hu + (p - (int)before);
            w = unit * dealU + r;
            dealt = dealU != 8;   // whole units of 8 ids keep an expert's workgroups on the XCDs the order below assumes
        }
        tile = w / a.n_tiles_n;
        nt = w - tile * a.n_tiles_n;
        if (halves) nt = 2 * nt + sub;   // index of the 128-feature tile the IB = 1 body works on
    }
    // Row tiles of one expert side by side.  The workgroups of an expert with n row tiles are a
    // contiguous span of n * n_tiles_n launch positions; the hardware deals workgroup id to XCD
    // id % 8, so the positions of the span that are 8 apart (one "class", position % 8) run on one
    // XCD, one after the other.  In plain tile-major order the n workgroups that read the same
    // weight panel are n_tiles_n positions apart: they start microseconds apart, on whatever XCD
    // that distance leads to, and an XCD's 4 MiB of L2 hold only about three k steps of its 32
    // workgroups' streams, so each of them fetches the panel from beyond L2 for itself.  Inside
    // the span the order is therefore (feature tile, row tile) per class: the n row tiles of a
    // panel are consecutive positions of one class, i.e. consecutive workgroups of one XCD, start
    // together and walk k in step.  A class of c positions holds c / n whole panels; the c % n
    // positions left over in each class take the remaining panels' tiles in turn (those panels are
    // spread over several XCDs; none when n_tiles_n is a multiple of 8).  A short last tile (a
    // different, faster body) would not stay in step anyway: those go to the end of the span.
    // (Mixtral shape, T=4096: layer -3 %; T=8192 -2 %; no effect on single-tile experts.)
    // The schedule entry is read once: the look-ups (block count, entry, expert offsets, for
    // the gate+up projection the source row) are dependent loads in front of the block's first
    // weight and tile loads, each worth several hundred nanoseconds of a ~100 us block.
    if (tile >= blocks) return false;
    const int bm = a.M < 256 ? a.M : 256;              // rows per schedule entry
    const int e = blist[2 * tile];
    const int r_in = blist[2 * tile + 1];
    const int seg0 = a.offsets[e];
    const int n_e = a.offsets[e + 1] - seg0;
    const int n = (n_e + bm - 1) / bm;                 // row tiles (schedule entries) of this expert
    int ti = r_in / bm;                                // which of them this workgroup is
    // see below; a.even: 0 never, 1 experts of up to three row tiles, 2 those while the launch is at most two rounds, 3 always
    const bool even = a.even == 3 || (n <= 3 && (a.even == 1 || (a.even == 2 && total <= 2 * a.slots)));
    // An expert whose span reaches into a split last round keeps the plain order in all of its
    // workgroups, the halves and the whole tiles before them alike: the two orders number the
    // positions of a span differently, so one span must use one of them throughout.
    const bool in_split = (tile - ti + n) * a.n_tiles_n > split_from;
    if (a.sib && !in_split && !dealt && n >= 2) {
        auto body = [](int rows) { const int c = (rows + 31) >> 5; return c > 7 ? 8 : c; };
        // tiles that run the same body as the first one (all of them when the rows are dealt evenly)
        const int nf = (even || body(n_e - (n - 1) * bm) == body(bm)) ? n : n - 1;
        const int l = ti * a.n_tiles_n + nt;           // position inside the expert's span
        const int span = nf * a.n_tiles_n;             // positions of the tiles that keep pace with each other
        if (l >= span) {
            ti = n - 1;
            nt = l - span;
        } else if (units) {
            nt = l / nf;
            ti = l - nt * nf;
        } else {
            const int cls = l & 7, j = l >> 3;         // class of the position, index inside the class
            int left_before = 0, whole = 0, mine = 0;
#pragma unroll
            for (int c = 0; c < 8; ++c) {
                const int positions = (span - c + 7) >> 3, panels = positions / nf;   // non-increasing in c
                if (c < cls) left_before += positions - panels * nf;
                if (c == cls) mine = panels;
                whole += panels;
            }
            if (j < mine * nf) {
                // the p-th whole panel of every class: panels p * 8 + class (at any time the XCDs work on neighbouring panels)
                nt = (j / nf) * 8 + cls;
                ti = j % nf;
            } else {
                const int m = left_before + (j - mine * nf);
                nt = whole + m / nf;
                ti = m % nf;
            }
        }
    }
    // Rows of a multi-tile expert dealt evenly over its n schedule entries, in whole 32-row blocks:
    // Algorithm 1 gives 1040 rows as 4 x 256 + 16, and the 16-row tile streams a whole weight
    // panel for 1/16 of the MFMA work, eight times faster through k than its siblings, so it
    // shares nothing with them (1040 instead of 1024 rows per expert cost +8 % on gate+up and
    // +15 % on the down projection).  5 x 224 (4 x 224 + 144) is the same number of 32-row MFMA
    // blocks, ceil(n_e / 32), in tiles that run at about the same pace.  Which rows a workgroup
    // computes does not change any row's result.  The CU time of the two divisions is about the
    // same (a 16-row tile costs a third of a full one); what differs is how the launch ends.
    // Experts of two or three row tiles, where the short tile's extra pass over the weight panel
    // is a third to a half of the expert's weight traffic, are dealt evenly (Mixtral shape T=1024
    // -4 %, T=2048 -5 %, Qwen2-MoE shape T=4096 -2 %); with four tiles or more the 224-row bodies
    // cost what the shared panel saves (gate+up at T=4096 +1.7 %).  Down projection (few, heavy
    // workgroups): only while the launch is at most two rounds, where equal tiles end together
    // (T=2048: 538 -> 455 us); with more rounds the quick short tiles fill the gaps better
    // (T=4096: 864 against 915 us).
    int row_in = ti * bm, rows = bm;
    if (even && n >= 2) {
        const int per = (((n_e + n - 1) / n) + 31) & ~31;   // <= 256
        row_in = ti * per;
        rows = per;
    }
    rows = (n_e - row_in) < rows ? (n_e - row_in) : rows;
    if (rows <= 0) return false;                            // (n >= 8 only: the rounding can empty the last entry)
    m.e = e;
    m.row0 = seg0 + row_in;
    m.rows = rows;
    m.n_e = n_e;
    m.nt = nt;
    m.halves = halves;
    m.chunked = units;
    m.stream = a.stream != 0 && n_e <= a.M && (!GATEUP || (multi == 0 && (long long)n_e * a.E <= 2ll * a.R && (a.P != nullptr || n_e <= 160)));
    m.deep = a.cus > 0 && (IB * (GATEUP ? 2 : 1) == 1 ? total % a.cus != 0 : 2 * total <= a.cus);   // see rows_body
    return true;
}

__device__ __forceinline__ int rotation(const GemmArgs& a, const MixedWork& m, bool multi) {
    const int apart = a.rot_mul, in_step = a.rot_mul_multi, chunk = a.rot_mul_chunk;   // values first: a choice between the fields' addresses puts the whole argument block in scratch memory
    return multi ? in_step : m.chunked ? chunk : apart;
}

// The kernel: what to work on from mixed_assign, the regime from the expert's rows, the body from the block's.
// PACKED: always true (kept because it is part of the kernel's name, which the library reports); row-major weights: tile_kernel.
template <int IB, bool GATEUP, bool WNT, bool HALF>
__device__ __forceinline__ void tile_mixed(const GemmArgs& a, uint16_t* xs) {
    MixedWork m;
    if (!mixed_assign<IB, GATEUP>(a, (int)blockIdx.x, m)) return;
    Tile t;
    const int nt = m.nt;
    const bool halves = m.halves;
    t.e = m.e;
    t.row0 = m.row0;
    t.rows = m.rows;
    t.n_e = m.n_e;
    t.stream = m.stream;
    // A short last tile of a multi-tile expert runs through k several times faster than its
    // siblings and shares nothing with them in time: it streams the panel like a single-block
    // expert does (non-temporal, k rotated), so that its stream does not evict the panels the
    // full tiles share.
    const bool multi = t.n_e > a.M && t.rows > a.short_nt;
    t.rot_mul = rotation(a, m, multi);
    const bool shared = multi || a.no_nt;
    if constexpr (IB == 2 && !GATEUP) {
        if (halves) {
            if (shared || !WNT) return dma_dispatch<1, GATEUP, false, HALF>(a, t, nt, xs);
            return dma_dispatch<1, GATEUP, WNT, HALF>(a, t, nt, xs);
        }
    }
    // Single-block tiles: weights through LDS where three ring buffers fit (rows_body); only taller ones are left
    // for the bodies below.  Not in the build for two workgroups per CU, whose half of LDS holds two buffers
    // (Qwen2-MoE shape, 100 tokens, gate+up 362 -> 384 us).
    constexpr int RM = HALF ? 0 : rows_max(IB * (GATEUP ? 2 : 1));
    if constexpr (RM > 0) {
        if (!multi && !(WNT && a.no_nt) && t.rows <= RM * 32)
            return rows_dispatch<IB, GATEUP, true, WNT, RM>(a, t, nt, m.deep, xs);
    }
    if (shared || !WNT) return dma_dispatch<IB, GATEUP, false, HALF>(a, t, nt, xs);
    if constexpr (WNT && RM < 8) dma_dispatch<IB, GATEUP, true, HALF, RM + 1>(a, t, nt, xs);
}

template <int IB, bool GATEUP, bool PACKED, bool WNT, bool HALF = false>
__global__ __launch_bounds__(kThreads, HALF ? 2 : 1) void tile_kernel_mixed(const GemmArgs a) {
    static_assert(PACKED, "row-major weights: tile_kernel");
    extern __shared__ __attribute__((aligned(1024))) uint16_t xs[];
    tile_mixed<IB, GATEUP, WNT, HALF>(a, xs);
}

// The gate+up projection with the permutation inside (permute_inside).
template <bool HALF>
__global__ __launch_bounds__(kThreads, HALF ? 2 : 1) void routed_tile_kernel_mixed(const GemmArgs a) {
    extern __shared__ __attribute__((aligned(1024))) uint16_t xs[];
    GemmArgs b = a;
    permute_inside(a, b, reinterpret_cast<int32_t*>(xs));
    tile_mixed<1, true, true, HALF>(b, xs);
}

// Row-major weights: the same launch orders and regimes, rows_body.
template <int IB, bool GATEUP>
__global__ __launch_bounds__(kThreads) void tile_kernel(const GemmArgs a) {
    extern __shared__ __attribute__((aligned(1024))) uint16_t xs[];
    MixedWork m;
    if (!mixed_assign<IB, GATEUP>(a, (int)blockIdx.x, m)) return;
    Tile t;
    t.e = m.e;
    t.row0 = m.row0;
    t.rows = m.rows;
    t.n_e = m.n_e;
    t.stream = m.stream;
    const bool multi = t.n_e > a.M && t.rows > a.short_nt;
    t.rot_mul = rotation(a, m, multi);
    if constexpr (IB == 2 && !GATEUP) {
        if (m.halves) return rows_dispatch<1, GATEUP, false, false, 8>(a, t, m.nt, m.deep, xs);
    }
    if (multi || a.no_nt) return rows_dispatch<IB, GATEUP, false, false, 8>(a, t, m.nt, m.deep, xs);
    rows_dispatch<IB, GATEUP, false, true, 8>(a, t, m.nt, m.deep, xs);
}

// =============================================================================================
// skinny_kernel: JB*32 <= 64 token rows, fragments straight from global memory, no LDS in the
// reduction loop.  SPLITK == 1: the four wavefronts own four different 32-row weight blocks.
// SPLITK == 4: they share one weight block and each reduces a quarter of K; partial sums are
// added in wavefront order through LDS (fixed order: bit-reproducible).
// Packed weights are loaded non-temporally, row-major ones are not: each of their 128-byte lines is consumed by
// the four loads of a step (down projection of the Mixtral shape, row-major, non-temporal / cached: 1 token 81 / 40 us,
// 2 tokens 169 / 93; packed 37 us at one token).
// =============================================================================================
template <int JB, bool GATEUP, int STAGES, int SPLITK, bool PACKED>
__global__ __launch_bounds__(kThreads) void skinny_kernel(const GemmArgs a) {
    constexpr int NM = GATEUP ? 2 : 1;
    constexpr int BM = JB * 32;
    constexpr int BN = (SPLITK == 1) ? 128 : 32;
    __shared__ float red[(SPLITK == 1) ? 1 : 3 * NM * JB * 16 * kWave];

    Tile t;
    int tile, nt;
    if (!map_workgroup(a, tile, nt) || !load_tile(a, tile, BM, t)) return;
    const int tid = threadIdx.x, wave = tid / kWave, lane = tid % kWave;
    const int li = lane & 31, half = lane >> 5;
    const int K = a.K, N = a.N;
    const int KT = K / kBK;
    const int n0w = nt * BN + (SPLITK == 1 ? wave * 32 : 0);
    const int per = (KT + SPLITK - 1) / SPLITK;
    const int kt_begin = (SPLITK == 1) ? 0 : wave * per;
    // last step of this wavefront's K range; below kt_begin when the range is empty
    const int kt_last = ((SPLITK == 1) ? KT : ((kt_begin + per) < KT ? (kt_begin + per) : KT)) - 1;

    typedef WAddr<PACKED, NM> WA;
    const uint16_t* wp[NM];
    static_for<NM>([&](auto m) { wp[m] = WA::base(a, t.e, n0w / 32, m, lane); });
    const uint16_t* xp[JB];
    static_for<JB>([&](auto j) {
        xp[j] = token_row(a, t.row0 + j * 32 + li) + half * 8;
    });

    f32x16 acc[NM][JB];
    static_for<NM>([&](auto i) {
        static_for<JB>([&](auto j) {
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[i][j][v] = 0.0f;
        });
    });

    uint4 wreg[STAGES][NM][4];
    uint4 xreg[STAGES][JB][4];
    auto load = [&](int kt, auto st) {
        int kc = kt < kt_last ? kt : kt_last;   // clamped into [0, KT): always in bounds
        kc = kc > 0 ? kc : 0;
        static_for<NM>([&](auto i) {
            static_for<4>([&](auto s) {
                wreg[st][i][s] = load_w16<PACKED>(wp[i] + (size_t)kc * WA::kStep + s * WA::sStep);
            });
        });
        static_for<JB>([&](auto j) {
            static_for<4>([&](auto s) {
                xreg[st][j][s] = *reinterpret_cast<const uint4*>(xp[j] + (size_t)kc * kBK + s * 16);
            });
        });
    };
    auto step = [&](int kt, auto st) {
        load(kt + STAGES - 1, std::integral_constant<int, (st + STAGES - 1) % STAGES>{});
        __builtin_amdgcn_sched_barrier(0);
        static_for<4>([&](auto s) {
            static_for<NM>([&](auto i) {
                static_for<JB>([&](auto j) {
                    acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(
                        __builtin_bit_cast(bf16x8, wreg[st][i][s]), __builtin_bit_cast(bf16x8, xreg[st][j][s]),
                        acc[i][j], 0, 0, 0);
                });
            });
        });
        __builtin_amdgcn_sched_barrier(0);
    };

    static_for<STAGES - 1>([&](auto st) { load(kt_begin + st, st); });
    int kt = kt_begin;
    for (; kt + STAGES - 1 <= kt_last; kt += STAGES) static_for<STAGES>([&](auto st) { step(kt + st, st); });
    static_for<STAGES>([&](auto st) {
        if (kt + st <= kt_last) step(kt + st, st);
    });

    if constexpr (SPLITK > 1) {
        // wavefronts 1..3 park their partial sums; wavefront 0 adds them in order 1, 2, 3
        constexpr int PER_WAVE = NM * JB * 16 * kWave;
        if (wave > 0) {
            static_for<NM>([&](auto i) {
                static_for<JB>([&](auto j) {
#pragma unroll
                    for (int v = 0; v < 16; ++v)
                        red[(wave - 1) * PER_WAVE + ((i * JB + j) * 16 + v) * kWave + lane] = acc[i][j][v];
                });
            });
        }
        __syncthreads();
        if (wave > 0) return;
        for (int w = 0; w < SPLITK - 1; ++w) {
            static_for<NM>([&](auto i) {
                static_for<JB>([&](auto j) {
#pragma unroll
                    for (int v = 0; v < 16; ++v)
                        acc[i][j][v] += red[w * PER_WAVE + ((i * JB + j) * 16 + v) * kWave + lane];
                });
            });
        }
    }
    static_for<JB>([&](auto j) {
        const int tr = j * 32 + li;
        const bool live = tr < t.rows;
        store_block<GATEUP>(acc[0][j], acc[GATEUP ? 1 : 0][j], a.Out + (size_t)(t.row0 + (live ? tr : 0)) * a.ldo, n0w,
                            half, N, live);
    });
}

// =============================================================================================
// launch helpers
// =============================================================================================
// k-loop rotation between the workgroups of an XCD, in steps.  Single-block experts (weights
// streamed once): 2, which spreads the row-strided token tile reads over the L2 channels.
// Multi-tile experts (the LDS-DMA kernels): 0, so that row tiles that share a weight panel, and
// feature tiles that share a token tile, walk k together and meet in L2 (measured: a third
// fewer L2 misses, ~3 % faster at Mixtral T=4096).
inline int rot_steps(bool dma) {
    const int v = knob(kKnobRot);
    return v >= 0 ? v : (dma ? 0 : 2);
}


// Launch order switches, feature-tile count and grid of a tile_kernel_mixed launch (host arithmetic
// only; `cus` = CUs of the device).  Returns the grid size.
template <int IB, bool GATEUP, bool WNT, bool HALF = false>
inline long long mixed_launch_shape(GemmArgs& args, int max_blocks, int cus) {
    constexpr int BN = 4 * IB * 32;
    args.n_tiles_n = (args.N + BN - 1) / BN;
    args.rot_mul = rot_steps(false);
    // Test knobs (see moe_internal.hpp) can override the three launch-order choices; -1 = the rule.
    args.sib = knob(kKnobSideBySide) >= 0 ? knob(kKnobSideBySide) : 1;
    args.even = knob(kKnobEvenRows) >= 0 ? knob(kKnobEvenRows) : (GATEUP ? 1 : 2);
    // Runs of consecutive positions per XCD (mixed_assign).  The token tile of an expert then comes from beyond L2 once, not once per
    // XCD; with 128 rows of a 256-expert layer that was a fifth of all bytes that the gate+up launch moved.
    //   Gate+up: where the workgroups of a block fit the CUs of an XCD (up to 32 feature tiles).  us, without / with: 128 experts of
    // 4096 x 1536, 2048 tokens 628 / 540; 256 of 7168 x 2048, 4096 tokens 2567 / 2320; Qwen2-MoE shape 1024
    // tokens 419 / 398; 16 experts of 6144 x 4096, 1000 tokens 270 / 264; at 112 and 128 feature tiles (Mixtral shapes) 325 / 328 and
    // 500 / 517.  From 64 rows per expert on (uniform routing): below, a token tile is too little to share, and what runs on an XCD at once
    // reads weight panels that lie a power of two apart at d = 4096 and 2048, out of few L2 channels: 128 experts of 4096 x 1536, 19 rows
    // 497 / 628, 44 rows 534 / 552, 62 rows 569 / 549; 64 of 4096 x 2048, 31 rows 349 / 404, 62 rows 366 / 356; 32 of 4096 x 4096, 31 rows
    // 336 / 392, 55 rows 336 / 349; other widths -3 to +2 %.  Row-major weights not at multiples of 16 tiles, whose runs are whole
    // experts: 64 experts of 2048 x 2048, 8 rows 167 / 178, 62 rows 183 / 190; 32 of 4096 x 4096, 100 rows 367 / 381; ahead at 128 of
    // 4096 x 1536, 69 rows 562 / 532, 125 rows 619 / 569.
    //   Down: 128 experts 354 / 333, 256 experts 2048 tokens 1499 / 1428, Qwen2-MoE shape 512 tokens 234 / 216.
    // The k loops of such workgroups walk in step, which is where they share most (gate+up of 128 experts of 4096 x 1536, 2048 tokens, one
    // step apart 599 / in step 534; down projection of 256 experts, 2048 tokens 1487 / 1409; Qwen2-MoE shape 512 tokens two apart 222 /
    // 218).  Two apart on loops over streamed weights beyond K = 4096, where either is within 3 % (us, two apart / in step: 6144 467 / 473; 6400 144 / 142; 8192
    // 178 / 172; 11264 129 / 125; 14336, 700 tokens 218 / 222); at 4096 two apart is 102 / 90.
    // Row-major weights, whose rows would all be read from one L2 channel in step (down projection of 256 experts, 512 tokens 1233 / 1388): one apart in gate+up, two
    // apart in the down projection, and there one contiguous eighth of the launch per XCD where every expert is one block, so that it runs through neighbouring rows.
    // Down projection, us, plain two apart / runs one apart / runs two apart / eighths: Mixtral-8x22B shape, 60 tokens 275 / 290 / 278 / 278, 300 tokens 325 / 346 / 312 /
    // 326, 8 tokens 258 / 262 / 249 / 249; 32 experts of 4096 x 4096, 20 tokens 153 / 162 / 159 / 151, 250 tokens 178 / 186 / 183 / 175; 64 of 2048 x 2048, 500 tokens
    // 106 / 98 / 107 / 97; 32 of 8192 x 1024, 250 tokens 104 / 108 / 102 / 101; 256 experts of DeepSeek-V3's widths, 1000 tokens 1305 / 1279 / 1303 / 1351.
    const bool packed = args.P != nullptr;
    const bool shares = !GATEUP || (args.n_tiles_n <= 32 && args.R >= 64ll * args.E && (packed || args.n_tiles_n % 16 != 0));
    args.chunk = knob(kKnobXcdChunk) >= 0 ? knob(kKnobXcdChunk) : shares ? 2 : 0;
    args.unit = (HALF ? 2 : 1) * (cus >= 16 ? cus / 16 : 16);
    // With multi-block experts: where the feature-tile count is no multiple of 8, or 8 or less (else the side-by-side order has the tiles
    // that share a panel on one XCD already), and the launch is four rounds or more, three in the down projection, because
    // an XCD's runs may hold more full tiles than another's (32 experts of 2880 x 2880, 1001 tokens at skew 1, gate+up 3.6 rounds 219 / 233 us; Mixtral
    // shape, 4096 tokens, down projection 2.2 rounds 814 / 927, gate+up with 112 tiles 1540 / 1600).  In the down projection in launches of any
    // length where a run holds a whole block: up to 16 feature tiles with streamed weights, up to 8 otherwise.  us, without / with: 64 experts of 896 x
    // 2048 (7 tiles), 1000 tokens, skew 0.6 87 / 71, skew 2 79 / 65; 60 of 1024 x 1408 (8), 300 tokens, skew 1.2 45 / 44, 128 of 640 x 1024 (5), 2000 tokens,
    // skew 0.6 55 / 49; 16 of 1792 x 3584 (14), 300 tokens 61 / 58, 700 tokens 84 / 86; cached weights, 16 of 1024 x 4096 (4), 2000 tokens, skew 0.6 100 / 91, but
    // 8 of 2880 x 2880 (12), 2000 tokens, skew 1.4 76 / 80.  With 23 tiles 101 / 112 (32 of 2880 x 2880, 300 tokens, skew 1.2).
    //   Gate+up: not beyond 20 tiles, and not where light blocks stand among the heavy ones, whose workgroups of one expert then meet on an XCD in a bunch:
    // up to 16 tiles as many light ones as heavy ones, beyond, where a block is longer than a run, two fifths.  us, without / with: 23 tiles, 32 experts of 2880 x
    // 2880, 1500 tokens at skew 1 268 / 277, 4000 tokens at skew 1.6 543 / 552; 20 tiles, Qwen2-MoE shape, 1000 tokens at skew 0.5 475 / 495, at skew
    // 1 489 / 513, 160 experts of 1536 x 2560, 2000 tokens at skew 1.6 241 / 261, but Qwen2-MoE shape 4096 tokens at skew 1 1141 / 1128, 3000 tokens 898 / 882;
    // 12 tiles, 128 experts of 4096 x 1536, 1500 tokens at skew 1.6 424 / 442, 4096 tokens at skew 0.5 936 / 887.  The Qwen2-MoE figures with
    // row-major weights: 1000 tokens at skew 0.5 501 / 532, 4096 tokens 1216 / 1187.
    //   Down: with a few blocks of multi-block experts, two weight blocks and streamed weights like without (16 tiles, 128 experts of 4096 x 1536, 500 tokens
    // at skew 0.6 310 / 294; 8 tiles, 60 of 2048 x 1408, 300 tokens 78 / 73); with one weight block rather not (23 tiles, above).
    const bool scattered = (args.n_tiles_n % 8 != 0 || args.n_tiles_n <= 8) && (!GATEUP || args.n_tiles_n <= 20);
    args.multi_from = !scattered ? INT_MAX : GATEUP ? 64 * args.unit : args.n_tiles_n <= (WNT ? 16 : 8) ? 0 : 48 * args.unit;
    args.few_from = !GATEUP && IB == 2 && WNT ? 0 : args.multi_from;
    args.light = !GATEUP ? 5 * 256 : args.n_tiles_n <= 16 ? 5 : 2;   // 256: the most single-block experts that there can be
    args.no_nt = knob(kKnobNoNt) > 0;
    args.short_nt = knob(kKnobShortNt) >= 0 ? knob(kKnobShortNt) : (GATEUP ? 64 : 0);
    args.eighths = !GATEUP && !packed;
    args.stream = (long long)args.R * args.N >= (1ll << 20) && (long long)args.E * args.N * args.K > (1ll << 26);
    args.rot_mul_multi = rot_steps(true);
    const int in_runs = !packed ? (GATEUP ? 1 : 2) : (!GATEUP && WNT && args.K > 4096) ? 2 : 0;
    args.rot_mul_chunk = knob(kKnobRot) >= 0 ? knob(kKnobRot) : in_runs;
    long long grid = ((long long)max_blocks * args.n_tiles_n + 7) / 8 * 8;   // as many for every XCD (the runs)
    args.slots = 0;
    args.cus = cus;
    if constexpr (IB == 2 && !GATEUP) {
        args.slots = cus;
        grid += cus / 2;     // a split last round has up to slots/2 extra workgroups
    }
    return grid;
}

inline int device_cus() {
    static const int cus = [] {
        int dev = 0, n = 0;
        if (hipGetDevice(&dev) != hipSuccess) return 0;
        if (hipDeviceGetAttribute(&n, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess) return 0;
        return n;
    }();
    return cus;
}

template <int IB, bool GATEUP, bool PACKED, bool WNT, bool HALF = false, bool ROUTED = false>
hipError_t launch_tile_mixed(const GemmArgs& a, int max_blocks, hipStream_t s) {
    // the DMA ring of tile_body_dma: XD+1 = 4 buffers of 256 (128) rows x 128 bytes; that of rows_body
    constexpr int ni = IB * (GATEUP ? 2 : 1), ring = 4 * (HALF ? 4 : 8) * 32 * 128, rows = HALF ? 0 : rows_lds(rows_max(ni), ni);
    constexpr int staged = store_lds(HALF ? 4 : 8, IB), loop = ring > rows ? ring : rows, lds = loop > staged ? loop : staged;
    static_assert(!ROUTED || (GATEUP && IB == 1 && PACKED && WNT), "permute_inside is part of the gate+up kernels");
    auto kern = [] {
        if constexpr (ROUTED) return routed_tile_kernel_mixed<HALF>;
        else return tile_kernel_mixed<IB, GATEUP, PACKED, WNT, HALF>;
    }();
    // once per process and kernel: not allowed while a stream is being captured into a graph
    static const hipError_t attr = hipFuncSetAttribute(reinterpret_cast<const void*>(kern),
                                                       hipFuncAttributeMaxDynamicSharedMemorySize, lds);
    if (attr != hipSuccess) return attr;
    GemmArgs args = a;
    const long long grid = mixed_launch_shape<IB, GATEUP, WNT, HALF>(args, max_blocks, device_cus());
    hipLaunchKernelGGL(kern, dim3((unsigned)grid), dim3(kThreads), lds, s, args);
    return hipGetLastError();
}

template <int IB, bool GATEUP>
hipError_t launch_rows(const GemmArgs& a, int max_blocks, hipStream_t s) {
    constexpr int NI = IB * (GATEUP ? 2 : 1);
    constexpr int loop = rows_lds(8, NI), staged = store_lds(8, IB), lds = loop > staged ? loop : staged;
    auto kern = tile_kernel<IB, GATEUP>;
    // once per process and kernel: not allowed while a stream is being captured into a graph
    static const hipError_t attr = hipFuncSetAttribute(reinterpret_cast<const void*>(kern),
                                                       hipFuncAttributeMaxDynamicSharedMemorySize, lds);
    if (attr != hipSuccess) return attr;
    GemmArgs args = a;
    const long long grid = mixed_launch_shape<IB, GATEUP, false>(args, max_blocks, device_cus());
    hipLaunchKernelGGL(kern, dim3((unsigned)grid), dim3(kThreads), lds, s, args);
    return hipGetLastError();
}

template <int JB, bool GATEUP, int STAGES, int SPLITK, bool PACKED>
hipError_t launch_skinny(const GemmArgs& a, int max_blocks, hipStream_t s) {
    constexpr int BN = (SPLITK == 1) ? 128 : 32;
    GemmArgs args = a;
    args.n_tiles_n = (a.N + BN - 1) / BN;
    const long long grid = (long long)max_blocks * args.n_tiles_n;
    hipLaunchKernelGGL((skinny_kernel<JB, GATEUP, STAGES, SPLITK, PACKED>), dim3((unsigned)grid), dim3(kThreads), 0,
                       s, args);
    return hipGetLastError();
}

struct Variant {
    int M;          // tallest block (Alg. 1's M) this variant can hold; it serves any schedule with M <= this
    bool packed;    // consumes moe_pack_weights' layout
    launch_fn fn;
    const char* name;   // kernel template instance, as rocprofv3 prints it (minus namespaces)
};

// A test may force a variant by table index through a knob; the index is ignored unless that
// variant matches the tile height and weight layout in use.
inline int forced_variant(int which, int count, int M, bool packed, const Variant* table) {
    const int id = knob(which);
    return (id >= 0 && id < count && table[id].M >= M && table[id].packed == packed) ? id : -1;
}

}  // namespace

}  // namespace moe

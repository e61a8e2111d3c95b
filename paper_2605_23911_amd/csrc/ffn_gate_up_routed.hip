// The gate+up kernels that permute up to 1024 rows by themselves (permute_inside), in a translation unit of their own to shorten the build.
#include "ffn_kernels.hpp"

namespace moe {

hipError_t launch_routed_mixed(const GemmArgs& a, int max_blocks, hipStream_t s) {
    return launch_tile_mixed<1, true, true, true, false, true>(a, max_blocks, s);
}

hipError_t launch_routed_mixed_half(const GemmArgs& a, int max_blocks, hipStream_t s) {
    return launch_tile_mixed<1, true, true, true, true, true>(a, max_blocks, s);
}

}  // namespace moe

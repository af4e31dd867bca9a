// Embedding kernels of the CTM chain in FP32 (see embed_tile.hpp).
#include "embed_tile.hpp"

namespace reach {

hipError_t launch_embed_ctm_f32(int, int E, int S, bool pair, const EmbedPass& a, int64_t grid,
                hipStream_t s) {
    return by_E<K_CTM, float, IN_SCALAR>(E, S, pair, a, grid, s);
}

}  // namespace reach

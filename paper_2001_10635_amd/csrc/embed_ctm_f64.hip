// Embedding kernels of the CTM chain in FP64 (see embed_tile.hpp).
#include "embed_tile.hpp"

namespace reach {

hipError_t launch_embed_ctm_f64(int, int E, int S, bool pair, const EmbedPass& a, int64_t grid,
                hipStream_t s) {
    return by_E<K_CTM, double, IN_SCALAR>(E, S, pair, a, grid, s);
}

}  // namespace reach

// Embedding kernels of the RD chain in FP64 (see embed_tile.hpp).
#include "embed_tile.hpp"

namespace reach {

hipError_t launch_embed_rd_f64(int mode, int E, int S, bool pair, const EmbedPass& a, int64_t grid,
                hipStream_t s) {
    return mode ? by_E<K_RD, double, IN_CELL>(E, S, pair, a, grid, s)
                : by_E<K_RD, double, IN_SCALAR>(E, S, pair, a, grid, s);
}

}  // namespace reach

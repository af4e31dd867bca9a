// Embedding kernels of the LIN3 chain in FP32 (see embed_tile.hpp).
#include "embed_tile.hpp"

namespace reach {

hipError_t launch_embed_lin3_f32(int mode, int E, int S, bool pair, const EmbedPass& a, int64_t grid,
                hipStream_t s) {
    // the left coupling crosses the sides (after the exchange of a.alt) or not
    if ((a.prm[0] < 0.0) != (a.alt != 0))
        return mode ? by_E<K_LIN3M, float, IN_CELL>(E, S, pair, a, grid, s)
                    : by_E<K_LIN3M, float, IN_ALT>(E, S, pair, a, grid, s);
    return mode ? by_E<K_LIN3C, float, IN_CELL>(E, S, pair, a, grid, s)
                : by_E<K_LIN3C, float, IN_ALT>(E, S, pair, a, grid, s);
}

}  // namespace reach

// Host-side check of the stage shapes of grouped batch launches (no GPU use): a member of any shape is planned with one
// that has a grouped kernel, its own where it has one.
#include <cstdio>

#include "batch_plan.hpp"

using namespace bub;

int main()
{
    int bad = 0;
    for (int ndim = 1; ndim <= 3; ++ndim)
        for (int tile = -1; tile < 8; ++tile) {
            const int g = group_tile(ndim, tile);
            const bool own = tile >= 0 && tile < GROUP_TILES[ndim];
            if (g < 0 || g >= GROUP_TILES[ndim] || (own && g != tile)) {
                std::printf("%dD shape %d: %d\n", ndim, tile, g);
                ++bad;
            }
        }
    if (GROUP_TILES[1] != 3) std::printf("1D: %d shapes\n", GROUP_TILES[1]), ++bad;   // the fourth has no grouped kernel
    return bad != 0;
}

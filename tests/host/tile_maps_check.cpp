// Host build of the map that deals a call's tiles to the XCDs
// (paper_2203_09384_amd/csrc/index_maps.hpp) for the CPU tests.
#include "index_maps.hpp"

extern "C" void tm_deal(int64_t batch, int64_t per, int64_t* b, int64_t* tile)
{
    for (int64_t block = 0; block < batch * per; block++) {
        const auto at = mifft::idx::xcd_deal_tile(block, batch, per);
        b[block] = at.b;
        tile[block] = at.tile;
    }
}

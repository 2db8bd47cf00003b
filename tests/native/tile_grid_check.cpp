// Host check of the tile grids and of the block order (lbm_kernels.h): reads
// "limits nx ny planes" or "visit nx ny planes" lines and prints, per tile shape, what
// the test compares.
#include <cstdio>
#include <cstring>
#include <vector>

#include "lbm_kernels.h"

using namespace cglbm;

template <int TX, int TY>
void limits(int nx, int ny, int planes)
{
    const dim3 g = tile_grid<TX, TY>(nx, ny, planes);
    printf("%llu %u %u %u\n", (unsigned long long)g.x * (TX * TY), g.x, g.y, g.z);
}

// tiles of the lattice that are not visited exactly once
template <int TX, int TY>
void visit(int nx, int ny, int planes)
{
    const dim3 g = tile_grid<TX, TY>(nx, ny, planes);
    const int T = (int)tiles_in_plane<TX, TY>(nx, ny);
    std::vector<int> seen((size_t)T * planes);
    long long wrong = 0;
    for (uint32_t by = 0; by < g.y; ++by)
        for (uint32_t bx = 0; bx < g.x; ++bx) {
            const TileOrder o = tile_of_block(g.x, g.y, bx, by, T, planes);
            if (!o.live) continue;
            if (o.b < 0 || o.b >= T || o.z < 0 || o.z >= planes)
                ++wrong;
            else
                ++seen[(size_t)o.z * T + o.b];
        }
    for (int s : seen) wrong += s != 1;
    printf("%lld\n", wrong);
}

int main()
{
    char what[16];
    int nx, ny, planes;
    while (scanf("%15s %d %d %d", what, &nx, &ny, &planes) == 4) {
        const bool lim = !strcmp(what, "limits");
        (lim ? limits<128, 2> : visit<128, 2>)(nx, ny, planes);  // state kernels, wide fused tiles
        (lim ? limits<128, 4> : visit<128, 4>)(nx, ny, planes);  // wide density tiles
        (lim ? limits<64, 4> : visit<64, 4>)(nx, ny, planes);    // narrow tiles
        (lim ? limits<64, 8> : visit<64, 8>)(nx, ny, planes);    // density tiles of the referenced forms
    }
    return 0;
}

// Host-only probe of the sweeps' tile rule (no kernel, no device call): for
// each nx ny nz triple on the command line and each sweep kind it prints the
// tile's width, height and chunk, its blocks, and the blocks that 66 x 7
// threads on the power-of-two chunks would take.
#include <cstdio>
#include <cstdlib>
#include "pt_internal.h"
int main(int argc, char** argv) {
    for (int a = 1; a + 2 < argc; a += 3) {
        ptk::Geom g{};
        g.nx = atoi(argv[a]); g.ny = atoi(argv[a + 1]); g.nz = atoi(argv[a + 2]);
        g.P = ((g.nx + 1 + 31) / 32) * 32; g.S = g.P * (g.ny + 1);
        const ptk::Tiling t = ptk::make_tiling(g);
        for (int k = 0; k < 4; ++k)
            printf("%d %d %d %d %d %d %d %lld %lld %lld\n", g.nx, g.ny, g.nz, k, t.shape[k].w, t.shape[k].h, t.shape[k].kz,
                   (long long)ptk::sweep_blocks(g, t.shape[k]), (long long)ptk::iter_grid_blocks(g, ptk::BX, 7),
                   (long long)t.most);
    }
    return 0;
}

// Prints how the gradient sums of a box are taken (kbc::grad_planes):
// nx ny nz -> planes per march of a tile (0: one node per thread) and the
// number of tiles.
#include <cstdio>
#include <cstdlib>

#include "kbc_internal.h"

int main(int argc, char** argv)
{
    if (argc != 4) return 2;
    kbc::Geom g{};
    g.nx = atoi(argv[1]);
    g.ny = atoi(argv[2]);
    g.nz = atoi(argv[3]);
    g.nnodes = g.nx * g.ny * g.nz;
    const uint32_t lz = kbc::grad_planes(g);
    std::printf("%u %llu\n", lz, lz ? (unsigned long long)kbc::grad_items(g, lz) : 0ull);
    return 0;
}

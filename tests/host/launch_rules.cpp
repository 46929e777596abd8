// Prints what the launch rules choose for a box: program, rule, then the
// rule's arguments.
#include <cstdio>
#include <cstdlib>
#include <cstring>

#include "kbc_internal.h"

using namespace kbc;

static Geom planes(char** a)
{
    Geom g{};
    g.nx = atoi(a[0]);
    g.ny = atoi(a[1]);
    g.nz = atoi(a[2]);
    g.nnodes = g.nx * g.ny * g.nz;
    geom_planes(g, 0);
    return g;
}

int main(int argc, char** argv)
{
    const char* rule = argc > 1 ? argv[1] : "";
    // curl nx ny nz: planes of a run, runs
    if (!strcmp(rule, "curl") && argc == 5) {
        const Geom g = planes(argv + 2);
        const uint32_t lz = curl_planes(g);
        printf("%u %llu\n", lz, (unsigned long long)g.nx * g.ny * ((g.nz + lz - 1) / lz));
        return 0;
    }
    // gamma nx ny nz: workgroups of the stabilizer statistics
    if (!strcmp(rule, "gamma") && argc == 5) {
        printf("%u\n", gamma_blocks(planes(argv + 2)));
        return 0;
    }
    // pair storage variant nx ny nz: 1 where a pull box takes its steps in pairs
    if (!strcmp(rule, "pair") && argc == 7) {
        const int storage = atoi(argv[2]), variant = atoi(argv[3]);
        Geom g = planes(argv + 4);
        // x-blocked where the lattice spans less than 4 GiB
        const double bytes = 27.0 * g.nnodes * (storage == ST_F64 ? 8 : (storage == ST_F16 ? 2 : 4));
        if (bytes < 4294967296.0) geom_blocked(g);
        PairTiles t;
        printf("%d\n", pair_plan(storage, variant, false, g, 256, &t) ? 1 : 0);
        return 0;
    }
    // aa storage nx ny nz: 1 where an in-place box stores through the caches
    if (!strcmp(rule, "aa") && argc == 6) {
        const Geom g = planes(argv + 3);
        const bool f64 = atoi(argv[2]) == ST_F64;
        const uint64_t plane = g.plane * (f64 ? 8 : 4);
        printf("%d\n", cached_stores(false, 27 * plane, plane, f64) ? 1 : 0);
        return 0;
    }
    return 2;
}

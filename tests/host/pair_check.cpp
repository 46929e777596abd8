// Host check of the pair sweep's plan and index rules (kbc::pair_plan and the
// slot and tile arithmetic of k_pair): every tile fits the workgroup and its
// LDS entries, the tiles' inner nodes cover the box once, every value that
// an inner node's second step gathers is handed over by a thread of its
// workgroup, at the slot the reader looks in; the padded layout is injective
// inside its extent.  Arguments after the program: storage nx ny nz variant;
// then only the plan is printed.
#include <cstdio>
#include <cstdlib>
#include <vector>

#include "kbc_internal.h"

using namespace kbc;

static Geom geom(uint32_t nx, uint32_t ny, uint32_t nz)
{
    Geom g{};
    g.nx = nx;
    g.ny = ny;
    g.nz = nz;
    g.nnodes = nx * ny * nz;
    geom_blocked(g);
    return g;
}

// The slots one workgroup writes and reads for `planes` planes, as k_pair
// numbers them: a reader must find the value of the plane it expects.
static long check_slots(uint32_t planes, uint32_t regs)
{
    const uint32_t plus_n = 9 - regs, n = 27 + 3 * plus_n + regs;
    std::vector<int> held(n, -1);
    long bad = 0;
    int h1 = -1, h2 = -1;
    for (uint32_t j = 0, j3 = 0; j < planes + 2; ++j) {
        const uint32_t zero = 9 + (j & 1) * 9, plus = 27 + j3 * plus_n;
        for (uint32_t k = 0; k < 9; ++k) {
            held[k] = (int)j;
            held[zero + k] = (int)j;
            held[k < plus_n ? plus + k : n - 1] = (int)j;
        }
        const uint32_t zero1 = 9 + ((j & 1) ^ 1) * 9, plus2 = 27 + (j3 == 2 ? 0 : j3 + 1) * plus_n;
        for (uint32_t k = 0; j >= 2 && k < 9; ++k) {
            bad += held[k] != (int)j;
            bad += held[zero1 + k] != (int)j - 1;
            bad += (k < plus_n ? held[plus2 + k] : h2) != (int)j - 2;
        }
        if (regs) {
            h2 = h1;
            h1 = held[n - 1];
        }
        j3 = j3 == 2 ? 0 : j3 + 1;
    }
    return bad;
}

static long check_tiles(const Geom& g, const PairTiles& p)
{
    long bad = 0;
    if ((p.tx + 2) * (p.ty + 2) > kPairBlock || p.tx * p.ty > kPairInner) ++bad;
    if (p.grid != p.ntx * p.nty * ((g.nz + p.lz - 1) / p.lz) || p.lz == 0) ++bad;
    std::vector<uint8_t> seen((size_t)g.nx * g.ny, 0);
    for (uint32_t tile = 0; tile < p.ntx * p.nty; ++tile) {
        const uint32_t x0 = tile % p.ntx * p.tx, y0 = tile / p.ntx * p.ty;
        const uint32_t rows = g.ny - y0 < p.ty ? g.ny - y0 : p.ty;
        // what the first step hands over: node computed -> entries written
        std::vector<int> from(9 * p.tx * p.ty, -1);
        for (uint32_t t = 0; t < kPairBlock; ++t) {
            const uint32_t ex = t % (p.tx + 2), ey = t / (p.tx + 2);
            if (ey >= rows + 2) continue;
            const uint32_t xa = (x0 + g.nx - 1 + ex) % g.nx, ya = (y0 + g.ny - 1 + ey) % g.ny;
            for (int k = 0; k < 9; ++k) {
                const int vx = k % 3 - 1, vy = k / 3 - 1;
                if (!(ex + vx - 1 < p.tx && ey + vy - 1 < p.ty)) continue;
                const uint32_t d = (ey - 1) * p.tx + (ex - 1) + vy * p.tx + vx;
                if (d >= p.tx * p.ty || from[9 * d + k] >= 0) ++bad;
                else from[9 * d + k] = (int)(xa + g.nx * ya);
            }
        }
        for (uint32_t t = 0; t < p.tx * p.ty; ++t) {
            const uint32_t x = x0 + t % p.tx, y = y0 + t / p.tx;
            if (x >= g.nx || y >= g.ny) continue;
            ++seen[x + (size_t)g.nx * y];
            for (int k = 0; k < 9; ++k) {
                const uint32_t xs = (x + g.nx - (k % 3 - 1)) % g.nx, ys = (y + g.ny - (k / 3 - 1)) % g.ny;
                if (from[9 * t + k] != (int)(xs + g.nx * ys)) ++bad;
            }
        }
    }
    for (uint8_t v : seen) bad += v != 1;
    return bad;
}

static long check_padded(Geom g)
{
    geom_blocked16(g);
    std::vector<uint8_t> seen(geom_extent(g), 0);
    long bad = 0;
    for (int s = 0; s < 27; ++s)
        for (uint32_t z = 0; z < g.nz; ++z)
            for (uint32_t y = 0; y < g.ny; ++y)
                for (uint32_t x = 0; x < g.nx; ++x) {
                    const uint64_t i = pop_index(g, s, x, y, z);
                    if (i >= seen.size() || seen[i]++) ++bad;
                    if (x % 16 == 0 && i % 16) ++bad;   // runs of 16 start on a line
                }
    return bad;
}

int main(int argc, char** argv)
{
    if (argc == 6) {
        PairTiles p;
        const Geom g = geom(atoi(argv[2]), atoi(argv[3]), atoi(argv[4]));
        const bool yes = pair_plan(atoi(argv[1]), atoi(argv[5]), false, g, 256, &p);
        printf("%s lz %u grid %u\n", yes ? "pairs" : "single", yes ? p.lz : 0, yes ? p.grid : 0);
        return 0;
    }
    long bad = 0, pairs = 0;
    for (uint32_t planes = 1; planes < 9; ++planes) bad += check_slots(planes, 0) + check_slots(planes, 1);
    const uint32_t nxs[] = {1, 2, 15, 16, 17, 33, 64, 65, 96, 100, 131, 256, 300};
    const uint32_t nys[] = {1, 3, 11, 12, 13, 50, 97, 256};
    const uint32_t nzs[] = {1, 2, 5, 61, 100, 256, 1000};
    for (uint32_t nx : nxs)
        for (uint32_t ny : nys)
            for (uint32_t nz : nzs)
                for (int storage = 0; storage < 4; ++storage)
                    for (int variant : {0, 3, 7})
                        for (uint32_t cus : {256u, 32u}) {
                            const Geom g = geom(nx, ny, nz);
                            PairTiles p;
                            if (pair_plan(storage, variant, true, g, cus, &p)) ++bad;
                            if (!pair_plan(storage, variant, false, g, cus, &p)) continue;
                            ++pairs;
                            if (variant == 3 && cus == 256) bad += check_tiles(g, p);
                        }
    for (uint32_t nx : {1u, 15u, 17u, 90u, 100u, 131u}) bad += check_padded(geom(nx, 5, 3));
    if (pairs < 100) ++bad;   // the rule must not have become empty
    if (bad) printf("%ld errors, %ld plans\n", bad, pairs);
    return bad ? 1 : 0;
}

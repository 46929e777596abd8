// kbc_internal.h -- host-side interface between the C-ABI layer and the
// kernel launchers (not part of the public ABI).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "kbc_device.h"

namespace kbc {

// Population storage layout of one box (all modes are [27][nz][ny][nx]):
//   pull:  buffer `cur` holds the post-collision P(t-1) so that
//          F_i(x, t) = cur[i][x - v_i] (at t = 0, cur[i][x] = f^eq_i(x + v_i));
//   AA:    even t: F_i(x, t) = buf[i][x]; odd t: F_i(x, t) = buf[26-i][x - v_i].
enum Layout : int { LY_PULL = 0, LY_AA_EVEN = 1, LY_AA_ODD = 2 };

// Population layouts of a box (see Geom).  Planes [27][nz][ny][nx], each
// followed by `pad` unused elements:
inline void geom_planes(Geom& g, uint64_t pad)
{
    g.plane = (uint64_t)g.nnodes + pad;
    g.row = g.nx;
    g.slab = g.nx * g.ny;
    g.chunk = 0;
    g.xshift = 31;
    g.xmask = 0x7fffffffu;
}

// x-blocked [nz][ny][nx/B][27][B]: the 27 populations of B nodes adjacent in
// x lie in one contiguous run, B = 64 or 32 where it divides nx, else B = nx.
inline void geom_blocked(Geom& g)
{
    const uint32_t b = g.nx % 64 == 0 ? 64 : (g.nx % 32 == 0 ? 32 : g.nx);
    g.plane = b;
    g.row = 27 * g.nx;
    g.slab = 27 * g.nx * g.ny;
    if (b == g.nx) {
        g.chunk = 0;
        g.xshift = 31;
        g.xmask = 0x7fffffffu;
    } else {
        g.chunk = 27 * b;
        g.xshift = b == 64 ? 6 : 5;
        g.xmask = b - 1;
    }
}

// The same with B = 16 for rows that 16 does not divide: the last chunk of a
// row is only partly used, so that every run of 16 nodes starts on a 128-byte
// line in FP64.
inline void geom_blocked16(Geom& g)
{
    const uint32_t chunks = (g.nx + 15) / 16;
    g.plane = 16;
    g.chunk = 27 * 16;
    g.row = g.chunk * chunks;
    g.slab = g.row * g.ny;
    g.xshift = 4;
    g.xmask = 15;
}

inline bool geom_is_planes(const Geom& g) { return g.row == g.nx && g.xshift == 31 && g.plane >= g.nnodes; }

// Elements of the buffer that the layout spans.
inline uint64_t geom_extent(const Geom& g) { return pop_index(g, 26, g.nx - 1, g.ny - 1, g.nz - 1) + 1; }

// Bytes spanned by the populations of one slot (the 32-bit offsets of the
// step kernels address within this span from the slot's base).
inline uint64_t geom_slot_span_bytes(const Geom& g, size_t elem)
{
    return (pop_index(g, 0, g.nx - 1, g.ny - 1, g.nz - 1) + 1) * elem;
}

// Record the message returned by kbc_last_error() on this thread.
void set_last_error(const char* msg);

// One time step of one box (src -> dst for pull; in place for AA).
// block: step_threads(); cached: cached_stores().
hipError_t launch_step(int storage, int variant, int sweep, bool exact_gamma, uint32_t block,
                       bool cached, const StepParams& p, hipStream_t stream);

// Whether a box's steps store through the caches instead of past them.  Stored
// past them (non-temporal), a population that the next step reads comes from
// the last-level cache or HBM, and where rows are no multiple of 128 bytes the
// lines at the ends of a wave's run are written in parts; stored through them,
// the lattice competes with the reads.  By the bytes of the box's lattices
// (32 MB of L2, 256 MB of last-level cache; us per step, past / through):
//   pull, more than the L2s and no more than the last-level cache: FP64 64^3
//   (113 MB, in pairs) 21.5 / 18.3, 80^3 33.8 / 26.9, FP32 64^3 (57 MB) 12.3 / 10.3, 131 x
//   97 x 61 (167 MB) 40.0 / 32.1, 104^3 (243 MB) 50.5 / 41.6;
//   above: FP64 88^3 (294 MB) 48.8 / 50.3, 128^3 129 / 142, FP32 128^3 73.6 / 76.4;
//   around the L2s' size: FP32 40^3 (14 MB) 6.3 / 6.9, 48^3 (24 MB) 7.9 / 9.0;
//   far below it: FP64 16^3 4.20 / 3.95, FP32 24^3 (3 MB) 4.47 / 4.14.
//   AA, more than the L2s: FP64 80^3 (110 MB) 44.2 / 39.8, 100^3 72.6 / 68.3,
//   200^3 (1.7 GB) 705 / 666, FP32 127^3 (221 MB) 89.8 / 77.2; the same from 2 GB
//   on (256^3 FP64 1347 / 1346); below: FP64 48^3 (24 MB) 10.3 / 11.0, 56^3 (38 MB) 15.7 /
//   16.1, 60^3 (47 MB) 18.8 / 19.2, while FP32 gains from there (72^3, 40 MB, 16.9 / 16.2).
//   AA, planes of exactly 16 MiB (453 MB), and of 32 MiB in FP64: stores past the caches
//   are faster, probably because the lines of 27 planes a power of two apart
//   compete for the same sets (over several allocations, FP64 128^3 178 / 179-190, 64 x 128 x 256 177-181 /
//   178-192, 512 x 64 x 64 174-187 / 181-199, 256 x 256 x 64 332 / 339, FP32-X 512 x 64 x 128
//   172-188 / 184-188; 160 x 128 x 128, planes of 20 MiB, 229 / 223, 192 x 128 x 128, of 24,
//   275 / 261; 128 x 128 x 64, of 8, fits the last-level cache: 90 / 71).
// plane_bytes: one direction plane of an AA box.
inline bool cached_stores(bool pull, uint64_t bytes, uint64_t plane_bytes, bool f64)
{
    constexpr uint64_t MB = 1000000, MiB = 1 << 20;
    if (!pull) {
        if (plane_bytes == 16 * MiB || (f64 && plane_bytes == 32 * MiB)) return false;
        return bytes > (f64 ? 50 : 36) * MB && bytes < 2000 * MB;
    }
    return bytes < 8 * MB || (bytes > 36 * MB && bytes <= 256 * MB);
}

// Threads of a workgroup of the step.  One wavefront for the exact stabilizer
// (two waves per SIMD, and LDS for 64 threads: `collide`).  Otherwise 256, and
// where fewer threads still give every CU no more than one workgroup, 128 or
// 64, so that a small box spreads over all the CUs (us per step with 256 /
// 128 / 64 threads, FP64 pull: 16^3 5.10 / 4.39 / 4.20, 32^3 6.48 / 4.88 /
// 4.96; FP64 AA 32^3 7.32 / 5.38 / 5.56, FP32 AA 5.40 / 4.23 / 4.26).  Past that line
// the larger workgroup is the better one or the same (FP32 pull 36^3 5.77 /
// 6.19 / 6.58; 64 in the largest boxes 17-33% slower for the AA sweeps).
inline uint32_t step_threads(bool exact_gamma, uint32_t nnodes, uint32_t cus)
{
    if (exact_gamma || nnodes <= 64 * cus) return 64;
    return nnodes <= 128 * cus ? 128 : 256;
}

// The kernel and launch shape launch_step uses (for building graphs of steps).
using StepFn = void (*)(StepParams);
hipError_t step_launch_shape(int storage, int variant, int sweep, bool exact_gamma, uint32_t block,
                             bool cached, const Geom& g, StepFn* fn, uint32_t* grid);

// ---------------------------------------------------------------------------
// Two steps of a pull box in one launch (k_pair, kbc_pair.h): a workgroup of
// kPairBlock threads owns a tile of tx x ty columns and lz planes.
// ---------------------------------------------------------------------------
constexpr uint32_t kPairBlock = 256;   // (tx + 2)(ty + 2), at most
constexpr uint32_t kPairInner = 192;   // tx ty, at most (three whole waves)

struct PairTiles {
    uint32_t tx, ty;     // columns of a tile
    uint32_t ntx, nty;   // tiles along x and y
    uint32_t lz;         // planes of a tile (the last one along z may have fewer)
    uint32_t grid;       // workgroups
};

// Waves per SIMD of k_pair: two by registers and LDS in FP64, three in FP32.
constexpr uint32_t pair_waves(int storage) { return storage == ST_F64 ? 2 : 3; }

// Whether a pull box takes its steps in pairs, and with which tiles.
//
// A tile row is one 128-byte line: tiles 18, 20, 22 or 30 wide, whose
// non-temporal stores are partial lines, ran 1.6-2.3x slower at 256^3.  16 x 12 in FP64 keeps 192 of the
// 252 nodes computed per plane.
//
// lz minimises plane iterations of the whole GPU, measured as rounds of
// resident workgroups times lz + 2 (a tile computes two planes more than it
// stores).  A last round that leaves half the slots empty runs its planes in
// 0.68 of the time.  Over cubes of 64-256 nodes the choice is the fastest of
// the measured lz or within 2% of it, except 6% at 240.
//
// `fill` is the share of the plane iterations' node capacity that the box
// uses.  Pairs against single steps, both storing as cached_stores has it;
// FP64, natural s: 48^3 (0.33) 0.87x, 64^3 (0.44) 1.00x, 60^3-63^3 1.04-1.20x, 80^3 (0.65)
// 1.31x, 128^3 (0.76) 1.20x, 256^3 (0.88) 1.45x, 25 boxes of 150,000 to 1.5 million
// nodes between 16 and 256 an axis 1.07-1.46x; central s, whose extra arithmetic is
// no longer hidden, 128^3 1.14x, 256^3 1.31x.  FP32 (32 x 5 tiles, more of the sweep
// is arithmetic): 128^3 1.08x, 160^3 (0.76) 1.10x, 192^3 1.12x, 256^3 (0.86) 1.26x; central
// 256^3 1.05x; flat boxes whose single steps store through the caches 0.95-1.02x
// (96 x 96 x 128 44.1 against 42.0 us, 256 x 240 x 12 26.7 / 25.7).  FP32 with the
// FP64-formed non-equilibrium ran 0.97x at 256^3 and FP16 is bound by arithmetic,
// so they keep single steps, as does the exact stabilizer.
//
// In planes (lattices of 4 GiB and more, each tile row in 27 lines far apart)
// the lines' alignment decides.  Pairs against single steps, FP64: rows of whole
// 64 bytes 1.05-1.34x (280^3 1.15x, 296^3 1.05x, 320^3 1.22x, 512^3 1.22x, 48 x 800 x 800
// 1.32x; central 280 x 300 x 300 1.12x); other rows lose (276^3 0.96x, 290^3 0.87x,
// 310^3 0.92x, 350^3 0.83x, 281 x 500 x 200 0.83x), except where every plane
// starts at an odd node, which slows the single step as much (301^3 1.11x,
// 285^3 1.05x, 341^3 1.00x, 395^3 1.00x, 305^3 0.96x).  FP32: rows up to 352 nodes 1.05-
// 1.25x (352^3, 256 x 512 x 320, 96 x 700 x 700), longer ones 0.80-1.02x (384^3 0.95x,
// 416^3 1.02x, 512^3 0.92x, 1024 x 256 x 160 0.80x).
inline bool pair_plan(int storage, int variant, bool exact_gamma, const Geom& g, uint32_t cus,
                      PairTiles* out)
{
    if (exact_gamma || (storage != ST_F64 && storage != ST_F32)) return false;
    if (storage == ST_F32 && (is_central(variant) || g.nx % 32)) return false;
    if (geom_is_planes(g)) {
        if (storage == ST_F64 && g.nx % 8 && g.nnodes % 2 == 0) return false;
        if (storage == ST_F32 && g.nx > 352) return false;
    }
    if (storage == ST_F32 && cached_stores(true, 2 * geom_extent(g) * sizeof(float), 0, false)) return false;
    PairTiles p;
    p.tx = storage == ST_F64 ? 16 : 32;
    p.ty = storage == ST_F64 ? 12 : 5;
    p.ntx = (g.nx + p.tx - 1) / p.tx;
    p.nty = (g.ny + p.ty - 1) / p.ty;
    const double slots = (double)cus * pair_waves(storage);
    const double tiles = (double)p.ntx * p.nty;
    double best = 0.0;
    p.lz = 0;
    for (uint32_t chunks = 1; chunks <= g.nz && chunks <= 64; ++chunks) {
        const uint32_t lz = (g.nz + chunks - 1) / chunks;
        const double w = tiles * ((g.nz + lz - 1) / lz) / slots;
        const double whole = (double)(uint64_t)w, part = w - whole;
        const double cost = (whole + (part == 0.0 ? 0.0 : (part <= 0.5 ? 0.68 : 1.0))) * (lz + 2);
        if (p.lz == 0 || cost < best) {
            best = cost;
            p.lz = lz;
        }
    }
    const double fill = (double)g.nnodes / (best * slots * p.tx * p.ty);
    const double least = storage == ST_F32 ? 0.72 : (is_central(variant) ? 0.6 : 0.42);
    if (fill < least) return false;
    p.grid = p.ntx * p.nty * ((g.nz + p.lz - 1) / p.lz);
    *out = p;
    return true;
}

struct PairParams {
    const void* src;
    void* dst;
    Geom g;
    Coll c;
    PairTiles p;
};
using PairFn = void (*)(PairParams);
// The kernel pair_plan's boxes run (storage FP64 or FP32 dev).
PairFn pair_step(int storage, int variant, bool cached);

// Write f^eq(rho, u) of device fields u [3][N], rho [N] (may be NULL) into the
// storage buffer in the given layout.
hipError_t launch_init_feq(int storage, int layout, void* buf, const Geom& g,
                           const float* scale, const double* u, const double* rho,
                           hipStream_t stream);

// Validity of an initial state: sets *flag (device int, pre-zeroed) to 1 if
// some |u_a| >= 1 or rho <= 0 or a value is not finite.
hipError_t launch_check_init(const Geom& g, const double* u, const double* rho, int* flag,
                             hipStream_t stream);

// Per-direction max |f^eq_i - W_i| over the box (device float[27], zeroed
// by the callee) for choosing FP16 scales.
hipError_t launch_feq_dev_max(const Geom& g, const double* u, const double* rho,
                              unsigned* max_bits, hipStream_t stream);

// Per-direction max |f_i - W_i| of a canonical FP64 population field.
hipError_t launch_pop_dev_max(const Geom& g, const double* f, unsigned* max_bits,
                              hipStream_t stream);

// Canonical F(t) [27][N] FP64 <-> storage in the given layout.
hipError_t launch_gather_pop(int storage, int layout, const void* buf, const Geom& g,
                             const float* inv_scale, double* f, hipStream_t stream);
hipError_t launch_scatter_pop(int storage, int layout, void* buf, const Geom& g,
                              const float* scale, const double* f, hipStream_t stream);

// F(t) at selected nodes: out [count][27] FP64, nodes [count] (in range).
hipError_t launch_sample_pop(int storage, int layout, const void* buf, const Geom& g,
                             const float* inv_scale, const uint32_t* nodes, int count,
                             double* out, hipStream_t stream);

// One pass over F(t): rho [N] (nullable) and u [3][N] (both NULL: not stored),
// and out[0..2] = sum_x u_a(x), out[3] = sum_x |u(x) - <u>|^2, out[4] = nodes
// where a value is not finite; the same bits whether u is stored or not.
// partial: device scratch of energy_partials() doubles; with
// log (may be NULL) it receives out[3], and out[6] becomes 1 if out[4] is not 0.
int energy_partials();
hipError_t launch_fields(int storage, int layout, const void* buf, const Geom& g,
                         const float* inv_scale, double* rho, double* u, double* partial,
                         double* out, double* log, hipStream_t stream);

// A step (estimate gamma only) that also leaves the sums of the state it reads in
// `runs`, series_partials(g) doubles, and the sums over `count` such arrays, one
// after the other: what launch_fields writes to log for each state goes to
// log[0 .. count), and out[6] becomes 1 if some node was not finite.
// groups: count * energy_partials() doubles.
size_t series_partials(const Geom& g);
hipError_t launch_step_series(int storage, int variant, int sweep, uint32_t block,
                              const StepParams& p, double* runs, hipStream_t stream);
hipError_t launch_series_sums(const Geom& g, int count, const double* runs, double* groups,
                              double* out, double* log, hipStream_t stream);

// Plain streaming copy of n16 16-byte words.
hipError_t launch_copy16(void* dst, const void* src, size_t n16, hipStream_t stream);
hipError_t launch_rewrite16(void* p, size_t n16, hipStream_t stream);

// Sums over a velocity field u [3][N], in a fixed order.
// *out = sum_x |curl_FD2 u(x)|^2; partial: reduce_partials().
// A thread sums a run of curl_planes() planes of one column: long runs read u the
// least, but where a plane has few nodes a wave's runs start far apart and
// there are few of them (us of kbc_enstrophy with 32 / 4 / 1 planes: 1 x 1 x 4,000,000
// 424 / 255 / 256, 1 x 1 x 65,536 71 / 36 / 35, 8 x 8 x 200,000 737 / 732 / 749, 15 x
// 17 x 60,000 893 / 876 / 897, 512^3 FP16 3241 / 3299 / 3554).
inline uint32_t curl_planes(const Geom& g) { return g.nx * g.ny < 256 ? 4 : 32; }
hipError_t launch_curl(const Geom& g, const double* u, double* partial, double* out,
                       hipStream_t stream);
// The kernel and tiles of the gradient sums: planes that a tile of kGradX x
// kGradY columns is marched through, 0 for one node per thread.  A march is a
// chain of plane loads: long ones leave the GPU idle on small boxes and their
// last round of workgroups unfilled on larger ones, short ones load their first
// planes for little (us of kbc_statistics at second / eighth order, marches of 32, 16 and
// 8 planes, nodes: 32^3 67 / 89, 53 / 64, 46 / 51, 38 / 42; 64^3 81 / 102, 64 / 75, 56 /
// 62, 51 / 59; 96^3 102 / 125, 86 / 99, 81 / 90, 80 / 105; 128^3 180 / 203, 166 / 185, 166 /
// 184, 168 / 224; 200^3 491 / 593, 508 / 569, 511 / 571, 536 / 822; 256^3 982 / 1038, 982 /
// 1051, 991 / 1064).  A short row or few rows leave lanes without a node
// (4 x 512 x 512, an eighth of the lanes filled: 122 / 158 in marches of 32, 128 / 170 of 8,
// 89 / 114 by nodes; 8 x 1024 x 1024, a quarter: 625 / 767, 636 / 800, 512 / 722; 16 x 400 x
// 400, half: 201 / 228, 189 / 221, 187 / 259; 1 x 1 x 4,000,000: 4.3 / 6.1, 4.7 / 7.3, 0.26 /
// 0.36 ms).
constexpr uint32_t kGradX = 32, kGradY = 8;
inline uint64_t grad_items(const Geom& g, uint32_t lz)
{
    return (uint64_t)((g.nx + kGradX - 1) / kGradX) * ((g.ny + kGradY - 1) / kGradY) * ((g.nz + lz - 1) / lz);
}
inline uint32_t grad_planes(const Geom& g)
{
    const double lanes = (double)grad_items(g, 1) * (kGradX * kGradY);
    if (g.nnodes <= 1u << 18 || g.nnodes < 0.4 * lanes) return 0;
    return grad_items(g, 16) < 512 ? 8 : 16;
}
// Flow statistics.  grad: out[8] = sums over nodes of |curl u|^2,
// sum_ab (d_a u_b + d_b u_a)^2, (div u)^2, (du_x/dx)^n for n = 2..6, with the
// central stencil of the given order (2 or 8); partial: reduce_partials() * 8.
hipError_t launch_grad_stats(int order, const Geom& g, const double* u, double* partial,
                             double* out, hipStream_t stream);
// gamma of the next collision at every node: out[4] = sum, sum of squares,
// min, max; partial: gamma_blocks() * 4.
// Workgroups of it: few waves fit a SIMD with the collision's registers, and
// further rounds of workgroups are further prologues and partial sums (us of
// kbc_gamma_statistics with 2048 / 1024, FP64: 512 x 512 x 4 in place 78 / 74, 100^3 75 /
// 72, 80^3 in place 55 / 52; the same from 160^3 on).
inline uint32_t gamma_blocks(const Geom& g)
{
    const uint32_t b = g.nnodes / 256 + (g.nnodes % 256 != 0);
    return b < 1024 ? b : 1024;
}
hipError_t launch_gamma_stats(int storage, int variant, bool exact_gamma, int layout,
                              const void* buf, const Geom& g, const Coll& c,
                              const float* inv_scale, double* partial, double* out,
                              hipStream_t stream);
// x-correlation sums: out[2r + c] = sum over nodes of u'_c(x) u'_c(x + r),
// c = 0 (x component), 1 (y component), r = 0..rmax; requires
// nx <= corr_max_nx(), rmax < corr_max_lags(); partial: corr_partials(g, rmax)
// doubles; mean_sum: the three sums of u.
int corr_max_nx();
int corr_max_lags();
size_t corr_partials(const Geom& g, int rmax);
hipError_t launch_corr_x(const Geom& g, const double* u, const double* mean_sum, int rmax,
                         double* partial, double* out, hipStream_t stream);

// Blocks of a reduction over u; `partial` holds up to 8 doubles for each.
int reduce_partials();

// ---------------------------------------------------------------------------
// Batched ensemble (pool): many independent AA boxes advanced by one launch.
// ---------------------------------------------------------------------------
struct PoolBox {
    void* buf;            // the box's population array (AA layout, in place)
    Geom g;
    Coll c;
    uint32_t tile0;       // first tile of the box in the current batch
    uint32_t ntiles;      // ceil(nnodes / (block * sub))
    int32_t parity0;      // t mod 2 at the start of the batch
    int32_t steps;        // steps the box takes in the current batch
    int8_t scale_exp[28]; // FP16 storage: stored = (f - W) * 2^scale_exp[i]
};

// One launch group of a batch: boxes[first .. first + n_active) of the
// batch's box table, all at the same parity, sorted by tile0 (tiles are
// numbered from 0 within the group).
struct PoolMeta {
    uint32_t first;       // index of the group's first box in the table
    uint32_t n_active;    // boxes in the group
    uint32_t n_tiles;     // tiles in the group
    uint32_t block;       // threads per block
    uint32_t sub;         // block-sized sub-tiles per tile
};

constexpr int kPoolMaxBlock = 512;

// Step k (0-based) of a batch for one launch group: every box of the group
// with k < steps applies the AA sweep `sweep` (SW_AA_EVEN or SW_AA_ODD).
// Persistent grid-stride loop over the group's tiles; block <= 512.
// boxes and tstart are the whole table (tstart[b] = boxes[b].tile0, a
// compact copy for the tile -> box search); meta is the group's entry.
// one: the launch has a block for every tile of the group and one run of
// nodes per tile (sub = 1), so the single-tile kernel applies
hipError_t launch_pool_step(int storage, int variant, int sweep, const PoolBox* boxes,
                            const uint32_t* tstart, const PoolMeta* meta, int k, int block,
                            int grid, bool one, hipStream_t stream);

// ---------------------------------------------------------------------------
// Kernel tables.  The step, pool and stabilizer-statistics kernels are
// instantiated in kbc_step_inst.hip, once per storage form S and stabilizer
// mode GX (exact root or estimate), so that the eight instances compile in
// parallel; these functions return the kernel for a variant and sweep.
// ---------------------------------------------------------------------------
struct LoadCtx {
    float inv_scale[27];
};
using PoolFn = void (*)(const PoolBox*, const uint32_t*, const PoolMeta*, int);
using SeriesFn = void (*)(StepParams, double*);
using GammaFn = void (*)(int, const void*, Geom, Coll, LoadCtx, double*);

// c64: the box is x-blocked in chunks of 64 nodes (a pull sweep may then
// take a kernel with that geometry compiled in)
template <int S, bool GX>
StepFn step_kernel(int variant, int sweep, bool c64, bool cached);
template <int S>
PairFn pair_kernel(int variant, bool cached);               // FP64 and FP32 dev, estimate gamma only
template <int S>
PoolFn pool_kernel(int variant, int sweep, bool one);   // estimate gamma only
template <int S>
SeriesFn series_kernel(int variant, int sweep, bool c64);   // estimate gamma only
template <int S, bool GX>
GammaFn gamma_kernel(int variant);

}  // namespace kbc

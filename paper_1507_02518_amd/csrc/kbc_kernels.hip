// kbc_kernels.hip -- gfx950 kernels of the D3Q27 KBC lattice Boltzmann box
// other than the step itself (kbc_step.h, instantiated in kbc_step_inst.hip):
// initialisation at the product-form equilibrium, layout conversion, FP64
// diagnostics, the streaming copy, and the launchers of all of them.
#include <hip/hip_runtime.h>
#include <math.h>

#include "kbc_device.h"
#include "kbc_fields.h"
#include "kbc_internal.h"
#include "kbc_step.h"

namespace kbc {

namespace {

template <int S>
__device__ __forceinline__ void store_full(void* buf, uint64_t idx, int slot, int i,
                                           const float* scale, double f)
{
    using T = typename Traits<S>::T;
    T* b = static_cast<T*>(buf);
    if constexpr (S == ST_F64) b[idx] = f;
    else if constexpr (S == ST_F32) b[idx] = (float)(f - weight(i));
    else b[idx] = (_Float16)((float)(f - weight(i)) * scale[slot]);
}

// Product-form equilibrium of section II through its one-dimensional
// marginals, in FP64: e_0 = (4 - 2S)/3, e_{+-1} = ((2S - 1)/3 +- u)/2.
__device__ __forceinline__ void marginals(double u, double e[3])
{
    const double q3 = 3.0 * u * u;
    const double sm1 = q3 / (1.0 + sqrt(1.0 + q3));
    e[1] = 2.0 / 3.0 - (2.0 / 3.0) * sm1;
    e[2] = 1.0 / 6.0 + sm1 / 3.0 + 0.5 * u;
    e[0] = 1.0 / 6.0 + sm1 / 3.0 - 0.5 * u;
}

struct StoreCtx {
    float scale[27];
};

template <int S>
__global__ void __launch_bounds__(kBlock) k_init_feq(int layout, void* buf, Geom g, StoreCtx sc,
                                                     const double* __restrict__ u,
                                                     const double* __restrict__ rho)
{
    const uint32_t n = blockIdx.x * kBlock + threadIdx.x;
    if (n >= g.nnodes) return;
    uint32_t x, y, z;
    node_xyz(n, g, x, y, z);
    const double r = rho ? rho[n] : 1.0;
    double ex[3], ey[3], ez[3];
    marginals(u[n], ex);
    marginals(u[g.nnodes + n], ey);
    marginals(u[2 * (size_t)g.nnodes + n], ez);
    for (int i = 0; i < 27; ++i) {
        const double feq = r * ex[i % 3] * ey[(i / 3) % 3] * ez[i / 9];
        int slot;
        const uint64_t idx = locate(layout, i, x, y, z, g, slot);
        store_full<S>(buf, idx, slot, i, sc.scale, feq);
    }
}

__global__ void __launch_bounds__(kBlock) k_check_init(Geom g, const double* __restrict__ u,
                                                       const double* __restrict__ rho, int* flag)
{
    const uint32_t n = blockIdx.x * kBlock + threadIdx.x;
    if (n >= g.nnodes) return;
    bool bad = false;
    for (int a = 0; a < 3; ++a) {
        const double v = u[a * (size_t)g.nnodes + n];
        bad |= !(fabs(v) < 1.0);
    }
    if (rho) bad |= !(rho[n] > 0.0 && isfinite(rho[n]));
    if (bad) atomicOr(flag, 1);
}

// Per-direction maximum over the block first (non-negative floats compare
// like their bit patterns), then one atomic per direction and block.
__device__ __forceinline__ void block_max_27(float (&d)[27], unsigned* max_bits)
{
    __shared__ unsigned red[27];
    if (threadIdx.x < 27) red[threadIdx.x] = 0u;
    __syncthreads();
    for (int i = 0; i < 27; ++i) {
        unsigned v = __float_as_uint(d[i]);
        for (int off = 32; off > 0; off >>= 1) v = max(v, (unsigned)__shfl_xor((int)v, off, 64));
        if ((threadIdx.x & 63) == 0) atomicMax(&red[i], v);
    }
    __syncthreads();
    if (threadIdx.x < 27) atomicMax(&max_bits[threadIdx.x], red[threadIdx.x]);
}

__global__ void __launch_bounds__(kBlock) k_feq_dev_max(Geom g, const double* __restrict__ u,
                                                        const double* __restrict__ rho,
                                                        unsigned* max_bits)
{
    const uint32_t n = blockIdx.x * kBlock + threadIdx.x;
    float d[27];
    for (int i = 0; i < 27; ++i) d[i] = 0.0f;
    if (n < g.nnodes) {
        const double r = rho ? rho[n] : 1.0;
        double ex[3], ey[3], ez[3];
        marginals(u[n], ex);
        marginals(u[g.nnodes + n], ey);
        marginals(u[2 * (size_t)g.nnodes + n], ez);
        for (int i = 0; i < 27; ++i)
            d[i] = (float)fabs(r * ex[i % 3] * ey[(i / 3) % 3] * ez[i / 9] - weight(i));
    }
    block_max_27(d, max_bits);
}

__global__ void __launch_bounds__(kBlock) k_pop_dev_max(Geom g, const double* __restrict__ f,
                                                        unsigned* max_bits)
{
    const uint32_t n = blockIdx.x * kBlock + threadIdx.x;
    float d[27];
    for (int i = 0; i < 27; ++i)
        d[i] = n < g.nnodes ? (float)fabs(f[i * (size_t)g.nnodes + n] - weight(i)) : 0.0f;
    block_max_27(d, max_bits);
}

template <int S>
__global__ void __launch_bounds__(kBlock) k_gather_pop(int layout, const void* buf, Geom g,
                                                       LoadCtx lc, double* __restrict__ f)
{
    const uint32_t n = blockIdx.x * kBlock + threadIdx.x;
    if (n >= g.nnodes) return;
    uint32_t x, y, z;
    node_xyz(n, g, x, y, z);
    for (int i = 0; i < 27; ++i) {
        int slot;
        const uint64_t idx = locate(layout, i, x, y, z, g, slot);
        f[i * (size_t)g.nnodes + n] = load_full<S>(buf, idx, slot, i, lc.inv_scale);
    }
}

template <int S>
__global__ void __launch_bounds__(kBlock) k_sample_pop(int layout, const void* buf, Geom g,
                                                       LoadCtx lc, const uint32_t* __restrict__ nodes,
                                                       int count, double* __restrict__ out)
{
    const int k = blockIdx.x * kBlock + threadIdx.x;
    if (k >= count) return;
    const uint32_t n = nodes[k];
    uint32_t x, y, z;
    node_xyz(n, g, x, y, z);
    for (int i = 0; i < 27; ++i) {
        int slot;
        const uint64_t idx = locate(layout, i, x, y, z, g, slot);
        out[27 * (size_t)k + i] = load_full<S>(buf, idx, slot, i, lc.inv_scale);
    }
}

template <int S>
__global__ void __launch_bounds__(kBlock) k_scatter_pop(int layout, void* buf, Geom g, StoreCtx sc,
                                                        const double* __restrict__ f)
{
    const uint32_t n = blockIdx.x * kBlock + threadIdx.x;
    if (n >= g.nnodes) return;
    uint32_t x, y, z;
    node_xyz(n, g, x, y, z);
    for (int i = 0; i < 27; ++i) {
        int slot;
        const uint64_t idx = locate(layout, i, x, y, z, g, slot);
        store_full<S>(buf, idx, slot, i, sc.scale, f[i * (size_t)g.nnodes + n]);
    }
}

// Density and velocity of F(t) and the kinetic-energy sums in one pass over the
// populations (kbc_fields.h on the order): wave w takes the runs w, w + waves,
// ... and writes its group's sums.  FIELDS: u (and rho where asked for) are
// stored too.  Bound by reading the populations: FP64 256^3 with u stored
// 0.87 -> 0.82 ms, FP16 512^3 5.41 -> 2.14 ms against the version with a
// 64-bit index and a wrap per population.
template <int S, int LY, bool FIELDS>
__global__ void __launch_bounds__(kBlock) k_fields(const void* buf, Geom g, LoadCtx lc,
                                                   double* __restrict__ rho,
                                                   double* __restrict__ u,
                                                   EnergySum* __restrict__ groups)
{
    using T = typename Traits<S>::T;
    using R = typename Traits<S>::R;
    const uint32_t runs = (g.nnodes + 63) / 64, lane = threadIdx.x & 63;
    const uint32_t wave = blockIdx.x * (kBlock / 64) + (threadIdx.x >> 6);
    const uint32_t waves = runs < kEnergyGroups ? runs : kEnergyGroups;
    if (wave >= waves) return;
    EnergyAcc acc;
    T v[27];
    auto fetch = [&](uint32_t j) {
        const uint32_t node = 64 * j + lane;
        load_node<S, LY>(buf, g, node < g.nnodes ? node : g.nnodes - 1, v);
    };
    fetch(wave);
    for (uint32_t j = wave; j < runs; j += waves) {
        const uint32_t node = 64 * j + lane;
        const bool real = node < g.nnodes;
        R f[27];
#pragma unroll
        for (int i = 0; i < 27; ++i) f[i] = decode<S>(v[i], lc.inv_scale[i]);
        // the next run's populations are on their way while this one is reduced
        if (j + waves < runs) fetch(j + waves);
        double m, uu[3];
        node_velocity<S>(f, m, uu);
        if constexpr (FIELDS) {
            if (real) {
                if (rho) rho[node] = m;
                u[node] = uu[0];
                u[g.nnodes + (size_t)node] = uu[1];
                u[2 * (size_t)g.nnodes + node] = uu[2];
            }
        }
        double inv;
        const double count = run_count(j, g.nnodes, inv);
        add_energy(acc, run_energy(real, count, inv, m, uu), count, inv, j == wave);
    }
    if (lane == 0) groups[wave] = total_energy(acc);
}

// Nodes of the group w.
__device__ __forceinline__ double group_count(uint32_t w, uint32_t nnodes)
{
    const uint32_t runs = (nnodes + 63) / 64, waves = runs < kEnergyGroups ? runs : kEnergyGroups;
    const uint32_t mine = (runs - w + waves - 1) / waves;
    // the last run may be short
    return 64.0 * mine - ((runs - 1) % waves == w ? 64.0 * runs - (double)nnodes : 0.0);
}

// The groups' sums from the runs' of blockIdx.y-th state, one thread each (the
// adding that k_fields does as it goes).
__global__ void __launch_bounds__(kBlock) k_energy_groups(const EnergySum* __restrict__ runs_of,
                                                          uint32_t nnodes,
                                                          EnergySum* __restrict__ groups)
{
    const uint32_t runs = (nnodes + 63) / 64, waves = runs < kEnergyGroups ? runs : kEnergyGroups;
    const uint32_t w = blockIdx.x * kBlock + threadIdx.x;
    if (w >= waves) return;
    runs_of += (size_t)blockIdx.y * runs;
    EnergyAcc acc;
    for (uint32_t j = w; j < runs; j += waves) {
        double inv;
        const double count = run_count(j, nnodes, inv);
        add_energy(acc, runs_of[j], count, inv, j == w);
    }
    groups[(size_t)blockIdx.y * kEnergyGroups + w] = total_energy(acc);
}

// The sums over all nodes from the groups': out[0..2] sum of u, [3] sum of
// |u - <u>|^2, [4] nodes that are not finite.  log (may be NULL) takes out[3],
// and out[6] then becomes 1 if some node was not finite.  One workgroup for each
// of gridDim.x states, the last of which fills out; every thread adds its
// groups to the deviations from the first group's mean, and the five sums
// are then plain ones.
constexpr int kFinalBlock = 1024;
__global__ void __launch_bounds__(kFinalBlock) k_energy_final(const EnergySum* __restrict__ groups,
                                                              uint32_t nnodes,
                                                              double* __restrict__ out,
                                                              double* __restrict__ log)
{
#pragma clang fp contract(off)
    __shared__ double part[kFinalBlock / 64][5];
    groups += (size_t)blockIdx.x * kEnergyGroups;
    const uint32_t runs = (nnodes + 63) / 64, waves = runs < kEnergyGroups ? runs : kEnergyGroups;
    const double r0 = 1.0 / group_count(0, nnodes);
    const double c[3] = {groups[0].s[0] * r0, groups[0].s[1] * r0, groups[0].s[2] * r0};
    double a[5] = {0.0, 0.0, 0.0, 0.0, 0.0};   // sums of n d, of m2 + n d^2, bad
    for (uint32_t w = threadIdx.x; w < waves; w += kFinalBlock) {
        const EnergySum e = groups[w];
        const double n = group_count(w, nnodes), r = 1.0 / n;
        double d2 = 0.0;
        for (int k = 0; k < 3; ++k) {
            const double d = e.s[k] * r - c[k];
            a[k] += n * d;
            d2 = k == 0 ? d * d : d2 + d * d;
        }
        a[3] += e.m2 + n * d2;
        a[4] += e.bad;
    }
    for (int k = 0; k < 5; ++k) a[k] = wave_sum(a[k]);
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    if (lane == 0)
        for (int k = 0; k < 5; ++k) part[wave][k] = a[k];
    __syncthreads();
    if (threadIdx.x == 0) {
        for (int k = 0; k < 5; ++k) {
            a[k] = part[0][k];
            for (int w = 1; w < kFinalBlock / 64; ++w) a[k] += part[w][k];
        }
        const double N = (double)nnodes;
        const double m2 = a[3] - ((a[0] * a[0] + a[1] * a[1]) + a[2] * a[2]) / N;
        if (blockIdx.x + 1 == gridDim.x) {
            for (int k = 0; k < 3; ++k) out[k] = N * c[k] + a[k];
            out[3] = m2;
            out[4] = a[4];
        }
        if (log) {
            log[blockIdx.x] = m2;
            if (a[4] != 0.0) out[6] = 1.0;
        }
    }
}

// ---------------------------------------------------------------------------
// Deterministic FP64 reductions: fixed grid, fixed per-thread order,
// butterfly within the wavefront, fixed order across wavefronts and blocks.
// ---------------------------------------------------------------------------
// Blocks of the reductions over a velocity field: eight per CU, all resident.
constexpr int kReduceBlocks = 2048;

// Per-block sums of |curl u|^2, second-order central differences on the
// periodic grid.  A thread marches a column of lz planes (curl_planes) and keeps
// u_x and u_y of three planes; an item is 256 of these runs, columns first, and
// the workgroups of one XCD take consecutive items, so that the rows a row
// is differenced with come from its L2.  Bound by reading u: 512^3 1.17 -> 0.97
// ms (3.2 GB) against one node per thread in the dispatch order.
__global__ void __launch_bounds__(kBlock) k_curl(Geom g, uint32_t lz, const double* __restrict__ u,
                                                 double* __restrict__ partial)
{
    const size_t N = g.nnodes;
    const double *ux = u, *uy = u + N, *uz = u + 2 * N;
    const uint32_t slab = g.nx * g.ny;
    const uint32_t runs = slab * ((g.nz + lz - 1) / lz), items = (runs + kBlock - 1) / kBlock;
    // eighth of the items of this XCD (workgroup b runs on XCD b mod 8)
    const uint32_t xcds = gridDim.x < 8 ? 1 : 8;
    const uint32_t j = blockIdx.x % xcds, q = items / xcds, r = items % xcds;
    const uint32_t first = j * q + (j < r ? j : r), last = first + q + (j < r ? 1 : 0);
    double acc[1] = {0.0};
    for (uint32_t it = first + blockIdx.x / xcds; it < last; it += (gridDim.x + xcds - 1 - j) / xcds) {
        const uint32_t run = it * kBlock + threadIdx.x;
        if (run >= runs) continue;
        const uint32_t z0 = run / slab * lz, c = run % slab;
        const uint32_t planes = g.nz - z0 < lz ? g.nz - z0 : lz;
        const uint32_t y = fdiv(c, g.dnx), x = c - y * g.nx;
        const uint32_t xp = x + 1 == g.nx ? c - x : c + 1, xm = x == 0 ? c + g.nx - 1 : c - 1;
        const uint32_t yp = y + 1 == g.ny ? c - y * g.nx : c + g.nx;
        const uint32_t ym = y == 0 ? c + (g.ny - 1) * g.nx : c - g.nx;
        size_t here = (size_t)z0 * slab;
        const size_t below = (size_t)(z0 == 0 ? g.nz - 1 : z0 - 1) * slab;
        double ax = ux[below + c], ay = uy[below + c];   // plane z - 1
        double bx = ux[here + c], by = uy[here + c];     // plane z
        for (uint32_t k = 0; k < planes; ++k) {
            const size_t up = z0 + k + 1 == g.nz ? 0 : here + slab;
            const double cx = ux[up + c], cy = uy[up + c];
            const double *px = ux + here, *py = uy + here, *pz = uz + here;
            const double wx = 0.5 * (pz[yp] - pz[ym]) - 0.5 * (cy - ay);
            const double wy = 0.5 * (cx - ax) - 0.5 * (pz[xp] - pz[xm]);
            const double wz = 0.5 * (py[xp] - py[xm]) - 0.5 * (px[yp] - px[ym]);
            acc[0] += wx * wx + wy * wy + wz * wz;
            ax = bx;
            ay = by;
            bx = cx;
            by = cy;
            here = up;
        }
    }
    block_sum<1>(acc, partial + blockIdx.x);
}

template <int K>
__global__ void __launch_bounds__(kBlock) k_reduce_final_k(const double* __restrict__ partial,
                                                           int count, double* __restrict__ out)
{
    double acc[K];
#pragma unroll
    for (int k = 0; k < K; ++k) acc[k] = 0.0;
    for (int b = threadIdx.x; b < count; b += kBlock)
#pragma unroll
        for (int k = 0; k < K; ++k) acc[k] += partial[K * b + k];
    block_sum<K>(acc, out);
}

// ---------------------------------------------------------------------------
// Flow statistics of section V from the velocity field u[3][N].
// ---------------------------------------------------------------------------

// Central first-derivative weights of f(x+m) - f(x-m): second order, and
// the nine-point eighth-order stencil.
template <int ORD> struct FdW;
template <> struct FdW<2> {
    static constexpr int M = 1;
    __device__ static constexpr double c(int) { return 0.5; }
};
template <> struct FdW<8> {
    static constexpr int M = 4;
    __device__ static constexpr double c(int m)
    {
        return m == 1 ? 4.0 / 5.0 : (m == 2 ? -1.0 / 5.0 : (m == 3 ? 4.0 / 105.0 : -1.0 / 280.0));
    }
};

// Adds a node's |curl u|^2, sum_ab (d_a u_b + d_b u_a)^2, (div u)^2 and
// (du_x/dx)^n for n = 2..6, given G[a][b] = d u_a / d x_b.
__device__ __forceinline__ void add_grad(const double (&G)[3][3], double (&acc)[8])
{
    const double wx = G[2][1] - G[1][2], wy = G[0][2] - G[2][0], wz = G[1][0] - G[0][1];
    acc[0] += wx * wx + wy * wy + wz * wz;
    double e = 0.0;
#pragma unroll
    for (int a = 0; a < 3; ++a)
#pragma unroll
        for (int b = 0; b < 3; ++b) {
            const double sab = G[a][b] + G[b][a];
            e += sab * sab;
        }
    acc[1] += e;
    const double dv = G[0][0] + G[1][1] + G[2][2];
    acc[2] += dv * dv;
    const double d1 = G[0][0], d2 = d1 * d1, d3 = d2 * d1;
    acc[3] += d2;
    acc[4] += d3;
    acc[5] += d2 * d2;
    acc[6] += d3 * d2;
    acc[7] += d3 * d3;
}

// Per-block sums of these, fixed order.  A workgroup marches a tile of
// 32 x 8 columns through lz planes (grad_planes): a thread keeps its column's
// 2M + 1 planes in registers for the z derivatives, and the plane's tile with
// its halo goes through LDS for the others, 10 loads per node and plane at
// eighth order instead of 72 with a 64-bit remainder for each neighbour.
// 200^3, eighth order: 0.45 -> 0.18 ms.
static_assert(kGradX * kGradY == kBlock, "one thread per column");

template <int ORD>
__global__ void __launch_bounds__(kBlock) k_grad_stats(Geom g, uint32_t lz,
                                                       const double* __restrict__ u,
                                                       double* __restrict__ partial)
{
    constexpr int M = FdW<ORD>::M;
    constexpr uint32_t W = kGradX + 2 * M, H = kGradY + 2 * M, PER = (W * H + kBlock - 1) / kBlock;
    __shared__ double tile[3][H * W];
    const size_t N = g.nnodes;
    const uint32_t t = threadIdx.x, tx = t % kGradX, ty = t / kGradX;
    const uint32_t slab = g.nx * g.ny;
    const uint32_t ntx = (g.nx + kGradX - 1) / kGradX, nty = (g.ny + kGradY - 1) / kGradY;
    const uint32_t items = ntx * nty * ((g.nz + lz - 1) / lz);
    double acc[8];
#pragma unroll
    for (int k = 0; k < 8; ++k) acc[k] = 0.0;
    for (uint32_t it = blockIdx.x; it < items; it += gridDim.x) {
        const uint32_t xi = it % ntx, yz = it / ntx, x0 = xi * kGradX, y0 = yz % nty * kGradY;
        const uint32_t z0 = yz / nty * lz;
        const uint32_t planes = g.nz - z0 < lz ? g.nz - z0 : lz;
        const bool real = x0 + tx < g.nx && y0 + ty < g.ny;
        const uint32_t own = ((y0 + ty) % g.ny) * g.nx + (x0 + tx) % g.nx;
        // tile element e = t + k 256 is node (x0 - M + e % W, y0 - M + e / W), periodic
        uint32_t from[PER];
#pragma unroll
        for (uint32_t k = 0; k < PER; ++k) {
            const uint32_t e = t + k * kBlock;
            const uint32_t x = periodic_minus(x0 + e % W, M, g.nx), y = periodic_minus(y0 + e / W, M, g.ny);
            from[k] = y * g.nx + x;
        }
        double col[3][2 * M + 1];   // [a][d]: u_a at plane z - M + d
#pragma unroll
        for (int d = 1; d <= 2 * M; ++d) {
            const size_t at = (size_t)periodic_minus(z0 + d - 1, M, g.nz) * slab + own;
#pragma unroll
            for (int a = 0; a < 3; ++a) col[a][d] = u[a * N + at];
        }
        for (uint32_t p = 0; p < planes; ++p) {
            const size_t at = (size_t)((z0 + p + M) % g.nz) * slab + own;
#pragma unroll
            for (int a = 0; a < 3; ++a) {
#pragma unroll
                for (int d = 0; d < 2 * M; ++d) col[a][d] = col[a][d + 1];
                col[a][2 * M] = u[a * N + at];
            }
            const double* plane = u + (size_t)(z0 + p) * slab;
            __syncthreads();
#pragma unroll
            for (uint32_t k = 0; k < PER; ++k) {
                const uint32_t e = t + k * kBlock;
                if (e < W * H)
#pragma unroll
                    for (int a = 0; a < 3; ++a) tile[a][e] = plane[a * N + from[k]];
            }
            __syncthreads();
            const uint32_t c = (ty + M) * W + tx + M;
            double G[3][3];  // G[a][b] = d u_a / d x_b
#pragma unroll
            for (int a = 0; a < 3; ++a) {
                double dx = 0.0, dy = 0.0, dz = 0.0;
#pragma unroll
                for (int m = 1; m <= M; ++m) {
                    dx += FdW<ORD>::c(m) * (tile[a][c + m] - tile[a][c - m]);
                    dy += FdW<ORD>::c(m) * (tile[a][c + m * W] - tile[a][c - m * W]);
                    dz += FdW<ORD>::c(m) * (col[a][M + m] - col[a][M - m]);
                }
                G[a][0] = dx;
                G[a][1] = dy;
                G[a][2] = dz;
            }
            if (!real) continue;
            add_grad(G, acc);
        }
    }
    __syncthreads();
    block_sum<8>(acc, partial + 8 * blockIdx.x);
}

// The same sums with one node per thread and its neighbours from the caches,
// for boxes that leave the tiles empty or too few (grad_planes).
template <int ORD>
__global__ void __launch_bounds__(kBlock) k_grad_nodes(Geom g, const double* __restrict__ u,
                                                       double* __restrict__ partial)
{
    constexpr int M = FdW<ORD>::M;
    const size_t N = g.nnodes;
    const uint32_t slab = g.nx * g.ny;
    double acc[8];
#pragma unroll
    for (int k = 0; k < 8; ++k) acc[k] = 0.0;
    for (uint32_t n = blockIdx.x * kBlock + threadIdx.x; n < g.nnodes; n += gridDim.x * kBlock) {
        uint32_t c[3];
        node_xyz(n, g, c[0], c[1], c[2]);
        const uint32_t len[3] = {g.nx, g.ny, g.nz}, step[3] = {1, g.nx, slab};
        double G[3][3];  // G[a][b] = d u_a / d x_b
#pragma unroll
        for (int b = 0; b < 3; ++b) {
            const uint32_t base = n - c[b] * step[b];
            uint32_t up = c[b], down = c[b];
#pragma unroll
            for (int a = 0; a < 3; ++a) G[a][b] = 0.0;
#pragma unroll
            for (int m = 1; m <= M; ++m) {
                up = wrap_add(up, 1, len[b]);
                down = wrap_add(down, -1, len[b]);
                const double *pu = u + (base + up * step[b]), *pd = u + (base + down * step[b]);
#pragma unroll
                for (int a = 0; a < 3; ++a) G[a][b] += FdW<ORD>::c(m) * (pu[a * N] - pd[a * N]);
            }
        }
        add_grad(G, acc);
    }
    block_sum<8>(acc, partial + 8 * blockIdx.x);
}

__global__ void __launch_bounds__(kBlock) k_gamma_final(const double* __restrict__ partial,
                                                        int count, double* __restrict__ out)
{
    double acc[2] = {0.0, 0.0};
    double lo = __builtin_inf(), hi = -__builtin_inf();
    for (int b = threadIdx.x; b < count; b += kBlock) {
        acc[0] += partial[4 * b];
        acc[1] += partial[4 * b + 1];
        lo = fmin(lo, partial[4 * b + 2]);
        hi = fmax(hi, partial[4 * b + 3]);
    }
    double tmp[2];
    block_sum<2>(acc, tmp);  // thread 0 holds the sums in tmp
    __shared__ double mn[kBlock / 64], mx[kBlock / 64];
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) {
        lo = fmin(lo, __shfl_xor(lo, off, 64));
        hi = fmax(hi, __shfl_xor(hi, off, 64));
    }
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    if (lane == 0) {
        mn[wave] = lo;
        mx[wave] = hi;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        for (int w = 0; w < kBlock / 64; ++w) {
            lo = fmin(lo, mn[w]);
            hi = fmax(hi, mx[w]);
        }
        out[0] = tmp[0];
        out[1] = tmp[1];
        out[2] = lo;
        out[3] = hi;
    }
}

// Sums over the (y, z) lines of u'_c(x) u'_c(x + r) for the components c = x, y
// and r = 0..rmax.  A workgroup stages a few lines of one component in
// LDS, each followed by its own start (so that x + r needs no wrap) and padded
// by one value in eight, and splits the products into tiles of 8 nodes x 8
// lags: 23 reads from LDS for 64 multiply-adds in registers, where one lag per
// thread and pass read two values for each.  Thread t has lags
// 8 (t mod lag_tiles) .. + 7 and the node tiles t / lag_tiles, + groups, ...;
// the padding puts the windows of neighbouring lag tiles 9 values apart, on
// different banks.  Bound by the FP64 multiply-adds and the LDS reads beside
// them: 200^3 with 101 lags 0.77 -> 0.15 ms.
constexpr int kCorrMaxN = 4096;
constexpr int kCorrMaxLags = 2048;
constexpr int kCorrTile = 8;
constexpr int kCorrBlocks = 1024;   // workgroups per component and lag range
__host__ __device__ constexpr uint32_t corr_pad(uint32_t i) { return i + i / 8; }

// Lag tiles of one workgroup, at most (more lags: further workgroups).
constexpr uint32_t kCorrLagTiles = 64;

struct CorrPlan {
    uint32_t lag_tiles;   // of one workgroup
    uint32_t ranges;      // lag ranges
    uint32_t lines;       // staged at a time
    uint32_t stride;      // LDS values per line
    uint32_t blocks;      // per component and range
};

inline CorrPlan corr_plan(const Geom& g, int rmax)
{
    CorrPlan p;
    const uint32_t tiles = (uint32_t)rmax / kCorrTile + 1;
    p.ranges = (tiles + kCorrLagTiles - 1) / kCorrLagTiles;
    p.lag_tiles = (tiles + p.ranges - 1) / p.ranges;
    // a line, its start again up to the last window's end
    p.stride = corr_pad(g.nx + p.ranges * p.lag_tiles * kCorrTile + 2 * kCorrTile) + 1;
    // several short lines at a time keep the threads' shares even; 32 KB
    p.lines = std::max<uint32_t>(1, std::min<uint32_t>(8, 4096 / p.stride));
    p.blocks = (uint32_t)std::min<uint64_t>(kCorrBlocks, ((uint64_t)g.ny * g.nz + p.lines - 1) / p.lines);
    return p;
}

__global__ void __launch_bounds__(kBlock) k_corr_x(Geom g, CorrPlan p, const double* __restrict__ u,
                                                   const double* __restrict__ mean_sum, int rmax,
                                                   double* __restrict__ partial)
{
    extern __shared__ double line[];
    const uint32_t comp = blockIdx.y, range = blockIdx.z, t = threadIdx.x;
    const size_t N = g.nnodes;
    const double mean = mean_sum[comp] / (double)N;
    const double* uc = u + comp * N;
    const uint32_t lines = g.ny * g.nz, groups = kBlock / p.lag_tiles;
    const uint32_t lt = t % p.lag_tiles, grp = t / p.lag_tiles;
    const uint32_t lag0 = (range * p.lag_tiles + lt) * kCorrTile;
    const uint32_t full = g.nx / kCorrTile, tail = g.nx % kCorrTile;
    const uint32_t ext = g.nx + p.ranges * p.lag_tiles * kCorrTile + 2 * kCorrTile;
    double acc[kCorrTile];
#pragma unroll
    for (int k = 0; k < kCorrTile; ++k) acc[k] = 0.0;
    for (uint32_t l0 = blockIdx.x * p.lines; l0 < lines; l0 += gridDim.x * p.lines) {
        const uint32_t here = lines - l0 < p.lines ? lines - l0 : p.lines;
        __syncthreads();
        for (uint32_t l = 0; l < here; ++l) {
            const double* src = uc + (size_t)(l0 + l) * g.nx;
            for (uint32_t i = t; i < ext; i += kBlock) line[l * p.stride + corr_pad(i)] = src[i % g.nx] - mean;
        }
        __syncthreads();
        if (grp < groups) {
            for (uint32_t it = grp; it < here * full; it += groups) {
                const uint32_t l = it / full, xt = it - l * full;
                // tiles start at multiples of 8: element k of a window is k + k / 8 on
                const double* a = line + l * p.stride + corr_pad(xt * kCorrTile);
                const double* b = line + l * p.stride + corr_pad(xt * kCorrTile + lag0);
                double av[8], bv[15];
#pragma unroll
                for (int k = 0; k < 8; ++k) av[k] = a[k];
#pragma unroll
                for (int k = 0; k < 15; ++k) bv[k] = b[k + k / 8];
#pragma unroll
                for (int i = 0; i < 8; ++i)
#pragma unroll
                    for (int k = 0; k < 8; ++k) acc[k] = fma(av[i], bv[i + k], acc[k]);
            }
            // the nodes past the last whole tile, one at a time
            for (uint32_t it = grp; it < here * tail; it += groups) {
                const uint32_t l = it / tail, x = full * kCorrTile + it - l * tail;
                const double av = line[l * p.stride + corr_pad(x)];
#pragma unroll
                for (int k = 0; k < 8; ++k) acc[k] = fma(av, line[l * p.stride + corr_pad(x + lag0 + k)], acc[k]);
            }
        }
    }
    // over the groups, in order
    __syncthreads();
    if (grp < groups)
#pragma unroll
        for (int k = 0; k < 8; ++k) line[(grp * p.lag_tiles + lt) * 8 + k] = acc[k];
    __syncthreads();
    for (uint32_t k = t; k < p.lag_tiles * 8; k += kBlock) {
        const uint32_t lag = range * p.lag_tiles * 8 + k;
        if (lag > (uint32_t)rmax) continue;
        double s = 0.0;
        for (uint32_t q = 0; q < groups; ++q) s += line[q * p.lag_tiles * 8 + k];
        partial[((size_t)lag * 2 + comp) * gridDim.x + blockIdx.x] = s;   // [2r + c][block]
    }
}

// out[2r + c] from the workgroups' sums, one workgroup each.
__global__ void __launch_bounds__(kBlock) k_corr_final(const double* __restrict__ partial,
                                                       int blocks, double* __restrict__ out)
{
    const double* p = partial + (size_t)blockIdx.x * blocks;
    double acc[1] = {0.0};
    for (int b = threadIdx.x; b < blocks; b += kBlock) acc[0] += p[b];
    block_sum<1>(acc, out + blockIdx.x);
}

inline unsigned grid_for(uint32_t n) { return (n + kBlock - 1) / kBlock; }

__global__ void k_zero_u32(unsigned* p, int n)
{
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) p[i] = 0u;
}

// Streaming copy: one 16-byte word per thread and iteration (ordinary
// loads, non-temporal stores); the grid covers up to 2^21 blocks, which is
// the whole array for copies up to 8 GiB.  This form measured fastest among
// the copies tried (16 B or 8 B per lane, 1 or 4 words per thread, with or
// without non-temporal loads).
typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));

__global__ void __launch_bounds__(kBlock) k_copy16(u32x4* __restrict__ dst,
                                                  const u32x4* __restrict__ src, size_t n16)
{
    const size_t stride = (size_t)gridDim.x * kBlock;
    for (size_t k = (size_t)blockIdx.x * kBlock + threadIdx.x; k < n16; k += stride)
        __builtin_nontemporal_store(src[k], &dst[k]);
}

// The same stream in place: every 16-byte word is read and written back to
// its own address, the access pattern of an in-place sweep.  `mask` is zero
// at run time (the data stays as it was); XOR-ing it into all four lanes
// keeps the compiler from dropping (or narrowing) the store of a value just
// loaded from the same address.
__global__ void __launch_bounds__(kBlock) k_rewrite16(u32x4* p, size_t n16, uint32_t mask)
{
    const size_t stride = (size_t)gridDim.x * kBlock;
    for (size_t k = (size_t)blockIdx.x * kBlock + threadIdx.x; k < n16; k += stride) {
        u32x4 v = p[k];
        v ^= mask;
        __builtin_nontemporal_store(v, &p[k]);
    }
}

}  // namespace

// ---------------------------------------------------------------------------
// Launchers
// ---------------------------------------------------------------------------
// x-blocked in chunks of 64 nodes (geom_blocked)
static bool chunks_of_64(const Geom& g)
{
    return g.xshift == 6 && g.xmask == 63 && g.plane == 64 && g.chunk == 27 * 64;
}

hipError_t step_launch_shape(int storage, int variant, int sweep, bool exact_gamma, uint32_t block,
                             bool cached, const Geom& g, StepFn* fn, uint32_t* grid)
{
    // whole waves, and the threads the kernel was compiled for
    if (block < 64 || block % 64 || block > (exact_gamma ? 64u : (uint32_t)kStepBlock)) return hipErrorInvalidValue;
    // the AA kernels address populations in planes (see node_update)
    if (sweep != SW_PULL && !geom_is_planes(g)) return hipErrorInvalidValue;
    const bool c64 = chunks_of_64(g);
    switch (storage) {
    case ST_F64: *fn = exact_gamma ? step_kernel<ST_F64, true>(variant, sweep, c64, cached) : step_kernel<ST_F64, false>(variant, sweep, c64, cached); break;
    case ST_F32: *fn = exact_gamma ? step_kernel<ST_F32, true>(variant, sweep, c64, cached) : step_kernel<ST_F32, false>(variant, sweep, c64, cached); break;
    case ST_F32X: *fn = exact_gamma ? step_kernel<ST_F32X, true>(variant, sweep, c64, cached) : step_kernel<ST_F32X, false>(variant, sweep, c64, cached); break;
    default: *fn = exact_gamma ? step_kernel<ST_F16, true>(variant, sweep, c64, cached) : step_kernel<ST_F16, false>(variant, sweep, c64, cached); break;
    }
    *grid = (g.nnodes + block - 1) / block;
    return hipSuccess;
}

hipError_t launch_step(int storage, int variant, int sweep, bool exact_gamma, uint32_t block,
                       bool cached, const StepParams& p, hipStream_t stream)
{
    StepFn fn;
    uint32_t grid;
    hipError_t e = step_launch_shape(storage, variant, sweep, exact_gamma, block, cached, p.g, &fn, &grid);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(fn, dim3(grid), dim3(block), 0, stream, p);
    return hipGetLastError();
}

PairFn pair_step(int storage, int variant, bool cached)
{
    return storage == ST_F64 ? pair_kernel<ST_F64>(variant, cached) : pair_kernel<ST_F32>(variant, cached);
}

hipError_t launch_pool_step(int storage, int variant, int sweep, const PoolBox* boxes,
                            const uint32_t* tstart, const PoolMeta* meta, int k, int block,
                            int grid, bool one, hipStream_t stream)
{
    if (block < 64 || block > kPoolMaxBlock || block % 64 || grid < 1) return hipErrorInvalidValue;
    if (sweep != SW_AA_EVEN && sweep != SW_AA_ODD) return hipErrorInvalidValue;
    PoolFn fn;
    switch (storage) {
    case ST_F64: fn = pool_kernel<ST_F64>(variant, sweep, one); break;
    case ST_F32: fn = pool_kernel<ST_F32>(variant, sweep, one); break;
    case ST_F32X: fn = pool_kernel<ST_F32X>(variant, sweep, one); break;
    default: fn = pool_kernel<ST_F16>(variant, sweep, one); break;
    }
    hipLaunchKernelGGL(fn, dim3(grid), dim3(block), 0, stream, boxes, tstart, meta, k);
    return hipGetLastError();
}

hipError_t launch_init_feq(int storage, int layout, void* buf, const Geom& g, const float* scale,
                           const double* u, const double* rho, hipStream_t stream)
{
    if (storage == ST_F32X) storage = ST_F32;  // same storage format
    StoreCtx sc;
    for (int i = 0; i < 27; ++i) sc.scale[i] = scale ? scale[i] : 1.0f;
    const dim3 grid(grid_for(g.nnodes)), block(kBlock);
    if (storage == ST_F64) hipLaunchKernelGGL(k_init_feq<ST_F64>, grid, block, 0, stream, layout, buf, g, sc, u, rho);
    else if (storage == ST_F32) hipLaunchKernelGGL(k_init_feq<ST_F32>, grid, block, 0, stream, layout, buf, g, sc, u, rho);
    else hipLaunchKernelGGL(k_init_feq<ST_F16>, grid, block, 0, stream, layout, buf, g, sc, u, rho);
    return hipGetLastError();
}

hipError_t launch_check_init(const Geom& g, const double* u, const double* rho, int* flag,
                             hipStream_t stream)
{
    hipLaunchKernelGGL(k_check_init, dim3(grid_for(g.nnodes)), dim3(kBlock), 0, stream, g, u, rho, flag);
    return hipGetLastError();
}

hipError_t launch_feq_dev_max(const Geom& g, const double* u, const double* rho, unsigned* max_bits,
                              hipStream_t stream)
{
    hipLaunchKernelGGL(k_zero_u32, dim3(1), dim3(64), 0, stream, max_bits, 27);
    hipLaunchKernelGGL(k_feq_dev_max, dim3(grid_for(g.nnodes)), dim3(kBlock), 0, stream, g, u, rho, max_bits);
    return hipGetLastError();
}

hipError_t launch_pop_dev_max(const Geom& g, const double* f, unsigned* max_bits, hipStream_t stream)
{
    hipLaunchKernelGGL(k_zero_u32, dim3(1), dim3(64), 0, stream, max_bits, 27);
    hipLaunchKernelGGL(k_pop_dev_max, dim3(grid_for(g.nnodes)), dim3(kBlock), 0, stream, g, f, max_bits);
    return hipGetLastError();
}

hipError_t launch_gather_pop(int storage, int layout, const void* buf, const Geom& g,
                             const float* inv_scale, double* f, hipStream_t stream)
{
    if (storage == ST_F32X) storage = ST_F32;  // same storage format
    LoadCtx lc;
    for (int i = 0; i < 27; ++i) lc.inv_scale[i] = inv_scale ? inv_scale[i] : 1.0f;
    const dim3 grid(grid_for(g.nnodes)), block(kBlock);
    if (storage == ST_F64) hipLaunchKernelGGL(k_gather_pop<ST_F64>, grid, block, 0, stream, layout, buf, g, lc, f);
    else if (storage == ST_F32) hipLaunchKernelGGL(k_gather_pop<ST_F32>, grid, block, 0, stream, layout, buf, g, lc, f);
    else hipLaunchKernelGGL(k_gather_pop<ST_F16>, grid, block, 0, stream, layout, buf, g, lc, f);
    return hipGetLastError();
}

hipError_t launch_sample_pop(int storage, int layout, const void* buf, const Geom& g,
                             const float* inv_scale, const uint32_t* nodes, int count,
                             double* out, hipStream_t stream)
{
    if (storage == ST_F32X) storage = ST_F32;  // same storage format
    LoadCtx lc;
    for (int i = 0; i < 27; ++i) lc.inv_scale[i] = inv_scale ? inv_scale[i] : 1.0f;
    const dim3 grid((count + kBlock - 1) / kBlock), block(kBlock);
    if (storage == ST_F64) hipLaunchKernelGGL(k_sample_pop<ST_F64>, grid, block, 0, stream, layout, buf, g, lc, nodes, count, out);
    else if (storage == ST_F32) hipLaunchKernelGGL(k_sample_pop<ST_F32>, grid, block, 0, stream, layout, buf, g, lc, nodes, count, out);
    else hipLaunchKernelGGL(k_sample_pop<ST_F16>, grid, block, 0, stream, layout, buf, g, lc, nodes, count, out);
    return hipGetLastError();
}

hipError_t launch_scatter_pop(int storage, int layout, void* buf, const Geom& g, const float* scale,
                              const double* f, hipStream_t stream)
{
    if (storage == ST_F32X) storage = ST_F32;  // same storage format
    StoreCtx sc;
    for (int i = 0; i < 27; ++i) sc.scale[i] = scale ? scale[i] : 1.0f;
    const dim3 grid(grid_for(g.nnodes)), block(kBlock);
    if (storage == ST_F64) hipLaunchKernelGGL(k_scatter_pop<ST_F64>, grid, block, 0, stream, layout, buf, g, sc, f);
    else if (storage == ST_F32) hipLaunchKernelGGL(k_scatter_pop<ST_F32>, grid, block, 0, stream, layout, buf, g, sc, f);
    else hipLaunchKernelGGL(k_scatter_pop<ST_F16>, grid, block, 0, stream, layout, buf, g, sc, f);
    return hipGetLastError();
}

namespace {

template <bool FIELDS>
using FieldsFn = void (*)(const void*, Geom, LoadCtx, double*, double*, EnergySum*);

template <int S, bool FIELDS>
FieldsFn<FIELDS> fields_kernel(int layout)
{
    return layout == LY_PULL ? k_fields<S, LY_PULL, FIELDS>
                             : (layout == LY_AA_EVEN ? k_fields<S, LY_AA_EVEN, FIELDS>
                                                     : k_fields<S, LY_AA_ODD, FIELDS>);
}

}  // namespace

static_assert(sizeof(EnergySum) == 5 * sizeof(double), "energy_partials() counts doubles");
int energy_partials() { return 5 * (int)kEnergyGroups; }

hipError_t launch_fields(int storage, int layout, const void* buf, const Geom& g,
                         const float* inv_scale, double* rho, double* u, double* partial,
                         double* out, double* log, hipStream_t stream)
{
    if (storage == ST_F32X) storage = ST_F32;  // same storage format
    // the AA layouts are planes (load_node)
    if (layout != LY_PULL && !geom_is_planes(g)) return hipErrorInvalidValue;
    LoadCtx lc;
    for (int i = 0; i < 27; ++i) lc.inv_scale[i] = inv_scale ? inv_scale[i] : 1.0f;
    const uint32_t runs = (uint32_t)(((uint64_t)g.nnodes + 63) / 64);
    const uint32_t waves = std::min(runs, kEnergyGroups);
    const dim3 grid((waves + kBlock / 64 - 1) / (kBlock / 64)), block(kBlock);
    EnergySum* groups = reinterpret_cast<EnergySum*>(partial);
    const auto fn = storage == ST_F64   ? (u ? fields_kernel<ST_F64, true>(layout) : fields_kernel<ST_F64, false>(layout))
                    : storage == ST_F32 ? (u ? fields_kernel<ST_F32, true>(layout) : fields_kernel<ST_F32, false>(layout))
                                        : (u ? fields_kernel<ST_F16, true>(layout) : fields_kernel<ST_F16, false>(layout));
    hipLaunchKernelGGL(fn, grid, block, 0, stream, buf, g, lc, rho, u, groups);
    hipLaunchKernelGGL(k_energy_final, dim3(1), dim3(kFinalBlock), 0, stream, groups, g.nnodes, out, log);
    return hipGetLastError();
}

size_t series_partials(const Geom& g)
{
    return ((uint64_t)g.nnodes + 63) / 64 * (sizeof(EnergySum) / sizeof(double));
}

hipError_t launch_step_series(int storage, int variant, int sweep, uint32_t block,
                              const StepParams& p, double* runs, hipStream_t stream)
{
    StepFn step;   // whose shape and chunks the series kernel takes
    uint32_t grid;
    hipError_t e = step_launch_shape(storage, variant, sweep, false, block, false, p.g, &step, &grid);
    if (e != hipSuccess) return e;
    const bool c64 = chunks_of_64(p.g);
    SeriesFn fn;
    switch (storage) {
    case ST_F64: fn = series_kernel<ST_F64>(variant, sweep, c64); break;
    case ST_F32: fn = series_kernel<ST_F32>(variant, sweep, c64); break;
    case ST_F32X: fn = series_kernel<ST_F32X>(variant, sweep, c64); break;
    default: fn = series_kernel<ST_F16>(variant, sweep, c64); break;
    }
    hipLaunchKernelGGL(fn, dim3(grid), dim3(block), 0, stream, p, runs);
    return hipGetLastError();
}

hipError_t launch_series_sums(const Geom& g, int count, const double* runs, double* groups,
                              double* out, double* log, hipStream_t stream)
{
    EnergySum* gr = reinterpret_cast<EnergySum*>(groups);
    hipLaunchKernelGGL(k_energy_groups, dim3(kEnergyGroups / kBlock, count), dim3(kBlock), 0, stream,
                       reinterpret_cast<const EnergySum*>(runs), g.nnodes, gr);
    hipLaunchKernelGGL(k_energy_final, dim3(count), dim3(kFinalBlock), 0, stream, gr, g.nnodes, out, log);
    return hipGetLastError();
}

hipError_t launch_copy16(void* dst, const void* src, size_t n16, hipStream_t stream)
{
    if (n16 == 0) return hipSuccess;
    const size_t want = (n16 + kBlock - 1) / kBlock;
    const unsigned blocks = (unsigned)std::min<size_t>(want, 1u << 21);
    hipLaunchKernelGGL(k_copy16, dim3(blocks), dim3(kBlock), 0, stream, static_cast<u32x4*>(dst),
                       static_cast<const u32x4*>(src), n16);
    return hipGetLastError();
}

hipError_t launch_rewrite16(void* p, size_t n16, hipStream_t stream)
{
    if (n16 == 0) return hipSuccess;
    const size_t want = (n16 + kBlock - 1) / kBlock;
    const unsigned blocks = (unsigned)std::min<size_t>(want, 1u << 21);
    hipLaunchKernelGGL(k_rewrite16, dim3(blocks), dim3(kBlock), 0, stream, static_cast<u32x4*>(p),
                       n16, 0u);
    return hipGetLastError();
}

int reduce_partials() { return kReduceBlocks; }

hipError_t launch_curl(const Geom& g, const double* u, double* partial, double* out,
                       hipStream_t stream)
{
    const uint32_t lz = curl_planes(g);
    const uint64_t runs = (uint64_t)g.nx * g.ny * ((g.nz + lz - 1) / lz);
    const unsigned blocks = (unsigned)std::min<uint64_t>(kReduceBlocks, (runs + kBlock - 1) / kBlock);
    hipLaunchKernelGGL(k_curl, dim3(blocks), dim3(kBlock), 0, stream, g, lz, u, partial);
    hipLaunchKernelGGL(k_reduce_final_k<1>, dim3(1), dim3(kBlock), 0, stream, partial, (int)blocks, out);
    return hipGetLastError();
}

hipError_t launch_grad_stats(int order, const Geom& g, const double* u, double* partial,
                             double* out, hipStream_t stream)
{
    const uint32_t lz = grad_planes(g);
    const bool nodes = lz == 0;
    const unsigned blocks = nodes ? std::min<unsigned>(kReduceBlocks, grid_for(g.nnodes))
                                  : (unsigned)std::min<uint64_t>(kReduceBlocks, grad_items(g, lz));
    if (nodes && order == 8) hipLaunchKernelGGL(k_grad_nodes<8>, dim3(blocks), dim3(kBlock), 0, stream, g, u, partial);
    else if (nodes) hipLaunchKernelGGL(k_grad_nodes<2>, dim3(blocks), dim3(kBlock), 0, stream, g, u, partial);
    else if (order == 8) hipLaunchKernelGGL(k_grad_stats<8>, dim3(blocks), dim3(kBlock), 0, stream, g, lz, u, partial);
    else hipLaunchKernelGGL(k_grad_stats<2>, dim3(blocks), dim3(kBlock), 0, stream, g, lz, u, partial);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(k_reduce_final_k<8>, dim3(1), dim3(kBlock), 0, stream, partial, (int)blocks, out);
    return hipGetLastError();
}


hipError_t launch_gamma_stats(int storage, int variant, bool exact_gamma, int layout,
                              const void* buf, const Geom& g, const Coll& c,
                              const float* inv_scale, double* partial, double* out,
                              hipStream_t stream)
{
    LoadCtx lc;
    for (int i = 0; i < 27; ++i) lc.inv_scale[i] = inv_scale ? inv_scale[i] : 1.0f;
    const unsigned blocks = gamma_blocks(g);
    GammaFn fn;
    switch (storage) {
    case ST_F64: fn = exact_gamma ? gamma_kernel<ST_F64, true>(variant) : gamma_kernel<ST_F64, false>(variant); break;
    case ST_F32: fn = exact_gamma ? gamma_kernel<ST_F32, true>(variant) : gamma_kernel<ST_F32, false>(variant); break;
    case ST_F32X: fn = exact_gamma ? gamma_kernel<ST_F32X, true>(variant) : gamma_kernel<ST_F32X, false>(variant); break;
    default: fn = exact_gamma ? gamma_kernel<ST_F16, true>(variant) : gamma_kernel<ST_F16, false>(variant); break;
    }
    hipLaunchKernelGGL(fn, dim3(blocks), dim3(kBlock), 0, stream, layout, buf, g, c, lc, partial);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(k_gamma_final, dim3(1), dim3(kBlock), 0, stream, partial, (int)blocks, out);
    return hipGetLastError();
}

int corr_max_nx() { return kCorrMaxN; }
int corr_max_lags() { return kCorrMaxLags; }
size_t corr_partials(const Geom& g, int rmax)
{
    return (size_t)corr_plan(g, rmax).blocks * 2 * (rmax + 1);
}

hipError_t launch_corr_x(const Geom& g, const double* u, const double* mean_sum, int rmax,
                         double* partial, double* out, hipStream_t stream)
{
    const CorrPlan p = corr_plan(g, rmax);
    const size_t reduce = (size_t)(kBlock / p.lag_tiles) * p.lag_tiles * 8;
    const size_t lds = std::max<size_t>((size_t)p.lines * p.stride, reduce) * sizeof(double);
    hipLaunchKernelGGL(k_corr_x, dim3(p.blocks, 2, p.ranges), dim3(kBlock), lds, stream, g, p, u,
                       mean_sum, rmax, partial);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(k_corr_final, dim3(2 * (rmax + 1)), dim3(kBlock), 0, stream, partial,
                       (int)p.blocks, out);
    return hipGetLastError();
}

}  // namespace kbc

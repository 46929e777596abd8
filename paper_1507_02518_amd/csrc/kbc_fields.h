// kbc_fields.h -- density and velocity of a node from its stored populations,
// and the kinetic-energy sums over nodes, shared by every kernel that needs
// them, so that they all see the same bits: no operation here is contracted
// (a kernel's surroundings must not decide which products fuse), and the sums
// are taken in one fixed order, which depends on the node count alone.
//
// Order of the energy sums: the nodes in runs of 64 (one wavefront, one node
// per lane), each reduced to its sum of u and its sum of squares about its
// own mean; run j belongs to group j mod kEnergyGroups, whose runs are added
// in increasing order, as deviations of their means from the first run's; the
// groups in a fixed tree, as deviations from the first group's mean.  No sum
// of squares is taken about a point far from its mean, so nothing cancels
// against the flow's mean.
#pragma once

#include "kbc_step.h"

namespace kbc {

namespace {

// Stored populations of F(t) at node n, in the layout LY (the gather of the
// sweep of the same name; see node_update on the addressing).
template <int S, int LY>
__device__ __forceinline__ void load_node(const void* bufv, const Geom& g, uint32_t n,
                                          typename Traits<S>::T (&v)[27])
{
    using T = typename Traits<S>::T;
    constexpr uint32_t EB = sizeof(T);
    const char* buf = static_cast<const char*>(bufv);
    const uint64_t planeb = g.plane * EB;
    if constexpr (LY == LY_AA_EVEN) {
        const uint32_t off = n * EB;
#pragma unroll
        for (int i = 0; i < 27; ++i) {
            gchar_t* q = (gchar_t*)(buf + i * planeb);
            asm volatile("" : "+s"(q));
            v[i] = *reinterpret_cast<const T*>((const char*)q + off);
        }
    } else {
        uint32_t x, y, z;
        node_xyz(n, g, x, y, z);
        const uint32_t rowb = g.row * EB, slabb = g.slab * EB;
        auto xoff = [&](uint32_t xx) -> uint32_t {
            if constexpr (LY == LY_PULL) return (xx >> g.xshift) * (g.chunk * EB) + (xx & g.xmask) * EB;
            else return xx * EB;
        };
        const uint32_t bx[3] = {xoff(x + 1 == g.nx ? 0 : x + 1), xoff(x), xoff(x == 0 ? g.nx - 1 : x - 1)};
        const uint32_t by[3] = {(y + 1 == g.ny ? 0 : y + 1) * rowb, y * rowb, (y == 0 ? g.ny - 1 : y - 1) * rowb};
        const uint32_t bz[3] = {(z + 1 == g.nz ? 0 : z + 1) * slabb, z * slabb, (z == 0 ? g.nz - 1 : z - 1) * slabb};
#pragma unroll
        for (int i = 0; i < 27; ++i) {
            const int slot = LY == LY_PULL ? i : opp(i);
            v[i] = *reinterpret_cast<const T*>(buf + slot * planeb + (bz[i / 9] + by[(i / 3) % 3] + bx[i % 3]));
        }
    }
}

// rho = sum_i f_i and u = sum_i v_i f_i / rho (section I) in FP64 from the
// decoded populations; deviation forms sum the deviations and add the
// weights' share (1, 0).
template <int S, typename R>
__device__ __forceinline__ void node_velocity(const R (&f)[27], double& m, double (&u)[3])
{
#pragma clang fp contract(off)
    double a0[9], a1[9];
#pragma unroll
    for (int yz = 0; yz < 9; ++yz) {
        const double fm = f[3 * yz], f0 = f[3 * yz + 1], fp = f[3 * yz + 2];
        a0[yz] = (fm + fp) + f0;
        a1[yz] = fp - fm;
    }
    double s[3], d[3];   // over y: sums and differences for each z
    double jx = 0.0;
#pragma unroll
    for (int z = 0; z < 3; ++z) {
        s[z] = (a0[3 * z] + a0[3 * z + 2]) + a0[3 * z + 1];
        d[z] = a0[3 * z + 2] - a0[3 * z];
        const double px = (a1[3 * z] + a1[3 * z + 2]) + a1[3 * z + 1];
        jx = z == 0 ? px : jx + px;
    }
    const double jy = (d[0] + d[2]) + d[1], jz = s[2] - s[0];
    m = (s[0] + s[2]) + s[1];
    if constexpr (S != ST_F64) m += 1.0;
    const double ir = 1.0 / m;
    u[0] = jx * ir;
    u[1] = jy * ir;
    u[2] = jz * ir;
}

// Sums of the velocity over a set of nodes: sum of u, sum of |u - mean|^2 over
// the set, and how many of its nodes are not finite.
struct EnergySum {
    double s[3], m2, bad;
};
constexpr uint32_t kEnergyGroups = 4096;

__device__ __forceinline__ double shfl_from(double v, int lane)
{
    return __hiloint2double(__builtin_amdgcn_readlane(__double2hiint(v), lane),
                            __builtin_amdgcn_readlane(__double2loint(v), lane));
}

// The sums of one run of nodes: lane l has node l where `real` (the first
// `count` lanes).  Every lane returns them.  Deviations from the first
// node's velocity keep the squares' rounding at that of the local variation;
// the four sums share the butterfly, which takes 7 exchanges instead of 24.
__device__ __forceinline__ EnergySum run_energy(bool real, double count, double inv, double m,
                                                const double (&u)[3])
{
#pragma clang fp contract(off)
    const double c[3] = {shfl_from(u[0], 0), shfl_from(u[1], 0), shfl_from(u[2], 0)};
    double v[4];
#pragma unroll
    for (int a = 0; a < 3; ++a) v[a] = real ? u[a] - c[a] : 0.0;
    v[3] = (v[0] * v[0] + v[1] * v[1]) + v[2] * v[2];
    const uint32_t lane = threadIdx.x & 63;
    // lanes with bit 5 keep the sums 2 and 3, those with bit 4 the odd one
    const bool b5 = lane & 32, b4 = lane & 16;
    double p = b5 ? v[2] : v[0], q = b5 ? v[3] : v[1];
    p += __shfl_xor(b5 ? v[0] : v[2], 32, 64);
    q += __shfl_xor(b5 ? v[1] : v[3], 32, 64);
    double r = b4 ? q : p;
    r += __shfl_xor(b4 ? p : q, 16, 64);
#pragma unroll
    for (int off = 8; off > 0; off >>= 1) r += __shfl_xor(r, off, 64);
    const double d[3] = {shfl_from(r, 0), shfl_from(r, 16), shfl_from(r, 32)};
    const double sq = shfl_from(r, 48);
    EnergySum e;
#pragma unroll
    for (int a = 0; a < 3; ++a) e.s[a] = count * c[a] + d[a];
    e.m2 = sq - ((d[0] * d[0] + d[1] * d[1]) + d[2] * d[2]) * inv;
    const bool bad = real && !(isfinite(m) && isfinite(u[0]) && isfinite(u[1]) && isfinite(u[2]));
    e.bad = (double)__popcll(__builtin_amdgcn_ballot_w64(bad));
    return e;
}

// Adds sets of nodes: deviations from the mean c of the first of them.
struct EnergyAcc {
    double c[3], d[3], q, n, bad;
};

// b: a set of nb nodes, rb = 1 / nb.
__device__ __forceinline__ void add_energy(EnergyAcc& a, const EnergySum& b, double nb, double rb,
                                           bool first)
{
#pragma clang fp contract(off)
    double d2 = 0.0;
#pragma unroll
    for (int k = 0; k < 3; ++k) {
        const double mean = b.s[k] * rb;
        if (first) a.c[k] = mean;
        const double d = mean - a.c[k];
        a.d[k] = first ? 0.0 : a.d[k] + nb * d;
        d2 = k == 0 ? d * d : d2 + d * d;
    }
    a.q = first ? b.m2 : a.q + (b.m2 + nb * d2);
    a.n = first ? nb : a.n + nb;
    a.bad = first ? b.bad : a.bad + b.bad;
}

__device__ __forceinline__ EnergySum total_energy(const EnergyAcc& a)
{
#pragma clang fp contract(off)
    EnergySum e;
#pragma unroll
    for (int k = 0; k < 3; ++k) e.s[k] = a.n * a.c[k] + a.d[k];
    e.m2 = a.q - ((a.d[0] * a.d[0] + a.d[1] * a.d[1]) + a.d[2] * a.d[2]) / a.n;
    e.bad = a.bad;
    return e;
}

// Nodes of run j, and one over that.
__device__ __forceinline__ double run_count(uint32_t j, uint32_t nnodes, double& inv)
{
    const uint32_t left = nnodes - 64 * j;
    inv = left < 64 ? 1.0 / left : 0.015625;
    return left < 64 ? (double)left : 64.0;
}

// One step of a box (k_step without the exact stabilizer) that also writes
// the energy sums of the state it reads, one per run: a step reads every
// population of F(t) anyway, so k after each of n steps takes no pass of its own
// but for the last.  FP64 128^3 (bound by memory): 162 us per step, 153 for the
// step alone and 235 with a pass over the populations after it.
template <int S, int V, int SW, bool C64 = false>
__global__ void __launch_bounds__(kStepBlock) __attribute__((amdgpu_waves_per_eu(1, 8)))
k_series(StepParams p, double* __restrict__ runs)
{
    using R = typename Traits<S>::R;
    uint32_t order = SW != SW_PULL ? p.xcd_order : ORDER_PLAIN;
    if (order == ORDER_PAIRS && p.g.nx <= blockDim.x) order = ORDER_PLAIN;
    const uint32_t n0 = step_block(blockIdx.x, gridDim.x, order) * blockDim.x;
    const uint32_t n = n0 + threadIdx.x;
    // a wave without a node has no run; the barrier of the aligned stores
    // still counts it
    const bool real = n < p.g.nnodes, run = (n & ~63u) < p.g.nnodes;
    auto pre = [&](R (&f)[27]) {
        double m, u[3], inv;
        node_velocity<S>(f, m, u);
        const uint32_t j = n >> 6;
        if (run) {
            const double count = run_count(j, p.g.nnodes, inv);
            const EnergySum e = run_energy(real, count, inv, m, u);
            if ((n & 63) == 0) reinterpret_cast<EnergySum*>(runs)[j] = e;
        }
        // the step's own arithmetic stays that of k_step
#pragma unroll
        for (int i = 0; i < 27; ++i) asm volatile("" : "+v"(f[i]));
    };
    constexpr bool ALN = SW == SW_AA_ODD && KBC_AA_ALIGNED && (S == ST_F64 || S == ST_F32X);
    node_update<S, V, SW, false, ALN, C64, false>(p.src, p.dst, p.g, p.c, p.scale_exp,
                                           real ? n : p.g.nnodes - 1, n0, real, pre);
}

}  // namespace

}  // namespace kbc

// kbc_pair.h -- two time steps of a pull box in one sweep over memory.
//
// A single step reads and writes every population once and runs at the copy
// bandwidth, so the steps of a box cost what their traffic costs.  k_pair
// takes two steps per read and write of the lattice: a workgroup marches a
// tile of tx x ty columns through z, collides the (tx + 2)(ty + 2) nodes of a
// plane that the second step gathers from, hands their post-collision values
// over in LDS, and collides and stores the tile's nodes one plane behind.
// Both collisions are the function of the single step, on the same inputs:
// the populations it writes are the same bits.
//
// What it measured (FP64, s = d+t+q, ms per step): 256^3 1.22 -> 0.84,
// 192^3 0.507 -> 0.370, 128^3 0.151 -> 0.126, 64^3 0.025 -> 0.021.  The
// halo costs 1.25 x the reads at 256^3 (FETCH_SIZE; the writes are 1.00 x), so
// a pair moves 8.2 GB between L2 and the fabric instead of 14.5 GB.  With
// both collisions taken out the sweep still needs 0.80 of its 0.84 ms: the
// data movement bounds it, at 5.1 TB/s where a copy marched through the same
// tiles reaches 5.2.
//
// Why this split: two 256-thread workgroups per CU (FP64: 240 VGPRs, 78 KB of
// LDS each) overlap one's loads with the other's collisions.  One workgroup
// of one wave per SIMD with the next plane's loads in flight during the second
// collision ran at 1.07 ms, and the same with three waves less in FP32 at
// 0.58 against 0.49 ms.
#pragma once

#include "kbc_step.h"

namespace kbc {

namespace {

// LDS holds the post-collision values of the tile's nodes by destination:
// entry [slot][inner node] is the value that streams to that node within its
// plane.  The node at plane z - 1 takes v_z = -1 values of plane z, v_z = 0
// values of plane z - 1 and v_z = +1 values of plane z - 2, so the groups are
// kept for one, two and three planes: 9 + 18 + 27 slots.  In FP64 that is 1 KB
// more than half of a CU's LDS, and the last v_z = +1 population is kept for
// one plane there and in two registers after that (52 slots).
// CACHED: stores through the caches (cached_stores).
template <int S, int V, bool CACHED>
__global__ void __launch_bounds__(kPairBlock, pair_waves(S)) k_pair(PairParams pp)
{
    using T = typename Traits<S>::T;
    static_assert(sizeof(T) == sizeof(typename Traits<S>::R), "LDS holds stored populations");
    constexpr uint32_t EB = sizeof(T);
    constexpr int kRegs = S == ST_F64 ? 1 : 0;   // v_z = +1 populations kept in registers
    constexpr uint32_t kPlus = 9 - kRegs;        // and those kept in LDS
    constexpr uint32_t kSlots = 27 + 3 * kPlus + kRegs;
    __shared__ T lds[kSlots * kPairInner];

    const Geom& g = pp.g;
    const uint32_t tx = pp.p.tx, ty = pp.p.ty;
    const uint32_t t = threadIdx.x;
    // Consecutive tiles (x fastest, then y, then z) to one XCD, so that the
    // columns that neighbouring tiles share meet in one L2: 0.84 against 0.97
    // ms in the dispatch order at 256^3.
    const uint32_t tile = step_block(blockIdx.x, gridDim.x, ORDER_EIGHTHS);
    const uint32_t tyz = tile / pp.p.ntx, tzi = tyz / pp.p.nty;
    const uint32_t x0 = (tile - tyz * pp.p.ntx) * tx, y0 = (tyz - tzi * pp.p.nty) * ty;
    const uint32_t z0 = tzi * pp.p.lz;
    const uint32_t planes = g.nz - z0 < pp.p.lz ? g.nz - z0 : pp.p.lz;

    // first step: thread t has node (x0 - 1 + ex, y0 - 1 + ey), periodic;
    // spare threads, and rows past the box's last one, repeat the first node
    uint32_t ex = t % (tx + 2), ey = t / (tx + 2);
    const uint32_t rows = g.ny - y0 < ty ? g.ny - y0 : ty;
    const bool outer = ey < rows + 2;
    if (!outer) ex = ey = 0;
    const uint32_t xa = (x0 + g.nx - 1 + ex) % g.nx, ya = (y0 + g.ny - 1 + ey) % g.ny;
    const uint32_t rowb = g.row * EB, slabb = g.slab * EB;
    auto xoff = [&](uint32_t xx) -> uint32_t {
        return (xx >> g.xshift) * (g.chunk * EB) + (xx & g.xmask) * EB;
    };
    const uint32_t bx[3] = {xoff(xa + 1 == g.nx ? 0 : xa + 1), xoff(xa),
                            xoff(xa == 0 ? g.nx - 1 : xa - 1)};
    const uint32_t by[3] = {(ya + 1 == g.ny ? 0 : ya + 1) * rowb, ya * rowb,
                            (ya == 0 ? g.ny - 1 : ya - 1) * rowb};
    // byte offset of (x - v_x, y - v_y) in a plane, index (v_x + 1) + 3 (v_y + 1)
    uint32_t off[9];
#pragma unroll
    for (int k = 0; k < 9; ++k) off[k] = by[k / 3] + bx[k % 3];
    // whether the value sent along v stays in the tile, and its entry there
    bool okx[3], oky[3];
#pragma unroll
    for (int v = -1; v < 2; ++v) {
        okx[v + 1] = outer && ex + v - 1 < tx;
        oky[v + 1] = ey + v - 1 < ty;
    }
    const uint32_t own = (ey - 1) * tx + (ex - 1);

    // second step: thread t < tx ty has node (x0 + t % tx, y0 + t / tx)
    const uint32_t inner = t < tx * ty ? t : tx * ty - 1;
    const uint32_t xb = x0 + inner % tx, yb = y0 + inner / tx;
    const bool stores = t < tx * ty && xb < g.nx && yb < g.ny;
    uint32_t out = stores ? yb * rowb + xoff(xb) : 0;

    const uint64_t planeb = g.plane * EB;
    const char* src = static_cast<const char*>(pp.src);
    char* dst = static_cast<char*>(pp.dst);
    // A slot's base address in scalar registers, hidden from the compiler,
    // which would keep 27 loop-invariant 64-bit vector addresses and spill;
    // the offsets are hidden in each pass for the same reason.
    auto scalar = [](auto* q) {
        gchar_t* h = (gchar_t*)q;
        asm volatile("" : "+s"(h));
        return (decltype(q))h;
    };

    T h1 = T(0), h2 = T(0);   // kRegs: the value one and two planes back
    uint32_t z = z0 == 0 ? g.nz - 1 : z0 - 1, j3 = 0;   // j3 = j mod 3
#pragma unroll 1
    for (uint32_t j = 0; j < planes + 2; ++j) {
        const uint32_t zm = z == 0 ? g.nz - 1 : z - 1, zp = z + 1 == g.nz ? 0 : z + 1;
        T f[27];
#pragma unroll
        for (int k = 0; k < 9; ++k) asm volatile("" : "+v"(off[k]));
#pragma unroll
        for (int az = 0; az < 3; ++az) {
            const uint64_t zb = az == 0 ? zp : (az == 1 ? z : zm);
            const char* base = src + (9 * az * planeb + zb * slabb);
#pragma unroll
            for (int k = 0; k < 9; ++k) {
                base = scalar(base);
                f[9 * az + k] = *reinterpret_cast<const T*>(base + off[k]);
                base += planeb;
            }
        }
        collide<S, V>(f, pp.c);
        // pinned, so that the relaxation fuses as in the single step
#pragma unroll
        for (int i = 0; i < 27; ++i) asm volatile("" : "+v"(f[i]));

        const uint32_t zero = 9 + (j & 1) * 9, plus = 27 + j3 * kPlus;
        __syncthreads();   // the second step of the plane before has read its slots
#pragma unroll
        for (uint32_t k = 0; k < 9; ++k) {
            if (okx[k % 3] && oky[k / 3]) {
                const uint32_t d = own + ((int)(k / 3) - 1) * tx + ((int)(k % 3) - 1);
                lds[k * kPairInner + d] = f[k];
                lds[(zero + k) * kPairInner + d] = f[9 + k];
                lds[(k < kPlus ? plus + k : kSlots - 1) * kPairInner + d] = f[18 + k];
            }
        }
        __syncthreads();
        if (t < kPairInner) {
            const uint32_t zero1 = 9 + ((j & 1) ^ 1) * 9;                 // j - 1
            const uint32_t plus2 = 27 + (j3 == 2 ? 0 : j3 + 1) * kPlus;   // j - 2
            auto keep = [&] {
                if constexpr (kRegs) {
                    h2 = h1;
                    h1 = lds[(kSlots - 1) * kPairInner + t];
                }
            };
            if (j >= 2) {
                T q[27];
#pragma unroll
                for (uint32_t k = 0; k < 9; ++k) {
                    q[k] = lds[k * kPairInner + t];
                    q[9 + k] = lds[(zero1 + k) * kPairInner + t];
                    q[18 + k] = k < kPlus ? lds[(plus2 + k) * kPairInner + t] : h2;
                }
                keep();
                collide<S, V>(q, pp.c);
#pragma unroll
                for (int i = 0; i < 27; ++i) asm volatile("" : "+v"(q[i]));
                if (stores) {
                    char* base = dst + (uint64_t)zm * slabb;
                    asm volatile("" : "+v"(out));
#pragma unroll
                    for (int i = 0; i < 27; ++i) {
                        base = scalar(base);
                        st_pop<CACHED>(reinterpret_cast<T*>(base + out), q[i]);
                        base += planeb;
                    }
                }
            } else {
                keep();
            }
        }
        z = zp;
        j3 = j3 == 2 ? 0 : j3 + 1;
    }
}

}  // namespace

}  // namespace kbc

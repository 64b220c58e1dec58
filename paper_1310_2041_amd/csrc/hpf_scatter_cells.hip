// Density assignment over the cell list (beads in hpf_sort_by_cell order).
//
// The paper gathers: one thread per mesh point collects the fractions of the
// beads in the eight cells around it (Algorithm 1 Kernel 2), so no two threads
// write one point. Here the deposit is pushed from the beads, but still
// without global atomics and with exact integer sums:
//
//   pass 1  one workgroup per B^3 brick of cells reads the beads listed in
//           the brick (a contiguous range after the sort) and accumulates
//           their fixed-point weights in an LDS box of P = B + 1 + 2h mesh
//           points per axis, h = drift halo in cells; the box is stored to a
//           per-brick partial buffer;
//   pass 2  one thread per mesh point adds the partial boxes covering it
//           (per axis the own brick and at most one neighbour) and stores the
//           count;
//   fixup   beads that moved more than h cells out of their brick since the
//           sort (listed by pass 1, long lists found by pass 2), and beads the
//           sort could not bin, are added with global u64 atomics.
//
// Every bead is deposited exactly once, integer addition is exact and order
// free, so the counts equal those of hpf_density_scatter bit for bit.
#include "hpf_common.hpp"

#include <algorithm>

namespace hpf {

constexpr int kTcThreads = 256;
constexpr int kTcMaxB = 16;
constexpr int kTcMaxHalo = 2;

struct TileK {
    MeshK m;
    int32_t B;          // brick edge (tile of owned mesh points)
    int32_t h;          // drift halo in cells
    int32_t nb[3];      // bricks per axis
    uint32_t NK;        // number of sort keys (bricks); key NK = beads that cannot be binned
    int32_t P;          // B + 1 + 2h: mesh points per axis of a brick's deposit box
    int64_t ntiles;
};

// c / B for 0 <= c < 2^20 and 1 <= B <= 16, exactly: with m = ceil(2^32 / B) the excess
// m B - 2^32 is below 16, so c times it stays below 2^32. m is the same for a whole launch.
__device__ __forceinline__ uint32_t div_brick(int c, int B)
{
    return B == 1 ? (uint32_t)c : __umulhi((uint32_t)c, 0xffffffffu / (uint32_t)B + 1u);
}

// Sort key of a cell: the index of its brick of B^3 cells, x fastest.
__device__ __forceinline__ uint32_t brick_of(int cx, int cy, int cz, int B, const int nb[3])
{
    return (div_brick(cz, B) * (uint32_t)nb[1] + div_brick(cy, B)) * (uint32_t)nb[0] + div_brick(cx, B);
}

__device__ __forceinline__ int wrap_idx(int c, int M)
{
    c %= M;
    return c < 0 ? c + M : c;
}

// Periodic difference a - b folded into [-M/2, M/2].
__device__ __forceinline__ int periodic_delta(int a, int b, int M)
{
    int d = a - b;
    if (d > M / 2)
        d -= M;
    else if (d < -(M / 2))
        d += M;
    return d;
}

__device__ __forceinline__ void lds_add_u64(unsigned long long* p, unsigned long long v)
{
    __hip_atomic_fetch_add(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
}


// Cell of bead b relative to the deposit box of the brick whose first cell is
// (x0, y0, z0) and whose width is (ox, oy, oz) cells: true, with the local
// cell (lx, ly, lz), when the bead's 8 corners lie in the part of the box that
// the sum pass reads (box points [0, o + 2h] per axis).
__device__ __forceinline__ bool brick_box_cell(const BeadCell& b, const MeshK& m, int x0, int y0, int z0, int ox,
                                               int oy, int oz, int h, int& lx, int& ly, int& lz)
{
    lx = periodic_delta(b.c[0], x0, m.M[0]) + h;
    ly = periodic_delta(b.c[1], y0, m.M[1]) + h;
    lz = periodic_delta(b.c[2], z0, m.M[2]) + h;
    return lx >= 0 && lx <= ox - 1 + 2 * h && ly >= 0 && ly <= oy - 1 + 2 * h && lz >= 0 && lz <= oz - 1 + 2 * h;
}

// yz * q for yz <= 2^32 and q < 2^16, exactly: two products of at most 17 x 16 bits,
// which the 24-bit multiplier forms at full rate.
__device__ __forceinline__ uint64_t mul_w16(uint64_t yz, uint32_t q)
{
    const uint32_t yh = (uint32_t)(yz >> HPF_FIX_BITS) & 0x1ffffu, yl = (uint32_t)yz & 0xffffu;
    return ((uint64_t)(yh * q) << HPF_FIX_BITS) + (uint64_t)(yl * q);
}

// Adds one bead's 8 fixed-point corner weights to species t of an LDS box of
// P^3 points at local cell (lx, ly, lz). The corner weights come from two
// products: with w0 = 2^S - w1 per axis, W(0, ., .) = 2^S W_yz - W(1, ., .),
// and likewise along y and z. Every q is below 2^16 (cell_coord), so the masks
// change nothing; they let the compiler use the 24-bit multiplier.

__device__ __forceinline__ void box_deposit(unsigned long long* box, int P, int t, int lx, int ly, int lz,
                                            const BeadCell& b)
{
    const int P2 = P * P;
    const uint32_t q0 = b.q[0] & 0xffffu, q1 = b.q[1] & 0xffffu, q2 = b.q[2] & 0xffffu;
    const uint32_t yz11 = q1 * q2;
    const uint32_t yz01 = (q2 << HPF_FIX_BITS) - yz11;   // wy0 wz1
    const uint32_t yz10 = (q1 << HPF_FIX_BITS) - yz11;   // wy1 wz0
    const uint64_t yz00 = ((uint64_t)kOne << HPF_FIX_BITS) - yz11 - yz01 - yz10;
    unsigned long long* c0 = box + t * P2 * P + (lz * P + ly) * P + lx;
    const uint64_t a00 = mul_w16(yz00, q0), a10 = mul_w16(yz10, q0);
    const uint64_t a01 = mul_w16(yz01, q0), a11 = mul_w16(yz11, q0);
    lds_add_u64(c0, (yz00 << HPF_FIX_BITS) - a00);
    lds_add_u64(c0 + 1, a00);
    lds_add_u64(c0 + P, ((uint64_t)yz10 << HPF_FIX_BITS) - a10);
    lds_add_u64(c0 + P + 1, a10);
    lds_add_u64(c0 + P2, ((uint64_t)yz01 << HPF_FIX_BITS) - a01);
    lds_add_u64(c0 + P2 + 1, a01);
    lds_add_u64(c0 + P2 + P, ((uint64_t)yz11 << HPF_FIX_BITS) - a11);
    lds_add_u64(c0 + P2 + P + 1, a11);
}

// Pass 1: one workgroup per brick deposits the beads listed in that brick --
// one contiguous range of the cell-sorted arrays -- into an LDS box of
// P = B + 1 + 2h mesh points per axis starting h points below the brick (a
// bead that drifted at most h cells reaches points [x0 - h, x0 + B + h]). A
// thread takes kScBatch consecutive beads, so the lanes of one LDS atomic
// mostly sit in different cells. The box goes to a per-brick partial buffer
// with plain stores.
//
// Beads outside the box (strays) are listed in place: the brick's own stretch
// of a buffer of one entry per bead holds them from its first entry on, and
// their number in its last. When all of the brick's beads are strays there is
// no entry to spare for the number and no need of a list. So nothing is
// cleared beforehand and no workgroup waits for another's reservation.
//
// A workgroup alone on its CU is bound by its own chain (clear the box, load, deposit, store), so
// it takes the most threads there are: that is where no CU gets a second one, for want of bricks
// or of LDS. Otherwise 512 threads measure best. The three passes, with 256 threads of four
// beads / 512 of two / 1024 of two: 20,000 beads in 27 bricks 15.1 / 12.4 / 11.7 us; 3M beads in
// 216 bricks of 16 cells 72.1 / 50.6 / 42.5, in 1,728 of 8 cells 39.6 / 38.8 / 50.6; 1M in 512
// bricks 22.5 / 19.3 / 21.1. Where LDS and bricks make at least kScManyPerCu workgroups a CU, 256
// threads of two fill it too, and wait less for each other (with 512: 10,648 bricks of 3 cells, 95
// beads each, 55 us against 75; 8,000 of 5 cells, 250 beads, 65 against 78; 1,728 of 8 cells, halo 1,
// K = 2, 95 beads 27 against 30, 1200 beads 34.5 against 37).
constexpr int kScBatch = 2;
constexpr int kScBrickThreads = 512;
constexpr int kScManyPerCu = 6;
constexpr int kScLoneThreads = 1024;
constexpr int64_t kCus = 256;
constexpr size_t kLdsPerCu = 160 * 1024;

// Deposit of the beads listed in `brick` (cell_start of this system, i.e.
// already offset for batched systems) into an LDS box, stored to `out`.
template <int kThreads>
__device__ __forceinline__ void scatter_brick_body(const float3* __restrict__ R, const uint8_t* __restrict__ T,
                                                   int K, const TileK& tk,
                                                   const uint32_t* __restrict__ cell_start, int64_t brick,
                                                   unsigned long long* __restrict__ out,
                                                   uint32_t* __restrict__ strays)
{
    extern __shared__ unsigned long long smem[];
    __shared__ uint32_t stray_n;
    const int tid = threadIdx.x;
    const int B = tk.B, h = tk.h, P = tk.P;
    const int Mx = tk.m.M[0], My = tk.m.M[1], Mz = tk.m.M[2];
    const uint32_t first = cell_start[brick];
    const uint32_t last = cell_start[brick + 1];
    const int bx = (int)(brick % tk.nb[0]);
    const int by = (int)((brick / tk.nb[0]) % tk.nb[1]);
    const int bz = (int)(brick / ((int64_t)tk.nb[0] * tk.nb[1]));
    const int x0 = bx * B, y0 = by * B, z0 = bz * B;
    const int ox = min(B, Mx - x0), oy = min(B, My - y0), oz = min(B, Mz - z0);
    const int P2 = P * P, P3 = P2 * P;
    const int nbox = K * P3;
    unsigned long long* box = smem;
    for (int e = tid; e < nbox; e += kThreads)
        box[e] = 0ull;
    if (tid == 0)
        stray_n = 0;
    __syncthreads();
    for (uint32_t j0 = first; j0 < last; j0 += kThreads * kScBatch) {
        float3 rj[kScBatch];
        int tj[kScBatch];
        const uint32_t jb = j0 + tid * kScBatch;
#pragma unroll
        for (int u = 0; u < kScBatch; ++u) {
            if (jb + u < last) {
                rj[u] = R[jb + u];
                tj[u] = T[jb + u];
            }
        }
#pragma unroll
        for (int u = 0; u < kScBatch; ++u) {
            const uint32_t p = jb + u;
            if (p >= last)
                continue;
            const int t = tj[u];
            BeadCell b;
            int lx, ly, lz;
            const bool ok = bead_cell(rj[u], tk.m, b) && t < K;
            if (!ok || !brick_box_cell(b, tk.m, x0, y0, z0, ox, oy, oz, h, lx, ly, lz)) {
                const uint32_t slot = first + atomicAdd(&stray_n, 1u);
                if (slot < last - 1)
                    strays[slot] = p;
                continue;
            }
            box_deposit(box, P, t, lx, ly, lz, b);
        }
    }
    __syncthreads();
    if (tid == 0 && first < last)
        strays[last - 1] = stray_n;
    for (int e = tid; e < nbox; e += kThreads)
        out[e] = box[e];
}

template <int kThreads>
__global__ __launch_bounds__(kThreads) void k_scatter_bricks(const float3* __restrict__ R,
                                                             const uint8_t* __restrict__ T, int K, TileK tk,
                                                             const uint32_t* __restrict__ cell_start,
                                                             unsigned long long* __restrict__ partials,
                                                             uint32_t* __restrict__ strays)
{
    const int64_t brick = xcd_block(blockIdx.x, gridDim.x);
    const int P = tk.P;
    scatter_brick_body<kThreads>(R, T, K, tk, cell_start, brick, partials + brick * (int64_t)K * P * P * P, strays);
}

// Pass 2: one thread per mesh point sums the partial boxes that cover it and
// stores the count. Along an axis the box of brick b spans points
// [bB - h, bB + ob + h] (ob = the brick's width), periodically. With h < B
// only bricks b0 - 2 .. b0 + 2 (b0 = v / B) can reach v; the +-2 ones matter
// only next to the periodic seam when the last brick is narrower than h.
struct Cover {
    int n;
    int64_t off[5];     // brick * (brick stride) + local * (point stride) along this axis
};

// Writes into c (in LDS) the boxes that cover coordinate v along one axis. A
// brick reached twice through the periodic wrap (fewer than five bricks on the
// axis) is listed once. Brick numbers are kept in registers (constant indices
// only), so nothing of this goes to scratch memory.
__device__ __forceinline__ void covering(Cover& c, int v, int B, int h, int nb, int M, int64_t bstride,
                                         int lstride)
{
    int n = 0;
    int seen[5];
    const int b0 = v / B;
#pragma unroll
    for (int q = 0; q < 5; ++q) {
        int b = b0 + q - 2;
        if (b < 0)
            b += nb;
        else if (b >= nb)
            b -= nb;
        bool ok = b >= 0 && b < nb;         // fewer than 3 bricks on this axis
        seen[q] = ok ? b : -1 - q;
#pragma unroll
        for (int r = 0; r < q; ++r)
            ok &= seen[r] != b;
        const int ob = min(B, M - b * B);
        int l = v - (b * B - h);
        if (l < 0)
            l += M;
        else if (l >= M)
            l -= M;
        if (ok && l <= ob + 2 * h) {
            c.off[n] = b * bstride + (int64_t)l * lstride;
            ++n;
        }
    }
    c.n = n;
}

// True when no point lies in more than two boxes along any axis: at least three bricks, each wider
// than the overhang of its two neighbours together.
static bool two_boxes_at_most(const TileK& tk)
{
    for (int d = 0; d < 3; ++d)
        if (tk.nb[d] < 3 || std::min(tk.B, tk.m.M[d] - (tk.nb[d] - 1) * tk.B) <= 2 * tk.h)
            return false;
    return true;
}

// The entries that cover one point when no axis has more than two covering
// boxes (the usual case): the eight offsets and which of them exist. Built and
// read with constant indices only, so it stays in registers.
struct Cover2 {
    int64_t e[8];
    bool use[8];
};

__device__ __forceinline__ bool cover2_ok(const Cover& cx, const Cover& cy, const Cover& cz)
{
    return cx.n <= 2 && cy.n <= 2 && cz.n <= 2;
}

__device__ __forceinline__ Cover2 cover2(const Cover& cx, const Cover& cy, const Cover& cz)
{
    const bool hx = cx.n > 1, hy = cy.n > 1, hz = cz.n > 1;
    const int64_t x[2] = {cx.off[0], hx ? cx.off[1] : cx.off[0]};
    const int64_t y[2] = {cy.off[0], hy ? cy.off[1] : cy.off[0]};
    const int64_t z[2] = {cz.off[0], hz ? cz.off[1] : cz.off[0]};
    Cover2 c;
#pragma unroll
    for (int q = 0; q < 8; ++q) {
        const int a = q >> 2, b = (q >> 1) & 1, d = q & 1;
        c.e[q] = z[a] + y[b] + x[d];
        c.use[q] = (a == 0 || hz) && (b == 0 || hy) && (d == 0 || hx);
    }
    return c;
}

// Sum of the covering entries of species block kb (= k * P^3); every load of
// the point is issued before the additions.
__device__ __forceinline__ unsigned long long cover2_sum(const unsigned long long* __restrict__ partials,
                                                         const Cover2& c, int64_t kb)
{
    unsigned long long v[8];
#pragma unroll
    for (int q = 0; q < 8; ++q)
        v[q] = c.use[q] ? partials[c.e[q] + kb] : 0ull;
    unsigned long long sum = 0;
#pragma unroll
    for (int q = 0; q < 8; ++q)
        sum += v[q];
    return sum;
}

// Adds the covering entries of K species (P3 apart) to n, for any number of boxes per axis: the
// points beside the periodic seam when the last brick is thin (three boxes an axis), and bricks
// hardly wider than the halo. The nine entries of a z are loaded together, a missing one as a copy
// of another (an address that is valid, its value dropped). One after the other, the 27 of a corner
// made the last bricks of a thin mesh the ones that the whole launch waits for: a mesh of 18^3
// points in bricks of 8, finish with the potential 16 us and with loads under conditions 15.5; now
// 11.4 (58^3: 10.6, now 8.9).
template <int K>
__device__ __forceinline__ void add_covers(const unsigned long long* __restrict__ partials, const Cover& cx,
                                           const Cover& cy, const Cover& cz, int64_t P3, unsigned long long (&n)[K])
{
    const int nx = cx.n, ny = cy.n, nz = cz.n;
    if (nx <= 3 && ny <= 3) {
        int64_t xo[3], yo[3];
#pragma unroll
        for (int c = 0; c < 3; ++c) {
            xo[c] = cx.off[min(c, nx - 1)];
            yo[c] = cy.off[min(c, ny - 1)];
        }
        for (int a = 0; a < nz; ++a) {
            const unsigned long long* z = partials + cz.off[a];
#pragma unroll
            for (int k = 0; k < K; ++k) {
                unsigned long long v[9];
#pragma unroll
                for (int q = 0; q < 9; ++q)
                    v[q] = z[yo[q / 3] + xo[q % 3] + k * P3];
#pragma unroll
                for (int q = 0; q < 9; ++q)
                    n[k] += q / 3 < ny && q % 3 < nx ? v[q] : 0ull;
            }
        }
        return;
    }
    for (int a = 0; a < nz; ++a)
        for (int b = 0; b < ny; ++b)
            for (int c = 0; c < nx; ++c)
#pragma unroll
                for (int k = 0; k < K; ++k)
                    n[k] += partials[cz.off[a] + cy.off[b] + cx.off[c] + k * P3];
}

// One of three values by axis, selected as values (the arguments are copies).
__device__ __forceinline__ int pick3(int d, int a, int b, int c) { return d == 0 ? a : d == 1 ? b : c; }

// Cover lists of one brick's coordinates along each axis, with the offsets of
// the covering boxes' entries precomputed per axis (the offset of an entry in
// the partial buffer is the sum of its three axis terms), so that a point's
// covering entries cost three additions each. Call with all threads; ends
// with a barrier.
__device__ __forceinline__ void brick_covers(Cover (&cov)[3][kTcMaxB], const TileK& tk, int K, const int bxyz[3],
                                             const int o[3])
{
    const int B = tk.B, h = tk.h, P = tk.P;
    const int64_t P3K = (int64_t)K * P * P * P;
    const int tid = threadIdx.x;
    if (tid < 3 * B) {
        // the axis is chosen among values: a run-time index into the per-axis arrays
        // (or a conditional over them, which selects an address) would place them in
        // scratch memory
        const int d = tid / B, i = tid % B;
        const int od = pick3(d, o[0], o[1], o[2]);
        if (i < od) {
            const int bd = pick3(d, bxyz[0], bxyz[1], bxyz[2]);
            const int nbd = pick3(d, tk.nb[0], tk.nb[1], tk.nb[2]);
            const int Md = pick3(d, tk.m.M[0], tk.m.M[1], tk.m.M[2]);
            const int64_t bstride = d == 0 ? P3K : d == 1 ? tk.nb[0] * P3K : (int64_t)tk.nb[0] * tk.nb[1] * P3K;
            const int lstride = pick3(d, 1, P, P * P);
            covering(cov[d][i], bd * B + i, B, h, nbd, Md, bstride, lstride);
        }
    }
    __syncthreads();
}

// Local coordinates of point e of a brick of o[0] x o[1] x o[2] points (x fastest).
__device__ __forceinline__ void brick_point(int e, const int o[3], int B, int& ix, int& iy, int& iz)
{
    if (B == 8 && o[0] == 8 && o[1] == 8) {
        ix = e & 7;
        iy = (e >> 3) & 7;
        iz = e >> 6;
    } else {
        ix = e % o[0];
        const int r1 = e / o[0];
        iy = r1 % o[1];
        iz = r1 / o[1];
    }
}

// One workgroup per brick: the cover lists of the brick's coordinates along
// each axis are built once in LDS, then each thread sums the partial boxes for
// its points (consecutive threads -> consecutive x -> coalesced reads).
// With kAdd the sums are added to the counts instead of stored.
template <bool kAdd = false>
__device__ __forceinline__ void scatter_sum_body(const unsigned long long* __restrict__ partials,
                                                 const TileK& tk, int K, int64_t brick,
                                                 unsigned long long* __restrict__ counts)
{
    __shared__ Cover cov[3][kTcMaxB];
    const int B = tk.B, P = tk.P, P3 = P * P * P;
    const int bxyz[3] = {(int)(brick % tk.nb[0]), (int)((brick / tk.nb[0]) % tk.nb[1]),
                         (int)(brick / ((int64_t)tk.nb[0] * tk.nb[1]))};
    int o[3];
#pragma unroll
    for (int d = 0; d < 3; ++d)
        o[d] = min(B, tk.m.M[d] - bxyz[d] * B);
    brick_covers(cov, tk, K, bxyz, o);
    const int npts = o[0] * o[1] * o[2];
    const int Mx = tk.m.M[0], My = tk.m.M[1];
    for (int e = threadIdx.x; e < npts; e += (int)blockDim.x) {
        int ix, iy, iz;
        brick_point(e, o, B, ix, iy, iz);
        const Cover& cx = cov[0][ix];
        const Cover& cy = cov[1][iy];
        const Cover& cz = cov[2][iz];
        const int64_t dst = ((int64_t)(bxyz[2] * B + iz) * My + (bxyz[1] * B + iy)) * Mx + bxyz[0] * B + ix;
        if (cover2_ok(cx, cy, cz)) {
            const Cover2 c2 = cover2(cx, cy, cz);
            for (int k = 0; k < K; ++k) {
                const unsigned long long sum = cover2_sum(partials, c2, (int64_t)k * P3);
                if (kAdd)
                    counts[(int64_t)k * tk.m.nm + dst] += sum;
                else
                    counts[(int64_t)k * tk.m.nm + dst] = sum;
            }
            continue;
        }
        for (int k = 0; k < K; ++k) {
            unsigned long long sum[1] = {0};
            add_covers<1>(partials + (int64_t)k * P3, cx, cy, cz, P3, sum);
            if (kAdd)
                counts[(int64_t)k * tk.m.nm + dst] += sum[0];
            else
                counts[(int64_t)k * tk.m.nm + dst] = sum[0];
        }
    }
}

// Up to one thread per point of the brick (B^3 <= 512): launched with 512
// threads when there are few bricks (a small mesh must still fill the chip),
// else with 256.
constexpr int kSumThreads = 512;
constexpr int64_t kSumFewBricks = 2048;

static dim3 sum_block(int64_t ntiles) { return dim3(ntiles < kSumFewBricks ? kSumThreads : kSumThreads / 2); }

// A brick's list of strays: its bead range and the list's length. Lengths are held to the
// range, so that a buffer that another call writes meanwhile gives wrong counts and no wild access.
struct StrayList {
    uint32_t at, beads, len;
    bool shared;
};

constexpr uint32_t kSharedList = 1u << 31;           // in a list's length: all workgroups take part
constexpr uint32_t kLongList = 2048;                 // strays above which a list is shared
constexpr uint32_t kLongLists = 31;                  // as many as the 64 entries behind the lists hold

__device__ __forceinline__ StrayList stray_list(const uint32_t* __restrict__ strays, uint32_t first, uint32_t last)
{
    StrayList l{first, 0u, 0u, false};
    if (first < last) {
        const uint32_t n = strays[last - 1];
        l.beads = last - first;
        l.len = min(n & ~kSharedList, l.beads);
        l.shared = (n & kSharedList) != 0;
    }
    return l;
}

// The box sums' launch ends before the strays' begins, so it finds the long lists for it, in one
// workgroup beside those of the bricks: marks them, and writes their number and ranges behind the
// lists (N entries). range(b, first, last) gives the bead range of list b < n. While a list was
// its brick's workgroup's alone, 1M beads that had all left one brick took 17.5 ms, and 3M in a
// droplet of 40^3 cells of 192^3 4.0; now 1.9 and 1.4.
constexpr int kScanLists = 4;

template <class Range>
__device__ __forceinline__ void find_long_lists(uint32_t* __restrict__ strays, int64_t N, int64_t n, Range range)
{
    __shared__ uint32_t found;
    if (threadIdx.x == 0)
        found = 0u;
    __syncthreads();
    uint32_t* out = strays + N;
    for (int64_t b0 = threadIdx.x; b0 < n; b0 += kScanLists * (int64_t)blockDim.x) {
        uint32_t first[kScanLists], last[kScanLists];
        StrayList l[kScanLists];
#pragma unroll
        for (int u = 0; u < kScanLists; ++u)
            range(min(b0 + u * (int64_t)blockDim.x, n - 1), first[u], last[u]);
#pragma unroll
        for (int u = 0; u < kScanLists; ++u)
            l[u] = stray_list(strays, first[u], last[u]);
#pragma unroll
        for (int u = 0; u < kScanLists; ++u) {
            if (b0 + u * (int64_t)blockDim.x >= n || l[u].len <= kLongList)
                continue;
            const uint32_t slot = atomicAdd(&found, 1u);
            if (slot < kLongLists) {
                out[1 + 2 * slot] = first[u];
                out[2 + 2 * slot] = last[u];
                strays[last[u] - 1] = l[u].len | kSharedList;
            }
        }
    }
    __syncthreads();
    if (threadIdx.x == 0)
        out[0] = min(found, kLongLists);
}

// Without kAdd (a scatter with strays) the launch has kFindBlocks workgroups before those of the
// bricks (a whole turn of the XCDs, so that a brick's stays on its own); the first finds the long
// lists. With it, N, cell_start and strays are not read.
constexpr int kFindBlocks = 8;

template <bool kAdd>
__global__ __launch_bounds__(kSumThreads) void k_scatter_sum(const unsigned long long* __restrict__ partials,
                                                     TileK tk, int K, int64_t N,
                                                     const uint32_t* __restrict__ cell_start,
                                                     uint32_t* __restrict__ strays,
                                                     unsigned long long* __restrict__ counts)
{
    constexpr int skip = kAdd ? 0 : kFindBlocks;
    if (!kAdd && (int)blockIdx.x < skip) {
        if (blockIdx.x == 0)
            find_long_lists(strays, N, tk.ntiles, [&](int64_t b, uint32_t& first, uint32_t& last) {
                first = cell_start[b];
                last = cell_start[b + 1];
            });
        return;
    }
    scatter_sum_body<kAdd>(partials, tk, K, xcd_block(blockIdx.x - skip, gridDim.x - skip), counts);
}

__device__ __forceinline__ void atomic_add_u64_agent(unsigned long long* p, unsigned long long v)
{
    __hip_atomic_fetch_add(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Eight global u64 atomics of one bead; false if it cannot be binned.
__device__ __forceinline__ bool deposit_global(const float3& r, int t, int K, const MeshK& m,
                                               unsigned long long* __restrict__ counts)
{
    BeadCell b;
    if (!(bead_cell(r, m, b) && t < K))
        return false;
    const int32_t x0 = b.c[0], x1 = next_wrap(x0, m.M[0]);
    const int32_t y0 = b.c[1], y1 = next_wrap(y0, m.M[1]);
    const int32_t z0 = b.c[2], z1 = next_wrap(z0, m.M[2]);
    const uint64_t wx0 = kOne - b.q[0], wx1 = b.q[0];
    const uint64_t wy0 = kOne - b.q[1], wy1 = b.q[1];
    const uint64_t wz0 = kOne - b.q[2], wz1 = b.q[2];
    unsigned long long* nk = counts + (int64_t)t * m.nm;
    const int64_t r00 = ((int64_t)z0 * m.M[1] + y0) * m.M[0];
    const int64_t r10 = ((int64_t)z0 * m.M[1] + y1) * m.M[0];
    const int64_t r01 = ((int64_t)z1 * m.M[1] + y0) * m.M[0];
    const int64_t r11 = ((int64_t)z1 * m.M[1] + y1) * m.M[0];
    atomic_add_u64_agent(nk + r00 + x0, wx0 * wy0 * wz0);
    atomic_add_u64_agent(nk + r00 + x1, wx1 * wy0 * wz0);
    atomic_add_u64_agent(nk + r10 + x0, wx0 * wy1 * wz0);
    atomic_add_u64_agent(nk + r10 + x1, wx1 * wy1 * wz0);
    atomic_add_u64_agent(nk + r01 + x0, wx0 * wy0 * wz1);
    atomic_add_u64_agent(nk + r01 + x1, wx1 * wy0 * wz1);
    atomic_add_u64_agent(nk + r11 + x0, wx0 * wy1 * wz1);
    atomic_add_u64_agent(nk + r11 + x1, wx1 * wy1 * wz1);
    return true;
}

// The strays of n <= kTcThreads lists, deposited by the whole workgroup; thread i < n brings
// list i (read by each thread for its own, so that the chain of reads is walked once and not
// list after list). With parts > 1, every parts-th turn of each list from `part` on.
template <class Deposit>
__device__ __forceinline__ void deposit_lists(const uint32_t* __restrict__ strays, int64_t n, int part, int parts,
                                              const StrayList& mine, Deposit deposit)
{
    __shared__ uint32_t at[kTcThreads], len[kTcThreads], beads[kTcThreads];
    const int tid = threadIdx.x;
    if (tid < n) {
        at[tid] = mine.at;
        beads[tid] = mine.beads;
        len[tid] = mine.len;
    }
    if (!__syncthreads_or(tid < n && mine.len != 0))
        return;
    for (int64_t q = 0; q < n; ++q)
        for (uint32_t i = part * kTcThreads + tid; i < len[q]; i += parts * kTcThreads) {
            const uint32_t p = len[q] == beads[q] ? at[q] + i : strays[at[q] + i];
            if (p - at[q] < beads[q])
                deposit(q, p);
        }
}

// The lists of this workgroup's bricks: list g, g + groups, ... of n (range as in
// find_long_lists), but for the shared ones; deposit(list, bead).
template <class Range, class Deposit>
__device__ __forceinline__ void deposit_own_lists(const uint32_t* __restrict__ strays, int64_t n, int64_t g,
                                                  int64_t groups, int part, int parts, Range range, Deposit deposit)
{
    for (int64_t b0 = g; b0 < n; b0 += groups * kTcThreads) {
        uint32_t first, last;
        range(min(b0 + groups * threadIdx.x, n - 1), first, last);
        StrayList l = stray_list(strays, first, last);
        if (l.shared)
            l.len = 0u;
        const int64_t here = min((int64_t)kTcThreads, (n - b0 + groups - 1) / groups);
        deposit_lists(strays, here, part, parts, l, [&](int64_t q, uint32_t p) { deposit(b0 + groups * q, p); });
        __syncthreads();
    }
}

// The shared lists, by all workgroups.
template <class Deposit>
__device__ __forceinline__ void deposit_shared_lists(const uint32_t* __restrict__ strays, int64_t N, Deposit deposit)
{
    const uint32_t* in = strays + N;
    const uint32_t n = min(in[0], kLongLists);
    if (n == 0)                          // uniform
        return;
    const uint32_t q = min(threadIdx.x, n - 1);
    const uint32_t last = min((int64_t)in[2 + 2 * q], N), first = min(in[1 + 2 * q], last);
    deposit_lists(strays, n, blockIdx.x, gridDim.x, stray_list(strays, first, last),
                  [&](int64_t, uint32_t p) { deposit(p); });
}

// Workgroups of the stray pass: up to kStrayBlocks bricks get one or several each. With more, a
// workgroup takes every kStrayGroups-th brick, so that neighbouring bricks, which tend to be as
// full as each other, go to different ones (a prime, which no mesh's strides have for a factor).
constexpr int kStrayBlocks = 512;
constexpr int kStrayGroups = 509;

// Global-atomic deposit of the stray beads and of the beads the sort could not
// bin (storage indices [cell_start[NK], N)).
__global__ __launch_bounds__(kTcThreads) void k_scatter_strays(const float3* __restrict__ R,
                                                               const uint8_t* __restrict__ T, int64_t N,
                                                               int K, MeshK m, uint32_t NK, int parts,
                                                               const uint32_t* __restrict__ cell_start,
                                                               const uint32_t* __restrict__ strays,
                                                               unsigned long long* __restrict__ counts)
{
    bool bad = false;
    auto deposit = [&](uint32_t p) { bad |= !deposit_global(R[p], T[p], K, m, counts); };
    deposit_own_lists(strays, NK, blockIdx.x / parts, gridDim.x / parts, blockIdx.x % parts, parts,
                      [&](int64_t b, uint32_t& first, uint32_t& last) {
                          first = cell_start[b];
                          last = cell_start[b + 1];
                      },
                      [&](int64_t, uint32_t p) { deposit(p); });
    deposit_shared_lists(strays, N, deposit);
    for (int64_t p = (int64_t)cell_start[NK] + (int64_t)blockIdx.x * kTcThreads + threadIdx.x; p < N;
         p += (int64_t)gridDim.x * kTcThreads)
        bad |= !deposit_global(R[p], T[p], K, m, counts);
    if (bad)
        raise_flag(HPF_FLAG_BAD_BEAD);
}

size_t scatter_cells_smem(int K, int P)
{
    return sizeof(unsigned long long) * (size_t)K * P * P * P;
}

// Whether LDS (smem bytes a workgroup) and bricks make kScManyPerCu workgroups a CU.
static bool many_bricks(const TileK& tk, size_t smem)
{
    return tk.ntiles >= kScManyPerCu * kCus && kScManyPerCu * smem <= kLdsPerCu;
}

size_t scatter_cells_partials(int64_t ntiles, int K, int P)
{
    return sizeof(unsigned long long) * (size_t)ntiles * K * P * P * P;
}

hpf_status_t launch_scatter_cells(const float* R, const uint8_t* T, int64_t N, const TileK& tk, int K,
                                  const uint32_t* cell_start, uint64_t* counts, uint32_t* strays,
                                  unsigned long long* partials, hipStream_t s)
{
    auto* c = reinterpret_cast<unsigned long long*>(counts);
    auto* Rp = reinterpret_cast<const float3*>(R);
    const size_t smem = scatter_cells_smem(K, tk.P);
    auto go = [&](auto kernel, int threads) {
        // gfx950 has 160 KiB of LDS per CU; opt in above the 64 KiB default
        if (smem > 65536 && hipFuncSetAttribute(reinterpret_cast<const void*>(kernel),
                                                hipFuncAttributeMaxDynamicSharedMemorySize,
                                                (int)smem) != hipSuccess)
            return HPF_EINVAL;
        hipLaunchKernelGGL(kernel, dim3((unsigned)tk.ntiles), dim3(threads), smem, s, Rp, T, K, tk, cell_start,
                           partials, strays);
        return HPF_OK;
    };
    const bool lone = tk.ntiles <= kCus || 2 * smem > kLdsPerCu;
    const bool many = many_bricks(tk, smem);
    const hpf_status_t st = lone   ? go(k_scatter_bricks<kScLoneThreads>, kScLoneThreads)
                            : many ? go(k_scatter_bricks<kTcThreads>, kTcThreads)
                                   : go(k_scatter_bricks<kScBrickThreads>, kScBrickThreads);
    if (st != HPF_OK)
        return st;
    hipLaunchKernelGGL(k_scatter_sum<false>, dim3((unsigned)tk.ntiles + kFindBlocks), sum_block(tk.ntiles), 0, s,
                       partials, tk, K, N, cell_start, strays, c);
    const int parts = (int)std::max<int64_t>(1, kStrayBlocks / tk.NK);
    const int blocks = tk.NK <= kStrayBlocks ? kStrayBlocks / parts * parts : kStrayGroups;
    hipLaunchKernelGGL(k_scatter_strays, dim3(blocks), dim3(kTcThreads), 0, s, Rp, T, N, K, tk.m, tk.NK, parts,
                       cell_start, strays, c);
    return hipGetLastError() == hipSuccess ? HPF_OK : HPF_EHIP;
}

}  // namespace hpf

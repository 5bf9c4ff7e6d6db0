// Owner-map maintenance and state import/export kernels (gfx950).
//
// The owner map is kept incrementally when spheres move, in one launch with
// one to four wavefronts per sphere, in any order:
//  - the sphere enters the nodes of its new ball that its old one did not
//    cover: it takes each unless a wall or a lower-index sphere whose new ball
//    also covers it owns it, by compare-and-swap from any other owner (a
//    higher index, the fluid, or a lower index that is leaving the node);
//  - it leaves the nodes of its old ball that its new one does not cover:
//    those it still owns turn fluid by compare-and-swap, and are refilled with
//    the equilibrium at rho0 and the velocity they had as a solid (the
//    solid-side Maxwell equilibrium of Sec. 2.3).
// A node in both balls needs a look only where balls overlap: a sphere that
// was refused a node of its ball, or lost one, is marked, and a marked sphere
// goes through its whole new ball in the next update.  An unmarked sphere owns
// every node of its ball that is not a wall's.
// Every node ends with the owner of the new geometry whatever the order of
// the wavefronts: the lowest-index sphere whose new ball covers it (walls
// first), else fluid.  A node refilled and then taken by another sphere was
// refilled for nothing: a solid node's populations are never read.
#include "lbm_device.h"
#include "lbm_internal.h"
#include "lbm_linkmath.h"

#include <hip/hip_runtime.h>
#include <math.h>

#include <algorithm>

namespace lbm {
namespace {

using namespace dev;

// A node of the lattice: wrapped coordinates and index.
struct Node {
    int px, py, pz;
    uint32_t n;
};

// Compare-and-swap of a 16-bit owner code (through its 32-bit word): the
// code found (expect on success).
__device__ __forceinline__ uint16_t cas_u16(uint16_t *addr, uint16_t expect, uint16_t val)
{
    unsigned int *w = (unsigned int *)((uintptr_t)addr & ~(uintptr_t)3);
    const unsigned int sh = ((uintptr_t)addr & 2) ? 16u : 0u;
    unsigned int old = __hip_atomic_load(w, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    while (true) {
        const uint16_t cur = (uint16_t)((old >> sh) & 0xffffu);
        if (cur != expect) return cur;
        const unsigned int nw = (old & ~(0xffffu << sh)) | ((unsigned int)val << sh);
        const unsigned int prev = atomicCAS(w, old, nw);
        if (prev == old) return expect;
        old = prev;  // this code or the other half of the word changed
    }
}

// The node turned from fluid to solid or back: its bit of the solid bitmap is
// flipped, with its periodic copies at the row's ends.  Every change of a
// node's owner is a compare-and-swap, so the changes of a node are in one
// order and its flips add up to its final state, in whatever order they land.
__device__ __forceinline__ void flip_bit(const GeomArgs &g, int px, int py, int pz)
{
    uint32_t *row = g.bits + (size_t)bit_row_words(g.nx) * ((size_t)py + (size_t)g.ny * pz);
    auto flip = [&](int p) { atomicXor(row + (p >> 5), 1u << (p & 31)); };
    flip(px + 1);
    if (px == 0) flip(g.nx + 1);
    if (px == g.nx - 1) flip(0);
}

// Sphere b is marked: it may not own every node of its new ball.
__device__ __forceinline__ void mark(const GeomArgs &g, int b)
{
    __hip_atomic_store(g.lost + b, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Sphere `id` (new geometry) takes node v, found with owner o.
__device__ __forceinline__ void enter_node(const GeomArgs &g, const Node &v, uint16_t o, uint16_t id)
{
    while (true) {
        if (o < g.n_walls || o == id) return;
        if (o < id) {
            // a lower-index sphere keeps the node if its new ball covers it
            const int b = o - g.n_walls;
            if (b < g.nb2) {
                const double *Bo = g.bodies2 + (size_t)b * kBodyStride;
                // (the record in one round trip: both tests without a branch)
                const double o4[10] = {Bo[0], Bo[1], Bo[2], 0.0, 0.0, 0.0, 0.0, 0.0, 0.0, Bo[9]};
                if ((int)body_ok(o4, g.nx, g.ny, g.nz) & (int)inside(o4, v.px, v.py, v.pz, g.nx, g.ny, g.nz)) {
                    mark(g, id - g.n_walls);
                    return;
                }
            }
        }
        const uint16_t prev = cas_u16(g.own + v.n, o, id);
        if (prev == o) {
            if (o >= kVacated) flip_bit(g, v.px, v.py, v.pz);
            else if (o > id && o - g.n_walls < g.nb2) mark(g, o - g.n_walls);
            return;
        }
        o = prev;
    }
}

// The nodes of ball B in the column (px, py) of the lattice: the unwrapped z
// range [lo, hi] (empty when lo > hi), exactly those for which inside() holds.
// The range is [Z - h, Z + h] with h^2 = R^2 - (dx^2 + dy^2).  A first pass
// in FP32 takes the offsets from the box origin (kx - ox for the column at
// box position kx; |offsets| <= R + 1) and bounds h^2 within +-eps2, an upper
// bound of its FP32 error with a wide margin; where both bounds give the same
// end nodes those are the ends of the exact range (the FP64 test of inside()
// differs from the exact one only within about 1e-13 of the surface).
// Otherwise the FP64 pass decides: dx^2 + dy^2 formed as inside() forms it
// and FP64 h settle every node farther than 1e-6 from both ends (their
// roundings move an end by about 2^-52 R^2 / h < 1e-7 while h > max(1e-4,
// 1e-8 R^2)), and inside() itself decides the rest: along a column |p - X|^2
// grows with |z - Z| (each rounding is monotone), so the nodes inside form
// one range.
struct BallCols {
    float ox, oy, oz;  // centre minus box origin, per axis
    float r2, eps2;    // R^2 and the error bound of h^2
    float m;           // bound of the error of a range end, with margin
};

__device__ __forceinline__ BallCols ball_cols(const double *B, const Box &bx)
{
    BallCols bc;
    bc.ox = (float)(B[0] - (double)bx.x0);
    bc.oy = (float)(B[1] - (double)bx.y0);
    bc.oz = (float)(B[2] - (double)bx.z0);
    bc.r2 = (float)(B[9] * B[9]);
    // the FP32 error of h^2 stays below 1e-6 (R + 1)^2 and that of an end
    // (the offset oz, the sums, the square root) below 1e-6 (R + 1): the
    // bounds below are ten times these
    bc.eps2 = 1e-5f * (bc.r2 + 1.0f) + 2e-5f * (float)B[9];
    bc.m = 1e-5f * ((float)B[9] + 1.0f);
    return bc;
}

__device__ __forceinline__ void column_range(const double *B, const Box &bx, const BallCols &bc, int kx, int ky,
                                             int px, int py, int nx, int ny, int nz, int &lo, int &hi)
{
#pragma clang fp contract(off)
    lo = 1;
    hi = 0;
    {
        const float dx = (float)kx - bc.ox, dy = (float)ky - bc.oy;
        const float h2 = bc.r2 - (dx * dx + dy * dy);
        if (h2 < -bc.eps2) return;  // no node of the column within R
        if (h2 > bc.eps2) {
            const float hl = __builtin_sqrtf(h2 - bc.eps2), hh = __builtin_sqrtf(h2 + bc.eps2);
            const float m = bc.m;
            // an end settled this way lies at least m / 2 from every node
            const int l0 = (int)ceilf(bc.oz - hh - m), l1 = (int)ceilf(bc.oz - hl + m);
            const int h0 = (int)floorf(bc.oz + hl - m), h1 = (int)floorf(bc.oz + hh + m);
            if (l0 == l1 && h0 == h1) {
                lo = bx.z0 + l0;
                hi = bx.z0 + h0;
                return;
            }
        }
    }
    const double r2 = B[9] * B[9];
    const double dx = min_image((double)px - B[0], nx);
    const double dy = min_image((double)py - B[1], ny);
    const double sxy = dx * dx + dy * dy;
    if (sxy > r2) return;  // |p - X|^2 >= sxy for every node of the column
    const double h = sqrt(r2 - sxy);
    const double za = B[2] - h, zb = B[2] + h;
    const double fa = floor(za), fb = floor(zb);
    lo = (int)fa + 1;
    hi = (int)fb;
    constexpr double kSure = 1e-6;
    if (h > 1e-4 && h > 1e-8 * r2 && za - fa > kSure && fa + 1.0 - za > kSure && zb - fb > kSure && fb + 1.0 - zb > kSure)
        return;
    const int zmin = (int)ceil(B[2] - B[9]), zmax = (int)floor(B[2] + B[9]);  // the ball's box
    lo = max(lo - 2, zmin);
    hi = min(hi + 1, zmax);
    while (lo <= hi && !inside(B, px, py, wrap1(lo, nz), nx, ny, nz)) ++lo;
    while (hi >= lo && !inside(B, px, py, wrap1(hi, nz), nx, ny, nz)) --hi;
}

__global__ __launch_bounds__(kBlock) void k_link_records(GeomArgs g, const double *wrec)
{
    const int i = blockIdx.x * kBlock + threadIdx.x;
    if (i >= g.n_walls + g.nb) return;
    static_cast<LinkRec *>(g.lrec)[i].k =
        sphere_k(i < g.n_walls ? wrec + (size_t)i * kBodyStride : g.bodies + (size_t)(i - g.n_walls) * kBodyStride);
}

// A sphere table of n doubles from pinned host memory, read over PCIe: one
// launch where a copy command and an event took two calls.  The last block to
// finish tells the host that the table has been read (seen, pinned; left:
// blocks done, 0 between launches).  With the forces written to pinned memory
// by the kernel that forms them, a step of a 96^3 box with 400 spheres, tables
// and forces on the host, takes 67 us instead of 81, of a 24x20x28 box 30
// instead of 34.
__global__ __launch_bounds__(kBlock) void k_take_table(const double *from, double *to, int n, unsigned *left,
                                                       unsigned *seen, unsigned ticket)
{
    const int i = blockIdx.x * kBlock + threadIdx.x;
    if (i < n) to[i] = from[i];
    __syncthreads();  // the block has read its part
    if (threadIdx.x != 0) return;
    if (__hip_atomic_fetch_add(left, 1u, __ATOMIC_ACQ_REL, __HIP_MEMORY_SCOPE_AGENT) != gridDim.x - 1) return;
    __hip_atomic_store(left, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    __hip_atomic_store(seen, ticket, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_SYSTEM);
}

__global__ __launch_bounds__(kBlock) void k_mark_all(int *lost, int n)
{
    const int i = blockIdx.x * kBlock + threadIdx.x;
    if (i < n) lost[i] = 1;
}

// The solid bitmap from the owner map, or (kWalls) that map and the bitmap of a
// lattice that holds only walls: one thread per bit, two words per wavefront
// from a ballot.  The bits of a row past its second periodic copy are 0.  (In
// rounds of the grid: a lattice one node wide has 32 bits per node, and a launch
// less than 2^32 threads.)
template <bool kWalls>
__global__ __launch_bounds__(kBlock) void k_solid_bits(GeomArgs g, const uint8_t *wall)
{
    const int rw = bit_row_words(g.nx);
    const size_t words = (size_t)rw * ((size_t)g.ny * (size_t)g.nz);
    for (size_t first = (size_t)blockIdx.x * kBlock; first < 32 * words; first += (size_t)gridDim.x * kBlock) {
        const size_t i = first + threadIdx.x;
        const size_t w = i >> 5, r = w / (size_t)rw;
        const int p = (int)(w - r * (size_t)rw) * 32 + (int)(i & 31);
        bool solid = false;
        if (w < words && p <= g.nx + 1) {
            const int x = p == 0 ? g.nx - 1 : (p == g.nx + 1 ? 0 : p - 1);
            const size_t n = (size_t)x + (size_t)g.nx * r;
            if constexpr (kWalls) {
                const uint8_t v = wall[n];
                solid = v != 0;
                if (p == x + 1) g.own[n] = solid ? (uint16_t)(v - 1) : kFluid;
            } else {
                solid = g.own[n] < kVacated;
            }
        }
        const unsigned long long m = __ballot(solid);
        if ((threadIdx.x & 31) == 0 && w < words) g.bits[w] = (uint32_t)(m >> (threadIdx.x & 32));
    }
}

// Lattice coordinates of node index n (a rare path: integer divisions).
__device__ __forceinline__ Node node_of(uint32_t n, int nx, int ny)
{
    const uint32_t plane = (uint32_t)nx * (uint32_t)ny, r = n % plane;
    return Node{(int)(r % (uint32_t)nx), (int)(r / (uint32_t)nx), (int)(n / plane), n};
}

// Position of wrapped coordinate p in a box that starts at x0 (the image
// nearest its origin).
__device__ __forceinline__ int box_pos(int p, int x0, int n)
{
    const int k = p - x0;
    return k < 0 ? k + n : (k >= n ? k - n : k);
}

constexpr int kGeomList = 192;  // changed nodes of a wavefront taken together
// leaving nodes of 64 from which a lane refills a whole node: 19 rounds of one
// direction, where three nodes take one round (8 balls of radius 14 that jump:
// 1.5 ms, three at a time 3.7 ms)
constexpr int kManyLeft = 12;
constexpr int kScan = 8;        // nodes of a lane whose owners are looked at together (a marked sphere's)

// The n listed nodes of a wavefront change hands: sphere `id` enters or leaves
// them.  Returns 0, the new length of the list.
template <int S>
__device__ __forceinline__ int work_off(const GeomArgs &g, const uint32_t *list, int n, uint16_t id,
                                        const double *bodies, int lane)
{
    using St = Store<S>;
    typename St::T *pop = static_cast<typename St::T *>(g.pop);
    __builtin_amdgcn_wave_barrier();
#pragma unroll 1
    for (int k0 = 0; k0 < n; k0 += 64) {
        bool left = false;
        if (k0 + lane < n) {
            const uint32_t e = list[k0 + lane], node = e & 0x7FFFFFFFu;
            const uint16_t o = g.own[node];
            const Node v = node_of(node, g.nx, g.ny);
            if (!(e >> 31)) {
                enter_node(g, v, o, id);
            } else if (o == id && cas_u16(g.own + node, id, kFluid) == id) {
                flip_bit(g, v.px, v.py, v.pz);
                left = true;
            }
        }
        // refill: three nodes at a time, 19 lanes each, or, where many leave,
        // a lane per node
        uint64_t m = __ballot(left);
        if (__popcll(m) >= kManyLeft) {
            m = 0;
            if (left) {
                const Node v = node_of(list[k0 + lane] & 0x7FFFFFFFu, g.nx, g.ny);
                double u0, u1, u2;
                sphere_velocity(bodies + (size_t)(id - g.n_walls) * kBodyStride, v.px, v.py, v.pz, g.nx, g.ny, g.nz, u0,
                                u1, u2);
#pragma unroll 1
                for (int i = 0; i < kQ; ++i)
                    St::st(at(pop + (size_t)i * g.Ns, v.n), (float)eq_dev(i, g.rho0, u0, u1, u2));
            }
        }
#pragma unroll 1
        while (m) {
            const int i = lane % kQ, third = lane / kQ;
            int from = -1;
#pragma unroll
            for (int t = 0; t < 3; ++t) {
                if (third == t && m) from = __builtin_ctzll(m);
                m &= m - 1;
            }
            if (from >= 0) {
                const Node v = node_of(list[k0 + from] & 0x7FFFFFFFu, g.nx, g.ny);
                double u0, u1, u2;
                sphere_velocity(bodies + (size_t)(id - g.n_walls) * kBodyStride, v.px, v.py, v.pz, g.nx, g.ny, g.nz, u0,
                                u1, u2);
                St::st(at(pop + (size_t)i * g.Ns, v.n), (float)eq_dev(i, g.rho0, u0, u1, u2));
            }
        }
    }
    __builtin_amdgcn_wave_barrier();
    return 0;
}

// The value of lane `l` (compile-time or uniform) on every lane, as a scalar.
__device__ __forceinline__ int lane_of(int v, int l) { return __builtin_amdgcn_readlane(v, l); }
__device__ __forceinline__ float lane_of(float v, int l)
{
    return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), l));
}

// The part of an arc of length `len` from 0 on a circle of nz nodes that an
// arc of length `other` from d (0 <= d < nz) does not cover: two runs [a1, a1 +
// n1) and [a2, a2 + n2), exact for arcs of any lengths below nz.
__device__ __forceinline__ void arc_less(int len, int d, int other, int nz, int &a1, int &n1, int &a2, int &n2)
{
    a1 = max(d + other - nz, 0);  // the other arc's part beyond nz
    n1 = max(min(d, len) - a1, 0);
    a2 = d + other;
    n2 = max(len - a2, 0);
}

// 1 << lw wavefronts of a workgroup per sphere.  The lanes take the (x, y)
// columns of the new ball's box, then those of the old ball's that lie beside
// it; the ends of a column's new and old ranges give the nodes the sphere
// enters and leaves there, which are listed in LDS.  A marked sphere lists
// every node of its new ball that it does not own.  The list is worked off by
// the whole wavefront: one lane per node for the owner's compare-and-swap, then
// the refills.  A sphere's wavefronts take its columns in turn, 64 at a time,
// or, where it has fewer, every second or fourth node of each column.
// What bounds it: one wavefront's chain of sphere record, column ranges, owner
// and compare-and-swap, through code that the step kernel's stream has pushed
// out of the caches; hence one copy of each part, the two balls side by side
// on two lanes, and no look at nodes that stay.  128x128x512 duct, 4000
// spheres, about one changed node per sphere: 25 us a step at its start, 44 us
// 1000 steps later, when most spheres overlap.  Where a marked sphere put every
// node of its ball on the list, and asked for a neighbour's record one value
// after the other, 26 and 52 us; with one wavefront per stamp and one per
// vacate, each looking at every node of its ball, 29 and 44.
template <int S>
__global__ __launch_bounds__(kBlock) void k_geometry(GeomArgs g, int lw)
{
    __shared__ uint32_t lists[kBlock / 64][kGeomList];  // node index, bit 31: left by the sphere
    // the sphere is the same on every lane of the wavefront: made uniform, so
    // that what follows from it is scalar
    const int wv = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const int b = ((int)blockIdx.x * (kBlock / 64) + wv) >> lw, sub = wv & ((1 << lw) - 1);
    const bool any = b < max(g.nb, g.nb2);
    const int lost = any ? g.lost_prev[b] : 0;
    if (lw) __syncthreads();  // every wavefront of the sphere has read its mark
    // a marked sphere goes through its whole new ball
    const bool whole = b < g.nb && __builtin_amdgcn_readfirstlane(lost) != 0;
    if (!any) return;
    const int lane = threadIdx.x & 63;
    const int nx = g.nx, ny = g.ny, nz = g.nz;
    const uint32_t plane = (uint32_t)nx * (uint32_t)ny;
    uint32_t *list = lists[wv];
    const uint16_t id = (uint16_t)(g.n_walls + b);
    // even lanes set up the new ball, odd lanes the old one
    const bool mine = (lane & 1) == 0 ? b < g.nb2 : b < g.nb;
    const double *table[2] = {g.bodies2, g.bodies};
    const double *B = (lane & 1 ? g.bodies : g.bodies2) + (mine ? (size_t)b * kBodyStride : (size_t)0);
    const int ok = mine && body_ok(B, nx, ny, nz);
    const Box bx = body_box(B, 0);
    const BallCols bc = ball_cols(B, bx);
    const int inv = (int)(0xFFFFFFFFu / (uint32_t)max(bx.ex, 1));
    int in_ball[2];
    Box box[2];
    BallCols cols[2];
    uint32_t invs[2];
#pragma unroll
    for (int t = 0; t < 2; ++t) {
        in_ball[t] = lane_of(ok, t);
        box[t] = Box{lane_of(bx.x0, t), lane_of(bx.y0, t), lane_of(bx.z0, t),
                     lane_of(bx.ex, t), lane_of(bx.ey, t), lane_of(bx.ez, t)};
        cols[t] = BallCols{lane_of(bc.ox, t), lane_of(bc.oy, t), lane_of(bc.oz, t),
                           lane_of(bc.r2, t), lane_of(bc.eps2, t), lane_of(bc.m, t)};
        invs[t] = (uint32_t)lane_of(inv, t);
    }
    if (lane == 0 && sub == 0) {
        g.lost_prev[b] = 0;  // the array takes the marks of the update after this one
        if (mine) static_cast<LinkRec *>(g.lrec)[g.n_walls + b].k = sphere_k(B);
    }
    const int n_new = in_ball[0] ? box[0].ex * box[0].ey : 0;
    const int n_cols = n_new + (in_ball[1] ? box[1].ex * box[1].ey : 0);
    // the sphere's wavefronts: 1 << lk share each 64 columns
    const int lk = max(lw - (n_cols > 192 ? 2 : (n_cols > 64 ? 1 : 0)), 0);
    const int step = 1 << lk, stride = 64 << (lw - lk);
    int n = 0;  // listed nodes
    for (int c0 = 64 * (sub >> lk); c0 < n_cols; c0 += stride) {
        // ---- 64 columns: the changed nodes of each
        int e1 = 0, e2 = 0, l1 = 0, l2 = 0;      // nodes entered and left: two runs of each
        int ze1 = 0, ze2 = 0, zl1 = 0, zl2 = 0;  // their first z (from that of the range)
        int start[2] = {0, 0}, len[2] = {0, 0};  // the column's ranges: wrapped start, length
        uint32_t col = 0;
        const int c = c0 + lane;
        if (c < n_cols) {
            const int t0 = c >= n_new, cc = t0 ? c - n_new : c;
            const int ex = t0 ? box[1].ex : box[0].ex;
            int ky = (int)__umulhi((uint32_t)cc, t0 ? invs[1] : invs[0]), kx = cc - ky * ex;
            if (kx >= ex) {
                ++ky;
                kx -= ex;
            }
            const int px = wrap1((t0 ? box[1].x0 : box[0].x0) + kx, nx), py = wrap1((t0 ? box[1].y0 : box[0].y0) + ky, ny);
            col = (uint32_t)px + (uint32_t)nx * (uint32_t)py;
            const bool in_new = in_ball[0] && box_pos(px, box[0].x0, nx) < box[0].ex && box_pos(py, box[0].y0, ny) < box[0].ey;
            if (!(t0 && in_new)) {  // (an old column inside the new box was taken with the new ones)
#pragma unroll 1
                for (int t = t0; t < 2; ++t) {
                    const Box &bt = t ? box[1] : box[0];
                    const int qx = box_pos(px, bt.x0, nx), qy = box_pos(py, bt.y0, ny);
                    if ((t ? in_ball[1] : in_ball[0]) && qx < bt.ex && qy < bt.ey) {
                        int lo, hi;
                        column_range(table[t] + (size_t)b * kBodyStride, bt, t ? cols[1] : cols[0], qx, qy, px, py, nx, ny,
                                     nz, lo, hi);
                        const int at0 = wrap1(lo, nz), m = max(hi - lo + 1, 0);
                        if (t) {
                            start[1] = at0;
                            len[1] = m;
                        } else {
                            start[0] = at0;
                            len[0] = m;
                        }
                    }
                }
            }
            const int d = start[1] - start[0];
            arc_less(len[0], d < 0 ? d + nz : d, len[1], nz, ze1, e1, ze2, e2);
            arc_less(len[1], d > 0 ? nz - d : -d, len[0], nz, zl1, l1, zl2, l2);
            if (whole) e1 = e2 = 0;  // (looked at with the rest of the ball)
        }
        // ---- listed, one node of each column at a time: the changed nodes,
        //      then those of a marked sphere's ball that are not its own
        const int cnt = e1 + e2 + l1 + l2, scan = whole ? len[0] : 0;
        uint32_t todo = 0;
        int k = sub & (step - 1), ks = k - kScan * step;
        while (true) {
            // ---- the listed nodes change hands when the list is full or
            //      there are no more
            const bool runs = __ballot(k < cnt) != 0;
            const bool more = runs || __ballot(todo != 0 || ks + kScan * step < scan) != 0;
            if (n > kGeomList - 64 || (!more && n && c0 + stride >= n_cols)) n = work_off<S>(g, list, n, id, g.bodies, lane);
            if (!more) break;
            bool changed, leaves = false;
            int z;
            if (runs) {
                leaves = k >= e1 + e2;
                z = k < e1 ? ze1 + k
                           : (!leaves ? ze2 + (k - e1) : (k < e1 + e2 + l1 ? zl1 + (k - e1 - e2) : zl2 + (k - e1 - e2 - l1)));
                changed = k < cnt;
                k += step;
            } else {
                if (!__ballot(todo != 0)) {
                    ks += kScan * step;
                    uint16_t o[kScan];
#pragma unroll
                    for (int u = 0; u < kScan; ++u) {
                        const int q = ks + u * step;
                        o[u] = id;
                        if (q < scan) o[u] = *at(g.own, col + plane * (uint32_t)wrap1(start[0] + q, nz));
                    }
#pragma unroll
                    for (int u = 0; u < kScan; ++u) todo |= (o[u] != id && o[u] >= g.n_walls) ? 1u << u : 0u;
                }
                changed = todo != 0;
                z = ks + (changed ? __builtin_ctz(todo) : 0) * step;
                todo &= todo - 1u;
            }
            const uint32_t node = col + plane * (uint32_t)wrap1((leaves ? start[1] : start[0]) + z, nz);
            const uint64_t m = __ballot(changed);
            if (changed)
                list[n + (int)__builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0u))] =
                    node | (leaves ? 0x80000000u : 0u);
            n += __popcll(m);
        }
    }
}

template <int S>
__global__ __launch_bounds__(kBlock) void k_init_pop(GeomArgs g, const double *rho, const double *u)
{
    using St = Store<S>;
    typename St::T *pop = static_cast<typename St::T *>(g.pop);
    const int n = blockIdx.x * kBlock + threadIdx.x;
    if (n >= g.N) return;
    const size_t N = (size_t)g.N;
    if (g.own[n] < kVacated) {
        for (int i = 0; i < kQ; ++i) St::st(pop + i * (size_t)g.Ns + n, 0.0f);
        return;
    }
    const double r = rho ? rho[n] : (double)g.rho0;
    const double u0 = u ? u[n] : 0.0, u1 = u ? u[N + n] : 0.0, u2 = u ? u[2 * N + n] : 0.0;
    const double uu = u0 * u0 + u1 * u1 + u2 * u2;
    for (int i = 0; i < kQ; ++i) {
        const double cu = dcx(i) * u0 + dcy(i) * u1 + dcz(i) * u2;
        const double dev = wgt(i) * (r - (double)g.rho0) + wgt(i) * r * (3.0 * cu + 4.5 * cu * cu - 1.5 * uu);
        St::st(pop + i * (size_t)g.Ns + n, (float)dev);
    }
}

__device__ __forceinline__ void solid_velocity(const GeomArgs &g, const double *walls, uint16_t o, int px, int py,
                                               int pz, double &u0, double &u1, double &u2)
{
    if (o < g.n_walls) {
        u0 = walls[o * kWallStride];
        u1 = walls[o * kWallStride + 1];
        u2 = walls[o * kWallStride + 2];
    } else {
        sphere_velocity(g.bodies + (o - g.n_walls) * kBodyStride, px, py, pz, g.nx, g.ny, g.nz, u0, u1, u2);
    }
}

template <int S>
__global__ __launch_bounds__(kBlock) void k_export_pop(GeomArgs g, const double *walls, int dir, double *out)
{
    using St = Store<S>;
    const typename St::T *pop = static_cast<const typename St::T *>(g.pop);
    const int n = blockIdx.x * kBlock + threadIdx.x;
    if (n >= g.N) return;
    const uint16_t o = g.own[n];
    if (o >= kVacated) {
        out[n] = (double)St::ld(pop + (size_t)dir * g.Ns + n) + wgt(dir) * (double)g.rho0;
        return;
    }
    const int px = n % g.nx, py = (n / g.nx) % g.ny, pz = n / (g.nx * g.ny);
    double u0, u1, u2;
    solid_velocity(g, walls, o, px, py, pz, u0, u1, u2);
    out[n] = wgt(dir) * (double)g.rho0 + eq_dev(dir, g.rho0, u0, u1, u2);
}

template <int S>
__global__ __launch_bounds__(kBlock) void k_import_pop(int N, int Ns, int dir, float rho0, const double *in, void *popv)
{
    using St = Store<S>;
    typename St::T *pop = static_cast<typename St::T *>(popv);
    const int n = blockIdx.x * kBlock + threadIdx.x;
    if (n < N) St::st(pop + (size_t)dir * Ns + n, (float)(in[n] - wgt(dir) * (double)rho0));
}

template <int S>
__global__ __launch_bounds__(kBlock) void k_export_macro(GeomArgs g, const double *walls, double fx, double fy,
                                                         double fz, double *rho, double *u)
{
    using St = Store<S>;
    const typename St::T *pop = static_cast<const typename St::T *>(g.pop);
    const int n = blockIdx.x * kBlock + threadIdx.x;
    if (n >= g.N) return;
    const size_t N = (size_t)g.N;
    const uint16_t o = g.own[n];
    if (o >= kVacated) {
        double r = 0.0, j0 = 0.0, j1 = 0.0, j2 = 0.0;
        for (int i = 0; i < kQ; ++i) {
            const double f = (double)St::ld(pop + i * (size_t)g.Ns + n) + wgt(i) * (double)g.rho0;
            r += f;
            j0 += dcx(i) * f;
            j1 += dcy(i) * f;
            j2 += dcz(i) * f;
        }
        rho[n] = r;
        u[n] = (j0 - 0.5 * fx) / r;
        u[N + n] = (j1 - 0.5 * fy) / r;
        u[2 * N + n] = (j2 - 0.5 * fz) / r;
        return;
    }
    const int px = n % g.nx, py = (n / g.nx) % g.ny, pz = n / (g.nx * g.ny);
    double u0, u1, u2;
    solid_velocity(g, walls, o, px, py, pz, u0, u1, u2);
    rho[n] = g.rho0;
    u[n] = u0;
    u[N + n] = u1;
    u[2 * N + n] = u2;
}

__global__ __launch_bounds__(kBlock) void k_export_owner(const uint16_t *own, int N, int32_t *out)
{
    const int n = blockIdx.x * kBlock + threadIdx.x;
    if (n < N) out[n] = own[n] >= kVacated ? -1 : (int32_t)own[n];
}

__global__ __launch_bounds__(kBlock) void k_zero(double *p, int n)
{
    const int i = blockIdx.x * kBlock + threadIdx.x;
    if (i < n) p[i] = 0.0;
}

__global__ __launch_bounds__(kBlock) void k_count_fluid(const uint16_t *own, int N, unsigned long long *count)
{
    __shared__ unsigned int s_cnt;
    if (threadIdx.x == 0) s_cnt = 0;
    __syncthreads();
    unsigned int c = 0;
    for (int n = blockIdx.x * kBlock + threadIdx.x; n < N; n += gridDim.x * kBlock) c += own[n] >= kVacated;
    atomicAdd(&s_cnt, c);
    __syncthreads();
    if (threadIdx.x == 0 && s_cnt) atomicAdd(count, (unsigned long long)s_cnt);
}

inline int nblk(long n) { return (int)((n + kBlock - 1) / kBlock); }

// Wavefronts of k_geometry per sphere, as a power of two: as many as the chip
// holds at once (its registers leave four to each of 1024 SIMDs), up to four.
// Few spheres leave most of it idle while a large, jumping or overlapped one
// makes a long chain; with many, each wavefront's set-up is what costs.  us per
// update with 1 / 2 / 4 wavefronts: one sphere of radius 30 in 96^3 239 / 132 / 72, 60
// of radius 8 to 14, most overlapping, 342 / 181 / 106; radius 4, 300 spheres
// 18.6 / 17.0 / 16.2, jumping 61 / 39 / 37, 1000 spheres 22.0 / 21.6 / 21.0; radius 3,
// 2000 spheres 21.6 / 22.0 / 26.5; the duct's 4000, in whole steps, 275.7 / 278.3 /
// 279.6; radius 2, 8000 spheres 29 / 40 / 59.
constexpr int kGeomWaves = 4096;
inline int geometry_split(int spheres) { return spheres <= kGeomWaves / 4 ? 2 : (spheres <= kGeomWaves / 2 ? 1 : 0); }

template <template <int> class K, typename... A>
hipError_t dispatch(int storage, dim3 grid, dim3 block, hipStream_t s, A... args)
{
    switch (storage) {
    case 0: hipLaunchKernelGGL(K<0>::fn, grid, block, 0, s, args...); break;
    case 1: hipLaunchKernelGGL(K<1>::fn, grid, block, 0, s, args...); break;
    case 2: hipLaunchKernelGGL(K<2>::fn, grid, block, 0, s, args...); break;
    default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

template <int S> struct GeomK { static constexpr auto fn = k_geometry<S>; };
template <int S> struct InitK { static constexpr auto fn = k_init_pop<S>; };
template <int S> struct ExportK { static constexpr auto fn = k_export_pop<S>; };
template <int S> struct ImportK { static constexpr auto fn = k_import_pop<S>; };
template <int S> struct MacroK { static constexpr auto fn = k_export_macro<S>; };

}  // namespace

hipError_t launch_link_records(const GeomArgs &g, const double *wrec, hipStream_t s)
{
    const int n = g.n_walls + g.nb;
    if (n <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_link_records, dim3(nblk(n)), dim3(kBlock), 0, s, g, wrec);
    return hipGetLastError();
}

hipError_t launch_take_table(const double *from, double *to, int n, unsigned *left, unsigned *seen, unsigned ticket,
                             hipStream_t s)
{
    if (n <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_take_table, dim3(nblk(n)), dim3(kBlock), 0, s, from, to, n, left, seen, ticket);
    return hipGetLastError();
}

hipError_t launch_mark_all(int *lost, int n, hipStream_t s)
{
    if (n <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_mark_all, dim3(nblk(n)), dim3(kBlock), 0, s, lost, n);
    return hipGetLastError();
}

static dim3 bits_grid(const GeomArgs &g)
{
    const size_t bits = 32 * (size_t)bit_row_words(g.nx) * ((size_t)g.ny * (size_t)g.nz);
    return dim3((unsigned)std::min((bits + kBlock - 1) / kBlock, (size_t)1 << 22));
}

hipError_t launch_walls_init(const GeomArgs &g, const uint8_t *wall, hipStream_t s)
{
    hipLaunchKernelGGL(k_solid_bits<true>, bits_grid(g), dim3(kBlock), 0, s, g, wall);
    return hipGetLastError();
}

hipError_t launch_solid_bits(const GeomArgs &g, hipStream_t s)
{
    hipLaunchKernelGGL(k_solid_bits<false>, bits_grid(g), dim3(kBlock), 0, s, g, (const uint8_t *)nullptr);
    return hipGetLastError();
}

hipError_t launch_geometry(int storage, const GeomArgs &g, hipStream_t s)
{
    const int spheres = std::max(g.nb, g.nb2);
    if (spheres <= 0) return hipSuccess;
    const int lw = geometry_split(spheres), per_block = (kBlock / 64) >> lw;
    return dispatch<GeomK>(storage, dim3((spheres + per_block - 1) / per_block), dim3(kBlock), s, g, lw);
}

hipError_t launch_init_pop(int storage, const GeomArgs &g, const double *rho, const double *u, hipStream_t s)
{
    return dispatch<InitK>(storage, dim3(nblk(g.N)), dim3(kBlock), s, g, rho, u);
}

hipError_t launch_export_pop(int storage, const GeomArgs &g, const double *walls, int dir, double *out,
                             hipStream_t s)
{
    return dispatch<ExportK>(storage, dim3(nblk(g.N)), dim3(kBlock), s, g, walls, dir, out);
}

hipError_t launch_import_pop(int storage, int N, int Ns, int dir, float rho0, const double *in, void *pop,
                             hipStream_t s)
{
    return dispatch<ImportK>(storage, dim3(nblk(N)), dim3(kBlock), s, N, Ns, dir, rho0, in, pop);
}

hipError_t launch_export_macro(int storage, const GeomArgs &g, const double *walls, double fx, double fy,
                               double fz, double *rho, double *u, hipStream_t s)
{
    return dispatch<MacroK>(storage, dim3(nblk(g.N)), dim3(kBlock), s, g, walls, fx, fy, fz, rho, u);
}

hipError_t launch_export_owner(const uint16_t *own, int N, int32_t *out, hipStream_t s)
{
    hipLaunchKernelGGL(k_export_owner, dim3(nblk(N)), dim3(kBlock), 0, s, own, N, out);
    return hipGetLastError();
}

hipError_t launch_zero(double *p, int n, hipStream_t s)
{
    if (n <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_zero, dim3(nblk(n)), dim3(kBlock), 0, s, p, n);
    return hipGetLastError();
}

hipError_t launch_count_fluid(const uint16_t *own, int N, unsigned long long *count, hipStream_t s)
{
    hipLaunchKernelGGL(k_count_fluid, dim3(std::min(nblk(N), 2048)), dim3(kBlock), 0, s, own, N, count);
    return hipGetLastError();
}

}  // namespace lbm

// The fused D3Q19 step on gfx950: boundary links, pull streaming, collision
// and store of a 256-node tile in one pass over HBM.
//
// Per tile (one workgroup, one node per thread):
//  1. Each wavefront reads which of its nodes and of their pull sources are
//     solid from the solid bitmap, as lane masks in scalar registers, and
//     issues the pulls of fluid nodes from fluid sources (the streaming
//     equation of Sec. 2.2) straight into the tile's LDS array of
//     populations.
//  2. A direction whose pull source is a solid node is a cut link (Sec. 2.3);
//     the links of the tile are listed in LDS and spread over the
//     workgroup's threads.  Per link: the value of the
//     population the node receives (the q < 1/2 and q >= 1/2 branches with
//     the moving-boundary term of eq. moving_boundary_velocity, walls at
//     q = 1/2), formed from the current state at the node and at the node
//     behind it, which the tile's pulls have brought into the caches; and
//     the momentum exchanged on the link (Sec. 2.3, force and torque), added
//     as 64-bit fixed point to the tile's LDS table of bodies.
//     The link's value goes into the LDS slot its pull would have filled.
//  3. Each node takes its 19 values from LDS; moments, the Smagorinsky
//     relaxation time, BGK + Guo collision and the store follow as in the
//     pull-collide kernel.
//  4. The tile's body sums go to the global fixed-point sums with one atomic
//     add per body and component; a small kernel turns them into the FP64
//     forces of the step.  Integer sums do not depend on the order of the
//     additions, so the forces are the same bit for bit for every launch,
//     tile shape and batch.
// What bounds it: with FP32 storage HBM and issue about equally, with 16-bit
// storage instruction issue.  A wavefront issues vector and scalar
// instructions on separate ports at the same rate (one per SIMD in four
// cycles), so both counts matter.  On the 128x128x512 duct with 4000 spheres,
// tile 64x2x2, per wavefront: 658 vector and 588 scalar instructions
// (FP16), 206 us per launch; with owner codes loaded per pull source and a scan over
// the workgroup (897 vector, 410 scalar, 18 loads more) it took 244 us, FP32
// 255 against 287 us.  Masks kept per direction for the pulls as well (1305
// scalar instructions) took 316 us: the pulls therefore go to every fluid
// lane, and the few values pulled from solid sources are replaced later.
//
// The link arithmetic is that of the boundary-link pass (lbm_linkmath.h), so
// the populations equal, bit for bit, those of the link pass followed by the
// pull-collide kernel.
#include "lbm_collide.h"
#include "lbm_device.h"
#include "lbm_internal.h"
#include "lbm_linkmath.h"

#include <hip/hip_ext.h>
#include <hip/hip_runtime.h>
#include <math.h>

#include <map>
#include <mutex>

namespace lbm {
namespace {

using namespace dev;

// LDS per workgroup is held to 23040 bytes, so that seven workgroups fit in
// a CU's 160 KB: 984 list items of 16 bits and two copies of a 16-body force
// table
// (with 8 bodies, tiles 64 nodes long often found the table full and sent
// their sums to global memory)
//
// A tile with more links than the list holds forms them in rounds, each with
// the masks read again and two more barriers.  With 492 items of 32 bits that
// were 3-4.5% of the duct's tiles: 7.15 against 6.96 ms per 30 FP16 steps, 8.32
// against 8.25 ms in FP32; on a lattice whose tiles all run at once the
// heaviest tile sets the time, 96x40x40 with 200 spheres 288 against 256 us per
// 20 steps.
constexpr int kLinkCap = 984;   // links of a tile listed at once (rounds beyond)
constexpr int kRec = 16;        // bodies of a tile with a slot in the LDS force table
constexpr int kCopies = 2;      // copies of the table's sums (by lane), so fewer lanes add to one address

struct FusedLds {
    uint16_t item[kLinkCap];          // link: node << 6 | I << 1 | (node behind solid)
    uint32_t val[kQ][kBlock];         // population i streamed to node n: val[i][n], as the stored value's
                                      // bits (16-bit storage: zero-extended)
    int key[kRec];                    // owner code of the body in a force slot, -1 free
    unsigned long long sum[kCopies][kRec][6];  // fixed-point F, T of that body
    int wtot[kBlock / 64];
};
static_assert(sizeof(FusedLds) <= 23040, "seven workgroups per CU");

// The step's arguments where they lie in memory (the kernel's argument
// segment, or a batch member's record), read by scalar loads: nothing writes
// them while a kernel runs.
typedef const __attribute__((address_space(4))) FusedArgs *ArgPtr;

// The same pointer, unknown to the compiler: what is read through it is
// loaded again.  A tile works in phases that need different arguments, and
// all of them together with the lane masks do not fit in scalar registers.
__device__ __forceinline__ ArgPtr reread(ArgPtr p)
{
    asm volatile("" : "+s"(p));
    return p;
}

// v 2^32 rounded to the nearest integer, ties to even, as a two's-complement
// 64-bit value.  While |v 2^32| < 2^51 one FP64 add of 1.5 2^52 leaves that
// integer in the low mantissa bits (to_fix_fast, for |v| < kFixFastLimit);
// larger values take the library conversion, which rounds the same way.
constexpr double kFixFastLimit = 524288.0;  // 2^19

__device__ __forceinline__ unsigned long long to_fix_fast(double v)
{
    constexpr double kMagic = 6755399441055744.0;  // 1.5 * 2^52
    const double t = __builtin_fma(v, kFixScale, kMagic);
    return (unsigned long long)(__double_as_longlong(t) - __double_as_longlong(kMagic));
}

__device__ __forceinline__ unsigned long long to_fix_slow(double v)
{
    return (unsigned long long)__double2ll_rn(v * kFixScale);
}

// Global fixed-point sums of owner code `key` (tile t picks the wall copy).
__device__ __forceinline__ unsigned long long *fix_slot(ArgPtr f, int key, int t)
{
    const int e = key < f->n_walls ? f->wall_base + key * kWallRep + (t & (kWallRep - 1)) : key - f->n_walls;
    return f->fsum + 6 * (size_t)e;
}

// Add one link's fixed-point force and torque to the tile's slot of body
// `key` (the lane's copy of the sums), or straight to the global sums when
// the table is full.  A slot is claimed once by compare-and-swap; later
// lookups read it.
__device__ __forceinline__ void table_add(ArgPtr f, FusedLds &lds, int key, const unsigned long long (&v)[6],
                                          int t)
{
    int s = key & (kRec - 1);
#pragma unroll 1
    for (int p = 0; p < kRec; ++p) {
        int cur = __hip_atomic_load(&lds.key[s], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
        if (cur == -1) cur = atomicCAS(&lds.key[s], -1, key);
        if (cur == -1 || cur == key) {
            unsigned long long *d = lds.sum[threadIdx.x & (kCopies - 1)][s];
#pragma unroll
            for (int c = 0; c < 6; ++c) atomicAdd(d + c, v[c]);  // zeros too: no test per component
            return;
        }
        s = (s + 1) & (kRec - 1);
    }
    unsigned long long *g = fix_slot(f, key, t);
#pragma unroll
    for (int c = 0; c < 6; ++c)
        if (v[c]) atomicAdd(g + c, v[c]);
}

// Wait until this wavefront's vector memory loads are complete, loads into
// LDS included (s_waitcnt vmcnt(0); the compiler does not track those).
__device__ __forceinline__ void wait_vmem() { __builtin_amdgcn_s_waitcnt(0x0F70); }

// Workgroup barrier for LDS only: this wavefront's LDS operations complete,
// then s_barrier; loads from global memory, those into LDS included, stay in
// flight (a full barrier, or a fence on LDS, waits for them all).  The asm
// clobbers memory, so the compiler moves no memory access across it.
__device__ __forceinline__ void lds_barrier() { asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory"); }

// Quotient and remainder of t / d for a uniform t >= 0, with inv =
// quick_inv(d).
__device__ __forceinline__ int quick_div(int t, int d, uint32_t inv, int &rem)
{
    int q = (int)__umulhi((uint32_t)t, inv);
    rem = t - q * d;
    if (rem >= d) {
        ++q;
        rem -= d;
    }
    return q;
}

typedef uint32_t uint32x2 __attribute__((ext_vector_type(2)));

// A wavefront's share of a tile, 64 / TX rows of TX nodes at z from row y on,
// as 64-bit lane masks in scalar registers: the lanes inside the lattice,
// those of fluid nodes, and per direction the fluid lanes whose pull source
// x - c_i is solid (a cut link).  Everything here is scalar: the windows of
// the solid bitmap are scalar loads, a direction's mask is a shift of one of
// them, and using a mask as the lanes of a load or store costs no vector
// instruction.  Scalar instructions count as vector ones do (see above): on
// lattices whose tiles all run at once the chain through them is what a step
// waits for.  With the masks set to zero where there are no links and 32-node
// rows combined by 64-bit shifts, 60 more per wavefront, 96x40x40 with 204
// spheres took 255 against 245 us per 20 steps (FP16 259 / 250), 160x128x128 FP16
// 3.14 against 3.01 ms per 50.
template <int TX>
struct WaveMasks {
    uint64_t in, fluid, cut[kQ];
};

// The rows of a wavefront (z, y .. y + R - 1) and their periodic neighbours, as
// scalars: y - 1 .. y + R and z - 1 .. z + 1.  A wavefront outside the lattice
// takes rows inside it.
template <int R>
struct WaveRows {
    int y[R + 2], z[3];
    __device__ __forceinline__ WaveRows(int wy, int wz, int ny, int nz)
    {
        y[1] = min(wy, ny - 1);
        y[0] = y[1] == 0 ? ny - 1 : y[1] - 1;
#pragma unroll
        for (int k = 2; k < R + 2; ++k) y[k] = y[k - 1] + 1 >= ny ? 0 : y[k - 1] + 1;
        z[1] = min(wz, nz - 1);
        z[0] = z[1] == 0 ? nz - 1 : z[1] - 1;
        z[2] = z[1] + 1 >= nz ? 0 : z[1] + 1;
    }
};

// Returns whether the wavefront has links; without any, cut is left unset.
template <int TX>
__device__ __forceinline__ bool wave_masks(ArgPtr f, int x0, int y, int z, const WaveRows<64 / TX> &w,
                                           WaveMasks<TX> &m)
{
    constexpr int R = 64 / TX;
    constexpr uint64_t kOnes = TX == 64 ? ~0ull : (1ull << (TX & 63)) - 1;
    typedef const __attribute__((address_space(4))) char *ScalarPtr;  // scalar loads: nothing writes it meanwhile
    typedef const __attribute__((address_space(4))) uint32_t *ScalarWords;
    const int nx = f->s.nx, ny = f->s.ny, nz = f->s.nz;
    m.in = 0;
    const uint64_t row_in = x0 + TX <= nx ? kOnes : (1ull << (nx - x0)) - 1;
#pragma unroll
    for (int r = 0; r < R; ++r)
        if (z < nz && y + r < ny) m.in |= row_in << (r * TX & 63);
    m.fluid = 0;
    if (!m.in) return false;
    const uint32_t rw = 4u * (uint32_t)bit_row_words(nx);
    const ScalarPtr bits = (ScalarPtr)(uintptr_t)f->bits;
    uint32_t yw[R + 2];  // byte offsets of the rows' windows within a plane
#pragma unroll
    for (int k = 0; k < R + 2; ++k) yw[k] = rw * (uint32_t)w.y[k] + (uint32_t)(x0 >> 5) * 4u;
    // solid bits of TX nodes of the rows y - 1 .. y + R and z - 1 .. z + 1:
    // of the nodes x - 1 (s = 0), x (1) and x + 1 (2)
    uint64_t lo[3][R + 2];
    uint32_t hi[3][R + 2];
#pragma unroll
    for (int dz = 0; dz < 3; ++dz) {
        const uint32_t zw = rw * (uint32_t)ny * (uint32_t)w.z[dz];
#pragma unroll
        for (int k = 0; k < R + 2; ++k) {
            const ScalarWords p = (ScalarWords)(bits + (uint64_t)(yw[k] + zw));
            lo[dz][k] = (uint64_t)p[0] | (uint64_t)p[1] << 32;
            hi[dz][k] = TX == 64 ? p[2] : 0u;
        }
    }
    const int half = TX == 16 ? (x0 & 16) : 0;
    auto window = [&](int dz, int k, int s) -> uint64_t {
        if (TX == 64) return s == 0 ? lo[dz][k] : lo[dz][k] >> s | (uint64_t)hi[dz][k] << ((64 - s) & 63);
        return (lo[dz][k] >> (half + s)) & kOnes;
    };
    auto rows = [&](int cx, int cy, int cz) {  // solid bits of the sources x - c of the wavefront's nodes
        if constexpr (TX == 32) {  // two registers side by side, nothing to shift and combine
            const uint32_t a = (uint32_t)(lo[1 - cz][1 - cy] >> (1 - cx)), b = (uint32_t)(lo[1 - cz][2 - cy] >> (1 - cx));
            return __builtin_bit_cast(uint64_t, uint32x2{a, b});
        }
        uint64_t v = 0;
#pragma unroll
        for (int r = 0; r < R; ++r) v |= window(1 - cz, r + 1 - cy, 1 - cx) << (r * TX & 63);
        return v;
    };
    m.fluid = m.in & ~rows(0, 0, 0);
    // nothing solid near the wavefront: no link
    uint64_t any = 0;
    uint32_t any_hi = 0;
#pragma unroll
    for (int dz = 0; dz < 3; ++dz)
#pragma unroll
        for (int k = 0; k < R + 2; ++k) {
            any |= lo[dz][k];
            any_hi |= hi[dz][k];
        }
    if (!(any | any_hi)) return false;
#pragma unroll
    for (int i = 1; i < kQ; ++i) m.cut[i] = m.fluid & rows(CX[i], CY[i], CZ[i]);
    return true;
}

// Item `it` of the tile's list: returns the link's value as the stored bits,
// its momentum goes into the force table.  Walls are records like spheres:
// reference point, velocity, no spin, q = 1/2 and no minimum image (their arm
// is about the reference point).
template <int S, int TX, int TY, int TZ>
__device__ __forceinline__ uint32_t fused_link(ArgPtr f, const typename Store<S>::T *__restrict__ src, FusedLds &lds,
                                               int x0, int y0, int z0, uint32_t it, int t)
{
    using St = Store<S>;
    using T = typename St::T;
    const size_t Ns = (size_t)f->s.Ns;
    const int nx = f->s.nx, ny = f->s.ny, nz = f->s.nz;
    const int nl = (int)(it >> 6), I = (int)((it >> 1) & 31u), K = I <= 9 ? I + 9 : I - 9;
    const bool behind = !(it & 1u);  // the node behind is fluid
    const int lx = nl % TX, ly = (nl / TX) % TY, lz = nl / (TX * TY);
    const int x = x0 + lx, y = y0 + ly, z = z0 + lz;
    const Comp cx = comp_x(I), cy = comp_y(I), cz = comp_z(I);
    const int nxy = nx * ny;
    // the node's index, without multiplications per lane
    uint32_t xi = (uint32_t)(x0 + nx * y0 + nxy * z0 + lx);
#pragma unroll
    for (int b = 1; b < TY; b <<= 1) xi += ly & b ? (uint32_t)(b * nx) : 0u;
#pragma unroll
    for (int b = 1; b < TZ; b <<= 1) xi += lz & b ? (uint32_t)(b * nxy) : 0u;
    // the solid node p = x - c_I and the node behind x, x + c_I: one step of
    // the index, or, in a wavefront with a node on the box's faces, with the
    // periodic wrap
    const uint32_t step = (uint32_t)(cx.value() + cy.times(nx) + cz.times(nxy));
    uint32_t pi = xi - step, bi = xi + step;
    if (__ballot((unsigned)(x - 1) >= (unsigned)(nx - 2) || (unsigned)(y - 1) >= (unsigned)(ny - 2) ||
                 (unsigned)(z - 1) >= (unsigned)(nz - 2))) {
        const int ax = cx.value(), ay = cy.value(), az = cz.value();
        pi = (uint32_t)(wrap_add(x, -ax, nx) + nx * (wrap_add(y, -ay, ny) + ny * wrap_add(z, -az, nz)));
        bi = (uint32_t)(wrap_add(x, ax, nx) + nx * (wrap_add(y, ay, ny) + ny * wrap_add(z, az, nz)));
    }
    // population d of node n, as stored
    auto stored = [&](int d, uint32_t n) { return src[(uint64_t)(uint32_t)d * (uint32_t)Ns + n]; };
    const int os = *at(f->s.own, pi);
    const bool sphere = os >= f->n_walls;
    const bool exact_q = sphere && !f->halfway;
    // the solid's record and the populations, in one round trip: the record
    // first, and the populations as stored values, converted only once all
    // are in flight (a conversion inside a branch would wait for its load,
    // and for everything issued before it)
    const SphereK sk = at(static_cast<const LinkRec *>(f->lrec), (uint32_t)os)->k;
    const T rk = stored(K, xi);
    T ra = T(0), rb = T(0);
    if (exact_q) {
        ra = stored(I, xi);
        if (behind) rb = stored(K, bi);
    }
    const float fk = St::cvt(rk), fa = St::cvt(ra), fb = St::cvt(rb);
    const LinkGeo g = link_geo(sk, exact_q, sphere, f->s.rho0, x, y, z, nx, ny, nz, I);
    const float vr = St::round(link_value(g.q, fk, fa, fb, behind, g.mw));
    double acc[6];
    const double mom = link_momentum(fk, vr, I, f->s.rho0);
    link_force_terms(mom, I, g, acc);
    unsigned long long v[6];
    // F = -mom c_I: its fixed-point components are -c M with M = fix(mom)
    // (the rounding is odd-symmetric).  One range test for the four
    // conversions (to_fix's two ways, taken together).
    unsigned long long M;
    const double big =
        fmax(fmax(__builtin_fabs(mom), __builtin_fabs(acc[3])), fmax(__builtin_fabs(acc[4]), __builtin_fabs(acc[5])));
    if (big < kFixFastLimit) {
        M = to_fix_fast(mom);
#pragma unroll
        for (int c = 3; c < 6; ++c) v[c] = to_fix_fast(acc[c]);
    } else {
        M = to_fix_slow(mom);
#pragma unroll
        for (int c = 3; c < 6; ++c) v[c] = to_fix_slow(acc[c]);
    }
    // -c M from the component's masks: M ^ s - s is -M where s is all ones
    auto signed_part = [&](const Comp &c) {
        const unsigned long long s = (unsigned long long)(long long)c.pos;
        return ((M ^ s) - s) & (unsigned long long)(long long)(c.pos | c.neg);
    };
    v[0] = signed_part(cx);
    v[1] = signed_part(cy);
    v[2] = signed_part(cz);
    table_add(f, lds, os, v, t);
    return St::to_bits(vr);
}

// Issue the pulls of directions I .. 18 of the active lanes into the row
// of lds.val that starts at node `first` (the wavefront's): xb, yb, zb are the
// byte offsets of the source by the component of -c_i (-1, 0, 1).
template <int S, int I>
__device__ __forceinline__ void pull_from(const char *src, size_t Ns, const uint32_t (&xb)[3], const uint32_t (&yb)[3],
                                          const uint32_t (&zb)[3], FusedLds &lds, int first)
{
    if constexpr (I < kQ) {
        using T = typename Store<S>::T;
        constexpr int kBytes = S == 0 ? 4 : 2;
        const uint32_t off = xb[1 - CX[I]] + (yb[1 - CY[I]] + zb[1 - CZ[I]]);
        const T *p = reinterpret_cast<const T *>(src + (size_t)I * Ns * sizeof(T) + off);
        __builtin_amdgcn_global_load_lds(p, (__attribute__((address_space(3))) void *)&lds.val[I][first], kBytes, 0, 0);
        pull_from<S, I + 1>(src, Ns, xb, yb, zb, lds, first);
    }
}

// Tile t of the lattice of f.  Every thread of the workgroup calls it (it
// holds barriers); lds may be reused by the next call.
template <int S, int TX, int TY, int TZ>
__device__ __forceinline__ void fused_tile(ArgPtr f, const void *srcv, void *dstv, int t, FusedLds &lds)
{
    static_assert(TX * TY * TZ == kBlock, "tile must hold one workgroup");
    using St = Store<S>;
    using T = typename St::T;
    const T *__restrict__ src = static_cast<const T *>(srcv);
    const size_t Ns = (size_t)f->s.Ns;
    const int nx = f->s.nx, ny = f->s.ny, nz = f->s.nz;

    constexpr int R = 64 / TX;  // rows of a wavefront
    // (opaque: a kernel that loops over tiles would keep what follows from the
    // thread index in registers from tile to tile)
    int tid = threadIdx.x;
    asm volatile("" : "+v"(tid));
    const int lane = tid & 63;
    const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);
    int tx, ty;
    const int r = quick_div(t, f->s.ntx, f->inv_ntx, tx);
    const int x0 = tx * TX, z0 = quick_div(r, f->s.nty, f->inv_nty, ty) * TZ, y0 = ty * TY;
    // the wavefront's rows: at z from wy on; the lane's node (x, y, z)
    const int wy = y0 + wv * R % TY, z = z0 + wv * R / TY;
    const int lx = lane % TX, x = x0 + lx, y = wy + lane / TX;

    // 1. which lanes are fluid, and which directions of each are cut
    const WaveRows<R> rows(wy, z, ny, nz);
    WaveMasks<TX> mk;
    const bool links = wave_masks<TX>(f, x0, wy, z, rows, mk);
    // byte offsets of the lane's pull sources x - c_i within a direction's
    // array (below 2^32): a lane part for the x neighbour and, where the
    // wavefront holds several rows, the y neighbour, and a scalar part for
    // the rest
    constexpr uint32_t kB = sizeof(T);
    const uint32_t xb[3] = {kB * (uint32_t)(x == 0 ? nx - 1 : x - 1), kB * (uint32_t)x,
                            kB * (uint32_t)(x + 1 >= nx ? 0 : x + 1)};
    uint32_t yb[3], zb[3];  // lane part of y (scalar where R == 1) and scalar part of z
#pragma unroll
    for (int k = 0; k < 3; ++k) {
        yb[k] = kB * (uint32_t)(nx * (R == 1 ? rows.y[k] : wrap1(y + k - 1, ny)));
        zb[k] = kB * (uint32_t)(nx * ny) * (uint32_t)rows.z[k];
    }

    lds_barrier();  // the previous tile's readers of lds are done
    // the pulls of the fluid nodes go straight from HBM into lds.val (one
    // word per lane, 16-bit values zero-extended), in flight while the tile's
    // links are listed and formed.  A pull from a solid source brings a value
    // that nobody reads: the link's value replaces it once it has landed.
    if (__builtin_amdgcn_inverse_ballot_w64(mk.fluid))
        pull_from<S, 0>(reinterpret_cast<const char *>(src), Ns, xb, yb, zb, lds, wv * 64);
    // listed links: not the inflow plane's directions from the removed domain
    const bool inflow = z == f->s.zieb_z;
    auto links_of = [&](const WaveMasks<TX> &m, int i) -> uint64_t { return inflow && CZ[i] == 1 ? 0ull : m.cut[i]; };
    int cnt = 0;
    if (links)
#pragma unroll
        for (int i = 1; i < kQ; ++i) cnt += __popcll(links_of(mk, i));
    for (int k = tid; k < kRec; k += kBlock) lds.key[k] = -1;
    for (int k = tid; k < kCopies * kRec * 6; k += kBlock) (&lds.sum[0][0][0])[k] = 0ull;
    if (lane == 0) lds.wtot[wv] = cnt | (mk.fluid ? 1 << 20 : 0);  // cnt <= 64 * 18
    lds_barrier();  // publishes the counts and the table's reset
    int tot = 0, first = 0, flags = 0;  // the tile's links, those of the wavefronts before, whether any node is fluid
#pragma unroll
    for (int w = 0; w < kBlock / 64; ++w) {
        const int v = __builtin_amdgcn_readfirstlane(lds.wtot[w]);
        if (w < wv) first += v & 0xFFFFF;
        tot += v & 0xFFFFF;
        flags |= v;
    }
    if (!(flags >> 20)) return;

    // 2. the tile's links, listed and spread over the workgroup, in rounds
    //    of kLinkCap.  An item is node << 6 | I << 1 | (the node behind x
    //    is solid).  A wavefront lists its links direction by
    //    direction, so that neighbouring items read neighbouring nodes of
    //    the same arrays.  The value of a thread's first link waits until
    //    every pull of the tile has landed, then replaces what was pulled.
    auto list = [&](const WaveMasks<TX> &m, int base, bool all) {  // all: or those in [base, base + kLinkCap)
        int k0 = -base;
#pragma unroll
        for (int i = 1; i < kQ; ++i) {
            const uint64_t c = links_of(m, i);
            if (__builtin_amdgcn_inverse_ballot_w64(c)) {
                const int k = (int)__builtin_amdgcn_mbcnt_hi((uint32_t)(c >> 32),
                                                             __builtin_amdgcn_mbcnt_lo((uint32_t)c, first + k0));
                // the source of opp(i) is the node behind x, x + c_i
                const uint32_t solid = __builtin_amdgcn_inverse_ballot_w64(m.cut[opp(i)]) ? 1u : 0u;
                if (all || (k >= 0 && k < kLinkCap)) lds.item[k] = (uint16_t)((uint32_t)tid << 6 | (uint32_t)i << 1 | solid);
            }
            k0 += __popcll(c);
        }
    };
    if (cnt) {
        if (tot <= kLinkCap) list(mk, 0, true);
        else list(mk, 0, false);
    }
    bool landed = false;  // every pull of the tile has landed
    for (int base = 0; base < tot; base += kLinkCap) {
        if (base) {
            lds_barrier();  // the previous round's list is processed
            WaveMasks<TX> again;  // (not kept: few tiles need a second round)
            if (wave_masks<TX>(reread(f), x0, wy, z, WaveRows<R>(wy, z, ny, nz), again)) list(again, base, false);
        }
        lds_barrier();  // the list is written (an LDS-only barrier: the pulls stay in flight)
        const int n = min(kLinkCap, tot - base);
        for (int j0 = 0; j0 < n; j0 += kBlock) {
            const int j = j0 + tid;
            uint32_t bits = 0, it = 0;
            if (j < n) {
                it = lds.item[j];
                bits = fused_link<S, TX, TY, TZ>(reread(f), src, lds, x0, y0, z0, it, t);
            }
            if (!landed) {
                wait_vmem();
                lds_barrier();
                landed = true;
            }
            if (j < n) lds.val[(it >> 1) & 31u][it >> 6] = bits;
        }
    }
    if (tot > 0) {
        lds_barrier();  // the link values and the tile's body sums are complete
        // 4. the tile's body sums, the copies added up: one thread per body
        //    and component, so that a body's six sums go out in one access
        if (tid < 6 * kRec) {
            const int slot = tid / 6, c = tid - 6 * slot;
            const int key = lds.key[slot];
            unsigned long long v = 0ull;
#pragma unroll
            for (int q = 0; q < kCopies; ++q) v += lds.sum[q][slot][c];
            if (key >= 0 && v) atomicAdd(fix_slot(f, key, t) + c, v);
        }
    }

    // 3. pull, collide and store (whole wavefronts; none with no fluid lane)
    if (!mk.fluid || !__builtin_amdgcn_inverse_ballot_w64(mk.in)) return;
    const bool fluid = __builtin_amdgcn_inverse_ballot_w64(mk.fluid);
    float g[kQ];
    wait_vmem();  // this wavefront's pulls have landed in lds.val (the link values are there since the barrier)
    if (!fluid) {
#pragma unroll
        for (int i = 0; i < kQ; ++i) g[i] = 0.0f;
    } else {
#pragma unroll
        for (int i = 0; i < kQ; ++i) g[i] = St::from_bits(lds.val[i][tid]);
    }
    f = reread(f);
    StepArgs a;  // what the collision reads
    a.Ns = f->s.Ns;
    a.tau0 = f->s.tau0;
    a.smag_k = f->s.smag_k;
    a.rho0 = f->s.rho0;
    a.fx = f->s.fx;
    a.fy = f->s.fy;
    a.fz = f->s.fz;
    a.flag = f->s.flag;
    a.stream_out = f->s.stream_out;
    a.zieb_state = f->s.zieb_state;
    // index of the lane's node
    const uint32_t idx = (uint32_t)x + (uint32_t)nx * ((uint32_t)y + (uint32_t)ny * (uint32_t)z);
    if (inflow && fluid) zieb_plane<S>(a, src, idx, g);
    collide_store<S>(a, g, fluid, idx, static_cast<T *>(dstv));
}

// Force entry i of a step (spheres, then walls) from its fixed-point sums,
// which are cleared.
__device__ __forceinline__ void finish_value(const FinishArgs &fa, int i)
{
    const int ns = 6 * fa.nb;
    unsigned long long sum;
    if (i < ns) {
        sum = fa.fsum[i];
        fa.fsum[i] = 0ull;
    } else {
        const int w = (i - ns) / 6, c = (i - ns) % 6;
        unsigned long long *p = fa.fsum + 6 * ((size_t)fa.wall_base + (size_t)w * kWallRep) + c;
        sum = 0ull;
        for (int r = 0; r < kWallRep; ++r) {
            sum += p[6 * r];
            p[6 * r] = 0ull;
        }
    }
    const double v = (double)(long long)sum * (1.0 / kFixScale);
    fa.out[i] = v;
    if (fa.out2) fa.out2[i] = v;
}

// Seven waves per SIMD: the LDS of a workgroup allows seven per CU, and the
// compiler then keeps the kernel within 72 VGPRs without spilling.
template <int S, int TX, int TY, int TZ>
__global__ __launch_bounds__(kBlock) __attribute__((amdgpu_waves_per_eu(7, 7))) void k_fused(FusedArgs f)
{
    __shared__ FusedLds lds;
    // the previous step's forces, if nobody has read them yet (their sums
    // are in the other buffer)
    // (a stride of 2^31 threads, a lattice of 2^23 tiles, would turn an int
    // negative and never end)
    if (f.fin.fsum)
        for (size_t i = (size_t)blockIdx.x * kBlock + threadIdx.x; i < 6 * (size_t)(f.fin.nb + f.fin.n_walls);
             i += (size_t)gridDim.x * kBlock)
            finish_value(f.fin, (int)i);
    // (f is the kernel's only argument: it lies at the segment's start)
    const ArgPtr p = (ArgPtr)__builtin_amdgcn_kernarg_segment_ptr();
    const int t = xcd_remap<kTileChunk<S>>(blockIdx.x, gridDim.x);
    fused_tile<S, TX, TY, TZ>(p, f.s.src, f.s.dst, f.s.backward ? (int)gridDim.x - 1 - t : t, lds);
}

// The spheres' entries, one per thread, by the first `sphere_blocks` blocks;
// then the walls', one per wavefront, whose lanes take the copies (a kWallRep
// of 64): all copies in one round trip.
__global__ __launch_bounds__(kBlock) void k_finish(FinishArgs fa, int sphere_blocks)
{
    static_assert(kWallRep == 64, "a lane per copy");
    if ((int)blockIdx.x < sphere_blocks) {
        const int i = blockIdx.x * kBlock + threadIdx.x;
        if (i < 6 * fa.nb) finish_value(fa, i);
        return;
    }
    const int e = ((int)blockIdx.x - sphere_blocks) * (kBlock / 64) + (int)(threadIdx.x >> 6), lane = threadIdx.x & 63;
    if (e >= 6 * fa.n_walls) return;
    const int w = e / 6, c = e - 6 * w;
    unsigned long long *p = fa.fsum + 6 * ((size_t)fa.wall_base + (size_t)w * kWallRep + lane) + c;
    unsigned long long sum = *p;
    *p = 0ull;
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) sum += __shfl_xor(sum, off);
    if (lane != 0) return;
    const double v = (double)(long long)sum * (1.0 / kFixScale);
    fa.out[6 * fa.nb + e] = v;
    if (fa.out2) fa.out2[6 * fa.nb + e] = v;
}

__global__ __launch_bounds__(kBlock) void k_zero_fix(unsigned long long *p, int n)
{
    const int i = blockIdx.x * kBlock + threadIdx.x;
    if (i < n) p[i] = 0ull;
}

// Persistent fused step over the tiles of many lattices, all with the
// batch's tile shape.  Member m owns the global tiles [tile_begin[m],
// tile_begin[m + 1]); XCD k (workgroups k, k + 8, ...) takes its share of
// the global tile range (runs of neighbouring tiles, by xcd_item) from its
// own queue, so that each XCD works on neighbouring tiles of the same
// members while every XCD draws from all of them.  Six waves per SIMD: its
// tile loop needs more registers than seven would leave.
template <int S, int TX, int TY, int TZ>
__global__ __launch_bounds__(kBlock) __attribute__((amdgpu_waves_per_eu(6, 6))) void k_batch_fused(BatchStepArgs b)
{
    __shared__ FusedLds lds;
    __shared__ int next[2];  // the workgroup's tile of this iteration and of the next, in turn
    const int xcd = blockIdx.x & 7;
    int *q = b.queue + xcd * kQueueStride;  // the XCD's tiles in turn, by xcd_item
    if (threadIdx.x == 0) next[0] = atomicAdd(q, 1);
    lds_barrier();
    // the member of the previous tile is kept: a workgroup's next tile is
    // usually in the same member
    int mb = 0, me = 0;
    ArgPtr f = nullptr;
    const void *src = nullptr;
    void *dst = nullptr;
    for (int k = 0;; ++k) {
        int gt = xcd_item<kTileChunk<S>>(xcd, __builtin_amdgcn_readfirstlane(next[k & 1]));
        if (gt >= b.total_tiles) break;  // the XCD's later items lie beyond too
        if (b.backward && b.cur[0]) gt = b.total_tiles - 1 - gt;
        // the next tile is taken now, its atomic in flight during this one
        int pre = 0;
        if (threadIdx.x == 0) pre = atomicAdd(q, 1);
        if (gt < mb || gt >= me) {
            int m = 0, top = b.n;  // largest m with tile_begin[m] <= gt
            while (top - m > 1) {
                const int mid = (m + top) >> 1;
                if (b.members[mid].tile_begin <= gt) m = mid;
                else top = mid;
            }
            m = __builtin_amdgcn_readfirstlane(m);
            const BatchMember &bm = b.members[m];
            mb = bm.tile_begin;
            me = m + 1 < b.n ? b.members[m + 1].tile_begin : b.total_tiles;
            f = (ArgPtr)(uintptr_t)&bm.f;
            const int c = __builtin_amdgcn_readfirstlane(b.cur[m]);
            src = c ? bm.pop[1] : bm.pop[0];
            dst = c ? bm.pop[0] : bm.pop[1];
        }
        fused_tile<S, TX, TY, TZ>(f, src, dst, gt - mb, lds);
        if (threadIdx.x == 0) next[(k + 1) & 1] = pre;
        lds_barrier();
    }
}

// Forces of every member of a batch: one thread per force entry.
__global__ __launch_bounds__(kBlock) void k_batch_finish(BatchStepArgs b)
{
    const int g = blockIdx.x * kBlock + threadIdx.x;
    if (g >= b.total_forces) return;
    int m = 0, top = b.n;  // largest m with force_begin[m] <= g
    while (top - m > 1) {
        const int mid = (m + top) >> 1;
        if (b.members[mid].force_begin <= g) m = mid;
        else top = mid;
    }
    finish_value(b.members[m].fin, g - b.members[m].force_begin);
}

__global__ __launch_bounds__(kBlock) void k_batch_flip(int *cur, int n, int *queue)
{
    const int i = blockIdx.x * kBlock + threadIdx.x;
    if (i < n) cur[i] ^= 1;
    if (i < kQueueInts) queue[i] = 0;  // the tile queues of the next step
}

template <int S>
hipError_t launch_fused_s(const FusedArgs &f, hipStream_t s, hipEvent_t start, hipEvent_t stop)
{
    const dim3 grid(f.s.n_tiles), block(kBlock);
    void (*k)(FusedArgs) = nullptr;
    switch (f.s.tile) {
    case kTile64x2x2: k = k_fused<S, 64, 2, 2>; break;
    case kTile32x4x2: k = k_fused<S, 32, 4, 2>; break;
    case kTile32x2x4: k = k_fused<S, 32, 2, 4>; break;
    case kTile16x8x2: k = k_fused<S, 16, 8, 2>; break;
    default: return hipErrorInvalidValue;
    }
    if (start || stop)
        hipExtLaunchKernelGGL(k, grid, block, 0, s, start, stop, 0, f);
    else
        hipLaunchKernelGGL(k, grid, block, 0, s, f);
    return hipGetLastError();
}

template <int S>
const void *batch_kernel_s(int shape)
{
    switch (shape) {
    case kTile64x2x2: return (const void *)k_batch_fused<S, 64, 2, 2>;
    case kTile32x4x2: return (const void *)k_batch_fused<S, 32, 4, 2>;
    case kTile32x2x4: return (const void *)k_batch_fused<S, 32, 2, 4>;
    case kTile16x8x2: return (const void *)k_batch_fused<S, 16, 8, 2>;
    default: return nullptr;
    }
}

const void *batch_kernel(int storage, int shape)
{
    switch (storage) {
    case 0: return batch_kernel_s<0>(shape);
    case 1: return batch_kernel_s<1>(shape);
    case 2: return batch_kernel_s<2>(shape);
    default: return nullptr;
    }
}

inline int nblk(long n) { return (int)((n + kBlock - 1) / kBlock); }

}  // namespace

hipError_t launch_fused(int storage, const FusedArgs &f, hipStream_t s, hipEvent_t start, hipEvent_t stop)
{
    switch (storage) {
    case 0: return launch_fused_s<0>(f, s, start, stop);
    case 1: return launch_fused_s<1>(f, s, start, stop);
    case 2: return launch_fused_s<2>(f, s, start, stop);
    default: return hipErrorInvalidValue;
    }
}

hipError_t launch_finish(const FinishArgs &fa, hipStream_t s)
{
    const int sphere_blocks = nblk(6 * fa.nb), wall_blocks = (6 * fa.n_walls + kBlock / 64 - 1) / (kBlock / 64);
    if (sphere_blocks + wall_blocks <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_finish, dim3(sphere_blocks + wall_blocks), dim3(kBlock), 0, s, fa, sphere_blocks);
    return hipGetLastError();
}

hipError_t launch_zero_fix(unsigned long long *p, int n, hipStream_t s)
{
    if (n <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_zero_fix, dim3(nblk(n)), dim3(kBlock), 0, s, p, n);
    return hipGetLastError();
}

// The device array behind lbm_step_noalloc's force sums.  Host code takes
// its address per device from static_fix_scratch and never uses the name.
static __device__ __align__(256) unsigned long long scratch[2 * kStaticFixHalf];

hipError_t static_fix_scratch(unsigned long long **out)
{
    static std::mutex mu;
    static std::map<int, unsigned long long *> addr;  // device -> address of scratch there
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    std::lock_guard<std::mutex> lock(mu);
    auto it = addr.find(dev);
    if (it == addr.end()) {
        void *p = nullptr;
        e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
        if (e != hipSuccess) return e;
        it = addr.emplace(dev, static_cast<unsigned long long *>(p)).first;
    }
    *out = it->second;
    return hipSuccess;
}

int batch_step_blocks_per_cu(int storage, int shape)
{
    const void *k = batch_kernel(storage, shape);
    int n = 0;
    if (!k || hipOccupancyMaxActiveBlocksPerMultiprocessor(&n, k, kBlock, 0) != hipSuccess || n < 1) return 1;
    return n;
}

hipError_t launch_batch_step(int storage, int shape, const BatchStepArgs &b, int grid, hipStream_t s)
{
    if (b.total_tiles <= 0) return hipSuccess;
    const void *k = batch_kernel(storage, shape);
    if (!k) return hipErrorInvalidValue;
    BatchStepArgs arg = b;
    void *args[] = {&arg};
    return hipLaunchKernel(k, dim3(grid), dim3(kBlock), args, 0, s);
}

hipError_t launch_batch_finish(const BatchStepArgs &b, hipStream_t s)
{
    if (b.total_forces <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_batch_finish, dim3(nblk(b.total_forces)), dim3(kBlock), 0, s, b);
    return hipGetLastError();
}

hipError_t launch_batch_flip(int *cur, int n, int *queue, hipStream_t s)
{
    hipLaunchKernelGGL(k_batch_flip, dim3(nblk(std::max(n, kQueueInts))), dim3(kBlock), 0, s, cur, n, queue);
    return hipGetLastError();
}

}  // namespace lbm

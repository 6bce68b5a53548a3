// Device building blocks of the fused step: the pull gather (streaming with
// the second-order interpolation and the impermeable-wall scheme).
//
// Storage.  Per species and node the state is kept as
//     plane 0:       P0 = f~_0                                (rest population)
//     plane a >= 1:  g_a = f~_a - (w_a/w_0) P0                (deviation from rest)
// i.e. the populations relative to the rest state of reference density
// r* = P0/w_0; the species density is rho = r* + sum_{a>=1} g_a.  This is the
// same information as the Q post-collision populations in the same number of
// floats, but the small deviations carry the low-order bits: the mass and the
// momentum -- small differences of O(rho) numbers in the plain representation
// -- are kept to FP32 precision of the deviations, not of rho (when P0 is
// rounded on store, its rounding error is moved isotropically into the g_a,
// so no mass is lost).  The gather never forms an O(rho) population: the
// reference part of a streamed population enters only through differences
// P0(O+k) - P0(O), which are exact or nearly so.
//
// Gather.  A work-group owns a block of cross-section columns (x in 2-D,
// (x, y) in 3-D); each thread owns one column and marches through layers
// [m0, m1) of the slowest axis (y in 2-D, z in 3-D).  The interpolation of
// eq. (Second_order_spatial_interpolation) is a product of 1-D quadratic
// Lagrange factors, applied as nested 1-D passes: the cross-section passes
// read neighbouring columns straight from memory (L1/L2 hits: the
// neighbouring lanes of the same instruction read the same rows), and the
// pass along the marching axis is carried in registers (two running partial
// sums per deviation plane, three layers of the reference stencil), so every
// value of a layer is fetched from HBM about once.  Species 1 (c = 1) is an
// exact one-node shift.
//
// Addressing.  Loads and stores are buffer instructions: one buffer resource
// per direction plane (formed by scalar adds where a layer uses it) and the
// node as a 32-bit per-lane byte offset, so no per-load 64-bit address
// arithmetic is needed (each species' Q planes stay below 2 GiB; a buffer
// holds up to 4 of them).  The plane is not a scalar offset of the
// instruction: one takes the vector memory pipe 9 cycles instead of 5.  (Where a
// thread holds every species it is: see SpanBuf.)
//
// For every node the gather hands over, per species s:
//   P0[s]     the stored rest population at the node (it does not stream),
//   F[s][a]   f_a(O) - w_a r*(O) for a >= 1, f_a the streamed population.
// With the FP32 weight triples summing to exactly 1 and the wall terms handing
// back the stored weights that a solid layer would have received (Appendix A),
// the update moves mass without systematic drift.
#pragma once

#include "common.hpp"
#include "lattice.hpp"

namespace lbmmc {

// Work-groups are dealt to the eight XCDs round-robin by work-group id.  Map
// the id to a "virtual" id so that the work-groups on one XCD take a
// contiguous range of the (spatially ordered) tile list and share its halo
// rows in their XCD's L2.  Bijective for any grid size G.
__device__ __forceinline__ int virtual_block(int G) {
    const int b = blockIdx.x;
    const int k = b & 7, idx = b >> 3, per = G >> 3, rem = G & 7;
    return k * per + (k < rem ? k : rem) + idx;
}

// View of the Q planes of one species of a lattice (plane a of the view is
// direction a of that species).
struct Buf {
    const char* base;   // plane 0
    unsigned pb;        // bytes per plane
    int bytes;          // range-checked bytes beyond a plane's base
};

__device__ __forceinline__ Buf make_buf(const float* base, int64_t floats, int64_t plane) {
    return Buf{reinterpret_cast<const char*>(base), (unsigned)(plane * 4), (int)(floats * 4)};
}

// Buffer resource of plane p.  (The product in 64 bits: the planes a layer
// reads in turn then follow each other by a 64-bit scalar add.)
__device__ __forceinline__ __amdgpu_buffer_rsrc_t plane_rsrc(const Buf& b, int p) {
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<char*>(b.base) + (size_t)p * b.pb,
                                             (short)0, b.bytes, 0x00020000);
}

// The view of species s of a lattice whose planes start at `lattice`.
template <int LAT>
__device__ __forceinline__ Buf species_buf(const float* lattice, int64_t plane, int s) {
    constexpr int Q = Lat<LAT>::Q;
    return make_buf(lattice + (int64_t)s * Q * plane, (int64_t)Q * plane, plane);
}

// The same view with one buffer resource over the species' planes and the plane
// as the instruction's scalar offset, for the kernels in which a thread holds
// every species: N Q resources do not fit the scalar registers there, and the
// compiler keeps what does not fit in lanes of VGPRs, four moves for each load that
// needs one (three species at the equilibrium boundary: 1311 scalars spilled, 29
// with this view).  us with resources per plane and with this view: a step with
// the equilibrium boundary 1024x64 three species 17.0, 11.0, 96x48x40 125, 44;
// with moving walls, 1024x64 in tiles of 8 rows, 69, 50; with resting walls 33.5,
// 26.2; the initial state's VJP on 128x64x64 with four species 149, 115.
struct SpanBuf {
    __amdgpu_buffer_rsrc_t r;
    int pb;             // bytes per plane
};

template <int LAT>
__device__ __forceinline__ SpanBuf species_span(const float* lattice, int64_t plane, int s) {
    constexpr int Q = Lat<LAT>::Q;
    return SpanBuf{__builtin_amdgcn_make_buffer_rsrc(
                       const_cast<float*>(lattice + (int64_t)s * Q * plane), (short)0,
                       (int)(Q * plane * 4), 0x00020000),
                   (int)(plane * 4)};
}

// Byte offset that lies beyond any species view (the host keeps every
// species below 2 GiB): a raw buffer load at it is range-checked and returns
// 0, which is exactly the contribution of a solid (beyond-the-wall) source.
constexpr unsigned kSolid = 0x80000000u;

// Sum of two byte offsets where either may carry kSolid.  Offsets are added as
// signed 32-bit values with saturation: an in-lattice offset plus a
// neighbour step stays exact, and a sum with kSolid in it stays at or below
// INT_MIN plus a few steps, out of range as an unsigned offset.  A plain add
// would let two markers (the node next to walls on two axes reading the
// corner source beyond both) cancel modulo 2^32 into an in-range read.
__device__ __forceinline__ unsigned oadd(unsigned a, unsigned b) {
    return (unsigned)__builtin_elementwise_add_sat((int)a, (int)b);
}

// value of plane p at byte offset `vb` (per lane)
__device__ __forceinline__ float ldb(const Buf& b, int p, unsigned vb) {
    return __builtin_bit_cast(
        float, __builtin_amdgcn_raw_buffer_load_b32(plane_rsrc(b, p), (int)vb, 0, 0));
}
__device__ __forceinline__ float ldb(const SpanBuf& b, int p, unsigned vb) {
    return __builtin_bit_cast(
        float, __builtin_amdgcn_raw_buffer_load_b32(b.r, (int)vb, p * b.pb, 0));
}
// Cache policy of the population stores (a launch writes every value once
// and reads none of them back).  kStoreNT, the non-temporal (`nt`) policy,
// suits states larger than the last-level cache; kStoreWT, device scope
// (`sc1`: written through to the last-level cache), suits states that fit in
// it and are read again from there by the next step.  kStoreWB, written back
// from the L2, is for stores that do not fill their lines (k_step_strip: two
// strips write the line between them).  Neither changes a value or a coherence
// rule; the host picks one per context by the size of the two population
// buffers.
constexpr int kStoreWB = 0;
constexpr int kStoreNT = 2;
constexpr int kStoreWT = 16;
template <int POL = kStoreNT>
__device__ __forceinline__ void stb(const Buf& b, int p, unsigned vb, float v) {
    __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(unsigned, v), plane_rsrc(b, p),
                                          (int)vb, 0, POL);
}
template <int POL = kStoreNT>
__device__ __forceinline__ void stb(const SpanBuf& b, int p, unsigned vb, float v) {
    __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(unsigned, v), b.r, (int)vb,
                                          p * b.pb, POL);
}

// Neighbour index i+k (k = -1, +1) on an axis of n nodes: wrapped when periodic
// (wall = 0), -1 when the source node is solid (beyond a wall, wall = -1).
// Written as selects: as branches the uniform uses cost a jump each on the
// critical path of every layer.
__device__ __forceinline__ int nbr(int i, int k, int n, int wall) {
    const int j = i + k;
    const int lo = j < 0 ? ((j + n) | wall) : j;
    return j >= n ? ((j - n) | wall) : lo;
}

// Weights of the source offsets -1, 0, +1 for a direction component of sign p
// of a species with triple L (given for Courant number +c).
struct W3 {
    float m, z, p;
};
__device__ __forceinline__ W3 wsel(int p, const float* L) {
    if (p > 0) return W3{L[0], L[1], L[2]};
    if (p < 0) return W3{L[2], L[1], L[0]};
    return W3{0.0f, 1.0f, 0.0f};
}

// Per-column geometry: byte offsets of the cross-section neighbours relative
// to the column (kSolid for a solid neighbour).
struct Col {
    unsigned bxm, bxp, bym, byp;
};

// Cross-lane moves along a wave: lane i takes lane i-1's (from_left) or lane
// i+1's (from_right) value; the lane with no such neighbour takes `old`.
__device__ __forceinline__ float from_left(float old, float v) {
    return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(
        __builtin_bit_cast(int, old), __builtin_bit_cast(int, v), 0x138, 0xF, 0xF, false));
}
__device__ __forceinline__ float from_right(float old, float v) {
    return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(
        __builtin_bit_cast(int, old), __builtin_bit_cast(int, v), 0x130, 0xF, 0xF, false));
}

// x-pass of a plane value z with its x neighbours m (x-1) and q (x+1).
__device__ __forceinline__ float xcomb(W3 w, float m, float z, float q) {
    float v = w.z * z;
    v = fmaf(w.m, m, v);
    v = fmaf(w.p, q, v);
    return v;
}

// Reference stencil of one layer around the column (rest populations P0):
// the centre and the differences to the four cross-section neighbours (a
// solid neighbour, or a whole solid layer, reads as 0).
struct RhoLayer {
    float c, dxm, dxp, dym, dyp;
};

// ---------------------------------------------- reads, one column per thread
// Every value and its x neighbours by loads of their own (any work-group
// shape).

// Cross-section pass of plane p of direction components (q0, q1) around byte
// offset `cen`.
template <int LAT, class View>
__device__ __forceinline__ float hpass_load(const View& b, int p, int q0, int q1, unsigned cen,
                                            const Col& c, const float* L) {
    const W3 wx = wsel(q0, L);
    auto row = [&](unsigned r) {
        if (q0 == 0) return ldb(b, p, r);
        return xcomb(wx, ldb(b, p, oadd(r, c.bxm)), ldb(b, p, r), ldb(b, p, oadd(r, c.bxp)));
    };
    if (Lat<LAT>::DIM == 2 || q1 == 0) return row(cen);
    const W3 wy = wsel(q1, L);
    float v = wy.z * row(cen);
    v = fmaf(wy.m, row(oadd(cen, c.bym)), v);
    v = fmaf(wy.p, row(oadd(cen, c.byp)), v);
    return v;
}

template <int LAT, class View>
__device__ __forceinline__ RhoLayer rho_load(const View& b, int p, unsigned cen, const Col& c) {
    RhoLayer r;
    r.c = ldb(b, p, cen);
    r.dxm = ldb(b, p, oadd(cen, c.bxm)) - r.c;
    r.dxp = ldb(b, p, oadd(cen, c.bxp)) - r.c;
    r.dym = r.dyp = 0.0f;
    if constexpr (Lat<LAT>::DIM == 3) {
        r.dym = ldb(b, p, oadd(cen, c.bym)) - r.c;
        r.dyp = ldb(b, p, oadd(cen, c.byp)) - r.c;
    }
    return r;
}

// Per-lattice constants the gather needs, kept in scalar registers.
struct GatherConst {
    int nx, ny, nz, pitch, nm, walls, lstride;   // walls: wall mask; lstride: floats per layer
    float lam[MAXS][3];
};

__device__ __forceinline__ GatherConst gather_const(const LatParams& P, int dim) {
    GatherConst g;
    g.nx = P.nx; g.ny = P.ny; g.nz = P.nz; g.pitch = P.pitch;
    g.nm = dim == 2 ? P.ny : P.nz;
    g.walls = P.wall_mask;
    g.lstride = dim == 2 ? P.pitch : P.ny * P.pitch;
#pragma unroll
    for (int s = 0; s < MAXS; ++s) {
        g.lam[s][0] = P.lam[s][0]; g.lam[s][1] = P.lam[s][1]; g.lam[s][2] = P.lam[s][2];
    }
    return g;
}

// Per-column geometry of a gather (shared by the joint and per-species forms).
struct ColGeom {
    Col col;
    int sx, sy;            // wall side of the column (-1, 0, +1) on x / y
    unsigned colbase;      // byte offset of the column in layer 0
    unsigned lsb;          // bytes per layer
    int wx, wy, wm;        // walls on x / y / the marching axis (-1: yes, 0: no)
};

template <int LAT>
__device__ __forceinline__ ColGeom col_geom(const GatherConst& G, int x, int y) {
    constexpr int DIM = Lat<LAT>::DIM;
    ColGeom g;
    g.wx = -(G.walls & 1);
    g.wy = DIM == 3 ? -((G.walls >> 1) & 1) : 0;
    g.wm = -((G.walls >> Frame<LAT>::MA) & 1);
    const int xm = nbr(x, -1, G.nx, g.wx), xp = nbr(x, 1, G.nx, g.wx);
    g.col.bxm = xm < 0 ? kSolid : (unsigned)(xm - x) * 4u;
    g.col.bxp = xp < 0 ? kSolid : (unsigned)(xp - x) * 4u;
    g.col.bym = g.col.byp = 0u;
    if constexpr (DIM == 3) {
        const int ym = nbr(y, -1, G.ny, g.wy), yp = nbr(y, 1, G.ny, g.wy);
        g.col.bym = ym < 0 ? kSolid : (unsigned)((ym - y) * G.pitch) * 4u;
        g.col.byp = yp < 0 ? kSolid : (unsigned)((yp - y) * G.pitch) * 4u;
    }
    g.sx = g.wx & (x == 0 ? -1 : (x == G.nx - 1 ? 1 : 0));
    g.sy = g.wy & (y == 0 ? -1 : (y == G.ny - 1 ? 1 : 0));
    g.colbase = (unsigned)((DIM == 2 ? 0 : y * G.pitch) + x) * 4u;
    g.lsb = (unsigned)G.lstride * 4u;
    return g;
}

// byte offset of layer ml (uniform over the wave; kSolid beyond a wall)
__device__ __forceinline__ unsigned layer_base(const ColGeom& g, int ml) {
    return ml < 0 ? kSolid : (unsigned)ml * g.lsb;
}

// byte offset of the column in layer ml (beyond the view beyond a wall)
__device__ __forceinline__ unsigned layer_off(const ColGeom& g, int ml) {
    return oadd(layer_base(g, ml), g.colbase);
}

// wall sides of the node at layer m along the lattice axes x, y, z (-1: next
// to the low wall, +1: next to the high wall, 0: not next to a wall)
struct Sides {
    int s[3];
    bool any;
};

// The equilibrium comparison boundary of Sec. 4.1 (the scheme the paper sets
// against Appendix A on the Loschmidt tube), for a node next to walls, added
// to a gather in which solid sources contributed nothing: a source node O + k
// beyond a wall holds the rest equilibrium w_a rho_s, rho_s the density of the
// fluid node it faces (O + k with each component that crosses a wall set to
// 0), and is interpolated over like any node (eq. Second_order_spatial_
// interpolation, the tensor product in 3-D), so f_a(O) gains
// w_a sum over solid k of Lambda_k(c_a) rho_s(k).  Densities from the stored
// form: rho = P0/w_0 + sum_{a>0} g_a.
template <int LAT, bool BATCH, class View>
__device__ __forceinline__ void eq_wall_terms(const View& B, const GatherConst& G,
                                              const ColGeom& g, int pb0, const float* L,
                                              unsigned own, int m, const Sides& sd,
                                              float (&F)[Lat<LAT>::Q]) {
    using Fr = Frame<LAT>;
    using La = Lat<LAT>;
    constexpr int Q = La::Q;
    constexpr int DIM = La::DIM;
    constexpr int K1 = DIM == 3 ? 1 : 0;
    const float iw0 = 1.0f / La::w(0);
    const int sx = sd.s[0], s1 = DIM == 3 ? sd.s[1] : 0, sm = sd.s[Fr::MA];
    auto pick = [](const W3& w, int k) { return k < 0 ? w.m : (k > 0 ? w.p : w.z); };
#pragma unroll
    for (int km = -1; km <= 1; ++km)
#pragma unroll
        for (int k1 = -K1; k1 <= K1; ++k1)
#pragma unroll
            for (int kx = -1; kx <= 1; ++kx) {
                const bool solx = kx != 0 && kx == sx;
                const bool sol1 = k1 != 0 && k1 == s1;
                const bool solm = km != 0 && km == sm;
                if (!(solx || sol1 || solm)) continue;
                // the facing fluid node: the in-lattice steps of k only
                unsigned cl = (km != 0 && !solm) ? layer_off(g, nbr(m, km, G.nm, g.wm)) : own;
                if (kx != 0 && !solx) cl += kx < 0 ? g.col.bxm : g.col.bxp;
                if (k1 != 0 && !sol1) cl += k1 < 0 ? g.col.bym : g.col.byp;
                float v[Q];
#pragma unroll
                for (int b = 0; b < Q; ++b) v[b] = ldb(B, pb0 + b, cl);
                // (one round trip, not one for each)
                if constexpr (BATCH) __builtin_amdgcn_sched_barrier(0);
                float rho = v[0] * iw0;
#pragma unroll
                for (int b = 1; b < Q; ++b) rho += v[b];
#pragma unroll
                for (int a = 1; a < Q; ++a) {
                    if ((Fr::p0(a) == 0 && kx != 0) || (Fr::p1(a) == 0 && k1 != 0) ||
                        (Fr::pm(a) == 0 && km != 0))
                        continue;
                    float wgt = pick(wsel(Fr::p0(a), L), kx) * pick(wsel(Fr::pm(a), L), km);
                    if constexpr (DIM == 3) wgt *= pick(wsel(Fr::p1(a), L), k1);
                    F[a] = fmaf(La::w(a) * wgt, rho, F[a]);
                }
            }
}

// Slot of direction a among the directions with a marching-axis component.
template <int LAT>
__host__ __device__ constexpr int mar_slot(int a) {
    int k = 0;
    for (int b = 1; b < a; ++b) k += Frame<LAT>::pm(b) != 0 ? 1 : 0;
    return k;
}
template <int LAT>
constexpr int kMarDirs = mar_slot<LAT>(Lat<LAT>::Q);

// The two marching-axis partial sums of every direction with a marching
// component (get/set(k, a): sum k of direction a), in registers.
template <int LAT, bool LDS = false>
struct MarchSums {
    float acc0[Lat<LAT>::Q], acc1[Lat<LAT>::Q];
    __device__ __forceinline__ float get(int k, int a) const { return k ? acc1[a] : acc0[a]; }
    __device__ __forceinline__ void set(int k, int a, float v) {
        if (k)
            acc1[a] = v;
        else
            acc0[a] = v;
    }
};
// The same sums in an LDS area of the wave's own ([2 kMarDirs][64] floats,
// each lane its column; no other lane reads them, so no barrier), so they
// hold no VGPRs.
template <int LAT>
struct MarchSums<LAT, true> {
    float* acc;   // this lane's element of slot 0
    __device__ __forceinline__ float get(int k, int a) const {
        return acc[(2 * mar_slot<LAT>(a) + k) * 64];
    }
    __device__ __forceinline__ void set(int k, int a, float v) {
        acc[(2 * mar_slot<LAT>(a) + k) * 64] = v;
    }
};

// Marching state of one heavier species: the marching-axis partial sums of
// its deviation planes and the reference stencil of layers m-1, m, m+1.
template <int LAT, bool LDS = false>
struct Heavy : MarchSums<LAT, LDS> {
    RhoLayer rl[3];
};

// One layer of a heavier species from what the gather read: the reference
// stencil of the next layer, the x-differences cxm/cxp of the reference in
// rows y-1 and y+1 of this layer (3-D edge directions in the cross-section),
// and hp(a), the cross-section pass of plane a in the next layer (directions
// with a marching component) or in this one.
template <int LAT, bool HL, class HP>
__device__ __forceinline__ void heavy_combine(const float* L, const RhoLayer& nxt,
                                              const float (&cxm)[2], const float (&cxp)[2], HP hp,
                                              Heavy<LAT, HL>& h, float& P0,
                                              float (&F)[Lat<LAT>::Q]) {
    using Fr = Frame<LAT>;
    using La = Lat<LAT>;
    h.rl[2] = nxt;
    const float rc = h.rl[1].c;
    P0 = rc;
    F[0] = 0.0f;
#pragma unroll
    for (int a = 1; a < La::Q; ++a) {
        const W3 wxw = wsel(Fr::p0(a), L);
        const W3 wyw = wsel(Fr::p1(a), L);
        // reference part: delta_a = sum_k Lambda_k P0(O+k) - P0(O)
        auto xpart = [&](const RhoLayer& r) {
            return Fr::p0(a) != 0 ? fmaf(wxw.m, r.dxm, wxw.p * r.dxp) : 0.0f;
        };
        auto ypart = [&](const RhoLayer& r) {
            return Fr::p1(a) != 0 ? fmaf(wyw.m, r.dym, wyw.p * r.dyp) : 0.0f;
        };
        float delta;
        if (Fr::p0(a) != 0 && Fr::p1(a) != 0) {
            // 3-D xy edge: nested pass over rows y-1, y, y+1 of layer m
            const RhoLayer& r = h.rl[1];
            float v = wyw.z * xpart(r);
            v = fmaf(wyw.m, r.dym + fmaf(wxw.m, cxm[0], wxw.p * cxp[0]), v);
            v = fmaf(wyw.p, r.dyp + fmaf(wxw.m, cxm[1], wxw.p * cxp[1]), v);
            delta = v;
        } else if (Fr::pm(a) == 0) {
            delta = xpart(h.rl[1]) + ypart(h.rl[1]);
        } else {
            const W3 wmw = wsel(Fr::pm(a), L);
            // a solid layer reads as zeros: its term is -rc
            const RhoLayer& lo = h.rl[0];
            const RhoLayer& hi = h.rl[2];
            const float tlo = (lo.c - rc) + xpart(lo) + ypart(lo);
            const float thi = (hi.c - rc) + xpart(hi) + ypart(hi);
            const float tmid = xpart(h.rl[1]) + ypart(h.rl[1]);
            delta = fmaf(wmw.p, thi, fmaf(wmw.m, tlo, wmw.z * tmid));
        }
        // deviation part
        float Gv;
        const float hv = hp(a);   // 0 beyond a wall
        if (Fr::pm(a) == 0) {
            Gv = hv;
        } else {
            const W3 wmar = wsel(Fr::pm(a), L);
            const float a0 = h.get(0, a), a1 = h.get(1, a);
            Gv = fmaf(wmar.p, hv, a0);
            h.set(0, a, fmaf(wmar.z, hv, a1));
            h.set(1, a, wmar.m * hv);
        }
        F[a] = fmaf(La::wr(a), delta, Gv);
    }
    h.rl[0] = h.rl[1];
    h.rl[1] = h.rl[2];
}

// Impermeable walls (Appendix A) at a node next to them.  Species 1 (c = 1):
// f_a(O) = f~_abar(O) for a pointing away from a wall (halfway bounce-back).
// The others: f_a(O) += lambda_+1(c) f~_a(O) + lambda_-1(c) f~_abar(O); with
// f~ = (w/w_0) P0 + g and w_a = w_abar the reference part is
// (w_a/w_0)(lambda_+1 + lambda_-1) P0(O).  Where walls meet, what the
// node's populations would stream beyond the walls returns to the node,
// split by the set of walls crossed: into the reversed direction if the
// population moves toward one of them, else into its own direction.
// For a direction pointing away from n_away of the node's walls and
// toward n_tow of them that gives
//   f_a += (1 - (1 - l+)^n_away) (1 - l-)^n_tow f~_a
//        + (1 - (1 - l-)^n_away) f~_abar,
// (l+- = lambda_+-1(c)), the Appendix A terms for a single wall.  The node's
// own planes are read in one batch and the terms taken by selects: one round
// trip for the waves next to a wall, which set a small lattice's step time.
template <int LAT, bool FIRST, class View>
__device__ __forceinline__ void wall_returns(const View& B, const GatherConst& G, const float* L,
                                             unsigned own, const Sides& sd, float rc,
                                             float (&F)[Lat<LAT>::Q]) {
    using La = Lat<LAT>;
    constexpr int Q = La::Q;
    float W[Q];
#pragma unroll
    for (int a = 1; a < Q; ++a) W[a] = ldb(B, a, own);
    // (what follows is kept in this rare branch: moved before the march it
    // would hold registers through every layer)
    int side[3] = {sd.s[0], sd.s[1], sd.s[2]}, walls = G.walls;
    float l0 = L[0], l2 = L[2];
    asm volatile("" : "+v"(side[0]), "+v"(side[1]), "+v"(side[2]), "+s"(walls), "+s"(l0), "+s"(l2));
    const bool meet = (walls & (walls - 1)) != 0;
    const float u0 = 1.0f - l0, u2 = 1.0f - l2;
#pragma unroll
    for (int a = 1; a < Q; ++a) {
        int na = 0, nt = 0;
#pragma unroll
        for (int ax = 0; ax < La::DIM; ++ax) {
            const int c = ax == 0 ? La::cx(a) : (ax == 1 ? La::cy(a) : La::cz(a));
            if (c == 0) continue;
            na += side[ax] == -c ? 1 : 0;
            nt += side[ax] == c ? 1 : 0;
        }
        const float ga = W[a], gb = W[La::opp(a)];
        if constexpr (FIRST) {
            F[a] = na > 0 ? gb : F[a];
        } else {
            float c1 = l2, c2 = l0;
            if (meet) {
                float p0a = na > 1 ? u0 * u0 : u0, p2a = na > 1 ? u2 * u2 : u2;
                if (La::DIM == 3) {
                    p0a = na > 2 ? p0a * u0 : p0a;
                    p2a = na > 2 ? p2a * u2 : p2a;
                }
                const float p0t = nt > 1 ? u0 * u0 : (nt > 0 ? u0 : 1.0f);
                const bool several = na > 1 || nt > 0;
                c1 = several ? (1.0f - p2a) * p0t : c1;
                c2 = several ? 1.0f - p0a : c2;
            }
            const float t = F[a] + (fmaf(c1, ga, c2 * gb) + La::wr(a) * (c1 + c2) * rc);
            F[a] = na > 0 ? t : F[a];
        }
    }
}

// ------------------------------------- gather, one thread per column, loads
// Species 1 (c = 1) at layer m: exact shift, f_a(O) = f~_a(O - c_a).  A solid
// source reads as 0; wall_returns (or, for the equilibrium comparison
// boundary, eq_wall_terms) puts in what the node gets instead.  lo, hi: the
// column in layers m-1 and m+1.
template <int LAT, bool BATCH = false, class View>
__device__ __forceinline__ void shift_load(const View& B, const ColGeom& g, unsigned own,
                                           unsigned lo, unsigned hi, float& P0,
                                           float (&F)[Lat<LAT>::Q]) {
    using Fr = Frame<LAT>;
    using La = Lat<LAT>;
    auto source = [&](int a) {
        const int c0 = Fr::p0(a), c1 = Fr::p1(a), cm = Fr::pm(a);
        unsigned src = cm > 0 ? lo : (cm < 0 ? hi : own);
        if (c0 != 0) src = oadd(src, c0 > 0 ? g.col.bxm : g.col.bxp);
        if (c1 != 0) src = oadd(src, c1 > 0 ? g.col.bym : g.col.byp);
        return src;
    };
    const float r0 = ldb(B, 0, own);
    P0 = r0;
    F[0] = 0.0f;
    if constexpr (BATCH && La::DIM == 2) {
        float ref[La::Q];
#pragma unroll
        for (int a = 1; a < La::Q; ++a) {
            const unsigned src = source(a);
            ref[a] = ldb(B, 0, src);
            F[a] = ldb(B, a, src);
        }
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int a = 1; a < La::Q; ++a) F[a] = fmaf(La::wr(a), ref[a] - r0, F[a]);
    } else {
#pragma unroll
        for (int a = 1; a < La::Q; ++a) {
            const unsigned src = source(a);
            F[a] = fmaf(La::wr(a), ldb(B, 0, src) - r0, ldb(B, a, src));
        }
    }
}

// Start the march of a heavier species (B its view) at layer m0.
template <int LAT, bool HL, class View>
__device__ __forceinline__ void heavy_begin(const View& B, const GatherConst& G, const ColGeom& g,
                                            const float* L, int m0, Heavy<LAT, HL>& h) {
    using Fr = Frame<LAT>;
    const unsigned cm_ = layer_off(g, nbr(m0, -1, G.nm, g.wm)), c0_ = layer_off(g, m0);
    h.rl[0] = rho_load<LAT>(B, 0, cm_, g.col);
    h.rl[1] = rho_load<LAT>(B, 0, c0_, g.col);
#pragma unroll
    for (int a = 1; a < Lat<LAT>::Q; ++a) {
        if (Fr::pm(a) != 0) {
            const W3 wmar = wsel(Fr::pm(a), L);
            const float hm = hpass_load<LAT>(B, a, Fr::p0(a), Fr::p1(a), cm_, g.col, L);
            const float h0 = hpass_load<LAT>(B, a, Fr::p0(a), Fr::p1(a), c0_, g.col, L);
            h.set(0, a, fmaf(wmar.z, h0, wmar.m * hm));
            h.set(1, a, wmar.m * h0);
        } else if constexpr (!HL) {
            h.set(0, a, 0.0f);
            h.set(1, a, 0.0f);
        }
    }
}

// One layer of a heavier species: second-order interpolation, without walls.
template <int LAT, bool BATCH = false, bool HL, class View>
__device__ __forceinline__ void heavy_layer(const View& B, const ColGeom& g, const float* L,
                                            unsigned own, unsigned nxt, Heavy<LAT, HL>& h,
                                            float& P0, float (&F)[Lat<LAT>::Q]) {
    using Fr = Frame<LAT>;
    float cxm[2] = {0.0f, 0.0f}, cxp[2] = {0.0f, 0.0f};
    if constexpr (BATCH && Lat<LAT>::DIM == 2) {
        constexpr int Q = Lat<LAT>::Q;
        const RhoLayer ref = rho_load<LAT>(B, 0, nxt, g.col);
        float vm[Q], vz[Q], vp[Q];
#pragma unroll
        for (int a = 1; a < Q; ++a) {
            const unsigned c = Fr::pm(a) != 0 ? nxt : own;
            vz[a] = ldb(B, a, c);
            if (Fr::p0(a) == 0) continue;
            vm[a] = ldb(B, a, oadd(c, g.col.bxm));
            vp[a] = ldb(B, a, oadd(c, g.col.bxp));
        }
        __builtin_amdgcn_sched_barrier(0);
        heavy_combine<LAT>(L, ref, cxm, cxp,
                           [&](int a) {
                               const W3 wx = wsel(Fr::p0(a), L);
                               return Fr::p0(a) == 0 ? vz[a] : xcomb(wx, vm[a], vz[a], vp[a]);
                           },
                           h, P0, F);
        return;
    }
    if constexpr (Lat<LAT>::DIM == 3) {
#pragma unroll
        for (int j = 0; j < 2; ++j) {
            const unsigned rr = oadd(own, j == 0 ? g.col.bym : g.col.byp);
            const float cc = ldb(B, 0, rr);
            cxm[j] = ldb(B, 0, oadd(rr, g.col.bxm)) - cc;
            cxp[j] = ldb(B, 0, oadd(rr, g.col.bxp)) - cc;
        }
    }
    heavy_combine<LAT>(L, rho_load<LAT>(B, 0, nxt, g.col), cxm, cxp,
                       [&](int a) {
                           return hpass_load<LAT>(B, a, Fr::p0(a), Fr::p1(a),
                                                  Fr::pm(a) != 0 ? nxt : own, g.col, L);
                       },
                       h, P0, F);
}

template <int LAT>
__device__ __forceinline__ Sides wall_sides(const GatherConst& G, const ColGeom& g, int m) {
    constexpr int DIM = Lat<LAT>::DIM;
    const int sm = g.wm & (m == 0 ? -1 : (m == G.nm - 1 ? 1 : 0));
    Sides r;
    r.s[0] = g.sx;
    r.s[1] = DIM == 2 ? sm : g.sy;
    r.s[2] = DIM == 3 ? sm : 0;
    r.any = (r.s[0] | r.s[1] | r.s[2]) != 0;
    return r;
}

// A buffer view whose plane stride the compiler cannot look through: the
// per-plane buffer resources are then formed where a layer uses them (scalar
// adds beside the loads) instead of once before the march, where dozens of
// them would spill to VGPR lanes.
__device__ __forceinline__ Buf fresh(Buf b) {
    b.pb = __builtin_amdgcn_readfirstlane(b.pb);
    asm volatile("" : "+s"(b.pb));
    return b;
}

// Whether the joint gather keeps the loads of a species together (BATCH): in 2-D
// all of a layer's go out before the first of them is used, in 3-D a species'
// before the next one's.  Left to itself the compiler orders a layer of every
// species for few live registers, in the kernels that have much of them live
// across it down to a load or two in flight; the resting walls do better so.  us
// per step without and with: equilibrium boundary 1024x64 three species 11.0,
// 8.9; 4096x1024 222, 217; 128x96x64 quaternary 1474, 512 (96x48x40 three
// species 44, 47: not taken); moving walls 1500x600 three species 57, 41; but
// resting walls 512x512 binary 19.1, 21.3.
template <int LAT, int NS, int EXT>
constexpr bool kBatchLoads = EXT >= 2 && (Lat<LAT>::DIM == 2 || (EXT == 3 && NS == 4));

__device__ __forceinline__ SpanBuf fresh(SpanBuf b) { return b; }

// Forward pull gather of one column through layers [m0, m1), all species
// (B: the species views); calls op(P0, F, m, own) for every layer m (own:
// byte offset of the node within a plane).
template <int LAT, int NS, bool EQ = false, bool BATCH = false, class Op>
__device__ __forceinline__ void march(const SpanBuf (&B)[NS], const GatherConst& G, int x, int y,
                                      int m0, int m1, Op& op) {
    constexpr int Q = Lat<LAT>::Q;
    const ColGeom g = col_geom<LAT>(G, x, y);
    Heavy<LAT> h[NS > 1 ? NS - 1 : 1];
#pragma unroll
    for (int s = 1; s < NS; ++s) heavy_begin<LAT>(B[s], G, g, G.lam[s], m0, h[s - 1]);
    for (int m = m0; m < m1; ++m) {
        const unsigned own = layer_off(g, m);
        const unsigned nxt = layer_off(g, nbr(m, 1, G.nm, g.wm));
        const Sides sd = wall_sides<LAT>(G, g, m);
        float P0[NS], F[NS][Q];
        shift_load<LAT, BATCH>(B[0], g, own, layer_off(g, nbr(m, -1, G.nm, g.wm)), nxt, P0[0],
                               F[0]);
#pragma unroll
        for (int s = 1; s < NS; ++s) {
            if constexpr (BATCH) __builtin_amdgcn_sched_barrier(0);
            heavy_layer<LAT, BATCH>(B[s], g, G.lam[s], own, nxt, h[s - 1], P0[s], F[s]);
        }
        if constexpr (BATCH) __builtin_amdgcn_sched_barrier(0);
        if (sd.any) {
#pragma unroll
            for (int s = 0; s < NS; ++s) {
                if constexpr (EQ)
                    eq_wall_terms<LAT, BATCH>(B[s], G, g, 0, G.lam[s], own, m, sd, F[s]);
                else if (s == 0)
                    wall_returns<LAT, true>(B[s], G, G.lam[s], own, sd, P0[s], F[s]);
                else
                    wall_returns<LAT, false>(B[s], G, G.lam[s], own, sd, P0[s], F[s]);
            }
        }
        op(P0, F, m, own);
    }
}

// --------------------------------- gather, one wave per 64 columns of a row
// What bounds these kernels besides HBM is the vector memory pipe of a
// compute unit: a load of 64 consecutive floats takes it 5 cycles, 9 with a
// scalar offset in the instruction, and 10 if lane 0 and lane 63 read a line
// of their own (measured, rows in L1).  So
//   - every plane gets a buffer resource of its own (scalar adds, no scalar
//     offset);
//   - a plane row is read once, and the x neighbours are taken from the
//     adjacent lanes;
//   - the values beyond the two ends of the wave (two a row, on lines of
//     their own) are read for all rows of a layer by one load: lane k < 32
//     reads the left one of the k-th row, lane 32 + k the right one, and
//     ds_bpermute hands them to lanes 0 and 63 where they are used.
// 2-D heavier species, per layer: 10 loads instead of 16.

// The rows a layer reads, in the order they are kept: `z` slots for the rows,
// `h` slots for the rows whose x neighbours are needed.  REV: the reversed
// gather of the adjoint (no reference stencil, plane 0 at the node itself).  (The
// halo slots and their codes serve 3-D; 2-D lays its halos out by plane, see
// PlaneSlots.)
template <int LAT, bool REV>
struct Slots {
    using Fr = Frame<LAT>;
    static constexpr int Q = Lat<LAT>::Q;
    static constexpr bool D3 = Lat<LAT>::DIM == 3;
    static constexpr int rows(int a) { return Fr::p1(a) != 0 ? 3 : 1; }
    // First slots of every plane.  Layer: z 0 is the reference in the next
    // layer (REV: plane 0 of this one), 3-D forward 1, 2 its rows y-1, y+1
    // and 3, 4 those of this layer; h 0 (3-D 0, 1, 2) is theirs.  Begin (b*):
    // the same for one of the two layers a march starts from, planes with a
    // marching component only.
    static constexpr int zbase = D3 && !REV ? 5 : 1;
    static constexpr int hbase = REV ? 0 : (D3 ? 3 : 1);
    static constexpr int bzbase = REV ? 0 : (D3 ? 3 : 1);
    static constexpr int bhbase = REV ? 0 : 1;
    struct Table {
        int z[Q + 1], h[Q + 1], bz[Q + 1], bh[Q + 1];
    };
    static constexpr Table make() {
        Table t{};
        t.z[1] = zbase;
        t.h[1] = hbase;
        t.bz[1] = bzbase;
        t.bh[1] = bhbase;
        for (int a = 1; a < Q; ++a) {
            const bool x = Fr::p0(a) != 0, m = Fr::pm(a) != 0;
            t.z[a + 1] = t.z[a] + rows(a);
            t.h[a + 1] = t.h[a] + (x ? rows(a) : 0);
            t.bz[a + 1] = t.bz[a] + (m ? rows(a) : 0);
            t.bh[a + 1] = t.bh[a] + (m && x ? 1 : 0);
        }
        return t;
    }
    static constexpr Table tab = make();
    static constexpr int Z = tab.z[Q], H = tab.h[Q], BZ = tab.bz[Q], BH = tab.bh[Q];
    static constexpr int z(int a) { return tab.z[a]; }
    static constexpr int h(int a) { return tab.h[a]; }
    static constexpr int bz(int a) { return tab.bz[a]; }
    static constexpr int bh(int a) { return tab.bh[a]; }
    // what h slot k reads: plane, row (0: y, 1: y-1, 2: y+1), next layer
    static constexpr unsigned code(int plane, int row, bool nxt) {
        return (unsigned)(plane | row << 5 | (nxt ? 128 : 0));
    }
    static constexpr unsigned layer_code(int k) {
        if (!REV && k == 0) return code(0, 0, true);
        if (!REV && D3 && k < 3) return code(0, k, false);
        for (int a = 1; a < Q; ++a)
            if (Fr::p0(a) != 0 && k >= h(a) && k < h(a) + rows(a))
                return code(a, k - h(a), Fr::pm(a) != 0);
        return 0;
    }
    // (nxt here: the march's first layer, else the one before it)
    static constexpr unsigned begin_code(int k) {
        const int r = k / BH, j = k % BH;
        if (!REV && j == 0) return code(0, 0, r != 0);
        for (int a = 1; a < Q; ++a)
            if (Fr::pm(a) != 0 && Fr::p0(a) != 0 && j == bh(a)) return code(a, 0, r != 0);
        return 0;
    }
    static constexpr uint64_t word(bool begin, int w) {
        uint64_t v = 0;
        for (int j = 0; j < 8; ++j) {
            const int k = 8 * w + j;
            if (k < (begin ? 2 * BH : H))
                v |= (uint64_t)(begin ? begin_code(k) : layer_code(k)) << (8 * j);
        }
        return v;
    }
};
static_assert(Slots<1, false>::H <= 32 && 2 * Slots<1, false>::BH <= 32, "halo slots per side");

// The wave's columns: per-lane geometry and, uniform over the wave, the byte
// offsets of the columns beyond its two ends and of rows y-1, y, y+1.
struct WaveGeom {
    ColGeom g;
    unsigned xl, xr, y0, ym, yp;
    int sel;   // ds_bpermute byte address of h slot 0 for this lane
};

template <int LAT>
__device__ __forceinline__ WaveGeom wave_geom(const GatherConst& G, int x0, int x, int y,
                                              bool lane_zero) {
    WaveGeom w;
    w.g = col_geom<LAT>(G, x, y);
    if (lane_zero) w.g.colbase += kSolid;
    x0 = __builtin_amdgcn_readfirstlane(x0);
    const int xm = nbr(x0, -1, G.nx, w.g.wx), xp = nbr(x0 + 63, 1, G.nx, w.g.wx);
    w.xl = xm < 0 || x0 >= G.nx ? kSolid : (unsigned)xm * 4u;
    // (no lane needs it where the row ends within the wave)
    w.xr = xp < 0 || x0 + 63 >= G.nx ? kSolid : (unsigned)xp * 4u;
    w.y0 = w.ym = w.yp = 0u;
    if constexpr (Lat<LAT>::DIM == 3) {
        const int yu = __builtin_amdgcn_readfirstlane(y);
        const int ym = nbr(yu, -1, G.ny, w.g.wy), yp = nbr(yu, 1, G.ny, w.g.wy);
        w.y0 = (unsigned)(yu * G.pitch) * 4u;
        w.ym = ym < 0 ? kSolid : (unsigned)(ym * G.pitch) * 4u;
        w.yp = yp < 0 ? kSolid : (unsigned)(yp * G.pitch) * 4u;
    }
    w.sel = __lane_id() == 63 ? 128 : 0;
    return w;
}

// This lane's part of the halo load: offset without the layer, and which of
// the two layers.
struct HaloLane {
    unsigned off;
    bool nxt;
};

template <int LAT, bool REV, bool BEGIN>
__device__ __forceinline__ HaloLane halo_lane(const Buf& B, const WaveGeom& w, int used) {
    using S = Slots<LAT, REV>;
    const int lane = (int)__lane_id();
    const int k = lane & 31;
    constexpr uint64_t w0 = S::word(BEGIN, 0), w1 = S::word(BEGIN, 1), w2 = S::word(BEGIN, 2);
    const uint64_t v = k < 8 ? w0 : (k < 16 ? w1 : w2);
    const unsigned code = (unsigned)(v >> (8 * (k & 7))) & 255u;
    const unsigned row = (code >> 5) & 3u;
    // (values, not fields: a conditional between fields is one between their
    // addresses, and puts the struct in scratch memory)
    const unsigned xl = w.xl, xr = w.xr, y0 = w.y0, ym = w.ym, yp = w.yp;
    unsigned off = lane < 32 ? xl : xr;
    off = oadd(off, row == 0 ? y0 : (row == 1 ? ym : yp));
    off = oadd(off, (code & 31u) * B.pb);
    return HaloLane{k < used ? off : kSolid, (code & 128u) != 0};
}

__device__ __forceinline__ float halo_load(const Buf& B, const HaloLane& h, unsigned lay,
                                           unsigned lay_nxt) {
    return ldb(B, 0, oadd(h.off, h.nxt ? lay_nxt : lay));
}

// The values beyond the two ends of a row (l taken by lane 0, r by lane 63).
struct Ends {
    float l, r;
};

// Cross-section pass of direction components (q0, q1) from the rows z(0), z(1),
// z(2) (y, y-1, y+1) and their halos h(0), ...
template <int LAT, class Z, class H>
__device__ __forceinline__ float hpass_wave(int q0, int q1, Z z, H h, const float* L) {
    const W3 wx = wsel(q0, L);
    auto row = [&](int j) {
        const float c = z(j);
        if (q0 == 0) return c;
        const Ends e = h(j);
        return xcomb(wx, from_left(e.l, c), c, from_right(e.r, c));
    };
    if (Lat<LAT>::DIM == 2 || q1 == 0) return row(0);
    const W3 wy = wsel(q1, L);
    float v = wy.z * row(0);
    v = fmaf(wy.m, row(1), v);
    v = fmaf(wy.p, row(2), v);
    return v;
}

// Rows of one layer of the forward gather, each by its load: ref(j), the
// reference (z slots 0 .. zbase-1 of Slots); dev(a, j), row j of plane a;
// shift(a), g_a(O - c_a).
template <int LAT>
struct WaveRows {
    const Buf& B;
    const Col& col;
    unsigned lo, own, nxt;
    __device__ __forceinline__ unsigned at(unsigned c, int j) const {
        return j == 0 ? c : oadd(c, j == 1 ? col.bym : col.byp);
    }
    __device__ __forceinline__ float ref(int j) const {
        return ldb(B, 0, j < 3 ? at(nxt, j) : at(own, j - 2));
    }
    __device__ __forceinline__ float dev(int a, int j) const {
        return ldb(B, a, at(Frame<LAT>::pm(a) != 0 ? nxt : own, j));
    }
    __device__ __forceinline__ float shift(int a) const {
        using Fr = Frame<LAT>;
        const int c0 = Fr::p0(a), c1 = Fr::p1(a), cm = Fr::pm(a);
        unsigned src = cm > 0 ? lo : (cm < 0 ? nxt : own);
        if (c0 != 0) src = oadd(src, c0 > 0 ? col.bxm : col.bxp);
        if (c1 != 0) src = oadd(src, c1 > 0 ? col.bym : col.byp);
        return ldb(B, a, src);
    }
};

// The same rows in registers (2-D: of the next layer; 3-D: the layer's own).
template <int LAT, bool REV>
struct WaveRaw {
    float v[Slots<LAT, REV>::Z];
    float hv;
    __device__ __forceinline__ float ref(int j) const { return v[j]; }
    __device__ __forceinline__ float dev(int a, int j) const {
        return v[Slots<LAT, REV>::z(a) + j];
    }
    __device__ __forceinline__ float shift(int a) const {
        return v[Slots<LAT, REV>::zbase + a - 1];
    }
};

template <int LAT>
__device__ __forceinline__ void wave_load(const WaveRows<LAT>& r, int s, WaveRaw<LAT, false>& raw) {
    using S = Slots<LAT, false>;
#pragma unroll
    for (int j = 0; j < S::zbase; ++j) raw.v[j] = r.ref(j);
    if (s == 0) {
#pragma unroll
        for (int a = 1; a < S::Q; ++a) raw.v[S::zbase + a - 1] = r.shift(a);
    } else {
#pragma unroll
        for (int a = 1; a < S::Q; ++a)
#pragma unroll
            for (int j = 0; j < S::rows(a); ++j) raw.v[S::z(a) + j] = r.dev(a, j);
    }
}

// The reference stencil of a layer from its rows c(0), c(1), c(2) and the halo
// of row 0.  Species 1 keeps the values themselves in it (its update takes
// differences to the node's own value, not to the row's centre).
template <int LAT, class C>
__device__ __forceinline__ RhoLayer wave_rho(int s, C c, Ends h) {
    RhoLayer r;
    r.c = c(0);
    const float b = s == 0 ? 0.0f : r.c;
    r.dxm = from_left(h.l, r.c) - b;
    r.dxp = from_right(h.r, r.c) - b;
    r.dym = r.dyp = 0.0f;
    if constexpr (Lat<LAT>::DIM == 3) {
        r.dym = c(1) - b;
        r.dyp = c(2) - b;
    }
    return r;
}

// Start of the march of one species: the stencils of layers m0-1 and m0 and
// (heavier species) the marching sums, from rows ref(j, k) and dev(a, j, k),
// k = 0, 1 the layer, and halos h(slot).
template <int LAT, bool HL, class R, class H>
__device__ __forceinline__ void wave_begin(int s, const float* L, const R& r, H hx,
                                           Heavy<LAT, HL>& h) {
    using Fr = Frame<LAT>;
    using S = Slots<LAT, false>;
    h.rl[0] = wave_rho<LAT>(s, [&](int j) { return r.ref(j, 0); }, hx.ref(0));
    h.rl[1] = wave_rho<LAT>(s, [&](int j) { return r.ref(j, 1); }, hx.ref(1));
    if constexpr (!HL) {
#pragma unroll
        for (int a = 1; a < S::Q; ++a) {
            h.set(0, a, 0.0f);
            h.set(1, a, 0.0f);
        }
    }
    if (s == 0) return;
#pragma unroll
    for (int a = 1; a < S::Q; ++a) {
        if (Fr::pm(a) == 0) continue;
        const W3 wmar = wsel(Fr::pm(a), L);
        auto hp = [&](int k) {
            return hpass_wave<LAT>(Fr::p0(a), Fr::p1(a), [&](int j) { return r.dev(a, j, k); },
                                   [&](int) { return hx.dev(a, k); }, L);
        };
        const float hm = hp(0), h0 = hp(1);
        h.set(0, a, fmaf(wmar.z, h0, wmar.m * hm));
        h.set(1, a, wmar.m * h0);
    }
}

// The rows wave_begin takes, by their loads, and loaded ahead.
template <int LAT>
struct BeginRows {
    const Buf& B;
    const Col& col;
    unsigned c0, c1;
    __device__ __forceinline__ unsigned at(int j, int k) const {
        const unsigned c = k ? c1 : c0;
        return j == 0 ? c : oadd(c, j == 1 ? col.bym : col.byp);
    }
    __device__ __forceinline__ float ref(int j, int k) const { return ldb(B, 0, at(j, k)); }
    __device__ __forceinline__ float dev(int a, int j, int k) const {
        return ldb(B, a, at(j, k));
    }
};
template <int LAT, bool REV>
struct BeginRaw {
    float v[2][Slots<LAT, REV>::BZ];
    __device__ __forceinline__ float ref(int j, int k) const { return v[k][j]; }
    __device__ __forceinline__ float dev(int a, int j, int k) const {
        return v[k][Slots<LAT, REV>::bz(a) + j];
    }
};

template <int LAT, bool REV>
__device__ __forceinline__ void begin_load(const BeginRows<LAT>& r, int s,
                                           BeginRaw<LAT, REV>& raw) {
    using S = Slots<LAT, REV>;
#pragma unroll
    for (int k = 0; k < 2; ++k)
#pragma unroll
        for (int j = 0; j < S::BZ; ++j) raw.v[k][j] = j < S::bzbase ? r.ref(j, k) : 0.0f;
    if (s == 0) return;
#pragma unroll
    for (int a = 1; a < S::Q; ++a) {
        if (Frame<LAT>::pm(a) == 0) continue;
#pragma unroll
        for (int k = 0; k < 2; ++k)
#pragma unroll
            for (int j = 0; j < S::rows(a); ++j) raw.v[k][S::bz(a) + j] = r.dev(a, j, k);
    }
}

// One layer of one species from its rows, without walls.
template <int LAT, bool HL, class R, class H>
__device__ __forceinline__ void wave_layer(int s, const float* L, const R& r, H hx,
                                           Heavy<LAT, HL>& h, float& P0,
                                           float (&F)[Lat<LAT>::Q]) {
    using Fr = Frame<LAT>;
    using La = Lat<LAT>;
    using S = Slots<LAT, false>;
    const RhoLayer nxt = wave_rho<LAT>(s, [&](int j) { return r.ref(j); }, hx.ref(0));
    float cxm[2] = {0.0f, 0.0f}, cxp[2] = {0.0f, 0.0f};
    if constexpr (S::D3) {
#pragma unroll
        for (int j = 0; j < 2; ++j) {
            const float c = r.ref(3 + j);
            const Ends e = hx.ref(1 + j);
            const float b = s == 0 ? 0.0f : c;
            cxm[j] = from_left(e.l, c) - b;
            cxp[j] = from_right(e.r, c) - b;
        }
    }
    if (s == 0) {
        h.rl[2] = nxt;
        const float r0 = h.rl[1].c;
        P0 = r0;
        F[0] = 0.0f;
#pragma unroll
        for (int a = 1; a < La::Q; ++a) {
            const int c0 = Fr::p0(a), c1 = Fr::p1(a), cm = Fr::pm(a);
            const RhoLayer& l = h.rl[cm > 0 ? 0 : (cm < 0 ? 2 : 1)];
            float v = l.c;
            if (c0 != 0 && c1 != 0)
                v = c0 > 0 ? cxm[c1 > 0 ? 0 : 1] : cxp[c1 > 0 ? 0 : 1];
            else if (c0 != 0)
                v = c0 > 0 ? l.dxm : l.dxp;
            else if (c1 != 0)
                v = c1 > 0 ? l.dym : l.dyp;
            F[a] = fmaf(La::wr(a), v - r0, r.shift(a));
        }
        h.rl[0] = h.rl[1];
        h.rl[1] = h.rl[2];
    } else {
        heavy_combine<LAT>(L, nxt, cxm, cxp,
                           [&](int a) {
                               return hpass_wave<LAT>(
                                   Fr::p0(a), Fr::p1(a), [&](int j) { return r.dev(a, j); },
                                   [&](int j) { return hx.dev(a, j); }, L);
                           },
                           h, P0, F);
    }
}

// The halos of a layer (BEGIN: of a march's start): ref(j) those of the
// reference rows, dev(a, j) of row j (BEGIN: of layer j) of plane a.
template <int LAT, bool REV, bool BEGIN>
struct HaloSlots {
    using S = Slots<LAT, REV>;
    static constexpr int N = BEGIN ? 2 * S::BH : S::H;
    static constexpr int ref_slot(int j) { return BEGIN ? j * S::BH : j; }
    static constexpr int dev_slot(int a, int j) {
        return BEGIN ? j * S::BH + S::bh(a) : S::h(a) + j;
    }
};
// 2-D.  The slots are laid out by plane, so that a lane finds its part by a
// few integer operations (on a small lattice the set-up before the first load
// counts): the first load of a march takes rows m0-1, m0 and m0+1, slot 9 row +
// plane; a later layer's takes the next row and, for the planes without a
// marching component, its own, slot = plane.  Slots nothing needs read nothing.
template <bool REV>
struct PlaneSlots {
    using Fr = Frame<0>;
    // whether plane a's halos are needed in a march's start rows / in the next
    // (or own) row of a layer
    static constexpr bool march(int a) {
        return a == 0 ? !REV : Fr::p0(a) != 0 && Fr::pm(a) != 0;
    }
    static constexpr bool own(int a) { return a != 0 && Fr::p0(a) != 0 && Fr::pm(a) == 0; }
    static constexpr unsigned first_mask(bool shift) {
        unsigned v = 0;
        for (int a = 0; a < 9; ++a) {
            const bool mr = march(a) && (!shift || a == 0);
            const bool ow = own(a) && !shift;
            v |= (mr ? 1u : 0u) << a | (mr || ow ? 1u : 0u) << (9 + a) |
                 (mr ? 1u : 0u) << (18 + a);
        }
        return v;
    }
    static constexpr unsigned layer_mask(bool shift) {
        unsigned v = 0;
        for (int a = 0; a < 9; ++a)
            v |= ((march(a) && (!shift || a == 0)) || (own(a) && !shift) ? 1u : 0u) << a;
        return v;
    }
};

// (shift: species 1, which needs the reference's halos only)
template <bool REV>
__device__ __forceinline__ float halo_first(const Buf& B, const WaveGeom& w, bool shift,
                                            unsigned lay_lo, unsigned lay, unsigned lay_nxt) {
    using S = PlaneSlots<REV>;
    const int lane = (int)__lane_id(), k = lane & 31;
    const unsigned mask = shift ? S::first_mask(true) : S::first_mask(false);
    const unsigned xl = w.xl, xr = w.xr;
    const int p = k >= 18 ? k - 18 : (k >= 9 ? k - 9 : k);
    const unsigned row = k >= 18 ? lay_nxt : (k >= 9 ? lay : lay_lo);
    const unsigned off = oadd(oadd(lane < 32 ? xl : xr, row), (unsigned)p * B.pb);
    return ldb(B, 0, (mask >> k) & 1u ? off : kSolid);
}
template <bool REV>
__device__ __forceinline__ HaloLane halo_lane2(const Buf& B, const WaveGeom& w, bool shift) {
    using S = PlaneSlots<REV>;
    const int lane = (int)__lane_id(), k = lane & 31;
    const unsigned mask = shift ? S::layer_mask(true) : S::layer_mask(false);
    const unsigned xl = w.xl, xr = w.xr;
    const unsigned off = oadd(lane < 32 ? xl : xr, (unsigned)k * B.pb);
    // planes 1 and 3 are the ones without a marching component
    return HaloLane{(mask >> k) & 1u ? off : kSolid, k != 1 && k != 3};
}

// The halos, exchanged by ds_bpermute in one batch (issued one by one where
// they are used, every exchange would wait for itself), which leaves the
// vector ALUs, the busiest unit of the 2-D step, alone.  sel: byte address of
// slot 0 of row 0, own and next for this lane.
struct HaloSel {
    int lo, own, nxt;
};
template <bool REV, bool BEGIN>
struct HalosBatch {
    using S = PlaneSlots<REV>;
    float v[3][9];
    __device__ __forceinline__ HalosBatch(const HaloSel& sel, float hv) {
        auto take = [&](int at) {
            return __builtin_bit_cast(
                float, __builtin_amdgcn_ds_bpermute(at, __builtin_bit_cast(int, hv)));
        };
#pragma unroll
        for (int a = 0; a < 9; ++a) {
            if (S::march(a) && BEGIN) {
                v[0][a] = take(sel.lo + 4 * a);
                v[1][a] = take(sel.own + 4 * a);
            }
            if (S::march(a) && !BEGIN) v[2][a] = take(sel.nxt + 4 * a);
            if (S::own(a) && !BEGIN) v[1][a] = take(sel.own + 4 * a);
        }
        __builtin_amdgcn_sched_barrier(0);
    }
    __device__ __forceinline__ Ends ref(int j) const {
        const float h = v[BEGIN ? j : 2][0];
        return Ends{h, h};
    }
    __device__ __forceinline__ Ends dev(int a, int j) const {
        const float h = v[BEGIN ? j : (Frame<0>::pm(a) != 0 ? 2 : 1)][a];
        return Ends{h, h};
    }
};
// 3-D: read into scalar registers where they are used (21 values a layer,
// which would not fit beside its rows).
template <int LAT, bool REV, bool BEGIN>
struct HalosRead : HaloSlots<LAT, REV, BEGIN> {
    using T = HaloSlots<LAT, REV, BEGIN>;
    int hv;
    __device__ __forceinline__ explicit HalosRead(float h) : hv(__builtin_bit_cast(int, h)) {}
    __device__ __forceinline__ Ends get(int k) const {
        return Ends{__builtin_bit_cast(float, __builtin_amdgcn_readlane(hv, k)),
                    __builtin_bit_cast(float, __builtin_amdgcn_readlane(hv, 32 + k))};
    }
    __device__ __forceinline__ Ends ref(int j) const { return get(T::ref_slot(j)); }
    __device__ __forceinline__ Ends dev(int a, int j) const { return get(T::dev_slot(a, j)); }
};
// The wave form of the march of one species.  PF (2-D): the loads of a layer
// are issued a layer ahead, before the previous layer's exchange and
// collision -- which hide their latency -- and before its stores, whose
// acknowledgements they would otherwise wait for (a wave's vector memory
// counter retires in order); the first layer's go out together with those of
// the march's start.  In 3-D the values of a layer do not fit beside the
// collision's registers.
template <int LAT, bool HL, bool PF>
struct FwdWave {
    using S = Slots<LAT, false>;
    static_assert(!PF || Lat<LAT>::DIM == 2, "rows loaded ahead in 2-D only");
    const Buf& B;
    const GatherConst& G;
    const WaveGeom& w;
    int s;
    Heavy<LAT, HL> h;
    HaloLane hl;               // this lane's part of a layer's halo load
    HaloSel sel;               // 2-D: where the current layer's halos are
    WaveRaw<LAT, false> raw;   // PF: the next layer's rows
    BeginRaw<LAT, false> rb;
    float hvb;
    __device__ __forceinline__ int lo(int m) const { return nbr(m, -1, G.nm, w.g.wm); }
    __device__ __forceinline__ int hi(int m) const { return nbr(m, 1, G.nm, w.g.wm); }
    __device__ __forceinline__ WaveRows<LAT> rows(const Buf& Bm, int m) const {
        return WaveRows<LAT>{Bm, w.g.col, layer_off(w.g, lo(m)), layer_off(w.g, m),
                             layer_off(w.g, hi(m))};
    }
    __device__ __forceinline__ float halos(const Buf& Bm, int m) const {
        return halo_load(Bm, hl, layer_base(w.g, m), layer_base(w.g, hi(m)));
    }
    __device__ __forceinline__ BeginRows<LAT> begin_rows(const Buf& Bm, int m0) const {
        return BeginRows<LAT>{Bm, w.g.col, layer_off(w.g, lo(m0)), layer_off(w.g, m0)};
    }
    // the loads of the march's start (PF: with the first layer's; begin() and
    // layer() then take them)
    __device__ __forceinline__ void begin_loads(int m0) {
        const Buf Bm = fresh(B);
        if constexpr (Lat<LAT>::DIM == 2) {
            // (the halos first: they are taken first, and loads return in order)
            hvb = halo_first<false>(Bm, w, s == 0, layer_base(w.g, lo(m0)), layer_base(w.g, m0),
                                    layer_base(w.g, hi(m0)));
            sel = HaloSel{w.sel, w.sel + 36, w.sel + 72};
            raw.hv = hvb;
            if constexpr (PF) {
                begin_load<LAT, false>(begin_rows(Bm, m0), s, rb);
                wave_load<LAT>(rows(Bm, m0), s, raw);
            }
        } else {
            hvb = halo_load(Bm, halo_lane<LAT, false, true>(B, w, 2 * S::BH),
                            layer_base(w.g, lo(m0)), layer_base(w.g, m0));
            hl = halo_lane<LAT, false, false>(B, w, s == 0 ? S::hbase : S::H);
        }
    }
    __device__ __forceinline__ void begin(const float (&L)[3], int m0) {
        if constexpr (Lat<LAT>::DIM == 2) {
            const HalosBatch<false, true> hx(sel, hvb);
            if constexpr (PF) {
                wave_begin<LAT>(s, L, rb, hx, h);
            } else {
                const Buf Bm = fresh(B);
                wave_begin<LAT>(s, L, begin_rows(Bm, m0), hx, h);
            }
        } else {
            const Buf Bm = fresh(B);
            wave_begin<LAT>(s, L, begin_rows(Bm, m0), HalosRead<LAT, false, true>(hvb), h);
        }
    }
    // 2-D: the halo lanes of the layers after the first one
    __device__ __forceinline__ void next_lanes() {
        if constexpr (Lat<LAT>::DIM == 2) hl = halo_lane2<false>(B, w, s == 0);
    }
    __device__ __forceinline__ void load(int m) {
        if constexpr (PF) {
            const Buf Bm = fresh(B);
            raw.hv = halos(Bm, m);
            wave_load<LAT>(rows(Bm, m), s, raw);
        }
    }
    // the gather of layer m, without walls
    __device__ __forceinline__ void layer(const float (&L)[3], int m, bool first, float& P0,
                                          float (&F)[Lat<LAT>::Q]) {
        if constexpr (Lat<LAT>::DIM == 2) {
            if constexpr (PF) {
                wave_layer<LAT>(s, L, raw, HalosBatch<false, false>(sel, raw.hv), h, P0, F);
            } else {
                const Buf Bm = fresh(B);
                const float hv = first ? hvb : halos(Bm, m);
                const WaveRows<LAT> rw = rows(Bm, m);
                WaveRaw<LAT, false> q;
                wave_load<LAT>(rw, s, q);
                wave_layer<LAT>(s, L, q, HalosBatch<false, false>(sel, hv), h, P0, F);
            }
            sel = HaloSel{w.sel, w.sel, w.sel};
        } else {
            // every row of the layer in flight at once: left to the scheduler
            // they go out a few at a time, each waiting for the last (the
            // 256x128x128 layer: 690 instead of 655 us a step)
            const Buf Bm = fresh(B);
            const WaveRows<LAT> rw = rows(Bm, m);
            const HalosRead<LAT, false, false> hx(halos(Bm, m));
            auto whole = [&](int first_species) {
                WaveRaw<LAT, false> q;
                wave_load<LAT>(rw, first_species, q);
                __builtin_amdgcn_sched_barrier(0);
                wave_layer<LAT>(first_species, L, q, hx, h, P0, F);
            };
            if (s == 0)
                whole(0);
            else
                whole(1);
        }
    }
};

template <int LAT, bool HL, bool PF, class Op>
__device__ __forceinline__ void march1_wave(const Buf& B, const GatherConst& G, int s,
                                            const float (&L)[3], const WaveGeom& w, int m0, int m1,
                                            Op& op, float* macc) {
    FwdWave<LAT, HL, PF> fw{B, G, w, s};
    if constexpr (HL) fw.h.acc = macc;
    fw.begin_loads(m0);
    fw.begin(L, m0);
    if (m0 + 1 < m1) fw.next_lanes();
    for (int m = m0; m < m1; ++m) {
        float P0, F[Lat<LAT>::Q];
        fw.layer(L, m, m == m0, P0, F);
        const unsigned own = layer_off(w.g, m);
        const Sides sd = wall_sides<LAT>(G, w.g, m);
        if (sd.any) {
            if (s == 0)
                wall_returns<LAT, true>(fresh(B), G, L, own, sd, P0, F);
            else
                wall_returns<LAT, false>(fresh(B), G, L, own, sd, P0, F);
        }
        if (PF && m + 1 < m1) fw.load(m + 1);
        op(P0, F, m, own);
    }
}

// The same gather for one species s (uniform over the wave; B its view) with
// weight triple L; calls op(P0, F, m, own) with the species' values.  WAVE:
// the wave's 64 lanes are 64 consecutive columns of one row (in order, starting
// at x0) and the wave form is used.  lane_zero marks a lane whose reads all
// return 0.  With HL the marching partial sums live in the LDS area macc (this
// lane's element of the wave's [2 kMarDirs][64] floats).
template <int LAT, bool WAVE, bool HL, bool PF, class Op>
__device__ __forceinline__ void march1(const Buf& B, const GatherConst& G, int s,
                                       const float (&L)[3], int x0, int x, int y, bool lane_zero,
                                       int m0, int m1, Op& op, float* macc) {
    if constexpr (WAVE) {
        march1_wave<LAT, HL, PF>(B, G, s, L, wave_geom<LAT>(G, x0, x, y, lane_zero), m0, m1, op,
                                 macc);
    } else {
        ColGeom g = col_geom<LAT>(G, x, y);
        if (lane_zero) g.colbase += kSolid;
        Heavy<LAT, HL> h;
        if constexpr (HL) h.acc = macc;
        if (s > 0) heavy_begin<LAT>(fresh(B), G, g, L, m0, h);
        for (int m = m0; m < m1; ++m) {
            const Buf Bm = fresh(B);
            const unsigned own = layer_off(g, m);
            const unsigned nxt = layer_off(g, nbr(m, 1, G.nm, g.wm));
            const Sides sd = wall_sides<LAT>(G, g, m);
            float P0, F[Lat<LAT>::Q];
            if (s == 0) {
                shift_load<LAT>(Bm, g, own, layer_off(g, nbr(m, -1, G.nm, g.wm)), nxt, P0, F);
                if (sd.any) wall_returns<LAT, true>(Bm, G, L, own, sd, P0, F);
            } else {
                heavy_layer<LAT>(Bm, g, L, own, nxt, h, P0, F);
                if (sd.any) wall_returns<LAT, false>(Bm, G, L, own, sd, P0, F);
            }
            op(P0, F, m, own);
        }
    }
}

// Column of lane `lane` of a tile of 64 columns: x fastest over bx columns,
// then y (3-D).  Returns whether the lane lies in the lattice; a lane beyond
// it stores nothing and reads column 0 when x is periodic (the right
// neighbour of the row's last column, for the cross-lane gather), or is a
// lane whose reads return 0 at an x wall (`zero`), and in y the last row.
template <int LAT>
__device__ __forceinline__ bool tile_column(const Tile& T, const LatParams& P, int lane, int bx,
                                            int& x, int& y, bool& zero) {
    constexpr int DIM = Lat<LAT>::DIM;
    x = T.x0 + (DIM == 3 ? lane % bx : lane);
    y = DIM == 3 ? T.y0 + lane / bx : 0;
    const bool over = x >= P.nx;
    const bool inside = !over && (DIM == 2 || y < P.ny);
    const int wall = -(P.wall_mask & 1);
    zero = over && wall != 0;
    x = over ? ((P.nx - 1) & wall) : x;
    if (DIM == 3) y = y < P.ny ? y : P.ny - 1;
    return inside;
}

// tile_column for a work-group of W segments of 64 columns (W = bx by / 64):
// with W = 1 the lanes are laid out as tile_column; with W > 1 (bx a multiple
// of 64) segment seg is the 64 columns starting at x0 + 64 (seg mod (bx/64))
// in row y0 + seg / (bx/64), lane = column.  xs: the segment's first column.
template <int LAT>
__device__ __forceinline__ bool tile_column_seg(const Tile& T, const LatParams& P, int lane, int bx,
                                                int seg, int W, int& xs, int& x, int& y,
                                                bool& zero) {
    Tile S = T;
    if (W > 1) {
        const int per_row = bx >> 6;
        int row = 0;
        for (; seg >= per_row; seg -= per_row) ++row;   // (W <= 4: no division)
        S.x0 = T.x0 + 64 * seg;
        S.y0 = T.y0 + row;
        bx = 64;
    }
    xs = S.x0;
    return tile_column<LAT>(S, P, lane, bx, x, y, zero);
}

}  // namespace lbmmc

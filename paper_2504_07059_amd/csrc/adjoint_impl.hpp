// Discrete adjoint of the fused step (reverse mode, written by hand).
//
// The forward step maps the stored state s(t-1) to s(t) = T C(S(T^-1 s(t-1))),
// with S the pull streaming with walls, C the collision, and T the linear
// change of variables of the storage (P0 = f~_0, g_a = f~_a - (w_a/w_0) f~_0).
// One reverse step, given lam_s(t) = dL/ds(t) and s(t-1):
//   kernel A (per node): f(t) = S(T^-1 s(t-1)) by the forward gather;
//            lam_f = T^T lam_s(t); mu = (dC/df)^T lam_f at f(t), stored in a
//            scratch buffer (population space); parameter gradients
//            (dC/dD)^T lam_f and (dC/dg)^T lam_f accumulated in FP64;
//   kernel B (per node): lam_f(t-1) = S^T mu, i.e. the gather of mu with the
//            velocities reversed plus the transposed wall terms; stored as
//            lam_s(t-1) = T^-T lam_f(t-1).
// In a sequence of reverse steps, kernel B of one step and kernel A of the
// step before it run as one fused pass that gathers lam_f from the later
// step's mu directly (T^-T followed by T^T is the identity).
// Both kernels run one wave per species over tiles of 64 columns (their own
// tile list, independent of the forward step's execution shape).  The state
// and adjoint are FP32; parameter gradients are summed in FP64 per thread,
// per work-group and then over work-groups in a fixed order.
#pragma once

#include <hip/hip_runtime.h>

#include <type_traits>

#include "adjoint.hpp"
#include "kernels.hpp"

namespace lbmmc {

// Block reduction of NG doubles, ADDED into this work-group's own partials
// (each slot has one writer, and the reverse steps of a sequence run in
// stream order, so the per-tile sums accumulate deterministically).
template <int NG>
__device__ __forceinline__ void block_reduce_add(double (&acc)[NG], double* __restrict__ out) {
    __shared__ double red[4][NG];
    const int tid = threadIdx.x + blockDim.x * threadIdx.y;
    const int lane = tid & 63, wave = tid >> 6;
    const int nwaves = (blockDim.x * blockDim.y + 63) >> 6;
#pragma unroll
    for (int q = 0; q < NG; ++q) {
        double v = acc[q];
#pragma unroll
        for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off, 64);
        if (lane == 0) red[wave][q] = v;
    }
    __syncthreads();
    if (tid < NG) {
        double s = 0.0;
        for (int w = 0; w < nwaves; ++w) s += red[w][tid];
        out[tid] += s;
    }
}

// ------------------------------------------------------------------ kernel A
// One wave per species over 64 columns.  Per layer: the wave gathers f(t) of
// its species from f~(t-1) and publishes its density and momentum in LDS;
// every wave recomputes the node's forward collision state; each wave runs
// its species' part of the reverse sweep and publishes its contributions to
// the shared adjoints (u, rho, the densities and velocities, y); every wave
// sums them in species order and runs the shared tail (mixture and
// cross-relaxation reverse), then finishes and stores its own species' mu.
template <int LAT, int NS, int POL>
struct AdjSplitOp {
    static constexpr int Q = Lat<LAT>::Q;
    static constexpr int NG = NS * (NS - 1) / 2 + 3;
    static constexpr int D = Lat<LAT>::DIM;
    // packed contribution floats per species
    static constexpr int KX = 3 * D + NS;
    Buf lam;      // lam_s(t), representation space (this species' view)
    Buf mu;       // scratch, population space (this species' view)
    CollConst C;
    float (*x1)[D + 1][64];
    float (*x2)[KX][64];
    int s, lane;
    bool inside;
    // Build of the fused pass for three waves per SIMD: 2-D, up to three
    // species, states beyond the last-level cache (non-temporal stores).
    // Its marching and gradient sums then live in LDS; on cache-resident
    // lattices, where one tile's chain sets the step time, the register build
    // is faster.
    static constexpr bool kThree = Lat<LAT>::DIM == 2 && NS <= 3 && POL == kStoreNT;
    // FP64 gradient sums of this lane, in registers, or in 3-D and for kThree
    // in LDS.  Every wave holds the same dL/dK: the species-0 wave alone adds
    // it (acck: this lane's element of the work-group's [pairs][64] doubles);
    // dL/dg is each species' own (accl: of the wave's [D][64] doubles).
    static constexpr int NP = NS * (NS - 1) / 2;
    static constexpr bool kLdsSums = Lat<LAT>::DIM == 3 || kThree;
    double accr[kLdsSums ? 1 : D];
    double acckr[kLdsSums ? 1 : NP];
    double* accl;
    double* acck;
    __device__ __forceinline__ double& accg(int d) {
        if constexpr (kLdsSums)
            return accl[d * 64];
        else
            return accr[d];
    }
    __device__ __forceinline__ double& accp(int k) {
        if constexpr (kLdsSums)
            return acck[k * 64];
        else
            return acckr[k];
    }
    __device__ __forceinline__ void clear_sums() {
#pragma unroll
        for (int d = 0; d < D; ++d) accg(d) = 0.0;
        if (s == 0) {
#pragma unroll
            for (int k = 0; k < NP; ++k) accp(k) = 0.0;
        }
    }
    // 2-D, up to three species: the loads of a layer are issued before the
    // collision VJP of the layer before it, whose two exchanges hide their
    // latency (with four species the held values would cost the fused pass
    // its second wave per SIMD)
    static constexpr bool kAhead = Lat<LAT>::DIM == 2 && NS < 4 && !kThree;
    unsigned skip;   // kSolid on lanes beyond the lattice: their stores drop
    // kernel A alone: lam_f = T^T lam_s(t) from the stored adjoint
    __device__ __forceinline__ void operator()(float P0, float (&F)[Q], int, unsigned own) {
        using L = Lat<LAT>;
        // lam_f0 = lam_P0 - sum_a (w_a/w_0) lam_ga, lam_fa = lam_ga
        const Buf Lm = fresh(lam);
        float lt[Q];
        float l0 = ldb(Lm, 0, own);
#pragma unroll
        for (int a = 1; a < Q; ++a) {
            lt[a] = ldb(Lm, a, own);
            l0 = fmaf(-L::wr(a), lt[a], l0);
        }
        lt[0] = l0;
        reverse(P0, F, lt, own);
    }
    // fused reverse step: lam_f(t) given in population space (the transposed
    // stream of the later step's mu, computed by the caller)
    __device__ __forceinline__ void operator()(float P0, float (&F)[Q], float (&lt)[Q],
                                               unsigned own) {
        reverse(P0, F, lt, own);
    }
    // the collision VJP at f(t) = (P0, F) of lam_f = lt; lt becomes mu
    __device__ __forceinline__ void reverse(float P0, float (&F)[Q], float (&lt)[Q],
                                            unsigned own) {
        using L = Lat<LAT>;
        // own density and momentum (sum_a w_a = 1, sum_a c_a w_a = 0)
        float sf = 0.0f, jx = 0.0f, jy = 0.0f, jz = 0.0f;
#pragma unroll
        for (int a = 1; a < Q; ++a) {
            const float v = F[a];
            sf += v;
            if (L::cx(a) == 1) jx += v; else if (L::cx(a) == -1) jx -= v;
            if (L::cy(a) == 1) jy += v; else if (L::cy(a) == -1) jy -= v;
            if (L::cz(a) == 1) jz += v; else if (L::cz(a) == -1) jz -= v;
        }
        x1[s][0][lane] = fmaf(P0, L::inv_w0, sf);
        x1[s][1][lane] = jx;
        x1[s][2][lane] = jy;
        if constexpr (D == 3) x1[s][3][lane] = jz;
        __syncthreads();
        float rho[NS], jm[NS][3];
#pragma unroll
        for (int j = 0; j < NS; ++j) {
            rho[j] = x1[j][0][lane];
            jm[j][0] = x1[j][1][lane];
            jm[j][1] = x1[j][2][lane];
            jm[j][2] = D == 3 ? x1[j][D == 3 ? 3 : 0][lane] : 0.0f;
        }
        VjpFwd<NS> f;
        vjp_forward<NS, Lat<LAT>::DIM>(rho, jm, C, f);
        float dg[3] = {0.0f, 0.0f, 0.0f};
        {
            VjpPart<NS> part;
#pragma unroll
            for (int i = 0; i < NS; ++i) {
                if (i != s) continue;
                vjp_species<LAT, NS>(i, rho, f, C, lt, part, dg);
                int k = 0;
#pragma unroll
                for (int d = 0; d < D; ++d) {
                    x2[s][k++][lane] = part.dU[d];
                    x2[s][k++][lane] = part.due[d];
                    x2[s][k++][lane] = part.gV[d];
                }
                x2[s][k++][lane] = part.drho;
#pragma unroll
                for (int j = 0; j < NS; ++j)
                    if (j != i) x2[s][k++][lane] = part.dW[j];
            }
        }
        __syncthreads();
        VjpAcc<NS> A;
        vjp_zero<NS>(A);
#pragma unroll
        for (int v = 0; v < NS; ++v) {
            VjpPart<NS> part;
            int k = 0;
#pragma unroll
            for (int d = 0; d < D; ++d) {
                part.dU[d] = x2[v][k++][lane];
                part.due[d] = x2[v][k++][lane];
                part.gV[d] = x2[v][k++][lane];
            }
            part.drho = x2[v][k++][lane];
#pragma unroll
            for (int j = 0; j < NS; ++j)
                if (j != v) part.dW[j] = x2[v][k++][lane];
            vjp_add<NS, D>(v, rho, f, part, A);
        }
        float dK[NS][NS];
#pragma unroll
        for (int i = 0; i < NS; ++i)
#pragma unroll
            for (int j = 0; j < NS; ++j) dK[i][j] = 0.0f;
        vjp_mixture<NS, Lat<LAT>::DIM>(rho, f, C, A, dK);
#pragma unroll
        for (int i = 0; i < NS; ++i) {
            if (i != s) continue;
            vjp_finish<LAT, NS>(i, rho, f, C, A, lt, dg);
        }
        const Buf Mm = fresh(mu);
        const unsigned at = oadd(own, skip);
#pragma unroll
        for (int a = 0; a < Q; ++a) stb<POL>(Mm, a, at, lt[a]);
        if (inside) {
            if (s == 0) {
                int k = 0;
#pragma unroll
                for (int i = 0; i < NS; ++i)
#pragma unroll
                    for (int j = i + 1; j < NS; ++j, ++k) accp(k) += (double)dK[i][j];
            }
#pragma unroll
            for (int d = 0; d < D; ++d) accg(d) += (double)dg[d];
        }
    }
    // the wave's sums, for the block reduction
    __device__ __forceinline__ void sums(double (&out)[NG]) {
#pragma unroll
        for (int k = 0; k < NP; ++k) out[k] = 0.0;
        if (s == 0) {
#pragma unroll
            for (int k = 0; k < NP; ++k) out[k] = accp(k);
        }
#pragma unroll
        for (int d = 0; d < 3; ++d) out[NP + d] = d < D ? accg(d < D ? d : 0) : 0.0;
    }
};

template <int LAT, int NS, int POL, bool WAVE>
__global__ void __launch_bounds__(256) k_adj_collide(const float* __restrict__ fprev,
                                                     const float* __restrict__ lam,
                                                     float* __restrict__ mu,
                                                     const LatParams* __restrict__ lps,
                                                     const Tile* __restrict__ tiles, int bx,
                                                     double* __restrict__ gpart) {
    constexpr int DIM = Lat<LAT>::DIM;
    using Op = AdjSplitOp<LAT, NS, POL>;
    __shared__ float x1[NS][DIM + 1][64];
    __shared__ float x2[NS][Op::KX][64];
    __shared__ double gsum[Op::kLdsSums ? NS : 1][Op::kLdsSums ? DIM : 1][64];
    __shared__ double ksum[Op::kLdsSums ? Op::NP : 1][64];
    // 3-D: the march's partial sums of every wave
    __shared__ float msum[Lat<LAT>::DIM == 3 ? NS - 1 : 1][2 * kMarDirs<LAT>][64];
    const int lane = (int)threadIdx.x;
    const int s = __builtin_amdgcn_readfirstlane((int)threadIdx.y);
    const int tb = virtual_block((int)gridDim.x);
    const Tile T = tiles[tb];
    const LatParams& P = lps[0];   // (single-lattice contexts)
    int x, y;
    bool zero;
    const bool inside = tile_column<LAT>(T, P, lane, bx, x, y, zero);
    Op op{species_buf<LAT>(lam + P.base, P.plane, s), species_buf<LAT>(mu + P.base, P.plane, s),
          coll_const(P), x1, x2, s, lane, inside, {}, {}, &gsum[Op::kLdsSums ? s : 0][0][lane],
          &ksum[0][lane],
          inside ? 0u : kSolid};
    op.clear_sums();
    const GatherConst G = gather_const(P, DIM);
    const float L[3] = {P.lam[s][0], P.lam[s][1], P.lam[s][2]};
    march1<LAT, WAVE, DIM == 3, Op::kAhead>(species_buf<LAT>(fprev + P.base, P.plane, s), G, s, L,
                                            T.x0, x, y, zero, T.m0, T.m1, op,
                                            &msum[DIM == 3 && s > 0 ? s - 1 : 0][0][lane]);
    double sums[Op::NG];
    op.sums(sums);
    block_reduce_add<Op::NG>(sums, gpart + (int64_t)tb * Op::NG);
}

// ------------------------------------------------------------------ kernel B
// lam_f(t-1)(X) = sum_k Lambda_k(-e) mu(X + k) over fluid sources X + k (the
// pull gather with the velocity reversed: Lambda_{-k}(e) = Lambda_k(-e)),
// plus the transposed wall terms; species 1 (c = 1): mu_a(X + c_a), or
// mu_abar(X) where X + c_a is solid.  Stored as lam_s = T^-T lam_f:
// lam_P0 = lam_f0 + sum_a (w_a/w_0) lam_fa, lam_ga = lam_fa.
// The same march as the forward gather: one wave per species over a tile's
// columns, the cross-section passes read per layer (the wave form for 64-column
// rows), the pass along the marching axis carried in two partial sums per
// plane, so every value of mu is read about once.  Direction a reversed has
// the components of opp(a).

// Marching state of the reversed gather of one heavier species: the
// marching-axis partial sums of its planes of mu.
template <int LAT, bool LDS = false>
using RevMarch = MarchSums<LAT, LDS>;

// Start of the reversed march of a heavier species from hp(a, j), the
// cross-section pass of plane a in the layer before the first (j = 0) and in
// the first one (j = 1).
template <int LAT, bool RL, class HP>
__device__ __forceinline__ void rev_start(const float (&L)[3], HP hp, RevMarch<LAT, RL>& r) {
    using Fr = Frame<LAT>;
#pragma unroll
    for (int a = 1; a < Lat<LAT>::Q; ++a) {
        if (Fr::pm(a) != 0) {
            const W3 wmar = wsel(-Fr::pm(a), L);
            const float hm = hp(a, 0), h0 = hp(a, 1);
            r.set(0, a, fmaf(wmar.z, h0, wmar.m * hm));
            r.set(1, a, wmar.m * h0);
        }
    }
}

// One layer of it from hp(a), the cross-section pass of plane a in the next
// layer (directions with a marching component) or in this one.
template <int LAT, bool RL, class HP>
__device__ __forceinline__ void rev_combine(const float (&L)[3], HP hp, RevMarch<LAT, RL>& r,
                                            float (&lf)[Lat<LAT>::Q]) {
    using Fr = Frame<LAT>;
#pragma unroll
    for (int a = 1; a < Lat<LAT>::Q; ++a) {
        const float hv = hp(a);   // 0 beyond a wall
        if (Fr::pm(a) == 0) {
            lf[a] = hv;
        } else {
            const W3 wmar = wsel(-Fr::pm(a), L);
            const float a0 = r.get(0, a), a1 = r.get(1, a);
            lf[a] = fmaf(wmar.p, hv, a0);
            r.set(0, a, fmaf(wmar.z, hv, a1));
            r.set(1, a, wmar.m * hv);
        }
    }
}

// Transposed wall terms (walls on one axis) at a node next to a wall.
// Species 1: the bounce-back transpose, mu_abar(X) where X + c_a is solid.
// The others: the forward adds lambda_+1 f~_a(X) + lambda_-1 f~_abar(X) to
// f_a(X) for a pointing away from the wall.
template <int LAT>
__device__ __forceinline__ void rev_walls(const Buf& M, int s, const float (&L)[3], unsigned own,
                                          const Sides& sd, float (&lf)[Lat<LAT>::Q]) {
    using Fr = Frame<LAT>;
    using La = Lat<LAT>;
    float W[La::Q];
#pragma unroll
    for (int a = 1; a < La::Q; ++a) W[a] = ldb(M, a, own);
    int side[3] = {sd.s[0], sd.s[1], sd.s[2]};   // (kept in this branch, as in wall_returns)
    asm volatile("" : "+v"(side[0]), "+v"(side[1]), "+v"(side[2]));
#pragma unroll
    for (int a = 1; a < La::Q; ++a) {
        bool away = false, toward = false;
#pragma unroll
        for (int ax = 0; ax < La::DIM; ++ax) {
            const int c = Fr::comp(a, ax);
            if (c == 0) continue;
            away = away || side[ax] == -c;
            toward = toward || side[ax] == c;
        }
        if (s == 0) {
            lf[a] = toward ? W[La::opp(a)] : lf[a];
        } else {
            lf[a] = away ? fmaf(L[2], W[a], lf[a]) : lf[a];
            lf[a] = toward ? fmaf(L[0], W[La::opp(a)], lf[a]) : lf[a];
        }
    }
}

// The shifted read of species 1: mu_a(X + c_a); 0 where it is solid.
template <int LAT>
__device__ __forceinline__ unsigned rev_source(const Col& col, int a, unsigned lo, unsigned own,
                                               unsigned hi) {
    using Fr = Frame<LAT>;
    const int c0 = Fr::p0(a), c1 = Fr::p1(a), cm = Fr::pm(a);
    unsigned src = cm > 0 ? hi : (cm < 0 ? lo : own);
    if (c0 != 0) src = oadd(src, c0 > 0 ? col.bxp : col.bxm);
    if (c1 != 0) src = oadd(src, c1 > 0 ? col.byp : col.bym);
    return src;
}

// ---- reads, one column per thread
template <int LAT, bool RL>
__device__ __forceinline__ void rev_begin(const Buf& M, const GatherConst& G, const ColGeom& g,
                                          int s, const float (&L)[3], int m0,
                                          RevMarch<LAT, RL>& r) {
    using Fr = Frame<LAT>;
    using La = Lat<LAT>;
    if (s == 0) return;
    const unsigned c[2] = {layer_off(g, nbr(m0, -1, G.nm, g.wm)), layer_off(g, m0)};
    rev_start<LAT>(L, [&](int a, int j) {
        return hpass_load<LAT>(M, a, Fr::p0(La::opp(a)), Fr::p1(La::opp(a)), c[j], g.col, L);
    }, r);
}

template <int LAT, bool RL>
__device__ __forceinline__ void rev_layer(const Buf& M, const GatherConst& G, const ColGeom& g,
                                          int s, const float (&L)[3], int m, RevMarch<LAT, RL>& r,
                                          float (&lf)[Lat<LAT>::Q]) {
    using Fr = Frame<LAT>;
    using La = Lat<LAT>;
    const unsigned own = layer_off(g, m), nxt = layer_off(g, nbr(m, 1, G.nm, g.wm));
    lf[0] = ldb(M, 0, own);
    if (s == 0) {
        const unsigned lo = layer_off(g, nbr(m, -1, G.nm, g.wm));
#pragma unroll
        for (int a = 1; a < La::Q; ++a)
            lf[a] = ldb(M, a, rev_source<LAT>(g.col, a, lo, own, nxt));
    } else {
        rev_combine<LAT>(L, [&](int a) {
            return hpass_load<LAT>(M, a, Fr::p0(La::opp(a)), Fr::p1(La::opp(a)),
                                   Fr::pm(a) != 0 ? nxt : own, g.col, L);
        }, r, lf);
    }
    const Sides sd = wall_sides<LAT>(G, g, m);
    if (sd.any) rev_walls<LAT>(M, s, L, own, sd, lf);
}

// ---- the wave form
// Rows of one layer by their loads: rest, plane 0 at the node; dev(a, j), row j
// of plane a; shift(a), mu_a(X + c_a).
template <int LAT>
struct RevRows {
    const Buf& M;
    const Col& col;
    unsigned lo, own, nxt;
    __device__ __forceinline__ float rest() const { return ldb(M, 0, own); }
    __device__ __forceinline__ float dev(int a, int j) const {
        const unsigned c = Frame<LAT>::pm(a) != 0 ? nxt : own;
        return ldb(M, a, j == 0 ? c : oadd(c, j == 1 ? col.bym : col.byp));
    }
    __device__ __forceinline__ float shift(int a) const {
        return ldb(M, a, rev_source<LAT>(col, a, lo, own, nxt));
    }
};
// The same rows in registers (2-D).
template <int LAT>
struct RevRaw : WaveRaw<LAT, true> {
    __device__ __forceinline__ float rest() const { return this->v[0]; }
};

template <int LAT>
__device__ __forceinline__ void rev_load(const RevRows<LAT>& r, int s, RevRaw<LAT>& raw) {
    using S = Slots<LAT, true>;
    if (s == 0) {
#pragma unroll
        for (int a = 1; a < S::Q; ++a) raw.v[S::zbase + a - 1] = r.shift(a);
    } else {
#pragma unroll
        for (int a = 1; a < S::Q; ++a)
#pragma unroll
            for (int j = 0; j < S::rows(a); ++j) raw.v[S::z(a) + j] = r.dev(a, j);
    }
    raw.v[0] = r.rest();
}

template <int LAT, bool RL, class R, class H>
__device__ __forceinline__ void rev_begin_wave(int s, const float (&L)[3], const R& r, H hx,
                                               RevMarch<LAT, RL>& h) {
    using Fr = Frame<LAT>;
    using La = Lat<LAT>;
    using S = Slots<LAT, true>;
    if constexpr (!RL) {
#pragma unroll
        for (int a = 1; a < S::Q; ++a) {
            h.set(0, a, 0.0f);
            h.set(1, a, 0.0f);
        }
    }
    if (s == 0) return;
    rev_start<LAT>(L, [&](int a, int k) {
        return hpass_wave<LAT>(Fr::p0(La::opp(a)), Fr::p1(La::opp(a)),
                               [&](int j) { return r.dev(a, j, k); },
                               [&](int) { return hx.dev(a, k); }, L);
    }, h);
}

template <int LAT, bool RL, class R, class H>
__device__ __forceinline__ void rev_layer_wave(int s, const float (&L)[3], const R& r, H hx,
                                               RevMarch<LAT, RL>& h, float (&lf)[Lat<LAT>::Q]) {
    using Fr = Frame<LAT>;
    using La = Lat<LAT>;
    using S = Slots<LAT, true>;
    lf[0] = r.rest();
    if (s == 0) {
#pragma unroll
        for (int a = 1; a < S::Q; ++a) lf[a] = r.shift(a);
    } else {
        rev_combine<LAT>(L, [&](int a) {
            return hpass_wave<LAT>(Fr::p0(La::opp(a)), Fr::p1(La::opp(a)),
                                   [&](int j) { return r.dev(a, j); },
                                   [&](int j) { return hx.dev(a, j); }, L);
        }, h, lf);
    }
}

// The reversed march of one species in the wave form (PF: loads a layer ahead).
template <int LAT, bool HL, bool PF>
struct RevWave {
    using S = Slots<LAT, true>;
    const Buf& M;
    const GatherConst& G;
    const WaveGeom& w;
    int s;
    RevMarch<LAT, HL> r;
    HaloLane hl;
    HaloSel sel;
    RevRaw<LAT> raw;       // PF: the next layer's rows
    BeginRaw<LAT, true> rb;
    float hvb;
    __device__ __forceinline__ int lo(int m) const { return nbr(m, -1, G.nm, w.g.wm); }
    __device__ __forceinline__ int hi(int m) const { return nbr(m, 1, G.nm, w.g.wm); }
    __device__ __forceinline__ RevRows<LAT> rows(const Buf& Mm, int m) const {
        return RevRows<LAT>{Mm, w.g.col, layer_off(w.g, lo(m)), layer_off(w.g, m),
                            layer_off(w.g, hi(m))};
    }
    __device__ __forceinline__ float halos(const Buf& Mm, int m) const {
        return halo_load(Mm, hl, layer_base(w.g, m), layer_base(w.g, hi(m)));
    }
    __device__ __forceinline__ BeginRows<LAT> begin_rows(const Buf& Mm, int m0) const {
        return BeginRows<LAT>{Mm, w.g.col, layer_off(w.g, lo(m0)), layer_off(w.g, m0)};
    }
    __device__ __forceinline__ void begin_loads(int m0) {
        const Buf Mm = fresh(M);
        if constexpr (Lat<LAT>::DIM == 2) {
            hvb = 0.0f;
            if (s > 0)
                hvb = halo_first<true>(Mm, w, false, layer_base(w.g, lo(m0)), layer_base(w.g, m0),
                                       layer_base(w.g, hi(m0)));
            sel = HaloSel{w.sel, w.sel + 36, w.sel + 72};
            raw.hv = hvb;
            if constexpr (PF) {
                begin_load<LAT, true>(begin_rows(Mm, m0), s, rb);
                rev_load<LAT>(rows(Mm, m0), s, raw);
            }
        } else {
            hvb = 0.0f;
            if (s > 0)
                hvb = halo_load(Mm, halo_lane<LAT, true, true>(M, w, 2 * S::BH),
                                layer_base(w.g, lo(m0)), layer_base(w.g, m0));
            hl = halo_lane<LAT, true, false>(M, w, S::H);
        }
    }
    __device__ __forceinline__ void begin(const float (&L)[3], int m0) {
        if constexpr (Lat<LAT>::DIM == 2) {
            const HalosBatch<true, true> hx(sel, hvb);
            if constexpr (PF) {
                rev_begin_wave<LAT>(s, L, rb, hx, r);
            } else {
                const Buf Mm = fresh(M);
                rev_begin_wave<LAT>(s, L, begin_rows(Mm, m0), hx, r);
            }
        } else {
            const Buf Mm = fresh(M);
            rev_begin_wave<LAT>(s, L, begin_rows(Mm, m0), HalosRead<LAT, true, true>(hvb), r);
        }
    }
    __device__ __forceinline__ void next_lanes() {
        if constexpr (Lat<LAT>::DIM == 2) hl = halo_lane2<true>(M, w, false);
    }
    __device__ __forceinline__ void load(int m) {
        if constexpr (PF) {
            const Buf Mm = fresh(M);
            if (s > 0) raw.hv = halos(Mm, m);
            rev_load<LAT>(rows(Mm, m), s, raw);
        }
    }
    // lam_f of layer m, without walls
    __device__ __forceinline__ void layer(const float (&L)[3], int m, bool first,
                                          float (&lf)[Lat<LAT>::Q]) {
        if constexpr (Lat<LAT>::DIM == 2) {
            if constexpr (PF) {
                rev_layer_wave<LAT>(s, L, raw, HalosBatch<true, false>(sel, raw.hv), r, lf);
            } else {
                const Buf Mm = fresh(M);
                float hv = hvb;
                if (s > 0 && !first) hv = halos(Mm, m);
                RevRaw<LAT> q;
                rev_load<LAT>(rows(Mm, m), s, q);
                rev_layer_wave<LAT>(s, L, q, HalosBatch<true, false>(sel, hv), r, lf);
            }
            sel = HaloSel{w.sel, w.sel, w.sel};
        } else {
            const Buf Mm = fresh(M);
            const float hv = s > 0 ? halos(Mm, m) : 0.0f;
            rev_layer_wave<LAT>(s, L, rows(Mm, m), HalosRead<LAT, true, false>(hv), r, lf);
        }
    }
};

// Kernel B over one column: op(lam_f, own) per layer.
template <int LAT, class Op>
__device__ __forceinline__ void rev_march(const Buf& M, const GatherConst& G, int s,
                                          const float (&L)[3], const ColGeom& g, int m0, int m1,
                                          Op op) {
    RevMarch<LAT> r;
    rev_begin<LAT>(fresh(M), G, g, s, L, m0, r);
    for (int m = m0; m < m1; ++m) {
        float lf[Lat<LAT>::Q];
        rev_layer<LAT>(fresh(M), G, g, s, L, m, r, lf);
        op(lf, layer_off(g, m));
    }
}

template <int LAT, class Op>
__device__ __forceinline__ void rev_march_wave(const Buf& M, const GatherConst& G, int s,
                                               const float (&L)[3], const WaveGeom& w, int m0,
                                               int m1, Op op) {
    constexpr bool PF = Lat<LAT>::DIM == 2;
    RevWave<LAT, false, PF> rv{M, G, w, s};
    rv.begin_loads(m0);
    rv.begin(L, m0);
    if (m0 + 1 < m1) rv.next_lanes();
    for (int m = m0; m < m1; ++m) {
        float lf[Lat<LAT>::Q];
        rv.layer(L, m, m == m0, lf);
        const unsigned own = layer_off(w.g, m);
        const Sides sd = wall_sides<LAT>(G, w.g, m);
        if (sd.any) rev_walls<LAT>(fresh(M), s, L, own, sd, lf);
        if (PF && m + 1 < m1) rv.load(m + 1);
        op(lf, own);
    }
}

// The fused reverse step's march over one column: per layer the forward
// gather of f(t) from f~(t-1) (B: the species' view of the state) and the
// reversed gather of the later step's mu (M), then op(P0, F, lam_f, own).
// Both marches' partial sums in LDS in 3-D (20 floats per lane each; species
// 0, the exact shift, has none), which keeps the fused pass at three waves per
// SIMD (two with four species), and for Op::kThree.
template <int LAT, class Op>
__device__ __forceinline__ void march_fused(const Buf& B, const Buf& M, const GatherConst& G,
                                            int s, const float (&L)[3], const ColGeom& g, int m0,
                                            int m1, Op& op, float* macc) {
    constexpr int Q = Lat<LAT>::Q;
    constexpr bool HL = Lat<LAT>::DIM == 3 || Op::kThree;
    Heavy<LAT, HL> h;
    RevMarch<LAT, HL> r;
    if constexpr (HL) {
        h.acc = macc;
        r.acc = macc + 2 * kMarDirs<LAT> * 64;
    }
    if (s > 0) heavy_begin<LAT>(fresh(B), G, g, L, m0, h);
    rev_begin<LAT>(fresh(M), G, g, s, L, m0, r);
    for (int m = m0; m < m1; ++m) {
        const Buf Bm = fresh(B);
        const unsigned own = layer_off(g, m);
        const unsigned nxt = layer_off(g, nbr(m, 1, G.nm, g.wm));
        const Sides sd = wall_sides<LAT>(G, g, m);
        float P0, F[Q], lf[Q];
        if (s == 0) {
            shift_load<LAT>(Bm, g, own, layer_off(g, nbr(m, -1, G.nm, g.wm)), nxt, P0, F);
            if (sd.any) wall_returns<LAT, true>(Bm, G, L, own, sd, P0, F);
        } else {
            heavy_layer<LAT>(Bm, g, L, own, nxt, h, P0, F);
            if (sd.any) wall_returns<LAT, false>(Bm, G, L, own, sd, P0, F);
        }
        rev_layer<LAT>(fresh(M), G, g, s, L, m, r, lf);
        op(P0, F, lf, own);
    }
}

template <int LAT, class Op>
__device__ __forceinline__ void march_fused_wave(const Buf& B, const Buf& M, const GatherConst& G,
                                                 int s, const float (&L)[3], const WaveGeom& w,
                                                 int m0, int m1, Op& op, float* macc) {
    constexpr int Q = Lat<LAT>::Q;
    constexpr bool HL = Lat<LAT>::DIM == 3 || Op::kThree;
    constexpr bool PF = Op::kAhead;
    FwdWave<LAT, HL, PF> fw{B, G, w, s};
    RevWave<LAT, HL, PF> rv{M, G, w, s};
    if constexpr (HL) {
        fw.h.acc = macc;
        rv.r.acc = macc + 2 * kMarDirs<LAT> * 64;
    }
    fw.begin_loads(m0);
    rv.begin_loads(m0);
    fw.begin(L, m0);
    rv.begin(L, m0);
    if (m0 + 1 < m1) {
        fw.next_lanes();
        rv.next_lanes();
    }
    for (int m = m0; m < m1; ++m) {
        float P0, F[Q], lf[Q];
        fw.layer(L, m, m == m0, P0, F);
        rv.layer(L, m, m == m0, lf);
        const unsigned own = layer_off(w.g, m);
        const Sides sd = wall_sides<LAT>(G, w.g, m);
        if (sd.any) {
            if (s == 0)
                wall_returns<LAT, true>(fresh(B), G, L, own, sd, P0, F);
            else
                wall_returns<LAT, false>(fresh(B), G, L, own, sd, P0, F);
            rev_walls<LAT>(fresh(M), s, L, own, sd, lf);
        }
        if (PF && m + 1 < m1) {
            fw.load(m + 1);
            rv.load(m + 1);
        }
        op(P0, F, lf, own);
    }
}

template <int LAT, int NS, int POL, bool WAVE>
__global__ void __launch_bounds__(256) k_adj_stream(const float* __restrict__ mu,
                                                    float* __restrict__ lamout,
                                                    const LatParams* __restrict__ lps,
                                                    const Tile* __restrict__ tiles, int bx) {
    constexpr int DIM = Lat<LAT>::DIM;
    const int lane = (int)threadIdx.x;
    const int s = __builtin_amdgcn_readfirstlane((int)threadIdx.y);
    const int tb = virtual_block((int)gridDim.x);
    const Tile T = tiles[tb];
    const LatParams& P = lps[0];   // (single-lattice contexts)
    // lanes beyond the lattice run along (their neighbours across lanes are
    // the row's last columns) and store nothing
    int x, y;
    bool zero;
    const bool inside = tile_column<LAT>(T, P, lane, bx, x, y, zero);
    const GatherConst G = gather_const(P, DIM);
    const Buf M = species_buf<LAT>(mu + P.base, P.plane, s);
    const Buf O = species_buf<LAT>(lamout + P.base, P.plane, s);
    const float L[3] = {P.lam[s][0], P.lam[s][1], P.lam[s][2]};
    const unsigned skip = inside ? 0u : kSolid;
    auto store = [&](float (&lf)[Lat<LAT>::Q], unsigned own) {
        using La = Lat<LAT>;
        const Buf Om = fresh(O);
        const unsigned at = oadd(own, skip);
        float lp0 = lf[0];
#pragma unroll
        for (int a = 1; a < La::Q; ++a) {
            lp0 = fmaf(La::wr(a), lf[a], lp0);
            stb<POL>(Om, a, at, lf[a]);
        }
        stb<POL>(Om, 0, at, lp0);
    };
    if constexpr (WAVE) {
        rev_march_wave<LAT>(M, G, s, L, wave_geom<LAT>(G, T.x0, x, y, zero), T.m0, T.m1, store);
    } else {
        ColGeom g = col_geom<LAT>(G, x, y);
        if (zero) g.colbase += kSolid;
        rev_march<LAT>(M, G, s, L, g, T.m0, T.m1, store);
    }
}

// ------------------------------------------------------- fused reverse step
// Kernel B of step t+1 and kernel A of step t in one pass: lam_f(t) = S^T
// mu(t+1) is gathered from the later step's scratch mu (mu_in) where kernel A
// would read lam_s(t); the adjoint stays in population space between the two,
// so the storage transform and its inverse drop out, and mu(t) goes to mu_out.
// The parameter gradients accumulate as in kernel A.
// Its two gathers and the collision VJP keep the vector units busy half of the
// time (2048x1024 with three species 0.53 at 2.3 waves per SIMD, 128x96x64 0.47 at
// 2.2); the rest is latency at these few waves.  In 2-D, vector components beyond
// the lattice's dimensions are neither computed nor exchanged (2048x1024 with three
// species 228 -> 215 us per reverse step).  In 3-D, asked for three waves per SIMD,
// the build takes 158 VGPRs for two species and 168 for three (192 before), and a
// compute unit holds more work-groups: 128x96x64 with three species 235 -> 167 us
// per reverse step, tiles and their order included.  With three species it spills
// for that: 10 registers, 44 B of scratch a lane (7 and 32 B in blocks of 32 x 2).
// Four take 214 and are left at the two waves that is.  Each species hands on the
// 3 D + N values that the others' shares follow from, instead of D + 1 +
// (D + 2) N shares, which saves LDS and arithmetic on the sending side: 216 ->
// 211 and 166 -> 160 us.
template <int LAT, int NS, int POL, bool WAVE>
__global__ void __launch_bounds__(256)
    __attribute__((amdgpu_waves_per_eu(
        AdjSplitOp<LAT, NS, POL>::kThree || (Lat<LAT>::DIM == 3 && NS < 4) ? 3 : 1)))
    k_adj_fused(const float* __restrict__ fprev, const float* __restrict__ mu_in,
                float* __restrict__ mu_out, const LatParams* __restrict__ lps,
                const Tile* __restrict__ tiles, int bx, double* __restrict__ gpart) {
    constexpr int DIM = Lat<LAT>::DIM;
    using Op = AdjSplitOp<LAT, NS, POL>;
    __shared__ float x1[NS][DIM + 1][64];
    __shared__ float x2[NS][Op::KX][64];
    // the two marches' partial sums of every wave (3-D and the three-wave
    // build)
    constexpr bool HL = Lat<LAT>::DIM == 3 || Op::kThree;
    __shared__ float msum[HL ? NS - 1 : 1][HL ? 4 * kMarDirs<LAT> : 1][64];
    __shared__ double gsum[Op::kLdsSums ? NS : 1][Op::kLdsSums ? DIM : 1][64];
    __shared__ double ksum[Op::kLdsSums ? Op::NP : 1][64];
    const int lane = (int)threadIdx.x;
    const int s = __builtin_amdgcn_readfirstlane((int)threadIdx.y);
    // (species 0, the exact shift, keeps no marching state)
    float* macc = &msum[HL && s > 0 ? s - 1 : 0][0][lane];
    const int tb = virtual_block((int)gridDim.x);
    const Tile T = tiles[tb];
    const LatParams& P = lps[0];   // (single-lattice contexts)
    int x, y;
    bool zero;
    const bool inside = tile_column<LAT>(T, P, lane, bx, x, y, zero);
    const Buf M = species_buf<LAT>(mu_in + P.base, P.plane, s);
    // (the op's stored-adjoint view is not read on this path)
    Op op{M, species_buf<LAT>(mu_out + P.base, P.plane, s), coll_const(P), x1, x2, s, lane,
          inside, {}, {}, &gsum[Op::kLdsSums ? s : 0][0][lane],
          &ksum[0][lane], inside ? 0u : kSolid};
    op.clear_sums();
    const GatherConst G = gather_const(P, DIM);
    const float L[3] = {P.lam[s][0], P.lam[s][1], P.lam[s][2]};
    const Buf B = species_buf<LAT>(fprev + P.base, P.plane, s);
    if constexpr (WAVE) {
        march_fused_wave<LAT>(B, M, G, s, L, wave_geom<LAT>(G, T.x0, x, y, zero), T.m0, T.m1, op,
                              macc);
    } else {
        ColGeom g = col_geom<LAT>(G, x, y);
        if (zero) g.colbase += kSolid;
        march_fused<LAT>(B, M, G, s, L, g, T.m0, T.m1, op, macc);
    }
    double sums[Op::NG];
    op.sums(sums);
    block_reduce_add<Op::NG>(sums, gpart + (int64_t)tb * Op::NG);
}

// ----------------------------------------------------------------- init VJP
// f~(0) = C(f(0; g)), f_ia(0) = w_a rho_i (1 - e.g/(2 c_s^2)): the collision
// VJP at f(0) plus df(0)/dg.
template <int LAT, int NS>
__global__ void __launch_bounds__(256) k_adj_init(const LatParams* __restrict__ lps,
                                                  const double* __restrict__ x0,
                                                  const float* __restrict__ lam,
                                                  double* __restrict__ gpart) {
    using L = Lat<LAT>;
    constexpr int Q = L::Q;
    constexpr int NG = NS * (NS - 1) / 2 + 3;
    const LatParams& P = lps[0];
    const int64_t nodes = (int64_t)P.nx * P.ny * P.nz;
    const CollConst C = coll_const(P);
    SpanBuf Lb[NS];
#pragma unroll
    for (int s = 0; s < NS; ++s) Lb[s] = species_span<LAT>(lam + P.base, P.plane, s);
    double acc[NG];
#pragma unroll
    for (int q = 0; q < NG; ++q) acc[q] = 0.0;
    for (int64_t id = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; id < nodes;
         id += (int64_t)gridDim.x * blockDim.x) {
        const int x = (int)(id % P.nx);
        const int64_t r = id / P.nx;
        const int yy = (int)(r % P.ny);
        const int z = (int)(r / P.ny);
        const unsigned own = (unsigned)(((int64_t)z * P.ny + yy) * P.pitch + x) * 4u;
        float lt[NS][Q], rho[NS], jm[NS][3];
#pragma unroll
        for (int s = 0; s < NS; ++s) {
            rho[s] = (float)(x0[s * nodes + id] * (double)P.M[s] * (double)P.n0);
            const float c = C.c[s], ics = C.inv_cs2[s];
            jm[s][0] = jm[s][1] = jm[s][2] = 0.0f;
#pragma unroll
            for (int a = 1; a < Q; ++a) {
                const float eu = c * cdot<LAT>(a, -0.5f * C.g[0], -0.5f * C.g[1], -0.5f * C.g[2]);
                const float fa = L::w(a) * rho[s] * (1.0f + ics * eu);
                if (L::cx(a)) jm[s][0] += (float)L::cx(a) * fa;
                if (L::cy(a)) jm[s][1] += (float)L::cy(a) * fa;
                if (L::cz(a)) jm[s][2] += (float)L::cz(a) * fa;
            }
            float l0 = ldb(Lb[s], 0, own);
#pragma unroll
            for (int a = 1; a < Q; ++a) {
                lt[s][a] = ldb(Lb[s], a, own);
                l0 = fmaf(-L::wr(a), lt[s][a], l0);
            }
            lt[s][0] = l0;
        }
        float dK[NS][NS], dg[3] = {0.0f, 0.0f, 0.0f};
#pragma unroll
        for (int i = 0; i < NS; ++i)
#pragma unroll
            for (int j = 0; j < NS; ++j) dK[i][j] = 0.0f;
        collide_vjp<LAT, NS>(rho, jm, lt, C, dK, dg);
        // f_ia(0) depends on g through -e.g/(2 c_s^2)
#pragma unroll
        for (int s = 0; s < NS; ++s) {
            const float c = C.c[s], ics = C.inv_cs2[s];
#pragma unroll
            for (int a = 1; a < Q; ++a) {
                const float k = -0.5f * L::w(a) * rho[s] * ics * c * lt[s][a];
                dg[0] += k * L::cx(a);
                dg[1] += k * L::cy(a);
                dg[2] += k * L::cz(a);
            }
        }
        int k = 0;
#pragma unroll
        for (int i = 0; i < NS; ++i)
#pragma unroll
            for (int j = i + 1; j < NS; ++j) acc[k++] += (double)dK[i][j];
#pragma unroll
        for (int d = 0; d < 3; ++d) acc[k + d] += (double)dg[d];
    }
    block_reduce_add<NG>(acc, gpart + (int64_t)blockIdx.x * NG);
}

// ---------------------------------------------------------------- launchers
// Calls go(store policy, wave form) for a launch's tiles: the wave form where
// a tile is 64 columns of one row (always in 2-D).
template <int LAT, class Go>
static void by_build(const Launch& L, Go go) {
    auto pick = [&](auto wave) {
        if (L.wt)
            go(std::integral_constant<int, kStoreWT>{}, wave);
        else
            go(std::integral_constant<int, kStoreNT>{}, wave);
    };
    if constexpr (Lat<LAT>::DIM == 3) {
        if (L.bx != 64) return pick(std::false_type{});
    }
    pick(std::true_type{});
}

template <int LAT, int NS>
static hipError_t adj_t(const Launch& L, const float* lam_in, float* mu, double* gpart) {
    if (L.bx * L.by != 64) return hipErrorInvalidValue;
    auto go = [&](auto pol, auto wave) {
        hipLaunchKernelGGL((k_adj_collide<LAT, NS, decltype(pol)::value, decltype(wave)::value>), dim3(L.ntiles),
                           dim3(64, NS), 0, L.stream, L.src, lam_in, mu, L.lp, L.tiles, L.bx,
                           gpart);
    };
    by_build<LAT>(L, go);
    return hipGetLastError();
}

template <int LAT>
hipError_t launch_adjoint_lat(int ns, const Launch& L, const float* lam_in, float* mu, double* gpart) {
    if (ns == 2) return adj_t<LAT, 2>(L, lam_in, mu, gpart);
    if (ns == 3) return adj_t<LAT, 3>(L, lam_in, mu, gpart);
    if (ns == 4) return adj_t<LAT, 4>(L, lam_in, mu, gpart);
    return hipErrorInvalidValue;
}

template <int LAT, int NS>
static hipError_t adjf_t(const Launch& L, const float* mu_in, float* mu_out, double* gpart) {
    if (L.bx * L.by != 64) return hipErrorInvalidValue;
    auto go = [&](auto pol, auto wave) {
        hipLaunchKernelGGL((k_adj_fused<LAT, NS, decltype(pol)::value, decltype(wave)::value>), dim3(L.ntiles),
                           dim3(64, NS), 0, L.stream, L.src, mu_in, mu_out, L.lp, L.tiles, L.bx,
                           gpart);
    };
    by_build<LAT>(L, go);
    return hipGetLastError();
}

template <int LAT>
hipError_t launch_adjoint_fused_lat(int ns, const Launch& L, const float* mu_in, float* mu_out,
                                    double* gpart) {
    if (ns == 2) return adjf_t<LAT, 2>(L, mu_in, mu_out, gpart);
    if (ns == 3) return adjf_t<LAT, 3>(L, mu_in, mu_out, gpart);
    if (ns == 4) return adjf_t<LAT, 4>(L, mu_in, mu_out, gpart);
    return hipErrorInvalidValue;
}

template <int LAT, int NS>
static hipError_t adjs_t(const Launch& L, const float* mu, float* lam_out) {
    if (L.bx * L.by != 64) return hipErrorInvalidValue;
    auto go = [&](auto pol, auto wave) {
        hipLaunchKernelGGL((k_adj_stream<LAT, NS, decltype(pol)::value, decltype(wave)::value>), dim3(L.ntiles),
                           dim3(64, NS), 0, L.stream, mu, lam_out, L.lp, L.tiles, L.bx);
    };
    by_build<LAT>(L, go);
    return hipGetLastError();
}

template <int LAT>
hipError_t launch_adjoint_stream_lat(int ns, const Launch& L, const float* mu, float* lam_out) {
    if (ns == 2) return adjs_t<LAT, 2>(L, mu, lam_out);
    if (ns == 3) return adjs_t<LAT, 3>(L, mu, lam_out);
    if (ns == 4) return adjs_t<LAT, 4>(L, mu, lam_out);
    return hipErrorInvalidValue;
}

template <int LAT, int NS>
static hipError_t adji_t(const LatParams* lp, const LatParams& h, const double* x0,
                         const float* lam0, double* gpart, int nblocks, hipStream_t s) {
    hipLaunchKernelGGL((k_adj_init<LAT, NS>), dim3(nblocks), dim3(256), 0, s, lp, x0, lam0, gpart);
    return hipGetLastError();
}

template <int LAT>
hipError_t launch_adjoint_init_lat(int ns, const LatParams* lp, const LatParams& h, const double* x0,
                                   const float* lam0, double* gpart, int nblocks, hipStream_t s) {
    if (ns == 2) return adji_t<LAT, 2>(lp, h, x0, lam0, gpart, nblocks, s);
    if (ns == 3) return adji_t<LAT, 3>(lp, h, x0, lam0, gpart, nblocks, s);
    if (ns == 4) return adji_t<LAT, 4>(lp, h, x0, lam0, gpart, nblocks, s);
    return hipErrorInvalidValue;
}

}  // namespace lbmmc

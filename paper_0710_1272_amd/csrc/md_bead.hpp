// md_bead.hpp -- the bead kernel k_md (gfx950) and its launch.
//
// k_md: one workgroup per replica.  Depending on the mode it performs
//   step 1 of Sec. II (arXiv:0710.1272): nearest-grid-point interpolation of the fluid
//          velocity at every bead, u_i = j/rho of the pre-collision populations of the
//          node floor(r + 1/2) (pull-gathered from the current post-collision buffer);
//   step 2: M substeps h = 1/M with u_i frozen: harmonic bonds, WCA between non-bonded
//          beads, WCA on the distance to the nearest solid surface and to free-slip
//          faces, the pulling force in the pore (Sec. III), drag -m gamma (v - u_i) and
//          the random force A c (Philox4x32-10, A = sqrt(24 m gamma kT / h)),
//          integrated kick-drift; Fbar_i = mean of drag + random force;
//   epilogue: translocation count N_T, centre of mass (FP64), completion latch, and a
//          deterministic per-node sum of Fbar (one leader bead per node).
// Bead positions are accumulated in FP64 (they integrate ~10^5-10^6 small increments);
// velocities and forces use the lattice's arithmetic type.  Positions live in LDS.
#pragma once

#include <algorithm>

#include <climits>

#include "lbmd_lattice.hpp"

namespace lbmd {

template <int S>
struct MDReal {
    using type = float;
};
template <>
struct MDReal<LB_STORE_F64> {
    using type = double;
};

template <class Real>
struct MDKArgs {
    const Replica* reps;
    MDDev md;
    BeadPtrs<Real> b;
    const void* cur;
    RunState* st;
    const long long* step_at;  // the step counter this launch goes by
    // the counter the next step goes by (null: none that this launch sets), and whether the run
    // state's counter moves with this step
    long long* step_next;
    int last;
    // one-launch step: the buffer it writes, the marks of this and of the next step (null: none to
    // follow)
    void* dst;
    Marks now, next;
    int mode;
    int nmax;
    int list_in_lds;
    int noise_in_lds;  // random forces of all substeps tabulated in LDS at step start
};

// nearest node: floor(r + 1/2); periodic axes wrap, free-slip axes clamp (NaN -> 0)
__device__ __forceinline__ void ngp3(const int* n, const int* fs, const double* r, int* g) {
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        double t = floor(r[a] + 0.5);
        if (!(t >= -1e15 && t <= 1e15)) t = 0.0;  // non-finite
        if (fs[a]) {
            t = t < 0.0 ? 0.0 : (t > n[a] - 1 ? (double)(n[a] - 1) : t);
        } else {
            t = t - n[a] * floor(t / n[a]);
        }
        g[a] = (int)t;
    }
}

// The part of a replica's description the substep loop reads, copied into registers
// at kernel entry (before any store, so the copy is made with scalar loads).
struct Geom {
    int n[3];
    int fs[3];
    int n_walls;
    int wall[LB_MAX_WALLS][6];
};

__device__ __forceinline__ bool is_solid(const Geom& G, int x, int y, int z) {
    bool s = false;
#pragma unroll
    for (int k = 0; k < LB_MAX_WALLS; ++k) {
        if (k >= G.n_walls) break;
        const int* w = G.wall[k];
        const bool pore = pore_open(w) && y >= w[2] && y <= w[3] && z >= w[4] && z <= w[5];
        s = s || (x >= w[0] && x <= w[1] && !pore);
    }
    return s;
}

// A scalar the optimiser may not see through: what is computed from it is computed where it is
// used instead of being held in registers across the substep loop.
__device__ __forceinline__ int here(int v) {
    asm volatile("" : "+s"(v));
    return v;
}

__device__ __forceinline__ Geom load_geom(const Replica& R) {
    // every field is the same for the whole workgroup: keep it in scalar registers
    auto u = [](int v) { return __builtin_amdgcn_readfirstlane(v); };
    Geom g;
#pragma unroll
    for (int a = 0; a < 3; ++a) g.fs[a] = u(R.fs[a]);
    g.n[0] = u(R.nx);
    g.n[1] = u(R.ny);
    g.n[2] = u(R.nz);
    g.n_walls = u(R.n_walls);
#pragma unroll
    for (int k = 0; k < LB_MAX_WALLS; ++k)
#pragma unroll
        for (int m = 0; m < 6; ++m) g.wall[k][m] = u(R.wall[k][m]);
    return g;
}

// A wall's slab X0..X1 and pore prism Y0..Y1 x Z0..Z1 (solid node cubes span [i - 1/2, i + 1/2]).
// Its pore nodes are those with lo[a] <= floor(r + 1/2) <= hi on every axis, or lo[a] <= t < hi1[a]
// for t = r + 1/2; on a free-slip axis the node index is clamped into the box, so that a bound on a
// face of the box holds for every t (of a bead less than kNowhere away).  A wall without a pore has
// bounds that nothing meets.
struct WallBounds {
    double x0, x1, y0, y1, z0, z1;
    double lo[3], hi1[3];
};
struct WallInts {
    int side[6], lo[3], hi1[3];
};
__device__ __forceinline__ WallInts wall_ints(const Geom& G, const int* w) {
    const bool open = pore_open(w);
    WallInts I{{w[0], w[1], open ? w[2] : INT_MAX, w[3], w[4], w[5]}, {}, {}};
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        I.lo[a] = !open ? INT_MAX : w[2 * a] <= 0 ? INT_MIN : w[2 * a];
        I.hi1[a] = w[2 * a + 1] >= G.n[a] - 1 ? INT_MAX : w[2 * a + 1] + 1;
    }
    return I;
}
__device__ __forceinline__ WallBounds wall_bounds(const WallInts& I) {
    return {I.side[0] - 0.5, I.side[1] + 0.5, I.side[2] - 0.5, I.side[3] + 0.5, I.side[4] - 0.5, I.side[5] + 0.5,
            {(double)I.lo[0], (double)I.lo[1], (double)I.lo[2]}, {(double)I.hi1[0], (double)I.hi1[1], (double)I.hi1[2]}};
}

// A bead that is nowhere: a coordinate is not finite or, on a free-slip axis, absurdly far out.  The
// branch-free wall terms below hold for all others.
constexpr double kNowhere = 1e9;
template <bool PERIODIC>
__device__ __forceinline__ bool is_nowhere(const Geom& G, const double* r) {
    bool out = false;
#pragma unroll
    for (int a = 0; a < 3; ++a) out = out | !(fabs(r[a]) < (PERIODIC && !G.fs[a] ? HUGE_VAL : kNowhere));
    return out;
}

// Whether the nearest node floor(r + 1/2) of r is a node of wall w's pore; a periodic axis wraps
// the index as the node lookup does.  NOWHERE: r may be nowhere; a bound on a free-slip face of the
// box holds for it as for any other (the lookup clamps the index into the box).
template <bool PERIODIC, bool NOWHERE = false>
__device__ __forceinline__ bool wall_pore_node(const Geom& G, const WallBounds& B, const int* w, const double* r) {
    if (PERIODIC && !pore_open(w)) return false;
    bool in = true;
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        const double t = r[a] + 0.5;
        if (PERIODIC && !G.fs[a]) {
            double f = floor(t);
            if (!(f >= -1e9 && f <= 1e9)) f = 0.0;  // non-finite or absurd
            int k = (int)f % G.n[a];
            if (k < 0) k += G.n[a];
            in = in && k >= w[2 * a] && k <= w[2 * a + 1];
        } else {
            bool lo = t >= B.lo[a], hi = t < B.hi1[a];
            if constexpr (NOWHERE) {
                lo = lo | (w[2 * a] <= 0);
                hi = hi | (w[2 * a + 1] >= G.n[a] - 1);
            }
            in = in & lo & hi;
        }
    }
    return in;
}

// Squared distance from r to the nearest solid surface of a wall, and the vector from that
// surface point to r (xw: x wrapped into the box on a periodic axis).  Outside the prism (in
// y, z) the nearest solid point lies straight along x, on the slab; inside it, on the nearest
// of the four prism sides, at x clamped into the slab.  Ties go to the sides in the order
// y-low, y-high, z-low, z-high.  No branches: in the bead kernel the one wave with beads at the
// wall holds up all others at the substep's barrier.
// Its dependent FP64 operations are what counts: minima in place of compare and select, bounds that
// already hold what a missing pore or a face of the box means, and lane masks for the flags took the
// coupled step of 128x64x64 with 100 beads (FP32) from 50.4 to 48.7 us and 25 solvent-free steps of
// 16 chains of 32 beads from 1062 to 1007 us.
template <bool PERIODIC>
__device__ __forceinline__ double wall_dist2(const Geom& G, const WallBounds& B, const double* rin, double xw,
                                             double* dv) {
    double ry = rin[1], rz = rin[2];
    if (PERIODIC && !G.fs[1]) ry -= G.n[1] * floor((ry + 0.5) / G.n[1]);
    if (PERIODIC && !G.fs[2]) rz -= G.n[2] * floor((rz + 0.5) / G.n[2]);
    const double dx = fmin(xw - B.x0, fmax(xw - B.x1, 0.0));
    // distances to the four sides; all are >= 0 exactly when (ry, rz) lies in the prism
    const double yl = ry - B.y0, yh = B.y1 - ry, zl = rz - B.z0, zh = B.z1 - rz;
    const bool yhi = yh < yl, zhi = zh < zl;
    const double ys = fmin(yl, yh), zs = fmin(zl, zh);
    const bool on_z = zs < ys;
    const bool prism = fmin(ys, zs) >= 0.0;
    const double dy = (prism & !on_z) ? (yhi ? -ys : ys) : 0.0;
    const double dz = (prism & on_z) ? (zhi ? -zs : zs) : 0.0;
    dv[0] = dx;
    dv[1] = dy;
    dv[2] = dz;
    return sum_sq(dx, dy, dz);
}

// The nearest solid surface over the walls (squared distance and vector, as wall_dist2) and whether
// the nearest node is a pore node, for a bead that is nowhere; other beads keep what they have.  It is
// at a wall only if its x is within reach, is in no pore's cross-section, and of its place there only
// the slab's distance counts.
template <bool PERIODIC>
__device__ __forceinline__ void walls_of_nowhere(const Geom& G, const double* r, double xw, double reach,
                                                 double* best2, double* dvw, bool* pore) {
    if (!is_nowhere<PERIODIC>(G, r)) return;
    *best2 = HUGE_VAL;
    dvw[0] = dvw[1] = dvw[2] = 0.0;
    *pore = false;
#pragma unroll
    for (int w = 0; w < LB_MAX_WALLS; ++w) {
        if (w >= G.n_walls) break;
        int wl[6];  // (nothing of this rare path is to be held through the substep loop)
#pragma unroll
        for (int m = 0; m < 6; ++m) wl[m] = here(G.wall[w][m]);
        const WallBounds B = wall_bounds(wall_ints(G, wl));
        if (!(xw > B.x0 - reach && xw < B.x1 + reach)) continue;
        const double dx = xw - fmin(fmax(xw, B.x0), B.x1);
        if (dx * dx < *best2) {
            *best2 = dx * dx;
            dvw[0] = dx;
        }
        *pore = *pore || (pore_open(wl) && wall_pore_node<PERIODIC, true>(G, B, wl, r));
    }
}

// 1/x: the hardware reciprocal in FP32 (about 1 ulp), an exact division in FP64
template <class Real>
__device__ __forceinline__ Real fast_rcp(Real x) {
    if constexpr (sizeof(Real) == 4) return __builtin_amdgcn_rcpf(x);
    else return Real(1) / x;
}

// 1/sqrt(x): the hardware reciprocal square root in FP32 (about 1 ulp), sqrt and an
// exact division in FP64
template <class Real>
__device__ __forceinline__ Real fast_rsqrt(Real x) {
    if constexpr (sizeof(Real) == 4) return __builtin_amdgcn_rsqf(x);
    else return Real(1) / sqrt(x);
}

// -(1/r) dV/dr of WCA at squared distance r2 (0 beyond the cutoff)
template <class Real>
__device__ __forceinline__ Real wca_coef(Real r2, Real eps, Real sig2, Real rc2) {
    if (!(r2 < rc2)) return Real(0);
    const Real ir2 = fast_rcp<Real>(r2);
    const Real s2 = sig2 * ir2;
    const Real s6 = s2 * s2 * s2;
    return Real(24) * eps * (Real(2) * s6 * s6 - s6) * ir2;
}

// Issues the loads of the pre-collision populations of fluid node g (storage chosen at run
// time) without using a value, so that all 19 share one round trip: the stored elements as
// they are, zero-extended.
template <class Real, class Raw>
__device__ __forceinline__ void load_node(int storage, const Replica& R, const void* cur, const int* g, Raw* raw) {
    const PullMap map = make_pull_map(R, g[0], g[1], g[2]);
    long long off[Q];
    for_pops([&](auto P) {
        constexpr int p = decltype(P)::value;
        off[p] = R.pop_base + pull_element<p>(R, map);
    });
    if constexpr (sizeof(Real) == 8) {
#pragma unroll
        for (int p = 0; p < Q; ++p) raw[p] = ((const uint64_t*)cur)[off[p]];
    } else if (storage == LB_STORE_F32) {
#pragma unroll
        for (int p = 0; p < Q; ++p) raw[p] = ((const uint32_t*)cur)[off[p]];
    } else {
#pragma unroll
        for (int p = 0; p < Q; ++p) raw[p] = ((const uint16_t*)cur)[off[p]];
    }
}

template <int S, class Real, class Raw>
__device__ __forceinline__ void node_moments(Real rho0, const Raw* raw, Real* rho, Real* j) {
    using C = Codec<S>;
    Real m = 0, jx = 0, jy = 0, jz = 0;
    for_pops([&](auto P) {
        constexpr int p = decltype(P)::value;
        typename C::T e;
        if constexpr (sizeof(typename C::T) == 2) e = __builtin_bit_cast(typename C::T, (uint16_t)raw[p]);
        else e = __builtin_bit_cast(typename C::T, raw[p]);
        Real fp = (Real)C::template load<p>(e);
        if constexpr (C::deviation) fp += w_of<Real>(p) * rho0;
        m += fp;
        if constexpr (cx_of(p) != 0) jx += Real(cx_of(p)) * fp;
        if constexpr (cy_of(p) != 0) jy += Real(cy_of(p)) * fp;
        if constexpr (cz_of(p) != 0) jz += Real(cz_of(p)) * fp;
    });
    *rho = m;
    j[0] = jx;
    j[1] = jy;
    j[2] = jz;
}

// fluid velocity u = j / rho from the elements load_node fetched
template <class Real, class Raw>
__device__ __forceinline__ void node_velocity(int storage, Real rho0, const Raw* raw, Real* u) {
    Real rho = 1, j[3] = {0, 0, 0};
    if constexpr (sizeof(Real) == 8) {
        node_moments<LB_STORE_F64, Real>(rho0, raw, &rho, j);
    } else {
        switch (storage) {
            case LB_STORE_F32: node_moments<LB_STORE_F32, Real>(rho0, raw, &rho, j); break;
            case LB_STORE_F16DEV: node_moments<LB_STORE_F16DEV, Real>(rho0, raw, &rho, j); break;
            default: node_moments<LB_STORE_BF16DEV, Real>(rho0, raw, &rho, j); break;
        }
    }
    u[0] = j[0] / rho;
    u[1] = j[1] / rho;
    u[2] = j[2] / rho;
}

// The lattice update of one node from the elements load_node fetched, without the reaction:
// what the sweep would store there.
template <int S, class Raw>
__device__ __forceinline__ void update_node(const Replica& R, const Raw* raw, void* dst, int node,
                                            RunState* st) {
    using C = Codec<S>;
    typename C::R f[Q];
    for_pops([&](auto P) {
        constexpr int p = decltype(P)::value;
        if constexpr (sizeof(typename C::T) == 2) f[p] = C::load_raw(__builtin_bit_cast(typename C::T, (uint16_t)raw[p]));
        else f[p] = C::load_raw(__builtin_bit_cast(typename C::T, raw[p]));
    });
    relax_node<S, false>(R, f, node, st);
    store_node<S, false>(R, f, (typename C::T*)dst, node);
}

// S_p = -(w_p / c_s^2) F . c_p with c_s^2 = 1/3, added to the populations at base (stride PS)
template <int S>
__device__ __forceinline__ void add_reaction(typename Codec<S>::T* __restrict__ base, long long PS,
                                             const typename Codec<S>::R* F) {
    using C = Codec<S>;
    using Rl = typename C::R;
    auto source = [&](auto P) {
        constexpr int p = decltype(P)::value;
        Rl fc = 0;
        if constexpr (cx_of(p) != 0) fc += Rl(cx_of(p)) * F[0];
        if constexpr (cy_of(p) != 0) fc += Rl(cy_of(p)) * F[1];
        if constexpr (cz_of(p) != 0) fc += Rl(cz_of(p)) * F[2];
        return -Rl(3) * w_of<Rl>(p) * fc;
    };
    if constexpr (S == LB_STORE_F32 || S == LB_STORE_F64) {
        // full-precision storage: hardware float atomics without return (each node has one
        // leader, so no two threads add to one element and the result is deterministic)
        for_pops([&](auto P) {
            constexpr int p = decltype(P)::value;
            if constexpr (p != 0) (void)unsafeAtomicAdd(&base[(long long)p * PS], source(P));
        });
    } else {
        // 16-bit storage: decode, add, re-encode; all 18 moving populations are read
        // before any is written
        Rl f[Q];
        for_pops([&](auto P) {
            constexpr int p = decltype(P)::value;
            if constexpr (p != 0) f[p] = C::template load<p>(base[(long long)p * PS]);
        });
        for_pops([&](auto P) {
            constexpr int p = decltype(P)::value;
            if constexpr (p != 0) base[(long long)p * PS] = C::template store<p>(f[p] + source(P));
        });
    }
}

// One DPP lane exchange (no LDS round trip): quad_perm [1,0,3,2] swaps neighbouring lanes,
// [2,3,0,1] swaps lane pairs, row_half_mirror reverses each group of 8 lanes, row_mirror
// each row of 16.
constexpr int kDppSwap1 = 0xB1, kDppSwap2 = 0x4E, kDppHalfMirror = 0x141, kDppMirror = 0x140;
// rotations of the lanes within each row of 16
constexpr int kDppRor1 = 0x121, kDppRor2 = 0x122, kDppRor4 = 0x124, kDppRor8 = 0x128;

template <int CTRL>
__device__ __forceinline__ int dpp_i(int v) {
    return __builtin_amdgcn_update_dpp(0, v, CTRL, 0xF, 0xF, false);
}
template <int CTRL>
__device__ __forceinline__ float dpp_x(float v) {
    return __int_as_float(dpp_i<CTRL>(__float_as_int(v)));
}
template <int CTRL>
__device__ __forceinline__ double dpp_x(double v) {
    const long long b = __double_as_longlong(v);
    const int lo = dpp_i<CTRL>((int)(b & 0xFFFFFFFFll));
    const int hi = dpp_i<CTRL>((int)(b >> 32));
    return __longlong_as_double((long long)(((unsigned long long)(unsigned)hi << 32) | (unsigned)lo));
}
template <int CTRL>
__device__ __forceinline__ int dpp_x(int v) {
    return dpp_i<CTRL>(v);
}

// Sums of NV doubles over the block's first `threads` threads (whole waves; the others have left),
// valid in every one of them; scratch: 16 NV doubles.  The wave's
// butterfly (partners 32, 16, 8, 4, 2, 1 lanes away) takes the last four from lane rotations
// within rows of 16, which need no LDS round trip: after the first two exchanges every lane holds
// the sum of its class modulo 16, and rotating by 8, 4, 2, 1 reaches the other half class.
template <int NV>
__device__ __forceinline__ void block_sums(double* vals, double* scratch, int threads) {
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, nw = (threads + 63) >> 6;
#pragma unroll
    for (int k = 0; k < NV; ++k) vals[k] += __shfl_xor(vals[k], 32, 64);
#pragma unroll
    for (int k = 0; k < NV; ++k) vals[k] += __shfl_xor(vals[k], 16, 64);
#pragma unroll
    for (int k = 0; k < NV; ++k) {
        vals[k] += dpp_x<kDppRor8>(vals[k]);
        vals[k] += dpp_x<kDppRor4>(vals[k]);
        vals[k] += dpp_x<kDppRor2>(vals[k]);
        vals[k] += dpp_x<kDppRor1>(vals[k]);
        if (lane == 0) scratch[k * 16 + wave] = vals[k];
    }
    __syncthreads();
#pragma unroll
    for (int k = 0; k < NV; ++k) {
        double t = 0.0;
        for (int w = 0; w < nw; ++w) t += scratch[k * 16 + w];
        vals[k] = t;
    }
    __syncthreads();
}

// Sum over the G consecutive lanes of a group (G a power of two <= 64).  Each step adds
// the partial sum of the partner half, so every lane of the group ends with the same
// bits (a + b and b + a round alike): the redundant per-bead state of the group's
// lanes stays identical.
template <int G, class T>
__device__ __forceinline__ T group_sum(T v) {
    if constexpr (G >= 2) v += dpp_x<kDppSwap1>(v);
    if constexpr (G >= 4) v += dpp_x<kDppSwap2>(v);
    if constexpr (G >= 8) v += dpp_x<kDppHalfMirror>(v);
    if constexpr (G >= 16) v += dpp_x<kDppMirror>(v);
    if constexpr (G >= 32) v += __shfl_xor(v, 16, 64);
    if constexpr (G >= 64) v += __shfl_xor(v, 32, 64);
    return v;
}

// Pairwise separation r_i - r_j as FP32/FP64 components (minimum image on periodic
// axes) and its square.
template <class Real, bool PERIODIC>
__device__ __forceinline__ Real separation_v(const double* ri, const double* pj, const int* per,
                                             const double* nd, Real* d) {
    double dd[3] = {ri[0] - pj[0], ri[1] - pj[1], ri[2] - pj[2]};
    if constexpr (PERIODIC) {
#pragma unroll
        for (int c = 0; c < 3; ++c)
            // (within half a box there is nothing to subtract, and most waves need no division: 700
            // beads on two periodic axes, FP32, 157 us a step with it, 126 without)
            if (per[c] && !(fabs(dd[c]) * 2.01 < nd[c])) dd[c] -= nd[c] * floor(dd[c] / nd[c] + 0.5);
    }
    d[0] = (Real)dd[0];
    d[1] = (Real)dd[1];
    d[2] = (Real)dd[2];
    return sum_sq(d[0], d[1], d[2]);
}

// Angular term of Sec. II at the middle bead of (a, b, c): V = kappa phi^2 / 2 with phi
// the angle between the consecutive bonds d1 = r_b - r_a and d2 = r_c - r_b (0 for a
// straight chain).  With cos(phi) = d1.d2 / (|d1||d2|), the forces are
// f_a = -kappa (phi / sin phi) dcos/dd1, f_c = kappa (phi / sin phi) dcos/dd2, and the
// middle bead takes -(f_a + f_c); phi / sin phi -> 1 as phi -> 0.
template <class Real, bool PERIODIC>
__device__ __forceinline__ void angle_forces(const double* ra, const double* rb, const double* rc, const int* per,
                                             const double* nd, Real kappa, Real* fa, Real* fc) {
    Real d1[3], d2[3];
    const Real q1 = separation_v<Real, PERIODIC>(rb, ra, per, nd, d1);
    const Real q2 = separation_v<Real, PERIODIC>(rc, rb, per, nd, d2);
    const Real l1 = sqrt(q1), l2 = sqrt(q2);
    const Real dot = d1[0] * d2[0] + d1[1] * d2[1] + d1[2] * d2[2];
    const Real cx = d1[1] * d2[2] - d1[2] * d2[1], cy = d1[2] * d2[0] - d1[0] * d2[2],
               cz = d1[0] * d2[1] - d1[1] * d2[0];
    const Real cross = sqrt(cx * cx + cy * cy + cz * cz);
    const Real phi = atan2(cross, dot);
    const Real il12 = Real(1) / (l1 * l2);
    const Real sn = cross * il12;
    const Real small = sizeof(Real) == 4 ? Real(1e-4) : Real(1e-8);
    const Real phi_over_sin = sn > small ? phi / sn : Real(1) + phi * phi / Real(6);
    const Real c = dot * il12;
    const Real kk = kappa * phi_over_sin;
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        fa[a] = -kk * (d2[a] * il12 - c * d1[a] / q1);
        fc[a] = kk * (d1[a] * il12 - c * d2[a] / q2);
    }
}

// 1/b in FP64 to about an ulp: the hardware estimate and two Newton steps (an IEEE division is
// twice as many dependent instructions)
__device__ __forceinline__ double rcp64(double b) {
    double r = __builtin_amdgcn_rcp(b);
    r = __builtin_fma(__builtin_fma(-b, r, 1.0), r, r);
    return __builtin_fma(__builtin_fma(-b, r, 1.0), r, r);
}

// Whether any thread of the block (of its waves still running) passes need = true.  Two words, used in turn by successive
// votes (stamp counts them), so that nothing has to be cleared; between two votes on one word
// lies the barrier of the vote in between.
__device__ __forceinline__ bool block_vote(int* words, int stamp, bool need) {
    if (__ballot(need) != 0ull && (threadIdx.x & 63) == 0) words[stamp & 1] = ~stamp;
    __syncthreads();
    return __builtin_amdgcn_readfirstlane(words[stamp & 1]) == ~stamp;
}

// One tridiagonal system a_t x_{t-1} + b_t x_t + c_t x_{t+1} = d_t per workgroup, row t
// held by thread t (t < m), solved by parallel cyclic reduction: at stride s each row
// eliminates its couplings to rows t - s and t + s, so after ceil(log2 m) levels x_t = d_t / b_t.
// A level is a chain of one LDS round trip, a dozen dependent FP64 operations and a barrier, and
// a rigid chain's step is mostly such chains: rows are published as (a, 1/b, c, d), two 16-byte
// reads a neighbour; a row's coupling beyond either end is zero from the start and stays zero,
// so that the neighbour index is only clamped; and the new 1/b is a refined estimate, not a
// division.  The coupled step of 128x64x64 with a rigid chain of 100 beads (M = 5, FP32) fell from
// 99.6 to 77.4 us with it (before: one 8-byte array per coefficient, an IEEE division and a bounds
// test per neighbour and level).  W: [2][nmax][4] doubles, the two halves used in turn.  Every
// thread of the block must call it; it ends behind a barrier.
struct alignas(16) PcrRow {
    double a, ib, c, d;
};
__device__ __forceinline__ double pcr_solve(PcrRow* W, int nmax, int m, int t, double a, double b, double c, double d) {
    const bool row = t < m;
    double ib = rcp64(b);
    if (row) W[t] = PcrRow{a, ib, c, d};
    __syncthreads();
    int from = 0;
    for (int s = 1; s < m; s <<= 1) {
        if (row) {
            const PcrRow l = W[from + (t - s > 0 ? t - s : 0)];
            const PcrRow h = W[from + (t + s < m ? t + s : m - 1)];
            const double k1 = a * l.ib, k2 = c * h.ib;
            b = b - l.c * k1 - h.a * k2;
            d = d - l.d * k1 - h.d * k2;
            a = -l.a * k1;
            c = -h.c * k2;
            ib = rcp64(b);
            if (2 * s < m) W[nmax - from + t] = PcrRow{a, ib, c, d};
        }
        from = nmax - from;
        __syncthreads();
    }
    return row ? d * ib : 0.0;
}

// Verlet-list entries each lane keeps in registers (slot s of lane gl is entry gl + s G);
// entries beyond them are read from the list
// (fewer under the 1024-thread bound, where registers are scarcer)
template <int G, int BPT, int MAXT>
struct SlotsPerLane {
    // One lane a bead below the 1024-thread bound (257 to 512 beads): the substeps go by a shorter
    // inner list.  More lanes hold a bead's entries in their slots already; beyond 512 beads there
    // are no registers left for the second reference position.
    // Tight: the 1024-thread bound leaves a lane 128 registers, so that nothing is held through a
    // substep that can be had again where it is used (slot positions, wall bounds), and list entries
    // are taken in small rounds, their positions one at a time.  Held as below that bound, they
    // spilled: 700 beads (FP32 / FP64) 102 / 130 us a step, so 90 / 109; 1500 beads 243 / 353, so
    // 213 / 262; 2400 beads 410 / 669, so 355 / 515.
    static constexpr bool tight = MAXT > 512;
    static constexpr bool inner = G == 1 && BPT == 1 && MAXT <= 512;
    static constexpr int K = MAXT > 512 ? (BPT > 1 ? 1 : 2) : (BPT > 1 ? 4 : (G >= 8 ? 1 : inner ? 6 : 8 / G));
};
// Inner list: the entries of the Verlet list closer than rc + kInnerSkin, in the list's order, taken
// again when a bead has moved kInnerSkin / 2 since.  A lane runs through its entries one after the
// other and a wave through its longest lane: 8 to 13 list entries a bead are 3 to 5 inner ones.  The
// entries left out would add zeros, so the sums stay what they are.  400 beads (256x128x128, FP16):
// the bead kernel 86 -> 68 us, the step 119 -> 95.5.
constexpr int kInnerMax = 16;  // entries held; a bead with more goes by the Verlet list

// Verlet list of bead i (group of G lanes): every non-bonded bead closer than the list
// radius, in lane-then-index order.  Returns the count (may exceed the capacity).
template <class Real, int G, bool PERIODIC, bool TIGHT, class List>
__device__ __forceinline__ int build_list(int i, int n, bool bn, bool bp, const double* ri, const double* PB,
                                          const int* per, const double* nd, Real rl2, int gl, List list,
                                          int stride) {
    // U candidates a round: their positions are loaded together, so that a round and not a
    // candidate costs an LDS round trip
    constexpr int U = TIGHT ? 1 : G == 1 ? 8 : 4;
    auto scan = [&](auto&& hit_at) {
        int m = 0;
        for (int j0 = gl; j0 < n; j0 += U * G, m += U) {
            double pj[U][3];
#pragma unroll
            for (int t = 0; t < U; ++t) {
                const int j = j0 + t * G < n ? j0 + t * G : i;
#pragma unroll
                for (int c = 0; c < 3; ++c) pj[t][c] = PB[3 * j + c];
            }
#pragma unroll
            for (int t = 0; t < U; ++t) {
                const int j = j0 + t * G;
                Real d[3];
                const Real r2 = separation_v<Real, PERIODIC>(ri, pj[t], per, nd, d);
                const bool skip = j >= n || j == i || (j == i + 1 && bn) || (j == i - 1 && bp);
                if (!skip && r2 < rl2) hit_at(j, m + t);
            }
        }
    };
    if constexpr (G == 1) {
        // one lane per bead: append directly, keep counting past the capacity
        int total = 0;
        scan([&](int j, int) {
            if (total < kNeighbourMax) list[(size_t)total * stride] = (unsigned short)j;
            ++total;
        });
        return total;
    } else {
        // one pass: each lane marks its hits j = gl + m G in a mask of 64 W bits, then the
        // group places them by an exclusive prefix of counts.  m < n / G: at most
        // 512 / G^2 <= 128 for G >= 4 (lanes x beads <= 512) and 256 for G = 2 (up to 512
        // beads)
        constexpr int W = G == 2 ? 4 : 2;
        unsigned long long hit[W];
#pragma unroll
        for (int w = 0; w < W; ++w) hit[w] = 0ull;
        int mine = 0;
        scan([&](int, int m) {
            const unsigned long long bit = 1ull << (m & 63);
#pragma unroll
            for (int w = 0; w < W; ++w) hit[w] |= (m >> 6) == w ? bit : 0ull;
            ++mine;
        });
        int incl = mine;
#pragma unroll
        for (int off = 1; off < G; off <<= 1) {
            const int t = __shfl_up(incl, off, G);
            if (gl >= off) incl += t;
        }
        int pos = incl - mine;
        const int total = __shfl(incl, G - 1, G);
        if (total <= kNeighbourMax) {
#pragma unroll
            for (int w = 0; w < W; ++w) {
                unsigned long long h = hit[w];
                while (h) {
                    const int b = __builtin_ctzll(h);
                    h &= h - 1;
                    list[(size_t)(pos++) * stride] = (unsigned short)(gl + (64 * w + b) * G);
                }
            }
        }
        return total;
    }
}

// Each bead is owned by a group of G lanes that split its neighbour loop; every lane
// of the group keeps the bead's state, so the per-bead terms are computed redundantly
// without divergence.  BPT beads per group when there are more beads than groups
// (then G = 1).  WCA pairs come from a Verlet list (radius rc + skin), kept across LB
// steps and rebuilt whenever a bead has moved skin/2 since the last build, so the set
// of interacting pairs is exactly that of the all-pairs definition.
// Positions are double-buffered in LDS: one barrier per substep.  POLY compiles in the
// angular term and rigid bonds (the kernel without them is the harmonic-chain model).
// Every store of this wave has reached its XCD's L2 when this returns: after a barrier that
// follows it, other waves of the workgroup may update the same memory there.
__device__ __forceinline__ void stores_done() {
    __threadfence_block();
    __builtin_amdgcn_s_waitcnt(0);
}

// The kernel's first argument, read from the argument segment by a pointer that the optimiser
// cannot tie to the argument it already holds.
template <class Args>
__device__ __forceinline__ const Args& reread_args() {
    auto* p = (const char __attribute__((address_space(4)))*)__builtin_amdgcn_kernarg_segment_ptr();
    asm volatile("" : "+s"(p));
    return *(const Args*)(const char*)p;
}

// threads: the block's threads that take part (whole waves)
// OWN: the storage when the block also updates the nodes its beads sit on (one-launch step), else -1
template <class Real, int G, int BPT, bool PERIODIC, int MAXT, bool POLY, int OWN = -1>
__device__ __forceinline__ void bead_step(const MDKArgs<Real>& a, const int storage, const int rep, const int threads,
                                          double* lds) {
    constexpr bool own_nodes = OWN >= 0;
    __shared__ double red[16 * 4];
    const int NG = threads / G;  // groups
    const Replica& R = a.reps[rep];
    const Geom GM = load_geom(R);
    const uint32_t seed_lo = R.seed_lo, seed_hi = R.seed_hi;
    const double xmid = R.xmid;
    const long long pop_base = R.pop_base;
    const int plane = R.S;
    const int n = R.n_beads;
    const long long step = *a.step_at;
    if (rep == 0 && threadIdx.x == 0) {
        // the counters the next step and the next call go by (nothing of this step reads them)
        if (a.step_next) *a.step_next = step + 1;
        if (a.last) a.st->step = step + 1;
    }
    if (n == 0) return;
    const int b0 = R.bead0, NT = a.b.ntot, tid = threadIdx.x, nmax = a.nmax;
    const int grp = tid / G, gl = tid % G;
    double* P = lds;                                    // [2][nmax][3] positions
    int* NODE = (int*)(P + 6 * nmax);                   // [nmax]
    unsigned char* BN = (unsigned char*)(NODE + nmax);  // [nmax]
    // Verlet lists: [kNeighbourMax][nmax] in LDS when they fit, else global memory.  Up to 512 beads
    // two pointers into their own address spaces: an LDS read and a global one instead of one flat
    // one, into which the compiler would merge them (100 beads in 64x48x48, FP32: 38.4 -> 37.7 us a
    // step).  Beyond, where most lists are in global memory, the flat read is the faster one (1500
    // beads: 211 us, 219 with two pointers).
    constexpr bool kTight = SlotsPerLane<G, BPT, MAXT>::tight;
    typedef std::conditional_t<kTight, unsigned short, __attribute__((address_space(3))) unsigned short> LdsIndex;
    typedef std::conditional_t<kTight, unsigned short, __attribute__((address_space(1))) unsigned short> GlobalIndex;
    LdsIndex* LL = (LdsIndex*)(unsigned short*)(BN + nmax);
    GlobalIndex* GL = (GlobalIndex*)(a.b.nlist + b0);
    const bool list_lds = a.list_in_lds != 0;
    auto list_at = [&](int q, int i) -> int { return list_lds ? LL[q * nmax + i] : GL[(size_t)q * NT + i]; };
    // inner lists [kInnerMax][nmax] and random forces [M][nmax][3], after the lists (or after BN
    // when the lists are global)
    LdsIndex* IL = LL + (list_lds ? kNeighbourMax * nmax : 0);
    constexpr bool INNER = SlotsPerLane<G, BPT, MAXT>::inner;
    Real* NZ = (Real*)((unsigned short*)(BN + nmax) + (list_lds ? kNeighbourMax * nmax : 0) +
                       (INNER ? kInnerMax * nmax : 0));
    const bool noise_lds = G > 1 && a.noise_in_lds;
    const MDDev md = a.md;
    // rigid bonds: SHAKE/RATTLE work area after the random-force table, doubles:
    // reference bond vectors [3][nmax], multipliers [nmax], velocities [3][nmax], and
    // the cyclic-reduction buffers [2][4][nmax]
    double* RW = (double*)((unsigned char*)NZ +
                           (noise_lds ? (size_t)md.M * 3 * nmax * sizeof(Real) : (size_t)0));
    double* SDV = RW;
    double* LAM = RW + 3 * nmax;
    double* VXV = RW + 4 * nmax;
    PcrRow* PCRW = (PcrRow*)(RW + 7 * nmax);
    const int M = md.M;
    const int* nn = GM.n;
    const double nd[3] = {(double)GM.n[0], (double)GM.n[1], (double)GM.n[2]};
    const int per[3] = {GM.fs[0] ? 0 : 1, GM.fs[1] ? 0 : 1, GM.fs[2] ? 0 : 1};
    unsigned flags = 0;
    int cur = 0;  // offset of the current position buffer: 0 or 3 nmax

    double r[BPT][3];
    Real v[BPT][3], u[BPT][3], fb[BPT][3];
    int node[BPT];
    bool own[BPT];
    // One round trip for everything that the step's start positions do not decide: the bead
    // state and, with one bead per lane, the kept Verlet list (its length, the positions it
    // was built at, the first PF entries of each lane).  Whether the list is still valid is
    // known later; what was fetched in vain is dropped.
    double* dg = a.b.diag + 8 * rep;
    const double kept = dg[7];
    constexpr int PF = BPT == 1 ? (G == 1 ? 12 : (16 + G - 1) / G) : 1;
    double rref[BPT][3];
    int cnt[BPT];
    unsigned short pre_list[PF];
#pragma unroll
    for (int k = 0; k < BPT; ++k) {
        const int i = grp + k * NG;
        own[k] = i < n;
        node[k] = -1;
        cnt[k] = 0;
#pragma unroll
        for (int c = 0; c < 3; ++c) { r[k][c] = 0; v[k][c] = 0; u[k][c] = 0; fb[k][c] = 0; rref[k][c] = 0; }
        if (own[k]) {
            const int g = b0 + i;
#pragma unroll
            for (int c = 0; c < 3; ++c) r[k][c] = a.b.r[c * NT + g];
#pragma unroll
            for (int c = 0; c < 3; ++c) v[k][c] = a.b.v[c * NT + g];
            if constexpr (BPT == 1) {
#pragma unroll
                for (int c = 0; c < 3; ++c) rref[k][c] = a.b.rref[c * NT + g];
                cnt[k] = a.b.ncount[g];
                if (list_lds) {
#pragma unroll
                    for (int t = 0; t < PF; ++t)
                        pre_list[t] = gl + t * G < kNeighbourMax ? a.b.nlist[(size_t)(gl + t * G) * NT + g]
                                                                 : (unsigned short)0;
                }
            }
            if (!(a.mode & (MD_INTERP | MD_NO_HYDRO))) {
                node[k] = a.b.node[g];
#pragma unroll
                for (int c = 0; c < 3; ++c) u[k][c] = a.b.u[c * NT + g];
            }  // without hydrodynamics: u = 0 and no node (nothing is spread)
            if (gl == 0) {
                BN[i] = a.b.bond_next[g];
#pragma unroll
                for (int c = 0; c < 3; ++c) P[3 * i + c] = r[k][c];
            }
        }
    }

    // Rebuild vote: a wave whose beads moved too far in substep s stores ~s into word s & 1
    // (not s + 1: merged with the loop's own increment that would make the substep number
    // divergent in the compiler's eyes, and every decision of the loop a vector branch).
    // Two words, so that one barrier per substep separates the writes of a substep from its
    // reads and from the next writes to the same word; nothing has to be cleared.
    __shared__ int vote[2], inner_vote[2], block_votes[2];
    if (tid < 2) vote[tid] = inner_vote[tid] = block_votes[tid] = 0;
    int votes = 0;  // votes taken with block_vote
    if (a.mode & MD_SUBSTEPS) __syncthreads();

    // Verlet lists: kept from the previous launch (stored with the positions they were
    // built at) unless a bead has moved skin/2 since, else rebuilt before the first substep
    const Real rl2 = (Real)md.rl2, hs2 = (Real)md.half_skin2;
    // (kept in a scalar: every later decision of the whole workgroup then is a scalar branch)
    bool build = __builtin_amdgcn_readfirstlane(kept == 0.0 ? 1 : 0) != 0;
    if (!build && (a.mode & MD_SUBSTEPS)) {
        bool moved = false;
#pragma unroll
        for (int k = 0; k < BPT; ++k) {
            const int gi = b0 + grp + k * NG;
            if (!own[k]) continue;
            if constexpr (BPT > 1) {
#pragma unroll
                for (int c = 0; c < 3; ++c) rref[k][c] = a.b.rref[c * NT + gi];
                cnt[k] = a.b.ncount[gi];
            }
            const Real disp2 = sum_sq((Real)(r[k][0] - rref[k][0]), (Real)(r[k][1] - rref[k][1]),
                                      (Real)(r[k][2] - rref[k][2]));
            moved = moved | !(disp2 <= hs2);
        }
        // (a vote of the waves that take part: the library's workgroup reductions are for all
        // threads of the workgroup, and in the one-launch step some have left)
        build = block_vote(block_votes, votes++, moved);
        if (!build && list_lds) {
            // the kept list into LDS: what was fetched ahead, then 8 entries a lane per round trip
#pragma unroll
            for (int k = 0; k < BPT; ++k) {
                const int i = grp + k * NG;
                if (!own[k]) continue;
                const int m = cnt[k] < kNeighbourMax ? cnt[k] : kNeighbourMax;
                if constexpr (BPT == 1) {
#pragma unroll
                    for (int t = 0; t < PF; ++t)
                        if (gl + t * G < m) LL[i + (gl + t * G) * nmax] = pre_list[t];
                }
                constexpr int U = 8;
                for (int q0 = gl + (BPT == 1 ? PF * G : 0); q0 < m; q0 += U * G) {
                    unsigned short e[U];
#pragma unroll
                    for (int t = 0; t < U; ++t) {
                        const int q = q0 + t * G;
                        e[t] = q < m ? a.b.nlist[(size_t)q * NT + b0 + i] : (unsigned short)0;
                    }
#pragma unroll
                    for (int t = 0; t < U; ++t) {
                        const int q = q0 + t * G;
                        if (q < m) LL[i + q * nmax] = e[t];
                    }
                }
            }
        }
    }
    const Real A = (Real)md.A;
    auto tabulate_noise = [&]() {
        // the G lanes of a bead share its M Philox draws instead of each lane drawing all
        // of them; the table is read from the next barrier on
        if (!noise_lds) return;
#pragma unroll
        for (int k = 0; k < BPT; ++k) {
            const int i = grp + k * NG;
            if (!own[k]) continue;
            for (int s = gl; s < M; s += G) {
                const U4 rnd = philox4x32_10(U4{(uint32_t)i, (uint32_t)step, (uint32_t)s, 1u}, seed_lo, seed_hi);
                NZ[(s * nmax + i) * 3 + 0] = A * centred_uniform<Real>(rnd.x);
                NZ[(s * nmax + i) * 3 + 1] = A * centred_uniform<Real>(rnd.y);
                NZ[(s * nmax + i) * 3 + 2] = A * centred_uniform<Real>(rnd.z);
            }
        }
    };
    if (a.mode & MD_INTERP) {
        // the loads of all 19 populations of every bead's node are in flight while the random
        // forces are drawn
        using Raw = std::conditional_t<sizeof(Real) == 8, uint64_t, uint32_t>;
        Raw raw[BPT][Q];
        bool fluid[BPT];
#pragma unroll
        for (int k = 0; k < BPT; ++k) {
            int g[3];
            ngp3(GM.n, GM.fs, r[k], g);
            fluid[k] = own[k] && !is_solid(GM, g[0], g[1], g[2]);
            node[k] = fluid[k] ? g[0] + GM.n[0] * (g[1] + GM.n[1] * g[2]) : -1;
            if (fluid[k]) load_node<Real>(storage, R, a.cur, g, raw[k]);
        }
        if (a.mode & MD_SUBSTEPS) tabulate_noise();
#pragma unroll
        for (int k = 0; k < BPT; ++k) {
            const int i = grp + k * NG;
            if (fluid[k]) node_velocity<Real>(storage, (Real)R.rho0, raw[k], u[k]);
            if constexpr (own_nodes) {
                if (fluid[k] && gl == 0) update_node<OWN>(R, raw[k], a.dst, node[k], a.st);
            }
            if (own[k] && gl == 0) {
                const int gi = b0 + i;
                a.b.node[gi] = node[k];
#pragma unroll
                for (int c = 0; c < 3; ++c) a.b.u[c * NT + gi] = u[k][c];
            }
        }
    } else if (a.mode & MD_SUBSTEPS) {
        tabulate_noise();
    }
    if (!(a.mode & MD_SUBSTEPS)) return;
#pragma unroll
    for (int k = 0; k < BPT; ++k) {
        const int i = grp + k * NG;
        if (own[k] && gl == 0) NODE[i] = node[k];
    }

    const Real h = (Real)md.h, hm = (Real)(md.h * md.inv_mass), invM = (Real)md.inv_M;
    const Real mg = (Real)(md.mass * md.gamma);
    const Real kb = (Real)md.k_bond, r0 = (Real)md.r0;
    const Real eps24 = (Real)(24.0 * md.eps), sig2 = (Real)md.sigma2, rc2 = (Real)md.rc2;
    const Real epsw = (Real)md.eps_w, sigw2 = (Real)md.sigma_w2, rcw2 = (Real)md.rcw2;
    // beyond this distance from a face the face WCA term is zero (a margin over the cutoff
    // keeps the skipped terms zero under any rounding of the distance)
    const Real rcw_gate = (Real)(md.rcw + 1e-3);
    const Real fdrive = (Real)md.f_drive;
    __syncthreads();

    // chain neighbours (constant over the step) and the register slots of the lists
    bool bnk[BPT], bpk[BPT], bnn[BPT], bpp[BPT];  // bonded to i+1, i-1, and i+1 to i+2, i-1 to i-2
#pragma unroll
    for (int k = 0; k < BPT; ++k) {
        const int i = grp + k * NG;
        bnk[k] = own[k] && BN[i] != 0;
        bpk[k] = own[k] && i > 0 && BN[i - 1] != 0;
        bnn[k] = POLY && bnk[k] && BN[i + 1] != 0;
        bpp[k] = POLY && bpk[k] && i > 1 && BN[i - 2] != 0;
    }
    // rigid chains (at most 512 beads, one bond row per thread) only run with one bead per group
    const bool rigid = POLY && BPT == 1 && md.rigid != 0;
    const Real kappa = POLY ? (Real)md.kappa_phi : Real(0);
    constexpr int K = SlotsPerLane<G, BPT, MAXT>::K;
    int slot3[BPT][K], prev3[BPT], next3[BPT];  // three times the bead index
    bool used[BPT][K];
    bool shared[BPT], before[BPT];
    int builds = 0;
    // Beads within reach of a wall slab or a free-slip face.  Decided at each list build
    // with the margin skin/2: until the next build no bead moves farther than that, so a
    // bead outside these zones needs none of the wall, pore or face terms (all zero) and
    // cannot have left the box.
    const bool x_periodic = PERIODIC && !GM.fs[0];
    const double zone = md.zone;
    // What any bead of the wave is near, in one scalar: bit w of wall w, kFace of a face, and kLost if
    // one of the beads at a wall is nowhere (a bead that gets there forces a build).
    constexpr unsigned kWalls = (1u << LB_MAX_WALLS) - 1u, kFace = 1u << LB_MAX_WALLS, kLost = 2u << LB_MAX_WALLS;
    unsigned near[BPT];
    bool more[BPT];  // whether any bead of the wave has list entries beyond the register slots
    int cin[BPT];    // entries the substeps go through: of the inner list, or of the Verlet list
    bool half[BPT];  // inner list: whether any bead of the wave has entries in the slots' upper half
    double iref[BPT][3];  // where the inner list was taken
    const Real rin2 = (Real)md.rin2;
    const Real his2 = (Real)(0.25 * kInnerSkin * kInnerSkin);
    auto entry_at = [&](int q, int i, int k) -> int {
        if constexpr (INNER) return cin[k] <= kInnerMax ? (int)IL[q * nmax + i] : list_at(q, i);
        else return list_at(q, i);
    };
    WallBounds WB[LB_MAX_WALLS];
#pragma unroll
    for (int w = 0; w < LB_MAX_WALLS; ++w) WB[w] = wall_bounds(wall_ints(GM, GM.wall[w]));
#pragma unroll
    for (int k = 0; k < BPT; ++k) {
        const int i = own[k] ? grp + k * NG : 0;
        prev3[k] = 3 * (bpk[k] ? i - 1 : i);
        next3[k] = 3 * (bnk[k] ? i + 1 : i);
        near[k] = 0;
    }

    Real bond_max = 0;  // largest squared bond length met
    unsigned long long in_solid = 0, outside = 0;  // the wave's lanes
    for (int sub = 0; sub < M; ++sub) {
        const double* PB = P + cur;
        double* QB = P + (3 * nmax - cur);
        // the register slots of the Verlet list are read together with the rebuild vote of the
        // last substep; after a rebuild they are read again
        double pj[BPT][K][3];
        auto read_slots = [&](int k0, int k1) {
#pragma unroll
            for (int k = k0; k < k1; ++k)
#pragma unroll
                for (int s = 0; s < K; ++s) {
                    if (INNER && s == K / 2 && !half[k]) break;
#pragma unroll
                    for (int c = 0; c < 3; ++c) pj[k][s][c] = PB[slot3[k][s] + c];
                }
        };
        bool refresh = sub == 0;
        if (sub > 0) {
            const int voted = vote[(sub - 1) & 1];
            const int inner_voted = INNER ? inner_vote[(sub - 1) & 1] : 0;
            if (!kTight) read_slots(0, BPT);
            build = __builtin_amdgcn_readfirstlane(voted) == -sub;  // ~(sub - 1)
            if (INNER) refresh = __builtin_amdgcn_readfirstlane(inner_voted) == -sub;
        }
        if (build) {
            ++builds;
#pragma unroll
            for (int k = 0; k < BPT; ++k) {
                const int i = grp + k * NG;
                cnt[k] = 0;
#pragma unroll
                for (int c = 0; c < 3; ++c) rref[k][c] = r[k][c];
                if (!own[k]) continue;
                if (list_lds)
                    cnt[k] = build_list<Real, G, PERIODIC, kTight>(i, n, bnk[k], bpk[k], r[k], PB, per, nd, rl2, gl, LL + i,
                                                           nmax);
                else
                    cnt[k] = build_list<Real, G, PERIODIC, kTight>(i, n, bnk[k], bpk[k], r[k], PB, per, nd, rl2, gl, GL + i,
                                                           NT);
            }
            __syncthreads();
        }
        if (build || refresh) {
#pragma unroll
            for (int k = 0; k < BPT; ++k) {
                const int i = grp + k * NG;
                const double xw = x_periodic ? r[k][0] - nd[0] * floor((r[k][0] + 0.5) / nd[0]) : r[k][0];
                bool f_near = false;
                unsigned m = 0;
#pragma unroll
                for (int w = 0; w < LB_MAX_WALLS; ++w) {
                    if (w >= GM.n_walls) break;
                    if (__ballot(own[k] && xw > GM.wall[w][0] - 0.5 - zone && xw < GM.wall[w][1] + 0.5 + zone) != 0ull)
                        m |= 1u << w;
                }
                if (m != 0u && __ballot(own[k] && is_nowhere<PERIODIC>(GM, r[k])) != 0ull) m |= kLost;
#pragma unroll
                for (int c = 0; c < 3; ++c)
                    if (GM.fs[c]) f_near = f_near || !(r[k][c] + 0.5 >= zone && (nn[c] - 0.5) - r[k][c] >= zone);
                if (__ballot(own[k] && f_near) != 0ull) m |= kFace;
                near[k] = __builtin_amdgcn_readfirstlane(m);
                cin[k] = cnt[k];
                if constexpr (INNER) {
#pragma unroll
                    for (int c = 0; c < 3; ++c) iref[k][c] = r[k][c];
                    if (own[k] && cnt[k] <= kNeighbourMax) {
                        int m = 0;
                        constexpr int U = 4;
                        for (int q0 = 0; q0 < cnt[k]; q0 += U) {
                            int j[U];
                            double pq[U][3];
#pragma unroll
                            for (int t = 0; t < U; ++t) j[t] = q0 + t < cnt[k] ? list_at(q0 + t, i) : i;
#pragma unroll
                            for (int t = 0; t < U; ++t)
#pragma unroll
                                for (int c = 0; c < 3; ++c) pq[t][c] = PB[3 * j[t] + c];
#pragma unroll
                            for (int t = 0; t < U; ++t) {
                                Real d[3];
                                if (q0 + t < cnt[k] && separation_v<Real, PERIODIC>(r[k], pq[t], per, nd, d) < rin2) {
                                    if (m < kInnerMax) IL[m * nmax + i] = (unsigned short)j[t];
                                    ++m;
                                }
                            }
                        }
                        if (m <= kInnerMax) cin[k] = m;
                        // a bead with more entries goes by the Verlet list, which is longer still
                    }
                }
#pragma unroll
                for (int s = 0; s < K; ++s) {
                    const int q = gl + s * G;
                    used[k][s] = own[k] && cnt[k] <= kNeighbourMax && q < cin[k];
                    // an unused slot reads the bead itself
                    slot3[k][s] = 3 * (used[k][s] ? entry_at(q, i, k) : own[k] ? i : 0);
                }
                half[k] = __ballot(own[k] && cin[k] > K / 2 * G) != 0ull;
                more[k] = __ballot(own[k] && cin[k] > K * G) != 0ull;
            }
            if (!kTight) read_slots(0, BPT);
        }
        if (sub == 0) {
            // Flag whether a bead shares its node and whether a lower-index bead does (then it
            // is not the node's leader).  Beads on one node lie in its unit cell, at most
            // sqrt(3) apart: when the WCA cutoff rc covers that, they are bonded neighbours or
            // in this list (which holds every non-bonded pair closer than rc); otherwise every
            // bead's node is scanned.
#pragma unroll
            for (int k = 0; k < BPT; ++k) {
                const int i = grp + k * NG;
                int sh = 0, bf = 0;
                if (own[k] && node[k] >= 0) {
                    const bool all = cnt[k] > kNeighbourMax || md.node_scan_all;
                    const int lim = all ? n : cnt[k] + 2;
                    for (int q = gl; q < lim; q += G) {
                        int j;
                        if (all) j = q;
                        else if (q < cnt[k]) j = list_at(q, i);
                        else j = (q == cnt[k]) ? i - 1 : i + 1;
                        if (j < 0 || j >= n || j == i || NODE[j] != node[k]) continue;
                        sh = 1;
                        if (j < i) bf = 1;
                    }
                }
                shared[k] = group_sum<G>(sh) != 0;
                before[k] = group_sum<G>(bf) != 0;
            }
        }
        // Forces.  Lanes without a bead compute on bead 0's neighbourhood and drop the result,
        // and whole waves skip the surface terms together: the common path of a substep has no
        // divergent branch.
        Real F[BPT][3];
#pragma unroll
        for (int k = 0; k < BPT; ++k) {
            const int i = own[k] ? grp + k * NG : 0;
            double pm[3], pp[3];
#pragma unroll
            for (int c = 0; c < 3; ++c) pm[c] = PB[prev3[k] + c];
#pragma unroll
            for (int c = 0; c < 3; ++c) pp[c] = PB[next3[k] + c];
            Real noise[3];
            if (noise_lds) {
#pragma unroll
                for (int c = 0; c < 3; ++c) noise[c] = NZ[(sub * nmax + i) * 3 + c];
            } else {
                const U4 rnd = philox4x32_10(U4{(uint32_t)i, (uint32_t)step, (uint32_t)sub, 1u}, seed_lo, seed_hi);
                noise[0] = A * centred_uniform<Real>(rnd.x);
                noise[1] = A * centred_uniform<Real>(rnd.y);
                noise[2] = A * centred_uniform<Real>(rnd.z);
            }
            // WCA against the Verlet neighbours: register slots, then any further list
            // entries, or all pairs if the list overflowed
            Real fx = 0, fy = 0, fz = 0;
            // without branches: an unused slot or a pair beyond the cutoff adds 0 (times a separation
            // that is finite, as that of every bead a list holds)
            auto add_pair = [&](const Real* d, Real r2, bool hit) {
                const Real ir2 = fast_rcp<Real>(hit ? r2 : Real(1));
                const Real s2 = sig2 * ir2;
                const Real s6 = s2 * s2 * s2;
                const Real c = hit ? eps24 * (Real(2) * s6 * s6 - s6) * ir2 : Real(0);
                fx += c * d[0];
                fy += c * d[1];
                fz += c * d[2];
            };
            auto pair = [&](const double* p, bool valid) {
                Real d[3];
                const Real r2 = separation_v<Real, PERIODIC>(r[k], p, per, nd, d);
                add_pair(d, r2, valid & (r2 < rc2));
            };
            if (kTight) read_slots(k, k + 1);
#pragma unroll
            for (int s = 0; s < K; ++s) {
                if (INNER && s == K / 2 && !half[k]) break;
                pair(pj[k][s], used[k][s]);
            }
            if (more[k]) {
                // entries beyond the register slots, U a lane and round: a round, not an entry,
                // costs the LDS round trips (entry, position)
                constexpr int U = G == 1 && !(kTight && BPT == 1) ? 4 : 2;
                const bool overflow = own[k] && cnt[k] > kNeighbourMax;
                const int lim = own[k] && !overflow ? cin[k] : 0;
                for (int q0 = gl + K * G; q0 < lim; q0 += U * G) {
                    int j[U];
                    bool ok[U];
#pragma unroll
                    for (int t = 0; t < U; ++t) {
                        const int q = q0 + t * G;
                        ok[t] = q < lim;
                        if constexpr (kTight) j[t] = ok[t] ? entry_at(q, i, k) : i;
                        else j[t] = entry_at(ok[t] ? q : q0, i, k);
                    }
                    if constexpr (kTight) {
                        // one position at a time, and a wave without a pair within the cutoff skips the rest
#pragma unroll
                        for (int t = 0; t < U; ++t) {
                            if (t > 0 && __ballot(ok[t]) == 0ull) break;
                            const double pq[3] = {PB[3 * j[t]], PB[3 * j[t] + 1], PB[3 * j[t] + 2]};
                            Real d[3];
                            const Real r2 = separation_v<Real, PERIODIC>(r[k], pq, per, nd, d);
                            const bool hit = ok[t] & (r2 < rc2);
                            if (__ballot(hit) != 0ull) add_pair(d, r2, hit);
                        }
                    } else {
                        double pq[U][3];
#pragma unroll
                        for (int t = 0; t < U; ++t)
#pragma unroll
                            for (int c = 0; c < 3; ++c) pq[t][c] = PB[3 * j[t] + c];
#pragma unroll
                        for (int t = 0; t < U; ++t) pair(pq[t], ok[t]);
                    }
                }
                // A list that overflowed: all beads, one after the other.  Among them are beads whose
                // position is not finite, which no list holds: only a pair within the cutoff is added.
                for (int q = gl; q < (overflow ? n : 0); q += G) {
                    if (q == i || (q == i + 1 && bnk[k]) || (q == i - 1 && bpk[k])) continue;
                    const double pq[3] = {PB[3 * q], PB[3 * q + 1], PB[3 * q + 2]};
                    Real d[3];
                    const Real r2 = separation_v<Real, PERIODIC>(r[k], pq, per, nd, d);
                    if (r2 < rc2) add_pair(d, r2, true);
                }
            }
            F[k][0] = group_sum<G>(fx);
            F[k][1] = group_sum<G>(fy);
            F[k][2] = group_sum<G>(fz);
            // harmonic bonds to the chain neighbours, -k (len - r0)/len d = -k (1 - r0/len) d
            // (d points from j to i: the bond pulls i towards j when stretched); an
            // absent neighbour is the bead itself and adds 0
            if (!rigid) {
#pragma unroll
                for (int side = 0; side < 2; ++side) {
                    const bool on = side == 0 ? bpk[k] : bnk[k];
                    Real d[3];
                    const Real b2 = separation_v<Real, PERIODIC>(r[k], side == 0 ? pm : pp, per, nd, d);
                    bond_max = (on & (b2 > bond_max)) ? b2 : bond_max;
                    const Real coef = on ? -kb * (Real(1) - r0 * fast_rsqrt<Real>(b2)) : Real(0);
#pragma unroll
                    for (int c = 0; c < 3; ++c) F[k][c] += coef * d[c];
                }
            }
            // angular terms centred on i - 1, i and i + 1 (each needs both of its bonds)
            if (POLY && kappa != Real(0) && (bpk[k] || bnk[k])) {
                const int jmm = bpp[k] ? i - 2 : i, jpp = bnn[k] ? i + 2 : i;
                const double pmm[3] = {PB[3 * jmm], PB[3 * jmm + 1], PB[3 * jmm + 2]};
                const double ppp[3] = {PB[3 * jpp], PB[3 * jpp + 1], PB[3 * jpp + 2]};
                Real fa[3], fc[3];
                if (bpk[k] && bnk[k]) {
                    angle_forces<Real, PERIODIC>(pm, r[k], pp, per, nd, kappa, fa, fc);
#pragma unroll
                    for (int c = 0; c < 3; ++c) F[k][c] -= fa[c] + fc[c];
                }
                if (bpp[k]) {
                    angle_forces<Real, PERIODIC>(pmm, pm, r[k], per, nd, kappa, fa, fc);
#pragma unroll
                    for (int c = 0; c < 3; ++c) F[k][c] += fc[c];
                }
                if (bnn[k]) {
                    angle_forces<Real, PERIODIC>(r[k], pp, ppp, per, nd, kappa, fa, fc);
#pragma unroll
                    for (int c = 0; c < 3; ++c) F[k][c] += fa[c];
                }
            }
            // a non-finite coordinate stays non-finite: looked at once
            if (sub == M - 1 && own[k] && !(isfinite(r[k][0]) && isfinite(r[k][1]) && isfinite(r[k][2])))
                flags |= LB_ERR_NONFINITE;
            // nearest solid surface over the walls (min, earlier wall on ties) and the pore
            // drive (a bead whose nearest node is a pore node lies within half a node of its
            // wall's slab, so inside the zone); beyond the zone both are zero
            if (near[k] & kWalls) {
                const double xw = x_periodic ? r[k][0] - nd[0] * floor((r[k][0] + 0.5) / nd[0]) : r[k][0];
                double best2 = HUGE_VAL, dvw[3] = {0.0, 0.0, 0.0};
                bool pore = false;
#pragma unroll
                for (int w = 0; w < LB_MAX_WALLS; ++w) {
                    if (!(near[k] >> w & 1u)) continue;
                    double dv[3];
                    // (held through a polymer model's loop, the bounds would push its constraint
                    // solve out of the registers)
                    WallBounds B = WB[w];
                    if (POLY || kTight) {
                        int wl[6];
#pragma unroll
                        for (int m = 0; m < 6; ++m) wl[m] = here(GM.wall[w][m]);
                        B = wall_bounds(wall_ints(GM, wl));
                    }
                    const double q = wall_dist2<PERIODIC>(GM, B, r[k], xw, dv);
                    const bool closer = w == 0 || q < best2;
                    best2 = closer ? q : best2;
#pragma unroll
                    for (int c = 0; c < 3; ++c) dvw[c] = closer ? dv[c] : dvw[c];
                    pore = pore | wall_pore_node<PERIODIC>(GM, B, GM.wall[w], r[k]);
                }
                if (__builtin_expect((near[k] & kLost) != 0u, 0))
                    walls_of_nowhere<PERIODIC>(GM, r[k], xw, md.rcw, &best2, dvw, &pore);
                in_solid |= __ballot(own[k] & (best2 == 0.0));
                const bool hit = (best2 < (double)rcw2) & (best2 > 0.0);
                const Real c = wca_coef<Real>(hit ? (Real)best2 : rcw2, epsw, sigw2, rcw2);
#pragma unroll
                for (int q = 0; q < 3; ++q) F[k][q] += c * (Real)dvw[q];
                F[k][0] += pore ? fdrive : Real(0);
            }
            // free-slip faces at -1/2 and n - 1/2 (the WCA terms only within the cutoff)
            if (near[k] & kFace) {
                // (without PERIODIC every axis has faces)
                Real dlo[3], dhi[3], least = rcw_gate;
#pragma unroll
                for (int c = 0; c < 3; ++c) {
                    dlo[c] = (Real)(r[k][c] + 0.5);
                    dhi[c] = (Real)((nn[c] - 0.5) - r[k][c]);
                    if (PERIODIC && !GM.fs[c]) continue;
                    outside |= __ballot(own[k] & (!(dlo[c] > Real(0)) | !(dhi[c] > Real(0))));
                    least = fmin(least, fmin(dlo[c], dhi[c]));
                }
                const bool close = least < rcw_gate;
                if (own[k] & close) {
#pragma unroll
                    for (int c = 0; c < 3; ++c) {
                        if ((PERIODIC && !GM.fs[c]) || !(dlo[c] > Real(0)) || !(dhi[c] > Real(0))) continue;
                        F[k][c] += wca_coef<Real>(dlo[c] * dlo[c], epsw, sigw2, rcw2) * dlo[c];
                        F[k][c] -= wca_coef<Real>(dhi[c] * dhi[c], epsw, sigw2, rcw2) * dhi[c];
                    }
                }
            }
            // drag against the frozen fluid velocity and the random force
#pragma unroll
            for (int c = 0; c < 3; ++c) {
                const Real drag = -mg * (v[k][c] - u[k][c]);
                F[k][c] += drag + noise[c];
                fb[k][c] += (drag + noise[c]) * invM;
            }
        }
        // kick-drift into the other position buffer; the single barrier below both
        // publishes the new positions and collects the rebuild vote
#pragma unroll
        for (int k = 0; k < BPT; ++k) {
            const int i = grp + k * NG;
#pragma unroll
            for (int c = 0; c < 3; ++c) {
                v[k][c] += hm * F[k][c];
                r[k][c] += (double)(h * v[k][c]);
            }
            if (own[k] && gl == 0) {
#pragma unroll
                for (int c = 0; c < 3; ++c) QB[3 * i + c] = r[k][c];
            }
        }
        if (POLY && rigid) {
            // SHAKE and RATTLE on the unconstrained positions now in QB (PB still holds
            // the positions of the start of the substep); row t of the bond systems is
            // thread t, bond t joining beads t and t + 1
            __syncthreads();
            const int m = n - 1, t = tid;
            const bool on = t < m && BN[t] != 0;
            const double ih = 1.0 / md.h, im = md.inv_mass;
            double dref[3] = {0.0, 0.0, 0.0}, ut[3] = {0.0, 0.0, 0.0}, ut1[3] = {0.0, 0.0, 0.0};
            if (on) {
                const double pa[3] = {PB[3 * t], PB[3 * t + 1], PB[3 * t + 2]};
                const double pb[3] = {PB[3 * t + 3], PB[3 * t + 4], PB[3 * t + 5]};
                (void)separation_v<double, PERIODIC>(pa, pb, per, nd, dref);
#pragma unroll
                for (int c = 0; c < 3; ++c) {
                    ut[c] = QB[3 * t + c];
                    ut1[c] = QB[3 * t + 3 + c];
                }
            }
            if (t < nmax) {
#pragma unroll
                for (int c = 0; c < 3; ++c) SDV[c * nmax + t] = dref[c];
                LAM[t] = 0.0;
            }
            __syncthreads();
            // Newton iterations on the multipliers: positions r'_i = u_i + (lam_i d_i -
            // lam_{i-1} d_{i-1})/m, residuals g_t = |r'_t - r'_{t+1}|^2 - b^2
            double dm1[3] = {0.0, 0.0, 0.0}, dp1[3] = {0.0, 0.0, 0.0};
            if (on) {
#pragma unroll
                for (int c = 0; c < 3; ++c) {
                    dm1[c] = t > 0 ? SDV[c * nmax + t - 1] : 0.0;
                    dp1[c] = t + 1 < m ? SDV[c * nmax + t + 1] : 0.0;
                }
            }
            for (int it = 0;; ++it) {
                double sv[3] = {0.0, 0.0, 0.0}, g = 0.0;
                if (on) {
                    const double lm = t > 0 ? LAM[t - 1] : 0.0, l0 = LAM[t], lp = t + 1 < m ? LAM[t + 1] : 0.0;
                    double ra[3], rb[3];
#pragma unroll
                    for (int c = 0; c < 3; ++c) {
                        ra[c] = ut[c] + im * (l0 * dref[c] - lm * dm1[c]);
                        rb[c] = ut1[c] + im * (lp * dp1[c] - l0 * dref[c]);
                    }
                    g = (double)separation_v<double, PERIODIC>(ra, rb, per, nd, sv) - md.b2;
                }
                const bool bad = on && !(fabs(g) <= md.shake_tol_b2);
                const double B = on ? 4.0 * im * (sv[0] * dref[0] + sv[1] * dref[1] + sv[2] * dref[2]) : 1.0;
                const double Aa = on ? -2.0 * im * (sv[0] * dm1[0] + sv[1] * dm1[1] + sv[2] * dm1[2]) : 0.0;
                const double Cc = on ? -2.0 * im * (sv[0] * dp1[0] + sv[1] * dp1[1] + sv[2] * dp1[2]) : 0.0;
                const bool any_bad = block_vote(block_votes, votes++, bad);
                if (!any_bad) break;
                if (it >= md.shake_iter) {
                    flags |= LB_ERR_CONSTRAINT;
                    break;
                }
                const double x = pcr_solve(PCRW, nmax, m, t, Aa, B, Cc, on ? -g : 0.0);
                if (on) LAM[t] += x;
                __syncthreads();
            }
            // constrained positions and velocities (v = (r' - r) / h) of every bead
#pragma unroll
            for (int k = 0; k < BPT; ++k) {
                const int i = grp + k * NG;
                if (!own[k]) continue;
                const double li = bnk[k] ? LAM[i] : 0.0, lm = bpk[k] ? LAM[i - 1] : 0.0;
                const double r_old[3] = {PB[3 * i], PB[3 * i + 1], PB[3 * i + 2]};
#pragma unroll
                for (int c = 0; c < 3; ++c) {
                    const double di = bnk[k] ? SDV[c * nmax + i] : 0.0, dmi = bpk[k] ? SDV[c * nmax + i - 1] : 0.0;
                    r[k][c] += im * (li * di - lm * dmi);
                    v[k][c] = (Real)((r[k][c] - r_old[c]) * ih);
                }
            }
            __syncthreads();  // every read of the multipliers and of QB is done
#pragma unroll
            for (int k = 0; k < BPT; ++k) {
                const int i = grp + k * NG;
                if (!own[k] || gl != 0) continue;
#pragma unroll
                for (int c = 0; c < 3; ++c) {
                    QB[3 * i + c] = r[k][c];
                    VXV[c * nmax + i] = (double)v[k][c];
                }
            }
            __syncthreads();
            // RATTLE: (v'_t - v'_{t+1}) . s_t = 0 with v'_i = v_i + (mu_i s_i - mu_{i-1} s_{i-1})/m
            {
                double st[3] = {0.0, 0.0, 0.0}, sm[3] = {0.0, 0.0, 0.0}, sp[3] = {0.0, 0.0, 0.0};
                double rel = 0.0;
                auto bondvec = [&](int j, double* out) {  // r'_j - r'_{j+1}
                    const double pa[3] = {QB[3 * j], QB[3 * j + 1], QB[3 * j + 2]};
                    const double pb[3] = {QB[3 * j + 3], QB[3 * j + 4], QB[3 * j + 5]};
                    (void)separation_v<double, PERIODIC>(pa, pb, per, nd, out);
                };
                if (on) {
                    bondvec(t, st);
                    if (t > 0 && BN[t - 1]) bondvec(t - 1, sm);
                    if (t + 1 < m && BN[t + 1]) bondvec(t + 1, sp);
#pragma unroll
                    for (int c = 0; c < 3; ++c) rel += (VXV[c * nmax + t] - VXV[c * nmax + t + 1]) * st[c];
                }
                const double B = on ? 2.0 * im * (st[0] * st[0] + st[1] * st[1] + st[2] * st[2]) : 1.0;
                const double Aa = on ? -im * (st[0] * sm[0] + st[1] * sm[1] + st[2] * sm[2]) : 0.0;
                const double Cc = on ? -im * (st[0] * sp[0] + st[1] * sp[1] + st[2] * sp[2]) : 0.0;
                const double mu = pcr_solve(PCRW, nmax, m, t, Aa, B, Cc, on ? -rel : 0.0);
                if (t < nmax) LAM[t] = on ? mu : 0.0;
                __syncthreads();
#pragma unroll
                for (int k = 0; k < BPT; ++k) {
                    const int i = grp + k * NG;
                    if (!own[k]) continue;
                    double si[3] = {0.0, 0.0, 0.0}, sim[3] = {0.0, 0.0, 0.0};
                    if (bnk[k]) bondvec(i, si);
                    if (bpk[k]) bondvec(i - 1, sim);
                    const double mi = bnk[k] ? LAM[i] : 0.0, mm = bpk[k] ? LAM[i - 1] : 0.0;
#pragma unroll
                    for (int c = 0; c < 3; ++c) v[k][c] = (Real)(VXV[c * nmax + i] + im * (mi * si[c] - mm * sim[c]));
                }
            }
        }
        bool moved = false, inner_moved = false;
#pragma unroll
        for (int k = 0; k < BPT; ++k) {
            const Real disp2 = sum_sq((Real)(r[k][0] - rref[k][0]), (Real)(r[k][1] - rref[k][1]),
                                      (Real)(r[k][2] - rref[k][2]));
            moved = moved | (own[k] & !(disp2 <= hs2));  // also catches a non-finite position
            if constexpr (INNER) {
                const Real in2 = sum_sq((Real)(r[k][0] - iref[k][0]), (Real)(r[k][1] - iref[k][1]),
                                        (Real)(r[k][2] - iref[k][2]));
                inner_moved = inner_moved | (own[k] & !(in2 <= his2));
            }
        }
        if (INNER && __ballot(inner_moved) != 0ull && (tid & 63) == 0) inner_vote[sub & 1] = ~sub;
        if (__ballot(moved) != 0ull && (tid & 63) == 0) vote[sub & 1] = ~sub;
        __syncthreads();
        cur = 3 * nmax - cur;
    }
    if (bond_max > Real(4) * r0 * r0) flags |= LB_ERR_BOND_STRETCH;
    if (in_solid) flags |= LB_ERR_BEAD_IN_SOLID;
    if (outside) flags |= LB_ERR_BEAD_OUTSIDE;

    // The arguments are read again from here on: held through the substeps, their pointers
    // push the loop's own scalars out of the scalar registers.
    const MDKArgs<Real>& E = reread_args<MDKArgs<Real>>();
    double* dgE = E.b.diag + 8 * rep;
    // The nodes of the next step, marked for its sweep in two passes (several beads may share
    // a 64-node chunk): the chunk's entry is opened here, the bits follow below, after a barrier.
    Marks next;
    if constexpr (own_nodes) next = E.next;
    int chunk[BPT];
    unsigned long long bit[BPT];
#pragma unroll
    for (int k = 0; k < BPT; ++k) {
        chunk[k] = -1;
        bit[k] = 0;
        if (!next.stamp || !own[k] || gl != 0) continue;
        int g[3];
        ngp3(GM.n, GM.fs, r[k], g);
        if (is_solid(GM, g[0], g[1], g[2])) continue;
        const int at = g[0] + GM.n[0] * (g[1] + GM.n[1] * g[2]);
        chunk[k] = at >> 6;
        bit[k] = 1ull << (at & 63);
        next.stamp[chunk[k]] = mark_stamp(step + 1);
        next.mask[chunk[k]] = 0;
    }

    // keep the lists for the next launch when they were (re)built in this one
    if (builds > 0) {
#pragma unroll
        for (int k = 0; k < BPT; ++k) {
            const int i = grp + k * NG;
            if (!own[k]) continue;
            const int gi = b0 + i;
            if (gl == 0) {
#pragma unroll
                for (int c = 0; c < 3; ++c) E.b.rref[c * NT + gi] = rref[k][c];
                E.b.ncount[gi] = cnt[k];
            }
            if (list_lds) {
                const int m = cnt[k] < kNeighbourMax ? cnt[k] : kNeighbourMax;
                for (int q = gl; q < m; q += G) E.b.nlist[(size_t)q * NT + gi] = LL[i + q * nmax];
            }
        }
    }

    // write back, translocation count, centre of mass
    double acc[4] = {0, 0, 0, 0};
#pragma unroll
    for (int k = 0; k < BPT; ++k) {
        const int i = grp + k * NG;
        if (!own[k] || gl != 0) continue;
        const int gi = b0 + i;
#pragma unroll
        for (int c = 0; c < 3; ++c) {
            E.b.r[c * NT + gi] = r[k][c];
            E.b.v[c * NT + gi] = v[k][c];
            E.b.fbar[c * NT + gi] = fb[k][c];
        }
        acc[0] += r[k][0] > xmid ? 1.0 : 0.0;
        acc[1] += r[k][0];
        acc[2] += r[k][1];
        acc[3] += r[k][2];
    }
    block_sums<4>(acc, red, threads);

    // one leader per occupied node (its lowest-index bead) sums the Fbar of the beads on
    // it in index order; a bead alone on its node is its own sum
    bool lead_at[BPT];
    Real lead_f[BPT][3];
    double* FX = P;  // positions are no longer needed
#pragma unroll
    for (int k = 0; k < BPT; ++k) {
        const int i = grp + k * NG;
        if (!own[k] || gl != 0) continue;
#pragma unroll
        for (int c = 0; c < 3; ++c) FX[c * nmax + i] = (double)fb[k][c];
    }
    __syncthreads();
#pragma unroll
    for (int k = 0; k < BPT; ++k) {
        const int i = grp + k * NG;
        const int me = node[k];
        const bool lead = own[k] && me >= 0 && !before[k];
        Real s[3] = {fb[k][0], fb[k][1], fb[k][2]};
        // The few leaders with followers are served one after the other by their whole wave, 64
        // beads a look: one lane scanning every bead behind it alone was a chain of n LDS round
        // trips (23 us of the bead kernel's 93 us for 400 beads).  Bead j's share goes to lane
        // (j - i - 1) mod G of the group and the lanes' shares are added as a group.
        unsigned long long todo = __ballot(lead && shared[k] && gl == 0);
        while (todo) {
            const int src = __builtin_ctzll(todo);
            todo &= todo - 1;
            const int li = __builtin_amdgcn_readlane(i, src), ln = __builtin_amdgcn_readlane(me, src);
            Real t[3] = {0, 0, 0};
            for (int j0 = (li + 1) & ~63; j0 < n; j0 += 64) {
                const int j = j0 + (tid & 63);
                unsigned long long hits = __ballot(j > li && j < n && NODE[j < n ? j : li] == ln);
                while (hits) {
                    const int jj = j0 + __builtin_ctzll(hits);
                    hits &= hits - 1;
                    if ((jj - li - 1) % G == gl) {
#pragma unroll
                        for (int c = 0; c < 3; ++c) t[c] += (Real)FX[c * nmax + jj];
                    }
                }
            }
#pragma unroll
            for (int c = 0; c < 3; ++c) {
                const Real sum = group_sum<G>(t[c]);
                if (i == li) s[c] += sum;
            }
        }
        if (own[k] && gl == 0) {
            const int gi = b0 + i;
            E.b.agg_at[gi] = lead ? pop_base + me : -1;
            E.b.agg_at[NT + gi] = plane;
#pragma unroll
            for (int c = 0; c < 3; ++c) E.b.agg_f[c * NT + gi] = lead ? s[c] : Real(0);
        }
        lead_at[k] = lead && gl == 0;
#pragma unroll
        for (int c = 0; c < 3; ++c) lead_f[k][c] = s[c];
    }
    if constexpr (own_nodes) {
        stores_done();
        __syncthreads();
#pragma unroll
        for (int k = 0; k < BPT; ++k) {
            if (chunk[k] >= 0) atomicOr(&next.mask[chunk[k]], bit[k]);
            if (!lead_at[k]) continue;
            using T = typename Codec<OWN>::T;
            add_reaction<OWN>((T*)E.dst + pop_base + node[k], plane, lead_f[k]);
        }
    }
    if (tid == 0) {
        dgE[0] = acc[0];
        if (dgE[1] < 0.0 && (int)acc[0] == n) dgE[1] = (double)(step + 1);
        dgE[2] = acc[1] / n;
        dgE[3] = acc[2] / n;
        dgE[4] = acc[3] / n;
        dgE[5] = (double)(step + 1);
        dgE[6] += (double)builds;
        if (builds > 0) dgE[7] = 1.0;
    }
    if (flags) atomicOr(&E.st->err, flags);
}

template <class Real, int G, int BPT, bool PERIODIC, int MAXT, bool POLY>
__global__ __launch_bounds__(MAXT) void k_md(MDKArgs<Real> a, int storage) {
    extern __shared__ __align__(16) double lds[];
    bead_step<Real, G, BPT, PERIODIC, MAXT, POLY>(a, storage, blockIdx.x, blockDim.x, lds);
}

// A whole coupled step of one box in one launch: block 0 takes the bead step, which updates the
// nodes its beads sit on (it has their populations for the interpolation) and adds the reaction
// there; the others sweep every other node.  Nobody waits for anybody, so that the launch boundary
// is the only ordering.  Bound by the bead step, a chain of latencies in one workgroup: as launches
// of their own it, the sweep and the spread also paid for a dependency between two queues and for
// the launch that followed (128x64x64, 100 beads, FP32: 42.0 us a step, here 35.8; rigid 70.5 and
// 67.3; 12 beads in 64x32x32: 31.4 and 26.9).  The sweep runs with the bead step's registers, two
// waves a SIMD, which it hides in a box this small.
template <int S, class Real, int G, bool POLY>
__global__ __launch_bounds__(512) void k_step_one(MDKArgs<Real> a, int bead_threads, int tiles) {
    extern __shared__ __align__(16) double lds[];
    if (blockIdx.x == 0) {
        // the bead step is what the launch waits for
        if ((int)threadIdx.x >= bead_threads) return;
        __builtin_amdgcn_s_setprio(3);
        bead_step<Real, G, 1, false, 512, POLY, S>(a, S, 0, bead_threads, lds);
        return;
    }
    using T = typename Codec<S>::T;
    const int tile = xcd_tile((int)blockIdx.x - 1, tiles, -1);
    const long long step = *a.step_at;
    sweep_node<S, false, false, true>(a.reps[0], tile * (int)blockDim.x + (int)threadIdx.x, MAP_FLAT, (const T*)a.cur,
                                (T*)a.dst, a.st, a.now, mark_stamp(step));
}

// ---------------------------------------------------------------------------------
// Host launch.
// ---------------------------------------------------------------------------------
static inline int md_nmax(const Context& c) { return (c.max_beads + 63) / 64 * 64; }

static constexpr size_t kMDLdsBudget = 150 * 1024;
// the bead kernel's static LDS (block sums 512 B, the words of three votes 24 B) stays below this
static constexpr int kMDStaticLds = 2048;

static inline size_t md_base_lds(size_t nmax) { return nmax * (6 * sizeof(double) + sizeof(int) + 1); }
// SHAKE/RATTLE work area of rigid chains: 15 doubles per bead, always in LDS
static inline size_t md_rigid_lds(const Context& c, size_t nmax) { return c.md.rigid ? nmax * 15 * sizeof(double) : 0; }
static inline size_t md_list_lds(size_t nmax) { return nmax * kNeighbourMax * sizeof(unsigned short); }
static inline size_t md_noise_lds(const Context& c, size_t nmax) {
    return (size_t)c.md.M * 3 * nmax * (c.storage == LB_STORE_F64 ? sizeof(double) : sizeof(float));
}

// Verlet lists go to LDS when positions (two buffers), node/bond arrays and lists fit
static inline bool md_lists_in_lds(const Context& c) {
    const size_t nmax = (size_t)md_nmax(c);
    return md_base_lds(nmax) + md_rigid_lds(c, nmax) + md_list_lds(nmax) <= kMDLdsBudget;
}

// the per-step table of random forces, when several lanes share a bead and it fits
static inline bool md_noise_in_lds(const Context& c, int G) {
    const size_t nmax = (size_t)md_nmax(c);
    size_t b = md_base_lds(nmax) + md_rigid_lds(c, nmax) + md_noise_lds(c, nmax);
    if (md_lists_in_lds(c)) b += md_list_lds(nmax);
    return G > 1 && b <= kMDLdsBudget;
}

static inline size_t md_lds_bytes(const Context& c, int G) {
    const size_t nmax = (size_t)md_nmax(c);
    const size_t inner = G == 1 && c.max_beads <= 512 ? nmax * kInnerMax * sizeof(unsigned short) : 0;
    size_t b = md_base_lds(nmax) + md_rigid_lds(c, nmax);
    if (md_lists_in_lds(c)) b += md_list_lds(nmax);
    if (md_noise_in_lds(c, G)) b += md_noise_lds(c, nmax);
    return b + inner;
}

template <class Real>
static inline MDKArgs<Real> md_args(const Context& c, const void* cur, int mode, int G, const StepCount& at = StepCount{}) {
    MDKArgs<Real> a{};
    a.reps = c.d_reps;
    a.md = c.md;
    a.b = *(const BeadPtrs<Real>*)c.bead_ptrs;
    a.cur = cur;
    a.st = c.d_state;
    a.mode = mode;
    a.nmax = md_nmax(c);
    a.list_in_lds = md_lists_in_lds(c) ? 1 : 0;
    a.noise_in_lds = md_noise_in_lds(c, G) ? 1 : 0;
    a.step_at = at.read ? at.read : &c.d_state->step;
    a.step_next = at.next;
    a.last = at.last ? 1 : 0;
    return a;
}

template <class Real, int G, int BPT, bool PER, int MAXT, bool POLY>
static hipError_t launch_md_t(const Context& c, const void* cur, int mode, int block, const StepCount& at,
                              hipStream_t s) {
    const MDKArgs<Real> a = md_args<Real>(c, cur, mode, G, at);
    const size_t lds = md_lds_bytes(c, G);
    static bool attr_set = false;
    if (!attr_set) {
        hipError_t e = hipFuncSetAttribute((const void*)k_md<Real, G, BPT, PER, MAXT, POLY>,
                                           hipFuncAttributeMaxDynamicSharedMemorySize,
                                           160 * 1024 - kMDStaticLds);
        if (e != hipSuccess) return e;
        attr_set = true;
    }
    hipLaunchKernelGGL((k_md<Real, G, BPT, PER, MAXT, POLY>), dim3((unsigned)c.reps.size()), dim3(block), lds, s, a,
                       c.storage);
    return hipGetLastError();
}

// threads of a workgroup of G lanes a bead for m beads
static inline int md_block(int G, int m) { return std::min(1024, (G * m + 63) / 64 * 64); }

// The kernel's LDS attribute, on the current device: lb_init sets it, so that no later call has to,
// least of all one inside a graph capture.
template <int S, class Real, int G, bool POLY>
static hipError_t prepare_step_one_t() {
    return hipFuncSetAttribute((const void*)k_step_one<S, Real, G, POLY>, hipFuncAttributeMaxDynamicSharedMemorySize,
                               160 * 1024 - kMDStaticLds);
}

template <int S, bool POLY>
hipError_t prepare_step_one_g() {
    using Real = typename MDReal<S>::type;
    hipError_t e = prepare_step_one_t<S, Real, 16, POLY>();
    if (e == hipSuccess) e = prepare_step_one_t<S, Real, 8, POLY>();
    if (e == hipSuccess) e = prepare_step_one_t<S, Real, 4, POLY>();
    if (e == hipSuccess) e = prepare_step_one_t<S, Real, 2, POLY>();
    return e;
}

template <int S, class Real, int G, bool POLY>
static hipError_t launch_step_one_t(const Context& c, int cur, bool last, hipStream_t s) {
    MDKArgs<Real> a = md_args<Real>(c, c.pops[cur], MD_COUPLED, G,
                                    {&c.d_state->step_of[cur], last ? nullptr : &c.d_state->step_of[1 - cur], last});
    a.dst = c.pops[1 - cur];
    a.now = c.marks[cur];
    if (!last) a.next = c.marks[1 - cur];
    // 512 threads whatever the beads need: the kernel's registers leave a compute unit two waves a
    // SIMD, and a block of fewer waves than those eight would leave some of them unused
    const int tiles = (c.reps[0].V + 511) / 512;
    hipLaunchKernelGGL((k_step_one<S, Real, G, POLY>), dim3(1 + tiles), dim3(512), md_lds_bytes(c, G), s, a,
                       md_block(G, std::max(c.max_beads, 1)), tiles);
    return hipGetLastError();
}

// one step in one launch for the storage S; hipErrorNotSupported for other lanes per bead than
// the 512-thread workgroups hold
template <int S, bool POLY>
hipError_t launch_step_one_g(const Context& c, int cur, bool last, hipStream_t s) {
    using Real = typename MDReal<S>::type;
    const int m = std::max(c.max_beads, 1);
    const int G = c.md_lanes > 0 ? c.md_lanes : md_default_lanes(m);
    if (md_block(G, m) > 512) return hipErrorNotSupported;
    switch (G) {
        case 16: return launch_step_one_t<S, Real, 16, POLY>(c, cur, last, s);
        case 8: return launch_step_one_t<S, Real, 8, POLY>(c, cur, last, s);
        case 4: return launch_step_one_t<S, Real, 4, POLY>(c, cur, last, s);
        case 2: return launch_step_one_t<S, Real, 2, POLY>(c, cur, last, s);
        default: return hipErrorNotSupported;
    }
}

template <class Real, bool PER, bool POLY>
hipError_t launch_md_g(const Context& c, const void* cur, int mode, const StepCount& at, hipStream_t s) {
    // G lanes per bead (the context's choice); with one lane per bead the 512-thread
    // bound up to 512 beads, the 1024-thread bound beyond, up to 4 beads per lane
    const int m = std::max(c.max_beads, 1);
    const int G = c.md_lanes > 0 ? c.md_lanes : md_default_lanes(m);
    if (!md_lanes_valid(G, m)) return hipErrorInvalidValue;
    auto blk = [](int t) { return md_block(1, t); };
    switch (G) {
        case 16: return launch_md_t<Real, 16, 1, PER, 512, POLY>(c, cur, mode, blk(16 * m), at, s);
        case 8: return launch_md_t<Real, 8, 1, PER, 512, POLY>(c, cur, mode, blk(8 * m), at, s);
        case 4: return launch_md_t<Real, 4, 1, PER, 512, POLY>(c, cur, mode, blk(4 * m), at, s);
        case 2:
            // two lanes per bead: up to 256 beads in the 512-thread bound, up to 512 in the
            // 1024-thread one
            if (2 * m <= 512) return launch_md_t<Real, 2, 1, PER, 512, POLY>(c, cur, mode, blk(2 * m), at, s);
            return launch_md_t<Real, 2, 1, PER, 1024, POLY>(c, cur, mode, blk(2 * m), at, s);
        default: break;
    }
    if (m <= 512) return launch_md_t<Real, 1, 1, PER, 512, POLY>(c, cur, mode, blk(m), at, s);
    if (m <= 1024) return launch_md_t<Real, 1, 1, PER, 1024, POLY>(c, cur, mode, blk(m), at, s);
    if (m <= 2048) return launch_md_t<Real, 1, 2, PER, 1024, POLY>(c, cur, mode, 1024, at, s);
    if (m <= 3072) return launch_md_t<Real, 1, 3, PER, 1024, POLY>(c, cur, mode, 1024, at, s);
    if (m <= 4096) return launch_md_t<Real, 1, 4, PER, 1024, POLY>(c, cur, mode, 1024, at, s);
    return hipErrorInvalidValue;
}

// the eight variants are compiled as objects of their own (md_bead.hip)
extern template hipError_t launch_md_g<float, false, false>(const Context&, const void*, int, const StepCount&,
                                                                  hipStream_t);
extern template hipError_t launch_md_g<float, true, false>(const Context&, const void*, int, const StepCount&,
                                                                  hipStream_t);
extern template hipError_t launch_md_g<float, false, true>(const Context&, const void*, int, const StepCount&,
                                                                  hipStream_t);
extern template hipError_t launch_md_g<float, true, true>(const Context&, const void*, int, const StepCount&,
                                                                  hipStream_t);
extern template hipError_t launch_md_g<double, false, false>(const Context&, const void*, int, const StepCount&,
                                                                  hipStream_t);
extern template hipError_t launch_md_g<double, true, false>(const Context&, const void*, int, const StepCount&,
                                                                  hipStream_t);
extern template hipError_t launch_md_g<double, false, true>(const Context&, const void*, int, const StepCount&,
                                                                  hipStream_t);
extern template hipError_t launch_md_g<double, true, true>(const Context&, const void*, int, const StepCount&,
                                                                  hipStream_t);
extern template hipError_t launch_step_one_g<LB_STORE_F64, false>(const Context&, int, bool, hipStream_t);
extern template hipError_t prepare_step_one_g<LB_STORE_F64, false>();
extern template hipError_t launch_step_one_g<LB_STORE_F64, true>(const Context&, int, bool, hipStream_t);
extern template hipError_t prepare_step_one_g<LB_STORE_F64, true>();
extern template hipError_t launch_step_one_g<LB_STORE_F32, false>(const Context&, int, bool, hipStream_t);
extern template hipError_t prepare_step_one_g<LB_STORE_F32, false>();
extern template hipError_t launch_step_one_g<LB_STORE_F32, true>(const Context&, int, bool, hipStream_t);
extern template hipError_t prepare_step_one_g<LB_STORE_F32, true>();
extern template hipError_t launch_step_one_g<LB_STORE_F16DEV, false>(const Context&, int, bool, hipStream_t);
extern template hipError_t prepare_step_one_g<LB_STORE_F16DEV, false>();
extern template hipError_t launch_step_one_g<LB_STORE_F16DEV, true>(const Context&, int, bool, hipStream_t);
extern template hipError_t prepare_step_one_g<LB_STORE_F16DEV, true>();
extern template hipError_t launch_step_one_g<LB_STORE_BF16DEV, false>(const Context&, int, bool, hipStream_t);
extern template hipError_t prepare_step_one_g<LB_STORE_BF16DEV, false>();
extern template hipError_t launch_step_one_g<LB_STORE_BF16DEV, true>(const Context&, int, bool, hipStream_t);
extern template hipError_t prepare_step_one_g<LB_STORE_BF16DEV, true>();

}  // namespace lbmd

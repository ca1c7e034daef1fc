// lbmd_lattice.hpp -- the lattice update of one node (gfx950): gathers, collision, thermal source.
// Shared by the sweep (lb_kernels.hip) and by the bead kernel, which updates the nodes its beads
// sit on (md_bead.hpp).
#pragma once

#include <type_traits>
#include <utility>

#include "lbmd_internal.hpp"

namespace lbmd {

template <class F, int... Ps>
__device__ __forceinline__ void for_pops_impl(F&& f, std::integer_sequence<int, Ps...>) {
    (f(std::integral_constant<int, Ps>{}), ...);
}
template <class F>
__device__ __forceinline__ void for_pops(F&& f) {
    for_pops_impl(f, std::make_integer_sequence<int, Q>{});
}

// Blocks are dealt round-robin to the 8 XCDs.  Tile order options:
//   C < 0: XCD j takes one contiguous eighth of the tiles (best for one big box);
//   C = 0: the hardware order;
//   C > 0: XCD j takes the chunks j, j+8, j+16, ... of C consecutive tiles, locality
//          with balance when the work per tile is uneven (many small replicas); the
//          partial super-chunk at the end keeps its order.
__device__ __forceinline__ int xcd_tile(int b, int G, int C) {
    if (C < 0) {
        const int per = G >> 3, rem = G & 7, j = b & 7;
        return j * per + (j < rem ? j : rem) + (b >> 3);
    }
    if (C == 0) return b;
    const int S = 8 * C;
    if (b >= (G / S) * S) return b;
    const int j = b & 7, l = b >> 3;
    return ((l / C) * 8 + j) * C + (l % C);
}

__device__ __forceinline__ int replica_of_tile(const int* __restrict__ prefix, int n_reps, int tile) {
    int lo = 0, hi = n_reps - 1;
    while (lo < hi) {
        int mid = (lo + hi + 1) >> 1;
        if (prefix[mid] <= tile) lo = mid;
        else hi = mid - 1;
    }
    return lo;
}

// Solidity of the 27 nodes (x+dx, y+dy, z+dz), dx, dy, dz in {-1, 0, 1}, as bit
// 9(dx+1) + 3(dy+1) + (dz+1): a neighbour is solid when its x plane is a wall plane and its
// (y, z) lies outside that wall's pore.
__device__ __forceinline__ unsigned solid_neighbours(const Replica& R, int x, int y, int z) {
    unsigned solid27 = 0u;
#pragma unroll
    for (int k = 0; k < LB_MAX_WALLS; ++k) {
        if (k >= R.n_walls) break;
        const int* w = R.wall[k];
        unsigned bx = 0, by = 0, bz = 0;
#pragma unroll
        for (int d = -1; d <= 1; ++d) {
            bx |= (unsigned)(x + d >= w[0] && x + d <= w[1]) << (d + 1);
            by |= (unsigned)(y + d >= w[2] && y + d <= w[3]) << (d + 1);
            bz |= (unsigned)(z + d >= w[4] && z + d <= w[5]) << (d + 1);
        }
        // pore membership of (y+dy, z+dz) for the 9 combinations, bit 3(dy+1) + (dz+1)
        unsigned m = 0;
        if (pore_open(w)) {
#pragma unroll
            for (int dy = 0; dy < 3; ++dy)
#pragma unroll
                for (int dz = 0; dz < 3; ++dz)
                    m |= (((by >> dy) & (bz >> dz)) & 1u) << (3 * dy + dz);
        }
        const unsigned closed = ~m & 0x1FFu;
#pragma unroll
        for (int dx = 0; dx < 3; ++dx) solid27 |= (0u - ((bx >> dx) & 1u)) & (closed << (9 * dx));
    }
    return solid27;
}

// whether x lies within one plane of a wall (only such nodes have solid sources)
__device__ __forceinline__ bool in_wall_zone(const Replica& R, int x) {
    bool zone = false;
#pragma unroll
    for (int k = 0; k < LB_MAX_WALLS; ++k) {
        if (k >= R.n_walls) break;
        zone = zone || (x >= R.wall[k][0] - 1 && x <= R.wall[k][1] + 1);
    }
    return zone;
}

enum GatherKind { G_INTERIOR = 0, G_FAST = 1, G_WALL_PLANE = 2, G_WALL = 3, G_FACE = 4, G_GENERIC = 5 };

// Element `node` of a population block that starts at the wave-uniform pointer bp.  The byte
// offset is formed in 32 bits (a replica's population block holds at most 4 GiB, which
// lb_validate_config enforces), so the load takes the scalar-base plus 32-bit-offset form
// and the address costs one vector instruction instead of a 64-bit multiply-add.
template <class T>
__device__ __forceinline__ T ld32(const T* __restrict__ bp, int node) {
    return *(const T*)((const char*)bp + (unsigned)node * (unsigned)sizeof(T));
}

// Incoming populations of one lane of the flattened mapping (64 consecutive nodes
// per wave, possibly spanning rows), as stored numbers (Codec::load_raw).
//  G_GENERIC:    any lane (full resolver, used by waves touching a y/z face and a wall);
//  G_FACE:       lanes on any face, no wall within one node;
//  G_WALL:       y and z interior, lanes may neighbour a wall and its pore (solid test per
//                source over the 27 neighbours);
//  G_WALL_PLANE: y and z interior, lanes may neighbour a wall but lie at least two nodes from
//                its pore in y or z, so that a source is solid exactly when its x plane is a
//                wall plane: only populations with c_x != 0 can bounce, on two per-lane bits;
//  G_FAST:       y and z interior, no wall within one node (only x faces need care);
//  G_INTERIOR:   no lane on any face or within one node of a wall (no test at all).
// Outside G_GENERIC and G_FACE each population is read from its own block at a 32-bit offset; a
// free-slip x face (the reflected population at the node itself) and a solid source (the
// node's own population opp(p), half-way bounce-back) are loads of their own, taken only
// by the lanes that need them.
// RAW: f receives the stored elements themselves (decoded later by the caller), so that no
// conversion sits between the loads of two nodes gathered one after the other.
template <int S, int KIND, bool RAW = false>
__device__ __forceinline__ void gather19(
    const Replica& R, const typename Codec<S>::T* __restrict__ src, int idx, int x, int y, int z,
    std::conditional_t<RAW, typename Codec<S>::T, typename Codec<S>::R>* f) {
    using C = Codec<S>;
    using T = typename C::T;
    auto cv = [](T v) {
        if constexpr (RAW) return v;
        else return C::load_raw(v);
    };
    const long long PS = R.S;  // population plane stride
    const int nx = R.nx, nxy = R.nx * R.ny;
    const T* __restrict__ base = src + R.pop_base;
    if constexpr (KIND == G_GENERIC || KIND == G_FACE) {
        constexpr bool walls = KIND == G_GENERIC;
        const PullMap map = make_pull_map<walls>(R, x, y, z);
        for_pops([&](auto P) {
            constexpr int p = decltype(P)::value;
            // the source population differs from p only by reflections or reversal, which
            // keep the weight class, so the codec scale of p applies to it
            f[p] = cv(base[pull_element<p, walls>(R, map)]);
        });
        return;
    }
    // per-wall 3-bit masks: bit (d+1) set when x+d is a wall plane / y+d, z+d in the pore.
    // 16-bit storage (half the bytes per node, so the sweep is closer to issue-bound) folds
    // them once into the solidity of the 27 neighbours (x+dx, y+dy, z+dz), bit
    // 9(dx+1) + 3(dy+1) + (dz+1), and tests one bit per population; measured slower for
    // FP32 storage, which tests the wall masks per population
    constexpr bool kMask27 = C::deviation;
    unsigned mx[LB_MAX_WALLS] = {0u, 0u}, mp[LB_MAX_WALLS] = {0u, 0u};
    unsigned solid27 = 0u;
    if constexpr (KIND == G_WALL) {
        if constexpr (kMask27) {
            solid27 = solid_neighbours(R, x, y, z);
        } else {
#pragma unroll
            for (int k = 0; k < LB_MAX_WALLS; ++k) {
                if (k >= R.n_walls) break;
                const int* w = R.wall[k];
                unsigned bx = 0, by = 0, bz = 0;
#pragma unroll
                for (int d = -1; d <= 1; ++d) {
                    bx |= (unsigned)(x + d >= w[0] && x + d <= w[1]) << (d + 1);
                    by |= (unsigned)(y + d >= w[2] && y + d <= w[3]) << (d + 1);
                    bz |= (unsigned)(z + d >= w[4] && z + d <= w[5]) << (d + 1);
                }
                // pore membership of (y+dy, z+dz) for the 9 combinations, bit 3*(dy+1)+(dz+1)
                unsigned m = 0;
                if (pore_open(w)) {
#pragma unroll
                    for (int dy = 0; dy < 3; ++dy)
#pragma unroll
                        for (int dz = 0; dz < 3; ++dz)
                            m |= (((by >> dy) & (bz >> dz)) & 1u) << (3 * dy + dz);
                }
                mx[k] = bx;
                mp[k] = m;
            }
        }
    }
    // G_WALL_PLANE: whether the planes x - 1 and x + 1 are wall planes (a fluid node far from
    // the pores is not on one itself, so its c_x = 0 sources are fluid)
    bool solid_m = false, solid_p = false;
    if constexpr (KIND == G_WALL_PLANE) {
#pragma unroll
        for (int k = 0; k < LB_MAX_WALLS; ++k) {
            if (k >= R.n_walls) break;
            solid_m = solid_m || (x - 1 >= R.wall[k][0] && x - 1 <= R.wall[k][1]);
            solid_p = solid_p || (x + 1 >= R.wall[k][0] && x + 1 <= R.wall[k][1]);
        }
    }
    const bool xlo = x == 0, xhi = x == nx - 1, fsx = R.fs[0] != 0;
    for_pops([&](auto P) {
        constexpr int p = decltype(P)::value;
        constexpr int cx = cx_of(p), cy = cy_of(p), cz = cz_of(p);
        int node = idx - (cx + cy * nx + cz * nxy);
        // at an x face the source row's node x itself (free slip, fixed below) or the
        // periodic image
        if constexpr (KIND != G_INTERIOR && cx == 1) {
            if (xlo) node += fsx ? 1 : nx;
        }
        if constexpr (KIND != G_INTERIOR && cx == -1) {
            if (xhi) node -= fsx ? 1 : nx;
        }
        f[p] = cv(ld32(base + (long long)p * PS, node));
        if constexpr (KIND == G_WALL && p != 0) {
            // source offset -c: neighbour bit 9(1 - c_x) + 3(1 - c_y) + (1 - c_z), or bit
            // (1 - c) of each wall's masks
            bool solid = false;
            if constexpr (kMask27) {
                constexpr int bit = 9 * (1 - cx) + 3 * (1 - cy) + (1 - cz);
                solid = (solid27 >> bit) & 1u;
            } else {
#pragma unroll
                for (int k = 0; k < LB_MAX_WALLS; ++k) {
                    if (k >= R.n_walls) break;
                    bool inx = (mx[k] >> (1 - cx)) & 1u;
                    bool inpore = (mp[k] >> (3 * (1 - cy) + (1 - cz))) & 1u;
                    solid = solid || (inx && !inpore);
                }
            }
            // half-way bounce-back: the node's own population opp(p) of the last collision
            if (solid) f[p] = cv(ld32(base + (long long)opp_of(p) * PS, idx));
        }
        if constexpr (KIND == G_WALL_PLANE && cx != 0) {
            if (cx == 1 ? solid_m : solid_p) f[p] = cv(ld32(base + (long long)opp_of(p) * PS, idx));
        }
    });
    if constexpr (KIND != G_INTERIOR) {
        // a free-slip x face: the populations arriving through it are those with c_x reflected,
        // from the node's own plane (one branch per face, taken by the lanes on it)
        if (fsx && xlo) {
            for_pops([&](auto P) {
                constexpr int p = decltype(P)::value;
                if constexpr (cx_of(p) == 1)
                    f[p] = cv(ld32(base + (long long)mirror_of(p, 0) * PS,
                                            idx - (cy_of(p) * nx + cz_of(p) * nxy)));
            });
        }
        if (fsx && xhi) {
            for_pops([&](auto P) {
                constexpr int p = decltype(P)::value;
                if constexpr (cx_of(p) == -1)
                    f[p] = cv(ld32(base + (long long)mirror_of(p, 0) * PS,
                                            idx - (cy_of(p) * nx + cz_of(p) * nxy)));
            });
        }
    }
}

// Whether (y, z) lies within one node of an open pore of a wall whose zone holds x (only then
// can a neighbour of a fluid node next to the wall lie in the pore).
__device__ __forceinline__ bool near_pore(const Replica& R, int x, int y, int z) {
    bool near = false;
#pragma unroll
    for (int k = 0; k < LB_MAX_WALLS; ++k) {
        if (k >= R.n_walls) break;
        const int* w = R.wall[k];
        near = near || (pore_open(w) && x >= w[0] - 1 && x <= w[1] + 1 && y >= w[2] - 1 && y <= w[3] + 1 &&
                        z >= w[4] - 1 && z <= w[5] + 1);
    }
    return near;
}

// Row-segment work units: one wave owns up to 64 consecutive x of one row (y, z) of
// one replica, so y, z and every face decision are uniform across the wave and a
// lane only has to care about its own x.  segs = ceil(nx / 64) units per row.
struct RowUnit {
    int y, z, x0;
    bool valid;
};

__device__ __forceinline__ RowUnit row_unit(const Replica& R, int unit) {
    RowUnit u;
    const int segs = (R.nx + 63) >> 6;
    const int rows = R.ny * R.nz;
    u.valid = unit < rows * segs;
    const int row = unit / segs;
    u.x0 = (unit - row * segs) << 6;
    u.z = row / R.ny;
    u.y = row - u.z * R.ny;
    return u;
}

// Incoming populations of one lane of a row unit.  Face handling is uniform (the wave's
// y and z, so the source population after a y or z reflection is uniform too); x faces
// are per lane.  WALL: the segment is within one node of a wall plane, so every source
// is tested for solidity (bounce-back); the pore test of a source depends only on
// (y - c_y, z - c_z) and is uniform.  f receives the stored elements, decoded once all loads are
// issued (a conversion beside each load makes the compiler wait for every load in turn: 28.9 us a
// sweep of 128x64x64 in 16-bit storage instead of 19.8).
template <int S, bool WALL>
__device__ __forceinline__ void gather_row(const Replica& R, const typename Codec<S>::T* __restrict__ src,
                                           int idx, int x, int y, int z, typename Codec<S>::T* f) {
    using T = typename Codec<S>::T;
    const long long PS = R.S;  // population plane stride
    const int nx = R.nx, ny = R.ny, nz = R.nz, nxy = R.nx * R.ny;
    const T* __restrict__ base = src + R.pop_base;
    const bool xlo = x == 0, xhi = x == nx - 1, fsx = R.fs[0] != 0;
    for_pops([&](auto P) {
        constexpr int p = decltype(P)::value;
        constexpr int cx = cx_of(p), cy = cy_of(p), cz = cz_of(p);
        int node = idx - (cx + cy * nx + cz * nxy);
        bool fy = false, fz = false;
        int sy = y - cy, sz = z - cz;
        if constexpr (cy != 0) {
            if (y == (cy > 0 ? 0 : ny - 1)) {
                if (R.fs[1]) { node += cy * nx; fy = true; sy = y; }
                else node += cy * nxy;
            }
        }
        if constexpr (cz != 0) {
            if (z == (cz > 0 ? 0 : nz - 1)) {
                if (R.fs[2]) { node += cz * nxy; fz = true; sz = z; }
                else node += cz * (long long)nxy * nz;
            }
        }
        if constexpr (cx == 1) {
            if (xlo) node += fsx ? 1 : nx;
        }
        if constexpr (cx == -1) {
            if (xhi) node -= fsx ? 1 : nx;
        }
        const int q = mirror_combo<p>(false, fy, fz);  // uniform over the wave
        f[p] = ld32(base + (long long)q * PS, node);
        if constexpr (cx != 0) {
            // free slip: the population with c_x reflected as well, from that node
            if (fsx && (cx == 1 ? xlo : xhi)) {
                const int m = mirror_combo<p>(true, fy, fz);
                f[p] = ld32(base + (long long)m * PS, node);
            }
        }
        if constexpr (WALL && p != 0) {
            // walls are at least two planes away from the x faces, so x - c_x is the
            // source plane of every lane that can see a wall
            bool solid = false;
#pragma unroll
            for (int k = 0; k < LB_MAX_WALLS; ++k) {
                if (k >= R.n_walls) break;
                const int* w = R.wall[k];
                const bool inpore = pore_open(w) && sy >= w[2] && sy <= w[3] && sz >= w[4] && sz <= w[5];
                solid = solid || (!inpore && x - cx >= w[0] && x - cx <= w[1]);
            }
            // half-way bounce-back: the node's own population opp(p) of the last collision
            if (solid) f[p] = ld32(base + (long long)opp_of(p) * PS, idx);
        }
    });
}

// BGK relaxation of one node (Eq. lbe with the f_eq equation), in place on the stored numbers
// h_p = k_p (f_p - o_p) with k_p the codec's scale and o_p = w_p rho0 for deviation storage
// (k_p = 1, o_p = 0 for full storage); returns rho.  The opposite populations p, opp(p) are
// taken as pairs: their sum and difference give the moments, and they share |c.u| in f_eq:
// f_eq,p - o_p = w_p (b + rho (4.5 (c.u)^2 - 1.5 u^2) +- 3 rho c.u) with b = sum_p (f_p - o_p),
// that is rho - rho0 for deviation storage and rho for full storage.  The relaxation
// h*_p = (1 - omega) h_p + omega k_p (f_eq,p - o_p) keeps every scale in a constant.
template <int S>
__device__ __forceinline__ typename Codec<S>::R collide(typename Codec<S>::R* h,
                                                        typename Codec<S>::R omega,
                                                        typename Codec<S>::R rho0) {
    using C = Codec<S>;
    using Rl = typename C::R;
    // moments from the pair sums and differences (the o_p cancel in j: sum_p w_p c_p = 0)
    Rl m0 = h[0] * (Rl(1) / C::template kScale<0>), jx = 0, jy = 0, jz = 0;
    for_pops([&](auto P) {
        constexpr int p = decltype(P)::value;
        if constexpr (p % 2 == 1) {
            constexpr Rl is = Rl(1) / C::template kScale<p>;  // opp(p) = p + 1 shares it
            const Rl sum = h[p] + h[p + 1], dif = h[p] - h[p + 1];
            m0 += sum * is;
            if constexpr (cx_of(p) != 0) jx += dif * Rl(cx_of(p) * is);
            if constexpr (cy_of(p) != 0) jy += dif * Rl(cy_of(p) * is);
            if constexpr (cz_of(p) != 0) jz += dif * Rl(cz_of(p) * is);
        }
    });
    // deviation storage: m0 = rho - rho0; full storage: m0 = rho
    const Rl rho = C::deviation ? rho0 + m0 : m0;
    Rl inv;
    if constexpr (sizeof(Rl) == 4) inv = __builtin_amdgcn_rcpf(rho);  // about 1 ulp
    else inv = Rl(1) / rho;
    // The fused multiply-adds are spelled out: left to the compiler, their choice differs between
    // the kernels this is compiled into, and a node must not depend on which of them updates it.
    const Rl ux = jx * inv, uy = jy * inv, uz = jz * inv;
    const Rl usq = Rl(1.5) * sum_sq(ux, uy, uz);
    const Rl rus = rho * usq;
    const Rl r3 = Rl(3) * rho, r45 = Rl(4.5) * rho;
    const Rl om1 = Rl(1) - omega;
    // omega k_p w_p per weight class (k_p is a power of two near 1/w_p)
    const Rl cw0 = omega * (w_of<Rl>(0) * C::template kScale<0>);
    const Rl cw1 = omega * (w_of<Rl>(1) * C::template kScale<1>);
    const Rl cw7 = omega * (w_of<Rl>(7) * C::template kScale<7>);
    h[0] = fused(om1, h[0], cw0 * fused(-rho, usq, m0));
    for_pops([&](auto P) {
        constexpr int p = decltype(P)::value;
        if constexpr (p % 2 == 1) {
            // c.u over the one or two axes of c
            Rl cu = 0;
            if constexpr (cx_of(p) != 0) cu = Rl(cx_of(p)) * ux;
            if constexpr (cy_of(p) != 0) cu = fused(Rl(cy_of(p)) * jy, inv, cu);
            if constexpr (cz_of(p) != 0) cu = fused(Rl(cz_of(p)) * jz, inv, cu);
            const Rl e = m0 + fused(r45 * cu, cu, -rus);  // b + rho (4.5 cu^2 - 1.5 u^2)
            const Rl cw = p <= 6 ? cw1 : cw7;
            h[p] = fused(om1, h[p], cw * fused(r3, cu, e));
            h[p + 1] = fused(om1, h[p + 1], cw * fused(-r3, cu, e));
        }
    });
    return rho;
}

// Thermal source F_p of Eq. lbe (the fluctuating LB that Sec. II adopts), added to the
// post-collision populations: F = phi Pi eta, eta_p = sqrt(w_p) xi_p with xi_p of zero
// mean and unit variance (sqrt(12) times a symmetric uniform from Philox words p of the
// counters (node, step, j, 2)), Pi x = x - w (sum x + 3 c . sum c x) (no density or
// momentum in the noise), phi^2 = (kT / c_s^2) (1 - gamma^2) rho.  Its covariance
// mu rho (1 - gamma^2) Pi W is what keeps the equilibrium fluctuations mu rho w_p of the
// populations through a BGK collision with rate omega = 1 - gamma.  f holds the codec's stored
// numbers, so the source of population p is added times its scale k_p.
template <class C, class Rl>
__device__ __forceinline__ void add_thermal(Rl* f, uint32_t node, uint32_t step, uint32_t k0, uint32_t k1,
                                            Rl phi) {
    Rl s0 = 0, sx = 0, sy = 0, sz = 0;
    U4 w{0u, 0u, 0u, 0u};
    for_pops([&](auto P) {
        constexpr int p = decltype(P)::value;
        if constexpr (p % 4 == 0) w = philox4x32_10(U4{node, step, (uint32_t)(p / 4), 2u}, k0, k1);
        uint32_t word;
        if constexpr (p % 4 == 0) word = w.x;
        else if constexpr (p % 4 == 1) word = w.y;
        else if constexpr (p % 4 == 2) word = w.z;
        else word = w.w;
        // sqrt(12 w_p): 2 for the rest population, sqrt(2/3) and sqrt(1/3) for faces and edges
        constexpr int c2 = cx_of(p) * cx_of(p) + cy_of(p) * cy_of(p) + cz_of(p) * cz_of(p);
        constexpr double amp = c2 == 0 ? 2.0 : c2 == 1 ? 0.81649658092772603 : 0.57735026918962576;
        const Rl eta = Rl(amp) * symmetric_uniform<Rl>(word);
        s0 += eta;
        if constexpr (cx_of(p) != 0) sx += Rl(cx_of(p)) * eta;
        if constexpr (cy_of(p) != 0) sy += Rl(cy_of(p)) * eta;
        if constexpr (cz_of(p) != 0) sz += Rl(cz_of(p)) * eta;
        f[p] += (phi * C::template kScale<p>) * eta;
    });
    for_pops([&](auto P) {
        constexpr int p = decltype(P)::value;
        Rl m = s0;
        if constexpr (cx_of(p) != 0) m += Rl(3 * cx_of(p)) * sx;
        if constexpr (cy_of(p) != 0) m += Rl(3 * cy_of(p)) * sy;
        if constexpr (cz_of(p) != 0) m += Rl(3 * cz_of(p)) * sz;
        f[p] -= phi * (w_of<Rl>(p) * C::template kScale<p>) * m;
    });
}

// Thread-to-node mappings of the lattice kernel.  MAP_SHIFTED is MAP_FLAT with every x-row
// rotated by the replica's x_shift, chosen on the host so that the planes within one node of a
// wall fall into as few 64-lane waves as possible: the other waves of a row then take the
// gather without solid tests (used when nx is a multiple of 64, so that waves are row segments).
// MAP_FLAT2: two nodes per lane, 64 apart (k_stream_collide_2n).
enum LatticeMapping { MAP_FLAT = 0, MAP_ROWS = 1, MAP_SHIFTED = 2, MAP_FLAT2 = 3 };

// Collision of one fluid node (Eq. lbe), the density check, and the thermal source F_p.
template <int S, bool TH>
__device__ __forceinline__ void relax_node(const Replica& R, typename Codec<S>::R* f, int idx,
                                           RunState* __restrict__ st) {
    using Rl = typename Codec<S>::R;
    const Rl rho = collide<S>(f, (Rl)R.omega, (Rl)R.rho0);
    if (!(rho > Rl(0)) || !(rho < Rl(1e30))) atomicOr(&st->err, LB_ERR_DENSITY);
    if constexpr (TH) {
        const Rl phi = sqrt(fmax((Rl)R.noise_c * rho, Rl(0)));
        // the step counter does not move during a sweep with a thermal source
        add_thermal<Codec<S>, Rl>(f, (uint32_t)idx, (uint32_t)st->step, R.seed_lo, R.seed_hi, phi);
    }
}

// The slots of a solid node: never read (a fluid node bounces back off its own slots, and the
// read-outs report zero there), but written with every sweep, the rest value w_p rho0 that
// lb_init leaves there, so that a store instruction of a wave covers whole cache lines.  A
// wave whose lanes skip their stores leaves partly written lines, which HBM completes with a
// read-modify-write: in 48-96 node rows, each crossing a wall, that cost the 16-bit sweep 40 %.
template <int S>
__device__ __forceinline__ void rest_slots(const Replica& R, typename Codec<S>::R* f) {
    using C = Codec<S>;
    using Rl = typename C::R;
    for_pops([&](auto P) {
        constexpr int p = decltype(P)::value;
        if constexpr (C::deviation) f[p] = Rl(0);
        else f[p] = w_of<Rl>(p) * (Rl)R.rho0;
    });
}

__device__ __forceinline__ bool node_marked(const Marks& m, int idx, long long stamp) {
    const int c = idx >> 6;
    return m.stamp[c] == stamp && ((m.mask[c] >> (idx & 63)) & 1ull);
}

// non-temporal stores keep a box larger than the last-level cache from evicting the next step's
// sources; a box that fits it is better left cached for the next sweep
template <int S, bool NT>
__device__ __forceinline__ void store_node(const Replica& R, const typename Codec<S>::R* f,
                                           typename Codec<S>::T* __restrict__ dst, int idx) {
    using C = Codec<S>;
    typename C::T* __restrict__ out = dst + R.pop_base + idx;
    const long long PS = R.S;  // population plane stride
    for_pops([&](auto P) {
        constexpr int p = decltype(P)::value;
        if constexpr (NT) __builtin_nontemporal_store(C::store_raw(f[p]), out + (long long)p * PS);
        else out[(long long)p * PS] = C::store_raw(f[p]);
    });
}

// One LB time step of node n of replica R, 64 consecutive nodes per wave (n in the flat or shifted
// order): waves that touch a y/z face take the general resolver, waves next to a wall the
// solid-testing one.  MARKED: the marked nodes are left to the bead kernel.
template <int S, bool NT, bool TH, bool MARKED>
__device__ __forceinline__ void sweep_node(const Replica& R, int n, int mapping,
                                           const typename Codec<S>::T* __restrict__ src,
                                           typename Codec<S>::T* __restrict__ dst, RunState* __restrict__ st,
                                           const Marks& marks = Marks{}, long long stamp = 0) {
    using C = Codec<S>;
    using Rl = typename C::R;
    const bool inside = n < R.V;
    bool active = inside;
    const uint32_t t = fdiv((uint32_t)n, R.div_nx);
    int x = n - (int)t * R.nx;
    if (mapping == MAP_SHIFTED) {
        x += R.x_shift;
        if (x >= R.nx) x -= R.nx;
    }
    const int idx = x + (int)t * R.nx;
    const uint32_t zz = fdiv(t, R.div_ny);
    const int y = (int)t - (int)zz * R.ny;
    const int z = (int)zz;
    bool face = false, zone = false, xface = false, pore = false;
    if (active) {
        if (is_solid(R, x, y, z)) active = false;
        face = y == 0 || y == R.ny - 1 || z == 0 || z == R.nz - 1;
        zone = in_wall_zone(R, x);
        xface = x == 0 || x == R.nx - 1;
        pore = near_pore(R, x, y, z);
    }
    const bool any_face = __ballot(face && active) != 0;
    const bool any_zone = __ballot(zone && active) != 0;
    const bool any_xface = __ballot(xface && active) != 0;
    const bool any_pore = __ballot(pore && active) != 0;
    if (!inside) return;
    // 16-bit elements are gathered as stored and decoded once all loads are issued: a conversion
    // beside each load makes the compiler wait for every load in turn (the 203x77x91 sweep in
    // BF16 then takes 35 us instead of 21)
    constexpr bool raw = C::deviation;
    using E = std::conditional_t<raw, typename C::T, Rl>;
    E g[Q];
    if (active) {
        if (any_face && any_zone) gather19<S, G_GENERIC, raw>(R, src, idx, x, y, z, g);
        else if (any_face) gather19<S, G_FACE, raw>(R, src, idx, x, y, z, g);
        else if (any_pore) gather19<S, G_WALL, raw>(R, src, idx, x, y, z, g);
        else if (any_zone) gather19<S, G_WALL_PLANE, raw>(R, src, idx, x, y, z, g);
        else if (any_xface) gather19<S, G_FAST, raw>(R, src, idx, x, y, z, g);
        else gather19<S, G_INTERIOR, raw>(R, src, idx, x, y, z, g);
    }
    Rl f[Q];
    for_pops([&](auto P) {
        constexpr int p = decltype(P)::value;
        if constexpr (raw) f[p] = C::load_raw(g[p]);
        else f[p] = g[p];
    });
    if (!active) rest_slots<S>(R, f);
    else relax_node<S, TH>(R, f, idx, st);
    if constexpr (MARKED) {
        if (node_marked(marks, idx, stamp)) return;
    }
    store_node<S, NT>(R, f, dst, idx);
}

}  // namespace lbmd

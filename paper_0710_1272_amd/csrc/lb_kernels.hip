// lb_kernels.hip -- lattice kernels (gfx950).
//
// k_stream_collide: one LB time step (arXiv:0710.1272 Sec. II, Eq. lbe with F_p = 0;
// the source S_p is added afterwards by the spread kernel) in pull form.  Each thread
// owns one node: it gathers the 19 post-collision populations that stream into the
// node (periodic wrap, specular free-slip faces, half-way bounce-back on solid nodes),
// forms rho and j (Eqs. dens, vel), relaxes towards f_eq (f_eq eq.) with
// omega = 1/tau, and writes its own 19 post-collision values, coalesced and
// non-temporal.  Per replica the populations form a [19][V] block with x fastest;
// 16-bit storage keeps s_p (f_p - w_p rho0).  HBM traffic per fluid node is
// 19 loads + 19 stores of the storage type, the kernel's roofline.
#include <type_traits>
#include <utility>

#include "lbmd_lattice.hpp"

namespace lbmd {

template <int S, int BLOCK, bool NT, bool TH>
__global__ __launch_bounds__(BLOCK) void k_stream_collide(const Replica* __restrict__ reps,
                                                          const int* __restrict__ prefix,
                                                          int n_reps,
                                                          const typename Codec<S>::T* __restrict__ src,
                                                          typename Codec<S>::T* __restrict__ dst,
                                                          RunState* __restrict__ st, int bump_step,
                                                          int xcd_chunk, int mapping) {
    using C = Codec<S>;
    using Rl = typename C::R;
    if (bump_step && blockIdx.x == 0 && threadIdx.x == 0) st->step += 1;
    const int tile = xcd_tile(blockIdx.x, gridDim.x, xcd_chunk);
    const int r = replica_of_tile(prefix, n_reps, tile);
    const Replica& R = reps[r];
    if (mapping != MAP_ROWS) {
        sweep_node<S, NT, TH, false>(R, (tile - prefix[r]) * BLOCK + threadIdx.x, mapping, src, dst, st);
        return;
    }
    // one wave per row segment: y, z and the face decisions are wave-uniform
    constexpr int W = BLOCK / 64;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const RowUnit U = row_unit(R, (tile - prefix[r]) * W + wave);
    if (!U.valid) return;
    const int x = U.x0 + (threadIdx.x & 63);
    const int y = U.y, z = U.z;
    if (x >= R.nx) return;
    const bool solid = is_solid(R, x, y, z);
    const int idx = x + R.nx * (y + R.ny * z);
    bool zone = false;
#pragma unroll
    for (int k = 0; k < LB_MAX_WALLS; ++k) {
        if (k >= R.n_walls) break;
        zone = zone || (U.x0 <= R.wall[k][1] + 1 && U.x0 + 63 >= R.wall[k][0] - 1);
    }
    typename C::T g[Q];
    if (!solid) {
        if (zone) gather_row<S, true>(R, src, idx, x, y, z, g);
        else gather_row<S, false>(R, src, idx, x, y, z, g);
    }
    Rl f[Q];
    for_pops([&](auto P) {
        constexpr int p = decltype(P)::value;
        f[p] = C::load_raw(g[p]);
    });
    if (solid) rest_slots<S>(R, f);
    else relax_node<S, TH>(R, f, idx, st);
    store_node<S, NT>(R, f, dst, idx);
}

template <int S, int KIND, class E>
__device__ __forceinline__ void gather_two(const Replica& R, const typename Codec<S>::T* __restrict__ src,
                                           const int* n, const int* x, const int* y, const int* z, E* f0,
                                           E* f1) {
    constexpr bool raw = !std::is_same_v<E, typename Codec<S>::R>;
    gather19<S, KIND, raw>(R, src, n[0], x[0], y[0], z[0], f0);
    gather19<S, KIND, raw>(R, src, n[1], x[1], y[1], z[1], f1);
}

// One LB step for two nodes per lane, 64 apart: a wave takes 128 consecutive nodes of a
// replica and every load still covers 64 consecutive elements.  Both nodes' 19 loads are
// issued before the first collision, so a wave keeps twice the bytes in flight while it
// computes (16-bit storage moves only 128 bytes per load).  Both gathers run for every lane:
// a solid node, or a lane past the end of the replica (which takes the last node), reads
// nodes of the box and its results are dropped; solid nodes store their rest slots.
template <int S, int BLOCK, bool NT, bool TH>
__global__ __launch_bounds__(BLOCK) void k_stream_collide_2n(const Replica* __restrict__ reps,
                                                             const int* __restrict__ prefix, int n_reps,
                                                             const typename Codec<S>::T* __restrict__ src,
                                                             typename Codec<S>::T* __restrict__ dst,
                                                             RunState* __restrict__ st, int bump_step,
                                                             int xcd_chunk) {
    using C = Codec<S>;
    using Rl = typename C::R;
    if (bump_step && blockIdx.x == 0 && threadIdx.x == 0) st->step += 1;
    const int tile = xcd_tile(blockIdx.x, gridDim.x, xcd_chunk);
    const int r = replica_of_tile(prefix, n_reps, tile);
    const Replica& R = reps[r];
    const int first = (tile - prefix[r]) * (2 * BLOCK) + (threadIdx.x >> 6) * 128 + (threadIdx.x & 63);
    int n[2], x[2], y[2], z[2];
    bool act[2], in[2];
    bool face = false, zone = false, xface = false, pore = false;
#pragma unroll
    for (int k = 0; k < 2; ++k) {
        int m = first + 64 * k;
        in[k] = m < R.V;
        act[k] = in[k];
        if (!in[k]) m = R.V - 1;
        const uint32_t t = fdiv((uint32_t)m, R.div_nx);
        x[k] = m - (int)t * R.nx;
        const uint32_t zz = fdiv(t, R.div_ny);
        y[k] = (int)t - (int)zz * R.ny;
        z[k] = (int)zz;
        n[k] = m;
        // the gather kind covers every node the lane reads around, solid or not
        face = face || y[k] == 0 || y[k] == R.ny - 1 || z[k] == 0 || z[k] == R.nz - 1;
        zone = zone || in_wall_zone(R, x[k]);
        xface = xface || x[k] == 0 || x[k] == R.nx - 1;
        pore = pore || near_pore(R, x[k], y[k], z[k]);
        act[k] = act[k] && !is_solid(R, x[k], y[k], z[k]);
    }
    const bool any_face = __ballot(face) != 0;
    const bool any_zone = __ballot(zone) != 0;
    const bool any_xface = __ballot(xface) != 0;
    const bool any_pore = __ballot(pore) != 0;
    if (!in[0]) return;  // then the second node is outside too
    // 16-bit elements are gathered as stored and decoded after both nodes' loads are issued
    using E = std::conditional_t<C::deviation, typename C::T, Rl>;
    E g0[Q], g1[Q];
    if (any_face && any_zone) gather_two<S, G_GENERIC>(R, src, n, x, y, z, g0, g1);
    else if (any_face) gather_two<S, G_FACE>(R, src, n, x, y, z, g0, g1);
    else if (any_pore) gather_two<S, G_WALL>(R, src, n, x, y, z, g0, g1);
    else if (any_zone) gather_two<S, G_WALL_PLANE>(R, src, n, x, y, z, g0, g1);
    else if (any_xface) gather_two<S, G_FAST>(R, src, n, x, y, z, g0, g1);
    else gather_two<S, G_INTERIOR>(R, src, n, x, y, z, g0, g1);
    Rl f0[Q], f1[Q];
    for_pops([&](auto P) {
        constexpr int p = decltype(P)::value;
        if constexpr (C::deviation) {
            f0[p] = C::load_raw(g0[p]);
            f1[p] = C::load_raw(g1[p]);
        } else {
            f0[p] = g0[p];
            f1[p] = g1[p];
        }
    });

    auto finish = [&](Rl* f, int idx, bool fluid) {
        if (fluid) relax_node<S, TH>(R, f, idx, st);
        else rest_slots<S>(R, f);
        store_node<S, NT>(R, f, dst, idx);
    };
    finish(f0, n[0], act[0]);
    if (in[1]) finish(f1, n[1], act[1]);
}

// Same-pattern reference of the lattice kernel: every population of every node read at the
// kernel's pull address (the node index minus c_p's offset, wrapped into the replica; no faces,
// no solids, no arithmetic) and written unchanged to the node's own slot of the other buffer,
// in the kernel's tile order and store policy, one node per lane.  Its bandwidth bounds what
// the sweep's access pattern can reach.
template <int S, int BLOCK, bool NT>
__global__ __launch_bounds__(BLOCK) void k_pattern(const Replica* __restrict__ reps, const int* __restrict__ prefix,
                                                   int n_reps, const typename Codec<S>::T* __restrict__ src,
                                                   typename Codec<S>::T* __restrict__ dst, int xcd_chunk) {
    using T = typename Codec<S>::T;
    const int tile = xcd_tile(blockIdx.x, gridDim.x, xcd_chunk);
    const int r = replica_of_tile(prefix, n_reps, tile);
    const Replica& R = reps[r];
    const long long V = R.V, PS = R.S;
    const long long n = (long long)(tile - prefix[r]) * BLOCK + threadIdx.x;
    if (n >= V) return;
    const T* __restrict__ base = src + R.pop_base;
    T* __restrict__ out = dst + R.pop_base;
    const long long nx = R.nx, nxy = (long long)R.nx * R.ny;
    T v[Q];
    for_pops([&](auto P) {
        constexpr int p = decltype(P)::value;
        long long s = n - (cx_of(p) + cy_of(p) * nx + cz_of(p) * nxy);
        if (s < 0) s += V;
        else if (s >= V) s -= V;
        v[p] = base[(long long)p * PS + s];
    });
    for_pops([&](auto P) {
        constexpr int p = decltype(P)::value;
        if constexpr (NT) __builtin_nontemporal_store(v[p], out + (long long)p * PS + n);
        else out[(long long)p * PS + n] = v[p];
    });
}

// ---------------------------------------------------------------------------------
// Initial state: a post-collision buffer whose pull reproduces wanted pre-collision
// populations f0 (given, or f_eq of given rho/u, or w_p rho0).  Slot (s, q) holds
// f0 at the push target (x, p) of (s, q).
// ---------------------------------------------------------------------------------
// f_eq of Sec. II for all 19 populations (c_s^2 = 1/3), in FP64
__device__ __forceinline__ void feq19(double rho, double ux, double uy, double uz, double* feq) {
    const double usq = 1.5 * (ux * ux + uy * uy + uz * uz);
    for_pops([&](auto P) {
        constexpr int p = decltype(P)::value;
        const double cu = cx_of(p) * ux + cy_of(p) * uy + cz_of(p) * uz;
        feq[p] = w_of<double>(p) * rho * (1.0 + 3.0 * cu + 4.5 * cu * cu - usq);
    });
}

// element p of a register array without dynamic indexing
__device__ __forceinline__ double pick19(const double* a, int p) {
    double v = 0.0;
    for_pops([&](auto P) {
        constexpr int k = decltype(P)::value;
        v = (p == k) ? a[k] : v;
    });
    return v;
}

template <int S>
__global__ __launch_bounds__(256) void k_init(const Replica* __restrict__ reps, int r,
                                              typename Codec<S>::T* __restrict__ dst,
                                              const double* __restrict__ rho_in,
                                              const double* __restrict__ u_in,
                                              const double* __restrict__ pops_in) {
    using C = Codec<S>;
    const Replica& R = reps[r];
    const int s = blockIdx.x * 256 + threadIdx.x;
    if (s >= R.V) return;
    const long long V = R.V;  // the given fields are dense [19][V] / [3][V]
    const int sx = s % R.nx, sy = (s / R.nx) % R.ny, sz = s / (R.nx * R.ny);
    const bool solid = is_solid(R, sx, sy, sz);
    typename C::T* out = dst + R.pop_base + s;
    // the wanted pre-collision population p at node x
    auto wanted = [&](int p, int x) -> double {
        if (pops_in) return pops_in[(long long)p * V + x];
        const double rho = rho_in ? rho_in[x] : R.rho0;
        double feq[Q];
        if (u_in) feq19(rho, u_in[x], u_in[V + x], u_in[2 * V + x], feq);
        else feq19(rho, 0.0, 0.0, 0.0, feq);
        return pick19(feq, p);
    };
    for_pops([&](auto P) {
        constexpr int q = decltype(P)::value;
        double val = w_of<double>(q) * R.rho0;
        int p;
        if (!solid) {
            const int x = push_target<q>(R, sx, sy, sz, &p);
            val = wanted(p, x);
        }
        if constexpr (C::deviation) val -= w_of<double>(q) * R.rho0;
        out[(long long)q * R.S] = C::template store<q>((typename C::R)val);
    });
}

// ---------------------------------------------------------------------------------
// Pre-collision view of the current state (lb_moments): pull-gather of one node,
// decoded to FP64 full populations.
// ---------------------------------------------------------------------------------
template <int S>
__device__ __forceinline__ void gather_f64(const Replica& R, const typename Codec<S>::T* __restrict__ src,
                                           int x, int y, int z, double* f) {
    using C = Codec<S>;
    const PullMap map = make_pull_map(R, x, y, z);
    typename C::T raw[Q];
    for_pops([&](auto P) {
        constexpr int p = decltype(P)::value;
        raw[p] = src[R.pop_base + pull_element<p>(R, map)];
    });
    for_pops([&](auto P) {
        constexpr int p = decltype(P)::value;
        double v = (double)C::template load<p>(raw[p]);
        if constexpr (C::deviation) v += w_of<double>(p) * R.rho0;
        f[p] = v;
    });
}

// mode 0: populations [19][count]; mode 1: rho, u_x, u_y, u_z [4][count]
template <int S>
__global__ __launch_bounds__(256) void k_gather(const Replica* __restrict__ reps, int r,
                                                const typename Codec<S>::T* __restrict__ src, int mode,
                                                long long node0, int count, double* __restrict__ out) {
    const Replica& R = reps[r];
    const int i = blockIdx.x * 256 + threadIdx.x;
    if (i >= count) return;
    const long long s = node0 + i;
    const int x = (int)(s % R.nx), y = (int)((s / R.nx) % R.ny), z = (int)(s / ((long long)R.nx * R.ny));
    double f[Q];
    if (is_solid(R, x, y, z)) {
        for_pops([&](auto P) { f[decltype(P)::value] = 0.0; });
    } else {
        gather_f64<S>(R, src, x, y, z, f);
    }
    if (mode == 0) {
        for_pops([&](auto P) {
            constexpr int p = decltype(P)::value;
            out[(long long)p * count + i] = f[p];
        });
    } else {
        double rho = 0, jx = 0, jy = 0, jz = 0;
        for_pops([&](auto P) {
            constexpr int p = decltype(P)::value;
            rho += f[p];
            jx += cx_of(p) * f[p];
            jy += cy_of(p) * f[p];
            jz += cz_of(p) * f[p];
        });
        const double inv = rho != 0.0 ? 1.0 / rho : 0.0;
        out[i] = rho;
        out[count + i] = jx * inv;
        out[2LL * count + i] = jy * inv;
        out[3LL * count + i] = jz * inv;
    }
}

// FP64 totals of rho and j over the fluid nodes of replica r (Eqs. dens, vel summed over the
// box): per-lane sums over a fixed sequence of 64-node chunks, wavefront butterfly, block
// tree, one partial per block; a second single-block pass adds the partials in a fixed order
// (deterministic for a given grid).
template <int S>
__global__ __launch_bounds__(256) void k_conserved_partial(const Replica R,
                                                           const typename Codec<S>::T* __restrict__ src,
                                                           double* __restrict__ partials) {
    using C = Codec<S>;
    using Rl = typename C::R;
    // 64 consecutive nodes per wave, dealt to the waves of the grid in a fixed order; each
    // wave takes the cheapest gather that covers its lanes, as the lattice kernel does
    double acc[4] = {0, 0, 0, 0};
    const int lane = threadIdx.x & 63;
    const long long chunks = (R.V + 63) / 64;
    for (long long ch = blockIdx.x * 4LL + (threadIdx.x >> 6); ch < chunks; ch += gridDim.x * 4LL) {
        const long long n = ch * 64 + lane;
        const bool inside = n < R.V;
        const int idx = inside ? (int)n : (int)(R.V - 1);
        const uint32_t t = fdiv((uint32_t)idx, R.div_nx);
        const int x = idx - (int)t * R.nx;
        const uint32_t zz = fdiv(t, R.div_ny);
        const int y = (int)t - (int)zz * R.ny;
        const int z = (int)zz;
        const bool fluid = inside && !is_solid(R, x, y, z);
        const bool any_face = __ballot(fluid && (y == 0 || y == R.ny - 1 || z == 0 || z == R.nz - 1)) != 0;
        const bool any_pore = __ballot(fluid && near_pore(R, x, y, z)) != 0;
        const bool any_zone = __ballot(fluid && in_wall_zone(R, x)) != 0;
        const bool any_xface = __ballot(fluid && (x == 0 || x == R.nx - 1)) != 0;
        if (!fluid) continue;
        Rl f[Q];
        if (any_face && any_zone) gather19<S, G_GENERIC>(R, src, idx, x, y, z, f);
        else if (any_face) gather19<S, G_FACE>(R, src, idx, x, y, z, f);
        else if (any_pore) gather19<S, G_WALL>(R, src, idx, x, y, z, f);
        else if (any_zone) gather19<S, G_WALL_PLANE>(R, src, idx, x, y, z, f);
        else if (any_xface) gather19<S, G_FAST>(R, src, idx, x, y, z, f);
        else gather19<S, G_INTERIOR>(R, src, idx, x, y, z, f);
        for_pops([&](auto P) {
            constexpr int p = decltype(P)::value;
            // the stored number decoded as Codec::load does, then the rest value added in FP64
            double v = (double)(f[p] * (Rl(1) / C::template kScale<p>));
            if constexpr (C::deviation) v += w_of<double>(p) * R.rho0;
            acc[0] += v;
            if constexpr (cx_of(p) != 0) acc[1] += cx_of(p) * v;
            if constexpr (cy_of(p) != 0) acc[2] += cy_of(p) * v;
            if constexpr (cz_of(p) != 0) acc[3] += cz_of(p) * v;
        });
    }
    __shared__ double red[4][256 / 64];
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        double v = acc[k];
#pragma unroll
        for (int off = 32; off >= 1; off >>= 1) v += __shfl_xor(v, off, 64);
        if ((threadIdx.x & 63) == 0) red[k][threadIdx.x >> 6] = v;
    }
    __syncthreads();
    if (threadIdx.x < 4) {
        double v = 0;
        for (int w = 0; w < 256 / 64; ++w) v += red[threadIdx.x][w];
        partials[blockIdx.x * 4 + threadIdx.x] = v;
    }
}

__global__ __launch_bounds__(256) void k_conserved_final(const double* __restrict__ partials, int nblk,
                                                         double* __restrict__ out4) {
    __shared__ double red[4][256];
    double acc[4] = {0, 0, 0, 0};
    // thread t adds partials t, t + 256, t + 512, ... in that order; eight rows are loaded
    // before they are added, so that their latencies overlap
    for (int b0 = threadIdx.x; b0 < nblk; b0 += 256 * 8) {
        double v[8][4];
#pragma unroll
        for (int u = 0; u < 8; ++u) {
            const int b = b0 + u * 256;
#pragma unroll
            for (int k = 0; k < 4; ++k) v[u][k] = b < nblk ? partials[b * 4 + k] : 0.0;
        }
#pragma unroll
        for (int u = 0; u < 8; ++u) {
            if (b0 + u * 256 >= nblk) break;
#pragma unroll
            for (int k = 0; k < 4; ++k) acc[k] += v[u][k];
        }
    }
    for (int k = 0; k < 4; ++k) red[k][threadIdx.x] = acc[k];
    __syncthreads();
    for (int half = 128; half >= 1; half >>= 1) {
        if (threadIdx.x < half)
            for (int k = 0; k < 4; ++k) red[k][threadIdx.x] += red[k][threadIdx.x + half];
        __syncthreads();
    }
    if (threadIdx.x < 4) out4[threadIdx.x] = red[threadIdx.x][0];
}

// ---------------------------------------------------------------------------------
// Host launchers.
// ---------------------------------------------------------------------------------
template <int S, int BLOCK, bool NT, bool TH>
static hipError_t launch_sc_n(const Context& c, const void* src, void* dst, bool bump, hipStream_t s) {
    using T = typename Codec<S>::T;
    if (c.lat.mapping == MAP_FLAT2) {
        if constexpr (BLOCK >= 128 && BLOCK <= 512) {
            hipLaunchKernelGGL((k_stream_collide_2n<S, BLOCK, NT, TH>), dim3(c.lat.total_tiles), dim3(BLOCK), 0, s,
                               c.d_reps, c.lat.d_prefix, (int)c.reps.size(), (const T*)src, (T*)dst, c.d_state,
                               bump ? 1 : 0, c.lat_chunk);
            return hipGetLastError();
        } else {
            return hipErrorInvalidValue;  // two nodes per lane: blocks of 128 to 512 threads
        }
    }
    hipLaunchKernelGGL((k_stream_collide<S, BLOCK, NT, TH>), dim3(c.lat.total_tiles), dim3(BLOCK), 0, s,
                       c.d_reps, c.lat.d_prefix, (int)c.reps.size(), (const T*)src, (T*)dst, c.d_state,
                       bump ? 1 : 0, c.lat_chunk, c.lat.mapping);
    return hipGetLastError();
}

template <int S, int BLOCK, bool NT>
static hipError_t launch_pattern_n(const Context& c, const void* src, void* dst, hipStream_t s) {
    using T = typename Codec<S>::T;
    // the flat tile table of this block size (the rows mapping has other tiles)
    const LatticeLaunch* L = nullptr;
    for (const auto& l : c.lat_all)
        if (l.block == BLOCK && l.mapping == MAP_FLAT) L = &l;
    if (!L) return hipErrorInvalidValue;
    hipLaunchKernelGGL((k_pattern<S, BLOCK, NT>), dim3(L->total_tiles), dim3(BLOCK), 0, s, c.d_reps, L->d_prefix,
                       (int)c.reps.size(), (const T*)src, (T*)dst, c.lat_chunk);
    return hipGetLastError();
}

template <int S, int BLOCK>
static hipError_t launch_pattern_t(const Context& c, const void* src, void* dst, hipStream_t s) {
    return c.lat_nt ? launch_pattern_n<S, BLOCK, true>(c, src, dst, s) : launch_pattern_n<S, BLOCK, false>(c, src, dst, s);
}

template <int S>
static hipError_t launch_pattern_s(const Context& c, const void* src, void* dst, hipStream_t s) {
    switch (c.lat.block) {
        case 64: return launch_pattern_t<S, 64>(c, src, dst, s);
        case 128: return launch_pattern_t<S, 128>(c, src, dst, s);
        case 256: return launch_pattern_t<S, 256>(c, src, dst, s);
        case 512: return launch_pattern_t<S, 512>(c, src, dst, s);
        case 1024: return launch_pattern_t<S, 1024>(c, src, dst, s);
        default: return hipErrorInvalidValue;
    }
}

hipError_t launch_pattern(const Context& c, const void* src, void* dst, hipStream_t s) {
    switch (c.storage) {
        case LB_STORE_F64: return launch_pattern_s<LB_STORE_F64>(c, src, dst, s);
        case LB_STORE_F32: return launch_pattern_s<LB_STORE_F32>(c, src, dst, s);
        case LB_STORE_F16DEV: return launch_pattern_s<LB_STORE_F16DEV>(c, src, dst, s);
        case LB_STORE_BF16DEV: return launch_pattern_s<LB_STORE_BF16DEV>(c, src, dst, s);
        default: return hipErrorInvalidValue;
    }
}

template <int S, int BLOCK>
static hipError_t launch_sc_t(const Context& c, const void* src, void* dst, bool bump, hipStream_t s) {
    if (c.thermal) {
        // the thermal source reads the step counter, which must not move during the sweep
        if (bump) return hipErrorInvalidValue;
        return c.lat_nt ? launch_sc_n<S, BLOCK, true, true>(c, src, dst, false, s)
                        : launch_sc_n<S, BLOCK, false, true>(c, src, dst, false, s);
    }
    return c.lat_nt ? launch_sc_n<S, BLOCK, true, false>(c, src, dst, bump, s)
                    : launch_sc_n<S, BLOCK, false, false>(c, src, dst, bump, s);
}

template <int S>
static hipError_t launch_sc_s(const Context& c, const void* src, void* dst, bool bump, hipStream_t s) {
    switch (c.lat.block) {
        case 64: return launch_sc_t<S, 64>(c, src, dst, bump, s);
        case 128: return launch_sc_t<S, 128>(c, src, dst, bump, s);
        case 256: return launch_sc_t<S, 256>(c, src, dst, bump, s);
        case 512: return launch_sc_t<S, 512>(c, src, dst, bump, s);
        case 1024: return launch_sc_t<S, 1024>(c, src, dst, bump, s);
        default: return hipErrorInvalidValue;
    }
}

hipError_t launch_stream_collide(const Context& c, const void* src, void* dst, bool bump, hipStream_t s) {
    switch (c.storage) {
        case LB_STORE_F64: return launch_sc_s<LB_STORE_F64>(c, src, dst, bump, s);
        case LB_STORE_F32: return launch_sc_s<LB_STORE_F32>(c, src, dst, bump, s);
        case LB_STORE_F16DEV: return launch_sc_s<LB_STORE_F16DEV>(c, src, dst, bump, s);
        case LB_STORE_BF16DEV: return launch_sc_s<LB_STORE_BF16DEV>(c, src, dst, bump, s);
        default: return hipErrorInvalidValue;
    }
}

template <int S>
static hipError_t launch_init_t(const Context& c, int r, void* dst, const double* rho, const double* u,
                                const double* pops, hipStream_t s) {
    using T = typename Codec<S>::T;
    const int V = c.reps[r].V;
    hipLaunchKernelGGL((k_init<S>), dim3((V + 255) / 256), dim3(256), 0, s, c.d_reps, r, (T*)dst, rho, u,
                       pops);
    return hipGetLastError();
}

hipError_t launch_init(const Context& c, int r, void* dst, const double* rho, const double* u,
                       const double* pops, hipStream_t s) {
    switch (c.storage) {
        case LB_STORE_F64: return launch_init_t<LB_STORE_F64>(c, r, dst, rho, u, pops, s);
        case LB_STORE_F32: return launch_init_t<LB_STORE_F32>(c, r, dst, rho, u, pops, s);
        case LB_STORE_F16DEV: return launch_init_t<LB_STORE_F16DEV>(c, r, dst, rho, u, pops, s);
        case LB_STORE_BF16DEV: return launch_init_t<LB_STORE_BF16DEV>(c, r, dst, rho, u, pops, s);
        default: return hipErrorInvalidValue;
    }
}

template <int S>
static hipError_t launch_gather_t(const Context& c, int r, const void* src, int mode, long long node0,
                                  int count, double* out, hipStream_t s) {
    using T = typename Codec<S>::T;
    hipLaunchKernelGGL((k_gather<S>), dim3((count + 255) / 256), dim3(256), 0, s, c.d_reps, r,
                       (const T*)src, mode, node0, count, out);
    return hipGetLastError();
}

hipError_t launch_gather(const Context& c, int r, const void* src, int mode, long long node0, int count,
                         double* out, hipStream_t s) {
    switch (c.storage) {
        case LB_STORE_F64: return launch_gather_t<LB_STORE_F64>(c, r, src, mode, node0, count, out, s);
        case LB_STORE_F32: return launch_gather_t<LB_STORE_F32>(c, r, src, mode, node0, count, out, s);
        case LB_STORE_F16DEV: return launch_gather_t<LB_STORE_F16DEV>(c, r, src, mode, node0, count, out, s);
        case LB_STORE_BF16DEV: return launch_gather_t<LB_STORE_BF16DEV>(c, r, src, mode, node0, count, out, s);
        default: return hipErrorInvalidValue;
    }
}

template <int S>
static hipError_t launch_conserved_t(const Replica& R, const void* src, double* partials, int nblk, double* out4,
                                     hipStream_t s) {
    using T = typename Codec<S>::T;
    hipLaunchKernelGGL((k_conserved_partial<S>), dim3(nblk), dim3(256), 0, s, R, (const T*)src, partials);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(k_conserved_final, dim3(1), dim3(256), 0, s, (const double*)partials, nblk, out4);
    return hipGetLastError();
}

hipError_t launch_conserved_desc(const Replica& R, int storage, const void* src, double* partials, int nblk,
                                 double* out4, hipStream_t s) {
    switch (storage) {
        case LB_STORE_F64: return launch_conserved_t<LB_STORE_F64>(R, src, partials, nblk, out4, s);
        case LB_STORE_F32: return launch_conserved_t<LB_STORE_F32>(R, src, partials, nblk, out4, s);
        case LB_STORE_F16DEV: return launch_conserved_t<LB_STORE_F16DEV>(R, src, partials, nblk, out4, s);
        case LB_STORE_BF16DEV: return launch_conserved_t<LB_STORE_BF16DEV>(R, src, partials, nblk, out4, s);
        default: return hipErrorInvalidValue;
    }
}

hipError_t launch_conserved(const Context& c, int r, const void* src, double* out4, hipStream_t s) {
    // one block of partial sums per 4096 nodes (16 chunks of 64 nodes per wave), and at least
    // 2048 blocks (8192 waves) so that a small box still has loads in flight everywhere: a
    // 512^3 box took 2.6 ms with 2048 blocks and 1.8 ms with 32768
    const long long want = (c.reps[r].V + 4095) / 4096;
    const int nblk = (int)std::min<long long>(c.partial_blocks, std::max<long long>(2048, want));
    return launch_conserved_desc(c.reps[r], c.storage, src, c.d_partials, nblk, out4, s);
}

}  // namespace lbmd

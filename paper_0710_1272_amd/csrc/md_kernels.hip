// md_kernels.hip -- spread, trilinear coupling and observable kernels, and the bead kernel's host side (gfx950).
//
// k_spread: step 3, S_p = -(w_p / c_s^2) Fbar . c_p added to the post-collision
// populations of each leader's node (S_p eq.); nodes are unique within a replica,
// so there are no write conflicts and no floating-point atomics.
#include <algorithm>
#include <utility>

#include "md_bead.hpp"

namespace lbmd {

template <int S>
__global__ __launch_bounds__(256) void k_spread(const Replica* __restrict__ reps,
                                                BeadPtrs<typename MDReal<S>::type> b,
                                                typename Codec<S>::T* __restrict__ dst, RunState* st,
                                                int bump_step) {
    using Rl = typename Codec<S>::R;
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (bump_step && i == 0) st->step += 1;
    if (i >= b.ntot) return;
    // one round trip for everything a leader needs: where, stride, force
    const long long at = b.agg_at[i];
    const long long PS = b.agg_at[b.ntot + i];
    const Rl F[3] = {(Rl)b.agg_f[i], (Rl)b.agg_f[b.ntot + i], (Rl)b.agg_f[2 * b.ntot + i]};
    if (at < 0) return;
    add_reaction<S>(dst + at, PS, F);
}

__global__ void k_bump(RunState* st) { st->step += 1; }

// Small read-outs straight into pinned host memory, the run state with them: one launch and one
// synchronisation a call.  Copy commands instead (one per component of each bead array, each
// with a synchronisation of its own) took 130 us for the bead state of 100 beads, 10 us of it
// the copies themselves; this takes 16 us.
//   beads:    out = [n][3] positions, [n][3] velocities
//   coupling: out = [n][3] u_i, [n][3] Fbar_i, [n] node index
//   transloc: out = the replica's 8 diagnostics
template <class Real>
__global__ __launch_bounds__(256) void k_readout(BeadPtrs<Real> b, const RunState* __restrict__ st, int what,
                                                 int replica, int b0, int n, double* __restrict__ out,
                                                 RunState* __restrict__ out_st) {
    const int i = blockIdx.x * 256 + threadIdx.x;
    if (i == 0) *out_st = *st;
    const int NT = b.ntot;
    if (what == READ_TRANSLOC) {
        if (i < 8) out[i] = b.diag[8 * replica + i];
        return;
    }
    if (i >= n || what == READ_STATE) return;
    const int g = b0 + i;
#pragma unroll
    for (int c = 0; c < 3; ++c) {
        out[3 * i + c] = what == READ_BEADS ? b.r[c * NT + g] : (double)b.u[c * NT + g];
        out[3 * (n + i) + c] = what == READ_BEADS ? (double)b.v[c * NT + g] : (double)b.fbar[c * NT + g];
    }
    if (what == READ_COUPLING) out[6 * n + i] = (double)b.node[g];
}

// Before a run of one-launch steps: the nodes of the
// first step are marked for its sweep and the step counter is copied to where that step reads it.
template <class Real>
__global__ __launch_bounds__(256) void k_mark(const Replica* __restrict__ reps, BeadPtrs<Real> b,
                                              const RunState* __restrict__ st, Marks marks, long long* step_of) {
    const Replica& R = reps[0];
    const long long step = st->step;
    if (threadIdx.x == 0) *step_of = step;
    const int n[3] = {R.nx, R.ny, R.nz}, fs[3] = {R.fs[0], R.fs[1], R.fs[2]};
    const int nb = R.n_beads, b0 = R.bead0, NT = b.ntot;
    for (int pass = 0; pass < 2; ++pass) {
        for (int i = threadIdx.x; i < nb; i += blockDim.x) {
            const double r[3] = {b.r[b0 + i], b.r[NT + b0 + i], b.r[2 * NT + b0 + i]};
            int g[3];
            ngp3(n, fs, r, g);
            if (is_solid(R, g[0], g[1], g[2])) continue;
            const int at = g[0] + R.nx * (g[1] + R.ny * g[2]);
            const int c = at >> 6;
            if (pass == 0) {
                marks.stamp[c] = mark_stamp(step);
                marks.mask[c] = 0;
            } else {
                atomicOr(&marks.mask[c], 1ull << (at & 63));
            }
        }
        if (pass == 0) {
            stores_done();
            __syncthreads();
        }
    }
}

// Observable record of the translocation analysis (Sec. III), one workgroup per replica,
// after the bead step and before the step counter moves: when (step + 1) is a multiple of
// obs_every, a row (step + 1, N_T, S_H = m gamma sum v.u, S_E = sum F_drive.v over beads on
// pore nodes, K = m/2 sum v^2, R_U^2, R_T^2, x of the centre of mass) is appended to the
// replica's record (rows beyond the capacity are counted, not kept).  FP64 sums in a fixed
// order; positions are taken relative to the pore centre, which keeps the second moments of
// the radii of gyration small.
template <class Real>
__global__ __launch_bounds__(256) void k_observe(const Replica* __restrict__ reps, BeadPtrs<Real> b,
                                                 const RunState* __restrict__ st, double mass_gamma,
                                                 double half_mass, double f_drive, int no_hydro) {
    __shared__ double red[16 * 12];
    const long long step = st->step;
    if ((step + 1) % b.obs_every != 0) return;
    const Replica& R = reps[blockIdx.x];
    const int n = R.n_beads;
    if (n == 0) return;
    const Geom GM = load_geom(R);
    const int b0 = R.bead0, NT = b.ntot;
    const double xmid = R.xmid;
    const double ref[3] = {xmid, 0.5 * R.ny, 0.5 * R.nz};
    // N_T, S_H, S_E, K, sum d (3), sum d^2, and over the translocated beads sum d (3), sum d^2
    double o[12] = {0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0};
    for (int i = threadIdx.x; i < n; i += blockDim.x) {
        const int g = b0 + i;
        double r[3], v[3], u[3], d[3], d2 = 0.0, vu = 0.0, vv = 0.0;
#pragma unroll
        for (int c = 0; c < 3; ++c) {
            r[c] = b.r[c * NT + g];
            v[c] = (double)b.v[c * NT + g];
            u[c] = no_hydro ? 0.0 : (double)b.u[c * NT + g];
            d[c] = r[c] - ref[c];
            d2 += d[c] * d[c];
            vu += v[c] * u[c];
            vv += v[c] * v[c];
        }
        bool pore = false;
#pragma unroll
        for (int w = 0; w < LB_MAX_WALLS; ++w) {
            if (w >= GM.n_walls) break;
            pore = pore || (pore_open(GM.wall[w]) &&
                            wall_pore_node<true, true>(GM, wall_bounds(wall_ints(GM, GM.wall[w])), GM.wall[w], r));
        }
        const bool tr = r[0] > xmid;
        o[0] += tr ? 1.0 : 0.0;
        o[1] += mass_gamma * vu;
        o[2] += pore ? f_drive * v[0] : 0.0;
        o[3] += half_mass * vv;
        o[4] += d[0];
        o[5] += d[1];
        o[6] += d[2];
        o[7] += d2;
        if (tr) {
            o[8] += d[0];
            o[9] += d[1];
            o[10] += d[2];
            o[11] += d2;
        }
    }
    block_sums<12>(o, red, blockDim.x);
    if (threadIdx.x != 0) return;
    double* rec = b.obs + (size_t)blockIdx.x * ((size_t)b.obs_cap + 1) * 8;
    const double cnt = rec[0];
    if (cnt < (double)b.obs_cap) {
        const double nT = o[0], nU = (double)n - o[0];
        double rT = 0.0, rU = 0.0;
        if (nT > 0) {
            const double c0 = o[8] / nT, c1 = o[9] / nT, c2 = o[10] / nT;
            rT = fmax(o[11] / nT - (c0 * c0 + c1 * c1 + c2 * c2), 0.0);
        }
        if (nU > 0) {
            const double c0 = (o[4] - o[8]) / nU, c1 = (o[5] - o[9]) / nU, c2 = (o[6] - o[10]) / nU;
            rU = fmax((o[7] - o[11]) / nU - (c0 * c0 + c1 * c1 + c2 * c2), 0.0);
        }
        double* row = rec + (size_t)(1 + (long long)cnt) * 8;
        row[0] = (double)(step + 1);
        row[1] = nT;
        row[2] = o[1];
        row[3] = o[2];
        row[4] = o[3];
        row[5] = rU;
        row[6] = rT;
        row[7] = ref[0] + o[4] / n;
    }
    rec[0] = cnt + 1.0;
}

// Trilinear stencil of a position: nodes floor(r_a) + {0, 1} per axis (periodic axes wrap,
// a node beyond a free-slip face is the face node) and the 1-D weights 1 - f, f.
__device__ __forceinline__ void trilinear_axes(const Replica& R, const double* r, int lo[3][2], double w1[3][2]) {
    const int n[3] = {R.nx, R.ny, R.nz};
    const int fs[3] = {R.fs[0], R.fs[1], R.fs[2]};
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        double t = floor(r[a]);
        if (!(t >= -1e9 && t <= 1e9)) t = 0.0;  // non-finite or absurd
        const double fr = r[a] - t;
        w1[a][0] = 1.0 - fr;
        w1[a][1] = fr;
#pragma unroll
        for (int s = 0; s < 2; ++s) {
            int k = (int)t + s;
            if (!fs[a]) {
                k %= n[a];
                if (k < 0) k += n[a];
            } else {
                k = k < 0 ? 0 : (k > n[a] - 1 ? n[a] - 1 : k);
            }
            lo[a][s] = k;
        }
    }
}

// Step 1 with the trilinear stencil, one thread per bead: u_i = sum_c w_c u(x_c) over the 8
// surrounding nodes (u = 0 on solid ones), from the pre-collision populations; the
// start-of-step position is kept for the spread and the bead has no single node (-1).
template <class Real>
__global__ __launch_bounds__(256) void k_interp_tri(const Replica* __restrict__ reps, BeadPtrs<Real> b,
                                                    const void* cur, int storage) {
    // eight lanes a bead, lane c of the group owning stencil node c: the 8 x 19 population
    // reads of a bead are issued by 8 lanes at once instead of one after the other
    const int t = blockIdx.x * blockDim.x + threadIdx.x;
    const int i = t >> 3, c = t & 7;
    if (i >= b.ntot) return;  // whole groups of eight leave together
    const int NT = b.ntot;
    const Replica& R = reps[b.rep_of[i]];
    const double r[3] = {b.r[i], b.r[NT + i], b.r[2 * NT + i]};
    int lo[3][2];
    double w1[3][2];
    trilinear_axes(R, r, lo, w1);
    const int g[3] = {lo[0][c & 1], lo[1][(c >> 1) & 1], lo[2][(c >> 2) & 1]};
    double part[3] = {0.0, 0.0, 0.0};
    if (!is_solid(R, g[0], g[1], g[2])) {
        const double w = w1[0][c & 1] * w1[1][(c >> 1) & 1] * w1[2][(c >> 2) & 1];
        Real uc[3];
        std::conditional_t<sizeof(Real) == 8, uint64_t, uint32_t> raw[Q];
        load_node<Real>(storage, R, cur, g, raw);
        node_velocity<Real>(storage, (Real)R.rho0, raw, uc);
#pragma unroll
        for (int a = 0; a < 3; ++a) part[a] = w * (double)uc[a];
    }
    // the group's first lane adds the eight parts in stencil order (a solid node adds 0)
    double u[3] = {0.0, 0.0, 0.0};
#pragma unroll
    for (int k = 0; k < 8; ++k)
#pragma unroll
        for (int a = 0; a < 3; ++a) u[a] += __shfl(part[a], k, 8);
    if (c == 0) {
#pragma unroll
        for (int a = 0; a < 3; ++a) {
            b.u[a * NT + i] = (Real)u[a];
            b.rs[a * NT + i] = r[a];
        }
        b.node[i] = -1;
    }
}

// Step 3 with the trilinear stencil, eight lanes a bead (FP32 and FP64 storage): -w_c (w_p /
// c_s^2) Fbar . c_p added to the post-collision populations of every fluid node of the
// start-of-step stencil.  Stencils of nearby beads share nodes, so the adds are atomic (their
// order, and so the last bits of FP32 sums, can differ between runs).  16-bit storage takes
// the fixed-point spread below.
template <int S>
__global__ __launch_bounds__(256) void k_spread_tri(const Replica* __restrict__ reps,
                                                    BeadPtrs<typename MDReal<S>::type> b,
                                                    typename Codec<S>::T* __restrict__ dst, RunState* st,
                                                    int bump_step) {
    using C = Codec<S>;
    using Rl = typename C::R;
    // eight lanes a bead, lane c adding to stencil node c
    const int t = blockIdx.x * blockDim.x + threadIdx.x;
    const int i = t >> 3, c = t & 7;
    if (bump_step && t == 0) st->step += 1;
    if (i >= b.ntot) return;
    const int NT = b.ntot;
    const Replica& R = reps[b.rep_of[i]];
    const double r[3] = {b.rs[i], b.rs[NT + i], b.rs[2 * NT + i]};
    const Rl F[3] = {(Rl)b.fbar[i], (Rl)b.fbar[NT + i], (Rl)b.fbar[2 * NT + i]};
    int lo[3][2];
    double w1[3][2];
    trilinear_axes(R, r, lo, w1);
    const long long PS = R.S;  // population plane stride
    {
        const int g[3] = {lo[0][c & 1], lo[1][(c >> 1) & 1], lo[2][(c >> 2) & 1]};
        if (is_solid(R, g[0], g[1], g[2])) return;
        const Rl w = (Rl)(w1[0][c & 1] * w1[1][(c >> 1) & 1] * w1[2][(c >> 2) & 1]);
        typename C::T* base = dst + R.pop_base + g[0] + (long long)R.nx * (g[1] + (long long)R.ny * g[2]);
        for_pops([&](auto P) {
            constexpr int p = decltype(P)::value;
            if constexpr (p != 0) {
                Rl fc = 0;
                if constexpr (cx_of(p) != 0) fc += Rl(cx_of(p)) * F[0];
                if constexpr (cy_of(p) != 0) fc += Rl(cy_of(p)) * F[1];
                if constexpr (cz_of(p) != 0) fc += Rl(cz_of(p)) * F[2];
                const Rl src = -Rl(3) * w_of<Rl>(p) * fc * w;
                (void)unsafeAtomicAdd(&base[(long long)p * PS], src);
            }
        });
    }
}

// Deterministic form of step 3 with the trilinear stencil.  Floating-point adds depend on
// their order, and the order of atomic adds changes from run to run; integer adds do not.
// Each contribution -w_c (w_p / c_s^2) Fbar . c_p is rounded once to a multiple of 2^-48
// (in FP64) and added as a 64-bit integer into a table entry of its node; a second pass adds
// each node's exact sums to its populations (one rounding each) and empties the entry.
// A contribution is at most 2^9 in magnitude (larger ones are dropped and flagged), so a
// node's signed 64-bit sum cannot overflow below 2^(63 - 48 - 9) = 64 contributions; a node
// collects one from each bead whose 8-node stencil holds it, a handful at WCA densities.
constexpr double kFxScale = 281474976710656.0;  // 2^48
constexpr double kFxLimit = 512.0;

// slot of a key: the splitmix64 finaliser (Steele, Lea and Flood, OOPSLA 2014) as a hash
__device__ __forceinline__ unsigned fx_hash(unsigned long long k, unsigned mask) {
    k ^= k >> 30;
    k *= 0xbf58476d1ce4e5b9ull;
    k ^= k >> 27;
    k *= 0x94d049bb133111ebull;
    k ^= k >> 31;
    return (unsigned)k & mask;
}

// Pass 1: the table entry of every fluid node of the start-of-step
// stencil (linear probing; the table holds at most 8 nodes a bead in 16 slots a bead, so a
// free slot is always found), then 18 integer atomic adds into it; eight lanes a bead.
template <class Real>
__global__ __launch_bounds__(64) void k_spread_tri_fx(const Replica* __restrict__ reps, BeadPtrs<Real> b,
                                                      RunState* st) {
    // eight lanes a bead, lane c inserting stencil node c (integer sums: the order of the
    // lanes' adds does not matter)
    const int lane8 = blockIdx.x * blockDim.x + threadIdx.x;
    const int i = lane8 >> 3, c = lane8 & 7;
    if (i >= b.ntot) return;
    const int NT = b.ntot;
    const Replica& R = reps[b.rep_of[i]];
    const double r[3] = {b.rs[i], b.rs[NT + i], b.rs[2 * NT + i]};
    const double F[3] = {(double)b.fbar[i], (double)b.fbar[NT + i], (double)b.fbar[2 * NT + i]};
    int lo[3][2];
    double w1[3][2];
    trilinear_axes(R, r, lo, w1);
    const unsigned mask = b.hcap - 1;
    unsigned flags = 0;
    do {
        const int g[3] = {lo[0][c & 1], lo[1][(c >> 1) & 1], lo[2][(c >> 2) & 1]};
        if (is_solid(R, g[0], g[1], g[2])) break;
        const double w = w1[0][c & 1] * w1[1][(c >> 1) & 1] * w1[2][(c >> 2) & 1];
        const unsigned long long key =
            (unsigned long long)(R.pop_base + g[0] + (long long)R.nx * (g[1] + (long long)R.ny * g[2])) + 1ull;
        unsigned h = fx_hash(key, mask);
        bool found = false;
        for (unsigned t = 0; t <= mask; ++t) {
            const unsigned long long old = atomicCAS(&b.hkey[h], 0ull, key);
            if (old == 0ull) b.hrep[h] = b.rep_of[i];  // this thread opened the entry
            if (old == 0ull || old == key) {
                found = true;
                break;
            }
            h = (h + 1) & mask;
        }
        if (!found) {
            flags |= LB_ERR_NONFINITE;
            break;
        }
        for_pops([&](auto P) {
            constexpr int p = decltype(P)::value;
            if constexpr (p != 0) {
                double fc = 0.0;
                if constexpr (cx_of(p) != 0) fc += cx_of(p) * F[0];
                if constexpr (cy_of(p) != 0) fc += cy_of(p) * F[1];
                if constexpr (cz_of(p) != 0) fc += cz_of(p) * F[2];
                const double src = -3.0 * w_of<double>(p) * fc * w;
                if (!(fabs(src) <= kFxLimit)) {
                    flags |= LB_ERR_NONFINITE;
                } else {
                    const long long q = (long long)rint(src * kFxScale);
                    (void)atomicAdd((unsigned long long*)&b.hsum[(size_t)(p - 1) * b.hcap + h], (unsigned long long)q);
                }
            }
        });
    } while (false);
    if (flags) atomicOr(&st->err, flags);
}

// Pass 2, one thread per table slot: adds an occupied entry's sums to the post-collision
// populations of its node (each node has one entry, so plain read-modify-writes) and empties
// the entry for the next step.
template <int S>
__global__ __launch_bounds__(256) void k_spread_fx_apply(const Replica* __restrict__ reps,
                                                         BeadPtrs<typename MDReal<S>::type> b,
                                                         typename Codec<S>::T* __restrict__ dst, RunState* st,
                                                         int bump_step) {
    using C = Codec<S>;
    using Rl = typename C::R;
    const unsigned h = blockIdx.x * blockDim.x + threadIdx.x;
    if (bump_step && h == 0) st->step += 1;
    if (h >= b.hcap) return;
    const unsigned long long key = b.hkey[h];
    if (key == 0ull) return;
    const long long PS = reps[b.hrep[h]].S;  // population plane stride
    typename C::T* __restrict__ base = dst + (long long)(key - 1ull);
    for_pops([&](auto P) {
        constexpr int p = decltype(P)::value;
        if constexpr (p != 0) {
            long long* cell = &b.hsum[(size_t)(p - 1) * b.hcap + h];
            const long long q = *cell;
            if (q != 0) {
                const Rl add = (Rl)((double)q * (1.0 / kFxScale));
                base[(long long)p * PS] = C::template store<p>(C::template load<p>(base[(long long)p * PS]) + add);
                *cell = 0;
            }
        }
    });
    b.hkey[h] = 0ull;
}

// ---------------------------------------------------------------------------------
// Host launchers.
// ---------------------------------------------------------------------------------
int md_max_beads(bool rigid) {
    const size_t per = 6 * sizeof(double) + sizeof(int) + 1 + (rigid ? 15 * sizeof(double) : 0);
    const size_t nmax = (size_t)(160 * 1024 - kMDStaticLds) / per / 64 * 64;
    return (int)std::min<size_t>(nmax, 4096);
}

int md_default_lanes(int max_beads) {
    // lanes per bead: up to ~512 threads, so that each SIMD has two waves to interleave
    // (measured faster than one wave per SIMD for 100 beads, although the per-bead work
    // is repeated by every lane of a group); beyond 256 beads one lane per bead
    const int m = std::max(max_beads, 1);
    if (m <= 32) return 16;
    if (m <= 64) return 8;
    if (m <= 128) return 4;
    if (m <= 256) return 2;
    return 1;
}

bool md_lanes_valid(int lanes, int max_beads) {
    if (lanes == 1) return max_beads <= 4096;
    if (lanes == 2) return max_beads <= 512;
    return (lanes == 4 || lanes == 8 || lanes == 16) && (long long)lanes * max_beads <= 512;
}

template <class Real>
static hipError_t launch_md_r(const Context& c, const void* cur, int mode, const StepCount& at, hipStream_t s) {
    bool any_periodic = false;
    for (const Replica& R : c.reps)
        if (R.n_beads > 0 && (!R.fs[0] || !R.fs[1] || !R.fs[2])) any_periodic = true;
    if (c.md.rigid || c.md.kappa_phi != 0.0)
        return any_periodic ? launch_md_g<Real, true, true>(c, cur, mode, at, s)
                            : launch_md_g<Real, false, true>(c, cur, mode, at, s);
    return any_periodic ? launch_md_g<Real, true, false>(c, cur, mode, at, s)
                        : launch_md_g<Real, false, false>(c, cur, mode, at, s);
}

hipError_t launch_md(const Context& c, const void* cur, int mode, hipStream_t s, const StepCount& at) {
    if (c.storage == LB_STORE_F64) return launch_md_r<double>(c, cur, mode, at, s);
    return launch_md_r<float>(c, cur, mode, at, s);
}

// One lane a bead (more than 256 beads by default) stays with separate launches: the bead step then
// needs every register, and beside the sweep's code it spills (400 beads in 96x48x48, FP32: 90.9 us a
// step in one launch, 83.8 apart; in 128x64x64 200 beads, two lanes each: 51.6 and 53.4; 100 beads
// 35.8 and 42.0, rigid 67.3 and 70.5; 12 beads in 64x32x32: 26.9 and 31.4).
bool step_one_fits(const Context& c) {
    if (!c.one_launch || !c.marks[0].stamp || c.obs_every > 0) return false;
    return step_one_lanes(c.md_lanes > 0 ? c.md_lanes : md_default_lanes(c.max_beads), c.max_beads);
}

bool step_one_lanes(int lanes, int max_beads) { return lanes > 1 && md_block(lanes, std::max(max_beads, 1)) <= 512; }

hipError_t prepare_step_one(const Context& c) {
    const bool poly = c.md.rigid || c.md.kappa_phi != 0.0;
    switch (c.storage) {
        case LB_STORE_F64: return poly ? prepare_step_one_g<LB_STORE_F64, true>() : prepare_step_one_g<LB_STORE_F64, false>();
        case LB_STORE_F32: return poly ? prepare_step_one_g<LB_STORE_F32, true>() : prepare_step_one_g<LB_STORE_F32, false>();
        case LB_STORE_F16DEV:
            return poly ? prepare_step_one_g<LB_STORE_F16DEV, true>() : prepare_step_one_g<LB_STORE_F16DEV, false>();
        case LB_STORE_BF16DEV:
            return poly ? prepare_step_one_g<LB_STORE_BF16DEV, true>() : prepare_step_one_g<LB_STORE_BF16DEV, false>();
        default: return hipErrorNotSupported;
    }
}

hipError_t launch_step_one(const Context& c, int cur, bool last, hipStream_t s) {
    const bool poly = c.md.rigid || c.md.kappa_phi != 0.0;
    switch (c.storage) {
        case LB_STORE_F64:
            return poly ? launch_step_one_g<LB_STORE_F64, true>(c, cur, last, s) : launch_step_one_g<LB_STORE_F64, false>(c, cur, last, s);
        case LB_STORE_F32:
            return poly ? launch_step_one_g<LB_STORE_F32, true>(c, cur, last, s) : launch_step_one_g<LB_STORE_F32, false>(c, cur, last, s);
        case LB_STORE_F16DEV:
            return poly ? launch_step_one_g<LB_STORE_F16DEV, true>(c, cur, last, s)
                        : launch_step_one_g<LB_STORE_F16DEV, false>(c, cur, last, s);
        case LB_STORE_BF16DEV:
            return poly ? launch_step_one_g<LB_STORE_BF16DEV, true>(c, cur, last, s)
                        : launch_step_one_g<LB_STORE_BF16DEV, false>(c, cur, last, s);
        default: return hipErrorNotSupported;
    }
}

template <class Real>
static hipError_t launch_mark_t(const Context& c, int cur, hipStream_t s) {
    const BeadPtrs<Real> b = *(const BeadPtrs<Real>*)c.bead_ptrs;
    hipLaunchKernelGGL((k_mark<Real>), dim3(1), dim3(256), 0, s, c.d_reps, b, c.d_state,
                       c.marks[cur], &c.d_state->step_of[cur]);
    return hipGetLastError();
}

hipError_t launch_mark(const Context& c, int cur, hipStream_t s) {
    return c.storage == LB_STORE_F64 ? launch_mark_t<double>(c, cur, s) : launch_mark_t<float>(c, cur, s);
}

template <int S>
static hipError_t launch_spread_t(const Context& c, void* dst, bool bump, hipStream_t s) {
    using Real = typename MDReal<S>::type;
    const BeadPtrs<Real> b = *(const BeadPtrs<Real>*)c.bead_ptrs;
    // 64 threads a block: each leader's 18 read-modify-writes miss the caches when the
    // sweep streamed the populations past them, and more compute units keep more of
    // these misses in flight
    const int grid = (c.ntot_beads + 63) / 64;
    hipLaunchKernelGGL((k_spread<S>), dim3(grid > 0 ? grid : 1), dim3(64), 0, s, c.d_reps, b,
                       (typename Codec<S>::T*)dst, c.d_state, bump ? 1 : 0);
    return hipGetLastError();
}

template <int S>
static hipError_t launch_spread_tri_t(const Context& c, void* dst, bool bump, hipStream_t s) {
    using Real = typename MDReal<S>::type;
    const BeadPtrs<Real> b = *(const BeadPtrs<Real>*)c.bead_ptrs;
    // eight lanes a bead in 64-thread blocks, as for the nearest-node spread
    const int grid = (8 * c.ntot_beads + 63) / 64;
    hipLaunchKernelGGL((k_spread_tri<S>), dim3(grid > 0 ? grid : 1), dim3(64), 0, s, c.d_reps, b,
                       (typename Codec<S>::T*)dst, c.d_state, bump ? 1 : 0);
    return hipGetLastError();
}

template <class Real>
static hipError_t launch_interp_tri_t(const Context& c, const void* cur, hipStream_t s) {
    const BeadPtrs<Real> b = *(const BeadPtrs<Real>*)c.bead_ptrs;
    // eight lanes a bead in 64-thread blocks: each bead's 8 x 19 population reads may miss
    // the caches, and more compute units keep more misses in flight
    const int grid = (8 * c.ntot_beads + 63) / 64;
    hipLaunchKernelGGL((k_interp_tri<Real>), dim3(grid > 0 ? grid : 1), dim3(64), 0, s, c.d_reps, b, cur,
                       c.storage);
    return hipGetLastError();
}

hipError_t launch_interp_trilinear(const Context& c, const void* cur, hipStream_t s) {
    if (c.ntot_beads == 0) return hipSuccess;
    return c.storage == LB_STORE_F64 ? launch_interp_tri_t<double>(c, cur, s)
                                     : launch_interp_tri_t<float>(c, cur, s);
}

template <int S>
static hipError_t launch_spread_fx_t(const Context& c, void* dst, bool bump, hipStream_t s) {
    using Real = typename MDReal<S>::type;
    const BeadPtrs<Real> b = *(const BeadPtrs<Real>*)c.bead_ptrs;
    const int grid = (8 * c.ntot_beads + 63) / 64;  // eight lanes a bead
    hipLaunchKernelGGL((k_spread_tri_fx<Real>), dim3(grid > 0 ? grid : 1), dim3(64), 0, s, c.d_reps, b, c.d_state);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL((k_spread_fx_apply<S>), dim3((b.hcap + 255) / 256), dim3(256), 0, s, c.d_reps, b,
                       (typename Codec<S>::T*)dst, c.d_state, bump ? 1 : 0);
    return hipGetLastError();
}

hipError_t launch_spread(const Context& c, void* dst, bool bump, hipStream_t s) {
    // the trilinear spread in fixed point when asked for reproducible results, and always in
    // 16-bit storage: there a floating-point add into one element is a compare-and-swap loop on
    // its 32-bit word, and the integer atomics and one read-modify-write per node took 23 us
    // against 44 us on 128x64x64 (N = 100)
    const bool half = c.storage == LB_STORE_F16DEV || c.storage == LB_STORE_BF16DEV;
    if (c.md.stencil == LB_STENCIL_TRILINEAR && (c.deterministic || half)) {
        switch (c.storage) {
            case LB_STORE_F64: return launch_spread_fx_t<LB_STORE_F64>(c, dst, bump, s);
            case LB_STORE_F32: return launch_spread_fx_t<LB_STORE_F32>(c, dst, bump, s);
            case LB_STORE_F16DEV: return launch_spread_fx_t<LB_STORE_F16DEV>(c, dst, bump, s);
            case LB_STORE_BF16DEV: return launch_spread_fx_t<LB_STORE_BF16DEV>(c, dst, bump, s);
            default: return hipErrorInvalidValue;
        }
    }
    if (c.md.stencil == LB_STENCIL_TRILINEAR) {
        switch (c.storage) {
            case LB_STORE_F64: return launch_spread_tri_t<LB_STORE_F64>(c, dst, bump, s);
            case LB_STORE_F32: return launch_spread_tri_t<LB_STORE_F32>(c, dst, bump, s);
            default: return hipErrorInvalidValue;  // 16-bit storage took the fixed-point path
        }
    }
    switch (c.storage) {
        case LB_STORE_F64: return launch_spread_t<LB_STORE_F64>(c, dst, bump, s);
        case LB_STORE_F32: return launch_spread_t<LB_STORE_F32>(c, dst, bump, s);
        case LB_STORE_F16DEV: return launch_spread_t<LB_STORE_F16DEV>(c, dst, bump, s);
        case LB_STORE_BF16DEV: return launch_spread_t<LB_STORE_BF16DEV>(c, dst, bump, s);
        default: return hipErrorInvalidValue;
    }
}

template <class Real>
static hipError_t launch_observe_t(const Context& c, bool no_hydro, hipStream_t s) {
    const BeadPtrs<Real> b = *(const BeadPtrs<Real>*)c.bead_ptrs;
    hipLaunchKernelGGL((k_observe<Real>), dim3((unsigned)c.reps.size()), dim3(256), 0, s, c.d_reps, b, c.d_state,
                       c.md.mass * c.md.gamma, 0.5 * c.md.mass, c.md.f_drive, no_hydro ? 1 : 0);
    return hipGetLastError();
}

hipError_t launch_observe(const Context& c, bool no_hydro, hipStream_t s) {
    if (c.obs_every <= 0 || c.ntot_beads == 0) return hipSuccess;
    return c.storage == LB_STORE_F64 ? launch_observe_t<double>(c, no_hydro, s)
                                     : launch_observe_t<float>(c, no_hydro, s);
}

template <class Real>
static hipError_t launch_readout_t(const Context& c, int what, int r, double* out, RunState* out_st, hipStream_t s) {
    const BeadPtrs<Real> b = *(const BeadPtrs<Real>*)c.bead_ptrs;
    const Replica& R = c.reps[r];
    const int grid = what == READ_BEADS || what == READ_COUPLING ? (R.n_beads + 255) / 256 : 1;
    hipLaunchKernelGGL((k_readout<Real>), dim3(grid > 0 ? grid : 1), dim3(256), 0, s, b, c.d_state, what, r, R.bead0,
                       R.n_beads, out, out_st);
    return hipGetLastError();
}

hipError_t launch_readout(const Context& c, int what, int r, double* out, RunState* out_st, hipStream_t s) {
    return c.storage == LB_STORE_F64 ? launch_readout_t<double>(c, what, r, out, out_st, s)
                                     : launch_readout_t<float>(c, what, r, out, out_st, s);
}

hipError_t launch_bump(const Context& c, hipStream_t s) {
    hipLaunchKernelGGL(k_bump, dim3(1), dim3(1), 0, s, c.d_state);
    return hipGetLastError();
}

}  // namespace lbmd

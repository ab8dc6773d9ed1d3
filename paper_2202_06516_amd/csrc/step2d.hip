// step2d.hip -- the single-launch D2Q9 step (step2d.hpp): kernels and launches.
#include <hip/hip_runtime.h>

#include <type_traits>

#include "lbm.h"
#include "fused.hpp"
#include "step2d.hpp"

namespace lbm {

namespace {

typedef D2Q9 L2;

constexpr int halo_of(int model) { return model == M2_CHEM ? 6 : (model == M2_PSEUDO ? 1 : 2); }

__device__ __forceinline__ int wrap_any(int v, int n) {
    v %= n;
    return v < 0 ? v + n : v;
}

// workgroup id -> tile, contiguous runs per XCD
__device__ __forceinline__ unsigned tile_slot(unsigned t, unsigned n) {
    const unsigned q = n >> 3, r = n & 7u, xcd = t & 7u, loc = t >> 3;
    return (xcd < r ? xcd * (q + 1) : r * (q + 1) + (xcd - r) * q) + loc;
}

template <int TW, int TH, int NT, int H>
__global__ void __launch_bounds__(NT) k_tiles2d_flags(Tile2d* __restrict__ tiles, const uint8_t* __restrict__ cls) {
    const Tile2d t = tiles[blockIdx.x];
    constexpr int RW = TW + 2 * H, RH = TH + 2 * H;
    bool any = false;
    for (int i = threadIdx.x; i < RW * RH; i += NT) {
        const int x = wrap_any(t.x0 - H + i % RW, t.nx), y = wrap_any(t.y0 - H + i / RW, t.ny);
        any = any || cls[(size_t)t.off + (size_t)y * t.px + x] != 0;
    }
    const int s = __syncthreads_or(any);
    // (a pull reaches one node beyond the halo)
    const bool edge = t.x0 - H - 1 < 0 || t.x0 + TW + H >= t.nx || t.y0 - H - 1 < 0 || t.y0 + TH + H >= t.ny;
    if (threadIdx.x == 0) tiles[blockIdx.x].flags = (s ? T2_SOLID : 0) | (edge ? T2_EDGE : 0);
}

// Barrier for what the threads exchange through LDS: waits for this wave's LDS
// operations only, so that global loads issued ahead stay in flight.
__device__ __forceinline__ void lds_sync() { asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory"); }

// A pointer held in scalar registers that the compiler does not take apart:
// accesses at a 32-bit vector offset from it then need no vector address
// arithmetic.
template <typename T>
using gptr = T __attribute__((address_space(1)))*;
template <typename T>
__device__ __forceinline__ gptr<T> scalar_base(T* p, long long shift) {
    unsigned long long a = (unsigned long long)(p + shift);
    asm volatile("" : "+s"(a));
    return (gptr<T>)a;
}
template <typename T>
__device__ __forceinline__ gptr<T> at_byte(gptr<T> p, uint32_t bytes) {
    return (gptr<T>)((unsigned long long)p + bytes);
}

// Populations S_t of a node (pull form), every load issued without waiting for
// an earlier one; m: wall mask of a boundary node (links to a solid, whose
// populations are the ones that left the node: halfway bounce-back), else 0.
// A solid node pulls like a fluid one: its loads are in bounds, its values unused.
template <typename R, bool SOLID, bool EDGE>
__device__ __forceinline__ void pull2d(const R* __restrict__ f, long long N, const Tile2d& t, uint32_t ix, int x, int y,
                                       uint32_t m, R S[L2::Q]) {
    if constexpr (!SOLID && !EDGE) {
        // the shift goes into the scalar base, so that all nine loads share one vector offset
#pragma unroll
        for (int i = 0; i < L2::Q; ++i)
            S[i] = *at_byte(scalar_base(f, (long long)i * N - (L2::E[i][0] + L2::E[i][1] * t.px)),
                            ix * (uint32_t)sizeof(R));
        return;
    }
    const int ox[3] = {EDGE && x + 1 >= t.nx ? 1 - t.nx : 1, 0, EDGE && x < 1 ? t.nx - 1 : -1};
    const int oy[3] = {(EDGE && y + 1 >= t.ny ? 1 - t.ny : 1) * t.px, 0, (EDGE && y < 1 ? t.ny - 1 : -1) * t.px};
#pragma unroll
    for (int i = 0; i < L2::Q; ++i) {
        const uint32_t a = ix + (uint32_t)(ox[1 + L2::E[i][0]] + oy[1 + L2::E[i][1]]);  // x - e_i
        const int j = L2::OPP[i];
        if (SOLID && i) {
            const bool back = (m >> j) & 1u;
            S[i] = at(f + (size_t)(back ? j : i) * N, back ? ix : a);
        } else {
            S[i] = at(f + (size_t)i * N, a);
        }
    }
}

// The BGK collision of one D2Q9 node (collide_values without MRT), its products
// and sums fused as the split step's kernels have them, so that both give the
// same bits: there each pair of directions is a basic block of its own, and
// only the first pair's -1.5 v.v is fused.  (Inlined here, the compiler would
// fuse across the pairs as well.)
template <typename R, typename C>
__device__ __forceinline__ void collide_bgk9(const R S[L2::Q], double rd, C Fx, C Fy, const Collision<C>& cp,
                                             R fo[L2::Q]) {
#pragma clang fp contract(off)
    auto fm = [](C a, C b, C c) -> C {
        if constexpr (sizeof(C) == 8) return __builtin_fma(a, b, c);
        else return __builtin_fmaf(a, b, c);
    };
    C ir, jx, jy;
    const C rs = (C)rd;
    if constexpr (sizeof(C) == 8) {
        ir = 1.0 / rd;
        jx = (C)S[1] - (C)S[3] + (C)S[5] - (C)S[6] - (C)S[7] + (C)S[8];
        jy = (C)S[2] - (C)S[4] + (C)S[5] + (C)S[6] - (C)S[7] - (C)S[8];
    } else {
        const C g = (C)S[5] - (C)S[7], h = (C)S[6] - (C)S[8];
        ir = __builtin_amdgcn_rcpf(rs);
        jx = ((C)S[1] - (C)S[3]) + g - h;
        jy = ((C)S[2] - (C)S[4]) + g + h;
    }
    const C ux = jx * ir, uy = jy * ir, vx = (jx + Fx) * ir, vy = (jy + Fy) * ir;
    const C uu = fm(uy, uy, ux * ux), vv = fm(vy, vy, vx * vx), hu = C(1.5) * uu, hv = C(1.5) * vv;
    const C om1 = C(1) - cp.omega;
    const bool relax = om1 != C(0);
#pragma unroll
    for (int i = 1; i < L2::Q; ++i) {
        if (L2::OPP[i] < i) continue;
        const int j = L2::OPP[i];
        const C wr = rs * C(L2::w(i)), w3 = wr * C(3);
        const C ev = L2::E[i][0] == 0 ? vy : (L2::E[i][1] == 0 ? vx : (L2::E[i][0] > 0 ? vx + vy : vy - vx));
        const C q = fm(ev, C(4.5) * ev, C(1)), sym = i == 1 ? fm(vv, C(-1.5), q) : q - hv, anti = w3 * ev;
        C vi = fm(wr, sym, anti), vj = fm(wr, sym, -anti);
        if (relax) {
            const C eu = L2::E[i][0] == 0 ? uy : (L2::E[i][1] == 0 ? ux : (L2::E[i][0] > 0 ? ux + uy : uy - ux));
            const C p = fm(eu, C(4.5) * eu, C(1)) - hu, au = w3 * eu;
            vi = fm(om1, (C)S[i] - fm(wr, p, au), vi);
            vj = fm(om1, (C)S[j] - fm(wr, p, -au), vj);
        }
        fo[i] = (R)vi;
        fo[j] = (R)vj;
    }
    if constexpr (sizeof(C) == 4) {
        double srest = 0.0;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            constexpr int order[4] = {1, 2, 5, 6};
            srest += (double)fo[order[i]];
            srest += (double)fo[L2::OPP[order[i]]];
        }
        fo[0] = (R)(rd - srest);
    } else {
        const C w0 = rs * C(L2::w(0));
        C v0 = w0 * (C(1) - hv);
        if (relax) v0 = fm(om1, fm(-w0, C(1) - hu, (C)S[0]), v0);
        fo[0] = (R)v0;
    }
}

// field and wall are one array in the phase-field model (phi of the fluid nodes
// and of the solid layers): a workgroup reads it at solid nodes only and stores,
// on measure steps, at fluid nodes only, so that no entry is both.  (Reading it
// at every node, its value unused at fluid ones, raced with those stores.)
template <typename R, typename C, bool MRT, int MODEL, int TW, int TH, int NT, int WPE>
__global__ void __launch_bounds__(NT) __attribute__((amdgpu_waves_per_eu(WPE))) k_step2d(const Tile2d* __restrict__ tiles, long long N,
                                               const R* __restrict__ fin, R* __restrict__ fout,
                                               const R* __restrict__ gin, R* __restrict__ gout, R* field,
                                               const R* wall, const uint8_t* __restrict__ cls, WallBC bc,
                                               Thermo th, Collision<C> cp, PhaseField pf, DevCtl* __restrict__ ctl,
                                               MeasureSlots* __restrict__ slots, double rho_m, R inv_b, int meas,
                                               int tick, int grav) {
    constexpr int H = halo_of(MODEL), OWN = TW * TH, K = OWN > NT ? OWN / NT : 1;
    static_assert((TW & (TW - 1)) == 0 && (OWN % NT == 0 || NT % OWN == 0), "whole threads per tile");
    constexpr int RW = TW + 2 * H, RH = TH + 2 * H;   // rho (psi, phi): the tile and its halo
    constexpr int MW = TW + 4, MH = TH + 4;           // mu of the chemical-potential model: halo 2
    __shared__ R rs[RH * RW];
    __shared__ R ms[MODEL == M2_CHEM ? MH * MW : 1];
    __shared__ uint8_t cl[RH * RW];

    const int tid = threadIdx.x;
    const Tile2d t = tiles[tile_slot(blockIdx.x, gridDim.x)];
    const bool solid = (t.flags & T2_SOLID) != 0, edge = (t.flags & T2_EDGE) != 0;
    auto node = [&](int x, int y) { return t.off + (uint32_t)y * (uint32_t)t.px + (uint32_t)x; };
    bool bad = false;
    // the density (phase field: order parameter) of gathered populations, rounded to storage
    auto moment = [&](const R S[L2::Q], bool fluid, double& s) -> R {
        s = 0.0;
#pragma unroll
        for (int i = 0; i < L2::Q; ++i) s += (double)S[i];
        if constexpr (MODEL == M2_PHASE) bad = bad || (fluid && !(fabs(s) < 1e300));
        else bad = bad || (fluid && !(s > 0.0 && s < (double)inv_b));
        return (R)s;
    };
    // what the stencils read at a fluid node of that moment
    auto staged = [&](R v) -> R {
        if constexpr (MODEL == M2_PSEUDO) return (R)(C(1) - exp(-(C)v));
        else return v;
    };

    // 1. The populations of the tile's nodes (kept in registers) and of its
    // halo (the rows below and above the tile, then the columns at its two
    // sides), summed into rs.  Work item w: the tile's nodes first, then the
    // halo's; a thread's items are unrolled, so that all their loads are in
    // flight together.
    R S[K][L2::Q], Sf[MODEL == M2_PHASE ? K : 1][L2::Q], r0[K];
    double rd[K];
    uint8_t co[K];
    auto gather_all = [&](auto solid_c, auto edge_c, auto halo_c) {
        constexpr bool SOLID = decltype(solid_c)::value, EDGE = decltype(edge_c)::value;
        constexpr int h = decltype(halo_c)::value, NROW = 2 * h * TW, ALL = OWN + NROW + 2 * h * (TH + 2 * h);
        constexpr int KT = (ALL + NT - 1) / NT;
        const R* src = MODEL == M2_PHASE ? gin : fin;
#pragma unroll
        for (int k = 0; k < KT; ++k) {
            const int w = tid + k * NT;
            if ((k + 1) * NT > ALL && w >= ALL) continue;
            int ox, oy;
            if (w < OWN + NROW) {
                // (NT is a multiple of TW: the column is that of the thread)
                const int r = w / TW;
                ox = w & (TW - 1);
                oy = r < TH ? r : (r < TH + h ? r - TH - h : r - h);
            } else {
                const int j = w - OWN - NROW, r = j / (2 * h), q = j - r * (2 * h);
                ox = q < h ? q - h : q - h + TW;
                oy = r - h;
            }
            int x = t.x0 + ox, y = t.y0 + oy;
            if (EDGE) {
                x = wrap_any(x, t.nx);
                y = wrap_any(y, t.ny);
            }
            const uint32_t ix = node(x, y);
            uint8_t c = 0;
            uint32_t m = 0;
            R wv = R(0);
            if (SOLID) {
                c = at(cls, ix);
                m = at(bc.nbmask, ix);
                if constexpr (MODEL != M2_PHASE) wv = at(wall, ix);
            }
            R Q[L2::Q];
            pull2d<R, SOLID, EDGE>(src, N, t, ix, x, y, m, Q);
            const bool fluid = (c & CLS_MASK) == CLS_FLUID;
            if constexpr (SOLID && MODEL == M2_PHASE)
                if (!fluid) wv = at(wall, ix);
            if constexpr (SOLID && MODEL != M2_PHASE) {
                if (bc.bouzidi && (c & CLS_CURVED)) {
                    Dims d;
                    d.nx = t.nx;
                    d.ny = t.ny;
                    d.nz = 1;
                    d.px = t.px;
                    d.N = N;
                    interp_wall<L2, R, C>(fin, d, ix, x, y, 0, m, bc, Q);
                }
            }
            double sum;
            const R v = moment(Q, fluid, sum);
            const int l = (oy + H) * RW + ox + H;
            if (SOLID) {
                cl[l] = c;
                rs[l] = fluid ? staged(v) : (MODEL == M2_CHEM ? R(0) : wv);
                if constexpr (MODEL == M2_CHEM)
                    if (!fluid && ox >= -2 && ox < TW + 2 && oy >= -2 && oy < TH + 2) ms[(oy + 2) * MW + ox + 2] = wv;
            } else {
                rs[l] = staged(v);
            }
            if (k < K) {  // (with more threads than nodes only the first OWN threads use it)
#pragma unroll
                for (int i = 0; i < L2::Q; ++i) S[k][i] = Q[i];
                r0[k] = v;
                rd[k] = sum;
                co[k] = c;
                if constexpr (MODEL == M2_PHASE) {
                    pull2d<R, SOLID, EDGE>(fin, N, t, ix, x, y, m, Sf[k]);
                    if constexpr (SOLID)
                        if (bc.bouzidi && (c & CLS_CURVED)) {
                            Dims d;
                            d.nx = t.nx;
                            d.ny = t.ny;
                            d.nz = 1;
                            d.px = t.px;
                            d.N = N;
                            interp_wall<L2, R, C>(fin, d, ix, x, y, 0, m, bc, Sf[k]);
                        }
                }
            }
        }
    };
    typedef std::integral_constant<bool, true> Y;
    typedef std::integral_constant<bool, false> No;
    typedef std::integral_constant<int, H> Full;
    typedef std::integral_constant<int, MODEL == M2_CHEM ? 4 : H> Plain;  // no solid in reach: stencils alone
    if (solid) {
        if (edge) gather_all(Y{}, Y{}, Full{});
        else gather_all(Y{}, No{}, Full{});
    } else {
        if (edge) gather_all(No{}, Y{}, Plain{});
        else gather_all(No{}, No{}, Plain{});
    }
    lds_sync();

    if constexpr (MODEL == M2_CHEM) {
        // 2. Eq. 14 on the solid layers in reach: the first layer from its fluid
        // neighbours, then the second from its first-layer neighbours
        auto fill = [&](auto layer_c) {
            constexpr int layer = decltype(layer_c)::value, W = RW - 2 * layer, n = W * (RH - 2 * layer);
            constexpr uint8_t want = layer == 1 ? CLS_FLUID : CLS_L1;
            for (int i = tid; i < n; i += NT) {
                const int l = (i / W + layer) * RW + i % W + layer;
                if ((cl[l] & CLS_MASK) != layer) continue;
                double den = 0.0;
                C num = C(0);
#pragma unroll
                for (int q = 1; q < L2::Q; ++q) {
                    const int o = l + L2::E[q][1] * RW + L2::E[q][0];
                    const R v = rs[o];
                    if ((cl[o] & CLS_MASK) != want) continue;
                    den += L2::w(q);
                    num += C(L2::w(q)) * (C)v;
                }
                rs[l] = (R)(num * (C)(R)(1.0 / den));
            }
            lds_sync();
        };
        if (solid) {
            fill(std::integral_constant<int, 1>{});
            fill(std::integral_constant<int, 2>{});
        }
        // 3. mu of the tile and two nodes around it (the solid layers already hold the wall value)
#pragma unroll
        for (int k = 0; k < (MW * MH + NT - 1) / NT; ++k) {
            const int w = tid + k * NT;
            if ((k + 1) * NT > MW * MH && w >= MW * MH) continue;
            // whole rows of the tile's columns first, then two columns at each side
            const int j = w - MH * TW;
            const int ry = w < MH * TW ? w / TW : j >> 2;
            const int rx = w < MH * TW ? (w & (TW - 1)) + 2 : (j & 1) + ((j & 2) ? TW + 2 : 0);
            const int l = (ry + H - 2) * RW + rx + H - 2, i = ry * MW + rx;
            if (solid && (cl[l] & CLS_MASK) != CLS_FLUID) continue;
            auto p = [&](int o) { return (C)rs[l + o]; };
            const C c0 = p(0);
            C lap = d2c<C>(p(-2), p(-1), c0, p(1), p(2));
            lap += d2c<C>(p(-2 * RW), p(-RW), c0, p(RW), p(2 * RW));
            ms[i] = (R)((psi_prime<C>(c0, th) - (C)th.mu_ref) - (C)th.kappa * lap);
        }
        lds_sync();
    }

    auto store_all = [&](const R fo[L2::Q], uint32_t ix) {
#pragma unroll
        for (int i = 0; i < L2::Q; ++i)
            __builtin_nontemporal_store(fo[i], at_byte(scalar_base(fout, (long long)i * N), ix * (uint32_t)sizeof(R)));
    };
    // 4. force and collision of the tile's nodes.  The force enters the
    // collision as an opaque value, as the split step's collision takes it.
    auto collide_store = [&](const R P[L2::Q], double rdens, C Fx, C Fy, uint32_t ix) {
        R fo[L2::Q];
        if constexpr (MRT) collide_values<L2, R, C, true, true>(P, Fx, Fy, C(0), cp, fo, rdens);
        else collide_bgk9<R, C>(P, rdens, Fx, Fy, cp, fo);
        store_all(fo, ix);
    };
    unsigned long long cnt = 0, sx = 0, sy = 0;
#pragma unroll
    for (int k = 0; k < K; ++k) {
        const int w = tid + k * NT, lx = w & (TW - 1), ly = w / TW;
        const int x = t.x0 + lx, y = t.y0 + ly;
        if ((NT > OWN && w >= OWN) || x >= t.nx || y >= t.ny || (co[k] & CLS_MASK) != CLS_FLUID) continue;
        const uint32_t ix = node(x, y);
        const int l = (ly + H) * RW + lx + H;
        typedef double D;
        auto pr = [&](int o) { return (D)rs[l + o]; };
        if (meas) {
            at(field, ix) = r0[k];
            if ((double)r0[k] >= rho_m) {
                cnt += 1;
                sx += (unsigned long long)x;
                sy += (unsigned long long)y;
            }
        }
        if constexpr (MODEL == M2_PHASE) {
            const D c0 = pr(0);
            D lap = d2c<D>(pr(-2), pr(-1), c0, pr(1), pr(2));
            lap += d2c<D>(pr(-2 * RW), pr(-RW), c0, pr(RW), pr(2 * RW));
            const R mu = (R)(pf.A * (c0 * c0 * c0 - c0) - pf.kappa * lap);
            double rho = 0.0;
#pragma unroll
            for (int i = 0; i < L2::Q; ++i) rho += (double)Sf[k][i];
            bad = bad || !(rho > 0.0 && rho < 1e300);
            double F[3];
            const double m0 = (double)mu;
            F[0] = m0 * d1c<double>(pr(-2), pr(-1), pr(1), pr(2));
            F[1] = m0 * d1c<double>(pr(-2 * RW), pr(-RW), pr(RW), pr(2 * RW));
            F[2] = 0.0;
            if (grav) {
#pragma unroll
                for (int a = 0; a < 3; ++a) F[a] += rho * cp.g[a];
            }
            C v[3];
            if constexpr (sizeof(R) == 8) {
                R fo[L2::Q];
                collide_values<L2, R, C, MRT, true>(Sf[k], (C)F[0], (C)F[1], (C)F[2], cp, fo, rho);
                store_all(fo, ix);
                pf_velocity<L2, R, C>(Sf[k], F, v);
            } else {
                C Fx = (C)F[0], Fy = (C)F[1];
                asm volatile("" : "+v"(Fx), "+v"(Fy));
                collide_store(Sf[k], rho, Fx, Fy, ix);
                if constexpr (sizeof(C) == 8) {
                    const double Fv[3] = {Fx, Fy, 0.0};
                    pf_velocity<L2, R, C>(Sf[k], Fv, v);
                } else {
                    // pf_velocity on values the compiler cannot share with the
                    // collision above: the split step's kernel forms the velocity
                    // in the order parameter's basic block
                    const C g = (C)Sf[k][5] - (C)Sf[k][7], h = (C)Sf[k][6] - (C)Sf[k][8];
                    C jx = ((C)Sf[k][1] - (C)Sf[k][3]) + g - h, jy = ((C)Sf[k][2] - (C)Sf[k][4]) + g + h, r = (C)rho;
                    asm volatile("" : "+v"(jx), "+v"(jy), "+v"(r), "+v"(Fx), "+v"(Fy));
                    const C ir = __builtin_amdgcn_rcpf(r);
                    v[0] = (jx + C(0.5) * Fx) * ir;
                    v[1] = (jy + C(0.5) * Fy) * ir;
                    v[2] = C(0);
                }
            }
            R go[L2::Q];
            pf_collide_g<L2, R, C>(S[k], v, (C)mu, pf, go);
#pragma unroll
            for (int i = 0; i < L2::Q; ++i)
                __builtin_nontemporal_store(go[i], at_byte(scalar_base(gout, (long long)i * N), ix * (uint32_t)sizeof(R)));
        } else {
            D fx, fy;
            const D rk = (D)r0[k];
            if constexpr (MODEL == M2_PSEUDO) {
                double ax = 0.0, ay = 0.0;
#pragma unroll
                for (int i = 1; i < L2::Q; ++i) {
                    const double v = L2::w(i) * pr(L2::E[i][1] * RW + L2::E[i][0]);
                    ax += v * L2::E[i][0];
                    ay += v * L2::E[i][1];
                }
                const double p0 = pr(0);
                fx = -cp.sc_G * p0 * ax;
                fy = -cp.sc_G * p0 * ay;
            } else {
                const int m = (ly + 2) * MW + lx + 2;
                auto pm = [&](int o) { return (D)ms[m + o]; };
                const D gmx = d1c<D>(pm(-2), pm(-1), pm(1), pm(2));
                const D grx = d1c<D>(pr(-2), pr(-1), pr(1), pr(2));
                const D gmy = d1c<D>(pm(-2 * MW), pm(-MW), pm(MW), pm(2 * MW));
                const D gry = d1c<D>(pr(-2 * RW), pr(-RW), pr(RW), pr(2 * RW));
                const D third = D(1.0 / 3.0);
                fx = -rk * gmx + grx * third;
                fy = -rk * gmy + gry * third;
            }
            if (grav) {
                fx += rk * (D)cp.g[0];
                fy += rk * (D)cp.g[1];
            }
            C Fx = (C)fx, Fy = (C)fy;
            asm volatile("" : "+v"(Fx), "+v"(Fy));
            collide_store(S[k], rd[k], Fx, Fy, ix);
        }
    }
    if (bad) atomicOr(&ctl->status, 1);
    if (tick && blockIdx.x == 0 && tid == 0) ctl->t += 1;
    if (meas) {
        // liquid centroid sums of the workgroup
        __shared__ unsigned long long red[NT / 64][3];
        unsigned long long v[3] = {cnt, sx, sy};
#pragma unroll
        for (int off = 32; off > 0; off >>= 1)
#pragma unroll
            for (int a = 0; a < 3; ++a) v[a] += __shfl_down(v[a], off, 64);
        if ((tid & 63) == 0)
            for (int a = 0; a < 3; ++a) red[tid >> 6][a] = v[a];
        __syncthreads();
        if (tid < 3) {
            unsigned long long s = 0;
            for (int w = 0; w < NT / 64; ++w) s += red[w][tid];
            if (s) atomicAdd((&slots[t.c].cnt) + tid, s);
        }
    }
}

// Tile shapes (tw, th, threads, waves per SIMD the registers are held to); shape2d_for says which one when.
#define SHAPES2D(X) X(0, 16, 16, 1024, 8) X(1, 64, 16, 1024, 8) X(2, 32, 16, 512, 4)

template <typename R, typename C, bool MRT, int MODEL>
void launch_shape(const Step2dArgs& a, const Thermo& th, const void* cp, hipStream_t st) {
    const Collision<C> c = *(const Collision<C>*)cp;
    constexpr bool F64 = sizeof(C) == 8;
    switch (a.shape) {
#define X(I, TW, TH, NT, WPE)                                                                                     \
    case I:                                                                                                       \
        if constexpr (I < 2 || (F64 && MODEL != M2_PHASE))                                                                   \
            k_step2d<R, C, MRT, MODEL, TW, TH, NT, F64 ? 4 : WPE><<<(unsigned)a.ntiles, NT, 0, st>>>(             \
                a.tiles, a.N, (const R*)a.fin, (R*)a.fout, (const R*)a.gin, (R*)a.gout, (R*)a.field,              \
                (const R*)a.wall, a.cls, a.bc, th, c, a.pf, a.ctl, a.slots, a.rho_m, (R)a.inv_b, a.meas, a.tick,  \
                a.grav);                                                                                          \
        break;
        SHAPES2D(X)
#undef X
    }
}

template <typename R, typename C>
void launch_model(const Step2dArgs& a, const Thermo& th, const void* cp, hipStream_t st) {
    if (a.model == M2_PSEUDO) {
        if (a.mrt) launch_shape<R, C, true, M2_PSEUDO>(a, th, cp, st);
        else launch_shape<R, C, false, M2_PSEUDO>(a, th, cp, st);
    } else if (a.model == M2_PHASE) {
        if (a.mrt) launch_shape<R, C, true, M2_PHASE>(a, th, cp, st);
        else launch_shape<R, C, false, M2_PHASE>(a, th, cp, st);
    } else {
        if (a.mrt) launch_shape<R, C, true, M2_CHEM>(a, th, cp, st);
        else launch_shape<R, C, false, M2_CHEM>(a, th, cp, st);
    }
}

}  // namespace

Shape2d shape2d(int k) {
    static const Shape2d s[] = {
#define X(I, TW, TH, NT, WPE) {TW, TH, NT},
        SHAPES2D(X)
#undef X
    };
    return s[k];
}

std::vector<Tile2d> tiles2d(const Dims* dims, int n, int shape) {
    const Shape2d s = shape2d(shape);
    std::vector<Tile2d> v;
    for (int c = 0; c < n; ++c)
        for (int y0 = 0; y0 < dims[c].ny; y0 += s.th)
            for (int x0 = 0; x0 < dims[c].nx; x0 += s.tw) v.push_back(Tile2d{c, x0, y0, 0, dims[c].nx, dims[c].ny, dims[c].px, (uint32_t)dims[c].off});
    return v;
}

// One launch of a small lattice lasts as long as one workgroup does, and 16 x 16
// tiles with a thread for every node of the halo as well (one gather per
// thread) are the shorter chain: chemical potential, MRT, us per step at 256^2
// 6.5 against 10.2 with 64 x 16 ones in FP32 (7.7 against 13.5 in FP64).  They
// fill the device with two workgroups per compute unit (512 tiles, 131,000
// nodes); beyond, the halo counts: near a solid 16 x 16 tiles gather 3.1 times
// the populations that they collide and 64 x 16 ones 2.1 times (elsewhere 2.25
// and 1.7; pseudopotential 1.27 and 1.16, phase field 1.56 and 1.33).  us per
// step of 16 x 16 and 64 x 16 tiles, MRT FP32 and FP64:
//            chemical potential       pseudopotential         phase field
//   340^2    7.8 10.3   12.2 14.0     4.7 5.4    6.4  6.8     6.4  8.2   10.6 11.2
//   380^2    9.3 10.4   13.1 16.0     6.2 5.4    7.5  6.6     8.4  9.0   15.4 12.0
//   420^2   10.6 10.5   16.6 14.6     6.5 5.3    8.5  7.4    11.8 10.2   17.6 13.8
//   460^2   11.0 10.4   19.1 15.0     7.0 5.6   11.1  7.8    14.7 11.6   21.6 14.1
// so they cross between 340^2 and 420^2 for every model; one line, at the last
// size where all of these are ahead, serves them all (with BGK the phase field
// in FP64 alone is behind there, 12.5 against 10.7).  With double arithmetic
// 32 x 16 tiles of 512 threads are ahead of 64 x 16 ones from about 400,000
// nodes (chemical potential FP64, 720^2: 27.9 against 33.2 us, 1400^2: 74.3
// against 83.2), except in the phase-field model, whose second population set
// fills the registers.
int shape2d_for(long long nodes, int precision, int model) {
    if (nodes <= 116000) return 0;
    return precision != LBM_F32 && nodes >= 400000 && model != M2_PHASE ? 2 : 1;
}

void tiles2d_flags(Tile2d* tiles, int ntiles, const uint8_t* cls, int model, int shape,
                   hipStream_t st) {
    if (ntiles < 1) return;
    switch (shape) {
#define X(I, TW, TH, NT, WPE)                                                                                          \
    case I:                                                                                                       \
        if (model == M2_CHEM) k_tiles2d_flags<TW, TH, NT, halo_of(M2_CHEM)><<<(unsigned)ntiles, NT, 0, st>>>(tiles, cls); \
        else if (model == M2_PSEUDO) k_tiles2d_flags<TW, TH, NT, halo_of(M2_PSEUDO)><<<(unsigned)ntiles, NT, 0, st>>>(tiles, cls); \
        else k_tiles2d_flags<TW, TH, NT, halo_of(M2_PHASE)><<<(unsigned)ntiles, NT, 0, st>>>(tiles, cls);   \
        break;
        SHAPES2D(X)
#undef X
    }
}

void step2d_launch(const Step2dArgs& a, const Thermo& th, const void* cp, hipStream_t st) {
    if (a.precision == LBM_F64) launch_model<double, double>(a, th, cp, st);
    else if (a.precision == LBM_F32_MIXED) launch_model<float, double>(a, th, cp, st);
    else launch_model<float, float>(a, th, cp, st);
}

}  // namespace lbm

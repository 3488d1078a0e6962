// Fluid kernels of the step: the fluid pass (density and pseudopotential, force, Guo-BGK
// collision, push streaming with moving-wall bounce-back, in one read of the populations) and
// the per-body force/torque sums.
#pragma once

#include "device_common.h"

namespace pfl {

// periodic neighbour offsets of one cell as unsigned index deltas (the sum with the cell index
// wraps modulo 2^32 onto the neighbour's index, which lets loads use a scalar base + 32-bit
// offset)
struct NbrU {
    uint32_t xp, xm, yp, ym, zp, zm;
    // scale: bytes per element for byte offsets, 1 for element indices
    __device__ __forceinline__ NbrU(int x, int y, int z, int nx, int ny, int nz, int scale) {
        const int pl = nx * ny;
        xp = (uint32_t)((x == nx - 1 ? 1 - nx : 1) * scale);
        xm = (uint32_t)((x == 0 ? nx - 1 : -1) * scale);
        yp = (uint32_t)((y == ny - 1 ? (1 - ny) * nx : nx) * scale);
        ym = (uint32_t)((y == 0 ? (ny - 1) * nx : -nx) * scale);
        zp = (uint32_t)((z == nz - 1 ? (1 - nz) * pl : pl) * scale);
        zm = (uint32_t)((z == 0 ? (nz - 1) * pl : -pl) * scale);
    }
    template <int I>
    __device__ __forceinline__ uint32_t at(uint32_t idx) const {
        uint32_t o = idx;
        if constexpr (Dir<I>::x == 1) o += xp;
        if constexpr (Dir<I>::x == -1) o += xm;
        if constexpr (Dir<I>::y == 1) o += yp;
        if constexpr (Dir<I>::y == -1) o += ym;
        if constexpr (Dir<I>::z == 1) o += zp;
        if constexpr (Dir<I>::z == -1) o += zm;
        return o;
    }
};

// periodic neighbour offsets of one cell (index deltas for +1 / -1 along each axis)
struct Nbr {
    int xp, xm, yp, ym, zp, zm;
    __device__ __forceinline__ Nbr(int x, int y, int z, int nx, int ny, int nz) {
        const int pl = nx * ny;
        xp = x == nx - 1 ? 1 - nx : 1;
        xm = x == 0 ? nx - 1 : -1;
        yp = y == ny - 1 ? (1 - ny) * nx : nx;
        ym = y == 0 ? (ny - 1) * nx : -nx;
        zp = z == nz - 1 ? (1 - nz) * pl : pl;
        zm = z == 0 ? (nz - 1) * pl : -pl;
    }
    template <int I>
    __device__ __forceinline__ int off() const {
        return (Dir<I>::x == 1 ? xp : (Dir<I>::x == -1 ? xm : 0)) + (Dir<I>::y == 1 ? yp : (Dir<I>::y == -1 ? ym : 0)) +
               (Dir<I>::z == 1 ? zp : (Dir<I>::z == -1 ? zm : 0));
    }
    // the same for a direction known only at run time
    __device__ __forceinline__ int off_rt(int i) const {
        const int cx = kCX[i], cy = kCY[i], cz = kCZ[i];
        return (cx > 0 ? xp : (cx < 0 ? xm : 0)) + (cy > 0 ? yp : (cy < 0 ? ym : 0)) + (cz > 0 ? zp : (cz < 0 ? zm : 0));
    }
};

// reciprocal: correctly rounded in FP64 (parity with the FP64 oracle), hardware rcp in FP32
__device__ __forceinline__ double recip(double x) { return 1.0 / x; }
__device__ __forceinline__ float recip(float x) { return __builtin_amdgcn_rcpf(x); }

// ---- the fluid pass: density, pseudopotential, force, collision and push streaming -----------
//
// One pass over the populations per step.  A block owns a tile of 64 x TY nodes in the x-y plane
// and marches a chunk of tz planes along z.  The Shan-Chen/Benzi force at a node needs the
// pseudopotential of its 18 (26) neighbours at the same time level, so the block keeps a window
// of three planes of psi for its tile and a one-node halo in LDS: before colliding plane z it
// forms rho and psi of plane z + 1 from the post-stream populations (the tile's own nodes and
// the halo), so every population is read from HBM once.  The tile's own populations of plane
// z + 1 wait in LDS (each thread in its own slots) until plane z + 1 is collided; halo nodes
// and the two planes before and after the chunk cost a density-only read (mostly served by L2,
// where the neighbouring tiles read the same lines).  The pseudopotential of every node is
// written once, for the force scan and read-out.

// Collision and streaming of one fluid node (Sec. 3.2.1, 3.2.2, 3.2.3): sv holds its stored
// post-stream populations, psin(I) the pseudopotential of its neighbour in direction I, psi0 its
// own.  Forms the force from the neighbours' psi (solid neighbours act with their wetting
// density), collides with BGK + Guo forcing at the half-force velocity, and pushes each
// post-collision population to its neighbour, or, when the neighbour is solid (bit i of
// solid_dirs), reflects it half-way into the node's own opposite slot (with the moving-wall term
// where wall_in_fluid_pass).  rin: reference density of the node's stored inputs (FP16 storage).
//
// Arithmetic is organised by opposite pairs (c_opp = -c): with cu = c.v, cF = c.F,
//   f*_i = (1 - 1/tau) f_i + w (even + odd),  f*_opp = (1 - 1/tau) f_opp + w (even - odd),
//   even = rho/tau (1 - 3/2 v.v) - 3 g v.F + 9/2 rho/tau cu^2 + 9 g cu cF,  odd = 3 rho/tau cu + 3 g cF,
// g = 1 - 1/(2 tau), which is the BGK relaxation to the second-order equilibrium plus the Guo term.
// Where the moving-wall term of the bounce-back is added (Sec. 3.2.2).  FP32 and FP64: by the force
// scan, which visits exactly the nodes next to solids, so the fluid pass needs no body data and
// stays lean.  FP16 storage: in the fluid pass, so that the reflected population f*_i + g_i is
// rounded to FP16 once (adding g to an already rounded f*_i and rounding again was measured to
// triple the body-force error of the form).
template <typename S>
constexpr bool wall_in_fluid_pass() {
    return sizeof(S) == 2;
}

// Motion of every body for the moving-wall term of the FP16 form, staged in LDS by the fluid pass
// (centre FP64 for the minimum-image lever arm, velocities as the FP32 arithmetic uses them).
struct WallMot {
    double X[PF_LBM_MAX_BODIES][3];
    float V[PF_LBM_MAX_BODIES][3], W[PF_LBM_MAX_BODIES][3];
};

// psin(I): psi of the neighbour in direction I; FP16 form: refn(I) its reference density R (the
// encode of a population pushed there) and rown the node's own (the encode of its own slots),
// both R(psi) of this step's psi, formed once per node with the window
// SUM: the density for the force scan is summed for every node (see there)
template <typename S, class L, bool SUM, typename PsiN, typename RefN>
__device__ __forceinline__ void collide_push(const Prm<ArT<S>> &p, const S *sv, ArT<S> rin, PsiN psin, RefN refn,
                                             ArT<S> psi0, ArT<S> rown, S *__restrict__ fout, uint32_t solid_dirs,
                                             int x, int y, int z, long long Np, const WallMot *wm,
                                             ArT<S> *__restrict__ rho_link) {
    using T = ArT<S>;
    const int nx = p.nx, ny = p.ny, nz = p.nz;
    const uint32_t idx = (uint32_t)(x + nx * (y + ny * z));
    const uint32_t is = idx * (uint32_t)sizeof(S);  // populations (storage type)
    const NbrU ns(x, y, z, nx, ny, nz, (int)sizeof(S));
    constexpr bool H = sizeof(S) == 2;  // FP16 storage: deviations from w_i R

    T f[L::Q];
    sfor<L::Q>([&](auto I) { f[I] = pop_get<S>(sv[I], Dir<decltype(I)::value, L>::template w<T>(), rin); });
    // The density of a node with links for the moving-wall term of the force scan, which would read the q
    // populations again for it.  FP32: summed in the order of the directions, as the scan would (the sums
    // on the bodies cancel to far below its rounding), here where a node has links, or (SUM) for every node
    // and stored with the streaming, so that no branch waits for the neighbour bits here.  FP64 stores the
    // collision's own there.
    T rlink = T(0);
    if constexpr (sizeof(S) == 4) {
        if (SUM || solid_dirs) sfor<L::Q>([&](auto I) { rlink += f[I]; });
        if constexpr (!SUM)
            if (solid_dirs) stb(rho_link, idx * (uint32_t)sizeof(T), rlink);
    }
    // moments from pair sums and differences
    T rho = f[0], jx = T(0), jy = T(0), jz = T(0);
    sfor<(L::Q - 1) / 2>([&](auto K) {
        constexpr int i = 2 * decltype(K)::value + 1;  // i and i + 1 are opposite
        const T sp = f[i] + f[i + 1], dm = f[i] - f[i + 1];
        rho += sp;
        if constexpr (Dir<i, L>::x == 1) jx += dm;
        if constexpr (Dir<i, L>::x == -1) jx -= dm;
        if constexpr (Dir<i, L>::y == 1) jy += dm;
        if constexpr (Dir<i, L>::y == -1) jy -= dm;
        if constexpr (Dir<i, L>::z == 1) jz += dm;
        if constexpr (Dir<i, L>::z == -1) jz -= dm;
    });

    // pseudopotential force from pair differences of the neighbours' psi
    T s1x = T(0), s1y = T(0), s1z = T(0), s2x = T(0), s2y = T(0), s2z = T(0), s3x = T(0), s3y = T(0), s3z = T(0);
    sfor<(L::Q - 1) / 2>([&](auto K) {
        constexpr int i = 2 * decltype(K)::value + 1;
        const T pa = psin(std::integral_constant<int, i>{}), pb = psin(std::integral_constant<int, i + 1>{});
        const T dp = pa - pb;
        if constexpr (Dir<i, L>::c2 == 1) {
            if constexpr (Dir<i, L>::x != 0) s1x += T(Dir<i, L>::x) * dp;
            if constexpr (Dir<i, L>::y != 0) s1y += T(Dir<i, L>::y) * dp;
            if constexpr (Dir<i, L>::z != 0) s1z += T(Dir<i, L>::z) * dp;
        } else if constexpr (Dir<i, L>::c2 == 2) {
            if constexpr (Dir<i, L>::x != 0) s2x += T(Dir<i, L>::x) * dp;
            if constexpr (Dir<i, L>::y != 0) s2y += T(Dir<i, L>::y) * dp;
            if constexpr (Dir<i, L>::z != 0) s2z += T(Dir<i, L>::z) * dp;
        } else {
            s3x += T(Dir<i, L>::x) * dp;
            s3y += T(Dir<i, L>::y) * dp;
            s3z += T(Dir<i, L>::z) * dp;
        }
    });
    const T gp = -p.G * psi0;
    const T w1 = T(L::wshell[1]), w2 = T(L::wshell[2]);
    T Fx = w1 * s1x + w2 * s2x, Fy = w1 * s1y + w2 * s2y, Fz = w1 * s1z + w2 * s2z;
    if constexpr (L::Q == 27) {
        const T w3 = T(L::wshell[3]);
        Fx += w3 * s3x;
        Fy += w3 * s3y;
        Fz += w3 * s3z;
    }
    Fx = gp * Fx + p.fext[0];
    Fy = gp * Fy + p.fext[1];
    Fz = gp * Fz + p.fext[2];

    // half-force velocity; an empty node has v = 0
    T ux = T(0), uy = T(0), uz = T(0);
    if (rho > T(0)) {
        const T inv = recip(rho);
        ux = (jx + T(0.5) * Fx) * inv;
        uy = (jy + T(0.5) * Fy) * inv;
        uz = (jz + T(0.5) * Fz) * inv;
    }
    const T om = p.omega, g = p.guo, omr = om * rho;
    const T A = omr * (T(1) - T(1.5) * (ux * ux + uy * uy + uz * uz)) - T(3) * g * (ux * Fx + uy * Fy + uz * Fz);
    const T B = T(3) * omr, C = T(4.5) * omr, D = T(3) * g, E = T(9) * g, keep = T(1) - om;
    f[0] = keep * f[0] + Dir<0, L>::template w<T>() * A;
    sfor<(L::Q - 1) / 2>([&](auto K) {
        constexpr int i = 2 * decltype(K)::value + 1;
        constexpr T w = Dir<i, L>::template w<T>();
        const T cu = T(Dir<i, L>::x) * ux + T(Dir<i, L>::y) * uy + T(Dir<i, L>::z) * uz;
        const T cF = T(Dir<i, L>::x) * Fx + T(Dir<i, L>::y) * Fy + T(Dir<i, L>::z) * Fz;
        const T even = A + cu * (C * cu + E * cF);
        const T odd = B * cu + D * cF;
        f[i] = keep * f[i] + w * (even + odd);
        f[i + 1] = keep * f[i + 1] + w * (even - odd);
    });

    // streaming: push to the neighbour, or reflect half-way into the node's own opposite slot
    // when the neighbour is solid
    T drho = T(0);
    if (!solid_dirs) {
        sfor<L::Q>([&](auto I) {
            constexpr int i = decltype(I)::value;
            if constexpr (i > 0)
                stb(fout + (long long)i * Np, ns.template at<i>(is), pop_put<S>(f[i], Dir<i, L>::template w<T>(), refn(I)));
        });
    } else if constexpr (!wall_in_fluid_pass<S>()) {
        // f*_i into slot opp(i); the force scan adds the moving-wall term and the mass correction
        if constexpr (SUM || sizeof(S) == 8) stb(rho_link, idx * (uint32_t)sizeof(T), SUM ? rlink : rho);
        sfor<L::Q>([&](auto I) {
            constexpr int i = decltype(I)::value;
            if constexpr (i > 0) {
                if (!(solid_dirs & (1u << i)))
                    stb(fout + (long long)i * Np, ns.template at<i>(is), pop_put<S>(f[i], Dir<i, L>::template w<T>(), refn(I)));
                else
                    stb(fout + (long long)Dir<i, L>::opp * Np, is, pop_put<S>(f[i], Dir<i, L>::template w<T>(), rown));
            }
        });
    } else {
        // f*_i + g_i into slot opp(i), g_i = -2 rho w_i (c_i . u_w) / c_s^2 with u_w the rigid
        // velocity at the link midpoint x + c_i / 2; the rest population gives back the g_i.  The
        // solid neighbour's owner comes from its window entry and the bodies' motion from LDS, so
        // the links wait for no global load.
        sfor<L::Q>([&](auto I) {
            constexpr int i = decltype(I)::value;
            if constexpr (i > 0) {
                if (!(solid_dirs & (1u << i))) {
                    stb(fout + (long long)i * Np, ns.template at<i>(is), pop_put<S>(f[i], Dir<i, L>::template w<T>(), refn(I)));
                } else {
                    // the FP16 form's collision arithmetic is FP32: the lever arm about the body
                    // centre (minimum image, FP64) and the wall velocity at the link midpoint in FP32
                    // (bounded to the body table whatever the entry holds)
                    const int o = __float_as_int(refn(I)) & (PF_LBM_MAX_BODIES - 1);
                    const T rx = (T)mimg_r(x - wm->X[o][0], nx, p.inv_n[0]) + T(0.5 * Dir<i, L>::x),
                            ry = (T)mimg_r(y - wm->X[o][1], ny, p.inv_n[1]) + T(0.5 * Dir<i, L>::y),
                            rz = (T)mimg_r(z - wm->X[o][2], nz, p.inv_n[2]) + T(0.5 * Dir<i, L>::z);
                    const T wx = wm->W[o][0], wy = wm->W[o][1], wz = wm->W[o][2];
                    const T uwx = wm->V[o][0] + (wy * rz - wz * ry), uwy = wm->V[o][1] + (wz * rx - wx * rz),
                            uwz = wm->V[o][2] + (wx * ry - wy * rx);
                    const T cuw = T(Dir<i, L>::x) * uwx + T(Dir<i, L>::y) * uwy + T(Dir<i, L>::z) * uwz;
                    const T gw = T(-6.0 * Dir<i, L>::template w<double>()) * cuw * rho;
                    stb(fout + (long long)Dir<i, L>::opp * Np, is, pop_put<S>(f[i] + gw, Dir<i, L>::template w<T>(), rown));
                    drho += gw;
                }
            }
        });
    }
    stb(fout, is, pop_put<S>(f[0] - drho, Dir<0, L>::template w<T>(), rown));
}

// LDS of the fluid pass: the psi window (3 planes of the tile and its halo, 66 x (TY + 2)), the
// tile's populations of the plane being collided ([direction][node of the tile], stored form),
// and, where the budget allows (DMA), the halo's populations, cell words and previous psi of
// two planes, loaded straight into LDS.
// entry of the psi window: psi, and in the FP16 form beside it the reference density R(psi) of a
// fluid node (formed once per node instead of once per population pushed to it) or, for a solid
// node (never a push destination), the index of its owner as an integer bit pattern (the moving-
// wall term of a link into it reads the owner from the window instead of the cell word)
template <typename S>
using WinE = std::conditional_t<sizeof(S) == 2, float2, ArT<S>>;
template <typename S>
__device__ __forceinline__ ArT<S> win_psi(const WinE<S> &e) {
    if constexpr (sizeof(S) == 2)
        return e.x;
    else
        return e;
}
template <typename S>
__device__ __forceinline__ ArT<S> win_ref(const WinE<S> &e) {
    if constexpr (sizeof(S) == 2)
        return e.y;
    else
        return ArT<S>(0);
}
template <typename S>
__device__ __forceinline__ WinE<S> win_entry(ArT<S> psi, ArT<S> rho0, cell_t m) {
    if constexpr (sizeof(S) == 2)
        return make_float2(psi, (m & C_SOLID) ? __int_as_float(owner_of(m)) : ref_density(psi, rho0));
    else
        return psi;
}

template <typename S, class L, int TY, bool DMA>
struct FluidLds {
    // halo entries: the rows below and above the tile (64 each), the two columns (TY + 2 each)
    static constexpr int NH = DMA ? 128 + 2 * (TY + 2) : 1, NB = DMA ? 2 : 1;
    WinE<S> ring[3][TY + 2][66];
    std::conditional_t<wall_in_fluid_pass<S>(), WallMot, char> wm;  // bodies' motion (FP16 form)
    S pop[L::Q][64 * TY];
    S hpop[NB][L::Q][NH];
    cell_t hmask[NB][NH];
};
// Tile shapes of the fluid pass: TY rows of 64 nodes, W waves per block, each thread owning
// RPT = TY / W rows.  LDS stays within 80 KB so that two blocks share a CU (160 KB).
template <int TY>
struct FluidShape {
    static constexpr int W = TY <= 4 ? 4 : 8, RPT = TY / W;
};
// FP32 D3Q27 tiles of 8 rows exist in two forms, as the register count ends just above 128: held to 128, so
// that two blocks of 8 waves share a CU (LONE false), and free, one block a CU (LONE true).
template <typename S, class L, int TY>
constexpr bool fluid_two_forms() {
    return L::Q == 27 && sizeof(S) == 4 && TY == 8;
}
// waves per SIMD that the registers have to allow
template <typename S, class L, int TY, bool LONE>
constexpr int fluid_min_waves() {
    return fluid_two_forms<S, L, TY>() && !LONE ? 4 : 1;
}
constexpr size_t FLUID_LDS_MAX = 80 * 1024;
template <typename S, class L, int TY>
constexpr bool fluid_tile_fits() {
    return sizeof(FluidLds<S, L, TY, false>) <= FLUID_LDS_MAX;
}
// direct loads into LDS move one dword per lane (a shorter element would still take a dword slot
// of LDS per lane): FP32 populations only
template <typename S, class L, int TY>
constexpr bool fluid_halo_dma() {
    return sizeof(S) == 4 && sizeof(FluidLds<S, L, TY, true>) <= FLUID_LDS_MAX;
}

// one node's inputs of one plane: its stored populations, cell word and (FP16) previous psi
template <typename S, class L>
struct NodeIn {
    S v[L::Q];
    cell_t m;
    ArT<S> pp;
};

// psi of a node from its inputs (Sec. 3.2.3): fluid 1 - exp(-rho/rho0) with rho the sum of the
// populations (FP16: rho = R + sum of the stored deviations, the weights summing to one); a
// solid node carries the value of its body's wetting density.  v(I): stored population I.
template <typename S, class L, typename V>
__device__ __forceinline__ ArT<S> node_psi_of(const Prm<ArT<S>> &p, const BodyDev *__restrict__ bodies, cell_t m,
                                              ArT<S> pp, V v) {
    using T = ArT<S>;
    if (m & C_SOLID) return (T)bodies[owner_of(m)].psi_s;
    T r = T(0);
    if constexpr (sizeof(S) == 2) r = ref_density(pp, p.rho0);
    sfor<L::Q>([&](auto I) { r += (T)v(I); });
    return -expm1(-r * p.inv_rho0);
}

// The fluid pass (see above).  Launch: 64 W threads per block (W waves, one x-row of 64 nodes
// per wave and row set), tiles of 64 x TY nodes (thread (tx, w) owns rows w, w + W, ..), a 1-D
// grid of ceil(nx/64) * ceil(ny/TY) * ceil(nz/tz) blocks; blocks are ordered so that each XCD
// holds a contiguous run of tiles (a z-chunk of neighbouring tiles shares an L2).
//
// Software pipeline along z: while plane z is collided, the tile's own populations of plane z + 2
// are in flight into registers and (DMA) the halo's straight into LDS; at the top of the next
// pass they have landed, psi of plane z + 2 is formed, and so on.  Instantiations whose halo
// buffers do not fit the LDS budget load the halo of each plane just before its psi is formed.
//
// With bodies, block 0 is an extra one that only publishes the step's box, solid radii, volume terms
// and event flag from the previous reclassification (publish_step_state): that reduction chain runs
// beside the tiles instead of costing a launch, or, on a small grid where every tile runs at once,
// instead of delaying the block that would run it first.
template <typename S, class L, int TY, bool LONE>
__global__ __launch_bounds__(64 * FluidShape<TY>::W, (fluid_min_waves<S, L, TY, LONE>())) void k_collide_stream(Prm<ArT<S>> p, const S *__restrict__ fin,
                                                                     S *__restrict__ fout, ArT<S> *__restrict__ psi,
                                                                     ArT<S> *__restrict__ psi_prev,
                                                                     const cell_t *__restrict__ mask, BodyDev *bodies,
                                                                     int parity, StepState *st,
                                                                     const ClassifyPart *__restrict__ cpart, int cblk,
                                                                     const uint32_t *__restrict__ nbw, int tz) {
    using T = ArT<S>;
    constexpr int W = FluidShape<TY>::W, RPT = FluidShape<TY>::RPT;
    constexpr bool DMA = fluid_halo_dma<S, L, TY>();
    static_assert(fluid_tile_fits<S, L, TY>(), "LDS of the fluid pass above its budget");
    __shared__ FluidLds<S, L, TY, DMA> lds;
    constexpr bool H = sizeof(S) == 2;
    const int tid = (int)threadIdx.x, tx = tid & 63, wv = tid >> 6;
    const int extra = cpart ? 1 : 0;
    if (extra && blockIdx.x == 0) {
        publish_step_state(wv, W, parity, p.nx, p.ny, p.nz, p.tn, p.nb, p.eta, st, bodies, cpart, cblk);
        return;
    }
    // FP16 form: the bodies' motion for the moving-wall term into LDS (ordered before its first
    // use by the prologue's barrier)
    if constexpr (wall_in_fluid_pass<S>()) {
        for (int k = tid; k < p.nb * 9; k += 64 * W) {
            const int b = k / 9, c = k % 9;
            if (c < 3)
                lds.wm.X[b][c] = bodies[b].X[c];
            else if (c < 6)
                lds.wm.V[b][c - 3] = (float)bodies[b].V[c - 3];
            else
                lds.wm.W[b][c - 6] = (float)bodies[b].W[c - 6];
        }
    }
    auto wall_mot = [&]() -> const WallMot * {
        if constexpr (wall_in_fluid_pass<S>())
            return &lds.wm;
        else
            return nullptr;
    };
    const int nx = p.nx, ny = p.ny, nz = p.nz;
    const int tiles_x = (nx + 63) / 64, tiles_y = (ny + TY - 1) / TY, tiles = tiles_x * tiles_y;
    const int b = xcd_block((int)blockIdx.x - extra, (int)gridDim.x - extra);
    const int chunk = b / tiles, tile = b - chunk * tiles;
    const int tyi = tile / tiles_x, txi = tile - tyi * tiles_x;
    const int x0 = txi * 64, y0 = tyi * TY, zs = chunk * tz, ze = min(zs + tz, nz);
    const int x = x0 + tx;
    const uint32_t pl = (uint32_t)nx * (uint32_t)ny;
    // rows of this thread: ty = wv + W r; the node whose psi its window entry holds (a partial
    // tile's entries past the grid edge hold the periodic images the last nodes need)
    bool valid[RPT];
    uint32_t own_xy[RPT];
#pragma unroll
    for (int r = 0; r < RPT; ++r) {
        const int y = y0 + wv + W * r;
        valid[r] = x < nx && y < ny;
        own_xy[r] = (uint32_t)wrapi(x, nx) + (uint32_t)nx * (uint32_t)wrapi(y, ny);
    }
    // halo entry of this thread: row ly = -1 (wave 0), row ly = TY (wave 1), the two columns
    // lx = -1 and 64 for ly = -1..TY (wave 3, lanes 0 .. 2 TY + 3); hs: the wave's 64 entries
    // in the halo buffers
    int hlx = 0, hly = 0, hs = 0;
    bool halo = false;
    if (wv == 0 || wv == 1) {
        halo = true;
        hlx = tx;
        hly = wv == 0 ? -1 : TY;
        hs = 64 * wv;
    } else if (wv == 3) {
        halo = tx < 2 * (TY + 2);
        hlx = (tx & 1) ? 64 : -1;
        hly = (tx >> 1) - 1;
        hs = 128;
    }
    const uint32_t halo_xy = (uint32_t)wrapi(x0 + hlx, nx) + (uint32_t)nx * (uint32_t)wrapi(y0 + hly, ny);
    auto slot = [&](int zz) { return (zz - zs + 1) % 3; };
    auto hbuf = [&](int zz) { return DMA ? ((zz - zs + 1) & 1) : 0; };
    // The plane stride is re-read (opaque to the compiler) in every pass of the loop, so the 2 Q
    // plane addresses are formed on the scalar unit where they are used instead of being hoisted
    // out of the loop, where they would occupy more scalar registers than there are.
    auto plane_stride = [&]() {
        long long np = p.Np;
        asm volatile("" : "+s"(np));
        return np;
    };
    // loads of the own nodes' inputs of plane zz (issued, not waited for)
    auto load_own = [&](int zz, NodeIn<S, L> (&o)[RPT]) {
        const uint32_t zo = pl * (uint32_t)wrapi(zz, nz);
        const long long np = plane_stride();
#pragma unroll
        for (int r = 0; r < RPT; ++r) {
            const uint32_t idx = own_xy[r] + zo;
            o[r].m = mask[idx];
            o[r].pp = H ? psi_prev[idx] : T(0);
            const uint32_t is = idx * (uint32_t)sizeof(S);
            sfor<L::Q>([&](auto I) { o[r].v[I] = ldb(fin + (long long)I * np, is); });
        }
    };
    // the halo's inputs of plane zz straight into LDS buffer hb (DMA)
    // halo inputs of the plane in flight, where they go through registers (no DMA): prefetched one
    // pass ahead in the FP16 form; the FP64 form, short of registers, loads them when it needs them
    constexpr bool HPRE = !DMA && sizeof(S) == 2;
    NodeIn<S, L> hin;
    auto halo_load = [&](int zz, NodeIn<S, L> &o) {
        const uint32_t hidx = halo_xy + pl * (uint32_t)wrapi(zz, nz);
        const long long np = plane_stride();
        o.m = mask[hidx];
        o.pp = H ? psi_prev[hidx] : T(0);
        const uint32_t is = hidx * (uint32_t)sizeof(S);
        sfor<L::Q>([&](auto I) { o.v[I] = ldb(fin + (long long)I * np, is); });
    };
    // the halo's inputs of plane zz: straight into LDS buffer hb (DMA), else into registers
    // (issued, not waited for; in the prologue, prefetch = false, halo_psi loads them itself)
    auto halo_issue = [&](int zz, int hb, bool prefetch) {
        if constexpr (!DMA) {
            if (HPRE && prefetch && halo) halo_load(zz, hin);
        } else {
            if (!halo) return;
            const uint32_t hidx = halo_xy + pl * (uint32_t)wrapi(zz, nz);
            const long long np = plane_stride();
            sfor<L::Q>([&](auto I) {
                __builtin_amdgcn_global_load_lds(
                    (const __attribute__((address_space(1))) void *)(fin + (long long)I * np + hidx),
                    (__attribute__((address_space(3))) void *)&lds.hpop[hb][I][hs], 4, 0, 0);
            });
            __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void *)(mask + hidx),
                                             (__attribute__((address_space(3))) void *)&lds.hmask[hb][hs], 4, 0, 0);
        }
    };
    // psi of the halo entry of plane zz into the window: from the LDS buffer (DMA), from the
    // registers prefetched one pass earlier (prefetched), or loaded now (prologue)
    auto halo_psi = [&](int zz, bool prefetched) {
        if (!halo) return;
        T hp;
        cell_t hm;
        if constexpr (DMA) {
            const int hb = hbuf(zz), k = hs + tx;
            hm = lds.hmask[hb][k];
            hp = node_psi_of<S, L>(p, bodies, hm, T(0), [&](auto I) { return lds.hpop[hb][decltype(I)::value][k]; });
        } else {
            if (!(HPRE && prefetched)) halo_load(zz, hin);
            hm = hin.m;
            hp = node_psi_of<S, L>(p, bodies, hin.m, hin.pp, [&](auto I) { return hin.v[decltype(I)::value]; });
        }
        lds.ring[slot(zz)][hly + 1][hlx + 1] = win_entry<S>(hp, p.rho0, hm);
    };
    auto own_psi = [&](int zz, const NodeIn<S, L> (&o)[RPT]) {
#pragma unroll
        for (int r = 0; r < RPT; ++r)
            lds.ring[slot(zz)][wv + W * r + 1][tx + 1] = win_entry<S>(
                node_psi_of<S, L>(p, bodies, o[r].m, o[r].pp, [&](auto I) { return o[r].v[decltype(I)::value]; }),
                p.rho0, o[r].m);
    };

    // D3Q27: the neighbour-bit words of the plane being collided are loaded ahead of plane z + 2, as the
    // collision needs them first and loads are waited for in their order (FP32, 64^3: 42.1 -> 39.8 us,
    // 130^3: 209 -> 203).  In FP64 and in the one-block form, where they are needed only for streaming, behind
    // it (FP64 64^3 in chunks of 8 planes: 45.2 us, loaded ahead 48.5; one block, 250^3: 977 and 1012).
    constexpr bool NBPRE = !L::kBits && sizeof(S) < 8 && !LONE;
    NodeIn<S, L> A[RPT], B[RPT];
    // prologue: psi of planes zs - 1 and zs, populations of plane zs into LDS, plane zs + 1 in
    // flight
    load_own(zs - 1, A);
    own_psi(zs - 1, A);
    halo_issue(zs - 1, hbuf(zs - 1), false);
    halo_issue(zs, hbuf(zs), false);
    load_own(zs, A);
    load_own(zs + 1, B);
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __syncthreads();
    halo_psi(zs - 1, false);
    halo_psi(zs, false);
    own_psi(zs, A);
#pragma unroll
    for (int r = 0; r < RPT; ++r) sfor<L::Q>([&](auto I) { lds.pop[I][tid + 64 * W * r] = A[r].v[I]; });
    cell_t cm[RPT];  // cell words of the plane being collided
    T cpp[RPT];      // and their previous psi (FP16)
#pragma unroll
    for (int r = 0; r < RPT; ++r) {
        cm[r] = A[r].m;
        cpp[r] = A[r].pp;
    }
    halo_issue(zs + 1, hbuf(zs + 1), true);
    for (int z = zs; z < ze; ++z) {
        // plane z + 1 has landed (own populations in B, halo in its LDS buffer); every wave is done
        // with the previous plane's window entries and halo buffer
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        __syncthreads();
        const uint32_t zo = pl * (uint32_t)z;
        uint32_t nb[RPT];
#pragma unroll
        for (int r = 0; r < RPT; ++r) nb[r] = NBPRE ? nbw[own_xy[r] + zo] : 0u;
        own_psi(z + 1, B);
        halo_psi(z + 1, true);
#pragma unroll
        for (int r = 0; r < RPT; ++r) A[r] = B[r];
        if (z + 2 <= ze) {
            load_own(z + 2, B);
            halo_issue(z + 2, hbuf(z + 2), true);
        }
        __syncthreads();
#pragma unroll
        for (int r = 0; r < RPT; ++r) {
            const int ty = wv + W * r;
            // own populations of plane z from LDS, those of plane z + 1 in their place
            S cur[L::Q];
            sfor<L::Q>([&](auto I) { cur[I] = lds.pop[I][tid + 64 * W * r]; });
            sfor<L::Q>([&](auto I) { lds.pop[I][tid + 64 * W * r] = A[r].v[I]; });
            // the stores stay here, ahead of the collision (sunk below it, they would keep the next
            // plane's populations in registers through the collision)
            asm volatile("" ::: "memory");
            if (valid[r]) {
                const uint32_t idx = own_xy[r] + zo;
                // the node's entry in each window plane: neighbours are fixed offsets from it
                const WinE<S> *rm = &lds.ring[slot(z - 1)][ty + 1][tx + 1], *r0 = &lds.ring[slot(z)][ty + 1][tx + 1],
                              *rp = &lds.ring[slot(z + 1)][ty + 1][tx + 1];
                const T psi0 = win_psi<S>(*r0);
                psi[idx] = psi0;
                const cell_t w0 = cm[r];
                if (!(w0 & C_SOLID)) {
                    // bit i: the neighbour in direction i is solid (D3Q19: kept in the cell word;
                    // D3Q27: the neighbour-bit word of the node)
                    uint32_t solid_dirs;
                    if constexpr (L::kBits)
                        solid_dirs = w0 & C_NBMASK;
                    else
                        solid_dirs = NBPRE ? nb[r] : nbw[idx];
                    const T rin = H ? ref_density(cpp[r], p.rho0) : T(0);  // reference of the inputs
                    // the neighbour's window entry: fixed offsets from the node's
                    auto nbr = [&](auto I) -> const WinE<S> & {
                        constexpr int i = decltype(I)::value;
                        constexpr int o = Dir<i, L>::y * 66 + Dir<i, L>::x;
                        return Dir<i, L>::z < 0 ? rm[o] : (Dir<i, L>::z > 0 ? rp[o] : r0[o]);
                    };
                    collide_push<S, L, LONE>(
                        p, cur, rin, [&](auto I) { return win_psi<S>(nbr(I)); },
                        [&](auto I) { return win_ref<S>(nbr(I)); }, psi0, win_ref<S>(*r0), fout, solid_dirs, x,
                        y0 + ty, z, plane_stride(), wall_mot(), psi_prev);
                }
            }
            cm[r] = A[r].m;
            cpp[r] = A[r].pp;
        }
    }
}

// Per-body force and torque sums of the step over the box nodes (Sec. 3.1.1, 3.1.2, 3.2.2):
//  * fluid nodes next to solid nodes: the fluid pass reflected each population f*_i heading into
//    a solid node into the node's opposite slot; unless the fluid pass did so (wall_in_fluid_pass),
//    this kernel completes the moving-wall bounce-back of Sec. 3.2.2 there -- the slot becomes
//    f*_i + g_i with g_i = -2 rho w_i (c_i . u_w) / c_s^2 and the rest population gives back the
//    sum of the g_i (mass correction) -- and it adds to body b the momentum exchange
//    c_i (2 f*_i + g_i) of each link into b, plus the pseudopotential reaction
//    +G psi(x) w_i psi(varrho_b) c_i (opposite of the fluid's share), with the link midpoint as
//    lever arm;
//  * solid nodes (repulsion enabled): between a node p of body b1 and a node q of body b2 > b1
//    with |p - q| < r_c, f = e0 (n/r_c) (p - q)/|p - q| |(|p - q| - r_c)/r_c|^(n-1) on b1 at p
//    and -f on b2 at q; only nodes within r_c of a higher-index body's solid radius search.
// Torques are about the body centres X_b (minimum image).  Each wave reduces its contributions
// per touched body (64-lane shuffles) into LDS in a fixed order and every block writes FP64
// partials [body * 6 + component][block], summed by the rigid-body update (k_tile_activity).
//
// What bounds it: each wave runs a chain of four or five dependent memory rounds once, so the
// kernel is bound by latency and by the number of instructions on a wave's path (a SIMD holds one
// or two waves here, which issue one instruction in four cycles at best, and code that every wave
// runs once is fetched cold).  The work of one node is therefore split over lanes: the links of a
// node over eight lanes, the offsets of the repulsion search over the whole wave, and the six sums
// of a body share one exchange tree.  On large boxes the cache lines of the scattered nodes bound it,
// so only the planes of real links are read and the density comes from the fluid pass.  Against one
// lane per node with unrolled searches (67 KB of code, now 14 KB), in FP32 unless noted: 61 x 45 x 50
// two spheres 15.7 -> 8.5 us, 128^3 two spheres 18.7 -> 13.9 (D3Q27 25.1 -> 16.2), 256^3 four spheres
// 42.9 -> 27.1 (FP16 storage 31.4 -> 27.4), 32^3 plates FP64 37.6 -> 23.0, and 17.2 with the repulsion
// search of eight nodes loaded in one round.
constexpr int FORCE_WAVES = 12;  // waves per block of the force scan (one block per CU)

// component d of direction i known only at run time, from two-bit fields; i may reach 32 (the last lane of
// a node's eight on D3Q27), where the shift by 64 wraps and the result is not used
__host__ __device__ __forceinline__ constexpr int dir_rt(int i, int d) {
    constexpr auto pack = [](const int *c) {
        unsigned long long v = 0;
        for (int k = 0; k < 27; ++k) v |= (unsigned long long)(c[k] + 1) << (2 * k);
        return v;
    };
    constexpr unsigned long long X = pack(kCX), Y = pack(kCY), Z = pack(kCZ);
    return (int)(((d == 0 ? X : (d == 1 ? Y : Z)) >> ((2 * i) & 63)) & 3u) - 1;
}
static_assert(dir_rt(32, 0) == dir_rt(0, 0) && dir_rt(26, 2) == kCZ[26], "directions defined for every lane");

// periodic wrap by repeated addition (usually none; several on an axis shorter than the offset)
__device__ __forceinline__ int wrapl(int i, int n) {
    while (i < 0) i += n;
    while (i >= n) i -= n;
    return i;
}

// Totals of six values over a wave, in a fixed order: three halving exchanges leave each lane one
// component's sum over the 8 lanes that share its low bits, three more finish it.  Lane l returns
// the total of component l >> 3 (0..5; 0 for 6 and 7).
__device__ __forceinline__ double wave_sum6(const double (&v)[6]) {
    const int lane = (int)(threadIdx.x & 63);
    const bool h5 = lane & 32, h4 = lane & 16, h3 = lane & 8;
    double a[4], b[2];
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        const double up = j < 2 ? v[(4 + j) % 6] : 0.0;
        a[j] = (h5 ? up : v[j]) + __shfl_xor(h5 ? v[j] : up, 32, 64);
    }
#pragma unroll
    for (int j = 0; j < 2; ++j) b[j] = (h4 ? a[2 + j] : a[j]) + __shfl_xor(h4 ? a[j] : a[2 + j], 16, 64);
    double c = (h3 ? b[1] : b[0]) + __shfl_xor(h3 ? b[0] : b[1], 8, 64);
#pragma unroll
    for (int off = 4; off > 0; off >>= 1) c += __shfl_xor(c, off, 64);
    return c;
}

// s plus m times the values that eight lanes hold of directions 1 + q, 9 + q, .. (v[k] of lane q:
// direction 1 + q + 8 k), added in the order of the directions with one rounding each, in each of
// the lanes
template <int Q, typename T, int NS>
__device__ __forceinline__ T ordered_sum(T s, const T (&v)[NS], T m) {
#pragma unroll
    for (int i = 1; i < Q; ++i) {
        const T x = __shfl(v[(i - 1) / 8], (i - 1) % 8, 8);
        if constexpr (sizeof(T) == 8)
            s = __builtin_fma(x, m, s);
        else
            s = __builtin_fmaf(x, m, s);
    }
    return s;
}

template <typename S, class L>
__global__ __launch_bounds__(64 * FORCE_WAVES) void k_body_forces(Prm<ArT<S>> p, int parity,
                                                     const StepState *st, const S *__restrict__ fin,
                                                     S *__restrict__ fpost, const ArT<S> *__restrict__ psi,
                                                     const ArT<S> *__restrict__ psi_prev,
                                                     const cell_t *__restrict__ mask,
                                                     const BodyDev *__restrict__ bodies, double *part,
                                                     const uint32_t *__restrict__ nbw) {
    using T = ArT<S>;
    constexpr int W = FORCE_WAVES, NT = 64 * W;
    __shared__ double acc[W][PF_LBM_MAX_BODIES][6];
    __shared__ double bt[PF_LBM_MAX_BODIES][10];  // X, V, W and psi of every body
    const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
    const int nbod = p.nb;
    // each wave clears and fills only its own row of the sums
    for (int k = lane; k < nbod * 6; k += 64) (&acc[wave][0][0])[k] = 0.0;
    if (tid < nbod * 10) {
        const BodyDev &B = bodies[tid / 10];
        const int c = tid % 10;
        bt[tid / 10][c] = c < 3 ? B.X[c] : (c < 6 ? B.V[c - 3] : (c < 9 ? B.W[c - 6] : B.psi_s));
    }
    __syncthreads();
    const BoxIter it(st->box[parity], p.nx, p.ny, p.nz);
    const int nx = p.nx, ny = p.ny, nz = p.nz;
    const long long Np = p.Np;
    const bool rep = nbod > 1 && (p.flags & PF_LBM_REPULSION);
    // offset of a point from the centre of body b (minimum image)
    auto lever = [&](int b, const int *c, double *r) {
        const double *BX = bt[b];
        r[0] = mimg_r(c[0] - BX[0], nx, p.inv_n[0]);
        r[1] = mimg_r(c[1] - BX[1], ny, p.inv_n[1]);
        r[2] = mimg_r(c[2] - BX[2], nz, p.inv_n[2]);
    };
    // the totals of one body over the wave into its sums
    auto add = [&](int b, const double (&v)[6]) {
        const double s = wave_sum6(v);
        if ((lane & 7) == 0 && lane < 48) acc[wave][b][lane >> 3] += s;
    };
    // A wave takes U rounds of 64 box cells, in runs of RUN consecutive cells, the runs nw * RUN cells
    // apart (nw waves in the grid), so that the cells with work -- clustered on the bodies'
    // surfaces and, for the repulsion, in the small caps where two bodies nearly touch -- spread
    // over all waves.  A first pass loads the cell words of the U rounds together and keeps the
    // cells that need work: from the front of the list the fluid cells with a solid neighbour, from
    // its back the solid cells within r_c of the solid radius of a higher-index body.  (Runs of 64
    // cells: 11.9 instead of 8.5 us at 61 x 45 x 50, 41.9 instead of 23.0 on the 32^3 plates,
    // before the search took eight nodes a round.)
    constexpr int U = 4, CAP = 64 * U, RUN = 16, RPW = 64 / RUN;
    __shared__ int keep[W][CAP];
    __shared__ unsigned char kown[W][CAP];  // owners of the kept solid cells
    const int gw = (int)blockIdx.x * W + wave, nw = (int)gridDim.x * W;
    // cell of this lane in round u of the runs that start at s0, and the first cell of the round
    auto cell_of = [&](long long s0, int u) { return ((s0 + u * RPW + lane / RUN) * nw + gw) * RUN + (lane & (RUN - 1)); };
    for (long long s0 = 0; (s0 * nw + gw) * RUN < it.vol; s0 += RPW * U) {
        int nlink = 0, nrepc = 0;
        {
            cell_t wk[U];
            uint32_t nbk[U];
            // rounds past the end of the box are skipped by the whole wave
#pragma unroll
            for (int u = 0; u < U; ++u) {
                wk[u] = nbk[u] = 0;
                if (((s0 + RPW * u) * nw + gw) * RUN < it.vol) {
                    const long long k = cell_of(s0, u);
                    if (k < it.vol) {
                        int uu[3], c[3];
                        it.cell((int)k, uu, c);
                        const int idx = c[0] + nx * (c[1] + ny * c[2]);
                        wk[u] = mask[idx];
                        if constexpr (!L::kBits) nbk[u] = nbw[idx];
                    }
                }
            }
#pragma unroll 1
            for (int u = 0; u < U; ++u) {
                const cell_t w = u == 0 ? wk[0] : (u == 1 ? wk[1] : (u == 2 ? wk[2] : wk[3]));
                const uint32_t nb = u == 0 ? nbk[0] : (u == 1 ? nbk[1] : (u == 2 ? nbk[2] : nbk[3]));
                const int k = (int)cell_of(s0, u);
                const bool solid = (w & C_SOLID) != 0;
                const bool link = !solid && (L::kBits ? w & C_NBMASK : nb) != 0;
                const uint64_t bal = __ballot(link);
                if (link) keep[wave][nlink + __popcll(bal & ((1ull << lane) - 1ull))] = k;
                nlink += __popcll(bal);
                if (rep && __ballot(solid)) {
                    bool need = false;
                    if (solid) {
                        int uu[3], c[3];
                        it.cell(k, uu, c);
                        for (int b2 = owner_of(w) + 1; b2 < nbod; ++b2) {
                            double r[3];
                            lever(b2, c, r);
                            const double reach = (double)st->srad[b2] + p.r_c + 1e-3;
                            need = need || r[0] * r[0] + r[1] * r[1] + r[2] * r[2] < reach * reach;
                        }
                    }
                    const uint64_t bas = __ballot(need);
                    if (need) {
                        const int slot = CAP - 1 - nrepc - __popcll(bas & ((1ull << lane) - 1ull));
                        keep[wave][slot] = k;
                        kown[wave][slot] = (unsigned char)owner_of(w);
                    }
                    nrepc += __popcll(bas);
                }
            }
        }
        __builtin_amdgcn_wave_barrier();
        // links: eight lanes per node, lane q of them takes the directions 1 + q, 9 + q, ...
        constexpr int NS = (L::Q + 6) / 8;
        for (int j0 = 0; j0 < nlink; j0 += 8) {
            // the lane's directions are formed anew in each round (opaque to the compiler, which would
            // keep their components, weights and offsets in registers across the whole kernel)
            int q = lane & 7;
            asm volatile("" : "+v"(q));
            const bool has = j0 + (lane >> 3) < nlink;
            uint32_t touched = 0;
            int c[3] = {0, 0, 0};
            uint32_t is = 0;
            T rho = T(0), rown = T(0), drho = T(0), f0 = T(0);
            // per link i into a solid neighbour: its owner (-1: no link), the reflected post-collision
            // population fr = f*_i and the body-independent part of the link force, a = 2 f*_i +
            // G psi(x) w_i psi(x + c_i); drho sums the moving-wall terms of the node's links
            int own[NS];
            T a[NS], fr[NS], fq[NS];
            if (has) {
                int u[3];
                it.cell(keep[wave][j0 + (lane >> 3)], u, c);
                const uint32_t idx = (uint32_t)(c[0] + nx * (c[1] + ny * c[2]));
                is = idx * (uint32_t)sizeof(S);
                const NbrU ne(c[0], c[1], c[2], nx, ny, nz, 1);
                uint32_t nbits;
                if constexpr (L::kBits)
                    nbits = mask[idx] & C_NBMASK;
                else
                    nbits = nbw[idx];
                // The gathers of the node are issued in one round and unconditionally, so the
                // per-link selects below wait for memory once; loads inside per-link branches were
                // serialised, one memory latency per link.  A direction without a link reads the node's
                // own word and rest population instead, so that no cache line is fetched for it (the
                // lines bound this kernel on large boxes: each holds one or two of the scattered nodes).
                // The psi of a solid neighbour is its owner's.
                cell_t mo[NS];
                S fo[NS], fi[NS + 1], fr0;
                fr0 = ldb(fpost, is);
                const T ps0 = psi[idx], pp = psi_prev[idx];
                if constexpr (wall_in_fluid_pass<S>()) fi[NS] = ldb(fin, is);
#pragma unroll
                for (int k = 0; k < NS; ++k) {
                    const int i = 1 + q + 8 * k;
                    const bool on = i < L::Q;
                    const int opp = (i & 1) ? i + 1 : i - 1;
                    if constexpr (wall_in_fluid_pass<S>()) fi[k] = ldb(fin + (long long)(on ? i : 0) * Np, is);
                    const int dx = dir_rt(i, 0), dy = dir_rt(i, 1), dz = dir_rt(i, 2);
                    const bool link = on && (nbits & (1u << i));
                    own[k] = link ? 0 : -1;
                    fo[k] = ldb(fpost + (long long)(link ? opp : 0) * Np, is);
                    const uint32_t n = link ? idx + (dx > 0 ? ne.xp : (dx < 0 ? ne.xm : 0u)) +
                                                  (dy > 0 ? ne.yp : (dy < 0 ? ne.ym : 0u)) +
                                                  (dz > 0 ? ne.zp : (dz < 0 ? ne.zm : 0u))
                                            : idx;
                    mo[k] = ldb(mask, n * 4u);
                }
                rown = sizeof(S) == 2 ? ref_density(ps0, p.rho0) : T(0);
                f0 = pop_get<S>(fr0, Dir<0, L>::template w<T>(), rown);
                // density of the node: left by the fluid pass, or (FP16) summed from its populations
                if constexpr (!wall_in_fluid_pass<S>())
                    rho = pp;
                else
                    rho = ref_density(pp, p.rho0) + (T)fi[NS];
                const T gp = p.G * ps0;
#pragma unroll
                for (int k = 0; k < NS; ++k) {
                    const int i = 1 + q + 8 * k;
                    if constexpr (wall_in_fluid_pass<S>()) fq[k] = (T)fi[k];
                    if (own[k] >= 0) own[k] = owner_of(mo[k]) & (PF_LBM_MAX_BODIES - 1);
                    touched |= own[k] >= 0 ? 1u << own[k] : 0u;
                    const int c2 = i <= 6 ? 1 : (i <= 18 ? 2 : 3);
                    const T w = T(L::wshell[1]) * T(c2 == 1) + T(L::wshell[2]) * T(c2 == 2) + T(L::wshell[3]) * T(c2 == 3);
                    // reflected value: f*_i, or f*_i + g_i where the fluid pass added g
                    fr[k] = pop_get<S>(fo[k], w, rown);
                    const T ps = (T)bt[max(own[k], 0)][9];
                    if constexpr (sizeof(S) == 2)
                        a[k] = __builtin_fmaf(gp * w, ps, T(2) * fr[k]);
                    else
                        a[k] = T(2) * fr[k] + gp * w * ps;
                }
            }
            if constexpr (wall_in_fluid_pass<S>()) rho = ordered_sum<L::Q>(rho, fq, T(1));
            for (int b = 0; b < nbod; ++b) {
                if (!__ballot(touched & (1u << b))) continue;
                double v[6] = {0, 0, 0, 0, 0, 0};
                T gs[NS] = {};
                if (touched & (1u << b)) {
                    // The link midpoint is x + c_i/2, so with r the node's offset from the centre:
                    // c_i . u_w(x + c_i/2) = c_i . u_w(x) (the term c_i . (W x c_i)/2 vanishes) and
                    // (r + c_i/2) x s c_i = r x s c_i.  The wall term needs the node's rigid velocity
                    // only, and the torque is r x (sum of the link forces).
                    const double *BV = bt[b] + 3, *BW = BV + 3;
                    double r[3];
                    lever(b, c, r);
                    const double u0x = BV[0] + (BW[1] * r[2] - BW[2] * r[1]), u0y = BV[1] + (BW[2] * r[0] - BW[0] * r[2]),
                                 u0z = BV[2] + (BW[0] * r[1] - BW[1] * r[0]);
#pragma unroll
                    for (int k = 0; k < NS; ++k) {
                        if (own[k] == b) {
                            const int i = 1 + q + 8 * k, opp = (i & 1) ? i + 1 : i - 1;
                            const double dx = dir_rt(i, 0), dy = dir_rt(i, 1), dz = dir_rt(i, 2);
                            const int c2 = i <= 6 ? 1 : (i <= 18 ? 2 : 3);
                            const double w = c2 == 1 ? L::wshell[1] : (c2 == 2 ? L::wshell[2] : L::wshell[3]);
                            const double cuw = dx * u0x + dy * u0y + dz * u0z;
                            // moving-wall term g: the reflected population becomes f*_i + g (Sec.
                            // 3.2.2); the link carries 2 f*_i + g to the body plus the
                            // pseudopotential reaction, both along c_i
                            const T gr = T(-6.0 * w * cuw), g = gr * rho;
                            double s;
                            if constexpr (!wall_in_fluid_pass<S>()) {
                                stb(fpost + (long long)opp * Np, is, pop_put<S>(fr[k] + g, (T)w, rown));
                                gs[k] = gr;
                                s = (double)(a[k] + g);
                            } else {
                                s = (double)(a[k] - g);  // 2 (f*_i + g) - g
                            }
                            v[0] += dx * s;
                            v[1] += dy * s;
                            v[2] += dz * s;
                        }
                    }
                    v[3] = r[1] * v[2] - r[2] * v[1];
                    v[4] = r[2] * v[0] - r[0] * v[2];
                    v[5] = r[0] * v[1] - r[1] * v[0];
                }
                add(b, v);
                if constexpr (!wall_in_fluid_pass<S>()) drho = ordered_sum<L::Q>(drho, gs, rho);
            }
            // the rest population gives back the moving-wall terms (mass correction, Sec. 3.2.2)
            if constexpr (!wall_in_fluid_pass<S>())
                if (has && q == 0) stb(fpost, is, pop_put<S>(f0 - drho, Dir<0, L>::template w<T>(), rown));
        }
        // Repulsion between a solid node p of body b1 and the solid nodes q = p + d of bodies above
        // b1: the force on b1 at p, its opposite on b2 at q.  The n_rep offsets lie across the lanes, two
        // rounds (r_c = 3 needs two, r_c = 4 four) of PN nodes loaded together; the sums run per body b2
        // met.  With r the offset of p from a centre, the torque of the reaction is r x (-s) - sum d x f.
        constexpr int PN = 8;
        const int nrep = nrepc ? st->n_rep : 0;
        for (int o0 = 0; o0 < nrep; o0 += 128) {
            int o[2], dx[2], dy[2], dz[2];
#pragma unroll
            for (int t = 0; t < 2; ++t) {
                o[t] = o0 + 64 * t + lane;
                const int w = st->rep_off[min(o[t], nrep - 1)];
                dx[t] = (w & 255) - 8;
                dy[t] = ((w >> 8) & 255) - 8;
                dz[t] = (w >> 16) - 8;
            }
            const int doff[2] = {dx[0] + nx * (dy[0] + ny * dz[0]), dx[1] + nx * (dy[1] + ny * dz[1])};
            for (int j0 = 0; j0 < nrepc; j0 += PN) {
                // lane j < PN: node j of the batch; away from the grid's faces its neighbours are fixed offsets
                int nd, bown, u[3], c[3];
                {
                    const int slot = CAP - 1 - min(j0 + (lane & (PN - 1)), nrepc - 1);
                    it.cell(keep[wave][slot], u, c);
                    nd = c[0] + nx * (c[1] + ny * c[2]);
                    bown = kown[wave][slot];
                }
                const bool inner = min(min(c[0], c[1]), c[2]) >= 4 && c[0] < nx - 4 && c[1] < ny - 4 && c[2] < nz - 4;
                uint32_t any = 0;  // pairs (node, round) of the batch that meet a body above the node's
                auto meets = [&](int j, int t, cell_t m) {
                    const bool on = (t ? o[1] : o[0]) < nrep && (m & C_SOLID);
                    if (__ballot(on && owner_of(m) > __builtin_amdgcn_readlane(bown, j))) any |= 1u << (2 * j + t);
                };
                if (!__ballot(!inner)) {
                    cell_t mq[PN][2];
#pragma unroll
                    for (int j = 0; j < PN; ++j)
#pragma unroll
                        for (int t = 0; t < 2; ++t) mq[j][t] = mask[__builtin_amdgcn_readlane(nd, j) + doff[t]];
#pragma unroll
                    for (int j = 0; j < PN; ++j)
#pragma unroll
                        for (int t = 0; t < 2; ++t) meets(j, t, mq[j][t]);
                } else {
#pragma unroll 1
                    for (int k = 0; k < 2 * PN; ++k) {
                        const int j = k >> 1, t = k & 1;
                        const int x = __builtin_amdgcn_readlane(c[0], j) + (t ? dx[1] : dx[0]),
                                  y = __builtin_amdgcn_readlane(c[1], j) + (t ? dy[1] : dy[0]),
                                  z = __builtin_amdgcn_readlane(c[2], j) + (t ? dz[1] : dz[0]);
                        meets(j, t, mask[wrapl(x, nx) + nx * (wrapl(y, ny) + ny * wrapl(z, nz))]);
                    }
                }
                if (nrepc - j0 < PN) any &= (1u << (2 * (nrepc - j0))) - 1u;
                while (any) {  // rare: one pair at a time, its words loaded again
                    const int pr = __ffs(any) - 1, t = pr & 1;
                    any &= any - 1;
                    const int slot = CAP - 1 - (j0 + (pr >> 1)), bj = kown[wave][slot];
                    int u[3], cj[3];
                    it.cell(keep[wave][slot], u, cj);
                    const int ot = t ? o[1] : o[0], ex = t ? dx[1] : dx[0], ey = t ? dy[1] : dy[0], ez = t ? dz[1] : dz[0];
                    const bool on = ot < nrep;
                    const cell_t m = mask[wrapl(cj[0] + ex, nx) + nx * (wrapl(cj[1] + ey, ny) + ny * wrapl(cj[2] + ez, nz))];
                    const int b2 = on && (m & C_SOLID) ? owner_of(m) : -1;
                    uint64_t hits = __ballot(b2 > bj);
                    double fx = 0.0, fy = 0.0, fz = 0.0;
                    if (on) {
                        fx = st->rep_f[ot][0];
                        fy = st->rep_f[ot][1];
                        fz = st->rep_f[ot][2];
                    }
                    while (hits) {
                        const int bb = __shfl(b2, (int)__builtin_ctzll(hits), 64);
                        const bool mine = b2 == bb;
                        hits &= ~__ballot(mine);
                        const double v[6] = {mine ? fx : 0.0,
                                             mine ? fy : 0.0,
                                             mine ? fz : 0.0,
                                             mine ? ey * fz - ez * fy : 0.0,
                                             mine ? ez * fx - ex * fz : 0.0,
                                             mine ? ex * fy - ey * fx : 0.0};
                        const double tot = wave_sum6(v);
                        double s[3], td[3], r1[3], r2[3];
                        for (int k = 0; k < 3; ++k) {
                            s[k] = __shfl(tot, 8 * k, 64);
                            td[k] = __shfl(tot, 8 * (3 + k), 64);
                        }
                        lever(bj, cj, r1);
                        lever(bb, cj, r2);
                        if (lane == 0) {
                            double *A = acc[wave][bj], *R = acc[wave][bb];
                            for (int k = 0; k < 3; ++k) {
                                const int m1 = (k + 1) % 3, m2 = (k + 2) % 3;
                                A[k] += s[k];
                                A[3 + k] += r1[m1] * s[m2] - r1[m2] * s[m1];
                                R[k] -= s[k];
                                R[3 + k] -= r2[m1] * s[m2] - r2[m2] * s[m1] + td[k];
                            }
                        }
                    }
                }
            }
        }
        __builtin_amdgcn_wave_barrier();
    }
    __syncthreads();
    for (int k = tid; k < nbod * 6; k += NT) {
        const int b = k / 6, c = k % 6;
        double s = 0.0;
        for (int w = 0; w < W; ++w) s += acc[w][b][c];
        part[(long long)k * gridDim.x + blockIdx.x] = s;
    }
}

}  // namespace pfl

// Several D2Q9 steps of a small lattice in one launch.
//
// A step of the other paths is 2 to 5 launches, each a chain of memory round
// trips: about 10 us (fused) or 20 us (x walls) whatever the lattice, where the
// arithmetic of a few hundred cells takes one or two.  Here a workgroup keeps a
// region of the lattice, a thread per cell, its populations in registers, and
// takes `steps` steps with the stencils and the streaming through LDS; nothing
// touches HBM in between.  A region is the whole lattice, or all rows of a run
// of own columns with 4 `steps` columns on either side: a step reaches four
// cells (streaming one, the collision's gradients one, the force one, the
// Laplacian one), so what the missing neighbours spoil stays outside the own
// columns.  Every cell's arithmetic is the same wherever it lies in a region:
// the result does not depend on the split.
//
// Bound by the latency of the arithmetic, one or two wavefronts per SIMD.
#pragma once

#include "lbm_fused.hpp"

namespace lbm {

template <class C, class T> struct Block2DArgs {
    Grid g;
    Phys<C> ph;
    RefPops ref;
    Walls w;
    int own;    // own columns per workgroup (nx: one workgroup, whole lattice)
    int halo;   // columns on either side of them (0: whole lattice)
    int steps;  // 4 steps <= halo, unless the region is the whole lattice
    int pull;   // form of the input set: 0 arrived, 1 post-collision
    C rsf_hi, rsf_lo, rsg_hi, rsg_lo;  // sums of the reference populations
    const T *fi;
    T *fo;
};

// In the arithmetic of the fused step.  WALL: diffuse-reflection x walls; the
// arrived set goes out, since what a wall's ghost emits has no place in the
// post-collision set, which goes out otherwise.  FP64 and FP32 storage, van der
// Waals.
//
// Larger lattices between walls take the multi-kernel step, whose divisions are
// rounded correctly.  In FP32 the hardware reciprocal of rho alone would make u
// drift away from FP64 faster than that step does (64 x 4 cells, 200 steps:
// errors 0.44, 1.24, 0.35, 0.34 of the multi-kernel step's in rho, u, T, P);
// corrected 0.23, 0.62, 0.04, 0.05 at 2.44 us per step against 2.41.  Correcting
// the other quotients too changed none of these.
template <class S, bool WALL, int NT>
__global__ void __launch_bounds__(NT) k_block2d(Block2DArgs<typename S::C, typename S::T> a) {
    using C = typename S::C;
    constexpr int Q = 9;
    __shared__ C sRho[NT], sLap[NT];
    __shared__ C sU[2][NT], sT[NT], sH[NT], sL[2][NT];
    __shared__ C sF[Q][NT], sG[Q][NT];
    __shared__ C sE[WALL ? 2 : 1][3][2][WALL ? NT : 1];  // emitted f, g by side, direction and ghost row
    const Grid g = a.g;
    Phys<C> ph = a.ph;
    ph.pr = 0;  // van der Waals only
    const int h = g.ny, rw = a.own + 2 * a.halo, n = rw * h;
    const bool live = (int)threadIdx.x < n;  // other threads keep to the barriers
    const int t = live ? threadIdx.x : n - 1;
    const int ry = t / rw, rx = t - ry * rw;
    const int x0 = blockIdx.x * a.own;
    const int gx = x0 - a.halo + rx;  // beyond the lattice in a halo: a periodic image, or a cell of no use
    int x = gx;
    if (g.clampx) x = min(max(x, 0), g.nx - 1);
    else {
        x %= g.nx;
        if (x < 0) x += g.nx;
    }
    const int y = ry;
    const bool own = live && rx >= a.halo && gx < min(x0 + a.own, g.nx) && rx < a.halo + a.own;
    // the cell's neighbours in the region; beyond a zero-gradient wall, and at
    // the region's own ends, the cell itself
    int xm = rx - 1, xp = rx + 1, ym = y - 1, yp = y + 1;
    if (g.clampx) {
        if (gx <= 0) xm = rx;
        if (gx >= g.nx - 1) xp = rx;
    } else if (a.halo == 0) {
        if (xm < 0) xm = rw - 1;
        if (xp >= rw) xp = 0;
    }
    xm = max(xm, 0);
    xp = min(xp, rw - 1);
    ym = ym < 0 ? (g.clampy ? 0 : h - 1) : ym;
    yp = yp >= h ? (g.clampy ? h - 1 : 0) : yp;
    const int cW = ry * rw + xm, cE = ry * rw + xp, cS = ym * rw + rx, cN = yp * rw + rx;
    // where the arrived population with velocity c comes from, per axis
    const int px[3] = {xp, rx, xm}, py[3] = {yp * rw, ry * rw, ym * rw};
    const bool wall_lo = WALL && gx == 0, wall_hi = WALL && gx == g.nx - 1;
    // the cell's walls: one each, so both sides go through the same
    // instructions, but on a lattice of one column
    const int nwall = g.nx == 1 ? 2 : 1;
    auto wall_of = [&](int k) { return g.nx == 1 ? k : (wall_hi ? 1 : 0); };

    C f[Q], gq[Q];
#pragma unroll
    for (int i = 0; i < Q; i++) {
        const PopPair<typename S::T> p = load_pair(a.fi, arrived_index<2>(g, i, x, y, 0, a.pull));
        f[i] = S::load(&p.f, 0, (C)a.ref.f[i]);
        gq[i] = S::load(&p.g, 0, (C)a.ref.g[i]);
    }
    for (int s = 0; s < a.steps; s++) {
        // -- moments ----------------------------------------------------------
        C rho, J[2], G;
        {
            C v[Q], tg;
#pragma unroll
            for (int i = 0; i < Q; i++) {
                v[i] = S::dev(&f[i], 0, (C)a.ref.f[i]);
                const C d = S::dev(&gq[i], 0, (C)a.ref.g[i]);
                tg = i == 0 ? d : tg + d;
            }
            const C r0 = v[0] + v[1] + v[2], r1 = v[3] + v[4] + v[5], r2 = v[6] + v[7] + v[8];
            rho = (r0 + r1 + r2 + a.rsf_lo) + a.rsf_hi;
            J[0] = (v[2] + v[5] + v[8]) - (v[0] + v[3] + v[6]);
            J[1] = r2 - r0;
            G = (tg + a.rsg_lo) + a.rsg_hi;
        }
        if (live) sRho[t] = rho;
        __syncthreads();
        {
            const C l = sRho[cE] + sRho[cW] - C(2) * rho + sRho[cN] + sRho[cS] - C(2) * rho;
            if (live) sLap[t] = l;
        }
        __syncthreads();
        // -- fields -----------------------------------------------------------
        const C inv_rho = reciprocal<WALL>(rho);
        C F[2], u[2], Lam[2];
        F[0] = ph.kappa * rho * (C(0.5) * (sLap[cE] - sLap[cW]));
        F[1] = ph.kappa * rho * (C(0.5) * (sLap[cN] - sLap[cS]));
        C uF = 0, u2 = 0;
        for (int d = 0; d < 2; d++) {
            u[d] = (J[d] + C(0.5) * F[d]) * inv_rho;
            uF += u[d] * F[d];
            u2 += u[d] * u[d];
        }
        const C e = (G + C(0.5) * uF) * inv_rho - C(0.5) * u2;
        const C T = (e + ph.a * rho) * ph.inv_cv;
        C P, cs2;
        vdw_p_cs2(ph, rho, T, P, cs2);
        const C theta = P * inv_rho;
        for (int d = 0; d < 2; d++) Lam[d] = rho * u[d] * (u[d] * u[d] + C(3) * (theta - C(1.0 / 3.0)));
        const C hh = e + theta;
        if (live) {
            sU[0][t] = u[0];
            sU[1][t] = u[1];
            sT[t] = T;
            sH[t] = hh;
            sL[0][t] = Lam[0];
            sL[1][t] = Lam[1];
        }
        __syncthreads();
        // -- collision ----------------------------------------------------------
        {
            CollideIn<C> in;
            in.rho = rho;
            in.P = P;
            in.e = e;
            in.cs2 = cs2;
            in.u[0] = u[0];
            in.u[1] = u[1];
            in.u[2] = C(0);
            in.F[0] = F[0];
            in.F[1] = F[1];
            in.F[2] = C(0);
            // u_x, h, T, Lambda_x beside the cell along x: a wall's ghost has its own
            C nu[2] = {sU[0][cW], sU[0][cE]}, nh[2] = {sH[cW], sH[cE]};
            C nT[2] = {sT[cW], sT[cE]}, nL[2] = {sL[0][cW], sL[0][cE]};
            if constexpr (WALL) {
                if (wall_lo || wall_hi) {
                    for (int q = 0; q < nwall; q++) {
                        const int k = wall_of(q);
                        const WallGhost<C> gs = wall_ghost(ph, a.w, k, rho);
#pragma unroll
                        for (int j = 0; j < 2; j++) {
                            nu[j] = j == k ? gs.u[0] : nu[j];
                            nh[j] = j == k ? gs.h : nh[j];
                            nT[j] = j == k ? gs.T : nT[j];
                            nL[j] = j == k ? gs.Lx : nL[j];
                        }
                    }
                }
            }
            in.du = C(0.5) * (nu[1] - nu[0]) + C(0.5) * (sU[1][cN] - sU[1][cS]);
            in.dh[0] = C(0.5) * (nh[1] - nh[0]);
            in.dh[1] = C(0.5) * (sH[cN] - sH[cS]);
            in.dT[0] = C(0.5) * (nT[1] - nT[0]);
            in.dT[1] = C(0.5) * (sT[cN] - sT[cS]);
            in.L0[0] = Lam[0];
            in.Lm[0] = nL[0];
            in.Lp[0] = nL[1];
            in.L0[1] = Lam[1];
            in.Lm[1] = sL[1][cS];
            in.Lp[1] = sL[1][cN];
            in.dT[2] = in.dh[2] = in.L0[2] = in.Lm[2] = in.Lp[2] = C(0);
            collide_cell<2, WALL>(ph, in, f, gq);
        }
        // the last step of the post-collision form ends here
        if (!WALL && s == a.steps - 1) break;
        // -- streaming ------------------------------------------------------------
        if (live) {
#pragma unroll
            for (int i = 0; i < Q; i++) {
                sF[i][t] = f[i];
                sG[i][t] = gq[i];
            }
        }
        __syncthreads();
        if constexpr (WALL) {
            // the ghost beside a boundary cell of row y takes in what left
            // towards it and emits; its emission along c arrives in row y + c_y
            if (live && (wall_lo || wall_hi)) {
                for (int q = 0; q < nwall; q++) {
                    // as k_wall_emit, along c_x = cin
                    const int k = wall_of(q), cin = k ? -1 : 1;
                    const WallGhost<C> gs = wall_ghost(ph, a.w, k, rho);
                    const AxisEq<C> ex = axis_eq(gs.u[0], gs.theta), ey = axis_eq(gs.u[1], gs.theta);
                    const C pxc = k ? ex.p.m : ex.p.p, qxc = k ? ex.q.m : ex.q.p;
                    C m = 0, sm = 0;
#pragma unroll
                    for (int cy = -1; cy <= 1; cy++) {
                        m += sF[1 - cin + 3 * (cy + 1)][py[cy + 1] + rx];
                        sm += pxc * pick(ey.p, cy);
                    }
                    const C rg = m / sm, eps = gs.e - gs.theta;
#pragma unroll
                    for (int cy = -1; cy <= 1; cy++) {
                        const C fe = rg * pxc * pick(ey.p, cy);
                        sE[k][cy + 1][0][y] = fe;
                        sE[k][cy + 1][1][y] = fe * eps + C(0.5) * rg * (qxc * pick(ey.p, cy) + pxc * pick(ey.q, cy));
                    }
                }
            }
            __syncthreads();
        }
#pragma unroll
        for (int i = 0; i < Q; i++) {
            const int src = py[cy_of(i) + 1] + px[cx_of(i) + 1];
            f[i] = sF[i][src];
            gq[i] = sG[i][src];
            if constexpr (WALL) {
                const bool ghost = cx_of(i) == 1 ? wall_lo : (cx_of(i) == -1 && wall_hi);
                if (ghost) {
                    const int from = cy_of(i) == 1 ? ym : (cy_of(i) == -1 ? yp : y);
                    f[i] = sE[cx_of(i) == 1 ? 0 : 1][cy_of(i) + 1][0][from];
                    gq[i] = sE[cx_of(i) == 1 ? 0 : 1][cy_of(i) + 1][1][from];
                }
            }
        }
    }
    if (own) {
#pragma unroll
        for (int i = 0; i < Q; i++)
            store_pair(a.fo, pop_index<Q>(g, i, 0, x + (long long)g.nx * y), S::enc(f[i], (C)a.ref.f[i]),
                       S::enc(gq[i], (C)a.ref.g[i]));
    }
}

}  // namespace lbm

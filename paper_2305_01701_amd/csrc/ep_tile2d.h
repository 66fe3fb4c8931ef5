// Fused 2D PT sweeps over a TX x TY tile of cells, up to K of them in a row
// (shared by the single-model launches and the batched persistent kernel).
//
// The workgroup holds the tile with a halo of 2 K points in registers, every
// thread NQ points of one column: iterates, increment-start stresses and
// cohesion (or the held Lambda) are loaded once, ns <= K sweeps are done and
// the tile's own points are stored.  A sweep moves information two points,
// so after s sweeps the outer 2 s points of the halo are stale and the tile
// itself is exact.  What neighbours exchange goes through LDS, four barriers
// a sweep: physical trials S at the vertices; centre update (pressure,
// deviatoric trial, return mapping of centre_return); vertex stresses from
// the averaged centre Lambda, T = tau_k/(G~ dtau) + S; velocities.  A caller
// that runs several tiles in one workgroup must put a barrier between them.
//
// What bounds it: small grids the launch (2 to 3 us) and the latency of the
// stages, large ones the traffic to the last-level cache; both are paid once
// per launch, and the redundant halo buys that.  Per sweep, one sweep per
// launch and now, in us: 63^2 FP64 7.5 and 3.1; 511^2 FP32 8.3 and 4.5, FP64
// 11.3 and 8.6; 1023^2 FP32 19.4 and 11.1; 777 x 1010 FP64 with a per-cell G
// 39.8 and 23.  Skipping the waves whose rows are stale by a later sweep of
// the launch gained nothing (1023^2 FP32 11.3 against 11.1 us).
#pragma once
#include "ep_device.h"

namespace ep {

template <typename R, int TX, int TY, int K, int MODE, int NT, bool HG>
__device__ __forceinline__ void sweep_tile_2d(const SweepArgs<R>& a, int bx, int by, int ns)
{
    // multiply-adds are fused only within one expression, so that every
    // caller (single-model or batched kernel) rounds each point identically
#pragma clang fp contract(on)
    constexpr int HL = 2 * K, W = TX + 4 * K, H = TY + 4 * K;
    static_assert(NT % W == 0, "a thread's points lie in one column");
    constexpr int NR = NT / W, NQ = (H + NR - 1) / NR;   // rows per pass, points per thread
    constexpr int NP = NQ * NT, PAD = W + 1;
    __shared__ R sm[PAD + 6 * NP + PAD];
    __shared__ double s_red[NT / 64];
    R* const s_vx = sm + PAD;
    R* const s_vy = s_vx + NP;
    R* const s_e = s_vy + NP;            // trials, then new stresses of the vertices
    R* const s_lam = s_e + NP;
    R* const s_xx = s_lam + NP;          // txx - p, tyy - p
    R* const s_yy = s_xx + NP;

    const int nx = a.nx, ny = a.ny, tid = threadIdx.x;
    const int la = tid % W, lb = tid / W;
    const int i = bx * TX - HL + la, j0 = by * TY - HL + lb;
    const R idx = a.idx, idy = a.idy, igt = a.igt, igd = a.igd, ikt = a.ikt, ikd = a.ikd, D = a.D;
    const int lam_mode = a.lam_mode;

    // points outside the domain read its nearest point (and are not used)
    R vx[NQ], vy[NQ], p[NQ], sx[NQ], sy[NQ], xy[NQ], po[NQ], sxo[NQ], syo[NQ], xyo[NQ], c[NQ], igc[HG ? NQ : 1], igv[HG ? NQ : 1];
    const int ci = min(max(i, 0), nx);
    const R* const cb = lam_mode == LAM_FROZEN ? a.lam : a.coh;
#pragma unroll
    for (int u = 0; u < NQ; ++u) {
        const long e = ci + (long)a.sy * min(max(j0 + u * NR, 0), ny);
        vx[u] = a.it[F_VX][e];
        vy[u] = a.it[F_VY][e];
        p[u] = a.it[F_P][e];
        sx[u] = a.it[F_TXX][e];
        sy[u] = a.it[F_TYY][e];
        xy[u] = a.it[F_TXY][e];
        po[u] = a.old[O_P][e];
        sxo[u] = a.old[O_TXX][e];
        syo[u] = a.old[O_TYY][e];
        xyo[u] = a.old[O_TXY][e];
        c[u] = cb[e];
        if (HG) {
            const int j = j0 + u * NR;
            igc[u] = a.igdc[e];
            igv[u] = i >= 1 && i <= nx - 1 && j >= 1 && j <= ny - 1 ? vertex_compliance(a.igdc, e, (long)a.sy) : igd;
        }
    }
    // rows of this thread's column: inside for x-faces / centres and for
    // vertices / y-faces
    const bool xc = i >= 0 && i < nx, xv = i >= 1 && i <= nx - 1;
    auto yc = [&](int u) { const int j = j0 + u * NR; return j >= 0 && j < ny; };
    auto yv = [&](int u) { const int j = j0 + u * NR; return j >= 1 && j <= ny - 1; };
    // owned points: the tile's cells; faces and vertices also on the far wall
    // when the tile ends there
    const bool ox = la >= HL && la < HL + TX && i < nx, oxw = ox || (la >= HL && la <= HL + TX && i == nx);
    auto oy = [&](int u) { const int l = lb + u * NR; return l >= HL && l < HL + TY && j0 + u * NR < ny; };
    auto oyw = [&](int u) { const int l = lb + u * NR; return oy(u) || (l >= HL && l <= HL + TY && j0 + u * NR == ny); };

    R rmax = R(0), mmax = R(0), vmax = R(0), smax = R(0);   // combined, momentum-only, |v|, |stress|
    bool held = lam_mode == LAM_FROZEN;                      // c holds Lambda
#pragma unroll
    for (int u = 0; u < NQ; ++u) {
        s_vx[tid + u * NT] = vx[u];
        s_vy[tid + u * NT] = vy[u];
    }
    __syncthreads();
    for (int s = 0; s < ns; ++s) {
        const bool last = MODE == MODE_CHECK && s == ns - 1;
        R T[NQ];
#pragma unroll
        for (int u = 0; u < NQ; ++u) {
            const int q = tid + u * NT;
            const R e2 = (vx[u] - s_vx[q - W]) * idy + (vy[u] - s_vy[q - 1]) * idx;
            R sv = xyo[u] * (HG ? igv[u] : igd) + e2;
            if (!(xv && yv(u))) sv = R(0);
            T[u] = xy[u] * igt + sv;
            s_e[q] = sv;
        }
        __syncthreads();
#pragma unroll
        for (int u = 0; u < NQ; ++u) {
            const int q = tid + u * NT;
            R dvx = (s_vx[q + 1] - vx[u]) * idx + a.ebx;
            R dvy = (s_vy[q + W] - vy[u]) * idy + a.eby;
            R div = dvx + dvy;
            const R pk = p[u], txk = sx[u], tyk = sy[u];
            R pn = (pk * ikt + po[u] * ikd - div) * a.ikk;
            // per-cell G: the cell's compliance, its physical Dp and its D
            const R ig = HG ? igc[u] : igd;
            const R Dp = HG ? ig + a.imus : a.Dp;
            const R invDp = HG ? R(1) / Dp : a.invDp;
            const R Dc = HG ? igt + Dp : D;
            const R invDc = HG ? R(1) / Dc : a.invD;
            const R div3 = third(div);
            const R Sxx = sxo[u] * ig + R(2) * (dvx - div3);
            const R Syy = syo[u] * ig + R(2) * (dvy - div3);
            const R Txx = txk * igt + Sxx, Tyy = tyk * igt + Syy;
            const R Sb = R(0.25) * (s_e[q] + s_e[q + 1] + s_e[q + W] + s_e[q + W + 1]);
            const R nS2 = R(0.5) * (Sxx * Sxx + Syy * Syy), sh2 = Sb * Sb;
            const R ptr = pn;
            R lam;
            if (held) {                                   // frozen plasticity: the held Lambda
                lam = c[u];
                // dilatancy of the held Lambda: lamdot = Lambda sqrt(J2(S)) / (Dp + Lambda)
                if (a.Cik != R(0)) pn = ptr + lam * fast_sqrt(nS2 + sh2) * fast_rcp(Dp + lam) * a.Cik;
            } else {
                lam = centre_return(R(0.5) * (Txx * Txx + Tyy * Tyy), nS2, sh2, Dp, invDp, Dc, invDc, pn, c[u], a.A,
                                    a.B, a.Cik, a.vp, a.blend);
                if (lam_mode == LAM_STORE) {              // stored for freezing, held from the next sweep on
                    c[u] = lam;
                    if (ox && oy(u)) a.lam[i + (long)a.sy * (j0 + u * NR)] = lam;
                }
            }
            const R sc_ = HG ? fast_rcp(Dc + lam) : rcp_sum(D, lam, a.invD);
            R txx = Txx * sc_, tyy = Tyy * sc_;
            if (!(xc && yc(u))) lam = pn = txx = tyy = R(0);
            p[u] = pn;
            sx[u] = txx;
            sy[u] = tyy;
            s_lam[q] = lam;
            s_xx[q] = txx - pn;
            s_yy[q] = tyy - pn;
            if (last && ox && oy(u)) {
                R dp = fabs(pn - pk) * a.rK;
                R dt = nmax(fabs(txx - txk), fabs(tyy - tyk)) * a.rG;
                rmax = nmax(rmax, nmax(dp, dt));
                smax = nmax(smax, nmax(nmax(fabs(pn), fabs(txx)), fabs(tyy)));
            }
        }
        held = held || lam_mode == LAM_STORE;
        __syncthreads();
#pragma unroll
        for (int u = 0; u < NQ; ++u) {
            const int q = tid + u * NT;
            const R lv = R(0.25) * (s_lam[q - W - 1] + s_lam[q - W] + s_lam[q - 1] + s_lam[q]);
            R t = T[u] * (HG ? fast_rcp(igt + igv[u] + a.imus + lv) : rcp_sum(D, lv, a.invD));
            if (!(xv && yv(u))) t = R(0);
            if (last && oxw && oyw(u)) rmax = nmax(rmax, fabs(t - xy[u]) * a.rG);
            xy[u] = t;
            s_e[q] = t;
        }
        __syncthreads();
#pragma unroll
        for (int u = 0; u < NQ; ++u) {
            const int q = tid + u * NT;
            R Rx = (s_xx[q] - s_xx[q - 1]) * idx + (s_e[q + W] - xy[u]) * idy;
            R Ry = (s_yy[q] - s_yy[q - W]) * idy + (s_e[q + 1] - xy[u]) * idx;
            if (xv && yc(u)) vx[u] = vx[u] + a.dtrho * Rx;
            else Rx = R(0);
            if (xc && yv(u)) vy[u] = vy[u] + a.dtrho * Ry;
            else Ry = R(0);
            s_vx[q] = vx[u];
            s_vy[q] = vy[u];
            if (MODE == MODE_PHYS || last) {
                if (oxw && oy(u)) {
                    mmax = nmax(mmax, fabs(Rx));
                    vmax = nmax(vmax, fabs(vx[u]));
                }
                if (ox && oyw(u)) {
                    mmax = nmax(mmax, fabs(Ry));
                    vmax = nmax(vmax, fabs(vy[u]));
                }
            }
        }
        if (s + 1 < ns) __syncthreads();
    }
#pragma unroll
    for (int u = 0; u < NQ; ++u) {
        const long e = i + (long)a.sy * (j0 + u * NR);
        if (ox && oy(u)) {
            a.nx_[F_P][e] = p[u];
            a.nx_[F_TXX][e] = sx[u];
            a.nx_[F_TYY][e] = sy[u];
        }
        if (oxw && oyw(u)) a.nx_[F_TXY][e] = xy[u];
        if (MODE != MODE_PHYS) {
            if (oxw && oy(u)) a.nx_[F_VX][e] = vx[u];
            if (ox && oyw(u)) a.nx_[F_VY][e] = vy[u];
        }
    }
    if (MODE != MODE_UPDATE) {
        block_max_to<NT>((double)mmax, a.red + RED_MOM, s_red);
        if (MODE == MODE_CHECK) {
            block_max_to<NT>((double)fmax(rmax, mmax), a.red + RED_RESID, s_red);
            block_max_to<NT>((double)vmax, a.red + RED_VMAX, s_red);
            block_max_to<NT>((double)smax, a.red + RED_SMAX, s_red);
        }
    }
}

}  // namespace ep

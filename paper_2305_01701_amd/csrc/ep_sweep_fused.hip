// Fused PT sweep: one kernel per pseudo-transient iteration.
//
// One iteration couples points up to two cells apart (v -> shear trial at
// edges -> 4-point mean at centres -> Lambda at centres -> mean back to
// edges -> velocity), so a workgroup that owns a tile recomputes a halo:
//
//   3D: a workgroup owns a TX x TY column of cells over a chunk of z-planes
//   and marches up the chunk.  What neighbours exchange lives in LDS as 2D
//   planes of (TX+4) x (TY+4) points (a 2-point x-y halo).  Step f of the
//   march forms the shear trials on the z-level f (xz, yz edges) and the
//   plane f-1 (xy edges), the centre update of plane f-1 (pressure, deviator,
//   return mapping), the new edge stresses of plane/level f-1, and the new
//   velocities of plane f-2 (vx, vy) and level f-1 (vz), then stores the
//   velocity planes of step f+1 to LDS: four workgroup barriers per step.
//   Each field is read from and written to HBM once per sweep (iteration-k
//   velocities twice, from L2); the halo reads of neighbouring tiles are
//   served by L2 (blocks are remapped so that spatial neighbours run on the
//   same XCD).
//   What bounds it: large grids the memory traffic (beyond the L2, 255^3 FP32:
//   2.45 GB per sweep, 1.48 times the algorithmic bytes, at 5.4 TB/s; 511^3
//   22.7 GB at 6.0), small ones the latency of a march step.  An earlier form
//   kept every plane twice in LDS, split the points over the threads once for
//   all stages and loaded behind branches: 80 vector registers with spills,
//   whose reloads waited for the loads of the next step.  Per sweep, then and
//   now, in us: 255^3 FP32 541 and 452, FP64 989 and 803; 190 x 127 x 101 FP64
//   247 and 159; 63^3 FP32 142 and 18.2, FP64 194 and 25.5 (short chunks
//   included).
//   2D: the same stages on a single TX x TY tile (ep_tile2d.h, run by the
//   tile-list kernel of ep_sweep_batch.hip for single models and batches).
//
// The arithmetic of every point is that of the unfused sweep (same formulas,
// same Jacobi order: all reads are of iteration k, all writes iteration k+1).
#include <cmath>
#include <type_traits>

#include "ep_device.h"

namespace ep {

namespace {

// Tile grid of a 3D sweep and its interior rectangle [bx0, bx1) x [by0,
// by1): tiles whose points, 2-point halo included, lie strictly inside the
// domain in x and y.
struct TileSet {
    int nbx, nby, nbz, zc;      // tiles per direction, planes per z chunk
    int bx0, bx1, by0, by1;
};

// Global memory is reached through buffer instructions: a field of the
// chunk is a resource (base of its first plane, 2 GiB range), a point a
// 32-bit in-plane offset per lane plus a uniform plane offset.  A lane that
// must not access memory carries the offset NOWHERE, which the range check
// turns into a load of 0 or a dropped store, and a store that a whole step
// must not do gets an empty range.  So every load and store is issued
// unconditionally, and the compiler knows how many memory operations are in
// flight when it waits for one (behind a branch it would have to assume the
// fewest, and wait for younger ones too).
constexpr unsigned NOWHERE = 0xffffffffu;
constexpr int RANGE = 0x7fffffff;

//
// Where the planes of a chunk reach beyond 2 GiB (long planes) the plane's
// offset is added to the base in 64 bits instead.
template <typename R, typename P>
__device__ __forceinline__ R buf_load(const char* base, bool go, unsigned off, P plane)
{
    if constexpr (sizeof(P) == 8) return buf_load<R>(base + plane, go, off, 0);
    const auto rs = __builtin_amdgcn_make_buffer_rsrc((void*)base, (short)0, go ? RANGE : 0, 0x00020000);
    if constexpr (sizeof(R) == 4) return __builtin_bit_cast(R, __builtin_amdgcn_raw_buffer_load_b32(rs, off, (int)plane, 0));
    else return __builtin_bit_cast(R, __builtin_amdgcn_raw_buffer_load_b64(rs, off, (int)plane, 0));
}

template <typename R, typename P>
__device__ __forceinline__ void buf_store(char* base, bool go, unsigned off, P plane, R v)
{
    if constexpr (sizeof(P) == 8) return buf_store<R>(base + plane, go, off, 0, v);
    typedef unsigned u2 __attribute__((ext_vector_type(2)));
    const auto rs = __builtin_amdgcn_make_buffer_rsrc((void*)base, (short)0, go ? RANGE : 0, 0x00020000);
    if constexpr (sizeof(R) == 4) __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(unsigned, v), rs, off, (int)plane, 0);
    else __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(u2, v), rs, off, (int)plane, 0);
}

// The value as it is, hidden from the compiler: an expression of it is not
// fused with the one that formed it.
template <typename R>
__device__ __forceinline__ R opaque(R v) { asm volatile("" : "+v"(v)); return v; }

// LDS planes.  Velocities, xz / yz trials and compliances come in pairs
// (planes of even and of odd z): slot 0 of all of them, then slot 1, so that
// one address per slot and an immediate offset reach every plane of a point.
// Of the rest one plane is kept: what a thread needs of the plane below it
// carries over in registers (sums and differences are formed in the order in
// which the two planes come by).
enum { L_VX = 0, L_VY, L_VZ, L_SXZ, L_SYZ, L_PAIRS, L_IG = L_PAIRS };
enum { L_SXY = 0, L_LAM, L_XX, L_YY, L_ZZ, L_NXY, L_NXZ, L_NYZ, L_SINGLE };

// ----------------------------------------------------------------------- 3D
// The workgroup's points are split over its threads anew for each stage, row
// by row of the stage's own region, so that no wave works for the halo of
// another stage: q over the plane with its 2-point halo (velocities,
// physical trials), r over the centres with a 1-point halo, e over the edges
// and faces.  What a stage takes from memory is loaded under the stage's own
// split one step ahead, right after the previous step's values have been
// used, into the same registers.
template <typename R, int TX, int TY, int MODE, int NT, int WPE, bool HG, bool FRZ, bool FAR>
__global__ __attribute__((amdgpu_flat_work_group_size(NT, NT), amdgpu_waves_per_eu(WPE)))
void k_fused_3d(SweepArgs<R> a, TileSet ts)
{
    constexpr int W = TX + 4, H = TY + 4, N = W * H;       // plane with its halo
    constexpr int CW = TX + 2, CN = CW * (TY + 2);         // centres
    constexpr int EW = TX + 1, EN = EW * (TY + 1);         // edges, faces
    constexpr int NP = N + 2;                              // + a place for the threads beyond the plane
    constexpr int PAD = W + 2;                             // the halo's outermost points read neighbours before it
    constexpr int NPAIR = L_PAIRS + (HG ? 1 : 0), SL = NPAIR * NP;
    constexpr int RW = (CN + 63) / 64, QW = (EN + 63) / 64;   // waves with centres, with edges
    static_assert(N <= NT, "one point per thread");
    __shared__ R sm[PAD + 2 * SL + L_SINGLE * NP + PAD];
    __shared__ double s_red[NT / 64];

    const int lb = xcd_remap(blockIdx.x, ts.nbx * ts.nby * ts.nbz);
    const int bx = lb % ts.nbx, by = (lb / ts.nbx) % ts.nby, bz = lb / (ts.nbx * ts.nby);
    // the same sweep, compiled twice: for tiles strictly inside the domain in
    // x and y no point needs a boundary test
    auto body = [&](auto interior) {
    constexpr bool INT = decltype(interior)::value;
    const int i0 = bx * TX, j0 = by * TY;
    const int nx = a.nx, ny = a.ny, nz = a.nz;
    const int k0 = bz * ts.zc, k1 = min(k0 + ts.zc, nz);
    const int tid = threadIdx.x;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int hx = (!INT && i0 + TX == nx) ? 1 : 0;     // owns the x = nx row when nx % TX == 0
    const int hy = (!INT && j0 + TY == ny) ? 1 : 0;
    const bool last_z = (k1 == nz);

    // fields: first plane of the chunk of the first field of a group, and the
    // uniform field stride in bytes
    using Plane = std::conditional_t<FAR, long, int>;
    const int kb = max(k0 - 2, 0);
    const Plane plane_bytes = (Plane)(a.sz * (long)sizeof(R));
    const long first = (long)kb * a.sz;
    const char* const itb = (const char*)(a.it[0] + first);
    char* const nxb = (char*)(a.nx_[0] + first);
    const char* const olb = (const char*)(a.old[0] + first);
    const char* const cob = (const char*)((FRZ ? a.lam : a.coh) + first);
    const char* const igb = HG ? (const char*)(a.igdc + first) : nullptr;
    char* const lmb = (char*)(a.lam + first);
    const bool keep_lam = !FRZ && a.lam_mode == LAM_STORE;
    long fs = a.fs * (long)sizeof(R);
    // byte offset of plane g in the chunk (planes outside the domain: the
    // nearest; what is read there is not used)
    auto plane = [&](int g) -> Plane { return (min(max(g, kb), nz) - kb) * plane_bytes; };
    auto off = [&](bool ok, int i, int j) -> unsigned {
        return ok && i >= 0 && i <= nx && j >= 0 && j <= ny ? (unsigned)(i + a.sy * j) * (unsigned)sizeof(R) : NOWHERE;
    };
    const R idx = a.idx, idy = a.idy, idz = a.idz, igt = a.igt, igd = a.igd, ikt = a.ikt, ikd = a.ikd;
    const R D = a.D;

    // q: this thread's plane point
    const int q = min(tid, N), qi = i0 - 2 + q % W, qj = j0 - 2 + q / W;
    const unsigned qo = off(tid < N, qi, qj);
    const bool q_xz = INT || (qi >= 1 && qi <= nx - 1 && qj >= 0 && qj < ny);
    const bool q_yz = INT || (qj >= 1 && qj <= ny - 1 && qi >= 0 && qi < nx);
    const bool q_xy = INT || (qi >= 1 && qi <= nx - 1 && qj >= 1 && qj <= ny - 1);
    // r: this thread's centre
    const int rr = min(tid, CN - 1), rla = 1 + rr % CW, rlb = 1 + rr / CW, rq = tid < CN ? rla + W * rlb : N;
    const int ri = i0 - 2 + rla, rj = j0 - 2 + rlb;
    const unsigned ro = off(tid < CN, ri, rj);
    const bool r_in = INT || (ri >= 0 && ri < nx && rj >= 0 && rj < ny);
    const bool r_own = tid < CN && r_in && rla >= 2 && rla < TX + 2 && rlb >= 2 && rlb < TY + 2;
    const unsigned ros = r_own ? ro : NOWHERE;
    // e: this thread's edge and face point
    const int ee = min(tid, EN - 1), ela = 2 + ee % EW, elb = 2 + ee / EW, eq = tid < EN ? ela + W * elb : N;
    const int ei = i0 - 2 + ela, ej = j0 - 2 + elb;
    const unsigned eo = off(tid < EN, ei, ej);
    const bool e_x = tid < EN && ela < TX + 2 + hx && (INT || ei <= nx), e_y = tid < EN && elb < TY + 2 + hy && (INT || ej <= ny);
    const bool e_xc = tid < EN && ela < TX + 2 && (INT || ei < nx), e_yc = tid < EN && elb < TY + 2 && (INT || ej < ny);
    const bool own_xy = e_x && e_y, own_xz = e_x && e_yc, own_yz = e_xc && e_y, own_c = e_xc && e_yc;
    const bool in_x = INT || (ei >= 1 && ei <= nx - 1), in_y = INT || (ej >= 1 && ej <= ny - 1);

    R* const s0 = sm + PAD;
    R* const s1 = s0 + 2 * SL;

    // velocities of plane (vx, vy) and level (vz) g, and the compliances
    R fvx, fvy, fvz, fig = R(0);
    auto load_v = [&](int g) {
        const Plane p = plane(g);
        const bool go = g <= k1 + 1;
        fvx = buf_load<R>(itb, go, qo, p);
        fvy = buf_load<R>(itb + fs, go, qo, p);
        fvz = buf_load<R>(itb + fs + fs, go, qo, p);
        if (HG) fig = buf_load<R>(igb, go, qo, p);
    };
    auto stage_v = [&](int slot) {
        R* const s = s0 + slot * SL + q;
        s[L_VX * NP] = fvx;
        s[L_VY * NP] = fvy;
        s[L_VZ * NP] = fvz;
        if (HG) s[L_IG * NP] = fig;
    };
    // increment-start edge stresses: xz, yz at level f, xy at plane f - 1
    R oxz, oyz, oxy;
    auto load_old = [&](int f) {
        const char* b = olb + 3 * fs;
        const bool go = f <= k1 + 1;
        oxy = buf_load<R>(b, go, qo, plane(f - 1));
        b += fs;
        oxz = buf_load<R>(b, go, qo, plane(f));
        b += fs;
        oyz = buf_load<R>(b, go, qo, plane(f));
    };
    // centre data of plane c
    R cp, cpo, csx, csxo, csy, csyo, cc;
    auto load_c = [&](int c) {
        const Plane p = plane(c);
        const bool go = c >= k0 - 1 && c <= k1;
        const char *b = itb + 3 * fs, *o = olb;
        cp = buf_load<R>(b, go, ro, p);
        cpo = buf_load<R>(o, go, ro, p);
        b += fs;
        o += fs;
        csx = buf_load<R>(b, go, ro, p);
        csxo = buf_load<R>(o, go, ro, p);
        b += fs;
        o += fs;
        csy = buf_load<R>(b, go, ro, p);
        csyo = buf_load<R>(o, go, ro, p);
        cc = buf_load<R>(cob, go, ro, p);
    };
    // edge stresses of iteration k of plane and level l
    R kxy, kxz, kyz;
    auto load_k = [&](int l) {
        const Plane p = plane(l);
        const bool go = l >= k0 && l <= k1;
        const char* b = itb + 6 * fs;
        kxy = buf_load<R>(b, go, eo, p);
        b += fs;
        kxz = buf_load<R>(b, go, eo, p);
        b += fs;
        kyz = buf_load<R>(b, go, eo, p);
    };
    // velocities of iteration k at the faces: vx, vy of plane p, vz of level p + 1
    R wvx, wvy, wvz;
    auto load_w = [&](int p) {
        const bool go = p >= k0 - 1 && p <= k1;
        wvx = buf_load<R>(itb, go, eo, plane(p));
        wvy = buf_load<R>(itb + fs, go, eo, plane(p));
        wvz = buf_load<R>(itb + fs + fs, go, eo, plane(p + 1));
    };

    // combined, momentum-only, |v|, |stress| maxima, kept in the field type
    // (maxima are exact) and widened for the block reduction
    R rmax = R(0), mmax = R(0), vmax = R(0), smax = R(0);
    // compliances of the xz, yz edges of the level of the next step
    R pgxz = igd, pgyz = igd;
    // of the previous step: sums of the Lambda of the plane's two centres at
    // the xz and yz edges, new xz and yz stresses, -sigma_zz, and the parts of
    // the x and y momentum residuals within the plane
    R mxz = R(0), myz = R(0), uxz = R(0), uyz = R(0), uzz = R(0), ux = R(0), uy = R(0);
    R txy = R(0), txz = R(0), tyz = R(0);      // new edge stresses of this step

    // nothing below plane 0 is used, so its chunk starts a step later (slabs of
    // 3 planes: 5 steps instead of 6)
    const int f0 = max(k0 - 1, 0);
    load_v(f0 - 1);
    stage_v((f0 & 1) ^ 1);
    load_v(f0);
    stage_v(f0 & 1);
    load_old(f0);
    load_c(f0 - 1);
    load_k(f0 - 1);
    load_w(f0 - 2);
    load_v(f0 + 1);
    __syncthreads();
    // f - 1 is the plane of the centres, f - 2 that of the vx and vy updates
    for (int f = f0; f <= k1 + 1; ++f) {
        asm volatile("" : "+s"(fs));
        const int sc = f & 1;                 // slot of plane f; plane f - 1 has the other one
        R* const sf = s0 + sc * SL;
        R* const sg = s0 + (sc ^ 1) * SL;

        // ---- S2: physical shear trials: xz, yz at level f; xy at plane f-1 --
        {
            R* const cu = sf + q;             // plane / level f
            R* const pr = sg + q;             // plane f - 1
            const bool inner = f >= 1 && f <= nz - 1;
            R gxy = igd, gxz = igd, gyz = igd;
            if (HG) {                         // compliance of an edge: mean of its four cells
                const R *c0 = cu + L_IG * NP, *c1 = pr + L_IG * NP;
                gxz = R(0.25) * (c1[-1] + c1[0] + c0[-1] + c0[0]);
                gyz = R(0.25) * (c1[-W] + c1[0] + c0[-W] + c0[0]);
                gxy = R(0.25) * (c1[-W - 1] + c1[-W] + c1[-1] + c1[0]);
            }
            const R vz0 = cu[L_VZ * NP], vx0 = cu[L_VX * NP], vy0 = cu[L_VY * NP];
            const R vx1 = pr[L_VX * NP], vy1 = pr[L_VY * NP];
            const R exz = (vx0 - vx1) * idz + (vz0 - cu[L_VZ * NP - 1]) * idx;
            const R eyz = (vy0 - vy1) * idz + (vz0 - cu[L_VZ * NP - W]) * idy;
            const R exy = (vx1 - pr[L_VX * NP - W]) * idy + (vy1 - pr[L_VY * NP - 1]) * idx;
            const R sxz = oxz * gxz + exz, syz = oyz * gyz + eyz, sxy = oxy * gxy + exy;
            cu[L_SXZ * NP] = inner && q_xz ? sxz : R(0);
            cu[L_SYZ * NP] = inner && q_yz ? syz : R(0);
            s1[L_SXY * NP + q] = q_xy ? sxy : R(0);
        }
        load_old(f + 1);
        __syncthreads();
        // ---- S3: centres of plane c = f-1 -----------------------------------
        {
            const int c = f - 1;
            R pn = R(0), txx = R(0), tyy = R(0), lam = R(0);
            if (wave < RW) {
                const R* const up = sf + rq;  // level c + 1
                const R* const at = sg + rq;  // plane, level c
                const R vz0 = at[L_VZ * NP];
                R dvx = (at[L_VX * NP + 1] - at[L_VX * NP]) * idx + a.ebx;
                R dvy = (at[L_VY * NP + W] - at[L_VY * NP]) * idy + a.eby;
                R dvz = (up[L_VZ * NP] - vz0) * idz + a.ebz;
                R div = dvx + dvy + dvz;
                const R pk = cp, txk = csx, tyk = csy;
                pn = (pk * ikt + cpo * ikd - div) * a.ikk;
                // per-cell G: the cell's compliance, its physical Dp and its D
                const R igc = HG ? at[L_IG * NP] : igd;
                const R Dp = HG ? igc + a.imus : a.Dp;
                const R invDp = HG ? fast_rcp(Dp) : a.invDp;
                const R Dc = HG ? igt + Dp : D;
                const R invDc = HG ? fast_rcp(Dc) : a.invD;
                const R Sxx = csxo * igc + R(2) * (dvx - div * R(1.0 / 3.0));
                const R Syy = csyo * igc + R(2) * (dvy - div * R(1.0 / 3.0));
                const R Szz = -(Sxx + Syy);
                const R Txx = txk * igt + Sxx, Tyy = tyk * igt + Syy, Tzz = -(Txx + Tyy);
                R* const one = s1 + rq;
                const R* const xy = one + L_SXY * NP;
                const R Sxyb = R(0.25) * (xy[0] + xy[1] + xy[W] + xy[W + 1]);
                const R Sxzb = R(0.25) * (at[L_SXZ * NP] + at[L_SXZ * NP + 1] + up[L_SXZ * NP] + up[L_SXZ * NP + 1]);
                const R Syzb = R(0.25) * (at[L_SYZ * NP] + at[L_SYZ * NP + W] + up[L_SYZ * NP] + up[L_SYZ * NP + W]);
                const R nS2 = R(0.5) * (Sxx * Sxx + Syy * Syy + Szz * Szz);
                const R sh2 = Sxyb * Sxyb + Sxzb * Sxzb + Syzb * Syzb;
                const R ptr = pn;
                if (FRZ) {                                       // frozen plasticity: the held Lambda
                    lam = cc;
                    // dilatancy of the held Lambda: lamdot = Lambda sqrt(J2(S)) / (Dp + Lambda)
                    if (a.Cik != R(0)) pn = ptr + lam * fast_sqrt(nS2 + sh2) * fast_rcp(Dp + lam) * a.Cik;
                } else {
                    lam = centre_return(R(0.5) * (Txx * Txx + Tyy * Tyy + Tzz * Tzz), nS2, sh2, Dp, invDp, Dc, invDc,
                                        pn, cc, a.A, a.B, a.Cik, a.vp, a.blend);
                }
                const R sc_ = fast_rcp(Dc + lam);
                txx = opaque(Txx * sc_);
                tyy = opaque(Tyy * sc_);
                pn = opaque(pn);
                if (!INT && !r_in) lam = pn = txx = tyy = R(0);
                one[L_LAM * NP] = lam;
                one[L_XX * NP] = txx - pn;
                one[L_YY * NP] = tyy - pn;
                one[L_ZZ * NP] = -(txx + tyy) - pn;
                if (MODE == MODE_CHECK && r_own && c >= k0 && c < k1) {
                    R dp = fabs(pn - pk) * a.rK;
                    R dtx = fabs(txx - txk), dty = fabs(tyy - tyk), dtz = fabs((txx + tyy) - (txk + tyk));
                    rmax = nmax(rmax, nmax(dp, nmax(nmax(dtx, dty), dtz) * a.rG));
                    smax = nmax(smax, nmax(nmax(fabs(pn), fabs(txx)), nmax(fabs(tyy), fabs(txx + tyy))));
                }
            }
            const bool go = c >= k0 && c < k1;
            const Plane p = plane(c);
            char* b = nxb + 3 * fs;
            buf_store(b, go, ros, p, pn);
            b += fs;
            buf_store(b, go, ros, p, txx);
            b += fs;
            buf_store(b, go, ros, p, tyy);
            if (keep_lam) buf_store(lmb, go, ros, p, lam);       // stored for freezing
        }
        load_c(f);
        __syncthreads();
        // ---- S4: new edge stresses: xy at plane f-1, xz / yz at level f-1:
        //      T = tau_k/(G~ dtau) + S ------------------------------------------
        {
            const int l = f - 1;
            const bool do_p = l >= k0 && l < k1, inner = l >= 1 && l <= nz - 1;
            const bool do_l = do_p || (l == nz && last_z);
            uxz = txz;
            uyz = tyz;
            if (wave < QW) {
                const R* const at = sg + eq;                    // level l
                R* const one = s1 + eq;
                const R* const la = one + L_LAM * NP;
                R gxy = igd, gxz = pgxz, gyz = pgyz;
                if (HG) {
                    const R *c0 = sf + L_IG * NP + eq, *c1 = sg + L_IG * NP + eq;
                    gxy = R(0.25) * (c1[-W - 1] + c1[-W] + c1[-1] + c1[0]);
                    pgxz = R(0.25) * (c1[-1] + c1[0] + c0[-1] + c0[0]);
                    pgyz = R(0.25) * (c1[-W] + c1[0] + c0[-W] + c0[0]);
                }
                const R l00 = la[0], l01 = la[-1], l10 = la[-W];
                const R vxy = R(0.25) * (la[-W - 1] + l10 + l01 + l00);
                const R vxz = R(0.25) * (mxz + l01 + l00);
                const R vyz = R(0.25) * (myz + l10 + l00);
                mxz = l01 + l00;
                myz = l10 + l00;
                txy = (kxy * igt + one[L_SXY * NP]) * fast_rcp((HG ? igt + gxy + a.imus : D) + vxy);
                txz = (kxz * igt + at[L_SXZ * NP]) * fast_rcp((HG ? igt + gxz + a.imus : D) + vxz);
                tyz = (kyz * igt + at[L_SYZ * NP]) * fast_rcp((HG ? igt + gyz + a.imus : D) + vyz);
                if (!INT && !(in_x && in_y)) txy = R(0);
                if (!inner || (!INT && !(in_x && e_yc))) txz = R(0);
                if (!inner || (!INT && !(in_y && e_xc))) tyz = R(0);
                one[L_NXY * NP] = txy;
                one[L_NXZ * NP] = txz;
                one[L_NYZ * NP] = tyz;
                if (MODE == MODE_CHECK) {
                    if (do_p && own_xy) rmax = nmax(rmax, fabs(txy - kxy) * a.rG);
                    if (do_l && own_xz) rmax = nmax(rmax, fabs(txz - kxz) * a.rG);
                    if (do_l && own_yz) rmax = nmax(rmax, fabs(tyz - kyz) * a.rG);
                }
            }
            const Plane p = plane(l);
            char* b = nxb + 6 * fs;
            buf_store(b, do_p, own_xy ? eo : NOWHERE, p, txy);
            b += fs;
            buf_store(b, do_l, own_xz ? eo : NOWHERE, p, txz);
            b += fs;
            buf_store(b, do_l, own_yz ? eo : NOWHERE, p, tyz);
        }
        load_k(f);
        __syncthreads();
        // ---- S5: velocities: vx, vy at plane f-2, vz at level f-1 ------------
        {
            const int p = f - 2, l = f - 1;
            const bool do_xy = p >= k0 && p < k1;
            const bool do_z = (l >= k0 && l < k1) || (l == nz && last_z);
            const bool inner = l >= 1 && l <= nz - 1;
            R vx = wvx, vy = wvy, vz = wvz;
            if (wave < QW) {
                const R* const one = s1 + eq;                   // plane, level l = p + 1
                R Rx = ux + (txz - uxz) * idz;
                R Ry = uy + (tyz - uyz) * idz;
                R Rz = (one[L_NXZ * NP + 1] - txz) * idx + (one[L_NYZ * NP + W] - tyz) * idy + (one[L_ZZ * NP] - uzz) * idz;
                ux = (one[L_XX * NP] - one[L_XX * NP - 1]) * idx + (one[L_NXY * NP + W] - txy) * idy;
                uy = (one[L_NXY * NP + 1] - txy) * idx + (one[L_YY * NP] - one[L_YY * NP - W]) * idy;
                uzz = one[L_ZZ * NP];
                if (!INT && !in_x) Rx = R(0);
                if (!INT && !in_y) Ry = R(0);
                if (!inner) Rz = R(0);
                vx = vx + a.dtrho * Rx;
                vy = vy + a.dtrho * Ry;
                vz = vz + a.dtrho * Rz;
                if (MODE != MODE_UPDATE) {
                    const bool ox = do_xy && own_xz, oy = do_xy && own_yz, oz = do_z && own_c;
                    if (ox) mmax = nmax(mmax, fabs(Rx));
                    if (oy) mmax = nmax(mmax, fabs(Ry));
                    if (oz) mmax = nmax(mmax, fabs(Rz));
                    if (ox) vmax = nmax(vmax, fabs(vx));
                    if (oy) vmax = nmax(vmax, fabs(vy));
                    if (oz) vmax = nmax(vmax, fabs(vz));
                }
            }
            if (MODE != MODE_PHYS) {
                buf_store(nxb, do_xy, own_xz ? eo : NOWHERE, plane(p), vx);
                buf_store(nxb + fs, do_xy, own_yz ? eo : NOWHERE, plane(p), vy);
                buf_store(nxb + fs + fs, do_z, own_c ? eo : NOWHERE, plane(l), vz);
            }
        }
        load_w(f - 1);
        // ---- S1 of step f + 1 -------------------------------------------------
        stage_v(sc ^ 1);
        load_v(f + 2);
        __syncthreads();
    }
    if (MODE != MODE_UPDATE) {
        block_max_to<NT>((double)mmax, a.red + RED_MOM, s_red);
        if (MODE == MODE_CHECK) {
            block_max_to<NT>((double)fmax(rmax, mmax), a.red + RED_RESID, s_red);
            block_max_to<NT>((double)vmax, a.red + RED_VMAX, s_red);
            block_max_to<NT>((double)smax, a.red + RED_SMAX, s_red);
        }
    }
    };
    if (bx >= ts.bx0 && bx < ts.bx1 && by >= ts.by0 && by < ts.by1) body(std::true_type{});
    else body(std::false_type{});
}

// Tiles (X, Y: column; T: threads, at least one per point of the plane with
// its halo, so that no wave does a second round of a stage while the others
// wait at its barrier; E: waves per SIMD to fit in registers).
//  - 64 x 11 (68 x 15 = 1020 points), FP32, 18 LDS planes = 74 KB, two
//    workgroups per CU: a row of 68 values touches 4 lines of 128 bytes for
//    the 2 it owns, one of 36 values 3 for 1, and the neighbours' lines are
//    the traffic that binds large grids.  511^3: 3.72 ms per sweep, 32 x 16
//    3.91, 48 x 10 3.80; 255^3: 0.464, 0.495, 0.521 ms.
//  - 32 x 16 (36 x 20 = 720 points), which fills the last round of
//    workgroups better on middle grids (127^3: 54 us, 64 x 11 65 us); with a
//    per-cell G the FP32 tile for all large grids (64 x 11 would need more
//    than half the LDS then).  FP64: one workgroup of 105 KB and 12 waves per
//    CU; 48 x 15 and 32 x 24 with 1024 threads are no faster (255^3: 0.81 ms
//    against 0.90 and 0.91).
//  - 16 x 8 (20 x 12 = 240 points), for grids that would leave most CUs
//    without work: its march step takes 1.5 us on an otherwise idle CU, that
//    of the larger tiles 2.5 to 3.5 us (63^3 FP32: 18.5 us, 32 x 16 21 us).
template <int X_, int Y_, int T_, int E_> struct Tile {
    static constexpr int X = X_, Y = Y_, T = T_, E = E_;
};
using TileF_wide = Tile<64, 11, 1024, 8>;
using TileF_square = Tile<32, 16, 768, 6>;
using TileF_small = Tile<16, 8, 256, 6>;
using TileD_square = Tile<32, 16, 768, 3>;
using TileD_small = Tile<16, 8, 256, 3>;
enum { TILE_WIDE = 0, TILE_SQUARE, TILE_SMALL };

// first and one-past-last tile index along an axis whose tiles lie strictly
// inside with their 2-point halo: 3 <= i0 and i0 + T + 2 <= n
inline void interior_range(int n, int T, int nb, int& b0, int& b1)
{
    b0 = (3 + T - 1) / T;
    b1 = (n - T - 2) >= 0 ? (n - T - 2) / T + 1 : 0;
    if (b1 > nb) b1 = nb;
    if (b1 < b0) b1 = b0;
}

// Whether a chunk of zc planes of `plane` bytes (with the planes around it)
// reaches beyond the 32-bit offsets of the buffer accesses.
inline bool far_planes(int zc, double plane) { return (zc + 8) * plane > 2147483647.0; }

template <typename S, typename R, int MODE, bool G = true, bool LONG = false>
void run_3d(const SweepArgs<R>& a, hipStream_t s)
{
    constexpr int TX = S::X, TY = S::Y, NT = S::T, WPE = S::E;
    TileSet ts;
    ts.zc = a.plan.zc;
    ts.nbx = (a.nx + TX - 1) / TX;
    ts.nby = (a.ny + TY - 1) / TY;
    ts.nbz = (a.nz + ts.zc - 1) / ts.zc;
    interior_range(a.nx, TX, ts.nbx, ts.bx0, ts.bx1);
    interior_range(a.ny, TY, ts.nby, ts.by0, ts.by1);
    const int nb = ts.nbx * ts.nby * ts.nbz;
    auto go = [&](auto hg, auto frz) {
        constexpr bool HG = decltype(hg)::value, FRZ = decltype(frz)::value;
        if constexpr (LONG) {
            if (far_planes(ts.zc, (double)a.sz * sizeof(R))) {
                k_fused_3d<R, TX, TY, MODE, NT, WPE, HG, FRZ, true><<<nb, NT, 0, s>>>(a, ts);
                return;
            }
        }
        k_fused_3d<R, TX, TY, MODE, NT, WPE, HG, FRZ, false><<<nb, NT, 0, s>>>(a, ts);
    };
    const bool frz = a.lam_mode == LAM_FROZEN;
    if constexpr (G) {
        if (a.igdc) {
            frz ? go(std::true_type{}, std::true_type{}) : go(std::true_type{}, std::false_type{});
            return;
        }
    }
    frz ? go(std::false_type{}, std::true_type{}) : go(std::false_type{}, std::false_type{});
}

template <typename R, int MODE>
void run_3d(const SweepArgs<R>& a, hipStream_t s)
{
    if constexpr (sizeof(R) == 8) {
        if (a.plan.tile == TILE_SMALL) run_3d<TileD_small, R, MODE>(a, s);
        else run_3d<TileD_square, R, MODE, true, true>(a, s);
    } else {
        if (a.plan.tile == TILE_SMALL) run_3d<TileF_small, R, MODE>(a, s);
        else if (a.plan.tile == TILE_WIDE) run_3d<TileF_wide, R, MODE, false>(a, s);
        else run_3d<TileF_square, R, MODE, true, true>(a, s);
    }
}

// Compute units of the current device.
int device_cus()
{
    int dev = 0, n = 0;
    if (hipGetDevice(&dev) != hipSuccess || hipDeviceGetAttribute(&n, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || n <= 0) {
        (void)hipGetLastError();
        return 256;
    }
    return n;
}

// What a sweep with a tile costs, in us: a march step of a workgroup alone
// on its CU, of a full round of `res` workgroups per CU, and the launch with
// the fill of the pipeline.
struct TileCost {
    int tile, x, y, res;
    double alone, full, launch;
};
template <typename T>
constexpr TileCost cost_of(int tile, int res, double alone, double full, double launch)
{
    return {tile, T::X, T::Y, res, alone, full, launch};
}
const TileCost kCost32[] = {cost_of<TileF_wide>(TILE_WIDE, 2, 3.5, 6.0, 5.0),
                            cost_of<TileF_square>(TILE_SQUARE, 2, 2.61, 5.23, 5.0),
                            cost_of<TileF_small>(TILE_SMALL, 8, 1.5, 5.8, 2.0)};
const TileCost kCost64[] = {cost_of<TileD_square>(TILE_SQUARE, 1, 3.0, 3.3, 5.0),
                            cost_of<TileD_small>(TILE_SMALL, 4, 1.9, 4.2, 2.0)};

}  // namespace

// Measured on MI355X at 255^3: fused 0.46 ms (FP32) and 0.81 ms (FP64) per
// sweep against 1.57 ms for the three unfused FP64 kernels.
bool fused_preferred(int, bool) { return true; }

// Tile and chunk length of a grid.  A workgroup marches zc + 3 planes one
// after the other, so short chunks cut the latency of a sweep where the
// chip has room for more workgroups (63^3: 18 us in chunks of 4 planes, 58 us
// in chunks of 32), and long ones the planes that are loaded and computed
// twice.  In between the rounds of resident workgroups decide: the rule
// takes the least modelled time.  The costs above, the share of the last
// round that overlaps the one before and the cost of long marches (the
// workgroups of an XCD drift apart in z and lose the halo lines they share
// in its L2: FP32 511^3 3.72 ms in chunks of 16 planes, 3.99 in 64) were
// fitted to sweeps timed on 28 grids from 20^3 to 511^3 with every tile and
// the chunk lengths below.  Over 55 grids and slabs, 72 timings per precision
// with the per-cell G, the choice is within 0.5 % of the best of any tile and
// length on average and 10 % (FP32: 100^3 51 us, 46 in chunks of 13) and 12 %
// (FP64: 190 x 127 x 101 157 us, 141 in chunks of 21) at worst: lengths that
// divide nz evenly are not all in the list.  FP64 chunks of 64 planes only where a plane has
// at most 1 MB: 255^3 0.81 against 0.85 ms in chunks of 32, but 511^3 7.75
// against 6.59 ms in chunks of 43.  The small FP32 tiles read 1.9 values per
// point, which at 5.1 TB/s takes longer than their march where they fill the
// chip (500 x 500 x 8: 79 us, 32 x 16 tiles 63; with a per-cell G and 12
// planes 150 and 106).
FusedPlan fused_plan_3d(bool fp32, bool has_g, int nx, int ny, int nz, long sz)
{
    static const int cus = device_cus();
    static const int kChunks[] = {3, 4, 5, 6, 8, 10, 12, 16, 20, 24, 28, 32, 43, 50, 64};
    const double drift = fp32 ? 120.0 : 1000.0, overlap = fp32 ? 0.65 : 0.19;
    const double plane = (double)sz * (fp32 ? 4.0 : 8.0);
    FusedPlan best{0, 0};
    double t_best = INFINITY;
    const TileCost* c = fp32 ? kCost32 : kCost64;
    for (int q = 0; q < (fp32 ? 3 : 2); ++q) {
        if (has_g && c[q].tile == TILE_WIDE) continue;
        const double columns = (double)((nx + c[q].x - 1) / c[q].x) * ((ny + c[q].y - 1) / c[q].y);
        for (int zc : kChunks) {
            // the planes of a chunk within the range of 32-bit offsets (the
            // 32 x 16 tiles: one plane), the workgroups within that of a launch
            const double nb = columns * ((nz + zc - 1) / zc);
            if (c[q].tile == TILE_SQUARE ? plane > 2147483647.0 : far_planes(zc, plane)) continue;
            if (nb * c[q].x * c[q].y > 2147483647.0) continue;
            if (!fp32 && zc > 50 && plane > 1048576.0) continue;
            const double rounds = std::floor(nb / (cus * c[q].res)), rest = nb - rounds * cus * c[q].res;
            double step = rounds * c[q].full * (1.0 + zc / drift);
            if (rest > 0.0) {
                const double m = std::ceil(rest / cus);
                double last = c[q].res > 1 ? c[q].alone + (c[q].full - c[q].alone) * (m - 1.0) / (c[q].res - 1.0) : c[q].full;
                if (rounds > 0.0) last = last * (1.0 - overlap) + c[q].full * overlap * rest / (cus * c[q].res);
                step += last;
            }
            double t = c[q].launch + (zc + 3) * step;
            // full rounds of the small FP32 tiles are bound by their halo's bytes
            if (fp32 && c[q].tile == TILE_SMALL) {
                const double halo = (double)((c[q].x + 4) * (c[q].y + 4)) / (c[q].x * c[q].y);
                const double planes = nz + 3.0 * ((nz + zc - 1) / zc);
                t = std::fmax(t, 4.0 * nx * ny * ((16.0 + has_g) * halo * planes + 9.0 * nz) / 5.1e6);
            }
            if (t < t_best) {
                t_best = t;
                best = FusedPlan{c[q].tile, zc};
            }
        }
    }
    return best;
}

template <typename R>
void launch_sweep_fused_3d(const SweepArgs<R>& a, int mode, hipStream_t s)
{
    if (mode == MODE_UPDATE) run_3d<R, MODE_UPDATE>(a, s);
    else if (mode == MODE_CHECK) run_3d<R, MODE_CHECK>(a, s);
    else run_3d<R, MODE_PHYS>(a, s);
}


template void launch_sweep_fused_3d<double>(const SweepArgs<double>&, int, hipStream_t);
template void launch_sweep_fused_3d<float>(const SweepArgs<float>&, int, hipStream_t);

}  // namespace ep

// adjoint.hip -- reverse-mode gradient of J = sum_r g_r fitness_r through the
// time steps, the spring parameters, the parallel-sum rule and the genome MLP.
//
// Forward step n (all nodes, positions x_n): F = springs(x_n, t_n) + gravity +
// ground(z_n); v' = v_n + dt F / m; v'' = friction(v', z_n); v_{n+1} = damping v'';
// x_{n+1} = x_n + dt v_{n+1}.  Its reverse, for adjoints (lx, lv) of (x_{n+1}, v_{n+1}):
//   lvt = damping (lv + dt lx);  lv' = friction Jacobian^T lvt (and a z term);
//   lF = dt/m lv';  lv_n = lv';  lx_n = lx + ground/friction z terms + sum over
//   springs of K_s (lF_hi - lF_lo) (to the lower end, minus to the upper end),
// with K_s = k [(1 - L/r)(I - d^ d^T) + d^ d^T] the spring Hessian.  Per spring
// dJ/dk += -(r - L) d^.(lF_hi - lF_lo) and dJ/dL = k d^.(lF_hi - lF_lo), split by
// L = L0 + L0 a (sin(w t) cos phi + cos(w t) sin phi) into sums GS, GC of
// dJ/dL times sin(w t_n) and cos(w t_n).  Contact and friction branches are those
// the forward run took (the recorded states decide them).
#include <cmath>

#include "spring.h"

namespace sr {

namespace {
typedef float f32x4 __attribute__((ext_vector_type(4)));

struct AArgs {
    const RobotInfo *robots;
    const int32_t *list;
    int count;
    Planes pl;
    const float4 *x0;
    const float4 *rec_x, *rec_v;  // [rec_steps * slot_base + t * slots + s]
    const float4 *rec_u;          // v_n (dashpots, damped ground), same layout
    float4 *rec_l;                // lambda_F of every step (split form), same layout
    int n_steps, rec_steps;       // this segment's steps, the steps a buffer holds for each robot
    const float2 *sc;
    float4 *lx, *lv;    // per slot
    float *gk, *gs, *gc;  // per stencil entry
    float *gd;            // dJ/dc per stencil entry (dashpots)
    SimConst c;
};

// The parameter-gradient terms of one spring at one step (d = x_hi - x_lo,
// u = lambda_F,hi - lambda_F,lo, r2 = |d|^2, ir = 1/r, kL = k L(t), du = d.u):
//   dJ/dk  += -(r - L(t)) du / r,   dJ/d(k L0 a cos phi) += k du / r S,
//   dJ/d(k L0 a sin phi) += k du / r C.
// One helper for the fused reverse step and the split gradient pass, so both
// take the same operations and give the same bits.
__device__ __forceinline__ void spring_grad_sums(float r2, float ir, float kL, float du, float k, float ik, float2 sct,
                                                 float &gk, float &gs, float &gc) {
    const float dhu = du * ir;
    gk = fmaf(-(r2 * ir - kL * ik), dhu, gk);
    const float gL = k * dhu;
    gs = fmaf(gL, sct.x, gs);
    gc = fmaf(gL, sct.y, gc);
}

// XCH: each spring's K_s (lF_hi - lF_lo) is computed once by its lower end and
// handed to the upper end through LDS (three rows per direction, PAD zero
// entries in front); otherwise the upper end recomputes it.  Both give the
// same bits.  The exchange keeps one position/adjoint buffer and adds a
// barrier per step.
// ALAG (exchange form): the position and adjoint reads of direction d + ALAG
// are issued before direction d's arithmetic, which waits for its own two reads
// only (ALAG 0: each read is waited for before the next is issued).
// ONEBUF (recompute form): one position/adjoint buffer instead of two, with a
// barrier at the start of each step, so that 12^3 robots fit in LDS.
// DASH (recompute form, one buffer; Table II model): the forces also depend on
// the velocities v_n of the step.  A spring's dashpot c (v_j - v_i).d^ adds,
// with d = x_j - x_i, u = lambda_F,j - lambda_F,i, w = (v_j - v_i).d and
// du = d.u,
//   lambda_x,i += c/r^2 [du (v_j - v_i) + w u - 2 w du d / r^2]  (minus at j),
//   lambda_v,i += c du d / r^2                                     (minus at j),
//   dJ/dc      += -w du / r^2,
// and the ground force N = k_g(-z) - c_g v_z (where it is not clamped at zero)
// feeds lambda_z and lambda_vz, with the friction threshold following N.
// FNC: a scheduling barrier after each direction's spring work, so the
// compiler does not hoist every neighbour read of the slot (which spilled the
// non-exchange form at 9^3: 1265 VGPRs without, 51 with)
// XCC (exchange form): the directions are taken in XCC chunks, each with its
// own forward half, barrier and receiving half, so that only one chunk's rows
// need LDS (at 9^3-12^3 all 13 directions' rows would not fit beside the
// state).  Each node then adds its forward springs' terms and subtracts its
// backward springs' chunk by chunk, so the sums round differently from one
// chunk (the oracle bounds both).
// NOG (split form): the reverse step keeps no parameter-gradient sums; it
// writes each step's lambda_F to rec_l instead, and k_adj_grad forms the sums
// from the recorded positions and those lambda_F afterwards.  The 13 springs'
// three sums per slot no longer take registers beside the adjoint recursion.
// GPAR (split chunked form): each chunk's spring parameters are read from the
// planes for every step (they stay in L2), issued after the previous chunk's
// forward half and so in flight over its barrier and receiving half, instead
// of held for all 13 directions of every slot: at 10^3-12^3 those did not fit
// the registers beside the recursion and were spilled to scratch, which reads
// the same bytes without overlap.  With dashpots (four planes) it is the better
// form from 10^3 on, without (two or three planes) only at 12^3: at 10^3 and
// 11^3 the held parameters spill 0 to 33 registers, and the extra reads cost
// more (11^3, 256 robots: 9.6 ms a backward of 400 steps held, 10.3 read).
// Together with a gradient pass without spills: backward of 400 steps, Table II
// model, 64 robots of 10^3 / 11^3 / 12^3 7.6 / 13.6 / 27.6 -> 6.1 / 7.8 / 12.8 ms,
// 256 robots 17.0 / 33.6 / 63.2 -> 13.2 / 21.2 / 27.7 ms (12^3 with the recording
// kernel of its own); without dashpots 256 of 12^3 16.4 -> 15.4 ms.
template <int N, int BS, bool PHASE, bool XCH, int ALAG = 0, bool ONEBUF = false, bool DASH = false, bool FNC = false,
          bool NOG = false, int XCC = 1, bool GPAR = false>
__global__ __launch_bounds__(BS) void k_adjoint(AArgs A) {
    static_assert(!GPAR || (XCH && NOG && XCC > 1), "parameters per chunk are a form of the split chunked exchange");
    static_assert(XCC == 1 || XCH, "direction chunks are a form of the exchange");
    static_assert(ALAG == 0 || XCH, "pipelined reads are for the exchange form");
    static_assert(!DASH || XCH || ONEBUF, "the dashpot adjoint keeps one buffer");
    static_assert(!DASH || ALAG == 0, "the dashpot exchange reads its neighbours in order");
    using G = Geo<N>;
    constexpr int SL = G::SL, PAD = G::PAD, XL = G::XL, CL = G::CL;
    constexpr int NPT = (SL + BS - 1) / BS;
    constexpr int NBUF = (XCH || ONEBUF) ? 1 : 2;
    constexpr int NQ = XCH ? 1 : NDIR;
    constexpr int NCH = XCH ? XCC : 1;                 // direction chunks
    constexpr int NDC = (NDIR + NCH - 1) / NCH;        // directions per chunk
    constexpr int NR = DASH ? 4 : 3;                   // exchange rows per direction
    __shared__ float4 xs[NBUF][XL];
    __shared__ float4 lf[NBUF][XL];
    __shared__ float4 vs[DASH ? NBUF : 1][DASH ? XL : 1];
    __shared__ float ku[XCH ? NR * NDC * CL : 1];
    const int tid = threadIdx.x;
    const SimConst c = A.c;
    const bool ground = c.ground != 0;
    const float fz = c.mu_kc_dt_m;  // d(dv)/d(-z) = mu kc dt / m

    for (int q = blockIdx.x; q < A.count; q += gridDim.x) {
        const int r = A.list[q];
        const int base = A.robots[r].slot_base;
        const int pbase = NDIR * base;
        const size_t rbase = (size_t)A.rec_steps * base;
        const float4 ghost = make_float4(1e4f, 1e4f, 1e4f, 0.f), zero = make_float4(0.f, 0.f, 0.f, 0.f);
        if (XCH)
            for (int i = tid; i < NR * NDC * CL; i += BS) ku[i] = 0.f;
        for (int i = tid; i < PAD; i += BS) {
#pragma unroll
            for (int b = 0; b < NBUF; ++b) {
                xs[b][i] = ghost;
                xs[b][PAD + SL + i] = ghost;
                lf[b][i] = zero;
                lf[b][PAD + SL + i] = zero;
                if constexpr (DASH) {
                    vs[b][i] = zero;
                    vs[b][PAD + SL + i] = zero;
                }
            }
        }

        bool pres[NPT];
        float3 X0[NPT], lx[NPT], lv[NPT];
        constexpr int NP = GPAR ? NDC : NDIR;  // directions whose parameters are held
        auto pi_ = [&](int d) { return GPAR ? d % NDC : d; };
        float pk[NPT][NP], pa[NPT][NP], pb[NPT][NP], pik[NPT][NOG ? 1 : NDIR];
        float qk[NPT][NQ], qa[NPT][NQ], qb[NPT][NQ];
        constexpr int NG = NOG ? 1 : NDIR;
        float gk[NPT][NG], gs[NPT][NG], gc[NPT][NG];
        float pd[NPT][DASH ? NP : 1], qd[NPT][DASH ? NQ : 1], gd[NPT][DASH && !NOG ? NDIR : 1];
#pragma unroll
        for (int k = 0; k < NPT; ++k) {
            const int s = tid + k * BS;
            const bool live = s < SL;
            const int sc_ = live ? s : 0;
            const float4 P0 = A.x0[base + sc_];
            pres[k] = live && P0.w != 0.f;
            X0[k] = make_float3(P0.x, P0.y, P0.z);
            const float4 LX = A.lx[base + sc_], LV = A.lv[base + sc_];
            lx[k] = make_float3(LX.x, LX.y, LX.z);
            lv[k] = make_float3(LV.x, LV.y, LV.z);
#pragma unroll
            for (int d = 0; d < NDIR; ++d) {
                if (d >= NP) continue;  // GPAR: the first chunk's
                const int pi = pbase + d * SL + sc_;
                const float kk = live ? A.pl.k[pi] : 0.f;
                pk[k][d] = kk;
                pa[k][d] = live ? A.pl.kal[pi] : 0.f;
                pb[k][d] = (live && PHASE) ? A.pl.kbe[pi] : 0.f;
                if constexpr (!NOG) {
                    pik[k][d] = kk != 0.f ? 1.0f / kk : 0.f;
                    gk[k][d] = live ? A.gk[pi] : 0.f;
                    gs[k][d] = live ? A.gs[pi] : 0.f;
                    gc[k][d] = live ? A.gc[pi] : 0.f;
                }
                if constexpr (DASH) {
                    pd[k][d] = live ? A.pl.kd[pi] : 0.f;
                    if constexpr (!NOG) gd[k][DASH && !NOG ? d : 0] = live ? A.gd[pi] : 0.f;
                }
            }
            if (!XCH) {
#pragma unroll
                for (int d = 0; d < NQ; ++d) {
                    const int lo = s - dir_off(d, N);
                    const bool ok = live && lo >= 0;
                    const int qi = pbase + d * SL + (ok ? lo : 0);
                    qk[k][d] = ok ? A.pl.k[qi] : 0.f;
                    qa[k][d] = ok ? A.pl.kal[qi] : 0.f;
                    qb[k][d] = (ok && PHASE) ? A.pl.kbe[qi] : 0.f;
                    if constexpr (DASH) qd[k][d] = ok ? A.pl.kd[qi] : 0.f;
                }
            }
        }
        __syncthreads();

        // the recorded state of each step is read one step ahead, so the global
        // loads are in flight during the previous step's spring part
        float4 XRn[NPT], VPn[NPT], VNn[DASH ? NPT : 1];
#pragma unroll
        for (int k = 0; k < NPT; ++k) {
            const int s = tid + k * BS;
            if (pres[k] && A.n_steps > 0) {
                XRn[k] = A.rec_x[rbase + (size_t)(A.n_steps - 1) * SL + s];
                VPn[k] = A.rec_v[rbase + (size_t)(A.n_steps - 1) * SL + s];
                if constexpr (DASH) VNn[k] = A.rec_u[rbase + (size_t)(A.n_steps - 1) * SL + s];
            } else {
                XRn[k] = make_float4(0.f, 0.f, 0.f, 0.f);
                VPn[k] = XRn[k];
                if constexpr (DASH) VNn[k] = XRn[k];
            }
        }
        float2 sc_next = A.n_steps > 0 ? A.sc[A.n_steps - 1] : make_float2(0.f, 0.f);
        for (int t = A.n_steps - 1; t >= 0; --t) {
            const int b = NBUF == 1 ? 0 : (t & 1);
            if (NBUF == 1) __syncthreads();  // the previous step's readers are done with the buffers
            const float2 sct = sc_next;
            if (t > 0) sc_next = A.sc[t - 1];
            float4 XRc[NPT], VPc[NPT], VNc[DASH ? NPT : 1];
#pragma unroll
            for (int k = 0; k < NPT; ++k) {
                const int s = tid + k * BS;
                XRc[k] = XRn[k];
                VPc[k] = VPn[k];
                if constexpr (DASH) VNc[k] = VNn[k];
                if (pres[k] && t > 0) {
                    XRn[k] = A.rec_x[rbase + (size_t)(t - 1) * SL + s];
                    VPn[k] = A.rec_v[rbase + (size_t)(t - 1) * SL + s];
                    if constexpr (DASH) VNn[k] = A.rec_u[rbase + (size_t)(t - 1) * SL + s];
                }
            }
            float3 Xr[NPT], LF[NPT], Vr[DASH ? NPT : 1];
            // node-local part of the reverse step
#pragma unroll
            for (int k = 0; k < NPT; ++k) {
                const int s = tid + k * BS;
                if (s >= SL) continue;
                float3 X = X0[k], lF = make_float3(0.f, 0.f, 0.f);
                if (pres[k]) {
                    const float4 XR = XRc[k];
                    const float4 VP = VPc[k];
                    X = make_float3(XR.x, XR.y, XR.z);
                    float ux = c.damping * fmaf(c.dt, lx[k].x, lv[k].x);
                    float uy = c.damping * fmaf(c.dt, lx[k].y, lv[k].y);
                    const float uz = c.damping * fmaf(c.dt, lx[k].z, lv[k].z);
                    const bool below = ground && X.z < 0.f;
                    if (DASH && c.gdamp) {
                        // the damped ground: N = max(k_g (-z) - c_g v_z, 0), the
                        // friction threshold follows N; the forward's operations
                        const float4 VN = VNc[DASH ? k : 0];
                        const float Nf = below ? fmaxf(fmaf(-c.cg, VN.z, c.kc * -X.z), 0.f) : 0.f;
                        float lN = 0.f;
                        if (Nf > 0.f) {
                            const float dv = c.mu_dt_m * Nf;
                            const float u = sqrtf(fmaf(VP.y, VP.y, VP.x * VP.x));
                            if (u <= fmaxf(dv, c.mus_dt_m * Nf)) {
                                ux = 0.f;
                                uy = 0.f;
                            } else {
                                const float hx = VP.x / u, hy = VP.y / u;
                                const float dot = fmaf(hy, uy, hx * ux);
                                lN = -c.mu_dt_m * dot;
                                const float cc = dv / u;
                                const float nx = ux - cc * (ux - hx * dot);
                                const float ny = uy - cc * (uy - hy * dot);
                                ux = nx;
                                uy = ny;
                            }
                        }
                        lF = make_float3(c.dt_m * ux, c.dt_m * uy, c.dt_m * uz);
                        float lvz = uz;
                        if (Nf > 0.f) {
                            lN += lF.z;
                            lx[k].z = fmaf(-c.kc, lN, lx[k].z);
                            lvz = fmaf(-c.cg, lN, lvz);
                        }
                        lv[k] = make_float3(ux, uy, lvz);
                    } else {
                        if (below) {
                            const float dv = c.mu_kc_dt_m * (-X.z);
                            const float u = sqrtf(fmaf(VP.y, VP.y, VP.x * VP.x));
                            if (u <= fmaxf(dv, c.mus_kc_dt_m * (-X.z))) {
                                ux = 0.f;
                                uy = 0.f;
                            } else {
                                const float hx = VP.x / u, hy = VP.y / u;
                                const float dot = fmaf(hy, uy, hx * ux);
                                lx[k].z = fmaf(fz, dot, lx[k].z);
                                const float cc = dv / u;
                                const float nx = ux - cc * (ux - hx * dot);
                                const float ny = uy - cc * (uy - hy * dot);
                                ux = nx;
                                uy = ny;
                            }
                        }
                        lv[k] = make_float3(ux, uy, uz);
                        lF = make_float3(c.dt_m * ux, c.dt_m * uy, c.dt_m * uz);
                        if (below) lx[k].z = fmaf(-c.kc, lF.z, lx[k].z);
                    }
                }
                Xr[k] = X;
                LF[k] = lF;
                if (NOG && pres[k]) A.rec_l[rbase + (size_t)t * SL + s] = make_float4(lF.x, lF.y, lF.z, 0.f);
                xs[b][PAD + s] = make_float4(X.x, X.y, X.z, 0.f);
                lf[b][PAD + s] = make_float4(lF.x, lF.y, lF.z, 0.f);
                if constexpr (DASH) {
                    const float4 VN = pres[k] ? VNc[DASH ? k : 0] : zero;
                    Vr[DASH ? k : 0] = make_float3(VN.x, VN.y, VN.z);
                    vs[DASH ? b : 0][PAD + s] = make_float4(VN.x, VN.y, VN.z, 0.f);
                }
            }
            __syncthreads();
            // spring part: every node takes K_s (lF_hi - lF_lo) from each spring it touches
            float3 accs[NPT], accv[DASH ? NPT : 1];
#pragma unroll
            for (int k = 0; k < NPT; ++k) {
                accs[k] = make_float3(0.f, 0.f, 0.f);
                if constexpr (DASH) accv[DASH ? k : 0] = make_float3(0.f, 0.f, 0.f);
            }
#pragma unroll
            for (int ch = 0; ch < NCH; ++ch) {
            const int d0 = ch * NDC, d1 = d0 + NDC < NDIR ? d0 + NDC : NDIR;
            if (ch > 0) __syncthreads();  // the previous chunk's receivers are done with the rows
#if SR_POISON_LDS
            // debug build: each thread's own exchange entries of the chunk hold NaN
            // until it writes them
            if (XCH)
                for (int k = 0; k < NPT; ++k) {
                    const int s = tid + k * BS;
                    if (s < SL && pres[k])  // absent slots never write theirs (they stay zero)
                        for (int q = 0; q < NR; ++q)
                            for (int j = 0; j < d1 - d0; ++j) ku[(q * NDC + j) * CL + PAD + s] = __builtin_nanf("");
                }
#endif
#pragma unroll
            for (int k = 0; k < NPT; ++k) {
                const int s = tid + k * BS;
                if (s >= SL || !pres[k]) continue;
                const float4 *xsb = xs[b] + s;
                const float4 *lfb = lf[b] + s;
                const float4 *vsb = vs[DASH ? b : 0] + s;
                float3 acc = accs[k], av = make_float3(0.f, 0.f, 0.f);
                if constexpr (DASH) av = accv[DASH ? k : 0];
                float4 QY[NDIR], QL[NDIR];
                if constexpr (ALAG > 0) {
#pragma unroll
                    for (int d = 0; d < NDIR; ++d) {
                        if (d < d0 || d >= d1 || d >= d0 + ALAG) continue;
                        QY[d] = xsb[PAD + dir_off(d, N)];
                        QL[d] = lfb[PAD + dir_off(d, N)];
                    }
                }
#pragma unroll
                for (int d = 0; d < NDIR; ++d) {
                    if (d < d0 || d >= d1) continue;
                    // forward spring: self is the lower end
                    float3 Y, LJ;
                    if constexpr (ALAG > 0) {
                        constexpr int dummy = 0;
                        const int e = d + ALAG < d1 ? d + ALAG : dummy;
                        if (d + ALAG < d1) {
                            QY[e] = xsb[PAD + dir_off(e, N)];
                            QL[e] = lfb[PAD + dir_off(e, N)];
                        }
                        keep_w(QY[d].w);
                        keep_w(QL[d].w);
                        Y = make_float3(QY[d].x, QY[d].y, QY[d].z);
                        LJ = make_float3(QL[d].x, QL[d].y, QL[d].z);
                    } else {
                        Y = ld3(xsb + (PAD + dir_off(d, N)));
                        LJ = ld3(lfb + (PAD + dir_off(d, N)));
                    }
                    const float dx = Y.x - Xr[k].x, dy = Y.y - Xr[k].y, dz = Y.z - Xr[k].z;
                    const float ux = LJ.x - LF[k].x, uy = LJ.y - LF[k].y, uz = LJ.z - LF[k].z;
                    const float r2 = len2(dx, dy, dz);
                    const float ir = __builtin_amdgcn_rsqf(r2);
                    const float kk = pk[k][pi_(d)];
                    float kL = fmaf(pa[k][pi_(d)], sct.x, kk * L0d(c, d));
                    if (PHASE) kL = fmaf(pb[k][pi_(d)], sct.y, kL);
                    const float c1 = fmaf(-kL, ir, kk);
                    const float du = fmaf(dz, uz, fmaf(dy, uy, dx * ux));
                    const float c2 = (kL * ir) * ir * ir * du;
                    float kx = fmaf(c1, ux, c2 * dx), ky = fmaf(c1, uy, c2 * dy), kz = fmaf(c1, uz, c2 * dz);
                    if constexpr (DASH) {
                        // dashpot beside the spring (self is the lower end i)
                        const float3 VJ = ld3(vsb + (PAD + dir_off(d, N)));
                        const float3 VI = Vr[DASH ? k : 0];
                        const float wx = VJ.x - VI.x, wy = VJ.y - VI.y, wz = VJ.z - VI.z;
                        const float cd = pd[k][DASH ? pi_(d) : 0];
                        const float ir2 = ir * ir;
                        const float wv = fmaf(dz, wz, fmaf(dy, wy, dx * wx));
                        const float ce = cd * ir2, q2 = -2.f * wv * du * ir2;
                        kx = fmaf(ce, fmaf(du, wx, fmaf(wv, ux, q2 * dx)), kx);
                        ky = fmaf(ce, fmaf(du, wy, fmaf(wv, uy, q2 * dy)), ky);
                        kz = fmaf(ce, fmaf(du, wz, fmaf(wv, uz, q2 * dz)), kz);
                        const float cv = ce * du;
                        av.x = fmaf(cv, dx, av.x);
                        av.y = fmaf(cv, dy, av.y);
                        av.z = fmaf(cv, dz, av.z);
                        // the upper end forms its velocity-adjoint term c du d / r^2
                        // from this scalar and its own difference vector
                        if (XCH) ku[(3 * NDC + d - d0) * CL + PAD + s] = cv;
                        if constexpr (!NOG) gd[k][DASH && !NOG ? d : 0] = fmaf(-wv * du, ir2, gd[k][DASH && !NOG ? d : 0]);
                    }
                    acc.x += kx;
                    acc.y += ky;
                    acc.z += kz;
                    if (XCH) {
                        ku[(0 * NDC + d - d0) * CL + PAD + s] = kx;
                        ku[(1 * NDC + d - d0) * CL + PAD + s] = ky;
                        ku[(2 * NDC + d - d0) * CL + PAD + s] = kz;
                    }
                    if constexpr (!NOG)
                        spring_grad_sums(r2, ir, kL, du, kk, pik[k][NOG ? 0 : d], sct, gk[k][NOG ? 0 : d], gs[k][NOG ? 0 : d],
                                         gc[k][NOG ? 0 : d]);
                    if (FNC) __builtin_amdgcn_sched_barrier(0);
                }
                if (!XCH) {
#pragma unroll
                    for (int d = 0; d < NQ; ++d) {
                        // backward spring: self is the upper end
                        const float3 Y = ld3(xsb + (PAD - dir_off(d, N)));
                        const float3 LI = ld3(lfb + (PAD - dir_off(d, N)));
                        const float dx = Xr[k].x - Y.x, dy = Xr[k].y - Y.y, dz = Xr[k].z - Y.z;
                        const float ux = LF[k].x - LI.x, uy = LF[k].y - LI.y, uz = LF[k].z - LI.z;
                        const float r2 = len2(dx, dy, dz);
                        const float ir = __builtin_amdgcn_rsqf(r2);
                        float kL = fmaf(qa[k][d], sct.x, qk[k][d] * L0d(c, d));
                        if (PHASE) kL = fmaf(qb[k][d], sct.y, kL);
                        const float c1 = fmaf(-kL, ir, qk[k][d]);
                        const float du = fmaf(dz, uz, fmaf(dy, uy, dx * ux));
                        const float c2 = (kL * ir) * ir * ir * du;
                        float kx = fmaf(c1, ux, c2 * dx), ky = fmaf(c1, uy, c2 * dy), kz = fmaf(c1, uz, c2 * dz);
                        if constexpr (DASH) {
                            // dashpot beside the spring (self is the upper end j)
                            const float3 VI = ld3(vsb + (PAD - dir_off(d, N)));
                            const float3 VJ = Vr[DASH ? k : 0];
                            const float wx = VJ.x - VI.x, wy = VJ.y - VI.y, wz = VJ.z - VI.z;
                            const float cd = qd[k][DASH ? d : 0];
                            const float ir2 = ir * ir;
                            const float wv = fmaf(dz, wz, fmaf(dy, wy, dx * wx));
                            const float ce = cd * ir2, q2 = -2.f * wv * du * ir2;
                            kx = fmaf(ce, fmaf(du, wx, fmaf(wv, ux, q2 * dx)), kx);
                            ky = fmaf(ce, fmaf(du, wy, fmaf(wv, uy, q2 * dy)), ky);
                            kz = fmaf(ce, fmaf(du, wz, fmaf(wv, uz, q2 * dz)), kz);
                            const float cv = ce * du;
                            av.x = fmaf(-cv, dx, av.x);
                            av.y = fmaf(-cv, dy, av.y);
                            av.z = fmaf(-cv, dz, av.z);
                        }
                        acc.x -= kx;
                        acc.y -= ky;
                        acc.z -= kz;
                        if (FNC) __builtin_amdgcn_sched_barrier(0);
                    }
                }
                accs[k] = acc;
                if constexpr (DASH) accv[DASH ? k : 0] = av;
            }
            if constexpr (GPAR) {
                // the next chunk's parameters (after the last, the next step's first)
                const int n0 = ch + 1 < NCH ? d1 : 0;
#pragma unroll
                for (int k = 0; k < NPT; ++k) {
                    int s = tid + k * BS;
                    __asm__ volatile("" : "+v"(s));  // not out of the time loop
#pragma unroll
                    for (int j = 0; j < NDC; ++j) {
                        const int d = n0 + j;
                        if (d >= NDIR || !pres[k]) continue;
                        const int pi = pbase + d * SL + s;
                        pk[k][j] = A.pl.k[pi];
                        pa[k][j] = A.pl.kal[pi];
                        if (PHASE) pb[k][j] = A.pl.kbe[pi];
                        if constexpr (DASH) pd[k][DASH ? j : 0] = A.pl.kd[pi];
                    }
                }
            }
            if (XCH) {
                __syncthreads();
#pragma unroll
                for (int k = 0; k < NPT; ++k) {
                    const int s = tid + k * BS;
                    if (s >= SL || !pres[k]) continue;
                    float3 acc = accs[k];
#pragma unroll
                    for (int d = 0; d < NDIR; ++d) {
                        if (d < d0 || d >= d1) continue;
                        const int lo = PAD + s - dir_off(d, N);
                        acc.x -= ku[(0 * NDC + d - d0) * CL + lo];
                        acc.y -= ku[(1 * NDC + d - d0) * CL + lo];
                        acc.z -= ku[(2 * NDC + d - d0) * CL + lo];
                    }
                    accs[k] = acc;
                    if constexpr (DASH) {
                        // the recompute form's operations at the upper end: d = x_hi - x_lo
                        float3 av = accv[DASH ? k : 0];
#pragma unroll
                        for (int d = 0; d < NDIR; ++d) {
                            if (d < d0 || d >= d1) continue;
                            const int lo = PAD + s - dir_off(d, N);
                            const float3 Y = ld3(xs[b] + lo);
                            const float cv = ku[(3 * NDC + d - d0) * CL + lo];
                            av.x = fmaf(-cv, Xr[k].x - Y.x, av.x);
                            av.y = fmaf(-cv, Xr[k].y - Y.y, av.y);
                            av.z = fmaf(-cv, Xr[k].z - Y.z, av.z);
                        }
                        accv[DASH ? k : 0] = av;
                    }
                }
            }
            }  // direction chunks
#pragma unroll
            for (int k = 0; k < NPT; ++k) {
                const int s = tid + k * BS;
                if (s >= SL || !pres[k]) continue;
                const float3 acc = accs[k];
                lx[k].x += acc.x;
                lx[k].y += acc.y;
                lx[k].z += acc.z;
                if constexpr (DASH) {
                    const float3 av = accv[DASH ? k : 0];
                    lv[k].x += av.x;
                    lv[k].y += av.y;
                    lv[k].z += av.z;
                }
            }
        }
        // the adjoint state and the gradient sums carry over to the previous segment
#pragma unroll
        for (int k = 0; k < NPT; ++k) {
            const int s = tid + k * BS;
            if (s >= SL) continue;
            A.lx[base + s] = make_float4(lx[k].x, lx[k].y, lx[k].z, 0.f);
            A.lv[base + s] = make_float4(lv[k].x, lv[k].y, lv[k].z, 0.f);
#pragma unroll
            for (int d = 0; d < NDIR; ++d) {
                const int pi = pbase + d * SL + s;
                if constexpr (!NOG) {
                    A.gk[pi] = gk[k][NOG ? 0 : d];
                    A.gs[pi] = gs[k][NOG ? 0 : d];
                    A.gc[pi] = gc[k][NOG ? 0 : d];
                }
                if constexpr (DASH && !NOG) A.gd[pi] = gd[k][DASH && !NOG ? d : 0];
            }
        }
        __syncthreads();
    }
}

// One forward spring of the split gradient pass at one step: self (X, lambda_F L,
// velocity V) is the lower end, (Y, LJ, VJ) the upper; with dashpots also dJ/dc,
// as in the fused reverse step.
template <bool PHASE, bool DASH>
__device__ __forceinline__ void grad_spring(float3 X, float3 L, float3 V, float3 Y, float3 LJ, float3 VJ, float L0,
                                            float pk, float pa, float pb, float pik, float2 sct, float &gk, float &gs,
                                            float &gc, float &gd) {
    const float dx = Y.x - X.x, dy = Y.y - X.y, dz = Y.z - X.z;
    const float ux = LJ.x - L.x, uy = LJ.y - L.y, uz = LJ.z - L.z;
    const float r2 = len2(dx, dy, dz);
    const float ir = __builtin_amdgcn_rsqf(r2);
    float kL = fmaf(pa, sct.x, pk * L0);
    if (PHASE) kL = fmaf(pb, sct.y, kL);
    const float du = fmaf(dz, uz, fmaf(dy, uy, dx * ux));
    spring_grad_sums(r2, ir, kL, du, pk, pik, sct, gk, gs, gc);
    if constexpr (DASH) {
        const float wx = VJ.x - V.x, wy = VJ.y - V.y, wz = VJ.z - V.z;
        const float ir2 = ir * ir;
        const float wv = fmaf(dz, wz, fmaf(dy, wy, dx * wx));
        gd = fmaf(-wv * du, ir2, gd);
    }
}

// Split form, second pass: the parameter-gradient sums of the forward springs
// of directions D0 .. D1 - 1 over one segment, from the recorded positions x_t
// (rec_x; an absent slot sits at its build position) and the reverse step's
// lambda_F (rec_l; zero on absent slots), step by step from the segment's end
// to its start as in the fused form, through the same helper: the same bits.
// One LDS buffer of positions and one of lambda_F, two barriers per step.
template <int N, int BS, bool PHASE, int D0, int D1, bool DASH>
__device__ __forceinline__ void adj_grad_robot(const AArgs &A, int q, float4 *xs, float4 *lf, float4 *vs) {
    using G = Geo<N>;
    constexpr int SL = G::SL, PAD = G::PAD;
    constexpr int NPT = (SL + BS - 1) / BS;
    constexpr int ND = D1 - D0;
    const int tid = threadIdx.x;
    const SimConst c = A.c;
    {
        const int r = A.list[q];
        const int base = A.robots[r].slot_base;
        const int pbase = NDIR * base;
        const size_t rbase = (size_t)A.rec_steps * base;
        const float4 ghost = make_float4(1e4f, 1e4f, 1e4f, 0.f), zero = make_float4(0.f, 0.f, 0.f, 0.f);
        for (int i = tid; i < PAD; i += BS) {
            xs[i] = ghost;
            xs[PAD + SL + i] = ghost;
            lf[i] = zero;
            lf[PAD + SL + i] = zero;
            if constexpr (DASH) {
                vs[i] = zero;
                vs[PAD + SL + i] = zero;
            }
        }
        bool pres[NPT];
        float3 X0[NPT];
        float pk[NPT][ND], pa[NPT][ND], pb[NPT][ND], pik[NPT][ND], gk[NPT][ND], gs[NPT][ND], gc[NPT][ND];
        float gd[NPT][DASH ? ND : 1];
#pragma unroll
        for (int k = 0; k < NPT; ++k) {
            const int s = tid + k * BS;
            const bool live = s < SL;
            const int sc_ = live ? s : 0;
            const float4 P0 = A.x0[base + sc_];
            pres[k] = live && P0.w != 0.f;
            X0[k] = make_float3(P0.x, P0.y, P0.z);
#pragma unroll
            for (int j = 0; j < ND; ++j) {
                const int pi = pbase + (D0 + j) * SL + sc_;
                const float kk = live ? A.pl.k[pi] : 0.f;
                pk[k][j] = kk;
                pa[k][j] = live ? A.pl.kal[pi] : 0.f;
                pb[k][j] = (live && PHASE) ? A.pl.kbe[pi] : 0.f;
                pik[k][j] = kk != 0.f ? 1.0f / kk : 0.f;
                gk[k][j] = live ? A.gk[pi] : 0.f;
                gs[k][j] = live ? A.gs[pi] : 0.f;
                gc[k][j] = live ? A.gc[pi] : 0.f;
                if constexpr (DASH) gd[k][DASH ? j : 0] = live ? A.gd[pi] : 0.f;
            }
        }
        // each step's recorded values are loaded one step ahead, so the global
        // loads are in flight during the previous step's spring work
        float4 XRn[NPT], LLn[NPT], VNn[DASH ? NPT : 1];
#pragma unroll
        for (int k = 0; k < NPT; ++k) {
            const int s = tid + k * BS;
            XRn[k] = zero;
            LLn[k] = zero;
            if constexpr (DASH) VNn[DASH ? k : 0] = zero;
            if (pres[k] && A.n_steps > 0) {
                XRn[k] = A.rec_x[rbase + (size_t)(A.n_steps - 1) * SL + s];
                LLn[k] = A.rec_l[rbase + (size_t)(A.n_steps - 1) * SL + s];
                if constexpr (DASH) VNn[DASH ? k : 0] = A.rec_u[rbase + (size_t)(A.n_steps - 1) * SL + s];
            }
        }
        for (int t = A.n_steps - 1; t >= 0; --t) {
            __syncthreads();  // the previous step's readers are done with the buffers
            const float2 sct = A.sc[t];
            float3 Xr[NPT], LF[NPT], Vr[DASH ? NPT : 1];
#pragma unroll
            for (int k = 0; k < NPT; ++k) {
                const int s = tid + k * BS;
                if (s >= SL) continue;
                float3 X = X0[k];
                float4 L = zero, V = zero;
                if (pres[k]) {
                    const float4 XR = XRn[k];
                    X = make_float3(XR.x, XR.y, XR.z);
                    L = LLn[k];
                    if constexpr (DASH) V = VNn[DASH ? k : 0];
                    if (t > 0) {
                        XRn[k] = A.rec_x[rbase + (size_t)(t - 1) * SL + s];
                        LLn[k] = A.rec_l[rbase + (size_t)(t - 1) * SL + s];
                        if constexpr (DASH) VNn[DASH ? k : 0] = A.rec_u[rbase + (size_t)(t - 1) * SL + s];
                    }
                }
                Xr[k] = X;
                LF[k] = make_float3(L.x, L.y, L.z);
                xs[PAD + s] = make_float4(X.x, X.y, X.z, 0.f);
                lf[PAD + s] = make_float4(L.x, L.y, L.z, 0.f);
                if constexpr (DASH) {
                    Vr[DASH ? k : 0] = make_float3(V.x, V.y, V.z);
                    vs[PAD + s] = make_float4(V.x, V.y, V.z, 0.f);
                }
            }
            __syncthreads();
#pragma unroll
            for (int k = 0; k < NPT; ++k) {
                const int s = tid + k * BS;
                if (s >= SL || !pres[k]) continue;
#pragma unroll
                for (int j = 0; j < ND; ++j) {
                    const int d = D0 + j;
                    const int at = s + PAD + dir_off(d, N);
                    float3 V = Xr[k], VJ = Xr[k];  // unused without dashpots
                    if constexpr (DASH) V = Vr[DASH ? k : 0], VJ = ld3(vs + at);
                    float none = 0.f;
                    grad_spring<PHASE, DASH>(Xr[k], LF[k], V, ld3(xs + at), ld3(lf + at), VJ, L0d(c, d), pk[k][j],
                                             pa[k][j], pb[k][j], pik[k][j], sct, gk[k][j], gs[k][j], gc[k][j],
                                             DASH ? gd[k][DASH ? j : 0] : none);
                    __builtin_amdgcn_sched_barrier(0);
                }
            }
        }
#pragma unroll
        for (int k = 0; k < NPT; ++k) {
            const int s = tid + k * BS;
            if (s >= SL) continue;
#pragma unroll
            for (int j = 0; j < ND; ++j) {
                const int pi = pbase + (D0 + j) * SL + s;
                A.gk[pi] = gk[k][j];
                A.gs[pi] = gs[k][j];
                A.gc[pi] = gc[k][j];
                if constexpr (DASH) A.gd[pi] = gd[k][DASH ? j : 0];
            }
        }
        __syncthreads();
    }
}

// The gradient pass over all directions in one workgroup per robot (PARTS 1),
// or over 0..6 and 7..12 in two side by side (PARTS 2; they write disjoint sums).
// It runs beside the next segment's reversal, whose workgroups take a whole CU
// each: few workgroups that fill a CU leave it the others.
// DASH: also dJ/dc of the spring dashpots, from the recorded velocities v_n.
template <int N, int BS, bool PHASE, int PARTS, bool DASH = false>
__global__ __launch_bounds__(BS) void k_adj_grad(AArgs A) {
    __shared__ float4 xs[Geo<N>::XL];
    __shared__ float4 lf[Geo<N>::XL];
    __shared__ float4 vs[DASH ? Geo<N>::XL : 1];
    for (int q = blockIdx.x; q < A.count; q += gridDim.x) {
        if constexpr (PARTS == 1) {
            adj_grad_robot<N, BS, PHASE, 0, 13, DASH>(A, q, xs, lf, vs);
        } else {
            if (blockIdx.y == 0)
                adj_grad_robot<N, BS, PHASE, 0, 7, DASH>(A, q, xs, lf, vs);
            else
                adj_grad_robot<N, BS, PHASE, 7, 13, DASH>(A, q, xs, lf, vs);
        }
    }
}

// The same sums in tiles of TS slots.  A spring's sums need only its two ends,
// and it is summed at its lower end, whose neighbours lie at higher slots: a
// workgroup takes TS consecutive slots, one a thread with all 13 directions, and
// stages them with the PAD slots above for each step (two buffers, one barrier a
// step, the next step's values in flight over the spring work).  Bound by the
// chain of a step in few waves (1.6 us a step in a small launch at any side, 2.2
// with dashpots) against 2.4 to 5.5 for the form above; the workgroups are
// numbered so that a robot's tiles share an XCD and its L2.  It is taken for the
// segment reversed last, whose pass has nothing beside it and ends the backward
// (64 robots, base model, 8^3 / 10^3: 242 / 294 -> 178 / 195 us of 100 steps; not at
// 8^3 with dashpots, 212 us in two parts against 219 at 3 robots), and
// for every segment at 12^3 and at 11^3 with dashpots (1200 steps backward, 256
// robots of 12^3 45 -> 34 ms, with dashpots 82 -> 68; 64 robots 17.1 -> 15.0 and
// 36.9 -> 34.4).  On smaller sides the
// many small workgroups beside a reversal leave its next launch no empty CU (10^3,
// 64 and 128 robots: 3.07 and 4.2 ms with the form above, 3.3 and 4.1 in tiles).
template <int N, int TS, bool PHASE, bool DASH>
__global__ __launch_bounds__(TS, 2) void k_adj_grad_tiles(AArgs A) {
    using G = Geo<N>;
    constexpr int SL = G::SL, PAD = G::PAD, TL = TS + PAD;
    constexpr int NT = (SL + TS - 1) / TS, NE = (TL + TS - 1) / TS;
    __shared__ float4 xs[2][TL + 1], lf[2][TL + 1], vs[DASH ? 2 : 1][DASH ? TL + 1 : 1];
    const int tid = threadIdx.x, T = A.n_steps;
    const SimConst c = A.c;
    if (T <= 0) return;
    for (int w = blockIdx.x; w < (A.count + 7) / 8 * 8 * NT; w += gridDim.x) {
        const int q = w / 8 / NT * 8 + w % 8, s0 = w / 8 % NT * TS;
        if (q >= A.count) continue;
        const int base = A.robots[A.list[q]].slot_base;
        const float4 zero = make_float4(0.f, 0.f, 0.f, 0.f);
        // Absent nodes rest at their places with no adjoint and ghosts lie far off:
        // both are written once, and their steps' values go to the entry past the
        // tile's, so that every thread has the same loads in flight.
        int to[NE], from[NE];
        bool pres = false;
#pragma unroll
        for (int e = 0; e < NE; ++e) {
            const int i = tid + e * TS, s = s0 + i;
            const bool in = i < TL && s < SL;
            float4 P0 = make_float4(1e4f, 1e4f, 1e4f, 0.f);
            if (in) P0 = A.x0[base + s];
            to[e] = P0.w != 0.f ? i : TL;
            from[e] = in ? s : s0;
            if (e == 0) pres = P0.w != 0.f;
            P0.w = 0.f;
            if (i < TL)
#pragma unroll
                for (int h = 0; h < 2; ++h) {
                    xs[h][i] = P0;
                    lf[h][i] = zero;
                    if constexpr (DASH) vs[h][i] = zero;
                }
        }
        if (!__syncthreads_or(pres)) continue;
        const int pbase = NDIR * base + s0 + tid;
        float pk[NDIR], pa[NDIR], pb[NDIR], pik[NDIR], gk[NDIR], gs[NDIR], gc[NDIR], gd[DASH ? NDIR : 1];
#pragma unroll
        for (int d = 0; d < NDIR; ++d) {
            const int pi = pbase + d * SL;
            pk[d] = pres ? A.pl.k[pi] : 0.f;
            pa[d] = pres ? A.pl.kal[pi] : 0.f;
            pb[d] = pres && PHASE ? A.pl.kbe[pi] : 0.f;
            pik[d] = pk[d] != 0.f ? 1.0f / pk[d] : 0.f;
            gk[d] = pres ? A.gk[pi] : 0.f;
            gs[d] = pres ? A.gs[pi] : 0.f;
            gc[d] = pres ? A.gc[pi] : 0.f;
            if constexpr (DASH) gd[d] = pres ? A.gd[pi] : 0.f;
        }
        f32x4 xn[NE], ln[NE], vn[DASH ? NE : 1];
        const size_t rbase = (size_t)A.rec_steps * base;
        auto fetch = [&](int t) {
            const size_t at = rbase + (size_t)t * SL;
#pragma unroll
            for (int e = 0; e < NE; ++e) {
                xn[e] = *(const f32x4 *)&A.rec_x[at + from[e]];
                ln[e] = *(const f32x4 *)&A.rec_l[at + from[e]];
                if constexpr (DASH) vn[e] = *(const f32x4 *)&A.rec_u[at + from[e]];
            }
        };
        auto stage = [&](int t) {
#pragma unroll
            for (int e = 0; e < NE; ++e) {
                *(f32x4 *)&xs[t & 1][to[e]] = xn[e];
                *(f32x4 *)&lf[t & 1][to[e]] = ln[e];
                if constexpr (DASH) *(f32x4 *)&vs[t & 1][to[e]] = vn[e];
            }
        };
        fetch(T - 1);
        stage(T - 1);
        fetch(T > 1 ? T - 2 : 0);
        __syncthreads();
        for (int t = T - 1; t >= 0; --t) {
            const float2 sct = A.sc[t];
            if (pres) {
                const float4 *xb = xs[t & 1] + tid, *lb = lf[t & 1] + tid, *vb = vs[DASH ? t & 1 : 0] + (DASH ? tid : 0);
                const float3 X = ld3(xb), L = ld3(lb), V = DASH ? ld3(vb) : X;
                // the reads of direction d + 1 are issued before direction d's arithmetic
                float3 Y = ld3(xb + dir_off(0, N)), LJ = ld3(lb + dir_off(0, N)), VJ = V;
                if constexpr (DASH) VJ = ld3(vb + dir_off(0, N));
#pragma unroll
                for (int d = 0; d < NDIR; ++d) {
                    const float3 Yd = Y, Ld = LJ, Vd = VJ;
                    if (d + 1 < NDIR) {
                        Y = ld3(xb + dir_off(d + 1, N));
                        LJ = ld3(lb + dir_off(d + 1, N));
                        if constexpr (DASH) VJ = ld3(vb + dir_off(d + 1, N));
                    }
                    float none = 0.f;
                    grad_spring<PHASE, DASH>(X, L, V, Yd, Ld, Vd, L0d(c, d), pk[d], pa[d], pb[d], pik[d], sct, gk[d],
                                             gs[d], gc[d], DASH ? gd[DASH ? d : 0] : none);
                    __builtin_amdgcn_sched_barrier(0);
                }
            }
            if (t > 0) {
                stage(t - 1);
                fetch(t > 1 ? t - 2 : 0);
            }
            __syncthreads();
        }
        if (!pres) continue;
#pragma unroll
        for (int d = 0; d < NDIR; ++d) {
            const int pi = pbase + d * SL;
            A.gk[pi] = gk[d];
            A.gs[pi] = gs[d];
            A.gc[pi] = gc[d];
            if constexpr (DASH) A.gd[pi] = gd[d];
        }
    }
}

// Terminal adjoint of J = sum_r g_r (1/M_r) sum_i (x_i,x - x0_i,x): lx = g_r / M_r e_x on
// present nodes, lv = 0, gradient sums zero.
__global__ void k_adj_init(const RobotInfo *robots, int total_slots, const int32_t *slot_robot, const float4 *x0,
                           const float *dJ, float4 *lx, float4 *lv, float *gk, float *gs, float *gc, float *gd) {
    const int g = blockIdx.x * blockDim.x + threadIdx.x;
    if (g >= total_slots) return;
    const int r = slot_robot[g];
    const RobotInfo ri = robots[r];
    const bool pres = x0[g].w != 0.f;
    const float val = (pres && ri.M > 0) ? dJ[r] / (float)ri.M : 0.f;
    lx[g] = make_float4(val, 0.f, 0.f, 0.f);
    lv[g] = make_float4(0.f, 0.f, 0.f, 0.f);
    const int s = g - ri.slot_base;
    for (int d = 0; d < NDIR; ++d) {
        const int pi = NDIR * ri.slot_base + d * ri.slots + s;
        gk[pi] = 0.f;
        gs[pi] = 0.f;
        gc[pi] = 0.f;
        if (gd) gd[pi] = 0.f;
    }
}

// Per spring: dJ/dk, dJ/da, dJ/dphi in canonical order, from the stencil sums.
__global__ __launch_bounds__(EACH_THREADS) void k_adj_springs(const RobotInfo *robots, int total_slots,
                                                            const int32_t *slot_robot, SpringIndex ix,
                                                            const int64_t *spring_off, Planes pl, float voxel_len,
                                                            const float *gk, const float *gs, const float *gc,
                                                            float *g_k, float *g_a, float *g_phi) {
    each_spring(robots, total_slots, slot_robot, ix, spring_off, [&](int64_t o, int, int d, int pi, int) {
        const float L0 = voxel_len * sqrtf((float)dir_len2(d));
        const float kL0 = pl.k[pi] * L0, kal = pl.kal[pi], kbe = pl.kbe[pi];
        float a = 0.f, cph = 1.f, sph = 0.f;
        if (kL0 != 0.f) {
            if (kbe == 0.f) a = kal / kL0;
            else {
                a = sqrtf(kal * kal + kbe * kbe) / kL0;
                const float ph = atan2f(kbe, kal);
                cph = cosf(ph);
                sph = sinf(ph);
            }
        }
        if (g_k) g_k[o] = gk[pi];
        if (g_a) g_a[o] = L0 * (gs[pi] * cph + gc[pi] * sph);
        if (g_phi) g_phi[o] = L0 * a * (gc[pi] * cph - gs[pi] * sph);
    });
}

// dJ/dw per voxel through the parallel-sum rule.  Write Z = k a e^{i phi} for a
// spring, so k L(t) = k L0 + L0 (Re Z sin wt + Im Z cos wt): then dJ/dRe Z =
// L0 gs / k, dJ/dIm Z = L0 gc / k and, at fixed Z, dJ/dk = gk - (kal gs + kbe gc) / k^2
// (gk is dJ/dk at fixed a, phi; gs, gc the sums of dJ/dL k sin wt, k cos wt).
// Voxel v adds k_c w to k and k_c w amp e^{i ph} to Z of each of its 28 springs,
// with (amp, ph) = (a_c, phi_c), or (w a_c, w phi_c) under weight-scaled
// actuation, whose w-derivative is k_c a_c (2 w + i w^2 phi_c) e^{i w phi_c};
// and zeta sqrt(2 m k_c w) to the spring's dashpot c, whose w-derivative is
// zeta sqrt(2 m k_c w) / (2 w).
struct DwArgs {
    const RobotInfo *robots;
    int total_vox;
    const int32_t *vox_robot;
    const uint8_t *kept;
    const float *w;
    Planes pl;
    const float *gk, *gs, *gc, *gd;
    float k_class[5], a_class[5], phi_class[5];
    int weight_act;
    float voxel_len;
    float dash_c;  // d c / d w of this voxel's dashpot, up to sqrt(k_c / w): zeta sqrt(2 m) / 2
    float *dJdw;
};

__global__ void k_adj_dw(DwArgs A) {
    const int gv = blockIdx.x * blockDim.x + threadIdx.x;
    if (gv >= A.total_vox) return;
    const int r = A.vox_robot[gv];
    const RobotInfo ri = A.robots[r];
    const int v = gv - ri.vox_base;
    const int c = A.kept[gv];
    if (c == 0) {
        A.dJdw[gv] = 0.f;
        return;
    }
    const int n = ri.n, N = ri.N;
    const int i = v % n, j = (v / n) % n, kk = v / (n * n);
    const float kc = A.k_class[c], ac = A.a_class[c], pc = A.phi_class[c], wv = A.w[gv];
    const float dcdw = (A.gd && wv > 0.f) ? A.dash_c * sqrtf(kc / wv) : 0.f;
    float dzr, dzi;  // d(k_c w amp e^{i ph})/dw
    if (A.weight_act) {
        const float cs = cosf(wv * pc), sn = sinf(wv * pc);
        dzr = kc * ac * (2.f * wv * cs - wv * wv * pc * sn);
        dzi = kc * ac * (2.f * wv * sn + wv * wv * pc * cs);
    } else {
        dzr = kc * ac * cosf(pc);
        dzi = kc * ac * sinf(pc);
    }
    float sum = 0.f;
    for (int c1 = 0; c1 < 8; ++c1) {
        const int a1 = i + (c1 & 1), b1 = j + ((c1 >> 1) & 1), z1 = kk + (c1 >> 2);
        const int l1 = a1 + N * (b1 + N * z1);
        for (int c2 = 0; c2 < 8; ++c2) {
            const int a2 = i + (c2 & 1), b2 = j + ((c2 >> 1) & 1), z2 = kk + (c2 >> 2);
            const int l2 = a2 + N * (b2 + N * z2);
            if (l2 <= l1) continue;
            // forward direction from corner 1 to corner 2
            const int dx = a2 - a1, dy = b2 - b1, dz = z2 - z1;
            int d = -1;
            for (int q = 0; q < NDIR; ++q)
                if (dir_dx(q) == dx && dir_dy(q) == dy && dir_dz(q) == dz) d = q;
            const int pi = NDIR * ri.slot_base + d * ri.slots + l1;
            const float ks = A.pl.k[pi];
            const float L0 = A.voxel_len * sqrtf((float)dir_len2(d));
            const float gs = A.gs[pi], gc = A.gc[pi];
            float t = kc * A.gk[pi];
            if (ks != 0.f) {
                const float ik = 1.f / ks;
                t -= kc * (A.pl.kal[pi] * gs + A.pl.kbe[pi] * gc) * ik * ik;
                t += L0 * ik * (dzr * gs + dzi * gc);
            }
            if (A.gd) t = fmaf(dcdw, A.gd[pi], t);
            sum += t;
        }
    }
    A.dJdw[gv] = sum;
}

// Genome gradient: for each voxel with dJ/dw != 0, recompute the FP32 forward
// (encoding, two tanh layers, sigmoid head), g5 = dJ/dw w (1 - w), then back
// through W3 row 5, W2 and W1.  One workgroup of 8 waves per robot takes tiles
// of 128 voxels: each wave first runs 16 of them through the network and back on
// v_mfma_f32_16x16x4_f32 (whose accumulation is an FMA chain in ascending k, so
// with the bias as the first C this is the scalar loop's arithmetic; layout as
// in the FP32 genome query: register b of lane quarter kq holds feature 4 b + kq
// of voxel `col`), and leaves the encodings, h1 and both layers' deltas in LDS;
// then the waves add the tile's outer products, again as matrix products with
// the voxels as k in ascending order, wave w the row block w / 2 and two column
// blocks of both weight gradients, which stay in registers to the end.  Bias and
// head sums are trees over the 16 voxels of a wave.
// LDS rows of 72 floats: a wave's writes (16 voxels x 4 features) and its
// fragment reads (4 voxels x 16 features) meet each bank at most twice.
// Bound by the tanh and sin/cos (VALU) and the matrix instructions in turn, about
// 17k cycles a tile.  Measured against one thread per voxel quarter with FMA
// loops over LDS, 30 uneven robots: 1274 -> 439 us (the 12^3 robots' 14 tiles in a row).
constexpr int OFF_W1 = 0, OFF_B1 = 4096, OFF_W2 = 4160, OFF_B2 = 8256, OFF_W3 = 8320, OFF_B3 = 8704;
constexpr int MBT = 512, MBV = 16 * (MBT / 64), MROW = 72;

// sum over the 16 lanes of a lane quarter, on every one of them (swaps within a
// quad, across the half row, across the row)
template <int CTRL>
__device__ __forceinline__ float dpp(float v) {
    return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), CTRL, 0xf, 0xf, true));
}
__device__ __forceinline__ float sum16(float v) {
    v += dpp<0xB1>(v);
    v += dpp<0x4E>(v);
    v += dpp<0x141>(v);
    v += dpp<0x140>(v);
    return v;
}

__global__ __launch_bounds__(MBT) void k_mlp_backward(const RobotInfo *robots, const float *genomes, const float *B,
                                                      const float *dJdw, float *g_gen) {
    __shared__ float gamS[MBV * MROW], h1S[MBV * MROW], d1S[MBV * MROW], d2S[MBV * MROW];
    __shared__ float Bs[96], b1s[64], b2s[64], w3s[64];
    const int r = blockIdx.x;
    const RobotInfo ri = robots[r];
    const int n = ri.n, nv = n * n * n;
    const float *g = genomes + (size_t)r * SR_GENOME_LEN;
    float *out = g_gen + (size_t)r * SR_GENOME_LEN;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int col = lane & 15, kq = lane >> 4;
    const int perm = 4 * (col & 3) + (col >> 2);  // weight row of A row `col` within its block
    if (tid < 64) {
        b1s[tid] = g[OFF_B1 + tid];
        b2s[tid] = g[OFF_B2 + tid];
        w3s[tid] = g[OFF_W3 + 5 * 64 + tid];
    }
    if (tid < 96) Bs[tid] = B[tid];
    const float b3 = g[OFF_B3 + 5];
    float w1[4][16];
#pragma unroll
    for (int m = 0; m < 4; ++m)
#pragma unroll
        for (int b = 0; b < 16; ++b) w1[m][b] = g[OFF_W1 + 64 * (16 * m + perm) + 4 * b + kq];
    __syncthreads();
    f32x4 a1[2], a2[2];  // gradient blocks of W1 and W2
#pragma unroll
    for (int e = 0; e < 2; ++e)
#pragma unroll
        for (int i = 0; i < 4; ++i) a1[e][i] = a2[e][i] = 0.f;
    float s1[16], s2[16], s3[16], s5 = 0.f;  // this wave's sums of d1, d2, g5 h2 (feature 4 b + kq) and g5
#pragma unroll
    for (int b = 0; b < 16; ++b) s1[b] = s2[b] = s3[b] = 0.f;
    const int rb = wave >> 1, cb = 2 * (wave & 1);
    const float inv = 1.0f / (float)n;
    for (int v0 = 0; v0 < nv; v0 += MBV) {
        const int vid = v0 + 16 * wave + col, row = (16 * wave + col) * MROW;
        const float dJ = vid < nv ? dJdw[ri.vox_base + vid] : 0.f;
        const bool act = vid < nv && dJ != 0.f;
        if (v0 + 16 * wave < nv) {
            // W2 is read for every tile (from the caches): held in registers beside
            // W1 and the sums it would spill
            int wo = 64 * perm + kq, wt = 64 * kq + perm;
            __asm__ volatile("" : "+v"(wo), "+v"(wt));
            const float *w2 = g + OFF_W2 + wo, *w2t = g + OFF_W2 + wt;
            float h1[16], h2[16];
            {
                const float vx = (((vid % n)) + 0.5f) * inv, vy = (((vid / n) % n) + 0.5f) * inv,
                            vz = ((vid / (n * n)) + 0.5f) * inv;
                float gam[16];
#pragma unroll
                for (int b = 0; b < 8; ++b) {
                    const int q = 4 * b + kq;
                    const float t = 2.0f * fmaf(Bs[3 * q + 2], vz, fmaf(Bs[3 * q + 1], vy, Bs[3 * q] * vx));
                    float sn, cs;
                    sincospif(t, &sn, &cs);
                    gam[b] = act ? cs : 0.f;
                    gam[8 + b] = act ? sn : 0.f;
                }
                f32x4 acc[4];
#pragma unroll
                for (int m = 0; m < 4; ++m)
#pragma unroll
                    for (int i = 0; i < 4; ++i) acc[m][i] = b1s[16 * m + 4 * i + kq];
#pragma unroll
                for (int b = 0; b < 16; ++b) {
                    gamS[row + 4 * b + kq] = gam[b];
#pragma unroll
                    for (int m = 0; m < 4; ++m)
                        acc[m] = __builtin_amdgcn_mfma_f32_16x16x4f32(w1[m][b], gam[b], acc[m], 0, 0, 0);
                }
#pragma unroll
                for (int b = 0; b < 16; ++b) {
                    h1[b] = act ? tanhf(acc[b >> 2][b & 3]) : 0.f;
                    h1S[row + 4 * b + kq] = h1[b];
                }
            }
            {
                f32x4 acc[4];
#pragma unroll
                for (int m = 0; m < 4; ++m)
#pragma unroll
                    for (int i = 0; i < 4; ++i) acc[m][i] = b2s[16 * m + 4 * i + kq];
#pragma unroll
                for (int b = 0; b < 16; ++b)
#pragma unroll
                    for (int m = 0; m < 4; ++m)
                        acc[m] = __builtin_amdgcn_mfma_f32_16x16x4f32(w2[64 * 16 * m + 4 * b], h1[b], acc[m], 0, 0, 0);
#pragma unroll
                for (int b = 0; b < 16; ++b) h2[b] = act ? tanhf(acc[b >> 2][b & 3]) : 0.f;
            }
            f32x4 head;  // row 0: the sigmoid logit
#pragma unroll
            for (int i = 0; i < 4; ++i) head[i] = lane < 16 && i == 0 ? b3 : 0.f;
#pragma unroll
            for (int b = 0; b < 16; ++b)
                head = __builtin_amdgcn_mfma_f32_16x16x4f32(col == 0 ? w3s[4 * b + kq] : 0.f, h2[b], head, 0, 0, 0);
            const float o5 = __shfl(head[0], col, 64);
            const float w = 1.0f / (1.0f + expf(-o5));
            const float g5 = act ? dJ * w * (1.0f - w) : 0.f;
            s5 += sum16(g5);
            f32x4 acc[4];
#pragma unroll
            for (int m = 0; m < 4; ++m)
#pragma unroll
                for (int i = 0; i < 4; ++i) acc[m][i] = 0.f;
            // d2 = g5 w3 (1 - h2^2), d1 = (W2^T d2) (1 - h1^2)
#pragma unroll
            for (int b = 0; b < 16; ++b) {
                const float hh = h2[b];
                const float d2 = g5 * w3s[4 * b + kq] * (1.0f - hh * hh);
                d2S[row + 4 * b + kq] = d2;
#pragma unroll
                for (int m = 0; m < 4; ++m)
                    acc[m] = __builtin_amdgcn_mfma_f32_16x16x4f32(w2t[64 * 4 * b + 16 * m], d2, acc[m], 0, 0, 0);
                s2[b] += sum16(d2);
                s3[b] += sum16(g5 * hh);
            }
#pragma unroll
            for (int b = 0; b < 16; ++b) {
                const float hh = h1[b];
                const float d1 = acc[b >> 2][b & 3] * (1.0f - hh * hh);
                d1S[row + 4 * b + kq] = d1;
                s1[b] += sum16(d1);
            }
        }
        __syncthreads();
        // outer products over the tile's waves that hold voxels; k = voxel
        const int left = (nv - v0 + 15) / 16 * 16, ke = left < MBV ? left : MBV;
        for (int q = 0; q < ke; q += 16)
#pragma unroll
            for (int v = 0; v < 16; v += 4) {
                const int at = (q + v + kq) * MROW + col;
                const float f1 = d1S[at + 16 * rb], f2 = d2S[at + 16 * rb];
#pragma unroll
                for (int e = 0; e < 2; ++e) {
                    a1[e] = __builtin_amdgcn_mfma_f32_16x16x4f32(f1, gamS[at + 16 * (cb + e)], a1[e], 0, 0, 0);
                    a2[e] = __builtin_amdgcn_mfma_f32_16x16x4f32(f2, h1S[at + 16 * (cb + e)], a2[e], 0, 0, 0);
                }
            }
        __syncthreads();
    }
#pragma unroll
    for (int e = 0; e < 2; ++e)
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const int at = 64 * (16 * rb + 4 * kq + i) + 16 * (cb + e) + col;
            out[OFF_W1 + at] = a1[e][i];
            out[OFF_W2 + at] = a2[e][i];
        }
    // the waves' sums, in wave order (the tiles' LDS is free now)
    if (col == 0) {
#pragma unroll
        for (int b = 0; b < 16; ++b) {
            gamS[64 * wave + 4 * b + kq] = s1[b];
            h1S[64 * wave + 4 * b + kq] = s2[b];
            d1S[64 * wave + 4 * b + kq] = s3[b];
        }
        if (kq == 0) d2S[wave] = s5;
    }
    __syncthreads();
    if (tid < 64) {
        float t1 = 0.f, t2 = 0.f, t3 = 0.f;
        for (int q = 0; q < MBT / 64; ++q) {
            t1 += gamS[64 * q + tid];
            t2 += h1S[64 * q + tid];
            t3 += d1S[64 * q + tid];
        }
        out[OFF_B1 + tid] = t1;
        out[OFF_B2 + tid] = t2;
        for (int q = 0; q < 6; ++q) out[OFF_W3 + q * 64 + tid] = q == 5 ? t3 : 0.f;
    }
    if (tid < 5) out[OFF_B3 + tid] = 0.f;  // class logits carry no gradient
    if (tid == 64) {
        float t5 = 0.f;
        for (int q = 0; q < MBT / 64; ++q) t5 += d2S[q];
        out[OFF_B3 + 5] = t5;
    }
}

typedef void (*AdjFn)(AArgs);
constexpr int GRAD_TILE = 256;
struct AdjEntry {
    int n, block;
    AdjFn fn, fn_phase;
    // split form: fn is the reverse step without gradient sums, gt (or null) the
    // gradient pass in tiles of GRAD_TILE slots, and g0 (or null: gt) the one
    // beside a reversal, gblock threads per workgroup on a grid of robots x gy
    AdjFn gt = nullptr, gt_phase = nullptr;
    int gblock = 0;
    AdjFn g0 = nullptr, g0_phase = nullptr;
    int gy = 1;
    // Tiles beside a reversal of few robots: up to this many rounds of tiles by
    // 128 workgroups end before the reversal does, and the other half of the CUs
    // is there when its next launch comes.  1200 steps backward, all tiles at
    // once / 128 workgroups: 12^3, 64 robots 16.7 / 15.0 ms, 128 (9 rounds) with
    // dashpots 45.4 / 39.0, 192 57.6 / 69.0; 11^3 with dashpots, 64 (4 rounds)
    // 20.7 / 19.2, 96 (6) 24.1 / 27.3.
    int rounds = 0;
};
#define SR_AE(NN, BS, X) \
    { NN, BS, k_adjoint<NN + 1, BS, false, X>, k_adjoint<NN + 1, BS, true, X> }
#define SR_AEL(NN, BS, LG) \
    { NN, BS, k_adjoint<NN + 1, BS, false, true, LG>, k_adjoint<NN + 1, BS, true, true, LG> }
#define SR_GT(NN, DASH) \
    k_adj_grad_tiles<NN + 1, GRAD_TILE, false, DASH>, k_adj_grad_tiles<NN + 1, GRAD_TILE, true, DASH>
// split exchange form with a one-launch gradient pass
#define SR_AESL(NN, BS, LG, GBS)                                                                                \
    {                                                                                                          \
        NN, BS, k_adjoint<NN + 1, BS, false, true, LG, false, false, false, true>,                              \
            k_adjoint<NN + 1, BS, true, true, LG, false, false, false, true>, SR_GT(NN, false), GBS,             \
            k_adj_grad<NN + 1, GBS, false, 1>, k_adj_grad<NN + 1, GBS, true, 1>                                  \
    }
// split exchange form in XC direction chunks (one chunk's rows in LDS at a
// time), parameters per chunk with GP; SR_AESCG: the gradient pass beside a
// reversal in GY workgroups per robot
#define SR_AESC_(NN, BS, LG, XC, GP)                                                                           \
    NN, BS, k_adjoint<NN + 1, BS, false, true, LG, false, false, false, true, XC, GP>,                          \
        k_adjoint<NN + 1, BS, true, true, LG, false, false, false, true, XC, GP>, SR_GT(NN, false)
#define SR_AESC(NN, BS, LG, XC, GP, ROUNDS) \
    { SR_AESC_(NN, BS, LG, XC, GP), 0, nullptr, nullptr, 1, ROUNDS }
#define SR_AESCG(NN, BS, LG, XC, GP, GBS, GY)                                                                  \
    {                                                                                                          \
        SR_AESC_(NN, BS, LG, XC, GP), GBS, k_adj_grad<NN + 1, GBS, false, GY>,                                  \
            k_adj_grad<NN + 1, GBS, true, GY>, GY                                                               \
    }
const AdjEntry kAdj[] = {SR_AE(1, 64, true),    SR_AE(2, 64, true),    SR_AE(3, 64, true),   SR_AEL(4, 128, 2),
                         SR_AEL(5, 256, 2),     SR_AEL(6, 384, 2),     SR_AEL(7, 512, 2),    SR_AESL(8, 768, 2, 768),
                         SR_AESCG(9, 1024, 2, 2, false, 1024, 1), SR_AESCG(10, 768, 2, 3, false, 704, 2),
                         SR_AESCG(11, 1024, 0, 4, false, 1024, 2), SR_AESC(12, 768, 0, 7, true, 9)};
// spring dashpots or the damped ground (Table II model): the one-buffer
// recompute form with the velocity terms
#define SR_AED(NN, BS) \
    { NN, BS, k_adjoint<NN + 1, BS, false, false, 0, true, true>, k_adjoint<NN + 1, BS, true, false, 0, true, true> }
// the exchange form with the velocity terms: four rows per direction (K_s u and
// the scalar of the upper end's velocity-adjoint term), XC direction chunks
#define SR_AEDX(NN, BS, XC)                                                                                    \
    {                                                                                                          \
        NN, BS, k_adjoint<NN + 1, BS, false, true, 0, false, true, false, false, XC>,                           \
            k_adjoint<NN + 1, BS, true, true, 0, false, true, false, false, XC>                                 \
    }
// split form of the above: the reverse recursion alone, then the gradient
// pass with the dashpot terms
#define SR_AEDS_(NN, BS, XC, GP, ...)                                                                          \
    NN, BS, k_adjoint<NN + 1, BS, false, true, 0, false, true, false, true, XC, GP>,                            \
        k_adjoint<NN + 1, BS, true, true, 0, false, true, false, true, XC, GP>, __VA_ARGS__
#define SR_AEDS(NN, BS, XC, GP, ROUNDS) \
    { SR_AEDS_(NN, BS, XC, GP, SR_GT(NN, true)), 0, nullptr, nullptr, 1, ROUNDS }
// last: SR_GT, or two nulls where the pass in GY workgroups is never slower
#define SR_AEDSG(NN, BS, XC, GP, GBS, GY, ...)                                                                 \
    {                                                                                                          \
        SR_AEDS_(NN, BS, XC, GP, __VA_ARGS__), GBS, k_adj_grad<NN + 1, GBS, false, GY, true>,                                \
            k_adj_grad<NN + 1, GBS, true, GY, true>, GY                                                         \
    }
const AdjEntry kAdjD[] = {SR_AED(1, 64),        SR_AED(2, 64),        SR_AED(3, 64),        SR_AEDX(4, 128, 1),
                          SR_AEDX(5, 256, 1),   SR_AEDX(6, 384, 1),   SR_AEDX(7, 512, 1),
                          SR_AEDSG(8, 768, 2, false, 768, 2, nullptr, nullptr),
                          SR_AEDSG(9, 1024, 3, false, 1024, 2, SR_GT(9, true)),
                          SR_AEDSG(10, 768, 5, true, 768, 2, SR_GT(10, true)), SR_AEDS(11, 1024, 7, true, 5),
                          SR_AEDS(12, 768, 13, true, 9)};

}  // namespace

bool adjoint_is_split(int n, bool vel) {
    for (const auto &q : (vel ? kAdjD : kAdj))
        if (q.n == n) return q.gt || q.g0;
    return false;
}

hipError_t launch_adjoint(int n, bool phase, const RobotInfo *robots, const int32_t *list, int count, Planes pl,
                          const float4 *x0, const float4 *rec_x, const float4 *rec_v, const float4 *rec_u,
                          float4 *rec_l, int n_steps, int rec_steps, const float2 *sc, float4 *lx, float4 *lv,
                          float *gk, float *gs, float *gc, float *gd, SimConst c, hipStream_t st) {
    const bool vel = c.dash || c.gdamp;  // forces that depend on the velocities
    if (vel && (!rec_u || !gd)) return hipErrorInvalidValue;
    const AdjEntry *e = nullptr;
    for (const auto &q : (vel ? kAdjD : kAdj))
        if (q.n == n) e = &q;
    if (!e) return hipErrorInvalidConfiguration;
    AArgs A;
    A.robots = robots;
    A.list = list;
    A.count = count;
    A.pl = pl;
    A.x0 = x0;
    A.rec_x = rec_x;
    A.rec_v = rec_v;
    A.rec_u = rec_u;
    A.rec_l = rec_l;
    A.n_steps = n_steps;
    A.rec_steps = rec_steps;
    A.sc = sc;
    A.lx = lx;
    A.lv = lv;
    A.gk = gk;
    A.gs = gs;
    A.gc = gc;
    A.gd = gd;
    A.c = c;
    if ((e->gt || e->g0) && !rec_l) return hipErrorInvalidValue;
    hipLaunchKernelGGL(phase ? e->fn_phase : e->fn, dim3(count), dim3(e->block), 0, st, A);
    return hipGetLastError();
}

hipError_t launch_adj_grad(int n, bool phase, const RobotInfo *robots, const int32_t *list, int count, Planes pl,
                           const float4 *x0, const float4 *rec_x, const float4 *rec_u, float4 *rec_l, int n_steps,
                           int rec_steps, const float2 *sc, float *gk, float *gs, float *gc, float *gd, SimConst c,
                           bool beside, bool room, hipStream_t st) {
    const bool vel = c.dash || c.gdamp;
    if (vel && (!rec_u || !gd)) return hipErrorInvalidValue;
    const AdjEntry *e = nullptr;
    for (const auto &q : (vel ? kAdjD : kAdj))
        if (q.n == n) e = &q;
    if (!e || !(e->gt || e->g0) || !rec_l) return hipErrorInvalidValue;
    AArgs A = {};
    A.robots = robots;
    A.list = list;
    A.count = count;
    A.pl = pl;
    A.x0 = x0;
    A.rec_x = rec_x;
    A.rec_u = rec_u;
    A.rec_l = rec_l;
    A.n_steps = n_steps;
    A.rec_steps = rec_steps;
    A.sc = sc;
    A.gk = gk;
    A.gs = gs;
    A.gc = gc;
    A.gd = gd;
    A.c = c;
    if (e->g0 && (beside || !e->gt)) {
        hipLaunchKernelGGL(phase ? e->g0_phase : e->g0, dim3(count, e->gy), dim3(e->gblock), 0, st, A);
    } else {
        const int slots = (n + 1) * (n + 1) * (n + 1), tiles = (slots + GRAD_TILE - 1) / GRAD_TILE;
        const int all = (count + 7) / 8 * 8 * tiles;
        const bool half = beside && room && (all + 127) / 128 <= e->rounds;
        const int grid = half && all > 128 ? 128 : all;
        hipLaunchKernelGGL(phase ? e->gt_phase : e->gt, dim3(grid), dim3(GRAD_TILE), 0, st, A);
    }
    return hipGetLastError();
}

hipError_t launch_adj_init(const RobotInfo *robots, int total_slots, const int32_t *slot_robot, const float4 *x0,
                           const float *dJ, float4 *lx, float4 *lv, float *gk, float *gs, float *gc, float *gd,
                           hipStream_t st) {
    hipLaunchKernelGGL(k_adj_init, dim3((total_slots + 255) / 256), dim3(256), 0, st, robots, total_slots, slot_robot,
                       x0, dJ, lx, lv, gk, gs, gc, gd);
    return hipGetLastError();
}

hipError_t launch_adj_springs(const RobotInfo *robots, int total_slots, const int32_t *slot_robot, SpringIndex ix,
                              const int64_t *spring_off, Planes pl, float voxel_len, const float *gk, const float *gs,
                              const float *gc, float *g_k, float *g_a, float *g_phi, hipStream_t st) {
    if (!g_k && !g_a && !g_phi) return hipSuccess;
    hipLaunchKernelGGL(k_adj_springs, dim3((total_slots + EACH_SLOTS - 1) / EACH_SLOTS), dim3(EACH_THREADS), 0, st,
                       robots, total_slots, slot_robot, ix, spring_off, pl, voxel_len, gk, gs, gc, g_k, g_a, g_phi);
    return hipGetLastError();
}

hipError_t launch_adj_genome(const RobotInfo *robots, int R, int total_vox, const int32_t *vox_robot,
                             const uint8_t *kept, const float *w, Planes pl, const float *gk, const float *gs,
                             const float *gc, const float *gd, const sr_sim_params &p, const float *genomes,
                             const float *B, float *dJdw, float *g_gen, hipStream_t st) {
    DwArgs A;
    A.robots = robots;
    A.total_vox = total_vox;
    A.vox_robot = vox_robot;
    A.kept = kept;
    A.w = w;
    A.pl = pl;
    A.gk = gk;
    A.gs = gs;
    A.gc = gc;
    A.gd = p.zeta_spring != 0.f ? gd : nullptr;
    A.dash_c = (float)(0.5 * (double)p.zeta_spring * sqrt(2.0 * (double)p.mass));
    for (int c = 0; c < 5; ++c) {
        A.k_class[c] = p.k_class[c];
        A.a_class[c] = p.a_class[c];
        A.phi_class[c] = p.phi_class[c];
    }
    A.weight_act = (p.flags & SR_WEIGHT_ACTUATION) != 0;
    A.voxel_len = p.voxel_len;
    A.dJdw = dJdw;
    hipLaunchKernelGGL(k_adj_dw, dim3((total_vox + 255) / 256), dim3(256), 0, st, A);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(k_mlp_backward, dim3(R), dim3(MBT), 0, st, robots, genomes, B, dJdw, g_gen);
    return hipGetLastError();
}

}  // namespace sr

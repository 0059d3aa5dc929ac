// es_flux.hpp -- the per-node and per-interface pieces of the ES flux
// (Sections 3.1-3.4) shared by the direction-sweep kernels of es_rhs.hip and
// the batched stage kernel of es_batch.hip.  Node quantities live in an LDS
// tile (NodeTile); the functions read them by tile index.
#pragma once
#include "es_kernels.hpp"

namespace es {

// R is the precision of the interface arithmetic.  The FP64 tile keeps the
// species entropy variables y_l (formed once per node, read by up to 18
// interface stencils of it); the FP32 one forms them per interface from the
// FP64 node logs.
template <int N, int D, int NN, typename R = double>
struct NodeTile {
    double rho[N][NN];     // species densities
    double lrho[N][NN];    // their logs
    double lrt[N == 2 ? NN : 1];  // log of the total density (N = 2)
    double v[D][NN];       // velocity
    double b[NN];          // beta = 1/T
    double lb[NN];         // log beta
    float ay[NN];          // sum_l |y_l| (species entropy variables), and
    float av[NN];          // beta |v|_1: row magnitudes for the sign test's zero tolerance
    double m[D + 1][NN];   // half the metrics of direction k: n_t/2, n_1/2..n_D/2 (an
                           // interface average is then one sum; halving is exact)
};

template <int N, int D, int NN>
struct NodeTile<N, D, NN, double> {
    double rho[N][NN];
    double lrho[N][NN];
    double v[D][NN];
    double b[NN];
    double lb[NN];
    double y[N][NN];       // y_l = c_vl ln beta + R_l ln rho_l + c_vl Gamma_l - beta |v|^2 / 2
    double m[D + 1][NN];
};

// mixture Gamma, gas constant and pressure of tile node q (N = 2)
template <int N, int D, int NN, typename R>
__device__ __forceinline__ void mixture(const Phys& ph, const NodeTile<N, D, NN, R>& S, int q,
                                        double& gm, double& rm, double& p)
{
    const double r0 = S.rho[0][q], r1 = S.rho[1][q];
    const double cvr = ph.cv[0] * r0 + ph.cv[1] * r1;
    const double rR = ph.Rg[0] * r0 + ph.Rg[1] * r1;
    gm = (ph.cvgam[0] * r0 + ph.cvgam[1] * r1) * rcp(cvr);
    rm = rR * rcp(r0 + r1);
    p = rR * rcp(S.b[q]) - ph.pinf_tot;
}

// two-point EC flux between tile nodes ia, ib (eq ECfluxMM), written in the
// direction-generic form n_t Utilde + sum_j n_j Ftilde_j:
//   M_l = {rho_l}^ln ({v}.n + n_t),  p^ = Pi - p_inf with Pi = sum R_l {rho_l} / {beta},
//   momentum = {v} sum M_l + p^ n,
//   energy = sum M_l (c_vl/{beta}^ln - {|v|^2}/2) + |{v}|^2 sum M_l + Pi {v}.n + p_inf n_t,
// with {|v|^2} the mean of squares.  The energy line is {v}.momentum +
// p_inf ({v}.n + n_t) with the two p_inf {v}.n terms cancelled by hand, and
// Pi is formed in FP64 in both precisions: with a stiffened gas Pi and
// p_inf are both ~p_inf, so neither difference may be left to FP32.
// (M: the halved metrics of the direction, indexed like the tile)
template <int N, int D, int NN, typename R>
__device__ __forceinline__ void ec_pair(const Phys& ph, const NodeTile<N, D, NN, R>& S, const double (*M)[NN],
                                        int ia, int ib, R* F)
{
    constexpr int NC = N + D + 1;
    const R nt = R(M[0][ia]) + R(M[0][ib]);
    R n[D], vm[D];
    R vdn = R(0), v2 = R(0);
#pragma unroll
    for (int j = 0; j < D; j++) {
        n[j] = R(M[1 + j][ia]) + R(M[1 + j][ib]);
        const R va = R(S.v[j][ia]), vb = R(S.v[j][ib]);
        vm[j] = R(0.5) * (va + vb);
        v2 += va * va + vb * vb;
        vdn += vm[j] * n[j];
    }
    v2 *= R(0.5);
    const R vn = vdn + nt;
    const R ibln = R(inv_logmean(S.b[ia], S.b[ib], S.lb[ia], S.lb[ib]));
    double Rr = 0.0;
#pragma unroll
    for (int l = 0; l < N; l++) Rr += ph.Rg[l] * (S.rho[l][ia] + S.rho[l][ib]);
    const double Pi = Rr * rcp(S.b[ia] + S.b[ib]);
    const R phat = R(Pi - ph.pinf_tot);
    R Mt = R(0), eng = R(0);
#pragma unroll
    for (int l = 0; l < N; l++) {
        const R rln = R(logmean(S.rho[l][ia], S.rho[l][ib], S.lrho[l][ia], S.lrho[l][ib]));
        const R Ml = rln * vn;
        F[l] = Ml;
        Mt += Ml;
        eng += Ml * (R(ph.cv[l]) * ibln - R(0.5) * v2);
    }
    R vv = R(0);
#pragma unroll
    for (int j = 0; j < D; j++) {
        F[N + j] = vm[j] * Mt + phat * n[j];
        vv += vm[j] * vm[j];
    }
    F[NC - 1] = eng + vv * Mt + R(Pi) * vdn + R(ph.pinf_tot) * nt;
}

// (ec_pair and dissipation serve the FP32 interface arithmetic of the mixed
// form; the FP64 sweeps take pair_means, ec_flux64 and dissipation64 below)
//
// ES dissipation 1/2 s T^T R Y [[W]]^WENO at the interface between tile
// nodes iL (= i) and iR (= i+1); st[t] are the tile indices of nodes
// i-2..i+3.  Interface metrics, averages and R follow Section 3.4.  MG: the
// acoustic and species fields in one group or two.
template <int N, int D, int NN, typename R, int MG>
__device__ __forceinline__ void dissipation(const Phys& ph, const NodeTile<N, D, NN, R>& S, const double (*M)[NN],
                                            const int st[6], const Weno<R>& Wc, R* Dout)
{
    constexpr int NC = N + D + 1;
    const int iL = st[2], iR = st[3];
    // interface metric: mean of the two nodes
    R n[D];
    const R nt = R(M[0][iL]) + R(M[0][iR]);
    R nn2 = R(0);
#pragma unroll
    for (int j = 0; j < D; j++) {
        n[j] = R(M[1 + j][iL]) + R(M[1 + j][iR]);
        nn2 += n[j] * n[j];
    }
    const bool nz = nn2 > R(0);
    const R inn = nz ? rsqrt_pos(nn2) : R(0);
    const R nn = nn2 * inn;
    Rot<D, R> T;
    make_rot<D, R>(n, inn, nz, T);
    // averaged state
    R vbar[D];
    R vn = R(0);
#pragma unroll
    for (int j = 0; j < D; j++) {
        vbar[j] = R(0.5) * (R(S.v[j][iL]) + R(S.v[j][iR]));
        vn += vbar[j] * n[j];
    }
    Frame<N, D, R> F;
    rot_apply<D, R>(T, vbar, F.vh);
    R vv = R(0);
#pragma unroll
    for (int j = 0; j < D; j++) vv += F.vh[j] * F.vh[j];
    F.K = R(0.5) * vv;
    const R Tbar = R(inv_logmean(S.b[iL], S.b[iR], S.lb[iL], S.lb[iR]));   // 1/{beta}^ln
    if constexpr (N == 1) {
        const R G = R(ph.gam[0]), Rg = R(ph.Rg[0]), cv = R(ph.cv[0]);
        const R rho = R(logmean(S.rho[0][iL], S.rho[0][iR], S.lrho[0][iL], S.lrho[0][iR]));
        F.c = sqrt_pos(G * Rg * Tbar);
        F.H = G * cv * Tbar + F.K;
        F.sa = sqrt_pos(rho * rcp(R(2) * G * Rg));
        F.se = sqrt_pos(rho * rcp(cv * G));
        F.st = sqrt_pos(rho * Tbar);
    } else {
        R rl[2];
        double gmL, gmR, rmL, rmR, pL, pR;
        mixture<N, D, NN, R>(ph, S, iL, gmL, rmL, pL);
        mixture<N, D, NN, R>(ph, S, iR, gmR, rmR, pR);
        const R Rm[2] = {R(rmL), R(rmR)};
        const R Gm[2] = {R(gmL), R(gmR)};
#pragma unroll
        for (int l = 0; l < 2; l++)
            rl[l] = R(logmean(S.rho[l][iL], S.rho[l][iR], S.lrho[l][iL], S.lrho[l][iR]));
        const double rL = S.rho[0][iL] + S.rho[1][iL], rR = S.rho[0][iR] + S.rho[1][iR];
        const R rho = R(logmean(rL, rR, S.lrt[iL], S.lrt[iR]));
        const R Rb = R(0.5) * (Rm[0] + Rm[1]);
        const R Gb = R(0.5) * (Gm[0] + Gm[1]);
        const R irho = rcp(rho);
        R rhoh = R(0.5) * (R(pL) + R(pR));
#pragma unroll
        for (int l = 0; l < 2; l++) rhoh += R(ph.cv[l]) * rl[l] * Tbar + R(ph.pinf[l]);
        F.H = rhoh * irho + F.K;
        F.Y[0] = rl[0] * irho;
        F.Y[1] = rl[1] * irho;
        const R igm1 = rcp(Gb - R(1));
#pragma unroll
        for (int l = 0; l < 2; l++)
            F.e2[l] = F.K - (R(ph.cv[l]) + R(ph.Rg[l]) - Gb * R(ph.cv[l])) * Tbar * igm1;
        F.c = sqrt_pos(Gb * Rb * Tbar);
        F.sq = sqrt_pos(rho * rcp(Gb * Rb));
        F.s2a = F.sq * R(0.70710678118654752440);
        const R yy = sqrt_pos(F.Y[0] * F.Y[1]);
        const R sg = sqrt_pos(Gb - R(1));
        const R syg = F.sq * yy * sqrt_pos(Gb);
        F.d11 = -syg * R(ph.sr21);
        F.d12 = F.sq * F.Y[0] * sg;
        F.d21 = syg * R(ph.isr21);
        F.d22 = F.sq * F.Y[1] * sg;
    }
    const R s = fabs(nt + vn) + nn * F.c;

    // scaled entropy variables W_j = R^T T V(U_j) of the stencil nodes
    // j = i-2..i+3, one group of characteristic fields at a time (the
    // tangential fields, then the acoustic and species fields, these two in
    // separate groups when MG = 2), each group's MR-WENO jumps taken as soon
    // as its stencil values exist.  The acoustic
    // and species fields see the rotated momentum variables only through
    // (T vbar).(T b v) = b vbar.v and the normal row of T v.
    R Z[NC];
    // MR-WENO on one scaled characteristic field, sign matrix Y: the WENO
    // jump and the jump agree in sign, and the jump is not zero to working
    // precision, i.e. above zero_tol times mag, a bound on the size of the
    // terms that make W_i and W_{i+1}: max_l |R_lc| sum_l |y_l| over the
    // species rows, plus sum_e |R_ec| a_e with a_e = beta |v|_1 (>= every
    // rotated |y_{N+j}|) for the momentum rows and beta for the energy row,
    // all summed over nodes i and i+1.  Across a contact the acoustic jumps vanish up to rounding, in an
    // isentropic flow the entropy field's do; those count as sign 0.
    auto weno_field = [&](const R (&w)[6], R mag) -> R {
        R jump;
        const R jw = mr5_jump<R>(w[0], w[1], w[2], w[3], w[4], w[5], Wc, jump);
        const bool y = (jw * jump > R(0)) && (fabs(jump) > Wc.zero_tol * mag);
        return y ? jw : R(0);
    };
    // row magnitudes of nodes i and i+1, summed (the node part of the zero
    // tolerance, kept per node in the tile): ay = sum_l |y_l|, av = beta
    // |v|_1, aE = beta
    auto node_scales = [&](R& ay, R& av, R& aE) {
        ay = R(S.ay[iL]) + R(S.ay[iR]);
        av = R(S.av[iL]) + R(S.av[iR]);
        aE = R(fabs(S.b[iL]) + fabs(S.b[iR]));
    };
    asm volatile("" ::: "memory");
    {
        R Wt[D - 1][6];
        const R sct = (N == 1) ? F.st : F.sq * F.c;   // scale of the tangential columns
#pragma unroll
        for (int t = 0; t < 6; t++) {
            const int q = st[t];
            const R bq = R(S.b[q]);
            R vq[D], vr[D];
#pragma unroll
            for (int j = 0; j < D; j++) vq[j] = R(S.v[j][q]);
            rot_apply<D, R>(T, vq, vr);
            R yt[D - 1];
#pragma unroll
            for (int j = 1; j < D; j++) yt[j - 1] = bq * vr[j];
            R wt[D - 1];
            frame_project_tan<N, D, R>(F, yt, -bq, wt);
#pragma unroll
            for (int j = 0; j < D - 1; j++) Wt[j][t] = wt[j];
        }
        R ay, av, aE;
        node_scales(ay, av, aE);
        R mt[D - 1];
        bool need = false;
#pragma unroll
        for (int j = 0; j < D - 1; j++) {
            mt[j] = sct * (av + fabs(F.vh[j + 1]) * aE);
            need = need || fabs(Wt[j][3] - Wt[j][2]) > Wc.zero_tol * mt[j];
        }
        // where no lane of the wave has a jump above the tolerance, every
        // field of the group has Y = 0 and its WENO jump is not needed (the
        // same for the second group)
        if (__any(need)) {
#pragma unroll
            for (int j = 0; j < D - 1; j++) Z[N + 1 + j] = weno_field(Wt[j], mt[j]);
        } else {
#pragma unroll
            for (int j = 0; j < D - 1; j++) Z[N + 1 + j] = R(0);
        }
    }
    // the acoustic and species (entropy) fields, as one group or (MG = 2)
    // two, the acoustic fields and then the species fields, each reloading
    // its node values from LDS rather than keeping the previous group's loads
    // live across its WENO: fewer registers for more loads
    {
        constexpr int NM = N + 2;                  // main fields 0..N and NC - 1
        constexpr int NGRP = MG;
        R mg[NM];
        {
            R ay, av, aE;
            node_scales(ay, av, aE);
            frame_scale_main<N, D, R>(F, ay, av, aE, mg);
        }
#pragma unroll
        for (int grp = 0; grp < NGRP; grp++) {
            asm volatile("" ::: "memory");
            // main field of the c-th member of this group, and its slot in Z
            const int nf = NGRP == 1 ? NM : (grp == 0 ? 2 : NM - 2);
            auto mfield = [&](int c) { return NGRP == 1 ? c : (grp == 0 ? (c == 0 ? 0 : NM - 1) : 1 + c); };
            auto zslot = [&](int m) { return m <= N ? m : NC - 1; };
            R Wg[NM][6];
#pragma unroll
            for (int t = 0; t < 6; t++) {
                const int q = st[t];
                const R bq = R(S.b[q]);
                R vq[D], vr[D];
                R v2 = R(0), vbv = R(0);
#pragma unroll
                for (int j = 0; j < D; j++) {
                    vq[j] = R(S.v[j][q]);
                    v2 += vq[j] * vq[j];
                    vbv += vbar[j] * vq[j];
                }
                R ys[N];
                const double lbq = S.lb[q];
#pragma unroll
                for (int l = 0; l < N; l++)
                    ys[l] = R(ph.cv[l] * lbq + ph.Rg[l] * S.lrho[l][q] + ph.cvgam[l]) - R(0.5) * bq * v2;
                rot_apply<D, R>(T, vq, vr);
                R wm[NM];
                frame_project_main<N, D, R>(F, ys, bq * vr[0], bq * vbv, -bq, wm);
#pragma unroll
                for (int c = 0; c < NM; c++)
                    if (c < nf) Wg[c][t] = wm[mfield(c)];
            }
            bool need = false;
#pragma unroll
            for (int c = 0; c < NM; c++)
                if (c < nf) need = need || fabs(Wg[c][3] - Wg[c][2]) > Wc.zero_tol * mg[mfield(c)];
            if (__any(need)) {
#pragma unroll
                for (int c = 0; c < NM; c++)
                    if (c < nf) Z[zslot(mfield(c))] = weno_field(Wg[c], mg[mfield(c)]);
            } else {
#pragma unroll
                for (int c = 0; c < NM; c++)
                    if (c < nf) Z[zslot(mfield(c))] = R(0);
            }
        }
    }
    R RZ[NC];
    frame_expand<N, D, R>(F, Z, RZ);
    const R hs = R(0.5) * s;
#pragma unroll
    for (int l = 0; l < N; l++) Dout[l] = hs * RZ[l];
    R mv[D], mo[D];
#pragma unroll
    for (int j = 0; j < D; j++) mv[j] = RZ[N + j];
    rot_apply_t<D, R>(T, mv, mo);
#pragma unroll
    for (int j = 0; j < D; j++) Dout[N + j] = hs * mo[j];
    Dout[NC - 1] = hs * RZ[NC - 1];
}

// ---------------------------------------------------------------------------
// FP64 interface arithmetic.  The sweeps issue FP64 instructions for most of
// their time, so the formulas of ec_pair and dissipation above are arranged
// here for the fewest of them (the frame, the sign matrix and its tolerance,
// the reconstruction and the fluxes are the same):
//   - every multiply-add is one instruction;
//   - the reciprocals of a pair are taken two at a time over their product;
//   - F(l, l+1) and the dissipation share their logarithmic means;
//   - W_m of a stencil node is a dot product with the scaled column of R,
//     folded into interface constants: with t = vbar.v,
//       acoustic  c0 y_0 + c1 y_1 + beta (cv.v - cH) -+ beta (cn.v - ck),
//       species   d1 y_0 + d2 y_1 + beta ((d1 + d2) t - ce),
//       tangential  beta (ct.v - ck);
//   - the two middle nodes' W decide whether the wave needs the other four
//     and the reconstruction, and before the frame is formed the entropy
//     variables of the two nodes decide whether the wave has any dissipation.
// Each node's W goes through one instruction sequence, so identical states
// give identical W.
// ---------------------------------------------------------------------------

// makes the compiler form x here: it otherwise sinks sums to their last use
// and holds every operand of them in registers until then
__device__ __forceinline__ void form_here(double& x) { asm volatile("" : "+v"(x)); }

// logarithmic means of a node pair: of the species densities and the inverse
// of that of beta
template <int N>
struct PairMeans {
    double rho[N], ib;
};

// x / atanh(x) and atanh(x) / x from u = x^2 < 1e-4 (the series of logmean
// and inv_logmean)
__device__ __forceinline__ double lm_series(double u)
{
    return fma(-u, fma(u, fma(u, 44.0 / 945.0, 4.0 / 45.0), 1.0 / 3.0), 1.0);
}
__device__ __forceinline__ double ilm_series(double u)
{
    return fma(u, fma(u, fma(u, 1.0 / 7.0, 1.0 / 5.0), 1.0 / 3.0), 1.0);
}

template <int N, int D, int NN>
__device__ __forceinline__ void pair_means(const NodeTile<N, D, NN, double>& S, int ia, int ib,
                                           PairMeans<N>& pm, double& isb)
{
    double d[N], s[N];
    bool ser[N];
    bool any = false;
#pragma unroll
    for (int l = 0; l < N; l++) {
        const double ra = S.rho[l][ia], rb = S.rho[l][ib];
        d[l] = ra - rb;
        s[l] = ra + rb;
        ser[l] = d[l] * d[l] < 1.0e-4 * (s[l] * s[l]);
        any = any || !ser[l];
    }
    const double ba = S.b[ia], bb = S.b[ib];
    const double db = ba - bb, sb = ba + bb;
    const bool serb = db * db < 1.0e-4 * (sb * sb);
    any = any || !serb;
    if (!__any(any)) {   // the whole wave on the series
        isb = rcp64(sb);
        const double f = db * isb;
        pm.ib = 2.0 * isb * ilm_series(f * f);
        double is[N];
        if constexpr (N == 2) {
            const double r = rcp64(s[0] * s[1]);
            is[0] = r * s[1];
            is[1] = r * s[0];
        } else {
            is[0] = rcp64(s[0]);
        }
#pragma unroll
        for (int l = 0; l < N; l++) {
            const double x = d[l] * is[l];
            pm.rho[l] = 0.5 * s[l] * lm_series(x * x);
        }
    } else {             // lane by lane, the divisor selected
        const double e = serb ? 1.0 : db;
        const double rb = rcp64(sb * e);
        isb = rb * e;
        const double f = db * isb;
        const double ibs = 2.0 * isb * ilm_series(f * f);
        const double ibl = (S.lb[ia] - S.lb[ib]) * (rb * sb);
        pm.ib = serb ? ibs : ibl;
        double q[N], iq[N];
#pragma unroll
        for (int l = 0; l < N; l++) q[l] = ser[l] ? s[l] : S.lrho[l][ia] - S.lrho[l][ib];
        if constexpr (N == 2) {
            const double r = rcp64(q[0] * q[1]);
            iq[0] = r * q[1];
            iq[1] = r * q[0];
        } else {
            iq[0] = rcp64(q[0]);
        }
#pragma unroll
        for (int l = 0; l < N; l++) {
            const double x = d[l] * iq[l];
            const double xs = 0.5 * s[l] * lm_series(x * x);
            pm.rho[l] = ser[l] ? xs : x;
        }
    }
}

// logarithmic mean of two positive values without node logs: off the series
// ln(a/b) is taken of the quotient (one logarithm where a lane needs it)
__device__ __forceinline__ double logmean64(double a, double b)
{
    const double d = a - b, s = a + b;
    const double f = d * rcp64(s), u = f * f;
    double r = 0.5 * s * lm_series(u);
    if (!(d * d < 1.0e-4 * (s * s))) r = d * rcp64(ln_pos(a * rcp64(b)));
    return r;
}

// the two-point flux of ec_pair from the pair's means; vs = v_a + v_b and
// n, nt are returned for the dissipation
template <int N, int D, int NN>
__device__ __forceinline__ void ec_flux64(const Phys& ph, const NodeTile<N, D, NN, double>& S,
                                          const double (*M)[NN], int ia, int ib, const PairMeans<N>& pm,
                                          double isb, double* F)
{
    constexpr int NC = N + D + 1;
    const double nt = M[0][ia] + M[0][ib];
    double n[D], vs[D];
    double w = 0.0, s2 = 0.0, vv = 0.0;   // 2 {v}.n, sum of squares, 4 |{v}|^2
#pragma unroll
    for (int j = 0; j < D; j++) {
        n[j] = M[1 + j][ia] + M[1 + j][ib];
        const double va = S.v[j][ia], vb = S.v[j][ib];
        vs[j] = va + vb;
        s2 = fma(va, va, fma(vb, vb, s2));
        w = fma(vs[j], n[j], w);
        vv = fma(vs[j], vs[j], vv);
    }
    const double vn = fma(0.5, w, nt);
    double Rr = ph.Rg[0] * (S.rho[0][ia] + S.rho[0][ib]);
    if constexpr (N == 2) Rr = fma(ph.Rg[1], S.rho[1][ia] + S.rho[1][ib], Rr);
    const double Pi = Rr * isb;
    const double phat = Pi - ph.pinf_tot;
    double Mt = 0.0, ce = 0.0;
#pragma unroll
    for (int l = 0; l < N; l++) {
        F[l] = pm.rho[l] * vn;
        Mt += F[l];
        ce = l == 0 ? ph.cv[0] * F[0] : fma(ph.cv[l], F[l], ce);
    }
    const double hM = 0.5 * Mt;
#pragma unroll
    for (int j = 0; j < D; j++) F[N + j] = fma(vs[j], hM, phat * n[j]);
    // energy = 1/{beta}^ln sum c_vl M_l + M (|{v}|^2 - {|v|^2}/2) + Pi {v}.n + p_inf n_t
    const double k = fma(0.25, vv, -0.25 * s2);
    F[NC - 1] = fma(ce, pm.ib, fma(Mt, k, fma(0.5 * Pi, w, ph.pinf_tot * nt)));
}

// ES dissipation of the interface (iL, iR) = (st[2], st[3]), in Dout
template <int N, int D, int NN, int RC>
__device__ __forceinline__ void dissipation64(const Phys& ph, const NodeTile<N, D, NN, double>& S,
                                              const double (*M)[NN], const int st[6],
                                              const PairMeans<N>& pm, double* Dout)
{
    constexpr int NC = N + D + 1;
    const int iL = st[2], iR = st[3];
    const double tol = ph.stol64;
#pragma unroll
    for (int c = 0; c < NC; c++) Dout[c] = 0.0;
    // node parts of the sign test's tolerance (see dissipation): sum_l |y_l|,
    // beta |v|_1 and beta of both nodes
    double ay = 0.0, av, aE;
    // B_m >= max_l |R_lm| ay + sum_e |R_em| av + |R_Em| aE, so where the
    // entropy variables of the two nodes differ by no more than the tolerance
    // times ay, av and aE every |[[W_m]]| <= tol B_m and Y = 0.  The computed
    // jump is within 16 u B_m of the exact one: the test keeps 32 u of distance,
    // and below that asks for equality.
    {
        const double tq = fmax(0.0, 0.99 * (tol - 7.2e-15));
        const double bL = S.b[iL], bR = S.b[iR];
        double dy = 0.0, dm = 0.0, aL = 0.0, aR = 0.0;
#pragma unroll
        for (int l = 0; l < N; l++) {
            const double yL = S.y[l][iL], yR = S.y[l][iR];
            dy += fabs(yL - yR);
            ay += fabs(yL);
            ay += fabs(yR);
        }
#pragma unroll
        for (int j = 0; j < D; j++) {
            const double vL = S.v[j][iL], vR = S.v[j][iR];
            dm += fabs(fma(bL, vL, -(bR * vR)));
            aL += fabs(vL);
            aR += fabs(vR);
        }
        aE = fabs(bL) + fabs(bR);
        av = fma(fabs(bL), aL, fabs(bR) * aR);
        const bool flat = (dy <= tq * ay) && (dm <= tq * av) && (fabs(bL - bR) <= tq * aE);
        if (!__any(!flat)) return;
    }
    // interface normal, its rotation rows and the averaged velocity
    // (read again from the tile by each group)
    auto averaged = [&](double (&vb)[D]) {
#pragma unroll
        for (int j = 0; j < D; j++) vb[j] = 0.5 * (S.v[j][iL] + S.v[j][iR]);
    };
    double n[D], vb[D];
    averaged(vb);
    const double nt = M[0][iL] + M[0][iR];
    double nn2 = 0.0, vn = 0.0, K = 0.0;
#pragma unroll
    for (int j = 0; j < D; j++) {
        n[j] = M[1 + j][iL] + M[1 + j][iR];
        nn2 = fma(n[j], n[j], nn2);
        vn = fma(vb[j], n[j], vn);
        K = fma(vb[j], vb[j], K);
    }
    K *= 0.5;
    const bool nz = nn2 > 0.0;
    const double inn = nz ? rsqrt64(nn2) : 0.0;
    const double nn = nn2 * inn;
    // the rotation's angle factors (its rows are formed where they are used)
    double ct, sn, cp = 1.0, sp = 0.0;
    if constexpr (D == 2) {
        ct = nz ? n[0] * inn : 1.0;
        sn = n[1] * inn;
    } else {
        const double r2 = fma(n[0], n[0], n[1] * n[1]);
        const bool tz = r2 > 0.0;
        const double ir = tz ? rsqrt64(r2) : 0.0;
        ct = tz ? n[0] * ir : 1.0;
        sn = n[1] * ir;
        cp = nz ? (r2 * ir) * inn : 1.0;
        sp = n[2] * inn;
    }
    // rotated averaged velocity and the sum of its tangential magnitudes
    auto rotated = [&](const double (&vb)[D], double (&vh)[D], double& vt) {
        const double a = fma(ct, vb[0], sn * vb[1]);
        vh[0] = a;
        vh[1] = fma(ct, vb[1], -(sn * vb[0]));
        if constexpr (D == 3) {
            vh[0] = fma(cp, a, sp * vb[2]);
            vh[2] = fma(cp, vb[2], -(sp * a));
        }
        vt = fabs(vh[1]);
        if constexpr (D == 3) vt += fabs(vh[2]);
    };
    // averaged state and the scaled columns of R
    const double Tb = pm.ib;
    double c, H, sa, irho = 0.0;
    double syg = 0.0, sqg = 0.0, e2[2] = {0.0, 0.0}, se = 0.0;
    if constexpr (N == 1) {
        c = sqrt64(ph.gam[0] * ph.Rg[0] * Tb);
        H = fma(ph.cvgam[0], Tb, K);
        sa = sqrt64(pm.rho[0] * ph.isa);
        se = sqrt64(pm.rho[0] * ph.ise);
    } else {
        // (the scheduling fences keep the steps from overlapping: together they
        // need more registers than four waves a SIMD have)
        __builtin_amdgcn_sched_barrier(0);
        double Gb, Rb, pp, rho;
        {
            const double r0L = S.rho[0][iL], r1L = S.rho[1][iL], r0R = S.rho[0][iR], r1R = S.rho[1][iR];
            const double rtL = r0L + r1L, rtR = r0R + r1R;
            // means of the mixture Gamma, R and p + p_inf, each over one divisor
            {
                const double cvL = fma(ph.cv[0], r0L, ph.cv[1] * r1L), cvR = fma(ph.cv[0], r0R, ph.cv[1] * r1R);
                const double cgL = fma(ph.cvgam[0], r0L, ph.cvgam[1] * r1L);
                const double cgR = fma(ph.cvgam[0], r0R, ph.cvgam[1] * r1R);
                Gb = 0.5 * fma(cgL, cvR, cgR * cvL) * rcp64(cvL * cvR);
            }
            __builtin_amdgcn_sched_barrier(0);
            const double RL = fma(ph.Rg[0], r0L, ph.Rg[1] * r1L), RR = fma(ph.Rg[0], r0R, ph.Rg[1] * r1R);
            Rb = 0.5 * fma(RL, rtR, RR * rtL) * rcp64(rtL * rtR);
            __builtin_amdgcn_sched_barrier(0);
            const double bL = S.b[iL], bR = S.b[iR];
            pp = 0.5 * fma(RL, bR, RR * bL) * rcp64(bL * bR);
            __builtin_amdgcn_sched_barrier(0);
            rho = logmean64(rtL, rtR);
        }
        __builtin_amdgcn_sched_barrier(0);
        const double Gm = Gb - 1.0;
        const double ig = rcp64(rho * Gm);
        irho = ig * Gm;
        // rho h = {p} + sum (c_vl rho_l T + p_inf,l): the p_inf cancel by hand
        H = fma(fma(fma(ph.cv[0], pm.rho[0], ph.cv[1] * pm.rho[1]), Tb, pp), irho, K);
        const double Tg = Tb * (ig * rho);
#pragma unroll
        for (int l = 0; l < 2; l++) e2[l] = fma(-(fma(-Gb, ph.cv[l], ph.cvgam[l])), Tg, K);
        __builtin_amdgcn_sched_barrier(0);
        const double GR = Gb * Rb, i = rcp64(GR);
        c = sqrt64(GR * Tb);
        __builtin_amdgcn_sched_barrier(0);
        const double q = rho * i;
        syg = sqrt64((pm.rho[0] * irho * pm.rho[1]) * (Gb * i));
        __builtin_amdgcn_sched_barrier(0);
        sa = sqrt64(q) * 0.70710678118654752440;
        __builtin_amdgcn_sched_barrier(0);
        sqg = sqrt64(q * Gm);
    }
    double hs = 0.5 * fma(nn, c, fabs(nt + vn));   // s / 2
    form_here(hs);

    // one characteristic field per column: w(q) at tile node q for the fields
    // of a group, NF of them; Z of the group
    auto group = [&](auto nf_, auto w, const double* mg, double* Z) {
        constexpr int NF = decltype(nf_)::value;
        double W[NF][6];
        {
            double a[NF], b[NF];
            w(st[2], a);
            w(st[3], b);
#pragma unroll
            for (int f = 0; f < NF; f++) { W[f][2] = a[f]; W[f][3] = b[f]; Z[f] = 0.0; }
        }
        bool need = false;
#pragma unroll
        for (int f = 0; f < NF; f++) need = need || fabs(W[f][3] - W[f][2]) > tol * mg[f];
        if (__any(need)) {
#pragma unroll
            for (int t = 0; t < 6; t++) {
                if (t == 2 || t == 3) continue;
                __builtin_amdgcn_sched_barrier(0);
                double a[NF];
                w(st[t], a);
#pragma unroll
                for (int f = 0; f < NF; f++) W[f][t] = a[f];
            }
#pragma unroll
            for (int f = 0; f < NF; f++) {
                double jump;
                __builtin_amdgcn_sched_barrier(0);
                const double jw = weno_jump64<RC == 1>(W[f], ph, jump);
                if ((jw * jump > 0.0) && (fabs(jump) > tol * mg[f])) Z[f] = jw;
            }
        }
    };
    auto dotv = [&](const double* a, int q, double c0) {
        double r = c0;
#pragma unroll
        for (int j = 0; j < D; j++) r = fma(a[j], S.v[j][q], r);
        return r;
    };

    // R Z: species rows R0, R1, the sum that multiplies vbar, the other momentum
    // parts mo and the energy row En
    double R0, R1 = 0.0, zsum, En, mo[D];
    // species (entropy) fields
    asm volatile("" ::: "memory");
    {
        constexpr int NF = N == 1 ? 1 : 2;
        double mg[NF], Z[NF], sd[NF], ce[NF], cd[NF][N];
        double vb[D], vh[D], vt;
        averaged(vb);
        rotated(vb, vh, vt);
        const double va = (fabs(vh[0]) + vt) * av;
        if constexpr (N == 1) {
            cd[0][0] = se;
            sd[0] = se;
            ce[0] = se * K;
            mg[0] = se * fma(K, aE, ay + va);
        } else {
            cd[0][0] = -syg * ph.sr21;
            cd[0][1] = syg * ph.isr21;
            cd[1][0] = pm.rho[0] * (irho * sqg);
            cd[1][1] = pm.rho[1] * (irho * sqg);
#pragma unroll
            for (int f = 0; f < 2; f++) {
                sd[f] = cd[f][0] + cd[f][1];
                ce[f] = fma(cd[f][0], e2[0], cd[f][1] * e2[1]);
                mg[f] = fma(fabs(ce[f]), aE, fma(fabs(sd[f]), va, fmax(fabs(cd[f][0]), fabs(cd[f][1])) * ay));
            }
        }
        group(std::integral_constant<int, NF>{},
              [&](int q, double* o) {
                  const double b = S.b[q];
                  const double t = dotv(vb, q, 0.0);
#pragma unroll
                  for (int f = 0; f < NF; f++) {
                      double r = b * fma(sd[f], t, -ce[f]);
#pragma unroll
                      for (int l = 0; l < N; l++) r = fma(cd[f][l], S.y[l][q], r);
                      o[f] = r;
                  }
              },
              mg, Z);
        if constexpr (N == 1) {
            const double z = se * Z[0];
            R0 = zsum = z;
            En = K * z;
        } else {
            const double z1 = fma(cd[0][0], Z[0], cd[1][0] * Z[1]), z2 = fma(cd[0][1], Z[0], cd[1][1] * Z[1]);
            R0 = z1;
            R1 = z2;
            zsum = z1 + z2;
            En = fma(ce[0], Z[0], ce[1] * Z[1]);
        }
    }
    form_here(R0);
    form_here(zsum);
    form_here(En);
    if constexpr (N == 2) form_here(R1);
    // tangential fields
    asm volatile("" ::: "memory");
    {
        const double sct = N == 1 ? sqrt64(pm.rho[0] * pm.ib) : 1.41421356237309504880 * sa * c;
        double tc[D - 1][D], ck[D - 1], mg[D - 1], Z[D - 1];
        double vb[D], vh[D], vt;
        averaged(vb);
        rotated(vb, vh, vt);
#pragma unroll
        for (int f = 0; f < D - 1; f++) {
#pragma unroll
            for (int j = 0; j < D; j++) tc[f][j] = 0.0;
            ck[f] = sct * vh[1 + f];
            mg[f] = fma(fabs(ck[f]), aE, sct * av);
        }
        tc[0][0] = -sct * sn;
        tc[0][1] = sct * ct;
        if constexpr (D == 3) {
            const double q = -sct * sp;
            tc[1][0] = q * ct;
            tc[1][1] = q * sn;
            tc[1][2] = sct * cp;
        }
        group(std::integral_constant<int, D - 1>{},
              [&](int q, double* o) {
                  const double b = S.b[q];
#pragma unroll
                  for (int f = 0; f < D - 1; f++) {
                      double r = fma(tc[f][0], S.v[0][q], -ck[f]);
                      r = fma(tc[f][1], S.v[1][q], r);
                      if (D == 3 && f == 1) r = fma(tc[f][D - 1], S.v[D - 1][q], r);
                      o[f] = b * r;
                  }
              },
              mg, Z);
#pragma unroll
        for (int j = 0; j < D; j++) mo[j] = tc[0][j] * Z[0];
        En = fma(ck[0], Z[0], En);
        if constexpr (D == 3) {
#pragma unroll
            for (int j = 0; j < D; j++) mo[j] = fma(tc[1][j], Z[1], mo[j]);
            En = fma(ck[1], Z[1], En);
        }
    }
    form_here(En);
#pragma unroll
    for (int j = 0; j < D; j++) form_here(mo[j]);
    // acoustic fields
    asm volatile("" ::: "memory");
    {
        double cv[D], cn[D], row[D], mg[2], Z[2], cY[N];
        double vb[D], vh[D], vt;
        averaged(vb);
        rotated(vb, vh, vt);
        const double cv0 = c * vh[0];
        row[0] = cp * ct;
        row[1] = cp * sn;
        if constexpr (D == 3) row[2] = sp;
        const double cH = sa * H, sc = sa * c, ck = sa * cv0;
#pragma unroll
        for (int j = 0; j < D; j++) {
            cv[j] = sa * vb[j];
            cn[j] = sc * row[j];
        }
#pragma unroll
        for (int l = 0; l < N; l++) cY[l] = N == 1 ? sa : pm.rho[l] * (irho * sa);
        double ya = ay;
        if constexpr (N == 2) ya = fmax(fabs(pm.rho[0]), fabs(pm.rho[1])) * fabs(irho) * ay;
        mg[0] = sa * fma(fabs(H - cv0), aE, fma(fabs(vh[0] - c) + vt, av, ya));
        mg[1] = sa * fma(fabs(H + cv0), aE, fma(fabs(vh[0] + c) + vt, av, ya));
        group(std::integral_constant<int, 2>{},
              [&](int q, double* o) {
                  const double b = S.b[q];
                  double r = b * dotv(cv, q, -cH);
#pragma unroll
                  for (int l = 0; l < N; l++) r = fma(cY[l], S.y[l][q], r);
                  const double u = b * dotv(cn, q, -ck);
                  o[0] = r - u;
                  o[1] = r + u;
              },
              mg, Z);
        const double zs = sa * (Z[0] + Z[1]), zd = sa * (Z[1] - Z[0]);
        zsum += zs;
        const double cz = c * zd;
#pragma unroll
        for (int j = 0; j < D; j++) mo[j] = fma(cz, row[j], mo[j]);
        En = fma(H, zs, fma(cv0, zd, En));
        if constexpr (N == 1) R0 += zs;
        else {
            const double zr = irho * zs;
            R0 = fma(pm.rho[0], zr, R0);
            R1 = fma(pm.rho[1], zr, R1);
        }
    }
    form_here(R0);
    form_here(zsum);
    form_here(En);
    if constexpr (N == 2) form_here(R1);
#pragma unroll
    for (int j = 0; j < D; j++) form_here(mo[j]);
    asm volatile("" ::: "memory");
    averaged(vb);
    Dout[0] = hs * R0;
    if constexpr (N == 2) Dout[1] = hs * R1;
#pragma unroll
    for (int j = 0; j < D; j++) Dout[N + j] = hs * fma(vb[j], zsum, mo[j]);
    Dout[NC - 1] = hs * En;
}

// two-point EC flux in the precision of the sweep
template <int N, int D, int NN, typename R>
__device__ __forceinline__ void two_point(const Phys& ph, const NodeTile<N, D, NN, R>& S, const double (*M)[NN],
                                          int ia, int ib, R* F)
{
    if constexpr (sizeof(R) == 8) {
        PairMeans<N> pm;
        double isb;
        pair_means<N, D, NN>(S, ia, ib, pm, isb);
        ec_flux64<N, D, NN>(ph, S, M, ia, ib, pm, isb, F);
    } else {
        ec_pair<N, D, NN, R>(ph, S, M, ia, ib, F);
    }
}

// Numerical flux at the TL + 1 interfaces of each of TC lines of a tile
// (the interface form of eq ECFlux_curv_2p minus the ES dissipation of eq
// HOstable), left in X slot f + 1 of line c.
//
// Interface slot f = 0..TL of a line has left node l = f + 2 (the tile's
// first own node is l = 3).  Its thread evaluates P_m = F(l, l+m), m = 1..3,
// and with B(f) = a3 P_3 and H(f) = a2 P_2 + B(f) the flux is
//   F_f = a1 P_1 - D_f + H(f) + H(f-1) + B(f-2),
// so each two-point flux is evaluated once.  X slot f + 2 carries B(f),
// then H(f), and finally slot f + 1 holds F_f.  The pairs F(0,3), F(1,4),
// F(1,3) left of the first interface (B(-2), B(-1), H(-1)) are taken by
// the lanes with hid = 0 .. 3 TC - 1 (one wave, chosen by the caller).
// lidx(l, c) is the tile index of node l of line c, xidx(s, c) the X index
// of slot s of line c, line_ok(c) whether line c exists; f_ok says that
// this thread's interface (fi, fc) exists and its six nodes are loaded.
// RC selects the reconstruction of the dissipation (0: multi-resolution
// WENO, 1: classical WENO5).  X overlays the node quantities of S (all but the metrics):
// every flux is then formed in registers first and X is written only after
// a barrier that ends all node reads.  Every thread of the block must call
// this (it holds barriers).
// (MG: the FP32 dissipation's acoustic and species fields in one group or two;
// the FP64 one takes them apart in any case)
// interface_fluxes_m is the general form: the metrics M of the direction
// are passed in, X rows are XS slots long, and the tile's TL and TC may be
// run-time values (a block that sweeps two directions at once picks them per
// wave), and pre() runs between the fluxes and the exchange (loads that the
// caller wants in flight through the latter); interface_fluxes takes the tile's own metrics, fixed sizes and
// one group.
template <int N, int D, int NN, int XS, int RC, typename R, int MG, typename LI, typename XI,
          typename LOK, typename PRE>
__device__ __forceinline__ void interface_fluxes_m(const Phys& ph, const NodeTile<N, D, NN, R>& S,
                                                   const double (*M)[NN], R (*X)[XS], LI lidx, XI xidx,
                                                   LOK line_ok, int fi, int fc, bool f_ok, int hid,
                                                   int TL, int TC, PRE pre)
{
    constexpr int NC = N + D + 1;
    const R a1 = R(ph.alpha[0]), a2 = R(ph.alpha[1]), a3 = R(ph.alpha[2]);
    const int fl = fi + 2;
    R G[NC], A2[NC], B3[NC];
    if (f_ok) {
        R F[NC];
        if constexpr (sizeof(R) == 8) {
            PairMeans<N> pm;
            double isb;
            pair_means<N, D, NN>(S, lidx(fl, fc), lidx(fl + 1, fc), pm, isb);
            if (ph.dissipation) {
                int st[6];
#pragma unroll
                for (int q = 0; q < 6; q++) st[q] = lidx(fl - 2 + q, fc);
                dissipation64<N, D, NN, RC>(ph, S, M, st, pm, G);
            } else {
#pragma unroll
                for (int cc = 0; cc < NC; cc++) G[cc] = 0.0;
            }
            // (1 / (beta_a + beta_b) is taken again and the node values are read
            // again: fewer registers across the dissipation)
            asm volatile("" ::: "memory");
            isb = rcp64(S.b[lidx(fl, fc)] + S.b[lidx(fl + 1, fc)]);
            ec_flux64<N, D, NN>(ph, S, M, lidx(fl, fc), lidx(fl + 1, fc), pm, isb, F);
        } else if (ph.dissipation) {
            // zero tolerance of the sign test, relative to the size of the
            // terms of W, in the precision of the arithmetic (0: the sign
            // test as printed)
            const Weno<R> Wc = make_weno<R>(ph.chi, ph.eps, ph.stol32);
            int st[6];
#pragma unroll
            for (int q = 0; q < 6; q++) st[q] = lidx(fl - 2 + q, fc);
            dissipation<N, D, NN, R, MG>(ph, S, M, st, Wc, G);
        } else {
#pragma unroll
            for (int cc = 0; cc < NC; cc++) G[cc] = R(0);
        }
        if constexpr (sizeof(R) == 4) ec_pair<N, D, NN, R>(ph, S, M, lidx(fl, fc), lidx(fl + 1, fc), F);
#pragma unroll
        for (int cc = 0; cc < NC; cc++) G[cc] = a1 * F[cc] - G[cc];
        if (a2 != R(0)) {
            two_point<N, D, NN, R>(ph, S, M, lidx(fl, fc), lidx(fl + 2, fc), F);
        } else {
#pragma unroll
            for (int cc = 0; cc < NC; cc++) F[cc] = R(0);
        }
#pragma unroll
        for (int cc = 0; cc < NC; cc++) A2[cc] = a2 * F[cc];
        if (a3 != R(0)) {
            two_point<N, D, NN, R>(ph, S, M, lidx(fl, fc), lidx(fl + 3, fc), F);
        } else {
#pragma unroll
            for (int cc = 0; cc < NC; cc++) F[cc] = R(0);
        }
#pragma unroll
        for (int cc = 0; cc < NC; cc++) B3[cc] = a3 * F[cc];
    }
    // the pairs F(0,3), F(1,4), F(1,3) left of the first interface
    const bool halo = hid >= 0 && hid < 3 * TC;
    R Bh[NC];
    int hslot = 0, hc = 0;
    if (halo) {
        const int h = hid / TC;
        hc = hid % TC;
        const R am = (h == 2) ? a2 : a3;
        hslot = (h == 0) ? 0 : ((h == 1) ? 1 : TL + 3);
        if (line_ok(hc) && am != R(0)) {
            two_point<N, D, NN, R>(ph, S, M, lidx(h == 0 ? 0 : 1, hc), lidx(h == 1 ? 4 : 3, hc), Bh);
        } else {
#pragma unroll
            for (int cc = 0; cc < NC; cc++) Bh[cc] = R(0);
        }
#pragma unroll
        for (int cc = 0; cc < NC; cc++) Bh[cc] = am * Bh[cc];
    }
    pre();
    __syncthreads();   // node reads end before X overwrites them
    if (halo) {
#pragma unroll
        for (int cc = 0; cc < NC; cc++) X[cc][xidx(hslot, hc)] = Bh[cc];
    }
    if (f_ok) {
#pragma unroll
        for (int cc = 0; cc < NC; cc++) X[cc][xidx(fi + 2, fc)] = B3[cc];
    }
    __syncthreads();
    R Hf[NC], Hm[NC];
    if (f_ok) {
#pragma unroll
        for (int cc = 0; cc < NC; cc++) {
            G[cc] += X[cc][xidx(fi, fc)];                   // + B(f-2)
            Hf[cc] = A2[cc] + X[cc][xidx(fi + 2, fc)];      // H(f)
        }
        if (fi == 0) {
#pragma unroll
            for (int cc = 0; cc < NC; cc++) Hm[cc] = X[cc][xidx(TL + 3, fc)] + X[cc][xidx(1, fc)];
        }
    }
    __syncthreads();
    if (f_ok) {
#pragma unroll
        for (int cc = 0; cc < NC; cc++) X[cc][xidx(fi + 2, fc)] = Hf[cc];
        if (fi == 0) {
#pragma unroll
            for (int cc = 0; cc < NC; cc++) X[cc][xidx(1, fc)] = Hm[cc];
        }
    }
    __syncthreads();
    if (f_ok) {
#pragma unroll
        for (int cc = 0; cc < NC; cc++) {
            const int xi = xidx(fi + 1, fc);
            X[cc][xi] = G[cc] + (Hf[cc] + X[cc][xi]);     // F_f into slot f+1
        }
    }
    __syncthreads();
}

template <int N, int D, int NN, int TL, int TC, int RC, typename R, typename LI, typename XI, typename LOK>
__device__ __forceinline__ void interface_fluxes(const Phys& ph, const NodeTile<N, D, NN, R>& S,
                                                 R (*X)[(TL + 4) * TC], LI lidx, XI xidx,
                                                 LOK line_ok, int fi, int fc, bool f_ok, int hid)
{
    interface_fluxes_m<N, D, NN, (TL + 4) * TC, RC, R, 1>(ph, S, S.m, X, lidx, xidx, line_ok, fi, fc, f_ok, hid,
                                                          TL, TC, [] {});
}

// J U and J of one node as loaded
template <int NC>
struct NodeRaw {
    double U[NC], J;
};

template <int NC>
__device__ __forceinline__ void node_load(NodeRaw<NC>& r, const double* __restrict__ JU,
                                          const double* __restrict__ Jv, long P, long gi)
{
    r.J = Jv[gi];
#pragma unroll
    for (int cc = 0; cc < NC; cc++) r.U[cc] = JU[cc * P + gi];
}

// the reciprocal of the sweep's precision R (see rcp64)
template <typename R>
__device__ __forceinline__ double inv(double x)
{
    if constexpr (sizeof(R) == 8) return rcp64(x);
    else return rcp(x);
}

// primitive node quantities of a loaded node into tile slot li; returns the
// status bits of the node (1: rho_l <= 0, T <= 0 or non-finite; 2: J <= 0)
template <int N, int D, int NN, typename R>
__device__ __forceinline__ unsigned node_state(const Phys& ph, NodeTile<N, D, NN, R>& S, int li,
                                               const NodeRaw<N + D + 1>& raw)
{
    constexpr int NC = N + D + 1;
    const double Jq = raw.J;
    const double iJ = inv<R>(Jq);
    double U[NC];
#pragma unroll
    for (int cc = 0; cc < NC; cc++) U[cc] = raw.U[cc] * iJ;
    double rt = 0.0, cvr = 0.0;
#pragma unroll
    for (int sp = 0; sp < N; sp++) {
        rt += U[sp];
        cvr += ph.cv[sp] * U[sp];
    }
    const double ir = inv<R>(rt);
    double kin = 0.0;
#pragma unroll
    for (int j = 0; j < D; j++) {
        const double vj = U[N + j] * ir;
        S.v[j][li] = vj;
        kin += 0.5 * U[N + j] * vj;
    }
    const double e = U[NC - 1] - kin - ph.pinf_tot;
    const double beta = cvr * inv<R>(e);
    S.b[li] = beta;
    const double lbeta = ln_pos(beta);
    S.lb[li] = lbeta;
    bool ok = (beta > 0.0) && isfinite(beta) && isfinite(kin);
    double v1 = 0.0, v2 = 0.0;
#pragma unroll
    for (int j = 0; j < D; j++) {
        const double vj = S.v[j][li];
        v1 += fabs(vj);
        v2 += vj * vj;
    }
    double ysum = 0.0;
#pragma unroll
    for (int sp = 0; sp < N; sp++) {
        S.rho[sp][li] = U[sp];
        const double lr = ln_pos(U[sp]);
        S.lrho[sp][li] = lr;
        if constexpr (sizeof(R) == 8) {
            const double y = fma(-0.5 * beta, v2, fma(ph.Rg[sp], lr, fma(ph.cv[sp], lbeta, ph.cvgam[sp])));
            S.y[sp][li] = y;
        } else {
            ysum += fabs(ph.cv[sp] * lbeta + ph.Rg[sp] * lr + ph.cvgam[sp] - 0.5 * beta * v2);
        }
        ok = ok && (U[sp] > 0.0);
    }
    if constexpr (sizeof(R) == 4) {
        S.ay[li] = float(ysum);
        S.av[li] = float(fabs(beta) * v1);
    }
    if constexpr (N == 2 && sizeof(R) == 4) S.lrt[li] = ln_pos(rt);
    unsigned bad = ok ? 0u : 1u;
    if (!(Jq > 0.0)) bad |= 2u;
    return bad;
}

}  // namespace es

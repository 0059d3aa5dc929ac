// es_rhs.hip -- the semi-discrete right-hand side (Sections 3.1-3.4) and the
// fused SSP-RK3 stage (Section 5) on gfx950.
//
// k_rhs_dir is one launch per direction k; k_rhs_xy (below) builds the x and
// y directions of a 3D grid in one launch.  A 3D stage takes the z sweep, which
// writes its term, and then k_rhs_xy, which adds the others and applies the
// stage combination: the z sweep is bound by HBM (its halo along z is read
// again by every tile), the x-y launch by FP64 issue, so the operands of the
// combination are read beside the latter (2.78 against 2.99 ms a stage at
// 256^3 with the combination in the z sweep).  In k_rhs_dir a block of 256
// threads owns a tile of TL nodes along k on TC grid lines (consecutive in the
// line ordering, so the fastest other index runs along the lines and global
// loads coalesce), stages the node quantities of the tile plus a 3-node halo
// along k in LDS, and builds the full numerical flux at each of the TL + 1
// interfaces of every line, one thread per interface:
//   F_{i+1/2} = sum_m alpha_m sum_{s<m} F(i-s, i-s+m)  -  D_{i+1/2}
// (the interface form of eq ECFlux_curv_2p minus the ES dissipation
// 1/2 s T^T R Y [[W]]^WENO of eq HOstable).  Each two-point flux
// F(a, a+m) is evaluated once, by the thread whose interface has left node
// a; the m interfaces that use it collect it through an LDS exchange in
// three barrier-separated steps.  The node update is then the interface
// difference plus the GCL term delta_k[n_t] (eq GCL_flux), times -1/dxi_k,
// accumulated into the output; the last launch's epilogue can apply the
// Shu-Osher stage combination.
#include "es_flux.hpp"

namespace es {

// What bounds a sweep: FP64 issue and the latency of its loads and barriers,
// hidden by four blocks a compute unit (39.7 KB of LDS and 118 registers for
// two species in 3D).  At 256^3 (water / air, moving mesh) a stage took 3.11 ms
// against 4.05 ms with the arithmetic written term by term (2.34 against
// 3.06 thousand VALU instructions a wave), the loads of a block's nodes waited for one
// after the other and the stage epilogue's loads and stores alternating.
// Waves per SIMD: four in FP64, three in FP32 (one field group: splitting it
// costs more than a fourth wave gains)
template <int N, int D, int K, int TL, int TC, int MODE, typename R, int RC>
__global__ void __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(sizeof(R) == 8 ? 4 : 3, 8)))
k_rhs_dir(Phys ph, Geo g, const double* __restrict__ JU, const double* __restrict__ Jv,
          const double* __restrict__ jxx, const double* __restrict__ jxt,
          double* __restrict__ accU, double* __restrict__ accJ, RkArgs rk,
          unsigned* __restrict__ status)
{
    constexpr int NT = 256;
    constexpr int NC = N + D + 1;
    constexpr int NL = TL + 6;          // nodes per line: tile + 3-node halo on each side
    constexpr int NN = NL * TC;
    constexpr int NI = (TL + 1) * TC;   // interfaces (one thread each)
    constexpr int NS = TL + 4;          // exchange slots per line
    constexpr int NX = NS * TC;
    static_assert(NI <= NT && 3 * TC <= 64 && TL * TC <= NT, "tile does not fit the block");
    constexpr int FA = (K == 0) ? 1 : 0;   // across index that runs fastest
    constexpr int SA = (K == 2) ? 1 : 2;   // slowest across index
    __shared__ NodeTile<N, D, NN, R> S;
    // the flux exchange overlays the node quantities (not the metrics, which
    // the GCL term reads afterwards): 37 KB of LDS in all for two species in
    // 3D, so four blocks share a compute unit
    static_assert(sizeof(R) * NC * NX <= sizeof(S) - sizeof(S.m), "exchange does not fit the tile");
    R (*X)[NX] = reinterpret_cast<R (*)[NX]>(&S.rho[0][0]);

    const long P = g.P;
    const int nK = g.n[K];
    const int nF = g.n[FA];
    const long nlines = (long)nF * ((SA < D) ? g.n[SA] : 1);
    const int nseg = (nK + TL - 1) / TL;
    const int seg0 = (int)(blockIdx.x % nseg) * TL;
    const long line0 = (long)(blockIdx.x / nseg) * TC;
    const long sK = dir_stride(g, K);
    const int t = threadIdx.x;

    // LDS layouts are line-fastest in every direction, so the lanes of a wave
    // (consecutive lines) read consecutive words; the x sweep still walks x
    // fastest in its global loads and stores
    auto lidx = [](int l, int c) { return c + TC * l; };
    auto xidx = [](int s, int c) { return c + TC * s; };
    // padded index of the node at along-index 0 of each line of the block,
    // tabulated once (the line index splits into the two across indices by a
    // division)
    __shared__ long s_base[TC];
    if (t < TC) {
        const int L = (int)line0 + t;
        int i[3];
        i[K] = 0;
        i[FA] = g.ng + L % nF;
        i[SA] = (SA < D) ? g.ng + L / nF : 0;
        s_base[t] = node_index(g, i[0], i[1], i[2]);
    }
    __syncthreads();

    // ---- phase 1: node quantities of the tile (+ halo) into LDS ----------
    // all loads of the thread's nodes are issued before the first is used:
    // the block then waits for memory once
    unsigned bad = 0;
    const double itd = rk.tdiv ? 1.0 / *rk.tdiv : 1.0;
    {
        constexpr int NQ = (NN + NT - 1) / NT;
        NodeRaw<NC> raw[NQ];
        double mt[NQ], mx[NQ][D];
        bool have[NQ];
        int li[NQ];
        const double* __restrict__ jt = jxt ? jxt : jxx;   // (a fixed mesh reads it and drops it)
#pragma unroll
        for (int r = 0; r < NQ; r++) {
            const int q = t + r * NT;
            const int l = (K == 0) ? (q % NL) : (q / TC);
            const int c = (K == 0) ? (q / NL) : (q % TC);
            const int along = g.ng + seg0 + l - 3;
            have[r] = q < NN && along < g.np[K] && line0 + c < nlines;
            li[r] = lidx(l, c);
            // (a node that does not exist reads the tile's first node: a branch
            // would make the loads wait for each other)
            const long gi = have[r] ? s_base[c] + along * sK : s_base[0] + (g.ng + seg0) * sK;
            node_load<NC>(raw[r], JU, Jv, P, gi);
            mt[r] = jt[(long)K * P + gi];
#pragma unroll
            for (int j = 0; j < D; j++) mx[r][j] = jxx[(long)(K * D + j) * P + gi];
        }
#pragma unroll
        for (int r = 0; r < NQ; r++) {
            if (have[r]) {
                bad |= node_state<N, D, NN, R>(ph, S, li[r], raw[r]);
                S.m[0][li[r]] = jxt ? 0.5 * (mt[r] * itd) : 0.0;
#pragma unroll
                for (int j = 0; j < D; j++) S.m[1 + j][li[r]] = 0.5 * mx[r][j];
            }
        }
    }
    if (bad) atomicOr(status, bad);
    __syncthreads();

    // ---- phase 2: interface fluxes --------------------------------------
    const int fi = t / TC;
    const int fc = t % TC;
    // node fi + 5 must be inside the padded grid (ragged last segment)
    const bool f_ok = (t < NI) && (line0 + fc < nlines) && (g.ng + seg0 + fi + 2 < g.np[K]);
    interface_fluxes<N, D, NN, TL, TC, true, RC, R>(ph, S, X, lidx, xidx,
                                          [&](int c) { return line0 + c < nlines; }, fi, fc, f_ok,
                                          t - (int)(blockIdx.x & 3) * 64);

    // ---- phase 3: interface differences at the tile's nodes --------------
    const double dt = (MODE == MODE_RK) ? *rk.dt : 0.0;
    if (t < TL * TC) {
        const int lo = (K == 0) ? (t % TL) : (t / TC);
        const int c = (K == 0) ? (t / TL) : (t % TC);
        if (seg0 + lo < nK && line0 + c < nlines) {
            const int l = lo + 3;
            double gcl = 0.0;
#pragma unroll
            for (int m = 1; m <= 3; m++)
                gcl += ph.alpha[m - 1] * (S.m[0][lidx(l + m, c)] - S.m[0][lidx(l - m, c)]);
            const long gi = s_base[c] + (g.ng + seg0 + lo) * sK;
            const double h = g.idxi[K];
            const double dJ = -gcl * h;   // S.m holds half the metrics
            // every operand is loaded before the first result is stored (the
            // output may be the accumulator or Q_n, so a load after a store
            // would wait for it: seven round trips to memory instead of one)
            double ac[NC + 1], qs[NC + 1], qn[NC + 1];
            // stage 0 has a = 0: Q_s stands in for Q_n, which is not read
            const double* qnU = MODE == MODE_RK && rk.a != 0.0 ? rk.JUn : JU;
            const double* qnJ = MODE == MODE_RK && rk.a != 0.0 ? rk.Jn : Jv;
#pragma unroll
            for (int cc = 0; cc <= NC; cc++) {
                if constexpr (MODE != MODE_WRITE) ac[cc] = cc < NC ? accU[cc * P + gi] : accJ[gi];
                if constexpr (MODE == MODE_RK) {
                    qs[cc] = cc < NC ? JU[cc * P + gi] : Jv[gi];
                    qn[cc] = cc < NC ? qnU[cc * P + gi] : qnJ[gi];
                }
            }
            double* oU = MODE == MODE_RK && rk.outU ? rk.outU : accU;
            double* oJ = MODE == MODE_RK && rk.outJ ? rk.outJ : accJ;
#pragma unroll
            for (int cc = 0; cc <= NC; cc++) {
                const double d = cc < NC ? -(double)(X[cc < NC ? cc : 0][xidx(lo + 2, c)] -
                                                     X[cc < NC ? cc : 0][xidx(lo + 1, c)]) * h
                                         : dJ;
                double o = d;
                if constexpr (MODE != MODE_WRITE) o = ac[cc] + d;
                if constexpr (MODE == MODE_RK) o = rk.a * qn[cc] + rk.b * (qs[cc] + dt * o);
                (cc < NC ? oU[cc * P + gi] : oJ[gi]) = o;
            }
        }
    }
}

// The x and y directions of a 3D grid in one launch.  A block of 512
// threads owns a TX x TY tile of one z plane: it stages the node quantities
// of the tile plus a 3-node halo along x and y (a plus-shaped patch; the
// corners are never read) and the halved metrics of both directions in LDS
// once, then waves 0-3 build the x fluxes of the tile's TY rows and waves
// 4-7 the y fluxes of its TX columns at the same time, each with the
// interface scheme of interface_fluxes.  A node's output is the x
// difference plus the y difference, each rounded on its own, plus the
// accumulated z term.  LDS: 70 KB at 16 x 15 with two species, two blocks
// (four waves per SIMD) per compute unit; bound by FP64 issue and by the
// waits of the two blocks' phases (VALU busy 65 % of the cycles).
template <int N, int TX, int TY, int MODE, typename R, int RC, int MG>
__global__ void __launch_bounds__(512) __attribute__((amdgpu_waves_per_eu(4, 8)))
k_rhs_xy(Phys ph, Geo g, const double* __restrict__ JU, const double* __restrict__ Jv,
         const double* __restrict__ jxx, const double* __restrict__ jxt, double* accU, double* accJ, RkArgs rk, unsigned* __restrict__ status)
{
    constexpr int D = 3;
    constexpr int NT = 512;
    constexpr int NC = N + D + 1;
    constexpr int NEX = TX + 6, NEY = TY + 6;
    constexpr int NN = NEX * NEY;
    constexpr int XSX = (TX + 4) * TY, XSY = (TY + 4) * TX;    // exchange slots per component
    constexpr int XS = XSX > XSY ? XSX : XSY;
    static_assert((TX + 1) * TY <= NT / 2 && (TY + 1) * TX <= NT / 2 && 3 * TX <= 64 && 3 * TY <= 64,
                  "tile does not fit the block");
    __shared__ NodeTile<N, D, NN, R> S;     // S.m: the x metrics
    __shared__ double My[D + 1][NN];     // the y metrics
    static_assert(sizeof(R) * 2 * NC * XS <= sizeof(S) - sizeof(S.m), "exchange does not fit the tile");
    R (*Xb)[XS] = reinterpret_cast<R (*)[XS]>(&S.rho[0][0]);   // x rows 0..NC-1, y rows NC..2NC-1

    const long P = g.P;
    const int ng = g.ng, np0 = g.np[0], np1 = g.np[1];
    const int nx = g.n[0], ny = g.n[1];
    int bx, by, bz;
    xcd_plane(bx, by, bz);
    const int ox = bx * TX, oy = by * TY;
    // padded index of patch node (0, 0), at interior (ox - 3, oy - 3) of plane bz
    const long base = ((long)(ng + bz) * np1 + (oy + ng - 3)) * np0 + (ox + ng - 3);
    const int t = threadIdx.x;

    // ---- node quantities and metrics of the patch -------------------------
    // one node a thread, all of its loads issued before the first is used
    static_assert(NN <= NT, "one node a thread");
    unsigned bad = 0;
    const double itd = rk.tdiv ? 1.0 / *rk.tdiv : 1.0;
    {
        const int lx = t % NEX, ly = t / NEX;
        const bool cx = lx >= 3 && lx < 3 + TX, cy = ly >= 3 && ly < 3 + TY;
        // corners are never read, nodes beyond a ragged tile do not exist
        const bool have = t < NN && (cx || cy) && ox + lx - 3 + ng < np0 && oy + ly - 3 + ng < np1;
        const long gi = base + (long)ly * np0 + lx;
        if (have) {
            NodeRaw<NC> raw;
            double mx[D + 1], my[D + 1];
            node_load<NC>(raw, JU, Jv, P, gi);
            const double* __restrict__ jt = jxt ? jxt : jxx;   // (a fixed mesh reads it and drops it)
            if (cy) {
                mx[0] = jt[gi];
#pragma unroll
                for (int j = 0; j < D; j++) mx[1 + j] = jxx[(long)j * P + gi];
            }
            if (cx) {
                my[0] = jt[P + gi];
#pragma unroll
                for (int j = 0; j < D; j++) my[1 + j] = jxx[(long)(D + j) * P + gi];
            }
            bad = node_state<N, D, NN, R>(ph, S, t, raw);
            if (cy) {
                S.m[0][t] = jxt ? 0.5 * (mx[0] * itd) : 0.0;
#pragma unroll
                for (int j = 0; j < D; j++) S.m[1 + j][t] = 0.5 * mx[1 + j];
            }
            if (cx) {
                My[0][t] = jxt ? 0.5 * (my[0] * itd) : 0.0;
#pragma unroll
                for (int j = 0; j < D; j++) My[1 + j][t] = 0.5 * my[1 + j];
            }
        }
    }
    if (bad) atomicOr(status, bad);
    __syncthreads();

    // ---- interface fluxes: x in waves 0-3, y in waves 4-7 ------------------
    // x: interface fi of row fc, rows fastest; y: interface fi of column fc,
    // interfaces fastest.  Either way consecutive lanes are one patch row
    // (22 doubles) apart: 16 of them fall on the even banks and the next 16,
    // one node on, on the odd ones.  (Lanes along the contiguous index break a
    // row every 16 or 17 lanes and met conflicts for a third of the LDS time.)
    // The direction is uniform over a wave; read from the first lane, everything
    // derived from it lives in scalar registers
    const bool ydir = __builtin_amdgcn_readfirstlane(t / (NT / 2)) != 0;
    const int u = t & (NT / 2 - 1);
    const int TL = ydir ? TY : TX, TC = ydir ? TX : TY;
    const int fi = ydir ? u % (TY + 1) : u / TY;
    const int fc = ydir ? u / (TY + 1) : u % TY;
    const int o_along = ydir ? oy : ox, o_line = ydir ? ox : oy;
    const int n_line = ydir ? nx : ny, np_along = ydir ? np1 : np0;
    const bool f_ok = (u < (TL + 1) * TC) && (o_line + fc < n_line) && (o_along + fi + 2 + ng < np_along);
    // one copy of the arithmetic for both directions, the tile strides,
    // metric array and exchange rows picked per wave (compiling each
    // direction's arithmetic on its own under a branch took 4 % longer: the
    // join spills registers)
    const int sl = ydir ? NEX : 1, sc = ydir ? 1 : NEX, l0 = ydir ? 3 : 3 * NEX;
    const int xl = ydir ? 1 : TY, xc = ydir ? TY + 4 : 1;
    // each half of the block writes half of the components (J U, then J) of the
    // tile's nodes; their operands are fetched before the exchange
    constexpr int NH = NC / 2 + 1;
    const int ni = u % TX, nj = u / TX, c0 = ydir ? NH : 0;
    const bool own = u < TX * TY && ox + ni < nx && oy + nj < ny;
    const long gn = own ? base + (long)(nj + 3) * np0 + (ni + 3) : base + 3L * np0 + 3;
    double ac[NH], qs[NH], qn[NH];
    auto fetch = [&] {
#pragma unroll
        for (int i = 0; i < NH; i++) {
            const int cc = c0 + i < NC ? c0 + i : NC;
            const bool isJ = cc == NC;
            if constexpr (MODE != MODE_WRITE) ac[i] = (isJ ? accJ : accU + cc * P)[gn];
            if constexpr (MODE == MODE_RK) {
                qs[i] = (isJ ? Jv : JU + cc * P)[gn];
                // stage 0 has a = 0: Q_s stands in for Q_n, which is not read
                const double* nU = rk.a != 0.0 ? rk.JUn : JU;
                const double* nJ = rk.a != 0.0 ? rk.Jn : Jv;
                qn[i] = (isJ ? nJ : nU + cc * P)[gn];
            }
        }
    };
    interface_fluxes_m<N, D, NN, XS, true, RC, R, MG>(
        ph, S, ydir ? My : S.m, ydir ? Xb + NC : Xb, [=](int l, int c) { return l0 + l * sl + c * sc; },
        [=](int s, int c) { return s * xl + c * xc; }, [=](int c) { return o_line + c < n_line; }, fi, fc,
        f_ok, u - (int)(blockIdx.x & 3) * 64, TL, TC, fetch);

    // ---- node outputs: z term + (x difference + y difference) --------------
    if (own) {
        const double hx = g.idxi[0], hy = g.idxi[1], dt = MODE == MODE_RK ? *rk.dt : 0.0;
        const R (*Xx)[XS] = Xb;
        const R (*Xy)[XS] = Xb + NC;
        auto xs = [&](int s) { return nj + TY * (ni + s); };
        auto ys = [&](int s) { return (nj + s) + (TY + 4) * ni; };
#pragma unroll
        for (int i = 0; i < NH; i++) {
            const int cc = c0 + i;
            if (cc > NC) break;
            double dx, dy;
            if (cc < NC) {
                dx = -(double)(Xx[cc][xs(2)] - Xx[cc][xs(1)]) * hx;
                dy = -(double)(Xy[cc][ys(2)] - Xy[cc][ys(1)]) * hy;
            } else {
                auto lx_ = [&](int l) { return l + NEX * (nj + 3); };
                auto ly_ = [&](int l) { return (ni + 3) + NEX * l; };
                double gx = 0.0, gy = 0.0;
#pragma unroll
                for (int m = 1; m <= 3; m++) {
                    gx += ph.alpha[m - 1] * (S.m[0][lx_(ni + 3 + m)] - S.m[0][lx_(ni + 3 - m)]);
                    gy += ph.alpha[m - 1] * (My[0][ly_(nj + 3 + m)] - My[0][ly_(nj + 3 - m)]);
                }
                dx = -gx * hx;   // S.m and My hold half the metrics
                dy = -gy * hy;
            }
            double o = dx + dy;
            if constexpr (MODE != MODE_WRITE) o = o + ac[i];
            if constexpr (MODE == MODE_RK) o = rk.a * qn[i] + rk.b * (qs[i] + dt * o);
            double* out = cc < NC ? (MODE == MODE_RK && rk.outU ? rk.outU : accU) + cc * P
                                  : (MODE == MODE_RK && rk.outJ ? rk.outJ : accJ);
            out[gn] = o;
        }
    }
}

// --------------------------------------------------------------------------
// host-side launch
// --------------------------------------------------------------------------
template <int N, int D, int K, int MODE, typename R, int RC>
static hipError_t launch_dir(const Phys& ph, const Geo& g, const double* JU, const double* J,
                             const double* jxx, const double* jxt, double* accU, double* accJ,
                             const RkArgs& rk, unsigned* status, hipStream_t s)
{
    // tile: TL nodes along k on TC lines.  The x sweep reads its lines along
    // the contiguous index, so a longer tile (24 on 10 lines: 250 interfaces)
    // cuts its halo re-reads (30/24 instead of 22/16 loaded per owned node,
    // -11% time); the y and z sweeps read rows of TC consecutive x values
    // across their lines, so they keep 15 lines (120-byte rows) of 16 nodes
    constexpr int TL = (K == 0) ? 24 : 16;
    constexpr int TC = (K == 0) ? 10 : 15;
    constexpr int FA = (K == 0) ? 1 : 0;
    constexpr int SA = (K == 2) ? 1 : 2;
    const long nseg = (g.n[K] + TL - 1) / TL;
    const long nlines = (long)g.n[FA] * ((SA < D) ? g.n[SA] : 1);
    const long nblk = nseg * ((nlines + TC - 1) / TC);
    if (nblk > 0x7fffffffL || nlines + TC > 0x7fffffffL) return hipErrorInvalidConfiguration;
    dim3 grid((unsigned)nblk);
    hipLaunchKernelGGL((k_rhs_dir<N, D, K, TL, TC, MODE, R, RC>), grid, dim3(256), 0, s, ph, g, JU, J,
                       jxx, jxt, accU, accJ, rk, status);
    return hipGetLastError();
}

// the x and y directions of a 3D grid in one launch (k_rhs_xy)
template <int N, int MODE, typename R, int RC, int MG>
static hipError_t launch_xy(const Phys& ph, const Geo& g, const double* JU, const double* J,
                            const double* jxx, const double* jxt, double* accU, double* accJ,
                            const RkArgs& rk, unsigned* status, hipStream_t s)
{
    constexpr int TX = 16, TY = 15;
    const long gx = (g.n[0] + TX - 1) / TX, gy = (g.n[1] + TY - 1) / TY, gz = g.n[2];
    if (g.ng < 3 || gx * gy * gz > 0x7fffffffL || gy > 65535 || gz > 65535) return hipErrorInvalidConfiguration;
    hipLaunchKernelGGL((k_rhs_xy<N, TX, TY, MODE, R, RC, MG>), dim3((unsigned)gx, (unsigned)gy, (unsigned)gz), dim3(512), 0, s,
                       ph, g, JU, J, jxx, jxt, accU, accJ, rk, status);
    return hipGetLastError();
}

template <int N, int D, typename R, int RC>
static hipError_t rhs_all(const Phys& ph, const Geo& g, const double* JU, const double* J,
                          const double* jxx, const double* jxt, double* outU, double* outJ,
                          const RkArgs* rk, unsigned* status, hipStream_t s)
{
    RkArgs none{nullptr, nullptr, nullptr, 0.0, 0.0};
    if (rk) none.tdiv = rk->tdiv;
    // 3D: the z sweep, then x and y in one launch with the stage combination
    // (two field groups in the FP32 dissipation, which keeps that launch at 90
    // registers)
    if constexpr (D == 3) {
        hipError_t e = launch_dir<N, D, 2, MODE_WRITE, R, RC>(ph, g, JU, J, jxx, jxt, outU, outJ, none, status, s);
        if (e != hipSuccess) return e;
        if (rk) return launch_xy<N, MODE_RK, R, RC, 2>(ph, g, JU, J, jxx, jxt, outU, outJ, *rk, status, s);
        return launch_xy<N, MODE_ADD, R, RC, 2>(ph, g, JU, J, jxx, jxt, outU, outJ, none, status, s);
    } else {
        hipError_t e = launch_dir<N, D, 0, MODE_WRITE, R, RC>(ph, g, JU, J, jxx, jxt, outU, outJ, none,
                                                          status, s);
        if (e != hipSuccess) return e;
        if constexpr (D == 2) {
            if (rk) return launch_dir<N, D, 1, MODE_RK, R, RC>(ph, g, JU, J, jxx, jxt, outU, outJ, *rk, status, s);
            return launch_dir<N, D, 1, MODE_ADD, R, RC>(ph, g, JU, J, jxx, jxt, outU, outJ, none, status, s);
        } else {
            e = launch_dir<N, D, 1, MODE_ADD, R, RC>(ph, g, JU, J, jxx, jxt, outU, outJ, none, status, s);
            if (e != hipSuccess) return e;
            if (rk) return launch_dir<N, D, 2, MODE_RK, R, RC>(ph, g, JU, J, jxx, jxt, outU, outJ, *rk, status, s);
            return launch_dir<N, D, 2, MODE_ADD, R, RC>(ph, g, JU, J, jxx, jxt, outU, outJ, none, status, s);
        }
    }
}

hipError_t launch_rhs(const Phys& ph, const Geo& g, int mixed, const double* JU, const double* J,
                      const double* jxx, const double* jxt, double* outU, double* outJ,
                      const RkArgs* rk, unsigned* status, hipStream_t s)
{
#define ES_RHS_CASE(NN_, DD_)                                                                          \
    if (ph.nspec == NN_ && g.dim == DD_) {                                                             \
        if (ph.recon == 1) {   /* classical WENO5: FP64 only (checked at create) */                 \
            if (mixed) return hipErrorInvalidValue;                                                    \
            return rhs_all<NN_, DD_, double, 1>(ph, g, JU, J, jxx, jxt, outU, outJ, rk, status, s);   \
        }                                                                                              \
        if (mixed) return rhs_all<NN_, DD_, float, 0>(ph, g, JU, J, jxx, jxt, outU, outJ, rk, status, s); \
        return rhs_all<NN_, DD_, double, 0>(ph, g, JU, J, jxx, jxt, outU, outJ, rk, status, s);       \
    }
    ES_RHS_CASE(1, 2)
    ES_RHS_CASE(2, 2)
    ES_RHS_CASE(1, 3)
    ES_RHS_CASE(2, 3)
#undef ES_RHS_CASE
    return hipErrorInvalidValue;
}

}  // namespace es

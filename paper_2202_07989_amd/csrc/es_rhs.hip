// es_rhs.hip -- the semi-discrete right-hand side (Sections 3.1-3.4) and the
// fused SSP-RK3 stage (Section 5) on gfx950.
//
// A 2D stage is one launch (k_rhs_xy).  A 3D stage takes the z sweep (k_rhs_z),
// which writes its term, and then k_rhs_xy, which adds the x and y terms and
// applies the stage combination: the z sweep is bound by HBM (its halo along
// z is read again by every tile), the x-y launch by FP64 issue, so the operands
// of the combination are read beside the latter (2.84 against 3.11 ms a stage
// at 256^3 with the combination in the z sweep).  Every block stages node
// quantities in LDS and builds the full numerical flux at its interfaces, one
// thread per interface:
//   F_{i+1/2} = sum_m alpha_m sum_{s<m} F(i-s, i-s+m)  -  D_{i+1/2}
// (the interface form of eq ECFlux_curv_2p minus the ES dissipation
// 1/2 s T^T R Y [[W]]^WENO of eq HOstable).  Each two-point flux
// F(a, a+m) is evaluated once, by the thread whose interface has left node
// a; the m interfaces that use it collect it through an LDS exchange in
// three barrier-separated steps.  The node's term is the interface
// difference plus the GCL term delta_k[n_t] (eq GCL_flux), times -1/dxi_k.
#include "es_tile.hpp"

namespace es {

// The z sweep.  A block of 256 threads owns TL nodes along z on TC lines of
// consecutive x (16 on 15: 255 interfaces, rows of 120 bytes) plus a 3-node
// halo along z.  What bounds it: HBM (5.4 GB in 1.2 ms at 256^3 with the stage
// combination here, 3.1 GB in 0.89 ms without) and the latency of its loads
// and barriers, hidden by four blocks a compute unit (39.7 KB of LDS, 118
// registers for two species).  Waves per SIMD: four in FP64, three in FP32
// (one field group: splitting it costs more than a fourth wave gains).
template <int N, int TL, int TC, typename R, int RC>
__global__ void __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(sizeof(R) == 8 ? 4 : 3, 8)))
k_rhs_z(Phys ph, Geo g, const double* __restrict__ JU, const double* __restrict__ Jv,
        const double* __restrict__ jxx, const double* __restrict__ jxt, double* __restrict__ outU,
        double* __restrict__ outJ, const double* __restrict__ tdiv, unsigned* __restrict__ status)
{
    constexpr int D = 3, K = 2;
    constexpr int NT = 256;
    constexpr int NC = N + D + 1;
    constexpr int NL = TL + 6;          // nodes per line: tile + 3-node halo on each side
    constexpr int NN = NL * TC;
    constexpr int NI = (TL + 1) * TC;   // interfaces (one thread each)
    constexpr int NS = TL + 4;          // exchange slots per line
    constexpr int NX = NS * TC;
    static_assert(NI <= NT && 3 * TC <= 64 && TL * TC <= NT, "tile does not fit the block");
    __shared__ NodeTile<N, D, NN, R> S;
    // the flux exchange overlays the node quantities (not the metrics, which
    // the GCL term reads afterwards), so four blocks share a compute unit
    static_assert(sizeof(R) * NC * NX <= sizeof(S) - sizeof(S.m), "exchange does not fit the tile");
    R (*X)[NX] = reinterpret_cast<R (*)[NX]>(&S.rho[0][0]);

    const long P = g.P;
    const int nK = g.n[2], nF = g.n[0];
    const long nlines = (long)nF * g.n[1];
    const int nseg = (nK + TL - 1) / TL;
    const int seg0 = (int)(blockIdx.x % nseg) * TL;
    const long line0 = (long)(blockIdx.x / nseg) * TC;
    const long sK = dir_stride(g, K);
    const int t = threadIdx.x;

    // LDS layouts are line-fastest, so the lanes of a wave (consecutive lines)
    // read consecutive words
    auto lidx = [](int l, int c) { return c + TC * l; };
    auto xidx = [](int s, int c) { return c + TC * s; };
    // padded index of the node at along-index 0 of each line of the block,
    // tabulated once (the line index splits into the two across indices by a
    // division)
    __shared__ long s_base[TC];
    if (t < TC) {
        const int L = (int)line0 + t;
        s_base[t] = node_index(g, g.ng + L % nF, g.ng + L / nF, 0);
    }
    __syncthreads();

    // ---- phase 1: node quantities of the tile (+ halo) into LDS ----------
    // all loads of the thread's nodes are issued before the first is used:
    // the block then waits for memory once
    unsigned bad = 0;
    const double itd = tdiv ? 1.0 / *tdiv : 1.0;
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
            const int l = q / TC;
            const int c = q % TC;
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
    interface_fluxes<N, D, NN, TL, TC, RC, R>(ph, S, X, lidx, xidx,
                                          [&](int c) { return line0 + c < nlines; }, fi, fc, f_ok,
                                          t - (int)(blockIdx.x & 3) * 64);

    // ---- phase 3: interface differences at the tile's nodes --------------
    if (t < TL * TC) {
        const int lo = t / TC;
        const int c = t % TC;
        if (seg0 + lo < nK && line0 + c < nlines) {
            const int l = lo + 3;
            double gcl = 0.0;
#pragma unroll
            for (int m = 1; m <= 3; m++)
                gcl += ph.alpha[m - 1] * (S.m[0][lidx(l + m, c)] - S.m[0][lidx(l - m, c)]);
            const long gi = s_base[c] + (g.ng + seg0 + lo) * sK;
            const double h = g.idxi[K];
#pragma unroll
            for (int cc = 0; cc < NC; cc++)
                outU[cc * P + gi] = -(double)(X[cc][xidx(lo + 2, c)] - X[cc][xidx(lo + 1, c)]) * h;
            outJ[gi] = -gcl * h;   // S.m holds half the metrics
        }
    }
}

enum { MODE_WRITE = 0, MODE_ADD = 1, MODE_RK = 2 };

// The x and y directions of a grid (xy_tile), written (2D right-hand side),
// added to the z term in the output (3D), or with the Shu-Osher combination
// (in 3D of the accumulated z term too).  A 2D stage takes one launch
// instead of two sweeps with the accumulator between them: 32.0 against 38.2 us
// at 512^2 (two species), 9.9 against 17.2 us at 64^2 (one species).
template <int N, int D, int TX, int TY, int MODE, typename R, int RC, int MG>
__global__ void __launch_bounds__(512) __attribute__((amdgpu_waves_per_eu(4, 8)))
k_rhs_xy(Phys ph, Geo g, const double* __restrict__ JU, const double* __restrict__ Jv,
         const double* __restrict__ jxx, const double* __restrict__ jxt, double* accU, double* accJ, RkArgs rk,
         unsigned* __restrict__ status)
{
    constexpr int NC = N + D + 1, NN = (TX + 6) * (TY + 6), NH = NC / 2 + 1;
    constexpr bool ACC = MODE == MODE_ADD || (MODE == MODE_RK && D == 3);
    __shared__ NodeTile<N, D, NN, R> S;
    __shared__ double My[D + 1][NN];
    const long P = g.P;
    int bx, by, bz;
    xcd_plane<D>((g.n[0] + TX - 1) / TX, (g.n[1] + TY - 1) / TY, bx, by, bz);
    const int ox = bx * TX, oy = by * TY;
    const PlaneIn in{JU, Jv, jxx, jxt, rk.tdiv ? 1.0 / *rk.tdiv : 1.0, P, g.ng, g.np[0], g.np[1], g.n[0], g.n[1]};
    // padded index of patch node (0, 0), at interior (ox - 3, oy - 3) of plane bz
    const long base = ((long)(D == 3 ? g.ng + bz : 0) * g.np[1] + (oy + g.ng - 3)) * g.np[0] + (ox + g.ng - 3);
    double ac[NH], qs[NH], qn[NH];
    const double dt = MODE == MODE_RK ? *rk.dt : 0.0;
    const unsigned bad = xy_tile<N, D, TX, TY, 512, R, RC, MG>(
        ph, S, My, in, ox, oy, base, g.idxi[0], g.idxi[1], (int)blockIdx.x,
        [&](int i, int cc, long gn) {
            const bool isJ = cc == NC;
            if constexpr (ACC) ac[i] = (isJ ? accJ : accU + cc * P)[gn];
            if constexpr (MODE == MODE_RK) {
                qs[i] = (isJ ? Jv : JU + cc * P)[gn];
                // stage 0 has a = 0: Q_s stands in for Q_n, which is not read
                const double* nU = rk.a != 0.0 ? rk.JUn : JU;
                const double* nJ = rk.a != 0.0 ? rk.Jn : Jv;
                qn[i] = (isJ ? nJ : nU + cc * P)[gn];
            }
        },
        [&](int i, int cc, long gn, int ni, int nj, double o) {
            if constexpr (ACC) o = o + ac[i];
            if constexpr (MODE == MODE_RK) o = rk.a * qn[i] + rk.b * (qs[i] + dt * o);
            double* to = cc < NC ? (MODE == MODE_RK && rk.outU ? rk.outU : accU) + cc * P
                                 : (MODE == MODE_RK && rk.outJ ? rk.outJ : accJ);
            to[gn] = o;
            if constexpr (D == 2 && MODE == MODE_RK) {
                if (rk.images)   // J and J U wrapped or mirrored, momentum k negated across a wall of direction k
                    for_images<2>(g, ox + ni, oy + nj, 0, [&](const int (&side)[3], long gi) {
                        const int k = cc - N;
                        const bool neg = k >= 0 && k < 2 && cc < NC && side[k == 1] != 0 &&
                                         g.bc[k == 1][side[k == 1] > 0] == BC_REFLECT;
                        to[gi] = neg ? -o : o;
                    });
            }
        });
    if (bad) atomicOr(status, bad);
}

// --------------------------------------------------------------------------
// host-side launch
// --------------------------------------------------------------------------
template <int N, typename R, int RC>
static hipError_t launch_z(const Phys& ph, const Geo& g, const double* JU, const double* J, const double* jxx,
                           const double* jxt, double* outU, double* outJ, const double* tdiv, unsigned* status,
                           hipStream_t s)
{
    // 16 nodes on 15 lines: longer tiles re-read less halo but read narrower rows
    constexpr int TL = 16, TC = 15;
    const long nseg = (g.n[2] + TL - 1) / TL;
    const long nlines = (long)g.n[0] * g.n[1];
    const long nblk = nseg * ((nlines + TC - 1) / TC);
    if (nblk > 0x7fffffffL || nlines + TC > 0x7fffffffL) return hipErrorInvalidConfiguration;
    hipLaunchKernelGGL((k_rhs_z<N, TL, TC, R, RC>), dim3((unsigned)nblk), dim3(256), 0, s, ph, g, JU, J, jxx, jxt,
                       outU, outJ, tdiv, status);
    return hipGetLastError();
}

template <int N, int D, int MODE, typename R, int RC>
static hipError_t launch_xy(const Phys& ph, const Geo& g, const double* JU, const double* J,
                            const double* jxx, const double* jxt, double* accU, double* accJ,
                            const RkArgs& rk, unsigned* status, hipStream_t s)
{
    constexpr int TX = 16, TY = 15;
    const long gx = (g.n[0] + TX - 1) / TX, gy = (g.n[1] + TY - 1) / TY, gz = D == 3 ? g.n[2] : 1;
    if (g.ng < 3 || gx * gy * gz > 0x7fffffffL) return hipErrorInvalidConfiguration;
    // two field groups in the FP32 dissipation keep that launch at 90 registers
    hipLaunchKernelGGL((k_rhs_xy<N, D, TX, TY, MODE, R, RC, 2>), dim3((unsigned)(gx * gy * gz)), dim3(512), 0, s, ph, g, JU, J, jxx, jxt,
                       accU, accJ, rk, status);
    return hipGetLastError();
}

template <int N, int D, typename R, int RC>
static hipError_t rhs_all(const Phys& ph, const Geo& g, const double* JU, const double* J,
                          const double* jxx, const double* jxt, double* outU, double* outJ,
                          const RkArgs* rk, unsigned* status, hipStream_t s)
{
    const RkArgs none{nullptr, nullptr, nullptr, 0.0, 0.0};
    if constexpr (D == 3) {
        const hipError_t e = launch_z<N, R, RC>(ph, g, JU, J, jxx, jxt, outU, outJ, rk ? rk->tdiv : nullptr, status, s);
        if (e != hipSuccess) return e;
        if (!rk) return launch_xy<N, D, MODE_ADD, R, RC>(ph, g, JU, J, jxx, jxt, outU, outJ, none, status, s);
    } else {
        if (!rk) return launch_xy<N, D, MODE_WRITE, R, RC>(ph, g, JU, J, jxx, jxt, outU, outJ, none, status, s);
    }
    return launch_xy<N, D, MODE_RK, R, RC>(ph, g, JU, J, jxx, jxt, outU, outJ, *rk, status, s);
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

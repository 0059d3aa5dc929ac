// es_tile.hpp -- the x and y directions of one tile of a plane by one block:
// shared by the single-grid launch of es_rhs.hip and the batched stage of
// es_batch.hip.
#pragma once
#include "es_flux.hpp"

namespace es {

// grid of the plane a tile lies in: J U, J and the metrics of directions 0
// and 1 (jt: the time metrics, null on a fixed mesh; read times itd), P the component
// stride, base the padded index of patch node (0, 0)
struct PlaneIn {
    const double *JU, *J, *jxx, *jxt;
    double itd;
    long P;
    int ng, np0, np1, nx, ny;
};

// A block of NT threads owns the TX x TY tile at (ox, oy) of a plane.  It
// stages the node quantities of the tile plus a 3-node halo along x and y (a
// plus-shaped patch; the corners are never read) and the halved metrics of
// both directions in LDS once; then the first half of its waves builds the x
// fluxes of the tile's TY rows and the second half the y fluxes of its TX
// columns at the same time, each with the interface scheme of
// interface_fluxes.  A node's term is the x difference plus the y difference,
// each rounded on its own.  Each half of the block writes half of the
// components (J U, then J) of the tile's nodes: fetch(i, cc, gn) runs before the
// exchange (component cc of padded node gn, the thread's i-th) and
// out(i, cc, gn, ni, nj, term) writes.  rot spreads the pairs
// left of a line's first interface over the waves.  Bound by FP64 issue and by
// the waits of a block's phases; two blocks of 512 threads (70 KB, 123
// registers for two species in 3D) share a compute unit.  Returns the status
// bits of the thread's node.
template <int N, int D, int TX, int TY, int NT, typename R, int RC, int MG, int NN, typename FETCH, typename OUT>
__device__ __forceinline__ unsigned xy_tile(const Phys& ph, NodeTile<N, D, NN, R>& S, double (*My)[NN],
                                            const PlaneIn& in, int ox, int oy, long base, double hx, double hy,
                                            int rot, FETCH fetch, OUT out)
{
    constexpr int NC = N + D + 1;
    constexpr int NEX = TX + 6, NEY = TY + 6;
    constexpr int XSX = (TX + 4) * TY, XSY = (TY + 4) * TX;    // exchange slots per component
    constexpr int XS = XSX > XSY ? XSX : XSY;
    static_assert(NN == NEX * NEY && NN <= NT, "one node a thread");
    static_assert((TX + 1) * TY <= NT / 2 && (TY + 1) * TX <= NT / 2 && 3 * TX <= 64 && 3 * TY <= 64 &&
                      NT % 128 == 0, "tile does not fit the block");
    // (S.m: the x metrics, My: the y metrics; the exchange overlays the rest)
    static_assert(sizeof(R) * 2 * NC * XS <= sizeof(S) - sizeof(S.m), "exchange does not fit the tile");
    R (*Xb)[XS] = reinterpret_cast<R (*)[XS]>(&S.rho[0][0]);   // x rows 0..NC-1, y rows NC..2NC-1
    const long P = in.P;
    const int ng = in.ng, np0 = in.np0, np1 = in.np1;
    int t = threadIdx.x;
    asm volatile("" : "+v"(t));   // (a caller's loop shall not keep what derives from it in registers)

    // ---- node quantities and metrics of the patch -------------------------
    // one node a thread, all of its loads issued before the first is used
    unsigned bad = 0;
    {
        const int lx = t % NEX, ly = t / NEX;
        const bool cx = lx >= 3 && lx < 3 + TX, cy = ly >= 3 && ly < 3 + TY;
        // corners are never read, nodes beyond a ragged tile do not exist
        const bool have = t < NN && (cx || cy) && ox + lx - 3 + ng < np0 && oy + ly - 3 + ng < np1;
        const long gi = base + (long)ly * np0 + lx;
        if (have) {
            NodeRaw<NC> raw;
            double mx[D + 1], my[D + 1];
            node_load<NC>(raw, in.JU, in.J, P, gi);
            const double* __restrict__ jxx = in.jxx;
            const double* __restrict__ jt = in.jxt ? in.jxt : jxx;   // (a fixed mesh reads it and drops it)
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
                S.m[0][t] = in.jxt ? 0.5 * (mx[0] * in.itd) : 0.0;
#pragma unroll
                for (int j = 0; j < D; j++) S.m[1 + j][t] = 0.5 * mx[1 + j];
            }
            if (cx) {
                My[0][t] = in.jxt ? 0.5 * (my[0] * in.itd) : 0.0;
#pragma unroll
                for (int j = 0; j < D; j++) My[1 + j][t] = 0.5 * my[1 + j];
            }
        }
    }
    __syncthreads();

    // ---- interface fluxes: x in the first half, y in the second ----
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
    const int n_line = ydir ? in.nx : in.ny, np_along = ydir ? np1 : np0;
    const bool f_ok = (u < (TL + 1) * TC) && (o_line + fc < n_line) && (o_along + fi + 2 + ng < np_along);
    // one copy of the arithmetic for both directions, the tile strides,
    // metric array and exchange rows picked per wave (compiling each
    // direction's arithmetic on its own under a branch took 4 % longer: the
    // join spills registers)
    const int sl = ydir ? NEX : 1, sc = ydir ? 1 : NEX, l0 = ydir ? 3 : 3 * NEX;
    const int xl = ydir ? 1 : TY, xc = ydir ? TY + 4 : 1;
    constexpr int NH = NC / 2 + 1;
    const int ni = u % TX, nj = u / TX, c0 = ydir ? NH : 0;
    const bool own = u < TX * TY && ox + ni < in.nx && oy + nj < in.ny;
    const long gn = own ? base + (long)(nj + 3) * np0 + (ni + 3) : base + 3L * np0 + 3;
    interface_fluxes_m<N, D, NN, XS, RC, R, MG>(
        ph, S, ydir ? My : S.m, ydir ? Xb + NC : Xb, [=](int l, int c) { return l0 + l * sl + c * sc; },
        [=](int s, int c) { return s * xl + c * xc; }, [=](int c) { return o_line + c < n_line; }, fi, fc,
        f_ok, u - (rot % (NT / 128)) * 64, TL, TC, [&] {
#pragma unroll
            for (int i = 0; i < NH; i++) fetch(i, c0 + i < NC ? c0 + i : NC, gn);
        });

    // ---- node outputs ------------------------------------------------------
    if (own) {
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
            out(i, cc, gn, ni, nj, dx + dy);
        }
    }
    return bad;
}

}  // namespace es

// es_batch.hip -- one SSP-RK3 stage (Section 5) of many independent 2D
// instances of uneven size in one launch; each instance is the
// semi-discrete scheme of Sections 3.1-3.4 on its own periodic grid.
//
// The work list holds regions of TX x TY nodes of every instance (the
// autotuner picks the shape).  A block builds the x and y terms of a region
// with xy_tile, both directions at once, and writes the Shu-Osher
// combination to the region's nodes and their periodic ghost images, so the
// next stage reads complete ghost layers with no fill.  A region's right-hand
// side depends only on its patch, so regions need no ordering and the launch
// has no grid-wide synchronisation.  LOOP: a persistent grid whose blocks take
// regions round-robin; else one block per region (the faster one here).  On
// the 64-instance batch (15.5 M cells, water / air) a stage of 16 x 15 regions
// takes 1.48 ms against 2.28 ms with the same arithmetic and the directions
// swept one after the other by 256 threads (two waves a SIMD: the right-hand
// sides stayed in registers across the sweeps).
#include "es_tile.hpp"

namespace es {

template <int N, int TX, int TY, int NT, bool LOOP, typename R, int RC>
__global__ void __launch_bounds__(NT) __attribute__((amdgpu_waves_per_eu(4, 8)))
k_stage2d_batched(Phys ph, const Geo* __restrict__ geos, const int4* __restrict__ tiles, int ntiles,
                  BatchTables tb, double ca, double cb, const double* __restrict__ dt_dev,
                  unsigned* __restrict__ status)
{
    constexpr int D = 2;
    constexpr int NC = N + D + 1, NN = (TX + 6) * (TY + 6), NH = NC / 2 + 1;
    __shared__ NodeTile<N, D, NN, R> S;
    __shared__ double My[D + 1][NN];
    unsigned bad = 0;
    for (int w = blockIdx.x; w < ntiles; w += gridDim.x) {
        const int4 tw = tiles[w];
        const int bi = tw.x, ox = tw.y, oy = tw.z;
        const Geo& g = geos[bi];
        const long P = g.P;
        const int nx = g.n[0], ny = g.n[1], np0 = g.np[0], ng = g.ng;
        const PlaneIn in{tb.JUs[bi], tb.Js[bi], tb.jxx[bi], tb.jxt ? tb.jxt[bi] : nullptr, 1.0, P, ng, np0,
                         g.np[1], nx, ny};
        const double dt = dt_dev[bi];
        const double* __restrict__ JUn = tb.JUn[bi];
        const double* __restrict__ Jn = tb.Jn[bi];
        double* JUo = tb.JUo[bi];
        double* Jo = tb.Jo[bi];
        const long base = (long)(oy + ng - 3) * np0 + (ox + ng - 3);
        double qs[NH], qn[NH];
        bad |= xy_tile<N, D, TX, TY, NT, R, RC, 2>(
            ph, S, My, in, ox, oy, base, g.idxi[0], g.idxi[1], w,
            [&](int i, int cc, long gn) {
                const bool isJ = cc == NC;
                qs[i] = (isJ ? in.J : in.JU + cc * P)[gn];
                // stage 0 has ca = 0: Q_s stands in for the state at t^n, which is not read
                const double* nU = ca != 0.0 ? JUn : in.JU;
                const double* nJ = ca != 0.0 ? Jn : in.J;
                qn[i] = (isJ ? nJ : nU + cc * P)[gn];
            },
            [&](int i, int cc, long gn, int ni, int nj, double L) {
                // the node and its ghost images
                const double o = ca * qn[i] + cb * (qs[i] + dt * L);
                double* to = cc < NC ? JUo + cc * P : Jo;
                to[gn] = o;
                const int gx = ox + ni, gy = oy + nj;
                if (gx < ng || gx >= nx - ng || gy < ng || gy >= ny - ng) {
#pragma unroll 1
                    for (int k = 0; k < 9; k++) {
                        const int xx = gx + (k % 3 - 1) * nx, yy = gy + (k / 3 - 1) * ny;
                        if (k != 4 && xx >= -ng && xx < nx + ng && yy >= -ng && yy < ny + ng)
                            to[(long)(yy + ng) * np0 + (xx + ng)] = o;
                    }
                }
            });
        if constexpr (!LOOP) break;
        __syncthreads();   // the next region overwrites the patch
    }
    if (bad) atomicOr(status, bad);
}

// the region shapes of the autotuner's search: (TX, TY, threads); each
// direction of a shape has at most half as many interfaces as threads
#define ES_BATCH_SHAPES(X) X(0, 10, 10, 256) X(1, 15, 15, 512) X(2, 16, 15, 512) X(3, 15, 16, 512) \
                           X(4, 18, 13, 512) X(5, 21, 21, 1024)

int batch_nshapes() { return 6; }

void batch_shape(int v, int* tx, int* ty, int* nt)
{
#define ES_SHAPE(V_, TX_, TY_, NT_) if (v == V_) { *tx = TX_; *ty = TY_; *nt = NT_; return; }
    ES_BATCH_SHAPES(ES_SHAPE)
#undef ES_SHAPE
    *tx = *ty = *nt = 0;
}

template <int N, typename R, int RC>
static hipError_t launch_variant(int v, const Phys& ph, const Geo* geos, const BatchTiling& tl,
                                 const BatchTables& tb, double ca, double cb, const double* dt_dev,
                                 unsigned* status, hipStream_t s)
{
#define ES_BATCH_CASE(V_, TX_, TY_, NT_)                                                             \
    if (v == V_) {                                                                                   \
        if (tl.blocks < tl.ntiles)                                                                   \
            hipLaunchKernelGGL((k_stage2d_batched<N, TX_, TY_, NT_, true, R, RC>), dim3(tl.blocks), dim3(NT_), 0, \
                               s, ph, geos, tl.tiles, tl.ntiles, tb, ca, cb, dt_dev, status);        \
        else                                                                                         \
            hipLaunchKernelGGL((k_stage2d_batched<N, TX_, TY_, NT_, false, R, RC>), dim3(tl.blocks), dim3(NT_), 0, \
                               s, ph, geos, tl.tiles, tl.ntiles, tb, ca, cb, dt_dev, status);        \
        return hipGetLastError();                                                                    \
    }
    ES_BATCH_SHAPES(ES_BATCH_CASE)
#undef ES_BATCH_CASE
    return hipErrorInvalidValue;
}

template <int N, typename R, int RC>
static hipError_t occupancy_variant(int v, int* blocks_per_cu)
{
#define ES_OCC_CASE(V_, TX_, TY_, NT_)                                                               \
    if (v == V_)                                                                                     \
        return hipOccupancyMaxActiveBlocksPerMultiprocessor(blocks_per_cu,                          \
                                                            k_stage2d_batched<N, TX_, TY_, NT_, true, R, RC>, NT_, 0);
    ES_BATCH_SHAPES(ES_OCC_CASE)
#undef ES_OCC_CASE
    return hipErrorInvalidValue;
}

hipError_t batch_occupancy(int nspec, int mixed, int recon, int v, int* blocks_per_cu)
{
    if (recon == 1) {   // classical WENO5: FP64 only
        if (mixed) return hipErrorInvalidValue;
        return nspec == 1 ? occupancy_variant<1, double, 1>(v, blocks_per_cu)
                          : occupancy_variant<2, double, 1>(v, blocks_per_cu);
    }
    if (nspec == 1)
        return mixed ? occupancy_variant<1, float, 0>(v, blocks_per_cu) : occupancy_variant<1, double, 0>(v, blocks_per_cu);
    return mixed ? occupancy_variant<2, float, 0>(v, blocks_per_cu) : occupancy_variant<2, double, 0>(v, blocks_per_cu);
}

hipError_t launch_stage_batched(const Phys& ph, const Geo* geos, int mixed, const BatchTiling& tl,
                                const BatchTables& tb, double ca, double cb, const double* dt_dev,
                                unsigned* status, hipStream_t s)
{
    if (tl.ntiles == 0) return hipSuccess;
    if (ph.recon == 1) {   // classical WENO5: FP64 only (checked at create)
        if (mixed) return hipErrorInvalidValue;
        return ph.nspec == 1 ? launch_variant<1, double, 1>(tl.v, ph, geos, tl, tb, ca, cb, dt_dev, status, s)
                             : launch_variant<2, double, 1>(tl.v, ph, geos, tl, tb, ca, cb, dt_dev, status, s);
    }
    if (ph.nspec == 1)
        return mixed ? launch_variant<1, float, 0>(tl.v, ph, geos, tl, tb, ca, cb, dt_dev, status, s)
                     : launch_variant<1, double, 0>(tl.v, ph, geos, tl, tb, ca, cb, dt_dev, status, s);
    return mixed ? launch_variant<2, float, 0>(tl.v, ph, geos, tl, tb, ca, cb, dt_dev, status, s)
                 : launch_variant<2, double, 0>(tl.v, ph, geos, tl, tb, ca, cb, dt_dev, status, s);
}

}  // namespace es

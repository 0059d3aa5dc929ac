// es_kernels.hip -- the HBM-bound steps of the path on gfx950: ghost
// layers, GCL metrics (Section 3.2), the CFL wave speed (Section 5),
// mesh redistribution (Section 4) and the FP64 entropy sums.
#include "es_kernels.hpp"

namespace es {

// ---------------------------------------------------------------------------
// Ghost layers in one launch per field: every ghost node (the shell of the
// padded box: the z slabs, then the y slabs over interior z, then the x slabs
// over interior y and z) takes the value of one interior node, with all of
// its out-of-range coordinates mapped at once.
//
// Periodic faces wrap (the mesh gains -L_k / +L_k in component k below /
// above the interior along k).  The boundary conditions of the paper's
// walled examples (reflecting walls, outflow, inflow) are taken with
// cell-centred nodes: the face lies halfway between the outermost node and
// the first ghost node, and the ghost node m layers outside mirrors the
// interior node m - 1 layers inside.  Across such a face the mesh is
// mirrored about the face's coordinate (x_k -> 2 wall - x_k), displacements
// and time metrics negate component k, and a metric J dxi_a/dx_b is negated
// when exactly one of a, b is k: the values the mirrored mesh has.  The
// state is filled by fill_state.
// ---------------------------------------------------------------------------
// (index arithmetic in 32 bits: a grid holds fewer than 2^31 / 9 points,
// which the context checks at creation, and 64-bit division is a long
// software sequence on the GPU)
__device__ __forceinline__ void shell_node(const Geo& g, long t, long nzs, long nys, int d[3])
{
    const unsigned ng = g.ng;
    const unsigned np0 = g.np[0], np1 = g.np[1];
    const unsigned n0 = g.n[0], n1 = g.n[1], n2 = g.n[2];
    const int z0 = g.dim == 3 ? (int)ng : 0;
    if (t < nzs) {                                   // z ghost planes
        const unsigned u = (unsigned)t, pl = np0 * np1;
        const unsigned k = u / pl, r = u - k * pl;
        d[2] = (int)(k < ng ? k : k + n2);
        const unsigned y = r / np0;
        d[1] = (int)y;
        d[0] = (int)(r - y * np0);
    } else if (t < nzs + nys) {                      // y ghost rows over interior z
        const unsigned u = (unsigned)(t - nzs), per = 2u * ng * np0;
        const unsigned zz = u / per, r = u - zz * per;
        d[2] = z0 + (int)zz;
        const unsigned k = r / np0;
        d[1] = (int)(k < ng ? k : k + n1);
        d[0] = (int)(r - k * np0);
    } else {                                         // x ghost columns over interior y, z
        const unsigned u = (unsigned)(t - nzs - nys), w = 2u * ng;
        const unsigned row = u / w, k = u - row * w;
        d[0] = (int)(k < ng ? k : k + n0);
        const unsigned zz = row / n1;
        d[1] = (int)(ng + (row - zz * n1));
        d[2] = z0 + (int)zz;
    }
}

// interior image of padded index i along k; side = -1 / +1 below / above
// the interior, 0 inside
__device__ __forceinline__ int ghost_image(const Geo& g, int k, int i, int& side)
{
    const int n = g.n[k], r = i - g.ng;
    side = r < 0 ? -1 : (r >= n ? 1 : 0);
    if (!side) return i;
    if (g.bc[k][side > 0] == BC_PERIODIC) return (side < 0 ? r + n : r - n) + g.ng;
    return (side < 0 ? -1 - r : 2 * n - 1 - r) + g.ng;
}

// ghost value of component c of a field of kind `what` from its image value v
__device__ __forceinline__ double ghost_value(const Geo& g, int what, int c, const int side[3], double v)
{
    for (int k = 0; k < g.dim; k++) {
        if (!side[k]) continue;
        if (g.bc[k][side[k] > 0] == BC_PERIODIC) {
            if (what == GH_MESH && c == k) v += side[k] * g.len[k];
            continue;
        }
        if (what == GH_MESH && c == k) v = 2.0 * g.wall[k][side[k] > 0] - v;
        if ((what == GH_DISP || what == GH_JXT) && c == k) v = -v;
        if (what == GH_JXX && ((c / g.dim == k) != (c % g.dim == k))) v = -v;
    }
    return v;
}

// ghost_value with the field's kind and component known at compile time
template <int WHAT, int D>
__device__ __forceinline__ double ghost_of(const Geo& g, int c, const int (&side)[3], double v)
{
#pragma unroll
    for (int k = 0; k < D; k++) {
        if constexpr (WHAT == GH_PLAIN) break;
        const bool hit = WHAT == GH_JXX ? ((c / D == k) != (c % D == k)) : c == k;
        if (!hit || !side[k]) continue;
        const bool hi = side[k] > 0, per = g.bc[k][hi] == BC_PERIODIC;
        if constexpr (WHAT == GH_MESH) {
            const double sg = per ? 1.0 : -1.0;
            const double off = per ? (hi ? g.len[k] : -g.len[k]) : 2.0 * (hi ? g.wall[k][1] : g.wall[k][0]);
            v = fma(sg, v, off);
        } else {
            v = per ? v : -v;
        }
    }
    return v;
}

// writes the D-dimensional interior node (i0, i1, i2) of an NCOMP-component
// field and its ghost images under the field's ghost rule
template <int D, int NCOMP, int WHAT>
__device__ __forceinline__ void put_images(const Geo& g, int i0, int i1, int i2, const double (&v)[NCOMP],
                                           double* __restrict__ a)
{
    const int ng = g.ng;
    const int z0 = D == 3 ? ng : 0;
    const long di = node_index(g, i0 + ng, i1 + ng, i2 + z0);
#pragma unroll
    for (int c = 0; c < NCOMP; c++) a[c * g.P + di] = v[c];
    for_images<D>(g, i0, i1, i2, [&](const int (&side)[3], long gi) {
#pragma unroll
        for (int c = 0; c < NCOMP; c++) a[c * g.P + gi] = ghost_of<WHAT, D>(g, c, side, v[c]);
    });
}

// interior coordinate (0 .. n-1) that coordinate i of direction k images, i any
// distance outside, and the mesh rule along the way: the mesh component k at
// i is sg times its value there plus off
__device__ __forceinline__ int mesh_image(const Geo& g, int k, int i, double& sg, double& off)
{
    const int n = g.n[k];
    sg = 1.0;
    off = 0.0;
    while (i < 0 || i >= n) {
        const int hi = i >= n;
        if (g.bc[k][hi] == BC_PERIODIC) {
            i += hi ? -n : n;
            off += sg * (hi ? g.len[k] : -g.len[k]);
        } else {
            i = hi ? 2 * n - 1 - i : -1 - i;
            off += sg * 2.0 * g.wall[k][hi];
            sg = -sg;
        }
    }
    return i;
}

// interior node q (0 .. nint-1) -> padded index
// (32-bit index arithmetic, as in shell_node)
__device__ __forceinline__ long interior_node(const Geo& g, long q, int& i0, int& i1, int& i2)
{
    const unsigned u = (unsigned)q, n0 = g.n[0], n1 = g.n[1];
    const unsigned r = u / n0, z = r / n1;
    i0 = (int)(u - r * n0) + g.ng;
    i1 = (int)(r - z * n1) + g.ng;
    i2 = (int)z + (g.dim == 3 ? g.ng : 0);
    return node_index(g, i0, i1, i2);
}

__device__ __forceinline__ long n_interior(const Geo& g)
{
    return (long)g.n[0] * g.n[1] * (g.dim == 3 ? g.n[2] : 1);
}

// one or two fields (a2 may be null) of their own kinds per launch; the
// first is skipped where skip_a is given and set (metrics kept from the step
// before have their ghost layers already)
__global__ void k_fill_shell(Geo g, double* __restrict__ a, int ncomp, int what, double* __restrict__ a2,
                             int ncomp2, int what2, long nzs, long nys, long nxs, const int* __restrict__ skip_a)
{
    if (skip_a && *skip_a) ncomp = 0;
    const long total = nzs + nys + nxs;
    for (long t = blockIdx.x * (long)blockDim.x + threadIdx.x; t < total; t += (long)gridDim.x * blockDim.x) {
        int d[3];
        shell_node(g, t, nzs, nys, d);
        int sidx[3] = {d[0], d[1], d[2]}, side[3] = {0, 0, 0};
        for (int k = 0; k < g.dim; k++) sidx[k] = ghost_image(g, k, d[k], side[k]);
        const long di = node_index(g, d[0], d[1], d[2]);
        const long si = node_index(g, sidx[0], sidx[1], sidx[2]);
        for (int c = 0; c < ncomp; c++) a[c * g.P + di] = ghost_value(g, what, c, side, a[c * g.P + si]);
        if (a2)
            for (int c = 0; c < ncomp2; c++) a2[c * g.P + di] = ghost_value(g, what2, c, side, a2[c * g.P + si]);
    }
}

// the state's ghosts: J is a plain field (wrapped or mirrored); a
// reflecting wall mirrors U with momentum component k negated, outflow
// copies U of the outermost interior node, inflow takes the face's
// prescribed state (the lowest direction's where several meet); JU = J
// (mirrored) times that U
__device__ __forceinline__ void fill_state_node(const Geo& g, const InflowStates& in, double* __restrict__ JU,
                                                double* __restrict__ J, int nc, int nspec, const int d[3])
{
    int src[3] = {d[0], d[1], d[2]}, img[3] = {d[0], d[1], d[2]};
    int flip = 0, uk = -1, us = 0;
    bool extrap = false;
    for (int k = 0; k < g.dim; k++) {
        int side;
        src[k] = ghost_image(g, k, d[k], side);
        img[k] = src[k];
        if (!side) continue;
        const int kind = g.bc[k][side > 0];
        if (kind == BC_REFLECT) flip |= 1 << k;
        if (kind == BC_OUTFLOW) {
            src[k] = side < 0 ? g.ng : g.ng + g.n[k] - 1;
            extrap = true;
        }
        if (kind == BC_INFLOW && uk < 0) {
            uk = k;
            us = side > 0;
        }
    }
    const long di = node_index(g, d[0], d[1], d[2]);
    const long si = node_index(g, src[0], src[1], src[2]);
    const double Jd = J[node_index(g, img[0], img[1], img[2])];
    J[di] = Jd;
    for (int c = 0; c < nc; c++) {
        double u;
        if (uk >= 0) u = Jd * in.u[uk][us][c];
        else if (extrap) u = Jd * (JU[c * g.P + si] / J[si]);
        else u = JU[c * g.P + si];
        if (uk < 0 && c >= nspec && c < nspec + g.dim && ((flip >> (c - nspec)) & 1)) u = -u;
        JU[c * g.P + di] = u;
    }
}

__global__ void k_fill_state(Geo g, InflowStates in, double* __restrict__ JU, double* __restrict__ J,
                             int nc, int nspec, long nzs, long nys, long nxs)
{
    const long total = nzs + nys + nxs;
    for (long t = blockIdx.x * (long)blockDim.x + threadIdx.x; t < total; t += (long)gridDim.x * blockDim.x) {
        int d[3];
        shell_node(g, t, nzs, nys, d);
        fill_state_node(g, in, JU, J, nc, nspec, d);
    }
}

// The start of a time step in one launch: the ghost layers of the state and of
// the mesh x, and *same cleared unless x (ghost layers included) holds the
// values of the kept mesh mx (a NaN never matches; the step before leaves *same
// set)
__global__ void k_step_begin(Geo g, InflowStates in, double* __restrict__ JU, double* __restrict__ J,
                             double* __restrict__ x, const double* __restrict__ mx, int* __restrict__ same, int nc,
                             int nspec, long nzs, long nys, long nxs)
{
    const long shell = nzs + nys + nxs, total = shell + n_interior(g);
    bool differ = false;
    for (long t = blockIdx.x * (long)blockDim.x + threadIdx.x; t < total; t += (long)gridDim.x * blockDim.x) {
        if (t < shell) {
            int d[3];
            shell_node(g, t, nzs, nys, d);
            fill_state_node(g, in, JU, J, nc, nspec, d);
            int sidx[3] = {d[0], d[1], d[2]}, side[3] = {0, 0, 0};
            for (int k = 0; k < g.dim; k++) sidx[k] = ghost_image(g, k, d[k], side[k]);
            const long di = node_index(g, d[0], d[1], d[2]), si = node_index(g, sidx[0], sidx[1], sidx[2]);
            for (int c = 0; c < g.dim; c++) {
                const double v = ghost_value(g, GH_MESH, c, side, x[c * g.P + si]);
                x[c * g.P + di] = v;
                differ |= !(v == mx[c * g.P + di]);
            }
        } else {
            int i0, i1, i2;
            const long i = interior_node(g, t - shell, i0, i1, i2);
            for (int c = 0; c < g.dim; c++) differ |= !(x[c * g.P + i] == mx[c * g.P + i]);
        }
    }
    if (differ) *same = 0;
}

// its end: the step's scalars to the caller's (where given), x^{n+1} from mx
// when the mesh moved, and the flag set for the next step
__global__ void k_step_end(const double* __restrict__ dt, double* __restrict__ dt_out, const double* __restrict__ dtau,
                           double* __restrict__ dtau_out, const double* __restrict__ mx, double* __restrict__ x, long n,
                           int* __restrict__ same)
{
    if (blockIdx.x == 0 && threadIdx.x == 0) {
        if (dt_out) *dt_out = *dt;
        if (dtau_out) *dtau_out = *dtau;
        *same = 1;
    }
    for (long t = blockIdx.x * (long)blockDim.x + threadIdx.x; t < n; t += (long)gridDim.x * blockDim.x) x[t] = mx[t];
}

static void shell_sizes(const Geo& g, long& nzs, long& nys, long& nxs)
{
    const long ng2 = 2L * g.ng;
    const long nz = g.dim == 3 ? g.n[2] : 1;
    nzs = g.dim == 3 ? ng2 * g.np[0] * g.np[1] : 0;
    nys = ng2 * g.np[0] * nz;
    nxs = ng2 * g.n[1] * nz;
}

hipError_t fill_ghosts2(const Geo& g, double* a, int ncomp, int what, double* a2, int ncomp2, int what2,
                       hipStream_t s, const int* skip_a = nullptr)
{
    long nzs, nys, nxs;
    shell_sizes(g, nzs, nys, nxs);
    const long total = nzs + nys + nxs;
    const int blocks = (int)std::min<long>((total + 255) / 256, 8192);
    hipLaunchKernelGGL(k_fill_shell, dim3(blocks), dim3(256), 0, s, g, a, ncomp, what, a2, ncomp2, what2, nzs,
                       nys, nxs, skip_a);
    return hipGetLastError();
}

hipError_t fill_ghosts(const Geo& g, double* a, int ncomp, int what, hipStream_t s)
{
    return fill_ghosts2(g, a, ncomp, what, nullptr, 0, GH_PLAIN, s);
}

hipError_t fill_state(const Geo& g, const InflowStates& in, double* JU, double* J, int nc, int nspec,
                      hipStream_t s)
{
    bool periodic = true;
    for (int k = 0; k < g.dim; k++) periodic = periodic && g.bc[k][0] == BC_PERIODIC;
    if (periodic) return fill_ghosts2(g, JU, nc, GH_PLAIN, J, 1, GH_PLAIN, s);   // plain wrapped copies
    long nzs, nys, nxs;
    shell_sizes(g, nzs, nys, nxs);
    const long total = nzs + nys + nxs;
    const int blocks = (int)std::min<long>((total + 255) / 256, 8192);
    hipLaunchKernelGGL(k_fill_state, dim3(blocks), dim3(256), 0, s, g, in, JU, J, nc, nspec, nzs, nys, nxs);
    return hipGetLastError();
}

__global__ void k_copy(const double* __restrict__ src, double* __restrict__ dst, long n)
{
    for (long t = blockIdx.x * (long)blockDim.x + threadIdx.x; t < n; t += (long)gridDim.x * blockDim.x)
        dst[t] = src[t];
}

__global__ void k_fill_value(double* __restrict__ dst, long n, double v)
{
    for (long t = blockIdx.x * (long)blockDim.x + threadIdx.x; t < n; t += (long)gridDim.x * blockDim.x)
        dst[t] = v;
}

__global__ void k_set_scalar(double* dst, double v) { if (threadIdx.x == 0 && blockIdx.x == 0) *dst = v; }

// dst = src over n values when *flag is zero
__global__ void k_copy_unless(const double* __restrict__ src, double* __restrict__ dst, long n,
                              const int* __restrict__ flag)
{
    if (*flag) return;
    for (long t = blockIdx.x * (long)blockDim.x + threadIdx.x; t < n; t += (long)gridDim.x * blockDim.x)
        dst[t] = src[t];
}

static int grid_for(long n) { return (int)std::max<long>(1, std::min<long>((n + 255) / 256, 16384)); }

hipError_t copy(const double* src, double* dst, long n, hipStream_t s)
{
    hipLaunchKernelGGL(k_copy, dim3(grid_for(n)), dim3(256), 0, s, src, dst, n);
    return hipGetLastError();
}
hipError_t fill_value(double* dst, long n, double v, hipStream_t s)
{
    hipLaunchKernelGGL(k_fill_value, dim3(grid_for(n)), dim3(256), 0, s, dst, n, v);
    return hipGetLastError();
}
hipError_t step_begin(const Geo& g, const InflowStates& in, double* JU, double* J, double* x, const double* mx,
                      int* same, int nc, int nspec, hipStream_t s)
{
    long nzs, nys, nxs;
    shell_sizes(g, nzs, nys, nxs);
    const long total = nzs + nys + nxs + (long)g.n[0] * g.n[1] * (g.dim == 3 ? g.n[2] : 1);
    hipLaunchKernelGGL(k_step_begin, dim3(grid_for(total)), dim3(256), 0, s, g, in, JU, J, x, mx, same, nc, nspec, nzs,
                       nys, nxs);
    return hipGetLastError();
}
hipError_t step_end(const double* dt, double* dt_out, const double* dtau, double* dtau_out, const double* mx, double* x,
                    long n, int* same, hipStream_t s)
{
    hipLaunchKernelGGL(k_step_end, dim3(grid_for(n)), dim3(256), 0, s, dt, dt_out, dtau, dtau_out, mx, x, n, same);
    return hipGetLastError();
}
hipError_t copy_unless(const double* src, double* dst, long n, const int* flag, hipStream_t s)
{
    hipLaunchKernelGGL(k_copy_unless, dim3(grid_for(n)), dim3(256), 0, s, src, dst, n, flag);
    return hipGetLastError();
}
hipError_t set_scalar(double* dst, double v, hipStream_t s)
{
    hipLaunchKernelGGL(k_set_scalar, dim3(1), dim3(64), 0, s, dst, v);
    return hipGetLastError();
}

// ---------------------------------------------------------------------------
// GCL metrics (eq SCLCoeff, eq VCLCoeff).  Stage mesh xs = x_n + c_s disp.
// ---------------------------------------------------------------------------
// a double of the `bytes` at base, both the same for the whole wave; a store at or
// past the end is dropped.  A marching kernel stores through it without a
// branch: behind a branch the compiler does not know how many stores follow a
// load, and its wait for a load of two planes ago also drains the last plane's
__device__ __forceinline__ double buffer_load(const double* base, unsigned bytes, unsigned at)
{
    const auto r = __builtin_amdgcn_make_buffer_rsrc(const_cast<double*>(base), 0, bytes, 0x00027000);
    return __builtin_bit_cast(double, __builtin_amdgcn_raw_buffer_load_b64(r, at, 0, 0));
}
__device__ __forceinline__ void buffer_store(double* base, unsigned bytes, unsigned at, double v)
{
    using U2 = __attribute__((__vector_size__(2 * sizeof(unsigned)))) unsigned;
    const auto r = __builtin_amdgcn_make_buffer_rsrc(base, 0, bytes, 0x00027000);
    __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(U2, v), r, at, 0, 0);
}
constexpr unsigned DROPPED = 0xfffffff8u;

// compute units of the device
constexpr int UNITS = 256;

// z chunks of nz planes for `cols` columns of blocks, `slots` blocks at a time (the
// launch's resident blocks a compute unit times the units):
// the number that leaves the shortest walk (rounds of blocks times planes a
// block), each walk taking `extra` planes more than it writes.  A block that has a
// compute unit to itself walks faster, by a third at least (64^3 mesh step 100 us; with
// the units doubled up for shorter chunks 111).  A multiple of 8, where each XCD
// walks whole chunks and so finds its tiles' neighbours in its own L2, may be a
// tenth longer (two Jacobi sweeps at 256^3: 8 chunks 280 us, 2 chunks 306)
static int z_chunk(int nz, long cols, int extra, int slots)
{
    double best = -1.0;
    int chunk = nz;
    // (past four rounds a shorter chunk only adds its extra planes)
    for (int c = 1; c <= std::max(1L, std::min((long)nz / 2, 4 * slots / cols + 8)); c++) {
        const int zc = (nz + c - 1) / c, n = (nz + zc - 1) / zc;
        const double rounds = slots > UNITS && cols * n <= UNITS ? 0.75 : (double)((cols * n + slots - 1) / slots);
        const double walk = rounds * (zc + extra) * (n % 8 == 0 ? 0.9 : 1.0);
        if (best < 0.0 || walk < best) {
            best = walk;
            chunk = zc;
        }
    }
    return chunk;
}

// 3D metrics in one walk along z.  The products
//   Pr[a][j] = delta_a[xs_p] xs_q,  (p, q) = (j+1, j+2) mod 3,
// are differenced again,
//   J dxi_k/dx_j = (delta_b[Pr[a][j]] - delta_a[Pr[b][j]]) / (dxi_a dxi_b),  (k, a, b) cyclic.
// delta is the 2w-order central difference 1/2 sum_m alpha_m (f_{+m} - f_{-m})
// (alpha_m = 0 for m > w).
//   A block owns (HX - 6) x (HY - 6) columns over a chunk of z planes and forms
// the products of these and of a 3-node halo around them, so they never go to
// memory: at 256^3 the walk moves 3.3 GB (2.4 GB of x, disp and the metrics
// themselves) where two passes with the nine products between them moved 7.2.
// Differences along z come from 7 planes of the thread's own column in
// registers: x, Pr[0] and Pr[1].  All three are 126 registers, two waves a SIMD,
// so two threads share a column: the first holds x and Pr[1] and gives
// Pr[2] and the metrics k = 0, the second holds Pr[0], brings x in and gives
// k = 1 and 2.  Neighbours in the plane are in LDS, both x and the products
// twice, so one barrier a plane is enough: products of plane k - 3 and x of
// plane k + 1 are written while the metrics of plane k - 4 are formed.
// x is loaded two planes ahead, and its wait comes before the plane's stores (behind
// them, in order, it would drain them first).
//   256^3, ghost fill included: 1040 us (two passes 1735 us).  Seven planes are
// unrolled, so that the rings stay in place (1153 us with the moves).  Bound by the
// stores, rows of 26 doubles at any alignment: without them 723 us; with the
// non-temporal hint, which keeps neighbouring tiles' parts of a line from meeting in
// the L2, 1143.  Two barriers a plane took 1249 us, one thread a column (512 of
// them) 1276, 48 x 10 columns of those 1537, 64 x 8 1610.
// (with the halves of alpha: the factor 1/2 of each difference is exact)
__device__ __forceinline__ double cdiff(const double* ah, double p1, double m1, double p2, double m2,
                                        double p3, double m3)
{
    double s = ah[0] * (p1 - m1);
    s += ah[1] * (p2 - m2);
    s += ah[2] * (p3 - m3);
    return s;
}

template <int HX, int HY, bool MOVED>
__global__ void __launch_bounds__(2 * HX * HY)
k_metric3(Geo g, Phys ph, const double* __restrict__ xn, const double* __restrict__ dx, double cs,
          const double* __restrict__ disp, const double* __restrict__ dt_dev, double* __restrict__ jxx,
          double* __restrict__ jxt, int zchunk, const int* __restrict__ reuse)
{
    if (reuse && *reuse) return;
    constexpr int TX = HX - 6, TY = HY - 6, NT = HX * HY;
    static_assert(NT % 64 == 0);
    __shared__ double X[2][3][NT + 6];    // xs of a plane (node t at t + 3)
    __shared__ double E[2][3][3][NT];     // Pr[a][j] of a plane
    const long P = g.P;
    const int np0 = g.np[0], np1 = g.np[1];
    int bx, by, bz;
    xcd_tile((g.n[0] + TX - 1) / TX, (g.n[1] + TY - 1) / TY, bx, by, bz);
    const bool first = __builtin_amdgcn_readfirstlane(threadIdx.x) < NT;
    const int t = first ? threadIdx.x : threadIdx.x - NT, lx = t % HX, ly = t / HX;
    const int gx = g.ng + bx * TX + lx - 3, gy = g.ng + by * TY + ly - 3;
    const int zc0 = g.ng + bz * zchunk, zc1 = min(zc0 + zchunk, g.ng + g.n[2]);
    if (zc0 >= zc1) return;   // uniform over the block
    const bool row = ly >= 3 && ly < TY + 3;
    const bool own = row && lx >= 3 && lx < TX + 3 && gx < g.ng + g.n[0] && gy < g.ng + g.n[1];
    // (a column beyond a ragged tile's halo reads the last padded node, which
    // no written node uses)
    const long sz = (long)np0 * np1;
    const double dt = dt_dev ? *dt_dev : 0.0;
    const double idt = dt > 0.0 ? 1.0 / dt : 0.0;   // mesh velocity = disp / dt
    const bool moving = jxt && disp && dt > 0.0;
    const double* wsrc = moving ? disp : xn;   // (read in any case)
    const double ah[3] = {0.5 * ph.alpha[0], 0.5 * ph.alpha[1], 0.5 * ph.alpha[2]};
    const double s01 = g.idxi[0] * g.idxi[1], s12 = g.idxi[1] * g.idxi[2], s20 = g.idxi[2] * g.idxi[0];
    const unsigned cb = (unsigned)((min(gy, np1 - 1) * np0 + min(gx, np0 - 1)) * sizeof(double));
    const unsigned plane = (unsigned)(sz * sizeof(double));
    auto load = [&](const double* f, int c, int z) { return buffer_load(f + (c * P + z * sz), plane, cb); };
    auto store = [&](double* f, int c, int z, double v) { buffer_store(f + (c * P + z * sz), plane, cb, v); };
    // the waves of the two halves take different walks, each with the same
    // barrier a plane
    auto walk = [&](auto half) {
        constexpr bool A = half == 0;
        // planes of the own column, plane zc0 - 3 + i in slot i % 7: Pr[1] (A) or Pr[0]; xs
        double pr[3][7], xr[A ? 3 : 1][7];
#pragma unroll
        for (int j = 0; j < 3; j++)
#pragma unroll
            for (int r = 0; r < 7; r++) {
                pr[j][r] = 0.0;
                if constexpr (A) xr[j][r] = 0.0;
            }
        double w[3] = {0.0, 0.0, 0.0}, nx[3], nd[3];
        auto fetch = [&](int z) {
#pragma unroll
            for (int p = 0; p < 3; p++) {
                nx[p] = load(xn, p, z);
                if constexpr (MOVED) nd[p] = load(dx, p, z);
            }
        };
        auto stage = [&](int z) {   // plane z into X; the next one on its way
#pragma unroll
            for (int p = 0; p < 3; p++) {
                if constexpr (MOVED) X[z & 1][p][t + 3] = nx[p] + cs * nd[p];
                else X[z & 1][p][t + 3] = nx[p];
            }
            fetch(min(z + 1, zc1 + 2));
        };
        if constexpr (!A) {
            fetch(zc0 - 3);
            stage(zc0 - 3);
        }
        __syncthreads();
        // (seven planes a pass, so that no ring is moved)
        for (int k0 = zc0 - 3;; k0 += 7)
#pragma unroll
        for (int u = 0; u < 7; u++) {
            const int k = k0 + u;
            // the metrics of plane z, whose products are in E since the last
            // barrier.  Each half folds its metrics into its time metrics (the
            // sum over j in the order of k_vcl)
            const int z = k - 4;
            if constexpr (!A)
                if (k + 1 < zc1 + 3) stage(k + 1);
            // difference along z of a ring at plane z, its last plane in slot u - 1
            auto zdiff = [&](const double (&q)[7], int u) {
                return cdiff(ah, q[(u + 4) % 7], q[(u + 2) % 7], q[(u + 5) % 7], q[(u + 1) % 7], q[(u + 6) % 7], q[u % 7]);
            };
            if (own && z >= zc0) {
                double nt[2] = {0.0, 0.0};
#pragma unroll
                for (int j = 0; j < 3; j++) {
                    const double v = moving ? w[j] * idt : 0.0;
                    const double *e0 = &E[z & 1][0][j][t], *e1 = &E[z & 1][1][j][t], *e2 = &E[z & 1][2][j][t];
                    const double zd = zdiff(pr[j], u);
                    if constexpr (A) {   // k = 0 (a = 1, b = 2): delta_2 Pr[1][j] - delta_1 Pr[2][j]
                        const double M = (zd - cdiff(ah, e2[HX], e2[-HX], e2[2 * HX], e2[-2 * HX], e2[3 * HX], e2[-3 * HX])) * s12;
                        store(jxx, j, z, M);
                        nt[0] -= v * M;
                    } else {
                        // k = 1 (a = 2, b = 0): delta_0 Pr[2][j] - delta_2 Pr[0][j]
                        const double M1 = (cdiff(ah, e2[1], e2[-1], e2[2], e2[-2], e2[3], e2[-3]) - zd) * s20;
                        // k = 2 (a = 0, b = 1): delta_1 Pr[0][j] - delta_0 Pr[1][j]
                        const double M2 = (cdiff(ah, e0[HX], e0[-HX], e0[2 * HX], e0[-2 * HX], e0[3 * HX], e0[-3 * HX]) -
                                           cdiff(ah, e1[1], e1[-1], e1[2], e1[-2], e1[3], e1[-3])) * s01;
                        store(jxx, 3 + j, z, M1);
                        store(jxx, 6 + j, z, M2);
                        nt[0] -= v * M1;
                        nt[1] -= v * M2;
                    }
                }
                if (jxt) {
                    store(jxt, A ? 0 : 1, z, nt[0]);
                    if constexpr (!A) store(jxt, 2, z, nt[1]);
                }
            }
            if (k == zc1 + 3) return;
            // Pr[1] (rows within the halo) or Pr[0] (columns within the halo) of plane k
            double d[3] = {0.0, 0.0, 0.0};
            if (!A || row)
#pragma unroll
                for (int p = 0; p < 3; p++) {
                    constexpr int st = A ? HX : 1;
                    const double* F = &X[k & 1][p][t + 3];
                    d[p] = cdiff(ah, F[st], F[-st], F[2 * st], F[-2 * st], F[3 * st], F[-3 * st]);
                }
            double v[3];
#pragma unroll
            for (int p = 0; p < 3; p++) v[p] = X[k & 1][p][t + 3];
            // and the products of plane k - 3
#pragma unroll
            for (int j = 0; j < 3; j++) {
                pr[j][u] = d[(j + 1) % 3] * v[(j + 2) % 3];
                if constexpr (A) xr[j][u] = v[j];
                E[(k + 1) & 1][A][j][t] = pr[j][(u + 4) % 7];
            }
            if constexpr (A) {
#pragma unroll
                for (int j = 0; j < 3; j++)
                    E[(k + 1) & 1][2][j][t] = zdiff(xr[(j + 1) % 3], u + 1) * xr[(j + 2) % 3][(u + 4) % 7];
            }
#pragma unroll
            for (int j = 0; j < 3; j++) w[j] = load(wsrc, j, max(k - 3, zc0));
            __syncthreads();
        }
    };
    if (first) walk(std::integral_constant<int, 0>{});
    else walk(std::integral_constant<int, 1>{});
}

// 2D: J dxi_1/dx = (delta_2 x_2, -delta_2 x_1)/dxi_2, J dxi_2/dx = (-delta_1 x_2, delta_1 x_1)/dxi_1,
// a node and its ghost images a thread.  With reuse set, jxx holds the metrics
// already (ghost layers included) and only the time metrics are formed.
// (One pass: the separate grid-stride passes over the nodes and the ghost shell,
// with divisions and the time metrics and ghost fill of kept metrics in
// launches of their own, took 12.3 + 4.1 + 4.8 us at 350 x 150; now 6.9 on
// average.)
__global__ void k_metric2(Geo g, Phys ph, const double* __restrict__ xn,
                          const double* __restrict__ disp, double cs, const double* __restrict__ dt_dev,
                          double* __restrict__ jxx, double* __restrict__ jxt, const int* __restrict__ reuse)
{
    const bool kept = reuse && *reuse;
    if (kept && !jxt) return;
    const long P = g.P;
    const long q = blockIdx.x * (long)blockDim.x + threadIdx.x;
    if (q >= n_interior(g)) return;
    const double dt = dt_dev ? *dt_dev : 0.0;
    int i0, i1, i2;
    const long i = interior_node(g, q, i0, i1, i2);
    double w[2] = {0.0, 0.0};   // the displacement, ahead of the stores
    if (jxt && disp && dt > 0.0) {
        w[0] = disp[i];
        w[1] = disp[P + i];
    }
    double M[4];
    if (kept) {
#pragma unroll
        for (int c = 0; c < 4; c++) M[c] = jxx[c * P + i];
    } else {
        const double ah[3] = {0.5 * ph.alpha[0], 0.5 * ph.alpha[1], 0.5 * ph.alpha[2]};   // 0 beyond w
        const bool moved = disp && cs != 0.0;
        // all loads first (one behind a branch is waited for on the spot)
        auto node = [&](int a, int p, int m) {   // +1 +2 +3 -1 -2 -3 along a, component p
            return p * P + i + (m < 3 ? m + 1 : 2 - m) * (a == 0 ? 1L : g.np[0]);
        };
        double f[2][2][6];
#pragma unroll
        for (int q = 0; q < 24; q++) f[q / 12][q / 6 % 2][q % 6] = xn[node(q / 12, q / 6 % 2, q % 6)];
        if (moved) {
            double e[2][2][6];
#pragma unroll
            for (int q = 0; q < 24; q++) e[q / 12][q / 6 % 2][q % 6] = disp[node(q / 12, q / 6 % 2, q % 6)];
#pragma unroll
            for (int q = 0; q < 24; q++) f[q / 12][q / 6 % 2][q % 6] += cs * e[q / 12][q / 6 % 2][q % 6];
        }
        double d[2][2];   // d[a][p] = delta_a[x_p]
#pragma unroll
        for (int a = 0; a < 2; a++)
#pragma unroll
            for (int p = 0; p < 2; p++) {
                const double* h = f[a][p];
                d[a][p] = cdiff(ah, h[0], h[3], h[1], h[4], h[2], h[5]);
            }
        M[0] = d[1][1] * g.idxi[1];
        M[1] = -d[1][0] * g.idxi[1];
        M[2] = -d[0][1] * g.idxi[0];
        M[3] = d[0][0] * g.idxi[0];
        put_images<2, 4, GH_JXX>(g, i0 - g.ng, i1 - g.ng, 0, M, jxx);
    }
    if (jxt) {
        const double idt = dt > 0.0 ? 1.0 / dt : 0.0;   // mesh velocity = disp / dt
        double nt[2] = {0.0, 0.0};
        if (disp && dt > 0.0)
#pragma unroll
            for (int k = 0; k < 2; k++)
#pragma unroll
                for (int j = 0; j < 2; j++) nt[k] -= (w[j] * idt) * M[k * 2 + j];
        put_images<2, 2, GH_JXT>(g, i0 - g.ng, i1 - g.ng, 0, nt, jxt);
    }
}

// jxi_t only, from an existing jxi_x (only when *only_if is set, if given)
__global__ void k_vcl(Geo g, const double* __restrict__ disp, const double* __restrict__ dt_dev,
                      const double* __restrict__ jxx, double* __restrict__ jxt, const int* __restrict__ only_if)
{
    if (only_if && !*only_if) return;
    const long P = g.P;
    const int D = g.dim;
    const long nint = n_interior(g);
    const double dt = dt_dev ? *dt_dev : 0.0;
    const double idt = dt > 0.0 ? 1.0 / dt : 0.0;   // mesh velocity = disp / dt
    for (long q = blockIdx.x * (long)blockDim.x + threadIdx.x; q < nint; q += (long)gridDim.x * blockDim.x) {
        int i0, i1, i2;
        const long i = interior_node(g, q, i0, i1, i2);
        for (int k = 0; k < D; k++) {
            double nt = 0.0;
            if (disp && dt > 0.0)
                for (int j = 0; j < D; j++) nt -= (disp[j * P + i] * idt) * jxx[(k * D + j) * P + i];
            jxt[k * P + i] = nt;
        }
    }
}

// discrete Jacobian of the mesh: J = (1/d) sum_k sum_j dx_j/dxi_k J dxi_k/dx_j
// (the cofactor expansion of det dx/dxi along each column k, averaged),
// dx_j/dxi_k by the 2w-order central difference of the metrics
__global__ void k_jacobian(Geo g, Phys ph, const double* __restrict__ x, const double* __restrict__ jxx,
                           double* __restrict__ J)
{
    const long P = g.P;
    const int d = g.dim;
    const long nint = n_interior(g);
    for (long q = blockIdx.x * (long)blockDim.x + threadIdx.x; q < nint; q += (long)gridDim.x * blockDim.x) {
        int i0, i1, i2;
        const long i = interior_node(g, q, i0, i1, i2);
        double s = 0.0;
        for (int k = 0; k < d; k++) {
            const long st = dir_stride(g, k);
            for (int j = 0; j < d; j++) {
                const double* a = x + j * P;
                double dk = 0.0;
                for (int m = 1; m <= ph.w; m++) dk += ph.alpha[m - 1] * (a[i + m * st] - a[i - m * st]);
                s += 0.5 * dk / g.dxi[k] * jxx[(k * d + j) * P + i];
            }
        }
        J[i] = s / d;
    }
}

hipError_t jacobian(const Phys& ph, const Geo& g, const double* x, const double* jxx, double* J, hipStream_t s)
{
    const long nint = (long)g.n[0] * g.n[1] * (g.dim == 3 ? g.n[2] : 1);
    hipLaunchKernelGGL(k_jacobian, dim3(grid_for(nint)), dim3(256), 0, s, g, ph, x, jxx, J);
    const hipError_t e = hipGetLastError();
    return e != hipSuccess ? e : fill_ghosts(g, J, 1, GH_PLAIN, s);
}

hipError_t metrics(const Phys& ph, const Geo& g, const double* xn, const double* disp, double cs,
                   const double* dt_dev, double* jxx, double* jxt, int vcl_only,
                   hipStream_t s, const int* reuse)
{
    const long nint = (long)g.n[0] * g.n[1] * (g.dim == 3 ? g.n[2] : 1);
    // the stage mesh reads the displacement only where c_s is not zero (the
    // 2D kernel tests c_s itself: it reads disp for the time metrics too)
    const double* dx = cs != 0.0 ? disp : nullptr;
    if (vcl_only) {
        if (!jxt) return hipSuccess;
        hipLaunchKernelGGL(k_vcl, dim3(grid_for(nint)), dim3(256), 0, s, g, disp, dt_dev, jxx, jxt,
                           (const int*)nullptr);
    } else if (g.dim == 2) {   // with its ghost layers
        hipLaunchKernelGGL(k_metric2, dim3((unsigned)((nint + 255) / 256)), dim3(256), 0, s, g, ph, xn, disp, cs,
                           dt_dev, jxx, jxt, reuse);
        return hipGetLastError();
    } else {
        constexpr int HX = 32, HY = 16;   // one block a compute unit
        const int gx = (g.n[0] + HX - 7) / (HX - 6), gy = (g.n[1] + HY - 7) / (HY - 6);
        const int zc = z_chunk(g.n[2], (long)gx * gy, 6, UNITS);
        hipLaunchKernelGGL((dx ? k_metric3<HX, HY, true> : k_metric3<HX, HY, false>), dim3(gx * gy * ((g.n[2] + zc - 1) / zc)), dim3(2 * HX * HY), 0, s, g, ph,
                           xn, dx, cs, disp, dt_dev, jxx, jxt, zc, reuse);
        if (reuse && jxt)
            hipLaunchKernelGGL(k_vcl, dim3(grid_for(nint)), dim3(256), 0, s, g, disp, dt_dev, jxx, jxt, reuse);
    }
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    if (!vcl_only) return fill_ghosts2(g, jxx, g.dim * g.dim, GH_JXX, jxt, g.dim, GH_JXT, s, reuse);
    if (jxt) e = fill_ghosts(g, jxt, g.dim, GH_JXT, s);
    return e;
}

// ---------------------------------------------------------------------------
// reductions: per-block partials in a fixed grid, then one block folds the
// partials in a fixed order (deterministic sums)
// ---------------------------------------------------------------------------
static constexpr int RED_BLOCKS = 2048;

// (the maximum is lambda: out[1] = a / lambda with a = cfl; the sum is scaled by a)
template <int OP>
__global__ void k_finish(const double* __restrict__ part, int nparts, double* __restrict__ out, double a)
{
    double v = OP == RED_MAX ? -INFINITY : 0.0;
    for (int t = threadIdx.x; t < nparts; t += blockDim.x) v = red_combine<OP>(v, part[t]);
    v = block_reduce<OP>(v);
    if (threadIdx.x == 0) {
        out[0] = OP == RED_MAX ? v : v * a;
        if (OP == RED_MAX) out[1] = a / v;
    }
}

// thermo of one node from JU/J
template <int N, int D>
struct NodeState {
    double U[N + D + 1];
    double rho, v[D], T, p, beta;
    bool ok;
};

template <int N, int D>
__device__ __forceinline__ void load_state(const Phys& ph, const double* JU, const double* Jv, long P,
                                           long i, NodeState<N, D>& s)
{
    constexpr int NC = N + D + 1;
    const double Jq = Jv[i];
#pragma unroll
    for (int c = 0; c < NC; c++) s.U[c] = JU[c * P + i] / Jq;
    double rt = 0.0, cvr = 0.0, rR = 0.0;
    bool ok = Jq > 0.0;
#pragma unroll
    for (int l = 0; l < N; l++) {
        rt += s.U[l];
        cvr += ph.cv[l] * s.U[l];
        rR += ph.Rg[l] * s.U[l];
        ok = ok && (s.U[l] > 0.0);
    }
    double kin = 0.0;
#pragma unroll
    for (int j = 0; j < D; j++) {
        s.v[j] = s.U[N + j] / rt;
        kin += 0.5 * s.U[N + j] * s.v[j];
    }
    s.rho = rt;
    s.T = (s.U[NC - 1] - kin - ph.pinf_tot) / cvr;
    s.beta = 1.0 / s.T;
    s.p = rR * s.T - ph.pinf_tot;
    s.ok = ok && (s.T > 0.0) && isfinite(s.T) && isfinite(kin);
}

template <int N, int D>
__global__ void k_wavespeed(Phys ph, Geo g, const double* __restrict__ JU, const double* __restrict__ Jv,
                            const double* __restrict__ jxx, double* __restrict__ part,
                            unsigned* __restrict__ status)
{
    const long P = g.P;
    const long nint = n_interior(g);
    double lam = 0.0;
    unsigned bad = 0;
    for (long q = blockIdx.x * (long)blockDim.x + threadIdx.x; q < nint; q += (long)gridDim.x * blockDim.x) {
        int i0, i1, i2;
        const long i = interior_node(g, q, i0, i1, i2);
        NodeState<N, D> s;
        load_state<N, D>(ph, JU, Jv, P, i, s);
        if (!s.ok) bad |= 1u;
        double cvr = 0.0, cg = 0.0, rR = 0.0;
#pragma unroll
        for (int l = 0; l < N; l++) {
            cvr += ph.cv[l] * s.U[l];
            cg += ph.cvgam[l] * s.U[l];
            rR += ph.Rg[l] * s.U[l];
        }
        const double c = sqrt((rR / s.rho) * (cg / cvr) * s.T);
        double sum = 0.0;
#pragma unroll
        for (int k = 0; k < D; k++) {
            double vn = 0.0, nn = 0.0;
#pragma unroll
            for (int j = 0; j < D; j++) {
                const double n = jxx[(k * D + j) * P + i];
                vn += s.v[j] * n;
                nn += n * n;
            }
            sum += (fabs(vn) + c * sqrt(nn)) / Jv[i] / g.dxi[k];
        }
        lam = fmax(lam, sum);
    }
    if (bad) atomicOr(status, bad);
    lam = block_reduce<RED_MAX>(lam);
    if (threadIdx.x == 0) part[blockIdx.x] = lam;
}

template <int N, int D>
__global__ void k_entropy(Phys ph, Geo g, const double* __restrict__ JU, const double* __restrict__ Jv,
                          const double* __restrict__ dJU, const double* __restrict__ dJ,
                          double* __restrict__ part)
{
    constexpr int NC = N + D + 1;
    const long P = g.P;
    const long nint = n_interior(g);
    double acc = 0.0;
    for (long q = blockIdx.x * (long)blockDim.x + threadIdx.x; q < nint; q += (long)gridDim.x * blockDim.x) {
        int i0, i1, i2;
        const long i = interior_node(g, q, i0, i1, i2);
        NodeState<N, D> s;
        load_state<N, D>(ph, JU, Jv, P, i, s);
        // logarithms as the flux kernels take them (within 2 ulp); a
        // non-positive T or rho_l is a non-physical state the steps report
        const double lT = ln_pos(s.T);
        if (!dJU) {   // J eta, eta = -sum rho_l (c_vl ln T - R_l ln rho_l)
            double eta = 0.0;
#pragma unroll
            for (int l = 0; l < N; l++) eta -= s.U[l] * (ph.cv[l] * lT - ph.Rg[l] * ln_pos(s.U[l]));
            acc += Jv[i] * eta;
        } else {      // V . dJU - phi dJ
            double v2 = 0.0;
#pragma unroll
            for (int j = 0; j < D; j++) v2 += s.v[j] * s.v[j];
            double t = 0.0, phi = 0.0;
#pragma unroll
            for (int l = 0; l < N; l++) {
                const double Vl = -(ph.cv[l] * lT - ph.Rg[l] * ln_pos(s.U[l])) - v2 / (2.0 * s.T) + ph.cvgam[l];
                t += Vl * dJU[l * P + i];
                phi += ph.Rg[l] * s.U[l] - ph.pinf[l] / s.T;
            }
#pragma unroll
            for (int j = 0; j < D; j++) t += (s.v[j] / s.T) * dJU[(N + j) * P + i];
            t += (-1.0 / s.T) * dJU[(NC - 1) * P + i];
            acc += t - phi * dJ[i];
        }
    }
    acc = block_reduce<RED_SUM>(acc);
    if (threadIdx.x == 0) part[blockIdx.x] = acc;
}

static int red_grid(long nint) { return (int)std::max<long>(1, std::min<long>((nint + 255) / 256, RED_BLOCKS)); }

int reduction_blocks(long nint) { return red_grid(nint); }

#define ES_DISPATCH_ND(ph, g, FN, ...)                                   \
    do {                                                                 \
        if (ph.nspec == 1 && g.dim == 2) FN<1, 2>(__VA_ARGS__);          \
        else if (ph.nspec == 2 && g.dim == 2) FN<2, 2>(__VA_ARGS__);     \
        else if (ph.nspec == 1 && g.dim == 3) FN<1, 3>(__VA_ARGS__);     \
        else FN<2, 3>(__VA_ARGS__);                                      \
    } while (0)

template <int N, int D>
static void launch_wavespeed(const Phys& ph, const Geo& g, const double* JU, const double* J,
                             const double* jxx, double* part, unsigned* status, int nb, hipStream_t s)
{
    hipLaunchKernelGGL((k_wavespeed<N, D>), dim3(nb), dim3(256), 0, s, ph, g, JU, J, jxx, part, status);
}

hipError_t wavespeed(const Phys& ph, const Geo& g, const double* JU, const double* J, const double* jxx,
                     double cfl, double* part, double* out2, unsigned* status, hipStream_t s)
{
    const long nint = (long)g.n[0] * g.n[1] * (g.dim == 3 ? g.n[2] : 1);
    const int nb = red_grid(nint);
    ES_DISPATCH_ND(ph, g, launch_wavespeed, ph, g, JU, J, jxx, part, status, nb, s);
    hipLaunchKernelGGL(k_finish<RED_MAX>, dim3(1), dim3(256), 0, s, part, nb, out2, cfl);
    return hipGetLastError();
}

// per-instance CFL wave speed of a batch of 2D instances (eq cfl for each):
// block (b, j0, j1) reduces rows j0..j1-1 of instance b; a second pass
// reduces each instance's blocks in a fixed order.
template <int N>
__global__ void k_wavespeed_batched(Phys ph, const Geo* __restrict__ geos, const int4* __restrict__ wl,
                                    const double* const* __restrict__ JUt,
                                    const double* const* __restrict__ Jt,
                                    const double* const* __restrict__ jxxt, double* __restrict__ part,
                                    unsigned* __restrict__ status)
{
    constexpr int D = 2;
    const int4 e = wl[blockIdx.x];
    const Geo g = geos[e.x];
    const double* JU = JUt[e.x];
    const double* Jv = Jt[e.x];
    const double* jxx = jxxt[e.x];
    const long P = g.P;
    const int n0 = g.n[0];
    const int cnt = (e.z - e.y) * n0;
    double lam = 0.0;
    unsigned bad = 0;
    for (int q = threadIdx.x; q < cnt; q += blockDim.x) {
        const long i = node_index(g, q % n0 + g.ng, e.y + q / n0 + g.ng, 0);
        NodeState<N, D> s;
        load_state<N, D>(ph, JU, Jv, P, i, s);
        if (!s.ok) bad |= 1u;
        double cvr = 0.0, cg = 0.0, rR = 0.0;
#pragma unroll
        for (int l = 0; l < N; l++) {
            cvr += ph.cv[l] * s.U[l];
            cg += ph.cvgam[l] * s.U[l];
            rR += ph.Rg[l] * s.U[l];
        }
        const double c = sqrt((rR / s.rho) * (cg / cvr) * s.T);
        double sum = 0.0;
#pragma unroll
        for (int k = 0; k < D; k++) {
            double vn = 0.0, nn = 0.0;
#pragma unroll
            for (int j = 0; j < D; j++) {
                const double n = jxx[(k * D + j) * P + i];
                vn += s.v[j] * n;
                nn += n * n;
            }
            sum += (fabs(vn) + c * sqrt(nn)) / Jv[i] / g.dxi[k];
        }
        lam = fmax(lam, sum);
    }
    if (bad) atomicOr(status, bad);
    lam = block_reduce<RED_MAX>(lam);
    if (threadIdx.x == 0) part[blockIdx.x] = lam;
}

__global__ void k_finish_batched(const double* __restrict__ part, const int* __restrict__ first, double cfl,
                                 double* __restrict__ lam_out, double* __restrict__ dt_out)
{
    const int b = blockIdx.x;
    double v = -INFINITY;
    for (int t = first[b] + threadIdx.x; t < first[b + 1]; t += blockDim.x) v = fmax(v, part[t]);
    v = block_reduce<RED_MAX>(v);
    if (threadIdx.x == 0) {
        if (lam_out) lam_out[b] = v;
        dt_out[b] = cfl / v;
    }
}

hipError_t wavespeed_batched(const Phys& ph, const Geo* geos, const int4* wl, int nwl, const int* first,
                             int count, const double* const* JU, const double* const* J,
                             const double* const* jxx, double cfl, double* part, double* lambda_out,
                             double* dt_out, unsigned* status, hipStream_t s)
{
    if (ph.nspec == 1)
        hipLaunchKernelGGL(k_wavespeed_batched<1>, dim3(nwl), dim3(256), 0, s, ph, geos, wl, JU, J, jxx,
                           part, status);
    else
        hipLaunchKernelGGL(k_wavespeed_batched<2>, dim3(nwl), dim3(256), 0, s, ph, geos, wl, JU, J, jxx,
                           part, status);
    hipLaunchKernelGGL(k_finish_batched, dim3(count), dim3(256), 0, s, part, first, cfl, lambda_out, dt_out);
    return hipGetLastError();
}

template <int N, int D>
static void launch_entropy(const Phys& ph, const Geo& g, const double* JU, const double* J,
                           const double* dJU, const double* dJ, double* part, int nb, hipStream_t s)
{
    hipLaunchKernelGGL((k_entropy<N, D>), dim3(nb), dim3(256), 0, s, ph, g, JU, J, dJU, dJ, part);
}

hipError_t entropy_sum(const Phys& ph, const Geo& g, const double* JU, const double* J, const double* dJU,
                       const double* dJ, double* part, double* out, hipStream_t s)
{
    const long nint = (long)g.n[0] * g.n[1] * (g.dim == 3 ? g.n[2] : 1);
    const int nb = red_grid(nint);
    double dv = 1.0;
    for (int k = 0; k < g.dim; k++) dv *= g.dxi[k];
    ES_DISPATCH_ND(ph, g, launch_entropy, ph, g, JU, J, dJU, dJ, part, nb, s);
    hipLaunchKernelGGL(k_finish<RED_SUM>, dim3(1), dim3(256), 0, s, part, nb, out, dv);
    return hipGetLastError();
}

// ---------------------------------------------------------------------------
// mesh redistribution (Section 4)
// ---------------------------------------------------------------------------
// The kernels keep a maximum or minimum over all blocks in a device scalar
// that the call's first launch resets (order does not matter, so the result
// is the two-pass reduction's): non-negative doubles compare like their bits.
// One thread a block takes part: the atomics of one address follow one another,
// and with one a wave the 64^3 monitor (480 blocks of eight) took 24.0 instead
// of 9.3 us.
__device__ __forceinline__ void scalar_max(double* a, double v)
{
    if (v > *(volatile double*)a)
        atomicMax((unsigned long long*)a, (unsigned long long)__double_as_longlong(v));
}

// any sign: bits that order like the doubles
__device__ __forceinline__ unsigned long long order_key(double v)
{
    const unsigned long long b = (unsigned long long)__double_as_longlong(v);
    return (b >> 63) ? ~b : (b | 0x8000000000000000ull);
}
__device__ __forceinline__ double order_value(unsigned long long k)
{
    return __longlong_as_double((long long)((k >> 63) ? (k & 0x7fffffffffffffffull) : ~k));
}

__device__ __forceinline__ void scalar_min(unsigned long long* key, double v)
{
    const unsigned long long k = order_key(v);
    if (k < *(volatile unsigned long long*)key) atomicMin(key, k);
}

// scal: the maxima [0..7] to 0, the limiter's key [8] to that of 1; the
// residuals to 0
__global__ void k_mesh_begin(double* __restrict__ scal, double* __restrict__ resid, int nresid)
{
    const int t = threadIdx.x;
    if (t < 8) scal[t] = 0.0;
    if (t == 8) ((unsigned long long*)scal)[8] = order_key(1.0);
    if (resid)
        for (int q = t; q < nresid; q += blockDim.x) resid[q] = 0.0;
}

// |grad_xi sigma| by second-order central differences, for each monitor
// variable, and its maximum.  The form with a Laplacian term also writes |lap_xi sigma| (second-order central
// differences) as channel nsig + s.  Variables: 0 rho, 1 rho_1, 2 rho_2,
// 3 p, 4 the speed |v| (the u of Example 5.9's monitor), 5 the schlieren
// function of eq schlieren, read from its array (with ghost layers).
// monitor variable sig at node i.  SIG: which variables the monitor may
// use, so that the kernels carry only the code (and registers) they need:
// 0 the densities (rho, rho_1, rho_2), 1 also the pressure, 2 also the
// speed and the schlieren function
template <int N, int D, int SIG = 0>
__device__ __forceinline__ double sigma_of(const Phys& ph, const double* JU, const double* Jv, long P,
                                           long i, int sig, const double* phi)
{
    if (SIG == 2 && sig == 5) return phi[i];
    const double Jq = Jv[i];
    if (SIG == 2 && sig == 4) {
        double r = 0.0, m2 = 0.0;
#pragma unroll
        for (int l = 0; l < N; l++) r += JU[l * P + i] / Jq;
#pragma unroll
        for (int j = 0; j < D; j++) {
            const double vj = (JU[(N + j) * P + i] / Jq) / r;
            m2 += vj * vj;
        }
        return sqrt(m2);
    }
    // (divisions, not a reciprocal of J: with the reciprocal the 3D gradient
    // took 310 instead of 240 us although it issues fewer instructions)
    if (sig == 0) {
        double r = 0.0;
#pragma unroll
        for (int l = 0; l < N; l++) r += JU[l * P + i] / Jq;
        return r;
    }
    if (sig == 1) return JU[i] / Jq;
    if (sig == 2 || SIG == 0) return JU[(N > 1 ? 1 : 0) * P + i] / Jq;
    NodeState<N, D> s;
    load_state<N, D>(ph, JU, Jv, P, i, s);
    return s.p;
}

// the value of the lane below or above this one in the wave (0 past its ends); every
// lane of the wave has to take part
template <int CTRL>
__device__ __forceinline__ double lane_shift(double v)
{
    const unsigned long long b = __builtin_bit_cast(unsigned long long, v);
    const unsigned lo = __builtin_amdgcn_update_dpp(0, (int)(unsigned)b, CTRL, 0xf, 0xf, true);
    const unsigned hi = __builtin_amdgcn_update_dpp(0, (int)(unsigned)(b >> 32), CTRL, 0xf, 0xf, true);
    return __builtin_bit_cast(double, (unsigned long long)hi << 32 | lo);
}
__device__ __forceinline__ double lane_below(double v) { return lane_shift<0x138>(v); }   // wave shift right by one
__device__ __forceinline__ double lane_above(double v) { return lane_shift<0x130>(v); }   // wave shift left by one

// 3D monitor gradient walking z (second-order central differences): a block owns
// 30 x 14 columns over a chunk of z planes, every thread a column of these and a
// one-node halo (a row is 32 lanes).  A variable is evaluated once per node of
// the patch, 1.2 times per owned node; its neighbours along x are the
// neighbouring lanes', along y in LDS (two planes), along z the thread's own
// (256^3, density: 160 us; 64 x 4 columns with all neighbours in LDS 205).
template <int N, int SIG>
__global__ void __launch_bounds__(512)
k_monitor_grad3(Phys ph, Geo g, MonitorP mo, const double* __restrict__ JU, const double* __restrict__ Jv,
                double* __restrict__ grad, double* __restrict__ gmax, int zchunk)
{
    constexpr int D = 3, TX = 30, TY = 14, HX = 32;
    __shared__ double Sg[2][512 + 2 * HX];   // (a row on either side, read and not used)
    __shared__ double part[8][MON_CH];       // the waves' maxima
    const long P = g.P;
    const int np0 = g.np[0], np1 = g.np[1];
    int bx, by, bz;
    xcd_tile((g.n[0] + TX - 1) / TX, (g.n[1] + TY - 1) / TY, bx, by, bz);
    const int t = threadIdx.x, lx = t % HX, ly = t / HX;
    const int gx = bx * TX + lx - 1, gy = by * TY + ly - 1;
    const bool own = lx >= 1 && lx <= TX && ly >= 1 && ly <= TY && gx < g.n[0] && gy < g.n[1];
    const int zc0 = bz * zchunk, zc1 = min(zc0 + zchunk, g.n[2]);
    if (zc0 >= zc1) return;   // uniform over the block
    // (a column beyond a ragged tile's halo reads the nearest one, which no written node uses)
    const long sz = (long)np0 * np1, col = (long)(min(gy, g.n[1]) + g.ng) * np0 + min(gx, g.n[0]) + g.ng;
    double ih[3];
#pragma unroll
    for (int k = 0; k < 3; k++) ih[k] = 1.0 / (2.0 * g.dxi[k]);
    for (int s = 0; s < mo.nsig; s++) {
        const int sg = mo.sigma[s];
        auto sigma = [&](int z) { return sigma_of<N, D, SIG>(ph, JU, Jv, P, col + (z + g.ng) * sz, sg, mo.phi); };
        double sm = sigma(zc0 - 1), s0 = sigma(zc0);
        double mg = 0.0, ml = 0.0;     // this channel's maxima over the column
        Sg[zc0 & 1][HX + t] = s0;
        __syncthreads();
        for (int z = zc0; z < zc1; z++) {
            const double sp = sigma(z + 1);
            const double xp = lane_above(s0), xm = lane_below(s0);
            const double* A = &Sg[z & 1][HX + t];
            const double yp = A[HX], ym = A[-HX];
            const double d0 = (xp - xm) * ih[0];
            const double d1 = (yp - ym) * ih[1];
            const double d2 = (sp - sm) * ih[2];
            const double gv = sqrt(d0 * d0 + d1 * d1 + d2 * d2);
            const long i = col + (z + g.ng) * sz;
            if (own) {
                grad[s * P + i] = gv;
                mg = fmax(mg, gv);
                if (mo.form) {   // directions 0, 1, 2 in order
                    double lap = (xp - 2.0 * s0 + xm) / (g.dxi[0] * g.dxi[0]);
                    lap += (yp - 2.0 * s0 + ym) / (g.dxi[1] * g.dxi[1]);
                    lap += (sp - 2.0 * s0 + sm) / (g.dxi[2] * g.dxi[2]);
                    grad[(mo.nsig + s) * P + i] = fabs(lap);
                    ml = fmax(ml, fabs(lap));
                }
            }
            Sg[(z + 1) & 1][HX + t] = sp;
            sm = s0;
            s0 = sp;
            __syncthreads();
        }
        mg = wave_max(mg);
        if (mo.form) ml = wave_max(ml);
        if ((t & 63) == 0) {
            part[t >> 6][s] = mg;
            if (mo.form) part[t >> 6][mo.nsig + s] = ml;
        }
    }
    __syncthreads();
    if (t < (mo.form ? 2 * mo.nsig : mo.nsig)) {
        double m = part[0][t];
        for (int q = 1; q < 8; q++) m = fmax(m, part[q][t]);
        scalar_max(gmax + t, m);
    }
}

// the schlieren function of eq schlieren, Phi = exp(-Psi |grad rho| /
// max |grad rho|), Psi = (psi_1 rho_1 + psi_2 rho_2) / rho: first
// |grad_xi rho| (the monitor's central differences) and its maximum, then Phi from the global maximum (1 where it is 0)
template <int N, int D>
__global__ void k_rho_grad(Phys ph, Geo g, const double* __restrict__ JU, const double* __restrict__ Jv,
                           double* __restrict__ gr, double* __restrict__ gmax)
{
    const long P = g.P;
    const long nint = n_interior(g);
    double gm = 0.0;
    for (long q = blockIdx.x * (long)blockDim.x + threadIdx.x; q < nint; q += (long)gridDim.x * blockDim.x) {
        int i0, i1, i2;
        const long i = interior_node(g, q, i0, i1, i2);
        double g2 = 0.0;
#pragma unroll
        for (int k = 0; k < D; k++) {
            const long st = dir_stride(g, k);
            const double sp = sigma_of<N, D>(ph, JU, Jv, P, i + st, 0, nullptr);
            const double sm = sigma_of<N, D>(ph, JU, Jv, P, i - st, 0, nullptr);
            const double dk = (sp - sm) / (2.0 * g.dxi[k]);
            g2 += dk * dk;
        }
        gr[i] = sqrt(g2);
        gm = fmax(gm, gr[i]);
    }
    const double r = block_reduce<RED_MAX>(gm);
    if (threadIdx.x == 0) scalar_max(gmax, r);
}

template <int N, int D>
__global__ void k_schlieren(Phys ph, Geo g, MonitorP mo, const double* __restrict__ JU,
                            const double* __restrict__ Jv, const double* __restrict__ gr,
                            const double* __restrict__ gmax, double* __restrict__ phi)
{
    const long P = g.P;
    const long nint = n_interior(g);
    const double G = *gmax;
    for (long q = blockIdx.x * (long)blockDim.x + threadIdx.x; q < nint; q += (long)gridDim.x * blockDim.x) {
        int i0, i1, i2;
        const long i = interior_node(g, q, i0, i1, i2);
        double psi = mo.psi[0];
        if (N == 2) {
            const double r1 = sigma_of<N, D>(ph, JU, Jv, P, i, 1, nullptr);
            const double r = sigma_of<N, D>(ph, JU, Jv, P, i, 0, nullptr);
            psi = (mo.psi[0] * r1 + mo.psi[1] * (r - r1)) / r;
        }
        const double v[1] = {G > 0.0 ? exp(-psi * gr[i] / G) : 1.0};
        put_images<D, 1, GH_PLAIN>(g, i0 - g.ng, i1 - g.ng, D == 3 ? i2 - g.ng : 0, v, phi);
    }
}

// channels of a monitor's gradients that theta is formed from (0 without gmax: the
// field is theta already), and a node's, all loaded before the first is used (a
// load behind the arithmetic of the one before is a round trip each)
__device__ __forceinline__ int theta_channels(const MonitorP& mo, const double* gmax)
{
    return !gmax ? 1 : (mo.form ? 2 * mo.nsig : mo.nsig);
}
__device__ __forceinline__ void theta_load(double (&raw)[MON_CH], const double* in, int nch, long P, long i)
{
#pragma unroll
    for (int c = 0; c < MON_CH; c++)
        if (c < nch) raw[c] = in[c * P + i];
}
__device__ __forceinline__ double theta_of(const MonitorP& mo, const double* gmax, const double (&raw)[MON_CH])
{
    if (!gmax) return raw[0];
    double th = 1.0;
#pragma unroll
    for (int s = 0; s < MON_CH; s++) {
        if (s >= mo.nsig) break;
        const double G = gmax[s];
        if (G > 0.0) {
            const double r = raw[s] / G;
            th += mo.form ? mo.alpha[s] * r : mo.alpha[s] * r * r;
        }
        if (s < 2 && mo.form && gmax[mo.nsig + s] > 0.0)   // (at most two variables)
            th += mo.beta[s] * ((mo.nsig == 1 ? raw[1] : raw[2 + s]) / gmax[mo.nsig + s]);
    }
    return sqrt(th);
}
__device__ __forceinline__ double theta_node(const MonitorP& mo, const double* grad, const double* gmax, long P,
                                             long i)
{
    double raw[MON_CH];
    theta_load(raw, grad, theta_channels(mo, gmax), P, i);
    return theta_of(mo, gmax, raw);
}

__global__ void k_theta(Geo g, MonitorP mo, const double* __restrict__ grad, const double* __restrict__ gmax,
                        double* __restrict__ theta)
{
    const long nint = n_interior(g);
    for (long q = blockIdx.x * (long)blockDim.x + threadIdx.x; q < nint; q += (long)gridDim.x * blockDim.x) {
        int i0, i1, i2;
        const long i = interior_node(g, q, i0, i1, i2);
        theta[i] = theta_node(mo, grad, gmax, g.P, i);
    }
}

// lim lowered to the movement limiter's bound for one coordinate that moves
// from x0 to xm between the neighbours lo and hi (1 if it does not move).  The
// quotient is taken only where a product says that it may be below lim, which at
// 1 is where a node moves half a spacing
__device__ __forceinline__ double limit(double lim, double xm, double x0, double lo, double hi)
{
    const double dx = xm - x0, n = (dx < 0.0 ? lo : hi) - x0, d = 2.0 * dx;
    const bool may = dx != 0.0 && !((dx < 0.0 ? -n : n) > lim * fabs(d) * (1.0 + 1e-15));
    return may ? fmin(lim, n / d) : lim;
}

// ---------------------------------------------------------------------------
// 2D: a few thousand to a few hundred thousand nodes, where a launch of a few
// microseconds costs more than its work.  Each block owns a 32 x 16 tile and
// takes several steps of the same kind in LDS on a halo that shrinks by one
// node a step (the halo's updates are computed again by the neighbours);
// nodes outside the grid are read through the face rules and updated like
// any other, which the updates commute with, so no launch needs or writes the
// ghost layers of Theta or of the moving mesh.  800 x 160, five-variable
// monitor, 3 filter passes, 10 Jacobi sweeps: 8 launches instead of 29, 52
// instead of 140 us.  A launch's loads are all issued before the first is used.
// The tile fills the device at that size (250 blocks) and leaves more than half of
// it idle at 350 x 150 (110); no other tile has been measured.
// ---------------------------------------------------------------------------
constexpr int TX2 = 32, TY2 = 16, STEPS2 = 5;
constexpr int RX2 = TX2 + 2 * STEPS2, RY2 = TY2 + 2 * STEPS2;

// the tiles of a 2D grid, one block index (a grid's second extent stops at
// 65535), and the first node of this block's
static dim3 tiles2(const Geo& g) { return dim3((unsigned)((g.n[0] + TX2 - 1) / TX2) * ((g.n[1] + TY2 - 1) / TY2)); }
__device__ __forceinline__ void tile2(const Geo& g, int& ox, int& oy)
{
    const unsigned tx = (g.n[0] + TX2 - 1) / TX2, row = blockIdx.x / tx;
    ox = (int)(blockIdx.x - row * tx) * TX2;
    oy = (int)row * TY2;
}

// the monitor variables of a tile and its one-node halo, evaluated once per
// node from one load of its state, then |grad| (and |lap|) at the tile's nodes
// and their maxima
template <int N, int SIG>
__global__ void __launch_bounds__(256)
k_monitor2(Phys ph, Geo g, MonitorP mo, const double* __restrict__ JU, const double* __restrict__ Jv,
           double* __restrict__ grad, double* __restrict__ gmax)
{
    constexpr int HX = TX2 + 2, HY = TY2 + 2, NV = SIG == 2 ? MON_CH : (SIG == 1 ? 4 : 3);
    __shared__ double Sg[NV][HY][HX];
    __shared__ double part[4][MON_CH];
    const long P = g.P;
    int ox, oy;
    tile2(g, ox, oy);
    const double ih0 = 1.0 / (2.0 * g.dxi[0]), ih1 = 1.0 / (2.0 * g.dxi[1]);
    const double il0 = 1.0 / (g.dxi[0] * g.dxi[0]), il1 = 1.0 / (g.dxi[1] * g.dxi[1]);
    // (a monitor may name a variable more than once; NV of them fit at a time)
    for (int s0 = 0; s0 < mo.nsig; s0 += NV) {
        const int ns = min(NV, mo.nsig - s0);
        for (int q = threadIdx.x; q < HX * HY; q += 256) {
            const int hx = q % HX, hy = q / HX;
            const int gx = ox + hx - 1 + g.ng, gy = oy + hy - 1 + g.ng;
            if (gx >= g.np[0] || gy >= g.np[1]) continue;
            const long i = (long)gy * g.np[0] + gx;
            double v[6];   // the variables by code
            if constexpr (SIG == 0) {
                const double Jq = Jv[i];
                v[1] = JU[i] / Jq;
                v[2] = N > 1 ? JU[P + i] / Jq : v[1];
                v[0] = N > 1 ? v[1] + v[2] : v[1];
            } else {
                NodeState<N, 2> st;
                load_state<N, 2>(ph, JU, Jv, P, i, st);
                v[0] = st.rho;
                v[1] = st.U[0];
                v[2] = st.U[N - 1];
                v[3] = st.p;
                if constexpr (SIG == 2) {
                    v[4] = sqrt(st.v[0] * st.v[0] + st.v[1] * st.v[1]);
                    v[5] = mo.phi ? mo.phi[i] : 0.0;
                }
            }
#pragma unroll
            for (int s = 0; s < NV; s++)
                if (s < ns) {
                    const int sig = mo.sigma[s0 + s];
                    double w = v[0];
#pragma unroll
                    for (int c = 1; c < (SIG == 2 ? 6 : (SIG == 1 ? 4 : 3)); c++) w = sig == c ? v[c] : w;
                    Sg[s][hy][hx] = w;
                }
        }
        __syncthreads();
        for (int s = 0; s < ns; s++) {
            double mg = 0.0, ml = 0.0;
            for (int q = threadIdx.x; q < TX2 * TY2; q += 256) {
                const int hx = q % TX2 + 1, hy = q / TX2 + 1;
                const int x = ox + hx - 1, y = oy + hy - 1;
                if (x >= g.n[0] || y >= g.n[1]) continue;
                const long i = (long)(y + g.ng) * g.np[0] + (x + g.ng);
                const double xp = Sg[s][hy][hx + 1], xm = Sg[s][hy][hx - 1];
                const double yp = Sg[s][hy + 1][hx], ym = Sg[s][hy - 1][hx];
                const double d0 = (xp - xm) * ih0, d1 = (yp - ym) * ih1;
                const double gv = sqrt(d0 * d0 + d1 * d1);
                grad[(s0 + s) * P + i] = gv;
                mg = fmax(mg, gv);
                if (mo.form) {
                    const double c0 = Sg[s][hy][hx];
                    const double lap = fabs((xp - 2.0 * c0 + xm) * il0 + (yp - 2.0 * c0 + ym) * il1);
                    grad[(mo.nsig + s0 + s) * P + i] = lap;
                    ml = fmax(ml, lap);
                }
            }
            mg = wave_max(mg);
            if (mo.form) ml = wave_max(ml);
            if ((threadIdx.x & 63) == 0) {
                part[threadIdx.x >> 6][s0 + s] = mg;
                if (mo.form) part[threadIdx.x >> 6][mo.nsig + s0 + s] = ml;
            }
        }
        __syncthreads();   // (the next variables overwrite the tile)
    }
    const int t = threadIdx.x;
    if (t < (mo.form ? 2 * mo.nsig : mo.nsig))
        scalar_max(gmax + t, fmax(fmax(part[0][t], part[1][t]), fmax(part[2][t], part[3][t])));
}

// The region of a tile: RX2 x RY2 nodes around it whatever the number of
// steps, R2S of them a thread (fixed positions, so no step divides an index); a
// node is at distance e outside the tile and takes part in step p while
// e <= steps - p.
constexpr int NT2 = 384, R2S = (RX2 * RY2 + NT2 - 1) / NT2;

struct Region2 {
    int x[R2S], y[R2S], e[R2S];
    __device__ __forceinline__ Region2(int t)
    {
#pragma unroll
        for (int r = 0; r < R2S; r++) {
            const int q = t + r * NT2;
            x[r] = q % RX2;
            y[r] = q / RX2;
            const int ex = max(STEPS2 - x[r], x[r] - (STEPS2 + TX2 - 1)), ey = max(STEPS2 - y[r], y[r] - (STEPS2 + TY2 - 1));
            e[r] = q < RX2 * RY2 ? max(0, max(ex, ey)) : 1 << 20;
        }
    }
};

// `steps` passes of the low-pass filter; with gmax, theta is formed from the
// monitor's gradients `in` first
__global__ void __launch_bounds__(NT2)
k_filter2(Geo g, MonitorP mo, const double* __restrict__ in, const double* __restrict__ gmax,
          double* __restrict__ out, int steps)
{
    __shared__ double F[2][RY2][RX2];
    int ox, oy;
    tile2(g, ox, oy);
    const Region2 R(threadIdx.x);
    // every load of the thread's nodes before the first is used
    const int nch = theta_channels(mo, gmax);
    double raw[R2S][MON_CH];
#pragma unroll
    for (int r = 0; r < R2S; r++) {
        double sg, off;
        const bool on = R.e[r] <= steps;
        const int ix = on ? mesh_image(g, 0, ox + R.x[r] - STEPS2, sg, off) : 0;
        const int iy = on ? mesh_image(g, 1, oy + R.y[r] - STEPS2, sg, off) : 0;
        theta_load(raw[r], in, nch, g.P, (long)(iy + g.ng) * g.np[0] + (ix + g.ng));
    }
#pragma unroll
    for (int r = 0; r < R2S; r++)
        if (R.e[r] <= steps) F[0][R.y[r]][R.x[r]] = theta_of(mo, gmax, raw[r]);
    __syncthreads();
    for (int p = 1; p <= steps; p++) {
        const double (*A)[RX2] = F[(p - 1) & 1];
        double (*B)[RX2] = F[p & 1];
#pragma unroll
        for (int r = 0; r < R2S; r++) {
            if (R.e[r] > steps - p) continue;
            const int x = R.x[r], y = R.y[r];
            const double r0 = 0.25 * A[y - 1][x - 1] + 0.5 * A[y - 1][x] + 0.25 * A[y - 1][x + 1];
            const double r1 = 0.25 * A[y][x - 1] + 0.5 * A[y][x] + 0.25 * A[y][x + 1];
            const double r2 = 0.25 * A[y + 1][x - 1] + 0.5 * A[y + 1][x] + 0.25 * A[y + 1][x + 1];
            B[y][x] = 0.25 * r0 + 0.5 * r1 + 0.25 * r2;
        }
        __syncthreads();
    }
#pragma unroll
    for (int r = 0; r < R2S; r++) {
        const int x = ox + R.x[r] - STEPS2, y = oy + R.y[r] - STEPS2;
        if (R.e[r] > 0 || x >= g.n[0] || y >= g.n[1]) continue;
        out[(long)(y + g.ng) * g.np[0] + (x + g.ng)] = F[steps & 1][R.y[r]][R.x[r]];
    }
}

// `steps` Jacobi sweeps of the mesh equations; resid: the sweeps' residuals;
// with xn (the last launch of a call) also the movement limiter's bound
// against it, into the ordered key `bound`.  Theta is frozen, so a node's four
// weights and the reciprocal of their sum stay in registers.
__global__ void __launch_bounds__(NT2)
k_jacobi2(Geo g, const double* __restrict__ th, const double* __restrict__ xa, double* __restrict__ xb, int steps,
          double* __restrict__ resid, const double* __restrict__ xn, unsigned long long* __restrict__ bound)
{
    __shared__ double Ts[RY2][RX2];
    __shared__ double Xs[2][2][RY2][RX2];   // buffer, component
    __shared__ double part[NT2 / 64];
    const long P = g.P;
    int ox, oy;
    tile2(g, ox, oy);
    const Region2 R(threadIdx.x);
    const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
    // every load of the thread's nodes before the first is used
    double t0[R2S], x0[R2S], x1[R2S], sg[R2S][2], of[R2S][2];
#pragma unroll
    for (int r = 0; r < R2S; r++) {
        const bool on = R.e[r] <= steps;
        const int ix = on ? mesh_image(g, 0, ox + R.x[r] - STEPS2, sg[r][0], of[r][0]) : 0;
        const int iy = on ? mesh_image(g, 1, oy + R.y[r] - STEPS2, sg[r][1], of[r][1]) : 0;
        const long i = (long)(iy + g.ng) * g.np[0] + (ix + g.ng);
        t0[r] = th[i];
        x0[r] = xa[i];
        x1[r] = xa[P + i];
    }
#pragma unroll
    for (int r = 0; r < R2S; r++) {
        if (R.e[r] > steps) continue;
        Ts[R.y[r]][R.x[r]] = t0[r];
        Xs[0][0][R.y[r]][R.x[r]] = fma(sg[r][0], x0[r], of[r][0]);
        Xs[0][1][R.y[r]][R.x[r]] = fma(sg[r][1], x1[r], of[r][1]);
    }
    __syncthreads();
    const double w0 = 1.0 / (g.dxi[0] * g.dxi[0]), w1 = 1.0 / (g.dxi[1] * g.dxi[1]);
    double tp0[R2S], tm0[R2S], tp1[R2S], tm1[R2S], iden[R2S];
#pragma unroll
    for (int r = 0; r < R2S; r++) {
        if (R.e[r] >= steps) continue;
        const int x = R.x[r], y = R.y[r];
        const double t0 = Ts[y][x];
        tp0[r] = 0.5 * (t0 + Ts[y][x + 1]) * w0;
        tm0[r] = 0.5 * (t0 + Ts[y][x - 1]) * w0;
        tp1[r] = 0.5 * (t0 + Ts[y + 1][x]) * w1;
        tm1[r] = 0.5 * (t0 + Ts[y - 1][x]) * w1;
        iden[r] = rcp((tp0[r] + tm0[r]) + (tp1[r] + tm1[r]));
    }
    for (int p = 1; p <= steps; p++) {
        const double (*A0)[RX2] = Xs[(p - 1) & 1][0];
        const double (*A1)[RX2] = Xs[(p - 1) & 1][1];
        double (*B0)[RX2] = Xs[p & 1][0];
        double (*B1)[RX2] = Xs[p & 1][1];
        double res = 0.0;
#pragma unroll
        for (int r = 0; r < R2S; r++) {
            if (R.e[r] > steps - p) continue;
            const int x = R.x[r], y = R.y[r];
            double n0 = tp0[r] * A0[y][x + 1] + tm0[r] * A0[y][x - 1];
            n0 += tp1[r] * A0[y + 1][x] + tm1[r] * A0[y - 1][x];
            double n1 = tp0[r] * A1[y][x + 1] + tm0[r] * A1[y][x - 1];
            n1 += tp1[r] * A1[y + 1][x] + tm1[r] * A1[y - 1][x];
            n0 *= iden[r];
            n1 *= iden[r];
            B0[y][x] = n0;
            B1[y][x] = n1;
            if (R.e[r] == 0 && ox + x - STEPS2 < g.n[0] && oy + y - STEPS2 < g.n[1])
                res = fmax(res, fmax(fabs(n0 - A0[y][x]), fabs(n1 - A1[y][x])));
        }
        if (resid) {
            res = wave_max(res);
            if (lane == 0) part[wid] = res;
        }
        __syncthreads();
        if (resid) {
            if (threadIdx.x == 0) {
                for (int q = 1; q < NT2 / 64; q++) res = fmax(res, part[q]);
                scalar_max(resid + p - 1, res);
            }
            __syncthreads();   // part is written again
        }
    }
    double b = 1.0;
    bool own[R2S];
    long at[R2S];
    double nb[R2S][6];   // x_n there and on either side
#pragma unroll
    for (int r = 0; r < R2S; r++) {
        const int x = ox + R.x[r] - STEPS2, y = oy + R.y[r] - STEPS2;
        own[r] = R.e[r] == 0 && x < g.n[0] && y < g.n[1];
        at[r] = own[r] ? (long)(y + g.ng) * g.np[0] + (x + g.ng) : (long)g.ng * g.np[0] + g.ng;
        if (xn) {
            const double *p = xn + at[r], *q = xn + P + at[r];
            const long n0 = g.np[0];
            nb[r][0] = p[0];
            nb[r][1] = p[-1];
            nb[r][2] = p[1];
            nb[r][3] = q[0];
            nb[r][4] = q[-n0];
            nb[r][5] = q[n0];
        }
    }
#pragma unroll
    for (int r = 0; r < R2S; r++) {
        if (!own[r]) continue;
        const double v[2] = {Xs[steps & 1][0][R.y[r]][R.x[r]], Xs[steps & 1][1][R.y[r]][R.x[r]]};
        if (xn) {
            b = limit(b, v[0], nb[r][0], nb[r][1], nb[r][2]);
            b = limit(b, v[1], nb[r][3], nb[r][4], nb[r][5]);
        }
        xb[at[r]] = v[0];
        xb[P + at[r]] = v[1];
    }
    if (xn) {
        b = wave_min(b);
        if (lane == 0) part[wid] = b;
        __syncthreads();
        if (threadIdx.x == 0) {
            for (int q = 1; q < NT2 / 64; q++) b = fmin(b, part[q]);
            scalar_min(bound, b);
        }
    }
}

// disp = Delta_tau (x^[mu] - x_n), and with xnext also x_{n+1} = x_n + disp; 2D with
// the ghost layers (each ghost node from its image node, as a ghost fill
// gives it), which a fill follows up in 3D.  The limiter's key is decoded here: Delta_tau = min(1, bound) into
// dtau and, when given, dtau_out
template <int D>
__global__ void k_disp(Geo g, const double* __restrict__ xmu, const double* __restrict__ xn,
                       const unsigned long long* __restrict__ bound, double* __restrict__ dtau,
                       double* __restrict__ dtau_out, double* __restrict__ disp, double* __restrict__ xnext,
                       unsigned* __restrict__ status)
{
    const long P = g.P;
    const double d = fmin(1.0, order_value(*bound));
    if (blockIdx.x == 0 && threadIdx.x == 0) {
        *dtau = d;
        if (dtau_out) *dtau_out = d;
        if (!(d > 0.0)) atomicOr(status, 2u);
    }
    const long q = blockIdx.x * (long)blockDim.x + threadIdx.x;
    if (q >= n_interior(g)) return;
    int i0, i1, i2;
    const long i = interior_node(g, q, i0, i1, i2);
    const int z = D == 3 ? i2 - g.ng : 0;
    double v[D], w[D];
#pragma unroll
    for (int c = 0; c < D; c++) {
        const double x0 = xn[c * P + i];
        v[c] = d * (xmu[c * P + i] - x0);
        w[c] = x0 + v[c];
    }
    if constexpr (D == 3) {   // (the images a thread cost 108 us at 256^3, the fill 45)
#pragma unroll
        for (int c = 0; c < D; c++) {
            disp[c * P + i] = v[c];
            if (xnext) xnext[c * P + i] = w[c];
        }
    } else {
        put_images<D, D, GH_DISP>(g, i0 - g.ng, i1 - g.ng, z, v, disp);
        if (xnext) put_images<D, D, GH_MESH>(g, i0 - g.ng, i1 - g.ng, z, w, xnext);
    }
}

// ---------------------------------------------------------------------------
// 3D: bound by HBM (two Jacobi sweeps move 1.25 GB at 4.4 TB/s), so several filter
// passes or Jacobi sweeps walk z together; three sweeps leave one block a
// compute unit and half of its columns halo, 3 + 2 sweeps took 73 us more than
// 2 + 2 + 1.  A block owns TX x TY columns over a chunk of z planes; every thread owns one
// column of the tile plus a halo of S nodes.  Step s of plane z runs as soon as
// step s - 1 has reached plane z + 1; the planes it needs along z are the
// thread's own registers, those in the plane are in LDS (double-buffered, one
// barrier a plane), and its halo is one node narrower.  Nodes outside the grid
// are read through the face rules, as in 2D.  A launch then reads and writes a
// field once for S steps: at 256^3 three filter passes take 123 us instead
// of 3 x 97 us and two Jacobi sweeps 300 us instead of 2 x 307 us (each with the
// ghost fill that they needed).
// ---------------------------------------------------------------------------
template <int TX, int TY, int S>
struct Column3 {
    static constexpr int HX = TX + 2 * S, HY = TY + 2 * S, HN = HX * HY, NT = (HN + 63) / 64 * 64;
};

// S passes of the low-pass filter: the weights 2^-(|j|_1 + 3), j in {-1,0,1}^3, are
// the product of (1/4, 1/2, 1/4) along each direction, so a pass is the
// in-plane sum q of each plane and out = q(z-1)/4 + q(z)/2 + q(z+1)/4.  The sum
// along x comes from the neighbouring lanes (a wave is two rows), which leaves two
// LDS reads a pass instead of nine: 172 instead of 260 us for three, and 123 with
// the monitor channels prefetched.  With
// gmax, theta is formed from the monitor's gradients `in` first
template <int TX, int TY, int S>
__global__ void __launch_bounds__((Column3<TX, TY, S>::NT))
k_filter3(Geo g, MonitorP mo, const double* __restrict__ in, const double* __restrict__ gmax,
          double* __restrict__ out, int zchunk)
{
    constexpr int HX = Column3<TX, TY, S>::HX, HN = Column3<TX, TY, S>::HN;
    static_assert(HX == 32 && HN % 64 == 0, "lanes of a row are neighbours");
    __shared__ double R[S][2][HN + 2 * HX];   // sums along x of the field after s passes, two planes
    int bx, by, bz;
    xcd_tile((g.n[0] + TX - 1) / TX, (g.n[1] + TY - 1) / TY, bx, by, bz);
    const int t = threadIdx.x, lx = t % HX, ly = t / HX;
    const int gx = bx * TX + lx - S, gy = by * TY + ly - S;
    const bool own = lx >= S && lx < S + TX && ly >= S && ly < S + TY && gx < g.n[0] && gy < g.n[1];
    const int zc0 = bz * zchunk, zc1 = min(zc0 + zchunk, g.n[2]);
    if (zc0 >= zc1) return;   // uniform over the block
    double sg, off;
    // (a column beyond a ragged tile's halo reads an image that no written node uses)
    const int ix = mesh_image(g, 0, min(gx, g.n[0] + S), sg, off), iy = mesh_image(g, 1, min(gy, g.n[1] + S), sg, off);
    const long col = (long)(iy + g.ng) * g.np[0] + (ix + g.ng), sz = (long)g.np[0] * g.np[1];
    // PF planes in flight (a plane a round trip to memory left the block waiting)
    constexpr int PF = 2;
    const int nch = theta_channels(mo, gmax);
    double next[PF][MON_CH];
    auto load = [&](int u, int z) {
        double s_, o_;
        theta_load(next[u], in, nch, g.P, col + (mesh_image(g, 2, min(z, zc1 + S - 1), s_, o_) + g.ng) * sz);
    };
    const int row = __builtin_amdgcn_readfirstlane(ly);   // the wave's rows: this one and the next
    double q[S][3];   // in-plane sums of the last three planes after s passes
    double rx[S];     // the own sum along x of the last plane
#pragma unroll
    for (int s = 0; s < S; s++) q[s][0] = q[s][1] = q[s][2] = rx[s] = 0.0;
    const unsigned plane = (unsigned)(sz * sizeof(double)), ob = own ? (unsigned)(col * sizeof(double)) : DROPPED;
    auto store = [&](int z, double v) {   // (a plane below the chunk: dropped)
        buffer_store(out + (max(z, zc0) + g.ng) * sz, z >= zc0 ? plane : 0u, ob, v);
    };
#pragma unroll
    for (int u = 0; u < PF; u++) {   // (with the store that a step has)
        load(u, zc0 - S + u);
        __builtin_amdgcn_sched_barrier(0);
        store(zc0 - 1 - u, 0.0);
        __builtin_amdgcn_sched_barrier(0);
    }
    // plane k enters; the field after s passes has reached plane k - 2 s
    const int kend = zc1 + 2 * S;
    int k0 = zc0 - S;
    do {   // (entered without a test, past which the first loads would sink)
#pragma unroll
        for (int u = 0; u < PF; u++) {
            const int k = k0 + u;
            if (k >= kend) break;   // uniform
            auto enter = [&](int s, double v) {
                rx[s] = 0.25 * lane_below(v) + 0.5 * v + 0.25 * lane_above(v);
                R[s][k & 1][HX + t] = rx[s];
            };
            double vo = 0.0;
#pragma unroll
            for (int s = S - 1; s >= 0; s--) {
                if (row + 1 < s + 1 || row > TY + 2 * S - 2 - s) continue;   // halo used up
                const double* A = &R[s][~k & 1][HX + t];
                q[s][0] = q[s][1];
                q[s][1] = q[s][2];
                q[s][2] = 0.25 * A[-HX] + 0.5 * rx[s] + 0.25 * A[HX];
                const double v = 0.25 * q[s][0] + 0.5 * q[s][1] + 0.25 * q[s][2];
                if (s + 1 < S) enter(s + 1, v);
                else vo = v;
            }
            store(k - 2 * S, vo);
            enter(0, theta_of(mo, gmax, next[u]));
            load(u, k + PF);
            __syncthreads();
        }
    } while ((k0 += PF) < kend);
}

// S Jacobi sweeps of the mesh equations (1 or 2); resid: their residuals; LIM (the
// last launch of a call): also the movement limiter's bound against x_n, whose
// planes walk along, into the ordered key `bound`.  Two blocks share a compute unit,
// but for two sweeps with the limiter: 81 KB and 144 registers a thread.  Within 128
// registers and 73 KB (no rows between the planes) 25 registers spill and ten sweeps
// at 256^3 take 2473 us, as it is 2153, and with the last two sweeps in launches of
// their own 2082, but six then take 1763 instead of 1555 and two 1087 instead of 938.
template <int TX, int TY, int S, bool LIM>
__global__ void __launch_bounds__((Column3<TX, TY, S>::NT)) __attribute__((amdgpu_waves_per_eu(S == 2 && LIM ? 2 : 4, 8)))
k_jacobi3(Geo g, const double* __restrict__ th, const double* __restrict__ xa, double* __restrict__ xb,
          double* __restrict__ resid, const double* __restrict__ xn, unsigned long long* __restrict__ bound,
          int zchunk)
{
    constexpr int HX = Column3<TX, TY, S>::HX, HN = Column3<TX, TY, S>::HN;
    static_assert(HX == 32 && HN % 64 == 0, "lanes of a row are neighbours");
    constexpr int HP = HN + 2 * HX;         // (a row on either side, read and not used)
    __shared__ double Ts[S + 1][HP];        // theta of the last planes
    __shared__ double Xs[S][2][3][HP];      // x before step s, two planes
    __shared__ double Ns[LIM ? S + 1 : 1][LIM ? HP : 1];   // x_n's second component
    __shared__ double part[S + LIM][HN / 64];   // the waves' maxima and minima
    const long P = g.P;
    int bx, by, bz;
    xcd_tile((g.n[0] + TX - 1) / TX, (g.n[1] + TY - 1) / TY, bx, by, bz);
    const int t = threadIdx.x, lx = t % HX, ly = t / HX;
    const int gx = bx * TX + lx - S, gy = by * TY + ly - S;
    const bool own = lx >= S && lx < S + TX && ly >= S && ly < S + TY && gx < g.n[0] && gy < g.n[1];
    const int row = __builtin_amdgcn_readfirstlane(ly);   // the wave's rows: this one and the next
    const int zc0 = bz * zchunk, zc1 = min(zc0 + zchunk, g.n[2]);
    if (zc0 >= zc1) return;   // uniform over the block
    const long sz = (long)g.np[0] * g.np[1];
    // (a column beyond a ragged tile's halo reads an image that no written node uses)
    double s0, b0, s1, b1;
    const int ix = mesh_image(g, 0, min(gx, g.n[0] + S), s0, b0), iy = mesh_image(g, 1, min(gy, g.n[1] + S), s1, b1);
    const unsigned cb = ((unsigned)(iy + g.ng) * g.np[0] + (ix + g.ng)) * (unsigned)sizeof(double);
    const unsigned ob = own ? cb : DROPPED, plane = (unsigned)(sz * sizeof(double));
    double h2[3];
#pragma unroll
    for (int k = 0; k < 3; k++) h2[k] = 0.5 / (g.dxi[k] * g.dxi[k]);
    double tr[S + 2];        // theta of the own column, planes k - S - 1 .. k
    double xr[S][3][3];      // x before step s, the last three planes
    double res[S];
    double lim = 1.0;
#pragma unroll
    for (int s = 0; s < S; s++) {
        res[s] = 0.0;
#pragma unroll
        for (int c = 0; c < 3; c++) xr[s][c][0] = xr[s][c][1] = xr[s][c][2] = 0.0;
    }
#pragma unroll
    for (int r = 0; r < S + 2; r++) tr[r] = 0.0;
    double nr[LIM ? 3 : 1][S + 2];   // x_n of the own column, planes k - S - 1 .. k
    // PF planes in flight
    constexpr int PF = 2;
    double tn[PF], pn[PF][3], nn[LIM ? PF : 1][3];
    auto fetch = [&](int u, int z) {
        double s2, b2;
        const long i = (mesh_image(g, 2, min(z, zc1 + S - 1), s2, b2) + g.ng) * sz;
        tn[u] = buffer_load(th + i, plane, cb);
#pragma unroll
        for (int c = 0; c < 3; c++) pn[u][c] = buffer_load(xa + c * P + i, plane, cb);
        if constexpr (LIM)
#pragma unroll
            for (int c = 0; c < 3; c++) nn[u][c] = buffer_load(xn + c * P + i, plane, cb);
    };
    auto store = [&](int z, const double (&v)[3]) {   // (a plane outside the chunk: dropped)
        const bool on = z >= zc0 && z < zc1;
#pragma unroll
        for (int c = 0; c < 3; c++)
            buffer_store(xb + c * P + ((on ? z : zc0) + g.ng) * sz, on ? plane : 0u, ob, v[c]);
    };
#pragma unroll
    for (int u = 0; u < PF; u++) {   // (with the stores that a step has)
        fetch(u, zc0 - S + u);
        __builtin_amdgcn_sched_barrier(0);
        store(zc0 - 1 - u, {0.0, 0.0, 0.0});
        __builtin_amdgcn_sched_barrier(0);
    }
    // plane k enters; step s (0 .. S-1) runs at plane k - 1 - s
    int k0 = zc0 - S;
    do {   // (entered without a test, past which the first loads would sink)
#pragma unroll
        for (int u = 0; u < PF; u++) {
            const int k = k0 + u;
            if (k >= zc1 + S) break;   // uniform
            double s2, b2;
            mesh_image(g, 2, k, s2, b2);
            const double sc[3] = {s0, s1, s2}, bc[3] = {b0, b1, b2};
#pragma unroll
            for (int r = 0; r < S + 1; r++) tr[r] = tr[r + 1];
            double t1 = tn[u];
            asm volatile("" : "+v"(t1));   // (a copy: a load into the register of a ring's value is moved, and so waited for, at once)
            tr[S + 1] = t1;
            Ts[(k + 3 * S + 3) % (S + 1)][HX + t] = t1;
#pragma unroll
            for (int c = 0; c < 3; c++) {
                const double x = fma(sc[c], pn[u][c], bc[c]);
                xr[0][c][0] = xr[0][c][1];
                xr[0][c][1] = xr[0][c][2];
                xr[0][c][2] = x;
                Xs[0][k & 1][c][HX + t] = x;
                if constexpr (LIM) {
                    const double y = fma(sc[c], nn[u][c], bc[c]);
#pragma unroll
                    for (int r = 0; r < S + 1; r++) nr[c][r] = nr[c][r + 1];
                    nr[c][S + 1] = y;
                    if (c == 1) Ns[(k + 3 * S + 3) % (S + 1)][HX + t] = y;
                }
            }
            fetch(u, k + PF);
            double v[3] = {0.0, 0.0, 0.0};
#pragma unroll
            for (int s = 0; s < S; s++) {
                const int z = k - 1 - s;
                if (row + 1 < s + 1 || row > TY + 2 * S - 2 - s) continue;   // halo used up
                const double* T = &Ts[(z + 3 * S + 3) % (S + 1)][HX + t];
                const double t0 = tr[S - s];
                double tp[3], tm[3];
                tp[0] = h2[0] * (t0 + T[1]);
                tm[0] = h2[0] * (t0 + T[-1]);
                tp[1] = h2[1] * (t0 + T[HX]);
                tm[1] = h2[1] * (t0 + T[-HX]);
                tp[2] = h2[2] * (t0 + tr[S - s + 1]);
                tm[2] = h2[2] * (t0 + tr[S - s - 1]);
                const double iden = rcp(((tp[0] + tm[0]) + (tp[1] + tm[1])) + (tp[2] + tm[2]));
                double r = res[s];
#pragma unroll
                for (int c = 0; c < 3; c++) {
                    const double* A = &Xs[s][z & 1][c][HX + t];
                    double num = tp[0] * A[1];
                    num = fma(tm[0], A[-1], num);
                    num = fma(tp[1], A[HX], num);
                    num = fma(tm[1], A[-HX], num);
                    num = fma(tp[2], xr[s][c][2], num);
                    num = fma(tm[2], xr[s][c][0], num);
                    v[c] = num * iden;
                    r = fmax(r, fabs(v[c] - xr[s][c][1]));
                }
                res[s] = own && z >= zc0 && z < zc1 ? r : res[s];
                if (s + 1 < S) {
#pragma unroll
                    for (int c = 0; c < 3; c++) {
                        xr[s + 1 < S ? s + 1 : s][c][0] = xr[s + 1 < S ? s + 1 : s][c][1];
                        xr[s + 1 < S ? s + 1 : s][c][1] = xr[s + 1 < S ? s + 1 : s][c][2];
                        xr[s + 1 < S ? s + 1 : s][c][2] = v[c];
                        Xs[s + 1 < S ? s + 1 : s][z & 1][c][HX + t] = v[c];
                    }
                } else {
                    double lo[3], hi[3];
                    if constexpr (LIM) {   // plane z = k - S: x_n's own column at nr[.][1], its neighbours
                        const double* A = &Ns[(z + 3 * S + 3) % (S + 1)][HX + t];
                        lo[0] = lane_below(nr[0][1]);
                        hi[0] = lane_above(nr[0][1]);
                        lo[1] = A[-HX];
                        hi[1] = A[HX];
                        lo[2] = nr[2][0];
                        hi[2] = nr[2][2];
                    }
                    if constexpr (LIM)
                        if (own && z >= zc0 && z < zc1)
#pragma unroll
                            for (int c = 0; c < 3; c++) lim = limit(lim, v[c], nr[c][1], lo[c], hi[c]);
                }
            }
            store(k - S, v);
            __syncthreads();
        }
    } while ((k0 += PF) < zc1 + S);
    if (!LIM && !resid) return;
#pragma unroll
    for (int s = 0; s < S; s++) {
        const double r = wave_max(res[s]);
        if ((t & 63) == 0) part[s][t >> 6] = r;
    }
    if constexpr (LIM) {
        lim = wave_min(lim);
        if ((t & 63) == 0) part[S][t >> 6] = lim;
    }
    __syncthreads();
    if (resid && t < S) {
        double r = part[t][0];
        for (int q = 1; q < HN / 64; q++) r = fmax(r, part[t][q]);
        scalar_max(resid + t, r);
    }
    if (LIM && t == S) {
        for (int q = 0; q < HN / 64; q++) lim = fmin(lim, part[S][q]);
        scalar_min(bound, lim);
    }
}

// |grad rho| into gr, then the schlieren function
template <int N, int D>
static void launch_schlieren(const Phys& ph, const Geo& g, const MonitorP& mo, const double* JU,
                             const double* J, double* gr, double* gmax, double* phi, int nb, int gi,
                             hipStream_t s)
{
    if constexpr (D == 2) {   // the monitor's gradient of one variable, the density
        MonitorP m{};
        m.nsig = 1;
        hipLaunchKernelGGL((k_monitor2<N, 0>), tiles2(g), dim3(256), 0, s, ph, g, m, JU, J, gr, gmax);
    } else {
        hipLaunchKernelGGL((k_rho_grad<N, D>), dim3(nb), dim3(256), 0, s, ph, g, JU, J, gr, gmax);
    }
    hipLaunchKernelGGL((k_schlieren<N, D>), dim3(gi), dim3(256), 0, s, ph, g, mo, JU, J, gr, gmax, phi);
}

template <int N>
static auto monitor2_kernel(int sigmode)
{
    return sigmode == 2 ? k_monitor2<N, 2> : (sigmode == 1 ? k_monitor2<N, 1> : k_monitor2<N, 0>);
}
template <int N>
static auto monitor3_kernel(int sigmode)
{
    return sigmode == 2 ? k_monitor_grad3<N, 2> : (sigmode == 1 ? k_monitor_grad3<N, 1> : k_monitor_grad3<N, 0>);
}

hipError_t mesh_redistribute(const Phys& ph, const Geo& g, const MonitorP& mo_in, const double* JU,
                             const double* J, const double* xn, double* disp, MeshWork& w,
                             double* dtau_out, double* resid_out, unsigned* status, hipStream_t s,
                             double* xnext)
{
    MonitorP mo = mo_in;
    mo.phi = w.phi;
    const bool d3 = g.dim == 3;
    const long nint = (long)g.n[0] * g.n[1] * (d3 ? g.n[2] : 1);
    // the schlieren function first when the monitor uses it (th1 holds
    // |grad rho| until the filter overwrites it)
    bool use_phi = false, ext = false, press = false;
    for (int q = 0; q < mo.nsig; q++) {
        use_phi = use_phi || mo.sigma[q] == 5;
        ext = ext || mo.sigma[q] >= 4;
        press = press || mo.sigma[q] == 3;
    }
    // the monitor kernels carry only the variables they are asked for
    const int sigmode = ext ? 2 : (press ? 1 : 0);
    hipLaunchKernelGGL(k_mesh_begin, dim3(1), dim3(256), 0, s, w.scal, resid_out, mo.n_sweeps);
    if (use_phi)
        ES_DISPATCH_ND(ph, g, launch_schlieren, ph, g, mo, JU, J, w.th1, w.scal + 7, w.phi, red_grid(nint),
                       grid_for(nint), s);
    // monitor and its global maxima (3D: three blocks a compute unit, two with the pressure)
    if (d3) {
        const int jx = (g.n[0] + 29) / 30, jy = (g.n[1] + 13) / 14, zc = z_chunk(g.n[2], (long)jx * jy, 2, (sigmode ? 2 : 3) * UNITS);
        hipLaunchKernelGGL(ph.nspec == 1 ? monitor3_kernel<1>(sigmode) : monitor3_kernel<2>(sigmode),
                           dim3(jx * jy * ((g.n[2] + zc - 1) / zc)), dim3(512), 0, s, ph, g, mo, JU, J, w.grad, w.scal, zc);
    } else {
        hipLaunchKernelGGL(ph.nspec == 1 ? monitor2_kernel<1>(sigmode) : monitor2_kernel<2>(sigmode), tiles2(g), dim3(256),
                           0, s, ph, g, mo, JU, J, w.grad, w.scal);
    }
    // 3D launches over z chunks of tiles of nt threads, `blocks` of them resident on a
    // compute unit
    auto march = [&](auto kern, int tx, int ty, int nt, int extra, int blocks, auto... args) {
        const int gx = (g.n[0] + tx - 1) / tx, gy = (g.n[1] + ty - 1) / ty;
        const int zc = z_chunk(g.n[2], (long)gx * gy, extra, blocks * UNITS);
        hipLaunchKernelGGL(kern, dim3(gx * gy * ((g.n[2] + zc - 1) / zc)), dim3(nt), 0, s, g, args..., zc);
    };
    // theta and the filter passes (none: theta alone)
    double *th = w.th0, *th2 = w.th1;
    for (int left = mo.n_smooth, first = 1; first || left > 0; first = 0) {
        const int steps = std::min(left, d3 ? 3 : STEPS2);
        const double* in = first ? w.grad : th;
        const double* gmax = first ? w.scal : nullptr;
        if (!d3) {
            hipLaunchKernelGGL(k_filter2, tiles2(g), dim3(NT2), 0, s, g, mo, in, gmax, th2, steps);
        } else if (steps == 0) {
            hipLaunchKernelGGL(k_theta, dim3(grid_for(nint)), dim3(256), 0, s, g, mo, in, gmax, th2);
        } else {
            if (steps == 1) march(k_filter3<30, 20, 1>, 30, 20, 704, 3, 2, mo, in, gmax, th2);
            else if (steps == 2) march(k_filter3<28, 18, 2>, 28, 18, 704, 6, 2, mo, in, gmax, th2);
            else march(k_filter3<26, 16, 3>, 26, 16, 704, 9, 2, mo, in, gmax, th2);
        }
        std::swap(th, th2);
        left -= steps;
    }
    // Jacobi sweeps: the first launch reads x_n itself, then xa and xb alternate;
    // the last one takes the limiter's bound
    const double* xcur = xn;
    double *xa = w.xa, *xb = w.xb;
    unsigned long long* key = reinterpret_cast<unsigned long long*>(w.scal + 8);
    for (int nu = 0; nu < mo.n_sweeps;) {
        const int steps = std::min(mo.n_sweeps - nu, d3 ? 2 : STEPS2);
        const double* xl = nu + steps == mo.n_sweeps ? xn : nullptr;
        double* res = resid_out ? resid_out + nu : nullptr;
        if (!d3) {
            hipLaunchKernelGGL(k_jacobi2, tiles2(g), dim3(NT2), 0, s, g, th, xcur, xa, steps, res, xl, key);
        } else {
            if (steps == 1 && xl) march(k_jacobi3<30, 14, 1, true>, 30, 14, 512, 2, 2, th, xcur, xa, res, xl, key);
            else if (steps == 1) march(k_jacobi3<30, 14, 1, false>, 30, 14, 512, 2, 2, th, xcur, xa, res, xl, key);
            else if (xl) march(k_jacobi3<28, 12, 2, true>, 28, 12, 512, 4, 1, th, xcur, xa, res, xl, key);
            else march(k_jacobi3<28, 12, 2, false>, 28, 12, 512, 4, 2, th, xcur, xa, res, xl, key);
        }
        xcur = xa;
        std::swap(xa, xb);
        nu += steps;
    }
    const dim3 nodes((unsigned)((nint + 255) / 256));
    if (d3) {
        hipLaunchKernelGGL(k_disp<3>, nodes, dim3(256), 0, s, g, xcur, xn, key, w.scal + 6, dtau_out, disp, xnext, status);
        const hipError_t e = hipGetLastError();
        return e != hipSuccess ? e : fill_ghosts2(g, disp, 3, GH_DISP, xnext, 3, GH_MESH, s);
    }
    hipLaunchKernelGGL(k_disp<2>, nodes, dim3(256), 0, s, g, xcur, xn, key, w.scal + 6, dtau_out, disp, xnext, status);
    return hipGetLastError();
}

}  // namespace es

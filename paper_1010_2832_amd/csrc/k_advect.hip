// Advection half of the fractional step (Section 10): first-order
// semi-Lagrangian advection of the face velocities (bilinear in 2D,
// trilinear in 3D) and of the nodal liquid level set, FP64.
//
// * Velocity extension: faces the last Stokes step defined (K > 0, or
//   W_F = 0) are known; each of `layers` passes gives every unknown face with
//   a known neighbour of the same component (one index step along an axis)
//   the mean of those neighbours, summed along x (i-1, i+1), then y, then z.
// * Interpolation of a sample type of stagger s at a point given in index
//   units of h from the box corner: continuous index P - s/2, clamped to
//   [0, shape - 1] per axis, base min(floor, shape - 2), multilinear weights.
// * Departure point of a sample: its position minus dt v / h (index units),
//   v the interpolated extended velocity.
#include "vfs_internal.h"

namespace vfs {
namespace {

enum : uint8_t { FK = 1 };

// Place of a point along an axis of a lattice of n samples of stagger s, by
// index units: base sample and weight of the next.
__device__ __forceinline__ void axis_weights(double P, int s, int n, int& i0, double& t) {
    double xi = P - 0.5 * s;
    xi = fmin(fmax(xi, 0.0), (double)(n - 1));
    int f = (int)floor(xi);
    i0 = min(f, max(n - 2, 0));
    t = xi - (double)i0;
}

// Multilinear value of the lattice at `src` (extents n, staggers s, element
// steps `step`) at the index-space point P.  The dimension is a compile-time
// constant and a corner is a step from the base: with the axes looped over at run
// time and an index product for each corner, address arithmetic took most of
// the time: at 256^3 the velocity took 5.37 ms and now 0.99, the level set 1.45 and
// 0.42 (0.2 and 0.15 for their bytes; the gathers' loads are what is left).  The
// roundings are those of the loops: weights multiplied x, y, z, one fused step a
// corner.
template <int DIM>
__device__ __forceinline__ double interp(const double* __restrict__ src, const int (&n)[DIM],
                                         const int (&s)[DIM], const long long (&step)[DIM],
                                         const double (&P)[DIM]) {
#pragma clang fp contract(off)
    double w[DIM][2];
    long long d[DIM];
#pragma unroll
    for (int b = 0; b < DIM; ++b) {
        int i0;
        double t;
        axis_weights(P[b], s[b], n[b], i0, t);
        w[b][0] = 1.0 - t;
        w[b][1] = t;
        src += i0 * step[b];
        d[b] = n[b] > 1 ? step[b] : 0;
    }
    double v[1 << DIM];
#pragma unroll
    for (int c = 0; c < 1 << DIM; ++c) {
        long long o = 0;
#pragma unroll
        for (int b = 0; b < DIM; ++b)
            if ((c >> b) & 1) o += d[b];
        v[c] = src[o];
    }
    double acc = 0.0;
#pragma unroll
    for (int c = 0; c < 1 << DIM; ++c) {
        double q = w[0][c & 1];
#pragma unroll
        for (int b = 1; b < DIM; ++b) q *= w[b][(c >> b) & 1];
        acc = __builtin_fma(q, v[c], acc);
    }
    return acc;
}

// value of face component a (padded slices `u`) at the index-space point P
template <int DIM>
__device__ __forceinline__ double interp_face(const Geo& g, const double* __restrict__ u, int a,
                                              const double (&P)[DIM]) {
    int n[DIM], s[DIM];
    long long step[DIM];
    const int nn[3] = {g.nx, g.ny, g.nz};
    const long long st[3] = {1, (long long)g.PX, (long long)g.PX * g.PY};
#pragma unroll
    for (int b = 0; b < DIM; ++b) {
        s[b] = b == a ? 0 : 1;
        n[b] = nn[b] + 1 - s[b];
        step[b] = st[b];
    }
    const long long base = DIM == 2 ? g.idx(0, 0) : g.idx(0, 0, 0);
    return interp<DIM>(u + (long long)a * g.NP + base, n, s, step, P);
}

__device__ __forceinline__ bool face_valid(const Geo& g, int a, int i, int j, int k) {
    const int n[3] = {g.nx, g.ny, g.nz};
    const int id[3] = {i, j, k};
    for (int b = 0; b < g.dim; ++b) {
        const int lim = n[b] + (b == a ? 1 : 0);
        if (id[b] < 0 || id[b] >= lim) return false;
    }
    return true;
}

__device__ __forceinline__ long long anchor(const Geo& g, int i, int j, int k) {
    return g.dim == 2 ? g.idx(i, j) : g.idx(i, j, k);
}

// known flags of the velocity of the last Stokes step
__global__ void k_known_faces(Geo g, const uint8_t* __restrict__ fflag,
                              const double* __restrict__ WF, uint8_t* __restrict__ known) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    const int j = blockIdx.y * blockDim.y + threadIdx.y;
    const int k = blockIdx.z * blockDim.z + threadIdx.z;
    if (i > g.nx || j > g.ny || k > (g.dim == 3 ? g.nz : 0)) return;
    const long long o = anchor(g, i, j, k);
    for (int a = 0; a < g.dim; ++a) {
        const long long q = (long long)a * g.NP + o;
        uint8_t kn = 0;
        if (face_valid(g, a, i, j, k))
            kn = ((fflag[q] & FK) || WF[(long long)(1 + a) * g.NP + o] == 0.0) ? 1 : 0;
        known[q] = kn;
    }
}

// one extension layer: vin/kin -> vout/kout
__global__ void k_extend(Geo g, const double* __restrict__ vin, const uint8_t* __restrict__ kin,
                         double* __restrict__ vout, uint8_t* __restrict__ kout) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    const int j = blockIdx.y * blockDim.y + threadIdx.y;
    const int k = blockIdx.z * blockDim.z + threadIdx.z;
    if (i > g.nx || j > g.ny || k > (g.dim == 3 ? g.nz : 0)) return;
    const long long o = anchor(g, i, j, k);
    const long long step[3] = {1, (long long)g.PX, (long long)g.PX * g.PY};
    const int id[3] = {i, j, k};
    for (int a = 0; a < g.dim; ++a) {
        const long long q = (long long)a * g.NP + o;
        if (!face_valid(g, a, i, j, k)) continue;
        if (kin[q]) {
            vout[q] = vin[q];
            kout[q] = 1;
            continue;
        }
        double acc = 0.0;
        int cnt = 0;
        for (int b = 0; b < g.dim; ++b) {
            int lo[3] = {id[0], id[1], id[2]};
            lo[b] -= 1;
            if (face_valid(g, a, lo[0], lo[1], lo[2]) && kin[q - step[b]]) {
                acc += vin[q - step[b]];
                ++cnt;
            }
            int hi[3] = {id[0], id[1], id[2]};
            hi[b] += 1;
            if (face_valid(g, a, hi[0], hi[1], hi[2]) && kin[q + step[b]]) {
                acc += vin[q + step[b]];
                ++cnt;
            }
        }
        if (cnt > 0) {
            vout[q] = acc / (double)cnt;
            kout[q] = 1;
        } else {
            vout[q] = vin[q];
            kout[q] = 0;
        }
    }
}

// semi-Lagrangian velocity: every valid face of every component
template <int DIM>
__global__ __launch_bounds__(256) void k_advect_u(Geo g, double dt, const double* __restrict__ uext,
                                                  double* __restrict__ uout) {
    const int id[3] = {(int)(blockIdx.x * blockDim.x + threadIdx.x),
                       (int)(blockIdx.y * blockDim.y + threadIdx.y),
                       (int)(blockIdx.z * blockDim.z + threadIdx.z)};
    if (id[0] > g.nx || id[1] > g.ny || (DIM == 3 && id[2] > g.nz)) return;
    const long long o = DIM == 2 ? g.idx(id[0], id[1]) : g.idx(id[0], id[1], id[2]);
    const double sc = dt / g.h;
#pragma unroll
    for (int a = 0; a < DIM; ++a) {
        if (!face_valid(g, a, id[0], id[1], id[2])) continue;
        double P[DIM], D[DIM];
#pragma unroll
        for (int b = 0; b < DIM; ++b) P[b] = (double)id[b] + (b != a ? 0.5 : 0.0);
#pragma unroll
        for (int b = 0; b < DIM; ++b) D[b] = __builtin_fma(-sc, interp_face<DIM>(g, uext, b, P), P[b]);
        uout[(long long)a * g.NP + o] = interp_face<DIM>(g, uext, a, D);
    }
}

// semi-Lagrangian level set at the nodes (compact arrays)
template <int DIM>
__global__ __launch_bounds__(256) void k_advect_phi(Geo g, double dt, const double* __restrict__ uext,
                                                    const double* __restrict__ phi,
                                                    double* __restrict__ out) {
    const int id[3] = {(int)(blockIdx.x * blockDim.x + threadIdx.x),
                       (int)(blockIdx.y * blockDim.y + threadIdx.y),
                       (int)(blockIdx.z * blockDim.z + threadIdx.z)};
    const int nn[3] = {g.nx + 1, g.ny + 1, DIM == 3 ? g.nz + 1 : 1};
    if (id[0] >= nn[0] || id[1] >= nn[1] || id[2] >= nn[2]) return;
    const long long st[3] = {1, nn[0], (long long)nn[0] * nn[1]};
    const double sc = dt / g.h;
    double P[DIM], D[DIM];
    int n[DIM], s[DIM];
    long long step[DIM];
#pragma unroll
    for (int b = 0; b < DIM; ++b) {
        P[b] = (double)id[b];
        n[b] = nn[b];
        s[b] = 0;
        step[b] = st[b];
    }
#pragma unroll
    for (int b = 0; b < DIM; ++b) D[b] = __builtin_fma(-sc, interp_face<DIM>(g, uext, b, P), P[b]);
    out[id[0] + st[1] * id[1] + st[2] * id[2]] = interp<DIM>(phi, n, s, step, D);
}

dim3 grid_of(const Geo& g, dim3 bs, int extra) {
    return dim3((g.nx + extra + bs.x - 1) / bs.x, (g.ny + extra + bs.y - 1) / bs.y,
                g.dim == 3 ? (g.nz + extra + bs.z - 1) / bs.z : 1);
}

dim3 block_of(const Geo& g) { return g.dim == 2 ? dim3(64, 4, 1) : dim3(64, 2, 2); }

}  // namespace

void launch_known_faces(const Geo& g, const uint8_t* fflag, const double* WF, uint8_t* known,
                        hipStream_t s) {
    const dim3 bs = block_of(g);
    hipLaunchKernelGGL(k_known_faces, grid_of(g, bs, 1), bs, 0, s, g, fflag, WF, known);
}

void launch_extend(const Geo& g, const double* vin, const uint8_t* kin, double* vout,
                   uint8_t* kout, hipStream_t s) {
    const dim3 bs = block_of(g);
    hipLaunchKernelGGL(k_extend, grid_of(g, bs, 1), bs, 0, s, g, vin, kin, vout, kout);
}

void launch_advect_u(const Geo& g, double dt, const double* uext, double* uout, hipStream_t s) {
    const dim3 bs = block_of(g);
    if (g.dim == 2)
        hipLaunchKernelGGL(k_advect_u<2>, grid_of(g, bs, 1), bs, 0, s, g, dt, uext, uout);
    else
        hipLaunchKernelGGL(k_advect_u<3>, grid_of(g, bs, 1), bs, 0, s, g, dt, uext, uout);
}

void launch_advect_phi(const Geo& g, double dt, const double* uext, const double* phi, double* out,
                       hipStream_t s) {
    const dim3 bs = block_of(g);
    if (g.dim == 2)
        hipLaunchKernelGGL(k_advect_phi<2>, grid_of(g, bs, 1), bs, 0, s, g, dt, uext, phi, out);
    else
        hipLaunchKernelGGL(k_advect_phi<3>, grid_of(g, bs, 1), bs, 0, s, g, dt, uext, phi, out);
}

}  // namespace vfs

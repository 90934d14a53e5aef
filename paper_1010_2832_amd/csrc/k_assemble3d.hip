// 3D assembly of the SPD stress/pressure system (paper eq.
// stokesmixedsystemspd, factored form of Section 7), null-space elimination
// (Section 8), moving-solid right-hand side (Section 6.2) and velocity
// recovery from the velocity row of eq. stokesmixedsystem.
//
// Samples (Section 5, Fig. 2): p, tau_xx, tau_yy at cells (tau_zz =
// -tau_xx - tau_yy); tau_xy on z-edges, tau_xz on y-edges, tau_yz on
// x-edges; u, v, w on faces.  Reduced deformation rows:
//   D_xx = u_x - w_z, D_yy = v_y - w_z, D_xy = u_y + v_x, D_xz = u_z + w_x,
//   D_yz = v_z + w_y.
// Compliance: (1/mu)[[1, 1/2], [1/2, 1]] on each cell's (tau_xx, tau_yy) and
// 1/mu on the edges, times W_F W_L of the sample.
//
// Slices: samples 0 p, 1 txx, 2 tyy, 3 txy (z-edge), 4 txz (y-edge),
// 5 tyz (x-edge); faces 0 u, 1 v, 2 w; weight sets 0 cell, 1 u, 2 v, 3 w,
// 4 z-edge, 5 y-edge, 6 x-edge.
#include "vfs_internal.h"

namespace vfs {
namespace {

enum : uint8_t { FK = 1, FBAD = 2, FINV = 4 };

struct FaceIn {
    const double* WL;
    double* WF;
    const double* rho;
    const double* u;
    double* ustar;
    double* rhof;
    double* K;
    uint8_t* fflag;
};

// Classification and coefficients of face slice `a` at anchor o.
// s0, s1: the two cells sharing the face (in-box flags lo_in / hi_in),
// e0..e3: edge samples whose stencil holds the face (set index + offsets).
__device__ __forceinline__ void face_one(const Geo& g, const FaceIn& f, int a, long long o,
                                         long long oc_lo, bool lo_in, bool hi_in,
                                         int set_e0, long long oe0, long long oe1, int set_e1,
                                         long long oe2, long long oe3, double sK, double dt,
                                         double ga) {
    const long long NP = g.NP;
    const double wl = f.WL[(1 + a) * NP + o];
    const double wf = f.WF[(1 + a) * NP + o];
    bool inval = false;
    if (wf > 0.0) {
        const double* WFc = f.WF;
        inval = WFc[oc_lo] == 0.0 || WFc[o] == 0.0 || f.WF[set_e0 * NP + oe0] == 0.0 ||
                f.WF[set_e0 * NP + oe1] == 0.0 || f.WF[set_e1 * NP + oe2] == 0.0 ||
                f.WF[set_e1 * NP + oe3] == 0.0;
    }
    const double wfe = inval ? 0.0 : wf;
    const bool kp = wfe > 0.0 && wl > 0.0;
    const bool bad = wfe > 0.0 && wl == 0.0;
    double r;
    if (lo_in && hi_in)
        r = (f.rho[oc_lo] + f.rho[o]) * 0.5;
    else
        r = lo_in ? f.rho[oc_lo] : f.rho[o];
    f.WF[(1 + a) * NP + o] = wfe;
    f.rhof[a * NP + o] = r;
    f.K[a * NP + o] = kp ? sK * (wfe / (r * wl)) : 0.0;
    f.fflag[a * NP + o] = (uint8_t)((kp ? FK : 0) | (bad ? FBAD : 0) | (inval ? FINV : 0));
    f.ustar[a * NP + o] = f.u[a * NP + o] + dt * ga;
}

__global__ void k_face3d(Geo g, double dt, double g0, double g1, double g2, FaceIn f) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    const int j = blockIdx.y * blockDim.y + threadIdx.y;
    const int k = blockIdx.z * blockDim.z + threadIdx.z;
    if (i > g.nx || j > g.ny || k > g.nz) return;
    const long long o = g.idx(i, j, k);
    const double sK = dt / (g.h * g.h);
    // u face (i,j,k): i <= nx, j < ny, k < nz. cells (i-1,j,k),(i,j,k);
    // z-edges (i,j,k),(i,j+1,k) [set 4]; y-edges (i,j,k),(i,j,k+1) [set 5]
    if (j < g.ny && k < g.nz)
        face_one(g, f, 0, o, g.idx(i - 1, j, k), i > 0, i < g.nx, 4, o, g.idx(i, j + 1, k), 5, o,
                 g.idx(i, j, k + 1), sK, dt, g0);
    // v face: i < nx, j <= ny, k < nz. cells (i,j-1,k),(i,j,k);
    // z-edges (i,j,k),(i+1,j,k) [4]; x-edges (i,j,k),(i,j,k+1) [6]
    if (i < g.nx && k < g.nz)
        face_one(g, f, 1, o, g.idx(i, j - 1, k), j > 0, j < g.ny, 4, o, g.idx(i + 1, j, k), 6, o,
                 g.idx(i, j, k + 1), sK, dt, g1);
    // w face: i < nx, j < ny, k <= nz. cells (i,j,k-1),(i,j,k);
    // y-edges (i,j,k),(i+1,j,k) [5]; x-edges (i,j,k),(i,j+1,k) [6]
    if (i < g.nx && j < g.ny)
        face_one(g, f, 2, o, g.idx(i, j, k - 1), k > 0, k < g.nz, 5, o, g.idx(i + 1, j, k), 6, o,
                 g.idx(i, j + 1, k), sK, dt, g2);
}

struct SampleIn {
    const double* WL;
    const double* WF;
    const double* mu;
    const double* K;
    const uint8_t* fflag;
    const double* ustar;
    const double* ubc;
    double* a;
    double* c;
    double* dinv;
    double* b;
};

// The twelve faces that the samples of an anchor meet.
enum Face3 { U0, UX, UY, UZ, V0, VY, VX, VZ, W0, WZ, WX, WY };   // at the anchor; one step along an axis
struct Faces3 {
    double K[12], y[12], ubc[12];   // y = W_F u* + W_S u_BC
};

// One sample with stencil faces f of signs sg (the reduced-D row, or -div for
// pressure), its weights given.
template <int NF>
__device__ __forceinline__ void sample_one(const Faces3& F, const int (&f)[NF], const int (&sg)[NF],
                                           bool pressure, double wl, double wf, double mu_s, double ih,
                                           double& a_out, double& c_out, double& d_out, double& b_out) {
#pragma clang fp contract(off)
    double sumK = F.K[f[0]], ty = 0.0, tb = 0.0;
#pragma unroll
    for (int q = 1; q < NF; ++q) sumK += F.K[f[q]];
#pragma unroll
    for (int q = 0; q < NF; ++q) {
        ty = sg[q] > 0 ? ty + F.y[f[q]] : ty - F.y[f[q]];
        tb = sg[q] > 0 ? tb + F.ubc[f[q]] : tb - F.ubc[f[q]];
    }
    a_out = wl;
    c_out = pressure ? 0.0 : wf * wl / mu_s;
    d_out = 1.0 / __builtin_fma(wl * wl, sumK, c_out);
    b_out = wl * __builtin_fma(ih, ty, -((1.0 - wf) * (tb * ih)));
}

__device__ __forceinline__ double mu_mean(const Geo& g, const double* mu, int i, int j, int k,
                                          int sx, int sy, int sz) {
    // mean of the in-box cells adjacent to a sample of stagger (sx,sy,sz)
    double s = 0.0;
    int n = 0;
    for (int di = (sx ? 0 : -1); di <= 0; ++di)
        for (int dj = (sy ? 0 : -1); dj <= 0; ++dj)
            for (int dk = (sz ? 0 : -1); dk <= 0; ++dk) {
                const int ci = i + di, cj = j + dj, ck = k + dk;
                if (ci < 0 || ci >= g.nx || cj < 0 || cj >= g.ny || ck < 0 || ck >= g.nz) continue;
                s += mu[g.idx(ci, cj, ck)];
                ++n;
            }
    return n ? s / (double)n : 1.0;
}

// An anchor's faces are read once for all its samples: read by each, under its own
// test, they took 130 loads of a thread, 2.05 ms at 256^3 (now 1.70; 5 GB, 1.1 ms).
// 128 registers, 14 spilled: with 196 and half the waves 1.90 ms, with 102 2.35.
__global__ __launch_bounds__(256, 4) void k_sample3d(Geo g, SampleIn s, Scalars* sc) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    const int j = blockIdx.y * blockDim.y + threadIdx.y;
    const int k = blockIdx.z * blockDim.z + threadIdx.z;
    int nact = 0;
    if (i <= g.nx && j <= g.ny && k <= g.nz) {
        const long long NP = g.NP;
        const long long o = g.idx(i, j, k);
        const double ih = 1.0 / g.h;
        double av[6], cv[6], dv[6], bv[6];
        for (int q = 0; q < 6; ++q) av[q] = cv[q] = dv[q] = bv[q] = 0.0;
        const long long sx = 1, sy = g.PX, sz = (long long)g.PX * g.PY;
        const long long at[12] = {o,      o + sx, o - sy, o - sz, NP + o,     NP + o + sy,
                                  NP + o - sx, NP + o - sz, 2 * NP + o, 2 * NP + o + sz, 2 * NP + o - sx,
                                  2 * NP + o - sy};
        // stencils: p -div; txx u_x - w_z; tyy v_y - w_z; txy u_y + v_x (z-edge);
        // txz u_z + w_x (y-edge); tyz v_z + w_y (x-edge)
        uint8_t fl[12];
#pragma unroll
        for (int q = 0; q < 12; ++q) fl[q] = s.fflag[at[q]];
        const bool cell = i < g.nx && j < g.ny && k < g.nz;
        const bool valid[6] = {cell, cell, cell, k < g.nz, j < g.ny, i < g.nx};
        const uint8_t met[6] = {(uint8_t)(fl[U0] | fl[UX] | fl[V0] | fl[VY] | fl[W0] | fl[WZ]),
                                (uint8_t)(fl[UX] | fl[U0] | fl[WZ] | fl[W0]),
                                (uint8_t)(fl[VY] | fl[V0] | fl[WZ] | fl[W0]),
                                (uint8_t)(fl[U0] | fl[UY] | fl[V0] | fl[VX]),
                                (uint8_t)(fl[U0] | fl[UZ] | fl[W0] | fl[WX]),
                                (uint8_t)(fl[V0] | fl[VZ] | fl[W0] | fl[WY])};
        constexpr int set[6] = {0, 0, 0, 4, 5, 6};
        double wl[6];
        bool act[6];
        // the (txx, tyy) compliance coupling: the diagonal of the 2x2 block is c;
        // Jacobi uses the diagonal entries only
#pragma unroll
        for (int q = 0; q < 6; ++q) {
            wl[q] = (q == 1 || q == 2) ? wl[0] : s.WL[set[q] * NP + o];
            act[q] = valid[q] && wl[q] > 0.0 && !(met[q] & FBAD) && (met[q] & FK);
            nact += act[q] ? 1 : 0;
        }
        if (nact) {
            Faces3 F;
#pragma unroll
            for (int q = 0; q < 12; ++q) {
#pragma clang fp contract(off)
                const double wf = s.WF[NP + at[q]], ubc = s.ubc[at[q]];
                F.K[q] = s.K[at[q]];
                F.ubc[q] = ubc;
                F.y[q] = __builtin_fma(wf, s.ustar[at[q]], (1.0 - wf) * ubc);
            }
            double wf[6];
#pragma unroll
            for (int q = 0; q < 6; ++q) wf[q] = (q == 1 || q == 2) ? wf[0] : s.WF[set[q] * NP + o];
            const double muc = cell ? s.mu[o] : 1.0;
            if (act[0])
                sample_one<6>(F, {U0, UX, V0, VY, W0, WZ}, {1, -1, 1, -1, 1, -1}, true, wl[0], wf[0], muc, ih,
                              av[0], cv[0], dv[0], bv[0]);
            if (act[1])
                sample_one<4>(F, {UX, U0, WZ, W0}, {1, -1, -1, 1}, false, wl[1], wf[1], muc, ih, av[1], cv[1],
                              dv[1], bv[1]);
            if (act[2])
                sample_one<4>(F, {VY, V0, WZ, W0}, {1, -1, -1, 1}, false, wl[2], wf[2], muc, ih, av[2], cv[2],
                              dv[2], bv[2]);
            if (act[3])
                sample_one<4>(F, {U0, UY, V0, VX}, {1, -1, 1, -1}, false, wl[3], wf[3],
                              mu_mean(g, s.mu, i, j, k, 0, 0, 1), ih, av[3], cv[3], dv[3], bv[3]);
            if (act[4])
                sample_one<4>(F, {U0, UZ, W0, WX}, {1, -1, 1, -1}, false, wl[4], wf[4],
                              mu_mean(g, s.mu, i, j, k, 0, 1, 0), ih, av[4], cv[4], dv[4], bv[4]);
            if (act[5])
                sample_one<4>(F, {V0, VZ, W0, WY}, {1, -1, 1, -1}, false, wl[5], wf[5],
                              mu_mean(g, s.mu, i, j, k, 1, 0, 0), ih, av[5], cv[5], dv[5], bv[5]);
        }
#pragma unroll
        for (int q = 0; q < 6; ++q) {
            s.a[q * NP + o] = av[q];
            s.c[q * NP + o] = cv[q];
            s.dinv[q * NP + o] = dv[q];
            s.b[q * NP + o] = bv[q];
        }
    }
    __shared__ int s_cnt;
    const int tid = threadIdx.x + blockDim.x * (threadIdx.y + blockDim.y * threadIdx.z);
    if (tid == 0) s_cnt = 0;
    __syncthreads();
    if (nact) atomicAdd(&s_cnt, nact);
    __syncthreads();
    if (tid == 0 && s_cnt) atomicAdd((unsigned long long*)&sc->n_active, (unsigned long long)s_cnt);
}

// Velocity recovery (3D): u = u* - dt (B x) / (rho W_L) where K > 0; u_BC
// where W_F = 0; 0 elsewhere.
__global__ void k_velocity3d(Geo g, double dt, const double* __restrict__ x,
                             const double* __restrict__ a, const double* __restrict__ ustar,
                             const double* __restrict__ ubc, const double* __restrict__ rhof,
                             const double* __restrict__ WL, const double* __restrict__ WF,
                             const uint8_t* __restrict__ fflag, double* __restrict__ u) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    const int j = blockIdx.y * blockDim.y + threadIdx.y;
    const int k = blockIdx.z * blockDim.z + threadIdx.z;
    if (i > g.nx || j > g.ny || k > g.nz) return;
    const long long NP = g.NP;
    const long long o = g.idx(i, j, k);
    auto W = [&](int s, long long off) { return a[s * NP + off] * x[s * NP + off]; };
    const double sc = dt / g.h;
    if (j < g.ny && k < g.nz) {
        double val;
        if (fflag[o] & FK) {
            const long long om = g.idx(i - 1, j, k);
            const double d = (W(0, o) - W(0, om)) + (W(1, om) - W(1, o)) +
                             (W(3, o) - W(3, g.idx(i, j + 1, k))) +
                             (W(4, o) - W(4, g.idx(i, j, k + 1)));
            val = ustar[o] - sc * d / (rhof[o] * WL[NP + o]);
        } else {
            val = WF[NP + o] == 0.0 ? ubc[o] : 0.0;
        }
        u[o] = val;
    }
    if (i < g.nx && k < g.nz) {
        double val;
        if (fflag[NP + o] & FK) {
            const long long om = g.idx(i, j - 1, k);
            const double d = (W(0, o) - W(0, om)) + (W(2, om) - W(2, o)) +
                             (W(3, o) - W(3, g.idx(i + 1, j, k))) +
                             (W(5, o) - W(5, g.idx(i, j, k + 1)));
            val = ustar[NP + o] - sc * d / (rhof[NP + o] * WL[2 * NP + o]);
        } else {
            val = WF[2 * NP + o] == 0.0 ? ubc[NP + o] : 0.0;
        }
        u[NP + o] = val;
    }
    if (i < g.nx && j < g.ny) {
        double val;
        if (fflag[2 * NP + o] & FK) {
            const long long om = g.idx(i, j, k - 1);
            const double d = (W(0, o) - W(0, om)) + (W(1, o) - W(1, om)) + (W(2, o) - W(2, om)) +
                             (W(4, o) - W(4, g.idx(i + 1, j, k))) +
                             (W(5, o) - W(5, g.idx(i, j + 1, k)));
            val = ustar[2 * NP + o] - sc * d / (rhof[2 * NP + o] * WL[3 * NP + o]);
        } else {
            val = WF[3 * NP + o] == 0.0 ? ubc[2 * NP + o] : 0.0;
        }
        u[2 * NP + o] = val;
    }
}

// Prescribed traction (Section 6.1), 3D counterpart of k_traction2d: on
// faces with K > 0, u* += dt f / (rho W_L), f = B0 (a y) - W_L (B0 y), with
// B0's stencils of k_velocity3d.
__global__ void k_traction3d(Geo g, double dt, const double* __restrict__ y,
                             const double* __restrict__ a, const double* __restrict__ rhof,
                             const double* __restrict__ WL, const uint8_t* __restrict__ fflag,
                             double* __restrict__ ustar) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    const int j = blockIdx.y * blockDim.y + threadIdx.y;
    const int k = blockIdx.z * blockDim.z + threadIdx.z;
    if (i > g.nx || j > g.ny || k > g.nz) return;
    const long long NP = g.NP;
    const long long o = g.idx(i, j, k);
    auto AY = [&](int s, long long off) { return a[s * NP + off] * y[s * NP + off]; };
    auto Y = [&](int s, long long off) { return y[s * NP + off]; };
    const double sc = dt / g.h;
    if (j < g.ny && k < g.nz && (fflag[o] & FK)) {
        const long long om = g.idx(i - 1, j, k), oy = g.idx(i, j + 1, k), oz = g.idx(i, j, k + 1);
        const double day = (AY(0, o) - AY(0, om)) + (AY(1, om) - AY(1, o)) + (AY(3, o) - AY(3, oy)) +
                           (AY(4, o) - AY(4, oz));
        const double dy = (Y(0, o) - Y(0, om)) + (Y(1, om) - Y(1, o)) + (Y(3, o) - Y(3, oy)) +
                          (Y(4, o) - Y(4, oz));
        const double wl = WL[NP + o];
        ustar[o] += sc * (day - wl * dy) / (rhof[o] * wl);
    }
    if (i < g.nx && k < g.nz && (fflag[NP + o] & FK)) {
        const long long om = g.idx(i, j - 1, k), ox = g.idx(i + 1, j, k), oz = g.idx(i, j, k + 1);
        const double day = (AY(0, o) - AY(0, om)) + (AY(2, om) - AY(2, o)) + (AY(3, o) - AY(3, ox)) +
                           (AY(5, o) - AY(5, oz));
        const double dy = (Y(0, o) - Y(0, om)) + (Y(2, om) - Y(2, o)) + (Y(3, o) - Y(3, ox)) +
                          (Y(5, o) - Y(5, oz));
        const double wl = WL[2 * NP + o];
        ustar[NP + o] += sc * (day - wl * dy) / (rhof[NP + o] * wl);
    }
    if (i < g.nx && j < g.ny && (fflag[2 * NP + o] & FK)) {
        const long long om = g.idx(i, j, k - 1), ox = g.idx(i + 1, j, k), oy = g.idx(i, j + 1, k);
        const double day = (AY(0, o) - AY(0, om)) + (AY(1, o) - AY(1, om)) + (AY(2, o) - AY(2, om)) +
                           (AY(4, o) - AY(4, ox)) + (AY(5, o) - AY(5, oy));
        const double dy = (Y(0, o) - Y(0, om)) + (Y(1, o) - Y(1, om)) + (Y(2, o) - Y(2, om)) +
                          (Y(4, o) - Y(4, ox)) + (Y(5, o) - Y(5, oy));
        const double wl = WL[3 * NP + o];
        ustar[2 * NP + o] += sc * (day - wl * dy) / (rhof[2 * NP + o] * wl);
    }
}

// A cell whose tau_xx is active and tau_yy eliminated (or the reverse): the
// eliminated stress holds its boundary value, and the compliance coupling
// (1/2) W_F W_L / mu of the pair moves that value times the coupling to the
// right-hand side of the active one.  c holds W_F W_L / mu on active stresses.
__global__ void k_traction_pair3d(Geo g, const double* __restrict__ y,
                                  const double* __restrict__ a, const double* __restrict__ c,
                                  double* __restrict__ b) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    const int j = blockIdx.y * blockDim.y + threadIdx.y;
    const int k = blockIdx.z * blockDim.z + threadIdx.z;
    if (i >= g.nx || j >= g.ny || k >= g.nz) return;
    const long long NP = g.NP;
    const long long o = g.idx(i, j, k);
    const bool ax = a[NP + o] != 0.0, ay = a[2 * NP + o] != 0.0;
    if (ax && !ay) b[NP + o] -= 0.5 * c[NP + o] * y[2 * NP + o];
    if (ay && !ax) b[2 * NP + o] -= 0.5 * c[2 * NP + o] * y[NP + o];
}

dim3 grid3(const Geo& g, dim3 bs) {
    return dim3((g.nx + 1 + bs.x - 1) / bs.x, (g.ny + 1 + bs.y - 1) / bs.y,
                (g.nz + 1 + bs.z - 1) / bs.z);
}

}  // namespace

void launch_face_coef3d(const Geo& g, double dt, const double* g3, const double* WL, double* WF,
                        const double* rho, const double* u, double* ustar, double* rhof,
                        double* K, uint8_t* fflag, hipStream_t s) {
    FaceIn f{WL, WF, rho, u, ustar, rhof, K, fflag};
    dim3 bs(64, 2, 2);
    hipLaunchKernelGGL(k_face3d, grid3(g, bs), bs, 0, s, g, dt, g3[0], g3[1], g3[2], f);
}

void launch_traction3d(const Geo& g, double dt, const double* y, const double* a,
                       const double* rhof, const double* WL, const uint8_t* fflag, double* ustar,
                       hipStream_t s) {
    dim3 bs(64, 2, 2);
    hipLaunchKernelGGL(k_traction3d, grid3(g, bs), bs, 0, s, g, dt, y, a, rhof, WL, fflag, ustar);
}

void launch_traction_pair3d(const Geo& g, const double* y, const double* a, const double* c,
                            double* b, hipStream_t s) {
    dim3 bs(64, 2, 2);
    hipLaunchKernelGGL(k_traction_pair3d, grid3(g, bs), bs, 0, s, g, y, a, c, b);
}

void launch_sample_coef3d(const Geo& g, const double* WL, const double* WF, const double* mu,
                          const double* K, const uint8_t* fflag, const double* ustar,
                          const double* ubc, double* a, double* c, double* dinv, double* b,
                          Scalars* sc, hipStream_t s) {
    SampleIn si{WL, WF, mu, K, fflag, ustar, ubc, a, c, dinv, b};
    dim3 bs(64, 2, 2);
    hipLaunchKernelGGL(k_sample3d, grid3(g, bs), bs, 0, s, g, si, sc);
}

void launch_velocity3d(const Geo& g, double dt, const double* x, const double* a,
                       const double* ustar, const double* ubc, const double* rhof,
                       const double* WL, const double* WF, const uint8_t* fflag, double* u,
                       hipStream_t s) {
    dim3 bs(64, 2, 2);
    hipLaunchKernelGGL(k_velocity3d, grid3(g, bs), bs, 0, s, g, dt, x, a, ustar, ubc, rhof, WL, WF,
                       fflag, u);
}

}  // namespace vfs

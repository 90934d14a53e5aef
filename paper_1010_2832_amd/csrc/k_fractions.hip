// Volume fractions of the sample control volumes (paper Section 5,
// Figs. 3-4: every term of the discrete functional is weighted by the
// fraction of material in an h-sized control volume around its sample).
//
// Estimator: nodal level set -> h/2 lattice by multilinear interpolation
// (midpoints averaged along x, then y, then z); each h/2 sub-cell split into
// Kuhn simplices sharing its min->max diagonal (2 triangles / 6 tetrahedra
// in axis-permutation order xyz, xzy, yxz, yzx, zxy, zyx); exact measure of
// {phi < 0} of each simplex under linear interpolation; control-volume
// weight = mean of its 2^d sub-cells, summed pairwise along x, then y, then
// z.  The operation order is part of the definition: together with
// -ffp-contract=off (set for this file by the build) it makes the weights,
// and therefore every classification decision taken on them, reproducible
// to the last bit.
//
// Box walls: sub-cells outside the box are solid (fluid fraction 0) and
// take the liquid fraction of the adjacent in-box sub-cell; faces on the
// box boundary have W_F = 0.  Weights below w_min are snapped to 0.
#include "vfs_internal.h"

namespace vfs {
namespace {

// Puts the negative values first, each kind in its order, and counts them:
// exchanges of neighbours, so that the values stay in registers.
template <int N>
__device__ __forceinline__ int negatives_first(double (&w)[N]) {
    int k = 0;
#pragma unroll
    for (int q = 0; q < N; ++q) k += w[q] < 0.0 ? 1 : 0;
#pragma unroll
    for (int r = N - 1; r > 0; --r)
#pragma unroll
        for (int q = 0; q < r; ++q) {
            const double u = w[q], v = w[q + 1];
            const bool swap = !(u < 0.0) && v < 0.0;
            w[q] = swap ? v : u;
            w[q + 1] = swap ? u : v;
        }
    return k;
}

// Fraction of a triangle with phi < 0 for vertex values v0, v1, v2.
// Negative values are taken first in vertex order, then the others.
__device__ __forceinline__ double tri_frac(double v0, double v1, double v2) {
    double w[3] = {v0, v1, v2};
    const int k = negatives_first(w);
    const double a = w[0], b = w[1], c = w[2];
    double f;
    if (k == 0) {
        f = 0.0;
    } else if (k == 3) {
        f = 1.0;
    } else if (k == 1) {
        f = (a * a) / ((a - b) * (a - c));
    } else {
        f = 1.0 - (c * c) / ((c - a) * (c - b));
    }
    return fmin(fmax(f, 0.0), 1.0);
}

// Fraction of a tetrahedron with phi < 0.
__device__ __forceinline__ double tet_frac(double v0, double v1, double v2, double v3) {
    double w[4] = {v0, v1, v2, v3};
    const int k = negatives_first(w);
    const double a = w[0], b = w[1], c = w[2], d = w[3];
    double num, den;
    if (k == 0) return 0.0;
    if (k == 4) return 1.0;
    // one division for the three cases
    if (k == 1) {
        num = (a * a) * a;
        den = ((a - b) * (a - c)) * (a - d);
    } else if (k == 2) {
        num = ((a * a) * (b * b) - ((a * b) * (a + b)) * (c + d)) +
              (c * d) * (((a * a) + (a * b)) + (b * b));
        den = ((a - c) * (a - d)) * ((b - c) * (b - d));
    } else {
        num = (d * d) * d;
        den = ((d - a) * (d - b)) * (d - c);
    }
    const double q = num / den, f = k == 3 ? 1.0 - q : q;
    return fmin(fmax(f, 0.0), 1.0);
}

// Value along an axis of the h/2 lattice inside a cell: its near node (0), the
// midpoint (1) or its far node (2).
__device__ __forceinline__ double half(double p, double q, int at) {
    return at == 0 ? p : (at == 1 ? (p + q) * 0.5 : q);
}

// Liquid fraction of sub-cell (ox, oy) of a cell with nodal values p[y][x].
// The value's sign is that of the nodes where these agree (a mean keeps it), and
// a sub-cell of one sign is 0 or 1 without a look at its triangles.
__device__ __forceinline__ double sub_frac(const double (&p)[2][2], int ox, int oy) {
    double c[2][2];
#pragma unroll
    for (int dy = 0; dy < 2; ++dy)
#pragma unroll
        for (int dx = 0; dx < 2; ++dx)
            c[dy][dx] = half(half(p[0][0], p[0][1], ox + dx), half(p[1][0], p[1][1], ox + dx), oy + dy);
    const double t1 = tri_frac(c[0][0], c[0][1], c[1][1]);
    const double t2 = tri_frac(c[0][0], c[1][0], c[1][1]);
    return (t1 + t2) * 0.5;
}

// The same in 3D, p[z][y][x].
__device__ __forceinline__ double sub_frac(const double (&p)[2][2][2], int ox, int oy, int oz) {
    double c[2][2][2];   // [x][y][z]
#pragma unroll
    for (int dz = 0; dz < 2; ++dz)
#pragma unroll
        for (int dy = 0; dy < 2; ++dy)
#pragma unroll
            for (int dx = 0; dx < 2; ++dx) {
                double z[2];
#pragma unroll
                for (int k = 0; k < 2; ++k)
                    z[k] = half(half(p[k][0][0], p[k][0][1], ox + dx), half(p[k][1][0], p[k][1][1], ox + dx),
                                oy + dy);
                c[dx][dy][dz] = half(z[0], z[1], oz + dz);
            }
    // permutations xyz, xzy, yxz, yzx, zxy, zyx: v1 = +e_p0, v2 = v1 + e_p1
    double acc;
    acc = tet_frac(c[0][0][0], c[1][0][0], c[1][1][0], c[1][1][1]);          // xyz
    acc = acc + tet_frac(c[0][0][0], c[1][0][0], c[1][0][1], c[1][1][1]);    // xzy
    acc = acc + tet_frac(c[0][0][0], c[0][1][0], c[1][1][0], c[1][1][1]);    // yxz
    acc = acc + tet_frac(c[0][0][0], c[0][1][0], c[0][1][1], c[1][1][1]);    // yzx
    acc = acc + tet_frac(c[0][0][0], c[0][0][1], c[1][0][1], c[1][1][1]);    // zxy
    acc = acc + tet_frac(c[0][0][0], c[0][0][1], c[0][1][1], c[1][1][1]);    // zyx
    return acc / 6.0;
}

// Nodal values of cell (i, j[, k]), and how many are negative.
__device__ __forceinline__ int cell_nodes(const double* __restrict__ phi, int NX1, int i, int j,
                                          double (&p)[2][2]) {
    const double* q = phi + (long long)j * NX1 + i;
    int neg = 0;
#pragma unroll
    for (int y = 0; y < 2; ++y)
#pragma unroll
        for (int x = 0; x < 2; ++x) {
            p[y][x] = q[y * NX1 + x];
            neg += p[y][x] < 0.0 ? 1 : 0;
        }
    return neg;
}

__device__ __forceinline__ int cell_nodes(const double* __restrict__ phi, int NX1, int NY1, int i, int j,
                                          int k, double (&p)[2][2][2]) {
    const long long plane = (long long)NX1 * NY1;
    const double* q = phi + k * plane + (long long)j * NX1 + i;
    int neg = 0;
#pragma unroll
    for (int z = 0; z < 2; ++z)
#pragma unroll
        for (int y = 0; y < 2; ++y)
#pragma unroll
            for (int x = 0; x < 2; ++x) {
                p[z][y][x] = q[z * plane + y * NX1 + x];
                neg += p[z][y][x] < 0.0 ? 1 : 0;
            }
    return neg;
}

__device__ __forceinline__ int clamp_cell(int A, int S) { return A < 0 ? 0 : (A >= S ? S - 1 : A); }

__device__ __forceinline__ double snap(double w, double w_min) { return w < w_min ? 0.0 : w; }

// Weights of all sample sets of a tile of anchors, both materials, in one pass.
// Writing the sub-cell fractions to memory and averaging them in a second kernel
// took 8.9 ms at 256^3 (a pool with a solid), this one takes 0.91, and the 2.1 GB
// it cannot do without about 0.45: every sub-cell ran its six tetrahedra, and
// 4.3 GB of fractions were written and read again.
// Here a tile's sub-cells live in LDS.  Anchor i averages sub-cells 2i - 1 to
// 2i + 1 of each axis, so TX anchors need 2 TX + 1 of them.  Cells whose nodes
// have one sign are filled in; the sub-cells of the others, few and unevenly
// spread, are listed and shared out over the whole workgroup.  x positions are
// split by parity, so that lanes read neighbouring words.
template <int DIM>
struct FTile {
    static constexpr int TX = 32, TY = DIM == 2 ? 8 : 4, TZ = DIM == 2 ? 1 : 4, NT = 256;
    static constexpr int CX = TX + 1, CY = TY + 1, CZ = DIM == 2 ? 1 : TZ + 1;   // cells
    static constexpr int SX = 2 * TX + 2, SY = 2 * TY + 1, SZ = DIM == 2 ? 1 : 2 * TZ + 1;
    static constexpr int cells = CX * CY * CZ, subs = 1 << DIM;
    static constexpr int per = TX * TY * TZ / NT;   // anchors per thread
};

template <int DIM>
struct FLds {
    double th[FTile<DIM>::SZ][FTile<DIM>::SY][FTile<DIM>::SX];
    short mixed[FTile<DIM>::cells];
    int n;
};

// Sub-cell fractions of the tile at (i0, j0, k0) into LDS.  Returns 0 or 1 when
// every sub-cell of the tile has that value (LDS is then not written), else -1.
template <int DIM>
__device__ __forceinline__ int tile_fractions(const Geo& g, int i0, int j0, int k0,
                                              const double* __restrict__ phi, bool complement,
                                              FLds<DIM>& sh) {
    using F = FTile<DIM>;
    const int tid = threadIdx.x, NX1 = g.nx + 1, NY1 = g.ny + 1;
    if (tid == 0) sh.n = 0;
    __syncthreads();
    constexpr int rounds = (F::cells + F::NT - 1) / F::NT;
    int kind[rounds];   // 1: fraction 0, 2: fraction 1, 4: both signs, 0: outside
    int any = 0;
    double p3[2][2][2], p2[2][2];
    auto cell = [&](int e, int& i, int& j, int& k) {
        i = i0 - 1 + e % F::CX;
        j = j0 - 1 + (e / F::CX) % F::CY;
        k = DIM == 2 ? 0 : k0 - 1 + e / (F::CX * F::CY);
        return i >= 0 && i < g.nx && j >= 0 && j < g.ny && (DIM == 2 || (k >= 0 && k < g.nz));
    };
#pragma unroll
    for (int r = 0; r < rounds; ++r) {
        const int e = tid + F::NT * r;
        int i, j, k;
        kind[r] = 0;
        if (e < F::cells && cell(e, i, j, k)) {
            const int neg = DIM == 2 ? cell_nodes(phi, NX1, i, j, p2) : cell_nodes(phi, NX1, NY1, i, j, k, p3);
            kind[r] = neg == 0 ? (complement ? 2 : 1) : (neg == F::subs ? (complement ? 1 : 2) : 4);
            if (kind[r] == 4) sh.mixed[atomicAdd(&sh.n, 1)] = (short)e;
        }
        any |= kind[r];
    }
    any = (__syncthreads_or(any & 1) ? 1 : 0) | (__syncthreads_or(any & 2) ? 2 : 0) |
          (sh.n ? 4 : 0);
    if (any == 1 || any == 2) return any - 1;
    auto at = [&](int e, int q) -> double* {
        // sub-cell q of cell e; the tile starts at the upper half of its first cell
        const int a = 2 * (e % F::CX) - 1 + (q & 1), b = 2 * ((e / F::CX) % F::CY) - 1 + ((q >> 1) & 1),
                  c = DIM == 2 ? 0 : 2 * (e / (F::CX * F::CY)) - 1 + (q >> 2);
        if (a < 0 || b < 0 || c < 0) return nullptr;
        return &sh.th[c][b][(a & 1) * (F::SX / 2) + (a >> 1)];
    };
#pragma unroll
    for (int r = 0; r < rounds; ++r)
        if (kind[r] == 1 || kind[r] == 2) {
            const double v = kind[r] == 2 ? 1.0 : 0.0;
#pragma unroll
            for (int q = 0; q < F::subs; ++q)
                if (double* d = at(tid + F::NT * r, q)) *d = v;
        }
    const int items = sh.n * F::subs;
    for (int t = tid; t < items; t += F::NT) {
        const int e = sh.mixed[t / F::subs], q = t % F::subs;
        double* d = at(e, q);
        if (!d) continue;
        int i, j, k;
        cell(e, i, j, k);
        double f;
        if constexpr (DIM == 2) {
            cell_nodes(phi, NX1, i, j, p2);
            f = sub_frac(p2, q & 1, q >> 1);
        } else {
            cell_nodes(phi, NX1, NY1, i, j, k, p3);
            f = sub_frac(p3, q & 1, (q >> 1) & 1, q >> 2);
        }
        *d = complement ? 1.0 - f : f;
    }
    __syncthreads();
    return -1;
}

// The sub-cells 2i - 1 to 2i + 1 of each axis around an anchor.  Box rule: liquid
// mirrors (clamps) into the box, fluid is 0 outside.
template <int DIM>
__device__ __forceinline__ void sub_cells(const Geo& g, const FLds<DIM>& sh, int uniform, bool liquid, int i0,
                                          int j0, int k0, int i, int j, int k,
                                          double (&t)[DIM == 2 ? 1 : 3][3][3]) {
    constexpr int NZ = DIM == 2 ? 1 : 3;
    int x[3], y[3], z[3];
    bool ox[3], oy[3], oz[3];
#pragma unroll
    for (int q = 0; q < 3; ++q) {
        const int A = 2 * i - 1 + q, B = 2 * j - 1 + q, C = 2 * k - 1 + q;
        const int a = clamp_cell(A, 2 * g.nx) - (2 * i0 - 1);
        x[q] = (a & 1) * (FTile<DIM>::SX / 2) + (a >> 1);
        y[q] = clamp_cell(B, 2 * g.ny) - (2 * j0 - 1);
        z[q] = DIM == 2 ? 0 : clamp_cell(C, 2 * g.nz) - (2 * k0 - 1);
        ox[q] = !liquid && (A < 0 || A >= 2 * g.nx);
        oy[q] = !liquid && (B < 0 || B >= 2 * g.ny);
        oz[q] = DIM == 3 && !liquid && (C < 0 || C >= 2 * g.nz);
    }
#pragma unroll
    for (int c = 0; c < NZ; ++c)
#pragma unroll
        for (int b = 0; b < 3; ++b)
#pragma unroll
            for (int a = 0; a < 3; ++a) {
                t[c][b][a] = uniform >= 0 ? (double)uniform : sh.th[z[c]][y[b]][x[a]];
                if (ox[a] || oy[b] || oz[c]) t[c][b][a] = 0.0;
            }
}

// Mean over the control volume of a sample of stagger (sx, sy, sz).
__device__ __forceinline__ double cv_mean(const double (&t)[1][3][3], int sx, int sy, int) {
    return ((t[0][sy][sx] + t[0][sy][sx + 1]) + (t[0][sy + 1][sx] + t[0][sy + 1][sx + 1])) * 0.25;
}
__device__ __forceinline__ double cv_mean(const double (&t)[3][3][3], int sx, int sy, int sz) {
    double z[2];
#pragma unroll
    for (int q = 0; q < 2; ++q)
        z[q] = (t[sz + q][sy][sx] + t[sz + q][sy][sx + 1]) + (t[sz + q][sy + 1][sx] + t[sz + q][sy + 1][sx + 1]);
    return (z[0] + z[1]) * 0.125;
}

// staggers of the sample sets:
// 2D 0 cell (1,1), 1 u (0,1), 2 v (1,0), 3 node (0,0)
// 3D 0 cell (1,1,1), 1 u (0,1,1), 2 v (1,0,1), 3 w (1,1,0),
//    4 z-edge (0,0,1), 5 y-edge (0,1,0), 6 x-edge (1,0,0)
template <int DIM>
__device__ __forceinline__ void stagger_of(int s, int& sx, int& sy, int& sz) {
    constexpr int x[7] = {1, 0, 1, 1, 0, 0, 1}, y[7] = {1, 1, 0, 1, 0, 1, 0}, z[7] = {1, 1, 1, 0, 1, 0, 0};
    sx = DIM == 2 ? (s == 0 || s == 2) : x[s];
    sy = DIM == 2 ? s < 2 : y[s];
    sz = DIM == 2 ? 1 : z[s];
}

template <int DIM>
__global__ __launch_bounds__(256) void k_weights(Geo g, const double* __restrict__ phi_l,
                                                 const double* __restrict__ phi_s, double w_min,
                                                 double* __restrict__ WL, double* __restrict__ WF) {
    using F = FTile<DIM>;
    __shared__ FLds<DIM> sh;
    const int i0 = blockIdx.x * F::TX, j0 = blockIdx.y * F::TY, k0 = blockIdx.z * F::TZ;
    for (int m = 0; m < 2; ++m) {
        const bool liquid = m == 0;
        const double* phi = liquid ? phi_l : phi_s;
        double* __restrict__ W = liquid ? WL : WF;
        const int uniform = phi ? tile_fractions<DIM>(g, i0, j0, k0, phi, !liquid, sh) : 1;
#pragma unroll 1
        for (int n = 0; n < F::per; ++n) {
            const int t = threadIdx.x + F::NT * n;
            const int i = i0 + t % F::TX, j = j0 + (t / F::TX) % F::TY, k = k0 + t / (F::TX * F::TY);
            if (i > g.nx || j > g.ny || (DIM == 3 && k > g.nz)) continue;
            const long long o = DIM == 2 ? g.idx(i, j) : g.idx(i, j, k);
            double th[DIM == 2 ? 1 : 3][3][3];
            sub_cells<DIM>(g, sh, uniform, liquid, i0, j0, k0, i, j, k, th);
#pragma unroll
            for (int s = 0; s < (DIM == 2 ? 4 : 7); ++s) {
                int sx, sy, sz;
                stagger_of<DIM>(s, sx, sy, sz);
                const bool valid = (i < g.nx + (sx ? 0 : 1)) && (j < g.ny + (sy ? 0 : 1)) &&
                                   (DIM == 2 || k < g.nz + (sz ? 0 : 1));
                if (!valid) continue;
                double w = snap(cv_mean(th, sx, sy, sz), w_min);
                if (!liquid && ((s == 1 && (i == 0 || i == g.nx)) || (s == 2 && (j == 0 || j == g.ny)) ||
                                (DIM == 3 && s == 3 && (k == 0 || k == g.nz))))
                    w = 0.0;
                W[s * g.NP + o] = w;
            }
        }
        __syncthreads();   // the next material reuses the LDS
    }
}

// Liquid weights of one sample set, to the caller's compact array.  The control
// volumes of one set share no sub-cell: a lane computes one, and the 2^d lanes of
// a sample add theirs in pairs along x, y and z.  3.4 us at 64^2, where the
// launches of filling, sub-cell, weight and unpack kernels took 18.
//
// KEEP: out may lie over phi, so the weights are kept in an array of the library's
// until all of phi is read (k_kept_out then copies them).
__device__ double kept[kMostSetValues];

template <int DIM, bool KEEP>
__global__ __launch_bounds__(256) void k_weights_set(Geo g, int n0, int n1, int n2, int sx, int sy, int sz,
                                                     const double* __restrict__ phi, double w_min,
                                                     double* __restrict__ out) {
    constexpr int subs = 1 << DIM;
    const long long t = (long long)blockIdx.x * blockDim.x + threadIdx.x, e = t / subs;
    const int q = (int)(t % subs);
    if (e >= (long long)n0 * n1 * n2) return;   // whole groups of lanes
    const int i = (int)(e % n0), j = (int)((e / n0) % n1), k = (int)(e / ((long long)n0 * n1));
    const int A = clamp_cell(2 * i + (sx ? 0 : -1) + (q & 1), 2 * g.nx),
              B = clamp_cell(2 * j + (sy ? 0 : -1) + ((q >> 1) & 1), 2 * g.ny);
    double f;
    if constexpr (DIM == 2) {
        double p[2][2];
        const int neg = cell_nodes(phi, g.nx + 1, A >> 1, B >> 1, p);
        f = neg == 0 ? 0.0 : (neg == 4 ? 1.0 : sub_frac(p, A & 1, B & 1));
    } else {
        const int C = clamp_cell(2 * k + (sz ? 0 : -1) + (q >> 2), 2 * g.nz);
        double p[2][2][2];
        const int neg = cell_nodes(phi, g.nx + 1, g.ny + 1, A >> 1, B >> 1, C >> 1, p);
        f = neg == 0 ? 0.0 : (neg == 8 ? 1.0 : sub_frac(p, A & 1, B & 1, C & 1));
    }
    f = f + __shfl_xor(f, 1);
    f = f + __shfl_xor(f, 2);
    if constexpr (DIM == 3) f = f + __shfl_xor(f, 4);
    if (q == 0) (KEEP ? kept : out)[e] = snap(f * (DIM == 2 ? 0.25 : 0.125), w_min);
}

__global__ __launch_bounds__(256) void k_kept_out(long long n, double* __restrict__ out) {
    const long long t = (long long)blockIdx.x * blockDim.x + threadIdx.x;
    if (t < n) out[t] = kept[t];
}

__global__ void k_fill(double* __restrict__ d, long long n, double v) {
    const long long t = (long long)blockIdx.x * blockDim.x + threadIdx.x;
    if (t < n) d[t] = v;
}

}  // namespace

void launch_fill(double* dst, long long n, double v, hipStream_t s) {
    const int bs = 256;
    if (n <= 0) return;
    hipLaunchKernelGGL(k_fill, dim3((unsigned)((n + bs - 1) / bs)), dim3(bs), 0, s, dst, n, v);
}

template <int DIM>
static void launch_weights_dim(const Geo& g, const double* phi_l, const double* phi_s, double w_min,
                               double* WL, double* WF, hipStream_t s) {
    using F = FTile<DIM>;
    const dim3 gs(g.nx / F::TX + 1, g.ny / F::TY + 1, DIM == 2 ? 1 : g.nz / F::TZ + 1);
    hipLaunchKernelGGL(k_weights<DIM>, gs, dim3(F::NT), 0, s, g, phi_l, phi_s, w_min, WL, WF);
}

void launch_weights(const Geo& g, const double* phi_l, const double* phi_s, double w_min, double* WL,
                    double* WF, hipStream_t s) {
    if (g.dim == 2)
        launch_weights_dim<2>(g, phi_l, phi_s, w_min, WL, WF, s);
    else
        launch_weights_dim<3>(g, phi_l, phi_s, w_min, WL, WF, s);
}

void launch_weights_set(const Geo& g, int set, const double* phi_l, double w_min, double* out,
                        hipStream_t s) {
    int shp[3];
    set_shape(g, set, shp);
    const long long n = (long long)shp[0] * shp[1] * (g.dim == 3 ? shp[2] : 1);
    const int sx = shp[0] == g.nx, sy = shp[1] == g.ny, sz = g.dim == 3 ? shp[2] == g.nz : 1;
    const unsigned nb = (unsigned)((n * (1 << g.dim) + 255) / 256);
    const long long nodes = (long long)(g.nx + 1) * (g.ny + 1) * (g.dim == 3 ? g.nz + 1 : 1);
    const bool keep = out < phi_l + nodes && phi_l < out + n;
    auto launch = [&](auto kernel) {
        hipLaunchKernelGGL(kernel, dim3(nb), dim3(256), 0, s, g, shp[0], shp[1], g.dim == 3 ? shp[2] : 1, sx,
                           sy, sz, phi_l, w_min, out);
    };
    if (g.dim == 2)
        keep ? launch(k_weights_set<2, true>) : launch(k_weights_set<2, false>);
    else
        keep ? launch(k_weights_set<3, true>) : launch(k_weights_set<3, false>);
    if (keep)
        hipLaunchKernelGGL(k_kept_out, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, n, out);
}

}  // namespace vfs

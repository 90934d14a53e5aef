// 3D Jacobi-preconditioned CG as one resident kernel: a whole solve in one
// launch, for active sets of at most one brick per compute unit.
//
// Launched once per iteration a short tile list is bound by the launch and by
// the chain of planes a workgroup marches through, and each 64 x 4 x 8 tile of
// it is mostly empty.  Here the active set is cut into small bricks whose
// vectors stay in registers; a workgroup forms its brick's faces in LDS and
// trades sums and rim values by stamped words (vfs_resident.h), as in 2D.  The
// halo of a brick is as large as the brick, so the exchange is what an iteration
// waits for: the rim goes out as one packed plane per side and sample.
//
// Bricks of 8 x 8 x 8 anchors (512 threads, one each); in FP32, where those are
// more than the compute units, 16 x 8 x 8 (1024 threads: with 512 of two anchors
// each the 226 spilled registers took 26 us an iteration at 64^3, against 18).
// In FP64 the wide brick's fields alone exceed the LDS.  c, K and 1 / a lie in
// LDS where the registers would spill.  Measured, us an iteration, launched and
// resident: FP32 128^3 column (76 000 unknowns) 19.1 and 5.7, 24^3 pool 16.0 and
// 7.5, 60 x 64 x 52 pool 25.7 and 16.2, 64^3 27.2 and 17.9; FP64 column 37.5 and
// 8.9, 24^3 19.0 and 10.0, 64 x 30 x 36 25.0 and 10.0.
//
// The vectors are kept weighted as in k_fused3d (R = e r, P = a p, Q = e A p,
// e = a D^-1; r, z and p from 1 / e and 1 / a), and in FP32 every rounding is
// that of k_fused3d, so a solve takes the same steps resident and not.  The
// compiler contracts A p = a S + c p differently in the two shapes of that
// kernel; `pair` says which one would have run, `fold` whether its last column
// is folded.
#include "vfs_internal.h"
#include "vfs_resident.h"

#include <algorithm>

namespace vfs {
namespace {

template <int BX, int BY, int BZ>
struct Brick {
    static constexpr int anchors = BX * BY * BZ;
    static constexpr int NT = anchors < 1024 ? anchors : 1024, NW = NT / 64;   // threads, waves
    static constexpr int RPT = anchors / NT;   // anchors per thread
    static constexpr int HX = BX + 2, HY = BY + 2, HZ = BZ + 2;
    static constexpr int ring = HX * HY * HZ - anchors;
    static constexpr int NR = (ring + NT - 1) / NT;
    // faces beyond the anchors' own: per axis the far plane, and the near
    // planes of the two other axes
    static constexpr int sx = BY * BZ, sy = BX * BZ, sz = BX * BY;
    static constexpr int extra = 3 * (sx + sy + sz);
    static constexpr int NE = (extra + NT - 1) / NT;
    // message: six planes (x low, x high, y low, ...) of six samples
    __host__ __device__ static constexpr int plane(int q) {
        return q < 2 ? q * 6 * sx : (q < 4 ? 12 * sx + (q - 2) * 6 * sy : 12 * (sx + sy) + (q - 4) * 6 * sz);
    }
    __host__ __device__ static constexpr int psize(int q) { return q < 2 ? sx : (q < 4 ? sy : sz); }
    static constexpr int values = 12 * (sx + sy + sz);
};

template <typename T>
struct Res3dArgs {
    Geo g;
    const T* r;      // residual the solve starts from (kept)
    T* x;            // iterate, updated at the end
    const T* e;      // FP32: a D^-1; FP64: D^-1
    const T* a;
    const T* c;
    const T* K;
    const int* list;   // bricks
    const int* rank;   // workgroup of every brick of the lattice, or -1
    int nbx, nby;      // bricks of the lattice along x and y
    LLWord* part;
    LLWord* msg;       // [2][kResMost][message]
    unsigned stamp;
    int set_bb;
    int pair;          // the launched iteration would run two threads an anchor
    int fold;          // and fold the column i = nx
    Scalars* sc;
};

// 1 / a, c and K in LDS: FP64 and the wide brick have too few registers (57 and
// 60 spilled so, 82 and 73 otherwise; the narrow FP32 brick spills none)
template <typename T, int BX, int BY, int BZ>
constexpr bool kCoefLds = sizeof(T) == 8 || Brick<BX, BY, BZ>::anchors > 512;
template <typename T, int BX, int BY, int BZ>
constexpr bool kInvLds = kCoefLds<T, BX, BY, BZ>;

template <typename T, int BX, int BY, int BZ>
struct Res3dLds {
    using B = Brick<BX, BY, BZ>;
    T w[6][B::HZ][B::HY][B::HX];                        // a p of the brick and its halo
    T gu[BZ + 1][BY + 1][BX + 1];                       // u at x 0.., y -1.., z -1..
    T gv[BZ + 1][BY + 1][BX + 1];                       // v at x -1.., y 0.., z -1..
    T gw[BZ + 1][BY + 1][BX + 1];                       // w at x -1.., y -1.., z 0..
    T x[6][B::anchors];
    T out[4][6][BX > BY ? BX * BZ : BY * BZ];           // x and y planes to send
    T ck[kCoefLds<T, BX, BY, BZ> ? 8 : 1][B::anchors];    // c of samples 1 to 5, K
    T ia[kInvLds<T, BX, BY, BZ> ? 6 : 1][B::anchors];     // 1 / a
    double tot[B::NW][8], part[B::NW][8];
    int abort;
};

// own anchors' share of the CG iteration; r_k of iteration 0 is the plain
// residual, later R / e
template <typename T, int BX, int BY, int BZ>
__global__ __launch_bounds__((Brick<BX, BY, BZ>::NT), 1) void k_resident3d(Res3dArgs<T> S) {
#pragma clang fp contract(off)
    using B = Brick<BX, BY, BZ>;
    constexpr int LW = kLLWords<T>;
    constexpr int RPT = B::RPT, NR = B::NR, NE = B::NE, NT = B::NT, NW = B::NW;
    constexpr int PS = NT / 8;   // workgroups whose sums are read at a time
    constexpr bool FP64 = sizeof(T) == 8;
    __shared__ Res3dLds<T, BX, BY, BZ> sh;
    const Geo& g = S.g;
    const long long NP = g.NP;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wid = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int W = gridDim.x, me = blockIdx.x;
    const int brick = S.list[me];
    const int bx = brick % S.nbx, by = (brick / S.nbx) % S.nby, bz = brick / (S.nbx * S.nby);
    const int i0 = bx * BX, j0 = by * BY, k0 = bz * BZ;
    auto inside = [&](int i, int j, int k) {
        return i >= 0 && i <= g.nx && j >= 0 && j <= g.ny && k >= 0 && k <= g.nz;
    };
    // samples outside the grid read offset 0, the zero pad of every slice
    auto off = [&](int i, int j, int k) { return inside(i, j, k) ? g.idx(i, j, k) : 0LL; };

    // own anchors
    T R[RPT][6], P[RPT][6], Q[RPT][6];
    constexpr bool CL = kCoefLds<T, BX, BY, BZ>, IL = kInvLds<T, BX, BY, BZ>;
    T A[RPT][6], IAr[RPT][6], E[RPT][6], IE[FP64 ? RPT : 1][6], CKr[RPT][8];
    auto CK = [&](int n, int s) { return CL ? sh.ck[CL ? s : 0][tid + NT * n] : CKr[n][s]; };
    auto IA = [&](int n, int s) { return IL ? sh.ia[IL ? s : 0][tid + NT * n] : IAr[n][s]; };
    auto set_ck = [&](int n, int s, T v) { (CL ? sh.ck[CL ? s : 0][tid + NT * n] : CKr[n][s]) = v; };
    int lx[RPT], ly[RPT], lz[RPT];
    bool last[RPT];   // the folded column
#pragma unroll
    for (int n = 0; n < RPT; ++n) {
        const int t = tid + NT * n;
        lx[n] = t % BX;
        ly[n] = (t / BX) % BY;
        lz[n] = t / (BX * BY);
        const long long o = off(i0 + lx[n], j0 + ly[n], k0 + lz[n]);
        last[n] = S.fold && i0 + lx[n] == g.nx;
#pragma unroll
        for (int s = 0; s < 6; ++s) {
            A[n][s] = S.a[s * NP + o];
            E[n][s] = FP64 ? A[n][s] * S.e[s * NP + o] : S.e[s * NP + o];
            (IL ? sh.ia[IL ? s : 0][t] : IAr[n][s]) = A[n][s] != T(0) ? T(1) / A[n][s] : T(0);
            if constexpr (FP64) IE[n][s] = E[n][s] != T(0) ? T(1) / E[n][s] : T(0);
            sh.x[s][t] = S.x[s * NP + o];
            P[n][s] = S.r[s * NP + o];   // plain residual, for iteration 0
            R[n][s] = E[n][s] * P[n][s];
            Q[n][s] = T(0);
            if (s > 0) set_ck(n, s > 0 ? s - 1 : 0, S.c[s * NP + o]);
        }
#pragma unroll
        for (int q = 0; q < 3; ++q) set_ck(n, 5 + q, S.K[q * NP + o]);
    }
    // faces this workgroup needs, in brick coordinates
    auto nu = [&](int x, int y, int z) {
        return (x >= 0 && x <= BX && y >= 0 && y < BY && z >= 0 && z < BZ) ||
               (x >= 0 && x < BX && ((y == -1 && z >= 0 && z < BZ) || (z == -1 && y >= 0 && y < BY)));
    };
    auto nv = [&](int x, int y, int z) {
        return (x >= 0 && x < BX && y >= 0 && y <= BY && z >= 0 && z < BZ) ||
               (y >= 0 && y < BY && ((x == -1 && z >= 0 && z < BZ) || (z == -1 && x >= 0 && x < BX)));
    };
    auto nw = [&](int x, int y, int z) {
        return (x >= 0 && x < BX && y >= 0 && y < BY && z >= 0 && z <= BZ) ||
               (z >= 0 && z < BZ && ((x == -1 && y >= 0 && y < BY) || (y == -1 && x >= 0 && x < BX)));
    };
    // halo positions: place in LDS, state, and the words they come by
    T rR[NR][6], rP[NR][6], rQ[NR][6];
    int rat[NR];            // index in one sample's LDS box, -1: none
    unsigned need[NR];      // samples awaited
    long long src[NR];      // word of sample 0
    int sstep[NR];          // words from one sample to the next
#pragma unroll
    for (int n = 0; n < NR; ++n) {
        const int h = tid + NT * n;
        rat[n] = -1;
        need[n] = 0;
        src[n] = 0;
        sstep[n] = 0;
#pragma unroll
        for (int s = 0; s < 6; ++s) rR[n][s] = rP[n][s] = rQ[n][s] = T(0);
        if (h < B::ring) {
            constexpr int cap = B::HX * B::HY, rim = cap - BX * BY;
            int x, y, z;
            if (h < 2 * cap) {
                z = h < cap ? -1 : BZ;
                const int e = h % cap;
                x = e % B::HX - 1;
                y = e / B::HX - 1;
            } else {
                const int e = (h - 2 * cap) % rim;
                z = (h - 2 * cap) / rim;
                if (e < 2 * B::HX) {
                    y = e < B::HX ? -1 : BY;
                    x = e % B::HX - 1;
                } else {
                    y = (e - 2 * B::HX) >> 1;
                    x = (e & 1) ? BX : -1;
                }
            }
            rat[n] = ((z + 1) * B::HY + y + 1) * B::HX + x + 1;
            const int i = i0 + x, j = j0 + y, k = k0 + z;
            if (inside(i, j, k)) {
                const long long o = g.idx(i, j, k);
                const bool use[6] = {
                    nu(x, y, z) || nu(x + 1, y, z) || nv(x, y, z) || nv(x, y + 1, z) || nw(x, y, z) ||
                        nw(x, y, z + 1),
                    nu(x, y, z) || nu(x + 1, y, z) || nw(x, y, z) || nw(x, y, z + 1),
                    nv(x, y, z) || nv(x, y + 1, z) || nw(x, y, z) || nw(x, y, z + 1),
                    nu(x, y, z) || nu(x, y - 1, z) || nv(x, y, z) || nv(x - 1, y, z),
                    nu(x, y, z) || nu(x, y, z - 1) || nw(x, y, z) || nw(x - 1, y, z),
                    nv(x, y, z) || nv(x, y, z - 1) || nw(x, y, z) || nw(x, y - 1, z)};
#pragma unroll
                for (int s = 0; s < 6; ++s)
                    if (const T a = S.a[s * NP + o]; use[s] && a != T(0)) {
                        const T e = FP64 ? a * S.e[s * NP + o] : S.e[s * NP + o];
                        need[n] |= 1u << s;
                        rR[n][s] = e * S.r[s * NP + o];
                    }
                if (need[n]) {
                    // an active sample's brick is in the list; the plane it is
                    // read from: along an axis on which it lies beyond this brick
                    const int dx = x < 0 ? -1 : x / BX, dy = y < 0 ? -1 : y / BY, dz = z < 0 ? -1 : z / BZ;
                    const int ux = x - dx * BX, uy = y - dy * BY, uz = z - dz * BZ;
                    const int who = S.rank[(bx + dx) + S.nbx * ((by + dy) + S.nby * (bz + dz))];
                    const int ax = dx ? 0 : (dy ? 1 : 2);
                    const int pl = 2 * ax + ((ax == 0 ? dx : (ax == 1 ? dy : dz)) < 0 ? 1 : 0);
                    const int at = ax == 0 ? uy + BY * uz : (ax == 1 ? ux + BX * uz : ux + BX * uy);
                    src[n] = ((long long)who * B::values + B::plane(pl) + at) * LW;
                    sstep[n] = B::psize(pl) * LW;
                    if (who < 0) need[n] = 0;
                }
            }
        }
    }
    // extra faces: kind 0..8 = (axis u, v, w) x (far plane, near planes)
    int ekind[NE], ex[NE], ey[NE], ez[NE];
    T eK[NE];
#pragma unroll
    for (int n = 0; n < NE; ++n) {
        int e = tid + NT * n;
        ekind[n] = -1;
        eK[n] = T(0);
        ex[n] = ey[n] = ez[n] = 0;
        constexpr int size[9] = {B::sx, B::sy, B::sz, B::sx, B::sy, B::sz, B::sx, B::sy, B::sz};
#pragma unroll
        for (int q = 0; q < 9; ++q) {
            if (ekind[n] < 0 && e < size[q]) {
                ekind[n] = q;
                const int ax = q % 3;   // the plane's axis
                const int u = ax == 0 ? e % BY : e % BX, w = ax == 0 ? e / BY : e / BX;
                const int at = ax == q / 3 ? (ax == 0 ? BX : (ax == 1 ? BY : BZ)) : -1;
                ex[n] = ax == 0 ? at : u;
                ey[n] = ax == 0 ? u : (ax == 1 ? at : w);
                ez[n] = ax == 2 ? at : w;
                const int i = i0 + ex[n], j = j0 + ey[n], k = k0 + ez[n];
                eK[n] = S.K[(q / 3) * NP + off(i, j, k)];
            } else if (ekind[n] < 0) {
                e -= size[q];
            }
        }
    }
    if (tid < 8 * NW) sh.part[tid >> 3][tid & 7] = 0.0;
    if (tid == 0) sh.abort = 0;
    const double tol2 = S.sc->tol2;
    const int max_iter = S.sc->max_iter;
    double bb = S.set_bb ? 0.0 : S.sc->bb;
    int* abort_flag = &S.sc->aborted;
    T* const w0 = &sh.w[0][0][0][0];
    constexpr int box = B::HX * B::HY * B::HZ;
    // numerators of the faces at brick coordinates (x, y, z), from LDS
    auto wat = [&](int s, int x, int y, int z) { return sh.w[s][z + 1][y + 1][x + 1]; };
    auto fu = [&](int x, int y, int z) {
        return (wat(0, x, y, z) - wat(0, x - 1, y, z)) + (wat(1, x - 1, y, z) - wat(1, x, y, z)) +
               (wat(3, x, y, z) - wat(3, x, y + 1, z)) + (wat(4, x, y, z) - wat(4, x, y, z + 1));
    };
    auto fv = [&](int x, int y, int z) {
        return (wat(0, x, y, z) - wat(0, x, y - 1, z)) + (wat(2, x, y - 1, z) - wat(2, x, y, z)) +
               (wat(3, x, y, z) - wat(3, x + 1, y, z)) + (wat(5, x, y, z) - wat(5, x, y, z + 1));
    };
    auto fw = [&](int x, int y, int z) {
        return (wat(0, x, y, z) - wat(0, x, y, z - 1)) + (wat(1, x, y, z) - wat(1, x, y, z - 1)) +
               (wat(2, x, y, z) - wat(2, x, y, z - 1)) + (wat(4, x, y, z) - wat(4, x + 1, y, z)) +
               (wat(5, x, y, z) - wat(5, x, y + 1, z));
    };

    auto total = [](const double (*s)[8]) {
        double t = waves_total8(s);
        if constexpr (NW == 16) t += waves_total8(s + 8);
        return t;
    };

    T alpha = T(0), beta = T(0);
    for (int k = 0;; ++k) {
        if (k > 0) {
            const unsigned want = S.stamp + (unsigned)k;
            double tot[5];
            if (W > 1) {
                const LLWord* msg = S.msg + (long long)(want & 1) * kResMost * B::values * LW;
                const LLWord* pw = S.part + (long long)(want & 1) * kResMost * 16 + 2 * min(tid & 7, 4);
                const int np = (W + PS - 1) / PS;
                double sum = 0.0;
                LLPatience wait;
                ll_first_wait(W);
                for (;;) {
                    LLSlot<double> ps[kResMost / PS];
                    LLSlot<T> rs[NR][6];
#pragma unroll
                    for (int m = 0; m < kResMost / PS; ++m)
                        if (m < np) ps[m].load(pw + min((tid >> 3) + PS * m, W - 1) * 16);
#pragma unroll
                    for (int n = 0; n < NR; ++n)
                        if (need[n]) {
#pragma unroll
                            for (int s = 0; s < 6; ++s) rs[n][s].load(msg + src[n] + s * sstep[n]);
                        }
                    bool got = true;
                    sum = 0.0;
#pragma unroll
                    for (int m = 0; m < kResMost / PS; ++m)
                        if (m < np) {
                            got &= ps[m].ready(want);
                            if ((tid >> 3) + PS * m < W) sum += ps[m].value();
                        }
#pragma unroll
                    for (int n = 0; n < NR; ++n)
#pragma unroll
                        for (int s = 0; s < 6; ++s) {
                            const bool nd = (need[n] >> s) & 1u;
                            got &= !nd || rs[n][s].ready(want);
                            rQ[n][s] = nd ? rs[n][s].value() : T(0);
                        }
                    if (__all(got)) break;
                    if (wait.over(abort_flag, nullptr)) {
                        sh.abort = 1;
                        break;
                    }
                }
                sum = swap_rows32(swap_rows16(sum + dpp_perm<0x128>(sum)));   // row_ror:8
                if (lane < 8) sh.tot[wid][lane] = sum;
                __syncthreads();
                if (sh.abort) return;
                const double t = total(sh.tot);
#pragma unroll
                for (int q = 0; q < 5; ++q) tot[q] = lane_value(t, q);
            } else {
                const double t = total(sh.part);
#pragma unroll
                for (int q = 0; q < 5; ++q) tot[q] = lane_value(t, q);
                __syncthreads();
            }
            if (S.set_bb && k == 1) bb = tot[4];
            const CgStep st = cg_step(tot, tol2, bb, k - 1, max_iter);
            if (st.stop) {
                if (me == 0 && tid == 0) {
                    Scalars* sc = S.sc;
                    sc->rr = tot[4];
                    sc->pq = tot[1];
                    if (S.set_bb) sc->bb = bb;
                    sc->iter = k - 1;
                    sc->done = st.stop;
                }
                break;
            }
            alpha = (T)st.alpha;
            beta = (T)st.beta;
        }
        const bool first = k == 0;
        double part[5] = {};
        // R_k, a p_k, x_k
#pragma unroll
        for (int n = 0; n < RPT; ++n) {
#pragma unroll
            for (int s = 0; s < 6; ++s) {
                const T ia = IA(n, s), pi = P[n][s] * ia;
                if (!first) sh.x[s][tid + NT * n] = ll_fma(alpha, pi, sh.x[s][tid + NT * n]);
                const T Rn = ll_fma(-alpha, Q[n][s], R[n][s]);
                T ie;
                if constexpr (FP64)
                    ie = IE[n][s];
                else
                    ie = E[n][s] != T(0) ? __builtin_amdgcn_rcpf(E[n][s]) : T(0);
                const T rn = first ? P[n][s] : Rn * ie;
                const T zn = Rn * ia;
                P[n][s] = first ? Rn : ll_fma(beta, P[n][s], Rn);
                R[n][s] = Rn;
                // inactive samples hold zeros, except a plain residual that the
                // caller may have left there
                if (A[n][s] != T(0)) {
                    part[0] = ll_fma((double)rn, (double)zn, part[0]);
                    part[4] = ll_fma((double)rn, (double)rn, part[4]);
                }
                sh.w[s][lz[n] + 1][ly[n] + 1][lx[n] + 1] = P[n][s];
            }
        }
#pragma unroll
        for (int n = 0; n < NR; ++n)
            if (rat[n] >= 0) {
#pragma unroll
                for (int s = 0; s < 6; ++s) {
                    rR[n][s] = ll_fma(-alpha, rQ[n][s], rR[n][s]);
                    rP[n][s] = ll_fma(beta, rP[n][s], rR[n][s]);
                    w0[s * box + rat[n]] = rP[n][s];
                }
            }
        __syncthreads();
        // faces
        T gu[RPT], gv[RPT], gw[RPT];
#pragma unroll
        for (int n = 0; n < RPT; ++n) {
            gu[n] = CK(n, 5) * fu(lx[n], ly[n], lz[n]);
            gv[n] = CK(n, 6) * fv(lx[n], ly[n], lz[n]);
            gw[n] = CK(n, 7) * fw(lx[n], ly[n], lz[n]);
            sh.gu[lz[n] + 1][ly[n] + 1][lx[n]] = gu[n];
            sh.gv[lz[n] + 1][ly[n]][lx[n] + 1] = gv[n];
            sh.gw[lz[n]][ly[n] + 1][lx[n] + 1] = gw[n];
        }
#pragma unroll
        for (int n = 0; n < NE; ++n) {
            const int ax = ekind[n] < 0 ? -1 : ekind[n] / 3;
            if (ax == 0) sh.gu[ez[n] + 1][ey[n] + 1][ex[n]] = eK[n] * fu(ex[n], ey[n], ez[n]);
            if (ax == 1) sh.gv[ez[n] + 1][ey[n]][ex[n] + 1] = eK[n] * fv(ex[n], ey[n], ez[n]);
            if (ax == 2) sh.gw[ez[n]][ey[n] + 1][ex[n] + 1] = eK[n] * fw(ex[n], ey[n], ez[n]);
        }
        __syncthreads();
        // A p at the own anchors
        const unsigned stamp = S.stamp + (unsigned)k + 1u;
        LLWord* out = S.msg + ((long long)(stamp & 1) * kResMost + me) * B::values * LW;
#pragma unroll
        for (int n = 0; n < RPT; ++n) {
            const int x = lx[n], y = ly[n], z = lz[n];
            const T gu0 = gu[n], gu1 = sh.gu[z + 1][y + 1][x + 1], gum = sh.gu[z + 1][y][x],
                    guz = sh.gu[z][y + 1][x];
            const T gv0 = gv[n], gv1 = sh.gv[z + 1][y + 1][x + 1], gvm = sh.gv[z + 1][y][x],
                    gvz = sh.gv[z][y][x + 1];
            const T gw0 = gw[n], gw1 = sh.gw[z + 1][y + 1][x + 1], gwx = sh.gw[z][y + 1][x],
                    gwy = sh.gw[z][y][x + 1];
            T p[6], ia[6];
#pragma unroll
            for (int s = 0; s < 6; ++s) {
                ia[s] = IA(n, s);
                p[s] = P[n][s] * ia[s];
            }
            const T cross = T(0.5) * fmin(CK(n, 0), CK(n, 1));
            // a S + c p, contracted on either product
            auto form = [&](int s, T S6, bool on_a) {
                const T a = A[n][s], c = CK(n, s - 1);
                return on_a ? ll_fma(a, S6, c * p[s]) : ll_fma(c, p[s], a * S6);
            };
            const bool pair = S.pair != 0;
            T y6[6];
            y6[0] = A[n][0] * ((gu0 - gu1) + (gv0 - gv1) + (gw0 - gw1));
            y6[1] = ll_fma(cross, p[2], form(1, (gu1 - gu0) + (gw0 - gw1), pair));
            y6[2] = ll_fma(cross, p[1], form(2, (gv1 - gv0) + (gw0 - gw1), false));
            y6[3] = form(3, (gu0 - gum) + (gv0 - gvm), pair || last[n]);
            y6[4] = form(4, (gu0 - guz) + (gw0 - gwx), pair || last[n]);
            y6[5] = form(5, (gv0 - gvz) + (gw0 - gwy), pair);
#pragma unroll
            for (int s = 0; s < 6; ++s) {
                const T dd = E[n][s] * ia[s], zn = R[n][s] * ia[s];
                const double yd = y6[s];
                part[1] = ll_fma((double)p[s], yd, part[1]);
                part[2] = ll_fma((double)zn, yd, part[2]);
                part[3] = ll_fma((double)dd * yd, yd, part[3]);
                Q[n][s] = (dd * A[n][s]) * y6[s];
                if (x == 0) sh.out[0][s][y + BY * z] = Q[n][s];
                if (x == BX - 1) sh.out[1][s][y + BY * z] = Q[n][s];
                if (y == 0) sh.out[2][s][x + BX * z] = Q[n][s];
                if (y == BY - 1) sh.out[3][s][x + BX * z] = Q[n][s];
                if (W > 1) {
                    if (z == 0) ll_put(out + (B::plane(4) + s * B::sz + x + BX * y) * LW, Q[n][s], stamp);
                    if (z == BZ - 1)
                        ll_put(out + (B::plane(5) + s * B::sz + x + BX * y) * LW, Q[n][s], stamp);
                }
            }
        }
        double four, fifth;
        wave_sum5(part, four, fifth);
        if (lane < 4) sh.part[wid][lane] = four;
        if (lane == 0) sh.part[wid][4] = fifth;
        __syncthreads();
        if (W > 1) {
            if (wid == 0) {
                const double t = total(sh.part);
                if (lane < 5)
                    ll_put(S.part + ((long long)(stamp & 1) * kResMost + me) * 16 + 2 * lane, t, stamp);
            }
            // x and y planes, 64 values a wave at a time
            constexpr int rx = 12 * B::sx / 64, ry = 12 * B::sy / 64;
            static_assert(B::sx % 64 == 0 && B::sy % 64 == 0, "whole waves a plane");
            for (int row = wid; row < rx + ry; row += NW) {
                const bool isx = row < rx;
                const int e = (isx ? row : row - rx) * 64 + lane, sz = isx ? B::sx : B::sy;
                const int q = e / (6 * sz), s = (e / sz) % 6, at = e % sz;
                ll_put(out + (B::plane((isx ? 0 : 2) + q) + s * sz + at) * LW, sh.out[(isx ? 0 : 2) + q][s][at],
                       stamp);
            }
        }
    }
#pragma unroll
    for (int n = 0; n < RPT; ++n) {
        const int i = i0 + lx[n], j = j0 + ly[n], k = k0 + lz[n];
        if (!inside(i, j, k)) continue;
        const long long o = g.idx(i, j, k);
#pragma unroll
        for (int s = 0; s < 6; ++s)
            if (A[n][s] != T(0)) S.x[s * NP + o] = sh.x[s][tid + NT * n];
    }
}

// flag of every brick: some sample has a != 0 (one workgroup a brick)
__global__ __launch_bounds__(256) void k_res3d_flags(Geo g, int bx, int by, int bz, int nbx, int nby,
                                                     const double* __restrict__ a,
                                                     const int* __restrict__ tflags, int ntx, int nty,
                                                     int* __restrict__ flags) {
    const int b = blockIdx.x;
    const int i0 = (b % nbx) * bx, j0 = ((b / nbx) % nby) * by, k0 = (b / (nbx * nby)) * bz;
    // a brick lies in two 64 x 4 x 8 tiles; most are in none that is active
    static_assert(kTile3X % 16 == 0 && kTile3Y == 4 && kTile3Z == 8, "bricks and tiles");
    const int t0 = i0 / kTile3X + ntx * (j0 / kTile3Y + nty * (k0 / kTile3Z));
    const bool second = j0 / kTile3Y + 1 < nty;
    if (!tflags[t0] && !(second && tflags[t0 + ntx])) {
        if (threadIdx.x == 0) flags[b] = 0;
        return;
    }
    int any = 0;
    for (int e = threadIdx.x; e < bx * by * bz; e += 256) {
        const int i = i0 + e % bx, j = j0 + (e / bx) % by, k = k0 + e / (bx * by);
        if (i <= g.nx && j <= g.ny && k <= g.nz)
            for (int s = 0; s < 6; ++s) any |= a[s * g.NP + g.idx(i, j, k)] != 0.0;
    }
    any = __syncthreads_or(any);
    if (threadIdx.x == 0) flags[b] = any;
}

// ordered list of the flagged bricks (its first kResMost), their number, and
// the place of every brick in it (-1: none); one workgroup
__global__ __launch_bounds__(1024) void k_res3d_list(int n, const int* __restrict__ flags,
                                                     int* __restrict__ list, int* __restrict__ rank,
                                                     int* __restrict__ count) {
    __shared__ int sCnt[16];
    const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
    int base = 0;
    for (int t0 = 0; t0 < n; t0 += 1024) {
        const int t = t0 + threadIdx.x;
        const int any = t < n ? flags[t] : 0;
        const unsigned long long m = __ballot(any);
        if (lane == 0) sCnt[wid] = __popcll(m);
        __syncthreads();
        int before = base, all = 0;
        for (int w = 0; w < 16; ++w) {
            if (w < wid) before += sCnt[w];
            all += sCnt[w];
        }
        const int at = before + __popcll(m & ((1ull << lane) - 1ull));
        if (t < n) rank[t] = any && at < kResMost ? at : -1;
        if (any && at < kResMost) list[at] = t;
        base += all;
        __syncthreads();
    }
    if (threadIdx.x == 0) *count = base;
}

struct Shape {
    int bx, by, bz;
};
Shape shape_of(int shape) { return shape == 0 ? Shape{8, 8, 8} : Shape{16, 8, 8}; }

template <typename T, int BX, int BY, int BZ>
void launch_shape(const Res3dArgs<T>& S, int count, hipStream_t s) {
    hipLaunchKernelGGL((k_resident3d<T, BX, BY, BZ>), dim3(count), dim3(Brick<BX, BY, BZ>::NT), 0, s, S);
}

}  // namespace

void res3d_lattice(const Geo& g, int shape, int& nbx, int& nby, int& nbz) {
    const Shape b = shape_of(shape);
    nbx = g.nx / b.bx + 1;
    nby = g.ny / b.by + 1;
    nbz = g.nz / b.bz + 1;
}

// words of the messages of kResMost workgroups, both parities; FP64 for the
// first shape, FP32 for the second
long long res3d_words() {
    return std::max(2LL * kResMost * Brick<8, 8, 8>::values * 2, 2LL * kResMost * Brick<16, 8, 8>::values);
}

void launch_res3d_lists(const Geo& g, int shape, const double* a, const int* tile_flags, int* flags,
                        int* list, int* rank, int* count, hipStream_t s) {
    int nbx, nby, nbz, ntx, nty, ntz;
    tile_dims(g, ntx, nty, ntz);
    res3d_lattice(g, shape, nbx, nby, nbz);
    const Shape b = shape_of(shape);
    const int n = nbx * nby * nbz;
    hipLaunchKernelGGL(k_res3d_flags, dim3(n), dim3(256), 0, s, g, b.bx, b.by, b.bz, nbx, nby, a,
                       tile_flags, ntx, nty, flags);
    hipLaunchKernelGGL(k_res3d_list, dim3(1), dim3(1024), 0, s, n, flags, list, rank, count);
}

template <typename T>
void launch_resident3d(const Geo& g, int shape, const int* list, const int* rank, int count, const T* r,
                       T* x, const T* e, const T* a, const T* c, const T* K, LLWordBuf part,
                       LLWordBuf msg, unsigned stamp, bool set_bb, bool pair, bool fold, Scalars* sc,
                       hipStream_t s) {
    int nbx, nby, nbz;
    res3d_lattice(g, shape, nbx, nby, nbz);
    const Res3dArgs<T> S{g,   r,    x,   e,     a,              c,            K,            list, rank, nbx, nby,
                         part, msg, stamp, set_bb ? 1 : 0, pair ? 1 : 0, fold ? 1 : 0, sc};
    if (shape == 0) launch_shape<T, 8, 8, 8>(S, count, s);
    else if constexpr (sizeof(T) == 4) launch_shape<T, 16, 8, 8>(S, count, s);
}

template void launch_resident3d<float>(const Geo&, int, const int*, const int*, int, const float*, float*,
                                       const float*, const float*, const float*, const float*, LLWordBuf,
                                       LLWordBuf, unsigned, bool, bool, bool, Scalars*, hipStream_t);
template void launch_resident3d<double>(const Geo&, int, const int*, const int*, int, const double*,
                                        double*, const double*, const double*, const double*, const double*,
                                        LLWordBuf, LLWordBuf, unsigned, bool, bool, bool, Scalars*,
                                        hipStream_t);

}  // namespace vfs

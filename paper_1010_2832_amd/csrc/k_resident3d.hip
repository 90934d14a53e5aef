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
// Bricks of 8 x 8 x 8 anchors (512 threads, one each).  Where those are more than
// the compute units: in FP32 16 x 8 x 8 (1024 threads); in FP64, where the wide
// brick's fields alone exceed the LDS, two small bricks to a unit, which keep only
// R, Q and the halo's R in registers and stream the rest (a, D^-1, c, K, x) from
// rows of their own.  Of those up to 512 workgroups the first adds the sums and
// writes each of the others its own line: 474 workgroups reading 474 lines, or all
// one line, slowed everything else (88 x 56 x 72: 100 and 330 ms a step, now 36 to 42).
// a p lies in LDS, c, K and 1 / a too, where the registers would spill, and
// addresses are renewed in every iteration (hoisted by the compiler they were
// spilled, and 64^3 took 17.9 us an iteration).  Measured, us an iteration,
// launched and resident: FP32 128^3 column (76 000 unknowns) 19.1 and 5.7, 24^3
// pool 16.0 and 7.0, 60 x 64 x 52 pool 25.7 and 9.7, 64^3 27.2 and 10.1; FP64
// column 37.5 and 7.5, 24^3 19.0 and 7.9, 64 x 30 x 36 25.0 and 8.7; two to a
// unit, 88 x 56 x 72, 81 and 46: 40% of it for the fields and what is spilled (172
// registers of 128), 300 MB an iteration from beyond the L2.
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

constexpr int kResStream = 26;   // fields that a streaming workgroup keeps in memory

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
    double* buf;       // streamed fields of every workgroup, or null
    LLWord* part;
    LLWord* msg;       // [2][workgroups][message]
    unsigned stamp;
    int set_bb;
    int pair;          // the launched iteration would run two threads an anchor
    int fold;          // and fold the column i = nx
    Scalars* sc;
};

// PER bricks share a compute unit: one, or two that stream what does not change
// and x from memory.
//
// 1 / a, c and K in LDS, and a p in LDS alone: FP64 and the wide brick have too few
// registers (with this none and 2 spilled, without 82 and 73)
template <typename T, int BX, int BY, int BZ, int PER>
constexpr bool kCoefLds = PER == 1 && (sizeof(T) == 8 || Brick<BX, BY, BZ>::anchors > 512);

template <typename T, int BX, int BY, int BZ, int PER>
struct Res3dLds {
    using B = Brick<BX, BY, BZ>;
    T w[6][B::HZ][B::HY][B::HX];                        // a p of the brick and its halo
    T gu[BZ + 1][BY + 1][BX + 1];                       // u at x 0.., y -1.., z -1..
    T gv[BZ + 1][BY + 1][BX + 1];                       // v at x -1.., y 0.., z -1..
    T gw[BZ + 1][BY + 1][BX + 1];                       // w at x -1.., y -1.., z 0..
    static constexpr bool coef = kCoefLds<T, BX, BY, BZ, PER>;
    T x[PER == 1 ? 6 : 1][PER == 1 ? B::anchors : 1];
    T out[4][6][BX > BY ? BX * BZ : BY * BZ];           // x and y planes to send
    T ck[coef ? 8 : 1][coef ? B::anchors : 1];           // c of samples 1 to 5, K
    T ia[coef ? 6 : 1][coef ? B::anchors : 1];           // 1 / a
    double tot[B::NW][8], part[B::NW][8];
    int abort;
};

// 1 / v, 0 for 0: v_rcp_f64 and two Newton steps
__device__ __forceinline__ double reciprocal(double v) {
    double r = __builtin_amdgcn_rcp(v);
    r = __builtin_fma(__builtin_fma(-v, r, 1.0), r, r);
    r = __builtin_fma(__builtin_fma(-v, r, 1.0), r, r);
    return v != 0.0 ? r : 0.0;
}

// a value that all lanes have, as a scalar
__device__ __forceinline__ double scalar(double v) {
    return __hiloint2double(__builtin_amdgcn_readfirstlane(__double2hiint(v)),
                            __builtin_amdgcn_readfirstlane(__double2loint(v)));
}
__device__ __forceinline__ float scalar(float v) {
    return __int_as_float(__builtin_amdgcn_readfirstlane(__float_as_int(v)));
}

// own anchors' share of the CG iteration; r_k of iteration 0 is the plain
// residual, later R / e
template <typename T, int BX, int BY, int BZ, int PER>
__global__ __launch_bounds__((Brick<BX, BY, BZ>::NT), (PER * Brick<BX, BY, BZ>::NW / 4)) void k_resident3d(
    Res3dArgs<T> S) {
#pragma clang fp contract(off)
    using B = Brick<BX, BY, BZ>;
    constexpr int LW = kLLWords<T>;
    constexpr int RPT = B::RPT, NR = B::NR, NE = B::NE, NT = B::NT, NW = B::NW;
    constexpr int PS = NT / 8;   // workgroups whose sums are read at a time
    constexpr int MP = PER * kResMost / PS;
    constexpr bool central = PER > 1;   // the first workgroup adds up for all
    constexpr bool FP64 = sizeof(T) == 8;
    constexpr bool stream = PER > 1;
    static_assert(!stream || (FP64 && RPT == 1), "streamed: FP64, one anchor a thread");
    __shared__ Res3dLds<T, BX, BY, BZ, PER> sh;
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

    T* const w0 = &sh.w[0][0][0][0];
    constexpr int box = B::HX * B::HY * B::HZ;

    // own anchors
    constexpr bool hold = !stream && !kCoefLds<T, BX, BY, BZ, PER>;   // a p in registers too
    T R[RPT][6], Q[RPT][6], Pk[hold ? RPT : 1][6];
    constexpr bool CL = kCoefLds<T, BX, BY, BZ, PER>;
    constexpr int held = stream ? 1 : RPT;
    T Ar[held][6], IAr[held][6], Er[held][6], IEr[FP64 ? held : 1][6], CKr[held][8];
    // places, renewed in every iteration: addresses hoisted out of the loop fill
    // the registers and come back from scratch memory
    int tt = tid;
    // streamed: the thread's own copies of a, D^-1, x (6 each), c and K, a row of NT
    // for each field (from the grid's slices, 64-byte rows of 26 arrays, a step at
    // 88 x 56 x 72 took 57.1 ms against 54.6)
    int mine = me * kResStream * NT;
    auto row = [&](int f) -> T& { return *(T*)((char*)S.buf + (unsigned)(mine + f * NT + tt) * 8u); };
    auto lx = [&](int n) { return (tt + NT * n) % BX; };
    auto ly = [&](int n) { return (tt + NT * n) / BX % BY; };
    auto lz = [&](int n) { return (tt + NT * n) / (BX * BY); };
    // streamed: a, D^-1, c and K of the iteration, loaded ahead of their use
    T As[stream ? 6 : 1], Ds[stream ? 6 : 1], CKs[stream ? 8 : 1];
    // c of samples 1 to 5 and K; 1 / a
    auto CK = [&](int n, int s) -> T {
        if constexpr (stream) return CKs[s];
        return CL ? sh.ck[CL ? s : 0][tid + NT * n] : CKr[n][s];
    };
    auto A = [&](int n, int s) -> T { return stream ? As[stream ? s : 0] : Ar[stream ? 0 : n][s]; };
    auto E = [&](int n, int s) -> T {
        return stream ? As[stream ? s : 0] * Ds[stream ? s : 0] : Er[stream ? 0 : n][s];
    };
    auto IA = [&](int n, int s) -> T {
        if constexpr (stream) return reciprocal(As[s]);
        return CL ? sh.ia[CL ? s : 0][tid + NT * n] : IAr[n][s];
    };
    auto IE = [&](int n, int s) -> T {
        if constexpr (stream) return reciprocal(E(n, s));
        else if constexpr (FP64) return IEr[n][s];
        else return Er[n][s] != T(0) ? __builtin_amdgcn_rcpf(Er[n][s]) : T(0);
    };
    auto load_ad = [&](int lo, int hi) {
        if constexpr (stream) {
#pragma unroll
            for (int s = lo; s < hi; ++s) {
                As[s] = row(s);
                Ds[s] = row(6 + s);
            }
        }
    };
    auto load_ck = [&] {
        if constexpr (stream) {
#pragma unroll
            for (int s = 0; s < 8; ++s) CKs[s] = row(18 + s);
        }
    };
    bool last[RPT];   // the folded column
#pragma unroll
    for (int n = 0; n < RPT; ++n) {
        const int t = tid + NT * n;
        const long long o = off(i0 + lx(n), j0 + ly(n), k0 + lz(n));
        last[n] = S.fold && i0 + lx(n) == g.nx;
#pragma unroll
        for (int s = 0; s < 6; ++s) {
            if constexpr (stream) {
                As[s] = row(s) = S.a[s * NP + o];
                Ds[s] = row(6 + s) = S.e[s * NP + o];
                row(12 + s) = S.x[s * NP + o];
                if (s > 0) row(17 + s) = S.c[s * NP + o];
                if (s < 3) row(23 + s) = S.K[s * NP + o];
            } else {
                const T a = S.a[s * NP + o], ia = a != T(0) ? T(1) / a : T(0);
                Ar[n][s] = a;
                Er[n][s] = FP64 ? a * S.e[s * NP + o] : S.e[s * NP + o];
                (CL ? sh.ia[CL ? s : 0][t] : IAr[n][s]) = ia;
                if constexpr (FP64) IEr[n][s] = Er[n][s] != T(0) ? T(1) / Er[n][s] : T(0);
                sh.x[s][t] = S.x[s * NP + o];
                if (s > 0) (CL ? sh.ck[CL ? s - 1 : 0][t] : CKr[n][s > 0 ? s - 1 : 0]) = S.c[s * NP + o];
                if (s < 3) (CL ? sh.ck[CL ? 5 + s : 0][t] : CKr[n][5 + s]) = S.K[s * NP + o];
            }
            const T r = S.r[s * NP + o];
            // plain residual, for iteration 0
            sh.w[s][lz(n) + 1][ly(n) + 1][lx(n) + 1] = r;
            if constexpr (hold) Pk[n][s] = r;
            R[n][s] = E(n, s) * r;
            Q[n][s] = T(0);
        }
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
    T rR[NR][6], rQ[NR][6], rP[hold ? NR : 1][6];
    // bits 0..: samples awaited, 6: by an x plane, 7: a place of the halo, 8..: its
    // index in one sample's LDS box
    unsigned ring[NR];
    int src[NR];   // word of sample 0
#pragma unroll
    for (int n = 0; n < NR; ++n) {
        const int h = tid + NT * n;
        ring[n] = 0;
        src[n] = 0;
#pragma unroll
        for (int s = 0; s < 6; ++s) rR[n][s] = rQ[n][s] = rP[hold ? n : 0][s] = T(0);
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
            const int place = ((z + 1) * B::HY + y + 1) * B::HX + x + 1;
            ring[n] = 128u | (unsigned)place << 8;
#pragma unroll
            for (int s = 0; s < 6; ++s) w0[s * box + place] = T(0);
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
                        ring[n] |= 1u << s;
                        rR[n][s] = e * S.r[s * NP + o];
                    }
                if (ring[n] & 63u) {
                    // an active sample's brick is in the list; the plane it is
                    // read from: along an axis on which it lies beyond this brick
                    const int dx = x < 0 ? -1 : x / BX, dy = y < 0 ? -1 : y / BY, dz = z < 0 ? -1 : z / BZ;
                    const int ux = x - dx * BX, uy = y - dy * BY, uz = z - dz * BZ;
                    const int who = S.rank[(bx + dx) + S.nbx * ((by + dy) + S.nby * (bz + dz))];
                    const int ax = dx ? 0 : (dy ? 1 : 2);
                    const int pl = 2 * ax + ((ax == 0 ? dx : (ax == 1 ? dy : dz)) < 0 ? 1 : 0);
                    const int at = ax == 0 ? uy + BY * uz : (ax == 1 ? ux + BX * uz : ux + BX * uy);
                    src[n] = (who * B::values + B::plane(pl) + at) * LW;
                    if (ax == 0) ring[n] |= 64u;
                    if (who < 0) ring[n] &= ~63u;
                }
            }
        }
    }
    // extra faces: kind 0..8 = (axis u, v, w) x (far plane, near planes)
    int extra[NE];   // bits 0..: kind, 4, 12, 20: place + 1; -1: none
    T eK[NE];
#pragma unroll
    for (int n = 0; n < NE; ++n) {
        int e = tid + NT * n;
        extra[n] = -1;
        eK[n] = T(0);
        constexpr int size[9] = {B::sx, B::sy, B::sz, B::sx, B::sy, B::sz, B::sx, B::sy, B::sz};
#pragma unroll
        for (int q = 0; q < 9; ++q) {
            if (extra[n] < 0 && e < size[q]) {
                const int ax = q % 3;   // the plane's axis
                const int u = ax == 0 ? e % BY : e % BX, w = ax == 0 ? e / BY : e / BX;
                const int at = ax == q / 3 ? (ax == 0 ? BX : (ax == 1 ? BY : BZ)) : -1;
                const int x = ax == 0 ? at : u, y = ax == 0 ? u : (ax == 1 ? at : w), z = ax == 2 ? at : w;
                extra[n] = q | (x + 1) << 4 | (y + 1) << 12 | (z + 1) << 20;
                eK[n] = S.K[(q / 3) * NP + off(i0 + x, j0 + y, k0 + z)];
            } else if (extra[n] < 0) {
                e -= size[q];
            }
        }
    }
    if (tid < 8 * NW) sh.part[tid >> 3][tid & 7] = 0.0;
    if (tid == 0) sh.abort = 0;
    const double tol2 = scalar(S.sc->tol2);
    const int max_iter = S.sc->max_iter;
    double bb = scalar(S.set_bb ? 0.0 : S.sc->bb);
    int* abort_flag = &S.sc->aborted;
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

    auto renew = [&] {
        if constexpr (stream || CL) {
            asm volatile("" : "+v"(tt), "+s"(mine));
#pragma unroll
            for (int n = 0; n < NE; ++n) asm volatile("" : "+v"(extra[n]));
#pragma unroll
            for (int n = 0; n < NR; ++n) asm volatile("" : "+v"(ring[n]), "+v"(src[n]));
        }
    };
    T alpha = T(0), beta = T(0);
    for (int k = 0;; ++k) {
        renew();
        if (k > 0) {
            const unsigned want = S.stamp + (unsigned)k;
            double tot[5];
            if (W > 1) {
                const LLWord* msg = S.msg + (long long)(want & 1) * W * B::values * LW;
                const LLWord* pw = S.part + (long long)(want & 1) * kRes3dMost * 16 + 2 * min(tt & 7, 4);
                LLWord* const all = S.part + (2 + (want & 1)) * (long long)kRes3dMost * 16;
                const int np = (W + PS - 1) / PS;
                double sum = 0.0;
                LLPatience wait;
                ll_first_wait(W);
                // sums of all workgroups: everyone adds them up, or the first does
                // for everyone
                LLSlot<double> ps[MP], ts;
                auto load_sums = [&] {
#pragma unroll
                    for (int m = 0; m < MP; ++m)
                        if (m < np) ps[m].load(pw + min((tt >> 3) + PS * m, W - 1) * 16);
                };
                auto add_sums = [&] {
                    bool got = true;
                    sum = 0.0;
#pragma unroll
                    for (int m = 0; m < MP; ++m)
                        if (m < np) {
                            got &= ps[m].ready(want);
                            if ((tt >> 3) + PS * m < W) sum += ps[m].value();
                        }
                    return got;
                };
                auto wave_sums = [&] {
                    sum = swap_rows32(swap_rows16(sum + dpp_perm<0x128>(sum)));   // row_ror:8
                    if ((tt & 63) < 8) sh.tot[wid][tt & 63] = sum;
                };
                if (central && me == 0) {
                    for (;;) {
                        load_sums();
                        if (__all(add_sums())) break;
                        if (wait.over(abort_flag, nullptr)) {
                            sh.abort = 1;
                            break;
                        }
                    }
                    wave_sums();
                    __syncthreads();
                    // a line for each: one line for all of them would be read in turn
                    const double t = total(sh.tot);
                    for (int e = tt >> 3; e < W && !sh.abort; e += PS)
                        if ((tt & 7) < 5) ll_put(all + e * 16 + 2 * (tt & 7), t, want);
                    __syncthreads();
                }
                for (;;) {
                    LLSlot<T> rs[NR][6];
                    if constexpr (central) {
                        if (wid == 0) ts.load(all + me * 16 + 2 * min(tt & 63, 4));
                    } else
                        load_sums();
#pragma unroll
                    for (int n = 0; n < NR; ++n)
                        if (ring[n] & 63u) {
#pragma unroll
                            for (int s = 0; s < 6; ++s) {
                                // planes across y and z are of one size
                                static_assert(B::sy == B::sz, "one step");
                                const int step = B::sx == B::sy || (ring[n] & 64u) ? B::sx : B::sy;
                                rs[n][s].load(msg + src[n] + s * step * LW);
                            }
                        }
                    bool got = central ? wid != 0 || ts.ready(want) : add_sums();
#pragma unroll
                    for (int n = 0; n < NR; ++n)
#pragma unroll
                        for (int s = 0; s < 6; ++s) {
                            const bool nd = (ring[n] >> s) & 1u;
                            got &= !nd || rs[n][s].ready(want);
                            rQ[n][s] = nd ? rs[n][s].value() : T(0);
                        }
                    if (__all(got)) break;
                    if (wait.over(abort_flag, nullptr)) {
                        sh.abort = 1;
                        break;
                    }
                }
                if constexpr (central) {
                    if (wid == 0 && (tt & 63) < 8) sh.tot[0][tt & 63] = ts.value();
                } else {
                    wave_sums();
                }
                __syncthreads();
                if (sh.abort) return;
                double t;
                if constexpr (central)
                    t = sh.tot[0][tt & 7];
                else
                    t = total(sh.tot);
#pragma unroll
                for (int q = 0; q < 5; ++q) tot[q] = lane_value(t, q);
            } else {
                const double t = total(sh.part);
#pragma unroll
                for (int q = 0; q < 5; ++q) tot[q] = lane_value(t, q);
                __syncthreads();
            }
            if (S.set_bb && k == 1) bb = scalar(tot[4]);
            const CgStep st = cg_step(tot, tol2, bb, k - 1, max_iter);
            if (st.stop) {
                if (me == 0 && tt == 0) {
                    Scalars* sc = S.sc;
                    sc->rr = tot[4];
                    sc->pq = tot[1];
                    if (S.set_bb) sc->bb = bb;
                    sc->iter = k - 1;
                    sc->done = st.stop;
                }
                break;
            }
            alpha = scalar((T)st.alpha);
            beta = scalar((T)st.beta);
        }
        const bool first = k == 0;
        renew();
        // the halo's a p_k, then the own R_k, a p_k, x_k
#pragma unroll
        for (int n = 0; n < NR; ++n)
            if (ring[n] & 128u) {
#pragma unroll
                for (int s = 0; s < 6; ++s) {
                    rR[n][s] = ll_fma(-alpha, rQ[n][s], rR[n][s]);
                    T& Pl = w0[s * box + (ring[n] >> 8)];
                    const T Pn = ll_fma(beta, hold ? rP[hold ? n : 0][s] : Pl, rR[n][s]);
                    if constexpr (hold) rP[n][s] = Pn;
                    Pl = Pn;
                }
            }
        double part[5] = {};
#pragma unroll
        for (int n = 0; n < RPT; ++n) {
            T xs[stream ? 6 : 1];
#pragma unroll
            for (int s = 0; s < 6; ++s) {
                if constexpr (stream) {   // three samples' values at a time
                    if (s == 3) __builtin_amdgcn_sched_barrier(0);
                    if (s % 3 == 0) {
                        load_ad(s, s + 3);
#pragma unroll
                        for (int u = s; u < s + 3; ++u) xs[u] = row(12 + u);
                    }
                }
                T& Pl = sh.w[s][lz(n) + 1][ly(n) + 1][lx(n) + 1];
                const T Po = hold ? Pk[hold ? n : 0][s] : Pl, ia = IA(n, s), pi = Po * ia;
                if constexpr (stream) {
                    if (!first) row(12 + s) = ll_fma(alpha, pi, xs[s]);
                } else {
                    if (!first) sh.x[s][tt + NT * n] = ll_fma(alpha, pi, sh.x[s][tt + NT * n]);
                }
                const T Rn = ll_fma(-alpha, Q[n][s], R[n][s]);
                const T rn = first ? Po : Rn * IE(n, s);
                const T zn = Rn * ia;
                const T Pn = first ? Rn : ll_fma(beta, Po, Rn);
                if constexpr (hold) Pk[n][s] = Pn;
                Pl = Pn;
                R[n][s] = Rn;
                // inactive samples hold zeros, except a plain residual that the
                // caller may have left there
                if (A(n, s) != T(0)) {
                    part[0] = ll_fma((double)rn, (double)zn, part[0]);
                    part[4] = ll_fma((double)rn, (double)rn, part[4]);
                }
            }
        }
        if (stream) __builtin_amdgcn_sched_barrier(0);
        renew();
        load_ck();
        load_ad(0, 6);
        __syncthreads();
        // faces
        renew();
        T gu[RPT], gv[RPT], gw[RPT];
#pragma unroll
        for (int n = 0; n < RPT; ++n) {
            gu[n] = CK(n, 5) * fu(lx(n), ly(n), lz(n));
            gv[n] = CK(n, 6) * fv(lx(n), ly(n), lz(n));
            gw[n] = CK(n, 7) * fw(lx(n), ly(n), lz(n));
            sh.gu[lz(n) + 1][ly(n) + 1][lx(n)] = gu[n];
            sh.gv[lz(n) + 1][ly(n)][lx(n) + 1] = gv[n];
            sh.gw[lz(n)][ly(n) + 1][lx(n) + 1] = gw[n];
        }
#pragma unroll
        for (int n = 0; n < NE; ++n) {
            const int ax = extra[n] < 0 ? -1 : (extra[n] & 15) / 3;
            const int x = (extra[n] >> 4 & 255) - 1, y = (extra[n] >> 12 & 255) - 1, z = (extra[n] >> 20) - 1;
            if (ax == 0) sh.gu[z + 1][y + 1][x] = eK[n] * fu(x, y, z);
            if (ax == 1) sh.gv[z + 1][y][x + 1] = eK[n] * fv(x, y, z);
            if (ax == 2) sh.gw[z][y + 1][x + 1] = eK[n] * fw(x, y, z);
        }
        __syncthreads();
        // A p at the own anchors
        renew();
        const unsigned stamp = S.stamp + (unsigned)k + 1u;
        LLWord* out = S.msg + ((long long)(stamp & 1) * W + me) * B::values * LW;
#pragma unroll
        for (int n = 0; n < RPT; ++n) {
            const int x = lx(n), y = ly(n), z = lz(n);
            auto Gu = [&](int dx, int dy, int dz) { return sh.gu[z + 1 + dz][y + 1 + dy][x + dx]; };
            auto Gv = [&](int dx, int dy, int dz) { return sh.gv[z + 1 + dz][y + dy][x + 1 + dx]; };
            auto Gw = [&](int dx, int dy, int dz) { return sh.gw[z + dz][y + 1 + dy][x + 1 + dx]; };
            const bool pair = S.pair != 0;
            T ia[6], p[6];
            auto point = [&](int s) {
                ia[s] = IA(n, s);
                p[s] = (hold ? Pk[hold ? n : 0][s] : wat(s, x, y, z)) * ia[s];
            };
            // a S + c p, contracted on either product
            auto form = [&](int s, T S6, bool on_a) {
                const T a = A(n, s), c = CK(n, s - 1);
                return on_a ? ll_fma(a, S6, c * p[s]) : ll_fma(c, p[s], a * S6);
            };
            auto finish = [&](int s, T y6) {
                const T dd = stream ? Ds[stream ? s : 0] : E(n, s) * ia[s], zn = R[n][s] * ia[s];
                const double yd = y6;
                part[1] = ll_fma((double)p[s], yd, part[1]);
                part[2] = ll_fma((double)zn, yd, part[2]);
                part[3] = ll_fma((double)dd * yd, yd, part[3]);
                Q[n][s] = (dd * A(n, s)) * y6;
                if (x == 0) sh.out[0][s][y + BY * z] = Q[n][s];
                if (x == BX - 1) sh.out[1][s][y + BY * z] = Q[n][s];
                if (y == 0) sh.out[2][s][x + BX * z] = Q[n][s];
                if (y == BY - 1) sh.out[3][s][x + BX * z] = Q[n][s];
                if (W > 1) {
                    if (z == 0) ll_put(out + (B::plane(4) + s * B::sz + x + BX * y) * LW, Q[n][s], stamp);
                    if (z == BZ - 1)
                        ll_put(out + (B::plane(5) + s * B::sz + x + BX * y) * LW, Q[n][s], stamp);
                }
            };
            const T gu0 = stream ? Gu(0, 0, 0) : gu[n], gv0 = stream ? Gv(0, 0, 0) : gv[n],
                    gw0 = stream ? Gw(0, 0, 0) : gw[n];
            {
                const T gu1 = Gu(1, 0, 0), gv1 = Gv(0, 1, 0), gw1 = Gw(0, 0, 1);
#pragma unroll
                for (int s = 0; s < 3; ++s) point(s);
                const T cross = T(0.5) * fmin(CK(n, 0), CK(n, 1));
                finish(0, A(n, 0) * ((gu0 - gu1) + (gv0 - gv1) + (gw0 - gw1)));
                finish(1, ll_fma(cross, p[2], form(1, (gu1 - gu0) + (gw0 - gw1), pair)));
                finish(2, ll_fma(cross, p[1], form(2, (gv1 - gv0) + (gw0 - gw1), false)));
            }
            {
                const T gum = Gu(0, -1, 0), guz = Gu(0, 0, -1), gvm = Gv(-1, 0, 0), gvz = Gv(0, 0, -1),
                        gwx = Gw(-1, 0, 0), gwy = Gw(0, -1, 0);
#pragma unroll
                for (int s = 3; s < 6; ++s) point(s);
                finish(3, form(3, (gu0 - gum) + (gv0 - gvm), pair || last[n]));
                finish(4, form(4, (gu0 - guz) + (gw0 - gwx), pair || last[n]));
                finish(5, form(5, (gv0 - gvz) + (gw0 - gwy), pair));
            }
        }
        double four, fifth;
        wave_sum5(part, four, fifth);
        if ((tt & 63) < 4) sh.part[wid][(tt & 63)] = four;
        if ((tt & 63) == 0) sh.part[wid][4] = fifth;
        __syncthreads();
        if (W > 1) {
            if (wid == 0) {
                const double t = total(sh.part);
                if ((tt & 63) < 5)
                    ll_put(S.part + ((long long)(stamp & 1) * kRes3dMost + me) * 16 + 2 * (tt & 63), t, stamp);
            }
            // x and y planes, 64 values a wave at a time
            constexpr int rx = 12 * B::sx / 64, ry = 12 * B::sy / 64;
            static_assert(B::sx % 64 == 0 && B::sy % 64 == 0, "whole waves a plane");
            for (int row = wid; row < rx + ry; row += NW) {
                const bool isx = row < rx;
                const int e = (isx ? row : row - rx) * 64 + (tt & 63), sz = isx ? B::sx : B::sy;
                const int q = e / (6 * sz), s = (e / sz) % 6, at = e % sz;
                ll_put(out + (B::plane((isx ? 0 : 2) + q) + s * sz + at) * LW, sh.out[(isx ? 0 : 2) + q][s][at],
                       stamp);
            }
        }
    }
#pragma unroll
    for (int n = 0; n < RPT; ++n) {
        const int i = i0 + lx(n), j = j0 + ly(n), k = k0 + lz(n);
        if (!inside(i, j, k)) continue;
        const long long o = g.idx(i, j, k);
#pragma unroll
        for (int s = 0; s < 6; ++s) {
            if constexpr (stream) {
                if (row(s) != T(0)) S.x[s * NP + o] = row(12 + s);
            } else {
                if (A(n, s) != T(0)) S.x[s * NP + o] = sh.x[s][tid + NT * n];
            }
        }
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

// ordered list of the flagged bricks (its first kRes3dMost), their number, and
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
        if (t < n) rank[t] = any && at < kRes3dMost ? at : -1;
        if (any && at < kRes3dMost) list[at] = t;
        base += all;
        __syncthreads();
    }
    if (threadIdx.x == 0) *count = base;
}

struct Shape {
    int bx, by, bz;
};
Shape shape_of(int shape) { return shape == 1 ? Shape{16, 8, 8} : Shape{8, 8, 8}; }

template <typename T, int BX, int BY, int BZ, int PER>
void launch_shape(const Res3dArgs<T>& S, int count, hipStream_t s) {
    hipLaunchKernelGGL((k_resident3d<T, BX, BY, BZ, PER>), dim3(count), dim3(Brick<BX, BY, BZ>::NT), 0, s, S);
}

}  // namespace

void res3d_lattice(const Geo& g, int shape, int& nbx, int& nby, int& nbz) {
    const Shape b = shape_of(shape);
    nbx = g.nx / b.bx + 1;
    nby = g.ny / b.by + 1;
    nbz = g.nz / b.bz + 1;
}

// words of the messages of the most workgroups a grid can need, both parities; FP64
// for the first shape, FP32 for the second
long long res3d_words(const Geo& g) {
    auto bricks = [&](int shape) {
        int x, y, z;
        res3d_lattice(g, shape, x, y, z);
        return std::min((long long)x * y * z, (long long)kRes3dMost);
    };
    return std::max(2 * bricks(0) * Brick<8, 8, 8>::values * 2, 2 * bricks(1) * Brick<16, 8, 8>::values);
}

// values of the streamed fields of n bricks
long long res3d_stream(int n) { return (long long)n * kResStream * Brick<8, 8, 8>::anchors; }

// whether two streaming bricks fit on a compute unit
bool res3d_two() {
    static const bool two = [] {
        int nb = 0;
        const auto k = k_resident3d<double, 8, 8, 8, 2>;
        return hipOccupancyMaxActiveBlocksPerMultiprocessor(&nb, k, Brick<8, 8, 8>::NT, 0) == hipSuccess &&
               nb >= 2;
    }();
    return two;
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
                       T* x, const T* e, const T* a, const T* c, const T* K, double* buf, LLWordBuf part,
                       LLWordBuf msg, unsigned stamp, bool set_bb, bool pair, bool fold, Scalars* sc,
                       hipStream_t s) {
    int nbx, nby, nbz;
    res3d_lattice(g, shape, nbx, nby, nbz);
    const Res3dArgs<T> S{g,   r,    x,   e,     a,              c,            K,            list, rank, nbx, nby,
                         buf,  part, msg, stamp, set_bb ? 1 : 0, pair ? 1 : 0, fold ? 1 : 0, sc};
    if (shape == 0)
        launch_shape<T, 8, 8, 8, 1>(S, count, s);
    else if constexpr (sizeof(T) == 4)
        launch_shape<T, 16, 8, 8, 1>(S, count, s);
    else
        launch_shape<T, 8, 8, 8, 2>(S, count, s);
}

template void launch_resident3d<float>(const Geo&, int, const int*, const int*, int, const float*, float*,
                                       const float*, const float*, const float*, const float*, double*,
                                       LLWordBuf, LLWordBuf, unsigned, bool, bool, bool, Scalars*, hipStream_t);
template void launch_resident3d<double>(const Geo&, int, const int*, const int*, int, const double*,
                                        double*, const double*, const double*, const double*, const double*,
                                        double*, LLWordBuf, LLWordBuf, unsigned, bool, bool, bool, Scalars*,
                                        hipStream_t);

}  // namespace vfs

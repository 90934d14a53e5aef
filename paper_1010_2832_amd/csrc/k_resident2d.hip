// 2D Jacobi-preconditioned CG as one resident kernel: a whole solve in one
// launch.
//
// The iteration is that of k_fused2d (one reduction per iteration, the next
// r.z from its expansion).  Launched once per iteration it is bound by the
// launch itself and by reading every vector back (8.2 us at 512^2 in FP32,
// 10.3 us for the FP64 pair of kernels at 300 x 212); here the vectors and
// coefficients of a tile stay in registers for the whole solve and only two
// things cross workgroups, both as stamped words (vfs_resident.h): the five
// partial sums, read by everybody, and A p at the anchors on a tile's rim.
// A workgroup keeps r and p of its halo itself, updating them by the owner's
// own expressions on the owner's A p, so both hold the same bits.
//
// A workgroup of 8 waves owns 62 x 8 RPT anchors: a wave holds RPT rows of 64
// lanes, lanes 1..62 own anchors and lanes 0 and 63 the halo columns, so
// x neighbours are a lane shift away and y neighbours mostly in the same
// thread; the rows at a wave's edge go through LDS.  The first and last wave
// also hold the halo rows.  The face rows between two waves are formed twice.
//
// What a round costs is set by the number of cache lines that are written and
// polled, so a workgroup's partial sums fill one line of their own and the rim
// goes out as one packed message per side (the columns are gathered in LDS
// first): with the rim scattered over the grid and the sums of one kind side
// by side, a round of 202 workgroups took 6 us instead of 2.5.
#include "vfs_internal.h"
#include "vfs_resident.h"

#include <algorithm>

namespace vfs {
namespace {

constexpr int NW = 8, NT = 64 * NW;
constexpr int BX = 62;

template <typename T>
struct Res2dArgs {
    Geo g;
    const T* r;      // residual the solve starts from (kept)
    T* x;            // iterate, updated at the end
    const T* dinv;
    const T* a;
    const T* c;
    const T* K;
    const int* tiles;
    int ntx;         // tiles per row of the tile lattice
    LLWord* part;    // [2][workgroups][16]: five sums, a line per workgroup
    LLWord* msg;     // [2][tiles of the lattice][message]
    long long slot;  // words from one parity's messages to the other's
    unsigned stamp;  // stamps of this solve start here
    int set_bb;
    Scalars* sc;
};

// A thread's share of a tile.  With RPT rows of 4 (FP64) or 8 (FP32) x would
// not fit in 256 registers beside the rest and lives in LDS.
template <typename T, int RPT>
struct Res2dState {
    T R[RPT][3], P[RPT][3], Q[RPT][3];
    T D[RPT][3], A[RPT][3], C[RPT][2], Ku[RPT], Kv[RPT];
    T Kum, Kvp;               // u faces of the row below, v faces of the row above
    T rR[3], rP[3], rQ[3], rD[3], rA[3];   // halo row (first and last wave)
};

// A tile's message: its first and last row (64 lanes, [sample][lane]), then its
// first and last own column ([sample][row]).
template <int RPT>
struct Msg {
    static constexpr int kRows = NW * RPT;
    static constexpr int row(int side) { return side * 3 * 64; }
    static constexpr int col(int side) { return 2 * 3 * 64 + side * 3 * kRows; }
    static constexpr int values = 2 * 3 * 64 + 2 * 3 * kRows;
};

template <typename T, int RPT>
__global__ __launch_bounds__(NT, 1) void k_resident2d(Res2dArgs<T> S) {
#pragma clang fp contract(off)
    // Every rounding is spelled out, as k_fused2d has them: both forms then give
    // the same iterates (their FP64 sums differ in order alone, which the
    // rounding of alpha and beta to FP32 hides).
    constexpr int LW = kLLWords<T>;
    constexpr bool XLDS = RPT * sizeof(T) >= 32;
    using M = Msg<RPT>;
    constexpr int NC = 3 * M::kRows, CL = (NC + 63) / 64;   // values of a column message
    __shared__ T sX[XLDS ? RPT : 1][3][XLDS ? NT : 1];
    T X[XLDS ? 1 : RPT][3];
    __shared__ T sLo[NW + 1][3][64];   // a p of a wave's first row; [NW]: halo row above
    __shared__ T sHi[NW + 1][3][64];   // a p of a wave's last row at [wave + 1]; [0]: below
    __shared__ T sIn[2][NC], sOut[2][NC];   // A p of the halo columns, of the own outer columns
    __shared__ double sTot[NW][8], sPart[NW][8];   // five sums a wave
    __shared__ int sAbort;
    const Geo& g = S.g;
    const long long NP = g.NP;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wid = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int W = gridDim.x, me = blockIdx.x;
    const int tile = S.tiles[me];
    const int tx = tile % S.ntx, ty = tile / S.ntx;
    const int i = tx * BX - 1 + lane;
    const int j0 = ty * (NW * RPT), jw = j0 + wid * RPT;
    const bool icol = i >= 0 && i <= g.nx;
    const bool mine = lane >= 1 && lane <= BX && icol;   // this lane owns its anchors
    const bool ring = wid == 0 || wid == NW - 1;
    const int jr = wid == 0 ? j0 - 1 : j0 + NW * RPT;
    const bool rin = ring && icol && jr >= 0 && jr <= g.ny;
    // samples outside the grid read offset 0, the zero pad of every slice
    auto off = [&](int j) { return icol && j >= 0 && j <= g.ny ? g.idx(i, j) : 0LL; };

    Res2dState<T, RPT> v;
#pragma unroll
    for (int q = 0; q < RPT; ++q) {
        const long long o = off(jw + q);
#pragma unroll
        for (int s = 0; s < 3; ++s) {
            v.R[q][s] = S.r[s * NP + o];
            v.D[q][s] = S.dinv[s * NP + o];
            v.A[q][s] = S.a[s * NP + o];
            const T x = S.x[s * NP + o];
            if constexpr (XLDS)
                sX[q][s][tid] = x;
            else
                X[q][s] = x;
            v.P[q][s] = v.Q[q][s] = T(0);
        }
        v.C[q][0] = S.c[NP + o];
        v.C[q][1] = S.c[2 * NP + o];
        v.Ku[q] = S.K[o];
        v.Kv[q] = S.K[NP + o];
    }
    v.Kum = S.K[off(jw - 1)];
    v.Kvp = S.K[NP + off(jw + RPT)];
    const long long ro = rin ? g.idx(i, jr) : 0LL;
#pragma unroll
    for (int s = 0; s < 3; ++s) {
        v.rR[s] = S.r[s * NP + ro];
        v.rD[s] = S.dinv[s * NP + ro];
        v.rA[s] = S.a[s * NP + ro];
        v.rP[s] = v.rQ[s] = T(0);
    }
    // messages: a halo value is awaited where its sample is active (then its
    // tile is in the list and publishes it); the others stay 0.  Tiles next to
    // the lattice's border wrap to some tile's message, which is not awaited.
    constexpr long long MW = (long long)M::values * LW;
    const long long mine_at = (long long)tile * MW;
    // halo row: lanes 1..62 from the tile below (above), lanes 0 and 63 from
    // the diagonal ones, whose lane 62 (1) that column is
    long long row_at = 0;
    if (rin) {
        const int ttx = lane == 0 ? tx - 1 : (lane == 63 ? tx + 1 : tx);
        const int src = lane == 0 ? BX : (lane == 63 ? 1 : lane);
        row_at = ((long long)(ttx + S.ntx * (wid == 0 ? ty - 1 : ty + 1)) * M::values +
                  M::row(wid == 0 ? 1 : 0) + src) * LW;
    }
    // halo columns: wave 1 polls the left one, wave 2 the right one
    const bool cols = wid == 1 || wid == 2;
    const int cside = wid - 1;
    long long col_at = 0;
    bool cneed[CL];
#pragma unroll
    for (int m = 0; m < CL; ++m) cneed[m] = false;
    if (cols) {
        const int ic = cside == 0 ? tx * BX - 1 : tx * BX + BX;
        if (ic >= 0 && ic <= g.nx) {
            col_at = ((long long)(tile + (cside == 0 ? -1 : 1)) * M::values + M::col(1 - cside)) * LW;
#pragma unroll
            for (int m = 0; m < CL; ++m) {
                const int e = lane + 64 * m, s = e / M::kRows, j = j0 + e % M::kRows;
                cneed[m] = e < NC && j <= g.ny && S.a[(e < NC ? s : 0) * NP + (j <= g.ny ? g.idx(ic, j) : 0)] != T(0);
            }
        }
    }
    for (int e = tid; e < 2 * NC; e += NT) sIn[e / NC][e % NC] = T(0);
    const double tol2 = S.sc->tol2;
    const int max_iter = S.sc->max_iter;
    double bb = S.set_bb ? 0.0 : S.sc->bb;
    int* abort_flag = &S.sc->aborted;
    if (tid == 0) sAbort = 0;
    if (tid < 8 * NW) sPart[tid >> 3][tid & 7] = 0.0;

    T alpha = T(0), beta = T(0);
    for (int k = 0;; ++k) {
        if (k > 0) {
            double tot[5];
            if (W > 1) {
                // A p of the halo and the partial sums of iteration k - 1; the
                // words of all of them are in flight together
                const unsigned want = S.stamp + (unsigned)k;
                const LLWord* msg = S.msg + ((k - 1) & 1) * S.slot;
                // thread t reads sum t % 8 of workgroups t / 8 + 64 m
                const LLWord* pw = S.part + ((long long)((k - 1) & 1) * kResMost) * 16 + 2 * min(tid & 7, 4);
                const int np = (W + 63) >> 6;
                double sum = 0.0;
                LLPatience wait;
                ll_first_wait(W);
                for (;;) {
                    LLSlot<double> ps[kResMost / 64];
                    LLSlot<T> rs[3], cs[CL];
#pragma unroll
                    for (int m = 0; m < kResMost / 64; ++m)
                        if (m < np) ps[m].load(pw + min((tid >> 3) + 64 * m, W - 1) * 16);
                    if (ring) {
#pragma unroll
                        for (int s = 0; s < 3; ++s) rs[s].load(msg + row_at + s * 64 * LW);
                    }
                    if (cols) {
#pragma unroll
                        for (int m = 0; m < CL; ++m)
                            cs[m].load(msg + col_at + min(lane + 64 * m, NC - 1) * LW);
                    }
                    bool got = true;
                    sum = 0.0;
#pragma unroll
                    for (int m = 0; m < kResMost / 64; ++m)
                        if (m < np) {
                            got &= ps[m].ready(want);
                            if ((tid >> 3) + 64 * m < W) sum += ps[m].value();
                        }
                    if (ring) {
#pragma unroll
                        for (int s = 0; s < 3; ++s) {
                            const bool need = v.rA[s] != T(0);
                            got &= !need || rs[s].ready(want);
                            v.rQ[s] = need ? rs[s].value() : T(0);
                        }
                    }
                    if (cols) {
#pragma unroll
                        for (int m = 0; m < CL; ++m) {
                            got &= !cneed[m] || cs[m].ready(want);
                            if (cneed[m]) sIn[cside][lane + 64 * m] = cs[m].value();
                        }
                    }
                    if (__all(got)) break;
                    if (wait.over(abort_flag)) {
                        sAbort = 1;
                        break;
                    }
                }
                // lanes of one sum are 8 apart
                sum = swap_rows32(swap_rows16(sum + dpp_perm<0x128>(sum)));   // row_ror:8
                if (lane < 8) sTot[wid][lane] = sum;
                __syncthreads();
                if (sAbort) return;
                const double t = waves_total8(sTot);
#pragma unroll
                for (int q = 0; q < 5; ++q) tot[q] = lane_value(t, q);
                if (lane == 0 || lane == 63) {
#pragma unroll
                    for (int q = 0; q < RPT; ++q)
#pragma unroll
                        for (int s = 0; s < 3; ++s)
                            v.Q[q][s] = sIn[lane == 0 ? 0 : 1][s * M::kRows + wid * RPT + q];
                }
            } else {
                const double t = waves_total8(sPart);
#pragma unroll
                for (int q = 0; q < 5; ++q) tot[q] = lane_value(t, q);
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

        // r_k, z_k, p_k, x_k and a p_k (iteration 0: p = z, alpha = beta = 0)
        double part[5] = {};
#pragma unroll
        for (int q = 0; q < RPT; ++q) {
#pragma unroll
            for (int s = 0; s < 3; ++s) {
                if constexpr (XLDS)
                    sX[q][s][tid] = ll_fma(alpha, v.P[q][s], sX[q][s][tid]);
                else
                    X[q][s] = ll_fma(alpha, v.P[q][s], X[q][s]);
                T zn;
                cg_advance(v.R[q][s], v.P[q][s], zn, v.Q[q][s], v.D[q][s], alpha, beta);
                const T rn = v.R[q][s];
                if (mine) {
                    part[0] = ll_fma((double)rn, (double)zn, part[0]);
                    part[4] = ll_fma((double)rn, (double)rn, part[4]);
                }
            }
        }
#pragma unroll
        for (int s = 0; s < 3; ++s) {
            sLo[wid][s][lane] = v.A[0][s] * v.P[0][s];
            sHi[wid + 1][s][lane] = v.A[RPT - 1][s] * v.P[RPT - 1][s];
        }
        if (ring) {
#pragma unroll
            for (int s = 0; s < 3; ++s) {
                T zn;
                cg_advance(v.rR[s], v.rP[s], zn, v.rQ[s], v.rD[s], alpha, beta);
                T* dst = wid == 0 ? &sHi[0][s][lane] : &sLo[NW][s][lane];
                *dst = v.rA[s] * v.rP[s];
            }
        }
        __syncthreads();

        // faces row by row, A p at the own anchors; a tile's outer rows are
        // published at once, its outer columns gathered in LDS
        const unsigned stamp = S.stamp + (unsigned)k + 1u;
        LLWord* out = S.msg + (k & 1) * S.slot + mine_at;
        T below[3], up[3];
#pragma unroll
        for (int s = 0; s < 3; ++s) {
            below[s] = sHi[wid][s][lane];
            up[s] = sLo[wid + 1][s][lane];
        }
        T w[3], wn[3];   // a p of the row and of the next one
#pragma unroll
        for (int s = 0; s < 3; ++s) w[s] = v.A[0][s] * v.P[0][s];
        T gum = v.Kum * ((below[0] - lane_left(below[0])) + (lane_left(below[1]) - below[1]) +
                         (below[2] - w[2]));
        T gv = v.Kv[0] * ((w[0] - below[0]) + (w[1] - below[1]) + (w[2] - lane_right(w[2])));
#pragma unroll
        for (int q = 0; q < RPT; ++q) {
            constexpr int last = RPT - 1;
            const int qn = q < last ? q + 1 : last;
#pragma unroll
            for (int s = 0; s < 3; ++s) wn[s] = q < last ? v.A[qn][s] * v.P[qn][s] : up[s];
            const T kv = q < last ? v.Kv[qn] : v.Kvp;
            const T gu = v.Ku[q] * ((w[0] - lane_left(w[0])) + (lane_left(w[1]) - w[1]) +
                                    (w[2] - wn[2]));
            const T gvn = kv * ((wn[0] - w[0]) + (wn[1] - w[1]) + (wn[2] - lane_right(wn[2])));
            const T gu1 = lane_right(gu), gvl = lane_left(gv);
            T y[3];
            y[0] = v.A[q][0] * ((gu - gu1) + (gv - gvn));
            y[1] = ll_fma(v.A[q][1], (gu1 - gu) + (gv - gvn), v.C[q][0] * v.P[q][1]);
            y[2] = ll_fma(v.A[q][2], (gu - gum) + (gv - gvl), v.C[q][1] * v.P[q][2]);
            if (mine) {
#pragma unroll
                for (int s = 0; s < 3; ++s) {
                    const double yd = y[s];
                    const T zn = v.D[q][s] * v.R[q][s];
                    part[1] = ll_fma((double)v.P[q][s], yd, part[1]);
                    part[2] = ll_fma((double)zn, yd, part[2]);
                    part[3] = ll_fma((double)v.D[q][s] * yd, yd, part[3]);
                }
            }
            if (W > 1) {
                if ((q == 0 && wid == 0) || (q == last && wid == NW - 1)) {
#pragma unroll
                    for (int s = 0; s < 3; ++s)
                        ll_put(out + (M::row(wid == 0 ? 0 : 1) + s * 64 + lane) * LW, y[s], stamp);
                }
                if (lane == 1 || lane == BX) {
#pragma unroll
                    for (int s = 0; s < 3; ++s)
                        sOut[lane == 1 ? 0 : 1][s * M::kRows + wid * RPT + q] = y[s];
                }
            }
#pragma unroll
            for (int s = 0; s < 3; ++s) {
                v.Q[q][s] = mine ? y[s] : T(0);
                w[s] = wn[s];
            }
            gum = gu;
            gv = gvn;
        }
        double four, fifth;
        wave_sum5(part, four, fifth);
        if (lane < 4) sPart[wid][lane] = four;
        if (lane == 0) sPart[wid][4] = fifth;
        __syncthreads();
        if (W > 1) {
            if (wid == 0) {
                const double t = waves_total8(sPart);
                if (lane < 5)
                    ll_put(S.part + ((long long)(k & 1) * kResMost + me) * 16 + 2 * lane, t,
                           stamp);
            }
            if (cols) {
#pragma unroll
                for (int m = 0; m < CL; ++m) {
                    const int e = lane + 64 * m;
                    if (e < NC) ll_put(out + (M::col(cside) + e) * LW, sOut[cside][e], stamp);
                }
            }
        }
    }
#pragma unroll
    for (int q = 0; q < RPT; ++q) {
        const int j = jw + q;
        if (mine && j <= g.ny) {
#pragma unroll
            for (int s = 0; s < 3; ++s) {
                if constexpr (XLDS)
                    S.x[s * NP + g.idx(i, j)] = sX[q][s][tid];
                else
                    S.x[s * NP + g.idx(i, j)] = X[q][s];
            }
        }
    }
}

// flag of every 62 x 8 strip of the tile lattice: some sample has a != 0
__global__ __launch_bounds__(512) void k_res2d_flags(Geo g, int ntx, const double* __restrict__ a,
                                                     int* __restrict__ flags) {
    const int t = blockIdx.x;
    const int i = (t % ntx) * BX + (threadIdx.x & 63), j = (t / ntx) * NW + (threadIdx.x >> 6);
    int any = 0;
    if ((threadIdx.x & 63) < BX && i <= g.nx && j <= g.ny)
        for (int s = 0; s < 3; ++s) any |= a[s * g.NP + g.idx(i, j)] != 0.0;
    any = __syncthreads_or(any);
    if (threadIdx.x == 0) flags[t] = any;
}

// ordered tile lists for RPT = 1, 2, 4, 8 (list b of workgroup b): a tile of
// RPT strips is listed if one of them is flagged
__global__ __launch_bounds__(1024) void k_res2d_lists(int ntx, int nty, const int* __restrict__ flags,
                                                      int* __restrict__ lists, int cap,
                                                      int* __restrict__ counts) {
    const int rpt = 1 << blockIdx.x;
    const int rows = (nty + rpt - 1) / rpt, n = ntx * rows;
    int* list = lists + (long long)blockIdx.x * cap;
    __shared__ int sCnt[16];
    const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
    int base = 0;
    for (int t0 = 0; t0 < n; t0 += 1024) {
        const int t = t0 + threadIdx.x;
        int any = 0;
        if (t < n) {
            const int tx = t % ntx, ty = t / ntx;
            for (int q = 0; q < rpt && ty * rpt + q < nty; ++q) any |= flags[tx + ntx * (ty * rpt + q)];
        }
        const unsigned long long m = __ballot(any);
        if (lane == 0) sCnt[wid] = __popcll(m);
        __syncthreads();
        int before = base, all = 0;
        for (int w = 0; w < 16; ++w) {
            if (w < wid) before += sCnt[w];
            all += sCnt[w];
        }
        const int at = before + __popcll(m & ((1ull << lane) - 1ull));
        if (any && at < cap) list[at] = t;
        base += all;
        __syncthreads();
    }
    if (threadIdx.x == 0) counts[blockIdx.x] = base;
}

template <typename T, int RPT>
void launch_rpt(const Res2dArgs<T>& S, int count, hipStream_t s) {
    hipLaunchKernelGGL((k_resident2d<T, RPT>), dim3(count), dim3(NT), 0, s, S);
}

}  // namespace

void res2d_lattice(const Geo& g, int& ntx, int& nty) {
    ntx = (g.nx + 1 + BX - 1) / BX;
    nty = (g.ny + 1 + NW - 1) / NW;
}

// words of the messages of one shape's lattice, both parities, FP64
long long res2d_words(const Geo& g, int shape) {
    int ntx, nty;
    res2d_lattice(g, ntx, nty);
    const int rpt = 1 << shape;
    return 2LL * 2 * ntx * ((nty + rpt - 1) / rpt) * (2 * 3 * 64 + 2 * 3 * NW * rpt);
}

void launch_res2d_lists(const Geo& g, const double* a, int* flags, int* lists, int cap, int* counts,
                        hipStream_t s) {
    int ntx, nty;
    res2d_lattice(g, ntx, nty);
    hipLaunchKernelGGL(k_res2d_flags, dim3(ntx * nty), dim3(512), 0, s, g, ntx, a, flags);
    hipLaunchKernelGGL(k_res2d_lists, dim3(kResShapes), dim3(1024), 0, s, ntx, nty, flags, lists,
                       cap, counts);
}

template <typename T>
void launch_resident2d(const Geo& g, int shape, const int* tiles, int count, const T* r, T* x,
                       const T* dinv, const T* a, const T* c, const T* K, LLWordBuf part,
                       LLWordBuf msg, unsigned stamp, bool set_bb, Scalars* sc, hipStream_t s) {
    int ntx, nty;
    res2d_lattice(g, ntx, nty);
    const long long slot = res2d_words(g, shape) / 4 * kLLWords<T>;
    const Res2dArgs<T> S{g,    r,   x,    dinv,  a,              c, K, tiles, ntx,
                         part, msg, slot, stamp, set_bb ? 1 : 0, sc};
    if (shape == 0) launch_rpt<T, 1>(S, count, s);
    else if (shape == 1) launch_rpt<T, 2>(S, count, s);
    else if (shape == 2) launch_rpt<T, 4>(S, count, s);
    else if constexpr (sizeof(T) == 4) launch_rpt<T, 8>(S, count, s);
}

template void launch_resident2d<float>(const Geo&, int, const int*, int, const float*, float*,
                                       const float*, const float*, const float*, const float*,
                                       LLWordBuf, LLWordBuf, unsigned, bool, Scalars*, hipStream_t);
template void launch_resident2d<double>(const Geo&, int, const int*, int, const double*, double*,
                                        const double*, const double*, const double*, const double*,
                                        LLWordBuf, LLWordBuf, unsigned, bool, Scalars*, hipStream_t);

}  // namespace vfs

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
// Where an iteration's time goes (300^2, 104 workgroups, FP32, 3.0 us): 0.3 us
// update, 0.5 faces and A p, 0.5 sums of the workgroup, 1.0 until the others'
// words are there, 0.6 totals and scalars.
//
// What a round costs is set by the number of cache lines that are written and
// polled, so a workgroup's partial sums fill one line of their own and the rim
// goes out as one packed message per side (the columns are gathered in LDS
// first): with the rim scattered over the grid and the sums of one kind side
// by side, a round of 202 workgroups took 6 us instead of 2.5.
#include "vfs_batch.h"
#include "vfs_internal.h"
#include "vfs_resident.h"

#include <algorithm>

namespace vfs {
namespace {

constexpr int NW = 8, NT = 64 * NW;
constexpr int BX = 62;

// A tile's message: its first and last row (64 lanes, [sample][lane]), then its
// first and last own column ([sample][row]).
template <int RPT>
struct Msg {
    static constexpr int kRows = NW * RPT;
    __host__ __device__ static constexpr int row(int side) { return side * 3 * 64; }
    __host__ __device__ static constexpr int col(int side) { return 2 * 3 * 64 + side * 3 * kRows; }
    static constexpr int values = 2 * 3 * 64 + 2 * 3 * kRows;
};

// Where the workgroups of one solve meet.
struct Meeting {
    LLWord* part;      // [2][kResMost][16]: five sums, a line per workgroup
    LLWord* msg;       // [2][tiles of the lattice][message]
    long long slot;    // words from one parity's messages to the other's
    int W, me;         // workgroups of this solve, and this one's number
    int* abort_flag;
    const unsigned* beat;   // moves while an earlier solve of these workgroups goes on
};

template <typename T, int RPT>
struct Res2dLds {
    static constexpr bool XLDS = RPT * sizeof(T) >= 16;
    static constexpr int NC = 3 * NW * RPT;
    T x[XLDS ? RPT : 1][3][XLDS ? NT : 1];
    T lo[NW + 1][3][64];      // a p of a wave's first row; [NW]: halo row above
    T hi[NW + 1][3][64];      // a p of a wave's last row at [wave + 1]; [0]: below
    T in[2][NC], out[2][NC];  // halo columns received, own outer columns to send
    double tot[NW][8], part[NW][8];   // five sums a wave
    int abort;
};

// One workgroup's tile: its place, a thread's share of its state and the
// traffic with the other workgroups.  With RPT rows of 2 (FP64) or 4 (FP32) and
// more, x lives in LDS: 256 registers would not hold it beside the rest (64 2D
// problems with 62 x 32 anchors a workgroup: 291 ms with x in registers, 261).
//
// WT: the vectors are kept weighted as in the batched iteration (R = e r, P = a
// p, Q = e A p with e = a D^-1; r, z and p come from 1 / e and 1 / a), so that
// a batch gives the same iterates resident and not.
template <typename T, int RPT, bool WT = false>
struct Res2d {
    static constexpr int LW = kLLWords<T>;
    using M = Msg<RPT>;
    using Lds = Res2dLds<T, RPT>;
    static constexpr int NC = Lds::NC, CL = (NC + 63) / 64;   // values of a column message

    // state: own rows, halo columns (lanes 0 and 63), halo row (first, last wave)
    T R[RPT][3], P[RPT][3], Q[RPT][3], X[Lds::XLDS ? 1 : RPT][3];
    T D[RPT][3], A[RPT][3], C[RPT][2], Ku[RPT], Kv[RPT];   // WT: D holds e
    T IA[WT ? RPT : 1][3];    // WT: 1 / a (0 where a = 0)
    T Kum, Kvp;               // u faces of the row below, v faces of the row above
    T rR[3], rP[3], rQ[3], rD[3], rA[3];
    // place
    int tid, lane, wid, tile, tx, ty, i, j0, jw, jr;
    bool icol, mine, ring, rin, cols;
    int cside;
    long long ro, mine_at, row_at, col_at;
    bool cneed[CL];

    __device__ __forceinline__ void place(const Geo& g, int tile_, int ntx) {
        tid = threadIdx.x;
        lane = tid & 63;
        wid = __builtin_amdgcn_readfirstlane(tid >> 6);
        tile = tile_;
        tx = tile % ntx;
        ty = tile / ntx;
        i = tx * BX - 1 + lane;
        j0 = ty * (NW * RPT);
        jw = j0 + wid * RPT;
        icol = i >= 0 && i <= g.nx;
        mine = lane >= 1 && lane <= BX && icol;   // this lane owns its anchors
        ring = wid == 0 || wid == NW - 1;
        jr = wid == 0 ? j0 - 1 : j0 + NW * RPT;
        rin = ring && icol && jr >= 0 && jr <= g.ny;
        ro = rin ? g.idx(i, jr) : 0LL;
    }
    // samples outside the grid read offset 0, the zero pad of every slice
    __device__ __forceinline__ long long off(const Geo& g, int j) const {
        return icol && j >= 0 && j <= g.ny ? g.idx(i, j) : 0LL;
    }

    // coefficients, and where this tile's messages come from: a halo value is
    // awaited where its sample is active (then its tile is in the list and
    // publishes it); the others stay 0
    __device__ __forceinline__ void load(const Geo& g, int ntx, const T* __restrict__ dinv,
                                         const T* __restrict__ a, const T* __restrict__ c,
                                         const T* __restrict__ K, Lds& sh) {
        const long long NP = g.NP;
#pragma unroll
        for (int q = 0; q < RPT; ++q) {
            const long long o = off(g, jw + q);
#pragma unroll
            for (int s = 0; s < 3; ++s) {
                D[q][s] = dinv[s * NP + o];
                A[q][s] = a[s * NP + o];
                if constexpr (WT) IA[q][s] = A[q][s] != T(0) ? T(1) / A[q][s] : T(0);
            }
            C[q][0] = c[NP + o];
            C[q][1] = c[2 * NP + o];
            Ku[q] = K[o];
            Kv[q] = K[NP + o];
        }
        Kum = K[off(g, jw - 1)];
        Kvp = K[NP + off(g, jw + RPT)];
#pragma unroll
        for (int s = 0; s < 3; ++s) {
            rD[s] = dinv[s * NP + ro];
            rA[s] = a[s * NP + ro];
        }
        mine_at = (long long)tile * M::values * LW;
        // halo row: lanes 1..62 from the tile below (above), lanes 0 and 63
        // from the diagonal ones, whose lane 62 (1) that column is
        row_at = 0;
        if (rin) {
            const int ttx = lane == 0 ? tx - 1 : (lane == 63 ? tx + 1 : tx);
            const int src = lane == 0 ? BX : (lane == 63 ? 1 : lane);
            row_at = ((long long)(ttx + ntx * (wid == 0 ? ty - 1 : ty + 1)) * M::values +
                      M::row(wid == 0 ? 1 : 0) + src) * LW;
        }
        // halo columns: wave 1 polls the left one, wave 2 the right one
        cols = wid == 1 || wid == 2;
        cside = wid - 1;
        col_at = 0;
#pragma unroll
        for (int m = 0; m < CL; ++m) cneed[m] = false;
        if (cols) {
            const int ic = cside == 0 ? tx * BX - 1 : tx * BX + BX;
            if (ic >= 0 && ic <= g.nx) {
                col_at = ((long long)(tile + (cside == 0 ? -1 : 1)) * M::values + M::col(1 - cside)) * LW;
#pragma unroll
                for (int m = 0; m < CL; ++m) {
                    const int e = lane + 64 * m, s = e < NC ? e / M::kRows : 0, j = j0 + e % M::kRows;
                    cneed[m] = e < NC && j <= g.ny && a[s * NP + (j <= g.ny ? g.idx(ic, j) : 0)] != T(0);
                }
            }
        }
        for (int e = tid; e < 2 * NC; e += NT) sh.in[e / NC][e % NC] = T(0);
        if (tid < 8 * NW) sh.part[tid >> 3][tid & 7] = 0.0;
        if (tid == 0) sh.abort = 0;
    }

    // Sends the outer rows' values of row q (y) at once, puts the outer columns'
    // into LDS for finish_round.
    __device__ __forceinline__ void send_row(const Meeting& mt, Lds& sh, int q, const T (&y)[3],
                                             unsigned stamp) const {
        constexpr int last = RPT - 1;
        LLWord* out = mt.msg + (stamp & 1) * mt.slot + mine_at;
        if ((q == 0 && wid == 0) || (q == last && wid == NW - 1)) {
#pragma unroll
            for (int s = 0; s < 3; ++s)
                ll_put(out + (M::row(wid == 0 ? 0 : 1) + s * 64 + lane) * LW, y[s], stamp);
        }
        if (lane == 1 || lane == BX) {
#pragma unroll
            for (int s = 0; s < 3; ++s) sh.out[lane == 1 ? 0 : 1][s * M::kRows + wid * RPT + q] = y[s];
        }
    }

    // Ends a round: the workgroup's sums and outer columns go out.  Contains a
    // barrier; every thread of the workgroup calls it.
    __device__ __forceinline__ void finish_round(const Meeting& mt, Lds& sh, const double (&part)[5],
                                                 unsigned stamp) const {
        double four, fifth;
        wave_sum5(part, four, fifth);
        if (lane < 4) sh.part[wid][lane] = four;
        if (lane == 0) sh.part[wid][4] = fifth;
        __syncthreads();
        if (mt.W > 1) {
            if (wid == 0) {
                const double t = waves_total8(sh.part);
                if (lane < 5)
                    ll_put(mt.part + ((long long)(stamp & 1) * kResMost + mt.me) * 16 + 2 * lane, t, stamp);
            }
            if (cols) {
                LLWord* out = mt.msg + (stamp & 1) * mt.slot + mine_at;
#pragma unroll
                for (int m = 0; m < CL; ++m) {
                    const int e = lane + 64 * m;
                    if (e < NC) ll_put(out + (M::col(cside) + e) * LW, sh.out[cside][e], stamp);
                }
            }
        }
    }

    // The totals of round `want`, and its halo values in Q (halo columns) and rQ
    // (halo row); the words of all of them are in flight together.  False when
    // the solve was given up.
    __device__ __forceinline__ bool collect(const Meeting& mt, Lds& sh, unsigned want, double (&tot)[5]) {
        if (mt.W == 1) {
            const double t = waves_total8(sh.part);
#pragma unroll
            for (int q = 0; q < 5; ++q) tot[q] = lane_value(t, q);
            __syncthreads();   // before the next round's sums take the place
            return true;
        }
        const LLWord* msg = mt.msg + (want & 1) * mt.slot;
        // thread t reads sum t % 8 of workgroups t / 8 + 64 m
        const LLWord* pw = mt.part + (long long)(want & 1) * kResMost * 16 + 2 * min(tid & 7, 4);
        const int np = (mt.W + 63) >> 6;
        double sum = 0.0;
        LLPatience wait;
        ll_first_wait(mt.W);
        for (;;) {
            LLSlot<double> ps[kResMost / 64];
            LLSlot<T> rs[3], cs[CL];
#pragma unroll
            for (int m = 0; m < kResMost / 64; ++m)
                if (m < np) ps[m].load(pw + min((tid >> 3) + 64 * m, mt.W - 1) * 16);
            if (ring) {
#pragma unroll
                for (int s = 0; s < 3; ++s) rs[s].load(msg + row_at + s * 64 * LW);
            }
            if (cols) {
#pragma unroll
                for (int m = 0; m < CL; ++m) cs[m].load(msg + col_at + min(lane + 64 * m, NC - 1) * LW);
            }
            bool got = true;
            sum = 0.0;
#pragma unroll
            for (int m = 0; m < kResMost / 64; ++m)
                if (m < np) {
                    got &= ps[m].ready(want);
                    if ((tid >> 3) + 64 * m < mt.W) sum += ps[m].value();
                }
            if (ring) {
#pragma unroll
                for (int s = 0; s < 3; ++s) {
                    const bool need = rA[s] != T(0);
                    got &= !need || rs[s].ready(want);
                    rQ[s] = need ? rs[s].value() : T(0);
                }
            }
            if (cols) {
#pragma unroll
                for (int m = 0; m < CL; ++m) {
                    got &= !cneed[m] || cs[m].ready(want);
                    if (cneed[m]) sh.in[cside][lane + 64 * m] = cs[m].value();
                }
            }
            if (__all(got)) break;
            if (wait.over(mt.abort_flag, mt.beat)) {
                sh.abort = 1;
                break;
            }
        }
        // lanes of one sum are 8 apart
        sum = swap_rows32(swap_rows16(sum + dpp_perm<0x128>(sum)));   // row_ror:8
        if (lane < 8) sh.tot[wid][lane] = sum;
        __syncthreads();
        if (sh.abort) return false;
        const double t = waves_total8(sh.tot);
#pragma unroll
        for (int q = 0; q < 5; ++q) tot[q] = lane_value(t, q);
        if (lane == 0 || lane == 63) {
#pragma unroll
            for (int q = 0; q < RPT; ++q)
#pragma unroll
                for (int s = 0; s < 3; ++s) Q[q][s] = sh.in[lane == 0 ? 0 : 1][s * M::kRows + wid * RPT + q];
        }
        return true;
    }

    // r_k, z_k, p_k, x_k, then A p_k (into Q) and the sums of iteration k; round
    // `stamp` is sent.  Every rounding is spelled out, as k_fused2d has them:
    // both forms then give the same iterates (their FP64 sums differ in order
    // alone, which the rounding of alpha and beta to FP32 hides).
    // `first`: iteration 0, where P holds the plain residual (WT).
    __device__ __forceinline__ void iterate(const Meeting& mt, Lds& sh, T alpha, T beta, unsigned stamp,
                                            bool first = false) {
#pragma clang fp contract(off)
        double part[5] = {};
#pragma unroll
        for (int q = 0; q < RPT; ++q) {
#pragma unroll
            for (int s = 0; s < 3; ++s) {
                T rn, zn;
                if constexpr (WT) {
                    const T pi = P[q][s] * IA[q][s];   // p of the last iteration
                    if constexpr (Lds::XLDS)
                        sh.x[q][s][tid] = ll_fma(alpha, pi, sh.x[q][s][tid]);
                    else
                        X[q][s] = ll_fma(alpha, pi, X[q][s]);
                    const T Rn = ll_fma(-alpha, Q[q][s], R[q][s]);
                    const T ie = D[q][s] != T(0) ? __builtin_amdgcn_rcpf(D[q][s]) : T(0);
                    rn = first ? P[q][s] : Rn * ie;
                    zn = Rn * IA[q][s];
                    P[q][s] = first ? Rn : ll_fma(beta, P[q][s], Rn);
                    R[q][s] = Rn;
                } else {
                    if constexpr (Lds::XLDS)
                        sh.x[q][s][tid] = ll_fma(alpha, P[q][s], sh.x[q][s][tid]);
                    else
                        X[q][s] = ll_fma(alpha, P[q][s], X[q][s]);
                    cg_advance(R[q][s], P[q][s], zn, Q[q][s], D[q][s], alpha, beta);
                    rn = R[q][s];
                }
                if (mine) {
                    part[0] = ll_fma((double)rn, (double)zn, part[0]);
                    part[4] = ll_fma((double)rn, (double)rn, part[4]);
                }
            }
        }
        // a p of row q
        auto ap = [&](int q, int s) { return WT ? P[q][s] : A[q][s] * P[q][s]; };
#pragma unroll
        for (int s = 0; s < 3; ++s) {
            sh.lo[wid][s][lane] = ap(0, s);
            sh.hi[wid + 1][s][lane] = ap(RPT - 1, s);
        }
        if (ring) {
#pragma unroll
            for (int s = 0; s < 3; ++s) {
                T* dst = wid == 0 ? &sh.hi[0][s][lane] : &sh.lo[NW][s][lane];
                if constexpr (WT) {
                    rR[s] = ll_fma(-alpha, rQ[s], rR[s]);
                    rP[s] = ll_fma(beta, rP[s], rR[s]);
                    *dst = rP[s];
                } else {
                    T zn;
                    cg_advance(rR[s], rP[s], zn, rQ[s], rD[s], alpha, beta);
                    *dst = rA[s] * rP[s];
                }
            }
        }
        __syncthreads();

        // faces row by row, A p at the own anchors
        T below[3], up[3];
#pragma unroll
        for (int s = 0; s < 3; ++s) {
            below[s] = sh.hi[wid][s][lane];
            up[s] = sh.lo[wid + 1][s][lane];
        }
        T w[3], wn[3];   // a p of the row and of the next one
#pragma unroll
        for (int s = 0; s < 3; ++s) w[s] = ap(0, s);
        T gum = Kum * ((below[0] - lane_left(below[0])) + (lane_left(below[1]) - below[1]) +
                       (below[2] - w[2]));
        T gv = Kv[0] * ((w[0] - below[0]) + (w[1] - below[1]) + (w[2] - lane_right(w[2])));
#pragma unroll
        for (int q = 0; q < RPT; ++q) {
            constexpr int last = RPT - 1;
            const int qn = q < last ? q + 1 : last;
#pragma unroll
            for (int s = 0; s < 3; ++s) wn[s] = q < last ? ap(qn, s) : up[s];
            const T kv = q < last ? Kv[qn] : Kvp;
            const T gu = Ku[q] * ((w[0] - lane_left(w[0])) + (lane_left(w[1]) - w[1]) + (w[2] - wn[2]));
            const T gvn = kv * ((wn[0] - w[0]) + (wn[1] - w[1]) + (wn[2] - lane_right(wn[2])));
            const T gu1 = lane_right(gu), gvl = lane_left(gv);
            auto pv = [&](int s) { return WT ? P[q][s] * IA[WT ? q : 0][s] : P[q][s]; };   // p
            T y[3];
            y[0] = A[q][0] * ((gu - gu1) + (gv - gvn));
            const T s1 = (gu1 - gu) + (gv - gvn), s2 = (gu - gum) + (gv - gvl);
            y[1] = WT ? ll_fma(C[q][0], pv(1), A[q][1] * s1) : ll_fma(A[q][1], s1, C[q][0] * pv(1));
            y[2] = WT ? ll_fma(C[q][1], pv(2), A[q][2] * s2) : ll_fma(A[q][2], s2, C[q][1] * pv(2));
#pragma unroll
            for (int s = 0; s < 3; ++s) {
                const T dd = WT ? D[q][s] * IA[WT ? q : 0][s] : D[q][s];
                const T zn = WT ? R[q][s] * IA[WT ? q : 0][s] : D[q][s] * R[q][s];
                if (mine) {
                    const double yd = y[s];
                    part[1] = ll_fma((double)pv(s), yd, part[1]);
                    part[2] = ll_fma((double)zn, yd, part[2]);
                    part[3] = ll_fma((double)dd * yd, yd, part[3]);
                }
                if (WT) y[s] = (dd * A[q][s]) * y[s];   // e A p
            }
            if (mt.W > 1) send_row(mt, sh, q, y, stamp);
#pragma unroll
            for (int s = 0; s < 3; ++s) {
                Q[q][s] = mine ? y[s] : T(0);
                w[s] = wn[s];
            }
            gum = gu;
            gv = gvn;
        }
        finish_round(mt, sh, part, stamp);
    }
};

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
    LLWord* part;
    LLWord* msg;
    long long slot;
    unsigned stamp;  // stamps of this solve start here
    int set_bb;
    Scalars* sc;
};

template <typename T, int RPT>
__global__ __launch_bounds__(NT, 1) void k_resident2d(Res2dArgs<T> S) {
    __shared__ Res2dLds<T, RPT> sh;
    const Geo& g = S.g;
    const long long NP = g.NP;
    Res2d<T, RPT> v;
    v.place(g, S.tiles[blockIdx.x], S.ntx);
    v.load(g, S.ntx, S.dinv, S.a, S.c, S.K, sh);
#pragma unroll
    for (int q = 0; q < RPT; ++q) {
        const long long o = v.off(g, v.jw + q);
#pragma unroll
        for (int s = 0; s < 3; ++s) {
            v.R[q][s] = S.r[s * NP + o];
            v.P[q][s] = v.Q[q][s] = T(0);
            const T x = S.x[s * NP + o];
            if constexpr (Res2dLds<T, RPT>::XLDS)
                sh.x[q][s][v.tid] = x;
            else
                v.X[q][s] = x;
        }
    }
#pragma unroll
    for (int s = 0; s < 3; ++s) {
        v.rR[s] = S.r[s * NP + v.ro];
        v.rP[s] = v.rQ[s] = T(0);
    }
    const double tol2 = S.sc->tol2;
    const int max_iter = S.sc->max_iter;
    double bb = S.set_bb ? 0.0 : S.sc->bb;
    const Meeting mt{S.part, S.msg, S.slot, (int)gridDim.x, (int)blockIdx.x, &S.sc->aborted, nullptr};

    // iteration 0: p = z
    v.iterate(mt, sh, T(0), T(0), S.stamp + 1u);
    for (int k = 1;; ++k) {
        double tot[5];
        if (!v.collect(mt, sh, S.stamp + (unsigned)k, tot)) return;
        if (S.set_bb && k == 1) bb = tot[4];
        const CgStep st = cg_step(tot, tol2, bb, k - 1, max_iter);
        if (st.stop) {
            if (mt.me == 0 && v.tid == 0) {
                Scalars* sc = S.sc;
                sc->rr = tot[4];
                sc->pq = tot[1];
                if (S.set_bb) sc->bb = bb;
                sc->iter = k - 1;
                sc->done = st.stop;
            }
            break;
        }
        v.iterate(mt, sh, (T)st.alpha, (T)st.beta, S.stamp + (unsigned)k + 1u);
    }
#pragma unroll
    for (int q = 0; q < RPT; ++q) {
        const int j = v.jw + q;
        if (v.mine && j <= g.ny) {
#pragma unroll
            for (int s = 0; s < 3; ++s) {
                if constexpr (Res2dLds<T, RPT>::XLDS)
                    S.x[s * NP + g.idx(v.i, j)] = sh.x[q][s][v.tid];
                else
                    S.x[s * NP + g.idx(v.i, j)] = v.X[q][s];
            }
        }
    }
}

// A batch of mixed solves.  The launched form walks all tiles of all problems
// once per iteration, each read from and written to memory, with a barrier over
// the whole chip in between (1.06 s for 64 problems of 64^2 to 512^2 to 1e-11);
// here a group of workgroups keeps one problem on the chip until it is solved,
// FP64 refinement included, and the groups do not wait for each other.  A pass
// is FP32 CG on r64 / |r64| to the pass's tolerance, x64 += |r64| x, the FP64
// residual.  x64, r64 and the residual's partial sums cross workgroups through
// memory, once a pass, behind fences; the residual and its norm are formed over
// 64 x 8 tiles with the roundings and the order of k_batch_resid.
__device__ __forceinline__ double batch_resid_at(const BProb& P, int i, int j) {
#pragma clang fp contract(off)
    const Geo& g = P.g;
    const long long NP = g.NP;
    auto W = [&](int s, int ii, int jj) {
        const long long o = s * NP + g.idx(ii, jj);
        return P.a64[o] * P.x64[o];
    };
    const long long o = g.idx(i, j);
    // the padding is zero, also past the upper edges
    auto u = [&](int ii, int jj) {
        return P.K64[g.idx(ii, jj)] * ((W(0, ii, jj) - W(0, ii - 1, jj)) + (W(1, ii - 1, jj) - W(1, ii, jj)) +
                                       (W(2, ii, jj) - W(2, ii, jj + 1)));
    };
    auto v = [&](int ii, int jj) {
        return P.K64[NP + g.idx(ii, jj)] *
               ((W(0, ii, jj) - W(0, ii, jj - 1)) + (W(1, ii, jj) - W(1, ii, jj - 1)) +
                (W(2, ii, jj) - W(2, ii + 1, jj)));
    };
    const double gu0 = u(i, j), gu1 = i < g.nx ? u(i + 1, j) : 0.0, gum = j > 0 ? u(i, j - 1) : 0.0;
    const double gv0 = v(i, j), gv1 = j < g.ny ? v(i, j + 1) : 0.0, gvm = i > 0 ? v(i - 1, j) : 0.0;
    const double r0 = ll_fma(-((gu0 - gu1) + (gv0 - gv1)), P.a64[o], P.b64[o]);
    const double y1 = ll_fma((gu1 - gu0) + (gv0 - gv1), P.a64[NP + o], P.c64[NP + o] * P.x64[NP + o]);
    const double y2 = ll_fma((gu0 - gum) + (gv0 - gvm), P.a64[2 * NP + o],
                             P.c64[2 * NP + o] * P.x64[2 * NP + o]);
    const double r1 = P.b64[NP + o] - y1, r2 = P.b64[2 * NP + o] - y2;
    P.r64[o] = r0;
    P.r64[NP + o] = r1;
    P.r64[2 * NP + o] = r2;
    return ll_fma(r2, r2, ll_fma(r0, r0, r1 * r1));
}

template <int RPT>
__global__ __launch_bounds__(NT, 1) void k_batch_resident(BatchArgs B, const BResProb* __restrict__ rp,
                                                          const BResWg* __restrict__ wgs,
                                                          const int* __restrict__ list,
                                                          unsigned* beats) {
    using Tile = Res2d<float, RPT, true>;
    __shared__ Res2dLds<float, RPT> sh;
    __shared__ double sSum[NW];
    const BResWg wg = wgs[blockIdx.x];
    const int me = (int)blockIdx.x - wg.group0;
    unsigned beat = 0;
    for (int e = 0; e < wg.nlist; ++e) {
        const int pr = list[wg.list0 + e];
        const BResProb rb = rp[pr];
        if (me >= rb.W) continue;
        const BProb& P = B.prob[pr];
        const Geo& g = P.g;
        const long long NP = g.NP;
        const Meeting mt{rb.part, rb.msg, rb.slot, rb.W, me, &B.ctl->abort, beats + wg.group};
        Tile v;
        __syncthreads();   // LDS of the previous problem is no longer read
        v.place(g, rb.tiles[me], rb.ntx);
        v.load(g, rb.ntx, P.ead, P.a, P.c, P.K, sh);
        __syncthreads();
        const bool lead = me == 0 && v.tid == 0;
        auto alive = [&]() {
            if (lead)
                __hip_atomic_store(beats + wg.group, ++beat, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        };
        unsigned stamp = rb.stamp;
        double tot[5];
        // everybody's stores before it are seen by everybody's loads after it
        // (a round without content)
        auto meet = [&]() {
            const double none[5] = {};
            const float zero[3] = {0.f, 0.f, 0.f};
            __threadfence();
            __syncthreads();
            ++stamp;
            alive();
            if (mt.W > 1) {
#pragma unroll
                for (int q = 0; q < RPT; ++q) v.send_row(mt, sh, q, zero, stamp);
            }
            v.finish_round(mt, sh, none, stamp);
            const bool ok = v.collect(mt, sh, stamp, tot);
            __threadfence();
            return ok;
        };
        // r64 = b - A x64 and |r64|^2
        auto residual = [&](double& norm2) {
            const int half = v.wid >> 2, row = v.wid & 3;
            for (int m = 0; m < rb.nt64; m += 2 * mt.W) {
                const int item = m + 2 * mt.me + half;
                double acc = 0.0;
                if (item < rb.nt64) {
                    const int t = rb.tiles64[item];
                    const int i = (t % rb.ntx64) * 64 + v.lane, j = (t / rb.ntx64) * 8 + row;
                    if (i <= g.nx && j <= g.ny) acc += batch_resid_at(P, i, j);
                    if (i <= g.nx && j + 4 <= g.ny) acc += batch_resid_at(P, i, j + 4);
                }
                const double s = wave_sum64(acc);
                if (v.lane == 0) sSum[v.wid] = s;
                __syncthreads();
                if (item < rb.nt64 && row == 0 && v.lane == 0)
                    rb.part64[item] = ((sSum[4 * half] + sSum[4 * half + 1]) + sSum[4 * half + 2]) + sSum[4 * half + 3];
                __syncthreads();
            }
            if (!meet()) return false;
            double s = 0.0;
            if (v.tid < 256)
                for (int b = v.tid; b < rb.nt64; b += 256) s += rb.part64[b];
            s = wave_sum64(s);
            if (v.lane == 0) sSum[v.wid] = s;
            __syncthreads();
            norm2 = ((sSum[0] + sSum[1]) + sSum[2]) + sSum[3];
            __syncthreads();
            return true;
        };
        double rho2;
        if (!residual(rho2)) return;
        const double bb64 = rho2;
        double rel = bb64 > 0.0 ? sqrt(rho2 / bb64) : 0.0;
        int iters = 0, passes = 0;
        while (rel > B.tol && isfinite(rel) && passes < B.max_passes && iters < B.max_iter) {
            double ti = 0.5 * B.tol / rel;
            ti = ti < 1e-5 ? 1e-5 : (ti > 0.5 ? 0.5 : ti);
            const double tol2 = ti * ti, rho = sqrt(rho2), inv = rho2 > 0.0 ? 1.0 / sqrt(rho2) : 0.0;
            // the pass starts from r = r64 / |r64|, weighted on tile and halo
#pragma unroll
            for (int q = 0; q < RPT; ++q) {
                const long long o = v.off(g, v.jw + q);
#pragma unroll
                for (int s = 0; s < 3; ++s) {
                    const float r = (float)(P.r64[s * NP + o] * inv);
                    v.P[q][s] = r;
                    v.R[q][s] = v.D[q][s] * r;
                    v.Q[q][s] = 0.f;
                    if constexpr (Res2dLds<float, RPT>::XLDS)
                        sh.x[q][s][v.tid] = 0.f;
                    else
                        v.X[q][s] = 0.f;
                }
            }
#pragma unroll
            for (int s = 0; s < 3; ++s) {
                v.rR[s] = v.rD[s] * (float)(P.r64[s * NP + v.ro] * inv);
                v.rP[s] = v.rQ[s] = 0.f;
            }
            double bb = 0.0;
            v.iterate(mt, sh, 0.f, 0.f, ++stamp, true);
            int k = 1;
            for (;; ++k) {
                if ((k & 255) == 0) alive();
                if (!v.collect(mt, sh, stamp, tot)) return;
                if (k == 1) bb = tot[4];
                const CgStep st = cg_step(tot, tol2, bb, k - 1, min(B.max_iter_pass, B.max_iter - iters));
                if (st.stop) break;
                v.iterate(mt, sh, (float)st.alpha, (float)st.beta, ++stamp);
            }
            iters += k - 1;
            // x64 += |r64| x at the own anchors
#pragma unroll
            for (int q = 0; q < RPT; ++q) {
                const int j = v.jw + q;
                if (v.mine && j <= g.ny) {
#pragma unroll
                    for (int s = 0; s < 3; ++s) {
                        double* x = P.x64 + s * NP + g.idx(v.i, j);
                        float d;
                        if constexpr (Res2dLds<float, RPT>::XLDS)
                            d = sh.x[q][s][v.tid];
                        else
                            d = v.X[q][s];
                        *x = ll_fma(rho, (double)d, *x);
                    }
                }
            }
            ++passes;
            if (!meet() || !residual(rho2)) return;
            rel = sqrt(rho2 / bb64);
        }
        if (lead) {
            BState& S = B.state[pr];
            S.bb64 = bb64;
            S.rho2 = rho2;
            S.rel = rel;
            S.iters_total = iters;
            S.passes = passes;
            S.stamp = stamp;
            S.t_done = wall_clock64();
        }
        alive();
    }
}

__global__ __launch_bounds__(256) void k_batch_resident_start(BatchArgs A, unsigned* beats, int give_up) {
    const int p = blockIdx.y;
    const BProb& P = A.prob[p];
    if (blockIdx.x == 0 && threadIdx.x == 0) {
        BState& S = A.state[p];
        S.t_start = wall_clock64();
        S.t_done = 0;
        S.rel = S.rho2 = S.bb64 = 0.0;
        S.iters_total = S.passes = S.needs = 0;
        S.stamp = 0;
        if (p == 0) A.ctl->abort = give_up;
    }
    if (p == 0 && blockIdx.x == 0) beats[threadIdx.x] = 0;
    const long long n = 3 * P.g.NP;
    for (long long e = (long long)blockIdx.x * 256 + threadIdx.x; e < n; e += (long long)gridDim.x * 256)
        P.x64[e] = P.r64[e] = 0.0;
}

// flag of every W x 8 strip of the tile lattice: some sample has a != 0
template <int W>
__global__ __launch_bounds__(512) void k_res2d_flags(Geo g, int ntx, const double* __restrict__ a,
                                                     int* __restrict__ flags) {
    const int t = blockIdx.x;
    const int i = (t % ntx) * W + (threadIdx.x & 63), j = (t / ntx) * NW + (threadIdx.x >> 6);
    int any = 0;
    if ((threadIdx.x & 63) < W && i <= g.nx && j <= g.ny)
        for (int s = 0; s < 3; ++s) any |= a[s * g.NP + g.idx(i, j)] != 0.0;
    any = __syncthreads_or(any);
    if (threadIdx.x == 0) flags[t] = any;
}

// ordered tile lists: workgroup b < kResShapes lists the tiles of 2^b strips
// (of which one is flagged) in list b, the last one the 64 x 8 tiles
struct Res2dLists {
    int ntx, nty, ntx64;
    const int* flags;
    const int* flags64;
    int* lists;
    int* list64;
    int* counts;
};
__global__ __launch_bounds__(1024) void k_res2d_lists(Res2dLists L) {
    const bool wide = blockIdx.x == kResShapes;
    const int rpt = wide ? 1 : 1 << blockIdx.x;
    const int ntx = wide ? L.ntx64 : L.ntx;
    const int rows = (L.nty + rpt - 1) / rpt, n = ntx * rows;
    const int* flags = wide ? L.flags64 : L.flags;
    int* list = wide ? L.list64 : L.lists + blockIdx.x * kResMost;
    const int cap = wide ? n : kResMost;
    __shared__ int sCnt[16];
    const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
    int base = 0;
    for (int t0 = 0; t0 < n; t0 += 1024) {
        const int t = t0 + threadIdx.x;
        int any = 0;
        if (t < n) {
            const int tx = t % ntx, ty = t / ntx;
            for (int q = 0; q < rpt && ty * rpt + q < L.nty; ++q) any |= flags[tx + ntx * (ty * rpt + q)];
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
    if (threadIdx.x == 0) L.counts[blockIdx.x] = base;
}

static_assert(kResMost == 256, "beats: one per thread of k_batch_resident_start");

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

int res2d_tiles64(const Geo& g) { return ((g.nx + 64) / 64) * ((g.ny + NW) / NW); }

void launch_res2d_lists(const Geo& g, const double* a, int* flags, int* lists, int* list64, int* counts,
                        hipStream_t s) {
    int ntx, nty;
    res2d_lattice(g, ntx, nty);
    const int ntx64 = (g.nx + 64) / 64;
    int* flags64 = flags + ntx * nty;
    hipLaunchKernelGGL((k_res2d_flags<BX>), dim3(ntx * nty), dim3(512), 0, s, g, ntx, a, flags);
    hipLaunchKernelGGL((k_res2d_flags<64>), dim3(ntx64 * nty), dim3(512), 0, s, g, ntx64, a, flags64);
    const Res2dLists L{ntx, nty, ntx64, flags, flags64, lists, list64, counts};
    hipLaunchKernelGGL(k_res2d_lists, dim3(kResShapes + 1), dim3(1024), 0, s, L);
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

void launch_batch_resident_start(const BatchArgs& A, unsigned* beats, bool give_up, hipStream_t s) {
    hipLaunchKernelGGL(k_batch_resident_start, dim3(64, A.nprob), dim3(256), 0, s, A, beats,
                       give_up ? 1 : 0);
}

void launch_batch_resident(int shape, const BatchArgs& A, const BResProb* rp, const BResWg* wg,
                           const int* list, unsigned* beats, int grid, hipStream_t s) {
    if (shape == 0)
        hipLaunchKernelGGL((k_batch_resident<1>), dim3(grid), dim3(NT), 0, s, A, rp, wg, list, beats);
    else if (shape == 1)
        hipLaunchKernelGGL((k_batch_resident<2>), dim3(grid), dim3(NT), 0, s, A, rp, wg, list, beats);
    else
        hipLaunchKernelGGL((k_batch_resident<4>), dim3(grid), dim3(NT), 0, s, A, rp, wg, list, beats);
}

template void launch_resident2d<float>(const Geo&, int, const int*, int, const float*, float*,
                                       const float*, const float*, const float*, const float*,
                                       LLWordBuf, LLWordBuf, unsigned, bool, Scalars*, hipStream_t);
template void launch_resident2d<double>(const Geo&, int, const int*, int, const double*, double*,
                                        const double*, const double*, const double*, const double*,
                                        LLWordBuf, LLWordBuf, unsigned, bool, Scalars*, hipStream_t);

}  // namespace vfs

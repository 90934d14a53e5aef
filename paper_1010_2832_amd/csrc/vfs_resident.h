// Exchange between the workgroups of a resident kernel: all of them stay on
// the chip for a whole solve and trade values through memory once per CG
// iteration, without a launch, a fence or a barrier.
//
// The words are those of low-latency collectives, which send a flag with every
// few bytes of data: every value travels as 8-byte words of 32 bits of payload
// and a 32-bit stamp, stored and polled with relaxed agent-scope atomics (which
// bypass the caches that are not shared), so a word that shows the expected
// stamp is the value itself: one trip through memory carries data and arrival.
// All participants reading ten words of each other took 1.4 us a round for 32
// workgroups and 2.3 us for 256 (a grid barrier with release and acquire: 12
// us for 256, because it writes back and invalidates the L2s).
//
// Two slots by iteration parity suffice: a workgroup stores iteration k + 1
// only after it has read the partial sums of iteration k from everybody, and
// everybody stores those after reading all it needs of iteration k - 1.
// Stamps grow over all solves of a context, so no slot has to be cleared but
// after a solve that was given up.
// Every wait ends: by arrival, by the abort flag of the solve, or by a
// deadline, which sets that flag.
#pragma once

#include <hip/hip_runtime.h>

#include "vfs_reduce.h"

namespace vfs {

using LLWord = unsigned long long;

// wall clock ticks (100 MHz) after which a wait gives up: 1 s
constexpr long long kResidentTicks = 100000000LL;

__device__ __forceinline__ LLWord ll_load(const LLWord* p) {
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ void ll_store(LLWord* p, unsigned payload, unsigned stamp) {
    __hip_atomic_store(p, ((LLWord)stamp << 32) | payload, __ATOMIC_RELAXED,
                       __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ bool ll_ready(LLWord w, unsigned stamp) {
    return (unsigned)(w >> 32) == stamp;
}

// words of one value
template <typename T>
constexpr int kLLWords = (int)sizeof(T) / 4;

__device__ __forceinline__ void ll_put(LLWord* p, float v, unsigned stamp) {
    ll_store(p, __float_as_uint(v), stamp);
}
__device__ __forceinline__ void ll_put(LLWord* p, double v, unsigned stamp, int step = 1) {
    ll_store(p, (unsigned)__double2loint(v), stamp);
    ll_store(p + step, (unsigned)__double2hiint(v), stamp);
}
// The words of one value, loaded first and looked at later: a poll issues the
// loads of everything it waits for before it waits for any of them.
template <typename T>
struct LLSlot;
template <>
struct LLSlot<float> {
    LLWord w;
    __device__ __forceinline__ void load(const LLWord* p) { w = ll_load(p); }
    __device__ __forceinline__ bool ready(unsigned stamp) const { return ll_ready(w, stamp); }
    __device__ __forceinline__ float value() const { return __uint_as_float((unsigned)w); }
};
template <>
struct LLSlot<double> {
    LLWord w0, w1;
    __device__ __forceinline__ void load(const LLWord* p, int step = 1) {
        w0 = ll_load(p);
        w1 = ll_load(p + step);
    }
    __device__ __forceinline__ bool ready(unsigned stamp) const {
        return ll_ready(w0, stamp) && ll_ready(w1, stamp);
    }
    __device__ __forceinline__ double value() const {
        return __hiloint2double((int)(unsigned)w1, (int)(unsigned)w0);
    }
};

// Pause before the first poll of a round.  What a workgroup waits for takes
// most of a microsecond to arrive; a poll sent at once comes back empty and
// the next one late.  Whole 2D iterations at 512^2 (202 workgroups) took 4.1 us
// without a pause, 3.7 with 768 clocks, 3.5 with 1024, 3.7 with 1536; at 300 x
// 212 (100) 3.5, 3.3, 3.1 and 3.2; at 32^2 (4 workgroups) 768 was best.
__device__ __forceinline__ void ll_first_wait(int workgroups) {
    if (workgroups <= 16)
        __builtin_amdgcn_s_sleep(12);
    else
        __builtin_amdgcn_s_sleep(16);
}

// Patience of one wait: true when it has to end (abort flag up, or the
// deadline, which raises it).  A workgroup may wait for others that are still
// busy with an earlier solve: while `beat` moves, the clock starts again.
struct LLPatience {
    long long t0 = 0;
    int spin = 0;
    unsigned last = 0;
    __device__ __forceinline__ bool over(int* abort_flag, const unsigned* beat) {
        if ((++spin & 63) != 0) return false;
        if (__hip_atomic_load(abort_flag, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) return true;
        const long long t = wall_clock64();
        if (beat) {
            const unsigned b = __hip_atomic_load(beat, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            if (b != last) t0 = 0;
            last = b;
        }
        if (t0 == 0) {
            t0 = t;
            return false;
        }
        if (t - t0 < kResidentTicks) return false;
        __hip_atomic_store(abort_flag, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        return true;
    }
};

// value of the lane to the left (lane - 1) or right (lane + 1); lane 0 or 63
// receives 0
__device__ __forceinline__ float lane_left(float v) {
    return __int_as_float(
        __builtin_amdgcn_update_dpp(0, __float_as_int(v), 0x138, 0xf, 0xf, true));   // wave_shr:1
}
__device__ __forceinline__ float lane_right(float v) {
    return __int_as_float(
        __builtin_amdgcn_update_dpp(0, __float_as_int(v), 0x130, 0xf, 0xf, true));   // wave_shl:1
}
__device__ __forceinline__ double lane_left(double v) { return dpp_move<0x138, 0xf>(v); }
__device__ __forceinline__ double lane_right(double v) { return dpp_move<0x130, 0xf>(v); }

// Sums of five values over the 64 lanes of a wave.  Two exchange steps leave
// each lane one of the first four values (the lane's number mod 4) and the
// fifth, so 13 additions do what five separate sums take 30 for; the rotations
// and swaps add the lanes of equal residue.  Lane l < 4 returns the total of
// v[l] in `four`, lane 0 that of v[4] in `fifth`.
template <int CTRL>
__device__ __forceinline__ double dpp_perm(double v) {
    return dpp_move<CTRL, 0xf>(v);
}
__device__ __forceinline__ double swap_rows16(double v) {
    const auto lo = __builtin_amdgcn_permlane16_swap((unsigned)__double2loint(v),
                                                     (unsigned)__double2loint(v), false, false);
    const auto hi = __builtin_amdgcn_permlane16_swap((unsigned)__double2hiint(v),
                                                     (unsigned)__double2hiint(v), false, false);
    return __hiloint2double((int)hi[0], (int)lo[0]) + __hiloint2double((int)hi[1], (int)lo[1]);
}
__device__ __forceinline__ double swap_rows32(double v) {
    const auto lo = __builtin_amdgcn_permlane32_swap((unsigned)__double2loint(v),
                                                     (unsigned)__double2loint(v), false, false);
    const auto hi = __builtin_amdgcn_permlane32_swap((unsigned)__double2hiint(v),
                                                     (unsigned)__double2hiint(v), false, false);
    return __hiloint2double((int)hi[0], (int)lo[0]) + __hiloint2double((int)hi[1], (int)lo[1]);
}
__device__ __forceinline__ void wave_sum5(const double (&v)[5], double& four, double& fifth) {
    const bool odd = threadIdx.x & 1, high = threadIdx.x & 2;
    // quad_perm [1,0,3,2] (0xb1): the neighbour; [2,3,0,1] (0x4e): two lanes on
    const double a = (odd ? v[1] : v[0]) + dpp_perm<0xb1>(odd ? v[0] : v[1]);
    const double b = (odd ? v[3] : v[2]) + dpp_perm<0xb1>(odd ? v[2] : v[3]);
    double e = v[4] + dpp_perm<0xb1>(v[4]);
    double q = (high ? b : a) + dpp_perm<0x4e>(high ? a : b);
    e += dpp_perm<0x4e>(e);
    q += dpp_perm<0x124>(q);   // row_ror:4
    e += dpp_perm<0x124>(e);
    q += dpp_perm<0x128>(q);   // row_ror:8
    e += dpp_perm<0x128>(e);
    four = swap_rows32(swap_rows16(q));
    fifth = swap_rows32(swap_rows16(e));
}

// Totals of [8 waves][8] values kept in LDS (five of the eight used), in every
// lane of each wave that calls it.
__device__ __forceinline__ double waves_total8(const double (*s)[8]) {
    const int lane = threadIdx.x & 63;
    const double v = s[lane >> 3][lane & 7];
    return swap_rows32(swap_rows16(v + dpp_perm<0x128>(v)));   // lane l: total of value l % 8
}
__device__ __forceinline__ double lane_value(double v, int lane) {
    return __hiloint2double(__builtin_amdgcn_readlane(__double2hiint(v), lane),
                            __builtin_amdgcn_readlane(__double2loint(v), lane));
}

// r -= alpha q and p = D^-1 r + beta p in a fixed order of roundings: the owner
// of a sample and every workgroup that keeps it as halo get the same bits.
__device__ __forceinline__ float ll_fma(float a, float b, float c) { return __builtin_fmaf(a, b, c); }
__device__ __forceinline__ double ll_fma(double a, double b, double c) { return __builtin_fma(a, b, c); }
template <typename T>
__device__ __forceinline__ void cg_advance(T& r, T& p, T& z, T q, T d, T alpha, T beta) {
#pragma clang fp contract(off)
    r = ll_fma(-alpha, q, r);
    z = d * r;
    p = ll_fma(beta, p, z);
}

// Stop decision and CG scalars of iteration k - 1 from its five totals (r.z,
// p.q, q.D^-1 r, q.D^-1 q, r.r), the rules of k_fused2d.
struct CgStep {
    int stop;
    double alpha, beta;
};
__device__ __forceinline__ CgStep cg_step(const double (&t)[5], double tol2, double bb, int done_iters,
                                          int max_iter) {
    const double rz = t[0], pq = t[1], qdr = t[2], qdq = t[3], rr = t[4];
    CgStep s{0, 0.0, 0.0};
    if (!isfinite(rz) || !isfinite(rr) || !isfinite(pq))
        s.stop = 3;
    else if (rr <= tol2 * bb)
        s.stop = 1;
    else if (done_iters >= max_iter)
        s.stop = 2;
    else if (!(pq > 0.0))
        s.stop = 3;
    if (s.stop) return s;
    // the two divisions do not wait for each other
    const double irz = 1.0 / rz;
    s.alpha = rz / pq;
    const double rzn = rz - 2.0 * s.alpha * qdr + s.alpha * s.alpha * qdq;
    s.beta = rz > 0.0 ? rzn * irz : 0.0;
    return s;
}

}  // namespace vfs

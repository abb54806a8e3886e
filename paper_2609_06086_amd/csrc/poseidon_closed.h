#pragma once
// Closed-form makespan of one candidate with a per-lane proof that it is
// exact (1F1B with M >= 2S + 2, Eager 1F1B with M >= 4S + 2).
//
// Stage x (0-based) runs m_x warm-up forwards (1F1B: S - x; Eager 1F1B:
// 2(S-1-x) + 1), then n_x = M - m_x pairs (B_i, F_{m_x+i}), then m_x drain
// backwards (1F1B's order F^{S-x-1} (F B)* B* is the same sequence).  Write
// r_x = F_x + B_x and e_x = cf_x + cb_x (boundary x, between stages x, x+1).
//
// Value.  For every stage x there is a path that reaches its first pair as
// late as any path, stays at the stage to the last pair and leaves along the
// heaviest way out:
//   T_x = U_x + n_x r_x + V_x,
//   U_x  = max(Fw_x, U_{x+1} + B_{x+1} + cb_x)          the start of B_{x,1},
//   Fw_x = (F_0 + .. + F_x) + (cf_0 + .. + cf_{x-1}) + (m_x - 1) max(F_0 .. F_x)
//          the finish of the last warm-up forward (a monotone path through
//          rows of constant weight spends its free steps on the heaviest),
// and V_x, from the finish of F_{x,M} to the end, the same with time reversed
// (F and B, cf and cb exchanged, the drain for the warm-up; with all-reduce
// nodes a drain path may end at any stage's R).  So T >= max_x T_x.
//
// Proof.  Let s be the stage with the largest rate among those a path visits
// in its pairs.  Every edge between pair nodes of 1F1B joins consecutive
// slots of the unit-weight schedule (an Eager forward edge spans 3), so a
// detour from s and back has as many nodes as the stay at s it replaces: c_y
// (F, B) couples at each stage y, and at most c_y crossings of y's edge
// towards s, and as many of the other one.  So if every stage y that is not
// in a set K of pairwise non-adjacent stages has
//   r_y + e_{y-1} + e_y <= r_k for all k in K                             (1)
// then no detour gains (each edge is charged to an end point outside K).
// Nor does entering the pairs elsewhere and walking to s: from a stage below,
// the walk's backwards are in U_s; from the warm-up of a stage above, it
// brought (m - 1) max(F_0 .. F_x) along, and is matched by Fw_s while that
// maximum is at most r_s; if it is larger, at stage j, the path that stays at
// j until it walks to s is heavier and has the larger rate, and the argument
// starts again from there.  Leaving is entering with time reversed.  Raising
// the rate of the stages outside K to r_y + g_y, g_y = e_{y-1} + e_y, makes
// (1) hold whichever of them a path visits (and its first and last pair may
// each gain g_y), so
//   T <= max( max_{k in K} T_k, max_{y not in K} T_y + (n_y + 1) g_y ).
// With K = the stages whose raised value or rate reaches the largest
// (T_x + (n_x + 1) g_x >= max T, or r_x + g_x >= max r) the right side is
// max_x T_x, and the lane holds the exact makespan if K satisfies (1) and has
// no adjacent stages.  Under Eager 1F1B a detour also takes two idle slots
// per crossing, which its forward and backward cover, and T = max_x T_x
// whenever no boundary weighs more than a stage's F or B.  The bounds on M
// leave room for the walks between stages.
//
// Lanes without proof are evaluated by the recurrence.  How many those are
// depends on the transfers.  1F1B, 16 and 8 stages of some 8-10 layers each:
// 0.4 % where cf + cb is a tenth to a third of a layer (also when every layer
// costs the same), 7 and 6 % at one to three layers, 36 and 25 % at three to
// ten.  Eager 1F1B's condition is the stricter one, over all stages and
// boundaries at once: none while no boundary outweighs the lightest layer on
// the fastest type, 9 % of the 16-stage synthetic workload, where some do, 94
// and 45 % at a quarter of a layer to one, and nearly all beyond.  (The value
// is exact for almost all of them.)
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "poseidon_internal.h"

namespace pk {

// k * x for a small k; U24: the full-rate 24-bit multiply (the problem's
// stage weights fit 24 bits).  The callers take U24 as a template argument
// and branch once on it, so that no select merges the two products into one
// slow 32-bit multiply.
template <bool U24>
__host__ __device__ __forceinline__ uint32_t mul_small(uint32_t x, uint32_t k) {
#if defined(__HIP_DEVICE_COMPILE__)
    return U24 ? __umul24(x, k) : x * k;
#else
    return x * k;   // (both products are below 2^32)
#endif
}
__host__ __device__ __forceinline__ uint32_t umax(uint32_t a, uint32_t b) { return a > b ? a : b; }
__host__ __device__ __forceinline__ uint32_t umin(uint32_t a, uint32_t b) { return a < b ? a : b; }

// m_x - 1 of 0-based stage x
template <int S, bool EAGER>
__host__ __device__ constexpr int warm_steps(int x) { return (EAGER ? 2 : 1) * (S - 1 - x); }

// The per-stage constants, read through a scalar pointer that the compiler
// cannot see through (one wide scalar load per row and candidate): as loop
// invariants they would hold some 60 scalar registers through the kernels
// and spill into vector lanes.
struct ClosedConst {
    const __attribute__((address_space(4))) uint32_t *c;
    __device__ __forceinline__ explicit ClosedConst(const KParams &p) {
        uint64_t a = reinterpret_cast<uint64_t>(p.ctab);
        asm volatile("" : "+s"(a));
        c = reinterpret_cast<const __attribute__((address_space(4))) uint32_t *>(a);
    }
    template <int ROW>
    __device__ __forceinline__ uint32_t at(int x) const { return c[ROW * kSMax + x]; }
};

// The same in host memory.
struct ClosedConstHost {
    const uint32_t *c;
    explicit ClosedConstHost(const KParams &p) : c(p.ctab) {}
    template <int ROW>
    uint32_t at(int x) const { return c[ROW * kSMax + x]; }
};

// The constants of a problem (host): fills ctab, and edge_max of p, from
// p.S, p.M, p.cf, p.cb and p.closed.
inline void closed_constants(KParams &p, uint32_t (&ctab)[kCRows * kSMax]) {
    for (uint32_t &v : ctab) v = 0;
    p.edge_max = 0;
    for (uint32_t s = 0; s < p.S; ++s) {
        auto row = [&](int r) { return ctab + (size_t)r * kSMax; };
        const uint32_t lo = s > 0 ? row(kCE)[s - 1] : 0u, hi = s + 1 < p.S ? p.cf[s] + p.cb[s] : 0u;
        row(kCE)[s] = hi;
        row(kCSum)[s] = s > 0 ? row(kCSum)[s - 1] + lo : 0u;
        row(kCE2)[s] = lo + hi;
        // (1F1B, M > S; at most M times the boundaries' sum, below 2^31)
        if (p.closed) row(kCE2n)[s] = (p.M - p.S + 1 + s) * (lo + hi);
        row(kCCb)[s] = s + 1 < p.S ? p.cb[s] : 0u;
        row(kCPsi)[s] = s > 0 ? row(kCPsi)[s - 1] + p.cb[s - 1] : 0u;
        p.edge_max = umax(p.edge_max, hi);
    }
}

// T = max_x T_x of one candidate (D: all-reduce weights, with AR); returns
// whether it is proven to be the makespan.
//
// The quantities are kept relative to the transfer times of the boundaries
// above their stage: U less Phi_x = cf_0 + .. + cf_{x-1}, V less Psi_x =
// cb_0 + .. + cb_{x-1}.  An input from the stage below then carries e_x, and
// T_x gains Phi_x + Psi_x = e_0 + .. + e_{x-1}.
template <int S, bool EAGER, bool AR, bool U24, typename CONST = ClosedConst>
__host__ __device__ __forceinline__ bool closed_form(const KParams &p, const uint32_t (&F)[S], const uint32_t (&B)[S],
                                            const uint32_t (&D)[S], uint32_t &T) {
    const CONST cc(p);
    // P[x] = Fw_x (later T_x), X[x] = the drain of stage x from the start of
    // its first backward
    uint32_t P[S], X[S];
    {
        uint32_t pre = 0, mx = 0;
#pragma unroll
        for (int x = 0; x < S; ++x) {
            pre += F[x];
            mx = umax(mx, F[x]);
            P[x] = pre + mul_small<U24>(mx, warm_steps<S, EAGER>(x));
        }
    }
    {
        uint32_t pre = 0, mx = 0, tail = 0, A[AR ? S : 1];
#pragma unroll
        for (int x = 0; x < S; ++x) {
            const uint32_t h = warm_steps<S, EAGER>(x);
            pre += B[x];
            if constexpr (!AR) {
                mx = umax(mx, B[x]);
                X[x] = pre + mul_small<U24>(mx, h);
            } else {
                // A[j] + h B_j (+ the path down to stage j): the drain that
                // takes its h free steps at stage j and then goes on to the
                // heaviest R
                tail = x == 0 ? D[0] : umax(D[x], tail + B[x > 0 ? x - 1 : 0] + cc.template at<kCCb>(x > 0 ? x - 1 : 0));
                A[x] = tail + B[x] - pre - cc.template at<kCPsi>(x);
                uint32_t m = 0;
#pragma unroll
                for (int j = 0; j <= x; ++j) m = umax(m, A[j] + mul_small<U24>(B[j], h));
                X[x] = pre + m;
            }
        }
    }
    // T_x, from the last stage up (n_x = M - 1 - (m_x - 1))
    uint32_t u = P[S - 1], v = X[S - 1], Tm = 0, rm = 0;
#pragma unroll
    for (int x = S - 1; x >= 0; --x) {
        if (x < S - 1) {
            const int b = x + 1 < S ? x + 1 : 0;   // the stage below
            u = umax(P[x], u + B[b] + cc.template at<kCE>(x));
            v = umax(X[x], v + F[b] + cc.template at<kCE>(x));
        }
        const uint32_t r = F[x] + B[x];
        P[x] = u + mul_small<U24>(r, p.M - 1 - warm_steps<S, EAGER>(x));
        P[x] += v + cc.template at<kCSum>(x);
        Tm = umax(Tm, P[x]);
        rm = umax(rm, r);
    }
    T = Tm;
    if constexpr (EAGER) {
        uint32_t mn = umin(F[0], B[0]);
#pragma unroll
        for (int x = 1; x < S; ++x) mn = umin(mn, umin(F[x], B[x]));
        return mn >= p.edge_max;
    } else {
        bool K[S];
        uint32_t low = 0xFFFFFFFFu;   // the smallest rate in K
#pragma unroll
        for (int x = 0; x < S; ++x) {
            const uint32_t r = F[x] + B[x];
            // (bitwise throughout: no branch per stage)
            K[x] = (int)(P[x] + cc.template at<kCE2n>(x) >= Tm) | (int)(r + cc.template at<kCE2>(x) >= rm);
            low = umin(low, K[x] ? r : 0xFFFFFFFFu);
        }
        bool ok = true;
#pragma unroll
        for (int x = 0; x < S; ++x) {
            ok &= (bool)((int)K[x] | (int)(F[x] + B[x] + cc.template at<kCE2>(x) <= low));
            if (x > 0) ok &= !((int)K[x] & (int)K[x > 0 ? x - 1 : 0]);
        }
        return ok;
    }
}

}  // namespace pk

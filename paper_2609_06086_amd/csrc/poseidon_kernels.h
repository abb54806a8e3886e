#pragma once
// Device code (templates) for batched evaluation of Poseidon's 1F1B-DAG training-time
// model on gfx950 (CDNA4), one candidate configuration per lane.
//
// Per lane the path is:
//   (a1) decode: index -> (composition rank, assignment) -> cut points, types
//   (a2) stage weights from per-type prefix sums held in LDS, memory check
//   (a3) the longest path of the schedule's DAG: its closed form with a
//        proof (poseidon_closed.h), and a register stencil for the lanes
//        and problems without one
//   (a4) a wave / block / grid min-reduction of (makespan, index) keys
// and, for the early-stop variant, (a5) the Eq. 2 lower bound with
// block-local compaction of the surviving candidates.
//
// The DAG's longest path is integer add/max work with no contraction, so
// it runs on the VALU; there is nothing here for the matrix cores.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <type_traits>
#include <utility>

#include "poseidon_closed.h"
#include "poseidon_internal.h"

namespace pk {

constexpr int kBlock = 256;            // 4 waves of 64
constexpr int kWaves = kBlock / 64;

// The kernel's arguments (its only parameter, at the start of the kernarg
// segment) through a pointer the compiler cannot see through: fields read
// through it are scalar loads at the point of use.  Read the plain way they
// are loop invariants, some 100 of them in fused_kernel, that are loaded once
// and then spilled into vector lanes (a VALU operation per reload).
__device__ __forceinline__ const KParams &fresh_args() {
    uint64_t a = reinterpret_cast<uint64_t>(__builtin_amdgcn_kernarg_segment_ptr());
    asm volatile("" : "+s"(a));
    return *(const KParams *)reinterpret_cast<const __attribute__((address_space(4))) KParams *>(a);
}

// ---------------------------------------------------------------------------
// LDS image of the context's tables (one copy per block)
// ---------------------------------------------------------------------------
struct Lds {
    const uint64_t *cost;   // [T][L+1]  (prefix bwd << 32) | prefix fwd
    const uint32_t *pm;     // [L+1]     prefix memory
    const uint32_t *cap;    // [T]
    const uint32_t *pd;     // [T][L+1]  prefix all-reduce time (when the problem has one)
};

// Layout: cost (8-byte entries) | pm | cap | pd.
__device__ __forceinline__ Lds stage_tables(const KParams &p, unsigned char *smem) {
    uint64_t *cost = reinterpret_cast<uint64_t *>(smem);
    const uint32_t ncost = p.T * (p.L + 1);
    uint32_t *pm = reinterpret_cast<uint32_t *>(cost + ncost);
    uint32_t *cap = pm + (p.L + 1);
    for (uint32_t i = threadIdx.x; i < ncost; i += kBlock) cost[i] = p.cost[i];
    for (uint32_t i = threadIdx.x; i <= p.L; i += kBlock) pm[i] = p.pm[i];
    for (uint32_t i = threadIdx.x; i < p.T; i += kBlock) cap[i] = p.cap[i];
    uint32_t *pd = cap + p.T;
    if (p.has_ar)
        for (uint32_t i = threadIdx.x; i < ncost; i += kBlock) pd[i] = p.pd[i];
    __syncthreads();
    return Lds{cost, pm, cap, pd};
}

// Stage entries of the evaluation and early-stop kernels.  For device type
// t and end point j = 0..L the fields
//   Pf_t[j], Pb_t[j]   prefix forward and backward time,
//   hm_t[j]            the largest end point h >= j with Pm[h] - Pm[j] <= cap[t],
//   Pd_t[j]            prefix all-reduce time (with all-reduce times only)
// are uint32 at byte t * erow + field * kEntField + 4 j.  A stage [c0, c1) on
// type t then has F = Pf(c1) - Pf(c0), B = Pb(c1) - Pb(c0) and fits its
// memory iff c1 <= hm_t[c0].  Every load is 4 bytes wide at a per-lane
// address and the fields of one end point are a constant distance apart
// (the load's immediate offset): wider loads at per-lane addresses
// serialise on the LDS banks.
//
// With base-T assignment digits and T <= 4, the digit table follows: for
// every r < T^4 the entry-block offsets of the four digits of r (most
// significant first) as 16-bit fields of a uint64, so the types of four
// stages cost one division by T^4 and one load.
struct Ent {
    const unsigned char *e;    // entry blocks (byte addressed)
    const uint64_t *dig;       // [T^4] packed offsets of four digits (dig_tg > 0)
};

template <int NT = kBlock>
__device__ __forceinline__ Ent entry_tables(const KParams &p, unsigned char *smem) {
    uint4 *e = reinterpret_cast<uint4 *>(smem);
    const uint4 *g = reinterpret_cast<const uint4 *>(p.ent);
    const uint32_t n = (p.ent_bytes + 8 * p.dig_tg) / 16;
    for (uint32_t i = threadIdx.x; i < n; i += NT) e[i] = g[i];
    if (threadIdx.x == 0 && (p.dig_tg & 1u))   // an odd number of 8-byte digit entries
        reinterpret_cast<uint64_t *>(smem + p.ent_bytes)[p.dig_tg - 1] =
            reinterpret_cast<const uint64_t *>(reinterpret_cast<const unsigned char *>(p.ent) + p.ent_bytes)[p.dig_tg - 1];
    __syncthreads();
    return Ent{smem, reinterpret_cast<const uint64_t *>(smem + p.ent_bytes)};
}

__device__ __forceinline__ Ent entry_global(const KParams &p) {
    const unsigned char *e = reinterpret_cast<const unsigned char *>(p.ent);
    return Ent{e, reinterpret_cast<const uint64_t *>(e + p.ent_bytes)};
}

// field F of end point c in the type block at byte offset `to` (= t * erow)
template <uint32_t F>
__device__ __forceinline__ uint32_t ent(const Ent &t, uint32_t c, uint32_t to) {
    return *reinterpret_cast<const uint32_t *>(t.e + ((c << 2) + to) + F * kEntField);
}

// ---------------------------------------------------------------------------
// (a1) decode
// ---------------------------------------------------------------------------

// Cut points of the composition with lexicographic rank r (sorted cut
// tuples c_1 < ... < c_{S-1} in 1 .. L-1).  The complements y_j = L - 1 - c_j
// run the other way, and lexicographic order of the cuts is the reverse of
// the co-lexicographic order of the complements, whose rank is
// sum_j C(y_j, S - j) (combinatorial number system).  So R = C(L-1, S-1) - 1
// - r is that rank, and the cuts follow greedily: y_j is the largest y with
// C(y, S - j) <= R, then R <- R - C(y_j, S - j); the last (S - j = 1) is
// y = R.  The kernels carry q = R + 1 and find n = y_j + 1 as the smallest n
// with C(n, S - j) >= q, by a search over column S - j of the Pascal table.
// Cut points in compact form: cut j (1-based) is byte (j-1) % 4 of word
// (j-1) / 4; a valid composition has c_1 >= 1, so an all-zero first byte
// marks an invalid candidate (for S = 1 the single byte is 1 when valid).
template <int S>
struct Codes {
    static constexpr int kWords = S > 1 ? (S - 1 + 3) / 4 : 1;
};

template <int S>
__device__ __forceinline__ void pack_cuts(const uint32_t (&cut)[S + 1], bool ok, uint32_t (&w)[Codes<S>::kWords]) {
#pragma unroll
    for (int k = 0; k < Codes<S>::kWords; ++k) w[k] = 0;
    if (S == 1) {
        w[0] = ok ? 1u : 0u;
        return;
    }
#pragma unroll
    for (int j = 1; j <= S - 1; ++j) w[(j - 1) / 4] |= (ok ? cut[j] : 0u) << (8 * ((j - 1) % 4));
}

template <int S>
__device__ __forceinline__ bool unpack_cuts(const uint32_t (&w)[Codes<S>::kWords], uint32_t L,
                                            uint32_t (&cut)[S + 1]) {
    cut[0] = 0;
    cut[S] = L;
#pragma unroll
    for (int j = 1; j <= S - 1; ++j) cut[j] = (w[(j - 1) / 4] >> (8 * ((j - 1) % 4))) & 0xFFu;
    return (w[0] & 0xFFu) != 0u;   // (an invalid candidate's words are all zero)
}

template <int S>
__device__ __forceinline__ void decode_types(const KParams &p, uint32_t a, uint32_t (&ty)[S]) {
    if (p.assign_mode == kAssignFixed) {
#pragma unroll
        for (int s = 0; s < S; ++s) ty[s] = (p.fixed_word[s / 4] >> (8 * (s % 4))) & 0xFFu;
    } else if (p.assign_mode == kAssignTable) {
        const uint8_t *row = p.assign + (uint64_t)a * S;
#pragma unroll
        for (int s = 0; s < S; ++s) ty[s] = row[s];
    } else {
        // base-T digits, stage 1 most significant.  q = umulhi(a, m) with
        // m = floor(2^32 / T) + 1 is floor(a / T) or one more; one
        // correction makes it exact for every 32-bit a.
#pragma unroll
        for (int s = S - 1; s >= 0; --s) {
            uint32_t q = __umulhi(a, p.magicT);
            int32_t rem = (int32_t)(a - q * p.T);
            if (rem < 0) { q -= 1; rem += (int32_t)p.T; }
            ty[s] = (uint32_t)rem;
            a = q;
        }
    }
}

// Stage types as byte offsets of their entry blocks (t * erow; both factors
// fit 24 bits, so this is the full-rate 24-bit multiply).  Base-T digits
// with T <= 4 go four stages at a time through the digit table: the stages
// S-4..S-1 are the digits of a mod T^4, the four before them those of
// (a div T^4) mod T^4, and so on (stage 1 most significant).
template <int S>
__device__ __forceinline__ void decode_toff(const KParams &p, const Ent &t, uint32_t a, uint32_t (&to)[S]) {
    if (p.assign_mode == kAssignDigits && p.dig_tg) {
        constexpr int NG = (S + 3) / 4;
        uint32_t q = a;
#pragma unroll
        for (int k = 0; k < NG; ++k) {
            uint32_t r = q;
            if (k + 1 < NG) {
                uint32_t d = __umulhi(q, p.dig_magic);   // floor(q / T^4) or one more
                int32_t rem = (int32_t)(q - d * p.dig_tg);
                if (rem < 0) { d -= 1; rem += (int32_t)p.dig_tg; }
                r = (uint32_t)rem;
                q = d;
            }
            const uint64_t w = t.dig[r];
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const int s = S - 4 * k - 4 + i;   // digit i (most significant first) of group k
                if (s >= 0) to[s] = (uint32_t)(w >> (16 * i)) & 0xFFFFu;
            }
        }
        return;
    }
    if (p.assign_mode == kAssignFixed) {
        // the same offsets for every candidate: four stage types a word, each
        // word passed through an empty asm so that the offsets are unpacked
        // (scalar instructions) where they are used instead of S loop-
        // invariant values holding scalar registers through the whole kernel
#pragma unroll
        for (int g = 0; g < (S + 3) / 4; ++g) {
            uint32_t wd = p.fixed_word[g];
            asm volatile("" : "+s"(wd));
#pragma unroll
            for (int i = 0; i < 4; ++i)
                if (4 * g + i < S) to[4 * g + i < S ? 4 * g + i : 0] = ((wd >> (8 * i)) & 0xFFu) * p.erow;
        }
        return;
    }
    uint32_t ty[S];
    decode_types<S>(p, a, ty);
#pragma unroll
    for (int s = 0; s < S; ++s) to[s] = __umul24(ty[s], p.erow);
}

// Joint index first + i = rank * A + assignment of candidate i of the call,
// range mode.  The host gives first = first_rank * A + first_asg; when
// first_asg plus a call's largest i fits 32 bits the rest is one 32-bit
// division by A: q = umulhi(v, floor(2^32 / A)) is floor(v / A) or one less.
// (The 64-bit division it replaces took most of the decode's operations.)
__device__ __forceinline__ void split_index(const KParams &p, uint32_t i, uint64_t &rank, uint64_t &asg) {
    if (p.div_magic) {
        const uint32_t v = p.first_asg + i, A = (uint32_t)p.A;
        uint32_t q = __umulhi(v, p.div_magic), r = v - q * A;
        if (r >= A) { q += 1; r -= A; }
        rank = p.first_rank + q;
        asg = r;
    } else {
        const uint64_t idx = p.first + i;
        rank = idx / p.A;
        asg = idx - rank * p.A;
    }
}

// Candidate i of the call -> (rank, assignment); false if out of range.
template <typename R>
__device__ __forceinline__ bool candidate(const KParams &p, uint64_t i, R &r, uint32_t &a) {
    uint64_t rank, asg;
    if (p.comp_rank) {
        rank = p.comp_rank[i];
        asg = p.assign_idx ? p.assign_idx[i] : 0u;
    } else {
        if (p.A == 1) { rank = p.first + i; asg = 0; }
        else { split_index(p, (uint32_t)i, rank, asg); }
    }
    const bool ok = rank < p.n_comp && asg < p.A;
    r = ok ? (R)rank : (R)0;
    a = ok ? (uint32_t)asg : 0u;
    return ok;
}

// Assignment index of candidate i (valid candidates only).
__device__ __forceinline__ uint32_t assign_of(const KParams &p, uint64_t i) {
    if (p.comp_rank) return p.assign_idx ? p.assign_idx[i] : 0u;
    if (p.A == 1) return 0u;
    uint64_t rank, asg;
    split_index(p, (uint32_t)i, rank, asg);
    return (uint32_t)asg;
}

// ---------------------------------------------------------------------------
// (a2) stage weights and memory feasibility
// ---------------------------------------------------------------------------
template <int S>
__device__ __forceinline__ bool stage_weights(const KParams &p, const Lds &t,
                                              const uint32_t (&cut)[S + 1], const uint32_t (&ty)[S],
                                              uint32_t (&F)[S], uint32_t (&B)[S]) {
    bool feas = true;
    const uint32_t row = p.L + 1;
#pragma unroll
    for (int s = 0; s < S; ++s) {
        const uint64_t *c = t.cost + ty[s] * row;
        const uint64_t hi = c[cut[s + 1]], lo = c[cut[s]];
        F[s] = (uint32_t)hi - (uint32_t)lo;
        B[s] = (uint32_t)(hi >> 32) - (uint32_t)(lo >> 32);
        const uint32_t mem = t.pm[cut[s + 1]] - t.pm[cut[s]];
        feas &= mem <= t.cap[ty[s]];   // (no short circuit: no branch per stage)
    }
    return feas;
}

// The same from the stage entries: no multiply, one address per end point.
template <int S>
__device__ __forceinline__ bool stage_weights(const KParams &p, const Ent &t, const uint32_t (&cut)[S + 1],
                                              const uint32_t (&to)[S], uint32_t (&F)[S], uint32_t (&B)[S]) {
    bool feas = true;
#pragma unroll
    for (int s = 0; s < S; ++s) {
        F[s] = ent<kEPf>(t, cut[s + 1], to[s]) - ent<kEPf>(t, cut[s], to[s]);
        B[s] = ent<kEPb>(t, cut[s + 1], to[s]) - ent<kEPb>(t, cut[s], to[s]);
        feas &= cut[s + 1] <= ent<kEHm>(t, cut[s], to[s]);   // (no short circuit: no branch per stage)
    }
    return feas;
}

// ---------------------------------------------------------------------------
// (a3) longest path of the 1F1B DAG
// ---------------------------------------------------------------------------
// With unit node weights the as-soon-as-possible start slot of every node
// puts at most one node per stage in a slot, and each cross-stage
// predecessor is still the newest node of its stage one slot later.  One
// register per stage, X[s] = finish time of stage s's newest node, therefore
// suffices: slot by slot every active stage updates from the previous
// slot's values,
//   forward : X[s] <- F_s + max(X[s], X[s-1] + cf_{s-1})
//   backward: X[s] <- B_s + max(X[s], X[s+1] + cb_s)
// and T = X[1] after the last slot (B_{1,M} is the DAG's only sink).
//
// The registers hold Y[s] = X[s] + phi_s with phi_s = cf_s + ... + cf_{S-1}
// (the transfer times of the boundaries below stage s).  A constant shift
// per stage does not change any max, and with this one the forward input
// Y[s-1] already contains cf_{s-1}, so the updates become
//   forward : Y[s] <- F_s + max(Y[s], Y[s-1])
//   backward: Y[s] <- B_s + max(Y[s], Y[s+1] + (cf_s + cb_s))
// which saves one add per forward node that has an upstream stage; the
// result is T = Y[1] - phi_1.
//
// For M >= S the 2(M+S-1) slots are a prologue of 2S-1 slots, a steady part
// in which stage s (1-based) runs a forward pass in slots k = s+1 (mod 2)
// and a backward pass in the others, and an epilogue of 2S-2 slots.

constexpr int kIdle = 0, kFwd = 1, kBwd = 2;

// slot k < 2S-1 (prologue), 1-based stage s
__host__ __device__ constexpr int pro_op(int S, int s, int k) {
    return (k >= s - 1 && k <= S - 1) ? kFwd
         : (k >= 2 * S - s + 1 && ((k - s - 1) & 1) == 0) ? kFwd
         : (k >= 2 * S - s && ((k - s) & 1) == 0) ? kBwd
         : kIdle;
}
// slot 2M + j, j < 2S-2 (epilogue)
__host__ __device__ constexpr int epi_op(int S, int s, int j) {
    return (((j - s - 1) & 1) == 0 && j <= s - 3) ? kFwd
         : (((j - s) & 1) == 0 && j <= 2 * S - s - 2) ? kBwd
         : kIdle;
}

// wave-uniform transfer weights after the shift (SGPRs)
template <int S>
struct Comm {
    uint32_t e[S > 1 ? S - 1 : 1];   // cf_s + cb_s, 0-based boundary s
    uint32_t phi0;                   // cf_0 + ... + cf_{S-2}
};

template <int S>
__device__ __forceinline__ uint32_t node(int op, int s, const uint32_t (&Y)[S], const uint32_t (&F)[S],
                                         const uint32_t (&B)[S], const Comm<S> &c) {
    // s is 0-based here
    if (op == kFwd) return F[s] + (s > 0 ? max(Y[s], Y[s > 0 ? s - 1 : 0]) : Y[s]);
    if (op == kBwd)
        return B[s] + (s < S - 1 ? max(Y[s], Y[s < S - 1 ? s + 1 : 0] + c.e[s < S - 1 ? s : 0]) : Y[s]);
    return Y[s];
}

// Registers before the first slot: stage 1 starts at phi_1 (its X is 0);
// every other stage's first node is a forward pass whose upstream input is
// at least phi_s, so 0 there leaves every max unchanged.
template <int S>
__device__ __forceinline__ void dp_init(uint32_t (&Y)[S], const Comm<S> &c) {
#pragma unroll
    for (int s = 0; s < S; ++s) Y[s] = 0;
    Y[0] = c.phi0;
}

template <int S>
__device__ __forceinline__ void steady_slot(int parity, uint32_t (&Y)[S], const uint32_t (&F)[S],
                                            const uint32_t (&B)[S], const Comm<S> &c) {
    uint32_t N[S];
#pragma unroll
    for (int s = 0; s < S; ++s) {
        // 1-based stage s+1 runs forward when k = s+2 (mod 2), i.e. k = s (mod 2)
        const int op = (((s & 1) == parity) ? kFwd : kBwd);
        N[s] = node<S>(op, s, Y, F, B, c);
    }
#pragma unroll
    for (int s = 0; s < S; ++s) Y[s] = N[s];
}

// Prologue (slots 0 .. 2S-2) with its warm-up forwards in closed form.
// Stage s (0-based) first runs S - s forwards F_{s,1..S-s} in slots
// s .. S-1; each reads only its own stage's previous forward and the same
// micro-batch's forward upstream, and with the potential shift every
// forward edge weighs 0.  So the longest path to F_{s,m} is the heaviest
// monotone path through a grid whose row i carries the constant weight F_i:
// it visits rows 0..s once each and spends its other m - 1 steps on the
// heaviest of them,
//     Y[s] = phi_0 + (F_0 + ... + F_s) + (m - 1) max(F_0, ..., F_s),  m = S - s.
// Slots S .. 2S-2 (the first backwards and the forwards between them) run
// on the stencil.  U24: every stage weight is below 2^24.
template <int S, bool U24>
__device__ __forceinline__ void dp_prologue_t(uint32_t (&Y)[S], const uint32_t (&F)[S], const uint32_t (&B)[S],
                                              const Comm<S> &c) {
    uint32_t pre = c.phi0, mx = 0;
#pragma unroll
    for (int s = 0; s < S; ++s) {
        pre += F[s];
        mx = max(mx, F[s]);
        Y[s] = pre + mul_small<U24>(mx, S - 1 - s);
    }
#pragma unroll
    for (int k = S; k < 2 * S - 1; ++k) {
        uint32_t N[S];
#pragma unroll
        for (int s = 0; s < S; ++s) N[s] = node<S>(pro_op(S, s + 1, k), s, Y, F, B, c);
#pragma unroll
        for (int s = 0; s < S; ++s) Y[s] = N[s];
    }
}

template <int S>
__device__ __forceinline__ void dp_prologue(uint32_t (&Y)[S], const uint32_t (&F)[S], const uint32_t (&B)[S],
                                            const Comm<S> &c, bool u24) {
    if (u24) dp_prologue_t<S, true>(Y, F, B, c);
    else dp_prologue_t<S, false>(Y, F, B, c);
}

// one steady iteration: an odd slot then an even slot (slots 2S-1+2i, 2S+2i)
template <int S>
__device__ __forceinline__ void dp_iter(uint32_t (&Y)[S], const uint32_t (&F)[S], const uint32_t (&B)[S],
                                        const Comm<S> &c) {
    steady_slot<S>(1, Y, F, B, c);
    steady_slot<S>(0, Y, F, B, c);
}

// the last steady slot (2M-1) and the epilogue; afterwards Y[s] holds the
// (shifted) finish of B_{s,M}, the last node of every stage
template <int S>
__device__ __forceinline__ void dp_finish(uint32_t (&Y)[S], const uint32_t (&F)[S], const uint32_t (&B)[S],
                                          const Comm<S> &c) {
    steady_slot<S>(1, Y, F, B, c);
#pragma unroll
    for (int j = 0; j < 2 * S - 2; ++j) {
        uint32_t N[S];
#pragma unroll
        for (int s = 0; s < S; ++s) N[s] = node<S>(epi_op(S, s + 1, j), s, Y, F, B, c);
#pragma unroll
        for (int s = 0; s < S; ++s) Y[s] = N[s];
    }
}

// The last steady slot and the epilogue with the drain in closed form, for
// the DAG without all-reduce nodes; returns T = finish(B_{1,M}).
// Stage s (0-based) ends with its last forward F_{s,M} and then its drain,
// the S - s backwards B_{s,m}, m = M-S+s+1 .. M.  Each drain node's
// predecessors are drain nodes, except at the drain's first node: its own
// stage's F_{s,M} and the stage below's last backward before its drain,
// B_{s+1,M-S+s+1} (edge cb_s); and no node outside the drains reads a drain
// node.  Inside the drains a path from stage s to B_{1,M} runs down the
// stages s, s-1, .., 0 (edges cb_i) and takes S - 1 - s more steps along
// its stages, best spent on the heaviest backward, so
//   T = max_s [ max(fin F_{s,M}, fin B_{s+1,M-S+s+1} + cb_s)
//              + (B_0 + .. + B_s) + (cb_0 + .. + cb_{s-1}) + (S-1-s) max(B_0 .. B_s) ].
// The stencil below computes only the nodes outside the drains and keeps,
// per stage, its register just before (Yb) and after (Yf) its last forward:
// the backward before F_{s,M} is B_{s,M-S+s}, the one stage s-1's drain
// starts from.  In shifted registers the bracket is
//   max(Yf[s], Yb[s+1] + cf_s + cb_s) - phi_s, and the constant
//   cb_0 + .. + cb_{s-1} - phi_s is -phi_0 + (cf_0 + cb_0) + .. + (cf_{s-1} + cb_{s-1})
// (modulo 2^32: every sum that reaches T is a path length below 2^31).
template <int S, bool U24>
__device__ __forceinline__ uint32_t dp_finish_t(const KParams &p, uint32_t (&Y)[S], const uint32_t (&F)[S],
                                                const uint32_t (&B)[S], const Comm<S> &c) {
    uint32_t Yf[S], Yb[S];
    Yf[0] = Y[0];                         // stage 0's last forward ran in slot 2M-2
    Yb[S > 1 ? 1 : 0] = Y[S > 1 ? 1 : 0];  // stage 1's runs in slot 2M-1
    {
        // slot 2M-1 without stage 0's backward (the first of its drain)
        uint32_t N[S];
#pragma unroll
        for (int s = 0; s < S; ++s) N[s] = node<S>(s == 0 ? kIdle : ((s & 1) ? kFwd : kBwd), s, Y, F, B, c);
#pragma unroll
        for (int s = 0; s < S; ++s) Y[s] = N[s];
    }
    if (S > 1) Yf[1] = Y[1];
    // epilogue slots 2M + j: stage s >= 2 runs its last forward at j = s - 2;
    // its backwards from j = s - 1 on are drain nodes
#pragma unroll
    for (int j = 0; j + 2 < S; ++j) {
        uint32_t N[S];
#pragma unroll
        for (int s = 0; s < S; ++s) {
            int op = epi_op(S, s + 1, j);
            if (op == kBwd && j >= s - 1) op = kIdle;
            if (op == kFwd && j == s - 2) Yb[s] = Y[s];
            N[s] = node<S>(op, s, Y, F, B, c);
        }
#pragma unroll
        for (int s = 0; s < S; ++s) {
            if (epi_op(S, s + 1, j) == kFwd && j == s - 2) Yf[s] = N[s];
            Y[s] = N[s];
        }
    }
    // ek = cb_0 + .. + cb_{s-1} - phi_s = -phi_0 + e_0 + .. + e_{s-1} (mod 2^32)
    uint32_t T = 0, pb = 0, mxb = 0, ek = 0u - c.phi0;
#pragma unroll
    for (int s = 0; s < S; ++s) {
        pb += B[s];
        mxb = max(mxb, B[s]);
        const uint32_t a = s + 1 < S ? max(Yf[s], Yb[s + 1 < S ? s + 1 : 0] + c.e[s + 1 < S ? s : 0]) : Yf[s];
        T = max(T, a + pb + mul_small<U24>(mxb, S - 1 - s) + ek);
        if (s + 1 < S) ek += c.e[s + 1 < S ? s : 0];
    }
    return T;
}

// The steady iteration is one fixed map Y -> A(Y) built from max and +
// only, so A(Y + c) = A(Y) + c for every constant c.  Once one iteration
// raises every stage by the same amount d, every later iteration does the
// same: after n more iterations the state is exactly Y + n d.  The kernels
// check this at a few iteration counts; a lane that passes jumps to the end
// of the steady part, the others are queued and resumed by the next level.
template <int S>
__device__ __forceinline__ bool dp_settled(const uint32_t (&Y)[S], const uint32_t (&Yp)[S], uint32_t &d) {
    d = Y[0] - Yp[0];
    bool same = true;
#pragma unroll
    for (int s = 1; s < S; ++s) same = same && (Y[s] - Yp[s] == d);
    return same;
}

// run iterations k0+1 .. k1 (k0 <= k1 <= nit); returns whether the state
// settled by iteration k1 and, if so, moves it to iteration `nit` (the end).
// With k1 = nit it simply runs to the end.
template <int S>
__device__ __forceinline__ bool dp_advance(uint32_t (&Y)[S], const uint32_t (&F)[S], const uint32_t (&B)[S],
                                           const Comm<S> &c, uint32_t k0, uint32_t k1, uint32_t nit) {
    if (k1 >= nit) {
        for (uint32_t it = k0; it < nit; ++it) dp_iter<S>(Y, F, B, c);
        return true;
    }
    for (uint32_t it = k0 + 1; it < k1; ++it) dp_iter<S>(Y, F, B, c);
    uint32_t Yp[S];
#pragma unroll
    for (int s = 0; s < S; ++s) Yp[s] = Y[s];
    dp_iter<S>(Y, F, B, c);
    uint32_t d;
    const bool ok = dp_settled<S>(Y, Yp, d);
    const uint32_t jump = ok ? (nit - k1) * d : 0u;
#pragma unroll
    for (int s = 0; s < S; ++s) Y[s] += jump;
    return ok;
}

// 1F1B with M < S: the slot schedule comes from a table of per-slot
// forward / backward stage masks built on the host (the host checks that
// every input is still its stage's newest node, so one register suffices).
template <int S>
__device__ __forceinline__ void dp_table(const KParams &p, const uint32_t (&F)[S], const uint32_t (&B)[S],
                                         const Comm<S> &c, uint32_t (&Y)[S]) {
    dp_init<S>(Y, c);
    for (uint32_t k = 0; k < p.nslots; ++k) {
        const uint32_t fm = p.slot_mask[3 * k], bm = p.slot_mask[3 * k + 2];
        uint32_t N[S];
#pragma unroll
        for (int s = 0; s < S; ++s) {
            const int op = ((fm >> s) & 1u) ? kFwd : (((bm >> s) & 1u) ? kBwd : kIdle);
            N[s] = node<S>(op, s, Y, F, B, c);
        }
#pragma unroll
        for (int s = 0; s < S; ++s) Y[s] = N[s];
    }
}

// Any schedule table (Eager 1F1B, Sec. 4.1.4 / App. B.1).  A stage can
// run ahead of its downstream neighbour by more than one forward pass, so
// a forward node may need the upstream stage's second-newest forward; the
// host marks those nodes in a third mask.  Per stage the registers are the
// newest node of either kind (Y), the newest and previous forward (Fn, Fp)
// and the newest backward (Bn), all shifted by the stage's potential.
template <int S>
__device__ __forceinline__ void dp_sched(const KParams &p, const uint32_t (&F)[S], const uint32_t (&B)[S],
                                         const Comm<S> &c, uint32_t (&Y)[S]) {
    uint32_t Fn[S], Fp[S], Bn[S];
    dp_init<S>(Y, c);
#pragma unroll
    for (int s = 0; s < S; ++s) { Fn[s] = 0; Fp[s] = 0; Bn[s] = 0; }
    for (uint32_t k = 0; k < p.nslots; ++k) {
        const uint32_t fm = p.slot_mask[3 * k], fd = p.slot_mask[3 * k + 1], bm = p.slot_mask[3 * k + 2];
        uint32_t N[S];
#pragma unroll
        for (int s = 0; s < S; ++s) {
            if ((fm >> s) & 1u) {
                const uint32_t in = s == 0 ? 0u : (((fd >> s) & 1u) ? Fp[s > 0 ? s - 1 : 0] : Fn[s > 0 ? s - 1 : 0]);
                N[s] = F[s] + max(Y[s], in);
            } else if ((bm >> s) & 1u) {
                N[s] = B[s] + (s < S - 1 ? max(Y[s], Bn[s < S - 1 ? s + 1 : 0] + c.e[s < S - 1 ? s : 0]) : Y[s]);
            } else {
                N[s] = Y[s];
            }
        }
#pragma unroll
        for (int s = 0; s < S; ++s) {
            if ((fm >> s) & 1u) { Fp[s] = Fn[s]; Fn[s] = N[s]; }
            if ((bm >> s) & 1u) Bn[s] = N[s];
            Y[s] = N[s];
        }
    }
}

// ---------------------------------------------------------------------------
// Eager 1F1B in closed form (M >= 2S-1).  Under unit weights, stage s
// (1-based) runs its 2(S-s)+1 warm-up forwards in slots s-1 .. 2S-s-1;
// from slot 2S-s on it runs a backward in every slot with k + s even and a
// forward in the others, up to its last forward in slot 2M-2S+3s-3; then
// backwards in the slots with k + s even up to 2M+2S-s-2.  That is
// 2(M+S-1) slots: a prologue of 2S-1 slots, M-2S+1 steady pairs of slots
// (2S-1+2i, 2S+2i) and an epilogue of 4S-3 slots.  A forward in the
// alternating part reads the upstream stage's previous forward (kFwdDeep),
// except the stage's last one, which reads the upstream's newest; a
// backward always reads the downstream stage's newest node.
// ---------------------------------------------------------------------------
constexpr int kFwdDeep = 3;

// prologue slot k (0 .. 2S-2), 1-based stage s
__host__ __device__ constexpr int eager_pro_op(int S, int s, int k) {
    return k < s - 1 ? kIdle : k <= 2 * S - s - 1 ? kFwd : (((k + s) & 1) == 0 ? kBwd : kFwdDeep);
}
// steady slot of parity `odd` (slot 2S-1+2i is odd)
__host__ __device__ constexpr int eager_steady_op(int s, int odd) {
    return odd ? ((s & 1) ? kBwd : kFwdDeep) : ((s & 1) ? (s == 1 ? kFwd : kFwdDeep) : kBwd);
}
// epilogue slot 2M-2S+1+j (j = 0 .. 4S-4)
__host__ __device__ constexpr int eager_epi_op(int S, int s, int j) {
    return j <= 3 * s - 4 ? (((j + 1 + s) & 1) == 0 ? kBwd : (j < 3 * s - 4 ? kFwdDeep : kFwd))
         : (j <= 4 * S - s - 3 && ((j + 1 + s) & 1) == 0) ? kBwd
         : kIdle;
}

// phase of a slot: prologue slot K, steady odd / even slot, epilogue slot K
enum EagerPhase { kPro = 0, kOdd = 1, kEven = 2, kEpi = 3 };

template <int S, int PH, int K>
__host__ __device__ constexpr int eager_op_at(int s) {
    return PH == kPro ? eager_pro_op(S, s, K)
         : PH == kOdd ? eager_steady_op(s, 1)
         : PH == kEven ? eager_steady_op(s, 0)
         : eager_epi_op(S, s, K);
}

// node of 0-based stage s with a compile-time op
template <int S, int OP, int s>
__device__ __forceinline__ uint32_t eager_node(const uint32_t (&Y)[S], const uint32_t (&Fn)[S],
                                               const uint32_t (&Fp)[S], const uint32_t (&F)[S],
                                               const uint32_t (&B)[S], const Comm<S> &c) {
    constexpr int u = s > 0 ? s - 1 : 0, d = s < S - 1 ? s + 1 : 0;
    if constexpr (OP == kFwd) return F[s] + (s > 0 ? max(Y[s], Fn[u]) : Y[s]);
    else if constexpr (OP == kFwdDeep) return F[s] + (s > 0 ? max(Y[s], Fp[u]) : Y[s]);
    else if constexpr (OP == kBwd) return B[s] + (s < S - 1 ? max(Y[s], Y[d] + c.e[d > 0 ? d - 1 : 0]) : Y[s]);
    else return Y[s];
}

template <int OP>
__device__ __forceinline__ void eager_store(uint32_t n, uint32_t &y, uint32_t &fn, uint32_t &fp) {
    if constexpr (OP == kFwd || OP == kFwdDeep) { fp = fn; fn = n; }
    y = n;
}

// one slot, every stage's op fixed at compile time (synchronous update)
template <int S, int PH, int K, int... I>
__device__ __forceinline__ void eager_slot(std::integer_sequence<int, I...>, uint32_t (&Y)[S], uint32_t (&Fn)[S],
                                           uint32_t (&Fp)[S], const uint32_t (&F)[S], const uint32_t (&B)[S],
                                           const Comm<S> &c) {
    uint32_t N[S];
    ((N[I] = eager_node<S, eager_op_at<S, PH, K>(I + 1), I>(Y, Fn, Fp, F, B, c)), ...);
    (eager_store<eager_op_at<S, PH, K>(I + 1)>(N[I], Y[I], Fn[I], Fp[I]), ...);
}

// the slots K... of a phase, in order
template <int S, int PH, int... K>
__device__ __forceinline__ void eager_run(std::integer_sequence<int, K...>, uint32_t (&Y)[S], uint32_t (&Fn)[S],
                                          uint32_t (&Fp)[S], const uint32_t (&F)[S], const uint32_t (&B)[S],
                                          const Comm<S> &c) {
    (eager_slot<S, PH, K>(std::make_integer_sequence<int, S>{}, Y, Fn, Fp, F, B, c), ...);
}

template <int S>
__device__ __forceinline__ void eager_pair(uint32_t (&Y)[S], uint32_t (&Fn)[S], uint32_t (&Fp)[S],
                                           const uint32_t (&F)[S], const uint32_t (&B)[S], const Comm<S> &c) {
    eager_slot<S, kOdd, 0>(std::make_integer_sequence<int, S>{}, Y, Fn, Fp, F, B, c);
    eager_slot<S, kEven, 0>(std::make_integer_sequence<int, S>{}, Y, Fn, Fp, F, B, c);
}

// n steady pairs, two per trip so that the forward registers come back to
// the same roles at the loop edge
template <int S>
__device__ __forceinline__ void eager_pairs(uint32_t n, uint32_t (&Y)[S], uint32_t (&Fn)[S], uint32_t (&Fp)[S],
                                            const uint32_t (&F)[S], const uint32_t (&B)[S], const Comm<S> &c) {
    for (uint32_t i = 1; i < n; i += 2) {
        eager_pair<S>(Y, Fn, Fp, F, B, c);
        eager_pair<S>(Y, Fn, Fp, F, B, c);
    }
    if (n & 1u) eager_pair<S>(Y, Fn, Fp, F, B, c);
}

template <int S>
__device__ __forceinline__ void eager_prologue(uint32_t (&Y)[S], uint32_t (&Fn)[S], uint32_t (&Fp)[S],
                                               const uint32_t (&F)[S], const uint32_t (&B)[S], const Comm<S> &c) {
    dp_init<S>(Y, c);
#pragma unroll
    for (int s = 0; s < S; ++s) { Fn[s] = 0; Fp[s] = 0; }
    eager_run<S, kPro>(std::make_integer_sequence<int, 2 * S - 1>{}, Y, Fn, Fp, F, B, c);
}

template <int S>
__device__ __forceinline__ void eager_epilogue(uint32_t (&Y)[S], uint32_t (&Fn)[S], uint32_t (&Fp)[S],
                                               const uint32_t (&F)[S], const uint32_t (&B)[S], const Comm<S> &c) {
    eager_run<S, kEpi>(std::make_integer_sequence<int, 4 * S - 3>{}, Y, Fn, Fp, F, B, c);
}

template <int S>
__device__ __forceinline__ void dp_eager(uint32_t M, const uint32_t (&F)[S], const uint32_t (&B)[S],
                                         const Comm<S> &c, uint32_t (&Y)[S]) {
    uint32_t Fn[S], Fp[S];
    eager_prologue<S>(Y, Fn, Fp, F, B, c);
    eager_pairs<S>(M - 2 * S + 1, Y, Fn, Fp, F, B, c);
    eager_epilogue<S>(Y, Fn, Fp, F, B, c);
}

// Between steady pairs the state that the rest of the DP reads is, per
// stage, the newest forward Fn and, for a stage with odd 1-based index (its
// newest node is that forward), the previous forward Fp, else the newest
// node Y (a backward; its Fp is rewritten before any read).  The pair map is
// built from max and + only, so once one pair raises all 2S values by the
// same d, every later pair does the same (as for 1F1B).  Checking it needs
// one saved value per stage: a pair moves the old Fn into Fp, so
// Fn - Fp is the forward's increment.
template <int S>
__device__ __forceinline__ bool eager_advance(uint32_t (&Y)[S], uint32_t (&Fn)[S], uint32_t (&Fp)[S],
                                              const uint32_t (&F)[S], const uint32_t (&B)[S], const Comm<S> &c,
                                              uint32_t k0, uint32_t k1, uint32_t npairs) {
    const bool last = k1 >= npairs;
    eager_pairs<S>(last ? npairs - k0 : k1 - k0 - 1, Y, Fn, Fp, F, B, c);
    if (last) return true;
    uint32_t Z[S];
#pragma unroll
    for (int s = 0; s < S; ++s) Z[s] = (s & 1) == 0 ? Fp[s] : Y[s];
    eager_pair<S>(Y, Fn, Fp, F, B, c);
    const uint32_t d = Fn[0] - Fp[0];
    bool ok = true;
#pragma unroll
    for (int s = 0; s < S; ++s)
        ok = ok && Fn[s] - Fp[s] == d && ((s & 1) == 0 ? Fp[s] : Y[s]) - Z[s] == d;
    const uint32_t jump = ok ? (npairs - k1) * d : 0u;
#pragma unroll
    for (int s = 0; s < S; ++s) { Y[s] += jump; Fn[s] += jump; Fp[s] += jump; }
    return ok;
}

// queue image of the state between pairs (2S words) and back
template <int S>
__device__ __forceinline__ void eager_pack(const uint32_t (&Y)[S], const uint32_t (&Fn)[S], const uint32_t (&Fp)[S],
                                           uint32_t (&X)[2 * S]) {
#pragma unroll
    for (int s = 0; s < S; ++s) { X[s] = Fn[s]; X[S + s] = (s & 1) == 0 ? Fp[s] : Y[s]; }
}

template <int S>
__device__ __forceinline__ void eager_unpack(const uint32_t (&X)[2 * S], uint32_t (&Y)[S], uint32_t (&Fn)[S],
                                             uint32_t (&Fp)[S]) {
#pragma unroll
    for (int s = 0; s < S; ++s) {
        Fn[s] = X[s];
        Y[s] = (s & 1) == 0 ? X[s] : X[S + s];
        Fp[s] = (s & 1) == 0 ? X[S + s] : 0u;
    }
}

// The whole DP for the few lanes of a wave that survive the early-stop test:
// the closed forms take the steady-state check every kSurvStep iterations,
// and the wave leaves the steady loop as soon as all its active lanes have
// settled (jumped to its end) or reached it.
constexpr uint32_t kSurvStep = 8;


template <int S>
__device__ __forceinline__ Comm<S> load_comm(const KParams &p) {
    Comm<S> c;
    uint32_t phi = 0;
#pragma unroll
    for (int s = 0; s < (S > 1 ? S - 1 : 1); ++s) {
        c.e[s] = p.cf[s] + p.cb[s];
        phi += p.cf[s];
    }
    c.phi0 = phi;
    return c;
}

// ---------------------------------------------------------------------------
// (a5) Eq. 2: g(S_x) = sum_{i<x} F_i + M (F_x + B_x) + max_{i<=x}(sum_{j=i}^{x-1} B_j + d_i)
// ---------------------------------------------------------------------------
// Classification of a candidate against the bound b over its stages
// 0 .. X-1 in pipeline order, as the search of Sec. 4.2.3 discards a
// partial configuration: out = some stage fails; over = the first failing
// stage exceeds its device's memory (tested first at a stage), not only
// g(S_x) <= b.  Both are lane masks in scalar registers, so that a stage
// costs two compares and no other vector operation for its tests.  The stage
// weights come from the stage entries.  Without all-reduce times the inner
// max of Eq. 2 is its whole sum, so g(S_x) = sum_{i<x} (F_i + B_i)
// + M (F_x + B_x) and the two times are needed only as their sum: field
// kEPf holds Pf + Pb then (SUM), or both are read.
template <int S, bool AR, int X, bool G24, bool SUM>
__device__ __forceinline__ void classify_g(const KParams &p, const Ent &t, const uint32_t (&cut)[S + 1],
                                           const uint32_t (&to)[S], uint32_t b, bool &out, bool &over) {
    uint32_t pre = 0, inner = 0, bprev = 0;
    const uint32_t M = p.M;
    out = over = false;
#pragma unroll
    for (int x = 0; x < X; ++x) {
        const uint32_t lo = cut[x], hi = cut[x + 1], tx = to[x];
        const bool m = hi > ent<kEHm>(t, lo, tx);
        uint32_t W = ent<kEPf>(t, hi, tx) - ent<kEPf>(t, lo, tx);
        uint32_t g;
        if constexpr (AR) {
            const uint32_t F = W, B = ent<kEPb>(t, hi, tx) - ent<kEPb>(t, lo, tx);
            const uint32_t D = ent<kEPd>(t, hi, tx) - ent<kEPd>(t, lo, tx);
            inner = x == 0 ? D : max(inner + bprev, D);
            // M (F + B) is below 2^31 like every path weight: a full-rate
            // 24-bit multiply when both factors fit
            g = pre + inner + (G24 ? __umul24(M, F + B) : M * (F + B));
            pre += F;
            bprev = B;
        } else {
            if constexpr (!SUM) W += ent<kEPb>(t, hi, tx) - ent<kEPb>(t, lo, tx);
            g = pre + (G24 ? __umul24(M, W) : M * W);
            pre += W;
        }
        over |= m & !out;
        out |= m | (g > b);
    }
}

template <int S, bool AR, int X, bool SUM>
__device__ __forceinline__ void classify(const KParams &p, const Ent &t, const uint32_t (&cut)[S + 1],
                                         const uint32_t (&to)[S], uint32_t b, bool &out, bool &over) {
    if (p.g24) classify_g<S, AR, X, true, SUM>(p, t, cut, to, b, out, over);
    else classify_g<S, AR, X, false, SUM>(p, t, cut, to, b, out, over);
}

// ---------------------------------------------------------------------------
// end of the iteration: the end node E follows every R_s (Sec. 4.1.1), and
// R_s follows B_{s,M} with the stage's summed per-layer all-reduce time
// (Sec. 4.1.3).  Without all-reduce times T = finish(B_{1,M}).
// ---------------------------------------------------------------------------
template <int S>
__device__ __forceinline__ void stage_allreduce(const KParams &p, const Lds &t, const uint32_t (&cut)[S + 1],
                                                const uint32_t (&ty)[S], uint32_t (&D)[S]) {
    const uint32_t row = p.L + 1;
#pragma unroll
    for (int s = 0; s < S; ++s) D[s] = t.pd[ty[s] * row + cut[s + 1]] - t.pd[ty[s] * row + cut[s]];
}

template <int S>
__device__ __forceinline__ void stage_allreduce(const KParams &p, const Ent &t, const uint32_t (&cut)[S + 1],
                                                const uint32_t (&to)[S], uint32_t (&D)[S]) {
#pragma unroll
    for (int s = 0; s < S; ++s) D[s] = ent<kEPd>(t, cut[s + 1], to[s]) - ent<kEPd>(t, cut[s], to[s]);
}

// T from the registers after the epilogue; with all-reduce times the
// stage's cut codes `w` and assignment `a` give R_s
template <int S, bool AR>
__device__ __forceinline__ uint32_t end_time(const KParams &p, const Lds &t, const uint32_t (&Y)[S],
                                             const Comm<S> &c, const uint32_t (&w)[Codes<S>::kWords], uint32_t a) {
    if (!AR) return Y[0] - c.phi0;
    uint32_t cut[S + 1], ty[S], D[S];
    unpack_cuts<S>(w, p.L, cut);
    decode_types<S>(p, a, ty);
    stage_allreduce<S>(p, t, cut, ty, D);
    // Y[s] - phi_s = finish(B_{s,M}); phi_0 - phi_s = psi_s
    uint32_t e = 0;
#pragma unroll
    for (int s = 0; s < S; ++s) e = max(e, Y[s] + p.psi[s] + D[s]);
    return e - c.phi0;
}

template <int S, bool AR>
__device__ __forceinline__ uint32_t end_time(const KParams &p, const Ent &t, const uint32_t (&Y)[S],
                                             const Comm<S> &c, const uint32_t (&w)[Codes<S>::kWords], uint32_t a) {
    if (!AR) return Y[0] - c.phi0;
    uint32_t cut[S + 1], to[S], D[S];
    unpack_cuts<S>(w, p.L, cut);
    decode_toff<S>(p, t, a, to);
    stage_allreduce<S>(p, t, cut, to, D);
    uint32_t e = 0;
#pragma unroll
    for (int s = 0; s < S; ++s) e = max(e, Y[s] + p.psi[s] + D[s]);
    return e - c.phi0;
}

// After the steady part: T from the last steady slot, the epilogue and the
// end node (1F1B; closed-form drain without all-reduce times).
template <int S, bool AR, typename TAB>
__device__ __forceinline__ uint32_t dp_end(const KParams &p, const TAB &t, uint32_t (&Y)[S], const uint32_t (&F)[S],
                                           const uint32_t (&B)[S], const Comm<S> &c,
                                           const uint32_t (&w)[Codes<S>::kWords], uint32_t a) {
    if constexpr (AR) {
        dp_finish<S>(Y, F, B, c);
        return end_time<S, true>(p, t, Y, c, w, a);
    } else {
        if (p.g24) return dp_finish_t<S, true>(p, Y, F, B, c);
        return dp_finish_t<S, false>(p, Y, F, B, c);
    }
}

// The whole DP of one candidate with a settle check every kSurvStep steady
// iterations (the wave leaves the steady loop once all its lanes settled),
// ending in T (the end node: closed-form drain for 1F1B without all-reduce
// times, else the full epilogue and the all-reduce nodes).
// CLOSED: the problem has a closed form (no slot table).
template <int S, bool SCH, bool AR, bool CLOSED = false, typename TAB>
__device__ __forceinline__ uint32_t dp_full_settle(const KParams &p, const TAB &t, const uint32_t (&F)[S],
                                                   const uint32_t (&B)[S], const Comm<S> &c,
                                                   const uint32_t (&w)[Codes<S>::kWords], uint32_t a) {
    const unsigned long long act = __ballot(true);
    uint32_t Y[S];
    if (SCH && (CLOSED || !p.nslots)) {
        uint32_t Fn[S], Fp[S];
        eager_prologue<S>(Y, Fn, Fp, F, B, c);
        const uint32_t np = p.M - 2 * S + 1;
        bool done = false;
        for (uint32_t k = 0; k < np;) {
            const uint32_t k1 = min(k + kSurvStep, np);
            if (!done) done = eager_advance<S>(Y, Fn, Fp, F, B, c, k, k1, np);
            k = k1;
            if (__ballot(done) == act) break;
        }
        eager_epilogue<S>(Y, Fn, Fp, F, B, c);
    } else if (!SCH && (CLOSED || p.M >= (uint32_t)S)) {
        dp_prologue<S>(Y, F, B, c, p.g24 != 0);
        const uint32_t nit = p.M - S;
        bool done = false;
        for (uint32_t k = 0; k < nit;) {
            const uint32_t k1 = min(k + kSurvStep, nit);
            if (!done) done = dp_advance<S>(Y, F, B, c, k, k1, nit);
            k = k1;
            if (__ballot(done) == act) break;
        }
        return dp_end<S, AR>(p, t, Y, F, B, c, w, a);
    } else if constexpr (SCH) {
        dp_sched<S>(p, F, B, c, Y);
    } else {
        dp_table<S>(p, F, B, c, Y);
    }
    return end_time<S, AR>(p, t, Y, c, w, a);
}

// ---------------------------------------------------------------------------
// (a4) reductions
// ---------------------------------------------------------------------------
__device__ __forceinline__ unsigned long long wave_min(unsigned long long v) {
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1) {
        const unsigned long long w = __shfl_xor(v, o, 64);
        v = w < v ? w : v;
    }
    return v;
}

// Block min of `v` over NT threads, folded into *acc (part: NT / 64 words of LDS).
template <int NT>
__device__ __forceinline__ void block_min(unsigned long long v, unsigned long long *acc, unsigned long long *part) {
    v = wave_min(v);
    if ((threadIdx.x & 63) == 0) part[threadIdx.x >> 6] = v;
    __syncthreads();
    if (threadIdx.x == 0) {
        unsigned long long m = part[0];
#pragma unroll
        for (int w = 1; w < NT / 64; ++w) m = part[w] < m ? part[w] : m;
        if (m != ~0ull) atomicMin(acc, m);
    }
}

// The words a host that waits for a call's result reads, written straight to
// its pinned memory by the call's last block: key, error flag, early-stop
// counters (earlier kernels' writes).  A copy after the kernels costs another
// launch and its wait, about 8 us of a small call's 30.
struct HostOut {
    unsigned long long *words = nullptr;   // null: nobody waits
    const unsigned int *err = nullptr;
    const unsigned long long *stats = nullptr;
};
__device__ __forceinline__ HostOut host_out(const KParams &p) { return HostOut{p.host_words, p.err, p.stats}; }
__device__ __forceinline__ void publish_host(const HostOut &h, unsigned long long key) {
    h.words[kHostKey] = key;
    h.words[kHostErr] = __hip_atomic_load(h.err, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    for (int i = 0; i < 3; ++i)
        h.words[kHostStats + i] = __hip_atomic_load(h.stats + i, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    __threadfence_system();
}

// Block min of `v`, folded into *acc.  When `finalize` is set (the last
// kernel of an evaluation chunk), the last block of the grid also moves *acc
// to *result (or folds it in, for the second and later chunks of a call,
// and/or into *run_best) and re-arms *acc and *done.
__device__ __forceinline__ void block_min_and_finish(unsigned long long v, unsigned long long *acc,
                                                     unsigned int *done, unsigned long long *result,
                                                     unsigned long long *run_best, bool finalize,
                                                     bool accumulate = false,
                                                     unsigned long long *snap = nullptr,
                                                     uint32_t nblocks = 0,
                                                     HostOut host = HostOut{}) {
    __shared__ unsigned long long part[kWaves];
    v = wave_min(v);
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    if (lane == 0) part[wave] = v;
    __syncthreads();
    if (threadIdx.x == 0) {
        unsigned long long m = part[0];
#pragma unroll
        for (int w = 1; w < kWaves; ++w) m = part[w] < m ? part[w] : m;
        if (m != ~0ull) atomicMin(acc, m);
        if (finalize) {
            __threadfence();
            const unsigned int ticket = atomicAdd(done, 1u);
            if (ticket == (nblocks ? nblocks : gridDim.x) - 1) {
                __threadfence();
                const unsigned long long k = atomicExch(acc, ~0ull);
                unsigned long long out = k;
                if (result) {
                    if (accumulate) {
                        const unsigned long long old = atomicMin(result, k);
                        out = old < k ? old : k;
                    } else {
                        atomicExch(result, k);
                    }
                }
                if (run_best) {
                    const unsigned long long old = atomicMin(run_best, k);
                    out = old < k ? old : k;
                    if (snap) atomicExch(snap, out);
                }
                atomicExch(done, 0u);
                if (host.words) publish_host(host, out);
            }
        }
    }
}

__device__ __forceinline__ unsigned long long wave_sum_u32(uint32_t v) {
    unsigned long long s = v;
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1) s += __shfl_xor(s, o, 64);
    return s;
}

// Exclusive prefix sum over the block's threads in thread order; every
// thread gets its offset and the block total.  All threads must call it.
__device__ __forceinline__ unsigned long long block_exclusive_scan_u64(unsigned long long v,
                                                                       unsigned long long &total) {
    __shared__ unsigned long long wtot[kWaves];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    unsigned long long inc = v;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        const unsigned long long u = __shfl_up(inc, o, 64);
        if (lane >= o) inc += u;
    }
    if (lane == 63) wtot[wave] = inc;
    __syncthreads();
    unsigned long long before = 0, all = 0;
#pragma unroll
    for (int k = 0; k < kWaves; ++k) {
        before += k < wave ? wtot[k] : 0ull;
        all += wtot[k];
    }
    __syncthreads();
    total = all;
    return before + inc - v;
}

// Exclusive scan of n per-block counts (of an earlier kernel) into LDS
// (pre[0 .. n-1]) with their total; the caller's next barrier publishes pre.
// The counts are staged in LDS by independent coalesced loads: a thread that
// loaded its own run of counts waited for each of them, which was most of
// the time of a kernel with a short list.
__device__ __forceinline__ void scan_counts(const unsigned int *counts, uint32_t n, uint32_t *pre, uint32_t &total) {
#pragma unroll 8
    for (uint32_t j = threadIdx.x; j < n; j += kBlock) pre[j] = counts[j];
    __syncthreads();
    const uint32_t per = (n + kBlock - 1) / kBlock, j0 = threadIdx.x * per;
    uint32_t mine = 0;
    for (uint32_t j = j0; j < j0 + per && j < n; ++j) mine += pre[j];
    unsigned long long all;
    uint32_t run = (uint32_t)block_exclusive_scan_u64(mine, all);
    for (uint32_t j = j0; j < j0 + per && j < n; ++j) {
        const uint32_t c = pre[j];
        pre[j] = run;
        run += c;
    }
    total = (uint32_t)all;
}

__device__ __forceinline__ unsigned long long make_key(bool feasible, uint32_t T, uint32_t i) {
    return ((unsigned long long)(feasible ? T : 0xFFFFFFFFu) << 32) | i;
}

// ---------------------------------------------------------------------------
// kernels
// ---------------------------------------------------------------------------

// Layout of one straggler queue (the cascades over HBM): idx[cap] | codes[kWords][cap] | asg[cap]
// (calls with a list of assignment indices) | Y[NX][cap].  The entry holds
// the assignment index rather than the next level re-reading it from the
// caller's list: a 4-byte read at a scattered index costs a whole memory
// sector.
template <int S>
struct QueueView {
    uint32_t *idx, *codes, *asg, *Y;
    __device__ __forceinline__ QueueView(const KParams &p, int which) {
        idx = p.queue[which];
        codes = idx + p.qcap;
        asg = codes + (uint64_t)Codes<S>::kWords * p.qcap;
        Y = asg + (p.qasg ? p.qcap : 0ull);
    }
};

// Queue a wave's unsettled lanes (candidate index, cut codes, assignment
// index, registers) for the next level.  Block b owns slots
// [b * seg_cap, (b + 1) * seg_cap) of the queue and counts its entries in
// LDS (*nq), so no global atomic is involved; every lane of the wave must
// call this.  The assignment index (list mode with assignment indices only)
// is `a`, or with a < 0 read again from the caller's list for candidate idx
// of the call: the evaluation kernels would otherwise keep it in a register
// through the DP, which costs them more than the reload of the few lanes
// that are queued.
template <int S, int NX>
__device__ __forceinline__ void enqueue(const KParams &p, int which, unsigned int *nq, bool want, uint32_t idx,
                                        const uint32_t (&w)[Codes<S>::kWords], int64_t a,
                                        const uint32_t (&Y)[NX]) {
    const unsigned long long m = __ballot(want);
    if (m == 0) return;
    const unsigned int lane = threadIdx.x & 63;
    unsigned int base = 0;
    if (lane == 0) base = atomicAdd(nq, (unsigned int)__popcll(m));
    base = __shfl(base, 0, 64);
    if (want) {
        const unsigned long long below = lane ? (m & ((1ull << lane) - 1ull)) : 0ull;
        // 32-bit word offsets: a queue holds fewer than 2^32 words
        const uint32_t slot = blockIdx.x * (uint32_t)p.seg_cap + base + __popcll(below), qcap = (uint32_t)p.qcap;
        const QueueView<S> q(p, which);
        q.idx[slot] = idx;
#pragma unroll
        for (int k = 0; k < Codes<S>::kWords; ++k) q.codes[k * qcap + slot] = w[k];
        if (p.qasg) q.asg[slot] = a >= 0 ? (uint32_t)a : __builtin_nontemporal_load(p.assign_idx + idx);
#pragma unroll
        for (int s = 0; s < NX; ++s) q.Y[s * qcap + slot] = Y[s];
    }
}

// (a1) Unrank every candidate of the chunk [p.first_i, p.first_i + p.n_i)
// into compact cut codes.  Each lane walks kIlp candidates through their
// searches together so that the dependent LDS reads of one overlap those of
// the others.  Invalid (rank, assignment) pairs get the invalid code and
// raise the error flag.
constexpr int kIlp = kDecodeIlp;

// kIlp candidates per lane.  A kernel holds the Pascal columns it searches
// in LDS, each sorted (2^H rows, then kBucketPad rows of the type's largest
// value) and with the host's bucket table (per bucket key, the first row
// whose entry reaches the bucket; the keys are defined with bucket_lo).  The
// search for the smallest n with C(n, c) >= Q starts at the row Q's bucket
// names and halves bucket_steps(w, H, c) times over the 2^steps rows after
// it, which hold every row a value of that bucket can land on.  The last cut
// needs no search (decode_range).
// One halving: t <- 2 t + (probe < Q), as a compare into VCC and an add with
// carry-in (the compiler's select and shift-or take one VALU operation more).
__device__ __forceinline__ uint32_t tree_step(uint32_t t, uint64_t probe, uint64_t q) {
    asm("v_cmp_lt_u64_e32 vcc, %1, %2\n\tv_addc_co_u32_e32 %0, vcc, %0, %0, vcc"
                 : "+v"(t) : "v"(probe), "v"(q) : "vcc");
    return t;
}
__device__ __forceinline__ uint32_t tree_step(uint32_t t, uint32_t probe, uint32_t q) {
    asm("v_cmp_lt_u32_e32 vcc, %1, %2\n\tv_addc_co_u32_e32 %0, vcc, %0, %0, vcc"
                 : "+v"(t) : "v"(probe), "v"(q) : "vcc");
    return t;
}

// Bucket key of Q >= 1, plus kBucketBias (a constant of the table's address).
__device__ __forceinline__ uint32_t bucket_key(uint64_t q) {
    float hi, lo;   // (two 32-bit conversions, spelled out: the compiler makes one of 64 bits, three times as long)
    asm("v_cvt_f32_u32_e32 %0, %1" : "=v"(hi) : "v"((uint32_t)(q >> 32)));
    asm("v_cvt_f32_u32_e32 %0, %1" : "=v"(lo) : "v"((uint32_t)q));
    const float f = __fmaf_rn(hi, 4294967296.0f, lo);
    return __float_as_uint(f) >> 19;
}
__device__ __forceinline__ uint32_t bucket_key(uint32_t q) { return __float_as_uint((float)q) >> 19; }

constexpr uint32_t kBucketPad = 8;   // rows past 2^H: a search reads at most 2^3 - 2 past its start
constexpr int kBucketStepsMax = 3;

// Halvings a search over column c needs after its bucket's start row: the
// most rows the values of one bucket can land on (2^H rows of C(n, c),
// w-bit entries saturated at the type's largest value, values up to the
// column's last entry), as a power of two.  Evaluated at compile time.
__host__ __device__ constexpr int bucket_steps(int w, int H, int c) {
    const int NH = 1 << H;
    const unsigned __int128 vmax = w == 64 ? (unsigned __int128)~0ull : (unsigned __int128)0xFFFFFFFFu;
    unsigned __int128 col[256] = {};
    unsigned __int128 v = c == 0 ? 1 : 0;   // C(n, c): 0 below n = c, then C(n-1, c) n / (n - c)
    for (int n = 0; n < NH; ++n) {
        if (n == c) v = 1;
        else if (n > c) v = v * (unsigned)n / (unsigned)(n - c);
        col[n] = v < vmax ? v : vmax;
    }
    const unsigned __int128 top = col[NH - 1];
    int most = 1;
    for (uint32_t key = 0; key < bucket_tab_bytes(w); ++key) {
        const unsigned __int128 lo = bucket_lo(key);
        const unsigned __int128 nx = bucket_hi(key), hi = nx < top + 1 ? nx : top + 1;   // values a search sees: [lo, hi)
        if (lo >= hi) continue;
        int a = 0, b = 0;
        for (int x = 0; x < 2; ++x) {   // first rows reaching lo and hi - 1
            const unsigned __int128 t = x == 0 ? lo : hi - 1;
            int l = 0, r = NH;
            while (l < r) {
                const int mid = (l + r) / 2;
                if (col[mid] < t) l = mid + 1;
                else r = mid;
            }
            (x == 0 ? a : b) = l;
        }
        most = b - a + 1 > most ? b - a + 1 : most;
    }
    int h = 0;
    while ((1 << h) < most) ++h;
    return h;
}
static_assert(bucket_steps(64, 7, 2) == 2 && bucket_steps(64, 7, 15) == 1 && bucket_steps(32, 7, 3) == 2,
              "bucket steps of the 7-level columns");

// With 64-bit ranks the searches over columns 0 .. kNarrow-1 run in 32 bits:
// C(n, k) < 2^32 for every n <= 255 and k <= 4, and at the search over
// column k the state q is at most C(y, k) for the previous cut's complement
// y <= 254 (or C(L-1, k) at the first cut), so q, every probe and the rank
// left fit 32 bits there.  Those columns are kept in LDS as uint32 (half the
// bytes per probe); the others as R.
template <int S, typename R>
__host__ __device__ constexpr int narrow_cols() {
    return sizeof(R) == 8 ? (S < 5 ? S : 5) : 0;
}

// One cut's search for NI candidates over column c of type V (R or uint32)
// with its bucket table.  q is the decode state (see decode_start): the cut's
// complement y = L - 1 - cut is the largest y with C(y, c) <= q - 1, so
// n = y + 1 is the smallest n with C(n, c) >= q; then q <- q - C(n - 1, c)
// and the cut is L - n.
template <typename V, typename R, int HS, int NI>
__device__ __forceinline__ void search_cut(const KParams &p, const V *col, const uint8_t *tab, R (&q)[NI],
                                           uint32_t (&cut)[NI]) {
    static_assert(HS <= kBucketStepsMax, "a bucket spans at most 2^3 rows (the padding)");
    V Q[NI];
    uint32_t n0[NI], t[NI];
#pragma unroll
    for (int u = 0; u < NI; ++u) Q[u] = (V)q[u];
#pragma unroll
    for (int u = 0; u < NI; ++u) {
        n0[u] = tab[bucket_key(Q[u]) - kBucketBias];
        t[u] = 0;
    }
    // halving d probes the last row of the left half of rows
    // [n0 + t 2^(HS-d), n0 + (t + 1) 2^(HS-d))
#pragma unroll
    for (int d = 0; d < HS; ++d) {
#pragma unroll
        for (int u = 0; u < NI; ++u) {
            const V probe = col[n0[u] + (t[u] << (HS - d)) + (1u << (HS - 1 - d)) - 1u];
            t[u] = d == 0 ? (uint32_t)(probe < Q[u]) : tree_step(t[u], probe, Q[u]);   // (no register to clear first)
        }
    }
#pragma unroll
    for (int u = 0; u < NI; ++u) {
        const uint32_t n = n0[u] + t[u];   // at least 1: C(0, c) = 0 < q
        q[u] = (R)(Q[u] - col[n - 1]);
        cut[u] = p.L - n;
    }
}

// LDS image of Pascal columns C0 .. C1, the ones a kernel searches (cut j
// searches column S - j, so no search reads columns 0 and 1): the wide
// columns among them (NN and up, NN = narrow_cols) as R, then the narrow ones
// as uint32, NP rows each, then their bucket tables in column order.
template <int S, typename R, int H, int C0 = 2, int C1 = S - 1>
struct Pascal {
    static constexpr uint32_t NH = 1u << H, NP = NH + kBucketPad;
    static constexpr int NN = narrow_cols<S, R>();
    static constexpr int WL = C0 > NN ? C0 : NN;              // first wide column held
    static constexpr int NWC = C1 >= WL ? C1 - WL + 1 : 0;   // wide columns held
    static constexpr int NHI = C1 < NN - 1 ? C1 : NN - 1;    // last narrow column held
    static constexpr int NNC = NHI >= C0 ? NHI - C0 + 1 : 0; // narrow columns held
    static constexpr size_t kWideBytes = (size_t)NWC * NP * sizeof(R), kNarrowBytes = (size_t)NNC * NP * 4;
    // bucket tables: the narrow columns' first, then the wide ones'
    static constexpr uint32_t kTabN = bucket_tab_bytes(32), kTabW = bucket_tab_bytes(8 * (int)sizeof(R));
    static constexpr size_t bytes() { return kWideBytes + kNarrowBytes + (size_t)NNC * kTabN + (size_t)NWC * kTabW; }
    const unsigned char *base;
    __device__ __forceinline__ explicit Pascal(const void *b) : base(reinterpret_cast<const unsigned char *>(b)) {}
    template <int c>
    __device__ __forceinline__ const auto *col() const {
        if constexpr (c >= NN) return reinterpret_cast<const R *>(base + (size_t)(c - WL) * NP * sizeof(R));
        else return reinterpret_cast<const uint32_t *>(base + kWideBytes + (size_t)(c - C0) * NP * 4);
    }
    template <int c>
    __device__ __forceinline__ const uint8_t *tab() const {
        if constexpr (c >= NN) return base + kWideBytes + kNarrowBytes + (size_t)NNC * kTabN + (size_t)(c - WL) * kTabW;
        else return base + kWideBytes + kNarrowBytes + (size_t)(c - C0) * kTabN;
    }
    // the search of a cut over column c, for NI candidates
    template <int c, int NI>
    __device__ __forceinline__ void search(const KParams &p, R (&q)[NI], uint32_t (&cut)[NI]) const {
        static_assert(c >= C0 && c <= C1, "column outside the window");
        using V = typename std::conditional<(c >= NN), R, uint32_t>::type;
        search_cut<V, R, bucket_steps(8 * (int)sizeof(V), H, c)>(p, col<c>(), tab<c>(), q, cut);
    }
};

// f(integral_constant<int, i>) for i = A .. B-1 (a loop whose index is a
// constant expression)
template <int A, int B, typename F>
__device__ __forceinline__ void static_for(F &&f) {
    if constexpr (A < B) {
        f(std::integral_constant<int, A>{});
        static_for<A + 1, B>(f);
    }
}

// The decode state of lexicographic rank r: q = C(L-1, S-1) - r, which is
// one more than the co-lexicographic rank of the cut complements
// y_j = L - 1 - c_j (so q >= 1 for every valid rank).
template <typename R>
__device__ __forceinline__ R decode_start(const KParams &p, R r) {
    return (R)(p.n_comp - (uint64_t)r);
}

// The checks of kIlp list entries whose ranks and assignment indices were all
// loaded before: candidate() on one after the other waits for memory kIlp
// times (early stop on 2^26 candidates at S = 8: 587 us so, 491 us together).
template <typename R>
__device__ __forceinline__ void check_entries(const KParams &p, const uint64_t (&rank)[kIlp], const uint32_t (&idx)[kIlp],
                                              const bool (&act)[kIlp], bool (&ok)[kIlp], uint32_t (&asg)[kIlp],
                                              R (&r)[kIlp]) {
#pragma unroll
    for (int u = 0; u < kIlp; ++u) {
        const bool in = rank[u] < p.n_comp && idx[u] < p.A;
        r[u] = in ? (R)rank[u] : (R)0;
        asg[u] = in ? idx[u] : 0u;
        ok[u] = in & act[u];
    }
}

// Candidates base + u * stride + lane (u < kIlp) of the piece, base the same
// for every lane of the wave (a list is then read at a scalar base and a
// 32-bit lane offset): call positions, ranks and assignment indices (0 where
// out of range: ok = false).  Lanes past the end take the last candidate,
// act = ok = false.
template <typename R>
__device__ __forceinline__ void load_candidates(const KParams &p, uint32_t base, uint32_t stride, uint32_t lane,
                                                bool (&act)[kIlp], bool (&ok)[kIlp], uint32_t (&pos)[kIlp],
                                                uint32_t (&asg)[kIlp], R (&r)[kIlp]) {
    const uint32_t n = (uint32_t)p.n_i, first_i = (uint32_t)p.first_i;
    uint32_t wb[kIlp], l[kIlp];
#pragma unroll
    for (int u = 0; u < kIlp; ++u) {
        const uint32_t i = base + u * stride;
        wb[u] = min(i, n - 1);
        l[u] = min(lane, n - 1 - wb[u]);
        wb[u] += first_i;
        act[u] = i + lane < n;
        pos[u] = wb[u] + l[u];
    }
    if (p.comp_rank) {
        uint64_t rank[kIlp];
        uint32_t idx[kIlp];
#pragma unroll
        for (int u = 0; u < kIlp; ++u)
            rank[u] = *reinterpret_cast<const uint64_t *>(reinterpret_cast<const char *>(p.comp_rank + wb[u]) + (l[u] << 3));
        if (p.assign_idx) {
#pragma unroll
            for (int u = 0; u < kIlp; ++u)
                idx[u] = *reinterpret_cast<const uint32_t *>(reinterpret_cast<const char *>(p.assign_idx + wb[u]) + (l[u] << 2));
        } else {
#pragma unroll
            for (int u = 0; u < kIlp; ++u) idx[u] = 0u;
        }
        check_entries<R>(p, rank, idx, act, ok, asg, r);
    } else {
#pragma unroll
        for (int u = 0; u < kIlp; ++u) ok[u] = candidate<R>(p, pos[u], r[u], asg[u]) & act[u];
    }
}

// The same at any call positions pos (valid positions also for lanes with
// act = false).
template <typename R>
__device__ __forceinline__ void gather_candidates(const KParams &p, const uint32_t (&pos)[kIlp], const bool (&act)[kIlp],
                                                  bool (&ok)[kIlp], uint32_t (&asg)[kIlp], R (&r)[kIlp]) {
    if (p.comp_rank) {
        uint64_t rank[kIlp];
        uint32_t idx[kIlp];
#pragma unroll
        for (int u = 0; u < kIlp; ++u) rank[u] = p.comp_rank[pos[u]];
#pragma unroll
        for (int u = 0; u < kIlp; ++u) idx[u] = p.assign_idx ? p.assign_idx[pos[u]] : 0u;
        check_entries<R>(p, rank, idx, act, ok, asg, r);
    } else {
#pragma unroll
        for (int u = 0; u < kIlp; ++u) ok[u] = candidate<R>(p, pos[u], r[u], asg[u]) & act[u];
    }
}

template <int S, typename R, int H, typename PC>
__device__ __forceinline__ void decode_ilp(const KParams &p, const PC &pc, uint32_t base,
                                           uint32_t stride, bool (&act)[kIlp], bool (&ok)[kIlp],
                                           uint32_t (&asg)[kIlp], uint32_t (&w)[kIlp][Codes<S>::kWords]) {
    constexpr int NW = Codes<S>::kWords;
    R q[kIlp];
    uint32_t pos[kIlp];
    load_candidates<R>(p, base, stride, threadIdx.x & 63, act, ok, pos, asg, q);
#pragma unroll
    for (int u = 0; u < kIlp; ++u) {
        q[u] = decode_start<R>(p, q[u]);
#pragma unroll
        for (int k = 0; k < NW; ++k) w[u][k] = 0;
    }
    // the searches, cut by cut, interleaved over the kIlp candidates; each
    // cut goes straight into its byte of the code words (cut j searches
    // column S - j)
    static_for<1, S - 1>([&](auto jc) {
        constexpr int j = decltype(jc)::value;
        uint32_t cut[kIlp];
        pc.template search<S - j>(p, q, cut);
#pragma unroll
        for (int u = 0; u < kIlp; ++u) w[u][(j - 1) / 4] |= cut[u] << (8 * ((j - 1) % 4));
    });
    if (S >= 2) {
#pragma unroll
        for (int u = 0; u < kIlp; ++u) w[u][(S - 2) / 4] |= (p.L - (uint32_t)q[u]) << (8 * ((S - 2) % 4));
    }
#pragma unroll
    for (int u = 0; u < kIlp; ++u) {
        if (S == 1) w[u][0] = 1u;
        if (!ok[u]) {
#pragma unroll
            for (int k = 0; k < NW; ++k) w[u][k] = 0u;
        }
    }
}

// Searches of cuts J0+1 .. J1 (J1 <= S - 1) of kIlp candidates from the
// decode state q after cut J0; cut S - 1, the last, needs no search (with
// one cut left, C(y, 1) = y: its complement is q - 1, so c_{S-1} = L - q).
template <int S, typename R, int H, int J0, int J1, typename PC>
__device__ __forceinline__ void decode_range(const KParams &p, const PC &pc, R (&q)[kIlp],
                                             uint32_t (&cut)[kIlp][S + 1]) {
    constexpr int JS = J1 < S - 2 ? J1 : S - 2;   // cuts found by a search
    static_for<J0 + 1, JS + 1>([&](auto jc) {
        constexpr int j = decltype(jc)::value;
        uint32_t cj[kIlp];
        pc.template search<S - j>(p, q, cj);
#pragma unroll
        for (int u = 0; u < kIlp; ++u) cut[u][j] = cj[u];
    });
    if (J1 == S - 1 && S >= 2) {
#pragma unroll
        for (int u = 0; u < kIlp; ++u) cut[u][S - 1] = p.L - (uint32_t)q[u];
    }
}

// Cuts c_1 .. c_J (J <= S - 1) of kIlp candidates at call positions pos
// (valid positions also for inactive lanes) into cut[u][0 .. J], with
// c_0 = 0 and c_S = L; q is left as decode_range needs it to go on.
// Invalid (rank, assignment) pairs get ok = false.
template <int S, typename R, int H, int J, typename PC>
__device__ __forceinline__ void decode_cuts(const KParams &p, const PC &pc,
                                            const uint32_t (&pos)[kIlp], const bool (&act)[kIlp],
                                            bool (&ok)[kIlp], uint32_t (&asg)[kIlp], R (&q)[kIlp],
                                            uint32_t (&cut)[kIlp][S + 1]) {
    gather_candidates<R>(p, pos, act, ok, asg, q);
#pragma unroll
    for (int u = 0; u < kIlp; ++u) {
        q[u] = decode_start<R>(p, q[u]);
        cut[u][0] = 0;
        cut[u][S] = p.L;
    }
    decode_range<S, R, H, 0, J>(p, pc, q, cut);
}

template <int S, typename R, int H, typename PC>
__device__ __forceinline__ void decode_batch(const KParams &p, const PC &pc, uint32_t base,
                                             uint32_t stride, bool &bad) {
    constexpr int NW = Codes<S>::kWords;
    bool act[kIlp], ok[kIlp];
    uint32_t asg[kIlp], w[kIlp][NW];
    decode_ilp<S, R, H>(p, pc, __builtin_amdgcn_readfirstlane(base), stride, act, ok, asg, w);
#pragma unroll
    for (int u = 0; u < kIlp; ++u) {
        const uint32_t i = base + u * stride;
        bad |= act[u] && !ok[u];
        if (act[u]) {
#pragma unroll
            for (int k = 0; k < NW; ++k) p.codes[k * (uint32_t)p.ccap + i] = w[u][k];
        }
    }
}

// Columns C0 .. C1 of the Pascal table into LDS (layout of
// Pascal<S, R, H, C0, C1>): 2^H rows each, then the padding rows of the
// type's largest value (so that the columns stay sorted), then the host's
// bucket tables of those columns.  Narrow columns saturate at 2^32 - 1 (no
// value of a column below 5 reaches it for n <= 255).
template <int S, typename R, int H, int C0 = 2, int C1 = S - 1, int NT = kBlock>
__device__ __forceinline__ void pascal_tables(const KParams &p, void *lds) {
    using PC = Pascal<S, R, H, C0, C1>;
    constexpr uint32_t NH = PC::NH, NP = PC::NP, NC = C1 >= C0 ? (uint32_t)(C1 - C0 + 1) : 0u;
    unsigned char *b = reinterpret_cast<unsigned char *>(lds);
    R *ws = reinterpret_cast<R *>(b);
    uint32_t *ns = reinterpret_cast<uint32_t *>(b + PC::kWideBytes);
    const R *gb = reinterpret_cast<const R *>(p.binom);
    for (uint32_t e = threadIdx.x; e < NC * NP; e += NT) {
        const uint32_t k = C0 + e / NP, i = e % NP;
        const R v = i < NH ? gb[k * kNB + i] : ~(R)0;
        if ((int)k >= PC::NN) ws[(k - PC::WL) * NP + i] = v;
        else ns[(k - C0) * NP + i] = v > (R)0xFFFFFFFFu ? 0xFFFFFFFFu : (uint32_t)v;
    }
    uint4 *lt = reinterpret_cast<uint4 *>(b + PC::kWideBytes + PC::kNarrowBytes);
    constexpr uint32_t n16 = PC::kTabN / 16, w16 = PC::kTabW / 16;
    for (uint32_t e = threadIdx.x; e < PC::NNC * n16; e += NT)
        lt[e] = reinterpret_cast<const uint4 *>(p.btab + (size_t)(C0 + e / n16) * kBucketTab)[e % n16];
    for (uint32_t e = threadIdx.x; e < PC::NWC * w16; e += NT)
        lt[PC::NNC * n16 + e] = reinterpret_cast<const uint4 *>(p.btab + (size_t)(PC::WL + e / w16) * kBucketTab)[e % w16];
}

// LDS bytes of Pascal columns C0 .. C1 with their bucket tables
template <int S, typename R, int C0 = 2, int C1 = S - 1>
__host__ __device__ constexpr size_t pascal_bytes(uint32_t L) {
    switch (decode_levels(L)) {
    case 8: return Pascal<S, R, 8, C0, C1>::bytes();
    case 7: return Pascal<S, R, 7, C0, C1>::bytes();
    case 6: return Pascal<S, R, 6, C0, C1>::bytes();
    default: return Pascal<S, R, 5, C0, C1>::bytes();
    }
}

// Range mode with one assignment: candidate i of the chunk is composition
// rank first + first_i + i, so consecutive candidates are consecutive
// ranks.  A lane takes kIlp consecutive candidates: it unranks the first
// (one search per cut) and steps to the others by the lexicographic
// successor, in which the last cut that can still grow (cut j may reach
// L - S + j) grows by one and the cuts after it follow it at distance 1.
// The lane's kIlp code words of one word index are contiguous: one 16-byte
// store (the code rows hold a multiple of 4 words).
template <int S>
__device__ __forceinline__ void next_cuts(uint32_t L, uint32_t (&c)[S + 1]) {
    // js = the last cut that can grow, b = c_js + 1 - js (no register index
    // is dynamic: both are selected in the scan)
    uint32_t js = 0, b = 1;
#pragma unroll
    for (int j = 1; j <= S - 1; ++j) {
        const bool grow = c[j] < L - S + j;
        js = grow ? (uint32_t)j : js;
        b = grow ? c[j] + 1 - j : b;
    }
#pragma unroll
    for (int m = 1; m <= S - 1; ++m) c[m] = (uint32_t)m < js ? c[m] : b + m;
}

template <int S, typename R, int H, typename PC>
__device__ __forceinline__ void decode_succ_words(const KParams &p, const PC &pc, uint32_t base,
                                                  uint32_t (&w)[kIlp][Codes<S>::kWords], bool &bad) {
    const uint64_t rank0 = p.first + (uint32_t)p.first_i + base;
    R q[1] = {decode_start<R>(p, (R)(rank0 < p.n_comp ? rank0 : 0))};
    uint32_t c[S + 1];
    c[0] = 0;
    c[S] = p.L;
    static_for<1, S - 1>([&](auto jc) {
        constexpr int j = decltype(jc)::value;
        uint32_t cj[1];
        pc.template search<S - j>(p, q, cj);
        c[j] = cj[0];
    });
    if (S >= 2) c[S - 1] = p.L - (uint32_t)q[0];
#pragma unroll
    for (int u = 0; u < kIlp; ++u) {
        if (u > 0) next_cuts<S>(p.L, c);
        const bool act = base + u < (uint32_t)p.n_i;
        const bool ok = rank0 + u < p.n_comp;
        bad |= act && !ok;
        pack_cuts<S>(c, ok, w[u]);
    }
}

template <int S, typename R, int H, typename PC>
__device__ __forceinline__ void decode_succ(const KParams &p, const PC &pc, uint32_t base, bool &bad) {
    static_assert(kIlp == 4, "one 16-byte store per code word");
    constexpr int NW = Codes<S>::kWords;
    uint32_t w[kIlp][NW];
    decode_succ_words<S, R, H>(p, pc, base, w, bad);
    const uint32_t ccap = (uint32_t)p.ccap;
#pragma unroll
    for (int k = 0; k < NW; ++k)
        *reinterpret_cast<uint4 *>(p.codes + k * ccap + base) = make_uint4(w[0][k], w[1][k], w[2][k], w[3][k]);
}

template <int S, typename R, int H>
__device__ __forceinline__ void decode_all(const KParams &p, void *lds, bool &bad) {
    pascal_tables<S, R, H>(p, lds);
    __syncthreads();
    const Pascal<S, R, H> pc(lds);
    if (!p.comp_rank && p.A == 1) {
        const uint32_t stride = gridDim.x * kBlock * kIlp, n_i = (uint32_t)p.n_i;
        for (uint32_t base = (blockIdx.x * kBlock + threadIdx.x) * kIlp; base < n_i; base += stride)
            decode_succ<S, R, H>(p, pc, base, bad);
        return;
    }
    // 32-bit positions: a chunk holds at most 2^26 candidates, a call fewer than 2^32
    const uint32_t stride = gridDim.x * kBlock, n_i = (uint32_t)p.n_i;
    for (uint32_t base = blockIdx.x * kBlock + threadIdx.x; base < n_i; base += kIlp * stride)
        decode_batch<S, R, H>(p, pc, base, stride, bad);
}

template <int S, typename R>
__global__ __launch_bounds__(kBlock) void decode_kernel(KParams p) {
    extern __shared__ __align__(16) unsigned char smem[];
    R *lds = reinterpret_cast<R *>(smem);
    bool bad = false;
    switch (decode_levels(p.L)) {
    case 8: decode_all<S, R, 8>(p, lds, bad); break;
    case 7: decode_all<S, R, 7>(p, lds, bad); break;
    case 6: decode_all<S, R, 6>(p, lds, bad); break;
    default: decode_all<S, R, 5>(p, lds, bad); break;
    }
    if (bad) atomicOr(p.err, 1u);
}

// Outputs of a wave's candidates gi (one per lane, 64 aligned consecutive
// positions: chunks start at multiples of 64): makespans of the lanes with
// `write` set and the packed feasibility bits.  They are read back only by
// the host or the argmin pass: stream them past the caches.
__device__ __forceinline__ void write_outputs(const KParams &p, uint32_t gi, bool write, uint32_t T, bool feas) {
    if (write && p.makespan_out) __builtin_nontemporal_store(T, p.makespan_out + gi);
    if (p.feas_bits_out) {
        const unsigned long long bits = __ballot(feas);
        const uint32_t w0 = (gi - (threadIdx.x & 63)) >> 5, nwords = (uint32_t)p.nwords;
        if ((threadIdx.x & 63) == 0 && w0 < nwords) __builtin_nontemporal_store((uint32_t)bits, p.feas_bits_out + w0);
        if ((threadIdx.x & 63) == 32 && w0 + 1 < nwords) __builtin_nontemporal_store((uint32_t)(bits >> 32), p.feas_bits_out + w0 + 1);
    }
}

// The same for a wave whose lanes hold kIlp consecutive candidates each
// (256 in all, from base = lane * kIlp on; gi their position in the call):
// makespans as one 16-byte store where the caller's array allows it, and the
// lanes' four feasibility bits joined to words of eight lanes.
__device__ __forceinline__ void write_quad(const KParams &p, uint32_t gi, uint32_t base, uint32_t n_i,
                                           const uint32_t (&T)[kIlp], uint32_t nib) {
    static_assert(kIlp == 4, "one 16-byte store");
    if (p.makespan_out) {
        uint32_t *o = p.makespan_out + gi;
        if (((uint64_t)(uintptr_t)p.makespan_out & 15u) == 0 && base + kIlp <= n_i) {   // (gi is a multiple of 4)
            typedef uint32_t v4 __attribute__((ext_vector_type(4)));
            __builtin_nontemporal_store((v4){T[0], T[1], T[2], T[3]}, reinterpret_cast<v4 *>(o));
        } else {
#pragma unroll
            for (int u = 0; u < kIlp; ++u)
                if (base + u < n_i) __builtin_nontemporal_store(T[u], o + u);
        }
    }
    if (p.feas_bits_out) {
        uint32_t v = nib << (4 * (threadIdx.x & 7));
#pragma unroll
        for (int o = 1; o < 8; o <<= 1) v |= __shfl_xor(v, o, 64);
        const uint32_t word = gi >> 5;
        if ((threadIdx.x & 7) == 0 && word < (uint32_t)p.nwords && base < n_i) __builtin_nontemporal_store(v, p.feas_bits_out + word);
    }
}

// (a2)-(a4), (a6) for the chunk by the recurrence alone (problems with too
// few micro-batches for the closed form, and the slot tables): stage weights
// from the cut codes, memory check, the DP and the reduction.  SCH: Eager
// 1F1B; TAB: the slot table instead of the compiled schedule.
template <int S, bool AR, bool SCH, bool TAB>
__global__ __launch_bounds__(kBlock) void eval_kernel(KParams p) {
    extern __shared__ __align__(16) unsigned char smem[];
    const Ent tab = entry_tables(p, smem);
    const Comm<S> comm = load_comm<S>(p);
    constexpr int NW = Codes<S>::kWords;
    unsigned long long best = ~0ull;
    // 32-bit positions: a chunk holds at most 2^26 candidates, a call fewer
    // than 2^32, and the code buffer fewer than 2^32 words (fewer scalar
    // registers than 64-bit ones, which this kernel is short of)
    const uint32_t stride = gridDim.x * kBlock, n_i = (uint32_t)p.n_i, ccap = (uint32_t)p.ccap;
    const uint32_t first_i = (uint32_t)p.first_i;
    // every wave runs the same trip count so that ballots see whole waves
    const uint32_t span = (n_i + stride - 1) / stride;
    uint32_t i = blockIdx.x * kBlock + threadIdx.x;
    for (uint32_t it = 0; it < span; ++it, i += stride) {
        const bool active = i < n_i;
        const uint32_t gi = first_i + i;   // index within the call
        uint32_t w[NW];
#pragma unroll
        for (int k = 0; k < NW; ++k) w[k] = active ? p.codes[k * ccap + i] : 0u;
        uint32_t cut[S + 1], to[S], F[S], B[S], Y[S];
        const bool ok = unpack_cuts<S>(w, p.L, cut);
        const uint32_t a = ok ? assign_of(p, gi) : 0u;
        decode_toff<S>(p, tab, a, to);
        const bool feas = stage_weights<S>(p, tab, cut, to, F, B) && ok && active;
        uint32_t T;
        if constexpr (TAB) {
            if constexpr (SCH) dp_sched<S>(p, F, B, comm, Y);
            else dp_table<S>(p, F, B, comm, Y);
            T = end_time<S, AR>(p, tab, Y, comm, w, a);
        } else if constexpr (SCH) {
            dp_eager<S>(p.M, F, B, comm, Y);
            T = end_time<S, AR>(p, tab, Y, comm, w, a);
        } else {
            dp_prologue<S>(Y, F, B, comm, p.g24 != 0);
            for (uint32_t k = S; k < p.M; ++k) dp_iter<S>(Y, F, B, comm);
            T = dp_end<S, AR>(p, tab, Y, F, B, comm, w, a);
        }
        if (!ok) T = 0xFFFFFFFFu;
        write_outputs(p, gi, active, T, feas);
        if (active) {
            const unsigned long long key = make_key(feas, T, gi);
            best = key < best ? key : best;
        }
    }
    block_min_and_finish(best, p.acc, p.done, p.result, nullptr, true, p.accumulate, nullptr, 0, host_out(p));
}

// (a2)-(a4), (a6) for a chunk of an Eager 1F1B problem whose candidates mostly
// have no closed-form proof: the recurrence for every candidate, in a cascade.
// A lane whose steady state has not settled by pair p.lvl_k[0] is queued for
// resume_kernel.  Held to 128 VGPRs (4 waves a SIMD instead of 3 at S = 16),
// where full_kernel has 2: with none of the candidates proven (transfers of
// 1-5 layers) 2^24 of 16 stages and 128 micro-batches take 3.28 ms so, 4.15
// with the closed form and full_kernel; 2^22 of 300 and 1,000 micro-batches
// 1.14 and 1.49 against 1.59 and 2.84.
template <int S, bool AR>
__global__ __launch_bounds__(kBlock) __attribute__((amdgpu_waves_per_eu(4, 8))) void cascade_kernel(KParams p) {
    extern __shared__ __align__(16) unsigned char smem[];
    const Ent tab = entry_tables(p, smem);
    const Comm<S> comm = load_comm<S>(p);
    constexpr int NW = Codes<S>::kWords, NX = 2 * S;
    unsigned long long best = ~0ull;
    // 32-bit positions and trip counts as in eval_kernel
    const uint32_t stride = gridDim.x * kBlock, n_i = (uint32_t)p.n_i, ccap = (uint32_t)p.ccap;
    const uint32_t first_i = (uint32_t)p.first_i;
    const uint32_t span = (n_i + stride - 1) / stride;
    const uint32_t nit = p.M - 2 * S + 1, k1 = p.nlevels ? p.lvl_k[0] : nit;
    __shared__ unsigned int nq;
    if (threadIdx.x == 0) nq = 0;
    __syncthreads();
    uint32_t i = blockIdx.x * kBlock + threadIdx.x;
    for (uint32_t it = 0; it < span; ++it, i += stride) {
        const bool active = i < n_i;
        const uint32_t gi = first_i + i;
        uint32_t w[NW];
#pragma unroll
        for (int k = 0; k < NW; ++k) w[k] = active ? p.codes[k * ccap + i] : 0u;
        uint32_t cut[S + 1], to[S], F[S], B[S], Y[S], Fn[S], Fp[S];
        const bool ok = unpack_cuts<S>(w, p.L, cut);
        const uint32_t a = ok ? assign_of(p, gi) : 0u;
        decode_toff<S>(p, tab, a, to);
        const bool feas = stage_weights<S>(p, tab, cut, to, F, B) && ok && active;
        eager_prologue<S>(Y, Fn, Fp, F, B, comm);
        const bool done_here = eager_advance<S>(Y, Fn, Fp, F, B, comm, 0, k1, nit);
        if (p.nlevels) {
            uint32_t X[NX];
            eager_pack<S>(Y, Fn, Fp, X);
            enqueue<S, NX>(p, 0, &nq, !done_here && active && ok, gi, w, -1, X);
        }
        eager_epilogue<S>(Y, Fn, Fp, F, B, comm);
        uint32_t T = end_time<S, AR>(p, tab, Y, comm, w, a);
        if (!ok) T = 0xFFFFFFFFu;
        const bool write = active && (done_here || !ok);
        write_outputs(p, gi, write, T, feas);
        if (write) {
            const unsigned long long key = make_key(feas, T, gi);
            best = key < best ? key : best;
        }
    }
    if (p.nlevels) {
        __syncthreads();
        if (threadIdx.x == 0) p.qcount[blockIdx.x] = nq;   // entries for level 1
    }
    block_min_and_finish(best, p.acc, p.done, p.result, nullptr, p.nlevels == 0, p.accumulate, nullptr, 0, host_out(p));
}

// Level `lvl` of that cascade: the queued lanes from steady pair
// p.lvl_k[lvl-1] to p.lvl_k[lvl] (the end at the last level).  Block b takes
// the segment that block b of the level before wrote.
template <int S, bool AR>
__global__ __launch_bounds__(kBlock) void resume_kernel(KParams p, uint32_t lvl) {
    extern __shared__ __align__(16) unsigned char smem[];
    const Ent tab = entry_tables(p, smem);
    const Comm<S> comm = load_comm<S>(p);
    constexpr int NW = Codes<S>::kWords, NX = 2 * S;
    const uint32_t nit = p.M - 2 * S + 1;
    const uint32_t k0 = p.lvl_k[lvl - 1];
    const uint32_t k1 = lvl < p.nlevels ? p.lvl_k[lvl] : nit;
    const uint32_t n = p.qcount[(uint64_t)(lvl - 1) * p.nseg + blockIdx.x];
    const QueueView<S> qin(p, (lvl - 1) & 1);
    __shared__ unsigned int nq;
    if (threadIdx.x == 0) nq = 0;
    __syncthreads();
    unsigned long long best = ~0ull;
    const uint32_t span = (n + kBlock - 1) / kBlock;
    // 32-bit word offsets: a queue holds fewer than 2^32 words
    const uint32_t seg = blockIdx.x * (uint32_t)p.seg_cap, qcap = (uint32_t)p.qcap;
    for (uint32_t it = 0; it < span; ++it) {
        const uint32_t q = seg + it * kBlock + threadIdx.x;
        const bool active = it * kBlock + threadIdx.x < n;
        const uint32_t i = active ? qin.idx[q] : 0u;
        uint32_t w[NW], cut[S + 1], to[S], F[S], B[S], X[NX], Y[S], Fn[S], Fp[S];
#pragma unroll
        for (int k = 0; k < NW; ++k) w[k] = active ? qin.codes[k * qcap + q] : 0u;
#pragma unroll
        for (int s = 0; s < NX; ++s) X[s] = active ? qin.Y[s * qcap + q] : 0u;
        unpack_cuts<S>(w, p.L, cut);   // (a queued entry's codes were valid when it was queued)
        const uint32_t a = !active ? 0u : p.qasg ? qin.asg[q] : assign_of(p, i);
        decode_toff<S>(p, tab, a, to);
        const bool feas = stage_weights<S>(p, tab, cut, to, F, B);
        eager_unpack<S>(X, Y, Fn, Fp);
        const bool settled = eager_advance<S>(Y, Fn, Fp, F, B, comm, k0, k1, nit);
        if (lvl < p.nlevels) {
            eager_pack<S>(Y, Fn, Fp, X);
            enqueue<S, NX>(p, lvl & 1, &nq, active && !settled, i, w, a, X);
        }
        eager_epilogue<S>(Y, Fn, Fp, F, B, comm);
        const uint32_t T = end_time<S, AR>(p, tab, Y, comm, w, a);
        if (active && settled) {
            // scattered one-word writes: the nontemporal hint keeps them out of L2 write-allocate
            if (p.makespan_out) __builtin_nontemporal_store(T, p.makespan_out + i);
            const unsigned long long key = make_key(feas, T, i);
            best = key < best ? key : best;
        }
    }
    if (lvl < p.nlevels) {
        __syncthreads();
        if (threadIdx.x == 0) p.qcount[(uint64_t)lvl * p.nseg + blockIdx.x] = nq;
    }
    block_min_and_finish(best, p.acc, p.done, p.result, nullptr, lvl == p.nlevels, p.accumulate, nullptr, 0, host_out(p));
}

// The list of candidates without a closed-form proof, arrays of ccap
// entries: call position, cut codes, assignment index.  Block b of
// closed_kernel fills slots [b * seg_cap, (b + 1) * seg_cap) and writes its
// count to fcount[b].
template <int S>
struct FullList {
    uint32_t *pos, *w, *asg;
    __device__ __forceinline__ explicit FullList(const KParams &p)
        : pos(p.flist), w(p.flist + p.ccap), asg(p.flist + (1 + Codes<S>::kWords) * p.ccap) {}
};

// One candidate per lane of a wave from its cut codes w (all zero: invalid),
// assignment a and position gi: stage weights, memory check, closed-form
// makespan (poseidon_closed.h).  Lanes whose value is not proven go to the
// block's segment of the list that full_kernel evaluates by the recurrence.
// Returns whether T is the candidate's makespan; all lanes call it.
template <int S, bool AR, bool SCH, bool U24>
__device__ __forceinline__ bool closed_one(const KParams &p, const Ent &tab, uint32_t seg, unsigned int *nq,
                                           bool active, uint32_t gi, uint32_t a,
                                           const uint32_t (&w)[Codes<S>::kWords], uint32_t &T, bool &feas) {
    constexpr int NW = Codes<S>::kWords;
    uint32_t cut[S + 1], to[S], F[S], B[S], D[S];
    const bool ok = unpack_cuts<S>(w, p.L, cut);
    decode_toff<S>(p, tab, a, to);
    feas = stage_weights<S>(p, tab, cut, to, F, B) && ok && active;
    if (AR) stage_allreduce<S>(p, tab, cut, to, D);
    const bool proven = closed_form<S, SCH, AR, U24>(p, F, B, D, T) || !ok;
    if (!ok) T = 0xFFFFFFFFu;
    const unsigned long long m = __ballot(active && !proven);
    if (m) {
        const unsigned int lane = threadIdx.x & 63;
        unsigned int base = 0;
        if (lane == 0) base = atomicAdd(nq, (unsigned int)__popcll(m));
        base = __shfl(base, 0, 64);
        if (active && !proven) {
            const uint32_t slot = seg + base + __popcll(lane ? (m & ((1ull << lane) - 1ull)) : 0ull);
            const FullList<S> l(p);
            l.pos[slot] = gi;
#pragma unroll
            for (int k = 0; k < NW; ++k) l.w[k * (uint32_t)p.ccap + slot] = w[k];
            l.asg[slot] = a;
        }
    }
    return active && proven;
}

// (a1)-(a4), (a6) for the chunk in one pass: every lane unranks kIlp
// candidates together (the decode's LDS chains overlap) and takes the closed
// form of one after the other from their packed cuts, which never leave its
// registers.  VALU-bound (79-89 % issue): about 26 operations a stage for
// the weights and the closed form and 15 a search, against 5 a stage for
// every one of the recurrence's steady iterations, at least S of them.
// 2^24 candidates of 16 stages: 401 us (decode 161 and closed form 346 as
// two kernels; decode 159 and the recurrence 1091 + 510 before); 2^26 of 8
// stages 776 us (297 + 761; 307 + 1415 + 653); the exhaustive 8-stage range
// 599 us (131 + 593; 133 + 1175 + 416).
// LDS: the Pascal columns at offset 0 (a compile-time size), then the stage
// entries at a constant offset (it folds into the loads' immediates; static
// __shared__ variables would move both), then a few words.  The columns have
// 2^7 or 2^8 rows: the shorter forms of the decode kernel save little here.
// 512 threads share one copy of the tables.
constexpr int kFuseBlock = (int)kFuseThreads;
constexpr size_t kFuseTail = 128;   // wave minima, list counter
__host__ __device__ constexpr uint32_t fuse_levels(uint32_t L) { return L > 128 ? 8u : 7u; }

template <int S, typename R, bool AR, bool SCH, int H>
__device__ __forceinline__ void fused_all(const KParams &p, unsigned char *smem) {
    using PC = Pascal<S, R, H>;
    constexpr int NW = Codes<S>::kWords, NT = kFuseBlock;
    static_assert(PC::bytes() % 16 == 0, "entries follow the columns at 16 bytes");
    pascal_tables<S, R, H, 2, S - 1, NT>(p, smem);
    unsigned char *tail = smem + PC::bytes() + p.ent_lds;
    unsigned long long *part = reinterpret_cast<unsigned long long *>(tail);
    unsigned int *nq = reinterpret_cast<unsigned int *>(tail + NT / 64 * 8);
    if (threadIdx.x == 0) *nq = 0;
    const Ent tab = entry_tables<NT>(p, smem + PC::bytes());   // (its barrier publishes all of it)
    const PC pc(smem);
    const uint32_t n_i = (uint32_t)p.n_i, first_i = (uint32_t)p.first_i, lane = threadIdx.x & 63;
    const uint32_t seg = blockIdx.x * (uint32_t)p.seg_cap;
    unsigned long long best = ~0ull;
    bool bad = false;
    if (!p.comp_rank && p.A == 1) {
        // consecutive ranks: a lane takes kIlp of them, the first unranked,
        // the others by the lexicographic successor
        const uint32_t stride = gridDim.x * NT * kIlp;
        for (uint32_t wb = (blockIdx.x * NT + (threadIdx.x - lane)) * kIlp; wb < n_i; wb += stride) {   // (wave-uniform)
            const uint32_t base = wb + lane * kIlp;
            uint32_t w[kIlp][NW];
            decode_succ_words<S, R, H>(fresh_args(), pc, base, w, bad);
            uint32_t Tq[kIlp], nib = 0;
#pragma unroll
            for (int u = 0; u < kIlp; ++u) Tq[u] = 0;
#pragma unroll 1
            for (uint32_t u = 0; u < (uint32_t)kIlp; ++u) {
                uint32_t T;
                bool feas;
                const bool done = closed_one<S, AR, SCH, true>(fresh_args(), tab, seg, nq, base + u < n_i, first_i + base + u, 0u, w[0], T, feas);
                // (an unproven lane's value is overwritten by full_kernel, which runs after this one)
                nib |= (feas ? 1u : 0u) << u;
                if (done) {
                    const unsigned long long key = make_key(feas, T, first_i + base + u);
                    best = key < best ? key : best;
                }
                // the next candidate's words, and the values in order (no dynamic register index)
#pragma unroll
                for (int v = 0; v + 1 < kIlp; ++v) {
#pragma unroll
                    for (int k = 0; k < NW; ++k) w[v][k] = w[v + 1][k];
                    Tq[v] = Tq[v + 1];
                }
                Tq[kIlp - 1] = T;
            }
            write_quad(fresh_args(), first_i + base, base, n_i, Tq, nib);
        }
    } else {
        const uint32_t stride = gridDim.x * NT;
        const uint32_t wave0 = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6) * 64;
        for (uint32_t wb = blockIdx.x * NT + wave0; wb < n_i; wb += kIlp * stride) {   // (wave-uniform)
            bool act[kIlp], ok[kIlp];
            uint32_t asg[kIlp], w[kIlp][NW];
            decode_ilp<S, R, H>(fresh_args(), pc, wb, stride, act, ok, asg, w);
#pragma unroll
            for (int u = 0; u < kIlp; ++u) bad |= act[u] && !ok[u];
#pragma unroll 1
            for (uint32_t u = 0; u < (uint32_t)kIlp; ++u) {
                const uint32_t i = wb + u * stride + lane;
                if (wb + u * stride >= n_i) break;   // (wave-uniform)
                uint32_t T;
                bool feas;
                const KParams &q = fresh_args();
                const bool write = closed_one<S, AR, SCH, true>(q, tab, seg, nq, i < n_i, first_i + i, asg[0], w[0], T, feas);
                write_outputs(q, first_i + i, write, T, feas);
                if (write) {
                    const unsigned long long key = make_key(feas, T, first_i + i);
                    best = key < best ? key : best;
                }
#pragma unroll
                for (int v = 0; v + 1 < kIlp; ++v) {
#pragma unroll
                    for (int k = 0; k < NW; ++k) w[v][k] = w[v + 1][k];
                    asg[v] = asg[v + 1];
                }
            }
        }
    }
    if (bad) atomicOr(p.err, 1u);
    __syncthreads();
    if (threadIdx.x == 0) p.fcount[blockIdx.x] = *nq;
    block_min<NT>(best, p.acc, part);
}

// (128 VGPRs: two blocks of eight waves a CU at S = 16.  With all-reduce times
// the drain keeps A, B and D of every stage, and at S = 16 70 registers, Eager
// 1F1B 49, go to scratch; without, and up to S = 13 with them, none)
template <int S, typename R, bool AR, bool SCH>
__global__ __launch_bounds__(kFuseBlock) __attribute__((amdgpu_waves_per_eu(4, 8))) void fused_kernel(KParams p) {
    extern __shared__ __align__(16) unsigned char smem[];
    if (fuse_levels(p.L) == 8) fused_all<S, R, AR, SCH, 8>(p, smem);
    else fused_all<S, R, AR, SCH, 7>(p, smem);
}

template <int S, typename R>
__host__ __device__ constexpr size_t fused_lds(uint32_t L, size_t ent_lds) {
    return (fuse_levels(L) == 8 ? Pascal<S, R, 8>::bytes() : Pascal<S, R, 7>::bytes()) + ent_lds + kFuseTail;
}

// The closed form from the decode kernel's cut codes, for stage weights above
// 24 bits (32-bit products).
template <int S, bool AR, bool SCH>
__global__ __launch_bounds__(kBlock) void closed_kernel(KParams p) {
    extern __shared__ __align__(16) unsigned char smem[];
    const Ent tab = entry_tables(p, smem);
    __shared__ unsigned int nq;
    if (threadIdx.x == 0) nq = 0;
    __syncthreads();
    constexpr int NW = Codes<S>::kWords;
    unsigned long long best = ~0ull;
    // 32-bit positions and word offsets, as in eval_kernel
    const uint32_t stride = gridDim.x * kBlock, n_i = (uint32_t)p.n_i, ccap = (uint32_t)p.ccap;
    const uint32_t first_i = (uint32_t)p.first_i, seg = blockIdx.x * (uint32_t)p.seg_cap, lane = threadIdx.x & 63;
    for (uint32_t wb = blockIdx.x * kBlock + (threadIdx.x - lane); wb < n_i; wb += stride) {   // (wave-uniform)
        const uint32_t i = wb + lane, gi = first_i + i;
        const bool active = i < n_i;
        uint32_t w[NW], T;
#pragma unroll
        for (int k = 0; k < NW; ++k) w[k] = active ? p.codes[k * ccap + i] : 0u;
        bool feas;
        const uint32_t a = (w[0] & 0xFFu) ? assign_of(p, gi) : 0u;
        const bool write = closed_one<S, AR, SCH, false>(p, tab, seg, &nq, active, gi, a, w, T, feas);
        write_outputs(p, gi, write, T, feas);
        if (write) {
            const unsigned long long key = make_key(feas, T, gi);
            best = key < best ? key : best;
        }
    }
    __syncthreads();
    if (threadIdx.x == 0) p.fcount[blockIdx.x] = nq;
    block_min_and_finish(best, p.acc, p.done, p.result, nullptr, false);
}

// The candidates of the list by the recurrence.  Every block scans the
// segment counts and takes an equal run of the list's entries (in segment
// order, whole waves), in tiles of p.tile: a tile's lanes run to the first
// checkpoint of the steady part, the ones that have not settled are packed
// into the block's queue and run to the next, and so on, so that the few
// long transients share waves.  Queue entries carry position, cut codes,
// assignment and the DP state; blocks share nothing.  Under 1F1B bound by
// latency: few lanes (0.2-0.5 % of a chunk with transfers of a tenth of a
// layer) on long serial chains, 18 % VALU issue.  It takes 83 us of the
// 8-stage and 58 us of the 16-stage calls (2^26, 2^24); the launches per
// checkpoint over the whole chunk's queue that it replaces took 653 and 510 us
// for the 20 % of lanes the stencil left unsettled.  Under Eager 1F1B the list
// is longer (9 % of the 16-stage workload: 422 of 775 us) and the state larger
// (192 VGPRs at S = 16, 2 waves a SIMD); calls that would list nearly
// everything take cascade_kernel instead.
template <int S, bool AR, bool SCH>
__global__ __launch_bounds__(kBlock) void full_kernel(KParams p, uint32_t nseg) {
    extern __shared__ __align__(16) unsigned char smem[];
    uint32_t *pre = reinterpret_cast<uint32_t *>(smem + p.ent_lds);   // nseg entries
    uint32_t n;
    scan_counts(p.fcount, nseg, pre, n);
    const uint32_t waves = (n + 63) / 64;
    const uint32_t share = (waves + gridDim.x - 1) / gridDim.x * 64;   // entries a block takes
    const uint32_t need = n == 0 ? 1u : (n + share - 1) / share;       // blocks that have any
    if (blockIdx.x >= need) return;   // (block-uniform)
    const Ent tab = entry_tables(p, smem);   // (its barrier also publishes pre)
    const Comm<S> comm = load_comm<S>(p);
    constexpr int NW = Codes<S>::kWords;
    constexpr int NX = SCH ? 2 * S : S;
    constexpr uint32_t kEntry = 2 + NW + NX;
    const uint32_t nit = SCH ? p.M - 2 * S + 1 : p.M - S, ccap = (uint32_t)p.ccap, tile = p.tile;
    const FullList<S> list(p);
    // the block's two queues: kEntry arrays of `tile` words each
    uint32_t *const q0 = p.tileq + (uint64_t)blockIdx.x * 2 * kEntry * tile;
    __shared__ unsigned int nq[2];
    unsigned long long best = ~0ull;
    const uint32_t e0 = blockIdx.x * share, e1 = min(n, e0 + share);
    for (uint32_t t0 = e0; t0 < e1; t0 += tile) {
        uint32_t cnt = min(tile, e1 - t0), k0 = 0;
        for (uint32_t lvl = 0; cnt; ++lvl) {
            const uint32_t k1 = lvl < p.nlevels ? p.lvl_k[lvl] : nit;
            const uint32_t *qin = q0 + ((lvl + 1) & 1) * (uint64_t)kEntry * tile;
            uint32_t *qout = q0 + (lvl & 1) * (uint64_t)kEntry * tile;
            if (threadIdx.x == 0) nq[lvl & 1] = 0;
            __syncthreads();
            for (uint32_t j0 = (threadIdx.x >> 6) * 64; j0 < cnt; j0 += kBlock) {   // (wave-uniform)
                const uint32_t j = j0 + (threadIdx.x & 63);
                const bool active = j < cnt;
                uint32_t i = 0, a = 0, w[NW], X[NX], cut[S + 1], to[S], F[S], B[S], Y[S];
                if (lvl == 0) {
                    // the last segment g with pre[g] <= entry holds it
                    const uint32_t e = t0 + (active ? j : 0u);
                    uint32_t lo = 0, hi = nseg;
                    while (hi - lo > 1) {
                        const uint32_t mid = (lo + hi) >> 1;
                        if (pre[mid] <= e) lo = mid;
                        else hi = mid;
                    }
                    const uint32_t at = lo * (uint32_t)p.seg_cap + (e - pre[lo]);
                    i = list.pos[at];
                    a = list.asg[at];
#pragma unroll
                    for (int k = 0; k < NW; ++k) w[k] = list.w[k * ccap + at];
                } else {
                    const uint32_t at = active ? j : 0u;
                    i = qin[at];
                    a = qin[tile + at];
#pragma unroll
                    for (int k = 0; k < NW; ++k) w[k] = qin[(2 + k) * tile + at];
#pragma unroll
                    for (int s = 0; s < NX; ++s) X[s] = qin[(2 + NW + s) * tile + at];
                }
                unpack_cuts<S>(w, p.L, cut);
                decode_toff<S>(p, tab, a, to);
                const bool feas = stage_weights<S>(p, tab, cut, to, F, B);
                bool settled;
                uint32_t T = 0;
                if constexpr (SCH) {
                    uint32_t Fn[S], Fp[S];
                    if (lvl == 0) eager_prologue<S>(Y, Fn, Fp, F, B, comm);
                    else eager_unpack<S>(X, Y, Fn, Fp);
                    settled = eager_advance<S>(Y, Fn, Fp, F, B, comm, k0, k1, nit);
                    eager_pack<S>(Y, Fn, Fp, X);
                    if (__ballot(active && settled)) {
                        eager_epilogue<S>(Y, Fn, Fp, F, B, comm);
                        T = end_time<S, AR>(p, tab, Y, comm, w, a);
                    }
                } else {
                    if (lvl == 0) {
                        dp_prologue<S>(Y, F, B, comm, p.g24 != 0);
                    } else {
#pragma unroll
                        for (int s = 0; s < S; ++s) Y[s] = X[s];
                    }
                    settled = dp_advance<S>(Y, F, B, comm, k0, k1, nit);
#pragma unroll
                    for (int s = 0; s < S; ++s) X[s] = Y[s];
                    if (__ballot(active && settled)) T = dp_end<S, AR>(p, tab, Y, F, B, comm, w, a);
                }
                const unsigned long long m = __ballot(active && !settled);
                if (m) {
                    const unsigned int lane = threadIdx.x & 63;
                    unsigned int base = 0;
                    if (lane == 0) base = atomicAdd(&nq[lvl & 1], (unsigned int)__popcll(m));
                    base = __shfl(base, 0, 64);
                    if (active && !settled) {
                        const uint32_t at = base + __popcll(lane ? (m & ((1ull << lane) - 1ull)) : 0ull);
                        qout[at] = i;
                        qout[tile + at] = a;
#pragma unroll
                        for (int k = 0; k < NW; ++k) qout[(2 + k) * tile + at] = w[k];
#pragma unroll
                        for (int s = 0; s < NX; ++s) qout[(2 + NW + s) * tile + at] = X[s];
                    }
                }
                if (active && settled) {
                    if (p.makespan_out) __builtin_nontemporal_store(T, p.makespan_out + i);
                    const unsigned long long key = make_key(feas, T, i);
                    best = key < best ? key : best;
                }
            }
            __syncthreads();   // the level's entries are written and counted
            cnt = nq[lvl & 1];
            k0 = k1;
        }
    }
    block_min_and_finish(best, p.acc, p.done, p.result, nullptr, true, p.accumulate, nullptr, need, host_out(p));
}

// Early stop (Eq. 2 / Theorem 1) over one piece of a chunk.  Against the
// bound b in force (min of the caller's bound and the best of the earlier
// chunks, fixed within a chunk) every candidate is classified by classify()
// over its stages in pipeline order; the ones no stage discards survive
// and are evaluated exactly.
//
// filter_kernel runs in one of three modes:
//  kFilterFull   decodes every cut (a1), builds the stage weights (a2) and
//                decides all S stages while the cuts are in registers; the
//                survivors go to a list (call position + cut codes), block b
//                filling segment b of seg_cap entries, counted in LDS (no
//                global atomic, whose single address would serialise waves);
//  kFilterPrefix decodes only the first X = filter_prefix<S>() cuts and
//                decides the stages they close; the candidates it keeps go
//                to a list in the same segments (counts in acount) with
//                what the decode needs to go on (AList);
//  kFilterGather takes block b's segment of that list in order (coalesced),
//                decodes the remaining cuts and goes on as kFilterFull.
// For S >= 4 a piece goes through kFilterPrefix, then kFilterGather: most
// candidates are discarded at one of their first stages, and only the rest
// pay for the searches of their later cuts.  surv_kernel evaluates the
// survivor list on the DAG (a3) and folds it into the running best (a4).
//
// The prefix pass on 2^26 candidates of 8 stages takes 351 us (394 before):
// 62 % VALU issue at 130 wave operations a candidate (230 before), and the
// LDS busy 53 % of the cycles, half of them bank conflicts of the searches'
// per-lane addresses; its list alone is 155 us of memory.  2^24 of 16 stages
// 173 us (232 before), the gather passes 64 and 34 us (86 and 44).
enum FilterMode { kFilterFull = 0, kFilterPrefix = 1, kFilterGather = 2 };
template <int S>
__host__ __device__ constexpr int filter_prefix() { return S >= 4 ? S / 2 : 0; }
// Pascal columns a mode searches: the prefix mode cuts 1 .. X (columns
// S-X .. S-1), the gather mode the cuts after them (columns 2 .. S-X-1), the
// full mode every cut (columns 2 .. S-1)
template <int S, int MODE>
__host__ __device__ constexpr int filter_col_lo() { return MODE == kFilterPrefix ? S - filter_prefix<S>() : 2; }
template <int S, int MODE>
__host__ __device__ constexpr int filter_col_hi() { return MODE == kFilterGather ? S - filter_prefix<S>() - 1 : S - 1; }

// The prefix list, arrays of ccap entries: call position, decode state q
// after the first X cuts (low and high words), assignment index, then the
// first X cuts as cut codes.
static_assert(4 + (filter_prefix<kSMax>() + 3) / 4 <= kAListWords, "first-stage list entry too small");
struct AList {
    uint32_t *pos, *rlo, *rhi, *asg, *w;
    __device__ __forceinline__ explicit AList(const KParams &p)
        : pos(p.alist), rlo(p.alist + p.ccap), rhi(p.alist + 2 * p.ccap), asg(p.alist + 3 * p.ccap),
          w(p.alist + 4 * p.ccap) {}
};

// Stage-1 screen of the prefix mode.  Stage 1 = [0, c_1) on type t fits its
// memory iff c_1 <= hm_t(0), and g(S_1) = M (F_1 + B_1) + d_1 only grows
// with c_1, so it passes Eq. 2 iff c_1 <= hb_t, the largest end point with
// g(S_1) <= b.  Ranks are lexicographic with c_1 the most significant cut,
// so the compositions with c_1 <= h hold the ranks below
//   N(h) = C(L-1, S-1) - C(L-1-h, S-1)
// (the others have all S-1 cuts in h+1 .. L-1).  A candidate therefore
// fails stage 1 iff its rank is at least N(min(hm_t, hb_t)), and fails it on
// memory (tested first at a stage) iff its rank is at least N(hm_t): one
// compare decides it before any cut is decoded.  thr[2t], thr[2t+1] = those
// two limits for every type t (threads t < T; the caller's barrier
// publishes them).
template <int S, typename R, bool SUM>
__device__ __forceinline__ void stage1_limits(const KParams &p, const Ent &tab, uint32_t b, unsigned long long *thr) {
    if (threadIdx.x >= p.T) return;
    const uint32_t to = threadIdx.x * p.erow, L = p.L, hmax = L - S + 1;   // hmax: the largest c_1
    // (the prefix sums start at 0)
    const uint32_t pd0 = p.has_ar ? ent<kEPd>(tab, 0, to) : 0u;
    // g(S_1) is nondecreasing in c_1: the largest passing end point by halving
    // steps (hb = 0: none passes; every c_1 is at least 1)
    uint32_t hb = 0;
    for (uint32_t st = 128; st; st >>= 1) {
        const uint32_t c = hb + st;
        if (c <= hmax) {
            const uint32_t W = ent<kEPf>(tab, c, to) + (SUM ? 0u : ent<kEPb>(tab, c, to));
            const uint32_t D = p.has_ar ? ent<kEPd>(tab, c, to) - pd0 : 0u;
            // M (F + B) + d_1 is an Eq. 2 value, below 2^31 like every path weight
            if (p.M * W + D <= b) hb = c;
        }
    }
    const uint32_t hm = min(ent<kEHm>(tab, 0, to), hmax), h1 = min(hb, hm);
    const R *bin = reinterpret_cast<const R *>(p.binom);
    thr[2 * threadIdx.x] = p.n_comp - (uint64_t)bin[(S - 1) * kNB + (L - 1 - h1)];
    thr[2 * threadIdx.x + 1] = p.n_comp - (uint64_t)bin[(S - 1) * kNB + (L - 1 - hm)];
}

// Type of stage 1 of assignment a (valid a).
template <int S>
__device__ __forceinline__ uint32_t first_stage_type(const KParams &p, uint32_t a) {
    if (p.assign_mode == kAssignFixed) return p.fixed_word[0] & 0xFFu;
    if (p.assign_mode == kAssignTable) return p.assign[(uint64_t)a * S];
    // the top base-T digit: floor(a / T^(S-1)), from a multiply-high that
    // gives it or one more
    uint32_t q = __umulhi(a, p.s1_magic);
    if ((uint64_t)q * p.s1_div > a) q -= 1;
    return q;
}

// LDS words that lanes of one wave wrote are visible to the wave's other
// lanes after this (their writes complete; no code moves across it).
__device__ __forceinline__ void wave_lds_sync() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// Buffered positions of one wave in the screened prefix mode: fewer than one
// batch of kIlp * 64 before a screened tile of as many adds to it.
constexpr uint32_t kScreenBuf = 2 * kIlp * 64;
// The screen costs a second load of every kept candidate at a scattered index
// and the buffer's bookkeeping, and saves the prefix work of the ones it
// discards.  Early stop on lists of 2^24 (8 stages without all-reduce times:
// 2^26), us with the screen / without: 6 stages 245 / 229, 8 stages 450 / 473,
// 10 stages 216 / 218, 12 stages 290 / 266, 16 stages 291 / 260; with
// all-reduce times 8 stages 205 / 226, 16 stages 351 / 307.  So: four or five
// prefix cuts, or fewer with the dearer tests; with more cuts the loads and
// the registers cost more than the searches saved.
template <int S, bool AR, int MODE>
__host__ __device__ constexpr bool filter_screens() {
    return MODE == kFilterPrefix && filter_prefix<S>() <= 5 && (AR || filter_prefix<S>() >= 4);
}
template <int S, bool AR, int MODE>
__host__ __device__ constexpr size_t filter_static_lds() {
    return filter_screens<S, AR, MODE>() ? (size_t)kScreenBuf * 4 * (kBlock / 64) + 16 * kTypesMax : 0;
}

// Of the set lanes of m, those below this lane.
__device__ __forceinline__ uint32_t lanes_below(unsigned long long m) {
    return __builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0u));
}

// Word at byte offset o of an array whose start is the same for every lane
// (a scalar base and a 32-bit lane offset: no 64-bit address per lane).
__device__ __forceinline__ uint32_t &word_at(uint32_t *a, uint32_t o) {
    return *reinterpret_cast<uint32_t *>(reinterpret_cast<char *>(a) + o);
}

// The tests of kIlp decoded candidates of one lane (cuts 1 .. X of
// filter_all's mode in cut[u]): classification, counts, and the list entry
// of each candidate kept (the prefix list, or the survivor list).  Every
// lane of the wave comes here; the counts are the wave's.
template <int S, typename R, bool AR, bool SUM, int MODE>
__device__ __forceinline__ void filter_emit(const KParams &p, const Ent &tab, uint32_t b, unsigned int *nq,
                                            const bool (&act)[kIlp], const bool (&ok)[kIlp],
                                            const uint32_t (&pos)[kIlp], const uint32_t (&asg)[kIlp],
                                            const R (&r)[kIlp], const uint32_t (&cut)[kIlp][S + 1],
                                            uint32_t &n_keep, uint32_t &n_pruned, uint32_t &n_infeas, bool &bad) {
    constexpr int X0 = filter_prefix<S>();
    constexpr int X = MODE == kFilterPrefix ? X0 : S;   // stages decided, cuts 1 .. X decoded
    constexpr int NW = Codes<S>::kWords;
    constexpr int AW = (X0 + 3) / 4;                    // code words of the prefix cuts
    const unsigned int lane = threadIdx.x & 63;
    unsigned long long m[kIlp];
    uint32_t total = 0;
#pragma unroll
    for (int u = 0; u < kIlp; ++u) {
        uint32_t to[S];
        decode_toff<S>(p, tab, ok[u] ? asg[u] : 0u, to);
        bool out, over;
        classify<S, AR, X, SUM>(p, tab, cut[u], to, b, out, over);
        bad |= act[u] & !ok[u];
        const bool valid = act[u] & ok[u];
        m[u] = __ballot(valid & !out);
        n_infeas += (uint32_t)__popcll(__ballot(valid & over));
        n_pruned += (uint32_t)__popcll(__ballot(valid & out & !over));
        total += (uint32_t)__popcll(m[u]);
    }
    if (total == 0) return;
    if (MODE != kFilterPrefix) n_keep += total;
    uint32_t slot0 = 0;
    if (lane == 0) slot0 = atomicAdd(nq, total);
    slot0 = __builtin_amdgcn_readfirstlane(slot0);
    // (32-bit word offsets of a segment: each list holds fewer than 2^32
    // words; byte offsets inside a segment, seg_cap entries, fit too)
    const uint32_t seg = blockIdx.x * (uint32_t)p.seg_cap, ccap = (uint32_t)p.ccap;
    const AList al(p);
#pragma unroll
    for (int u = 0; u < kIlp; ++u) {
        if ((m[u] >> lane) & 1) {
            const uint32_t o = (slot0 + lanes_below(m[u])) << 2;
            if constexpr (MODE == kFilterPrefix) {
                uint32_t w[AW];
#pragma unroll
                for (int k = 0; k < AW; ++k) w[k] = 0;
#pragma unroll
                for (int j = 1; j <= X0; ++j) w[(j - 1) / 4] |= cut[u][j] << (8 * ((j - 1) % 4));
                word_at(al.pos + seg, o) = pos[u];
                word_at(al.asg + seg, o) = asg[u];
                word_at(al.rlo + seg, o) = (uint32_t)r[u];
                if (sizeof(R) == 8) word_at(al.rhi + seg, o) = (uint32_t)((uint64_t)r[u] >> 32);
#pragma unroll
                for (int k = 0; k < AW; ++k) word_at(al.w + (k * ccap + seg), o) = w[k];
            } else {
                uint32_t w[NW];
                pack_cuts<S>(cut[u], true, w);
                word_at(p.sidx + seg, o) = pos[u];
#pragma unroll
                for (int k = 0; k < NW; ++k) word_at(p.codes + (k * ccap + seg), o) = w[k];
            }
        }
        slot0 += (uint32_t)__popcll(m[u]);
    }
}

// Prefix mode: each wave screens tiles of kIlp * 64 consecutive candidates
// of the piece (its stream: tiles gw, gw + nwave, ...) on stage 1 alone
// (stage1_limits), keeps the positions of the rest in its LDS buffer buf,
// and decodes and tests them kIlp * 64 at a time, so that the searches of
// the first cuts run only for candidates that pass stage 1 (about two in
// three on the workloads here) and every lane has a candidate to decode.
template <int S, typename R, int H, bool AR, bool SUM, typename PC>
__device__ __forceinline__ void filter_screened(const KParams &p0, const PC &pc, const Ent &tab,
                                                uint32_t b, unsigned int *nq, uint32_t *buf,
                                                const unsigned long long *thr, uint32_t &n_keep,
                                                uint32_t &n_pruned, uint32_t &n_infeas, bool &bad) {
    constexpr int X0 = filter_prefix<S>();
    constexpr uint32_t kTile = kIlp * 64;
    const unsigned int lane = threadIdx.x & 63;
    // 32-bit positions: a piece holds at most 2^26 candidates, a call fewer than 2^32
    const uint32_t n = (uint32_t)p0.n_i, first_i = (uint32_t)p0.first_i;
    const uint32_t nwave = gridDim.x * (kBlock / 64);
    // next tile of the stream (the same for every lane)
    uint32_t tile = blockIdx.x * (kBlock / 64) + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    uint32_t cnt = 0;                                                  // positions in buf
    for (;;) {
        // screen tiles until a batch is buffered or the stream ends
        while (cnt < kTile && tile * kTile < n) {
            const KParams &p = fresh_args();
            const uint32_t t0 = tile * kTile;
            tile += nwave;
            bool act[kIlp], ok[kIlp];
            uint32_t pos[kIlp], a[kIlp];
            R r[kIlp];
            load_candidates<R>(p, t0, 64, lane, act, ok, pos, a, r);
#pragma unroll
            for (int u = 0; u < kIlp; ++u) {
                const uint32_t t = first_stage_type<S>(p, a[u]);
                const uint64_t rk = (uint64_t)r[u];
                const bool fail = rk >= thr[2 * t], over = rk >= thr[2 * t + 1];
                // (out of range: kept, the batch raises the error flag)
                const bool keep = act[u] & !(ok[u] & fail);
                const unsigned long long m = __ballot(keep);
                n_infeas += (uint32_t)__popcll(__ballot(ok[u] & fail & over));
                n_pruned += (uint32_t)__popcll(__ballot(ok[u] & fail & !over));
                if (keep) buf[cnt + lanes_below(m)] = pos[u] - first_i;
                cnt += (uint32_t)__popcll(m);
            }
        }
        if (cnt == 0) break;
        const KParams &p = fresh_args();
        wave_lds_sync();
        const uint32_t nb = cnt < kTile ? cnt : kTile;
        bool act[kIlp], ok[kIlp];
        uint32_t pos[kIlp], asg[kIlp], cut[kIlp][S + 1];
        R r[kIlp];
#pragma unroll
        for (int u = 0; u < kIlp; ++u) {
            const uint32_t j = (uint32_t)u * 64 + lane;
            act[u] = j < nb;
            pos[u] = first_i + (act[u] ? buf[j] : 0u);   // (position 0 of the piece for idle lanes)
        }
        decode_cuts<S, R, H, X0>(p, pc, pos, act, ok, asg, r, cut);
        filter_emit<S, R, AR, SUM, kFilterPrefix>(p, tab, b, nq, act, ok, pos, asg, r, cut, n_keep, n_pruned, n_infeas, bad);
        // the positions past the batch (fewer than kTile) move to the front
        if (cnt > kTile) {
            uint32_t v[kIlp];
#pragma unroll
            for (int u = 0; u < kIlp; ++u) {
                const uint32_t j = kTile + (uint32_t)u * 64 + lane;
                v[u] = j < cnt ? buf[j] : 0u;
            }
            wave_lds_sync();
#pragma unroll
            for (int u = 0; u < kIlp; ++u) {
                const uint32_t j = (uint32_t)u * 64 + lane;
                if (kTile + j < cnt) buf[j] = v[u];
            }
        }
        cnt -= nb;
        wave_lds_sync();
    }
}

template <int S, typename R, int H, bool AR, bool SUM, int MODE>
__device__ __forceinline__ void filter_all(const KParams &p, const R *pas, const Ent &tab, uint32_t b,
                                           unsigned int *nq, uint32_t *buf, const unsigned long long *thr,
                                           uint32_t &n_keep, uint32_t &n_pruned, uint32_t &n_infeas, bool &bad) {
    constexpr int X0 = filter_prefix<S>();
    constexpr int AW = (X0 + 3) / 4;                    // code words of the prefix cuts
    const Pascal<S, R, H, filter_col_lo<S, MODE>(), filter_col_hi<S, MODE>()> pc(pas);
    if constexpr (filter_screens<S, AR, MODE>()) {
        filter_screened<S, R, H, AR, SUM>(p, pc, tab, b, nq, buf, thr, n_keep, n_pruned, n_infeas, bad);
        return;
    }
    // 32-bit positions and word offsets: a piece holds at most 2^26
    // candidates, a call fewer than 2^32, and each list fewer than 2^32
    // words (fewer scalar registers than 64-bit ones)
    const uint32_t seg = blockIdx.x * (uint32_t)p.seg_cap, ccap = (uint32_t)p.ccap;
    const uint32_t lane = threadIdx.x & 63;
    // full, prefix: the piece, kIlp candidates a lane, strided over the grid;
    // gather: this block's segment of the list, strided over the block.  The
    // loop runs over whole waves: base is the same for every lane.
    const uint32_t n = MODE == kFilterGather ? p.acount[blockIdx.x] : (uint32_t)p.n_i;
    const uint32_t stride = MODE == kFilterGather ? (uint32_t)kBlock : gridDim.x * kBlock;
    const uint32_t wave0 = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6) * 64;
    const uint32_t start = MODE == kFilterGather ? wave0 : blockIdx.x * kBlock + wave0;
    for (uint32_t base = start; base < n; base += kIlp * stride) {
        const KParams &p = fresh_args();
        bool act[kIlp], ok[kIlp];
        uint32_t pos[kIlp];
        uint32_t asg[kIlp], cut[kIlp][S + 1];
        R r[kIlp];
        if constexpr (MODE != kFilterGather) load_candidates<R>(p, base, stride, lane, act, ok, pos, asg, r);
#pragma unroll
        for (int u = 0; u < kIlp; ++u) {
            cut[u][0] = 0;
            cut[u][S] = p.L;
            if constexpr (MODE == kFilterGather) {
                // lanes past the end take the last entry (not counted)
                const uint32_t i = base + u * stride, wb = min(i, n - 1), l = min(lane, n - 1 - wb);
                act[u] = i + lane < n;
                const AList al(p);
                const uint32_t s0 = seg + wb, o = l << 2;
                ok[u] = act[u];
                pos[u] = word_at(al.pos + s0, o);
                asg[u] = word_at(al.asg + s0, o);
                r[u] = (R)word_at(al.rlo + s0, o);
                if constexpr (sizeof(R) == 8) r[u] |= (R)((uint64_t)word_at(al.rhi + s0, o) << 32);
                uint32_t w[AW + 1];
#pragma unroll
                for (int k = 0; k < AW; ++k) w[k] = word_at(al.w + (k * ccap + s0), o);
#pragma unroll
                for (int j = 1; j <= X0; ++j) cut[u][j] = (w[(j - 1) / 4] >> (8 * ((j - 1) % 4))) & 0xFFu;
            } else {
                r[u] = decode_start<R>(p, r[u]);
            }
        }
        if constexpr (MODE == kFilterGather) decode_range<S, R, H, X0, S - 1>(p, pc, r, cut);
        else decode_range<S, R, H, 0, MODE == kFilterPrefix ? X0 : S - 1>(p, pc, r, cut);
        filter_emit<S, R, AR, SUM, MODE>(p, tab, b, nq, act, ok, pos, asg, r, cut, n_keep, n_pruned, n_infeas, bad);
    }
}

// GTAB: the stage entries are read from global memory (L2) instead of LDS,
// when they and the Pascal columns together exceed the 64 KB of LDS one
// block may use (the largest columns: L > 128 with 64-bit ranks).  LDS:
// the stage entries first (unless GTAB), then the Pascal columns.
template <int S, typename R, bool AR, bool GTAB, int MODE>
__global__ __launch_bounds__(kBlock) __attribute__((amdgpu_waves_per_eu(4, 8))) void filter_kernel(KParams p) {
    extern __shared__ __align__(16) unsigned char smem[];
    constexpr bool SUM = !AR && !GTAB;   // field kEPf holds Pf + Pb (classify)
    const uint32_t H = decode_levels(p.L);
    Ent tab;
    R *pas;
    if constexpr (GTAB) {
        tab = entry_global(p);
        pas = reinterpret_cast<R *>(smem);
    } else {
        pas = reinterpret_cast<R *>(smem + p.ent_lds);
        tab = entry_tables(p, smem);
        if constexpr (SUM) {   // (the barrier after the Pascal columns publishes the sums)
            uint32_t *e = reinterpret_cast<uint32_t *>(smem);
            for (uint32_t t = 0; t < p.T; ++t, e += p.erow / 4)
                for (uint32_t i = threadIdx.x; i < kEntRow; i += kBlock) e[i] += e[i + (kEPb - kEPf) * kEntRow];
        }
    }
    // bound in force: min(caller's bound, best of the chunks before this one)
    const unsigned long long rb = __hip_atomic_load(p.snap, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    const uint32_t rbT = (uint32_t)(rb >> 32);
    const uint32_t b = rbT < p.es_bound ? rbT : p.es_bound;
    uint32_t n_keep = 0, n_pruned = 0, n_infeas = 0;
    bool bad = false;
    __shared__ unsigned int nq;
    if (threadIdx.x == 0) nq = 0;
    // prefix mode: the waves' position buffers and the stage-1 rank limits
    // (published by the barrier after the Pascal columns)
    uint32_t *buf = nullptr;
    const unsigned long long *thr = nullptr;
    if constexpr (filter_screens<S, AR, MODE>()) {
        __shared__ uint32_t screen_buf[kScreenBuf * (kBlock / 64)];
        __shared__ unsigned long long screen_thr[2 * kTypesMax];
        if constexpr (SUM) __syncthreads();   // (the sums)
        stage1_limits<S, R, SUM>(p, tab, b, screen_thr);
        buf = screen_buf + (threadIdx.x >> 6) * kScreenBuf;
        thr = screen_thr;
    }
    switch (H) {
    case 8: pascal_tables<S, R, 8, filter_col_lo<S, MODE>(), filter_col_hi<S, MODE>()>(p, pas); __syncthreads(); filter_all<S, R, 8, AR, SUM, MODE>(p, pas, tab, b, &nq, buf, thr, n_keep, n_pruned, n_infeas, bad); break;
    case 7: pascal_tables<S, R, 7, filter_col_lo<S, MODE>(), filter_col_hi<S, MODE>()>(p, pas); __syncthreads(); filter_all<S, R, 7, AR, SUM, MODE>(p, pas, tab, b, &nq, buf, thr, n_keep, n_pruned, n_infeas, bad); break;
    case 6: pascal_tables<S, R, 6, filter_col_lo<S, MODE>(), filter_col_hi<S, MODE>()>(p, pas); __syncthreads(); filter_all<S, R, 6, AR, SUM, MODE>(p, pas, tab, b, &nq, buf, thr, n_keep, n_pruned, n_infeas, bad); break;
    default: pascal_tables<S, R, 5, filter_col_lo<S, MODE>(), filter_col_hi<S, MODE>()>(p, pas); __syncthreads(); filter_all<S, R, 5, AR, SUM, MODE>(p, pas, tab, b, &nq, buf, thr, n_keep, n_pruned, n_infeas, bad); break;
    }
    // per-block sums (the counts are the waves'), one global atomic per
    // counter and block
    __shared__ unsigned long long cnt[3];
    if (threadIdx.x < 3) cnt[threadIdx.x] = 0;
    __syncthreads();
    if ((threadIdx.x & 63) == 0) {
        if (n_keep) atomicAdd(&cnt[0], (unsigned long long)n_keep);
        if (n_pruned) atomicAdd(&cnt[1], (unsigned long long)n_pruned);
        if (n_infeas) atomicAdd(&cnt[2], (unsigned long long)n_infeas);
    }
    __syncthreads();
    if (threadIdx.x < 3 && cnt[threadIdx.x]) atomicAdd(&p.stats[threadIdx.x], cnt[threadIdx.x]);
    // (after the barrier above: every wave has added)
    if (threadIdx.x == 0) (MODE == kFilterPrefix ? p.acount : p.scount)[blockIdx.x] = nq;
    if (bad) atomicOr(p.err, 1u);
}

// Where only the best candidate of a list is wanted (early stop, search), a
// candidate whose closed form is not proven needs the recurrence only if its
// value, a lower bound of its makespan, could still win: its key
// (value << 32 | position) is below the best known one.  Each wave keeps such
// candidates in a list in LDS and runs the recurrence on them when 64 have
// gathered, and on the rest once the block's proven candidates are known.
// (Problems without a closed form put every candidate there, with value 0.)
// The best known key is the block's own, in LDS: read from a global word by
// every wave it cost more than it saved (that word's line serialises them).
struct Pend {
    uint32_t *at, *low;            // the wave's [128]: where the candidate is, and its value
    unsigned long long *known;     // the block's best key so far (starts at the largest that counts)
    uint32_t n;                    // entries (wave-uniform)
};
struct PendLds {
    uint32_t at[kWaves][128], low[kWaves][128];
    unsigned long long known;
};
__device__ __forceinline__ Pend pend_init(PendLds &l, unsigned long long limit) {
    if (threadIdx.x == 0) l.known = limit;   // (published by the caller's next barrier)
    return Pend{l.at[threadIdx.x >> 6], l.low[threadIdx.x >> 6], &l.known, 0u};
}

// f(at) = exact key, for entries 0 .. n-1 that can still win (n <= 64).
template <typename F>
__device__ __forceinline__ void pend_run(const Pend &l, uint32_t first, uint32_t n, unsigned long long &best, F &&f) {
    wave_lds_sync();
    const uint32_t lane = threadIdx.x & 63;
    if (lane < n && (unsigned long long)l.low[first + lane] << 32 <= *l.known) {
        const unsigned long long key = f(l.at[first + lane]);
        best = key < best ? key : best;
    }
    wave_lds_sync();
}

// One batch of a wave: `proven` lanes offer their key, the other lanes with
// `want` set are kept; then the wave runs a full batch if it has one.
template <typename F>
__device__ __forceinline__ void pend_add(Pend &l, bool want, bool proven, uint32_t at, uint32_t T, uint32_t pos,
                                         unsigned long long &best, F &&f, uint32_t batch = 64) {
    const uint32_t lane = threadIdx.x & 63;
    if (want && proven) {
        const unsigned long long key = make_key(true, T, pos);
        if (key < best) {
            best = key;
            if (key < *l.known) atomicMin(l.known, key);
        }
    }
    const bool keep = want && !proven && (unsigned long long)T << 32 <= *l.known;
    const unsigned long long m = __ballot(keep);
    if (m == 0) return;
    if (keep) {
        const uint32_t j = l.n + __popcll(lane ? (m & ((1ull << lane) - 1ull)) : 0ull);
        l.at[j] = at;
        l.low[j] = T;
    }
    l.n += __popcll(m);
    if (l.n >= batch) {   // (without a closed form: every batch at once)
        const uint32_t n = min(l.n, 64u);
        l.n -= n;
        pend_run(l, l.n, n, best, f);   // (the last ones: the rest stays in place)
    }
}

// After a block's last batch (all threads): the rest of the lists against
// the block's best and *acc.  Returns the thread's best key.
template <typename F>
__device__ __forceinline__ unsigned long long pend_finish(Pend &l, unsigned long long best, unsigned long long *acc, F &&f) {
    if (__syncthreads_or(l.n != 0)) {
        if (threadIdx.x == 0)
            atomicMin(l.known, __hip_atomic_load(acc, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT));
        __syncthreads();
        pend_run(l, 0u, l.n, best, f);
    }
    return best;
}

// One candidate's closed form on its stage weights: true if T is exact,
// else T is a lower bound.
template <int S, bool AR, bool SCH>
__device__ __forceinline__ bool closed_or_bound(const KParams &p, const Ent &tab, const uint32_t (&cut)[S + 1],
                                                const uint32_t (&to)[S], const uint32_t (&F)[S],
                                                const uint32_t (&B)[S], uint32_t &T) {
    uint32_t D[S];
    if (AR) stage_allreduce<S>(p, tab, cut, to, D);
    return p.g24 ? closed_form<S, SCH, AR, true>(p, F, B, D, T) : closed_form<S, SCH, AR, false>(p, F, B, D, T);
}

// surv_kernel takes the survivor list as one sequence in segment order
// (segment j: scount[j] entries from j seg_cap).  Every block scans the nseg
// segment counts into LDS, after the stage entries; survivor k then goes to
// thread k mod (grid kBlock), found by a binary search of the scan, so the
// survivors spread over the whole grid, 64 to a wave.  Only the blocks the
// list needs (one per kBlock survivors, at least one) go on: the others
// leave before loading the entries and take no ticket on the done counter.
// Bound by latency (0.1-0.8 % of the candidates come here).  With few batches
// a wave the closed form does not shorten the chain: some lane of some wave
// needs the recurrence all the same, after it, unless they are so few that
// all have the proof.  So from p.surv_least survivors up to p.surv_direct
// quarters of a batch per wave all take the recurrence at once (the limits
// and what they were measured on are at their rule in the host code).
// 8 stages, 7.0e4 survivors of 2^26: 25 us, 29 with the closed form first; 16
// stages, 1.0e5 of 2^24: 51 us with it first, 62 at once.
template <int S, bool AR, bool SCH>
__global__ __launch_bounds__(kBlock) void surv_kernel(KParams p, uint32_t publish, uint32_t nseg) {
    extern __shared__ __align__(16) unsigned char smem[];
    __shared__ PendLds pend;
    // a makespan above the caller's bound never becomes the result
    Pend l = pend_init(pend, (unsigned long long)p.es_bound << 32 | 0xFFFFFFFFu);
    uint32_t *pre = reinterpret_cast<uint32_t *>(smem + p.ent_lds);   // nseg + 1 entries
    uint32_t n;
    scan_counts(p.scount, nseg, pre, n);
    const uint32_t need = n == 0 ? 1u : min(gridDim.x, (n + kBlock - 1) / kBlock);
    if (blockIdx.x >= need) return;   // (block-uniform: every thread has the same n)
    const Ent tab = entry_tables(p, smem);   // (its barrier also publishes pre)
    const Comm<S> comm = load_comm<S>(p);
    constexpr int NW = Codes<S>::kWords;
    auto load = [&](uint32_t at, uint32_t &i, uint32_t &a, uint32_t (&w)[NW], uint32_t (&cut)[S + 1], uint32_t (&to)[S],
                    uint32_t (&F)[S], uint32_t (&B)[S]) {
        i = p.sidx[at];
#pragma unroll
        for (int kk = 0; kk < NW; ++kk) w[kk] = p.codes[kk * (uint32_t)p.ccap + at];
        unpack_cuts<S>(w, p.L, cut);
        a = assign_of(p, i);
        decode_toff<S>(p, tab, a, to);
        stage_weights<S>(p, tab, cut, to, F, B);
    };
    auto full = [&](uint32_t at) {
        uint32_t i, a, w[NW], cut[S + 1], to[S], F[S], B[S];
        load(at, i, a, w, cut, to, F, B);
        return make_key(true, dp_full_settle<S, SCH, AR>(p, tab, F, B, comm, w, a), i);
    };
    unsigned long long best = ~0ull;
    const bool closed = p.closed && (n < p.surv_least || (uint64_t)n * 4 > (uint64_t)p.surv_direct * (gridDim.x * kBlock));
    const uint32_t lane = threadIdx.x & 63;
    for (uint32_t k0 = blockIdx.x * kBlock + (threadIdx.x - lane); k0 < n; k0 += gridDim.x * kBlock) {   // (wave-uniform)
        const uint32_t k = k0 + lane;
        uint32_t at = 0, i = 0, T = 0;
        bool proven = false;
        if (k < n) {
            // the last segment j with pre[j] <= k holds survivor k
            uint32_t lo = 0, hi = nseg;
            while (hi - lo > 1) {
                const uint32_t mid = (lo + hi) >> 1;
                if (pre[mid] <= k) lo = mid;
                else hi = mid;
            }
            at = lo * (uint32_t)p.seg_cap + (k - pre[lo]);
            if (closed) {
                uint32_t a, w[NW], cut[S + 1], to[S], F[S], B[S];
                load(at, i, a, w, cut, to, F, B);
                proven = closed_or_bound<S, AR, SCH>(p, tab, cut, to, F, B, T);
            }
        }
        pend_add(l, k < n, proven, at, T, i, best, full, closed ? 64u : 1u);
    }
    best = pend_finish(l, best, p.acc, full);
    block_min_and_finish(best, p.acc, p.done, nullptr, p.run_best, true, false, publish ? p.snap : nullptr, need, host_out(p));
}

constexpr size_t kLdsBlockMax = 64 * 1024;   // LDS bytes one block of these kernels may use
constexpr size_t kLdsCu = 160 * 1024;          // (fused_kernel: all a CU has)

// host-side launchers
// ---------------------------------------------------------------------------
template <int S>
hipError_t launch_eval_s(const KParams &p, const LaunchCfg &lc, hipStream_t st) {
    const dim3 g(lc.grid), b(kBlock);
    const bool sch = p.sched != 0, ar = p.has_ar != 0, tab = p.nslots != 0;
    const int k = (ar ? 4 : 0) | (sch ? 2 : 0) | (tab ? 1 : 0);
    switch (k) {
    case 0: hipLaunchKernelGGL((eval_kernel<S, false, false, false>), g, b, lc.lds_bytes, st, p); break;
    case 1: hipLaunchKernelGGL((eval_kernel<S, false, false, true>), g, b, lc.lds_bytes, st, p); break;
    case 2: hipLaunchKernelGGL((eval_kernel<S, false, true, false>), g, b, lc.lds_bytes, st, p); break;
    case 3: hipLaunchKernelGGL((eval_kernel<S, false, true, true>), g, b, lc.lds_bytes, st, p); break;
    case 4: hipLaunchKernelGGL((eval_kernel<S, true, false, false>), g, b, lc.lds_bytes, st, p); break;
    case 5: hipLaunchKernelGGL((eval_kernel<S, true, false, true>), g, b, lc.lds_bytes, st, p); break;
    case 6: hipLaunchKernelGGL((eval_kernel<S, true, true, false>), g, b, lc.lds_bytes, st, p); break;
    default: hipLaunchKernelGGL((eval_kernel<S, true, true, true>), g, b, lc.lds_bytes, st, p); break;
    }
    return hipGetLastError();
}

// The kernels of one schedule and end node: f(integral constants AR, SCH)
template <typename F>
auto with_variant(const KParams &p, F &&f) {
    using std::false_type;
    using std::true_type;
    if (p.has_ar) return p.sched ? f(true_type{}, true_type{}) : f(true_type{}, false_type{});
    return p.sched ? f(false_type{}, true_type{}) : f(false_type{}, false_type{});
}

template <int S>
hipError_t launch_closed_s(const KParams &p, const LaunchCfg &lc, hipStream_t st) {
    return with_variant(p, [&](auto ar, auto sch) {
        hipLaunchKernelGGL((closed_kernel<S, decltype(ar)::value, decltype(sch)::value>), dim3(lc.grid), dim3(kBlock),
                           lc.lds_bytes, st, p);
        return hipGetLastError();
    });
}

// The recurrence over a chunk, then its cascade's levels (p.nlevels + 1
// launches on lc.grid blocks).
template <int S, bool AR>
hipError_t launch_cascade_ar(const KParams &p, const LaunchCfg &lc, hipStream_t st) {
    const dim3 g(lc.grid), b(kBlock);
    hipLaunchKernelGGL((cascade_kernel<S, AR>), g, b, lc.lds_bytes, st, p);
    hipError_t e = hipGetLastError();
    for (uint32_t l = 1; l <= p.nlevels && e == hipSuccess; ++l) {
        hipLaunchKernelGGL((resume_kernel<S, AR>), g, b, lc.lds_bytes, st, p, l);
        e = hipGetLastError();
    }
    return e;
}
template <int S>
hipError_t launch_cascade_s(const KParams &p, const LaunchCfg &lc, hipStream_t st) {
    return p.has_ar ? launch_cascade_ar<S, true>(p, lc, st) : launch_cascade_ar<S, false>(p, lc, st);
}

// Resident blocks per CU of its first kernel.
template <int S>
hipError_t cascade_occupancy_s(const KParams &p, size_t lds, int *blocks) {
    if (p.has_ar) return hipOccupancyMaxActiveBlocksPerMultiprocessor(blocks, cascade_kernel<S, true>, kBlock, lds);
    return hipOccupancyMaxActiveBlocksPerMultiprocessor(blocks, cascade_kernel<S, false>, kBlock, lds);
}

template <int S, typename R>
hipError_t launch_fused_s(const KParams &p, const LaunchCfg &lc, hipStream_t st) {
    const size_t lds = fused_lds<S, R>(p.L, p.ent_lds);
    return with_variant(p, [&](auto ar, auto sch) {
        hipLaunchKernelGGL((fused_kernel<S, R, decltype(ar)::value, decltype(sch)::value>), dim3(lc.grid),
                           dim3(kFuseBlock), lds, st, p);
        return hipGetLastError();
    });
}

// Resident blocks per CU of fused_kernel (0: its tables exceed a CU's LDS).
template <int S, typename R>
hipError_t fused_occupancy_s(const KParams &p, int *blocks) {
    const size_t lds = fused_lds<S, R>(p.L, p.ent_lds);
    *blocks = 0;
    if (lds > kLdsCu) return hipSuccess;
    return with_variant(p, [&](auto ar, auto sch) {
        return hipOccupancyMaxActiveBlocksPerMultiprocessor(blocks, fused_kernel<S, R, decltype(ar)::value, decltype(sch)::value>,
                                                            kFuseBlock, lds);
    });
}

// full_kernel on lc.grid2 blocks (LDS: the stage entries, then the scan of
// the lc.grid segment counts)
template <int S>
hipError_t launch_full_s(const KParams &p, const LaunchCfg &lc, hipStream_t st) {
    const size_t lds = (size_t)p.ent_lds + (size_t)lc.grid * 4;
    if (lds > kLdsBlockMax || lc.grid2 == 0) return hipErrorInvalidValue;
    return with_variant(p, [&](auto ar, auto sch) {
        hipLaunchKernelGGL((full_kernel<S, decltype(ar)::value, decltype(sch)::value>), dim3(lc.grid2), dim3(kBlock),
                           lds, st, p, lc.grid);
        return hipGetLastError();
    });
}

template <int S, typename R>
hipError_t launch_decode_s(const KParams &p, const LaunchCfg &lc, hipStream_t st) {
    const size_t lds = pascal_bytes<S, R>(p.L);   // (columns 2 .. S-1)
    hipLaunchKernelGGL((decode_kernel<S, R>), dim3(lc.grid), dim3(kBlock), lds, st, p);
    return hipGetLastError();
}

// One piece of an early-stop chunk: filter_kernel on the grid in lc (LDS:
// Pascal columns, then the stage tables of lc.lds_bytes), in prefix then
// gather mode for S >= 4, else in full mode; then surv_kernel on lc.grid2
// blocks (LDS: the stage entries, then the scan of the lc.grid segment
// counts).
template <int S, typename R, int MODE>
hipError_t launch_filter_s(const KParams &p, const LaunchCfg &lc, hipStream_t st) {
    const size_t pas = pascal_bytes<S, R, filter_col_lo<S, MODE>(), filter_col_hi<S, MODE>()>(p.L);
    const size_t fixed = p.has_ar ? filter_static_lds<S, true, MODE>() : filter_static_lds<S, false, MODE>();
    const dim3 fg(lc.grid), fb(kBlock);
    if (pas + lc.lds_bytes + fixed > kLdsBlockMax) {
        if (p.has_ar) hipLaunchKernelGGL((filter_kernel<S, R, true, true, MODE>), fg, fb, pas, st, p);
        else hipLaunchKernelGGL((filter_kernel<S, R, false, true, MODE>), fg, fb, pas, st, p);
    } else {
        const size_t lds = pas + lc.lds_bytes;
        if (p.has_ar) hipLaunchKernelGGL((filter_kernel<S, R, true, false, MODE>), fg, fb, lds, st, p);
        else hipLaunchKernelGGL((filter_kernel<S, R, false, false, MODE>), fg, fb, lds, st, p);
    }
    return hipGetLastError();
}

template <int S, typename R>
hipError_t launch_bounded_s(const KParams &p, const LaunchCfg &lc, hipStream_t st, uint32_t publish) {
    hipError_t e;
    if constexpr (filter_prefix<S>() > 0) {
        e = launch_filter_s<S, R, kFilterPrefix>(p, lc, st);
        if (e == hipSuccess) e = launch_filter_s<S, R, kFilterGather>(p, lc, st);
    } else {
        e = launch_filter_s<S, R, kFilterFull>(p, lc, st);
    }
    if (e != hipSuccess) return e;
    const uint32_t nseg = lc.grid;
    const dim3 g(lc.grid2), b(kBlock);
    const size_t sl = (size_t)p.ent_lds + ((size_t)nseg + 1) * 4;
    if (sl > kLdsBlockMax || lc.grid2 == 0) return hipErrorInvalidValue;
    const bool sch = p.sched != 0;
    if (p.has_ar && sch) hipLaunchKernelGGL((surv_kernel<S, true, true>), g, b, sl, st, p, publish, nseg);
    else if (p.has_ar) hipLaunchKernelGGL((surv_kernel<S, true, false>), g, b, sl, st, p, publish, nseg);
    else if (sch) hipLaunchKernelGGL((surv_kernel<S, false, true>), g, b, sl, st, p, publish, nseg);
    else hipLaunchKernelGGL((surv_kernel<S, false, false>), g, b, sl, st, p, publish, nseg);
    return hipGetLastError();
}

// Resident blocks per CU of the early-stop filter instances launch_bounded_s
// picks (their LDS: the Pascal columns plus the stage entries of `ent_lds`);
// with two modes the smaller of their counts, so that the second runs its
// blocks, one per segment of the first's list, in one wave too.
template <int S, typename R, int MODE>
hipError_t filter_occupancy_mode(const KParams &p, size_t ent_lds, int *blocks) {
    const size_t pas = pascal_bytes<S, R, filter_col_lo<S, MODE>(), filter_col_hi<S, MODE>()>(p.L);
    const size_t fixed = p.has_ar ? filter_static_lds<S, true, MODE>() : filter_static_lds<S, false, MODE>();
    if (pas + ent_lds + fixed > kLdsBlockMax) {
        if (p.has_ar) return hipOccupancyMaxActiveBlocksPerMultiprocessor(blocks, filter_kernel<S, R, true, true, MODE>, kBlock, pas);
        return hipOccupancyMaxActiveBlocksPerMultiprocessor(blocks, filter_kernel<S, R, false, true, MODE>, kBlock, pas);
    }
    if (p.has_ar)
        return hipOccupancyMaxActiveBlocksPerMultiprocessor(blocks, filter_kernel<S, R, true, false, MODE>, kBlock, pas + ent_lds);
    return hipOccupancyMaxActiveBlocksPerMultiprocessor(blocks, filter_kernel<S, R, false, false, MODE>, kBlock, pas + ent_lds);
}

template <int S, typename R>
hipError_t filter_occupancy_s(const KParams &p, size_t ent_lds, int *blocks) {
    if constexpr (filter_prefix<S>() > 0) {
        int a = 0, b = 0;
        hipError_t e = filter_occupancy_mode<S, R, kFilterPrefix>(p, ent_lds, &a);
        if (e == hipSuccess) e = filter_occupancy_mode<S, R, kFilterGather>(p, ent_lds, &b);
        *blocks = a < b ? a : b;
        return e;
    } else {
        return filter_occupancy_mode<S, R, kFilterFull>(p, ent_lds, blocks);
    }
}

// Resident blocks per CU of the kernel that evaluates a problem's candidates
// (`blocks`) and, with the closed form, of full_kernel (`full`).
template <int S>
hipError_t occupancy_s(const KParams &p, size_t lds, int *blocks, int *full) {
    return with_variant(p, [&](auto arc, auto schc) {
        constexpr bool ar = decltype(arc)::value, sch = decltype(schc)::value;
        if (!p.closed) {
            *full = 0;
            if (p.nslots) return hipOccupancyMaxActiveBlocksPerMultiprocessor(blocks, eval_kernel<S, ar, sch, true>, kBlock, lds);
            return hipOccupancyMaxActiveBlocksPerMultiprocessor(blocks, eval_kernel<S, ar, sch, false>, kBlock, lds);
        }
        const hipError_t e = hipOccupancyMaxActiveBlocksPerMultiprocessor(blocks, closed_kernel<S, ar, sch>, kBlock, lds);
        if (e != hipSuccess) return e;
        return hipOccupancyMaxActiveBlocksPerMultiprocessor(full, full_kernel<S, ar, sch>, kBlock, lds);
    });
}

}  // namespace pk

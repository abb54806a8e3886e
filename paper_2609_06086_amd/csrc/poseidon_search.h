#pragma once
// Device code of the pruned configuration search (Sec. 4.2.3): stage-level
// pruning with Eq. 2 (Theorem 1) and layer-level pruning with the ridge
// pattern (Theorem 2) over partial configurations, level by level.
//
// A frontier node is a partial configuration of one assignment row: the
// row and the cut codes of stages 1..x (one byte per cut).  Every quantity
// the tests need (prefix forward time, the inner max of Eq. 2, the last
// backward time, the ridge state of a type) is recomputed from the cuts and
// the LDS prefix tables, so a node is 4 + 4 * ceil((S-1)/4) bytes.
//
// Level x -> x+1 runs two kernels over the frontier.  The children of a node
// are the end points hi = c_x+1, c_x+2, ... of stage x+1 up to the first
// one that fails a test: the memory sum and g(S_{x+1}) only grow with hi,
// and once a type's counts are falling the ridge test fails for every
// larger count too, so the accepted children form one contiguous range,
// whose length a binary search finds.
// search_count_kernel counts them per block; search_scan_kernel turns the
// block counts into offsets; search_write_kernel writes the children in
// node order (a block-local scan places each node's range), so the next
// frontier is again in search order (row, then composition rank).  The
// nodes of level S-3 go to search_last_kernel, which expands them through the
// level that fixes the last cut, tests the last stage, which that cut
// determines, and evaluates the configurations that pass, so neither of the
// two widest levels is written.  search_leaf_kernel evaluates the single
// configurations of S = 1.
#include "poseidon_kernels.h"

namespace pk {

constexpr uint32_t kSearchRidge = 1u, kSearchNoStage = 2u;

struct SearchNode {
    uint32_t row, lo, t;          // row, c_x, type of stage x+1
    uint32_t pre_f, inner, last_b;
    int32_t last_l;               // last layer count of type t among stages 1..x (-1: none)
    bool falling;                 // type t's counts have started to fall
    uint32_t tS;                  // type of stage S, with its ridge state over stages 1..x
    int32_t last_lS;
    bool fallingS;
    uint32_t tN;                  // type of stage x+2, with its ridge state over stages 1..x
    int32_t last_lN;              // (what a child's own stage test needs)
    bool fallingN;
};

// Prefix quantities of a node at level x (stages 1..x fixed).
template <int S, bool AR>
__device__ __forceinline__ SearchNode search_node(const KParams &p, const Lds &tab, uint32_t row,
                                                  const uint32_t (&w)[Codes<S>::kWords], uint32_t x,
                                                  uint32_t (&ty)[S], uint32_t (&cut)[S + 1]) {
    decode_types<S>(p, row, ty);
    cut[0] = 0;
#pragma unroll
    for (int s = 1; s < S; ++s) cut[s] = (w[(s - 1) >> 2] >> (8 * ((s - 1) & 3))) & 0xFFu;
    cut[S] = p.L;
    SearchNode n;
    n.row = row;
    n.lo = 0;
    n.t = ty[0];
    n.pre_f = 0;
    n.inner = 0;
    n.last_b = 0;
#pragma unroll
    for (int s = 0; s < S; ++s) {
        if ((uint32_t)s == x) { n.lo = cut[s]; n.t = ty[s]; }
    }
    n.last_l = -1;
    n.falling = false;
    n.tS = ty[S - 1];
    n.last_lS = -1;
    n.fallingS = false;
    n.tN = ty[0];
#pragma unroll
    for (int s = 0; s < S; ++s) {
        if ((uint32_t)s == x + 1) n.tN = ty[s];
    }
    n.last_lN = -1;
    n.fallingN = false;
    const uint32_t row_len = p.L + 1;
#pragma unroll
    for (int s = 0; s < S; ++s) {
        if ((uint32_t)s < x) {
            const uint64_t *c = tab.cost + ty[s] * row_len;
            const uint64_t hi = c[cut[s + 1]], lo = c[cut[s]];
            const uint32_t f = (uint32_t)hi - (uint32_t)lo, b = (uint32_t)(hi >> 32) - (uint32_t)(lo >> 32);
            const uint32_t d = AR ? tab.pd[ty[s] * row_len + cut[s + 1]] - tab.pd[ty[s] * row_len + cut[s]] : 0u;
            n.inner = s == 0 ? d : max(n.inner + n.last_b, d);
            n.pre_f += f;
            n.last_b = b;
            const int32_t l = (int32_t)(cut[s + 1] - cut[s]);
            if (ty[s] == n.t) {
                if (n.last_l >= 0 && l < n.last_l) n.falling = true;
                n.last_l = l;
            }
            if (ty[s] == n.tS) {
                if (n.last_lS >= 0 && l < n.last_lS) n.fallingS = true;
                n.last_lS = l;
            }
            if (ty[s] == n.tN) {
                if (n.last_lN >= 0 && l < n.last_lN) n.fallingN = true;
                n.last_lN = l;
            }
        }
    }
    return n;
}

// The child of a node at level x with stage x+1 = [lo, c): its prefix
// quantities at level x+1, extended by that one stage (the type of its
// stage x+3 is not tracked: used for the level that fixes the last cut,
// whose children are complete).
template <bool AR>
__device__ __forceinline__ SearchNode search_child(const KParams &p, const Lds &tab, const SearchNode &n, uint32_t x,
                                                   uint32_t c) {
    const uint32_t row_len = p.L + 1;
    const uint64_t *ct = tab.cost + n.t * row_len;
    const uint64_t ch = ct[c], cl = ct[n.lo];
    const uint32_t f = (uint32_t)ch - (uint32_t)cl, b = (uint32_t)(ch >> 32) - (uint32_t)(cl >> 32);
    const uint32_t d = AR ? tab.pd[n.t * row_len + c] - tab.pd[n.t * row_len + n.lo] : 0u;
    const int32_t l = (int32_t)(c - n.lo);
    SearchNode m = n;
    m.lo = c;
    m.t = n.tN;
    m.inner = x == 0 ? d : max(n.inner + n.last_b, d);
    m.pre_f = n.pre_f + f;
    m.last_b = b;
    m.last_l = n.last_lN;
    m.falling = n.fallingN;
    if (n.t == n.tN) {
        m.falling = m.falling || (m.last_l >= 0 && l < m.last_l);
        m.last_l = l;
    }
    if (n.t == n.tS) {
        m.fallingS = m.fallingS || (m.last_lS >= 0 && l < m.last_lS);
        m.last_lS = l;
    }
    return m;
}

// Outcome of trying stage x+1 = [lo, hi): 0 accepted, 1 memory, 2 ridge, 3 bound.
template <bool AR>
__device__ __forceinline__ int search_try(const KParams &p, const Lds &tab, const SearchNode &n, uint32_t x,
                                          uint32_t hi, uint32_t flags, uint32_t bound) {
    const uint32_t row_len = p.L + 1;
    if (tab.pm[hi] - tab.pm[n.lo] > tab.cap[n.t]) return 1;
    const int32_t l = (int32_t)(hi - n.lo);
    if ((flags & kSearchRidge) && n.last_l >= 0 && n.falling && l > n.last_l) return 2;
    if (!(flags & kSearchNoStage)) {
        const uint64_t *c = tab.cost + n.t * row_len;
        const uint64_t ch = c[hi], cl = c[n.lo];
        const uint32_t f = (uint32_t)ch - (uint32_t)cl, b = (uint32_t)(ch >> 32) - (uint32_t)(cl >> 32);
        const uint32_t d = AR ? tab.pd[n.t * row_len + hi] - tab.pd[n.t * row_len + n.lo] : 0u;
        const uint32_t inn = x == 0 ? d : max(n.inner + n.last_b, d);
        // Eq. 2: g(S_{x+1}) = sum_{i<=x} F_i + M (F_{x+1} + B_{x+1}) + inner
        if (n.pre_f + p.M * (f + b) + inn > bound) return 3;
    }
    return 0;
}

// Per-type tables of the stage tests, built in LDS behind the stage tables
// by the count kernel and the last pass: fb = prefix fwd + prefix bwd, mfb = M fb
// (below 2^31 like every path weight, checked at load), and hm[t][lo] = the
// largest h with layers [lo, h) within type t's memory cap.  Without
// all-reduce times a stage's Eq. 2 test is then one compare, mfb[h] against
// a per-node threshold, and its memory test a cap on the range.
struct SearchTab {
    const uint32_t *fb, *mfb, *hm;
};

// LDS bytes of the stage tables (the layout of stage_tables), where the
// search tables start; the host sizes the launch the same way.
__device__ __forceinline__ uint32_t search_tab_offset(const KParams &p) {
    const uint32_t n = p.T * (p.L + 1);
    return (n * 8 + (p.L + 1) * 4 + p.T * 4 + (p.has_ar ? n * 4 : 0) + 15) & ~15u;
}

// where search_last_kernel's stage entries start, behind the search tables
__device__ __forceinline__ uint32_t search_ent_offset(const KParams &p) {
    return search_tab_offset(p) + ((3 * p.T * (p.L + 1) * 4 + 15) & ~15u);
}

__device__ __forceinline__ SearchTab search_tables(const KParams &p, const Lds &tab, unsigned char *smem) {
    const uint32_t row = p.L + 1, n = p.T * row;
    uint32_t *fb = reinterpret_cast<uint32_t *>(smem + search_tab_offset(p)), *mfb = fb + n, *hm = mfb + n;
    for (uint32_t i = threadIdx.x; i < n; i += kBlock) {
        const uint64_t c = tab.cost[i];
        const uint32_t v = (uint32_t)c + (uint32_t)(c >> 32);
        fb[i] = v;
        mfb[i] = p.M * v;
        const uint32_t t = i / row, lo = i - t * row;
        // pm only grows: the largest h that fits, by halving steps from lo
        uint32_t h = lo;
        for (uint32_t st = 256; st; st >>= 1)
            if (h + st <= p.L && tab.pm[h + st] - tab.pm[lo] <= tab.cap[t]) h += st;
        hm[i] = h;
    }
    __syncthreads();
    return SearchTab{fb, mfb, hm};
}

// The rule that ended a node's accepted range of k end points (0: it ran to
// hmax): the first test end point lo+k+1 fails, in the order memory, ridge,
// bound.  Without all-reduce times the memory and ridge outcomes are range
// limits, and a maximal range that neither ended must have met the bound.
template <bool AR>
__device__ __forceinline__ int search_stop(const KParams &p, const Lds &tab, const SearchTab &sx,
                                           const SearchNode &n, uint32_t x, uint32_t k, uint32_t hmax,
                                           uint32_t flags, uint32_t bound) {
    const uint32_t h = n.lo + k + 1;
    if (h > hmax) return 0;
    if (AR) return search_try<AR>(p, tab, n, x, h, flags, bound);
    if (h > sx.hm[n.t * (p.L + 1) + n.lo]) return 1;
    if ((flags & kSearchRidge) && n.last_l >= 0 && n.falling && (int32_t)(h - n.lo) > n.last_l) return 2;
    return 3;
}

// Outcomes of the last-stage test of the children of one node.
struct LastStage {
    uint32_t pass = 0, mem = 0, ridge = 0, bound = 0;
};

// Number k of accepted choices of stage x+1: the end points lo+1 .. lo+k
// pass the memory, ridge and Eq. 2 tests and lo+k+1 (if <= hmax) fails one.
// Each test, once failed, fails for every larger end point (the memory sum
// and g(S_{x+1}) only grow with it; a falling type's ridge test fails for
// every count above its last one), so k is found by a binary search over
// the end points instead of trying them one by one.
template <bool AR>
__device__ __forceinline__ uint32_t search_accepted(const KParams &p, const Lds &tab, const SearchTab &sx,
                                                    const SearchNode &n, uint32_t x, uint32_t hmax, uint32_t flags,
                                                    uint32_t bound) {
    const uint32_t row_len = p.L + 1;
    uint32_t len = hmax - n.lo;
    if ((flags & kSearchRidge) && n.last_l >= 0 && n.falling) len = min(len, (uint32_t)n.last_l);
    const int H = (int)decode_levels(p.L);   // (uniform: the steps above it are skipped by scalar branches)
    if (!AR) {
        // memory caps the range; Eq. 2, pre_f + M (fb[h] - fb[lo]) + inn <= bound
        // with inn = inner + last_b (0 for the first stage), is mfb[h] <= thr
        const uint32_t *mf = sx.mfb + n.t * row_len;
        len = min(len, sx.hm[n.t * row_len + n.lo] - n.lo);
        if (flags & kSearchNoStage) return len;
        const int64_t thr64 = (int64_t)bound + mf[n.lo] - n.pre_f - (x == 0 ? 0u : n.inner + n.last_b);
        const int32_t thr = thr64 > INT32_MAX ? INT32_MAX : thr64 < 0 ? -1 : (int32_t)thr64;
        // each step loads (an in-range entry) and combines its tests without
        // branches, so the wave never splits over them
        uint32_t k = 0;
#pragma unroll
        for (int b = 7; b >= 0; --b) {
            if (b >= H) continue;
            const uint32_t t = k + (1u << b);
            const int32_t v = (int32_t)mf[n.lo + min(t, len)];
            k = ((t <= len) & (v <= thr)) ? t : k;
        }
        return k;
    }
    const uint64_t *ct = tab.cost + n.t * row_len;
    const uint64_t cl = ct[n.lo];
    const uint32_t pml = tab.pm[n.lo], capt = tab.cap[n.t];
    // with all-reduce times: each probe evaluates the memory and Eq. 2 tests
    const uint32_t *pdt = tab.pd + n.t * row_len;
    const uint32_t dl = pdt[n.lo];
    const bool stage = !(flags & kSearchNoStage);
    const uint32_t carry = n.inner + n.last_b;
    uint32_t k = 0;
#pragma unroll
    for (int b = 7; b >= 0; --b) {
        if (b >= H) continue;
        const uint32_t t = k + (1u << b);
        const uint32_t h = n.lo + min(t, len);
        bool ok = tab.pm[h] - pml <= capt;
        if (stage) {
            const uint64_t ch = ct[h];
            const uint32_t f = (uint32_t)ch - (uint32_t)cl, bw = (uint32_t)(ch >> 32) - (uint32_t)(cl >> 32);
            const uint32_t d = pdt[h] - dl;
            const uint32_t inn = x == 0 ? d : max(carry, d);
            ok = ok && n.pre_f + p.M * (f + bw) + inn <= bound;
        }
        k = (t <= len && ok) ? t : k;
    }
    return k;
}

// Children lo+1 .. lo+k of a node at the level that fixes the last cut
// (x + 2 == S): each fixes every cut, so the last stage [hi, L) is tested
// here (memory in closed form through last_lo, then ridge, then Eq. 2) and
// only children that pass it are kept; lp counts the outcomes.
// search_last_range gives the kept ones as a range [g0, h1] (its return
// value is their number) where the closed form below applies; elsewhere
// search_last_test tries one end point.
//
// Without all-reduce times the last stage's Eq. 2 splits into a per-node
// constant and a function of hi alone:
//   g(S_S) = C + G(hi),  G(hi) = Pf_t[hi] + Pb_t[hi] - M (Pf_tS[hi] + Pb_tS[hi])
// (t, tS the types of stages S-1 and S, Pf / Pb the prefix times).  G falls
// as hi grows when no layer's forward + backward time on t exceeds M times
// that on tS (checked per type pair on the host: bit 8 t + tS of p.g_mono), and the
// last stage's ridge test fails on a prefix of the end points too, so then
// every outcome count is a range length: the ridge prefix in closed form,
// the bound prefix by a binary search.  Otherwise the end points are tried
// one by one.
template <int S>
__device__ __forceinline__ void search_write_child(const SearchParams &q, uint64_t o, uint32_t row, uint32_t x,
                                                   uint32_t hi, const uint32_t (&w)[Codes<S>::kWords]) {
    q.out_row[o] = row;
#pragma unroll
    for (int k = 0; k < Codes<S>::kWords; ++k) {
        const uint32_t v = (uint32_t)k == (x >> 2) ? (w[k] | (hi << (8 * (x & 3)))) : w[k];
        q.out_codes[(uint64_t)k * q.out_cap + o] = v;
    }
}

// the end points memory allows: hi < last_lo[type] exceeds the last stage's cap
__device__ __forceinline__ void search_last_limits(const KParams &p, const SearchNode &n, uint32_t k, LastStage &lp,
                                                   uint32_t &h0, uint32_t &h1) {
    h0 = max(n.lo + 1, p.last_lo[n.tS]);
    h1 = n.lo + k;
    lp.mem += (h0 <= h1 ? h0 : h1 + 1) - (n.lo + 1);
}

__device__ __forceinline__ uint32_t search_last_range(const KParams &p, const SearchTab &sx, const SearchNode &n,
                                                      uint32_t x, uint32_t h0, uint32_t h1, uint32_t flags,
                                                      uint32_t bound, LastStage &lp, uint32_t &g0out) {
    const uint32_t row_len = p.L + 1;
    const bool ridge = (flags & kSearchRidge) != 0, stage = !(flags & kSearchNoStage);
    const bool same = n.t == n.tS;
    if (h0 > h1) return 0;
    // ridge: the end points below r0 fail
    uint32_t r0 = h0;
    if (ridge) {
        if (same) {
            // counts of type t fall before lo + last_lS (or throughout), and the
            // last stage is then longer than stage S-1 below ceil((L + lo) / 2)
            const uint32_t e1 = (p.L + n.lo + 1) / 2;
            const uint32_t e2 = n.fallingS ? 0xFFFFFFFFu : (n.last_lS >= 0 ? n.lo + (uint32_t)n.last_lS : 0u);
            r0 = max(h0, min(e1, e2));
        } else if (n.last_lS >= 0 && n.fallingS) {
            r0 = max(h0, p.L - (uint32_t)n.last_lS);
        }
        r0 = min(r0, h1 + 1);
        lp.ridge += r0 - h0;
    }
    // Eq. 2: the end points below g0 fail
    uint32_t g0 = r0;
    if (stage && r0 <= h1) {
        const uint32_t *ft = sx.fb + n.t * row_len, *ms = sx.mfb + n.tS * row_len;
        // g(hi) = C + G(hi), G(hi) = fb_t[hi] - mfb_tS[hi].  g is an Eq. 2
        // value, below 2^31 like every path weight (checked at load), so
        // C + G evaluates exactly in 32-bit modular arithmetic
        const uint32_t C = n.pre_f - ft[n.lo] + (x == 0 ? 0u : n.inner + n.last_b) + ms[p.L];
        const uint32_t len = h1 + 1 - r0;
        // g is smallest at h1: if even that fails, every end point does
        // (the usual case, so the search below mostly runs on no lane)
        uint32_t j = len;
        if (C + ft[h1] - ms[h1] <= bound) {
            const int H = (int)decode_levels(p.L);
            j = 0;
#pragma unroll
            for (int b = 7; b >= 0; --b) {
                if (b >= H) continue;
                const uint32_t t = j + (1u << b);
                const uint32_t h = r0 + min(t, len) - 1;
                j = ((t <= len) & (C + ft[h] - ms[h] > bound)) ? t : j;
            }
        }
        g0 = r0 + j;
        lp.bound += j;
    }
    lp.pass += h1 + 1 - g0;
    g0out = g0;
    return h1 + 1 - g0;
}

// The constant C of a node's g(hi) = C + fb_t[hi] - mfb_tS[hi] (above; the
// formula itself needs no monotone pair), without all-reduce times.
struct SearchLast {
    uint32_t C;
};
template <bool AR>
__device__ __forceinline__ SearchLast search_last_one(const KParams &p, const SearchTab &sx, const SearchNode &n, uint32_t x) {
    if constexpr (AR) return SearchLast{0u};
    const uint32_t row_len = p.L + 1;
    return SearchLast{n.pre_f - sx.fb[n.t * row_len + n.lo] + (x == 0 ? 0u : n.inner + n.last_b) + sx.mfb[n.tS * row_len + p.L]};
}

template <bool AR>
__device__ __forceinline__ bool search_last_test(const KParams &p, const Lds &tab, const SearchTab &sx, const SearchNode &n,
                                                 const SearchLast &one, uint32_t x, uint32_t hi, uint32_t flags,
                                                 uint32_t bound, LastStage &lp) {
    const uint32_t row_len = p.L + 1;
    if (flags & kSearchRidge) {
        // type tS's counts with stage x+1 appended when it has that type
        const int32_t l = (int32_t)(hi - n.lo);
        int32_t ll = n.last_lS;
        bool fall = n.fallingS;
        if (n.t == n.tS) {
            fall = fall || (ll >= 0 && l < ll);
            ll = l;
        }
        if (ll >= 0 && fall && (int32_t)(p.L - hi) > ll) {
            lp.ridge += 1;
            return false;
        }
    }
    if (!(flags & kSearchNoStage)) {
        uint32_t g;
        if constexpr (!AR) {
            g = one.C + sx.fb[n.t * row_len + hi] - sx.mfb[n.tS * row_len + hi];
        } else {
            const uint64_t *ct = tab.cost + n.t * row_len, *cs = tab.cost + n.tS * row_len;
            const uint64_t cl = ct[n.lo], cL = cs[p.L], ch = ct[hi], sh = cs[hi];
            const uint32_t f = (uint32_t)ch - (uint32_t)cl, b = (uint32_t)(ch >> 32) - (uint32_t)(cl >> 32);
            const uint32_t d = tab.pd[n.t * row_len + hi] - tab.pd[n.t * row_len + n.lo];
            const uint32_t inn = x == 0 ? d : max(n.inner + n.last_b, d);
            const uint32_t fS = (uint32_t)cL - (uint32_t)sh, bS = (uint32_t)(cL >> 32) - (uint32_t)(sh >> 32);
            const uint32_t dS = tab.pd[n.tS * row_len + p.L] - tab.pd[n.tS * row_len + hi];
            // Eq. 2 for the last stage: g(S_S) = sum_{i<S} F_i + M (F_S + B_S) + max(inner + B_{S-1}, d_S)
            g = n.pre_f + f + p.M * (fS + bS) + max(inn + b, dS);
        }
        if (g > bound) {
            lp.bound += 1;
            return false;
        }
    }
    lp.pass += 1;
    return true;
}

__device__ __forceinline__ void search_flush(const SearchParams &q, unsigned int visited, unsigned int evaluated,
                                             unsigned int mem, unsigned int ridge, unsigned int bound) {
    __shared__ unsigned int c[5];
    if (threadIdx.x < 5) c[threadIdx.x] = 0;
    __syncthreads();
    if (visited) atomicAdd(&c[0], visited);
    if (evaluated) atomicAdd(&c[1], evaluated);
    if (mem) atomicAdd(&c[2], mem);
    if (ridge) atomicAdd(&c[3], ridge);
    if (bound) atomicAdd(&c[4], bound);
    __syncthreads();
    if (threadIdx.x < 5 && c[threadIdx.x]) atomicAdd(&q.stats[threadIdx.x], (unsigned long long)c[threadIdx.x]);
}

// The count kernel's counters: summed over the block in LDS, then one
// atomic per counter into the block's slot of q.stats_part.
__device__ __forceinline__ void search_block_counts(const SearchParams &q, unsigned int visited, unsigned int evaluated,
                                                    unsigned int mem, unsigned int ridge, unsigned int bound) {
    __shared__ unsigned int c[5];
    if (threadIdx.x < 5) c[threadIdx.x] = 0;
    __syncthreads();
    if (visited) atomicAdd(&c[0], visited);
    if (evaluated) atomicAdd(&c[1], evaluated);
    if (mem) atomicAdd(&c[2], mem);
    if (ridge) atomicAdd(&c[3], ridge);
    if (bound) atomicAdd(&c[4], bound);
    __syncthreads();
    if (threadIdx.x < 5 && c[threadIdx.x])
        atomicAdd(&q.stats_part[threadIdx.x * kStatSlots + blockIdx.x % kStatSlots], (unsigned long long)c[threadIdx.x]);
}

template <int S>
__device__ __forceinline__ void search_load(const SearchParams &q, uint32_t i, bool active, uint32_t &row,
                                            uint32_t (&w)[Codes<S>::kWords]) {
    row = active ? q.in_row[i] : 0u;
#pragma unroll
    for (int k = 0; k < Codes<S>::kWords; ++k) w[k] = active ? q.in_codes[(uint64_t)k * q.in_cap + i] : 0u;
}

// Nodes of the level: counted on the device by the previous level's scan
// when the host launched on an upper bound (q.n_dev), else q.n_in.
__device__ __forceinline__ uint32_t search_n_in(const SearchParams &q) {
    return q.n_dev ? (uint32_t)*q.n_dev : q.n_in;
}

// Count the children of every node of the piece; one total per block.  The
// kernel waits on chains of dependent LDS loads (binary searches), so it
// asks for 7 waves per SIMD (72 VGPRs, no spills for any S) rather than the
// compiler's choice of 6.
template <int S, bool AR>
__global__ __launch_bounds__(kBlock) __attribute__((amdgpu_waves_per_eu(7, 8))) void search_count_kernel(KParams p, SearchParams q) {
    extern __shared__ __align__(16) unsigned char smem[];
    const uint32_t n_in = search_n_in(q);
    if (blockIdx.x * kBlock >= n_in) {
        // a block past the level's nodes (grid from an upper bound): zero total
        if (threadIdx.x == 0) q.blk_tot[blockIdx.x] = 0;
        return;
    }
    const Lds tab = stage_tables(p, smem);
    const SearchTab sx = search_tables(p, tab, smem);
    const uint32_t i = blockIdx.x * kBlock + threadIdx.x;
    const bool active = i < n_in;
    const uint32_t bound = *q.bound;
    uint32_t row, w[Codes<S>::kWords], ty[S], cut[S + 1];
    search_load<S>(q, i, active, row, w);
    uint32_t cnt = 0, why_mem = 0, why_ridge = 0, why_bound = 0;
    if (active) {
        const uint32_t x = q.level;
        const SearchNode n = search_node<S, AR>(p, tab, row, w, x, ty, cut);
        const uint32_t hmax = p.L - (S - 1 - x);   // every later stage keeps one layer
        cnt = search_accepted<AR>(p, tab, sx, n, x, hmax, q.flags, bound);
        // the rule that stopped the range (0: it ran to its structural end)
        const int why = search_stop<AR>(p, tab, sx, n, x, cnt, hmax, q.flags, bound);
        why_mem = why == 1;
        why_ridge = why == 2;
        why_bound = why == 3;
        q.node_cnt[i] = (uint16_t)cnt;   // at most L - 1 children
    }
    __shared__ unsigned int tot;
    if (threadIdx.x == 0) tot = 0;
    __syncthreads();
    const unsigned int wsum = (unsigned int)wave_sum_u32(cnt);
    if ((threadIdx.x & 63) == 0 && wsum) atomicAdd(&tot, wsum);
    search_block_counts(q, cnt, 0, why_mem, why_ridge, why_bound);
    if (threadIdx.x == 0) q.blk_tot[blockIdx.x] = tot;
}

// Write the children of blocks [blk_base, blk_base + gridDim.x) in node
// order, the first one at position 0 of the output.
template <int S>
__global__ __launch_bounds__(kBlock) void search_write_kernel(KParams p, SearchParams q) {
    const uint32_t blk = q.blk_base + blockIdx.x;
    const uint32_t n_in = search_n_in(q);
    if (blk * kBlock >= n_in) return;   // past the level's nodes
    constexpr int NW = Codes<S>::kWords;
    const uint32_t i = blk * kBlock + threadIdx.x;
    const bool active = i < n_in;
    const uint32_t x = q.level;
    // the count kernel left each node's number of children
    const uint32_t cnt = active ? q.node_cnt[i] : 0u;
    unsigned long long total;
    const unsigned long long local = block_exclusive_scan_u64(cnt, total);
    if (total == 0) return;   // no child in the block
    const uint64_t blk0 = q.blk_off[blk] - q.blk_off[q.blk_base];
    // every accepted choice is a child: c_{x+1} = lo+1 .. lo+cnt.  The
    // wave writes the children of its nodes together, 64 consecutive ones
    // per store: lane j takes child o0 + j of the wave's run, and its
    // parent is the first lane whose inclusive count exceeds that
    // (a binary search over the lanes)
    uint32_t row, w[NW];
    search_load<S>(q, i, active, row, w);
    uint32_t lo = 0;
#pragma unroll
    for (int s = 1; s < S; ++s)
        if ((uint32_t)s == x) lo = (w[(s - 1) >> 2] >> (8 * ((s - 1) & 3))) & 0xFFu;
    const uint32_t lane = threadIdx.x & 63;
    const unsigned long long l0 = __shfl(local, 0, 64);
    const uint32_t incl = (uint32_t)(local - l0) + cnt;
    const uint32_t wtot = __shfl(incl, 63, 64);
    for (uint32_t o0 = 0; o0 < wtot; o0 += 64) {
        const uint32_t o = o0 + lane;
        uint32_t pl = 0;
#pragma unroll
        for (uint32_t b = 32; b; b >>= 1) pl = __shfl(incl, (int)(pl + b - 1), 64) <= o ? pl + b : pl;
        const uint32_t first = __shfl(incl - cnt, (int)pl, 64);
        const uint32_t prow = __shfl(row, (int)pl, 64), plo = __shfl(lo, (int)pl, 64);
        uint32_t pw[NW];
#pragma unroll
        for (int k = 0; k < NW; ++k) pw[k] = __shfl(w[k], (int)pl, 64);
        if (o < wtot) search_write_child<S>(q, blk0 + l0 + o, prow, x, plo + 1 + (o - first), pw);
    }
}

// c_{S-1} of complete cut codes
template <int S>
__device__ __forceinline__ uint32_t last_cut(const uint32_t (&w)[Codes<S>::kWords]) {
    return (w[(S - 2) / 4] >> (8 * ((S - 2) % 4))) & 0xFFu;
}

// The block's best of its threads' bests, (key, last cut) the smallest, with
// the configuration that has it, to the block's slot.
template <int S>
struct BlockBest {
    unsigned long long key[kWaves];
    uint32_t sub[kWaves], row[kWaves], w[kWaves][Codes<S>::kWords];
};
template <int S>
__device__ __forceinline__ void block_best(const SearchParams &q, unsigned long long best, uint32_t bsub, uint32_t brow,
                                           const uint32_t (&bw)[Codes<S>::kWords], BlockBest<S> &sh) {
    constexpr int NW = Codes<S>::kWords;
    const uint32_t lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const unsigned long long wbest = wave_min(best);
    uint32_t s = best == wbest ? bsub : 0xFFFFFFFFu;
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1) s = min(s, (uint32_t)__shfl_xor((int)s, o, 64));
    const unsigned long long win = __ballot(best == wbest && bsub == s);
    if (lane == (uint32_t)__ffsll((long long)win) - 1u) {
        sh.key[wave] = wbest;
        sh.sub[wave] = s;
        sh.row[wave] = brow;
#pragma unroll
        for (int k = 0; k < NW; ++k) sh.w[wave][k] = bw[k];
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        int v = 0;
#pragma unroll
        for (int k = 1; k < kWaves; ++k) v = sh.key[k] < sh.key[v] || (sh.key[k] == sh.key[v] && sh.sub[k] < sh.sub[v]) ? k : v;
        q.slot_key[blockIdx.x] = sh.key[v];
        q.slot_row[blockIdx.x] = sh.row[v];
#pragma unroll
        for (int k = 0; k < NW; ++k) q.slot_w[k * kSlotMax + blockIdx.x] = sh.w[v][k];
        if (sh.key[v] != ~0ull) atomicMin(q.acc, sh.key[v]);
    }
}

constexpr uint32_t kRunCap = 192;   // runs a wave gathers: handed out from 128 on
template <int S>
struct LastPend {
    uint32_t row[128], at[128], low[128], w[Codes<S>::kWords][128];
};
template <int S>
struct LastLds {
    uint32_t run[kWaves][kRunCap];
    LastPend<S> pend[kWaves];
    unsigned long long known;
    BlockBest<S> best;
};

// The last levels in one pass: the nodes of level S-3 (S >= 3), or S-2
// (S = 2), are expanded through the level that fixes the last cut, and the
// complete configurations that pass the last stage are evaluated at once, so
// the widest level is neither written nor read, needs no frontier memory and
// no host round trip per piece of it.  The kept end points of one choice of
// stage S-1 are a run [hi0, hi0 + cnt), and the wave's runs gather in LDS
// until it hands them out, 64 configurations at a time whichever node they
// come from.  Most configurations end with their closed form; see Pend for
// the others.  Ties go to the first in search order: (node, end point of
// stage S-2's choice, last cut).
//
// The pass's unit is an item: one of the `parts` equal shares of a node's
// choices of stage S-2 (choices part + 1, part + 1 + parts, ..).  A wave
// takes `width` items at a time.  With nodes for every lane of the grid a
// node is one item.  With fewer, its choices spread over as many lanes as the
// grid has, and the items over as many waves: one node of a 200-layer model
// has 2e4 configurations, and a lane that expands them all and a wave that
// hands them out leave the chip waiting (one row of 3 stages, 574 us so and
// 81 now; 512 rows of 3 stages and 256 layers with all-reduce times 13.2 and
// 1.0 ms).  Parts and spread nodes where the grid is full anyway cost more
// (the 8-stage search below: 18.9 ms with 2 parts, 21 with spread nodes, 17.1):
// neighbours are alike, and most nodes have few choices.
//
// Without a closed form (!CLOSED) a configuration costs its whole recurrence,
// and the wave whose neighbours are wide would run thousands of them, so the
// pass writes them to a list that search_list_kernel evaluates with the whole
// grid (6 stages, 1 micro-batch, 1.4e6 configurations: 1.7 ms a search, 3.8
// evaluated in place); those that the list has no room for are evaluated here.
// (Before the pass: a count and a scan of those nodes, then some 90 write
// launches of 110 us, 90-170 blocks wide each, and as many leaf launches of 42
// us; the 8-stage search with 3.8e8 complete configurations took 33.9 ms, now
// 16.)  Held to 128 VGPRs for S <= 8: 299 us a launch of that search against
// 355 us at the 130 the compiler takes (3 waves a SIMD); 5 waves a SIMD spill
// in every variant and are slower at every size tried (6 and 8 stages, with
// and without all-reduce times).  At 128 the common variant of 8 stages has
// no spills, those with all-reduce times or one-by-one last stages up to 44
// registers.
template <int S, bool AR, bool MONO, bool SCH, bool CLOSED>
__global__ __launch_bounds__(kBlock) __attribute__((amdgpu_waves_per_eu(S <= 8 ? 4 : 3, 8))) void search_last_kernel(KParams p, SearchParams q) {
    extern __shared__ __align__(16) unsigned char smem[];
    const uint32_t n_in = search_n_in(q), nwave = gridDim.x * kWaves;
    const uint32_t parts = S >= 3 ? min(max(64 * nwave / max(n_in, 1u), 1u), p.L - S + 1) : 1u;   // (at most L-S+1 choices)
    const uint32_t items = n_in * parts;   // (at most the larger of n_in and the grid's lanes)
    const uint32_t width = min(max((items + nwave - 1) / nwave, 1u), 64u);
    if (blockIdx.x * kWaves * width >= items) {   // past the level's nodes
        if (threadIdx.x == 0) q.slot_key[blockIdx.x] = ~0ull;
        return;
    }
    constexpr int NW = Codes<S>::kWords;
    constexpr uint32_t x = S >= 3 ? S - 3 : 0;   // the nodes' level
    __shared__ LastLds<S> sh;
    const Lds tab = stage_tables(p, smem);
    const SearchTab sx = search_tables(p, tab, smem);
    const Ent ent_tab = entry_tables(p, smem + search_ent_offset(p));
    const Comm<S> comm = load_comm<S>(p);
    const uint32_t bound = *q.bound, lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const unsigned long long lanes_below = lane ? (~0ull >> (64 - lane)) : 0ull;
    // a makespan above the bound or not below the best of the earlier pieces
    // never becomes the result
    const unsigned long long had = q.best[0];
    const uint32_t most = had <= bound ? (had ? (uint32_t)had - 1u : 0u) : bound;
    if (threadIdx.x == 0) sh.known = (unsigned long long)most << 32 | 0xFFFFFFFFu;
    __syncthreads();
    uint32_t *run = sh.run[wave];
    LastPend<S> &pend = sh.pend[wave];
    uint32_t nrun = 0, npend = CLOSED ? 0u : blockIdx.x * kWaves + wave;   // (wave-uniform)
    // the thread's best: (T << 32 | node << 8 | end point of stage S-2's choice), then
    // the last cut, then what names it
    unsigned long long best = ~0ull;
    uint32_t bsub = 0, brow = 0, bw[NW];
#pragma unroll
    for (int k = 0; k < NW; ++k) bw[k] = 0;
    auto offer = [&](uint32_t T, uint32_t at, uint32_t row, const uint32_t (&w)[NW]) __attribute__((always_inline)) {
        const unsigned long long key = make_key(true, T, at);
        if (key > best) return;
        const uint32_t sub = last_cut<S>(w);
        if (key == best && sub >= bsub) return;
        best = key;
        bsub = sub;
        brow = row;
#pragma unroll
        for (int k = 0; k < NW; ++k) bw[k] = w[k];
        if (key < sh.known) atomicMin(&sh.known, key);
    };
    auto run_pend = [&](uint32_t first, uint32_t n) __attribute__((always_inline)) {   // the recurrence for n <= 64 kept entries
        wave_lds_sync();
        if (lane < n && (unsigned long long)pend.low[first + lane] << 32 <= sh.known) {
            const uint32_t e = first + lane, row = pend.row[e];
            uint32_t w[NW], cut[S + 1], to[S], F[S], B[S];
#pragma unroll
            for (int k = 0; k < NW; ++k) w[k] = pend.w[k][e];
            unpack_cuts<S>(w, p.L, cut);
            decode_toff<S>(p, ent_tab, row, to);
            stage_weights<S>(p, ent_tab, cut, to, F, B);
            offer(dp_full_settle<S, SCH, AR, true>(p, ent_tab, F, B, comm, w, row), pend.at[e], row, w);
        }
        wave_lds_sync();
    };
    // hand out the gathered runs (node, row, w: the lanes' nodes)
    auto hand_out = [&](uint32_t node, uint32_t row, const uint32_t (&w)[NW]) __attribute__((always_inline)) {
        wave_lds_sync();
        for (uint32_t r0 = 0; r0 < nrun; r0 += 64) {
            const uint32_t rw = r0 + lane < nrun ? run[r0 + lane] : 0u, cnt = rw >> 22;
            uint32_t incl = cnt;
#pragma unroll
            for (int o = 1; o < 64; o <<= 1) {
                const uint32_t u = __shfl_up(incl, o, 64);
                if (lane >= (uint32_t)o) incl += u;
            }
            const uint32_t total = __shfl(incl, 63, 64);
            uint32_t slot = kListCap, lpart = 0;
            if constexpr (!CLOSED) {   // room for all of them in one part of the list (the parts in turn)
                if (q.list) {
                    lpart = npend++ % kListParts;
                    if (lane == 0) slot = atomicAdd(&q.list_n[lpart], total);
                    slot = __builtin_amdgcn_readfirstlane(slot);
                }
            }
            for (uint32_t o0 = 0; o0 < total; o0 += 64) {
                const uint32_t o = o0 + lane;
                uint32_t pl = 0;   // the run that holds configuration o: the first whose inclusive count exceeds it
#pragma unroll
                for (uint32_t b = 32; b; b >>= 1) pl = __shfl(incl, (int)(pl + b - 1), 64) <= o ? pl + b : pl;
                const bool on = o < total;
                pl = on ? pl : 0u;
                const uint32_t rp = __shfl(rw, (int)pl, 64), first = __shfl(incl - cnt, (int)pl, 64);
                const uint32_t src = rp & 63u, hi = ((rp >> 14) & 0xFFu) + (on ? o - first : 0u);
                const uint32_t prow = __shfl(row, (int)src, 64);
                const uint32_t at = __shfl(node, (int)src, 64) << 8 | ((rp >> 6) & 0xFFu);
                uint32_t pw[NW];
#pragma unroll
                for (int k = 0; k < NW; ++k) pw[k] = __shfl(w[k], (int)src, 64);
                if constexpr (S >= 3) {
                    pw[x / 4] |= ((rp >> 6) & 0xFFu) << (8 * (x % 4));
                    pw[(x + 1) / 4] |= hi << (8 * ((x + 1) % 4));
                } else {
                    pw[0] |= hi;
                }
                bool eval = on;
                if constexpr (!CLOSED) {
                    // to the list, while its part has room
                    eval = on && slot + o >= kListCap;
                    if (on && !eval) {
                        uint32_t *l = q.list + lpart * kListCap + slot + o;
                        l[0] = at;
                        l[kListParts * kListCap] = prow;
#pragma unroll
                        for (int k = 0; k < NW; ++k) l[(2 + k) * kListParts * kListCap] = pw[k];
                    }
                    if (__ballot(eval) == 0) continue;
                }
                uint32_t cut[S + 1], to[S], F[S], B[S], T;
                unpack_cuts<S>(pw, p.L, cut);
                decode_toff<S>(p, ent_tab, prow, to);
                stage_weights<S>(p, ent_tab, cut, to, F, B);
                if constexpr (!CLOSED) {
                    if (eval) {
                        T = dp_full_settle<S, SCH, AR>(p, ent_tab, F, B, comm, pw, prow);
                        if (T <= bound) offer(T, at, prow, pw);
                    }
                    continue;
                }
                const bool proven = closed_or_bound<S, AR, SCH>(p, ent_tab, cut, to, F, B, T);
                if (on && proven && T <= bound) offer(T, at, prow, pw);
                const bool keep = on && !proven && (unsigned long long)T << 32 <= sh.known;
                const unsigned long long m = __ballot(keep);
                if (m) {
                    if (keep) {
                        const uint32_t e = npend + (uint32_t)__popcll(m & lanes_below);
                        pend.row[e] = prow;
                        pend.at[e] = at;
                        pend.low[e] = T;
#pragma unroll
                        for (int k = 0; k < NW; ++k) pend.w[k][e] = pw[k];
                    }
                    npend += (uint32_t)__popcll(m);
                    if (npend >= 64) {
                        npend -= 64;
                        run_pend(npend, 64u);
                    }
                }
            }
        }
        nrun = 0;
        wave_lds_sync();
    };
    uint32_t visited = 0, why_mem = 0, why_ridge = 0, why_bound = 0;
    LastStage lp;
    for (uint32_t base = (blockIdx.x * kWaves + wave) * width; base < items; base += nwave * width) {   // (wave-uniform)
        const bool active = lane < width && base + lane < items;
        const uint32_t node = active ? (base + lane) / parts : 0u, part = active ? base + lane - node * parts : 0u;
        uint32_t row, w[NW], ty[S], cut[S + 1];
        search_load<S>(q, node, active, row, w);
        const SearchNode n = search_node<S, AR>(p, tab, row, w, x, ty, cut);
        auto add_run = [&](bool want, uint32_t c, uint32_t hi0, uint32_t cnt) __attribute__((always_inline)) {
            const unsigned long long m = __ballot(want);
            if (m == 0) return;
            if (want) run[nrun + (uint32_t)__popcll(m & lanes_below)] = lane | c << 6 | hi0 << 14 | cnt << 22;
            nrun += (uint32_t)__popcll(m);
        };
        // the kept children of a node at the level that fixes the last cut, as runs
        auto last_children = [&](bool on, const SearchNode &m, uint32_t lx, uint32_t acc, uint32_t c) __attribute__((always_inline)) {
            uint32_t h0 = 1, h1 = 0;
            if (on) search_last_limits(p, m, acc, lp, h0, h1);
            bool range = !AR;
            if (!AR && !MONO) range = (p.g_mono >> (8 * m.t + m.tS)) & 1ull;
            uint32_t g0 = 0, cnt = 0;
            if (on && range) cnt = search_last_range(p, sx, m, lx, h0, h1, q.flags, bound, lp, g0);
            add_run(cnt != 0, c, g0, cnt);
            if constexpr (AR || !MONO) {
                // one by one; consecutive end points that pass make a run
                const SearchLast one = search_last_one<AR>(p, sx, m, lx);
                cnt = 0;
                for (uint32_t hi = h0; __ballot(on && !range && hi <= h1); ++hi) {
                    const bool t = on && !range && hi <= h1 && search_last_test<AR>(p, tab, sx, m, one, lx, hi, q.flags, bound, lp);
                    const bool flush = cnt != 0 && !t;
                    if (nrun > kRunCap - 64) hand_out(node, row, w);
                    add_run(flush, c, g0, cnt);
                    g0 = cnt == 0 ? hi : g0;
                    cnt = t ? cnt + 1 : 0u;
                }
                if (nrun > kRunCap - 64) hand_out(node, row, w);
                add_run(cnt != 0, c, g0, cnt);
            }
        };
        const uint32_t hmax = p.L - (S - 1 - x);   // every later stage keeps one layer
        const uint32_t acc = active ? search_accepted<AR>(p, tab, sx, n, x, hmax, q.flags, bound) : 0u;
        // the rule that stopped the range (0: it ran to its structural end), counted by the node's first item
        const bool first = active && part == 0;
        const int why = first ? search_stop<AR>(p, tab, sx, n, x, acc, hmax, q.flags, bound) : 0;
        visited += first ? acc : 0u;
        why_mem += why == 1;
        why_ridge += why == 2;
        why_bound += why == 3;
        // (the runs are handed out when the next choice's might not fit, and
        // at the end, before the lanes move on to other nodes)
        for (uint32_t k = 1 + part;; k += parts) {
            const bool more = S >= 3 ? __ballot(k <= acc) != 0 : k == 1;   // (S = 2: one part)
            if (more) {
                if constexpr (S >= 3) {
                    const bool on = k <= acc;
                    const uint32_t c = n.lo + (on ? k : 0u);
                    SearchNode m = n;
                    uint32_t acc2 = 0;
                    if (on) {
                        m = search_child<AR>(p, tab, n, x, c);
                        acc2 = search_accepted<AR>(p, tab, sx, m, x + 1, p.L - 1, q.flags, bound);
                        const int why2 = search_stop<AR>(p, tab, sx, m, x + 1, acc2, p.L - 1, q.flags, bound);
                        visited += acc2;
                        why_mem += why2 == 1;
                        why_ridge += why2 == 2;
                        why_bound += why2 == 3;
                    }
                    last_children(on, m, x + 1, acc2, c);
                } else {
                    last_children(active, n, x, acc, 0u);
                }
            }
            if (!more || nrun > kRunCap - 64) hand_out(node, row, w);
            if (!more) break;
        }
    }
    // what the lists still hold, against the best of the block and the piece
    __syncthreads();
    if (threadIdx.x == 0) atomicMin(&sh.known, __hip_atomic_load(q.acc, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT));
    __syncthreads();
    if constexpr (CLOSED) run_pend(0u, npend);
    // a makespan from the recurrence can lie above the bound
    if ((uint32_t)(best >> 32) > bound) best = ~0ull;
    // a configuration that passes the last stage counts as visited twice (its
    // stages S-1 and S) and evaluated
    search_block_counts(q, visited + lp.pass, lp.pass, why_mem + lp.mem, why_ridge + lp.ridge, why_bound + lp.bound);
    block_best<S>(q, best, bsub, brow, bw, sh.best);
}

// Problems without a closed form: the list's configurations by the
// recurrence, 64 to a wave, over the whole grid.
template <int S, bool AR, bool SCH>
__global__ __launch_bounds__(kBlock) void search_list_kernel(KParams p, SearchParams q) {
    extern __shared__ __align__(16) unsigned char smem[];
    __shared__ BlockBest<S> bb;
    constexpr int NW = Codes<S>::kWords;
    const uint32_t lane = threadIdx.x & 63, bound = *q.bound;
    static_assert(kListParts == 64, "a lane per part");
    uint32_t incl = min(q.list_n[lane], kListCap);
    const uint32_t mine = incl;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        const uint32_t u = __shfl_up(incl, o, 64);
        if (lane >= (uint32_t)o) incl += u;
    }
    const uint32_t n = __shfl(incl, 63, 64);
    if (blockIdx.x * kBlock >= n) return;   // (block-uniform; the slot keeps the last pass's best)
    const Ent tab = entry_tables(p, smem);
    const Comm<S> comm = load_comm<S>(p);
    unsigned long long best = ~0ull;
    uint32_t bsub = 0, brow = 0, bw[NW];
#pragma unroll
    for (int k = 0; k < NW; ++k) bw[k] = 0;
    for (uint32_t k0 = blockIdx.x * kBlock + (threadIdx.x - lane); k0 < n; k0 += gridDim.x * kBlock) {   // (wave-uniform)
        const uint32_t o = k0 + lane;
        uint32_t pl = 0;   // the part that holds entry o
#pragma unroll
        for (uint32_t b = 32; b; b >>= 1) pl = __shfl(incl, (int)(pl + b - 1), 64) <= o ? pl + b : pl;
        pl = o < n ? pl : 0u;
        const uint32_t first = __shfl(incl - mine, (int)pl, 64);
        if (o >= n) continue;
        const uint32_t *l = q.list + pl * kListCap + (o - first);
        const uint32_t at = l[0], row = l[kListParts * kListCap];
        uint32_t w[NW], cut[S + 1], to[S], F[S], B[S];
#pragma unroll
        for (int k = 0; k < NW; ++k) w[k] = l[(2 + k) * kListParts * kListCap];
        unpack_cuts<S>(w, p.L, cut);
        decode_toff<S>(p, tab, row, to);
        stage_weights<S>(p, tab, cut, to, F, B);
        const uint32_t T = dp_full_settle<S, SCH, AR>(p, tab, F, B, comm, w, row);
        if (T > bound) continue;
        const unsigned long long key = make_key(true, T, at);
        const uint32_t sub = last_cut<S>(w);
        if (key < best || (key == best && sub < bsub)) {
            best = key;
            bsub = sub;
            brow = row;
#pragma unroll
            for (int k = 0; k < NW; ++k) bw[k] = w[k];
        }
    }
    // the slot holds the last pass's best of that block: the better one stays
    if (threadIdx.x == 0) {
        const unsigned long long key = q.slot_key[blockIdx.x];
        uint32_t w[NW];
#pragma unroll
        for (int k = 0; k < NW; ++k) w[k] = q.slot_w[k * kSlotMax + blockIdx.x];
        if (key < best || (key == best && key != ~0ull && last_cut<S>(w) < bsub)) {
            best = key;
            bsub = last_cut<S>(w);
            brow = q.slot_row[blockIdx.x];
#pragma unroll
            for (int k = 0; k < NW; ++k) bw[k] = w[k];
        }
    }
    block_best<S>(q, best, bsub, brow, bw, bb);
}

// A lone stage (S = 1): one configuration per row, tested here like any
// stage, then evaluated; block b's best goes to slot b.
template <bool AR, bool SCH>
__global__ __launch_bounds__(kBlock) void search_leaf_kernel(KParams p, SearchParams q) {
    extern __shared__ __align__(16) unsigned char smem[];
    const uint32_t n_in = search_n_in(q), bound = *q.bound;
    const Lds tab = stage_tables(p, smem);
    const uint32_t i = blockIdx.x * kBlock + threadIdx.x;
    uint32_t row, w[1], ty[1], cut[2];
    search_load<1>(q, i, i < n_in, row, w);
    int why = 4;
    unsigned long long key = ~0ull;
    if (i < n_in) {
        const SearchNode n = search_node<1, AR>(p, tab, row, w, 0, ty, cut);
        why = search_try<AR>(p, tab, n, 0, p.L, q.flags, bound);
        if (why == 0) {
            uint32_t F[1], B[1];
            stage_weights<1>(p, tab, cut, ty, F, B);
            const uint32_t T = dp_full_settle<1, SCH, AR>(p, tab, F, B, load_comm<1>(p), w, row);
            if (T <= bound) key = ((unsigned long long)T << 32) | i;
        }
    }
    search_flush(q, why == 0, why == 0, why == 1, why == 2, why == 3);
    block_min_and_finish(key, q.acc, nullptr, nullptr, nullptr, false);
}

// After a piece: its best configuration replaces the best so far only if
// strictly better (earlier pieces and chunks come first in search order).
// best[0..2] = makespan, row, composition rank.  The configuration is in the
// slot whose key is the piece's best (S = 1: there is no cut, and the row is
// the one at that position).
template <typename R>
__global__ __launch_bounds__(kBlock) void search_merge_kernel(KParams p, SearchParams q, uint32_t nslot) {
    const unsigned long long key = *q.acc, had = q.best[0];
    __shared__ uint32_t slot;
    if (threadIdx.x == 0) slot = 0xFFFFFFFFu;
    __syncthreads();
    if (threadIdx.x == 0) *q.acc = ~0ull;
    if (q.list_n && threadIdx.x < kListParts) q.list_n[threadIdx.x] = 0u;
    if (key == ~0ull || (key >> 32) >= had) return;   // (the same for every thread)
    const uint32_t S = p.S, L = p.L;
    uint64_t rank = 0;
    uint32_t row = 0;
    if (S == 1) {
        if (threadIdx.x != 0) return;
        row = q.in_row[(uint32_t)key];
    } else {
        // the slot with that key (of equal ones the smallest last cut)
        auto last = [&](uint32_t b) { return (q.slot_w[((S - 2) >> 2) * kSlotMax + b] >> (8 * ((S - 2) & 3))) & 0xFFu; };
        static_assert(kSlotMax <= 1u << 16, "a slot in 16 bits");
        for (uint32_t b = threadIdx.x; b < nslot; b += kBlock)
            if (q.slot_key[b] == key) atomicMin(&slot, last(b) << 16 | b);
        __syncthreads();
        if (threadIdx.x != 0) return;
        const uint32_t b = slot & 0xFFFFu;
        row = q.slot_row[b];
        const R *binom = reinterpret_cast<const R *>(p.binom);
        // rank = sum_j C(L - 1 - c_{j-1}, S - j) - C(L - c_j, S - j)   (hockey-stick identity)
        uint32_t prev = 0;
        for (uint32_t j = 1; j < S; ++j) {
            const uint32_t c = (q.slot_w[((j - 1) >> 2) * kSlotMax + b] >> (8 * ((j - 1) & 3))) & 0xFFu;
            const uint32_t k = S - j;
            rank += (uint64_t)binom[k * kNB + (L - 1 - prev)] - (uint64_t)binom[k * kNB + (L - c)];
            prev = c;
        }
    }
    q.best[0] = key >> 32;
    q.best[1] = row;
    q.best[2] = rank;
}

// Roots of a piece of rows: level-0 nodes with no cut.
template <int S>
__global__ __launch_bounds__(kBlock) void search_root_kernel(SearchParams q, uint32_t first_row, uint32_t n) {
    const uint32_t i = blockIdx.x * kBlock + threadIdx.x;
    if (i >= n) return;
    q.out_row[i] = first_row + i;
#pragma unroll
    for (int k = 0; k < Codes<S>::kWords; ++k) q.out_codes[(uint64_t)k * q.out_cap + i] = 0u;
}

// ---------------------------------------------------------------------------
template <int S, typename R>
hipError_t launch_search_s(int op, const KParams &p, const SearchParams &q, uint32_t grid, size_t lds,
                           hipStream_t st) {
    const dim3 g(grid), b(kBlock);
    switch (op) {
    case kSearchOpCount:
        if (p.has_ar) hipLaunchKernelGGL((search_count_kernel<S, true>), g, b, lds, st, p, q);
        else hipLaunchKernelGGL((search_count_kernel<S, false>), g, b, lds, st, p, q);
        break;
    case kSearchOpWrite: hipLaunchKernelGGL((search_write_kernel<S>), g, b, 0, st, p, q); break;
    case kSearchOpLast:
        return with_variant(p, [&](auto arc, auto schc) {
            constexpr bool ar = decltype(arc)::value, sch = decltype(schc)::value;
            if constexpr (S == 1) {
                hipLaunchKernelGGL((search_leaf_kernel<ar, sch>), g, b, lds, st, p, q);
            } else {
                if (!p.closed) hipLaunchKernelGGL((search_last_kernel<S, ar, false, sch, false>), g, b, lds, st, p, q);
                else if (!ar && p.g_mono_all) hipLaunchKernelGGL((search_last_kernel<S, ar, !ar, sch, true>), g, b, lds, st, p, q);
                else hipLaunchKernelGGL((search_last_kernel<S, ar, false, sch, true>), g, b, lds, st, p, q);
            }
            return hipGetLastError();
        });
    case kSearchOpList:
        return with_variant(p, [&](auto arc, auto schc) {
            if constexpr (S > 1)
                hipLaunchKernelGGL((search_list_kernel<S, decltype(arc)::value, decltype(schc)::value>), g, b, lds, st, p, q);
            return hipGetLastError();
        });
    case kSearchOpMerge: hipLaunchKernelGGL((search_merge_kernel<R>), dim3(1), dim3(kBlock), 0, st, p, q, q.n_in); break;
    case kSearchOpRoot: hipLaunchKernelGGL((search_root_kernel<S>), g, b, 0, st, q, q.root_first, q.n_in); break;
    default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

}  // namespace pk

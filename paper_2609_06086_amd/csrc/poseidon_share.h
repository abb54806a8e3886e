#pragma once
// How many of a problem's candidates have no closed-form proof, estimated on
// the host when the costs are loaded: the proof of poseidon_closed.h on a
// fixed set of candidates (random compositions and assignments, the same ones
// for every load).  Only the choice between passes of equal results depends
// on it.
#include <stdint.h>

#include "poseidon_closed.h"

namespace pk {

constexpr uint32_t kShareSamples = 64;

// the loaded tables on the host: [T][L+1] prefix times, assignment rows
// [A][S] (null: every base-T row)
struct ShareTables {
    const uint64_t *cost;   // (prefix bwd << 32) | prefix fwd
    const uint32_t *pd;     // prefix all-reduce times, or null
    const uint8_t *assign;
};

// Candidates without a proof among kShareSamples (p.ctab in host memory).
template <int S, bool EAGER, bool AR>
inline uint32_t share_of(const KParams &p, const ShareTables &t) {
    uint64_t state = 0x9E3779B97F4A7C15ull;
    auto below = [&](uint32_t n) {   // (splitmix64, multiply-shift)
        uint64_t z = (state += 0x9E3779B97F4A7C15ull);
        z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ull;
        z = (z ^ (z >> 27)) * 0x94D049BB133111EBull;
        return (uint32_t)((((z ^ (z >> 31)) & 0xFFFFFFFFull) * n) >> 32);
    };
    uint32_t open = 0;
    for (uint32_t i = 0; i < kShareSamples; ++i) {
        // S-1 of the L-1 cut points, all subsets equally likely
        uint32_t cut[S + 1], k = 0;
        cut[0] = 0;
        for (uint32_t c = 1; c < p.L && k < S - 1u; ++c)
            if (below(p.L - c) < S - 1u - k) cut[++k] = c;
        cut[S] = p.L;
        const uint64_t row = t.assign ? below((uint32_t)(p.A < 0xFFFFFFFFull ? p.A : 0xFFFFFFFFull)) : 0u;
        uint32_t F[S], B[S], D[S], T;
        for (int s = 0; s < S; ++s) {
            const uint32_t ty = t.assign ? t.assign[row * S + s] : below(p.T);
            const uint64_t lo = t.cost[(size_t)ty * (p.L + 1) + cut[s]], hi = t.cost[(size_t)ty * (p.L + 1) + cut[s + 1]];
            F[s] = (uint32_t)hi - (uint32_t)lo;
            B[s] = (uint32_t)(hi >> 32) - (uint32_t)(lo >> 32);
            D[s] = AR ? t.pd[(size_t)ty * (p.L + 1) + cut[s + 1]] - t.pd[(size_t)ty * (p.L + 1) + cut[s]] : 0u;
        }
        open += !closed_form<S, EAGER, AR, false, ClosedConstHost>(p, F, B, D, T);
    }
    return open;
}

template <int S>
inline uint32_t share_dispatch(const KParams &p, const ShareTables &t) {
    if (p.S != (uint32_t)S) {
        if constexpr (S < kSMax) return share_dispatch<S + 1>(p, t);
        return 0;
    }
    if (p.sched) return t.pd ? share_of<S, true, true>(p, t) : share_of<S, true, false>(p, t);
    return t.pd ? share_of<S, false, true>(p, t) : share_of<S, false, false>(p, t);
}

// Share of the candidates of a problem with p.closed that have no proof
// (0 .. 1).
inline double unproven_share(const KParams &p, const ShareTables &t) {
    return share_dispatch<1>(p, t) / (double)kShareSamples;
}

}  // namespace pk

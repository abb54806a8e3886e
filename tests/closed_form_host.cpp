// Host build of the closed form and of the estimate of how many candidates
// have a proof, for tests/test_closed_form_cpu.py (compiled by the test, host
// code only).
#include <stdint.h>

#include <vector>

#include "../paper_2609_06086_amd/csrc/poseidon_share.h"

namespace {

template <int S, bool EAGER, bool AR>
void eval(const pk::KParams &p, uint32_t n, const uint32_t *F, const uint32_t *B, const uint32_t *D, uint32_t *T,
          uint8_t *proven) {
    for (uint32_t i = 0; i < n; ++i) {
        uint32_t f[S], b[S], d[S];
        for (int s = 0; s < S; ++s) {
            f[s] = F[(size_t)i * S + s];
            b[s] = B[(size_t)i * S + s];
            d[s] = AR ? D[(size_t)i * S + s] : 0u;
        }
        proven[i] = pk::closed_form<S, EAGER, AR, false, pk::ClosedConstHost>(p, f, b, d, T[i]);
    }
}

template <int S>
void dispatch(const pk::KParams &p, uint32_t n, const uint32_t *F, const uint32_t *B, const uint32_t *D, uint32_t *T,
              uint8_t *proven) {
    if (p.S != (uint32_t)S) {
        if constexpr (S < pk::kSMax) dispatch<S + 1>(p, n, F, B, D, T, proven);
        return;
    }
    if (p.sched) D ? eval<S, true, true>(p, n, F, B, D, T, proven) : eval<S, true, false>(p, n, F, B, D, T, proven);
    else D ? eval<S, false, true>(p, n, F, B, D, T, proven) : eval<S, false, false>(p, n, F, B, D, T, proven);
}

pk::KParams params(uint32_t L, uint32_t S, uint32_t M, uint32_t T, uint32_t sched, const uint32_t *cf,
                   const uint32_t *cb, uint32_t (&ctab)[pk::kCRows * pk::kSMax]) {
    pk::KParams p{};
    p.L = L; p.S = S; p.M = M; p.T = T; p.sched = sched; p.closed = 1;
    for (uint32_t s = 0; s + 1 < S; ++s) { p.cf[s] = cf[s]; p.cb[s] = cb[s]; }
    pk::closed_constants(p, ctab);
    p.ctab = ctab;
    return p;
}

}  // namespace

extern "C" {

// n candidates of S stages with weights F, B (and all-reduce weights D, or
// null) [n][S]: the closed form's value and whether it is proven.
void cf_eval(uint32_t S, uint32_t M, uint32_t sched, uint32_t n, const uint32_t *F, const uint32_t *B,
             const uint32_t *D, const uint32_t *cf, const uint32_t *cb, uint32_t *T, uint8_t *proven) {
    uint32_t ctab[pk::kCRows * pk::kSMax];
    const pk::KParams p = params(S, S, M, 1, sched, cf, cb, ctab);
    dispatch<1>(p, n, F, B, D, T, proven);
}

// the estimated share of a problem's candidates without a proof
double cf_share(uint32_t L, uint32_t S, uint32_t M, uint32_t T, uint32_t sched, const uint32_t *fwd,
                const uint32_t *bwd, const uint32_t *allreduce, const uint32_t *cf, const uint32_t *cb,
                const uint8_t *assign, uint64_t A) {
    uint32_t ctab[pk::kCRows * pk::kSMax];
    pk::KParams p = params(L, S, M, T, sched, cf, cb, ctab);
    p.A = A;
    std::vector<uint64_t> cost((size_t)T * (L + 1));
    std::vector<uint32_t> pd(allreduce ? cost.size() : 0);
    for (uint32_t t = 0; t < T; ++t) {
        uint32_t f = 0, b = 0, d = 0;
        for (uint32_t l = 0; l <= L; ++l) {
            cost[(size_t)t * (L + 1) + l] = (uint64_t)b << 32 | f;
            if (allreduce) pd[(size_t)t * (L + 1) + l] = d;
            if (l == L) break;
            f += fwd[(size_t)t * L + l];
            b += bwd[(size_t)t * L + l];
            if (allreduce) d += allreduce[(size_t)t * L + l];
        }
    }
    return pk::unproven_share(p, pk::ShareTables{cost.data(), allreduce ? pd.data() : nullptr, assign});
}

}  // extern "C"

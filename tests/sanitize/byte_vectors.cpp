// Host check of the edge kernels' entry code (csrc/taps_entry.h, compiled for
// the host) against the step-by-step form in steps.h: unification,
// Algorithm 1, "rearrange" and "remove" of random strategy pairs of random
// operators (1-8 axes, tensors of rank 0-8) on 1-256 devices, for 1-4 link
// classes at random boundaries, every field of every candidate, also where the
// degrees multiply to less than the devices (the tensors are replicated along
// the levels left); of every candidate rank of every set of partitionable axes
// the level runs, cuts and packed descriptor against their definition; and
// strategies stored at any address.  Prints "N compared, 0 mismatches".
#include <cstdio>
#include <cstdint>
#include <cstring>

#include "steps.h"
#include "taps_entry.h"

namespace {

uint64_t rng_state = 88172645463325252ull;
uint32_t rnd() {
    rng_state ^= rng_state << 13;
    rng_state ^= rng_state >> 7;
    rng_state ^= rng_state << 17;
    return (uint32_t)(rng_state >> 16);
}

const taps_completion_table kW = taps_make_completions();
const taps_top_table kT = taps_make_tops();
uint64_t compared = 0, bad = 0;

uint32_t candidates(uint32_t part, uint32_t n) { return kW.v[(taps_popc(part) * 9u + n) * 9u]; }

taps_desc describe(const taps_nibbles &S) {
    uint32_t expo[8];
    int32_t pos[8];
    for (uint32_t a = 0; a < 8u; ++a) {
        expo[a] = taps_nib(S.expo, a);
        pos[a] = expo[a] ? (int32_t)taps_nib(S.pos, a) : -1;
    }
    return taps_describe(8u, expo, pos);
}

void check(bool ok, const char *what, uint32_t n, uint32_t x) {
    ++compared;
    if (!ok && bad++ < 8) printf("%s: n %u, %u\n", what, n, x);
}

// Ranks are strategies in canonical order, each once; their layout.
void layouts() {
    for (uint32_t n = 0; n <= 8u; ++n)
        for (uint32_t part = 0; part < 256u; part += n > 5u ? 5u : 1u) {
            const uint32_t total = candidates(part, n), step = total > 400u ? total / 400u : 1u;
            for (uint32_t r = 0; r < total; r += step) {
                const taps_nibbles S = taps_unrank(part, n, r, kW.v);
                const taps_runs R = taps_lay_out(S, part, n);
                const taps_desc D = describe(S);
                uint32_t sum = 0, positions = 0, split = 0;
                bool ok = R.cuts == D.cuts && R.width == D.width;
                for (uint32_t a = 0; a < 8u; ++a) {
                    const uint32_t w = taps_nib(S.expo, a);
                    sum += w;
                    ok = ok && (w == 0u || ((part >> a) & 1u));
                    if (w) positions |= 1u << taps_nib(S.pos, a), ++split;
                    ok = ok && ((taps_u64(R.packed.runs) >> (8u * a + 4u)) & 15u) == w;
                    ok = ok && taps_axis_levels(R.packed, a) ==
                                   taps_levels(taps_nib(D.lo, a), taps_nib(D.width, a));
                }
                ok = ok && sum == n && positions == taps_low_mask(split);
                for (uint32_t l = 0; l < n; ++l) {
                    const uint32_t s = taps_nibble_shift(l), a = taps_nib(D.owner, l);
                    const uint32_t lo = taps_nib(D.lo, a), end = lo + taps_nib(D.width, a);
                    ok = ok && ((R.packed.owner >> s) & 15u) == a;
                    ok = ok && ((R.packed.place >> s) & 15u) == (end - 1u - l) + (l == lo ? 8u : 0u);
                }
                if (r + step < total && step == 1u) {   // ascending degrees, descending positions
                    const taps_nibbles N = taps_unrank(part, n, r + 1u, kW.v);
                    int order = 0;
                    for (uint32_t a = 0; a < 8u && !order; ++a)
                        order = (int)taps_nib(N.expo, a) - (int)taps_nib(S.expo, a);
                    for (uint32_t a = 0; a < 8u && !order; ++a)
                        if (taps_nib(S.expo, a)) order = (int)taps_nib(S.pos, a) - (int)taps_nib(N.pos, a);
                    ok = ok && order > 0;
                }
                check(ok, "layout", n, r);
            }
        }
}

// A strategy at every address, also one that no wider type starts at.
void stores() {
    alignas(16) uint8_t b[48];
    for (uint32_t at = 0; at < 17u; ++at) {
        std::memset(b, 0xEE, sizeof b);
        taps_store_strategy(b + at, {0x03020100u, 0x07060504u}, {0x0B0A0908u, 0x0F0E0D0Cu});
        bool ok = true;
        for (uint32_t k = 0; k < 48u; ++k) ok = ok && b[k] == (k - at < 16u ? k - at : 0xEEu);
        check(ok, "strategy store", at, 0);
    }
}

uint32_t pick_axes(uint32_t of, uint32_t rank) {
    uint32_t ax[8], r = 0;
    for (uint32_t i = 0; i < of; ++i) ax[i] = i;
    for (uint32_t i = 0; i < rank; ++i) {
        const uint32_t j = i + rnd() % (of - i), t = ax[i];
        ax[i] = ax[j];
        ax[j] = t;
        r |= ax[i] << (4u * i);
    }
    return r;
}

// A random strategy over the axes of `mask` on 2^n devices, or (partial) one whose
// degrees may multiply to less.
taps_nibbles draw_strategy(uint32_t mask, uint32_t n, bool partial) {
    uint32_t k = n;
    if (partial)
        do k = rnd() % (n + 1u);
        while (!candidates(mask, k));
    return taps_unrank(mask, k, rnd() % candidates(mask, k), kW.v);
}

// Whether the levels that S's runs cover end at a boundary of the unified axes.
// (Elsewhere an axis lies partly in a run and partly above it, and the step-by-step
// form slices into levels that are no axis's top.)
bool ends_at_a_boundary(const taps_nibbles &S, uint32_t tops) {
    uint32_t covered = 0;
    for (uint32_t a = 0; a < 8u; ++a) covered += taps_nib(S.expo, a);
    return covered == 0u || ((tops >> (covered - 1u)) & 1u);
}

template <uint32_t C>
void entries(uint64_t budget, bool partial) {
    const taps_width_table widths = taps_make_widths();
    const taps_a2a_table a2a = taps_make_a2a();
    const taps_expand_table ex = taps_make_expand();
    static taps_pair expand[256], cls_rows[256 * TAPS_D_MAX_CLASSES];
    static taps_a2a_row rows[256];
    static taps_top_row tops[256];
    static taps_b8 low[256];
    static uint8_t rank_table[256];
    for (uint32_t x = 0; x < 256u; ++x) expand[x] = taps_pair{ex.lo[x], ex.hi[x]};
    const uint64_t until = compared + budget;
    for (uint32_t trial = 0; compared < until; ++trial) {
        const uint32_t n = trial % 9u;
        uint32_t b[TAPS_D_MAX_CLASSES] = {0, 0, 0, 0};   // boundaries, non-decreasing
        for (uint32_t c = 0; c + 1u < C; ++c) b[c] = rnd() % (n + 1u);
        for (uint32_t c = 1; c + 1u < C; ++c)
            if (b[c] < b[c - 1u]) b[c] = b[c - 1u];
        taps_hier_steps H;
        std::memset(&H, 0, sizeof(H));
        H.n_classes = C;
        H.a2a_own = 1;   // AllToAlls of class 0 apart
        for (uint32_t l = 0; l < 8u; ++l) {
            uint32_t cls = 0, beta = 0;
            for (uint32_t c = 0; c + 1u < C; ++c)
                if (b[c] <= l) {
                    ++cls;
                    beta = b[c];
                }
            H.cls_of_top |= cls << (4u * l);
            H.beta_of_top |= beta << (4u * l);
            H.levels_of_cls[cls] |= 1u << l;
            H.beta_of_cls[cls] = beta;
        }
        const taps_levels_model m = taps_make_levels(n, C, b);
        const uint32_t lam = C > 1 ? b[0] : n;
        const uint32_t in_lo = lam >= 4u ? ~0u : (1u << (8u * lam)) - 1u;
        const uint32_t in_hi = lam <= 4u ? 0u : lam >= 8u ? ~0u : (1u << (8u * (lam - 4u))) - 1u;
        for (uint32_t x = 0; x < 256u; ++x) {
            tops[x] = taps_make_top_row(kT, x, m, low[x]);
            rows[x] = taps_a2a_row{a2a.lo[x], a2a.hi[x], a2a.lo[x] & in_lo, a2a.hi[x] & in_hi};
            for (uint32_t c = 0; c < TAPS_D_MAX_CLASSES; ++c) {
                const uint32_t lv = c < C ? H.levels_of_cls[c] & 0xFFu : 0u;
                cls_rows[x * TAPS_D_MAX_CLASSES + c] =
                    taps_pair{a2a.lo[x] & (ex.lo[lv] * 0xFFu), a2a.hi[x] & (ex.hi[lv] * 0xFFu)};
            }
        }
        const uint32_t na = 1u + rnd() % 8u, nb = 1u + rnd() % 8u;
        const uint32_t pm = rnd() & taps_low_mask(na), qm = rnd() & taps_low_mask(nb);
        const uint32_t tp = candidates(pm, n), tq = candidates(qm, n);
        if (!partial && (!tp || !tq)) continue;
        const uint32_t rank = rnd() % ((na < nb ? na : nb) + 1u);
        const uint32_t pax = pick_axes(na, rank), qax = pick_axes(nb, rank);
        const taps_side from = taps_make_side(pax, rank), to = taps_make_side(qax, rank);
        for (uint32_t i = 0; i < 8u; ++i) {
            const taps_nibbles Sp = draw_strategy(pm, n, partial);
            taps_row P;
            taps_make_row(P, describe(Sp), pax, rank, n, lam);
            taps_fill_rank_table(P, rank_table, 0, 1);
            P.to_rank = rank_table;
            P.widths = widths.v;
            P.a2a = rows;
            P.expand = expand;
            P.a2a_cls = cls_rows;
            const taps_source S = taps_make_source<C>(taps_lay_out(Sp, pm, n).packed, from, to,
                                                         rank, m);
            for (uint32_t j = 0; j < 24u; ++j) {
                const taps_nibbles Sq = draw_strategy(qm, n, partial);
                taps_col Q;
                std::memset(&Q, 0, sizeof(Q));
                taps_make_col(Q, describe(Sq), qax, rank);
                taps_lv L;
                taps_unify(P, Q, L);
                if (!ends_at_a_boundary(Sp, L.tp) || !ends_at_a_boundary(Sq, L.tp)) continue;
                const taps_start st = taps_begin(P, L);
                taps_fach want[3];
                const taps_hier_model_t<C> M{&H, cls_rows, expand};
                want[0] = taps_alg1_t(P, L, M, st);
                want[1] = taps_rearrange_t(P, L, M, st);
                want[2] = taps_remove_h(P, L, M);
                taps_three<C> got;
                taps_three_candidates<C>(S, taps_lay_out(Sq, qm, n).packed,
                                         taps_in_tensor(to, rank), m, tops, low, got);
                bool ok = got.a2a_in == want[0].xa;
                for (uint32_t k = 0; k < 3u; ++k) {
                    const uint32_t link[3] = {want[k].x1, want[k].x2, want[k].x3};
                    ok = ok && got.c[k].vol == want[k].vol && got.c[k].ct == want[k].ct &&
                         got.c[k].in == want[k].x0 + want[k].xa;
                    for (uint32_t c = 1; c < C; ++c) ok = ok && got.c[k].link[c - 1u] == link[c - 1u];
                }
                const uint32_t coll = taps_collectives_h(L, H);
                ok = ok && got.coll == (((coll & 0xFFu) << 2) | ((coll >> 8) << 7));
                if (C == 2) {   // the two-class closed forms
                    const taps_fac two[3] = {taps_alg1(P, L, st),
                                             taps_rearrange(P, L, st),
                                             taps_remove(P, L)};
                    for (uint32_t k = 0; k < 3u; ++k)
                        ok = ok && two[k].vol == got.c[k].vol && two[k].intra == got.c[k].in &&
                             two[k].inter == got.c[k].link[0] && two[k].ct == got.c[k].ct;
                }
                check(ok, partial ? "entry of partial strategies" : "entry", n, C);
            }
        }
    }
}

}  // namespace

int main() {
    layouts();
    stores();
    for (const bool partial : {false, true}) {
        entries<1>(20000, partial);
        entries<2>(150000, partial);
        entries<3>(100000, partial);
        entries<4>(100000, partial);
    }
    printf("%llu compared, %llu mismatches\n", (unsigned long long)compared,
           (unsigned long long)bad);
    return bad != 0;
}

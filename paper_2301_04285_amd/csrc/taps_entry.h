// taps_entry.h -- the candidates of one edge entry on byte vectors.
//
// The edge tensor T leaves its source under strategy P and enters its target
// under strategy Q.  Both device matrices and the tensor's shape are unified
// (Table 1) by closing the strategies' cuts, boundaries between adjacent levels,
// under the maps between their sides: a cut inside one side's run of a dimension
// forces the cut at the same bit of that dimension on the other side.  An axis of
// the unified matrix is named by its top level.  Position t of dimension d, the
// part that starts at its bit t, is held on either side by the axis whose top is
// the dimension's run's end less 1 + t; so every relation between the two tensor
// maps that Algorithm 1 needs is a map between levels.  With e = n - (levels the
// map uses) a device's shard is tbytes * 2^e nb, and the volumes of Eq. 9, 10
// and 14 follow from the state each axis is moved at (in factor units: taps_fac).
//
// Laid out for one entry per lane with no loop over dimensions and no table per
// row, so that the lanes of a wavefront may hold different rows:
//
//   * A set of levels is a vector of 8 bytes (two registers), byte l = FF when
//     level l is in it.  A map between levels is a vector of 8 indices, and
//     v_perm_b32 applies it: two instructions carry a whole set or a whole
//     vector of widths through a map, whatever the tensor's rank.  An index of
//     0x0D or more gives FF ("no level"), and so maps compose.
//   * Everything that propagates along chains of positions -- the cuts of the
//     unification, the AllToAll closures -- is found by pointer doubling: three
//     steps cover the at most seven hops, with no loop that would run until the
//     wavefront's slowest lane is done.
//   * The state of a sequence is one byte G: the shard's exponent in the low
//     bits and the number of free levels inside a node in the upper 3.  A
//     gather of an axis adds the axis's byte of `D` (its width, and its levels
//     inside a node << 5), a slice subtracts it.  Where the order of the gathers
//     is known beforehand ("remove", "rearrange", either kind of gather of
//     Algorithm 1) the states before all of them come from one prefix sum over
//     bytes in producer order: a multiplication by 0x01010101 per half.
//   * Algorithm 1's loop over gathers is in closed form too: which axes it
//     gathers, which move after which of them, and which slices come a pass
//     late, follow from the producer's order along the chains.  As a loop it
//     took 74 instructions per round, 2.0 rounds for the slowest of 64 lanes;
//     without it the 96-layer GPT's tables take 1409 us instead of 1529.
//   * Each axis held off its target is moved exactly once by every candidate,
//     so a candidate is described by the state each axis was moved at.  Powers
//     of two of a byte are a table lookup by v_perm_b32, a gather's volume fits
//     a byte (its exponent and width add up to at most 8), and the sums over the
//     axes are byte dot products.  Whether a level lies inside a node is the
//     same for every lane, so either kind's levels are brought to the low bytes
//     of one register by a uniform selection.
#pragma once

#include "taps_device.h"

// ---------------------------------------------------------------------------
// Vectors of 8 bytes
// ---------------------------------------------------------------------------
struct taps_b8 {
    uint32_t lo, hi;   // bytes 0-3, 4-7
};

// v_perm_b32: byte k of the result is byte sel_k of (hi, lo) for sel_k < 8,
// 0 for 0x0C, FF for 0x0D and above (8-11, the signs of odd bytes, are used
// by taps_not_lowest alone).
__host__ __device__ inline uint32_t taps_perm(uint32_t hi, uint32_t lo, uint32_t sel) {
#if defined(__HIP_DEVICE_COMPILE__)
    return __builtin_amdgcn_perm(hi, lo, sel);
#else
    const uint64_t d = ((uint64_t)hi << 32) | lo;
    uint32_t r = 0;
    for (uint32_t k = 0; k < 4u; ++k) {
        const uint32_t s = (sel >> (8u * k)) & 0xFFu;
        uint32_t b = 0xFFu;
        if (s < 8u)
            b = (uint32_t)(d >> (8u * s)) & 0xFFu;
        else if (s < 12u)
            b = ((d >> (16u * (s - 8u) + 15u)) & 1u) ? 0xFFu : 0u;
        else if (s == 12u)
            b = 0u;
        r |= b << (8u * k);
    }
    return r;
#endif
}

__host__ __device__ inline taps_b8 taps_map(const taps_b8 &x, const taps_b8 &index) {
    return {taps_perm(x.hi, x.lo, index.lo), taps_perm(x.hi, x.lo, index.hi)};
}

// v_bitop3_b32 (the issue rate of a 32-bit add); truth table T, bit 4a + 2b + c.
template <uint32_t T>
__host__ __device__ inline uint32_t taps_bitop3(uint32_t a, uint32_t b, uint32_t c) {
#if defined(__HIP_DEVICE_COMPILE__)
    return __builtin_amdgcn_bitop3_b32(a, b, c, T);
#else
    uint32_t r = 0;
    for (uint32_t k = 0; k < 8u; ++k)
        if ((T >> k) & 1u) r |= ((k & 4u) ? a : ~a) & ((k & 2u) ? b : ~b) & ((k & 1u) ? c : ~c);
    return r;
#endif
}
template <uint32_t T>
__host__ __device__ inline taps_b8 taps_bitop3(const taps_b8 &a, const taps_b8 &b, const taps_b8 &c) {
    return {taps_bitop3<T>(a.lo, b.lo, c.lo), taps_bitop3<T>(a.hi, b.hi, c.hi)};
}
constexpr uint32_t TAPS_A = 0xF0, TAPS_B = 0xCC, TAPS_C = 0xAA;   // the operands' truth tables
constexpr uint32_t TAPS_AND3 = TAPS_A & TAPS_B & TAPS_C;
constexpr uint32_t TAPS_A_NOTB_C = TAPS_A & (0xFFu ^ TAPS_B) & TAPS_C;

__host__ __device__ inline taps_b8 operator&(const taps_b8 &a, const taps_b8 &b) {
    return {a.lo & b.lo, a.hi & b.hi};
}
__host__ __device__ inline taps_b8 operator|(const taps_b8 &a, const taps_b8 &b) {
    return {a.lo | b.lo, a.hi | b.hi};
}
__host__ __device__ inline taps_b8 operator~(const taps_b8 &a) { return {~a.lo, ~a.hi}; }
// Byte sums and differences; no byte may carry or borrow.
__host__ __device__ inline taps_b8 operator+(const taps_b8 &a, const taps_b8 &b) {
    return {a.lo + b.lo, a.hi + b.hi};
}
__host__ __device__ inline taps_b8 operator-(const taps_b8 &a, const taps_b8 &b) {
    return {a.lo - b.lo, a.hi - b.hi};
}
__host__ __device__ inline taps_b8 taps_all(uint32_t word) { return {word, word}; }
__host__ __device__ inline bool taps_any(const taps_b8 &a) { return (a.lo | a.hi) != 0u; }
__host__ __device__ inline uint64_t taps_u64(const taps_b8 &a) { return ((uint64_t)a.hi << 32) | a.lo; }
__host__ __device__ inline taps_b8 taps_from(uint64_t x) { return {(uint32_t)x, (uint32_t)(x >> 32)}; }

// a in the bits of m, b in the others.
__host__ __device__ inline taps_b8 taps_blend(const taps_b8 &m, const taps_b8 &a, const taps_b8 &b) {
    return taps_bitop3<(TAPS_A & TAPS_B) | ((0xFFu ^ TAPS_A) & TAPS_C)>(m, a, b);
}

// FF where bit 7 of the byte is set (an index that names no level), else 0.
__host__ __device__ inline taps_b8 taps_none(const taps_b8 &x) {
    return {taps_perm(0u, 0u, x.lo & 0x80808080u), taps_perm(0u, 0u, x.hi & 0x80808080u)};
}

// FF where the byte is above 0x0C, else 0; an index that names no level is.
__host__ __device__ inline taps_b8 taps_above(const taps_b8 &x) {
    return {taps_perm(0u, 0u, x.lo), taps_perm(0u, 0u, x.hi)};
}

// FF where bit 3 is clear, 0 where it is set (selector 8 reads a sign that is 0).
__host__ __device__ inline taps_b8 taps_not_lowest(const taps_b8 &x) {
    return {taps_perm(0u, 0xFFu, x.lo & 0x08080808u), taps_perm(0u, 0xFFu, x.hi & 0x08080808u)};
}

// c plus the sum of the bytes.
__host__ __device__ inline uint32_t taps_sum(const taps_b8 &x, uint32_t c) {
    return taps_dot4(x.hi, 0x01010101u, taps_dot4(x.lo, 0x01010101u, c));
}

// 2^x for bytes x < 8.
__host__ __device__ inline uint32_t taps_pow2(uint32_t x) {
    return taps_perm(0x80402010u, 0x08040201u, x);
}

// Selector of levels l .. l + 3, 0 from `end` on.
__host__ __device__ inline uint32_t taps_four(uint32_t l, uint32_t end) {
    const uint32_t idx = 0x03020100u + l * 0x01010101u;
    const uint32_t k = end - l;   // 0 where a launch has no such levels
    const uint32_t keep = k >= 4u ? ~0u : (1u << (8u * k)) - 1u;
    return (idx & keep) | (0x0C0C0C0Cu & ~keep);
}

// Whether any lane of the wavefront (on the host: this one) has c.
__host__ __device__ inline bool taps_wave_any(bool c) {
#if defined(__HIP_DEVICE_COMPILE__)
    return __any(c);
#else
    return c;
#endif
}

// The set as a bit mask.
__host__ __device__ inline uint32_t taps_bits(const taps_b8 &x) {
    return taps_dot4(x.hi & 0x01010101u, 0x80402010u, taps_dot4(x.lo & 0x01010101u, 0x08040201u, 0u));
}

// States before each of the steps whose changes are the bytes of e, from state
// g, in ascending bytes; `end` receives the state after the last.  The changes may be negative
// (e is then the plain 32-bit sum of its bytes' values): every state is a byte,
// so the sums below come out digit by digit.
__host__ __device__ inline taps_b8 taps_states(const taps_b8 &e, uint32_t g, uint32_t &end) {
    taps_b8 x;
    x.lo = ((e.lo << 8) + g) * 0x01010101u;
    const uint32_t mid = (x.lo + e.lo) >> 24;
    x.hi = ((e.hi << 8) + mid) * 0x01010101u;
    end = (x.hi + e.hi) >> 24;
    return x;
}

// ---------------------------------------------------------------------------
// Strategy descriptors
// ---------------------------------------------------------------------------

// A strategy on binary levels.  owner and place are 8 indexed nibbles in the
// order that two masks turn into a byte vector: index k < 4 in the low nibble
// of byte k, k >= 4 in the high nibble of byte k - 4.
struct taps_packed {
    uint32_t owner;   // per level: the op axis that owns it (0x0C: none, the degrees multiply to less
                      // than 2^n; 0 above the last level)
    uint32_t place;   // per level: its distance from the top of its axis's run, + 8 when it is the
                      // run's lowest level (7: no owner; 15 above the last level)
    taps_b8 runs;     // per op axis: top level + 1 of its run, and << 4 the run's width (0: not split)
};

__host__ __device__ inline taps_b8 taps_unnibble(uint32_t x) {
    return {x & 0x0F0F0F0Fu, (x >> 4) & 0x0F0F0F0Fu};
}
__host__ __device__ inline uint32_t taps_nibble_shift(uint32_t k) {
    return k < 4u ? 8u * k : 8u * k - 28u;
}
// nibbles 0-3 of x (< 2^16) to the low nibbles of four bytes
__host__ __device__ inline uint32_t taps_spread(uint32_t x) {
    x = (x | (x << 8)) & 0x00FF00FFu;
    return (x | (x << 4)) & 0x0F0F0F0Fu;
}
// nibbles 0-7 in ascending order (taps_nib) to the order above
__host__ __device__ inline uint32_t taps_deal(uint32_t x) {
    return taps_spread(x & 0xFFFFu) | (taps_spread(x >> 16) << 4);
}

// The level runs of a strategy: the axis at position 0 owns the lowest levels.
// Positions past 7 leave an axis whole; a malformed strategy gives meaningless
// numbers but never an out-of-range index.
struct taps_runs {
    taps_packed packed;
    uint32_t lo, width;   // nibble a: lowest level and width of axis a's run (width 0: not split)
    uint32_t cuts;        // bit c: levels c - 1 and c belong to different axes
};

// axes: the axes that may be split (others are whole).
__host__ __device__ inline taps_runs taps_lay_out(const taps_nibbles &S, uint32_t axes, uint32_t n) {
    taps_runs R = {{0u, 0u, 0u, 0u}, 0u, 0u, 0u};
    uint32_t by_pos = 0;   // nibble p: width of the axis at position p
#pragma unroll
    for (uint32_t a = 0; a < TAPS_D_MAX_AXES; ++a) {
        if (!((axes >> a) & 1u)) continue;
        const uint32_t p = taps_nib(S.pos, a), w = p < 8u ? taps_nib(S.expo, a) : 0u;
        R.width |= w << (4u * a);
        by_pos |= w << (4u * (p & 7u));
    }
    const uint32_t first = (by_pos << 4) * 0x11111111u;   // nibble p: levels below position p
    uint32_t owner = 0, place = 0, end = 0;
#pragma unroll
    for (uint32_t a = 0; a < TAPS_D_MAX_AXES; ++a) {
        if (!((axes >> a) & 1u)) continue;
        const uint32_t w = taps_nib(R.width, a);
        if (w == 0u) continue;
        const uint32_t lo = taps_nib(first, taps_nib(S.pos, a) & 7u);
        const uint32_t at = (4u * lo) & 31u, cut = (32u - 4u * w) & 31u;
        R.lo |= lo << (4u * a);
        end |= ((lo + w) & 15u) << (4u * a);
        owner |= ((a * 0x11111111u) >> cut) << at;
        // w - 1, ..., 1, 0 upwards, the lowest level flagged
        place |= ((0x01234567u >> cut) | 8u) << at;
        R.cuts |= 1u << lo;
    }
    R.cuts &= ~1u;
    const uint32_t above = n < 8u ? ~0u << (4u * n) : 0u;
    // levels past the last run, if the degrees multiply to less than 2^n: no axis
    // holds them (the tensors are replicated along them), and no cut lies below
    const uint32_t covered = (first >> 28) + (by_pos >> 28);
    const uint32_t idle = covered < n ? ~above & (~0u << (4u * covered)) : 0u;
    R.packed.owner = taps_deal((owner & ~above) | (0xCCCCCCCCu & idle));
    R.packed.place = taps_deal(place | above | (0x77777777u & idle));
    R.packed.runs = {taps_spread(end & 0xFFFFu) | (taps_spread(R.width & 0xFFFFu) << 4),
                     taps_spread(end >> 16) | (taps_spread(R.width >> 16) << 4)};
    return R;
}

// Levels of op axis a.
__host__ __device__ inline uint32_t taps_axis_levels(const taps_packed &p, uint32_t a) {
    const uint32_t run = (a < 4u ? p.runs.lo : p.runs.hi) >> (8u * (a & 3u));
    const uint32_t w = (run >> 4) & 15u, end = run & 15u;
    return taps_levels(end < w ? 0u : end - w, w);
}

// A strategy's 16 bytes, degrees then positions, to any address: the caller's
// array may start anywhere (still one 16-byte store, which global memory takes
// unaligned).
__host__ __device__ inline void taps_store_strategy(void *at, const taps_b8 &degrees,
                                                    const taps_b8 &positions) {
    const taps_b8 bytes[2] = {degrees, positions};
    __builtin_memcpy(at, bytes, sizeof bytes);
}

// One side of an edge: which tensor dimension an op axis carries (7: none; a
// tensor of rank 8 uses every axis) and which axis a dimension lies on (0x0C:
// none), as nibbles in the order of taps_packed.
struct taps_side {
    uint32_t dim_of, axis_of;
};

__host__ __device__ inline taps_side taps_make_side(uint32_t axes, uint32_t rank) {
    taps_side s = {0x77777777u, 0xCCCCCCCCu};
    for (uint32_t d = 0; d < rank && d < TAPS_D_MAX_RANK; ++d) {
        const uint32_t a = taps_nib(axes, d) & 7u;
        const uint32_t sa = taps_nibble_shift(a), sd = taps_nibble_shift(d);
        s.dim_of = (s.dim_of & ~(15u << sa)) | (d << sa);
        s.axis_of = (s.axis_of & ~(15u << sd)) | (a << sd);
    }
    return s;
}

// FF at the op axes that an edge's tensor has on this side.
__host__ __device__ inline taps_b8 taps_in_tensor(const taps_side &s, uint32_t rank) {
    // dimension 7 stands for "none" below rank 8
    const taps_b8 dim = taps_unnibble(s.dim_of);
    const uint32_t hi = rank < TAPS_D_MAX_RANK ? 0x00FFFFFFu : 0xFFFFFFFFu;
    return {taps_perm(hi, 0xFFFFFFFFu, dim.lo), taps_perm(hi, 0xFFFFFFFFu, dim.hi)};
}

// ---------------------------------------------------------------------------
// What a launch, an edge and a row fix
// ---------------------------------------------------------------------------

// Levels and link classes (uniform over a launch).  Class 0 lies inside a
// node; class c >= 1 holds the levels first[c] .. first[c + 1] - 1, whose
// groups share the links of blocks of 2^beta[c] ranks (beta[c] = first[c]; 0
// for a class without levels).  The paper's two classes are C = 2.
struct taps_levels_model {
    uint32_t n;       // levels
    uint32_t full;    // taps_low_mask(n)
    uint32_t first[TAPS_D_MAX_CLASSES + 1];
    uint32_t beta[TAPS_D_MAX_CLASSES];
    taps_b8 in01;     // 01 at the levels inside a node
    taps_b8 coll;     // an axis's collective at its places in meta: 4, and 128 more outside a node
    taps_b8 share[TAPS_D_MAX_CLASSES];   // byte u: 2^(beta - u), the groups that share a link of the
                                         // class when u of the levels below beta are free
};

// Bytes 01 at the levels lo .. hi - 1.
__host__ __device__ inline taps_b8 taps_range(uint32_t lo, uint32_t hi) {
    uint64_t m = 0;
#pragma unroll
    for (uint32_t l = 0; l < TAPS_D_MAX_LEVELS; ++l)
        if (l >= lo && l < hi) m |= 1ull << (8u * l);
    return taps_from(m);
}

// n_classes classes, class c >= 1 from level boundary[c - 1] up (non-decreasing).
__host__ __device__ inline taps_levels_model taps_make_levels(uint32_t n, uint32_t n_classes,
                                                              const uint32_t *boundary) {
    taps_levels_model m;
    m.n = n;
    m.full = taps_low_mask(n);
    m.first[0] = 0u;
    for (uint32_t c = 1; c <= TAPS_D_MAX_CLASSES; ++c)
        m.first[c] = c < n_classes && boundary[c - 1u] < n ? boundary[c - 1u] : n;
    for (uint32_t c = 0; c < TAPS_D_MAX_CLASSES; ++c) {
        m.beta[c] = c && m.first[c] < m.first[c + 1u] ? m.first[c] : 0u;
        uint64_t share = 0;
        for (uint32_t u = 0; u < 8u && u <= m.beta[c]; ++u)
            share |= (uint64_t)(1u << (m.beta[c] - u)) << (8u * u);
        m.share[c] = taps_from(share);
    }
    m.in01 = taps_range(0u, m.first[1]);
    m.coll = {0x84848484u - m.in01.lo * 0x80u, 0x84848484u - m.in01.hi * 0x80u};
    return m;
}
__host__ __device__ inline taps_levels_model taps_make_levels(uint32_t n, uint32_t lam) {
    return taps_make_levels(n, 2u, &lam);
}

// By tops mask, in LDS.  For every top t, with w the width of its axis and k_c
// the axis's levels below beta[c]: byte t of d is w + (k_1 << 5), of low (more
// than two classes) k_2 + (k_3 << 4), of tops FF, of a2a 256 - 2^(8 - w) (an
// AllToAll moves all but 2^-w of the shard, Eq. 10), of link 256 - 2^(8 - w + k)
// with k that of the axis's own class (of that, all but what stays inside the
// blocks, Eq. 14; 0 inside a node).  0 at the other levels.
struct alignas(16) taps_top_row {
    taps_b8 d, tops, a2a, link;
};

// Of the axes with widths w (bytes at the tops), the levels below beta: all of
// an axis that ends below it, and of those above only the lowest can reach there.
__host__ __device__ inline taps_b8 taps_levels_below(const taps_b8 &w, uint32_t tp, uint32_t beta) {
    const taps_b8 r = taps_range(0u, beta);
    uint64_t k = taps_u64(w & taps_b8{r.lo * 0xFFu, r.hi * 0xFFu});
    const uint32_t above = tp >> beta;
    if (above) {
        const uint32_t s = beta + taps_ctz(above);
        const uint32_t ws = (uint32_t)(taps_u64(w) >> (8u * s)) & 15u;
        if (ws > s + 1u - beta) k |= (uint64_t)(ws - (s + 1u - beta)) << (8u * s);
    }
    return taps_from(k);
}

// The axes' widths by tops mask.
struct taps_top_table {
    uint32_t w_lo[256], w_hi[256];
};

__host__ __device__ constexpr taps_top_table taps_make_tops() {
    taps_top_table t{};
    for (uint32_t m = 0; m < 256u; ++m) {
        uint64_t w = 0;
        uint32_t lo = 0;
        for (uint32_t l = 0; l < 8u; ++l)
            if ((m >> l) & 1u) {
                w |= (uint64_t)(l + 1u - lo) << (8u * l);
                lo = l + 1u;
            }
        t.w_lo[m] = (uint32_t)w;
        t.w_hi[m] = (uint32_t)(w >> 32);
    }
    return t;
}

__host__ __device__ inline taps_top_row taps_make_top_row(const taps_top_table &T, uint32_t tp,
                                                          const taps_levels_model &m, taps_b8 &low) {
    const taps_b8 w = {T.w_lo[tp], T.w_hi[tp]};
    // FF where a width (at most 8) is not 0
    const taps_b8 tops = taps_none(w + taps_all(0x7F7F7F7Fu));
    const taps_b8 one = tops & taps_all(0x01010101u);
    // 256 - 2^(8 - x) for x = 1 .. 8 by x - 1
    const taps_b8 parts = {0xF0E0C080u, 0xFFFEFCF8u};
    taps_top_row row = {w, tops, taps_map(parts, w - one) & tops, {0u, 0u}};
    low = {0u, 0u};
#pragma unroll
    for (uint32_t c = 1; c < TAPS_D_MAX_CLASSES; ++c) {
        if (m.first[c] >= m.first[c + 1u]) continue;   // uniform
        const taps_b8 k = m.beta[c] ? taps_levels_below(w, tp, m.beta[c]) : taps_b8{0u, 0u};
        const uint64_t k64 = taps_u64(k);
        if (c == 1u) row.d = row.d | taps_from(k64 << 5);
        if (c == 2u) low = low | k;
        if (c == 3u) low = low | taps_from(k64 << 4);
        const taps_b8 r = taps_range(m.first[c], m.first[c + 1u]);
        const taps_b8 mine = tops & taps_b8{r.lo * 0xFFu, r.hi * 0xFFu};
        row.link = row.link | (taps_map(parts, w - one - (k & mine)) & mine);
    }
    return row;
}

// The source side of a row: its levels' positions as the target side's axes
// meet them, and the target's axes that carry their dimensions.
struct taps_source {
    taps_b8 axis;     // per level: the target's axis of its tensor dimension (0x0C: none)
    taps_b8 from;     // per level: 7F - its position bit in the dimension (taps_packed::place
                      // without the flag), 77 without an owner
    taps_b8 below;    // per level: 7E - that bit, at most 76 for a run's lowest level (77: no owner)
    taps_b8 top;      // per target axis: 7F + end of the run on its dimension
    taps_b8 room;     // per target axis: 80 - width of that run
    taps_b8 held;     // FF at the levels the tensor's map uses
    taps_b8 uncut;    // FF where no cut lies below the level
    taps_b8 rank;     // per level: its place among the positions in order (dimension, then bit)
    taps_b8 order;    // per place in that order: the level (0x0C: none)
    uint32_t g;       // the state G before the first step: the shard's exponent, and << 5 the
                      // free levels below beta[1]
    uint32_t h;       // more than two classes: the free levels below beta[2], and << 4 below beta[3]
};

template <uint32_t C>
__host__ __device__ inline taps_source taps_make_source(const taps_packed &p, const taps_side &side,
                                                        const taps_side &to, uint32_t rank,
                                                        const taps_levels_model &m) {
    taps_source P;
    const taps_b8 owner = taps_unnibble(p.owner);
    const taps_b8 dim = taps_map(taps_unnibble(side.dim_of), owner);
    P.axis = taps_map(taps_unnibble(to.axis_of), dim);
    const taps_b8 flagged = taps_unnibble(p.place);
    const taps_b8 place = flagged & taps_all(0x07070707u);
    // 77 at a level without an owner: past every run of the target's side
    const taps_b8 idle = {(owner.lo >> 3) & 0x01010101u, (owner.hi >> 3) & 0x01010101u};
    P.from = taps_all(0x7F7F7F7Fu) - place - idle;
    P.below = taps_all(0x7E7E7E7Eu) - flagged;
    const taps_b8 runs = taps_map(p.runs, taps_unnibble(side.axis_of));
    const taps_b8 width = {(runs.lo >> 4) & 0x0F0F0F0Fu, (runs.hi >> 4) & 0x0F0F0F0Fu};
    const taps_b8 dim_of = taps_unnibble(to.dim_of);
    P.top = taps_map((runs & taps_all(0x0F0F0F0Fu)) + taps_all(0x7F7F7F7Fu), dim_of);
    P.room = taps_map(taps_all(0x80808080u) - width, dim_of);
    P.held = taps_map(taps_in_tensor(side, rank), owner);
    P.uncut = taps_not_lowest(flagged);
    uint32_t used;
    const taps_b8 first = taps_states(width, 0u, used);   // positions before each dimension
    P.rank = (taps_map(first, dim) + place) & taps_all(0x07070707u);
    uint64_t order = 0x0C0C0C0C0C0C0C0Cull;
#pragma unroll
    for (uint32_t l = 0; l < TAPS_D_MAX_LEVELS; ++l) {
        const uint32_t rank_l = ((l < 4u ? P.rank.lo : P.rank.hi) >> (8u * (l & 3u))) & 7u;
        const uint32_t held_l = ((l < 4u ? P.held.lo : P.held.hi) >> (8u * (l & 3u))) & 0xFFu;
        if (l < m.n) order ^= (uint64_t)((l ^ 0x0Cu) & held_l) << (8u * rank_l);
    }
    P.order = taps_from(order);
    uint32_t free_below[TAPS_D_MAX_CLASSES];
#pragma unroll
    for (uint32_t c = 1; c < TAPS_D_MAX_CLASSES; ++c)
        free_below[c] = c < C && m.beta[c]
                            ? m.beta[c] - taps_sum(P.held & taps_range(0u, m.beta[c]), 0u) : 0u;
    P.g = ((m.n - used) & 15u) | (free_below[1] << 5);
    P.h = free_below[2] | (free_below[3] << 4);
    return P;
}

// ---------------------------------------------------------------------------
// One entry
// ---------------------------------------------------------------------------

// One candidate in factor units (taps_fac), by link class: volume, what class
// 0 carries, what class c carries over its links times the sharing groups, and
// the sum of the group counts.
template <uint32_t C>
struct taps_cost_c {
    uint32_t vol, in, link[C > 1 ? C - 1 : 1], ct;
};

// Replace (Algorithm 1), rearrange (the same without AllToAll) and remove.
template <uint32_t C>
struct taps_three {
    taps_cost_c<C> c[3];
    uint32_t a2a_in;   // what AllToAlls carry of c[0].in
    uint32_t coll;     // collectives of every candidate and inter-node ones among them, at their
                       // places in the record's meta (bits 2 and 7 up)
};

// One pointer-doubling step of "not reached": x stays FF only where the level
// it points to is FF too.
__host__ __device__ inline taps_b8 taps_hop(const taps_b8 &x, const taps_b8 &to) {
    return x & taps_map(x, to);
}

// in_tensor: taps_in_tensor of the target side; tab, low: taps_make_top_row's
// by tops mask (low is read for more than two classes).
template <uint32_t C>
__host__ __device__ inline void taps_three_candidates(const taps_source &P, const taps_packed &q,
                                                      const taps_b8 &in_tensor,
                                                      const taps_levels_model &m,
                                                      const taps_top_row *tab, const taps_b8 *low,
                                                      taps_three<C> &out) {
    constexpr bool kLow = C > 2;   // the free levels below further boundaries are followed too
    const taps_b8 owner = taps_unnibble(q.owner), flagged = taps_unnibble(q.place);
    const taps_b8 place = flagged & taps_all(0x07070707u);
    // of the target's runs on the source levels' dimensions
    const taps_b8 runs = taps_map(q.runs, P.axis), end = runs & taps_all(0x0F0F0F0Fu);
    const taps_b8 width_p = {(runs.lo >> 4) & 0x0F0F0F0Fu, (runs.hi >> 4) & 0x0F0F0F0Fu};

    // prev[c]: the source level at the position that target level c goes to;
    // next[p]: the target level that goes to source level p's position.  The
    // byte differences keep bit 7 set; place + 80 - width has it set when the
    // position lies past the other side's run (7F - place + width, clear).  A
    // target level without an owner reads 0 for top and room: its difference
    // borrows, from levels above it alone, and is 78 or 79 below bit 7, no level.
    // below_*: the same for the cuts inside what both sides split (all levels
    // there but the lowest).
    constexpr uint32_t kPast = (TAPS_A & TAPS_B) | ((0xFFu ^ TAPS_A) & TAPS_C);
    constexpr uint32_t kNotPast = (TAPS_A & (0xFFu ^ TAPS_B)) | ((0xFFu ^ TAPS_A) & TAPS_C);
    const taps_b8 high = taps_all(0x80808080u);
    const taps_b8 past = taps_map(P.room, owner), from = taps_map(P.top, owner) - place;
    const taps_b8 prev = taps_bitop3<kPast>(high, place + past, from);
    taps_b8 below_c = taps_bitop3<kPast>(high, flagged + taps_all(0x01010101u) + past, from);
    const taps_b8 from_p = end + P.from;
    const taps_b8 next = taps_bitop3<kNotPast>(high, P.from + width_p, from_p);
    taps_b8 below_p = taps_bitop3<kNotPast>(high, P.below + width_p, from_p);

    // unification (Table 1): the cuts of both sides, closed under both maps
    taps_b8 uncut = taps_not_lowest(flagged) & P.uncut;
    uncut = taps_bitop3<TAPS_AND3>(uncut, taps_map(uncut, below_c), taps_map(uncut, below_p));
    below_c = taps_map(below_c, below_c);
    below_p = taps_map(below_p, below_p);
    uncut = taps_bitop3<TAPS_AND3>(uncut, taps_map(uncut, below_c), taps_map(uncut, below_p));
    below_c = taps_map(below_c, below_c);
    below_p = taps_map(below_p, below_p);
    uncut = taps_bitop3<TAPS_AND3>(uncut, taps_map(uncut, below_c), taps_map(uncut, below_p));
    // a level is a top if a cut lies below the next: of FF bytes at the levels with
    // none, the sum by the weights of the levels below them is, up to bit 7, -1 less
    const uint32_t tp = m.full & taps_dot4(uncut.hi, 0x40201008u,
                                           taps_dot4(uncut.lo, 0x04020100u, ~0u));
    const taps_top_row row = taps_entry<5>(tab, tp);
    const taps_b8 D = row.d;
    taps_b8 D2 = {0u, 0u};
    if (kLow) D2 = taps_entry<3>(low, tp);

    // away: not at the same position on both sides
    const taps_b8 away = {taps_perm(0xFFFFFFFFu, 0xFFFFFF00u, prev.lo ^ 0x03020100u),
                          taps_perm(0xFFFFFFFFu, 0xFFFFFF00u, prev.hi ^ 0x07060504u)};
    const taps_b8 dst = row.tops & taps_map(in_tensor, owner);
    const taps_b8 held = taps_bitop3<TAPS_AND3>(row.tops, P.held, away);
    const taps_b8 unwanted = taps_above(next);   // source positions no target axis goes to
    const taps_b8 ns = taps_map(next, P.order);
    // the common start of Algorithm 1 and "rearrange": the first InferSlice
    const taps_b8 open = taps_map(~held, prev);   // targets no held axis blocks
    const taps_b8 todo0 = dst & away;
    const taps_b8 sliced = taps_bitop3<TAPS_A_NOTB_C>(todo0, held, open);
    const taps_b8 todo = todo0 & ~sliced;
    const uint32_t G = P.g - taps_sum(D & sliced, 0u);
    const uint32_t H = kLow ? P.h - taps_sum(D2 & sliced, 0u) : 0u;

    // ---- Algorithm 1 ("replace" in Table 2): the state every axis is moved at, and
    // the axes that AllToAlls move.  The printed loop comes to this:
    //   * one pass of the inner loop is InferSlice, then InferAll2All until nothing
    //     moves; a slice frees no position, so a second pass can only slice (targets
    //     that the AllToAlls freed) and a third finds nothing;
    //   * an AllGather of an axis whose position no target axis goes to frees nothing
    //     that anyone waits for, and the axis cannot be sliced back (with a free
    //     target it would have moved): such gathers run back to back, in producer
    //     order, but the first alone before the slices still pending;
    //   * the axes left sit at targeted positions, and AllGatherFirstUndoneDim takes
    //     the first in producer order, a pass after each;
    //   * with nothing held at a source position only slices remain, which are free.
    taps_b8 at, at2 = {0u, 0u}, a2a;   // at2: the free levels of H
    {
        // the first closure: movable axes, then those whose targets they free
        const taps_b8 movers = todo & held;
        taps_b8 stay = ~(movers & open);
        const taps_b8 hop1 = taps_bitop3<(TAPS_A | (0xFFu ^ TAPS_B) | TAPS_C)>(prev, movers, open);
        stay = taps_hop(stay, hop1);
        const taps_b8 hop2 = taps_map(hop1, hop1);
        stay = taps_hop(stay, hop2);
        const taps_b8 hop4 = taps_map(hop2, hop2);
        stay = taps_hop(stay, hop4);
        a2a = ~stay;
        at = taps_all(G * 0x01010101u) & a2a;
        if (kLow) at2 = taps_all(H * 0x01010101u) & a2a;
        const taps_b8 left = held & stay, wait = todo & stay;
        if (taps_wave_any(taps_any(left))) {
            // the slices those moves make possible: at once if the first InferSlice
            // found something, else after the next gather, whose state is higher then
            const taps_b8 ug = left & unwanted;
            const taps_b8 freed = taps_bitop3<TAPS_A_NOTB_C>(wait, left, taps_map(~left, prev));
            const bool now = taps_any(sliced), gathers = taps_any(ug);
            uint32_t pending = taps_sum(D & freed, 0u), g = G - pending;
            pending = now ? 0u : pending;
            uint32_t pending2 = kLow ? taps_sum(D2 & freed, 0u) : 0u, h = H - pending2;
            pending2 = now ? 0u : pending2;
            // untargeted gathers in producer order
            if (taps_wave_any(gathers)) {
                const taps_b8 us = taps_map(ug, P.order);   // its lowest byte: the first
                const uint32_t f_lo = us.lo & (0u - us.lo), f_hi = us.lo ? 0u : us.hi & (0u - us.hi);
                taps_b8 s = taps_states(taps_map(D & ug, P.order), g, g);
                s = s + taps_b8{f_lo * pending, f_hi * pending};
                at = taps_blend(ug, taps_map(s, P.rank), at);
                pending = gathers ? 0u : pending;
                if (kLow) {
                    s = taps_states(taps_map(D2 & ug, P.order), h, h);
                    s = s + taps_b8{f_lo * pending2, f_hi * pending2};
                    at2 = taps_blend(ug, taps_map(s, P.rank), at2);
                    pending2 = gathers ? 0u : pending2;
                }
            }
            // What is left blocks itself: cycles, and chains down to an axis without a
            // target.  AllGatherFirstUndoneDim takes the first in the producer's order,
            // which frees all that wait for it along the chain; so an axis is gathered
            // if it comes before all that its own target waits for (of a cycle, the
            // first), and is moved else, after the next one along the chain that is.
            // The last that waits before a gathered axis is sliced in the same pass.
            const taps_b8 rest = left & ~ug;
            if (taps_wave_any(taps_any(rest))) {
                // ranks not met along the chain, and those below the axis's own
                taps_b8 unmet = {taps_perm(0x7FBFDFEFu, 0xF7FBFDFEu, P.rank.lo),
                                 taps_perm(0x7FBFDFEFu, 0xF7FBFDFEu, P.rank.hi)};
                const taps_b8 under = {taps_perm(0x7F3F1F0Fu, 0x07030100u, P.rank.lo),
                                       taps_perm(0x7F3F1F0Fu, 0x07030100u, P.rank.hi)};
                unmet = taps_hop(unmet, hop1);
                unmet = taps_hop(unmet, hop2);
                unmet = taps_hop(unmet, hop4);
                const taps_b8 moved = rest & taps_above((under & ~unmet) + taps_all(0x0C0C0C0Cu));
                const taps_b8 taken = rest & ~moved;
                const taps_b8 self = {0x03020100u, 0x07060504u};
                // the gathered axis along the chain, and the axis that waits up to it
                taps_b8 to = taps_blend(taken, self, prev), up = taps_blend(moved, next, self);
                to = taps_map(to, to);
                up = taps_map(up, up);
                to = taps_map(to, to);
                up = taps_map(up, up);
                to = taps_map(to, to);
                up = taps_map(taps_map(up, up), next);
                const taps_b8 xs = taps_map(taken, P.order), rank_to = taps_map(P.rank, to);
                const taps_b8 plus = taps_map(D, P.order) & xs;
                const taps_b8 minus = taps_map(taps_map(D & todo, up), P.order) & xs;
                taps_b8 s = taps_states(plus - minus, g, g), s2 = {0u, 0u};
                const taps_b8 after = s + plus;
                taps_b8 after2 = {0u, 0u}, minus2 = {0u, 0u};
                if (kLow) {
                    const taps_b8 plus2 = taps_map(D2, P.order) & xs;
                    minus2 = taps_map(taps_map(D2 & todo, up), P.order) & xs;
                    s2 = taps_states(plus2 - minus2, h, h);
                    after2 = s2 + plus2;
                }
                // A slice that only the AllToAlls of its pass make possible waits for the
                // next pass, after its gather, unless InferSlice found something before
                // them: an earlier such slice, or one into the gathered axis's position.
                // bit k of gathers_at: a gather at place k; bit k of late: a slice of the
                // gather at place k - 1 (0: pending) may wait so
                const taps_b8 via = taps_bitop3<TAPS_AND3>(taps_map(moved, ns), xs,
                                                           taps_all(0x01010101u));
                const uint32_t gathers_at = taps_bits(xs);
                uint32_t late = 2u * taps_dot4(via.hi, 0x80402010u, taps_dot4(via.lo, 0x08040201u, 0u)) +
                                ((pending | pending2) ? 1u : 0u);
                uint32_t higher = gathers_at & (late | (0u - late));   // from the first such on
                if (taps_wave_any(higher != 0u)) {
                    const uint64_t by = (taps_u64(minus) << 8) | (pending & 0xFFu);
                    const uint64_t by2 = kLow ? (taps_u64(minus2) << 8) | (pending2 & 0xFFu) : 0u;
                    for (uint32_t it = 0; it < TAPS_D_MAX_LEVELS && higher; ++it) {
                        const uint32_t from = 8u * taps_ctz(late), to_byte = 8u * taps_ctz(higher);
                        s = taps_from(taps_u64(s) + (((by >> from) & 0xFFu) << to_byte));
                        if (kLow) s2 = taps_from(taps_u64(s2) + (((by2 >> from) & 0xFFu) << to_byte));
                        // that gather's own slice does not wait
                        late &= (late - 1u) & ~(2u * (higher & (0u - higher)));
                        higher = gathers_at & (late | (0u - late));
                    }
                }
                a2a = a2a | moved;
                at = taps_blend(taken, taps_map(s, rank_to), at);
                at = taps_blend(moved, taps_map(after, rank_to), at);
                if (kLow) {
                    at2 = taps_blend(taken, taps_map(s2, rank_to), at2);
                    at2 = taps_blend(moved, taps_map(after2, rank_to), at2);
                }
            }
        }
    }

    // ---- "rearrange" (Algorithm 1 without AllToAll): untargeted axes in producer
    // order, then targeted ones; each is sliced back at once if its target is open,
    // and what waits for its position is sliced into that
    taps_b8 at_r, at_r2 = {0u, 0u};
    {
        // a targeted axis whose blocker comes before it
        const taps_b8 before = taps_above((P.rank + taps_all(0x0C0C0C0Cu)) -
                                          (taps_map(P.rank, prev) & taps_all(0x07070707u)));
        const taps_b8 ready = open | taps_bitop3<TAPS_A_NOTB_C>(held, unwanted, before);
        // sliced straight back when its target is open by then; the others stay
        // gathered and are sliced, like the axes not held at all, when their
        // blocker is gathered
        const taps_b8 kept = taps_bitop3<TAPS_A & (0xFFu ^ (TAPS_B & TAPS_C))>(held, dst, ready);
        const taps_b8 later = todo & ~ready;
        const taps_b8 us = taps_map(unwanted, P.order);
        const taps_b8 plus = taps_map(D & kept, P.order);
        const taps_b8 minus = taps_map(D & later, ns) & ~us;
        uint32_t g;
        const taps_b8 first = taps_states(plus & us, G, g);
        const taps_b8 then = taps_states((plus & ~us) - minus, g, g);
        at_r = taps_map(taps_blend(us, first, then), P.rank);
        if (kLow) {
            const taps_b8 plus2 = taps_map(D2 & kept, P.order);
            const taps_b8 minus2 = taps_map(D2 & later, ns) & ~us;
            uint32_t h;
            const taps_b8 first2 = taps_states(plus2 & us, H, h);
            const taps_b8 then2 = taps_states((plus2 & ~us) - minus2, h, h);
            at_r2 = taps_map(taps_blend(us, first2, then2), P.rank);
        }
    }

    // ---- "remove": every axis gathered in producer order.  ("Naive", the fourth of
    // Table 2, gathers a superset of these in the same order: never cheaper, and it
    // wins no tie.)
    const taps_b8 Dh = D & held;
    uint32_t g_end;
    const taps_b8 at_m = taps_map(taps_states(taps_map(Dh, P.order), P.g, g_end), P.rank);
    taps_b8 at_m2 = {0u, 0u}, Dh2 = {0u, 0u};
    if (kLow) {
        uint32_t h_end;
        Dh2 = D2 & held;
        at_m2 = taps_map(taps_states(taps_map(Dh2, P.order), P.h, h_end), P.rank);
    }

    // ---- costs.  A gather of an axis of width w at shard 2^e (e + w <= 8) moves
    // 2^(e + w) - 2^e (Eq. 9), an AllToAll 2^e - 2^(e - w) (Eq. 10); out of a block,
    // 2^(beta - u) groups share the link, u the free levels below beta, the
    // axis's own among them (Algorithm 3).
    const taps_b8 width = Dh & taps_all(0x0F0F0F0Fu);
    uint32_t in1 = 0, in2 = 0, a2a_in = 0, out1 = 0, out2 = 0, out3 = 0, a2a_out = 0;
    uint32_t ct1 = 0, ct2 = 0, ct3 = 0;
    uint32_t link1[TAPS_D_MAX_CLASSES] = {0u}, link2[TAPS_D_MAX_CLASSES] = {0u};
    uint32_t link3[TAPS_D_MAX_CLASSES] = {0u}, a2a_link[TAPS_D_MAX_CLASSES] = {0u};
    const taps_b8 more = width - (held & taps_all(0x01010101u));   // w - 1
    auto inside = [&](uint32_t l) {   // levels l .. l + 3 inside a node
        const uint32_t sel = taps_four(l, m.first[1]);
        const uint32_t hm = taps_perm(held.hi, held.lo, sel), mo = taps_perm(more.hi, more.lo, sel);
        const uint32_t am = taps_perm(a2a.hi, a2a.lo, sel);
        // 2^w - 1 of the axes held, and of those gathered
        const uint32_t gain = taps_perm(0xFF7F3F1Fu, 0x0F070301u, mo) & hm;
        const uint32_t e1 = taps_pow2(taps_perm(at.hi, at.lo, sel) & 0x07070707u);
        const uint32_t e2 = taps_pow2(taps_perm(at_r.hi, at_r.lo, sel) & 0x07070707u);
        in1 = taps_dot4(gain & ~am, e1, in1);
        in2 = taps_dot4(gain, e2, in2);
        a2a_in = taps_dot4(taps_perm(row.a2a.hi, row.a2a.lo, sel) & am, e1, a2a_in);
    };
    auto outside = [&](uint32_t c, uint32_t l) {   // levels l .. l + 3 of class c
        const uint32_t sel = taps_four(l, m.first[c + 1u]);
        const uint32_t hm = taps_perm(held.hi, held.lo, sel), mo = taps_perm(more.hi, more.lo, sel);
        const uint32_t am = taps_perm(a2a.hi, a2a.lo, sel), one = hm & 0x01010101u;
        const uint32_t y1 = taps_perm(at.hi, at.lo, sel), y2 = taps_perm(at_r.hi, at_r.lo, sel);
        const uint32_t y3 = taps_perm(at_m.hi, at_m.lo, sel);
        // the axes' own levels below this class's boundary, and with them the free ones
        const uint32_t own = c == 1u ? taps_perm(Dh.hi, Dh.lo, sel) & 0xE0E0E0E0u
                                     : taps_perm(Dh2.hi, Dh2.lo, sel);
        auto u_of = [&](uint32_t y, const taps_b8 &z) {
            const uint32_t f = (c == 1u ? y : taps_perm(z.hi, z.lo, sel)) + own;
            return (c == 1u ? f >> 5 : c == 2u ? f : f >> 4) & 0x07070707u;
        };
        const uint32_t u1 = u_of(y1, at2);
        const taps_b8 share = m.share[c];
        const uint32_t s1 = taps_perm(share.hi, share.lo, u1);
        const uint32_t s2 = taps_perm(share.hi, share.lo, u_of(y2, at_r2));
        const uint32_t s3 = taps_perm(share.hi, share.lo, u_of(y3, at_m2));
        // the gathers' volumes, a byte each, of the axes in mask
        auto volumes = [&](uint32_t e, uint32_t mask) {
            const uint32_t hi = taps_perm(0xFF7F3F1Fu, 0x0F070301u, e + mo);   // 2^(k + 1) - 1
            const uint32_t lo = taps_perm(0x7F3F1F0Fu, 0x07030100u, e);        // 2^k - 1
            return taps_bitop3<TAPS_A & (0xFFu ^ TAPS_B) & TAPS_C>(hi, lo, mask);
        };
        const uint32_t e = y1 & 0x07070707u;
        const uint32_t v1 = volumes(e, hm & ~am), v2 = volumes(y2 & 0x07070707u, hm);
        const uint32_t v3 = volumes(y3 & 0x07070707u, hm);
        out1 = taps_dot4(v1, 0x01010101u, out1);
        out2 = taps_dot4(v2, 0x01010101u, out2);
        out3 = taps_dot4(v3, 0x01010101u, out3);
        link1[c] = taps_dot4(v1, s1, link1[c]);
        link2[c] = taps_dot4(v2, s2, link2[c]);
        link3[c] = taps_dot4(v3, s3, link3[c]);
        ct1 = taps_dot4(one, s1, ct1);
        ct2 = taps_dot4(one, s2, ct2);
        ct3 = taps_dot4(one, s3, ct3);
        // AllToAlls: the link carries 2^e times the share without the axis's own
        // levels, 2^x with x up to 14: the bytes of x < 8 and of x >= 8 apart
        a2a_out = taps_dot4(taps_perm(row.a2a.hi, row.a2a.lo, sel) & am, taps_pow2(e), a2a_out);
        const uint32_t kap = (c == 1u ? own >> 5 : c == 2u ? own : own >> 4) & 0x07070707u;
        const uint32_t x = e + m.beta[c] * 0x01010101u - (u1 & hm) + kap;
        const uint32_t part = taps_perm(row.link.hi, row.link.lo, sel) & am;
        const uint32_t p = taps_pow2(x & 0x07070707u);
        const uint32_t big = part & taps_perm(0u, 0x00008000u, x & 0x08080808u);
        a2a_link[c] += taps_dot4(part, p, 0u) + taps_dot4(big, p, 0u) * 255u;
    };
    inside(0u);
    if (m.first[1] > 4u) inside(4u);   // uniform, as below
#pragma unroll
    for (uint32_t c = 1; c < C; ++c) {
        if (C == 2 || m.first[c] < m.first[c + 1u]) outside(c, m.first[c]);
        if (m.first[c + 1u] - m.first[c] > 4u) outside(c, m.first[c] + 4u);
    }
    const uint32_t in_1 = (in1 << 8) + a2a_in, out_1 = (out1 << 8) + a2a_out;
    const uint32_t vol_m = (1u << (g_end & 15u)) - (1u << (P.g & 15u));   // telescopes
    out.c[0].vol = in_1 + out_1;
    out.c[0].in = in_1;
    out.c[0].ct = ct1;
    out.c[1].vol = (in2 + out2) << 8;
    out.c[1].in = in2 << 8;
    out.c[1].ct = ct2;
    out.c[2].vol = vol_m << 8;
    out.c[2].in = (vol_m - out3) << 8;
    out.c[2].ct = ct3;
#pragma unroll
    for (uint32_t c = 1; c < C; ++c) {
        out.c[0].link[c - 1u] = (link1[c] << 8) + a2a_link[c];
        out.c[1].link[c - 1u] = link2[c] << 8;
        out.c[2].link[c - 1u] = link3[c] << 8;
    }
    out.a2a_in = a2a_in;
    const taps_b8 h01 = held & taps_all(0x01010101u);
    out.coll = taps_dot4(h01.hi, m.coll.hi, taps_dot4(h01.lo, m.coll.lo, 0u));
}

// taps_device.h -- what the TAPS cost-table kernels and the host plan share:
// strategies in canonical order, the intra-op costs, records and link classes.
//
// Every device count here is a power of two, N = 2^n devices with L = 2^lam
// per node, so a device matrix is described by its binary levels 0..n-1
// (level 0 innermost; a device's rank bit l is its coordinate bit on level
// l; levels < lam lie inside one node).  A strategy gives each split op axis
// a contiguous run of levels; a tensor dimension inherits the run of its op
// axis.  All set operations of the cost model become bit operations on
// at most 8 levels:
//
//   * intra-op AllReduce of a tensor (Eq. 5-7, Algorithm 2): the group spans
//     the levels G the tensor does not use; ct is 0 when G lies below lam,
//     else 2^(lam - |G below lam|);
//   * the redistribution of an edge's tensor: taps_entry.h.
//
// Volumes are integers in "nb" (bytes x N), which makes every per-device
// volume exact.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#define TAPS_D_MAX_AXES 8
#define TAPS_D_MAX_RANK 8
#define TAPS_D_MAX_LEVELS 8
#define TAPS_D_MAX_CLASSES 4

__host__ __device__ inline uint32_t taps_nib(uint32_t v, uint32_t k) { return (v >> (4u * k)) & 15u; }

__host__ __device__ inline uint32_t taps_popc(uint32_t v) { return (uint32_t)__builtin_popcount(v); }

__host__ __device__ inline uint32_t taps_ctz(uint32_t v) { return (uint32_t)__builtin_ctz(v); }

__host__ __device__ inline uint32_t taps_low_mask(uint32_t k) { return k >= 32u ? ~0u : ((1u << k) - 1u); }

// Bits 0..k-1 for k < 32.
__host__ __device__ inline uint32_t taps_below(uint32_t k) { return (1u << k) - 1u; }

// w one-bits starting at bit o, ((1 << w) - 1) << o, for w, o < 32 and w + o <= 32:
// one v_bfm_b32 on the device.
__host__ __device__ inline uint32_t taps_bfm(uint32_t w, uint32_t o) {
#if defined(__HIP_DEVICE_COMPILE__)
    uint32_t r;
    __asm__("v_bfm_b32 %0, %1, %2" : "=v"(r) : "v"(w), "v"(o));
    return r;
#else
    return ((1u << w) - 1u) << o;
#endif
}

// x << K for a result below 2^16, the shift an inline constant.
template <uint32_t K>
__host__ __device__ inline uint32_t taps_shl16c(uint32_t x) {
#if defined(__HIP_DEVICE_COMPILE__)
    uint32_t r;
    __asm__("v_lshlrev_b16 %0, %2, %1" : "=v"(r) : "v"(x), "i"(K));
    return r;
#else
    return (x << K) & 0xFFFFu;
#endif
}

// Entry i (< 2^16 / sizeof(T)) of a small table: the byte offset by a 16-bit shift.
template <uint32_t LogSize, typename T>
__host__ __device__ inline const T &taps_entry(const T *tab, uint32_t i) {
    static_assert(sizeof(T) == (1u << LogSize), "entry size");
    return *(const T *)((const char *)tab + taps_shl16c<LogSize>(i));
}

// Levels lo .. lo+w-1 (lo + w <= 8).
__host__ __device__ inline uint32_t taps_levels(uint32_t lo, uint32_t w) {
    return taps_below(lo + w) & ~taps_below(lo);
}

// ---------------------------------------------------------------------------
// GenerateStrategySet in canonical order (Auxiliary Graph section, Table 3).
//
// Order: the exponent tuple (log2 degree per op axis, axis 0 most
// significant) ascending; within one exponent tuple the device-map tuple
// (position per split axis, in axis order) descending.  Counting is done
// with w(k, s, z) = the number of strategies that complete a prefix with z
// split axes so far, s levels still to hand out and k partitionable axes
// left: sum_j C(k, j) C(s-1, j-1) (z+j)!  (s = 0: z!).  With k = p, s = n,
// z = 0 this is the paper's count sum_i i! C(p,i) C(n-1,i-1).
// ---------------------------------------------------------------------------

__host__ __device__ constexpr uint32_t taps_binom(uint32_t a, uint32_t b) {
    if (b > a) return 0;
    uint32_t r = 1;
    for (uint32_t x = 1; x <= b; ++x) r = r * (a - b + x) / x;
    return r;
}

__host__ __device__ constexpr uint32_t taps_fact(uint32_t a) {
    uint32_t r = 1;
    for (uint32_t x = 2; x <= a; ++x) r *= x;
    return r;
}

// w(k, s, z); only states with z + s <= 8 occur (each split axis takes at
// least one level), where every term has z + j <= 8 and the sum stays below
// 2^32; other entries are never read.
__host__ __device__ constexpr uint32_t taps_completions(uint32_t k, uint32_t s, uint32_t z) {
    if (z + s > TAPS_D_MAX_LEVELS) return 0;
    if (s == 0) return taps_fact(z);
    uint32_t tot = 0;
    const uint32_t jmax = k < s ? k : s;
    for (uint32_t j = 1; j <= jmax; ++j)
        tot += taps_binom(k, j) * taps_binom(s - 1, j - 1) * taps_fact(z + j);
    return tot;
}

struct taps_completion_table {
    uint32_t v[9 * 9 * 9];   // index (k * 9 + s) * 9 + z
};

__host__ __device__ constexpr taps_completion_table taps_make_completions() {
    taps_completion_table t{};
    for (uint32_t x = 0; x < 9u * 9u * 9u; ++x) t.v[x] = taps_completions(x / 81u, (x / 9u) % 9u, x % 9u);
    return t;
}

// A strategy as nibbles by op axis: log2 degrees and device-matrix positions
// (15: not split).
struct taps_nibbles {
    uint32_t expo, pos;
};

// Decodes candidate r (0 <= r < w(p, n, 0)) of the partitionable axes `part`;
// W: the completion table (in LDS on the device).  No array is indexed by a
// value that varies over a wavefront, so everything stays in registers.
__host__ __device__ inline taps_nibbles taps_unrank(uint32_t part, uint32_t n, uint32_t r,
                                                    const uint32_t *W) {
    taps_nibbles S = {0u, ~0u};
    uint32_t s = n, z = 0;
    for (uint32_t m = part; m; m &= m - 1u) {   // uniform
        const uint32_t k = taps_popc(m) - 1u, a = taps_ctz(m);
        const uint32_t *row = W + k * 81u + z;
        const uint32_t none = row[s * 9u];
        if (r < none) continue;
        r -= none;
        uint32_t e = 1;
        for (; e < s; ++e) {   // the last exponent takes what is left
            const uint32_t c = row[(s - e) * 9u + 1u];
            if (r < c) break;
            r -= c;
        }
        S.expo |= e << (4u * a);
        s = s > e ? s - e : 0u;
        ++z;
    }
    // r is now the rank of the position tuple among the z! orderings, in
    // descending order: the (z! - 1 - r)-th ascending permutation, its digits
    // (how many of the j positions left are passed over) from the last
    uint32_t q = taps_fact(z) - 1u - r, digits = 0;
#pragma unroll
    for (uint32_t j = 2; j <= 8u; ++j) {
        const uint32_t d = q / j;
        digits |= (q - d * j) << (4u * (j - 1u));
        q = d;
    }
    uint32_t left = 0x76543210u;   // the free positions, ascending
    for (uint32_t m = part; m; m &= m - 1u) {   // uniform
        const uint32_t a4 = 4u * taps_ctz(m);
        if (!((S.expo >> a4) & 15u)) continue;
        --z;
        const uint32_t d4 = 4u * ((digits >> (4u * z)) & 7u);
        const uint32_t below = (1u << d4) - 1u, p = (left >> d4) & 15u;
        left = (left & below) | ((left >> 4) & ~below);
        S.pos = (S.pos & ~(15u << a4)) | (p << a4);
    }
    return S;
}

// ---------------------------------------------------------------------------
// Records
// ---------------------------------------------------------------------------

struct taps_acc {
    uint64_t vol, intra, inter;
    uint32_t n_coll, n_inter, sum_ct;
};

__host__ __device__ inline void taps_acc_zero(taps_acc &c) {
    c.vol = c.intra = c.inter = 0;
    c.n_coll = c.n_inter = c.sum_ct = 0;
}

__host__ __device__ inline uint32_t taps_meta(uint32_t cand, const taps_acc &c) {
    return cand | (c.n_coll << 2) | (c.n_inter << 7) | (c.sum_ct << 12);
}

// ---------------------------------------------------------------------------
// Intra-op cost (Eq. 5-8 with Algorithm 2 and Eq. 11-12): one ring AllReduce
// over the levels a tensor does not use.  bytes = elements x dtype bytes.
// ---------------------------------------------------------------------------
__host__ __device__ inline void taps_allreduce(taps_acc &c, uint32_t missing, uint64_t bytes,
                                               uint32_t lam) {
    if (!missing) return;
    uint32_t lg = taps_popc(missing);
    uint64_t V = ((bytes << lg) - bytes) << 1;   // 2 (g - 1) |tensor| bytes, in nb
    c.vol += V;
    c.n_coll += 1;
    if ((missing >> lam) == 0) {
        c.intra += V;
        return;
    }
    uint32_t lct = lam - taps_popc(missing & taps_low_mask(lam));
    c.inter += V << lct;
    c.n_inter += 1;
    c.sum_ct += 1u << lct;
}

// Sum of the four byte products of a and b, plus c: one v_dot4_u32_u8.
__host__ __device__ inline uint32_t taps_dot4(uint32_t a, uint32_t b, uint32_t c) {
#if defined(__HIP_DEVICE_COMPILE__)
    return __builtin_amdgcn_udot4(a, b, c, false);
#else
    for (uint32_t k = 0; k < 32u; k += 8u) c += ((a >> k) & 0xFFu) * ((b >> k) & 0xFFu);
    return c;
#endif
}

// ---------------------------------------------------------------------------
// Edge records
// ---------------------------------------------------------------------------

// One candidate of an edge entry under the paper's two link classes.  An edge's
// volumes are its tensor's bytes times a power of two times a small integer, so
// they are counted in units of tbytes / 256 ("factor units", 32 bits) and
// scaled by tbytes once, exactly, at the end; comparing two candidates of one
// entry does not need tbytes at all.  ct: the sum of the inter-node group
// counts (Algorithm 3) of its collectives.
struct taps_fac {
    uint32_t vol, intra, inter;
    uint32_t ct;
};

// Exact order of intra/(N B_intra) + inter/(N B_inter) between candidates:
// intra * bi + inter * ba with bi = B_inter / g, ba = B_intra / g
// (g = gcd of the two).  Both products fit 64 bits when bi, ba < 2^32.
struct taps_keys {
    uint64_t b_inter_red, b_intra_red;
    bool narrow;   // both reduced bandwidths below 2^32
};

__host__ __device__ inline uint64_t taps_key64(const taps_fac &a, const taps_keys &K) {
    return (uint64_t)a.intra * (uint32_t)K.b_inter_red + (uint64_t)a.inter * (uint32_t)K.b_intra_red;
}

__host__ __device__ inline bool taps_less(const taps_fac &a, const taps_fac &b,
                                          const taps_keys &K) {
    if (K.narrow) return taps_key64(a, K) < taps_key64(b, K);
    const unsigned __int128 ka =
        (unsigned __int128)a.intra * K.b_inter_red + (unsigned __int128)a.inter * K.b_intra_red;
    const unsigned __int128 kb =
        (unsigned __int128)b.intra * K.b_inter_red + (unsigned __int128)b.inter * K.b_intra_red;
    return ka < kb;
}

// How the factor-unit sums of one edge become record numbers (uniform over
// the edge): volumes are tbytes * f / 256 nb, exact; t uses the per-unit
// seconds a = tbytes / 256 / (N B).
struct taps_scaler {
    uint64_t tbytes;
    uint32_t q;         // tbytes / 256 when that is exact and below 2^32, else 0
    double a_intra;     // tbytes / 256 / (N B_intra)
    double a_inter;     // tbytes / 256 / (N B_inter)
};

__host__ __device__ inline taps_scaler taps_make_scaler(uint64_t tbytes, double inv_n_bintra,
                                                        double inv_n_binter) {
    taps_scaler S;
    S.tbytes = tbytes;
    S.q = (tbytes & 255u) == 0 && (tbytes >> 40) == 0 ? (uint32_t)(tbytes >> 8) : 0u;
    const double unit = (double)tbytes * (1.0 / 256.0);   // exact: tbytes < 2^53
    S.a_intra = unit * inv_n_bintra;
    S.a_inter = unit * inv_n_binter;
    return S;
}

// tbytes * f / 256, exact (the result is an integer volume in nb < 2^64).
__host__ __device__ inline uint64_t taps_scale(const taps_scaler &S, uint32_t f) {
    if (S.q) return (uint64_t)S.q * f;
    return (((S.tbytes & 0xFFFFFFFFull) * f) >> 8) + (((S.tbytes >> 32) * f) << 24);
}

struct taps_entry_out {
    double t;
    uint64_t vol, intra, inter;
    uint32_t meta;
};

// ---------------------------------------------------------------------------
// Link-class hierarchies (an extension of the paper's two classes).
//
// Blocks of 2^beta_0 <= 2^beta_1 <= ... consecutive ranks (a node, a group of
// nodes, ...; the last class spans all devices).  A collective belongs to
// the smallest block that holds each of its groups: with top level t that is
// class c = the number of boundaries beta <= t; it pays bw[c] divided by the
// number of groups sharing the uplink of one block of the largest boundary
// beta <= t (Algorithm 2 / 3 and the AllToAll paragraph with "node" read as
// that block).  With one boundary (beta = lam) this is the two-class model.
// Volumes are factor units (taps_fac), accumulated per class, and candidates
// compare by the exact key sum_c x_c w_c with w_c = lcm(bw) / bw_c.
// ---------------------------------------------------------------------------
struct taps_hier {
    uint32_t n_classes;     // 1 .. TAPS_D_MAX_CLASSES
    uint32_t cls_of_top;    // nibble t: class of a collective whose top level is t
    uint32_t beta_of_top;   // nibble t: the largest boundary <= t (0 for class 0)
    uint32_t pad;
    uint64_t w[TAPS_D_MAX_CLASSES];        // exact-order weights, each below 2^30
    double inv_n_bw[TAPS_D_MAX_CLASSES];   // 1 / (N bw[c])
    uint64_t w_a2a;          // weight of the in-block AllToAll volume (0: priced as class 0)
    double inv_n_bw_a2a;     // 1 / (N bw_a2a)
    uint32_t a2a_own;        // 1: in-block AllToAlls have a bandwidth of their own
    uint32_t pad2;
    uint32_t boundary[TAPS_D_MAX_CLASSES];        // log2 of the block below class c >= 1
};

// Intra-op AllReduce (Eq. 5-8) of a tensor missing the levels `missing`,
// under link classes: nb volumes per class.
struct taps_acch {
    uint64_t vol, x0, x1, x2, x3;
    uint32_t n_coll, n_inter, sum_ct;
};

__host__ __device__ inline uint32_t taps_msb(uint32_t v) { return 31u - (uint32_t)__builtin_clz(v); }

__host__ __device__ inline void taps_allreduce_h(taps_acch &c, uint32_t missing, uint64_t bytes,
                                                 const taps_hier &H) {
    if (!missing) return;
    const uint32_t lg = taps_popc(missing);
    const uint64_t V = ((bytes << lg) - bytes) << 1;   // 2 (g - 1) |tensor| bytes, in nb
    const uint32_t top = taps_msb(missing);
    const uint32_t cls = taps_nib(H.cls_of_top, top);
    c.vol += V;
    c.n_coll += 1;
    if (!cls) {
        c.x0 += V;
        return;
    }
    const uint32_t beta = taps_nib(H.beta_of_top, top);
    const uint32_t lct = beta - taps_popc(missing & taps_below(beta));
    const uint64_t X = V << lct;
    c.x1 += cls == 1 ? X : 0u;
    c.x2 += cls == 2 ? X : 0u;
    c.x3 += cls == 3 ? X : 0u;
    c.n_inter += 1;
    c.sum_ct += 1u << lct;
}

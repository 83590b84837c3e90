// taps_kernels.hip -- gfx950 kernels of the TAPS cost tables.
//
//   k_build_strategies  one workgroup per chunk of 256 candidate ranks of an
//                 operator: GenerateStrategySet in canonical order at
//                 host-counted offsets (ballot, LDS scan), optionally each
//                 strategy's descriptor and node record
//   k_node_costs  one thread per strategy: the intra-op AllReduces
//   k_memory_costs one thread per strategy: weight and output shard bytes
//   k_edge_front  the descriptors of given strategies, one thread each, and the
//                 edge plan: one thread per computed edge (its constants), one
//                 per window (the edge it starts in)
//   k_build_front k_build_strategies and the edge plan in one launch
//   k_edge_costs  one wavefront per window of aligned 64-entry tiles of the
//                 concatenated tables, one entry per lane whatever its row
//                 (taps_entry.h); whole-line stores
//   k_edge_costs_sweep  the same at several bandwidth points: the candidates
//                 once per entry, one selection and store per point
//   k_edge_costs_h  the same under a hierarchy of link classes
//   k_*_crowded   the windows in which many small tables meet, a lane its own
//   k_copy_tables shared tables: one workgroup per chunk of a computed
//                 table, written to every table that shares it
//   k_pull        a call's upload, read from pinned host memory
#include <cstddef>

#include "taps_internal.h"

namespace {

constexpr uint32_t kWave = 64;

// Widths of the unified axes by their tops.
__constant__ taps_top_table kTops = taps_make_tops();
// Completion counts w(k, s, z) for k, s, z in 0..8 (see taps_completions),
// evaluated by the compiler.
__constant__ taps_completion_table kCompletions = taps_make_completions();

template <typename T>
__device__ inline T *at_byte(T *base, uint32_t offset) {
    return (T *)((char *)base + offset);
}

// Entry row + j (of a window: row uniform, j the lane; 32-bit byte offsets from
// the five scalar bases).  Non-temporal stores: a tile of one edge is whole
// 128-byte lines where the tables lie end to end from a line on, as in a build
// without sharing, and nothing is left to merge (cached stores take the 24-layer
// GPT's build from 80.6 to 82.5 us; arrays that start between lines, the
// 96-layer GPT's edges from 1284 to 1326).  Cached: ordinary stores, into the
// tables of several bandwidth points (TAPS_WINDOW_SWEEP has both).
template <bool Cached>
__device__ inline void store_entry(const taps_table &out, uint64_t row, uint32_t j,
                                   const taps_entry_out &o, uint32_t meta) {
    uint32_t o8 = j * 8u, o4 = j * 4u;
    // made here and not kept across the loop as five 64-bit addresses
    __asm__ volatile("" : "+v"(o8), "+v"(o4));
    if (Cached) {
        *at_byte(out.t + row, o8) = o.t;
        *at_byte(out.vol + row, o8) = o.vol;
        *at_byte(out.intra + row, o8) = o.intra;
        *at_byte(out.inter + row, o8) = o.inter;
        *at_byte(out.meta + row, o4) = meta;
        return;
    }
    __builtin_nontemporal_store(o.t, at_byte(out.t + row, o8));
    __builtin_nontemporal_store(o.vol, at_byte(out.vol + row, o8));
    __builtin_nontemporal_store(o.intra, at_byte(out.intra + row, o8));
    __builtin_nontemporal_store(o.inter, at_byte(out.inter + row, o8));
    __builtin_nontemporal_store(meta, at_byte(out.meta + row, o4));
}

__device__ inline uint32_t lanes_below(uint64_t mask) {
    return __builtin_amdgcn_mbcnt_hi((uint32_t)(mask >> 32),
                                     __builtin_amdgcn_mbcnt_lo((uint32_t)mask, 0u));
}

// A strategy's bytes as nibbles (positions past 7 or negative: 15).
__device__ inline taps_nibbles strategy_nibbles(const taps_strategy &st) {
    taps_nibbles S = {0u, 0u};
#pragma unroll
    for (uint32_t a = 0; a < TAPS_MAX_AXES; ++a) {
        const uint32_t p = (uint8_t)st.pos[a];
        S.expo |= (uint32_t)(st.log2_deg[a] & 15u) << (4u * a);
        S.pos |= (p < 8u ? p : 15u) << (4u * a);
    }
    return S;
}

// largest k in [0, n) with offsets[k] <= x
__device__ inline uint32_t find_owner(const uint64_t *offsets, uint32_t n, uint64_t x) {
    uint32_t lo = 0, hi = n;
    while (hi - lo > 1) {
        uint32_t mid = (lo + hi) >> 1;
        if (offsets[mid] <= x)
            lo = mid;
        else
            hi = mid;
    }
    return lo;
}

// The owner of a wavefront's lane's x (x of lane l: first + l, or less at the
// end), as find_owner: 64 offsets per step for the first lane's, then the
// offsets after that one, at most one per lane as every range holds something.
// All lanes take part.
__device__ inline uint32_t wave_owner(const uint64_t *offsets, uint32_t n, uint64_t x) {
    const uint32_t lane = threadIdx.x % kWave;
    const uint64_t first = ((uint64_t)__builtin_amdgcn_readfirstlane((uint32_t)(x >> 32)) << 32) |
                           __builtin_amdgcn_readfirstlane((uint32_t)x);
    uint32_t lo = 0, size = n;   // largest k in [lo, lo + size) with offsets[k] <= first
    for (;;) {
        const uint32_t stride = (size + kWave - 1u) / kWave, k = lane * stride;
        const uint64_t m = __ballot(k < size && offsets[lo + (k < size ? k : 0u)] <= first);
        const uint32_t j = ((uint32_t)__builtin_popcountll(m) - 1u) * stride;
        lo += j;
        if (stride == 1u) break;
        size = size - j < stride ? size - j : stride;
    }
    const uint64_t next = offsets[n - lo > lane + 1u ? lo + lane + 1u : n];
    uint32_t more = 0;
#pragma unroll
    for (uint32_t step = kWave / 2; step; step /= 2) {
        const uint32_t at = more + step - 1u;
        const uint64_t o = ((uint64_t)__shfl((uint32_t)(next >> 32), at) << 32) |
                           __shfl((uint32_t)next, at);
        more += o <= x ? step : 0u;
    }
    return lo + more;
}

// An operator's description in registers, read as words all at once: its bytes
// one by one are a chain of some 30 dependent loads.
struct op_words {
    uint32_t w[sizeof(taps_op) / 4u];
    __device__ uint32_t byte(uint32_t at) const { return (w[at / 4u] >> (8u * (at % 4u))) & 0xFFu; }
    __device__ uint64_t length(uint32_t a) const {
        const uint32_t at = offsetof(taps_op, axis_len) / 4u + 2u * a;
        return ((uint64_t)w[at + 1u] << 32) | w[at];
    }
    // the axes of the tensor at byte `at`, which names an axis at most once
    __device__ uint32_t axes(uint32_t at) const {
        const uint32_t rank = byte(at);
        uint32_t m = 0;
#pragma unroll
        for (uint32_t d = 0; d < TAPS_MAX_RANK; ++d)
            if (d < rank) m |= 1u << (byte(at + 1u + d) & 7u);
        return m;
    }
    // f(at) for the output, the inputs and the weights
    template <typename F> __device__ void tensors(bool inputs, const F &f) const {
        const uint32_t n_in = inputs ? byte(offsetof(taps_op, n_in)) : 0u;
        const uint32_t n_w = byte(offsetof(taps_op, n_w));
        f(offsetof(taps_op, out));
#pragma unroll
        for (uint32_t q = 0; q < TAPS_MAX_INPUTS; ++q)
            if (q < n_in) f(offsetof(taps_op, in) + q * sizeof(taps_tensor));
#pragma unroll
        for (uint32_t q = 0; q < TAPS_MAX_WEIGHTS; ++q)
            if (q < n_w) f(offsetof(taps_op, w) + q * sizeof(taps_tensor));
    }
};

// A lane's own operator.
__device__ inline op_words read_op(const taps_op *op) {
    static_assert(sizeof(taps_op) % 16 == 0, "16-byte loads of operators");
    op_words o;
#pragma unroll
    for (uint32_t x = 0; x < sizeof(taps_op) / 16u; ++x) {
        const uint4 v = ((const uint4 *)op)[x];
        o.w[4 * x] = v.x, o.w[4 * x + 1] = v.y, o.w[4 * x + 2] = v.z, o.w[4 * x + 3] = v.w;
    }
    return o;
}

// add(levels without the tensor, its bytes) for every tensor of an operator;
// byte a of (hi, lo): the levels of axis a.
template <typename Add>
__device__ inline void node_tensors(const op_words &op, uint32_t lo, uint32_t hi, uint32_t full,
                                    const Add &add) {
    op.tensors(true, [&](uint32_t at) {
        const uint32_t axes = op.axes(at);
        uint64_t size = op.byte(offsetof(taps_op, dtype_bytes));
        uint32_t used = 0;
#pragma unroll
        for (uint32_t a = 0; a < TAPS_MAX_AXES; ++a)
            if ((axes >> a) & 1u) {
                size *= op.length(a);
                used |= (a < 4u ? lo : hi) >> (8u * (a & 3u));
            }
        add(full & ~used, size);
    });
}

// The same for strategy s of a lane's own operator.
template <typename Add>
__device__ inline void strategy_tensors(const taps_op *op, const taps_strategy &s, uint32_t n,
                                        const Add &add) {
    const op_words o = read_op(op);
    const taps_packed D = taps_lay_out(strategy_nibbles(s), 0xFFu, n).packed;
    uint32_t lo = 0, hi = 0;
#pragma unroll
    for (uint32_t a = 0; a < TAPS_MAX_AXES; ++a)
        (a < 4u ? lo : hi) |= (taps_axis_levels(D, a) & 0xFFu) << (8u * (a & 3u));
    node_tensors(o, lo, hi, taps_low_mask(n), add);
}

__device__ inline void store_node(const taps_table &node, uint64_t idx, const taps_acc &c,
                                  const taps_launch &lp) {
    node.t[idx] = (double)c.intra * lp.inv_n_bintra + (double)c.inter * lp.inv_n_binter;
    node.vol[idx] = c.vol;
    node.intra[idx] = c.intra;
    node.inter[idx] = c.inter;
    node.meta[idx] = taps_meta(0, c);
}

// One thread per strategy, from the strategies themselves.  Bound by latency:
// the owner's offsets, then operator and strategy together, then arithmetic
// (6,400 strategies 4.9 us, 9.3 with descriptors from a launch of their own and
// the operators read byte by byte; k_memory_costs 3.8, 6.4 before).
__global__ __launch_bounds__(256) void k_node_costs(const taps_op *__restrict__ ops, uint32_t n_ops,
                                                    const uint64_t *__restrict__ offsets,
                                                    const taps_strategy *__restrict__ strategies,
                                                    uint64_t total, taps_launch lp, taps_table out) {
    const uint64_t idx = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const uint64_t x = idx < total ? idx : total - 1u;
    const taps_op *op = ops + wave_owner(offsets, n_ops, x);
    taps_acc c;
    taps_acc_zero(c);
    strategy_tensors(op, strategies[x], lp.n, [&](uint32_t missing, uint64_t bytes) {
        taps_allreduce(c, missing, bytes, lp.lam);
    });
    if (idx < total) store_node(out, idx, c, lp);
}

// GenerateStrategySet, and the whole strategy side of a single-call build, in
// one launch: one workgroup per chunk of 256 consecutive candidate ranks of
// one operator (only chunks that hold a strategy are launched) tests its
// candidates in canonical order (a ballot per wavefront, the four wavefront
// counts scanned in LDS) and writes every valid strategy together with, when
// asked (desc and node.t not NULL), its descriptor and its node (intra-op)
// record.  A chunk's strategies go to [base, base + count), where the host
// counted them with the same unranking and filter (plan_build checks the
// chunks' counts against the exact per-operator count); nothing is written
// outside that range.
constexpr uint32_t kBuildThreads = TAPS_BUILD_CHUNK;

// The strategies of one chunk of candidate ranks (a whole workgroup).
__device__ inline void build_chunk(const taps_build_chunk &ck, const taps_op *__restrict__ ops,
                                   uint32_t allowed_cuts, const taps_launch &lp,
                                   taps_strategy *__restrict__ out,
                                   taps_packed *__restrict__ desc, const taps_table &node) {
    __shared__ uint32_t W[9 * 9 * 9];
    __shared__ uint32_t wave_count[kBuildThreads / kWave];
    const uint32_t tid = threadIdx.x, lane = tid % kWave, wave = tid / kWave;
    for (uint32_t x = tid; x < 9u * 9u * 9u; x += blockDim.x) W[x] = kCompletions.v[x];
    // the operator, the same for the whole workgroup: read as words (scalar loads;
    // its bytes one by one were a chain of some 30 dependent vector loads, most of
    // this kernel's time) and taken apart on the scalar unit
    const uint32_t *words = (const uint32_t *)(ops + ck.op);
    op_words op;
#pragma unroll
    for (uint32_t x = 0; x < sizeof(taps_op) / 4u; ++x) op.w[x] = words[x];
    const uint32_t part = op.byte(offsetof(taps_op, part_mask));
    uint32_t most = 0;   // nibble a: the largest exponent that divides axis a's length
#pragma unroll
    for (uint32_t a = 0; a < TAPS_MAX_AXES; ++a) {
        const uint64_t len = op.length(a) | 256u;   // exponents end at 8
        most |= (uint32_t)__builtin_ctzll(len) << (4u * a);
    }
    __syncthreads();
    const uint32_t total = W[(taps_popc(part) * 9u + lp.n) * 9u];
    const uint32_t full = taps_low_mask(lp.n);
    const uint32_t r = ck.first + tid;
    bool valid = r < total;
    const taps_nibbles S = taps_unrank(part, lp.n, valid ? r : 0u, W);
#pragma unroll
    for (uint32_t a = 0; a < TAPS_MAX_AXES; ++a)
        valid = valid && taps_nib(S.expo, a) <= taps_nib(most, a);
    const taps_runs R = taps_lay_out(S, part, lp.n);
    valid = valid && (R.cuts & ~allowed_cuts) == 0u;
    const uint64_t m = __ballot(valid);
    if (lane == 0) wave_count[wave] = (uint32_t)__builtin_popcountll(m);
    __syncthreads();
    uint32_t before = 0;
    for (uint32_t w = 0; w < wave; ++w) before += wave_count[w];
    const uint32_t k = before + lanes_below(m);
    if (!valid || k >= ck.count) return;
    const uint64_t idx = ck.base + k;
    // bytes: degrees, then positions (-1: not split)
    const uint32_t whole = ~(S.pos & (S.pos >> 1) & (S.pos >> 2) & (S.pos >> 3)) & 0x11111111u;
    auto bytes = [](uint32_t nibbles) { return taps_spread(nibbles & 0xFFFFu); };
    const uint32_t not_lo = bytes(0x11111111u & ~whole) * 0xFFu;
    const uint32_t not_hi = bytes((0x11111111u & ~whole) >> 16) * 0xFFu;
    taps_store_strategy(out + idx, {bytes(S.expo), bytes(S.expo >> 16)},
                        {bytes(S.pos) | not_lo, bytes(S.pos >> 16) | not_hi});
    if (desc) desc[idx] = R.packed;   // uniform: descriptors and node records are optional
    if (!node.t) return;
    // levels of every axis, a byte each
    uint32_t lv_lo = 0, lv_hi = 0;
#pragma unroll
    for (uint32_t a = 0; a < TAPS_MAX_AXES; ++a) {
        if (!((part >> a) & 1u)) continue;
        const uint32_t v = taps_bfm(taps_nib(R.width, a), taps_nib(R.lo, a)) & 0xFFu;
        (a < 4u ? lv_lo : lv_hi) |= v << (8u * (a & 3u));
    }
    taps_acc c;
    taps_acc_zero(c);
    node_tensors(op, lv_lo, lv_hi, full, [&](uint32_t missing, uint64_t bytes) {
        taps_allreduce(c, missing, bytes, lp.lam);
    });
    store_node(node, idx, c, lp);
}

__global__ __launch_bounds__(kBuildThreads) void k_build_strategies(
    const taps_op *__restrict__ ops, const taps_build_chunk *__restrict__ chunks,
    uint32_t allowed_cuts, taps_launch lp, taps_strategy *__restrict__ out,
    taps_packed *__restrict__ desc, taps_table node) {
    build_chunk(chunks[blockIdx.x], ops, allowed_cuts, lp, out, desc, node);
}

// Bytes of one shard of the output and of every weight: each dimension's
// length divided by its split degree, times the element size.
__global__ __launch_bounds__(256) void k_memory_costs(const taps_op *__restrict__ ops,
                                                      uint32_t n_ops,
                                                      const uint64_t *__restrict__ offsets,
                                                      const taps_strategy *__restrict__ strategies,
                                                      uint64_t total, uint64_t *__restrict__ memory) {
    const uint64_t idx = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const uint64_t x = idx < total ? idx : total - 1u;
    const op_words op = read_op(ops + wave_owner(offsets, n_ops, x));
    const taps_strategy s = strategies[x];
    uint64_t m = 0;
    op.tensors(false, [&](uint32_t at) {
        const uint32_t axes = op.axes(at);
        uint64_t b = op.byte(offsetof(taps_op, dtype_bytes));
#pragma unroll
        for (uint32_t a = 0; a < TAPS_MAX_AXES; ++a)
            if ((axes >> a) & 1u) b *= op.length(a) >> (s.pos[a] >= 0 ? (s.log2_deg[a] & 15u) : 0u);
        m += b;
    });
    if (idx < total) memory[idx] = m;
}

// Constants of computed edge k.
__device__ inline void edge_setup_one(uint32_t k, const taps_plan_args &pa, const taps_launch &lp) {
    const uint32_t e = pa.computed ? pa.computed[k] : k;
    const taps_edge E = pa.edges[e];
    const taps_op &src = pa.ops[E.src_op];
    const taps_op &dst = pa.ops[E.dst_op];
    const taps_tensor &T = src.out;
    const taps_tensor &Tc = dst.in[E.dst_slot];
    taps_edge_params p;
    p.out_offset = pa.edge_offsets[e];
    uint64_t bytes = src.dtype_bytes;
    uint32_t pax = 0, cax = 0;
    for (uint32_t d = 0; d < T.rank && d < TAPS_MAX_RANK; ++d) {
        bytes *= (uint64_t)src.axis_len[T.axis[d] & 7u];
        pax |= (uint32_t)(T.axis[d] & 7u) << (4u * d);
        cax |= (uint32_t)(Tc.axis[d] & 7u) << (4u * d);
    }
    p.scale = taps_make_scaler(bytes, lp.inv_n_bintra, lp.inv_n_binter);
    // the source side of the redistribution: the producer's output map, or for
    // the backward tables the consumer's input map (the gradient moves back)
    const uint32_t from = pa.reverse ? E.dst_op : E.src_op, to = pa.reverse ? E.src_op : E.dst_op;
    p.src_base = (uint32_t)pa.op_offsets[from];
    p.dst_base = (uint32_t)pa.op_offsets[to];
    p.ns = (uint32_t)(pa.op_offsets[from + 1] - pa.op_offsets[from]);
    p.nd = (uint32_t)(pa.op_offsets[to + 1] - pa.op_offsets[to]);
    p.rank = T.rank;
    p.from = taps_make_side(pa.reverse ? cax : pax, T.rank);
    p.to = taps_make_side(pa.reverse ? pax : cax, T.rank);
    p.pad = 0;
    pa.params[k] = p;
}

// The computed edge that holds the first entry of window w, ~0 for a crowded window.
__device__ inline void window_one(uint64_t w, const taps_plan_args &pa) {
    uint32_t e = find_owner(pa.starts, pa.n_edges, w * pa.window);
    if (pa.crowded && pa.n_edges - e > pa.crowded &&   // uniform, mostly 0
        pa.starts[e + pa.crowded] < (w + 1u) * pa.window)
        e = ~0u;
    pa.window_edge[w] = e;
}

// The edge plan in one launch: blocks [0, setup_blocks) set up the edges (the
// first also the edge kernels' table by tops mask), the rest map the windows.
__device__ inline void edge_plan_block(uint32_t b, uint32_t setup_blocks, const taps_plan_args &pa,
                                       const taps_launch &lp) {
    if (b == 0u && threadIdx.x < 256u) {
        taps_b8 low;
        pa.tops[threadIdx.x] = taps_make_top_row(kTops, threadIdx.x, pa.model, low);
        ((taps_b8 *)(pa.tops + 256))[threadIdx.x] = low;
    }
    if (b < setup_blocks) {
        const uint32_t e = b * blockDim.x + threadIdx.x;
        if (e < pa.n_edges) edge_setup_one(e, pa, lp);
    } else {
        const uint64_t w = (uint64_t)(b - setup_blocks) * blockDim.x + threadIdx.x;
        if (w < pa.n_windows) window_one(w, pa);
    }
}

// The front of an edge call on given strategies: their descriptors, then the
// edge plan, in one launch (two take 3 us more on the host and on the GPU).
__global__ __launch_bounds__(256) void k_edge_front(const taps_strategy *__restrict__ s,
                                                    uint64_t total, uint32_t describe_blocks,
                                                    taps_packed *__restrict__ desc,
                                                    taps_plan_args pa, taps_launch lp,
                                                    uint32_t setup_blocks) {
    if (blockIdx.x >= describe_blocks) {
        edge_plan_block(blockIdx.x - describe_blocks, setup_blocks, pa, lp);
        return;
    }
    const uint64_t idx = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (idx < total) desc[idx] = taps_lay_out(strategy_nibbles(s[idx]), 0xFFu, lp.n).packed;
}

// The front of a single-call build: the strategy chunks, then the edge plan
// (which needs only the strategy offsets, which the host counted), in one
// launch.
__global__ __launch_bounds__(kBuildThreads) void k_build_front(
    const taps_op *__restrict__ ops, const taps_build_chunk *__restrict__ chunks, uint32_t n_chunks,
    uint32_t allowed_cuts, taps_launch lp, taps_strategy *__restrict__ out,
    taps_packed *__restrict__ desc, taps_table node, taps_plan_args pa, uint32_t setup_blocks) {
    if (blockIdx.x < n_chunks)
        build_chunk(chunks[blockIdx.x], ops, allowed_cuts, lp, out, desc, node);
    else
        edge_plan_block(blockIdx.x - n_chunks, setup_blocks, pa, lp);
}

// ---------------------------------------------------------------------------
// The edge kernels.
//
// Wavefront w takes window w, one 64-entry tile at a time, lane l entry l of
// the tile: its edge is uniform (a tile that runs into the next edge is taken
// in two passes), its row and column are its own.  Rows shorter than a wavefront
// leave no lane idle, and a tile of one edge is stored in whole 128-byte lines
// (but for shared tables, whose places in the output are not their windows', and
// arrays that start between lines).  The
// source side of a lane's row is made again only in tiles where a lane's row
// changes.
//
// Bound by the issue of vector instructions, hence by their number per tile: 531
// at 3.9 cycles of a SIMD each.  The ones used most (v_perm_b32, v_dot4_u32_u8,
// v_mul_lo_u32, v_mad_u64_u32) take 4.1-4.2 alone, v_and_b32 and v_bitop3_b32
// 2.3, but in turns with v_perm_b32 3.9: a mixture gains little from its fast
// half (4.0 at the 4 wavefronts per SIMD that run here).
// Everything a row fixes is made with the row (positions as the target's axes
// meet them), places in a window are 32-bit scalars, and the addresses of the
// five stores are scalar bases and one offset: together 1409 -> 1299 us on the
// 96-layer GPT's build.
// ---------------------------------------------------------------------------
constexpr uint32_t kWindowsPerBlock = 4;

// A lane's row and column; `mul`: how often nd < 64 goes into up to 127.
struct cell {
    uint32_t i, j;
};
__device__ inline uint32_t row_multiplier(uint32_t nd) { return 65535u / nd + 1u; }
__device__ inline void wrap(cell &c, uint32_t nd, uint32_t mul) {
    if (nd >= kWave) {   // uniform; j < nd + 64
        const uint32_t over = c.j >= nd ? 1u : 0u;
        c.i += over;
        c.j -= over ? nd : 0u;
    } else {
        const uint32_t q = (c.j * mul) >> 16;
        c.i += q;
        c.j -= q * nd;
    }
}

// A value that is the same in every lane, in scalar registers.
__device__ inline uint64_t uniform(uint64_t x) {
    const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)x);
    const uint32_t hi = __builtin_amdgcn_readfirstlane((uint32_t)(x >> 32));
    return ((uint64_t)hi << 32) | lo;
}

// The source sides of 64 consecutive rows of an edge, kept in LDS by each
// wavefront: lane l makes row first + l, once for the 1024 entries of a window
// as a rule, and a lane reads its own row's when that changes (5 LDS reads
// against the 125 instructions of taps_make_source).
struct row_cache {
    uint4 w[kWave][5];
};
static_assert(sizeof(taps_source) <= sizeof(uint4) * 5, "a row's source side");

__device__ inline void fill_rows(row_cache &cache, const taps_source &P, uint32_t lane) {
    uint32_t w[20] = {};
    __builtin_memcpy(w, &P, sizeof P);
    // the wavefront's earlier reads come before these writes, its later ones after
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
#pragma unroll
    for (uint32_t k = 0; k < 5u; ++k)
        cache.w[lane][k] = uint4{w[4 * k], w[4 * k + 1], w[4 * k + 2], w[4 * k + 3]};
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

__device__ inline taps_source read_row(const row_cache &cache, uint32_t r) {
    uint32_t w[20];
#pragma unroll
    for (uint32_t k = 0; k < 5u; ++k) {
        const uint4 x = cache.w[r][k];
        w[4 * k] = x.x, w[4 * k + 1] = x.y, w[4 * k + 2] = x.z, w[4 * k + 3] = x.w;
    }
    taps_source P;
    __builtin_memcpy(&P, w, sizeof P);
    return P;
}

// The table by tops mask, into LDS (a whole workgroup).
template <uint32_t C>
__device__ inline void load_tops(const taps_windows &win, taps_top_row *tops, taps_b8 *low) {
    for (uint32_t x = threadIdx.x; x < 256u; x += blockDim.x) {
        tops[x] = win.tops[x];
        if (C > 2) low[x] = ((const taps_b8 *)(win.tops + 256))[x];
    }
    __syncthreads();
}

// Emit(E, at, lane, r): stores the entry at + lane of an edge with constants E
// from its candidates r.
template <uint32_t C, typename Emit>
__device__ inline void run_window(const taps_windows &win, const taps_packed *__restrict__ desc,
                                  const Emit &emit) {
    __shared__ taps_top_row tops[256];
    __shared__ taps_b8 low[C > 2 ? 256 : 1];
    __shared__ row_cache rows[kWindowsPerBlock];
    const taps_levels_model &m = win.model;
    load_tops<C>(win, tops, low);
    const uint32_t lane = threadIdx.x % kWave;
    const uint32_t wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
    const uint64_t w = (uint64_t)blockIdx.x * kWindowsPerBlock + wave;
    if (w >= win.n_windows) return;
    const uint64_t span = (uint64_t)win.tiles * kWave;
    const uint64_t begin = w * span;
    // places in the window, 32 bits each (a scalar compare; 64 bits take vector ones)
    const uint32_t size = (uint32_t)(win.total - begin < span ? win.total - begin : span);
    uint32_t e = win.window_edge[w];
    if (e == ~0u) return;   // crowded
    taps_edge_params E = win.params[e];
    taps_b8 in_tensor = taps_in_tensor(E.to, E.rank);
    uint64_t e_start = uniform(win.starts[e]), e_end = uniform(win.starts[e + 1u]);
    auto place = [&](uint64_t x) {   // of entry x, one past the window's for all behind it
        return x - begin > size ? size + 1u : (uint32_t)(x - begin);
    };
    uint32_t stop = place(e_end);
    uint64_t to_out = begin + uniform(E.out_offset) - e_start;
    uint32_t mul = row_multiplier(E.nd);
    const uint64_t local = begin - e_start;   // below ns * nd
    cell c;
    c.i = (uint32_t)(local / E.nd);
    c.j = (uint32_t)(local % E.nd) + lane;
    wrap(c, E.nd, mul);
    taps_source P = {};
    uint32_t row = ~0u;              // the row P holds
    uint32_t cached = ~0u - kWave;   // the cache holds rows cached .. cached + 63 of edge e
    taps_packed q = desc[E.dst_base + (c.i < E.ns ? c.j : 0u)];
    for (uint32_t v = 0; v < size; v += kWave) {
        const uint32_t tile_end = size - v < kWave ? size : v + kWave;
        // the next tile's target side, asked for a tile ahead (before this tile's
        // stores, which a later load would wait for)
        cell next = c;
        taps_packed next_q = q;
        if (stop > tile_end) {   // uniform
            next.j += kWave;
            wrap(next, E.nd, mul);
            next_q = desc[E.dst_base + (next.i < E.ns ? next.j : 0u)];
        }
        uint32_t first = 0;   // lanes below this are done
        for (;;) {            // uniform: one edge per pass
            const uint32_t last = (stop < tile_end ? stop : tile_end) - v;
            const bool mine = lane - first < last - first;
            if (__any(mine && c.i != row)) {
                if (__any(mine && c.i - cached >= kWave)) {
                    cached = __builtin_amdgcn_readlane(c.i, first);
                    const uint32_t r = cached + lane;
                    fill_rows(rows[wave],
                              taps_make_source<C>(desc[E.src_base + (r < E.ns ? r : cached)],
                                                  E.from, E.to, E.rank, m), lane);
                }
                // (an entry's row is within 63 of the first's, as every row has one at least)
                P = read_row(rows[wave], mine ? c.i - cached : 0u);
                row = mine ? c.i : ~0u;
            }
            // every lane, so that the branches on the node boundary stay uniform
            // (a lane without an entry computes one that it does not store)
            taps_three<C> r;
            taps_three_candidates<C>(P, q, in_tensor, m, tops, low, r);
            if (mine) emit(E, to_out + v, lane, r);
            if (stop >= tile_end && (stop > tile_end || tile_end == size)) break;
            // the next edge starts in this tile, or with the next one
            first = last;
            ++e;
            E = win.params[e];
            in_tensor = taps_in_tensor(E.to, E.rank);
            e_start = e_end;
            e_end = uniform(win.starts[e + 1u]);
            stop = place(e_end);
            to_out = begin + uniform(E.out_offset) - e_start;
            mul = row_multiplier(E.nd);
            row = ~0u;
            cached = ~0u - kWave;
            c.i = 0u;
            c.j = lane - first;   // lanes below `first` come to this edge with the next tile
            if (lane >= first) wrap(c, E.nd, mul);
            next = c;
            if (lane < first) next.i = 0u;
            next.j += kWave;
            if (first == tile_end - v) {
                // it starts with the next tile (first == 64): lane l there is its entry l
                wrap(next, E.nd, mul);
                next_q = desc[E.dst_base + (next.i < E.ns ? next.j : 0u)];
                break;
            }
            wrap(next, E.nd, mul);
            q = desc[E.dst_base + (lane >= first && c.i < E.ns ? c.j : 0u)];
            next_q = desc[E.dst_base + (next.i < E.ns ? next.j : 0u)];
        }
        c = next;
        q = next_q;
    }
}

// A crowded window: one wavefront per tile, a lane's edge, row and column its
// own.  Bound by latency: the chain from the starts over the edge's constants
// to the descriptors, and the candidates once.
template <uint32_t C, typename Emit>
__device__ inline void run_crowded(const taps_windows &win, const taps_packed *__restrict__ desc,
                                   const Emit &emit) {
    __shared__ taps_top_row tops[256];
    __shared__ taps_b8 low[C > 2 ? 256 : 1];
    load_tops<C>(win, tops, low);
    const uint32_t lane = threadIdx.x % kWave;
    const uint64_t k = (uint64_t)blockIdx.x * kWindowsPerBlock + threadIdx.x / kWave;
    if (k >= (uint64_t)win.n_crowded * win.tiles) return;
    const uint64_t tile = (uint64_t)win.crowded[k / win.tiles] * win.tiles + k % win.tiles;
    if (tile * kWave >= win.total) return;   // the last window may be shorter
    const uint64_t at = tile * kWave + lane, x = at < win.total ? at : win.total - 1u;
    const uint32_t e = wave_owner(win.starts, win.n_edges, x);
    const taps_edge_params E = win.params[e];
    const uint64_t local = x - win.starts[e];   // below ns * nd
    const uint32_t i = (uint32_t)(local / E.nd), j = (uint32_t)(local % E.nd);
    const taps_packed q = desc[E.dst_base + j];
    const taps_source P =
        taps_make_source<C>(desc[E.src_base + i], E.from, E.to, E.rank, win.model);
    taps_three<C> r;
    taps_three_candidates<C>(P, q, taps_in_tensor(E.to, E.rank), win.model, tops, low, r);
    if (at < win.total) emit(E, E.out_offset + local, 0u, r);
}

// Selection among the candidates under one bandwidth point's keys (ties go to
// the earlier candidate), scaled.  Narrow: 64-bit keys.
template <bool Narrow>
__device__ inline taps_entry_out select_entry(const taps_three<2> &r, const taps_keys &K,
                                              const taps_scaler &S) {
    auto fac = [&](uint32_t c) {
        return taps_fac{r.c[c].vol, r.c[c].in, r.c[c].link[0], r.c[c].ct};
    };
    uint32_t intra = r.c[0].in, inter = r.c[0].link[0], ct = r.c[0].ct, cand = 0u;
    if (Narrow) {
        uint64_t best = taps_key64(fac(0), K);
        const uint64_t k1 = taps_key64(fac(1), K), k2 = taps_key64(fac(2), K);
#pragma unroll
        for (uint32_t c = 1; c < 3u; ++c) {
            const uint64_t k = c == 1u ? k1 : k2;
            const bool less = k < best;
            best = less ? k : best;
            intra = less ? r.c[c].in : intra;
            inter = less ? r.c[c].link[0] : inter;
            ct = less ? r.c[c].ct : ct;
            cand = less ? c : cand;
        }
    } else {
        taps_fac best = fac(0);
#pragma unroll
        for (uint32_t c = 1; c < 3u; ++c)
            if (taps_less(fac(c), best, K)) {
                best = fac(c);
                cand = c;
            }
        intra = best.intra;
        inter = best.inter;
        ct = best.ct;
    }
    uint32_t vol = r.c[1].vol < r.c[0].vol ? r.c[1].vol : r.c[0].vol;
    vol = r.c[2].vol < vol ? r.c[2].vol : vol;
    taps_entry_out o;
    if (S.q) {   // uniform over the edge
        o.vol = (uint64_t)S.q * vol;
        o.intra = (uint64_t)S.q * intra;
        o.inter = (uint64_t)S.q * inter;
    } else {
        o.vol = taps_scale(S, vol);
        o.intra = taps_scale(S, intra);
        o.inter = taps_scale(S, inter);
    }
    o.t = (double)intra * S.a_intra + (double)inter * S.a_inter;
    o.meta = cand | r.coll | (ct << 12);
    return o;
}

// Narrow: both reduced bandwidths are below 2^32 (64-bit keys).
template <bool Narrow>
struct emit_one {
    const taps_keys &K;
    const taps_table &out;
    __device__ void operator()(const taps_edge_params &E, uint64_t at, uint32_t lane,
                               const taps_three<2> &r) const {
        const taps_entry_out o = select_entry<Narrow>(r, K, E.scale);
        store_entry<false>(out, at, lane, o, o.meta);
    }
};

template <bool Narrow>
__global__ __launch_bounds__(256) void k_edge_costs(taps_windows win,
                                                    const taps_packed *__restrict__ desc,
                                                    taps_launch lp, taps_table out) {
    const taps_keys K = {lp.b_inter_red, lp.b_intra_red, Narrow};
    run_window<2>(win, desc, emit_one<Narrow>{K, out});
}

template <bool Narrow>
__global__ __launch_bounds__(256) void k_edge_costs_crowded(taps_windows win,
                                                            const taps_packed *__restrict__ desc,
                                                            taps_launch lp, taps_table out) {
    const taps_keys K = {lp.b_inter_red, lp.b_intra_red, Narrow};
    run_crowded<2>(win, desc, emit_one<Narrow>{K, out});
}

// Several bandwidth points: the candidates of each entry are costed once and
// selected, scaled and stored once per point.  Bound by the stores, which spread
// over five arrays per point (window lengths by points: TAPS_WINDOW_SWEEP).
template <bool Narrow>
struct emit_sweep {
    const taps_sweep &sw;
    __device__ void operator()(const taps_edge_params &E, uint64_t at, uint32_t lane,
                               const taps_three<2> &r) const {
        for (uint32_t k = 0; k < sw.count; ++k) {
            // Narrow: 64-bit keys at every point
            const taps_keys K = {sw.b_inter_red[k], sw.b_intra_red[k], Narrow || sw.narrow[k] != 0};
            const taps_scaler S =
                taps_make_scaler(E.scale.tbytes, sw.inv_n_bintra[k], sw.inv_n_binter[k]);
            const taps_entry_out o = Narrow || K.narrow ? select_entry<true>(r, K, S)
                                                        : select_entry<false>(r, K, S);
            store_entry<true>(sw.out[k], at, lane, o, o.meta);
        }
    }
};

template <bool Narrow>
__global__ __launch_bounds__(256) void k_edge_costs_sweep(taps_windows win,
                                                          const taps_packed *__restrict__ desc,
                                                          taps_sweep sw) {
    run_window<2>(win, desc, emit_sweep<Narrow>{sw});
}

template <bool Narrow>
__global__ __launch_bounds__(256) void k_edge_costs_sweep_crowded(
    taps_windows win, const taps_packed *__restrict__ desc, taps_sweep sw) {
    run_crowded<2>(win, desc, emit_sweep<Narrow>{sw});
}

// Link-class hierarchies: each entry selected by the exact key over the classes
// of H and scaled.  C: the hierarchy's number of classes.
template <uint32_t C>
__device__ inline taps_entry_out select_entry_h(const taps_three<C> &r, const taps_hier &H,
                                                const taps_scaler &S) {
    // AllToAlls inside a node at their own bandwidth, if it is set
    const uint32_t own = H.a2a_own ? r.a2a_in : 0u;
    auto key = [&](uint32_t c) {
        uint64_t k = (uint64_t)(r.c[c].in - (c ? 0u : own)) * H.w[0];
#pragma unroll
        for (uint32_t x = 1; x < C; ++x) k += (uint64_t)r.c[c].link[x - 1u] * H.w[x];
        return c ? k : k + (uint64_t)own * H.w_a2a;
    };
    const uint64_t k0 = key(0), k1 = key(1), k2 = key(2);
    const bool one = k1 < k0, two = k2 < (one ? k1 : k0);
    auto pick = [&](uint32_t a, uint32_t b, uint32_t c) { return two ? c : one ? b : a; };
    taps_cost_c<C> best;
    best.in = pick(r.c[0].in, r.c[1].in, r.c[2].in);
    best.ct = pick(r.c[0].ct, r.c[1].ct, r.c[2].ct);
#pragma unroll
    for (uint32_t x = 0; x + 1u < C; ++x)
        best.link[x] = pick(r.c[0].link[x], r.c[1].link[x], r.c[2].link[x]);
    best.vol = r.c[1].vol < r.c[0].vol ? r.c[1].vol : r.c[0].vol;   // the smallest of all
    best.vol = r.c[2].vol < best.vol ? r.c[2].vol : best.vol;
    const uint32_t cand = pick(0u, 1u, 2u), xa = pick(own, 0u, 0u);
    uint32_t links = 0;   // below 2^29: 8 axes, 2^16 units, 2^7 groups and 3 classes
    const double unit = (double)S.tbytes * (1.0 / 256.0);
    taps_entry_out o;
    o.t = (double)(best.in - xa) * (unit * H.inv_n_bw[0]);
#pragma unroll
    for (uint32_t x = 1; x < C; ++x) {
        links += best.link[x - 1u];
        o.t += (double)best.link[x - 1u] * (unit * H.inv_n_bw[x]);
    }
    o.t += (double)xa * (unit * H.inv_n_bw_a2a);
    if (S.q) {   // uniform over the edge
        o.vol = (uint64_t)S.q * best.vol;
        o.intra = (uint64_t)S.q * best.in;
        o.inter = (uint64_t)S.q * links;
    } else {
        o.vol = taps_scale(S, best.vol);
        o.intra = taps_scale(S, best.in);
        o.inter = taps_scale(S, links);
    }
    o.meta = cand | r.coll | (best.ct << 12);
    return o;
}

template <uint32_t C>
struct emit_classes {
    const taps_hier &H;
    const taps_table &out;
    __device__ void operator()(const taps_edge_params &E, uint64_t at, uint32_t lane,
                               const taps_three<C> &r) const {
        const taps_entry_out o = select_entry_h<C>(r, H, E.scale);
        store_entry<false>(out, at, lane, o, o.meta);
    }
};

// At least 4 wavefronts per SIMD: three classes take 140 registers without the
// bound (3 wavefronts: 2220 us on the 96-layer GPT's build against 2180).
template <uint32_t C>
__global__ __launch_bounds__(256, 4) void k_edge_costs_h(taps_windows win,
                                                      const taps_packed *__restrict__ desc,
                                                      taps_hier H, taps_table out) {
    run_window<C>(win, desc, emit_classes<C>{H, out});
}

template <uint32_t C>
__global__ __launch_bounds__(256) void k_edge_costs_h_crowded(taps_windows win,
                                                              const taps_packed *__restrict__ desc,
                                                              taps_hier H, taps_table out) {
    run_crowded<C>(win, desc, emit_classes<C>{H, out});
}

__global__ __launch_bounds__(256) void k_node_costs_h(const taps_op *__restrict__ ops,
                                                      uint32_t n_ops,
                                                      const uint64_t *__restrict__ offsets,
                                                      const taps_strategy *__restrict__ strategies,
                                                      uint64_t total, uint32_t n, taps_hier H,
                                                      taps_table out) {
    const uint64_t idx = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const uint64_t x = idx < total ? idx : total - 1u;
    const taps_op *op = ops + wave_owner(offsets, n_ops, x);
    taps_acch c = {0, 0, 0, 0, 0, 0, 0, 0};
    strategy_tensors(op, strategies[x], n, [&](uint32_t missing, uint64_t bytes) {
        taps_allreduce_h(c, missing, bytes, H);
    });
    if (idx >= total) return;
    out.t[idx] = (double)c.x0 * H.inv_n_bw[0] + (double)c.x1 * H.inv_n_bw[1] +
                 (double)c.x2 * H.inv_n_bw[2] + (double)c.x3 * H.inv_n_bw[3];
    out.vol[idx] = c.vol;
    out.intra[idx] = c.x0;
    out.inter[idx] = c.x1 + c.x2 + c.x3;
    out.meta[idx] = (c.n_coll << 2) | (c.n_inter << 7) | (c.sum_ct << 12);
}

// Shared tables: each task holds `count` (<= TAPS_COPY_CHUNK) consecutive
// entries of a computed table, staged once in LDS with the `extra` entries
// after them and stored into every table that shares it; blockIdx.y picks the
// array.  The tables start at arbitrary entries, so into each destination a
// task stores the whole 128-byte lines that its entries end: from the first
// line boundary at or after them to the one at or after their end (LDS absorbs
// the difference in alignment), with single entries only at a table's ends.
// Bound by the stores: the 96-layer GPT's 3.5 GB take 688 us when each task
// stores just its entries, in cached stores, which leaves a part of a line at
// either end of each to merge; 640 us so, 5.5 TB/s (a plain store of five
// arrays side by side: 570 - 640 us).
constexpr uint32_t kCopyThreads = 512;

template <typename T>
__device__ inline void copy_range(T *base, const taps_copy_task &c,
                                  const uint64_t *__restrict__ dst_list, T *stage) {
    constexpr uint32_t kV = 16 / sizeof(T);      // entries per 16-byte store
    constexpr uint32_t kLine = 128 / sizeof(T);  // and per line
    static_assert(kLine <= TAPS_COPY_EXTRA && TAPS_COPY_CHUNK % kLine == 0, "whole lines per task");
    typedef uint32_t quad __attribute__((ext_vector_type(4)));
    const T *s = base + c.src;
    const uint32_t have = c.count + c.extra;
    for (uint32_t x = threadIdx.x; x < have; x += blockDim.x) stage[x] = s[x];
    __syncthreads();
    for (uint32_t k = 0; k < c.n_dst; ++k) {
        T *d = base + dst_list[c.dst_begin + k] + c.offset;
        const uint32_t mis = (uint32_t)(((uintptr_t)d & 127u) / sizeof(T));
        const uint32_t skip = mis ? kLine - mis : 0u;   // entries before the first line boundary
        const uint32_t lo = skip < have ? skip : have;
        const uint32_t hi = c.count + skip < have ? c.count + skip : have;
        const uint32_t n_vec = (hi - lo) / kV, tail = lo + n_vec * kV;
        if (c.offset == 0 && threadIdx.x < lo) d[threadIdx.x] = stage[threadIdx.x];
        for (uint32_t v = threadIdx.x; v < n_vec; v += blockDim.x) {
            quad val;
            __builtin_memcpy(&val, stage + lo + v * kV, 16);
            __builtin_nontemporal_store(val, (quad *)(d + lo) + v);
        }
        if (tail + threadIdx.x < hi) d[tail + threadIdx.x] = stage[tail + threadIdx.x];
    }
}

// An upload without the copy engine: the plan is read straight from
// fine-grained pinned host memory, 16 bytes per thread and step, so the
// build's kernels follow it on the same queue with no hand-over.
__global__ __launch_bounds__(256) void k_pull(const uint4 *__restrict__ src,
                                              uint4 *__restrict__ dst, uint32_t n16) {
    for (uint32_t k = blockIdx.x * 256u + threadIdx.x; k < n16; k += gridDim.x * 256u)
        dst[k] = src[k];
}

__global__ __launch_bounds__(kCopyThreads) void k_copy_tables(const taps_copy_task *__restrict__ tasks,
                                                     const uint64_t *__restrict__ dst_list,
                                                     taps_table out) {
    __shared__ uint64_t stage[TAPS_COPY_CHUNK + TAPS_COPY_EXTRA];
    const taps_copy_task c = tasks[blockIdx.x];
    switch (blockIdx.y) {
    case 0: copy_range(out.t, c, dst_list, (double *)stage); break;
    case 1: copy_range(out.vol, c, dst_list, stage); break;
    case 2: copy_range(out.intra, c, dst_list, stage); break;
    case 3: copy_range(out.inter, c, dst_list, stage); break;
    default: copy_range(out.meta, c, dst_list, (uint32_t *)stage); break;
    }
}

// One workgroup per pair of strategy ranges; flags[p] = any entry differs.
__global__ __launch_bounds__(256) void k_same_ranges(const taps_strategy *__restrict__ s,
                                                     const uint64_t *__restrict__ pairs,
                                                     uint32_t *__restrict__ flags) {
    const uint64_t a = pairs[3 * blockIdx.x], b = pairs[3 * blockIdx.x + 1];
    const uint64_t count = pairs[3 * blockIdx.x + 2];
    int differ = 0;
    for (uint64_t k = threadIdx.x; k < count; k += blockDim.x) {
        const taps_strategy x = s[a + k], y = s[b + k];
        for (uint32_t q = 0; q < TAPS_MAX_AXES; ++q)
            differ |= (x.log2_deg[q] != y.log2_deg[q]) | (x.pos[q] != y.pos[q]);
    }
    differ = __syncthreads_or(differ);
    if (threadIdx.x == 0) flags[blockIdx.x] = differ ? 1u : 0u;
}

inline uint32_t blocks_for(uint64_t n, uint32_t per) { return (uint32_t)((n + per - 1) / per); }

}  // namespace

hipError_t taps_launch_node_costs(const taps_op *ops, uint32_t n_ops, const uint64_t *offsets,
                                  const taps_strategy *strategies, uint64_t total,
                                  const taps_launch &lp, taps_table out, hipStream_t stream) {
    if (total == 0) return hipSuccess;
    hipLaunchKernelGGL(k_node_costs, dim3(blocks_for(total, 256)), dim3(256), 0, stream, ops,
                       n_ops, offsets, strategies, total, lp, out);
    return hipGetLastError();
}

hipError_t taps_launch_memory_costs(const taps_op *ops, uint32_t n_ops, const uint64_t *offsets,
                                   const taps_strategy *s, uint64_t total, uint64_t *memory,
                                   hipStream_t stream) {
    if (total == 0) return hipSuccess;
    hipLaunchKernelGGL(k_memory_costs, dim3(blocks_for(total, 256)), dim3(256), 0, stream, ops,
                       n_ops, offsets, s, total, memory);
    return hipGetLastError();
}

hipError_t taps_launch_edge_front(const taps_strategy *strategies, uint64_t total,
                                  taps_packed *desc, const taps_plan_args &pa,
                                  const taps_launch &lp, hipStream_t stream) {
    if (pa.n_edges == 0) return hipSuccess;
    const uint32_t describe_blocks = blocks_for(total, 256);
    const uint32_t setup_blocks = blocks_for(pa.n_edges, 256);
    const uint32_t map_blocks = blocks_for(pa.n_windows, 256);
    hipLaunchKernelGGL(k_edge_front, dim3(describe_blocks + setup_blocks + map_blocks), dim3(256),
                       0, stream, strategies, total, describe_blocks, desc, pa, lp, setup_blocks);
    return hipGetLastError();
}

namespace {

// The window kernel over the windows, unless all are crowded, then the other one over the
// tiles of those.
template <typename Kernel, typename... Args>
hipError_t launch_windows(const taps_windows &win, hipStream_t stream, Kernel windows,
                          Kernel crowded, Args... args) {
    const dim3 block(kWave * kWindowsPerBlock);
    if (win.n_windows > win.n_crowded)
        hipLaunchKernelGGL(windows, dim3(blocks_for(win.n_windows, kWindowsPerBlock)), block, 0,
                           stream, win, args...);
    if (win.n_crowded)
        hipLaunchKernelGGL(crowded,
                           dim3(blocks_for((uint64_t)win.n_crowded * win.tiles, kWindowsPerBlock)),
                           block, 0, stream, win, args...);
    return hipGetLastError();
}

}  // namespace

hipError_t taps_launch_edge_costs(const taps_windows &win, const taps_packed *desc,
                                  const taps_launch &lp, taps_table out, hipStream_t stream) {
    return lp.narrow ? launch_windows(win, stream, k_edge_costs<true>, k_edge_costs_crowded<true>,
                                      desc, lp, out)
                     : launch_windows(win, stream, k_edge_costs<false>, k_edge_costs_crowded<false>,
                                      desc, lp, out);
}

hipError_t taps_launch_edge_costs_sweep(const taps_windows &win, const taps_packed *desc,
                                        const taps_sweep &sw, hipStream_t stream) {
    bool narrow = true;
    for (uint32_t k = 0; k < sw.count; ++k) narrow = narrow && sw.narrow[k] != 0;
    return narrow ? launch_windows(win, stream, k_edge_costs_sweep<true>,
                                   k_edge_costs_sweep_crowded<true>, desc, sw)
                  : launch_windows(win, stream, k_edge_costs_sweep<false>,
                                   k_edge_costs_sweep_crowded<false>, desc, sw);
}

hipError_t taps_launch_build_strategies(const taps_op *ops, const taps_build_chunk *chunks,
                                        uint32_t n_chunks, uint32_t allowed_cuts,
                                        const taps_launch &lp, taps_strategy *out,
                                        taps_packed *desc, taps_table node, hipStream_t stream) {
    if (n_chunks == 0) return hipSuccess;
    hipLaunchKernelGGL(k_build_strategies, dim3(n_chunks), dim3(kBuildThreads), 0, stream, ops,
                       chunks, allowed_cuts, lp, out, desc, node);
    return hipGetLastError();
}

hipError_t taps_launch_build_front(const taps_build_chunk *chunks, uint32_t n_chunks,
                                   uint32_t allowed_cuts, const taps_launch &lp, taps_strategy *out,
                                   taps_packed *desc, taps_table node, const taps_plan_args &pa,
                                   hipStream_t stream) {
    const uint32_t setup_blocks = blocks_for(pa.n_edges, 256);
    const uint32_t blocks = n_chunks + setup_blocks + blocks_for(pa.n_windows, 256);
    if (blocks == 0) return hipSuccess;
    hipLaunchKernelGGL(k_build_front, dim3(blocks), dim3(kBuildThreads), 0, stream, pa.ops, chunks,
                       n_chunks, allowed_cuts, lp, out, desc, node, pa, setup_blocks);
    return hipGetLastError();
}

hipError_t taps_launch_edge_costs_h(const taps_windows &win, const taps_packed *desc,
                                    const taps_hier &H, taps_table out, hipStream_t stream) {
    auto launch = [&](auto windows, auto crowded) {
        return launch_windows(win, stream, windows, crowded, desc, H, out);
    };
    switch (H.n_classes) {
    case 1: return launch(k_edge_costs_h<1>, k_edge_costs_h_crowded<1>);
    case 2: return launch(k_edge_costs_h<2>, k_edge_costs_h_crowded<2>);
    case 3: return launch(k_edge_costs_h<3>, k_edge_costs_h_crowded<3>);
    default: return launch(k_edge_costs_h<4>, k_edge_costs_h_crowded<4>);
    }
}

hipError_t taps_launch_node_costs_h(const taps_op *ops, uint32_t n_ops, const uint64_t *offsets,
                                    const taps_strategy *strategies, uint64_t total, uint32_t n,
                                    const taps_hier &H, taps_table out, hipStream_t stream) {
    if (total == 0) return hipSuccess;
    hipLaunchKernelGGL(k_node_costs_h, dim3(blocks_for(total, 256)), dim3(256), 0, stream, ops,
                       n_ops, offsets, strategies, total, n, H, out);
    return hipGetLastError();
}

hipError_t taps_launch_pull(const void *src, void *dst, uint64_t bytes, hipStream_t stream) {
    const uint64_t n16 = bytes / 16;
    if (n16 == 0) return hipSuccess;
    const uint64_t blocks = (n16 + 255) / 256 < 256 ? (n16 + 255) / 256 : 256;
    hipLaunchKernelGGL(k_pull, dim3((uint32_t)blocks), dim3(256), 0, stream, (const uint4 *)src,
                       (uint4 *)dst, (uint32_t)n16);
    return hipGetLastError();
}

hipError_t taps_launch_copy_tables(const taps_copy_task *tasks, uint32_t n_tasks,
                                   const uint64_t *dst_list, taps_table out, hipStream_t stream) {
    if (n_tasks == 0) return hipSuccess;
    hipLaunchKernelGGL(k_copy_tables, dim3(n_tasks, 5), dim3(kCopyThreads), 0, stream, tasks, dst_list,
                       out);
    return hipGetLastError();
}

hipError_t taps_launch_same_ranges(const taps_strategy *strategies, const uint64_t *pairs,
                                   uint32_t n_pairs, uint32_t *flags, hipStream_t stream) {
    if (n_pairs == 0) return hipSuccess;
    hipLaunchKernelGGL(k_same_ranges, dim3(n_pairs), dim3(256), 0, stream, strategies, pairs,
                       flags);
    return hipGetLastError();
}

// taps_internal.h -- launch interface between the C ABI and the kernels.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "taps.h"
#include "taps_device.h"
#include "taps_entry.h"

// Uniform parameters of a table launch.
struct taps_launch {
    uint32_t n;             // log2 N
    uint32_t lam;           // log2 L
    uint64_t b_inter_red;   // B_inter / gcd(B_intra, B_inter)
    uint64_t b_intra_red;   // B_intra / gcd(B_intra, B_inter)
    double inv_n_bintra;    // 1 / (N B_intra)
    double inv_n_binter;    // 1 / (N B_inter)
    uint32_t narrow;        // both reduced bandwidths below 2^32
};

// Per-edge constants of the edge-table kernel.
struct taps_edge_params {
    uint64_t out_offset;   // first entry of the edge's table
    taps_scaler scale;     // tbytes and the per-unit seconds of the edge tensor
    uint32_t src_base;     // first strategy of the source side (producer; consumer for
    uint32_t dst_base;     //   the backward tables) and of the target side
    uint32_t ns, nd;       // their strategy counts
    uint32_t rank, pad;
    taps_side from, to;    // tensor dimensions and op axes of the two sides
};

// Shared tables: entries [src, src + count) of every array are copied to
// [dst[k] + offset, dst[k] + offset + count) for the n_dst table starts
// dst[k] = dst_list[dst_begin + k].
struct taps_copy_task {
    uint64_t src, offset;
    uint32_t count, dst_begin, n_dst;
    uint32_t extra;   // entries of the table after these, at most TAPS_COPY_EXTRA
};
#define TAPS_COPY_CHUNK 2048    // entries per copy task (4 per thread of 512; 1024 and 4096 are slower)
#define TAPS_COPY_DSTS 6        // tables one copy task writes (4, 8 and 12 measure within 1 %)
#define TAPS_COPY_EXTRA 32u     // entries of a 128-byte line, of the narrowest array

// The edge kernels run over windows: window w is the 64 T entries
// [64 T w, 64 T (w + 1)) of the computed tables laid end to end (aligned, so
// that tiles are whole lines of the output, unless tables are shared or the
// arrays start between lines), taken by one wavefront 64 at a time.
#define TAPS_TILE_COLS 64
// Entries of one call: its tiles, and so its windows and blocks, stay below 2^31.
#define TAPS_MAX_ENTRIES (0x7FFFFFFFull * TAPS_TILE_COLS)
// T: a window's set-up (its place, the row cache, the LDS table) is paid once
// per T tiles, and the launch's end leaves wavefronts idle for up to a window,
// so T grows with the square root of the tiles, up to TAPS_WINDOW_LONG, which
// launches of at least taps_set_long_segments_min() such windows take.
// Measured (us, T = 1 / 2 / 4 / 8 / 16 / 32): 1.5 M tiles 2233 / 1858 / 1680 /
// 1600 / 1561 / 1565, 145 k tiles 215 / 183 / 169 / 165 / 170 / 197, 64 k tiles
// 120 / 106 / 101 / 102 / 105 / 119, 16 k tiles 99 / 95 / 94 / 96 / 105 / 131
// (whole builds).  Several bandwidth points are bound by their stores, into five
// arrays per point.  The fewer the points, the longer the windows may be (1.5 M
// tiles, us, T = 1 / 2 / 3 / 4 / 8, cached stores, then non-temporal ones):
//   2 points  2393 / 1984 / 1806 / 1710 / 1567,  2069 / 1759 / 1612 / 1576 / 1508
//   3 points  2718 / 2208 / 1954 / 1877 / 1922,  2200 / 1915 / 1946 / 1989 / 2002
//   4 points  2991 / 2403 / 2643 / 2664 / 2651,  2564 / 2630 / 2700 / 2693 / 2673
//   5 points  3308 / 3260 / 3295 / 3291 / 3275,  3447 / 3265 / 3313 / 3334 / 3327
//   8 points  5482 / 5356 / 5380 / 5343 / 5368,  5518 / 5434 / 5434 / 5461 / 5486
// and alike on 215 k tiles (2 points 405 / 345 / 320 / 309 / 298, 4 points 471 /
// 405 / 451 / 453 / 465).  Why four points have their best at two tiles is not known.
#define TAPS_WINDOW_LONG 16
#define TAPS_WINDOW_SWEEP(points) ((points) == 2 ? 8 : (points) == 3 ? 4 : 2)
#define TAPS_LONG_SEGS_MIN 32768
// A wavefront takes the tables that meet in its window one after the other,
// about 1.6 us each.  A window that holds entries of more than TAPS_CROWDED(T)
// tables goes to the k_*_crowded kernels instead, a lane its own table (calls,
// us, as windows / crowded: 255 tables of one entry 129 / 23, 1,000 tables of
// 3,969 entries and of one in turns of a hundred 206 / 58, 199 of 9 entries, eight
// to a tile and not crowded, 31).
#define TAPS_CROWDED(tiles) (2u * (tiles) + 6u)

hipError_t taps_launch_node_costs(const taps_op *ops, uint32_t n_ops, const uint64_t *offsets,
                                  const taps_strategy *strategies, uint64_t total,
                                  const taps_launch &lp, taps_table out, hipStream_t stream);
// The edge plan of a launch (device arrays): the constants of the n_edges
// computed edges (edge computed[k], or k without that list) into params, and
// the edge that each window starts in (~0: a crowded one).  starts: n_edges + 1
// first entries of the computed tables laid end to end; window: entries per
// window; reverse: the backward tables (source side = the consumer's input map).
struct taps_plan_args {
    const taps_op *ops;
    const taps_edge *edges;
    const uint64_t *op_offsets;
    const uint64_t *edge_offsets;
    const uint32_t *computed;
    const uint64_t *starts;
    taps_edge_params *params;
    uint32_t *window_edge;
    taps_top_row *tops;          // TAPS_TOPS_BYTES: 256 rows, then their `low` bytes
    uint64_t n_windows;
    uint32_t n_edges, window, reverse;
    uint32_t crowded;            // tables from which on a window is (0: no window is)
    taps_levels_model model;
};
#define TAPS_TOPS_BYTES ((sizeof(taps_top_row) + sizeof(taps_b8)) * 256)
// The plan and the `total` strategies' descriptors.
hipError_t taps_launch_edge_front(const taps_strategy *strategies, uint64_t total,
                                  taps_packed *desc, const taps_plan_args &pa,
                                  const taps_launch &lp, hipStream_t stream);
// What the edge kernels run over (the plan's results).
struct taps_windows {
    const taps_edge_params *params;
    const uint64_t *starts;
    const uint32_t *window_edge;
    const taps_top_row *tops;
    const uint32_t *crowded;     // the crowded windows
    uint64_t n_windows, total;   // total: computed entries
    uint32_t tiles;              // tiles per window
    uint32_t n_edges, n_crowded, pad;
    taps_levels_model model;
};
hipError_t taps_launch_edge_costs(const taps_windows &win, const taps_packed *desc,
                                  const taps_launch &lp, taps_table out, hipStream_t stream);
hipError_t taps_launch_memory_costs(const taps_op *ops, uint32_t n_ops, const uint64_t *offsets,
                                   const taps_strategy *s, uint64_t total, uint64_t *memory,
                                   hipStream_t stream);
// Bandwidth points of one sweep: the keys and per-unit seconds of each, and
// the table each writes.
struct taps_sweep {
    uint32_t count;
    uint32_t narrow[TAPS_MAX_SWEEP];
    uint64_t b_inter_red[TAPS_MAX_SWEEP];
    uint64_t b_intra_red[TAPS_MAX_SWEEP];
    double inv_n_bintra[TAPS_MAX_SWEEP];
    double inv_n_binter[TAPS_MAX_SWEEP];
    taps_table out[TAPS_MAX_SWEEP];
};
hipError_t taps_launch_edge_costs_sweep(const taps_windows &win, const taps_packed *desc,
                                        const taps_sweep &sw, hipStream_t stream);
// One workgroup of k_build_strategies: candidate ranks [first, first +
// TAPS_BUILD_CHUNK) of operator `op`, of which `count` pass the filter; they
// are strategies base, base + 1, ... in rank order.
#define TAPS_BUILD_CHUNK 256
struct taps_build_chunk {
    uint64_t base;
    uint32_t op, first, count, pad;
};
// Strategies of every operator in one launch (one workgroup per chunk of
// candidate ranks that holds a strategy), with their descriptors and node
// records unless desc / node.t are NULL.
hipError_t taps_launch_build_strategies(const taps_op *ops, const taps_build_chunk *chunks,
                                        uint32_t n_chunks, uint32_t allowed_cuts,
                                        const taps_launch &lp, taps_strategy *out,
                                        taps_packed *desc, taps_table node, hipStream_t stream);
// taps_launch_build_strategies and the edge plan as one launch (the
// plan needs only the host-counted strategy offsets).
hipError_t taps_launch_build_front(const taps_build_chunk *chunks, uint32_t n_chunks,
                                   uint32_t allowed_cuts, const taps_launch &lp, taps_strategy *out,
                                   taps_packed *desc, taps_table node, const taps_plan_args &pa,
                                   hipStream_t stream);
// Link-class hierarchies: the edge and node tables under the classes of H.
hipError_t taps_launch_edge_costs_h(const taps_windows &win, const taps_packed *desc,
                                    const taps_hier &H, taps_table out, hipStream_t stream);
hipError_t taps_launch_node_costs_h(const taps_op *ops, uint32_t n_ops, const uint64_t *offsets,
                                    const taps_strategy *strategies, uint64_t total, uint32_t n,
                                    const taps_hier &H, taps_table out, hipStream_t stream);
// Copies `bytes` (a multiple of 16, below 2^36) from src, fine-grained pinned
// host memory mapped for the device, to device memory at dst.
hipError_t taps_launch_pull(const void *src, void *dst, uint64_t bytes, hipStream_t stream);
hipError_t taps_launch_copy_tables(const taps_copy_task *tasks, uint32_t n_tasks,
                                   const uint64_t *dst_list, taps_table out, hipStream_t stream);
// For each pair p: flags[p] = 0 if strategies[first_a .. +count) equals
// strategies[first_b .. +count), else 1.  pairs: (first_a, first_b, count) as
// three uint64 each.
hipError_t taps_launch_same_ranges(const taps_strategy *strategies, const uint64_t *pairs,
                                   uint32_t n_pairs, uint32_t *flags, hipStream_t stream);

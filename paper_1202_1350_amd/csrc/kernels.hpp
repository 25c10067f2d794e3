// kernels.hpp -- launchers of the verifier's kernels (kernels.hip).
//
// Every launcher enqueues on `st` and returns the launch status; none of
// them synchronises.  Device pointers only.  Reductions write one row of
// partial sums per workgroup; the host adds the rows.
#pragma once
#include <algorithm>

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace gkr {

typedef uint64_t u64;
typedef uint32_t u32;
typedef uint8_t u8;

// Layer gate mix: the kernels drop the type array when a layer is uniform.
enum Kind { KIND_ADD = 0, KIND_MUL = 1, KIND_MIXED = 2 };

// Workgroup size of every reduction kernel, and the cap on workgroups per
// launch (8 per CU on 256 CUs).
constexpr int BLOCK = 256;
constexpr int MAX_BLOCKS = 2048;

// Workgroups for n work items at `per` items per thread.
inline int blocks_for(u64 n, u64 per = 1) {
    u64 t = (n + per - 1) / per;
    u64 b = (t + BLOCK - 1) / BLOCK;
    if (b < 1) b = 1;
    if (b > (u64)MAX_BLOCKS) b = MAX_BLOCKS;
    return (int)b;
}

// ---- verifier (a10) ---------------------------------------------------------
// A layer whose add~ and mult~ at (a*, b*, c*) take a pass over its gates.
// Its eq half tables (entry x of a point's halves: chi_x = lo[x mod 2^L]
// hi[x >> L]) sit one after another from tab: a* (2^La, 2^{s-La}), b* and c*
// (2^Lb, 2^{sp-Lb} each).  One launch forms the tables of every such layer and
// one passes over all their gates; workgroups [eq0, next eq0) and [block0,
// next block0) of them belong to the layer.
struct WireLayer {
    u32 kind, S, s, sp, La, Lb;
    u32 pt;            // a*, b*, c* in the points
    u32 eq0, block0;
    u32 pad;
    const u8 *type;
    const u32 *in1, *in2;
    u64 *tab;
};
u64 wire_table_words(u32 s, u32 sp);
u32 wire_eq_blocks(u32 s, u32 sp);
// Workgroups of a layer of S gates: two gates a thread before another starts,
// a share of WIRE_BLOCKS when the launch's layers want more in all
// (blocks_all, the sum of what they want), at least one.
constexpr u64 WIRE_BLOCKS = 2048;
inline u64 wire_blocks_wanted(u32 S) { return std::max<u64>(1, ((u64)S + 2 * BLOCK - 1) / (2 * BLOCK)); }
u32 wire_gate_blocks(u32 S, u64 blocks_all);
// L: n descriptors on the device, then one whose eq0 and block0 are the totals.
// out[2b], out[2b+1]: workgroup b's sums over ADD and MUL gates.
hipError_t launch_wiring(hipStream_t st, const WireLayer *L, u32 n, u32 eq_blocks, u32 gate_blocks, const u64 *pts,
                         u64 *out);
// Multilinear extension of T (n values, u64 or u32) at the point pt (s
// coordinates, the others 0): partial sums of nb workgroups, stored, or added
// to the sums already there (accumulate).  A chunk of a longer table starts
// at x0, a multiple of 2^12.  *bad = 1 if a u64 value is not below p.
struct MlePoint {
    u32 s;
    u64 r[36];
};
constexpr int MLE_BLOCKS = 2048;
int mle_blocks(u64 n);
hipError_t launch_mle(hipStream_t st, u64 n, const u64 *T64, const u32 *T32, const MlePoint &pt, u64 x0, u64 *partials,
                      int nb, int accumulate, u32 *bad);
// ---- field check ----------------------------------------------------------
hipError_t launch_field_op(hipStream_t st, int op, const u64 *a, const u64 *b, u64 *out, u64 n);

}  // namespace gkr

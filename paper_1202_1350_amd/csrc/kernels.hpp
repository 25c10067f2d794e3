// kernels.hpp -- launchers of the GKR / sum-check kernels (kernels.hip).
//
// Every launcher enqueues on `st` and returns the launch status; none of
// them synchronises.  Device pointers only.  Reductions write one row of
// partial sums per workgroup into `partials`; a *_final kernel (one
// workgroup) folds the rows, writes the round message into the transcript,
// and only then draws the next challenge.
#pragma once
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

// ---- proof bookkeeping ----------------------------------------------------
// eq half tables of a point pt[0..s): lo[x] = chi_x(pt[0..L)) for x < 2^L,
// hi[y] = chi_y(pt[L..s)) for y < 2^{s-L}; chi_x(pt) = lo[x & (2^L-1)] * hi[x >> L].
hipError_t launch_eq_halves(hipStream_t st, const u64 *pt, u32 s, u32 L, u64 *lo, u64 *hi);

// ---- verifier (a10) ---------------------------------------------------------
// Per workgroup (add~, mult~) partial sums at (a*, b*, c*) from half tables.
struct WiringArgs {
    int kind;
    u32 S;
    const u8 *type;
    const u32 *in1, *in2;
    const u64 *alo, *ahi;
    u32 La;
    const u64 *blo, *bhi;
    u32 Lb;
    const u64 *clo, *chi;
    u32 Lc;
    u64 *partials;
};
hipError_t launch_wiring(hipStream_t st, const WiringArgs &a, int *nblocks);
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
// Fold nparts rows of K partial sums into out[0..K).
hipError_t launch_reduce_rows(hipStream_t st, int nparts, int K, const u64 *partials, u64 *out);

// ---- field check ----------------------------------------------------------
hipError_t launch_field_op(hipStream_t st, int op, const u64 *a, const u64 *b, u64 *out, u64 n);

}  // namespace gkr

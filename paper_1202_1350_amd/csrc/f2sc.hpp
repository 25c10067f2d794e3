// f2sc.hpp -- launchers of the interactive F2 sum-check's prover (f2sc.hip).
//
// A proof over n = 2^l counts is f2sc_passes(l) grid passes of three rounds
// each, then one tail.  Pass p sums the Gram matrix of level 3p's octs into
// rows of F2SC_ROW words (one a workgroup, f2sc_rows(l, p) of them) and, for
// p >= 1, stores the level; the launch after it draws the three challenges
// and forms its messages.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace gkr {

typedef uint64_t u64;
typedef uint32_t u32;

constexpr int F2SC_ROW = 40;        // words of a row: five slots a lane of an oct
constexpr int F2SC_MAX_ROWS = 1024;
constexpr int F2SC_TAIL_LOG = 11;   // the tail's largest level, 2^11 entries
constexpr int F2SC_TAIL = 1 << F2SC_TAIL_LOG;
constexpr int F2SC_MAX_PASSES = 7;  // l <= 32

// Device state of a proof: rng[p] is the challenge stream's state before
// draw 3p (rng[0] comes from the seed), written by the launch that finishes
// pass p - 1.
struct F2scState {
    u64 rng[F2SC_MAX_PASSES + 1];
};

struct F2scPass {
    u32 p, prev_nrows;
    u64 seed;
    F2scState *ps;
    const u64 *prev_rows;  // pass p - 1's
    u64 *rows;             // this pass's
    u64 *msgs, *chals;     // the transcript's bases
};

u32 f2sc_passes(u32 l);
u32 f2sc_rows(u32 l, u32 p);
// Pass p < f2sc_passes(l): p = 0 reads the counts; p = 1 folds them, p >= 2
// folds src (level 3(p-1)), into dst (level 3p).
hipError_t launch_f2sc_pass(hipStream_t st, const F2scPass &a, u32 l, const u32 *a32, const u64 *src, u64 *dst);
// Rounds 3p .. l-1, p = f2sc_passes(l), from the counts (p <= 1) or src.
hipError_t launch_f2sc_tail(hipStream_t st, const F2scPass &a, u32 l, const u32 *a32, const u64 *src);

}  // namespace gkr

// steps.hpp -- the prover as a program of steps, executed by one kernel.
//
// A proof is a fixed sequence of steps (evaluation of each layer, the
// circuit's first small layers whole in one step that also evaluates them,
// then per layer: the p-phase, several rounds a step; the two omega phases,
// three rounds a step, after the eq tables of a* and b* where the level-0
// steps do not form them; and the line: V_{i+1} folded along it for layers of
// 2^11 entries and more, else the line points' eq tables and the line sums).
// Most steps are one grid pass; a step that ends sum-check rounds leaves one
// row of partial sums per workgroup.
//
// Every workgroup of the next step draws the round's challenge from the
// same SplitMix64 state (the verifier's coins do not depend on the
// messages), so no step ever synchronises workgroups inside a kernel; its
// workgroup 0 records the challenge and does the part of the round's finish
// that later rounds need (the beta prefix, v1 / v2, the next layer's z).
// Folding the rows into the message values is needed by nothing but the
// transcript, so every reducing step keeps rows of its own and one last
// step, ST_FINISH, folds all of them at once, one workgroup per message.
// The challenge of round j is used only after message j's sums are complete:
// in a later launch, or past a barrier of the one workgroup that ends a phase.
//
// One launch runs one step of each of several proofs (a job table maps
// workgroups to (proof, step)); a single proof is the one-job case.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace gkr {

typedef uint64_t u64;
typedef uint32_t u32;
typedef int32_t i32;
typedef uint8_t u8;

constexpr int SBLOCK = 512;      // threads per workgroup of the step kernel
constexpr int SMAX_BLOCKS = 512; // workgroups per step (2 per CU)
constexpr int LINE_CHUNK = 16;   // line points summed per workgroup
constexpr int ROW_STRIDE = 16;   // u64 per partial-sum row

enum StepKind : u32 {
    ST_EVAL = 0,   // V_i[g] = V_{i+1}[in1] op V_{i+1}[in2]
    ST_START,      // outputs into the transcript, z_0 drawn
    ST_EQ,         // eq half tables of a point (a* or b*)
    ST_P,          // p-phase, three to seven rounds (a-variables)
    ST_W,          // one omega round (b- or c-variables), gate by gate
    ST_FOLD,       // fold of V_{i+1}'s table by the last challenge
    ST_LT,         // eq tables of the line points
    ST_LINE,       // line sums h(t), t = 2..s'
    ST_SGE,        // next layer has one gate: v1 = v2 = V_{i+1}[0]
    ST_END,        // nothing but the prologue
    ST_WAGG,       // omega phase, tables: per-gate weights summed by bound wire
    ST_WT0,        // omega phase, tables: level-0 tables and rounds 0 to 2
    ST_WT,         // omega phase, tables: rounds k to k + 2 (fold, then sum)
    ST_WTAIL,      // omega phase, tables: remaining rounds in one workgroup
    ST_PTAIL,      // p-phase: remaining rounds in one workgroup
    ST_LOAD,       // inputs (pointer in state[3]) into V_d, range check
    ST_WA0,        // omega phase, tables: ST_WAGG and ST_WT0 in one pass, for
                   // layers whose wires each carry at most one chunk of gates
    ST_FINISH,     // every round's rows into its message values
    ST_WSMALL,     // omega phase of a small layer: eq table, level-0 tables, all rounds
    ST_TOP,        // the first layers whose tables all fit a tail, whole, in one workgroup
    ST_LFOLD,      // line of a wide layer: V_{i+1} folded along the line, 2^(tb+9) entries a workgroup
};

enum FinKind : u32 {
    FIN_NONE = 0,
    FIN_P,     // R p-phase messages from rows of 2^R column sums
    FIN_W,     // omega message from rows of (E0, E1, O0, O1)
    FIN_LINE,  // h(t) values from rows of line sums; then tau and z_{i+1}
    FIN_T,     // three table-round messages from rows of an oct's sums (T_ROW)
};

// Several rounds per launch.  The sums of a later round are, before the
// challenges between are known, polynomials in them with coefficients that are
// sums over the present tables: a step also sums those coefficients, and the
// messages follow from its rows and the challenges.
//   p-phase, R rounds: V_j's entries with equal low R index bits x, weighted
//     by eq(z, their other bits), add up to 2^R column sums T[x]; round k's
//     S_t = sum over x with bit k = t of T[x] prod_{i<k} eq(x_i, r_i)
//     prod_{i>k} eq(x_i, z_i), at one product an entry.
//   table rounds, three: A F + C over an oct of entries is a polynomial of
//     degree two in each of the three variables the rounds bind; its values at
//     {0, 1, inf}^3 (inf: the leading coefficient, a product of differences),
//     summed over the octs, are 27 words from which the three messages follow.

constexpr u32 KALL = 0xFFFF;  // kind resolved at run time (mixed batches)

// The finishes (bit f for FinKind f) a step of the given kind can carry;
// each kernel instantiation compiles only these.
__host__ __device__ constexpr u32 fin_mask(u32 kind) {
    return kind == KALL                              ? 0xFFu
           : kind == ST_P                            ? (1u << FIN_P) | (1u << FIN_LINE)
           : kind == ST_PTAIL                        ? (1u << FIN_P) | (1u << FIN_LINE)
           : kind == ST_WT                           ? 1u << FIN_T
           : kind == ST_WTAIL                        ? 1u << FIN_T
           : kind == ST_EQ                           ? (1u << FIN_LINE) | (1u << FIN_W)
           : kind == ST_END                          ? 1u << FIN_LINE
           : (kind == ST_W || kind == ST_FOLD || kind == ST_LT || kind == ST_LFOLD) ? 1u << FIN_W
                                                     : 0u;
}

// Largest table (entries at the level a tail starts from, after its fold)
// that a one-workgroup tail keeps in LDS.
constexpr int TAIL_LIM = 1024;
constexpr int TAIL_LOG = 10;  // log2(TAIL_LIM): rounds of a tail

// Per-proof device state shared by all steps of a proof.
struct ProofPtrs {
    u64 *msgs;   // transcript
    u64 *chals;  // challenges
    u64 *rngst;  // rngst[c] = SplitMix64 state before challenge c
    u64 *zbuf;   // z of the current layer
    u64 *state;  // [0] beta prefix C, [1] v1, [2] seed, [3] input pointer,
                 // [4] nonzero if an input is not below p
};

// Prologue: finish the previous round and/or draw challenge `draw`.  The
// message values themselves are written by ST_FINISH from `rows` (and, for
// p-phase rounds, the beta prefix and z values recorded in `rec`, P_REC words).
constexpr u32 P_ROUNDS = 7;  // most p-phase rounds a step sums (2^7 columns)
constexpr u32 P_REC = 16;    // C and up to 15 z values
constexpr u32 T_ROW = 32;    // an oct's sums: four slots for each of its eight lanes
constexpr u32 WT_COLS = 4 * T_ROW;  // the sums of a tail's steps of three rounds
constexpr u32 P_LAST = 5;    // a tail's last rounds, summed together
constexpr u32 PT_COLS = 64;  // words of a tail's columns: its first rounds' at 0, the last ones' at 32
struct Fin {
    u32 kind;          // FinKind
    i32 draw;          // challenge index drawn here (-1: none)
    const u64 *rows;   // partial rows of the previous step
    u32 nrows;
    u64 *rec;          // FIN_P: C, z_j .. z_{j+R-1} at the time of the rounds
    u32 j;             // FIN_P: first round's index (z_j)
    u32 R;             // FIN_P: rounds finished (challenges draw .. draw + R - 1)
    u32 last;          // FIN_W: 1 / 2 = end of phase 1 / 2 (v1 / v2)
    u32 T;             // FIN_LINE: number of line values
    u32 sp;            // FIN_LINE: coordinates of z_{i+1}
    u32 chunk_blocks;  // FIN_LINE: workgroups per chunk of line points
    u32 ch;            // FIN_LINE: line points per chunk
    const u64 *F;      // FIN_W last: the 2-entry table
    u64 *msg;          // where the message goes
    u64 *vout;         // FIN_W last: transcript slot of v1 / v2
    const u64 *bstar, *cstar;  // FIN_LINE: line endpoints (chals)
};

// One message (or one chunk of line values) of ST_FINISH.
struct FinItem {
    u32 kind;          // FinKind
    u32 nrows;
    const u64 *rows;
    u64 *msg;
    const u64 *rec;    // FIN_P
    i32 draw;          // FIN_T: the first round's challenge; FIN_P: the challenge of rec's first z
    u32 nvals;         // FIN_LINE: values of this chunk; FIN_P, FIN_T: rounds
    u32 pre;           // FIN_P: rounds between rec's C and the first of these
};
struct FinishArgs {
    const FinItem *items;  // one per workgroup
    const u64 *chals;
};

struct EvalArgs {
    u32 kind, S;
    u64 npad;
    const u8 *type;
    const u32 *in1, *in2;
    const u64 *Vn;
    u64 *V;
};
struct LoadArgs {
    u32 S;
    u64 npad;
    u64 *V;
};
struct StartArgs {
    u32 s0, S0;
    const u64 *V0;
};
struct EqArgs {
    u32 n;      // coordinates: challenges chals[base .. base+n) (the last may be drawn now)
    u32 L;      // lo table covers coordinates [0, L)
    u32 base;
    u64 *lo, *hi;
    u32 beta_lo;  // a*: lo entries times beta(z, a*) (state[0]), so that a gate's
                  // weight beta chi_g(a*) is lo[g mod 2^L] hi[g >> L]
};
// p-phase grid step.  pend = 0: rounds 0 .. R-1 of V_i, its column sums
// weighted by eq over z_i[R..s), in runs of SBLOCK entries (nu of them).
// pend >= 3: V^(j) from V^(j-pend) folded by the pend challenges just drawn,
// stored, and its 2^3 column sums (R = 3); a unit is eight entries of V^(j),
// of which live are not zero.
struct PArgs {
    u32 pend, R, s, j;
    u64 nu, live;
    const u64 *Vsrc;
    u64 *Vout;
};
struct WArgs {
    u32 kind, ph, init, write_w, inline_fold;
    u32 S, k;
    u64 nfold;
    const u32 *idx, *oth;
    const u8 *type;
    const u64 *F, *Vn;
    u64 *Fout;
    const u64 *alo, *ahi;
    u32 La;
    const u64 *blo, *bhi;
    u32 Lb;
    i32 rchal;  // non-inline rounds k > 0: index of r_{k-1} in chals
    u64 *w, *off;
};
struct FoldArgs {
    u64 nh;
    const u64 *src;
    u64 *dst;
};
struct LtArgs {
    u32 sp, L, M;
    u32 bbase, cbase;  // challenge indices of b* and c*
    u64 *lo, *hl, *hh;
};
// Line sums: chunk q of the workgroups takes points t' = q ch .. q ch + ch - 1
// (ch in {4, 8, 12, 16}, chunks of equal size); workgroups [q chunk_blocks,
// (q+1) chunk_blocks) make up a chunk.
struct LineArgs {
    u32 sp, L, M, T, chunk_blocks, ch;
    const u64 *V, *lo, *hl, *hh;
};
// Line of a layer with 2^11 <= 2^s' <= 2^32 by folding (ST_LFOLD):
// h(t) = ~V_{i+1}(b* + t (c* - b*)) is a polynomial of degree s' in t; V is
// folded coordinate by coordinate, each entry pair becoming a polynomial one
// degree higher.  With D = tb + 9, workgroup g (one per 2^D entries below
// S_{i+1}) folds entries [g 2^D, (g+1) 2^D) along coordinates 0..D-1 into
// a polynomial of degree D and writes its term of h(t), weighted along
// coordinates D..s'-1, for t = 2..s' as rows: value j in row
// (j / ROW_STRIDE) nwg + g, column j % ROW_STRIDE (nwg workgroups).
// ST_FINISH adds the rows up into h(2..s') as it does for the line sums'
// rows.
constexpr u32 LFOLD_MIN = 11, LFOLD_MAX = 32;
// Entries a thread folds, 2^tb: 128 to 256 workgroups from 2^17 to 2^22
// entries (a workgroup's time is set mostly by its LDS levels, not by tb), as
// many as there are below, and 2^(s' - 14) above (tb = 5 at most: more
// polynomials in registers would spill).
constexpr u32 lfold_tb(u32 sp) { return sp <= 17 ? 1 : sp == 18 ? 2 : sp <= 20 ? 3 : sp == 21 ? 4 : 5; }
static_assert(LFOLD_MIN >= 1 + 9, "a workgroup folds at least 2^(1 + 9) entries");
constexpr u32 lfold_wg(u32 sp) { return 1u << (sp - lfold_tb(sp) - 9); }
// Workgroups that cover the first n entries (V_{i+1} is zero from S_{i+1}
// on, so the blocks above hold zero polynomials and write no rows).
constexpr u32 lfold_wg_live(u32 sp, u64 n) {
    const u64 need = (n + (1ull << (lfold_tb(sp) + 9)) - 1) >> (lfold_tb(sp) + 9);
    return need < 1 ? 1u : need > lfold_wg(sp) ? lfold_wg(sp) : (u32)need;
}
constexpr u32 LFOLD_CHUNKS = 2;  // most rows a workgroup: h(2..s'), s' - 1 <= 2 ROW_STRIDE values
static_assert(LFOLD_MAX - 1 <= LFOLD_CHUNKS * ROW_STRIDE, "h(2..s') fits a workgroup's rows");
static_assert(LFOLD_MAX <= 32, "b*_k and c*_k - b*_k of the line sit in 32 words of LDS each");
struct LfoldArgs {
    u32 sp, tb, bbase, cbase;  // coordinates; 2^tb entries a thread; challenge indices of b* and c*
    const u64 *V;              // V_{i+1}
    u64 *rows;                 // nwg rows of ROW_STRIDE words for every ROW_STRIDE values
    const u64 *chals;
};
struct SgeArgs {
    const u64 *Vn;
    u64 *vslot;
};
// Tables of an omega phase: A[x] (weights) and C[x] (additive part) over
// the bound wire x, with F the fold of V_{i+1}:
//   G_k(t) = sum_m A_k(t, m) F_k(t, m) + C_k(t, m).
// Tiles of whole chunks spanning at most TILE_POS sorted positions (one
// wave each in the per-chunk sums), or a single big chunk of a heavy wire:
// tile t holds chunks [tch[t], tch[t+1]).
constexpr u32 TILE_POS = 64;
// Widest point whose eq tables a level-0 step forms in LDS: thirds of at most
// 2^7 entries.  Up to here an ST_EQ launch (4.2 us) costs more than the step's
// own tables (about 1 us) and the further products; at 2^22 gates these cost
// more than the launch.
constexpr u32 EQ_THIRDS = 20, EQ_THIRD = 128;
struct WaggArgs {
    u32 kind, ph;
    u32 nch;                 // chunks: sorted positions [cstart[ch], cstart[ch+1]) share one wire x
    const u32 *perm, *cstart;  // perm[p]: the gate at sorted position p
    const u32 *oths;         // other wire (ph 1: in2; ph 2: in1) by sorted position
    const u8 *types;         // gate type by sorted position (mixed layers)
    const u64 *Vn;
    const u64 *alo, *ahi;
    u32 La;
    const u64 *blo, *bhi;
    u32 Lb;
    u64 *partA, *partC;      // per chunk (ph 2: sums over ADD / MUL gates)
    u32 ntiles;              // tiles of whole chunks, at most 64 sorted positions each:
    const u32 *tch;          // tile t holds chunks [tch[t], tch[t+1])
};
// sum: whether the step sums rounds 0..2 (else it only forms the tables); nw
// wires, whole octs if it does.
struct Wt0Args {
    u32 ph, hasC, sum;
    u64 nw;
    const u32 *xch;          // chunks of wire x: [xch[x], xch[x+1])
    const u64 *partA, *partC;
    const u64 *F;            // V_{i+1}
    u64 *A, *C;              // level-0 tables
};
// ST_WA0: wire x's gates sit at sorted positions [rowptr[x], rowptr[x+1])
// (at most one chunk of gates per wire).  eqL > 0: the step forms the eq
// tables of a* (and b*, phase 2) itself, in LDS, as thirds of eqL coordinates
// each (an entry weighs one entry of each third): a launch less, a product
// more a point and gate than from the halves of an ST_EQ step.  The line:
// EQ_THIRDS coordinates (see there).
struct Wa0Args {
    u32 kind, ph, hasC, sum;
    u32 eqL, s, sp, co;      // coordinates of a* and b*, challenge index of a* (b* follows)
    u64 nw;
    const u32 *perm, *rowptr;
    const u32 *oths;
    const u8 *types;
    const u64 *Vn;           // V_{i+1}: gathered operands and the table F
    const u64 *alo, *ahi;
    u32 La;
    const u64 *blo, *bhi;
    u32 Lb;
    u64 *A, *C;              // level-0 tables
};
// Table step: level k folded by its three challenges to level k + 3, stored,
// and that level's sums; a unit is an entry of level k + 3 (whole octs).
struct WtArgs {
    u32 hasC;
    u64 nu;
    const u64 *A, *C, *F;    // level k
    u64 *An, *Cn, *Fn;       // level k + 3
};
struct WtailArgs {
    u32 k0, sp, hasC, last;
    u32 pend;                // challenges this step draws first: level k0 - pend is in memory (3, or 0)
    u32 live;                // level-k0 entries [live, 2^{sp-k0}) are zero (not read)
    const u64 *A, *C, *F;    // level k0-pend, 2^{sp-k0+pend} entries
    u32 c0;                  // challenge index of round k0
    u64 *cols;               // WT_COLS words
    u64 *vout;
};
struct PtailArgs {
    u32 j0, s;
    u32 pend;                // challenges the prologue drew (3; 0 when j0 = 0)
    u32 live;                // entries [live, 2^{s-j0}) of V^(j0) are zero (not read)
    const u64 *V;            // V^(j0-pend)
    u32 c0;                  // challenge index of round j0
    u64 *msg;                // message slot of round j0
    u64 *rec;                // C and z of the pending and the tail's rounds
    u64 *cols;               // PT_COLS words
};

// A small layer's whole omega phase in one workgroup: w as for ST_WA0
// (its eq table pointers are where this step writes the table of the
// phase's point), then rounds 0 .. sp-1 as a tail.
struct WsmallArgs {
    Wa0Args w;
    u32 eqn, eqL, eqbase;  // the point: coordinates, lo-table coordinates, challenge index
    u64 *eqlo, *eqhi;
    u32 sp, last, c0;       // last = phase (1: v1 into state[1]); c0: challenge index of round 0
    u64 *cols, *vout;       // cols: WT_COLS words
};

// ST_TOP: the sum-check of layers 0 .. nl-1 in one workgroup.  Every one of
// them has 2^s_i and 2^s_{i+1} (1 <= s_{i+1}) at most TAIL_LIM entries and
// one chunk of gates per wire in both omega phases.  Its p-phase, omega
// phases and line run as tails over tables kept in LDS from one layer to the
// next (V_{i+1}, read for the omega phases, is the next layer's V_i).
struct TopLayer {
    u32 s, sp, kind, co;       // s_i, s_{i+1}, gate mix, challenge index of round 0
    u64 *msg;                  // 3 n_i round values, v1, v2, h(2..s_{i+1})
    const u64 *Vn;             // V_{i+1}
    const u32 *rowptr[2], *perm[2], *oths[2];  // wire groups by in1 (phase 1) and in2 (phase 2)
    const u8 *types[2];        // gate types in sorted order (mixed layers)
    u32 S;                     // gates of layer i
    const u32 *in1, *in2;      // its wiring (evaluation)
    const u8 *type;            // its gate types (mixed layers)
    u64 *V;                    // V_i, written by the evaluation
    u64 *rec, *cols;           // the p-phase's record and columns (as PtailArgs)
    u64 *wcols[2];             // the omega phases' sums (WT_COLS words each)
};
// ST_TOP also evaluates its layers, nl - 1 down to 0, from V_nl (the layer
// below them, evaluated by ST_EVAL launches), and starts the proof as
// ST_START does (the randomness of z_0 and the outputs into the transcript).
struct TopArgs {
    u32 nl;
    const TopLayer *L;         // nl descriptors (device memory)
    const u64 *V0;             // V_0
};

struct StepDesc {
    u32 kind;
    u32 nblocks;
    u32 reduces;   // 1 if the step writes partial rows
    u32 K;         // values per row
    u64 *rows;     // this step's partial rows
    Fin fin;
    ProofPtrs pp;
    union {
        EvalArgs eval;
        StartArgs start;
        EqArgs eq;
        PArgs p;
        WArgs w;
        FoldArgs fold;
        LtArgs lt;
        LineArgs line;
        SgeArgs sge;
        WaggArgs wagg;
        Wt0Args wt0;
        WtArgs wt;
        WtailArgs wtail;
        PtailArgs ptail;
        LoadArgs load;
        Wa0Args wa0;
        FinishArgs finish;
        WsmallArgs wsmall;
        TopArgs top;
        LfoldArgs lfold;
    } u;
};

// One (proof, step) of a launch; workgroups [block0, next block0) run it.
struct JobEntry {
    const StepDesc *step;
    u32 block0;
    u32 pad;
};

// Workgroups a step needs.
u32 step_grid(const StepDesc &sd);
// One step of one proof (descriptor passed by value); ev0 / ev1 (or NULL)
// are recorded at the start and end of the dispatch.
hipError_t launch_step(hipStream_t st, const StepDesc &sd, hipEvent_t ev0 = nullptr,
                       hipEvent_t ev1 = nullptr);
// One step of each of njobs proofs (entries in device memory, sorted by
// block0, followed by a sentinel whose block0 is the total; each job spans
// step_grid(*step) workgroups).
hipError_t launch_steps(hipStream_t st, const JobEntry *jobs, u32 njobs, u32 total_blocks,
                        hipEvent_t ev0 = nullptr, hipEvent_t ev1 = nullptr);

// A launch's jobs passed by value (serving: the mix changes every launch).
constexpr int MAX_TABLE_JOBS = 128;
struct JobTable {
    u32 n, total;
    JobEntry e[MAX_TABLE_JOBS];
};
hipError_t launch_step_table(hipStream_t st, const JobTable &t);

// One proof of a batch: where its seed and input pointer go, and where its
// transcript is gathered.
struct BatchSlot {
    u64 *state;
    u64 seed, input;
    const u64 *msgs;
    u64 n_msgs, out_off, flag_off;
};
hipError_t launch_batch_setup(hipStream_t st, const BatchSlot *slots, u32 n);
// most_msgs: the longest transcript.
hipError_t launch_batch_gather(hipStream_t st, const BatchSlot *slots, u32 n, u64 most_msgs, u64 *out);

}  // namespace gkr

// steps.hip -- the step kernel: one launch runs one step of each job.
//
// Sec. 4.1.1 of the paper: every gate (or table entry) contributes
// independently to the prover's message, so a step is a grid-stride pass in
// which each workgroup sums its share (exchanges within a wave, matrix
// products of digits where a thread has several entries, then LDS) into one
// row of partial sums.  All arithmetic is exact in F_p (Sec. 6.1), so the
// result does not depend on the summation order.
#include <hip/hip_ext.h>

#include "lanes.hpp"
#include "steps.hpp"

namespace gkr {

using fp::add;
using fp::mul;
using fp::P;
using fp::sub;
using fp::u128;

struct alignas(16) u64x2 {
    u64 x, y;
};
__device__ __forceinline__ u64x2 ld2(const u64 *p, u64 i) { return *reinterpret_cast<const u64x2 *>(p + i); }
__device__ __forceinline__ void st2(u64 *p, u64 i, u64 a, u64 b) {
    u64x2 v;
    v.x = a;
    v.y = b;
    *reinterpret_cast<u64x2 *>(p + i) = v;
}

constexpr int NWAVES = SBLOCK / 64;
// LDS entries per table of an omega tail: 2^10 and the levels of an eighth, a
// 64th and a 512th after it (and room below for eq halves).
constexpr int TAIL_TAB = TAIL_LIM + TAIL_LIM / 4;
constexpr int TAIL_EXTRA = 8 + 2 * T_ROW + 16;  // weights, partial sums, challenges and RNG state after the three tables

// Words for workgroup sums, beside the body's.
__device__ __forceinline__ u64 *sum_lds() {
    __shared__ __align__(16) u64 t[NWAVES * ROW_STRIDE + ROW_STRIDE];
    return t;
}

// Sum over the wave, left in lane 63: prefix sums within each row of 16
// lanes (shifts 1, 2, 4, 8), then row 0's total into row 1 and row 2's into
// row 3, then lane 31's into rows 2 and 3.  Lanes a shift leaves without a
// source read 0.
__device__ __forceinline__ u64 wave_sum63(u64 v) {
    v = add(v, dppx<0x111, 0xf>(v));  // row_shr:1
    v = add(v, dppx<0x112, 0xf>(v));  // row_shr:2
    v = add(v, dppx<0x114, 0xf>(v));  // row_shr:4
    v = add(v, dppx<0x118, 0xf>(v));  // row_shr:8
    v = add(v, dppx<0x142, 0xa>(v));  // row_bcast:15 into rows 1, 3
    v = add(v, dppx<0x143, 0xc>(v));  // row_bcast:31 into rows 2, 3
    return v;
}

// Workgroup sum of v; thread k < K writes total k to out[k].
template <int K>
__device__ __forceinline__ void block_store(u64 (&v)[K], u64 *out) {
    static_assert(K <= ROW_STRIDE, "sum_lds");
    u64 (*sm)[NWAVES] = reinterpret_cast<u64 (*)[NWAVES]>(sum_lds());
#pragma unroll
    for (int k = 0; k < K; k++) v[k] = wave_sum63(v[k]);
    const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
    if (lane == 63) {
#pragma unroll
        for (int k = 0; k < K; k++) sm[k][wid] = v[k];
    }
    __syncthreads();
    if (threadIdx.x < K) {
        u64 a = 0;
#pragma unroll
        for (int w = 0; w < NWAVES; w++) a = add(a, sm[threadIdx.x][w]);
        out[threadIdx.x] = a;
    }
    __syncthreads();
}

__device__ __forceinline__ u64 xor64(u64 v, int m) {
    const int lo = __shfl_xor((int)(u32)v, m), hi = __shfl_xor((int)(u32)(v >> 32), m);
    return ((u64)(u32)hi << 32) | (u64)(u32)lo;
}

// Sum rows [first, first + n) of K <= ROW_STRIDE values; every thread of the
// workgroup receives the totals.  Lane l of a wave reads column l % 16 of
// row l / 16, so one load brings four whole rows and the rows stream in as
// coalesced, independent loads (sixteen in flight per lane); the four
// lanes of a column are then summed across the wave and the waves in LDS.
template <int K>
__device__ __forceinline__ void rows_total(const u64 *rows, u32 first, u32 n, u64 (&tot)[K]) {
    static_assert(K <= ROW_STRIDE, "a row holds at most ROW_STRIDE values");
    constexpr u32 STEP = NWAVES * 4;  // rows per pass of the workgroup
    constexpr u32 U = 16;             // passes per batch of loads
    u64 (*part)[ROW_STRIDE] = reinterpret_cast<u64 (*)[ROW_STRIDE]>(sum_lds());
    u64 *res = sum_lds() + NWAVES * ROW_STRIDE;
    const u32 lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
    const u32 r0 = wid * 4 + (lane >> 4);
    const u64 *p = rows + ((u64)first + wid * 4) * ROW_STRIDE + lane;  // row first + r0, column lane % 16
    const u32 passes = r0 < n ? (n - r0 + STEP - 1) / STEP : 0;
    u64 acc[4] = {0, 0, 0, 0};
    for (u32 j = 0; j < passes; j += U) {  // a batch's loads are all issued before any add
        u64 x[U];
#pragma unroll
        for (int q = 0; q < (int)U; q++) x[q] = j + q < passes ? p[(u64)(j + q) * STEP * ROW_STRIDE] : 0;
#pragma unroll
        for (int q = 0; q < (int)U; q++) acc[q & 3] = add(acc[q & 3], x[q]);
    }
    u64 v = add(add(acc[0], acc[1]), add(acc[2], acc[3]));
    v = add(v, xor64(v, 16));
    v = add(v, xor64(v, 32));
    if (lane < (u32)K) part[wid][lane] = v;
    __syncthreads();
    if (threadIdx.x < (u32)K) {
        u64 t = part[0][threadIdx.x];
#pragma unroll
        for (int w = 1; w < NWAVES; w++) t = add(t, part[w][threadIdx.x]);
        res[threadIdx.x] = t;
    }
    __syncthreads();
#pragma unroll
    for (int k = 0; k < K; k++) tot[k] = res[k];
}

// chi of the bits of x over coordinates pt[0..n)
__device__ __forceinline__ u64 chi_bits(u64 x, const u64 *pt, u32 n) {
    u64 e = 1;
    for (u32 k = 0; k < n; k++) e = mul(e, fp::eqbit((u32)((x >> k) & 1), pt[k]));
    return e;
}

struct Ctx {
    u64 *lds;        // lds_words(kind) words: every kind lays its arrays over the same ones
    u32 lb, nb;      // this workgroup within the step, workgroups of the step
    u64 gtid, gstride;
    u64 r;           // challenge drawn in the prologue
    u64 rl;          // lane k: the k-th challenge drawn
};

// What a tail takes over from its launch's prologue: the RNG state after the
// drawn challenges (if the prologue drew any).
struct TailIn {
    u64 st;
    u32 drew;
};

// Value t of a p-phase message from the two sums: G(0) = C (1-z) S0,
// G(1) = C z S1, G(2) = C (3z - 1)(2 S1 - S0); t is chosen per lane.
__device__ __forceinline__ u64 p_value(u32 t, u64 C, u64 z, u64 S0, u64 S1) {
    const u64 e = t == 0 ? sub(1, z) : (t == 1 ? z : sub(add(add(z, z), z), 1));
    const u64 S = t == 0 ? S0 : (t == 1 ? S1 : sub(add(S1, S1), S0));
    return mul(mul(C, e), S);
}

// Value k of tot, k chosen per lane.
template <int K>
__device__ __forceinline__ u64 pick(const u64 (&tot)[K], u32 k) {
    u64 v = 0;
#pragma unroll
    for (int q = 0; q < K; q++) v = k == (u32)q ? tot[q] : v;
    return v;
}

// The part of a round's finish that later rounds need; it reads no rows.
// The first wave records the beta prefix C and the z values of p-phase rounds
// for their messages and advances C by the drawn challenges; thread 0,
// at the end of an omega phase folds the last pair into v1 / v2; the line
// finish stores z_{i+1}.
template <u32 KIND>
__device__ __forceinline__ void fin_inline(const StepDesc &sd, const Ctx &c, const u64 *s_pt) {
    const Fin &f = sd.fin;
    const ProofPtrs &pp = sd.pp;
    constexpr u32 FM = fin_mask(KIND);
    const u32 tid = threadIdx.x;
    if ((FM & (1u << FIN_P)) && f.kind == FIN_P) {
        if (tid < 64) {  // lane k: round j + k
            const bool on = tid < f.R;
            const u64 z = on ? pp.zbuf[f.j + tid] : 0, C = pp.state[0];
            if (on) f.rec[1 + tid] = z;
            const u64 e = row_product(on ? fp::eq(z, c.rl) : 1);
            if (tid == 0) {
                f.rec[0] = C;
                pp.state[0] = mul(C, e);  // beta prefix over r_0 .. r_{j+R-1}
            }
        }
    } else if ((FM & (1u << FIN_W)) && f.kind == FIN_W) {
        if (f.last && tid == 0) {
            const u64 f0 = f.F[0], f1 = f.F[1];
            const u64 v = add(f0, mul(c.r, sub(f1, f0)));
            *f.vout = v;
            if (f.last == 1) pp.state[1] = v;
        }
    } else if ((FM & (1u << FIN_LINE)) && f.kind == FIN_LINE) {
        if (tid < f.sp) pp.zbuf[tid] = s_pt[tid];
        if (tid == 0) pp.state[0] = 1;  // the next layer's a-variables start unbound
    }
}

// Message of p-phase round k of the R summed in the columns T (2^R words of
// LDS), z and r the rounds' coordinates and challenges, C the beta prefix
// before round k; one wave.
__device__ __forceinline__ void p_message(const u64 *T, u32 R, u32 k, const u64 *z, const u64 *r, u64 C, u64 *msg) {
    const u32 lane = threadIdx.x & 63;
    u64 S0 = 0, S1 = 0;
    for (u32 x = lane; x < (1u << R); x += 64) {
        u64 w = T[x];
        for (u32 i = 0; i < R; i++)  // (uniform)
            if (i != k) w = mul(w, fp::eqbit((x >> i) & 1, i < k ? r[i] : z[i]));
        if ((x >> k) & 1)
            S1 = add(S1, w);
        else
            S0 = add(S0, w);
    }
    S0 = wave_total(S0);
    S1 = wave_total(S1);
    if (lane < 3) msg[lane] = p_value(lane, C, z[k], S0, S1);
}
// The beta prefix after rounds 0 .. k-1 (k <= 16): C0 prod eq(z_i, r_i), in
// every lane.
__device__ __forceinline__ u64 beta_prefix(u64 C0, u32 k, const u64 *z, const u64 *r) {
    const u32 lane = threadIdx.x & 63;
    return uniform(mul(C0, row_product(lane < k ? fp::eq(z[lane], r[lane]) : 1)));
}

// Three table rounds from octs of entries, one entry a lane (lane j of the
// oct: bits x, y, z of j).  At a point of {0, 1, inf}^3 the term is a product
// of A's and F's values there, a difference along every inf axis (either sign:
// both factors share it), plus C at the corners.  Lane j takes four of the 27:
//   slot 0: corner j;
//   slot 1: x inf (lanes x = 0); x, z inf (x = 1, z = 0); all inf (lane 5);
//   slot 2: y inf (lanes y = 0); x, y inf (y = 1, x = 0);
//   slot 3: z inf (lanes z = 0); y, z inf (z = 1, y = 0).
// Every lane runs the same instructions (operands chosen by its bits).  o: this
// lane's factors of slots 1..3, below 2p.
__device__ __forceinline__ void oct_factors(u32 lane, u64 v, u64 (&o)[3]) {
    const bool x = lane & 1, y = lane & 2, z = lane & 4;
    const u64 dx = v + (P - from1(v)), dy = v + (P - from2(v)), dz = v + (P - from4(v));
    const u64 dxz = fp::fold64_mad(dx + (2 * P - from4(dx))), dxy = fp::fold64_mad(dx + (2 * P - from2(dx)));
    const u64 dyz = fp::fold64_mad(dy + (2 * P - from4(dy)));
    const u64 dxyz = fp::fold64_mad(dxz + (2 * P - from2(dxz)));  // (dxz below 2^61 + 8)
    o[0] = !x ? dx : (!z ? dxz : dxyz);
    o[1] = !y ? dy : dxy;
    o[2] = !z ? dz : dyz;
}
// One slot's factor alone (SLOT 1..3), as oct_factors forms it.
template <int SLOT>
__device__ __forceinline__ u64 oct_factor(u32 lane, u64 v) {
    const bool x = lane & 1, y = lane & 2, z = lane & 4;
    if (SLOT == 1) {
        const u64 dx = v + (P - from1(v)), dxz = fp::fold64_mad(dx + (2 * P - from4(dx)));
        const u64 dxyz = fp::fold64_mad(dxz + (2 * P - from2(dxz)));
        return !x ? dx : (!z ? dxz : dxyz);
    }
    const u64 dy = v + (P - from2(v));
    if (SLOT == 2) {
        const u64 dx = v + (P - from1(v)), dxy = fp::fold64_mad(dx + (2 * P - from2(dx)));
        return !y ? dy : dxy;
    }
    const u64 dz = v + (P - from4(v)), dyz = fp::fold64_mad(dy + (2 * P - from4(dy)));
    return !z ? dz : dyz;
}
// Sums of the lane's four slots: products below 2^124, up to eight between
// reductions.
struct OctSums {
    u128 acc[4] = {0, 0, 0, 0};
    u64 s[4] = {0, 0, 0, 0};
    u32 terms = 0;
};
__device__ __forceinline__ void oct_flush(OctSums &q) {
    q.terms = 0;
#pragma unroll
    for (int k = 0; k < 4; k++) {
        q.s[k] = add(q.s[k], fp::red128(q.acc[k]));
        q.acc[k] = 0;
    }
}
__device__ __forceinline__ void oct_add(u32 lane, u64 A, u64 C, u64 F, OctSums &q) {
    u64 a[3], f[3];
    oct_factors(lane, A, a);
    oct_factors(lane, F, f);
    q.acc[0] += fp::wide(A, F) + C;
#pragma unroll
    for (int k = 0; k < 3; k++) q.acc[k + 1] += fp::wide(a[k], f[k]);
    if (++q.terms == 8) oct_flush(q);
}
// The wave's sums into out[4 j + k]: lanes of equal j = lane mod 8 added, the
// slots spread over the lanes on the way (an exchange of two slots leaves one
// sum of each in either half): a narrow step ends with this, and runs each of
// its instructions once; summing every slot in every lane made the steps 0.6
// (ST_WT) and 1.1 us (ST_WA0) longer at 2^17 wires.
__device__ __forceinline__ void oct_wave(OctSums &q, u64 *out) {
    const u32 lane = threadIdx.x & 63;
    oct_flush(q);
    const u64 v = swap16_sum(swap32_sum(q.s[0], q.s[1]), swap32_sum(q.s[2], q.s[3]));  // (four values below p)
    const u64 t = reduced(v + from8(v));
    if (!(lane & 8)) out[4 * (lane & 7) + ((lane >> 4) & 1) * 2 + (lane >> 5)] = t;
}
// A grid step's row.
__device__ __forceinline__ void oct_row(OctSums &q, u64 *part, u64 *row) {
    oct_wave(q, part + (threadIdx.x >> 6) * T_ROW);
    __syncthreads();
    if (threadIdx.x < T_ROW) {
        u64 t = 0;  // (eight values below p)
#pragma unroll
        for (int w = 0; w < NWAVES; w++) t += part[w * T_ROW + threadIdx.x];
        row[threadIdx.x] = reduced(t);
    }
}
// LDS written before by this wave's lanes is read after (one wave's LDS
// operations stay in order; this keeps the compiler's order).
__device__ __forceinline__ void wave_lds() {
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
}
// Word of a row that holds the point (x, y, z), 2 for inf.
__device__ __forceinline__ u32 point_word(u32 x, u32 y, u32 z) {
    if (x < 2 && y < 2 && z < 2) return 4 * (x + 2 * y + 4 * z);
    if (x == 2 && y < 2) return 4 * (z < 2 ? 2 * y + 4 * z : 1 + 2 * y) + 1;
    if (x == 2 && z == 2) return 4 * 5 + 1;
    if (y == 2 && z < 2) return 4 * (x < 2 ? x + 4 * z : 2 + 4 * z) + 2;
    return 4 * (y == 2 ? x + 4 : x + 2 * y) + 3;
}

// The octs' sums on the matrix cores, for steps whose threads take several
// entries.  Every one of the 27 sums is a combination of the 64 sums S_ij =
// sum over the octs of A_i F_j, and with the entries written in eight signed
// digits, v = sum_l d_l(v) 256^l with -128 <= d_l < 128, those are
// combinations of the 64 x 64 sums of products of digits: one product of
// bytes, contracted over the octs, exact in 32 bits for below 2^17 octs a
// wave.  A wave collects 32 octs, four entries a lane (entry lane mod 8 of
// octs lane / 8 + 8 u, u < 4), takes the bytes of its four entries apart by
// digit and passes them through LDS to the lanes that own rows (digit l, entry
// i): row l' 8 + i of the tile of digits 4 t + l'.  About 22 instructions an
// entry against 180 of oct_add, but some 500 at a workgroup's end: a step of
// fewer than four entries a thread stays with oct_add.  The level-0 step of a
// layer of 2^22 gates 55 -> 44 us, of 2^24 wires 212 -> 172; the table steps
// (ST_WT) gain nothing, near the rate of memory at such sizes.
typedef int i32x4 __attribute__((ext_vector_type(4)));
typedef int i32x16 __attribute__((ext_vector_type(16)));
constexpr u32 GRAM_DIG = 68;               // LDS dwords a digit: 64 lanes, padded (reads without bank conflicts)
constexpr u32 GRAM_WORDS = 8 * GRAM_DIG / 2;  // LDS words a wave
struct Gram {
    i32x16 acc[2][2];  // by tile of A's and F's digits
    u64 c;             // sum of the lane's C entries, below 2^61 + 8
};
// (A last turn that some waves lack stays with oct_add as well: 786,500 wires,
// just above three a thread, prove in 437 us so and in 425 with oct_add, 900,001
// in 448 and 441, 1,040,001 in 473 and 467; 2^20, four a thread, in 472.)
__device__ __forceinline__ bool gram_fits(u64 n, u64 stride) {  // (uniform)
    return n >= 4 * stride && n <= (stride << 13);               // at most 2^16 octs a wave
}
// The lane's operands (both digit tiles) of its four entries v.
__device__ __forceinline__ void gram_operand(u32 lane, const u64 (&v)[4], u32 *stage, i32x4 (&op)[2]) {
    constexpr u64 H = 0x8080808080808080ull;
    u32 lo[4], hi[4];
#pragma unroll
    for (u32 u = 0; u < 4; u++) {
        const u64 d = (v[u] + H) ^ H;  // (v < 2^61: nothing is carried out of the top digit)
        lo[u] = (u32)d;
        hi[u] = (u32)(d >> 32);
    }
    auto put = [&](u32 l, const u32 (&x)[4]) {  // digits l .. l + 3, a dword of four octs each
        const u32 a = __builtin_amdgcn_perm(x[1], x[0], 0x05010400), b = __builtin_amdgcn_perm(x[3], x[2], 0x05010400);
        const u32 e = __builtin_amdgcn_perm(x[1], x[0], 0x07030602), f = __builtin_amdgcn_perm(x[3], x[2], 0x07030602);
        u32 *o = stage + l * GRAM_DIG + (lane & 7) * 8 + (lane >> 3);
        o[0] = __builtin_amdgcn_perm(b, a, 0x05040100);
        o[GRAM_DIG] = __builtin_amdgcn_perm(b, a, 0x07060302);
        o[2 * GRAM_DIG] = __builtin_amdgcn_perm(f, e, 0x05040100);
        o[3 * GRAM_DIG] = __builtin_amdgcn_perm(f, e, 0x07060302);
    };
    put(0, lo);
    put(4, hi);
    wave_lds();
#pragma unroll
    for (u32 t = 0; t < 2; t++)
        op[t] = *reinterpret_cast<const i32x4 *>(stage + (4 * t + (lane & 31) / 8) * GRAM_DIG + (lane & 7) * 8 +
                                                 (lane >> 5) * 4);
    wave_lds();
}
__device__ __forceinline__ void gram_add(u32 lane, const u64 (&A)[4], const u64 (&F)[4], u32 *stage, Gram &g) {
    i32x4 a[2], f[2];
    gram_operand(lane, A, stage, a);
    gram_operand(lane, F, stage, f);
#pragma unroll
    for (u32 t = 0; t < 2; t++)
#pragma unroll
        for (u32 m = 0; m < 2; m++)
            g.acc[t][m] = __builtin_amdgcn_mfma_i32_32x32x32_i8(a[t], f[m], g.acc[t][m], 0, 0, 0);
}
// The workgroup's row from its waves' sums; lds: GRAM_WORDS a wave.
__device__ __forceinline__ void gram_row(const Gram &g, u64 *lds, u64 *row) {
    const u32 lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    // Lane: column (digit m' of the tile, entry j of F), rows (digit l', entry
    // i = 4 (lane / 32) + r of A) in word 4 l' + r.
    const u32 sh = 8 * ((lane >> 3) & 3);
    u64 s = 0;
#pragma unroll
    for (u32 r = 0; r < 4; r++) {
        int64_t x[2][2];
#pragma unroll
        for (u32 t = 0; t < 2; t++)
#pragma unroll
            for (u32 m = 0; m < 2; m++) {
                x[t][m] = g.acc[t][m][12 + r];
#pragma unroll
                for (int l = 2; l >= 0; l--) x[t][m] = x[t][m] * 256 + g.acc[t][m][4 * l + r];  // below 2^56
            }
        // (a multiple of p above 2^121 makes the sum positive)
        const u64 v = fp::red128(((u128)P << 61) + (u128)x[0][0] + ((u128)(x[0][1] + x[1][0]) << 32) +
                                 ((u128)x[1][1] << 64));
        const u64 q = ((v << sh) & P) | (v >> (61 - sh));  // times 256^m'
        const u64 tot = reduced(plus16(q + from8(q)));     // over m'
        if (((lane >> 3) & 3) == r) s = tot;
    }
    const u64 c = reduced(plus32(plus16(reduced(g.c) + from8(reduced(g.c)))));
    u64 *part = lds + w * GRAM_WORDS;
    part[(4 * (lane >> 5) + ((lane >> 3) & 3)) * 8 + (lane & 7)] = s;  // S_ij
    if (lane < 8) part[64 + lane] = c;
    __syncthreads();
    u64 *b0 = lds + 80, *b1 = b0 + 72;  // (past the first wave's part)
    if (threadIdx.x < 72) {
        u64 t = 0;
#pragma unroll
        for (u32 k = 0; k < NWAVES; k++) t = add(t, lds[k * GRAM_WORDS + threadIdx.x]);
        b0[threadIdx.x] = t;
    }
    __syncthreads();
    if (w) return;
    // One variable after another: its bits (i, j) = (0, 0), (1, 1) give the
    // points 0 and 1, (1 - 0)(1 - 0) the point inf.
    u64 *src = b0, *dst = b1;
#pragma unroll
    for (u32 v = 0; v < 3; v++) {
        const u32 np = v == 0 ? 1 : (v == 1 ? 3 : 9), nb = 4 >> v;  // points so far; entries left a side
        const u32 rest = lane % (nb * nb), pd = lane / (nb * nb);
        u64 x = 0;
        if (pd < 3 * np) {
            const u32 p = pd % np, d = pd / np;
            const u64 *S = src + p * 4 * nb * nb + (rest / nb) * 4 * nb + 2 * (rest % nb);
            const u64 s00 = S[0], s01 = S[1], s10 = S[2 * nb], s11 = S[2 * nb + 1];
            x = d == 0 ? s00 : (d == 1 ? s11 : sub(add(s00, s11), add(s01, s10)));
        }
        wave_lds();
        dst[lane] = x;
        wave_lds();
        u64 *t = src;
        src = dst;
        dst = t;
    }
    // points (x, y, z) in src[x + 3 y + 9 z]
    const u32 x = lane % 3, y = (lane / 3) % 3, z = lane / 9;
    const u64 val = add(src[lane], x < 2 && y < 2 && z < 2 ? b0[64 + x + 2 * y + 4 * z] : 0);
    if (lane < T_ROW) dst[lane] = 0;
    wave_lds();
    if (lane < 27) dst[point_word(x, y, z)] = val;
    wave_lds();
    if (lane < T_ROW) row[lane] = dst[lane];
}
// Message k of the three rounds from the octs' sums E (T_ROW words, LDS): lane
// x + 3 y + 9 z holds the point (x, y, z), 2 for inf.  The rounds before k are
// bound (a quadratic is q0 (1 - r) + q1 r + qinf (r^2 - r)), those after it
// summed over 0 and 1; G(2) = 2 G(1) - G(0) + 2 G(inf).  One wave.
__device__ __forceinline__ void t_message(const u64 *E, u32 k, const u64 *r, u64 *msg) {
    const u32 lane = threadIdx.x & 63;
    const u32 d[3] = {lane % 3, (lane / 3) % 3, lane / 9};
    const u32 x = d[0], y = d[1], z = d[2];
    u64 v = lane < 27 ? E[point_word(x, y, z)] : 0;
#pragma unroll
    for (u32 i = 0; i < 3; i++) {
        if (i < k) {  // (uniform)
            const u64 ri = r[i];
            v = mul(v, d[i] == 0 ? sub(1, ri) : (d[i] == 1 ? ri : sub(mul(ri, ri), ri)));
        } else if (i > k && d[i] == 2) {
            v = 0;
        }
    }
    const u32 dk = k == 0 ? x : (k == 1 ? y : z);
    const u64 q0 = wave_total(dk == 0 ? v : 0), q1 = wave_total(dk == 1 ? v : 0), q2 = wave_total(dk == 2 ? v : 0);
    if (lane < 3) msg[lane] = lane == 0 ? q0 : (lane == 1 ? q1 : sub(add(add(q1, q1), add(q2, q2)), q0));
}

// One item of ST_FINISH: the rows of one round (FIN_W), of the rounds a step
// summed (FIN_P, FIN_T: the columns are added up, then a wave forms each
// message) or of a chunk of line values into the transcript.
__device__ __forceinline__ void step_finish(const FinishArgs &a, const Ctx &c) {
    const FinItem &it = a.items[c.lb];
    const u32 tid = threadIdx.x;
    switch (it.kind) {
        case FIN_P: {  // column sums, then a wave a message
            u64 *s_col = c.lds;
            const u32 R = it.nvals, x = tid & ((1u << R) - 1), G = SBLOCK >> R;
            u64 t = 0;
            constexpr u32 U = 16;  // loads in flight
            for (u32 q0 = tid >> R; q0 < it.nrows; q0 += G * U) {
                u64 v[U];
#pragma unroll
                for (u32 i = 0; i < U; i++) {
                    const u32 q = q0 + i * G;
                    v[i] = q < it.nrows ? it.rows[((u64)q << R) + x] : 0;
                }
#pragma unroll
                for (u32 i = 0; i < U; i++) t = add(t, v[i]);
            }
            s_col[tid] = t;
            __syncthreads();
            for (u32 h = SBLOCK / 2; h >= (1u << R); h >>= 1) {
                if (tid < h) s_col[tid] = add(s_col[tid], s_col[tid + h]);
                __syncthreads();
            }
            const u32 k = tid >> 6;
            if (k < R) {
                const u64 *z = it.rec + 1, *r = a.chals + it.draw;
                p_message(s_col, R, k, z + it.pre, r + it.pre, beta_prefix(it.rec[0], it.pre + k, z, r), it.msg + 3 * k);
            }
            break;
        }
        case FIN_W: {
            u64 t[4];
            rows_total<4>(it.rows, 0, it.nrows, t);
            if (tid == 0) {
                const u64 E0 = t[0], E1 = t[1], O0 = t[2], O1 = t[3];
                it.msg[0] = E0;
                it.msg[1] = O1;
                u64 o4 = add(O1, O1);
                o4 = add(o4, o4);
                it.msg[2] = sub(add(sub(E0, add(E1, E1)), o4), add(O0, O0));
            }
            break;
        }
        case FIN_T: {  // the octs' sums, then a wave a message
            u64 *s_col = c.lds;
            const u32 x = tid & (T_ROW - 1);
            constexpr u32 G = SBLOCK / T_ROW, U = 16;
            u64 t = 0;
            for (u32 q0 = tid / T_ROW; q0 < it.nrows; q0 += G * U) {
                u64 v[U];
#pragma unroll
                for (u32 i = 0; i < U; i++) {
                    const u32 q = q0 + i * G;
                    v[i] = q < it.nrows ? it.rows[(u64)q * T_ROW + x] : 0;
                }
#pragma unroll
                for (u32 i = 0; i < U; i++) t = add(t, v[i]);
            }
            s_col[tid] = t;
            __syncthreads();
            for (u32 h = SBLOCK / 2; h >= T_ROW; h >>= 1) {
                if (tid < h) s_col[tid] = add(s_col[tid], s_col[tid + h]);
                __syncthreads();
            }
            const u32 k = tid >> 6;
            if (k < it.nvals) t_message(s_col, k, a.chals + it.draw, it.msg + 3 * k);
            break;
        }
        case FIN_LINE: {
            u64 t[LINE_CHUNK];
            rows_total<LINE_CHUNK>(it.rows, 0, it.nrows, t);
            if (tid < it.nvals) it.msg[tid] = pick(t, tid);
            break;
        }
        default: break;
    }
}

// ------------------------------------------------------------ step bodies

__device__ __forceinline__ void step_load(const LoadArgs &a, const ProofPtrs &pp, const Ctx &c) {
    const u64 *src = reinterpret_cast<const u64 *>(pp.state[3]);
    u64 bad = 0;
    for (u64 g = c.gtid; g < a.npad; g += c.gstride) {
        u64 v = 0;
        if (g < a.S) {
            v = src[g];
            bad |= v >= P;
        }
        a.V[g] = v;
    }
    if (bad) atomicOr(reinterpret_cast<unsigned long long *>(pp.state + 4), 1ull);
}

__device__ __forceinline__ void step_eval(const EvalArgs &a, const Ctx &c) {
    for (u64 g = c.gtid; g < a.npad; g += c.gstride) {
        u64 v = 0;
        if (g < a.S) {
            const u64 x = a.Vn[a.in1[g]], y = a.Vn[a.in2[g]];
            const bool ismul = a.kind == 1 || (a.kind == 2 && a.type[g]);
            v = ismul ? mul(x, y) : add(x, y);
        }
        a.V[g] = v;
    }
}

__device__ __forceinline__ void step_start(const StartArgs &a, const ProofPtrs &pp, const Ctx &c) {
    if (c.lb == 0 && threadIdx.x == 0) {
        u64 st = fp::sm_state(pp.state[2], fp::PURPOSE_GKR);  // state[2] = seed
        pp.rngst[0] = st;
        for (u32 k = 0; k < a.s0; k++) {
            const u64 z = fp::sm_field(st);
            pp.chals[k] = z;
            pp.zbuf[k] = z;
            pp.rngst[k + 1] = st;
        }
        pp.state[0] = 1;
        pp.state[1] = 0;
    }
    for (u64 g = c.gtid; g < a.S0; g += c.gstride) pp.msgs[g] = a.V0[g];
}

__device__ __forceinline__ void step_eq(const EqArgs &a, const Ctx &c, const u64 *pt, const ProofPtrs &pp) {
    const u64 nlo = 1ull << a.L, nhi = 1ull << (a.n - a.L);
    const u64 beta = a.beta_lo ? pp.state[0] : 1;
    for (u64 x = c.gtid; x < nlo + nhi; x += c.gstride) {
        if (x < nlo)
            a.lo[x] = a.beta_lo ? mul(beta, chi_bits(x, pt, a.L)) : chi_bits(x, pt, a.L);
        else
            a.hi[x - nlo] = chi_bits(x - nlo, pt + a.L, a.n - a.L);
    }
}

// x1 - x0 + p, not reduced (canonical x0, x1: below 2 p).
__device__ __forceinline__ u64 diff_lz(u64 x1, u64 x0) { return x1 + (fp::P - x0); }

// p-phase grid steps (see PArgs).  zp: z_i in LDS (first step) or memory.
// FIRST: whether this is the phase's first step, compile-time (1, 0; one
// kernel each) or -1 to take a.pend.
//
// First step: bound by the read of V_i and one product an entry.  A thread
// keeps its place in the SBLOCK-entry runs, so its entry's weight is one
// scalar a run times a factor of its own, applied once at the end.  A narrow
// one is the chain of its loads: the first runs' values and the line's points
// are asked for before the wait for the challenge state, and a run's weight is
// a product over lanes (6.4 -> 5.4 us at 2^17 entries).
struct Runs {  // a thread's values in its workgroup's next four runs
    u64 v[4];
};
__device__ __forceinline__ Runs load_runs(const PArgs &a, const Ctx &c, u64 q0, u32 n) {
    const u64 *src = a.Vsrc + q0 * SBLOCK + threadIdx.x;
    Runs r;
#pragma unroll
    for (u32 i = 0; i < 4; i++) r.v[i] = i < n ? src[(u64)i * c.nb * SBLOCK] : 0;
    return r;
}
__device__ __forceinline__ u32 runs_from(const PArgs &a, const Ctx &c, u64 q0) {  // 0 .. 64
    if (q0 >= a.nu) return 0;
    const u64 left = (a.nu - q0 + c.nb - 1) / c.nb;
    return left < 64 ? (u32)left : 64;
}
// x: the first runs' values (under way since before the prologue's wait).
__device__ __forceinline__ void step_p_first(const PArgs &a, const Ctx &c, const u64 *zp, u64 *row, Runs x) {
    u64 *s_w = c.lds, (*s_sum)[64] = reinterpret_cast<u64 (*)[64]>(s_w + 64);
    constexpr u32 LB = 9;
    static_assert((1 << LB) == SBLOCK, "SBLOCK");
    const u32 tid = threadIdx.x, lane = tid & 63, R = a.R;
    u64 own = 1;  // the weight of the thread's place in a run
    for (u32 k = R; k < LB; k++) own = mul(own, fp::eqbit((tid >> k) & 1, zp[k]));
    u64 t = 0;
    for (u64 q0 = c.lb; q0 < a.nu; q0 += 64ull * c.nb) {  // 64 runs of this workgroup at a time
        const u32 n = runs_from(a, c, q0);
        if (q0 != c.lb) x = load_runs(a, c, q0, n);
        // their weights: a row of 16 lanes a run, a coordinate a lane
        for (u32 i = tid >> 4; i < n; i += SBLOCK / 16) {
            const u64 q = q0 + (u64)i * c.nb;
            u64 w = 1;
            for (u32 k = LB + (tid & 15); k < a.s; k += 16) w = mul(w, fp::eqbit((u32)(q >> (k - LB)) & 1, zp[k]));
            s_w[i] = row_product(w);
        }
        __syncthreads();
        u128 acc = 0;
        for (u32 i0 = 0; i0 < n; i0 += 4) {
            if (i0) x = load_runs(a, c, q0 + (u64)i0 * c.nb, n - i0);
#pragma unroll
            for (u32 i = 0; i < 4; i++)  // (up to 64 products below 2^122)
                if (i0 + i < n) acc += fp::wide(s_w[i0 + i], x.v[i]);
        }
        t = add(t, fp::red128(acc));
        __syncthreads();  // s_w is read
    }
    t = mul(t, own);
    // threads of equal column tid mod 2^R, over the wave and the waves
    for (u32 b = R; b < 6; b++) t = plus_bit(t, b);
    s_sum[tid >> 6][lane] = t;
    __syncthreads();
    if (tid < (1u << R)) {
        const u32 w0 = tid >> 6, step = R > 6 ? 1u << (R - 6) : 1;
        u64 s = 0;
        for (u32 w = w0; w < (u32)NWAVES; w += step) s = add(s, s_sum[w][tid & 63]);
        row[tid] = s;
    }
}

// Later steps: eight lanes form an entry of V^(j) from its 2^pend entries of
// V^(j-pend) and a wave a unit of eight entries, lane group g holding column g.
// The first unit's loads are issued before draw() waits for the challenge
// state: a step this small is a chain of memory round trips.
template <typename Draw>
__device__ __forceinline__ void step_p_next(const PArgs &a, const Ctx &c, const u64 *zp, u64 *row, Draw draw) {
    u64 *s_chi = c.lds, (*s_sum)[8] = reinterpret_cast<u64 (*)[8]>(s_chi + (1 << P_ROUNDS));
    const u32 tid = threadIdx.x, lane = tid & 63, wid = tid >> 6, l = lane & 7, g = lane >> 3, pend = a.pend;
    const u64 ustep = (u64)c.nb * NWAVES;
    u64 u = (u64)c.lb * NWAVES + wid;
    // a lane's entries of unit u: one (pend = 3), or two of each 16
    constexpr u32 MX = 1 << (P_ROUNDS - 4);
    const u32 n = pend == 3 ? 0 : 1u << (pend - 4);
    u64x2 x[MX];
    auto load = [&](u64 uu) {
        const u64 m = 8 * uu + g;
        const bool on = uu < a.nu && m < a.live;
        const u64 *src = a.Vsrc + (m << pend);
        if (n == 0) x[0].x = on ? src[l] : 0;
#pragma unroll
        for (u32 i = 0; i < MX; i++)
            if (i < n) {
                x[i].x = x[i].y = 0;
                if (on) x[i] = ld2(src, 16 * i + 2 * l);
            }
    };
    load(u);
    // lane k < nz of each row of 16: coordinate k of a unit's index (usually
    // all s - j - 3 of them)
    const u32 nz = a.s - a.j - 3, kz = lane & 15;
    const u64 z1 = kz < nz ? zp[a.j + 3 + kz] : 0;
    draw();
    if (tid < (1u << pend)) {  // chi_tid of the drawn challenges
        u64 w = 1;
        for (u32 k = 0; k < pend; k++) w = mul(w, fp::eqbit((tid >> k) & 1, lane_value(c.rl, k)));
        s_chi[tid] = w;
    }
    __syncthreads();
    u64 sum = 0;
    while (u < a.nu) {  // (wave-uniform)
        const u64 m = 8 * u + g;
        u64 v;
        if (n == 0) {
            v = mul(s_chi[l], x[0].x);
        } else {
            u128 acc = 0;
#pragma unroll
            for (u32 i = 0; i < MX; i++)
                if (i < n) {
                    const u64x2 w = ld2(s_chi, 16 * i + 2 * l);
                    acc += fp::wide(w.x, x[i].x) + fp::wide(w.y, x[i].y);
                }
            v = fp::red128(acc);
        }
        v = reduced(oct_total(v));
        if (l == 0) a.Vout[m] = v;
        u64 w = row_product(kz < nz ? fp::eqbit((u32)(u >> kz) & 1, z1) : 1);
        for (u32 k = 16; k < nz; k++) w = mul(w, fp::eqbit((u32)(u >> k) & 1, zp[a.j + 3 + k]));
        sum = add(sum, mul(w, v));
        u += ustep;
        load(u);
    }
    if (l == 0) s_sum[wid][g] = sum;
    __syncthreads();
    if (tid < 8) {
        u64 s = 0;
#pragma unroll
        for (int w = 0; w < NWAVES; w++) s = add(s, s_sum[w][tid]);
        row[tid] = s;
    }
}

template <int FIRST, typename Draw>
__device__ __forceinline__ void step_p(const PArgs &a, const Ctx &c, const u64 *zp, u64 *row, Draw draw, Runs x) {
    if (FIRST == 1 || (FIRST < 0 && a.pend == 0))
        step_p_first(a, c, zp, row, FIRST == 1 ? x : load_runs(a, c, c.lb, runs_from(a, c, c.lb)));
    else
        step_p_next(a, c, zp, row, draw);
}

// Gate g with bound-wire index idx, at round k of its phase:
//   term_g(t) = w_g eq(bit_k(idx), t) (F(t) + off_g)
// with F(t) = (1-t) F[2m] + t F[2m+1], m = idx >> (k+1), the extension of
// V_{i+1} at the partially bound point.  MUL gates carry their fixed
// operand inside w (off = 0), ADD gates in off.  With P0 = w (F[2m] + off),
// P1 = w (F[2m+1] + off):  bit 0 adds P0 at t=0 and P0 - 2 P1 at t=2;
// bit 1 adds P1 at t=1 and 4 P1 - 2 P0 at t=2.  The row holds (E0, E1)
// = sums of (P0, P1) over bit-0 gates and (O0, O1) over bit-1 gates.
template <int KIND, int PH>
__device__ __forceinline__ void step_w(const WArgs &a, const Ctx &c, const ProofPtrs &pp, u64 *row) {
    const bool init = a.init, inl = a.inline_fold, wr = a.write_w;
    u64 r = 0, omr = 0;
    if (!init) {
        r = inl ? c.r : pp.chals[a.rchal];
        omr = sub(1, r);
    }
    const u64 v1 = PH == 2 ? pp.state[1] : 0;
    const u64 amask = (1ull << a.La) - 1, bmask = (1ull << a.Lb) - 1;
    const u32 k = a.k;
    if (inl) {
        // this round's table F^(k) = F^(k-1) folded by r, for the next round
        for (u64 m = c.gtid; m < a.nfold; m += c.gstride) {
            const u64x2 p = ld2(a.F, 2 * m);
            a.Fout[m] = add(p.x, mul(r, sub(p.y, p.x)));
        }
    }
    u64 acc[4] = {0, 0, 0, 0};
    for (u64 g = c.gtid; g < a.S; g += c.gstride) {
        const u32 idx = a.idx[g];
        const bool ismul = KIND == 1 || (KIND == 2 && a.type[g]);
        u64 wt, of;
        if (init) {
            u64 wg = mul(a.alo[g & amask], a.ahi[g >> a.La]);  // beta chi_g(a*): lo carries beta
            if (PH == 1) {
                const u64 y = a.Vn[a.oth[g]];
                wt = ismul ? mul(wg, y) : wg;
                of = ismul ? 0 : y;
                if (KIND != 1) a.off[g] = of;
            } else {
                const u32 i1 = a.oth[g];
                wg = mul(wg, mul(a.blo[i1 & bmask], a.bhi[i1 >> a.Lb]));
                wt = ismul ? mul(wg, v1) : wg;
                of = ismul ? 0 : v1;
            }
        } else {
            wt = mul(a.w[g], ((idx >> (k - 1)) & 1) ? r : omr);
            if (PH == 1)
                of = KIND == 1 ? 0 : a.off[g];
            else
                of = ismul ? 0 : v1;
        }
        u64 f0, f1;
        if (inl) {
            const u64 q = ((u64)idx >> (k + 1)) << 2;
            const u64x2 p0 = ld2(a.F, q), p1 = ld2(a.F, q + 2);
            f0 = add(p0.x, mul(r, sub(p0.y, p0.x)));
            f1 = add(p1.x, mul(r, sub(p1.y, p1.x)));
        } else {
            const u64x2 f = ld2(a.F, ((u64)idx >> (k + 1)) << 1);
            f0 = f.x;
            f1 = f.y;
        }
        const u64 P0 = mul(wt, add(f0, of)), P1 = mul(wt, add(f1, of));
        if ((idx >> k) & 1) {
            acc[2] = add(acc[2], P0);
            acc[3] = add(acc[3], P1);
        } else {
            acc[0] = add(acc[0], P0);
            acc[1] = add(acc[1], P1);
        }
        if (wr) a.w[g] = wt;
    }
    block_store<4>(acc, row);
}

__device__ __forceinline__ void step_fold(const FoldArgs &a, const Ctx &c) {
    const u64 r = c.r;
    for (u64 m = c.gtid; m < a.nh; m += c.gstride) {
        const u64x2 p = ld2(a.src, 2 * m);
        a.dst[m] = add(p.x, mul(r, sub(p.y, p.x)));
    }
}

// Line step (a9).  h(t) = ~V_{i+1}(l(t)) for t = 2..s', l(t) = b* + t (c* - b*).
// x = (hh 2^M + mid) 2^L + lane: chi_x(l(t)) = Hh_t[hh] Hl_t[mid] lo_t[lane].
// Tables: lo [T][2^L], hl [T][2^M], hh [2^H][T].
__device__ __forceinline__ void step_lt(const LtArgs &a, const Ctx &c, const u64 *bstar, const u64 *cstar) {
    if (a.sp < 2) return;  // no line points
    const u32 T = a.sp - 1, H = a.sp - a.L - a.M;
    const u64 nlo = 1ull << a.L, nhl = 1ull << a.M, nhh = 1ull << H;
    const u64 per = nlo + nhl + nhh;
    for (u64 e = c.gtid; e < (u64)T * per; e += c.gstride) {
        const u32 tp = (u32)(e / per);
        const u64 x = e % per;
        const u64 t = tp + 2;
        u32 base, n;
        u64 bits;
        if (x < nlo) {
            base = 0; n = a.L; bits = x;
        } else if (x < nlo + nhl) {
            base = a.L; n = a.M; bits = x - nlo;
        } else {
            base = a.L + a.M; n = H; bits = x - nlo - nhl;
        }
        u64 v = 1;
        for (u32 k = 0; k < n; k++) {
            const u64 b = bstar[base + k], cc = cstar[base + k];
            const u64 l = add(b, mul(t, sub(cc, b)));
            v = mul(v, fp::eqbit((u32)((bits >> k) & 1), l));
        }
        if (x < nlo)
            a.lo[(u64)tp * nlo + bits] = v;
        else if (x < nlo + nhl)
            a.hl[(u64)tp * nhl + bits] = v;
        else
            a.hh[bits * T + tp] = v;
    }
}

// Workgroups [q * chunk_blocks, (q+1) * chunk_blocks) sum line points
// t' = 16 q .. 16 q + 15; within a chunk, wave `mid` walks hh.
// The weights hh[h][t] of 64 consecutive h pass through LDS (one read per
// tile, broadcast reads in the loop); every lane runs the loop, lanes past
// the table adding zeros.  Products are summed exactly in 128 bits and
// reduced once per tile (<= 64 terms).
template <int CH>
__device__ void line_sums(const LineArgs &a, const Ctx &c, u64 *row) {
    u64 (*s_w)[CH] = reinterpret_cast<u64 (*)[CH]>(c.lds);
    const u32 T = a.T, H = a.sp - a.L - a.M;
    const u64 nlo = 1ull << a.L, nhl = 1ull << a.M, nhh = 1ull << H;
    const u32 chunk = c.lb / a.chunk_blocks;
    const u32 t0 = chunk * CH;
    const u32 lane = threadIdx.x & 63;
    const u64 mid = (u64)(c.lb - chunk * a.chunk_blocks) * NWAVES + (threadIdx.x >> 6);
    const bool ok = lane < nlo && mid < nhl;
    const u64 x0 = ok ? (mid << a.L) + lane : 0;
    u64 s[CH];
#pragma unroll
    for (int t = 0; t < CH; t++) s[t] = 0;
    for (u64 h0 = 0; h0 < nhh; h0 += 64) {
        const u32 nh = nhh - h0 < 64 ? (u32)(nhh - h0) : 64u;
        __syncthreads();  // the previous tile's weights are read
        for (u32 i = threadIdx.x; i < 64u * CH; i += SBLOCK) {
            const u32 hl = i / CH, t = i % CH;
            s_w[hl][t] = hl < nh && t0 + t < T ? a.hh[(h0 + hl) * T + t0 + t] : 0;
        }
        __syncthreads();
        u128 w128[CH];
#pragma unroll
        for (int t = 0; t < CH; t++) w128[t] = s[t];
        for (u32 hl = 0; hl < nh; hl++) {
            const u64 v = ok ? a.V[((h0 + hl) << (a.M + a.L)) + x0] : 0;
#pragma unroll
            for (int t = 0; t < CH; t++) w128[t] += fp::wide(s_w[hl][t], v);
        }
#pragma unroll
        for (int t = 0; t < CH; t++) s[t] = fp::red128(w128[t]);
    }
    u64 acc[LINE_CHUNK];
#pragma unroll
    for (int t = 0; t < LINE_CHUNK; t++) {
        acc[t] = 0;
        if (t < CH && t0 + t < T && ok)
            acc[t] = mul(s[t < CH ? t : 0], mul(a.hl[(u64)(t0 + t) * nhl + mid], a.lo[(u64)(t0 + t) * nlo + lane]));
    }
    block_store<LINE_CHUNK>(acc, row);
}

__device__ __forceinline__ void step_line(const LineArgs &a, const Ctx &c, u64 *row) {
    switch (a.ch) {
        case 4: line_sums<4>(a, c, row); break;
        case 8: line_sums<8>(a, c, row); break;
        case 12: line_sums<12>(a, c, row); break;
        default: line_sums<16>(a, c, row); break;
    }
}

// ------------------------------------------- omega phases over tables
//
// Grouping the gates of an omega phase by the wire x they bind, the
// per-gate terms w_g eq(bit_k(x), t) (F(t) + off_g) of round k sum to
//   G_k(t) = sum_m A_k(t, m) F_k(t, m) + C_k(t, m),
// with A_0[x] = sum of w_g over the gates on x, C_0[x] = sum of w_g off_g,
// and A_k, C_k, F_k the folds of A_0, C_0 and V_{i+1} by the phase's first
// k challenges (all three are multilinear in the bound bits).  The gates are
// read once per phase instead of once per round.

// Sums over the gates perm[p0 .. p1) of one wire x.  Phase 1: MUL gates
// put w V[in2] on x's value (sA), ADD gates put w on it (sA) and add
// w V[in2] (sC).  Phase 2: sums of the weights over ADD gates (sA) and MUL
// gates (sC); v1 enters when the level-0 tables are formed.
// GK, PH: the layer's gate mix (0 ADD, 1 MUL, 2 mixed) and the phase when
// known at compile time, -1 and 0 to read them from a.
// wa(g): beta chi_g(a*); wb(i): chi_i(b*).
template <int GK, int PH, typename Args, typename Wa, typename Wb>
__device__ __forceinline__ void wire_sums_of(const Args &a, u32 p0, u32 p1, u64 &sA_out, u64 &sC_out, Wa wa, Wb wb) {
    const u32 kind = GK >= 0 ? (u32)GK : a.kind, ph = PH > 0 ? (u32)PH : a.ph;
    // branch-free updates keep both sums in registers; a sum that a gate
    // mix leaves at zero is not updated
    u64 sA = 0, sC = 0;
    for (u32 p = p0; p < p1; p++) {
        const u32 g = a.perm[p], o = a.oths[p];
        const bool ismul = kind == 1 || (kind == 2 && a.types[p]);
        u64 w = wa(g);
        if (ph == 1) {
            const u64 wy = mul(w, a.Vn[o]);
            if (kind == 1) {
                sA = add(sA, wy);
            } else {
                sA = add(sA, ismul ? wy : w);
                sC = add(sC, ismul ? 0 : wy);
            }
        } else {
            w = mul(w, wb(o));
            if (kind == 1) {
                sC = add(sC, w);
            } else if (kind == 0) {
                sA = add(sA, w);
            } else {
                sA = add(sA, ismul ? 0 : w);
                sC = add(sC, ismul ? w : 0);
            }
        }
    }
    sA_out = sA;
    sC_out = sC;
}
template <int GK = -1, int PH = 0, typename Args>
__device__ __forceinline__ void wire_sums(const Args &a, u32 p0, u32 p1, u64 &sA_out, u64 &sC_out) {
    const u64 amask = (1ull << a.La) - 1, bmask = (1ull << a.Lb) - 1;
    wire_sums_of<GK, PH>(
        a, p0, p1, sA_out, sC_out, [&](u32 g) { return mul(a.alo[g & amask], a.ahi[g >> a.La]); },
        [&](u32 i) { return mul(a.blo[i & bmask], a.bhi[i >> a.Lb]); });
}

// Value v of lane l (l uniform or not; every lane of the wave takes part).
__device__ __forceinline__ u64 bperm64(u64 v, u32 l) {
    const int lo = __builtin_amdgcn_ds_bpermute((int)(l << 2), (int)(u32)v);
    const int hi = __builtin_amdgcn_ds_bpermute((int)(l << 2), (int)(u32)(v >> 32));
    return ((u64)(u32)hi << 32) | (u64)(u32)lo;
}

// Per-chunk sums of the gates' terms (wires with more than one chunk).  A
// wave takes a tile of whole chunks (at most 64 sorted positions) and lane
// l the gate at the tile's position l, so the gate arrays are read in
// coalesced runs; the inclusive scan of the terms over the wave gives each
// chunk's sum as the scan at its last position minus the scan just before
// its first.  Terms as in wire_sums (beta(z, a*), which multiplies every
// term, comes with the lo half of a*'s eq table).
// GK, PH: the gate mix and phase, compile-time (one kernel each) or -1, 0.
template <int GK, int PH>
__device__ __forceinline__ void step_wagg(const WaggArgs &a, const ProofPtrs &pp, const Ctx &c) {
    (void)pp;  // beta(z, a*) is in the lo half of a*'s eq table
    const u32 kind = GK >= 0 ? (u32)GK : a.kind, ph = PH > 0 ? (u32)PH : a.ph;
    const u32 lane = threadIdx.x & 63;
    const u64 amask = (1ull << a.La) - 1, bmask = (1ull << a.Lb) - 1;
    const u64 nwaves = c.gstride >> 6;
    for (u64 t = c.gtid >> 6; t < a.ntiles; t += nwaves) {  // wave-uniform
        const u32 c0 = a.tch[t], nc = a.tch[t + 1] - c0;
        if (nc == 0) continue;  // (a group without gates has one empty tile)
        const u32 base = a.cstart[c0], end = a.cstart[c0 + nc];
        if (end - base > TILE_POS) {  // one big chunk of a heavy wire: lanes stride over it
            u64 sA = 0, sC = 0;
#pragma unroll 4
            for (u32 q = base + lane; q < end; q += 64) {
                const u32 g = a.perm[q], o = a.oths[q];
                const bool ismul = kind == 1 || (kind == 2 && a.types[q]);
                u64 w = mul(a.alo[g & amask], a.ahi[g >> a.La]);
                if (ph == 1) {
                    const u64 wy = mul(w, a.Vn[o]);
                    sA = add(sA, ismul ? wy : w);
                    sC = add(sC, ismul ? 0 : wy);
                } else {
                    w = mul(w, mul(a.blo[o & bmask], a.bhi[o >> a.Lb]));
                    sA = add(sA, ismul ? 0 : w);
                    sC = add(sC, ismul ? w : 0);
                }
            }
            sA = wave_sum63(sA);
            sC = wave_sum63(sC);
            if (lane == 63) {
                a.partA[c0] = sA;
                a.partC[c0] = sC;
            }
            continue;
        }
        const u32 p = base + lane;
        u64 vA = 0, vC = 0;
        if (p < end) {
            const u32 g = a.perm[p], o = a.oths[p];
            const bool ismul = kind == 1 || (kind == 2 && a.types[p]);
            u64 w = mul(a.alo[g & amask], a.ahi[g >> a.La]);
            if (ph == 1) {
                const u64 wy = mul(w, a.Vn[o]);
                vA = ismul ? wy : w;
                vC = ismul ? 0 : wy;
            } else {
                w = mul(w, mul(a.blo[o & bmask], a.bhi[o >> a.Lb]));
                vA = ismul ? 0 : w;
                vC = ismul ? w : 0;
            }
        }
        const u64 sA = wave_sum63(vA), sC = wave_sum63(vC);  // inclusive scans
        const bool mine = lane < nc;  // lane k writes chunk c0 + k
        const u32 k = mine ? lane : 0;
        const u32 first = a.cstart[c0 + k] - base, last = a.cstart[c0 + k + 1] - base - 1;
        const u32 before = first ? first - 1 : 0;
        const u64 A1 = bperm64(sA, last), C1 = bperm64(sC, last);
        const u64 A0 = bperm64(sA, before), C0 = bperm64(sC, before);
        if (mine) {
            a.partA[c0 + k] = first ? sub(A1, A0) : A1;
            a.partC[c0 + k] = first ? sub(C1, C0) : C1;
        }
    }
}

// Level-0 entries from a wire's sums (phase 2: ADD gates w (v1 + G(t)),
// MUL gates w v1 G(t)).
__device__ __forceinline__ void level0(u32 ph, u64 v1, u64 sA, u64 sC, u64 &A, u64 &C) {
    if (ph == 2) {
        A = add(sA, mul(v1, sC));
        C = mul(v1, sA);
    } else {
        A = sA;
        C = sC;
    }
}

// Level-0 tables of an omega phase and the sums of its first three rounds
// (sum); a lane takes a wire, so eight adjacent lanes hold an oct (nw and the
// stride are multiples of 8).  wire(x, sA, sC) gives the sums of wire x's
// gates.  GK, PH: the gate mix and phase when known at compile time (-1, 0: ph
// and hasC).
template <int GK, int PH, typename Wire>
__device__ __forceinline__ void level0_round(u32 ph_rt, u32 hasC_rt, u32 sum, u64 nw, const u64 *F, u64 *At, u64 *Ct,
                                             const ProofPtrs &pp, const Ctx &c, u64 *row, u64 *stage, Wire wire) {
    const u32 ph = PH > 0 ? (u32)PH : ph_rt;
    const bool hasC = GK >= 0 ? GK != 1 : hasC_rt != 0;
    const u64 v1 = ph == 2 ? pp.state[1] : 0;
    const u32 lane = threadIdx.x & 63;
    auto entry = [&](u64 x, u64 &A, u64 &C, u64 &f) {
        f = F[x];
        u64 sA, sC;
        wire(x, sA, sC);
        if (GK == 1 && ph == 2) {  // MUL gates only: sA is zero
            A = mul(v1, sC);
            C = 0;
        } else {
            level0(ph, v1, sA, sC, A, C);
        }
        if (!hasC) C = 0;
        At[x] = A;
        if (hasC) Ct[x] = C;
    };
    if (GK >= 0 && sum && gram_fits(nw, c.gstride)) {  // (uniform)
        u32 *st = reinterpret_cast<u32 *>(stage + (threadIdx.x >> 6) * GRAM_WORDS);
        Gram g = {};
        for (u64 b = c.gtid - lane; b < nw; b += 4 * c.gstride) {  // (whole waves)
            u64 A[4] = {0, 0, 0, 0}, f[4] = {0, 0, 0, 0};
#pragma unroll
            for (u32 u = 0; u < 4; u++) {
                const u64 x = b + u * c.gstride + lane;
                u64 C = 0;
                if (x < nw) entry(x, A[u], C, f[u]);
                if (hasC) g.c = fp::fold64(g.c + C);
            }
            gram_add(lane, A, f, st, g);
        }
        gram_row(g, stage, row);
        return;
    }
    OctSums q;
    for (u64 x = c.gtid; x < nw; x += c.gstride) {
        u64 A, C, f;
        entry(x, A, C, f);
        if (sum) oct_add(lane, A, C, f, q);  // (uniform)
    }
    if (sum) oct_row(q, c.lds, row);
}

// Level 0 from the chunk sums: wire x's sums add its chunks
// [xch[x], xch[x+1]).  A lane adds the chunks of its own wire when they are
// few; a wire with more (the pattern entries of pattern matching feed up to
// 2^18 gates) is summed by the whole wave, lanes striding over its chunks,
// one such wire after another.  Whole waves iterate together, so the wave
// reductions see every lane.
constexpr u32 WT0_LANE_CHUNKS = 64;
__device__ __forceinline__ void step_wt0(const Wt0Args &a, const ProofPtrs &pp, const Ctx &c, u64 *row) {
    const u64 v1 = a.ph == 2 ? pp.state[1] : 0;
    const u32 lane = threadIdx.x & 63;
    OctSums q;
    for (u64 base = c.gtid - lane; base < a.nw; base += c.gstride) {  // wave-uniform
        const u64 x = base + lane;
        const bool on = x < a.nw;
        u32 c0 = 0, c1 = 0;
        if (on) {
            c0 = a.xch[x];
            c1 = a.xch[x + 1];
        }
        const bool many = c1 - c0 > WT0_LANE_CHUNKS;
        u64 sA = 0, sC = 0;
        if (!many) {
            for (u32 ch = c0; ch < c1; ch++) {
                sA = add(sA, a.partA[ch]);
                sC = add(sC, a.partC[ch]);
            }
        }
        for (u64 hm = __ballot(many); hm; hm &= hm - 1) {
            const u32 l = (u32)__ffsll((long long)hm) - 1;  // uniform
            const u32 b0 = (u32)__builtin_amdgcn_readlane((int)c0, l);
            const u32 b1 = (u32)__builtin_amdgcn_readlane((int)c1, l);
            u64 wA = 0, wC = 0;
#pragma unroll 4
            for (u32 ch = b0 + lane; ch < b1; ch += 64) {
                wA = add(wA, a.partA[ch]);
                wC = add(wC, a.partC[ch]);
            }
            wA = lane_value(wave_sum63(wA), 63);
            wC = lane_value(wave_sum63(wC), 63);
            if (lane == l) {
                sA = wA;
                sC = wC;
            }
        }
        u64 A, C, f = 0;
        level0(a.ph, v1, sA, sC, A, C);
        if (!a.hasC) C = 0;
        if (on) {
            a.A[x] = A;
            if (a.hasC) a.C[x] = C;
            f = a.F[x];
        } else {
            A = C = 0;
        }
        if (a.sum) oct_add(lane, A, C, f, q);  // (uniform)
    }
    if (a.sum) oct_row(q, c.lds, row);
}

// Thirds of the eq table of the n coordinates pt (chals): entry (q, x) of tab,
// x < 2^L, is chi of x over coordinates q L .. (q+1) L - 1 (those past n are 0),
// times scale in third 0.  One entry a thread and turn.
__device__ __forceinline__ void eq_thirds(u64 *tab, const u64 *pt, u32 n, u32 L, u64 scale, u32 first, u32 step) {
    for (u32 e = first; e < (3u << L); e += step) {
        const u32 q = e >> L, x = e & ((1u << L) - 1);
        u64 f[7];  // (L <= 7)
#pragma unroll
        for (u32 k = 0; k < 7; k++) {
            const u32 j = q * L + k;
            const u64 r = k < L && j < n ? pt[j] : 0;
            f[k] = fp::eqbit((x >> k) & 1, r);
        }
        const u64 v = mul(mul(mul(f[0], f[1]), mul(f[2], f[3])), mul(mul(f[4], f[5]), f[6]));
        tab[q * EQ_THIRD + x] = q == 0 ? mul(scale, v) : v;
    }
}
static_assert(EQ_THIRD == 1 << 7 && EQ_THIRDS <= 3 * 7, "thirds of at most 7 coordinates");

// GK, PH: the gate mix and phase, compile-time (one kernel each) or -1, 0.
template <int GK, int PH>
__device__ __forceinline__ void step_wa0(const Wa0Args &a, const ProofPtrs &pp, const Ctx &c, u64 *row) {
    u64 *stage = c.lds + NWAVES * T_ROW + 6 * EQ_THIRD;
    if (a.eqL) {  // (uniform)
        const u32 ph = PH > 0 ? (u32)PH : a.ph, L = a.eqL, m = (1u << L) - 1;
        u64 *ta = c.lds + NWAVES * T_ROW, *tb = ta + 3 * EQ_THIRD;
        const u32 half = SBLOCK / 2, tid = threadIdx.x;
        if (ph == 1)
            eq_thirds(ta, pp.chals + a.co, a.s, L, pp.state[0], tid, SBLOCK);
        else if (tid < half)  // (the two tables side by side)
            eq_thirds(ta, pp.chals + a.co, a.s, L, pp.state[0], tid, half);
        else
            eq_thirds(tb, pp.chals + a.co + a.s, a.sp, L, 1, tid - half, half);
        __syncthreads();
        auto chi = [&](const u64 *t, u32 x) {
            return mul(mul(t[x & m], t[EQ_THIRD + ((x >> L) & m)]), t[2 * EQ_THIRD + (x >> (2 * L))]);
        };
        level0_round<GK, PH>(a.ph, a.hasC, a.sum, a.nw, a.Vn, a.A, a.C, pp, c, row, stage, [&](u64 x, u64 &sA, u64 &sC) {
            wire_sums_of<GK, PH>(
                a, a.rowptr[x], a.rowptr[x + 1], sA, sC, [&](u32 g) { return chi(ta, g); },
                [&](u32 i) { return chi(tb, i); });
        });
        return;
    }
    level0_round<GK, PH>(a.ph, a.hasC, a.sum, a.nw, a.Vn, a.A, a.C, pp, c, row, stage, [&](u64 x, u64 &sA, u64 &sC) {
        wire_sums<GK, PH>(a, a.rowptr[x], a.rowptr[x + 1], sA, sC);
    });
}

// The eight entries of one entry of the level three below, and their fold by
// three challenges (chi: the eight weights).
struct Eight {
    u64x2 p[4];
};
__device__ __forceinline__ Eight ld8(const u64 *X, u64 g) {
    Eight e;
#pragma unroll
    for (u32 k = 0; k < 4; k++) e.p[k] = ld2(X, 8 * g + 2 * k);
    return e;
}
__device__ __forceinline__ u64 fold3(const Eight &e, const u64 (&chi)[8]) {
    u128 t = 0;
#pragma unroll
    for (u32 k = 0; k < 4; k++) t += fp::wide(chi[2 * k], e.p[k].x) + fp::wide(chi[2 * k + 1], e.p[k].y);
    return fp::red128(t);
}
// The weights of a fold by the challenges in lanes off .. off + 2 of rl: one a
// lane, then scalars.
__device__ __forceinline__ void chi8(u64 rl, u64 (&chi)[8]) {
    const u32 lane = threadIdx.x;
    const u64 x = mul(mul(fp::eqbit(lane & 1, lane_value(rl, 0)), fp::eqbit((lane >> 1) & 1, lane_value(rl, 1))),
                      fp::eqbit((lane >> 2) & 1, lane_value(rl, 2)));
#pragma unroll
    for (u32 e = 0; e < 8; e++) chi[e] = lane_value(x, e);
}

// HC: whether the layer has a C table, compile-time (one kernel each) or -1.
// The first entries' loads are issued before draw() waits for the challenge
// state.
template <int HC, typename Draw>
__device__ __forceinline__ void step_wt(const WtArgs &a, const Ctx &c, u64 *row, Draw draw) {
    const bool hasC = HC >= 0 ? HC != 0 : a.hasC != 0;
    const u32 lane = threadIdx.x & 63;
    u64 g = c.gtid;
    Eight A = {}, F = {}, C = {};
    auto load = [&](u64 e) {
        if (e < a.nu) {
            A = ld8(a.A, e);
            F = ld8(a.F, e);
            if (hasC) C = ld8(a.C, e);
        }
    };
    load(g);
    draw();
    u64 chi[8];
    chi8(c.rl, chi);
    OctSums q;
    for (; g < a.nu; g += c.gstride) {  // (whole octs)
        const u64 vA = fold3(A, chi), vF = fold3(F, chi), vC = hasC ? fold3(C, chi) : 0;
        a.An[g] = vA;
        a.Fn[g] = vF;
        if (hasC) a.Cn[g] = vC;
        oct_add(lane, vA, vC, vF, q);
        load(g + c.gstride);  // (48 registers: not held across oct_add)
    }
    oct_row(q, c.lds, row);
}

// ------------------------------------------------------------------ tails
//
// An omega tail runs the last rounds of a phase in one workgroup, three rounds
// at a time (see FIN_T) over tables in LDS: the sums of a level's octs are
// complete at a barrier, the level is folded by the three challenges, one
// thread a table and entry, and a second barrier publishes the next level, an
// eighth as long.  A wave issues an instruction every four to six cycles and
// waits for the instruction cache on code it has not run yet, so the tail's
// length is what one wave runs between barriers, and every level runs the same
// code: a wave sums one of the octs' four slots, the last wave draws the
// challenges and forms the fold's weights.  ST_FINISH forms the messages from
// the sums.
static_assert((1 << TAIL_LOG) == TAIL_LIM, "TAIL_LOG");
static_assert(NWAVES == 8, "two waves a slot");
static_assert(3 * TAIL_LIM / 8 <= SBLOCK, "one thread a table and folded entry");

// RNG state of the tail's first round: the prologue drew the pending
// challenges and left the state after them; a tail without them reads it.
__device__ __forceinline__ u64 tail_state(const ProofPtrs &pp, u32 c0, u32 drew, u64 st) {
    __shared__ u64 s_st;
    if (drew) return uniform(st);
    if (threadIdx.x == 0) s_st = pp.rngst[c0];
    __syncthreads();
    return uniform(s_st);
}

// The rounds of an omega tail over tables A, C, F in LDS (areas of TAIL_TAB
// entries one after another from tab, then TAIL_EXTRA words).  Level 0, 2^L
// entries, is at the start of each area, complete at a barrier.  The steps'
// sums go to cols, challenges c0, c0 + 1, ... are recorded (and into rec, in
// LDS, when rec is not NULL) with the RNG state after them; F's last entry is v1
// (last = 1) or v2, to *vout and left in tab[2 TAIL_TAB + TAIL_TAB - 1].  Returns
// the RNG state after the last round.
// HC: whether the phase has a C table, compile-time (1, 0) or -1 to take hc_rt.
template <int HC = -1>
__device__ __forceinline__ u64 wtail_rounds(u64 *tab, u32 L, bool hc_rt, u64 st, u64 *cols, u32 c0, u32 last, u64 *vout,
                                            const ProofPtrs &pp, u64 *rec = nullptr) {
    const bool hc = HC >= 0 ? HC != 0 : hc_rt;
    u64 *A = tab, *Ct = tab + TAIL_TAB, *F = tab + 2 * TAIL_TAB;
    u64 *s_w = tab + 3 * TAIL_TAB, *part = s_w + 8, *s_r = part + 2 * T_ROW, *s_st = s_r + 15;
    const u32 tid = threadIdx.x, lane = tid & 63;
    const u32 w = (u32)__builtin_amdgcn_readfirstlane((int)(tid >> 6));  // wave-uniform
    const u32 slot = w & 3, half = w >> 2;
    u32 n = 1u << L, base = 0;
    u64 rl = 0;  // last wave, lane k: challenge k
    for (u32 k0 = 0;; k0 += 3) {
        const u32 nr = L - k0 < 3 ? L - k0 : 3;
        const bool end = k0 + 3 >= L;
        // this wave's slot of entries 64 q + lane, q = half, half + 2, ... (at
        // most eight products below 2^124)
        if (64 * half < n) {
            u128 acc = 0;
            auto sums = [&](auto term) {  // term(a, f, e, on) of each entry
                for (u32 q = half; 64 * q < n; q += 2) {
                    const u32 e = 64 * q + lane;
                    const bool on = e < n;
                    acc += term(on ? A[base + e] : 0, on ? F[base + e] : 0, e, on);
                }
            };
            switch (slot) {
                case 0:
                    sums([&](u64 a, u64 f, u32 e, bool on) {
                        return fp::wide(a, f) + (on && hc ? Ct[base + e] : 0);
                    });
                    break;
                case 1:
                    sums([&](u64 a, u64 f, u32, bool) { return fp::wide(oct_factor<1>(lane, a), oct_factor<1>(lane, f)); });
                    break;
                case 2:
                    sums([&](u64 a, u64 f, u32, bool) { return fp::wide(oct_factor<2>(lane, a), oct_factor<2>(lane, f)); });
                    break;
                default:
                    sums([&](u64 a, u64 f, u32, bool) { return fp::wide(oct_factor<3>(lane, a), oct_factor<3>(lane, f)); });
                    break;
            }
            const u64 p = fp::red128(acc), v = reduced(plus32(plus16(p + from8(p))));
            if (lane < 8) part[half * T_ROW + 4 * lane + slot] = v;
        }
        if (w == NWAVES - 1) {  // the challenges (used after the sums are complete) and their fold's weights
            rl = draw_lanes(st, nr, k0, rl);
            u64 f[3];
#pragma unroll
            for (u32 k = 0; k < 3; k++)  // (entries past the level weigh 0)
                f[k] = fp::eqbit((lane >> k) & 1, k < nr ? lane_value(rl, k0 + k) : 0);
            const u64 x = mul(mul(f[0], f[1]), f[2]);
            if (lane < 8) s_w[lane] = x;
            if (end && lane < L) s_r[lane] = rl;
            if (end && lane == 0) *s_st = st;
        }
        __syncthreads();  // the sums of these rounds are complete
        if (tid >= SBLOCK - T_ROW) {  // (the last wave is idle in the fold)
            const u32 x = tid - (SBLOCK - T_ROW);
            cols[k0 / 3 * T_ROW + x] = n > 64 ? add(part[x], part[T_ROW + x]) : part[x];
        }
        const u32 lo = n > 8 ? 31 - (u32)__builtin_clz(n >> 3) : 0, no = 1u << lo;  // entries of the next level
        const u32 t = tid >> lo, o = tid & (no - 1);
        if (t < (end ? 1u : (hc ? 3u : 2u))) {  // F, A, C
            u64 *X = t == 0 ? F : (t == 1 ? A : Ct);
            u128 s = 0;
            if (n >= 8) {
                const u64 *src = X + base + 8 * o;
#pragma unroll
                for (u32 k = 0; k < 8; k += 2) {
                    const u64x2 x = ld2(src, k), wk = ld2(s_w, k);
                    s += fp::wide(wk.x, x.x) + fp::wide(wk.y, x.y);
                }
            } else {
                for (u32 k = 0; k < n; k++) s += fp::wide(s_w[k], X[base + k]);
            }
            X[end ? TAIL_TAB - 1 : base + n + o] = fp::red128(s);
        }
        __syncthreads();  // the next level is complete, the weights and partial sums are read
        if (end) break;
        base += n;
        n = no;
    }
    if (tid < L) {
        const u64 r = s_r[tid];
        pp.chals[c0 + tid] = r;
        if (rec) rec[tid] = r;
    }
    st = uniform(*s_st);
    if (tid == 0) {
        const u64 v = F[TAIL_TAB - 1];
        pp.rngst[c0 + L] = st;
        *vout = v;
        if (last == 1) pp.state[1] = v;
    }
    return st;
}

// HC: whether the phase has a C table, compile-time (one kernel each) or -1.
// After pend = 3 rounds this step finishes them itself: its first loads are
// issued before the wait for the challenge state.
template <int HC>
__device__ __forceinline__ void step_wtail(const WtailArgs &a, const ProofPtrs &pp, const Ctx c, u64 st_raw) {
    u64 *tab = c.lds;
    const u32 tid = threadIdx.x, lane = tid & 63;
    const bool hc = HC >= 0 ? HC != 0 : a.hasC != 0;
    const u32 L = a.sp - a.k0;  // 2^L entries of level k0, at most TAIL_LIM
    u64 st;
    if (a.pend) {
        Eight A = {}, F = {}, C = {};
        auto load = [&](u32 e) {
            if (e < a.live) {  // (the grid steps wrote level k0 - 3 below 8 live)
                A = ld8(a.A, e);
                F = ld8(a.F, e);
                if (hc) C = ld8(a.C, e);
            }
        };
        load(tid);
        st = uniform(st_raw);
        const u64 rl = draw_lanes(st, 3);
        u64 chi[8];
        chi8(rl, chi);
        if (tid < 3) pp.chals[a.c0 - 3 + lane] = rl;
#pragma unroll
        for (u32 i = 0; i < 2; i++) {
            const u32 e = tid + i * SBLOCK;
            if (i && (1u << L) > SBLOCK) load(e);
            if (e < (1u << L)) {
                const bool on = e < a.live;
                tab[e] = on ? fold3(A, chi) : 0;
                if (hc) tab[TAIL_TAB + e] = on ? fold3(C, chi) : 0;
                tab[2 * TAIL_TAB + e] = on ? fold3(F, chi) : 0;
            }
        }
    } else {
        for (u32 e = tid; e < (1u << L); e += SBLOCK) {
            const bool on = e < a.live;
            tab[e] = on ? a.A[e] : 0;
            if (hc) tab[TAIL_TAB + e] = on ? a.C[e] : 0;
            tab[2 * TAIL_TAB + e] = on ? a.F[e] : 0;
        }
        st = tail_state(pp, a.c0, 0, 0);
    }
    __syncthreads();
    wtail_rounds<HC>(tab, L, hc, st, a.cols, a.c0, a.last, a.vout, pp);
}

// A whole omega phase of a small layer in one workgroup: the eq table of
// the phase's point (a* in phase 1, b* in phase 2) into the workspace, the
// level-0 tables from the wiring (as ST_WA0 forms them) into LDS, then
// every round as a tail.
__device__ __forceinline__ void step_wsmall(const WsmallArgs &a, const ProofPtrs &pp, const Ctx c) {
    u64 *tab = c.lds;
    const u32 tid = threadIdx.x;
    {
        const u64 *pt = pp.chals + a.eqbase;
        const u64 nlo = 1ull << a.eqL, nhi = 1ull << (a.eqn - a.eqL);
        const u64 beta = pp.state[0];  // phase 1: a*'s lo half carries beta(z, a*)
        for (u64 x = tid; x < nlo + nhi; x += SBLOCK) {
            if (x < nlo)
                a.eqlo[x] = a.w.ph == 1 ? mul(beta, chi_bits(x, pt, a.eqL)) : chi_bits(x, pt, a.eqL);
            else
                a.eqhi[x - nlo] = chi_bits(x - nlo, pt + a.eqL, a.eqn - a.eqL);
        }
    }
    __syncthreads();  // the eq table is read back by this workgroup
    const Wa0Args &w = a.w;
    const bool hc = w.hasC != 0;
    const u64 v1 = w.ph == 2 ? pp.state[1] : 0;
    const u32 n = 1u << a.sp;
    for (u32 x = tid; x < n; x += SBLOCK) {
        u64 sA, sC, A, C;
        wire_sums(w, w.rowptr[x], w.rowptr[x + 1], sA, sC);
        level0(w.ph, v1, sA, sC, A, C);
        tab[x] = A;
        if (hc) tab[TAIL_TAB + x] = C;
        tab[2 * TAIL_TAB + x] = w.Vn[x];
    }
    const u64 st = tail_state(pp, a.c0, 0, 0);
    __syncthreads();
    wtail_rounds(tab, a.sp, hc, st, a.cols, a.c0, a.last, a.vout, pp);
}

// p-phase rounds in one workgroup over v, the level's 2^L <= TAIL_LIM entries
// (thread tid holds entries tid and tid + SBLOCK, 0 past the end).  The column
// sums of the first L - 5 rounds (see FIN_P: weights of the other five
// coordinates, one product an entry) are complete at a barrier; the entries
// are then folded by those rounds' challenges at once, and the 32 (or fewer)
// left are the last five rounds' column sums themselves.  Both go to cols;
// ST_FINISH forms the messages from them.  Lane off + k of every wave holds
// z of round k in zl and receives its challenge in rl; st becomes the state
// after them.  lds: PT_LDS words.  A round at a time (sums, barrier, fold,
// barrier, ten times) took 13.9 us a tail; this takes 6.5.
constexpr u32 PT_LDS = 32 * (3 + NWAVES);
__device__ __forceinline__ void ptail_rounds(const u64 (&v)[2], u32 L, u32 off, u64 zl, u64 &rl, u64 &st, u64 *cols,
                                             u64 *lds) {
    u64 *s_w = lds, *s_chi = lds + 32, *s_v = lds + 64, (*s_part)[32] = reinterpret_cast<u64 (*)[32]>(lds + 96);
    const u32 tid = threadIdx.x, lane = tid & 63;
    const u32 w = (u32)__builtin_amdgcn_readfirstlane((int)(tid >> 6));  // wave-uniform
    const u32 Ra = L > P_LAST ? L - P_LAST : 0, Rb = L - Ra, nc = 1u << Ra;
    if (Ra) {
        rl = draw_lanes(st, Ra, off, rl);  // used after the sums are complete
        if (w == 0 && lane < 32) {  // weights of the last coordinates (Rb = P_LAST)
            u64 f[P_LAST];
#pragma unroll
            for (u32 k = 0; k < P_LAST; k++) f[k] = fp::eqbit((lane >> k) & 1, lane_value(zl, off + Ra + k));
            s_w[lane] = mul(mul(mul(f[0], f[1]), mul(f[2], f[3])), f[4]);
        }
        if (w == NWAVES - 1 && lane < 32) {
            u64 f[P_LAST];
#pragma unroll
            for (u32 k = 0; k < P_LAST; k++) f[k] = k < Ra ? fp::eqbit((lane >> k) & 1, lane_value(rl, off + k)) : 1;
            s_chi[lane] = mul(mul(mul(f[0], f[1]), mul(f[2], f[3])), f[4]);
        }
        __syncthreads();
        u64 t = fp::red128(fp::wide(v[0], s_w[(tid >> Ra) & 31]) + fp::wide(v[1], s_w[((tid + SBLOCK) >> Ra) & 31]));
        for (u32 b = Ra; b < 6; b++) t = plus_bit(t, b);
        if (lane < nc) s_part[w][lane] = t;
        __syncthreads();  // the column sums are complete
        const u64 chi = s_chi[tid & (nc - 1)];
        u64 x[2] = {mul(chi, v[0]), mul(chi, v[1])};
        for (u32 b = 0; b < Ra; b++) {
            x[0] = plus_bit(x[0], b);
            x[1] = plus_bit(x[1], b);
        }
        if ((tid & (nc - 1)) == 0) {
            if (tid < (1u << L)) s_v[tid >> Ra] = x[0];
            if (tid + SBLOCK < (1u << L)) s_v[(tid + SBLOCK) >> Ra] = x[1];
        }
        if (tid < nc) {
            u64 s = 0;
#pragma unroll
            for (int q = 0; q < NWAVES; q++) s = add(s, s_part[q][tid]);
            cols[tid] = s;
        }
        __syncthreads();  // the last rounds' column sums are complete
        if (tid < 32) cols[32 + tid] = s_v[tid];
    } else if (tid < (1u << L)) {
        cols[32 + tid] = v[0];
    }
    rl = draw_lanes(st, Rb, off + Ra, rl);
}

// Remaining p-phase rounds j0..s-1 (ST_PTAIL), after pend = 3 rounds whose
// finish this step does itself (everything it reads is loaded before the first
// wait), or from round 0 (pend = 0).
__device__ __forceinline__ void step_ptail(const PtailArgs &a, const ProofPtrs &pp, Ctx c, u32 drew, u64 st0,
                                           u64 st_raw) {
    const u32 tid = threadIdx.x, lane = tid & 63, pend = a.pend;
    const u32 L = a.s - a.j0;  // 2^L entries of V^(j0), at most TAIL_LIM
    u64x2 p[2][4];
#pragma unroll
    for (u32 i = 0; i < 2; i++) {
        const u32 e = tid + i * SBLOCK;
#pragma unroll
        for (u32 k = 0; k < 4; k++) {
            p[i][k].x = p[i][k].y = 0;
            if (e < a.live) {
                if (pend)
                    p[i][k] = ld2(a.V, 8 * e + 2 * k);
                else if (k == 0)
                    p[i][k].x = a.V[e];
            }
        }
    }
    const u64 zl = lane < pend + L ? pp.zbuf[a.j0 - pend + lane] : 0;  // z of the pending rounds, then the tail's
    const u64 C0 = pp.state[0];
    u64 rl = 0, st, v[2];
    if (pend) {
        st = uniform(st_raw);
        rl = draw_lanes(st, 3);
        const u64 x = mul(mul(fp::eqbit(lane & 1, lane_value(rl, 0)), fp::eqbit((lane >> 1) & 1, lane_value(rl, 1))),
                          fp::eqbit((lane >> 2) & 1, lane_value(rl, 2)));
        u64 chi[8];  // one weight a lane, then scalars
#pragma unroll
        for (u32 e = 0; e < 8; e++) chi[e] = lane_value(x, e);
#pragma unroll
        for (u32 i = 0; i < 2; i++) {
            u128 t = 0;
#pragma unroll
            for (u32 k = 0; k < 4; k++) t += fp::wide(chi[2 * k], p[i][k].x) + fp::wide(chi[2 * k + 1], p[i][k].y);
            v[i] = fp::red128(t);
        }
    } else {
        st = tail_state(pp, a.c0, drew, st0);
        v[0] = p[0][0].x;
        v[1] = p[1][0].x;
    }
    ptail_rounds(v, L, pend, zl, rl, st, a.cols, c.lds);
    if (tid < 64) {
        const bool on = lane < pend + L;
        const u64 C = uniform(mul(C0, row_product(on ? fp::eq(zl, rl) : 1)));
        if (on) {
            pp.chals[a.c0 - pend + lane] = rl;
            a.rec[1 + lane] = zl;
        }
        if (tid == 0) {
            a.rec[0] = C0;
            pp.state[0] = C;  // beta(z, a*)
            pp.rngst[a.c0 + L] = st;
        }
    }
}

// ---------------------------------------------------------- line by folding
//
// h(t) = ~V_{i+1}(l(t)), l(t) = b* + t (c* - b*), is a polynomial of degree
// s' in t.  Folding V along the line coordinate by coordinate (bit k of the
// index, LSB first) turns each entry pair into a polynomial one degree
// higher: with D = P1 - P0 and d_k = c_k - b_k, the fold is
// P0(t) + (b_k + t d_k) D(t), whose coefficient j is P0_j + b_k D_j +
// d_k D_{j-1}.  After all s' folds the one polynomial left is h.  About four
// products an entry, against one per entry and line point for the sums over
// eq tables (ST_LT, ST_LINE), so wide layers take this path.  A thread folds
// 2^tb entries in registers (tb coordinates, 1 <= tb <= 5); the workgroup's 512
// polynomials of degree tb lose six more coordinates in LDS, two a level, one
// coefficient per work item; and the eight polynomials left, of degree
// tb + 6, are evaluated at t = 2..s', an item per point and polynomial, and
// weighted along every coordinate from tb + 6 on, prod_k (bit ? l_k(t) :
// 1 - l_k(t)) (a row of 16 lanes forms a point's weights beside the second
// and third level).  The workgroup's sums are written as a row (two rows: 16
// values a row); ST_FINISH adds the rows up.
// A workgroup's time is its chain of levels: nine levels of one coordinate,
// Horner's rule and the weights one after another took 10.2 us a launch at
// 2^17 entries, this takes 7.2 (27.1 -> 24.8 at 2^22, 73 -> 68 at 2^24).
constexpr u32 LF_POLYS = 8;  // polynomials left after the levels in LDS
constexpr u32 LF_LDS = 9;    // coordinates below a workgroup's in LDS: SBLOCK = 2^9 polynomials
static_assert((1 << LF_LDS) == SBLOCK && (SBLOCK >> 6) == LF_POLYS, "512 polynomials, three levels of two coordinates");

// The fold of a and b (degree D, in registers) into o (degree D + 1).
template <int D>
__device__ __forceinline__ void fold_poly(const u64 (&a)[D + 1], const u64 (&b)[D + 1], u64 bk, u64 dk,
                                          u64 (&o)[D + 2]) {
    u64 Dprev = 0;
#pragma unroll
    for (int j = 0; j <= D + 1; j++) {
        const int jj = j <= D ? j : D;  // (in range for the unrolled loads)
        const u64 Dj = j <= D ? diff_lz(b[jj], a[jj]) : 0;  // (< 2p: the sum stays below 2^125)
        const u64 a0 = j <= D ? a[jj] : 0;
        o[j] = fp::red128((u128)a0 + fp::wide(bk, Dj) + fp::wide(dk, Dprev));
        Dprev = Dj;
    }
}

template <int N, int D>
__device__ __forceinline__ void fold_level_reg(const u64 (&p)[N][D + 1], u64 (&q)[N / 2][D + 2], u64 bk, u64 dk) {
#pragma unroll
    for (int m = 0; m < N / 2; m++) fold_poly<D>(p[2 * m], p[2 * m + 1], bk, dk, q[m]);
}

// Two coordinates of the 4M polynomials of degree d at src folded into M of
// degree d + 2 at dst; coefficient j of polynomial m of n is word j n + m, so
// a work item reads a coefficient of its four polynomials in two 16-byte
// loads.  With l0, l1 the coordinates' lines, D0 = P1 - P0, D1 = P2 - P0 and
// D01 = P3 - P2 - P1 + P0, the fold is P0 + l0 D0 + l1 D1 + l0 l1 D01; e holds
// l0 l1's coefficients.
template <u32 M>
__device__ __forceinline__ void lds_fold2(const u64 *src, u64 *dst, u32 d, const u64 *b, const u64 *dl, const u64 *e) {
    const u64 b0 = b[0], d0 = dl[0], b1 = b[1], d1 = dl[1], e0 = e[0], e1 = e[1], e2 = e[2];
    for (u32 it = threadIdx.x; it < M * (d + 3); it += SBLOCK) {
        const u32 j = it / M, m = it % M;
        u64 p0 = 0, D0[2] = {0, 0}, D1[2] = {0, 0}, D01[3] = {0, 0, 0};
#pragma unroll
        for (u32 q = 0; q < 3; q++) {
            if (j < q || j - q > d) continue;
            const u64 *S = src + (j - q) * (4 * M) + 4 * m;
            const u64x2 lo = ld2(S, 0), hi = ld2(S, 2);
            if (q == 0) p0 = lo.x;
            if (q < 2) {
                D0[q] = diff_lz(lo.y, lo.x);  // (< 2p)
                D1[q] = diff_lz(hi.x, lo.x);
            }
            D01[q] = (hi.y + lo.x) + (2 * P - hi.x - lo.y);  // (< 4p)
        }
        // below 2^61 + 4 2^123 + 3 2^124 < 2^127
        dst[it] = fp::red128((u128)p0 + fp::wide(b0, D0[0]) + fp::wide(d0, D0[1]) + fp::wide(b1, D1[0]) +
                             fp::wide(d1, D1[1]) + fp::wide(e0, D01[0]) + fp::wide(e1, D01[1]) + fp::wide(e2, D01[2]));
    }
}

// Register levels D .. TB-1 of N polynomials of degree D; the one left
// (degree TB) goes to out, a coefficient every SBLOCK words.
template <int N, int D, int TB>
__device__ __forceinline__ void fold_regs(const u64 (&p)[N][D + 1], const u64 *bk, const u64 *dk, u64 *out) {
    if constexpr (D == TB) {
        static_assert(N == 1, "2^TB entries make one polynomial of degree TB");
#pragma unroll
        for (int j = 0; j <= TB; j++) out[j * SBLOCK] = p[0][j];
    } else {
        u64 q[N / 2][D + 2];
        fold_level_reg<N, D>(p, q, bk[D], dk[D]);
        fold_regs<N / 2, D + 1, TB>(q, bk, dk, out);
    }
}

template <int TB>
__device__ __forceinline__ void lfold_body(const LfoldArgs &a, const Ctx &c, i32 draw) {
    constexpr int E = 1 << TB;  // entries a thread folds
    u64 *bk = c.lds, *dk = bk + 32, *ee = dk + 32, *wt = ee + 16;  // l_k = b_k + t d_k; products of pairs; weights
    u64 *buf0 = wt + 32 * LF_POLYS, *buf1 = buf0 + SBLOCK * (TB + 1);  // 512 x (TB + 1), then 128 x (TB + 3) words
    const u32 tid = threadIdx.x;
    // the thread's entries (loaded before the line's coordinates are read)
    const u64 *src = a.V + ((u64)c.lb << (TB + LF_LDS)) + ((u64)tid << TB);
    u64 x[E][1];
#pragma unroll
    for (int e = 0; e < E; e += 2) {
        const u64x2 v = ld2(src, e);
        x[e][0] = v.x;
        x[e + 1][0] = v.y;
    }
    if (tid < a.sp) {  // (the challenge drawn by this launch's prologue is c.r, not yet in chals)
        const i32 bi = (i32)(a.bbase + tid), ci = (i32)(a.cbase + tid);
        const u64 b = bi == draw ? c.r : a.chals[bi], cc = ci == draw ? c.r : a.chals[ci];
        bk[tid] = b;
        dk[tid] = sub(cc, b);
    }
    __syncthreads();
    if (tid >= SBLOCK - 9) {  // coefficient i of l_k l_{k+1}, k = TB + 2 q
        const u32 q = (SBLOCK - 1 - tid) / 3, i = (SBLOCK - 1 - tid) % 3, k = TB + 2 * q;
        const u64 u = i == 2 ? dk[k] : bk[k], v = i ? dk[k + 1] : bk[k + 1];
        ee[3 * q + i] = fp::red128(fp::wide(u, v) + (i == 1 ? fp::wide(dk[k], bk[k + 1]) : 0));
    }
    fold_regs<E, 0, TB>(x, bk, dk, buf0 + tid);
    __syncthreads();
    lds_fold2<128>(buf0, buf1, TB, bk + TB, dk + TB, ee);
    __syncthreads();
    // Beside the second and third level, from the last row of lanes down: the
    // row of point t = 2 + pt multiplies the factors of the workgroup's own
    // bits, then each of its first eight lanes those of its polynomial's.
    const u32 T = a.sp - 1, pt = (SBLOCK - 1 - tid) / 16, l16 = tid % 16;
    constexpr u32 K8 = TB + 6, D = TB + LF_LDS;
    const auto factor = [&](u32 k, u32 bit, u64 t) { return fp::eqbit(bit, add(bk[k], mul(t, dk[k]))); };
    lds_fold2<32>(buf1, buf0, TB + 2, bk + TB + 2, dk + TB + 2, ee + 3);
    u64 w = 1;
    if (pt < T) {
        for (u32 k = D + l16; k < a.sp; k += 16) w = mul(w, factor(k, (c.lb >> (k - D)) & 1, pt + 2));
        w = row_product(w);
    }
    __syncthreads();
    lds_fold2<LF_POLYS>(buf0, buf1, TB + 4, bk + TB + 4, dk + TB + 4, ee + 6);
    if (pt < T && l16 < LF_POLYS) {
        const u64 f = mul(factor(K8, l16 & 1, pt + 2), factor(K8 + 1, (l16 >> 1) & 1, pt + 2));
        wt[pt * LF_POLYS + l16] = mul(mul(w, factor(K8 + 2, l16 >> 2, pt + 2)), f);
    }
    __syncthreads();
    const u32 tp = tid / LF_POLYS, m = tid % LF_POLYS;
    if (tp < T) {  // (whole octs of lanes)
        u64 pw = 1;  // t^j <= 32^11
        u128 v = 0;
#pragma unroll
        for (u32 j = 0; j <= K8; j++) {
            v += fp::wide(buf1[j * LF_POLYS + m], pw);
            pw *= tp + 2;
        }
        const u64 h = reduced(oct_total(mul(fp::red128(v), wt[tid])));
        if (m == 0) a.rows[((u64)(tp / ROW_STRIDE) * c.nb + c.lb) * ROW_STRIDE + tp % ROW_STRIDE] = h;
    }
}

// draw: the challenge index drawn by the launch's prologue (one round's
// finish at most: FIN_W or none), -1 if none.
__device__ __forceinline__ void step_lfold(const LfoldArgs &a, const Ctx &c, i32 draw) {
    switch (a.tb) {
        case 1: lfold_body<1>(a, c, draw); break;
        case 2: lfold_body<2>(a, c, draw); break;
        case 3: lfold_body<3>(a, c, draw); break;
        case 4: lfold_body<4>(a, c, draw); break;
        default: lfold_body<5>(a, c, draw); break;
    }
}

// ---------------------------------------------------------------- top layers
//
// ST_TOP runs the sum-check of the circuit's first layers in one
// workgroup, one layer after the other, as the tails run a phase: the
// p-phase over V_i, the two omega phases over A, C and F = V_{i+1}, and the
// line through b* and c*.  The tables stay in LDS between layers: the
// omega phases leave V_{i+1} as level 0 of F, which is the next layer's
// V_i, so global memory is read only for each V_{i+1} and the wiring and
// written only for messages, challenges and RNG states.  LDS areas (TAIL_TAB
// entries each): X holds the p-phase's sums, A (omega phases) and the line's point
// tables; Y holds C and, in its last 128 entries, the eq halves of a* and
// b* while the level-0 tables are formed; Z holds V_i, then F.

// lo[x] = chi_x(pt[0..L)) for x < 2^L and hi[x] = chi_x(pt[L..n)) for
// x < 2^(n-L), L = n / 2, so chi_x(pt) = lo[x mod 2^L] hi[x >> L].
__device__ __forceinline__ void eq_halves_lds(const u64 *pt, u32 n, u64 *lo, u64 *hi) {
    const u32 L = n / 2, nlo = 1u << L, nhi = 1u << (n - L);
    for (u32 x = threadIdx.x; x < nlo + nhi; x += SBLOCK) {
        if (x < nlo)
            lo[x] = chi_bits(x, pt, L);
        else
            hi[x - nlo] = chi_bits(x - nlo, pt + L, n - L);
    }
}

// Level 0 of omega phase ph of a top layer: wire x's gates (one chunk)
// summed as wire_sums sums them, with chi_g(a*) and (phase 2)
// chi_in1(b*) from the eq halves in LDS and phase 1's operand V_{i+1}[in2]
// from F in LDS.
__device__ __forceinline__ void top_level0(const TopLayer &Ld, u32 ph, u64 beta, u64 v1, const u64 *ea, u32 La,
                                           const u64 *eb, u32 Lb, const u64 *F, u64 *A, u64 *C, bool hc) {
    const u32 N = 1u << Ld.sp, q = ph - 1;
    const u32 *rowptr = Ld.rowptr[q], *perm = Ld.perm[q], *oths = Ld.oths[q];
    const u8 *types = Ld.types[q];
    const u32 amask = (1u << La) - 1, bmask = (1u << Lb) - 1;
    const u64 *ea_hi = ea + 32, *eb_hi = eb + 32;
    for (u32 x = threadIdx.x; x < N; x += SBLOCK) {
        u64 sA = 0, sC = 0;
        const u32 p0 = rowptr[x], p1 = rowptr[x + 1];
        for (u32 p = p0; p < p1; p++) {
            const u32 g = perm[p], o = oths[p];
            const bool ismul = Ld.kind == 1 || (Ld.kind == 2 && types[p]);  // MUL, or a MUL gate of a mixed layer
            u64 w = mul(beta, mul(ea[g & amask], ea_hi[g >> La]));
            if (ph == 1) {
                const u64 wy = mul(w, F[o]);
                sA = add(sA, ismul ? wy : w);
                sC = add(sC, ismul ? 0 : wy);
            } else {
                w = mul(w, mul(eb[o & bmask], eb_hi[o >> Lb]));
                sA = add(sA, ismul ? 0 : w);
                sC = add(sC, ismul ? w : 0);
            }
        }
        u64 a, c;
        level0(ph, v1, sA, sC, a, c);
        A[x] = a;
        if (hc) C[x] = c;
    }
}

// The line of a top layer: h(t) = ~V_{i+1}(l(t)) for t = 2..sp, l(t) =
// b* + t (c* - b*), over level 0 of F.  The eq halves of point t go to
// tb + 64 (t - 2) (lo, 32 entries) and 32 past it (hi); wave w sums points
// t - 2 = w, w + NWAVES, ..., each lane adding hi lo V over every 64th
// entry in 128 bits, and lane 63 writes h(t) to out[t - 2].
__device__ __forceinline__ void top_line(u32 sp, const u64 *bst, const u64 *cst, const u64 *F, u64 *tb, u64 *out) {
    const u32 T = sp - 1, Ll = sp / 2, Lh = sp - Ll;
    for (u32 e = threadIdx.x; e < T * 64; e += SBLOCK) {
        const u32 tp = e >> 6, j = e & 63;
        const u64 t = tp + 2;
        const bool lo = j < 32;
        const u32 x = lo ? j : j - 32, nb = lo ? Ll : Lh, base = lo ? 0 : Ll;
        if (x < (1u << nb)) {
            u64 v = 1;
            for (u32 k = 0; k < nb; k++) {
                const u64 b = bst[base + k], c = cst[base + k];
                v = mul(v, fp::eqbit((x >> k) & 1, add(b, mul(t, sub(c, b)))));
            }
            tb[e] = v;
        }
    }
    __syncthreads();
    const u32 lane = threadIdx.x & 63;
    const u32 w = (u32)__builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));  // wave-uniform
    const u32 N = 1u << sp, m = (1u << Ll) - 1;
    for (u32 tp = w; tp < T; tp += NWAVES) {
        const u64 *lo = tb + 64 * tp, *hi = lo + 32;
        u128 acc = 0;  // at most 16 products below 2^122
        for (u32 x = lane; x < N; x += 64) acc += fp::wide(hi[x >> Ll], mul(lo[x & m], F[x]));
        const u64 v = wave_sum63(fp::red128(acc));
        if (lane == 63) out[tp] = v;
    }
}

__device__ __forceinline__ void step_top(const TopArgs &a, const ProofPtrs &pp, const Ctx c) {
    __shared__ u64 s_r[3 * TAIL_LOG];  // the layer's challenges: a*, then b*, then c*
    __shared__ u64 s_st;
    u64 *tab = c.lds;
    u64 *X = tab, *Y = tab + TAIL_TAB, *Z = tab + 2 * TAIL_TAB;
    u64 *eqa = Y + TAIL_TAB - 128, *eqb = eqa + 64;  // eq halves: lo in [0, 32), hi in [32, 64)
    const u32 tid = threadIdx.x, lane = tid & 63;
    // Evaluation of the layers, nl - 1 down to 0, each from the one below it
    // in LDS (X and Y in turn; Z is not touched), every table also written
    // to memory as ST_EVAL writes it.
    {
        const TopLayer &Lk = a.L[a.nl - 1];
        u64 *src = X, *dst = Y;
        for (u32 e = tid; e < (1u << Lk.sp); e += SBLOCK) src[e] = Lk.Vn[e];
        __syncthreads();
        for (u32 i = a.nl; i-- > 0;) {
            const TopLayer &Ld = a.L[i];
            for (u32 g = tid; g < (1u << Ld.s); g += SBLOCK) {
                u64 v = 0;
                if (g < Ld.S) {
                    const u64 x = src[Ld.in1[g]], y = src[Ld.in2[g]];
                    const bool ismul = Ld.kind == 1 || (Ld.kind == 2 && Ld.type[g]);
                    v = ismul ? mul(x, y) : add(x, y);
                }
                dst[g] = v;
                Ld.V[g] = v;
            }
            __syncthreads();
            u64 *t = src;
            src = dst;
            dst = t;
        }
        // the start (as ST_START): z_0 from the seed's stream, the outputs
        // (V_0, now in src) into the transcript
        const TopLayer &L0 = a.L[0];
        if (tid == 0) {
            u64 st = fp::sm_state(pp.state[2], fp::PURPOSE_GKR);  // state[2] = seed
            pp.rngst[0] = st;
            for (u32 k = 0; k < L0.s; k++) {
                const u64 z = fp::sm_field(st);
                pp.chals[k] = z;
                pp.zbuf[k] = z;
                pp.rngst[k + 1] = st;
            }
            pp.state[0] = 1;
            pp.state[1] = 0;
        }
        for (u32 g = tid; g < L0.S; g += SBLOCK) pp.msgs[g] = src[g];
        __syncthreads();  // the tables, z_0 and the RNG state are read back below
    }
    // V_0, z_0 and the RNG state of the start
    {
        const TopLayer &L0 = a.L[0];
        for (u32 e = tid; e < (1u << L0.s); e += SBLOCK) Z[e] = a.V0[e];
        if (tid == 0) s_st = pp.rngst[L0.co];
    }
    u64 zr = lane < a.L[0].s ? pp.zbuf[lane] : 0;  // z_l of the layer in lane l
    __syncthreads();
    u64 st = uniform(s_st);
    for (u32 i = 0; i < a.nl; i++) {
        const TopLayer &Ld = a.L[i];
        const u32 s = Ld.s, sp = Ld.sp, n = s + 2 * sp, N = 1u << sp;
        const bool hc = Ld.kind != 1;  // a layer with ADD gates has a C table
        // p-phase over V_i (level 0 of Z); beta starts at 1
        u64 beta = 1;
        if (s > 0) {
            u64 v[2], rl = 0;
#pragma unroll
            for (u32 e = 0; e < 2; e++) v[e] = tid + e * SBLOCK < (1u << s) ? Z[tid + e * SBLOCK] : 0;
            ptail_rounds(v, s, 0, zr, rl, st, Ld.cols, X);
            beta = uniform(row_product(lane < s ? fp::eq(zr, rl) : 1));
            if (tid < s) {
                pp.chals[Ld.co + tid] = s_r[tid] = rl;
                Ld.rec[1 + tid] = zr;
            }
            if (tid == 0) Ld.rec[0] = 1;
        }
        __syncthreads();  // the p-phase's reads of Z are done
        // phase 1: F = V_{i+1} into Z, A and C from the gates on in1
        for (u32 e = tid; e < N; e += SBLOCK) Z[e] = Ld.Vn[e];
        eq_halves_lds(s_r, s, eqa, eqa + 32);
        __syncthreads();
        top_level0(Ld, 1, beta, 0, eqa, s / 2, eqb, 0, Z, X, Y, hc);
        __syncthreads();
        st = wtail_rounds(tab, sp, hc, st, Ld.wcols[0], Ld.co + s, 1, Ld.msg + 3 * n, pp, s_r + s);
        const u64 v1 = Z[TAIL_TAB - 1];  // F bound in every variable
        __syncthreads();  // phase 1's partial sums are read; its tree in Y is no longer needed
        // phase 2: the gates on in2, with v1
        eq_halves_lds(s_r, s, eqa, eqa + 32);
        eq_halves_lds(s_r + s, sp, eqb, eqb + 32);
        __syncthreads();
        top_level0(Ld, 2, beta, v1, eqa, s / 2, eqb, sp / 2, Z, X, Y, hc);
        __syncthreads();
        st = wtail_rounds(tab, sp, hc, st, Ld.wcols[1], Ld.co + s + sp, 2, Ld.msg + 3 * n + 1, pp, s_r + s + sp);
        __syncthreads();
        // the line (level 0 of Z is still V_{i+1}); its point tables in X
        if (sp >= 2) {
            top_line(sp, s_r + s, s_r + s + sp, Z, X, Ld.msg + 3 * n + 2);
            __syncthreads();
        }
        // tau and z_{i+1} = l(tau) for the next layer of this step (the
        // step after it draws the last layer's tau)
        if (i + 1 < a.nl) {
            const u64 tau = fp::sm_field(st);
            if (tid == 0) {
                pp.chals[Ld.co + n] = tau;
                pp.rngst[Ld.co + n + 1] = st;
            }
            const u64 b = lane < sp ? s_r[s + lane] : 0, c = lane < sp ? s_r[s + sp + lane] : 0;
            zr = add(b, mul(tau, sub(c, b)));
            __syncthreads();  // s_r is read before the next layer records into it
        }
    }
}

// ---------------------------------------------------------------- kernel

// One step on workgroup lb.  Workgroups [0, nblocks) run the body; a step
// that finishes the previous round has one more workgroup, lb == nblocks,
// which only folds the previous rows into the message (so that work runs
// beside the body instead of ahead of it) and records the drawn challenge.
template <u32 KIND, int GK, int PH>
__device__ __forceinline__ void run_step(const StepDesc &sd, u32 lb, u64 *lds) {
    __shared__ u64 s_pt[64];  // a point (EQ), or b* and c* (LT), or z_{i+1} (FIN_LINE)
    const Fin &f = sd.fin;
    const ProofPtrs &pp = sd.pp;
    const u32 kind = KIND == KALL ? sd.kind : KIND;
    const bool tail = kind == ST_WTAIL || kind == ST_PTAIL || kind == ST_WSMALL ||
                      kind == ST_TOP;  // one workgroup does everything
    const bool has_fin = f.kind != FIN_NONE;
    const bool split = has_fin && !tail;  // workgroup nblocks finishes, the others run the body
    const bool fin_block = split && lb == sd.nblocks;
    const bool recorder = split ? fin_block : lb == 0;
    Ctx c;
    c.lds = lds;
    c.lb = lb;
    c.nb = sd.nblocks;
    c.gtid = (u64)c.lb * SBLOCK + threadIdx.x;
    c.gstride = (u64)c.nb * SBLOCK;

    // --- prologue: the challenge.  Every thread of every workgroup draws the
    // same value from the state in memory (a uniform load), so nothing waits
    // for a barrier before the body's first loads.
    u64 st_after = 0;
    c.r = 0;
    c.rl = 0;
    const u64 st_raw = f.draw >= 0 ? pp.rngst[f.draw] : 0;
    auto draw = [&]() {
        if (f.draw < 0) return;
        u64 st = uniform(st_raw);
        const u32 nd = f.kind == FIN_T ? 3 : ((fin_mask(KIND) & (1u << FIN_P)) && f.kind == FIN_P ? f.R : 1);
        c.rl = draw_lanes(st, nd);
        c.r = lane_value(c.rl, 0);
        if (recorder && threadIdx.x < nd) pp.chals[f.draw + threadIdx.x] = c.rl;
        if (recorder && threadIdx.x == 0) pp.rngst[f.draw + nd] = st;
        st_after = st;  // the state after the drawn challenge(s)
    };
    // a tail finishes the rounds before it itself; a table step's body and a
    // later p-phase step's draw after issuing their loads
    const bool own_fin = tail && (f.kind == FIN_P || f.kind == FIN_T);
    const bool pfirst = (KIND == ST_P || KIND == KALL) && kind == ST_P && sd.u.p.pend == 0;
    const bool late = own_fin || (((kind == ST_P && !pfirst) || kind == ST_WT) && !fin_block);
    const bool line_fin = (fin_mask(KIND) & (1u << FIN_LINE)) && f.kind == FIN_LINE;
    u64 bb = 0, cc = 0;
    auto line_points = [&]() {
        if (line_fin && threadIdx.x < f.sp) {
            bb = f.bstar[threadIdx.x];
            cc = f.cstar[threadIdx.x];
        }
    };
    if (KIND != KALL) line_points();  // (the kernel of every kind would spill more)
    Runs px = {};
    if (KIND == ST_P && GK == 1 && !fin_block) px = load_runs(sd.u.p, c, lb, runs_from(sd.u.p, c, lb));
    if (!late) draw();
    TailIn ti = {st_after, f.draw >= 0 ? 1u : 0u};
    // points assembled in LDS (challenges drawn by earlier launches are in
    // chals; the one drawn just now is c.r)
    if (line_fin || kind == ST_EQ || kind == ST_LT || pfirst) {  // (uniform)
        if (KIND == KALL) line_points();
        if (line_fin && threadIdx.x < f.sp)
            s_pt[threadIdx.x] = add(bb, mul(c.r, sub(cc, bb)));  // z_{i+1} = l(tau)
        if (pfirst && !line_fin && threadIdx.x < sd.u.p.s)
            s_pt[threadIdx.x] = pp.zbuf[threadIdx.x];  // z of the layer, already recorded
        if (kind == ST_EQ && threadIdx.x < sd.u.eq.n) {
            const i32 ci = (i32)(sd.u.eq.base + threadIdx.x);
            s_pt[threadIdx.x] = ci == f.draw ? c.r : pp.chals[ci];
        }
        if (kind == ST_LT && threadIdx.x < 2 * sd.u.lt.sp) {
            const u32 sp = sd.u.lt.sp;
            const i32 ci = (i32)(threadIdx.x < sp ? sd.u.lt.bbase + threadIdx.x
                                                  : sd.u.lt.cbase + threadIdx.x - sp);
            s_pt[threadIdx.x] = ci == f.draw ? c.r : pp.chals[ci];
        }
        __syncthreads();
    }
    if (fin_block || (tail && has_fin && !own_fin)) {
        fin_inline<KIND>(sd, c, s_pt);
        if (fin_block) return;
    }
    if (tail && has_fin) {
        if ((fin_mask(KIND) & (1u << FIN_LINE)) && f.kind == FIN_LINE) __syncthreads();  // z_{i+1} stored
    }

    // --- body
    u64 *row = sd.rows ? sd.rows + (u64)c.lb * ROW_STRIDE : nullptr;
    u64 *trow = sd.rows + (u64)c.lb * T_ROW;  // of table rounds
    switch (kind) {
        case ST_LOAD: step_load(sd.u.load, pp, c); break;
        case ST_EVAL: step_eval(sd.u.eval, c); break;
        case ST_START: step_start(sd.u.start, pp, c); break;
        case ST_EQ:
            step_eq(sd.u.eq, c, s_pt, pp);
            break;
        case ST_P:
            step_p<KIND == ST_P ? GK : -1>(sd.u.p, c, pfirst ? s_pt : pp.zbuf,
                                           sd.rows + ((u64)c.lb << sd.u.p.R), draw, px);
            break;
        case ST_W: {
            const WArgs &a = sd.u.w;
            if (GK >= 0) {
                step_w<GK < 0 ? 0 : GK, PH < 1 ? 1 : PH>(a, c, pp, row);
            } else if (a.ph == 1) {
                if (a.kind == 0) step_w<0, 1>(a, c, pp, row);
                else if (a.kind == 1) step_w<1, 1>(a, c, pp, row);
                else step_w<2, 1>(a, c, pp, row);
            } else {
                if (a.kind == 0) step_w<0, 2>(a, c, pp, row);
                else if (a.kind == 1) step_w<1, 2>(a, c, pp, row);
                else step_w<2, 2>(a, c, pp, row);
            }
            break;
        }
        case ST_FOLD: step_fold(sd.u.fold, c); break;
        case ST_LT: step_lt(sd.u.lt, c, s_pt, s_pt + sd.u.lt.sp); break;
        case ST_LINE: step_line(sd.u.line, c, row); break;
        case ST_WAGG: step_wagg<KIND == ST_WAGG ? GK : -1, KIND == ST_WAGG ? PH : 0>(sd.u.wagg, pp, c); break;
        case ST_WT0: step_wt0(sd.u.wt0, pp, c, trow); break;
        case ST_WA0: step_wa0<KIND == ST_WA0 ? GK : -1, KIND == ST_WA0 ? PH : 0>(sd.u.wa0, pp, c, trow); break;
        case ST_WT: step_wt<KIND == ST_WT ? GK : -1>(sd.u.wt, c, trow, draw); break;
        case ST_WTAIL: step_wtail<KIND == ST_WTAIL ? GK : -1>(sd.u.wtail, pp, c, st_raw); break;
        case ST_PTAIL: step_ptail(sd.u.ptail, pp, c, ti.drew, ti.st, st_raw); break;
        case ST_FINISH: step_finish(sd.u.finish, c); break;
        case ST_WSMALL: step_wsmall(sd.u.wsmall, pp, c); break;
        case ST_TOP: step_top(sd.u.top, pp, c); break;
        case ST_LFOLD: step_lfold(sd.u.lfold, c, f.draw); break;
        case ST_SGE:
            if (c.lb == 0 && threadIdx.x == 0) {
                const u64 v = sd.u.sge.Vn[0];
                sd.u.sge.vslot[0] = v;
                sd.u.sge.vslot[1] = v;
                pp.state[1] = v;
            }
            break;
        default: break;
    }
}

// LDS words of a kind's body (the kernel of mixed batches holds every kind's
// code, and its LDS decides how many workgroups a CU takes).
constexpr u32 TAIL_WORDS = 3 * TAIL_TAB + TAIL_EXTRA, LFOLD_WORDS = 80 + 32 * LF_POLYS + SBLOCK * 6 + 128 * 8;
constexpr u32 lds_words(u32 kind) {
    return kind == ST_P       ? 64 + NWAVES * 64
           : kind == ST_PTAIL ? PT_LDS
           : kind == ST_FINISH ? SBLOCK
           : kind == ST_LINE   ? 64 * LINE_CHUNK
           : kind == ST_LFOLD  ? LFOLD_WORDS
           : kind == ST_WA0 ? NWAVES * T_ROW + 6 * EQ_THIRD + NWAVES * GRAM_WORDS
           : kind == ST_WT0 || kind == ST_WT ? NWAVES * T_ROW
           : kind == ST_WTAIL || kind == ST_WSMALL || kind == ST_TOP ? TAIL_WORDS
           : kind == KALL ? (TAIL_WORDS > LFOLD_WORDS ? TAIL_WORDS : LFOLD_WORDS)
                          : 2;
}
static_assert(64 + NWAVES * 64 >= (1 << P_ROUNDS) + NWAVES * 8, "lds_words");

// A single proof's step, its descriptor passed by value as kernel argument;
// one instantiation per step kind (and per gate mix and phase for omega
// rounds) keeps each kernel's code and registers to what the kind needs.
template <u32 KIND, int GK, int PH>
__global__ void __launch_bounds__(SBLOCK, 4) k_step_one(const StepDesc sd) {
    __shared__ __align__(16) u64 lds[lds_words(KIND)];
    run_step<KIND, GK, PH>(sd, blockIdx.x, lds);
}

// One step of each of several proofs.
__global__ void __launch_bounds__(SBLOCK, 4) k_step_jobs(const JobEntry *__restrict__ jobs, u32 njobs) {
    u32 lo = 0, hi = njobs;
    const u32 b = blockIdx.x;
    while (hi - lo > 1) {
        const u32 mid = (lo + hi) >> 1;
        if (jobs[mid].block0 <= b) lo = mid; else hi = mid;
    }
    __shared__ __align__(16) u64 lds[lds_words(KALL)];
    run_step<KALL, -1, 0>(*jobs[lo].step, b - jobs[lo].block0, lds);
}

// One step of each of several proofs, the job table in the kernel arguments.
__global__ void __launch_bounds__(SBLOCK, 4) k_step_table(const JobTable t) {
    u32 lo = 0, hi = t.n;
    const u32 b = blockIdx.x;
    while (hi - lo > 1) {
        const u32 mid = (lo + hi) >> 1;
        if (t.e[mid].block0 <= b) lo = mid; else hi = mid;
    }
    __shared__ __align__(16) u64 lds[lds_words(KALL)];
    run_step<KALL, -1, 0>(*t.e[lo].step, b - t.e[lo].block0, lds);
}

hipError_t launch_step_table(hipStream_t st, const JobTable &t) {
    hipLaunchKernelGGL(k_step_table, dim3(t.total), dim3(SBLOCK), 0, st, t);
    return hipGetLastError();
}

u32 step_grid(const StepDesc &sd) {
    if (sd.kind == ST_WTAIL || sd.kind == ST_PTAIL || sd.kind == ST_WSMALL || sd.kind == ST_TOP) return 1;
    return sd.nblocks + (sd.fin.kind != FIN_NONE ? 1 : 0);
}

hipError_t launch_step(hipStream_t st, const StepDesc &sd, hipEvent_t ev0, hipEvent_t ev1) {
    const dim3 g(step_grid(sd)), b(SBLOCK);
    // with events: the dispatch itself is timed (hipExtLaunchKernelGGL)
#define L1(K) hipExtLaunchKernelGGL((k_step_one<K, -1, 0>), g, b, 0, st, ev0, ev1, 0, sd)
#define LW(G, PH) hipExtLaunchKernelGGL((k_step_one<ST_W, G, PH>), g, b, 0, st, ev0, ev1, 0, sd)
#define LK(K, G, PH) hipExtLaunchKernelGGL((k_step_one<K, G, PH>), g, b, 0, st, ev0, ev1, 0, sd)
    switch (sd.kind) {
        case ST_LOAD: L1(ST_LOAD); break;
        case ST_EVAL: L1(ST_EVAL); break;
        case ST_START: L1(ST_START); break;
        case ST_EQ: L1(ST_EQ); break;
        case ST_P:  // one kernel for the phase's first step, one for the others
            if (sd.u.p.pend == 0) LK(ST_P, 1, 0); else LK(ST_P, 0, 0);
            break;
        case ST_W:
            if (sd.u.w.ph == 1) {
                if (sd.u.w.kind == 0) LW(0, 1); else if (sd.u.w.kind == 1) LW(1, 1); else LW(2, 1);
            } else {
                if (sd.u.w.kind == 0) LW(0, 2); else if (sd.u.w.kind == 1) LW(1, 2); else LW(2, 2);
            }
            break;
        case ST_FOLD: L1(ST_FOLD); break;
        case ST_LT: L1(ST_LT); break;
        case ST_LINE: L1(ST_LINE); break;
        case ST_SGE: L1(ST_SGE); break;
        case ST_WAGG: {  // one kernel per gate mix and phase
            const u32 k = sd.u.wagg.kind, ph = sd.u.wagg.ph;
            if (ph == 1) {
                if (k == 0) LK(ST_WAGG, 0, 1); else if (k == 1) LK(ST_WAGG, 1, 1); else LK(ST_WAGG, 2, 1);
            } else {
                if (k == 0) LK(ST_WAGG, 0, 2); else if (k == 1) LK(ST_WAGG, 1, 2); else LK(ST_WAGG, 2, 2);
            }
            break;
        }
        case ST_WT0: L1(ST_WT0); break;
        case ST_WA0: {  // one kernel per gate mix and phase
            const u32 k = sd.u.wa0.kind, ph = sd.u.wa0.ph;
            if (ph == 1) {
                if (k == 0) LK(ST_WA0, 0, 1); else if (k == 1) LK(ST_WA0, 1, 1); else LK(ST_WA0, 2, 1);
            } else {
                if (k == 0) LK(ST_WA0, 0, 2); else if (k == 1) LK(ST_WA0, 1, 2); else LK(ST_WA0, 2, 2);
            }
            break;
        }
        case ST_WT:  // one kernel with a C table, one without
            if (sd.u.wt.hasC) LK(ST_WT, 1, 0); else LK(ST_WT, 0, 0);
            break;
        case ST_WTAIL:  // one kernel with a C table, one without
            if (sd.u.wtail.hasC) LK(ST_WTAIL, 1, 0); else LK(ST_WTAIL, 0, 0);
            break;
        case ST_PTAIL: L1(ST_PTAIL); break;
        case ST_FINISH: L1(ST_FINISH); break;
        case ST_WSMALL: L1(ST_WSMALL); break;
        case ST_TOP: L1(ST_TOP); break;
        case ST_LFOLD: L1(ST_LFOLD); break;
        default: L1(ST_END); break;
    }
#undef L1
#undef LW
#undef LK
    return hipGetLastError();
}

hipError_t launch_steps(hipStream_t st, const JobEntry *jobs, u32 njobs, u32 total_blocks,
                        hipEvent_t ev0, hipEvent_t ev1) {
    hipExtLaunchKernelGGL(k_step_jobs, dim3(total_blocks), dim3(SBLOCK), 0, st, ev0, ev1, 0, jobs, njobs);
    return hipGetLastError();
}

// ------------------------------------------------------------- batches

// Proof q's seed and input pointer into its state; range flag cleared.
__global__ void k_batch_setup(const BatchSlot *slots, u32 n) {
    const u32 q = blockIdx.x * blockDim.x + threadIdx.x;
    if (q < n) {
        u64 *st = slots[q].state;
        st[2] = slots[q].seed;
        st[3] = slots[q].input;
        st[4] = 0;
    }
}

// Transcripts (and range flags) of the batch into one contiguous buffer:
// proof q's msgs at out[slots[q].out_off ...], its flag at out[slots[q].flag_off].
// A workgroup copies GATHER words at a time, blockIdx.x the proof (one
// workgroup a proof took 460 us for 6 MB).
constexpr u32 GATHER = 2048;
__global__ void k_batch_gather(const BatchSlot *slots, u32 n, u64 *out) {
    const BatchSlot &s = slots[blockIdx.x];
    for (u64 k0 = (u64)blockIdx.y * GATHER; k0 < s.n_msgs; k0 += (u64)gridDim.y * GATHER) {
        const u64 k1 = k0 + GATHER < s.n_msgs ? k0 + GATHER : s.n_msgs;
        for (u64 k = k0 + threadIdx.x; k < k1; k += blockDim.x) out[s.out_off + k] = s.msgs[k];
    }
    if (blockIdx.y == 0 && threadIdx.x == 0) out[s.flag_off] = s.state[4];
}

hipError_t launch_batch_setup(hipStream_t st, const BatchSlot *slots, u32 n) {
    hipLaunchKernelGGL(k_batch_setup, dim3((n + 255) / 256), dim3(256), 0, st, slots, n);
    return hipGetLastError();
}

hipError_t launch_batch_gather(hipStream_t st, const BatchSlot *slots, u32 n, u64 most_msgs, u64 *out) {
    const u64 nb = (most_msgs + GATHER - 1) / GATHER;
    hipLaunchKernelGGL(k_batch_gather, dim3(n, (u32)(nb < 1 ? 1 : nb > 1024 ? 1024 : nb)), dim3(256), 0, st, slots, n, out);
    return hipGetLastError();
}

}  // namespace gkr

// f2sc.hip -- the interactive F2 sum-check's prover on gfx950 (Sec. 3.2,
// Sec. 7): G_j(t) = sum_m ((1-t) A[2m] + t A[2m+1])^2 over the table A folded
// by the earlier challenges.
//
// Three rounds a pass.  Before r_j is known, the sums of rounds j, j+1 and
// j+2 are quadratic forms in the challenges whose coefficients are the Gram
// matrix M[x][y] = sum over octs of A[8o + x] A[8o + y] of the level-j table
// (x, y < 8: the three variables the rounds bind).  A pass folds the level
// three below by its three challenges, stores the level (one eighth of what
// it read) and sums the Gram matrix of its octs; the next launch draws the
// three challenges, after every sum of theirs is complete, and one workgroup
// of it turns the rows into the nine message values beside the body.  Against
// a launch per round this reads every level once per three rounds and stores
// an eighth of it instead of a half: for 2^26 counts 0.7 GB move instead of
// 1.6 GB, in 6 launches instead of 16 (proof 412 -> 180 us; 2^10 counts,
// one launch instead of four and no copies, 42 -> 25 us).
#include "f2sc.hpp"
#include "lanes.hpp"

namespace gkr {

using fp::add;
using fp::mul;
using fp::P;
using fp::sub;
using fp::u128;

namespace {

constexpr int FB = 512;           // threads per workgroup
constexpr int FW = FB / 64;       // waves
constexpr int OCT = 8;            // lanes sharing an oct, one entry each
constexpr int SLOTS = 5;          // Gram sums a lane keeps
static_assert(OCT * SLOTS == F2SC_ROW, "a row holds every lane's slots");

// The 36 products of an oct over its eight lanes: lane j takes the partners
// j, j ^ (1 or 3), j ^ (2 or 6), j ^ (4 or 5), j ^ 7, the first of each pair
// where j lacks that bit, so that every unordered pair of lanes is taken once
// (slot 4 twice: only lanes without bit 0 are read).
__device__ __forceinline__ void gram_add(u32 j, u64 v, u128 (&acc)[SLOTS]) {
    // (every lane takes part in every exchange; the selects come after)
    const u64 v1 = from1(v), v2 = from2(v), v3 = from3(v), v7 = from7(v);
    const u64 v6 = from1(v7), v5 = from2(v7), v4 = from3(v7);  // j ^ 6 = (j ^ 7) ^ 1, ...
    const u64 o1 = j & 1 ? v3 : v1, o2 = j & 2 ? v6 : v2, o3 = j & 4 ? v5 : v4;
    acc[0] += fp::wide(v, v);
    acc[1] += fp::wide(v, o1);
    acc[2] += fp::wide(v, o2);
    acc[3] += fp::wide(v, o3);
    acc[4] += fp::wide(v, v7);
}

// Where M[x][y] sits among the 40 slots of a row.
__device__ __forceinline__ u32 gram_slot(u32 x, u32 y) {
    const u32 d = x ^ y;
    u32 s, j;
    if (d == 0) {
        s = 0, j = x;
    } else if (d == 1 || d == 3) {
        s = 1, j = (x & 1) == (d == 3 ? 1u : 0u) ? x : y;
    } else if (d == 2 || d == 6) {
        s = 2, j = ((x >> 1) & 1) == (d == 6 ? 1u : 0u) ? x : y;
    } else if (d == 4 || d == 5) {
        s = 3, j = ((x >> 2) & 1) == (d == 5 ? 1u : 0u) ? x : y;
    } else {
        s = 4, j = x & 1 ? y : x;
    }
    return j * SLOTS + s;
}

// chi_e(r) of lane e's three bits: the weight of entry e in a fold by three challenges.
__device__ __forceinline__ u64 chi3(u32 e, const u64 (&r)[3]) {
    return mul(mul(fp::eqbit(e & 1, r[0]), fp::eqbit((e >> 1) & 1, r[1])), fp::eqbit((e >> 2) & 1, r[2]));
}

struct Weights {
    u64 w[OCT];
};
__device__ __forceinline__ Weights fold_weights(const u64 (&r)[3]) {
    const u64 mine = chi3(threadIdx.x & 7, r);  // one weight a lane, then scalars
    Weights q;
#pragma unroll
    for (int e = 0; e < OCT; e++) {
        const u32 lo = (u32)__builtin_amdgcn_readlane((int)(u32)mine, e);
        const u32 hi = (u32)__builtin_amdgcn_readlane((int)(u32)(mine >> 32), e);
        q.w[e] = ((u64)hi << 32) | lo;
    }
    return q;
}

// Four counts in one 16-byte load; the caller's vector may start at any count,
// so nothing beyond 4-byte alignment is promised (the load is the same
// instruction either way).
__device__ __forceinline__ uint4 counts4(const u32 *p) {
    uint4 v;
    __builtin_memcpy(&v, p, sizeof v);
    return v;
}

// Entry g of a level from the eight entries below it.
__device__ __forceinline__ u64 fold8(const u32 *src, u64 g, const Weights &q) {
    const uint4 a = counts4(src + OCT * g), b = counts4(src + OCT * g + 4);
    return fp::red128(fp::wide(q.w[0], a.x) + fp::wide(q.w[1], a.y) + fp::wide(q.w[2], a.z) + fp::wide(q.w[3], a.w) +
                      fp::wide(q.w[4], b.x) + fp::wide(q.w[5], b.y) + fp::wide(q.w[6], b.z) + fp::wide(q.w[7], b.w));
}
struct alignas(16) u64x2 {
    u64 x, y;
};
__device__ __forceinline__ u64 fold8(const u64 *src, u64 g, const Weights &q) {
    u128 s = 0;
#pragma unroll
    for (int e = 0; e < OCT; e += 2) {
        const u64x2 p = *reinterpret_cast<const u64x2 *>(src + OCT * g + e);
        s += fp::wide(q.w[e], p.x) + fp::wide(q.w[e + 1], p.y);
    }
    return fp::red128(s);  // (eight products below 2^122)
}

// Sum over the lanes with equal j = lane % 8, in every lane, of canonical
// values: eight of them, below 2^64, not reduced.
__device__ __forceinline__ u64 lane_sums(u64 v) { return plus32(plus16(v + from8(v))); }

// A wave's Gram sums into part[wave].
__device__ __forceinline__ void wave_gram(u64 (&s)[SLOTS], u64 (*part)[F2SC_ROW]) {
    const u32 lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
#pragma unroll
    for (int k = 0; k < SLOTS; k++) s[k] = lane_sums(s[k]);
    if (lane < OCT) {
#pragma unroll
        for (int k = 0; k < SLOTS; k++) part[wid][lane * SLOTS + k] = reduced(s[k]);
    }
}

// Message k < 3 of three rounds from their Gram matrix, lane x + 8 y of the
// wave holding M[x][y], and their challenges: with a_x the entries folded so
// far, G(0) and G(1) add M over equal x, y with the round's bit 0 or 1, and
// G(2) = sum (2 a_1 - a_0)^2 = 4 G(1) + G(0) - 4 sum a_0 a_1.  The earlier
// rounds' variables are first bound in both indices, by weights and a sum
// over their lane bits.  *f2 (if not NULL) receives G(0) + G(1).
__device__ __forceinline__ void gram_message(u64 m, u32 k, const u64 *r, u64 *msg, u64 *f2) {
    const u32 lane = threadIdx.x & 63, x = lane & 7, y = lane >> 3;
    for (u32 b = 0; b < k; b++) {
        m = mul(m, mul(fp::eqbit((x >> b) & 1, r[b]), fp::eqbit((y >> b) & 1, r[b])));
        m = plus_bit(plus_bit(m, b), 3 + b);
    }
    const u32 xk = (x >> k) & 1, yk = (y >> k) & 1, low = (1u << k) - 1;
    const bool on = !(x & low) && !(y & low) && (x >> (k + 1)) == (y >> (k + 1));
    const u64 g0 = wave_total(on && !xk && !yk ? m : 0), g1 = wave_total(on && xk && yk ? m : 0);
    const u64 c = wave_total(on && !xk && yk ? m : 0);
    if (lane == 0) {
        const u64 d = sub(g1, c), d2 = add(d, d);
        msg[0] = g0;
        msg[1] = g1;
        msg[2] = add(g0, add(d2, d2));
        if (f2) *f2 = add(g0, g1);
    }
}

// The state of the challenge stream before draw 3p, and the three draws of
// pass p's rounds from it.
__device__ __forceinline__ u64 state_at(const F2scState *ps, u64 seed, u32 p) {
    return uniform(p ? ps->rng[p] : fp::sm_state(seed, fp::PURPOSE_F2SC));
}

// One workgroup: pass p's rows into its nine messages, its challenges and
// the state after them.
__device__ void finish_pass(const F2scPass &a, u32 p, u32 nrows, const u64 *rows) {
    __shared__ u64 sm[FB / F2SC_ROW][F2SC_ROW];
    u64 st = state_at(a.ps, a.seed, p);
    const u64 r[3] = {fp::sm_field(st), fp::sm_field(st), fp::sm_field(st)};
    const u32 tid = threadIdx.x;
    constexpr u32 GRP = FB / F2SC_ROW;  // rows in flight, a thread a column
    if (tid < GRP * F2SC_ROW) {
        u64 s = 0;
        constexpr u32 U = 16;  // loads in flight: a row at a time waits a memory round trip each
        for (u32 q0 = tid / F2SC_ROW; q0 < nrows; q0 += GRP * U) {
            u64 x[U];
#pragma unroll
            for (u32 i = 0; i < U; i++) {
                const u32 q = q0 + i * GRP;
                x[i] = q < nrows ? rows[(u64)q * F2SC_ROW + tid % F2SC_ROW] : 0;
            }
#pragma unroll
            for (u32 i = 0; i < U; i++) s = add(s, x[i]);
        }
        sm[tid / F2SC_ROW][tid % F2SC_ROW] = s;
    }
    __syncthreads();
    const u32 k = tid >> 6;  // a wave a message
    if (k >= 3) return;
    if (tid == 0) {
        a.ps->rng[p + 1] = st;
        for (int i = 0; i < 3; i++) a.chals[3 * p + i] = r[i];
    }
    const u32 slot = gram_slot(tid & 7, (tid >> 3) & 7);
    u64 m = 0;
    for (u32 g = 0; g < GRP; g++) m = add(m, sm[g][slot]);
    gram_message(m, k, r, a.msgs + 1 + 9 * p + 3 * k, p || k ? nullptr : a.msgs);
}

// Rounds 0..2 over the counts: two lanes hold an oct (four counts each); lane
// h sums the ten products among its own counts and eight of the sixteen
// across, exactly in 96 bits (one multiply-add and one carry a product).
// Bound by the read of the counts: 268 MB in 54 us at 2^26, 5.0 TB/s (one round
// alone read them in 66 us).
__device__ __forceinline__ void acc96(u64 &lo, u32 &hi, u32 a, u32 b) {
    asm("v_mad_u64_u32 %0, vcc, %2, %3, %0\n\tv_addc_co_u32 %1, vcc, 0, %1, vcc"
        : "+v"(lo), "+v"(hi) : "v"(a), "v"(b) : "vcc");
}
__device__ __forceinline__ u32 swap1(u32 v) { return (u32)__builtin_amdgcn_update_dpp(0, (int)v, 0xB1, 0xf, 0xf, true); }

__global__ void __launch_bounds__(FB) k_f2sc_first(const F2scPass a, u64 nq, const u32 *__restrict__ src) {
    constexpr int K = 18;
    u64 lo[K];
    u32 hi[K];
#pragma unroll
    for (int k = 0; k < K; k++) lo[k] = 0, hi[k] = 0;
    const u32 h = threadIdx.x & 1;
    const u64 stride = (u64)gridDim.x * FB;
    auto oct_half = [&](const uint4 &v4) {
        const u32 v[4] = {v4.x, v4.y, v4.z, v4.w};
        const u32 o[4] = {swap1(v4.x), swap1(v4.y), swap1(v4.z), swap1(v4.w)};
        int k = 0;
#pragma unroll
        for (int x = 0; x < 4; x++)
#pragma unroll
            for (int y = x; y < 4; y++, k++) acc96(lo[k], hi[k], v[x], v[y]);
        // across: counts 0, 1 of lane 0 and 2, 3 of lane 0 (lane 1's partner) with lane 1's four
#pragma unroll
        for (int x = 0; x < 2; x++)
#pragma unroll
            for (int y = 0; y < 4; y++, k++) acc96(lo[k], hi[k], h ? o[2 + x] : v[x], h ? v[y] : o[y]);
    };
    // four loads in flight a lane (nq and the stride are even: an oct's lanes stay together)
    constexpr u32 U = 4;
    u64 q = (u64)blockIdx.x * FB + threadIdx.x;
    for (; q + (U - 1) * stride < nq; q += U * stride) {
        uint4 v[U];
#pragma unroll
        for (u32 i = 0; i < U; i++) v[i] = counts4(src + 4 * (q + i * stride));
#pragma unroll
        for (u32 i = 0; i < U; i++) oct_half(v[i]);
    }
    for (; q < nq; q += stride) oct_half(counts4(src + 4 * q));
    // sums over the lanes with equal h, into the row's slots
    __shared__ u64 part[FW][F2SC_ROW];
    const u32 lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
    u64 s[K];
#pragma unroll
    for (int k = 0; k < K; k++) {
        u64 t = fp::red128(((u128)hi[k] << 64) + lo[k]);
        t += dppx<0x112>(t);  // row_shr:2, 4, 8: eight values below p stay below 2^64
        t += dppx<0x114>(t);
        t += dppx<0x118>(t);
        s[k] = reduced(plus32(plus16(reduced(t))));  // (lanes 14, 15)
    }
    if (lane < F2SC_ROW) part[wid][lane] = 0;  // (slot 4 of lanes with bit 0 is not used)
    __builtin_amdgcn_wave_barrier();
    if (lane == 14 || lane == 15) {
        int k = 0;
#pragma unroll
        for (int x = 0; x < 4; x++)
#pragma unroll
            for (int y = x; y < 4; y++, k++) part[wid][gram_slot(4 * h + x, 4 * h + y)] = s[k];
#pragma unroll
        for (int x = 0; x < 2; x++)
#pragma unroll
            for (int y = 0; y < 4; y++, k++) part[wid][gram_slot(2 * h + x, 4 + y)] = s[k];
    }
    __syncthreads();
    if (threadIdx.x < F2SC_ROW) {
        u64 t = 0;
#pragma unroll
        for (int w = 0; w < FW; w++) t = add(t, part[w][threadIdx.x]);
        a.rows[(u64)blockIdx.x * F2SC_ROW + threadIdx.x] = t;
    }
}

// Pass p >= 1: entry g of level 3p from the eight of level 3(p-1) (the counts
// themselves when p = 1), stored, and the level's Gram sums.  Workgroup 0
// finishes pass p - 1.  Lanes own one entry, so loads and stores
// are contiguous over the wave; n is a multiple of 64.  Bound by memory: from
// 2^26 counts 335 MB in 56 us, 6.0 TB/s (98 us for 805 MB as one round).
template <typename T>
__global__ void __launch_bounds__(FB, 8) k_f2sc_pass(const F2scPass a, u64 n, const T *__restrict__ src, u64 *dst) {
    if (blockIdx.x == 0) {  // (dispatched first: the last one would wait for a body workgroup to end)
        finish_pass(a, a.p - 1, a.prev_nrows, a.prev_rows);
        return;
    }
    const u32 nb = gridDim.x - 1, lb = blockIdx.x - 1;
    u64 st = state_at(a.ps, a.seed, a.p - 1);
    const u64 r[3] = {fp::sm_field(st), fp::sm_field(st), fp::sm_field(st)};
    const Weights q = fold_weights(r);
    const u32 j = threadIdx.x & 7;
    u128 acc[SLOTS] = {0, 0, 0, 0, 0};
    u64 s[SLOTS] = {0, 0, 0, 0, 0};
    u32 terms = 0;
    for (u64 g = (u64)lb * FB + threadIdx.x; g < n; g += (u64)nb * FB) {
        const u64 v = fold8(src, g, q);
        dst[g] = v;
        gram_add(j, v, acc);
        if (++terms == 32) {  // (64 products below 2^122 would fit)
            terms = 0;
#pragma unroll
            for (int k = 0; k < SLOTS; k++) s[k] = add(s[k], fp::red128(acc[k])), acc[k] = 0;
        }
    }
    __shared__ u64 part[FW][F2SC_ROW];
#pragma unroll
    for (int k = 0; k < SLOTS; k++) s[k] = add(s[k], fp::red128(acc[k]));
    wave_gram(s, part);
    __syncthreads();
    if (threadIdx.x < F2SC_ROW) {
        u64 t = 0;
#pragma unroll
        for (int w = 0; w < FW; w++) t = add(t, part[w][threadIdx.x]);
        a.rows[(u64)lb * F2SC_ROW + threadIdx.x] = t;
    }
}

// The last rounds in one workgroup (workgroup 1 finishes pass p - 1): level
// 3p, 2^L <= F2SC_TAIL entries, folded from the level below (p >= 1) or read
// (p = 0), then three rounds at a time: Gram sums into LDS, a barrier that
// completes them, the fold by the three challenges, a barrier; the messages
// are formed from the sums at the end.  A wave issues an instruction every
// four to six cycles, so the length of the tail is the instructions one wave
// runs between barriers: below 512 entries the slots of a level go to
// different waves, one wave draws the challenges and their eight weights
// while the others sum (they are read after the barrier), and each message
// has a wave of its own.  8.4 us from 2^10 counts (13.6 us as a round at a
// time; 12.5 us with every slot in the entry's wave and each three rounds'
// messages in one).
template <typename T>
__global__ void __launch_bounds__(FB) k_f2sc_tail(const F2scPass a, u32 L, const T *__restrict__ src) {
    constexpr int PER = F2SC_TAIL / FB;
    constexpr int STEPS = (F2SC_TAIL_LOG + 2) / 3;
    __shared__ u64 tab[F2SC_TAIL / OCT], part[STEPS][FW][F2SC_ROW], s_r[STEPS][3], s_w[OCT];
    if (blockIdx.x == 1) {
        finish_pass(a, a.p - 1, a.prev_nrows, a.prev_rows);
        return;
    }
    const u32 tid = threadIdx.x, lane = tid & 63, j = tid & 7;
    const u32 wid = (u32)__builtin_amdgcn_readfirstlane((int)(tid >> 6));
    u64 st;
    u64 x[PER];  // entries tid, tid + FB, ... of the first level (0 past its end)
    const u32 n0 = 1u << L;
    if (a.p) {
        st = state_at(a.ps, a.seed, a.p - 1);
        const u64 r[3] = {fp::sm_field(st), fp::sm_field(st), fp::sm_field(st)};
        const Weights q = fold_weights(r);
#pragma unroll
        for (int i = 0; i < PER; i++) x[i] = tid + i * FB < n0 ? fold8(src, tid + i * FB, q) : 0;
    } else {
        st = state_at(a.ps, a.seed, 0);
#pragma unroll
        for (int i = 0; i < PER; i++) x[i] = tid + i * FB < n0 ? (u64)src[tid + i * FB] : 0;
    }
    // (wave FW - 1) three challenges for s_r[step] and the weights of their fold
    auto draw = [&](u32 step) {
        if (wid == FW - 1) {
            const u64 r[3] = {fp::sm_field(st), fp::sm_field(st), fp::sm_field(st)};
            if (lane < OCT) s_w[lane] = chi3(lane, r);
            if (lane < 3) s_r[step][lane] = lane == 0 ? r[0] : (lane == 1 ? r[1] : r[2]);
        }
    };
    draw(0);
    if ((tid & ~63u) < n0) {
        u128 acc[SLOTS] = {0, 0, 0, 0, 0};
#pragma unroll
        for (int i = 0; i < PER; i++)
            if (i * FB < (int)n0) gram_add(j, x[i], acc);
        u64 s[SLOTS];
#pragma unroll
        for (int k = 0; k < SLOTS; k++) s[k] = fp::red128(acc[k]);
        wave_gram(s, part[0]);
    }
    __syncthreads();  // the sums of the first three rounds are complete
    u32 n = n0, steps = (L + 2) / 3;
    for (u32 step = 0; step + 1 < steps; step++) {
        // the oct's eight weighted entries added over its lanes: below 8 p < 2^64
        const u64 w = s_w[j];
        if (step == 0) {
#pragma unroll
            for (int i = 0; i < PER; i++) {
                if (i * FB < (int)n0) {
                    const u64 v = oct_total(mul(w, x[i]));
                    if (j == 0 && tid + i * FB < n) tab[(tid + i * FB) >> 3] = reduced(v);
                }
            }
        } else {  // (at most F2SC_TAIL / 8 entries, in tab[0 .. n))
            if ((tid & ~63u) < n) {
                const u64 v = oct_total(mul(w, tid < n ? x[0] : 0));
                if (j == 0 && tid < n) tab[tid >> 3] = reduced(v);
            }
        }
        n >>= 3;
        __syncthreads();  // the next level is complete, and s_w is read
        x[0] = tid < n ? tab[tid] : 0;
        draw(step + 1);
        // task (slot, 64 entries): one product a lane, partners as gram_add's
        const u32 ew = (n + 63) >> 6;
        for (u32 t = wid; t < SLOTS * ew; t += FW) {
            const u32 k = t / ew, q = t - k * ew, e = q * 64 + lane;
            const u32 d = k == 0 ? 0 : k == 4 ? 7 : k == 1 ? (j & 1 ? 3 : 1) : k == 2 ? (j & 2 ? 6 : 2) : (j & 4 ? 5 : 4);
            const u64 v = e < n ? tab[e] : 0, o = (e ^ d) < n ? tab[e ^ d] : 0;
            const u64 s = reduced(lane_sums(mul(v, o)));
            if (lane < OCT) part[step + 1][q][lane * SLOTS + k] = s;
        }
        __syncthreads();  // the sums of these rounds are complete
    }
    const u32 base = 3 * a.p;
    if (tid < L) a.chals[base + tid] = s_r[tid / 3][tid % 3];
    const u32 slot = gram_slot(lane & 7, lane >> 3);
    for (u32 t = wid; t < L; t += FW) {  // message t: a wave each, the last rounds' (most binds) not together
        const u32 step = t / 3, k = t - 3 * step;
        const u32 nlev = n0 >> (3 * step);
        const u32 nw = nlev < (u32)FB ? (nlev + 63) >> 6 : FW;
        u64 m = 0;
        for (u32 w = 0; w < nw; w++) m = add(m, part[step][w][slot]);
        gram_message(m, k, s_r[step], a.msgs + 1 + 3 * (base + t), base + t == 0 ? a.msgs : nullptr);
    }
}

// n == 1: the transcript is F2 = a[0]^2.
__global__ void k_f2sc_single(const u32 *a32, u64 *msg) {
    if (threadIdx.x == 0) {
        const u64 v = a32[0];
        msg[0] = mul(v, v);
    }
}

}  // namespace

u32 f2sc_passes(u32 l) { return l <= (u32)F2SC_TAIL_LOG ? 0 : (l - F2SC_TAIL_LOG + 2) / 3; }

u32 f2sc_rows(u32 l, u32 p) {
    // lanes of the pass: two an oct over the counts, one an entry later.  Four
    // a thread before another workgroup starts, as many workgroups as the
    // chip holds at once: two a CU with the first pass's registers, four with
    // the later ones' (the finisher reads a row of each).
    const u64 lanes = p == 0 ? (1ull << l) / 4 : (1ull << l) >> (3 * p);
    const u64 b = (lanes + 4 * FB - 1) / (4 * FB), most = p == 0 ? 512 : F2SC_MAX_ROWS - 1;
    return (u32)(b < 1 ? 1 : b > most ? most : b);
}

hipError_t launch_f2sc_pass(hipStream_t st, const F2scPass &a, u32 l, const u32 *a32, const u64 *src, u64 *dst) {
    const u32 nb = f2sc_rows(l, a.p);
    const u64 n = (1ull << l) >> (3 * a.p);
    if (a.p == 0)
        hipLaunchKernelGGL(k_f2sc_first, dim3(nb), dim3(FB), 0, st, a, n / 4, a32);
    else if (a.p == 1)
        hipLaunchKernelGGL(k_f2sc_pass<u32>, dim3(nb + 1), dim3(FB), 0, st, a, n, a32, dst);
    else
        hipLaunchKernelGGL(k_f2sc_pass<u64>, dim3(nb + 1), dim3(FB), 0, st, a, n, src, dst);
    return hipGetLastError();
}

hipError_t launch_f2sc_tail(hipStream_t st, const F2scPass &a, u32 l, const u32 *a32, const u64 *src) {
    const u32 L = l - 3 * a.p;
    const dim3 g(a.p ? 2 : 1), b(FB);
    if (l == 0)
        hipLaunchKernelGGL(k_f2sc_single, dim3(1), dim3(64), 0, st, a32, a.msgs);
    else if (a.p <= 1)
        hipLaunchKernelGGL(k_f2sc_tail<u32>, g, b, 0, st, a, L, a32);
    else
        hipLaunchKernelGGL(k_f2sc_tail<u64>, g, b, 0, st, a, L, src);
    return hipGetLastError();
}

}  // namespace gkr

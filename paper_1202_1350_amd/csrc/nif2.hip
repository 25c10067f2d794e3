// nif2.hip -- the non-interactive F2 protocol (Sec. 3.2, 4.2) on
// gfx950: the prover's prime factor transforms of the grid rows and the
// column square-sums of its proof, and the verifier's row evaluations.
//
// The universe is a v x h grid, cell (row y, column j) = a_{j v + y}, so
// element j of every row is one contiguous run of v words: a thread per
// (row, line of a pass) reads and writes coalesced, the layout the paper
// reaches by transposing the grid (Sec. 6.2.1).  Row y is the polynomial
// f_y of degree < h through the order-h subgroup H = <w>; the proof is
// g = sum_y f_y^2 on the order-2h subgroup <xi> (xi^2 = w): the even points
// are the data squared, the odd points are f_y on the coset xi H, obtained
// from an inverse transform (values -> coefficients c), a twist
// c_k xi^k / h and a forward transform.
#include "lanes.hpp"
#include "nif2.hpp"

namespace gkr {

using fp::add;
using fp::mul;
using fp::P;
using fp::sub;
using fp::u128;

constexpr int NT = 256;  // threads per workgroup of these kernels

struct PassArgs {
    PfaPlan pl;
    u64 n, v;
    u32 dim;       // digit transformed by this pass
    u64 wp[25];    // powers 0 .. F-1 of the pass's root
};

__device__ __forceinline__ u32 good_index(const PfaPlan &pl, u64 pos) {
    u64 g = 0;
    for (u32 i = 0; i < pl.nf; i++) g += (pos / pl.stride[i]) % pl.F[i] * pl.gstep[i];
    return (u32)(g % pl.h);
}
__device__ __forceinline__ u32 crt_index(const PfaPlan &pl, u64 pos) {
    u64 c = 0;
    for (u32 i = 0; i < pl.nf; i++) c += (pos / pl.stride[i]) % pl.F[i] * pl.cstep[i];
    return (u32)(c % pl.h);
}

// One pass: the F-point DFT along digit `dim` of every line of every row.
// MODE 1 gathers the row from a in Good order (the first inverse pass);
// MODE 2 twists by tw[CRT(position)] as it loads (the first forward pass).
template <int F, int MODE>
__global__ void __launch_bounds__(NT) k_pfa_pass(const PassArgs pa, const u64 *__restrict__ a,
                                                 const u64 *__restrict__ tw, u64 *W) {
    const PfaPlan &pl = pa.pl;
    const u64 v = pa.v, s = pl.stride[pa.dim];
    const u64 total = (u64)(pl.h / F) * v;
    for (u64 gid = (u64)blockIdx.x * NT + threadIdx.x; gid < total; gid += (u64)gridDim.x * NT) {
        const u64 y = gid % v, l = gid / v;
        const u64 base = (l % s) + (l / s) * s * F;
        u64 x[F];
        if (MODE == 1) {
            const u32 g0 = good_index(pl, base), gs = pl.gstep[pa.dim];
#pragma unroll
            for (int m = 0; m < F; m++) {
                const u64 j = (g0 + (u64)m * gs) % pl.h, i = j * v + y;
                x[m] = i < pa.n ? a[i] : 0;
            }
        } else if (MODE == 2) {
            const u32 c0 = crt_index(pl, base), cs = pl.cstep[pa.dim];
#pragma unroll
            for (int m = 0; m < F; m++)
                x[m] = mul(W[(base + m * s) * v + y], tw[(c0 + (u64)m * cs) % pl.h]);
        } else {
#pragma unroll
            for (int m = 0; m < F; m++) x[m] = W[(base + m * s) * v + y];
        }
        if constexpr (F == 25) {
            // 25 = 5 x 5: n = 5 n1 + n2, k = k1 + 5 k2, w^{nk} = u^{n1 k1} w^{n2 k1} u^{n2 k2}
            // with u = w^5: five 5-point DFTs over n1 (in place), twiddles w^{n2 k1},
            // five 5-point DFTs over n2 written out
#pragma unroll
            for (int n2 = 0; n2 < 5; n2++) {
                u64 t[5];
#pragma unroll
                for (int k1 = 0; k1 < 5; k1++) {
                    u128 acc = 0;
#pragma unroll
                    for (int n1 = 0; n1 < 5; n1++) acc += fp::wide(x[5 * n1 + n2], pa.wp[(5 * n1 * k1) % 25]);
                    t[k1] = fp::red128(acc);
                }
#pragma unroll
                for (int k1 = 0; k1 < 5; k1++) x[5 * k1 + n2] = (n2 * k1) ? mul(t[k1], pa.wp[n2 * k1]) : t[k1];
            }
#pragma unroll
            for (int k1 = 0; k1 < 5; k1++) {
#pragma unroll
                for (int k2 = 0; k2 < 5; k2++) {
                    u128 acc = 0;
#pragma unroll
                    for (int n2 = 0; n2 < 5; n2++) acc += fp::wide(x[5 * k1 + n2], pa.wp[(5 * n2 * k2) % 25]);
                    W[(base + (k1 + 5 * k2) * s) * v + y] = fp::red128(acc);
                }
            }
        } else {
#pragma unroll
            for (int k = 0; k < F; k++) {
                u128 acc = 0;
#pragma unroll
                for (int m = 0; m < F; m++) acc += fp::wide(x[m], pa.wp[(m * k) % F]);  // F < 32 terms < 2^127
                W[(base + k * s) * v + y] = fp::red128(acc);
            }
        }
    }
}

static u32 grid_of(u64 items) {
    const u64 b = (items + NT - 1) / NT;
    return (u32)std::max<u64>(1, std::min<u64>(b, 4096));
}

template <int MODE>
static hipError_t pass(hipStream_t st, const PassArgs &pa, const u64 *a, const u64 *tw, u64 *W) {
    const u32 F = pa.pl.F[pa.dim];
    const dim3 g(grid_of((u64)(pa.pl.h / F) * pa.v)), b(NT);
    switch (F) {
#define PF(N) case N: hipLaunchKernelGGL((k_pfa_pass<N, MODE>), g, b, 0, st, pa, a, tw, W); break;
        PF(3) PF(5) PF(7) PF(9) PF(11) PF(13) PF(25)
#undef PF
        default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

hipError_t launch_nif2_transform(hipStream_t st, const PfaPlan &pl, const u64 *a, u64 n, u64 v,
                                 const u64 *tw, u64 *W) {
    PassArgs pa;
    pa.pl = pl;
    pa.n = n;
    pa.v = v;
    // inverse transform: values on H (Good order) -> coefficients (CRT order)
    for (u32 d = 0; d < pl.nf; d++) {
        pa.dim = d;
        u64 w = 1;
        for (u32 m = 0; m < pl.F[d]; m++, w = mul(w, pl.winv[d])) pa.wp[m] = w;
        const hipError_t e = d == 0 ? pass<1>(st, pa, a, tw, W) : pass<0>(st, pa, a, tw, W);
        if (e != hipSuccess) return e;
    }
    // twist by xi^k / h, forward transform: CRT order -> f_y(xi w^j) in Good order
    for (u32 d = 0; d < pl.nf; d++) {
        pa.dim = d;
        u64 w = 1;
        for (u32 m = 0; m < pl.F[d]; m++, w = mul(w, pl.wfwd[d])) pa.wp[m] = w;
        const hipError_t e = d == 0 ? pass<2>(st, pa, a, tw, W) : pass<0>(st, pa, a, tw, W);
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

// ------------------------------------------------------- rows kept in LDS
//
// Rows of up to NIF2_LDS_H values (every row length of Table 3) go through
// both transforms without leaving the chip: a workgroup takes a tile of TY
// adjacent rows (their elements of a column are adjacent words), reads it
// once, adds its squares into the even points' sums, runs the passes of both
// transforms in LDS, and adds the squares of what is left into the odd
// points' sums, kept in registers over all of the workgroup's tiles.  Against
// a launch a pass with the grid in memory (six reads and six writes of 200 MB
// for h = 2475, the columns read once more and the range check once before)
// the grid is read once, and the time is the transforms' arithmetic: h = 2475
// over 25 million values 795 -> 413 us a proof, this kernel 380 us with the
// VALU issuing 82% of it (172 million wave instructions, 440 a value).
//
// A DFT of odd length F pairs x_m with x_{F-m}: with s = x_m + x_{F-m},
// d = x_m - x_{F-m}, c_j = (w^j + w^-j) / 2 and t_j = (w^j - w^-j) / 2,
//   X_k, X_{F-k} = (x_0 + sum_m s_m c_{mk}) +- sum_m d_m t_{mk},
// (F-1)^2 / 2 products instead of F^2 (50 for 121 at F = 11); 25 is 5 x 5
// with twiddles.  X_0 is a sum.
constexpr int RB = 512;  // threads per workgroup of the row kernel

struct Half {
    u32 l, h;
};
struct RowArgs {
    u32 h, nf, logty, ntiles;
    u32 full;         // columns all of whose v rows hold values
    u64 rem;          // rows of the next column that do
    u32 F[NIF2_LDS_NF], stride[NIF2_LDS_NF];
    u64 v;
    const u64 *a;
    const u32 *pos;   // column j's position (Good order)
    const u64 *tw;    // by position: xi^k / h of coefficient k there (CRT order)
    u64 *part;        // [workgroup][2][h], by position: even, odd points
    u32 *flag;        // set when a value is not below p
    u32 root_at[2 * NIF2_LDS_NF];  // per pass: its roots in `roots`
    Half roots[NIF2_LDS_ROOTS];
};

//
// The passes are bound by VALU instructions, so the products are sums over
// halves: x = xh 2^31 + xl (xl < 2^31) makes a product the three sums
// xl yl, xl yh + xh yl, xh yh of weights 1, 2^31, 2^62 = 2, four multiply-adds
// and no carries while at most four terms are summed; a u128 sum takes 12
// instructions a term.  Values between passes are congruent, not canonical,
// and below 3 2^61 + 16; a folded value is below 2^61 + 8, its high half at
// most 2^30.

__device__ __forceinline__ Half halves(u64 x) { return {(u32)x & 0x7fffffffu, (u32)(x >> 31)}; }
__device__ __forceinline__ u64 fold(u64 x) { return fp::fold64_mad(x); }
struct Sums {
    u64 ll = 0, mm = 0, hh = 0;
};
// (a term is at most 2^62, 2^62, 2^60 + 2^31)
__device__ __forceinline__ void mac(Sums &a, Half x, Half y) {
    a.ll += (u64)x.l * y.l;
    a.mm += (u64)x.l * y.h;
    a.mm += (u64)x.h * y.l;
    a.hh += (u64)x.h * y.h;
}
// The value of N <= 7 terms' sums plus x0, below 2^61 + 8:
// ll + mm 2^31 + 2 hh with 2^31 mm = (mm >> 30) + (mm mod 2^30) 2^31.  Before
// the last fold ll is folded (2^61), mm's parts are 2^34 and 2^61, and 2 hh is
// 2^61 a term (for more than four terms hh is folded first: 2^62).  With four
// terms x0 is below 2^61 + 8: 7 2^61 and less than 2^36 in all, below 2^64.
// Where F = 9 moves one of its four terms into x0 (below 2^62 + 32 then) three
// are left: 7 2^61 and less than 2^36 again.
template <int N>
__device__ __forceinline__ u64 total(const Sums &a, u64 x0 = 0) {
    const u64 t = fold(a.ll) + x0 + (a.mm >> 30) + (u64)((u32)a.mm & 0x3fffffffu) * 0x80000000u;
    return fold(t + 2 * (N <= 4 ? a.hh : fold(a.hh)));
}
__device__ __forceinline__ u64 mul_lz(u64 x, Half y) {
    Sums a;
    mac(a, halves(fold(x)), y);
    return total<1>(a);
}

// x := its DFT, c_j at rt[j - 1] for j <= M = (F-1)/2, t_j at rt[M + j - 1] for j < F.
template <int F>
__device__ __forceinline__ void dft_odd(u64 (&x)[F], const Half *rt) {
    constexpr int M = (F - 1) / 2;
    Half s[M], d[M];
    const u64 x0 = fold(x[0]);
    u64 tot = x0;
#pragma unroll
    for (int m = 1; m <= M; m++) {
        const u64 sm = fold(x[m] + x[F - m]);  // (below 3 2^62 + 32 before)
        s[m - 1] = halves(sm);
        d[m - 1] = halves(fold(x[m] + (4 * P - x[F - m])));  // (below 3 2^61 + 2^63 + 16)
        tot += sm;  // (M + 1 <= 7 values below 2^61 + 8: no overflow)
    }
#pragma unroll
    for (int k = 1; k <= M; k++) {
        Sums A, B;
        u64 extra = x0;
        int ta = 0;
#pragma unroll
        for (int m = 1; m <= M; m++) {
            const int j = (m * k) % F;
            if (j == 0) {  // (F = 9: c_0 = 1, t_0 = 0)
                extra += ((u64)s[m - 1].h << 31) + s[m - 1].l;
                continue;
            }
            if (ta++ == 4) {  // room for three more terms
                A.ll = fold(A.ll);
                A.mm = fold(A.mm);
                B.ll = fold(B.ll);
                B.mm = fold(B.mm);
            }
            mac(A, s[m - 1], rt[(j <= M ? j : F - j) - 1]);
            mac(B, d[m - 1], rt[M + j - 1]);
        }
        const u64 p = total<M>(A, extra), q = total<M>(B);
        x[k] = p + q;
        x[F - k] = p + (2 * P - q);
    }
    x[0] = fold(tot);
}

// 25 = 5 x 5: n = 5 n1 + n2, k = k1 + 5 k2; the 5-point roots at rt, the
// twiddles w^{n2 k1} (n2, k1 = 1..4) at rt + 6.  out(k, X_k) takes the results.
template <typename Out>
__device__ __forceinline__ void dft25(u64 (&x)[25], const Half *rt, Out out) {
#pragma unroll
    for (int n2 = 0; n2 < 5; n2++) {
        u64 t[5] = {x[n2], x[5 + n2], x[10 + n2], x[15 + n2], x[20 + n2]};
        dft_odd<5>(t, rt);
        x[n2] = t[0];
#pragma unroll
        for (int k1 = 1; k1 < 5; k1++) x[5 * k1 + n2] = n2 ? mul_lz(t[k1], rt[6 + 4 * (n2 - 1) + k1 - 1]) : t[k1];
    }
#pragma unroll
    for (int k1 = 0; k1 < 5; k1++) {
        u64 t[5] = {x[5 * k1], x[5 * k1 + 1], x[5 * k1 + 2], x[5 * k1 + 3], x[5 * k1 + 4]};
        dft_odd<5>(t, rt);
#pragma unroll
        for (int k2 = 0; k2 < 5; k2++) out(k1 + 5 * k2, t[k2]);
    }
}

// One pass over the tile in LDS: the F-point DFT along a digit of stride s.
template <int F>
__device__ __forceinline__ void row_pass(u64 *W, u32 h, u32 s, u32 logty, const Half *rt, const u64 *tw) {
    const u32 ty = 1u << logty, items = (h / F) << logty;
    for (u32 it = threadIdx.x; it < items; it += RB) {
        const u32 y = it & (ty - 1), l = it >> logty;
        const u32 q = l / s, base = l - q * s + q * s * F;
        const u32 step = s << logty;
        u32 at = (base << logty) + y;
        u64 x[F];
#pragma unroll
        for (int m = 0; m < F; m++) x[m] = W[at + m * step];
        if (tw) {  // (uniform)
#pragma unroll
            for (int m = 0; m < F; m++) x[m] = mul_lz(x[m], halves(tw[base + m * s]));
        }
        asm("" : "+v"(at));  // the stores' addresses are formed again: F of them would be held in registers
        if constexpr (F == 25) {
            dft25(x, rt, [&](int k, u64 X) { W[at + k * step] = X; });
        } else {
            dft_odd<F>(x, rt);
#pragma unroll
            for (int m = 0; m < F; m++) W[at + m * step] = x[m];
        }
    }
}

// The square of a value, added to sums of at most four terms.
__device__ __forceinline__ void square(Sums &s, u64 v) {
    const Half x = halves(fold(v));
    s.ll += (u64)x.l * x.l;
    s.mm += (u64)x.l * (2 * x.h);
    s.hh += (u64)x.h * x.h;
}
// Squares of the tile's values added per position.  Tiles of few rows (long
// ones): a thread sums its positions' TY values into acc.
template <int NC>
__device__ __forceinline__ void square_sums(const u64 *W, u32 h, u32 logty, u64 (&acc)[NC]) {
#pragma unroll
    for (int c = 0; c < NC; c++) {
        const u32 p = threadIdx.x + c * RB;
        if (p < h) {
            u64 t = acc[c];
            for (u32 y = 0; y < (1u << logty); y += 4) {
                Sums s;
#pragma unroll
                for (u32 i = 0; i < 4; i++) square(s, W[(p << logty) + y + i]);
                t = fold(t + total<4>(s));
            }
            acc[c] = t;
        }
    }
}
// Short rows, and one row or two: a row a lane (a thread a position would leave
// most threads idle), summed over the lanes of a position into s_acc, LDS.
__device__ __forceinline__ void square_lanes(const u64 *W, u32 h, u32 logty, u64 *s_acc) {
    const u32 lane = threadIdx.x & 63, w = threadIdx.x >> 6, lw = logty < 6 ? logty : 6;  // log2 lanes a position
    const u32 y0 = lane & ((1u << lw) - 1), per = 64 >> lw;
    for (u32 p0 = w * per; p0 < h; p0 += RB / 64 * per) {  // (wave-uniform)
        const u32 p = p0 + (lane >> lw);
        u64 t = 0;
        if (p < h) {
            for (u32 y = y0; y < (1u << logty); y += 64 * 4) {
                Sums s;
#pragma unroll
                for (u32 i = 0; i < 4; i++)
                    if (y + 64 * i < (1u << logty)) square(s, W[(p << logty) + y + 64 * i]);
                t = fold(t + total<4>(s));
            }
        }
        t = fp::canon(t);
        for (u32 b = 0; b < lw; b++) t = plus_bit(t, b);  // (uniform)
        if (y0 == 0 && p < h) s_acc[p] = add(s_acc[p], t);
    }
}

// NC: positions a thread accumulates, ceil(h / RB); 0: positions accumulated in
// LDS, after the tile.
template <int NC>
__global__ void __launch_bounds__(RB, NC <= 5 ? 4 : 2) k_nif2_rows_lds(const RowArgs a) {
    extern __shared__ u64 W[];
    constexpr int NA = NC ? NC : 1;
    const u32 tid = threadIdx.x, ty = 1u << a.logty;
    u64 *s_acc = W + ((u64)a.h << a.logty);
    u64 even[NA], odd[NA];
#pragma unroll
    for (int c = 0; c < NA; c++) even[c] = odd[c] = 0;
    if (!NC)
        for (u32 p = tid; p < 2 * a.h; p += RB) s_acc[p] = 0;
    // Adjacent tiles share cache lines, so workgroups of one XCD (equal
    // blockIdx mod 8) take adjacent tiles.
    const u32 xcd = blockIdx.x & 7, per = (a.ntiles + 7) / 8;
    u64 bad = 0;
    for (u32 k = blockIdx.x >> 3; k < per; k += gridDim.x >> 3) {
        const u32 tile = xcd * per + k;
        if (tile >= a.ntiles) break;  // (uniform)
        const u64 y0 = (u64)tile << a.logty;
        __syncthreads();  // the previous tile's sums are done with W
        {
            // column j of row y0 + y is a value while j < cols; a thread keeps
            // its row and takes every dj-th column, eight loads in flight
            const u32 y = tid & (ty - 1), dj = RB >> a.logty;
            const u64 row = y0 + y;
            const u32 cols = row < a.v ? a.full + (row < a.rem ? 1u : 0u) : 0u;
            u32 j = tid >> a.logty;
            const u64 *src = a.a + (u64)j * a.v + row;
            const u64 step = (u64)dj * a.v;
            constexpr u32 U = 8;
            for (; j < a.h; j += U * dj, src += U * step) {
                u64 x[U];
                u32 p[U];
#pragma unroll
                for (u32 i = 0; i < U; i++) {
                    p[i] = j + i * dj < a.h ? a.pos[j + i * dj] : 0;
                    x[i] = j + i * dj < cols ? src[i * step] : 0;
                }
#pragma unroll
                for (u32 i = 0; i < U; i++) {
                    bad |= x[i] >= P;
                    if (j + i * dj < a.h) W[(p[i] << a.logty) + y] = x[i];
                }
            }
        }
        __syncthreads();
        if (NC) square_sums<NA>(W, a.h, a.logty, even); else square_lanes(W, a.h, a.logty, s_acc);
        for (u32 q = 0; q < 2 * a.nf; q++) {
            const u32 d = q < a.nf ? q : q - a.nf;
            const Half *rt = a.roots + a.root_at[q];
            const u64 *tw = q == a.nf ? a.tw : nullptr;
            __syncthreads();
            switch (a.F[d]) {
#define RP(N) case N: row_pass<N>(W, a.h, a.stride[d], a.logty, rt, tw); break;
                RP(3) RP(5) RP(7) RP(9) RP(11) RP(13) RP(25)
#undef RP
                default: break;
            }
        }
        __syncthreads();
        if (NC) square_sums<NA>(W, a.h, a.logty, odd); else square_lanes(W, a.h, a.logty, s_acc + a.h);
    }
    if (!NC) {
        __syncthreads();
        for (u32 p = tid; p < 2 * a.h; p += RB) a.part[(u64)blockIdx.x * 2 * a.h + p] = s_acc[p];
    }
#pragma unroll
    for (int c = 0; c < NC; c++) {
        const u32 p = tid + c * RB;
        if (p < a.h) {
            a.part[(u64)blockIdx.x * 2 * a.h + p] = fp::canon(even[c]);
            a.part[((u64)blockIdx.x * 2 + 1) * a.h + p] = fp::canon(odd[c]);
        }
    }
    if (bad) a.flag[0] = 1;
}

// By position p: pos[Good(p)] = p and tw[p] = xi^CRT(p) / h.
__global__ void k_nif2_tables(const PfaPlan pl, u64 xi, u64 hinv, u32 *pos, u64 *tw) {
    const u32 p = blockIdx.x * NT + threadIdx.x;
    if (p >= pl.h) return;
    pos[good_index(pl, p)] = p;
    tw[p] = mul(fp::pow(xi, crt_index(pl, p)), hinv);
}

// msgs[2j + o] = the sum over the workgroups of the parts at column j's
// position (o: even or odd points); 32 threads share a position, 32 adjacent
// positions a workgroup.
__global__ void __launch_bounds__(1024) k_nif2_parts(const PfaPlan pl, const u64 *__restrict__ part, u32 nwg, u64 *msgs) {
    __shared__ u64 sm[32][32];
    const u32 t = threadIdx.x & 31, g = threadIdx.x >> 5, c = blockIdx.x * 32 + t;  // c = o h + position
    u64 s = 0;
    if (c < 2 * pl.h) {
#pragma unroll 16
        for (u32 w = g; w < nwg; w += 32) s = add(s, part[(u64)w * 2 * pl.h + c]);
    }
    sm[g][t] = s;
    __syncthreads();
    if (g == 0 && c < 2 * pl.h) {
        for (u32 k = 1; k < 32; k++) s = add(s, sm[k][t]);
        const u32 o = c >= pl.h;
        msgs[2 * good_index(pl, o ? c - pl.h : c) + o] = s;
    }
}

// Rows a tile holds: a power of two, at least 4, at most 80 KB of LDS (two
// workgroups a CU: one loads while the other transforms), except that rows of
// more than 2560 values take 160 KB with 4.  Rows of fewer than 64 values
// accumulate over lanes in LDS with up to 512 a tile, longer ones over threads'
// positions with up to 64: 24 million values at h = 9 take 190 us so (820 with
// a thread a position), at h = 99 302 us (400 over lanes), at 225 373 (491).
// Fewer rows than fill the chip so are cut into lower tiles, down to one row
// (below four over lanes: the squares of a position come in fours), while half
// the height makes at most one tile a CU and leaves half the threads a value:
// 5 10^4 values took 130 us in 3 tiles of 4 rows at h = 5005 and take 85 in
// 10 of one, 52 -> 40 at h = 45 (9 tiles -> 139), 5 10^5 values 131 -> 91 at
// 5005, 70 -> 50 at 585 (54 -> 214).  More tiles than CUs gain nothing: 5 10^5
// values at h = 225 take 52 us in 139, 56 in 278, 62 in 556.
static bool over_lanes(u32 h, u32 l) { return h < 64 || l < 2; }
static u64 tile_bytes(u32 h, u32 l) { return 8ull * h * ((1ull << l) + (over_lanes(h, l) ? 2 : 0)); }
static u64 tile_count(u64 v, u32 l) { return (v + (1ull << l) - 1) >> l; }
static u32 tile_log(u32 h, u64 v) {
    u32 l = 2;
    const u32 most = over_lanes(h, l) ? 9 : 6;
    while (l < most && tile_bytes(h, l + 1) <= 80 * 1024) l++;
    while (l > 0 && tile_count(v, l - 1) <= 256 && (h << (l - 1)) >= RB / 2) l--;
    return l;
}
static_assert(8ull * NIF2_LDS_H * 4 <= 160 * 1024, "two rows and their sums fit LDS");
u32 nif2_lds_groups(u32 h, u64 v) {
    const u32 l = tile_log(h, v);
    const u64 tiles = tile_count(v, l), most = 256 * std::min<u64>(4, 160 * 1024 / tile_bytes(h, l));
    return (u32)((std::min<u64>(tiles, most) + 7) / 8 * 8);
}

hipError_t launch_nif2_rows_lds(hipStream_t st, const PfaPlan &pl, const u64 *a, u64 n, u64 v, u64 xi, u32 *pos,
                                u64 *tw, u64 *part, u64 *msgs, u32 *flag) {
    RowArgs r;
    r.h = pl.h;
    r.nf = pl.nf;
    r.logty = tile_log(pl.h, v);
    r.ntiles = (u32)tile_count(v, r.logty);
    r.full = (u32)(n / v);
    r.rem = n % v;
    r.v = v;
    r.a = a;
    r.pos = pos;
    r.tw = tw;
    r.part = part;
    r.flag = flag;
    u32 at = 0;
    const u64 half = 1ull << 60;  // 1/2
    for (u32 q = 0; q < 2 * pl.nf; q++) {
        const u32 d = q < pl.nf ? q : q - pl.nf, F = pl.F[d], f = F == 25 ? 5 : F, M = (f - 1) / 2;
        const u64 w = q < pl.nf ? pl.winv[d] : pl.wfwd[d], wi = q < pl.nf ? pl.wfwd[d] : pl.winv[d];
        const u64 u = F == 25 ? fp::pow(w, 5) : w, ui = F == 25 ? fp::pow(wi, 5) : wi;
        r.F[d] = F;
        r.stride[d] = pl.stride[d];
        r.root_at[q] = at;
        if (at + M + f - 1 + 16 > NIF2_LDS_ROOTS) return hipErrorInvalidValue;
        auto put = [&](u64 c) { r.roots[at++] = Half{(u32)c & 0x7fffffffu, (u32)(c >> 31)}; };
        for (u32 j = 1; j <= M; j++) put(mul(add(fp::pow(u, j), fp::pow(ui, j)), half));
        for (u32 j = 1; j < f; j++) put(mul(sub(fp::pow(u, j), fp::pow(ui, j)), half));
        if (F == 25)
            for (u32 n2 = 1; n2 < 5; n2++)
                for (u32 k1 = 1; k1 < 5; k1++) put(fp::pow(w, n2 * k1));
    }
    const u32 nwg = nif2_lds_groups(pl.h, v), lds = (u32)tile_bytes(pl.h, r.logty);
    hipLaunchKernelGGL(k_nif2_tables, dim3((pl.h + NT - 1) / NT), dim3(NT), 0, st, pl, xi, fp::inv(pl.h), pos, tw);
    const u32 nc = (pl.h + RB - 1) / RB;
#define RK(N) hipLaunchKernelGGL(k_nif2_rows_lds<N>, dim3(nwg), dim3(RB), lds, st, r)
    if (over_lanes(pl.h, r.logty)) RK(0);
    else if (nc <= 1) RK(1);
    else if (nc <= 3) RK(3);
    else if (nc <= 5) RK(5);
    else RK(10);
#undef RK
    hipLaunchKernelGGL(k_nif2_parts, dim3((2 * pl.h + 31) / 32), dim3(1024), 0, st, pl, part, nwg, msgs);
    return hipGetLastError();
}

// ------------------------------------------------------------ reductions

// Sum of one value per thread over the first NT threads, returned to thread 0.
__device__ __forceinline__ u64 group_sum(u64 v) {
    __shared__ u64 sm[NT / 64];
    for (int o = 32; o > 0; o >>= 1) {
        const int lo = __shfl_down((int)(u32)v, o), hi = __shfl_down((int)(u32)(v >> 32), o);
        v = add(v, ((u64)(u32)hi << 32) | (u32)lo);
    }
    if ((threadIdx.x & 63) == 0 && threadIdx.x < NT) sm[threadIdx.x >> 6] = v;
    __syncthreads();
    u64 t = 0;
    if (threadIdx.x == 0)
        for (int w = 0; w < NT / 64; w++) t = add(t, sm[w]);
    return t;
}

// Sum of squares of `cnt` words at src[0 .. cnt) (only i < lim count), in
// u128 with a reduction every 16 terms.
__device__ __forceinline__ u64 sq_sum(const u64 *src, u64 cnt, u64 off, u64 lim) {
    u64 s = 0;
    u128 acc = 0;
    u32 t = 0;
    for (u64 y = threadIdx.x; y < cnt; y += NT) {
        const u64 x = off + y < lim ? src[y] : 0;
        acc += fp::wide(x, x);
        if (++t == 16) {
            s = add(s, fp::red128(acc));
            acc = 0;
            t = 0;
        }
    }
    return add(s, fp::red128(acc));
}

// Workgroup (k, c): the part of g(xi^k) = sum_y (value k of row y)^2 over
// rows [c ch, (c + 1) ch), into part[k S + c].
__global__ void __launch_bounds__(NT) k_nif2_colsum(const PfaPlan pl, const u64 *__restrict__ a, u64 n, u64 v,
                                                    const u64 *__restrict__ W, u64 ch, u32 S, u64 *part) {
    const u32 k = blockIdx.x / S, c = blockIdx.x % S;
    const u64 y0 = c * ch, cnt = y0 < v ? std::min<u64>(ch, v - y0) : 0;
    const u64 j = k >> 1;
    u64 s;
    if ((k & 1) == 0) {
        s = sq_sum(a + j * v + y0, cnt, j * v + y0, n);
    } else {
        u64 pos = 0;  // f_y(xi w^j) sits at the position whose Good index is j
        for (u32 i = 0; i < pl.nf; i++) pos += (j * pl.ginv[i] % pl.F[i]) * pl.stride[i];
        s = sq_sum(W + pos * v + y0, cnt, 0, cnt);
    }
    s = group_sum(s);
    if (threadIdx.x == 0) part[(u64)k * S + c] = s;
}

// msgs[k] = sum_c part[k S + c]
__global__ void k_nif2_colfin(const u64 *__restrict__ part, u32 S, u32 K, u64 *msgs) {
    const u32 k = blockIdx.x * NT + threadIdx.x;
    if (k >= K) return;
    u64 s = 0;
    for (u32 c = 0; c < S; c++) s = add(s, part[(u64)k * S + c]);
    msgs[k] = s;
}

u32 nif2_colsum_split(u32 h, u64 v) {
    // about 2048 workgroups in all, each over at least 4096 rows
    const u64 want = std::max<u64>(1, 2048 / (2ull * h));
    return (u32)std::max<u64>(1, std::min<u64>(want, v / 4096));
}

hipError_t launch_nif2_colsum(hipStream_t st, const PfaPlan &pl, const u64 *a, u64 n, u64 v, const u64 *W,
                              u64 *part, u64 *msgs) {
    const u32 S = nif2_colsum_split(pl.h, v);
    const u64 ch = (v + S - 1) / S;
    hipLaunchKernelGGL(k_nif2_colsum, dim3(2 * pl.h * S), dim3(NT), 0, st, pl, a, n, v, W, ch, S, part);
    hipLaunchKernelGGL(k_nif2_colfin, dim3((2 * pl.h + NT - 1) / NT), dim3(NT), 0, st, part, S, 2 * pl.h, msgs);
    return hipGetLastError();
}

__global__ void k_nif2_twist(u32 h, u64 xi, u64 hinv, u64 *tw) {
    const u32 k = blockIdx.x * NT + threadIdx.x;
    if (k < h) tw[k] = mul(fp::pow(xi, k), hinv);
}

hipError_t launch_nif2_twist(hipStream_t st, u32 h, u64 xi, u64 *tw) {
    hipLaunchKernelGGL(k_nif2_twist, dim3((h + NT - 1) / NT), dim3(NT), 0, st, h, xi, fp::inv(h), tw);
    return hipGetLastError();
}

// ------------------------------------------------------------- verifier

// The Lagrange bases at r of the order-h subgroup <w> (L[j], j < h) and the
// order-2h subgroup <xi> (L[h + k], k < 2h): w^j (r^N - 1) / (N (r - w^j)), or
// [w^j == r] when r^N = 1.  Clears the flag as well.
__global__ void k_nif2_bases(u64 w, u64 xi, u64 h, u64 r, u64 rh1, u64 r2h1, u64 *L, u32 *flag) {
    const u64 t = (u64)blockIdx.x * NT + threadIdx.x;
    if (t == 0) *flag = 0;
    if (t >= 3 * h) return;
    const u64 N = t < h ? h : 2 * h, rN1 = t < h ? rh1 : r2h1;
    const u64 wj = t < h ? fp::pow(w, t) : fp::pow(xi, t - h);
    if (rN1 == 0)
        L[t] = wj == r ? 1 : 0;
    else
        L[t] = mul(mul(wj, rN1), fp::inv(mul(N % P, sub(r, wj))));
}

// Verifier's pass over the grid: out[pb + b] = the sum over workgroup pb + b's
// rows y of (sum_j a(j, y) L[j])^2, and out[0 .. pb) add up to sum_k msgs[k]
// L[h + k], PROOF_WORDS of the proof a workgroup, all its loads in flight: the
// proof is in host memory, and one workgroup for all of it waited a trip over
// the link for every 512 words (a verification of 5 10^4 values at h = 225225
// 1497 us, now 736; at h = 5005 60, now 56).  RW adjacent rows at a time, RB / RW threads a row taking every
// (RB / RW)-th column, eight loads in flight; values are checked against p as
// they pass.  One read of the grid: 200 MB in 37 us at h = 585 (a range check,
// a pass of 32-column parts and their squares before: 72 us in three).
constexpr u32 PROOF_WORDS = 4 * RB;
static_assert((2 * NIF2_MAX_H + PROOF_WORDS - 1) / PROOF_WORDS < NIF2_ROW_BLOCKS, "workgroups left for the rows");
template <int RW>
__global__ void __launch_bounds__(RB) k_nif2_rowsum(const u64 *__restrict__ a, u32 h, u32 full, u64 rem, u64 v,
                                                    const u64 *__restrict__ L, const u64 *__restrict__ msgs, u32 pb,
                                                    u64 *out, u32 *flag) {
    constexpr u32 G = RB / RW, U = 8;
    __shared__ u64 sm[G][RW];
    const u32 tid = threadIdx.x, y = tid % RW, g = tid / RW;
    u64 s = 0;
    if (blockIdx.x < pb) {
        constexpr u32 W = PROOF_WORDS / RB;
        const u32 k0 = blockIdx.x * PROOF_WORDS + tid;
        u64 m[W];
#pragma unroll
        for (u32 i = 0; i < W; i++) m[i] = k0 + i * RB < 2 * h ? msgs[k0 + i * RB] : 0;
#pragma unroll
        for (u32 i = 0; i < W; i++)
            if (k0 + i * RB < 2 * h) s = add(s, mul(m[i], L[h + k0 + i * RB]));
    } else {
        u64 bad = 0;
        for (u64 y0 = (u64)(blockIdx.x - pb) * RW; y0 < v; y0 += (u64)(gridDim.x - pb) * RW) {
            const u64 row = y0 + y;
            const u32 cols = row < v ? full + (row < rem ? 1u : 0u) : 0u;
            u64 t = 0;
            for (u32 j0 = g; j0 < cols; j0 += G * U) {
                u64 x[U], w[U];
#pragma unroll
                for (u32 i = 0; i < U; i++) {
                    const u32 j = j0 + i * G;
                    x[i] = j < cols ? a[(u64)j * v + row] : 0;
                    w[i] = j < cols ? L[j] : 0;
                }
                u128 acc = 0;
#pragma unroll
                for (u32 i = 0; i < U; i++) {
                    bad |= x[i] >= P;
                    acc += fp::wide(x[i], w[i]);
                }
                t = add(t, fp::red128(acc));
            }
            __syncthreads();  // the previous rows' sums are read
            sm[g][y] = t;
            __syncthreads();
            if (tid < RW) {
                for (u32 k = 1; k < G; k++) t = add(t, sm[k][y]);
                s = add(s, mul(t, t));
            }
        }
        if (bad) *flag = 1;
    }
    // (RB threads; NT of them hold a group_sum)
    __shared__ u64 half[RB - NT];
    __syncthreads();
    if (tid >= NT) half[tid - NT] = s;
    __syncthreads();
    if (tid < RB - NT) s = add(s, half[tid]);
    s = group_sum(s);
    if (tid == 0) out[blockIdx.x] = s;
}

// Rows a workgroup takes at a time: 512, a thread a row, where rows are short;
// else 64 while they fill the chip.
static u64 rowsum_rows(u32 h, u64 v) { return v < 64 * 512 ? 16 : h > 64 ? 64 : 512; }
u32 nif2_proof_blocks(u32 h) { return (2 * h + PROOF_WORDS - 1) / PROOF_WORDS; }
u32 nif2_rowsum_blocks(u32 h, u64 v) {
    const u64 rw = rowsum_rows(h, v), b = (v + rw - 1) / rw;
    return nif2_proof_blocks(h) + (u32)std::min<u64>(b, NIF2_ROW_BLOCKS - nif2_proof_blocks(h));
}

hipError_t launch_nif2_verify(hipStream_t st, const u64 *a, u64 n, u64 v, u32 h, u64 w, u64 xi, u64 r, u64 *L,
                              const u64 *msgs, u64 *out, u32 *flag) {
    const u64 rh = fp::pow(r, h);
    hipLaunchKernelGGL(k_nif2_bases, dim3((3 * h + NT - 1) / NT), dim3(NT), 0, st, w, xi, (u64)h, r, sub(rh, 1),
                       sub(mul(rh, rh), 1), L, flag);
    const dim3 g(nif2_rowsum_blocks(h, v));
    const u64 rw = rowsum_rows(h, v);
    const u32 full = (u32)(n / v), pb = nif2_proof_blocks(h);
    const u64 rem = n % v;
    if (rw == 512)
        hipLaunchKernelGGL(k_nif2_rowsum<512>, g, dim3(RB), 0, st, a, h, full, rem, v, L, msgs, pb, out, flag);
    else if (rw == 64)
        hipLaunchKernelGGL(k_nif2_rowsum<64>, g, dim3(RB), 0, st, a, h, full, rem, v, L, msgs, pb, out, flag);
    else
        hipLaunchKernelGGL(k_nif2_rowsum<16>, g, dim3(RB), 0, st, a, h, full, rem, v, L, msgs, pb, out, flag);
    return hipGetLastError();
}

__global__ void k_nif2_range(const u64 *__restrict__ a, u64 n, u32 *flag) {
    for (u64 i = (u64)blockIdx.x * NT + threadIdx.x; i < n; i += (u64)gridDim.x * NT)
        if (a[i] >= P) flag[0] = 1;
}

hipError_t launch_nif2_range(hipStream_t st, const u64 *a, u64 n, u32 *flag) {
    hipLaunchKernelGGL(k_nif2_range, dim3(grid_of(n)), dim3(NT), 0, st, a, n, flag);
    return hipGetLastError();
}

}  // namespace gkr

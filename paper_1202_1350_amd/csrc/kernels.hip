// kernels.hip -- HIP kernels (gfx950) of the GKR verifier over F_p, p =
// 2^61 - 1: the wiring predicates at a point and the inputs' extension.
//
// A workgroup sums its share (wave64 shuffles, then LDS) into one row of
// partial sums, which the host adds up.  All arithmetic is exact modular
// integer arithmetic (no floating point, Sec. 6.1), so any summation order
// gives identical bits.
#include <algorithm>

#include "fp61.hpp"
#include "kernels.hpp"

namespace gkr {

using fp::add;
using fp::mul;
using fp::P;
using fp::sub;

#define GTID ((u64)blockIdx.x * blockDim.x + threadIdx.x)
#define GSTRIDE ((u64)gridDim.x * blockDim.x)

// ---------------------------------------------------------------- reductions

template <int K>
__device__ __forceinline__ void wave_reduce(u64 (&v)[K]) {
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) {
#pragma unroll
        for (int k = 0; k < K; k++) v[k] = add(v[k], __shfl_xor(v[k], o));
    }
}

// Sum v over the workgroup; thread k < K writes total k to out[k].
template <int K>
__device__ __forceinline__ void block_store(u64 (&v)[K], u64 *out) {
    __shared__ u64 sm[K][BLOCK / 64];
    wave_reduce<K>(v);
    const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
    if (lane == 0) {
#pragma unroll
        for (int k = 0; k < K; k++) sm[k][wid] = v[k];
    }
    __syncthreads();
    if (threadIdx.x < K) {
        u64 a = 0;
#pragma unroll
        for (int w = 0; w < BLOCK / 64; w++) a = add(a, sm[threadIdx.x][w]);
        out[threadIdx.x] = a;
    }
}

// --------------------------------------------------------- proof bookkeeping

// chi over the bits of x of the coordinates pt[0..n)
__device__ __forceinline__ u64 chi_bits(u64 x, const u64 *pt, u32 n) {
    u64 e = 1;
    for (u32 k = 0; k < n; k++) e = mul(e, fp::eqbit((u32)((x >> k) & 1), pt[k]));
    return e;
}

// ---------------------------------------------------------- verifier (a10)
//
// All layers in two launches: a layer's own launches (three tables, a pass, a
// reduction) are a few thousand gates' work and cost their launch latencies
// (the MatMult check at N = 64, 66 such layers: 330 launches, 1.5 ms a
// verification; two launches, with the host's replay beside them, 0.07 ms).

// The layer of workgroup b.
template <u32 WireLayer::*FIRST>
__device__ __forceinline__ u32 layer_of(const WireLayer *L, u32 n, u32 b) {
    u32 lo = 0, hi = n;
    while (hi - lo > 1) {
        const u32 mid = (lo + hi) >> 1;
        if (L[mid].*FIRST <= b) lo = mid; else hi = mid;
    }
    return lo;
}

__global__ void __launch_bounds__(BLOCK) k_wire_eq(const WireLayer *__restrict__ L, u32 n, const u64 *__restrict__ pts) {
    const WireLayer &w = L[layer_of<&WireLayer::eq0>(L, n, blockIdx.x)];
    u64 x = (u64)(blockIdx.x - w.eq0) * BLOCK + threadIdx.x;
    u64 *tab = w.tab + x;
    // the half this entry is of
    const u32 bits[6] = {w.La, w.s - w.La, w.Lb, w.sp - w.Lb, w.Lb, w.sp - w.Lb};
    u32 at = w.pt;
#pragma unroll
    for (u32 h = 0; h < 6; h++) {
        const u64 len = 1ull << bits[h];
        if (x < len) {
            *tab = chi_bits(x, pts + at, bits[h]);
            return;
        }
        x -= len;
        at += bits[h];
    }
}

__global__ void __launch_bounds__(BLOCK) k_wiring(const WireLayer *__restrict__ L, u32 n, u64 *out) {
    const u32 q = layer_of<&WireLayer::block0>(L, n, blockIdx.x);
    const WireLayer &w = L[q];
    const u32 lb = blockIdx.x - w.block0, nb = L[q + 1].block0 - w.block0;
    const u64 am = (1ull << w.La) - 1, bm = (1ull << w.Lb) - 1;
    const u64 *alo = w.tab, *ahi = alo + (1ull << w.La), *blo = ahi + (1ull << (w.s - w.La));
    const u64 *bhi = blo + (1ull << w.Lb), *clo = bhi + (1ull << (w.sp - w.Lb)), *chi = clo + (1ull << w.Lb);
    u64 acc[2] = {0, 0};
    for (u64 g = (u64)lb * BLOCK + threadIdx.x; g < w.S; g += (u64)nb * BLOCK) {
        const u32 i1 = w.in1[g], i2 = w.in2[g];
        const u64 ea = mul(alo[g & am], ahi[g >> w.La]);
        const u64 eb = mul(blo[i1 & bm], bhi[i1 >> w.Lb]);
        const u64 ec = mul(clo[i2 & bm], chi[i2 >> w.Lb]);
        const u64 e = mul(ea, mul(eb, ec));
        const bool ismul = w.kind == KIND_MUL || (w.kind == KIND_MIXED && w.type[g]);
        acc[0] = add(acc[0], ismul ? 0 : e);
        acc[1] = add(acc[1], ismul ? e : 0);
    }
    block_store<2>(acc, out + 2 * (u64)blockIdx.x);
}

u64 wire_table_words(u32 s, u32 sp) {
    return (1ull << (s / 2)) + (1ull << (s - s / 2)) + 2 * ((1ull << (sp / 2)) + (1ull << (sp - sp / 2)));
}
u32 wire_eq_blocks(u32 s, u32 sp) { return (u32)((wire_table_words(s, sp) + BLOCK - 1) / BLOCK); }
u32 wire_gate_blocks(u32 S, u64 blocks_all) {
    // The layers of a launch share WIRE_BLOCKS workgroups (eight a CU, all the
    // chip holds at once) by gates: a thread's gates are a chain of dependent
    // gathers, so one wide layer needs them all (2^24 gates: 218 us a
    // verification, 302 with 256 workgroups a layer), and many layers no more
    // (78 layers of F0 on 100003 values 117 us, 147 with two gates a thread).
    const u64 b = wire_blocks_wanted(S);
    return (u32)(blocks_all <= WIRE_BLOCKS ? b : std::max<u64>(1, b * WIRE_BLOCKS / blocks_all));
}

hipError_t launch_wiring(hipStream_t st, const WireLayer *L, u32 n, u32 eq_blocks, u32 gate_blocks, const u64 *pts,
                         u64 *out) {
    hipLaunchKernelGGL(k_wire_eq, dim3(eq_blocks), dim3(BLOCK), 0, st, L, n, pts);
    hipLaunchKernelGGL(k_wiring, dim3(gate_blocks), dim3(BLOCK), 0, st, L, n, out);
    return hipGetLastError();
}

// Multilinear extension of T at the point pt: a workgroup takes tiles of
// BLOCK * E values, a thread the same E places of every tile, so a value's
// weight is chi of the tile's index (one scalar a tile, formed ahead in LDS,
// 256 tiles at a time) times chi of its place in the tile (E weights a
// thread, applied once at the end).  Bound by the read of T: 268 MB of counts
// in 52 us, 5.2 TB/s (58 us with a weight table read and a four-byte load a
// value).  VEC values a load: 16 bytes, or one value from unaligned input.
template <typename T, int VEC>
struct alignas(sizeof(T) * VEC) Vec {
    T v[VEC];
};
template <typename T, int VEC>
__global__ void __launch_bounds__(BLOCK) k_mle(u64 n, const T *__restrict__ in, const MlePoint pt, u64 x0, u64 *partials,
                                               int accumulate, u32 *bad) {
    constexpr int LN = VEC == 4 ? 1 : 2, NL = 1 << LN;  // loads a thread and tile
    constexpr int LV = VEC == 4 ? 2 : VEC == 2 ? 1 : 0, E = NL * VEC;
    constexpr int LT = LN + LV + 8;  // log2 of the tile
    static_assert(BLOCK == 256 && (1 << LT) == BLOCK * E, "a tile is 2^LT values");
    // sums of products below 2^122 are reduced every 32 tiles; those of
    // 32-bit counts (below 2^93) hold all of a workgroup's tiles
    constexpr bool REDUCE = sizeof(T) == 8;
    __shared__ u64 s_w[BLOCK];
    const u32 tid = threadIdx.x;
    const u64 tiles = (n + (1u << LT) - 1) >> LT;
    fp::u128 acc[E];
    u64 sum[E];
#pragma unroll
    for (int e = 0; e < E; e++) acc[e] = 0, sum[e] = 0;
    u32 terms = 0;
    u64 over = 0;
    for (u64 q0 = blockIdx.x; q0 < tiles; q0 += (u64)BLOCK * gridDim.x) {
        {  // weights of this workgroup's next tiles
            const u64 q = q0 + (u64)tid * gridDim.x, hi = (x0 >> LT) + q;
            u64 w = 1;
            if (q < tiles)
                for (u32 k = LT; k < pt.s; k++) w = mul(w, fp::eqbit((u32)(hi >> (k - LT)) & 1, pt.r[k]));
            __syncthreads();
            s_w[tid] = w;
            __syncthreads();
        }
        for (u32 k = 0; k < BLOCK; k++) {
            const u64 q = q0 + (u64)k * gridDim.x;
            if (q >= tiles) break;  // (uniform)
            const u64 base = q << LT, w = s_w[k];
            T v[E];
            if (base + (1u << LT) <= n) {
#pragma unroll
                for (int i = 0; i < NL; i++) {
                    const Vec<T, VEC> x = *reinterpret_cast<const Vec<T, VEC> *>(in + base + ((u64)i * BLOCK + tid) * VEC);
#pragma unroll
                    for (int c = 0; c < VEC; c++) v[i * VEC + c] = x.v[c];
                }
            } else {
#pragma unroll
                for (int e = 0; e < E; e++) {
                    const u64 x = base + ((u64)(e / VEC) * BLOCK + tid) * VEC + e % VEC;
                    v[e] = x < n ? in[x] : 0;
                }
            }
#pragma unroll
            for (int e = 0; e < E; e++) {
                if (sizeof(T) == 8) over |= (u64)v[e] >= P;
                acc[e] += fp::wide(w, (u64)v[e]);
            }
            if (REDUCE && ++terms == 32) {
                terms = 0;
#pragma unroll
                for (int e = 0; e < E; e++) sum[e] = add(sum[e], fp::red128(acc[e])), acc[e] = 0;
            }
        }
    }
    // weights of the thread's places: bits [0, LV) of the value in its load,
    // then the thread's eight, then the load's LN (a point's missing
    // coordinates are 0: their factor is 1)
    u64 tot[1] = {0};
    u64 wt = 1;
    for (u32 k = 0; k < 8; k++) wt = mul(wt, fp::eqbit((tid >> k) & 1, pt.r[LV + k]));
#pragma unroll
    for (int i = 0; i < NL; i++) {
        fp::u128 t = 0;
#pragma unroll
        for (int c = 0; c < VEC; c++) {
            u64 wc = 1;
#pragma unroll
            for (int b = 0; b < LV; b++) wc = mul(wc, fp::eqbit((c >> b) & 1, pt.r[b]));
            t += fp::wide(wc, add(sum[i * VEC + c], fp::red128(acc[i * VEC + c])));
        }
        u64 wi = fp::eqbit(i & 1, pt.r[LV + 8]);
        if (LN == 2) wi = mul(wi, fp::eqbit(i >> 1, pt.r[LV + 9]));
        tot[0] = add(tot[0], mul(fp::red128(t), wi));
    }
    tot[0] = mul(tot[0], wt);
    if (sizeof(T) == 8 && over) *bad = 1;
    __shared__ u64 res[1];
    block_store<1>(tot, res);
    __syncthreads();
    if (tid == 0) partials[blockIdx.x] = accumulate ? add(partials[blockIdx.x], res[0]) : res[0];
}

int mle_blocks(u64 n) {
    // 16 values a thread before another workgroup starts, eight workgroups a CU
    return (int)std::max<u64>(1, std::min<u64>(MLE_BLOCKS, (n + 16 * BLOCK - 1) / (16 * BLOCK)));
}

hipError_t launch_mle(hipStream_t st, u64 n, const u64 *T64, const u32 *T32, const MlePoint &pt, u64 x0, u64 *partials,
                      int nb, int accumulate, u32 *bad) {
    const bool wide16 = ((uintptr_t)(T64 ? (const void *)T64 : (const void *)T32) & 15) == 0;
    const dim3 g(nb), b(BLOCK);
    if (T64 && wide16)
        hipLaunchKernelGGL((k_mle<u64, 2>), g, b, 0, st, n, T64, pt, x0, partials, accumulate, bad);
    else if (T64)
        hipLaunchKernelGGL((k_mle<u64, 1>), g, b, 0, st, n, T64, pt, x0, partials, accumulate, bad);
    else if (wide16)
        hipLaunchKernelGGL((k_mle<u32, 4>), g, b, 0, st, n, T32, pt, x0, partials, accumulate, bad);
    else
        hipLaunchKernelGGL((k_mle<u32, 1>), g, b, 0, st, n, T32, pt, x0, partials, accumulate, bad);
    return hipGetLastError();
}

// ------------------------------------------------------------ field check

__global__ void __launch_bounds__(BLOCK) k_field_op(int op, const u64 *a, const u64 *b, u64 *out,
                                                    u64 n) {
    for (u64 i = GTID; i < n; i += GSTRIDE) {
        if (op == 4) {
            // 256 dependent products per element: independent chains across
            // elements, for measuring the product rate
            u64 x = a[i];
            const u64 y = b[i];
#pragma unroll 16
            for (int k = 0; k < 256; k++) x = mul(x, y);
            out[i] = x;
            continue;
        }
        if (op == 3) {
            fp::u128 s = 0;
            for (u64 j = 0; j < 64; j++) {
                const u64 k = (i + j) % n;
                s += fp::wide(a[k], b[k]);
            }
            out[i] = fp::red128(s);
            continue;
        }
        const u64 x = a[i], y = b[i];
        out[i] = op == 0 ? add(x, y) : (op == 1 ? sub(x, y) : mul(x, y));
    }
}

hipError_t launch_field_op(hipStream_t st, int op, const u64 *a, const u64 *b, u64 *out, u64 n) {
    hipLaunchKernelGGL(k_field_op, dim3(blocks_for(n, 4)), dim3(BLOCK), 0, st, op, a, b, out, n);
    return hipGetLastError();
}

}  // namespace gkr

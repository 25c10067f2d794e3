// kernels.hip -- HIP kernels (gfx950) of the GKR prover's per-layer
// sum-check over F_p, p = 2^61 - 1, and of its verifier.
//
// Sec. 4.1.1: each gate contributes independently to the prover's message;
// a workgroup sums its gates' contributions (wave64 shuffles, then LDS),
// writes one row of partial sums, and a one-workgroup *_final kernel folds
// the rows, writes the message and only then draws the next challenge on
// the device.  All arithmetic is exact modular integer arithmetic (no
// floating point, Sec. 6.1), so any summation order gives identical bits.
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

// ----------------------------------------------------------- evaluation (a3)

__global__ void __launch_bounds__(BLOCK) k_load_inputs(const u64 *src, u32 S, u64 npad, u64 *V,
                                                       u32 *bad) {
    u32 flag = 0;
    for (u64 g = GTID; g < npad; g += GSTRIDE) {
        u64 v = 0;
        if (g < S) {
            v = src[g];
            if (v >= P) flag = 1;
        }
        V[g] = v;
    }
    if (flag) atomicOr(bad, 1u);
}

hipError_t launch_load_inputs(hipStream_t st, const u64 *src, u32 S, u64 npad, u64 *V,
                              u32 *bad_flag) {
    hipLaunchKernelGGL(k_load_inputs, dim3(blocks_for(npad, 4)), dim3(BLOCK), 0, st, src, S, npad,
                       V, bad_flag);
    return hipGetLastError();
}

__global__ void __launch_bounds__(BLOCK) k_check_range(const u64 *src, u64 n, u32 *bad) {
    u32 flag = 0;
    for (u64 g = GTID; g < n; g += GSTRIDE) flag |= src[g] >= P;
    if (flag) atomicOr(bad, 1u);
}

hipError_t launch_check_range(hipStream_t st, const u64 *src, u64 n, u32 *bad_flag) {
    hipLaunchKernelGGL(k_check_range, dim3(blocks_for(n, 4)), dim3(BLOCK), 0, st, src, n, bad_flag);
    return hipGetLastError();
}

// --------------------------------------------------------- proof bookkeeping

// chi over the bits of x of the coordinates pt[0..n)
__device__ __forceinline__ u64 chi_bits(u64 x, const u64 *pt, u32 n) {
    u64 e = 1;
    for (u32 k = 0; k < n; k++) e = mul(e, fp::eqbit((u32)((x >> k) & 1), pt[k]));
    return e;
}

__global__ void __launch_bounds__(BLOCK) k_eq_halves(const u64 *pt, u32 s, u32 L, u64 *lo, u64 *hi) {
    const u64 nlo = 1ull << L, nhi = 1ull << (s - L);
    for (u64 x = GTID; x < nlo + nhi; x += GSTRIDE) {
        if (x < nlo)
            lo[x] = chi_bits(x, pt, L);
        else
            hi[x - nlo] = chi_bits(x - nlo, pt + L, s - L);
    }
}

hipError_t launch_eq_halves(hipStream_t st, const u64 *pt, u32 s, u32 L, u64 *lo, u64 *hi) {
    u64 n = (1ull << L) + (1ull << (s - L));
    hipLaunchKernelGGL(k_eq_halves, dim3(blocks_for(n)), dim3(BLOCK), 0, st, pt, s, L, lo, hi);
    return hipGetLastError();
}

// ---------------------------------------------------------- verifier (a10)

template <int KIND>
__global__ void __launch_bounds__(BLOCK) k_wiring(WiringArgs a) {
    const u64 am = (1ull << a.La) - 1, bm = (1ull << a.Lb) - 1, cm = (1ull << a.Lc) - 1;
    u64 acc[2] = {0, 0};
    for (u64 g = GTID; g < a.S; g += GSTRIDE) {
        const u32 i1 = a.in1[g], i2 = a.in2[g];
        const u64 ea = mul(a.alo[g & am], a.ahi[g >> a.La]);
        const u64 eb = mul(a.blo[i1 & bm], a.bhi[i1 >> a.Lb]);
        const u64 ec = mul(a.clo[i2 & cm], a.chi[i2 >> a.Lc]);
        const u64 e = mul(ea, mul(eb, ec));
        const bool ismul = KIND == KIND_MUL || (KIND == KIND_MIXED && a.type[g]);
        if (ismul)
            acc[1] = add(acc[1], e);
        else
            acc[0] = add(acc[0], e);
    }
    block_store<2>(acc, a.partials + 2 * (u64)blockIdx.x);
}

hipError_t launch_wiring(hipStream_t st, const WiringArgs &a, int *nblocks) {
    int nb = blocks_for(a.S, 4);
    *nblocks = nb;
    dim3 g(nb), b(BLOCK);
    if (a.kind == KIND_ADD) hipLaunchKernelGGL(k_wiring<KIND_ADD>, g, b, 0, st, a);
    else if (a.kind == KIND_MUL) hipLaunchKernelGGL(k_wiring<KIND_MUL>, g, b, 0, st, a);
    else hipLaunchKernelGGL(k_wiring<KIND_MIXED>, g, b, 0, st, a);
    return hipGetLastError();
}

template <bool WIDE>
__global__ void __launch_bounds__(BLOCK) k_mle(u64 n, const u64 *T64, const u32 *T32, const u64 *lo,
                                               const u64 *hi, u32 L, u64 *partials, int accumulate) {
    const u64 mask = (1ull << L) - 1;
    u64 acc[1] = {0};
    if ((GSTRIDE & mask) == 0) {
        // every x of this thread has the same low bits: chi_x = lo[x & mask]
        // hi[x >> L], so the thread sums hi[x >> L] v_x exactly in 128 bits
        // (reduced every 32 terms: 32 products below 2^122 fit) and
        // multiplies by its lo once
        u64 s = 0;
        fp::u128 w = 0;
        u32 k = 0;
        for (u64 x = GTID; x < n; x += GSTRIDE) {
            w += WIDE ? fp::wide(hi[x >> L], T64[x]) : fp::wide(hi[x >> L], (u64)T32[x]);
            if (++k == 32) {
                s = add(s, fp::red128(w));
                w = 0;
                k = 0;
            }
        }
        s = add(s, fp::red128(w));
        acc[0] = GTID < n ? mul(s, lo[GTID & mask]) : 0;
    } else {
        for (u64 x = GTID; x < n; x += GSTRIDE) {
            const u64 v = WIDE ? T64[x] : (u64)T32[x];
            acc[0] = add(acc[0], mul(mul(lo[x & mask], hi[x >> L]), v));
        }
    }
    __shared__ u64 tot[1];
    block_store<1>(acc, tot);
    __syncthreads();
    if (threadIdx.x == 0) partials[blockIdx.x] = accumulate ? add(partials[blockIdx.x], tot[0]) : tot[0];
}

hipError_t launch_mle(hipStream_t st, u64 n, const u64 *T64, const u32 *T32, const u64 *lo,
                      const u64 *hi, u32 L, u64 *partials, int *nblocks, int accumulate, int nb_fixed) {
    const int nb = nb_fixed > 0 ? nb_fixed : blocks_for(n, 8);
    *nblocks = nb;
    if (T64)
        hipLaunchKernelGGL(k_mle<true>, dim3(nb), dim3(BLOCK), 0, st, n, T64, T32, lo, hi, L, partials,
                           accumulate);
    else
        hipLaunchKernelGGL(k_mle<false>, dim3(nb), dim3(BLOCK), 0, st, n, T64, T32, lo, hi, L,
                           partials, accumulate);
    return hipGetLastError();
}

__global__ void __launch_bounds__(BLOCK) k_reduce_rows(int nparts, int K, const u64 *partials, u64 *out) {
    u64 v[4] = {0, 0, 0, 0};
    for (int r = threadIdx.x; r < nparts; r += BLOCK)
        for (int k = 0; k < K; k++) v[k] = add(v[k], partials[(u64)r * K + k]);
    __shared__ u64 res[4];
    block_store<4>(v, res);
    __syncthreads();
    if (threadIdx.x < K) out[threadIdx.x] = res[threadIdx.x];
}

hipError_t launch_reduce_rows(hipStream_t st, int nparts, int K, const u64 *partials, u64 *out) {
    hipLaunchKernelGGL(k_reduce_rows, dim3(1), dim3(BLOCK), 0, st, nparts, K, partials, out);
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

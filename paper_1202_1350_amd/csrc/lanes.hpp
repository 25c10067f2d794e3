// lanes.hpp -- exchanges and sums of u64 values over the lanes of a 64-wide
// wave (gfx950).  Every lane of the wave takes part in every call: select
// operands after an exchange, never around it.
#pragma once
#include "fp61.hpp"

namespace gkr {

using fp::u32;
using fp::u64;

// DPP move of one u64 as two 32-bit halves; lanes without a source read 0.
template <int CTRL, int ROWS = 0xf>
__device__ __forceinline__ u64 dppx(u64 v) {
    const int lo = __builtin_amdgcn_update_dpp(0, (int)(u32)v, CTRL, ROWS, 0xf, true);
    const int hi = __builtin_amdgcn_update_dpp(0, (int)(u32)(v >> 32), CTRL, ROWS, 0xf, true);
    return ((u64)(u32)hi << 32) | (u64)(u32)lo;
}
__device__ __forceinline__ u64 from1(u64 v) { return dppx<0xB1>(v); }       // lane ^ 1
__device__ __forceinline__ u64 from2(u64 v) { return dppx<0x4E>(v); }       // lane ^ 2
__device__ __forceinline__ u64 from3(u64 v) { return dppx<0x1B>(v); }       // lane ^ 3
__device__ __forceinline__ u64 from7(u64 v) { return dppx<0x141>(v); }      // lane ^ 7 (row_half_mirror)
__device__ __forceinline__ u64 from4(u64 v) { return from3(from7(v)); }     // lane ^ 4
__device__ __forceinline__ u64 from8(u64 v) { return dppx<0x128>(v); }      // lane ^ 8 (row_ror:8)

// v + its value in lane ^ 16 or ^ 32 (the swaps leave the two halves' values
// of every lane pair in both results).
typedef unsigned int u32x2 __attribute__((ext_vector_type(2)));
__device__ __forceinline__ u64 plus16(u64 v) {
    const u32x2 a = __builtin_amdgcn_permlane16_swap((u32)v, (u32)v, false, false);
    const u32x2 b = __builtin_amdgcn_permlane16_swap((u32)(v >> 32), (u32)(v >> 32), false, false);
    return (((u64)b.x << 32) | a.x) + (((u64)b.y << 32) | a.y);
}
__device__ __forceinline__ u64 plus32(u64 v) {
    const u32x2 a = __builtin_amdgcn_permlane32_swap((u32)v, (u32)v, false, false);
    const u32x2 b = __builtin_amdgcn_permlane32_swap((u32)(v >> 32), (u32)(v >> 32), false, false);
    return (((u64)b.x << 32) | a.x) + (((u64)b.y << 32) | a.y);
}
// The sum over lanes l and l ^ 32 (l ^ 16) of a in the lanes with that bit clear,
// of b in the others; not reduced.
__device__ __forceinline__ u64 swap32_sum(u64 a, u64 b) {
    const u32x2 x = __builtin_amdgcn_permlane32_swap((u32)a, (u32)b, false, false);
    const u32x2 y = __builtin_amdgcn_permlane32_swap((u32)(a >> 32), (u32)(b >> 32), false, false);
    return (((u64)y.x << 32) | x.x) + (((u64)y.y << 32) | x.y);
}
__device__ __forceinline__ u64 swap16_sum(u64 a, u64 b) {
    const u32x2 x = __builtin_amdgcn_permlane16_swap((u32)a, (u32)b, false, false);
    const u32x2 y = __builtin_amdgcn_permlane16_swap((u32)(a >> 32), (u32)(b >> 32), false, false);
    return (((u64)y.x << 32) | x.x) + (((u64)y.y << 32) | x.y);
}

// A value every lane holds the same copy of, moved to scalar registers.
__device__ __forceinline__ u64 uniform(u64 v) {
    const u32 lo = (u32)__builtin_amdgcn_readfirstlane((int)(u32)v);
    const u32 hi = (u32)__builtin_amdgcn_readfirstlane((int)(u32)(v >> 32));
    return ((u64)hi << 32) | lo;
}
__device__ __forceinline__ u64 lane_value(u64 v, u32 l) {  // l uniform
    const u32 lo = (u32)__builtin_amdgcn_readlane((int)(u32)v, l);
    const u32 hi = (u32)__builtin_amdgcn_readlane((int)(u32)(v >> 32), l);
    return ((u64)hi << 32) | lo;
}

__device__ __forceinline__ u64 reduced(u64 v) { return fp::canon(fp::fold64(v)); }

// Lane l ^ (1 << b)'s value, b < 4 uniform.
__device__ __forceinline__ u64 from_bit(u64 v, u32 b) {
    switch (b) {
        case 0: return from1(v);
        case 1: return from2(v);
        case 2: return from4(v);
        default: return from8(v);
    }
}
// v + lane ^ (1 << b)'s value, canonical, b uniform.
__device__ __forceinline__ u64 plus_bit(u64 v, u32 b) {
    if (b < 4) return fp::add(v, from_bit(v, b));
    return reduced(b == 4 ? plus16(v) : plus32(v));
}

// Sum over the wave of canonical values, in every lane: DPP prefix steps
// (eight values below p stay below 2^64, so three steps go unreduced), then
// lane 63's total.
__device__ __forceinline__ u64 wave_total(u64 v) {
    v += dppx<0x111>(v);  // row_shr:1, 2, 4
    v += dppx<0x112>(v);
    v += dppx<0x114>(v);
    v = reduced(v);
    v += dppx<0x118>(v);       // row_shr:8
    v += dppx<0x142, 0xa>(v);  // row_bcast:15 into rows 1, 3
    v += dppx<0x143, 0xc>(v);  // row_bcast:31 into rows 2, 3
    return lane_value(reduced(v), 63);
}

// Sum of canonical values over the eight lanes 8m .. 8m + 7, in each of them,
// below 2^64 and not reduced.
__device__ __forceinline__ u64 oct_total(u64 v) {
    v += from1(v);
    v += from2(v);
    return v + from7(v);
}
// Product over the lanes 16m .. 16m + 15, in each of them.
__device__ __forceinline__ u64 row_product(u64 v) {
    v = fp::mul(v, from1(v));
    v = fp::mul(v, from2(v));
    v = fp::mul(v, from7(v));
    return fp::mul(v, from8(v));
}

// Lane off + k (k < n, off + n <= 64) receives draw k of the challenge stream
// after state st (uniform), the other lanes x; st becomes the state after the
// draws.  A draw is the mix of its own counter, so the lanes draw side by
// side, unless one of them has to be redrawn (once in 2^61): then one after
// the other.
__device__ __forceinline__ u64 draw_lanes(u64 &st, u32 n, u32 off = 0, u64 x = 0) {
    const u32 k = (threadIdx.x & 63) - off;
    const u64 v = fp::sm_mix(st + fp::SM_GAMMA * (k + 1)) & fp::P;
    if (__builtin_expect(__ballot(k < n && v == fp::P) != 0, 0)) {
        for (u32 q = 0; q < n; q++) {
            const u64 r = fp::sm_field(st);
            if (k == q) x = r;
        }
        return x;
    }
    st += fp::SM_GAMMA * n;
    return k < n ? v : x;
}

}  // namespace gkr

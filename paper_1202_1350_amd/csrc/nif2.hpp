// nif2.hpp -- kernels of the non-interactive F2 protocol (Sec. 3.2,
// 4.2): the prover's per-row transforms over F_p and the column
// square-sums that form its proof, and the verifier's row evaluations.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace gkr {

typedef uint64_t u64;
typedef uint32_t u32;

constexpr int NIF2_MAXF = 5;  // coprime factors of h (3, 5, 7, 9, 11, 13, 25)

// The prime factor transform of a row of length h = F_0 ... F_{nf-1}
// (pairwise coprime): position P = sum d_i stride_i (mixed radix, digit
// d_i < F_i) holds index Good(P) = sum d_i (h / F_i) mod h before a
// transform and CRT(P) = sum d_i e_i mod h after it (e_i = 1 mod F_i,
// 0 mod F_j), or the other way round; the transform is then a product of
// F_i-point DFTs along the digits, with roots w^(h/F_i).
struct PfaPlan {
    u32 h, nf;
    u32 F[NIF2_MAXF], stride[NIF2_MAXF], gstep[NIF2_MAXF], cstep[NIF2_MAXF], ginv[NIF2_MAXF];
    u64 wfwd[NIF2_MAXF], winv[NIF2_MAXF];  // w^(h/F_i), w^(-h/F_i)
};

// Grid: element (position P, row y) of the transform buffer W at P v + y;
// input a_i at i = j v + y for row y, column j (zero for i >= n).
hipError_t launch_nif2_transform(hipStream_t st, const PfaPlan &pl, const u64 *a, u64 n, u64 v,
                                 const u64 *tw, u64 *W);
// Rows of at most NIF2_LDS_H values: the whole proof msgs[0 .. 2h) with each
// row transformed in LDS (no transform buffer), the range check included
// (flag[0] = 1 if some a_i >= p).  pos: h, tw: h, part: nif2_lds_groups(h, v)
// 2h words of scratch.
constexpr u32 NIF2_LDS_H = 5120;
constexpr int NIF2_LDS_NF = 4;      // factors of such an h (3 5 7 11 13 = 15015 is longer)
constexpr int NIF2_LDS_ROOTS = 160; // words of roots: at most 22 a pass
u32 nif2_lds_groups(u32 h, u64 v);
hipError_t launch_nif2_rows_lds(hipStream_t st, const PfaPlan &pl, const u64 *a, u64 n, u64 v, u64 xi, u32 *pos,
                                u64 *tw, u64 *part, u64 *msgs, u32 *flag);
// msgs[k] = sum_y (value k of row y)^2, k < 2h: even k from a, odd from W;
// each column is split over nif2_colsum_split(h, v) workgroups whose sums
// go through part (2h times that many words).
u32 nif2_colsum_split(u32 h, u64 v);
hipError_t launch_nif2_colsum(hipStream_t st, const PfaPlan &pl, const u64 *a, u64 n, u64 v,
                              const u64 *W, u64 *part, u64 *msgs);
// tw[k] = xi^k / h, k < h.
hipError_t launch_nif2_twist(hipStream_t st, u32 h, u64 xi, u64 *tw);
// The verifier at the secret r: out[0 .. nif2_proof_blocks(h)) add up to the
// value at r of the polynomial through the 2h proof values msgs
// (device-visible), out[nif2_proof_blocks(h) .. nif2_rowsum_blocks(h, v)) to
// sum_y f_y(r)^2; *flag = 1 if some a_i >= p (cleared first).  L: 3h scratch
// words.
constexpr u32 NIF2_ROW_BLOCKS = 1024;
constexpr u32 NIF2_MAX_H = 9 * 25 * 7 * 11 * 13;  // the longest row of the supported factors
u32 nif2_proof_blocks(u32 h);
u32 nif2_rowsum_blocks(u32 h, u64 v);
hipError_t launch_nif2_verify(hipStream_t st, const u64 *a, u64 n, u64 v, u32 h, u64 w, u64 xi, u64 r, u64 *L,
                              const u64 *msgs, u64 *out, u32 *flag);
// flag[0] = 1 if some a_i >= p.
hipError_t launch_nif2_range(hipStream_t st, const u64 *a, u64 n, u32 *flag);

}  // namespace gkr

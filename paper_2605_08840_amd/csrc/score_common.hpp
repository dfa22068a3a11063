// Pieces shared by the FP32 and the MFMA scoring paths: scratch pointers and the kernel
// that merges the key splits of the attention pass into per-query statistics.
#pragma once

#include <type_traits>

#include "common.hpp"

namespace restkv {

struct ScorePtrs {
  float* part_m; float* part_mx; int* part_n; float* part_ref; float* part_l; float* part_z;
  float* rs_m; float* rs_l; float* rs_zz; int* rs_nstar; float* rs_istar;
  float* vv;
  uint16_t* op;
};

inline ScorePtrs score_ptrs(char* ws, const ScoreWs& lay) {
  ScorePtrs p;
  p.part_m = (float*)(ws + lay.part_m); p.part_mx = (float*)(ws + lay.part_mx);
  p.part_n = (int*)(ws + lay.part_n);
  p.part_ref = (float*)(ws + lay.part_ref); p.part_l = (float*)(ws + lay.part_l);
  p.part_z = (float*)(ws + lay.part_z);
  p.rs_m = (float*)(ws + lay.rs_m); p.rs_l = (float*)(ws + lay.rs_l); p.rs_zz = (float*)(ws + lay.rs_zz);
  p.rs_nstar = (int*)(ws + lay.rs_nstar); p.rs_istar = (float*)(ws + lay.rs_istar);
  p.vv = (float*)(ws + lay.vv);
  p.op = (uint16_t*)(ws + lay.op);
  return p;
}

// One 1 KiB asynchronous copy global -> LDS: lane i moves the 16 bytes at base + voff_i to LDS bytes
// [16 i, 16 i + 16) of lds_dst.  base and lds_dst are wave-uniform.  Issued from inline asm and waited for
// with explicit s_waitcnt vmcnt(n).
__device__ __forceinline__ void dma_1k(const void* base, uint32_t voff, void* lds_dst) {
  const uint32_t dst =
      __builtin_amdgcn_readfirstlane((uint32_t)(uintptr_t)(__attribute__((address_space(3))) void*)lds_dst);
  const uint64_t sb = (uint64_t)base;
  const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)sb);
  const uint32_t hi = __builtin_amdgcn_readfirstlane((uint32_t)(sb >> 32));
  const uint64_t ub = ((uint64_t)hi << 32) | lo;
  asm volatile("s_mov_b32 m0, %2\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, %1" ::"v"(voff), "s"(ub), "s"(dst)
               : "memory", "m0");
}

// ---- planes -------------------------------------------------------------------
// FP32 values as bf16 planes: x = h + m + l, h the bf16 nearest to x, m the nearest to what is left, l the rest
// (exact, 8 + 8 + 8 bits, where PlaneRange says so).  A bf16 value has one plane.
typedef float f32x2 __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
template <typename T> inline constexpr int planes_of = 3;
template <> inline constexpr int planes_of<bf16_t> = 1;

// NP planes of eight values, as operand registers
template <int NP>
struct Op { uint4 p[NP]; };
__device__ __forceinline__ bf16x8 as_bf16x8(uint4 u) {
  union { uint4 u; bf16x8 b; } x;
  x.u = u;
  return x.b;
}
template <int NP>
__device__ __forceinline__ Op<NP> split8(const float (&x)[8]) {
  Op<NP> o;
  uint32_t w[NP][4];
  // (-1, 0) and (0, -1) as scalar registers: which half an inline constant of this instruction fills is not relied on
  uint32_t lo = 0x0000BF80u, hi = 0xBF800000u;
  if (NP > 1) asm("" : "+s"(lo), "+s"(hi));
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    float a = x[2 * e], b = x[2 * e + 1];
#pragma unroll
    for (int p = 0; p < NP; ++p) {
      const bf16x2 h = __builtin_convertvector(f32x2{a, b}, bf16x2);
      w[p][e] = __builtin_bit_cast(uint32_t, h);
      if (p + 1 < NP) {      // what is left (exact), each in one instruction
        a = __builtin_amdgcn_fdot2_f32_bf16(h, __builtin_bit_cast(bf16x2, lo), a, false);
        b = __builtin_amdgcn_fdot2_f32_bf16(h, __builtin_bit_cast(bf16x2, hi), b, false);
      }
    }
  }
#pragma unroll
  for (int p = 0; p < NP; ++p) o.p[p] = make_uint4(w[p][0], w[p][1], w[p][2], w[p][3]);
  return o;
}
template <int NP>
__device__ __forceinline__ Op<NP> split8(float4 a, float4 b) {
  const float x[8] = {a.x, a.y, a.z, a.w, b.x, b.y, b.z, b.w};
  return split8<NP>(x);
}

// Planes give products as the FP32 instruction does between values of which one side (q rows, u rows, Gram entries) lies in this
// range: groups of eight whose largest lies in (2^-40, 2^60), or of zeros.  What the other side's l plane loses below the bf16
// subnormals is then below 2^-73, and products of planes are normal numbers.  A value beyond the bf16 range, or an
// infinity, leaves inf - inf in its planes (and in its neighbour's, 0 * inf in the two-term product): every product with it is NaN.
// Whoever finds a value out of range, or such a sum, takes the FP32 instruction.
struct PlaneRange {
  uint32_t worst = 0u;                  // in halves: largest upper 16 bits of the groups' largest magnitudes, and of their negatives
  __device__ __forceinline__ void take(float4 a, float4 b) {
    float m = a.x;
    asm("v_max3_f32 %0, |%1|, |%2|, |%0|" : "+v"(m) : "v"(a.y), "v"(a.z));
    asm("v_max3_f32 %0, |%1|, |%2|, %0" : "+v"(m) : "v"(a.w), "v"(b.x));
    asm("v_max3_f32 %0, |%1|, |%2|, %0" : "+v"(m) : "v"(b.y), "v"(b.z));
    asm("v_max_f32_e64 %0, |%1|, %0" : "+v"(m) : "v"(b.w));
    const uint32_t u = __float_as_uint(m), both = __builtin_amdgcn_perm(u, 0u - u, 0x07060302u);
    asm("v_pk_max_u16 %0, %0, %1" : "+v"(worst) : "v"(both));
  }
  __device__ __forceinline__ bool out() const { return worst >= 0x5D800000u || (worst & 0xFFFFu) >= 0xD480u; }
};

// Rows of a head as the FP32 score pass takes them, an item per 32 window positions of a query head and kind (q, u):
// the planes in operand order ([plane][d/16][lane half][32 rows][8] bf16, so that an operand register is one 1 KiB
// run), then the rows' statistics ([32][4] f32; q: maximum, denominator; u: zz, champion, its score), the last of which is
// 1.0 for a row out of the planes' range, whose values are there in FP32: of eight the first four in the place of their
// h plane, the others in that of m.
constexpr int row_item(int d) { return (3 * d / 16 + 1) * 1024; }
inline __host__ __device__ int row_items(int W) { return (W + 31) / 32; }

// Per split s and query row the attention pass leaves (all logits in log2 units, scaled):
//   part_m    largest logit seen, -inf if the split saw no key
//   part_mx   logit of the key the split kept OUT of its sums (valid if part_n >= 0)
//   part_n    index of that key; without one -2 - (index of the largest logit's key) where the pass
//             tracks it (FP32 path, which keeps a key out only while it is the largest), else -1
//   part_ref  reference the sums are relative to
//   part_l    sum over the included keys of 2^(logit - ref)
//   part_z    sum over the included keys of 2^(logit - ref) * v
// A split keeps a key out when, on arrival, it is the largest so far and holds more than half
// of the mass seen so far (always true for a key that ends with more than half of the total).
// part_ref never follows a kept-out key, only keys that are part of the sums (on the matrix-core
// path: exactly the logit of a key that was heavy among the others when it arrived, so that its
// bf16 weight is exact).
// The merge keeps out the excluded key that is the overall maximum (if any) and folds every
// other excluded key back in.  With a key kept out ("champion", weight A* = 1/l):
//   l = 1 + l_rest, z = (v* + z_rest)/l, u = z M_h, zz = u.z, and the champion's indicator in its
//   leave-one-out form I* = A* ||(z_rest/l_rest - v*) W_O||  (Eq. ori with Eq. relation; equals
//   Eq. rec_ei).  Without one, l and z are the plain softmax sums relative to the maximum; the largest
//   key, where its index is known, then has A* <= 1/2, and the same form is the difference
//   A*/(1 - A*) ||(z - v*) W_O||.  Either way the difference is taken before its norm: the expanded
//   distance of the score pass cancels where v* lies near z.

// Statistics of a caller's own attention kernel come in as ONE split: the log-sum-exp of a row (pb.ext_lse, natural log) is
// both the reference and the "largest logit", the sum of weights is 1, no key is kept out, and the caller's attention
// output [Hq*W, d] is part_z (EXT; a launch that wrote them out took 2.3 us, and a test at run time costs every other
// merge 0.7 us).

// Merge of the key splits and the per-row quantities of the score pass, RQ query rows of one head
// per workgroup of 4 D threads.
//   * One wavefront per row brings in the row's per-split scalars (a lane each, S <= 64) and leaves
//     the splits' factors, the list of kept-out keys that join the sums, and the row's scalars.
//   * The sums over the splits: a thread owns four columns of a row; 16 / RQ threads share a row's
//     columns and take every (16 / RQ)-th split, so that few rows still mean many loads in flight.
//   * u = z M_h (and y = x M_h where a row has a champion) is a 16-row product on
//     v_mfma_f32_16x16x4_f32: a wavefront owns 16 columns, its Gram entries stay in registers
//     (loaded first, every entry needed by exactly one lane), z and x are LDS operands.  Up to eight rows
//     z and x share the block (a second block for x: whole path at 2112 tokens 70.5 us instead of 67.7).
// Bound by latency (three dependent round trips to memory) until the rows fill the chip, then by the
// partial sums, Gram matrices and operands it moves.  Against a kernel of four rows per workgroup
// with u on the vector ALU and value rows fetched for every split: 65536 rows x 1 split (32 layers of
// 2112 tokens folded) 207 -> 66 us, 2048 rows x 17 splits 15.8 -> 13.2 us, 1024 rows (window 32) 13.1
// -> 10.8 us, 4096 rows x 32 splits 24.6 -> 14.7 us, 2048 rows x 32 splits 19.5 -> 17.5 us.
// Workgroups of one KV head follow each other on one XCD (ids 8 apart): its L2 holds their Gram matrices
// and completes the cache lines that the heads of a group write in pieces.
// grid (Hq * ceil(W / RQ)), 4 D threads.
typedef float f32x4_t __attribute__((ext_vector_type(4)));

// reductions over groups of `w` lanes (a power of two)
__device__ __forceinline__ float group_sum(float x, int w) {
  for (int sh = w >> 1; sh >= 1; sh >>= 1) x += __shfl_xor(x, sh, 64);
  return x;
}
__device__ __forceinline__ float group_max(float x, int w) {
  for (int sh = w >> 1; sh >= 1; sh >>= 1) x = fmaxf(x, __shfl_xor(x, sh, 64));
  return x;
}
// sum over each row of 16 lanes (rotations, no LDS traffic)
__device__ __forceinline__ float row16_sum(float x) {
#define RK_ROR(n) x += __uint_as_float(__builtin_amdgcn_update_dpp(0u, __float_as_uint(x), 0x120 + (n), 0xF, 0xF, false))
  RK_ROR(8); RK_ROR(4); RK_ROR(2); RK_ROR(1);
#undef RK_ROR
  return x;
}
// four consecutive elements of a row, whatever its alignment
__device__ __forceinline__ f32x4_t quad_of(const float* p) {
  f32x4_t x;
  __builtin_memcpy(&x, p, 16);
  return x;
}
__device__ __forceinline__ f32x4_t quad_of(const bf16_t* p) {
  uint2 u;
  __builtin_memcpy(&u, p, 8);
  return f32x4_t{__uint_as_float(u.x << 16), __uint_as_float(u.x & 0xFFFF0000u), __uint_as_float(u.y << 16),
                 __uint_as_float(u.y & 0xFFFF0000u)};
}

// splits that the LDS lists of a workgroup hold (many rows come with few splits)
constexpr int combine_max_splits(int rq) { return rq >= 64 ? 8 : (rq >= 32 ? 16 : 64); }

template <typename T, int D, int RQ, int USE_OP, bool EXT>
__global__ __launch_bounds__(4 * D, 4) void k_attn_combine(Prob pb, const T* __restrict__ v, int S,
                                                           const float* __restrict__ gram, ScorePtrs o,
                                                           const float* __restrict__ part_z, const T* __restrict__ q,
                                                           int log2gp, int nwb) {
  constexpr int SMAX = combine_max_splits(RQ), NT = 4 * D, NWV = D / 16, CQ = D / 4, ZST = D + 4;
  constexpr int NP = RQ < 16 ? 16 / RQ : 1;              // threads that share a row's columns
  constexpr int MB = RQ < 16 ? 1 : RQ / 16;              // rows per thread, 16-row blocks of the product
  constexpr int SB = MB >= 4 ? 2 : (RQ <= 8 ? 8 : 4);    // splits in flight per row
  constexpr int JB = MB >= 2 || sizeof(T) == 4 ? 4 : 8;  // joining keys in flight per row (eight of float spill registers at D = 128)
  __shared__ __attribute__((aligned(16))) float zs[RQ][ZST];             // z of the rows
  __shared__ __attribute__((aligned(16))) float xs[RQ * NP][ZST];        // partial sums of the splits, then x, then u
  __shared__ float red[NWV][RQ][2];
  __shared__ float s_w[RQ][SMAX], s_jw[RQ][SMAX];
  __shared__ int s_jn[RQ][SMAX];
  __shared__ float s_fr[RQ], s_lrest[RQ];
  __shared__ int s_nj[RQ], s_nstar[RQ];
  const int tid = threadIdx.x, l = tid & 63, wv = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int npg = (pb.W + RQ - 1) / RQ;
  const int per = pb.G * npg, id = blockIdx.x, full = (pb.Hkv & ~7) * per;      // workgroups per KV head
  const int g = id < full ? (id / (8 * per)) * 8 + (id & 7) : id / per;
  const int wg = id < full ? (id >> 3) % per : id % per;
  const int h = g * pb.G + wg / npg, i0 = wg % npg * RQ;
  const T* vg = v + (int64_t)g * pb.kv_sh;
  const int SW = S <= 1 ? 1 : 1 << (32 - __builtin_clz((unsigned)(S - 1)));      // lanes per row
  const int sub = l & (SW - 1);
  // FP32 score pass: statistic k of window position i with the q rows (which = 0) or the u rows
  char* const items = (char*)o.op + (int64_t)h * row_items(pb.W) * 2 * row_item(D);
  auto item_of = [&](int i, int which) { return items + ((i >> 5) * 2 + which) * (int64_t)row_item(D); };
  auto stat = [&](int i, int which, int k) { return (float*)(item_of(i, which) + 3 * D / 16 * 1024) + (i & 31) * 4 + k; };
  const unsigned long long mine = SW >= 64 ? ~0ull : ((1ull << SW) - 1ull) << (l & ~(SW - 1));
  // what the workgroup needs from memory is asked for in the order in which it will be waited for:
  // the scalars, the first splits' sums, the Gram entries
  float pm, pmx, pref, pl;
  int pn;
  auto fetch_scalars = [&](int r) {
    const int64_t po = (int64_t)(h * pb.W + min(i0 + r, pb.W - 1)) * S + min(sub, S - 1);
    if constexpr (EXT) {
      pm = pref = pb.ext_lse[po] * 1.4426950408889634f; pmx = 0.f; pn = -1; pl = 1.f;
    } else {
      pm = o.part_m[po]; pmx = o.part_mx[po]; pn = o.part_n[po]; pref = o.part_ref[po]; pl = o.part_l[po];
    }
  };
  fetch_scalars(min(tid / SW, RQ - 1));
  const int c4 = 4 * (tid % CQ), rz = (tid / CQ) % (RQ / MB), part = tid / (CQ * (RQ / MB));
  const float* pz[MB];
  f32x4_t t[MB][SB];
#pragma unroll
  for (int m = 0; m < MB; ++m) pz[m] = part_z + (int64_t)(h * pb.W + min(i0 + rz + 16 * m, pb.W - 1)) * S * D + c4;
  auto fetch_splits = [&](int m, int s) {
#pragma unroll
    for (int k = 0; k < SB; ++k) t[m][k] = quad_of(pz[m] + (int64_t)min(s + k * NP, S - 1) * D);
  };
#pragma unroll
  for (int m = 0; m < MB; ++m) fetch_splits(m, part);
  // Gram entries of this lane: column 16 wv + l % 16, the K index of step 4 a + e being 16 a + 4 (l / 16) + e.  Heads of 128 read
  // them along rows of M (8/8 heads, 3.8k tokens 7.8 -> 7.3 us for the merge), heads of 64, a quarter of the entries, from the
  // row of the same number (M is symmetric), four at a time (32/8 heads, two layers of 3.5k, statistics in: 5.5 us against 5.7.  bf16
  // alone: in the FP32 path the same, 5.0 against 5.6, moves the code of the merge for heads of 128, which then takes 11.8 us for
  // 11.1 at 8k with not an instruction changed).
  f32x4_t mreg[D / 16];
  if (gram) {
    if constexpr (D == 64 && USE_OP == 1) {
      const float* Mh = gram + ((int64_t)h * D + 16 * wv + (l & 15)) * D + 4 * (l >> 4);
#pragma unroll
      for (int a = 0; a < D / 16; ++a) mreg[a] = quad_of(Mh + 16 * a);
    } else {
      const float* Mh = gram + ((int64_t)h * D + 4 * (l >> 4)) * D + 16 * wv + (l & 15);
#pragma unroll
      for (int a = 0; a < D / 16; ++a)
#pragma unroll
        for (int e = 0; e < 4; ++e) mreg[a][e] = Mh[(16 * a + e) * D];
    }
  }
  for (int r = tid / SW; r < RQ; r += NT / SW) {
    const int row = h * pb.W + min(i0 + r, pb.W - 1);
    if (r >= NT / SW) fetch_scalars(r);
    if (sub >= S) { pm = -INFINITY; pn = -1; }
    const float M0 = group_max(pm, SW);
    // split whose kept-out key is the overall maximum: the earliest one (= lowest key)
    const unsigned long long cand = __ballot(pn >= 0 && pmx == M0) & mine;
    const int sl = cand ? __builtin_ctzll(cand) : -1;      // its lane
    // a split adds to the merged sums if it saw a key and its own sums are not empty; its
    // kept-out key joins them unless it is the overall maximum
    const bool has = pm != -INFINITY && pl > 0.f;
    const bool joins = pm != -INFINITY && pn >= 0 && l != sl;
    // The merged sums are relative to R, the largest logit that is part of them (reference of a
    // split, logit of a joining key), NOT to the overall maximum M0: a kept-out key may be any
    // distance above the rest without the rest's sums underflowing.
    float R = has ? pref : -INFINITY;
    if (joins) R = fmaxf(R, pmx);
    R = group_max(R, SW);
    const float w = has ? exp2f(pref - R) : 0.f;
    const float wj = joins ? exp2f(pmx - R) : 0.f;
    const float lrest = group_sum((has ? w * pl : 0.f) + wj, SW);    // (an empty split's sums may hold anything)
    const unsigned long long jm = __ballot(wj != 0.f) & mine;
    if (wj != 0.f) {
      const int e = __popcll(jm & ((1ull << l) - 1ull));
      s_jw[r][e] = wj;
      s_jn[r][e] = pn;
    }
    s_w[r][sub] = w;
    // without one: the earliest split whose largest logit, part of its sums, is the overall maximum
    const unsigned long long cin = __ballot(pn <= -2 && pm == M0) & mine;
    const int sc = cand ? sl : (cin ? __builtin_ctzll(cin) : -1);
    const int nst = __shfl(pn, sc < 0 ? l : sc, 64);
    if (sub == 0) {
      s_fr[r] = R == -INFINITY ? 0.f : exp2f(R - M0);
      s_lrest[r] = lrest;
      s_nj[r] = __popcll(jm);
      s_nstar[r] = sc >= 0 ? nst : -1;       // as part_n
      if (i0 + r < pb.W) *(USE_OP == 1 ? o.rs_m + row : stat(i0 + r, 0, 0)) = M0;
    }
  }
  __syncthreads();
  // the key that the score pass is to evaluate in its leave-one-out form
  auto key_of = [](int n) { return n >= 0 ? n : (n <= -2 ? -2 - n : -1); };
  auto loo = [&](int r) { return pb.ind == 0 ? key_of(s_nstar[r]) : -1; };
  // rows that have one (a bit each), and the slot of a row's x among them
  unsigned long long cm = __ballot(loo(l & (RQ - 1)) >= 0);
  if constexpr (RQ < 64) cm &= (1ull << RQ) - 1ull;
  const bool champ = cm != 0ull;
  auto slot_of = [&](int r) { return RQ <= 8 ? r : __popcll(cm & ((1ull << r) - 1ull)); };
#pragma unroll
  for (int m = 0; m < MB; ++m) {
    const int r = rz + 16 * m;
    // value rows of the kept-out keys: the overall maximum's, and those that join, the first JB of them
    // (kept as they are stored until they are used)
    const int nj = s_nj[r], nstar = s_nstar[r];
    T tj[JB][4];
    auto fetch_joins = [&](int j) {
#pragma unroll
      for (int k = 0; k < JB; ++k)
        __builtin_memcpy(&tj[k][0], vg + (int64_t)s_jn[r][min(j + k * NP, nj - 1)] * pb.kv_st + c4, 4 * sizeof(T));
    };
    const f32x4_t vs = quad_of(vg + (int64_t)max(key_of(nstar), 0) * pb.kv_st + c4);
    if (part < nj) fetch_joins(part);
    f32x4_t z = {0.f, 0.f, 0.f, 0.f};
    for (int s = part; s < S; s += SB * NP) {
      if (s != part) fetch_splits(m, s);
#pragma unroll
      for (int k = 0; k < SB; ++k) {
        const float wk = s + k * NP < S ? s_w[r][s + k * NP] : 0.f;
#pragma unroll
        for (int e = 0; e < 4; ++e) z[e] = fmaf(wk, wk != 0.f ? t[m][k][e] : 0.f, z[e]);
      }
    }
    for (int j = part; j < nj; j += JB * NP) {
      if (j != part) fetch_joins(j);
#pragma unroll
      for (int k = 0; k < JB; ++k) {
        const float wk = j + k * NP < nj ? s_jw[r][j + k * NP] : 0.f;
        const f32x4_t x = quad_of(&tj[k][0]);
#pragma unroll
        for (int e = 0; e < 4; ++e) z[e] = fmaf(wk, x[e], z[e]);
      }
    }
    if constexpr (NP > 1) {
      *(f32x4_t*)&xs[part * RQ + r][c4] = z;
      __syncthreads();
    }
    if (part == 0) {
#pragma unroll
      for (int k = 1; k < NP; ++k) z += *(const f32x4_t*)&xs[k * RQ + r][c4];
      // rest -> units of the overall maximum (0 when the rest is below FP32 range next to the kept-out key)
      const float fr = s_fr[r], lrest = s_lrest[r];
      f32x4_t zz, x = {0.f, 0.f, 0.f, 0.f};
      if (nstar >= 0) {
        const float l_ = 1.f + lrest * fr;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          zz[e] = (vs[e] + z[e] * fr) / l_;
          x[e] = lrest > 0.f ? z[e] / lrest - vs[e] : 0.f;     // z_without_champion - v_champion
        }
      } else {
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          zz[e] = z[e] / lrest;
          x[e] = nstar <= -2 ? zz[e] - vs[e] : 0.f;
        }
      }
      *(f32x4_t*)&zs[r][c4] = zz;
      if (RQ <= 8 || ((cm >> r) & 1ull)) *(f32x4_t*)&xs[slot_of(r)][c4] = x;      // (its own partial sum, or nothing, was there)
    }
  }
  __syncthreads();
  // u and y: register j of a lane is row 4 (l / 16) + j of a 16-row block, column 16 wv + l % 16.  With at
  // most eight rows z takes the first half of one block and x the second; with more, the x of the rows
  // that have one follow in blocks of their own.
  const int c = 16 * wv + (l & 15), kq = l >> 4;
  // acc[m]: product of block m, whose row i lies in LDS at row_of(m, i)
  auto product = [&](auto row_of, auto& acc) {
    constexpr int NB = sizeof(acc) / sizeof(f32x4_t);
#pragma unroll
    for (int m = 0; m < NB; ++m) acc[m] = f32x4_t{0.f, 0.f, 0.f, 0.f};
    // (attention-weight and value-norm indicators: no output term (u = 0, zz = 0), no key is evaluated by the
    // leave-one-out form; the score pass then sees sqrt(vv) with vv = 1 or ||v||^2)
    if (pb.ind != 0) return;
    if (gram) {
#pragma unroll
      for (int a = 0; a < D / 16; ++a) {
        f32x4_t xa[NB];
#pragma unroll
        for (int m = 0; m < NB; ++m) xa[m] = *(const f32x4_t*)&row_of(m, l & 15)[16 * a + 4 * kq];
#pragma unroll
        for (int e = 0; e < 4; ++e)
#pragma unroll
          for (int m = 0; m < NB; ++m) acc[m] = __builtin_amdgcn_mfma_f32_16x16x4f32(xa[m][e], mreg[a][e], acc[m], 0, 0, 0);
      }
      // wait states between the last MFMA and the first read of its result, spelled out because a
      // branch lies in between (the compiler inserts too few on one of the merging paths)
#pragma unroll
      for (int m = 0; m < NB; ++m) asm volatile("s_nop 15" : "+v"(acc[m]));
    } else {
#pragma unroll
      for (int m = 0; m < NB; ++m)
#pragma unroll
        for (int j = 0; j < 4; ++j) acc[m][j] = row_of(m, 4 * kq + j)[c];
    }
  };
  // zz = u.z and |x|_M^2 = y.x: sums over 16 lanes here, across the wavefronts below
  f32x4_t u[MB];
  if constexpr (RQ <= 8) {
    auto row_of = [&](int, int i) -> const float* { return i < 8 ? zs[i & (RQ - 1)] : xs[i & (RQ - 1)]; };
    product(row_of, u);
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const int i = 4 * kq + j;
      const float s0 = row16_sum(u[0][j] * row_of(0, i)[c]);
      if ((i & 7) < RQ && (l & 15) == 0) red[wv][i & 7][i >> 3] = s0;
    }
  } else {
    product([&](int m, int i) -> const float* { return zs[16 * m + i]; }, u);
#pragma unroll
    for (int m = 0; m < MB; ++m)
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const float s0 = row16_sum(u[m][j] * zs[16 * m + 4 * kq + j][c]);
        if ((l & 15) == 0) red[wv][16 * m + 4 * kq + j][0] = s0;
      }
    const int nx = __popcll(cm);
    for (int m0 = 0; m0 < nx; m0 += 16) {        // (rows past the last are whatever LDS holds, and are not used)
      auto row_of = [&](int, int i) -> const float* { return xs[m0 + i]; };
      f32x4_t y[1];
      product(row_of, y);
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const float s1 = row16_sum(y[0][j] * row_of(0, 4 * kq + j)[c]);
        if ((l & 15) == 0) red[wv][m0 + 4 * kq + j][1] = s1;
      }
    }
  }
  // u takes the place of the x that have been read, or of partial sums that nobody reads any more
  constexpr int UB = RQ <= 8 ? RQ : 0;
  if (RQ > 8 && champ) __syncthreads();
#pragma unroll
  for (int m = 0; m < MB; ++m)
#pragma unroll
    for (int j = 0; j < 4; ++j)
      if (16 * m + 4 * kq + j < RQ) xs[UB + 16 * m + 4 * kq + j][c] = u[m][j];
  __syncthreads();
  for (int r = tid; r < RQ; r += NT) {
    if (i0 + r >= pb.W) break;
    const int row = h * pb.W + i0 + r;
    const bool has_x = (cm >> r) & 1ull;
    const int sl = has_x ? slot_of(r) : 0;
    float zz = 0.f, qx = 0.f;
#pragma unroll
    for (int k = 0; k < NWV; ++k) { zz += red[k][r][0]; qx += has_x ? red[k][sl][1] : 0.f; }
    const float lr = s_lrest[r] * s_fr[r], l_ = s_nstar[r] >= 0 ? 1.f + lr : lr;
    // A* ||(z_rest - v*) W_O|| with A* = 1/l, or A*/(1 - A*) ||(z - v*) W_O|| with A*/(1 - A*) = 1/(l - 1)
    const float is = sqrtf(fmaxf(qx, 0.f)) / (s_nstar[r] >= 0 ? l_ : l_ - 1.f);
    if constexpr (USE_OP == 1) {
      o.rs_l[row] = l_;
      o.rs_zz[row] = zz;
      o.rs_nstar[row] = loo(r);
      o.rs_istar[row] = is;
    } else {
      *stat(i0 + r, 0, 1) = l_;
      *stat(i0 + r, 1, 0) = zz;
      *stat(i0 + r, 1, 1) = __int_as_float(loo(r));
      *stat(i0 + r, 1, 2) = is;
    }
  }
  if constexpr (USE_OP == 1) {
    // q, and u split into bf16 high and low parts, in the order the score pass feeds them to the
    // matrix cores: [which][32-row block][d/16][lane half][local row][8], local row =
    // position * Gp + head, so that a wavefront fetches each operand register as one 1 KiB run
    const int head = h - g * pb.G, log2iw = 5 - log2gp;
    const int64_t plane = (int64_t)pb.Hkv * nwb * (D / 16) * 2 * 32 * 8;
    for (int x = tid; x < RQ * (D / 8); x += NT) {
      const int r = x / (D / 8), c8 = x % (D / 8), i = i0 + r;
      if (i >= pb.W) continue;
      const int wb = i >> log2iw, m_ = ((i & ((1 << log2iw) - 1)) << log2gp) + head;
      const int64_t at = ((((int64_t)(g * nwb + wb) * (D / 16) + (c8 >> 1)) * 2 + (c8 & 1)) * 32 + m_) * 8;
      uint32_t hi[4], lo[4];
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        const float ue = xs[UB + r][8 * c8 + e];
        const uint32_t ub = __float_as_uint(ue);
        const uint32_t hb = (ub + 0x7FFFu + ((ub >> 16) & 1u)) & 0xFFFF0000u;      // round to nearest even (u is finite)
        const uint32_t lb = __float_as_uint(ue - __uint_as_float(hb));
        const uint32_t lw = (lb + 0x7FFFu + ((lb >> 16) & 1u)) >> 16;
        hi[e >> 1] = e & 1 ? (hi[e >> 1] | hb) : (hb >> 16);
        lo[e >> 1] = e & 1 ? (lo[e >> 1] | (lw << 16)) : lw;
      }
      *(uint4*)(o.op + at) = *(const uint4*)(q + (int64_t)h * pb.q_sh + (int64_t)i * pb.q_st + 8 * c8);   // (16-byte rows: checked on the host)
      *(uint4*)(o.op + plane + at) = make_uint4(hi[0], hi[1], hi[2], hi[3]);
      *(uint4*)(o.op + 2 * plane + at) = make_uint4(lo[0], lo[1], lo[2], lo[3]);
    }
  } else {
    // planes of q and u (see row_item)
    constexpr int LPR = D / 8;                             // lanes of a row
    for (int x = tid; x < RQ * LPR; x += NT) {
      const int r = x / LPR, c8 = x % LPR, i = i0 + r;
      const bool there = i < pb.W;
      const T* qp = q + (int64_t)h * pb.q_sh + (int64_t)min(i, pb.W - 1) * pb.q_st + 8 * c8;
      const f32x4_t qa = quad_of(qp), qb = quad_of(qp + 4);
      const f32x4_t ua = *(const f32x4_t*)&xs[UB + r][8 * c8], ub = *(const f32x4_t*)&xs[UB + r][8 * c8 + 4];
      auto put = [&](int which, const f32x4_t& va, const f32x4_t& vb, bool small, auto np) {
        constexpr int N = decltype(np)::value;
        const float4 a = make_float4(va[0], va[1], va[2], va[3]), b = make_float4(vb[0], vb[1], vb[2], vb[3]);
        PlaneRange in;
        in.take(a, b);
        // (a bf16 row is its own plane, whatever it holds; the lanes of a row are neighbours)
        const unsigned long long mine = ((1ull << LPR) - 1ull) << (l & ~(LPR - 1));
        const bool raw = N > 1 && (__ballot(in.out() || small) & mine) != 0ull;
        if (!there) return;
        char* const at = item_of(i, which) + c8 * 512 + (i & 31) * 16;
        const Op<N> o8 = split8<N>(a, b);
        if (raw) {
          *(float4*)at = a;
          *(float4*)(at + (D / 16) * 1024) = b;
        } else {
#pragma unroll
          for (int p = 0; p < N; ++p) *(uint4*)(at + p * (D / 16) * 1024) = o8.p[p];
        }
        if (c8 == 0) *stat(i, which, 3) = raw ? 1.f : 0.f;
      };
      put(0, qa, qb, false, std::integral_constant<int, planes_of<T>>{});
      // (a row whose u.v the score pass sets against a zz so much smaller than u that values' low planes count)
      float um = 0.f;
#pragma unroll
      for (int e = 0; e < 4; ++e) um = fmaxf(um, fmaxf(fabsf(ua[e]), fabsf(ub[e])));
      float zz = 0.f;
#pragma unroll
      for (int k = 0; k < NWV; ++k) zz += red[k][r][0];
      put(1, ua, ub, fabsf(zz) < 0x1p-90f * um, std::integral_constant<int, 3>{});
    }
  }
}

// USE_OP: what the score pass takes, 1: operands of the bf16 path, 2: items of the FP32 path.
template <typename T, int D, int RQ, int USE_OP>
inline void launch_combine_rows(const Prob& pb, const T* v, int S, const float* gram, const ScorePtrs& w, const float* part_z,
                                const T* q, int log2gp, int nwb, hipStream_t st) {
  const dim3 gr(pb.Hq * ((pb.W + RQ - 1) / RQ));
  if constexpr (RQ > 4) {                          // (four rows only with several splits)
    if (pb.ext_lse) {
      RK_LAUNCH(ST_COMBINE, st, (k_attn_combine<T, D, RQ, USE_OP, true>), gr, dim3(4 * D), 0, st, pb, v, S, gram, w, part_z, q, log2gp, nwb);
      return;
    }
  }
  RK_LAUNCH(ST_COMBINE, st, (k_attn_combine<T, D, RQ, USE_OP, false>), gr, dim3(4 * D), 0, st, pb, v, S, gram, w, part_z, q, log2gp, nwb);
}
template <typename T, int D, int USE_OP>
inline void launch_combine(const Prob& pb, const T* v, int S, const float* gram, const ScorePtrs& w, const float* part_z,
                           const T* q, int log2gp, int nwb, hipStream_t st) {
  // As many rows per workgroup (one chain of round trips, one read of the Gram matrix) as still leave
  // a workgroup for every compute unit; where eight rows do not, four rows whose splits are shared by
  // four threads (1024 rows: 10.8 us against 14.1 with eight; 2048 rows, score + smoothing, eight against four: 2112
  // tokens 56.2 / 59.8 us, 24k 142.0 / 144.6, 32k 176.0 / 178.7; one split has nothing to share).
  auto fills = [&](int rq) { return S <= combine_max_splits(rq) && pb.W > rq / 2 && (int64_t)pb.Hq * ((pb.W + rq - 1) / rq) >= n_cu(); };
  if (fills(64)) launch_combine_rows<T, D, 64, USE_OP>(pb, v, S, gram, w, part_z, q, log2gp, nwb, st);
  else if (fills(32)) launch_combine_rows<T, D, 32, USE_OP>(pb, v, S, gram, w, part_z, q, log2gp, nwb, st);
  else if (fills(16)) launch_combine_rows<T, D, 16, USE_OP>(pb, v, S, gram, w, part_z, q, log2gp, nwb, st);
  else if (S > 1 && (int64_t)pb.Hq * ((pb.W + 7) / 8) < n_cu()) launch_combine_rows<T, D, 4, USE_OP>(pb, v, S, gram, w, part_z, q, log2gp, nwb, st);
  else launch_combine_rows<T, D, 8, USE_OP>(pb, v, S, gram, w, part_z, q, log2gp, nwb, st);
}

}  // namespace restkv

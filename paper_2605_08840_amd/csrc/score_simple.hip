// Reconstruction indicator in FP32 (float32 inputs, and bf16 inputs whose shape or alignment the
// bf16 path does not take).
//
// The same four stages and scratch layout as the bf16 path.  Every product of FP32 values runs on
// v_mfma_f32_32x32x16_bf16 with both sides cut into planes: x = h + m + l, each a bf16 (h the nearest
// to x, m the nearest to what is left, l the rest: 8 + 8 + 8 bits), and x y as the six products
// h h, h m, m h, m m, h l, l h with FP32 accumulation; what is dropped (m l, l m, l l) is below
// 2^-25 |x y|, less than the rounding of one FP32 addition.  Six bf16 instructions of 32 cycles take
// 16 K indices, eight v_mfma_f32_32x32x2_f32 of 64 cycles take the same: 2.7 times the rate.  A bf16
// input has one plane (it is exact), so its products with FP32 values are three.  Scores are nearer to 64 bits than
// with FP32 products: 0.81 of the distance (2-norm, mean of 70 shapes; with sinks, where a few entries carry the
// norm, 0.79 to 0.90 over 60 seeds of five shapes).
// Planes hold values of ordinary size (PlaneRange).  Where operands are not, each kernel notices at the end of its work, by
// sums that are not finite or by the range of q, u and Gram entries, and does that part again on the FP32 instruction.
// 8k tokens, 32/8 heads of 128, window 32, against kernels of FP32 products: attention pass 52 -> 39 us, value-Gram pass
// 54 -> 35, score pass 58 -> 42; score and smoothing 177 -> 132 us.  What bounds them now: per 32 keys a wavefront has 96 to 120 MFMAs
// (3.1k to 3.8k cycles) and 200 to 350 vector instructions that cut values into planes, and both wavefronts of a
// SIMD are in the same phase most of the time.
//
//   C layout of a 32x32 block:  register j of lane l holds
//       M index = 8*(j/4) + 4*(l/32) + (j%4),   N index = l % 32;
//   A / B operands: lane l holds M (or N) index l % 32 and 8 K indices, chosen by l / 32.
//
// Which 16 K indices a step multiplies in which order is free as long as A and B agree.  The
// contraction over the keys (P.V) and the one with the Gram matrix take the K indices that the
// registers of a C block hold in the two lane halves, so that attention weights are operands as they
// stand, and the value entries a lane holds as operands are the ones its row dots need.
#include <algorithm>
#include <type_traits>

#include "score_common.hpp"

namespace restkv {

namespace {

typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef short s16x4 __attribute__((ext_vector_type(4)));
typedef short s16x8 __attribute__((ext_vector_type(8)));

constexpr int KB = 32;      // keys per block (one side of an MFMA)
constexpr float LOG2E = 1.4426950408889634f;
constexpr float RESCALE_TH = 8.0f;  // log2 units a joining logit may run ahead of the reference

// the FP32 instruction, for what planes do not hold (PlaneRange): a lane has ONE K index, chosen by its half
#define MFMA32(a, b, c) __builtin_amdgcn_mfma_f32_32x32x2f32((a), (b), (c), 0, 0, 0)
__device__ __forceinline__ void mul4(f32x16& acc, float4 a, float4 b) {
  acc = MFMA32(a.x, b.x, acc);
  acc = MFMA32(a.y, b.y, acc);
  acc = MFMA32(a.z, b.z, acc);
  acc = MFMA32(a.w, b.w, acc);
}

// acc + registers 4 jq .. of a block times four values
__device__ __forceinline__ float dot4(const f32x16& y, int jq, float4 x, float acc) {
  return fmaf(y[4 * jq + 3], x.w, fmaf(y[4 * jq + 2], x.z, fmaf(y[4 * jq + 1], x.y, fmaf(y[4 * jq], x.x, acc))));
}

// Wait states between the last MFMA on a block and the first read of its result, spelled out: where
// branches lie in between, hipcc 7.2 inserts too few on some path, and the last registers of the block
// come out stale.
__device__ __forceinline__ void settle(f32x16& x) { asm volatile("s_nop 15\n\ts_nop 3" : "+v"(x)); }

__device__ __forceinline__ float half_max(float x) {   // with the lane 32 away
  const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  return fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1]));
}
__device__ __forceinline__ float half_sum(float x) {
  const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}
__device__ __forceinline__ int half_min(int x) {
  const auto r = __builtin_amdgcn_permlane32_swap((unsigned)x, (unsigned)x, false, false);
  return min((int)r[0], (int)r[1]);
}
__device__ __forceinline__ constexpr int cidx(int j, int hf) { return 8 * (j >> 2) + 4 * hf + (j & 3); }

// four consecutive elements of a row; VEC: the address is a multiple of four elements
template <bool VEC>
__device__ __forceinline__ float4 load4(const float* p) {
  if constexpr (VEC) return *(const float4*)p;
  else return make_float4(p[0], p[1], p[2], p[3]);
}
template <bool VEC>
__device__ __forceinline__ float4 load4(const bf16_t* p) {
  if constexpr (VEC) {
    const uint2 u = *(const uint2*)p;
    return make_float4(__uint_as_float(u.x << 16), __uint_as_float(u.x & 0xFFFF0000u), __uint_as_float(u.y << 16),
                       __uint_as_float(u.y & 0xFFFF0000u));
  } else {
    return make_float4(to_float(p[0]), to_float(p[1]), to_float(p[2]), to_float(p[3]));
  }
}

// acc += a b over the 16 K indices of a step, the small products first
template <int NA, int NB>
__device__ __forceinline__ void mul(f32x16& acc, const Op<NA>& a, const Op<NB>& b) {
#pragma unroll
  for (int s = NA + NB - 2 < 2 ? NA + NB - 2 : 2; s >= 0; --s)
#pragma unroll
    for (int i = 0; i < NA; ++i)
      if (s - i >= 0 && s - i < NB)
        acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(as_bf16x8(a.p[i]), as_bf16x8(b.p[s - i]), acc, 0, 0, 0);
}

// acc(a) += step a of KS whose A side comes from LDS, read(a, p) being plane p of step a: a plane of the
// next step is asked for as soon as the current one is done with (l after one product, m after three).  Left to
// itself the compiler asks for everything first, which spills, or for each operand right before its use, which leaves
// the matrix cores idle half of the time.
template <int NA, int NB, int KS, typename Acc, typename F, typename G>
__device__ __forceinline__ void contract(Acc acc, F read, G other) {
  uint4 x[NA];
#pragma unroll
  for (int p = 0; p < NA; ++p) x[p] = read(0, p);
#pragma unroll
  for (int a = 0; a < KS; ++a) {
    const Op<NB> b = other(a);
#pragma unroll
    for (int p = NA - 1; p >= 0; --p) {
      __builtin_amdgcn_sched_barrier(0);
      uint4 next;
      if (p == 0 && a + 1 < KS) next = read(a + 1, 0);
#pragma unroll
      for (int i = (NB - 1 < 2 - p ? NB - 1 : 2 - p); i >= 0; --i)
        acc(a) = __builtin_amdgcn_mfma_f32_32x32x16_bf16(as_bf16x8(x[p]), as_bf16x8(b.p[i]), acc(a), 0, 0, 0);
      if (p > 0 && a + 1 < KS) next = read(a + 1, p);
      x[p] = next;
    }
  }
  __builtin_amdgcn_sched_barrier(0);
}

// Planes of KB rows of D values in LDS, read as operand columns (32 rows x 8 K indices): chunk c (8 values) of a row
// lies c column strides from the first, which keeps one address per lane for all reads, and the odd stride spreads
// the writes of a row's chunks over the banks.
template <int D, int NP>
struct ColTile {
  static constexpr int CST = KB * 8 + 8, PLANE = D / 8 * CST;      // (in bf16)
  uint16_t x[NP][PLANE];
  __device__ static __forceinline__ int at(int r, int c) { return c * CST + r * 8; }
  // plane p of the operand of step ks: rows rr on one side, K indices 16 ks + 8 hf .. + 7
  __device__ __forceinline__ uint4 cols(int rr, int hf, int ks, int p) const { return *(const uint4*)&x[p][at(rr, hf) + 2 * ks * CST]; }
};
// The same read through the transposing 8-byte read (4 rows x 4 chunks per lane half): a row is D bf16, its groups of
// four chunks permuted by the row.
template <int D, int NP>
struct RowTile {
  static constexpr int CH = D / 8, SH = CH == 16 ? 0 : 1;
  uint16_t x[NP][KB * D];
  __device__ static __forceinline__ int at(int r, int c) { return r * D + ((c ^ (((r >> SH) & (CH / 4 - 1)) << 2)) << 3); }
  // plane p of the operand with the 32 columns 32 cb .. on one side and the rows (keys) 16 grp .. as K indices in the order
  // of the registers of a C block; r0, c0: row and column of this lane's 8 bytes inside a 16 x 32 piece
  __device__ __forceinline__ uint4 rows(int grp, int cb, int r0, int c0, int p) const {
    const int c = 32 * cb + c0;
    const uint16_t* b = &x[p][at(r0, c >> 3) + (c & 7) + 16 * grp * D];           // rows r, r + 8 and r + 16 share their permutation
    const s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) s16x4*)(b));
    const s16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) s16x4*)(b + 8 * D));
    union { s16x8 s; uint4 u; } a;
    a.s = __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
    return a.u;
  }
};

// A block of KB rows of D values on its way from global memory to a tile through NT threads' registers.
template <int D, int NT>
struct Stage {
  static constexpr int CH = D / 8, N = KB * CH / NT;
  static_assert(KB * CH % NT == 0, "every thread takes the same number of chunks");
  float4 r[N][2];
  // the first of `rows` rows (the others become zeros) at base (wave-uniform), `stride` elements apart
  template <bool VEC, typename T>
  __device__ __forceinline__ void fetch(const T* base, int64_t stride, int rows) {
    const int row = (int)threadIdx.x / CH, c = (int)threadIdx.x % CH;
    const int64_t lane = row * stride + 8 * c;
#pragma unroll
    for (int j = 0; j < N; ++j) {
      const T* p = base + (int64_t)(j * (NT / CH)) * stride + lane;
      if (rows < KB && row + j * (NT / CH) >= rows) p = base;
      r[j][0] = load4<VEC>(p);
      r[j][1] = load4<VEC>(p + 4);
    }
    if (rows < KB)                                     // (uniform)
#pragma unroll
      for (int j = 0; j < N; ++j)
        if (row + j * (NT / CH) >= rows) r[j][0] = r[j][1] = make_float4(0.f, 0.f, 0.f, 0.f);
  }
  template <typename Tile>
  __device__ __forceinline__ void store(Tile& t) const {
    constexpr int NP = sizeof(t.x) / sizeof(t.x[0]);
#pragma unroll
    for (int j = 0; j < N; ++j) {
      const int x = (int)threadIdx.x + j * NT, row = x / CH, c = x % CH;
      const Op<NP> o = split8<NP>(r[j][0], r[j][1]);
      const int at = t.at(row, c);
#pragma unroll
      for (int p = 0; p < NP; ++p) *(uint4*)&t.x[p][at] = o.p[p];
    }
  }
};

// Attention pass: per key split, online softmax of every window query with its dominant key kept
// out of the sums (outputs described in score_common.hpp).  A wavefront owns 32 query rows, on the
// N side: a lane is half of a row, its softmax state is scalar.  The planes of a K and a V block of 32
// keys are in LDS (48 KiB for D = 128, two workgroups per compute unit); the next block's loads are in
// flight while a block is worked on, its K planes are written when the logits have been formed, its V
// planes when the values have been added up: two barriers per block of 96 MFMAs per wavefront.
// Workgroups: S splits x ceil(R / (32 NW)) row blocks x KV heads, 64 NW threads.
template <int D, int NP, int NW>
struct AttnSmem {
  __attribute__((aligned(16))) ColTile<D, NP> Ks;
  __attribute__((aligned(16))) RowTile<D, NP> Vs;
  int beyond[NW];                       // a wavefront has found that planes do not hold a value of this split or of its rows
};
template <typename T, int D, int NW, bool VEC>
__device__ __forceinline__ void attn_pass(const Prob& pb, int s, int yb, int g, AttnSmem<D, planes_of<T>, NW>& sm, const T* __restrict__ q,
                                          const T* __restrict__ k, const T* __restrict__ v, int S, int kps, const ScorePtrs& o) {
  constexpr int CB = D / 32, NP = planes_of<T>;
  auto& Ks = sm.Ks;
  auto& Vs = sm.Vs;
  auto& beyond = sm.beyond;
  const int l = threadIdx.x & 63, wv = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6)), rr = l & 31, hf = l >> 5;
  const int r = (yb * NW + wv) * 32 + rr;               // row inside the KV head
  const bool valid = r < pb.R;
  const int hl = valid ? r / pb.W : 0, i = valid ? r % pb.W : 0;
  const int vis_last = (pb.causal && valid) ? pb.P + i : pb.L - 1;
  const T* kg = k + (int64_t)g * pb.kv_sh;
  const T* vg = v + (int64_t)g * pb.kv_sh;
  const int kbeg = s * kps, kend = min(pb.L, kbeg + kps);
  const int nblk = kend > kbeg ? (kend - kbeg + KB - 1) / KB : 0;

  bool out;
  Op<NP> qf[D / 16];
  {
    PlaneRange in;
    const T* qp = q + (int64_t)(g * pb.G + hl) * pb.q_sh + (int64_t)i * pb.q_st + 8 * hf;
#pragma unroll
    for (int a = 0; a < D / 16; ++a) {
      const float4 x = load4<VEC>(qp + 16 * a), y = load4<VEC>(qp + 16 * a + 4);
      qf[a] = split8<NP>(x, y);
      in.take(x, y);
    }
    out = __ballot(in.out()) != 0ull;
  }
  // row and column of the 8 bytes that this lane contributes to a transposing read
  const int s16 = l & 15, vrow = 4 * hf + (s16 >> 2), vcol = 16 * ((l >> 4) & 1) + 4 * (s16 & 3);
  const float c2 = pb.scale * LOG2E;
  float mall, mref, mx, lsum;
  int nx;                            // key kept out of the sums, -1: none
  int ni;                            // key of the largest logit (the one kept out, if any)
  f32x16 oacc[CB];

  // moves the reference onto a logit that runs far ahead of it (also if there is none yet: 2^-inf = 0)
  auto rescale = [&](float to) {
    const bool mv = (to - mref) * c2 > RESCALE_TH;
    const float f = mv ? __builtin_amdgcn_exp2f((mref - to) * c2) : 1.f;
    lsum *= f;
#pragma unroll
    for (int cb = 0; cb < CB; ++cb)
#pragma unroll
      for (int j = 0; j < 16; ++j) oacc[cb][j] *= f;
    mref = mv ? to : mref;
  };
  Stage<D, NW * 64> sg;                // K rows, then V rows of the next block on their way to LDS
  auto fetch = [&](const T* base, int t) {
    const int k0 = kbeg + t * KB;
    sg.template fetch<VEC>(base + (int64_t)k0 * pb.kv_st, pb.kv_st, kend - k0);
  };
  // the split in planes, or (raw) every product on the FP32 instruction with operands straight from memory
  auto walk = [&](auto raw) {
    constexpr bool RAW = decltype(raw)::value;
    mall = mref = mx = -INFINITY;
    lsum = 0.f;
    nx = -1;
    ni = 0;
#pragma unroll
    for (int cb = 0; cb < CB; ++cb)
#pragma unroll
      for (int j = 0; j < 16; ++j) oacc[cb][j] = 0.f;
    if (!RAW && nblk > 0) {
      fetch(kg, 0);
      const Stage<D, NW * 64> sk = sg;
      fetch(vg, 0);
      sk.store(Ks);
      sg.store(Vs);
      __syncthreads();
    }
    for (int t = 0; t < nblk; ++t) {
      const int k0 = kbeg + t * KB;
      f32x16 sacc;
#pragma unroll
      for (int j = 0; j < 16; ++j) sacc[j] = 0.f;
      if constexpr (RAW) {
        int r2 = r;
        asm volatile("" : "+v"(r2));     // (formed here, not kept in registers through the walk in planes)
        const T* qr = q + (int64_t)(g * pb.G + (valid ? r2 / pb.W : 0)) * pb.q_sh + (int64_t)(valid ? r2 % pb.W : 0) * pb.q_st;
        const T* kr = kg + (int64_t)min(k0 + rr, kend - 1) * pb.kv_st + 4 * hf;
#pragma unroll 4
        for (int a = 0; a < D; a += 8) mul4(sacc, load4<VEC>(kr + a), load4<VEC>(qr + 4 * hf + a));
      } else {
        if (t + 1 < nblk) fetch(kg, t + 1);
        contract<NP, NP, D / 16>([&](int) -> f32x16& { return sacc; }, [&](int a, int p) { return Ks.cols(rr, hf, a, p); }, [&](int a) { return qf[a]; });
        __syncthreads();                 // the K planes have been read, the V planes of this block are complete
        if (t + 1 < nblk) {
          sg.store(Ks);
          fetch(vg, t + 1);
        }
      }
      settle(sacc);
      if (k0 + KB > kend || (pb.causal && k0 + KB - 1 > pb.P)) {
#pragma unroll
        for (int j = 0; j < 16; ++j) {
          const int n = k0 + cidx(j, hf);
          if (n >= kend || n > vis_last) sacc[j] = -INFINITY;
        }
      }
      float tm = sacc[0];
#pragma unroll
      for (int j = 1; j < 16; ++j) tm = fmaxf(tm, sacc[j]);
      tm = half_max(tm);
      // The reference of the exponentials is a logit that is part of the sums; it moves when a
      // joining logit runs RESCALE_TH ahead of it.  A key is kept out when it is the largest so far
      // and holds more than half of the mass including its own block's (what a key that ends with
      // more than half of the total always does), and only as long as it is the largest.
      const bool newmax = tm > mall;
      mall = fmaxf(mall, tm);
      float tinc = tm;                   // largest logit of the block that joins the sums
      if (__ballot(newmax) != 0ull) {
        int cand = 0x7FFFFFFF;
#pragma unroll
        for (int j = 0; j < 16; ++j)
          if (sacc[j] == tm) cand = min(cand, k0 + cidx(j, hf));
        cand = half_min(cand);
        ni = newmax ? cand : ni;
        // (this lane's share of the sum alone outweighs most candidates)
        bool dominant = newmax && tm > -INFINITY && lsum < 1.0002f * __builtin_amdgcn_exp2f((tm - mref) * c2);
        if (__ballot(dominant) != 0ull) {
          // mass without the candidate, relative to the candidate itself
          float rest = lsum * __builtin_amdgcn_exp2f((mref - tm) * c2);    // (empty sums: 0 * 0)
#pragma unroll
          for (int j = 0; j < 16; ++j) rest += __builtin_amdgcn_exp2f((sacc[j] - tm) * c2);
          rest = half_sum(rest) - 1.f;
          if (nx >= 0) rest += __builtin_amdgcn_exp2f((mx - tm) * c2);
          // (rest carries the rounding of the sum it was taken from: a tie may go either way)
          dominant = dominant && rest < 1.0001f;
        }
        const bool joins = newmax && nx >= 0;          // the key kept out so far is not the largest any more: it joins the sums
        if (__ballot(dominant || joins) != 0ull) {
          const int cz = dominant ? cand : -1;
          tinc = -INFINITY;
#pragma unroll
          for (int j = 0; j < 16; ++j) {
            sacc[j] = k0 + cidx(j, hf) == cz ? -INFINITY : sacc[j];
            tinc = fmaxf(tinc, sacc[j]);
          }
          tinc = half_max(tinc);
          if (joins) tinc = fmaxf(tinc, mx);
          rescale(tinc);
          if (joins) {
            const float w = __builtin_amdgcn_exp2f((mx - mref) * c2);
            if (hf == 0) lsum += w;
            const T* vr = vg + (int64_t)nx * pb.kv_st + 4 * hf;
#pragma unroll
            for (int cb = 0; cb < CB; ++cb)
#pragma unroll
              for (int jq = 0; jq < 4; ++jq) {
                const float4 x = load4<VEC>(vr + 32 * cb + 8 * jq);
                oacc[cb][4 * jq + 0] = fmaf(w, x.x, oacc[cb][4 * jq + 0]);
                oacc[cb][4 * jq + 1] = fmaf(w, x.y, oacc[cb][4 * jq + 1]);
                oacc[cb][4 * jq + 2] = fmaf(w, x.z, oacc[cb][4 * jq + 2]);
                oacc[cb][4 * jq + 3] = fmaf(w, x.w, oacc[cb][4 * jq + 3]);
              }
          }
          if (dominant || joins) {
            mx = tm;
            nx = dominant ? cand : -1;
          }
        }
      }
      if (__ballot((tinc - mref) * c2 > RESCALE_TH) != 0ull) rescale(tinc);
      // weights relative to the reference (a row that has none yet has nothing to add).  The instruction
      // makes 0 of weights below 2^-126: the sums hold the reference's own weight, 1, and do not notice.
      const float nm = mref == -INFINITY ? 0.f : -mref * c2;
#pragma unroll
      for (int j = 0; j < 16; ++j) sacc[j] = __builtin_amdgcn_exp2f(fmaf(sacc[j], c2, nm));
      lsum += ((sacc[0] + sacc[1]) + (sacc[2] + sacc[3])) + ((sacc[4] + sacc[5]) + (sacc[6] + sacc[7])) +
              (((sacc[8] + sacc[9]) + (sacc[10] + sacc[11])) + ((sacc[12] + sacc[13]) + (sacc[14] + sacc[15])));
      if constexpr (RAW) {
#pragma unroll
        for (int j = 0; j < 16; ++j) {
          const int n = k0 + cidx(j, hf);
          const T* vr = vg + (int64_t)min(n, kend - 1) * pb.kv_st + rr;
#pragma unroll
          for (int cb = 0; cb < CB; ++cb) {
            const float x = to_float(vr[32 * cb]);
            oacc[cb] = MFMA32(n < kend ? x : 0.f, sacc[j], oacc[cb]);
          }
          __builtin_amdgcn_sched_barrier(0);
        }
#pragma unroll
        for (int cb = 0; cb < CB; ++cb) settle(oacc[cb]);
      } else {
#pragma unroll
        for (int grp = 0; grp < 2; ++grp) {
          float pe[8];
#pragma unroll
          for (int e = 0; e < 8; ++e) pe[e] = sacc[8 * grp + e];
          const Op<3> pv = split8<3>(pe);
          contract<NP, 3, CB>([&](int cb) -> f32x16& { return oacc[cb]; }, [&](int cb, int p) { return Vs.rows(grp, cb, vrow, vcol, p); },
                              [&](int) { return pv; });
        }
        if (t + 1 < nblk) {
          __syncthreads();               // the V planes have been read, the K planes of the next block are complete
          sg.store(Vs);
        }
      }
    }
#pragma unroll
    for (int cb = 0; cb < CB; ++cb) settle(oacc[cb]);
  };
  walk(std::false_type{});
  if (nblk > 0) {
    // With queries in the planes' range, a key or value beyond it has made a sum NaN or infinite (a key whose logits are all
    // -inf: no largest logit where there is a visible key), and values that are all so small that their low planes are
    // lost (2^-133 each) have made sums below 2^-90 of the weights'.
    float big = 0.f, t = lsum;
#pragma unroll
    for (int cb = 0; cb < CB; ++cb)
#pragma unroll
      for (int j = 0; j < 16; j += 2) {
        big = fmaxf(big, fmaxf(fabsf(oacc[cb][j]), fabsf(oacc[cb][j + 1])));
        t += oacc[cb][j] * oacc[cb][j + 1];
      }
    big = half_max(big);
    out |= __ballot(!(fabsf(t) < INFINITY) || (big != 0.f && big < 0x1p-90f * lsum) ||
                    (valid && mall == -INFINITY && kbeg <= vis_last)) != 0ull;
    beyond[wv] = out;
    __syncthreads();
    int any = 0;
#pragma unroll
    for (int k = 0; k < NW; ++k) any |= beyond[k];
    if (__builtin_expect(__builtin_amdgcn_readfirstlane(any), 0)) walk(std::true_type{});
  }
  const float ltot = half_sum(lsum);
  if (valid) {
    const int64_t po = ((int64_t)g * pb.R + r) * S + s;
    if (hf == 0) {
      o.part_m[po] = mall * c2;
      o.part_mx[po] = mx * c2;
      o.part_n[po] = nx >= 0 ? nx : -2 - ni;
      o.part_ref[po] = mref == -INFINITY ? 0.f : mref * c2;
      o.part_l[po] = ltot;
    }
    float* zp = o.part_z + po * D + 4 * hf;
#pragma unroll
    for (int cb = 0; cb < CB; ++cb)
#pragma unroll
      for (int jq = 0; jq < 4; ++jq)
        *(float4*)(zp + 32 * cb + 8 * jq) =
            make_float4(oacc[cb][4 * jq], oacc[cb][4 * jq + 1], oacc[cb][4 * jq + 2], oacc[cb][4 * jq + 3]);
  }
}

// vv[h, n] = v_n M_h v_n^T = sum_i v_i (T v)_i with the upper triangular T = diag(M) + 2 triu(M, 1)
// (M is symmetric), so that 32x16 pieces below the diagonal are skipped.  The planes of T of the
// workgroup's head stay in LDS in operand order (one 1 KiB run per piece and plane); a wavefront takes
// 32 keys at a time, on the N side.  K indices are taken in the order of a C block's registers: the
// values a lane holds as operands are also the factors of its row dots.  Workgroups: chunks x query heads, 64 NW threads.
template <int D, int NW>
struct VvSmem {
  static constexpr int NB = D / 32 * (D / 32 + 1);     // pieces on or above the diagonal: KS - 2 cb of row block cb
  __attribute__((aligned(16))) uint4 Ts[NB][3][64];
  int beyond[NW];                                      // a wavefront has found that planes do not hold an entry of T
};
template <typename T, int D, int NW, bool VEC>
__device__ __forceinline__ void vv_pass(const Prob& pb, int chunk, int chunks, int h, VvSmem<D, NW>& sm, const T* __restrict__ v,
                                        const float* __restrict__ gram, float* __restrict__ vv, int ldv) {
  constexpr int CB = D / 32, KS = D / 16, NP = planes_of<T>, NB = VvSmem<D, NW>::NB;
  auto& Ts = sm.Ts;
  auto& beyond = sm.beyond;
  const int g = h / pb.G, stride = NW * chunks;
  const int l = threadIdx.x & 63, wv = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6)), rr = l & 31, hf = l >> 5;
  const T* vg = v + (int64_t)g * pb.kv_sh;
  const int nb = (pb.P + KB - 1) / KB;
  float4 vf[KS][2];                                    // dims 16 ks + 4 hf .. + 3 and 16 ks + 8 + 4 hf .. + 3 of key rr
  auto fetch = [&](int b) {
    const T* vr = vg + (int64_t)min(b * KB + rr, pb.P - 1) * pb.kv_st + 4 * hf;
#pragma unroll
    for (int a = 0; a < KS; ++a) {
      vf[a][0] = load4<VEC>(vr + 16 * a);
      vf[a][1] = load4<VEC>(vr + 16 * a + 8);
    }
  };
  int b = chunk * NW + wv;
  if (b < nb) fetch(b);
  PlaneRange seen;                                     // of the Gram entries this thread has cut into planes
  // (all loads first: one round trip)
  constexpr int NPC = (NB + NW - 1) / NW;                   // pieces per wavefront
  const float* Mh = gram + (int64_t)h * D * D;
  f32x4_t m[NPC][2];
#pragma unroll
  for (int j = 0; j < NPC; ++j) {
    int cb = 0, a = min(wv + NW * j, NB - 1);           // piece: row block cb, step 2 cb + a
    while (a >= KS - 2 * cb) { a -= KS - 2 * cb; ++cb; }
    const float* p = Mh + (32 * cb + rr) * D + 16 * (2 * cb + a) + 4 * hf;
    m[j][0] = quad_of(p);
    m[j][1] = quad_of(p + 8);
  }
#pragma unroll
  for (int j = 0; j < NPC; ++j) {
    if (wv + NW * j >= NB) break;
    int cb = 0, a = wv + NW * j;
    while (a >= KS - 2 * cb) { a -= KS - 2 * cb; ++cb; }
    const int i = 32 * cb + rr, j0 = 16 * (2 * cb + a) + 4 * hf;
    float x[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      const int c = j0 + 8 * (e >> 2) + (e & 3);
      const float f = m[j][e >> 2][e & 3];
      x[e] = c > i ? 2.f * f : (c == i ? f : 0.f);
    }
    const Op<3> t = split8<3>(x);
    seen.take(make_float4(x[0], x[1], x[2], x[3]), make_float4(x[4], x[5], x[6], x[7]));
#pragma unroll
    for (int p = 0; p < 3; ++p) Ts[wv + NW * j][p][l] = t.p[p];
  }
  beyond[wv] = __ballot(seen.out()) != 0ull;
  __syncthreads();
  int any = 0;
#pragma unroll
  for (int j = 0; j < NW; ++j) any |= beyond[j];
  bool raw = __builtin_amdgcn_readfirstlane(any);
  for (; b < nb; b += stride) {
    Op<NP> vo[KS];
#pragma unroll
    for (int a = 0; a < KS; ++a) vo[a] = split8<NP>(vf[a][0], vf[a][1]);
    float acc = 0.f;
#pragma unroll
    for (int cb = 0; cb < CB; ++cb) {
      f32x16 y;
#pragma unroll
      for (int j = 0; j < 16; ++j) y[j] = 0.f;
#pragma unroll
      for (int a = 2 * cb; a < KS; ++a) {
        Op<3> t;
#pragma unroll
        for (int p = 0; p < 3; ++p) t.p[p] = Ts[cb * (KS + 1 - cb) + a - 2 * cb][p][l];
        mul(y, t, vo[a]);
      }
      settle(y);
#pragma unroll
      for (int jq = 0; jq < 4; ++jq) acc = dot4(y, jq, vf[2 * cb + (jq >> 1)][jq & 1], acc);
    }
    const int n = b * KB + rr;
    raw |= __ballot(!(fabsf(acc) < INFINITY)) != 0ull;
    acc = half_sum(acc);
    if (b + stride < nb) fetch(b + stride);
    if (hf == 0 && n < pb.P) vv[(int64_t)h * ldv + n] = acc;
  }
  if (__builtin_expect(!raw, 1)) return;
  // This wavefront's blocks once more, on the FP32 instruction with everything from memory: planes do not hold T or a value.  (A
  // value beyond them has made a sum NaN or infinite; with T in their range one too small for them has a square below FP32.)
#pragma unroll 1
  for (int b = chunk * NW + wv; b < nb; b += stride) {
    const int n = b * KB + rr;
    const T* vr = vg + (int64_t)min(n, pb.P - 1) * pb.kv_st + 4 * hf;
    float acc = 0.f;
#pragma unroll 1
    for (int cb = 0; cb < CB; ++cb) {
      const int i = 32 * cb + rr;
      f32x16 y;
#pragma unroll
      for (int j = 0; j < 16; ++j) y[j] = 0.f;
#pragma unroll 1
      for (int k = 32 * cb; k < D; k += 8) {
        const int c = k + 4 * hf;
        const f32x4_t m = quad_of(Mh + i * D + c);
        auto up = [&](int e) { return c + e > i ? 2.f * m[e] : (c + e == i ? m[e] : 0.f); };
        mul4(y, make_float4(up(0), up(1), up(2), up(3)), load4<VEC>(vr + k));
      }
      settle(y);
#pragma unroll
      for (int jq = 0; jq < 4; ++jq) acc = dot4(y, jq, load4<VEC>(vr + 32 * cb + 8 * jq), acc);
    }
    acc = half_sum(acc);
    if (hf == 0 && n < pb.P) vv[(int64_t)h * ldv + n] = acc;
  }
}

// The two passes that need nothing of each other, one launch: the first workgroups are the attention pass's (split fastest,
// then row block, then head), the others the value-Gram pass's (chunk fastest).  Either one is five to forty microseconds of
// workgroups of few blocks, and its start and end hide behind the other's.  Score + smoothing, 32/8 heads of 128, window 32: 8k tokens 131 ->
// 128 us, 1.5k 77.6 -> 72.5; 28/4 heads, 5k 130 -> 115; 4/2 heads, 16k 88 -> 77; heads of 64, 8/8, 12k 75 -> 67; four heads of 64, 1k, whole
// path 41.7 -> 37.0.  (With the value-Gram pass first 4/2 heads, 16k 91.)  Where the launch is not taken (see run): 16/4 heads of 128,
// window 16, 16k 126 us in two launches, 137 in one; 8/8 heads, window 32, 8k 75.7 and 77.4, 16k 116 and 118; 28/4, window 8, 8k 133 and 131, 16k 190 and 195.
//
// ATTN, VV: whether that pass is there; alone it has a grid of its own dimensions, (S, gy, Hkv) or (chunks, Hq).  64 NW threads.
struct AttnArgs { int S, gy, kps; };
struct VvArgs { int at, chunks, ldv; };               // workgroups from `at` on
template <typename T, int D, int NW, bool VEC, bool ATTN, bool VV>
__global__ __launch_bounds__(NW * 64, NW == 2 ? 1 : 2) void k_attn_vv_f32(Prob pb, const T* __restrict__ q, const T* __restrict__ k,
                                                                          const T* __restrict__ v, const float* __restrict__ gram,
                                                                          ScorePtrs o, AttnArgs aa, VvArgs va) {
  __shared__ union { AttnSmem<ATTN ? D : 32, planes_of<T>, NW> a; VvSmem<VV ? D : 32, NW> v; } sm;
  if constexpr (!VV) {
    attn_pass<T, D, NW, VEC>(pb, blockIdx.x, blockIdx.y, blockIdx.z, sm.a, q, k, v, aa.S, aa.kps, o);
  } else if constexpr (!ATTN) {
    vv_pass<T, D, NW, VEC>(pb, blockIdx.x, va.chunks, blockIdx.y, sm.v, v, gram, o.vv, va.ldv);
  } else {
    const int id = blockIdx.x;
    if (id < va.at) {
      const int y = id / aa.S;
      attn_pass<T, D, NW, VEC>(pb, id - y * aa.S, y % aa.gy, y / aa.gy, sm.a, q, k, v, aa.S, aa.kps, o);
    } else {
      const int x = id - va.at, h = x / va.chunks;
      vv_pass<T, D, NW, VEC>(pb, x - h * va.chunks, va.chunks, h, sm.v, v, gram, o.vv, va.ldv);
    }
  }
}

// vv without a projection: squared norm of the value row (1 for the attention-weight indicator,
// which has no value term).  grid (ceil(P/256), Hkv), 256 threads
template <typename T, int D>
__global__ __launch_bounds__(256) void k_vnorm2_f32(Prob pb, const T* __restrict__ v, float* __restrict__ vv, int ldv) {
  const int g = blockIdx.y, n = blockIdx.x * 256 + threadIdx.x;
  if (n >= pb.P) return;
  const T* vr = v + (int64_t)g * pb.kv_sh + (int64_t)n * pb.kv_st;
  float acc[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll 8
  for (int c = 0; c < D; c += 4)
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const float x = to_float(vr[c + e]);
      acc[e] = fmaf(x, x, acc[e]);
    }
  const float sum = pb.ind == 1 ? 1.f : (acc[0] + acc[1]) + (acc[2] + acc[3]);
  for (int hl = 0; hl < pb.G; ++hl) vv[(int64_t)(g * pb.G + hl) * ldv + n] = sum;
}

// a / b as the operator gives it but for one quotient in a million, which comes out one unit in the last place off: the
// approximation's residual is one rounding from exact, and is added once.  Five instructions for the operator's eleven
// (with those and the library's square root score + smoothing takes 2 to 12 % longer: 28/4 heads of 64, 5k, 85.0 us with the
// bare approximations, 87.7 with these, 95.6).
__device__ __forceinline__ float quotient(float a, float b) {
  const float r = __builtin_amdgcn_rcpf(b), q = a * r;
  return __builtin_amdgcn_div_fixupf(fmaf(fmaf(-b, q, a), r, q), b, a);
}
// Square roots in the same way; the library's where a residual may be subnormal, or for an infinity.
__device__ __forceinline__ void roots(float (&x)[4]) {
  const float low = fminf(fminf(x[0], x[1]), fminf(x[2], x[3])), high = fmaxf(fmaxf(x[0], x[1]), fmaxf(x[2], x[3]));
  if (__ballot(low < 1e-25f || high > 1e38f) != 0ull) {
#pragma unroll
    for (int e = 0; e < 4; ++e) x[e] = sqrtf(x[e]);
  } else {
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const float y = __builtin_amdgcn_rsqf(x[e]), s = x[e] * y;
      x[e] = fmaf(fmaf(-s, s, x[e]), 0.5f * y, s);
    }
  }
}

// Score pass: logits again, cross term u.v_n, closed form, mean (or maximum) over the group.  A
// wavefront owns 32 keys (N side: a store writes 32 consecutive keys of a row) and 32 window positions
// (M side), and walks the heads of the group HC at a time: first the logits of HC heads with the planes
// of its K rows in registers, then the cross terms with the planes of its V rows in the same registers
// (both at once are 192 registers, and two wavefronts per SIMD have 256 each).  The planes of a head's
// q and u rows pass through double-buffered LDS, shared by the workgroup's wavefronts, the next rows' loads in
// flight while a head is worked on.  grid (ceil(P / (32 NW)), ceil(W / 32), Hkv), 64 NW threads.
//
// HS: the wavefronts of a workgroup share 32 keys and divide the heads of the group; each has the planes of the K and V rows in
// registers and an LDS buffer of its own for its heads' rows, and their sums meet in LDS at the end.  One wavefront per 32 keys
// that walks all heads is a serial chain: per head 96 products on one accumulator and 600 vector instructions, at one
// instruction per six cycles for a wavefront that has a SIMD to itself.  Score + smoothing, one wavefront walking the heads and HS:
// 32/8 heads of 128, window 32, 1k tokens 60.3 -> 48.2 us; 28/4, 2k 90.7 -> 66.5; 64/8, 1k 98.1 -> 70.4; 4/2, 4k 51.0 -> 46.7; 4/1 heads
// of 128, 2k, whole path 56.0 -> 44.5; 4/2 heads of 64, 1k, whole path 35.8 -> 34.5.  grid (ceil(P / 32), ceil(W / 32), Hkv).
template <typename T, int D, int NW, bool VEC, bool HS>
__global__ __launch_bounds__(NW * 64, NW == 1 || HS ? 1 : 2) void k_score_f32(Prob pb, const T* __restrict__ q, const T* __restrict__ k,
                                                          const T* __restrict__ v, ScorePtrs o, int ldv,
                                                          float* __restrict__ score) {
  constexpr int KS = D / 16, NP = planes_of<T>, HC = 2;
  constexpr int PL = 3 * KS * 1024;          // planes of an item
  __shared__ __attribute__((aligned(1024))) char rows[HS ? NW : 2][row_item(D) + (HS ? 1024 : 0)];
  const int g = blockIdx.z, i0 = blockIdx.y * 32;
  const int l = threadIdx.x & 63, wv = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6)), rr = l & 31, hf = l >> 5;
  const int n = (HS ? blockIdx.x : blockIdx.x * NW + wv) * KB + rr, nc = min(n, pb.P - 1);
  const T* kr = k + (int64_t)g * pb.kv_sh + (int64_t)nc * pb.kv_st + 8 * hf;
  const T* vr = v + (int64_t)g * pb.kv_sh + (int64_t)nc * pb.kv_st + 8 * hf;
  const float c2 = pb.scale * LOG2E;
  // The attention-weight and value-norm indicators come out of the same expression without the
  // 1 - A (their u, zz and champion are empty, vv is 1 or ||v||^2).
  const float rec = pb.ind == 0 ? 1.f : 0.f;
  // Item (head, which) on its way to LDS: q rows with the statistics of their weights (maximum, denominator), or
  // u rows with zz, the champion's key and its score.
  const char* const items = (const char*)o.op + (int64_t)(g * pb.G * gridDim.y + blockIdx.y) * 2 * row_item(D);
  auto planes = [&](int bf) { return &rows[HS ? wv : bf][0]; };      // (HS: one buffer for the planes, two for the statistics)
  auto stats = [&](int bf) { return planes(bf) + PL + (HS ? bf * 1024 : 0); };
  auto copy_item = [&](int hl, int which, int bf) {
    const int np = which ? 3 : NP;
    const char* src = items + ((int64_t)hl * gridDim.y * 2 + which) * row_item(D);
    // (a row past the window's end becomes a copy of the last one)
    const int row = min(rr, pb.W - 1 - i0);
    for (int x = HS ? 0 : wv; x < np * KS; x += HS ? 1 : NW) dma_1k(src + x * 1024, 16u * (uint32_t)(32 * hf + row), planes(bf) + x * 1024);
    if (HS || wv == NW - 1) dma_1k(src + PL, 16u * (uint32_t)row, stats(bf));
  };
  auto stat = [&](int bf, int j) { return *(const float4*)(stats(bf) + cidx(j, hf) * 16); };
  auto row_op = [&](int bf, int a, int p) { return *(const uint4*)(planes(bf) + (p * KS + a) * 1024 + l * 16); };
  // row rr: in FP32 if it is out of the planes' range; four of its values, those from 8 a + 4 hf on
  auto raw_row = [&](int bf) { return *(const float*)(stats(bf) + rr * 16 + 12) != 0.f; };
  auto row_quad = [&](int bf, int a, bool raw, auto np) {
    const char* const at = planes(bf) + (a >> 1) * 1024 + (a & 1) * 512 + rr * 16;
    const float4 x = *(const float4*)(at + hf * KS * 1024);
    f32x4_t s = quad_of((const bf16_t*)(at + 8 * hf));
#pragma unroll
    for (int p = 1; p < decltype(np)::value; ++p) s += quad_of((const bf16_t*)(at + p * KS * 1024 + 8 * hf));
    return raw ? x : make_float4(s[0], s[1], s[2], s[3]);
  };
  // acc += rows x keys on the FP32 instruction: a key's row from memory
  auto raw_product = [&](f32x16& acc, int bf, const T* key, auto np) {
    const bool raw = raw_row(bf);
#pragma unroll
    for (int j = 0; j < 16; ++j) acc[j] = 0.f;
#pragma unroll 1
    for (int a = 0; a < D / 8; ++a) mul4(acc, row_quad(bf, a, raw, np), load4<VEC>(key - 4 * hf + 8 * a));
  };
  // what has been copied is complete, and what was read is free, after this
  auto turn = [] {
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __syncthreads();
  };
  Op<NP> kv[KS];                  // planes of this lane's K row, then of its V row
  // One wavefront in a workgroup has registers for both rows: asked for at once and before the first turn, they are one round trip.
  constexpr bool BOTH = NW == 1 || HS;
  Op<NP> kk[BOTH ? KS : 1], vo[BOTH ? KS : 1];
  if constexpr (BOTH) {
    float4 x[2 * KS], y[2 * KS];
#pragma unroll
    for (int a = 0; a < KS; ++a) {
      x[2 * a] = load4<VEC>(kr + 16 * a); x[2 * a + 1] = load4<VEC>(kr + 16 * a + 4);
      y[2 * a] = load4<VEC>(vr + 16 * a); y[2 * a + 1] = load4<VEC>(vr + 16 * a + 4);
    }
    if (!HS || wv < pb.G) copy_item(HS ? wv : 0, 0, 0);
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int a = 0; a < KS; ++a) {
      kk[a] = split8<NP>(x[2 * a], x[2 * a + 1]);
      vo[a] = split8<NP>(y[2 * a], y[2 * a + 1]);
    }
  }
  auto load_kv = [&](const T* p) {
    int o = 0;                    // (both rows' planes would be taken out of the loop over the chunks, and spill)
    asm volatile("" : "+v"(o));
    p += o;
#pragma unroll
    for (int a = 0; a < KS; ++a) {
      kv[a] = split8<NP>(load4<VEC>(p + 16 * a), load4<VEC>(p + 16 * a + 4));
      if (a % 4 == 3) __builtin_amdgcn_sched_barrier(0);      // (eight loads in flight)
    }
  };
  // Whether planes do not hold the operands of a product: the row (known from its item), or a key or value beyond them, which
  // has made its sums NaN or infinite.
  auto sums_of = [&](const f32x16& acc) {
    float t[2] = {0.f, 0.f};
#pragma unroll
    for (int j = 0; j < 16; j += 2) t[(j >> 1) & 1] = fmaf(acc[j], acc[j + 1], t[(j >> 1) & 1]);
    return t[0] + t[1];
  };
  auto beyond = [](float t, bool raw) { return __builtin_expect(__ballot(raw || !(fabsf(t) < INFINITY)) != 0ull, 0); };
  // logits -> A / (1 - A).  Attention weights relative to the row's maximum: the instruction makes 0 of one below 2^-126, and where
  // a wavefront has such a weight the library call, which scales it, takes all of them (for every
  // weight it costs the pass 3 %).
  auto weigh = [&](f32x16& s, int bf) {
    float low = INFINITY;
#pragma unroll
    for (int j = 0; j < 16; ++j) {
      s[j] = fmaf(s[j], c2, -stat(bf, j).x);           // maximum
      low = fminf(low, s[j]);
    }
    if (__ballot(low < -126.f) != 0ull) {
#pragma unroll
      for (int j = 0; j < 16; ++j) {
        s[j] = exp2f(s[j]);
        if (j % 4 == 3) __builtin_amdgcn_sched_barrier(0);
      }
    } else {
#pragma unroll
      for (int j = 0; j < 16; ++j) s[j] = __builtin_amdgcn_exp2f(s[j]);
    }
#pragma unroll
    for (int j = 0; j < 16; ++j) s[j] = quotient(s[j], fmaf(-rec, s[j], stat(bf, j).y));      // denominator
  };
  // cross terms -> indicators
  auto measure = [&](f32x16& s, const f32x16& w, int bf, float vvn) {
#pragma unroll
    for (int jq = 0; jq < 4; ++jq) {
      float4 r[4];                                     // zz, champion, its score
      float x[4];
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        r[e] = stat(bf, 4 * jq + e);
        x[e] = fmaxf(fmaf(-2.f, s[4 * jq + e], r[e].x) + vvn, 0.f);
      }
      roots(x);
#pragma unroll
      for (int e = 0; e < 4; ++e) s[4 * jq + e] = n == __float_as_int(r[e].y) ? r[e].z : w[4 * jq + e] * x[e];
    }
  };
  float out[16];
#pragma unroll
  for (int j = 0; j < 16; ++j) out[j] = 0.f;
  if constexpr (HS) {
    // this wavefront's heads; nothing is shared until the end
    auto landed = [] { asm volatile("s_waitcnt vmcnt(0)" ::: "memory"); };
    for (int h = wv; h < pb.G; h += NW) {
      const float vvn = o.vv[(int64_t)(g * pb.G + h) * ldv + nc];
      f32x16 wt, cacc;
#pragma unroll
      for (int j = 0; j < 16; ++j) { wt[j] = 0.f; cacc[j] = 0.f; }
      landed();
      bool raw = raw_row(0);
      contract<NP, NP, KS>([&](int) -> f32x16& { return wt; }, [&](int a, int p) { return row_op(0, a, p); }, [&](int a) { return kk[a]; });
      settle(wt);
      if (beyond(sums_of(wt), raw)) {
        raw_product(wt, 0, kr, std::integral_constant<int, NP>{});
        settle(wt);
      }
      copy_item(h, 1, 1);                              // (the q planes have been read; their statistics stay)
      weigh(wt, 0);
      landed();
      raw = raw_row(1);
      contract<3, NP, KS>([&](int) -> f32x16& { return cacc; }, [&](int a, int p) { return row_op(1, a, p); }, [&](int a) { return vo[a]; });
      settle(cacc);
      if (beyond(sums_of(cacc), raw)) {
        raw_product(cacc, 1, vr, std::integral_constant<int, 3>{});
        settle(cacc);
      }
      if (h + NW < pb.G) copy_item(h + NW, 0, 0);
      measure(cacc, wt, 1, vvn);
#pragma unroll
      for (int j = 0; j < 16; ++j) out[j] = pb.gmax ? fmaxf(out[j], cacc[j]) : out[j] + cacc[j];
    }
    // the heads of the group meet, in the order of the wavefronts, which take 1 / NW of the rows each
    float* const sums = (float*)&rows[0][0];
    __syncthreads();                                   // every wavefront is done with its buffer
#pragma unroll
    for (int j = 0; j < 16; ++j) sums[(wv * 16 + j) * 64 + l] = out[j];
    __syncthreads();
    const float invG = pb.gmax ? 1.f : 1.0f / (float)pb.G;
#pragma unroll
    for (int jj = 0; jj < 16 / NW; ++jj) {
      const int j = wv * (16 / NW) + jj, i = i0 + 8 * (j >> 2) + 4 * hf + (j & 3);
      float x = sums[j * 64 + l];
#pragma unroll
      for (int k = 1; k < NW; ++k) {
        const float y = sums[(k * 16 + j) * 64 + l];
        x = pb.gmax ? fmaxf(x, y) : x + y;
      }
      if (n < pb.P && i < pb.W) score[((int64_t)g * pb.W + i) * pb.ld + n] = x * invG;
    }
    return;
  }
  if constexpr (!BOTH) copy_item(0, 0, 0);
  turn();
  int bf = 0;                     // buffer of the current rows; the other one was last read before the last barrier
  for (int h0 = 0; h0 < pb.G; h0 += HC) {
    f32x16 wt[HC];                // logits, then A / (1 - A), of the heads of this chunk
    float vvn[HC];
#pragma unroll
    for (int c = 0; c < HC; ++c) vvn[c] = o.vv[(int64_t)(g * pb.G + min(h0 + c, pb.G - 1)) * ldv + nc];
    if constexpr (!BOTH) load_kv(kr);
#pragma unroll
    for (int c = 0; c < HC; ++c) {
      if (h0 + c >= pb.G) break;                       // (uniform)
      const bool last = c == HC - 1 || h0 + c + 1 == pb.G;
      if (last) copy_item(h0, 1, bf ^ 1); else copy_item(h0 + c + 1, 0, bf ^ 1);
      f32x16 sacc;
#pragma unroll
      for (int j = 0; j < 16; ++j) sacc[j] = 0.f;
      const bool raw = raw_row(bf);
      contract<NP, NP, KS>([&](int) -> f32x16& { return sacc; }, [&](int a, int p) { return row_op(bf, a, p); }, [&](int a) { return BOTH ? kk[BOTH ? a : 0] : kv[a]; });
      settle(sacc);
      const float t = sums_of(sacc);
      weigh(sacc, bf);
      if (beyond(t, raw)) {
        raw_product(sacc, bf, kr, std::integral_constant<int, NP>{});
        settle(sacc);
        weigh(sacc, bf);
      }
      wt[c] = sacc;
      turn();
      bf ^= 1;
    }
    if constexpr (!BOTH) load_kv(vr);
#pragma unroll
    for (int c = 0; c < HC; ++c) {
      if (h0 + c >= pb.G) break;
      const bool last = c == HC - 1 || h0 + c + 1 == pb.G, end = h0 + c + 1 == pb.G;
      if (!last) copy_item(h0 + c + 1, 1, bf ^ 1); else if (!end) copy_item(h0 + HC, 0, bf ^ 1);
      f32x16 cacc;
#pragma unroll
      for (int j = 0; j < 16; ++j) cacc[j] = 0.f;
      const bool raw = raw_row(bf);
      contract<3, NP, KS>([&](int) -> f32x16& { return cacc; }, [&](int a, int p) { return row_op(bf, a, p); }, [&](int a) { return BOTH ? vo[BOTH ? a : 0] : kv[a]; });
      settle(cacc);
      const float t = sums_of(cacc);
      measure(cacc, wt[c], bf, vvn[c]);
      if (beyond(t, raw)) {
        raw_product(cacc, bf, vr, std::integral_constant<int, 3>{});
        settle(cacc);
        measure(cacc, wt[c], bf, vvn[c]);
      }
#pragma unroll
      for (int j = 0; j < 16; ++j) out[j] = pb.gmax ? fmaxf(out[j], cacc[j]) : out[j] + cacc[j];
      if (!end) {
        turn();
        bf ^= 1;
      }
    }
  }
  const float invG = pb.gmax ? 1.f : 1.0f / (float)pb.G;
  if (n < pb.P) {
#pragma unroll
    for (int j = 0; j < 16; ++j) {
      const int i = i0 + cidx(j, hf);
      if (i < pb.W) score[((int64_t)g * pb.W + i) * pb.ld + n] = out[j] * invG;
    }
  }
}

// How the passes of a layer are launched.
struct Plan {
  int nw, gy, S, kps;       // attention pass: wavefronts of a workgroup, row blocks, key splits, keys of a split
  int na;                   // its workgroups
  bool joint;               // the value-Gram pass is in its launch
  int nb, gw;               // blocks of keys, and of window positions, of the score pass
  int snw;                  // wavefronts of a workgroup of the score pass
  bool hs;                  // they divide the heads of the group
};
Plan plan_f32(const Prob& pb, int s_max, bool gram) {
  Plan x;
  const int cu = n_cu();
  // four wavefronts of 32 rows per workgroup where there are rows for them; splits until about two
  // workgroups per compute unit, at least one block of keys each
  x.nw = pb.R > 64 ? 4 : 2;
  x.gy = (pb.R + 32 * x.nw - 1) / (32 * x.nw);
  int S = (2 * cu + pb.Hkv * x.gy - 1) / (pb.Hkv * x.gy);
  S = std::max(1, std::min(std::min(S, s_max), (pb.L + KB - 1) / KB));
  x.kps = ((pb.L + S - 1) / S + KB - 1) / KB * KB;
  // (one "split": the caller's attention output and log-sum-exp stand in for the pass)
  x.S = pb.ext_lse ? 1 : (pb.L + x.kps - 1) / x.kps;
  x.na = x.S * x.gy * pb.Hkv;
  // Together, unless two wavefronts hold all rows of a head of 128 and have their splits on every compute unit: with 350 registers
  // each they are one to a SIMD, where the value-Gram pass wants two.
  x.joint = gram && !pb.ext_lse && (pb.d == 64 || x.nw == 4 || 2 * x.na <= cu);
  // The heads of a group on up to four wavefronts while a workgroup of them for every 32 keys and positions fits the chip at once (D =
  // 128: one to a compute unit by registers and LDS, two rounds still pay; D = 64: two), else four wavefronts of 32 keys that share the
  // staged rows.  Score + smoothing, both sides of the limits: heads of 128, 500 workgroups, 28/4 heads 96 us against 104, 4/2 heads 57.2 /
  // 59.9, 1000 workgroups, 32/8 heads 110 / 94; heads of 64, 750 workgroups, 28/4 heads 68.9 / 77.5, 32/8 57.2 / 59.8, 1000 workgroups,
  // 16/4 heads 58.3 / 57.2, 32/8 61.6 / 61.3.  A group of one head has one wavefront while that leaves compute units idle.
  x.nb = (pb.P + KB - 1) / KB;
  x.gw = (pb.W + 31) / 32;
  const int64_t nwg = (int64_t)x.nb * x.gw * pb.Hkv;
  x.hs = pb.G >= 2 && nwg <= (pb.d == 64 ? 3 : 2) * cu;
  x.snw = x.hs ? (pb.G == 2 ? 2 : 4) : nwg <= 2 * cu ? 1 : 4;
  return x;
}

template <typename T, int D, bool VEC>
int run(const Prob& pb, const void* q, const void* k, const void* v, const float* gram,
        float* score, char* ws, const ScoreWs& lay, hipStream_t st) {
  const T* qq = (const T*)q;
  const T* kk = (const T*)k;
  const T* vp = (const T*)v;
  const ScorePtrs w = score_ptrs(ws, lay);
  if (pb.ind != 0) gram = nullptr;                 // no projection: vv becomes the squared norm of the value row
  const Plan pl = plan_f32(pb, lay.S_max, gram != nullptr);
  const int cu = n_cu(), S = pl.S, na = pl.na, nb = pl.nb;
  const bool joint = pl.joint;
  const float* part_z = pb.ext_lse ? pb.ext_out : w.part_z;
  const AttnArgs aa = {S, pl.gy, pl.kps};
  auto attn_vv = [&](auto nwc, auto attn, auto vvp, const dim3& gr, const VvArgs& va) {
    constexpr int NW = decltype(nwc)::value;
    constexpr bool ATTN = decltype(attn)::value, VV = decltype(vvp)::value;
    RK_LAUNCH(ATTN ? ST_ATTN : ST_VV, st, (k_attn_vv_f32<T, D, NW, VEC, ATTN, VV>), gr, dim3(64 * NW), 0, st, pb, qq, kk, vp, gram, w,
              aa, va);
  };
  auto chunks_of = [&](int nwv) { return std::min((2 * cu + pb.Hq - 1) / pb.Hq, (nb + nwv - 1) / nwv); };
  auto attn = [&](auto nwc) {
    const int chunks = chunks_of(decltype(nwc)::value);
    if (joint) attn_vv(nwc, std::true_type{}, std::true_type{}, dim3(na + chunks * pb.Hq), VvArgs{na, chunks, lay.ldv});
    else attn_vv(nwc, std::true_type{}, std::false_type{}, dim3(S, pl.gy, pb.Hkv), VvArgs{});
  };
  const std::integral_constant<int, 4> four;
  if (!pb.ext_lse) {
    if (pl.nw == 4) attn(four);
    else attn(std::integral_constant<int, 2>{});
  }
  if (gram && !joint) attn_vv(four, std::false_type{}, std::true_type{}, dim3(chunks_of(4), pb.Hq), VvArgs{0, chunks_of(4), lay.ldv});
  if (!gram) RK_LAUNCH(ST_VV, st, (k_vnorm2_f32<T, D>), dim3((pb.P + 255) / 256, pb.Hkv), dim3(256), 0, st, pb, vp, w.vv, lay.ldv);
  launch_combine<T, D, 2>(pb, vp, S, gram, w, part_z, qq, 0, 0, st);
  auto score_pass = [&](auto nwc, auto hs) {
    constexpr int NW = decltype(nwc)::value;
    constexpr bool HS = decltype(hs)::value;
    RK_LAUNCH(ST_SCORE, st, (k_score_f32<T, D, NW, VEC, HS>), dim3(HS ? nb : (nb + NW - 1) / NW, pl.gw, pb.Hkv), dim3(64 * NW), 0, st, pb, qq, kk,
              vp, w, lay.ldv, score);
  };
  if (pl.hs && pl.snw == 2) score_pass(std::integral_constant<int, 2>{}, std::true_type{});
  else if (pl.hs) score_pass(four, std::true_type{});
  else if (pl.snw == 1) score_pass(std::integral_constant<int, 1>{}, std::false_type{});
  else score_pass(four, std::false_type{});
  return hip_status();
}

template <typename T, int D>
int pick(const Prob& pb, const void* q, const void* k, const void* v, const float* gram, float* score, char* ws,
         const ScoreWs& lay, hipStream_t st) {
  // 4-element accesses (16 or 8 bytes) where every row starts on such a boundary
  const bool vec = (((uintptr_t)q | (uintptr_t)k | (uintptr_t)v) & (4 * sizeof(T) - 1)) == 0 &&
                   ((pb.q_sh | pb.q_st | pb.kv_sh | pb.kv_st) & 3) == 0;
  return vec ? run<T, D, true>(pb, q, k, v, gram, score, ws, lay, st) : run<T, D, false>(pb, q, k, v, gram, score, ws, lay, st);
}

}  // namespace

int fp32_plan(const Prob& pb, int32_t* plan) {
  if (pb.dtype != RESTKV_F32) return RESTKV_EUNSUPPORTED;
  const Plan x = plan_f32(pb, score_ws(pb).S_max, pb.ind == 0);
  plan[0] = x.S;
  plan[1] = x.joint;
  plan[2] = x.snw;
  plan[3] = x.hs;
  return RESTKV_OK;
}

int launch_score_simple(const Prob& pb, const void* q, const void* k, const void* v,
                        const float* gram, float* score, char* ws, const ScoreWs& lay,
                        hipStream_t st) {
  if (pb.dtype == RESTKV_F32) {
    return pb.d == 64 ? pick<float, 64>(pb, q, k, v, gram, score, ws, lay, st)
                      : pick<float, 128>(pb, q, k, v, gram, score, ws, lay, st);
  }
  return pb.d == 64 ? pick<bf16_t, 64>(pb, q, k, v, gram, score, ws, lay, st)
                    : pick<bf16_t, 128>(pb, q, k, v, gram, score, ws, lay, st);
}

}  // namespace restkv

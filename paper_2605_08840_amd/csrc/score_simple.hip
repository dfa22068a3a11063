// Reconstruction indicator in FP32 (float32 inputs, and bf16 inputs whose shape or alignment the
// bf16 path does not take).
//
// The same four stages and scratch layout as the bf16 path, every product in FP32 on
// v_mfma_f32_32x32x2_f32:
//
//   C layout of a 32x32 block:  register j of lane l holds
//       M index = 8*(j/4) + 4*(l/32) + (j%4),   N index = l % 32;
//   A / B operands: lane l holds M (or N) index l % 32 and ONE K index, chosen by l / 32.
//
// Which two K indices a step multiplies is free as long as A and B agree.  Contractions over the
// head dimension take (8a + e, 8a + 4 + e): a lane then reads its operands of four steps as one
// 16-byte piece.  The contraction over the keys (P.V) takes the pair of keys that register j of a
// logit block holds in the two lane halves, so the attention weights are operands as they stand.
// An instruction is 64 cycles for one operand register each: what bounds these kernels is the
// matrix pipe (157 TFLOP/s), not LDS nor HBM.  Measured at 8k tokens, 32/8 heads of 128, window 32,
// against vector-ALU kernels that read two LDS words per multiply-add: attention pass 338 -> 55 us,
// value-Gram pass 478 -> 56 us, score pass 266 -> 60 us (14 GFLOP executed: 82 TFLOP/s).
#include <algorithm>

#include "score_common.hpp"

namespace restkv {

namespace {

typedef float f32x16 __attribute__((ext_vector_type(16)));

constexpr int KB = 32;      // keys per block (one side of an MFMA)
constexpr float LOG2E = 1.4426950408889634f;
constexpr float RESCALE_TH = 8.0f;  // log2 units a joining logit may run ahead of the reference

#define MFMA32(a, b, c) __builtin_amdgcn_mfma_f32_32x32x2f32((a), (b), (c), 0, 0, 0)

// Wait states between the last MFMA on a block and the first read of its result, spelled out (18 for
// a 16-pass instruction): where branches lie in between, hipcc 7.2 inserts too few on some path, and
// the last registers of the block come out stale.
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

// A block of KB rows of D floats on its way from global memory to LDS through NT threads' registers.
template <int D, int NT>
struct Stage {
  static constexpr int N = KB * D / 4 / NT;
  float4 r[N];
  // ptr_of(row): address of a row's first element, or nullptr for a row of zeros
  template <bool VEC, typename F>
  __device__ __forceinline__ void fetch(F ptr_of) {
#pragma unroll
    for (int j = 0; j < N; ++j) {
      const int x = (int)threadIdx.x + j * NT, row = x / (D / 4), c4 = x % (D / 4);
      const auto p = ptr_of(row);
      r[j] = p ? load4<VEC>(p + 4 * c4) : make_float4(0.f, 0.f, 0.f, 0.f);
    }
  }
  __device__ __forceinline__ void store(float* lds, int stride) const {
#pragma unroll
    for (int j = 0; j < N; ++j) {
      const int x = (int)threadIdx.x + j * NT, row = x / (D / 4), c4 = x % (D / 4);
      *(float4*)&lds[row * stride + 4 * c4] = r[j];
    }
  }
};

// Attention pass: per key split, online softmax of every window query with its dominant key kept
// out of the sums (outputs described in score_common.hpp).  A wavefront owns 32 query rows, on the
// N side: a lane is half of a row, its softmax state is scalar.  K and V blocks of 32 keys are
// double-buffered in LDS, the next block's loads are in flight while a block is worked on.  Row
// strides in LDS: D + 4 floats for K (16-byte reads down the rows), D + 8 for V (4-byte reads along
// a row, the lane halves four rows apart), so that neither read meets a bank twice.
// grid (S, ceil(R / (32 NW)), Hkv), 64 NW threads.
template <typename T, int D, int NW, bool VEC>
__global__ __launch_bounds__(NW * 64, 2) void k_attn_f32(Prob pb, const T* __restrict__ q, const T* __restrict__ k,
                                                         const T* __restrict__ v, int S, int kps, ScorePtrs o) {
  constexpr int CB = D / 32, KST = D + 4, VST = D + 8;
  __shared__ __attribute__((aligned(16))) float Ks[2][KB * KST];
  __shared__ __attribute__((aligned(16))) float Vs[2][KB * VST];
  const int s = blockIdx.x, g = blockIdx.z;
  const int l = threadIdx.x & 63, wv = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6)), rr = l & 31, hf = l >> 5;
  const int r = (blockIdx.y * NW + wv) * 32 + rr;       // row inside the KV head
  const bool valid = r < pb.R;
  const int hl = valid ? r / pb.W : 0, i = valid ? r % pb.W : 0;
  const int vis_last = (pb.causal && valid) ? pb.P + i : pb.L - 1;
  const T* kg = k + (int64_t)g * pb.kv_sh;
  const T* vg = v + (int64_t)g * pb.kv_sh;
  const int kbeg = s * kps, kend = min(pb.L, kbeg + kps);
  const int nblk = kend > kbeg ? (kend - kbeg + KB - 1) / KB : 0;

  float4 qf[D / 8];
  {
    const T* qp = q + (int64_t)(g * pb.G + hl) * pb.q_sh + (int64_t)i * pb.q_st + 4 * hf;
#pragma unroll
    for (int a = 0; a < D / 8; ++a) qf[a] = load4<VEC>(qp + 8 * a);
  }
  const float c2 = pb.scale * LOG2E;
  float mall = -INFINITY, mref = -INFINITY, mx = -INFINITY, lsum = 0.f;
  int nx = -1;                       // key kept out of the sums, -1: none
  int ni = 0;                        // key of the largest logit (the one kept out, if any)
  f32x16 oacc[CB];
#pragma unroll
  for (int cb = 0; cb < CB; ++cb)
#pragma unroll
    for (int j = 0; j < 16; ++j) oacc[cb][j] = 0.f;

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
  Stage<D, NW * 64> sk, sv;
  auto fetch = [&](int t) {
    const int k0 = kbeg + t * KB;
    sk.template fetch<VEC>([&](int row) { return k0 + row < kend ? kg + (int64_t)(k0 + row) * pb.kv_st : nullptr; });
    sv.template fetch<VEC>([&](int row) { return k0 + row < kend ? vg + (int64_t)(k0 + row) * pb.kv_st : nullptr; });
  };
  if (nblk > 0) {
    fetch(0);
    sk.store(Ks[0], KST);
    sv.store(Vs[0], VST);
    __syncthreads();
  }
  for (int t = 0; t < nblk; ++t) {
    const int k0 = kbeg + t * KB;
    if (t + 1 < nblk) fetch(t + 1);
    f32x16 sacc;
#pragma unroll
    for (int j = 0; j < 16; ++j) sacc[j] = 0.f;
    const float* kt = &Ks[t & 1][rr * KST + 4 * hf];
#pragma unroll
    for (int a = 0; a < D / 8; ++a) {
      const float4 kf = *(const float4*)(kt + 8 * a);
      sacc = MFMA32(kf.x, qf[a].x, sacc);
      sacc = MFMA32(kf.y, qf[a].y, sacc);
      sacc = MFMA32(kf.z, qf[a].z, sacc);
      sacc = MFMA32(kf.w, qf[a].w, sacc);
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
      // mass without the candidate, relative to the candidate itself
      float rest = lsum * __builtin_amdgcn_exp2f((mref - tm) * c2);    // (empty sums: 0 * 0)
      int cand = 0x7FFFFFFF;
#pragma unroll
      for (int j = 0; j < 16; ++j) {
        rest += __builtin_amdgcn_exp2f((sacc[j] - tm) * c2);
        if (sacc[j] == tm) cand = min(cand, k0 + cidx(j, hf));
      }
      rest = half_sum(rest) - 1.f;
      cand = half_min(cand);
      ni = newmax ? cand : ni;
      if (nx >= 0) rest += __builtin_amdgcn_exp2f((mx - tm) * c2);
      // (rest carries the rounding of the sum it was taken from: a tie may go either way)
      const bool dominant = newmax && tm > -INFINITY && rest < 1.0001f;
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
    const float* vt = &Vs[t & 1][4 * hf * VST + rr];
#pragma unroll
    for (int j = 0; j < 16; ++j)
#pragma unroll
      for (int cb = 0; cb < CB; ++cb)
        oacc[cb] = MFMA32(vt[(8 * (j >> 2) + (j & 3)) * VST + 32 * cb], sacc[j], oacc[cb]);
    if (t + 1 < nblk) {                // the other buffers were last read before the barrier that ended block t-1
      sk.store(Ks[(t + 1) & 1], KST);
      sv.store(Vs[(t + 1) & 1], VST);
      __syncthreads();
    }
  }
#pragma unroll
  for (int cb = 0; cb < CB; ++cb) settle(oacc[cb]);
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
// (M is symmetric), so that 32x32 blocks below the diagonal are skipped.  T of the workgroup's head
// stays in LDS (row stride D + 4 floats); a wavefront takes 32 keys at a time, on the N side, whose
// values are operand registers and, because the K pairs were chosen like the rows a lane holds in
// the C layout, also exactly the factors of the row dot.  grid (chunks, Hq), 256 threads.
template <typename T, int D, bool VEC>
__global__ __launch_bounds__(256, 2) void k_vv_f32(Prob pb, const T* __restrict__ v, const float* __restrict__ gram,
                                                   float* __restrict__ vv, int ldv) {
  constexpr int CB = D / 32, ST = D + 4;
  __shared__ __attribute__((aligned(16))) float Ts[D * ST];
  const int h = blockIdx.y, g = h / pb.G;
  const int l = threadIdx.x & 63, wv = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6)), rr = l & 31, hf = l >> 5;
  const T* vg = v + (int64_t)g * pb.kv_sh;
  const int nb = (pb.P + KB - 1) / KB;
  float4 vf[D / 8];
  auto fetch = [&](int b) {
    const T* vr = vg + (int64_t)min(b * KB + rr, pb.P - 1) * pb.kv_st + 4 * hf;
#pragma unroll
    for (int a = 0; a < D / 8; ++a) vf[a] = load4<VEC>(vr + 8 * a);
  };
  int b = blockIdx.x * 4 + wv;
  if (b < nb) fetch(b);
  const float* Mh = gram + (int64_t)h * D * D;
  for (int x = threadIdx.x; x < D * D / 4; x += 256) {
    const int i = x / (D / 4), j0 = 4 * (x % (D / 4));
    float m[4] = {Mh[i * D + j0], Mh[i * D + j0 + 1], Mh[i * D + j0 + 2], Mh[i * D + j0 + 3]};
#pragma unroll
    for (int e = 0; e < 4; ++e) m[e] = j0 + e > i ? 2.f * m[e] : (j0 + e == i ? m[e] : 0.f);
    *(float4*)&Ts[i * ST + j0] = make_float4(m[0], m[1], m[2], m[3]);
  }
  __syncthreads();
  for (; b < nb; b += 4 * gridDim.x) {
    float acc = 0.f;
#pragma unroll
    for (int cb = 0; cb < CB; ++cb) {
      f32x16 y;
#pragma unroll
      for (int j = 0; j < 16; ++j) y[j] = 0.f;
      const float* tr = &Ts[(32 * cb + rr) * ST + 4 * hf];
#pragma unroll
      for (int a = 4 * cb; a < D / 8; ++a) {
        const float4 tf = *(const float4*)(tr + 8 * a);
        y = MFMA32(tf.x, vf[a].x, y);
        y = MFMA32(tf.y, vf[a].y, y);
        y = MFMA32(tf.z, vf[a].z, y);
        y = MFMA32(tf.w, vf[a].w, y);
      }
      settle(y);
#pragma unroll
      for (int jq = 0; jq < 4; ++jq) {
        const float4 x = vf[4 * cb + jq];
        acc = fmaf(y[4 * jq + 0], x.x, acc);
        acc = fmaf(y[4 * jq + 1], x.y, acc);
        acc = fmaf(y[4 * jq + 2], x.z, acc);
        acc = fmaf(y[4 * jq + 3], x.w, acc);
      }
    }
    const int n = b * KB + rr;
    acc = half_sum(acc);
    if (b + 4 * (int)gridDim.x < nb) fetch(b + 4 * gridDim.x);
    if (hf == 0 && n < pb.P) vv[(int64_t)h * ldv + n] = acc;
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

// Score pass: logits again, cross term u.v_n, closed form, mean (or maximum) over the group.  A
// wavefront owns 32 keys (N side: a store writes 32 consecutive keys of a row), whose K and V rows
// are its B operands in registers for the whole kernel, and 32 window positions (M side); it walks
// the heads of the group, whose q and u rows and statistics all wavefronts share through double-
// buffered LDS.  grid (ceil(P / (32 NW)), ceil(W / 32), Hkv), 64 NW threads.
template <typename T, int D, int NW, bool VEC>
__global__ __launch_bounds__(NW * 64, NW == 1 ? 1 : 2) void k_score_f32(Prob pb, const T* __restrict__ q, const T* __restrict__ k,
                                                          const T* __restrict__ v, ScorePtrs o, int ldv,
                                                          float* __restrict__ score) {
  constexpr int ST = D + 4, NT = NW * 64;
  __shared__ __attribute__((aligned(16))) float Qs[2][KB * ST];
  __shared__ __attribute__((aligned(16))) float Us[2][KB * ST];
  __shared__ __attribute__((aligned(16))) float st[2][5][32];    // per row: max, denominator, zz, champion key, its score
  const int g = blockIdx.z, i0 = blockIdx.y * 32;
  const int l = threadIdx.x & 63, wv = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6)), rr = l & 31, hf = l >> 5;
  const int n = (blockIdx.x * NW + wv) * KB + rr, nc = min(n, pb.P - 1);
  float4 kf[D / 8], vf[D / 8];
  {
    const T* kr = k + (int64_t)g * pb.kv_sh + (int64_t)nc * pb.kv_st + 4 * hf;
    const T* vr = v + (int64_t)g * pb.kv_sh + (int64_t)nc * pb.kv_st + 4 * hf;
#pragma unroll
    for (int a = 0; a < D / 8; ++a) kf[a] = load4<VEC>(kr + 8 * a);
#pragma unroll
    for (int a = 0; a < D / 8; ++a) vf[a] = load4<VEC>(vr + 8 * a);
  }
  const float c2 = pb.scale * LOG2E;
  // The attention-weight and value-norm indicators come out of the same expression without the
  // 1 - A (their u, zz and champion are empty, vv is 1 or ||v||^2).
  const float rec = pb.ind == 0 ? 1.f : 0.f;
  Stage<D, NT> sg;                // q, then u of the next head on its way to LDS
  float sst[3];
  auto fetch_q = [&](int hl) {
    const int h = g * pb.G + hl;
    sg.template fetch<VEC>([&](int row) { return i0 + row < pb.W ? q + (int64_t)h * pb.q_sh + (int64_t)(i0 + row) * pb.q_st : nullptr; });
  };
  // u, and the rows' statistics through the first 32 threads (max, denominator, zz) and the last 32 (champion)
  auto fetch_u = [&](int hl) {
    const int h = g * pb.G + hl;
    sg.template fetch<true>([&](int row) { return i0 + row < pb.W ? o.rs_u + ((int64_t)h * pb.W + i0 + row) * D : (const float*)nullptr; });
    if (threadIdx.x < 32) {
      const int row = h * pb.W + min(i0 + (int)threadIdx.x, pb.W - 1);
      sst[0] = o.rs_m[row]; sst[1] = o.rs_l[row]; sst[2] = o.rs_zz[row];
    } else if (threadIdx.x >= NT - 32) {
      const int row = h * pb.W + min(i0 + (int)threadIdx.x - (NT - 32), pb.W - 1);
      sst[0] = __int_as_float(o.rs_nstar[row]); sst[1] = o.rs_istar[row];
    }
  };
  auto store_u = [&](int bf) {
    sg.store(Us[bf], ST);
    if (threadIdx.x < 32) {
      st[bf][0][threadIdx.x] = sst[0]; st[bf][1][threadIdx.x] = sst[1]; st[bf][2][threadIdx.x] = sst[2];
    } else if (threadIdx.x >= NT - 32) {
      st[bf][3][threadIdx.x - (NT - 32)] = sst[0]; st[bf][4][threadIdx.x - (NT - 32)] = sst[1];
    }
  };
  float out[16];
#pragma unroll
  for (int j = 0; j < 16; ++j) out[j] = 0.f;
  fetch_q(0);
  sg.store(Qs[0], ST);
  fetch_u(0);
  store_u(0);
  __syncthreads();
  for (int hl = 0; hl < pb.G; ++hl) {
    const int bf = hl & 1;
    const bool more = hl + 1 < pb.G;
    const float vvn = o.vv[(int64_t)(g * pb.G + hl) * ldv + nc];
    if (more) fetch_q(hl + 1);
    f32x16 sacc, cacc;
#pragma unroll
    for (int j = 0; j < 16; ++j) { sacc[j] = 0.f; cacc[j] = 0.f; }
    const float* qt = &Qs[bf][rr * ST + 4 * hf];
    const float* ut = &Us[bf][rr * ST + 4 * hf];
#pragma unroll
    for (int a = 0; a < D / 8; ++a) {
      const float4 qa = *(const float4*)(qt + 8 * a);
      sacc = MFMA32(qa.x, kf[a].x, sacc);
      sacc = MFMA32(qa.y, kf[a].y, sacc);
      sacc = MFMA32(qa.z, kf[a].z, sacc);
      sacc = MFMA32(qa.w, kf[a].w, sacc);
    }
    if (more) {                       // the other buffers were last read before the barrier that ended the last head
      sg.store(Qs[bf ^ 1], ST);
      fetch_u(hl + 1);
    }
#pragma unroll
    for (int a = 0; a < D / 8; ++a) {
      const float4 ua = *(const float4*)(ut + 8 * a);
      cacc = MFMA32(ua.x, vf[a].x, cacc);
      cacc = MFMA32(ua.y, vf[a].y, cacc);
      cacc = MFMA32(ua.z, vf[a].z, cacc);
      cacc = MFMA32(ua.w, vf[a].w, cacc);
    }
    settle(sacc);
    settle(cacc);
    // Attention weights relative to the row's maximum.  The instruction makes 0 of one below 2^-126: where
    // a wavefront has such a weight the library call, which scales it, takes all of them (for every
    // weight it costs the pass 3 %).
    float low = INFINITY;
#pragma unroll
    for (int jq = 0; jq < 4; ++jq) {
      const float4 rm = *(const float4*)&st[bf][0][8 * jq + 4 * hf];
      const float m_[4] = {rm.x, rm.y, rm.z, rm.w};
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        sacc[4 * jq + e] = fmaf(sacc[4 * jq + e], c2, -m_[e]);
        low = fminf(low, sacc[4 * jq + e]);
      }
    }
    if (__ballot(low < -126.f) != 0ull) {
#pragma unroll
      for (int j = 0; j < 16; ++j) sacc[j] = exp2f(sacc[j]);
    } else {
#pragma unroll
      for (int j = 0; j < 16; ++j) sacc[j] = __builtin_amdgcn_exp2f(sacc[j]);
    }
#pragma unroll
    for (int jq = 0; jq < 4; ++jq) {
      const int m0 = 8 * jq + 4 * hf;
      const float4 rl = *(const float4*)&st[bf][1][m0], rz = *(const float4*)&st[bf][2][m0],
                   rn = *(const float4*)&st[bf][3][m0], ri = *(const float4*)&st[bf][4][m0];
      const float l_[4] = {rl.x, rl.y, rl.z, rl.w}, z_[4] = {rz.x, rz.y, rz.z, rz.w},
                  n_[4] = {rn.x, rn.y, rn.z, rn.w}, s_[4] = {ri.x, ri.y, ri.z, ri.w};
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const int j = 4 * jq + e;
        const float ex = sacc[j];
        const float dist2 = fmaf(-2.f, cacc[j], z_[e]) + vvn;
        float val = ex / fmaf(-rec, ex, l_[e]) * sqrtf(fmaxf(dist2, 0.f));
        val = n == __float_as_int(n_[e]) ? s_[e] : val;
        out[j] = pb.gmax ? fmaxf(out[j], val) : out[j] + val;
      }
    }
    if (more) {
      store_u(bf ^ 1);
      __syncthreads();
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

template <typename T, int D, bool VEC>
int run(const Prob& pb, const void* q, const void* k, const void* v, const float* gram,
        float* score, char* ws, const ScoreWs& lay, hipStream_t st) {
  const T* qq = (const T*)q;
  const T* kk = (const T*)k;
  const T* vp = (const T*)v;
  const ScorePtrs w = score_ptrs(ws, lay);
  const int cu = n_cu();
  // four wavefronts of 32 rows per workgroup where there are rows for them; splits until about two
  // workgroups per compute unit, at least one block of keys each
  const int nw = pb.R > 64 ? 4 : 2;
  const int gy = (pb.R + 32 * nw - 1) / (32 * nw);
  int S = (2 * cu + pb.Hkv * gy - 1) / (pb.Hkv * gy);
  S = std::max(1, std::min(std::min(S, lay.S_max), (pb.L + KB - 1) / KB));
  const int kps = ((pb.L + S - 1) / S + KB - 1) / KB * KB;
  S = (pb.L + kps - 1) / kps;
  if (pb.ind != 0) gram = nullptr;                 // no projection: vv becomes the squared norm of the value row
  const float* part_z = w.part_z;
  if (pb.ext_lse) {
    // the caller's attention output and log-sum-exp stand in for the attention pass: one "split"
    S = 1;
    const int rows = pb.Hq * pb.W;
    RK_LAUNCH(ST_ATTN, st, (k_stats_fill<0>), dim3((rows + 255) / 256), dim3(256), 0, st, rows, pb.ext_lse,
              w.part_m, w.part_mx, w.part_n, w.part_ref, w.part_l);
    part_z = pb.ext_out;
  } else {
    if (nw == 4)
      RK_LAUNCH(ST_ATTN, st, (k_attn_f32<T, D, 4, VEC>), dim3(S, gy, pb.Hkv), dim3(256), 0, st, pb, qq, kk, vp, S, kps, w);
    else
      RK_LAUNCH(ST_ATTN, st, (k_attn_f32<T, D, 2, VEC>), dim3(S, gy, pb.Hkv), dim3(128), 0, st, pb, qq, kk, vp, S, kps, w);
  }
  launch_combine<T, D>(pb, vp, S, gram, w, part_z, (const T*)nullptr, 0, 0, 0, st);
  const int nb = (pb.P + KB - 1) / KB;               // blocks of keys
  if (gram) {
    int chunks = (2 * cu + pb.Hq - 1) / pb.Hq;
    chunks = std::min(chunks, (nb + 3) / 4);
    RK_LAUNCH(ST_VV, st, (k_vv_f32<T, D, VEC>), dim3(chunks, pb.Hq), dim3(256), 0, st, pb, vp, gram, w.vv, lay.ldv);
  } else {
    RK_LAUNCH(ST_VV, st, (k_vnorm2_f32<T, D>), dim3((pb.P + 255) / 256, pb.Hkv), dim3(256), 0, st, pb, vp, w.vv, lay.ldv);
  }
  // one wavefront per workgroup while that leaves compute units idle, else four that share the staged rows
  const int gw = (pb.W + 31) / 32;
  if ((int64_t)nb * gw * pb.Hkv <= 2 * cu)
    RK_LAUNCH(ST_SCORE, st, (k_score_f32<T, D, 1, VEC>), dim3(nb, gw, pb.Hkv), dim3(64), 0, st, pb, qq, kk, vp, w, lay.ldv, score);
  else
    RK_LAUNCH(ST_SCORE, st, (k_score_f32<T, D, 4, VEC>), dim3((nb + 3) / 4, gw, pb.Hkv), dim3(256), 0, st, pb, qq, kk, vp, w, lay.ldv,
              score);
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

// Reconstruction indicator on the matrix cores (bf16 inputs, FP32 accumulation), gfx950.
//
// Same four stages and scratch layout as the FP32 path: attention pass per key split, merge
// (score_common.hpp), value Gram pass vv, score pass.  Every contraction runs on
// v_mfma_f32_32x32x16_bf16:
//
//   C layout of a 32x32 block:  register j of lane l holds
//       M index = 8*(j/4) + 4*(l/32) + (j%4),   N index = l % 32.
//   A / B operands: lane l holds M (or N) index l % 32 and the 8 consecutive
//       K indices 8*(l/32) .. 8*(l/32)+7 of each 16-wide K step.
//
// The attention pass puts the 32 query rows of a wavefront on the N side (lane % 32 = query
// row, keys or value columns on the M side), so the softmax statistics and the champion
// bookkeeping are per-lane scalars.  The score pass puts the query rows on the M side and the
// keys on the N side, with the heads of a group in consecutive registers, so the mean over
// the group is a few in-lane adds and a store writes 32 consecutive keys of one row.
//
// All three kernels are persistent (about one 8-wavefront workgroup per compute unit walking a
// run of 64-key tiles) and stream their K/V tiles through asynchronous LDS rings (TileRing).
#include <limits.h>

#include <algorithm>
#include <type_traits>

#include "score_common.hpp"

namespace restkv {

namespace {

typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef short s16x4 __attribute__((ext_vector_type(4)));
typedef short s16x8 __attribute__((ext_vector_type(8)));
typedef unsigned int u32x2 __attribute__((ext_vector_type(2)));

constexpr int TN = 64;                 // keys per LDS tile
constexpr float LOG2E = 1.4426950408889634f;
// A joining key that holds more than 1/9 of the others' sum on arrival becomes the reference of its row, so that its
// weight is exact.  Side by side with the value-Gram pass (share_the_chip) there may be fewer splits than there are alone,
// hence fewer keys that are a split's first or kept out, and more weights enter the sums as bf16.  Splits of up to LO_TILES
// tiles, or half as many as alone, then take the weights above 1/16 of the row's sum so far (half of which a lane has: LO_SHARE) in two bf16 parts,
// 16 keys at a time, with a second product for the remainders.  Scores then lie nearer to 64 bits than with all splits,
// whatever the logits.  Distance (2-norm) over that of all splits, plain / sinks / clustered logits, 55 shapes each: mean
// 0.72 / 0.66 / 0.35, worst 0.99 / 0.98 / 0.72; without the second part 1.01 / 1.00 / 1.22 and 1.17 / 1.43 / 1.94.
// Score + smoothing with and without it, 32/8 heads, window 64: 4k 56.8 / 54.9 us, clustered 62.9 / 59.5; 16k 108.7 / 108.0,
// clustered 133.8 / 123.5.  Longer splits lose nothing by being fewer with a limit of 1/33 (clustered, 16k to 50k: 0.80 to
// 1.02 of the distance; 512/64 heads, 3186 tokens, two splits for four 1.18), and would pay up to 11 % (64/8 heads, 32k, clustered).
constexpr float HEAVY_SPLITS = 8.0f, HEAVY_SIDE = 32.0f, HEAVY_LO = 16.0f, LO_SHARE = 8.0f;
constexpr int LO_TILES = 24;
static_assert(HEAVY_LO >= LO_SHARE, "the branch that looks for heavy weights is entered for all of them");
constexpr float RESCALE_TH = 8.0f;  // log2 units a row maximum may run ahead of its reference

#define MFMA(a, b, c) __builtin_amdgcn_mfma_f32_32x32x16_bf16((a), (b), (c), 0, 0, 0)

__device__ __forceinline__ float xhalf_max(float x) {   // max with the lane 32 away
  const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  return fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1]));
}
__device__ __forceinline__ float xhalf_sum(float x) {
  const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}
__device__ __forceinline__ int xhalf_min(int x) {
  const auto r = __builtin_amdgcn_permlane32_swap((unsigned)x, (unsigned)x, false, false);
  return min((int)r[0], (int)r[1]);
}
__device__ __forceinline__ float bf16_to_f(uint16_t b) { return __uint_as_float(((uint32_t)b) << 16); }

// Bit string of a comparison: bits = 16 bits + (x == t), one bit for each x in order.  And x[] = v where register number X + i is n.  In
// groups of four for the distance between a compare and the instruction that reads its outcome (see shift_in_gt_2x2).
__device__ __forceinline__ void shift_in_eq4(uint32_t& bits, float x0, float x1, float x2, float x3, float t) {
  unsigned long long c0, c1, c2;
  asm("v_cmp_eq_f32_e64 %1, %4, %8\n\t"
      "v_cmp_eq_f32_e64 %2, %5, %8\n\t"
      "v_cmp_eq_f32_e64 %3, %6, %8\n\t"
      "v_cmp_eq_f32_e32 vcc, %7, %8\n\t"
      "v_addc_co_u32_e64 %0, %1, %0, %0, %1\n\t"
      "v_addc_co_u32_e64 %0, %2, %0, %0, %2\n\t"
      "v_addc_co_u32_e64 %0, %3, %0, %0, %3\n\t"
      "v_addc_co_u32_e32 %0, vcc, %0, %0, vcc"
      : "+v"(bits), "=&s"(c0), "=&s"(c1), "=&s"(c2)
      : "v"(x0), "v"(x1), "v"(x2), "v"(x3), "v"(t)
      : "vcc");
}
template <int X>
__device__ __forceinline__ void set_where4(float& x0, float& x1, float& x2, float& x3, int n, float v) {
  unsigned long long c0, c1, c2;
  asm("v_cmp_eq_u32_e64 %4, %8, %7\n\t"
      "v_cmp_eq_u32_e64 %5, %9, %7\n\t"
      "v_cmp_eq_u32_e64 %6, %10, %7\n\t"
      "v_cmp_eq_u32_e32 vcc, %11, %7\n\t"
      "v_cndmask_b32_e64 %0, %0, %12, %4\n\t"
      "v_cndmask_b32_e64 %1, %1, %12, %5\n\t"
      "v_cndmask_b32_e64 %2, %2, %12, %6\n\t"
      "v_cndmask_b32_e32 %3, %3, %12, vcc"
      : "+v"(x0), "+v"(x1), "+v"(x2), "+v"(x3), "=&s"(c0), "=&s"(c1), "=&s"(c2)
      : "v"(n), "n"(X), "n"(X + 1), "n"(X + 2), "n"(X + 3), "v"(v)
      : "vcc");
}

// key (or value-column) index of register j of a 32x32 block for this lane half
__device__ __forceinline__ constexpr int cidx(int j, int hf) { return 8 * (j >> 2) + 4 * hf + (j & 3); }

struct RowInfo {
  int hloc, i, h, row;   // head inside the group, window position, query head, global row h*W+i
  bool valid;
};
__device__ __forceinline__ RowInfo row_info(const Prob& pb, int g, int wave_block, int lane, int log2iw) {
  RowInfo r;
  const int rr = lane & 31;
  const int iw = 1 << log2iw;
  r.hloc = rr >> log2iw;
  r.i = wave_block * iw + (rr & (iw - 1));
  r.valid = r.hloc < pb.G && r.i < pb.W;
  r.h = g * pb.G + (r.valid ? r.hloc : 0);
  r.row = r.h * pb.W + (r.valid ? r.i : 0);
  return r;
}

// vv without a projection: squared norm of the value row (1 for the attention-weight
// indicator, which has no value term).  grid (ceil(P/256), Hkv)
template <int D>
__global__ __launch_bounds__(256) void k_vnorm2(Prob pb, const uint16_t* __restrict__ v,
                                                float* __restrict__ vv, int ldv) {
  const int g = blockIdx.y, n = blockIdx.x * 256 + threadIdx.x;
  if (n >= pb.P) return;
  if (pb.ind == 1) {
    for (int hl = 0; hl < pb.G; ++hl) vv[(int64_t)(g * pb.G + hl) * ldv + n] = 1.0f;
    return;
  }
  const uint16_t* vr = v + (int64_t)g * pb.kv_sh + (int64_t)n * pb.kv_st;
  float acc = 0.f;
#pragma unroll
  for (int c8 = 0; c8 < D / 8; ++c8) {
    const uint4 u = *(const uint4*)(vr + 8 * c8);
    const uint32_t w[4] = {u.x, u.y, u.z, u.w};
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const float a = __uint_as_float(w[e] << 16), b = __uint_as_float(w[e] & 0xFFFF0000u);
      acc = fmaf(a, a, acc);
      acc = fmaf(b, b, acc);
    }
  }
  for (int hl = 0; hl < pb.G; ++hl) vv[(int64_t)(g * pb.G + hl) * ldv + n] = acc;
}

constexpr int ilog2(int x) { return x <= 1 ? 0 : 1 + ilog2(x / 2); }

// ------------------------------------------------------------------------------------------
// Order of the workgroups of the three passes over (KV head, row block, key chunk).  Workgroups go
// round the eight XCDs by their id.  With a multiple of eight KV heads of 128 the head runs fastest: a
// head's workgroups then share one XCD, whose L2 holds the head's Gram matrices, queries and operands,
// and what one pass leaves (split sums, vv, operands) is read by the next on the same XCD.  Score +
// smoothing, 32/8 heads, 8k tokens, window 32: 72.3 -> 70.4 us; 64k and 128k unchanged.  Otherwise the
// chunk runs fastest: with four heads (28/4 of 64, 20k tokens) the row blocks of a key chunk would land
// on two XCDs and fetch its tiles twice, 82.2 -> 84.2 us, and choosing at run time costs the kernels for
// heads of 64 1 %.
template <int D>
__host__ __device__ __forceinline__ bool heads_first(const Prob& pb) { return D == 128 && (pb.Hkv & 7) == 0; }
struct WgAt { int chunk, y, g; };
// workgroup id of a pass of chunks x ny x Hkv workgroups
template <int D>
__device__ __forceinline__ WgAt wg_at(const Prob& pb, int id, int chunks, int ny) {
  const int n0 = heads_first<D>(pb) ? pb.Hkv : chunks, x = id % n0, r = id / n0;
  return heads_first<D>(pb) ? WgAt{r / ny, r % ny, x} : WgAt{x, r % ny, r / ny};
}

// ------------------------------------------------------------------------------------------
// Asynchronous tile ring shared by the pipelined kernels.
//
// A 64-key tile of a [tokens, D] bf16 matrix is copied global -> LDS by global_load_lds_dwordx4:
// each wave-instruction moves 1 KiB (64 lanes x 16 B) to consecutive LDS bytes, while every
// lane picks its own global source.  Inside a tile row the 16-byte chunks are permuted by a
// row-dependent XOR (see TileRing) so that the lanes of one LDS read instruction, which walk
// down the rows at a fixed chunk, spread over all banks without padding between the rows.
// The copies are issued from inline asm and waited for with explicit s_waitcnt
// vmcnt(n): a wave's loads retire in order, and a later store can only make the count higher,
// so "count <= number of loads issued after the group" implies that the group has landed.
// dma_1k with the LDS byte address given as a number (wave-uniform, like base): nothing of the
// copy's addressing is left to the vector ALU but the lane's own offset.
__device__ __forceinline__ void dma_1k_to(const void* base, uint32_t voff, uint32_t lds_dst) {
  asm volatile("s_mov_b32 m0, %2\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, %1" ::"v"(voff), "s"(base), "s"(lds_dst)
               : "memory", "m0");
}
// the same with a 64-bit address per lane
__device__ __forceinline__ void dma_1k_from(const void* src, uint32_t lds_dst) {
  asm volatile("s_mov_b32 m0, %1\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, off" ::"v"(src), "s"(lds_dst) : "memory", "m0");
}
// LDS byte address of a __shared__ object
__device__ __forceinline__ uint32_t lds_addr(const void* p) {
  return (uint32_t)(uintptr_t)(__attribute__((address_space(3))) const void*)p;
}
// The wavefront's index inside its workgroup as a scalar: what is derived from it (ring slots,
// row blocks, the early / late split) then lives in scalar registers and branches.
__device__ __forceinline__ int wave_index() { return __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6)); }
// KIND 0: tile read as MFMA operand columns (16 rows x one 16-byte chunk per instruction):
//         chunk c of row r sits at chunk position c ^ key, key = (r >> log2(16/CH)) & (CH-1).
// KIND 1: tile read through the transposing 8-byte LDS read (4 rows x 4 consecutive chunks per
//         half wave): the GROUP of four chunks c>>2 sits at group position (c>>2) ^ key,
//         key = r & 3 (D = 128) or (r >> 1) & 1 (D = 64).
template <int D, int KIND = 0>
struct TileRing {
  static constexpr int CH = D / 8;                 // 16-byte chunks per row
  static constexpr int RPI = 64 / CH;              // rows per wave-instruction
  static constexpr int NI = TN / RPI;              // wave-instructions per tile
  static constexpr int SH = CH == 16 ? 0 : 1;      // D = 128: 0, D = 64: 1
  __device__ static __forceinline__ int swz(int r, int c) {
    if constexpr (KIND == 0) return c ^ ((r >> SH) & (CH - 1));
    else return c ^ (((r >> SH) & (CH / 4 - 1)) << 2);
  }
  // offset in uint16 units of chunk c of row r
  __device__ static __forceinline__ int off(int r, int c) { return r * D + (swz(r, c) << 3); }
  // wave wv of NW issues its share of one tile: rows [kb, kb+64) of the matrix at `base`
  // (wave-uniform pointer, row pitch `pitch` bytes), clamped to row L-1.  Byte offsets are 32-bit:
  // the host checks that the matrix of one head spans less than 4 GiB.
  template <int NW>
  __device__ static __forceinline__ void issue(const uint16_t* base, uint32_t pitch, int kb, int L,
                                               uint16_t* lds_tile, int wv, int lane) {
    issue_rows<NW>(base, pitch, [&](int r) { return min(kb + r, L - 1); }, lds_tile, wv, lane);
  }
  // the same with an arbitrary matrix row for every tile row r (row_of(r) must be a valid row)
  template <int NW, typename F>
  __device__ static __forceinline__ void issue_rows(const uint16_t* base, uint32_t pitch, F row_of,
                                                    uint16_t* lds_tile, int wv, int lane) {
    static_assert(NI % NW == 0, "tile instructions must divide over the wavefronts");
#pragma unroll
    for (int j = 0; j < NI / NW; ++j) {
      const int blk = wv * (NI / NW) + j;
      const int r = blk * RPI + lane / CH, cs = lane % CH;
      const uint32_t voff = (uint32_t)row_of(r) * pitch + (uint32_t)(swz(r, cs) * 16);
      dma_1k(base, voff, lds_tile + blk * 512);
    }
  }
  // The fast path for tiles that lie wholly inside the matrix (no row clamp): the lane's byte
  // offsets inside a tile are computed once per kernel (plan), a copy then takes the tile's
  // wave-uniform address (tile_base = base + first row * pitch) and LDS address and no vector
  // arithmetic at all.
  template <int NW>
  __device__ static __forceinline__ void plan(uint32_t pitch, int wv, int lane, uint32_t (&off)[NI / NW]) {
#pragma unroll
    for (int j = 0; j < NI / NW; ++j) {
      const int blk = wv * (NI / NW) + j;
      const int r = blk * RPI + lane / CH, cs = lane % CH;
      off[j] = (uint32_t)r * pitch + (uint32_t)(swz(r, cs) * 16);
    }
  }
  template <int NW>
  __device__ static __forceinline__ void issue_whole(const void* tile_base, const uint32_t (&off)[NI / NW],
                                                     uint32_t lds_tile, int wv) {
#pragma unroll
    for (int j = 0; j < NI / NW; ++j) dma_1k_to(tile_base, off[j], lds_tile + (uint32_t)(wv * (NI / NW) + j) * 1024u);
  }
};
// Workgroup barrier without the full fence of __syncthreads (which would also wait for the
// asynchronous tile copies in flight): the wavefront's own LDS accesses are drained first, the
// copies are accounted for separately with wait_vm.
__device__ __forceinline__ void wg_barrier() { asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory"); }
template <int N>
__device__ __forceinline__ void wait_vm() {
  static_assert(N == 0 || N == 1 || N == 2 || N == 3 || N == 4 || N == 5 || N == 8, "add the literal");
  if constexpr (N == 1) asm volatile("s_waitcnt vmcnt(1)" ::: "memory");
  if constexpr (N == 0) asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  if constexpr (N == 2) asm volatile("s_waitcnt vmcnt(2)" ::: "memory");
  if constexpr (N == 4) asm volatile("s_waitcnt vmcnt(4)" ::: "memory");
  if constexpr (N == 8) asm volatile("s_waitcnt vmcnt(8)" ::: "memory");
  if constexpr (N == 3) asm volatile("s_waitcnt vmcnt(3)" ::: "memory");
  if constexpr (N == 5) asm volatile("s_waitcnt vmcnt(5)" ::: "memory");
}

// ------------------------------------------------------------------------------------------
// vv[h, n] = v_n M_h v_n^T with the symmetric Gram matrix M_h, as  sum_j v_j (T v)_j  with the
// lower triangular T = (diag(M) + 2 triu(M, 1))^T, of which half is kept: only the 32 x 32 blocks on or below the diagonal
// are multiplied (10 of 16 for D = 128).  Y^T = T V^T runs on the MFMA with T split into bf16
// high and low parts that stay in registers for the whole kernel; row block rb needs the k-steps
// up to 2 rb + 1, so a wavefront takes the row blocks pr and D/32 - 1 - pr of one head: D/16 + 2
// k-steps whatever pr.  (Lower, so that the lanes of a load, which are rows of T, read along a row of M: with the
// upper triangle every lane read its own row, a cache line per lane and instruction, and a workgroup's Gram entries took 6 us;
// scores from statistics + smoothing, 32/8 heads, 32k, 136.0 -> 133.3 us with the same in the merge.)  The value tiles arrive through a 4-deep asynchronous LDS ring and are
// the B operand shared by all wavefronts; the partial dots of a head's wavefronts meet in LDS.
// A tile has a matrix part (two 32-key halves of 20 MFMAs) and a vector part (the row dots);
// wavefronts 0..3 and 4..7 run them in complementary order (see the loop), so the matrix cores
// stay fed.  The two wavefronts of a head are in the same group.
// The rows of T are taken in the order in which a lane's registers of the product are the value entries that it already
// holds as operands, so the row dots read nothing more from LDS (a third of the reads, and 15 registers): 32/8 heads, 128k
// score + smoothing 598 -> 592 us, 64/8 heads 1014 -> 1003, 256 KV heads of 2112 tokens 374 -> 371.
// KS2 (few heads per KV head): wavefronts 0..3 take keys 0..31 of a tile and wavefronts 4..7 keys
// 32..63 of the same heads, so that a workgroup holds half as many heads.  A wavefront without a head
// only copies.
// Workgroups: key chunks x ceil(G/HPW) x KV heads, 512 threads; HPW = 4 heads per workgroup (8 for D = 64), half
// of that with KS2.
template <int D, bool KS2>
struct VvSmem {
  static constexpr int HPW = 8 / (D / 64) / (KS2 ? 2 : 1);
  __attribute__((aligned(1024))) uint16_t Vs[4][TN * D];
  float part[2][HPW][D / 64][TN];
};
template <int D, bool KS2>
__device__ __forceinline__ void vv_pass(const Prob& pb, WgAt at, VvSmem<D, KS2>& sm, const uint16_t* __restrict__ v,
                                        const float* __restrict__ gram, float* __restrict__ vv,
                                        int ldv, int tiles_per_wg) {
  constexpr int NW = 8, KS = D / 16, CB = D / 32, WPH = CB / 2, HPW = NW / WPH / (KS2 ? 2 : 1);
  constexpr int NMB = KS2 ? 1 : 2;                  // 32-key blocks of a tile per wavefront
  using Ring = TileRing<D, 0>;
  constexpr int NG = Ring::NI / NW;                 // copies per wavefront and tile
  auto& Vs = sm.Vs;
  auto& part = sm.part;
  const int g = at.g;
  const int l = threadIdx.x & 63, wv = threadIdx.x >> 6, rr = l & 31, hf = l >> 5;
  const int wvs = wave_index();                     // the same as a scalar, for the copies' addresses
  const int wr = KS2 ? wvs % (NW / 2) : wvs, ko = KS2 ? 32 * (wvs / (NW / 2)) : 0;   // first key of this wavefront in a tile
  const int hw = wr / WPH, pr = wr % WPH;           // head inside the workgroup, row block pair
  const int hloc = at.y * HPW + hw;
  const int h = g * pb.G + (hloc < pb.G ? hloc : 0);
  const uint16_t* vg = v + (int64_t)g * pb.kv_sh;
  const uint32_t pitch = (uint32_t)pb.kv_st * 2u;

  const int NT = (pb.P + TN - 1) / TN;
  const int t0 = at.chunk * tiles_per_wg;
  const int t1 = min(NT, t0 + tiles_per_wg);
  if (t0 >= t1) return;
  uint32_t voff[NG];
  Ring::template plan<NW>(pitch, wvs, l, voff);
  const uint32_t vs_base = lds_addr(&Vs[0][0]);
  auto issue_tile = [&](int t) {
    const int kb = min(t, t1 - 1) * TN;
    if (kb + TN <= pb.L)
      Ring::template issue_whole<NW>((const char*)vg + (uint64_t)kb * pitch, voff, vs_base + (uint32_t)(t & 3) * (TN * D * 2), wvs);
    else
      Ring::template issue<NW>(vg, pitch, kb, pb.L, Vs[t & 3], wv, l);
  };
  issue_tile(t0);
  issue_tile(t0 + 1);
  if (hloc >= pb.G) {                               // no head: this wavefront's share of the copies only
    wait_vm<NG>();
    wg_barrier();
    for (int t = t0; t < t1; ++t) {
      issue_tile(t + 2);
      wait_vm<NG>();
      wg_barrier();
    }
    wg_barrier();
    wait_vm<0>();
    return;
  }

  auto body = [&](auto prc) {
    constexpr int PR = decltype(prc)::value;
    constexpr int RB0 = CB - 1 - PR, RB1 = PR;      // RB0 >= RB1
    constexpr int N0 = 2 * (RB0 + 1), N1 = 2 * (RB1 + 1);
    bf16x8 ahi0[N0], alo0[N0], ahi1[N1], alo1[N1];
    auto load_frag = [&](int rb, int ks, bf16x8& hi8, bf16x8& lo8) {
      // Column of the Gram matrix that is this lane's row of T: the rows of a block in the order in which a lane's
      // registers of the product (rows 8 a + 4 hf + b) are the value entries that it holds as operands (16 (a / 2) + 8 hf + 4 (a % 2) + b)
      const int j = 32 * rb + ((rr & 0x13) | (rr & 4) << 1 | (rr & 8) >> 1);
      const float* mcol = gram + ((int64_t)h * D + 16 * ks + 8 * hf) * D + j;
      float x[8];
#pragma unroll
      for (int e = 0; e < 8; ++e) x[e] = mcol[e * D];
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        const int i = 16 * ks + 8 * hf + e;
        if (ks >= 2 * rb) x[e] = i < j ? x[e] : (i == j ? 0.5f * x[e] : 0.f);    // (else: left of the diagonal block)
      }
      const Op<2> o = split8<2>(x);
      hi8 = as_bf16x8(o.p[0]);
      lo8 = as_bf16x8(o.p[1]);
    };
#pragma unroll
    for (int a = 0; a < N0; ++a) load_frag(RB0, a, ahi0[a], alo0[a]);
#pragma unroll
    for (int a = 0; a < N1; ++a) load_frag(RB1, a, ahi1[a], alo1[a]);

    // vv of one tile of this wavefront's head: the partial dots of the head's wavefronts meet here
    auto head_sum = [&](int t) {
      if (PR == 0) {
        const int n = t * TN + ko + l;
        if (n < pb.P && (!KS2 || l < 32)) {
          float sum = 0.f;
#pragma unroll
          for (int m2 = 0; m2 < WPH; ++m2) sum += part[(t - t0) & 1][hw][m2][KS2 ? ko + (l & 31) : l];
          vv[(int64_t)h * ldv + n] = 2.f * sum;
        }
      }
    };
    f32x16 y0[NMB], y1[NMB];
    uint4 vq0[NMB][2], vq1[NMB][2];      // the operands that hold the value entries of the two row blocks, for the row dots
    // matrix quarter: Y^T = T V^T for block nb of this wavefront's 32-key blocks of tile t
    auto mat = [&](int nb, int t) {
      const uint16_t* vt = Vs[t & 3];
      __builtin_amdgcn_s_setprio(2);
#pragma unroll
      for (int j = 0; j < 16; ++j) { y0[nb][j] = 0.f; y1[nb][j] = 0.f; }
      // all operand reads of the quarter first: the MFMAs then run back to back instead of one
      // LDS round trip per k-step
      bf16x8 b[N0];
#pragma unroll
      for (int a = 0; a < N0; ++a) b[a] = as_bf16x8(*(const uint4*)&vt[Ring::off(ko + 32 * nb + rr, 2 * a + hf)]);
#pragma unroll
      for (int a = 0; a < 2; ++a) {
        vq0[nb][a] = __builtin_bit_cast(uint4, b[N0 - 2 + a]);
        vq1[nb][a] = __builtin_bit_cast(uint4, b[N1 - 2 + a]);
      }
#pragma unroll
      for (int ks = 0; ks < N0; ++ks) {
        y0[nb] = MFMA(ahi0[ks], b[ks], y0[nb]);
        if (ks < N1) y1[nb] = MFMA(ahi1[ks], b[ks], y1[nb]);
        y0[nb] = MFMA(alo0[ks], b[ks], y0[nb]);
        if (ks < N1) y1[nb] = MFMA(alo1[ks], b[ks], y1[nb]);
      }
      __builtin_amdgcn_s_setprio(0);
    };
    // vector quarter: row dot with v_n (register j of a block is the Gram row of entry 4 (j/4 % 2) + j%4 of operand j/8)
    auto dot = [&](int nb, int t) {
      float a0[4], a1[4];              // four independent chains per row block
#pragma unroll
      for (int jq = 0; jq < 4; ++jq) {
        const uint4 w0 = vq0[nb][jq >> 1], w1 = vq1[nb][jq >> 1];
        const uint2 u0 = jq & 1 ? make_uint2(w0.z, w0.w) : make_uint2(w0.x, w0.y);
        const uint2 u1 = jq & 1 ? make_uint2(w1.z, w1.w) : make_uint2(w1.x, w1.y);
        a0[jq] = y0[nb][4 * jq + 0] * __uint_as_float(u0.x << 16);
        a1[jq] = y1[nb][4 * jq + 0] * __uint_as_float(u1.x << 16);
        a0[jq] = fmaf(y0[nb][4 * jq + 1], __uint_as_float(u0.x & 0xFFFF0000u), a0[jq]);
        a1[jq] = fmaf(y1[nb][4 * jq + 1], __uint_as_float(u1.x & 0xFFFF0000u), a1[jq]);
        a0[jq] = fmaf(y0[nb][4 * jq + 2], __uint_as_float(u0.y << 16), a0[jq]);
        a1[jq] = fmaf(y1[nb][4 * jq + 2], __uint_as_float(u1.y << 16), a1[jq]);
        a0[jq] = fmaf(y0[nb][4 * jq + 3], __uint_as_float(u0.y & 0xFFFF0000u), a0[jq]);
        a1[jq] = fmaf(y1[nb][4 * jq + 3], __uint_as_float(u1.y & 0xFFFF0000u), a1[jq]);
      }
      const float acc0 = (a0[0] + a0[1]) + (a0[2] + a0[3]), acc1 = (a1[0] + a1[1]) + (a1[2] + a1[3]);
      const float acc = xhalf_sum(acc0 + acc1);
      if (hf == 0) part[(t - t0) & 1][hw][PR][ko + 32 * nb + rr] = acc;
    };

    // Steps H_t, one tile each, separated by workgroup barriers.  Wavefronts 0..3 run
    //   H_t: matrix(0,t) matrix(1,t) dot(0,t) dot(1,t),
    // wavefronts 4..7 the complementary order, one tile behind with their row dots,
    //   H_t: dot(0,t-1) dot(1,t-1) matrix(0,t) matrix(1,t),
    // so that on every SIMD one wavefront feeds the matrix cores while the other does its vector
    // work.  Tile t is read in H_t only; the copy of tile t+2 is issued at the top of H_t (its
    // slot held tile t-2); a wavefront waits for its share of tile t+1 before the barrier that
    // ends H_t, when only the copy of tile t+2 is younger.  The partial dots of tile t meet in LDS
    // one step after they were written (two buffers).
    const bool late = wv >= NW / 2;
    wait_vm<NG>();           // own share of tile t0 (compiler-issued loads above are older or waited for)
    wg_barrier();
    for (int t = t0; t < t1; ++t) {
      issue_tile(t + 2);     // into the slot of tile t-2
      if (!late) {
        if (t > t0) head_sum(t - 1);
        mat(0, t);
        if constexpr (NMB > 1) mat(1, t);
        dot(0, t);
        if constexpr (NMB > 1) dot(1, t);
      } else {
        if (t > t0 + 1) head_sum(t - 2);
        if (t > t0) {
          dot(0, t - 1);
          if constexpr (NMB > 1) dot(1, t - 1);
        }
        mat(0, t);
        if constexpr (NMB > 1) mat(1, t);
      }
      wait_vm<NG>();         // own share of tile t+1 (only the copy of tile t+2 is younger)
      wg_barrier();
    }
    if (late) {
      dot(0, t1 - 1);
      if constexpr (NMB > 1) dot(1, t1 - 1);
      if (t1 - 2 >= t0) head_sum(t1 - 2);
    } else {
      head_sum(t1 - 1);
    }
    wg_barrier();
    if (late) head_sum(t1 - 1);
    wait_vm<0>();            // no copy may land in LDS after the workgroup has gone
  };
  if constexpr (WPH == 1) {
    body(std::integral_constant<int, 0>{});
  } else {
    if (pr == 0) body(std::integral_constant<int, 0>{});
    else body(std::integral_constant<int, 1>{});
  }
}

// ------------------------------------------------------------------------------------------
// Attention pass, pipelined: per key split, champion-excluded online softmax statistics and
// A.V sums (outputs: the per-split statistics described in score_common.hpp).
// Workgroups: splits x row blocks x KV heads, 512 threads.
//
// K tiles travel through a 3-deep, V tiles through a 4-deep asynchronous LDS ring.  A step t has a
// matrix half (P.V of tile t-1, then Q.K of tile t: 48 MFMAs) and a vector half (softmax
// bookkeeping of tile t).  Every wavefront passes ONE workgroup barrier per step: wavefronts 0..3
// after the vector half, wavefronts 4..7 between the halves, so that the two wavefronts of a SIMD
// alternate between the matrix cores and the vector ALUs without meeting twice per tile.  With
// B_t the barrier of step t: K tile t and V tile t-1 are read between B_t-1 and B_t+1 at the
// latest by the matrix halves of step t (early wavefronts: before B_t, late ones: before their
// B_t too); the copy of tile t+2 is issued at the top of step t, after B_t-1, into the K slot of
// tile t-1 and the V slot of tile t-2, both last read by a matrix half that precedes B_t-1; every
// wavefront waits for its share of tile t+1 (only tile t+2 is younger) before its B_t, the first
// barrier after which tile t+1 is read.
//
// KS2 (row blocks of 32 that fill at most half of the eight wavefronts): a workgroup holds four row
// blocks, wavefronts 0..3 take keys 0..31 of every tile and wavefronts 4..7 keys 32..63, and the two
// halves meet in LDS at the end, so that a split leaves one set of sums either way.  A wavefront
// without rows only copies.
//
// Query rows and sums pass through LDS on their way in and out, so that accesses to memory run along rows: with an access of
// every lane to its own row the rows took 1.3 us and the sums 2 to 3.6 us of a workgroup's time (score + smoothing, 32/8 heads, 8k,
// window 32: 59.3 -> 58.0 us with the Gram entries of the other pass and of the merge read along rows; 28/4 heads of 64,
// 20k 81.4 -> 79.6; 256 KV heads of 2112 tokens 368 -> 358).
//
// LO: groups of 16 keys that hold a heavy weight enter P.V a second time with what bf16 has left of their weights.
template <int D>
struct AttnSmem { __attribute__((aligned(1024))) uint16_t ring[7][TN * D]; };
template <int D, bool KS2, bool LO>
__device__ __forceinline__ void attn_pass(const Prob& pb, WgAt at, AttnSmem<D>& sm, const uint16_t* __restrict__ q,
                                          const uint16_t* __restrict__ k,
                                          const uint16_t* __restrict__ v, int S, int kps,
                                          int log2iw, float heavy, const ScorePtrs& o) {
  constexpr int NW = 8, KS = D / 16, CB = D / 32, RB = KS2 ? 4 : 8, NMB = KS2 ? 1 : 2;
  using RingK = TileRing<D, 0>;
  using RingV = TileRing<D, 1>;
  constexpr int NG = 2 * (RingK::NI / NW);          // copies per wavefront and tile
  auto& ring = sm.ring;
  uint16_t (*Ks)[TN * D] = ring, (*Vs)[TN * D] = ring + 3;

  const int s = at.chunk, g = at.g;
  const int l = threadIdx.x & 63, wv = wave_index(), rr = l & 31, hf = l >> 5;
  const RowInfo ri = row_info(pb, g, at.y * RB + wv % RB, l, log2iw);
  const int ko = KS2 ? 32 * (wv / RB) : 0;          // first key of this wavefront in a tile
  const bool idle = (at.y * RB + wv % RB) << log2iw >= pb.W;   // no row here: this wavefront only copies
  const uint16_t* kg = k + (int64_t)g * pb.kv_sh;
  const uint16_t* vg = v + (int64_t)g * pb.kv_sh;

  const int kbeg = s * kps;
  const int kend = min(pb.L, kbeg + kps);
  const int ntiles = kend > kbeg ? (kend - kbeg + TN - 1) / TN : 0;
  const uint32_t pitch = (uint32_t)pb.kv_st * 2u;
  uint32_t koff[NG / 2], voff[NG / 2];
  RingK::template plan<NW>(pitch, wv, l, koff);
  RingV::template plan<NW>(pitch, wv, l, voff);
  const uint32_t ks_base = lds_addr(&Ks[0][0]), vs_base = lds_addr(&Vs[0][0]);
  auto issue_tile = [&](int t) {
    const int kb = kbeg + min(t, ntiles - 1) * TN;   // past the end: harmless repeat into a free slot
    if (kb + TN <= pb.L) {
      const uint64_t tb = (uint64_t)kb * pitch;
      RingK::template issue_whole<NW>((const char*)kg + tb, koff, ks_base + (uint32_t)(t % 3) * (TN * D * 2), wv);
      RingV::template issue_whole<NW>((const char*)vg + tb, voff, vs_base + (uint32_t)(t & 3) * (TN * D * 2), wv);
    } else {
      RingK::template issue<NW>(kg, pitch, kb, pb.L, Ks[t % 3], wv, l);
      RingV::template issue<NW>(vg, pitch, kb, pb.L, Vs[t & 3], wv, l);
    }
  };
  // The wavefront's query rows come through LDS, in the slots of K tiles 1, 2 and V tiles 1, 2 (half a slot each): a lane that
  // loads its own row's operands touches a cache line per lane and instruction.  (Copies for wavefronts without rows too held up
  // the first tile: 8/8 heads of 128 without the other pass, window 16, 3.8k tokens 8.0 us against 8.4; heads of 64, 12k, with it 17.7
  // against 18.4.  Tile 1 of K on its way before the rows are read, V tile 1 in the slot that is free then: the second wait in
  // the loop costs 32k clustered 91.7 against 91.1, 256 KV heads of 2112 tokens 150.4 against 148.8.)
  const int row_blk = at.y * RB + wv % RB;
  uint16_t* const qs = ring[(wv < NW / 2 ? 1 : 4) + (wv >> 1 & 1)] + (wv & 1) * (32 * D);
  constexpr int QI = 32 / RingK::RPI;               // copies of a wavefront's query rows
  if (ntiles > 0) {
    const uint32_t qd = lds_addr(qs);
    if (!idle) {
#pragma unroll
      for (int j = 0; j < QI; ++j) {                // (an absent row: row (h, 0) once more, masked below)
        const int r = j * RingK::RPI + l / RingK::CH;
        const RowInfo x = row_info(pb, g, row_blk, r, log2iw);
        dma_1k_from(q + (int64_t)x.h * pb.q_sh + (int64_t)(x.valid ? x.i : 0) * pb.q_st + 8 * RingK::swz(r, l % RingK::CH),
                    qd + (uint32_t)j * 1024u);
      }
    }
    issue_tile(0);
  }
  bf16x8 qf[KS];
  const int vis_last = (pb.causal && ri.valid) ? pb.P + ri.i : pb.L - 1;
  const float c2 = pb.scale * LOG2E;

  float mall = -INFINITY, mref = -INFINITY, mx = -INFINITY, lsum = 0.f;
  int nx = -1;                       // key kept out of the sums, -1: none
  f32x16 oacc[CB];
#pragma unroll
  for (int cb = 0; cb < CB; ++cb)
#pragma unroll
    for (int j = 0; j < 16; ++j) oacc[cb][j] = 0.f;
  bf16x8 pv[NMB][2], pr[NMB][2];     // weights; LO: their remainders in the groups that have a bit in `two`
  uint32_t two = 0;

  // lane-constant part of the transposing LDS read of the value tile: row and column of the
  // 8 bytes this lane contributes to a 16 x 16 block
  const int s16 = l & 15;
  const int vrow = 4 * hf + (s16 >> 2), vcol = 16 * ((l >> 4) & 1) + 4 * (s16 & 3);

  // Operand i of P.V (O^T[c, row] += V^T P^T: 16-key group i / CB, columns 32 (i % CB) ..), of Q.K (k-step i / NMB, keys
  // 32 (i % NMB) ..).
  // One address per lane and tile: the permutation is an XOR of address bits that the row's pitch leaves alone (rows 8, 16, 32
  // apart share it), so the chunks of a k-step or column block are an XOR with a constant away.
  typedef __attribute__((address_space(3))) s16x4 lds_s16x4;
  typedef __attribute__((address_space(3))) const bf16x8 lds_bf16x8;
  const uint32_t v_lane = vs_base + 2u * (uint32_t)(RingV::off(ko + vrow, vcol >> 3) + (vcol & 7));
  const uint32_t k_lane = ks_base + 2u * (uint32_t)RingK::off(ko + rr, hf);
  auto v_tile = [&](int t) { return v_lane + (uint32_t)(t & 3) * (TN * D * 2); };
  auto k_tile = [&](int t) { return k_lane + (uint32_t)(t % 3) * (TN * D * 2); };
  auto read_v = [&](uint32_t vt, int i) {
    const uint32_t at = (vt ^ ((uint32_t)(i % CB) << 6)) + (uint32_t)(i / CB) * (16 * D * 2);
    const s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4*)at);
    const s16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4*)(at + 8 * D * 2));
    union { s16x8 s; bf16x8 b; } a;
    a.s = __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
    return a.b;
  };
  auto read_k = [&](uint32_t kt, int i) {
    return *(lds_bf16x8*)((kt ^ ((uint32_t)(i / NMB) << 5)) + (uint32_t)(i % NMB) * (32 * D * 2));
  };
  constexpr int NPV = 2 * NMB * CB, NQK = NMB * KS;
  // The products of a step are one stream with RD operands read ahead (a product is 32 cycles, an LDS round trip four or five): left
  // to itself the compiler asks for an operand right before its product.  Score + smoothing, 32/8 heads, 128k 590 -> 583 us, 32k
  // clustered 209 -> 203; the latter 201 with the search of a key to keep out in groups of four compares.  (LO: five, with six a
  // register goes to scratch.)
  constexpr int RD = NPV < 6 ? NPV : LO ? 5 : 6;
  bf16x8 op[RD];
  // P.V of a tile; next(i): operand i of what follows (nothing after the last tile).  LO: remainders of heavy weights go in
  // ahead of their group's products, with the operands that these have asked for (with reads of their own ahead of the stream, this launch,
  // clustered, window 64: 16/4 heads of 128, 4k 25.7 us against 24.1, 32/8, 8k 40.6 against 38.0; 8/8, window 16, 4k 14.0 / 13.4).
  auto accumulate = [&](uint32_t vt, auto next) {
#pragma unroll
    for (int i = 0; i < RD; ++i) op[i] = read_v(vt, i);
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int i = 0; i < NPV; ++i) {
      if (LO && i % CB == 0 && (two >> i / CB & 1u)) {     // (uniform)
#pragma unroll
        for (int cb = 0; cb < CB; ++cb) oacc[cb] = MFMA(op[(i + cb) % RD], pr[i / (2 * CB)][i / CB & 1], oacc[cb]);
      }
      oacc[i % CB] = MFMA(op[i % RD], pv[i / (2 * CB)][i / CB & 1], oacc[i % CB]);
      if (i + RD < NPV) op[i % RD] = read_v(vt, i + RD);
      else op[i % RD] = next(i + RD - NPV, op[i % RD]);
      __builtin_amdgcn_sched_barrier(0);
    }
  };

  if (ntiles > 0 && idle) {
    wait_vm<0>();
    wg_barrier();
    issue_tile(1);
    for (int t = 0; t < ntiles; ++t) {
      issue_tile(t + 2);
      wait_vm<NG>();
      wg_barrier();
    }
    wait_vm<0>();
  } else if (ntiles > 0) {
    wait_vm<NG>();           // the query rows
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) {
      const uint4 u = *(const uint4*)&qs[RingK::off(rr, 2 * ks + hf)];
      qf[ks] = as_bf16x8(ri.valid ? u : make_uint4(0, 0, 0, 0));
    }
    wait_vm<0>();            // own share of tile 0
    wg_barrier();            // B_-1: every wavefront has its query rows in registers
    issue_tile(1);
    const bool late = wv >= NW / 2;
    constexpr int S0 = NPV % RD;         // place of the first operand of Q.K
#pragma unroll
    for (int i = 0; i < RD; ++i) op[(S0 + i) % RD] = read_k(k_tile(0), i);

    for (int t = 0; t < ntiles; ++t) {
      const int kb = kbeg + t * TN;
      issue_tile(t + 2);     // into the K slot of tile t-1 and the V slot of tile t-2, both last read before B_t-1
      __builtin_amdgcn_s_setprio(0);
      // ---- matrix half: P.V of the previous tile, logits S^T[key, row] = K Q^T of this one ----
      const uint32_t kt = k_tile(t);
      if (t > 0) accumulate(v_tile(t - 1), [&](int i, bf16x8) { return read_k(kt, i); });
      f32x16 sacc[NMB];
#pragma unroll
      for (int mb = 0; mb < NMB; ++mb)
#pragma unroll
        for (int j = 0; j < 16; ++j) sacc[mb][j] = 0.f;
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int i = 0; i < NQK; ++i) {
        sacc[i % NMB] = MFMA(op[(S0 + i) % RD], qf[i / NMB], sacc[i % NMB]);
        if (i + RD < NQK) op[(S0 + i) % RD] = read_k(kt, i + RD);
        __builtin_amdgcn_sched_barrier(0);
      }
      __builtin_amdgcn_s_setprio(2);
      if (late) {            // B_t of the late wavefronts: between the halves
        wait_vm<NG>();       // own share of tile t+1 (only the copies of tile t+2 are younger)
        wg_barrier();
      }
      // ---- vector half ----
      const bool tile_mask = (kb + TN > kend) || (pb.causal && kb + TN - 1 > pb.P);
      if (tile_mask) {
        const int lim = min(kend - 1, vis_last) - (kb + ko + 4 * hf);
#pragma unroll
        for (int mb = 0; mb < NMB; ++mb)
#pragma unroll
          for (int j = 0; j < 16; ++j)
            if (32 * mb + cidx(j, 0) > lim) sacc[mb][j] = -INFINITY;
      }
      // (only one wavefront of the SIMD is in its vector half: independent chains, not one long one)
      auto tile_max = [&] {
        float tq[4];
#pragma unroll
        for (int c = 0; c < 4; ++c) {
          tq[c] = fmaxf(fmaxf(sacc[0][c], sacc[0][4 + c]), sacc[0][8 + c]);
          if constexpr (NMB > 1) {
            tq[c] = fmaxf(fmaxf(tq[c], sacc[0][12 + c]), sacc[NMB - 1][c]);
            tq[c] = fmaxf(fmaxf(tq[c], sacc[NMB - 1][4 + c]), sacc[NMB - 1][8 + c]);
            tq[c] = fmaxf(tq[c], sacc[NMB - 1][12 + c]);
          } else {
            tq[c] = fmaxf(tq[c], sacc[0][12 + c]);
          }
        }
        return xhalf_max(fmaxf(fmaxf(tq[0], tq[1]), fmaxf(tq[2], tq[3])));
      };
      const float tm = tile_max();

      // A key is kept out of the sums only if, on arrival, it is the largest so far AND holds
      // more than half of the mass seen so far (what a key that ends with A > 1/2 always does);
      // such keys are rare after the first tile, so the expensive part of the bookkeeping (index
      // search, folding the previous kept-out key back in) almost never runs.  The weights that enter the P.V product are rounded to bf16;
      // that costs nothing where a key holds a small share of the sums, and would cost up to
      // 2^-9 of a heavy key's share.  So the reference of the exponentials is always a logit that
      // is PART of the sums (never the kept-out key's, which may be any distance above), it is
      // moved exactly onto the largest joining logit of a tile whenever that key is heavy among
      // the others (its weight is then exactly 1, which bf16 holds), and lazily otherwise.
      const bool newmax = tm > mall;
      const float pl = __builtin_amdgcn_exp2f((tm - mref) * c2);   // tile maximum in the current frame (inf on the first tile)
      mall = fmaxf(mall, tm);
      // Nothing to do unless the reference has to move or the tile maximum may be heavy: lsum is
      // this lane's share of the row's sum, so the comparison is a necessary condition for both
      // "kept out" and "heavy", which are settled below.
      bool any_heavy = false;
      if (__ballot((tm - mref) * c2 > RESCALE_TH || pl * heavy > lsum) != 0ull) {
        if (LO) any_heavy = __ballot(pl * LO_SHARE > lsum) != 0ull;
        const float oth = xhalf_sum(lsum);
        bool dominant = false;
        if (newmax) {
          float total = oth;
          if (nx >= 0) total += __builtin_amdgcn_exp2f((mx - mref) * c2);
          // total = inf: the key kept out so far is the whole mass in FP32, and tm is above it
          dominant = pl > total || total == INFINITY;
        }
        float tinc = tm;                 // largest logit of the tile that joins the sums
        int cand = INT_MAX;
        if (__ballot(dominant) != 0ull) {
          // first register of the lane that holds the maximum (-1: none), and the key of it
          uint32_t eq = 0;
#pragma unroll
          for (int mb = 0; mb < NMB; ++mb)
#pragma unroll
            for (int j = 0; j < 16; j += 4) shift_in_eq4(eq, sacc[mb][j], sacc[mb][j + 1], sacc[mb][j + 2], sacc[mb][j + 3], tm);
          const int cj = eq ? __builtin_clz(eq) - (32 - 16 * NMB) : -1;
          const int mine = cj >= 0 && dominant ? kb + ko + 4 * hf + 2 * (cj & ~3) + (cj & 3) : INT_MAX;
          cand = xhalf_min(mine);
          // the new kept-out key leaves the tile: its weight below is exp2(-inf) = 0
          const int cz = dominant && mine == cand ? cj : -1;
          const float none = -INFINITY;
          auto leave = [&](auto x) {
            constexpr int X = decltype(x)::value, MB = X >> 4, J = X & 15;
            float x0 = sacc[MB][J], x1 = sacc[MB][J + 1], x2 = sacc[MB][J + 2], x3 = sacc[MB][J + 3];
            set_where4<X>(x0, x1, x2, x3, cz, none);
            sacc[MB][J] = x0; sacc[MB][J + 1] = x1; sacc[MB][J + 2] = x2; sacc[MB][J + 3] = x3;
          };
          leave(std::integral_constant<int, 0>()); leave(std::integral_constant<int, 4>());
          leave(std::integral_constant<int, 8>()); leave(std::integral_constant<int, 12>());
          if constexpr (NMB > 1) {
            leave(std::integral_constant<int, 16>()); leave(std::integral_constant<int, 20>());
            leave(std::integral_constant<int, 24>()); leave(std::integral_constant<int, 28>());
          }
          tinc = tile_max();
        }
        // Where nothing of the tile joins (one visible key, and it is kept out) the reference
        // stays; a row without any reference yet takes the kept-out key's logit (any finite
        // value will do: its sums are empty).
        float tref = mref;
        if (tinc == -INFINITY) {
          if (mref == -INFINITY) tref = tm;
        } else {
          const float pinc = tinc == tm ? pl : __builtin_amdgcn_exp2f((tinc - mref) * c2);   // inf without a reference
          if (pinc * heavy > oth || (tinc - mref) * c2 > RESCALE_TH) tref = tinc;
        }
        // The key kept out so far joins the sums too (in FP32, below): the reference may not
        // stay far under it, however far it lies above the rest.
        if (dominant && nx >= 0 && (mx - tref) * c2 > RESCALE_TH) tref = mx;
        if (tref != mref) {
          const float f = __builtin_amdgcn_exp2f((mref - tref) * c2);   // first tile: 2^-inf = 0
          lsum *= f;
          if (t > 0)                   // (the first tile finds empty sums)
#pragma unroll
            for (int cb = 0; cb < CB; ++cb)
#pragma unroll
              for (int j = 0; j < 16; ++j) oacc[cb][j] *= f;
          mref = tref;
        }
        if (dominant) {
          if (nx >= 0) {               // the key kept out so far joins the running sums, in FP32
            const float w = __builtin_amdgcn_exp2f((mx - mref) * c2);
            if (hf == 0) lsum += w;
            const uint16_t* vr = vg + (int64_t)nx * pb.kv_st;
#pragma unroll
            for (int cb = 0; cb < CB; ++cb)
#pragma unroll
              for (int jq = 0; jq < 4; ++jq) {
                const uint2 u = *(const uint2*)(vr + 32 * cb + 8 * jq + 4 * hf);
                oacc[cb][4 * jq + 0] += w * __uint_as_float(u.x << 16);
                oacc[cb][4 * jq + 1] += w * __uint_as_float(u.x & 0xFFFF0000u);
                oacc[cb][4 * jq + 2] += w * __uint_as_float(u.y << 16);
                oacc[cb][4 * jq + 3] += w * __uint_as_float(u.y & 0xFFFF0000u);
              }
          }
          mx = tm;
          nx = cand;
        }
      }
      // ---- weights relative to the reference ----
      const float nm = -mref * c2;
      {
        float ls[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int mb = 0; mb < NMB; ++mb)
#pragma unroll
          for (int b8 = 0; b8 < 16; b8 += 8) {
            float pe[8];
#pragma unroll
            for (int e = 0; e < 8; ++e) pe[e] = fmaf(sacc[mb][b8 + e], c2, nm);
#pragma unroll
            for (int e = 0; e < 8; ++e) pe[e] = __builtin_amdgcn_exp2f(pe[e]);
            if (LO)
#pragma unroll
              for (int e = 0; e < 8; ++e) sacc[mb][b8 + e] = pe[e];
#pragma unroll
            for (int e = 0; e < 8; ++e) ls[e & 3] += pe[e];
#pragma unroll
            for (int e = 0; e < 8; ++e) pv[mb][b8 >> 3][e] = (__bf16)pe[e];
          }
        lsum += (ls[0] + ls[1]) + (ls[2] + ls[3]);
      }
      if (LO) {
        two = 0;
        if (any_heavy) {
#pragma unroll
          for (int grp = 0; grp < 2 * NMB; ++grp) {
            const int mb = grp >> 1, b8 = 8 * (grp & 1);
            float gm = sacc[mb][b8];
#pragma unroll
            for (int e = 1; e < 8; ++e) gm = fmaxf(gm, sacc[mb][b8 + e]);
            if (__ballot(gm * LO_SHARE > lsum) != 0ull) {
              two |= 1u << grp;
#pragma unroll
              for (int e = 0; e < 8; ++e) pr[mb][grp & 1][e] = (__bf16)(sacc[mb][b8 + e] - (float)pv[mb][grp & 1][e]);
            }
          }
        }
      }
      if (!late) {           // B_t of the early wavefronts: after both halves
        wait_vm<NG>();
        wg_barrier();
      }
    }
    accumulate(v_tile(ntiles - 1), [](int, bf16x8 x) { return x; });   // its slot is not a target of the copies still in flight
    wait_vm<0>();            // no copy may land in LDS after the workgroup has gone
  }
  float ltot = xhalf_sum(lsum);
  if constexpr (KS2) {
    // The two key halves of a row meet in the ring's memory (every copy has landed, every read is done
    // after the first barrier).  As in the merge of the splits: a kept-out key stays out if it is the
    // largest logit of both halves, otherwise it joins the sums, and the reference is the largest
    // logit that is part of them.  Each half brings its own sums to the common reference, then
    // wavefronts 4..7 hand theirs over.
    constexpr int NX = CB * 16 + 1;
    float* const hx = (float*)&ring[0][0] + (wv % RB) * (NX * 64) + l;                  // sums of the second half
    float* const sc = (float*)&ring[0][0] + (RB * NX + (wv % RB) * 10 + wv / RB * 5) * 64 + l;   // scalars of the halves
    const float* const sco = sc + (wv < RB ? 5 : -5) * 64;
    uint2 vr[CB][4];                       // value row of the own kept-out key
    const uint16_t* const vp = vg + (int64_t)max(nx, 0) * pb.kv_st + 4 * hf;
#pragma unroll
    for (int cb = 0; cb < CB; ++cb)
#pragma unroll
      for (int jq = 0; jq < 4; ++jq) vr[cb][jq] = *(const uint2*)(vp + 32 * cb + 8 * jq);
    wg_barrier();
    sc[0] = mall; sc[64] = mx; sc[128] = __int_as_float(nx); sc[192] = mref; sc[256] = ltot;
    wg_barrier();
    const float mall1 = sco[0], mx1 = sco[64], mref1 = sco[192], l1 = sco[256];
    const int nx1 = __float_as_int(sco[128]);
    const float M = fmaxf(mall, mall1);
    // (the sums of a half without a key may hold anything)
    const bool has0 = mall != -INFINITY && ltot > 0.f, has1 = mall1 != -INFINITY && l1 > 0.f;
    const bool out0 = nx >= 0 && mx == M, out1 = nx1 >= 0 && mx1 == M;
    const bool keep0 = out0 && !(out1 && nx1 < nx), keep1 = out1 && !keep0;
    const bool join0 = nx >= 0 && !keep0, join1 = nx1 >= 0 && !keep1;
    float R = -INFINITY;
    if (has0) R = mref;
    if (has1) R = fmaxf(R, mref1);
    if (join0) R = fmaxf(R, mx);
    if (join1) R = fmaxf(R, mx1);
    if (R == -INFINITY) R = M;             // nothing is part of the sums
    const float w0 = has0 ? __builtin_amdgcn_exp2f((mref - R) * c2) : 0.f;
    const float wj = join0 ? __builtin_amdgcn_exp2f((mx - R) * c2) : 0.f;
    ltot = (has0 ? w0 * ltot : 0.f) + wj;
#pragma unroll
    for (int cb = 0; cb < CB; ++cb)
#pragma unroll
      for (int j = 0; j < 16; ++j) {
        const uint2 u = vr[cb][j >> 2];
        const uint32_t e = j & 2 ? u.y : u.x;
        const float ve = __uint_as_float(j & 1 ? e & 0xFFFF0000u : e << 16);
        oacc[cb][j] = fmaf(wj, join0 ? ve : 0.f, has0 ? w0 * oacc[cb][j] : 0.f);
      }
    if (wv >= RB) {
#pragma unroll
      for (int cb = 0; cb < CB; ++cb)
#pragma unroll
        for (int j = 0; j < 16; ++j) hx[(16 * cb + j) * 64] = oacc[cb][j];
      hx[16 * CB * 64] = ltot;
    }
    wg_barrier();
    if (wv >= RB) return;
#pragma unroll
    for (int cb = 0; cb < CB; ++cb)
#pragma unroll
      for (int j = 0; j < 16; ++j) oacc[cb][j] += hx[(16 * cb + j) * 64];
    ltot += hx[16 * CB * 64];
    nx = keep0 ? nx : (keep1 ? nx1 : -1);
    mx = M;
    mall = M;
    mref = R;
  }
  if (ri.valid) {
    const int64_t po = (int64_t)ri.row * S + s;
    if (hf == 0) {
      o.part_m[po] = mall * c2;
      o.part_mx[po] = mx * c2;
      o.part_n[po] = nx;
      o.part_ref[po] = ntiles > 0 ? mref * c2 : 0.f;
      o.part_l[po] = ltot;
    }
  }
  // The sums leave through LDS, 32 columns at a time, so that a store instruction writes whole cache lines (eight rows) and not
  // 16 bytes of 32 rows.  The memory is the wavefront's own: where its half's sums were, or a part of the ring that nobody reads
  // or copies to any more.
  if constexpr (!KS2) wg_barrier();
  float* const zb = KS2 ? (float*)&ring[0][0] + (wv % RB) * ((CB * 16 + 1) * 64) : (float*)&ring[0][0] + wv * (32 * 32 * (D / 64));
  RowInfo zr[4];
#pragma unroll
  for (int k = 0; k < 4; ++k) zr[k] = row_info(pb, g, row_blk, 8 * k + (l >> 3), log2iw);
#pragma unroll
  for (int cb = 0; cb < CB; ++cb) {
    float* const zc = zb + (cb & (D / 64 - 1)) * (32 * 32);        // 16-byte chunk c of row r at c ^ (r % 8)
#pragma unroll
    for (int jq = 0; jq < 4; ++jq) {
      const f32x4 x = {oacc[cb][4 * jq], oacc[cb][4 * jq + 1], oacc[cb][4 * jq + 2], oacc[cb][4 * jq + 3]};
      *(f32x4*)(zc + 32 * rr + 4 * ((2 * jq + hf) ^ (rr & 7))) = x;
    }
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      const int r = 8 * k + (l >> 3);
      const f32x4 x = *(const f32x4*)(zc + 32 * r + 4 * ((l & 7) ^ (r & 7)));
      if (zr[k].valid) *(f32x4*)(o.part_z + ((int64_t)zr[k].row * S + s) * D + 32 * cb + 4 * (l & 7)) = x;
    }
  }
}

// The two passes that need nothing of each other, one launch: workgroups [va.at, va.at + va.n) are the value-Gram pass's,
// the others the attention pass's; the second pass's start as the first one's end.  By registers (heads of 128 205 to 251, heads
// of 64 up to 167) a compute unit holds one workgroup; only where both passes split their tiles in heads of 64 (127: the bound) two.
// ATTN, VV: 0 that pass is not there, 1 it is, 2 with KS2, 3 with LO.  512 threads.
struct AttnArgs { int S, ny, kps, log2iw; float heavy; };
struct VvArgs { int at, n, chunks, ny, ldv, tiles_per_wg; };
template <int D, int ATTN, int VV>
__global__ __launch_bounds__(512, D == 64 && ATTN == 2 && VV != 1 ? 4 : 2) void k_attn_vv(Prob pb, const uint16_t* __restrict__ q, const uint16_t* __restrict__ k,
                                                 const uint16_t* __restrict__ v, const float* __restrict__ gram,
                                                 ScorePtrs o, AttnArgs aa, VvArgs va) {
  __shared__ union { AttnSmem<ATTN ? D : 64> a; VvSmem<D, VV == 2> v; } sm;
  const int id = blockIdx.x;
  if (VV && (!ATTN || (unsigned)(id - va.at) < (unsigned)va.n)) {
    if constexpr (VV != 0)
      vv_pass<D, VV == 2>(pb, wg_at<D>(pb, id - va.at, va.chunks, va.ny), sm.v, v, gram, o.vv, va.ldv, va.tiles_per_wg);
  } else {
    if constexpr (ATTN != 0)
      attn_pass<D, ATTN == 2, ATTN == 3>(pb, wg_at<D>(pb, id - (va.at ? 0 : va.n), aa.S, aa.ny), sm.a, q, k, v, aa.S, aa.kps, aa.log2iw,
                              aa.heavy, o);
  }
}

// ------------------------------------------------------------------------------------------
// Score pass: logits again, cross term u.v_n, closed form, mean over the group.
// Workgroups: key chunks x row blocks x KV heads, 512 threads = 8 wavefronts of 32 query rows each.
//
// Per element (query row r of head h, key n), with M, l, zz the row's softmax maximum,
// denominator and z M_h z^T from the attention pass:
//   a = 2^(s c2 - M - log2(G l)) = A / G,   den = 1 - G a = 1 - A,
//   x = vv[h,n] - 2 (u.v_n - zz/2),          I/G = a sqrt(x) / den = a x rsq(x den^2)
// (1/G of the group mean and 1/l are folded into the exponent, zz/2 into the accumulator's
// start value).  Here the query rows sit on the M side of the MFMA and the keys on the N side:
// a lane owns ONE key of each 32-key block and 16 query rows, ordered so that the heads of a
// group that share a window position are consecutive registers of one lane (local row =
// position * Gp + head).  The group mean is then a few in-lane adds (plus one half swap from
// Gp = 8 on), and a store instruction writes 32 consecutive keys of a row.
//
// Schedule:
//   * K, V and vv tiles arrive through a 3-deep (vv: 4-deep) asynchronous LDS ring, two tiles
//     ahead of their use, so no wavefront waits on a global load in the steady state;
//   * every tile has a matrix half-step (48 MFMAs per wavefront) and a vector half-step
//     (closed form, group mean, stores) separated by workgroup barriers, and wavefronts 4..7
//     run ONE half-step behind wavefronts 0..3 (they pass one extra barrier before the loop,
//     the others one extra after it).  The two wavefronts of a SIMD are therefore always in
//     different half-steps: one feeds the matrix cores while the other uses the vector ALUs;
//   * a workgroup walks a long run of tiles, so the per-row setup is paid once.
// Ring safety, with barriers E_0, E_1, ... and tile t handled by the early half in
// (E_2t, E_2t+2) and by the late half in (E_2t+1, E_2t+3):  the copy of tile t+2 is issued at
// the top of a wavefront's step t, i.e. after E_2t at the earliest, into the K/V slot of tile
// t-1 (last read before E_2t) and the vv slot of tile t-2 (last read before E_2t-1); each
// wavefront waits for its own share of tile t+1 before its mid-step barrier, which for both
// halves precedes E_2t+2, the first barrier after which tile t+1 is read.
// KS2: as in the attention pass, four row blocks per workgroup and 32 keys of a tile per wavefront.
template <int D, int GP, bool KS2>
__global__ __launch_bounds__(512) void k_score_pipe(Prob pb, const uint16_t* __restrict__ q,
                                                    const uint16_t* __restrict__ k,
                                                    const uint16_t* __restrict__ v, ScorePtrs o, int ldv,
                                                    float* __restrict__ score, int tiles_per_wg, int nwb, int chunks, int ny) {
  constexpr int NW = 8, KS = D / 16, LG = ilog2(GP), IW = 32 / GP, RB = KS2 ? 4 : 8, NMB = KS2 ? 1 : 2;
  constexpr int GV = GP < 4 ? 4 : GP;               // vv rows per ring slot (whole 1 KiB copies)
  constexpr int NVB = GV / 4;                       // 1 KiB copies per vv tile
  constexpr int ND = GP <= 4 ? GP : GP / 2;         // distinct heads among a lane's 16 registers
  using Ring = TileRing<D>;
  constexpr int NG = 2 * (Ring::NI / NW) + 1;       // copies per wavefront and tile
  __shared__ __attribute__((aligned(1024))) uint16_t Ks[3][TN * D];
  __shared__ __attribute__((aligned(1024))) uint16_t Vs[3][TN * D];
  __shared__ __attribute__((aligned(1024))) float vvs[4][GV][TN];
  __shared__ __attribute__((aligned(16))) float rowc[NW][4][32];   // per local row: accumulator start values, champion key and score

  const WgAt at = wg_at<D>(pb, blockIdx.x, chunks, ny);
  const int g = at.g;
  const int l = threadIdx.x & 63, wv = threadIdx.x >> 6, rr = l & 31, hf = l >> 5;
  const int wvs = wave_index();                     // the same as a scalar, for the copies' addresses
  const int wb = at.y * RB + wvs % RB;        // block of IW window positions
  const int ko = KS2 ? 32 * (wvs / RB) : 0;         // first key of this wavefront in a tile
  const uint16_t* kg = k + (int64_t)g * pb.kv_sh;
  const uint16_t* vg = v + (int64_t)g * pb.kv_sh;

  const int NT = (pb.P + TN - 1) / TN;
  const int t0 = at.chunk * tiles_per_wg;
  const int t1 = min(NT, t0 + tiles_per_wg);
  if (t0 >= t1) return;

  // vv copy of this wavefront: block wv % NVB (duplicates write identical bytes)
  const int vb = wvs % NVB;
  const float* vv_g = o.vv + (int64_t)g * pb.G * ldv;                    // vv rows of this group
  const uint32_t vv_row = (uint32_t)min(4 * vb + (l >> 4), pb.G - 1) * (uint32_t)ldv;
  const uint32_t pitch = (uint32_t)pb.kv_st * 2u;
  uint32_t kvoff[(NG - 1) / 2];
  Ring::template plan<NW>(pitch, wvs, l, kvoff);
  const uint32_t vvoff = (vv_row + 4u * (uint32_t)(l & 15)) * 4u;
  const uint32_t ks_base = lds_addr(&Ks[0][0]), vs_base = lds_addr(&Vs[0][0]), vv_base = lds_addr(&vvs[0][0][0]);
  auto issue_tile = [&](int t) {
    const int tt = min(t, t1 - 1);                  // past the end: harmless repeat into a free slot
    const int kb = tt * TN;
    if (kb + TN <= pb.L && kb + TN <= ldv) {   // whole tile, no clamp anywhere
      const uint64_t tb = (uint64_t)kb * pitch;
      const uint32_t slot = (uint32_t)(t % 3) * (TN * D * 2);
      Ring::template issue_whole<NW>((const char*)kg + tb, kvoff, ks_base + slot, wvs);
      Ring::template issue_whole<NW>((const char*)vg + tb, kvoff, vs_base + slot, wvs);
      dma_1k_to(vv_g + kb, vvoff, vv_base + (uint32_t)((t & 3) * GV + 4 * vb) * (TN * 4));
    } else {
      Ring::template issue<NW>(kg, pitch, kb, pb.L, Ks[t % 3], wv, l);
      Ring::template issue<NW>(vg, pitch, kb, pb.L, Vs[t % 3], wv, l);
      dma_1k(vv_g, (vv_row + (uint32_t)min(kb + 4 * (l & 15), ldv - 4)) * 4u, &vvs[t & 3][4 * vb][0]);
    }
  };
  issue_tile(t0);          // ring indices run on the absolute tile number
  issue_tile(t0 + 1);

  // A operands: local row rr = position * GP + head
  const float c2 = pb.scale * LOG2E;
  // Gf: what the exponent and the leave-one-out value fold in (G for the mean over the group,
  // 1 for the maximum); Gd: the factor in 1 - A (0 for the indicators without 1 / (1 - A))
  const float Gf = pb.gmax ? 1.f : (float)pb.G, invG = 1.f / Gf;
  const float Gd = pb.ind != 0 ? 0.f : Gf;
  bf16x8 qf[KS], uhi[KS], ulo[KS];
  int nslane = -1;                                   // champion key of local row rr (for the tile test)
  {
    const int head = rr & (GP - 1), i = wb * IW + (rr >> LG);
    const bool valid = head < pb.G && i < pb.W;
    const int h = g * pb.G + (valid ? head : 0);
    const int row = h * pb.W + (valid ? i : 0);
    // operand-ordered copies left by the merge kernel: one 1 KiB run per wavefront and register
    const int64_t plane = (int64_t)pb.Hkv * nwb * (KS * 2 * 32 * 8);
    // (loaded whether the row exists or not, then masked: the buffer holds every padded row of the
    // nwb blocks, a wavefront without a block reads the last one, and unconditional loads are all in
    // flight together)
    const uint16_t* ob = o.op + (((int64_t)(g * nwb + min(wb, nwb - 1)) * KS * 2 + hf) * 32 + rr) * 8;
    const uint4 zero4 = make_uint4(0, 0, 0, 0);
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) {
      const uint16_t* pk = ob + ks * (2 * 32 * 8);
      const uint4 a = *(const uint4*)pk;
      const uint4 b = *(const uint4*)(pk + plane);
      const uint4 c = *(const uint4*)(pk + 2 * plane);
      qf[ks] = as_bf16x8(valid ? a : zero4);
      uhi[ks] = as_bf16x8(valid ? b : zero4);
      ulo[ks] = as_bf16x8(valid ? c : zero4);
    }
    // Start values of the two accumulators of this row, so that the MFMAs deliver
    //   s + (-M - log2(G l)) / c2   and   u.v_n - zz/2   directly.
    // An idle row starts at -inf (its q is zero): its exponential, hence its score, is exactly 0.
    if (valid) nslane = o.rs_nstar[row];
    if (hf == 0) {
      rowc[wv][0][rr] = valid ? (-o.rs_m[row] - log2f(Gf * o.rs_l[row])) / c2 : -INFINITY;
      rowc[wv][1][rr] = valid ? -0.5f * o.rs_zz[row] : 0.f;
      rowc[wv][2][rr] = __int_as_float(nslane);
      rowc[wv][3][rr] = valid ? o.rs_istar[row] * invG : 0.f;
    }
  }
  const float* vvlane = &vvs[0][0][0] + ko + rr;
  // Output a of a lane (after the group mean) belongs to window position i0 + out_pos0(a):
  //   Gp <= 4: registers Gp a .. Gp a + Gp - 1, local row 8 (Gp a / 4) + 4 hf + (Gp a) % 4;
  //   Gp 8, 16: position 2 a + hf after the half swap;   Gp 32: position 0 in both halves.
  constexpr int NOUT = GP <= 4 ? 16 / GP : (GP == 8 ? 2 : 1);
  constexpr int HS = GP <= 4 ? 4 / GP : (GP == 32 ? 0 : 1);   // position step between the lane halves
  auto out_pos0 = [](int a) constexpr {
    return GP <= 4 ? (8 * ((GP * a) >> 2) + ((GP * a) & 3)) >> LG : 2 * a;
  };
  const int i0 = wb * IW + hf * HS;
  const bool rows_full = wb * IW + IW <= pb.W;       // wave-uniform: every position of the block exists
  char* sbase = (char*)(score + (int64_t)g * pb.W * pb.ld);
  const uint32_t ld4 = (uint32_t)pb.ld * 4u;
  const uint32_t voff0 = (uint32_t)i0 * ld4 + (uint32_t)(ko + rr) * 4u;   // 32-bit: checked on the host

  wait_vm<NG>();           // own share of tile t0
  wg_barrier();            // E_2t0
  const bool late = wv >= NW / 2;
  if (late) wg_barrier();

  if (wb >= nwb) {         // no row here: this wavefront's share of the copies only
    for (int t = t0; t < t1; ++t) {
      issue_tile(t + 2);
      wait_vm<NG>();
      wg_barrier();
      wg_barrier();
    }
    if (!late) wg_barrier();
    wait_vm<0>();
    return;
  }
  for (int t = t0; t < t1; ++t) {
    // The wavefront in its vector half-step goes first at the issue port: it is the one with many
    // short instructions, and the half-step that bounds the tile time; the MFMAs of the other
    // wavefront of the SIMD need one issue slot in eight and find it in the gaps (measured: 1.4 %
    // against the opposite order, which is how the kernel was first written).
    __builtin_amdgcn_s_setprio(0);
    issue_tile(t + 2);
    // ---- matrix half-step ----
    const uint16_t* kt = Ks[t % 3];
    const uint16_t* vt = Vs[t % 3];
    f32x16 sacc[NMB], cacc[NMB];
#pragma unroll
    for (int a = 0; a < 4; ++a) {
      const f32x4 s0 = *(const f32x4*)&rowc[wv][0][8 * a + 4 * hf];
      const f32x4 c0 = *(const f32x4*)&rowc[wv][1][8 * a + 4 * hf];
#pragma unroll
      for (int e = 0; e < 4; ++e) {
#pragma unroll
        for (int mb = 0; mb < NMB; ++mb) { sacc[mb][4 * a + e] = s0[e]; cacc[mb][4 * a + e] = c0[e]; }
      }
    }
    // consecutive MFMAs never touch the same accumulator
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) {
      bf16x8 bk[NMB], bv[NMB];
#pragma unroll
      for (int mb = 0; mb < NMB; ++mb) {
        const int of = Ring::off(ko + 32 * mb + rr, 2 * ks + hf);
        bk[mb] = as_bf16x8(*(const uint4*)&kt[of]);
        bv[mb] = as_bf16x8(*(const uint4*)&vt[of]);
      }
#pragma unroll
      for (int mb = 0; mb < NMB; ++mb) {
        sacc[mb] = MFMA(qf[ks], bk[mb], sacc[mb]);
        cacc[mb] = MFMA(uhi[ks], bv[mb], cacc[mb]);
      }
#pragma unroll
      for (int mb = 0; mb < NMB; ++mb) cacc[mb] = MFMA(ulo[ks], bv[mb], cacc[mb]);
    }
    wait_vm<NG>();         // own share of tile t+1 (only the copies of tile t+2 are younger)
    wg_barrier();
    __builtin_amdgcn_s_setprio(2);
    // ---- vector half-step ----
    const int kb = t * TN;
    const float* vvt = vvlane + (t & 3) * (GV * TN);
#pragma unroll
    for (int mb = 0; mb < NMB; ++mb) {
      float vvh[ND];
#pragma unroll
      for (int jd = 0; jd < ND; ++jd)
        vvh[jd] = vvt[((8 * (jd >> 2) + 4 * hf + (jd & 3)) & (GP - 1)) * TN + 32 * mb];
      // stage by stage over 8 registers: eight independent chains in flight
#pragma unroll
      for (int b8 = 0; b8 < 16; b8 += 8) {
        float a[8], x[8], den[8];
#pragma unroll
        for (int e = 0; e < 8; ++e) a[e] = sacc[mb][b8 + e] * c2;
#pragma unroll
        for (int e = 0; e < 8; ++e) x[e] = fmaf(-2.f, cacc[mb][b8 + e], vvh[(b8 + e) % ND]);
#pragma unroll
        for (int e = 0; e < 8; ++e) a[e] = __builtin_amdgcn_exp2f(a[e]);
#pragma unroll
        for (int e = 0; e < 8; ++e) den[e] = fmaf(-Gd, a[e], 1.f);
#pragma unroll
        for (int e = 0; e < 8; ++e) a[e] *= fabsf(x[e]);
#pragma unroll
        for (int e = 0; e < 8; ++e) x[e] = fabsf(x[e]) * den[e];
        // the tiny addend keeps rsq finite when x is exactly 0 (the score is then 0, not NaN)
#pragma unroll
        for (int e = 0; e < 8; ++e) x[e] = fmaf(x[e], den[e], 1e-37f);
#pragma unroll
        for (int e = 0; e < 8; ++e) x[e] = __builtin_amdgcn_rsqf(x[e]);
#pragma unroll
        for (int e = 0; e < 8; ++e) sacc[mb][b8 + e] = a[e] * x[e];
      }
    }
    // key of this lane in the two 32-key blocks of the tile
    int nk[NMB];
#pragma unroll
    for (int mb = 0; mb < NMB; ++mb) nk[mb] = kb + ko + 32 * mb + rr;
    const bool champ_here = nslane >= kb && nslane < kb + TN;
    if (__ballot(champ_here) != 0ull) {    // a champion of this wavefront is here
#pragma unroll
      for (int j = 0; j < 16; ++j) {       // register j of lane half hf is local row 8 (j/4) + 4 hf + j%4
        const int m_ = 8 * (j >> 2) + 4 * hf + (j & 3);
        const int ns = __float_as_int(rowc[wv][2][m_]);
        const float is = rowc[wv][3][m_];
#pragma unroll
        for (int mb = 0; mb < NMB; ++mb)
          if (nk[mb] == ns) sacc[mb][j] = is;
      }
    }
    // ---- mean (or maximum) over the group (in-lane, one half swap from GP = 8 on), store ----
    float outv[NMB][NOUT];
    auto group_reduce = [&](auto maxc) {
      auto comb = [](float x, float y) { return decltype(maxc)::value ? fmaxf(x, y) : x + y; };
#pragma unroll
      for (int mb = 0; mb < NMB; ++mb) {
        if constexpr (GP <= 4) {
#pragma unroll
          for (int a = 0; a < NOUT; ++a) {
            float s = sacc[mb][GP * a];
#pragma unroll
            for (int e = 1; e < GP; ++e) s = comb(s, sacc[mb][GP * a + e]);
            outv[mb][a] = s;
          }
        } else {
          constexpr int RPG = GP / 2;                 // registers per group inside one lane half
          float s[16 / RPG];
#pragma unroll
          for (int a = 0; a < 16 / RPG; ++a) {
            s[a] = sacc[mb][RPG * a];
#pragma unroll
            for (int e = 1; e < RPG; ++e) s[a] = comb(s[a], sacc[mb][RPG * a + e]);
          }
          if constexpr (16 / RPG >= 2) {
#pragma unroll
            for (int a = 0; a < 16 / RPG; a += 2) {
              // lower half ends up with the total of position a, upper half with that of a + 1
              const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(s[a]), __float_as_uint(s[a + 1]),
                                                              false, false);
              outv[mb][a / 2] = comb(__uint_as_float(r[0]), __uint_as_float(r[1]));
            }
          } else {
            // both halves hold (and store) the same total
            outv[mb][0] = decltype(maxc)::value ? xhalf_max(s[0]) : xhalf_sum(s[0]);
          }
        }
      }
    };
    if (pb.gmax) group_reduce(std::true_type{}); else group_reduce(std::false_type{});
    const uint32_t toff = (uint32_t)kb * 4u;
    if (rows_full && kb + TN <= pb.P) {             // wave-uniform: no lane needs a guard
#pragma unroll
      for (int mb = 0; mb < NMB; ++mb)
#pragma unroll
        for (int a = 0; a < NOUT; ++a)
          *(float*)(sbase + (voff0 + toff + (uint32_t)(128 * mb) + (uint32_t)out_pos0(a) * ld4)) = outv[mb][a];
    } else {
#pragma unroll
      for (int mb = 0; mb < NMB; ++mb)
#pragma unroll
        for (int a = 0; a < NOUT; ++a)
          if (i0 + out_pos0(a) < pb.W && kb + ko + 32 * mb + rr < pb.P)
            *(float*)(sbase + (voff0 + toff + (uint32_t)(128 * mb) + (uint32_t)out_pos0(a) * ld4)) = outv[mb][a];
    }
    wg_barrier();
  }
  if (!late) wg_barrier();
  wait_vm<0>();            // no copy may land in LDS after the workgroup has gone
}

// Tiles that the busiest compute unit walks when `per` workgroups share every tile of the nt and each
// takes a run of them: a run, twice if the workgroups are more than the compute units.
int64_t span_tiles(int nt, int64_t per) {
  const int64_t tpw = std::max<int64_t>(1, (nt * per + n_cu() - 1) / n_cu());
  return tpw * (((nt + tpw - 1) / tpw * per + n_cu() - 1) / n_cu());
}

// Row blocks of 32 (padded group x window positions) that a workgroup of 8 wavefronts holds: eight, or
// four whose tiles are split between two wavefronts (KS2).  KS2 where a workgroup walks at least
// min_tiles tiles of n and either four row blocks are all there is, or (wide) the busiest compute unit walks
// at most 3/2 of the tiles, which cost 0.6 each: heads of 64 with nine to twelve blocks, if the workgroups fit the chip
// at once.  Score pass, heads of 64, twelve blocks: 4 KV heads, 20k tokens 25.9 us against 28.2; 8 KV heads
// (264 workgroups), 100k tokens 270 against 207.  Fifteen blocks for eight 1285 against 1006.  With heads of
// 128 a tile costs 0.7: nine to twelve blocks 31.7 against 31.6 and 36.5 against 33.3.  Attention pass, nine and
// ten blocks, 16 tiles for every KV head 69.2 against 67.5, 49 tiles 173 ... 184 against 182 ... 189.
struct RowGeom { int gp, log2iw, nwr, gy; bool ks2; };
RowGeom row_geom(const Prob& pb, int n, int min_tiles, bool wide) {
  RowGeom r;
  r.gp = 1;
  while (r.gp < pb.G) r.gp <<= 1;
  const int iw = 32 / r.gp;
  r.log2iw = ilog2(iw);
  const int nwr = (pb.W + iw - 1) / iw;            // wavefronts needed to cover the window
  const int gy4 = (nwr + 3) / 4, gy8 = (nwr + 7) / 8, nt = (n + TN - 1) / TN;
  r.ks2 = (int64_t)nt * gy4 * pb.Hkv >= (int64_t)min_tiles * n_cu() &&
          (gy4 == gy8 || (wide && 2 * span_tiles(nt, (int64_t)gy4 * pb.Hkv) <= 3 * span_tiles(nt, (int64_t)gy8 * pb.Hkv)));
  r.gy = r.ks2 ? gy4 : gy8;
  r.nwr = nwr;
  return r;
}
// Both halves of a tile pay the first tile's bookkeeping and meet at the end (4-5 us).  32/8 heads of 128,
// window 32: four tiles a workgroup 19.8 us against 23.4 with KS2, 16 tiles 36.4 against 37.8, 32 tiles 65.6
// against 58.9; window 16: eight tiles 23.0 against 23.2, 16 tiles 32.3 against 31.2; six shapes at 16 tiles -1.1 ... +1.4.
constexpr int ATTN_KS2_TILES = 16;
// Score pass, window 32: two tiles a workgroup 12.2 us against 12.6, four 16.5 against 15.8, 32 tiles 72.6 against 63.8.
constexpr int SCORE_KS2_TILES = 4;
// Value-Gram pass, heads of 128 in groups of 2: one tile a workgroup 8.1 us against 10.3, four 12.3 against 13.4,
// eight 17.3 against 17.3, 32 tiles 45.1 against 41.7; groups of 1: 7.1 and 8.0, 11.0 and 10.7, 15.8 and 14.5, 42.8
// and 34.9; heads of 64 in groups of 4: 7.0 and 8.1, 10.2 and 10.4, 14.4 and 13.5, 36.1 and 30.0.
constexpr int VV_KS2_TILES = 6;

template <int D, int GP>
void launch_score_pipe(const Prob& pb, const uint16_t* q, const uint16_t* k, const uint16_t* v, const ScorePtrs& w, int ldv,
                       float* score, int nwb, hipStream_t st) {
  const RowGeom rg = row_geom(pb, pb.P, SCORE_KS2_TILES, D == 64);
  // one resident workgroup per compute unit, each walking a run of tiles
  const int NT = (pb.P + TN - 1) / TN;
  const int tpp = max(1, (int)(((int64_t)NT * rg.gy * pb.Hkv + n_cu() - 1) / n_cu()));
  const int chunks = (NT + tpp - 1) / tpp;
  const dim3 gr(chunks * rg.gy * pb.Hkv);
  if (rg.ks2)
    RK_LAUNCH(ST_SCORE, st, (k_score_pipe<D, GP, true>), gr, dim3(512), 0, st, pb, q, k, v, w, ldv, score, tpp, nwb, chunks, rg.gy);
  else
    RK_LAUNCH(ST_SCORE, st, (k_score_pipe<D, GP, false>), gr, dim3(512), 0, st, pb, q, k, v, w, ldv, score, tpp, nwb, chunks, rg.gy);
}

// (whole tiles: with S splits asked for the last ones may have nothing left)
inline int split_tiles(int nt, int S) { return (nt + S - 1) / S; }
inline int splits_of(int nt, int S) { const int t = split_tiles(nt, S); return (nt + t - 1) / t; }
// S splits beside the value-Gram pass take heavy weights in two parts (S1: splits of the pass alone; see HEAVY_SIDE).
inline bool two_parts(int nt, int S, int S1) {
  const int s = splits_of(nt, S), alone = splits_of(nt, S1);
  return s < alone && (split_tiles(nt, S) <= LO_TILES || 2 * s <= alone);
}

// Attention pass and value-Gram pass side by side, each on a part of the compute units, where that ends earlier than
// one after the other on all of them: fixed parts (launch, operands, first tile, sums) overlap, fewer splits are fewer
// sums for the merge, and a unit bound by vector instructions next to one bound by the matrix cores runs at a higher
// clock.  Model: a workgroup of the attention pass takes A0 + a t us for t tiles, one of the value-Gram pass V0 + v t, one
// after the other V1 more and 6 % more per tile; clustered logits take up to SLOW a.  Where the workgroups of all
// splits leave half of the units free (one or two KV heads, whose splits are as many as the merge takes), the splits stay as
// many and the value-Gram pass has the other units.  Else taken is the split count with the smallest sum of plain and
// clustered time (SPLIT us for each split) that wins for plain logits and loses at most LOSS by the model, which is nothing
// by measurement, for clustered ones; weights in two parts cost clustered ones PARTS a tile, and then they may not lose.
// Score + smoothing, plain / clustered logits, against one after the other in two launches: 32/8 heads, window 64, 4k
// 0.82 / 0.88, 8k 0.88 / 0.96, 16k 0.88 / 0.98, 32k 0.93 / 0.96, 64k 0.94 / 0.96; window 16, 4k 0.84 / 0.90; 64/8, 4k 0.90 / 0.93;
// 8/8, 4k 0.89 / 0.94; 16/4, 4k 0.85 / 0.95, 8k 0.88 / 0.97, 32k 0.91 / 1.02; 28/4, window 32, 32k 0.91 / 1.07, the worst of
// 500 shapes; 4/2, 4k 0.89 / 0.88, 8k 0.89 / 0.89, 16k 0.89 / 0.90; 4/1, 8k 0.86 / 0.87.  (With SPLIT 1.3 for any number of
// heads 4/2, 8k 1.01 / 1.20, 4/1, 16k 0.98 / 1.10, 16/4, 8k, window 16 0.93 / 1.06; with 0.65 32/8, 4k, window 16 0.92.
// With weights in two parts let off as lightly as others 128/32 heads, 4k, one split for two 0.96 / 1.12.)
// Only where the workgroups have equal work: a last row block or head group that
// is mostly empty ends early and leaves its unit idle (28/4 heads, 30k, window 33, clustered 155 us against 161).  Not for heads
// of 64, whose workgroups do less per tile than these constants say (28/4 heads, 50k, clustered 174 us against 192).
inline int share_the_chip(const Prob& pb, int nt, int nwr, int S1, const VvArgs& va, int ny, int* chunks) {
  constexpr float A0 = 10.f, V0 = 6.f, V1 = 4.f, A = 1.5f, V = 1.2f, SEQ = 1.06f, SLOW = 1.5f, LOSS = 1.08f, SPLIT = 0.9f, PARTS = 1.1f;
  if ((ny > 1 && (nwr - 1) % 8 < 4) || (va.ny > 1 && (pb.G - 1) % 4 < 2)) return 0;
  const int ntv = (pb.P + TN - 1) / TN;
  auto tiles = [](int n, int parts) { return (float)((n + parts - 1) / parts); };
  auto seq = [&](float a) { return A0 + V0 + V1 + SEQ * (a * tiles(nt, S1) + V * va.tiles_per_wg); };
  const float seq1 = seq(A), seq2 = seq(SLOW * A);
  float best = INFINITY;
  int bs = 0;
  for (int S = S1; S >= 1; --S) {
    const int c = min(ntv, (n_cu() - S * ny * pb.Hkv) / (va.ny * pb.Hkv));     // chunks for the value-Gram pass
    if (c < 1) continue;
    const bool lo = two_parts(nt, S, S1);
    const float tv = V0 + V * tiles(ntv, c), t1 = max(A0 + A * tiles(nt, S), tv);
    const float t2 = max(A0 + (lo ? PARTS : 1.f) * SLOW * A * tiles(nt, S), tv);
    if (t1 >= seq1 || t2 > (lo ? 1.f : LOSS) * seq2 || t1 + t2 + SPLIT * S > best) continue;
    best = t1 + t2 + SPLIT * S;
    bs = S;
    *chunks = c;
    if (S == S1 && t2 <= seq2 && 2 * S * ny * pb.Hkv <= n_cu()) break;
  }
  return bs;
}

// How the two passes of a layer are launched.
struct AttnVvPlan { RowGeom rg; AttnArgs aa; VvArgs va; bool vks2, side, lo; };
template <int D>
AttnVvPlan plan_attn_vv(const Prob& pb, const ScoreWs& lay, bool gram) {
  AttnVvPlan pl = {row_geom(pb, pb.L, ATTN_KS2_TILES, false), {}, {0, 0, 0, 0, lay.ldv, 0}, false, false, false};
  const RowGeom& rg = pl.rg;
  VvArgs& va = pl.va;
  AttnArgs& aa = pl.aa;
  const int ntv = (pb.P + TN - 1) / TN;
  if (gram) {
    constexpr int HPW = D == 128 ? 4 : 8;
    // as for the rows: half as many heads per workgroup, at most 3/2 of the tiles, VV_KS2_TILES of them
    const int hg4 = (pb.G + HPW / 2 - 1) / (HPW / 2), hg8 = (pb.G + HPW - 1) / HPW;
    const int64_t t4 = span_tiles(ntv, (int64_t)hg4 * pb.Hkv);
    pl.vks2 = t4 >= VV_KS2_TILES && 2 * t4 <= 3 * span_tiles(ntv, (int64_t)hg8 * pb.Hkv);
    va.ny = pl.vks2 ? hg4 : hg8;
    va.tiles_per_wg = max(1, (int)(((int64_t)ntv * va.ny * pb.Hkv + n_cu() - 1) / n_cu()));
    va.chunks = (ntv + va.tiles_per_wg - 1) / va.tiles_per_wg;
  }
  aa = {0, rg.gy, 0, rg.log2iw, HEAVY_SPLITS};
  if (!pb.ext_lse) {
    // attention pass: about one workgroup per compute unit, whole tiles per split
    const int nt = (pb.L + TN - 1) / TN;
    auto set_splits = [&](int S) {
      aa.kps = split_tiles(nt, S) * TN;
      aa.S = splits_of(nt, S);
    };
    const int S1 = max(1, min(min(n_cu() / (pb.Hkv * rg.gy), nt), lay.S_max));
    set_splits(S1);
    int chunks = 0;
    if (const int S2 = D == 128 && gram && !rg.ks2 && !pl.vks2 ? share_the_chip(pb, nt, rg.nwr, S1, va, rg.gy, &chunks) : 0) {
      pl.side = true;
      set_splits(S2);
      pl.lo = two_parts(nt, S2, S1);
      aa.heavy = pl.lo ? HEAVY_LO : HEAVY_SIDE;
      va.tiles_per_wg = (ntv + chunks - 1) / chunks;
      va.chunks = (ntv + va.tiles_per_wg - 1) / va.tiles_per_wg;
    }
  }
  // The attention pass first: the value-Gram pass leaves the values in cache for the score pass (8/8 heads of 128, 71k 220 us
  // against 227, 82k 299 / 311; 32/8, window 32, 64k 259 / 263).  Heads of 64 and rows of one split (many heads, whose sums
  // the merge then finds in cache) take it second (64/8 heads of 64, 40k 266 us against 271; 256 KV heads of 2112 tokens
  // 372 / 376).
  va.n = va.chunks * va.ny * pb.Hkv;
  va.at = D == 64 || aa.S <= 1 ? 0 : aa.S * aa.ny * pb.Hkv;
  return pl;
}

template <int D>
int run_mfma(const Prob& pb, const void* q, const void* k, const void* v, const float* gram,
             float* score, char* ws, const ScoreWs& lay, hipStream_t st) {
  const uint16_t* qq = (const uint16_t*)q;
  const uint16_t* kk = (const uint16_t*)k;
  const uint16_t* vp = (const uint16_t*)v;
  const ScorePtrs w = score_ptrs(ws, lay);
  if (pb.ind != 0) gram = nullptr;                 // the attention-weight and value-norm indicators have no projection
  const AttnVvPlan pl = plan_attn_vv<D>(pb, lay, gram != nullptr);
  const RowGeom& rg = pl.rg;
  const AttnArgs aa = pl.aa;
  const VvArgs va = pl.va;
  if (!gram) {
    RK_LAUNCH(ST_VV, st, (k_vnorm2<D>), dim3((pb.P + 255) / 256, pb.Hkv), dim3(256), 0, st, pb, vp,
              w.vv, lay.ldv);
  }
  const dim3 gav(va.n + aa.S * aa.ny * pb.Hkv);
  auto attn_vv = [&](auto a, auto b) {
    RK_LAUNCH(decltype(a)::value ? ST_ATTN : ST_VV, st, (k_attn_vv<D, decltype(a)::value, decltype(b)::value>), gav, dim3(512), 0, st,
              pb, qq, kk, vp, gram, w, aa, va);
  };
  const std::integral_constant<int, 0> no;
  const std::integral_constant<int, 1> plain;
  const std::integral_constant<int, 2> split;
  auto with_vv = [&](auto a) {
    if (!gram) { if constexpr (decltype(a)::value != 0) attn_vv(a, no); }
    else if (pl.vks2) attn_vv(a, split);
    else attn_vv(a, plain);
  };
  const float* part_z = w.part_z;
  auto combine = [&](int S) {
    launch_combine<bf16_t, D, 1>(pb, (const bf16_t*)v, S, gram, w, part_z, (const bf16_t*)q, ilog2(rg.gp), lay.nwb, st);
  };
  if (pb.ext_lse) {
    // the caller's attention output and log-sum-exp stand in for the attention pass: one "split"
    part_z = pb.ext_out;
    combine(1);
    with_vv(no);
  } else {
    if (rg.ks2) {
      with_vv(split);
    } else if (pl.lo) {
      if constexpr (D == 128) attn_vv(std::integral_constant<int, 3>(), plain);
    } else {
      with_vv(plain);
    }
    combine(aa.S);
  }
#define RK_SCORE(GPV) launch_score_pipe<D, GPV>(pb, qq, kk, vp, w, lay.ldv, score, lay.nwb, st)
  switch (rg.gp) {
    case 1: RK_SCORE(1); break;
    case 2: RK_SCORE(2); break;
    case 4: RK_SCORE(4); break;
    case 8: RK_SCORE(8); break;
    case 16: RK_SCORE(16); break;
    case 32: RK_SCORE(32); break;
    default: break;
  }
#undef RK_SCORE
  return hip_status();
}

}  // namespace

bool mfma_eligible(const Prob& pb, const void* q, const void* k, const void* v) {
  if (pb.dtype != RESTKV_BF16) return false;
  if ((((uintptr_t)q | (uintptr_t)k | (uintptr_t)v) & 15u) != 0) return false;
  if ((pb.q_sh | pb.q_st | pb.kv_sh | pb.kv_st) & 7) return false;
  if (pb.G > 32) return false;
  // 32-bit byte offsets inside one head's K/V matrix and inside one group's vv rows
  if ((uint64_t)pb.L * (uint64_t)pb.kv_st * 2u >= (1ull << 32)) return false;
  if ((uint64_t)pb.G * (uint64_t)((pb.P + 3) / 4 * 4) * 4u >= (1ull << 32)) return false;
  if ((uint64_t)(pb.W + 32) * (uint64_t)pb.ld * 4u >= (1ull << 32)) return false;   // one head's score rows
  return true;
}

int score_plan(const Prob& pb, int32_t* plan) {
  if (!mfma_eligible(pb, nullptr, nullptr, nullptr)) return RESTKV_EUNSUPPORTED;
  const ScoreWs lay = score_ws(pb);
  const AttnVvPlan pl = pb.d == 64 ? plan_attn_vv<64>(pb, lay, pb.ind == 0) : plan_attn_vv<128>(pb, lay, pb.ind == 0);
  plan[0] = pl.aa.S;
  plan[1] = pl.aa.kps / TN;
  plan[2] = pl.side;
  plan[3] = pl.lo;
  return RESTKV_OK;
}

int launch_score_mfma(const Prob& pb, const void* q, const void* k, const void* v, const float* gram,
                      float* score, char* ws, const ScoreWs& lay, hipStream_t st) {
  return pb.d == 64 ? run_mfma<64>(pb, q, k, v, gram, score, ws, lay, st)
                    : run_mfma<128>(pb, q, k, v, gram, score, ws, lay, st);
}

}  // namespace restkv

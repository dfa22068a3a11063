// Block-wide top-k searches of rows of floats (gfx950, 64-wide waves).
//
// Rows, or candidates of a row, that fit a block's registers: a histogram over the keys' own range whose
// threshold bin is ranked directly (block_cut).  A long row is bracketed from a sample first (block_bracket), so
// that one streaming pass leaves few candidates.  Where the bracket misses or holds too many, the row
// is searched exactly in global memory: a radix select on the order-preserving integer image of the
// floats (three histogram passes of 11 + 11 + 10 bits), then, in position order, the entries equal to the
// threshold, lowest positions first.
#pragma once

#include <type_traits>

#include "common.hpp"

namespace restkv {

constexpr int SEL_NT = 1024;             // threads per block
constexpr int SEL_NW = SEL_NT / 64;      // wavefronts per block
constexpr int SEL_BINS = 2048;

struct SelectSmem {
  uint32_t hist[SEL_BINS];
  uint32_t wsum[SEL_NW];
  uint32_t cnt_gt[SEL_NW];
  uint32_t cnt_eq[SEL_NW];
  uint32_t bin, below, take;             // results of one digit search
  unsigned long long isum[SEL_NW];
};

// inclusive scan over the block of one value per thread (thread order)
__device__ __forceinline__ uint32_t block_incl_scan(uint32_t x, uint32_t* wsum) {
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) {
    const uint32_t y = __shfl_up(x, o, 64);
    if (lane >= o) x += y;
  }
  __syncthreads();
  if (lane == 63) wsum[w] = x;
  __syncthreads();
  uint32_t base = 0;
  for (int j = 0; j < w; ++j) base += wsum[j];
  return x + base;
}

// number of set bits of `ballot` below this lane
__device__ __forceinline__ uint32_t rank_in_ballot(unsigned long long ballot) {
  const uint32_t lane = threadIdx.x & 63;
  const unsigned long long below = lane ? (ballot & (~0ull >> (64 - lane))) : 0ull;
  return (uint32_t)__popcll(below);
}

// Threshold of the k-th largest (1 <= k <= n): on return `tau` is its key, `n_eq` the number of
// keys equal to it and `k_eq` how many of these belong to the top k (>= 1).  All threads of the
// block must call; all receive the result.
// Any block of 64 .. SEL_NT threads whose size divides SEL_BINS.
// Bound by the latency of the row's loads, eight of which a thread has in flight, and by LDS atomics on
// few bins (keys of one exponent, equal keys): a wavefront adds the entries of its first entry's bin at once.
__device__ inline void block_kth_key(const float* __restrict__ row, int n, int k, SelectSmem& sm,
                                     uint32_t& tau, uint32_t& n_eq, uint32_t& k_eq) {
  uint32_t prefix = 0, mask = 0, krem = (uint32_t)k;
  const int shifts[3] = {21, 10, 0};
  const int nbits[3] = {11, 11, 10};
#pragma unroll
  for (int pass = 0; pass < 3; ++pass) {
    const int sh = shifts[pass];
    const uint32_t nb = 1u << nbits[pass];
    const int nt = (int)blockDim.x, bpt = SEL_BINS / nt;
    for (int b = threadIdx.x; b < SEL_BINS; b += nt) sm.hist[b] = 0;
    __syncthreads();
    for (int x0 = 0; x0 < n; x0 += 8 * nt) {     // (block-uniform: every lane takes part in the ballots)
      float f[8];
#pragma unroll
      for (int u = 0; u < 8; ++u) f[u] = row[min(x0 + u * nt + (int)threadIdx.x, n - 1)];
      uint32_t bin[8];
      unsigned long long all[8], same[8];
      int lead[8];
#pragma unroll
      for (int u = 0; u < 8; ++u) {
        const uint32_t key = float_key(f[u]);
        const bool in = x0 + u * nt + (int)threadIdx.x < n && (key & mask) == prefix;
        bin[u] = in ? (key >> sh) & (nb - 1) : 0xFFFFFFFFu;
        all[u] = __ballot(in);
      }
#pragma unroll
      for (int u = 0; u < 8; ++u) {
        lead[u] = all[u] ? __builtin_ctzll(all[u]) : 0;
        same[u] = __ballot(bin[u] == (uint32_t)__builtin_amdgcn_readlane((int)bin[u], lead[u]));
      }
#pragma unroll
      for (int u = 0; u < 8; ++u) {
        if (all[u] == 0ull) continue;
        if ((int)(threadIdx.x & 63) == lead[u]) atomicAdd(&sm.hist[bin[u]], (uint32_t)__popcll(same[u]));
        else if (((all[u] & ~same[u]) >> (threadIdx.x & 63)) & 1ull) atomicAdd(&sm.hist[bin[u]], 1u);
      }
    }
    __syncthreads();
    // bins in descending order: thread t owns the reversed bins bpt t .. bpt t + bpt - 1
    const int r0 = bpt * (int)threadIdx.x;
    uint32_t own = 0;
    for (int j = 0; j < bpt; ++j) own += r0 + j < (int)nb ? sm.hist[nb - 1 - (r0 + j)] : 0u;
    const uint32_t incl = block_incl_scan(own, sm.wsum);
    uint32_t before = incl - own;
    if (before < krem && krem <= incl) {        // exactly one thread
      for (int j = 0; j < bpt; ++j) {
        const uint32_t hj = r0 + j < (int)nb ? sm.hist[nb - 1 - (r0 + j)] : 0u;
        if (krem <= before + hj) { sm.bin = nb - 1 - (r0 + j); sm.below = before; sm.take = hj; break; }
        before += hj;
      }
    }
    __syncthreads();
    prefix |= sm.bin << sh;
    mask |= (nb - 1) << sh;
    krem -= sm.below;
    n_eq = sm.take;
    __syncthreads();
  }
  tau = prefix;
  k_eq = krem;
}

// Position of the k_eq-th entry (1 <= k_eq <= their number) whose key is tau, in position order: a
// wavefront counts them in its part of the row, the one that has it looks again.  All threads of
// the block must call; all receive the result.
__device__ inline uint32_t block_tie_cut(const float* __restrict__ row, int n, uint32_t tau, uint32_t k_eq, SelectSmem& sm) {
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6, nw = (int)(blockDim.x >> 6);
  const int seg = ((n + nw - 1) / nw + 63) / 64 * 64;
  const int beg = min(n, w * seg), end = min(n, beg + seg);
  auto each = [&](auto f) {                      // f(position of lane 0, ballot of the ties), until it returns false
    for (int x0 = beg; x0 < end; x0 += 512) {
      float v[8];
#pragma unroll
      for (int u = 0; u < 8; ++u) v[u] = row[min(x0 + 64 * u + lane, n - 1)];
#pragma unroll
      for (int u = 0; u < 8; ++u)
        if (!f(x0 + 64 * u, __ballot(x0 + 64 * u + lane < end && float_key(v[u]) == tau))) return;
    }
  };
  uint32_t c = 0;
  each([&](int, unsigned long long b) { c += (uint32_t)__popcll(b); return true; });
  __syncthreads();
  if (lane == 0) sm.cnt_eq[w] = c;
  __syncthreads();
  uint32_t run = 0;
  for (int j = 0; j < w; ++j) run += sm.cnt_eq[j];
  if (run < k_eq && k_eq <= run + c) {           // exactly one wavefront
    each([&](int x0, unsigned long long b) {
      const uint32_t m = (uint32_t)__popcll(b);
      if (run + m < k_eq) { run += m; return true; }
      if (((b >> lane) & 1ull) && rank_in_ballot(b) == k_eq - run - 1u) sm.bin = (uint32_t)(x0 + lane);
      return false;
    });
  }
  __syncthreads();
  return sm.bin;
}

__device__ __forceinline__ float key_float(uint32_t k) {
  return __uint_as_float((k & 0x80000000u) ? (k ^ 0x80000000u) : ~k);
}

constexpr int SEL_NS = 4096;     // samples of the bracketed search

// largest / smallest value of the 64 lanes, in every lane (no LDS traffic)
__device__ __forceinline__ uint32_t wave_max_u(uint32_t x) {
#define RK_ROR(n) x = max(x, (uint32_t)__builtin_amdgcn_update_dpp(0u, x, 0x120 + (n), 0xF, 0xF, false))
  RK_ROR(1); RK_ROR(2); RK_ROR(4); RK_ROR(8);
#undef RK_ROR
  auto r = __builtin_amdgcn_permlane16_swap(x, x, false, false);
  x = max(r[0], r[1]);
  r = __builtin_amdgcn_permlane32_swap(x, x, false, false);
  return max(r[0], r[1]);
}
// inclusive sum over the lanes up to this one
__device__ __forceinline__ uint32_t wave_incl_scan(uint32_t x) {
#define RK_DPP(ctrl, rows) x += __builtin_amdgcn_update_dpp(0u, x, (ctrl), (rows), 0xF, false)
  RK_DPP(0x111, 0xF); RK_DPP(0x112, 0xF); RK_DPP(0x114, 0xF); RK_DPP(0x118, 0xF);   // row_shr 1, 2, 4, 8
  RK_DPP(0x142, 0xA); RK_DPP(0x143, 0xC);                                           // row_bcast 15, 31
#undef RK_DPP
  return x;
}

// ---- selection among keys held in registers ---------------------------------------------------
// A histogram over the keys' own range (2048 bins in LDS, equally wide on the order-preserving
// integer image, i.e. logarithmic with linear pieces in value) finds the bin of the k-th largest
// key; its few members are then ranked one against the other, or the bin is cut again.  Five
// barriers for one round against the ten to twenty of a bisection on the key's bits.
constexpr int CUT_BINS = 2048;
constexpr int CUT_MEMB = 64;
struct CutSmem {
  uint32_t hist[CUT_BINS];
  uint32_t ws[2][SEL_NW];
  uint32_t res[2][3];                    // bin, entries above it, entries in it (per wanted rank)
  uint32_t n;
  uint32_t ck[CUT_MEMB], cp[CUT_MEMB];
};

// a value that is the same in every lane, for the compiler: held in a scalar register from here on
__device__ __forceinline__ uint32_t uniform(uint32_t x) { return (uint32_t)__builtin_amdgcn_readfirstlane((int)x); }

// Smallest and largest key of the block, empty slots (key 0) aside; lo = 0xFFFFFFFF and hi = 0 if
// there is no key.  One barrier; nothing of sm but ws is touched.
template <int NT, int NPT>
__device__ __forceinline__ void block_range(const uint32_t (&key)[NPT], CutSmem& sm, uint32_t& lo, uint32_t& hi) {
  uint32_t nlo = 0u, mx = 0u;            // largest inverted key = smallest key
#pragma unroll
  for (int j = 0; j < NPT; ++j) {
    mx = max(mx, key[j]);
    nlo = key[j] ? max(nlo, ~key[j]) : nlo;
  }
  mx = wave_max_u(mx);
  nlo = wave_max_u(nlo);
  if ((threadIdx.x & 63) == 0) { sm.ws[0][threadIdx.x >> 6] = mx; sm.ws[1][threadIdx.x >> 6] = nlo; }
  __syncthreads();
#pragma unroll
  for (int j = 0; j < NT / 64; ++j) { mx = max(mx, sm.ws[0][j]); nlo = max(nlo, sm.ws[1][j]); }
  // (scalars where vector registers are short: a spill in the 1024 x 16 kernel costs 3 us; rows of 20k and more,
  // with registers to spare, are 0.2 us faster without the two instructions)
  lo = NPT <= 16 ? uniform(~nlo) : ~nlo;
  hi = NPT <= 16 ? uniform(mx) : mx;
}

// width of a bin (log2) that covers [lo, hi] with CUT_BINS of them
__device__ __forceinline__ int cut_shift(uint32_t lo, uint32_t hi) {
  const uint32_t range = hi - lo;
  return range < (uint32_t)CUT_BINS ? 0 : 21 - __builtin_clz(range);
}

// Histogram of val(j), j < NPT, over [lo, hi] (values outside are left out; 0 never counts: lo >= 1),
// then the bins that hold the ranks k[r] (1-based, from the top): res[r], with 0 entries in the bin if
// there is no such rank.  Four barriers, the first of which also separates this from what used sm before.
template <int NT, int NPT, int NR, typename V>
__device__ __forceinline__ void block_bins(V val, uint32_t lo, uint32_t hi, int shift, const uint32_t (&k)[NR],
                                           CutSmem& sm) {
  constexpr int R = CUT_BINS / NT;
  __syncthreads();
#pragma unroll
  for (int i = 0; i < R; ++i) sm.hist[threadIdx.x + i * NT] = 0u;
  if (threadIdx.x == 0) {
    sm.n = 0u;
#pragma unroll
    for (int r = 0; r < NR; ++r) sm.res[r][2] = 0u;
  }
  __syncthreads();
#pragma unroll
  for (int j = 0; j < NPT; ++j) {
    const uint32_t d = val(j) - lo;
    if (d <= hi - lo) atomicAdd(&sm.hist[d >> shift], 1u);
  }
  __syncthreads();
  // thread t owns the bins CUT_BINS - R (t + 1) .. + R - 1: thread order is descending
  const int base = CUT_BINS - R * ((int)threadIdx.x + 1), w = threadIdx.x >> 6;
  uint32_t h[R], own = 0;
#pragma unroll
  for (int i = 0; i < R; ++i) { h[i] = sm.hist[base + i]; own += h[i]; }
  uint32_t incl = wave_incl_scan(own);
  if ((threadIdx.x & 63) == 63) sm.ws[0][w] = incl;
  __syncthreads();
#pragma unroll
  for (int j = 0; j < NT / 64 - 1; ++j) incl += j < w ? sm.ws[0][j] : 0u;
#pragma unroll
  for (int r = 0; r < NR; ++r) {
    uint32_t before = incl - own;
    if (before < k[r] && k[r] <= incl) {           // exactly one thread
#pragma unroll
      for (int i = R - 1; i >= 0; --i) {
        if (before < k[r] && k[r] <= before + h[i]) {
          sm.res[r][0] = (uint32_t)(base + i); sm.res[r][1] = before; sm.res[r][2] = h[i];
        }
        before += h[i];
      }
    }
  }
  __syncthreads();
}

// Cut of the k largest entries: an entry is one of them iff (key, ~position) >= (tau, ~cut), i.e.
// equal keys are taken lowest position first.  key: NPT per thread, 0 where a slot is empty; pos(j):
// position of slot j (below 2^31); every key lies in [lo, hi] (lo >= 1) and there are at least k >= 1
// of them.  False (nothing found) where there are fewer: the caller then searches the row in another way.
// WHOLE: the keys are a whole row of at least k entries (every float is one, whatever its bits) and [lo, hi] is
// their block_range, so that every rank exists and the way out for one that does not, which costs
// the 1024 x 16 kernel two spilled registers, is left out.  Either way each round narrows the range, and
// the search ends.  All NT threads call, all receive the result.  pos gets the thread index as an argument
// that the compiler cannot see through: it would keep NPT positions in registers otherwise.
template <int NT, bool WHOLE, int NPT, typename P>
__device__ __forceinline__ bool block_cut(const uint32_t (&key)[NPT], P pos, uint32_t k, uint32_t lo, uint32_t hi,
                                          CutSmem& sm, uint32_t& tau, uint32_t& cut) {
  bool tie = false;                      // equal keys straddle the cut: the search goes on over inverted positions
  uint32_t tkey = 0;
  for (;;) {                             // (block-uniform; the range shrinks by 2^11 a round)
    int t = threadIdx.x;
    asm volatile("" : "+v"(t));
    auto val = [&](int j) { return tie ? (key[j] == tkey ? ~(uint32_t)pos(j, t) : 0u) : key[j]; };
    const int shift = cut_shift(lo, hi);
    const uint32_t kk[1] = {k};
    if (tie) block_bins<NT, NPT, 1>(val, lo, hi, shift, kk, sm);
    else block_bins<NT, NPT, 1>([&](int j) { return key[j]; }, lo, hi, shift, kk, sm);
    const uint32_t cnt = uniform(sm.res[0][2]);
    if (!WHOLE && cnt == 0u) return false;
    k -= uniform(sm.res[0][1]);
    const uint32_t off = uniform(sm.res[0][0]) << shift;
    hi = lo + off + min(hi - lo - off, (1u << shift) - 1u);      // (no sum that could wrap)
    lo += off;
    if (cnt == k) {                      // the whole bin is taken
      tau = tie ? tkey : lo;
      cut = tie ? ~lo : 0xFFFFFFFFu;
      return true;
    }
    if (cnt <= (uint32_t)CUT_MEMB) {
#pragma unroll
      for (int j = 0; j < NPT; ++j) {
        const uint32_t d = val(j) - lo;
        if (d <= hi - lo) {
          const uint32_t e = atomicAdd(&sm.n, 1u);
          sm.ck[e] = key[j];
          sm.cp[e] = (uint32_t)pos(j, t);
        }
      }
      __syncthreads();
      // every wavefront ranks the members for itself
      const uint32_t l = threadIdx.x & 63;
      const uint32_t mk = l < cnt ? sm.ck[l] : 0u, mp = l < cnt ? sm.cp[l] : 0u;
      const unsigned long long mine = ((unsigned long long)mk << 32) | (unsigned long long)(uint32_t)~mp;
      uint32_t rank = 0;
      for (uint32_t e = 0; e < cnt; ++e) {
        const unsigned long long x = ((unsigned long long)sm.ck[e] << 32) | (unsigned long long)(uint32_t)~sm.cp[e];
        rank += x > mine ? 1u : 0u;
      }
      const int sel = __builtin_ctzll(__ballot(l < cnt && rank == k - 1u));
      tau = (uint32_t)__builtin_amdgcn_readlane((int)mk, sel);
      cut = (uint32_t)__builtin_amdgcn_readlane((int)mp, sel);
      return true;
    }
    bool equal = shift == 0;
    if (NPT <= 16 && !tie && !equal && cnt > 2u * NT) {
      // That many entries in one bin are nearly always equal ones at its lower end (the smallest of the row: scores that
      // underflowed to 0).  The further histograms would be chains of adds to one word: count them.  (512 rows
      // of 16384 scores, 99.9 % zeros: 233 -> 109 us.  Not for any bin that is cut again: 256 heavy-tailed rows of
      // 10k 12.4 -> 16.0 us.  Not with 32 entries per thread, where the longer code costs every row of 20k 2 % and
      // one workgroup fills a compute unit.)
      uint32_t c = 0;
#pragma unroll
      for (int j = 0; j < NPT; ++j) c += (uint32_t)__popcll(__ballot(key[j] == lo));
      if ((threadIdx.x & 63) == 0) atomicAdd(&sm.n, c);
      __syncthreads();
      equal = uniform(sm.n) == cnt;
    }
    if (equal) {                         // more equal keys than members are ranked
      tie = true;
      tkey = lo;
      lo = 0x80000000u;
      hi = 0xFFFFFFFFu;
    }
  }
}
// (key, inverted position) of an entry and of a cut as one comparison.  (The form "key > tau ||
// (key == tau && position <= cut)" is miscompiled by hipcc 7.2 at -O3: the addend of the tie case is dropped.)
__device__ __forceinline__ bool in_cut(uint32_t key, uint32_t pos, uint32_t tau, uint32_t cut) {
  const unsigned long long a = ((unsigned long long)key << 32) | (unsigned long long)(uint32_t)~pos;
  const unsigned long long b = ((unsigned long long)tau << 32) | (unsigned long long)(uint32_t)~cut;
  return a >= b;
}

// One row of floats in the registers of a block of NT threads (NPT each): its keys, 0 past the end.
// VEC (the row 16-byte aligned, readable up to the next multiple of four): quads NT apart.
template <int NT, int NPT, bool VEC>
__device__ __forceinline__ int row_pos(int j, int t) {
  return VEC ? 4 * ((j >> 2) * NT + t) + (j & 3) : j * NT + t;
}
template <int NT, int NPT, bool VEC>
__device__ __forceinline__ void load_row_keys(const float* __restrict__ row, int n, uint32_t (&key)[NPT]) {
  float f[NPT];
  if constexpr (VEC) {
    const int last = (n - 1) & ~3;
#pragma unroll
    for (int q = 0; q < NPT / 4; ++q) {
      const float4 v4 = *(const float4*)(row + min(4 * (q * NT + (int)threadIdx.x), last));
      f[4 * q] = v4.x; f[4 * q + 1] = v4.y; f[4 * q + 2] = v4.z; f[4 * q + 3] = v4.w;
    }
  } else {
#pragma unroll
    for (int j = 0; j < NPT; ++j) f[j] = row[min(j * NT + (int)threadIdx.x, n - 1)];
  }
#pragma unroll
  for (int j = 0; j < NPT; ++j) key[j] = row_pos<NT, NPT, VEC>(j, threadIdx.x) < n ? float_key(f[j]) : 0u;
}
// largest row that load_row_keys is instantiated for, and f(NT, NPT) with the instance for n <= that
constexpr int ROW_REG_MAX = 32768;
template <typename F>
inline void with_row_block(int n, F f) {
  if (n <= 2048) f(std::integral_constant<int, 256>{}, std::integral_constant<int, 8>{});
  else if (n <= 4096) f(std::integral_constant<int, 256>{}, std::integral_constant<int, 16>{});
  else if (n <= 8192) f(std::integral_constant<int, 512>{}, std::integral_constant<int, 16>{});
  else if (n <= 16384) f(std::integral_constant<int, 1024>{}, std::integral_constant<int, 16>{});
  else f(std::integral_constant<int, 1024>{}, std::integral_constant<int, 32>{});
}

// Sample ranks that bracket the k-th largest of a population of n from a sample of ns
// (1-based, descending order): five standard deviations of the hypergeometric rank plus 2.
__device__ __forceinline__ void bracket_ranks(int n, int ns, int k, int& r_hi, int& r_lo) {
  const float f = (float)ns / (float)n;
  const float kp = (float)k * f;
  const int margin = (int)(5.0f * sqrtf(fmaxf(kp * (1.0f - f), 0.f))) + 2;
  r_hi = (int)kp - margin;          // <= 0: no upper bound
  r_lo = (int)kp + 2 + margin;      // > ns: no lower bound
}

// Evenly spread sample of a row of more than NPT * blockDim.x entries in runs of RUN consecutive floats, NPT
// keys per thread.  Returns the sample size.
template <int NPT, int RUN>
__device__ inline int block_sample_regs(const float* __restrict__ row, int n, uint32_t (&k)[NPT]) {
  const int cap = NPT * blockDim.x, nch = cap / RUN;
  const double step = (double)(n - RUN) / (double)(nch - 1);     // no integer division per sample
#pragma unroll
  for (int j = 0; j < NPT; ++j) {
    const int x = threadIdx.x + j * blockDim.x;
    const int c = x / RUN, e = x % RUN;
    const int start = min((int)((double)c * step), n - RUN);
    k[j] = float_key(row[start + e]);
  }
  return cap;
}

// Bracket {klo, khi} (keys) of the k-th largest of row[0..n): the k-th largest key lies in
// (klo, khi] unless the sample misled us.  khi = 0xFFFFFFFF / klo = 0 mean "unbounded".  The bins of
// the two ranks are bracket enough, unless a few outliers stretch the bins until they are wide
// next to the bracket itself: then the range between them is cut again.  (Bins up to 1/32 of it pass:
// log-normal scores need no second cut, which costs 1 us; with 1/64, rows of 40k of them do.  With 1/16,
// rows of 150k scores, four of them 2^60 above the rest, held more than 4096 candidates and were
// searched exactly: smoothing 386 us against 103.)
template <int NT, int NPT, int RUN>
__device__ __forceinline__ void block_bracket(const float* __restrict__ row, int n, int k, CutSmem& sm, uint32_t& klo,
                                              uint32_t& khi) {
  uint32_t keys[NPT];
  const int ns = block_sample_regs<NPT, RUN>(row, n, keys);
  int r_hi, r_lo;
  bracket_ranks(n, ns, k, r_hi, r_lo);
  uint32_t lo, hi;
  block_range<NT>(keys, sm, lo, hi);
  const bool up = r_hi >= 1, dn = r_lo <= ns;
  uint32_t kk[2] = {(uint32_t)max(r_hi, 1), (uint32_t)min(r_lo, ns)};
  for (int round = 0; round < 2; ++round) {
    const int shift = cut_shift(lo, hi);
    block_bins<NT, NPT, 2>([&](int j) { return keys[j]; }, lo, hi, shift, kk, sm);
    const uint32_t off = sm.res[0][0] << shift, bot = lo + (sm.res[1][0] << shift);
    const uint32_t top = lo + off + min(hi - lo - off, (1u << shift) - 1u);
    const uint32_t above = sm.res[0][1];
    hi = top;
    lo = bot;
    if (shift == 0 || (1u << shift) <= ((hi - lo) >> 5)) break;     // (block-uniform)
    kk[0] -= above;
    kk[1] -= above;
  }
  khi = up ? hi : 0xFFFFFFFFu;
  klo = dn ? lo - 1u : 0u;
}

// The bracket (klo, khi] as floats {x, y} for comparisons: "above" is f > y, "inside" is x < f, not
// above.  Comparisons and keys order the same, but for -0 = +0 where the keys of the zeros differ: an
// end between the two moves outwards past both, so that what is counted by comparison and what is
// ranked by key are the same entries.  (A NaN is neither above nor inside.)
__device__ __forceinline__ float2 bracket_ends(uint32_t klo, uint32_t khi) {
  constexpr uint32_t NEG0 = 0x7FFFFFFFu;       // key of -0
  klo = klo == NEG0 ? NEG0 - 1u : klo;
  khi = khi == NEG0 ? NEG0 + 1u : khi;
  return make_float2(klo ? key_float(klo) : -INFINITY, khi != 0xFFFFFFFFu ? key_float(khi) : INFINITY);
}

// Calls f(word index, word) for every 32-bit word of a row of ndw mask words (ndw a multiple of
// 4, the row 16-byte aligned): 16-byte loads, four of them in flight per thread (NT threads).
template <int NT, typename F>
__device__ __forceinline__ void for_each_mask_word(const uint32_t* __restrict__ mrow, int ndw, F f) {
  const int nq = ndw >> 2;
  for (int q0 = 0; q0 < nq; q0 += 4 * NT) {
    uint4 v[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const int q = q0 + u * NT + (int)threadIdx.x;
      v[u] = ((const uint4*)mrow)[min(q, nq - 1)];
    }
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const int q = q0 + u * NT + (int)threadIdx.x;
      if (q < nq) { f(4 * q, v[u].x); f(4 * q + 1, v[u].y); f(4 * q + 2, v[u].z); f(4 * q + 3, v[u].w); }
    }
  }
}

// Visits row[0..n) in position order, wave after wave; f(position, selected_rank)
// is called for every selected element, ranks ascending with position.
// Returns through `sm.cnt_*` nothing the caller needs.
template <typename F>
__device__ inline void block_visit_topk(const float* __restrict__ row, int n, uint32_t tau,
                                        uint32_t k_eq, SelectSmem& sm, F f) {
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6, nw = (int)(blockDim.x >> 6);
  int seg = (n + nw - 1) / nw;
  seg = (seg + 63) / 64 * 64;
  const int beg = min(n, w * seg), end = min(n, beg + seg);
  uint32_t cgt = 0, ceq = 0;
  for (int x0 = beg; x0 < end; x0 += 512) {
    uint32_t kk[8];
#pragma unroll
    for (int u = 0; u < 8; ++u) {
      const int x = x0 + 64 * u + lane;
      kk[u] = x < end ? float_key(row[x]) : 0u;
    }
#pragma unroll
    for (int u = 0; u < 8; ++u) {
      const bool ok = x0 + 64 * u + lane < end;
      cgt += __popcll(__ballot(ok && kk[u] > tau));
      ceq += __popcll(__ballot(ok && kk[u] == tau));
    }
  }
  __syncthreads();
  if (lane == 0) { sm.cnt_gt[w] = cgt; sm.cnt_eq[w] = ceq; }
  __syncthreads();
  uint32_t eq_run = 0, out_run = 0;
  for (int j = 0; j < w; ++j) {
    out_run += sm.cnt_gt[j] + min(sm.cnt_eq[j], k_eq - min(k_eq, eq_run));
    eq_run += sm.cnt_eq[j];
  }
  for (int x0 = beg; x0 < end; x0 += 512) {
    uint32_t kk[8];
#pragma unroll
    for (int u = 0; u < 8; ++u) {
      const int x = x0 + 64 * u + lane;
      kk[u] = x < end ? float_key(row[x]) : 0u;
    }
#pragma unroll
    for (int u = 0; u < 8; ++u) {
      const int x = x0 + 64 * u + lane;
      const bool ok = x < end;
      const bool gt = ok && kk[u] > tau, eq = ok && kk[u] == tau;
      const unsigned long long beq = __ballot(eq);
      const bool take = gt || (eq && eq_run + rank_in_ballot(beq) < k_eq);
      const unsigned long long btk = __ballot(take);
      if (take) f(x, out_run + rank_in_ballot(btk));
      eq_run += __popcll(beq);
      out_run += __popcll(btk);
    }
  }
}

}  // namespace restkv

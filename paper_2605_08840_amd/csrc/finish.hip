// Spatial smoothing, selection and gather of a short layer in one launch (Sec. 3.3, Eq. final_ei and topk).
//
// After the statistics of a short prefix (k_short_rows) three launches are left: box mean, selection, gather.  At these sizes each
// of them is a launch and a chain of round trips with most of the chip idle.  Here every workgroup of a head smooths the head's whole
// row and searches its cut for itself, then gathers its own part of the kept rows.
#include "rowselect.hpp"
#include "window.hpp"

namespace restkv {

namespace {

constexpr int FIN_REACH = 64;        // widest window that the launch takes (its shift is half of that at most)
constexpr int FIN_PAD = FIN_REACH + 2;
constexpr int FIN_ROWS = 64;         // kept rows that a workgroup gathers, at most

// Widest window that the head statistics could ask for: |D_front - D_rear| < P.
bool narrow_window(const Prob& pb) {
  return pb.base_k + (pb.adaptive ? 2.0 * floor((double)pb.P / (double)pb.beta) : 0.0) <= (double)FIN_REACH;
}

// Bound by latency: the head's index sums and smoothed scores (one round trip), the search (five barriers), the gather (a
// second round trip).  The results are those of k_box, k_sel_row and k_compact, bit for bit.  Whole path in three launches and in
// this one, 32/8 heads of 128: 2112 tokens 55.3 -> 48.5 us, two layers 68.4 -> 62.1, four 92.3 -> 86.3, eight 149 -> 146; 4160 tokens 66.8 ->
// 61.8, 8k 85.4 -> 81.7, 16k 120.4 -> 118.6; four float32 heads of 64, 1k 45.5 -> 40.8.
// grid (Hkv, parts), NT threads; a workgroup gathers `rows` kept rows of `cpr` 16-byte chunks each.
template <int NT, int NPT>
__global__ __launch_bounds__(NT, NT == 1024 ? 4 : 1) void k_finish(Prob pb, const float* __restrict__ ema,
                                                                  const unsigned long long* __restrict__ rowsum,
                                                                  float* __restrict__ fin, int32_t* __restrict__ aws_info,
                                                                  double* __restrict__ aws_d, int32_t* __restrict__ idx,
                                                                  const uint4* __restrict__ k, const uint4* __restrict__ v,
                                                                  uint4* __restrict__ k_out, uint4* __restrict__ v_out, int rows,
                                                                  int cpr, int64_t sh16, int64_t st16) {
  constexpr int N = NT * NPT, NWORD = N / 32;
  __shared__ AwsSmem aw;
  __shared__ CutSmem cs;
  __shared__ float tile[N + 2 * FIN_PAD];
  __shared__ uint32_t bits[NWORD];
  __shared__ int sel[FIN_ROWS];
  const int g = blockIdx.x, part = blockIdx.y, tid = threadIdx.x;
  const float* e = ema + (int64_t)g * pb.ld;
  const float pad = pb.pmax ? -INFINITY : 0.f;
  float x[NPT];
#pragma unroll
  for (int j = 0; j < NPT; ++j) x[j] = e[min(j * NT + tid, pb.P - 1)];
  int w_s, gamma;
  head_window<NT>(pb, g, rowsum, part == 0, aws_info, aws_d, aw, w_s, gamma);
#pragma unroll
  for (int j = 0; j < NPT; ++j) tile[FIN_PAD + j * NT + tid] = j * NT + tid < pb.P ? x[j] : pad;
  for (int i = tid; i < FIN_PAD; i += NT) { tile[i] = pad; tile[FIN_PAD + N + i] = pad; }
  __syncthreads();
  // the window's terms lowest index first, as the launch for long rows adds them
  const float* t0 = tile + FIN_PAD + gamma - w_s / 2 + tid;
#pragma unroll
  for (int j = 0; j < NPT; ++j) x[j] = pad;
  if (pb.pmax) {
    for (int u = 0; u < w_s; ++u)
#pragma unroll
      for (int j = 0; j < NPT; ++j) x[j] = fmaxf(x[j], t0[j * NT + u]);
#pragma unroll
    for (int j = 0; j < NPT; ++j) x[j] = x[j] == -INFINITY ? 0.f : x[j];
  } else {
    for (int u = 0; u < w_s; ++u)
#pragma unroll
      for (int j = 0; j < NPT; ++j) x[j] += t0[j * NT + u];
#pragma unroll
    for (int j = 0; j < NPT; ++j) x[j] = x[j] / (float)w_s;
  }
  // every part writes the scores of every parts-th run of NT positions
#pragma unroll
  for (int j = 0; j < NPT; ++j)
    if ((unsigned)j % gridDim.y == (unsigned)part && j * NT + tid < pb.P) fin[(int64_t)g * pb.ld + j * NT + tid] = x[j];

  const int kept = pb.B - pb.W;                      // of the prefix
  const int r0 = part * rows, r1 = min(pb.B, r0 + rows);
  if (kept < pb.P) {
    uint32_t key[NPT], lo, hi, tau, cut;
    auto pos = [](int j, int t) { return j * NT + t; };
#pragma unroll
    for (int j = 0; j < NPT; ++j) key[j] = pos(j, tid) < pb.P ? float_key(x[j]) : 0u;
    block_range<NT>(key, cs, lo, hi);
    block_cut<NT, true>(key, pos, (uint32_t)kept, lo, hi, cs, tau, cut);
#pragma unroll
    for (int j = 0; j < NPT; ++j) {
      const unsigned long long b = __ballot(in_cut(key[j], (uint32_t)pos(j, tid), tau, cut));
      if ((tid & 63) < 2) bits[(j * NT + (tid & ~63)) / 32 + (tid & 63)] = (uint32_t)(b >> (32 * (tid & 63)));
    }
    __syncthreads();
    // ordered list, of which this workgroup keeps its own part
    constexpr int WPT = (NWORD + NT - 1) / NT;
    uint32_t c = 0;
#pragma unroll
    for (int u = 0; u < WPT; ++u) c += tid * WPT + u < NWORD ? (uint32_t)__popc(bits[tid * WPT + u]) : 0u;
    uint32_t at = wave_incl_scan(c);
    if ((tid & 63) == 63) cs.ws[1][tid >> 6] = at;
    __syncthreads();
    at -= c;
    for (int j = 0; j < (tid >> 6); ++j) at += cs.ws[1][j];
#pragma unroll
    for (int u = 0; u < WPT; ++u)
      if (tid * WPT + u < NWORD)
        for (uint32_t m = bits[tid * WPT + u]; m; m &= m - 1) {
          if (at - (uint32_t)r0 < (uint32_t)rows) sel[at - r0] = 32 * (tid * WPT + u) + __builtin_ctz(m);
          ++at;
        }
    for (int r = max(r0, kept) + tid; r < r1; r += NT) sel[r - r0] = pb.P + r - kept;
  } else {
    for (int r = r0 + tid; r < r1; r += NT) sel[r - r0] = r;      // everything is kept, in order
  }
  __syncthreads();
  for (int r = r0 + tid; r < r1; r += NT) idx[(int64_t)g * pb.B + r] = sel[r - r0];
  // four chunks of K and V in flight per thread
  const int n = (r1 - r0) * cpr;
  const uint4 *kg = k + (int64_t)g * sh16, *vg = v + (int64_t)g * sh16;
  const int64_t o0 = ((int64_t)g * pb.B + r0) * cpr;
  for (int c0 = tid; c0 < n; c0 += 4 * NT) {
    uint4 a[4], b[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const int c = min(c0 + u * NT, n - 1);
      const int64_t at = (int64_t)sel[c / cpr] * st16 + c % cpr;
      a[u] = kg[at];
      b[u] = vg[at];
    }
#pragma unroll
    for (int u = 0; u < 4; ++u)
      if (c0 + u * NT < n) { k_out[o0 + c0 + u * NT] = a[u]; v_out[o0 + c0 + u * NT] = b[u]; }
  }
}

}  // namespace

// The search is repeated by every workgroup, so their number times the row may be what the chip does at once (16384 positions a
// compute unit): eight layers of 2112 tokens (2048 workgroups) 149 against 146 us with this launch, 32 layers 431 against 457;
// 8k tokens, four layers 196 against 202.
bool finish_eligible(const Prob& pb, const void* k, const void* v, const void* k_out, const void* v_out) {
  const int per16 = pb.dtype == RESTKV_F32 ? 4 : 8;
  const int64_t parts = (pb.B + FIN_ROWS - 1) / FIN_ROWS;
  return !pb.hb && pb.P <= FINISH_MAX && narrow_window(pb) && parts * pb.Hkv * pb.P <= FINISH_MAX * (int64_t)n_cu() && parts < 65536 &&
         pb.kv_sh % per16 == 0 && pb.kv_st % per16 == 0 &&
         (((uintptr_t)k | (uintptr_t)v | (uintptr_t)k_out | (uintptr_t)v_out) & 15u) == 0;
}

int launch_finish(const Prob& pb, const float* ema, const unsigned long long* rowsum, float* fin, int32_t* aws_info,
                  double* aws_d, int32_t* idx, const void* k, const void* v, void* k_out, void* v_out, hipStream_t st) {
  const int per16 = pb.dtype == RESTKV_F32 ? 4 : 8, cpr = pb.d / per16;
  // as many workgroups as there are compute units, 16 rows or more each
  int rows = FIN_ROWS;
  while (rows > 16 && (int64_t)((pb.B + rows / 2 - 1) / (rows / 2)) * pb.Hkv <= n_cu()) rows /= 2;
  with_row_block(pb.P, [&](auto nt, auto npt) {
    constexpr int NT = decltype(nt)::value, NPT = decltype(npt)::value;
    if constexpr (NT * NPT <= FINISH_MAX)
      RK_LAUNCH(ST_SELECT, st, (k_finish<NT, NPT>), dim3(pb.Hkv, (pb.B + rows - 1) / rows), dim3(NT), 0, st, pb, ema, rowsum, fin,
                aws_info, aws_d, idx, (const uint4*)k, (const uint4*)v, (uint4*)k_out, (uint4*)v_out, rows, cpr, pb.kv_sh / per16,
                pb.kv_st / per16);
  });
  return hip_status();
}

}  // namespace restkv

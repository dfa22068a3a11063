// Per-head selection (Sec. 3.3, Eq. topk): top-(B-W) prefix positions in ascending order,
// window positions appended.
//
// A prefix of at most ROW_REG_MAX positions fits the registers of one workgroup, which does it all
// (k_sel_row).  A longer row is cut into chunks that many workgroups work on in parallel:
//   scan    : per chunk: a sample of the row brackets the threshold of the top-(B-W) (every
//             workgroup of the head repeats this search); count the entries above the bracket;
//             those inside it leave as bit masks
//   emit    : every workgroup of the head finds the exact threshold among the candidates (or by a
//             radix search of the whole row if the bracket missed), counts the selected entries
//             before its own chunks and writes theirs in order
#include <mutex>

#include "rowselect.hpp"

namespace restkv {

namespace {

// Scratch of restkv_select_static: one array per GPU, held until the process ends.  Host code
// never passes the array's name to a kernel: its device address is looked up once per device.
constexpr size_t STATIC_SCRATCH_BYTES = (size_t)4 << 20;
static __device__ __align__(256) unsigned char scratch[STATIC_SCRATCH_BYTES];

constexpr int MAX_DEVICES = 64;
std::mutex g_scratch_mu;
char* g_scratch_ptr[MAX_DEVICES];    // device address of `scratch` on each GPU, nullptr until asked for

// Device address of the current GPU's copy of `scratch` (RESTKV_EHIP if the runtime refuses).
int static_scratch(char** out) {
  int dev = -1;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= MAX_DEVICES) return RESTKV_EHIP;
  std::lock_guard<std::mutex> lk(g_scratch_mu);
  if (!g_scratch_ptr[dev]) {
    void* ptr = nullptr;
    if (hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch)) != hipSuccess || !ptr) return RESTKV_EHIP;
    g_scratch_ptr[dev] = (char*)ptr;
  }
  *out = g_scratch_ptr[dev];
  return RESTKV_OK;
}

constexpr int SCH = 4096;            // positions per chunk = workgroup of the scan (16 per thread)
constexpr int SCAP = 4096;           // candidates the finishing step can take
constexpr int EMIT_WGS = 32;         // workgroups per head of the emission, at most

struct SelPtrs {
  float2* thr;            // [Hkv] bracket of the head's threshold
  uint32_t* above;        // [Hkv, nchunks] entries above the bracket
  uint16_t* cmask;        // [Hkv, nchunks * 256] entries inside the bracket: 16 bits per thread of the scan
};

SelPtrs sel_ptrs(const Prob& pb, char* ws, size_t* bytes) {
  const size_t nch = (size_t)(pb.P + SCH - 1) / SCH;
  size_t off = 0;
  auto take = [&](size_t b) { char* p = ws ? ws + off : nullptr; off = align_up(off + b); return p; };
  SelPtrs w;
  w.thr = (float2*)take((size_t)pb.Hkv * 8);
  w.above = (uint32_t*)take((size_t)pb.Hkv * nch * 4);
  w.cmask = (uint16_t*)take((size_t)pb.Hkv * nch * 512);
  if (bytes) *bytes = off;
  return w;
}

// One head by one workgroup, its row in registers: cut, selected positions as a bit per position in
// LDS, ordered write.  Three launches (scan, finish, emission) took 25.9 us at 2k tokens, 8 heads, and
// 22 us at 1k, 2 heads; this takes 6.3 and 4.2.  At the longest row that fits, 32768 positions, 8 heads:
// 12.3 us, and 14.9 by the two launches for longer rows.  grid (Hkv), NT threads.
template <int NT, int NPT, bool VEC>
__global__ __launch_bounds__(NT, NT == 1024 ? 4 : 1) void k_sel_row(Prob pb, const float* __restrict__ fin,
                                                                   int32_t* __restrict__ idx) {
  constexpr int NWORD = NT * NPT / 32, WPT = (NWORD + NT - 1) / NT;     // words of 32 positions, per thread
  __shared__ CutSmem cs;
  __shared__ uint32_t bits[NWORD];
  const int g = blockIdx.x, tid = threadIdx.x;
  const int bg = head_budget(pb, g), k = bg - pb.W;
  int32_t* out = idx + (int64_t)g * pb.B;
  for (int j = tid; j < pb.W; j += NT) out[k + j] = pb.P + j;
  for (int j = bg + tid; j < pb.B; j += NT) out[j] = -1;       // a smaller per-head budget: unused tail
  if (k >= pb.P) {                                             // everything is kept
    for (int j = tid; j < pb.P; j += NT) out[j] = j;
    return;
  }
  uint32_t key[NPT], lo, hi, tau, cut;
  load_row_keys<NT, NPT, VEC>(fin + (int64_t)g * pb.ld, pb.P, key);
  for (int x = tid; x < NWORD; x += NT) bits[x] = 0u;
  block_range<NT>(key, cs, lo, hi);
  auto pos = [](int j, int t) { return row_pos<NT, NPT, VEC>(j, t); };
  block_cut<NT, true>(key, pos, (uint32_t)k, lo, hi, cs, tau, cut);
#pragma unroll
  for (int j0 = 0; j0 < NPT; j0 += 4) {
    uint32_t m[4];
#pragma unroll
    for (int e = 0; e < 4; ++e) m[e] = in_cut(key[j0 + e], (uint32_t)pos(j0 + e, tid), tau, cut) ? 1u : 0u;
    if constexpr (VEC) {               // four consecutive positions of one word
      const uint32_t q = m[0] | (m[1] << 1) | (m[2] << 2) | (m[3] << 3);
      if (q) atomicOr(&bits[pos(j0, tid) >> 5], q << (pos(j0, tid) & 31));
    } else {
#pragma unroll
      for (int e = 0; e < 4; ++e)
        if (m[e]) atomicOr(&bits[pos(j0 + e, tid) >> 5], 1u << (pos(j0 + e, tid) & 31));
    }
  }
  __syncthreads();
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
      for (uint32_t m = bits[tid * WPT + u]; m; m &= m - 1) out[at++] = 32 * (tid * WPT + u) + __builtin_ctz(m);
}

// Bracket and scan of one chunk of a head's final scores.  Every workgroup of a head first
// brackets the head's top-(B-W) threshold from the same sample of the row (same arithmetic, same
// result: thirty-two workgroups repeating a search that would otherwise leave all but eight
// compute units idle behind a launch of its own), with the loads of its own chunk already in
// flight.  Thread t then owns positions chunk * 4096 + 16 t .. + 15: the entries above the bracket
// are counted (one count per chunk), the entries inside it leave as a 16-bit mask per thread
// (element e at bit 15 - e).  head_grid: parts = chunks, 256 threads.
template <bool BY8>
__global__ __launch_bounds__(256) void k_sel_scan(Prob pb, const float* __restrict__ fin, SelPtrs w,
                                                  int nchunks, int vec) {
  __shared__ CutSmem cs;
  __shared__ uint32_t red[4];
  const HeadPart hp = head_part<BY8>(pb);
  const int g = hp.g, ch = hp.x, tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
  const float* row = fin + (int64_t)g * pb.ld;
  const int n0 = ch * SCH + 16 * tid;
  float x[16];
  if (vec && n0 + 15 < pb.P) {
#pragma unroll
    for (int q4 = 0; q4 < 4; ++q4) {
      const float4 v4 = *(const float4*)(row + n0 + 4 * q4);
      x[4 * q4] = v4.x; x[4 * q4 + 1] = v4.y; x[4 * q4 + 2] = v4.z; x[4 * q4 + 3] = v4.w;
    }
  } else {
#pragma unroll
    for (int e = 0; e < 16; ++e) x[e] = row[min(n0 + e, pb.P - 1)];     // unconditional, masked below
#pragma unroll
    for (int e = 0; e < 16; ++e) x[e] = n0 + e < pb.P ? x[e] : -INFINITY;
  }
  const int k = head_budget(pb, g) - pb.W;
  float2 th = make_float2(INFINITY, INFINITY);          // everything is kept: nothing above, nothing inside
  if (k < pb.P) {                                       // block-uniform
    uint32_t klo, khi;
    block_bracket<256, SEL_NS / 256, 1>(row, pb.P, k, cs, klo, khi);   // smoothed rows: single, spread samples
    th = bracket_ends(klo, khi);
  }
  if (ch == 0 && tid == 0) w.thr[g] = th;
  float tlo = __builtin_bit_cast(float, __builtin_amdgcn_readfirstlane(__builtin_bit_cast(int, th.x)));
  float thi = __builtin_bit_cast(float, __builtin_amdgcn_readfirstlane(__builtin_bit_cast(int, th.y)));
  settle_scalars(tlo, thi);
  uint32_t hb = 0, lb = 0;
#pragma unroll
  for (int e = 0; e < 16; e += 2) shift_in_gt_2x2(hb, lb, x[e], x[e + 1], thi, tlo);
  w.cmask[((int64_t)g * nchunks + ch) * 256 + tid] = (uint16_t)(lb & ~hb);
  const uint32_t c = wave_sum((uint32_t)__popc(hb));
  if (lane == 0) red[wv] = c;
  __syncthreads();
  if (tid == 0) w.above[g * nchunks + ch] = red[0] + red[1] + red[2] + red[3];
}

// Exact threshold of a head and ordered emission.  Every workgroup of the head repeats the search (a
// launch of one workgroup per head that leaves the result for another launch costs more than
// thirty-two workgroups repeating it on compute units that have nothing else to do; 128k tokens, 8
// heads: 16.5 + 15.8 + 4.0 us in three launches, 11.3 + 11.6 in two):
//   * it adds up the chunks' counts, expands the head's masks into candidate positions, fetches
//     their values (at most SCAP) and finds the cut among them;
//   * or, if the bracket missed or holds too many candidates, searches the row exactly (every workgroup
//     of the head on its own: 128k equal scores, 8 heads, 182 us, 400k distinct ones 404; with one
//     workgroup per head and a launch in between, a load in flight per thread, 461 and 463);
//   * the selected entries before its first chunk are the counts above the bracket plus the
//     selected candidates there; from there on it emits its chunks (thread t owns 8 consecutive
//     positions of each).  Window tokens and the unused tail of a smaller per-head budget are
//     written by the first workgroup.
// head_grid: parts = workgroups of a head, 512 threads; workgroup x owns the chunks [x cpw, (x + 1) cpw).
template <bool BY8>
__global__ __launch_bounds__(512) void k_sel_emit(Prob pb, const float* __restrict__ fin, SelPtrs w,
                                                  int nchunks, int cpw, int vec, int32_t* __restrict__ idx) {
  constexpr int NT = 512, NW = NT / 64, FPT = SCAP / NT;
  __shared__ CutSmem cs;
  __shared__ SelectSmem sm;                      // (exact search only)
  __shared__ uint32_t red[2][NW];
  __shared__ uint32_t flag;
  __shared__ int cpos[SCAP];
  const HeadPart hp = head_part<BY8>(pb);
  const int g = hp.g, tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
  const float* row = fin + (int64_t)g * pb.ld;
  const int bg = head_budget(pb, g), k = bg - pb.W;
  int32_t* out = idx + (int64_t)g * pb.B;
  const uint32_t* above = w.above + (int64_t)g * nchunks;
  const int ch0 = hp.x * cpw, ch1 = min(nchunks, ch0 + cpw);
  const uint32_t first = (uint32_t)ch0 * (uint32_t)SCH;         // first position that is this workgroup's
  if (hp.x == 0) {
    for (int j = tid; j < pb.W; j += NT) out[k + j] = pb.P + j;
    for (int j = bg + tid; j < pb.B; j += NT) out[j] = -1;
  }
  uint32_t tau = 0u, cut = 0xFFFFFFFFu, off = first;             // (everything is kept)
  if (k < pb.P) {                                // workgroup-uniform
    const float2 th = w.thr[g];
    // counts above the bracket, in all chunks and in those before, and number of candidates
    const int ndw = nchunks * 128;               // two threads of the scan per 32-bit word
    const uint32_t* mrow = (const uint32_t*)(w.cmask + (int64_t)g * nchunks * 256);
    uint32_t c_mine = 0, a_mine = 0, b_mine = 0;
    for_each_mask_word<NT>(mrow, ndw, [&](int, uint32_t m) { c_mine += (uint32_t)__popc(m); });
    for (int c = tid; c < nchunks; c += NT) { const uint32_t a = above[c]; a_mine += a; b_mine += c < ch0 ? a : 0u; }
    const uint32_t incl = block_incl_scan(c_mine, sm.wsum);
    a_mine = wave_sum(a_mine);
    b_mine = wave_sum(b_mine);
    if (lane == 0) { red[0][wv] = a_mine; red[1][wv] = b_mine; }
    if (tid == NT - 1) flag = incl;
    __syncthreads();
    const uint32_t nc = flag;
    uint32_t n_above = 0, n_before = 0;
#pragma unroll
    for (int j = 0; j < NW; ++j) { n_above += red[0][j]; n_before += red[1][j]; }
    uint32_t sel_before = 0;                     // this thread's share of the selected candidates before `first`
    bool found = n_above < (uint32_t)k && (uint32_t)k <= n_above + nc && nc <= (uint32_t)SCAP;      // workgroup-uniform
    if (found) {
      uint32_t slot = incl - c_mine;
      for_each_mask_word<NT>(mrow, ndw, [&](int x, uint32_t m) {
        while (m) {
          const int b = __builtin_ctz(m);
          m &= m - 1;
          cpos[slot++] = 16 * (2 * x + (b >> 4)) + 15 - (b & 15);  // half word = thread of the scan, bit 15 - e = element e
        }
      });
      __syncthreads();
      uint32_t ck[FPT];
      float fv[FPT];
      int iv[FPT];
#pragma unroll
      for (int j = 0; j < FPT; ++j) {            // unconditional loads, masked afterwards: all in flight at once
        const uint32_t x = tid + j * NT;
        iv[j] = cpos[x < nc ? x : 0u];
        fv[j] = row[iv[j]];
      }
#pragma unroll
      for (int j = 0; j < FPT; ++j) ck[j] = (uint32_t)(tid + j * NT) < nc ? float_key(fv[j]) : 0u;
      // every candidate lies inside the bracket (th.x, th.y]
      found = block_cut<NT, false>(ck, [&](int j, int) { return iv[j]; }, (uint32_t)k - n_above, float_key(th.x) + 1u, float_key(th.y), cs, tau, cut);
#pragma unroll
      for (int j = 0; j < FPT; ++j)
        sel_before += ck[j] && (uint32_t)iv[j] < first && in_cut(ck[j], (uint32_t)iv[j], tau, cut) ? 1u : 0u;
    }
    if (!found) {
      // exact search of the whole row: threshold, the last tie that is taken, and a count of the
      // selected entries before this workgroup's
      uint32_t n_eq, k_eq;
      block_kth_key(row, pb.P, k, sm, tau, n_eq, k_eq);
      cut = k_eq < n_eq ? block_tie_cut(row, pb.P, tau, k_eq, sm) : 0xFFFFFFFFu;
      sel_before = 0;
      for (uint32_t x0 = tid; x0 < first; x0 += 8u * NT) {
        float f[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) f[u] = row[min(x0 + (uint32_t)(u * NT), first - 1u)];
#pragma unroll
        for (int u = 0; u < 8; ++u)
          sel_before += x0 + (uint32_t)(u * NT) < first && in_cut(float_key(f[u]), x0 + (uint32_t)(u * NT), tau, cut) ? 1u : 0u;
      }
      n_before = 0;                              // (every entry has been counted)
    }
    __syncthreads();
    sel_before = wave_sum(sel_before);
    if (lane == 0) red[0][wv] = sel_before;
    __syncthreads();
    off = n_before;
#pragma unroll
    for (int j = 0; j < NW; ++j) off += red[0][j];
  }
  for (int ch = ch0; ch < ch1; ++ch) {
    const int n0 = ch * SCH + tid * (SCH / NT);
    float x[SCH / NT];
    if (vec && n0 + SCH / NT - 1 < pb.P) {
#pragma unroll
      for (int q4 = 0; q4 < SCH / NT / 4; ++q4) {
        const float4 v4 = *(const float4*)(row + n0 + 4 * q4);
        x[4 * q4] = v4.x; x[4 * q4 + 1] = v4.y; x[4 * q4 + 2] = v4.z; x[4 * q4 + 3] = v4.w;
      }
    } else {
#pragma unroll
      for (int e = 0; e < SCH / NT; ++e) x[e] = row[min(n0 + e, pb.P - 1)];
    }
    uint32_t mask = 0;
#pragma unroll
    for (int e = 0; e < SCH / NT; ++e)
      if (n0 + e < pb.P && in_cut(float_key(x[e]), (uint32_t)(n0 + e), tau, cut)) mask |= 1u << e;
    const uint32_t c = (uint32_t)__popc(mask);
    const uint32_t incl = wave_incl_scan(c);
    __syncthreads();
    if (lane == 63) red[1][wv] = incl;
    __syncthreads();
    uint32_t at = off + incl - c;
    for (int j = 0; j < NW; ++j) {
      const uint32_t r = red[1][j];
      at += j < wv ? r : 0u;
      off += r;
    }
    for (uint32_t m = mask; m; m &= m - 1) {
      if (at < (uint32_t)k) out[at] = n0 + __builtin_ctz(m);
      ++at;
    }
  }
}

}  // namespace

size_t select_ws_bytes(const Prob& pb) {
  size_t n = 0;
  sel_ptrs(pb, nullptr, &n);
  return n;
}

int launch_select(const Prob& pb, const float* fin, int32_t* idx, char* ws, hipStream_t st) {
  const bool vec = (pb.ld & 3) == 0 && ((uintptr_t)fin & 15u) == 0;
  if (pb.P <= ROW_REG_MAX) {
    with_row_block(pb.P, [&](auto nt, auto npt) {
      constexpr int NT = decltype(nt)::value, NPT = decltype(npt)::value;
      if (vec) RK_LAUNCH(ST_SELECT, st, (k_sel_row<NT, NPT, true>), dim3(pb.Hkv), dim3(NT), 0, st, pb, fin, idx);
      else RK_LAUNCH(ST_SELECT, st, (k_sel_row<NT, NPT, false>), dim3(pb.Hkv), dim3(NT), 0, st, pb, fin, idx);
    });
    return hip_status();
  }
  const int nch = (pb.P + SCH - 1) / SCH;
  const SelPtrs w = sel_ptrs(pb, ws, nullptr);
  const int cpw = (nch + EMIT_WGS - 1) / EMIT_WGS;
  by_heads(pb, [&](auto by8) {
    constexpr bool BY8 = decltype(by8)::value;
    RK_LAUNCH(ST_SELECT, st, k_sel_scan<BY8>, head_grid(pb, nch), dim3(256), 0, st, pb, fin, w, nch, vec ? 1 : 0);
    RK_LAUNCH(ST_SELECT, st, k_sel_emit<BY8>, head_grid(pb, (nch + cpw - 1) / cpw), dim3(512), 0, st, pb, fin, w, nch, cpw, vec ? 1 : 0, idx);
  });
  return hip_status();
}

size_t select_static_capacity() { return STATIC_SCRATCH_BYTES; }

int launch_select_static(const Prob& pb, const float* fin, int32_t* idx, hipStream_t st) {
  if (select_ws_bytes(pb) > STATIC_SCRATCH_BYTES) return RESTKV_EWORKSPACE;
  char* ws = nullptr;
  const int rc = static_scratch(&ws);
  if (rc) return rc;
  return launch_select(pb, fin, idx, ws, st);
}

}  // namespace restkv

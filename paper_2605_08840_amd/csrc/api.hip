// C ABI of the ReST-KV eviction library: argument validation, scratch layout, dispatch.
// Everything behind these entry points is a hand-written HIP kernel for gfx950.
#include <math.h>

#include <algorithm>

#include "score_common.hpp"

namespace restkv {

int resolve(const restkv_params* p, Prob* o) {
  if (!p || !o) return RESTKV_EINVAL;
  if (p->n_q_heads <= 0 || p->n_kv_heads <= 0 || p->n_q_heads % p->n_kv_heads) return RESTKV_EINVAL;
  if (p->seq_len < 2 || p->window < 1 || p->window >= p->seq_len) return RESTKV_EINVAL;
  if (p->budget <= p->window || p->budget > p->seq_len) return RESTKV_EINVAL;
  if (p->base_window < 1 || !(p->base_window & 1)) return RESTKV_EINVAL;
  if (p->variant & ~0x77) return RESTKV_EINVAL;
  if ((p->variant & 3) == 3 || ((p->variant >> 4) & 3) == 3) return RESTKV_EINVAL;
  if (!(p->ema_alpha >= 0.f && p->ema_alpha <= 1.f)) return RESTKV_EINVAL;
  if (p->adaptive && !(p->beta > 0.f)) return RESTKV_EINVAL;
  // |D_front - D_rear| < L, so floor(|x| / beta) stays a 32-bit integer with room to spare
  if (p->adaptive && (double)p->seq_len / (double)p->beta >= 1073741824.0) return RESTKV_EINVAL;
  if (!(p->scale >= 0.f) || isinf(p->scale)) return RESTKV_EINVAL;
  if (p->head_dim != 64 && p->head_dim != 128) return RESTKV_EUNSUPPORTED;
  if (p->dtype != RESTKV_F32 && p->dtype != RESTKV_BF16) return RESTKV_EUNSUPPORTED;
  o->Hq = p->n_q_heads; o->Hkv = p->n_kv_heads; o->G = o->Hq / o->Hkv;
  o->d = p->head_dim; o->L = p->seq_len; o->W = p->window; o->P = o->L - o->W;
  o->B = p->budget; o->R = o->G * o->W; o->hb = nullptr; o->ext_out = nullptr; o->ext_lse = nullptr;
  if ((int64_t)o->G * o->W > 4096) return RESTKV_EUNSUPPORTED;
  o->dtype = p->dtype; o->causal = p->causal ? 1 : 0; o->base_k = p->base_window;
  o->ind = p->variant & 3; o->gmax = (p->variant >> 2) & 1; o->tmode = (p->variant >> 4) & 3;
  o->pmax = (p->variant >> 6) & 1;
  o->adaptive = (p->adaptive && o->W >= 2) ? 1 : 0;
  o->scale = p->scale > 0.f ? p->scale : 1.0f / sqrtf((float)o->d);
  o->alpha = p->ema_alpha; o->beta = p->beta;
  o->q_st = p->q_stride_t ? p->q_stride_t : o->d;
  o->q_sh = p->q_stride_h ? p->q_stride_h : (int64_t)o->W * o->d;
  o->kv_st = p->kv_stride_t ? p->kv_stride_t : o->d;
  o->kv_sh = p->kv_stride_h ? p->kv_stride_h : (int64_t)o->L * o->d;
  o->ld = p->ld_score ? p->ld_score : o->P;
  if (o->q_st < o->d || o->kv_st < o->d || o->q_sh < 0 || o->kv_sh < 0 || o->ld < o->P) return RESTKV_EINVAL;
  return RESTKV_OK;
}

ScoreWs score_ws(const Prob& pb) {
  ScoreWs w;
  w.S_max = 64;
  const int S = w.S_max;
  w.ldv = (pb.P + 3) / 4 * 4;
  const size_t rows = (size_t)pb.Hq * pb.W;
  size_t off = 0;
  auto take = [&](size_t bytes) { size_t o = off; off = align_up(off + bytes); return o; };
  w.part_m = take(rows * S * 4);
  w.part_mx = take(rows * S * 4);
  w.part_n = take(rows * S * 4);
  w.part_ref = take(rows * S * 4);
  w.part_l = take(rows * S * 4);
  w.part_z = take(rows * S * (size_t)pb.d * 4);
  w.rs_m = take(rows * 4);
  w.rs_l = take(rows * 4);
  w.rs_zz = take(rows * 4);
  w.rs_nstar = take(rows * 4);
  w.rs_istar = take(rows * 4);
  w.vv = take((size_t)pb.Hq * w.ldv * 4);
  // operand-ordered copies for the matrix-core path: 32-row blocks hold Gp (power of two >= G)
  // heads of 32/Gp window positions
  w.nwb = 0;
  if (pb.G <= 32) {
    int gp = 1;
    while (gp < pb.G) gp <<= 1;
    const int iw = 32 / gp;
    w.nwb = (pb.W + iw - 1) / iw;
  }
  // (the FP32 path leaves q and u of every head in planes there instead)
  w.op = take(std::max((size_t)3 * pb.Hkv * w.nwb * 32 * pb.d * 2, (size_t)pb.Hq * row_items(pb.W) * 2 * row_item(pb.d)));
  w.bytes = off;
  return w;
}

SmoothWs smooth_ws(const Prob& pb) {
  SmoothWs w;
  size_t off = 0;
  auto take = [&](size_t bytes) { size_t o = off; off = align_up(off + bytes); return o; };
  w.rowsum = take((size_t)pb.Hkv * pb.W * 8);
  w.ema = take((size_t)pb.Hkv * pb.ld * 4);
  const size_t rows = (size_t)pb.Hkv * pb.W;
  w.thr = take(rows * 8);
  w.cnt_hi = take(rows * 4);
  w.sum_hi = take(rows * 8);
  w.cmask = take(rows * (size_t)((pb.P + 1023) / 1024) * 64 * 2);
  w.bytes = off;
  return w;
}

// compute units of the current device (queried once)
int n_cu() {
  static int n = 0;
  if (n == 0) {
    int dev = 0, v = 0;
    if (hipGetDevice(&dev) == hipSuccess &&
        hipDeviceGetAttribute(&v, hipDeviceAttributeMultiprocessorCount, dev) == hipSuccess && v > 0)
      n = v;
    else
      n = 256;
  }
  return n;
}

static bool g_force_fp32 = false;   // see restkv_debug_force_fp32

static int check_ws(const void* ws, size_t have, size_t need) {
  if (!ws || ((uintptr_t)ws & 255u) || have < need) return RESTKV_EWORKSPACE;
  return RESTKV_OK;
}

}  // namespace restkv

using namespace restkv;

extern "C" {

size_t restkv_workspace_bytes(const restkv_params* p) {
  Prob pb;
  if (resolve(p, &pb) != RESTKV_OK) return 0;
  size_t n = score_ws(pb).bytes;
  if (smooth_ws(pb).bytes > n) n = smooth_ws(pb).bytes;
  if (select_ws_bytes(pb) > n) n = select_ws_bytes(pb);
  return n;
}

int restkv_prepare_wo(const restkv_params* p, const float* w_o, int64_t d_model, float* gram,
                      restkv_stream_t stream) {
  Prob pb;
  int rc = resolve(p, &pb);
  if (rc) return rc;
  if (!w_o || !gram || d_model < 1) return RESTKV_EINVAL;
  return launch_gram(pb, w_o, d_model, gram, (hipStream_t)stream);
}

int restkv_score(const restkv_params* p, const void* q, const void* k, const void* v,
                 const float* gram, float* score, void* workspace, size_t workspace_bytes,
                 restkv_stream_t stream) {
  Prob pb;
  int rc = resolve(p, &pb);
  if (rc) return rc;
  if (!q || !k || !v || !score) return RESTKV_EINVAL;
  const ScoreWs lay = score_ws(pb);
  rc = check_ws(workspace, workspace_bytes, lay.bytes);
  if (rc) return rc;
  if (mfma_eligible(pb, q, k, v) && !g_force_fp32)
    return launch_score_mfma(pb, q, k, v, gram, score, (char*)workspace, lay, (hipStream_t)stream);
  return launch_score_simple(pb, q, k, v, gram, score, (char*)workspace, lay, (hipStream_t)stream);
}

int restkv_score_from_attention(const restkv_params* p, const void* q, const void* k, const void* v,
                                const float* gram, const float* attn_out, const float* lse, float* score,
                                void* workspace, size_t workspace_bytes, restkv_stream_t stream) {
  Prob pb;
  int rc = resolve(p, &pb);
  if (rc) return rc;
  if (!q || !k || !v || !score || !attn_out || !lse) return RESTKV_EINVAL;
  pb.ext_out = attn_out;
  pb.ext_lse = lse;
  const ScoreWs lay = score_ws(pb);
  rc = check_ws(workspace, workspace_bytes, lay.bytes);
  if (rc) return rc;
  if (mfma_eligible(pb, q, k, v) && !g_force_fp32)
    return launch_score_mfma(pb, q, k, v, gram, score, (char*)workspace, lay, (hipStream_t)stream);
  return launch_score_simple(pb, q, k, v, gram, score, (char*)workspace, lay, (hipStream_t)stream);
}

static int smooth_impl(const restkv_params* p, const float* score, const int32_t* head_budget, float* ema,
                       float* final_score, int32_t* aws_info, double* aws_d, void* workspace,
                       size_t workspace_bytes, restkv_stream_t stream) {
  Prob pb;
  int rc = resolve(p, &pb);
  if (rc) return rc;
  if (!score || !final_score) return RESTKV_EINVAL;
  pb.hb = head_budget;
  const SmoothWs lay = smooth_ws(pb);
  rc = check_ws(workspace, workspace_bytes, lay.bytes);
  if (rc) return rc;
  return launch_smooth(pb, score, ema, final_score, aws_info, aws_d, (char*)workspace, lay,
                       (hipStream_t)stream);
}

int restkv_smooth(const restkv_params* p, const float* score, float* ema, float* final_score,
                  int32_t* aws_info, double* aws_d, void* workspace, size_t workspace_bytes,
                  restkv_stream_t stream) {
  return smooth_impl(p, score, nullptr, ema, final_score, aws_info, aws_d, workspace, workspace_bytes, stream);
}

int restkv_smooth_b(const restkv_params* p, const float* score, const int32_t* head_budget, float* ema,
                    float* final_score, int32_t* aws_info, double* aws_d, void* workspace,
                    size_t workspace_bytes, restkv_stream_t stream) {
  if (!head_budget) return RESTKV_EINVAL;
  return smooth_impl(p, score, head_budget, ema, final_score, aws_info, aws_d, workspace, workspace_bytes, stream);
}

int restkv_score_smooth(const restkv_params* p, const void* q, const void* k, const void* v,
                        const float* gram, float* score, float* ema, float* final_score,
                        int32_t* aws_info, double* aws_d, void* workspace, size_t workspace_bytes,
                        restkv_stream_t stream) {
  Prob pb;
  int rc = resolve(p, &pb);
  if (rc) return rc;
  if (!q || !k || !v || !score || !final_score) return RESTKV_EINVAL;
  // Both sizes are checked first so that nothing is enqueued when the second call would fail.  The two
  // use the workspace one after the other.
  const size_t a = score_ws(pb).bytes, b = smooth_ws(pb).bytes;
  rc = check_ws(workspace, workspace_bytes, a > b ? a : b);
  if (rc) return rc;
  // A score pass that accumulated the smoothing itself (temporal sums and top-B statistics against
  // brackets from a sampled pass, prefixes from 32k on) was slower at every size it took: 32/8 heads
  // of 128, window 64: 269 against 213 us at 32k tokens, 407 against 347 at 64k, 697 against 645 at
  // 128k; 64/8 heads at 128k 789 against 730.  Its vector work costs more than the read it saves.
  rc = restkv_score(p, q, k, v, gram, score, workspace, workspace_bytes, stream);
  if (rc) return rc;
  return restkv_smooth(p, score, ema, final_score, aws_info, aws_d, workspace, workspace_bytes, stream);
}

static int select_impl(const restkv_params* p, const float* final_score, const int32_t* head_budget,
                       int32_t* idx, void* workspace, size_t workspace_bytes, restkv_stream_t stream) {
  Prob pb;
  int rc = resolve(p, &pb);
  if (rc) return rc;
  if (!final_score || !idx) return RESTKV_EINVAL;
  pb.hb = head_budget;
  rc = check_ws(workspace, workspace_bytes, select_ws_bytes(pb));
  if (rc) return rc;
  return launch_select(pb, final_score, idx, (char*)workspace, (hipStream_t)stream);
}

int restkv_select(const restkv_params* p, const float* final_score, int32_t* idx, void* workspace,
                  size_t workspace_bytes, restkv_stream_t stream) {
  return select_impl(p, final_score, nullptr, idx, workspace, workspace_bytes, stream);
}

int restkv_select_b(const restkv_params* p, const float* final_score, const int32_t* head_budget,
                    int32_t* idx, void* workspace, size_t workspace_bytes, restkv_stream_t stream) {
  if (!head_budget) return RESTKV_EINVAL;
  return select_impl(p, final_score, head_budget, idx, workspace, workspace_bytes, stream);
}

int restkv_select_static(const restkv_params* p, const float* final_score, int32_t* idx,
                         restkv_stream_t stream) {
  Prob pb;
  int rc = resolve(p, &pb);
  if (rc) return rc;
  if (!final_score || !idx) return RESTKV_EINVAL;
  return launch_select_static(pb, final_score, idx, (hipStream_t)stream);
}

size_t restkv_select_static_capacity(void) { return select_static_capacity(); }

int restkv_compact(const restkv_params* p, const void* k, const void* v, const int32_t* idx,
                   void* k_out, void* v_out, restkv_stream_t stream) {
  Prob pb;
  int rc = resolve(p, &pb);
  if (rc) return rc;
  if (!k || !v || !idx || !k_out || !v_out) return RESTKV_EINVAL;
  return launch_compact(pb, k, v, idx, k_out, v_out, (hipStream_t)stream);
}

int restkv_evict(const restkv_params* p, const void* q, const void* k, const void* v, const float* gram, float* score,
                 float* ema, float* final_score, int32_t* aws_info, double* aws_d, int32_t* idx, void* k_out, void* v_out,
                 void* workspace, size_t workspace_bytes, restkv_stream_t stream) {
  Prob pb;
  int rc = resolve(p, &pb);
  if (rc) return rc;
  if (!q || !k || !v || !score || !final_score || !idx || !k_out || !v_out) return RESTKV_EINVAL;
  // (all sizes first, so that nothing is enqueued when a later stage would fail; the stages use the workspace one after the other)
  const SmoothWs lay = smooth_ws(pb);
  rc = check_ws(workspace, workspace_bytes, std::max(std::max(score_ws(pb).bytes, lay.bytes), select_ws_bytes(pb)));
  if (rc) return rc;
  rc = restkv_score(p, q, k, v, gram, score, workspace, workspace_bytes, stream);
  if (rc) return rc;
  if (short_rows(pb) && finish_eligible(pb, k, v, k_out, v_out)) {
    unsigned long long* rowsum = (unsigned long long*)((char*)workspace + lay.rowsum);
    float* e = ema ? ema : (float*)((char*)workspace + lay.ema);
    launch_short_rows(pb, score, e, rowsum, (hipStream_t)stream);
    return launch_finish(pb, e, rowsum, final_score, aws_info, aws_d, idx, k, v, k_out, v_out, (hipStream_t)stream);
  }
  rc = restkv_smooth(p, score, ema, final_score, aws_info, aws_d, workspace, workspace_bytes, stream);
  if (!rc) rc = restkv_select(p, final_score, idx, workspace, workspace_bytes, stream);
  if (!rc) rc = restkv_compact(p, k, v, idx, k_out, v_out, stream);
  return rc;
}

const char* restkv_strerror(int code) {
  switch (code) {
    case RESTKV_OK: return "ok";
    case RESTKV_EINVAL: return "invalid argument (null pointer, inconsistent shape or budget outside (W, L])";
    case RESTKV_EUNSUPPORTED: return "unsupported configuration (head_dim must be 64 or 128; dtype f32 or bf16)";
    case RESTKV_EWORKSPACE: return "workspace missing, not 256-byte aligned or smaller than restkv_workspace_bytes() (restkv_select_static: the problem needs more than the library's static scratch)";
    case RESTKV_EHIP: return "HIP runtime error at kernel launch";
    default: return "unknown error code";
  }
}

int restkv_version(void) { return 100; }

int restkv_debug_force_fp32(int on) {
  g_force_fp32 = on != 0;
  return RESTKV_OK;
}

int restkv_debug_score_plan(const restkv_params* p, int32_t* plan) {
  Prob pb;
  int rc = resolve(p, &pb);
  if (rc) return rc;
  if (!plan) return RESTKV_EINVAL;
  return score_plan(pb, plan);
}

int restkv_debug_fp32_plan(const restkv_params* p, int32_t* plan) {
  Prob pb;
  int rc = resolve(p, &pb);
  if (rc) return rc;
  if (!plan) return RESTKV_EINVAL;
  return fp32_plan(pb, plan);
}

}  // extern "C"

// Adaptive window of a KV head (Sec. 3.3): size and shift of the spatial smoothing from the drift of the per-query top-B
// positions.
#pragma once

#include "common.hpp"

namespace restkv {

// Window size and shift from the drift statistic (device function so that every block of
// the box kernel derives the same integers without a host round trip).
// (front and rear index sums come in already added up)
__device__ inline void aws_window(const Prob& pb, unsigned long long sf, unsigned long long sr, int g,
                                  int& w_s, int& gamma, double& d_front, double& d_rear) {
  w_s = pb.base_k; gamma = 0; d_front = 0.0; d_rear = 0.0;
  if (!pb.adaptive) return;
  const int nf = pb.W / 2;
  const double bt = (double)min(head_budget(pb, g), pb.P);
  d_front = (double)sf / (bt * (double)nf);
  d_rear = (double)sr / (bt * (double)(pb.W - nf));
  const double x = d_front - d_rear;
  const double beta = (double)pb.beta;
  w_s = pb.base_k + 2 * (int)floor(fabs(x) / beta);
  const int f = (int)floor(x / beta);
  gamma = x > 0.0 ? f : f + 1;
}

struct AwsSmem {
  alignas(16) unsigned long long sum[2][16];
  int w_s, gamma;
};
// Window of head g from the index sums of its W queries, for every thread of the block: all loads in flight at once, wavefront
// sums, then thread 0, which also writes them out where `leave` says so.  Two barriers.
template <int NT>
__device__ __forceinline__ void head_window(const Prob& pb, int g, const unsigned long long* __restrict__ rowsum, bool leave,
                                            int32_t* __restrict__ aws_info, double* __restrict__ aws_d, AwsSmem& sm, int& w_s,
                                            int& gamma) {
  unsigned long long sf = 0, sr = 0;
  if (pb.adaptive)
    for (int i = threadIdx.x; i < pb.W; i += NT) {
      const unsigned long long s = rowsum[g * pb.W + i];
      if (i < pb.W / 2) sf += s; else sr += s;
    }
#pragma unroll
  for (int o = 32; o >= 1; o >>= 1) { sf += __shfl_xor(sf, o, 64); sr += __shfl_xor(sr, o, 64); }
  if ((threadIdx.x & 63) == 0) { sm.sum[0][threadIdx.x >> 6] = sf; sm.sum[1][threadIdx.x >> 6] = sr; }
  __syncthreads();
  if (threadIdx.x == 0) {
    sf = sr = 0;
#pragma unroll
    for (int j = 0; j < NT / 64; ++j) { sf += sm.sum[0][j]; sr += sm.sum[1][j]; }
    int w_s0, gamma0;
    double df, dr;
    aws_window(pb, sf, sr, g, w_s0, gamma0, df, dr);
    sm.w_s = w_s0; sm.gamma = gamma0;
    if (leave) {
      if (aws_info) { aws_info[2 * g] = w_s0; aws_info[2 * g + 1] = gamma0; }
      if (aws_d) { aws_d[2 * g] = df; aws_d[2 * g + 1] = dr; }
    }
  }
  __syncthreads();
  w_s = sm.w_s; gamma = sm.gamma;
}

}  // namespace restkv

// Stage I pruning and the ordering of Eq. 3-9: per image, the tokens by descending score, equal scores by ascending
// index; the first k_prune are written out.
#include "tc_internal.h"

namespace tc {

// The place of a token is the number of tokens that precede it.  One workgroup counts for 64 tokens against all N keys in
// LDS, each of its four wavefronts for a quarter of them: N^2 comparisons, but spread over the chip and without a barrier
// per step (a bitonic sort by one workgroup per image is log^2 N of them: 55 at 576 tokens; 30 -> 5 us for one image, 31 -> 6 for
// 64, 93 -> 15 for 8 of 2880 tokens).
__global__ __launch_bounds__(256) void topk_kernel(const float* __restrict__ E, int32_t* __restrict__ order, int N, int kp) {
  extern __shared__ __attribute__((aligned(16))) unsigned long long keys[];  // round_up(N, 8)
  typedef __attribute__((ext_vector_type(2))) unsigned long long k2;
  __shared__ int part[4][64];
  const int b = blockIdx.y, tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int n8 = round_up(N, 8);
  for (int i = tid; i < n8; i += 256) {
    float v = i < N ? E[(size_t)b * N + i] : 0.f;
    if (v != v) v = -INFINITY;  // NaN scores rank last
    keys[i] = i < N ? order_key(v, i) : 0ull;  // (zero precedes nobody)
  }
  __syncthreads();
  const int x = blockIdx.x * 64 + lane;
  const unsigned long long mine = keys[min(x, N - 1)];
  const int per = (n8 / 2 + 3) / 4, e0 = wave * per, e1 = min(n8 / 2, e0 + per);
  const k2* kk = reinterpret_cast<const k2*>(keys);
  int rank = 0;
#pragma unroll 8
  for (int e = e0; e < e1; e++) {
    const k2 v = kk[e];
    rank += (v.x > mine ? 1 : 0) + (v.y > mine ? 1 : 0);
  }
  part[wave][lane] = rank;
  __syncthreads();
  if (wave == 0 && x < N) {
    rank = (part[0][lane] + part[1][lane]) + (part[2][lane] + part[3][lane]);
    if (rank < kp) order[(size_t)b * kp + rank] = x;
  }
}

int launch_topk(const Plan& pl, const float* E, int32_t* order, hipStream_t st) {
  TC_TIMED(PK_TOPK, 0, st, (topk_kernel<<<dim3((pl.N + 63) / 64, pl.B), 256, (size_t)round_up(pl.N, 8) * 8, st>>>(E, order, pl.N, pl.kp)));
  return check_launch();
}

}  // namespace tc

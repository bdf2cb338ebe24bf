// Per-node softmax statistics of the verifier logits.
//
// The scheduler of §4 reads the target's top-1 probability p0 at the
// verifier's last position; §3 / Appendix A use the entropy of the same
// distribution as the regime signal.  For every logits row the kernel
// produces the lowest-index argmax, p1 = 1/Z and the entropy
// H = ln Z - sum (y - m) e^(y - m) / Z with y = inv_temp * z, m = max y.
//
// One workgroup per row.  A slab of the row (up to 32768 entries, 16384 where V
// is no multiple of four: up to 64 registers a thread) has all its loads in
// flight at once, and a row of one slab stays in registers for both steps
// (max / argmax, then the two sums); longer rows are read twice, the second
// time from L2.  With a load a loop trip the kernel waited out a memory latency
// per 2048 entries (per 512 where V is no multiple of four): 26 rows of 32000
// 12.7 -> 11.9 us, of 24001 19.2 -> 13.6; the exponentials of one CU are what
// is left.  Reductions use wave shuffles and a fixed-order combine of the
// per-wave results, so the result does not depend on scheduling.
#include <cfloat>
#include <climits>

#include "common.hpp"

namespace entmtp {
namespace {

constexpr int kStatsThreads = 512;
constexpr int kStatsWaves = kStatsThreads / 64;

// (value, index) pair ordered by value descending, then index ascending:
// an associative total order, so any reduction tree gives the same winner.
__device__ __forceinline__ void take_best(float& v, int& i, float v2, int i2) {
  if (v2 > v || (v2 == v && i2 < i)) {
    v = v2;
    i = i2;
  }
}

// VEC: V is a multiple of four (rows of 16-byte units), else units of one entry.
// R: units per thread and slab.
template <bool VEC, int R>
__global__ __launch_bounds__(kStatsThreads) void logit_stats_kernel(
    const float* __restrict__ logits, int V, float inv_temp, float* __restrict__ entropy,
    float* __restrict__ top1p, int* __restrict__ argmax) {
  __shared__ float s_v[kStatsWaves];
  __shared__ int s_i[kStatsWaves];
  __shared__ float s_z[kStatsWaves], s_s[kStatsWaves];

  constexpr int E = VEC ? 4 : 1;             // entries per unit
  const float* z = logits + static_cast<size_t>(blockIdx.x) * V;
  const int tid = threadIdx.x;
  const int lane = tid & 63, wave = tid >> 6;
  const int n = V / E;
  const bool one = n <= R * kStatsThreads;   // one slab: it stays in registers
  float x[R][E];
  auto load = [&](int u0) {   // (past the row: its last unit, not used)
#pragma unroll
    for (int i = 0; i < R; ++i) {
      if (u0 + kStatsThreads * i >= n) break;   // (uniform)
      const int u = min(u0 + tid + kStatsThreads * i, n - 1);
      if constexpr (VEC) {
        const float4 v = reinterpret_cast<const float4*>(z)[u];
        x[i][0] = v.x;
        x[i][1] = v.y;
        x[i][2] = v.z;
        x[i][3] = v.w;
      } else {
        x[i][0] = z[u];
      }
    }
  };
  auto each = [&](int u0, auto f) {   // f(entry, index) in index order
#pragma unroll
    for (int i = 0; i < R; ++i) {
      if (u0 + kStatsThreads * i >= n) break;
      const int u = u0 + tid + kStatsThreads * i;
      if (u < n) {
#pragma unroll
        for (int e = 0; e < E; ++e) f(x[i][e], E * u + e);
      }
    }
  };

  // ---- max and lowest index attaining it
  float best = -INFINITY;
  int bidx = INT_MAX;
  for (int u0 = 0; u0 < n; u0 += R * kStatsThreads) {
    load(u0);
    each(u0, [&](float v, int i) { take_best(best, bidx, v, i); });
  }
#pragma unroll
  for (int off = 32; off >= 1; off >>= 1)
    take_best(best, bidx, __shfl_xor(best, off, 64), __shfl_xor(bidx, off, 64));
  if (lane == 0) {
    s_v[wave] = best;
    s_i[wave] = bidx;
  }
  __syncthreads();
  best = s_v[0];
  bidx = s_i[0];
  for (int w = 1; w < kStatsWaves; ++w) take_best(best, bidx, s_v[w], s_i[w]);

  // ---- Z = sum e^(y-m), S = sum (y-m) e^(y-m)
  // (the difference of the raw logits first: exact or nearly, 0 for the largest)
  float Z = 0.f, S = 0.f;
  for (int u0 = 0; u0 < n; u0 += R * kStatsThreads) {
    if (!one) load(u0);
    each(u0, [&](float v, int) {
      const float t = (v - best) * inv_temp;
      const float e = expf(t);
      Z += e;
      if (e > 0.f) S += t * e;  // keeps (-inf) * 0 out of the sum
    });
  }
#pragma unroll
  for (int off = 32; off >= 1; off >>= 1) {
    Z += __shfl_xor(Z, off, 64);
    S += __shfl_xor(S, off, 64);
  }
  if (lane == 0) {
    s_z[wave] = Z;
    s_s[wave] = S;
  }
  __syncthreads();
  if (tid == 0) {
    float Zt = 0.f, St = 0.f;
    for (int w = 0; w < kStatsWaves; ++w) {
      Zt += s_z[w];
      St += s_s[w];
    }
    if (entropy) entropy[blockIdx.x] = logf(Zt) - St / Zt;
    if (top1p) top1p[blockIdx.x] = 1.f / Zt;
    if (argmax) argmax[blockIdx.x] = bidx;
  }
}

}  // namespace
}  // namespace entmtp

using namespace entmtp;

extern "C" int32_t entmtp_logit_stats(const float* logits, int32_t T, int32_t V, float inv_temp,
                                      float* entropy, float* top1p, int32_t* argmax,
                                      void* stream) {
  clear_error();
  ENTMTP_CHECK_ARG(logits != nullptr, ENTMTP_EINVAL, "logits is NULL");
  ENTMTP_CHECK_ARG(T >= 1 && V >= 1, ENTMTP_EINVAL, "T = %d, V = %d must be >= 1", T, V);
  ENTMTP_CHECK_ARG(inv_temp > 0.f && inv_temp < INFINITY, ENTMTP_EINVAL,
                   "inv_temp = %g must be positive and finite", static_cast<double>(inv_temp));
  ENTMTP_CHECK_ARG(aligned16(logits), ENTMTP_EINVAL, "logits must be 16-byte aligned");
  if (!entropy && !top1p && !argmax) return ENTMTP_OK;
  auto go = [&](auto kernel) {
    hipLaunchKernelGGL(kernel, dim3(T), dim3(kStatsThreads), 0, static_cast<hipStream_t>(stream), logits,
                       V, inv_temp, entropy, top1p, argmax);
  };
  // Short rows take a slab of a quarter: at 40 registers a thread instead of 88
  // four workgroups share a CU, which more rows than CUs need (300 rows of 1000
  // to 4000 entries 6.3 - 7.1 us in the long form, loads past the row included,
  // 4.4 - 5.4 in this one); longer rows want every load of theirs in flight.
  if ((V & 3) == 0)
    V <= 16 * kStatsThreads ? go(logit_stats_kernel<true, 4>) : go(logit_stats_kernel<true, 16>);
  else
    V <= 8 * kStatsThreads ? go(logit_stats_kernel<false, 8>) : go(logit_stats_kernel<false, 32>);
  return launch_status("logit_stats launch");
}

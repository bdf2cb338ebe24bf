// Speculative-sampling verification of a draft tree (§2.1).
//
// §2.1 states the rule for one chain: a draft token t is kept with
// probability min(1, p(t) / p_hat(t)), p the target's distribution and p_hat
// the draft's, left to right; at the first rejection the rest is dropped and
// a replacement is drawn from norm(max(0, p - p_hat)).  On a tree the walk
// starts at the root with r = p there and tries the current node's children
// in index (rank) order, all drafted from the node's draft distribution q:
// child c passes when u_c * q(t_c) < r(t_c); the first that passes becomes
// the current node (r = p at it), and each one that fails replaces r by
// norm(max(0, r - q)) before the next sibling is tried.  When no child
// passes, or the node is a leaf, the bonus token is drawn from r by inverse
// CDF over the vocabulary in index order.  For a chain this is the rule
// above; the uniforms are inputs, so a run is reproducible.
//
// One workgroup of 1024 threads walks the tree.  The target's distribution at
// a node comes from its logits and the statistics the LM head already
// produced at the same temperature (argmax and top-1 probability:
// p(v) = exp((z_v - z_argmax) * inv_temp) * top1p), so a level that accepts
// costs no pass over the vocabulary.  The walk is sequential in its
// decisions, so the kernel is bound by its memory round trips (one CU reads a
// row): the per-node inputs come in with the first of them, a node's children
// are looked up together, and a pass over the vocabulary has 32 loads of each
// thread in flight.  Up to 32768 entries the node's row (p, then the residual)
// stays in LDS (r as it is: p, then the normalised residual), so passes after
// the first read only q, and the draw reads the LDS; a rejection's values wait
// in registers for their mass.  (The row itself in registers spilled: 16 waves
// leave 128 a lane, 134 us.)  What is left is one CU's arithmetic: an
// exponential an entry and node, a division an entry and rejection.  Sums keep
// one order in both forms (a thread's entries v = tid, tid + 1024, ... for the
// mass, its contiguous chunk for the draw, then lanes, then wavefronts).
// Statistics and walk, whole calls, 32000 entries: 26 nodes 69 -> 35 us (the
// walk about 56 -> 21), 60 nodes 104 -> 44; 128256 entries, 64 nodes 612 -> 252
// (before: a load a trip, each waited for, and three passes a rejection).
#include "common.hpp"
#include "stream_pipe.hpp"

namespace entmtp {
namespace {

constexpr int kSpecThreads = 1024;
constexpr int kSpecWaves = kSpecThreads / 64;

// Sum in a fixed order: lanes by butterfly, then the wavefronts in order.
__device__ __forceinline__ float block_sum(float v, float* red) {
#pragma unroll
  for (int off = 32; off >= 1; off >>= 1) v += __shfl_xor(v, off, 64);
  __syncthreads();
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = v;
  __syncthreads();
  float s = red[0];
#pragma unroll
  for (int w = 1; w < kSpecWaves; ++w) s += red[w];
  return s;
}

constexpr int kSpecRegs = 32;        // entries a thread of the longest row kept in LDS
constexpr int kSpecShortRegs = 8;    // and of the short ones
constexpr int kSpecTinyRegs = 2;
constexpr int kSpecBatch = 16;                           // else: loads of each row in flight per thread
constexpr int kSpecSeg = 16;                             // entries of each chunk staged at a time (draw)
constexpr int kSpecSegLd = kSpecSeg + 1;

// Dynamic LDS of the form that keeps a row of R entries a thread (and its
// padding), or with R = 0 a segment of every thread's chunk.
constexpr size_t spec_lds(int R) {
  return (R > 0 ? R * kSpecThreads + 3 * (R * kSpecThreads / 32) : kSpecThreads * kSpecSegLd) * sizeof(float);
}

constexpr size_t kSpecStaticLds = 11 * 1024;   // (the per-node arrays, rounded up)
static_assert(spec_lds(kSpecRegs) + kSpecStaticLds <= 160 * 1024, "the resident row fits in the LDS of a CU");

// R > 0: the vocabulary has at most R entries a thread, and its row is kept.
template <int R>
__global__ __launch_bounds__(kSpecThreads) void accept_stochastic_kernel(
    const int* __restrict__ parent, const int* __restrict__ depth,
    const int* __restrict__ path_tab, int T, int D, const int* __restrict__ tok,
    const float* __restrict__ z, const float* __restrict__ q, int V, float inv_temp,
    const int* __restrict__ amax, const float* __restrict__ top1p,
    const float* __restrict__ u_accept, const float* __restrict__ u_sample, float* __restrict__ w,
    int* __restrict__ accept_len, int* __restrict__ path_out, int path_cap,
    int* __restrict__ bonus) {
  constexpr bool RES = R > 0;
  constexpr int NR = RES ? R : 1;   // entries a thread
  extern __shared__ float s_row[];
  __shared__ float red[kSpecWaves];
  __shared__ float s_scan[kSpecWaves];
  __shared__ int s_parent[ENTMTP_T_MAX], s_tok[ENTMTP_T_MAX], s_amax[ENTMTP_T_MAX];
  __shared__ float s_top1p[ENTMTP_T_MAX], s_ua[ENTMTP_T_MAX], s_us[ENTMTP_T_MAX];
  __shared__ int s_depth[ENTMTP_T_MAX];
  __shared__ int s_children[ENTMTP_T_MAX];
  __shared__ float s_zc[ENTMTP_T_MAX], s_qc[ENTMTP_T_MAX];   // the children's tokens in cur's rows
  __shared__ int s_count[ENTMTP_T_MAX / 64];
  __shared__ float s_zm;
  __shared__ int s_claim, s_last;
  __shared__ float s_excl;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  if (tid < T) {
    s_parent[tid] = parent[tid];
    s_tok[tid] = tok[tid];
    s_amax[tid] = amax[tid];
    s_top1p[tid] = top1p[tid];
    s_ua[tid] = u_accept[tid];
    s_us[tid] = u_sample[tid];
    s_depth[tid] = depth[tid];
  }
  static_assert(kSpecThreads >= ENTMTP_T_MAX, "one thread per node");
  // The draw gives thread t the contiguous chunk [t * chunk, (t + 1) * chunk).
  // Resident entry v lies at v + 3 (v / 32): chunks of any length up to 32 then
  // start in different banks (conflicts of two to four lanes at the worst), and
  // a thread's entries tid + 1024 i at a constant stride.
  const int chunk = (V + kSpecThreads - 1) / kSpecThreads;
  auto at = [](int v) { return v + 3 * (v >> 5); };
  constexpr int kStride = kSpecThreads + 3 * (kSpecThreads / 32);
  float* const mine_row = s_row + at(tid);
  // entries tid + 1024 i, i < R, of a row (zeros past its end)
  auto load_row = [&](const float* row, float (&x)[NR]) {
    const __amdgpu_buffer_rsrc_t buf = dma_buffer(row, static_cast<uint32_t>(V) * 4u);
#pragma unroll
    for (int i = 0; i < NR; ++i) x[i] = buf_load(buf, (tid + i * kSpecThreads) * 4u);
  };
  __syncthreads();
  int cur = 0;
  // each level descends one depth, so the walk ends within D + 1 levels
  for (int level = 0; level <= D; ++level) {
    const float* zr = z + static_cast<size_t>(cur) * V;
    const float* qr = q + static_cast<size_t>(cur) * V;
    // cur's children in index order, each with its token's logit and draft
    // probability, and the largest logit
    bool mine = false;
    int rank = 0;
    float zc = 0.f, qc = 0.f;
    if (tid < ENTMTP_T_MAX) {   // whole wavefronts
      mine = tid > cur && tid < T && s_parent[tid < T ? tid : 0] == cur;
      const unsigned long long m = __ballot(mine);
      rank = __popcll(m & ((1ull << lane) - 1ull));
      if (lane == 0) s_count[wave] = __popcll(m);
      const int t = mine ? s_tok[tid] : -1;
      if (t >= 0 && t < V) {
        zc = zr[t];
        qc = qr[t];
      }
    } else if (tid == ENTMTP_T_MAX) {
      s_zm = zr[s_amax[cur]];
    }
    __syncthreads();
    int nchild = 0;
#pragma unroll
    for (int k = 0; k < ENTMTP_T_MAX / 64; ++k) {
      if (k < wave) rank += s_count[k];
      nchild += s_count[k];
    }
    if (mine) {
      s_children[rank] = tid;
      s_zc[rank] = zc;
      s_qc[rank] = qc;
    }
    __syncthreads();
    // target distribution at cur: p(v) = exp((z_v - z_max) * inv_temp) * top1p
    const float zm = s_zm, p1 = s_top1p[cur];
    auto p_of = [&](float x) { return expf((x - zm) * inv_temp) * p1; };
    bool resid = false;   // r(v) = p(v), or once resid the normalised residual (s_row or w)
    int next = -1;
    bool loaded = false;   // (RES) s_row holds r
    auto fill = [&]() {
      loaded = true;
      float a[NR];
      load_row(zr, a);
#pragma unroll
      for (int i = 0; i < NR; ++i) {   // (zeros past the row: they stay so in every residual)
        mine_row[i * kStride] = tid < V - kSpecThreads * i ? p_of(a[i]) : 0.f;
        if (i % 8 == 7) __builtin_amdgcn_sched_barrier(0);   // (all at once would spill)
      }
    };
    // f(v, r(v), q(v)) of this thread's entries, in index order; src: where r
    // lies (z: as logits)
    auto each = [&](const float* src, auto f) {
      for (int v0 = tid; v0 < V; v0 += kSpecBatch * kSpecThreads) {
        float a[kSpecBatch], b[kSpecBatch];
#pragma unroll
        for (int i = 0; i < kSpecBatch; ++i) {   // (past the row: its last entry, not used)
          const int v = min(v0 + kSpecThreads * i, V - 1);
          a[i] = src[v];
          b[i] = qr[v];
        }
#pragma unroll
        for (int i = 0; i < kSpecBatch; ++i)
          if (v0 + kSpecThreads * i < V) f(v0 + kSpecThreads * i, a[i], b[i]);
      }
    };
    for (int j = 0; j < nchild; ++j) {
      const int c = s_children[j];
      const int t = s_tok[c];
      const bool in_v = t >= 0 && t < V;
      const float qt = s_qc[j];
      float rt = 0.f;
      if (in_v) rt = resid ? (RES ? s_row[at(t)] : w[t]) : p_of(s_zc[j]);
      if (qt > 0.f ? (s_ua[c] * qt < rt) : (rt > 0.f)) {   // (the same in every thread)
        next = c;
        break;
      }
      // residual max(0, r - q): its mass, then (if any: else r stays as it is)
      // the values over it
      float part = 0.f;
      if constexpr (RES) {
        if (!loaded) fill();
        float x[NR];
        load_row(qr, x);
#pragma unroll
        for (int i = 0; i < NR; ++i) {
          x[i] = fmaxf(mine_row[i * kStride] - x[i], 0.f);
          part += x[i];
        }
        const float mass = block_sum(part, red);
        if (mass > 0.f) {
          resid = true;
#pragma unroll
          for (int i = 0; i < NR; ++i) {
            mine_row[i * kStride] = x[i] / mass;
            if (i % 8 == 7) __builtin_amdgcn_sched_barrier(0);
          }
        }
      } else if (!resid) {   // (w is free: the values go there, whatever their mass)
        each(zr, [&](int v, float x, float qx) {
          const float y = fmaxf(p_of(x) - qx, 0.f);
          part += y;
          w[v] = y;
        });
        const float mass = block_sum(part, red);
        if (mass > 0.f) {
          resid = true;
          each(w, [&](int v, float x, float) { w[v] = x / mass; });
        }
      } else {
        each(w, [&](int, float x, float qx) { part += fmaxf(x - qx, 0.f); });
        const float mass = block_sum(part, red);
        if (mass > 0.f) each(w, [&](int v, float x, float qx) { w[v] = fmaxf(x - qx, 0.f) / mass; });
      }
      __syncthreads();   // the residual is written before its entries are read
    }
    if (next >= 0) {
      cur = __builtin_amdgcn_readfirstlane(next);   // (the same in every thread)
      __syncthreads();   // s_children is rebuilt for the next level
      continue;
    }
    // draw from r: contiguous chunks per thread, exclusive scan of their sums
    const int a = s_depth[cur];
    const int pnode = tid <= D ? path_tab[cur * (D + 1) + tid] : -1;   // (ahead of the draw's passes)
    const int v0 = tid * chunk, v1 = min(V, v0 + chunk);
    float cs = 0.f;
    int last = -1;   // this chunk's last token with mass
    if constexpr (RES) {
      if (!loaded) fill();
      __syncthreads();   // the row's entries are read by other threads
#pragma unroll 8
      for (int v = v0; v < v1; ++v) {
        const float r = s_row[at(v)];
        cs += r;
        if (r > 0.f) last = v;
      }
    } else {
      // a segment of every chunk at a time through the LDS
      const float* src = resid ? w : zr;
      for (int s0 = 0; s0 < chunk; s0 += kSpecSeg) {
        float x[kSpecSeg];
        const int o = tid & (kSpecSeg - 1);
#pragma unroll
        for (int k = 0; k < kSpecSeg; ++k) {
          const long long v = static_cast<long long>((tid / kSpecSeg) + (kSpecThreads / kSpecSeg) * k) * chunk + s0 + o;
          x[k] = src[v < V ? v : V - 1];
        }
        __syncthreads();   // the previous segment is read out
#pragma unroll
        for (int k = 0; k < kSpecSeg; ++k)
          s_row[((tid / kSpecSeg) + (kSpecThreads / kSpecSeg) * k) * kSpecSegLd + o] = resid ? x[k] : p_of(x[k]);
        __syncthreads();
        for (int i = 0; i < kSpecSeg; ++i) {
          const int v = v0 + s0 + i;
          if (s0 + i < chunk && v < V) {
            const float r = s_row[tid * kSpecSegLd + i];
            cs += r;
            if (r > 0.f) last = v;
          }
        }
      }
    }
    float incl = cs;   // inclusive scan within the wavefront
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) {
      const float o = __shfl_up(incl, off, 64);
      if (lane >= off) incl += o;
    }
    if (lane == 63) s_scan[wave] = incl;
    if (tid == 0) {
      s_claim = 0x7fffffff;
      s_last = -1;
    }
    __syncthreads();
    float base = 0.f, total = 0.f;
    for (int wv = 0; wv < kSpecWaves; ++wv) {
      if (wv < wave) base += s_scan[wv];
      total += s_scan[wv];
    }
    const float excl = base + incl - cs;
    const float target = s_us[cur] * total;
    // the chunk the target falls in (rounding at a chunk boundary could let
    // two chunks claim it: the first), and the last token with mass
    const bool claims = cs > 0.f && excl <= target && target < excl + cs;
    if (claims) atomicMin(&s_claim, tid);
    const unsigned long long has = __ballot(last >= 0);
    if (has && lane == 63 - __clzll(has)) atomicMax(&s_last, last);
    __syncthreads();
    const int claim = s_claim;
    if (tid == claim) s_excl = excl;
    int hit = s_last;   // past the rounded total (no chunk claims the target)
    if (claim != 0x7fffffff) {
      // the claimed chunk, entry by entry (its r staged by the workgroup)
      const int c0 = claim * chunk, c1 = min(V, c0 + chunk);
      float acc = 0.f;
      hit = c1 - 1;
      bool found = false;
      for (int s0 = c0; s0 < c1; s0 += kSpecThreads) {
        __syncthreads();   // s_excl is written; the previous piece is read out
        float x = 0.f;
        if (s0 + tid < c1) {
          if constexpr (RES) x = s_row[at(s0 + tid)];
          else x = resid ? w[s0 + tid] : p_of(zr[s0 + tid]);
        }
        __syncthreads();   // (the row's entries are read before the piece overwrites them)
        s_row[tid] = x;
        __syncthreads();
        if (s0 == c0) acc = s_excl;
        if (tid == 0 && !found) {   // (every thread makes every round: they hold barriers)
          const int n = min(kSpecThreads, c1 - s0);
#pragma unroll 8
          for (int i = 0; i < n && !found; ++i) {
            acc += s_row[i];
            if (acc > target) {
              hit = s0 + i;
              found = true;
            }
          }
        }
      }
    }
    if (tid < path_cap) path_out[tid] = tid <= a ? pnode : -1;
    if (tid == 0) {
      *accept_len = a;
      *bonus = hit;
    }
    return;
  }
}

}  // namespace
}  // namespace entmtp

using namespace entmtp;

extern "C" int32_t entmtp_accept_stochastic(const entmtp_bank* bank, int32_t topo,
                                            const int32_t* draft_tokens, const float* logits,
                                            const float* q, int32_t V, float inv_temp,
                                            const int32_t* argmax, const float* top1p,
                                            const float* u_accept, const float* u_sample,
                                            float* workspace, int32_t* accept_len,
                                            int32_t* path, int32_t* bonus, void* stream) {
  clear_error();
  ENTMTP_CHECK_ARG(draft_tokens && logits && q && argmax && top1p && u_accept && u_sample &&
                       workspace && accept_len && path && bonus,
                   ENTMTP_EINVAL, "pointers must be non-NULL");
  ENTMTP_CHECK_ARG(V >= 1, ENTMTP_EINVAL, "V = %d < 1", V);
  ENTMTP_CHECK_ARG(inv_temp > 0.f && inv_temp < INFINITY, ENTMTP_EINVAL,
                   "inv_temp must be positive and finite");
  if (int32_t rc = check_device_bank(bank, topo)) return rc;
  const TopoDesc& d = bank->desc[topo];
  auto go = [&](auto kernel, size_t lds) {
    hipLaunchKernelGGL(kernel, dim3(1), dim3(kSpecThreads), lds, static_cast<hipStream_t>(stream),
                       bank_ptr<int>(bank, d.off_parent), bank_ptr<int>(bank, d.off_depth),
                       bank_ptr<int>(bank, d.off_path), d.T, d.D, draft_tokens, logits, q, V, inv_temp,
                       argmax, top1p, u_accept, u_sample, workspace, accept_len, path, d.D + 1, bonus);
  };
  // a row in the LDS of one CU up to 32 entries a thread (140 KB of it), else a
  // segment at a time.  Short rows have instances of their own: with the long
  // row's 32 exponentials and divisions a thread a pass over 1000 entries took
  // 20.5 us a walk of 8 nodes, 9.0 with two (12.0 in a loop of loads), and one
  // over 4000 11.9, 8.1 with eight (10.5)
  if (V <= kSpecTinyRegs * kSpecThreads)
    go(accept_stochastic_kernel<kSpecTinyRegs>, spec_lds(kSpecTinyRegs));
  else if (V <= kSpecShortRegs * kSpecThreads)
    go(accept_stochastic_kernel<kSpecShortRegs>, spec_lds(kSpecShortRegs));
  else if (V <= kSpecRegs * kSpecThreads)
    go(accept_stochastic_kernel<kSpecRegs>, spec_lds(kSpecRegs));
  else
    go(accept_stochastic_kernel<0>, spec_lds(0));
  return launch_status("accept_stochastic launch");
}

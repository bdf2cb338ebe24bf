// Tree-masked attention of the verification pass.
//
// §2.3: the draft tree is verified in a single sparse forward pass of the
// target model with a precomputed tree attention mask and position offsets;
// §3.2 names the mask size among the per-step verifier costs.  Node i of the
// tree attends to the whole prefix and to the nodes on its own root-to-node
// path; it sits at sequence position prefix_len + depth(i).
//
// Two kernels, both on the caller's stream:
//  1. attend: flash-decoding over the cache.  The queries and the tree's keys
//     are rotated to their positions as they are loaded (fp64 angles from a
//     per-workgroup LDS table over the tree's depths, one bf16 rounding); the
//     tree's keys and values come from the step's inputs rather than the
//     cache, and the workgroups of the first query group write them (keys
//     rotated) into cache slots [L, L+T) for the steps after this one.
//     A workgroup owns one (KV head, group of four 32-row query tiles, key
//     split), a tile per wave, and the waves walk the same 32-key blocks,
//     copied once per workgroup straight into a ring in LDS, so a block is
//     read once per 128 rows.  Trees of one tile run the same kernel with
//     three waves only loading: a block then costs one wave 0.55 us, and the
//     form that split the keys over the waves instead (a wave's keys in
//     registers, merged through LDS at the end) took 14.6 us and a merge of
//     4.1 where this one, unsplit, takes 12.8 (27 nodes, prefix 256), and
//     43.3 us a call against 40.3 at prefix 8192 with 40 heads.
//     S^T = K Q^T and O^T += V^T P^T run on v_mfma_f32_32x32x16_bf16, V
//     transposed by the LDS read, P never leaving registers (the S^T accumulator
//     layout is re-read as the B operand of the PV product after a fixed key
//     permutation).  Blocks wholly inside the prefix skip the mask; the
//     others take a 32-bit window cut from the node's ancestor bitmask.
//     Online softmax in fp32, base 2, with a lazily raised running max (the
//     accumulators are rescaled only when a block's max passes the reference
//     by more than 2^8).  A weight equal to the reference is exact in bf16, so
//     fewer references cost trees of one tile a little: error against 64 bits
//     3.27e-3 where four waves with a reference each had 3.13e-3; raising it at
//     every block gives 3.17e-3 and takes 3 - 10 % longer.
//  2. merge: combines the splits' partials: (max, sum) in fp32 and the
//     output normalised by its sum, in bf16 (half the bytes of fp32; a
//     normalised partial stays within the range of the values).
//     Skipped when a single split covers the keys.
#include <algorithm>
#include <cfloat>
#include <cmath>
#include <mutex>
#include <type_traits>

#include "common.hpp"
#include "stream_pipe.hpp"

namespace entmtp {
namespace {

typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef float f32x2 __attribute__((ext_vector_type(2)));

constexpr int HD = ENTMTP_HEAD_DIM;  // 128
constexpr int kAttnThreads = 256;
constexpr int KB = 32;               // keys per block
constexpr int kQTile = 32;           // query rows per tile
constexpr float kLazyLog2 = 8.f;     // the running max is raised only past this many doublings
constexpr int kMaxSplits = 32;
constexpr int kMinBlocksPerSplit = 4;
// Sequences of up to this many key blocks are not split: a merge (launch,
// partials, its gap) costs as much as the blocks it saves.  Captured calls back
// to back, split / unsplit, 32 KV heads: 9 blocks 12.5 / 12.2 us (27 nodes), 10
// 14.1 / 14.4 (64), 11 12.3 / 12.9 (7) and 12.5 / 13.0 (27), where calls from
// Python still gain unsplit (13.9 / 13.1); 12 13.6 / 15.3 (64), 13 12.3 / 14.3,
// 20 13.7 / 18.9 (27).  4 and 8 KV heads alike.
constexpr int kLoneBlocks = 11;
constexpr int kTilesPerWg = 4;       // query tiles per workgroup, one per wave
constexpr int kWgPerCu = 2;          // attend workgroups resident per CU (registers, LDS)
constexpr int kMaxSeqs = ENTMTP_B_MAX;

__host__ __device__ inline int rows_padded(int G, int T) {
  return (G * T + kQTile - 1) / kQTile * kQTile;
}

// Workgroups along the query rows: groups of four 32-row tiles.
__host__ __device__ inline int query_groups(int nqt) { return (nqt + kTilesPerWg - 1) / kTilesPerWg; }

__host__ __device__ inline int split_bound(int nblocks) {
  if (nblocks <= kLoneBlocks) return 1;
  const int b = nblocks / kMinBlocksPerSplit;
  return b > kMaxSplits ? kMaxSplits : b;
}

// Split count of a lone sequence: pick the count that fills the resident
// workgroups (slots) in whole rounds -- the first (1..bound) whose last
// round is at least 90% full, else the fullest one seen (integer arithmetic,
// so that the host and the device choose alike).
__host__ __device__ inline int split_for_bound(int bound, int base_wg, int slots) {
  int best = 1;
  long long best_wg = 0, best_rounds = 1;
  for (int ns = 1; ns <= bound; ++ns) {
    const long long wg = static_cast<long long>(base_wg) * ns;
    const long long rounds = (wg + slots - 1) / slots;
    if (wg * best_rounds > best_wg * rounds) {   // fill wg / (rounds * cus) improves
      best_wg = wg;
      best_rounds = rounds;
      best = ns;
    }
    if (10 * wg >= 9 * rounds * slots) break;
  }
  return best;
}

__host__ __device__ inline int split_single(int nblocks, int base_wg, int cus) {
  return split_for_bound(split_bound(nblocks), base_wg, cus * kWgPerCu);
}

// Where split k of ns begins: even shares of nblocks + tree_extra blocks, the
// last split, which holds the tree's keys, shorter by tree_extra.  A block of
// tree keys is rotated and staged through registers (about two prefix blocks'
// time) after a table of fp64 angles (two more): given an even share that
// workgroup ended 8 us after the others at 128 nodes and prefix 8192 (43.8
// against a median of 35), 4 us at 27 nodes and prefix 2048.
constexpr int kTreeSetup = 2;
__host__ __device__ inline int tree_extra(int nblocks, int L, int ns) {
  const int extra = kTreeSetup + nblocks - L / KB, share = nblocks / ns;
  return extra < share ? extra : share;   // (the last split keeps a block)
}
__device__ __forceinline__ int split_begin(int k, int ns, int nblocks, int extra) {
  return k < ns ? static_cast<int>(static_cast<unsigned>(k) * static_cast<unsigned>(nblocks + extra) / ns)
                : nblocks;
}

// A batch of several sequences shares one blocks-per-split target t: sequence
// b, with H_b streams (KV heads x query groups) of nb_b blocks, takes
// ns_b(t) = ceil(nb_b / t) splits (clipped to [1, split_bound]).  Every
// workgroup costs its blocks and a fixed part, and the chip runs `slots` of
// them at a time, so the target minimises
//   rounds(sum H_b ns_b(t)) * (kWgFixed + t)  (+ kMergeCost when any is split)
// over kTargets candidates: the last one splits nothing (t = the longest),
// the others are multiples of the even share work / slots, from half of it
// (two rounds) up.  A fixed number of workgroups per CU instead (three, at two
// resident) left the second round half empty: eight GQA sequences 103 us
// against 88, at prefixes up to 4096 62 us a call against 48.
constexpr int kTargets = 16;
constexpr int kWgFixed = 6;      // a workgroup's fixed part, in blocks (8 us at 1.3-1.7 us a block)
constexpr int kMergeCost = 4;    // the merge kernel, in blocks
__host__ __device__ inline int target_sixteenths(int k) {   // of the even share
  constexpr unsigned long long lo = 0x1413121110'0a0908ull;   // 8 9 10 16 17 18 19 20
  constexpr unsigned long long hi = 0x60402820'1e1c1816ull;   // 22 24 28 30 32 40 64 96
  return static_cast<int>((k < 8 ? lo >> (8 * k) : hi >> (8 * (k - 8))) & 0xff);
}
__host__ __device__ inline int batch_target(int k, long long work, int nb_max, int slots) {
  if (k == kTargets - 1) return nb_max > 1 ? nb_max : 1;
  const long long t = (work * target_sixteenths(k) + 16LL * slots - 1) / (16LL * slots);
  return static_cast<int>(t > kMinBlocksPerSplit ? (t < nb_max ? t : nb_max) : kMinBlocksPerSplit);
}
__host__ __device__ inline int batch_splits(int nb, int t) {
  const int ns = (nb + t - 1) / t, bound = split_bound(nb);
  return ns < 1 ? 1 : (ns > bound ? bound : ns);
}
// One key per candidate: the smallest wins (the lowest candidate among equals).
__host__ __device__ inline unsigned long long batch_cost(int k, int t, long long items, bool split,
                                                         int slots) {
  const long long rounds = (items + slots - 1) / slots;
  return (static_cast<unsigned long long>(rounds * (kWgFixed + t) + (split ? kMergeCost : 0)) << 8) | k;
}
// Most workgroups a planned batch can have (padding aside) when its streams
// number at most `streams`: the two-round candidates are allowed only where
// the streams alone nearly fill the chip, and a split count is below
// nb / t + 1, so the items stay below work / t + streams.
__host__ __device__ inline bool two_rounds(long long streams_bound, int slots) {
  return 4 * streams_bound > 3LL * slots;
}

// ----------------------------------------------------------- descriptors --

// One sequence of a (possibly batched) call, planned on the host.
struct SeqPlan {
  uint16_t* kc;            // [Hkv][cap][HD] this sequence's cache
  uint16_t* vc;
  const uint32_t* mask;    // [T][ENTMTP_MASK_WORDS] its tree's ancestor bitmask
  const int* depth;        // [T]
  int T, L, row0;          // nodes, prefix length, first row in the concatenated q / out
  int D;                   // depth of the tree's deepest node
  int rows_pad, nqt, nqg, nsplit;   // padded rows, query tiles, query groups, splits
  int item0;               // first attend workgroup of the sequence
  int merge0;              // first merge block of the sequence
  long long part_off;      // row offset of its split partials
};

// A bank tree as a device-planned batch finds it (kernel arguments).
struct TreeHdr {
  int T, D, off_mask, off_depth;
};
constexpr int kMaxTreesArg = 32;   // bank trees a device-planned batch can name

struct BatchArgs {
  SeqPlan s[kMaxSeqs];
  // device-planned batch: sequence b's tree, prefix length and first row
  // come from device arrays (topo_dev[b], len_dev[b], row_off_dev[b]); the
  // host fixed its caches and partial range (at strides sized for the bank's
  // largest plan), and every workgroup derives the plan the host would have
  // made (plan_call), its own place in it included, from those arrays
  const int32_t* topo_dev;
  const int32_t* len_dev;
  const int32_t* row_off_dev;   // [B + 1]
  int rows_cap;                 // rows q / k_tree / v_tree / out hold
  int n_trees;
  TreeHdr trees[kMaxTreesArg];
  // device-planned single sequence (a tree chosen on the GPU): when dev is
  // set, sequence 0's tree, prefix length and split plan come from *dev, the
  // bank descriptors and the CU count, and the grids are sized for the
  // largest plan
  const DevStep* dev;
  const DevTopo* topos;
  const uint8_t* arena;
  int cus;
  int two_rounds;          // device-planned batch: two_rounds() of the streams the host can bound
  int B, G, Hq, Hkv, cap;
  float scale_log2;
  double theta;            // rotation base (0: no rotation)
  double freq[HD / 2];     // theta^(-2c/d) of pair c, computed on the host
  const uint16_t* q;       // [rows][Hq][HD] (rows = sum of T, sequence after sequence)
  const uint16_t* kt;      // [rows][Hkv][HD]
  const uint16_t* vt;
  uint16_t* part_o;        // [part rows][HD] bf16: the split's output, normalised by its sum
  float* part_ml;          // [part rows][2]
  uint16_t* out;           // [rows][Hq][HD]
};
static_assert(sizeof(BatchArgs) <= 4096, "kernel arguments are limited to 4 KB");

// Sequence that owns index `x` of a grid whose per-sequence ranges start at
// `first(b)`, in increasing order (uniform per workgroup): lane i compares
// with sequence i's start, so a batch costs one memory round trip however
// many sequences it has.  Called by whole wavefronts.
template <typename F>
__device__ __forceinline__ int seq_of(const BatchArgs& p, int x, F first) {
  if (p.B == 1) return 0;
  const int lane = threadIdx.x & 63;
  const bool owns = lane < p.B && x >= first(p.s[lane < p.B ? lane : 0]);
  return __popcll(__ballot(owns)) - 1;
}

// Rows a merge block covers (a half-wavefront each).
constexpr int kMergeRows = 8;

// Plan of sequence b: the host's, or -- for a device-planned call -- the
// plan the host would make for the tree and prefix length the device holds
// (same arithmetic), with the caches the host passed.
__device__ __forceinline__ SeqPlan resolve(const BatchArgs& p, int b) {
  if (!p.dev) return p.s[b];
  SeqPlan q = p.s[0];
  const DevStep st = *p.dev;
  const DevTopo* t = p.topos + st.rung;   // read in place (no local copy to index)
  q.T = st.T;
  q.L = st.L;
  q.D = t->D;
  if (q.L < 0 || q.T < 1 || q.L + q.T > p.cap) {   // outside the cache: no attention at all
    q.T = 0;
    q.L = 0;
    q.nsplit = 1;
    q.nqt = 0;
    q.nqg = 0;
    return q;
  }
  q.mask = reinterpret_cast<const uint32_t*>(p.arena + t->off_mask);
  q.depth = reinterpret_cast<const int*>(p.arena + t->off_depth);
  q.row0 = 0;
  q.rows_pad = rows_padded(p.G, q.T);
  q.nqt = q.rows_pad / kQTile;
  q.nqg = query_groups(q.nqt);
  const int nblocks = (q.L + q.T + KB - 1) / KB;
  q.nsplit = t->splits[split_bound(nblocks)];   // = split_single(nblocks, Hkv * nqg, cus)
  q.item0 = 0;
  q.merge0 = 0;
  q.part_off = 0;
  return q;
}

__device__ __forceinline__ long long uniform(long long x) {
  const uint32_t lo = __builtin_amdgcn_readfirstlane(static_cast<int>(x));
  const uint32_t hi = __builtin_amdgcn_readfirstlane(static_cast<int>(x >> 32));
  return static_cast<long long>((static_cast<unsigned long long>(hi) << 32) | lo);
}

// The sequence that owns index x of a device-planned batch's attend or merge
// grid (MERGE), its plan included; T = 0 for an index past the last; total:
// where the indexes end.  Lane i
// of each wavefront reads sequence i's entries; a sequence whose tree index
// lies outside the bank, whose prefix length is negative or leaves no room
// for its tree in the cache, or whose tree rows [row_off[b], row_off[b] + T)
// do not lie in [row_off[b], row_off[b + 1]) and the row capacity has no work
// (T = 0) and counts for nothing in the batch plan.
// The rest is plan_call's arithmetic, the grid ranges a prefix sum over the
// sequences, so that the grid is as long as the plan (the host bounds it) and
// not as long as the largest plan of every sequence: those grids' empty
// workgroups took as long as the attention (185 us a call against 109
// planned on the host).  Called by whole wavefronts.
template <bool MERGE>
__device__ __forceinline__ SeqPlan resolve_batch(const BatchArgs& p, int x, int tid, int& total) {
  const int lane = tid & 63;
  int tr = -1, L = -1, r0 = -1, r1 = -1;
  if (lane < p.B) {
    tr = p.topo_dev[lane];
    L = p.len_dev[lane];
    r0 = p.row_off_dev[lane];
    r1 = p.row_off_dev[lane + 1];
  }
  // every bank tree's size, lane k holding tree k's (requested with the
  // entries above, so one memory round trip covers both)
  const int tree_T = lane < p.n_trees ? p.trees[lane].T : 0;
  const bool named = lane < p.B && tr >= 0 && tr < p.n_trees;
  const int T_named = __shfl(tree_T, named ? tr : 0, 64);
  int T = named ? T_named : 0;
  const long long end = static_cast<long long>(r0) + T;   // (64-bit: the entries are unchecked)
  const bool ok = named && L >= 0 && static_cast<long long>(L) + T <= p.cap && r0 >= 0 &&
                  end <= r1 && end <= p.rows_cap;
  if (!ok) T = 0;
  const int nb = T ? (L + T + KB - 1) / KB : 0;
  const int rows_pad = rows_padded(p.G, T);
  const int nqg = query_groups(rows_pad / kQTile);
  const int H = p.Hkv * nqg;
  int ns = 1;
  const int slots = p.cus * kWgPerCu;
  if (p.B == 1) {
    if (T) ns = split_single(nb, H, p.cus);
  } else {
    // lane k (mod 16) weighs candidate k; the four lanes of a candidate take
    // every fourth sequence
    static_assert(kMaxSeqs == 16 && kTargets == 16, "16 lanes hold the sequences, 16 the candidates");
    long long work = static_cast<long long>(H) * nb;
    int nb_max = nb;
#pragma unroll
    for (int off = 8; off >= 1; off >>= 1) {
      work += __shfl_xor(work, off, 64);
      nb_max = max(nb_max, __shfl_xor(nb_max, off, 64));
    }
    work = uniform(work);   // (lane 0's 16 lanes hold every sequence)
    nb_max = __builtin_amdgcn_readfirstlane(nb_max);
    const int k = lane & 15;
    const int t = batch_target(k, work, nb_max, slots);
    long long items = 0;
    int split = 0;
#pragma unroll
    for (int u = 0; u < kMaxSeqs / 4; ++u) {
      const int b = (lane >> 4) + 4 * u;
      const int nbb = __shfl(nb, b, 64), Hb = __shfl(H, b, 64);
      const int n = batch_splits(nbb, t);
      items += static_cast<long long>(Hb) * n;
      split |= Hb > 0 && n > 1;
    }
#pragma unroll
    for (int off = 16; off <= 32; off <<= 1) {
      items += __shfl_xor(items, off, 64);
      split |= __shfl_xor(split, off, 64);
    }
    unsigned long long cost = batch_cost(k, t, items, split, slots);
    if (target_sixteenths(k) < 16 && !p.two_rounds) cost = ~0ull;
#pragma unroll
    for (int off = 8; off >= 1; off >>= 1) {
      const unsigned long long o = __shfl_xor(cost, off, 64);
      cost = o < cost ? o : cost;
    }
    const int best = __builtin_amdgcn_readfirstlane(static_cast<int>(cost & 0xff));
    ns = batch_splits(nb, __builtin_amdgcn_readlane(t, best));
  }
  // this sequence's range of the grid, and the sequence x lies in
  const int len = MERGE ? (ns > 1 ? (p.Hkv * p.G * T + kMergeRows - 1) / kMergeRows : 0)
                        : (T ? (p.Hkv * ns + 7) / 8 * 8 * nqg : 0);
  int last = len;   // inclusive prefix sum
#pragma unroll
  for (int off = 1; off < kMaxSeqs; off <<= 1) {
    const int o = __shfl_up(last, off, 64);
    if (lane >= off) last += o;
  }
  const unsigned long long past = __ballot(lane < p.B && x >= last);
  const int b = __popcll(past);
  total = __builtin_amdgcn_readlane(last, p.B - 1);
  SeqPlan q = p.s[b < p.B ? b : 0];   // caches and the partial range
  if (b >= p.B) {
    q.T = 0;
    return q;
  }
  // (readlane: the plan stays in scalar registers, and with it the buffer
  // descriptors of the copies; through shuffles a block took 1.0 us, not 0.8)
  auto at = [&](int v) { return __builtin_amdgcn_readlane(v, b); };
  const TreeHdr& h = p.trees[at(tr)];
  q.T = at(T);
  q.L = at(L);
  q.row0 = at(r0);
  q.D = h.D;
  q.mask = reinterpret_cast<const uint32_t*>(p.arena + h.off_mask);
  q.depth = reinterpret_cast<const int*>(p.arena + h.off_depth);
  q.rows_pad = at(rows_pad);
  q.nqt = q.rows_pad / kQTile;
  q.nqg = at(nqg);
  q.nsplit = at(ns);
  q.item0 = q.merge0 = at(last - len);
  return q;
}

// Calls work(plan, x, thread) for the index x this workgroup has in the attend
// or (MERGE) merge grid.  A device-planned batch's grid is as long as any plan
// of sequences whose rows are their own; where row ranges overlap (the entries
// are the device's) the plan can be longer, and a workgroup takes every
// gridDim.x-th index.  The attend kernel takes its first index outside the
// loop: one loop over all of them took 102.1 us for eight GQA sequences, this
// form 100.0, and the first index alone, which left such sequences out, 99.3.
// (The merge is faster in one loop, by 1.9 us.)  What follows from the thread's
// number must not be kept from one index for the next, in registers that spilled
// (84): it is taken anew each time.
template <bool DEVB, bool MERGE, typename F>
__device__ __forceinline__ void for_items(const BatchArgs& p, F work) {
  int x = static_cast<int>(blockIdx.x), tid = static_cast<int>(threadIdx.x);
  if constexpr (DEVB) {
    int total = x + 1;
    if constexpr (!MERGE) {
      const SeqPlan first = resolve_batch<MERGE>(p, x, tid, total);
      if (first.T == 0) return;
      work(first, x, tid);
      x += static_cast<int>(gridDim.x);
    }
    for (; x < total; x += static_cast<int>(gridDim.x)) {
      if constexpr (!MERGE) __syncthreads();   // the LDS of one index is read out
      asm volatile("" : "+v"(tid));
      const SeqPlan sq = resolve_batch<MERGE>(p, x, tid, total);
      work(sq, x, tid);
    }
  } else {
    work(resolve(p, seq_of(p, x, [](const SeqPlan& q) { return MERGE ? q.merge0 : q.item0; })), x, tid);
  }
}

// ------------------------------------------------------------------ RoPE --

// Angles of a tree's positions: the turn of pair (c, c + 64) at position
// L + d, d = 0..D, in fp64 (pos * freq[c], freq[c] = theta^(-2c/d) from the
// host), tabulated as (cos, sin) by the workgroup's threads (a multiple of
// 64: each keeps one pair's frequency).
constexpr int kRopePairs = HD / 2;
inline void set_rope(BatchArgs& a, float rope_theta) {
  a.theta = static_cast<double>(rope_theta);
  // (a model has one base: its 64 powers are kept, per thread, for the next call)
  thread_local double last_theta = -1.0, freq[kRopePairs];
  if (a.theta != last_theta) {
    for (int c = 0; c < kRopePairs; ++c) freq[c] = a.theta > 0.0 ? std::pow(a.theta, -2.0 * c / HD) : 0.0;
    last_theta = a.theta;
  }
  std::copy(freq, freq + kRopePairs, a.freq);
}
// sin and cos of x in fp64, 0 <= x < 2^31 (positions times frequencies up to
// one radian, those of a base of one or more): x less the nearest multiple n of pi/2 (pi/2 as a sum of two
// doubles, each product exact in its fused multiply-add: the remainder is
// off by a rounding of its own size), then the Taylor series on [-pi/4,
// pi/4], cut where the next term is below 1e-17 of the value.  About 40 fp64
// instructions; the library's sincos, made for all arguments, took most of
// the attention kernels' prologue.  It stays for bases below one, whose
// frequencies grow to 1 / base: the angle of an ordinary position then leaves
// this range (base 1e-6: from position 4200 on), so those calls have an
// instance of the kernel of their own (wide_angles) and the others keep theirs
// as it is.
__device__ __forceinline__ double2 cos_sin(double x) {
  const double n = rint(x * 0.63661977236758134308);   // 2 / pi
  const double r = fma(-n, 6.123233995736766035869e-17, fma(-n, 1.57079632679489655800, x));
  const double z = r * r;
  double s = 1.0 / 355687428096000.0;                  // 1 / 17!
  s = fma(s, z, -1.0 / 1307674368000.0);
  s = fma(s, z, 1.0 / 6227020800.0);
  s = fma(s, z, -1.0 / 39916800.0);
  s = fma(s, z, 1.0 / 362880.0);
  s = fma(s, z, -1.0 / 5040.0);
  s = fma(s, z, 1.0 / 120.0);
  s = fma(s, z, -1.0 / 6.0);
  s = fma(s * z, r, r);
  double c = 1.0 / 20922789888000.0;                   // 1 / 16!
  c = fma(c, z, -1.0 / 87178291200.0);
  c = fma(c, z, 1.0 / 479001600.0);
  c = fma(c, z, -1.0 / 3628800.0);
  c = fma(c, z, 1.0 / 40320.0);
  c = fma(c, z, -1.0 / 720.0);
  c = fma(c, z, 1.0 / 24.0);
  c = fma(c, z, -0.5);
  c = fma(c, z, 1.0);
  const int q = static_cast<int>(n) & 3;   // quarter turns
  const double a = q & 1 ? s : c, b = q & 1 ? c : s;
  return make_double2(q == 1 || q == 2 ? -a : a, q >= 2 ? -b : b);
}

inline bool wide_angles(double theta) { return theta > 0.0 && theta < 1.0; }

// Calls put(d, c, (cos, sin)) for the angles of positions L + d, d = 0..D,
// over the workgroup.  f: thread tid's pair frequency, freq[tid % 64], loaded by the caller ahead of its bulk loads (a load issued behind
// them would wait for them).
template <bool WIDE, typename F>
__device__ __forceinline__ void rope_table(int tid, int D, int L, double f, F put) {
  const int c = tid % kRopePairs;
  for (int d = tid / kRopePairs; d <= D; d += kAttnThreads / kRopePairs) {
    const double x = (static_cast<double>(L) + static_cast<double>(d)) * f;
    if constexpr (WIDE) {
      double sn, cs;
      sincos(x, &sn, &cs);
      put(d, c, make_double2(cs, sn));
    } else {
      put(d, c, cos_sin(x));
    }
  }
}

// Turns the 8 pairs (c0 + e, c0 + e + 64), e < 8, whose halves lo / hi hold
// (bf16), by the angles at t[0 .. 7] (t = the position's table row at c0, its
// eight entries at index ^ swz, so that the lanes of a row read other banks):
// lo cos - hi sin and hi cos + lo sin in fp64 (each product rounded, then
// the sum: no fused multiply-add), each rounded to bf16 once.
__device__ __forceinline__ void rope_pairs(u32x4& lo, u32x4& hi, const double2* t, int swz) {
#pragma clang fp contract(off)
#pragma unroll
  for (int w = 0; w < 4; ++w) {
    uint32_t nl = 0u, nh = 0u;
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      const double2 a = t[(2 * w + h) ^ swz];
      const double x = bf16_to_f64(static_cast<uint16_t>(lo[w] >> (16 * h)));
      const double y = bf16_to_f64(static_cast<uint16_t>(hi[w] >> (16 * h)));
      nl |= f64_to_bf16_rne(x * a.x - y * a.y) << (16 * h);
      nh |= f64_to_bf16_rne(y * a.x + x * a.y) << (16 * h);
    }
    lo[w] = nl;
    hi[w] = nh;
  }
}

// The same turn of pairs c0 .. c0 + 7 in fp32 with fp32 angles (pair c at
// t[c ^ swz]: lanes at other depths read other banks), rounded to bf16 by the hardware
// (for the queries, which only enter bf16 products: the cache keeps the
// fp64 form's keys).  Which product is fused is spelled out, so that every
// instance of the kernel rounds alike.
__device__ __forceinline__ void rope_pairs_f32(u32x4& lo, u32x4& hi, const float2* t, int c0, int swz) {
#pragma unroll
  for (int w = 0; w < 4; ++w) {
    const float4 a = *reinterpret_cast<const float4*>(t + ((c0 + 2 * w) ^ swz));   // (swz is even)
    const float2 a0 = make_float2(a.x, a.y), a1 = make_float2(a.z, a.w);
    const float x0 = bf16_lo(lo[w]), x1 = bf16_hi(lo[w]);
    const float y0 = bf16_lo(hi[w]), y1 = bf16_hi(hi[w]);
    lo[w] = __builtin_bit_cast(uint32_t, __builtin_convertvector(
                                             (f32x2{fmaf(x0, a0.x, -(y0 * a0.y)), fmaf(x1, a1.x, -(y1 * a1.y))}), bf16x2));
    hi[w] = __builtin_bit_cast(uint32_t, __builtin_convertvector(
                                             (f32x2{fmaf(x0, a0.y, y0 * a0.x), fmaf(x1, a1.y, y1 * a1.x)}), bf16x2));
  }
}

// ---------------------------------------------------------------- attend --

// Four query tiles per workgroup, one per wave (waves past the tree's last
// tile only load).  The
// four waves walk the same key blocks, which reach LDS by direct global->LDS
// copies (no registers, no LDS stores) into a ring of kRing slots, one
// barrier per block; K and V lie there as 256-byte rows, their 16-byte chunks
// XOR-swizzled by row through the copies' source addresses.  The K Q^T
// product reads K rows as they lie; the V^T operand of the P V product comes
// from the transposing LDS read (ds_read_b64_tr_b16), four keys of one dim a
// lane.  A KV block is then read once per 128 query rows, no cross-wave merge
// is needed, and two workgroups share a CU.
constexpr int kRing = 4;
constexpr int kRingK = KB * HD * 2;          // bytes of a slot's K rows (V follows)
constexpr int kRingSlot = 2 * kRingK;        // 16 KB
constexpr int kRingLoads = kRingSlot / 16 / kAttnThreads;   // copies per thread and block

typedef short s16x4 __attribute__((ext_vector_type(4)));

// Four 16-bit elements of one column of a 4 x 16 block, the 16 lanes of a
// group holding the block's columns: lane j of the group passes the address
// of elements 4 (j % 4) .. + 3 of row j / 4 and receives column j.  (In a
// device-only function, as lds_dma16.)
__device__ __forceinline__ uint2 lds_read_tr(const uint8_t* p) {
  typedef __attribute__((address_space(3))) s16x4 lds_s16x4;
  return __builtin_bit_cast(uint2, __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4*)p));
}

// The larger of a lane's value and that of the lane 32 away.
__device__ __forceinline__ float max_halves(float x) {
  const uint32_t u = __float_as_uint(x);
  const auto r = __builtin_amdgcn_permlane32_swap(u, u, false, false);
  return fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1]));
}

// Chunk c (16 bytes) of row r of a slot lies at chunk position c ^ k_swz(r)
// (K) or c ^ v_swz(r) (V): a K fragment read takes one chunk of 16 rows, a
// transposing read 32 lanes' 64 bytes of four rows; both then cover all banks.
__device__ __forceinline__ int k_swz(int r) { return r & 15; }
__device__ __forceinline__ int v_swz(int r) { return 4 * (r & 3); }

// WIDE: the rotation's angles may pass the short sine's range (wide_angles).
template <bool WIDE>
__device__ __forceinline__ void attend_item(const BatchArgs& p, const SeqPlan& sq, int x, int tid) {
  // blockIdx -> sequence, then (kv head, split) group and query-tile group;
  // the query groups of one (head, split) land on the same XCD (dispatch is
  // round-robin over 8 XCDs and every sequence's range starts at a multiple
  // of 8), so their K/V reads share that XCD's L2.
  if (sq.T == 0) return;
  const int bid = x - sq.item0;
  const int qg = (bid >> 3) % sq.nqg;
  const int gc = ((bid >> 3) / sq.nqg) * 8 + (bid & 7);
  if (gc >= p.Hkv * sq.nsplit) return;
  const int g = gc / sq.nsplit, split = gc % sq.nsplit;
  const int T = sq.T, L = sq.L, nkeys = sq.L + sq.T, rows_pad = sq.rows_pad;
  const int nsplit = sq.nsplit;
  const int lane = tid & 63, wave = tid >> 6;
  const int li = lane & 31, lh = lane >> 5;
  const int GT = p.G * T;
  const int qt = qg * 4 + wave;           // this wave's query tile
  const bool live = qt < sq.nqt;          // (uniform per wave)

  // one LDS object per slot, so that the compiler can tell the slot being
  // read from the slots the copies in flight write to
  __shared__ __attribute__((aligned(16))) uint8_t slot0[kRingSlot];
  __shared__ __attribute__((aligned(16))) uint8_t slot1[kRingSlot];
  __shared__ __attribute__((aligned(16))) uint8_t slot2[kRingSlot];
  __shared__ __attribute__((aligned(16))) uint8_t slot3[kRingSlot];
  __shared__ uint8_t s_depth[ENTMTP_T_MAX];
  uint8_t* const ring[4] = {slot0, slot1, slot2, slot3};
  static_assert(kRing == 4, "the ring's slots");

  const size_t head_off = static_cast<size_t>(g) * p.cap * HD;
  uint16_t* const kc_head = sq.kc + head_off;
  uint16_t* const vc_head = sq.vc + head_off;
  const float c = p.scale_log2;
  const int nblocks = (nkeys + KB - 1) / KB;
  const int extra = tree_extra(nblocks, L, nsplit);
  const int blk_lo = split_begin(split, nsplit, nblocks, extra);
  const int blk_hi = split_begin(split + 1, nsplit, nblocks, extra);
  const int nb = blk_hi - blk_lo;
  const bool rope = p.theta > 0.0;
  // the first query group's workgroups keep the tree's keys (rotated) and
  // values in the cache (slots L .. L + T - 1) for the steps after this one
  const bool keeper = qg == 0;

  // the split's first np blocks lie wholly in the prefix
  const int np = max(0, min(nb, L / KB - blk_lo));

  // copies of prefix block i (past the last: that one again) into a slot:
  // instruction j of wave w fills rows 8 w + 4 j .. + 3 of K and of V, lane l
  // the chunk position l % 16 of row l / 16 among them.  The buffers span the
  // block; without a prefix block they are empty and the copies bring zeros
  // that nothing reads, so that every path carries the same count.
  const uint32_t blk_bytes = np > 0 ? kRingK : 0;
  uint32_t koff[kRingLoads / 2], voffs[kRingLoads / 2];
#pragma unroll
  for (int j = 0; j < kRingLoads / 2; ++j) {
    const int r = 4 * (wave * (kRingLoads / 2) + j) + (lane >> 4);
    koff[j] = r * 256 + (((lane & 15) ^ k_swz(r)) << 4);
    voffs[j] = r * 256 + (((lane & 15) ^ v_swz(r)) << 4);
  }
  auto gload = [&](uint8_t* slot, int i) {
    const size_t off = static_cast<size_t>(blk_lo + min(i, max(np - 1, 0))) * (KB * HD);   // (uniform)
    const __amdgpu_buffer_rsrc_t kbuf = dma_buffer(kc_head + off, blk_bytes);
    const __amdgpu_buffer_rsrc_t vbuf = dma_buffer(vc_head + off, blk_bytes);
#pragma unroll
    for (int j = 0; j < kRingLoads / 2; ++j) {
      const int r0 = 4 * (wave * (kRingLoads / 2) + j);
      buf_dma16(kbuf, koff[j], slot + r0 * 256);
      buf_dma16(vbuf, voffs[j], slot + kRingK + r0 * 256);
    }
  };

  // Blocks that hold tree keys go through registers instead: thread (row
  // tid / 8, cc = tid % 8) takes chunks cc and cc + 8 of its key and value
  // row (the two halves of pairs 8 cc .. 8 cc + 7), rotates a tree key, and
  // the keeper writes it and its value to the cache.  (In the main loop an
  // ordinary load or an LDS store would wait for every copy in flight.)
  auto tab64 = [&](int d) {   // angles at depth d (pair c at tab64_at), 16 depths a slot
    return reinterpret_cast<double2*>(d < 16 ? slot2 : slot3) + (d & 15) * kRopePairs;
  };
  static_assert(16 * kRopePairs * sizeof(double2) <= kRingSlot && ENTMTP_D_MAX < 32, "the angles fit in two slots");
  struct TreeRegs {
    u32x4 k0, k1, v0, v1;
  };
  const int trow = tid >> 3, tcc = tid & 7;
  auto tree_load = [&](TreeRegs& t, int i) {
    const int key = min((blk_lo + min(i, nb - 1)) * KB + trow, nkeys - 1);
    const size_t pre = static_cast<size_t>(key) * HD;
    const size_t own = (static_cast<size_t>(sq.row0 + key - L) * p.Hkv + g) * HD;
    const uint16_t* kp = (key < L ? kc_head + pre : p.kt + own) + 8 * tcc;
    const uint16_t* vp = (key < L ? vc_head + pre : p.vt + own) + 8 * tcc;
    t.k0 = *reinterpret_cast<const u32x4*>(kp);
    t.k1 = *reinterpret_cast<const u32x4*>(kp + HD / 2);
    t.v0 = *reinterpret_cast<const u32x4*>(vp);
    t.v1 = *reinterpret_cast<const u32x4*>(vp + HD / 2);
  };
  auto tree_stage = [&](uint8_t* slot, TreeRegs& t, int i) {
    const int key = (blk_lo + i) * KB + trow;
    if (key >= L && key < nkeys) {
      if (rope) rope_pairs(t.k0, t.k1, tab64(s_depth[key - L]) + 8 * tcc, tcc & 7);
      if (keeper) {
        uint16_t* kd = kc_head + static_cast<size_t>(key) * HD + 8 * tcc;
        uint16_t* vd = vc_head + static_cast<size_t>(key) * HD + 8 * tcc;
        *reinterpret_cast<u32x4*>(kd) = t.k0;
        *reinterpret_cast<u32x4*>(kd + HD / 2) = t.k1;
        *reinterpret_cast<u32x4*>(vd) = t.v0;
        *reinterpret_cast<u32x4*>(vd + HD / 2) = t.v1;
      }
    }
    uint8_t* const row = slot + trow * 256;
    *reinterpret_cast<u32x4*>(row + ((tcc ^ k_swz(trow)) << 4)) = t.k0;
    *reinterpret_cast<u32x4*>(row + (((tcc + 8) ^ k_swz(trow)) << 4)) = t.k1;
    *reinterpret_cast<u32x4*>(row + kRingK + ((tcc ^ v_swz(trow)) << 4)) = t.v0;
    *reinterpret_cast<u32x4*>(row + kRingK + (((tcc + 8) ^ v_swz(trow)) << 4)) = t.v1;
  };

  double freq = p.freq[tid % kRopePairs];
  TreeRegs tregs;
  if (nb > np) tree_load(tregs, np);

  // The small loads go first (this wave's Q fragments, its rows' depths and
  // masks, all unconditional: rows past the tree read row 0 and are never
  // stored): behind the key blocks they would wait for every workgroup's
  // burst.  Query row r of KV head g is (head g * G + r / T, node r % T);
  // chunks s and s + 4 hold the two halves of pairs 16s + 8lh + e.
  u32x4 qf[8];
  const int qrow = qt * kQTile + li;
  const bool qlive = qrow < GT;
  const int qnode = qlive ? qrow % T : 0;
  {
    const uint16_t* qp = p.q + (static_cast<size_t>(sq.row0 + qnode) * p.Hq + g * p.G + (qlive ? qrow / T : 0)) * HD +
                         8 * lh;
#pragma unroll
    for (int s = 0; s < 8; ++s) qf[s] = *reinterpret_cast<const u32x4*>(qp + 16 * s);
  }
  const int qdepth = sq.depth[qnode];
  const int tdepth = sq.depth[min(tid, T - 1)];
  u32x4 mlo = *reinterpret_cast<const u32x4*>(sq.mask + qnode * ENTMTP_MASK_WORDS);
  u32x4 mhi = *reinterpret_cast<const u32x4*>(sq.mask + qnode * ENTMTP_MASK_WORDS + 4);
  static_assert(ENTMTP_MASK_WORDS == 8, "a mask row is two 16-byte loads");
#pragma unroll
  for (int k = 0; k < kRing - 1; ++k) gload(ring[k], k);
  // the angles, while the blocks arrive: the queries' fp32 table lies in the
  // last slot, free until the loop's first copies
  asm volatile("" : "+v"(freq));   // (the compiler would sink its load below the copies)
  float2* const tab32 = reinterpret_cast<float2*>(slot3);
  static_assert((ENTMTP_D_MAX + 1) * kRopePairs * sizeof(float2) <= kRingSlot, "the angles fit in a slot");
  if (rope) rope_table<WIDE>(tid, sq.D, L, freq, [&](int d, int pr, double2 cs) {
    tab32[d * kRopePairs + (pr ^ (2 * (d & 31)))] = make_float2(static_cast<float>(cs.x), static_cast<float>(cs.y));
  });
  s_depth[tid] = static_cast<uint8_t>(tdepth);
  static_assert(kAttnThreads >= ENTMTP_T_MAX, "one thread per node");
  wait_lds();
  stage_barrier();
  if (!qlive) mlo = mhi = u32x4{~0u, ~0u, ~0u, ~0u};   // padding rows see every key
  if (rope) {
    const float2* tr = tab32 + qdepth * kRopePairs;
#pragma unroll
    for (int s = 0; s < 4; ++s) rope_pairs_f32(qf[s], qf[s + 4], tr, 16 * s + 8 * lh, 2 * (qdepth & 31));
  }

  // l_run: the sum of this lane's half of the keys (the halves meet at the end)
  float m_run = -INFINITY, l_run = 0.f;
  f32x16 o[4];
#pragma unroll
  for (int ct = 0; ct < 4; ++ct)
#pragma unroll
    for (int r = 0; r < 16; ++r) o[ct][r] = 0.f;

  // fragment addresses within a slot: K row li, chunk 2 s + lh; the
  // transposing reads of V: row 4 lh + (lane % 16) / 4 of each 8 rows, dims
  // 32 ct + 16 (li / 16) + 4 (lane % 4)
  const int kx = lh ^ k_swz(li);
  const int vrow = 4 * lh + ((lane & 15) >> 2);
  const int vx = (2 * ((lane >> 4) & 1) + ((lane & 3) >> 1)) ^ v_swz(vrow);
  const int voff = kRingK + vrow * 256 + 8 * (lane & 1);

  // S^T = K Q^T of the block in a slot
  auto scores = [&](const uint8_t* slot, f32x16& sacc) {
#pragma unroll
    for (int r = 0; r < 16; ++r) sacc[r] = 0.f;
#pragma unroll
    for (int s = 0; s < 8; ++s) {
      const u32x4 kf = *reinterpret_cast<const u32x4*>(slot + li * 256 + ((kx ^ (2 * s)) << 4));
      sacc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(as_bf16x8(kf), as_bf16x8(qf[s]), sacc, 0, 0, 0);
    }
  };
  // block i's softmax (lazily raised max) and
  // O^T += V^T P^T from its slot; prefix: every key of the block is visible
  auto attend = [&](int i, const uint8_t* slot, f32x16& sacc, auto prefix) {
    float bmax = -INFINITY;
    if constexpr (decltype(prefix)::value) {
#pragma unroll
      for (int r = 0; r < 16; ++r) bmax = fmaxf(bmax, sacc[r]);
    } else {
      const int kb = (blk_lo + i) * KB;
      uint32_t win = 0xFFFFFFFFu;
      const int rel = kb - L;
      auto word = [&](int w) {   // (w is uniform)
        uint32_t x = 0u;
#pragma unroll
        for (int k = 0; k < 8; ++k) x = w == k ? (k < 4 ? mlo[k & 3] : mhi[k & 3]) : x;
        return x;
      };
      if (rel < 0) {
        const int npre = -rel;
        win = (0xFFFFFFFFu >> (32 - npre)) | (mlo[0] << npre);
      } else {
        const int wi = rel >> 5, sh = rel & 31;
        const uint32_t lo = word(wi), hi = word(wi + 1);
        win = sh ? (lo >> sh) | (hi << (32 - sh)) : lo;
      }
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        const int n = 8 * (r >> 2) + 4 * lh + (r & 3);
        const bool vis = ((win >> n) & 1u) && (kb + n < nkeys);
        sacc[r] = vis ? sacc[r] : -INFINITY;
        bmax = fmaxf(bmax, sacc[r]);
      }
    }
    bmax = max_halves(bmax);
    const float mb = bmax * c;
    const bool need = mb > m_run + kLazyLog2;
    if (__any(need)) {
      const float mn = need ? mb : m_run;
      const float alpha = !need ? 1.f : (m_run == -INFINITY ? 0.f : __builtin_amdgcn_exp2f(m_run - mn));
      l_run *= alpha;
#pragma unroll
      for (int ct = 0; ct < 4; ++ct)
#pragma unroll
        for (int r = 0; r < 16; ++r) o[ct][r] *= alpha;
      m_run = mn;
    }
    const float mneg = m_run == -INFINITY ? 0.f : -m_run;
    float pr[16];
    float rsum = 0.f;
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      pr[r] = __builtin_amdgcn_exp2f(fmaf(sacc[r], c, mneg));
      rsum += pr[r];
    }
    l_run += rsum;
    bf16x8 pf[2];
#pragma unroll
    for (int u = 0; u < 2; ++u) {
      u32x4 w;
#pragma unroll
      for (int e = 0; e < 4; ++e)
        w[e] = __builtin_bit_cast(uint32_t, __builtin_convertvector(
                                               (f32x2{pr[8 * u + 2 * e], pr[8 * u + 2 * e + 1]}), bf16x2));
      pf[u] = as_bf16x8(w);
    }
#pragma unroll
    for (int ct = 0; ct < 4; ++ct) {
      const uint8_t* vp = slot + voff + ((vx ^ (4 * ct)) << 4);
#pragma unroll
      for (int u = 0; u < 2; ++u) {
        const uint2 x0 = lds_read_tr(vp + 16 * u * 256);
        const uint2 x1 = lds_read_tr(vp + (16 * u + 8) * 256);
        const u32x4 w = {x0.x, x0.y, x1.x, x1.y};
        o[ct] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(as_bf16x8(w), pf[u], o[ct], 0, 0, 0);
      }
    }
  };

  // The prefix's blocks.  Step i takes the scores of block i + 1 ahead of
  // block i's softmax, so that a wave has products to issue beside its
  // exponentials; blocks i + 2 and i + 3 are in flight, the latter's copies
  // going into the slot block i - 1 left, behind the barrier every wave
  // reaches after its products.  Copies past the last block fetch it again,
  // so the count in flight is always the same.
  f32x16 sa, sb;
  wait_vmcnt<(kRing - 2) * kRingLoads>();
  stage_barrier();
  if (live) scores(ring[0], sa);
  int i0 = 0;
  for (; i0 + kRing <= np; i0 += kRing) {
#pragma unroll
    for (int k = 0; k < kRing; ++k) {
      wait_vmcnt<(kRing - 3) * kRingLoads>();
      stage_barrier();
      gload(ring[(k + kRing - 1) % kRing], i0 + k + kRing - 1);
      if (live) {
        f32x16& cur = k & 1 ? sb : sa;
        scores(ring[(k + 1) % kRing], k & 1 ? sa : sb);
        attend(i0 + k, ring[k], cur, std::true_type{});
      }
    }
  }
  // the last np % kRing blocks are in flight (a loop left from within its
  // round would make the compiler add full waits)
  wait_vmcnt<0>();
  stage_barrier();
  if (live) {
#pragma unroll
    for (int k = 0; k < kRing - 1; ++k)
      if (i0 + k < np) {
        f32x16& cur = k & 1 ? sb : sa;
        if (k + 1 < kRing - 1) scores(ring[k + 1], k & 1 ? sa : sb);
        attend(i0 + k, ring[k], cur, std::true_type{});
      }
  }

  // the blocks that hold tree keys: staged into two of the slots in turn, the
  // next block's loads ahead of this one's products, the keys' fp64 angles in
  // the other two
  if (nb > np) {
    __syncthreads();
    if (rope) {
      rope_table<WIDE>(tid, sq.D, L, freq, [&](int d, int pr, double2 cs) { tab64(d)[pr ^ ((pr >> 3) & 7)] = cs; });
      __syncthreads();
    }
    tree_stage(slot0, tregs, np);
    for (int i = np;; i += 2) {
      tree_load(tregs, i + 1);
      __syncthreads();
      if (live) {
        scores(slot0, sa);
        attend(i, slot0, sa, std::false_type{});
      }
      if (i + 1 >= nb) break;
      tree_stage(slot1, tregs, i + 1);
      tree_load(tregs, i + 2);
      __syncthreads();
      if (live) {
        scores(slot1, sa);
        attend(i + 1, slot1, sa, std::false_type{});
      }
      if (i + 2 >= nb) break;
      tree_stage(slot0, tregs, i + 2);
    }
  }

  // this wave's tile: the output (one split) or its partial.  Lane (query li,
  // half lh) holds dims 32 ct + 8 j + 4 lh + i in o[ct][4 j + i]; the halves
  // trade a chunk so that each stores 16 bytes: lane 0..31 dims 8 j .. 8 j + 7
  // of even j, lane 32..63 of odd j.
  if (!live) return;
  l_run += __shfl_xor(l_run, 32, 64);
  const int row = qt * kQTile + li;
  uint16_t* dst;
  if (nsplit == 1) {
    const int r = row < GT ? row : 0;
    dst = p.out + (static_cast<size_t>(sq.row0 + r % T) * p.Hq + g * p.G + r / T) * HD;
  } else {
    const size_t prow = sq.part_off + (static_cast<size_t>(split) * p.Hkv + g) * rows_pad + row;
    dst = p.part_o + prow * HD;
    if (lh == 0 && row < GT) {
      p.part_ml[prow * 2 + 0] = m_run;
      p.part_ml[prow * 2 + 1] = l_run;
    }
  }
  const float il = l_run > 0.f ? 1.f / l_run : 0.f;   // 0: no key of the split is visible
  auto pack = [&](float x, float y) {
    return __builtin_bit_cast(uint32_t, __builtin_convertvector((f32x2{x * il, y * il}), bf16x2));
  };
#pragma unroll
  for (int ct = 0; ct < 4; ++ct)
#pragma unroll
    for (int j = 0; j < 4; j += 2) {
      const f32x16& a = o[ct];
      const auto x = __builtin_amdgcn_permlane32_swap(pack(a[4 * j], a[4 * j + 1]),
                                                      pack(a[4 * j + 4], a[4 * j + 5]), false, false);
      const auto y = __builtin_amdgcn_permlane32_swap(pack(a[4 * j + 2], a[4 * j + 3]),
                                                      pack(a[4 * j + 6], a[4 * j + 7]), false, false);
      if (row < GT) *reinterpret_cast<u32x4*>(dst + 32 * ct + 8 * (j + lh)) = u32x4{x[0], y[0], x[1], y[1]};
    }
}

template <bool DEVB, bool WIDE>
__global__ __launch_bounds__(kAttnThreads, 2) void tree_attn_kernel(BatchArgs p) {
  for_items<DEVB, false>(p, [&](const SeqPlan& sq, int x, int tid) { attend_item<WIDE>(p, sq, x, tid); });
}

// ----------------------------------------------------------------- merge --

// One half-wavefront per output row (kMergeRows rows per block): lane c <
// nsplit reads split c's (max, sum) and every lane then requests its four
// dims of the first kMergeBatch splits' partial outputs at once (one memory
// latency instead of one per four splits: the kernel's time was those
// rounds), the group reduces the (max, sum) pairs to the common max and the
// normalised split weights, and combines; splits past the batch follow four
// at a time.
constexpr int kMergeBatch = 16;   // splits whose partials are requested together
constexpr int kMergeThreads = 32 * kMergeRows;
static_assert(kMaxSplits <= 32, "a half-wavefront holds one lane per split");

__device__ __forceinline__ void merge_item(const BatchArgs& p, const SeqPlan& sq, int x, int tid) {
  if (sq.nsplit == 1 || sq.T == 0) return;   // written by the attend kernel, or nothing to do
  const int GT = p.G * sq.T;
  const int local = (x - sq.merge0) * kMergeRows + (tid >> 5);
  if (local >= p.Hkv * GT) return;   // past the last row (device-planned grids cover the largest tree)
  const int g = local / GT, row = local % GT;
  const int lane = tid & 31;
  const int nsplit = sq.nsplit;
  auto prow_of = [&](int c) {
    return sq.part_off + (static_cast<size_t>(c) * p.Hkv + g) * sq.rows_pad + row;
  };
  float mc = -INFINITY, lc = 0.f;
  if (lane < nsplit) {
    const float2 ml = *reinterpret_cast<const float2*>(p.part_ml + prow_of(lane) * 2);
    mc = ml.x;
    lc = ml.y;
  }
  const int d4 = 4 * lane;
  uint2 ob[kMergeBatch];
#pragma unroll
  for (int c = 0; c < kMergeBatch; ++c)
    ob[c] = *reinterpret_cast<const uint2*>(p.part_o + prow_of(min(c, nsplit - 1)) * HD + d4);
  float M = mc;
#pragma unroll
  for (int off = 16; off >= 1; off >>= 1) M = fmaxf(M, __shfl_xor(M, off, 32));
  const float w = mc == -INFINITY ? 0.f : __builtin_amdgcn_exp2f(mc - M);
  float lsum = lc * w;
#pragma unroll
  for (int off = 16; off >= 1; off >>= 1) lsum += __shfl_xor(lsum, off, 32);
  const float wn = w * lc / lsum;   // the split's share of the row
  float4 acc = make_float4(0.f, 0.f, 0.f, 0.f);
  auto add = [&](float wc, uint2 v) {
    acc.x += wc * __uint_as_float(v.x << 16);
    acc.y += wc * __uint_as_float(v.x & 0xffff0000u);
    acc.z += wc * __uint_as_float(v.y << 16);
    acc.w += wc * __uint_as_float(v.y & 0xffff0000u);
  };
#pragma unroll
  for (int c = 0; c < kMergeBatch; ++c) add(c < nsplit ? __shfl(wn, c, 32) : 0.f, ob[c]);
  for (int c0 = kMergeBatch; c0 < nsplit; c0 += 4) {   // four splits' loads in flight at a time
    uint2 o[4];
    float wc[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      const int c = min(c0 + k, nsplit - 1);
      wc[k] = c0 + k < nsplit ? __shfl(wn, c, 32) : 0.f;
      o[k] = *reinterpret_cast<const uint2*>(p.part_o + prow_of(c) * HD + d4);
    }
#pragma unroll
    for (int k = 0; k < 4; ++k) add(wc[k], o[k]);
  }
  const int gh = row / sq.T, node = row % sq.T;
  uint2 pk;
  pk.x = f32_to_bf16_rne(acc.x) | (f32_to_bf16_rne(acc.y) << 16);
  pk.y = f32_to_bf16_rne(acc.z) | (f32_to_bf16_rne(acc.w) << 16);
  *reinterpret_cast<uint2*>(p.out + (static_cast<size_t>(sq.row0 + node) * p.Hq + g * p.G + gh) * HD + d4) = pk;
}

template <bool DEVB>
__global__ __launch_bounds__(kMergeThreads) void attn_merge_kernel(BatchArgs p) {
  for_items<DEVB, true>(p, [&](const SeqPlan& sq, int x, int tid) { merge_item(p, sq, x, tid); });
}

// ------------------------------------------------------------------ host --

size_t al256(size_t x) { return (x + 255) & ~size_t(255); }

template <bool DEVB = false>
void launch_attend(const BatchArgs& a, int items, hipStream_t s) {
  auto go = [&](auto kernel) { hipLaunchKernelGGL(kernel, dim3(items), dim3(kAttnThreads), 0, s, a); };
  if (wide_angles(a.theta))
    go(tree_attn_kernel<DEVB, true>);
  else
    go(tree_attn_kernel<DEVB, false>);
}

int device_cus() {
  static int cus[64] = {0};
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) return 256;
  if (cus[dev] == 0) {
    int n = 0;
    if (hipDeviceGetAttribute(&n, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || n <= 0) n = 256;
    cus[dev] = n;
  }
  return cus[dev];
}

// Grid sizes of one call.
struct CallShape {
  int rows = 0;          // concatenated tree rows
  int items = 0;         // attend workgroups
  int merge_blocks = 0;  // merge blocks
  size_t need = 0;       // workspace bytes
};

int bank_rows(const entmtp_bank* bank) {   // nodes of the largest tree
  int T = 0;
  for (const TopoDesc& td : bank->desc) T = td.T > T ? td.T : T;
  return T;
}

// Streams a batch can have at most, whatever trees of at most `rows` rows
// together it names: a sequence's query groups number at most G T / 128 + 1.
long long streams_bound(int B, int Hkv, int G, long long rows) {
  return Hkv * (rows * G / (kTilesPerWg * kQTile) + B);
}

// Plans the sequences of one call: per-sequence split counts (a lone
// sequence fills the CUs by itself; a batch shares one blocks-per-split
// target, batch_cost), grid ranges and the packed workspace layout (output partials, then (max, sum) partials).
CallShape plan_call(const entmtp_bank* bank, int B, const int32_t* topo, const int32_t* L,
                    entmtp_bf16* const* kc, entmtp_bf16* const* vc, int cap, int Hq, int Hkv,
                    BatchArgs& a) {
  a.dev = nullptr;
  a.topos = nullptr;
  a.arena = nullptr;
  a.topo_dev = nullptr;
  a.len_dev = nullptr;
  a.row_off_dev = nullptr;
  a.B = B;
  a.G = Hq / Hkv;
  a.Hq = Hq;
  a.Hkv = Hkv;
  a.cap = cap;
  const int cus = device_cus();
  a.cus = cus;
  const int slots = cus * kWgPerCu;
  int target = 1;   // blocks per split (a batch of several)
  if (B > 1) {
    int nb[kMaxSeqs], H[kMaxSeqs], nb_max = 0;
    long long work = 0;   // key-block streams
    for (int b = 0; b < B; ++b) {
      const int T = bank->desc[topo[b]].T;
      H[b] = Hkv * query_groups(rows_padded(a.G, T) / kQTile);
      nb[b] = (L[b] + T + KB - 1) / KB;
      nb_max = nb[b] > nb_max ? nb[b] : nb_max;
      work += static_cast<long long>(H[b]) * nb[b];
    }
    // (by the bank, not the trees named: a device-planned batch decides alike)
    const bool two = two_rounds(streams_bound(B, Hkv, a.G, static_cast<long long>(B) * bank_rows(bank)), slots);
    unsigned long long best = ~0ull;
    for (int k = 0; k < kTargets; ++k) {
      if (target_sixteenths(k) < 16 && !two) continue;
      const int t = batch_target(k, work, nb_max, slots);
      long long items = 0;
      bool split = false;
      for (int b = 0; b < B; ++b) {
        const int n = batch_splits(nb[b], t);
        items += static_cast<long long>(H[b]) * n;
        split = split || n > 1;
      }
      const unsigned long long cost = batch_cost(k, t, items, split, slots);
      if (cost < best) {
        best = cost;
        target = t;
      }
    }
  }

  CallShape sh;
  long long part_rows = 0;
  for (int b = 0; b < B; ++b) {
    const TopoDesc& td = bank->desc[topo[b]];
    SeqPlan& q = a.s[b];
    q.kc = kc[b];
    q.vc = vc[b];
    q.mask = bank_ptr<uint32_t>(bank, td.off_mask);
    q.depth = bank_ptr<int>(bank, td.off_depth);
    q.T = td.T;
    q.D = td.D;
    q.L = L[b];
    q.row0 = sh.rows;
    q.rows_pad = rows_padded(a.G, q.T);
    q.nqt = q.rows_pad / kQTile;
    q.nqg = query_groups(q.nqt);
    const int nblocks = (q.L + q.T + KB - 1) / KB;
    q.nsplit = B == 1 ? split_single(nblocks, Hkv * q.nqg, cus) : batch_splits(nblocks, target);
    q.item0 = sh.items;
    q.merge0 = sh.merge_blocks;
    q.part_off = part_rows;
    sh.rows += q.T;
    sh.items += (Hkv * q.nsplit + 7) / 8 * 8 * q.nqg;
    if (q.nsplit > 1) {
      sh.merge_blocks += (Hkv * a.G * q.T + kMergeRows - 1) / kMergeRows;
      part_rows += static_cast<long long>(q.nsplit) * Hkv * q.rows_pad;
    }
  }
  const size_t po = static_cast<size_t>(part_rows) * HD * sizeof(uint16_t);
  const size_t pml = static_cast<size_t>(part_rows) * 2 * 4;
  sh.need = al256(po) + al256(pml);
  return sh;
}

// Points the planned call at its workspace and launches attend and (when
// some sequence has several splits) merge.
int32_t launch_call(BatchArgs& a, const CallShape& sh, void* workspace, hipStream_t s) {
  uint8_t* ws = static_cast<uint8_t*>(workspace);
  long long part_rows = 0;
  for (int b = 0; b < a.B; ++b)
    if (a.s[b].nsplit > 1) part_rows += static_cast<long long>(a.s[b].nsplit) * a.Hkv * a.s[b].rows_pad;
  const size_t po = static_cast<size_t>(part_rows) * HD * sizeof(uint16_t);
  a.part_o = reinterpret_cast<uint16_t*>(ws);
  a.part_ml = reinterpret_cast<float*>(ws + al256(po));
  launch_attend(a, sh.items, s);
  if (int32_t rc = launch_status("tree_attn launch")) return rc;
  if (sh.merge_blocks > 0) {
    hipLaunchKernelGGL(attn_merge_kernel<false>, dim3(sh.merge_blocks), dim3(kMergeThreads), 0, s, a);
    if (int32_t rc = launch_status("tree_attn merge launch")) return rc;
  }
  return ENTMTP_OK;
}

size_t workspace_bytes(int T, int Hq, int Hkv, int L) {
  // sized with the largest split count a plan can choose, so the figure
  // never shrinks when T or L grows
  const int G = Hq / Hkv;
  const int rows_pad = rows_padded(G, T);
  const int nblocks = (L + T + KB - 1) / KB;
  const size_t bound = split_bound(nblocks);
  return al256(bound * Hkv * rows_pad * HD * sizeof(uint16_t)) + al256(bound * Hkv * rows_pad * 2 * 4);
}

// Checks shared by the single and batched entry points.
int32_t check_common(int32_t Hq, int32_t Hkv, int32_t d, float scale, float rope_theta,
                     const void* q, const void* k_tree, const void* v_tree, const void* out,
                     const void* workspace) {
  ENTMTP_CHECK_ARG(q && k_tree && v_tree && out && workspace, ENTMTP_EINVAL,
                   "tensor and workspace pointers must be non-NULL");
  ENTMTP_CHECK_ARG(d == HD, ENTMTP_EINVAL, "head dim %d unsupported (built for %d)", d, HD);
  ENTMTP_CHECK_ARG(Hq >= 1 && Hkv >= 1, ENTMTP_EINVAL, "Hq = %d, Hkv = %d must be >= 1", Hq, Hkv);
  ENTMTP_CHECK_ARG(Hq % Hkv == 0, ENTMTP_ERANGE, "Hq = %d is not a multiple of Hkv = %d", Hq, Hkv);
  ENTMTP_CHECK_ARG(Hq / Hkv <= 32, ENTMTP_ERANGE, "query group %d too large", Hq / Hkv);
  ENTMTP_CHECK_ARG(scale > 0.f && scale < INFINITY, ENTMTP_EINVAL, "scale must be positive");
  ENTMTP_CHECK_ARG(rope_theta >= 0.f && rope_theta < INFINITY, ENTMTP_EINVAL,
                   "rope_theta must be >= 0");
  ENTMTP_CHECK_ARG(aligned16(q) && aligned16(k_tree) && aligned16(v_tree) && aligned16(out) &&
                       aligned16(workspace),
                   ENTMTP_EINVAL, "tensors and workspace must be 16-byte aligned");
  return ENTMTP_OK;
}

int32_t check_sequence(const entmtp_bank* bank, int32_t topo, int32_t prefix_len,
                       const void* kc, const void* vc, int32_t cap, int b) {
  if (int32_t rc = check_device_bank(bank, topo)) return rc;
  ENTMTP_CHECK_ARG(kc && vc && aligned16(kc) && aligned16(vc), ENTMTP_EINVAL,
                   "sequence %d: caches must be non-NULL and 16-byte aligned", b);
  ENTMTP_CHECK_ARG(prefix_len >= 0, ENTMTP_EINVAL, "sequence %d: prefix_len = %d < 0", b,
                   prefix_len);
  const int T = bank->desc[topo].T;
  ENTMTP_CHECK_ARG(static_cast<int64_t>(prefix_len) + T <= cap, ENTMTP_ERANGE,
                   "sequence %d: cache capacity %d below prefix_len + T = %d", b, cap,
                   prefix_len + T);
  return ENTMTP_OK;
}

}  // namespace

int32_t attn_device_shape(const entmtp_bank* bank, int Hq, int Hkv, int cap, DevAttnShape* out) {
  const int cus = device_cus();
  const int G = Hq / Hkv;
  DevAttnShape sh;
  for (const TopoDesc& td : bank->desc) {
    sh.T_max = td.T > sh.T_max ? td.T : sh.T_max;
    const int nqg = query_groups(rows_padded(G, td.T) / kQTile);
    const int max_blocks = (cap + KB - 1) / KB;
    for (int nblocks = 1; nblocks <= max_blocks; ++nblocks) {
      const int ns = split_single(nblocks, Hkv * nqg, cus);
      const int items = (Hkv * ns + 7) / 8 * 8 * nqg;
      sh.items = items > sh.items ? items : sh.items;
    }
  }
  sh.rows = sh.T_max;
  sh.merge_blocks = (Hkv * G * sh.T_max + kMergeRows - 1) / kMergeRows;
  sh.need = workspace_bytes(sh.T_max, Hq, Hkv, cap);
  *out = sh;
  return ENTMTP_OK;
}

void attn_device_splits(const entmtp_bank* bank, int Hq, int Hkv, DevTopo* topos) {
  const int cus = device_cus();
  const int G = Hq / Hkv;
  for (size_t k = 0; k < bank->desc.size(); ++k) {
    const int nqg = query_groups(rows_padded(G, bank->desc[k].T) / kQTile);
    topos[k].splits[0] = 1;
    for (int b = 1; b <= kMaxSplits; ++b)
      topos[k].splits[b] = static_cast<unsigned char>(split_for_bound(b, Hkv * nqg, cus * kWgPerCu));
  }
}

int32_t launch_attn_device(const entmtp_bank* bank, const DevStep* dev, const DevTopo* topos,
                           const DevAttnShape& sh, const entmtp_bf16* q, const entmtp_bf16* k_tree,
                           const entmtp_bf16* v_tree, entmtp_bf16* k_cache, entmtp_bf16* v_cache,
                           int cap, int Hq, int Hkv, float scale, float rope_theta,
                           entmtp_bf16* out, void* workspace, hipStream_t s) {
  BatchArgs a{};
  a.dev = dev;
  a.topos = topos;
  a.arena = bank->arena;
  a.cus = device_cus();
  a.B = 1;
  a.G = Hq / Hkv;
  a.Hq = Hq;
  a.Hkv = Hkv;
  a.cap = cap;
  a.s[0].kc = k_cache;
  a.s[0].vc = v_cache;
  a.scale_log2 = scale * 1.4426950408889634f;
  set_rope(a, rope_theta);
  a.q = q;
  a.kt = k_tree;
  a.vt = v_tree;
  a.out = out;
  // the workspace regions at the bounds workspace_bytes() sizes them with
  const int rows_pad = rows_padded(a.G, sh.T_max);
  const size_t bound = split_bound((cap + sh.T_max + KB - 1) / KB);
  const size_t po = bound * Hkv * rows_pad * HD * sizeof(uint16_t);
  uint8_t* ws = static_cast<uint8_t*>(workspace);
  a.part_o = reinterpret_cast<uint16_t*>(ws);
  a.part_ml = reinterpret_cast<float*>(ws + al256(po));
  launch_attend(a, sh.items, s);
  if (int32_t rc = launch_status("tree_attn launch")) return rc;
  hipLaunchKernelGGL(attn_merge_kernel<false>, dim3(sh.merge_blocks), dim3(kMergeThreads), 0, s, a);
  return launch_status("tree_attn merge launch");
}

// What the host fixes of a device-planned batch: grids that cover every plan
// the device can make (of sequences with rows of their own: for_items), and
// per-sequence partial ranges sized for the largest plan any bank tree can need
// at prefix lengths up to cap - T.
struct BatchDevShape {
  int items = 0;             // attend workgroups
  int merge_blocks = 0;
  bool two = false;          // two-round candidates allowed (two_rounds)
  long long part_rows = 0;   // partial rows per sequence
  size_t need = 0;           // workspace bytes for B sequences
};

BatchDevShape batch_dev_shape(const entmtp_bank* bank, int B, int Hq, int Hkv, int cap, int rows_cap) {
  BatchDevShape sh;
  const int G = Hq / Hkv;
  const int slots = device_cus() * kWgPerCu;
  const int bound = split_bound((cap + KB - 1) / KB);
  const int T_max = bank_rows(bank);
  sh.two = two_rounds(streams_bound(B, Hkv, G, static_cast<long long>(B) * T_max), slots);
  // tree rows of the batch, where no two sequences share one
  const long long rows = std::min<long long>(rows_cap, static_cast<long long>(B) * T_max);
  const long long streams = streams_bound(B, Hkv, G, rows);
  // items of a batch: at most work / t + streams (t at least half the even
  // share with two rounds, else the whole of it), or every sequence at its
  // bound; the padding of a (KV head, split) range to eight adds up to seven
  // workgroups per query group
  const long long groups = rows * G / (kTilesPerWg * kQTile) + B;
  const int nqg = query_groups(rows_padded(G, T_max) / kQTile);
  const long long most = B == 1 ? static_cast<long long>(Hkv) * bound * nqg
                                : (sh.two ? 2LL : 1LL) * slots + streams;
  const long long all = static_cast<long long>(B) * ((Hkv * bound + 7) / 8 * 8) * nqg;
  sh.items = static_cast<int>(std::min(most + 7 * groups, all));
  // merge blocks: a row of Hq heads per tree row, kMergeRows to a block
  sh.merge_blocks = static_cast<int>(rows * Hq / kMergeRows + B);
  sh.part_rows = static_cast<long long>(bound) * Hkv * rows_padded(G, T_max);
  const size_t prows = static_cast<size_t>(B) * sh.part_rows;
  sh.need = al256(prows * HD * sizeof(uint16_t)) + al256(prows * 2 * 4);
  return sh;
}

}  // namespace entmtp

// Workspace of entmtp_tree_attn_noalloc, for callers that cannot allocate:
// one array per device, held until the process ends.  Host code never
// passes `scratch` itself to a kernel (in host code the name is a host-side
// stand-in): it takes the device address looked up below.
static __device__ __align__(256) uint8_t scratch[ENTMTP_NOALLOC_SCRATCH_BYTES];

namespace {

constexpr int kMaxScratchDevices = 64;
std::mutex g_scratch_mu;
void* g_scratch_dev[kMaxScratchDevices] = {};

// Device address of `scratch` on the current device, looked up (with that
// device current) the first time a call runs on it.
int32_t scratch_address(void** out) {
  int dev = -1;
  if (int32_t rc = entmtp::hip_status(hipGetDevice(&dev), "hipGetDevice")) return rc;
  ENTMTP_CHECK_ARG(dev >= 0 && dev < kMaxScratchDevices, ENTMTP_EINVAL,
                   "device %d outside the %d devices the static scratch is tracked for", dev,
                   kMaxScratchDevices);
  std::lock_guard<std::mutex> lock(g_scratch_mu);
  if (g_scratch_dev[dev] == nullptr) {
    void* p = nullptr;
    if (int32_t rc = entmtp::hip_status(hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)),
                                        "hipGetSymbolAddress (static scratch)"))
      return rc;
    ENTMTP_CHECK_ARG(p != nullptr, ENTMTP_EHIP, "hipGetSymbolAddress returned NULL for the scratch");
    g_scratch_dev[dev] = p;
  }
  *out = g_scratch_dev[dev];
  return ENTMTP_OK;
}

}  // namespace

using namespace entmtp;

extern "C" size_t entmtp_tree_attn_workspace(int32_t T, int32_t Hq, int32_t Hkv, int32_t d,
                                             int32_t prefix_len) {
  if (T < 1 || T > ENTMTP_T_MAX || Hq < 1 || Hkv < 1 || Hq % Hkv || d != HD || prefix_len < 0)
    return 0;
  return workspace_bytes(T, Hq, Hkv, prefix_len);
}

extern "C" size_t entmtp_tree_attn_batched_workspace(int32_t B, int32_t T_max, int32_t Hq,
                                                     int32_t Hkv, int32_t d,
                                                     int32_t max_prefix_len) {
  if (B < 1 || B > ENTMTP_B_MAX) return 0;
  return static_cast<size_t>(B) * entmtp_tree_attn_workspace(T_max, Hq, Hkv, d, max_prefix_len);
}

extern "C" int32_t entmtp_tree_attn(const entmtp_bank* bank, int32_t topo, const entmtp_bf16* q,
                                    const entmtp_bf16* k_tree, const entmtp_bf16* v_tree,
                                    entmtp_bf16* k_cache, entmtp_bf16* v_cache, int32_t cap,
                                    int32_t prefix_len, int32_t Hq, int32_t Hkv, int32_t d,
                                    float scale, float rope_theta, entmtp_bf16* out,
                                    void* workspace, size_t ws_bytes, void* stream) {
  clear_error();
  if (int32_t rc = check_sequence(bank, topo, prefix_len, k_cache, v_cache, cap, 0)) return rc;
  if (int32_t rc = check_common(Hq, Hkv, d, scale, rope_theta, q, k_tree, v_tree, out, workspace))
    return rc;
  const int T = bank->desc[topo].T;
  ENTMTP_CHECK_ARG(ws_bytes >= workspace_bytes(T, Hq, Hkv, prefix_len), ENTMTP_ENOSPC,
                   "workspace has %zu bytes, needs %zu", ws_bytes,
                   workspace_bytes(T, Hq, Hkv, prefix_len));
  BatchArgs a;
  const CallShape sh = plan_call(bank, 1, &topo, &prefix_len, &k_cache, &v_cache, cap, Hq, Hkv, a);
  a.scale_log2 = scale * 1.4426950408889634f;
  set_rope(a, rope_theta);
  a.q = q;
  a.kt = k_tree;
  a.vt = v_tree;
  a.out = out;
  return launch_call(a, sh, workspace, static_cast<hipStream_t>(stream));
}

extern "C" int32_t entmtp_tree_attn_noalloc(const entmtp_bank* bank, int32_t topo,
                                            const entmtp_bf16* q, const entmtp_bf16* k_tree,
                                            const entmtp_bf16* v_tree, entmtp_bf16* k_cache,
                                            entmtp_bf16* v_cache, int32_t cap, int32_t prefix_len,
                                            int32_t Hq, int32_t Hkv, int32_t d, float scale,
                                            float rope_theta, entmtp_bf16* out, void* stream) {
  clear_error();
  if (int32_t rc = check_sequence(bank, topo, prefix_len, k_cache, v_cache, cap, 0)) return rc;
  // (the workspace check of check_common is met by the static array)
  if (int32_t rc = check_common(Hq, Hkv, d, scale, rope_theta, q, k_tree, v_tree, out, scratch))
    return rc;
  const int T = bank->desc[topo].T;
  // the bound entmtp_tree_attn_workspace() states covers every plan of the
  // call, so an accepted call stays inside the array
  const size_t need = workspace_bytes(T, Hq, Hkv, prefix_len);
  ENTMTP_CHECK_ARG(need <= ENTMTP_NOALLOC_SCRATCH_BYTES, ENTMTP_ENOSPC,
                   "the call needs %zu bytes of workspace, the static scratch holds %zu", need,
                   static_cast<size_t>(ENTMTP_NOALLOC_SCRATCH_BYTES));
  void* ws = nullptr;
  if (int32_t rc = scratch_address(&ws)) return rc;
  BatchArgs a;
  const CallShape sh = plan_call(bank, 1, &topo, &prefix_len, &k_cache, &v_cache, cap, Hq, Hkv, a);
  a.scale_log2 = scale * 1.4426950408889634f;
  set_rope(a, rope_theta);
  a.q = q;
  a.kt = k_tree;
  a.vt = v_tree;
  a.out = out;
  return launch_call(a, sh, ws, static_cast<hipStream_t>(stream));
}

extern "C" int32_t entmtp_tree_attn_batched(
    const entmtp_bank* bank, int32_t B, const int32_t* topo, const int32_t* prefix_len,
    const entmtp_bf16* q, const entmtp_bf16* k_tree, const entmtp_bf16* v_tree,
    entmtp_bf16* const* k_caches, entmtp_bf16* const* v_caches, int32_t cap, int32_t Hq,
    int32_t Hkv, int32_t d, float scale, float rope_theta, entmtp_bf16* out, void* workspace,
    size_t ws_bytes, void* stream) {
  clear_error();
  ENTMTP_CHECK_ARG(B >= 1 && B <= ENTMTP_B_MAX, ENTMTP_EINVAL, "B = %d outside [1, %d]", B,
                   ENTMTP_B_MAX);
  ENTMTP_CHECK_ARG(topo && prefix_len && k_caches && v_caches, ENTMTP_EINVAL,
                   "topo, prefix_len, k_caches and v_caches must be non-NULL host arrays");
  for (int b = 0; b < B; ++b)
    if (int32_t rc = check_sequence(bank, topo[b], prefix_len[b], k_caches[b], v_caches[b], cap, b))
      return rc;
  if (int32_t rc = check_common(Hq, Hkv, d, scale, rope_theta, q, k_tree, v_tree, out, workspace))
    return rc;
  BatchArgs a;
  const CallShape sh = plan_call(bank, B, topo, prefix_len, k_caches, v_caches, cap, Hq, Hkv, a);
  ENTMTP_CHECK_ARG(ws_bytes >= sh.need, ENTMTP_ENOSPC, "workspace has %zu bytes, needs %zu",
                   ws_bytes, sh.need);
  a.scale_log2 = scale * 1.4426950408889634f;
  set_rope(a, rope_theta);
  a.q = q;
  a.kt = k_tree;
  a.vt = v_tree;
  a.out = out;
  return launch_call(a, sh, workspace, static_cast<hipStream_t>(stream));
}

extern "C" size_t entmtp_tree_attn_batched_device_workspace(const entmtp_bank* bank, int32_t B,
                                                            int32_t Hq, int32_t Hkv, int32_t d,
                                                            int32_t cap) {
  if (!bank || bank->desc.empty() || B < 1 || B > ENTMTP_B_MAX || Hq < 1 || Hkv < 1 ||
      Hq % Hkv || d != HD || cap < 1)
    return 0;
  return batch_dev_shape(bank, B, Hq, Hkv, cap, 1).need;   // (not a matter of the rows)
}

extern "C" int32_t entmtp_tree_attn_batched_device(
    const entmtp_bank* bank, int32_t B, const int32_t* topo, const int32_t* prefix_len,
    const int32_t* row_off, int32_t rows_cap, const entmtp_bf16* q, const entmtp_bf16* k_tree,
    const entmtp_bf16* v_tree, entmtp_bf16* const* k_caches, entmtp_bf16* const* v_caches,
    int32_t cap, int32_t Hq, int32_t Hkv, int32_t d, float scale, float rope_theta,
    entmtp_bf16* out, void* workspace, size_t ws_bytes, void* stream) {
  clear_error();
  ENTMTP_CHECK_ARG(B >= 1 && B <= ENTMTP_B_MAX, ENTMTP_EINVAL, "B = %d outside [1, %d]", B,
                   ENTMTP_B_MAX);
  if (int32_t rc = check_device_bank(bank, 0)) return rc;
  ENTMTP_CHECK_ARG(static_cast<int>(bank->desc.size()) <= kMaxTreesArg, ENTMTP_ERANGE,
                   "a device-planned batch names at most %d bank trees (bank has %zu)",
                   kMaxTreesArg, bank->desc.size());
  ENTMTP_CHECK_ARG(topo && prefix_len && row_off, ENTMTP_EINVAL,
                   "topo, prefix_len and row_off must be non-NULL device arrays");
  ENTMTP_CHECK_ARG(k_caches && v_caches, ENTMTP_EINVAL,
                   "k_caches and v_caches must be non-NULL host arrays");
  ENTMTP_CHECK_ARG(rows_cap >= 1, ENTMTP_EINVAL, "rows_cap = %d < 1", rows_cap);
  ENTMTP_CHECK_ARG(cap >= 1, ENTMTP_EINVAL, "cap = %d < 1", cap);
  for (int b = 0; b < B; ++b)
    ENTMTP_CHECK_ARG(k_caches[b] && v_caches[b] && aligned16(k_caches[b]) && aligned16(v_caches[b]),
                     ENTMTP_EINVAL, "sequence %d: caches must be non-NULL and 16-byte aligned", b);
  if (int32_t rc = check_common(Hq, Hkv, d, scale, rope_theta, q, k_tree, v_tree, out, workspace))
    return rc;
  const BatchDevShape sh = batch_dev_shape(bank, B, Hq, Hkv, cap, rows_cap);
  ENTMTP_CHECK_ARG(ws_bytes >= sh.need, ENTMTP_ENOSPC, "workspace has %zu bytes, needs %zu",
                   ws_bytes, sh.need);
  BatchArgs a{};
  a.topo_dev = topo;
  a.len_dev = prefix_len;
  a.row_off_dev = row_off;
  a.rows_cap = rows_cap;
  a.n_trees = static_cast<int>(bank->desc.size());
  for (int k = 0; k < a.n_trees; ++k) {
    const TopoDesc& td = bank->desc[k];
    ENTMTP_CHECK_ARG(td.off_mask <= INT32_MAX && td.off_depth <= INT32_MAX, ENTMTP_ERANGE,
                     "bank arena offsets past 2 GiB");
    a.trees[k] = TreeHdr{td.T, td.D, static_cast<int>(td.off_mask), static_cast<int>(td.off_depth)};
  }
  a.arena = bank->arena;
  a.cus = device_cus();
  a.B = B;
  a.G = Hq / Hkv;
  a.Hq = Hq;
  a.Hkv = Hkv;
  a.cap = cap;
  a.scale_log2 = scale * 1.4426950408889634f;
  set_rope(a, rope_theta);
  a.q = q;
  a.kt = k_tree;
  a.vt = v_tree;
  a.out = out;
  const size_t rows = static_cast<size_t>(B) * sh.part_rows;
  uint8_t* ws = static_cast<uint8_t*>(workspace);
  a.part_o = reinterpret_cast<uint16_t*>(ws);
  a.part_ml = reinterpret_cast<float*>(ws + al256(rows * HD * sizeof(uint16_t)));
  for (int b = 0; b < B; ++b) {
    a.s[b].kc = k_caches[b];
    a.s[b].vc = v_caches[b];
    a.s[b].part_off = b * sh.part_rows;
  }
  const hipStream_t s = static_cast<hipStream_t>(stream);
  a.two_rounds = sh.two;
  launch_attend<true>(a, sh.items, s);
  if (int32_t rc = launch_status("tree_attn (device-planned batch) launch")) return rc;
  hipLaunchKernelGGL(attn_merge_kernel<true>, dim3(sh.merge_blocks), dim3(kMergeThreads), 0, s, a);
  return launch_status("tree_attn (device-planned batch) merge launch");
}

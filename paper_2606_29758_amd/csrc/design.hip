// Cutoff design of PS-PPO ("Computing xi" of Algorithm 1; Sec. 3.3, App. E, F).
//
// Weights.  For prompt p (completions r = pK .. pK+K-1, lengths T_r,
// T_p = max_r T_r) and step t = 1..T_p, over the n_t completions alive at t
// (T_r >= t):
//   gbar_t = (1/n_t) sum_r gamma_r(t)                 (output-head score proxy, App. D)
//   u_t    = 1/2 - 1/(2 n_t) || sum_{r in G_t} pi_r(.|t) - sum_{r in B_t} pi_r(.|t) ||_1
//            (reward-uncertainty proxy, App. E, with p = |G_t|/n_t; G_t / B_t the
//            successful / unsuccessful completions)
//   w_t    = gbar_t u_t.
// Each pi_r(.|t) is given by its top-k entries (token id, log-prob); the mass
// left outside them is one further coordinate shared by every completion.
//
// Design.  Per prompt, minimise sum_t w_t / xi_t subject to sum_t xi_t = B and
// 1 >= xi_1 >= ... >= xi_T > 0 (Eq. design_problem): Pooling Adjacent
// Violators builds contiguous blocks with non-increasing scores
// s_m = sqrt(W_m / L_m) (App. F); the optimum is xi = min(1, kappa s_m), the
// cap saturating a prefix of blocks and kappa spending the rest of the budget
// on the others.  Variants: Heuristic (the unconstrained closed form
// B sqrt(w_t) / sum_j sqrt(w_j), capped, then a running minimum), Uniform
// (H uniform on 1..T) and Time prior (xi_t = exp(-lambda (t-1))).  Every xi is
// floored at 2^-32, the resolution of the sampler's thresholds.
//
// Both kernels work in float64.
#include <cmath>
#include <mutex>
#include <string>

#include "common.h"

namespace pspo {
namespace {

constexpr int kDesignMaxEntries = 256;   // K * topk per step
constexpr double kXiFloor = 0x1p-32;

__device__ __forceinline__ double wave_sum(double v) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o);
  return v;
}

// Sum over groups of G consecutive lanes (all lanes active; every lane of a
// group gets it): lane exchanges inside 16-lane rows as DPP moves.
template <int kCtrl>
__device__ __forceinline__ double dpp(double v) {
  const uint64_t u = __builtin_bit_cast(uint64_t, v);
  const uint32_t lo = (uint32_t)__builtin_amdgcn_mov_dpp((int)(uint32_t)u, kCtrl, 0xF, 0xF, true);
  const uint32_t hi = (uint32_t)__builtin_amdgcn_mov_dpp((int)(uint32_t)(u >> 32), kCtrl, 0xF, 0xF, true);
  return __builtin_bit_cast(double, (uint64_t)hi << 32 | lo);
}
template <int G>
__device__ __forceinline__ double group_sum(double v) {
  static_assert(G >= 4 && G <= 64, "groups of 4 to 64 lanes");
  v += dpp<0xB1>(v);                      // lane ^ 1
  v += dpp<0x4E>(v);                      // lane ^ 2
  if constexpr (G >= 8) v += dpp<0x141>(v);    // the other quad of the half row (mirrored)
  if constexpr (G >= 16) v += dpp<0x140>(v);   // the other half of the row (mirrored)
  if constexpr (G >= 32) v += __shfl_xor(v, 16);
  if constexpr (G >= 64) v += __shfl_xor(v, 32);
  return v;
}

__device__ __forceinline__ double lane_value(double x, int lane) {
  const uint64_t u = __builtin_bit_cast(uint64_t, x);
  const uint32_t lo = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)u, lane);
  const uint32_t hi = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(u >> 32), lane);
  return __builtin_bit_cast(double, (uint64_t)hi << 32 | lo);
}

// The prompt of step g: the last p with xi_off[p] <= g (0 if none).  Called by a
// whole wave whose steps are first + (lane * kSteps / 64).  Up to 64 prompts: one
// load, and the offsets are counted by a ballot for each of the wave's steps (a
// binary search is a chain of loads, and a wave's time in the weights' kernels is
// mostly load latency).
template <int kSteps>
__device__ __forceinline__ int prompt_of(const int64_t* __restrict__ xi_off, int P, int64_t total, int64_t first) {
  const int lane = threadIdx.x & 63, mine = lane / (64 / kSteps);
  int lo = 0;
  if (P <= 64) {
    const int64_t off = lane < P ? xi_off[lane] : INT64_MAX;
    for (int s = 0; s < kSteps; ++s) {
      const int before = __popcll(__ballot(off <= first + s));
      if (mine == s) lo = max(before - 1, 0);
    }
  } else {
    const int64_t g = first + mine;
    int hi = P - 1;
    while (g < total && lo < hi) {
      const int mid = (lo + hi + 1) >> 1;
      if (xi_off[mid] <= g) lo = mid;
      else hi = mid - 1;
    }
  }
  return lo;
}

// The outputs of step g from its sums over the alive completions.
__device__ __forceinline__ void write_weight(int64_t g, double gsum, double nalive, double nsucc, double l1,
                                             double rest, double* __restrict__ w, double* __restrict__ gbar_out,
                                             double* __restrict__ u_out, int32_t* __restrict__ err_flag) {
  if (nalive == 0.0) {   // the table is longer than every completion of the prompt
    if (err_flag) atomicOr(err_flag, PSPO_DEVERR_BAD_XI);
    w[g] = NAN;
    return;
  }
  const double gb = gsum / nalive;
  // equal rewards among the alive completions: p is 0 or 1 and the norm is exactly 1,
  // so u = 0 (taken exactly); otherwise ||.||_1 <= 1 by the triangle inequality, so
  // u >= 0 and rounding below it is clamped
  const double u = (nsucc == 0.0 || nsucc == nalive) ? 0.0 : fmax(0.0, 0.5 - 0.5 * (l1 + fabs(rest)) / nalive);
  w[g] = gb * u;
  if (gbar_out) gbar_out[g] = gb;
  if (u_out) u_out[g] = u;
}

// The weights: a group of G lanes (a power of two >= topk, up to 64) per
// (prompt, step), 64 / G steps per one-wave block.  The completions are taken
// in order; each entry of a completion's list finds its token id's slot in a
// hash table of the step in LDS (open addressing, at most half full) and adds
// its signed probability there, so every id's terms are added in the order of the
// completions; the entries of kListsAhead completions are read together.  Two orders
// rest on the wave, whose LDS atomics the hardware carries out lane by lane, always in
// the same order, and on the table being this wave's alone: which of two new ids of
// one list that meet in a slot takes it (the final sum goes through the slots), and
// the terms of an id that one list holds twice.  So a call repeats its bits.  One wave
// per step compared every entry with every other one from LDS, and 8 of its lanes
// summed the lists' masses with an exp per entry of their own: 160 us for 35,000
// steps of 8 top-16 lists (19 MB of lists), 26 us now.
constexpr int kListsAhead = 4;
template <int G>
__global__ __launch_bounds__(64) void design_weights_kernel(
    const float* __restrict__ gamma, const int32_t* __restrict__ topk_ids, const float* __restrict__ topk_logp,
    int topk, const int32_t* __restrict__ lengths, const int32_t* __restrict__ full_off,
    const float* __restrict__ rewards, const int64_t* __restrict__ xi_off, int P, int K, int64_t total, int slots,
    double* __restrict__ w, double* __restrict__ gbar_out, double* __restrict__ u_out, int32_t* __restrict__ err_flag) {
  extern __shared__ __attribute__((aligned(16))) unsigned char lds[];
  constexpr int kSteps = 64 / G;
  const int lane = threadIdx.x, e = lane % G;
  double* all_sums = reinterpret_cast<double*>(lds);                       // [steps][slots]
  int32_t* all_ids = reinterpret_cast<int32_t*>(lds + (int64_t)kSteps * slots * 8);
  for (int i = lane; i < kSteps * slots; i += 64) {
    all_sums[i] = 0.0;
    all_ids[i] = -1;
  }
  double* sums = all_sums + lane / G * slots;
  int32_t* ids = all_ids + lane / G * slots;
  const int shift = __builtin_clz(slots) + 1;   // a hash's top log2(slots) bits
  const int64_t g = (int64_t)blockIdx.x * kSteps + lane / G;
  const bool live = g < total;
  const int p = prompt_of<kSteps>(xi_off, P, total, (int64_t)blockIdx.x * kSteps);
  const int t = live ? (int)(g - xi_off[p]) + 1 : 0;
  __syncthreads();

  double rest = 0.0, gsum = 0.0, nalive = 0.0, nsucc = 0.0;
  for (int k0 = 0; k0 < K; k0 += G) {
    // lane e: the row of completion k0 + e at this step (-1: not alive) and its sign
    int64_t row = -1;
    bool succ = false;
    if (live && k0 + e < K) {
      const int r = p * K + k0 + e;
      const int len = lengths[r], first = full_off[r];   // (loaded together)
      const float reward = rewards[r];
      if (len >= t) {
        row = (int64_t)first + t - 1;
        succ = reward > 0.5f;
        gsum += (double)gamma[row];
        nalive += 1.0;
        nsucc += succ ? 1.0 : 0.0;
      }
    }
    const int kn = min(G, K - k0);
    for (int kb = 0; kb < kn; kb += kListsAhead) {
      int64_t rows[kListsAhead];
      int32_t list_id[kListsAhead];
      float list_lp[kListsAhead];
#pragma unroll
      for (int q = 0; q < kListsAhead; ++q) {
        rows[q] = __shfl(row, min(kb + q, kn - 1), G);
        if (kb + q >= kn) rows[q] = -1;
        const bool on = rows[q] >= 0 && e < topk;
        list_id[q] = on ? topk_ids[rows[q] * topk + e] : -1;
        list_lp[q] = on ? topk_logp[rows[q] * topk + e] : 0.f;
      }
#pragma unroll
      for (int q = 0; q < kListsAhead; ++q) {
        const int64_t now = rows[q];
        int32_t id = list_id[q];
        float lp = list_lp[q];
        const double sign = __shfl((int)succ, min(kb + q, kn - 1), G) ? 1.0 : -1.0;
        double mass = 0.0;
        if (now >= 0) {
          for (int e1 = e;;) {
            if (e1 < topk) {
              const double pr = exp((double)lp);
              mass += pr;
              if (id >= 0) {
                int slot = (int)((uint32_t)id * 0x9E3779B1u >> shift);
                for (;;) {           // ends: the table has more slots than entries
                  const int32_t old = atomicCAS(&ids[slot], -1, id);
                  if (old == -1 || old == id) break;
                  slot = (slot + 1) & (slots - 1);
                }
                unsafeAtomicAdd(&sums[slot], sign * pr);   // (one row's ids may repeat)
              }
            }
            e1 += G;
            if (e1 - e >= topk) break;
            if (e1 < topk) {         // lists longer than a wave
              id = topk_ids[now * topk + e1];
              lp = topk_logp[now * topk + e1];
            }
          }
        }
        mass = group_sum<G>(mass);
        if (now >= 0) rest += sign * fmax(0.0, 1.0 - mass);
      }
    }
  }
  __syncthreads();
  double l1 = 0.0;
  for (int i = e; i < slots; i += G) l1 += fabs(sums[i]);
  l1 = group_sum<G>(l1);
  gsum = group_sum<G>(gsum);
  nalive = group_sum<G>(nalive);
  nsucc = group_sum<G>(nsucc);
  if (live && e == 0) write_weight(g, gsum, nalive, nsucc, l1, rest, w, gbar_out, u_out, err_flag);
}

// The weights where many lists have few entries: a wave per step, entry j = k topk + i
// of its K lists in lane j % 64 (E entries a lane), the entries of an id found by a
// ballot: the order of every sum is that of the entries.
template <int E>
__global__ __launch_bounds__(64) void design_weights_short_kernel(
    const float* __restrict__ gamma, const int32_t* __restrict__ topk_ids, const float* __restrict__ topk_logp,
    int topk, const int32_t* __restrict__ lengths, const int32_t* __restrict__ full_off,
    const float* __restrict__ rewards, const int64_t* __restrict__ xi_off, int P, int K, int64_t total,
    double* __restrict__ w, double* __restrict__ gbar_out, double* __restrict__ u_out, int32_t* __restrict__ err_flag) {
  const int lane = threadIdx.x;
  const int64_t g = blockIdx.x;
  const int p = prompt_of<1>(xi_off, P, total, g);
  const int t = (int)(g - xi_off[p]) + 1;
  // lane k: the row of completion k at this step (-1: not alive)
  int64_t row = -1;
  double gsum = 0.0;
  bool succ = false;
  if (lane < K) {
    const int r = p * K + lane;
    const int len = lengths[r], first = full_off[r];
    const float reward = rewards[r];
    if (len >= t) {
      row = (int64_t)first + t - 1;
      gsum = (double)gamma[row];
      succ = reward > 0.5f;
    }
  }
  const uint64_t alive = __ballot(row >= 0), good = __ballot(succ);
  const int ne = K * topk;
  int32_t id[E];
  double pr[E], v[E];
#pragma unroll
  for (int u = 0; u < E; ++u) {
    const int j = lane + 64 * u, k = min(j / topk, 63);
    const int64_t from = __shfl(row, k);
    const bool on = j < ne && from >= 0;
    id[u] = on ? topk_ids[from * topk + (j - k * topk)] : -1;
    pr[u] = on ? exp((double)topk_logp[from * topk + (j - k * topk)]) : 0.0;
    v[u] = good >> k & 1 ? pr[u] : -pr[u];
  }
  // lane k: the mass outside its completion's list
  double mass = 0.0;
  for (int i = 0; i < topk; ++i) {
    const int j = lane * topk + i;
    double x = __shfl(pr[0], j & 63);
    if constexpr (E > 1) {
      const double y = __shfl(pr[1], j & 63);
      x = j < 64 ? x : y;
    }
    mass += x;
  }
  double rest = row >= 0 ? (succ ? 1.0 : -1.0) * fmax(0.0, 1.0 - mass) : 0.0;
  // each distinct id once: an id of one entry is that entry's value already; the
  // values of a repeated one are added in the order of the entries, for its first
  double sum[E];
  uint64_t left[E];
#pragma unroll
  for (int u = 0; u < E; ++u) {
    sum[u] = id[u] >= 0 ? v[u] : 0.0;
    left[u] = __ballot(id[u] >= 0);
  }
#pragma unroll
  for (int q = 0; q < E; ++q) {
    while (left[q] != 0) {
      const int i = __builtin_ctzll(left[q]);
      const int32_t other = __builtin_amdgcn_readlane(id[q], i);
      uint64_t same[E];
      int n = 0;
#pragma unroll
      for (int u = 0; u < E; ++u) {
        same[u] = __ballot(id[u] == other);
        left[u] &= ~same[u];
        n += __popcll(same[u]);
      }
      if (n == 1) continue;   // uniform over the wave
      double x = 0.0;
#pragma unroll
      for (int u = 0; u < E; ++u) {
        for (uint64_t m = same[u]; m != 0; m &= m - 1) x += lane_value(v[u], __builtin_ctzll(m));
        if (id[u] == other) sum[u] = 0.0;
      }
      if (lane == i) sum[q] = x;
    }
  }
  double l1 = 0.0;
#pragma unroll
  for (int u = 0; u < E; ++u) l1 += fabs(sum[u]);
  l1 = wave_sum(l1);
  rest = wave_sum(rest);
  gsum = wave_sum(gsum);
  if (lane == 0)
    write_weight(g, gsum, (double)__popcll(alive), (double)__popcll(good), l1, rest, w, gbar_out, u_out, err_flag);
}

// A launch takes fewer than 2^32 threads: one-wave blocks per launch.
constexpr int64_t kMaxWaveBlocks = (int64_t(1) << 32) / 64 - 1;

// Whether a step's entries are compared within a wave (design_weights_short_kernel)
// rather than gathered in its table: many lists of few entries, which a group of four
// lanes passes four at a time (0.7 us a completion, however few the steps), while a
// wave per step takes 5 us and, past some 5,000 steps, 0.5 to 1.9 ns a step.  us a
// call, table / wave: 8 lists of 1 entry 7.4 / 4.7 at 16 steps and 8.5 / 9.6 at 15,582;
// 16 of 4 18.6 / 6.3 at 1,961 and 20.7 / 17.1 at 15,752; 24 of 1 22.9 / 21.1 at 31,462;
// 64 of 1 103.8 / 32.2 at 31,766; 64 of 2 52.2 / 10.3 at 1,989.  Up to four lists
// the table is as fast at any number of steps (4.8 to 7.1).
inline bool short_lists_pay(int K, int topk, int64_t total_T) {
  if (K <= 4 || topk > 4 || K * topk > 128) return false;
  return total_T <= (K >= 24 ? kMaxWaveBlocks : 1300 * K);
}

// Groups of G lanes: the smallest power of two >= topk (at least 4, at most 64)
// whose 64 / G tables stay within 24 KB of LDS, so that six blocks or more share a CU.
struct WeightsShape {
  int group, slots;
};
WeightsShape weights_shape(int K, int topk) {
  WeightsShape s{4, 16};
  while (s.slots < 2 * K * topk) s.slots *= 2;   // <= 512
  while (s.group < 64 && (s.group < topk || 64 / s.group * s.slots * 12 > 24 * 1024)) s.group *= 2;
  return s;
}

// The budgeted monotone solve (App. F).  One thread per prompt ran Pooling
// Adjacent Violators over the steps, one dependent chain of LDS accesses and
// branches per step, and then summed, searched and wrote the table alone:
// 1,922 us for 8 prompts of 2,500 to 6,900 steps, 44 us with what follows.
//
// The blocks are found by all threads: blocks of steps are joined pairwise up a
// tree, where only the blocks at the joint can violate, and pooling adjacent
// violators in any order ends at the same blocks.  A block's weight is summed in
// the order of the tree (float64: at most log2(T) + the block's joins roundings,
// where one after another it was its length; against sums in extended precision
// 9.2e-17 relative, rms over the steps of six batches of that size, where one
// after another is off by 1.7e-16).  Scores, the search for the first
// unsaturated block and the table are spread over the threads.
constexpr int kDesignThreads = 1024;

// Storage of one prompt's blocks, all of one memory kind (LDS or the workspace).
// ln[t] > 0: a block of ln[t] steps starts at t, its summed weight (later its
// score) at wv[t]; the last step e of a block of L >= 2 steps holds ln[e] = -L,
// so that the block can be found from its end; ln is 0 or stale but not
// positive at every other step.  heads: bit t % 64 of word t / 64.
struct Blocks {
  double* wv;
  int32_t* ln;
  uint64_t* heads;
};

// Joins the blocks of [a, m) and [m, b): pools the two blocks at m while the left
// one's mean is below the right one's, then on to both sides.  Scores
// sqrt(W / L) are in the order of the means, and W1 / L1 < W2 / L2 exactly when
// W1 L2 < W2 L1: two products and no division (a product rounds to 2^-53
// relative, so the decision can differ from the exact one only for blocks whose
// means agree to that; pooling or not such a pair moves the table by the same
// relative amount).
__device__ __forceinline__ void join_blocks(const Blocks& bl, int a, int m, int b) {
  int l = abs(bl.ln[m - 1]), r = bl.ln[m];
  int s = m - l, e = m;            // the pooled block is [s, e) once a pair has been pooled
  double W = bl.wv[s], V = bl.wv[m];
  if (!(W * (double)r < V * (double)l)) return;
  bool pool_right = true;
  for (;;) {
    if (pool_right) {              // [s, e) and the block of r steps at e
      bl.ln[e] = 0;
      W += V;
      l += r;
      e += r;
    }
    pool_right = false;
    if (e < b) {
      r = bl.ln[e];
      V = bl.wv[e];
      pool_right = W * (double)r < V * (double)l;
    }
    if (pool_right) continue;
    if (s == a) break;
    const int tl = abs(bl.ln[s - 1]);
    const double tw = bl.wv[s - tl];
    if (!(tw * (double)l < W * (double)tl)) break;
    bl.ln[s] = 0;
    s -= tl;
    l += tl;
    W += tw;
  }
  bl.ln[s] = l;
  bl.ln[e - 1] = -l;
  bl.wv[s] = W;
}

// Bits of the first step of every block over [0, n).
__device__ __forceinline__ void mark_heads(const Blocks& bl, int n) {
  for (int t = threadIdx.x; t < (n + 63) / 64 * 64; t += kDesignThreads) {
    const uint64_t m = __ballot(t < n && bl.ln[t] > 0);
    if ((threadIdx.x & 63) == 0) bl.heads[t / 64] = m;
  }
}

// The solve of one prompt of T steps whose last positive weight is step n - 1
// (trailing steps of weight 0 are blocks of their own and pool with nothing).
__device__ __forceinline__ void solve_prompt(const Blocks& bl, const double* wp, int T, int n, double budget,
                                             double* xp) {
  __shared__ int sh_saturated;
  __shared__ double sh_kappa;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
#pragma unroll 4
  for (int t = tid; t < n; t += kDesignThreads) {
    bl.ln[t] = 1;
    bl.wv[t] = wp[t];
  }
  __syncthreads();
  // (64-bit positions: twice the half length can pass 2^31)
  for (int64_t half = 1; half < n; half *= 2) {
    for (int64_t a = 2 * half * tid; a + half < n; a += 2 * half * kDesignThreads)
      join_blocks(bl, (int)a, (int)(a + half), (int)min(a + 2 * half, (int64_t)n));
    __syncthreads();
  }
  const int words = (n + 63) / 64;
  mark_heads(bl, n);
  __syncthreads();
  // the block scores sqrt(W_m / L_m)
  for (int t = tid; t < n; t += kDesignThreads)
    if (bl.ln[t] > 0) bl.wv[t] = sqrt(bl.wv[t] / (double)bl.ln[t]);
  __syncthreads();
  // Suffix sums of L_m s_m (accumulated from the last block), and the first
  // unsaturated block: kappa(m) = (B - start_m) / sum_{j>=m} L_j s_j with
  // kappa(m) s_m <= 1.  The first block of weight 0 from which only such blocks
  // follow (if there is one) is step n: kappa < 0 stands for it.
  if (wave == 0) {
    double acc = 0.0, kappa = -1.0;
    int saturated = n;
    bool found = n < T;            // false: until a block qualifies, the last block's kappa stands
    for (int word = words - 1; word >= 0; --word) {
      const uint64_t heads = bl.heads[word];
      if (heads == 0) continue;
      const int t = word * 64 + lane;
      const bool head = (heads >> lane) & 1;
      const double score = head ? bl.wv[t] : 0.0;
      const int len = head ? bl.ln[t] : 0;
      double rest = 0.0;           // of this lane's block
      for (uint64_t m = heads; m != 0;) {
        const int k = 63 - __builtin_clzll(m);
        m ^= 1ull << k;
        acc += (double)__builtin_amdgcn_readlane(len, k) * lane_value(score, k);
        if (lane == k) rest = acc;
      }
      const bool none = head && rest == 0.0;
      const double mine = none ? -1.0 : (budget - (double)t) / rest;
      const uint64_t ok = __ballot(none || (head && mine * score <= 1.0));
      if (ok != 0) {
        const int k = __builtin_ctzll(ok);
        kappa = lane_value(mine, k);
        saturated = word * 64 + k;
        found = true;
      } else if (!found) {
        kappa = lane_value(mine, 63 - __builtin_clzll(heads));
        found = true;
      }
    }
    if (lane == 0) {
      sh_kappa = kappa;
      sh_saturated = saturated;
    }
  }
  __syncthreads();
  const double kappa = sh_kappa;
  const int saturated = sh_saturated;
  const double even = (budget - (double)saturated) / (double)(T - saturated);   // used where kappa < 0
  for (int t = tid; t < T; t += kDesignThreads) {
    int start = t;                 // of t's block
    double score = 0.0;
    if (t < n) {
      int word = t / 64;
      uint64_t m = bl.heads[word] & (~0ull >> (63 - (t & 63)));
      while (m == 0) m = bl.heads[--word];   // step 0 starts a block
      start = word * 64 + 63 - __builtin_clzll(m);
      score = bl.wv[start];
    }
    const double v = kappa < 0.0 ? (start < saturated ? 1.0 : even) : fmin(1.0, kappa * score);
    xp[t] = fmax(v, kXiFloor);
  }
}

// The sum of the square roots of the weights, by one wave: lane l takes the
// steps l, l + 64, ... in order, then a fixed butterfly over the lanes.
__device__ __forceinline__ double root_sum(const double* wp, int T) {
  double part = 0.0;
#pragma unroll 8
  for (int t = threadIdx.x & 63; t < T; t += 64) part += sqrt(wp[t]);
  return wave_sum(part);
}

// LDS of a design block: its blocks of steps (12 bytes and a bit per step) when
// they fit.
constexpr int kDesignLdsBytes = 156 * 1024;
constexpr int kDesignLdsSteps = kDesignLdsBytes / 98 * 8;   // 12.25 bytes per step: room for the last word

// One block per prompt: T <= kDesignLdsSteps steps in LDS, otherwise in the workspace.
__global__ __launch_bounds__(kDesignThreads) void design_cutoffs_kernel(
    const double* __restrict__ w, const int64_t* __restrict__ xi_off, double budget, int variant, double lambda,
    double* __restrict__ xi, int32_t* __restrict__ blen, double* __restrict__ bval, int32_t* __restrict__ spare,
    int32_t* __restrict__ err_flag) {
  __shared__ __attribute__((aligned(16))) unsigned char lds[kDesignLdsBytes];
  __shared__ int sh_bad, sh_n;
  __shared__ double sh_root, sh_run[kDesignThreads / 64];
  const int p = blockIdx.x, tid = threadIdx.x;
  const int64_t a = xi_off[p];
  const int T = (int)(xi_off[p + 1] - a);
  const double* wp = w + a;
  double* xp = xi + a;
  if (variant == PSPO_DESIGN_UNIFORM) {
    for (int t = tid; t < T; t += kDesignThreads) xp[t] = (double)(T - t) / (double)T;
    return;
  }
  if (variant == PSPO_DESIGN_TIME_PRIOR) {
    for (int t = tid; t < T; t += kDesignThreads) xp[t] = fmax(exp(-lambda * (double)t), kXiFloor);
    return;
  }
  // the weights checked, and the last positive one
  if (tid == 0) sh_bad = sh_n = 0;
  __syncthreads();
  int n = 0;
  bool bad = false;
#pragma unroll 4
  for (int t = tid; t < T; t += kDesignThreads) {
    const double v = wp[t];
    if (!(v >= 0.0) || isinf(v)) bad = true;
    if (v > 0.0) n = t + 1;
  }
  if (bad) atomicOr(&sh_bad, 1);
  if (n > 0) atomicMax(&sh_n, n);
  __syncthreads();
  n = sh_n;
  double all = -1.0;   // >= 0 or NAN: every step's value
  if (sh_bad) {
    if (tid == 0 && err_flag) atomicOr(err_flag, PSPO_DEVERR_BAD_XI);
    all = NAN;
  } else if (budget >= (double)T) {
    all = 1.0;
  } else if (n == 0) {   // every weight zero: any feasible table is optimal
    all = budget / (double)T;
  }
  if (!(all < 0.0)) {
    for (int t = tid; t < T; t += kDesignThreads) xp[t] = all;
    return;
  }
  if (variant == PSPO_DESIGN_HEURISTIC) {
    // a running minimum: of each wave's 64 steps, then over the waves
    if (tid < 64) {
      const double r = root_sum(wp, T);
      if (tid == 0) sh_root = r;
    }
    __syncthreads();
    const double root = sh_root;
    double before = 1.0;
    for (int t0 = 0; t0 < T; t0 += kDesignThreads) {
      const int t = t0 + tid;
      double v = t < T ? fmin(1.0, budget * sqrt(wp[t]) / root) : 1.0;
#pragma unroll
      for (int o = 1; o < 64; o <<= 1) {
        const double u = __shfl_up(v, o);
        if ((tid & 63) >= o) v = fmin(v, u);
      }
      if ((tid & 63) == 63) sh_run[tid >> 6] = v;
      __syncthreads();
      double run = before;
      for (int k = 0; k < kDesignThreads / 64; ++k) {
        if (k == (tid >> 6)) v = fmin(v, run);
        run = fmin(run, sh_run[k]);
      }
      before = run;
      if (t < T) xp[t] = fmax(v, kXiFloor);
      __syncthreads();
    }
    return;
  }
  if (T <= kDesignLdsSteps)
    solve_prompt(Blocks{reinterpret_cast<double*>(lds), reinterpret_cast<int32_t*>(lds + (int64_t)kDesignLdsSteps * 8),
                        reinterpret_cast<uint64_t*>(lds + (int64_t)kDesignLdsSteps * 12)},
                 wp, T, n, budget, xp);
  else
    solve_prompt(Blocks{bval + a, blen + a, reinterpret_cast<uint64_t*>(spare + (a + 1) / 2 * 2)}, wp, T, n, budget,
                 xp);
}

// Argument checks shared by the design entry points (host only).
int check_design_args(const double* w, const int64_t* xi_off, int32_t P, int64_t total_T, double budget,
                      int32_t variant, double lambda, const double* xi) {
  PSPO_REQUIRE(P >= 1 && total_T >= 0, PSPO_ERR_INVALID_ARG, "need P >= 1 and total_T >= 0");
  PSPO_REQUIRE(variant >= PSPO_DESIGN_OPTIMIZED && variant <= PSPO_DESIGN_TIME_PRIOR, PSPO_ERR_INVALID_ARG,
               "unknown design variant");
  PSPO_REQUIRE(std::isfinite(budget) && budget > 0.0, PSPO_ERR_INVALID_ARG, "budget must be finite and > 0");
  PSPO_REQUIRE(std::isfinite(lambda) && lambda >= 0.0, PSPO_ERR_INVALID_ARG, "lambda must be finite and >= 0");
  if (total_T == 0) return PSPO_OK;
  PSPO_REQUIRE(w && xi_off && xi, PSPO_ERR_INVALID_ARG, "null pointer");
  PSPO_REQUIRE(aligned(w, 8) && aligned(xi_off, 8) && aligned(xi, 8), PSPO_ERR_INVALID_ARG,
               "misaligned pointer");
  return PSPO_OK;
}

// The blocks of the prompts that do not fit in LDS (summed weight, length and
// the bits of the first steps) carved from `ws`
// (pspo_design_workspace_bytes(total_T)), then the solve.  The kernel writes
// every entry before reading it, so the memory needs no clearing.
int launch_design(const double* w, const int64_t* xi_off, int32_t P, int64_t total_T, double budget, int32_t variant,
                  double lambda, double* xi, char* ws, int32_t* err_flag, hipStream_t stream) {
  int32_t* blen = reinterpret_cast<int32_t*>(ws + round_up(total_T * 4, 256));
  double* bval = reinterpret_cast<double*>(ws + 2 * round_up(total_T * 4, 256));
  int32_t* spare = reinterpret_cast<int32_t*>(ws);
  hipLaunchKernelGGL(design_cutoffs_kernel, dim3((unsigned)P), dim3(kDesignThreads), 0, stream, w, xi_off, budget,
                     variant, lambda, xi, blen, bval, spare, err_flag);
  PSPO_LAUNCHED("design_cutoffs_kernel", stream);
  return PSPO_OK;
}

}  // namespace

// Scratch of the no-allocation entry point: a file-scope device array, one copy
// per GPU, held until the process ends.  Host code never uses its name as an
// address (on the host it is a stand-in symbol): the device address comes from
// hipGetSymbolAddress, taken once per device with that device current.
constexpr size_t kNoAllocScratchBytes = size_t(8) << 20;   // total_T <= 2^19 steps
static __device__ __align__(256) unsigned char scratch[kNoAllocScratchBytes];

namespace {

constexpr int kMaxDevices = 64;
std::mutex g_scratch_mu;
char* g_scratch[kMaxDevices] = {};

// The current device's address of `scratch` (looked up on the first call on
// that device).
int scratch_address(char** out) {
  int dev = 0;
  PSPO_HIP_CHECK(hipGetDevice(&dev));
  PSPO_REQUIRE(dev >= 0 && dev < kMaxDevices, PSPO_ERR_UNSUPPORTED, "device id out of range");
  std::lock_guard<std::mutex> lock(g_scratch_mu);
  if (g_scratch[dev] == nullptr) {
    void* p = nullptr;
    PSPO_HIP_CHECK(hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)));
    PSPO_REQUIRE(p != nullptr && aligned(p, 256), PSPO_ERR_HIP, "scratch has no usable device address");
    g_scratch[dev] = static_cast<char*>(p);
  }
  *out = g_scratch[dev];
  return PSPO_OK;
}

}  // namespace
}  // namespace pspo

extern "C" {

int pspo_design_weights(const float* gamma, const int32_t* topk_ids, const float* topk_logp, int32_t topk,
                        const int32_t* lengths, const int32_t* full_off, const float* rewards, const int64_t* xi_off,
                        int32_t P, int32_t K, int64_t total_T, double* w, double* gamma_bar, double* u,
                        int32_t* err_flag, hipStream_t stream) {
  using namespace pspo;
  clear_last_error();
  TraceRange trace_range("pspo_design_weights");
  PSPO_REQUIRE(P >= 1 && K >= 1 && total_T >= 0, PSPO_ERR_INVALID_ARG, "need P >= 1, K >= 1, total_T >= 0");
  PSPO_REQUIRE(K <= 64, PSPO_ERR_UNSUPPORTED, "K must be <= 64");
  PSPO_REQUIRE(topk >= 1 && (int64_t)K * topk <= kDesignMaxEntries, PSPO_ERR_UNSUPPORTED,
               "need topk >= 1 and K * topk <= 256");
  if (total_T == 0) return PSPO_OK;
  PSPO_REQUIRE(gamma && topk_ids && topk_logp && lengths && full_off && rewards && xi_off && w, PSPO_ERR_INVALID_ARG,
               "null pointer");
  PSPO_REQUIRE(aligned(w, 8) && aligned(gamma_bar, 8) && aligned(u, 8) && aligned(xi_off, 8), PSPO_ERR_INVALID_ARG,
               "misaligned float64 / int64 pointer");
  const int ne = K * topk;
  const bool few = short_lists_pay(K, topk, total_T);
  const WeightsShape shape = weights_shape(K, topk);
  const int steps = few ? 1 : 64 / shape.group;
  const int64_t blocks = total_T / steps + (total_T % steps != 0 ? 1 : 0);
  PSPO_REQUIRE(blocks <= kMaxWaveBlocks, PSPO_ERR_UNSUPPORTED,
               "problem too large: at most " + std::to_string(kMaxWaveBlocks * steps) + " steps at this K and topk");
  if (int rc = require_gfx950()) return rc;
  auto launch = [&](auto kernel, auto... slots) {
    hipLaunchKernelGGL(kernel, dim3((unsigned)blocks), dim3(64), few ? 0u : (unsigned)(steps * shape.slots * 12), stream,
                       gamma, topk_ids, topk_logp, topk, lengths, full_off, rewards, xi_off, P, K, total_T, slots..., w,
                       gamma_bar, u, err_flag);
  };
  if (few && ne <= 64) launch(design_weights_short_kernel<1>);
  else if (few) launch(design_weights_short_kernel<2>);
  else if (shape.group == 4) launch(design_weights_kernel<4>, shape.slots);
  else if (shape.group == 8) launch(design_weights_kernel<8>, shape.slots);
  else if (shape.group == 16) launch(design_weights_kernel<16>, shape.slots);
  else if (shape.group == 32) launch(design_weights_kernel<32>, shape.slots);
  else launch(design_weights_kernel<64>, shape.slots);
  PSPO_LAUNCHED("design_weights_kernel", stream);
  return PSPO_OK;
}

size_t pspo_design_workspace_bytes(int64_t total_T) {
  using pspo::round_up;
  if (total_T < 0) return 0;
  return (size_t)(round_up(total_T * 4, 256) * 2 + round_up(total_T * 8, 256));
}

int pspo_design_cutoffs(const double* w, const int64_t* xi_off, int32_t P, int64_t total_T, double budget,
                        int32_t variant, double lambda, double* xi, void* workspace, size_t workspace_bytes,
                        int32_t* err_flag, hipStream_t stream) {
  using namespace pspo;
  clear_last_error();
  TraceRange trace_range("pspo_design_cutoffs");
  if (int rc = check_design_args(w, xi_off, P, total_T, budget, variant, lambda, xi)) return rc;
  if (total_T == 0) return PSPO_OK;
  PSPO_REQUIRE(workspace && aligned(workspace, 256), PSPO_ERR_INVALID_ARG,
               "workspace must be non-NULL and 256-byte aligned");
  PSPO_REQUIRE(workspace_bytes >= pspo_design_workspace_bytes(total_T), PSPO_ERR_WORKSPACE,
               "workspace too small: need " + std::to_string(pspo_design_workspace_bytes(total_T)) + " bytes");
  if (int rc = require_gfx950()) return rc;
  return launch_design(w, xi_off, P, total_T, budget, variant, lambda, xi, static_cast<char*>(workspace), err_flag,
                       stream);
}

int pspo_design_cutoffs_noalloc(const double* w, const int64_t* xi_off, int32_t P, int64_t total_T, double budget,
                                int32_t variant, double lambda, double* xi, int32_t* err_flag, hipStream_t stream) {
  using namespace pspo;
  clear_last_error();
  TraceRange trace_range("pspo_design_cutoffs_noalloc");
  if (int rc = check_design_args(w, xi_off, P, total_T, budget, variant, lambda, xi)) return rc;
  if (total_T == 0) return PSPO_OK;
  PSPO_REQUIRE(pspo_design_workspace_bytes(total_T) <= kNoAllocScratchBytes, PSPO_ERR_UNSUPPORTED,
               "total_T = " + std::to_string(total_T) + " needs " +
                   std::to_string(pspo_design_workspace_bytes(total_T)) + " bytes of scratch; the no-allocation "
                   "entry point has " + std::to_string(kNoAllocScratchBytes) + " (total_T <= 2^19)");
  if (int rc = require_gfx950()) return rc;
  char* ws = nullptr;
  if (int rc = scratch_address(&ws)) return rc;
  return launch_design(w, xi_off, P, total_T, budget, variant, lambda, xi, ws, err_flag, stream);
}

}  // extern "C"

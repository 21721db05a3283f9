// Agent- and turn-wise grouping and group-relative advantages (gfx950).
//
// Alg. 1 of the paper keys every sampled candidate by g = hash(e, i, t); Eq. (1) normalises the
// rewards inside each group.  Here the key is the injective packing
//   key = (e * n_agent + i) * n_turn + t,
// groups are numbered densely in ascending key order, and the responses of a group are listed in
// ascending original index (a stable sort by key).  Members are first listed per key in arbitrary order (the
// return value of a histogram atomic), then ordered by counting inside their group, which makes every output
// deterministic.  Three paths by size, with the same arithmetic per group:
//   k_ga_range   up to 65536 responses over as many keys: one launch, two beyond 4096 responses.  Every workgroup owns a
//                range of keys and scans all keys (they are in L2); nothing passes between workgroups.
//   k_gp_*       pools of up to 16 million responses: partition by key range, each range finished in LDS, results gathered
//                back in response order.
//   k_ga_hist .. anything else (very many keys per response, or few keys with very many members): histogram over the key
//                box, scans, scatter, finish.
#include <algorithm>
#include <mutex>

#include "common.hpp"

namespace atg {

namespace {

constexpr int kKeysPerBlock = 2048;
constexpr int kSmallGroup = 16;

struct GaArgs {
  int32_t n_resp, n_env, n_agent, n_turn;
  const int32_t* env_id;
  const int32_t* agent_id;
  const int32_t* turn_id;
  const float* reward;
  int32_t group_by;          // at_grpo_group_by
  int32_t n_sample;          // extent of sample_id (AT_GRPO_GROUP_BY_PARALLEL only)
  const int32_t* sample_id;  // candidate index c of each response (AT_GRPO_GROUP_BY_PARALLEL only)
};

// Key of a response under the chosen grouping (ascending key = canonical group order):
//   AGENT_TURN  (e, i, t)                         the paper's grouping (Alg. 1, Sec. 4.1)
//   TRAJECTORY  e                                 all candidates of a task in one group, whatever agent
//                                                 and turn produced them (GRPO applied to the whole MAS)
//   PARALLEL    (e, i, t, c if t > 0 else 0)      K trajectories sampled in parallel share a state only at
//                                                 the first turn; later turns are groups of one (Sec. 4.1)
// A response with an id outside its extent has no key.
__device__ __forceinline__ int64_t key_of(const GaArgs& a, int r, bool* ok) {
  const int e = a.env_id[r], i = a.agent_id[r], t = a.turn_id[r];
  bool in = e >= 0 && e < a.n_env && i >= 0 && i < a.n_agent && t >= 0 && t < a.n_turn;
  int64_t key;
  if (a.group_by == AT_GRPO_GROUP_BY_TRAJECTORY) {
    key = e;
  } else {
    key = (static_cast<int64_t>(e) * a.n_agent + i) * a.n_turn + t;
    if (a.group_by == AT_GRPO_GROUP_BY_PARALLEL) {
      const int c = a.sample_id[r];
      in = in && c >= 0 && c < a.n_sample;
      key = key * a.n_sample + (t > 0 ? c : 0);
    }
  }
  *ok = in;
  return key;
}

__device__ __forceinline__ bool finite_reward(float x) { return fabsf(x) <= 3.402823466e38f; }

// hist[key] += 1 for the wavefront's lanes with key >= 0; returns the lane's arrival rank inside its group.  Neighbouring lanes
// with the same key (candidates of one group emitted together, the order a rollout produces) are folded into one atomic
// per run.  Every lane of the wavefront calls it.
__device__ __forceinline__ int count_runs(int32_t* hist, int key) {
  const int lane = threadIdx.x & 63;
  const int prev = __shfl_up(key, 1, 64);
  const bool head = (lane == 0) || (key != prev);
  const unsigned long long heads = __builtin_amdgcn_ballot_w64(head);
  const unsigned long long below = heads & ((2ull << lane) - 1ull);          // heads at or below this lane
  const int start = 63 - __builtin_clzll(below);
  const unsigned long long above = (lane == 63) ? 0ull : (heads >> (lane + 1)) << (lane + 1);
  const int next = above ? __builtin_ctzll(above) : 64;
  int base = 0;
  if (head && key >= 0) base = atomicAdd(&hist[key], next - lane);
  base = __shfl(base, start, 64);
  return base + (lane - start);
}

// histogram over the key box
__global__ __launch_bounds__(256) void k_ga_hist(GaArgs a, int32_t* __restrict__ err,
                                                 int32_t* __restrict__ hist, int32_t* __restrict__ key_of_resp,
                                                 int32_t* __restrict__ rank_of_resp) {
  const int r = blockIdx.x * 256 + threadIdx.x;
  int key = -1;
  if (r < a.n_resp) {
    bool ok;
    const int64_t k64 = key_of(a, r, &ok);
    if (!ok) {
      atomicOr(err, AT_GRPO_DATA_ID_RANGE);
    } else if (!finite_reward(a.reward[r])) {
      atomicOr(err, AT_GRPO_DATA_REWARD);     // takes no part: no group, advantage 0
    } else {
      key = static_cast<int32_t>(k64);
    }
    key_of_resp[r] = key;
  }
  const int rank = count_runs(hist, key);
  if (r < a.n_resp && key >= 0) rank_of_resp[r] = rank;
}

// per-block sums of (key present, members) over 2048 keys
__global__ __launch_bounds__(256) void k_ga_scan_partial(const int32_t* __restrict__ hist, int64_t n_keys,
                                                         int32_t* __restrict__ bsum_p,
                                                         int32_t* __restrict__ bsum_c) {
  __shared__ int lds4[4];
  const int64_t k0 = static_cast<int64_t>(blockIdx.x) * kKeysPerBlock + threadIdx.x * 8;
  int p = 0, c = 0;
#pragma unroll
  for (int e = 0; e < 8; ++e) {
    const int h = (k0 + e < n_keys) ? hist[k0 + e] : 0;
    p += (h > 0);
    c += h;
  }
  const int tp = block_sum_256_int(p, lds4);
  const int tcn = block_sum_256_int(c, lds4);
  if (threadIdx.x == 0) {
    bsum_p[blockIdx.x] = tp;
    bsum_c[blockIdx.x] = tcn;
  }
}

// single block: exclusive scan of the block sums; totals -> n_groups and the closing CSR offset
__global__ __launch_bounds__(256) void k_ga_scan_top(int64_t n_blocks, int32_t* __restrict__ bsum_p,
                                                     int32_t* __restrict__ bsum_c,
                                                     int32_t* __restrict__ n_groups,
                                                     int32_t* __restrict__ seg_offsets) {
  __shared__ int lds4[4];
  int run_p = 0, run_c = 0;
  for (int64_t base = 0; base < n_blocks; base += 256) {
    const int64_t b = base + threadIdx.x;
    const int vp = (b < n_blocks) ? bsum_p[b] : 0;
    const int vc = (b < n_blocks) ? bsum_c[b] : 0;
    int tp, tcn;
    const int ep = block_exclusive_scan<256>(vp, lds4, &tp);
    const int ec = block_exclusive_scan<256>(vc, lds4, &tcn);
    if (b < n_blocks) {
      bsum_p[b] = run_p + ep;
      bsum_c[b] = run_c + ec;
    }
    run_p += tp;
    run_c += tcn;
  }
  if (threadIdx.x == 0) {
    *n_groups = run_p;
    seg_offsets[run_p] = run_c;
  }
}

// dense id of every present key and CSR offset of every group
__global__ __launch_bounds__(256) void k_ga_scan_apply(const int32_t* __restrict__ hist, int64_t n_keys,
                                                       const int32_t* __restrict__ boff_p,
                                                       const int32_t* __restrict__ boff_c,
                                                       int32_t* __restrict__ gid_of_key,
                                                       int32_t* __restrict__ seg_offsets) {
  __shared__ int lds4[4];
  const int64_t k0 = static_cast<int64_t>(blockIdx.x) * kKeysPerBlock + threadIdx.x * 8;
  int h[8];
  int p = 0, c = 0;
#pragma unroll
  for (int e = 0; e < 8; ++e) {
    h[e] = (k0 + e < n_keys) ? hist[k0 + e] : 0;
    p += (h[e] > 0);
    c += h[e];
  }
  int tp, tcn;
  int gp = boff_p[blockIdx.x] + block_exclusive_scan<256>(p, lds4, &tp);
  int gc = boff_c[blockIdx.x] + block_exclusive_scan<256>(c, lds4, &tcn);
#pragma unroll
  for (int e = 0; e < 8; ++e) {
    if (h[e] > 0) {
      gid_of_key[k0 + e] = gp;
      seg_offsets[gp] = gc;
      ++gp;
      gc += h[e];
    }
  }
}

__global__ __launch_bounds__(256) void k_ga_scatter(int n_resp, const int32_t* __restrict__ key_of_resp,
                                                    const int32_t* __restrict__ rank_of_resp,
                                                    const int32_t* __restrict__ gid_of_key,
                                                    const int32_t* __restrict__ seg_offsets,
                                                    int32_t* __restrict__ group_id,
                                                    int32_t* __restrict__ arrival,
                                                    float* __restrict__ adv) {
  const int r = blockIdx.x * 256 + threadIdx.x;
  if (r >= n_resp) return;
  const int key = key_of_resp[r];
  if (key < 0) {
    group_id[r] = -1;
    adv[r] = 0.f;
    return;
  }
  const int g = gid_of_key[key];
  group_id[r] = g;
  arrival[seg_offsets[g] + rank_of_resp[r]] = r;
}

struct GaStat {
  float eps_std;
  int ddof, norm;
};

// One group of at most N <= 16 members, handled by one thread, in registers: ranks by counting, sums in ascending-index
// order (fp32, two passes).  id(j), x(j): index and reward of member j in arrival order; put_perm(rank, id) and
// put_adv(j, id, a) store; *best gets the first of the members with the largest reward.
template <int N, typename Id, typename X, typename PutPerm, typename PutAdv>
__device__ __forceinline__ void finish_small(int n, Id id_of, X x_of, PutPerm put_perm, PutAdv put_adv, const GaStat& st,
                                             float* mean_out, float* std_out, int* best) {
  int id[N];
  float x[N];
#pragma unroll
  for (int j = 0; j < N; ++j) id[j] = (j < n) ? id_of(j) : 0x7fffffff;
#pragma unroll
  for (int j = 0; j < N; ++j) x[j] = (j < n) ? x_of(j) : 0.f;
  float xs[N];      // rewards in perm order
  int rank[N];
#pragma unroll
  for (int j = 0; j < N; ++j) {
    int c = 0;
#pragma unroll
    for (int i = 0; i < N; ++i) c += (id[i] < id[j]);
    rank[j] = c;
  }
#pragma unroll
  for (int pos = 0; pos < N; ++pos) {
    float v = 0.f;
#pragma unroll
    for (int j = 0; j < N; ++j) v = (rank[j] == pos && j < n) ? x[j] : v;
    xs[pos] = v;
  }
  float sum = 0.f;
  bool same = true;
#pragma unroll
  for (int pos = 0; pos < N; ++pos)
    if (pos < n) {
      sum += xs[pos];
      same = same && (xs[pos] == xs[0]);
    }
  const float mean = same ? xs[0] : sum / static_cast<float>(n);
  float sd = 0.f, ss = 0.f;
#pragma unroll
  for (int pos = 0; pos < N; ++pos)
    if (pos < n) {
      const float d = xs[pos] - mean;
      ss += d * d;
    }
  const int denom = n - st.ddof;
  if (!same) sd = denom > 0 ? sqrtf(ss / static_cast<float>(denom)) : 0.f;
  int top = id[0];
  float xt = x[0];
#pragma unroll
  for (int j = 0; j < N; ++j)
    if (j < n) {
      put_perm(rank[j], id[j]);
      float a = 0.f;
      if (!same) a = (st.norm == AT_GRPO_NORM_STD) ? (x[j] - mean) / (sd + st.eps_std) : (x[j] - mean);
      put_adv(j, id[j], a);
      if (x[j] > xt || (x[j] == xt && id[j] < top)) {
        xt = x[j];
        top = id[j];
      }
    }
  *mean_out = mean;
  *std_out = sd;
  *best = top;
}

template <typename Id, typename X, typename PutPerm, typename PutAdv>
__device__ __forceinline__ void finish_by_thread(int n, Id id_of, X x_of, PutPerm put_perm, PutAdv put_adv, const GaStat& st,
                                                 float* mean, float* sd, int* best) {
  if (n <= 8) finish_small<8>(n, id_of, x_of, put_perm, put_adv, st, mean, sd, best);
  else finish_small<kSmallGroup>(n, id_of, x_of, put_perm, put_adv, st, mean, sd, best);
}

// One larger group, handled by one wavefront: ranks by counting, statistics as 64 lane-strided partial sums over the
// ordered members, combined in a fixed order.  perm: the group's part of the output (global memory); reward(r): reward of
// response r.
template <typename Id, typename X, typename Reward, typename PutAdv>
__device__ __forceinline__ void finish_by_wave(int n, int lane, Id id_of, X x_of, Reward reward, int32_t* perm, PutAdv put_adv,
                                               const GaStat& st, float* mean_out, float* std_out, int* best) {
  n = __builtin_amdgcn_readfirstlane(n);
  if (n <= 64) {       // a member per lane: compared in registers (3.1 million responses in groups of 24: 208 -> 185 us)
    const int mine = lane < n ? id_of(lane) : 0x7fffffff;
    int rank = 0;
    for (int i = 0; i < n; ++i) rank += __builtin_amdgcn_readlane(mine, i) < mine;
    if (lane < n) perm[rank] = mine;
  } else {
    for (int j = lane; j < n; j += 64) {
      const int rj = id_of(j);
      int rank = 0;
      for (int i = 0; i < n; ++i) rank += (id_of(i) < rj);
      perm[rank] = rj;
    }
  }
  // the ranks are read back by other lanes of this wavefront: a fence of the workgroup is enough, and a device-wide one writes
  // back the L2 for every group (2^20 responses in groups of 24: 797 us in rollout order and 914 shuffled, now 123 and 153)
  __threadfence_block();
  const float x0 = reward(perm[0]);
  float sum = 0.f, xt = -INFINITY;
  int same = 1, top = 0x7fffffff;
  for (int j = lane; j < n; j += 64) {
    const int r = perm[j];
    const float x = reward(r);
    sum += x;
    same &= (x == x0);
    if (x > xt) {        // ascending indices: the first of equal rewards stays
      xt = x;
      top = r;
    }
  }
  sum = wave_sum(sum);
  sum = __shfl(sum, 0, 64);
  same = __builtin_amdgcn_ballot_w64(same == 0) == 0ull;
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) {
    const float xo = __shfl_xor(xt, o, 64);
    const int to = __shfl_xor(top, o, 64);
    if (xo > xt || (xo == xt && to < top)) {
      xt = xo;
      top = to;
    }
  }
  float mean = sum / static_cast<float>(n), sd = 0.f;
  if (same) {
    mean = x0;
  } else {
    float ss = 0.f;
    for (int j = lane; j < n; j += 64) {
      const float d = reward(perm[j]) - mean;
      ss += d * d;
    }
    ss = wave_sum(ss);
    ss = __shfl(ss, 0, 64);
    const int denom = n - st.ddof;
    sd = denom > 0 ? sqrtf(ss / static_cast<float>(denom)) : 0.f;
  }
  for (int j = lane; j < n; j += 64) {
    const float x = x_of(j);
    const float a = same ? 0.f : (st.norm == AT_GRPO_NORM_STD) ? (x - mean) / (sd + st.eps_std) : (x - mean);
    put_adv(j, id_of(j), a);
  }
  *mean_out = mean;
  *std_out = sd;
  *best = top;
}

// The group outputs, and how many groups the buffers hold; with `fill` the entries behind the last group and behind the
// last listed response are set to zero (best: -1).
struct GaOut {
  int32_t* group_id;
  int32_t* n_groups;
  int32_t* seg_offsets;
  int32_t* perm;
  float* adv;
  float* mean;     // may be null
  float* std;      // may be null
  int32_t* best;   // may be null
  int32_t g_max;
  int32_t fill;
};

__device__ __forceinline__ void put_stats(const GaOut& o, int g, float mean, float sd, int best) {
  if (o.mean) o.mean[g] = mean;
  if (o.std) o.std[g] = sd;
  if (o.best) o.best[g] = best;
}

// fills the outputs behind group G - 1 and listed response n_listed - 1, with `threads` threads of which this is `tid`
__device__ __forceinline__ void fill_tails(const GaOut& o, int G, int n_listed, int n_resp, int64_t tid, int64_t threads) {
  if (!o.fill) return;
  for (int64_t g = G + tid; g < o.g_max; g += threads) {
    o.seg_offsets[g + 1] = 0;
    put_stats(o, static_cast<int>(g), 0.f, 0.f, -1);
  }
  for (int64_t r = n_listed + tid; r < n_resp; r += threads) o.perm[r] = 0;
}

// Groups 0 .. n - 1 of a list of members in arrival order, outputs from group g0 on: off(i) is the first member of group i,
// off(n) the end of the last.  The groups are shared by `parts` workgroups of 256 threads (a thread per small group) or by
// `waves` wavefronts (one per larger group).
template <typename Off>
__device__ __forceinline__ void finish_small_groups(int n, int g0, int part, int parts, int t, Off off, const int32_t* arrival,
                                                    const float* reward, const GaStat& st, const GaOut& o) {
  for (int g = part * 256 + t; g < n; g += parts * 256) {
    const int from = off(g), members = off(g + 1) - from;
    if (members > kSmallGroup) continue;
    float mean, sd;
    int best;
    finish_by_thread(
        members, [&](int j) { return arrival[from + j]; }, [&](int j) { return reward[arrival[from + j]]; },
        [&](int rank, int r) { o.perm[from + rank] = r; }, [&](int, int r, float v) { o.adv[r] = v; }, st, &mean, &sd, &best);
    put_stats(o, g0 + g, mean, sd, best);
  }
}

// A wavefront looks at the sizes of up to 64 consecutive groups at once: one group at a time, a million groups of one member
// took 16384 wavefronts 64 dependent pairs of loads each (129 us in rollout order and 206 shuffled, now 52 and 130).
template <typename Off>
__device__ __forceinline__ void finish_large_groups(int n, int g0, int wave, int waves, Off off, const int32_t* arrival,
                                                    const float* reward, const GaStat& st, const GaOut& o) {
  const int lane = threadIdx.x & 63;
  const int per = min(64, (n + waves - 1) / waves);
  for (int64_t first = static_cast<int64_t>(wave) * per; first < n; first += static_cast<int64_t>(waves) * per) {
    int from = 0, members = 0;
    if (lane < per && first + lane < n) {
      from = off(static_cast<int>(first) + lane);
      members = off(static_cast<int>(first) + lane + 1) - from;
    }
    for (uint64_t large = __builtin_amdgcn_ballot_w64(members > kSmallGroup); large != 0; large &= large - 1) {
      const int j = __builtin_ctzll(large);
      const int f = __shfl(from, j, 64), m = __shfl(members, j, 64);
      float mean, sd;
      int best;
      finish_by_wave(
          m, lane, [&](int i) { return arrival[f + i]; }, [&](int i) { return reward[arrival[f + i]]; },
          [&](int r) { return reward[r]; }, o.perm + f, [&](int, int r, float v) { o.adv[r] = v; }, st, &mean, &sd, &best);
      if (lane == 0) put_stats(o, g0 + static_cast<int>(first) + j, mean, sd, best);
    }
  }
}

// Eq. (3): r = alpha * r_team + r_loc.  One fp32 multiplication, then one fp32 addition (never
// contracted to an fma): the result decides which groups count as all-equal and which candidate
// is the arg max, so its rounding is part of the definition.
// reward may be r_team or r_loc itself.
__global__ __launch_bounds__(256) void k_ga_mix(int n, const float* r_team, const float* r_loc, float alpha, float* reward) {
#pragma clang fp contract(off)
  const int r = blockIdx.x * 256 + threadIdx.x;
  if (r < n) {
    const float prod = alpha * r_team[r];
    reward[r] = prod + r_loc[r];
  }
}

struct GaMix {
  const float* r_team;
  const float* r_loc;
  float alpha;
  float* reward_out;
};

// the reward of response r: given, or mixed by Eq. (3)
__device__ __forceinline__ float reward_of(const GaArgs& a, const GaMix& mix, int r) {
#pragma clang fp contract(off)
  if (!mix.r_team) return a.reward[r];
  const float prod = mix.alpha * mix.r_team[r];
  return prod + mix.r_loc[r];
}

// ------------------------------------------------------------------------------------------------
// The sizes a training step has, in one launch (two beyond 4096 responses, so that the keys are only computed once).
// Workgroup b owns the keys [b * n_own, (b + 1) * n_own).  It scans the keys of all responses, counts those that are
// smaller and marks which smaller ones occur (one bit each): that is all it needs to know of the others to place its own
// groups.  Its own members go through an LDS list.  Bound by latency: launches, the scan (from L2), a dozen workgroup
// barriers.  Whole calls: 128 responses 43 -> 16 us (the outputs were cleared by fills of their own), 20480 mixed rewards
// 71 -> 23 us (seven launches and the fills before).  The kernel itself with the keys held from one pass to the next and one scan
// for all four sums: 64 responses 7.4 -> 6.6 us, 20480 14.6 -> 13.0, 8100 groups of one 11.8 -> 10.2, 32000 shuffled 25.3 -> 24.7.
// ------------------------------------------------------------------------------------------------
constexpr int kRangeMaxResp = 65536, kRangeMaxKeys = 65528;
constexpr int kRangeList = 4096;         // members listed in LDS; more go to global scratch
constexpr int kRangeDirect = 4096;       // responses up to which every workgroup computes the keys itself
constexpr int kRangeFew = 1024;          // responses up to which 256 threads do
constexpr int kRangeRounds = 4;          // responses per thread whose ids are in flight together
static_assert(kRangeFew <= kRangeRounds * 256 && kRangeDirect <= kRangeRounds * 1024, "the keys of all responses stay in registers");
constexpr int kRangeKept = kRangeMaxResp / 8 / 1024;      // pieces of eight keys that a thread of 1024 holds from one pass to the next
constexpr int kRangeOwn = 128;           // keys of a workgroup beyond which its list may be left to the whole grid
constexpr int kRangeBlocks = 512;        // workgroups of such calls: 256 responses or 1024 keys each (more than kRangeOwn)
static_assert(kRangeMaxKeys / kRangeOwn <= kRangeBlocks, "one word pair each");
constexpr int kLeftBlocks = 128;         // workgroups that finish what others left (512: the launch that finds nothing to do takes
                                         // 4 us instead of 2)

// key of a response in 16 bits, or why it has none
enum : int { kKeyNone = 0xfffd, kKeyBadReward = 0xfffe, kKeyBadId = 0xffff };

__device__ __forceinline__ int key16(const GaArgs& a, const GaMix& mix, int r, float* x) {
  bool ok;
  const int64_t key = key_of(a, r, &ok);
  *x = reward_of(a, mix, r);
  return !ok ? kKeyBadId : (!finite_reward(*x) ? kKeyBadReward : static_cast<int>(key));
}

// the keys of all responses, padded to a multiple of 8 (the array holds 256 bytes at the least); the mixed rewards, which may
// take the place of what they are mixed from
__global__ __launch_bounds__(256) void k_ga_keys(GaArgs a, GaMix mix, uint16_t* __restrict__ keys) {
  const int r = blockIdx.x * 256 + threadIdx.x;
  if (r >= (a.n_resp + 7) / 8 * 8) return;
  float x = 0.f;
  const int key = r < a.n_resp ? key16(a, mix, r, &x) : kKeyNone;
  keys[r] = static_cast<uint16_t>(key);
  if (mix.reward_out && r < a.n_resp) mix.reward_out[r] = x;
}

// eight keys that are all the same (responses of a larger group side by side): counted at once, since 64 lanes' atomics on one LDS
// word take turns (65536 responses in groups of 256, all in one workgroup's keys: its kernel 115 -> 73 us)
__device__ __forceinline__ bool all_equal(const uint4& v) {
  return v.x == v.y && v.x == v.z && v.x == v.w && (v.x >> 16) == (v.x & 0xffff);
}

struct RangeSums {
  int below, g_below, own_groups, own_members, g_own, f_own;
};

// Sums of `below` and `bits` over the workgroup, exclusive prefixes and sums of (c > 0) and c: one barrier, where four scans took eight.
template <int NT>
__device__ __forceinline__ RangeSums range_sums(int below, int bits, int c, int (&lds)[3][NT / 64]) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  constexpr int kShift = 17;                        // c adds up to kRangeMaxResp at most
  static_assert(kRangeMaxResp < (1 << kShift) && NT <= (1 << (31 - kShift - 1)), "both prefixes fit a word");
  const int v = (c > 0 ? 1 << kShift : 0) + c;
  int incl = v;
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) {
    const int up = __shfl_up(incl, o, 64);
    if (lane >= o) incl += up;
    below += __shfl_xor(below, o, 64);
    bits += __shfl_xor(bits, o, 64);
  }
  if (lane == 63) {
    lds[0][wave] = incl;
    lds[1][wave] = below;
    lds[2][wave] = bits;
  }
  __syncthreads();
  RangeSums s{0, 0, 0, 0, 0, 0};
  int before = incl - v, total = 0;
#pragma unroll
  for (int w = 0; w < NT / 64; ++w) {
    const int t = lds[0][w];
    before += w < wave ? t : 0;
    total += t;
    s.below += lds[1][w];
    s.g_below += lds[2][w];
  }
  constexpr int kMask = (1 << kShift) - 1;
  s.own_groups = total >> kShift;
  s.own_members = total & kMask;
  s.g_own = before >> kShift;
  s.f_own = before & kMask;
  return s;
}

// NT threads, each with at most one own key.  keys16: the keys (then a.reward holds the rewards), or null.
// Where the responses lie in the key range is only seen here: a workgroup whose members do not fit its list finishes them out of
// global scratch, or, with `left`, leaves them to k_ga_left and says which groups those are: left[2 b] groups from left[2 b + 1].
template <int NT>
__global__ __launch_bounds__(NT) void k_ga_range(GaArgs a, GaMix mix, GaStat st, int n_keys, int n_own,
                                                 const uint16_t* __restrict__ keys16, int32_t* __restrict__ err,
                                                 int32_t* __restrict__ arrival, int32_t* __restrict__ left, GaOut o) {
  __shared__ int present[(kRangeMaxKeys + 31) / 32];
  __shared__ int count[NT], cursor[NT], first[NT], gid[NT];
  __shared__ int list_id[kRangeList];
  __shared__ float list_x[kRangeList];
  __shared__ int lds_sums[3][NT / 64];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int b = blockIdx.x, lo = b * n_own, own = min(n_own, n_keys - lo);
  for (int k = tid; k < (lo + 31) / 32; k += NT) present[k] = 0;
  count[tid] = 0;
  __syncthreads();

  int keys[kRangeRounds];          // without keys16
  int below = 0, bad = 0;
  // (keys that stand for "none" are above every range); workgroup 0 has no smaller keys and looks for bad ones instead
  auto look = [&](int key, bool new_run, int members) {
    below += key < lo ? members : 0;
    const unsigned d = static_cast<unsigned>(key - lo);
    if (d < static_cast<unsigned>(own)) atomicAdd(&count[d], members);
    if (b == 0) {
      bad |= key == kKeyBadId ? AT_GRPO_DATA_ID_RANGE : (key == kKeyBadReward ? AT_GRPO_DATA_REWARD : 0);
    } else if (key < lo && new_run) {
      atomicOr(&present[key >> 5], 1 << (key & 31));   // once per run of equal keys
    }
  };
  uint4 kept[kRangeKept];          // with keys16: eight keys each
  if (keys16) {
    const int pieces = (a.n_resp + 7) / 8;
#pragma unroll
    for (int u = 0; u < kRangeKept; ++u)
      if (u * NT < pieces) kept[u] = reinterpret_cast<const uint4*>(keys16)[min(u * NT + tid, pieces - 1)];
#pragma unroll
    for (int u = 0; u < kRangeKept; ++u) {
      if (u * NT + tid >= pieces) break;
      const uint4 v = kept[u];
      if (all_equal(v)) {
        look(v.x & 0xffff, true, 8);
        continue;
      }
      const uint32_t w[4] = {v.x, v.y, v.z, v.w};
      int prev = -1;
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        const int key = (w[e >> 1] >> (16 * (e & 1))) & 0xffff;
        look(key, key != prev, 1);
        prev = key;
      }
    }
  } else {
    float x[kRangeRounds];
#pragma unroll
    for (int u = 0; u < kRangeRounds; ++u) {
      const int r = u * NT + tid;
      x[u] = 0.f;
      keys[u] = r < a.n_resp ? key16(a, mix, r, &x[u]) : kKeyNone;
    }
#pragma unroll
    for (int u = 0; u < kRangeRounds; ++u) {
      const int r = u * NT + tid;
      if (mix.reward_out && r < a.n_resp && b == 0) mix.reward_out[r] = x[u];
      const int prev = __shfl_up(keys[u], 1, 64);
      look(keys[u], lane == 0 || prev != keys[u], 1);
    }
  }
  __syncthreads();                 // every bit is set
  int bits = 0;
  for (int k = tid; k < (lo + 31) / 32; k += NT) bits += __popc(present[k]);
  // smaller keys: members and groups, a word each; own keys: dense ids and offsets, at most 1024 groups above at most 65536 members in
  // one word.  One scan for the three
  const int c = tid < own ? count[tid] : 0;
  const RangeSums sums = range_sums<NT>(below, bits, c, lds_sums);
  below = sums.below;
  const int g_below = sums.g_below, own_groups = sums.own_groups, own_members = sums.own_members, g_own = sums.g_own, f_own = sums.f_own;
  first[tid] = f_own;
  cursor[tid] = f_own;
  gid[tid] = g_below + g_own;
  if (c > 0) o.seg_offsets[g_below + g_own] = below + f_own;
  const bool in_lds = own_members <= kRangeList;
  __syncthreads();

  // list the own members
  auto enlist = [&](int r0, int key, int members) {    // responses r0 .. of one key
    const unsigned d = static_cast<unsigned>(key - lo);
    if (d < static_cast<unsigned>(own)) {
      const int at = atomicAdd(&cursor[d], members);
      for (int e = 0; e < members; ++e) {
        if (in_lds) list_id[at + e] = r0 + e;
        else arrival[below + at + e] = r0 + e;
        o.group_id[r0 + e] = gid[d];
      }
    }
    if (b == 0 && key > kKeyNone) {
      for (int e = 0; e < members; ++e) {
        o.group_id[r0 + e] = -1;
        o.adv[r0 + e] = 0.f;
      }
    }
  };
  if (keys16) {
#pragma unroll
    for (int u = 0; u < kRangeKept; ++u) {
      const int cc = u * NT + tid;
      if (cc * 8 >= a.n_resp) break;
      const uint4 v = kept[u];
      if (all_equal(v)) {
        enlist(cc * 8, v.x & 0xffff, 8);
        continue;
      }
      const uint32_t w[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
      for (int e = 0; e < 8; ++e) enlist(cc * 8 + e, (w[e >> 1] >> (16 * (e & 1))) & 0xffff, 1);
    }
  } else {
#pragma unroll
    for (int u = 0; u < kRangeRounds; ++u) enlist(u * NT + tid, keys[u], 1);
  }
  __syncthreads();
  if (in_lds) {      // all rewards at once: one load latency instead of one per member met above
    for (int i = tid; i < own_members; i += NT) list_x[i] = reward_of(a, mix, list_id[i]);
    __syncthreads();
  }

  auto reward = [&](int r) { return reward_of(a, mix, r); };
  auto finish = [&](auto id_of, auto x_of) {
    if (c > 0 && c <= kSmallGroup) {
      float mean, sd;
      int best;
      int32_t* perm = o.perm + below + f_own;
      finish_by_thread(
          c, [&](int j) { return id_of(f_own + j); }, [&](int j) { return x_of(f_own + j); },
          [&](int rank, int r) { perm[rank] = r; }, [&](int, int r, float v) { o.adv[r] = v; }, st, &mean, &sd, &best);
      put_stats(o, g_below + g_own, mean, sd, best);
    }
    for (int k = wave; k < own; k += NT / 64) {
      const int n = count[k], f = first[k];
      if (n <= kSmallGroup) continue;
      float mean, sd;
      int best;
      finish_by_wave(
          n, lane, [&](int j) { return id_of(f + j); }, [&](int j) { return x_of(f + j); }, reward, o.perm + below + f,
          [&](int, int r, float v) { o.adv[r] = v; }, st, &mean, &sd, &best);
      if (lane == 0) put_stats(o, gid[k], mean, sd, best);
    }
  };
  if (left && tid == 0) {
    left[2 * b] = in_lds ? 0 : own_groups;
    left[2 * b + 1] = g_below;
  }
  if (in_lds) finish([&](int j) { return list_id[j]; }, [&](int j) { return list_x[j]; });
  else if (!left) finish([&](int j) { return arrival[below + j]; }, [&](int j) { return reward(arrival[below + j]); });

  if (b == 0) {
    const int id_bad = __syncthreads_or(bad & AT_GRPO_DATA_ID_RANGE), x_bad = __syncthreads_or(bad & AT_GRPO_DATA_REWARD);
    if (tid == 0) *err = (id_bad ? AT_GRPO_DATA_ID_RANGE : 0) | (x_bad ? AT_GRPO_DATA_REWARD : 0);
  }
  if (b == static_cast<int>(gridDim.x) - 1) {
    const int G = g_below + own_groups, listed = below + own_members;
    if (tid == 0) {
      *o.n_groups = G;
      o.seg_offsets[G] = listed;
    }
    fill_tails(o, G, listed, a.n_resp, tid, NT);
  }
}

// The groups that workgroups of k_ga_range left, shared by the grid.
__global__ __launch_bounds__(256) void k_ga_left(int n_blocks, const int32_t* __restrict__ left, const int32_t* __restrict__ arrival,
                                                 const float* __restrict__ reward, GaStat st, GaOut o) {
  __shared__ int groups[kRangeBlocks];
  int any = 0;
  for (int b = threadIdx.x; b < n_blocks; b += 256) any |= groups[b] = left[2 * b];
  if (!__syncthreads_or(any)) return;
  for (int b = 0; b < n_blocks; ++b) {
    const int n = groups[b];
    if (n == 0) continue;
    const int g0 = left[2 * b + 1];
    auto off = [&](int g) { return o.seg_offsets[g0 + g]; };
    finish_small_groups(n, g0, static_cast<int>(blockIdx.x), static_cast<int>(gridDim.x), threadIdx.x, off, arrival, reward, st, o);
    finish_large_groups(n, g0, static_cast<int>(blockIdx.x * 256 + threadIdx.x) >> 6, static_cast<int>(gridDim.x) * 4, off, arrival,
                        reward, st, o);
  }
}

// ------------------------------------------------------------------------------------------------
// Pools.  A response needs four accesses at unrelated addresses if histogram, ranks, lists and results live in global memory
// (2^22 shuffled responses: 440 us on the stream).  Instead the responses are partitioned by key range ("bins" of 3072 to 4096
// responses) with LDS counters, so that every run written is a few entries long; each bin is finished by one workgroup in
// LDS; and one last pass in response order gathers the results, again in runs.  About 84 bytes per response, all streamed.
// Whole calls in groups of 8, shuffled and in rollout order (in brackets: the histogram path): 2^20 responses 69 and 47 us (113
// and 57), 2^22 159 and 118 (454 and 120), 2^24 614 and 400 (2054 and 453).
//
// How many responses a bin has depends on where the ids lie in their extents, which only the device sees.  Bins that do not
// fit LDS (a pool from a part of the extents, say) are therefore not left to one workgroup: from the partition on their
// responses go the way of the histogram path (ranks from global counters, member lists by group, groups shared by the whole
// grid), inside the launches that the other bins need anyway.  262144 responses in groups of 128 that lie in one bin of
// 2^19 keys: 8275 us by one workgroup, 57 now; in groups of 8 from a quarter of their extents, in rollout order and shuffled: 2^20
// responses 104 and 138 us by a workgroup per bin, 54 and 115 now, 2^22 176 and 351, now 126 and 441 (130 and 461 by histogram).
// ------------------------------------------------------------------------------------------------
constexpr int kPoolThreads = 1024;       // of a partitioning workgroup
constexpr int kPoolMaxBins = 4096, kPoolMinBins = 256, kPoolRound = 512;
constexpr int kPoolPerBin = 4096, kPoolFewPerBin = 3072;      // responses per bin
constexpr int kPoolMaxKeys = 2048;       // keys of a bin
constexpr int kPoolCap = 6016;           // responses of a bin that fit its lists; a bin with more is "large"
constexpr int kBinThreads = 512, kBinPer = (kPoolCap + kBinThreads - 1) / kBinThreads;
static_assert(kPoolMaxKeys <= kPoolCap, "a large bin has more responses than keys");
static_assert(kPoolCap < 65536 && kPoolMaxKeys < 32768, "place and group share a word");
constexpr int kLargeBlocks = 1024;       // workgroups that finish the groups of the large bins (2^22 responses in 342 large bins:
                                         // 148 us, with 512 workgroups 170)

constexpr int kTicketBins = 32;    // bins that draw tickets from one counter (one for all: 446 us instead of 441 where all bins are large)
constexpr int kSortPer = 16;       // responses per thread of the pools whose blocks are sorted
constexpr int kSortUsed = kPoolThreads * kSortPer / 64;      // bins that a sorted block uses at the least (runs of 64)
constexpr int kSortLds = (2 * kPoolThreads * kSortPer + kPoolMaxBins) * 4, kTurnLds = kPoolThreads * kSortPer * 8;

struct PoolPlan {
  int width, bins;           // bin of a key = key / width
  int per;                   // responses per thread of a partitioning workgroup, a multiple of 4
  int32_t* key;              // [R]
  int32_t* slot;             // [R] place of the response in the partitioned order; of a large bin: bit 31 and rank inside its group.
                             // Of a sorted block (see k_gp_partition): places of its responses in ascending order
  uint16_t* member;          // [R] of a sorted block: which response of the block has that place
  int32_t* sorted;           // [blocks] of a sorted block (one that may be one, before it is partitioned): its responses with a key (0),
                             // else -1
  int32_t* list;             // [R] members of the large bins, by group
  int32_t* hist;             // [keys] of a large bin: members
  int2* kr;                  // [R] (key, response), partitioned.  Of a large bin: (first member's place in `list`, group inside the bin)
                             // of its keys in turn, which are fewer than its responses
  float* x;                  // [R] rewards, partitioned
  float2* result;            // [R] (advantage, group inside the bin), partitioned
  float4* stats;             // [R] (mean, std, best, offset) of group i of the bin at bin_base + i
  int32_t* blk;              // [blocks][bins]
  int32_t* bin_cnt;          // [bins]
  int32_t* bin_base;         // [bins + 1]
  int32_t* cursor;           // [bins] of a large bin: has it groups of more than kSmallGroup?
  int32_t* bin_groups;       // [bins]
  int32_t* gid_base;         // [bins + 1]
  int32_t* bins_done;        // workgroups of k_gp_bin that have counted their groups: [1 + i] of the bins of i in turn, [0] full ones
  int32_t* large;            // [bins + 1] number of large bins, then which ones they are
};

// atomicAdd(&counter[bin], 1) of every active lane.  In rollout order all lanes of a wavefront name the same bin, and 64 atomics
// on one LDS word take turns: the lanes that agree with the first one share a single addition
// (300000 responses over 37500 keys in rollout order 65 -> 55 us, shuffled 74 -> 72).
__device__ __forceinline__ int count_in_bin(int* counter, int bin) {
  const int first = __builtin_amdgcn_readfirstlane(bin);
  const uint64_t same = __builtin_amdgcn_ballot_w64(bin == first);
  if (bin != first) return atomicAdd(&counter[bin], 1);
  const int lane = threadIdx.x & 63;
  int at = 0;
  if ((same & ((uint64_t{1} << lane) - 1)) == 0) at = atomicAdd(&counter[first], static_cast<int>(__popcll(same)));
  return __builtin_amdgcn_readfirstlane(at) + static_cast<int>(__popcll(same & ((uint64_t{1} << lane) - 1)));
}

__global__ __launch_bounds__(kPoolThreads) void k_gp_init(int32_t* __restrict__ bin_cnt, int bins, int32_t* __restrict__ err) {
  for (int i = threadIdx.x; i < bins; i += kPoolThreads) bin_cnt[i] = 0;
  if (threadIdx.x == 0) *err = 0;
}

__global__ __launch_bounds__(kPoolThreads) void k_gp_count(GaArgs a, GaMix mix, PoolPlan p, int32_t* __restrict__ err) {
  __shared__ int hist[kPoolMaxBins];
  __shared__ int used;
  for (int i = threadIdx.x; i < p.bins; i += kPoolThreads) hist[i] = 0;
  __syncthreads();
  const int64_t r0 = static_cast<int64_t>(blockIdx.x) * kPoolThreads * p.per + threadIdx.x;
  int bad = 0;
#pragma unroll 4
  for (int u = 0; u < p.per; ++u) {
    const int64_t r = r0 + u * kPoolThreads;
    if (r < a.n_resp) {
      bool ok;
      const int64_t k64 = key_of(a, static_cast<int>(r), &ok);
      const float x = reward_of(a, mix, static_cast<int>(r));
      if (mix.reward_out) mix.reward_out[r] = x;
      int key = -1;
      if (!ok) bad |= AT_GRPO_DATA_ID_RANGE;
      else if (!finite_reward(x)) bad |= AT_GRPO_DATA_REWARD;
      else key = static_cast<int>(k64);
      p.key[r] = key;
      if (key >= 0) count_in_bin(hist, static_cast<int>(static_cast<unsigned>(key) / static_cast<unsigned>(p.width)));
    }
  }
  if (bad) atomicOr(err, bad);
  if (threadIdx.x == 0) used = 0;
  __syncthreads();
  int mine = 0;
  for (int i = threadIdx.x; i < p.bins; i += kPoolThreads) {
    const int c = hist[i];
    p.blk[static_cast<size_t>(blockIdx.x) * p.bins + i] = c;
    if (c) atomicAdd(&p.bin_cnt[i], c);
    mine += c ? 1 : 0;
  }
  if (p.per == kSortPer) {
    if (mine) atomicAdd(&used, mine);
    __syncthreads();
    if (threadIdx.x == 0) p.sorted[blockIdx.x] = used >= kSortUsed ? 0 : -1;
  }
}

// exclusive scan of n <= kPoolMaxBins counts `in(i)` by one workgroup of NT threads; out[n] = total, which is returned
template <int NT, typename In>
__device__ __forceinline__ int scan_small(In in, int n, int32_t* out, int32_t* out2, int* lds) {
  constexpr int kPer = kPoolMaxBins / NT;
  int v[kPer], sum = 0;
#pragma unroll
  for (int e = 0; e < kPer; ++e) {
    const int i = threadIdx.x * kPer + e;
    v[e] = i < n ? in(i) : 0;
    sum += v[e];
  }
  int total;
  int at = block_exclusive_scan<NT>(sum, lds, &total);
#pragma unroll
  for (int e = 0; e < kPer; ++e) {
    const int i = threadIdx.x * kPer + e;
    if (i < n) {
      out[i] = at;
      if (out2) out2[i] = at;
    }
    at += v[e];
  }
  if (threadIdx.x == 0) out[n] = total;
  return total;
}

// workgroup 0: bases of the bins, list of the large ones; the others clear the counters of the large bins' keys, a wavefront per
// bin
constexpr int kBasesBins = kPoolThreads / 64;

__global__ __launch_bounds__(kPoolThreads) void k_gp_bases(PoolPlan p, int64_t n_keys) {
  __shared__ int lds16[16];
  __shared__ int n_large;
  if (blockIdx.x == 0) {
    if (threadIdx.x == 0) n_large = 0;
    if (threadIdx.x <= kPoolMaxBins / kTicketBins) p.bins_done[threadIdx.x] = 0;
    scan_small<kPoolThreads>([&](int i) { return p.bin_cnt[i]; }, p.bins, p.bin_base, p.cursor, lds16);
    __syncthreads();
    for (int i = threadIdx.x; i < p.bins; i += kPoolThreads)
      if (p.bin_cnt[i] > kPoolCap) p.large[1 + atomicAdd(&n_large, 1)] = i;
    __syncthreads();
    if (threadIdx.x == 0) p.large[0] = n_large;
    return;
  }
  const int bin = (blockIdx.x - 1) * kBasesBins + (threadIdx.x >> 6);
  if (bin >= p.bins || p.bin_cnt[bin] <= kPoolCap) return;
  const int64_t lo = static_cast<int64_t>(bin) * p.width, end = min(lo + p.width, n_keys);
  for (int64_t k = lo + (threadIdx.x & 63); k < end; k += 64) p.hist[k] = 0;
}

// every response of the block stored where it belongs; next: [bins] in LDS
__device__ __forceinline__ void partition_block(int n_resp, const float* __restrict__ reward, const PoolPlan& p, int* next) {
  for (int i = threadIdx.x; i < p.bins; i += kPoolThreads) {
    const int c = p.blk[static_cast<size_t>(blockIdx.x) * p.bins + i];
    next[i] = c == 0 ? 0 : (p.bin_cnt[i] > kPoolCap ? INT32_MIN : atomicAdd(&p.cursor[i], c));   // places in large bins: below zero
  }
  __syncthreads();
  const int64_t r0 = static_cast<int64_t>(blockIdx.x) * kPoolThreads * p.per + threadIdx.x;
  for (int u0 = 0; u0 < p.per; u0 += 4) {
    int key[4];
    float x[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const int64_t r = r0 + (u0 + u) * kPoolThreads;
      key[u] = r < n_resp ? p.key[r] : -1;
      x[u] = r < n_resp ? reward[r] : 0.f;
    }
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const int r = static_cast<int>(r0 + (u0 + u) * kPoolThreads);
      int at = 0;
      if (key[u] >= 0) {
        at = count_in_bin(next, static_cast<int>(static_cast<unsigned>(key[u]) / static_cast<unsigned>(p.width)));
        if (at >= 0) {
          p.kr[at] = make_int2(key[u], r);
          p.x[at] = x[u];
          p.slot[r] = at;
        }
      }
      if (__builtin_amdgcn_ballot_w64(at < 0) != 0) {
        const int rank = count_runs(p.hist, at < 0 ? key[u] : -1);
        if (at < 0) p.slot[r] = INT32_MIN | rank;
      }
    }
  }
}

// A block of the largest pools whose responses lie in many bins (shuffled, it has 16 responses per bin): stored one by one where
// they belong, the lanes' stores would reach 1024 places a run apart, each a little at a time, and the L2 of an XCD does not hold
// the lines that its 32 workgroups have begun.  Such a block is sorted by bin in LDS first, and leaves field by field in whole
// runs; its results come back the same way (k_gp_turn).  Shuffled pools in groups of 8, partition and results in response order:
// 2^22 93 + 55 us one by one, 48 + 30 sorted; 2^24 524 + 279 and 222 + 149.  Bound by the latency of its passes through LDS, one
// workgroup on each compute unit.  Other blocks gain nothing: in rollout order consecutive lanes have consecutive places, and
// blocks with members of large bins rank them one by one in any case.  Pools of less than 2.4 million have fewer responses per
// block, and runs that stay in L2 (2^20 shuffled: 20 us, 31 sorted).
// ALL: blocks that are not sorted are done here too; otherwise they are left to k_gp_partition, which takes two workgroups per
// compute unit where this one's LDS leaves room for one (2^24 in rollout order: 69 us, here 100).
template <bool ALL>
__global__ __launch_bounds__(kPoolThreads) void k_gp_partition_sorted(int n_resp, const float* __restrict__ reward, PoolPlan p) {
  constexpr int PER = kSortPer, B = kPoolThreads * PER;
  extern __shared__ __attribute__((aligned(16))) int lds[];
  __shared__ int lds16[16];
  int* place = lds;                // [B]
  int* field = lds + B;            // [B]; until the places are known: distance of a bin's places from its local ones
  int* next = lds + 2 * B;         // [bins], at most kPoolMaxBins
  const int tid = threadIdx.x;
  if (p.sorted[blockIdx.x] < 0) {
    if (ALL) partition_block(n_resp, reward, p, next);
    return;
  }
  const int32_t* blk = p.blk + static_cast<size_t>(blockIdx.x) * p.bins;
  const int64_t block0 = static_cast<int64_t>(blockIdx.x) * B, r0 = block0 + tid;
  // each thread owns a run of bins
  constexpr int kPer = kPoolMaxBins / kPoolThreads;
  int c[kPer], members = 0;
  bool large = false;
#pragma unroll
  for (int e = 0; e < kPer; ++e) {
    const int i = tid * kPer + e;
    c[e] = i < p.bins ? blk[i] : 0;
    members += c[e];
    large = large || (c[e] > 0 && p.bin_cnt[i] > kPoolCap);
  }
  if (__syncthreads_or(large)) {
    if (tid == 0) p.sorted[blockIdx.x] = -1;
    if (ALL) partition_block(n_resp, reward, p, next);
    return;
  }
  int key[PER];
  float x[PER];
#pragma unroll
  for (int u = 0; u < PER; ++u) {
    const int64_t r = r0 + u * kPoolThreads;
    key[u] = r < n_resp ? p.key[r] : -1;
    x[u] = r < n_resp ? reward[r] : 0.f;
  }
  int total;
  int at = block_exclusive_scan<kPoolThreads>(members, lds16, &total);
  if (tid == 0) p.sorted[blockIdx.x] = total;
#pragma unroll
  for (int e = 0; e < kPer; ++e) {
    const int i = tid * kPer + e;
    if (i >= p.bins) continue;
    next[i] = at;
    if (c[e] > 0) field[i] = atomicAdd(&p.cursor[i], c[e]) - at;
    at += c[e];
  }
  __syncthreads();
  int local[PER];                  // place inside the block, in the order of the bins
#pragma unroll
  for (int u = 0; u < PER; ++u) {
    local[u] = -1;
    if (key[u] < 0) continue;
    const int bin = static_cast<int>(static_cast<unsigned>(key[u]) / static_cast<unsigned>(p.width));
    local[u] = atomicAdd(&next[bin], 1);
    place[local[u]] = local[u] + field[bin];
  }
  __syncthreads();
  int to[PER];
#pragma unroll
  for (int i = 0; i < PER; ++i) {
    const int j = tid + i * kPoolThreads;
    to[i] = j < total ? place[j] : -1;
    if (j >= total && block0 + j < n_resp) p.slot[block0 + j] = 0;      // not a place in a large bin
  }
  // one field after the other goes through LDS into that order and out
  auto leave = [&](auto value, auto put) {
#pragma unroll
    for (int u = 0; u < PER; ++u)
      if (local[u] >= 0) field[local[u]] = value(u);
    __syncthreads();
#pragma unroll
    for (int i = 0; i < PER; ++i)
      if (to[i] >= 0) put(i, to[i], field[tid + i * kPoolThreads]);
    __syncthreads();
  };
  leave([&](int u) { return __float_as_int(x[u]); }, [&](int, int t, int v) { p.x[t] = __int_as_float(v); });
  int k_out[PER];
  leave([&](int u) { return key[u]; }, [&](int i, int, int v) { k_out[i] = v; });
  leave([&](int u) { return tid + u * kPoolThreads; },
        [&](int i, int t, int v) {
          const int64_t j = block0 + tid + i * kPoolThreads;
          p.kr[t] = make_int2(k_out[i], static_cast<int>(block0) + v);
          p.slot[j] = t;
          p.member[j] = static_cast<uint16_t>(v);
        });
}

// sorted: blocks that k_gp_partition_sorted has done are skipped
__global__ __launch_bounds__(kPoolThreads) void k_gp_partition(int n_resp, const float* __restrict__ reward, PoolPlan p, int sorted) {
  __shared__ int next[kPoolMaxBins];
  if (sorted && p.sorted[blockIdx.x] >= 0) return;
  partition_block(n_resp, reward, p, next);
}

// Place of list entry f in LDS.  A thread walks its own group, so 64 lanes read entries that lie a group's size apart; groups of
// 8 would meet in 8 of the 64 banks.
__device__ __forceinline__ int bin_at(int f) { return f ^ ((f >> 6) & 7); }
static_assert(kPoolCap % 8 == 0, "entries move inside blocks of eight");

__global__ __launch_bounds__(kBinThreads, 4) void k_gp_bin(PoolPlan p, const float* __restrict__ reward, GaStat st, int64_t n_keys,
                                                        GaOut o) {
  __shared__ int list_id[kPoolCap];
  __shared__ float list_x[kPoolCap];
  __shared__ int count[kPoolMaxKeys], next[kPoolMaxKeys];
  __shared__ uint16_t gid[kPoolMaxKeys];
  __shared__ int wsum[2][kBinThreads / 64];
  __shared__ int last;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int bin = blockIdx.x, base = p.bin_base[bin], m = p.bin_base[bin + 1] - base;
  const int lo = bin * p.width;
  const int own = static_cast<int>(min(static_cast<int64_t>(p.width), n_keys - lo));
  // The workgroup that is the last to have counted its bin's groups turns the counts into ids of first groups: 3 to 5 us in this
  // launch, where one of its own took 6.5 and its gap.  Only the counts have to be in order with the tickets, and they are atomics,
  // performed where all XCDs meet.  So it takes no more than that the exchange has returned before the ticket is drawn: the
  // statement between them needs its result, and no access to memory passes it in either direction.  (With a release on the ticket
  // and an acquire on the last one instead, every workgroup writes its L2 back: 2^22 shuffled 159 -> 176 us, in rollout order 120 ->
  // 138, 2^24 620 -> 757 and 403 -> 537.)  The reading side is behind the barrier that hands `last` on.
  int before = 0, ticket = 0;
  auto publish = [&](int n_groups) { if (tid == 0) before = atomicExch(&p.bin_groups[bin], n_groups); };
  auto draw = [&] {
    if (tid != 0) return;
    asm volatile("" : "+v"(before) : : "memory");
    ticket = atomicAdd(&p.bins_done[1 + bin / kTicketBins], 1);
  };
  auto scan_if_last = [&] {
    if (tid == 0) {
      const int first = bin / kTicketBins * kTicketBins;
      last = ticket == min(kTicketBins, p.bins - first) - 1 &&
             atomicAdd(p.bins_done, 1) == (p.bins + kTicketBins - 1) / kTicketBins - 1;
    }
    __syncthreads();
    if (!last) return;
    const int G = scan_small<kBinThreads>(
        [&](int i) { return __hip_atomic_load(&p.bin_groups[i], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }, p.bins, p.gid_base,
        nullptr, wsum[0]);
    if (tid != 0) return;
    *o.n_groups = G;
    o.seg_offsets[G] = p.bin_base[p.bins];
  };
  if (m == 0) {
    publish(0);
    draw();
    scan_if_last();
    return;
  }
  const bool large = m > kPoolCap;
  for (int k = tid; k < own; k += kBinThreads) count[k] = large ? p.hist[lo + k] : 0;
  __syncthreads();
  // The bin's members stay in registers from here on: one wait for memory instead of one per pass and member.  2^24 responses in
  // rollout order: 245 us with three reads of kr and the members' order stored from here one by one, 156 with kr in registers,
  // 147 with whole lines of perm (512 threads; 215 with 1024, whose groups leave half of them idle).
  int2 kr[kBinPer];
  float x[kBinPer];
  if (!large) {
#pragma unroll
    for (int i = 0; i < kBinPer; ++i) {
      const int e = tid + i * kBinThreads;
      kr[i] = e < m ? p.kr[base + e] : make_int2(-1, 0);
      x[i] = e < m ? p.x[base + e] : 0.f;
    }
#pragma unroll
    for (int i = 0; i < kBinPer; ++i)
      if (kr[i].x >= 0) atomicAdd(&count[kr[i].x - lo], 1);
  }
  __syncthreads();
  // offsets and ids of the keys that occur: each thread owns a run of keys
  constexpr int kPer = kPoolMaxKeys / kBinThreads;
  int c[kPer], members = 0, groups = 0;
#pragma unroll
  for (int e = 0; e < kPer; ++e) {
    const int k = tid * kPer + e;
    c[e] = k < own ? count[k] : 0;
    members += c[e];
    groups += c[e] > 0;
  }
  int im = members, ig = groups;
#pragma unroll
  for (int d = 1; d < 64; d <<= 1) {
    const int um = __shfl_up(im, d, 64), ug = __shfl_up(ig, d, 64);
    if (lane >= d) {
      im += um;
      ig += ug;
    }
  }
  if (lane == 63) {
    wsum[0][wave] = im;
    wsum[1][wave] = ig;
  }
  __syncthreads();
  int at = im - members, g = ig - groups, n_groups = 0;
#pragma unroll
  for (int w = 0; w < kBinThreads / 64; ++w) {
    if (w < wave) {
      at += wsum[0][w];
      g += wsum[1][w];
    }
    n_groups += wsum[1][w];
  }
#pragma unroll
  for (int e = 0; e < kPer; ++e) {
    const int k = tid * kPer + e;
    if (k < own) {
      next[k] = at;
      gid[k] = static_cast<uint16_t>(g);
      if (large && c[e] > 0) {
        p.kr[base + k] = make_int2(base + at, g);
        p.stats[base + g].w = __int_as_float(base + at);
      }
      at += c[e];
      g += c[e] > 0;
    }
  }
  publish(n_groups);
  if (large) {
    bool wave_groups = false;
#pragma unroll
    for (int e = 0; e < kPer; ++e) wave_groups = wave_groups || c[e] > kSmallGroup;
    const int any = __syncthreads_or(wave_groups);
    if (tid == 0) p.cursor[bin] = any;
    draw();
    scan_if_last();
    return;
  }
  __syncthreads();
  int place[kBinPer];        // place in the lists, and the group in the upper half
#pragma unroll
  for (int i = 0; i < kBinPer; ++i) {
    place[i] = -1;
    if (kr[i].x < 0) continue;
    const int k = kr[i].x - lo, f = atomicAdd(&next[k], 1);
    list_id[bin_at(f)] = kr[i].y;
    list_x[bin_at(f)] = x[i];
    place[i] = f | static_cast<int>(gid[k]) << 16;
  }
  __syncthreads();
  // next[k] is now one past the members of key k.  A member's advantage takes the place of its reward, which only its own group
  // reads, and the ordered members of a small group that of its list, so that both leave in whole lines.
  auto id_of = [&](int j) { return list_id[bin_at(j)]; };
  auto x_of = [&](int j) { return list_x[bin_at(j)]; };
  for (int k = tid; k < own; k += kBinThreads) {
    const int n = count[k], f = next[k] - n;
    if (n == 0 || n > kSmallGroup) continue;
    float mean, sd;
    int best;
    finish_by_thread(
        n, [&](int j) { return id_of(f + j); }, [&](int j) { return x_of(f + j); },
        [&](int rank, int r) { list_id[bin_at(f + rank)] = r; }, [&](int j, int, float v) { list_x[bin_at(f + j)] = v; }, st,
        &mean, &sd, &best);
    p.stats[base + gid[k]] = make_float4(mean, sd, __int_as_float(best), __int_as_float(base + f));
  }
  for (int k = wave; k < own; k += kBinThreads / 64) {
    const int n = count[k], f = next[k] - n;
    if (n <= kSmallGroup) continue;
    float mean, sd;
    int best;
    finish_by_wave(
        n, lane, [&](int j) { return id_of(f + j); }, [&](int j) { return x_of(f + j); }, [&](int r) { return reward[r]; },
        o.perm + base + f,
        [&](int j, int, float v) {
          list_x[bin_at(f + j)] = v;
          list_id[bin_at(f + j)] = -1;      // its place among the members is stored already
        },
        st, &mean, &sd, &best);
    if (lane == 0) p.stats[base + gid[k]] = make_float4(mean, sd, __int_as_float(best), __int_as_float(base + f));
  }
  draw();
  __syncthreads();
  for (int e = tid; e < m; e += kBinThreads) {
    const int r = list_id[bin_at(e)];
    if (r >= 0) o.perm[base + e] = r;
  }
#pragma unroll
  for (int i = 0; i < kBinPer; ++i)
    if (place[i] >= 0)
      p.result[base + tid + i * kBinThreads] = make_float2(list_x[bin_at(place[i] & 0xffff)], __int_as_float(place[i] >> 16));
  scan_if_last();
}

// results in response order; the blocks behind `resp_blocks` write the groups of a bin each, the last ones fill the tails.
// Members of the large bins are listed; their advantages and groups are left to k_gp_large.
__global__ __launch_bounds__(256) void k_gp_out(PoolPlan p, int n_resp, int resp_blocks, GaOut o) {
  if (static_cast<int>(blockIdx.x) < resp_blocks) {
    // the loads of a thread's four responses go out together
    if (p.per == kSortPer && p.sorted[blockIdx.x / kSortPer] >= 0) return;      // left to k_gp_turn
    const int64_t r0 = static_cast<int64_t>(blockIdx.x) * 1024 + threadIdx.x;
    int key[4], at[4], gid0[4], first[4];
    float2 res[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const int64_t r = r0 + u * 256;
      key[u] = r < n_resp ? p.key[r] : -1;
      at[u] = r < n_resp ? p.slot[r] : 0;      // no slot without a key
    }
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const bool in_large = key[u] >= 0 && at[u] < 0;
      const int bin = key[u] < 0 ? 0 : static_cast<int>(static_cast<unsigned>(key[u]) / static_cast<unsigned>(p.width));
      gid0[u] = p.gid_base[bin];
      const int2 g = in_large ? p.kr[p.bin_base[bin] + (key[u] - bin * p.width)] : make_int2(0, 0);
      first[u] = g.x;
      res[u] = in_large ? make_float2(0.f, __int_as_float(g.y)) : (key[u] >= 0 ? p.result[at[u]] : make_float2(0.f, 0.f));
    }
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const int64_t r = r0 + u * 256;
      if (r >= n_resp) break;
      if (key[u] < 0) {
        o.group_id[r] = -1;
        o.adv[r] = 0.f;
      } else {
        o.group_id[r] = gid0[u] + __float_as_int(res[u].y);
        if (at[u] >= 0) o.adv[r] = res[u].x;
        else p.list[first[u] + (at[u] & 0x7fffffff)] = static_cast<int>(r);
      }
    }
    return;
  }
  const int bin = blockIdx.x - resp_blocks;
  if (bin < p.bins) {
    const int g0 = p.gid_base[bin], n = p.gid_base[bin + 1] - g0, base = p.bin_base[bin];
    if (p.bin_cnt[bin] > kPoolCap) return;
    for (int i = threadIdx.x; i < n; i += 256) {
      const float4 s = p.stats[base + i];
      o.seg_offsets[g0 + i] = __float_as_int(s.w);
      put_stats(o, g0 + i, s.x, s.y, __float_as_int(s.z));
    }
    return;
  }
  const int64_t tid = static_cast<int64_t>(bin - p.bins) * 256 + threadIdx.x;
  fill_tails(o, p.gid_base[p.bins], p.bin_base[p.bins], n_resp, tid,
             static_cast<int64_t>(gridDim.x - resp_blocks - p.bins) * 256);
}

// The groups of the large bins, shared by `units` units of 256 threads of which this is number `unit`, with thread `t` of them.
__device__ __forceinline__ void finish_large_bins(const PoolPlan& p, const float* __restrict__ reward, const GaStat& st, const GaOut& o,
                                                  int unit, int units, int t) {
  const int n_large = p.large[0];
  if (n_large == 0) return;
  // the bins' first parts come first: consecutive workgroups, which the hardware deals to the XCDs in turn, have equal work
  const int teams = min(n_large, units), parts = units / teams;
  const int part = unit / teams;
  if (part >= parts) return;
  for (int i = unit % teams; i < n_large; i += teams) {
    const int bin = p.large[1 + i], base = p.bin_base[bin], end = p.bin_base[bin + 1];
    const int g0 = p.gid_base[bin], n = p.gid_base[bin + 1] - g0;
    const bool wave_groups = p.cursor[bin] != 0;
    if (part * 256 >= n && !wave_groups) continue;
    auto off = [&](int g) { return g < n ? __float_as_int(p.stats[base + g].w) : end; };
    for (int g = part * 256 + t; g < n; g += parts * 256) o.seg_offsets[g0 + g] = off(g);
    finish_small_groups(n, g0, part, parts, t, off, p.list, reward, st, o);
    if (wave_groups) finish_large_groups(n, g0, part * 4 + (t >> 6), parts * 4, off, p.list, reward, st, o);
  }
}

// A launch of its own: it returns at once where there are no large bins (2 to 5 us), and the registers of the finishing code would cost
// k_gp_out its wavefronts.  Pools whose blocks may be sorted have k_gp_turn do it.
__global__ __launch_bounds__(256) void k_gp_large(PoolPlan p, const float* __restrict__ reward, GaStat st, GaOut o) {
  finish_large_bins(p, reward, st, o, blockIdx.x, gridDim.x, threadIdx.x);
}

// Results of the sorted blocks in response order: read in the order of their places, run by run, and turned in LDS.  Then the
// groups of the large bins: a launch that finds nothing to do takes 4.6 us at 2^22 responses, and one of those is enough.
__device__ __forceinline__ void turn_block(const PoolPlan& p, int n_resp, const GaOut& o, float2* turned) {
  constexpr int PER = kSortPer;
  const int64_t block0 = static_cast<int64_t>(blockIdx.x) * kPoolThreads * PER, r0 = block0 + threadIdx.x;
  const int sorted = p.sorted[blockIdx.x];
  if (sorted < 0) return;
  int at[PER], who[PER];
  float2 res[PER];
#pragma unroll
  for (int i = 0; i < PER; ++i) {
    const int j = threadIdx.x + i * kPoolThreads;
    at[i] = j < sorted ? p.slot[block0 + j] : -1;
  }
#pragma unroll
  for (int i = 0; i < PER; ++i) {
    const int j = threadIdx.x + i * kPoolThreads;
    who[i] = j < sorted ? p.member[block0 + j] : -1;
    res[i] = at[i] >= 0 ? p.result[at[i]] : make_float2(0.f, 0.f);
  }
#pragma unroll
  for (int i = 0; i < PER; ++i)
    if (who[i] >= 0) turned[who[i]] = res[i];
  int key[PER];
#pragma unroll
  for (int u = 0; u < PER; ++u) {
    const int64_t r = r0 + u * kPoolThreads;
    key[u] = r < n_resp ? p.key[r] : -1;
  }
  __syncthreads();
#pragma unroll
  for (int u = 0; u < PER; ++u) {
    const int64_t r = r0 + u * kPoolThreads;
    if (r >= n_resp) break;
    const float2 v = key[u] < 0 ? make_float2(0.f, 0.f) : turned[threadIdx.x + u * kPoolThreads];
    o.group_id[r] = key[u] < 0 ? -1 : p.gid_base[static_cast<unsigned>(key[u]) / static_cast<unsigned>(p.width)] + __float_as_int(v.y);
    o.adv[r] = v.x;
  }
}

__global__ __launch_bounds__(kPoolThreads) void k_gp_turn(PoolPlan p, int n_resp, int blocks, const float* __restrict__ reward, GaStat st, GaOut o) {
  extern __shared__ __attribute__((aligned(16))) float2 turned[];      // [kPoolThreads * kSortPer]
  if (static_cast<int>(blockIdx.x) < blocks) turn_block(p, n_resp, o, turned);
  constexpr int kUnits = kPoolThreads / 256;
  const int sub = static_cast<int>(threadIdx.x) >> 8;
  finish_large_bins(p, reward, st, o, sub * static_cast<int>(gridDim.x) + static_cast<int>(blockIdx.x),
                    kUnits * static_cast<int>(gridDim.x), threadIdx.x & 255);
}

// both finishing roles in one launch: the first n_small blocks take the small groups (a thread each), the next n_large the
// larger ones (a wavefront each), the rest the tails
__global__ __launch_bounds__(256) void k_ga_finish(int n_small, int n_large, int n_resp, const int32_t* __restrict__ arrival,
                                                   const float* __restrict__ reward, GaStat st, GaOut o) {
  const int G = *o.n_groups, b = blockIdx.x;
  auto off = [&](int g) { return o.seg_offsets[g]; };
  if (b < n_small)
    finish_small_groups(G, 0, b, n_small, threadIdx.x, off, arrival, reward, st, o);
  else if (b < n_small + n_large)
    finish_large_groups(G, 0, ((b - n_small) * 256 + static_cast<int>(threadIdx.x)) >> 6, (n_large * 256) >> 6, off, arrival,
                        reward, st, o);
  else
    fill_tails(o, G, o.seg_offsets[G], n_resp, static_cast<int64_t>(b - n_small - n_large) * 256 + threadIdx.x,
               static_cast<int64_t>(gridDim.x - n_small - n_large) * 256);
}

// clears two ranges in one launch
__global__ void k_ga_clear2(int32_t* __restrict__ p, int64_t n, int32_t* __restrict__ q, int64_t nq) {
  const int64_t stride = static_cast<int64_t>(gridDim.x) * blockDim.x;
  for (int64_t i = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x; i < n; i += stride) p[i] = 0;
  for (int64_t i = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x; i < nq; i += stride) q[i] = 0;
}

struct GaPlan {
  int64_t n_keys, n_blocks;
  bool pooled;
  PoolPlan pool;
  int32_t *err, *hist, *gid_of_key, *key_of_resp, *rank_of_resp, *arrival, *bsum_p, *bsum_c;
};

int64_t key_box(int32_t n_env, int32_t n_agent, int32_t n_turn, int32_t group_by, int32_t n_sample) {
  if (group_by == AT_GRPO_GROUP_BY_TRAJECTORY) return n_env;
  const int64_t eit = static_cast<int64_t>(n_env) * n_agent * n_turn;
  if (group_by == AT_GRPO_GROUP_BY_PARALLEL) return n_sample > 0 && eit <= (int64_t{1} << 28) ? eit * n_sample : -1;
  return eit;
}

bool plan(int32_t n_resp, int32_t n_env, int32_t n_agent, int32_t n_turn, int32_t group_by, int32_t n_sample,
          WsAlloc& ws, GaPlan* p) {
  if (n_resp <= 0 || n_env <= 0 || n_agent <= 0 || n_turn <= 0) return false;
  const int64_t n_keys = key_box(n_env, n_agent, n_turn, group_by, n_sample);
  if (n_keys <= 0 || n_keys > (int64_t{1} << 28)) return false;
  p->n_keys = n_keys;
  p->n_blocks = ceil_div(n_keys, kKeysPerBlock);
  p->err = ws.take<int32_t>(64);
  p->hist = ws.take<int32_t>(static_cast<size_t>(n_keys));
  p->gid_of_key = ws.take<int32_t>(static_cast<size_t>(n_keys));
  p->key_of_resp = ws.take<int32_t>(static_cast<size_t>(n_resp));
  p->rank_of_resp = ws.take<int32_t>(static_cast<size_t>(n_resp));
  p->arrival = ws.take<int32_t>(static_cast<size_t>(n_resp));
  p->bsum_p = ws.take<int32_t>(static_cast<size_t>(p->n_blocks));
  p->bsum_c = ws.take<int32_t>(static_cast<size_t>(p->n_blocks));
  return true;
}

// The pool path's scratch, behind the common part; false if the path does not apply: too few responses to fill the chip
// with bins, bins of too many keys, or so few keys that the bins overflow.
bool plan_pool(int32_t n_resp, WsAlloc& ws, GaPlan* p) {
  if (n_resp <= kRangeMaxResp && p->n_keys <= kRangeMaxKeys) return false;
  // Whole rounds of two workgroups per compute unit: a bin takes as long as its members, a started round as long as a full one
  // (2^22 responses in groups of 8, 1366 bins and 1024: in rollout order 120 and 113 us, environments shuffled 130 and 120, all
  // shuffled 243 and 226; 2 million in groups of 24, 652 and 512: 156 and 127).  One workgroup per compute unit does up to
  // 786432 (10^6 responses in groups of two, 256 bins and 512: 71 and 60).  More bins where so few would span too many keys.
  int64_t want = ceil_div(n_resp, kPoolPerBin * kPoolRound) * kPoolRound, most = ceil_div(n_resp, kPoolFewPerBin);
  if (most < kPoolMinBins) most = want = kPoolMinBins;
  if (most > kPoolMaxBins) most = kPoolMaxBins;
  if (want > kPoolMaxBins) want = kPoolMaxBins;
  // about a response per key: the histogram is as fast in any order (10^6 responses in groups of one: 51 us, 75 in bins)
  if (ceil_div(p->n_keys, most) > kPoolMaxKeys) return false;
  if (ceil_div(p->n_keys, want) > kPoolMaxKeys) want = most;
  const int64_t width = ceil_div(p->n_keys, want);
  PoolPlan& q = p->pool;
  q.width = static_cast<int>(width);
  q.bins = static_cast<int>(ceil_div(p->n_keys, width));
  if (n_resp < kRangeMaxResp / 2) return false;
  if (static_cast<int64_t>(n_resp) > static_cast<int64_t>(q.bins) * kPoolCap * 3 / 4) return false;
  // 16 responses per thread make the longest runs; smaller pools take fewer, so that most compute units have a workgroup (2^20
  // responses, 64 workgroups and 256: counting 17 and 7 us, partition in rollout order 11 and 7, shuffled 30 and 19).  Two and a
  // half million, whole call with 153 and 306 workgroups: rollout order 87 and 81 us, shuffled 145 and 160.
  q.per = 16;
  while (q.per > 4 && ceil_div(n_resp, kPoolThreads * q.per) < 144) q.per /= 2;
  const size_t R = static_cast<size_t>(n_resp), blocks = static_cast<size_t>(ceil_div(n_resp, kPoolThreads * q.per));
  q.key = p->key_of_resp;
  q.slot = p->rank_of_resp;
  q.list = p->arrival;
  q.hist = p->hist;
  q.kr = ws.take<int2>(R);
  q.x = ws.take<float>(R);
  q.member = ws.take<uint16_t>(blocks * kPoolThreads * q.per);
  q.sorted = ws.take<int32_t>(blocks);
  q.result = ws.take<float2>(R);
  q.stats = ws.take<float4>(R);
  q.blk = ws.take<int32_t>(blocks * static_cast<size_t>(q.bins));
  q.bin_cnt = ws.take<int32_t>(static_cast<size_t>(q.bins));
  q.bin_base = ws.take<int32_t>(static_cast<size_t>(q.bins) + 1);
  q.cursor = ws.take<int32_t>(static_cast<size_t>(q.bins));
  q.bin_groups = ws.take<int32_t>(static_cast<size_t>(q.bins));
  q.gid_base = ws.take<int32_t>(static_cast<size_t>(q.bins) + 1);
  q.bins_done = ws.take<int32_t>(1 + kPoolMaxBins / kTicketBins);
  q.large = ws.take<int32_t>(static_cast<size_t>(q.bins) + 1);
  return true;
}

}  // namespace

size_t group_advantage_workspace(int32_t n_resp, int32_t n_env, int32_t n_agent, int32_t n_turn, int32_t group_by,
                                 int32_t n_sample) {
  WsAlloc ws(nullptr);
  GaPlan p;
  if (!plan(n_resp, n_env, n_agent, n_turn, group_by, n_sample, ws, &p)) return 0;
  plan_pool(n_resp, ws, &p);
  return ws.bytes();
}

size_t group_advantage_workspace(int32_t n_resp, int32_t n_env, int32_t n_agent, int32_t n_turn) {
  return group_advantage_workspace(n_resp, n_env, n_agent, n_turn, AT_GRPO_GROUP_BY_AGENT_TURN, 1);
}

// what the call can do with at the least (the pool path needs more and is left out then)
size_t group_advantage_least_workspace(int32_t n_resp, int32_t n_env, int32_t n_agent, int32_t n_turn) {
  WsAlloc ws(nullptr);
  GaPlan p;
  if (!plan(n_resp, n_env, n_agent, n_turn, AT_GRPO_GROUP_BY_AGENT_TURN, 1, ws, &p)) return 0;
  return ws.bytes();
}

}  // namespace atg

using namespace atg;

namespace {

// do n elements at a and m elements at b (4 bytes each) have memory in common?
bool overlap(const void* a, int64_t n, const void* b, int64_t m) {
  const uintptr_t x = reinterpret_cast<uintptr_t>(a), y = reinterpret_cast<uintptr_t>(b);
  return a && b && x < y + static_cast<uintptr_t>(m) * 4 && y < x + static_cast<uintptr_t>(n) * 4;
}

int run_group_advantage(int32_t n_resp, int32_t n_env, int32_t n_agent, int32_t n_turn,
                        const int32_t* env_id, const int32_t* agent_id, const int32_t* turn_id,
                        const float* reward, float eps_std, int32_t ddof, int32_t norm, int32_t* group_id,
                        int32_t* n_groups, int32_t* seg_offsets, int32_t* perm, float* adv,
                        float* group_mean, float* group_std, const float* r_team, const float* r_loc,
                        float alpha, float* reward_out, int32_t* best, void* workspace,
                        size_t workspace_bytes, void* hip_stream,
                        int32_t group_by = AT_GRPO_GROUP_BY_AGENT_TURN, const int32_t* sample_id = nullptr,
                        int32_t n_sample = 1) {
  if (!env_id || !agent_id || !turn_id || !group_id || !n_groups || !seg_offsets || !perm || !adv)
    return AT_GRPO_EINVAL;
  if (n_resp <= 0 || n_env <= 0 || n_agent <= 0 || n_turn <= 0) return AT_GRPO_EINVAL;
  if (group_by != AT_GRPO_GROUP_BY_AGENT_TURN && group_by != AT_GRPO_GROUP_BY_TRAJECTORY &&
      group_by != AT_GRPO_GROUP_BY_PARALLEL)
    return AT_GRPO_EINVAL;
  if (group_by == AT_GRPO_GROUP_BY_PARALLEL && (!sample_id || n_sample <= 0)) return AT_GRPO_EINVAL;
  if (ddof != 0 && ddof != 1) return AT_GRPO_EINVAL;
  const int32_t fill = (norm & AT_GRPO_NORM_FILL) != 0;
  norm &= ~AT_GRPO_NORM_FILL;
  if (norm != AT_GRPO_NORM_STD && norm != AT_GRPO_NORM_NONE) return AT_GRPO_EINVAL;
  if (!(eps_std >= 0.f)) return AT_GRPO_EINVAL;
  WsAlloc ws(workspace);
  GaPlan p;
  if (!plan(n_resp, n_env, n_agent, n_turn, group_by, n_sample, ws, &p)) return AT_GRPO_EUNSUPPORTED;
  if (!workspace || (reinterpret_cast<uintptr_t>(workspace) & 255) || workspace_bytes < ws.bytes())
    return AT_GRPO_EWORKSPACE;
  hipStream_t s = static_cast<hipStream_t>(hip_stream);
  ProfScope ps(PROF_GROUP, s);

  const GaMix mix{r_team, r_loc, alpha, r_team ? reward_out : nullptr};
  GaArgs a{n_resp, n_env, n_agent, n_turn, env_id, agent_id, turn_id, reward, group_by, n_sample, sample_id};
  const GaStat st{eps_std, ddof, norm};
  const int64_t g_max = n_resp < p.n_keys ? n_resp : p.n_keys;      // most groups there can be
  const GaOut o{group_id, n_groups, seg_offsets, perm, adv, group_mean, group_std, best, static_cast<int32_t>(g_max), fill};

  if (n_resp <= kRangeMaxResp && p.n_keys <= kRangeMaxKeys) {
    // A workgroup per 256 responses, and enough that each has at most one key per thread.  Every workgroup scans all keys, so
    // large calls take more threads.  Measured on the stream, launch gaps included, 256 / 1024 threads: 64 responses 11 / 12 us,
    // 1024: 12 / 13, 4096: 25 / 14; 65536 responses with a workgroup per 128 / 256 / 512: 49 / 31 / 32 us.
    // Where an output lies on an input (rewards mixed in place), one workgroup's results could reach another that still has
    // inputs to read: the keys then go through a launch of their own, behind which a reward is only read for its own group.
    const auto in_place = [&] {
      for (const void* in : {static_cast<const void*>(env_id), static_cast<const void*>(agent_id), static_cast<const void*>(turn_id),
                             static_cast<const void*>(sample_id), static_cast<const void*>(reward),
                             static_cast<const void*>(r_team), static_cast<const void*>(r_loc)}) {
        if (!in) continue;
        for (const void* out : {static_cast<const void*>(mix.reward_out), static_cast<const void*>(group_id),
                                static_cast<const void*>(perm), static_cast<const void*>(adv)})
          if (overlap(in, n_resp, out, n_resp)) return true;
        for (const void* out : {static_cast<const void*>(group_mean), static_cast<const void*>(group_std),
                                static_cast<const void*>(best), static_cast<const void*>(seg_offsets)})
          if (overlap(in, n_resp, out, g_max + 1)) return true;
        if (overlap(in, n_resp, n_groups, 1)) return true;
      }
      return false;
    };
    const bool direct = n_resp <= kRangeDirect && !in_place();
    const int threads = n_resp <= kRangeFew ? 256 : 1024;
    const int64_t by_resp = ceil_div(n_resp, 256), by_keys = ceil_div(p.n_keys, threads);
    const int64_t blocks = by_resp > by_keys ? by_resp : by_keys;
    const int own = static_cast<int>(ceil_div(p.n_keys, blocks));
    const dim3 grid(static_cast<unsigned>(ceil_div(p.n_keys, own)));
    uint16_t* keys16 = direct ? nullptr : reinterpret_cast<uint16_t*>(p.key_of_resp);
    GaMix given = mix;
    if (!direct) {
      hipLaunchKernelGGL(k_ga_keys, dim3(static_cast<unsigned>(ceil_div(n_resp, 256) + 1)), dim3(256), 0, s, a, mix, keys16);
      ATG_LAUNCH_CHECK();
      if (r_team) a.reward = reward_out;
      given = GaMix{nullptr, nullptr, 0.f, nullptr};
    }
    // Many keys per workgroup are few responses per key.  If the responses lie in a few workgroups' keys all the same (ids from
    // a part of their extents), those workgroups' large groups go to a third launch, which costs the others 2 us: 65536
    // responses in groups of 256, all in one workgroup's keys, took it 1834 us, now 164; 32768 in groups of 64: 318, now 52.
    // Up to kRangeOwn keys a wavefront has at most eight large groups.
    int32_t* left = n_resp > kRangeList && own > kRangeOwn ? p.hist : nullptr;
    if (threads == 256)
      hipLaunchKernelGGL(k_ga_range<256>, grid, dim3(256), 0, s, a, given, st, static_cast<int>(p.n_keys), own, keys16, p.err,
                         p.arrival, left, o);
    else
      hipLaunchKernelGGL(k_ga_range<1024>, grid, dim3(1024), 0, s, a, given, st, static_cast<int>(p.n_keys), own, keys16, p.err,
                         p.arrival, left, o);
    ATG_LAUNCH_CHECK();
    if (left) {
      hipLaunchKernelGGL(k_ga_left, dim3(kLeftBlocks), dim3(256), 0, s, static_cast<int>(grid.x), left, p.arrival, a.reward, st,
                         o);
      ATG_LAUNCH_CHECK();
    }
    return AT_GRPO_OK;
  }
  if (plan_pool(n_resp, ws, &p) && workspace_bytes >= ws.bytes()) {
    const unsigned blocks = static_cast<unsigned>(ceil_div(n_resp, kPoolThreads * p.pool.per));
    const float* rw = r_team ? reward_out : reward;
    hipLaunchKernelGGL(k_gp_init, dim3(1), dim3(kPoolThreads), 0, s, p.pool.bin_cnt, p.pool.bins, p.err);
    ATG_LAUNCH_CHECK();
    hipLaunchKernelGGL(k_gp_count, dim3(blocks), dim3(kPoolThreads), 0, s, a, mix, p.pool, p.err);
    ATG_LAUNCH_CHECK();
    hipLaunchKernelGGL(k_gp_bases, dim3(static_cast<unsigned>(1 + ceil_div(p.pool.bins, kBasesBins))), dim3(kPoolThreads), 0, s,
                       p.pool, p.n_keys);
    ATG_LAUNCH_CHECK();
    // Blocks that are one round of workgroups are partitioned by one launch, whose LDS leaves room for one per compute unit (2^22 in
    // rollout order 19 us; k_gp_partition 18 and the launch in front of it 5); more of them take a second one for those not sorted.
    const bool may_sort = p.pool.per == kSortPer, one_round = blocks <= static_cast<unsigned>(device_cu_count());
    if (may_sort) {
      auto k = one_round ? k_gp_partition_sorted<true> : k_gp_partition_sorted<false>;
      ATG_TRY(allow_big_lds(k, kSortLds));
      hipLaunchKernelGGL(k, dim3(blocks), dim3(kPoolThreads), kSortLds, s, n_resp, rw, p.pool);
      ATG_LAUNCH_CHECK();
    }
    if (!may_sort || !one_round) {
      hipLaunchKernelGGL(k_gp_partition, dim3(blocks), dim3(kPoolThreads), 0, s, n_resp, rw, p.pool, may_sort ? 1 : 0);
      ATG_LAUNCH_CHECK();
    }
    hipLaunchKernelGGL(k_gp_bin, dim3(p.pool.bins), dim3(kBinThreads), 0, s, p.pool, rw, st, p.n_keys, o);
    ATG_LAUNCH_CHECK();
    const int resp_blocks = static_cast<int>(ceil_div(n_resp, 1024));
    hipLaunchKernelGGL(k_gp_out, dim3(static_cast<unsigned>(resp_blocks + p.pool.bins + (fill ? 64 : 0))), dim3(256), 0, s,
                       p.pool, n_resp, resp_blocks, o);
    ATG_LAUNCH_CHECK();
    // both behind k_gp_out, which lists the members of the large bins
    if (may_sort) {
      ATG_TRY(allow_big_lds(k_gp_turn, kTurnLds));
      hipLaunchKernelGGL(k_gp_turn, dim3(std::max(blocks, static_cast<unsigned>(kLargeBlocks * 256 / kPoolThreads))), dim3(kPoolThreads),
                         kTurnLds, s, p.pool, n_resp, static_cast<int>(blocks), rw, st, o);
      ATG_LAUNCH_CHECK();
    } else {
      hipLaunchKernelGGL(k_gp_large, dim3(kLargeBlocks), dim3(256), 0, s, p.pool, rw, st, o);
      ATG_LAUNCH_CHECK();
    }
    return AT_GRPO_OK;
  }
  if (r_team) {
    // the mixed reward is an output; everything below reads it
    hipLaunchKernelGGL(k_ga_mix, dim3(static_cast<unsigned>(ceil_div(n_resp, 256))), dim3(256), 0, s, n_resp,
                       r_team, r_loc, alpha, reward_out);
    ATG_LAUNCH_CHECK();
    a.reward = reward = reward_out;
  }
  const unsigned rb = static_cast<unsigned>(ceil_div(n_resp, 256));
  const unsigned kb = static_cast<unsigned>(p.n_blocks);

  hipLaunchKernelGGL(k_ga_clear2, dim3(static_cast<unsigned>(ceil_div(p.n_keys, 1024) > 4096 ? 4096 : ceil_div(p.n_keys, 1024))),
                     dim3(256), 0, s, p.hist, p.n_keys, p.err, int64_t{64});
  ATG_LAUNCH_CHECK();
  hipLaunchKernelGGL(k_ga_hist, dim3(rb), dim3(256), 0, s, a, p.err, p.hist, p.key_of_resp, p.rank_of_resp);
  ATG_LAUNCH_CHECK();
  hipLaunchKernelGGL(k_ga_scan_partial, dim3(kb), dim3(256), 0, s, p.hist, p.n_keys, p.bsum_p, p.bsum_c);
  ATG_LAUNCH_CHECK();
  hipLaunchKernelGGL(k_ga_scan_top, dim3(1), dim3(256), 0, s, p.n_blocks, p.bsum_p, p.bsum_c, n_groups, seg_offsets);
  ATG_LAUNCH_CHECK();
  hipLaunchKernelGGL(k_ga_scan_apply, dim3(kb), dim3(256), 0, s, p.hist, p.n_keys, p.bsum_p, p.bsum_c,
                     p.gid_of_key, seg_offsets);
  ATG_LAUNCH_CHECK();
  hipLaunchKernelGGL(k_ga_scatter, dim3(rb), dim3(256), 0, s, n_resp, p.key_of_resp, p.rank_of_resp,
                     p.gid_of_key, seg_offsets, group_id, p.arrival, adv);
  ATG_LAUNCH_CHECK();
  // at most min(R, keys) groups exist; both finishing roles stride over them
  const int fs = static_cast<int>(ceil_div(g_max, 256) > 4096 ? 4096 : ceil_div(g_max, 256));
  const int fl = static_cast<int>(ceil_div(g_max, 4) > 4096 ? 4096 : ceil_div(g_max, 4));
  hipLaunchKernelGGL(k_ga_finish, dim3(static_cast<unsigned>(fs + fl + (fill ? 64 : 0))), dim3(256), 0, s, fs, fl, n_resp,
                     p.arrival, reward, st, o);
  ATG_LAUNCH_CHECK();
  return AT_GRPO_OK;
}

}  // namespace

extern "C" int at_grpo_group_advantage(int32_t n_resp, int32_t n_env, int32_t n_agent, int32_t n_turn,
                                       const int32_t* env_id, const int32_t* agent_id,
                                       const int32_t* turn_id, const float* reward, float eps_std,
                                       int32_t ddof, int32_t norm, int32_t* group_id, int32_t* n_groups,
                                       int32_t* seg_offsets, int32_t* perm, float* adv, float* group_mean,
                                       float* group_std, void* workspace, size_t workspace_bytes,
                                       void* hip_stream) {
  if (!reward) return AT_GRPO_EINVAL;
  return run_group_advantage(n_resp, n_env, n_agent, n_turn, env_id, agent_id, turn_id, reward, eps_std, ddof,
                             norm, group_id, n_groups, seg_offsets, perm, adv, group_mean, group_std, nullptr,
                             nullptr, 0.f, nullptr, nullptr, workspace, workspace_bytes, hip_stream);
}

extern "C" int at_grpo_group_advantage_mixed(int32_t n_resp, int32_t n_env, int32_t n_agent, int32_t n_turn,
                                             const int32_t* env_id, const int32_t* agent_id,
                                             const int32_t* turn_id, const float* r_team,
                                             const float* r_loc, float alpha, float eps_std, int32_t ddof,
                                             int32_t norm, float* reward, int32_t* group_id,
                                             int32_t* n_groups, int32_t* seg_offsets, int32_t* perm,
                                             float* adv, float* group_mean, float* group_std,
                                             int32_t* best, void* workspace, size_t workspace_bytes,
                                             void* hip_stream) {
  if (!r_team || !r_loc || !reward) return AT_GRPO_EINVAL;
  if (!(fabsf(alpha) <= 3.402823466e38f)) return AT_GRPO_EINVAL;
  return run_group_advantage(n_resp, n_env, n_agent, n_turn, env_id, agent_id, turn_id, reward, eps_std, ddof,
                             norm, group_id, n_groups, seg_offsets, perm, adv, group_mean, group_std, r_team,
                             r_loc, alpha, reward, best, workspace, workspace_bytes, hip_stream);
}


extern "C" int at_grpo_group_advantage_keyed(int32_t group_by, int32_t n_resp, int32_t n_env, int32_t n_agent,
                                             int32_t n_turn, int32_t n_sample, const int32_t* env_id,
                                             const int32_t* agent_id, const int32_t* turn_id,
                                             const int32_t* sample_id, const float* reward, float eps_std,
                                             int32_t ddof, int32_t norm, int32_t* group_id, int32_t* n_groups,
                                             int32_t* seg_offsets, int32_t* perm, float* adv, float* group_mean,
                                             float* group_std, void* workspace, size_t workspace_bytes,
                                             void* hip_stream) {
  if (!reward) return AT_GRPO_EINVAL;
  return run_group_advantage(n_resp, n_env, n_agent, n_turn, env_id, agent_id, turn_id, reward, eps_std, ddof,
                             norm, group_id, n_groups, seg_offsets, perm, adv, group_mean, group_std, nullptr,
                             nullptr, 0.f, nullptr, nullptr, workspace, workspace_bytes, hip_stream, group_by,
                             sample_id, n_sample);
}

extern "C" size_t at_grpo_group_advantage_keyed_workspace_bytes(int32_t group_by, int32_t n_resp, int32_t n_env,
                                                                int32_t n_agent, int32_t n_turn, int32_t n_sample) {
  if (group_by != AT_GRPO_GROUP_BY_AGENT_TURN && group_by != AT_GRPO_GROUP_BY_TRAJECTORY &&
      group_by != AT_GRPO_GROUP_BY_PARALLEL)
    return 0;
  return group_advantage_workspace(n_resp, n_env, n_agent, n_turn, group_by, n_sample);
}

// ------------------------------------------------------------------------------------------------
// The same call for callers that cannot allocate or hand over device scratch: the workspace is a
// fixed array in device memory that belongs to the library.  Every GPU the library runs on holds
// its own copy of the array (at its own address) until the process ends.
// ------------------------------------------------------------------------------------------------
namespace {

constexpr size_t kStaticScratchBytes = size_t{2} << 20;
static __device__ __align__(256) unsigned char scratch[kStaticScratchBytes];

constexpr int kMaxDevices = 64;
std::mutex g_scratch_mutex;
void* g_scratch_ptr[kMaxDevices] = {nullptr};

// Device address of `scratch` on the current device (looked up once per device; the array's name
// is only a host-side handle and must never be passed to a kernel or a memory call).
int static_scratch(void** out) {
  int dev = -1;
  ATG_HIP_TRY(hipGetDevice(&dev));
  if (dev < 0 || dev >= kMaxDevices) return AT_GRPO_EUNSUPPORTED;
  std::lock_guard<std::mutex> lock(g_scratch_mutex);
  if (!g_scratch_ptr[dev]) {
    void* p = nullptr;
    ATG_HIP_TRY(hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)));
    if (!p || (reinterpret_cast<uintptr_t>(p) & 255)) return AT_GRPO_EHIP;
    g_scratch_ptr[dev] = p;
  }
  *out = g_scratch_ptr[dev];
  return AT_GRPO_OK;
}

__global__ void k_ga_copy_error(const int32_t* __restrict__ err, int32_t* __restrict__ out) { *out = *err; }

}  // namespace

extern "C" size_t at_grpo_static_scratch_bytes(void) { return kStaticScratchBytes; }

extern "C" int at_grpo_group_advantage_static(int32_t n_resp, int32_t n_env, int32_t n_agent, int32_t n_turn,
                                              const int32_t* env_id, const int32_t* agent_id,
                                              const int32_t* turn_id, const float* reward, float eps_std,
                                              int32_t ddof, int32_t norm, int32_t* group_id,
                                              int32_t* n_groups, int32_t* seg_offsets, int32_t* perm,
                                              float* adv, float* group_mean, float* group_std,
                                              int32_t* data_error, void* hip_stream) {
  if (!reward) return AT_GRPO_EINVAL;
  if (n_resp <= 0 || n_env <= 0 || n_agent <= 0 || n_turn <= 0) return AT_GRPO_EINVAL;
  const size_t need = group_advantage_least_workspace(n_resp, n_env, n_agent, n_turn);
  if (need == 0 || need > kStaticScratchBytes) return AT_GRPO_ESCRATCH;
  void* ws = nullptr;
  ATG_TRY(static_scratch(&ws));
  ATG_TRY(run_group_advantage(n_resp, n_env, n_agent, n_turn, env_id, agent_id, turn_id, reward, eps_std, ddof,
                              norm, group_id, n_groups, seg_offsets, perm, adv, group_mean, group_std, nullptr,
                              nullptr, 0.f, nullptr, nullptr, ws, kStaticScratchBytes, hip_stream));
  if (data_error) {
    hipLaunchKernelGGL(k_ga_copy_error, dim3(1), dim3(1), 0, static_cast<hipStream_t>(hip_stream),
                       static_cast<const int32_t*>(ws), data_error);
    ATG_LAUNCH_CHECK();
  }
  return AT_GRPO_OK;
}

// fcp_plan_groups: the FCP scheduler's two stages on the host (paper Sec. 4.4): memory-aware packing of the
// micro-batch's sequences into atomic groups (best-fit decreasing) and the 2D dynamic programme that gives
// every group its CP degree so that the slowest group is as fast as possible (Eq. 2, Eq. 11, Alg. 1), with the
// group time model of Eq. 8-10.  Host only; nothing here touches the GPU.
//
// Readings where the paper is silent or at odds with itself (they are the header's contract):
//   * capacity is given in tokens per rank, (E - M_ms) / M_token: Cond. 3 with Eq. 7 is a ratio of token counts;
//   * the compute terms of Eq. 8 are divided by the degree (Eq. 11 needs T(G, d); CP splits a sequence evenly,
//     Sec. 4.3); a degree-1 group has no ring and no exchange; all CP traffic is the attention's KV ring, so
//     Eq. 10 hides min(attention compute, exchange);
//   * every table entry but DP[0][0] starts at +inf; Cond. 6 is "at most N ranks", so the answer is taken at the
//     smallest rank count that attains the least makespan (with an exchange term more ranks can be slower).
#include <algorithm>
#include <array>
#include <cmath>
#include <limits>
#include <vector>

#include "fcp.h"
#include "fcp_internal.h"

namespace {

struct Group {
  int64_t load = 0;               // tokens
  int32_t d_min = 0;
  // sums that T(G, d) needs, accumulated in increasing sequence index
  double quad = 0.0, lin = 0.0, tokens = 0.0;
};

// Eq. 8-10 for one group at degrees lo .. hi
inline void group_times(const Group& g, int lo, int hi, const fcp_cost_model& cm, double* __restrict__ t) {
  const double quad = g.quad, lin = g.lin, beta1 = cm.beta1, t_ring = cm.alpha3_over_v * g.tokens + cm.beta2;
  for (int d = lo; d <= hi; ++d) {
    const double t_cpa = quad / d, t_cm = d == 1 ? 0.0 : t_ring;
    t[d] = t_cpa + lin / d + beta1 + t_cm - std::min(t_cpa, t_cm);
  }
}

// The two inner loops of a plan are worked in four lanes where the processor has them.
#if defined(__x86_64__) && !defined(__HIP_DEVICE_COMPILE__)
#define FCP_WIDE_LANES __attribute__((target_clones("avx2", "default")))
#else
#define FCP_WIDE_LANES
#endif

// The first of the least rooms that hold s tokens, or -1.
FCP_WIDE_LANES int best_fit(const int64_t* __restrict__ room, int n, int64_t s) {
  int64_t least = INT64_MAX;
  for (int g = 0; g < n; ++g) {
    const int64_t r = room[g] < s ? INT64_MAX : room[g];
    least = r < least ? r : least;
  }
  if (least == INT64_MAX) return -1;               // (a room is less than that: a sequence has been taken off it)
  int g = 0;
  while (room[g] != least) ++g;
  return g;
}

// One degree of a group against adjacent rank counts: the least makespan so far and its degree.
FCP_WIDE_LANES void relax(const double* __restrict__ prev, double t, double d, double* __restrict__ best, double* __restrict__ degree, int n) {
  for (int x = 0; x < n; ++x) {
    const double cost = prev[x] < t ? t : prev[x];
    const bool less = cost < best[x];
    best[x] = less ? cost : best[x];
    degree[x] = less ? d : degree[x];
  }
}

// Sequence indices by decreasing length, equal lengths in input order: a byte-wise radix sort, least byte first, without the
// bytes that all lengths share.
std::vector<int32_t> longest_first(const int32_t* len, int32_t n) {
  std::vector<int32_t> order(n), other(n);
  std::array<std::array<int32_t, 256>, 4> count{};
  for (int32_t k = 0; k < n; ++k) {
    order[k] = k;
    for (int b = 0; b < 4; ++b) ++count[b][~((uint32_t)len[k] >> (8 * b)) & 255];
  }
  for (int b = 0; b < 4; ++b) {
    auto& at = count[b];
    if (n == 0 || at[~((uint32_t)len[0] >> (8 * b)) & 255] == n) continue;
    int32_t sum = 0;
    for (int32_t& c : at) { const int32_t x = c; c = sum; sum += x; }
    for (int32_t k : order) other[at[~((uint32_t)len[k] >> (8 * b)) & 255]++] = k;
    std::swap(order, other);
  }
  return order;
}

}  // namespace

extern "C" int fcp_plan_groups(const int32_t* seq_lens, const float* eta, int32_t n_seqs, int32_t n_ranks,
                               int64_t tokens_per_rank, const fcp_cost_model* cm, int32_t* group_of_seq,
                               int32_t* n_groups, int32_t* group_d_min, int32_t* group_degree,
                               int32_t* group_base_rank, double* makespan) {
  using fcp::fail;
  fcp::clear_error();
  if (!seq_lens || !cm || !group_of_seq || !n_groups || !group_d_min || !group_degree || !group_base_rank || !makespan)
    return fail(FCP_ERR_INVALID_ARG, "fcp_plan_groups: null argument");
  if (n_seqs < 0 || n_ranks < 1 || tokens_per_rank < 1)
    return fail(FCP_ERR_INVALID_ARG, "fcp_plan_groups: n_seqs < 0, n_ranks < 1 or tokens_per_rank < 1");
  if (n_ranks > (1 << 16)) return fail(FCP_ERR_UNSUPPORTED, "fcp_plan_groups: more than 65536 ranks");
  for (int32_t k = 0; k < n_seqs; ++k) {
    if (seq_lens[k] < 1) return fail(FCP_ERR_INVALID_ARG, "fcp_plan_groups: seq_lens[%d] = %d < 1", k, seq_lens[k]);
    if (eta && !(eta[k] >= 0.f)) return fail(FCP_ERR_INVALID_ARG, "fcp_plan_groups: eta[%d] negative or NaN", k);
  }
  if (!(cm->alpha1 >= 0.0) || !(cm->alpha2 >= 0.0) || !(cm->beta1 >= 0.0) || !(cm->alpha3_over_v >= 0.0) || !(cm->beta2 >= 0.0))
    return fail(FCP_ERR_INVALID_ARG, "fcp_plan_groups: cost coefficients must be non-negative numbers");

  // ---- Stage 1: best-fit decreasing.  Longest first (equal lengths in input order); a sequence goes to the open
  // group with the least headroom that still holds it (the group opened first among equals), else opens a group
  // of d_min = ceil(len / capacity) ranks.
  // (The rooms of the open groups lie side by side, so that the search is one pass over a few cache lines.)
  const std::vector<int32_t> order = longest_first(seq_lens, n_seqs);
  std::vector<Group> groups;
  std::vector<int64_t> room_of;
  for (int32_t k : order) {
    const int64_t s = seq_lens[k];
    int best = best_fit(room_of.data(), (int)room_of.size(), s);
    if (best < 0) {
      Group g;
      const int64_t dm = (s + tokens_per_rank - 1) / tokens_per_rank;
      if (dm > n_ranks) {
        *n_groups = 0;
        return fail(FCP_ERR_CAPACITY, "fcp_plan_groups: sequence %d (%d tokens) needs %lld ranks of %lld tokens, %d available",
                    k, seq_lens[k], (long long)dm, (long long)tokens_per_rank, n_ranks);
      }
      g.d_min = (int32_t)dm;
      groups.push_back(g);
      room_of.push_back(dm * tokens_per_rank);
      best = (int)groups.size() - 1;
    }
    room_of[best] -= s;
    group_of_seq[k] = best;
  }
  const int kp = (int)groups.size();
  *n_groups = kp;
  // cost sums in increasing sequence index
  for (int32_t k = 0; k < n_seqs; ++k) {
    Group& g = groups[group_of_seq[k]];
    g.load += seq_lens[k];
    const double s = (double)seq_lens[k];
    g.quad += cm->alpha1 * (1.0 + (eta ? (double)eta[k] : 0.0)) * s * s;
    g.lin += cm->alpha2 * s;
  }
  int64_t need = 0;
  for (int g = 0; g < kp; ++g) {
    groups[g].tokens = (double)groups[g].load;
    group_d_min[g] = groups[g].d_min;
    need += groups[g].d_min;
  }
  if (need > n_ranks)
    return fail(FCP_ERR_CAPACITY, "fcp_plan_groups: the groups need %lld ranks at their minimum degrees, %d available",
                (long long)need, n_ranks);
  if (kp == 0) {
    *makespan = 0.0;
    return FCP_OK;
  }

  // ---- Stage 2: DP[i][j] = least makespan of the first i groups on exactly j ranks (Eq. 11)
  const double inf = std::numeric_limits<double>::infinity();
  const int N = n_ranks;
  std::vector<double> prev(N + 1, inf), cur(N + 1, inf);
  std::vector<int32_t> path((size_t)kp * (N + 1), 0);
  prev[0] = 0.0;
  int64_t before = 0;                       // sum of d_min of the groups before group i
  std::vector<double> t(N + 1), pick(N + 1);   // (degrees as doubles: lanes of one width)
  for (int i = 0; i < kp; ++i) {
    const int dm = groups[i].d_min;
    const int d_hi = N - (int)(need - dm);  // no count leaves more than this for group i
    group_times(groups[i], dm, d_hi, *cm, t.data());
    // Rank counts from before + dm (less is infeasible) to what leaves the later groups their minimum.  The degree is the
    // outer loop, so that the inner one runs over adjacent entries without a dependence and is vectorised; for each count the
    // degrees are still tried in increasing order and the first of equals stays.
    const int j_lo = (int)before + dm, j_hi = N - (int)(need - before - dm);
    std::fill(cur.begin(), cur.end(), inf);
    std::fill(pick.begin(), pick.end(), 0.0);
    for (int d = dm; d <= j_hi - (int)before; ++d) {
      relax(prev.data() + before, t[d], d, cur.data() + before + d, pick.data() + before + d, j_hi - (int)before - d + 1);
    }
    for (int j = j_lo; j <= j_hi; ++j) path[(size_t)i * (N + 1) + j] = (int32_t)pick[j];
    before += dm;
    std::swap(prev, cur);
  }
  int best_j = 0;
  for (int j = 1; j <= N; ++j)
    if (prev[j] < prev[best_j]) best_j = j;
  if (!(prev[best_j] < inf)) return fail(FCP_ERR_CAPACITY, "fcp_plan_groups: no feasible allocation found");
  *makespan = prev[best_j];
  int j = best_j;
  for (int i = kp - 1; i >= 0; --i) {
    group_degree[i] = path[(size_t)i * (N + 1) + j];
    j -= group_degree[i];
  }
  int32_t base = 0;
  for (int i = 0; i < kp; ++i) {
    group_base_rank[i] = base;
    base += group_degree[i];
  }
  return FCP_OK;
}

// The paper's atomic groups run as one CP group (Sec. 4.4): every sequence of a group takes the group's degree
// and base rank.
extern "C" int fcp_group_shard_args(const int32_t* group_of_seq, int32_t n_seqs, const int32_t* group_degree,
                                    const int32_t* group_base_rank, int32_t n_groups, int32_t* cp_degree,
                                    int32_t* base_rank) {
  using fcp::fail;
  fcp::clear_error();
  if (n_seqs < 0 || n_groups < 0 || (n_seqs > 0 && (!group_of_seq || !cp_degree || !base_rank)) ||
      (n_groups > 0 && (!group_degree || !group_base_rank)))
    return fail(FCP_ERR_INVALID_ARG, "fcp_group_shard_args: null argument or negative count");
  for (int32_t g = 0; g < n_groups; ++g)
    if (group_degree[g] < 1 || group_base_rank[g] < 0)
      return fail(FCP_ERR_INVALID_ARG, "fcp_group_shard_args: group %d has degree %d, base rank %d", g, group_degree[g],
                  group_base_rank[g]);
  for (int32_t k = 0; k < n_seqs; ++k) {
    const int32_t g = group_of_seq[k];
    if (g < 0 || g >= n_groups)
      return fail(FCP_ERR_INVALID_ARG, "fcp_group_shard_args: group_of_seq[%d] = %d out of range", k, g);
    cp_degree[k] = group_degree[g];
    base_rank[k] = group_base_rank[g];
  }
  return FCP_OK;
}

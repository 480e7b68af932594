// Host-side parts of libfcp: error reporting and the shard plan.
#include <algorithm>
#include <cstdarg>
#include <cstdio>
#include <vector>

#include "fcp_internal.h"

namespace fcp {

static thread_local char g_err[512] = "";

int fail(int code, const char* fmt, ...) {
  va_list ap;
  va_start(ap, fmt);
  vsnprintf(g_err, sizeof(g_err), fmt, ap);
  va_end(ap);
  return code;
}

void clear_error() { g_err[0] = 0; }

}  // namespace fcp

extern "C" const char* fcp_last_error(void) { return fcp::g_err; }

namespace {

// Full-attention spans of every sequence as (start, end) pairs in increasing order, and the mask they imply in
// the form the kernels use: a row at position i sees the keys 0 .. limit(i); a key at position j is seen by the
// rows from(j) .. L-1.  Outside a span both are the position itself (causal), inside a span its last and its
// first position.
struct SpanIndex {
  std::vector<std::vector<std::pair<int32_t, int32_t>>> by_seq;
  const std::pair<int32_t, int32_t>* find(int32_t seq, int32_t pos) const {
    const auto& v = by_seq[seq];
    auto it = std::upper_bound(v.begin(), v.end(), pos,
                               [](int32_t x, const std::pair<int32_t, int32_t>& sp) { return x < sp.first; });
    if (it == v.begin()) return nullptr;
    --it;
    return pos < it->second ? &*it : nullptr;
  }
  int32_t limit(int32_t seq, int32_t pos) const { auto sp = find(seq, pos); return sp ? sp->second - 1 : pos; }
  int32_t from(int32_t seq, int32_t pos) const { auto sp = find(seq, pos); return sp ? sp->first : pos; }
};

int build_span_index(const char* who, const int32_t* seq_lens, int32_t n_seqs, const fcp_span* spans, int32_t n_spans,
                     SpanIndex* out) {
  using fcp::fail;
  if (n_spans < 0 || (n_spans > 0 && !spans)) return fail(FCP_ERR_INVALID_ARG, "%s: bad span list", who);
  out->by_seq.assign((size_t)n_seqs, {});
  for (int32_t i = 0; i < n_spans; ++i) {
    const fcp_span& sp = spans[i];
    if (sp.seq < 0 || sp.seq >= n_seqs) return fail(FCP_ERR_INVALID_ARG, "%s: spans[%d].seq = %d out of range", who, i, sp.seq);
    if (sp.start < 0 || sp.len < 1 || (int64_t)sp.start + sp.len > (int64_t)seq_lens[sp.seq])
      return fail(FCP_ERR_INVALID_ARG, "%s: spans[%d] = [%d, +%d) leaves sequence %d of %d tokens", who, i, sp.start,
                  sp.len, sp.seq, seq_lens[sp.seq]);
    if (i > 0 && (spans[i - 1].seq > sp.seq || (spans[i - 1].seq == sp.seq && spans[i - 1].start + spans[i - 1].len > sp.start)))
      return fail(FCP_ERR_INVALID_ARG, "%s: spans must be sorted by (seq, start) and must not overlap (entry %d)", who, i);
    out->by_seq[sp.seq].emplace_back(sp.start, sp.start + sp.len);
  }
  return FCP_OK;
}

}  // namespace

// Zigzag shard plan.  The paper fixes only an even split of every sequence over the d ranks of its group (Sec. 4.3)
// and that d may be any positive integer (Sec. 4.2); the 2d-chunk zigzag with the remainder spread over
// the first chunks is the load-balanced form of that split for a causal mask.  With full-attention
// spans (Sec. 4.3, time estimation) the chunks stay the same and a query chunk additionally gets the
// later key chunks that a span reaching over the chunk border makes visible.
static int shard_plan(const char* who, const int32_t* seq_lens, const int32_t* cp_degree,
                      const int32_t* base_rank, int32_t n_seqs, const fcp_span* spans, int32_t n_spans,
                      fcp_chunk_desc* chunks, int64_t chunk_cap, int64_t* n_chunks, fcp_work_desc* work,
                      int64_t work_cap, int64_t* n_work) {
  using fcp::fail;
  fcp::clear_error();
  if (!seq_lens || !cp_degree || !n_chunks || !n_work || n_seqs < 0)
    return fail(FCP_ERR_INVALID_ARG, "%s: null argument or negative n_seqs", who);
  int64_t total = 0;
  for (int32_t s = 0; s < n_seqs; ++s) {
    if (seq_lens[s] < 1) return fail(FCP_ERR_INVALID_ARG, "%s: seq_lens[%d] = %d < 1", who, s, seq_lens[s]);
    if (cp_degree[s] < 1 || cp_degree[s] > (1 << 20))
      return fail(FCP_ERR_INVALID_ARG, "%s: cp_degree[%d] = %d out of range", who, s, cp_degree[s]);
    if (base_rank && base_rank[s] < 0) return fail(FCP_ERR_INVALID_ARG, "%s: base_rank[%d] < 0", who, s);
    total += seq_lens[s];
  }
  if (total > INT32_MAX) return fail(FCP_ERR_UNSUPPORTED, "%s: more than 2^31-1 tokens", who);
  SpanIndex mask;
  if (n_spans != 0)
    if (int rc = build_span_index(who, seq_lens, n_seqs, spans, n_spans, &mask)) return rc;

  // Nothing below is sorted and no table is kept: chunk c of a sequence of L tokens at degree d starts at c q + min(c, r) (q, r: quotient and
  // remainder of L / 2d), and walking the sequences in order visits the entries of every (rank) and (rank, step) in the order
  // they are listed in, so that each entry can be written to its place once the entries per (rank) and (rank, step) have been
  // counted.  (Building the two tables and sorting them took 86 % of the time of a plan of 512 sequences on 64 ranks.)
  struct Cut {
    int32_t n, quot, rem, d, base;                   // chunks of the sequence; degree, first rank
    int64_t r;                                       // its dense number (below)
    int32_t start(int32_t c) const { return c * quot + std::min(c, rem); }
    int32_t len(int32_t c) const { return quot + (c < rem ? 1 : 0); }
    int32_t filled() const { return quot > 0 ? n : rem; }       // chunks with tokens come first
  };
  // chunks that query chunk c of sequence s sees: those with a smaller number
  auto n_seen = [&](int32_t s, const Cut& cut, int32_t c) -> int32_t {
    if (n_spans == 0 || c >= cut.filled()) return c < cut.filled() ? c + 1 : 0;
    const int32_t last_seen = mask.limit(s, cut.start(c) + cut.len(c) - 1);   // by the chunk's last row, hence by any
    int32_t v = c + 1;
    while (v < cut.filled() && cut.start(v) <= last_seen) ++v;
    return v;
  };

  // Only the counts: a query chunk has an item for every owner whose first chunk it sees, min(d, chunks seen) of them.  (The first of a caller's two calls; through
  // the counters per rank and step below it took 7.6 us for 512 sequences on 64 ranks, now 3.2 with the call itself.)
  if (!chunks && !work) {
    *n_chunks = *n_work = 0;
    for (int32_t s = 0; s < n_seqs; ++s) {
      const int32_t d = cp_degree[s], n = d == 1 ? 1 : 2 * d;
      *n_chunks += n;
      if (n_spans == 0 && seq_lens[s] >= n) {        // no chunk is empty, and chunk c sees c + 1
        *n_work += d == 1 ? 1 : (int64_t)d * (d + 1) / 2 + (int64_t)d * d;
      } else {
        const int32_t quot = seq_lens[s] / n;
        const Cut c = {n, quot, seq_lens[s] - quot * n, d, 0, 0};
        for (int32_t i = 0; i < n; ++i) *n_work += std::min(d, n_seen(s, c, i));
      }
    }
    return FCP_OK;
  }

  // Ranks as dense numbers: the ranks themselves from the least one on, or, where the base ranks lie far apart, their places
  // among the ranks in use.
  std::vector<Cut> cuts(n_seqs);
  int64_t nc = 0, r_lo = INT64_MAX, r_hi = 0;
  for (int32_t s = 0; s < n_seqs; ++s) {
    const int32_t d = cp_degree[s], n = d == 1 ? 1 : 2 * d, base = base_rank ? base_rank[s] : 0;
    const int32_t quot = seq_lens[s] / n;
    cuts[s] = {n, quot, seq_lens[s] - quot * n, d, base, base};
    nc += n;
    r_lo = std::min<int64_t>(r_lo, base);
    r_hi = std::max<int64_t>(r_hi, (int64_t)base + d);
  }
  int64_t n_dense = n_seqs == 0 ? 0 : r_hi - r_lo;
  if (n_dense > 4 * nc + 1024) {
    std::vector<int64_t> in_use;
    for (const Cut& c : cuts)
      for (int32_t i = 0; i < c.d; ++i) in_use.push_back((int64_t)c.base + i);
    std::sort(in_use.begin(), in_use.end());
    in_use.erase(std::unique(in_use.begin(), in_use.end()), in_use.end());
    for (Cut& c : cuts) c.r = std::lower_bound(in_use.begin(), in_use.end(), (int64_t)c.base) - in_use.begin();
    n_dense = (int64_t)in_use.size();
  } else {
    for (Cut& c : cuts) c.r -= r_lo;
  }

  // Entries per rank, and the first place of every rank's steps among the (rank, step) counters.  (An owner of empty
  // chunks has no items, nor has any after it.)
  std::vector<int64_t> chunk_at(n_dense + 1, 0), step_at(n_dense + 1, 0);
  for (const Cut& c : cuts)
    for (int32_t i = 0; i < c.d; ++i) {
      chunk_at[c.r + i + 1] += c.d == 1 ? 1 : 2;
      if (i < c.filled()) step_at[c.r + i + 1] = std::max<int64_t>(step_at[c.r + i + 1], c.d);
    }
  for (int64_t r = 0; r < n_dense; ++r) { chunk_at[r + 1] += chunk_at[r]; step_at[r + 1] += step_at[r]; }
  // Items per (rank, step).  The step's keys belong to owner j; chunk j is its first one in memory, so a query chunk that sees
  // j or more chunks has an item.
  std::vector<int64_t> work_at(step_at[n_dense] + 1, 0);
  for (int32_t s = 0; s < n_seqs; ++s) {
    const Cut& c = cuts[s];
    for (int32_t i = 0; i < std::min(c.d, c.filled()); ++i) {
      const int32_t lo = n_seen(s, c, i), hi = c.d == 1 ? 0 : n_seen(s, c, 2 * c.d - 1 - i);
      int64_t* const at = work_at.data() + step_at[c.r + i] + 1;
      for (int32_t step = 0, j = i; step < c.d; ++step, j = j == 0 ? c.d - 1 : j - 1) at[step] += (j < lo) + (j < hi);
    }
  }
  for (size_t i = 1; i < work_at.size(); ++i) work_at[i] += work_at[i - 1];

  *n_chunks = nc;
  *n_work = work_at.back();
  if ((chunks && chunk_cap < *n_chunks) || (work && work_cap < *n_work))
    return fail(FCP_ERR_CAPACITY, "%s: need %lld chunk and %lld work entries", who,
                (long long)*n_chunks, (long long)*n_work);

  // Rank-local packed offsets: per rank, sequences in input order, early chunk before late.
  std::vector<int32_t> used(n_dense, 0);             // rows of the rank so far
  for (int32_t s = 0; s < n_seqs; ++s) {
    const Cut& cut = cuts[s];
    const int32_t d = cut.d;
    for (int32_t i = 0; i < d; ++i) {
      const int32_t ca = i, cb = 2 * d - 1 - i;      // the owner's chunks (the second one: d > 1)
      const int32_t off = used[cut.r + i], len_a = cut.len(ca), len_b = d == 1 ? 0 : cut.len(cb);
      used[cut.r + i] = off + len_a + len_b;
      if (chunks) {
        chunks[chunk_at[cut.r + i]++] = {s, cut.base + i, ca, cut.start(ca), len_a, off};
        if (d > 1) chunks[chunk_at[cut.r + i]++] = {s, cut.base + i, cb, cut.start(cb), len_b, off + len_a};
      }
      if (!work || i >= cut.filled()) continue;
      const int32_t lo = n_seen(s, cut, ca), hi = d == 1 ? 0 : n_seen(s, cut, cb);
      int64_t* const at = work_at.data() + step_at[cut.r + i];
      for (int32_t step = 0, j = i; step < d; ++step, j = j == 0 ? d - 1 : j - 1) {
        const int32_t j2 = 2 * d - 1 - j;
        fcp_work_desc w = {s, cut.base + i, step, off, cut.start(ca), len_a, 1, {cut.start(j), 0}, {cut.len(j), 0}};
        const int32_t k1 = cut.start(j2), n1 = cut.len(j2);
        if (j < lo) {
          if (d > 1 && j2 < lo) { w.n_seg = 2; w.k_seq_start[1] = k1; w.k_len[1] = n1; }
          work[at[step]++] = w;
        }
        if (j < hi) {
          const bool two = j2 < hi;
          w.q_local_off = off + len_a; w.q_seq_start = cut.start(cb); w.q_len = len_b;
          w.n_seg = two ? 2 : 1; w.k_seq_start[1] = two ? k1 : 0; w.k_len[1] = two ? n1 : 0;
          work[at[step]++] = w;
        }
      }
    }
  }
  return FCP_OK;
}

extern "C" int fcp_shard_plan(const int32_t* seq_lens, const int32_t* cp_degree,
                              const int32_t* base_rank, int32_t n_seqs, fcp_chunk_desc* chunks,
                              int64_t chunk_cap, int64_t* n_chunks, fcp_work_desc* work,
                              int64_t work_cap, int64_t* n_work) {
  return shard_plan("fcp_shard_plan", seq_lens, cp_degree, base_rank, n_seqs, nullptr, 0, chunks, chunk_cap, n_chunks,
                    work, work_cap, n_work);
}

extern "C" int fcp_shard_plan_mixed(const int32_t* seq_lens, const int32_t* cp_degree,
                                    const int32_t* base_rank, int32_t n_seqs, const fcp_span* spans,
                                    int32_t n_spans, fcp_chunk_desc* chunks, int64_t chunk_cap,
                                    int64_t* n_chunks, fcp_work_desc* work, int64_t work_cap, int64_t* n_work) {
  return shard_plan("fcp_shard_plan_mixed", seq_lens, cp_degree, base_rank, n_seqs, spans, n_spans, chunks, chunk_cap,
                    n_chunks, work, work_cap, n_work);
}

extern "C" int fcp_mask_tables(const int32_t* seq_lens, int32_t n_seqs, const fcp_span* spans, int32_t n_spans,
                               const fcp_chunk_desc* chunks, int64_t n_chunks, int32_t rank, int32_t* q_limit,
                               int64_t q_limit_cap, int64_t* n_q, int32_t* k_from, float* eta) {
  using fcp::fail;
  fcp::clear_error();
  const char* who = "fcp_mask_tables";
  if (!seq_lens || n_seqs < 0 || n_chunks < 0 || (n_chunks > 0 && !chunks))
    return fail(FCP_ERR_INVALID_ARG, "%s: null argument or negative count", who);
  for (int32_t s = 0; s < n_seqs; ++s)
    if (seq_lens[s] < 1) return fail(FCP_ERR_INVALID_ARG, "%s: seq_lens[%d] = %d < 1", who, s, seq_lens[s]);
  SpanIndex mask;
  if (int rc = build_span_index(who, seq_lens, n_seqs, spans, n_spans, &mask)) return rc;
  int64_t rows = 0;
  for (int64_t i = 0; i < n_chunks; ++i) {
    const fcp_chunk_desc& c = chunks[i];
    if (c.rank != rank) continue;
    if (c.seq < 0 || c.seq >= n_seqs || c.seq_start < 0 || c.len < 0 || c.local_off < 0 ||
        (int64_t)c.seq_start + c.len > (int64_t)seq_lens[c.seq])
      return fail(FCP_ERR_INVALID_ARG, "%s: chunks[%lld] does not fit its sequence", who, (long long)i);
    rows = std::max<int64_t>(rows, (int64_t)c.local_off + c.len);
  }
  if (n_q) *n_q = rows;
  if (q_limit) {
    if (q_limit_cap < rows) return fail(FCP_ERR_CAPACITY, "%s: q_limit needs %lld entries", who, (long long)rows);
    for (int64_t i = 0; i < n_chunks; ++i) {
      const fcp_chunk_desc& c = chunks[i];
      if (c.rank != rank) continue;
      for (int32_t r = 0; r < c.len; ++r) q_limit[c.local_off + r] = mask.limit(c.seq, c.seq_start + r);
    }
  }
  int64_t t0 = 0;
  for (int32_t s = 0; s < n_seqs; ++s) {
    const int64_t L = seq_lens[s];
    if (k_from)
      for (int32_t pos = 0; pos < L; ++pos) k_from[t0 + pos] = mask.from(s, pos);
    if (eta) {
      int64_t extra = 0;       // pairs above the diagonal: n (n - 1) / 2 per span of n tokens
      for (const auto& sp : mask.by_seq[s]) extra += (int64_t)(sp.second - sp.first) * (sp.second - sp.first - 1) / 2;
      eta[s] = (float)((double)extra / (double)(L * (L + 1) / 2));
    }
    t0 += L;
  }
  return FCP_OK;
}

// Device-side tile scheduler for the attention kernels.
//
// The paper's motivation (Sec. 4.1) is that heterogeneous lengths leave some compute units
// as stragglers; inside one rank the same holds for tiles: a query block at the end of a long
// chunk has hundreds of key blocks, one from a short sequence has one.  This kernel turns the
// rank's work items (device memory) into a list of tiles sorted by DECREASING cost, which the
// persistent attention kernels pull from shared counters (longest-first list scheduling).
// Fully masked key blocks never enter the cost or the kernels' loops.
//
// It also validates every work item against the extents the caller passed, so that no
// attention kernel can be steered out of bounds by a bad descriptor: a rejected item gets
// no tiles and is counted in the header.
//
// A list is one block's work between two launches that wait for it, so what counts is the chain of dependent steps: trips to global memory and
// block barriers.  Items are fetched once into LDS with everything that depends on global memory (their sequence's place, what their last row
// sees), the exclusivity flags take the cheapest of three ways, nothing is indexed in scratch memory.  Time from the first
// to the last instruction of a list, forward / backward: 1 item 8.2 -> 5.6 us, 28 items 18 / 31 -> 11 / 13 us, 71 items 37 / 48 -> 14 / 12 us,
// 1000 items 64 / 65 -> 14 / 23 us.
#include "fcp_items.h"

namespace fcp {

namespace {

constexpr int kSchedThreads = 1024;
constexpr int kBuckets = 2048;
constexpr int kMaxExclusiveScan = kMaxFlaggedItems;   // longer lists are not staged in LDS and have no exclusivity flags

constexpr int kItemWords = 13;      // in LDS: the item, then the first flag block of its chain or the first turn number of its tiles (an odd stride: no bank conflicts)
using ItemSlot = int32_t[kItemWords];
__device__ inline void put_item(ItemSlot& r, const Item& it) {
  const int32_t w[12] = {it.seq, it.q_off, it.q_len, it.q_pos, it.k0, it.n0, it.k1, it.n1, it.base, it.vis0, it.vis1, it.step};
#pragma unroll
  for (int i = 0; i < 12; ++i) r[i] = w[i];
}
__device__ inline Item get_item(const ItemSlot& r) {
  return {r[0], r[1], r[2], r[3], r[4], r[5], r[6], r[7], r[8], r[9], r[10], r[11]};
}

// The thread's item of a list that is staged in LDS (none: rejected).
__device__ inline Item my_item(const ListArgs& a, const MaskTables& m) {
  if (a.n_work <= kMaxExclusiveScan && (int32_t)threadIdx.x < a.n_work) return load_item(a, m, threadIdx.x);
  return {-1, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0};
}

// query tile qt (of `tile` rows): cost = key blocks (of `inner` keys) its last row sees
__device__ inline int32_t fwd_cost(const MaskTables& m, const Item& it, int32_t qt, int32_t tile, int32_t inner) {
  const int64_t limit = m.limit(it, min((qt + 1) * tile, it.q_len) - 1);
  return ceil_div(seen_keys(it, 0, limit), inner) + (it.n1 > 0 ? ceil_div(seen_keys(it, 1, limit), inner) : 0);
}

// key tile kt (of `tile` keys) of segment s: the item's first row that sees its first key
__device__ inline int32_t first_row_of(const MaskTables& m, const Item& it, int s, int32_t kt, int32_t tile) {
  return (int32_t)max((int64_t)0, min((int64_t)it.q_len - 1, m.from(it, (int64_t)it.k(s) + (int64_t)kt * tile) - it.q_pos));
}
// ... and its cost = query blocks (of `inner` rows) from that row on; in a chained list blocks counted from the item's first row
template <bool Chain>
__device__ inline int32_t bwd_cost(const MaskTables& m, const Item& it, int s, int32_t kt, int32_t tile, int32_t inner) {
  const int32_t row = first_row_of(m, it, s, kt, tile);
  return Chain ? ceil_div(it.q_len, inner) - row / inner : ceil_div(it.q_len - row, inner);
}

// Exclusive block scan of one value per thread; returns the exclusive prefix and sets
// `total` (same for every thread).  `s_wave` holds one slot per wave.
__device__ inline int32_t block_exclusive_scan(int32_t v, int32_t* s_wave, int32_t& total) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  int32_t inc = v;
  for (int off = 1; off < 64; off <<= 1) {
    int32_t t = __shfl_up(inc, off, 64);
    if (lane >= off) inc += t;
  }
  __syncthreads();
  if (lane == 63) s_wave[wave] = inc;
  __syncthreads();
  int32_t base = 0, tot = 0;
  for (int w = 0; w < kSchedThreads / 64; ++w) {
    const int32_t x = s_wave[w];
    if (w < wave) base += x;
    tot += x;
  }
  total = tot;
  return base + inc - v;
}

// Exclusivity flags: an item whose query rows (key segments) no other valid item of this launch touches lets the
// backward kernels add to dQ (dK/dV) without atomics, or write the final result directly.
// Flags of all items at once (n_work <= kMaxExclusiveScan, staged in LDS).  Query rows are one set of intervals over all valid items, key segments
// one set of up to two per item, ordered by (sequence, start): only segments of the same sequence can overlap, and an item's own two
// segments count like anybody else's.  Three ways:
//   * a list in row order, every interval behind the one before (packed whole sequences): one look at the neighbour finds that out;
//   * up to kSmallList items: all pairs;
//   * else by sorting: intervals sorted by their start overlap an earlier one iff the largest end so far exceeds their start, and a
//     later one iff the next start lies before their end.  The sequence enters the sort key with its low 21 bits: two
//     sequences that collide there are treated as one, which can only clear a flag that could have been set (the safe side).
// `key`: LDS work area of 2 * kMaxExclusiveScan entries; `fl`: LDS, one word per item, written here.
__device__ inline void bitonic_sort(uint64_t* key, int32_t n_pow2) {
  // A list written in row order (the usual case: items by sequence, chunks by position) is sorted already: one pass
  // over the neighbours finds that out, and the log^2 rounds of exchanges and block barriers are skipped.
  int ordered = 1;
  for (int32_t t = threadIdx.x; t + 1 < n_pow2; t += kSchedThreads) ordered &= key[t] <= key[t + 1];
  if (__syncthreads_and(ordered)) return;
  for (int32_t k = 2; k <= n_pow2; k <<= 1)
    for (int32_t j = k >> 1; j > 0; j >>= 1) {
      for (int32_t t = threadIdx.x; t < n_pow2 / 2; t += kSchedThreads) {
        const int32_t i = ((t & ~(j - 1)) << 1) | (t & (j - 1)), l = i | j;
        const uint64_t a = key[i], b = key[l];
        if ((a > b) == ((i & k) == 0)) { key[i] = b; key[l] = a; }
      }
      __syncthreads();
    }
}

// Inclusive running maximum over the block's values in thread order (two per thread: v0 then v1).  `s_wmax`: 16 slots.
__device__ inline void block_running_max(uint64_t v0, uint64_t v1, uint64_t* s_wmax, uint64_t& before0, uint64_t& before1) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  uint64_t inc = v0 > v1 ? v0 : v1;
  for (int off = 1; off < 64; off <<= 1) {
    const uint64_t o = __shfl_up(inc, off, 64);
    if (lane >= off && o > inc) inc = o;
  }
  __syncthreads();
  if (lane == 63) s_wmax[wave] = inc;
  __syncthreads();
  uint64_t base = 0;
  for (int w = 0; w < wave; ++w) base = s_wmax[w] > base ? s_wmax[w] : base;
  uint64_t prev = __shfl_up(inc, 1, 64);        // maximum up to and including the thread before, inside the wave
  if (lane == 0) prev = 0;
  before0 = prev > base ? prev : base;          // maximum of everything before v0
  before1 = before0 > v0 ? before0 : v0;        // ... before v1
}

constexpr int kSmallList = 256;   // (all pairs take about 5 us there, the two sorts 25 at any length)

__device__ inline void exclusive_flags_all(const ItemSlot* item, int32_t n_work, uint64_t* key, uint64_t* s_wmax, int32_t* fl) {
  const int tid = threadIdx.x;
  constexpr uint64_t kNone = ~(uint64_t)0;
  constexpr int32_t kAll = kFlagQExclusive | kFlagSeg0Exclusive | kFlagSeg1Exclusive;
  static_assert(kMaxExclusiveScan <= kSchedThreads, "one item per thread");
  bool in_order = true;
  if (tid < n_work) {
    const Item a = get_item(item[tid]);
    fl[tid] = a.seq < 0 ? 0 : kAll;
    in_order = a.seq >= 0 && (a.n1 == 0 || a.k1 >= a.k0 + a.n0);
    if (tid > 0) {
      const Item b = get_item(item[tid - 1]);
      in_order &= a.q_off >= b.q_off + b.q_len && (a.seq > b.seq || (a.seq == b.seq && a.k0 >= (b.n1 > 0 ? b.k1 + b.n1 : b.k0 + b.n0)));
    }
  }
  if (__syncthreads_and(in_order)) return;
  if (n_work <= kSmallList) {
    // thread = (item, share of the others); the lanes of a wave look at the same other item
    int32_t p = 1;
    while (p < n_work) p <<= 1;
    const int32_t ia = tid & (p - 1), parts = kSchedThreads / p;
    if (ia < n_work && fl[ia] != 0) {
      const Item a = get_item(item[ia]);
      int32_t lost = a.n1 > 0 && a.k0 < a.k1 + a.n1 && a.k1 < a.k0 + a.n0 ? kFlagSeg0Exclusive | kFlagSeg1Exclusive : 0;
      for (int32_t ib = tid / p; ib < n_work; ib += parts) {
        const Item b = get_item(item[ib]);
        if (ib == ia || b.seq < 0) continue;
        if (a.q_off < b.q_off + b.q_len && b.q_off < a.q_off + a.q_len) lost |= kFlagQExclusive;
        if (a.seq != b.seq) continue;
        auto meets = [](int32_t k, int32_t n, int32_t ks, int32_t ns) { return n > 0 && ns > 0 && k < ks + ns && ks < k + n; };
        if (meets(a.k0, a.n0, b.k0, b.n0) || meets(a.k0, a.n0, b.k1, b.n1)) lost |= kFlagSeg0Exclusive;
        if (meets(a.k1, a.n1, b.k0, b.n0) || meets(a.k1, a.n1, b.k1, b.n1)) lost |= kFlagSeg1Exclusive;
      }
      if (lost) atomicAnd(&fl[ia], ~lost);
    }
    __syncthreads();
    return;
  }
  // ---- query rows: key = start << 11 | item
  int32_t np = 2;
  while (np < n_work) np <<= 1;
  for (int32_t i = tid; i < np; i += kSchedThreads)
    key[i] = (i < n_work && item[i][0] >= 0) ? ((uint64_t)(uint32_t)item[i][1] << 11) | (uint64_t)i : kNone;
  __syncthreads();
  bitonic_sort(key, np);
  {
    // one element per thread (np <= kSchedThreads): value of the running maximum = end
    const uint64_t k0 = tid < np ? key[tid] : kNone;
    const bool live = k0 != kNone;
    const int32_t i = live ? (int32_t)(k0 & 2047) : 0;
    const uint64_t end = live ? (uint64_t)(uint32_t)(item[i][1] + item[i][2]) : 0;
    uint64_t before, unused;
    block_running_max(end, 0, s_wmax, before, unused);
    if (live) {
      const uint64_t start = k0 >> 11;
      const uint64_t nxt = tid + 1 < np ? key[tid + 1] : kNone;
      const bool hit = before > start || (nxt != kNone && (nxt >> 11) < end);
      if (hit) atomicAnd(&fl[i], ~kFlagQExclusive);
    }
  }
  __syncthreads();
  // ---- key segments: key = seq (21 bits) << 43 | start (31 bits) << 12 | slot (item * 2 + segment)
  int32_t np2 = 2;
  while (np2 < 2 * n_work) np2 <<= 1;
  for (int32_t sl = tid; sl < np2; sl += kSchedThreads) {
    const int32_t i = sl >> 1, sg = sl & 1;
    uint64_t k = kNone;
    if (i < n_work && item[i][0] >= 0 && item[i][5 + 2 * sg] > 0)
      k = ((uint64_t)(item[i][0] & 0x1FFFFF) << 43) | ((uint64_t)(uint32_t)item[i][4 + 2 * sg] << 12) | (uint64_t)sl;
    key[sl] = k;
  }
  __syncthreads();
  bitonic_sort(key, np2);
  {
    // two consecutive elements per thread; value of the running maximum = seq << 32 | end
    auto unpack = [&](uint64_t k, uint64_t& val, uint64_t& seqm, uint64_t& start, int32_t& slot) {
      slot = (int32_t)(k & 4095);
      start = (k >> 12) & 0x7FFFFFFFu;
      seqm = k >> 43;
      const ItemSlot& r = item[slot >> 1];
      val = (seqm << 32) | (uint64_t)(uint32_t)(r[4 + 2 * (slot & 1)] + r[5 + 2 * (slot & 1)]);
    };
    const int32_t p0 = 2 * tid, p1 = 2 * tid + 1;
    const uint64_t k0 = p0 < np2 ? key[p0] : kNone, k1 = p1 < np2 ? key[p1] : kNone;
    uint64_t v0 = 0, v1 = 0, q0 = 0, q1 = 0, st0 = 0, st1 = 0;
    int32_t sl0 = 0, sl1 = 0;
    if (k0 != kNone) unpack(k0, v0, q0, st0, sl0);
    if (k1 != kNone) unpack(k1, v1, q1, st1, sl1);
    uint64_t b0, b1;
    block_running_max(v0, v1, s_wmax, b0, b1);
    const uint64_t k2 = p1 + 1 < np2 ? key[p1 + 1] : kNone;
    auto test = [&](uint64_t k, uint64_t val, uint64_t seqm, uint64_t start, int32_t slot, uint64_t before, uint64_t nxt) {
      if (k == kNone) return;
      bool hit = (before >> 32) == seqm && (before & 0xFFFFFFFFu) > start;            // an earlier segment of the sequence ends after this start
      if (nxt != kNone && (nxt >> 43) == seqm && ((nxt >> 12) & 0x7FFFFFFFu) < (val & 0xFFFFFFFFu)) hit = true;   // the next one starts before this end
      if (hit) atomicAnd(&fl[slot >> 1], ~((slot & 1) ? kFlagSeg1Exclusive : kFlagSeg0Exclusive));
    };
    test(k0, v0, q0, st0, sl0, b0, k1);
    test(k1, v1, q1, st1, sl1, b1, k2);
  }
  __syncthreads();
}

// What the key-tile and query-tile lists of a backward are like: one unit per tile; the chains of the one-pass kernel; tiles split where
// whole ones would leave most of the chip idle (see split_sizes).
enum ListMode { kWhole, kChained, kSplit };

// Split tiles.  A unit is a serial loop over the 32-row blocks (key tiles: of every query head of the KV head) or the 32-key
// blocks (query tiles) that the tile meets.  On small problems the longest of these loops, not the sum of the work, sets the time: a
// sequence of 4096 tokens with 3 query heads per KV head has a key tile of 384 steps where an even spread over the CUs would
// be 37.  So a key tile's rows are cut into pieces of `rows` rows of the item, a query tile's keys into pieces of `keys` keys of a segment, and
// every piece is a unit; the pieces of a tile add to its accumulators with atomics, and where one item owns the rows they take turns
// (see wait_turn in csrc/fcp_bwd.h), so that the sums of such rows repeat bit for bit as those of whole tiles do.
// Size of a piece, in steps: a CU's even share of all steps; not less than sqrt(steps / 8), where the loop of a piece and the atomics of all of them
// take the same time (a piece's 32 K elements go at one element per L2 channel and clock, an eighth of a step's time); not less
// than sqrt(kTurnSteps longest loop), where the loop of a piece and the turns of its tile take the same time; not less
// than min_steps, a unit's own beginning and end.  Nothing is split unless the longest loop is clearly longer than what the pieces
// take: the share, half a piece at the end of the list, the atomics of the items whose tiles are longer than a piece, the turns.
struct SplitArgs { int32_t group, kv_units, q_units, dq_tile, n_cu, min_steps, key_turns, row_turns, blocks_per_cu, many_short; };
struct SplitSizes { int32_t rows, keys; };
constexpr int32_t kNoPieces = 1 << 24;
// Least ratio of the longest loop to what the pieces take.  Key tiles, two blocks per CU and three (64 channels): the blocks share the CU's matrix units, so
// that on a filled chip a loop takes longer than its steps say (64 channels, at 1.15 / 0.85 / 0.6: 8192 tokens, 4 heads 222 / 186 / 186 us; 30 sequences of
// 20011 tokens, the longest over 3 ranks, 110 / 110 / 132; 8192 tokens, 40 heads on 8 1207 / 1207 / 1507).  Query tiles have a second way to
// shorten their loops, halves (see bwd_lists_kernel), which lists with pieces of query tiles do without: 24 sequences of 32768 tokens, 4 heads of 64
// channels, just below 1.18, 350 us whole and 422 in pieces.
constexpr float kSplitGainKeys2 = 1.12f, kSplitGainKeys3 = 0.85f, kSplitGainRows = 1.18f;
constexpr float kTurnSteps = 4.f;      // one piece's turn, in steps: its atomics, their acknowledgement, the word (1.5 to 6 within 5 % of each other)

// Called by every thread of the block, with its item (rejected: none).  Every block that asks gets the same answer: sums are formed in a fixed
// order, and nothing is contracted differently where the function is inlined twice.
__device__ inline SplitSizes split_sizes(const SplitArgs& a, const MaskTables& m, const Item& it, int32_t fl, int32_t n_work) {
#pragma clang fp contract(off)
  __shared__ float s_part[kSchedThreads / 64][8];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, n_waves = (n_work + 63) >> 6;
  // the item's steps (the average of its first and last tile times the tiles) and its longest tile, also among those it owns: key tiles, query tiles
  float steps[2] = {0.f, 0.f}, longest[2] = {0.f, 0.f}, owned[2] = {0.f, 0.f};
  if (it.seq >= 0) {
#pragma unroll
    for (int s = 0; s < 2; ++s) {
      const int32_t nt = ceil_div(it.vis(s), kBwdBN);
      if (nt == 0) continue;
      const int32_t c0 = bwd_cost<false>(m, it, s, 0, kBwdBN, kBwdBM), c1 = bwd_cost<false>(m, it, s, nt - 1, kBwdBN, kBwdBM);
      steps[0] += 0.5f * nt * (c0 + c1) * a.group * a.kv_units;
      longest[0] = fmaxf(longest[0], c0 * a.group);
      if (fl & (s ? kFlagSeg1Exclusive : kFlagSeg0Exclusive)) owned[0] = fmaxf(owned[0], c0 * a.group);
    }
    const int32_t nq = ceil_div(it.q_len, a.dq_tile);
    longest[1] = ceil_div(it.vis0, kDqBN) + ceil_div(it.vis1, kDqBN);
    if (fl & kFlagQExclusive) owned[1] = longest[1];
    // (a row unit's step is half of what a CU does at a time)
    steps[1] = 0.25f * nq * (fwd_cost(m, it, 0, a.dq_tile, kDqBN) + longest[1]) * a.q_units;
  }
  auto wave_sum = [](float v) { for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64); return v; };
  auto wave_max = [](float v) { for (int o = 32; o > 0; o >>= 1) v = fmaxf(v, __shfl_xor(v, o, 64)); return v; };
  if (wave < n_waves) {
    const float p[6] = {wave_sum(steps[0]), wave_sum(steps[1]), wave_max(longest[0]), wave_max(longest[1]), wave_max(owned[0]), wave_max(owned[1])};
    if (lane == 0)
#pragma unroll
      for (int i = 0; i < 6; ++i) s_part[wave][i] = p[i];
  }
  __syncthreads();
  float all[2] = {0.f, 0.f}, top[2] = {0.f, 0.f}, turns[2] = {0.f, 0.f}, piece[2];
  for (int w = 0; w < n_waves; ++w)
#pragma unroll
    for (int l = 0; l < 2; ++l) {
      all[l] += s_part[w][l];
      top[l] = fmaxf(top[l], s_part[w][2 + l]);
      turns[l] = fmaxf(turns[l], kTurnSteps * s_part[w][4 + l]);
    }
#pragma unroll
  for (int l = 0; l < 2; ++l)
    piece[l] = fmaxf(fmaxf(all[l] / a.n_cu, sqrtf(all[l] * 0.125f)), fmaxf(sqrtf(turns[l]), (float)a.min_steps));
  if (wave < n_waves) {
    const float p[2] = {wave_sum(longest[0] > piece[0] ? steps[0] : 0.f), wave_sum(longest[1] > piece[1] ? steps[1] : 0.f)};
    if (lane == 0) { s_part[wave][6] = p[0]; s_part[wave][7] = p[1]; }
  }
  __syncthreads();
#pragma unroll
  for (int l = 0; l < 2; ++l) {
    float heavy = 0.f;
    for (int w = 0; w < n_waves; ++w) heavy += s_part[w][6 + l];
    const float pieces = all[l] / a.n_cu + 0.5f * piece[l] + 0.125f * heavy / piece[l] + turns[l] / piece[l] + 4.f;
    const float gain = l ? kSplitGainRows : a.blocks_per_cu > 2 ? kSplitGainKeys3 : kSplitGainKeys2;
    if (top[l] < gain * pieces) piece[l] = kNoPieces;
  }
  return {piece[0] < kNoPieces ? 32 * max(1, (int32_t)piece[0] / a.group) : 32 * kNoPieces, 32 * (int32_t)piece[1]};
}

// One pass or two, where the longest item decides (lists of several short items that the caller may have put a long one among).  Estimated times
// in us, from the list: tiles and steps per CU and the longest tile's loop.  In one pass a chain is a serial loop as long as its first tile's, and with
// several query heads per KV head its other tiles keep that tile's pace through all heads: `idle` steps, those that they lack
// against it.  Fitted to 124 lists of 30 to 1000 short sequences and one of 512 to 65536 tokens, 1, 2 and 4 heads per KV head (5 and 10 % off on
// average).  On these and on 117 others (log-normal lengths, several long ones, 1 to 8 heads per KV head) the way chosen takes 0.4 % longer than the
// faster one on average and 17 % at most; one pass for all of them 4 % and 57 %.
// The kernel of many short sequences (a.many_short), fitted to 60 lists of 120 to 1000 short sequences with and without one of 512 to 16384 tokens, 1 to 5 heads per
// KV head: the way chosen takes 0.2 % longer than the faster one on average and 9 % at most; one pass for all of them 19 %.
// Called by every thread of the block, with its item.  Every block that asks gets the same answer.
__device__ inline bool one_pass_pays(const SplitArgs& a, const MaskTables& m, const Item& it, int32_t n_work) {
#pragma clang fp contract(off)
  __shared__ float s_part[kSchedThreads / 64][4];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, n_waves = (n_work + 63) >> 6;
  float units = 0.f, steps = 0.f, idle = 0.f, longest = 0.f;
  if (it.seq >= 0) {
#pragma unroll
    for (int s = 0; s < 2; ++s) {
      const int32_t nt = ceil_div(it.vis(s), kBwdBN);
      if (nt == 0) continue;
      const int32_t c0 = bwd_cost<true>(m, it, s, 0, kBwdBN, kBwdBM), c1 = bwd_cost<true>(m, it, s, nt - 1, kBwdBN, kBwdBM);
      units += nt;
      steps += 0.5f * nt * (c0 + c1) * a.group;
      idle += 0.5f * nt * (c0 - c1) * a.group;
      longest = fmaxf(longest, (float)(c0 * a.group));
    }
  }
  if (wave < n_waves) {
    for (int o = 32; o > 0; o >>= 1) {
      units += __shfl_xor(units, o, 64);
      steps += __shfl_xor(steps, o, 64);
      idle += __shfl_xor(idle, o, 64);
      longest = fmaxf(longest, __shfl_xor(longest, o, 64));
    }
    if (lane == 0) { s_part[wave][0] = units; s_part[wave][1] = steps; s_part[wave][2] = idle; s_part[wave][3] = longest; }
  }
  __syncthreads();
  units = steps = idle = longest = 0.f;
  for (int w = 0; w < n_waves; ++w) {
    units += s_part[w][0];
    steps += s_part[w][1];
    idle += s_part[w][2];
    longest = fmaxf(longest, s_part[w][3]);
  }
  const float per_cu = (float)a.kv_units / a.n_cu;
  if (a.many_short) {
    const float work = (4.04f * units + 1.17f * steps + 1.02f * idle) * per_cu, chain = 2.72f * longest;
    return 25.f + sqrtf(sqrtf(work * work * work * work + chain * chain * chain * chain)) <= 18.5f + (6.9f * units + 1.74f * steps) * per_cu;
  }
  const float one = 21.f + fmaxf((7.9f * units + 1.36f * steps + (a.group > 1 ? 0.64f : 0.41f) * idle) * per_cu, 1.46f * longest);
  const float two = 47.f + fmaxf((12.9f * units + 1.65f * steps) * per_cu, 1.12f * longest);
  return one <= two;
}

// Pieces of a query tile: up to this many, those of segment 0 first (one for a tile that is not split).
__device__ inline int32_t key_slots(const Item& it, int32_t keys) { return max(1, ceil_div(it.vis0, keys) + ceil_div(it.vis1, keys)); }
// The pieces of a key tile: numbers first .. first + count - 1.  A later tile of the segment lacks the leading ones.
struct RowPieces { int32_t first, count; };
__device__ inline RowPieces row_pieces(const MaskTables& m, const Item& it, int s, int32_t kt, int32_t rows) {
  const int32_t first = first_row_of(m, it, s, kt, kBwdBN) / rows;
  return {first, ceil_div(it.q_len, rows) - first};
}

// Pieces of a tile stand in the list by bucket (decreasing), then in the order of their flat numbers.  How many stand before piece `offset` of
// run `at`, for pieces that come in runs of equal buckets.
struct PieceRun { int32_t count, bucket; };
template <int N>
__device__ inline int32_t pieces_before(const PieceRun (&run)[N], int at, int32_t offset) {
  int32_t n = offset, mine = 0;
#pragma unroll
  for (int i = 0; i < N; ++i) mine = i == at ? run[i].bucket : mine;
#pragma unroll
  for (int i = 0; i < N; ++i)
    if (i != at && (run[i].bucket > mine || (i < at && run[i].bucket == mine))) n += run[i].count;
  return n;
}

// LDS shared between the flags' sort (first) and the list builder's histogram and offsets (afterwards).
struct SortArea {
  union {
    uint64_t key[2 * kMaxExclusiveScan];
    struct { int32_t hist[kBuckets]; int32_t off[kMaxExclusiveScan + 1]; } later;
  };
  uint64_t wmax[kSchedThreads / 64];
};

// One tile list, built by one block.
template <ListMode Mode, bool ManyShort = false>
__device__ void build_list(
    bool backward, int32_t tile, int32_t inner, const ListArgs& args, const MaskTables& m,
    int32_t tile_cap, SchedHeader* hdr, int32_t* item_off, Tile* tiles,
    ItemSlot* s_item,                    // LDS, kMaxExclusiveScan slots
    SortArea* area, int32_t* s_fl,       // LDS: sort keys (later the histogram and the offsets), one flag word per item
    int32_t* chain,                      // kChained: the tiles' chain records
    const SplitArgs& sargs,              // kSplit
    bool stable,                         // tiles of one bucket in the order of their numbers (chains and pieces always)
    const Item& mine) {                  // staged lists: the thread's item, or a rejected one
  __shared__ int32_t s_wave[kSchedThreads / 64];
  __shared__ int32_t s_max, s_rej;
  constexpr bool Chain = Mode == kChained;
  int32_t* const s_hist = area->later.hist;
  int32_t* const s_off = area->later.off;          // item_off for staged lists
  const int tid = threadIdx.x, lane = tid & 63;
  const int32_t n_work = args.n_work;
  const bool staged = n_work <= kMaxExclusiveScan;
  SplitSizes split{};
  bool cut = false;                                // tiles are split (the same for every thread)
  int32_t path = Mode == kChained ? kPathOnePass : 0;
  if (tid == 0) { s_max = 0; s_rej = 0; }
  if (staged && tid < n_work) put_item(s_item[tid], mine);
  __syncthreads();                                 // (for every list: the other waves add to s_max and s_rej below)
  if (staged) {
    exclusive_flags_all(s_item, n_work, area->key, area->wmax, s_fl);
    if constexpr (Mode == kSplit) {
      split = split_sizes(sargs, m, mine, tid < n_work ? s_fl[tid] : 0, n_work);
      cut = (backward ? split.rows : split.keys) < 32 * kNoPieces;
      path = (split.rows < 32 * kNoPieces ? kPathSplitKeys : 0) | (split.keys < 32 * kNoPieces ? kPathSplitRows : 0);
    }
  }
  auto fetch = [&](int32_t i) { return staged ? get_item(s_item[i]) : load_item(args, m, i); };
  for (int b = tid; b < kBuckets; b += kSchedThreads) s_hist[b] = 0;   // (the sort keys are done with)

  // Chains (key tiles only, at most kMaxExclusiveScan items): the flags of the query blocks of the items that own their rows.
  if constexpr (Chain) {
    const int32_t nb = tid < n_work && (s_fl[tid] & kFlagQExclusive) ? ceil_div(mine.q_len, inner) : 0;
    int32_t total;
    const int32_t ex = block_exclusive_scan(nb, s_wave, total);
    if (tid < n_work) s_item[tid][12] = ex;
  }

  // Split tiles: the first turn number of the tiles of the items that own their rows (query tiles) or of the segments that own their keys.
  if (Mode == kSplit && cut) {
    int32_t nt = 0;
    if (tid < n_work) {
      const int32_t fl = s_fl[tid];
      if (backward) nt = (fl & kFlagSeg0Exclusive ? ceil_div(mine.vis0, tile) : 0) + (fl & kFlagSeg1Exclusive ? ceil_div(mine.vis1, tile) : 0);
      else nt = fl & kFlagQExclusive ? ceil_div(mine.q_len, tile) : 0;
    }
    int32_t total;
    const int32_t ex = block_exclusive_scan(nt, s_wave, total);
    if (tid < n_work) s_item[tid][12] = ex;
  }

  // Pass 1: count tiles per item, exclusive offsets.
  int32_t total_tiles = 0;
  for (int32_t base = 0; base < n_work; base += kSchedThreads) {
    const int32_t i = base + tid;
    int32_t cnt = 0, cost = 0, bad = 0;
    if (i < n_work) {
      const Item it = staged ? mine : load_item(args, m, i);
      if (it.seq < 0) {
        bad = 1;
      } else if (!backward) {
        cnt = ceil_div(it.q_len, tile);
        cost = ceil_div(it.vis0, inner) + ceil_div(it.vis1, inner);
        if (Mode == kSplit && cut) cnt *= key_slots(it, split.keys);
      } else {
        const int32_t nt0 = ceil_div(it.vis0, tile), nt1 = ceil_div(it.vis1, tile);
        cnt = nt0 + nt1;
        cost = ceil_div(it.q_len, inner);
        if (Mode == kSplit && cut)
          cnt = (nt0 > 0 ? nt0 * row_pieces(m, it, 0, 0, split.rows).count : 0) + (nt1 > 0 ? nt1 * row_pieces(m, it, 1, 0, split.rows).count : 0);
      }
    }
    for (int o = 32; o > 0; o >>= 1) cost = max(cost, __shfl_xor(cost, o, 64));
    const uint64_t n_bad = __builtin_amdgcn_ballot_w64(bad != 0);
    if (lane == 0) {
      if (cost > 0) atomicMax(&s_max, cost);
      if (n_bad) atomicAdd(&s_rej, __builtin_popcountll(n_bad));
    }
    int32_t total;
    const int32_t ex = block_exclusive_scan(cnt, s_wave, total);
    if (i < n_work) (staged ? s_off : item_off)[i] = total_tiles + ex;
    total_tiles += total;
  }
  __syncthreads();
  const int32_t n_tiles = min(total_tiles, tile_cap);
  if (tid == 0 && total_tiles > tile_cap) s_rej += total_tiles - tile_cap;
  int shift = 0;
  while ((s_max >> shift) >= kBuckets) ++shift;

  // Pass 2 and 3 share the decode of a flat tile number into its resolved record and cost.
  auto item_of = [&](int32_t t) {
    int32_t lo = 0, hi = n_work - 1;               // last item with item_off <= t
    while (lo < hi) {
      const int32_t mid = (lo + hi + 1) >> 1;
      if ((staged ? s_off[mid] : item_off[mid]) <= t) lo = mid; else hi = mid - 1;
    }
    return lo;
  };
  auto bucket_of = [&](int32_t cost) { return min(cost >> shift, kBuckets - 1); };
  // What a tile is sorted by: its cost.  For the kernel of many short sequences, in lists of four units per block and more, the chained tiles of an item with
  // one segment all stand where its longest does, one after the other: the Q and dO rows, and what a tile leaves of dQ, are then still in the caches for
  // the next tile, which works a step behind it.  (By their own cost the second tiles come after all first ones.  Scheduling and one-pass launch, by cost / by
  // item: 400 sequences of 256 tokens, 32 query heads on 8 1322 / 1203 us, 1000 of 128 on average 1289 / 1294, with 8 heads 527 / 507; but 60 of 160, less than
  // two units per block, 137 / 156: second tiles then wait for first ones that begin with them.)
  // (Compiled only into the launches that can be followed by that kernel: a longer one begins later, 1 us of 40 on 30 sequences of 100.)
  const bool by_item = ManyShort && sargs.many_short && (int64_t)n_tiles * sargs.kv_units >= 8 * sargs.n_cu;
  auto place_of = [&](int32_t t, int32_t cost) {
    if (ManyShort && by_item) {
      const Item it = get_item(s_item[item_of(t)]);
      if (it.vis0 == 0 || it.vis1 == 0) return bucket_of(ceil_div(it.q_len, inner));
    }
    return bucket_of(cost);
  };
  auto decode = [&](int32_t t, Tile& out) -> int32_t {
    const int32_t at = item_of(t);
    const Item it = fetch(at);
    const int32_t local = t - (staged ? s_off[at] : item_off[at]);
    const int32_t fl = staged ? s_fl[at] : 0;
    if (!backward) {
      int32_t slots = 1, qt = local;
      if (Mode == kSplit && cut) {
        slots = key_slots(it, split.keys);
        qt = local / slots;
      }
      QTile q{};
      const int32_t r0 = qt * tile;
      q.q_row0 = it.q_off + r0;
      q.q_pos0 = it.q_pos + r0;
      q.rows = min(tile, it.q_len - r0);
      q.step = it.step;
      const int64_t limit = m.limit(it, r0 + q.rows - 1);
      const int32_t v0 = seen_keys(it, 0, limit), v1 = it.n1 > 0 ? seen_keys(it, 1, limit) : 0;
      q.kv_row0[0] = it.base + it.k0;
      q.k_pos0[0] = it.k0;
      q.vis[0] = v0;
      q.kv_row0[1] = it.n1 > 0 ? it.base + it.k1 : 0;
      q.k_pos0[1] = it.k1;
      q.vis[1] = v1;
      q.flags = fl;
      int32_t cost = ceil_div(v0, inner) + ceil_div(v1, inner);
      if (Mode == kSplit && cut) {
        int32_t slot = local - qt * slots;
        if (v0 + v1 > split.keys) {
          const int32_t c0 = ceil_div(it.vis0, split.keys);
          const int sg = slot < c0 ? 0 : 1;
          const int32_t first = (slot - (sg ? c0 : 0)) * split.keys;
          const int32_t vis = min(split.keys, (sg ? v1 : v0) - first);
          q.kv_row0[0] = it.base + it.k(sg) + first;
          q.k_pos0[0] = it.k(sg) + first;
          q.vis[0] = vis;
          q.kv_row0[1] = q.k_pos0[1] = q.vis[1] = 0;
          q.flags = fl & ~kFlagQExclusive;
          cost = vis > 0 ? ceil_div(vis, inner) : -1;
          q.turn = s_item[at][12] + qt;
          if (vis > 0 && (fl & kFlagQExclusive) && q.turn < sargs.row_turns && total_tiles <= tile_cap) {
            // runs: the full pieces of segment 0, its last one, those of segment 1
            const int32_t n0 = ceil_div(v0, split.keys), n1 = ceil_div(v1, split.keys), full = split.keys / inner;
            const int32_t t0 = ceil_div(v0 - (n0 - 1) * split.keys, inner), t1 = ceil_div(v1 - (n1 - 1) * split.keys, inner);
            const PieceRun run[4] = {{max(0, n0 - 1), bucket_of(full)}, {min(n0, 1), bucket_of(t0)},
                                     {max(0, n1 - 1), bucket_of(full)}, {min(n1, 1), bucket_of(t1)}};
            const int32_t i = slot - (sg ? c0 : 0), last = (sg ? n1 : n0) - 1;
            q.flags |= kFlagInTurn | pieces_before(run, 2 * sg + (i == last ? 1 : 0), i == last ? 0 : i) << kPieceShift;
          }
        } else if (slot > 0) {
          cost = -1;
        }
      }
      out = __builtin_bit_cast(Tile, q);
      return cost;
    }
    const int32_t nt0 = ceil_div(it.vis0, tile);
    int sg = local >= nt0 ? 1 : 0;
    int32_t kt = local - (sg ? nt0 : 0);
    int32_t row0 = 0, row1 = it.q_len;               // the unit's rows of the item
    bool whole = true;
    if (Mode == kSplit && cut) {
      RowPieces pc = nt0 > 0 ? row_pieces(m, it, 0, 0, split.rows) : RowPieces{0, 1};
      sg = local >= nt0 * pc.count ? 1 : 0;
      const int32_t l = local - (sg ? nt0 * pc.count : 0);
      if (sg) pc = row_pieces(m, it, 1, 0, split.rows);
      kt = l / pc.count;
      row0 = (pc.first + l - kt * pc.count) * split.rows;
      row1 = min(it.q_len, row0 + split.rows);
      if (first_row_of(m, it, sg, kt, tile) >= row1) return -1;
      whole = row_pieces(m, it, sg, kt, split.rows).count == 1;
      if (whole) { row0 = 0; row1 = it.q_len; }
    }
    KTile k{};
    k.k_pos0 = it.k(sg) + kt * tile;
    k.kv_row0 = it.base + k.k_pos0;
    k.n_keys = min(tile, it.vis(sg) - kt * tile);
    const int64_t last_q_pos = (int64_t)it.q_pos + row1 - 1;
    int32_t from[8];                                 // of every group's first and last key
#pragma unroll
    for (int g = 0; g < 8; ++g) from[g] = min(16 * (g & ~1) + 31 * (g & 1), k.n_keys - 1);
    if (m.k_from) {                                  // (one branch: the eight loads are in flight together)
#pragma unroll
      for (int g = 0; g < 8; ++g) from[g] = m.k_from[k.kv_row0 + from[g]];
    } else {
#pragma unroll
      for (int g = 0; g < 8; ++g) from[g] += k.k_pos0;
    }
#pragma unroll
    for (int g = 0; g < 8; ++g) {
      const int32_t f = (int32_t)min(last_q_pos, (int64_t)from[g]);
      if (g & 1) k.from_last[g / 2] = f; else k.from_first[g / 2] = f;
    }
    k.q_local_off = it.q_off + row0;
    k.q_seq_start = it.q_pos + row0;
    k.q_len = row1 - row0;
    const bool owned = (fl & (sg ? kFlagSeg1Exclusive : kFlagSeg0Exclusive)) != 0;
    k.flags = whole && owned ? kFlagSeg0Exclusive : 0;
    if (Mode == kSplit && !whole && owned) {
      k.turn = s_item[at][12] + (sg && (fl & kFlagSeg0Exclusive) ? nt0 : 0) + kt;
      if (k.turn < sargs.key_turns && total_tiles <= tile_cap) {
        // runs: the first piece (from the first row that sees the tile on), the full ones, the last one
        const RowPieces pc = row_pieces(m, it, sg, kt, split.rows);
        const int32_t end = (pc.first + 1) * split.rows, last0 = (pc.first + pc.count - 1) * split.rows;
        const PieceRun run[3] = {{1, bucket_of(ceil_div(end - first_row_of(m, it, sg, kt, tile), inner))}, {pc.count - 2, bucket_of(split.rows / inner)},
                                 {1, bucket_of(ceil_div(it.q_len - last0, inner))}};
        const int32_t i = row0 / split.rows - pc.first;
        const int ra = i == 0 ? 0 : i == pc.count - 1 ? 2 : 1;
        k.flags = kFlagInTurn | pieces_before(run, ra, ra == 1 ? i - 1 : 0) << kPieceShift;
      }
    }
    out = __builtin_bit_cast(Tile, k);
    const int32_t first = k.from_first[0] - it.q_pos;      // (first_row_of, before it is clamped)
    if (Chain) return ceil_div(it.q_len, inner) - max(0, first) / inner;
    return ceil_div(row1 - max(row0, first), inner);
  };

  // Place of key tile t in the chain of its item, if the item owns its query rows (else the tile adds with atomics, rank -1):
  // rank = number of the item's tiles before it, `next` = first query block of the tile after it (or past the last block),
  // `first` = its own first block, flag0 = the item's first flag block.  Order: by place (see place_of), then by flat number, which for an item of one
  // segment is that of its tiles' buckets too; for one of two segments: by bucket (decreasing), then by flat number.  Inside a
  // segment the buckets do not grow with the key, so the tiles of the other segment that come before are found by bisection.
  // Blocks are counted so that tiles of one bucket start at the same one: a tile later in the chain never starts at an earlier block.
  auto chain_place = [&](int32_t t, int32_t bucket, int32_t& rank, int32_t& next, int32_t& first, int32_t& flag0) {
    const int32_t at = item_of(t);
    const Item it = get_item(s_item[at]);
    const int32_t nqb = ceil_div(it.q_len, inner);
    auto first_block = [&](int32_t b) {               // first block of the tiles of bucket b
      const int64_t most = (((int64_t)b + 1) << shift) - 1;
      return b >= kBuckets - 1 || most >= nqb ? 0 : nqb - (int32_t)most;
    };
    first = first_block(bucket);
    next = nqb;
    rank = -1;
    flag0 = 0;
    // (a list that is cut lacks tiles that others would wait for: all of it adds with atomics)
    if (!(s_fl[at] & kFlagQExclusive) || total_tiles > tile_cap) return;
    flag0 = s_item[at][12];
    const int32_t nt0 = ceil_div(it.vis0, tile);
    const int32_t my_seg = t - s_off[at] >= nt0 ? 1 : 0;
    const int32_t my_kt = t - s_off[at] - (my_seg ? nt0 : 0);
    rank = my_kt;
#pragma unroll
    for (int sg = 0; sg < 2; ++sg) {
      const int32_t nt = ceil_div(it.vis(sg), tile);
      auto tile_bucket = [&](int32_t kt) { return bucket_of(bwd_cost<Chain>(m, it, sg, kt, tile, inner)); };
      int32_t a;                                      // the segment's first tile after t
      if (sg == my_seg) {
        a = my_kt + 1;
      } else {
        int32_t b = nt;                               // first kt with bucket < `bucket` (ties stand before t) or <= `bucket`
        a = 0;
        while (a < b) {
          const int32_t mid = (a + b) >> 1, bm = tile_bucket(mid);
          if (sg < my_seg ? bm < bucket : bm <= bucket) b = mid; else a = mid + 1;
        }
        rank += a;
      }
      if (a < nt) next = min(next, first_block(tile_bucket(a)));
    }
    if (rank == 0) first = 0;                         // rows that see no key get their zeros from the item's first tile
  };

  // (a thread's first tile and its cost stay in registers for the scatter pass: with up to 1024 tiles, all of them)
  Tile first_tile;
  int32_t first_cost = 0;
  for (int32_t t = tid; t < n_tiles; t += kSchedThreads) {
    Tile tl;
    const int32_t c = decode(t, tl);
    if (t == tid) { first_tile = tl; first_cost = c; }
    if (Mode != kSplit || c >= 0) atomicAdd(&s_hist[place_of(t, c)], 1);   // (-1: no such piece)
  }
  __syncthreads();
  // Descending-cost start offset of every bucket: scan the histogram from the top.
  int32_t n_listed;
  {
    static_assert(kBuckets == 2 * kSchedThreads, "two buckets per thread");
    const int b_hi = kBuckets - 1 - 2 * tid, b_lo = b_hi - 1;
    const int32_t h_hi = s_hist[b_hi], h_lo = s_hist[b_lo];
    const int32_t ex = block_exclusive_scan(h_hi + h_lo, s_wave, n_listed);
    __syncthreads();
    s_hist[b_hi] = ex;
    s_hist[b_lo] = ex + h_hi;
  }
  __syncthreads();
  if (!stable && (Mode == kWhole || (Mode == kSplit && !cut))) {
    for (int32_t t = tid; t < n_tiles; t += kSchedThreads) {
      Tile tl;
      int32_t c;
      if (t == tid) { tl = first_tile; c = first_cost; }
      else c = decode(t, tl);
      const int32_t pos = atomicAdd(&s_hist[bucket_of(c)], 1);
      tiles[pos] = tl;
    }
  } else {
    // The tiles of a chain, and the pieces of a tile, must stand in the list in the order in which they take turns: by bucket, then in the
    // order of the flat tile numbers, i.e. the scatter has to be stable (chained: by place, see above); so has that of the backward's query tiles, whose place says whether they are worked in halves.  A wave groups its lanes by bucket, the waves
    // take their places one after the other.
    for (int32_t base = 0; base < n_tiles; base += kSchedThreads) {
      const int32_t t = base + tid;
      Tile tl;
      int32_t c = -1, bucket = -1 - tid, rank = -1, next = 0, first = 0, flag0 = 0;
      if (t < n_tiles) {
        if (base == 0) { tl = first_tile; c = first_cost; }
        else c = decode(t, tl);
      }
      const bool live = c >= 0;                       // (kSplit, -1: no such piece)
      if (live) {
        if constexpr (Chain) chain_place(t, bucket_of(c), rank, next, first, flag0);
        bucket = place_of(t, c);
      }
      const int lane = tid & 63;
      uint64_t mine = 0;                              // lanes of the wave with this lane's bucket
      for (uint64_t todo = __builtin_amdgcn_ballot_w64(live); todo;) {
        const int l = __builtin_ctzll(todo);
        const int32_t bl = __builtin_amdgcn_readlane(bucket, l);
        const uint64_t m = __builtin_amdgcn_ballot_w64(live && bucket == bl);
        if (bucket == bl) mine = m;
        todo &= ~m;
      }
      const int before = __builtin_popcountll(mine & (((uint64_t)1 << lane) - 1));
      const int n_waves = min(kSchedThreads, n_tiles - base + 63) / 64;
      int32_t pos = 0;
      for (int w = 0; w < n_waves; ++w) {
        if ((tid >> 6) == w && live) {
          pos = s_hist[bucket] + before;
          if (before == 0) s_hist[bucket] = pos + __builtin_popcountll(mine);
        }
        __syncthreads();
      }
      if (live) {
        tiles[pos] = tl;
        if constexpr (Chain) {
          int32_t* r = chain + (int64_t)pos * kChainWords;
          r[0] = rank; r[1] = next; r[2] = flag0; r[3] = first;
        }
      }
    }
  }
  if (tid == 0) {
    hdr->n_tiles = n_listed;
    hdr->n_rejected = s_rej;
    hdr->max_cost = s_max;
    hdr->path = path;
    hdr->n_stalled = 0;
    for (int c = 0; c < 3; ++c) hdr->pad[c] = 0;
    for (int c = 0; c < kNumXcd; ++c) hdr->counter[c] = hdr->claimed[c] = 0;
  }
}

// Direct mode of the backward: where does the result of every query row / pool key come from?  State 0: no unit of
// this launch touches it (the result is zero); 1: it is accumulated in fp32 (several units, atomics) and converted
// afterwards - its accumulator row is cleared here; 2: one unit owns it and writes the final bf16 row itself.  The
// states follow the same exclusivity flags the kernels act on.  One lane per row, 64-row batches dealt out to the blocks in turn.
struct RowStateJob {
  uint8_t* q_state;        // NULL: no row states in this launch
  uint8_t* kv_state;       // NULL: query rows only (forward)
  float* dq_acc;           // accumulators whose state-1 rows are cleared, or NULL
  float* dk_acc;
  float* dv_acc;
  int32_t q_row_elems, kv_row_elems;
  int32_t n_parts, check_step;   // the validity rules of the list the states go with
  uint32_t* o_none;        // forward with one partial slot (see RowStates), or NULL
  float* lse_none;
  int32_t hq;
};
// The blocks `first` .. `first + count - 1` of the launch share the rows; LDS arrays come from the kernel.  `split`: the rows of split tiles are
// accumulated into.
template <bool Split>
__device__ void row_states(int first, int count, const RowStateJob& job, const ListArgs& args, const MaskTables& m, ItemSlot* s_item,
                           int32_t* s_fl, SortArea* area, const SplitArgs& sargs, const Item& item) {
  uint8_t* __restrict__ q_state = job.q_state;
  uint8_t* __restrict__ kv_state = job.kv_state;
  float* __restrict__ dq_acc = job.dq_acc;
  float* __restrict__ dk_acc = job.dk_acc;
  float* __restrict__ dv_acc = job.dv_acc;
  const int32_t q_row_elems = job.q_row_elems, kv_row_elems = job.kv_row_elems;
  const int32_t tq = args.tq, n_work = args.n_work, n_kv_rows = kv_state ? args.tkv : 0;
  const int tid = threadIdx.x, lane = tid & 63;
  if (tid < n_work) put_item(s_item[tid], item);
  __syncthreads();
  exclusive_flags_all(s_item, n_work, area->key, area->wmax, s_fl);
  SplitSizes split{};
  bool cut = false;
  if constexpr (Split) {
    split = split_sizes(sargs, m, item, tid < n_work ? s_fl[tid] : 0, n_work);
    cut = min(split.rows, split.keys) < 32 * kNoPieces;
  }
  // Only the keys that some row sees matter here.  A rejected item has empty ranges, so the passes over the list below carry no test
  // of validity.  An item without such keys has no key tile: in the backward its rows are untouched.
  if (n_kv_rows > 0 && tid < n_work && item.vis0 + item.vis1 == 0) s_item[tid][2] = 0;
  __syncthreads();

  // Rows are taken in batches of 64, one LANE per row.  Batch f belongs to block f mod count, so every block's batches
  // are spread evenly over all rows: any run of rows that must be cleared is shared by all blocks, and a block still
  // meets only the items that reach into one of its batches (for many short sequences a small part of the list),
  // which it picks first.  A wave then walks the picked items for its 64 rows (all lanes read the same item, an LDS
  // broadcast; nothing is exchanged between lanes).  The rows that are accumulated into go to a list in LDS, and the
  // block's 16 waves clear them in turn.  (Every row against every item, one wave per row and a search of cu_seqlens
  // per pool row, took 0.33 ms for 256 K rows and 1000 items.)
  const int64_t n_rows = (int64_t)tq + n_kv_rows;     // (the forward classifies its query rows only)
  const int64_t n_batches = (n_rows + 63) >> 6;
  const int64_t blk = blockIdx.x - first;
  const int wave = tid >> 6;
  int32_t* s_pick = reinterpret_cast<int32_t*>(area->key);                       // free again once the flags are known
  int64_t* s_clear = reinterpret_cast<int64_t*>(area->key + kMaxExclusiveScan);  // kSchedThreads rows at most
  int32_t* s_cnt = reinterpret_cast<int32_t*>(&area->wmax[0]);                   // [0] items picked, [1] rows to clear
  if (tid == 0) s_cnt[0] = 0;
  __syncthreads();
  {
    // do the n rows from s0 on meet a batch of this block?  The first batch at or after s0 / 64 that is ours.
    auto ours = [&](int64_t s0, int32_t n) {
      if (n <= 0) return false;
      const int64_t fs = s0 >> 6;
      int64_t d = (blk - fs) % count;
      if (d < 0) d += count;
      return ((fs + d) << 6) < s0 + n;
    };
    for (int32_t i = tid; i < n_work; i += kSchedThreads) {
      const Item it = get_item(s_item[i]);
      bool hit = ours(it.q_off, it.q_len);
      if (n_kv_rows > 0) hit = hit || ours((int64_t)tq + it.base + it.k0, it.vis0) || ours((int64_t)tq + it.base + it.k1, it.vis1);
      if (hit) s_pick[atomicAdd(&s_cnt[0], 1)] = i;
    }
  }
  __syncthreads();
  const int32_t n_cand = s_cnt[0];
  const float4 zero = make_float4(0.f, 0.f, 0.f, 0.f);
  const int64_t per_round = (int64_t)count * (kSchedThreads / 64);
  for (int64_t f0 = 0; f0 < n_batches; f0 += per_round) {    // the same trip count for every wave of the block
    if (tid == 0) s_cnt[1] = 0;
    const int64_t f = f0 + (int64_t)wave * count + blk;
    const int64_t r0 = f << 6, r = r0 + lane;
    const bool live = r < n_rows;
    int32_t at = 0, at_seg = 0;          // the last one found (kSplit)
    int32_t cnt = 0, own = 0;            // covering (item, segment) pairs; flags bit of the last one found
    // (no branch inside these loops: the reads of several items are in flight together)
    if (r0 + 63 < tq) {                  // 64 query rows
      const int32_t x = (int32_t)r;
#pragma unroll 4
      for (int32_t c = 0; c < n_cand; ++c) {
        const int32_t j = s_pick[c];
        const bool hit = (uint32_t)(x - s_item[j][1]) < (uint32_t)s_item[j][2];
        cnt += hit;
        own = hit ? s_fl[j] & kFlagQExclusive : own;
        if constexpr (Split) at = hit ? j : at;
      }
    } else if (r0 < n_rows) {            // pool rows, or the batch with the last query rows and the first pool rows
      const bool is_q = r < tq;
      const int32_t x = (int32_t)(is_q ? r : r - tq);
#pragma unroll 4
      for (int32_t c = 0; c < n_cand; ++c) {
        const int32_t j = s_pick[c];
        const int32_t fj = s_fl[j];
        const int32_t (&it)[kItemWords] = s_item[j];
        const int32_t y = x - it[8];
        const bool hq = is_q && (uint32_t)(x - it[1]) < (uint32_t)it[2];
        const bool h0 = !is_q && (uint32_t)(y - it[4]) < (uint32_t)it[9];
        const bool h1 = !is_q && (uint32_t)(y - it[6]) < (uint32_t)it[10];
        cnt += (int)hq + (int)h0 + (int)h1;
        own = hq ? fj & kFlagQExclusive : own;
        own = h0 ? fj & kFlagSeg0Exclusive : own;
        own = h1 ? fj & kFlagSeg1Exclusive : own;
        if constexpr (Split) { at = hq || h0 || h1 ? j : at; at_seg = h1 ? 1 : h0 ? 0 : at_seg; }
      }
    }
    if (Split && cut) {
      if (cnt == 1 && own != 0) {        // is the row's tile one of several units?
        const Item it = get_item(s_item[at]);
        if (r < tq) {
          const int32_t last = min(((int32_t)r - it.q_off) / sargs.dq_tile * sargs.dq_tile + sargs.dq_tile, it.q_len) - 1;
          const int64_t limit = m.limit(it, last);
          if (seen_keys(it, 0, limit) + (it.n1 > 0 ? seen_keys(it, 1, limit) : 0) > split.keys) own = 0;
        } else {
          const int32_t kt = ((int32_t)(r - tq) - it.base - it.k(at_seg)) / kBwdBN;
          if (row_pieces(m, it, at_seg, kt, split.rows).count > 1) own = 0;
        }
      }
    }
    const int state = cnt == 0 ? 0 : (cnt == 1 && own != 0) || job.o_none ? 2 : 1;
    if (live) {
      if (r < tq) q_state[r] = (uint8_t)state;
      else kv_state[r - tq] = (uint8_t)state;
    }
    __syncthreads();
    const bool clear = live && (job.o_none ? state == 0 : state == 1 && (r >= tq || dq_acc != nullptr));
    const uint64_t todo = __builtin_amdgcn_ballot_w64(clear);
    if (todo) {
      int32_t base = 0;
      if (lane == 0) base = atomicAdd(&s_cnt[1], __builtin_popcountll(todo));
      base = __builtin_amdgcn_readfirstlane(base);
      const int32_t pos = base + (int32_t)__builtin_amdgcn_mbcnt_hi((uint32_t)(todo >> 32),
                                                                     __builtin_amdgcn_mbcnt_lo((uint32_t)todo, 0));
      if (clear) s_clear[pos] = r;
    }
    __syncthreads();
    const int32_t n_clear = s_cnt[1];
    for (int32_t c = wave; c < n_clear; c += kSchedThreads / 64) {
      const int64_t rr = s_clear[c];
      if (job.o_none) {
        uint4* row = reinterpret_cast<uint4*>(job.o_none + rr * (q_row_elems / 2));
        for (int32_t e = lane; e < q_row_elems / 8; e += 64) row[e] = make_uint4(0, 0, 0, 0);
        for (int32_t h = lane; h < job.hq; h += 64) job.lse_none[(int64_t)h * tq + rr] = -INFINITY;
        continue;
      }
      if (rr < tq) {
        float4* row = reinterpret_cast<float4*>(dq_acc + rr * q_row_elems);
        for (int32_t e = lane; e < q_row_elems / 4; e += 64) row[e] = zero;
      } else {
        const int64_t kr = rr - tq;
        float4* rk = reinterpret_cast<float4*>(dk_acc + kr * kv_row_elems);
        float4* rv = reinterpret_cast<float4*>(dv_acc + kr * kv_row_elems);
        for (int32_t e = lane; e < kv_row_elems / 4; e += 64) { rk[e] = zero; rv[e] = zero; }
      }
    }
    __syncthreads();
  }
}

// The row states alone (launches that build no list).
__global__ __launch_bounds__(kSchedThreads) void row_state_kernel(const RowStateJob job, const ListArgs args, const MaskTables m) {
  __shared__ ItemSlot s_item[kMaxExclusiveScan];
  __shared__ int32_t s_fl[kMaxExclusiveScan];
  __shared__ SortArea s_area;
  row_states<false>(0, gridDim.x, job, args, m, s_item, s_fl, &s_area, SplitArgs{}, my_item(args, m));
}

struct ListJob {
  int32_t tile, inner, tile_cap;
  SchedHeader* hdr;
  int32_t* item_off;
  Tile* tiles;
};

// Forward (and the lists of empty calls): block 0 builds the list, the next `fill_blocks` blocks pre-fill the partial LSE with -inf,
// the blocks after those classify the rows (direct mode).
__global__ __launch_bounds__(kSchedThreads) void sched_kernel(
    int backward, const ListJob j, const ListArgs args, const MaskTables m,
    float* lse_fill, int64_t lse_fill_n, int fill_blocks, const RowStateJob states) {
  __shared__ ItemSlot s_item[kMaxExclusiveScan];
  __shared__ int32_t s_fl[kMaxExclusiveScan];
  __shared__ SortArea s_area;
  const int b = blockIdx.x;
  if (b == 0) {
    build_list<kWhole>(backward != 0, j.tile, j.inner, args, m, j.tile_cap, j.hdr, j.item_off, j.tiles, s_item, &s_area, s_fl, nullptr, SplitArgs{}, false, my_item(args, m));
  } else if (b <= fill_blocks) {
    const int64_t stride = (int64_t)fill_blocks * kSchedThreads;
    for (int64_t i = (int64_t)(b - 1) * kSchedThreads + threadIdx.x; i < lse_fill_n; i += stride)
      lse_fill[i] = -INFINITY;
  } else {
    row_states<false>(1 + fill_blocks, gridDim.x - 1 - fill_blocks, states, args, m, s_item, s_fl, &s_area, SplitArgs{}, my_item(args, m));
  }
}

// Backward: one launch for everything that precedes the attention kernels.  Block 0 builds the key-tile list
// (dK, dV), block 1 the query-tile list (dQ), the other blocks write the row statistics in the form
// the kernels consume: plane 0 = -LSE log2 e (-inf for a row without keys, so that its probabilities vanish),
// plane 1 = -delta.
// Other != Mode: the list decides which of the two it is (see one_pass_pays).
template <ListMode Mode, ListMode Other = Mode>
__global__ __launch_bounds__(kSchedThreads) void sched_bwd_kernel(
    const ListJob kv, const ListJob qt, const ListArgs args, const MaskTables m,
    const float* __restrict__ lse, const float* __restrict__ delta, int64_t n_stats, float* __restrict__ stats,
    int stat_blocks, int32_t* __restrict__ chain, int32_t* __restrict__ flags, int64_t n_flags, const SplitArgs split,
    const RowStateJob states) {
  __shared__ ItemSlot s_item[kMaxExclusiveScan];
  __shared__ int32_t s_fl[kMaxExclusiveScan];
  __shared__ SortArea s_area;
  const int b = blockIdx.x;
  if (b < 2) {
    const ListJob& j = b == 0 ? kv : qt;
    const Item mine = my_item(args, m);
    if (Other != Mode && !one_pass_pays(split, m, mine, args.n_work)) {
      build_list<Other>(b == 0, j.tile, j.inner, args, m, j.tile_cap, j.hdr, j.item_off, j.tiles, s_item, &s_area, s_fl, nullptr, split, b == 1, mine);
    } else if (Mode == kChained && b == 1) {        // the one-pass kernel has key tiles only
      if (Other != Mode && threadIdx.x == 0) {
        j.hdr->n_tiles = 0;
        j.hdr->path = kPathOnePass;
      }
    } else {
      build_list<Mode, Mode == kChained && Other != Mode>(b == 0, j.tile, j.inner, args, m, j.tile_cap, j.hdr, j.item_off, j.tiles, s_item, &s_area, s_fl, chain, split, b == 1, mine);
    }
  } else if (b < 2 + stat_blocks) {
    const int64_t stride = (int64_t)stat_blocks * kSchedThreads;
    for (int64_t i = (int64_t)(b - 2) * kSchedThreads + threadIdx.x; i < n_stats; i += stride) {
      const float l = lse[i];
      stats[i] = l == -INFINITY ? -INFINITY : -l * 1.4426950408889634f;
      stats[n_stats + i] = -delta[i];
    }
    if constexpr (Mode != kWhole)
      for (int64_t i = (int64_t)(b - 2) * kSchedThreads + threadIdx.x; i < n_flags; i += stride) flags[i] = 0;
  } else {   // direct mode: the row states, and the accumulator rows that are accumulated into cleared
    const Item mine = my_item(args, m);
    const int first = 2 + stat_blocks, count = gridDim.x - first;
    if (Other == kSplit && Other != Mode && !one_pass_pays(split, m, mine, args.n_work))
      row_states<true>(first, count, states, args, m, s_item, s_fl, &s_area, split, mine);
    else
      row_states<Mode == kSplit>(first, count, states, args, m, s_item, s_fl, &s_area, split, mine);
  }
}

}  // namespace

constexpr int kRowStateBlocks = 128;
static int row_state_blocks(int32_t tq, int32_t n_kv_rows) {
  int64_t blocks = ((int64_t)tq + n_kv_rows + kSchedThreads / 64 - 1) / (kSchedThreads / 64);
  // Every block stages the whole work list first, so few blocks with several rows per wave.  Measured on the 32K
  // workload (forward / backward scheduling launch): 64 blocks 34 / 81 us, 128 blocks 28 / 50, 256 blocks - / 57,
  // 512 blocks 41 / 58.
  if (blocks > kRowStateBlocks) blocks = kRowStateBlocks;
  return blocks < 1 ? 1 : (int)blocks;
}

static RowStateJob make_job(const RowStates* rs) {
  RowStateJob j{};
  if (rs) {
    j.q_state = rs->q_state; j.kv_state = rs->kv_state;
    j.dq_acc = rs->dq_acc; j.dk_acc = rs->dk_acc; j.dv_acc = rs->dv_acc;
    j.q_row_elems = rs->q_row_elems; j.kv_row_elems = rs->kv_row_elems;
    j.n_parts = rs->n_parts; j.check_step = rs->check_step ? 1 : 0;
    j.o_none = (uint32_t*)rs->o_none; j.lse_none = rs->lse_none; j.hq = rs->hq;
  }
  return j;
}

static ListArgs list_args(int64_t kv_row_bytes, const fcp_work_desc* work, int64_t n_work, const int32_t* cu, int32_t n_seqs, int32_t tq,
                          int32_t tkv, int32_t n_parts, bool check_step) {
  return {work, cu, (int32_t)n_work, n_seqs, tq, tkv, n_parts, max_segment_keys(kv_row_bytes), check_step};
}
static ListJob list_job(void* region, int64_t n_work, int32_t tile, int32_t inner, int64_t cap) {
  return {tile, inner, (int32_t)cap, reinterpret_cast<SchedHeader*>(region),
          reinterpret_cast<int32_t*>(static_cast<char*>(region) + sizeof(SchedHeader)), const_cast<Tile*>(sched_tiles(region, n_work))};
}

int check_row_states(int64_t n_work) {
  if (n_work > kMaxExclusiveScan)
    return fail(FCP_ERR_UNSUPPORTED, "direct mode: more than %d work items (use the plain entry point)", kMaxExclusiveScan);
  return FCP_OK;
}

int launch_row_states(int64_t kv_row_bytes, const RowStates& rs, const int32_t* q_limit, const int32_t* k_from,
                      const fcp_work_desc* work, int64_t n_work, const int32_t* cu_seqlens_kv, int32_t n_seqs,
                      int32_t tq, int32_t tkv, hipStream_t stream) {
  int rc = check_row_states(n_work);
  if (rc != FCP_OK) return rc;
  hipLaunchKernelGGL(row_state_kernel, dim3((unsigned)row_state_blocks(tq, rs.kv_state ? tkv : 0)), dim3(kSchedThreads), 0,
                     stream, make_job(&rs), list_args(kv_row_bytes, work, n_work, cu_seqlens_kv, n_seqs, tq, tkv, rs.n_parts, rs.check_step),
                     MaskTables{q_limit, k_from});
  FCP_HIP_CHECK(hipGetLastError());
  return FCP_OK;
}

int launch_schedule(bool backward, int32_t tile, int32_t inner, int64_t kv_row_bytes,
                    const int32_t* q_limit, const int32_t* k_from,
                    const fcp_work_desc* work, int64_t n_work,
                    const int32_t* cu_seqlens_kv, int32_t n_seqs, int32_t tq, int32_t tkv,
                    int32_t n_parts, int64_t tile_cap, void* region, float* lse_fill,
                    int64_t lse_fill_n, hipStream_t stream, const RowStates* states) {
  if (states) { const int rcs = check_row_states(n_work); if (rcs != FCP_OK) return rcs; }
  int fill_blocks = 0;
  if (lse_fill && lse_fill_n > 0) {
    fill_blocks = (int)((lse_fill_n + kSchedThreads * 4 - 1) / (kSchedThreads * 4));
    if (fill_blocks > 1024) fill_blocks = 1024;
    if (fill_blocks < 1) fill_blocks = 1;
  }
  const int state_blocks = states ? row_state_blocks(tq, states->kv_state ? tkv : 0) : 0;
  hipLaunchKernelGGL(sched_kernel, dim3(1 + fill_blocks + state_blocks), dim3(kSchedThreads), 0, stream,
                     backward ? 1 : 0, list_job(region, n_work, tile, inner, tile_cap),
                     list_args(kv_row_bytes, work, n_work, cu_seqlens_kv, n_seqs, tq, tkv, n_parts, lse_fill != nullptr || states != nullptr),
                     MaskTables{q_limit, k_from}, lse_fill, lse_fill_n, fill_blocks, make_job(states));
  FCP_HIP_CHECK(hipGetLastError());
  return FCP_OK;
}

int launch_schedule_bwd(int64_t kv_row_bytes, const int32_t* q_limit, const int32_t* k_from,
                        const fcp_work_desc* work, int64_t n_work, const int32_t* cu_seqlens_kv, int32_t n_seqs,
                        int32_t tq, int32_t tkv, int64_t cap_kv, void* region_kv, int32_t dq_tile, int64_t cap_q, void* region_q,
                        const float* lse, const float* delta, int64_t n_stats, float* stats, hipStream_t stream,
                        const RowStates* states, int32_t* chain, int32_t* flags, int64_t n_flags, const SplitTiles* split, bool either) {
  int64_t stat_blocks = (n_stats + kSchedThreads * 4 - 1) / (kSchedThreads * 4);
  if (stat_blocks > 1024) stat_blocks = 1024;
  if (stat_blocks < 1) stat_blocks = 1;
  const int state_blocks = states ? row_state_blocks(tq, states->kv_state ? tkv : 0) : 0;
  SplitArgs sp{};
  if (split) sp = {split->group, split->kv_units, split->q_units, dq_tile, split->n_cu, split->min_steps, split->key_turns, split->row_turns, split->blocks_per_cu, split->many_short ? 1 : 0};
  // (a kernel of its own for each mode: a longer one begins later)
  const bool cuts = split && split->cuts;
  const auto kernel = chain && either ? (cuts ? sched_bwd_kernel<kChained, kSplit> : sched_bwd_kernel<kChained, kWhole>)
                      : chain ? sched_bwd_kernel<kChained> : cuts ? sched_bwd_kernel<kSplit> : sched_bwd_kernel<kWhole>;
  hipLaunchKernelGGL(kernel, dim3((unsigned)(2 + stat_blocks + state_blocks)), dim3(kSchedThreads), 0, stream,
                     list_job(region_kv, n_work, kBwdBN, kBwdBM, cap_kv), list_job(region_q, n_work, dq_tile, kDqBN, cap_q),
                     list_args(kv_row_bytes, work, n_work, cu_seqlens_kv, n_seqs, tq, tkv, 1, false),
                     MaskTables{q_limit, k_from}, lse, delta, n_stats, stats, (int)stat_blocks, chain, flags, n_flags, sp, make_job(states));
  FCP_HIP_CHECK(hipGetLastError());
  return FCP_OK;
}

}  // namespace fcp

extern "C" size_t fcp_scratch_bytes(int which, int32_t tq, int32_t tkv, int32_t hq, int32_t hkv,
                                    int32_t head_dim, int64_t n_work, int32_t n_parts) {
  if (tq < 0 || tkv < 0 || n_work < 0 || n_parts < 0) return 0;
  if (which == FCP_SCRATCH_BWD)   // key-tile list, query-tile list, packed row statistics,
                                  // row states
    return fcp::sched_region_bytes(n_work, fcp::bwd_kv_cap(tkv, n_work)) +
           fcp::sched_region_bytes(n_work, fcp::bwd_q_cap(tq, tkv, n_work)) +
           fcp::pad_to((size_t)hq * (size_t)tq * 8, 256) +
           fcp::pad_to((size_t)tq, 256) + fcp::pad_to((size_t)tkv, 256) +  // + row states of the direct mode
           fcp::turn_bytes(tq, tkv, hq, hkv, n_work) +                     // + turns of split tiles
           fcp::chain_bytes(tq, tkv, hq, hkv, head_dim, n_work);                // + chains of the one-pass kernel
  return fcp::fwd_scratch_bytes(tq, tkv, n_work, n_parts);
}

extern "C" int fcp_scratch_status(const void* scratch, void* stream, int32_t* n_tiles, int32_t* n_rejected) {
  fcp::clear_error();
  if (!scratch) return fcp::fail(FCP_ERR_INVALID_ARG, "fcp_scratch_status: scratch is NULL");
  fcp::SchedHeader h;
  FCP_HIP_CHECK(hipMemcpyAsync(&h, scratch, sizeof(h), hipMemcpyDeviceToHost, (hipStream_t)stream));
  FCP_HIP_CHECK(hipStreamSynchronize((hipStream_t)stream));
  if (n_tiles) *n_tiles = h.n_tiles;
  if (n_rejected) *n_rejected = h.n_rejected;
  if (h.n_stalled != 0)
    return fcp::fail(FCP_ERR_STALLED, "fcp_scratch_status: %d waits for another unit's turn ran out; the rows concerned are NaN", (int)h.n_stalled);
  return FCP_OK;
}

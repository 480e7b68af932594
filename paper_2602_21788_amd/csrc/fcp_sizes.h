// Sizes and choices that follow from a call's arguments alone: room in the tile lists, the forward's form and its list (not installed).
// Plain C++, so that they can be checked without a device.
#pragma once
#include <stddef.h>
#include <stdint.h>

#include <algorithm>

#ifdef __HIPCC__
#define FCP_HD __host__ __device__
#else
#define FCP_HD
#endif

namespace fcp {

constexpr int kFwdBM = 256;      // query rows per forward unit
constexpr int kMinFwdTile = 32;  // smallest query tile of the forward (sizes its tile list; the backward's is kDqBM)
constexpr int kBwdBN = 128;      // keys per dK/dV unit
constexpr int kDqBM = 64;        // query rows per dQ unit (two heads of a KV head), twice that for a single head

constexpr size_t kSchedHeaderBytes = 128, kTileBytes = 64;
constexpr int64_t kMaxTiles = INT32_MAX / 64;   // of a list

inline size_t pad_to(size_t x, size_t a) { return (x + a - 1) / a * a; }

// Upper bounds on the number of tiles of a valid plan (anything beyond is dropped and
// counted as rejected).  Query tiles: every (row, slot) belongs to at most one item, and over
// a rank's items the query chunks of a sequence add up to at most its length.  Key tiles:
// over a rank's items the key segments of a sequence add up to at most twice its length.
inline int64_t q_tile_cap(int32_t tq, int32_t tkv, int64_t n_work, int32_t n_parts, int32_t rows) {   // rows: least rows of a tile
  const int64_t by_slots = (int64_t)n_parts * ((tq + (int64_t)rows - 1) / rows);
  const int64_t by_tokens = (tkv + (int64_t)rows - 1) / rows;
  return n_work + std::min(by_slots, by_tokens);
}
inline int64_t kv_tile_cap(int32_t tkv, int64_t n_work) {
  return 2 * n_work + 2 * (int64_t)((tkv + kBwdBN - 1) / kBwdBN);
}

// Room for the backward's lists when tiles are split (split_sizes, csrc/fcp_sched.hip).  A tile has at most two pieces more than its loop divided by the size of a
// piece.  Over all tiles that quotient is 4 per CU at most: a piece is no less than a CU's share of all steps, which counts a key tile's loop at half its
// length or more (the average of the first and the last tile), and a query tile's at a quarter (a row unit's step is half of what a CU does at a
// time); and a piece in whole steps is half of its size at least (key tiles, whose pieces are whole blocks of 32 rows for all heads of the group), 12 / 13
// of it (query tiles, by the least size).  So 2048 is enough for 472 CUs.
inline int64_t bwd_kv_cap(int32_t tkv, int64_t n_work) { return 2 * kv_tile_cap(tkv, n_work) + 2048; }
inline int64_t bwd_q_cap(int32_t tq, int32_t tkv, int64_t n_work) { return 2 * q_tile_cap(tq, tkv, n_work, 1 << 20, kDqBM) + 2048; }

// One schedule region: SchedHeader | item offsets int32[n_work+1] | Tile[cap]; every part padded to 64 bytes, the region to 256.
inline size_t sched_item_off_bytes(int64_t n_work) { return pad_to((size_t)(n_work + 1) * sizeof(int32_t), 64); }
inline size_t sched_region_bytes(int64_t n_work, int64_t cap) {
  return pad_to(kSchedHeaderBytes + sched_item_off_bytes(n_work) + (size_t)cap * kTileBytes, 256);
}

// ---- grids of the persistent kernels and the first units of their blocks ----------------
constexpr int kNumXcd = 8;

// Blocks of a launch: as many as are resident, or as there are units, and a multiple of the XCD count: block b is number b / 8 of the grid / 8 blocks
// of queue b % 8.  With 300 resident blocks a 38th block of some queues would begin with a unit that the counter deals out too.
inline int64_t persistent_blocks(int64_t resident, int64_t units) {
  const int64_t most = resident / kNumXcd * kNumXcd, wanted = (units + kNumXcd - 1) / kNumXcd * kNumXcd;
  return std::max<int64_t>(kNumXcd, std::min(most, wanted));
}

// The heads of a tile (`per_tile`: heads, or pairs of them) and the queues.  `queues` > 1, or a list whose units wait for each other (`in_turn`): every queue
// has as many heads as every other and works all tiles for them, in list order; its blocks are b = queue mod `queues`.  A unit then waits for units of its
// own queue only (the pieces of a tile for one head), which running blocks have taken before it: blocks that cannot start, because something else
// holds their CUs, hold up nobody who runs.  (A power of two: as many blocks for every queue.)  `queues` = 1 else: one numbering, which the eight counters
// deal out in turn.
FCP_HD inline int head_queues(int per_tile, bool in_turn) {
  if (per_tile % kNumXcd == 0) return kNumXcd;
  return !in_turn ? 1 : per_tile % 4 == 0 ? 4 : per_tile % 2 == 0 ? 2 : 1;
}
// Which counter a block takes numbers from, and the unit that number i is of the queue's heads: mul i + add.
struct UnitNumbers { int counter, mul, add; };
FCP_HD inline UnitNumbers unit_numbers(int block, int queues, bool in_turn) {
  if (queues > 1 || in_turn) return {block % queues, 1, 0};
  return {block % kNumXcd, kNumXcd, block % kNumXcd};
}

// Do the blocks of a queue begin with units by their numbers, instead of taking them from the queue's counter?  A launch then begins with one trip to memory
// instead of three in a row, on lines that all blocks are after.  But the first units are the longest, and one of a block that cannot start, because
// something else holds its CU, waits until a block of the launch has run dry.  So only in launches of few units per block, fewer of long ones (`longest`:
// the key rows of the longest loop, at most), where the beginning counts.  By number / by counter, us: forward, 300 sequences of 120 tokens, 8 heads (6 units per
// block) 94 / 101, 32 heads on 8 (12) 199 / 209, 412 of 149, 40 on 8 (30) 460 / 471; both lists, 36 sequences of 104, 40 on 8 of 64 channels (3) 67 / 71,
// 340 of 67, 8 on one (3) 68 / 72, 43864 tokens in 11 sequences over 8 ranks, 32 on 8 (14) equal.  While 16 of 256 CUs are held: both lists, 32768 tokens
// in 24 sequences, 32 on 8 (20) 2950 / 2700, 65536 over 4 ranks (16) 29420 / 28790; the forward's wide form there 9590 / 9030, which never begins by
// number.  Never for units that wait for each other.
constexpr int kDealForward = 32, kDealLists = 4, kDealKeys = 1024;
FCP_HD inline bool deals_first(int units, int blocks, int per_block, int longest) { return units <= (longest > kDealKeys ? 2 : per_block) * blocks; }
// When does a block ask the counter for its next unit?  With loops of some length in the unit's last step (`take`): the trip is over before the epilogue is,
// and what is left goes to whoever comes first.  Blocks that begin by number, with short loops, have it in reserve from the unit before: their
// units are too short to cover the trip, and too short for the end to become uneven.  A long unit in reserve is begun late, after the block's own long
// one.  In reserve / taken in the last step, us: forward, 35768 tokens in 53 sequences over 2 ranks, 8 heads on one 418 / 358; 42000 in 60, 6
// on 2 269 / 236; 28000 in 40 over 4 ranks, 10 on 2 200 / 191; 18000 tokens, 8 of 64 channels (by number) 413 / 398; 9 sequences of 1000, 8 heads (by
// number) 87 / 77; both lists, 18000 tokens, 8 of 64 channels 1220 / 1171.  (In reserve but for the last three units per block: 53860 tokens in 5 sequences
// over 3 ranks, 8 on one 684, where reserve 597, last step 589.)
FCP_HD inline bool keeps_reserve(bool dealt, int longest) { return dealt && longest <= kDealKeys; }

// Two lists worked by the same blocks (csrc/fcp_attn_bwd_lists.hip): what block `place` of the `places` of its queue begins with, the key units of the queue
// being `key_units`, `n_long` of them (`places` at most) longer than any row unit.  The long key units go to the first blocks, then key units and row
// units in turn, then row units.  The counters deal out the rest: key units from `key_dealt` on, row units from places - key_dealt on.
struct FirstUnit { int key_dealt, key, row; };     // (-1: none of that list)
FCP_HD inline FirstUnit first_unit(int place, int places, int key_units, int n_long) {
  const int alternate = n_long + (places - n_long + 1) / 2;
  const int key_dealt = key_units < alternate ? key_units : alternate;
  const int k = place - n_long, pairs = 2 * (key_dealt - n_long);
  if (k < 0) return {key_dealt, place, -1};
  if (k >= pairs) return {key_dealt, -1, k - pairs / 2};
  return (k & 1) ? FirstUnit{key_dealt, -1, k >> 1} : FirstUnit{key_dealt, n_long + (k >> 1), -1};
}

// ---- the forward ------------------------------------------------------------------------
// The forms of the forward.  Rows per unit (of two heads each half as many where the heads of a KV head pair up):
enum FwdForm {
  kFwdWide,      // 256 rows: eight waves in lock step, one block per CU (csrc/fcp_attn_fwd.hip, 128 channels)
  kFwdSmall,     // 128 rows: four waves, two blocks per CU (64 channels: three; csrc/fcp_attn_fwd_small.hip, as those below)
  kFwdShort,     // 128 rows: four waves, three blocks per CU (128 channels)
  kFwdSplit2,    // 64 rows: two waves share 32 rows and divide the keys
  kFwdSplit4,    // four waves do; 64 rows of eight waves with 128 channels, 32 rows of four waves and one head with 64
};
inline int fwd_unit_rows(FwdForm f, int head_dim) { return f == kFwdWide ? kFwdBM : f == kFwdSplit2 ? 64 : f == kFwdSplit4 ? (head_dim == 64 ? 32 : 64) : 128; }

// Which form works a list.  The items are in device memory; the host has their mean length and the work per CU (units of 128 rows of one head, a
// row counted once per item that covers it).  Measured, forward step with its scheduling launch, wide / the form chosen, us:
//   few units, and loops long enough to be divided: the longest unit's loop sets the time.  128 channels, 8 heads: 2000 tokens 59 / 38 (four waves
//     a row; two 44), 4096 tokens 102 / 75 (two), 4096 tokens over 3 ranks 53 / 43.  64 channels, 4 heads, undivided / divided: 512 tokens 23 / 23, 4096 68 /
//     38 (four; two 50); several sequences have a longer longest loop for the same work: 16 of 16384 tokens 72 / 57 (two).  Where units abound it is slower:
//     60000 tokens in 16 sequences, 32 heads on 8 of 128 channels 3940 / 5230.
//   64 channels otherwise: blocks of four waves, three per CU, at every size (against the wide form when it had 64 channels: 60000 tokens in 16 sequences,
//     40 heads on 8 4100 / 3760; 1000 of 128 1050 / 737).
//   128 channels: short items are mostly beginnings and ends of units, which other blocks of the CU cover: 1000 of 128, 32 heads on 8 956 / 681 (two
//     blocks per CU 718), 200 of 80000 tokens 1172 / 1071 (1157); with few units per CU two blocks with 64-key tiles do better than three with
//     32-key tiles: 4000 tokens in 8 sequences, 32 heads on 8, 62 / 62 (three: 64), 8192 tokens of 8 heads 193 / 183 (206).  Long items: the wide form (60000
//     tokens in 16 sequences 3940; 4030 with three blocks, 4180 with two).
inline FwdForm fwd_form(int head_dim, int hq, int64_t tq, int64_t tkv, int64_t n_work, int64_t n_parts, int n_cu) {
  const int64_t rows = std::min(n_parts * tq, tkv);          // of all items together, at most
  const int64_t mean = n_work > 0 ? rows / n_work : 0;
  const double per_cu = (double)rows * hq / (128. * n_cu);
  if (head_dim == 64) {
    if (mean >= 256 && (per_cu <= 0.5 || (per_cu <= 1. && mean >= 1024))) return kFwdSplit4;
    return mean >= 256 && per_cu <= (tq == tkv && n_work >= 8 ? 2.5 : 1.6) ? kFwdSplit2 : kFwdSmall;
  }
  if (mean >= 256 && per_cu <= 1.1) return per_cu <= 0.55 ? kFwdSplit4 : kFwdSplit2;
  const int64_t units = (rows / 128 + n_work) * hq;
  if (mean <= 640) return units <= 12 * (int64_t)n_cu ? kFwdSmall : kFwdShort;
  return units <= 6 * (int64_t)n_cu ? kFwdSmall : kFwdWide;
}

// The form and its list: two heads of one KV head per unit when the heads pair up (and a unit has rows for two), else twice the rows for one head.
// The list has to fit `area` bytes.  Where that of the form's tiles does not (the static work area is checked for tiles of 128 rows), units
// of 128 rows of one head take their place, whose tiles are the largest that every head layout and both widths have.
struct FwdPlan { FwdForm form; int32_t head_pair, tile; int64_t cap; };
inline FwdPlan fwd_plan(int head_dim, int hq, int hkv, int32_t tq, int32_t tkv, int64_t n_work, int32_t n_parts, int n_cu, size_t area) {
  auto with = [&](FwdForm f, bool pair) {
    const int rows = fwd_unit_rows(f, head_dim);
    const int32_t tile = pair ? rows / 2 : rows;
    return FwdPlan{f, pair ? 1 : 0, tile, q_tile_cap(tq, tkv, n_work, n_parts, tile)};
  };
  const FwdForm form = fwd_form(head_dim, hq, tq, tkv, n_work, n_parts, n_cu);
  const FwdPlan p = with(form, (hq / hkv) % 2 == 0 && fwd_unit_rows(form, head_dim) > 32);
  if (p.cap <= kMaxTiles && sched_region_bytes(n_work, p.cap) <= area) return p;
  return with(kFwdSmall, false);
}

// Blocks of the form that a CU holds.
inline int fwd_blocks_per_cu(FwdForm f, int head_dim) {
  if (head_dim == 64) return f == kFwdSplit4 ? 2 : 3;
  return f == kFwdWide || f == kFwdSplit4 ? 1 : f == kFwdShort ? 3 : 2;
}
// Does the launch do without a list?  Its blocks then have one unit each, which they find from the items themselves (one item per lane, the slots of a row in
// one word), and as many blocks as there can be units are launched: there is no scheduling launch to wait for (7 to 10 us), but a block begins with one or
// two trips to memory more, and the order of the tiles is an estimate (alone_order).  With up to 2.5 units per resident block that pays.  The two calls of the direct
// forward in a graph, with a list / without, us: 512 tokens, 4 heads of 64 channels (0.13 units per block) 16.0 / 9.3; 4096, the same heads (1.0) 33.6 / 27.9; 4096 over 3
// ranks, 8 heads (1.1) 43.7 / 37.0; 30 of 667, 6 on 2 of 64 (1.5) 41.6 / 29.2; 40 sequences of 300, the same heads (1.8) 35.3 / 24.5; 30 of 100, 32 on 8 (2.2) 29.7 / 22.6; 4096 over 8,
// 32 on 8 (2.4) 57.0 / 47.8.  Past that less, and not always: 20000 over 8 ranks, 8 heads (2.6) 133 / 129, 64 of 300, 8 heads (3.2) 53.6 / 52.3, 60 of 500, 10 on 2 of 64 (3.7)
// 57.0 / 54.6, 6 of 2000, 32 on 8 of 64 134.6 / 134.8; of 149 lists of more than 8192 tokens with 2.5 to 3 units per block 21 take more than 1 % longer without, the worst 6 %.
constexpr int kAloneItems = 64, kAloneParts = 32;
inline bool fwd_alone(FwdForm f, int head_dim, int64_t n_work, int32_t n_parts, int64_t units, int n_cu) {
  return f != kFwdWide && n_work >= 1 && n_work <= kAloneItems && n_parts <= kAloneParts && 2 * units <= 5 * (int64_t)n_cu * fwd_blocks_per_cu(f, head_dim);
}

// In which order such a launch has its tiles (alone_record in csrc/fcp_attn_fwd_small.hip).  Blocks begin in the order of their numbers, so that with more than one unit
// per CU the order decides which units share a CU and which begin late.  The two calls of the direct forward in a graph, us, with a list / by items, the one with the
// costliest last tile first, its tiles from the end on / by tiles, each by its own cost:
//   128 rows a unit: 25834 tokens, one sequence of 16481 over 2 ranks, 4 heads 184 / 226 / 177; 18232 over 2, 4 of 64 channels 141 / 172 / 135; 8642 over 2, 8 heads 108 / 127 /
//     102; 30 of 667, 6 on 2 of 64 42 / 35 / 30; 16 of 200, 32 on 8 of 64 29 / 19 / 17; but 55 of 80, 8 of 64 22.8 / 10.3 / 11.1 (the search, about 0.3 us for few items and 0.8
//     for many).  Of 1992 calls of all kinds 123 by items and 25 by tiles took more than 1 % longer than before there were launches without a list, the worst 24 and 9 %;
//   keys divided among the waves (64 and 32 rows a unit): several short units one after the other take as long as a long one, and by tiles the short ones of all items come
//     last: 2 of 1200, 8 on one of 64 23.7 / 19.9 / 22.6, 5096 over 2, 6 on 2 of 64 43.8 / 36.8 / 40.1;
//   up to a unit per CU any order does, and none has to be found.
enum AloneOrder { kInListOrder, kByItems, kByTiles };
inline AloneOrder alone_order(FwdForm f, int64_t n_work, int64_t units, int n_cu) {
  if (n_work == 1 || units <= n_cu) return kInListOrder;
  return f == kFwdSplit2 || f == kFwdSplit4 ? kByItems : kByTiles;
}

// What a call must bring: the list of the smallest tiles and the direct mode's row states; for the static area (no row states, and the plan goes by
// what fits) the list of 128-row tiles, with tq bytes to spare.
inline size_t fwd_area_bytes(int32_t tq, int32_t tkv, int64_t n_work, int32_t n_parts) {
  return sched_region_bytes(n_work, q_tile_cap(tq, tkv, n_work, n_parts, kMinFwdTile));
}
inline size_t fwd_scratch_bytes(int32_t tq, int32_t tkv, int64_t n_work, int32_t n_parts) {
  return fwd_area_bytes(tq, tkv, n_work, n_parts) + pad_to((size_t)tq, 256);
}
inline size_t fwd_static_bytes(int32_t tq, int32_t tkv, int64_t n_work, int32_t n_parts) {
  return sched_region_bytes(n_work, q_tile_cap(tq, tkv, n_work, n_parts, kFwdBM / 2)) + pad_to((size_t)tq, 256);
}

// ---- the backward -----------------------------------------------------------------------
// Does delta read dO as a stream, past the caches?  The attention kernel reads dO next.  Where the L2s (8 of 4 MB) can hold it, it is found there, and chains of short
// sequences wait for nothing longer; larger ones would not be found anyway, and push other lines out.  Delta, lists and conversion, dO streamed / not, us: 6603 tokens in
// 12 sequences, 8 heads on 8 (13.5 MB) 187 / 168, 4545 in 45, 32 on 8 (38 MB) 88 / 83; by bytes of dO, mean over calls of all kinds: 4 to 8 MB 1.003 / 0.995 of the time with
// neither O nor dO streamed, 16 to 28 0.991 / 0.993, 40 to 48 0.983 / 0.991, 64 to 96 0.974 / 0.984.
inline bool delta_streams_do(int32_t tq, int32_t hq, int32_t head_dim) { return 2 * (int64_t)tq * hq * head_dim > (int64_t)kNumXcd * 4 << 20; }
inline bool one_pass_heads(int32_t hkv, int32_t head_dim) { return head_dim == 128 && hkv % kNumXcd == 0; }

// One pass or two lists.  The one-pass kernel (csrc/fcp_attn_bwd_fused.hip) forms S and dP once and needs no query tiles; it has the
// units of key tiles only, which take turns at the dQ rows of a sequence.  That pays where sequences are short and few of them follow each
// other through the same rows: whole sequences (tq == tkv) with 256 rows or less per item, one or two heads per KV head or a tile per CU.  Scheduling and
// attention launches, one pass / two lists, us: 8 query heads on 8: 60 sequences of 130 tokens on average 54 / 58, 100 of 130 75 / 83, 30 of 190 49 / 56; 16 on 8:
// 60 of 130 67 / 75; 32 on 8: 60 of 100 74 / 79, 100 of 130 158 / 179; 40 on 8: 60 of 160 176 / 194.  With one query head per KV head, up to four tiles per
// CU, also a dozen sequences and more with a mean of 768 rows at most (as the kernels are now 9 to 12 % slower there: 12 of 6000 tokens in all 111 / 99); not
// longer ones (one of 512 tokens 37 / 33, 4096 210 / 160, 8192 518 / 466, 14400 1378 / 1301, 16384 1772 / 1616, 4 of 15000 798 / 744).
// Sharded lists (tq < tkv) have the whole sequence's tiles over a part of its rows: they stay with two lists.
// The rows per item are an average, and the items are in device memory: where one of them could be long enough to turn the comparison
// round (16384 rows with one query head per KV head, else 2048 and 512 rows of two and four heads), the scheduler decides when it sees them
// (one_pass_pays in csrc/fcp_sched.hip), and the launches of the other way end at once: 3 to 5 us, which lists of two heads per KV
// head and less than 8 K tokens on 8 KV heads are spared.
// Many short sequences, 2.5 key tiles per CU and more, go to blocks of four waves (csrc/fcp_attn_bwd_short.hip), scheduling and attention launches, twelve waves /
// four: 200 sequences of 60 tokens on average, 32 query heads on 8, 154 / 126 us, 1000 of 40 534 / 375, 1000 of 128 1419 / 1295; with fewer tiles there are
// few blocks for the chip (30 of 100, 16 on 8, 47 / 51), and with means above 192 rows most tiles are in chains, whose steps take longer there
// (400 of 256, 40 on 8, 1608 / 1590).  Below four tiles per CU that is so from smaller means on, the smaller the more heads a chain's steps have: 70 of 155, 8 on
// 8 70 / 72, 32 on 8 146 / 161, 40 on 8 177 / 203; 75 of 158, 24 on 8 144 / 156; 80 of 133, 40 on 8 173 / 200, 64 on 8 239 / 271; but 110 of 95, 40 on 8 155 / 146,
// 85 of 132, 24 on 8 132 / 122, 75 of 158, 8 on 8 77 / 72.  One long sequence sets the time there sooner (a step of its chain 2.5 us), so the scheduler always decides.
struct BwdWay { bool one_pass, many_short, either; };     // either: the scheduler decides between one pass and two lists
inline BwdWay bwd_way(int32_t hq, int32_t hkv, int32_t head_dim, int32_t tq, int32_t tkv, int64_t n_work, int n_cu) {
  const int group = hq / hkv;
  const int64_t key_units = (int64_t)tkv * hkv / kBwdBN;
  // (The kernel's queues are those of eight XCDs: not on a part of the chip.)
  const bool one_pass = one_pass_heads(hkv, head_dim) && n_work >= 1 && n_work <= 1024 && tq == tkv && n_cu == 256 &&
                        ((tkv <= 256 * n_work && (group <= 2 || key_units >= n_cu)) ||
                         (group == 1 && key_units <= 4 * n_cu && n_work >= 12 && tkv <= 768 * n_work));
  const bool many_short = one_pass && tkv <= 192 * n_work && 2 * key_units >= 5 * n_cu &&
                          (tkv <= (group <= 4 ? 144 : 112) * n_work || 4 * key_units >= (group <= 2 ? 11 : 16) * n_cu);
  const int64_t longest_item = (int64_t)tkv - n_work + 1;      // (with a row at least in each of the others)
  const bool either = many_short || (one_pass && group * longest_item > (group == 1 ? 16384 : group == 2 ? 4096 : 2048) && (group > 2 || key_units >= 2 * n_cu));
  return {one_pass, many_short, either};
}

}  // namespace fcp

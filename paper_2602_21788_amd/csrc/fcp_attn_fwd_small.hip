// The forward's forms for short documents, small problems and 64 channels per head: blocks of four waves, two or three blocks per CU.
//
// Same function as fwd_kernel (csrc/fcp_attn_fwd.hip).  There a CU works on one unit at a time, eight waves in lock step: the best form for a
// long row of key tiles of 128 channels, but whatever the unit waits for at its two ends (record, first tiles and Q rows on their way in, O
// rows on their way out) the whole CU waits for, and a unit of 256 rows x heads is a serial loop over all their keys while most
// of the chip may have no unit at all.  Here
//   * a block has one wave per SIMD and two LDS stages: several blocks share a CU without any lock step, one's beginning and end meet the others'
//     matrix work, and so do one's exponentials.  64 channels: three blocks of 140 registers (four, with two of them spilled, are as
//     fast).  128 channels: two with 64-key stages, or three of 168 registers with 32-key stages, which is what the LDS holds;
//   * a unit = 64 rows x two query heads of one KV head (even number of heads per KV head) or 128 rows of one head; every wave owns 32 rows, all
//     share the stages, one barrier per stage: scores, softmax and P V of a stage in turn (the fragments requested AH matrix instructions ahead;
//     all at once is slower with three blocks, the compiler's own order with two);
//   * SPLIT = 2, 4: groups of SPLIT waves own the same 32 rows and divide the keys of every stage among them, 32 keys each; their
//     (maximum, sum, O) meet in LDS at the unit's end.  Half (a quarter) of the rows per unit, half (a quarter) of the serial loop, for problems
//     that would otherwise leave CUs without a unit.  A stage's fills then serve fewer matrix instructions, so it does not pay where units
//     abound (60000 tokens in 16 sequences, 32 heads on 8: 4180 -> 5230 us with two).
//   * small launches have no list (fwd_alone in csrc/fcp_sizes.h): a block finds its unit from the work items, and further blocks do what else the
//     scheduling launch does (row states, empty slots, the header's counts).  No block waits for another one.
// Priorities as in fwd_kernel (matrix stream first) gain 1 % on long items and lose 1 to 3 % elsewhere; none are set.
// Times of the forms beside each other and where each is taken: fwd_form in csrc/fcp_sizes.h.
#include "fcp_fwd.h"

namespace fcp {
namespace {

template <int D, int NW, int SPLIT, int SKEYS>
struct SmallCfg {
  static constexpr int NWAVE = NW;
  static constexpr int RG = NWAVE / SPLIT;        // groups of 32 rows (of one or two heads)
  static constexpr int SK = SKEYS;                // keys per stage
  static constexpr int NB = SK / 32 / SPLIT;      // 32-key blocks of a stage per wave
  using KT = RowTile<D>;
  using VT = TrTile<D>;
  using QT = DualTile<D>;
  static constexpr int KBYTES = KT::bytes(SK);
  static constexpr int STAGE = KBYTES + VT::bytes(SK);
  static constexpr int max_of(int a, int b) { return a > b ? a : b; }
  static constexpr int LDS_BYTES = max_of(max_of(2 * STAGE, STAGE + NWAVE * QT::bytes(32)), SPLIT > 1 ? NWAVE * 32 * D * 4 : NWAVE * RowStage<D>::BYTES);
  static constexpr int RPW = SK / NWAVE;          // tile rows each wave fills
  static constexpr int IPT = RPW / KT::RPI;       // fill instructions per wave, stage and tensor
  static constexpr int NKF = D == 128 || IPT == 1 ? 1 : 2;    // distinct lane offsets of K fills (the row permutation of D = 64 has a period of 16 rows)
  static constexpr int NKA = D == 128 ? 2 : 4;    // distinct per-lane K read addresses
  static constexpr int NVA = D / 32;              // distinct per-lane V^T read addresses
  static constexpr int NS = D / 16;               // MFMAs of one 32 x 32 score block
  static constexpr int KB_STRIDE = KT::row_base(32);
  static constexpr int PARTS = SPLIT < NVA ? SPLIT : NVA;   // waves of a group that combine, each NVA / PARTS channel blocks
  static_assert(RPW % KT::RPI == 0 && KT::row_base(RPW * 3 + KT::RPI) == KT::row_base(RPW * 3) + KT::row_base(KT::RPI), "a wave's rows start on a padding group boundary");
};

// ---- launches without a list (fwd_alone): one item per lane -------------------------------
typedef i32x4 __attribute__((may_alias)) i32x4_any;    // (the rows' lists lie in the stages)
static_assert(kAloneItems == 64 && kAloneParts == 32, "a lane per item, a bit per slot");
__device__ inline Item lane_item(const FwdParams& p, int lane) {
  Item it{-1, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0};
  if (lane < p.list.n_work) it = load_item(p.list, MaskTables{p.q_limit, nullptr}, lane);
  return it;
}
// Tiles of the lane's item that the launch works.  It has blocks for tile_cap tiles; of a list with more of them, in the order of the list, the rest is dropped and
// counted as rejected, as in a list.  `ahead`: tiles of the items that the list has before this one.
__device__ inline int32_t alone_tiles(const FwdParams& p, int32_t tiles, int32_t ahead) { return min(tiles, max(p.tile_cap - ahead, 0)); }
// The block's record, of the launch's tile `number`.  Where more than one unit comes to a CU the tiles stand in the order of what they cost, so that the longest units
// begin first and are spread over the CUs, and short ones lie beside them (AloneOrder in csrc/fcp_sizes.h, with times).  The order has to be every block's own and to need
// no list: the costs of an item's tiles are taken as a line from its first tile (its rows' own positions, also under a mask) to its last, which tells how many of them cost
// C or more.  A lane counts these for a C of its own over all items (the waves share long lists): the greatest C with more than `number` such tiles has the tile, among those
// of that cost in the order of the items.
// Every thread calls it; the answer (is there such a tile?) is wave 0's.
constexpr int kShareItems = 8;
template <int NW>
__device__ inline bool alone_record(const FwdParams& p, int number, float (*s_sums)[64], int32_t* s_rec) {
  const int lane = lane_id(), wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
  const int waves = p.order != kInListOrder && p.list.n_work > kShareItems ? NW : 1;
  if (wave >= waves) return true;
  const Item it = lane_item(p, lane);
  int32_t tiles = it.seq >= 0 ? ceil_div(it.q_len, p.tile) : 0;
  const int32_t upto = wave_prefix_sum(tiles), ahead = upto - tiles;
  if (number >= min(__builtin_amdgcn_readlane(upto, 63), p.tile_cap)) return false;
  tiles = alone_tiles(p, tiles, ahead);
  int32_t place = number - ahead, here = tiles, above = 0;    // the item's tiles from its end on: those in front, those among which `place` is
  if (p.order != kInListOrder) {
    const int32_t last = ceil_div(it.vis0, kFwdBN) + ceil_div(it.vis1, kFwdBN);
    const int64_t limit = (int64_t)it.q_pos + p.tile - 1;
    const int32_t first = ceil_div(seen_keys(it, 0, limit), kFwdBN) + (it.n1 > 0 ? ceil_div(seen_keys(it, 1, limit), kFwdBN) : 0);
    const bool rises = p.order == kByTiles && tiles > 1 && last > first;
    const float n = (float)tiles, from = (float)(rises ? first : last), per_step = rises ? (n - 1.f) / (float)(last - first) : n;
    // (C = 0: all of the item.  Past its last tile's cost: none.  A segment has 2^23 keys at most, max_segment_keys, so costs are below 2^19 and their differences exact, and
    // the product's rounding, 2^-23 of n at most, is less than per_step.)
    auto count = [](float c, float n, float from, float per_step) {
      return __builtin_amdgcn_fmed3f(n - __builtin_ceilf((c - from) * per_step), 0.f, n);
    };
    const float step = (float)(wave_max(last) / 64 + 1);
    float sum = 0.f;
#pragma unroll 4
    for (int i = wave; i < p.list.n_work; i += waves) {
      auto of = [&](float v) { return __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int32_t, v), i)); };
      sum += count((float)lane * step, of(n), of(from), of(per_step));
    }
    if (waves > 1) {
      s_sums[wave][lane] = sum;
      __syncthreads();
      if (wave != 0) return true;
#pragma unroll
      for (int w = 1; w < NW; ++w) sum += s_sums[w][lane];
    }
    const float c = (float)(__builtin_popcountll(__builtin_amdgcn_ballot_w64(sum > (float)number)) - 1) * step;
    above = (int32_t)count(c + step, n, from, per_step);
    here = (int32_t)count(c, n, from, per_step) - above;
    place = number - __builtin_amdgcn_readlane(wave_prefix_sum(above), 63) - (wave_prefix_sum(here) - here);
  }
  const uint64_t mine = __builtin_amdgcn_ballot_w64(place >= 0 && place < here);
  if (mine == 0) return false;                      // (does not occur: one lane has the place)
  const int at = __builtin_ctzll(mine);
  int32_t tile = tiles - 1 - above - place;
  tile = __builtin_amdgcn_readlane(tile, at);
  auto of = [&](int32_t v) { return __builtin_amdgcn_readlane(v, at); };
  const Item u{0, of(it.q_off), of(it.q_len), of(it.q_pos), of(it.k0), of(it.n0), of(it.k1), of(it.n1), of(it.base), 0, 0, of(it.step)};
  const bool shared = __builtin_amdgcn_ballot_w64(lane != at && it.seq >= 0 && it.q_off < u.q_off + u.q_len && u.q_off < it.q_off + it.q_len) != 0;
  const int32_t r0 = tile * p.tile;
  const int32_t rows = min(p.tile, u.q_len - r0);
  const int64_t limit = MaskTables{p.q_limit, nullptr}.limit(u, r0 + rows - 1);
  if (lane == 0) {
    const int32_t w[12] = {u.q_off + r0, u.q_pos + r0, rows, u.step, u.base + u.k0, u.n1 > 0 ? u.base + u.k1 : 0, u.k0, u.k1,
                           seen_keys(u, 0, limit), u.n1 > 0 ? seen_keys(u, 1, limit) : 0, shared ? 0 : kFlagQExclusive, 0};
#pragma unroll
    for (int i = 0; i < 12; ++i) s_rec[i] = w[i];
  }
  return true;
}
// What the scheduling launch does beside the list: the rows' states (direct mode), -inf in the partial slots of rows that no item covers there, O = 0 and
// LSE = -inf of rows without an item where no merge follows, and the counts of the header.  A row per thread.
template <int D>
__device__ inline void alone_rows(const FwdParams& p, i32x4_any* s_lists) {
  const int lane = lane_id(), n_work = p.list.n_work;
  s_lists += 64 * (threadIdx.x >> 6);
  const Item it = lane_item(p, lane);
  const int block = (int)blockIdx.x - p.unit_blocks;
  const int32_t tiles = it.seq >= 0 ? ceil_div(it.q_len, p.tile) : 0;
  const int32_t upto = wave_prefix_sum(tiles);
  if (block == 0 && threadIdx.x < 64) {
    const int32_t n_tiles = __builtin_amdgcn_readlane(upto, 63);
    const int n_bad = __builtin_popcountll(__builtin_amdgcn_ballot_w64(lane < n_work && it.seq < 0));
    if (lane == 0) {
      SchedHeader h{};
      h.n_tiles = min(n_tiles, p.tile_cap);
      h.n_rejected = n_bad + max(n_tiles - p.tile_cap, 0);
      h.path = kPathNoList;
      *p.hdr = h;
    }
  }
  if (p.running) return;
  const int32_t row = block * (int)blockDim.x + (int)threadIdx.x;
  const int32_t len = it.seq >= 0 ? it.q_len : 0;
  int32_t shared = 0, hits = 0, lost = 0;
  uint32_t slots = 0;
  s_lists[lane] = i32x4{it.q_off, len, it.step & 31, 0};
  wave_exchange();
#pragma unroll 4
  for (int j = 0; j < n_work; ++j) {
    const i32x4 o = s_lists[j];
    shared |= j != lane && o[1] > 0 && it.q_off < o[0] + o[1] && o[0] < it.q_off + len;
  }
  wave_exchange();
  // (rows of dropped tiles are like rows that the item does not have)
  s_lists[lane] = i32x4{it.q_off, min(len, alone_tiles(p, tiles, upto - tiles) * p.tile), it.step & 31, shared};
  wave_exchange();
#pragma unroll 4
  for (int j = 0; j < n_work; ++j) {
    const i32x4 o = s_lists[j];
    const bool hit = (uint32_t)(row - o[0]) < (uint32_t)o[1];
    hits += hit;
    lost |= hit ? o[3] : 0;
    slots |= hit ? 1u << o[2] : 0;
  }
  if (row >= p.tq) return;
  const int state = hits == 0 ? 0 : p.direct > 1 || (hits == 1 && !lost) ? 2 : 1;
  if (p.direct) p.q_state[row] = (uint8_t)state;
  if (p.direct > 1) {
    if (state != 0) return;
    u32x4* const o = reinterpret_cast<u32x4*>(p.o_out + (int64_t)row * p.hq * D);
    for (int e = 0; e < p.hq * D / 8; ++e) o[e] = u32x4{0, 0, 0, 0};
    for (int h = 0; h < p.hq; ++h) p.lse_out[(int64_t)h * p.tq + row] = -INFINITY;
  } else if (!p.direct || state != 2) {            // (the slots of a row that has its result are not read)
    for (int s = 0; s < p.list.n_parts; ++s) {
      if (slots >> s & 1) continue;
      for (int h = 0; h < p.hq; ++h) p.lse_part[((int64_t)s * p.hq + h) * p.tq + row] = -INFINITY;
    }
  }
}

template <int D, int NW, int SPLIT, int SKEYS, int OCC, int AH>
__global__ __launch_bounds__(64 * NW, OCC) void fwd_small_kernel(const FwdParams p) {
  using C = SmallCfg<D, NW, SPLIT, SKEYS>;
  using KT = typename C::KT;
  using VT = typename C::VT;
  using QT = typename C::QT;
  extern __shared__ __attribute__((aligned(256))) unsigned char smem[];
  __shared__ int32_t s_next_unit;
  __shared__ int32_t s_rec[16];
  __shared__ __attribute__((aligned(16))) float s_rowf[C::NWAVE][32];   // per wave: one factor per query row
  __shared__ __attribute__((aligned(16))) float s_rowl[C::NWAVE][32];   // SPLIT > 1: ... and its share of the row sum

  const int tid = threadIdx.x;
  const int lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int share = wave % SPLIT;                 // which 32 (or 64) keys of a stage
  const int group = wave / SPLIT;
  const int l32 = lane & 31, g2 = lane >> 5;
  const int G = p.hq / p.hkv;
  const uint32_t lds0 = lds_offset(smem);

  // unit numbering as in fwd_kernel: each XCD owns a contiguous eighth of the heads where they split evenly
  const int hpu = p.head_pair ? 2 : 1;
  const bool per_xcd = (p.hq % (kNumXcd * hpu)) == 0;
  const int xcd = per_xcd ? (int)(blockIdx.x % kNumXcd) : 0;
  const int heads_here = per_xcd ? p.hq / kNumXcd : p.hq;
  const int units_per_tile = heads_here / hpu;
  UnitQueue uq;
  if (p.unit_blocks > 0) {
    if ((int)blockIdx.x >= p.unit_blocks) return alone_rows<D>(p, reinterpret_cast<i32x4_any*>(smem));
    const int place = per_xcd ? blockIdx.x / kNumXcd : blockIdx.x;
    const bool found = alone_record<NW>(p, place / units_per_tile, reinterpret_cast<float (*)[64]>(smem), s_rec);
    uq.init_alone(units_per_tile, place % units_per_tile, found, &s_next_unit);
  } else {
    uq.init_dealt(p.hdr, p.tiles, xcd, units_per_tile, per_xcd ? blockIdx.x / kNumXcd : blockIdx.x, per_xcd ? gridDim.x / kNumXcd : gridDim.x, p.tile_cap,
                  &s_next_unit, s_rec);
  }

  const int kv_row_bytes = p.hkv * D * 2;
  int kfill[C::NKF];
#pragma unroll
  for (int i = 0; i < C::NKF; ++i) kfill[i] = fill_voff<KT>(C::RPW, wave, i, lane, kv_row_bytes) - i * KT::RPI * kv_row_bytes;
  const int vfill = fill_voff<VT>(C::RPW, wave, 0, lane, kv_row_bytes);
  // fragment addresses as in fwd_kernel, from the wave's first key block of a stage on
  int kaddr[C::NKA];
#pragma unroll
  for (int j = 0; j < C::NKA; ++j) kaddr[j] = tile_off<KT>(l32, 2 * j + g2) + (SPLIT > 1 ? share * C::KB_STRIDE : 0);
  int vaddr[C::NVA];
  {
    const int row0 = 4 * g2 + ((lane & 15) >> 2);
    const int chunk0 = 2 * ((lane >> 4) & 1) + ((lane & 3) >> 1);
#pragma unroll
    for (int db = 0; db < C::NVA; ++db)
      vaddr[db] = C::KBYTES + tile_off<VT>(row0, 4 * db + chunk0) + 8 * (lane & 1) + (SPLIT > 1 ? share * VT::row_base(32) : 0);
  }

  for (;;) {
    const int unit = uq.current(&s_next_unit);
    if (unit >= uq.n_units) break;
    const QTile t = read_record<QTile, 12>(s_rec);
    const int second = p.head_pair && C::RG > 1 ? group / (C::RG / 2 > 0 ? C::RG / 2 : 1) : 0;
    const int head = xcd * heads_here + (unit % units_per_tile) * hpu + second;
    const int kvh = head / G;

    const int wave_r0 = 32 * (p.head_pair ? group % (C::RG / 2 > 0 ? C::RG / 2 : 1) : group);
    const bool wave_active = wave_r0 < t.rows;
    const int my_row = wave_r0 + l32;
    const bool row_valid = my_row < t.rows;
    const int row_ld = min(my_row, t.rows - 1);
    // last key position the lane's row sees, and the least and greatest such limit among the wave's rows
    int q_lim = t.q_pos0 + my_row;
    int wave_first_lim = t.q_pos0 + wave_r0;
    int wave_last_lim = t.q_pos0 + min(wave_r0 + 31, t.rows - 1);
    if (p.q_limit) {
      const int32_t* ql = p.q_limit + t.q_row0;
      q_lim = ql[row_ld];
      wave_first_lim = __builtin_amdgcn_readfirstlane(ql[min(wave_r0, t.rows - 1)]);
      wave_last_lim = __builtin_amdgcn_readfirstlane(ql[min(wave_r0 + 31, t.rows - 1)]);
      __builtin_amdgcn_s_waitcnt(kWaitVm0);
    }
    // the two segments' fields as scalars (indexed with a run-time segment number the record would land in scratch memory)
    const int vis0 = t.vis[0], vis1 = t.vis[1], kpos0 = t.k_pos0[0], kpos1 = t.k_pos0[1];
    const int nt0 = (vis0 + C::SK - 1) / C::SK, nt1 = (vis1 + C::SK - 1) / C::SK;
    const int n_iter = nt0 + nt1;

    // ---- fills: as in fwd_kernel, stage by stage in list order
    i32x4 f_rk, f_rv;
    auto f_resources = [&](int64_t row0, int vis) {
      const int64_t off = (row0 * p.hkv + kvh) * D;
      const int bytes = vis > 0 ? (vis - 1) * kv_row_bytes + D * 2 : 0;
      f_rk = buffer_rsrc(p.k + off, bytes);
      f_rv = buffer_rsrc(p.v + off, bytes);
    };
    f_resources(t.kv_row0[0], vis0);
    int f_left = nt0, f_soff = 0;
    bool f_seg0 = true;
    uint32_t f_dst = 0;
    const uint32_t f_k = lds0 + KT::row_base(C::RPW * wave), f_v = lds0 + C::KBYTES + VT::row_base(C::RPW * wave);
    auto fill_next = [&]() {
      if (f_seg0 && f_left == 0) { f_resources(t.kv_row0[1], vis1); f_seg0 = false; f_soff = 0; }
#pragma unroll
      for (int i = 0; i < C::IPT; ++i) {
        const int so = f_soff + i * KT::RPI * kv_row_bytes;
        lds_fill_b128(f_rk, f_k + f_dst + KT::row_base(KT::RPI * i), kfill[i % C::NKF], so);
        lds_fill_b128(f_rv, f_v + f_dst + VT::row_base(VT::RPI * i), vfill, so);
      }
      --f_left;
      f_soff += C::SK * kv_row_bytes;
      f_dst = C::STAGE - f_dst;
    };

    // Prologue: the first stage and the wave's Q rows (whole rows through the second stage, which the first fill of the loop takes over
    // after the barrier that ends the reads here).
    if (n_iter > 0) fill_next();
    bf16x8 qf[C::NS];
    {
      int lane_p = lane;                            // addresses formed here, not ahead of the unit loop (registers)
      asm volatile("" : "+v"(lane_p));
      const int q_row_bytes = p.hq * D * 2;
      const int n_wave_rows = t.rows - wave_r0;
      const i32x4 rq = buffer_rsrc(p.q + ((int64_t)(t.q_row0 + wave_r0) * p.hq + head) * D,
                                   n_wave_rows > 0 ? (min(n_wave_rows, 32) - 1) * q_row_bytes + D * 2 : 0);
      const int area = C::STAGE + wave * QT::bytes(32);
#pragma unroll
      for (int i = 0; i < 32 / QT::RPI; ++i)
        lds_fill_b128(rq, lds0 + area + QT::row_base(QT::RPI * i), fill_voff<QT>(32, 0, i, lane_p, q_row_bytes), 0);
      __builtin_amdgcn_s_waitcnt(kWaitVm0);
#pragma unroll
      for (int ks = 0; ks < C::NS; ++ks)
        qf[ks] = *reinterpret_cast<const bf16x8*>(smem + area + tile_off<QT>(lane_p & 31, 2 * ks + (lane_p >> 5)));
      __builtin_amdgcn_s_waitcnt(0xC07F);           // lgkmcnt(0): in registers before anybody fills the second stage
    }
    f32x16 oacc[C::NVA];
#pragma unroll
    for (int db = 0; db < C::NVA; ++db) oacc[db] = zero16();
    float m_run = -INFINITY;   // running maximum in log2 units (score * scale_log2)
    float l_run = 0.f;         // this lane's share of the running sum
    const int slot = p.running ? 0 : t.step;
    if (p.running && share == 0) {                  // the caller's merged result is one more block of keys, see fwd_kernel
      const float lse_prev = p.lse_part[(int64_t)head * p.tq + t.q_row0 + row_ld];
      const int row_bytes = fresh_uniform(p.hq * D * 4);   // (the rows' offsets are formed here, not ahead of the unit loop)
      const int n_wave_rows = t.rows - wave_r0;
      const __amdgpu_buffer_rsrc_t ri = __builtin_amdgcn_make_buffer_rsrc(
          (void*)(p.o_part + ((int64_t)(t.q_row0 + wave_r0) * p.hq + head) * D), (short)0,
          n_wave_rows > 0 ? (n_wave_rows - 1) * row_bytes + D * 4 : 0, 0x00020000);
      const int o_voff = 4 * g2 * row_bytes + 4 * l32;
#pragma unroll
      for (int db = 0; db < C::NVA; ++db)
#pragma unroll
        for (int i = 0; i < 16; ++i)
          oacc[db][i] = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(
              ri, o_voff, (8 * (i / 4) + (i % 4)) * row_bytes + 128 * db, 0));
      const bool has_prev = lse_prev > -INFINITY;
      if (has_prev) {
        m_run = lse_prev * kLog2e;
        l_run = g2 == 0 ? 1.f : 0.f;
      }
      __builtin_amdgcn_s_waitcnt(kWaitVm0);
      s_rowf[wave][l32] = has_prev ? 1.f : 0.f;
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const f32x4 a = *reinterpret_cast<const f32x4*>(&s_rowf[wave][8 * j + 4 * g2]);
#pragma unroll
        for (int db = 0; db < C::NVA; ++db)
#pragma unroll
          for (int e = 0; e < 4; ++e) oacc[db][4 * j + e] = a[e] != 0.f ? oacc[db][4 * j + e] : 0.f;
      }
    }
    auto scale_rows = [&](float f) {                // see fwd_kernel
      s_rowf[wave][l32] = f;
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const f32x4 a = *reinterpret_cast<const f32x4*>(&s_rowf[wave][8 * j + 4 * g2]);
#pragma unroll
        for (int db = 0; db < C::NVA; ++db)
#pragma unroll
          for (int e = 0; e < 4; ++e) oacc[db][4 * j + e] *= a[e];
      }
    };

    // ---- the unit: per stage one barrier, then scores, softmax and P V of the wave's keys.  At the barrier the wave's part of the stage has
    // landed; the other stage was last read before it.
    for (int it = 0; it < n_iter; ++it) {
      __builtin_amdgcn_s_waitcnt(kWaitVm0);
      __syncthreads();
      if (__builtin_expect(it + 1 < n_iter, 1)) fill_next(); else uq.take(wave);
      const bool seg1 = it >= nt0;
      const int k0 = (it - (seg1 ? nt0 : 0)) * C::SK + (SPLIT > 1 ? 32 * share : 0);    // the wave's first key of the segment
      const int k_pos = (seg1 ? kpos1 : kpos0) + k0;
      const int n_valid = (seg1 ? vis1 : vis0) - k0;
      if (!wave_active || n_valid <= 0 || k_pos > wave_last_lim) continue;
      const unsigned char* const stage = smem + (it & 1) * C::STAGE;
      constexpr int kAhead = AH;
      f32x16 sacc[C::NB];
      {
        constexpr int N = C::NB * C::NS;
        bf16x8 fr[N];
        auto request = [&](int f) {
          if (f >= N) return;
          const int kb = f / C::NS, ks = f % C::NS;
          fr[f] = *reinterpret_cast<const bf16x8*>(stage + kaddr[ks % C::NKA] + (ks / C::NKA) * (C::NKA * 32) + kb * C::KB_STRIDE);
        };
#pragma unroll
        for (int x = 0; x < kAhead; ++x) request(x);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int x = 0; x < N; ++x) {
          sacc[x / C::NS] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fr[x], qf[x % C::NS], x % C::NS == 0 ? zero16() : sacc[x / C::NS], 0, 0, 0);
          request(x + kAhead);
          __builtin_amdgcn_sched_barrier(0);
        }
      }
      constexpr int NV = 2 * C::NB * C::NVA;
      bf16x8 vf[NV];
      auto v_request = [&](int f) {
        if (f >= NV) return;
        const int tt = f / C::NVA, db = f % C::NVA;
        vf[f] = tr_read_8(stage + vaddr[db] + tt * (16 * VT::row_base(1)), 8 * VT::row_base(1));
      };
#pragma unroll
      for (int x = 0; x < kAhead; ++x) v_request(x);
      // mask, lazy running maximum, exponentials, row sum, conversion: see fwd_kernel
      if (k_pos + 32 * C::NB - 1 > wave_first_lim || n_valid < 32 * C::NB) {
        const int lim = min(n_valid, q_lim - k_pos + 1) - 4 * g2;
#pragma unroll
        for (int kb = 0; kb < C::NB; ++kb)
#pragma unroll
          for (int i = 0; i < 16; ++i)
            if (32 * kb + 8 * (i / 4) + (i % 4) >= lim) sacc[kb][i] = -INFINITY;
      }
      float mx = max3(sacc[0][0], sacc[0][1], sacc[C::NB - 1][0]);
#pragma unroll
      for (int kb = 0; kb < C::NB; ++kb)
#pragma unroll
        for (int i = kb == 0 ? 2 : 0; i < 16; i += 2) mx = max3(mx, sacc[kb][i], sacc[kb][i + 1]);
      mx = lane32_partner_max(mx) * p.scale_log2;
      if (__builtin_amdgcn_ballot_w64(mx > m_run + kRescaleThreshold) != 0) {
        const float m_new = fmaxf(m_run, mx);
        const float alpha = __builtin_amdgcn_exp2f(m_run - (m_new == -INFINITY ? 0.f : m_new));
        m_run = m_new;
        l_run *= alpha;
        scale_rows(alpha);
      }
      const float m_use = m_run == -INFINITY ? 0.f : m_run;
      float psum = 0.f;
      bf16x8 pf[2 * C::NB];
#pragma unroll
      for (int e = 0; e < 16 * C::NB; e += 2) {
        const float e0 = __builtin_amdgcn_exp2f(fmaf(sacc[e / 16][e % 16], p.scale_log2, -m_use));
        const float e1 = __builtin_amdgcn_exp2f(fmaf(sacc[e / 16][e % 16 + 1], p.scale_log2, -m_use));
        psum += e0;
        psum += e1;
        pf[e / 8][e % 8] = (__bf16)e0;
        pf[e / 8][e % 8 + 1] = (__bf16)e1;
      }
      l_run += psum;
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int x = 0; x < NV; ++x) {
        oacc[x % C::NVA] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(pf[x / C::NVA], vf[x], oacc[x % C::NVA], 0, 0, 0);
        v_request(x + kAhead);
        __builtin_amdgcn_sched_barrier(0);
      }
    }
    __syncthreads();                                // the stages are free
    if (n_iter == 0) uq.take(wave);
    uq.prefetch();                                  // ahead of the epilogue's stores, see fwd_kernel

    // ---- epilogue
    float l_tot = lane32_partner_sum(l_run);
    if constexpr (SPLIT > 1) {
      // The group's waves leave (maximum, sum, O) in LDS, lane by lane in the accumulator layout; wave `share` of PARTS combines its channel blocks.
      s_rowf[wave][l32] = m_run;
      s_rowl[wave][l32] = l_tot;
      unsigned char* const mine = smem + wave * (32 * D * 4);
#pragma unroll
      for (int db = 0; db < C::NVA; ++db)
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          f32x4 v;
#pragma unroll
          for (int e = 0; e < 4; ++e) v[e] = oacc[db][4 * j + e];
          *reinterpret_cast<f32x4*>(mine + (db * 4 + j) * 1024 + lane * 16) = v;
        }
      __syncthreads();
      const int w0 = group * SPLIT;
      auto at = [&](const float (*a)[32], int w, int j) { return *reinterpret_cast<const f32x4*>(&a[w0 + w][8 * j + 4 * g2]); };
      m_run = s_rowf[w0][l32];
#pragma unroll
      for (int w = 1; w < SPLIT; ++w) m_run = fmaxf(m_run, s_rowf[w0 + w][l32]);
      l_tot = 0.f;
#pragma unroll
      for (int w = 0; w < SPLIT; ++w) l_tot += s_rowl[w0 + w][l32] * __builtin_amdgcn_exp2f(s_rowf[w0 + w][l32] - (m_run == -INFINITY ? 0.f : m_run));
      constexpr int NO = C::NVA / C::PARTS;         // channel blocks per combining wave: db = share * NO + o
      f32x16 out[NO];
#pragma unroll
      for (int j = 0; j < 4; ++j) {                 // four rows at a time, see scale_rows
        f32x4 m4 = at(s_rowf, 0, j), f4[SPLIT], l4 = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int w = 1; w < SPLIT; ++w)
#pragma unroll
          for (int e = 0; e < 4; ++e) m4[e] = fmaxf(m4[e], at(s_rowf, w, j)[e]);
#pragma unroll
        for (int w = 0; w < SPLIT; ++w)
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            f4[w][e] = __builtin_amdgcn_exp2f(at(s_rowf, w, j)[e] - (m4[e] == -INFINITY ? 0.f : m4[e]));
            l4[e] += f4[w][e] * at(s_rowl, w, j)[e];
          }
#pragma unroll
        for (int e = 0; e < 4; ++e) l4[e] = l4[e] > 0.f ? 1.f / l4[e] : 0.f;
#pragma unroll
        for (int o = 0; o < NO; ++o) {
          f32x4 acc = {0.f, 0.f, 0.f, 0.f};
          const int db = (share < C::PARTS ? share : 0) * NO + o;
#pragma unroll
          for (int w = 0; w < SPLIT; ++w) {
            const f32x4 v = *reinterpret_cast<const f32x4*>(smem + (w0 + w) * (32 * D * 4) + (db * 4 + j) * 1024 + lane * 16);
#pragma unroll
            for (int e = 0; e < 4; ++e) acc[e] += f4[w][e] * v[e];
          }
#pragma unroll
          for (int e = 0; e < 4; ++e) out[o][4 * j + e] = acc[e] * l4[e];
        }
      }
#pragma unroll
      for (int o = 0; o < NO; ++o) oacc[o] = out[o];
    } else {
      scale_rows(l_tot > 0.f ? 1.f / l_tot : 0.f);
    }
    // Direct mode: the tile's rows get all their keys in this unit, so the normalised O is the final one.
    const bool direct = p.direct > 1 || (p.direct && (t.flags & kFlagQExclusive) != 0);
    int lane_e = lane;                              // see RowStage::flush
    asm volatile("" : "+v"(lane_e));
    const int l32e = lane_e & 31, g2e = lane_e >> 5;
    const int n_wave_rows = t.rows - wave_r0;
    auto rows_of = [&](void* base, int row_bytes, int elem_bytes) {   // the wave's rows, ending with the tile's last
      return __builtin_amdgcn_make_buffer_rsrc(base, (short)0, n_wave_rows > 0 ? (n_wave_rows - 1) * row_bytes + D * elem_bytes : 0, 0x00020000);
    };
    float* const po = p.o_part + (int64_t)slot * ((int64_t)p.tq * p.hq * D) + ((int64_t)(t.q_row0 + wave_r0) * p.hq + head) * D;
    uint16_t* const pb = p.o_out + ((int64_t)(t.q_row0 + wave_r0) * p.hq + head) * D;
    if constexpr (SPLIT > 1) {
      // (a wave has 32 or 64 channels of every row here: stored straight from the registers)
      if (share < C::PARTS) {
        constexpr int NO = C::NVA / C::PARTS;
        if (!direct) {
          const int row_bytes = fresh_uniform(p.hq * D * 4);
          const __amdgpu_buffer_rsrc_t ro = rows_of(po, row_bytes, 4);
#pragma unroll
          for (int o = 0; o < NO; ++o)
#pragma unroll
            for (int i = 0; i < 16; ++i)
              __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(unsigned, (float)oacc[o][i]), ro, 4 * g2e * row_bytes + 4 * l32e,
                                                    (8 * (i / 4) + (i % 4)) * row_bytes + 128 * (share * NO + o), 0);
        }
        if (p.o_out && (p.running || direct)) {
          const int row_bytes = fresh_uniform(p.hq * D * 2);
          const __amdgpu_buffer_rsrc_t rb = rows_of(pb, row_bytes, 2);
#pragma unroll
          for (int o = 0; o < NO; ++o)
#pragma unroll
            for (int i = 0; i < 16; ++i)
              __builtin_amdgcn_raw_buffer_store_b16(__builtin_bit_cast(short, (__bf16)oacc[o][i]), rb, 4 * g2e * row_bytes + 2 * l32e,
                                                    (8 * (i / 4) + (i % 4)) * row_bytes + 64 * (share * NO + o), 0);
        }
      }
    } else {
      using OUT = RowStage<D>;
      unsigned char* const obuf = smem + wave * OUT::BYTES;
      if (!direct) {                                  // partial O, fp32: D / 2 channels per pass
        const int row_bytes = fresh_uniform(p.hq * D * 4);
        const __amdgpu_buffer_rsrc_t ro = rows_of(po, row_bytes, 4);
#pragma unroll
        for (int h = 0; h < 2; ++h) {
#pragma unroll
          for (int db = 0; db < D / 64; ++db)
#pragma unroll
            for (int i = 0; i < 16; ++i)
              OUT::put_f32(obuf, OUT::reg_row(i, g2e), 32 * db + l32e, oacc[h * (D / 64) + db][i]);
          OUT::flush(obuf, lane_e, ro, row_bytes, h * D * 2);
        }
      }
      if (p.o_out && (p.running || direct)) {         // the final rows as bf16
        const int row_bytes = fresh_uniform(p.hq * D * 2);
        const __amdgpu_buffer_rsrc_t rb = rows_of(pb, row_bytes, 2);
#pragma unroll
        for (int db = 0; db < D / 32; ++db)
#pragma unroll
          for (int i = 0; i < 16; ++i) OUT::put_bf16(obuf, OUT::reg_row(i, g2e), 32 * db + l32e, oacc[db][i]);
        OUT::template flush<true>(obuf, lane_e, rb, row_bytes, 0);
      }
    }
    if (row_valid && g2 == 0 && share == 0) {
      const float lse = l_tot > 0.f ? (m_run + __builtin_amdgcn_logf(l_tot)) * kLn2 : -INFINITY;
      float* dst = direct ? p.lse_out : p.lse_part + (int64_t)slot * ((int64_t)p.hq * p.tq);
      dst[(int64_t)head * p.tq + t.q_row0 + my_row] = lse;
    }
    uq.advance(&s_next_unit, s_rec);   // barrier: the LDS stages are free for the next unit's fills
  }
}

template <int D, int NW, int SPLIT, int SKEYS, int OCC, int AH>
int launch_one(FwdParams p, int64_t units, bool alone, int n_cu, hipStream_t stream) {
  using C = SmallCfg<D, NW, SPLIT, SKEYS>;
  static std::atomic<uint64_t> lds_done;
  const auto kernel = fwd_small_kernel<D, NW, SPLIT, SKEYS, OCC, AH>;
  const int rc = raise_lds_limit((const void*)kernel, C::LDS_BYTES, lds_done);
  if (rc != FCP_OK) return rc;
  int64_t blocks = persistent_blocks((int64_t)n_cu * (OCC * 4 / NW), units);
  p.unit_blocks = alone ? (int32_t)units : 0;
  if (alone) blocks = units + (p.running ? 1 : (p.tq + 64 * NW - 1) / (64 * NW));
  hipLaunchKernelGGL(kernel, dim3((unsigned)blocks), dim3(64 * NW), C::LDS_BYTES, stream, p);
  FCP_HIP_CHECK(hipGetLastError());
  return FCP_OK;
}

}  // namespace

int launch_fwd_small(FwdParams p, int head_dim, FwdForm form, int64_t units, bool alone, int n_cu, hipStream_t stream) {
  p.order = alone_order(form, p.list.n_work, units, n_cu);
  if (head_dim == 64)
    return form == kFwdSplit4   ? launch_one<64, 4, 4, 128, 2, 4>(p, units, alone, n_cu, stream)
           : form == kFwdSplit2 ? launch_one<64, 4, 2, 64, 3, 4>(p, units, alone, n_cu, stream)
                                : launch_one<64, 4, 1, 64, 3, 4>(p, units, alone, n_cu, stream);
  return form == kFwdSplit4   ? launch_one<128, 8, 4, 128, 2, 4>(p, units, alone, n_cu, stream)
         : form == kFwdSplit2 ? launch_one<128, 4, 2, 64, 2, 4>(p, units, alone, n_cu, stream)
         : form == kFwdSmall  ? launch_one<128, 4, 1, 64, 2, 4>(p, units, alone, n_cu, stream)
                              : launch_one<128, 4, 1, 32, 3, 3>(p, units, alone, n_cu, stream);
}

}  // namespace fcp

// dQ, dK and dV in one pass over key tiles by blocks of four waves, two per CU: the backward kernel of lists of many short sequences with 128
// channels per head.
//
// The function, the chain of tiles that adds up dQ through the L2 of one XCD, and the queues are those of csrc/fcp_attn_bwd_fused.hip, whose head
// explains them.  That kernel is one block of twelve waves per CU in lock step: a step costs little where one chain sets the time, but a unit's beginning and
// end (its K and V rows, three iterations of the pipeline) stand still as long as five steps, and a short sequence has four.  Here a wave does everything
// for 32 keys as in the key units of csrc/fcp_attn_bwd_lists.hip (S, dP, P, dS, dV and dK in its registers), leaves dS in LDS, and after a barrier forms the
// step's dQ for 32 channels of all 32 rows from the dS of all waves: two barriers per step, and while one block of the CU waits the other works.
//   * 253 registers (dV and dK 128, V fragments 32) and 75 KB of LDS (two stages of Q and dO, the K rows, which S reads as rows and dQ transposed, dS);
//   * dQ^T as [channel x query]: a lane has four consecutive channels of a query in four registers, exchanged with the other half of the wave
//     to stores of 16 bytes; the final rows of a sequence of one tile go straight to bf16;
//   * the flag of a chain's step is set most of a step later, when its stores have arrived anyway.
//   * a store or load takes about a clock for every line it touches, however little of it: the final rows leave 64 bytes of a row at a time, and a sum on its way
//     from one tile to the next lies where an instruction's lines are whole, not where row and channel belong (scheduling and one-pass launch, us, before / now: 1000
//     sequences of 128 on average, 32 query heads on 8 KV heads 1247 / 1210, 8 heads 504 / 464, 1000 of 60 482 / 465, 120 of 150 235 / 219).
// What bounds it: memory.  1000 sequences of 128 tokens, 32 query heads on 8 KV heads, are 4.2 GB of Q, dO, dQ, K, V, dK and dV: 0.89 ms with the scheduling launch
// (4.7 TB/s, what a large copy reaches, by count), 64 tokens each 0.45 ms; the twelve-wave kernel 1.01 and 0.64.  Sequences of two tiles move a part of dQ as fp32 and
// read Q and dO again: 1000 of 128 on average 1.42 -> 1.21 ms (5.2 GB by the counters; 8 heads 667 -> 464 us), 1000 of 40 534 -> 376 us (8 heads 318 -> 206).
// Where one chain sets the time a step takes 2.5 us against 1.5: the rule is bwd_way in csrc/fcp_sizes.h.
// Tried: the sums of earlier tiles requested before the barrier (a chain's step 2.5 -> 2.2 us, but many short sequences 2 % slower: the extra loads
// are issued for every step); fragments two or four instructions ahead, no priority for the matrix stream: equal.
#include "fcp_bwd.h"

namespace fcp {
namespace {

template <int D>
struct ShortCfg {
  static constexpr int NWAVE = 4;
  static constexpr int BM = kBwdBM;                // 32 query rows per step
  static constexpr int BN = kBwdBN;                // 128 keys per unit, 32 per wave
  using DT = DualTile<D>;
  static constexpr int TILE = DT::bytes(BM);       // one Q or dO block
  static constexpr int SLOT = 256;                 // one statistics plane of a step: 64 floats (32 used)
  static constexpr int STAGE = 2 * TILE + 2 * SLOT;
  static constexpr int KOFF = 2 * STAGE;           // the unit's K rows
  static constexpr int XGROUP = 32 * 32 * 2;       // dS of one key group, bf16
  static constexpr int XOFF = KOFF + DT::bytes(BN);
  static constexpr int max_of(int a, int b) { return a > b ? a : b; }
  static constexpr int LDS_BYTES = max_of(XOFF + NWAVE * XGROUP, NWAVE * RowStage<D>::BYTES);
  static constexpr int NS = D / 16;                // MFMAs of one 32 x 32 block of S or dP
  static constexpr int NVA = D / 32;               // 32-channel blocks of dK, dV
  static constexpr int IPT = BM / DT::RPI / 2;     // fill instructions per wave and step: waves 0, 1 fill Q, waves 2, 3 dO
  static_assert(D == 128, "four 32-channel slices of dQ, one per wave");
  static_assert(2 * STAGE >= DT::bytes(BN), "the V tile passes through the stages at the start of a unit");
  static_assert(STAGE % 256 == 0 && TILE % 256 == 0 && XOFF % 256 == 0, "the address permutations stay below bit 8");
  static_assert(LDS_BYTES <= 80 * 1024 - 256, "two blocks per CU");
};

__device__ inline void lds_barrier() { asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory"); }
template <int N>
__device__ inline void wait_vmem() { asm volatile("s_waitcnt vmcnt(%0)" :: "n"(N) : "memory"); }

constexpr int kCacheBypass = 16;   // sc1: the load goes past the CU's vector cache, which may hold what the line was when this CU last read it
constexpr int kClaimed = 1 << 30;      // counter of a claimed queue: past every unit; the claiming XCD from bit kClaimShift on (home blocks count below it)
constexpr int kClaimShift = 24;
constexpr int kClaimPolls = 16;
constexpr int kSpinLimit = 1 << 18;    // polls of a wave per unit, about half a second: a chain that cannot go on ends, its rows become NaN and the
                                       // header says so
// what eight rows further change in a chunk's place, besides the row itself
template <int D> constexpr int kTr8 = (DualTile<D>::key(0) ^ DualTile<D>::key(8)) << 4;
constexpr int kShortAhead = 3;         // LDS fragments are requested this many matrix instructions ahead

template <int D>
__global__ __launch_bounds__(256, 2) void bwd_short_kernel(const BwdParams p) {
  using C = ShortCfg<D>;
  using DT = typename C::DT;
  extern __shared__ __attribute__((aligned(256))) unsigned char smem[];
  __shared__ int32_t s_next_unit;
  __shared__ int32_t s_queue[2];                   // queue that units are taken from; this block's XCD
  __shared__ int32_t s_rec[20];                    // tile record, then chain record

  if (p.either && !(p.hdr->path & kPathOnePass)) return;
  const int lane = lane_id(), wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int l32 = lane & 31, g2 = lane >> 5;
  const int G = p.hq / p.hkv;
  const uint32_t lds0 = lds_offset(smem);
  // the queue of the XCD this block really runs on
  if (threadIdx.x == 0) s_queue[0] = s_queue[1] = __builtin_amdgcn_s_getreg(20 | (0 << 6) | (3 << 11)) & (kNumXcd - 1);   // HW_REG_XCC_ID, bits 3:0
  const int kvh_here = p.hkv / kNumXcd;
  const int n_units = p.hdr->n_tiles * kvh_here;

  // Units are taken one at a time, two steps before the block needs one: a unit that a block holds in reserve
  // holds up the units after it in its chains.
  int32_t pend = 0, recw = 0;
  auto take = [&]() {
    const int home = __builtin_amdgcn_readfirstlane(s_queue[1]), q = __builtin_amdgcn_readfirstlane(s_queue[0]);
    if (lane_id() == 0) pend = atomicAdd(q == home ? &p.hdr->counter[q] : &p.hdr->claimed[q], 1);
  };
  auto fetch = [&](int unit) {
    const int l = lane_id();
    if (unit < n_units) {
      const int64_t tile = unit / kvh_here;
      if (l < 16) recw = reinterpret_cast<const int32_t*>(p.tiles)[tile * 16 + l];
      else if (l < 20) recw = p.chain[tile * kChainWords + l - 16];
    }
  };
  auto publish = [&](int unit) {
    const int l = lane_id();
    if (l < 20) s_rec[l] = recw;
    if (l == 0) s_next_unit = unit;
  };
  // Blocks are dealt to the XCDs in turn, so every queue has its blocks.  An XCD that has begun nothing while a block of another one
  // has run out of units is late (its CUs are held by something else) or got no block: after a few polls (about 30 us) its
  // queue is claimed as a whole for the XCD of that block, and all blocks of that XCD which run out work it off together.  None of them
  // leaves before the last claim: a block leaves when every queue is begun.
  auto take_elsewhere = [&](int unit) {
    if (unit < n_units || n_units == 0) return;
    const int home = __builtin_amdgcn_readfirstlane(s_queue[1]);
    const int l = lane_id();
    for (int polls = 0;; ++polls) {
      int32_t c = 1;
      if (l < kNumXcd) c = __hip_atomic_load(&p.hdr->counter[l], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      uint64_t ours = __builtin_amdgcn_ballot_w64(c >= kClaimed && (c - kClaimed) >> kClaimShift == home);
      const uint64_t idle = __builtin_amdgcn_ballot_w64(c == 0);
      if (idle && polls >= kClaimPolls) {
        const int q = __builtin_ctzll(idle);
        int32_t old = 0;
        if (l == 0) old = atomicCAS(&p.hdr->counter[q], 0, kClaimed + (home << kClaimShift));
        if (__builtin_amdgcn_readfirstlane(old) == 0) ours |= (uint64_t)1 << q;
      }
      for (; ours && unit >= n_units; ours &= ours - 1) {
        const int q = __builtin_ctzll(ours);
        int32_t v = 0;
        if (l == 0) v = atomicAdd(&p.hdr->claimed[q], 1);
        unit = __builtin_amdgcn_readfirstlane(v);
        if (l == 0) s_queue[0] = q;
      }
      if (unit < n_units || !idle) break;
      __builtin_amdgcn_s_sleep(32);
    }
    fetch(unit);
    publish(unit);
  };
  if (wave == 0) {
    take();
    const int unit = __builtin_amdgcn_readfirstlane(pend);
    fetch(unit);
    publish(unit);
    take_elsewhere(unit);
  }
  lds_barrier();

  const int q_row_bytes = p.hq * D * 2, dq_row_bytes = p.hq * D * 4;
  const int kv_row_bytes = p.hkv * D * 2;
  const bool fill_is_do = wave >= 2;
  const int fill_row0 = 16 * (wave & 1);
  // fill instruction i covers rows fill_row0 + RPI i + lane / CPR: its chunk permutation is that of i = 0 with key(RPI i) on top
  const int tfill = (fill_row0 + lane / DT::CPR) * q_row_bytes + (((lane % DT::CPR) ^ DT::key(lane / DT::CPR)) << 4);
  const int row0 = tile_off<DT>(l32, g2);          // row fragment ks (row l32, channels 16 ks + 8 g2 ..) at row0 ^ (ks << 5)
  // Transposed fragments (one channel per lane; k-slots = rows 16 t + {4 g2 + [0,4), 8 + 4 g2 + [0,4)}): channel block db of the first four rows
  // at tr0 ^ (db << 6), of the four rows eight further at that ^ kTr8, eight rows on
  const int tr0 = tile_off<DT>(4 * g2 + ((lane & 15) >> 2), 2 * ((lane >> 4) & 1) + ((lane & 3) >> 1)) + 8 * (lane & 1);
  // dS of a key group: 16 bytes per (key, g2) and half t of the rows = rows 16 t + 4 g2 + [0,4) and 16 t + 8 + 4 g2 + [0,4).  The key is permuted by 8 g2 + 4 t,
  // so that the transposed reads of four keys x 32 rows fall into different banks.
  const int ds_put = (lane * 16) ^ (g2 << 7);       // half t at (ds_put ^ (t << 6)) + t * 1024
  // read with the query on the lane, k-slots = keys 16 x + {4 g2 + [0,4), 8 + 4 g2 + [0,4)}: the keys eight further at ^ 128, sixteen further at + 256
  const int ds_get = C::XOFF + ((lane >> 4) & 1) * 1024 + (lane & 1) * 512 +
                     (((4 * g2 + ((lane & 15) >> 2)) ^ (8 * (lane & 1) + 4 * ((lane >> 4) & 1))) << 4) + ((lane & 3) >> 1) * 8;

  for (;;) {
    const int unit = __builtin_amdgcn_readfirstlane(s_next_unit);
    if (unit >= n_units) break;
    const KTile t = read_record<KTile, 15>(s_rec);
    // place in the chain (-1: atomics), first block that a later tile reaches, first flag block, first query block
    const int rank = __builtin_amdgcn_readfirstlane(s_rec[16]), qb_next = __builtin_amdgcn_readfirstlane(s_rec[17]);
    const int flag_base = __builtin_amdgcn_readfirstlane(s_rec[18]), qb0 = __builtin_amdgcn_readfirstlane(s_rec[19]);
    const int kvh = __builtin_amdgcn_readfirstlane(s_queue[0]) * kvh_here + unit % kvh_here;
    const bool exclusive = (t.flags & kFlagSeg0Exclusive) != 0;
    const bool direct = exclusive && p.dk_out != nullptr;
    const int n_keys = t.n_keys;
    const int my_key = 32 * wave + l32;
    const int64_t kv_row0 = t.kv_row0;
    const int nqb = (t.q_len + C::BM - 1) / C::BM - qb0;
    const int n_iter = nqb * G;

    // ---- fills: step s = (query head s / nqb of the KV head, query block qb0 + nqb - 1 - s % nqb), strictly in order.  Rows past the item's
    // last row lie outside the resources' range and arrive as zeros.
    const int q_bytes = (t.q_len - 1) * q_row_bytes + D * 2;
    const int64_t plane = (int64_t)p.hq * p.tq;
    const int f_row0 = (qb0 + nqb - 1) * C::BM;
    int f_head = kvh * G, f_left = nqb;
    int f_soff = f_row0 * q_row_bytes, f_ssoff = f_row0 * 4;
    i32x4 f_rt, f_rst;
    auto f_resources = [&]() {
      f_rt = buffer_rsrc((fill_is_do ? p.d_o : p.q) + ((int64_t)t.q_local_off * p.hq + f_head) * D, q_bytes);
      f_rst = buffer_rsrc(p.stats + (wave & 1) * plane + (int64_t)f_head * p.tq + t.q_local_off, t.q_len * 4);
    };
    f_resources();
    uint32_t f_dst = 0;
    auto fill_next = [&]() {
      if (f_left == 0) {
        ++f_head;
        f_left = nqb;
        f_soff = f_row0 * q_row_bytes;
        f_ssoff = f_row0 * 4;
        f_resources();
      }
      const int tf = fresh(tfill);
#pragma unroll
      for (int i = 0; i < C::IPT; ++i)
        lds_fill_b128(f_rt, lds0 + f_dst + (fill_is_do ? C::TILE : 0) + DT::row_base(fill_row0 + DT::RPI * i), tf ^ (DT::key(DT::RPI * i) << 4),
                      f_soff + i * DT::RPI * q_row_bytes);
      if (wave < 2) lds_fill_b32(f_rst, lds0 + f_dst + 2 * C::TILE + wave * C::SLOT, fresh(lane) * 4, f_ssoff);
      --f_left;
      f_soff -= C::BM * q_row_bytes;
      f_ssoff -= C::BM * 4;
      f_dst = C::STAGE - f_dst;
    };

    // ---- the wave's K rows, and its V rows through the stages into registers.  Keys past the tile's last arrive as zeros.
    int my_key_from = t.k_pos0 + my_key;            // position of the first query that sees the lane's key
    if (p.k_from) my_key_from = p.k_from[kv_row0 + min(my_key, n_keys - 1)];
    bf16x8 vf[C::NS];
    {
      const int lane_p = fresh(lane);
      const int bytes = (n_keys - 1) * kv_row_bytes + D * 2;
      const int64_t base = (kv_row0 * p.hkv + kvh) * D;
      auto fill_rows = [&](const uint16_t* src, int area) {
        const i32x4 r = buffer_rsrc(src + base, bytes);
#pragma unroll
        for (int i = 0; i < 32 / DT::RPI; ++i)
          lds_fill_b128(r, lds0 + area + DT::row_base(32 * wave + DT::RPI * i), fill_voff<DT>(32, wave, i, lane_p, kv_row_bytes), 0);
      };
      fill_rows(p.v, 0);
      fill_rows(p.k, C::KOFF);
      wait_vmem<0>();
      const int r32 = DT::row_base(32) * wave + fresh(row0);
#pragma unroll
      for (int ks = 0; ks < C::NS; ++ks) vf[ks] = *reinterpret_cast<const bf16x8*>(smem + (r32 ^ (ks << 5)));
      lds_barrier();                                // the stages are free, the K tile is whole
    }
    my_key_from = (my_key < n_keys ? my_key_from : 1 << 29) - 4 * g2;   // masked: rows (minus 4 g2) below it
    fill_next();

    // a key group takes part in the blocks from j_act on and needs no mask from j_unmasked on (blocks from qb0)
    auto pick = [](const int32_t (&a)[4], int grp) { return grp == 0 ? a[0] : grp == 1 ? a[1] : grp == 2 ? a[2] : a[3]; };
    int j_actg[4];
#pragma unroll
    for (int g = 0; g < 4; ++g) {
      const int ta = t.from_first[g] - t.q_seq_start;
      j_actg[g] = (32 * g >= n_keys || ta > t.q_len - 1) ? nqb : max(0, (max(ta, 0) >> 5) - qb0);
    }
    const int j_act = pick(j_actg, wave);
    const int j_all = max(max(j_actg[0], j_actg[1]), max(j_actg[2], j_actg[3]));
    const int j_unmasked = 32 * wave + 32 > n_keys ? nqb : max(0, ((max(pick(t.from_last, wave) - t.q_seq_start, 0) + 31) >> 5) - qb0);
    // dV, dK [32-channel block] as [key x channel]: the channel is on the lane, register i is key 8 (i/4) + 4 g2 + i%4 of the wave's 32.  The keys are reached
    // through a buffer resource that ends with the tile's last key (reads past it give zero, writes are dropped).
    f32x16 dv[C::NVA], dk[C::NVA];
    const int n_wave_keys = n_keys - 32 * wave;
    const int64_t out0 = ((kv_row0 + 32 * wave) * p.hkv + kvh) * D;
    auto rsrc = [&](void* base, int row_bytes, int bytes) {
      return __builtin_amdgcn_make_buffer_rsrc(base, (short)0, n_wave_keys > 0 ? (min(n_wave_keys, 32) - 1) * row_bytes + D * bytes : 0, 0x00020000);
    };
#pragma unroll
    for (int db = 0; db < C::NVA; ++db) dv[db] = dk[db] = zero16();
    if (exclusive && !direct) {                     // start from the caller's values
      const int row_bytes = fresh_uniform(p.hkv * D * 4);
      const __amdgpu_buffer_rsrc_t rv = rsrc(p.dv + out0, row_bytes, 4), rk = rsrc(p.dk + out0, row_bytes, 4);
      const float inv = 1.f / p.scale;
#pragma unroll
      for (int db = 0; db < C::NVA; ++db)
#pragma unroll
        for (int i = 0; i < 16; ++i) {
          const int so = (8 * (i / 4) + (i % 4)) * row_bytes + 128 * db;
          dv[db][i] = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(rv, 4 * g2 * row_bytes + 4 * l32, so, 0));
          dk[db][i] = inv * __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(rk, 4 * g2 * row_bytes + 4 * l32, so, 0));
        }
    }

    // ---- dQ of a step: the wave's 32 channels of all 32 rows, the query on the lane.  One resource per unit, ending with the item's last row (rows
    // past it read as zero and are not written); a step's place in it is a scalar offset.
    const bool chained = rank >= 0, dq_direct = chained && p.dq_out != nullptr;
    const bool loads = chained && (rank > 0 || !dq_direct);
    const int64_t dq0 = ((int64_t)t.q_local_off * p.hq + kvh * G) * D + 32 * wave;
    const uint32_t dq_bytes = (uint32_t)(t.q_len - 1) * (uint32_t)dq_row_bytes + (G - 1) * D * 4 + 128;
    const __amdgpu_buffer_rsrc_t rq = __builtin_amdgcn_make_buffer_rsrc((void*)(p.dq + dq0), (short)0, (int)dq_bytes, 0x00020000);
    const __amdgpu_buffer_rsrc_t rf = __builtin_amdgcn_make_buffer_rsrc((void*)(p.flags + ((int64_t)flag_base * p.hq + kvh * G) * kChainSlices + wave),
                                                                       (short)0, 1 << 30, 0x00020000);
    const int blk = C::BM * dq_row_bytes, fblk = p.hq * kChainSlices * 4;   // a block further, in dQ and in the flags
    int so = (qb0 + nqb - 1) * blk, fo = (qb0 + nqb - 1) * fblk, fo_done = -1;   // (fo_done: flag of the step before, still to be set)
    int spin_left = kSpinLimit;
    const int it_take = max(n_iter - 2, 0);

    int j = nqb - 1, at0 = 0;
    for (int it = 0; it < n_iter; ++it) {
      // This step's rows have landed; of the instructions after their fill the final stores of dQ (two) or its atomics (sixteen) may still be under way, the
      // stores of sums that a later tile reads may not.
      if (it == 0) wait_vmem<0>();
      else if (fo_done >= 0) wait_vmem<4>();
      else if (chained) wait_vmem<2>();
      else wait_vmem<16>();
      lds_barrier();
      int seen = rank;
      if (rank > 0) seen = __builtin_amdgcn_raw_buffer_load_b32(rf, 0, fo, kCacheBypass);
      if (it + 1 < n_iter) fill_next();
      if (wave == 0 && it == it_take) take();

      f32x16 dq;
      if (j >= j_act) {
        const float* const stat = reinterpret_cast<const float*>(smem + at0 + 2 * C::TILE) + 4 * g2;
        f32x16 s, dp;
#pragma unroll
        for (int q = 0; q < 4; ++q) {               // the accumulator starts at -delta of its rows
          const f32x4 nd = *reinterpret_cast<const f32x4*>(stat + C::SLOT / 4 + 8 * q);
#pragma unroll
          for (int e = 0; e < 4; ++e) dp[4 * q + e] = nd[e];
        }
        // The step's 4 NS matrix instructions are one stream: the fragments of instruction k are requested A instructions ahead, across the borders
        // of S, dP, dV and dK.
        constexpr int NS = C::NS, A = kShortAhead;
        static_assert(2 * C::NVA == NS, "as many instructions in each of the four parts");
        int xr[NS], ta[C::NVA];
        const int k_at = C::KOFF + DT::row_base(32) * wave - at0;
        {
          const int r = fresh(row0);
#pragma unroll
          for (int ks = 0; ks < NS; ++ks) xr[ks] = (r ^ (ks << 5)) + at0;
        }
        bf16x8 fa[4 * NS], fb[NS];
        auto tr = [&](int tile, int x) {
          const unsigned char* b0 = smem + tile + (x / C::NVA) * (16 * DT::row_base(1));
          return tr_read_8(b0 + ta[x % C::NVA], b0 + 8 * DT::row_base(1) + (ta[x % C::NVA] ^ kTr8<D>));
        };
        auto request = [&](int k) {
          if (k < NS) {
            fa[k] = *reinterpret_cast<const bf16x8*>(smem + xr[k]);
            fb[k] = *reinterpret_cast<const bf16x8*>(smem + xr[k] + k_at);
          }
          else if (k < 2 * NS) fa[k] = *reinterpret_cast<const bf16x8*>(smem + xr[k - NS] + C::TILE);
          else if (k < 3 * NS) fa[k] = tr(C::TILE, k - 2 * NS);
          else if (k < 4 * NS) fa[k] = tr(0, k - 3 * NS);
        };
#pragma unroll
        for (int k = 0; k < A; ++k) request(k);
        __builtin_amdgcn_s_setprio(1);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int x = 0; x < NS; ++x) {              // S
          s = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fa[x], fb[x], x == 0 ? zero16() : s, 0, 0, 0);
          request(x + A);
          __builtin_amdgcn_sched_barrier(0);
        }
        {
          const int r = fresh(tr0);
#pragma unroll
          for (int db = 0; db < C::NVA; ++db) ta[db] = (r ^ (db << 6)) + at0;
        }
        bf16x8 pb[2], dsb[2];
        f32x4 nl[4];
        // element i of a 16-element part belongs to instruction x of a part's NS, from the second on
        auto first_of = [](int x) { return x < 1 ? 0 : 16 * (x - 1) / (C::NS - 1); };
#pragma unroll
        for (int x = 0; x < NS; ++x) {              // dP with P in its shadow
          dp = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fa[NS + x], vf[x], dp, 0, 0, 0);
          request(NS + x + A);
          if (x == 0) nl[0] = *reinterpret_cast<const f32x4*>(stat);
#pragma unroll
          for (int i = first_of(x); i < first_of(x + 1); ++i) {
            if (i % 4 == 0 && i < 12) nl[i / 4 + 1] = *reinterpret_cast<const f32x4*>(stat + 2 * i + 8);
            s[i] = __builtin_amdgcn_exp2f(fmaf(s[i], p.scale_log2, nl[i / 4][i % 4]));
          }
          __builtin_amdgcn_sched_barrier(0);
        }
        // The masked variants: the causal edge and the keys past the tile's last (always masked).  Rows past the item's last need no mask:
        // their dO and statistics arrive as zeros, so P = 1 meets zeros in dV and dS.  A masked pair is selected away, not multiplied by zero:
        // a row must not see what a key after it holds, an infinity or a NaN included.
        if (j < j_unmasked) {
          int lo = my_key_from - (t.q_seq_start + (qb0 + j) * C::BM);
          asm volatile("; masked variant" : "+v"(lo));
#pragma unroll
          for (int i = 0; i < 16; ++i) s[i] = 8 * (i / 4) + (i % 4) < lo ? 0.f : s[i];
#pragma unroll
          for (int i = 0; i < 16; ++i) dp[i] = 8 * (i / 4) + (i % 4) < lo ? 0.f : dp[i];
        }
#pragma unroll
        for (int i = 0; i < 16; ++i) pb[i / 8][i % 8] = (__bf16)s[i];
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int x = 0; x < NS; ++x) {              // dV with dS in its shadow
          dv[x % C::NVA] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(pb[x / C::NVA], fa[2 * NS + x], dv[x % C::NVA], 0, 0, 0);
          request(2 * NS + x + A);
#pragma unroll
          for (int i = first_of(x); i < first_of(x + 1); ++i) dsb[i / 8][i % 8] = (__bf16)(s[i] * dp[i]);
          __builtin_amdgcn_sched_barrier(0);
        }
        {
          const int dl = fresh(ds_put) + (C::XOFF + C::XGROUP * wave);
#pragma unroll
          for (int q = 0; q < 2; ++q) *reinterpret_cast<bf16x8*>(smem + (dl ^ (q << 6)) + q * 1024) = dsb[q];
        }
#pragma unroll
        for (int x = 0; x < NS; ++x) {              // dK
          dk[x % C::NVA] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(dsb[x / C::NVA], fa[3 * NS + x], dk[x % C::NVA], 0, 0, 0);
          request(3 * NS + x + A);
          __builtin_amdgcn_sched_barrier(0);
        }
        __builtin_amdgcn_s_setprio(0);
      }
      if (fo_done >= 0) {
        wait_vmem<0>();
        __builtin_amdgcn_raw_buffer_store_b32((unsigned)(rank + 1), rf, fresh(lane) == 0 ? 0 : 1 << 30, fo_done, 0);
        fo_done = -1;
      }
      lds_barrier();                                // dS of the key groups is there
      {
        const int kt = C::KOFF + (fresh(tr0) ^ (wave << 6)), dg = fresh(ds_get);
        auto kt_frag = [&](int x) {
          const unsigned char* b = smem + x * 16 * DT::row_base(1);
          return tr_read_8(b + kt, b + 8 * DT::row_base(1) + (kt ^ kTr8<D>));
        };
        auto ds_frag = [&](int x) {
          const unsigned char* b = smem + (x >> 1) * C::XGROUP + (x & 1) * 256;
          return tr_read_8(b + dg, b + (dg ^ 128));
        };
        if (j < j_all) {                            // (causal edge: a group that the block does not see is left out, its keys may hold anything)
          dq = zero16();
#pragma unroll
          for (int g = 0; g < 4; ++g)
            if (j >= j_actg[g]) {
#pragma unroll
              for (int h = 0; h < 2; ++h) dq = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kt_frag(2 * g + h), ds_frag(2 * g + h), dq, 0, 0, 0);
            }
        } else {
          constexpr int NX = C::BN / 16, A = kShortAhead;
          bf16x8 fk[NX], fd[NX];
#pragma unroll
          for (int x = 0; x < A; ++x) { fk[x] = kt_frag(x); fd[x] = ds_frag(x); }
          __builtin_amdgcn_sched_barrier(0);
#pragma unroll
          for (int x = 0; x < NX; ++x) {
            dq = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fk[x], fd[x], x == 0 ? zero16() : dq, 0, 0, 0);
            if (x + A < NX) { fk[x + A] = kt_frag(x + A); fd[x + A] = ds_frag(x + A); }
            __builtin_amdgcn_sched_barrier(0);
          }
        }
      }
      // dq[4 q + e] is channel 8 q + 4 g2 + e of the lane's query
      const int l = fresh(lane);
      if (loads) {
        while (__builtin_amdgcn_readfirstlane(seen) != rank && spin_left > 0) {
          __builtin_amdgcn_s_sleep(1);
          seen = __builtin_amdgcn_raw_buffer_load_b32(rf, 0, fo, kCacheBypass);
          --spin_left;
        }
        asm volatile("" ::: "memory");              // (what the block holds is read after that)
      }
      const float dq_mul = spin_left > 0 ? p.scale : NAN;            // (see kSpinLimit)
      const int dq_voff = (l & 31) * dq_row_bytes + 16 * (l >> 5);
      // Sums on their way from one tile to the next lie where an instruction's lines are whole: 16 bytes per lane of eight rows x 128 bytes.  In their own
      // places they lie where they come from and go to the caller, and in a last block of less than 32 rows.
      const bool whole = 32 * (qb0 + j + 1) <= t.q_len, get_lines = whole && rank > 0, put_lines = whole && qb0 + j >= qb_next;
      const int lines = (l >> 3) * dq_row_bytes + 16 * (l & 7);
      if (loads) {
        f32x4 v[4];
        const int at = get_lines ? lines : dq_voff, step = get_lines ? 8 * dq_row_bytes : 32;
#pragma unroll
        for (int q = 0; q < 4; ++q) v[q] = __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(rq, at, so + q * step, kCacheBypass));
        if (get_lines != put_lines) wait_vmem<0>(); // (all of it is read before any of it is written)
#pragma unroll
        for (int q = 0; q < 4; ++q)
#pragma unroll
          for (int e = 0; e < 4; ++e) dq[4 * q + e] = fmaf(dq[4 * q + e], dq_mul, v[q][e]);
      } else {
#pragma unroll
        for (int i = 0; i < 16; ++i) dq[i] *= dq_mul;
      }
      if (dq_direct && qb0 + j < qb_next) {         // no later tile reaches the block: the final rows
        const __amdgpu_buffer_rsrc_t rb = __builtin_amdgcn_make_buffer_rsrc((void*)(p.dq_out + dq0), (short)0, (int)(dq_bytes / 2), 0x00020000);
        u32x2 w[4];
#pragma unroll
        for (int q = 0; q < 4; ++q)
          w[q] = __builtin_bit_cast(u32x2, bf16x4{(__bf16)dq[4 * q], (__bf16)dq[4 * q + 1], (__bf16)dq[4 * q + 2], (__bf16)dq[4 * q + 3]});
        u32x4 x[2];
#pragma unroll
        for (int q = 0; q < 2; ++q) {               // lanes below 32 end up with channels 8 q .. 8 q + 7, the others with 16 + 8 q ..
          const auto a = __builtin_amdgcn_permlane32_swap(w[q][0], w[q + 2][0], false, false);
          const auto b = __builtin_amdgcn_permlane32_swap(w[q][1], w[q + 2][1], false, false);
          x[q] = u32x4{(uint32_t)a[0], (uint32_t)b[0], (uint32_t)a[1], (uint32_t)b[1]};
        }
#pragma unroll
        for (int e = 0; e < 4; ++e) {               // x[0]: all 32 channels of the first sixteen rows, x[1]: of the others (64 bytes of a row an instruction, not twice 16)
          const auto a = __builtin_amdgcn_permlane16_swap(x[0][e], x[1][e], false, false);
          x[0][e] = (uint32_t)a[0];
          x[1][e] = (uint32_t)a[1];
        }
#pragma unroll
        for (int q = 0; q < 2; ++q) {
          __builtin_amdgcn_raw_buffer_store_b128(x[q], rb, (16 * q + (l & 15)) * (dq_row_bytes / 2) + 32 * (l >> 5) + (l & 16) + (int)((uint32_t)so / 2), 0, 0);
          asm volatile("s_nop 1" :: "v"(x[q]));        // (see RowStage::flush)
        }
      } else if (chained) {
        const int at = (put_lines ? lines : dq_voff) + so, step = put_lines ? 8 * dq_row_bytes : 32;
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          const u32x4 x = __builtin_bit_cast(u32x4, f32x4{dq[4 * q], dq[4 * q + 1], dq[4 * q + 2], dq[4 * q + 3]});
          __builtin_amdgcn_raw_buffer_store_b128(x, rq, at + q * step, 0, 0);
          asm volatile("s_nop 1" :: "v"(x));
        }
        fo_done = fo;
      } else {
#pragma unroll
        for (int i = 0; i < 16; ++i) __builtin_amdgcn_raw_ptr_buffer_atomic_fadd_f32(dq[i], rq, dq_voff + 32 * (i / 4) + 4 * (i % 4), so, 0);
      }
      at0 = C::STAGE - at0;
      if (--j < 0) {                                // the next head's last block
        j = nqb - 1;
        so += (nqb - 1) * blk + D * 4;
        fo += (nqb - 1) * fblk + kChainSlices * 4;
      } else {
        so -= blk;
        fo -= fblk;
      }
    }
    if (fo_done >= 0) {
      wait_vmem<0>();
      __builtin_amdgcn_raw_buffer_store_b32((unsigned)(rank + 1), rf, fresh(lane) == 0 ? 0 : 1 << 30, fo_done, 0);
    }
    if (spin_left <= 0 && lane == 0) atomicAdd(&p.hdr->n_stalled, 1);
    int unit_next = 0;
    if (wave == 0) {
      unit_next = __builtin_amdgcn_readfirstlane(pend);
      fetch(unit_next);
    }
    lds_barrier();                                  // the LDS is free
    // ---- epilogue
    const int lane_e = fresh(lane), l32e = lane_e & 31, g2e = lane_e >> 5;
    if (direct) {
      using OUT = RowStage<D>;
      unsigned char* const obuf = smem + wave * OUT::BYTES;
      const int row_bytes = fresh_uniform(p.hkv * D * 2);
#pragma unroll
      for (int m = 0; m < 2; ++m) {
        const __amdgpu_buffer_rsrc_t r = rsrc((m ? p.dk_out : p.dv_out) + out0, row_bytes, 2);
        const float mul = m ? p.scale : 1.f;
#pragma unroll
        for (int db = 0; db < C::NVA; ++db)
#pragma unroll
          for (int i = 0; i < 16; ++i) OUT::put_bf16(obuf, OUT::reg_row(i, g2e), 32 * db + l32e, (m ? dk : dv)[db][i] * mul);
        OUT::template flush<true>(obuf, lane_e, r, row_bytes, 0);
      }
    } else {
      const int row_bytes = fresh_uniform(p.hkv * D * 4);
#pragma unroll
      for (int m = 0; m < 2; ++m) {
        const __amdgpu_buffer_rsrc_t r = rsrc((m ? p.dk : p.dv) + out0, row_bytes, 4);
        const float mul = m ? p.scale : 1.f;
#pragma unroll
        for (int db = 0; db < C::NVA; ++db)
#pragma unroll
          for (int i = 0; i < 16; ++i) {
            const float val = (m ? dk : dv)[db][i] * mul;
            const int o = (8 * (i / 4) + (i % 4)) * row_bytes + 128 * db;
            if (exclusive) __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(unsigned, val), r, 4 * g2e * row_bytes + 4 * l32e, o, 0);
            else __builtin_amdgcn_raw_ptr_buffer_atomic_fadd_f32(val, r, 4 * g2e * row_bytes + 4 * l32e, o, 0);
          }
      }
    }
    if (wave == 0) {
      publish(unit_next);
      take_elsewhere(unit_next);                    // (rare)
    }
    lds_barrier();                                  // the LDS is free for the next unit; these stores stay in flight
  }
}

}  // namespace

int launch_bwd_short(const BwdParams& p, int64_t units, int n_cu, hipStream_t stream) {
  const int64_t blocks = persistent_blocks(2 * (int64_t)n_cu, units);   // as many as are resident
  static std::atomic<uint64_t> lds_done;
  const int rc = raise_lds_limit((const void*)bwd_short_kernel<128>, ShortCfg<128>::LDS_BYTES, lds_done);
  if (rc != FCP_OK) return rc;
  hipLaunchKernelGGL(bwd_short_kernel<128>, dim3((unsigned)blocks), dim3(256), ShortCfg<128>::LDS_BYTES, stream, p);
  FCP_HIP_CHECK(hipGetLastError());
  return FCP_OK;
}

}  // namespace fcp

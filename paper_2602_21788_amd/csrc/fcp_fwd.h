// Declarations shared by the forward kernels' translation units (not installed).
#pragma once
#include "fcp_device.h"
#include "fcp_items.h"

namespace fcp {

struct FwdParams {
  const uint16_t* q;
  const uint16_t* k;
  const uint16_t* v;
  SchedHeader* hdr;
  const Tile* tiles;
  float* o_part;
  float* lse_part;
  const int32_t* q_limit;   // [tq] last key position each local query row sees, NULL = its own position (causal)
  uint16_t* o_out;          // running and direct mode: final O as bf16 [tq,hq,D], or NULL
  float* lse_out;           // direct mode: final LSE [hq,tq]
  int32_t running;          // 1: slot 0 of o_part / lse_part is the caller's running result, continued and rewritten
  int32_t direct;           // 1: a tile whose rows no other item of the launch covers writes o_out / lse_out, no partial; 2: every tile (one partial slot)
  int32_t tq, hq, hkv;
  int32_t head_pair;  // 1: a unit is a tile for TWO heads of one KV head; 0: a tile of twice the rows for one head
  int32_t tile_cap;   // tiles that the list has room for
  float scale_log2;   // softmax_scale * log2(e)
  // A launch without a list (fwd_alone in csrc/fcp_sizes.h): block b < unit_blocks finds unit b by itself, the blocks behind them classify the rows.
  int32_t unit_blocks;      // 0: the list tells
  int32_t tile;             // query rows per tile
  AloneOrder order;         // of the units
  uint8_t* q_state;         // direct mode
  ListArgs list;
};

constexpr float kRescaleThreshold = 8.f;   // log2 units

// (p.unit_blocks and p.order are set by the launch: `alone`)
int launch_fwd_small(FwdParams p, int head_dim, FwdForm form, int64_t units, bool alone, int n_cu, hipStream_t stream);

}  // namespace fcp

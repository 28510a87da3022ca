// Host representation of a rank view (the opaque fc_view).
#pragma once

#include <algorithm>
#include <cstdint>
#include <vector>

#include "../kernels/launch.hpp"
#include "flashcp.h"

namespace fc {

struct View {
  int32_t hq = 0, hkv = 0, d = 0, heads_per_tile = 1;
  int32_t bm_fwd = 0, bn_fwd = 0, bm_bwd = 0, bn_bwd = 0;

  std::vector<int32_t> q_gpos, recv_gpos;   // global positions, local / receive order
  std::vector<int32_t> seg_doc, q_cu, recv_cu, seg_piece;
  std::vector<int32_t> pieces;              // 5 per piece: seg, q_start, q_end, g_start, n_P
  std::vector<int32_t> lim;                 // receive index end seen by each query
  int64_t pairs_loc = 0, pairs_recv = 0;

  // work lists, 8 int32 per item (layout documented in flashcp.h), in map
  // order, and their largest-first launch orders
  std::vector<int32_t> fwd_local, fwd_recv, fwd_fused, bwd;
  std::vector<int32_t> perm_fwd_local, perm_fwd_recv, perm_fwd_fused, perm_bwd;
  // backward launch list, largest first: the key-major items with long query
  // ranges split into parts that write partial dK/dV (last field: partial
  // slot, -1 for a direct write), and one reduce entry per split key tile
  // (src, k0, k1, first slot, slot count, 0, 0, 0)
  std::vector<int32_t> bwd_launch, bwd_reduce;
  int32_t n_bwd_slots = 0;
  // per launch item, per 32-key wave: first query row that sees its first key
  std::vector<int32_t> bwd_qfirst;
  // dQ work of the one-launch backward where long key ranges are split over
  // workgroups (empty: the fused forward items are taken whole): items in
  // launch order, last field the partial slot or -1, and one entry per split
  // query tile (q0, q1, first slot, slot count, 0, 0, 0, 0)
  std::vector<int32_t> dq_items, dq_comb;
  int32_t n_dq_slots = 0;
  // forward of a split view: key tiles per chunk of a source (0: the view is
  // not split), the chunks as work items in launch order (forward items over
  // one source each, last field the partial slot), and per query tile of the
  // fused items q0, q1, first slot, received chunks, local chunks, 0, 0, 0
  // (its slots: the received chunks, then the local ones)
  int32_t fwd_chunk = 0;
  // whether the local, the received partial pass by itself takes the slots
  bool partial_slots[2] = {false, false};
  std::vector<int32_t> fwd_units, fwd_comb;

  // device blob: every table above that a kernel reads (the forward lists in
  // launch order), int32, sections aligned to 256 bytes; `off` holds section
  // offsets in int32 elements
  std::vector<int32_t> meta;
  struct {
    int64_t fwd_local, fwd_recv, fwd_fused;
    int64_t q_gpos, recv_gpos, lim;
    int64_t bwd_launch, bwd_reduce, bwd_qfirst;
    int64_t dq_items, dq_comb;
    int64_t fwd_units, fwd_comb;
  } off{};
  const int32_t* dev_meta = nullptr;        // set by fc_view_bind
  // a split view's own slots, behind the tables in the bound buffer (null: the
  // buffer holds the tables alone), for the partial passes
  float* dev_slots = nullptr;
  mutable fck::SlotGuard slot_guard[2];     // of the local, the received chunks' slots
  size_t table_bytes() const { return meta.size() * sizeof(int32_t); }

  int32_t t_q() const { return int32_t(q_gpos.size()); }
  int32_t t_recv() const { return int32_t(recv_gpos.size()); }
  void build_tiles();
  void build_bwd_launch();
  void build_dq_split();
  void build_fwd_split();
  int32_t head_chunks() const { return hq / hkv / heads_per_tile; }
  // backward workspace: delta, the split key tiles' partial dK/dV, the split
  // query tiles' partial dQ
  size_t delta_bytes() const { return (size_t(t_q()) * hq * sizeof(float) + 255) / 256 * 256; }
  size_t part_bytes() const {
    return 2 * size_t(n_bwd_slots) * hkv * bn_bwd * d * sizeof(float);
  }
  // one partial slot of a split query tile (forward or dQ): 128 rows x d
  size_t slot_bytes() const { return size_t(hkv) * head_chunks() * 128 * d * sizeof(float); }
  // the most bytes the slots of either direction may take: a view keeps the
  // forward's as long as it is bound, and a caller's workspaces hold both. Splits
  // gain most on ranks with a small share of a long context, where ten times
  // the output is common and small. By the estimated time, 256 MiB leave all but 1
  // of 700 split views over 2K to 256K tokens their fastest split (3% slower);
  // four times the output alone would slow half of them, by up to 3.9 times.
  size_t slots_most() const {
    return std::max(size_t(256) << 20, size_t(4) * t_q() * hq * d * sizeof(float));
  }
  size_t dq_part_bytes() const { return size_t(n_dq_slots) * slot_bytes(); }
  // the split forward's slots, and behind them 128 LSEs per slot
  size_t fwd_slots_bytes() const { return fwd_units.size() / 8 * slot_bytes(); }
  size_t fwd_split_bytes() const { return fwd_slots_bytes() + fwd_slots_bytes() / d; }
  void build_meta();
  int check_tables() const;
};

int build_view(const int32_t* cu, int32_t n_docs, const fc_shard* shards, int64_t n_shards,
               int32_t cp, int32_t rank, int32_t hq, int32_t hkv, int32_t d,
               const fc_tile_cfg* tiles, View& v);

}  // namespace fc

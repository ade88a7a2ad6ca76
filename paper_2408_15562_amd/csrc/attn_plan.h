// How a bf16 tree-attention call is laid out: rows per workgroup, and the number of workgroups that share its keys. Plain
// host code, no HIP in it.
#ifndef FSPAD_ATTN_PLAN_H
#define FSPAD_ATTN_PLAN_H

#include <stdint.h>

#include "fspad.h"

namespace fspad_detail {

constexpr int kBlockKeys = 32;          // keys per streamed block

struct Plan {
  bool shared_stage;   // the kernel whose wavefronts share K/V blocks through LDS (WS = 4 or 8 slabs of 32 rows)
  int QT, NS, WS, GY, D;
  int rows_per_unit;
  int n_wgs;           // workgroups for the largest slice of sequences
  int64_t total_blocks;
};

constexpr int64_t kComputeUnits = 256;
constexpr int64_t kMaxWorkgroups = 32768;
constexpr int kMaxQT = 4;                   // 16-row tiles per wavefront at most
constexpr int kMaxForcedWorkgroups = 4096;  // upper limit of fspad_attn_desc.workgroups

// Row tiling of one kv head's N*G query rows: up to 128 rows one or two slabs of 16*QT rows, one workgroup's. More:
// the shared-stage kernel's slabs of 32 rows, one per wavefront, four per workgroup (32/8 heads, 4096 keys, 60 nodes: 24.9 us
// against 29.9 us for 64-row tiles with two slabs).
inline void plan_rows(const fspad_attn_desc& d, Plan& pl) {
  const int rows = d.n_nodes_max * (d.n_q_heads / d.n_kv_heads);
  pl.D = d.head_dim;
  pl.shared_stage = rows > 4 * 32;
  if (pl.shared_stage) {
    pl.QT = 2;
    pl.NS = (rows + 31) / 32;
    pl.WS = 4;
    pl.GY = (pl.NS + pl.WS - 1) / pl.WS;
  } else {
    int best_cost = 1 << 30;
    for (int qt = kMaxQT; qt >= 1; --qt) {  // ties go to the larger tile: fewer re-reads of K/V
      const int ns = (rows + 16 * qt - 1) / (16 * qt);
      if (ns > 2) break;
      if (ns * qt < best_cost) { best_cost = ns * qt; pl.QT = qt; pl.NS = pl.WS = ns; }
    }
    pl.GY = 1;
  }
  pl.rows_per_unit = pl.WS * 16 * pl.QT;
}

inline int blocks_of(int kv_len, int n_nodes) {
  return (kv_len + kBlockKeys - 1) / kBlockKeys + (n_nodes + kBlockKeys - 1) / kBlockKeys;
}

// Wavefront sets that split a workgroup's keys: the two key groups of the shared-stage kernel, or
// the wavefronts that do not take a row slab of their own.
inline int key_waves(const Plan& pl) { return pl.shared_stage ? 2 : 4 / pl.WS; }

// Workgroup count for `total_blocks` flat blocks in `units` units: two resident workgroups per
// compute unit for 16-row tiles, one otherwise, but no workgroup with fewer
// than 2 blocks per key-splitting wave.
// When all units are equally long, the count is a multiple of the unit count where that pays: every unit is then cut
// into the same number of pieces, or not at all, and no workgroup straddles two units (a second segment costs a
// workgroup as much as 20 to 30 blocks do). Measured with 4 x 52 heads, 26 nodes: 1500 keys 28 us (208 workgroups) against
// 34 (256 unaligned ones), 4096 keys 77 against 79 (85 with 512); 4 x 40 heads, 60 nodes: 500 keys 19 us (160) against 33 (256),
// 4096 keys 78 against 80; 2 x 40 heads, 2048 keys, 60 nodes: 28 us (240) against 35 (256). One workgroup per compute unit
// at most: a second one shares its instruction issue and finishes last (32 heads, 4096 keys, 26 nodes: 19 us against 21 with 512).
// Not where it leaves more than two fifths of the compute units idle, nor for long streams (100 blocks of a cut
// unit, 200 of a whole one on fewer than three quarters of them), which straddling costs less than idle units do (4 x 40 heads, 8192 keys, 4 nodes: whole
// units 134 us, cut ones 107; 2 x 52 heads: two pieces each 76, cut anywhere 72), nor where 16-row tiles fill two workgroups per unit evenly
// (32 heads, 8192 keys, 4 nodes: 34 us against 31). Units of a few blocks per wavefront stay whole when there
// are enough of them (a quarter of the compute units, at most 5 blocks each): the merge costs more than the blocks
// (D = 128, 60 nodes, 17 blocks: 104 units 18.1 us whole, 21.5 in two pieces each, 29.4 unaligned; 64 units 17.7, 19.4, 28.1).
inline int plan_wgs(const Plan& pl, int64_t total_blocks, int64_t units, bool uniform, int forced) {
  const int KW = key_waves(pl);
  // (the shared-stage kernel's eight wavefronts of up to 256 registers fill a compute unit by themselves)
  // (a second resident workgroup of 32-row tiles pays where whole units outnumber the compute units, not for cut ones)
  const int64_t resident = pl.QT == 1 ? 2 * kComputeUnits : kComputeUnits;
  int64_t wgs = resident;
  const int64_t cap = total_blocks / (2 * KW);
  if (wgs > cap) wgs = cap;
  if (uniform && units <= total_blocks) {
    const int64_t rounds = (units + resident - 1) / resident;
    const int64_t blocks_per_unit = total_blocks / units;
    if (units <= kComputeUnits) {
      int64_t pieces = (blocks_per_unit + 2 * KW - 1) / (2 * KW);
      if (pieces > kComputeUnits / units) pieces = kComputeUnits / units;
      const bool few_blocks = units >= kComputeUnits / 4 && blocks_per_unit <= 5 * KW;
      if (few_blocks) pieces = 1;
      const bool is_short = few_blocks || blocks_per_unit <= 4 * KW * pieces;   // at most 4 (5 in whole units) blocks per wave
      const bool fills = 5 * units * pieces >= 3 * (wgs < kComputeUnits ? wgs : kComputeUnits);
      const bool even_anyway = pl.QT == 1 && (2 * kComputeUnits) % units == 0;
      const int64_t longest = pieces > 1 ? 100 * pieces : (4 * units >= 3 * kComputeUnits ? total_blocks : 200);
      if (is_short ? fills || pieces == 1 : fills && !even_anyway && blocks_per_unit <= longest)
        wgs = units * pieces;
    }
    if (4 * units >= 3 * rounds * resident) wgs = units;   // whole units fill the chip
    // D = 64, 32-row tiles: two workgroups fit on a compute unit, and share it with profit where the units would leave
    // more than two turns unevenly filled (13 x 40 heads, 26 nodes: 300 keys 19.6 us, one workgroup each 22.4; 3000 keys 78, 83)
    else if (units > 2 * kComputeUnits && pl.QT == 2 && !pl.shared_stage && pl.D == 64) wgs = cap < 2 * kComputeUnits ? cap : 2 * kComputeUnits;
  }
  if (forced > 0) wgs = forced < kMaxForcedWorkgroups ? forced : kMaxForcedWorkgroups;
  if (wgs > kMaxWorkgroups) wgs = kMaxWorkgroups;  // the kernels form w * (T mod W) in 32 bits
  if (wgs > total_blocks) wgs = total_blocks;
  if (wgs < 1) wgs = 1;
  return (int)wgs;
}

}  // namespace fspad_detail

#endif

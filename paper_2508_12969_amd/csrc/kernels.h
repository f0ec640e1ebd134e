// Launch interfaces of the device kernels.  Each launcher validates nothing: api.cpp has
// already checked shapes, alignment and support before it calls them.
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>
#include <type_traits>

#include "layout.h"

namespace ca {

struct PermuteArgs {
  const void* src;
  void* dst;
  int32_t T, H, W, tt, th, tw, nH, nW;
  int64_t n_vid, B, N_real, N_pad, N_video;
  int64_t planes;     // batch * num_heads
  int32_t row_bytes;  // head_dim * sizeof(element), a multiple of 16
  int32_t inverse;    // 0, 1, or one of these + kPermuteMany: then this is a PermuteManyArgs
};
constexpr int32_t kPermuteMany = 2;
// Several tensors in a launch, and room at the end of a plane of the tensors in natural order.
struct PermuteManyArgs : PermuteArgs {
  int32_t tensors;       // 1 to 3
  const void* srcs[3];   // in the place of src and dst
  void* dsts[3];
  int64_t natural_rows;  // of a plane, at least N_real; inverse: rows past N_real are written as zero
};
hipError_t launch_permute(const PermuteArgs& a, hipStream_t stream);

struct AttnArgs {
  const void* q;
  const void* k;
  const void* v;
  void* out;
  const int64_t* row_ptr;      // device; null selects the dense walk: every row uses col_meta[0..n)
  const int32_t* col_meta;     // device; per kept tile: tile id | padding class << 24; readable two words past the end
  const int32_t* order;        // device [entries]; the launch order: row ids; null = identity
  int64_t entries;             // launch-order entries per batch entry (num_heads * n rows, or fewer entries when query tiles are packed)
  int32_t simd_waves;          // one-tile kernel, 64-token tiles of head dim 64: waves per SIMD, 2 or 3
  Ways ways;                   // bf16 kernels: which of the kernels of attn_bf16_ways.hip, on `order` as rows, or kWaysNone = the others; fp32: which of attn_f32_planes.hip
  int32_t packed;              // 1: `order` also holds workgroups of two packed query tiles, as the complement of their index in the pair tables
  const int32_t* pair_rows;    // device [2*num_pairs]; row ids of the two query tiles of a workgroup (-1: none), paired kernel only
  int64_t num_pairs;
  const int32_t* pair_desc;    // device [num_pairs]; wave assignment of every workgroup of the paired kernel (layout.h)
  uint64_t upper_empty_classes; // bit c: tiles of padding class c hold no token in the upper half of their slots (paired kernel, 128-token tiles)
  const int64_t* pair_walk_ptr; // device [num_pairs + 1]; null selects the dense walk: every pair uses pair_walk[0..n)
  const int32_t* pair_walk;     // device; per walked tile: tile id | padding class << 24 | kPairInFirst | kPairInSecond,
                                // readable two words past the last entry
  const int32_t* tile_class;   // device [n]
  const SlotMask* class_mask;  // device
  const uint8_t* class_perm;   // device [num_classes * 128]; per class: valid slots ascending, then padding slots ascending
  int32_t num_classes;
  uint64_t class_valid;        // byte c: tokens of a tile of padding class c (the first eight classes)
  int32_t batch, num_heads;
  int64_t n;                   // tiles
  int32_t B, D;
  float scale;
  // natural-order variant (bf16 kernels): q, k, v, out are [batch, heads, N_real, D] and the kernel gathers / scatters
  int32_t natural;
  const int32_t* tile_origin;  // device [n]; natural-order row of slot 0 of every tile
  int32_t H, W, th, tw;
  int64_t n_vid, N_real;
  // bf16 kernels: workgroup ids below static_items map to launch-order entries through the XCD-aware
  // order; the pool_wgs workgroups after them draw a ticket from *pool_counter and take entry
  // static_items + ticket while that is below static_items + pool_items (the rest have nothing to do)
  int64_t static_items;
  int32_t pool_items, pool_wgs;
  int32_t* pool_counter;       // device; zero before and after every launch
};
// What the kernels of rows split along the keys are given besides; the others do not get it, so that their arguments lie
// as they did and their code is what it was.
struct SplitArgs : AttnArgs {
  const WorkItem* items;       // device [num_items]; null: rows are not split
  const MergeItem* merges;     // device [num_merges]
  int64_t num_items, num_merges; // of one batch entry
  int32_t share_waves;         // 32-query waves of a share
  int64_t shares;              // of one batch entry
  void* share_stats;           // device workspace of batch * shares shares: (reference, sum) of the lanes, and O
  void* share_o;
};
// The same for fp32 on the bf16 matrix instructions.
struct PlaneArgs : AttnArgs {
  void* units;                 // device workspace of plane_bytes (layout.h)
};
template <bool kSplit>
using LaunchArgs = std::conditional_t<kSplit, SplitArgs, AttnArgs>;
// fp32 problems, B <= 128, D in {32, 64, 128}
hipError_t launch_attn_f32(const AttnArgs& a, hipStream_t stream);
// the part of it with a.ways != kWaysNone, which says that `a` is a PlaneArgs
hipError_t launch_attn_f32_planes(const PlaneArgs& a, hipStream_t stream);
// bf16 problems, (B, D) in {64,128} x {64,128}
hipError_t launch_attn_bf16(const SplitArgs& a, hipStream_t stream);
// the part of it with a.ways != kWaysNone
hipError_t launch_attn_bf16_ways(const SplitArgs& a, hipStream_t stream);
// adds up the shares of split rows (after the launch that left them)
hipError_t launch_attn_bf16_merge(const SplitArgs& a, hipStream_t stream);
// bf16 problems with D = 128: workgroups that serve two query tiles (B = 64: every pair of neighbours; B = 128: the
// packed tiles of the grid's padded faces)
hipError_t launch_attn_bf16_pair(const SplitArgs& a, hipStream_t stream);

// The tile-mass kernel works on kMassQueries queries at a time: one query tile of 128 tokens, or two neighbours of 64.
constexpr int kMassQueries = 128;
inline int64_t mass_row_groups(int64_t n, int64_t B) { return (n * B + kMassQueries - 1) / kMassQueries; }
// Workgroups of four waves that a CU holds: the kernel is bound by the vector ALU (an exponential per
// score), and a third wave per SIMD fills what two leave; 128-token tiles of head dim 128 take too much LDS.
constexpr int mass_workgroups_per_cu(int64_t B, int D) { return B == 128 && D == 128 ? 2 : 3; }
constexpr int mass_step_keys(int64_t B, int D) { return B == 64 && D == 128 ? 64 : 128; }  // keys a workgroup stages at a time
constexpr int kMassMergeTiles = 32;  // key tiles that a workgroup of the merge adds up
// Workgroups that share the key tiles of a row group, `steps` steps of the kernel.  Four where that fills the card better: up to
// 1.5 launches of as many workgroups as it holds, of which at least 15 % of the places would stay empty, and a walk long enough to
// pay for the merge (4 us).  Measured, whole / four shares: head dim 64, 320 groups on 768 places 491 / 324 us, 565 256 / 210 us,
// 1120 496 / 428 us; head dim 128, 280 groups on 512 255 / 182 us, 560 459 / 313 us, 882 on 768 1191 / 1141 us.  Past the lines:
// 704 on 768 217 / 218 us, 1356 479 / 495 us, 1808 623 / 658 us, 192 groups of 16 steps 26 / 31 us (32 steps: 41 / 38, 32 groups
// of 16 steps 22 / 15).  Two or eight shares are 0-30 % slower, but for a few shapes where eight are up to 6 % faster.
inline int64_t mass_shares(int64_t groups, int64_t places, int64_t steps) {
  const int64_t rounds = (groups + places - 1) / places;
  if (2 * groups > 3 * places || 20 * groups > 17 * rounds * places) return 1;
  return steps >= (16 * groups <= places ? 16 : 32) ? 4 : 1;
}

struct MassArgs {
  const void* q;               // [batch, heads, N_pad, D] tile order, bf16
  const void* k;
  float* mass;                 // [batch, heads, n, n]
  float* partial;              // device workspace, partial_rows * n * kMassQueries * 2 floats: per query and key tile (sum,
                               // reference) of the row group a workgroup is working on (of every row group, where these
                               // have several shares)
  int64_t partial_rows;        // blocks of the workspace = most workgroups a launch may have, or the row groups where these have several shares
  int64_t places;              // workgroups that the device holds at a time
  int32_t shares;              // workgroups that share the key tiles of a row group, see mass_shares
  float* share_stats;          // device, where shares > 1: [row groups][shares][kMassQueries] (sum, reference)
  int32_t* counter;            // device; the ticket counter, zero before and after every launch
  const int32_t* dense_meta;   // device [n + 2]; per key tile: tile id | padding class << 24 | bit 31: upper key blocks empty
  const int32_t* tile_class;   // device [n]
  const SlotMask* class_mask;  // device
  const uint8_t* class_perm;   // device [num_classes * 128]
  int32_t batch, num_heads;
  int64_t n;
  int32_t B, D;
  float scale;
  int32_t num_classes;         // at most eight
  uint64_t class_valid;        // byte c: tokens of a tile of padding class c
  int32_t tokens_first;        // read where B is 128: the rows of padded tiles are brought into the order of class_perm
};
// bf16 problems, (B, D) in {64,128} x {64,128}
hipError_t launch_tile_mass(const MassArgs& a, hipStream_t stream);

}  // namespace ca

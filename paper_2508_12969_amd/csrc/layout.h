// Internal representation of a built layout.  Host tables are filled by layout.cpp (no HIP
// calls); device copies are created by api.cpp and consumed by the kernels.
#pragma once

#include <atomic>
#include <cstdint>
#include <memory>
#include <mutex>
#include <utility>
#include <vector>

#include "compact_attn.h"

namespace ca {

// Membership bits of a walk word of the paired kernel (bits 30 and 31; the tile id is below bit 24).
constexpr uint32_t kPairInFirst = 1u << 30, kPairInSecond = 1u << 31;

// How the four waves of a workgroup of the paired kernel are assigned (one word per workgroup):
// bit w: wave w works for the second query tile of the pair (else the first); bit 4 + w: wave w has
// queries at all; bits 8 + 4w .. 11 + 4w: the wave's first query slot / 32, counted in the tile's
// token-holding-slots-first order.  The plain pair of two 64-token tiles is kPairPlain: waves 0-1 hold
// slots 0-63 of the first tile, waves 2-3 those of the second.
constexpr uint32_t kPairPlain = 0xCu | 0xF0u | (0x1010u << 8);
constexpr uint32_t pair_desc_wave(int wave, int second, int first_slot32) {
  return ((uint32_t)second << wave) | (1u << (4 + wave)) | ((uint32_t)first_slot32 << (8 + 4 * wave));
}

// Validity of the B token slots of a tile, one bit per slot (B <= 128).
struct SlotMask {
  uint32_t w[4];
};

// How the entries of a launch order (rows or pairs of one batch entry, sorted by descending length)
// are handed out: the first static_entries by workgroup id, the remaining pool_entries by ticket.
struct LaunchSplit {
  int64_t static_entries = 0;
  int32_t pool_entries = 0;
};
constexpr int kPoolSlots = 64;          // pool counters per layout
constexpr int64_t kPoolMinItems = 4096; // smaller launches are dealt statically as a whole
// `work[i]`: cost of launch-order entry i (tile steps); returns the split of one batch entry's launch.
LaunchSplit split_launch(const int64_t* work, int64_t entries);

constexpr int kXcdChunk = 64;           // consecutive launch-order entries handed to one XCD
constexpr int kXcdSplitChunk = 32;      // the same where rows are split along the keys: such launches are small

// Launch-order entry of a workgroup id.  Workgroup ids are dealt round-robin to the 8 XCDs, each
// with an L2 of its own; they are remapped so that the workgroups resident on one XCD at a time
// (64: two per CU) are kXcdChunk consecutive entries of the launch order (same head, neighbouring
// query tiles, equal list lengths) instead of every eighth entry: their key-tile lists overlap, so
// more of the K/V tile copies hit that L2.  The order is sorted by descending list length, so in a
// round of 8 chunks the first chunk is the longest; rounds are therefore dealt to the XCDs in
// alternating direction, which evens out the work per XCD (measured at the 130K-token layouts:
// 1.4 % faster at 65 % sparsity, 2.3 % at 80 %, against chunks of 32 always dealt in the same
// direction).  Ids past the last full round keep their place.
constexpr int64_t xcd_launch_order(int64_t id, int64_t total, int64_t chunk = kXcdChunk) {
  const int64_t span = 8 * chunk;
  if (id >= total / span * span) return id;
  const int64_t xcd = id & 7, seq = id >> 3, round = seq / chunk;
  return round * span + ((round & 1) ? 7 - xcd : xcd) * chunk + seq % chunk;
}

// Chunk of launches of few rounds: with kXcdChunk the XCD of the first chunk gets the 64 longest rows and ends last.  Measured, 64 / 8, fp32 and
// ways-4x4 launches from 512 to 4095 workgroups: 1.04 times as fast over 44 of them (0.985 to 1.25); 8 heads of 7K tokens, fp32, head dim
// 128 754 / 660 us.  4 and 16 gave the same.  Below one span of large chunks all ids keep their place, which is the best there (chunks of 4, 8, 16: up to
// 1.08, but 0.78 to 0.86 on three of 20 launches of little more than one workgroup per CU); the kernels of eight waves were between 0.965 and 1.04
// and keep kXcdChunk.  launch_time goes on with kXcdChunk, which its constants were fitted with.
constexpr int64_t kXcdFewRows = 4096;
constexpr int kXcdFewChunk = 8;
constexpr int64_t xcd_chunk(int64_t total) { return total < kXcdFewRows && total >= 8 * kXcdChunk ? kXcdFewChunk : kXcdChunk; }

// The kernels of attn_bf16_ways.hip: waves of a workgroup x 32-query waves side by side; and those of attn_f32_planes.hip:
// 32-query waves side by side x waves that share the keys of a query.
enum Ways : int32_t { kWaysNone = 0, kWays4x4, kWays8x4, kWays8x2, kPlanes2x2, kPlanes2x4, kPlanes1x4 };

// Launches whose longest rows would outlast everything else, or that leave CUs without work, are split along the
// keys: a workgroup takes `count` tiles of the list of a launch-order
// entry (a row, or the complement of a workgroup of two query tiles), from its `first` on, and leaves what it has summed up to then in
// a workspace, from which a second kernel adds up the shares of a row.  place: part of the row's query slots | (share + 1) << 2,
// without a share for a row that is one item and writes its output itself.
struct WorkItem {
  int32_t entry, first, count, place;
};
struct MergeItem {
  int32_t entry, part, first_share, shares;
};
struct SplitPlan {  // of one batch entry; empty: rows are not split
  Ways ways = kWaysNone;
  std::vector<WorkItem> items;    // longest first
  std::vector<MergeItem> merges;
  int32_t shares = 0;
  int32_t waves = 0;              // 32-query waves of an item
};
constexpr int64_t kMaxSplitItems = 8192;
constexpr int64_t kMaxShareBytes = (int64_t)64 << 20;  // of all batch entries
// A share of `queries` queries: (reference, sum) of every lane of its 32-query waves, and O in fp32.
constexpr int64_t share_stats_bytes(int64_t queries) { return queries / 32 * 64 * 8; }
constexpr int64_t share_bytes(int64_t queries, int64_t head_dim) { return share_stats_bytes(queries) + queries * head_dim * 4; }
inline int64_t workspace_bytes(const SplitPlan& plan, int64_t batch, int64_t head_dim) {
  return plan.shares * batch * share_bytes(32 * plan.waves, head_dim);
}

// 16-query groups side by side in a workgroup of attn_f32.hip: as many as the tile has, because they share the staged keys; fewer, with
// the keys of a query split over the waves instead, while the launch has less than five workgroups
// per CU.  Measured: 1128 rows of 64 tokens at D = 128, 4 / 2 groups: 1.27 / 1.20 ms; 732 rows of 60 at
// D = 32, 4 / 2 / 1: 0.63 / 0.65 / 0.69 ms, where the one line for all head dims takes 2 and is 3 % off.  At D = 128, one group fills the LDS of a CU with one
// workgroup and waits for copies (240 rows of 128 tokens, 2 / 1 groups: 0.31 / 0.37 ms): small tiles only.
inline int f32_query_groups(int64_t rows, int64_t B, int64_t head_dim) {
  constexpr int64_t kMinWorkgroups = 1280;
  const int fewest = head_dim == 128 ? 2 : 1;
  int qw = B <= 16 ? 1 : B <= 32 ? 2 : 4;
  while (qw > fewest && rows * ((B + 16 * qw - 1) / (16 * qw)) < kMinWorkgroups) qw /= 2;
  return qw;
}

// fp32 attention on the bf16 matrix instructions (attn_f32_planes.hip): K and V are split into three bf16 values each, in units
// of 16 tokens.
constexpr int64_t kMaxPlaneBytes = (int64_t)8 << 30;  // of a call; of the copies of a dense call too
inline int64_t plane_bytes(int64_t planes, int64_t n, int64_t B, int64_t head_dim) { return planes * n * ((B + 15) / 16) * 16 * head_dim * 12; }

// Device-resident tables, parts of one block of device memory owned by the layout.
struct DeviceTables {
  unsigned char* block = nullptr;
  int64_t* row_ptr = nullptr;    // [num_heads*n + 1] offsets into col_idx (global over heads)
  int32_t* col_meta = nullptr;   // [nnz] kept key tiles, ascending inside each row: tile id | class << 24
  int32_t* dense_meta = nullptr; // [n] the same packing for the list 0..n-1 (dense walk)
  int32_t* order = nullptr;      // [num_heads*n] launch order of row ids head*n + tile
  int32_t* launch_rows = nullptr; // [num_launch_rows] launch order when query tiles are packed (row ids, and ~i for packed workgroup i); else null: `order`
  int64_t num_launch_rows = 0;
  int32_t* pair_desc = nullptr;  // [num_pairs] wave assignment of every workgroup of the paired kernel
  int32_t* pair_rows = nullptr;  // [2*num_pairs] row ids of the two query tiles a workgroup of the paired kernel owns (-1: none), in launch order
  int64_t num_pairs = 0;
  int64_t* pair_walk_ptr = nullptr;   // [num_pairs + 1]
  int32_t* pair_walk = nullptr;       // packed walk words (tile id | class << 24 | membership bits), two words of padding
  int32_t* dense_pair_walk = nullptr; // [n + 2] the walk 0..n-1 kept by both tiles (dense path)
  int32_t* tile_class = nullptr; // [n] index into class_mask; 0 = every slot holds a token
  SlotMask* class_mask = nullptr; // [num_classes]
  uint8_t* class_perm = nullptr;  // [num_classes * 128] per class: its valid slots ascending, then its padding slots ascending
  int32_t* tile_origin = nullptr; // [n] natural-order row of slot 0 of every tile
  WorkItem *split_items = nullptr, *split_items_dense = nullptr;      // SplitPlan of the sparse and of the dense walk
  MergeItem *split_merges = nullptr, *split_merges_dense = nullptr;
  int32_t* pool_counters = nullptr; // [pool_slots] tickets of the dynamically drawn tail of a launch; zero between launches
  int32_t pool_slots = 0;           // concurrent launches on one layout take different counters, round-robin
  float* mass_partial = nullptr;   // workspace of the tile-mass kernel, allocated at its first call: mass_partial_rows (= most
                                   // workgroups of its launch) * n * kMassQueries * 2 floats
  int64_t mass_partial_rows = 0;
  int64_t mass_places = 0;         // workgroups of it that the device holds at a time
  int32_t mass_shares = 1;         // workgroups that share the key tiles of a row group
  float* mass_share_stats = nullptr;  // inside the same allocation, as the counter is
  int32_t* mass_counter = nullptr; // its ticket counter
};

}  // namespace ca

struct ca_layout {
  ca_problem prob{};
  int32_t nT = 0, nH = 0, nW = 0;
  int64_t B = 0, n_vid = 0, n_txt = 0, n = 0, N_real = 0, N_pad = 0;
  float scale = 0.f;

  // host tables
  std::vector<int64_t> row_ptr;             // [num_heads*n + 1], global offsets
  std::vector<int32_t> col_idx;             // [nnz]
  std::vector<std::vector<int64_t>> head_row_ptr;  // per head, relative offsets (C-ABI view)
  std::vector<int32_t> order;               // [num_heads*n]
  std::vector<int32_t> pair_rows;           // [2*num_pairs], empty unless the paired kernel serves (part of) this layout
  std::vector<int32_t> pair_desc;           // [num_pairs] wave assignment (kPairPlain for a plain pair)
  // 128-token tiles, head dim 128: query tiles whose tokens fill fewer than four waves (tiles on a
  // padded face of the grid) are packed several to a workgroup (pair_rows, pair_desc), and
  // `launch_rows` is the launch order of everything, longest first: `order` without the packed
  // rows, and the complement ~i of packed workgroup i.
  bool packed_faces = false;
  std::vector<int32_t> launch_rows;
  std::vector<int64_t> pair_walk_ptr;       // [num_pairs + 1] offsets into pair_walk
  std::vector<int32_t> pair_walk;           // per pair: union of its two rows, tile id | kPairInFirst | kPairInSecond
  std::vector<int32_t> tile_class;          // [n]
  std::vector<ca::SlotMask> class_mask;     // class 0 = all valid
  bool mass_tokens_first = false;           // tile mass: the padded tiles' tokens are brought to the front, see build_slot_masks

  // A launch deals most of its workgroups to the XCDs statically and
  // leaves the cheapest entries at the end of the launch order to be drawn by whichever XCD gets there
  // first: rows / pairs of the sparse and of the dense walk.
  ca::LaunchSplit split_rows, split_rows_dense, split_pairs, split_pairs_dense;
  int32_t simd_waves = 2, simd_waves_dense = 2;               // waves per SIMD of the one-tile kernel (choose_simd_waves)
  ca::Ways ways = ca::kWaysNone, ways_dense = ca::kWaysNone;  // kernel of the sparse and of the dense walk, natural order included
  ca::SplitPlan split, split_dense;                           // rows split along the keys, for calls that bring a workspace
  ca::Ways planes = ca::kWaysNone, planes_dense = ca::kWaysNone;  // fp32: kernel of calls that bring a workspace, kWaysNone = attn_f32.hip
  // Dense walks do not depend on the tiles.  Where that is predicted to be faster, dense calls run on this layout of the same tokens
  // in natural order, cut into tiles of 128 without padding but at the end: on copies in a workspace, or on the tensors as
  // they are (closed_in_place: no tile is padded and 64-token tiles are taken two by two).  Only its dense tables are used.
  std::unique_ptr<ca_layout> closed;
  bool closed_in_place = false, is_closed = false;
  double closed_us = 0;  // predicted time of dense calls, infinite if they are not priced
  mutable std::atomic<uint32_t> launch_seq{0};  // picks the pool counter of a launch

  // device tables, created once
  std::mutex upload_mutex;
  bool uploaded = false;
  int device = -1;
  ca::DeviceTables dev;

  // The tables of the sparse forward as one block of bytes with 256-byte aligned parts, ready to be
  // copied into a fixed device array (compact_attn_forward_static); packed on first use.
  uint64_t serial = 0;                      // unique per layout object, never reused
  std::vector<unsigned char> static_image;
  struct StaticOffsets {
    size_t row_ptr = 0, col_meta = 0, order = 0, pair_rows = 0, pair_walk_ptr = 0, pair_walk = 0, tile_class = 0,
           class_mask = 0, class_perm = 0, pool_counter = 0, pair_desc = 0, launch_rows = 0, split_items = 0, split_merges = 0;
  } static_off;
};

namespace ca {

void set_error(const char* fmt, ...);
void clear_error();
const char* last_error();

// Fills every host table of `L` from L.prob and the head descriptions.  Returns a ca_status.
int build_host_tables(ca_layout& L, const ca_head* heads);
// The same from per-head CSR arrays (validated: extents, ids in range, strictly ascending rows).
int import_host_tables(ca_layout& L, const int64_t* const* row_ptr, const int32_t* const* col_idx);
// Row-wise union of two layouts of the same geometry and head count.
int union_host_tables(ca_layout& L, const ca_layout& a, const ca_layout& b);
// |A and B| / |A or B| over the tile pairs of head `ha` of a and head `hb` of b (1 if both are empty).
double head_similarity(const ca_layout& a, int32_t ha, const ca_layout& b, int32_t hb);
// Window search of one head (search.cpp); mass is host float [n*n], groups_out has num_groups entries.
int search_head_windows(const ca_layout& L, const float* mass, const int32_t* group_max_dt, int32_t num_groups, double tau,
                        double lambda, int32_t pattern, ca_group* groups_out, double* recall_out, double* kept_out);
// Host images of the tables the kernels read, packed from the layout's host tables (no HIP calls).
struct PackedTables {
  std::vector<int32_t> col_meta, dense_meta, pair_walk, dense_pair_walk, tile_origin;
  std::vector<uint8_t> class_perm;
};
// `forward_only` leaves out what only the dense and the natural-order walks read.  Returns a ca_status.
int pack_device_tables(const ca_layout& layout, bool forward_only, PackedTables& t);
// Kernel of the sparse or the dense walk, and the figures of the tiles it goes by; at most about `max_words` kept
// tiles are looked at.
constexpr int64_t kSampledWords = 500000;
Ways choose_ways(const ca_layout& L, bool dense, int64_t max_words, SplitPlan* plan = nullptr, double* predicted_us = nullptr);
Ways choose_planes(const ca_layout& L, bool dense, int64_t max_words);
std::pair<double, double> granules_per_tile(const ca_layout& L, bool dense, int64_t max_words);
// Bytes of a tensor of a bf16 layout in tile order.
inline int64_t tensor_bytes(const ca_layout& L) { return (int64_t)L.prob.batch * L.prob.num_heads * L.N_pad * L.prob.head_dim * 2; }
// Bytes that a sparse or a dense attention call can make use of.
inline int64_t call_workspace_bytes(const ca_layout& L, bool dense) {
  const ca_problem& p = L.prob;
  if (dense && L.closed) return (L.closed_in_place ? 0 : 4 * tensor_bytes(*L.closed)) + workspace_bytes(L.closed->split_dense, p.batch, p.head_dim);
  if (dense ? L.planes_dense : L.planes) return plane_bytes((int64_t)p.batch * p.num_heads, L.n, L.B, p.head_dim);
  return workspace_bytes(dense ? L.split_dense : L.split, p.batch, p.head_dim);
}
// Derived tables (per-head views, launch order, padding classes) once row_ptr / col_idx are set.
void finish_host_tables(ca_layout& L);

}  // namespace ca

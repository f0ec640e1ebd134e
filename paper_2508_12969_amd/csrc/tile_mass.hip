// Attention mass per tile pair on bf16 MFMA (Sec. 4.2 of the paper: masks are searched by the
// recall they keep, i.e. by how much of the full attention's probability mass falls on the kept
// tile pairs).  For every (batch, head, query tile a) the kernel produces, for all key tiles b,
//     mass[a, b] = sum_{i in a} sum_{j in b} softmax_row_i(scale * Q K^T)[j]
// over real tokens only (padding queries add nothing, padding keys are never attended).
//
// Same decomposition as the attention kernel in attn_bf16.hip: a wave owns 32 queries, transposed
// product S^T = K Q^T so that a lane owns one query (QueryWave in attn_bf16_common.h), K tiles copied
// into swizzled LDS, two buffers.  There is no V.
//
// What bounds it: the vector ALU.  Per score there is a multiply, an exponential (measured 3.6 ns per wave
// and SIMD, a multiply 1.1) and an add, about as many cycles as the matrix instructions at head dim 128 and twice
// as many at 64, so the
// exponentials of a tile are laid out to run beside the products of the next (one straight line of
// code per step, the rare cases aside) and the CU holds as many waves as the registers allow.
//
// One product per tile pair.  The normaliser l_i of a query is known only after its last key tile,
// so the walk over the n key tiles keeps what it cannot finish: per query i and key tile b the
// unnormalised sum  e[b][i] = sum_{j in b} exp2(scale' * (s_ij - m)), together with the exponent
// reference m it was taken against (it moves when a sum outgrows it, rarely), two floats, written to a workspace in
// device memory (2 * n * 128 floats per workgroup).  After the walk the workgroup reads its
// block back (or, where a launch would leave places empty and several workgroups share the key tiles, a second kernel
// reads theirs), brings every sum to the query's final reference and reduces over the queries,
//     mass[a, b] = sum_i e[b][i] * exp2(scale' * (m[b][i] - m_i)) / l_i,
// in a fixed order, so the result is run-to-run identical.  (The alternative without a workspace
// walks every row twice and multiplies twice; it measured twice the time per product.)
#include <algorithm>
#include <type_traits>

#include "attn_bf16_common.h"

namespace ca {
namespace {

// exp2 of a reference against the final one.  None lies above that but those of shares without a finite score, whose sums
// are zero and must stay so; NaN stays NaN.
__device__ __forceinline__ float ref_factor(float x) { return __builtin_amdgcn_exp2f(x > 0.f ? 0.f : x); }

constexpr float kSumLimit = 0x1p40f;  // a tile's row sum beyond this moves the query's exponent reference

// 128 queries per workgroup: one query tile of 128 tokens or two neighbours of 64 (the walk is the same
// for all rows of a head), and 128 keys per step, two tiles of 64 tokens; 64 keys where only that leaves
// LDS for a third workgroup on the CU (64-token tiles, head dim 128).
// Measured (all with 0.1 us more per group than now, see the end of the kernel), against one query tile and one key tile
// at a time and two waves per SIMD: 64-token tiles of head dim 64, 14.4K queries x 14.4K keys, 12 heads 771 -> 623 us, 80.6K x 80.6K, 8 heads 12.1 -> 10.0 ms;
// of head dim 128, 8 heads of 75.6K 17.9 -> 14.4 ms (15.7 ms with two workgroups of 128-key steps).
// 256-key steps at head dim 64 with two workgroups: 685 us and 11.1 ms; four workgroups: 625 us, 10.2 ms.
template <int B, int D>
struct MassShape {
  static constexpr int kQueries = kMassQueries, kRowTiles = kQueries / B;
  static constexpr int kStepKeys = mass_step_keys(B, D), kStepTiles = kStepKeys / B;
  struct Tile : Shape<B, D, 4> {        // what a wave multiplies at a time
    // without it the reads of a whole tile are requested at once (212 instead of 186 registers), and the
    // call takes 53.0 instead of 50.0 ms at the 119K-token layout of 12 heads
    static constexpr int kLeadK = 6;
  };
  using Step = Shape<kStepKeys, D, 4>;  // what the workgroup copies at a time
};

// mass[a, b] = sum_i e[b][i] * exp2(scale' * (m[b][i] - m_i)) / l_i of the key tiles begin .. end - 1 of a row group, by 256
// threads; part: its block of the workspace, rows: query tiles from its first one to the last of the plane.
// nan_from (shared key tiles): per query tile the first key tile of a later share than one with an infinite score.
template <int B, bool kSplit>
__device__ __forceinline__ void reduce_tiles(const float2* part, const float* inv_of, const float* ref_of, const int* nan_from, float c2, int begin,
                                             int end, int n, int64_t rows, float* out) {
  constexpr int kLanesPerTile = kMassQueries / 4;  // a key tile's pairs, four per lane
  constexpr int kTilesPerPass = 256 / kLanesPerTile;
  const int sub = threadIdx.x / kLanesPerTile, l4 = threadIdx.x % kLanesPerTile;
  const int row_of_lane = l4 * 4 / B;   // which of the workgroup's query tiles
  const bool stores = l4 * 4 % B == 0 && row_of_lane < rows;
  const float4 inv = *reinterpret_cast<const float4*>(&inv_of[4 * l4]);
  const float4 ref = *reinterpret_cast<const float4*>(&ref_of[4 * l4]);
  // kBatch key tiles per lane at a time, all loads requested before the first is used
  constexpr int kBatch = 4;
  static_assert(kBatch * kTilesPerPass == kMassMergeTiles, "a workgroup of the merge takes one batch");
  for (int b0 = begin + sub; b0 < end; b0 += kBatch * kTilesPerPass) {
    float4 p01[kBatch], p23[kBatch];  // (e0, m0, e1, m1), (e2, m2, e3, m3)
#pragma unroll
    for (int u = 0; u < kBatch; ++u) {
      const int b = min(b0 + u * kTilesPerPass, end - 1);  // past the end: a valid tile, not stored
      const float4* p = reinterpret_cast<const float4*>(part + (int64_t)b * kMassQueries + 4 * l4);
      p01[u] = p[0];
      p23[u] = p[1];
    }
#pragma unroll
    for (int u = 0; u < kBatch; ++u) {
      const int b = b0 + u * kTilesPerPass;
      const float t0 = p01[u].x * ref_factor((p01[u].y - ref.x) * c2) * inv.x;
      const float t1 = p01[u].z * ref_factor((p01[u].w - ref.y) * c2) * inv.y;
      const float t2 = p23[u].x * ref_factor((p23[u].y - ref.z) * c2) * inv.z;
      const float t3 = p23[u].z * ref_factor((p23[u].w - ref.w) * c2) * inv.w;
      float s = (t0 + t1) + (t2 + t3);
#pragma unroll
      for (int sh = B / 8; sh >= 1; sh >>= 1) s += __shfl_xor(s, sh, 64);
      if constexpr (kSplit) s = b < nan_from[row_of_lane] ? s : __builtin_nanf("");
      if (stores && b < end) out[row_of_lane * (int64_t)n + b] = s;
    }
  }
}

// The slots of a tile, those that hold a token first, of every padding class.
__device__ __forceinline__ uint8_t* lds_perm() {
  __shared__ uint8_t perm[8 * 128];
  return perm;
}

__device__ __forceinline__ int class_of(int32_t word) { return (word >> 24) & 0x7f; }

__device__ __forceinline__ int tokens_of(int32_t word, uint64_t class_valid) { return (int)((class_valid >> (8 * class_of(word))) & 0xffu); }

// f(blocks of 32 keys that hold a token, tokens of the last of them) for a tile of 128
template <class F>
__device__ __forceinline__ auto by_blocks(int tokens, F&& f) {
  if (tokens > 96) return f(std::integral_constant<int, 4>{}, tokens - 96);
  if (tokens > 64) return f(std::integral_constant<int, 3>{}, tokens - 64);
  if (tokens > 32) return f(std::integral_constant<int, 2>{}, tokens - 32);
  return f(std::integral_constant<int, 1>{}, tokens);
}

template <class W, class Blocks, class Acc>
__device__ __forceinline__ void scores_tokens_first(W& w, LdsTile tile, Blocks blocks, int last, Acc& acc) {
  w.template qk<0, blocks()>(tile, acc);
  if (last < 32) mask_granules(acc[blocks() - 1], min(16, last), max(0, last - 16));
}

// This wave's part of key tile `step`, whose word it is, into its buffer.
template <class M, class Loader>
__device__ __forceinline__ void issue_tokens_first(const Loader& loader, const char* Kp, int32_t word, int step, uint32_t lds_k_addr, int wave) {
  using S = typename M::Step;
  static_assert(M::kStepTiles == 1, "a step is one tile");
  const char* const from = Kp + (int64_t)step * S::kTileBytes;
  const uint32_t to = lds_k_addr + (step & 1) * S::kTileBytes;
  const int c = class_of(word);
  if (c == 0) {
    loader.issue(from, to, wave);
    return;
  }
  const int in_block = (threadIdx.x & 63) / S::kChunksPerRow;
#pragma unroll
  for (int i = 0; i < S::kLoadsPerThread; ++i) {
    const int block = wave * S::kLoadsPerThread + i;
    const int slot = lds_perm()[c * 128 + block * S::kRowsPerLoad + in_block];
    copy_rows(to + (uint32_t)block * 1024u, from, (uint32_t)((slot - in_block) * S::kRowBytes) + loader.voff[i & 3]);
  }
}

// kSplit: the key tiles of a row group are shared by several workgroups, see mass_shares.  Each leaves its sums and, for
// every query, its total and reference; tile_mass_merge_kernel finishes.
// kTokensFirst (128-token tiles, chosen by build_slot_masks): the rows of a padded tile are copied token-holding slots first,
// each from an address of its own, and blocks of 32 keys that are then without a token are neither multiplied nor summed; else
// the tile's order and a mask per slot.
template <int B, int D, bool kSplit, bool kTokensFirst>
__global__ __attribute__((amdgpu_flat_work_group_size(256, 256), amdgpu_waves_per_eu(mass_workgroups_per_cu(B, D), mass_workgroups_per_cu(B, D))))
void tile_mass_kernel(MassArgs a) {
  using M = MassShape<B, D>;
  using S = typename M::Tile;
  constexpr int KT = M::kStepTiles, Q = M::kQueries;
  __shared__ __attribute__((aligned(1024))) char lds_k[2 * M::Step::kTileBytes];
  __shared__ __attribute__((aligned(16))) float lds_inv[Q];  // 1 / l_i
  __shared__ __attribute__((aligned(16))) float lds_ref[Q];  // m_i
  __shared__ int lds_ticket;
  if constexpr (kTokensFirst) {
    for (int e = threadIdx.x; e < a.num_classes * 128; e += 256) lds_perm()[e] = a.class_perm[e];  // visible from the first ticket on
  }

  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int64_t groups = (a.n + M::kRowTiles - 1) / M::kRowTiles;  // per head
  const int shares = kSplit ? a.shares : 1;  // items per row group, each a part of its key tiles
  const int total = (int)((int64_t)a.batch * a.num_heads * groups) * shares;
  // one packed word per key tile 0..n-1: tile id | padding class << 24 | bit 31: upper key blocks empty
  const auto meta = CONST_PTR(int32_t, a.dense_meta);
  const auto class_mask = CONST_PTR(uint32_t, a.class_mask);  // 4 words per class
  const int n = (int)a.n;
  const int steps = (n + KT - 1) / KT;
  const TileLoader<typename M::Step, false> k_loader(wave, lane);
  const int my_key_tile = wave * KT / 4;  // the tile of a step this wave copies (a part of)
  const uint32_t lds_k_addr = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) char*)lds_k;
  const LdsTile k_tile = (LdsTile)lds_k;

  // The grid is at most as many workgroups as the card holds at a time; each takes (batch, head, row
  // group, share) items of the launch by ticket until none is left, so an XCD that runs faster takes more.
  // Every workgroup draws once more than it has items; whoever draws the last ticket of all zeroes the
  // counter for the next launch.
  for (;;) {
  if (threadIdx.x == 0) {
    const int t = atomicAdd(a.counter, 1);
    if (t == total + (int)gridDim.x - 1) __hip_atomic_store(a.counter, 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    lds_ticket = t;
  }
  __syncthreads();
  if (lds_ticket >= total) return;  // all threads of the workgroup alike
  const int64_t item = kSplit ? lds_ticket / shares : lds_ticket;  // (batch, head, row group), row-major
  const int share = kSplit ? lds_ticket % shares : 0;
  const int first_step = kSplit ? (int)((int64_t)share * steps / shares) : 0;
  const int end_step = kSplit ? (int)((int64_t)(share + 1) * steps / shares) : steps;
  // the block of the workspace, [n][Q] pairs (sum, reference): the row group's if several workgroups fill it, else the
  // workgroup's own, reused item after item
  float2* part = reinterpret_cast<float2*>(a.partial) + (kSplit ? item : (int64_t)blockIdx.x) * a.n * Q;
  const int64_t plane_id = item / groups;        // (batch, head)
  const int64_t first_row = item % groups * M::kRowTiles;
  const int64_t plane = plane_id * a.n * (int64_t)S::kTileBytes;
  const char* Kp = static_cast<const char*>(a.k) + plane;
  float* out = a.mass + (plane_id * a.n + first_row) * a.n;

  // A wave without a query tile or a real query (see query_slot) takes part in the tile copies and barriers only.
  QueryWave<S> w(lane, a.scale);
  const int64_t my_row = first_row + wave * 32 / B;
  const bool has_row = my_row < a.n;
  const int64_t q_tile = has_row ? my_row : first_row;
  const QuerySlot qs = query_slot<B>(a, q_tile, wave * 32 % B, w.qi);
  const bool wave_active = has_row && qs.wave_active;
  w.load_q(static_cast<const char*>(a.q) + plane + (q_tile * B + qs.slot) * S::kRowBytes);
  const int mine = wave * 32 + w.qi;  // this lane's query in the workspace block and in lds_inv
  const bool writer = w.g == 0;       // both lanes of a pair hold the query's sum; the lower one stores it

  if (first_step * KT + my_key_tile < n) {
    if constexpr (kTokensFirst) issue_tokens_first<M>(k_loader, Kp, meta[first_step], first_step, lds_k_addr, wave);
    else k_loader.issue(Kp + (int64_t)first_step * M::Step::kTileBytes, lds_k_addr + (first_step & 1) * M::Step::kTileBytes, wave);
  }
  float2 prev[KT];     // the previous step's sums and their references, stored at the head of the next step
  float m_run = 0.f;   // its exponent reference
  float l_row = 0.f;   // the query's running sum over the item's key tiles (both lanes of a pair hold it)
  float limit = -1.f;  // a row sum beyond it moves the reference: kSumLimit, and every sum before the query's first finite score
  auto store_step = [&](int step) {
#pragma unroll
    for (int t = 0; t < KT; ++t)
      if (writer && step * KT + t < n) part[(int64_t)(step * KT + t) * Q + mine] = prev[t];
  };

  // Where the loop's code lies matters, with a period of 32 bytes: moved 4 bytes at a time, 119K tokens x 12 heads of head dim 128 take
  // 49.1 to 50.5 ms, 12 heads x 20K of 128-token tiles and head dim 64 1.239 to 1.265 ms.  This is the first of eight places for
  // whole row groups; shared ones lie well without it (144 us at 3 heads x 12.5K of head dim 64, 146 us with it).
  if constexpr (!kSplit) asm volatile("s_nop 0");
  for (int j = first_step; j < end_step; ++j) {
    int32_t words[KT];  // past the end: tile 0's, not used
#pragma unroll
    for (int t = 0; t < KT; ++t) words[t] = meta[j * KT + t < n ? j * KT + t : 0];
    int32_t next_word = 0;
    if constexpr (kTokensFirst) next_word = meta[min(j + 1, n - 1)];
    // K(j) landed and visible, buffer (j+1)%2 free, the previous step's stores have been written
    WAIT_VMCNT(0);
    BARRIER();
    if ((!kSplit || j + 1 < end_step) && (j + 1) * KT + my_key_tile < n) {
      if constexpr (kTokensFirst) issue_tokens_first<M>(k_loader, Kp, next_word, j + 1, lds_k_addr, wave);
      else k_loader.issue(Kp + (int64_t)(j + 1) * M::Step::kTileBytes, lds_k_addr + ((j + 1) & 1) * M::Step::kTileBytes, wave);
    }
    if (j > first_step) store_step(j - 1);  // a whole step to complete
    const LdsTile k_step = k_tile + (j & 1) * M::Step::kTileBytes;

    constexpr std::integral_constant<int, S::kKeyBlocks> all_blocks;
    auto row_sum = [&](const floatx16 (&acc)[S::kKeyBlocks], auto blocks) {
      float e4[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int kb = 0; kb < blocks(); ++kb)
#pragma unroll
        for (int r = 0; r < 16; ++r) e4[r & 3] += __builtin_amdgcn_exp2f(acc[kb][r] * w.c2);
      return sum_with_partner((e4[0] + e4[1]) + (e4[2] + e4[3]));
    };
    float e[KT];
#pragma unroll
    for (int t = 0; t < KT; ++t) e[t] = 0.f;
    if (wave_active) {
      // The exponent reference is the row maximum of the first tile with a finite score.  Afterwards no maximum is
      // taken: the sums of a step are formed against the reference as it stands, and only if a tile's row sum leaves
      // [0, kSumLimit] for some query (it overflows, or is about to), or a query's sum is still zero (it has met
      // scores of minus infinity alone), the step is done again tile by tile,
      // with the tile's row maximum as the new reference of such queries.  Numerator and denominator
      // of a query always share one reference after the final pass, so the masses are those of the
      // exact softmax.
      bool by_tile = j == first_step || (j + 1) * KT > n;
      if (!by_tile) {
        bool move = false;
        int padding = 0;
#pragma unroll
        for (int t = 0; t < KT; ++t) padding |= words[t] >> 24;
        if (padding == 0) {
          // one straight line of code, so that the products of a tile can run beside the exponentials of
          // the one before
#pragma unroll
          for (int t = 0; t < KT; ++t) {
            floatx16 acc_s[S::kKeyBlocks];
            w.template qk<0, S::kKeyBlocks>(k_step + t * S::kTileBytes, acc_s);
            e[t] = row_sum(acc_s, all_blocks);
            move = move || !(e[t] <= limit);  // also true for inf and NaN
          }
        } else if constexpr (kTokensFirst) {
          e[0] = by_blocks(tokens_of(words[0], a.class_valid), [&](auto blocks, int last) {
            floatx16 acc_s[S::kKeyBlocks];
            scores_tokens_first(w, k_step, blocks, last, acc_s);
            return row_sum(acc_s, blocks);
          });
          move = !(e[0] <= limit);
        } else {
#pragma unroll
          for (int t = 0; t < KT; ++t) {
            floatx16 acc_s[S::kKeyBlocks];
            w.qk_tile(k_step + t * S::kTileBytes, acc_s, words[t] >= 0);
            w.mask_padding_keys(acc_s, (words[t] >> 24) & 0x7f, class_mask);
            e[t] = row_sum(acc_s, all_blocks);
            move = move || !(e[t] <= limit);
          }
        }
        const uint64_t movers = __builtin_amdgcn_ballot_w64(move);
        by_tile = __builtin_amdgcn_readfirstlane((uint32_t)movers | (uint32_t)(movers >> 32)) != 0;
        if (!by_tile) {
#pragma unroll
          for (int t = 0; t < KT; ++t) {
            prev[t] = float2{e[t], m_run};
            l_row += e[t];
          }
        }
      }
      if (by_tile) {
#pragma unroll
        for (int t = 0; t < KT; ++t) {
          if (j * KT + t >= n) break;
          floatx16 acc_s[S::kKeyBlocks];
          if constexpr (kTokensFirst) {
            by_blocks(tokens_of(words[t], a.class_valid), [&](auto blocks, int last) {
              scores_tokens_first(w, k_step, blocks, last, acc_s);
#pragma unroll
              for (int kb = blocks(); kb < S::kKeyBlocks; ++kb)
#pragma unroll
                for (int r = 0; r < 16; ++r) acc_s[kb][r] = kMinusInf;
            });
          } else {
            w.qk_tile(k_step + t * S::kTileBytes, acc_s, words[t] >= 0);
            w.mask_padding_keys(acc_s, (words[t] >> 24) & 0x7f, class_mask);
          }
          bool move = true;  // this lane's query takes a new reference (every query on the first tile)
          if (j > first_step || t > 0) {
            e[t] = row_sum(acc_s, all_blocks);
            move = !(e[t] <= limit);
          }
          const uint64_t movers = __builtin_amdgcn_ballot_w64(move);
          if (__builtin_amdgcn_readfirstlane((uint32_t)movers | (uint32_t)(movers >> 32)) != 0) {
            float mx = acc_s[0][0];
#pragma unroll
            for (int kb = 0; kb < S::kKeyBlocks; ++kb)
#pragma unroll
              for (int r = 0; r < 16; ++r) mx = fmaxf(mx, acc_s[kb][r]);
            mx = max_with_partner(mx);
            float delta = move ? mx : 0.f;
            if (delta == kMinusInf) delta = 0.f;  // a row that has seen no real key yet keeps its reference
            m_run += delta;
            // the reference only rises after the first finite score; before it nothing is summed, and a first maximum
            // far below zero must not make the factor infinite
            l_row *= __builtin_amdgcn_exp2f(fminf(-delta * w.c2, 0.f));
#pragma unroll
            for (int kb = 0; kb < S::kKeyBlocks; ++kb)
#pragma unroll
              for (int r = 0; r < 16; ++r) acc_s[kb][r] -= delta;
#pragma unroll
            for (int r = 0; r < 16; ++r) w.neg_m[r] = -m_run;
            e[t] = row_sum(acc_s, all_blocks);
          }
          l_row += e[t];
          if (l_row != 0.f) limit = kSumLimit;
          prev[t] = float2{e[t], m_run};
        }
      }
    } else {
#pragma unroll
      for (int t = 0; t < KT; ++t) prev[t] = float2{0.f, 0.f};
    }
  }

  // ---- mass[a, b] = sum_i e[b][i] * exp2(scale' * (m[b][i] - m_i)) / l_i --------------------------
  store_step(end_step - 1);
  if constexpr (kSplit) {
    if (writer) reinterpret_cast<float2*>(a.share_stats)[(item * shares + share) * Q + mine] = float2{qs.real ? l_row : 0.f, m_run};
    WAIT_VMCNT(0);
    __syncthreads();  // as below: the next item writes the staged tiles
    continue;
  }
  if (writer) {
    lds_inv[mine] = (qs.real && l_row > 0.f) ? 1.0f / l_row : 0.f;  // a padding query adds nothing
    lds_ref[mine] = m_run;
  }
  // The stored pairs are read back by other waves of this workgroup only, which share an L1: waiting for the stores and the
  // barrier's order are enough.  A device-wide fence in every wave writes back the XCD's L2 each time, for all of its
  // workgroups, 0.1 us per group of queries: 12 heads of 12.5K tokens of head dim 64 627 -> 482 us without it, 6 heads of 4K 57 -> 44 us.
  WAIT_VMCNT(0);
  __syncthreads();
  reduce_tiles<B, false>(part, lds_inv, lds_ref, nullptr, w.c2, 0, n, n, a.n - first_row, out);
  __syncthreads();  // the item is done: its ticket and its LDS tables may be overwritten
  }
}

// The last pass over row groups whose key tiles were shared: kMassMergeTiles key tiles of one row group per workgroup.  The
// shares are added in their order, so the result is run-to-run identical.  Bound: latency and the launch.
// Scores without a softmax come out as a single walk leaves them: after an infinity the reference is infinite, which gives
// zeros before its key tile and NaN from there on; a tile of NaN makes the reference NaN, and with it every mass.
template <int B>
__global__ __launch_bounds__(256) void tile_mass_merge_kernel(MassArgs a) {
  constexpr int Q = kMassQueries;
  __shared__ __attribute__((aligned(16))) float lds_inv[Q], lds_ref[Q];
  __shared__ int lds_nan_from[Q / B];
  const int64_t groups = (a.n + Q / B - 1) / (Q / B), item = blockIdx.x;
  const int64_t plane_id = item / groups, first_row = item % groups * (Q / B);
  const int n = (int)a.n, begin = blockIdx.y * kMassMergeTiles;
  const float c2 = a.scale * kLog2e;
  if (threadIdx.x < Q / B) lds_nan_from[threadIdx.x] = n;
  __syncthreads();
  if (threadIdx.x < Q) {
    const float2* stats = reinterpret_cast<const float2*>(a.share_stats) + item * a.shares * Q + threadIdx.x;
    float top = kMinusInf, sum = 0.f;
    for (int s = 0; s < a.shares; ++s) {
      const float2 st = stats[s * Q];
      if (st.x <= 0.f) continue;  // a share without a finite score has no reference of its own
      if (st.y == -kMinusInf && top != st.y) {  // the first infinite one: the walk of the tile's later shares would go on with it
        const int step_tiles = mass_step_keys(B, a.D) / B, steps = (n + step_tiles - 1) / step_tiles;
        atomicMin(&lds_nan_from[threadIdx.x / B], (int)((int64_t)(s + 1) * steps / a.shares) * step_tiles);
      }
      top = st.y > top || st.y != st.y ? st.y : top;
    }
    for (int s = 0; s < a.shares; ++s) sum += stats[s * Q].x * ref_factor((stats[s * Q].y - top) * c2);
    lds_inv[threadIdx.x] = sum > 0.f ? 1.0f / sum : 0.f;
    lds_ref[threadIdx.x] = top;
  }
  __syncthreads();
  reduce_tiles<B, true>(reinterpret_cast<const float2*>(a.partial) + item * a.n * Q, lds_inv, lds_ref, lds_nan_from, c2, begin,
                        min(begin + kMassMergeTiles, n), n, a.n - first_row, a.mass + (plane_id * a.n + first_row) * a.n);
}

template <int B, int D, bool kTokensFirst = false>
hipError_t launch(const MassArgs& a, int64_t items, hipStream_t stream) {
  if constexpr (B == 128 && !kTokensFirst) {
    if (a.tokens_first) return launch<B, D, true>(a, items, stream);
  }
  if (a.shares == 1) {
    hipLaunchKernelGGL((tile_mass_kernel<B, D, false, kTokensFirst>), dim3((unsigned)std::min(items, a.partial_rows)), dim3(256), 0, stream, a);
    return hipGetLastError();
  }
  const int64_t chunks = (a.n + kMassMergeTiles - 1) / kMassMergeTiles;
  if (chunks > 65535 || items > 0x7fffff) return hipErrorInvalidValue;
  hipLaunchKernelGGL((tile_mass_kernel<B, D, true, kTokensFirst>), dim3((unsigned)std::min(items * a.shares, a.places)), dim3(256), 0, stream, a);
  hipLaunchKernelGGL((tile_mass_merge_kernel<B>), dim3((unsigned)items, (unsigned)chunks), dim3(256), 0, stream, a);
  return hipGetLastError();
}

}  // namespace

hipError_t launch_tile_mass(const MassArgs& a, hipStream_t stream) {
  const int64_t items = (int64_t)a.batch * a.num_heads * mass_row_groups(a.n, a.B);
  if (items == 0) return hipSuccess;
  if (!a.partial || !a.counter || a.partial_rows < 1) return hipErrorInvalidValue;
  if (a.shares < 1 || items * a.shares + std::max(a.places, a.partial_rows) > 0x7fffffff) return hipErrorInvalidValue;
  if (a.shares > 1 && (items > a.partial_rows || a.places < 1 || !a.share_stats)) return hipErrorInvalidValue;
  if (a.B == 128 && a.D == 128) return launch<128, 128>(a, items, stream);
  if (a.B == 128 && a.D == 64) return launch<128, 64>(a, items, stream);
  if (a.B == 64 && a.D == 128) return launch<64, 128>(a, items, stream);
  if (a.B == 64 && a.D == 64) return launch<64, 64>(a, items, stream);
  return hipErrorInvalidValue;
}

}  // namespace ca

// Block-sparse attention forward on bf16 MFMA for launches that the one-tile-per-workgroup kernels serve
// badly: few rows or long walks (the card is not filled, or waits for its longest row), and grids whose
// tiles are padded on many sides.  choose_ways in layout.cpp says which launches come here.
//
// A workgroup of NW waves owns 32 * NQ query slots of one row (batch, head, query tile): NQ waves side by
// side hold 32 queries each, and NK = NW / NQ waves (ways) share a group of queries, way kw multiplying
// its share of every stage of keys with an online softmax of its own (QueryWave in attn_bf16_common.h);
// the ways are merged once, through LDS, lane by lane (all ways hold the same queries and channels in the
// same lanes).
//
// What bounds it there is the time of a stage, not a rate: a wave alone on its SIMD takes about 1.1 us for
// the products, the exponentials (two issue slots each) and the waits of 64 keys.  Splitting the keys of a
// stage over four ways and a 128-token tile over two workgroups (NW 8, NQ 2) makes the longest walk about
// twice as short and a full card 1.7 times slower.  Measured, one-tile kernel / NW 4, NQ 4 / NW 8, NQ 4 /
// NW 8, NQ 2: 86 rows of 43 tiles, head dim 128, 92 / 47 / 38 / 33 us; 100 rows of 50 tiles, head dim 64,
// 79 / 64 / - / 38 us; 1107 rows of 128 tokens on a 46 x 59 x 10 grid 883 / 649 / 547 / 797 us; 7680 rows
// on an unpadded grid, head dim 128, 15.9 / 18.0 / 18.9 / 27.8 ms.  (Granules past the end of a walk are not copied;
// copying the last one again took 757 us instead of 547.)
//
// Stages, not tiles.  Keys are staged by LDS DMA in granules of 16 tokens, one per wave and stage, two
// stages in LDS, one barrier per stage.  Only tokens are staged: the slots of a padded tile are taken
// token-holding slots first (class_perm), and a stage is filled from as many consecutive kept tiles as it
// takes.  A granule's rows past its tile's last token are masked by count: K repeats that token there, and V is
// zero, because a weight of zero does not cancel an infinity.  What a padding slot holds is never read.  (Three or four stages in LDS, copies issued after the first
// product phase, and the list's words in a vector register instead of scalar loads all measured the same
// or slower.)
#include "attn_bf16_common.h"

namespace ca {
namespace {

template <int D, int NW, int NQ_>
struct WayShape : Shape<128, D, NW> {
  static constexpr int NQ = NQ_, NK = NW / NQ_;
  static constexpr int kStageKeys = 16 * NW;                 // one 16-token granule per wave
  static constexpr int kKeyBlocks = kStageKeys / 32 / NK;    // 32-key blocks of a stage that one wave multiplies
  static constexpr int kStageBytes = kStageKeys * D * 2;     // of K, and of V
  static constexpr int kRowsPerLoad = 1024 / (D * 2);
  static constexpr int kLoads = 16 / kRowsPerLoad;           // of K, and of V, per wave and stage
  static constexpr int kLeadK = 6, kLeadV = 4;               // 3 - 6 % against the compiler's order at head dim 128
  // Eight waves and a stage of 64 KB.  Copies are asked for after the scores instead of before, because the waves wait for their turn at
  // asking and would start their products late; and a wave without a real query has a loop of its own, without which the
  // compiler copied all of O (64 registers) once a stage in 8x2.  Together, 192 rows of 64 tiles, 8x2, 62.2 / 56.3 us (57.1 with the
  // loop alone), 256 rows of 256 tiles 222 / 199 us (203); nine drawn launches of 8x2 1.09 times, three of 8x4 1.03.  With four waves or half
  // the bytes (head dim 64) neither gains anything (0.98 to 1.03), and the keys' branch stays.
  static constexpr bool kLateCopies = D == 128 && NW == 8;
  static_assert(kKeyBlocks >= 1 && kKeyBlocks * 32 * NK == kStageKeys && NW <= 8, "whole blocks per way, a byte of every granule's count");
};

// Copies a granule that is contiguous in memory (all slots of the tile hold tokens, tile order): the
// instruction offset moves the global and the LDS address together, so one M0 value and one base serve
// all of its loads.
template <int kLoads>
__device__ __forceinline__ void copy_granule(uint32_t m0, const char* base, const uint32_t (&lane_off)[kLoads]) {
  static_assert(kLoads == 2 || kLoads == 4, "16 rows of head dim 64 or 128");
  if constexpr (kLoads == 4) {
    asm volatile(
        "s_mov_b32 m0, %[m0]\n\ts_nop 0\n\t"
        "global_load_lds_dwordx4 %[v0], %[sb] offset:0\n\t"
        "global_load_lds_dwordx4 %[v1], %[sb] offset:1024\n\t"
        "global_load_lds_dwordx4 %[v2], %[sb] offset:2048\n\t"
        "global_load_lds_dwordx4 %[v3], %[sb] offset:3072\n\t"
        :
        : [m0] "s"(m0), [v0] "v"(lane_off[0]), [v1] "v"(lane_off[1]), [v2] "v"(lane_off[2]), [v3] "v"(lane_off[3]), [sb] "s"(base)
        : "memory");
  } else {
    asm volatile(
        "s_mov_b32 m0, %[m0]\n\ts_nop 0\n\t"
        "global_load_lds_dwordx4 %[v0], %[sb] offset:0\n\t"
        "global_load_lds_dwordx4 %[v1], %[sb] offset:1024\n\t"
        :
        : [m0] "s"(m0), [v0] "v"(lane_off[0]), [v1] "v"(lane_off[1]), [sb] "s"(base)
        : "memory");
  }
}

template <int D, int NW, int NQ, bool kNat, bool kSplit>
__global__ __attribute__((amdgpu_flat_work_group_size(NW * 64, NW * 64), amdgpu_waves_per_eu(D == 64 && (NW == 4 || kSplit) ? 4 : 2)))
void attn_bf16_ways_kernel(LaunchArgs<kSplit> a, int parts) {
  using S = WayShape<D, NW, NQ>;
  __shared__ __attribute__((aligned(1024))) char lds[4 * S::kStageBytes];  // K, V of stage 0, K, V of stage 1
  __shared__ float2 lds_stats[S::NK > 1 ? (NW - NQ) * 64 : 1];
  __shared__ uint8_t lds_perm[8 * 128];
  __shared__ int lds_row[kNat ? 128 : 1];  // natural order: row of a video tile's slot, from its first
  __shared__ __attribute__((aligned(16))) uint8_t lds_keys[2][8];

  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int qw = wave % NQ, kw = wave / NQ;
  int64_t batch, row, share = -1;
  int part, first_tile = 0, count;
  if constexpr (kSplit) {
    const LaunchItem it = split_item(a);
    batch = it.batch, row = it.entry, part = it.part, first_tile = it.first, count = it.count, share = it.share;
  } else {
    const int64_t linear = xcd_launch_order(blockIdx.x, gridDim.x, NW == 4 ? xcd_chunk(gridDim.x) : kXcdChunk);  // (batch, launch-order row, part)
    const int64_t rows = (int64_t)a.num_heads * a.n, item = linear / parts % rows;
    part = (int)(linear % parts);
    batch = linear / parts / rows;
    row = a.order ? CONST_PTR(int32_t, a.order)[item] : item;
    count = (int)(a.row_ptr ? CONST_PTR(int64_t, a.row_ptr)[row + 1] - CONST_PTR(int64_t, a.row_ptr)[row] : a.n);
  }
  const int64_t head = row / a.n, q_tile = row - head * a.n;
  const int64_t plane = (batch * a.num_heads + head) * (kNat ? a.N_real : a.n * (int64_t)a.B) * S::kRowBytes;
  const char* Kp = static_cast<const char*>(a.k) + plane;
  const char* Vp = static_cast<const char*>(a.v) + plane;
  const int64_t begin = (a.row_ptr ? CONST_PTR(int64_t, a.row_ptr)[row] : 0) + first_tile;
  const auto meta = CONST_PTR(int32_t, a.col_meta + begin);
  const auto tile_origin = CONST_PTR(int32_t, a.tile_origin);

  // ---- queries --------------------------------------------------------------------------------------
  QueryWave<S> w(lane, a.scale);
  const int first_slot = (part * NQ + qw) * 32;
  const QuerySlot qs = query_slot<128>(a, q_tile, first_slot, w.qi);
  int64_t q_row;
  if constexpr (kNat) {
    q_row = natural_query_row(a, q_tile, qs.slot);
  } else {
    q_row = q_tile * a.B + qs.slot;
  }
  char* out_row = static_cast<char*>(a.out) + plane + q_row * S::kRowBytes;
  // the slots that hold tokens come first: if the workgroup's first holds none, nobody's does
  if (!query_slot<128>(a, q_tile, part * NQ * 32, 0).wave_active) {
    if (kw == 0) w.store(out_row, false, !kNat);
    return;
  }
  for (int e = threadIdx.x; e < a.num_classes * 128; e += NW * 64) lds_perm[e] = a.class_perm[e];
  if constexpr (kNat)
    if (threadIdx.x < 128) {
      const int dx = threadIdx.x % a.tw, run = threadIdx.x / a.tw, dy = run % a.th, dt = run / a.th;
      lds_row[threadIdx.x] = (dt * a.H + dy) * a.W + dx;
    }
  w.load_q(static_cast<const char*>(a.q) + plane + q_row * S::kRowBytes);

  // ---- the walk: this wave's granule of every stage (every NW-th of the row) --------------------------
  const bool padded = a.num_classes > 1 || a.B % S::kStageKeys != 0;  // else every granule is full
  const int tile_granules = a.B >> 4;
  int j = 0, first = 0;
  int32_t word = count > 0 ? meta[0] : 0, word1 = count > 0 ? meta[1] : 0;
  auto tokens_of = [&](int32_t wd) { return (int)((a.class_valid >> (((uint32_t)wd >> 21) & 0x38)) & 0xffu); };
  auto advance = [&](int granules) {
    int left = padded ? (tokens_of(word) - first + 15) >> 4 : tile_granules - (first >> 4);
    while (granules >= left && j + 1 < count) {
      granules -= left;
      first = 0;
      ++j;
      word = word1;
      word1 = meta[j + 1];
      left = padded ? (tokens_of(word) + 15) >> 4 : tile_granules;
    }
    if (granules >= left) {  // past the end: nothing is copied
      granules = left - 1;
      j = count;
    }
    first += 16 * granules;
  };
  const uint32_t lds_addr = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) char*)lds + (uint32_t)(wave * 16 * S::kRowBytes);
  const int my_row = lane / S::kChunksPerRow, my_chunk = lane % S::kChunksPerRow;
  uint32_t k_lane[S::kLoads], v_lane[S::kLoads];  // offsets inside a contiguous KiB block
#pragma unroll
  for (int i = 0; i < S::kLoads; ++i) {
    const int r = i * S::kRowsPerLoad + my_row;  // of the granule; 16 rows do not change the swizzles
    k_lane[i] = (uint32_t)(my_row * S::kRowBytes + ((my_chunk ^ k_swizzle<D>(r)) << 4));
    v_lane[i] = (uint32_t)(my_row * S::kRowBytes + ((my_chunk ^ v_swizzle<D>(r)) << 4));
  }
  auto issue = [&](int buf) {
    const int tile = __builtin_amdgcn_readfirstlane(word) & 0xffffff, cls = (word >> 24) & 7;
    const int last = tokens_of(word) - 1;
    const int tokens = j < count ? min(16, last + 1 - first) : 0;  // of the granule
    char* const v_lds = lds + (buf * 2 + 1) * S::kStageBytes + wave * 16 * S::kRowBytes + lane * 16;
    if (padded && lane == 0) lds_keys[buf][wave] = (uint8_t)tokens;
    if (tokens == 0) {  // past the end
#pragma unroll
      for (int i = 0; i < S::kLoads; ++i) zero_lds16(v_lds + i * 1024);
      return;
    }
    const uint32_t m0 = __builtin_amdgcn_readfirstlane(lds_addr + (uint32_t)(buf * 2 * S::kStageBytes));
    int64_t row0;  // of the tile's slot 0
    bool text = false;
    if constexpr (kNat) {
      row0 = tile_origin[tile];
      text = tile >= a.n_vid;
    } else {
      row0 = (int64_t)tile * a.B;
    }
    const char *kb = Kp + row0 * S::kRowBytes, *vb = Vp + row0 * S::kRowBytes;
    if (!kNat && cls == 0) {
      const int skip = __builtin_amdgcn_readfirstlane(first * S::kRowBytes);
      copy_granule<S::kLoads>(m0, kb + skip, k_lane);
      copy_granule<S::kLoads>(m0 + (uint32_t)S::kStageBytes, vb + skip, v_lane);
    } else {
      int slot[S::kLoads];
#pragma unroll
      for (int i = 0; i < S::kLoads; ++i) {
        slot[i] = first + i * S::kRowsPerLoad + my_row;
        if (cls != 0) slot[i] = lds_perm[cls * 128 + min(slot[i], last)];
        if constexpr (kNat)
          if (!text) slot[i] = lds_row[slot[i]];
      }
#pragma unroll
      for (int i = 0; i < S::kLoads; ++i) {  // k_lane counts my_row from the load's first row: here the slot takes its place
        const uint32_t row_off = (uint32_t)((slot[i] - my_row) * S::kRowBytes);
        copy_rows(m0 + (uint32_t)(i * 1024), kb, row_off + k_lane[i]);
        if (i * S::kRowsPerLoad + my_row < tokens) copy_rows(m0 + (uint32_t)(S::kStageBytes + i * 1024), vb, row_off + v_lane[i]);
        else zero_lds16(v_lds + i * 1024);
      }
    }
  };

  __syncthreads();  // the tables in LDS are complete
  // Tokens of the stage's granules, one byte each.  On a grid without padded tiles all granules are full
  // and the number of stages is known; else each wave publishes the counts of what it copies.
  uint64_t keys = 0;
  int stages_left = (int)(((int64_t)count * a.B + S::kStageKeys - 1) / S::kStageKeys);
  auto landed = [&](int buf) {
    WAIT_VMCNT(0);
    WAIT_LGKMCNT0();
    BARRIER();  // the stage has landed, and every wave is done with the one before it
    if (!padded) {
      keys = --stages_left >= 0 ? 0x1010101010101010ull : 0;
      return;
    }
    const uint2 k2 = *reinterpret_cast<const uint2*>(lds_keys[buf]);
    keys = (uint64_t)__builtin_amdgcn_readfirstlane(k2.x);
    if (NW > 4) keys |= (uint64_t)__builtin_amdgcn_readfirstlane(k2.y) << 32;
  };
  if (count > 0) {
    advance(wave);
    issue(0);
    landed(0);
  }
  if constexpr (S::kLateCopies) {
    if (!qs.wave_active)  // takes part in the copies and barriers only
      for (int buf = 0; (keys & 0xff) != 0; buf ^= 1) {
        advance(NW);
        issue(buf ^ 1);
        landed(buf ^ 1);
      }
  }
  for (int buf = 0; (keys & 0xff) != 0; buf ^= 1) {
    advance(NW);
    if constexpr (!S::kLateCopies) issue(buf ^ 1);
    // this way's granules: 2 * kKeyBlocks bytes; in the last stage they may all be empty
    const uint64_t own = keys >> (16 * S::kKeyBlocks * kw);
    if (S::kLateCopies || (qs.wave_active && (own & 0xff) != 0)) {
      const int share = buf * 2 * S::kStageBytes + kw * S::kKeyBlocks * 32 * S::kRowBytes;
      const LdsTile k_tile = (LdsTile)lds + share, v_tile = k_tile + S::kStageBytes;
      floatx16 acc_s[S::kKeyBlocks];
      w.qk_tile(k_tile, acc_s, true);
      __builtin_amdgcn_sched_barrier(0);  // V fragments requested before the softmax would spill
      if constexpr (S::kLateCopies) {
        issue(buf ^ 1);
        __builtin_amdgcn_sched_barrier(0);
      }
#pragma unroll
      for (int kb = 0; kb < S::kKeyBlocks; ++kb) {
        const int c0 = (int)(own >> (16 * kb)) & 0xff, c1 = (int)(own >> (16 * kb + 8)) & 0xff;
        if (c0 + c1 != 32) mask_granules(acc_s[kb], c0, c1);
      }
      bf16x8 pf[S::kKeyBlocks][2];
      w.softmax(acc_s, pf);
      __builtin_amdgcn_sched_barrier(0);
      w.pv_tile(v_tile, pf, true);
      __builtin_amdgcn_sched_barrier(0);
    }
    landed(buf ^ 1);
  }

  // ---- merge: ways 1 .. NK - 1 hand over (reference, sum, O), way 0 adds them up and stores -----------
  constexpr int kOBytes = 32 * D * 4;
  static_assert((NW - NQ) * kOBytes <= 4 * S::kStageBytes, "the shares fit the stage buffers");
  float ref = w.reference();
  if constexpr (S::NK > 1) {
    __syncthreads();  // the stage buffers are free
    if (kw > 0) {
      const int from = wave - NQ;
      float4* o = reinterpret_cast<float4*>(lds + from * kOBytes);
#pragma unroll
      for (int i = 0; i < S::kDBlocks * 4; ++i)
        o[i * 64 + lane] = float4{w.acc_o[i / 4][i % 4 * 4], w.acc_o[i / 4][i % 4 * 4 + 1], w.acc_o[i / 4][i % 4 * 4 + 2], w.acc_o[i / 4][i % 4 * 4 + 3]};
      lds_stats[from * 64 + lane] = float2{ref, w.l_run};
    }
    __syncthreads();
    if (kw > 0) return;
    float top = ref;
#pragma unroll
    for (int k = 1; k < S::NK; ++k) top = fmaxf(top, lds_stats[((k - 1) * NQ + qw) * 64 + lane].x);
    // a way without a key has weight 0, also where no way has one (top is -inf)
    const float f0 = ref == kMinusInf ? 0.f : __builtin_amdgcn_exp2f((ref - top) * w.c2);
    ref = top;
    w.l_run *= f0;
#pragma unroll
    for (int db = 0; db < S::kDBlocks; ++db) w.acc_o[db] *= f0;
#pragma unroll 1
    for (int k = 1; k < S::NK; ++k) {
      const int from = (k - 1) * NQ + qw;
      const float2 st = lds_stats[from * 64 + lane];
      const float f = st.x == kMinusInf ? 0.f : __builtin_amdgcn_exp2f((st.x - top) * w.c2);
      w.l_run += st.y * f;
      const float4* o = reinterpret_cast<const float4*>(lds + from * kOBytes);
#pragma unroll
      for (int i = 0; i < S::kDBlocks * 4; ++i) {
        const float4 x = o[i * 64 + lane];
        w.acc_o[i / 4][i % 4 * 4 + 0] += x.x * f;
        w.acc_o[i / 4][i % 4 * 4 + 1] += x.y * f;
        w.acc_o[i / 4][i % 4 * 4 + 2] += x.z * f;
        w.acc_o[i / 4][i % 4 * 4 + 3] += x.w * f;
      }
    }
  }
  if constexpr (kSplit) {
    if (share >= 0) {
      if (qs.wave_active) w.store_share(a, share * NQ + qw, lane, ref);
      return;
    }
  }
  w.store(out_row, qs.real, !kNat || qs.real);
}

template <int D, int NW, int NQ>
hipError_t launch(const SplitArgs& a, hipStream_t stream) {
  const int parts = a.B / (32 * NQ);
  const int64_t entries = a.items ? a.num_items : (int64_t)a.num_heads * a.n * parts;
  const int64_t workgroups = a.batch * entries;
  if (parts < 1 || workgroups > 0xffffffffll / (NW * 64)) return hipErrorInvalidValue;
  const dim3 grid((unsigned)workgroups), block(NW * 64);
  if (a.items) {
    const auto kernel = a.natural ? attn_bf16_ways_kernel<D, NW, NQ, true, true> : attn_bf16_ways_kernel<D, NW, NQ, false, true>;
    hipLaunchKernelGGL(kernel, grid, block, 0, stream, a, parts);
  } else {
    const auto kernel = a.natural ? attn_bf16_ways_kernel<D, NW, NQ, true, false> : attn_bf16_ways_kernel<D, NW, NQ, false, false>;
    hipLaunchKernelGGL(kernel, grid, block, 0, stream, static_cast<const AttnArgs&>(a), parts);
  }
  return hipGetLastError();
}

}  // namespace

hipError_t launch_attn_bf16_ways(const SplitArgs& a, hipStream_t stream) {
  if ((int64_t)a.batch * a.num_heads * a.n == 0) return hipSuccess;
  if (a.num_classes < 1 || a.num_classes > 8) return hipErrorInvalidValue;
  if (a.D == 128 && a.ways == kWays4x4) return launch<128, 4, 4>(a, stream);
  if (a.D == 128 && a.ways == kWays8x4) return launch<128, 8, 4>(a, stream);
  if (a.D == 128 && a.ways == kWays8x2) return launch<128, 8, 2>(a, stream);
  if (a.D == 64 && a.ways == kWays4x4) return launch<64, 4, 4>(a, stream);
  if (a.D == 64 && a.ways == kWays8x2) return launch<64, 8, 2>(a, stream);
  return hipErrorInvalidValue;
}

}  // namespace ca

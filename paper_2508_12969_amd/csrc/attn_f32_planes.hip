// Block-sparse attention forward in fp32 on the bf16 matrix instructions: every fp32 operand is the sum of three
// bf16 values, and a product is the six partial products that reach 2^-24 of it, summed in fp32.
//
// Why: the f32 matrix instructions, on which attn_f32.hip runs, do 1/16 of the bf16 rate; six bf16 products per
// fp32 one are 2.7 times as fast.
//
// The split.  a = a1 + a2 + a3 with a1 the bf16 value nearest to a, a2 the one nearest to a - a1 and a3 the rest, at most 2^-8
// and 2^-17 of the power of two below a: 24 bits, which is all of a.  (Three-way bf16 splits: Henry, Tang, Heinecke, Leveraging
// the bfloat16 artificial intelligence datatype for higher-precision computations, ARITH 2019.)  Left out of a product are
// a2 b3, a3 b2 and a3 b3, at most 2^-24 of it and of either sign; with parts cut off instead of rounded it would be 2^-21,
// always to the same side.
// What is split is multiplied by 2^24 first, so that the parts of small values, subnormals included, hold all of their bits too.
// Infinities, NaN and values from 2^96 on are NaN in all three parts; queries whose sums are infinite or NaN, which
// they also become by V above about 2^60 and products of q and k above 2^79, are walked a second time, on the f32 matrix instructions.
//
// K and V are split once per call by a kernel of their own, into a workspace, as "units" of 16 tokens in
// the order in which the matrix instructions read them; the slots of a padded tile are taken token-holding slots
// first, and a unit's rows past its tile's last token are zero.  So the attention kernel copies plain blocks of memory
// (LDS DMA) and reads LDS in plain 16-byte rows: no gather, no swizzle, no transposing read.  Queries and
// probabilities are split in registers.
//
// Decomposition.  A way is two waves that hold 32 queries each, and a workgroup has NK ways for the same 64 query
// slots, way kw taking every NK-th stage of two units (32 keys) with an online softmax of its own; the ways are merged once,
// through LDS.  A way has room for three units in LDS (36 KB at head dim 128, so four ways fit a CU, two waves per
// SIMD): K of both units and V of the first; V of the second takes the place of K's first unit, and so on round, so that every copy
// is under way while one of the three product phases of a stage (scores, and 16 keys of O at a time) runs.  At head dims 32 and 64
// there is room for V of both units and a stage has two phases.
//
// What bounds it: the bf16 matrix instructions.  Measured, attn_f32.hip / this with the split of K and V: 8 heads of 8K tokens,
// dense, head dim 128 2.47 / 1.38 ms (1200 TFLOP/s of bf16 products), 64 1.29 / 0.73 ms, 32 0.65 / 0.42 ms; 8 heads of 7K tokens, head
// dim 128, 1128 rows of unequal length 1.18 / 0.64 ms (of which the split takes 0.026; 0.72 with launches of few rounds dealt in chunks of 64, see xcd_chunk); 1 head of 1.9K 115 / 80 us.  Four ways and
// one wave of queries (1x4) make the walk of a small launch shortest, two and two a full card fastest (choose_planes in layout.cpp).
#include <algorithm>
#include <type_traits>

#include "attn_bf16_common.h"

namespace ca {
namespace {

typedef __attribute__((ext_vector_type(4))) float f32x4;
typedef __attribute__((ext_vector_type(4))) uint32_t u32x4;
constexpr float kTop = 0x1p96f;             // operands from here on go the second way
constexpr float kLift = 0x1p24f;            // what is split is multiplied by this: third parts of the smallest values are no subnormals
constexpr float kDropScores = 0x1p-48f;     // and what comes of it by one of these
constexpr float kDropResult = 0x1p-24f;

template <int D>
struct UnitShape {
  static constexpr int kPlaneBytes = 16 * D * 2;        // one of the three parts of 16 rows
  static constexpr int kBytes = 3 * kPlaneBytes;        // of K, and of V behind it
  static constexpr int kLoads = kBytes / 1024;          // wave-wide 16-byte copies
  static constexpr int kPlaces = D == 128 ? 3 : 4;      // units that a way has room for
  static constexpr int kSteps = D / 16;                 // contraction steps of the scores
  static constexpr int kDBlocks = D / 32;
};

// Parts of two values, packed for the matrix instructions: word i holds part i + 1 of `even` below that of `odd`.
// kAnyValue: operands; else weights, which are 0 to 2^kLazyLog2, or NaN, and already multiplied by kLift.
template <bool kAnyValue>
__device__ __forceinline__ void split_pair(float even, float odd, uint32_t (&word)[3]) {
  if constexpr (kAnyValue) {
    even = fabsf(even) < kTop ? even * kLift : __builtin_nanf("");
    odd = fabsf(odd) < kTop ? odd * kLift : __builtin_nanf("");
  }
#pragma unroll
  for (int p = 0; p < 3; ++p) {
    word[p] = __builtin_bit_cast(uint32_t, bf16x2{(__bf16)even, (__bf16)odd});  // to nearest
    even -= __builtin_bit_cast(float, word[p] << 16);
    odd -= __builtin_bit_cast(float, word[p] & 0xffff0000u);
  }
}

// ---- K and V to units ---------------------------------------------------------------------------------
// One workgroup per unit, bound by memory: 4 bytes read and 6 written per element.  K part: [part][step of 16
// channels][half of 8 channels][key] and V part: [part][32-channel block][half of the keys][channel], 16 bytes each:
// eight channels of a key, or a channel of keys 4 h .. + 3 and 8 + 4 h .. + 3 (the keys whose scores a lane holds).
template <int D>
__global__ __attribute__((amdgpu_flat_work_group_size(2 * D, 2 * D)))
void split_units_kernel(AttnArgs a, char* units, int tile_units, int64_t total) {
  using U = UnitShape<D>;
  constexpr int kThreads = 2 * D, kRow = D + 4;  // floats; a row of LDS starts four banks on
  __shared__ __attribute__((aligned(16))) float lds[2 * 16 * kRow];
  const int64_t id = (int64_t)blockIdx.y * gridDim.x + blockIdx.x;
  if (id >= total) return;
  const int u = (int)(id % tile_units);
  const int64_t plane_tile = id / tile_units;  // (batch, head) plane * n + tile
  const int cls = CONST_PTR(int32_t, a.tile_class)[plane_tile % a.n];
  const int valid = (int)((a.class_valid >> (8 * cls)) & 0xffu);
  if (16 * u >= valid) return;
#pragma unroll
  for (int i = 0; i < 2; ++i) {
    const int e = threadIdx.x + i * kThreads, row = e / (D / 4), chunk = e % (D / 4), pos = 16 * u + row;
    f32x4 k = {0.f, 0.f, 0.f, 0.f}, v = k;
    if (pos < valid) {
      const int64_t at = (plane_tile * a.B + a.class_perm[cls * 128 + pos]) * D + chunk * 4;
      k = *reinterpret_cast<const f32x4*>(static_cast<const float*>(a.k) + at);
      v = *reinterpret_cast<const f32x4*>(static_cast<const float*>(a.v) + at);
    }
    *reinterpret_cast<f32x4*>(lds + row * kRow + chunk * 4) = k;
    *reinterpret_cast<f32x4*>(lds + (16 + row) * kRow + chunk * 4) = v;
  }
  __syncthreads();
  const int c = threadIdx.x;
  char* const out = units + id * 2 * U::kBytes + c * 16;
  float k[8], v[8];
#pragma unroll
  for (int i = 0; i < 8; ++i) {
    k[i] = lds[c % 16 * kRow + c / 16 * 8 + i];
    v[i] = lds[(16 + i / 4 * 8 + c / 32 % 2 * 4 + i % 4) * kRow + c / 64 * 32 + c % 32];
  }
  u32x4 kp[3], vp[3];
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    uint32_t word[3];
    split_pair<true>(k[2 * i], k[2 * i + 1], word);
#pragma unroll
    for (int p = 0; p < 3; ++p) kp[p][i] = word[p];
    split_pair<true>(v[2 * i], v[2 * i + 1], word);
#pragma unroll
    for (int p = 0; p < 3; ++p) vp[p][i] = word[p];
  }
#pragma unroll
  for (int p = 0; p < 3; ++p) {
    *reinterpret_cast<u32x4*>(out + p * U::kPlaneBytes) = kp[p];
    *reinterpret_cast<u32x4*>(out + U::kBytes + p * U::kPlaneBytes) = vp[p];
  }
}

// Five of the six products of (a1 + a2 + a3) (b1 + b2 + b3), the small ones first; a1 b1 is the sixth.
__device__ __forceinline__ floatx16 small_products(const bf16x8 (&a)[3], const bf16x8 (&b)[3], floatx16 acc) {
  acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[2], b[0], acc, 0, 0, 0);
  acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[1], b[1], acc, 0, 0, 0);
  acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[0], b[2], acc, 0, 0, 0);
  acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[1], b[0], acc, 0, 0, 0);
  return __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[0], b[1], acc, 0, 0, 0);
}
__device__ __forceinline__ floatx16 zeros() {
  floatx16 x;
#pragma unroll
  for (int r = 0; r < 16; ++r) x[r] = 0.f;
  return x;
}

// Copies kLoads consecutive KiB, or one less; the instruction offset moves the global and the LDS address together.
template <int kLoads, bool kEven>
__device__ __forceinline__ void copy_blocks(uint32_t m0, const char* base, uint32_t lane_off, bool all) {
#pragma unroll
  for (int i = 0; i < kLoads; i += 4) {
    const uint32_t m = m0 + (uint32_t)i * 1024;
    const char* const b = base + i * 1024;
    constexpr int kGroup = 4;
    if (kLoads - i >= kGroup) {
      asm volatile(
          "s_mov_b32 m0, %[m0]\n\ts_nop 0\n\t"
          "global_load_lds_dwordx4 %[v], %[sb] offset:0\n\t"
          "global_load_lds_dwordx4 %[v], %[sb] offset:1024\n\t"
          "global_load_lds_dwordx4 %[v], %[sb] offset:2048\n\t"
          "global_load_lds_dwordx4 %[v], %[sb] offset:3072\n\t"
          :
          : [m0] "s"(m), [v] "v"(lane_off), [sb] "s"(b)
          : "memory");
    } else if (kLoads - i == 3) {
      asm volatile(
          "s_mov_b32 m0, %[m0]\n\ts_nop 0\n\t"
          "global_load_lds_dwordx4 %[v], %[sb] offset:0\n\t"
          "global_load_lds_dwordx4 %[v], %[sb] offset:1024\n\t"
          "global_load_lds_dwordx4 %[v], %[sb] offset:2048\n\t"
          :
          : [m0] "s"(m), [v] "v"(lane_off), [sb] "s"(b)
          : "memory");
    } else if (kEven || all) {
      asm volatile(
          "s_mov_b32 m0, %[m0]\n\ts_nop 0\n\t"
          "global_load_lds_dwordx4 %[v], %[sb] offset:0\n\t"
          "global_load_lds_dwordx4 %[v], %[sb] offset:1024\n\t"
          :
          : [m0] "s"(m), [v] "v"(lane_off), [sb] "s"(b)
          : "memory");
    } else {
      copy_rows(m, b, lane_off);
    }
  }
}

// A place in the walk over the units of a row (wave-uniform).
struct UnitCursor {
  int j, unit, over;     // tile of the list, unit of it; over: units past the end of the row, -1 inside
  int valid;             // tokens of the tile
  int32_t word, word1;   // of this tile and the next
};

template <int D, int QN, int NK>
__global__ __attribute__((amdgpu_flat_work_group_size(64 * QN * NK, 64 * QN * NK), amdgpu_waves_per_eu(2)))
void attn_f32_planes_kernel(AttnArgs a, const char* units, int tile_units, int parts, int64_t workgroups) {
  using U = UnitShape<D>;
  constexpr int kMine = (U::kLoads + QN - 1) / QN;  // of a unit's copies one wave issues this many (or one less)
  __shared__ __attribute__((aligned(1024))) char lds[NK * U::kPlaces * U::kBytes];
  __shared__ float2 lds_stats[(NK - 1) * QN * 64];
  __shared__ int lds_again[QN];

  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int qw = wave % QN, kw = wave / QN;
  const int qi = lane & 31, g = lane >> 5;
  const int64_t id = (int64_t)blockIdx.y * gridDim.x + blockIdx.x;
  if (id >= workgroups) return;
  const int64_t linear = xcd_launch_order(id, workgroups, xcd_chunk(workgroups));
  const int64_t rows = (int64_t)a.num_heads * a.n;
  const int part = (int)(linear % parts);
  const int64_t item = (linear / parts) % rows, batch = linear / parts / rows;
  const int64_t row = a.order ? CONST_PTR(int32_t, a.order)[item] : item;
  const int64_t head = row / a.n, q_tile = row - head * a.n;
  const int64_t plane_tiles = (batch * a.num_heads + head) * a.n;
  const char* plane_units = units + plane_tiles * tile_units * (2 * U::kBytes);
  const int64_t tile_at = (plane_tiles + q_tile) * a.B * (int64_t)(D * 4);
  const int64_t begin = a.row_ptr ? CONST_PTR(int64_t, a.row_ptr)[row] : 0;
  const int count = (int)(a.row_ptr ? CONST_PTR(int64_t, a.row_ptr)[row + 1] - begin : a.n);
  const auto meta = CONST_PTR(int32_t, a.col_meta + begin);

  // ---- queries: positions of the tile's token order; a position past the tile has no row of the output -----
  const int q_cls = CONST_PTR(int32_t, a.tile_class)[q_tile];
  const int q_valid = (int)((a.class_valid >> (8 * q_cls)) & 0xffu);
  const int q_pos = (part * QN + qw) * 32 + qi;
  const bool q_in = q_pos < a.B;
  const int q_slot = a.class_perm[q_cls * 128 + (q_in ? q_pos : 0)];
  const bool wave_active = (part * QN + qw) * 32 < q_valid;
  char* const out_row = static_cast<char*>(a.out) + tile_at + (int64_t)q_slot * (D * 4);
  if (part * QN * 32 >= q_valid) {  // padding slots only: zero rows
    if (kw == 0 && q_in)
#pragma unroll
      for (int i = 0; i < D / 8; ++i) *reinterpret_cast<f32x4*>(out_row + (2 * i + g) * 16) = f32x4{0.f, 0.f, 0.f, 0.f};
    return;
  }
  bf16x8 qf[U::kSteps][3];  // B operand of S^T: the lane's query, channels 16 s + 8 g .. + 7
  {
    const char* const q_row = static_cast<const char*>(a.q) + tile_at + (int64_t)q_slot * (D * 4) + g * 32;
#pragma unroll
    for (int s = 0; s < U::kSteps; ++s) {
      const f32x4 x[2] = {*reinterpret_cast<const f32x4*>(q_row + s * 64), *reinterpret_cast<const f32x4*>(q_row + s * 64 + 16)};
      u32x4 w[3];
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        uint32_t word[3];
        split_pair<true>(x[i / 2][2 * (i % 2)], x[i / 2][2 * (i % 2) + 1], word);
#pragma unroll
        for (int p = 0; p < 3; ++p) w[p][i] = word[p];
      }
#pragma unroll
      for (int p = 0; p < 3; ++p) {
        qf[s][p] = __builtin_bit_cast(bf16x8, w[p]);
        asm volatile("" : "+v"(qf[s][p]));  // waited for here: in the loop the counter belongs to the copies
      }
    }
  }
  floatx16 acc_o[U::kDBlocks];
#pragma unroll
  for (int db = 0; db < U::kDBlocks; ++db)
#pragma unroll
    for (int r = 0; r < 16; ++r) acc_o[db][r] = 0.f;
  const float c2 = a.scale * kLog2e * kDropScores;
  float ref = -1e30f, l_run = 0.f;  // exponent reference of the query in log2 units; this lane's share of its row sum

  // ---- the walk ----------------------------------------------------------------------------------------
  auto tokens_of = [&](int32_t word) { return (int)((a.class_valid >> (((uint32_t)word >> 21) & 0x38)) & 0xffu); };
  auto advance = [&](UnitCursor& c, int by) {
    if (c.over >= 0) {
      c.over += by;
      return;
    }
    c.unit += by;
    while (16 * c.unit >= c.valid) {
      const int past = c.unit - ((c.valid + 15) >> 4);
      if (c.j + 1 >= count) {
        c.over = past;
        return;
      }
      c.unit = past;
      ++c.j;
      c.word = c.word1;
      c.word1 = meta[c.j + 1];
      c.valid = tokens_of(c.word);
    }
  };
  auto tokens_at = [&](const UnitCursor& c) { return c.over >= 0 ? 0 : min(16, c.valid - 16 * c.unit); };
  auto address = [&](const UnitCursor& c) { return plane_units + ((int64_t)(c.word & 0xffffff) * tile_units + c.unit) * (2 * U::kBytes); };

  const uint32_t lds_addr = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) char*)lds + (uint32_t)(kw * U::kPlaces * U::kBytes);
  const LdsTile lds_way = (LdsTile)lds + kw * U::kPlaces * U::kBytes;
  const uint32_t lane_off = (uint32_t)lane * 16;
  auto copy = [&](const char* from, int place) {  // this wave's share of a unit of K or of V
    const int first = qw * kMine * 1024;
    copy_blocks<kMine, U::kLoads % QN == 0>(lds_addr + (uint32_t)(place + first), from + first, lane_off, qw * kMine + kMine <= U::kLoads);
  };
  auto landed = [&](bool later) {  // later: one more unit has been asked for since
    if (later) WAIT_VMCNT(U::kLoads / QN);
    else WAIT_VMCNT(0);
    WAIT_LGKMCNT0();
    BARRIER();
  };
  auto fragments = [&](LdsTile at, bf16x8 (&f)[3]) {
#pragma unroll
    for (int p = 0; p < 3; ++p) f[p] = *reinterpret_cast<const __attribute__((address_space(3))) bf16x8*>(at + p * U::kPlaneBytes);
  };
  // O^T += V^T P^T for 16 keys, or 32.  The matrix instructions cut what they add to a larger sum, and always to the same side:
  // one sum over the whole walk was off by 2e-6 after 7K keys (5e-7 in attn_f32.hip), sums of their own, small products first, by
  // 2e-7, for 5 % of the time.  Likewise the five small products of the scores have a sum of their own.
  auto add_values = [&](auto two, const bf16x8 (&pf)[2][3], int t, int place) {
#pragma unroll
    for (int db = 0; db < U::kDBlocks; ++db) {
      bf16x8 vf[2][3];
      fragments(lds_way + place + db * 1024 + lane * 16, vf[0]);
      floatx16 sum = small_products(vf[0], pf[t], zeros());
      if constexpr (two()) {
        fragments(lds_way + place + U::kBytes + db * 1024 + lane * 16, vf[1]);
        sum = small_products(vf[1], pf[1], sum);
      }
      sum = __builtin_amdgcn_mfma_f32_32x32x16_bf16(vf[0][0], pf[t][0], sum, 0, 0, 0);
      if constexpr (two()) sum = __builtin_amdgcn_mfma_f32_32x32x16_bf16(vf[1][0], pf[1][0], sum, 0, 0, 0);
#pragma unroll
      for (int r = 0; r < 16; ++r) acc_o[db][r] += sum[r];
    }
  };

  // at: the first unit of this way's stage; of the second, k1 tokens and the address of K are kept
  UnitCursor at{0, 0, count > 0 ? -1 : 0, 0, count > 0 ? meta[0] : 0, count > 0 ? meta[1] : 0};
  at.valid = tokens_of(at.word);
  advance(at, 2 * kw);
  int k0 = tokens_at(at);
  const char* u0 = address(at);
  bool more = at.over < 2 * kw;  // way 0, the first to start a round of stages, still has one
  advance(at, 1);
  int k1 = tokens_at(at);
  const char* u1 = address(at);
  int pa = 0, pb = U::kBytes, pc = 2 * U::kBytes;  // places: K of the two units, V
  if (k0 > 0) copy(u0, pa);
  if (k1 > 0) copy(u1, pb);
  landed(false);
  if (k0 > 0) copy(u0 + U::kBytes, pc);
  if (U::kPlaces == 4 && k1 > 0) copy(u1 + U::kBytes, 3 * U::kBytes);
  while (more) {
    advance(at, 2 * NK - 1);
    const int next0 = tokens_at(at);
    const char* const v1 = address(at);
    more = at.over < 2 * kw;
    advance(at, 1);
    const int next1 = tokens_at(at);
    const char* const w1 = address(at);

    const bool work = wave_active && k0 > 0;
    bf16x8 pf[2][3];
    if (work) {
      floatx16 sc = zeros(), small = zeros();
      const LdsTile k_row = lds_way + (qi < 16 ? pa : pb) + g * 256 + (qi & 15) * 16;
#pragma unroll
      for (int s = 0; s < U::kSteps; ++s) {
        bf16x8 kf[3];
        fragments(k_row + s * 512, kf);
        small = small_products(kf, qf[s], small);
        sc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kf[0], qf[s][0], sc, 0, 0, 0);
      }
#pragma unroll
      for (int r = 0; r < 16; ++r) sc[r] += small[r];
      if (k0 + k1 != 32) mask_granules(sc, k0, k1);
      // ---- online softmax; the reference follows the running maximum with a lag of 2^kLazyLog2 at most
      float mx = sc[0];
#pragma unroll
      for (int r = 1; r < 16; ++r) mx = fmaxf(mx, sc[r]);
      mx = max_with_partner(mx);
      if (__any(mx * c2 > ref + kLazyLog2)) {
        const float ref_new = fmaxf(ref, mx * c2), alpha = __builtin_amdgcn_exp2f(ref - ref_new);
        l_run *= alpha;
#pragma unroll
        for (int db = 0; db < U::kDBlocks; ++db)
#pragma unroll
          for (int r = 0; r < 16; ++r) acc_o[db][r] *= alpha;
        ref = ref_new;
      }
#pragma unroll
      for (int t = 0; t < 2; ++t) {
        u32x4 w[3];
        float sum[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const float p0 = kLift * __builtin_amdgcn_exp2f(fmaf(sc[8 * t + 2 * i], c2, -ref)), p1 = kLift * __builtin_amdgcn_exp2f(fmaf(sc[8 * t + 2 * i + 1], c2, -ref));
          sum[i] = p0 + p1;
          uint32_t word[3];
          split_pair<false>(p0, p1, word);
#pragma unroll
          for (int p = 0; p < 3; ++p) w[p][i] = word[p];
        }
#pragma unroll
        for (int p = 0; p < 3; ++p) pf[t][p] = __builtin_bit_cast(bf16x8, w[p]);
        l_run += (sum[0] + sum[1]) + (sum[2] + sum[3]);
      }
    }
    landed(false);  // V (of the first unit); the places of K are free
    if constexpr (U::kPlaces == 4) {
      if (next0 > 0) copy(v1, pa);
      if (next1 > 0) copy(w1, pb);
      if (work && k1 > 0) add_values(std::true_type{}, pf, 0, pc);
      else if (work) add_values(std::false_type{}, pf, 0, pc);
      landed(false);  // K of the next stage; the places of V are free
      if (next0 > 0) copy(v1 + U::kBytes, pc);
      if (next1 > 0) copy(w1 + U::kBytes, 3 * U::kBytes);
    } else {
      if (k1 > 0) copy(u1 + U::kBytes, pa);
      if (work) add_values(std::false_type{}, pf, 0, pc);
      if (next0 > 0) copy(v1, pb);  // after the products: 1.02 times (0.99 to 1.03) before them, where waves wait for their turn at asking
      landed(next0 > 0);  // V of the second; the first one's place is free
      if (next1 > 0) copy(w1, pc);
      if (work && k1 > 0) add_values(std::false_type{}, pf, 1, pa);
      landed(false);  // K of the next stage; the place of V is free
      if (next0 > 0) copy(v1 + U::kBytes, pa);
      const int free_place = pa;
      pa = pb;
      pb = pc;
      pc = free_place;
    }
    k0 = next0;
    k1 = next1;
    u1 = w1;
  }

  // ---- merge of the ways: all hold the same queries and channels in the same lanes; way 0 gets the sums ------
  auto merge = [&] {
    if constexpr (NK > 1) {
      constexpr int kOBytes = 32 * D * 4;
      static_assert((NK - 1) * QN * kOBytes <= NK * U::kPlaces * U::kBytes, "the shares fit the places of the units");
      __syncthreads();
      if (kw > 0) {
        f32x4* const o = reinterpret_cast<f32x4*>(lds + (wave - QN) * kOBytes);
#pragma unroll
        for (int i = 0; i < U::kDBlocks * 4; ++i)
          o[i * 64 + lane] = f32x4{acc_o[i / 4][i % 4 * 4], acc_o[i / 4][i % 4 * 4 + 1], acc_o[i / 4][i % 4 * 4 + 2], acc_o[i / 4][i % 4 * 4 + 3]};
        lds_stats[(wave - QN) * 64 + lane] = float2{ref, l_run};
      }
      __syncthreads();
      if (kw > 0) return;
      float top = ref;
#pragma unroll
      for (int k = 1; k < NK; ++k) top = fmaxf(top, lds_stats[((k - 1) * QN + qw) * 64 + lane].x);
      const float own = __builtin_amdgcn_exp2f(ref - top);
      l_run *= own;
#pragma unroll
      for (int db = 0; db < U::kDBlocks; ++db)
#pragma unroll
        for (int r = 0; r < 16; ++r) acc_o[db][r] *= own;
#pragma unroll 1
      for (int k = 1; k < NK; ++k) {
        const int from = (k - 1) * QN + qw;
        const float2 st = lds_stats[from * 64 + lane];
        const float f = __builtin_amdgcn_exp2f(st.x - top);
        l_run += st.y * f;
        const f32x4* const o = reinterpret_cast<const f32x4*>(lds + from * kOBytes);
#pragma unroll
        for (int i = 0; i < U::kDBlocks * 4; ++i) {
          const f32x4 x = o[i * 64 + lane];
#pragma unroll
          for (int e = 0; e < 4; ++e) acc_o[i / 4][i % 4 * 4 + e] += x[e] * f;
        }
      }
    }
  };
  const bool real = q_pos < q_valid;  // a padding row is zero whatever its sums are
  auto store = [&](float l, float drop) {
    const float inv = l > 0.f ? 1.0f / l * drop : 0.f;
#pragma unroll
    for (int i = 0; i < U::kDBlocks * 4; ++i) {  // channels 32 db + 8 r4 + 4 g .. + 3
      f32x4 o;
#pragma unroll
      for (int e = 0; e < 4; ++e) o[e] = real ? acc_o[i / 4][i % 4 * 4 + e] * inv : 0.f;
      *reinterpret_cast<f32x4*>(out_row + (8 * i + 4 * g) * 4) = o;
    }
  };
  merge();
  bool again = false;  // this query did not come out finite, see the second walk
  if (kw == 0) {
    const float l = sum_with_partner(l_run);
    float z = 0.f * l;  // NaN if the sum or a channel is infinite or NaN
#pragma unroll
    for (int db = 0; db < U::kDBlocks; ++db)
#pragma unroll
      for (int r = 0; r < 16; ++r) z = fmaf(acc_o[db][r], 0.f, z);
    again = real && count > 0 && !(sum_with_partner(z) == 0.f && l > 0.f);
    const bool any = __any(again);
    if (lane == 0) lds_again[qw] = any;
    if (q_in) store(l, kDropResult);
  }
  __syncthreads();
  bool once_more = false;
#pragma unroll
  for (int i = 0; i < QN; ++i) once_more = once_more || lds_again[i];
  if (!once_more) return;

  // ---- second walk: queries whose sums are infinite, NaN or zero, on the f32 matrix instructions -------------
  // What six partial products and a lagging reference cannot do as fp32 does it ends in such sums: an infinity, which would meet parts
  // that are zero or of the other sign, and V near the top of the range times a weight above one.  So infinities and NaN are
  // where attn_f32.hip has them.  Operands come straight from memory: 8 heads of 7K tokens, head dim 128, 0.75 ms
  // without such queries, 1.8 with one, 3.7 if all are (1.22 in attn_f32.hip; in one run); the check costs nothing (638 / 639 us).
  {
    const bool mine = lds_again[qw];
    const char* const plane_k = static_cast<const char*>(a.k) + plane_tiles * a.B * (int64_t)(D * 4);
    const char* const plane_v = static_cast<const char*>(a.v) + plane_tiles * a.B * (int64_t)(D * 4);
    const float* const q_row = reinterpret_cast<const float*>(static_cast<const char*>(a.q) + tile_at + (int64_t)q_slot * (D * 4)) + g * (D / 2);
    const float c2_plain = a.scale * kLog2e;
    ref = -1e30f;
    l_run = 0.f;
#pragma unroll
    for (int db = 0; db < U::kDBlocks; ++db) acc_o[db] = zeros();
    int turn = 0;
#pragma unroll 1
    for (int j = 0; j < count; ++j) {
      const int32_t word = meta[j];
      const int valid = tokens_of(word);
      const int64_t tile_bytes = (int64_t)(word & 0xffffff) * a.B * (D * 4);
      const uint8_t* const perm = a.class_perm + (((uint32_t)word >> 24) & 7) * 128;
#pragma unroll 1
      for (int first = 0; first < valid; first += 32, turn = turn + 1 < NK ? turn + 1 : 0) {
        if (turn != kw || !mine) continue;
        const int keys = min(32, valid - first);
        floatx16 sc = zeros();
        const float* const k_row = reinterpret_cast<const float*>(plane_k + tile_bytes + (int64_t)perm[first + min(qi, keys - 1)] * (D * 4)) + g * (D / 2);
#pragma unroll 2
        for (int c = 0; c < D / 2; c += 4) {
          const f32x4 kf = *reinterpret_cast<const f32x4*>(k_row + c), qx = *reinterpret_cast<const f32x4*>(q_row + c);
#pragma unroll
          for (int e = 0; e < 4; ++e) sc = __builtin_amdgcn_mfma_f32_32x32x2f32(kf[e], qx[e], sc, 0, 0, 0);
        }
        float mx = kMinusInf;
#pragma unroll
        for (int r = 0; r < 16; ++r) {
          sc[r] = r / 4 * 8 + 4 * g + r % 4 < keys ? sc[r] : kMinusInf;
          mx = fmaxf(mx, sc[r]);
        }
        const float ref_new = fmaxf(ref, max_with_partner(mx) * c2_plain), alpha = __builtin_amdgcn_exp2f(ref - ref_new);
        if (__any(ref_new > ref)) {
          l_run *= alpha;
#pragma unroll
          for (int db = 0; db < U::kDBlocks; ++db)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc_o[db][r] *= alpha;
          ref = ref_new;
        }
#pragma unroll
        for (int r = 0; r < 16; ++r) {
          const int key = r / 4 * 8 + 4 * g + r % 4;
          const float p = __builtin_amdgcn_exp2f(fmaf(sc[r], c2_plain, -ref));
          l_run += p;
          const float* const v_row = reinterpret_cast<const float*>(plane_v + tile_bytes + (int64_t)perm[first + min(key, keys - 1)] * (D * 4)) + qi;
#pragma unroll
          for (int db = 0; db < U::kDBlocks; ++db)
            acc_o[db] = __builtin_amdgcn_mfma_f32_32x32x2f32(key < keys ? v_row[32 * db] : 0.f, p, acc_o[db], 0, 0, 0);
        }
      }
    }
    merge();
    if (kw > 0) return;
    const float l = sum_with_partner(l_run);
    if (again) store(l, 1.f);
  }
}

dim3 grid_of(int64_t workgroups) {
  const int64_t width = std::min(workgroups, (int64_t)1 << 23);  // a grid dimension holds fewer than 2^32 threads
  return dim3((unsigned)width, (unsigned)((workgroups + width - 1) / width));
}

template <int D, int QN, int NK>
hipError_t launch(const AttnArgs& a, char* units, hipStream_t stream) {
  const int tile_units = (a.B + 15) / 16, parts = (a.B + 32 * QN - 1) / (32 * QN);
  const int64_t rows = (int64_t)a.batch * a.num_heads * a.n, total = rows * tile_units, workgroups = rows * parts;
  if (total > (int64_t)1 << 38) return hipErrorInvalidValue;
  hipLaunchKernelGGL((split_units_kernel<D>), grid_of(total), dim3(2 * D), 0, stream, a, units, tile_units, total);
  const hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL((attn_f32_planes_kernel<D, QN, NK>), grid_of(workgroups), dim3(64 * QN * NK), 0, stream, a, units, tile_units, parts, workgroups);
  return hipGetLastError();
}

template <int D>
hipError_t launch(const PlaneArgs& a, hipStream_t stream) {
  char* const units = static_cast<char*>(a.units);
  if (a.ways == kPlanes2x2) return launch<D, 2, 2>(a, units, stream);
  if (a.ways == kPlanes2x4) return launch<D, 2, 4>(a, units, stream);
  if constexpr (D != 64)
    if (a.ways == kPlanes1x4) return launch<D, 1, 4>(a, units, stream);
  return hipErrorInvalidValue;
}

}  // namespace

hipError_t launch_attn_f32_planes(const PlaneArgs& a, hipStream_t stream) {
  if ((int64_t)a.batch * a.num_heads * a.n == 0) return hipSuccess;
  if (a.B > 128 || a.num_classes < 1 || a.num_classes > 8) return hipErrorInvalidValue;
  switch (a.D) {
    case 32: return launch<32>(a, stream);
    case 64: return launch<64>(a, stream);
    case 128: return launch<128>(a, stream);
    default: return hipErrorInvalidValue;
  }
}

}  // namespace ca

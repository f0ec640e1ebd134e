// Block-sparse attention forward in full fp32 on the f32 matrix instructions of gfx950 (Appendix D's
// block loop with online softmax), for fp32 problems of any tile size up to 128 tokens.
//
// What bounds it: v_mfma_f32_16x16x4_f32 (a multiply-add in full fp32; a large fp32 matrix product
// reaches 152 TFLOP/s on this card).  8 heads of 7K tokens, head dim 128, 0.094 TFLOP on real tokens:
// 1.18 ms (launches dealt in chunks of 64 rows, see xcd_chunk), 21.4 ms with one thread per query; 2 heads of 256 tokens: 11 us, 222 us.  Per 16 keys and 16 queries a wave
// issues D / 2 of them, 32 cycles each, beside D / 8 16-byte LDS reads and four exponentials, so
// everything else fits beside the matrix pipe.
//
// Decomposition.  A workgroup of four waves owns 16 * QW query slots of one row (batch, head, query
// tile); QW waves side by side hold 16 queries each, and KW = 4 / QW of them share a query group and
// take every KW-th block of 16 keys, each with an online softmax of its own, merged once at the end.
// QW = 4 reads every staged key for the most queries; QW = 1 gives the most workgroups and the
// shortest walk, which is what small tiles and small launches need (see launch_attn_f32).
//
// Transposed products, as in the bf16 kernels: S^T = K Q^T leaves a lane with one query (lane % 16)
// and keys 4 * (lane / 16) + r of the block in register r, which is the B operand of O^T = V^T P^T
// for the four keys {4 g + r}: nothing is exchanged between the products.  The order of the head dim
// inside a contraction is free, so the lane of group g takes d = 16 s + 4 g .. + 3 as one 16-byte read
// for four products; the rows of O^T are permuted likewise, so that one 16-byte read of V serves four
// products and a lane ends up with consecutive output channels.
//
// Keys are staged by LDS DMA, two buffers, one barrier per stage.  Only tokens are staged: the slots of
// a padded tile are taken token-holding slots first (class_perm), in blocks of 16, and a stage is filled
// from as many consecutive kept tiles as it takes.  A block's rows past its last token are masked by count:
// K repeats that token there, and V is zero, because a weight of zero does not cancel an infinity.  A
// padding slot is never read.
#include <algorithm>
#include <type_traits>

#include "attn_bf16_common.h"

namespace ca {
namespace {

typedef __attribute__((ext_vector_type(4))) float f32x4;
typedef __attribute__((ext_vector_type(2))) float f32x2;

template <int D_, int QW_>
struct F32Shape {
  static constexpr int D = D_, QW = QW_, KW = 4 / QW_;
  static constexpr int kStageKeys = (D == 128 && QW > 1) ? 32 : 64;  // 64 KB of LDS and two workgroups per CU (QW = 1 at D = 128: one)
  static constexpr int kBlocks = kStageKeys / 16;       // 16-key blocks of a stage
  static constexpr int kMine = kBlocks / KW;            // of which one wave multiplies
  static constexpr int kRowBytes = D * 4;
  static constexpr int kChunks = D / 4;                 // 16-byte chunks of a row
  static constexpr int kRowsPerLoad = 64 / kChunks;     // rows covered by one wave-wide 16-byte load
  static constexpr int kWaveRows = kStageKeys / 4;      // rows of a stage one wave copies
  static constexpr int kLoads = kWaveRows / kRowsPerLoad;
  static constexpr int kStageBytes = kStageKeys * kRowBytes;
  static constexpr int kVec = D >= 64 ? 4 : 2;          // floats of a V read
  static constexpr int kVecBlocks = D / (16 * kVec);
  static_assert(kMine >= 1 && 16 % kWaveRows == 0, "a wave multiplies whole blocks and copies rows of one block");
  static_assert(4 * 16 * D * 4 + 2 * 4 * 16 * 4 <= 4 * kStageBytes, "the merge fits the stage buffers");
};

// K is read by 16 rows at one logical chunk: physical chunk = logical ^ f(row) puts them on different
// banks.  V is read along its rows and needs no swizzle.
template <int D>
__device__ __forceinline__ int f32_k_swizzle(int row) {
  return D >= 64 ? (row & 15) : ((row >> 1) & 7);
}

// One load with an address of its own for every lane; lanes without a token take zeros instead.  Measured against
// V repeating the last token (and an infinity there giving NaN): 7K tokens, head dim 128, 1.175 / 1.180 ms; grids whose
// tiles are padded on many sides 0-7 % slower.  Lanes without a token that leave the copy out and write zeros
// to LDS: 1.227 ms and 3-8 %.
static __device__ const __attribute__((aligned(16))) uint32_t kZeros[4] = {0, 0, 0, 0};
__device__ __forceinline__ void copy_rows_or_zeros(uint32_t m0, const char* base, uint32_t lane_off, bool token) {
  const char* src = token ? base + lane_off : reinterpret_cast<const char*>(kZeros);
  asm volatile(
      "s_mov_b32 m0, %[m0]\n\ts_nop 0\n\t"
      "global_load_lds_dwordx4 %[v], off\n\t"
      :
      : [m0] "s"(m0), [v] "v"(src)
      : "memory");
}

// The 16-key blocks of one stage (wave-uniform): tile, first position in the tile's token order, tokens.
template <int N>
struct StageBlocks {
  int tile[N], first[N], valid[N], cls[N], keys[N];  // valid: tokens of the tile; keys: tokens of the block, 0 past the end of the row
};

template <int D, int QW>
__global__ __attribute__((amdgpu_flat_work_group_size(256, 256), amdgpu_waves_per_eu(2)))
void attn_f32_kernel(AttnArgs a, int parts, int64_t workgroups) {
  using S = F32Shape<D, QW>;
  constexpr int KW = S::KW;
  __shared__ __attribute__((aligned(1024))) char lds[4 * S::kStageBytes];  // K, V of stage 0, K, V of stage 1
  __shared__ uint8_t lds_perm[8 * 128];

  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int qw = wave % QW, kw = wave / QW;
  const int qi = lane & 15, g = lane >> 4;
  const int64_t id = (int64_t)blockIdx.y * gridDim.x + blockIdx.x;
  if (id >= workgroups) return;
  const int64_t linear = xcd_launch_order(id, workgroups, xcd_chunk(workgroups));
  const int64_t rows = (int64_t)a.num_heads * a.n;
  const int part = (int)(linear % parts);
  const int64_t item = (linear / parts) % rows, batch = linear / parts / rows;
  const int64_t row = a.order ? CONST_PTR(int32_t, a.order)[item] : item;
  const int64_t head = row / a.n, q_tile = row - head * a.n;
  const int64_t plane = (batch * a.num_heads + head) * a.n * a.B * (int64_t)S::kRowBytes;
  const char* Kp = static_cast<const char*>(a.k) + plane;
  const char* Vp = static_cast<const char*>(a.v) + plane;
  const int64_t tile_bytes = (int64_t)a.B * S::kRowBytes;
  const int64_t begin = a.row_ptr ? CONST_PTR(int64_t, a.row_ptr)[row] : 0;
  const int count = (int)(a.row_ptr ? CONST_PTR(int64_t, a.row_ptr)[row + 1] - begin : a.n);
  const auto meta = CONST_PTR(int32_t, a.col_meta + begin);

  for (int e = threadIdx.x; e < a.num_classes * 128; e += 256) lds_perm[e] = a.class_perm[e];

  // queries: positions of the tile's token order; a position past the tile has no row of the output
  const int q_cls = CONST_PTR(int32_t, a.tile_class)[q_tile];
  const int q_valid = (int)((a.class_valid >> (8 * q_cls)) & 0xffu);
  const int q_first = (part * QW + qw) * 16;
  const int q_pos = q_first + qi;
  const bool q_in = q_pos < a.B;
  const int q_slot = a.class_perm[q_cls * 128 + (q_in ? q_pos : 0)];
  const bool wave_active = q_first < q_valid;
  const char* tile_q = static_cast<const char*>(a.q) + plane + q_tile * tile_bytes;
  char* tile_o = static_cast<char*>(a.out) + plane + q_tile * tile_bytes;
  if (part * QW * 16 >= q_valid) {  // padding slots only: zero rows
    for (int e = threadIdx.x; e < QW * 16 * S::kChunks; e += 256) {
      const int pos = part * QW * 16 + e / S::kChunks;
      if (pos < a.B) *reinterpret_cast<f32x4*>(tile_o + (int64_t)a.class_perm[q_cls * 128 + pos] * S::kRowBytes + e % S::kChunks * 16) = f32x4{0.f, 0.f, 0.f, 0.f};
    }
    return;
  }
  f32x4 qf[D / 16];
#pragma unroll
  for (int s = 0; s < D / 16; ++s) qf[s] = *reinterpret_cast<const f32x4*>(tile_q + (int64_t)q_slot * S::kRowBytes + (16 * s + 4 * g) * 4);
#pragma unroll
  for (int s = 0; s < D / 16; ++s) asm volatile("" : "+v"(qf[s]));  // waited for here: in the loop the counter belongs to the copies

  f32x4 acc_o[D / 16];
#pragma unroll
  for (int i = 0; i < D / 16; ++i) acc_o[i] = f32x4{0.f, 0.f, 0.f, 0.f};
  const float c2 = a.scale * kLog2e;
  float ref = -1e30f, l_run = 0.f;  // exponent reference of the query in log2 units; this lane's share of its row sum

  // ---- the walk: blocks of 16 tokens of the kept tiles in order, the words two tiles ahead -----------
  int j = 0, first = 0;
  int32_t word = count > 0 ? meta[0] : 0, word1 = count > 0 ? meta[1] : 0;
  auto next_stage = [&](StageBlocks<S::kBlocks>& st) {
#pragma unroll
    for (int b = 0; b < S::kBlocks; ++b) {
      st.tile[b] = word & 0xffffff;
      st.cls[b] = (word >> 24) & 7;
      st.valid[b] = (int)((a.class_valid >> (8 * st.cls[b])) & 0xffu);
      st.first[b] = first;
      st.keys[b] = j < count ? min(16, st.valid[b] - first) : 0;
      if (j < count) {
        first += 16;
        if (first >= st.valid[b]) {
          first = 0;
          ++j;
          word = word1;
          if (j < count) word1 = meta[j + 1];
        }
      }
    }
  };
  // ---- this wave's rows of a stage, all in one block ---------------------------------------------------
  const uint32_t lds_addr = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) char*)lds;
  const int my_block = wave * S::kWaveRows / 16;
  auto issue = [&](const StageBlocks<S::kBlocks>& st, int buf) {
    int tile = 0, pos0 = 0, valid = 0, cls = 0, keys = 0;
#pragma unroll
    for (int b = 0; b < S::kBlocks; ++b)
      if (b == my_block) tile = st.tile[b], pos0 = st.first[b], valid = st.valid[b], cls = st.cls[b], keys = st.keys[b];
    if (keys == 0) return;
    const char* kb = Kp + tile * tile_bytes;
    const char* vb = Vp + tile * tile_bytes;
    auto copy = [&](auto full) {  // full: sixteen tokens, which the rows of most blocks are
#pragma unroll
      for (int i = 0; i < S::kLoads; ++i) {
        const int row0 = wave * S::kWaveRows + i * S::kRowsPerLoad;  // of the stage
        const int r = row0 + lane / S::kChunks;
        int slot = full() ? pos0 + (r & 15) : min(pos0 + (r & 15), valid - 1);
        if (cls != 0) slot = lds_perm[cls * 128 + slot];
        const int phys = lane % S::kChunks;
        const uint32_t k_off = (uint32_t)(slot * S::kRowBytes + (phys ^ f32_k_swizzle<D>(r)) * 16);
        const uint32_t v_off = (uint32_t)(slot * S::kRowBytes + phys * 16);
        const uint32_t k_lds = lds_addr + (uint32_t)(buf * 2 * S::kStageBytes + row0 * S::kRowBytes);
        if constexpr (full()) {
          asm volatile(
              "s_mov_b32 m0, %[mk]\n\ts_nop 0\n\t"
              "global_load_lds_dwordx4 %[ko], %[kb]\n\t"
              "s_mov_b32 m0, %[mv]\n\ts_nop 0\n\t"
              "global_load_lds_dwordx4 %[vo], %[vb]\n\t"
              :
              : [mk] "s"(k_lds), [mv] "s"(k_lds + (uint32_t)S::kStageBytes), [ko] "v"(k_off), [vo] "v"(v_off), [kb] "s"(kb), [vb] "s"(vb)
              : "memory");
        } else {
          copy_rows(k_lds, kb, k_off);
          copy_rows_or_zeros(k_lds + (uint32_t)S::kStageBytes, vb, v_off, (r & 15) < keys);
        }
      }
    };
    if (keys == 16) copy(std::true_type{});
    else copy(std::false_type{});
  };

  StageBlocks<S::kBlocks> cur, nxt;
  next_stage(cur);
  __syncthreads();  // lds_perm is complete
  issue(cur, 0);
  for (int buf = 0; cur.keys[0] > 0; buf ^= 1) {
    WAIT_VMCNT(0);
    WAIT_LGKMCNT0();
    BARRIER();  // this stage has landed, and every wave is done with the other buffer
    next_stage(nxt);
    issue(nxt, buf ^ 1);

    int keys[S::kMine];
    bool work = false;
#pragma unroll
    for (int x = 0; x < S::kMine; ++x) {
      keys[x] = 0;
#pragma unroll
      for (int b = 0; b < S::kBlocks; ++b)
        if (b == x * KW + kw) keys[x] = cur.keys[b];
    }
    work = wave_active && keys[0] > 0;  // blocks are filled in order
    if (work) {
      const LdsTile lds_k = (LdsTile)lds + buf * 2 * S::kStageBytes, lds_v = lds_k + S::kStageBytes;
      // ---- S^T = K Q^T; a lone block is summed in two chains so that its products do not wait for each other
      constexpr int kChains = S::kMine == 1 ? 2 : 1;
      f32x4 sc[S::kMine][kChains];
#pragma unroll
      for (int x = 0; x < S::kMine; ++x)
#pragma unroll
        for (int c = 0; c < kChains; ++c) sc[x][c] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int s = 0; s < D / 16; ++s) {
        f32x4 kf[S::kMine];
#pragma unroll
        for (int x = 0; x < S::kMine; ++x) {
          const int r = (x * KW + kw) * 16 + qi;
          kf[x] = *reinterpret_cast<const __attribute__((address_space(3))) f32x4*>(lds_k + r * S::kRowBytes + (((4 * s + g) ^ f32_k_swizzle<D>(qi)) << 4));
        }
#pragma unroll
        for (int t = 0; t < 4; ++t)
#pragma unroll
          for (int x = 0; x < S::kMine; ++x)
            sc[x][t % kChains] = __builtin_amdgcn_mfma_f32_16x16x4f32(kf[x][t], qf[s][t], sc[x][t % kChains], 0, 0, 0);
      }
      // ---- online softmax, the reference is the running maximum --------------------------------------
      float mx = kMinusInf;
#pragma unroll
      for (int x = 0; x < S::kMine; ++x) {
        if (kChains == 2) sc[x][0] += sc[x][kChains - 1];
        if (keys[x] < 16) {
#pragma unroll
          for (int r = 0; r < 4; ++r) sc[x][0][r] = 4 * g + r < keys[x] ? sc[x][0][r] : kMinusInf;
        }
#pragma unroll
        for (int r = 0; r < 4; ++r) mx = fmaxf(mx, sc[x][0][r]);
      }
      mx = fmaxf(mx, __shfl_xor(mx, 16, 64));
      mx = fmaxf(mx, __shfl_xor(mx, 32, 64));
      const float ref_new = fmaxf(ref, mx * c2);
      if (__any(ref_new > ref)) {
        const float alpha = __builtin_amdgcn_exp2f(ref - ref_new);
        l_run *= alpha;
#pragma unroll
        for (int i = 0; i < D / 16; ++i) acc_o[i] *= alpha;
        ref = ref_new;
      }
#pragma unroll
      for (int x = 0; x < S::kMine; ++x)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          sc[x][0][r] = __builtin_amdgcn_exp2f(fmaf(sc[x][0][r], c2, -ref));
          l_run += sc[x][0][r];
        }
      // ---- O^T += V^T P^T -------------------------------------------------------------------------------
#pragma unroll
      for (int x = 0; x < S::kMine; ++x) {
        if (x > 0 && keys[x] == 0) break;  // nothing was staged
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const LdsTile v_row = lds_v + ((x * KW + kw) * 16 + 4 * g + r) * S::kRowBytes;
#pragma unroll
          for (int vb = 0; vb < S::kVecBlocks; ++vb) {
            if constexpr (S::kVec == 4) {
              const f32x4 vf = *reinterpret_cast<const __attribute__((address_space(3))) f32x4*>(v_row + (16 * vb + qi) * 16);
#pragma unroll
              for (int t = 0; t < 4; ++t) acc_o[4 * vb + t] = __builtin_amdgcn_mfma_f32_16x16x4f32(vf[t], sc[x][0][r], acc_o[4 * vb + t], 0, 0, 0);
            } else {
              const f32x2 vf = *reinterpret_cast<const __attribute__((address_space(3))) f32x2*>(v_row + qi * 8);
#pragma unroll
              for (int t = 0; t < 2; ++t) acc_o[t] = __builtin_amdgcn_mfma_f32_16x16x4f32(vf[t], sc[x][0][r], acc_o[t], 0, 0, 0);
            }
          }
        }
      }
    }
    cur = nxt;
  }

  // ---- merge of the KW shares of a query, O = O^T / l, store -------------------------------------------
  l_run += __shfl_xor(l_run, 16, 64);
  l_run += __shfl_xor(l_run, 32, 64);
  // channels of a lane: kVec * 4 consecutive ones from 16 * kVec * vb + 4 * kVec * g on, kVec per register r
  if constexpr (KW == 1) {
    const float inv = (q_pos < q_valid && l_run > 0.f) ? 1.0f / l_run : 0.f;
    if (!q_in) return;
    char* out = tile_o + (int64_t)q_slot * S::kRowBytes;
#pragma unroll
    for (int vb = 0; vb < S::kVecBlocks; ++vb)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int d0 = 16 * S::kVec * vb + 4 * S::kVec * g + S::kVec * r;
        if constexpr (S::kVec == 4) {
          *reinterpret_cast<f32x4*>(out + d0 * 4) = f32x4{acc_o[4 * vb][r], acc_o[4 * vb + 1][r], acc_o[4 * vb + 2][r], acc_o[4 * vb + 3][r]} * inv;
        } else {
          *reinterpret_cast<f32x2*>(out + d0 * 4) = f32x2{acc_o[0][r], acc_o[1][r]} * inv;
        }
      }
  } else {
    float* red_ref = reinterpret_cast<float*>(lds);   // [4 waves][16]
    float* red_sum = red_ref + 64;                    // [4][16]
    float* red_o = red_ref + 128;                     // [4][16][D]
    __syncthreads();  // the stage buffers are free
    if (g == 0) red_ref[wave * 16 + qi] = ref;
    __syncthreads();
    float top = kMinusInf;
#pragma unroll
    for (int k = 0; k < KW; ++k) top = fmaxf(top, red_ref[(k * QW + qw) * 16 + qi]);
    const float f = __builtin_amdgcn_exp2f(ref - top);
    if (g == 0) red_sum[wave * 16 + qi] = l_run * f;
#pragma unroll
    for (int vb = 0; vb < S::kVecBlocks; ++vb)
#pragma unroll
      for (int r = 0; r < 4; ++r)
#pragma unroll
        for (int t = 0; t < S::kVec; ++t)
          red_o[(wave * 16 + qi) * D + 16 * S::kVec * vb + 4 * S::kVec * g + S::kVec * r + t] = acc_o[S::kVec * vb + t][r] * f;
    __syncthreads();
    for (int e = threadIdx.x; e < QW * 16 * S::kChunks; e += 256) {
      const int q = e / S::kChunks, c = e % S::kChunks;
      const int pos = part * QW * 16 + q;
      if (pos >= a.B) continue;
      float l = 0.f;
      f32x4 o = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int k = 0; k < KW; ++k) {
        l += red_sum[k * QW * 16 + q];
        o += *reinterpret_cast<const f32x4*>(&red_o[(k * QW * 16 + q) * D + 4 * c]);
      }
      const float inv = (pos < q_valid && l > 0.f) ? 1.0f / l : 0.f;
      *reinterpret_cast<f32x4*>(tile_o + (int64_t)lds_perm[q_cls * 128 + pos] * S::kRowBytes + c * 16) = o * inv;
    }
  }
}

template <int D>
hipError_t launch(const AttnArgs& a, hipStream_t stream) {
  const int64_t rows = (int64_t)a.batch * a.num_heads * a.n;
  const int qw = f32_query_groups(rows, a.B, D), parts = (a.B + 16 * qw - 1) / (16 * qw);
  const int64_t workgroups = rows * parts, width = std::min(workgroups, (int64_t)1 << 23);  // a grid dimension holds fewer than 2^32 threads
  if (workgroups > (int64_t)1 << 38) return hipErrorInvalidValue;
  const dim3 grid((unsigned)width, (unsigned)((workgroups + width - 1) / width)), block(256);
  if (qw == 4) hipLaunchKernelGGL((attn_f32_kernel<D, 4>), grid, block, 0, stream, a, parts, workgroups);
  else if (qw == 2) hipLaunchKernelGGL((attn_f32_kernel<D, 2>), grid, block, 0, stream, a, parts, workgroups);
  else hipLaunchKernelGGL((attn_f32_kernel<D, 1>), grid, block, 0, stream, a, parts, workgroups);
  return hipGetLastError();
}

}  // namespace

hipError_t launch_attn_f32(const AttnArgs& a, hipStream_t stream) {
  if (a.ways != kWaysNone) return launch_attn_f32_planes(static_cast<const PlaneArgs&>(a), stream);
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

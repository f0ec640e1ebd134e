// Rows split along the keys (SplitPlan in layout.h): adds up what the shares of a row have left in the workspace and
// writes the output.
//
// Bound: latency.  A share of 32 queries is 16.5 KB at head dim 128, a launch leaves kMaxShareBytes at most, and most leave a
// tenth of that.  A workgroup takes 32 queries, a wave 32 channels of them, lane by lane as the attention kernels left them,
// so that all reads are whole lines; the shares are added in their order, so the result is run-to-run identical.
#include "attn_bf16_common.h"

namespace ca {
namespace {

template <int D, bool kNat>
__global__ __launch_bounds__(D * 2) void attn_bf16_merge_kernel(SplitArgs a) {
  constexpr int kRowBytes = D * 2;
  const int lane = threadIdx.x & 63, db = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int waves = a.share_waves, wave = (int)(blockIdx.x % (unsigned)waves);
  const int64_t linear = blockIdx.x / (unsigned)waves, batch = linear / a.num_merges;
  const auto item = CONST_PTR(int32_t, a.merges + linear % a.num_merges);
  const int64_t entry = item[0];
  const int shares = item[3];
  const int64_t first = batch * a.shares + item[2];
  int64_t row = entry;
  int first_slot = (item[1] * waves + wave) * 32;
  if (entry < 0) {  // a workgroup of two query tiles, see attn_pair_body
    const uint32_t desc = (uint32_t)CONST_PTR(int32_t, a.pair_desc)[~entry];
    if (((desc >> (4 + wave)) & 1u) == 0) return;
    row = CONST_PTR(int32_t, a.pair_rows)[2 * ~entry + (int)((desc >> wave) & 1u)];
    if (row < 0) return;
    first_slot = (int)((desc >> (8 + 4 * wave)) & 0xFu) * 32;
  }
  const int64_t head = row / a.n, q_tile = row - head * a.n;
  const int64_t plane = (batch * a.num_heads + head) * (kNat ? a.N_real : a.n * (int64_t)a.B) * kRowBytes;
  const int qi = lane & 31, g = lane >> 5;
  const QuerySlot qs = query_slot<128>(a, q_tile, first_slot, qi);
  const int64_t q_row = kNat ? natural_query_row(a, q_tile, qs.slot) : q_tile * a.B + qs.slot;
  const float c2 = a.scale * kLog2e;
  float l_run = 0.f;
  floatx16 acc;
#pragma unroll
  for (int r = 0; r < 16; ++r) acc[r] = 0.f;
  if (qs.wave_active) {
    const float2* stats = static_cast<const float2*>(a.share_stats) + (first * waves + wave) * 64 + lane;
    const float4* o = static_cast<const float4*>(a.share_o) + ((first * waves + wave) * (D / 8) + db * 4) * 64 + lane;
    float top = kMinusInf;
    for (int k = 0; k < shares; ++k) top = fmaxf(top, stats[(int64_t)k * waves * 64].x);
#pragma unroll 2
    for (int k = 0; k < shares; ++k) {
      const float2 st = stats[(int64_t)k * waves * 64];
      const float f = st.x == kMinusInf ? 0.f : __builtin_amdgcn_exp2f((st.x - top) * c2);  // no key: weight 0
      l_run += st.y * f;
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const float4 x = o[((int64_t)k * waves * (D / 8) + i) * 64];
        acc[4 * i + 0] += x.x * f;
        acc[4 * i + 1] += x.y * f;
        acc[4 * i + 2] += x.z * f;
        acc[4 * i + 3] += x.w * f;
      }
    }
  }
  const float l_tot = sum_with_partner(l_run);
  const float inv = (qs.real && l_tot > 0.f) ? 1.0f / l_tot : 0.f;
  if (!kNat || qs.real) {
    char* out_row = static_cast<char*>(a.out) + plane + q_row * kRowBytes;
#pragma unroll
    for (int r4 = 0; r4 < 4; ++r4) {
      bf16x4 o4;
#pragma unroll
      for (int e = 0; e < 4; ++e) o4[e] = (__bf16)(acc[4 * r4 + e] * inv);
      *reinterpret_cast<bf16x4*>(out_row + (db * 32 + 8 * r4 + 4 * g) * 2) = o4;
    }
  }
  if (!kNat && entry < 0 && db == 0 && a.B > 64) zero_unowned_rows<D>(a, static_cast<char*>(a.out) + plane, q_tile, first_slot, lane);
}

}  // namespace

hipError_t launch_attn_bf16_merge(const SplitArgs& a, hipStream_t stream) {
  const int64_t blocks = a.batch * a.num_merges * a.share_waves;
  if (blocks < 1 || blocks > 0x7fffff || !a.merges || !a.share_stats || !a.share_o) return hipErrorInvalidValue;
  if (a.D != 64 && a.D != 128) return hipErrorInvalidValue;
  const auto kernel = a.D == 128 ? (a.natural ? attn_bf16_merge_kernel<128, true> : attn_bf16_merge_kernel<128, false>)
                                 : (a.natural ? attn_bf16_merge_kernel<64, true> : attn_bf16_merge_kernel<64, false>);
  hipLaunchKernelGGL(kernel, dim3((unsigned)blocks), dim3(a.D * 2), 0, stream, a);
  return hipGetLastError();
}

}  // namespace ca

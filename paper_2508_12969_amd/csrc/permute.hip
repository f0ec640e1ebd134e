// Tile-order flattening of the token sequence and its inverse (Sec. 3.1 / Appendix D of the
// paper): every run of B consecutive tokens of the permuted sequence is one tt x th x tw tile.
//
// HBM-bound copy.  One workgroup moves one tile of one (batch, head) plane.  Inside a tile the
// tw tokens that share (frame, row) are contiguous in both orders, so the unit of work is such a
// run: a wave derives the run's two offsets with scalar arithmetic and its lanes move 16-byte
// chunks, which keeps every access a full-width contiguous burst.  Padding slots are written as
// zero on the way in and skipped on the way out.
#include "kernels.h"

namespace ca {
namespace {

typedef __attribute__((ext_vector_type(4))) uint32_t u32x4;

constexpr int kThreads = 256;
constexpr int kWaves = kThreads / 64;

// kMany: a kernel of its own, because the few instructions more cost the others 0.3 us of 2.
template <bool kMany>
__global__ __launch_bounds__(kThreads) void permute_kernel(std::conditional_t<kMany, PermuteManyArgs, PermuteArgs> a) {
  const int64_t tile = blockIdx.x;
  const int64_t plane = blockIdx.y;
  int64_t natural_rows = a.N_real;
  const void* src = a.src;
  void* dst = a.dst;
  const bool inverse = (a.inverse & 1) != 0;
  if constexpr (kMany) {  // (an index that is not a constant would put the arguments into scratch memory)
    src = blockIdx.z == 0 ? a.srcs[0] : blockIdx.z == 1 ? a.srcs[1] : a.srcs[2];
    dst = blockIdx.z == 0 ? a.dsts[0] : blockIdx.z == 1 ? a.dsts[1] : a.dsts[2];
    natural_rows = a.natural_rows;
  }
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int lane = threadIdx.x & 63;
  const int64_t rb = a.row_bytes;

  const char* nat = static_cast<const char*>(inverse ? (const void*)dst : src) + plane * natural_rows * rb;
  const char* til = static_cast<const char*>(inverse ? src : (const void*)dst) + plane * a.N_pad * rb;
  if constexpr (kMany) {
    if (tile * a.B >= a.N_pad) {  // the last workgroup of a plane with room at its end
      for (int64_t c = threadIdx.x; c < (natural_rows - a.N_real) * rb >> 4; c += kThreads)
        reinterpret_cast<u32x4*>(const_cast<char*>(nat) + a.N_real * rb)[c] = u32x4{0u, 0u, 0u, 0u};
      return;
    }
  }

  const int runs = a.tt * a.th;                      // runs of tw tokens in a tile
  const int run_chunks = (int)((a.tw * rb) >> 4);    // 16-byte chunks per run
  int kt = 0, kh = 0, kw = 0;
  const bool text = tile >= a.n_vid;
  if (!text) {
    kw = (int)(tile % a.nW);
    const int64_t r = tile / a.nW;
    kh = (int)(r % a.nH);
    kt = (int)(r / a.nH);
  }
  for (int run = wave; run < runs; run += kWaves) {
    int64_t nat_off;   // byte offset of the run's first token in natural order
    int valid_chunks;  // chunks of the run that hold real tokens
    if (text) {
      nat_off = (a.N_video + (tile - a.n_vid) * a.B + (int64_t)run * a.tw) * rb;
      valid_chunks = run_chunks;
    } else {
      const int dt = run / a.th, dy = run - dt * a.th;
      const int t = kt * a.tt + dt, y = kh * a.th + dy, x0 = kw * a.tw;
      const int xs = (t < a.T && y < a.H) ? min(a.tw, a.W - x0) : 0;
      nat_off = (((int64_t)t * a.H + y) * a.W + x0) * rb;
      valid_chunks = (int)((xs * rb) >> 4);
    }
    const int64_t til_off = (tile * a.B + (int64_t)run * a.tw) * rb;
    if (!inverse) {
      for (int c = lane; c < run_chunks; c += 64) {
        u32x4 val = {0u, 0u, 0u, 0u};
        if (c < valid_chunks) val = __builtin_nontemporal_load(reinterpret_cast<const u32x4*>(nat + nat_off) + c);
        __builtin_nontemporal_store(val, reinterpret_cast<u32x4*>(const_cast<char*>(til) + til_off) + c);
      }
    } else {
      for (int c = lane; c < valid_chunks; c += 64) {
        const u32x4 val = __builtin_nontemporal_load(reinterpret_cast<const u32x4*>(til + til_off) + c);
        __builtin_nontemporal_store(val, reinterpret_cast<u32x4*>(const_cast<char*>(nat) + nat_off) + c);
      }
    }
  }
}

}  // namespace

hipError_t launch_permute(const PermuteArgs& a, hipStream_t stream) {
  const int64_t n_tiles = a.N_pad / a.B;
  if (n_tiles == 0 || a.planes == 0) return hipSuccess;
  if (a.planes > 65535) return hipErrorInvalidValue;
  dim3 grid((unsigned)n_tiles, (unsigned)a.planes, 1);
  if (a.inverse < kPermuteMany) {
    hipLaunchKernelGGL(permute_kernel<false>, grid, dim3(kThreads), 0, stream, a);
    return hipGetLastError();
  }
  const PermuteManyArgs& many = static_cast<const PermuteManyArgs&>(a);
  if (many.tensors < 1 || many.tensors > 3 || many.natural_rows < a.N_real) return hipErrorInvalidValue;
  if (a.inverse == kPermuteMany + 1 && many.natural_rows > a.N_real) grid.x += 1;
  grid.z = (unsigned)many.tensors;
  hipLaunchKernelGGL(permute_kernel<true>, grid, dim3(kThreads), 0, stream, many);
  return hipGetLastError();
}

}  // namespace ca

// Router-weighted combine: the k expert rows of a token are summed with the
// router weights in fp32, in slot order from +0.0, then rounded once to bf16
// (the paper's router-weighted F32 accumulation followed by conversion back
// to the hidden type).  Products and sums are rounded separately (FMA
// contraction is switched off in add_slots), which is the exact order of the
// definition, so the result is bit-identical to it for given rows.
//
// Memory bound: k * 4 bytes read + 2 bytes written per output element.
// Thread = 4 consecutive outputs (one 16-byte load per slot, one 8-byte
// store), so that a wave reads whole 1 KB pieces of a row; workgroup = 256
// threads = 1024 outputs of one token.  The rows are read once, by
// non-temporal loads, which leave the caches to others, but for 170 to 300 MB of
// rows: most of those are still in the Infinity Cache (256 MB) from the down
// projection that wrote them, and non-temporal loads of them were the slower
// ones.  (Fewer rows take the same time either way, and plain loads of them cost
// the next gate/up launch 2 to 3 us where its weights are in that cache: H 2048, I
// 768, 128 experts, 509 tokens 98.7 -> 100.9 us.)  Non-temporal loads need whole
// pieces and no row read twice: with 8 outputs per thread (two loads half a
// KB apart by lane) they were slower than plain ones, and
// reloading a slot in place of those past k (as plain loads did, from L1)
// took 24.7 instead of 15.1 us at k = 2.
// Measured, rows written just before, us (8 outputs per thread with plain
// loads | non-temporal | plain):
//   H 7168, k 8:  69 MB of rows 14.9 | 14.5 | 14.5    161 MB 29.0 | 28.9 | 28.7
//                235 MB 43.9 | 45.6 | 42.6    275 MB 54.7 | 54.5 | 53.8
//                344 MB 75.9 | 68.8 | 74.3
//               1879 MB 403 | 374 | 402 (5.7 TB/s of rows and outputs, rocprofv3)
//   H 2048, k 8: 229 MB 42.3 | 45.7 | 41.9    328 MB 71.2 | 67.1 | 70.0
//   H 4096, k 2: 197 MB 53.1 | 46.9 | 40.5    262 MB 70.6 | 55.7 | 58.6
#include <algorithm>

#include "common.h"

namespace moe {
namespace {

constexpr double kCachedRowsMin = 170e6, kCachedRowsMax = 300e6;  // bytes of rows read by plain loads

// Slots j0 .. j0 + N - 1 added to acc: their row indices and weights are
// loaded first, then the N rows (N loads in flight per thread), then the
// products are added in slot order.
template <bool NT, int N>
__device__ __forceinline__ void add_slots(float (&acc)[4], const float* __restrict__ y,
                                          const int32_t* __restrict__ dest, const float* __restrict__ w, int H,
                                          int n) {
#pragma clang fp contract(off)
  int64_t p[N];
  float wj[N];
  v4f v[N];
#pragma unroll
  for (int u = 0; u < N; ++u) {
    p[u] = dest[u];
    wj[u] = w[u];
  }
#pragma unroll
  for (int u = 0; u < N; ++u) {
    const v4f* row = reinterpret_cast<const v4f*>(y + p[u] * H + n);
    v[u] = NT ? __builtin_nontemporal_load(row) : *row;
  }
#pragma unroll
  for (int u = 0; u < N; ++u)
#pragma unroll
    for (int i = 0; i < 4; ++i) acc[i] = acc[i] + wj[u] * v[u][i];
}

// Token t's outputs n .. n + 3: slots in batches of 8, then the remaining 0
// to 7 in one batch of their own, so that no row is loaded twice.  Same
// arithmetic and order as combine8_of (the fused decode kernel's combine), so
// the same bits.
template <bool NT>
__device__ __forceinline__ uint2 combine4_batched(const float* __restrict__ y, const int32_t* __restrict__ dest,
                                                  const float* __restrict__ w, int k, int H, int64_t t, int n) {
  float acc[4] = {0.0f, 0.0f, 0.0f, 0.0f};
  dest += t * k;
  w += t * k;
  for (; k >= 8; k -= 8, dest += 8, w += 8) add_slots<NT, 8>(acc, y, dest, w, H, n);
  switch (k) {
    case 1: add_slots<NT, 1>(acc, y, dest, w, H, n); break;
    case 2: add_slots<NT, 2>(acc, y, dest, w, H, n); break;
    case 3: add_slots<NT, 3>(acc, y, dest, w, H, n); break;
    case 4: add_slots<NT, 4>(acc, y, dest, w, H, n); break;
    case 5: add_slots<NT, 5>(acc, y, dest, w, H, n); break;
    case 6: add_slots<NT, 6>(acc, y, dest, w, H, n); break;
    case 7: add_slots<NT, 7>(acc, y, dest, w, H, n); break;
    default: break;
  }
  return make_uint2((uint32_t)f32_to_bf16_rne(acc[0]) | ((uint32_t)f32_to_bf16_rne(acc[1]) << 16),
                    (uint32_t)f32_to_bf16_rne(acc[2]) | ((uint32_t)f32_to_bf16_rne(acc[3]) << 16));
}

template <bool NT>
__global__ __launch_bounds__(256) void combine_kernel(const float* __restrict__ y, const int32_t* __restrict__ dest,
                                                      const float* __restrict__ w, int k, int H, int blocks_per_tok,
                                                      uint16_t* __restrict__ out) {
  const int64_t t = blockIdx.x / blocks_per_tok;
  const int n = ((int)(blockIdx.x - t * blocks_per_tok) * 256 + (int)threadIdx.x) * 4;
  if (n >= H) return;
  *reinterpret_cast<uint2*>(out + t * H + n) = combine4_batched<NT>(y, dest, w, k, H, t, n);
}

}  // namespace
}  // namespace moe

using namespace moe;

extern "C" moe_status_t moe_combine(const float* y_rows, const int32_t* dest_row, const float* topk_w, int32_t T,
                                    int32_t k, int32_t H, uint16_t* out_bf16, hipStream_t stream) {
  if (T < 0 || k < 1 || H <= 0) return fail(MOE_ERR_INVALID_ARG, "moe_combine: T=%d k=%d H=%d", T, k, H);
  if (H % kBlock) return fail(MOE_ERR_UNSUPPORTED_SHAPE, "moe_combine: H=%d not a multiple of 128", H);
  if (T == 0) return MOE_OK;
  if (!y_rows || !dest_row || !topk_w || !out_bf16) return fail(MOE_ERR_INVALID_ARG, "moe_combine: null pointer");
  if (!aligned(y_rows, 16) || !aligned(out_bf16, 16))
    return fail(MOE_ERR_INVALID_ARG, "moe_combine: misaligned pointer");
  const int bpt = (H + 1023) / 1024;
  const int64_t blocks = (int64_t)T * bpt;
  if (blocks > 0x7fffffff) return fail(MOE_ERR_UNSUPPORTED_SHAPE, "moe_combine: too many tokens");
  const double row_bytes = (double)T * k * H * sizeof(float);
  const bool nt = row_bytes < kCachedRowsMin || row_bytes > kCachedRowsMax;
  // A grid has less than 2^32 threads: the tokens of one launch.
  const int64_t span = std::min<int64_t>(T, ((1 << 24) - 1) / bpt);
  for (int64_t t0 = 0; t0 < T; t0 += span) {
    const int64_t n = std::min<int64_t>(span, T - t0);
    const auto kernel = nt ? combine_kernel<true> : combine_kernel<false>;
    MOE_LAUNCH("combine", kernel, dim3((unsigned)(n * bpt)), dim3(256), 0, stream, y_rows, dest_row + t0 * k,
               topk_w + t0 * k, k, H, bpt, out_bf16 + t0 * H);
  }
  return check_launch("moe_combine");
}

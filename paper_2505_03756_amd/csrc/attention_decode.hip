// Paged attention of single new tokens (decode) on the matrix cores, for 16-bit pools with head_dim 128 and up to 16
// query heads per kv head.
//
// Bound by the K/V traffic: one token makes G = n_q / n_kv products per K/V element, so what counts is that every
// K/V byte is read once for all G heads, that enough loads are in flight, and that a wave spends few instructions
// per byte.  One WAVE owns the G rows of one (token, kv head) over a run of 16-position groups and walks it 32
// positions at a time; the pieces of a long context are merged afterwards.  Nothing is staged in LDS (no byte is used
// twice) and no wave waits for another one: the 16 loads (16 KiB) of the next 32 positions are in flight while the
// present ones are multiplied, 8 such waves per CU.
//
// S^T = K Q^T is computed transposed with 16x16x32 instructions: a lane holds one query row (column l % 16) and, with the
// keys fed in the order key(m) = 8 (m / 4) + 4 t + m % 4 for row m of instruction t, the 8 consecutive positions
// 8 (l / 16) ... + 7, which are also the positions of its 16-byte run of the transposed V of a pool block.
//
// O^T = V^T P^T takes fp32 weights and sums with three 16x16x32 instructions per weight: its value in the pool's type,
// the remainder, and the remainder of that; a product of two 16-bit numbers is exact in fp32.
//   bf16   8 bits each, so a weight is exactly the sum of its pieces.  Taken times 2^16 it keeps the last one a normal
//          number down to 2^-126 of the largest weight.
//   fp16   11 bits each; weights are taken times 2^15 and every remainder times 2^11, and the tile's sums are scaled back from
//          piece to piece.  Exact down to 2^-38 of the largest weight; below, at most 2^-62 of the largest is lost, which
//          times 65504 and a million positions is still less than half the smallest fp16 number.
// What the pieces cannot express is an infinite or overflowing product (0 x inf, inf - inf): a wave whose sums are not all
// finite walks its piece of the context again with 16x16x4 fp32 instructions on the widened V, so infinities and NaN
// in V come out as an fp32 multiply-add makes them.  The rows past the last head repeat it.
//
// The wave's work is in attention_decode_wave.h: beside tiles it runs in the tiled kernel's launch.
//
// Measured, whole steps on MI355X.  Before this kernel (a wave per query head on the vector units, fp32, nothing loaded
// ahead), then with weights as value and remainder only (16 bits of them in bf16), 16x16x4 throughout, three pieces:
//   256 sequences of 512-4096 positions, 32 / 32 heads, bf16, 9.8 GB of K/V    1941   1865   1903   1867 us
//   6 sequences of 8-16 k positions, 64 / 8 heads, bf16                         234    137    143    137 us
//   layer with 200 decode tokens, 32 / 32 heads, bf16                          1092   1047   1064   1046 us
#include <hip/hip_runtime.h>

#include "attention_decode_wave.h"
#include "flp_internal.h"

namespace {

template <typename M>
__global__ __launch_bounds__(256, 2) void attn_decode_kernel(FlpAttnArgs a, const FlpAttnUnit* __restrict__ units) {
  const int g = blockIdx.y * 4 + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  if (g < a.n_kv) flp_decode::decode_unit<M>(a, units[blockIdx.x], g);      // waves share nothing
}

}  // namespace

flp_status flp_launch_attn_decode(int dtype, const FlpAttnArgs& a, const FlpAttnUnit* units_dev, int32_t n_units,
                                  hipStream_t stream) {
  if (n_units <= 0) return FLP_OK;
  const dim3 grid((unsigned)n_units, (unsigned)((a.n_kv + 3) / 4));
  if (dtype == FLP_F16)
    hipLaunchKernelGGL((attn_decode_kernel<flp_decode::DF16>), grid, dim3(256), 0, stream, a, units_dev);
  else if (dtype == FLP_BF16)
    hipLaunchKernelGGL((attn_decode_kernel<flp_decode::DBF16>), grid, dim3(256), 0, stream, a, units_dev);
  else {
    flp_set_error("attention (decode path): dtype %d not supported", dtype);
    return FLP_ENOTSUP;
  }
  FLP_TRY_HIP(hipGetLastError());
  return FLP_OK;
}

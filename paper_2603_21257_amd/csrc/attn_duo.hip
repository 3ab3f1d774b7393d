// The small-tile shape of the pipelined attention kernel (attn_pipeline.h): workgroup = 4 query heads of one KV group x one
// token tile of 32 (128 rows in any case), four waves of 32 rows, two workgroups per CU (80 KiB of LDS each: K and V rings
// of five 8 KiB slots), so the two waves of a SIMD belong to different workgroups.  With the short queries of the paper's
// Table 1 (28 / 61 / 209 tokens) half of a 64-token tile's rows would be empty.
#include "attn_pipeline.h"

namespace calvo {
namespace duo {

using namespace attn;
using Cfg = PipeCfg<4, 5, 1>;
// with the rows of several tiles from the caller's arrays: a kernel of its own, the choice of the address costs every launch
// 0.4 us (28096+28 tokens 28.2 -> 28.6 us a call, 18624+7 18.1 -> 18.4)
using CfgSuffix = PipeCfg<4, 5, 1, true>;

__global__ void __launch_bounds__(256, 2) __attribute__((amdgpu_num_vgpr(120))) attn_duo_kernel(AttnParams p) {
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  clock_begin(p.clock);
  if (append_wg(p)) return;
  attn_pipeline<Cfg>(p, smem);
}


__global__ void __launch_bounds__(256, 2) __attribute__((amdgpu_num_vgpr(120))) attn_duo_suffix_kernel(AttnParams p) {
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  clock_begin(p.clock);
  if (append_wg(p)) return;
  attn_pipeline<CfgSuffix>(p, smem);
}

}  // namespace duo

int attn_duo_tile_tokens(int heads_per_wg) { return 32 * (4 / heads_per_wg); }

hipError_t attn_duo_prepare() {
  for (const void* k : {(const void*)duo::attn_duo_kernel, (const void*)duo::attn_duo_suffix_kernel}) {
    const hipError_t e = hipFuncSetAttribute(k, hipFuncAttributeMaxDynamicSharedMemorySize, duo::Cfg::LDS_BYTES);
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}

// one_tile: no request's suffix is longer than a tile
hipError_t launch_attn_duo(const AttnParams& p, bool one_tile, hipStream_t stream) {
  if (p.n_items <= 0) return hipSuccess;
  const unsigned grid = (unsigned)p.n_items * (unsigned)(p.n_q_heads / p.heads_per_wg);
  hipLaunchKernelGGL(p.k_suffix && !one_tile ? duo::attn_duo_suffix_kernel : duo::attn_duo_kernel, dim3(grid + attn::append_wgs(p)), dim3(256), duo::Cfg::LDS_BYTES, stream, p);
  return hipGetLastError();
}

}  // namespace calvo

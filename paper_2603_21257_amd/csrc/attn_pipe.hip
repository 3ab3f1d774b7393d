// The attention kernel for long suffixes (attn_pipeline.h): workgroup = 4 query heads of one KV group x 64 tokens (256 rows in
// any case), four waves of 64 rows, one workgroup per CU, K and V rings of eight 8 KiB slots.
// Also the kernel that merges the partial results of tiles whose context was cut into pieces.
#include "attn_pipeline.h"

namespace calvo {
namespace pipe {

using namespace attn;
using Cfg = PipeCfg<4, 8, 2>;

// 480 of the 512 registers that a wave alone on its SIMD may have (the attribute counts half of
// the unified VGPR+AGPR file on this target): the remaining 32 per SIMD lane let a wave of the
// ingest scatter kernel become resident next to the attention waves, so the loading stage keeps
// moving while attention occupies every CU.
__global__ void __launch_bounds__(256, 1) __attribute__((amdgpu_num_vgpr(240))) attn_pipe_kernel(AttnParams p) {
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  clock_begin(p.clock);
  if (append_wg(p)) return;
  attn_pipeline<Cfg>(p, smem);
}

// Combines the pieces of split tiles: for every row and head, with m = max_c m_c,
//     O = sum_c 2^(m_c - m) O_c  /  sum_c 2^(m_c - m) l_c
// (the pieces' O_c, l_c are sums of weights 2^(x - m_c), x the exponent of a score).  A piece in which a
// row saw no key has l_c = 0 and drops out; every other one counts, also with l_c = NaN or a weight that is 0 here.
// What counts is how many loads are in flight and how often a chain of loads is paid: the partials are a few MB to a few tens
// of MB that the caches still hold.  A wave merges ROWS rows: lane (row, i) reads (m, l) of piece i of its row, the maximum and
// the denominator are reductions over the row's lanes, and the O rows (64 lanes x 8 bytes) are fetched LOADS at a time -
// LOADS / ROWS pieces of ROWS rows - with each piece's weight taken from its lane.  The first of them are asked for before the
// weights are known, and the work item holds what is needed of its request, so that two loads in a row stand in front of
// them, both on the scalar unit (a vector load each and the request behind them before).
// ROWS = 1 while a wave per row fits the chip's wave slots, with all of 32 pieces in flight while half of them do; ROWS = 4 beyond
// (32000 rows x 4 pieces: 10.8 us, bandwidth; a wave per row 22.6 in four rounds).
// us a call of one caller, 16 loads behind the weights / this: 28096+28 tokens 31.1 / 30.2, 8192+1 15.8 / 15.3, 2048+209 27.7 / 26.0,
// 8192+28 (16Q/2KV) 20.1 / 19.1, 4096+1000 80.8 / 79.4.
constexpr unsigned kMergeSingleRows = 8192;      // 256 CUs x 32 waves

template <int ROWS, int LOADS>
__global__ void __launch_bounds__(256) merge_splits_kernel(AttnParams p, const int32_t* split_tiles) {
  const int NW = p.row_blocks_per_wg;
  const int HW = p.heads_per_wg, NHG = p.n_q_heads / HW, TPW = NW / HW;
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  constexpr int kLanes = 64 / ROWS, kPieces = LOADS / ROWS;
  constexpr int kWgs = 8 / ROWS;                                 // workgroups per 32-row slot
  // a head group is merged on the XCD whose L2 its pieces were written through (the workgroup order of
  // attn_pipeline.h): 2048+209 tokens 33.8 -> 28.3 us a call of one caller, 21.5 -> 20.7 with three in turn, 4096+28 20.2 -> 17.8
  // and 14.1 -> 13.3
  int hg, rest = blockIdx.x;
  if ((NHG & 7) == 0) {
    const int per = NHG >> 3;
    hg = (rest & 7) * per + (rest >> 3) % per;
    rest = (rest >> 3) / per;
  } else {
    hg = rest % NHG;
    rest /= NHG;
  }
  const int row0 = ((rest % kWgs) * 4 + wave) * ROWS;
  const int slot_id = rest / kWgs;
  const int wave_slot = slot_id % NW;
  const int first = ((const_i32p)(uintptr_t)split_tiles)[slot_id / NW];
  const WorkItem wi = load_item(p.items, first);
  const int tok0 = wi.q_tile * 32 * TPW + (wave_slot / HW) * 32 + row0;
  const int n_rows = min(ROWS, wi.suffix_len - tok0);
  if (n_rows <= 0) return;
  const int hq = hg * HW + wave_slot % HW;
  const int n = wi.n_splits;
  // row r of piece c: base + c * step + r
  const int64_t base = (((int64_t)first * NHG + hg) * NW + wave_slot) * 32 + row0;
  const int64_t step = (int64_t)NHG * NW * 32;
  const int my_row = lane / kLanes, my_c = lane % kLanes;
  const bool row_ok = my_row < n_rows;            // rows past the suffix were never written
  const f32x2* ml = (const f32x2*)p.part_ml + base + my_row;
  const f32x2* po = (const f32x2*)(p.part_o + base * kD) + lane;
  auto piece_ml = [&](int c) -> f32x2 { return row_ok && c < n ? ml[c * step] : (f32x2){-INFINITY, 0.f}; };
  f32x2 v[kPieces][ROWS];
  auto fetch = [&](int c) {                       // past the end: the last piece / row again, dropped below
#pragma unroll
    for (int i = 0; i < kPieces; i++)
#pragma unroll
      for (int r = 0; r < ROWS; r++) v[i][r] = po[min(c + i, n - 1) * step * (kD / 2) + min(r, n_rows - 1) * (kD / 2)];
  };

  f32x2 mine = piece_ml(my_c);
  fetch(0);                                       // on their way while the weights are found
  __builtin_amdgcn_sched_barrier(0);
  float m = mine[0];
  for (int c = my_c + kLanes; c < n; c += kLanes) m = fmaxf(m, piece_ml(c)[0]);
#pragma unroll
  for (int o = kLanes / 2; o > 0; o >>= 1) m = fmaxf(m, __shfl_xor(m, o));
  float l = 0.f, wgt = -1.f;                      // a negative weight drops out
  f32x2 acc[ROWS];
#pragma unroll
  for (int r = 0; r < ROWS; r++) acc[r] = (f32x2){0.f, 0.f};
  for (int c0 = 0; c0 < n; c0 += kPieces) {
    const int in_lanes = c0 % kLanes;
    if (in_lanes == 0) {                          // this lane's piece of the next kLanes
      if (c0) mine = piece_ml(c0 + my_c);
      wgt = -1.f;
      if (row_ok && c0 + my_c < n && mine[1] != 0.f) {
        wgt = __builtin_amdgcn_exp2f(mine[0] - m);
        l = __builtin_fmaf(wgt, mine[1], l);
      }
    }
    if (c0) fetch(c0);
#pragma unroll
    for (int i = 0; i < kPieces; i++) {
      if (c0 + i >= n) break;
#pragma unroll
      for (int r = 0; r < ROWS; r++) {
        const float w = __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, wgt), r * kLanes + in_lanes + i));
        if (!(w < 0.f)) {
          acc[r][0] = __builtin_fmaf(w, v[i][r][0], acc[r][0]);
          acc[r][1] = __builtin_fmaf(w, v[i][r][1], acc[r][1]);
        }
      }
    }
  }
#pragma unroll
  for (int o = kLanes / 2; o > 0; o >>= 1) l += __shfl_xor(l, o);
  unsigned short* out = (unsigned short*)p.out + ((int64_t)(wi.q_off + tok0) * p.n_q_heads + hq) * kD + 2 * lane;
#pragma unroll
  for (int r = 0; r < ROWS; r++) {
    if (r >= n_rows) break;
    const float inv = 1.f / __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, l), r * kLanes));
    bf16x2 w;
    w[0] = (__bf16)(acc[r][0] * inv);
    w[1] = (__bf16)(acc[r][1] * inv);
    *(unsigned int*)(out + (int64_t)r * p.n_q_heads * kD) = __builtin_bit_cast(unsigned int, w);
  }
  if (threadIdx.x == 0) clock_end_tail(p.clock.words);
}

}  // namespace pipe

int attn_pipe_tile_tokens(int heads_per_wg) { return 32 * pipe::Cfg::HB * pipe::Cfg::NW / heads_per_wg; }

hipError_t attn_pipe_prepare() {
  return hipFuncSetAttribute((const void*)pipe::attn_pipe_kernel, hipFuncAttributeMaxDynamicSharedMemorySize,
                             pipe::Cfg::LDS_BYTES);
}

hipError_t launch_attn_pipe(const AttnParams& p, hipStream_t stream) {
  if (p.n_items <= 0) return hipSuccess;
  const unsigned grid = (unsigned)p.n_items * (unsigned)(p.n_q_heads / p.heads_per_wg);
  hipLaunchKernelGGL(pipe::attn_pipe_kernel, dim3(grid + attn::append_wgs(p)), dim3(64 * pipe::Cfg::NW), pipe::Cfg::LDS_BYTES, stream, p);
  return hipGetLastError();
}

hipError_t launch_merge_splits(const AttnParams& p, const int32_t* split_tiles, int n_split_tiles, hipStream_t stream) {
  if (n_split_tiles <= 0) return hipSuccess;
  const unsigned slots = (unsigned)n_split_tiles * (unsigned)(p.n_q_heads / p.heads_per_wg) * (unsigned)p.row_blocks_per_wg;
  if (slots * 32u <= pipe::kMergeSingleRows / 2)
    hipLaunchKernelGGL((pipe::merge_splits_kernel<1, 32>), dim3(slots * 8u), dim3(256), 0, stream, p, split_tiles);
  else if (slots * 32u <= pipe::kMergeSingleRows)
    hipLaunchKernelGGL((pipe::merge_splits_kernel<1, 16>), dim3(slots * 8u), dim3(256), 0, stream, p, split_tiles);
  else
    hipLaunchKernelGGL((pipe::merge_splits_kernel<4, 16>), dim3(slots * 2u), dim3(256), 0, stream, p, split_tiles);
  return hipGetLastError();
}

}  // namespace calvo

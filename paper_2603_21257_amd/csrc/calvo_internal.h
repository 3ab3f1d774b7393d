// Internal declarations shared by the host API and the HIP kernels of libcalvo.
// Not part of the public ABI (see include/calvo.h).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "attn_plan.h"

namespace calvo {

// One request as the attention kernels see it (int32 x 4, device memory).
struct ReqDesc {
  int32_t table_off;  // offset of this request's block table inside the table array
  int32_t prefix_len; // P (tokens)
  int32_t suffix_len; // S (tokens)
  int32_t q_off;      // first row of this request inside q / out / k_suffix / v_suffix
};


// When an attention launch ran, in ticks of the constant counter (100 MHz), in device memory per layer: the
// first workgroup stores the start, the first wave of every workgroup raises an end when it is done (the counter
// only grows, so the words need no reset between launches).  A pair of timing events around the launch costs 8 us of host time and two
// barrier packets per call, more than the launch itself (2.5 us).  The ends are kept in sixteen words a cache
// line apart: on a single word 2048 workgroups that finish together queue up for 18 us.
constexpr int kClockEnds = 16, kClockStride = 16;                              // words; stride in 8-byte words
constexpr int kClockWords = (1 + kClockEnds) * kClockStride;                   // per layer: the start's line, then the ends
struct LaunchClock {
  unsigned long long* words;
  int32_t starts;           // this launch is the first of its call
};
__device__ inline void clock_begin(const LaunchClock& k) {
  // a scalar branch: all lanes of the first wave store the same value
  if (k.starts && blockIdx.x == 0 && __builtin_amdgcn_readfirstlane(threadIdx.x) == 0) k.words[0] = wall_clock64();
}
__device__ inline void clock_end(unsigned long long* words) {
  atomicMax(words + (1 + blockIdx.x % kClockEnds) * kClockStride, (unsigned long long)wall_clock64());
}
// for launches of many short workgroups: the last ones to be dispatched stand for all
__device__ inline void clock_end_tail(unsigned long long* words) {
  if (blockIdx.x + 256 >= gridDim.x) clock_end(words);
}

struct AttnParams {
  const void* q;
  void* out;
  const void* pool_layer;   // this layer's [pool_blocks][2][B][Hkv][D]
  const ReqDesc* reqs;
  const WorkItem* items;
  const int32_t* item_index; // NULL, or n_items indices into items: the work items of this launch
  const int32_t* tables;    // per request: its block table, padded with copies of the last entry
  const int64_t* blk_offs;  // per request: slot * block_bytes of the even blocks, then of the odd blocks
  int32_t n_items;          // tiles over all requests
  int32_t n_q_heads, n_kv_heads, head_dim;
  int32_t heads_per_wg;     // MFMA kernel: 1, 2 or 4 query heads of one KV group per workgroup
  int32_t tile_tokens;      // suffix tokens per work item
  int32_t row_blocks_per_wg;     // blocks of 32 query rows in an attention workgroup (8 or 4): layout of the split-KV partials
  float scale;              // softmax scale (natural-exponent units)
  // split-KV partial results, used by work items with n_splits > 1: per work item, head group, block of 32 rows
  // (head of the group x 32-token block of the tile): part_o [32 rows][D] fp32 unnormalised,
  // part_ml [32 rows][2] = (softmax reference in exponent units, i.e. score * scale * log2 e, row sum)
  float* part_o;
  float* part_ml;
  // Suffix K / V, or NULL: the keys past the prefixes are then read from here and stored to the pool by the launch itself
  // (tables), no append launch in front of it.
  const void* k_suffix;
  const void* v_suffix;
  LaunchClock clock;
  int32_t n_reqs, total_tokens;
  int32_t attn_wgs;         // workgroups of the grid that work on tiles; those behind them append the suffix rows
};

// workgroups that append the suffix rows in a launch of the pipelined kernels: four 16-byte chunks of K and of V per thread
inline unsigned append_wgs(int total_tokens, int n_kv_heads) { return (unsigned)(((int64_t)total_tokens * n_kv_heads * 16 + 1023) / 1024); }

struct AppendParams {
  const void* k_suffix;
  const void* v_suffix;
  void* pool_layer;
  const ReqDesc* reqs;
  const int32_t* tables;
  int32_t n_reqs;
  int32_t total_tokens;
  int32_t row_chunks;       // 16-byte chunks in one token's K (or V) row: Hkv*D*elt/16
};

// Scatter n_blocks consecutive source blocks to the pool slots table[0..n_blocks).
hipError_t launch_scatter_blocks(const void* src, void* pool_layer, const int32_t* table, int64_t n_blocks,
                                 int32_t blk_bytes, int grid, hipStream_t stream);
hipError_t launch_suffix_append(const AppendParams& p, hipStream_t stream);
// n_words 32-bit words of page-locked host memory to the device; both 16-byte aligned
hipError_t launch_upload_words(const int32_t* pinned_src, int32_t* dst, size_t n_words, hipStream_t stream);
// start and end of a layer's attention launch (LaunchClock) to two words of page-locked host memory
hipError_t launch_clock_out(const unsigned long long* words, unsigned long long* pinned, hipStream_t stream);
// test hook: occupies `stream` for about us microseconds (bounded), see kernels_ingest.hip
hipError_t launch_delay(int us, hipStream_t stream);

// The packed-rows kernel (attn_rows.hip): fp32 pools and head widths other than 128.
struct RowsParams {
  const void* q;
  const void* k_suffix;     // suffix K and V are read from here and stored to the pool by the launch ...
  const void* v_suffix;     // ... or NULL: they are in the pool already
  void* out;
  void* pool_layer;
  const ReqDesc* reqs;      // read if n_reqs > 1 ...
  ReqDesc one;              // ... the request of a batch of one: no descriptor load in front of the block table
  const WorkItem* items;    // NULL: uncut tiles, found by counting through the requests
  const int32_t* tables;
  int32_t n_reqs;
  int32_t n_q_heads, n_kv_heads, head_dim;
  uint32_t group;           // query heads per KV head
  float scale;
  // partial results of cut tiles: per work item and KV head [rows][padded head_dim] in part_o, [rows][2] in part_ml
  float* part_o;
  float* part_ml;
  LaunchClock clock;
};
// raises the kernel's dynamic LDS limit; once per device and shape, before the first launch
hipError_t attn_rows_prepare(int dtype, int head_dim, int tile_rows);
hipError_t launch_attn_rows(const RowsParams& p, int dtype, int tile_rows, int n_items, const int32_t* split_tiles, int n_split_tiles,
                            hipStream_t stream);
// The pipelined bf16 / head-dim-128 kernels (attn_pipeline.h).  The *_prepare calls raise the
// kernels' dynamic LDS limit; once per device, before the first launch.
hipError_t attn_pipe_prepare();
hipError_t attn_duo_prepare();
hipError_t launch_attn_pipe(const AttnParams& p, hipStream_t stream);
hipError_t launch_attn_duo(const AttnParams& p, bool one_tile, hipStream_t stream);
int attn_duo_tile_tokens(int heads_per_wg);
// combines the pieces of every split tile into out (bf16); n_split_tiles entries in split_tiles =
// indices of the first work item of each split tile
hipError_t launch_merge_splits(const AttnParams& p, const int32_t* split_tiles, int n_split_tiles, hipStream_t stream);
int attn_pipe_tile_tokens(int heads_per_wg);

constexpr int kBlockTokens = 16;
// Entries appended to every request's device-side block table (copies of its last entry).  No kernel needs more than the one
// that makes the count even; the rest keeps the two halves of the block offsets (even and odd blocks, calvo_api.hip), which the waves
// of a workgroup read side by side, from lying a power of two apart: with 4096 or 8192 blocks and no padding they do, and
// 61440+4096 tokens take 3083 -> 3160 us a call, 122880+8192 (64Q/8KV) 24500 -> 24860.
constexpr int kTablePad = 32;
}  // namespace calvo

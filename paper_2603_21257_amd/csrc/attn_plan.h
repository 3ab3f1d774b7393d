// Host-side planning of an attention launch: which kernel, which tiles, how many split-KV pieces.
// No device types here: the file is shared by the HIP translation units and by plain C++.
#pragma once
#include <cmath>
#include <cstdint>
#include <utility>
#include <vector>

namespace calvo {

// which of the bf16 / head-dim-128 kernels serves a batch with these lengths (attn_plan.cpp);
// the other calls take its answer
constexpr int kAttnPipe = 3;   // 64 query rows per wave, 64-token tiles
constexpr int kAttnDuo = 4;    // 32 query rows per wave, two workgroups per CU, 32-token tiles
int attn_mfma_choose(const int32_t* prefix_blocks, const int32_t* suffix_lens, int n_reqs, int heads_per_wg, int n_head_groups, int n_cus,
                     bool by_rows = false);      // by_rows: by the empty rows of the tiles alone
int attn_mfma_tile_tokens(int variant, int heads_per_wg);
int attn_mfma_row_blocks(int variant);           // blocks of 32 query rows in a workgroup

// query heads of one KV group that share a workgroup: 4, 2 or 1 (the largest that divides the group)
inline int attn_heads_per_wg(int n_q_heads, int n_kv_heads) {
  const int g = n_q_heads / n_kv_heads;
  return (g % 4 == 0) ? 4 : (g % 2 == 0) ? 2 : 1;
}

struct PlanTile {
  int32_t req, tile;
  int32_t n_sub;      // 32-key sub-tiles its rows see (prefix + the suffix up to the tile's end)
};

struct PlanParams {
  int n_head_groups;  // workgroups per work item
  int wg_slots;       // workgroups resident on the device at a time
  int split_min;      // shortest piece of a long tile, in sub-tiles (plan_piece_len scales it down for short ones)
  int split_fill;     // cost of a workgroup's pipeline fill and drain, in sub-tile steps
  int force_splits;   // > 0: cut every tile into this many pieces (test knob)
  // Few partial results: pieces never below split_min, the same number of every tile, no counts between the coarse ones.
  bool long_pieces = false;
  int step_cost = 0;  // packed-rows kernel: cost of a wave's 32-key step, in units of split_fill; else 0
  int alone = 0;      // > 0: up to this many workgroups have a CU each, which makes them faster (attn_plan.cpp)
  bool rounded = false;   // piece lengths of the form 8k + 2 instead of even ones
};

// A work item is one workgroup's share of the attention of one request: a tile of suffix tokens
// (tile_tokens of them) over the sub-tile range [sub_begin, sub_end) of its context (32-key
// sub-tiles).  Normally a tile is one work item covering its whole context; a tile may be cut into
// n_splits > 1 pieces (split-KV), which then run as separate workgroups, write partial results
// (unnormalised O, running maximum, row sum) and are combined by a merge kernel; the pieces of one
// tile are consecutive work items.  The device reads this struct as it is.
struct WorkItem {
  int32_t req;
  int32_t q_tile;     // tile index inside the request's suffix
  int32_t sub_begin;  // first 32-key sub-tile of this piece
  int32_t sub_end;    // one past its last sub-tile (the last piece ends at the tile's causal limit)
  int32_t n_splits;   // pieces the tile is cut into; 1 = the kernel writes the final output itself
  int32_t first_item; // index of the tile's first piece
  // of the request, so that the merge reads them from here (build_descriptor_blob)
  int32_t q_off, suffix_len;
};

struct PlanItems {
  std::vector<WorkItem> items;
  std::vector<int32_t> split_tiles;              // first work item of every cut tile
  std::vector<std::vector<int32_t>> groups;      // chunk-granular layers: work item indices per launch; else empty
};

// the batch's tiles of tile_tokens suffix tokens, heaviest first
std::vector<PlanTile> plan_tiles(const int32_t* prefix_blocks, const int32_t* suffix_lens, int n_reqs, int tile_tokens);

// length of the pieces a tile of n_sub sub-tiles is cut into when `want` pieces are asked for of the
// longest tile, which has n_max
int plan_piece_len(int n_sub, int n_max, int want, const PlanParams& p);

// pieces of the longest tile to ask for (1 = no cut), from a replay of the launch; a cut makes at most max_slots
// (piece, head group) pairs (partial results there is room for).  found, if asked for: what the replay makes of them, in units
// of split_fill; 0 where the number of pieces is forced, infinite where no launch is shorter than limit
struct PlanCost {
  double span = 0.;   // length of the launch and its merge
  double load = 0.;   // what they keep the whole chip busy for
};
int plan_pieces(const std::vector<PlanTile>& tiles, const PlanParams& p, int64_t max_slots = INT64_MAX, PlanCost* found = nullptr,
                double limit = HUGE_VAL);

// work items of a whole-layer launch: every tile cut into pieces of plan_piece_len
PlanItems plan_items(const std::vector<PlanTile>& tiles, int want, const PlanParams& p);

// Tilings of the packed-rows kernel (attn_rows.hip): (token, head) rows of one KV head per work item, what a wave's step of
// 32 keys costs and what the start and end of a workgroup do.
struct RowsShape {
  int tile_rows, step_cost, fill;
  int slots;          // partial-result slots (32 rows of 128 floats) of a work item and KV head
};
bool attn_rows_has_large(bool f32, int head_dim);
RowsShape attn_rows_shape(bool f32, int head_dim, bool large);

// The tiling of a batch, its tiles and the pieces that the longest is asked to be cut into.  force_tile: 1 takes the smaller
// tiling, 2 the larger one where there is one.
struct RowsPlan {
  RowsShape shape;
  std::vector<PlanTile> tiles;
  int want;
  bool large;
};
RowsPlan plan_rows(bool f32, int head_dim, const int32_t* prefix_blocks, const int32_t* suffix_lens, int n_reqs, int group,
                   int n_kv_heads, int n_cus, int force_splits, int64_t max_slots, int force_tile = 0);

// A decision about tiling and pieces (a replay of the launch), which depends only on the batch's lengths, and the lengths that it
// was made for: the following layers take it over.
struct KeptPlan {
  int want = 1;
  bool large = false;      // packed rows: the tiling
  // decide() sets them, unless they are those of these lengths already.  If it throws, no lengths are known.
  template <typename F>
  const KeptPlan& of(int variant, const int32_t* prefix_blocks, const int32_t* suffix_lens, int n_reqs, F&& decide) {
    std::vector<int64_t> mine;
    mine.reserve(2 * (size_t)n_reqs + 1);
    mine.push_back(variant);
    for (int r = 0; r < n_reqs; r++) { mine.push_back(prefix_blocks[r]); mine.push_back(suffix_lens[r]); }
    if (mine == key) return *this;
    key.clear();
    decide(*this);
    key = std::move(mine);
    return *this;
  }

 private:
  std::vector<int64_t> key;
};

// the batch's tiles of tile_rows rows, heaviest first (group: query heads per KV head)
std::vector<PlanTile> plan_row_tiles(const int32_t* prefix_blocks, const int32_t* suffix_lens, int n_reqs, int group, int tile_rows);
PlanParams rows_plan_params(RowsShape shape, int n_kv_heads, int n_cus, int force_splits);

// Work items of a layer that was loaded in n_chunks chunks of chunk_blocks block indices (even): piece
// k of a tile covers the sub-tiles of chunk k that lie wholly inside the request's prefix and goes
// into launch k, which needs blocks below (k + 1) * chunk_blocks only; what is left of the tile (the
// end of the prefix that shares a sub-tile with the suffix, the suffix itself) is its last piece, in
// launch n_chunks, which needs the whole layer.
PlanItems plan_items_chunked(const std::vector<PlanTile>& tiles, const int32_t* prefix_blocks, int chunk_blocks, int n_chunks);

}  // namespace calvo

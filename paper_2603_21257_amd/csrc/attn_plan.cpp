// Planning of an attention launch on the host.  A tile of suffix tokens normally is one work item
// that walks its whole context.  Short suffixes over long contexts (the paper's main regime,
// Section 2.2 and Table 1) give too few tiles for the chip, and some batches give a workgroup
// count just above a whole number of rounds; in both cases every tile's context is cut into pieces
// that run as separate workgroups and are merged afterwards.  How many pieces is decided by
// replaying the launch: workgroups start in grid order on the first free workgroup slot, a piece
// costs its sub-tiles plus a fixed pipeline fill and drain, cut tiles pay the merge.
#include "attn_plan.h"

#include <algorithm>
#include <cstdlib>
#include <functional>

#include "../../include/calvo.h"

namespace calvo {

int attn_pipe_tile_tokens(int heads_per_wg);
int attn_duo_tile_tokens(int heads_per_wg);

// Two kernels serve bf16 / head-dim-128 batches: kAttnPipe (64 query rows per wave, 64-token tiles for four
// heads: half the K/V traffic into LDS and out of it per query row) and kAttnDuo (32 rows per wave, two
// 4-wave workgroups per CU, 32-token tiles).  The smaller tiles win where half of a 64-token tile would be empty (the short
// queries of the paper's Table 1), and where the whole batch is little work: they spread it over twice as many workgroups,
// which fill and drain faster.  Measured, us a call of one caller, kAttnPipe / kAttnDuo (in brackets the 32-key steps of
// kAttnPipe per CU):
//   32Q/8KV  0+1024 tokens (8.5) 34.8 / 25.6, 1024+1000 (25) 52.0 / 38.7, 8192+256 (33) 49.0 / 50.2, 2048+1000 (41) 59.6 / 50.9,
//            16384+256 (65) 72.1 / 75.9, 4096+1000 (73) 82.8 / 79.1, 61440+4096 2961 / 3362
//   64Q/8KV  1024+1000 (49) 57.2 / 55.2, 4096+512 (68) 79.5 / 72.4, 2048+1000 (80) 80.9 / 82.2
//   40Q/8KV  (tiles of 256 / 128) 4096+512 (44) 61.9 / 60.9, 2048+1000 (52) 76.7 / 67.1, 4096+1000 (92) 114.6 / 107.8
//   16Q/8KV  (128 / 64) 4096+1000 (36) 54.4 / 55.9        8Q/8KV  (256 / 128) 4096+1000 (18) 43.6 / 40.8
// Over 1009 random batches of six layouts the sides cross at 100 steps and more where tiles are short; where they have 250
// steps and more (8K tokens of context), fill, drain and diagonal of the larger tiles matter less and the sides cross from 40
// on.  Between 40 and 60 steps the smaller tiles take 0.91 of the time on average (0.76 to 1.04): 2048+1000 as above, 40Q/8KV
// 688+412,480+924,1008+438,736+233 78.4 / 61.9, 16Q/8KV 80+446,8752+647 79.9 / 67.3.  One request whose suffix is a single
// tile of kAttnPipe has no more tiles to gain from, and takes its append along where launch_layer allows it: 2048+64 (2) 23.1 / 20.7,
// 8192+64 (8) 29.6 / 26.2, 16384+64 (16)
// 35.7 / 33.6, 64Q/8KV 16384+64 (32) 45.9 / 49.6, 40Q/8KV 8192+256 (41) 56.9 / 57.9, 8Q/8KV 16384+256 (16) 38.9 / 33.9; without suffix
// arrays 16384+64 35.4 / 31.3, 64Q/8KV 16384+64 45.2 / 47.4.  The sides cross between 16 and 32 there, above the line.  The environment
// variable CALVO_ATTN_VARIANT (3 or 4, read per call: tests switch it inside one process) forces one.
constexpr int kPipeStepsPerCu = 60, kPipeStepsPerCuLong = 40, kLongTile = 250, kPipeStepsPerCuOneTile = 12;

int attn_mfma_choose(const int32_t* prefix_blocks, const int32_t* suffix_lens, int n_reqs, int heads_per_wg, int n_head_groups, int n_cus,
                     bool by_rows) {
  const char* e = getenv("CALVO_ATTN_VARIANT");
  if (e && (e[0] == '3' || e[0] == '4') && e[1] == 0) return e[0] - '0';
  // query rows the tiles of each kernel would hold, empty ones included, and the steps of kAttnPipe
  const int t3 = attn_pipe_tile_tokens(heads_per_wg), t4 = attn_duo_tile_tokens(heads_per_wg);
  int64_t rows3 = 0, rows4 = 0, steps = 0, n_tiles = 0;
  for (int r = 0; r < n_reqs; r++) {
    const int64_t tiles = (suffix_lens[r] + t3 - 1) / t3;
    rows3 += tiles * t3;
    n_tiles += tiles;
    rows4 += (int64_t)((suffix_lens[r] + t4 - 1) / t4) * t4;
    steps += tiles * (16 * (int64_t)prefix_blocks[r] + (suffix_lens[r] + t3) / 2) / 32;
  }
  if (rows3 * 9 > rows4 * 10) return kAttnDuo;                // the larger tiles would carry over 10 % more rows
  const int line = n_reqs == 1 && suffix_lens[0] <= t3 ? kPipeStepsPerCuOneTile
                   : steps >= kLongTile * n_tiles     ? kPipeStepsPerCuLong
                                                      : kPipeStepsPerCu;
  return !by_rows && steps * n_head_groups < (int64_t)line * n_cus ? kAttnDuo : kAttnPipe;
}

// blocks of 32 query rows in a workgroup: a wave each, but two per wave in kAttnPipe
int attn_mfma_row_blocks(int variant) { return variant == kAttnPipe ? 8 : 4; }

int attn_mfma_tile_tokens(int variant, int heads_per_wg) {
  return variant == kAttnDuo ? attn_duo_tile_tokens(heads_per_wg) : attn_pipe_tile_tokens(heads_per_wg);
}

std::vector<PlanTile> plan_tiles(const int32_t* prefix_blocks, const int32_t* suffix_lens, int n_reqs, int tile_tokens) {
  std::vector<PlanTile> tiles;
  for (int r = 0; r < n_reqs; r++) {
    const int nt = (suffix_lens[r] + tile_tokens - 1) / tile_tokens;
    for (int t = 0; t < nt; t++) {
      const int64_t keys = (int64_t)prefix_blocks[r] * 16 + std::min<int64_t>((int64_t)(t + 1) * tile_tokens, suffix_lens[r]);
      tiles.push_back({r, t, (int32_t)((keys + 31) / 32)});
    }
  }
  std::stable_sort(tiles.begin(), tiles.end(), [](const PlanTile& a, const PlanTile& b) { return a.n_sub > b.n_sub; });
  return tiles;
}

// The kernels run a piece of n sub-tiles as a fill step, pairs of steady steps and one (n even) or two drain steps.
// The shortest piece is a 32nd of the tile, between 8 and split_min (48): a piece of 8 sub-tiles is mostly
// fill, but with one or two tiles the alternative is an idle chip.  Measured with the kernels before the present ones (8B
// shape, us a call with three callers in turn, floor 48 -> this): 2048+1 tokens 29.2 -> 13.7, 8192+1 31.0 -> 14.1, 16384+28
// 34.2 -> 23.0, 2048+209 34.3 -> 23.8; from 28K cached tokens on the two differ by less than 4 %.
int plan_piece_len(int n_sub, int n_max, int want, const PlanParams& p) {
  const int floor = p.step_cost ? 1 : p.long_pieces ? p.split_min : std::min(p.split_min, std::max(8, n_sub / 32));
  // a shorter tile gets as many pieces as it has of the longest tile's piece lengths (a quarter over is let go)
  if (!p.force_splits && !p.long_pieces) want = (int)(((int64_t)4 * n_sub * want + 3 * (int64_t)n_max - 1) / (4 * (int64_t)n_max));
  const int n = std::max(1, std::min(want, p.force_splits ? n_sub : n_sub / floor));
  int len = (n_sub + n - 1) / n;
  if (p.step_cost) return (len + 3) / 4 * 4;       // packed rows: the same number of wave steps on each of the four SIMDs
  if (n > 1 && !p.force_splits) len = p.rounded ? (len + 5) / 8 * 8 + 2 : (len + 1) / 2 * 2;
  return len;
}

// kAttnDuo: what a step of a workgroup costs that has its CU to itself, of a step of one that shares it (32Q/8KV, 0.69 us
// against 0.95 at 65536+100 tokens).  What this decides: 61440+28 tokens in 30 pieces (240 workgroups) 51 us a call, in 39 (312) 66;
// 8192+100 in 8 pieces (256) 31.9, in 16 (512) 36.3.  An uncut launch that is alone saves a merge at the cost of such steps, not
// at its full price: 1648+7 tokens (16Q/8KV, 8 workgroups uncut) take 14.5 us a call in 6 pieces, 27.2 uncut, and 1712+428
// (64Q/8KV, 224 uncut) 38.9 uncut, 49.1 in two.
constexpr double kAlone = 0.7;

int plan_pieces(const std::vector<PlanTile>& tiles, const PlanParams& p, int64_t max_slots, PlanCost* found, double limit) {
  if (found) *found = {};
  if (p.force_splits) return p.force_splits;
  const int64_t wgs = (int64_t)tiles.size() * p.n_head_groups;
  if (wgs <= 0) return 1;
  auto cost_of = [&](int64_t subs) { return (p.step_cost ? (subs + 3) / 4 * p.step_cost : subs) + p.split_fill; };
  if (wgs > 16 * (int64_t)p.wg_slots) {                         // many rounds: the last one hardly matters
    if (found) {
      for (const PlanTile& t : tiles) found->span += (double)(cost_of(t.n_sub) * p.n_head_groups) / p.wg_slots;
      found->load = found->span;
    }
    return 1;
  }
  static const std::vector<int> all = {1, 2, 3, 4, 5, 6, 7, 8, 9, 10, 11, 12, 13, 14, 15, 16, 20, 24, 32, 48, 64};
  static const std::vector<int> coarse = {1, 2, 3, 4, 5, 6, 8, 12, 16, 24, 32, 48, 64};
  const int n_max = tiles.front().n_sub;           // heaviest first
  int want = 1;
  double best = limit / 0.98;
  if (found) found->span = HUGE_VAL;
  std::vector<int64_t> heap;
  for (int n : p.long_pieces ? coarse : all) {
    if (n > 1 && wgs * n > (p.step_cost ? 4 : 16) * (int64_t)p.wg_slots) break;
    bool cut = false;
    int64_t end = 0, slots = 0, work = 0, longest = 0;
    for (const PlanTile& t : tiles) {
      const int len = plan_piece_len(t.n_sub, n_max, n, p);
      const int np = (t.n_sub + len - 1) / len;
      cut |= np > 1;
      slots += (int64_t)np * p.n_head_groups;
      work += ((np - 1) * cost_of(len) + cost_of(t.n_sub - (np - 1) * len)) * p.n_head_groups;
      longest = std::max(longest, cost_of(std::min(len, t.n_sub)));
    }
    if (n > 1 && slots > max_slots) break;
    // no order of the pieces beats the average load or the longest piece: most candidates need no replay
    const double step = slots <= p.alone ? kAlone : 1.;
    const double merge = (cut ? 1. : 1. - step) * p.split_fill;
    if (step * (double)std::max(work / p.wg_slots, longest) + merge >= best * 0.98) {
      if (!cut && n > 1) break;
      continue;
    }
    heap.assign((size_t)p.wg_slots, 0);            // min-heap of the times at which workgroup slots become free
    auto cmp = std::greater<int64_t>();
    for (const PlanTile& t : tiles) {
      const int len = plan_piece_len(t.n_sub, n_max, n, p);
      const int np = (t.n_sub + len - 1) / len;
      for (int k = 0; k < np; k++) {
        const int64_t cost = cost_of(std::min(t.n_sub, (k + 1) * len) - k * len);
        for (int h = 0; h < p.n_head_groups; h++) {
          std::pop_heap(heap.begin(), heap.end(), cmp);
          heap.back() += cost;
          end = std::max(end, heap.back());
          std::push_heap(heap.begin(), heap.end(), cmp);
        }
      }
    }
    const double span = step * (double)end + merge;
    if (span < best * 0.98) {                      // a cut has to win by 2 % over what is chosen so far
      best = span;
      want = n;
      if (found) *found = {span, (double)work / p.wg_slots + (cut ? p.split_fill : 0)};
    }
    if (!cut && n > 1) break;                       // longer cuts are refused by split_min: nothing changes
  }
  return want;
}

PlanItems plan_items(const std::vector<PlanTile>& tiles, int want, const PlanParams& p) {
  PlanItems out;
  for (const PlanTile& t : tiles) {
    const int len = plan_piece_len(t.n_sub, tiles.front().n_sub, want, p);
    const int n = (t.n_sub + len - 1) / len;
    const int32_t first = (int32_t)out.items.size();
    if (n > 1) out.split_tiles.push_back(first);
    for (int k = 0; k < n; k++) out.items.push_back({t.req, t.tile, k * len, std::min(t.n_sub, (k + 1) * len), n, first, 0, 0});
  }
  return out;
}

std::vector<PlanTile> plan_row_tiles(const int32_t* prefix_blocks, const int32_t* suffix_lens, int n_reqs, int group, int tile_rows) {
  std::vector<PlanTile> tiles;
  for (int r = 0; r < n_reqs; r++) {
    const int64_t rows = (int64_t)suffix_lens[r] * group;
    for (int64_t t = 0; t * tile_rows < rows; t++) {
      const int64_t keys = (int64_t)prefix_blocks[r] * 16 + (std::min((t + 1) * tile_rows, rows) - 1) / group + 1;
      tiles.push_back({r, (int32_t)t, (int32_t)((keys + 31) / 32)});
    }
  }
  std::stable_sort(tiles.begin(), tiles.end(), [](const PlanTile& a, const PlanTile& b) { return a.n_sub > b.n_sub; });
  return tiles;
}

// Packed-rows kernel, in tenths of a microsecond: start and end of a workgroup (a merge launch costs as much), and 32 keys for one wave's
// rows while the other waves of its SIMD are at work (measured per element type and padded head width).
// bf16, and fp32 above 128-wide heads, have a tiling of twice the rows, which reads K and V half as often: with the other one a workgroup waits for them (D = 64,
// 8192+512 tokens, 32Q/8KV: 96 us a call, 74 without the requests for K, 95 with a third of the products for the weights; 72 with twice
// the rows).  A step of twice the rows costs 1.0 (D = 256: one wave of a SIMD either way) to 1.8 as much.  The replay of both
// launches decides: the larger tiling where twice the length of its launch and once what it keeps the chip busy for come to 3 %
// less - unless its launch is the longer one and the smaller tiling leaves some of the chip idle (kFull) or is a tenth shorter.  One caller waits for a
// longer launch, whatever it leaves free for others: D = 256, 256+150 (6Q/3KV) 9.9 / 11.0 with three callers, 12.6 / 16.4 with one, D = 200,
// 432+31 (32Q/8KV) 10.0 / 11.1 and 13.2 / 16.7, D = 120, 0+515 (16Q/4KV) 10.2 / 10.7 and 12.5 / 16.0.  Time of the larger tiling over that of
// the smaller one with one caller and with three: over 46 such batches 1.27 and 1.02; longer launches of a full chip (46
// batches) 1.07 and 0.90; over 48 whose launch it makes up to a fifth shorter 0.96 and 0.91.
// us a call, three callers, 32Q/8KV, smaller / larger tiling, D = 64, 96, 256:
//   2048+64    10.0 / 12.7   16.1 / 16.1   26.8 / 21.7          2048+256   16.7 / 21.1   23.0 / 25.4   84.7 / 46.8
//   8192+128   29.3 / 27.3   41.6 / 39.3   148.2 / 83.7         0+512      11.8 / 10.7   16.3 / 12.8   37.4 / 25.9
//   5008+300   46.9 / 43.2   71.4 / 62.4   242.3 / 148.3        512+400 (8Q/8KV)   7.7 / 10.1   10.3 / 16.2   17.0 / 17.3
// fp32, D = 256, three callers (one): 2048+256 166.6 / 150.8 (169.5 / 156.9), 8192+512 1244 / 1073 (1220 / 1073), 4096+300 16Q/4KV 228.2 /
// 203.2 (232.3 / 209.5); the smaller one stays for 2048+64 58.7 / 54.8 (52.6 / 58.2), D = 200 48.4 / 51.7 (47.9 / 55.7), 1024+60 8Q/2KV
// 18.0 / 20.3 (20.4 / 25.4).  Up to D = 128 twice the rows gain nothing (matrix pipes): 8192+256, D = 64 136 / 141.
bool attn_rows_has_large(bool f32, int head_dim) { return !f32 || head_dim > 128; }

RowsShape attn_rows_shape(bool f32, int head_dim, bool large) {
  if (f32 && head_dim <= 128) return {32, head_dim <= 64 ? 23 : 48, 60, 1};
  if (f32) return large ? RowsShape{32, 78, 90, 2} : RowsShape{16, 43, 60, 1};
  if (head_dim <= 64) return large ? RowsShape{64, 10, 65, 2} : RowsShape{32, 6, 60, 1};
  if (head_dim <= 128) return large ? RowsShape{64, 16, 65, 2} : RowsShape{32, 9, 60, 1};
  return large ? RowsShape{32, 22, 90, 2} : RowsShape{16, 21, 60, 1};
}

PlanParams rows_plan_params(RowsShape shape, int n_kv_heads, int n_cus, int force_splits) {
  return {n_kv_heads, n_cus, 1, shape.fill, force_splits, false, shape.step_cost};
}

constexpr double kFull = 0.92;     // load of a launch that fills the chip, of its length
constexpr double kLonger = 1.1;

RowsPlan plan_rows(bool f32, int head_dim, const int32_t* prefix_blocks, const int32_t* suffix_lens, int n_reqs, int group,
                   int n_kv_heads, int n_cus, int force_splits, int64_t max_slots, int force_tile) {
  RowsPlan best;
  PlanCost best_cost;
  for (const bool large : {false, true}) {
    if (large && (!attn_rows_has_large(f32, head_dim) || force_tile == 1)) break;
    RowsPlan p;
    p.large = large;
    p.shape = attn_rows_shape(f32, head_dim, large);
    p.tiles = plan_row_tiles(prefix_blocks, suffix_lens, n_reqs, group, p.shape.tile_rows);
    const bool forced = !large || force_tile == 2;
    const double limit = forced ? HUGE_VAL : (best_cost.load >= kFull * best_cost.span ? kLonger : 1.) * best_cost.span + 0.5;
    PlanCost cost;
    p.want = plan_pieces(p.tiles, rows_plan_params(p.shape, n_kv_heads, n_cus, force_splits), max_slots / p.shape.slots, &cost, limit);
    if (forced || 2. * cost.span + cost.load < 0.97 * (2. * best_cost.span + best_cost.load)) {
      best = std::move(p);
      best_cost = cost;
    }
  }
  return best;
}

PlanItems plan_items_chunked(const std::vector<PlanTile>& tiles, const int32_t* prefix_blocks, int chunk_blocks, int n_chunks) {
  PlanItems out;
  out.groups.assign((size_t)n_chunks + 1, {});
  const int sub_per_chunk = chunk_blocks / 2;
  for (const PlanTile& t : tiles) {
    const int full = prefix_blocks[t.req] / 2;                   // sub-tiles wholly inside the prefix
    const int32_t first = (int32_t)out.items.size();
    const int n = (full + sub_per_chunk - 1) / sub_per_chunk;    // pieces that follow the chunks
    const int cut_end = std::min(full, n * sub_per_chunk);
    const int total = n + (cut_end < t.n_sub ? 1 : 0);
    if (total > 1) out.split_tiles.push_back(first);
    for (int k = 0; k < n; k++) {
      out.groups[(size_t)std::min(k, n_chunks)].push_back((int32_t)out.items.size());
      out.items.push_back({t.req, t.tile, k * sub_per_chunk, std::min(full, (k + 1) * sub_per_chunk), total, first, 0, 0});
    }
    if (cut_end < t.n_sub) {
      out.groups[(size_t)n_chunks].push_back((int32_t)out.items.size());
      out.items.push_back({t.req, t.tile, cut_end, t.n_sub, total, first, 0, 0});
    }
  }
  return out;
}

}  // namespace calvo

extern "C" int calvo_attn_plan_items(int32_t n_q_heads, int32_t n_kv_heads, int32_t n_cus, const int32_t* prefix_blocks,
                                     const int32_t* suffix_lens, int32_t n_reqs, int32_t chunk_blocks, int32_t* items,
                                     int32_t capacity, int32_t* n_items) {
  using namespace calvo;
  if (n_q_heads <= 0 || n_kv_heads <= 0 || n_q_heads % n_kv_heads != 0 || n_cus <= 0 || n_reqs < 0) return CALVO_EINVAL;
  if (n_reqs > 0 && (!prefix_blocks || !suffix_lens)) return CALVO_EINVAL;
  if (chunk_blocks < 0 || (chunk_blocks & 1) || capacity < 0 || (capacity > 0 && !items) || !n_items) return CALVO_EINVAL;
  int max_blocks = 0;
  for (int r = 0; r < n_reqs; r++) {
    if (prefix_blocks[r] < 0 || suffix_lens[r] < 0) return CALVO_EINVAL;
    max_blocks = std::max(max_blocks, prefix_blocks[r]);
  }
  const int hw = attn_heads_per_wg(n_q_heads, n_kv_heads);
  const int variant = attn_mfma_choose(prefix_blocks, suffix_lens, n_reqs, hw, n_q_heads / hw, n_cus);
  const std::vector<PlanTile> tiles = plan_tiles(prefix_blocks, suffix_lens, n_reqs, attn_mfma_tile_tokens(variant, hw));
  const PlanParams p{n_q_heads / hw, n_cus * (8 / attn_mfma_row_blocks(variant)), 48, 30, 0, false, 0, variant == kAttnDuo ? n_cus : 0};
  PlanItems pi;
  if (chunk_blocks > 0) {
    pi = plan_items_chunked(tiles, prefix_blocks, chunk_blocks, (max_blocks + chunk_blocks - 1) / chunk_blocks);
  } else {
    pi = plan_items(tiles, plan_pieces(tiles, p), p);
  }
  *n_items = (int32_t)pi.items.size();
  if ((int64_t)pi.items.size() > capacity) return CALVO_ENOMEM;
  std::vector<int32_t> launch(pi.items.size(), 0);
  for (size_t g = 0; g < pi.groups.size(); g++)
    for (int32_t i : pi.groups[g]) launch[(size_t)i] = (int32_t)g;
  for (size_t i = 0; i < pi.items.size(); i++) {
    const WorkItem& w = pi.items[i];
    int32_t* o = items + 6 * i;
    o[0] = w.req; o[1] = w.q_tile; o[2] = w.sub_begin; o[3] = w.sub_end; o[4] = w.n_splits; o[5] = launch[i];
  }
  return CALVO_OK;
}

extern "C" int calvo_attn_plan(int32_t n_q_heads, int32_t n_kv_heads, int32_t n_cus, const int32_t* prefix_blocks,
                               const int32_t* suffix_lens, int32_t n_reqs, int32_t* kernel, int32_t* tile_tokens,
                               int32_t* pieces, int32_t* n_workgroups) {
  using namespace calvo;
  if (n_q_heads <= 0 || n_kv_heads <= 0 || n_q_heads % n_kv_heads != 0 || n_cus <= 0 || n_reqs < 0) return CALVO_EINVAL;
  if (n_reqs > 0 && (!prefix_blocks || !suffix_lens)) return CALVO_EINVAL;
  for (int r = 0; r < n_reqs; r++)
    if (prefix_blocks[r] < 0 || suffix_lens[r] < 0) return CALVO_EINVAL;
  const int hw = attn_heads_per_wg(n_q_heads, n_kv_heads);
  const int variant = attn_mfma_choose(prefix_blocks, suffix_lens, n_reqs, hw, n_q_heads / hw, n_cus);
  const int tt = attn_mfma_tile_tokens(variant, hw);
  const std::vector<PlanTile> tiles = plan_tiles(prefix_blocks, suffix_lens, n_reqs, tt);
  PlanParams p{n_q_heads / hw, n_cus * (8 / attn_mfma_row_blocks(variant)), 48, 30, 0, false, 0, variant == kAttnDuo ? n_cus : 0};
  const int want = plan_pieces(tiles, p);
  int64_t items = 0;
  for (const PlanTile& t : tiles) {
    const int len = plan_piece_len(t.n_sub, tiles.front().n_sub, want, p);
    items += (t.n_sub + len - 1) / len;
  }
  if (kernel) *kernel = variant;
  if (tile_tokens) *tile_tokens = tt;
  if (pieces) *pieces = want;
  if (n_workgroups) *n_workgroups = (int32_t)(items * p.n_head_groups);
  return CALVO_OK;
}

// Paged causal GQA prefill attention on packed query rows: any head_dim <= 256 (multiple of 8), fp32 or
// bf16 storage, any group size.  This is the path for fp32 pools and for head widths the pipelined
// kernels (attn_pipeline.h) do not cover.
//
// Rows.  The (token, query head) pairs of one KV head are numbered row = token * group + head of the
// group; a workgroup owns NQB blocks of 16 consecutive rows, so that a one-token query with four heads per
// group fills a quarter of a block instead of one row of four tiles, and any group size packs without gaps.
//
// Both contractions run on the matrix pipes with the transposed formulation of attn_pipeline.h: lane
// (c = lane % 16, g = lane / 16) of a score tile holds query row c and keys 4g + r, r = 0..3, which is
// the operand order of the second product, so weights never cross lanes.
//   fp32: v_mfma_f32_16x16x4_f32 for both products (fp32 products and sums, as on the vector ALU).  The
//         k-slots may be any permutation of d if K and Q use the same one: a lane reads 16 bytes of its
//         key row (d = 16j + 4g ..) that feed four instructions.  For the second product a lane reads 16
//         bytes of a V row (d = 64q + 4c ..); output row m of instruction e is then d = 64q + 4m + e.
//   bf16: v_mfma_f32_16x16x32_bf16.  V rows are read 8 or 16 bytes per lane in the same way and the four
//         keys of a lane are brought together with v_perm_b32.  The weights stay fp32: each is split into
//         three bf16 terms (24 significant bits), three products with the exact bf16 V.  Two tilings (attn_rows_shape).
// Neither product tells an infinite or NaN V of a key that a row does not see from one that it does (0 times
// infinity), and the lower terms of a weight may be 0.  Such V leave sums that are not finite; a wave
// that finds one, or sums so large that weights above 1 (see the softmax reference) could be the reason, walks
// its keys again with every row adding its own keys' fp32 products, weights at most 1 (walk_by_row).
//
// No LDS on the way in: 16 keys are exactly one pool block, so a block's address is one scalar table
// lookup and the lanes' offsets inside it are constants; K and V go straight to registers, K(next) is
// requested as soon as the scores have consumed K and V(next) after the second product, or as soon as V is in
// operand order where all of it fits the registers that way (V_FIRST).  All waves of a
// workgroup work on the same rows: they take alternate steps of the keys and are combined through LDS at
// the end, which keeps short queries from being one long serial walk.  (Waves with rows of their own,
// which read the same K and V through the L1, were measured: the same within 3 % where there are rows
// enough to fill the chip, slower elsewhere.)  Contexts are cut into pieces across workgroups as well
// (attn_plan.cpp) and merged by merge_rows_kernel.
//
// The suffix's K and V are read from the caller's arrays where the launch is given them, and stored
// to the pool on the side; the append launch and its dependency go away.
//
// Softmax reference raised lazily: weights are taken against the maximum of an earlier step and the reference
// moves only when a score passes it by 2^16 (attn_pipeline.h, where it lies 16 above that maximum instead).
//
// What bounds it: fp32 the matrix pipes (a large fp32 product reaches 153 TFLOP/s on this part, a
// sixteenth of bf16; 2.3 us per 32 keys of a wave's 32 rows at D = 64 against 1.8 us of MFMA), bf16 the
// vector ALU (exponentials, weight split; at D = 64 in the larger tiling 0.9 us per step against 0.45 us of MFMA) and, in the
// smaller tiling, K and V on their way from L2.
// Measured against the kernel it replaces (one wave per token and head on the vector ALU), us a call:
// fp32 8Q/2KV D = 64, 1024+128 tokens 193 -> 12.5; bf16 16Q/4KV D = 64, 4096+300 tokens 1168 -> 22.7.
#include "attn_common.h"
#include "../../include/calvo.h"

#include <cfloat>

namespace calvo {
namespace rows {

using namespace attn;


// T_: storage.  DP: head_dim rounded up to 64, 128 or 256.  NQB: 16-row blocks of a tile.  KB: 16-key
// blocks per step.  NW: waves per workgroup.  FULL: head_dim == DP, no lane of a K or Q operand is past the end.
template <typename T_, int DP_, int NQB_, int KB_, int NW_, bool FULL_>
struct RowsCfg {
  typedef T_ T;
  static constexpr int DP = DP_, NQB = NQB_, KB = KB_, NW = NW_;
  static constexpr bool FULL = FULL_, F32 = sizeof(T_) == 4;
  static constexpr int E = sizeof(T_);
  static constexpr int KJ = F32 ? DP / 16 : DP / 32;         // 16-byte operand chunks of a K or Q row per lane
  static constexpr int VW = F32 ? 4 : (DP % 128 == 0 ? 8 : 4);   // consecutive d a lane reads of a V row
  static constexpr int VQ = DP / (16 * VW);                  // such reads per row
  static constexpr int NACC = VQ * VW;                       // 16 x 16 output tiles per 16-row block
  static constexpr bool V_FIRST = NACC <= (NW == 4 ? 8 : 4);      // V operands of a step in registers at a time
  static constexpr int ROWS = 16 * NQB;                      // rows of a tile
  static constexpr int UNITS = NQB * VQ * 4;                 // (row block, q, r): VW consecutive d of a lane's row
  static constexpr int LDS_O = NW * UNITS * VW * 64 * 4;     // all waves' accumulators
  static constexpr int LDS_BYTES = LDS_O + NW * ROWS * 8;
};

// Buffer resources: no stride, 32-bit data; an offset that lies in none
constexpr unsigned kPastEnd = 0xfffff000u, kBufferWord3 = 0x00020000u;

// by value: __builtin_bit_cast applied to an element of a vector reads element 0 with this compiler
__device__ inline float as_float(unsigned x) { return __builtin_bit_cast(float, x); }
__device__ inline unsigned bf16_rne(float x) {
  return (unsigned)__builtin_bit_cast(unsigned short, (__bf16)x);
}
__device__ inline float bf16_widen(unsigned b) { return __builtin_bit_cast(float, b << 16); }

template <class C>
__global__ void __launch_bounds__(64 * C::NW) attn_rows_kernel(RowsParams p) {
  typedef typename C::T T;
  constexpr int DP = C::DP, NQB = C::NQB, KB = C::KB, NW = C::NW, KJ = C::KJ, VW = C::VW, VQ = C::VQ, E = C::E;
  constexpr bool F32 = C::F32;
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  clock_begin(p.clock);
  const int c = lane & 15, g = lane >> 4;
  const int Hkv = p.n_kv_heads, Hq = p.n_q_heads, D = p.head_dim;
  const unsigned G = p.group;
  constexpr unsigned RT = C::ROWS;                             // rows of a work item

  // ---- work item (wave-uniform); a KV head's workgroups stay on one XCD where the heads divide over the eight
  int it, kv;
  {
    const int bid = blockIdx.x;
    if ((Hkv & 7) == 0) {
      const int per = Hkv >> 3, rest = bid >> 3;
      kv = (bid & 7) * per + rest % per;
      it = rest / per;
    } else {
      kv = bid % Hkv;
      it = bid / Hkv;
    }
  }
  int tile, sub_begin = 0, sub_end, n_splits = 1;
  bool first_piece = true;
  ReqDesc rd = p.one;                                          // a batch of one request comes with the launch
  if (p.items) {
    const WorkItem wi = p.items[it];
    tile = wi.q_tile; sub_begin = wi.sub_begin; sub_end = wi.sub_end; n_splits = wi.n_splits;
    first_piece = wi.first_item == it;
    if (p.n_reqs > 1) rd = p.reqs[wi.req];
  } else {
    // uncut tiles without a work item list (one request, or descriptors that have to stay small): count them
    int t = it, nt, req = 0;
    for (;;) {
      if (p.n_reqs > 1) rd = p.reqs[req];
      nt = (int)(((unsigned)rd.suffix_len * G + RT - 1) / RT);
      if (t < nt || req + 1 == p.n_reqs) break;
      t -= nt;
      req++;
    }
    tile = nt - 1 - t;                                         // longest context first
    const unsigned last = min((unsigned)rd.suffix_len * G, (unsigned)(tile + 1) * RT) - 1;
    sub_end = (rd.prefix_len + (int)(last / G) + 32) / 32;
  }
  const int P = rd.prefix_len, S = rd.suffix_len, ctx_len = P + S;
  const unsigned n_rows = (unsigned)S * G, row0 = (unsigned)tile * RT;

  // ---- rows of this lane: row 16 * qb + c of the tile
  int64_t qrow[NQB];                                           // row of q / out, in heads
  int posq[NQB];
  bool ok[NQB];
#pragma unroll
  for (int qb = 0; qb < NQB; qb++) {
    const unsigned rho = row0 + 16 * qb + c;
    ok[qb] = rho < n_rows;
    const unsigned rr = ok[qb] ? rho : n_rows - 1, tok = rr / G;
    posq[qb] = P + (int)tok;
    qrow[qb] = (int64_t)(rd.q_off + (int)tok) * Hq + kv * (int)G + (int)(rr - tok * G);
  }
  // first and last row of the tile
  const int pos_min = __builtin_amdgcn_readfirstlane(posq[0]), pos_max = __builtin_amdgcn_readlane(posq[NQB - 1], 15);

  // ---- addressing: block b of the request; 16-byte offsets inside it
  const unsigned char* pool = (const unsigned char*)p.pool_layer;
  const unsigned rs = (unsigned)(Hkv * D * E);                 // bytes between token rows
  const unsigned half = kBlockTokens * rs;
  const const_i32p table = (const_i32p)(uintptr_t)(p.tables + rd.table_off);
  const int p_blk = P / kBlockTokens, last_blk = (ctx_len + kBlockTokens - 1) / kBlockTokens - 1;
  const unsigned char* ks = (const unsigned char*)p.k_suffix;
  const unsigned char* vs = (const unsigned char*)p.v_suffix;
  const int64_t s_base = (int64_t)rd.q_off * rs;
  const bool from_suffix = ks != nullptr;
  const unsigned head_b = (unsigned)(kv * D * E);
  bool k_ok[KJ];                                               // operand chunk j of this lane lies inside the head
  unsigned q_off[KJ];
#pragma unroll
  for (int j = 0; j < KJ; j++) {
    const int d = F32 ? 16 * j + 4 * g : 32 * j + 8 * g;
    k_ok[j] = C::FULL || d < D;
    q_off[j] = (unsigned)((k_ok[j] ? d : 0) * E);
  }
  // A block's K or V half is a buffer of the token rows that the context has there: a base that a step computes on the scalar
  // unit, 32-bit offsets that stay.  What lies outside reads zeros, without an instruction that waits for the data: rows past
  // the end of the context (their scores are masked), K past the head (in place of Q's zeros there) and V past the head (output rows
  // that are not stored).
  auto buffer = [&](const unsigned char* base, int b) {
    const int rows = min(kBlockTokens, ctx_len - kBlockTokens * b);
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<unsigned char*>(base), 0, (unsigned)rows * rs, kBufferWord3);
  };
  auto k_at = [&](int j) {
    const unsigned at = head_b + c * rs + 16 * g;
    return k_ok[j] ? at + (F32 ? 16 * j : 32 * j) * E : kPastEnd;
  };
  auto v_at = [&](int r, int q) {
    const unsigned at = head_b + (4 * g + r) * rs + VW * E * c;
    return C::FULL || VW * (16 * q + c) < D ? at + VW * E * 16 * q : kPastEnd;
  };
  typedef typename std::conditional<(VW * E == 16), u32x4, u32x2>::type vreg;

  u32x4 kreg[KB][KJ];
  vreg vr[KB][4][VQ];
  int slot[KB];                                                // pool slots of the step that load_k takes next
  const unsigned char* vp[KB];                                 // V rows of the step that load_v takes next
  auto look_up = [&](int st) {
#pragma unroll
    for (int kb = 0; kb < KB; kb++) slot[kb] = table[min(st * KB + kb, last_blk)];
  };
  const unsigned char *v_pool = pool + half, *k_sfx = ks + s_base, *v_sfx = vs + s_base;
  const int sfx_blk = from_suffix ? p_blk : last_blk + 1;      // from this block on the caller's arrays
  auto load_k = [&](int st) {
#pragma unroll
    for (int kb = 0; kb < KB; kb++) {
      const int b = min(st * KB + kb, last_blk);
      const bool sfx = b >= sfx_blk;
      const uint64_t off = (uint64_t)(unsigned)(sfx ? b - p_blk : 2 * slot[kb]) * half;
      const auto buf = buffer((sfx ? k_sfx : pool) + off, b);
      vp[kb] = (sfx ? v_sfx : v_pool) + off;
#pragma unroll
      for (int j = 0; j < KJ; j++) kreg[kb][j] = __builtin_amdgcn_raw_buffer_load_b128(buf, k_at(j), 0, 0);
    }
  };
  auto load_v = [&](int st) {
#pragma unroll
    for (int kb = 0; kb < KB; kb++) {
      const auto buf = buffer(vp[kb], min(st * KB + kb, last_blk));
#pragma unroll
      for (int r = 0; r < 4; r++)
#pragma unroll
        for (int q = 0; q < VQ; q++) {
          if constexpr (VW * E == 16) vr[kb][r][q] = __builtin_amdgcn_raw_buffer_load_b128(buf, v_at(r, q), 0, 0);
          else vr[kb][r][q] = __builtin_amdgcn_raw_buffer_load_b64(buf, v_at(r, q), 0, 0);
        }
    }
  };

  // ---- this wave's steps: KB blocks each, alternating between the key waves
  constexpr int SPS = 2 / KB;                                  // steps per 32-key sub-tile
  const int st_begin = sub_begin * SPS + wave;
  int st = st_begin;
  const int st_end = min(sub_end * SPS, pos_max / (kBlockTokens * KB) + 1);
  u32x4 qreg[NQB][KJ];
  const f32x4 zero4 = {0.f, 0.f, 0.f, 0.f};
  f32x4 o[NQB][C::NACC];                                       // tile (q, e): d = VW * (16q + 4g + r) + e of query row c
#pragma unroll
  for (int qb = 0; qb < NQB; qb++)
#pragma unroll
    for (int a = 0; a < C::NACC; a++) o[qb][a] = zero4;
  // Softmax reference (exponent units), negated and 0 while no key has been seen; the score above which it moves, -inf until
  // then; row sum of this lane.
  float nref[NQB], bound[NQB], l[NQB];
#pragma unroll
  for (int qb = 0; qb < NQB; qb++) { nref[qb] = 0.f; bound[qb] = -INFINITY; l[qb] = 0.f; }
  const float c2 = p.scale * 1.4426950408889634f, inv_c2 = 1.f / c2;
  auto reference = [&](int qb) { return bound[qb] == -INFINITY ? -INFINITY : -nref[qb]; };
  // The score 16 above a reference.  Product and 1 / c2 are rounded: a 2^21st is taken off, so that no score above it stays below
  // the bound (at 2^30 exponent units its weight would not be finite), and a reference of finite scores keeps a finite bound.
  auto score_above = [&](float ref) {
    const float b = fminf((ref + 16.f) * inv_c2, FLT_MAX);
    return fmaxf(b - 0x1p-21f * __builtin_fabsf(b), -FLT_MAX);
  };

  // Weights of a row block as three bf16 terms: the upper half cut off, which leaves an exact rest, twice.  (Of a pair one
  // instruction packs them, two each clear and subtract; rounding the terms takes two more.)
  auto weights_bf16 = [&](const float (&w)[KB][4], bf16x8 (&pb)[3]) {
    u32x4 x[3];
#pragma unroll
    for (int i = 0; i < 4; i++) {
      float v[2] = {w[(KB - 1) & (i >> 1)][2 * (i & 1)], w[(KB - 1) & (i >> 1)][2 * (i & 1) + 1]};
#pragma unroll
      for (int t = 0; t < 3; t++) {
        const unsigned b0 = __builtin_bit_cast(unsigned, v[0]), b1 = __builtin_bit_cast(unsigned, v[1]);
        x[t][i] = __builtin_amdgcn_perm(b1, b0, 0x07060302u);
        v[0] -= as_float(b0 & 0xffff0000u);
        v[1] -= as_float(b1 & 0xffff0000u);
      }
    }
#pragma unroll
    for (int t = 0; t < 3; t++) pb[t] = __builtin_bit_cast(bf16x8, x[t]);
  };
  // V^T operand of tile (q, e): the lane's keys in k-slot order (kb, r)
  auto v_bf16 = [&](int q, int e) {
    u32x4 x;
#pragma unroll
    for (int i = 0; i < 4; i++)
      x[i] = __builtin_amdgcn_perm(vr[(KB - 1) & (i >> 1)][2 * (i & 1) + 1][q][e >> 1],
                                   vr[(KB - 1) & (i >> 1)][2 * (i & 1)][q][e >> 1], e & 1 ? 0x07060302u : 0x05040100u);
    return __builtin_bit_cast(bf16x8, x);
  };
  // Weights of row block qb, from its scores
  auto weigh = [&](const f32x4 (&s)[KB][NQB], int qb, float (&w)[KB][4]) {
    float sum = 0.f;
#pragma unroll
    for (int kb = 0; kb < KB; kb++)
#pragma unroll
      for (int r = 0; r < 4; r++) {
        w[kb][r] = __builtin_amdgcn_exp2f(__builtin_fmaf(s[kb][qb][r], c2, nref[qb]));
        sum += w[kb][r];
      }
    l[qb] += sum;
  };

  // One step.  DIAG: some row does not see all of its keys.  MORE: the wave has another step, which this one asks for.
  auto step = [&](auto diag_tag, auto more_tag) {
    constexpr bool DIAG = decltype(diag_tag)::value != 0, MORE = decltype(more_tag)::value != 0;
    const int k0 = st * (kBlockTokens * KB);
    f32x4 s[KB][NQB];
#pragma unroll
    for (int kb = 0; kb < KB; kb++)
#pragma unroll
      for (int qb = 0; qb < NQB; qb++) s[kb][qb] = zero4;
#pragma unroll
    for (int j = 0; j < KJ; j++) {
      if constexpr (F32) {
#pragma unroll
        for (int i = 0; i < 4; i++)
#pragma unroll
          for (int kb = 0; kb < KB; kb++)
#pragma unroll
            for (int qb = 0; qb < NQB; qb++)
              s[kb][qb] = __builtin_amdgcn_mfma_f32_16x16x4f32(as_float(kreg[kb][j][i]),
                                                               as_float(qreg[qb][j][i]), s[kb][qb], 0, 0, 0);
      } else {
#pragma unroll
        for (int kb = 0; kb < KB; kb++)
#pragma unroll
          for (int qb = 0; qb < NQB; qb++)
            s[kb][qb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, kreg[kb][j]),
                                                                __builtin_bit_cast(bf16x8, qreg[qb][j]), s[kb][qb], 0, 0, 0);
      }
    }
    if constexpr (MORE) {
      load_k(st + NW);
      look_up(st + 2 * NW);                                    // clamped to the last block
    }
    if constexpr (DIAG) {
#pragma unroll
      for (int kb = 0; kb < KB; kb++)
#pragma unroll
        for (int qb = 0; qb < NQB; qb++)
#pragma unroll
          for (int r = 0; r < 4; r++)
            if (k0 + 16 * kb + 4 * g + r > posq[qb]) s[kb][qb][r] = -INFINITY;
    }
    float mx[NQB];
    bool raise = false;
#pragma unroll
    for (int qb = 0; qb < NQB; qb++) {
      mx[qb] = -INFINITY;
#pragma unroll
      for (int kb = 0; kb < KB; kb++)
#pragma unroll
        for (int r = 0; r < 4; r++) mx[qb] = fmaxf(mx[qb], s[kb][qb][r]);
      raise |= mx[qb] > bound[qb];
    }
    if (__builtin_amdgcn_ballot_w64(raise) != 0) {
#pragma unroll
      for (int qb = 0; qb < NQB; qb++) {
        const float old = reference(qb), mn = fmaxf(old, quad_max(mx[qb]) * c2);
        nref[qb] = mn == -INFINITY ? 0.f : -mn;                // a row that has seen no key yet: all its weights are 0
        bound[qb] = mn == -INFINITY ? -INFINITY : score_above(mn);
        const float a = __builtin_amdgcn_exp2f(old + nref[qb]);
        l[qb] *= a;
#pragma unroll
        for (int i = 0; i < C::NACC; i++) o[qb][i] *= a;
      }
    }
    // Second product: o += V^T * w
    if constexpr (F32) {
      float w[NQB][KB][4];
#pragma unroll
      for (int qb = 0; qb < NQB; qb++) weigh(s, qb, w[qb]);
#pragma unroll
      for (int kb = 0; kb < KB; kb++)
#pragma unroll
        for (int r = 0; r < 4; r++)
#pragma unroll
          for (int q = 0; q < VQ; q++)
#pragma unroll
            for (int e = 0; e < VW; e++)
#pragma unroll
              for (int qb = 0; qb < NQB; qb++)
                o[qb][q * VW + e] = __builtin_amdgcn_mfma_f32_16x16x4f32(as_float(vr[kb][r][q][e]), w[qb][kb][r],
                                                                         o[qb][q * VW + e], 0, 0, 0);
      if constexpr (MORE) load_v(st + NW);
    } else if constexpr (C::V_FIRST) {
      // V into operand order, which frees its registers for the next step's, then one row block after the other
      bf16x8 a[C::NACC];
#pragma unroll
      for (int i = 0; i < C::NACC; i++) a[i] = v_bf16(i / VW, i % VW);
      if constexpr (MORE) {
        __builtin_amdgcn_sched_barrier(0);
        load_v(st + NW);
      }
#pragma unroll
      for (int qb = 0; qb < NQB; qb++) {
        float w[KB][4];
        bf16x8 pb[3];
        weigh(s, qb, w);
        weights_bf16(w, pb);
#pragma unroll
        for (int t = 0; t < 3; t++)
#pragma unroll
          for (int i = 0; i < C::NACC; i++) o[qb][i] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[i], pb[t], o[qb][i], 0, 0, 0);
      }
    } else {
      bf16x8 pb[NQB][3];
#pragma unroll
      for (int qb = 0; qb < NQB; qb++) {
        float w[KB][4];
        weigh(s, qb, w);
        weights_bf16(w, pb[qb]);
      }
#pragma unroll
      for (int q = 0; q < VQ; q++)
#pragma unroll
        for (int e0 = 0; e0 < VW; e0 += 4) {
          bf16x8 a[4];
#pragma unroll
          for (int e = 0; e < 4; e++) a[e] = v_bf16(q, e0 + e);
#pragma unroll
          for (int t = 0; t < 3; t++)
#pragma unroll
            for (int e = 0; e < 4; e++)
#pragma unroll
              for (int qb = 0; qb < NQB; qb++)
                o[qb][q * VW + e0 + e] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[e], pb[qb][t], o[qb][q * VW + e0 + e], 0, 0, 0);
          __builtin_amdgcn_sched_barrier(0);                   // one group's operands at a time in registers
        }
      if constexpr (MORE) load_v(st + NW);
    }
  };

  if (st < st_end) {
    // Requested Q, K, V, as in the loop, and Q waited for before it: a wait for K is then a wait for all but the V requests behind
    // it.  (Left to the scheduler, or with a test around the requests of a step, every step waited for the V it had just asked for.)
    look_up(st);
#pragma unroll
    for (int qb = 0; qb < NQB; qb++)
#pragma unroll
      for (int j = 0; j < KJ; j++) qreg[qb][j] = *(const u32x4*)((const unsigned char*)p.q + qrow[qb] * (D * E) + q_off[j]);
    __builtin_amdgcn_sched_barrier(0);
    load_k(st);
    look_up(st + NW);
    __builtin_amdgcn_sched_barrier(0);
    load_v(st);
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int qb = 0; qb < NQB; qb++)
#pragma unroll
      for (int j = 0; j < KJ; j++) {
        if (!C::FULL && !k_ok[j]) qreg[qb][j] = (u32x4){0u, 0u, 0u, 0u};
        asm volatile("" : "+v"(qreg[qb][j]));
      }
    // Two loops: the steps that every row sees in full spend nothing on masks.  The last step has nothing to ask for.
    const int st_last = st_end - NW, st_full = min(st_last, (pos_min + 1) / (kBlockTokens * KB));
    for (; st < st_full; st += NW) step(Tag<0>{}, Tag<1>{});
    for (; st < st_last; st += NW) step(Tag<1>{}, Tag<1>{});
    step(Tag<1>{}, Tag<0>{});
  }

  float m[NQB];
#pragma unroll
  for (int qb = 0; qb < NQB; qb++) m[qb] = reference(qb);

  // The same keys for the rows of one block, a key at a time: a row adds weight times V of the keys that it sees and
  // touches no other.  Weights are taken against the running maximum: sums stay within those of a textbook loop.
  // Rare, so it is written for few registers.
  auto walk_by_row = [&](auto qb_tag) {
    constexpr int qb = decltype(qb_tag)::value;
    const unsigned char* qp = (const unsigned char*)p.q + qrow[qb] * (D * E);
#pragma unroll
    for (int a = 0; a < C::NACC; a++) o[qb][a] = zero4;
    m[qb] = -INFINITY;
    l[qb] = 0.f;
#pragma unroll 1
    for (int s0 = st_begin; s0 < st_end; s0 += NW)
#pragma unroll 1
      for (int b = s0 * KB; b < (s0 + 1) * KB; b++) {
        const int k0 = kBlockTokens * b;
        if (k0 > pos_max) break;
        const bool sfx = from_suffix && b >= p_blk;
        const int64_t off = (sfx ? s_base + (int64_t)(b - p_blk) * half : (int64_t)table[b] * (2 * half)) + head_b;
        const unsigned char* kp = (sfx ? ks : pool) + off;
        const unsigned char* vb = sfx ? vs + off : kp + half;
        const int rest = min(kBlockTokens, ctx_len - k0);      // token rows the block holds
        kp += (int64_t)min(c, rest - 1) * rs;
        f32x4 s = zero4;
#pragma unroll 1
        for (int j = 0; j < KJ; j++) {
          const int d = F32 ? 16 * j + 4 * g : 32 * j + 8 * g;
          u32x4 kx = {0u, 0u, 0u, 0u}, qx = kx;
          if (C::FULL || d < D) {
            kx = *(const u32x4*)(kp + d * E);
            qx = *(const u32x4*)(qp + d * E);
          }
          if constexpr (F32) {
#pragma unroll
            for (int i = 0; i < 4; i++) s = __builtin_amdgcn_mfma_f32_16x16x4f32(as_float(kx[i]), as_float(qx[i]), s, 0, 0, 0);
          } else {
            s = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, kx), __builtin_bit_cast(bf16x8, qx), s, 0, 0, 0);
          }
        }
        float mx = -INFINITY, sum = 0.f, w[4];
#pragma unroll
        for (int r = 0; r < 4; r++) {
          if (k0 + 4 * g + r > posq[qb]) s[r] = -INFINITY;
          mx = fmaxf(mx, s[r]);
        }
        const float mn = fmaxf(m[qb], quad_max(mx) * c2), ref = mn == -INFINITY ? 0.f : mn;
        const float a = __builtin_amdgcn_exp2f(m[qb] - ref);
#pragma unroll
        for (int r = 0; r < 4; r++) {
          w[r] = __builtin_amdgcn_exp2f(__builtin_fmaf(s[r], c2, -ref));
          sum += w[r];
        }
        m[qb] = mn;
        l[qb] = l[qb] * a + sum;
#pragma unroll
        for (int i = 0; i < C::NACC; i++) o[qb][i] *= a;
#pragma unroll 1
        for (int key = 0; key < rest; key++) {
          const float w4 = key & 2 ? (key & 1 ? w[3] : w[2]) : (key & 1 ? w[1] : w[0]);
          const float wk = __shfl(w4, 16 * (key >> 2) + c);
          const bool sees = k0 + key <= posq[qb];
          const unsigned char* vrow = vb + (int64_t)key * rs;
#pragma unroll
          for (int q = 0; q < VQ; q++)
#pragma unroll
            for (int r = 0; r < 4; r++) {
              const int d = VW * (16 * q + 4 * g + r);
              if (!sees || !(C::FULL || d < D)) continue;
              const vreg x = *(const vreg*)(vrow + d * E);
#pragma unroll
              for (int e = 0; e < VW; e++) {
                float v;
                if constexpr (F32) v = as_float(x[e]);
                else v = e & 1 ? as_float(x[e >> 1] & 0xffff0000u) : bf16_widen(x[e >> 1] & 0xffffu);
                o[qb][q * VW + e][r] = __builtin_fmaf(wk, v, o[qb][q * VW + e][r]);
              }
            }
        }
      }
  };
  // With sums below 2^110 a wave's share leaves 18 powers of two for adding 8 waves and 64 pieces.
  float mag[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int qb = 0; qb < NQB; qb++)
#pragma unroll
    for (int a = 0; a < C::NACC; a++)
#pragma unroll
      for (int r = 0; r < 4; r++) mag[r] += __builtin_fabsf(o[qb][a][r]);
  if (__builtin_amdgcn_ballot_w64(!((mag[0] + mag[1]) + (mag[2] + mag[3]) < 0x1p110f)) != 0)
    static_for<0, NQB>(walk_by_row);

  // ---- suffix rows of the tokens whose first row lies in this tile: caller's arrays -> pool.  The first
  // chunk of every thread is on its way while the key waves are combined.
  const int cpr = D * E / 16;
  int n_copy = 0, t0 = 0;
  if (from_suffix && first_piece) {
    t0 = (int)((tile * RT + G - 1) / G);
    n_copy = ((int)((min((tile + 1) * RT, n_rows) + G - 1) / G) - t0) * cpr;
  }
  auto copy_at = [&](int i, int64_t& src, int64_t& dst) {
    const int tok = t0 + i / cpr, pos = P + tok;
    const unsigned in_row = head_b + 16 * (i % cpr);
    src = s_base + (int64_t)tok * rs + in_row;
    dst = (int64_t)p.tables[rd.table_off + pos / kBlockTokens] * (2 * half) + (int64_t)(pos % kBlockTokens) * rs + in_row;
  };
  unsigned char* wpool = (unsigned char*)p.pool_layer;
  u32x4 copy_k, copy_v;
  int64_t copy_dst = 0;
  if ((int)threadIdx.x < n_copy) {
    int64_t src;
    copy_at(threadIdx.x, src, copy_dst);
    copy_k = *(const u32x4*)(ks + src);
    copy_v = *(const u32x4*)(vs + src);
  }

  // ---- row sums over the four lanes of a row, then over the waves
  float* lds_o = (float*)smem + (size_t)wave * (C::UNITS * VW * 64) + lane;
  float* lds_ml = (float*)(smem + C::LDS_O);
#pragma unroll
  for (int qb = 0; qb < NQB; qb++)
    l[qb] = quad_sum(l[qb]);
#pragma unroll
  for (int qb = 0; qb < NQB; qb++)
    if (g == 0) *(f32x2*)(lds_ml + (wave * C::ROWS + 16 * qb + c) * 2) = (f32x2){m[qb], l[qb]};
  __syncthreads();
#pragma unroll
  for (int qb = 0; qb < NQB; qb++) {
    const f32x2* ml = (const f32x2*)lds_ml + 16 * qb + c;
    f32x2 x[NW];
    float all = -INFINITY, sum = 0.f;
#pragma unroll
    for (int k = 0; k < NW; k++) x[k] = ml[k * C::ROWS];
#pragma unroll
    for (int k = 0; k < NW; k++) all = fmaxf(all, x[k][0]);
    const float ref = all == -INFINITY ? 0.f : all;
    const float a = __builtin_amdgcn_exp2f(m[qb] - ref);
#pragma unroll
    for (int k = 0; k < NW; k++) sum += __builtin_amdgcn_exp2f(x[k][0] - ref) * x[k][1];
    m[qb] = all;
    l[qb] = sum;
#pragma unroll
    for (int q = 0; q < VQ; q++)
#pragma unroll
      for (int r = 0; r < 4; r++)
#pragma unroll
        for (int e = 0; e < VW; e++) lds_o[(((qb * VQ + q) * 4 + r) * VW + e) * 64] = o[qb][q * VW + e][r] * a;
  }
  __syncthreads();
  if ((int)threadIdx.x < n_copy) {
    *(u32x4*)(wpool + copy_dst) = copy_k;
    *(u32x4*)(wpool + copy_dst + half) = copy_v;
    for (int i = threadIdx.x + 64 * NW; i < n_copy; i += 64 * NW) {
      int64_t src, dst;
      copy_at(i, src, dst);
      *(u32x4*)(wpool + dst) = *(const u32x4*)(ks + src);
      *(u32x4*)(wpool + dst + half) = *(const u32x4*)(vs + src);
    }
  }
  const int64_t part = (int64_t)it * Hkv + kv;
  if (n_splits > 1 && wave == 0 && g == 0) {
#pragma unroll
    for (int qb = 0; qb < NQB; qb++) {
      float* pm = p.part_ml + (part * C::ROWS + 16 * qb + c) * 2;
      pm[0] = m[qb];
      pm[1] = l[qb];
    }
  }
#pragma unroll
  for (int qb = 0; qb < NQB; qb++)
#pragma unroll
    for (int q = 0; q < VQ; q++)
#pragma unroll
      for (int r = 0; r < 4; r++) {
        const int unit = (qb * VQ + q) * 4 + r;
        if (unit % NW != wave) continue;                       // the waves share the stores
        const float* src = (const float*)smem + unit * VW * 64 + lane;
        float v[NW][VW], x[VW];
#pragma unroll
        for (int k = 0; k < NW; k++)
#pragma unroll
          for (int e = 0; e < VW; e++) v[k][e] = src[(k * C::UNITS * VW + e) * 64];
#pragma unroll
        for (int e = 0; e < VW; e++) {
          x[e] = v[0][e];
#pragma unroll
          for (int k = 1; k < NW; k++) x[e] += v[k][e];
        }
        const int d = VW * (16 * q + 4 * g + r);
        if (n_splits > 1) {
          float* po = p.part_o + (part * C::ROWS + 16 * qb + c) * DP + d;
#pragma unroll
          for (int e = 0; e < VW; e += 4) *(f32x4*)(po + e) = (f32x4){x[e], x[e + 1], x[e + 2], x[e + 3]};
        } else if (ok[qb] && (C::FULL || d < D)) {
          const float inv = 1.f / l[qb];
          T* po = (T*)p.out + qrow[qb] * D + d;
          if constexpr (F32) {
            *(f32x4*)po = (f32x4){x[0] * inv, x[1] * inv, x[2] * inv, x[3] * inv};
          } else {
            vreg v;
#pragma unroll
            for (int e = 0; e < VW; e += 2) v[e / 2] = bf16_rne(x[e] * inv) | bf16_rne(x[e + 1] * inv) << 16;
            *(vreg*)po = v;
          }
        }
      }
  if (threadIdx.x == 0) clock_end(p.clock.words);
}

// Combines the pieces of cut tiles as merge_splits_kernel does, for this file's layout: one wave per row.
// us a call of one caller, 8 loads behind the weights / in front of them, 16 at D = 64: fp32 1024+128, 8Q/2KV, D = 64 15.8 / 14.4,
// bf16 8192+20, 16Q/4KV, D = 64 16.9 / 12.8; wider heads, where loads past the last piece are left out: fp32 8192+4, 8Q/2KV, D = 128 28.1 / 19.5,
// bf16 8192+4, 8Q/2KV, D = 256 22.6 / 15.8 (four in front 21.1), fp32 3040+1, 16Q/4KV, D = 256 22.0 / 16.4 (20.8).
// A row that saw no key in a piece has m = -inf, l = 0, O = 0 there and adds nothing.
template <typename T, int DP, int ROWS>
__global__ void __launch_bounds__(256) merge_rows_kernel(RowsParams p, const int32_t* split_tiles) {
  constexpr int W = DP / 64;                                   // consecutive floats of a lane
  typedef typename std::conditional<W == 4, f32x4, typename std::conditional<W == 2, f32x2, float>::type>::type vec;
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int Hkv = p.n_kv_heads, Hq = p.n_q_heads, D = p.head_dim;
  const unsigned G = p.group;
  const int row = (blockIdx.x % (ROWS / 4)) * 4 + wave;
  const int slot_id = blockIdx.x / (ROWS / 4), kv = slot_id % Hkv, first = ((const_i32p)(uintptr_t)split_tiles)[slot_id / Hkv];
  const WorkItem wi = load_item(p.items, first);
  const unsigned rho = (unsigned)wi.q_tile * ROWS + row;
  if (rho >= (unsigned)wi.suffix_len * G) return;
  const int n = wi.n_splits;
  const int64_t base = ((int64_t)first * Hkv + kv) * ROWS + row;
  const int64_t step = (int64_t)Hkv * ROWS;
  const f32x2* ml = (const f32x2*)p.part_ml + base;
  const float* po = p.part_o + base * DP + W * lane;
  // at most 64 pieces per tile (attn_plan.cpp): lane i holds piece i
  const f32x2 mine = lane < n ? ml[lane * step] : (f32x2){-INFINITY, 0.f};
  constexpr int B = W > 2 ? 8 : 16 / W;                        // loads in flight: the first are on their way while the weights are found
  vec v[B];
  // Past the end nothing, or (4 bytes a lane) the last piece again, which costs no more than the branch
  auto fetch = [&](int c0) {
#pragma unroll
    for (int i = 0; i < B; i++)
      if (W == 1 || c0 + i < n) v[i] = *(const vec*)(po + min(c0 + i, n - 1) * step * DP);
  };
  fetch(0);
  __builtin_amdgcn_sched_barrier(0);
  float all = mine[0];
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) all = fmaxf(all, __shfl_xor(all, o));
  const float wgt = mine[0] == -INFINITY ? 0.f : __builtin_amdgcn_exp2f(mine[0] - all);
  float l = wgt * mine[1];
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) l += __shfl_xor(l, o);
  float acc[W];
#pragma unroll
  for (int e = 0; e < W; e++) acc[e] = 0.f;
  for (int c0 = 0; c0 < n; c0 += B) {
    if (c0) fetch(c0);
#pragma unroll
    for (int i = 0; i < B; i++) {
      if (c0 + i >= n) break;
      const float w = __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, wgt), c0 + i));
#pragma unroll
      for (int e = 0; e < W; e++) {
        float x;
        if constexpr (W == 1) x = v[i];
        else x = v[i][e];
        acc[e] = __builtin_fmaf(w, x, acc[e]);
      }
    }
  }
  if (threadIdx.x == 0) clock_end_tail(p.clock.words);
  const int d = W * lane;
  if (d >= D) return;
  const float inv = 1.f / l;
  const unsigned tok = rho / G;
  T* out = (T*)p.out + ((int64_t)(wi.q_off + (int)tok) * Hq + kv * (int)G + (int)(rho - tok * G)) * D + d;
#pragma unroll
  for (int e = 0; e < W; e++) {
    if constexpr (sizeof(T) == 4) out[e] = acc[e] * inv;
    else out[e] = (T)bf16_rne(acc[e] * inv);
  }
}

template <class C>
hipError_t launch(const RowsParams& p, unsigned grid, const int32_t* split_tiles, int n_split_tiles, hipStream_t stream) {
  hipLaunchKernelGGL(attn_rows_kernel<C>, dim3(grid), dim3(64 * C::NW), C::LDS_BYTES, stream, p);
  if (n_split_tiles > 0) {
    const unsigned slots = (unsigned)n_split_tiles * (unsigned)p.n_kv_heads;
    hipLaunchKernelGGL((merge_rows_kernel<typename C::T, C::DP, C::ROWS>), dim3(slots * (C::ROWS / 4)), dim3(256), 0, stream, p,
                       split_tiles);
  }
  return hipGetLastError();
}

// f(configuration) for an element type, head width and tiling (attn_rows_shape)
template <typename F>
auto with_cfg(int dtype, int head_dim, int tile_rows, F&& f) {
  typedef uint16_t B16;
  if (dtype == CALVO_F32) {
    if (head_dim == 64) return f(RowsCfg<float, 64, 2, 2, 8, true>{});
    if (head_dim < 64) return f(RowsCfg<float, 64, 2, 2, 8, false>{});
    if (head_dim == 128) return f(RowsCfg<float, 128, 2, 1, 4, true>{});
    if (head_dim < 128) return f(RowsCfg<float, 128, 2, 1, 4, false>{});
    if (head_dim == 256) return tile_rows == 32 ? f(RowsCfg<float, 256, 2, 1, 4, true>{}) : f(RowsCfg<float, 256, 1, 1, 4, true>{});
    return tile_rows == 32 ? f(RowsCfg<float, 256, 2, 1, 4, false>{}) : f(RowsCfg<float, 256, 1, 1, 4, false>{});
  }
  if (head_dim == 64) return tile_rows == 64 ? f(RowsCfg<B16, 64, 4, 2, 8, true>{}) : f(RowsCfg<B16, 64, 2, 2, 8, true>{});
  if (head_dim < 64) return tile_rows == 64 ? f(RowsCfg<B16, 64, 4, 2, 8, false>{}) : f(RowsCfg<B16, 64, 2, 2, 8, false>{});
  if (head_dim <= 128)                                          // 128 itself: attn_pipeline.h
    return tile_rows == 64 ? f(RowsCfg<B16, 128, 4, 2, 4, false>{}) : f(RowsCfg<B16, 128, 2, 2, 8, false>{});
  if (head_dim == 256) return tile_rows == 32 ? f(RowsCfg<B16, 256, 2, 2, 4, true>{}) : f(RowsCfg<B16, 256, 1, 2, 4, true>{});
  return tile_rows == 32 ? f(RowsCfg<B16, 256, 2, 2, 4, false>{}) : f(RowsCfg<B16, 256, 1, 2, 4, false>{});
}

}  // namespace rows

hipError_t attn_rows_prepare(int dtype, int head_dim, int tile_rows) {
  return rows::with_cfg(dtype, head_dim, tile_rows, [](auto cfg) {
    typedef decltype(cfg) C;
    return hipFuncSetAttribute((const void*)rows::attn_rows_kernel<C>, hipFuncAttributeMaxDynamicSharedMemorySize, C::LDS_BYTES);
  });
}

hipError_t launch_attn_rows(const RowsParams& p, int dtype, int tile_rows, int n_items, const int32_t* split_tiles, int n_split_tiles,
                            hipStream_t stream) {
  if (n_items <= 0) return hipSuccess;
  const unsigned grid = (unsigned)n_items * (unsigned)p.n_kv_heads;
  return rows::with_cfg(dtype, p.head_dim, tile_rows, [&](auto cfg) {
    return rows::launch<decltype(cfg)>(p, grid, split_tiles, n_split_tiles, stream);
  });
}

}  // namespace calvo

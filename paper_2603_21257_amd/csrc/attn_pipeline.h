// Paged causal GQA prefill attention for gfx950 (CDNA4), software-pipelined kernel body: bf16 storage, head_dim 128,
// v_mfma_f32_16x16x32_bf16 for both contractions, fp32 online softmax.  Two shapes of it (PipeCfg):
//   HB = 2: a wave owns 64 query rows and has a SIMD to itself (512 registers), one workgroup per CU (attn_pipe.hip)
//   HB = 1: 32 query rows per wave, two workgroups per CU: tiles half as large, for short suffixes (attn_duo.hip)
//
// Why the 16x16x32 shape: the part is power limited under matrix load, and on normally
// distributed operands this shape sustains 12 % more flop/s than 32x32x16 at the power limit
// (2010-2040 against 1800-1820 TFLOP/s with nothing but MFMAs on every SIMD: half the accumulator
// traffic per product).  It costs issue slots (twice the instructions; on all-zero data, where
// nothing limits the clock, the kernel is slower), and wins on real data.
//
// Transposed formulation (every softmax statistic stays in a lane's own registers):
//   S^T[key][query] = K[key][:] . Q[query][:]       A = K rows from LDS, B = Q in registers
//   O^T[d][query]  += V^T[d][key] * P^T[key][query]  A = V^T, B = P^T
// A wave owns QB blocks of 16 queries (qb); a 32-key sub-tile is two blocks of 16 keys (kb).
// Lane (c = lane % 16, g = lane / 16) of a 16x16 accumulator tile (kb, qb) holds query 16qb + c and
// the keys 16kb + 4g + r, r = 0..3: a lane works on QB query columns with 8 keys each, the four
// lanes c, c+16, c+32, c+48 share a query (row max and row sum cross them only in the rare slow
// path and at the end), the O rescale is one scalar per lane and query block, and the weights of a
// lane are exactly the eight k-slots 8g..8g+7 of the B operand of the second MFMA when the k-slot
// order is taken as (kb, r): slot 8g + 4kb + r <-> key 16kb + 4g + r.  V stays token-major in LDS
// (as in the pool); the d-major A operand in that key order comes from two LDS transpose reads
// (ds_read_b64_tr_b16: keys 4g..4g+3 and 16+4g..16+4g+3 for d = 16db + c).
//
// Schedule.  The key loop advances in 32-key sub-tiles.  Steady step t:
//     QK(t+1):  S_t+1 = K_t+1 Q^T                               8 QB MFMA
//     SM(t):    P_t = 2^(c (S_t - m)), row sums                 vector ALU, in between
//     PV(t-1):  O^T += V_t-1^T P_t-1^T                          8 QB MFMA
// S and P are double-buffered; each of the 16 A operands of a step (8 of K: 16 keys x 32 d, 8 of V^T: 16 d x 32 keys) is read
// from LDS PD operands ahead and feeds QB MFMAs.  The loop is unrolled by the ring depth so that ring slots are immediates.
// Measured for one wave alone on its SIMD: an MFMA of this shape holds the matrix pipe for 16 cycles and the wave's vector
// instructions back for 8, anything else for 4; a vector instruction takes 4 cycles, an exponential 8.  So behind every
// MFMA goes at most one instruction of another kind (LDS read, request, wait), which is free, and then two vector
// instructions or one exponential, which fill the 16 cycles.  A step of HB = 2 (64 MFMAs, 32 exponentials, 83 other vector
// instructions, 24 LDS reads) takes 1220 cycles that way, 1320 with the same instructions in the order of the dependences;
// 1380 in the kernel, with the requests and the barrier.
// The query blocks of an operand are walked there and back: from one MFMA to the next either A or B stays the same.
// At the power limit operands that change cost clock: MFMAs alone on N(0,1) data sustain 1915 TFLOP/s where both change every
// time, 1975 where A is held for four and then both change, 2025 there and back.  In the kernel it is worth no more than what runs differ
// by (three in turn, with one order / there and back: 61440+4096 tokens 3084 / 3073 us a call, 16384+2048 424.7 / 423.8, 38304+209
// (40Q/8KV) 162.7 / 162.4; one caller 2943 / 2926, 432 / 429, 159 / 159) and costs nothing; the same bits, each sum keeps its order.
// The step is written in this order, with scheduling barriers in between.  MFMAs are inline assembly so that their results
// stay in place, O of HB = 2 in accumulation registers: left to the compiler, every value that vector instructions
// touch as well is moved back and forth (45 to 250 moves a step).  What the compiler then does not know are the wait states
// between an MFMA and vector instructions around it; in a step the operands are at least eight MFMAs apart, elsewhere
// mfma_settle() is in between.  A spilled register would break that: the kernels must compile without any
// (tests/test_attn_registers.py).
//
// Why 64 rows per wave: under matrix load the part is at its power limit, and what a step costs beyond its MFMAs is K and
// V: 16 KB a step from L2 into LDS, and out of LDS once per wave.  With 64 rows every operand read feeds four MFMAs, half the
// LDS reads per product of 32 rows.  61440+4096 tokens, 32Q/8KV, against the kernel before (32 rows per wave, the two waves
// of a SIMD taking turns on the matrix pipe and the vector ALU): 3170 -> 2960 us on N(0,1) data, 2605 -> 2370 on zeros
// (where no power limit hides the schedule); without the requests (wrong results, timing only) 2720 and 2200, so what is
// left there is the movement of K and V itself.  The schedule alone, at 32 rows per wave and two workgroups per CU, against
// SM(t) followed by its MFMAs: 28096+28 tokens 34.3 -> 31.0 us a call, three short queries over 28K-38K tokens
// 202 -> 187, 512+1 15.3 -> 13.2, 0+1024 29.1 -> 25.3.
// v_mfma_f32_32x32x16_bf16 was measured in the schedule of HB = 2: 2304 us on zeros, 3292 on N(0,1) data (against 2632 and
// 3080 of this shape at that point): fewer issue slots, more power.
//
// Softmax with a lazily raised reference.  A weight is 2^(c s - c m) with c = scale * log2(e); the row
// sum adds the fp32 weights with v_add_f32, the PV product takes them rounded to bf16 (nearest even,
// unbiased; a row's result moves by at most 2^-9 relative, the size of the output's own rounding).
// The row sum must not use v_dot2_f32_bf16: measured on MI355X, a dot-product instruction waits for
// the matrix pipe (16 of them take 616 cycles beside another wave's MFMA stream against 104 alone),
// whereas v_exp_f32, v_fma_f32, v_add_f32 and v_cvt_pk_bf16_f32 issue in the shadow of MFMAs.
// m is not the running maximum: it lies 16 (kRefShift) above the maximum of some earlier sub-tile.  The weights of a sub-tile
// are computed against the current m, and only if a lane's partial row sum passes 1 (kLazyBound), i.e. a score is
// about 16 powers of two above that maximum, is the sub-tile's own taken, m raised, l and O rescaled and the weights computed
// again.  So no weight is above 1, as in the textbook recurrence: a sum w V leaves the range of fp32 only where that one's
// does.  The largest weight of a row is at least 2^-16: scores down to 2^-110 of the largest count, and with fp32
// accumulation and bf16 weights (relative precision) the result is the textbook one's up to rounding; the products keep
// subnormal sums (measured: the error is the same down to |V| of 2^-120).
//
// Data movement.  K and V go from the pool straight into LDS with global_load_lds_dwordx4 (no register staging), 1 KiB
// (4 token rows x 256 B) per wave instruction, into two rings (K and V) of RING 8 KiB slots.  Step t requests K(t+KA) and
// V(t+VA), reads K(t+1), V(t-1) and the first operands of K(t+2).  A ring of eight has one barrier for two steps; HB = 1 has
// a ring of five, the most that two workgroups leave each other of a CU's LDS, and one for each.
// Rows are unpadded; 16-byte chunks are XOR-swizzled on the way in (the lane that owns LDS chunk
// position c fetches logical chunk c ^ f(row)) so that operand reads are bank-conflict free:
// K f = row & 15 (a 16-lane group reads one chunk of 16 different rows), V f = (row & 7) << 1 (half
// a wave reads two chunks of 8 different rows).  Operand addresses are lane constants plus immediates.
// Cache policy bits on the requests (nt, sc0, sc1) do nothing or harm (nt: +5 %).
//
// Sub-tiles that touch the causal diagonal or the end of the context are not pipelined: they are at most a handful per
// workgroup, are requested before the drain of the pipeline and run QK -> mask -> SM -> PV.
#pragma once
#include "attn_common.h"

namespace calvo {
namespace attn {

template <int NW_, int RING_, int HB_, bool SFX_ = false>
struct PipeCfg {
  // The suffix rows come from the caller's arrays in the pipelined sub-tiles too, not only in those on the diagonal
  static constexpr bool SFX = SFX_;
  static constexpr int NW = NW_;                       // waves per workgroup
  static constexpr int HB = HB_;                       // blocks of 32 query rows per wave
  static constexpr int QB = 2 * HB_;                   // blocks of 16
  static constexpr int RING = RING_;                   // LDS ring slots per operand
  static constexpr bool BAR2 = RING_ == 8;             // one barrier for two steps, else one for each
  static constexpr int KA = BAR2 ? RING_ - 1 : RING_;  // step t requests K(t + KA) ...
  static constexpr int VA = KA - 2;                    // ... and V(t + VA)
  static constexpr int NI = 8 / NW_;                   // 1 KiB requests per wave, operand and sub-tile
  static constexpr int UNROLL = RING_ % 2 ? 2 * RING_ : RING_;
  static constexpr int PD = 4;         // LDS operand reads run this many operands ahead
  static constexpr int LDS_BYTES = 2 * RING_ * kSlot;
};

// m0 = lds_base + off for the dma_1k_m0 that follows at least one instruction later
template <int OFF>
__device__ inline void set_m0(unsigned lds_base, Tag<OFF>) {
  asm volatile("s_add_u32 m0, %0, %1" : : "s"(lds_base), "n"(OFF) : "scc");
}
__device__ inline void set_m0(unsigned lds_base, int off) {
  asm volatile("s_add_u32 m0, %0, %1" : : "s"(lds_base), "s"(off) : "scc");
}
// 64 lanes x 16 bytes from sbase + voff to 1 KiB of LDS at m0
__device__ inline void dma_1k_m0(const unsigned char* sbase, unsigned voff) {
  asm volatile("global_load_lds_dwordx4 %0, %1" : : "v"(voff), "s"(sbase));
}
// byte offset of a ring slot, for slots known at compile time and for others
template <int S, int ADD>
__device__ inline constexpr Tag<S * kSlot + ADD> slot_off(Tag<S>, Tag<ADD>) { return {}; }
template <int ADD>
__device__ inline int slot_off(int s, Tag<ADD>) { return s * kSlot + ADD; }
template <int V>
__device__ inline void opaque(Tag<V>&) {}
__device__ inline void opaque(int& s) { asm volatile("" : "+s"(s)); }
template <int V>
__device__ inline constexpr int value_of(Tag<V>) { return V; }
__device__ inline int value_of(int v) { return v; }

// o += a * b.  ACC: o in accumulation registers (where the wave has the SIMD's 512 registers, of which vector
// instructions reach 256), else in architectural ones.
template <bool ACC>
__device__ inline void mfma_acc(f32x4& o, const bf16x8& a, const bf16x8& b) {
  if constexpr (ACC) asm volatile("v_mfma_f32_16x16x32_bf16 %0, %1, %2, %0" : "+a"(o) : "v"(a), "v"(b));
  else asm volatile("v_mfma_f32_16x16x32_bf16 %0, %1, %2, %0" : "+v"(o) : "v"(a), "v"(b));
}
template <bool ACC>
__device__ inline void pin_acc(f32x4& o) {
  if constexpr (ACC) asm volatile("" : "+a"(o));
  else asm volatile("" : "+v"(o));
}
// s = a * b (+ s), in architectural registers
__device__ inline void mfma_first(f32x4& s, const bf16x8& a, const bf16x8& b) {
  asm volatile("v_mfma_f32_16x16x32_bf16 %0, %1, %2, 0" : "=&v"(s) : "v"(a), "v"(b));
}
__device__ inline void mfma_next(f32x4& s, const bf16x8& a, const bf16x8& b) {
  asm volatile("v_mfma_f32_16x16x32_bf16 %0, %1, %2, %0" : "+v"(s) : "v"(a), "v"(b));
}
// The compiler knows nothing of the waits that these need where vector instructions write an operand or touch a result
// before or after them.  A value pinned on both sides of this keeps its vector instructions out of the way on either.
__device__ inline void mfma_settle() { asm volatile("s_nop 15"); }
template <bool ACC, int QB>
__device__ inline void pin_all(f32x4 (&o)[8][QB]) {
#pragma unroll
  for (int db = 0; db < 8; db++)
#pragma unroll
    for (int qb = 0; qb < QB; qb++) pin_acc<ACC>(o[db][qb]);
}
template <bool ACC, int QB>
__device__ inline void acc_ready(f32x4 (&o)[8][QB]) {
  pin_all<ACC>(o);
  mfma_settle();
  pin_all<ACC>(o);
}

// largest of the numbers (a NaN counts as nothing)
__device__ inline float max_of(const float (&v)[4]) {
  float m;
  asm("v_max3_f32 %0, %1, %2, %3\n\tv_max_f32 %0, %0, %4" : "=&v"(m) : "v"(v[0]), "v"(v[1]), "v"(v[2]), "v"(v[3]));
  return m;
}
__device__ inline float max_of(const float (&v)[2]) {
  float m;
  asm("v_max_f32 %0, %1, %2" : "=v"(m) : "v"(v[0]), "v"(v[1]));
  return m;
}

template <class Cfg_>
__device__ __forceinline__ void attn_pipeline(const AttnParams& p, unsigned char* smem) {
  constexpr int NW = Cfg_::NW, HB = Cfg_::HB, QB = Cfg_::QB, RING = Cfg_::RING, KA = Cfg_::KA, VA = Cfg_::VA, NI = Cfg_::NI, PD = Cfg_::PD;
  constexpr bool ACC = HB == 2;
  constexpr int kVBase = RING * kSlot;                 // V ring follows the K ring
  const lds_u8* lds = (const lds_u8*)smem;
  const unsigned lds0 = (unsigned)(size_t)lds;
  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int c = lane & 15;
  const int g = lane >> 4;

  // ---- work item decode (wave-uniform)
  const int HW = p.heads_per_wg;
  const int TPW = HB * NW / HW;                        // 32-token blocks of the tile
  const int NHG = p.n_q_heads / HW;
  int it, hg;
  {
    const int bid = blockIdx.x;
    if ((NHG & 7) == 0) {
      const int per = NHG >> 3, rest = bid >> 3;
      hg = (bid & 7) * per + rest % per;
      it = rest / per;
    } else {
      hg = bid % NHG;
      it = bid / NHG;
    }
  }
  if (p.item_index) it = p.item_index[it];
  const WorkItem wi = p.items[it];
  const ReqDesc rd = p.reqs[wi.req];
  const int P = rd.prefix_len, S = rd.suffix_len;
  const int TQ = 32 * TPW;
  const int q_base = wi.q_tile * TQ;
  const int Hkv = p.n_kv_heads, Hq = p.n_q_heads;
  const int kv = hg * HW / (Hq / Hkv);
  // A wave owns HB of the tile's row blocks of 32, one from either end: block vw is (head vw % HW, token block vw / HW).
  // Blocks with later tokens see more of the diagonal, so the waves have about the same number of sub-tiles there.
  int hq[HB], wq0[HB];
  auto row_block = [&](int h) { return h ? HB * NW - 1 - wave : wave; };
#pragma unroll
  for (int h = 0; h < HB; h++) {
    const int vw = row_block(h);
    hq[h] = hg * HW + vw % HW;
    wq0[h] = q_base + (vw / HW) * 32;
  }
  const int ctx_len = P + S;
  const int jb = wi.sub_begin;
  const int n_sub = wi.sub_end - jb;
  const int n_pipe = max(0, min(wi.sub_end, (P + q_base + 1) / kSK) - jb);
  const int last_blk = (ctx_len + kBlockTokens - 1) / kBlockTokens - 1;
  typedef const __attribute__((address_space(4))) int64_t* const_i64p;
  const int n_blk_pad = last_blk + 1 + kTablePad + ((last_blk + 1) & 1);
  const int wblk = wave / (NW / 2);
  const const_i64p boffs = (const_i64p)(uintptr_t)(p.blk_offs + rd.table_off + wblk * (n_blk_pad >> 1));
  const float c2 = p.scale * 1.4426950408889634f;

  // ---- pool -> LDS
  const unsigned char* pool = (const unsigned char*)p.pool_layer;
  const unsigned row_b = (unsigned)(Hkv * kD * 2);
  const unsigned half_b = kBlockTokens * row_b;
  const int brow0 = (32 / NW) * (wave % (NW / 2)) + (lane >> 4);
  unsigned voff_k[NI], voff_v[NI];
#pragma unroll
  for (int h = 0; h < NI; h++) {
    const int row = brow0 + 4 * h;
    voff_k[h] = row * row_b + kv * kRow + (((lane & 15) ^ (row & 15)) << 4);
    voff_v[h] = half_b + row * row_b + kv * kRow + (((lane & 15) ^ ((row & 7) << 1)) << 4);
  }
  const unsigned dma_lds = lds0 + wave * (1024 * NI);

  auto fetch_off = [&](int j) -> int64_t { return boffs[jb + j]; };
  // Where the launch takes the suffix along, its rows are read from the caller's arrays: a 16-key block lies wholly in the
  // prefix or wholly in the suffix.  The first tile of a suffix meets such blocks on its diagonal only, later ones (SFX) in
  // the pipelined part as well.  There the turns within the prefix come first, those that choose an address after them: 4096+700
  // tokens 55.0 us a call, with the choice in every turn 58.5; 448+400 13.8, with run-time ring slots outside the prefix 15.6.
  constexpr bool SFX = Cfg_::SFX;
  typedef const __attribute__((address_space(4))) AttnParams* const_paramsp;
  const int p_blk = P / kBlockTokens;
  const int n_pool = SFX ? max(0, min(n_pipe, p_blk / 2 - jb)) : n_pipe;     // pipelined sub-tiles that lie in the prefix
  // Addresses of the request's suffix block 0 in the caller's arrays, as bases for voff_k and voff_v
  struct SuffixBases {
    const unsigned char *k, *v;
  };
  auto suffix_bases = [&](const void* k, const void* v) -> SuffixBases {
    const int64_t off = (int64_t)rd.q_off * row_b;
    return {(const unsigned char*)k + off, (const unsigned char*)v + off - half_b};
  };
  // K (V) of pipelined sub-tile j, at offset off of the pool: base for voff_k (voff_v)
  auto kv_base = [&](int j, int64_t off, const unsigned char* sfx) -> const unsigned char* {
    if constexpr (SFX) {
      const int sfx_blk = 2 * (jb + j) + wblk - p_blk;
      const bool in_sfx = sfx_blk >= 0;
      return (in_sfx ? sfx : pool) + (in_sfx ? (int64_t)sfx_blk * half_b : off);
    }
    return pool + off;
  };
  // request I of a step: the NI of a K sub-tile, then the NI of a V sub-tile, into their ring slots
  auto request_m0 = [&](auto kslot, auto vslot, auto idx) {
    constexpr int I = decltype(idx)::value;
    if constexpr (I < NI) set_m0(dma_lds, slot_off(kslot, Tag<I * 1024>{}));
    else set_m0(dma_lds, slot_off(vslot, Tag<kVBase + (I - NI) * 1024>{}));
  };
  auto request_one = [&](const unsigned char* kbase, const unsigned char* vbase, auto idx) {
    constexpr int I = decltype(idx)::value;
    if constexpr (I < NI) dma_1k_m0(kbase, voff_k[I]);
    else dma_1k_m0(vbase, voff_v[I - NI]);
  };

  // ---- Q as the B operand of QK^T
  bf16x8 qB[QB][4];
  {
    const unsigned short* q = (const unsigned short*)p.q;
#pragma unroll
    for (int qb = 0; qb < QB; qb++) {
      const int tokq = wq0[qb >> 1] + 16 * (qb & 1) + c;
      const bool ok = tokq < S;
      const unsigned short* row = q + ((int64_t)(rd.q_off + (ok ? tokq : 0)) * Hq + hq[qb >> 1]) * kD + 8 * g;
#pragma unroll
      for (int ks = 0; ks < 4; ks++) {
        u32x4 v = {0u, 0u, 0u, 0u};
        if (ok) v = *(const u32x4*)(row + 32 * ks);
        qB[qb][ks] = __builtin_bit_cast(bf16x8, v);
      }
    }
  }

  const f32x4 zero4 = {0.f, 0.f, 0.f, 0.f};
  f32x4 o[8][QB];
  float m_run[QB], l_run[QB];
#pragma unroll
  for (int qb = 0; qb < QB; qb++) { m_run[qb] = -INFINITY; l_run[qb] = 0.f; }

  // ---- lane-constant operand addresses inside a slot
  const lds_u8* ka_addr[4];
#pragma unroll
  for (int ks = 0; ks < 4; ks++) ka_addr[ks] = lds + c * kRow + (((4 * ks + g) ^ c) << 4);
  const int v_row = 4 * g + (c >> 2);
  const lds_u8* va_addr[8];
#pragma unroll
  for (int db = 0; db < 8; db++)
    va_addr[db] = lds + kVBase + v_row * kRow + ((2 * (db ^ (v_row & 7)) + ((c & 3) >> 1)) << 4) + (c & 1) * 8;

  f32x4 sb[2][2][QB];                                  // [parity][kb][qb]
  bf16x8 pb[2][QB];

  auto expo = [&](float s, int qb) -> float { return __builtin_fmaf(s, c2, -m_run[qb]); };
  auto row_max = [&](const f32x4& a, const f32x4& b) -> float {
    float mx = fmaxf(fmaxf(a[0], a[1]), fmaxf(a[2], a[3]));
    mx = fmaxf(mx, fmaxf(fmaxf(b[0], b[1]), fmaxf(b[2], b[3])));
    return quad_max(mx);
  };
  auto weights_of = [&](const f32x4& s0, const f32x4& s1, int qb, float& ps, bf16x8& pw) {
    float w[8];
#pragma unroll
    for (int e = 0; e < 8; e++) w[e] = __builtin_amdgcn_exp2f(expo(e < 4 ? s0[e & 3] : s1[e & 3], qb));
    ps = ((w[0] + w[1]) + (w[2] + w[3])) + ((w[4] + w[5]) + (w[6] + w[7]));
    pw = __builtin_bit_cast(bf16x8, (u32x4){pack_bf16(w[0], w[1]), pack_bf16(w[2], w[3]), pack_bf16(w[4], w[5]), pack_bf16(w[6], w[7])});
  };
  // Softmax of query blocks QB0 .. QB0 + N - 1 of one sub-tile (scores possibly masked with -inf): weights against the
  // current reference, unless a partial row sum passes the bound (or is not a number, or there is no reference yet).
  auto softmax = [&](auto qb0, auto&& s, bf16x8* pw) {
    constexpr int QB0 = decltype(qb0)::value, N = sizeof(s[0]) / sizeof(f32x4);
    float ps[N];
    bool above = false;
#pragma unroll
    for (int q = 0; q < N; q++) {
      weights_of(s[0][q], s[1][q], QB0 + q, ps[q], pw[q]);
      above |= !(ps[q] <= kLazyBound);
    }
    if (__builtin_amdgcn_ballot_w64(above) != 0) {
      float alpha[N];
      bool changed = false;
#pragma unroll
      for (int q = 0; q < N; q++) {
        const int qb = QB0 + q;
        const float m_new = fmaxf(m_run[qb], __builtin_fmaf(row_max(s[0][q], s[1][q]), c2, kRefShift));
        alpha[q] = __builtin_amdgcn_exp2f(m_run[qb] - m_new);
        changed |= m_run[qb] != -INFINITY && !(alpha[q] == 1.f);         // without a reference O is 0
        m_run[qb] = m_new;
        l_run[qb] = l_run[qb] * alpha[q];
        weights_of(s[0][q], s[1][q], qb, ps[q], pw[q]);
      }
      if (__builtin_amdgcn_ballot_w64(changed) != 0) {
        acc_ready<ACC>(o);
#pragma unroll
        for (int db = 0; db < 8; db++)
#pragma unroll
          for (int q = 0; q < N; q++) o[db][QB0 + q] *= alpha[q];
      }
    }
#pragma unroll
    for (int q = 0; q < N; q++) l_run[QB0 + q] += ps[q];
  };
  // S of N query blocks from QB0 on
  auto qk = [&](int slot, auto qb0, auto&& s) {
    constexpr int QB0 = decltype(qb0)::value, N = sizeof(s[0]) / sizeof(f32x4);
#pragma unroll
    for (int kb = 0; kb < 2; kb++)
#pragma unroll
      for (int ks = 0; ks < 4; ks++) {
        const bf16x8 ka = read_k(ka_addr[ks] + 16 * kb * kRow + slot * kSlot);
#pragma unroll
        for (int q = 0; q < N; q++) {
          if (ks == 0) mfma_first(s[kb][q], ka, qB[QB0 + q][ks]);
          else mfma_next(s[kb][q], ka, qB[QB0 + q][ks]);
        }
      }
    mfma_settle();
#pragma unroll
    for (int q = 0; q < N; q++) asm volatile("" : "+v"(s[0][q]), "+v"(s[1][q]));
  };
  // O of N query blocks from QB0 on
  auto pv = [&](int slot, auto qb0, auto n, bf16x8* pw) {
    constexpr int QB0 = decltype(qb0)::value, N = decltype(n)::value;
#pragma unroll
    for (int q = 0; q < N; q++) pin(pw[q]);
    acc_ready<ACC>(o);
#pragma unroll
    for (int q = 0; q < N; q++) pin(pw[q]);
#pragma unroll
    for (int db = 0; db < 8; db++) {
      const bf16x8 a = read_vt(va_addr[db] + slot * kSlot);
#pragma unroll
      for (int q = 0; q < N; q++) mfma_acc<ACC>(o[db][QB0 + q], a, pw[q]);
    }
  };
  auto qk_all = [&](int slot, f32x4 (&s)[2][QB]) { qk(slot, Tag<0>{}, s); };
  auto softmax_all = [&](const f32x4 (&s)[2][QB], bf16x8 (&pw)[QB]) { softmax(Tag<0>{}, s, pw); };
  auto pv_all = [&](int slot, bf16x8 (&pw)[QB]) { pv(slot, Tag<0>{}, Tag<QB>{}, pw); };

  // operand i of a step: K operand (key block i%2, d slice i/2) for i < 8, V^T operand of d block i - 8 beyond
  auto load_opnd = [&](auto idx, auto ks, auto vs) -> bf16x8 {
    constexpr int i = decltype(idx)::value, k = i & 7;
    if constexpr (i >= 8) return read_vt(va_addr[k] + value_of(slot_off(vs, Tag<0>{})));
    else return read_k(ka_addr[k >> 1] + value_of(slot_off(ks, Tag<16 * (k & 1) * kRow>{})));
  };
  auto ring_slot = [](int j) { return (int)((unsigned)j % (unsigned)RING); };
  bf16x8 pre[PD];

  // ---- steady step t in ring slot TR: QK(t+1), SM(t), PV(t-1); requests K and V of t + LA from base
  auto step = [&](auto par, auto&& slot, const unsigned char* kbase, const unsigned char* vbase) {
    constexpr int C = decltype(par)::value;
    auto KS = slot(Tag<1>{});
    auto VS = slot(Tag<-1>{});
    auto KN = slot(Tag<2>{});
    const auto KR = slot(Tag<KA>{});
    const auto VR = slot(Tag<VA>{});
    opaque(KS);                                          // run-time slots: operand addresses are made where they are used,
    opaque(VS);                                          // not kept in registers through the step
    opaque(KN);
    f32x4 (&s)[2][QB] = sb[C];
    f32x4 (&sn)[2][QB] = sb[C ^ 1];
    const bf16x8 (&pp)[QB] = pb[C ^ 1];
    u32x4 pn[QB];
    float x[2], ps[QB], w[2];
    bf16x8 op[16 + PD];
    static_for<0, PD>([&](auto idx) { op[decltype(idx)::value] = pre[decltype(idx)::value]; });
    static_for<0, 16>([&](auto idx) {
      constexpr int i = decltype(idx)::value, k = i & 7;
      // request of this group, where a group reads one operand half only
      constexpr int rq = i < 4 ? i * NI / 4 : i >= 12 ? NI + (i - 12) * NI / 4 : -1;
      constexpr bool rq_on = NI == 4 ? rq >= 0 : rq >= 0 && (i & 1) == 0;
      static_for<0, QB>([&](auto qtag) {
        constexpr int qb = decltype(qtag)::value, kb = k & 1, ks = k >> 1;
        // four MFMAs per pair of weights: query block, key block and row of the pair
        constexpr int n = i * QB + qb, pair = n >> 2, part = n & 3, wq = pair >> 2, wkb = (pair >> 1) & 1, wr = 2 * (pair & 1);
        constexpr int qm = i & 1 ? QB - 1 - qb : qb;                  // there and back: either A or B stays from one MFMA to the next
        if constexpr (i >= 8) mfma_acc<ACC>(o[k][qm], op[i], pp[qm]);
        else if constexpr (ks == 0) mfma_first(sn[kb][qm], op[i], qB[qm][ks]);
        else mfma_next(sn[kb][qm], op[i], qB[qm][ks]);
        __builtin_amdgcn_sched_barrier(0);
        // what is free behind an MFMA
        if constexpr (qb == 0) {
          if constexpr (i + PD < 16) op[i + PD] = load_opnd(Tag<i + PD>{}, KS, VS);
          else op[i + PD] = load_opnd(Tag<i + PD - 16>{}, KN, VS);
        }
        if constexpr (rq_on && qb == QB / 2 - 1) request_m0(KR, VR, Tag<rq>{});
        if constexpr (rq_on && qb == QB / 2) request_one(kbase, vbase, Tag<rq>{});
        if constexpr (qb == QB - 1 && i < 15) pin(op[i + 1]);         // its wait goes here
        __builtin_amdgcn_sched_barrier(0);
        if constexpr (part == 0) {
          x[0] = expo(s[wkb][wq][wr], wq);
          x[1] = expo(s[wkb][wq][wr + 1], wq);
        } else if constexpr (part == 1) {
          w[0] = __builtin_amdgcn_exp2f(x[0]);
          pin(w[0]);
        } else if constexpr (part == 2) {
          w[1] = __builtin_amdgcn_exp2f(x[1]);
          pin(w[1]);
        } else {
          ps[wq] = (pair & 3) == 0 ? w[0] + w[1] : (ps[wq] + w[0]) + w[1];
          unsigned pk = pack_bf16(w[0], w[1]);
          pin(pk);
          pn[wq][pair & 3] = pk;
          pin(ps[wq]);
        }
        __builtin_amdgcn_sched_barrier(0);
      });
    });
    static_for<0, PD>([&](auto idx) { pre[decltype(idx)::value] = op[16 + decltype(idx)::value]; });
#pragma unroll
    for (int qb = 0; qb < QB; qb++) pb[C][qb] = __builtin_bit_cast(bf16x8, pn[qb]);
    if (__builtin_expect(__builtin_amdgcn_ballot_w64(!(max_of(ps) <= kLazyBound)) != 0, 0)) {
      acc_ready<ACC>(o);
#pragma unroll
      for (int qb = 0; qb < QB; qb++) {
        const float d = fmaxf(expo(row_max(s[0][qb], s[1][qb]), qb) + kRefShift, 0.f);
        const float a = __builtin_amdgcn_exp2f(-d);
        l_run[qb] *= a;
        m_run[qb] += d;
        weights_of(s[0][qb], s[1][qb], qb, ps[qb], pb[C][qb]);
#pragma unroll
        for (int db = 0; db < 8; db++) o[db][qb] *= a;
      }
      acc_ready<ACC>(o);
    }
#pragma unroll
    for (int qb = 0; qb < QB; qb++) l_run[qb] += ps[qb];
    // What the next steps read and prefetch has landed; their requests go into slots that nobody reads until the next
    // barrier.  One barrier for two steps: at the end of an even step t K up to t + 4 and V up to t + 2, i.e. everything
    // but the requests of the last three steps.  One for each: K up to t + 3 and V up to t, i.e. everything but the requests
    // of the last two steps and those for V before them.
    if constexpr (!Cfg_::BAR2) {
      wait_vm<5 * NI>();
      __syncthreads();
    } else if constexpr (C == 0) {
      wait_vm<3 * 2 * NI>();
      __syncthreads();
    }
  };

  // ---- fill: one sub-tile of K or of V into its slot
  const SuffixBases sfx0 = suffix_bases(p.k_suffix, p.v_suffix);
  auto request_k = [&](auto j) {
    constexpr int J = decltype(j)::value;
    const int sub = min(J, n_pipe - 1);
    const unsigned char* base = kv_base(sub, fetch_off(sub), sfx0.k);
    static_for<0, NI>([&](auto idx) {
      request_m0(Tag<J % RING>{}, Tag<0>{}, idx);
      asm volatile("s_nop 0");
      request_one(base, base, idx);
    });
  };
  auto request_v = [&](auto j) {
    constexpr int J = decltype(j)::value;
    const int sub = min(J, n_pipe - 1);
    const unsigned char* base = kv_base(sub, fetch_off(sub), sfx0.v);
    static_for<NI, 2 * NI>([&](auto idx) {
      request_m0(Tag<0>{}, Tag<J % RING>{}, idx);
      asm volatile("s_nop 0");
      request_one(base, base, idx);
    });
  };
  int t = 0;
  // What the first sub-tile needs comes first: the wait for Q, which the compiler puts in front of the first product, is a
  // wait for every request before it.
  if (n_pipe > 0) {
    request_k(Tag<0>{});
    request_v(Tag<0>{});
    request_k(Tag<1>{});
  }
#pragma unroll
  for (int db = 0; db < 8; db++)
#pragma unroll
    for (int qb = 0; qb < QB; qb++) {
      o[db][qb] = zero4;
      pin_acc<ACC>(o[db][qb]);                          // set here, under the first requests
    }
  if (n_pipe > 0) {
#pragma unroll
    for (int qb = 0; qb < QB; qb++)
#pragma unroll
      for (int ks = 0; ks < 4; ks++) pin(qB[qb][ks]);
    wait_vm<0>();
    __syncthreads();
    // K(0..K2-1), V(0), V(1): what the first steady steps read.  The rest in the order in which steps would have asked for
    // it, K(j) in front of V(j - KA + VA): the waits of the steady steps count on that order.
    constexpr int K2 = Cfg_::BAR2 ? 5 : 4, DV = KA - VA;
    static_for<2, K2>([&](auto j) { request_k(j); });
    static_for<1, K2 - DV>([&](auto j) { request_v(j); });
    static_for<K2, RING>([&](auto j) {
      request_k(j);
      request_v(Tag<decltype(j)::value - DV>{});
    });
    qk_all(0, sb[0]);
    softmax_all(sb[0], pb[0]);
    t = 1;
    if (n_pipe > 1) {
      qk_all(1, sb[1]);
      // K(0), whose slot is asked for next, is done with
      wait_vm<((K2 - DV - 2) + 2 * (RING - K2)) * NI>();
      __syncthreads();
      if constexpr (KA == RING) {
        request_k(Tag<KA>{});
        request_v(Tag<VA>{});
      }
      if (t + 2 < n_pipe) {
        static_for<0, PD>([&](auto idx) { pre[decltype(idx)::value] = load_opnd(idx, Tag<2>{}, Tag<0>{}); });
        constexpr int U = Cfg_::UNROLL;
        const_paramsp ps = (const_paramsp)__builtin_amdgcn_kernarg_segment_ptr();
        const SuffixBases sfx = suffix_bases(ps->k_suffix, ps->v_suffix);
        if (t + U < n_pipe) {
          // offsets of sub-tiles t + VA .. t + KA + RING - 1
          int64_t off_cur[U + DV], off_nxt[U];
#pragma unroll
          for (int i = 0; i < U + DV; i++) off_cur[i] = fetch_off(min(t + VA + i, n_pipe - 1));
          auto turns = [&](auto sfx_tag, int end) {
            for (; t + U <= end; t += U) {
#pragma unroll
              for (int i = 0; i < U; i++) off_nxt[i] = fetch_off(min(t + KA + U + i, n_pipe - 1));
              static_for<0, U>([&](auto h) {
                constexpr int H = decltype(h)::value;
                auto base = [&](int j, int64_t off, const unsigned char* s) {
                  if constexpr (decltype(sfx_tag)::value != 0) return kv_base(min(j, n_pipe - 1), off, s);
                  else return pool + off;
                };
                step(Tag<(H + 1) & 1>{}, [](auto d) { return Tag<(H + 1 + decltype(d)::value + RING) % RING>{}; },
                     base(t + H + KA, off_cur[H + DV], sfx.k), base(t + H + VA, off_cur[H], sfx.v));
              });
#pragma unroll
              for (int i = 0; i < DV; i++) off_cur[i] = off_cur[U + i];
#pragma unroll
              for (int i = 0; i < U; i++) off_cur[DV + i] = off_nxt[i];
            }
          };
          // a turn asks for sub-tiles up to t + KA + U - 1, past the last one for that one again
          turns(Tag<0>{}, !SFX || n_pool == n_pipe ? n_pipe - 1 : min(n_pipe - 1, n_pool - KA));
          if constexpr (SFX) turns(Tag<1>{}, n_pipe - 1);
        }
        // pairs of steps, ring slots at run time
        for (; t + 2 < n_pipe; t += 2) {
          auto base = [&](int j, const unsigned char* s) { return kv_base(min(j, n_pipe - 1), fetch_off(min(j, n_pipe - 1)), s); };
          const unsigned char *k0 = base(t + KA, sfx.k), *k1 = base(t + 1 + KA, sfx.k), *v0 = base(t + VA, sfx.v), *v1 = base(t + 1 + VA, sfx.v);
          step(Tag<1>{}, [&](auto d) -> int { return ring_slot(t + decltype(d)::value); }, k0, v0);
          step(Tag<0>{}, [&](auto d) -> int { return ring_slot(t + 1 + decltype(d)::value); }, k1, v1);
        }
      }
    }
  }

  const_paramsp pe = (const_paramsp)__builtin_amdgcn_kernarg_segment_ptr();
  asm volatile("" : "+s"(pe));

  // ---- sub-tiles on or past the diagonal: requested in groups of at most RING - 2
  const unsigned char* ks = (const unsigned char*)pe->k_suffix;
  const unsigned char* vs = (const unsigned char*)pe->v_suffix;
  auto request_tail = [&](int j) {
    const int sfx_blk = 2 * (jb + j) + wblk - P / kBlockTokens;
    const int64_t boff = fetch_off(j);
    const unsigned char *kb = pool + boff, *vb = kb;
    if (ks && sfx_blk >= 0) {
      const int64_t soff = (int64_t)rd.q_off * row_b + (int64_t)sfx_blk * half_b;
      kb = ks + soff;
      vb = vs + soff - half_b;
    }
#pragma unroll
    for (int h = 0; h < NI; h++) {
      const bool live = (jb + j) * kSK + wblk * 16 + brow0 + 4 * h < ctx_len;
      const unsigned l_k = __builtin_amdgcn_readfirstlane(dma_lds + ring_slot(j) * kSlot + h * 1024);
      if (live) {
        dma_1k(scalar_ptr(kb), voff_k[h], l_k);
        dma_1k(scalar_ptr(vb), voff_v[h], l_k + kVBase);
      } else {
        *(u32x4*)(smem + (l_k - lds0) + kVBase + (lane << 4)) = (u32x4){0u, 0u, 0u, 0u};
      }
    }
  };
  constexpr int TG = RING - 2;
  auto request_group = [&](int j0) {
    for (int j = j0; j < min(n_sub, j0 + TG); j++) request_tail(j);
  };

  // ---- drain: PV(t-1), then the one or two sub-tiles that are left; S(t) is in sb[1] (t odd), P(t-1) in pb[0].  The first
  // group of the tail is requested before them: the slots of sub-tiles t and t + 1 are not among its own.
  if (n_pipe > 0) pv_all(ring_slot(t - 1), pb[0]);
  wait_vm<0>();
  __syncthreads();
  request_group(n_pipe);
  if (t > 0 && t < n_pipe) {
    softmax_all(sb[1], pb[1]);
    pv_all(ring_slot(t), pb[1]);
    if (t + 1 < n_pipe) {
      qk_all(ring_slot(t + 1), sb[0]);
      softmax_all(sb[0], pb[0]);
      pv_all(ring_slot(t + 1), pb[0]);
    }
  }
  for (int j0 = n_pipe; j0 < n_sub; j0 += TG) {
    if (j0 > n_pipe) {
      __syncthreads();                                   // everyone has read the group before
      request_group(j0);
    }
    wait_vm<0>();
    __syncthreads();
    for (int j = j0; j < min(n_sub, j0 + TG); j++) {
      const int k0 = (jb + j) * kSK;
      // row block by row block: V of a sub-tile that a block sees nothing of stays away from it (0 times infinity)
      static_for<0, HB>([&](auto hh) {
        constexpr int H = decltype(hh)::value;
        const int pq_min = P + wq0[H];
        if (!(wq0[H] < S && k0 <= P + min(wq0[H] + 32, S) - 1)) return;
        f32x4 s2[2][2];
        qk(ring_slot(j), Tag<2 * H>{}, s2);
        if (k0 + 31 > pq_min) {
#pragma unroll
          for (int kb = 0; kb < 2; kb++)
#pragma unroll
            for (int q = 0; q < 2; q++)
#pragma unroll
              for (int r = 0; r < 4; r++)
                if (k0 + 16 * kb + 4 * g + r > pq_min + 16 * q + c) s2[kb][q][r] = -INFINITY;
        }
        bf16x8 pw[2];
        softmax(Tag<2 * H>{}, s2, pw);
        pv(ring_slot(j), Tag<2 * H>{}, Tag<2>{}, pw);
      });
    }
  }

  // ---- results: of a cut tile's piece the unnormalised O, the reference (exponent units) and the row sum, else the output
  acc_ready<ACC>(o);
#pragma unroll
  for (int qb = 0; qb < QB; qb++) {
    if (wq0[qb >> 1] + 16 * (qb & 1) >= S) continue;     // wave-uniform: every lane takes part in the exchanges
    const float lt = quad_sum(l_run[qb]);
    const int tokq = wq0[qb >> 1] + 16 * (qb & 1) + c;
    if (wi.n_splits > 1) {
      const int64_t slot = ((int64_t)it * NHG + hg) * (HB * NW) + row_block(qb >> 1);
      // a row that lies before the piece's first key saw none: a row sum of 0 says so
      if (tokq < S) {
        const int64_t prow = slot * 32 + 16 * (qb & 1) + c;
        store_piece(pe->part_o + prow * kD, g, o, qb);
        if (g == 0) *(f32x2*)(pe->part_ml + prow * 2) = (f32x2){m_run[qb], P + tokq < jb * kSK ? 0.f : lt};
      }
    } else {
      const float inv = 1.f / lt;
      unsigned short* row = (unsigned short*)pe->out + ((int64_t)(rd.q_off + tokq) * Hq + hq[qb >> 1]) * kD;
#pragma unroll
      for (int d = 0; d < 4; d++) store_out(row, d, g, o[2 * d][qb], o[2 * d + 1][qb], inv, tokq < S);
    }
  }
  if (threadIdx.x == 0) clock_end(pe->clock.words);
}

}  // namespace attn
}  // namespace calvo

// Device helpers shared by the pipelined attention kernels (attn_pipe.hip, attn_duo.hip): vector
// types, the geometry of a 32-key sub-tile in LDS, compile-time loops, the lane-half exchange,
// pool -> LDS requests, and the two LDS operand reads.
#pragma once
#include "calvo_internal.h"

namespace calvo {
namespace attn {

typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;
typedef __attribute__((ext_vector_type(2))) __bf16 bf16x2;
typedef __attribute__((ext_vector_type(4))) float f32x4;
typedef __attribute__((ext_vector_type(2))) float f32x2;
typedef __attribute__((ext_vector_type(4))) unsigned int u32x4;
typedef __attribute__((ext_vector_type(2))) unsigned int u32x2;
typedef __attribute__((ext_vector_type(4))) short s16x4;
typedef __attribute__((ext_vector_type(8))) short s16x8;
typedef __attribute__((address_space(3))) unsigned char lds_u8;
// descriptor words, which a launch in front of these kernels wrote (launch_upload_words) and none of them does: read on the scalar unit
typedef const __attribute__((address_space(4))) int32_t* const_i32p;
__device__ inline WorkItem load_item(const WorkItem* items, int i) {
  const const_i32p w = (const_i32p)(uintptr_t)(items + i);
  return {w[0], w[1], w[2], w[3], w[4], w[5], w[6], w[7]};
}

constexpr int kD = 128;
constexpr int kSK = 32;                        // keys per sub-tile / ring slot
constexpr int kRow = 256;                      // bytes per token row of one head
constexpr int kSlot = kSK * kRow;              // 8192
template <int V>
struct Tag { static constexpr int value = V; };
// f(Tag<B>{}), f(Tag<B+1>{}), ... f(Tag<E-1>{}): a loop whose index is a compile-time constant
template <int B, int E, typename F>
__device__ inline void static_for(F&& f) {
  if constexpr (B < E) {
    f(Tag<B>{});
    static_for<B + 1, E>(f);
  }
}
constexpr float kRefShift = 16.f;       // the softmax reference is this far above the maximum it was taken from (exponent units)
constexpr float kLazyBound = 1.f;       // a lane's partial row sum of a sub-tile may reach this before the reference is raised

// lanes [32,64) of a <-> lanes [0,32) of b (the compiler builtin for this instruction returns
// its first result twice, hence inline asm)
__device__ inline void half_swap(float& a, float& b) {
  asm volatile("s_nop 1\n\tv_permlane32_swap_b32 %0, %1" : "+v"(a), "+v"(b));
}
__device__ inline float half_swap_max(float v) {
  float a = v, b = v;
  half_swap(a, b);
  return fmaxf(a, b);
}
__device__ inline float half_swap_sum(float v) {
  float a = v, b = v;
  half_swap(a, b);
  return a + b;
}

// maximum / sum over the four lanes c, c+16, c+32, c+48 (the lanes that share a query): every lane
// of the wave must call these
__device__ inline float quad_max(float v) {
  v = fmaxf(v, __shfl_xor(v, 16, 64));
  return half_swap_max(v);
}
__device__ inline float quad_sum(float v) {
  v += __shfl_xor(v, 16, 64);
  return half_swap_sum(v);
}

// two weights rounded to bf16 (nearest even), packed
__device__ inline unsigned pack_bf16(float a, float b) {
  bf16x2 w;
  w[0] = (__bf16)a;
  w[1] = (__bf16)b;
  return __builtin_bit_cast(unsigned, w);
}

// odd rows of 16 lanes of a <-> even rows of b
__device__ inline void row_swap(unsigned& a, unsigned& b) {
  asm volatile("s_nop 1\n\tv_permlane16_swap_b32 %0, %1" : "+v"(a), "+v"(b));
}
// One output row's d = 32p .. 32p + 31 from two accumulator tiles (d blocks 2p and 2p + 1, lane (c, g): d = 4g + r of
// row c), times inv, as 16 bytes per lane; row: the lane's output row.  Lanes g and g ^ 1 exchange halves first: 64
// consecutive bytes per row and instruction instead of 32.
__device__ inline void store_out(unsigned short* row, int p, int g, const f32x4& a, const f32x4& b, float inv, bool ok) {
  unsigned a0 = pack_bf16(a[0] * inv, a[1] * inv), a1 = pack_bf16(a[2] * inv, a[3] * inv);
  unsigned b0 = pack_bf16(b[0] * inv, b[1] * inv), b1 = pack_bf16(b[2] * inv, b[3] * inv);
  row_swap(a0, b0);
  row_swap(a1, b1);
  if (ok) *(u32x4*)(row + 32 * p + 16 * (g & 1) + 8 * (g >> 1)) = (u32x4){a0, a1, b0, b1};
}

// O of one block of 16 rows of a piece (tile db: d = 16db + 4g + r of row c); po: the lane's row
template <int QB>
__device__ inline void store_piece(float* po, int g, const f32x4 (&o)[8][QB], int qb) {
#pragma unroll
  for (int db = 0; db < 8; db++) *(f32x4*)(po + 16 * db + 4 * g) = o[db][qb];
}

// Suffix token i of request r sits at absolute position P_r + i: slot table_r[pos / 16], row pos % 16 of the K half and of the
// V half.  One thread per 16-byte chunk of a row, four chunks of K and of V in flight: this is workgroup wg of n_wgs with 256 threads.
// A row looks for its request by halving: one after the other, 256 requests cost a workgroup some 60 us of waiting for descriptors (256
// requests of 1024+64 tokens 725 us a call of three callers, 380 this way; 128 of 1024+256, 8Q/8KV, 639 and 297).
__device__ inline void append_suffix(const AppendParams& p, int wg, int n_wgs, int tid) {
  const int64_t n = (int64_t)p.total_tokens * p.row_chunks, stride = (int64_t)n_wgs * 256;
  const int64_t half_chunks = (int64_t)kBlockTokens * p.row_chunks;   // one K (or V) half of a block
  const u32x4* ks = (const u32x4*)p.k_suffix;
  const u32x4* vs = (const u32x4*)p.v_suffix;
  u32x4* pool = (u32x4*)p.pool_layer;
  auto move = [&](int64_t i0, auto count) {
    constexpr int N = decltype(count)::value;
    u32x4 k[N], v[N];
    int64_t dst[N];
#pragma unroll
    for (int u = 0; u < N; u++) {
      const int64_t i = i0 + u * stride;
      k[u] = ks[i];
      v[u] = vs[i];
    }
#pragma unroll
    for (int u = 0; u < N; u++) {
      const int64_t i = i0 + u * stride;
      const int32_t tok = (int32_t)(i / p.row_chunks);
      const int32_t c = (int32_t)(i - (int64_t)tok * p.row_chunks);
      int r = 0;                                                      // the last request that begins at or before the token
      for (int end = p.n_reqs; end - r > 1;) {
        const int mid = (r + end) / 2;
        if (tok >= p.reqs[mid].q_off) r = mid;
        else end = mid;
      }
      const ReqDesc rd = p.reqs[r];
      const int32_t pos = rd.prefix_len + (tok - rd.q_off);
      const int64_t slot = p.tables[rd.table_off + pos / kBlockTokens];
      dst[u] = slot * 2 * half_chunks + (int64_t)(pos % kBlockTokens) * p.row_chunks + c;
    }
#pragma unroll
    for (int u = 0; u < N; u++) {
      pool[dst[u]] = k[u];
      pool[dst[u] + half_chunks] = v[u];
    }
  };
  int64_t i = (int64_t)wg * 256 + tid;
  for (; i + 3 * stride < n; i += 4 * stride) move(i, Tag<4>{});
  for (; i < n; i += stride) move(i, Tag<1>{});
}

// Workgroups behind those of the tiles in a launch that takes the suffix rows along (append_wgs).  They run beside the
// tiles; at the end of a tile's workgroup the rows were in the way of its results (us a call of one caller, there / here: 3072+40
// tokens, 8Q/8KV, 15.6 / 14.4, 512+1 13.3 / 12.9, 448+155 18.2 / 17.7).
inline unsigned append_wgs(const AttnParams& p) { return p.k_suffix ? calvo::append_wgs(p.total_tokens, p.n_kv_heads) : 0; }
__device__ inline bool append_wg(const AttnParams& p) {
  if ((int)blockIdx.x < p.attn_wgs) return false;
  AppendParams app{p.k_suffix, p.v_suffix, const_cast<void*>(p.pool_layer), p.reqs, p.tables, p.n_reqs, p.total_tokens,
                   p.n_kv_heads * (kRow / 16)};
  append_suffix(app, blockIdx.x - p.attn_wgs, gridDim.x - p.attn_wgs, threadIdx.x);
  if (threadIdx.x == 0) clock_end(p.clock.words);
  return true;
}

// 64 lanes x 16 bytes from global memory (uniform base + per-lane byte offset) to 1 KiB of LDS
// starting at lds_addr (uniform).  Completion is tracked by vmcnt.  No "memory" clobber on
// purpose: every read of the deposited data sits behind wait_vm + a workgroup barrier, and a
// clobber would stop the compiler from keeping the block-table loads on the scalar unit.
__device__ inline void dma_1k(const unsigned char* sbase, unsigned voff, unsigned lds_addr) {
  asm volatile("s_mov_b32 m0, %2\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, %1"
               :
               : "v"(voff), "s"(sbase), "s"(lds_addr));
}
// a wave-uniform address that the compiler keeps in vector registers, back in scalar ones
__device__ inline const unsigned char* scalar_ptr(const unsigned char* p) {
  const unsigned long long x = (unsigned long long)p;
  return (const unsigned char*)((unsigned long long)(unsigned)__builtin_amdgcn_readfirstlane((int)x) |
                                (unsigned long long)(unsigned)__builtin_amdgcn_readfirstlane((int)(x >> 32)) << 32);
}
// compiler-level fence for one value: it is 'rewritten' here, so its producers stay above this
// point and its consumers below it; emits no instruction
template <typename T>
__device__ inline void pin(T& x) {
  asm volatile("" : "+v"(x));
}
template <int N>
__device__ inline void wait_vm() {
  asm volatile("s_waitcnt vmcnt(%0)" : : "n"(N));
}

__device__ inline bf16x8 read_k(const lds_u8* a) { return *(const __attribute__((address_space(3))) bf16x8*)a; }
// V^T operand of a 16x16x32 MFMA: four keys for the lane's d from the rows the 16-lane group points
// at, and four more from 16 rows further on
__device__ inline bf16x8 read_vt(const lds_u8* a) {
  const s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((s16x4 __attribute__((address_space(3)))*)(a));
  const s16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((s16x4 __attribute__((address_space(3)))*)(a + 16 * kRow));
  const s16x8 both = __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
  return __builtin_bit_cast(bf16x8, both);
}

}  // namespace attn
}  // namespace calvo

// Ragged paged split-KV decode attention for gfx950 (MI355X).
//
// One decode step of one layer over Tangram's ragged cache (Section 4.2 of
// arXiv 2606.06302): every KV head h of request b keeps its own number of
// retained rows, stored in the pages of its head group.  The host partition
// (tg_build_plan, Algorithm 1's proportional rule or the sequential fill)
// cuts every (b, h) into page-aligned chunks and places them on n_bins bins;
// worker k of the launch runs bin k (a wave in the bf16 matrix-core kernel, a
// workgroup in the fp32 one and in the vector kernel, which few query heads and
// few bins take).  A chunk of a split unit writes an fp32 partial (o, lse), and
// the partials of every split unit are combined with a log-sum-exp merge
// (split-KV decoding, Section 2.2.3): by a merge kernel launched right after on
// the same stream, or, with arrival counters, inside the head_dim-128 bf16
// launch by the piece that finishes last (plans of few pieces per unit).  The
// in-launch merge orders partials and counters with device-scope stores, loads
// and atomics only: a fence for ordinary stores would write back and invalidate
// the whole L2 of an XCD.
//
// Open-ended items (the chunk that ends a unit in a plan built for several
// steps) run to the unit's live length, and can append the step's new token
// themselves: the row is taken from the token buffer instead of the pool,
// then stored into the pool, and the live length advanced, at the item's end.
//
// The workgroup kernels deal the pages of an item round-robin to their 4 waves;
// every wave keeps its own online-softmax state and the states are merged
// through LDS at the end of the item.  The wave index is made
// wave-uniform (readfirstlane) so that all item/page bookkeeping is scalar.
#include <hip/hip_runtime.h>

#include <array>
#include <cmath>
#include <cstring>
#include <mutex>
#include <utility>

#include "tg_device.h"
#include "tg_internal.h"

namespace {

using namespace tgd;

constexpr int kWaves = 4;
constexpr int kBlock = 64 * kWaves;
constexpr int kPage = 16;

// 16 bytes as a native vector so staged page data stays in VGPRs
typedef uint32_t u4 __attribute__((ext_vector_type(4)));

template <typename T>
struct Store;
template <>
struct Store<float> {
  static constexpr int kBytes = 4;
};
template <>
struct Store<uint16_t> {
  static constexpr int kBytes = 2;
};

// Partial dot product of one 16-byte chunk of K with the matching q chunk.
template <typename T>
__device__ __forceinline__ float chunk_dot(const u4& k, const u4& q, float acc);
template <>
__device__ __forceinline__ float chunk_dot<uint16_t>(const u4& k, const u4& q, float acc) {
  acc = dot2_bf16(k.x, q.x, acc);
  acc = dot2_bf16(k.y, q.y, acc);
  acc = dot2_bf16(k.z, q.z, acc);
  acc = dot2_bf16(k.w, q.w, acc);
  return acc;
}
template <>
__device__ __forceinline__ float chunk_dot<float>(const u4& k, const u4& q, float acc) {
  acc = fmaf(__uint_as_float(k.x), __uint_as_float(q.x), acc);
  acc = fmaf(__uint_as_float(k.y), __uint_as_float(q.y), acc);
  acc = fmaf(__uint_as_float(k.z), __uint_as_float(q.z), acc);
  acc = fmaf(__uint_as_float(k.w), __uint_as_float(q.w), acc);
  return acc;
}

// Unpack a 16-byte chunk of V into fp32.
template <typename T>
__device__ __forceinline__ void chunk_unpack(const u4& v, float* f);
template <>
__device__ __forceinline__ void chunk_unpack<uint16_t>(const u4& v, float* f) {
  f[0] = bf16_lo(v.x); f[1] = bf16_hi(v.x);
  f[2] = bf16_lo(v.y); f[3] = bf16_hi(v.y);
  f[4] = bf16_lo(v.z); f[5] = bf16_hi(v.z);
  f[6] = bf16_lo(v.w); f[7] = bf16_hi(v.w);
}
template <>
__device__ __forceinline__ void chunk_unpack<float>(const u4& v, float* f) {
  f[0] = __uint_as_float(v.x); f[1] = __uint_as_float(v.y);
  f[2] = __uint_as_float(v.z); f[3] = __uint_as_float(v.w);
}

template <typename T>
__device__ __forceinline__ void store_out(T* dst, float v);
template <>
__device__ __forceinline__ void store_out<float>(float* dst, float v) { *dst = v; }
template <>
__device__ __forceinline__ void store_out<uint16_t>(uint16_t* dst, float v) { *dst = f32_to_bf16(v); }

// four consecutive outputs, one 16- or 8-byte store (dst 16- or 8-byte aligned)
template <typename T>
__device__ __forceinline__ void store_out4(T* dst, float v0, float v1, float v2, float v3);
template <>
__device__ __forceinline__ void store_out4<float>(float* dst, float v0, float v1, float v2, float v3) {
  *reinterpret_cast<float4*>(dst) = make_float4(v0, v1, v2, v3);
}
template <>
__device__ __forceinline__ void store_out4<uint16_t>(uint16_t* dst, float v0, float v1, float v2, float v3) {
  *reinterpret_cast<uint2*>(dst) = make_uint2(uint32_t(f32_to_bf16(v0)) | (uint32_t(f32_to_bf16(v1)) << 16),
                                              uint32_t(f32_to_bf16(v2)) | (uint32_t(f32_to_bf16(v3)) << 16));
}

struct DecodeParams {
  const void* q;
  const u4* pool;            // 16-byte view of the page pool
  const int32_t* pt_pages;
  const tg_work_item* items;
  const int32_t* bin_offsets;
  const int32_t* unit_splits;
  const int32_t* unit_partial_base;
  void* out;
  float* lse;
  float* part_o;             // [num_partials][gqa][d]
  float* part_lse;           // [num_partials][gqa]
  int64_t page_chunks;       // 16-byte chunks per physical page
  int32_t heads_per_group;
  int32_t num_q_heads;
  int32_t num_kv_heads;
  int32_t n_bins;
  int32_t gqa;               // query heads per KV head
  uint64_t* timestamps;      // [n_bins][2] start / end stamps, or NULL
  const int32_t* live;       // live lengths of this layer: live[b * live_stride + h], or NULL
  int32_t live_stride;
  float scale_log2;          // sm_scale * log2(e)
  float scale;               // sm_scale
  int32_t* merge_counters;   // [B*H] arrival counters of the in-launch merge, or NULL
  // in-launch decode-token append (open items only), or append_k == NULL
  const u4* append_k;        // [B][H] token rows, 16-byte chunks
  const u4* append_v;
  u4* pool_w;                // the pool, written at the appended rows only
  int32_t* live_w;           // = live, written by the open items
  int32_t* append_full;      // set when a unit cannot take its token, or NULL
};

// An open-ended item (tok_end = -capacity) runs to the head's live length n,
// kept within [tok_begin + 1, capacity]; without live lengths, to capacity.
// With the in-launch append, an open item with tok_begin <= n < capacity
// takes the new token as entry n and runs to n + 1 (*arow = n); otherwise
// *arow = -1, and -2 for an open item that cannot take the token.
__device__ __forceinline__ int resolve_open(int tok_begin, int tok_end, int n, bool append, int* arow) {
  const int cap = -tok_end;
  if (append && n >= tok_begin && n < cap) {
    *arow = n;
    return n + 1;
  }
  *arow = append ? -2 : -1;
  return min(max(n, tok_begin + 1), cap);
}

__device__ __forceinline__ int resolve_end(int tok_begin, int tok_end, int b, int h, const DecodeParams& p,
                                           int* arow) {
  *arow = -1;
  if (tok_end >= 0) return tok_end;
  const int n = p.live ? p.live[(int64_t)b * p.live_stride + h] : -tok_end;
  return resolve_open(tok_begin, tok_end, n, p.append_k != nullptr, arow);
}

__device__ __forceinline__ int wave_id() { return __builtin_amdgcn_readfirstlane(threadIdx.x >> 6); }

// End of an item: combine the per-wave states (m, l in LDS [kWaves][G],
// accumulators at acc + w*acc_stride + g*D + e) and write the final output or
// this chunk's fp32 partial (normalised o and its lse).  Called by the whole
// workgroup after a barrier.
template <typename T, int G, int D>
__device__ __forceinline__ void finish_item(const DecodeParams& p, const tg_work_item& item, const float (*sm_m)[G],
                                            const float (*sm_l)[G], const float* acc, int acc_stride) {
  const float cs = p.scale_log2;
  const int qh0 = item.kv_head * G;
  for (int o = threadIdx.x; o < G * D; o += kBlock) {
    const int g = o / D, e = o % D;
    float M = sm_m[0][g];
#pragma unroll
    for (int w = 1; w < kWaves; ++w) M = fmaxf(M, sm_m[w][g]);
    float L = 0.f, A = 0.f;
#pragma unroll
    for (int w = 0; w < kWaves; ++w) {
      const float f = fast_exp2((sm_m[w][g] - M) * cs);   // 0 for a wave that saw no rows
      L = fmaf(sm_l[w][g], f, L);
      A = fmaf(acc[w * acc_stride + g * D + e], f, A);
    }
    const float O = A / L;
    const float lse_nat = M * p.scale + logf(L);
    if (item.out_idx < 0) {
      store_out<T>(static_cast<T*>(p.out) + ((int64_t)item.b * p.num_q_heads + qh0 + g) * D + e, O);
      if (p.lse && e == 0) p.lse[(int64_t)item.b * p.num_q_heads + qh0 + g] = lse_nat;
    } else {
      p.part_o[((int64_t)item.out_idx * G + g) * D + e] = O;
      if (e == 0) p.part_lse[(int64_t)item.out_idx * G + g] = lse_nat;
    }
  }
}

// ---------------------------------------------------------------------------
// Vector kernel for few query heads and for few bins (vector_kernel_pays()
// below): the 4 waves of a workgroup share a bin, and with 1 to 4 query heads
// per KV head the vector ALU keeps up with them.  A page slab (P=16 rows of one head, d*sizeof(T) bytes each) is read
// with one 16-byte load per lane per 64 chunks; lane l owns chunk l % CPR of
// token row l / CPR (CPR = 16-byte chunks per row).  q.k uses v_dot2_f32_bf16
// on raw bf16 pairs (fp32 FMAs for fp32 data) and a DPP all-reduce over the CPR
// lanes of a row; the per-page max uses the gfx950 permlane16/32 swaps.
template <typename T, int D>
struct Tile {
  static constexpr int kRowBytes = D * Store<T>::kBytes;
  static constexpr int kCPR = kRowBytes / 16;
  static constexpr int kEPC = 16 / Store<T>::kBytes;
  static constexpr int kTPL = 64 / kCPR;
  static constexpr int kSlots = kPage / kTPL;
  static constexpr int kSlabChunks = kPage * kCPR;
  static_assert(kCPR == 8 || kCPR == 16 || kCPR == 32, "unsupported row size");
};

template <typename T, int D, int GQA>
__global__ void __launch_bounds__(kBlock) tg_decode_kernel(DecodeParams p, const tg_work_item* __restrict__ items,
                                                          const int32_t* __restrict__ pt_pages,
                                                          const int32_t* __restrict__ bin_offsets,
                                                          const u4* __restrict__ pool) {
  using TL = Tile<T, D>;
  constexpr int CPR = TL::kCPR, EPC = TL::kEPC, TPL = TL::kTPL, NS = TL::kSlots;

  __shared__ float sm_m[kWaves][GQA];
  __shared__ float sm_l[kWaves][GQA];
  __shared__ float sm_acc[kWaves][GQA][D];

  const int lane = threadIdx.x & 63;
  const int wave = wave_id();
  const int c = lane % CPR;
  const int r = lane / CPR;
  const int it_begin = bin_offsets[blockIdx.x], it_end = bin_offsets[blockIdx.x + 1];
  const float cs = p.scale_log2;
  const uint64_t t_start = __builtin_amdgcn_s_memrealtime();

  for (int it = it_begin; it < it_end; ++it) {
    tg_work_item item = items[it];
    int arow;   // entry that takes the appended token, or < 0
    item.tok_end = resolve_end(item.tok_begin, item.tok_end, item.b, item.kv_head, p, &arow);
    const int qh0 = item.kv_head * GQA;
    const int64_t toff = ((int64_t)item.b * p.num_kv_heads + item.kv_head) * CPR;   // token row, in chunks
    u4 qv[GQA];
    {
      const u4* qbase = reinterpret_cast<const u4*>(static_cast<const T*>(p.q) +
                                                    ((int64_t)item.b * p.num_q_heads + qh0) * D);
#pragma unroll
      for (int g = 0; g < GQA; ++g) qv[g] = qbase[g * CPR + c];
    }
    float m[GQA], l[GQA], acc[GQA][EPC];
#pragma unroll
    for (int g = 0; g < GQA; ++g) {
      m[g] = -INFINITY;
      l[g] = 0.f;
#pragma unroll
      for (int e = 0; e < EPC; ++e) acc[g][e] = 0.f;
    }
    const int ntok = item.tok_end - item.tok_begin;
    const int npages = (ntok + kPage - 1) / kPage;
    const int32_t* pt = pt_pages + item.pt_base + item.tok_begin / kPage;
    const int64_t slab_k = (int64_t)item.slot * TL::kSlabChunks;
    const int64_t slab_v = ((int64_t)p.heads_per_group + item.slot) * TL::kSlabChunks;
    for (int pi = wave; pi < npages; pi += kWaves) {
      u4 kc[NS], vc[NS];
      {
        const int64_t pg = (int64_t)pt[pi] * p.page_chunks;
        const u4* kb = pool + pg + slab_k + lane;
        const u4* vb = pool + pg + slab_v + lane;
#pragma unroll
        for (int j = 0; j < NS; ++j) {
          kc[j] = kb[j * 64];
          vc[j] = vb[j * 64];
        }
      }
      if (arow >= 0 && pi == npages - 1) {   // the appended entry is the item's last: its row comes from the token
#pragma unroll
        for (int j = 0; j < NS; ++j)
          if (j * TPL + r == (arow & (kPage - 1))) {
            kc[j] = p.append_k[toff + c];
            vc[j] = p.append_v[toff + c];
          }
      }
      const int nvalid = min(kPage, ntok - pi * kPage);
      float s[NS][GQA];
#pragma unroll
      for (int j = 0; j < NS; ++j) {
#pragma unroll
        for (int g = 0; g < GQA; ++g) {
          float d = chunk_dot<T>(kc[j], qv[g], 0.f);
          if constexpr (CPR == 32) d = swap16_sum(group_sum<16>(d));
          else d = group_sum<CPR>(d);
          s[j][g] = d;
        }
      }
      if (nvalid < kPage) {
#pragma unroll
        for (int j = 0; j < NS; ++j) {
          const bool ok = j * TPL + r < nvalid;
#pragma unroll
          for (int g = 0; g < GQA; ++g) s[j][g] = ok ? s[j][g] : -INFINITY;
          if (!ok) vc[j] = u4(0u);
        }
      }
#pragma unroll
      for (int g = 0; g < GQA; ++g) {
        float mx = s[0][g];
#pragma unroll
        for (int j = 1; j < NS; ++j) mx = fmaxf(mx, s[j][g]);
        mx = rows_max<CPR>(mx);
        if (mx > m[g]) {
          const float alpha = fast_exp2((m[g] - mx) * cs);
          m[g] = mx;
          l[g] *= alpha;
#pragma unroll
          for (int e = 0; e < EPC; ++e) acc[g][e] *= alpha;
        }
      }
#pragma unroll
      for (int j = 0; j < NS; ++j) {
        float vf[EPC];
        chunk_unpack<T>(vc[j], vf);
#pragma unroll
        for (int g = 0; g < GQA; ++g) {
          const float pj = fast_exp2(fmaf(s[j][g], cs, -m[g] * cs));
          l[g] += pj;
#pragma unroll
          for (int e = 0; e < EPC; ++e) acc[g][e] = fmaf(pj, vf[e], acc[g][e]);
        }
      }
    }
#pragma unroll
    for (int g = 0; g < GQA; ++g) {
      l[g] = rows_sum<CPR>(l[g]);
#pragma unroll
      for (int e = 0; e < EPC; ++e) acc[g][e] = rows_sum<CPR>(acc[g][e]);
    }
    if (lane == 0) {
#pragma unroll
      for (int g = 0; g < GQA; ++g) {
        sm_m[wave][g] = m[g];
        sm_l[wave][g] = l[g];
      }
    }
    if (r == 0) {
#pragma unroll
      for (int g = 0; g < GQA; ++g)
#pragma unroll
        for (int e = 0; e < EPC; ++e) sm_acc[wave][g][c * EPC + e] = acc[g][e];
    }
    __syncthreads();
    finish_item<T, GQA, D>(p, item, sm_m, sm_l, &sm_acc[0][0][0], GQA * D);
    if (arow >= 0) {   // the token becomes entry arow of the cache; every thread read the length above
      if (threadIdx.x < 2 * CPR) {
        const bool is_k = threadIdx.x < CPR;
        const int ch = threadIdx.x % CPR;
        const int64_t pg = (int64_t)pt_pages[item.pt_base + arow / kPage] * p.page_chunks;
        p.pool_w[pg + (is_k ? slab_k : slab_v) + (arow % kPage) * CPR + ch] =
            is_k ? p.append_k[toff + ch] : p.append_v[toff + ch];
      }
      if (threadIdx.x == 0) p.live_w[(int64_t)item.b * p.live_stride + item.kv_head] = arow + 1;
    } else if (arow == -2 && threadIdx.x == 0 && p.append_full) {
      *p.append_full = 1;
    }
    __syncthreads();
  }
  if (p.timestamps && threadIdx.x == 0) {   // one lane, vector stores
    p.timestamps[2 * blockIdx.x] = t_start;
    p.timestamps[2 * blockIdx.x + 1] = __builtin_amdgcn_s_memrealtime();
  }
}

// ---------------------------------------------------------------------------
// bf16, head_dim D = 64 or 128, any gqa G in 1..16: matrix cores.
//
// Every wave is an independent worker: bin 4*blockIdx.x + wave of the plan.
// There is no barrier and no cross-wave merge; a wave runs its bin's items one
// after the other in steps of 128/D pages (8 KiB: one page of 16 tokens at
// head_dim 128, two pages at 64; the last step of an item of odd pages reads
// its one page twice and masks the second).
//
// Data movement.  Steps stream from HBM straight into a ring of R buffers
// in the wave's own LDS with gfx950's global_load_lds_dwordx4 (no staging
// registers): step k+R-1 is issued before step k is computed, so R-1 steps
// (8 KiB each) stay in flight while the wave computes.  The DMA is issued from
// inline assembly, invisible to the compiler's wait-count pass (which would
// otherwise drain every load before each LDS read), and the wave waits for
// step k with an explicit vmcnt that counts the DMA instructions issued after
// it; any other vector memory operation issued later (output stores) only
// makes that wait stricter.  Page ids and work items are read through the
// constant address space, i.e. with scalar loads, which the vector memory
// counter does not see.  The queries of an item are DMA'd with its first step
// into one of R-1 per-wave q slots and moved to registers when the item starts.
//
// Arithmetic, per 16-token page, with the query heads of the KV head as the
// 16 columns of the MFMA tiles (columns past G repeat a real head and are
// never stored):
//   * S^T[16 tok][16 heads] = K q^T: D/32 x v_mfma_f32_16x16x32_bf16, A = K rows
//     read from LDS (16 bytes per lane), B = q from registers.  Lane
//     (col, rb) = (lane % 16, lane / 16) receives tokens 4rb..4rb+3 of head col.
//   * online softmax on a step's 4 (or 8) values per lane; the row max and sum of a head
//     combine the 4 lanes of its column with the gfx950 permlane swaps.  The
//     running max is only raised when a step exceeds it by more than 8 (in
//     log2 units), so rescales are rare and p stays <= 2^8.
//   * O^T[16 dims][16 heads] += V^T P^T, one product per 16 dims: 16 tokens deep
//     (v_mfma_f32_16x16x16_bf16) at head_dim 128, 32 deep (16x16x32, k index
//     8rb+i = token 4rb+i of the first page, then of the second) at 64, there
//     once for each of three bf16 parts of P, which hold its 24 bits (fp32
//     partials are 5.9e-8 from 64 bits, 6.1e-8 on the vector kernel; with two
//     parts 1.0e-6, at 1 to 5 % less time).  P^T is the S^T tile of the same
//     lane (the result layout of the first product is the operand layout of the
//     second; rounded to bf16 at head_dim 128), and V^T comes from LDS with
//     ds_read_b64_tr_b16, whose 4x4 lane transpose turns row-major V rows into
//     the 4-consecutive-token operand.
//   * LDS layout: chunk c (16 bytes) of token row r sits at position c ^ k_swz(r)
//     in the K slab and at c ^ v_swz(r) in the V slab (the DMA lanes pick their
//     source chunk accordingly), so both operand reads are bank-conflict free:
//     r and 2r mod 16 with 256-byte rows; with 128-byte rows, where two rows
//     fill the 64 banks, (r/2) mod 8 and 2((r/2) mod 4).
// The accumulator of a lane belongs to one head, so rescaling and the final
// normalisation need no cross-lane traffic.
//
// Bound by HBM.  At head_dim 64 a page holds half the bytes for the same
// softmax; two pages per step keep the wave's instructions per byte near those
// at 128.  32 requests, gqa 4, 2048 to 16384 tokens (182 and 88 MB a layer): 33
// and 20 us, 5.6 and 4.4 TB/s, against 42 and 26 us on the vector kernel.

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef short s16x4 __attribute__((ext_vector_type(4)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef __bf16 bf16x4_vs __attribute__((__vector_size__(4 * sizeof(__bf16))));

#define TG_CONST __attribute__((address_space(4)))
#define TG_LDS __attribute__((address_space(3)))

__device__ __forceinline__ uint32_t lds_address(const void* ptr) {
  return static_cast<uint32_t>(reinterpret_cast<uintptr_t>((const TG_LDS void*)ptr));
}

// 16 bytes per lane from global memory into LDS at m0_base + 16 * lane.  A
// decode step reads every retained K/V byte exactly once, so the loads carry
// the non-temporal (streaming) policy, at device scope.
__device__ __forceinline__ void lds_dma16(const void* src, uint32_t m0_base) {
  asm volatile("global_load_lds_dwordx4 %0, off nt sc1" ::"v"(src), "{m0}"(m0_base) : "memory");
}

// vmcnt(n) with expcnt/lgkmcnt left alone; the memory clobber keeps LDS reads
// below it.
template <int N>
__device__ __forceinline__ void wait_vmcnt() {
  static_assert(N >= 0 && N < 64, "vmcnt is 6 bits");
  asm volatile("s_waitcnt vmcnt(%0)" ::"n"(N) : "memory");
}

__device__ __forceinline__ void wait_lgkmcnt0() { asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory"); }

// field-wise copy: the implicit copy constructor cannot bind a constant-space object
// (live lengths too: the open item that appends writes its length only after
// its last scalar read of it)
__device__ __forceinline__ tg_work_item load_item(const TG_CONST tg_work_item* src, const DecodeParams& p, int* arow) {
  tg_work_item r;
  r.pt_base = src->pt_base;
  r.b = src->b;
  r.kv_head = src->kv_head;
  r.slot = src->slot;
  r.tok_begin = src->tok_begin;
  r.tok_end = src->tok_end;
  r.out_idx = src->out_idx;
  *arow = -1;
  if (r.tok_end < 0) {
    const TG_CONST int32_t* live = (const TG_CONST int32_t*)p.live;
    const int n = live ? live[(int64_t)r.b * p.live_stride + r.kv_head] : -r.tok_end;
    r.tok_end = resolve_open(r.tok_begin, r.tok_end, n, p.append_k != nullptr, arow);
  }
  return r;
}

// two fp32 values as one 64-bit word (lo first, as they sit in memory)
__device__ __forceinline__ uint64_t pack_f32x2(float lo, float hi) {
  return (uint64_t)__float_as_uint(lo) | ((uint64_t)__float_as_uint(hi) << 32);
}

__device__ __forceinline__ f32x4 mfma_qk(const u4& a, const u4& b, const f32x4& c) {
  return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, a), __builtin_bit_cast(bf16x8, b), c, 0, 0,
                                                 0);
}
__device__ __forceinline__ f32x4 mfma_pv(const s16x4& a, const s16x4& b, const f32x4& c) {
  return __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(a, b, c, 0, 0, 0);
}
// 8 k-values of an operand from two halves of 4
__device__ __forceinline__ u4 join(const s16x4& lo, const s16x4& hi) {
  const uint2 a = __builtin_bit_cast(uint2, lo), b = __builtin_bit_cast(uint2, hi);
  return u4{a.x, a.y, b.x, b.y};
}
// Lane l of each 16-lane block receives element l % 4 of the 8-byte rows
// addressed by lanes l/4, l/4 + 4, l/4 + 8, l/4 + 12 of the block.
__device__ __forceinline__ s16x4 lds_read_tr16(const void* ptr) {
  return __builtin_bit_cast(s16x4, __builtin_amdgcn_ds_read_tr16_b64_v4bf16((TG_LDS bf16x4_vs*)ptr));
}

// This file is built with -mllvm -amdgpu-mfma-vgpr-form: the accumulators stay
// in VGPRs, where the rescale multiplies them in place, instead of being
// copied between AGPRs and VGPRs on every page.
template <int D, int QMAX>   // QMAX 8 or 16: the q slots hold up to QMAX query heads
__global__ void __launch_bounds__(kBlock) tg_decode_mfma_kernel(DecodeParams p, const tg_work_item* __restrict__ items_g,
                                                               const int32_t* __restrict__ pt_g,
                                                               const int32_t* __restrict__ bin_offsets_g,
                                                               const u4* __restrict__ pool) {
  static_assert(D == 64 || D == 128, "head_dim 64 or 128");
  constexpr int KP = 128 / D;            // pages per step
  constexpr int kStep = KP * kPage;      // tokens per step
  constexpr int CPR = D / 8;             // 16-byte chunks per row
  constexpr int kSlab = kPage * CPR;     // chunks per K or V slab of a page
  constexpr int R = QMAX * D <= 1024 ? 4 : 3;   // LDS step buffers per wave (160 KiB a CU)
  constexpr int NQ = R - 1;              // LDS query buffers per wave
  constexpr int kQChunks = QMAX * CPR;
  constexpr int kDma = 8;                // DMA instructions per step: 4 K + 4 V
  constexpr float kSlack = 8.0f;
  static_assert(kPage == 16 && KP * kSlab == 256, "one step is 4 KiB of K and 4 KiB of V");
  auto k_swz = [](int r) { return D == 128 ? r & 15 : (r >> 1) & 7; };
  auto v_swz = [](int r) { return D == 128 ? (2 * r) & 15 : 2 * ((r >> 1) & 3); };

  __shared__ u4 sm_ring[kWaves][R][512];   // step: K slabs, then V slabs
  __shared__ u4 sm_q[kWaves][NQ][kQChunks];

  const TG_CONST tg_work_item* const items = (const TG_CONST tg_work_item*)items_g;
  const TG_CONST int32_t* const pt = (const TG_CONST int32_t*)pt_g;
  const TG_CONST int32_t* const bin_offsets = (const TG_CONST int32_t*)bin_offsets_g;

  const int lane = threadIdx.x & 63;
  const int wave = wave_id();
  const int bin = blockIdx.x * (blockDim.x / 64) + wave;   // one to four workers per workgroup
  if (bin >= p.n_bins) return;
  const uint64_t t_start = __builtin_amdgcn_s_memrealtime();
  const int it_begin = bin_offsets[bin], it_end = bin_offsets[bin + 1];
  if (it_begin >= it_end) {
    if (p.timestamps && lane == 0) {   // one lane, vector stores
      p.timestamps[2 * bin] = t_start;
      p.timestamps[2 * bin + 1] = t_start;
    }
    return;
  }
  const int G = p.gqa;
  const int col = lane & 15;            // head column of the MFMA tiles
  const int rb = lane >> 4;             // row block: tokens / dims 4rb..4rb+3
  const int hq = col < G ? col : col % G;
  const float cs = p.scale_log2;
  const uint32_t ring_lds = lds_address(&sm_ring[wave][0][0]);
  const uint32_t q_lds = lds_address(&sm_q[wave][0][0]);
  const u4* const qsrc = static_cast<const u4*>(p.q);
  const int nq = G * CPR;               // 16-byte chunks of one item's queries

  // DMA cursor over every step of every item of the bin (pi: step, ns: steps);
  // it caches the item's page count, table base, slot and query offset.
  struct Cursor {
    int it, pi, ns, np, slot, arow;
    int64_t pbase, qoff;
  };
  auto enter = [&](Cursor& cu, int it) {
    int arow;
    const tg_work_item im = load_item(items + it, p, &arow);
    cu.it = it;
    cu.pi = 0;
    cu.np = (im.tok_end - im.tok_begin + kPage - 1) / kPage;
    cu.ns = (cu.np + KP - 1) / KP;
    cu.slot = im.slot;
    cu.arow = arow >= 0 ? (arow - im.tok_begin) % kStep : -1;   // row of the last step that takes the new token
    cu.pbase = im.pt_base + im.tok_begin / kPage;
    cu.qoff = ((int64_t)im.b * p.num_q_heads + (int64_t)im.kv_head * G) * CPR;
  };
  auto advance = [&](Cursor& cu) {   // false (cursor unchanged) past the bin's last page
    if (cu.pi + 1 < cu.ns) {
      ++cu.pi;
      return true;
    }
    if (cu.it + 1 < it_end) {
      enter(cu, cu.it + 1);
      return true;
    }
    return false;
  };
  // page ids of the cursor's step (an odd item's last page twice)
  struct Ids {
    int32_t v[KP];
  };
  auto page_ids = [&](const Cursor& cu) {
    Ids r;
#pragma unroll
    for (int k = 0; k < KP; ++k) r.v[k] = pt[cu.pbase + (KP == 1 ? cu.pi : min(KP * cu.pi + k, cu.np - 1))];
    return r;
  };
  // queries (on an item's first step), then the step's K slabs, then its V slabs
  auto issue = [&](const Cursor& cu, const Ids& id, int ring) {
    if (cu.pi == 0) {
      const u4* qb = qsrc + cu.qoff;
      const uint32_t dst = q_lds + ((cu.it - it_begin) % NQ) * (kQChunks * 16);
#pragma unroll
      for (int j = 0; j < kQChunks / 64; ++j)
        if (j * 64 < nq) lds_dma16(qb + min(j * 64 + lane, nq - 1), dst + j * 1024);
    }
    constexpr int kPerPage = 4 / KP;       // 1 KiB instructions per slab
    constexpr int kRowsPerDma = 64 / CPR;
    const uint32_t dst = ring_lds + ring * 8192;
    const int pos = lane % CPR;            // chunk position within the row
    if (cu.arow >= 0 && cu.pi == cu.ns - 1) {   // the step that takes the new token: that row from the token
      const int64_t toff = ((int64_t)items[cu.it].b * p.num_kv_heads + items[cu.it].kv_head) * CPR;
      const u4* tk = p.append_k + toff;
      const u4* tv = p.append_v + toff;
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const u4* kb = pool + (int64_t)id.v[j / kPerPage] * p.page_chunks + cu.slot * kSlab;
        const int r = (j % kPerPage) * kRowsPerDma + lane / CPR;   // token row of the page
        const int c = pos ^ k_swz(r);
        lds_dma16((j / kPerPage) * kPage + r == cu.arow ? tk + c : kb + r * CPR + c, dst + j * 1024);
      }
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const u4* vb = pool + (int64_t)id.v[j / kPerPage] * p.page_chunks + (p.heads_per_group + cu.slot) * kSlab;
        const int r = (j % kPerPage) * kRowsPerDma + lane / CPR;
        const int c = pos ^ v_swz(r);
        lds_dma16((j / kPerPage) * kPage + r == cu.arow ? tv + c : vb + r * CPR + c, dst + 4096 + j * 1024);
      }
      return;
    }
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const u4* kb = pool + (int64_t)id.v[j / kPerPage] * p.page_chunks + cu.slot * kSlab;
      const int r = (j % kPerPage) * kRowsPerDma + lane / CPR;   // token row of the page, written by this lane
      lds_dma16(kb + r * CPR + (pos ^ k_swz(r)), dst + j * 1024);
    }
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const u4* vb = pool + (int64_t)id.v[j / kPerPage] * p.page_chunks + (p.heads_per_group + cu.slot) * kSlab;
      const int r = (j % kPerPage) * kRowsPerDma + lane / CPR;
      lds_dma16(vb + r * CPR + (pos ^ v_swz(r)), dst + 4096 + j * 1024);
    }
  };

  Cursor d;
  enter(d, it_begin);
  bool d_live = true;
  Ids d_id = page_ids(d);
#pragma unroll
  for (int r = 0; r < R - 1; ++r) {
    if (d_live) {
      issue(d, d_id, r);
      d_live = advance(d);
      if (d_live) d_id = page_ids(d);
    }
  }

  // lane-constant parts of the operand addresses
  const int k_off = col * CPR;                                 // A of q.k: token row col
  const int v_tok = lane >> 2;                                 // source row of the transposed read
  const int v_off = 4096 + v_tok * (CPR * 16) + (lane & 3) * 8;   // bytes within the step buffer
  const int v_x = v_swz(v_tok) >> 1;                           // 32-byte pairs of chunks are swizzled as one

  int it = it_begin, pi = 0, ns = 0, ntok = 0, k = 0, arow = -1;
  tg_work_item item;
  u4 qv[D / 32];
  float m = -INFINITY, l = 0.f;
  // acc2 (head_dim 64): what the lower parts of P add
  f32x4 acc[D / 16], acc2[D / 16];
  for (;;) {
    if (pi == 0) {   // item start: its queries were DMA'd just before its first step
      item = load_item(items + it, p, &arow);
      ntok = item.tok_end - item.tok_begin;
      ns = (ntok + kStep - 1) / kStep;
      if (d_live)
        wait_vmcnt<kDma * (R - 1)>();
      else
        wait_vmcnt<0>();
      const u4* qrow = &sm_q[wave][(it - it_begin) % NQ][hq * CPR + rb];
#pragma unroll
      for (int c = 0; c < D / 32; ++c) qv[c] = qrow[4 * c];
      wait_lgkmcnt0();   // the slot may be refilled by the DMA issued next
      m = -INFINITY;
      l = 0.f;
#pragma unroll
      for (int mm = 0; mm < D / 16; ++mm) acc[mm] = acc2[mm] = f32x4{0.f, 0.f, 0.f, 0.f};
    }
    if (d_live) {   // keep R-1 steps in flight: issue step k+R-1, then wait for step k
      issue(d, d_id, (k + R - 1) % R);
      d_live = advance(d);
      if (d_live) d_id = page_ids(d);
      wait_vmcnt<kDma * (R - 1)>();
    } else {
      wait_vmcnt<0>();
    }
    const int rs = k % R;
    const u4* const kbuf = &sm_ring[wave][rs][0];
    const char* const pbuf = reinterpret_cast<const char*>(&sm_ring[wave][rs][0]);
    const int nvalid = min(kStep, ntok - pi * kStep);

    // S^T = K q^T
    float sv[4 * KP];
#pragma unroll
    for (int t = 0; t < KP; ++t) {
      f32x4 s = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int c = 0; c < D / 32; ++c) s = mfma_qk(kbuf[t * kSlab + k_off + ((4 * c + rb) ^ k_swz(col))], qv[c], s);
#pragma unroll
      for (int i = 0; i < 4; ++i) sv[4 * t + i] = t * kPage + 4 * rb + i < nvalid ? s[i] : -INFINITY;
    }
    float mx = sv[0];
#pragma unroll
    for (int i = 1; i < 4 * KP; ++i) mx = fmaxf(mx, sv[i]);
    mx = swap32_max(swap16_max(mx));
    const bool raise = (mx - m) * cs > kSlack;
    if (__any(raise)) {
      const float m_new = raise ? mx : m;
      const float alpha = fast_exp2((m - m_new) * cs);   // 0 when m was -inf
      l *= alpha;
      m = m_new;
#pragma unroll
      for (int mm = 0; mm < D / 16; ++mm) {
        acc[mm] *= alpha;
        if constexpr (KP == 2) acc2[mm] *= alpha;
      }
    }
    const float mcs = m * cs;
    s16x4 pb[KP], pm[KP], pl[KP];   // P as bf16, and (head_dim 64) the two parts that left
#pragma unroll
    for (int i = 0; i < 4 * KP; ++i) {
      const float pk = fast_exp2(fmaf(sv[i], cs, -mcs));
      if constexpr (KP == 1) {
        l += pk;
        pb[i / 4][i % 4] = (short)f32_to_bf16(pk);
      } else {
        // three parts of 8 bits, cut and not rounded: their sum is p.  No part
        // of a p > 0 is 0, so that none makes NaN of an infinite V: a part
        // below the smallest normal number becomes that (p itself is 0 below
        // it), an error of 2^-126 at most
        const uint32_t tiny = __float_as_uint(fminf(pk, 0x1p-126f));
        const uint32_t hi = __float_as_uint(pk) & 0xffff0000u;
        const float r1 = pk - __uint_as_float(hi);
        const uint32_t mid = __float_as_uint(r1) & 0xffff0000u;
        const uint32_t lo = __float_as_uint(r1 - __uint_as_float(mid));
        pb[i / 4][i % 4] = (short)(hi >> 16);
        pm[i / 4][i % 4] = (short)(max(mid, tiny) >> 16);   // as integers: the parts are not negative
        pl[i / 4][i % 4] = (short)(max(lo, tiny) >> 16);
        sv[i] = pk;
      }
    }
    if constexpr (KP == 2) l += ((sv[0] + sv[1]) + (sv[2] + sv[3])) + ((sv[4] + sv[5]) + (sv[6] + sv[7]));
    // O^T += V^T P^T
    const bool partial = nvalid < kStep;
#pragma unroll
    for (int mm = 0; mm < D / 16; ++mm) {
      s16x4 a[KP];
#pragma unroll
      for (int t = 0; t < KP; ++t) {
        a[t] = lds_read_tr16(pbuf + v_off + t * (kSlab * 16) + ((mm ^ v_x) << 5));
        if (partial) {   // rows past the retained length may hold anything
#pragma unroll
          for (int j = 0; j < 4; ++j)
            if (t * kPage + 4 * rb + j >= nvalid) a[t][j] = 0;
        }
      }
      if constexpr (KP == 1) {
        acc[mm] = mfma_pv(a[0], pb[0], acc[mm]);
      } else {
        const u4 v = join(a[0], a[1]);
        acc[mm] = mfma_qk(v, join(pb[0], pb[1]), acc[mm]);
        acc2[mm] = mfma_qk(v, join(pm[0], pm[1]), acc2[mm]);   // apart: one rounding of acc a step
        acc2[mm] = mfma_qk(v, join(pl[0], pl[1]), acc2[mm]);
      }
    }
    ++k;
    if (++pi < ns) continue;

    if (arow >= 0) {
      // the new token becomes entry arow of the cache: its rows are in this
      // step's LDS buffer (refilled only by the next issue), CPR lanes for K
      // and CPR for V, stored with ordinary vector stores, which the DMA waits
      // above only count as extra (later) operations
      const int r = arow % kPage;
      const int64_t pg = (int64_t)pt[item.pt_base + arow / kPage] * p.page_chunks;
      if (lane < 2 * CPR) {
        const int ch = lane % CPR;
        const bool is_k = lane < CPR;
        const int row = ((arow - item.tok_begin) % kStep) * CPR;   // of the step
        const u4 v = is_k ? kbuf[row + (ch ^ k_swz(r))] : kbuf[256 + row + (ch ^ v_swz(r))];
        p.pool_w[pg + (is_k ? item.slot : p.heads_per_group + item.slot) * kSlab + r * CPR + ch] = v;
      }
      if (lane == 0) p.live_w[(int64_t)item.b * p.live_stride + item.kv_head] = arow + 1;
    } else if (arow == -2 && lane == 0 && p.append_full) {
      *p.append_full = 1;
    }

    // item end: the head's sum over all 16 token rows, then normalise and store
    l = swap32_sum(swap16_sum(l));
    if (col < G) {
      const float lse_nat = m * p.scale + logf(l);
      const float inv = 1.f / l;
      if constexpr (KP == 2) {
#pragma unroll
        for (int mm = 0; mm < D / 16; ++mm) acc[mm] += acc2[mm];
      }
      const int qh = item.kv_head * G + col;
      if (item.out_idx < 0) {
        uint2* orow = reinterpret_cast<uint2*>(static_cast<uint16_t*>(p.out) +
                                               ((int64_t)item.b * p.num_q_heads + qh) * D + 4 * rb);
#pragma unroll
        for (int mm = 0; mm < D / 16; ++mm) {
          const f32x4 o = acc[mm] * inv;
          orow[mm * 4] = make_uint2(uint32_t(f32_to_bf16(o[0])) | (uint32_t(f32_to_bf16(o[1])) << 16),
                                    uint32_t(f32_to_bf16(o[2])) | (uint32_t(f32_to_bf16(o[3])) << 16));
        }
        if (p.lse && rb == 0) p.lse[(int64_t)item.b * p.num_q_heads + qh] = lse_nat;
      } else if (D == 128 && p.merge_counters) {
        // read in this launch by whichever worker merges the unit, maybe on
        // another XCD: device-scope stores, written through to where every
        // XCD's device-scope loads read
        uint64_t* prow = reinterpret_cast<uint64_t*>(p.part_o + ((int64_t)item.out_idx * G + col) * D + 4 * rb);
#pragma unroll
        for (int mm = 0; mm < D / 16; ++mm) {
          const f32x4 o = acc[mm] * inv;
          __hip_atomic_store(prow + mm * 8, pack_f32x2(o[0], o[1]), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
          __hip_atomic_store(prow + mm * 8 + 1, pack_f32x2(o[2], o[3]), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
        if (rb == 0)
          __hip_atomic_store(p.part_lse + (int64_t)item.out_idx * G + col, lse_nat, __ATOMIC_RELAXED,
                             __HIP_MEMORY_SCOPE_AGENT);
      } else {
        f32x4* prow = reinterpret_cast<f32x4*>(p.part_o + ((int64_t)item.out_idx * G + col) * D + 4 * rb);
#pragma unroll
        for (int mm = 0; mm < D / 16; ++mm) prow[mm * 4] = acc[mm] * inv;
        if (rb == 0) p.part_lse[(int64_t)item.out_idx * G + col] = lse_nat;
      }
    }
    pi = 0;
    if (++it == it_end) break;
  }
  wait_vmcnt<0>();   // every page and every partial of this worker is complete

  // In-launch log-sum-exp merge (split-KV decoding, Section 2.2.3).  Each split
  // piece this worker ran counts itself on its unit's arrival counter; the
  // piece that arrives last merges the unit's partials and resets the counter
  // for the next call.  The partials were written with device-scope stores and
  // are complete (the wait above) before the worker's increments; the merging
  // worker reads them with device-scope loads issued after its increment
  // returned.  This is the ordering a release/acquire pair gives for data
  // written and read by device-scope atomics, without the writeback and
  // invalidation of a whole L2 that a fence for ordinary data needs.
  if constexpr (D == 128) if (p.merge_counters) {
    const TG_CONST int32_t* const unit_splits = (const TG_CONST int32_t*)p.unit_splits;
    const TG_CONST int32_t* const unit_base = (const TG_CONST int32_t*)p.unit_partial_base;
    // the split items of the bin, up to kBatch at a time: all their arrivals
    // go out before the first result is waited for, so a worker pays one
    // round trip for them, not one per item
    constexpr int kBatch = 4;
    int it2 = it_begin;
    while (it2 < it_end) {
      int su[kBatch], nb = 0;   // item indices of this batch's split items
      for (; it2 < it_end && nb < kBatch; ++it2)
        if (items[it2].out_idx >= 0) su[nb++] = it2;
      if (nb == 0) break;
      int arrived[kBatch];
#pragma unroll
      for (int j = 0; j < kBatch; ++j) {
        arrived[j] = 0;
        if (j < nb && lane == 0) {
          const int u = items[su[j]].b * p.num_kv_heads + items[su[j]].kv_head;
          arrived[j] = __hip_atomic_fetch_add(p.merge_counters + u, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
      }
#pragma unroll
      for (int j = 0; j < kBatch; ++j) {
        if (j >= nb) break;
        const int b = items[su[j]].b, h = items[su[j]].kv_head;
        const int u = b * p.num_kv_heads + h;
        const int s = unit_splits[u], base = unit_base[u];
        if (__builtin_amdgcn_readfirstlane(arrived[j]) != s - 1) continue;
        if (col < G) {
          float mr = -INFINITY, L = 0.f;
          f32x4 A[8];
#pragma unroll
          for (int mm = 0; mm < 8; ++mm) A[mm] = f32x4{0.f, 0.f, 0.f, 0.f};
          // up to kSplitBatch partials are requested before the first is
          // used: one round trip for a unit of that many splits (indices past
          // the last re-read it, and selects discard their steps)
          constexpr int kSplitBatch = 4;
          for (int i0 = 0; i0 < s; i0 += kSplitBatch) {
            float lv[kSplitBatch];
            f32x4 ov[kSplitBatch][8];
#pragma unroll
            for (int jj = 0; jj < kSplitBatch; ++jj) {
              const int64_t pidx = (int64_t)base + min(i0 + jj, s - 1);
              lv[jj] = __hip_atomic_load(p.part_lse + pidx * G + col, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
              const uint64_t* prow = reinterpret_cast<const uint64_t*>(p.part_o + (pidx * G + col) * D + 4 * rb);
#pragma unroll
              for (int mm = 0; mm < 8; ++mm) {
                const uint64_t lo = __hip_atomic_load(prow + mm * 8, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                const uint64_t hi = __hip_atomic_load(prow + mm * 8 + 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                ov[jj][mm] = f32x4{__uint_as_float((uint32_t)lo), __uint_as_float((uint32_t)(lo >> 32)),
                                   __uint_as_float((uint32_t)hi), __uint_as_float((uint32_t)(hi >> 32))};
              }
            }
            // the same running-max recurrence, in the same order, as tg_merge_kernel
#pragma unroll
            for (int jj = 0; jj < kSplitBatch; ++jj) {
              const bool use = i0 + jj < s;
              const float mn = fmaxf(mr, lv[jj]);
              const float a = __expf(mr - mn), w = __expf(lv[jj] - mn);
              const float Ln = fmaf(L, a, w);
#pragma unroll
              for (int mm = 0; mm < 8; ++mm)
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                  const float An = fmaf(A[mm][q], a, w * ov[jj][mm][q]);
                  A[mm][q] = use ? An : A[mm][q];
                }
              L = use ? Ln : L;
              mr = use ? mn : mr;
            }
          }
          const int qh = h * G + col;
          uint2* orow =
              reinterpret_cast<uint2*>(static_cast<uint16_t*>(p.out) + ((int64_t)b * p.num_q_heads + qh) * D + 4 * rb);
#pragma unroll
          for (int mm = 0; mm < 8; ++mm)
            orow[mm * 4] =
                make_uint2(uint32_t(f32_to_bf16(A[mm][0] / L)) | (uint32_t(f32_to_bf16(A[mm][1] / L)) << 16),
                           uint32_t(f32_to_bf16(A[mm][2] / L)) | (uint32_t(f32_to_bf16(A[mm][3] / L)) << 16));
          if (p.lse && rb == 0) p.lse[(int64_t)b * p.num_q_heads + qh] = mr + logf(L);
        }
        if (lane == 0) __hip_atomic_store(p.merge_counters + u, 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      }
    }
  }
  if (p.timestamps && lane == 0) {   // one lane, vector stores
    p.timestamps[2 * bin] = t_start;
    p.timestamps[2 * bin + 1] = __builtin_amdgcn_s_memrealtime();
  }
}

// ---------------------------------------------------------------------------
// fp32, head_dim D = 64 or 128, any gqa G in 1..16: the fp32 matrix
// instructions, pages straight from HBM into registers.
//
// A workgroup runs one bin.  The pages of an item are dealt round-robin to its
// 4 waves; every wave keeps its own online-softmax state, merged through LDS at
// the end of the item.
//
// An fp32 operand lane holds one value per product, so any order of the
// contraction index will do as long as both operands use it, and the lane that
// loads 16 consecutive bytes feeds four products from them without LDS:
//   * S^T[16 tok][16 heads] = K q^T: D/4 x v_mfma_f32_16x16x4_f32; lane (col, rb)
//     = (lane % 16, lane / 16) holds dims 16c + 4rb + i of token col (and of
//     head col for q) for product (c, i);
//   * O^T[dims][16 heads] += V^T P^T: product (i, m, j) contracts tokens 4rb + i
//     for dims 64m + 4col + j: the lane's own S^T value i is the B operand, and
//     float j of its 16-byte load at dims 64m + 4col of token 4rb + i the A
//     operand.  The result lane holds dims 64m + 16rb + 4r + j, so j = 0..3 are
//     again 16 bytes.
// K's registers are reloaded for the wave's next page as soon as q.k has read
// them, V's after p.v, so a page is always in flight; page ids are read a page
// ahead.  The reloads are unconditional (a wave's last page is read once more,
// from cache): behind a branch the compiler would have to wait for every load
// in flight before each product (a unit per bin: 168 -> 128 us at head_dim 64).
// Bound by HBM; the 64 products of a page at head_dim 128 take about 1 us of
// the 5 a page is given then.  16 requests, gqa 4, 223 MB: 41 us, 5.4 TB/s,
// against 50 on the vector kernel; gqa 16, 134 MB: 97 -> 36 us with the merge.
// The non-temporal loads pay past the 256 MB the caches hold (gqa 4, 582 MB: 104
// us, plain 112; 792 MB at head_dim 64: 132, plain 145) and cost repeated
// passes over less (198 MB: 42, plain 38; after the caches were replaced both
// 45).  Loading an item's queries while the item before runs, into a second
// buffer, measured slower at 64 (14.2 -> 15.8 us at 31 MB) and level at 128.
template <int D>
__global__ void __launch_bounds__(kBlock, 2) tg_decode_f32_kernel(DecodeParams p, const tg_work_item* __restrict__ items_g,
                                                                 const int32_t* __restrict__ pt_g,
                                                                 const int32_t* __restrict__ bin_offsets_g,
                                                                 const u4* __restrict__ pool_g) {
  static_assert(D == 64 || D == 128, "head_dim 64 or 128");
  constexpr int CPR = D / 4;             // 16-byte chunks per row
  constexpr int kSlab = kPage * CPR;     // chunks per K or V slab of a page
  constexpr int NC = D / 16;             // 16-dim groups of q.k
  constexpr int NM = D / 64;             // 64-dim groups of p.v
  constexpr int kAcc = D == 64 ? 4 : 2;  // accumulators a wave's tokens are dealt to
  constexpr float kSlack = 8.0f;

  __shared__ f32x4 sm_acc[kWaves][16][CPR + 1];   // padded: the rows of different heads on different banks
  __shared__ f32x4 sm_q[16][CPR + 1];
  __shared__ float sm_m[kWaves][16], sm_l[kWaves][16];

  const TG_CONST tg_work_item* const items = (const TG_CONST tg_work_item*)items_g;
  const TG_CONST int32_t* const pt = (const TG_CONST int32_t*)pt_g;
  const TG_CONST int32_t* const bin_offsets = (const TG_CONST int32_t*)bin_offsets_g;
  const f32x4* const pool = reinterpret_cast<const f32x4*>(pool_g);

  const int lane = threadIdx.x & 63;
  const int wave = wave_id();
  const int G = p.gqa;
  const int col = lane & 15;
  const int rb = lane >> 4;
  const int hq = col < G ? col : col % G;   // columns past G repeat a real head and are never stored
  const int it_begin = bin_offsets[blockIdx.x], it_end = bin_offsets[blockIdx.x + 1];
  const float cs = p.scale_log2;
  const uint64_t t_start = __builtin_amdgcn_s_memrealtime();

  // load cursor over the pages of the bin that are this wave's
  struct Cursor {
    int it, pi, np, slot, arow;
    int64_t pbase;
  };
  auto enter = [&](Cursor& cu, int it) {   // the wave's first page at or after item it; false (cursor unchanged) if none
    for (; it < it_end; ++it) {
      int arow;
      const tg_work_item im = load_item(items + it, p, &arow);
      const int np = (im.tok_end - im.tok_begin + kPage - 1) / kPage;
      if (wave >= np) continue;
      cu.it = it;
      cu.pi = wave;
      cu.np = np;
      cu.slot = im.slot;
      cu.arow = arow >= 0 ? arow % kPage : -1;   // row of the last page that takes the new token
      cu.pbase = im.pt_base + im.tok_begin / kPage;
      return true;
    }
    return false;
  };
  auto advance = [&](Cursor& cu) {   // stays on the wave's last page
    if (cu.pi + kWaves < cu.np)
      cu.pi += kWaves;
    else
      enter(cu, cu.it + 1);
  };
  // every cached row is read once: non-temporal loads
  f32x4 kc[NC], vc[4][NM];
  auto load_k = [&](const Cursor& cu, int32_t id) {
    const bool takes_token = cu.arow >= 0 && cu.pi == cu.np - 1;
    const f32x4* tok = nullptr;
    if (takes_token)
      tok = reinterpret_cast<const f32x4*>(p.append_k) +
            ((int64_t)items[cu.it].b * p.num_kv_heads + items[cu.it].kv_head) * CPR + rb;
    const f32x4* src = pool + (int64_t)id * p.page_chunks + cu.slot * kSlab + col * CPR + rb;
    if (takes_token && col == cu.arow) src = tok;
#pragma unroll
    for (int c = 0; c < NC; ++c) kc[c] = __builtin_nontemporal_load(src + 4 * c);
  };
  auto load_v = [&](const Cursor& cu, int32_t id) {
    const bool takes_token = cu.arow >= 0 && cu.pi == cu.np - 1;
    const f32x4* tok = nullptr;
    if (takes_token)
      tok = reinterpret_cast<const f32x4*>(p.append_v) +
            ((int64_t)items[cu.it].b * p.num_kv_heads + items[cu.it].kv_head) * CPR + col;
    const f32x4* src = pool + (int64_t)id * p.page_chunks + (p.heads_per_group + cu.slot) * kSlab + 4 * rb * CPR + col;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const f32x4* row = takes_token && 4 * rb + i == cu.arow ? tok : src + i * CPR;
#pragma unroll
      for (int m = 0; m < NM; ++m) vc[i][m] = __builtin_nontemporal_load(row + 16 * m);
    }
  };

  Cursor d = {};
  int32_t d_id = 0;
  if (enter(d, it_begin)) {   // a wave without a page loads nothing and meets the others at the barriers
    d_id = pt[d.pbase + d.pi];
    load_k(d, d_id);
    load_v(d, d_id);
    advance(d);
    d_id = pt[d.pbase + d.pi];
  }

  for (int it = it_begin; it < it_end; ++it) {
    int arow;   // entry that takes the appended token, or < 0
    const tg_work_item item = load_item(items + it, p, &arow);
    const int ntok = item.tok_end - item.tok_begin;
    const int np = (ntok + kPage - 1) / kPage;
    {   // the item's queries through LDS: in registers they would cost a wave its second accumulator
      const f32x4* qrow = reinterpret_cast<const f32x4*>(p.q) +
                          ((int64_t)item.b * p.num_q_heads + item.kv_head * G) * CPR;
      for (int o = threadIdx.x; o < G * CPR; o += kBlock) sm_q[o / CPR][o % CPR] = qrow[o];
      __syncthreads();
    }
    const f32x4* const qv = &sm_q[hq][rb];
    float m = -INFINITY, l = 0.f;
    // added at the item's end, for short chains of roundings: as many as the
    // vector kernel has, 16 in a workgroup at head_dim 64 and 8 at 128, where
    // four a wave would not fit the registers.  With two at 64, long units were
    // up to 1.13 times further from 64 bits than there; now 0.98 over the range
    // (1.05 at most), for 0.3 us of 13 in short batches, none in long ones
    f32x4 acc[kAcc][NM][4];
#pragma unroll
    for (int e = 0; e < kAcc; ++e)
#pragma unroll
      for (int mm = 0; mm < NM; ++mm)
#pragma unroll
        for (int j = 0; j < 4; ++j) acc[e][mm][j] = f32x4{0.f, 0.f, 0.f, 0.f};

    for (int pi = wave; pi < np; pi += kWaves) {
      const int nvalid = min(kPage, ntok - pi * kPage);
      // S^T = K q^T: sums over 8 dims, then a tree: few rounding steps in a row
      f32x4 s[NC];
#pragma unroll
      for (int c = 0; c < NC; ++c) {
        const f32x4 q = qv[4 * c];
        f32x4 a = {0.f, 0.f, 0.f, 0.f}, b = a;
#pragma unroll
        for (int i = 0; i < 2; ++i) {
          a = __builtin_amdgcn_mfma_f32_16x16x4f32(kc[c][i], q[i], a, 0, 0, 0);
          b = __builtin_amdgcn_mfma_f32_16x16x4f32(kc[c][i + 2], q[i + 2], b, 0, 0, 0);
        }
        s[c] = a + b;
        if (c % 2 == 1) {
          s[c - 1] += s[c];
          __builtin_amdgcn_sched_barrier(0);   // at most two groups' sums at once: registers
        }
      }
#pragma unroll
      for (int n = 2; n < NC; n *= 2)
#pragma unroll
        for (int c = 0; c < NC; c += 2 * n) s[c] += s[c + n];
      load_k(d, d_id);
      float sv[4];
#pragma unroll
      for (int i = 0; i < 4; ++i) sv[i] = 4 * rb + i < nvalid ? s[0][i] : -INFINITY;
      float mx = fmaxf(fmaxf(sv[0], sv[1]), fmaxf(sv[2], sv[3]));
      mx = swap32_max(swap16_max(mx));
      const bool raise = (mx - m) * cs > kSlack;   // rescale only when it matters: p <= 2^8
      if (__any(raise)) {
        const float m_new = raise ? mx : m;
        const float alpha = fast_exp2((m - m_new) * cs);   // 0 when m was -inf
        l *= alpha;
        m = m_new;
#pragma unroll
        for (int mm = 0; mm < NM; ++mm)
#pragma unroll
          for (int j = 0; j < 4; ++j)
#pragma unroll
            for (int e = 0; e < kAcc; ++e) acc[e][mm][j] *= alpha;
      }
      // relative to m itself, not to a rounded m * cs: the state's m is what
      // the waves' and the pieces' states are weighted by
#pragma unroll
      for (int i = 0; i < 4; ++i) sv[i] = fast_exp2((sv[i] - m) * cs);
      l += (sv[0] + sv[1]) + (sv[2] + sv[3]);   // one rounding step a page in the long sum
      // O^T += V^T P^T
      const bool partial = nvalid < kPage;
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        if (partial && 4 * rb + i >= nvalid) {   // rows past the retained length may hold anything
#pragma unroll
          for (int mm = 0; mm < NM; ++mm) vc[i][mm] = f32x4{0.f, 0.f, 0.f, 0.f};
        }
#pragma unroll
        for (int mm = 0; mm < NM; ++mm)
#pragma unroll
          for (int j = 0; j < 4; ++j)
            acc[i % kAcc][mm][j] =
                __builtin_amdgcn_mfma_f32_16x16x4f32(vc[i][mm][j], sv[i], acc[i % kAcc][mm][j], 0, 0, 0);
      }
      load_v(d, d_id);
      advance(d);
      d_id = pt[d.pbase + d.pi];
    }

    // item end: the waves' states through LDS (a wave that saw no row has m =
    // -inf and weight 0), then the output or this piece's partial
    l = swap32_sum(swap16_sum(l));
    if (col < G) {
#pragma unroll
      for (int mm = 0; mm < NM; ++mm) {
        if constexpr (kAcc == 4) {
#pragma unroll
          for (int j = 0; j < 4; ++j) {
            acc[0][mm][j] += acc[2][mm][j];
            acc[1][mm][j] += acc[3][mm][j];
          }
        }
#pragma unroll
        for (int r = 0; r < 4; ++r)
          sm_acc[wave][col][16 * mm + 4 * rb + r] =
              f32x4{acc[0][mm][0][r] + acc[1][mm][0][r], acc[0][mm][1][r] + acc[1][mm][1][r],
                    acc[0][mm][2][r] + acc[1][mm][2][r], acc[0][mm][3][r] + acc[1][mm][3][r]};
      }
      if (rb == 0) {
        sm_m[wave][col] = m;
        sm_l[wave][col] = l;
      }
    }
    __syncthreads();
    for (int o = threadIdx.x; o < G * CPR; o += kBlock) {
      const int g = o / CPR, c = o % CPR;
      float M = sm_m[0][g];
#pragma unroll
      for (int w = 1; w < kWaves; ++w) M = fmaxf(M, sm_m[w][g]);
      float L = 0.f;
      f32x4 A = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int w = 0; w < kWaves; ++w) {
        const float f = fast_exp2((sm_m[w][g] - M) * cs);
        L = fmaf(sm_l[w][g], f, L);
#pragma unroll
        for (int q = 0; q < 4; ++q) A[q] = fmaf(sm_acc[w][g][c][q], f, A[q]);
      }
      const f32x4 O = {A[0] / L, A[1] / L, A[2] / L, A[3] / L};
      const int64_t row = item.out_idx < 0 ? (int64_t)item.b * p.num_q_heads + item.kv_head * G + g
                                           : (int64_t)item.out_idx * G + g;
      reinterpret_cast<f32x4*>(item.out_idx < 0 ? static_cast<float*>(p.out) : p.part_o)[row * CPR + c] = O;
      float* lse = item.out_idx < 0 ? p.lse : p.part_lse;
      if (lse && c == 0) lse[row] = M * p.scale + logf(L);
    }
    if (arow >= 0) {   // the token becomes entry arow of the cache; every wave read the length above
      if (threadIdx.x < 2 * CPR) {
        const bool is_k = threadIdx.x < CPR;
        const int ch = threadIdx.x % CPR;
        const int64_t toff = ((int64_t)item.b * p.num_kv_heads + item.kv_head) * CPR;
        const int64_t pg = (int64_t)pt[item.pt_base + arow / kPage] * p.page_chunks;
        p.pool_w[pg + (is_k ? item.slot : p.heads_per_group + item.slot) * kSlab + (arow % kPage) * CPR + ch] =
            is_k ? p.append_k[toff + ch] : p.append_v[toff + ch];
      }
      if (threadIdx.x == 0) p.live_w[(int64_t)item.b * p.live_stride + item.kv_head] = arow + 1;
    } else if (arow == -2 && threadIdx.x == 0 && p.append_full) {
      *p.append_full = 1;
    }
    __syncthreads();   // the states may be overwritten
  }
  if (p.timestamps && threadIdx.x == 0) {   // one lane, vector stores
    p.timestamps[2 * blockIdx.x] = t_start;
    p.timestamps[2 * blockIdx.x + 1] = __builtin_amdgcn_s_memrealtime();
  }
}

// ---------------------------------------------------------------------------
// Log-sum-exp merge of the split partials of every unit (b, h) with more than
// one split: lse* = log sum_i e^{lse_i}, O = sum_i e^{lse_i - lse*} o_i.
// Grid (units, ceil(gqa*D / 1024)): each thread owns four consecutive output
// elements (16-byte partial loads) and makes a single pass with a running
// max, so the loads of consecutive splits are independent and issue back to
// back.
template <typename T, int D>
__global__ void __launch_bounds__(kBlock) tg_merge_kernel(const int32_t* __restrict__ unit_splits,
                                                         const int32_t* __restrict__ unit_base,
                                                         const float* __restrict__ part_o,
                                                         const float* __restrict__ part_lse, void* out, float* lse,
                                                         int32_t num_kv_heads, int32_t gqa) {
  const int u = blockIdx.x;
  const int s = unit_splits[u];
  const int base = unit_base[u];
  // both reads in flight together, before the exit test (the compiler would
  // otherwise sink the second behind it: two round trips instead of one)
  asm volatile("" ::"s"(s), "s"(base));
  const int o = (blockIdx.y * kBlock + threadIdx.x) * 4;
  if (s <= 1 || o >= gqa * D) return;
  const int b = u / num_kv_heads, h = u % num_kv_heads;
  const int64_t row0 = (int64_t)b * num_kv_heads * gqa + (int64_t)h * gqa;
  const int g = o / D, e = o % D;   // D is a multiple of 4: the four outputs share g
  const float* pl = part_lse + (int64_t)base * gqa + g;
  const f32x4* po = reinterpret_cast<const f32x4*>(part_o + ((int64_t)base * gqa + g) * D + e);
  float m = -INFINITY, L = 0.f;
  f32x4 A = {0.f, 0.f, 0.f, 0.f};
  // kBatch splits' loads go out before the first is used, so a unit of up to
  // kBatch splits pays one memory round trip, not one per split.  Indices past
  // the last split re-read it; their steps are computed and then discarded by
  // selects (a branch would let the compiler sink the loads behind it).
  constexpr int kBatch = 4;
  for (int i0 = 0; i0 < s; i0 += kBatch) {
    float lv[kBatch];
    f32x4 ov[kBatch];
#pragma unroll
    for (int j = 0; j < kBatch; ++j) {
      const int64_t i = min(i0 + j, s - 1);
      lv[j] = pl[i * gqa];
      ov[j] = po[i * gqa * (D / 4)];
    }
#pragma unroll
    for (int j = 0; j < kBatch; ++j) {
      const bool use = i0 + j < s;
      const float mn = fmaxf(m, lv[j]);
      const float a = __expf(m - mn), w = __expf(lv[j] - mn);
      const float Ln = fmaf(L, a, w);
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const float An = fmaf(A[q], a, w * ov[j][q]);
        A[q] = use ? An : A[q];
      }
      L = use ? Ln : L;
      m = use ? mn : m;
    }
  }
  store_out4<T>(static_cast<T*>(out) + (row0 + g) * D + e, A[0] / L, A[1] / L, A[2] / L, A[3] / L);
  if (lse && e == 0) lse[row0 + g] = m + logf(L);
}

// The same merge for units cut into many pieces: W chains per unit and head,
// chain w taking pieces w, w + W, ... with the recurrence above, then the
// chains combined in order at the largest of their maxima.  One workgroup per
// (unit, head): D/4 threads per chain, four outputs each.
// What bounds the single chain is latency: it pays a memory round trip per
// kBatch pieces, and one request's long context on 1024 workers leaves units
// of hundreds of pieces on a handful of workgroups.  Measured (gqa 8, head_dim
// 128, 8 units with 1027 pieces, at most 368 per unit): 44 us in one chain,
// 14, 8.1, 5.6 and 5.8 us in 4, 8, 16 and 32.
template <typename T, int D, int W>
__global__ void __launch_bounds__(D / 4 * W) tg_merge_chains_kernel(
    const int32_t* __restrict__ unit_splits, const int32_t* __restrict__ unit_base, const float* __restrict__ part_o,
    const float* __restrict__ part_lse, void* out, float* lse, int32_t num_kv_heads, int32_t gqa) {
  constexpr int kTpc = D / 4;   // threads per chain
  __shared__ f32x4 sm_A[W][kTpc];
  __shared__ float sm_m[W], sm_L[W];
  const int u = blockIdx.x, g = blockIdx.y;
  const int s = unit_splits[u];
  const int base = unit_base[u];
  asm volatile("" ::"s"(s), "s"(base));   // both reads in flight before the exit test
  if (s <= 1) return;
  const int t = threadIdx.x % kTpc, w = threadIdx.x / kTpc;
  const float* pl = part_lse + (int64_t)base * gqa + g;
  const f32x4* po = reinterpret_cast<const f32x4*>(part_o + ((int64_t)base * gqa + g) * D) + t;
  float m = -INFINITY, L = 0.f;
  f32x4 A = {0.f, 0.f, 0.f, 0.f};
  constexpr int kBatch = 4;
  for (int i0 = w; i0 < s; i0 += kBatch * W) {
    float lv[kBatch];
    f32x4 ov[kBatch];
#pragma unroll
    for (int j = 0; j < kBatch; ++j) {
      const int64_t i = min(i0 + j * W, s - 1);
      lv[j] = pl[i * gqa];
      ov[j] = po[i * gqa * kTpc];
    }
#pragma unroll
    for (int j = 0; j < kBatch; ++j) {
      const bool use = i0 + j * W < s;
      const float mn = fmaxf(m, lv[j]);
      const float a = __expf(m - mn), wt = __expf(lv[j] - mn);
      const float Ln = fmaf(L, a, wt);
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const float An = fmaf(A[q], a, wt * ov[j][q]);
        A[q] = use ? An : A[q];
      }
      L = use ? Ln : L;
      m = use ? mn : m;
    }
  }
  sm_A[w][t] = A;
  if (t == 0) {
    sm_m[w] = m;
    sm_L[w] = L;
  }
  __syncthreads();
  if (w > 0) return;
  const int n = min(W, s);   // chains that hold a piece
  float M = -INFINITY;
  for (int c = 0; c < n; ++c) M = fmaxf(M, sm_m[c]);
  L = 0.f;
  A = f32x4{0.f, 0.f, 0.f, 0.f};
  for (int c = 0; c < n; ++c) {
    const float f = __expf(sm_m[c] - M);
    const f32x4 Ac = sm_A[c][t];
    L = fmaf(sm_L[c], f, L);
#pragma unroll
    for (int q = 0; q < 4; ++q) A[q] = fmaf(Ac[q], f, A[q]);
  }
  const int b = u / num_kv_heads, h = u % num_kv_heads;
  const int64_t row = (int64_t)b * num_kv_heads * gqa + (int64_t)h * gqa + g;
  store_out4<T>(static_cast<T*>(out) + row * D + 4 * t, A[0] / L, A[1] / L, A[2] / L, A[3] / L);
  if (lse && t == 0) lse[row] = M + logf(L);
}

using MergeFn = void (*)(const int32_t*, const int32_t*, const float*, const float*, void*, float*, int32_t,
                         int32_t);

// Chains a unit's partials are merged in, by the plan's pieces per unit (the
// lengths are ragged: the longest units hold about three times the mean).
// Measured, one chain against 16 (gqa 4 unless said): 6.3 pieces per unit (192
// units) 4.8 against 4.7 us, 6.9 (128 units, f32) 6.9 against 4.8, 17 (64
// units) 7.4 against 4.6, 33 (32 units, gqa 8) 13.2 against 3.9; with 5 per
// unit (256 units, gqa 8) the 16 chains' workgroups cost more than the round
// trips they save, 6.0 against 4.7.  8 chains are level with 16 up to 17
// pieces and behind above; 32 are never ahead by more than 0.7 us.
constexpr int kMergeLanes = 16;
int merge_lanes(int64_t num_partials, int64_t units) { return num_partials < 6 * units ? 1 : kMergeLanes; }

template <typename T, int D>
MergeFn pick_merge_lanes(int lanes) {
  return lanes == 1 ? &tg_merge_kernel<T, D> : &tg_merge_chains_kernel<T, D, kMergeLanes>;
}

MergeFn pick_merge(int dtype, int d, int lanes) {
  if (dtype == TG_F32 && d == 64) return pick_merge_lanes<float, 64>(lanes);
  if (dtype == TG_F32 && d == 128) return pick_merge_lanes<float, 128>(lanes);
  if (dtype == TG_BF16 && d == 64) return pick_merge_lanes<uint16_t, 64>(lanes);
  if (dtype == TG_BF16 && d == 128) return pick_merge_lanes<uint16_t, 128>(lanes);
  return nullptr;
}

using DecodeFn = void (*)(DecodeParams, const tg_work_item*, const int32_t*, const int32_t*, const u4*);

constexpr int kMaxGqa = 16;

// Where the vector kernel runs.  With few query heads the matrix kernels' 16
// columns stay mostly empty and their few, large workgroups wait longer for
// each item's queries, barriers and rounds than the vector kernel's many small
// ones; there it runs at any number of bins, each plan at the bins its own
// occupancy gives (8 KV heads, vector against matrix kernel, repeated passes /
// after the caches were replaced, us):
//   f32 gqa 1, 64 requests of 200 to 1000 tokens: head_dim 64 17 / 22 against
//     21 / 26, 128 23 / 29 against 31 / 36; gqa 3 19 / 24 against 21 / 26 and
//     29 / 36 against 32 / 38; 12 of 2000 to 8000 tokens, 128: gqa 1 35 / 44
//     against 42 / 45, gqa 3 39 / 48 against 42 / 45.  At gqa 4 the matrix
//     kernel is ahead or level everywhere (32 / 38 against 31 / 37, 42 / 51
//     against 42 / 45).  Past the 256 MB the caches hold, it is ahead by 6 to
//     10 % at any gqa (582 MB, gqa 1: 110 against 103), which a plan does not
//     show on the host.
//   bf16 head_dim 64, gqa 1: 64 requests of 200 to 1000 tokens 13.1 against 14.0
//     (19 against 19), 32 of 300 to 3000 11.6 against 15.0 (17 against 20);
//     396 MB 81 against 70.  With few requests level, but for one very long
//     context, whose more pieces the merge pays for (40000 tokens, 8 KV heads
//     14.5 against 13.1, 2 heads 19.4 against 14.4).
// Plans of few bins (one worker per unit, say) are bound by one worker, and
// four waves on a bin win at up to four heads: 128 bins of one unit each (16
// requests, 8192 tokens), bf16 head_dim 64, gqa 4 133 against 204 us, gqa 8 (64
// bins) 194 against 189; 256 bins of equal shares gqa 4 31 against 37, at 1024
// 26 against 19.
bool vector_kernel_pays(int dtype, int d, int gqa, int n_bins) {
  if (dtype == TG_F32) return gqa <= 3;
  return d == 64 && (gqa == 1 || (gqa <= 4 && n_bins <= 384));
}

template <typename T, int D>
DecodeFn pick_vector(int gqa) {
  if (gqa == 1) return &tg_decode_kernel<T, D, 1>;
  if (gqa == 2) return &tg_decode_kernel<T, D, 2>;
  if constexpr (sizeof(T) == 2) {
    if (gqa == 4) return &tg_decode_kernel<T, D, 4>;
  }
  return &tg_decode_kernel<T, D, 3>;
}

DecodeFn pick_decode(int dtype, int d, int gqa, int n_bins) {
  if (gqa < 1 || gqa > kMaxGqa) return nullptr;
  if (vector_kernel_pays(dtype, d, gqa, n_bins)) {
    if (dtype == TG_BF16) return pick_vector<uint16_t, 64>(gqa);
    return d == 64 ? pick_vector<float, 64>(gqa) : pick_vector<float, 128>(gqa);
  }
  if (dtype == TG_BF16 && d == 128) return gqa <= 8 ? &tg_decode_mfma_kernel<128, 8> : &tg_decode_mfma_kernel<128, 16>;
  if (dtype == TG_BF16 && d == 64) return gqa <= 8 ? &tg_decode_mfma_kernel<64, 8> : &tg_decode_mfma_kernel<64, 16>;
  if (dtype == TG_F32 && d == 64) return &tg_decode_f32_kernel<64>;
  if (dtype == TG_F32 && d == 128) return &tg_decode_f32_kernel<128>;
  return nullptr;
}

// whether every wave runs a bin of its own (the bf16 matrix kernel)
bool wave_per_bin(int dtype, int d, int gqa, int n_bins) {
  return dtype == TG_BF16 && !vector_kernel_pays(dtype, d, gqa, n_bins);
}

// Waves per workgroup of the bf16 kernel, each with a bin of its own.  Its LDS
// limits a CU to one workgroup of up to four waves, so plans of fewer bins than
// four per CU take fewer waves per workgroup and spread over more CUs: over all
// of them at multiples of 256 bins, over 129 to 255 between, where the time
// keeps falling with the bins (16 requests of 8192 tokens, gqa 4, 256 / 257 /
// 300 / 400 / 512 / 513 / 768 / 1024 bins: 62 / 63 / 54 / 43 / 36 / 36 / 29 / 29
// us at head_dim 128, 32 / 33 / 32 / 31 / 26 / 27 / 21 / 19 at 64).  256 bins in
// workgroups of four: 60.5 against 58.2 us at 128, 38.8 against 36.6 at 64.
int waves_per_wg(int n_bins) {
  constexpr int kCus = 256;
  const int w = n_bins / kCus + (n_bins % kCus != 0);
  return w < kWaves ? w : kWaves;
}

int bins_per_wg(int dtype, int d, int gqa, int n_bins) {
  return wave_per_bin(dtype, d, gqa, n_bins) ? waves_per_wg(n_bins) : 1;
}

int32_t check_decode_shape(const tg_geometry* g, int dtype) {
  if (int32_t rc = tg::check_geometry(g)) return rc;
  if (dtype != TG_F32 && dtype != TG_BF16) return tg::fail(TG_ERR_INVALID_ARG, "unknown dtype %d", dtype);
  if (g->page_size != kPage) return tg::fail(TG_ERR_UNSUPPORTED, "decode supports page_size 16 only (got %d)", g->page_size);
  if (g->head_dim != 64 && g->head_dim != 128)
    return tg::fail(TG_ERR_UNSUPPORTED, "decode supports head_dim 64 or 128 (got %d)", g->head_dim);
  const int gqa = g->num_q_heads / g->num_kv_heads;
  if (gqa < 1 || gqa > kMaxGqa) return tg::fail(TG_ERR_UNSUPPORTED, "decode supports 1..16 query heads per KV head");
  return TG_OK;
}

size_t align256(size_t x) { return (x + 255) & ~size_t(255); }

}  // namespace

// ---------------------------------------------------------------------------
// Static scratch of tg_decode_noalloc: the split partials of one call, for
// callers that cannot allocate device memory.  Every device the library runs
// on holds its own copy of this array until the process ends.  In host code
// `scratch` is only a stand-in symbol: its device address is looked up once
// per device (hipGetSymbolAddress, with that device current) and that address
// is what the kernels get.
static __device__ __align__(256) unsigned char scratch[TG_DECODE_NOALLOC_MAX_BYTES];

namespace {

constexpr int kMaxDevices = 64;
constexpr size_t kScratchCounters = 64 << 10;   // merge arrival counters: up to 16384 (request, KV head) units
std::mutex g_scratch_mu;
void* g_scratch_ptr[kMaxDevices] = {};

int32_t scratch_address(void** out) {
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess) return tg::fail(TG_ERR_HIP, "hipGetDevice failed");
  if (dev < 0 || dev >= kMaxDevices) return tg::fail(TG_ERR_UNSUPPORTED, "device %d: at most %d devices", dev, kMaxDevices);
  std::lock_guard<std::mutex> lock(g_scratch_mu);
  if (!g_scratch_ptr[dev]) {
    void* p = nullptr;
    const hipError_t e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
    if (e != hipSuccess || !p)
      return tg::fail(TG_ERR_HIP, "hipGetSymbolAddress(scratch) failed on device %d: %s", dev, hipGetErrorString(e));
    g_scratch_ptr[dev] = p;
  }
  *out = g_scratch_ptr[dev];
  return TG_OK;
}

// tg_decode with the partials' memory passed in: ws (ws_bytes bytes) stands for
// the caller's workspace.
int32_t decode_impl(const tg_decode_args* a, void* ws_ptr, size_t ws_bytes, void* hip_stream) {
  if (!a) return tg::fail(TG_ERR_INVALID_ARG, "args is NULL");
  if (int32_t rc = check_decode_shape(&a->geom, a->dtype)) return rc;
  const tg_geometry& g = a->geom;
  if (a->batch < 1 || a->n_bins < 1 || a->num_items < 0 || a->num_partials < 0)
    return tg::fail(TG_ERR_INVALID_ARG, "batch, n_bins must be >= 1; counts >= 0");
  if (!a->q || !a->kv_pool || !a->pt_pages || !a->items || !a->bin_offsets || !a->out)
    return tg::fail(TG_ERR_INVALID_ARG, "NULL device pointer");
  if (a->num_partials > 0 && (!a->unit_splits || !a->unit_partial_base))
    return tg::fail(TG_ERR_INVALID_ARG, "split plan needs unit_splits and unit_partial_base");
  const size_t need = tg_decode_workspace_bytes(&g, a->batch, a->num_partials);
  if (a->num_partials > 0 && (!ws_ptr || ws_bytes < need))
    return tg::fail(TG_ERR_BUFFER_TOO_SMALL, "workspace holds %zu bytes, need %zu", ws_bytes, need);
  if (!tg::aligned16({a->q, a->kv_pool, a->out, a->append_k, a->append_v, a->num_partials > 0 ? ws_ptr : nullptr}))
    return tg::fail(TG_ERR_INVALID_ARG, "device buffers must be 16-byte aligned");
  const int gqa = g.num_q_heads / g.num_kv_heads;
  const int esz = a->dtype == TG_F32 ? 4 : 2;
  const size_t o_bytes = align256((size_t)a->num_partials * gqa * g.head_dim * 4);
  char* ws = static_cast<char*>(ws_ptr);
  DecodeParams p;
  p.q = a->q;
  p.pool = static_cast<const u4*>(a->kv_pool);
  p.pt_pages = a->pt_pages;
  p.items = a->items;
  p.bin_offsets = a->bin_offsets;
  p.unit_splits = a->unit_splits;
  p.unit_partial_base = a->unit_partial_base;
  p.out = a->out;
  p.lse = a->lse;
  p.part_o = ws ? reinterpret_cast<float*>(ws) : nullptr;
  p.part_lse = ws ? reinterpret_cast<float*>(ws + o_bytes) : nullptr;
  p.page_chunks = (int64_t)g.heads_per_group * 2 * kPage * g.head_dim * esz / 16;
  p.heads_per_group = g.heads_per_group;
  p.num_q_heads = g.num_q_heads;
  p.num_kv_heads = g.num_kv_heads;
  p.n_bins = a->n_bins;
  p.gqa = gqa;
  p.timestamps = a->timestamps;
  if (a->live_len && (a->layer < 0 || a->layer >= g.num_layers))
    return tg::fail(TG_ERR_INVALID_ARG, "layer %d out of range", a->layer);
  p.live = a->live_len ? a->live_len + (int64_t)a->layer * g.num_kv_heads : nullptr;
  p.live_stride = g.num_layers * g.num_kv_heads;
  if ((a->append_k == nullptr) != (a->append_v == nullptr))
    return tg::fail(TG_ERR_INVALID_ARG, "append_k and append_v go together");
  if (a->append_k && !a->live_len) return tg::fail(TG_ERR_INVALID_ARG, "the in-launch append needs live_len");
  p.append_k = static_cast<const u4*>(a->append_k);
  p.append_v = static_cast<const u4*>(a->append_v);
  p.pool_w = static_cast<u4*>(a->kv_pool);
  p.live_w = a->append_k ? a->live_len + (int64_t)a->layer * g.num_kv_heads : nullptr;
  p.append_full = a->append_full;
  // the bf16 head_dim-128 kernel merges split units inside its launch when the
  // caller passes arrival counters and one chain is enough; every other case
  // merges in a second launch.  With several chains one wave would walk them
  // all: 24 requests of 2000 to 16000 tokens (6.2 pieces per unit) 92 us there,
  // 65 in one chain there, 53 with the second launch; 16 requests (8.9) 76, 52
  // and 36; one of 40000 tokens (129) 211, 158 and 17.
  const int lanes = merge_lanes(a->num_partials, (int64_t)a->batch * g.num_kv_heads);
  const bool fused_merge =
      a->merge_counters && a->num_partials > 0 && lanes == 1 && a->dtype == TG_BF16 && g.head_dim == 128;
  p.merge_counters = fused_merge ? a->merge_counters : nullptr;
  p.scale = a->sm_scale != 0.f ? a->sm_scale : 1.0f / std::sqrt((float)g.head_dim);
  p.scale_log2 = p.scale * kLog2e;
  if (a->num_items == 0) return TG_OK;
  hipStream_t st = static_cast<hipStream_t>(hip_stream);
  DecodeFn fn = pick_decode(a->dtype, g.head_dim, gqa, a->n_bins);
  const int bins = bins_per_wg(a->dtype, g.head_dim, gqa, a->n_bins);   // bins per workgroup
  const int waves = wave_per_bin(a->dtype, g.head_dim, gqa, a->n_bins) ? bins : kWaves;
  hipLaunchKernelGGL(fn, dim3((a->n_bins + bins - 1) / bins), dim3(64 * waves), 0, st, p, a->items, a->pt_pages,
                     a->bin_offsets, p.pool);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return tg::fail(TG_ERR_HIP, "decode launch failed: %s", hipGetErrorString(e));
  if (a->num_partials > 0 && !fused_merge) {
    MergeFn mf = pick_merge(a->dtype, g.head_dim, lanes);
    // one chain: four outputs per thread; several: a workgroup per (unit, head), D/4 threads per chain
    const int block = lanes == 1 ? kBlock : g.head_dim / 4 * lanes;
    const int grid_y = lanes == 1 ? (gqa * g.head_dim / 4 + kBlock - 1) / kBlock : gqa;
    hipLaunchKernelGGL(mf, dim3(a->batch * g.num_kv_heads, grid_y), dim3(block), 0, st, a->unit_splits,
                       a->unit_partial_base, p.part_o, p.part_lse, a->out, a->lse, g.num_kv_heads, gqa);
    e = hipGetLastError();
    if (e != hipSuccess) return tg::fail(TG_ERR_HIP, "merge launch failed: %s", hipGetErrorString(e));
  }
  return TG_OK;
}


}  // namespace

extern "C" {

size_t tg_decode_workspace_bytes(const tg_geometry* geom, int32_t batch, int32_t num_partials) {
  if (!geom || geom->num_kv_heads < 1 || geom->num_q_heads < geom->num_kv_heads || num_partials < 0 || batch < 0)
    return 0;
  const size_t gqa = (size_t)(geom->num_q_heads / geom->num_kv_heads);
  const size_t d = (size_t)geom->head_dim;
  // fp32 partial outputs, then their lse
  return align256((size_t)num_partials * gqa * d * sizeof(float)) +
         align256((size_t)num_partials * gqa * sizeof(float));
}

int32_t tg_decode_bins_per_workgroup(const tg_geometry* geom, int32_t dtype, int32_t n_bins, int32_t* bins) {
  if (!bins) return tg::fail(TG_ERR_INVALID_ARG, "bins is NULL");
  if (n_bins < 1) return tg::fail(TG_ERR_INVALID_ARG, "n_bins must be >= 1");
  if (int32_t rc = check_decode_shape(geom, dtype)) return rc;
  *bins = bins_per_wg(dtype, geom->head_dim, geom->num_q_heads / geom->num_kv_heads, n_bins);
  return TG_OK;
}

int32_t tg_decode_max_ctas(const tg_geometry* geom, int32_t dtype, int32_t device, int32_t* n_cta) {
  if (!n_cta) return tg::fail(TG_ERR_INVALID_ARG, "n_cta is NULL");
  if (int32_t rc = check_decode_shape(geom, dtype)) return rc;
  // the kernel that a plan of as many bins as fit runs on
  const int gqa = geom->num_q_heads / geom->num_kv_heads;
  DecodeFn fn = pick_decode(dtype, geom->head_dim, gqa, INT32_MAX);
  int cus = 0, per_cu = 0;
  if (hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, device) != hipSuccess)
    return tg::fail(TG_ERR_HIP, "hipDeviceGetAttribute failed for device %d", device);
  int prev = 0;
  if (hipGetDevice(&prev) != hipSuccess) return tg::fail(TG_ERR_HIP, "hipGetDevice failed");
  if (prev != device && hipSetDevice(device) != hipSuccess) return tg::fail(TG_ERR_HIP, "hipSetDevice failed");
  hipError_t e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, reinterpret_cast<const void*>(fn), kBlock, 0);
  if (prev != device) (void)hipSetDevice(prev);
  if (e != hipSuccess) return tg::fail(TG_ERR_HIP, "occupancy query failed: %s", hipGetErrorString(e));
  *n_cta = per_cu * cus * (wave_per_bin(dtype, geom->head_dim, gqa, INT32_MAX) ? kWaves : 1);
  return TG_OK;
}

int32_t tg_decode(const tg_decode_args* a, void* hip_stream) {
  if (!a) return tg::fail(TG_ERR_INVALID_ARG, "args is NULL");
  return decode_impl(a, a->workspace, a->workspace_bytes, hip_stream);
}

int32_t tg_decode_noalloc(const tg_decode_args* a, void* hip_stream) {
  if (!a) return tg::fail(TG_ERR_INVALID_ARG, "args is NULL");
  if (int32_t rc = check_decode_shape(&a->geom, a->dtype)) return rc;
  if (a->batch < 1 || a->num_partials < 0) return tg::fail(TG_ERR_INVALID_ARG, "batch must be >= 1, num_partials >= 0");
  const size_t need = tg_decode_workspace_bytes(&a->geom, a->batch, a->num_partials);
  if (need > (size_t)TG_DECODE_NOALLOC_MAX_BYTES - kScratchCounters)
    return tg::fail(TG_ERR_BUFFER_TOO_SMALL,
                    "tg_decode_noalloc: %d partials need %zu bytes of scratch, the static scratch holds %zu",
                    a->num_partials, need, (size_t)TG_DECODE_NOALLOC_MAX_BYTES - kScratchCounters);
  void* ws = nullptr;
  if (int32_t rc = scratch_address(&ws)) return rc;
  // the scratch starts with kScratchCounters bytes of merge arrival counters
  // (zero at load; every call leaves them zero), then the partials
  tg_decode_args b = *a;
  char* base = static_cast<char*>(ws);
  const bool counters_fit = (size_t)a->batch * a->geom.num_kv_heads * sizeof(int32_t) <= kScratchCounters;
  b.merge_counters = a->merge_counters && counters_fit ? reinterpret_cast<int32_t*>(base) : nullptr;
  return decode_impl(&b, base + kScratchCounters, (size_t)TG_DECODE_NOALLOC_MAX_BYTES - kScratchCounters, hip_stream);
}

}  // extern "C"

// Ragged chunked-prefill attention for gfx950 (MI355X), bf16 MFMA.
//
// Chunked prefill (Section 2.2.1 of arXiv 2606.06302) over Tangram's ragged
// compressed cache (Section 4.2): row i of request b's chunk, query head
// qh = h*gqa + j, attends to the kv_len[b][layer][h] retained history rows of
// KV head h (all visible) followed by chunk keys 0..i (causal, inclusive).
//
// Work decomposition.  The gqa query heads of a KV head are packed into the
// row dimension (row r = i*gqa + j), so every K/V tile is reused by gqa*rows
// queries.  One workgroup (8 waves, two per SIMD) owns 256 consecutive rows
// of one (b, h); wave w owns 32 of them (one 32-row MFMA column block).  With
// two waves per SIMD the matrix core runs one wave's products while the other
// does its softmax.  Key tiles of 64 keys:
// first the paged history (four pages per tile), then the chunk's own keys up
// to the workgroup's last row.  Blocks are placed XCD-aware: all row tiles of
// a (b, h) run on the same XCD (block id mod 8), so the history they share is
// read into one L2; the host schedule (tg_prefill_schedule) balances the units
// over the XCDs by their tile counts and starts the longest blocks first.  Given
// a workspace, blocks much longer than the rest are cut by keys (key-split
// launch, below).
//
// Data movement.  Tiles stream into a 4-deep LDS ring with gfx950's
// global_load_lds_dwordx4 (no staging registers); wave w fetches key rows
// 8w..8w+7 of a tile (half a page of history).  The DMA is issued from inline
// assembly (invisible to the compiler's wait-count pass), every wave waits for
// its own part with an explicit vmcnt, and one barrier per tile then makes the
// whole tile visible and retires every read of the slot the next DMA refills.
// Page ids and table entries are read with scalar loads.
//
// Per 32-key block and 32-row column block (v_mfma_f32_32x32x16_bf16, fp32
// accumulate):
//   S^T[key][row] = K Q^T   (A = K rows from LDS, B = Q rows in registers)
//   online softmax per row  (a lane owns one row: max over its 16 keys plus
//                            one permlane32 swap with the lane holding the rest)
//   O^T[dv][row] += V^T P^T (B = P^T straight from the lane's own S^T
//                            registers, rounded to bf16; A = V^T read from the
//                            row-major V tile with ds_read_b64_tr_b16)
// The lane in half hf = lane / 32 holds S^T keys {4hf..4hf+3, 8+4hf..8+4hf+3}
// of each 16-key half block and feeds them as B's 8 k-indices, so the A
// operand takes the same keys: two transposed reads of 4 consecutive keys.
// V rows of the last history tile past the retained length are zeroed in LDS
// by the wave that fetched them, so the PV loop needs no mask.
// LDS layout: chunk c (16 bytes) of key row r sits at position c ^ (r mod 16)
// in the K tile and c ^ 4(r mod 4) in the V tile, so the K operand reads and
// the transposed V reads are bank-conflict free.
#include <hip/hip_runtime.h>

#include <cmath>

#include "tg_device.h"
#include "tg_internal.h"

namespace {

using namespace tgd;

typedef uint32_t u4 __attribute__((ext_vector_type(4)));
typedef uint32_t u2v __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x4_vs __attribute__((__vector_size__(4 * sizeof(__bf16))));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef float f32x2 __attribute__((ext_vector_type(2)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef __bf16 bf16x2v __attribute__((ext_vector_type(2)));

#define TG_CONST __attribute__((address_space(4)))
#define TG_LDS __attribute__((address_space(3)))

constexpr int kPage = 16;
constexpr int kWaves = 8;
constexpr int kBlock = 64 * kWaves;
constexpr int kCB = 1;                         // 32-row MFMA column blocks per wave
constexpr int kRowsPerWave = 32 * kCB;
constexpr int kRows = kRowsPerWave * kWaves;   // query rows per workgroup
constexpr int kTile = 64;                      // keys per tile = 4 pages
static_assert(kRows == TG_PREFILL_ROWS && kTile == TG_PREFILL_TILE, "tg_prefill_schedule costs these tiles");
constexpr int kRing = 4;                       // LDS tile buffers
static_assert(kRing >= 2 && kRing <= 4, "the wait below covers up to two tiles in flight after the current one");
constexpr int kDmaRows = kTile / kWaves;       // key rows each wave fetches per tile
constexpr float kSlack = 8.0f;

// Shape constants of the kernel for head_dim D (64 or 128).  A key row is
// 2*D bytes = kChunks 16-byte chunks; one 1 KiB DMA instruction (64 lanes x
// 16 bytes) moves kRowsPerDma rows.  LDS swizzles: chunk c of key row r of a
// tile sits at position c ^ k_swz(r) in the K tile and c ^ v_swz(r) in the V
// tile (r taken mod 16, which is also the row within its page), chosen so
// that the q.k operand reads and the transposed V reads are bank-conflict free.
template <int D>
struct Shape {
  static_assert(D == 64 || D == 128, "head_dim 64 or 128");
  static constexpr int kChunks = D / 8;
  static constexpr int kRowsPerDma = 64 / kChunks;
  static constexpr int kDmaInst = kDmaRows / kRowsPerDma;   // 1 KiB instructions per K or V slab and wave
  static constexpr int kDmaPerTile = 2 * kDmaInst;
  static constexpr int kTileBytes = 2 * kTile * D * 2;      // K + V
  static constexpr int kK = D / 16;                         // 16-deep k steps of q.k
  static constexpr int kDB = D / 32;                        // 32-dim blocks of the output
  __device__ static constexpr int k_swz(int r) { return D == 128 ? (r & 15) : ((r >> 1) & 7); }
  __device__ static constexpr int v_swz(int r) { return D == 128 ? 4 * (r & 3) : 2 * (r & 3); }
};

struct PrefillParams {
  const uint16_t* q;        // [B][C][Hq][d]
  const u4* k_new;          // [B][C][H][d]
  const u4* v_new;
  const u4* pool;           // [pages][2][Hp][P][d]
  const int32_t* pt_pages;
  const int64_t* pt_offsets;
  const int32_t* kv_len;    // [B][L][H]
  const int32_t* group_of;  // [L][H]
  const int32_t* slot_of;
  uint16_t* out;            // [B][C][Hq][d]
  const int32_t* block_order;   // [gridDim.x] (unit * row_tiles + row tile) or -1, or NULL
  int32_t batch, chunk, layer, num_layers, num_kv_heads, num_groups, heads_per_group, gqa;
  int32_t row_tiles;        // ceil(chunk*gqa / kRows)
  float scale_log2;
  // key-split launch only
  f32x4* part_o;            // [kSplitSlots][part_waves][D/4][32 rows] unnormalised fp32 outputs
  float* part_ml;           // [kSplitSlots][part_waves][2][32 rows]: reference maximum, sum
  int2* pieces;             // [units * row_tiles]: first partial slot and piece count of every block
  int32_t part_waves;       // waves of a block that own rows: min(8, ceil(chunk*gqa / 32))
  int32_t last_tiles;       // key tiles of the chunk that a unit's last row tile sees
};

// Key-split launch.  The longest block bounds a launch of few or very unequal
// blocks: one request of 8 KV heads, chunk 512, is 64 blocks on 256 CUs, and
// the two long heads' 16 blocks hold 65 % of the key tiles.  With a workspace,
// blocks of more than T key tiles are cut into equal pieces of at most T, one
// workgroup each, which leave fp32 partials (accumulator, reference maximum,
// sum) for a second launch to merge.  T = max(kSplitMinTiles, total / target),
// so there are at most `target` pieces more than blocks.  Every workgroup
// derives the cut from the lengths itself: one thread per unit, the cut units
// first, then the others in seven classes of descending length, so that the
// longest pieces start first.  The row tiles of one (unit, piece) share its keys and run side
// by side on one XCD (workgroup id mod 8), the (unit, piece) groups
// round-robin over the XCDs.
//
// Measured, whole blocks against cut ones: one request, head_dim 128, chunk
// 512 over a 16384-token history 440 -> 76 us, chunk 16 over 8192 153 -> 20
// us; four requests, chunk 512 over 8192 166 -> 117 us; head_dim 64, five
// requests, chunk 333, 74 -> 45 us.  Where no block is much longer than the
// mean per CU the merge costs more than the cut saves (four requests, chunk
// 512 over 2048 tokens: 61 against 72 us): the caller gives no workspace there
// (tg_prefill_split_pays).
constexpr int kSplitMinTiles = tg::kPrefillSplitMinTiles;
static_assert(tg::kPrefillSplitMaxUnits == kBlock, "one thread per unit");
constexpr int split_target(int d) { return tg::prefill_split_target(d); }
// a cut unit of n tiles has at most n / T + 1 <= 2n / T pieces
constexpr int split_slots(int d) { return 2 * split_target(d); }

__device__ __forceinline__ f32x16 mfma(const u4& a, const u4& b, const f32x16& c) {
  return __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, a), __builtin_bit_cast(bf16x8, b), c, 0, 0,
                                                 0);
}

__device__ __forceinline__ uint32_t lds_address(const void* ptr) {
  return static_cast<uint32_t>(reinterpret_cast<uintptr_t>((const TG_LDS void*)ptr));
}

// 16 bytes per lane from global memory (a wave-uniform base plus 16 * chunk
// bytes per lane) into LDS at m0_base + 16 * lane.  The scalar base keeps
// 64-bit addresses out of the vector registers.
__device__ __forceinline__ void lds_dma16(const u4* base, uint32_t chunk, uint32_t m0_base) {
  asm volatile("global_load_lds_dwordx4 %0, %1" ::"v"(chunk * 16), "s"(base), "{m0}"(m0_base) : "memory");
}

template <int N>
__device__ __forceinline__ void wait_vmcnt() {
  static_assert(N >= 0 && N < 64, "vmcnt is 6 bits");
  asm volatile("s_waitcnt vmcnt(%0)" ::"n"(N) : "memory");
}

__device__ __forceinline__ void barrier() { asm volatile("s_barrier" ::: "memory"); }

// (lo, hi) rounded to bf16 and packed into one dword (one v_cvt_pk_bf16_f32)
__device__ __forceinline__ uint32_t pack_bf16(float lo, float hi) {
  return __builtin_bit_cast(uint32_t, __builtin_convertvector(f32x2{lo, hi}, bf16x2v));
}

// Lane l of each 16-lane block receives element l % 4 of the 8-byte rows
// addressed by lanes l/4, l/4 + 4, l/4 + 8, l/4 + 12 of the block.
__device__ __forceinline__ u2v lds_read_tr16(const void* ptr) {
  return __builtin_bit_cast(u2v, __builtin_amdgcn_ds_read_tr16_b64_v4bf16((TG_LDS bf16x4_vs*)ptr));
}

// Inclusive sum over the lanes of a wave.
__device__ __forceinline__ int wave_inclusive_sum(int x) {
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) {
    const int y = __shfl_up(x, o);
    if ((int)(threadIdx.x & 63) >= o) x += y;
  }
  return x;
}

// Registers: 222 and 226 (key-split) at head_dim 128, 128 at 64, none in scratch.
// A reload from scratch would wait for every DMA in flight: with 64-bit lane
// addresses for the DMA, six reloads a tile at head_dim 64 drained the ring
// (five requests, chunk 333, 49.4 us against 45.1; the blocks of one request,
// chunk 512 over 16384 tokens, 58 against 54).
template <int D, bool kSplit, int kWavesPerSimd>
__global__ void __launch_bounds__(kBlock, kWavesPerSimd) tg_prefill_kernel(PrefillParams p) {
  using S = Shape<D>;
  constexpr int kChunks = S::kChunks, kDmaInst = S::kDmaInst, kDmaPerTile = S::kDmaPerTile;
  constexpr int kTileBytes = S::kTileBytes, kRowsPerDma = S::kRowsPerDma;
  __shared__ u4 ring[kRing][2][kTile * kChunks];   // [slot][K, V][key row * kChunks + chunk position]
  // key-split launch: a sum and the group counts per (class, wave), this workgroup's piece
  __shared__ int64_t wave_sum[kSplit ? kWaves : 1];
  __shared__ int32_t class_groups[kSplit ? 64 : 1];
  __shared__ int32_t mine[kSplit ? 3 : 1];

  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int n_units = p.batch * p.num_kv_heads;
  const int C = p.chunk, gqa = p.gqa;
  const int Hq = p.num_kv_heads * gqa;
  const int rows_total = C * gqa;

  const TG_CONST int32_t* kv_len = (const TG_CONST int32_t*)p.kv_len;
  const TG_CONST int32_t* group_of = (const TG_CONST int32_t*)p.group_of;
  const TG_CONST int32_t* slot_of = (const TG_CONST int32_t*)p.slot_of;
  const TG_CONST int64_t* pt_offsets = (const TG_CONST int64_t*)p.pt_offsets;
  const TG_CONST int32_t* pt_pages = (const TG_CONST int32_t*)p.pt_pages;

  // block -> (unit, row tile): the host schedule, or units round-robin over
  // the 8 XCDs (all row tiles of a unit on one XCD either way); in the
  // key-split launch, this workgroup's piece of a block
  int unit, rt;
  int piece = 0, first_slot = 0, piece_tiles = 0;   // key-split launch
  if constexpr (kSplit) {
    const int u = threadIdx.x;
    int n = 0;
    if (u < n_units) {
      const int ub = u / p.num_kv_heads, uh = u % p.num_kv_heads;
      const int64_t ti = ((int64_t)ub * p.num_layers + p.layer) * p.num_groups +
                         p.group_of[(int64_t)p.layer * p.num_kv_heads + uh];
      const int64_t ucap = (p.pt_offsets[ti + 1] - p.pt_offsets[ti]) * kPage;
      const int64_t len = p.kv_len[((int64_t)ub * p.num_layers + p.layer) * p.num_kv_heads + uh];
      n = (int)((max<int64_t>(0, min<int64_t>(len, ucap)) + kTile - 1) / kTile) + p.last_tiles;
    }
    int64_t sum = n;
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) sum += __shfl_xor((long long)sum, o);
    if (lane == 0) wave_sum[wave] = sum;
    if (threadIdx.x == 0) mine[0] = -1;
    __syncthreads();
    sum = 0;
#pragma unroll
    for (int w = 0; w < kWaves; ++w) sum += wave_sum[w];
    constexpr int kTarget = split_target(D);
    const int64_t total = sum * p.row_tiles;
    piece_tiles = (int)max<int64_t>(kSplitMinTiles, (total + kTarget - 1) / kTarget);
    const int np = (n + piece_tiles - 1) / piece_tiles;   // 0 past the last unit
    // the unit's place in the order: its class's first group, then units by
    // index; class 0 is the cut units, 1..7 the others by descending length
    const int cls = np > 1 ? 0 : 7 - (int)((int64_t)min(n, piece_tiles) * 6 / piece_tiles);
    int before = 0;    // groups before this unit's within its class and wave
    int count = 0;     // lane c: groups of class c in this wave
#pragma unroll
    for (int c = 1; c < 8; ++c) {
      const uint64_t in = __ballot(np == 1 && cls == c);
      if (cls == c) before = (int)__builtin_amdgcn_mbcnt_hi((uint32_t)(in >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)in, 0u));
      if (lane == c) count = __popcll(in);
    }
    const int cut = np > 1 ? np : 0;
    const int cut_sum = wave_inclusive_sum(cut);
    if (cls == 0) before = cut_sum - cut;
    const int cut_all = __shfl(cut_sum, 63);
    if (lane == 0) count = cut_all;
    if (lane < 8) class_groups[8 * lane + wave] = count;
    __syncthreads();
    const int in_order = class_groups[lane];   // (class, wave) in order
    before += __shfl(wave_inclusive_sum(in_order) - in_order, 8 * cls + wave);
    const int g = ((int)blockIdx.x >> 3) / p.row_tiles * 8 + (blockIdx.x & 7);   // (unit, piece) group
    rt = ((int)blockIdx.x >> 3) % p.row_tiles;
    if (before <= g && g < before + np) {   // exactly one unit, or none past the last group
      mine[0] = u;
      mine[1] = g - before;
      mine[2] = before;   // the cut units come first: their groups are the partial slots
    }
    __syncthreads();
    unit = __builtin_amdgcn_readfirstlane(mine[0]);
    piece = __builtin_amdgcn_readfirstlane(mine[1]);
    first_slot = __builtin_amdgcn_readfirstlane(mine[2]);
    piece_tiles = __builtin_amdgcn_readfirstlane(piece_tiles);
    if (unit < 0) return;
  } else if (p.block_order) {
    const int code = ((const TG_CONST int32_t*)p.block_order)[blockIdx.x];
    if (code < 0 || code >= n_units * p.row_tiles) return;
    unit = code / p.row_tiles;
    rt = code % p.row_tiles;
  } else {
    const int xcd = blockIdx.x & 7, local = blockIdx.x >> 3;
    unit = xcd + 8 * (local / p.row_tiles);
    rt = local % p.row_tiles;
    if (unit >= n_units) return;
  }

  const int b = unit / p.num_kv_heads, h = unit % p.num_kv_heads;
  const int grp = group_of[(int64_t)p.layer * p.num_kv_heads + h];
  const int slot = slot_of[(int64_t)p.layer * p.num_kv_heads + h];
  const int64_t tidx = ((int64_t)b * p.num_layers + p.layer) * p.num_groups + grp;
  const int64_t tbase = pt_offsets[tidx];
  // the history is clamped to the head's table: [0, pages * page_size]
  const int64_t cap = (pt_offsets[tidx + 1] - tbase) * kPage;
  const int hist = (int)max<int64_t>(0, min<int64_t>(kv_len[((int64_t)b * p.num_layers + p.layer) * p.num_kv_heads + h], cap));
  const int npages = (hist + kPage - 1) / kPage;
  const int n_hist_tiles = (hist + kTile - 1) / kTile;
  const int row0 = rt * kRows;
  const int i_last = min(C - 1, (min(row0 + kRows, rows_total) - 1) / gqa);   // last chunk row of the block
  const int n_tiles = n_hist_tiles + (i_last + kTile) / kTile;
  int t_begin = 0, t_end = n_tiles, np = 1;
  if constexpr (kSplit) {
    np = (n_tiles + piece_tiles - 1) / piece_tiles;   // fewer than the unit's where the row tile sees less of the chunk
    if (piece == 0 && threadIdx.x == 0) p.pieces[unit * p.row_tiles + rt] = make_int2(first_slot * p.row_tiles + rt, np);
    if (piece >= np) return;
    t_begin = (int)((int64_t)piece * n_tiles / np);
    t_end = (int)((int64_t)(piece + 1) * n_tiles / np);
  }

  const int hf = lane >> 5;
  const int wave_i_max = min(C - 1, (min(row0 + wave * kRowsPerWave + kRowsPerWave, rows_total) - 1) / gqa);
  const int wave_i_min = min(C - 1, (row0 + wave * kRowsPerWave) / gqa);

  // DMA of this wave's share (key rows kDmaRows*w .. kDmaRows*(w+1)-1) of tile
  // t into ring slot s
  const uint32_t ring_lds = lds_address(&ring[0][0][0]);
  const int rl = lane / kChunks;   // row within a DMA instruction
  const int pos = lane % kChunks;  // chunk position within the row
  const int rb0 = (wave * kDmaRows) % kPage;   // first row of the share within its page
  auto issue = [&](int t, int s) {
    const uint32_t dst = ring_lds + (uint32_t)s * kTileBytes + (uint32_t)wave * (kDmaRows * kChunks * 16);
    if (t < n_hist_tiles) {
      // past the history: any valid page, masked later
      const int pg = min(t * (kTile / kPage) + wave * kDmaRows / kPage, npages - 1);
      const int64_t id = pt_pages[tbase + pg];
      const u4* kb = p.pool + ((id * 2 + 0) * p.heads_per_group + slot) * (kPage * kChunks);
      const u4* vb = p.pool + ((id * 2 + 1) * p.heads_per_group + slot) * (kPage * kChunks);
#pragma unroll
      for (int j = 0; j < kDmaInst; ++j) {
        const int r = rb0 + j * kRowsPerDma + rl;   // key row within the page (== tile row mod 16)
        lds_dma16(kb, r * kChunks + (pos ^ S::k_swz(r)), dst + j * 1024);
        lds_dma16(vb, r * kChunks + (pos ^ S::v_swz(r)), dst + kTile * kChunks * 16 + j * 1024);
      }
    } else {
      const int c0 = min((t - n_hist_tiles) * kTile + wave * kDmaRows, C - 1);   // first chunk key of the share
      const int64_t first = (((int64_t)b * C + c0) * p.num_kv_heads + h) * kChunks;
      const u4* kb = p.k_new + first;
      const u4* vb = p.v_new + first;
#pragma unroll
      for (int j = 0; j < kDmaInst; ++j) {
        const int r = j * kRowsPerDma + rl;
        const int rr = rb0 + r;             // tile row mod 16
        const int roff = min(r, C - 1 - c0) * p.num_kv_heads * kChunks;   // rows past the chunk repeat its last key (masked later)
        lds_dma16(kb, roff + (pos ^ S::k_swz(rr)), dst + j * 1024);
        lds_dma16(vb, roff + (pos ^ S::v_swz(rr)), dst + kTile * kChunks * 16 + j * 1024);
      }
    }
  };

  f32x16 acc[kCB][S::kDB];
  float m[kCB], l[kCB];
#pragma unroll
  for (int cb = 0; cb < kCB; ++cb) {
#pragma unroll
    for (int d = 0; d < S::kDB; ++d) acc[cb][d] = f32x16(0.f);
    m[cb] = -INFINITY;
    l[cb] = 0.f;
  }
  const float cs = p.scale_log2;

  // lane-constant parts of the LDS operand addresses
  const int k_row = lane & 31;                                  // A of S^T: key row kb*32 + k_row
  const int tr_key = (lane & 15) >> 2;                          // transposed read: key within a group of 4
  const int tr_dim = 16 * ((lane >> 4) & 1) + 4 * (lane & 3);   // dims within a 32-dim block
  const int tr_chunk = tr_dim >> 3, tr_half = (tr_dim >> 2) & 1;

  // this lane's query row
  int my_i[kCB];
  bool row_ok[kCB];
  u4 qb[kCB][S::kK];
#pragma unroll
  for (int cb = 0; cb < kCB; ++cb) {
    const int r = row0 + wave * kRowsPerWave + cb * 32 + (lane & 31);
    row_ok[cb] = r < rows_total;
    my_i[cb] = row_ok[cb] ? r / gqa : 0;
    const int j = row_ok[cb] ? r % gqa : 0;
    const u4* qp = reinterpret_cast<const u4*>(p.q + (((int64_t)b * C + my_i[cb]) * Hq + h * gqa + j) * D);
#pragma unroll
    for (int kk = 0; kk < S::kK; ++kk) qb[cb][kk] = row_ok[cb] ? qp[kk * 2 + hf] : u4(0u);
  }
  // Settle the query loads here, once: the compiler's wait-count pass cannot
  // see the inline-assembly LDS DMAs, so a load still pending at the loop
  // entry would make it wait for vmcnt(0) - every DMA in flight - at the first
  // use of qb on every tile.  Routing qb through an empty asm places that one
  // wait before the loop and leaves no compiler-tracked load behind.
#pragma unroll
  for (int cb = 0; cb < kCB; ++cb)
#pragma unroll
    for (int kk = 0; kk < S::kK; ++kk) asm volatile("" : "+v"(qb[cb][kk]));
  // prologue: the first kRing-1 tiles in flight (ring slot = tile - t_begin
  // modulo kRing)
#pragma unroll
  for (int r = 0; r < kRing - 1; ++r)
    if (t_begin + r < t_end) issue(t_begin + r, r);

  for (int t = t_begin; t < t_end; ++t) {
    // tile t has landed once at most the DMAs of the tiles after it are pending
    const int after = min(kRing - 2, t_end - 1 - t);
    if (after >= 2)
      wait_vmcnt<2 * kDmaPerTile>();
    else if (after == 1)
      wait_vmcnt<kDmaPerTile>();
    else
      wait_vmcnt<0>();
    if (t < n_hist_tiles && t * kTile + wave * kDmaRows + kDmaRows > hist) {
      // this wave's share holds V rows past the retained history: they may
      // hold anything (NaN included) and p = 0 does not cancel NaN, so zero them
      u4* vq = &ring[(t - t_begin) % kRing][1][wave * kDmaRows * kChunks];
#pragma unroll
      for (int j = 0; j < kDmaInst; ++j)
        if (t * kTile + wave * kDmaRows + j * kRowsPerDma + rl >= hist) vq[j * 64 + lane] = u4(0u);
      asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    }
    barrier();   // tile t complete in LDS; every wave is done with tile t-1
    if (t + kRing - 1 < t_end) issue(t + kRing - 1, (t - t_begin + kRing - 1) % kRing);

    const int s = (t - t_begin) % kRing;
    const unsigned char* kt = reinterpret_cast<const unsigned char*>(&ring[s][0][0]);
    const unsigned char* vt = reinterpret_cast<const unsigned char*>(&ring[s][1][0]);
    const bool is_chunk = t >= n_hist_tiles;
    const int key0 = is_chunk ? (t - n_hist_tiles) * kTile : t * kTile;   // first key of the tile
    const int key_end = is_chunk ? C : hist;                                 // keys >= this are invalid
    if (is_chunk && key0 > wave_i_max) continue;   // tile entirely in the future of this wave's rows

#pragma unroll
    for (int kb = 0; kb < 2; ++kb) {
      const int kbase = key0 + kb * 32;
      if (is_chunk && kbase > wave_i_max) break;
      // S^T for both column blocks; the K operand is read once
      f32x16 sc[kCB];
#pragma unroll
      for (int cb = 0; cb < kCB; ++cb) sc[cb] = f32x16(0.f);
      const int krow = kb * 32 + k_row;
      // all eight K operands of the block, and the V^T operands of its p.v
      // products (they do not depend on p), are requested before the first
      // product, so their LDS latency hides under q.k and the softmax
      u4 ka[S::kK];
#pragma unroll
      for (int kk = 0; kk < S::kK; ++kk)
        ka[kk] = *reinterpret_cast<const u4*>(kt + krow * (2 * D) + (((kk * 2 + hf) ^ S::k_swz(krow)) << 4));
      u4 va[2][S::kDB];
#pragma unroll
      for (int q16 = 0; q16 < 2; ++q16) {
        const int g0 = kb * 32 + q16 * 16 + 4 * hf;    // tile row of the A operand's first key
        const int r0 = g0 + tr_key, r1 = g0 + 8 + tr_key;  // source rows of the two transposed reads
#pragma unroll
        for (int db = 0; db < S::kDB; ++db) {
          const int c = 4 * db + tr_chunk;
          const u2v lo = lds_read_tr16(vt + r0 * (2 * D) + ((c ^ S::v_swz(r0)) << 4) + tr_half * 8);
          const u2v hi = lds_read_tr16(vt + r1 * (2 * D) + ((c ^ S::v_swz(r1)) << 4) + tr_half * 8);
          va[q16][db] = u4{lo.x, lo.y, hi.x, hi.y};
        }
      }
      __builtin_amdgcn_sched_barrier(0);   // keep the reads ahead of the products
#pragma unroll
      for (int kk = 0; kk < S::kK; ++kk)
#pragma unroll
        for (int cb = 0; cb < kCB; ++cb) sc[cb] = mfma(ka[kk], qb[cb][kk], sc[cb]);
      // only the block holding the end of the history and the chunk blocks
      // that reach past the wave's first row need a mask
      const bool masked = is_chunk ? kbase + 31 > wave_i_min : kbase + 32 > hist;
      if (masked) {
#pragma unroll
        for (int cb = 0; cb < kCB; ++cb)
#pragma unroll
          for (int r = 0; r < 16; ++r) {
            // lane holds keys n(r) = 8*(r/4) + 4*hf + r%4 of its row
            const int key = kbase + 8 * (r >> 2) + 4 * hf + (r & 3);
            const bool ok = key < key_end && (!is_chunk || key <= my_i[cb]);
            sc[cb][r] = ok ? sc[cb][r] : -INFINITY;
          }
      }
      u4 pb[kCB][2];
#pragma unroll
      for (int cb = 0; cb < kCB; ++cb) {
        float mx = -INFINITY;
#pragma unroll
        for (int r = 0; r < 16; ++r) mx = fmaxf(mx, sc[cb][r]);
        mx = swap32_max(mx);
        const bool raise = (mx - m[cb]) * cs > kSlack;
        if (__any(raise)) {   // raise the running max (rare after the first block)
          const float m_new = raise ? mx : m[cb];
          // 0 when m was -inf, and 1, not NaN, where it still is beside a row that raises
          const float alpha = kSplit && !raise ? 1.f : fast_exp2((m[cb] - m_new) * cs);
          m[cb] = m_new;
          l[cb] *= alpha;
#pragma unroll
          for (int d = 0; d < S::kDB; ++d) acc[cb][d] *= alpha;
        }
        // key-split launch: a row whose scores so far are all -inf has no
        // probabilities yet, not NaN (rows past the chunk's end are such, and
        // rows that meet infinite scores first)
        const float mcs = (kSplit && m[cb] == -INFINITY ? 0.f : m[cb]) * cs;
        uint32_t pw[8];
#pragma unroll
        for (int r = 0; r < 16; r += 2) {
          const float p0 = fast_exp2(fmaf(sc[cb][r], cs, -mcs));
          const float p1 = fast_exp2(fmaf(sc[cb][r + 1], cs, -mcs));
          l[cb] += p0 + p1;
          pw[r >> 1] = pack_bf16(p0, p1);
        }
        pb[cb][0] = u4{pw[0], pw[1], pw[2], pw[3]};
        pb[cb][1] = u4{pw[4], pw[5], pw[6], pw[7]};
      }
      // O^T += V^T P^T over the two 16-key halves of the block
#pragma unroll
      for (int q16 = 0; q16 < 2; ++q16)
#pragma unroll
        for (int db = 0; db < S::kDB; ++db)
#pragma unroll
          for (int cb = 0; cb < kCB; ++cb) acc[cb][db] = mfma(va[q16][db], pb[cb][q16], acc[cb][db]);
    }
  }
  wait_vmcnt<0>();
  // row sum over both halves of the row, then O = O^T / l
#pragma unroll
  for (int cb = 0; cb < kCB; ++cb) {
    const float lt = swap32_sum(l[cb]);
    if constexpr (kSplit) {
      static_assert(kCB == 1, "one partial row per lane pair");
      if (np > 1) {   // a piece: its partials, 16-byte stores contiguous over the 32 rows
        if (wave < p.part_waves) {
          const int64_t part = ((int64_t)(first_slot + piece) * p.row_tiles + rt) * p.part_waves + wave;
          f32x4* po = p.part_o + part * (D / 4) * 32 + (lane & 31);
#pragma unroll
          for (int db = 0; db < S::kDB; ++db)
#pragma unroll
            for (int r4 = 0; r4 < 4; ++r4)
              po[(db * 8 + 2 * r4 + hf) * 32] = f32x4{acc[cb][db][r4 * 4 + 0], acc[cb][db][r4 * 4 + 1],
                                                     acc[cb][db][r4 * 4 + 2], acc[cb][db][r4 * 4 + 3]};
          p.part_ml[part * 64 + lane] = hf ? lt : m[cb];
        }
        continue;
      }
    }
    if (!row_ok[cb]) continue;
    const int r = row0 + wave * kRowsPerWave + cb * 32 + (lane & 31);
    const int i = r / gqa, j = r % gqa;
    const float inv = 1.f / lt;
    uint16_t* orow = p.out + (((int64_t)b * C + i) * Hq + h * gqa + j) * D;
#pragma unroll
    for (int db = 0; db < S::kDB; ++db)
#pragma unroll
      for (int r4 = 0; r4 < 4; ++r4) {
        const int dv = db * 32 + 8 * r4 + 4 * hf;
        const uint32_t w0 = pack_bf16(acc[cb][db][r4 * 4 + 0] * inv, acc[cb][db][r4 * 4 + 1] * inv);
        const uint32_t w1 = pack_bf16(acc[cb][db][r4 * 4 + 2] * inv, acc[cb][db][r4 * 4 + 3] * inv);
        *reinterpret_cast<uint2*>(orow + dv) = make_uint2(w0, w1);
      }
  }
}

// Merge of the key-split launch: the pieces of a block are combined at the
// largest of their reference maxima (the pieces' sums and accumulators are
// relative to them).  Grid (blocks, waves with rows x D/32): thread = (row,
// four consecutive dims), so partial loads are contiguous over a wave's 32
// rows.  Bound by reading the partials back: 9 us for 220 pieces of 256 rows
// (29 MB).
template <int D>
__global__ void __launch_bounds__(256) tg_prefill_merge_kernel(PrefillParams p) {
  const int2 k = p.pieces[blockIdx.x];
  const int n = k.y;
  if (n <= 1) return;
  constexpr int kParts = D / 32;   // workgroups per 32 rows
  const int unit = blockIdx.x / p.row_tiles, rt = blockIdx.x % p.row_tiles;
  const int wave = blockIdx.y / kParts;
  const int chunk = (threadIdx.x >> 5) + 8 * (blockIdx.y % kParts);
  const int b = unit / p.num_kv_heads, h = unit % p.num_kv_heads;
  const int row = threadIdx.x & 31;
  const int r = rt * kRows + wave * kRowsPerWave + row;
  if (r >= p.chunk * p.gqa) return;
  auto part = [&](int i) { return ((int64_t)k.x + (int64_t)i * p.row_tiles) * p.part_waves + wave; };
  constexpr int kBatch = 4;
  float M = -INFINITY, L = 0.f;
  f32x4 A = f32x4(0.f);
  // kBatch pieces are requested before the first is used; past the last piece
  // it is read again and not used
  for (int i0 = 0; i0 < n; i0 += kBatch) {
    float mv[kBatch], lv[kBatch];
    f32x4 ov[kBatch];
#pragma unroll
    for (int j = 0; j < kBatch; ++j) {
      const int64_t pt = part(min(i0 + j, n - 1));
      mv[j] = p.part_ml[pt * 64 + row];
      lv[j] = p.part_ml[pt * 64 + 32 + row];
      ov[j] = p.part_o[(pt * (D / 4) + chunk) * 32 + row];
    }
    float Mn = M;
#pragma unroll
    for (int j = 0; j < kBatch; ++j) Mn = fmaxf(Mn, mv[j]);
    // a piece of chunk tiles that all lie in a wave's future leaves m = -inf and
    // zeros; while there is no other, nothing is rescaled and the weights are 0
    const float Mr = Mn == -INFINITY ? 0.f : Mn;
    const float a = fast_exp2((M - Mr) * p.scale_log2);
    L *= a;
    A *= a;
#pragma unroll
    for (int j = 0; j < kBatch; ++j) {
      const bool use = i0 + j < n;
      const float w = fast_exp2((mv[j] - Mr) * p.scale_log2);   // 0 for a piece with no visible key
      L = use ? fmaf(lv[j], w, L) : L;
#pragma unroll
      for (int q = 0; q < 4; ++q) A[q] = use ? fmaf(ov[j][q], w, A[q]) : A[q];
    }
    M = Mn;
  }
  const float inv = 1.f / L;
  const int Hq = p.num_kv_heads * p.gqa;
  uint16_t* orow = p.out + (((int64_t)b * p.chunk + r / p.gqa) * Hq + h * p.gqa + r % p.gqa) * D;
  *reinterpret_cast<uint2*>(orow + 4 * chunk) =
      make_uint2(pack_bf16(A[0] * inv, A[1] * inv), pack_bf16(A[2] * inv, A[3] * inv));
}

size_t align256(size_t x) { return (x + 255) & ~size_t(255); }

// Workspace of the key-split launch for this shape, 0 where it is not taken.
struct SplitLayout {
  int row_tiles, part_waves, groups;
  size_t o_bytes, ml_bytes, bytes;
};

SplitLayout split_layout(const tg_geometry& g, int batch, int chunk_len) {
  SplitLayout s = {};
  const int64_t rows = (int64_t)chunk_len * (g.num_q_heads / g.num_kv_heads);
  const int64_t row_tiles = (rows + kRows - 1) / kRows;
  const int64_t units = (int64_t)batch * g.num_kv_heads;
  if (units > tg::kPrefillSplitMaxUnits || units * row_tiles > tg::kPrefillSplitMaxBlocks) return s;
  s.row_tiles = (int)row_tiles;
  s.part_waves = (int)((rows < kRows ? rows : kRows) + 31) / 32;
  s.groups = split_target(g.head_dim) / s.row_tiles + (int)units;   // sum over units of ceil(n / T)
  const size_t parts = (size_t)split_slots(g.head_dim) * s.part_waves;
  s.o_bytes = align256(parts * 32 * g.head_dim * sizeof(float));
  s.ml_bytes = align256(parts * 64 * sizeof(float));
  s.bytes = s.o_bytes + s.ml_bytes + align256((size_t)(units * row_tiles) * sizeof(int2));
  return s;
}

int32_t check_prefill(const tg_prefill_args* a) {
  if (!a) return tg::fail(TG_ERR_INVALID_ARG, "args is NULL");
  const tg_geometry& g = a->geom;
  if (int32_t rc = tg::check_geometry(&g)) return rc;
  if (a->dtype != TG_BF16) return tg::fail(TG_ERR_UNSUPPORTED, "prefill supports bf16 only");
  if (g.head_dim != 64 && g.head_dim != 128)
    return tg::fail(TG_ERR_UNSUPPORTED, "prefill supports head_dim 64 or 128 (got %d)", g.head_dim);
  if (g.page_size != kPage) return tg::fail(TG_ERR_UNSUPPORTED, "prefill supports page_size 16 only");
  const int gqa = g.num_q_heads / g.num_kv_heads;
  if (gqa < 1 || gqa > 16) return tg::fail(TG_ERR_UNSUPPORTED, "prefill supports 1..16 query heads per KV head");
  if (a->batch < 1 || a->chunk_len < 1 || a->layer < 0 || a->layer >= g.num_layers)
    return tg::fail(TG_ERR_INVALID_ARG, "batch and chunk_len must be >= 1, layer in range");
  return TG_OK;
}

}  // namespace

extern "C" {

size_t tg_prefill_workspace_bytes(const tg_prefill_args* args) {
  if (check_prefill(args) != TG_OK) return 0;
  return split_layout(args->geom, args->batch, args->chunk_len).bytes;
}

int32_t tg_prefill(const tg_prefill_args* a, void* hip_stream) {
  if (int32_t rc = check_prefill(a)) return rc;
  const tg_geometry& g = a->geom;
  const int gqa = g.num_q_heads / g.num_kv_heads;
  if (!a->q || !a->k_new || !a->v_new || !a->kv_pool || !a->pt_pages || !a->pt_offsets || !a->kv_len ||
      !a->group_of || !a->slot_of || !a->out)
    return tg::fail(TG_ERR_INVALID_ARG, "NULL device pointer");
  if (!tg::aligned16({a->q, a->k_new, a->v_new, a->kv_pool, a->out}))
    return tg::fail(TG_ERR_INVALID_ARG, "device buffers must be 16-byte aligned");
  PrefillParams p;
  p.q = static_cast<const uint16_t*>(a->q);
  p.k_new = static_cast<const u4*>(a->k_new);
  p.v_new = static_cast<const u4*>(a->v_new);
  p.pool = static_cast<const u4*>(a->kv_pool);
  p.pt_pages = a->pt_pages;
  p.pt_offsets = a->pt_offsets;
  p.kv_len = a->kv_len;
  p.group_of = a->group_of;
  p.slot_of = a->slot_of;
  p.out = static_cast<uint16_t*>(a->out);
  p.block_order = a->block_order;
  p.batch = a->batch;
  p.chunk = a->chunk_len;
  p.layer = a->layer;
  p.num_layers = g.num_layers;
  p.num_kv_heads = g.num_kv_heads;
  p.num_groups = g.num_kv_heads / g.heads_per_group;
  p.heads_per_group = g.heads_per_group;
  p.gqa = gqa;
  p.row_tiles = (a->chunk_len * gqa + kRows - 1) / kRows;
  const float scale = a->sm_scale != 0.f ? a->sm_scale : 1.0f / std::sqrt((float)g.head_dim);
  p.scale_log2 = scale * kLog2e;
  const int units = a->batch * g.num_kv_heads;
  if (a->block_order && a->num_blocks < 1) return tg::fail(TG_ERR_INVALID_ARG, "block_order needs num_blocks >= 1");
  const int blocks = a->block_order ? a->num_blocks : 8 * ((units + 7) / 8) * p.row_tiles;
  hipStream_t st = static_cast<hipStream_t>(hip_stream);
  const SplitLayout sl = split_layout(g, a->batch, a->chunk_len);
  if (sl.bytes > 0 && a->workspace && a->workspace_bytes >= sl.bytes && tg::aligned16({a->workspace})) {
    char* ws = static_cast<char*>(a->workspace);
    p.part_o = reinterpret_cast<f32x4*>(ws);
    p.part_ml = reinterpret_cast<float*>(ws + sl.o_bytes);
    p.pieces = reinterpret_cast<int2*>(ws + sl.o_bytes + sl.ml_bytes);
    p.part_waves = sl.part_waves;
    p.last_tiles = (a->chunk_len - 1 + kTile) / kTile;
    auto split = g.head_dim == 128 ? tg_prefill_kernel<128, true, 2> : tg_prefill_kernel<64, true, 4>;
    auto merge = g.head_dim == 128 ? tg_prefill_merge_kernel<128> : tg_prefill_merge_kernel<64>;
    hipLaunchKernelGGL(split, dim3((sl.groups + 7) / 8 * 8 * sl.row_tiles), dim3(kBlock), 0, st, p);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return tg::fail(TG_ERR_HIP, "prefill launch failed: %s", hipGetErrorString(e));
    hipLaunchKernelGGL(merge, dim3(units * p.row_tiles, sl.part_waves * (g.head_dim / 32)), dim3(256), 0, st, p);
    e = hipGetLastError();
    if (e != hipSuccess) return tg::fail(TG_ERR_HIP, "prefill merge launch failed: %s", hipGetErrorString(e));
    return TG_OK;
  }
  // head_dim 64: two workgroups fit a CU (64 KiB rings, 128 registers), which
  // pays once there are more than two blocks per CU: 1024 blocks (16 requests,
  // chunk 512 over 4096) 177 -> 150 us, 640 blocks 91 -> 90.  Fewer blocks even
  // out better over the CUs one at a time, the longest first (512 blocks of 8
  // requests 63 us against 65, 336 of 14 37 against 38): LDS that is not used
  // keeps the second workgroup off.
  const size_t one_per_cu = g.head_dim == 64 && blocks <= tg::kPrefillOnePerCuBlocks ? 24 << 10 : 0;
  auto kernel = g.head_dim == 128 ? tg_prefill_kernel<128, false, 2> : tg_prefill_kernel<64, false, 2>;
  hipLaunchKernelGGL(kernel, dim3(blocks), dim3(kBlock), one_per_cu, st, p);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return tg::fail(TG_ERR_HIP, "prefill launch failed: %s", hipGetErrorString(e));
  return TG_OK;
}

}  // extern "C"

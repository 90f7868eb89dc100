// Internal helpers shared by the host and device translation units of
// libtangram.so (not part of the public ABI).
#pragma once
#include <cstdarg>
#include <cstdint>
#include <cstdio>
#include <initializer_list>

#include "tangram.h"

namespace tg {

// Records a thread-local message for tg_last_error() and returns `code`.
int32_t fail(int32_t code, const char* fmt, ...);

// Validates a geometry for the host integer calls.  On failure records a
// message and returns TG_ERR_INVALID_ARG.
int32_t check_geometry(const tg_geometry* g);

inline int64_t ceil_div(int64_t a, int64_t b) { return (a + b - 1) / b; }

// True when every pointer given is 16-byte aligned (NULL counts as aligned):
// the device calls move Q, K, V, outputs, partials and pool rows with 8- and
// 16-byte vector accesses.
inline bool aligned16(std::initializer_list<const void*> ptrs) {
  for (const void* q : ptrs)
    if (reinterpret_cast<uintptr_t>(q) & 15u) return false;
  return true;
}

// The cut of the key-split prefill launch, made on the device and foreseen by
// tg_prefill_split_pays: pieces of at least kPrefillSplitMinTiles key tiles,
// about prefill_split_target() of them, for at most so many units and blocks.
constexpr int kPrefillSplitMinTiles = 3;
constexpr int kPrefillSplitMaxUnits = 512;    // one thread of a workgroup per unit
constexpr int kPrefillSplitMaxBlocks = 1024;  // past it blocks outnumber the CUs by far and even out by themselves
// A little under the workgroups that run at once (one per CU at head_dim 128,
// two at 64), because cutting into equal pieces rounds up.  One request, chunk
// 512, 16384 tokens, with 160 / 208 / 256 / 320: 94 / 81 / 110 / 99 us at 128.
// At 64, chunk 512, with 352 / 448 / 512: one request over 16384 tokens 60 / 56
// / 65 us, two over 8192 61 / 57 / 68, four 95 / 109 / 110; over 57 shapes 0.99
// / 1 / 1.02.
constexpr int prefill_split_target(int head_dim) { return head_dim == 128 ? 208 : 448; }
// Whole-block launches of head_dim 64 with more blocks than this run two
// workgroups per CU.
constexpr int kPrefillOnePerCuBlocks = 512;

}  // namespace tg

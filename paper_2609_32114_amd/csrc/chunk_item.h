// chunk_item.h -- the (chunk, value head) work items of the chunk-local
// kernels and the LDS tile swizzle they share.
#pragma once

#include "device.h"
#include "prefill.h"

namespace hagdn {

// XOR-swizzled row-major tiles (rows of LD elements, a multiple of 128 bytes):
// 16-byte chunk q of row r is stored at chunk q ^ (r & 7), so the eight rows
// a fragment read touches in one LDS cycle hit eight different bank groups
// with no padding.
template <typename E, int LD>
__device__ __forceinline__ int swz(int r, int e) {
  constexpr int CH = 16 / (int)sizeof(E);
  return r * LD + ((e / CH) ^ (r & 7)) * CH + e % CH;
}
// One (chunk, value head) work item: chunk c = item / Hv, head h = item % Hv.
struct LocalItem {
  int c, h, start, len;  // len 0: past the last chunk
};
// Workgroup b -> item: the value heads of one q/k group (grouped heads share
// q and k) take consecutive ids of one XCD (ids b, b+8, ... share an XCD and
// its L2), so all but the first read q and k from L2.  Without grouping this
// is the identity.  The grid is padded to whole rounds of 8 groups.
__device__ __forceinline__ LocalItem local_item(const PrefillArgs &a, int b) {
  LocalItem it{0, 0, 0, 0};
  const int G = a.Hv / a.Hqk;  // value heads per q/k head
  const int xcd = b % 8, slot = b / 8;
  const int grp = (slot / G) * 8 + xcd;  // (chunk, q/k head) group
  if (grp < a.max_chunks * a.Hqk) {
    it.c = grp / a.Hqk;
    it.h = (grp % a.Hqk) * G + slot % G;
    if (a.single) {  // chunk c of the only sequence (tokens [0, T))
      it.start = it.c * kChunk;
      it.len = max(0, min(kChunk, a.T - it.start));
    } else {
      const int4 ci = a.chunk_info[it.c];
      it.start = ci.y;
      it.len = ci.z;
    }
  }
  return it;
}

// Workgroups of a chunk-local launch: one per (chunk, value head) block, padded
// to whole rounds of 8 q/k groups.
inline long local_grid(const PrefillArgs &a) {
  const long groups = (long)a.max_chunks * a.Hqk;
  return (groups + 7) / 8 * 8 * (a.Hv / a.Hqk);
}

}  // namespace hagdn

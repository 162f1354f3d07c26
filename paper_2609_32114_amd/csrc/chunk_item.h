// chunk_item.h -- the (chunk, value head) work items of the chunk-local
// kernels and the LDS tile swizzle they share.
#pragma once

#include "device.h"
#include "gate_map.h"
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

// ------------------------------------------------------------------ operator #3
// T = (I + A)^-1, unit lower triangular, fp32, blocked by 16, by four waves.
// Wave w holds its diagonal block of A transposed in accumulator order (lane
// (col, grp), element e = A[16w + col][16w + 4grp + e]) and inverts it from its
// registers; with A's strictly lower blocks and every T_ii in LDS, it then
// solves COLUMN block w: T_iw = -T_ii sum_{k=w}^{i-1} A_ik T_kw needs no other
// wave's blocks, so the rows follow one another without a barrier.

// fp32 16 x 16 x 16 product from operands in accumulator order: a[st] holds
// A[col][4grp + st], b[st] holds B[4grp + st][col].
__device__ __forceinline__ f32x4 mma16(f32x4 acc, f32x4 a, f32x4 b) {
#pragma unroll
  for (int st = 0; st < 4; ++st) acc = __builtin_amdgcn_mfma_f32_16x16x4f32(a[st], b[st], acc, 0, 0, 0);
  return acc;
}

__device__ __forceinline__ float lane_value(float x, int lane) {
  return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(x), lane));
}

// (I + A_ww)^-1 by forward substitution, column `col` per lane with A's elements
// broadcast from their lanes; returned in accumulator order (rows 4grp + e,
// column col).
__device__ __forceinline__ f32x4 invert_unit_lower(f32x4 ad) {
  const int col = threadIdx.x & 15, grp = (threadIdx.x >> 4) & 3;
  float x[16];
#pragma unroll
  for (int i = 0; i < 16; ++i) {
    float acc = i == col ? 1.f : 0.f;
#pragma unroll
    for (int s = 0; s < i; ++s) acc -= lane_value(ad[s & 3], i + 16 * (s >> 2)) * x[s];
    x[i] = acc;
  }
  f32x4 t;
#pragma unroll
  for (int e = 0; e < 4; ++e) t[e] = grp < 2 ? (grp == 0 ? x[e] : x[4 + e]) : (grp == 2 ? x[8 + e] : x[12 + e]);
  return t;
}

// Block (i, k) of the [64][64] tile: row col, columns 4grp .. +3.
__device__ __forceinline__ f32x4 block_rows(const float *sA, int i, int k) {
  const int col = threadIdx.x & 15, grp = (threadIdx.x >> 4) & 3;
  return *reinterpret_cast<const f32x4 *>(sA + swz<float, kChunk>(16 * i + col, 16 * k + 4 * grp));
}

// Blocks (i, wave), i > wave, of T from sA (strictly lower blocks: A; diagonal
// blocks: T_ii); `tw`: T_ww in accumulator order.  put(i, t) receives T_iw
// transposed (lane (col, grp), element e = T[16i + col][16 wave + 4grp + e]): the
// last product taken with its operands swapped.
template <typename Put>
__device__ __forceinline__ void solve_column(const float *sA, int wave, f32x4 tw, Put put) {
  f32x4 t[4];  // T_kw, k = wave .. 3
  t[0] = tw;
#pragma unroll
  for (int d = 1; d < 4; ++d) {
    const int i = wave + d;
    if (i < 4) {  // uniform for the wave
      f32x4 y = zero4();
#pragma unroll
      for (int k = 0; k < d; ++k) y = mma16(y, block_rows(sA, i, wave + k), t[k]);
      const f32x4 tii = block_rows(sA, i, i);
      if (i < 3) t[d] = -mma16(zero4(), tii, y);
      put(i, -mma16(zero4(), y, tii));
    }
  }
}

// Workgroups of a chunk-local launch: one per (chunk, value head) block, padded
// to whole rounds of 8 q/k groups.
inline long local_grid(const PrefillArgs &a) {
  const long groups = (long)a.max_chunks * a.Hqk;
  return (groups + 7) / 8 * 8 * (a.Hv / a.Hqk);
}

}  // namespace hagdn

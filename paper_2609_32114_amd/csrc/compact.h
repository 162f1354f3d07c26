// compact.h -- the compact factors of GDN prefill in bf16, and what their
// producer (k1_compact.hip) and consumers (k2_compact.hip) share.
//
// Per (chunk, value head) block the compact path keeps only what depends on
// more than one token of the chunk and not on the state.  With gamma the
// inclusive cumulative log-gate, T = (I + A)^-1 and P the operators #2 and #3
// (k1_chunk_local.hip):
//   T' = T Diag(b)                       P' = scale P
//   ek = nk e^gamma    kd = nk e^(gamma_last - gamma)    eq = scale nq e^gamma
// (nk, nq: the tokens' L2 factors of raw keys and queries, else 1).  The walk
// reads k, q and v themselves and carries the state S^T_c (d_k x d_v) through
//   X = V - Diag(ek) K S^T_c            U = T' X
//   S^T_{c+1} = e^gamma_last S^T_c + K^T Diag(kd) U
//   O = Diag(eq) Q S^T_c + P' U
// three dependent products per chunk where the affine factors (prefill.h) need
// one, but 13 KiB per block through memory instead of 96 KiB: T' and P' are
// lower triangular, 6 of their 8 operand blocks each.
//
// Block layout, kCompactBytes apart, from the start of the NM region: T' then
// P' (operand blocks of 64 lanes x 8 elements, block tri_block(nt, kb): row
// tile nt, k-block kb; slot j of lane (col, grp) = M[16nt + col][32kb + kmap(grp, j)]),
// then the 64-token vectors ek, kd, eq and 64 floats whose first is e^gamma_last.
#pragma once

#include "device.h"
#include "prefill.h"

namespace hagdn {

constexpr int kTriBlocks = 6;
constexpr int kTriBytes = kTriBlocks * 1024;
constexpr int kVecBytes = 4 * kChunk * 4;
constexpr int kCompactBytes = 2 * kTriBytes + kVecBytes;

// Operand block (row tile nt, 32-column block kb <= nt / 2) of a lower triangle.
__host__ __device__ __forceinline__ constexpr int tri_block(int nt, int kb) { return nt < 2 ? nt : 2 * nt - 2 + kb; }

// State row (d_k) held by row i (0..15) of accumulator tile rt: the fragment
// of a 32-row block made of two tiles (frag_from_acc) then holds eight
// consecutive d_k per lane, as a key or query row holds them in memory.
__host__ __device__ __forceinline__ constexpr int dk_of(int rt, int i) {
  return 32 * (rt >> 1) + 8 * (i >> 2) + 4 * (rt & 1) + (i & 3);
}

// Direct memory-to-LDS loads: lane l's 16 bytes land at l * 16 of the (wave
// uniform) LDS address.
__device__ __forceinline__ void lds_copy16(const void *g, void *l) {
  __builtin_amdgcn_global_load_lds(g, (__attribute__((address_space(3))) void *)l, 16, 0, 0);
}
// s_waitcnt vmcnt(N) alone (export and LDS counters at their maxima; gfx9 encoding)
template <int N>
__device__ __forceinline__ void wait_loads() {
  static_assert(N >= 0 && N < 64, "vmcnt range");
  __builtin_amdgcn_s_waitcnt((N & 0xF) | ((N >> 4) << 14) | 0x70 | 0xF00);
}

// Token rows in LDS (a stage of k2_compact.hip, the keys of k1_compact.hip):
// rows of ROW bytes, the 16-byte piece q of row r stored at piece
// q ^ row_swz(r).  Over 16 (ROW 256) or 8 consecutive rows row_swz takes every
// value, so an operand read (one piece of 16 rows) meets no bank twice; its
// upper bits follow r's lowest ones, so the four rows of a transposed read's
// 16-lane group (four pieces each) cover all pieces of a row.  With the plain
// r mod 16 those four rows meet in the same four pieces.
template <int ROW>
__device__ __forceinline__ constexpr int row_swz(int r) {
  return ROW >= 256 ? ((r & 3) << 2) | ((r >> 2) & 3) : ROW == 128 ? ((r & 1) << 2) | ((r >> 1) & 3) : r & (ROW / 16 - 1);
}

}  // namespace hagdn

// k2_compact.hip -- the Reduce phase and the last Map phase of the compact path
// (compact.h; paper Sec. 2.1, operators #5 H and #6 O): GDN in bf16.
//   compact_walk_kernel  a head (or a segment of one) per workgroup, four waves of
//                        two 16-column tiles: each operand crosses the CU once for
//                        all tiles.  64 chunks: 130 us with 64 heads (a step of
//                        2 us: the tile waves' instruction stream and LDS reads),
//                        254 us with 256 (4 us: the rate of a large copy; the
//                        affine staged walk's step moved 112 KiB for 77);
//   compact_row_kernel   one or two tiles per workgroup (below);
//   compact_map_kernel   both maps of a segment, compact_scan_kernel their
//                        composition: 89 + 14 us at 1 x 32768 tokens, 16 heads,
//                        where the affine maps took 147 and every segment applied
//                        the earlier maps itself (201 us for the segment walks,
//                        130 now).
// The workgroups of a head share an XCD and its L2 (consecutive workgroup ids are
// dealt round-robin to the 8 XCDs).
#include <atomic>

#include "compact.h"

namespace hagdn {
namespace {

constexpr int kXcds = 8;
constexpr int kLdsBytes = 160 * 1024;
typedef short s16x4 __attribute__((ext_vector_type(4)));
typedef unsigned u32x2 __attribute__((ext_vector_type(2)));

// Workgroup barrier that waits only for this wave's LDS operations; the fences
// keep the compiler from moving memory accesses across it.
__device__ __forceinline__ void stage_barrier() {
  __builtin_amdgcn_s_waitcnt(0xC07F);  // lgkmcnt(0)
  __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
  __builtin_amdgcn_s_barrier();
  __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
}

// One chunk's operands in LDS, shared by the CT column tiles of a workgroup, in
// two rings: A holds key rows [64][DK] and value rows [64][VC] (swizzled,
// compact.h) and T', B the vectors and, for a walk with outputs, P' and the
// query rows.  A ring three chunks deep keeps up to two chunks in flight behind
// the one in use; at d_k = d_v = 128 with all eight tiles of a head, A three
// and B two deep take the CU's 160 KiB exactly.
// RESERVED: LDS bytes the kernel keeps for other use.
template <int DK, int CT, bool OUT, int RESERVED = 0>
struct Stage {
  static constexpr int VC = 16 * (CT < 2 ? 2 : CT);  // staged value columns: whole tile pairs
  static constexpr int KROW = DK * 2, VROW = VC * 2;
  // ring A
  static constexpr int off_k = 0;
  static constexpr int off_t = off_k + kChunk * KROW;
  static constexpr int off_v = off_t + kTriBytes;
  static constexpr int A_BYTES = off_v + kChunk * VROW;
  // ring B
  static constexpr int off_vec = 0;
  static constexpr int off_p = off_vec + kVecBytes;
  static constexpr int off_q = off_p + (OUT ? kTriBytes : 0);
  static constexpr int B_BYTES = off_q + (OUT ? kChunk * KROW : 0);
  static constexpr int NA = 3;
  static constexpr int NB = NA * A_BYTES + 3 * B_BYTES + RESERVED <= kLdsBytes ? 3 : 2;
  static constexpr int BYTES = NA * A_BYTES + NB * B_BYTES;
  static_assert(BYTES + RESERVED <= kLdsBytes, "the rings fit the LDS");
  static constexpr int A_LOADS = A_BYTES / 1024, B_LOADS = B_BYTES / 1024;
  static_assert(A_LOADS < 64, "one chunk's loads fit the vector memory counter");
};

// Four rows (4grp .. +3 of the 16 at `rows`) of one column per lane, from
// row-major LDS: lane l of a 16-lane group passes the address of row l / 4,
// column piece l % 4 (four columns), and receives column l of the four rows.
__device__ __forceinline__ s16x4 read_tr(const unsigned char *p) {
  return __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) s16x4 *)p);
}
__device__ __forceinline__ bf16x8 frag_of(s16x4 lo, s16x4 hi) {
  typedef short s16x8 __attribute__((ext_vector_type(8)));
  return __builtin_bit_cast(bf16x8, (s16x8)__builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7));
}
__device__ __forceinline__ f32x4 to_f32(s16x4 v) {
  const u32x2 u = __builtin_bit_cast(u32x2, v);
  f32x4 r;
  r[0] = __uint_as_float(u[0] << 16);
  r[1] = __uint_as_float(u[0] & 0xffff0000u);
  r[2] = __uint_as_float(u[1] << 16);
  r[3] = __uint_as_float(u[1] & 0xffff0000u);
  return r;
}
__device__ __forceinline__ bf16x8 lds_frag(const unsigned char *p) {
  return __builtin_bit_cast(bf16x8, *reinterpret_cast<const u32x4 *>(p));
}

// Range-checked stores through a buffer resource over [base, base + bytes):
// lanes whose byte offset falls outside store nothing.
__device__ __forceinline__ __amdgpu_buffer_rsrc_t rows_buffer(void *base, uint32_t bytes) {
  return __builtin_amdgcn_make_buffer_rsrc(base, (short)0, (int)bytes, 0x00020000);  // gfx9 raw buffer word 3
}

// A chunk's kChunk rows of ROW bytes, `stride` bytes apart in memory (at most
// 64 x 16 MiB: 32-bit offsets), to LDS at `dst`, 1 KiB per direct load (lane l's
// 16 bytes land at l * 16); rows past `last` repeat it.
template <int ROW>
__device__ __forceinline__ void load_rows(const unsigned char *src, uint32_t stride, int last, unsigned char *dst, int lane) {
  constexpr int P = ROW / 16, RPB = 1024 / ROW, NB = kChunk / RPB;
  constexpr int REP = RPB >= 16 ? 1 : 16 / RPB;  // the swizzle repeats every 16 rows
  const int r0 = lane / P, piece = lane % P;
  if (last >= kChunk - 1) {  // uniform: whole chunk
    uint32_t off[REP];
#pragma unroll
    for (int i = 0; i < REP; ++i) off[i] = r0 * stride + (uint32_t)((piece ^ row_swz<ROW>(i * RPB + r0)) << 4);
#pragma unroll
    for (int b = 0; b < NB; ++b) lds_copy16(src + (uint32_t)(b * RPB) * stride + off[b % REP], dst + b * 1024);
  } else {
#pragma unroll
    for (int b = 0; b < NB; ++b) {
      const int row = b * RPB + r0;
      lds_copy16(src + ((uint32_t)min(row, last) * stride + (uint32_t)((piece ^ row_swz<ROW>(row)) << 4)), dst + b * 1024);
    }
  }
}
// N consecutive KiB.
template <int N>
__device__ __forceinline__ void load_block(const unsigned char *src, unsigned char *dst, int lane) {
#pragma unroll
  for (int j = 0; j < N; ++j) lds_copy16(src + j * 1024 + lane * 16, dst + j * 1024);
}

// The chunks one workgroup walks: first block, chunks, first token, tokens from
// there to the end of the sequence.
struct Span {
  int chunk0, nch, tok0, len;
};

// Keeps a ring of D slots filled with the span's chunks: chunk c has landed
// before the barrier that opens step c, and is loaded behind the barrier that
// ends the reads of the slot's last tenant.  ROWS: the row walk's protocol of
// three barriers a step: chunk c + 1 has landed before the second barrier of
// step c, and the slot of chunk c is free behind the third.
template <int D, int LOADS, bool ROWS, typename Issue>
__device__ __forceinline__ void fill_ring(int nch, Issue issue) {
  static_assert((D - 2) * LOADS < 64, "loads left in flight fit the vector memory counter");
  if constexpr (ROWS) {
#pragma unroll
    for (int c = 0; c < D; ++c)
      if (c < nch) issue(c);
    for (int c = -1; c < nch; ++c) {  // step c; -1: before the first one
      if (c >= 0) stage_barrier();
      if (c + D - 1 < nch) wait_loads<(D - 2) * LOADS>();  // chunks c + 2 .. c + D - 1 may be in flight
      else wait_loads<0>();
      stage_barrier();
      if (c >= 0) {
        stage_barrier();
        if (c + D < nch) issue(c + D);
      }
    }
    return;
  }
#pragma unroll
  for (int c = 0; c < D - 1; ++c)
    if (c < nch) issue(c);
  for (int c = 0; c <= nch; ++c) {
    if (c + D - 2 < nch) wait_loads<(D - 2) * LOADS>();
    else wait_loads<0>();
    stage_barrier();
    if (c + D - 1 < nch) issue(c + D - 1);
  }
}

// The two loader waves of a workgroup, one per ring; values: columns col0 .. of
// the head.
template <int DK, int DV, int CT, bool OUT, bool ROWS = false, int RESERVED = 0>
__device__ __forceinline__ void load_chunks(const PrefillArgs &a, const Span &sp, int h, int col0, unsigned char *lds,
                                            int ring, int lane) {
  using S = Stage<DK, CT, OUT, RESERVED>;
  if (sp.nch <= 0) return;
  const int hk = h / (a.Hv / a.Hqk);
  const size_t kst = (size_t)a.Hqk * DK * 2, vst = (size_t)a.Hv * DV * 2;
  const unsigned char *k0 = static_cast<const unsigned char *>(a.k) + (size_t)sp.tok0 * kst + (size_t)hk * S::KROW;
  const unsigned char *q0 = static_cast<const unsigned char *>(a.q) + (size_t)sp.tok0 * kst + (size_t)hk * S::KROW;
  const unsigned char *v0 =
      static_cast<const unsigned char *>(a.v) + (size_t)sp.tok0 * vst + ((size_t)h * DV + col0) * 2;
  const unsigned char *f0 =
      static_cast<const unsigned char *>(a.NM) + ((size_t)sp.chunk0 * a.Hv + h) * kCompactBytes;
  auto last = [&](int c) { return min(kChunk, sp.len - c * kChunk) - 1; };
  auto fac = [&](int c) { return f0 + (size_t)c * a.Hv * kCompactBytes; };
  if (ring == 0) {
    fill_ring<S::NA, S::A_LOADS, ROWS>(sp.nch, [&](int c) {
      unsigned char *st = lds + (c % S::NA) * S::A_BYTES;
      load_rows<S::KROW>(k0 + (size_t)c * kChunk * kst, (uint32_t)kst, last(c), st + S::off_k, lane);
      load_block<kTriBlocks>(fac(c), st + S::off_t, lane);
      load_rows<S::VROW>(v0 + (size_t)c * kChunk * vst, (uint32_t)vst, last(c), st + S::off_v, lane);
    });
  } else {
    fill_ring<S::NB, S::B_LOADS, ROWS>(sp.nch, [&](int c) {
      unsigned char *st = lds + S::NA * S::A_BYTES + (c % S::NB) * S::B_BYTES;
      load_block<1>(fac(c) + 2 * kTriBytes, st + S::off_vec, lane);
      if constexpr (OUT) {
        load_block<kTriBlocks>(fac(c) + kTriBytes, st + S::off_p, lane);
        load_rows<S::KROW>(q0 + (size_t)c * kChunk * kst, (uint32_t)kst, last(c), st + S::off_q, lane);
      }
    });
  }
}

// The state of two adjacent column tiles of one head in one wave, and one
// chunk step of it: H[t][rt][e] = S^T[dk_of(rt, 4grp + e)][dv_of(tile0 + t, col)].
// VALUES: the tiles take the chunks' value terms (the map of a state alone
// does not).
template <int DK, int DV, int CT, bool OUT, bool VALUES>
struct TileWalk {
  using S = Stage<DK, CT, OUT>;
  static constexpr int TW = 2, RT = DK / 16, KB = DK / 32;
  f32x4 H[TW][RT];
  int lane, col, grp;
  int koff[KB];      // natural key / query operand: row col, piece 4kb + grp
  int ktoff[KB];     // transposed key operand: row 4grp + col / 4, piece 4 (rt / 2) + col % 4
  int voff;          // transposed value tile pair of this wave (first tile of the pair)

  __device__ __forceinline__ void init(int tile_in_wg) {
    lane = threadIdx.x & 63;
    col = lane & 15;
    grp = lane >> 4;
    const int tr = 4 * grp + (col >> 2);
#pragma unroll
    for (int kb = 0; kb < KB; ++kb) {
      koff[kb] = col * S::KROW + (((4 * kb + grp) ^ row_swz<S::KROW>(col)) << 4);
      ktoff[kb] = tr * S::KROW + (((4 * kb + (col & 3)) ^ row_swz<S::KROW>(tr)) << 4);
    }
    voff = tr * S::VROW + (((4 * (tile_in_wg >> 1) + (col & 3)) ^ row_swz<S::VROW>(tr)) << 4);
  }

  // Operand groups of one chunk, in the order the step consumes them: four K
  // k-blocks, Q k-blocks, T', Q k-blocks, K^T in quarters, P'.  Each group is
  // read from LDS while the group before it is multiplied.
  bf16x8 f[2][8];
  __device__ __forceinline__ void read_k(const unsigned char *st, int kb, bf16x8 (&d)[8]) {
#pragma unroll
    for (int nt = 0; nt < 4; ++nt) d[nt] = lds_frag(st + S::off_k + koff[kb] + nt * 16 * S::KROW);
  }
  __device__ __forceinline__ void read_q(const unsigned char *st, int kb, bf16x8 (&d)[8]) {
#pragma unroll
    for (int nt = 0; nt < 4; ++nt) d[nt] = lds_frag(st + S::off_q + koff[kb] + nt * 16 * S::KROW);
  }
  __device__ __forceinline__ void read_tri(const unsigned char *p, bf16x8 (&d)[8]) {
#pragma unroll
    for (int j = 0; j < kTriBlocks; ++j) d[j] = lds_frag(p + lane * 16 + j * 1024);
  }
  // K^T row tiles 4q .. 4q + 3 (all RT of them for d_k = 64), tokens of k-block kb
  __device__ __forceinline__ void read_kt(const unsigned char *st, int kb, int q, bf16x8 (&d)[8]) {
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int rt = 4 * q + i;
      const unsigned char *p = st + S::off_k + ktoff[rt >> 1] + 32 * kb * S::KROW + 8 * (rt & 1);
      d[i] = frag_of(read_tr(p), read_tr(p + 16 * S::KROW));
    }
  }

  // S_c as bf16 operands.  A walk without outputs needs each k-block once and
  // rounds it as it gets there: with eight tile waves and two loaders a wave has
  // 168 registers.
  bf16x8 hb[TW][OUT ? KB : 1];
  __device__ __forceinline__ void round_state(int kb) {
#pragma unroll
    for (int t = 0; t < TW; ++t) hb[t][OUT ? kb : 0] = frag_from_acc<bf16_t>(H[t][2 * kb], H[t][2 * kb + 1]);
  }

  // The ring slots of chunk c.
  const unsigned char *st, *sb;
  __device__ __forceinline__ void slots(const unsigned char *lds, int c) {
    st = lds + __builtin_amdgcn_readfirstlane((c % S::NA) * S::A_BYTES);
    sb = lds + __builtin_amdgcn_readfirstlane(S::NA * S::A_BYTES + (c % S::NB) * S::B_BYTES);
  }
  // Before the first step: the barrier that publishes chunk 0.
  __device__ __forceinline__ void begin(const unsigned char *lds) {
    stage_barrier();
    slots(lds, 0);
    if constexpr (OUT) {
#pragma unroll
      for (int kb = 0; kb < KB; ++kb) round_state(kb);
    }
    read_k(st, 0, f[0]);
  }

  // S_c -> S_{c+1}; with OUT also the chunk's outputs, handed to store(o):
  // O^T[t][nt], token 16nt + col, columns dv_of(tile0 + t, 4grp .. +3).
  template <typename Store>
  __device__ __forceinline__ void step(const unsigned char *lds, int c, Store store) {
    const unsigned char *stv = st + S::off_v + voff;
    const float *vec = reinterpret_cast<const float *>(sb + S::off_vec);
    int cur = 0;
    f32x4 o[TW][4];
    // ---- K S_c; meanwhile the state's decay and the value rows
    f32x4 x[TW][4];
    s16x4 v[TW][4];
    const float dec = vec[3 * kChunk];
#pragma unroll
    for (int nt = 0; nt < 4; ++nt)
#pragma unroll
      for (int t = 0; t < TW; ++t) {
        x[t][nt] = zero4();
        if constexpr (OUT && VALUES) v[t][nt] = read_tr(stv + nt * 16 * S::VROW + 8 * t);
      }
#pragma unroll
    for (int kb = 0; kb < KB; ++kb) {
      if (kb + 1 < KB) read_k(st, kb + 1, f[cur ^ 1]);
      else if constexpr (OUT) read_q(sb, 0, f[cur ^ 1]);
      if constexpr (!OUT) round_state(kb);
#pragma unroll
      for (int nt = 0; nt < 4; ++nt)
#pragma unroll
        for (int t = 0; t < TW; ++t) x[t][nt] = mma(x[t][nt], f[cur][nt], hb[t][OUT ? kb : 0]);
#pragma unroll
      for (int t = 0; t < TW; ++t) {
        H[t][2 * kb] = H[t][2 * kb] * dec;
        H[t][2 * kb + 1] = H[t][2 * kb + 1] * dec;
      }
      mix<4 * TW, 3>();
      cur ^= 1;
    }
    // ---- first half of Q S_c; meanwhile X = V - Diag(ek) K S_c
    bf16x8 xf[TW][2];
    auto form_x = [&]() {
#pragma unroll
      for (int nt = 0; nt < 4; ++nt) {
        const f32x4 ek = *reinterpret_cast<const f32x4 *>(vec + 16 * nt + 4 * grp);
#pragma unroll
        for (int t = 0; t < TW; ++t) x[t][nt] = (VALUES ? to_f32(v[t][nt]) : zero4()) - ek * x[t][nt];
      }
#pragma unroll
      for (int t = 0; t < TW; ++t)
#pragma unroll
        for (int kb = 0; kb < 2; ++kb) xf[t][kb] = frag_from_acc<bf16_t>(x[t][2 * kb], x[t][2 * kb + 1]);
    };
    auto mul_q = [&](int kb) {
#pragma unroll
      for (int nt = 0; nt < 4; ++nt)
#pragma unroll
        for (int t = 0; t < TW; ++t) o[t][nt] = mma(kb == 0 ? zero4() : o[t][nt], hb[t][kb], f[cur][nt]);
    };
    if constexpr (OUT) {
      form_x();
#pragma unroll
      for (int kb = 0; kb < KB / 2; ++kb) {
        if (kb + 1 < KB / 2) read_q(sb, kb + 1, f[cur ^ 1]);
        else read_tri(st + S::off_t, f[cur ^ 1]);
        mul_q(kb);
        cur ^= 1;
      }
      mix<KB / 2 * 4 * TW, 3>();
    } else {
      read_tri(st + S::off_t, f[cur]);
      if constexpr (VALUES) {
#pragma unroll
        for (int nt = 0; nt < 4; ++nt)
#pragma unroll
          for (int t = 0; t < TW; ++t) v[t][nt] = read_tr(stv + nt * 16 * S::VROW + 8 * t);
      }
      form_x();
    }
    // ---- U = T' X
    f32x4 u[TW][4];
    if constexpr (OUT) read_q(sb, KB / 2, f[cur ^ 1]);
    else read_kt(st, 0, 0, f[cur ^ 1]);
#pragma unroll
    for (int kb = 0; kb < 2; ++kb)
#pragma unroll
      for (int nt = 2 * kb; nt < 4; ++nt)
#pragma unroll
        for (int t = 0; t < TW; ++t) u[t][nt] = mma(kb == 0 ? zero4() : u[t][nt], f[cur][tri_block(nt, kb)], xf[t][kb]);
    cur ^= 1;
    // ---- second half of Q S_c; meanwhile U and Diag(kd) U as operands
    bf16x8 uf[TW][2], ud[TW][2];
#pragma unroll
    for (int kb = 0; kb < 2; ++kb) {
      const f32x4 d0 = *reinterpret_cast<const f32x4 *>(vec + kChunk + 32 * kb + 4 * grp);
      const f32x4 d1 = *reinterpret_cast<const f32x4 *>(vec + kChunk + 32 * kb + 16 + 4 * grp);
#pragma unroll
      for (int t = 0; t < TW; ++t) {
        ud[t][kb] = frag_from_acc<bf16_t>(u[t][2 * kb] * d0, u[t][2 * kb + 1] * d1);
        if constexpr (OUT) uf[t][kb] = frag_from_acc<bf16_t>(u[t][2 * kb], u[t][2 * kb + 1]);
      }
    }
    if constexpr (OUT) {
#pragma unroll
      for (int kb = KB / 2; kb < KB; ++kb) {
        if (kb + 1 < KB) read_q(sb, kb + 1, f[cur ^ 1]);
        mul_q(kb);
        cur ^= 1;
      }
      mix<KB / 2 * 4 * TW, 3>();
      cur ^= 1;  // (the last group read nothing ahead)
    }
    // ---- O = Diag(eq) Q S_c + P' U, stored during the state update: behind the
    //      step's barrier the loaders' burst of loads fills the address unit, and
    //      a store there held its wave for a fifth of the step
    if constexpr (OUT) {
      read_tri(sb + S::off_p, f[cur ^ 1]);
#pragma unroll
      for (int nt = 0; nt < 4; ++nt) {
        const float eq = vec[2 * kChunk + 16 * nt + col];
#pragma unroll
        for (int t = 0; t < TW; ++t) o[t][nt] = o[t][nt] * eq;
      }
      cur ^= 1;
      read_kt(st, 0, 0, f[cur ^ 1]);
#pragma unroll
      for (int kb = 0; kb < 2; ++kb)
#pragma unroll
        for (int nt = 2 * kb; nt < 4; ++nt)
#pragma unroll
          for (int t = 0; t < TW; ++t) o[t][nt] = mma(o[t][nt], uf[t][kb], f[cur][tri_block(nt, kb)]);
      mix<6 * TW, 3>();
      cur ^= 1;
    }
    // ---- S_{c+1} = e^gamma_last S_c + K^T Diag(kd) U; behind the barrier the next
    //      chunk's first keys
    constexpr int NQ = RT / 4;  // row tile quarters
#pragma unroll
    for (int kb = 0; kb < 2; ++kb)
#pragma unroll
      for (int q = 0; q < NQ; ++q) {
        const bool lastg = kb == 1 && q == NQ - 1;
        if (!lastg) {
          read_kt(st, q + 1 < NQ ? kb : kb + 1, q + 1 < NQ ? q + 1 : 0, f[cur ^ 1]);
          if constexpr (OUT) {
            if (kb == 0 && q == 0) store(o);
          }
        } else {
          stage_barrier();  // chunk c + 1 has landed; every read of chunk c is done
          slots(lds, c + 1);
          read_k(st, 0, f[cur ^ 1]);
        }
#pragma unroll
        for (int i = 0; i < 4; ++i)
#pragma unroll
          for (int t = 0; t < TW; ++t) H[t][4 * q + i] = mma(H[t][4 * q + i], f[cur][i], ud[t][kb]);
        if constexpr (OUT) {
          if (kb == 1 && q > 0) {
            round_state(2 * q - 2);
            round_state(2 * q - 1);
          }
        }
        mix<4 * TW, 3>();
        cur ^= 1;
      }
    if constexpr (OUT) {
      round_state(KB - 2);
      round_state(KB - 1);
    }
    if (cur == 1) {  // the next step starts from buffer 0
#pragma unroll
      for (int i = 0; i < 4; ++i) f[0][i] = f[1][i];
    }
  }
  // Scheduling of the group just issued: N times one MFMA and V vector ALU
  // instructions, then the region ends.
  template <int N, int V>
  __device__ __forceinline__ static void mix() {
#pragma unroll
    for (int i = 0; i < N; ++i) {
      __builtin_amdgcn_sched_group_barrier(0x8, 1, 0);
      __builtin_amdgcn_sched_group_barrier(0x2, V, 0);
    }
    __builtin_amdgcn_sched_barrier(0);
  }
};

// The outputs of one chunk: tokens 16nt + col, the tile pair's eight consecutive
// columns.
__device__ __forceinline__ void store_chunk(__amdgpu_buffer_rsrc_t rsrc, int off, int step, const f32x4 (&o)[2][4]) {
#pragma unroll
  for (int nt = 0; nt < 4; ++nt)
    __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4, frag_from_acc<bf16_t>(o[0][nt], o[1][nt])), rsrc,
                                           off + nt * step, 0, 0);
}

// Head walk, state and outputs: one workgroup of d_v / 32 tile waves (two
// adjacent 16-column tiles each) and two loader waves per (sequence, value
// head), or with SEG per (segment, value head).
template <int DK, int DV, bool SINGLE, bool SEG>
__device__ __forceinline__ void head_walk(const PrefillArgs &a, int pair) {
  constexpr int TW = 2, NW = DV / 32, CT = DV / 16, RT = DK / 16;
  extern __shared__ __align__(16) unsigned char lds[];
  const int s = pair / a.Hv, h = pair % a.Hv;           // sequence or segment, value head
  int4 sg = {s, 0, 0, 0};  // {sequence, first chunk, chunks, index in sequence}
  if constexpr (SEG) sg = seg_info_at<SINGLE>(a, s);
  if (SEG && sg.x < 0) return;
  const int n = sg.x;
  const int4 si = seq_info_at<SINGLE>(a, n);  // {first chunk, chunks, start, length}
  const int2 ss = SEG ? seq_seg_at<SINGLE>(a, n) : make_int2(0, 1);  // {first segment, segments}
  const int skip = SEG ? sg.w * a.seg_chunks * kChunk : 0;           // tokens before the segment
  const Span sp = SEG ? Span{sg.y, sg.z, si.z + skip, si.w - skip} : Span{si.x, si.y, si.z, si.w};
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;

  if (wave >= NW) {
    load_chunks<DK, DV, CT, true>(a, sp, h, 0, lds, wave - NW, lane);
    return;
  }

  // ---- tile wave
  const int tile0 = wave * TW;
  TileWalk<DK, DV, CT, true, true> w;
  w.init(tile0);
  const int col = w.col, grp = w.grp;
  const size_t sbase = ((size_t)n * a.Hv + h) * DK * DV;
  if (SEG && sg.w > 0) {
    // the state entering this segment (compact_scan_kernel)
    const float *bm = a.Bseg + ((size_t)(s - 1) * a.Hv + h) * ((size_t)DK * DV);
#pragma unroll
    for (int t = 0; t < TW; ++t)
#pragma unroll
      for (int rt = 0; rt < RT; ++rt) w.H[t][rt] = load4(bm + ((size_t)((tile0 + t) * RT + rt) * 64 + lane) * 4);
  } else {
    // s0 itself only when this workgroup is its columns' only writer of
    // s_final; else the copy the segment maps made (s_final may alias s0)
    const float *src = a.s0 ? (ss.y > 1 ? a.s0c : a.s0) : nullptr;
#pragma unroll
    for (int t = 0; t < TW; ++t)
#pragma unroll
      for (int rt = 0; rt < RT; ++rt)
#pragma unroll
        for (int e = 0; e < 4; ++e)
          w.H[t][rt][e] = src ? src[sbase + (size_t)dk_of(rt, 4 * grp + e) * DV + dv_of(tile0 + t, col)] : 0.f;
  }
  if (sp.nch > 0) {
    const size_t row_bytes = (size_t)a.Hv * DV * 2;
    const __amdgpu_buffer_rsrc_t orsrc = rows_buffer(static_cast<unsigned char *>(a.o) + (size_t)sp.tok0 * row_bytes,
                                                     (uint32_t)(min(sp.len, sp.nch * kChunk) * row_bytes));
    const int orow = (col * a.Hv + h) * DV * 2 + dv_of(tile0, 4 * grp) * 2, ostep = 16 * (int)row_bytes;
    w.begin(lds);
    for (int c = 0; c < sp.nch; ++c) {
      w.step(lds, c, [&](const f32x4(&o)[TW][4]) { store_chunk(orsrc, orow + 4 * c * ostep, ostep, o); });
    }
  }
  if (a.s_final && sg.w == ss.y - 1) {
#pragma unroll
    for (int t = 0; t < TW; ++t)
#pragma unroll
      for (int rt = 0; rt < RT; ++rt)
#pragma unroll
        for (int e = 0; e < 4; ++e)
          a.s_final[sbase + (size_t)dk_of(rt, 4 * grp + e) * DV + dv_of(tile0 + t, col)] = w.H[t][rt][e];
  }
}

template <int DK, int DV, bool SINGLE, bool SEG>
__global__ __launch_bounds__(64 * (DV / 32 + 2), 1) void compact_walk_kernel(PrefillArgs a) {
  single_status<SINGLE>(a);
  head_walk<DK, DV, SINGLE, SEG>(a, blockIdx.x);
}

// ---------------------------------------------------------------------------
// Row walk: the latency form of the state walk, for calls whose column tiles do
// not outnumber the CUs much.  Four waves share TW tiles: wave w owns token tile
// w of K S, X, U and O and state row tiles w RT/4 .. of the update, so the three
// dependent products of a step are a few MFMAs each, and S, X and U pass
// between the waves as operand fragments through LDS (three barriers a step).
// A step takes ~2,000 cycles (62 us for 64 chunks), against ~3,200 for one wave
// per tile: at d_k = 128 and one tile the LDS moves ~165 KiB in it (49 staged, 66
// read as operands, 50 exchanged), 1,300 cycles at 128 bytes a clock.  Q, T' and P'
// straight to their one reader's registers (two chunks ahead, or one behind a loader
// that touched their lines) took 74 and 78 us: the waits for those loads cost more
// than the LDS bytes they save.
template <int DK, int TW>
struct RowExchange {
  static constexpr int KB = DK / 32;
  static constexpr int off_s = 0, off_x = TW * KB * 1024, off_u = off_x + TW * 2048, off_d = off_u + TW * 2048;
  static constexpr int BYTES = off_d + TW * 2048;
};

// Column tiles tg TW .. of chain `pair`; LONG: its sequence is marked as long.
template <int DK, int DV, int TW, bool SINGLE, bool SEG, bool LONG = false>
__device__ __forceinline__ void row_walk(const PrefillArgs &a, int pair, int tg) {
  constexpr int RT = DK / 16, KB = DK / 32, RPW = RT / 4;
  using X = RowExchange<DK, TW>;
  using S = Stage<DK, TW, true, X::BYTES>;
  extern __shared__ __align__(16) unsigned char lds[];
  const int s = pair / a.Hv, h = pair % a.Hv;            // sequence or segment, value head
  int4 sg = {s, 0, 0, 0};  // {sequence, first chunk, chunks, index in sequence}
  if constexpr (SEG) sg = seg_info_at<SINGLE>(a, s);
  if (SEG && sg.x < 0) return;
  const int n = sg.x;
  int4 si = seq_info_at<SINGLE>(a, n);  // {first chunk, chunks, start, length}
  if constexpr (LONG) si.x &= ~kLongMark;
  const int2 ss = SEG ? seq_seg_at<SINGLE>(a, n) : make_int2(0, 1);  // {first segment, segments}
  const int skip = SEG ? sg.w * a.seg_chunks * kChunk : 0;           // tokens before the segment
  const Span sp = SEG ? Span{sg.y, sg.z, si.z + skip, si.w - skip} : Span{si.x, si.y, si.z, si.w};
  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
  const int tile0 = tg * TW;
  if (w >= 4) {
    load_chunks<DK, DV, TW, true, true, X::BYTES>(a, sp, h, 32 * (tile0 >> 1), lds, w - 4, lane);
    return;
  }
  const int col = lane & 15, grp = lane >> 4;
  f32x4 H[TW][RPW];  // rows dk_of(w RPW + i, 4grp + e)
  const size_t sbase = ((size_t)n * a.Hv + h) * DK * DV;
  if (SEG && sg.w > 0) {
    // the state entering this segment (compact_scan_kernel)
    const float *bm = a.Bseg + ((size_t)(s - 1) * a.Hv + h) * ((size_t)DK * DV);
#pragma unroll
    for (int t = 0; t < TW; ++t)
#pragma unroll
      for (int i = 0; i < RPW; ++i)
        H[t][i] = load4(bm + ((size_t)((tile0 + t) * RT + w * RPW + i) * 64 + lane) * 4);
  } else {
    // s0 itself only where one workgroup reads and writes its columns; else the
    // copy the segment maps made (s_final may alias s0)
    const float *src = SEG && ss.y > 1 && a.s0 ? a.s0c : a.s0;
#pragma unroll
    for (int t = 0; t < TW; ++t)
#pragma unroll
      for (int i = 0; i < RPW; ++i)
#pragma unroll
        for (int e = 0; e < 4; ++e)
          H[t][i][e] = src ? src[sbase + (size_t)dk_of(w * RPW + i, 4 * grp + e) * DV + dv_of(tile0 + t, col)] : 0.f;
  }

  // LDS addresses, from a slot's base: key / query rows of token tile w, the
  // transposed keys of this wave's row tiles, the transposed values
  int koff[KB], ktoff[RPW];
  const int tr = 4 * grp + (col >> 2);
#pragma unroll
  for (int kb = 0; kb < KB; ++kb)
    koff[kb] = (16 * w + col) * S::KROW + (((4 * kb + grp) ^ row_swz<S::KROW>(col)) << 4);
#pragma unroll
  for (int i = 0; i < RPW; ++i) {
    const int rt = w * RPW + i;
    ktoff[i] = tr * S::KROW + (((4 * (rt >> 1) + (col & 3)) ^ row_swz<S::KROW>(tr)) << 4) + 8 * (rt & 1);
  }
  const int voff = (16 * w + tr) * S::VROW + (((col & 3) ^ row_swz<S::VROW>(16 * w + tr)) << 4) + (TW == 1 ? 8 * (tile0 & 1) : 0);
  const bool low = w >= 2;  // token tiles 2, 3 also meet the triangles' second k-block
  const int tri0 = tri_block(w, 0) * 1024 + lane * 16, tri1 = low ? tri0 + 1024 : tri0;
  unsigned char *xch = lds + S::BYTES;
  unsigned char *xs = xch + X::off_s + lane * 16, *xx = xch + X::off_x + lane * 16, *xu = xch + X::off_u + lane * 16,
                *xd = xch + X::off_d + lane * 16;
  const int half = (w >> 1) * 1024 + 8 * (w & 1);  // this token tile's half of a fragment
  auto put_half = [](unsigned char *p, f32x4 v) {
    *reinterpret_cast<u32x2 *>(p) = __builtin_bit_cast(u32x2, __builtin_convertvector(v, bf16x4));
  };
  const bf16x8 zero = zero_frag<bf16_t>();

  const size_t row_bytes = (size_t)a.Hv * DV * 2;
  const __amdgpu_buffer_rsrc_t orsrc =
      rows_buffer(static_cast<unsigned char *>(a.o) + (size_t)sp.tok0 * row_bytes,
                  (uint32_t)((SEG ? min(sp.len, sp.nch * kChunk) : sp.len) * row_bytes));
  int ooff = ((16 * w + col) * a.Hv + h) * DV * 2 + dv_of(tile0, 4 * grp) * 2;
  // ---- operands of chunk c, each read behind the barrier after its last use
  bf16x8 kf[KB], qf[KB], tf[2], pf[2], kt[RPW][2];
  s16x4 v[TW];
  f32x4 ek;
  auto slot_a = [&](int c) { return lds + __builtin_amdgcn_readfirstlane((c % S::NA) * S::A_BYTES); };
  auto slot_b = [&](int c) {
    return lds + __builtin_amdgcn_readfirstlane(S::NA * S::A_BYTES + (c % S::NB) * S::B_BYTES);
  };
  auto read_keys = [&](int c) {
    const unsigned char *st = slot_a(c);
#pragma unroll
    for (int kb = 0; kb < KB; ++kb) kf[kb] = lds_frag(st + S::off_k + koff[kb]);
#pragma unroll
    for (int t = 0; t < TW; ++t) v[t] = read_tr(st + S::off_v + voff + 8 * t);
    ek = *reinterpret_cast<const f32x4 *>(slot_b(c) + S::off_vec + (16 * w + 4 * grp) * 4);
  };
  auto read_queries = [&](int c) {
    const unsigned char *sb = slot_b(c);
#pragma unroll
    for (int kb = 0; kb < KB; ++kb) qf[kb] = lds_frag(sb + S::off_q + koff[kb]);
  };
  auto put_state = [&]() {
#pragma unroll
    for (int t = 0; t < TW; ++t) {
      if constexpr (RPW == 2) {
        *reinterpret_cast<u32x4 *>(xs + (t * KB + w) * 1024) =
            __builtin_bit_cast(u32x4, frag_from_acc<bf16_t>(H[t][0], H[t][1]));
      } else {
        put_half(xs + t * KB * 1024 + half, H[t][0]);
      }
    }
  };
  if (sp.nch > 0) {
    stage_barrier();  // chunk 0 has landed
    read_keys(0);
    read_queries(0);
    put_state();
  }
  for (int c = 0; c < sp.nch; ++c) {
    const unsigned char *st = slot_a(c), *sb = slot_b(c);
    const float *vec = reinterpret_cast<const float *>(sb + S::off_vec);
    stage_barrier();  // S_c is there
    bf16x8 hb[TW][KB];
#pragma unroll
    for (int kb = 0; kb < KB; ++kb)
#pragma unroll
      for (int t = 0; t < TW; ++t) hb[t][kb] = lds_frag(xs + (t * KB + kb) * 1024);
    __builtin_amdgcn_sched_barrier(0);
    tf[0] = lds_frag(st + S::off_t + tri0);
    tf[1] = lds_frag(st + S::off_t + tri1);
    const f32x4 kd = *reinterpret_cast<const f32x4 *>(vec + kChunk + 16 * w + 4 * grp);
    const float dec = vec[3 * kChunk], eq = vec[2 * kChunk + 16 * w + col];
    // ---- X = V - Diag(ek) K S_c (two chains over the k-blocks)
#pragma unroll
    for (int t = 0; t < TW; ++t) {
      f32x4 x0 = zero4(), x1 = zero4();
#pragma unroll
      for (int kb = 0; kb < KB; kb += 2) {
        x0 = mma(x0, kf[kb], hb[t][kb]);
        x1 = mma(x1, kf[kb + 1], hb[t][kb + 1]);
      }
      put_half(xx + t * 2048 + half, to_f32(v[t]) - ek * (x0 + x1));
    }
    __builtin_amdgcn_sched_barrier(0);
    // ---- Q S_c and the decay, while X crosses
    f32x4 o[TW];
#pragma unroll
    for (int t = 0; t < TW; ++t) {
      f32x4 q0 = zero4(), q1 = zero4();
#pragma unroll
      for (int kb = 0; kb < KB; kb += 2) {
        q0 = mma(q0, hb[t][kb], qf[kb]);
        q1 = mma(q1, hb[t][kb + 1], qf[kb + 1]);
      }
      o[t] = q0 + q1;
    }
    stage_barrier();  // X is there, and chunk c + 1 has landed
    // ---- U = T' X
    bf16x8 xf[TW][2];
#pragma unroll
    for (int t = 0; t < TW; ++t)
#pragma unroll
      for (int kb = 0; kb < 2; ++kb) xf[t][kb] = lds_frag(xx + (2 * t + kb) * 1024);
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int i = 0; i < RPW; ++i)
#pragma unroll
      for (int kb = 0; kb < 2; ++kb) {
        const unsigned char *p = st + S::off_k + ktoff[i] + 32 * kb * S::KROW;
        kt[i][kb] = frag_of(read_tr(p), read_tr(p + 16 * S::KROW));
      }
    pf[0] = lds_frag(sb + S::off_p + tri0);
    pf[1] = lds_frag(sb + S::off_p + tri1);
    if (!low) tf[1] = pf[1] = zero;
#pragma unroll
    for (int t = 0; t < TW; ++t) {
      f32x4 u = mma(zero4(), tf[0], xf[t][0]);
      u = mma(u, tf[1], xf[t][1]);
      put_half(xd + t * 2048 + half, u * kd);
      put_half(xu + t * 2048 + half, u);
    }
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int t = 0; t < TW; ++t) {
      o[t] = o[t] * eq;
#pragma unroll
      for (int i = 0; i < RPW; ++i) H[t][i] = H[t][i] * dec;
    }
    stage_barrier();  // U is there
    // ---- S_{c+1} = e^gamma_last S_c + K^T Diag(kd) U, then O = Diag(eq) Q S_c + P' U
    bf16x8 df[TW][2], uf[TW][2];
#pragma unroll
    for (int t = 0; t < TW; ++t)
#pragma unroll
      for (int kb = 0; kb < 2; ++kb) df[t][kb] = lds_frag(xd + (2 * t + kb) * 1024);
#pragma unroll
    for (int t = 0; t < TW; ++t)
#pragma unroll
      for (int kb = 0; kb < 2; ++kb) uf[t][kb] = lds_frag(xu + (2 * t + kb) * 1024);
    __builtin_amdgcn_sched_barrier(0);
    // the next chunk's operands: at d_k = 64 the keys before the update's products
    // and the queries before the outputs', at 128 all behind them (the products of a
    // step then wait for fewer reads; 64 chunks with 20 heads, either order left to
    // the compiler: 65-77 us against 62-73 at 64, 81 against 77 at 128)
    if constexpr (DK == 64) {
      read_keys(c + 1);
      __builtin_amdgcn_sched_barrier(0);
    }
#pragma unroll
    for (int kb = 0; kb < 2; ++kb)
#pragma unroll
      for (int t = 0; t < TW; ++t)
#pragma unroll
        for (int i = 0; i < RPW; ++i) H[t][i] = mma(H[t][i], kt[i][kb], df[t][kb]);
    put_state();
    __builtin_amdgcn_sched_barrier(0);
    if constexpr (DK == 64) {
      read_queries(c + 1);
      __builtin_amdgcn_sched_barrier(0);
    }
#pragma unroll
    for (int t = 0; t < TW; ++t) {
      o[t] = mma(o[t], uf[t][0], pf[0]);
      o[t] = mma(o[t], uf[t][1], pf[1]);
    }
    if constexpr (DK != 64) {
      read_keys(c + 1);
      read_queries(c + 1);
      __builtin_amdgcn_sched_barrier(0);
    }
    if constexpr (TW == 2) {
      __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4, frag_from_acc<bf16_t>(o[0], o[1])), orsrc, ooff, 0,
                                             0);
    } else {
      __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(u32x2, __builtin_convertvector(o[0], bf16x4)), orsrc, ooff,
                                            0, 0);
    }
    ooff += kChunk * (int)row_bytes;
  }
  if (a.s_final && sg.w == ss.y - 1) {
#pragma unroll
    for (int t = 0; t < TW; ++t)
#pragma unroll
      for (int i = 0; i < RPW; ++i)
#pragma unroll
        for (int e = 0; e < 4; ++e)
          a.s_final[sbase + (size_t)dk_of(w * RPW + i, 4 * grp + e) * DV + dv_of(tile0 + t, col)] = H[t][i][e];
  }
}

// Workgroup b of a launch of NG workgroups per chain: the chain and its part.  The
// workgroups of a head share an XCD.
template <int NG>
__device__ __forceinline__ int chain_of(int b) {
  return (b / kXcds / NG) * kXcds + b % kXcds;
}
template <int NG>
__device__ __forceinline__ int part_of(int b) {
  return (b / kXcds) % NG;
}

template <int DK, int DV, int TW, bool SINGLE, bool SEG>
__global__ __launch_bounds__(64 * 6, 1) void compact_row_kernel(PrefillArgs a) {
  constexpr int NG = DV / (16 * TW);
  single_status<SINGLE>(a);
  const int b = blockIdx.x, pair = chain_of<NG>(b);
  if (pair >= (SEG ? a.max_segs : a.N) * a.Hv) return;  // uniform for the workgroup
  row_walk<DK, DV, TW, SINGLE, SEG>(a, pair, part_of<NG>(b));
}

// Whole chains of a batch that has more column tiles than CUs and may hold chains much
// longer than the others (prefill.h, is_long_chain): the long ones' tiles first, one to
// a workgroup (row walk), then the other chains as a launch without them would walk
// them, in tile pairs (PAIR) or whole heads.  The chunk index kernel left the long
// sequences in a.ovl and a mark in their entries, so a workgroup reads nothing more
// than the plain walk does (with the count read first by every workgroup, 201 short
// sequences of 32 heads took 7 % longer).  Walked like the others, one 4,096-token
// chain among empty ones took 78 (pairs) or 122 us at d = 128 and 58 or 84 at 64, for
// the row walk's 60 and 50; calls with such a chain were up to 1.48 times as long as
// with the affine factors.
template <int DK, int DV, bool PAIR>
__global__ __launch_bounds__(64 * 6, 1) void compact_mixed_kernel(PrefillArgs a) {
  constexpr int NT = DV / 16, NG = PAIR ? NT / 2 : 1;
  const int b = blockIdx.x;
  if (b < a.long_rows) {
    const int i = chain_of<NT>(b);
    if (i >= a.ovl[0] * a.Hv) return;  // uniform for the workgroup, as every return here
    row_walk<DK, DV, 1, false, false, true>(a, a.ovl[1 + i / a.Hv] * a.Hv + i % a.Hv, part_of<NT>(b));
    return;
  }
  const int pair = chain_of<NG>(b - a.long_rows);
  if (pair >= a.N * a.Hv || a.seq_info[pair / a.Hv].x < 0) return;
  if constexpr (PAIR) {
    row_walk<DK, DV, 2, false, false>(a, pair, part_of<NG>(b - a.long_rows));
  } else {
    if (threadIdx.x >= 64 * (DV / 32 + 2)) return;  // whole waves (ended waves do not count at a barrier)
    head_walk<DK, DV, false, false>(a, pair);
  }
}

// Segment maps (the Chunk-Seg-Seg path, paper Sec. 4): S^T_out = A S^T_in +
// B_seg over a segment's chunks.  A is the walk of the d_k x d_k identity
// without the chunks' values, B_seg the walk of a zero state with them (the
// first segment's starts from the initial state and has no A, prefill.h).  One
// workgroup per (segment, value head), for segments that another one of the
// same sequence follows: d_k / 32 tile waves for A and d_v / 32 for B_seg (two
// tiles each) share the rings, so a chunk's keys cross the CU once for both
// maps, and every SIMD has two tile waves to hide each other's latency.  A
// leaves as bf16 operand blocks of the walk's own orders (row tile rt, k-block
// kb: lane (col, grp), slot j = A[dk_of(rt, col)][32kb + 8grp + j]), B_seg in
// fp32 as the accumulators stand.
template <int DK, int DV>
struct MapWaves {
  static constexpr int A = DK / 32, B = DV / 32, ALL = A + B + 2;
};

template <int DK, int DV, bool APART>
__device__ __forceinline__ void map_tiles(const PrefillArgs &a, int s, int h, int4 sg, int wave, unsigned char *lds) {
  constexpr int RT = DK / 16, KB = DK / 32, NT = DV / 16;
  const int lane = threadIdx.x & 63;
  const int nch = sg.z;
  TileWalk<DK, DV, NT, false, !APART> w;
  w.init(APART ? 0 : wave * 2);
  const int col = w.col, grp = w.grp;
  const bool from_s0 = !APART && sg.w == 0 && a.s0;
  const size_t sbase = ((size_t)sg.x * a.Hv + h) * DK * DV;
#pragma unroll
  for (int t = 0; t < 2; ++t)
#pragma unroll
    for (int rt = 0; rt < RT; ++rt)
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const int row = dk_of(rt, 4 * grp + e);
        float x = APART && row == 32 * wave + 16 * t + col ? 1.f : 0.f;
        if (from_s0) {  // uniform for the workgroup
          const size_t i = sbase + (size_t)row * DV + dv_of(2 * wave + t, col);
          x = a.s0[i];
          a.s0c[i] = x;
        }
        w.H[t][rt][e] = x;
      }
  if (nch > 0) {
    w.begin(lds);
    for (int c = 0; c < nch; ++c) {
      w.step(lds, c, [](const f32x4(&)[2][4]) {});
    }
  }
  stage_barrier();  // every read of the rings is done
  const size_t mblk = (size_t)s * a.Hv + h;
  if constexpr (!APART) {
    float *bm = a.Bseg + mblk * ((size_t)DK * DV);
#pragma unroll
    for (int t = 0; t < 2; ++t)
#pragma unroll
      for (int rt = 0; rt < RT; ++rt)
        *reinterpret_cast<f32x4 *>(bm + ((size_t)((2 * wave + t) * RT + rt) * 64 + lane) * 4) = w.H[t][rt];
    stage_barrier();
  } else {
    // row-major in LDS (rows padded by 8 elements), then operand blocks
    constexpr int LD = DK + 8;
    bf16_t *sA = reinterpret_cast<bf16_t *>(lds);
#pragma unroll
    for (int t = 0; t < 2; ++t)
#pragma unroll
      for (int rt = 0; rt < RT; ++rt)
#pragma unroll
        for (int e = 0; e < 4; ++e)
          sA[dk_of(rt, 4 * grp + e) * LD + 32 * wave + 16 * t + col] = f32_to_bf16(w.H[t][rt][e]);
    stage_barrier();
    bf16_t *am = static_cast<bf16_t *>(a.Aseg) + mblk * ((size_t)DK * DK);
    for (int q = wave; q < RT * KB; q += MapWaves<DK, DV>::A)
      store_frag_at(am + ((size_t)q * 64 + lane) * 8, load_frag(sA + dk_of(q / KB, col) * LD + 32 * (q % KB), grp));
  }
}

template <int DK, int DV, bool SINGLE>
__global__ __launch_bounds__(64 * (DK / 32 + DV / 32 + 2), 1) void compact_map_kernel(PrefillArgs a) {
  using MW = MapWaves<DK, DV>;
  extern __shared__ __align__(16) unsigned char lds[];
  const int pair = blockIdx.x;  // (segment, value head)
  const int s = pair / a.Hv, h = pair % a.Hv;
  const int4 sg = seg_info_at<SINGLE>(a, s);  // {sequence, first chunk, chunks, index in sequence}
  if (sg.x < 0) return;
  if (sg.w == seq_seg_at<SINGLE>(a, sg.x).y - 1) return;  // the last segment's map is never applied
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  if (wave >= MW::A + MW::B) {
    const int4 si = seq_info_at<SINGLE>(a, sg.x);
    const int skip = sg.w * a.seg_chunks * kChunk;
    load_chunks<DK, DV, DV / 16, false>(a, Span{sg.y, sg.z, si.z + skip, si.w - skip}, h, 0, lds, wave - MW::A - MW::B,
                                        threadIdx.x & 63);
  } else if (wave >= MW::A) {
    map_tiles<DK, DV, false>(a, s, h, sg, wave - MW::A, lds);
  } else if (sg.w > 0) {
    map_tiles<DK, DV, true>(a, s, h, sg, wave, lds);
  }  // else: the first segment has no A (ended waves do not count at a barrier)
}

// The states entering the segments: S_{j+1} = A_j S_j + B_j, j = 1 .. of each
// sequence, in place of the maps' B_j (B_0 is S_1 already).  One workgroup of
// d_k / 32 waves per (sequence, value head, 16-column tile); wave w owns state
// rows of tiles 2w, 2w + 1 and publishes them as one operand fragment per step.
// Walked by every segment from the start instead, these products took 5 us a
// map and 14 maps for the last segment of 16.
template <int DK, int DV, bool SINGLE>
__global__ __launch_bounds__(64 * (DK / 32), 1) void compact_scan_kernel(PrefillArgs a) {
  constexpr int RT = DK / 16, KB = DK / 32, NT = DV / 16, D = 3;  // maps in flight
  __shared__ bf16x8 xch[2][KB][64];
  const int b = blockIdx.x;
  const int pair = (b / kXcds / NT) * kXcds + b % kXcds, tile = (b / kXcds) % NT;
  if (pair >= a.N * a.Hv) return;  // uniform for the workgroup
  const int n = pair / a.Hv, h = pair % a.Hv;
  const int2 ss = seq_seg_at<SINGLE>(a, n);  // {first segment, segments}
  const int maps = ss.y - 2;                 // of segments 1 .. ss.y - 2
  if (maps <= 0) return;
  const int w = threadIdx.x >> 6, lane = threadIdx.x & 63;
  auto bseg = [&](int j) {  // B of the sequence's segment j, this wave's tiles
    return a.Bseg + ((size_t)(ss.x + j) * a.Hv + h) * ((size_t)DK * DV) + ((size_t)(tile * RT + 2 * w) * 64 + lane) * 4;
  };
  f32x4 H[2] = {load4(bseg(0)), load4(bseg(0) + 256)};
  struct Map {
    bf16x8 m[2][KB];
    f32x4 b[2];
  } ring[D];
  auto fetch = [&](Map &r, int j) {
    j = min(j, maps);  // segments 1 .. maps
    const bf16_t *am =
        static_cast<const bf16_t *>(a.Aseg) + ((size_t)(ss.x + j) * a.Hv + h) * ((size_t)DK * DK) + lane * 8;
#pragma unroll
    for (int i = 0; i < 2; ++i) {
#pragma unroll
      for (int kb = 0; kb < KB; ++kb) r.m[i][kb] = load_frag_at(am + (size_t)((2 * w + i) * KB + kb) * 512);
      r.b[i] = load4(bseg(j) + 256 * i);
    }
  };
  auto step = [&](Map &r, int j) {
    xch[j & 1][w][lane] = frag_from_acc<bf16_t>(H[0], H[1]);
    __syncthreads();
#pragma unroll
    for (int i = 0; i < 2; ++i) H[i] = r.b[i];
#pragma unroll
    for (int kb = 0; kb < KB; ++kb) {
      const bf16x8 f = xch[j & 1][kb][lane];
#pragma unroll
      for (int i = 0; i < 2; ++i) H[i] = mma(H[i], r.m[i][kb], f);
    }
#pragma unroll
    for (int i = 0; i < 2; ++i) store4(bseg(j) + 256 * i, H[i]);
  };
#pragma unroll
  for (int u = 0; u < D; ++u) fetch(ring[u], 1 + u);
  for (int j = 1; j <= maps; j += D) {
#pragma unroll
    for (int u = 0; u < D; ++u)
      if (j + u <= maps) {  // uniform for the workgroup
        step(ring[u], j + u);
        fetch(ring[u], j + u + D);
      }
  }
}

constexpr int kMaxDevices = 64;

// Raises a kernel's dynamic LDS limit to `lds` bytes, once per device (`done`:
// the kernel's own marks).
hipError_t raise_lds(const void *kern, int lds, std::atomic<bool> (&done)[kMaxDevices]) {
  int dev = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return e;
  if (dev < 0 || dev >= kMaxDevices || !done[dev].load(std::memory_order_relaxed)) {
    if ((e = hipFuncSetAttribute(kern, hipFuncAttributeMaxDynamicSharedMemorySize, lds)) != hipSuccess) return e;
    if (dev >= 0 && dev < kMaxDevices) done[dev].store(true, std::memory_order_relaxed);
  }
  return hipSuccess;
}

template <int DK, int DV, bool SINGLE, bool SEG>
hipError_t launch_walk_t(const PrefillArgs &a, hipStream_t stream) {
  constexpr int lds = Stage<DK, DV / 16, true>::BYTES;
  const void *kern = reinterpret_cast<const void *>(&compact_walk_kernel<DK, DV, SINGLE, SEG>);
  static std::atomic<bool> done[kMaxDevices];
  hipError_t e = raise_lds(kern, lds, done);
  if (e != hipSuccess) return e;
  const long blocks = (long)(SEG ? a.max_segs : a.N) * a.Hv;
  hipLaunchKernelGGL((compact_walk_kernel<DK, DV, SINGLE, SEG>), dim3((unsigned)blocks), dim3(64 * (DV / 32 + 2)), lds,
                     stream, a);
  return hipGetLastError();
}

template <int DK, int DV, int TW, bool SINGLE, bool SEG>
hipError_t launch_row_t(const PrefillArgs &a, hipStream_t stream) {
  using X = RowExchange<DK, TW>;
  constexpr int lds = Stage<DK, TW, true, X::BYTES>::BYTES + X::BYTES;
  const void *kern = reinterpret_cast<const void *>(&compact_row_kernel<DK, DV, TW, SINGLE, SEG>);
  static std::atomic<bool> done[kMaxDevices];
  hipError_t e = raise_lds(kern, lds, done);
  if (e != hipSuccess) return e;
  const long groups = ((long)(SEG ? a.max_segs : a.N) * a.Hv + kXcds - 1) / kXcds;
  const long blocks = groups * kXcds * (DV / (16 * TW));
  hipLaunchKernelGGL((compact_row_kernel<DK, DV, TW, SINGLE, SEG>), dim3((unsigned)blocks), dim3(64 * 6), lds, stream,
                     a);
  return hipGetLastError();
}

template <int DK, int DV, bool PAIR>
hipError_t launch_mixed_t(const PrefillArgs &a, hipStream_t stream) {
  using X1 = RowExchange<DK, 1>;
  using X2 = RowExchange<DK, 2>;
  constexpr int lds1 = Stage<DK, 1, true, X1::BYTES>::BYTES + X1::BYTES;
  constexpr int lds2 = PAIR ? Stage<DK, 2, true, X2::BYTES>::BYTES + X2::BYTES : Stage<DK, DV / 16, true>::BYTES;
  constexpr int lds = lds1 > lds2 ? lds1 : lds2, NT = DV / 16;
  const void *kern = reinterpret_cast<const void *>(&compact_mixed_kernel<DK, DV, PAIR>);
  static std::atomic<bool> done[kMaxDevices];
  hipError_t e = raise_lds(kern, lds, done);
  if (e != hipSuccess) return e;
  const long rest = ((long)a.N * a.Hv + kXcds - 1) / kXcds * kXcds * (PAIR ? NT / 2 : 1);
  hipLaunchKernelGGL((compact_mixed_kernel<DK, DV, PAIR>), dim3((unsigned)(a.long_rows + rest)), dim3(64 * 6), lds, stream, a);
  return hipGetLastError();
}

template <int DK, int DV, bool SINGLE>
hipError_t launch_map_t(const PrefillArgs &a, hipStream_t stream) {
  constexpr int rings = Stage<DK, DV / 16, false>::BYTES, tr = DK * (DK + 8) * 2;
  constexpr int lds = rings > tr ? rings : tr;
  const void *kern = reinterpret_cast<const void *>(&compact_map_kernel<DK, DV, SINGLE>);
  static std::atomic<bool> done[kMaxDevices];
  hipError_t e = raise_lds(kern, lds, done);
  if (e != hipSuccess) return e;
  const long blocks = (long)a.max_segs * a.Hv;
  hipLaunchKernelGGL((compact_map_kernel<DK, DV, SINGLE>), dim3((unsigned)blocks), dim3(64 * MapWaves<DK, DV>::ALL), lds,
                     stream, a);
  if ((e = hipGetLastError()) != hipSuccess) return e;
  // a sequence of T tokens has at most this many segments; a third one needs the scan
  if (((long)a.T + kChunk - 1) / kChunk <= 2L * a.seg_chunks) return hipSuccess;
  const long groups = ((long)a.N * a.Hv + kXcds - 1) / kXcds;
  hipLaunchKernelGGL((compact_scan_kernel<DK, DV, SINGLE>), dim3((unsigned)(groups * kXcds * (DV / 16))),
                     dim3(64 * (DK / 32)), 0, stream, a);
  return hipGetLastError();
}

enum class Part { kWalk, kMaps, kSegments };

// Whole chains, or segments with SEG.  The row walk while the column tiles, one
// or two to a workgroup, fit the CUs in one round; beyond that a whole head per
// workgroup, which moves each operand once for all its tiles.  Walk of 64 chunks,
// us, row walk against the whole head: 32 heads 69 / 124 (one tile), 48 heads 90 /
// 127 and 64 heads 104 / 129 (two tiles).  Segments of 1 x 7700 tokens, us per
// call, the same way: d = 64, 1 head 42 / 48, 4 heads 47 / 52; d = 128, 1 head 57 /
// 69 (the affine kernels took 42 and 50 at d = 64).
template <int DK, int DV, bool SINGLE, bool SEG>
hipError_t launch_walks(const PrefillArgs &a, hipStream_t s) {
  const long tiles = ((long)(SEG ? a.max_segs : a.N) * a.Hv + kXcds - 1) / kXcds * kXcds * (DV / 16);
  if (tiles <= a.cus) return launch_row_t<DK, DV, 1, SINGLE, SEG>(a, s);
  if constexpr (!SINGLE && !SEG) {
    if (a.long_rows > 0)
      return tiles <= 2L * a.cus ? launch_mixed_t<DK, DV, true>(a, s) : launch_mixed_t<DK, DV, false>(a, s);
  }
  if (tiles <= 2L * a.cus) return launch_row_t<DK, DV, 2, SINGLE, SEG>(a, s);
  return launch_walk_t<DK, DV, SINGLE, SEG>(a, s);
}

template <int DK, int DV, bool SINGLE>
hipError_t launch_dims(const PrefillArgs &a, Part part, hipStream_t s) {
  if (part == Part::kMaps) return launch_map_t<DK, DV, SINGLE>(a, s);
  if (part == Part::kSegments) return launch_walks<DK, DV, SINGLE, true>(a, s);
  return launch_walks<DK, DV, SINGLE, false>(a, s);
}

template <bool SINGLE>
hipError_t launch_part(const PrefillArgs &a, Part part, hipStream_t s) {
  if (a.Dk == 64 && a.Dv == 64) return launch_dims<64, 64, SINGLE>(a, part, s);
  if (a.Dk == 64 && a.Dv == 128) return launch_dims<64, 128, SINGLE>(a, part, s);
  if (a.Dk == 128 && a.Dv == 64) return launch_dims<128, 64, SINGLE>(a, part, s);
  return launch_dims<128, 128, SINGLE>(a, part, s);
}

hipError_t launch(const PrefillArgs &a, Part part, hipStream_t s) {
  return a.single ? launch_part<true>(a, part, s) : launch_part<false>(a, part, s);
}

}  // namespace

hipError_t launch_compact_walk(const PrefillArgs &a, hipStream_t s) { return launch(a, Part::kWalk, s); }
hipError_t launch_compact_maps(const PrefillArgs &a, hipStream_t s) { return launch(a, Part::kMaps, s); }
hipError_t launch_compact_segments(const PrefillArgs &a, hipStream_t s) { return launch(a, Part::kSegments, s); }

}  // namespace hagdn

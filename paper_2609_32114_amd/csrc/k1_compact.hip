// k1_compact.hip -- the first Map phase for the compact path (compact.h): the
// parts of operators #1-#3 (paper Sec. 2.1: Gate, KKT, Solve) that the state
// walk cannot redo per column tile, T' = T Diag(b), P' and the decay vectors,
// for GDN in bf16.  One workgroup of four waves per (chunk, value head).
//
// The affine chunk-local kernel (k1_chunk_local.hip) is bound by its factor
// stores on long calls (96 KiB written per 48 KiB read) and by its dependent
// phases on short ones.  This one reads keys and queries only, writes 13 KiB,
// and drops operator #4 and the reduce-side products; what is left is a chain
// of load, two 64 x 64 products, and the triangular solve.
//
// Wave i computes row block i of A and P transposed (token r = 16i + col per
// lane column), so the P accumulators are P' operand fragments as they stand.
// It then inverts its diagonal block and solves column block i of T
// (chunk_item.h), whose transposed blocks are halves of T' operand blocks.
// Four barriers in all (keys staged, and free again, A and the T_ii published,
// and with raw keys their L2 factors).  Five workgroups share a CU, as many as the
// registers allow (under 96).  A takes the keys' place in LDS: 17 KiB a workgroup;
// with a place of its own, 33 KiB, at four per CU and one barrier less, the last
// three calls below took 162-183, 44 and 90.  us, affine kernel against this one: one
// block per CU 19.7 / 8; 1,024
// blocks 47.5 / 15.6; 17,408 with two heads per key head 604-669 / 148-167; 3,200
// raw ones 134-145 / 42; 8,192 with 1 x 32768 tokens 293-326 / 76-87 (411 MB, the
// rate of a large copy).  Six per CU spill.
#include "chunk_item.h"
#include "compact.h"

namespace hagdn {
namespace {

constexpr int kThreads = 256;

template <int DK, bool PRE>
__global__ __launch_bounds__(kThreads, 5) void chunk_compact_kernel(PrefillArgs a) {
  constexpr int KB = DK / 32, ROW = DK * 2, PIECES = ROW / 16;
  constexpr int RPB = 1024 / ROW;       // rows of one 1 KiB load
  constexpr int LPW = kChunk / RPB / 4; // loads per wave
  // keys until op #2 is done with them, then A (strictly lower blocks) and T_ii
  // (diagonal blocks): 17 KiB a workgroup with the token vectors
  constexpr int kTile = kChunk * ROW > kChunk * kChunk * 4 ? kChunk * ROW : kChunk * kChunk * 4;
  __shared__ __align__(16) unsigned char sK[kTile];
  float *sA = reinterpret_cast<float *>(sK);
  __shared__ double sGam[kChunk];
  __shared__ __align__(16) float sBeta[kChunk], sNk[kChunk];
  const LocalItem cur = local_item(a, blockIdx.x);
  if (cur.len <= 0) return;  // past the last chunk: uniform for the workgroup
  const int tid = threadIdx.x, lane = tid & 63, col = lane & 15, grp = lane >> 4;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int h = cur.h, start = cur.start, len = cur.len, last = len - 1;
  const int hk = h / (a.Hv / a.Hqk);
  const size_t qk_row = (size_t)a.Hqk * DK;
  const bf16_t *kbase = static_cast<const bf16_t *>(a.k) + (size_t)start * qk_row + (size_t)hk * DK;
  const bf16_t *qbase = static_cast<const bf16_t *>(a.q) + (size_t)start * qk_row + (size_t)hk * DK;

  // ---- loads: keys to LDS (rows past the chunk's end repeat its last row:
  //      their b is 0), this lane's query row and token as operands
#pragma unroll
  for (int u = 0; u < LPW; ++u) {
    const int b = wave * LPW + u, r = b * RPB + lane / PIECES;
    const int piece = (lane % PIECES) ^ row_swz<ROW>(r);
    lds_copy16(kbase + (size_t)min(r, last) * qk_row + piece * 8, sK + b * 1024);
  }
  const int r = 16 * wave + col;  // the token of this lane's column of A^T and P^T
  bf16x8 qf[KB];
#pragma unroll
  for (int kb = 0; kb < KB; ++kb) qf[kb] = load_frag(qbase + (size_t)min(r, last) * qk_row + kb * 32, grp);
  if (wave == 0) {
    const size_t at = (size_t)(start + min(lane, last)) * a.Hv + h;
    const float graw = a.g[at], braw = a.beta[at];
    const float gx = (PRE && (a.pre & kPreGateSoftplus)) ? neg_softplus(graw) : graw;
    const float bx = (PRE && (a.pre & kPreBetaSigmoid)) ? sigmoid(braw) : braw;
    sBeta[lane] = lane < len ? bx : 0.f;
    // op #1 in fp64: gamma reaches thousands where gates are near 0, and the
    // decays are exponentials of its differences
    double x = lane < len ? gx : 0.f;
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) {
      const double y = __shfl_up(x, off);
      if (lane >= off) x += y;
    }
    sGam[lane] = x;
  }
  wait_loads<0>();
  __syncthreads();

  auto key_frag = [&](int row, int kb) {  // keys' channels 32kb + 8grp .. +7 of a token row
    return __builtin_bit_cast(bf16x8, *reinterpret_cast<const u32x4 *>(
        sK + row * ROW + (((4 * kb + grp) ^ row_swz<ROW>(row)) << 4)));
  };
  bf16x8 kr[KB];
#pragma unroll
  for (int kb = 0; kb < KB; ++kb) kr[kb] = key_frag(r, kb);
  float nk = 1.f, nq = 1.f;  // L2 factors of token r's key and query
  if constexpr (PRE) {
    if (a.pre & kPreQkNorm) {
      float ks = 0.f, qs = 0.f;
#pragma unroll
      for (int kb = 0; kb < KB; ++kb)
#pragma unroll
        for (int j = 0; j < 8; ++j) {
          const float x = frag_elem(kr[kb], j), y = frag_elem(qf[kb], j);
          ks += x * x;
          qs += y * y;
        }
      ks += __shfl_xor(ks, 16);
      ks += __shfl_xor(ks, 32);
      qs += __shfl_xor(qs, 16);
      qs += __shfl_xor(qs, 32);
      nk = inv_l2(ks);
      nq = inv_l2(qs);
      if (grp == 0) sNk[r] = nk;
      __syncthreads();
    }
  }
  const double gr = sGam[r];
  const float br = sBeta[r] * nk;

  // ---- op #2, transposed: A[r][s] and P[r][s], s = 16j + 4grp + e, j <= wave
  f32x4 accA[4], accP[4];
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    accA[j] = accP[j] = zero4();
    if (j <= wave) {  // uniform for the wave
#pragma unroll
      for (int kb = 0; kb < KB; ++kb) {
        const bf16x8 ks = key_frag(16 * j + col, kb);
        accA[j] = mma(accA[j], ks, kr[kb]);
        accP[j] = mma(accP[j], ks, qf[kb]);
      }
      f32x4 ns = {1.f, 1.f, 1.f, 1.f};
      if constexpr (PRE) {
        if (a.pre & kPreQkNorm) ns = *reinterpret_cast<const f32x4 *>(sNk + 16 * j + 4 * grp);
      }
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const int s = 16 * j + 4 * grp + e;
        float dec = s <= r ? __expf((float)(gr - sGam[s])) : 0.f;
        if constexpr (PRE) dec *= ns[e];
        accA[j][e] = (s < r && r < len) ? br * accA[j][e] * dec : 0.f;
        accP[j][e] = s <= r ? accP[j][e] * dec * (a.scale * nq) : 0.f;
      }
    }
  }

  __syncthreads();  // every wave is done with the keys
#pragma unroll
  for (int j = 0; j < 3; ++j)
    if (j < wave) *reinterpret_cast<f32x4 *>(sA + swz<float, kChunk>(r, 16 * j + 4 * grp)) = accA[j];

  // ---- op #3, diagonal block: column `col` of (I + A_ii)^-1 by forward
  //      substitution; A_ii[x][y] sits in lane x + 16 (y / 4), element y % 4
  f32x4 ad = accA[0];
#pragma unroll
  for (int j = 1; j < 4; ++j)
    if (j == wave) ad = accA[j];
  const f32x4 tj = invert_unit_lower(ad);
#pragma unroll
  for (int e = 0; e < 4; ++e) sA[swz<float, kChunk>(16 * wave + 4 * grp + e, 16 * wave + col)] = tj[e];

  // ---- P' operand blocks (row tile wave) and the vectors
  unsigned char *out = static_cast<unsigned char *>(a.NM) + ((size_t)cur.c * a.Hv + h) * kCompactBytes;
#pragma unroll
  for (int kb = 0; kb < 2; ++kb)
    if (kb <= (wave >> 1))
      store_frag_at(reinterpret_cast<bf16_t *>(out + kTriBytes + tri_block(wave, kb) * 1024) + lane * 8,
                    frag_from_acc<bf16_t>(accP[2 * kb], accP[2 * kb + 1]));
  if (grp == 0) {
    float *vec = reinterpret_cast<float *>(out + 2 * kTriBytes);
    const double gl = sGam[kChunk - 1];
    const float eg = __expf((float)gr);
    vec[r] = nk * eg;
    vec[kChunk + r] = nk * __expf((float)(gl - gr));
    vec[2 * kChunk + r] = a.scale * nq * eg;
    vec[3 * kChunk + r] = __expf((float)gl);
  }
  __syncthreads();

  // ---- op #3, column block j = wave of T, and its T' halves: slots 4 (j & 1)
  //      .. +3 of the blocks (i, j / 2), lane (col, grp) = T[16i + col][16j + 4grp + e] b_s
  const f32x4 bs = *reinterpret_cast<const f32x4 *>(sBeta + 16 * wave + 4 * grp);
  auto put = [&](int i, f32x4 t) {
    store4(reinterpret_cast<bf16_t *>(out + tri_block(i, wave >> 1) * 1024) + lane * 8 + 4 * (wave & 1), t * bs);
  };
  put(wave, block_rows(sA, wave, wave));
  if (wave & 1) put(wave - 1, zero4());  // the block above the diagonal
  solve_column(sA, wave, tj, [&](int i, f32x4 tt) { put(i, tt); });
}

template <int DK, bool PRE>
hipError_t launch_t(const PrefillArgs &a, hipStream_t stream) {
  hipLaunchKernelGGL((chunk_compact_kernel<DK, PRE>), dim3((unsigned)local_grid(a)), dim3(kThreads), 0, stream, a);
  return hipGetLastError();
}

}  // namespace

hipError_t launch_chunk_compact(const PrefillArgs &a, hipStream_t s) {
  if (a.max_chunks == 0) return hipSuccess;
  if (a.Dk == 64) return a.pre ? launch_t<64, true>(a, s) : launch_t<64, false>(a, s);
  return a.pre ? launch_t<128, true>(a, s) : launch_t<128, false>(a, s);
}

}  // namespace hagdn

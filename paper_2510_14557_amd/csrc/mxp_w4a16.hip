// mxp_gemm_w4a16 : D[M][N] = A[M][K] (bf16, not quantized) x deq(W)[N][K]^T, W in canonical MXFP4 / MXFP4+ / MXFP4++
// (few rows: a weight-read-bound kernel; many rows: a tiled kernel, which also takes MXFP6(+) / MXFP8(+) weights and, for
// the MXFP8+ products of mxp_gemm, quantized eight-bit activations), and mxp_gemm_w4a16_ws, which may de-convert W once
// into a workspace ahead of the bf16 product of mxp_bf16.hip.
//
// The conversion-based use of the formats (Sec. 5: on hardware that lacks low-precision units, or for weight-only
// quantization, the blocks are de-converted to a wider type the hardware multiplies, Eq. 2 inside the kernel; the BM
// needs one extra select per block).  Here the wider type is bf16 and the multiplier is the bf16 MFMA; the weights are
// read in their canonical 4.25 / 4.5-bit form, so for few activation rows the product is bound by 0.53-0.56 bytes per
// weight element.
#include "mxp_common.h"
#include "mxp_decode.h"
#include <cmath>

namespace {

using namespace mxp;
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
typedef __bf16 v8bf __attribute__((ext_vector_type(8)));
typedef float v16f __attribute__((ext_vector_type(16)));

__device__ __forceinline__ uint32_t f32_to_bf16_rne_bits(float v) {
  uint32_t u = __float_as_uint(v);
  if ((u & 0x7FFFFFFFu) > 0x7F800000u) return (u >> 16) | 0x0040u;
  return (u + 0x7FFFu + ((u >> 16) & 1u)) >> 16;
}

__device__ __forceinline__ v8bf as_v8bf(const uint32_t (&d)[4]) {
  union { u32x4 u; v8bf b; } c;
  c.u = (u32x4){d[0], d[1], d[2], d[3]};
  return c.b;
}

// ---- few activation rows (M <= 64): one workgroup per 32 CT weight rows, K split over its wavefronts ------------------
// A 32x32x16 bf16 MFMA operand lane l holds row l % 32 and eight k-slots 8 (l / 32) .. +7.  The sum over k does not care
// which k sits in which slot as long as both operands agree, so the two lane halves take two different MX blocks: in
// "super-step" t (64 elements of K) lane (n, h) de-converts block 2t + h of weight row n and feeds its 32 values to four
// MFMAs, eight at a time; the activation lane (m, h) loads the same eight k per MFMA.  The W operand goes first, so
// accumulator register r of lane l is D[m = l % 32][n = 8 (r / 4) + 4 (l / 32) + r % 4].
// A wavefront takes groups of 8 blocks (256 elements of K) of 32 rows: it reads them the way they lie in memory
// (8 lanes per row: 128 contiguous bytes), passes them through a private LDS patch, and picks them up in operand order.
constexpr int kW4RowStride = 144;                            // 8 blocks x 16 B + 16 B padding against bank conflicts
constexpr int kW4PatchBytes = 32 * kW4RowStride + 256 + 256; // elements, scale bytes [32][8], index bytes [32][8]

// 32 codes -> 32 bf16 (16 dwords of pairs), Eq. 2.  The unpack-convert instruction runs over the whole block with the
// NBM scale; the BM's code is taken out of the codes first (code 0 converts to +0), and its value, an exponent and mantissa in
// place, is or-ed onto its pair: put at its place in a group of four pairs first, then one and-or per pair with the group's mask
// (76 vector instructions; compared with and selected into each pair 110).  Six more mask the codes of a flushed block (scale byte 0)
// away: weights may hold many such blocks, and with one in fifty of them the general way below makes a call 2.0 to 2.6 times as long
// (masks after the conversion, where a lane needs them, 1.26; these take 0.7 % of a call without such blocks).  Only when some lane of the
// wavefront holds a block of NaNs (255), or one whose values may leave the bf16 normal range, does the wavefront take the general
// de-conversion, which builds the patterns from integer fields.
template <int MODE>
__device__ __forceinline__ void decode_block_bf16(const u32x4 q, uint32_t sbyte, uint32_t ib, uint32_t (&w)[16]) {
  uint32_t n[4] = {q.x, q.y, q.z, q.w};
  const uint32_t delta = MODE == 2 ? ib >> 5 : 0u, idx = ib & 31u;
  const bool plain = sbyte >= 2u + delta && sbyte <= 250u, flushed = sbyte == 0u;
  uint32_t put = 0;
  if (MODE >= 1) {
    const FourAt at(idx);
    const uint32_t nib = at.get(n);
    at.put(nib, n);
    put = (((nib & 8u) << 12) | ((sbyte + 2u) << 7) | ((nib & 7u) << 4)) << (16u * (idx & 1u));   // 2^e_max * 1.mmm * X
  }
  const uint32_t keep = flushed ? 0u : ~0u;                  // a flushed block is zero whatever its codes say
  n[0] &= keep; n[1] &= keep; n[2] &= keep; n[3] &= keep; put &= keep;
  const float X = __uint_as_float((plain ? sbyte - delta : 127u) << 23);
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    union { v2bf v; uint32_t u; } c0, c1, c2, c3;
    c0.v = __builtin_amdgcn_cvt_scalef32_pk_bf16_fp4(n[j], X, 0);
    c1.v = __builtin_amdgcn_cvt_scalef32_pk_bf16_fp4(n[j], X, 1);
    c2.v = __builtin_amdgcn_cvt_scalef32_pk_bf16_fp4(n[j], X, 2);
    c3.v = __builtin_amdgcn_cvt_scalef32_pk_bf16_fp4(n[j], X, 3);
    w[4 * j] = c0.u; w[4 * j + 1] = c1.u; w[4 * j + 2] = c2.u; w[4 * j + 3] = c3.u;
  }
  if (MODE >= 1) or_onto_pair(idx, put, w);
  if (__builtin_amdgcn_ballot_w64(!plain && !flushed) != 0) {
#pragma unroll 1
    for (uint32_t s = 0; s < 4; ++s) {                       // (in one loop: four copies cost the kernels their registers)
      uint32_t out[8];
      decode_group<(MODE >= 1), true>(s == 0 ? q.x : s == 1 ? q.y : s == 2 ? q.z : q.w, sbyte, MODE >= 1 ? idx : 64u, s, out, delta);
#pragma unroll
      for (int j = 0; j < 16; ++j) w[j] = s == (uint32_t)(j >> 2) ? out[j & 3] : w[j];
    }
  }
}

template <int MODE, int TMR, int CT, bool OUT_BF16, int WAVES>
__global__ void __launch_bounds__(64 * WAVES) w4a16_skinny_kernel(const uint16_t* __restrict__ A, int64_t lda,
                                                                  const u32x4* __restrict__ w_el, const uint8_t* __restrict__ w_sc,
                                                                  const uint8_t* __restrict__ w_ix, int64_t nbk, int64_t M, int64_t N,
                                                                  void* __restrict__ Dv, int64_t ldd) {
  extern __shared__ __attribute__((aligned(16))) uint8_t lds_raw[];
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  uint8_t* patches = lds_raw + wave * (CT * kW4PatchBytes);  // private to this wavefront (LDS operations of a wavefront run in order)
  const int h = lane >> 5, nl = lane & 31;
  const int64_t n0 = (int64_t)blockIdx.x * (32 * CT);
  const int64_t groups = (nbk + 7) / 8;
  const bool meta_dwords = (nbk & 3) == 0;                  // scale / index bytes of 4 blocks can be read as one dword
  v16f acc[TMR][CT];
  const uint16_t* a_row[TMR];
  bool a_ok[TMR];
#pragma unroll
  for (int i = 0; i < TMR; ++i) {
#pragma unroll
    for (int j = 0; j < CT; ++j)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.0f;
    a_ok[i] = 32 * i + nl < M;
    a_row[i] = A + (a_ok[i] ? (int64_t)(32 * i + nl) * lda : 0) + h * 32;
  }

  // loads of one group in memory order: elements, 8 lanes per row; scale and index bytes, 2 lanes per row.  Absent blocks (rows past
  // N, whose outputs are not stored; past K, where the activations are zero) are zeros with an ordinary scale byte.
  u32x4 q[CT][4];
  uint32_t sc4[CT], ix4[CT];
  auto load_group = [&](int64_t g) {
    const int64_t kb0 = 8 * g;
#pragma unroll
    for (int j = 0; j < CT; ++j) {
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const int64_t n = n0 + 32 * j + 8 * i + (lane >> 3), kb = kb0 + (lane & 7);
        q[j][i] = (u32x4){0, 0, 0, 0};
        if (n < N && kb < nbk) q[j][i] = __builtin_nontemporal_load(w_el + n * nbk + kb);
      }
      sc4[j] = 0x7F7F7F7Fu;
      ix4[j] = 0;
      const int64_t n = n0 + 32 * j + (lane >> 1), kb = kb0 + 4 * (lane & 1);
      if (n < N && kb < nbk) {
        const int64_t b = n * nbk + kb;
        if (meta_dwords) {
          sc4[j] = *reinterpret_cast<const uint32_t*>(w_sc + b);
          if (MODE >= 1) ix4[j] = *reinterpret_cast<const uint32_t*>(w_ix + b);
        } else {
#pragma unroll
          for (int t = 0; t < 4; ++t) {
            if (kb + t < nbk) {
              sc4[j] = (sc4[j] & ~(0xFFu << (8 * t))) | (uint32_t)w_sc[b + t] << (8 * t);
              if (MODE >= 1) ix4[j] |= (uint32_t)w_ix[b + t] << (8 * t);
            }
          }
        }
      }
    }
  };
  if (wave < groups) load_group(wave);
  for (int64_t g = wave; g < groups; g += WAVES) {
    const int64_t kb0 = 8 * g;
    // ---- through the patches into operand order
#pragma unroll
    for (int j = 0; j < CT; ++j) {
      uint8_t* patch = patches + j * kW4PatchBytes;
#pragma unroll
      for (int i = 0; i < 4; ++i)
        *reinterpret_cast<u32x4*>(patch + (8 * i + (lane >> 3)) * kW4RowStride + (lane & 7) * 16) = q[j][i];
      *reinterpret_cast<uint32_t*>(patch + 32 * kW4RowStride + (lane >> 1) * 8 + 4 * (lane & 1)) = sc4[j];
      if (MODE >= 1) *reinterpret_cast<uint32_t*>(patch + 32 * kW4RowStride + 256 + (lane >> 1) * 8 + 4 * (lane & 1)) = ix4[j];
    }
    if (g + WAVES < groups) load_group(g + WAVES);          // the next group's loads fly while this one is multiplied
#pragma unroll
    for (int t = 0; t < 4; ++t) {
      const int bl = 2 * t + h;                             // block of the group this lane de-converts
      // activations: lane (m, h) needs, for MFMA s, eight k of the same block (they stay in cache: A is small)
      u32x4 a[TMR][4];
#pragma unroll
      for (int i = 0; i < TMR; ++i) {
        const uint16_t* ap = a_row[i] + kb0 * 32 + t * 64;   // a_row already points at this lane's row and block half
        const bool ok = a_ok[i] && kb0 + bl < nbk;
#pragma unroll
        for (int s = 0; s < 4; ++s) {
          a[i][s] = (u32x4){0, 0, 0, 0};
          if (ok) a[i][s] = *reinterpret_cast<const u32x4*>(ap + 8 * s);
        }
      }
#pragma unroll
      for (int j = 0; j < CT; ++j) {
        const uint8_t *patch = patches + j * kW4PatchBytes, *p_sc = patch + 32 * kW4RowStride;
        const u32x4 qq = *reinterpret_cast<const u32x4*>(patch + nl * kW4RowStride + bl * 16);
        const uint32_t sb = p_sc[nl * 8 + bl];
        const uint32_t ib = MODE >= 1 ? (uint32_t)p_sc[256 + nl * 8 + bl] : 0u;
        uint32_t w[16];
        decode_block_bf16<MODE>(qq, sb, ib, w);
#pragma unroll
        for (int s = 0; s < 4; ++s) {
          const uint32_t w4[4] = {w[4 * s], w[4 * s + 1], w[4 * s + 2], w[4 * s + 3]};
          const v8bf wv = as_v8bf(w4);
#pragma unroll
          for (int i = 0; i < TMR; ++i) {
            const uint32_t a4[4] = {a[i][s].x, a[i][s].y, a[i][s].z, a[i][s].w};
            acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(wv, as_v8bf(a4), acc[i][j], 0, 0, 0);
          }
        }
      }
    }
  }
  __syncthreads();                                          // the patches are dead: the same LDS now collects the partial tiles
  float (*part)[TMR * CT][16][64] = reinterpret_cast<float (*)[TMR * CT][16][64]>(lds_raw);
#pragma unroll
  for (int i = 0; i < TMR; ++i)
#pragma unroll
    for (int j = 0; j < CT; ++j)
#pragma unroll
      for (int r = 0; r < 16; ++r) part[wave][i * CT + j][r][lane] = acc[i][j][r];
  __syncthreads();
  for (int e = tid; e < TMR * CT * 16 * 64; e += 64 * WAVES) {
    const int l = e & 63, r = (e >> 6) & 15, ij = e >> 10, i = ij / CT, j = ij % CT;
    float v = 0.0f;
#pragma unroll
    for (int w = 0; w < WAVES; ++w) v += part[w][ij][r][l];
    const int64_t row = 32 * i + (l & 31);
    const int64_t col = n0 + 32 * j + 8 * (r >> 2) + 4 * (l >> 5) + (r & 3);
    if (row < M && col < N) {
      if (OUT_BF16) static_cast<uint16_t*>(Dv)[row * ldd + col] = (uint16_t)f32_to_bf16_rne_bits(v);
      else static_cast<float*>(Dv)[row * ldd + col] = v;
    }
  }
}

template <int MODE, int TMR, int CT, bool OUT_BF16, int WAVES>
void launch_skinny(hipStream_t s, const void* A, int64_t lda, const uint8_t* we, const uint8_t* ws, const uint8_t* wi, int64_t nbk, int64_t M,
                   int64_t N, void* D, int64_t ldd) {
  constexpr int lds_part = WAVES * TMR * CT * 16 * 64 * 4, lds_patch = WAVES * CT * kW4PatchBytes;
  constexpr int lds = lds_part > lds_patch ? lds_part : lds_patch;
  static_assert(lds <= 160 * 1024, "LDS");
  allow_dynamic_lds<&w4a16_skinny_kernel<MODE, TMR, CT, OUT_BF16, WAVES>>((int)lds);
  hipLaunchKernelGGL((w4a16_skinny_kernel<MODE, TMR, CT, OUT_BF16, WAVES>), dim3((unsigned)((N + 32 * CT - 1) / (32 * CT))), dim3(64 * WAVES), lds, s,
                     static_cast<const uint16_t*>(A), lda, reinterpret_cast<const u32x4*>(we), ws, wi, nbk, M, N, D, ldd);
}

template <int MODE>
int dispatch_skinny(int64_t M, int64_t N, int64_t K, const void* A, int64_t lda, const uint8_t* we, const uint8_t* ws,
                    const uint8_t* wi, void* D, int d_dtype, int64_t ldd, hipStream_t s) {
  const int64_t ct = (N + 31) / 32, nbk = K / kBlock;
  if (ct > 2147483647LL) return MXP_ERR_UNSUPPORTED;
#define MXP_SKINNY(TMR, CT, WAVES)                                                                                  \
  do {                                                                                                              \
    if (d_dtype == MXP_BF16) launch_skinny<MODE, TMR, CT, true, WAVES>(s, A, lda, we, ws, wi, nbk, M, N, D, ldd);   \
    else launch_skinny<MODE, TMR, CT, false, WAVES>(s, A, lda, we, ws, wi, nbk, M, N, D, ldd);                      \
  } while (0)
  // What bounds this kernel is the reads of A (every workgroup reads all of it) and the vector instructions of the conversion, at the same
  // time: 13 x 28672 x 8192 MXFP4+ 64 us, 49 without the reads, 62 without the conversion, 32 without either (before the block maximum
  // went in by masks; now 52).  Two column tiles share the reads from the 257th tile on (us, replayed from a graph, one tile of sixteen
  // wavefronts -> here: 32 x 10000 x 4096 23.0 -> 15.8, 13 x 14336 x 4096 17.1 -> 15.0 and MXFP4 15.1 -> 11.3, 64 x 14336 x 4096
  // 38.9 -> 24.8); up to 256 tiles they would leave compute units idle (8 x 4096 x 4096 7.9 | 13.7), and up to 8 rows one tile of eight
  // wavefronts is ahead (4 x 10000 x 4096 15.1 -> 12.9 | 14.8 with two, x 1024 8.4 -> 5.4 | 6.3).
  // So it is where the last round of pairs of tiles would be nearly empty, up to 2^16 values of A (11 x 18389 x 4512 MXFP4+ 40.5 with
  // two, 30.2 with one of eight; 9 - 32 rows, 459 shapes of 513 - 768 tiles, geometric means against one of sixteen 0.78 with one of
  // eight, 1.03 with two); above that sixteen are (158 shapes, 1.01 and 1.11).
  const int64_t pairs = (ct + 1) / 2;
  const bool one_round = ct <= kNumCU;
  const bool last_empty = (pairs > kNumCU && 2 * pairs <= 3 * kNumCU) || (pairs > 2 * kNumCU && 4 * pairs <= 9 * kNumCU);
  if (M > 32) {
    if (one_round) MXP_SKINNY(2, 1, 8);                      // (sixteen wavefronts would spill)
    else MXP_SKINNY(2, 2, 8);
  } else {
    if (one_round || (last_empty && M * K > 65536)) MXP_SKINNY(1, 1, 16);
    else if (M <= 8 || last_empty) MXP_SKINNY(1, 1, 8);
    else MXP_SKINNY(1, 2, 8);
  }
#undef MXP_SKINNY
  return launch_status();
}

// ---- tiled product on de-converted operands: 256 x 256 output tiles ------------------------------------------------
// Many activation rows (prefill with weight-only quantization), weights of any block format; and the product of two
// quantized operands whose BM fits no block-scaled MFMA element (MXFP8+): every format's values are bf16 numbers, so
// the product of the de-converted operands on the bf16 MFMA is the exact product (fp32 accumulation).
// A workgroup of 2 x 4 wavefronts (two per SIMD, so that one's conversions and LDS traffic run under the other's MFMAs)
// computes 256 rows of A x 256 rows of W; each wavefront 4 x 2 MFMA tiles of 32 x 32.  K is walked in steps of 64 (two
// MX blocks: the two lane halves of an operand take one each, as above).  Both operands of a step lie in LDS as bf16,
// 256 rows each, double-buffered: un-quantized activations are copied, quantized operands are de-converted (Eq. 2) on
// the way in -- thread (n, b) of the workgroup owns block b of row n in every step, one block per thread and step, so
// each block is converted once per workgroup.  Rows are 144 bytes apart in LDS (128 + 16 of padding): the 16 lanes that
// read the same chunk of 16 consecutive rows then hit 16 different 16-byte bank groups (9 r mod 16), and the chunk is an
// immediate offset of the read.  Global loads run one step (un-quantized rows) or two (codes) ahead of the MFMAs that
// use them and are written to the other LDS stage behind the MFMAs of the step before; one barrier per step.
constexpr int kTRow = 144;                                   // bytes per operand row in LDS: 64 bf16 + 16 B of padding
constexpr int kTOperand = 256 * kTRow;                       // one operand of one step: 256 rows x 64 bf16
constexpr int kTStage = 2 * kTOperand;                       // activations, then weights
constexpr int kTiledLds = 2 * kTStage;
constexpr int kTiledThreads = 512;

// operand kinds
constexpr int kRawBf16 = 0, kFp4 = 1 /* + MODE: 1, 2, 3 */, kFp6 = 4, kFp8 = 6;   // six- / eight-bit: plain or + by a flag

struct QBlock {                                              // one block of codes with its scale and index bytes
  uint32_t raw[8];
  uint32_t sb, ib;
};

template <int KIND>
__device__ __forceinline__ QBlock q_load(bool ok, const uint8_t* el, const uint8_t* sc, const uint8_t* ix, int64_t b, bool has_ix) {
  QBlock r;
#pragma unroll
  for (int j = 0; j < 8; ++j) r.raw[j] = 0;
  r.sb = 0;                                                  // blocks past the matrix: scale byte 0, an all-zero block
  r.ib = 0;
  if (ok) {
    if (KIND == kFp6) {
      const u32x2* p = reinterpret_cast<const u32x2*>(el + b * 24);
      const u32x2 d0 = p[0], d1 = p[1], d2 = p[2];
      r.raw[0] = d0.x; r.raw[1] = d0.y; r.raw[2] = d1.x; r.raw[3] = d1.y; r.raw[4] = d2.x; r.raw[5] = d2.y;
    } else if (KIND == kFp8) {
      const u32x4* p = reinterpret_cast<const u32x4*>(el + b * 32);
      const u32x4 d0 = p[0], d1 = p[1];
      r.raw[0] = d0.x; r.raw[1] = d0.y; r.raw[2] = d0.z; r.raw[3] = d0.w;
      r.raw[4] = d1.x; r.raw[5] = d1.y; r.raw[6] = d1.z; r.raw[7] = d1.w;
    } else {
      const u32x4 d0 = *reinterpret_cast<const u32x4*>(el + b * 16);
      r.raw[0] = d0.x; r.raw[1] = d0.y; r.raw[2] = d0.z; r.raw[3] = d0.w;
    }
    r.sb = sc[b];
    if (has_ix) r.ib = ix[b];
  }
  return r;
}

// Four-bit block -> 64 bytes of bf16 at `dst`.  As decode_block_bf16, except that the rare cases are kept out of the
// registers: the 32 elements are converted with the NBM scale and stored, then the BM is written over its two bytes
// with one LDS store, and blocks with a reserved scale byte (all-zero, NaN) are overwritten by the lanes that hold one
// (LDS operations of a wavefront execute in order).  Wavefronts with a block below the bf16 normal range take the
// general routine.
template <int MODE>
__device__ __forceinline__ void q_store_fp4(const QBlock& r, uint8_t* dst) {
  const uint32_t delta = MODE == 2 ? r.ib >> 5 : 0u;
  const bool tiny = r.sb != 0u && r.sb < 2u + delta;
  if (__builtin_amdgcn_ballot_w64(tiny) != 0) {
    uint32_t w[16];
    decode_block_bf16<MODE>((u32x4){r.raw[0], r.raw[1], r.raw[2], r.raw[3]}, r.sb, r.ib, w);
#pragma unroll
    for (int s4 = 0; s4 < 4; ++s4)
      *reinterpret_cast<u32x4*>(dst + 16 * s4) = (u32x4){w[4 * s4], w[4 * s4 + 1], w[4 * s4 + 2], w[4 * s4 + 3]};
    return;
  }
  const bool special = r.sb == 0u || r.sb == 255u;
  const float X = __uint_as_float((special ? 127u : r.sb - delta) << 23);
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    union { v2bf v; uint32_t u; } c0, c1, c2, c3;
    c0.v = __builtin_amdgcn_cvt_scalef32_pk_bf16_fp4(r.raw[j], X, 0);
    c1.v = __builtin_amdgcn_cvt_scalef32_pk_bf16_fp4(r.raw[j], X, 1);
    c2.v = __builtin_amdgcn_cvt_scalef32_pk_bf16_fp4(r.raw[j], X, 2);
    c3.v = __builtin_amdgcn_cvt_scalef32_pk_bf16_fp4(r.raw[j], X, 3);
    *reinterpret_cast<u32x4*>(dst + 16 * j) = (u32x4){c0.u, c1.u, c2.u, c3.u};
  }
  if (MODE >= 1 && !special) {
    const uint32_t idx = r.ib & 31u;
    const uint32_t qd = idx < 8u ? r.raw[0] : idx < 16u ? r.raw[1] : idx < 24u ? r.raw[2] : r.raw[3];
    const uint32_t nib = (qd >> (4u * (idx & 7u))) & 15u;
    const float XB = __uint_as_float(r.sb << 23);
    const uint32_t bm = ((nib & 8u) << 12) | (__float_as_uint((float)(8u + (nib & 7u)) * (XB * 0.5f)) >> 16);   // exact: 4 bits
    *reinterpret_cast<uint16_t*>(dst + 2u * idx) = (uint16_t)bm;
  }
  if (__builtin_amdgcn_ballot_w64(special) != 0) {
    if (special) {
      const uint32_t v = r.sb == 0u ? 0u : 0x7FC07FC0u;
#pragma unroll
      for (int s4 = 0; s4 < 4; ++s4) *reinterpret_cast<u32x4*>(dst + 16 * s4) = (u32x4){v, v, v, v};
    }
  }
}

// de-convert the block and store its 64 bytes of bf16 at `dst` (the block's place in its LDS row)
template <int KIND>
__device__ __forceinline__ void q_store(const QBlock& r, bool plus, uint8_t* dst) {
  if constexpr (KIND >= 1 && KIND <= 3) {
    q_store_fp4<KIND - 1>(r, dst);
    return;
  }
  uint32_t w[16];
  if (KIND == kFp6 || KIND == kFp8) {
    constexpr int BITS = KIND == kFp6 ? 6 : 8;
    const bool general = __builtin_amdgcn_ballot_w64(!wide_block_is_plain<BITS>(r.raw, r.sb, plus ? (r.ib & 31u) : 64u)) != 0;
    decode_wide_block_bf16<BITS>(r.raw, r.sb, r.ib, plus, general, w);
  } else {
    decode_block_bf16<(KIND >= 1 && KIND <= 3 ? KIND - 1 : 0)>((u32x4){r.raw[0], r.raw[1], r.raw[2], r.raw[3]}, r.sb, r.ib, w);
  }
#pragma unroll
  for (int s4 = 0; s4 < 4; ++s4)
    *reinterpret_cast<u32x4*>(dst + 16 * s4) = (u32x4){w[4 * s4], w[4 * s4 + 1], w[4 * s4 + 2], w[4 * s4 + 3]};
}

struct QOperand {                                            // a quantized operand: codes, scale bytes, index bytes
  const uint8_t *el, *sc, *ix;
  int plus;                                                  // six- / eight-bit kinds: the + form
};

template <int AK, int WK, bool OUT_BF16, int WI>
__global__ void __launch_bounds__(kTiledThreads) deconv_tiled_kernel(const uint16_t* __restrict__ A, int64_t lda, QOperand qa,
                                                                     QOperand qw, int64_t nbk, int64_t M, int64_t N,
                                                                     void* __restrict__ Dv, int64_t ldd, int tiles_n) {
  extern __shared__ __attribute__((aligned(16))) uint8_t lds_raw[];
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  // WI row tiles per wavefront: 4 -> 256 rows of A per workgroup; 2 -> 128 rows, for launches that would otherwise leave
  // most compute units without a tile
  constexpr int NJ = 2, WAVES_N = 4, TROWS = 64 * WI, PA = TROWS * 8 / kTiledThreads;
  const int wm = wave / WAVES_N, wn = wave % WAVES_N, h = lane >> 5, nl = lane & 31;
  const int64_t m0 = (int64_t)(blockIdx.x / tiles_n) * TROWS, n0 = (int64_t)(blockIdx.x % tiles_n) * 256;
  const int64_t nks = (nbk + 1) / 2;

  v16f acc[WI][NJ];
#pragma unroll
  for (int i = 0; i < WI; ++i)
#pragma unroll
    for (int j = 0; j < NJ; ++j)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.0f;

  // un-quantized activations: chunk kc = tid % 8 of rows tid / 8 + 64 u
  const int a_row = tid >> 3, a_kc = tid & 7;
  const uint32_t a_off = (uint32_t)(a_row * kTRow + (a_kc << 4));
  constexpr int A_STEP = kTiledThreads / 8;
  const uint16_t* a_ptr[PA];
  bool a_ok[PA];
#pragma unroll
  for (int u = 0; u < PA; ++u) {
    a_ok[u] = AK == kRawBf16 && m0 + a_row + A_STEP * u < M;
    a_ptr[u] = A + (a_ok[u] ? (m0 + a_row + A_STEP * u) * lda : 0) + a_kc * 8;
  }
  // quantized operands: block b = tid % 2 of row tid / 2 in every step
  const int q_row = tid >> 1, q_b = tid & 1;
  const uint32_t q_off = (uint32_t)(q_row * kTRow + 64 * q_b);
  const bool qa_ok = AK != kRawBf16 && q_row < TROWS && m0 + q_row < M, qw_ok = n0 + q_row < N;
  const int64_t qa_base = qa_ok ? (m0 + q_row) * nbk + q_b : 0, qw_base = qw_ok ? (n0 + q_row) * nbk + q_b : 0;
  const bool a_has_ix = AK == 2 || AK == 3 || ((AK == kFp6 || AK == kFp8) && qa.plus);
  const bool w_has_ix = WK == 2 || WK == 3 || ((WK == kFp6 || WK == kFp8) && qw.plus);

  struct ABlock {
    u32x4 v[PA];
  };
  auto load_a = [&](int64_t ks) {
    ABlock r;
    const bool k_ok = 2 * ks + (a_kc >> 2) < nbk;            // the chunk's block exists (K % 32 == 0: chunks are whole)
#pragma unroll
    for (int u = 0; u < PA; ++u) {
      r.v[u] = (u32x4){0, 0, 0, 0};
      if (a_ok[u] && k_ok) r.v[u] = *reinterpret_cast<const u32x4*>(a_ptr[u] + ks * 64);
    }
    return r;
  };
  auto store_a = [&](int buf, const ABlock& r) {
#pragma unroll
    for (int u = 0; u < PA; ++u) *reinterpret_cast<u32x4*>(lds_raw + buf * kTStage + a_off + u * (A_STEP * kTRow)) = r.v[u];
  };
  auto load_qa = [&](int64_t ks) { return q_load<AK>(qa_ok && 2 * ks + q_b < nbk, qa.el, qa.sc, qa.ix, qa_base + 2 * ks, a_has_ix); };
  auto load_qw = [&](int64_t ks) { return q_load<WK>(qw_ok && 2 * ks + q_b < nbk, qw.el, qw.sc, qw.ix, qw_base + 2 * ks, w_has_ix); };

  // operand reads: lane (nl, h) of tile row / column r takes chunk 4 h + s4 (an immediate offset from these bases)
  uint32_t rd_a[WI], rd_w[NJ];
#pragma unroll
  for (int i = 0; i < WI; ++i) rd_a[i] = (uint32_t)((wm * (32 * WI) + 32 * i + nl) * kTRow + 64 * h);
#pragma unroll
  for (int j = 0; j < NJ; ++j) rd_w[j] = (uint32_t)(kTOperand + (wn * (32 * NJ) + 32 * j + nl) * kTRow + 64 * h);

  ABlock a1;
  QBlock qa1, qa2, qw1, qw2;
  if (AK == kRawBf16) {
    a1 = load_a(0);
    store_a(0, a1);
  } else {
    qa1 = load_qa(0);
    q_store<AK>(qa1, qa.plus != 0, lds_raw + q_off);
    qa1 = load_qa(1);
  }
  qw1 = load_qw(0);
  q_store<WK>(qw1, qw.plus != 0, lds_raw + kTOperand + q_off);
  qw1 = load_qw(1);
  __syncthreads();
  for (int64_t ks = 0; ks < nks; ++ks) {
    const bool more = ks + 1 < nks;
    const uint8_t* st = lds_raw + (ks & 1) * kTStage;
    uint8_t* nxt = lds_raw + ((ks + 1) & 1) * kTStage;
    if (AK == kRawBf16) {
      if (more) a1 = load_a(ks + 1);
    } else {
      qa2 = load_qa(ks + 2);
    }
    qw2 = load_qw(ks + 2);
    // the MFMAs of one eighth of K per slice (k-slots 8 s4 .. 8 s4 + 7 of both blocks)
#pragma unroll
    for (int s4 = 0; s4 < 4; ++s4) {
      v8bf wv[NJ];
#pragma unroll
      for (int j = 0; j < NJ; ++j) {
        const u32x4 v = *reinterpret_cast<const u32x4*>(st + rd_w[j] + 16 * s4);
        const uint32_t v4[4] = {v.x, v.y, v.z, v.w};
        wv[j] = as_v8bf(v4);
      }
#pragma unroll
      for (int i = 0; i < WI; ++i) {
        const u32x4 v = *reinterpret_cast<const u32x4*>(st + rd_a[i] + 16 * s4);
        const uint32_t v4[4] = {v.x, v.y, v.z, v.w};
        const v8bf a8 = as_v8bf(v4);
#pragma unroll
        for (int j = 0; j < NJ; ++j) acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a8, wv[j], acc[i][j], 0, 0, 0);
      }
    }
    // the next step's operands go into the other stage.  (Measured alternatives that were slower: stores placed between
    // the MFMA slices -- the branches of the de-conversion cut the MFMA sequence --, activations loaded two steps ahead,
    // the two wavefronts of a SIMD running half a step out of phase, 2 x 2 wavefronts of 4 x 4 tiles.)
    if (more) {
      if (AK == kRawBf16) store_a((int)((ks + 1) & 1), a1);
      else q_store<AK>(qa1, qa.plus != 0, nxt + q_off);
      q_store<WK>(qw1, qw.plus != 0, nxt + kTOperand + q_off);
    }
    if (AK != kRawBf16) qa1 = qa2;
    qw1 = qw2;
    __syncthreads();
  }
  // accumulator register r of lane l: D[8 (r / 4) + 4 (l / 32) + r % 4][l % 32] of the 32 x 32 tile
  const bool whole = m0 + TROWS <= M && n0 + 256 <= N;
#pragma unroll
  for (int i = 0; i < WI; ++i)
#pragma unroll
    for (int j = 0; j < NJ; ++j) {
      const int64_t col = n0 + wn * (32 * NJ) + 32 * j + nl;
      const int64_t row0 = m0 + wm * (32 * WI) + 32 * i + 4 * h;
      if (whole) {                                           // tile inside the matrix (uniform): no per-element tests
#pragma unroll
        for (int r = 0; r < 16; ++r) {
          const int64_t o = (row0 + 8 * (r >> 2) + (r & 3)) * ldd + col;
          if (OUT_BF16) static_cast<uint16_t*>(Dv)[o] = (uint16_t)f32_to_bf16_rne_bits(acc[i][j][r]);
          else static_cast<float*>(Dv)[o] = acc[i][j][r];
        }
      } else {
#pragma unroll
        for (int r = 0; r < 16; ++r) {
          const int64_t row = row0 + 8 * (r >> 2) + (r & 3);
          if (row < M && col < N) {
            if (OUT_BF16) static_cast<uint16_t*>(Dv)[row * ldd + col] = (uint16_t)f32_to_bf16_rne_bits(acc[i][j][r]);
            else static_cast<float*>(Dv)[row * ldd + col] = acc[i][j][r];
          }
        }
      }
    }
}

template <int AK, int WK, int WI = 4>
int launch_deconv(int64_t M, int64_t N, int64_t K, const void* A, int64_t lda, const QOperand& qa, const QOperand& qw, void* D,
                  int d_dtype, int64_t ldd, hipStream_t s) {
  const int64_t tm = (M + 64 * WI - 1) / (64 * WI), tn = (N + 255) / 256;
  if (tm * tn > 2147483647LL || tn > 2147483647LL) return MXP_ERR_UNSUPPORTED;
  const dim3 grid((unsigned)(tm * tn));
  const int64_t nbk = K / kBlock;
  static_assert(kTiledLds <= 160 * 1024, "LDS");
  if (d_dtype == MXP_BF16) {
    allow_dynamic_lds<&deconv_tiled_kernel<AK, WK, true, WI>>(kTiledLds);
    hipLaunchKernelGGL((deconv_tiled_kernel<AK, WK, true, WI>), grid, dim3(kTiledThreads), kTiledLds, s, static_cast<const uint16_t*>(A),
                       lda, qa, qw, nbk, M, N, D, ldd, (int)tn);
  } else {
    allow_dynamic_lds<&deconv_tiled_kernel<AK, WK, false, WI>>(kTiledLds);
    hipLaunchKernelGGL((deconv_tiled_kernel<AK, WK, false, WI>), grid, dim3(kTiledThreads), kTiledLds, s, static_cast<const uint16_t*>(A),
                       lda, qa, qw, nbk, M, N, D, ldd, (int)tn);
  }
  return launch_status();
}

// kind of the tiled kernel's operand loader for a block format, and whether it is the + form
inline int kind_of(int fmt) {
  switch (fmt) {
    case MXP_FMT_MXFP4: return 1;
    case MXP_FMT_MXFP4P: return 2;
    case MXP_FMT_MXFP4PP: return 3;
    case MXP_FMT_MXFP6: case MXP_FMT_MXFP6P: return kFp6;
    default: return kFp8;
  }
}
inline int64_t block_bytes(int fmt) { return fmt < MXP_FMT_MXFP6 ? 16 : fmt < MXP_FMT_MXFP8 ? 24 : 32; }   // codes of one block
inline int plus_of(int fmt) { return fmt == MXP_FMT_MXFP6P || fmt == MXP_FMT_MXFP8P; }

// fewer than ~200 tiles of 256 rows: tiles of 128 rows, twice as many workgroups (four-bit weights only)
inline bool tiles_of_128_rows(int64_t M, int64_t N) { return ((M + 255) / 256) * ((N + 255) / 256) < 200 && M > 128; }

// un-quantized bf16 activations x weights of any block format
int dispatch_tiled(int64_t M, int64_t N, int64_t K, const void* A, int64_t lda, const uint8_t* we, const uint8_t* ws,
                   const uint8_t* wi, int fmtW, void* D, int d_dtype, int64_t ldd, hipStream_t s) {
  const QOperand none = {nullptr, nullptr, nullptr, 0}, qw = {we, ws, wi, plus_of(fmtW)};
  if (tiles_of_128_rows(M, N) && kind_of(fmtW) <= 3) {
    switch (kind_of(fmtW)) {
      case 1: return launch_deconv<kRawBf16, 1, 2>(M, N, K, A, lda, none, qw, D, d_dtype, ldd, s);
      case 2: return launch_deconv<kRawBf16, 2, 2>(M, N, K, A, lda, none, qw, D, d_dtype, ldd, s);
      default: return launch_deconv<kRawBf16, 3, 2>(M, N, K, A, lda, none, qw, D, d_dtype, ldd, s);
    }
  }
  switch (kind_of(fmtW)) {
    case 1: return launch_deconv<kRawBf16, 1>(M, N, K, A, lda, none, qw, D, d_dtype, ldd, s);
    case 2: return launch_deconv<kRawBf16, 2>(M, N, K, A, lda, none, qw, D, d_dtype, ldd, s);
    case 3: return launch_deconv<kRawBf16, 3>(M, N, K, A, lda, none, qw, D, d_dtype, ldd, s);
    case kFp6: return launch_deconv<kRawBf16, kFp6>(M, N, K, A, lda, none, qw, D, d_dtype, ldd, s);
    default: return launch_deconv<kRawBf16, kFp8>(M, N, K, A, lda, none, qw, D, d_dtype, ldd, s);
  }
}

}  // namespace

namespace mxp {
// Both operands quantized, at least one of them eight-bit (MXFP8 / MXFP8+ with each other or with any narrower format), or
// a six-bit format next to MXFP4++: the product of the de-converted operands.
int deconv_gemm_launch(int64_t M, int64_t N, int64_t K, const uint8_t* ae, const uint8_t* as, const uint8_t* ai, int fmtA,
                           const uint8_t* be, const uint8_t* bs, const uint8_t* bi, int fmtB, void* D, int d_dtype, int64_t ldd,
                           hipStream_t s) {
  const QOperand qa = {ae, as, ai, plus_of(fmtA)}, qb = {be, bs, bi, plus_of(fmtB)};
  const int ka = kind_of(fmtA), kb = kind_of(fmtB);
#define MXP_DECONV(AKV, BKV) return launch_deconv<AKV, BKV>(M, N, K, nullptr, 0, qa, qb, D, d_dtype, ldd, s)
  if (ka == kFp8) {
    switch (kb) {
      case 1: MXP_DECONV(kFp8, 1);
      case 2: MXP_DECONV(kFp8, 2);
      case 3: MXP_DECONV(kFp8, 3);
      case kFp6: MXP_DECONV(kFp8, kFp6);
      default: MXP_DECONV(kFp8, kFp8);
    }
  }
  if (ka == kFp6 && kb == 3) MXP_DECONV(kFp6, 3);              // six-bit next to MXFP4++: no block-scaled image pairing for it
  if (ka == 3 && kb == kFp6) MXP_DECONV(3, kFp6);
  if (kb != kFp8) return MXP_ERR_UNSUPPORTED;
  switch (ka) {
    case 1: MXP_DECONV(1, kFp8);
    case 2: MXP_DECONV(2, kFp8);
    case 3: MXP_DECONV(3, kFp8);
    default: MXP_DECONV(kFp6, kFp8);
  }
#undef MXP_DECONV
}
}  // namespace mxp

namespace {
// W de-converted once, as bf16, ahead of a plain bf16 product -- or in the product kernel, again for each row of its tiles.
// Which is faster follows from what either makes of a shape: rounds of tiles over the chip that each walk along K, against
// a pass over W and fewer, faster rounds.  Both are estimated (us) with the rates that the two routes measured over 3700
// shapes (1 - 4096 rows, N 200 - 60000, K 256 - 30000, six formats; the estimates are off by 9 and 11 %), and W is de-converted
// once where that is ahead by a margin.  In the kernel -> once, us, bf16 out:
//   MXFP4+, 14336 x 4096: 160 rows 88.6 -> 60.5, 1024 131 -> 115, 4096 501 -> 363; 4096 x 14336: 160 rows 296 -> 110, 2048 331 -> 205
//   MXFP8+, 14336 x 4096: 1024 rows 170 -> 119, 4096 668 -> 374
// and where it stays in the kernel (column tiles fill the chip, few rows of them repeat the work; W in slabs that do not):
//   MXFP4+, 28672 x 8192: 129 rows 202 | 265, 512 267 | 347; 28672 x 14336: 512 rows 464 | 880; 14336 x 256: 512 rows 13.6 | 17.3
// Of the 3700 shapes 13 are slower than in the kernel by more than 3 % (11 % at most), 92 would gain more than 5 % (14 % on average).
double in_kernel_us(int64_t M, int64_t N, int64_t K, int fmtW) {
  const bool four = fmtW < MXP_FMT_MXFP6, halves = four && tiles_of_128_rows(M, N);
  // ns per element of K and round, by what a block's de-conversion takes
  const double c = halves ? 20.0 : four ? 27.0 : fmtW == MXP_FMT_MXFP6 ? 28.0 : fmtW == MXP_FMT_MXFP6P ? 33.5 : fmtW == MXP_FMT_MXFP8 ? 30.0 : 39.0;
  const double tiles = (double)((M + (halves ? 127 : 255)) / (halves ? 128 : 256)) * (double)((N + 255) / 256);
  return (four ? 8.0 : 10.0) + (double)K * c * (std::ceil(tiles / mxp::kNumCU) + 0.28 * tiles / mxp::kNumCU) * 1e-3 + (double)M * N / 1.75e6;
}
double once_us(int64_t M, int64_t n, int64_t K, int fmtW, bool d_vectors) {          // n rows of W
  const double blocks = (double)((M + 127) / 128) * (double)((n + 127) / 128), tiles = (double)((M + 255) / 256) * (double)((n + 255) / 256);
  const double rounds = std::floor(tiles / mxp::kNumCU), rem = tiles - rounds * mxp::kNumCU;
  const double walk = blocks <= mxp::kNumCU ? 5.5 + 1.6 * blocks / mxp::kNumCU
                                            : 19.5 * rounds + (rem == 0 ? 0.0 : rem <= mxp::kNumCU / 2 ? 12.0 : 19.5);   // ns per element of K
  const double bytes = 2.0 + (double)block_bytes(fmtW) / 32 + 1.0 / 16;               // bf16, codes, scale and index
  return 10.0 + bytes * (double)n * (double)K / 5e6 + (double)K * walk * 1e-3 + (double)M * n / 1.75e6 + (d_vectors ? 0.0 : (double)M * n / 1.05e6);
}

// Six- and eight-bit W next to 33 to 64 rows: rounds of the few-row kernel's workgroups (32 columns, one per compute unit), and the
// workgroups of the last one.
struct FewRounds {
  int64_t rounds, last;
  explicit FewRounds(int64_t N) : rounds(((N + 31) / 32 + mxp::kNumCU - 1) / mxp::kNumCU), last((N + 31) / 32 - (rounds - 1) * mxp::kNumCU) {}
};
// Where W as bf16 is ahead of that kernel: many of those rows, its last round up to two fifths full, and K between what a second launch
// and pass over W cost and what the last-level cache holds of it (us, few-row kernel | W once: MXFP6+ 57 x 8950 x 7424 92.2 | 73.1,
// 52 x 18895 x 3968 73.1 | 60.7, but MXFP6 58 x 8526 x 320 8.9 | 12.0; over 17000 shapes of 4096 - 32768 columns this choice is 0.4 % behind
// the better of the two, the kernel alone 0.7 %, W once below three fifths of a second round 8 %).
bool once_beats_few_rows(int64_t M, int64_t N, int64_t K, int fmtW) {
  const FewRounds r(N);
  const bool plus = fmtW == MXP_FMT_MXFP6P || fmtW == MXP_FMT_MXFP8P;
  return M > (plus ? 44 : 52) && r.rounds >= 2 && 5 * r.last <= 2 * mxp::kNumCU && K * (r.rounds - 1) >= 3072 && K * r.rounds <= 16384;
}
// Where the tiled kernel is: three and more rounds of it, each a step or two of K that one of its eight wavefronts takes (MXFP6+
// 50 x 24923 x 64 16.3 | 10.4, x 128 at 24600 - 32768 columns a fifth slower; at 192 the same).
bool tiles_beat_few_rows(int64_t M, int64_t N, int64_t K) {
  const FewRounds r(N);
  return M > 32 && K <= 192 && K <= 64 * (r.rounds - 2);
}

// Rows of W that are de-converted at a time, given room for so many bytes of them; 0: de-conversion stays in the kernel.
// Slabs are whole tiles and as even as that allows.  d_vectors: the rows of D start at 16-byte addresses.
int64_t slab_rows(int64_t M, int64_t N, int64_t K, int64_t lda, int fmtW, bool d_vectors, size_t bytes) {
  const bool four = fmtW < MXP_FMT_MXFP6;
  // few rows have kernels of their own: four-bit W up to 128 (16 / 64 rows x 14336 x 4096: 14.9 / 24.8 us against 60), wider W up to 64
  if ((four && M <= 128) || K < 256 || !mxp::bf16_gemm_takes(M, N, K, lda)) return 0;
  if (!four && M <= 64) return once_beats_few_rows(M, N, K, fmtW) && bytes / (2 * (size_t)K) >= (size_t)N ? N : 0;
  int64_t rows = N, n = 1;
  if (bytes / (2 * (size_t)K) < (size_t)N) {
    rows = (int64_t)(bytes / (2 * (size_t)K)) / 256 * 256;
    if (rows == 0) return 0;
    n = (N + rows - 1) / rows;
    rows = ((N + n - 1) / n + 255) / 256 * 256;
  }
  const double once = (double)(n - 1) * once_us(M, rows, K, fmtW, d_vectors) + once_us(M, N - (n - 1) * rows, K, fmtW, d_vectors);
  // short K and many columns: the second launch and the pass over W weigh more than the rates say (MXFP4+ 512 x 14336 x 512
  // 20.5 | 27.0, 512 x 14336 x 1024 31.1 | 35.3, estimated 4 and 11 % the other way; MXFP6 1024 x 14336 x 256
  // 20.4 | 22.5, MXFP8+ 512 x 57344 x 256 46.3 | 50.5)
  const bool short_k = four ? K < 1280 && N > 4608 : K < 640 && N > 12288;
  return once * (short_k ? 1.25 : n == 1 ? 1.02 : 1.1) < in_kernel_us(M, N, K, fmtW) ? rows : 0;
}
// Room asked for at most: what the last-level cache holds, which the product then reads a slab from (us in slabs of 128 MiB | of
// 256 | W whole: MXFP4+ 1024 x 28672 x 8192 499 | 440 | 467, 2048 x 57344 x 4096 836 | 782 | 787, 2048 x 28672 x 14336 1444 | 1325 |
// 1326; few rows and long K would gain from more, 768 x 14336 x 28672 1291 | 903 | 761, which a caller may give).
constexpr size_t kSlabBytes = (size_t)256 << 20;
}  // namespace

extern "C" size_t mxp_gemm_w4a16_workspace_bytes(int64_t M, int64_t N, int64_t K, int fmtW) {
  if (M <= 0 || N <= 0 || K <= 0 || K > mxp::kMaxGemmK || fmtW < MXP_FMT_MXFP4 || fmtW > MXP_FMT_MXFP8P) return 0;
  return ((size_t)slab_rows(M, N, K, K, fmtW, N % 4 == 0, kSlabBytes) * (size_t)K * 2 + 255) / 256 * 256;
}

extern "C" int mxp_gemm_w4a16(int64_t M, int64_t N, int64_t K, const void* A, int a_dtype, int64_t lda,
                              const uint8_t* W_elems, const uint8_t* W_scales, const uint8_t* W_idx, int fmtW, void* D,
                              int d_dtype, int64_t ldd, void* stream) {
  return mxp_gemm_w4a16_ws(M, N, K, A, a_dtype, lda, W_elems, W_scales, W_idx, fmtW, D, d_dtype, ldd, nullptr, 0, stream);
}

extern "C" int mxp_gemm_w4a16_ws(int64_t M, int64_t N, int64_t K, const void* A, int a_dtype, int64_t lda,
                                 const uint8_t* W_elems, const uint8_t* W_scales, const uint8_t* W_idx, int fmtW, void* D,
                                 int d_dtype, int64_t ldd, void* workspace, size_t workspace_bytes, void* stream) {
  using namespace mxp;
  if (fmtW < MXP_FMT_MXFP4 || fmtW > MXP_FMT_MXFP8P) return MXP_ERR_FORMAT;
  const bool wide_w = fmtW >= MXP_FMT_MXFP6;
  if (a_dtype != MXP_BF16 && a_dtype != MXP_F32) return MXP_ERR_DTYPE;
  const int rc0 = check_gemm(M, N, K, D, d_dtype, ldd);
  if (rc0 != MXP_OK || M == 0 || N == 0) return rc0;
  hipStream_t s = static_cast<hipStream_t>(stream);
  if (K == 0) return zero_output(D, d_dtype, M, N, ldd, s);
  if (!A || !W_elems || !W_scales || (fmtW != MXP_FMT_MXFP4 && !plain_wide_format(fmtW) && !W_idx)) return MXP_ERR_NULL;
  if (lda < K) return MXP_ERR_SHAPE;
  if (a_dtype != MXP_BF16) return MXP_ERR_UNSUPPORTED;      // the activations are multiplied as bf16
  if (!aligned16(A) || !aligned16(W_elems) || !aligned16(W_scales) || (W_idx && !aligned16(W_idx)) || (lda * 2) % 16 != 0)
    return MXP_ERR_ALIGN;
  const int64_t slab =
      workspace && aligned16(workspace) ? slab_rows(M, N, K, lda, fmtW, ldd % 4 == 0 && aligned16(D), workspace_bytes) : 0;
  if (slab) {
    const int64_t nbk = K / kBlock, esz = d_dtype == MXP_BF16 ? 2 : 4, row_bytes = nbk * block_bytes(fmtW);
    for (int64_t n0 = 0; n0 < N; n0 += slab) {
      const int64_t nr = N - n0 < slab ? N - n0 : slab;
      int rc = dequantize_bf16_launch(W_elems + n0 * row_bytes, W_scales + n0 * nbk, W_idx ? W_idx + n0 * nbk : nullptr, fmtW, nr, K,
                                      workspace, s);
      if (rc != MXP_OK) return rc;
      rc = bf16_gemm_launch(M, nr, K, A, lda, workspace, K, static_cast<uint8_t*>(D) + n0 * esz, d_dtype, ldd, s);
      if (rc != MXP_OK) return rc;
    }
    return MXP_OK;
  }
  // six- and eight-bit weights: a kernel of their own up to 64 rows (above, W read twice is no faster than W as bf16: 100 rows x
  // 4096 x 4096 MXFP8+ 38.3 us), the tiled kernel beyond and for many columns of the shortest K
  if (wide_w && M <= 64 && !tiles_beat_few_rows(M, N, K))
    return few_rows_launch(M, N, K, A, lda, W_elems, W_scales, W_idx, fmtW, D, d_dtype, ldd, s);
  if (wide_w) return dispatch_tiled(M, N, K, A, lda, W_elems, W_scales, W_idx, fmtW, D, d_dtype, ldd, s);
  if (M > 64 && M <= 128) {
    // two passes of the few-row kernel read the weights twice and still beat one row of 256 x 256 tiles here
    const int64_t esz = d_dtype == MXP_BF16 ? 2 : 4;
    for (int64_t r0 = 0; r0 < M; r0 += 64) {
      const int64_t mr = M - r0 < 64 ? M - r0 : 64;
      const void* Ar = static_cast<const uint16_t*>(A) + r0 * lda;
      void* Dr = static_cast<uint8_t*>(D) + r0 * ldd * esz;
      const int rc = fmtW == MXP_FMT_MXFP4PP  ? dispatch_skinny<2>(mr, N, K, Ar, lda, W_elems, W_scales, W_idx, Dr, d_dtype, ldd, s)
                     : fmtW == MXP_FMT_MXFP4P ? dispatch_skinny<1>(mr, N, K, Ar, lda, W_elems, W_scales, W_idx, Dr, d_dtype, ldd, s)
                                              : dispatch_skinny<0>(mr, N, K, Ar, lda, W_elems, W_scales, W_idx, Dr, d_dtype, ldd, s);
      if (rc != MXP_OK) return rc;
    }
    return MXP_OK;
  }
  if (M > 64) return dispatch_tiled(M, N, K, A, lda, W_elems, W_scales, W_idx, fmtW, D, d_dtype, ldd, s);
  if (fmtW == MXP_FMT_MXFP4PP) return dispatch_skinny<2>(M, N, K, A, lda, W_elems, W_scales, W_idx, D, d_dtype, ldd, s);
  if (fmtW == MXP_FMT_MXFP4P) return dispatch_skinny<1>(M, N, K, A, lda, W_elems, W_scales, W_idx, D, d_dtype, ldd, s);
  return dispatch_skinny<0>(M, N, K, A, lda, W_elems, W_scales, W_idx, D, d_dtype, ldd, s);
}

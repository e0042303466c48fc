// D[M][N] = A[M][K] (bf16) x deq(W)[N][K]^T for few rows of A and six- or eight-bit W: W read once, in its canonical bytes, and
// de-converted to bf16 (Eq. 2) by the lane that feeds it to the bf16 MFMA.  Weight-only quantization in the decode stage, and the
// products of mxp_gemm on de-converted operands with few rows.  Otherwise W is written as bf16 and read back: us per call, replayed
// from a graph, that way -> here, 1 x 4096 x 4096 MXFP8+ 37.5 -> 8.2, 13 x 14336 x 4096 MXFP8+ 53.6 -> 26.6, MXFP6+ 52.3 -> 30.1,
// 64 x 8192 x 8192 MXFP8+ 76.8 -> 51.4.  (Four-bit W keeps the kernel of mxp_w4a16.hip: 13 x 14336 x 4096 MXFP4+ 15.0 there | 20.4 here.)
//
// v_mfma_f32_16x16x32_bf16: lane l holds row l % 16 of an operand and eight k-slots of group l / 16.  The sum over k does not care
// which k sits in which slot as long as both operands agree, so the four lane groups take four consecutive MX blocks: in a step of
// 128 of K lane (n, g) loads block g of weight row n as it lies in memory (four lanes: 64 contiguous bytes of a row), de-converts
// its 32 values, and feeds them to four MFMAs, eight at a time; lane (m, g) has the same eight k of activation row m.  W goes first:
// accumulator register r of lane l is D[m = l % 16][n = 4 (l / 16) + r].
// A workgroup owns 16 CT columns and up to 16 MT rows; its wavefronts split K in chunks of two steps, each with all
// loads of a chunk in flight, and the partial tiles are summed through LDS in a fixed order.  Bound by what its two wavefronts a SIMD
// wait for: by counters (13 x 14336 x 4096 MXFP8+ | MXFP6+) the vector ALU is busy 30 | 22 % of the time with the conversion (about 80
// instructions a block), wavefronts are held before an instruction issues 55 | 59 %, in waits 28 %; above 16 rows the reads of A
// come on top: every workgroup reads all of it.
#include "mxp_common.h"
#include "mxp_decode.h"

namespace {

using namespace mxp;
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
typedef __bf16 v8bf __attribute__((ext_vector_type(8)));
typedef float v4f __attribute__((ext_vector_type(4)));

constexpr int kWaves = 8;                                    // wavefronts of a workgroup, which split K

template <int FMT>
struct Few {
  static constexpr bool PLUS = FMT == MXP_FMT_MXFP6P || FMT == MXP_FMT_MXFP8P;
  static constexpr int BITS = FMT < MXP_FMT_MXFP8 ? 6 : 8, DW = BITS;   // dwords of a block's codes
};

// bf16 pair i (elements 2 i, 2 i + 1) of a block, from integer fields: what the de-conversion kernels give
template <int FMT>
__device__ uint32_t general_pair(const uint32_t (&raw)[Few<FMT>::DW], uint32_t sb, uint32_t ib, uint32_t i) {
  constexpr int BITS = Few<FMT>::BITS;
  if (sb == 0u) return 0u;
  if (sb == 255u) return 0x7FC07FC0u;
  const uint32_t bm = Few<FMT>::PLUS ? ib & 31u : 64u;
  uint32_t out = 0;
#pragma unroll
  for (uint32_t e = 0; e < 2; ++e) {
    const uint32_t el = 2u * i + e, bit = (uint32_t)BITS * el, w = bit >> 5, sh = bit & 31u;
    uint32_t lo = 0, hi = 0;
#pragma unroll
    for (int j = 0; j < Few<FMT>::DW; ++j) {
      lo = w == (uint32_t)j ? raw[j] : lo;
      hi = w + 1u == (uint32_t)j ? raw[j] : hi;
    }
    const uint32_t c = (uint32_t)((((uint64_t)hi << 32) | lo) >> sh) & ((1u << BITS) - 1u);
    const uint32_t sign = c >> (BITS - 1), mag = c & ((1u << (BITS - 1)) - 1u);
    constexpr int MB = 3, BIAS = BITS == 6 ? 1 : 7, EMAX = BITS == 6 ? 2 : 8;
    uint32_t bits;
    if (bm == el) {
      bits = wide_f32_bits(sign, (1u << (BITS - 1)) | mag, EMAX - (BITS - 1) + (int)sb - 127);
    } else {
      const uint32_t x = mag >> MB, m = mag & ((1u << MB) - 1u);
      bits = wide_f32_bits(sign, x ? ((1u << MB) | m) : m, (int)(x ? x : 1u) - BIAS - MB + (int)sb - 127);
    }
    const uint32_t h = wide_bf16_rne(bits);
    out |= (h & 0xFFFFu) << (16u * e);
  }
  return out;
}

// 32 codes -> 32 bf16 (16 dwords of pairs).  The unpack-convert instructions run over the whole block with the scale of the ordinary
// elements; the BM's code is taken out of the codes first (code 0 converts to +0) and its value, an exponent and
// mantissa in place, is or-ed onto its pair: the pair of a group of four first, then one and-or per pair with the group's mask.
// Flushed blocks and blocks of NaNs are selected where a lane of the wavefront has one (weights may hold many of the former: one in
// fifty 1.2 times as long as none; pair by pair 5 to 6 times); blocks with E4M3's NaN code, and those whose values may leave the
// bf16 normal range, are made pair by pair, for the whole wavefront.
template <int FMT>
__device__ __forceinline__ void decode(const uint32_t (&raw)[Few<FMT>::DW], uint32_t sb, uint32_t ib, uint32_t (&w)[16]) {
  constexpr int BITS = Few<FMT>::BITS;
  constexpr bool PLUS = Few<FMT>::PLUS;
  constexpr uint32_t EMAX = BITS == 8 ? 8u : 2u;
  const uint32_t idx = ib & 31u;
  uint32_t n[Few<FMT>::DW];
#pragma unroll
  for (int j = 0; j < Few<FMT>::DW; ++j) n[j] = raw[j];
  uint32_t put = 0;
  if constexpr (PLUS) {
    uint32_t code;
    if constexpr (BITS == 6) {
      const SixAt at(idx);
      code = at.get(n);
      at.put(code, n);
      put = ((code & 0x20u) << 10) | ((sb + EMAX) << 7) | ((code & 0x1Fu) << 2);
    } else {
      uint32_t d = n[0];
#pragma unroll
      for (int j = 1; j < 8; ++j) d = (idx >> 2) == (uint32_t)j ? n[j] : d;
      const uint32_t sh = 8u * (idx & 3u);
      code = (d >> sh) & 0xFFu;
#pragma unroll
      for (int j = 0; j < 8; ++j) n[j] ^= (idx >> 2) == (uint32_t)j ? code << sh : 0u;
      put = ((code & 0x80u) << 8) | ((sb + EMAX) << 7) | (code & 0x7Fu);
    }
    put <<= 16u * (idx & 1u);
  }
  // the range in which every value is a normal bf16 number (E4M3 goes 2^9 below X)
  bool plain = sb >= 16u && sb <= 240u;
  if constexpr (BITS == 8) {
    uint32_t nanlike = 0;
#pragma unroll
    for (int j = 0; j < 8; ++j) nanlike |= ((n[j] & 0x7F7F7F7Fu) + 0x01010101u) & 0x80808080u;
    plain = plain && nanlike == 0u;
  }
  const float X = __uint_as_float((plain ? sb : 127u) << 23);
  if constexpr (BITS == 6) {
    union { v32bf_dec v; uint32_t u[16]; } c;
    c.v = __builtin_amdgcn_cvt_scalef32_pk32_bf16_fp6((v6u_dec){n[0], n[1], n[2], n[3], n[4], n[5]}, X);
#pragma unroll
    for (int j = 0; j < 16; ++j) w[j] = c.u[j];
  } else {
#pragma unroll
    for (int j = 0; j < 8; ++j) {
      union { v2bf v; uint32_t u; } c0, c1;
      c0.v = __builtin_amdgcn_cvt_scalef32_pk_bf16_fp8(n[j], X, false);
      c1.v = __builtin_amdgcn_cvt_scalef32_pk_bf16_fp8(n[j], X, true);
      w[2 * j] = c0.u; w[2 * j + 1] = c1.u;
    }
  }
  if constexpr (PLUS) or_onto_pair(idx, put, w);
  if (__builtin_amdgcn_ballot_w64(!plain) == 0) return;
  const bool reserved = sb == 0u || sb == 255u;              // zeros, NaN
  const uint32_t special = sb == 0u ? 0u : 0x7FC07FC0u;
#pragma unroll
  for (int j = 0; j < 16; ++j) w[j] = reserved ? special : w[j];
  if (__builtin_amdgcn_ballot_w64(!plain && !reserved) != 0) {
#pragma unroll 1
    for (uint32_t i = 0; i < 16; ++i) {
      const uint32_t v = general_pair<FMT>(raw, sb, ib, i);
#pragma unroll
      for (int j = 0; j < 16; ++j) w[j] = !plain && i == (uint32_t)j ? v : w[j];
    }
  }
}

template <int FMT, int MT, int CT>
__global__ void __launch_bounds__(64 * kWaves) few_rows_kernel(const uint16_t* __restrict__ A, int64_t lda, const uint8_t* __restrict__ w_el,
                                                              const uint8_t* __restrict__ w_sc, const uint8_t* __restrict__ w_ix, int nbk,
                                                              int M, int64_t N, void* __restrict__ Dv, int64_t ldd, int d_bf16) {
  using F = Few<FMT>;
  constexpr int STEPS = 2;                                   // steps of a chunk
  extern __shared__ __attribute__((aligned(16))) uint8_t lds_raw[];
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int r = lane & 15, g = lane >> 4;
  const int64_t n0 = (int64_t)blockIdx.x * (16 * CT);
  // blocks from the workgroup's first weight row on; rows past N repeat the last one, into columns that are not stored
  const uint8_t *el = w_el + n0 * nbk * (4 * F::DW), *sc = w_sc + n0 * nbk, *ix = F::PLUS ? w_ix + n0 * nbk : nullptr;
  uint32_t off[CT];
#pragma unroll
  for (int j = 0; j < CT; ++j) off[j] = (uint32_t)(n0 + 16 * j + r < N ? 16 * j + r : N - 1 - n0) * (uint32_t)nbk;
  const uint16_t* a_row[MT];
  bool a_ok[MT];
#pragma unroll
  for (int i = 0; i < MT; ++i) {
    a_ok[i] = 16 * i + r < M;
    a_row[i] = A + (a_ok[i] ? (int64_t)(16 * i + r) * lda : 0);
  }
  v4f acc[MT][CT];
#pragma unroll
  for (int i = 0; i < MT; ++i)
#pragma unroll
    for (int j = 0; j < CT; ++j) acc[i][j] = (v4f){0.0f, 0.0f, 0.0f, 0.0f};

  struct Chunk {
    uint32_t raw[STEPS][CT][F::DW], sb[STEPS][CT], ib[STEPS][CT];
  };
  auto load_w = [&](int ci, Chunk& c) {
#pragma unroll
    for (int t = 0; t < STEPS; ++t) {
      const int b = (ci * STEPS + t) * 4 + g;
      const uint32_t bc = (uint32_t)(b < nbk ? b : nbk - 1);   // past the end: A is zero there
#pragma unroll
      for (int j = 0; j < CT; ++j) {
        if constexpr (F::DW == 6) {
          const u32x2* p = reinterpret_cast<const u32x2*>(el + (off[j] + bc) * 24u);
          const u32x2 d0 = __builtin_nontemporal_load(p), d1 = __builtin_nontemporal_load(p + 1), d2 = __builtin_nontemporal_load(p + 2);
          c.raw[t][j][0] = d0.x; c.raw[t][j][1] = d0.y; c.raw[t][j][2] = d1.x; c.raw[t][j][3] = d1.y; c.raw[t][j][4] = d2.x; c.raw[t][j][5] = d2.y;
        } else {
#pragma unroll
          for (int q = 0; q < F::DW / 4; ++q) {
            const u32x4 d = __builtin_nontemporal_load(reinterpret_cast<const u32x4*>(el + (off[j] + bc) * (4u * F::DW) + 16 * q));
            c.raw[t][j][4 * q] = d.x; c.raw[t][j][4 * q + 1] = d.y; c.raw[t][j][4 * q + 2] = d.z; c.raw[t][j][4 * q + 3] = d.w;
          }
        }
        c.sb[t][j] = sc[off[j] + bc];
        c.ib[t][j] = F::PLUS ? (uint32_t)ix[off[j] + bc] : 0u;
      }
    }
  };
  const int n_chunks = (nbk + 4 * STEPS - 1) / (4 * STEPS);
  const int first = (int)((blockIdx.x * 5u) % (uint32_t)n_chunks);   // (workgroups start their walk at different chunks)
  for (int ci = wave; ci < n_chunks; ci += kWaves) {
    const int q = ci + first < n_chunks ? ci + first : ci + first - n_chunks;
    Chunk c;
    load_w(q, c);
    u32x4 a[STEPS][MT][4];
#pragma unroll
    for (int t = 0; t < STEPS; ++t) {
      const int b = (q * STEPS + t) * 4 + g;
      const bool in = b < nbk;
#pragma unroll
      for (int i = 0; i < MT; ++i)
#pragma unroll
        for (int s = 0; s < 4; ++s) {
          a[t][i][s] = (u32x4){0, 0, 0, 0};
          if (a_ok[i] && in) a[t][i][s] = *reinterpret_cast<const u32x4*>(a_row[i] + (int64_t)b * 32 + 8 * s);
        }
    }
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int t = 0; t < STEPS; ++t) {
      const bool in = (q * STEPS + t) * 4 + g < nbk;
#pragma unroll
      for (int j = 0; j < CT; ++j) {
        uint32_t w[16];
        decode<FMT>(c.raw[t][j], in ? c.sb[t][j] : 127u, c.ib[t][j], w);   // (past K any finite number does: A is zero there)
#pragma unroll
        for (int s = 0; s < 4; ++s) {
          union { u32x4 u; v8bf b; } x, y;
          x.u = (u32x4){w[4 * s], w[4 * s + 1], w[4 * s + 2], w[4 * s + 3]};
#pragma unroll
          for (int i = 0; i < MT; ++i) {
            y.u = a[t][i][s];
            acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(x.b, y.b, acc[i][j], 0, 0, 0);
          }
        }
      }
    }
  }
  // partial tiles: register r of a tile 66 floats on, so that the four columns of a lane lie on different banks
  constexpr int TILE = 4 * 66;
  float* part = reinterpret_cast<float*>(lds_raw);          // [kWaves][MT * CT][TILE]
#pragma unroll
  for (int i = 0; i < MT; ++i)
#pragma unroll
    for (int j = 0; j < CT; ++j)
#pragma unroll
      for (int q = 0; q < 4; ++q) part[(wave * MT * CT + i * CT + j) * TILE + q * 66 + lane] = acc[i][j][q];
  __syncthreads();
  constexpr int COLS = 16 * CT;
  for (int e = tid; e < MT * 16 * COLS; e += 64 * kWaves) {
    const int row = e / COLS, c = e % COLS, i = row >> 4, j = c >> 4;
    const float* p = part + (i * CT + j) * TILE + (c & 3) * 66 + (row & 15) + 16 * ((c & 15) >> 2);
    float v = 0.0f;
#pragma unroll
    for (int w = 0; w < kWaves; ++w) v += p[w * MT * CT * TILE];
    const int64_t col = n0 + c;
    if (row < M && col < N) {
      if (d_bf16) {
        const uint32_t u = __float_as_uint(v);
        static_cast<uint16_t*>(Dv)[row * ldd + col] =
            (uint16_t)((u & 0x7FFFFFFFu) > 0x7F800000u ? (u >> 16) | 0x0040u : (u + 0x7FFFu + ((u >> 16) & 1u)) >> 16);
      } else {
        static_cast<float*>(Dv)[row * ldd + col] = v;
      }
    }
  }
}

template <int FMT, int MT, int CT>
int launch_few(int64_t M, int64_t N, int64_t K, const void* A, int64_t lda, const uint8_t* we, const uint8_t* ws, const uint8_t* wi, void* D,
               int d_dtype, int64_t ldd, hipStream_t s) {
  constexpr int lds = kWaves * MT * CT * 4 * 66 * 4;
  static_assert(lds <= 160 * 1024, "LDS");
  const int64_t grid = (N + 16 * CT - 1) / (16 * CT);
  if (grid > 2147483647LL) return MXP_ERR_UNSUPPORTED;
  allow_dynamic_lds<&few_rows_kernel<FMT, MT, CT>>(lds);
  hipLaunchKernelGGL((few_rows_kernel<FMT, MT, CT>), dim3((unsigned)grid), dim3(64 * kWaves), lds, s, static_cast<const uint16_t*>(A), lda, we, ws,
                     wi, (int)(K / kBlock), (int)M, N, D, ldd, d_dtype == MXP_BF16 ? 1 : 0);
  return launch_status();
}

// Columns per workgroup: 16 while that fills one round of the chip (M = 16, K = 4096: N = 3000 11 us with 16 columns | 16 with 32),
// then 32 (N = 5000 18.8 | 16.3, K = 8192 and N = 8192 36.0 | 31.1), and 64 from 700 tiles of 16 on, where the reads of A weigh more
// (K = 8192, N = 14336: 16 rows 55.5 with 32 | 51.6 with 64, 32 rows 73.1 | 60.3); above 32 rows 64 columns do not fit the registers.
template <int FMT>
int launch_few_format(int64_t M, int64_t N, int64_t K, const void* A, int64_t lda, const uint8_t* we, const uint8_t* ws, const uint8_t* wi,
                      void* D, int d_dtype, int64_t ldd, hipStream_t s) {
#define MXP_FEW(MT, CT) return launch_few<FMT, MT, CT>(M, N, K, A, lda, we, ws, wi, D, d_dtype, ldd, s)
  const int64_t c16 = (N + 15) / 16;
  if (M <= 16) {
    if (c16 <= kNumCU) MXP_FEW(1, 1);
    if (c16 <= 700) MXP_FEW(1, 2);
    MXP_FEW(1, 4);
  }
  if (M <= 32) {
    if (c16 <= kNumCU) MXP_FEW(2, 1);
    if (c16 <= 2 * kNumCU) MXP_FEW(2, 2);                    // (one workgroup per compute unit: a second round would be nearly empty)
    MXP_FEW(2, 4);
  }
  if (c16 <= kNumCU) MXP_FEW(4, 1);
  MXP_FEW(4, 2);
#undef MXP_FEW
}

}  // namespace

namespace mxp {
int few_rows_launch(int64_t M, int64_t N, int64_t K, const void* A, int64_t lda, const uint8_t* we, const uint8_t* ws, const uint8_t* wi, int fmtW,
                    void* D, int d_dtype, int64_t ldd, hipStream_t s) {
  switch (fmtW) {
    case MXP_FMT_MXFP6: return launch_few_format<MXP_FMT_MXFP6>(M, N, K, A, lda, we, ws, wi, D, d_dtype, ldd, s);
    case MXP_FMT_MXFP6P: return launch_few_format<MXP_FMT_MXFP6P>(M, N, K, A, lda, we, ws, wi, D, d_dtype, ldd, s);
    case MXP_FMT_MXFP8: return launch_few_format<MXP_FMT_MXFP8>(M, N, K, A, lda, we, ws, wi, D, d_dtype, ldd, s);
    default: return launch_few_format<MXP_FMT_MXFP8P>(M, N, K, A, lda, we, ws, wi, D, d_dtype, ldd, s);
  }
}
}  // namespace mxp

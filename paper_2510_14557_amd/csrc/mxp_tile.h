// Epilogue and work-list pieces shared by the tiled products.  Device code only.
#pragma once
#include "mxp_common.h"

namespace mxp {

typedef float v16f __attribute__((ext_vector_type(16)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));

// fp32 -> bf16, round to nearest even, NaN stays NaN: the CDNA4 pack-convert instruction (one per two values).
typedef float f32x2 __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
__device__ __forceinline__ uint32_t pack_bf16x2(float lo, float hi) {
  union { bf16x2 v; uint32_t u; } c;
  c.v = __builtin_convertvector((f32x2){lo, hi}, bf16x2);
  return c.u;
}
__device__ __forceinline__ uint32_t f32_to_bf16_rne(float v) { return pack_bf16x2(v, 0.0f) & 0xFFFFu; }

// Epilogue through LDS for the large kernel.  Stored straight from the accumulator layout, a store instruction touches
// 64 different 128-byte lines with 16 bytes each, and the L2 then sees 4096 partial-line writes per wavefront tile.
// Each 32 x 32 tile is therefore passed through a private 32 x 36-float LDS patch (rows padded by 16 bytes against bank
// conflicts; LDS operations of one wavefront execute in order, so no wait is needed between the write and the read)
// and comes back with 8 consecutive lanes holding the 128 contiguous bytes of one row: every store instruction
// writes 8 full lines.  `patch` is this wavefront's scratch, two patches of kPatchBytes.  STREAM: streaming stores.
// COLUMNS: a lane per column where rows of D do not start at 16-byte addresses.
constexpr int kPatchStride = 144;                 // bytes per patch row: 32 floats + 16
constexpr int kPatchBytes = 32 * kPatchStride;

template <int TWM, int TWN, bool OUT_BF16, bool STREAM = true, bool COLUMNS = false>
__device__ __forceinline__ void store_tile_lds(const v16f (&acc)[TWM][TWN], int64_t tile_m, int64_t tile_n, int lane, int64_t M,
                                               int64_t N, void* __restrict__ Dv, int64_t ldd, uint8_t* patch) {
  typedef float f32x4 __attribute__((ext_vector_type(4)));
  const bool vec_ok = (ldd % 4 == 0) && ((reinterpret_cast<uintptr_t>(Dv) & 15u) == 0);
  auto put = [](auto* at, auto v) {
    if constexpr (STREAM) __builtin_nontemporal_store(v, at);
    else *at = v;
  };
  const int wr = (lane & 31) * kPatchStride + 16 * (lane >> 5);   // + 32 g
  const int rd = (lane >> 3) * kPatchStride + (lane & 7) * 16;    // + 8 k rows
  if (OUT_BF16 && vec_ok && TWN % 2 == 0) {
    // bf16: a row of one tile is only 64 bytes.  Two neighbouring tiles go through the two patches together and 16
    // consecutive lanes then hold the 128 contiguous bytes of one row (64 columns), so every store writes whole lines.
    const int rd2 = (lane >> 4) * kPatchStride + (lane & 7) * 16;  // + 4 k rows; patch (lane & 15) >> 3
    const uint8_t* pr = patch + ((lane & 15) >> 3) * kPatchBytes;
#pragma unroll
    for (int i = 0; i < TWM; ++i) {
#pragma unroll
      for (int j = 0; j < TWN; j += 2) {
#pragma unroll
        for (int t = 0; t < 2; ++t)
#pragma unroll
          for (int g = 0; g < 4; ++g) {
            f32x4 q = {acc[i][j + t][4 * g], acc[i][j + t][4 * g + 1], acc[i][j + t][4 * g + 2], acc[i][j + t][4 * g + 3]};
            *reinterpret_cast<f32x4*>(patch + t * kPatchBytes + wr + 32 * g) = q;
          }
        const int64_t col = (tile_n + j) * 32 + 4 * (lane & 15);
#pragma unroll
        for (int k = 0; k < 8; ++k) {
          const f32x4 v = *reinterpret_cast<const f32x4*>(pr + rd2 + 4 * k * kPatchStride);
          const int64_t row = (tile_m + i) * 32 + 4 * k + (lane >> 4);
          if (row >= M || col >= N) continue;
          if (col + 3 < N) {
            u32x2 o = {pack_bf16x2(v[0], v[1]), pack_bf16x2(v[2], v[3])};
            put(reinterpret_cast<u32x2*>(static_cast<uint16_t*>(Dv) + row * ldd + col), o);
          } else {
#pragma unroll
            for (int q = 0; q < 4; ++q)
              if (col + q < N) static_cast<uint16_t*>(Dv)[row * ldd + col + q] = (uint16_t)f32_to_bf16_rne(v[q]);
          }
        }
      }
    }
    return;
  }
#pragma unroll
  for (int i = 0; i < TWM; ++i) {
#pragma unroll
    for (int j = 0; j < TWN; ++j) {
      uint8_t* pb = patch + ((i * TWN + j) & 1) * kPatchBytes;
#pragma unroll
      for (int g = 0; g < 4; ++g) {
        f32x4 q = {acc[i][j][4 * g], acc[i][j][4 * g + 1], acc[i][j][4 * g + 2], acc[i][j][4 * g + 3]};
        *reinterpret_cast<f32x4*>(pb + wr + 32 * g) = q;
      }
      if (COLUMNS && !vec_ok) {
        // rows of D anywhere: a lane per column, so that a store instruction covers two whole rows of the tile.
        // (Not in the large kernels, whose loops lose registers to it: the 4096 x 14336 x 4096 step 172 | 181 us.)
        const int64_t col = (tile_n + j) * 32 + (lane & 31);
#pragma unroll
        for (int k = 0; k < 16; ++k) {
          const float v = *reinterpret_cast<const float*>(pb + (2 * k + (lane >> 5)) * kPatchStride + 4 * (lane & 31));
          const int64_t row = (tile_m + i) * 32 + 2 * k + (lane >> 5);
          if (row >= M || col >= N) continue;
          if (OUT_BF16) static_cast<uint16_t*>(Dv)[row * ldd + col] = (uint16_t)f32_to_bf16_rne(v);
          else static_cast<float*>(Dv)[row * ldd + col] = v;
        }
        continue;
      }
      const int64_t col = (tile_n + j) * 32 + 4 * (lane & 7);
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        const f32x4 v = *reinterpret_cast<const f32x4*>(pb + rd + 8 * k * kPatchStride);
        const int64_t row = (tile_m + i) * 32 + 8 * k + (lane >> 3);
        if (row >= M || col >= N) continue;
        if (vec_ok && col + 3 < N) {
          if (OUT_BF16) {
            u32x2 o = {pack_bf16x2(v[0], v[1]), pack_bf16x2(v[2], v[3])};
            put(reinterpret_cast<u32x2*>(static_cast<uint16_t*>(Dv) + row * ldd + col), o);
          } else {
            put(reinterpret_cast<f32x4*>(static_cast<float*>(Dv) + row * ldd + col), v);
          }
        } else {
#pragma unroll
          for (int q = 0; q < 4; ++q) {
            if (col + q < N) {
              if (OUT_BF16) static_cast<uint16_t*>(Dv)[row * ldd + col + q] = (uint16_t)f32_to_bf16_rne(v[q]);
              else static_cast<float*>(Dv)[row * ldd + col + q] = v[q];
            }
          }
        }
      }
    }
  }
}

constexpr int kBand = 4;

__device__ __forceinline__ void band_decode(int p, int rows, int cols, int& r, int& c, int band_cols = kBand) {
  const int per_band = band_cols * rows;
  const int band = p / per_band, q = p - band * per_band;
  const int c0 = band * band_cols;
  const int w = cols - c0 < band_cols ? cols - c0 : band_cols;
  r = q / w;
  c = c0 + (q - r * w);
}

}  // namespace mxp

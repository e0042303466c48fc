// mxp_gemm on canonical four- and six-bit operands without images: D[M][N] = deq(A)[M][K] x deq(B)[N][K]^T, every block
// brought into the form of a block-scaled MFMA operand inside the product kernel, once per workgroup.
//
// An operand image (mxp_prepack and its relatives) pays where it is read many times: by a product of many tiles, or by many
// products.  A product of one round of workgroups reads each block a few times only, and there the images cost more than the
// product: two launches ahead of it and 6.25 or, over two K segments, 12.5 bits an element written and read back.  Here a
// workgroup reads the 4.5 bits.
//
// One workgroup computes a tile of 64 WI x 64 WJ outputs.  K goes by in steps of KS blocks.  Four wavefronts multiply, 2 x 2 over the
// tile; eight convert: thread t of these owns block t % KS of rows t / KS, t / KS + 512 / KS, ... of a step, loads their codes,
// scale and index bytes three steps ahead of the products (128 contiguous bytes of a row by eight lanes), and stores the operand
// terms that they make to the LDS stage of the step that is multiplied next.  One barrier per step.  No unit bounds a step alone:
// 1024 x 4096 x 4096 MXFP4++ x MXFP4+ 1.7 us a step, of which (variants without them) the stores 0.7, at the 64 bytes a clock that
// LDS takes, the conversions 0.6, the products and their operand reads 1.0, partly at the same time; loads alone nearly nothing.  By
// counters (1037 x 3001 x 4128, 37.7 us) the vector ALU is busy 57 % of the time, LDS 29 %, the matrix cores 21 %.
// Measured and slower, us a call for that product | MXFP4+ x MXFP4: this 36 | 27 (replayed from a graph 33.6 | 24.8);
// conversions between the MFMAs of the same eight wavefronts 46 | 36; canonical bytes through LDS and K split over four wavefronts
// that convert in operand order 43 | 34; four converting wavefronts 45 | 32; four-byte loads of scale and index bytes, shared by a
// quad, 36 | 28.
//
// Terms of a block, each an exact E2M1 or E2M3 operand with a scale byte of its own (Sec. 4.2, 4.3; Eq. 3):
//   MXFP4    the codes as they are (E2M1)
//   MXFP4+   one E2M3 term: codes widened, the BM at exponent e_max
//   MXFP4++  the codes without the BM (E2M1), scale lowered by delta | the BM alone (E2M3)
//   MXFP6    the codes as they are (E2M3)
//   MXFP6+   the codes with BM_H in the BM's place (E2M3) | BM_L alone (E2M3)
// A pair of blocks takes as many MFMAs as the product of their numbers of terms.
#include "mxp_common.h"
#include "mxp_decode.h"
#include "mxp_prepack_body.h"
#include "mxp_tile.h"
#include <type_traits>

namespace {

using namespace mxp;
typedef int v8i __attribute__((ext_vector_type(8)));

constexpr int kConverting = 8;                               // converting wavefronts of a workgroup (four: 36 -> 45 us, head of this file)
constexpr int kE2M3 = 2, kE2M1 = 4;                          // element format codes of the f8f6f4 MFMA

// Element formats of the terms and bytes of a canonical block, by format code (MXP_FMT_*)
template <int FMT>
struct Kind {
  static constexpr bool PLUS = FMT == MXP_FMT_MXFP4P || FMT == MXP_FMT_MXFP4PP || FMT == MXP_FMT_MXFP6P;   // has index bytes
  static constexpr bool SIX = FMT == MXP_FMT_MXFP6 || FMT == MXP_FMT_MXFP6P;
  static constexpr int TERMS = FMT == MXP_FMT_MXFP4PP || FMT == MXP_FMT_MXFP6P ? 2 : 1;
  static constexpr int F0 = FMT == MXP_FMT_MXFP4 || FMT == MXP_FMT_MXFP4PP ? kE2M1 : kE2M3, F1 = kE2M3;
  static constexpr bool OWN_SCALE = FMT == MXP_FMT_MXFP4PP;  // the terms' scale bytes differ
  static constexpr int BLOCK = SIX ? 24 : 16;
};

// One operand of a step in LDS: for every term [row tile][block] runs of 32 rows x 16 bytes and, for E2M3 terms, of 32 rows x 8
// bytes; then the scale bytes, [block][row of a tile] dwords whose byte q belongs to row tile q.  The runs are padded by 32 bytes
// (the scale runs by 16): a store instruction of the threads of 8 rows x 8 blocks then covers all banks once, as does a read of 64
// consecutive lanes.
constexpr int kLoRun = 32 * 16 + 16, kHiRun = 32 * 8 + 16, kScRun = 32 * 4 + 8;
template <int FMT, int TILES, int KS>
struct Region {
  using K = Kind<FMT>;
  static constexpr int LO = TILES * KS * kLoRun, HI = TILES * KS * kHiRun;
  static constexpr int TERM0 = 0, TERM1 = LO + (K::F0 == kE2M3 ? HI : 0);
  static constexpr int SC0 = TERM1 + (K::TERMS == 2 ? LO + HI : 0), SC1 = SC0 + (K::OWN_SCALE ? KS * kScRun : 0);
  static constexpr int BYTES = SC1 + KS * kScRun;
};

template <int FMT>
struct Block {                                               // a canonical block as loaded
  uint32_t raw[Kind<FMT>::SIX ? 6 : 4];
  uint32_t sb, ib;
};

template <int FMT>
__device__ __forceinline__ Block<FMT> load_block(const uint8_t* el, const uint8_t* sc, const uint8_t* ix, uint32_t b) {
  Block<FMT> r;
  if constexpr (Kind<FMT>::SIX) {
    const u32x2* p = reinterpret_cast<const u32x2*>(el + b * 24u);
    const u32x2 d0 = p[0], d1 = p[1], d2 = p[2];
    r.raw[0] = d0.x; r.raw[1] = d0.y; r.raw[2] = d1.x; r.raw[3] = d1.y; r.raw[4] = d2.x; r.raw[5] = d2.y;
  } else {
    const u32x4 d = *reinterpret_cast<const u32x4*>(el + b * 16u);
    r.raw[0] = d.x; r.raw[1] = d.y; r.raw[2] = d.z; r.raw[3] = d.w;
  }
  r.sb = sc[b];
  r.ib = Kind<FMT>::PLUS ? (uint32_t)ix[b] : 0u;
  return r;
}

// Block -> terms t0, t1 (four dwords count of an E2M1 term, six of an E2M3 one) and their scale bytes.  A block outside the
// matrix (!ok) counts as a flushed one: scale byte 0, zeros whatever its codes say.
template <int FMT>
__device__ __forceinline__ void to_terms(const Block<FMT>& r, bool ok, uint32_t (&t0)[6], uint32_t (&t1)[6], uint32_t& s0, uint32_t& s1) {
  constexpr int W = Kind<FMT>::SIX ? 6 : 4;
  const uint32_t sb = ok ? r.sb : 0u;
  const bool flushed = sb == 0u, live = sb - 1u < 254u;      // live: neither flushed nor NaN, the block has a BM
  uint32_t n[W];
#pragma unroll
  for (int j = 0; j < W; ++j) n[j] = flushed ? 0u : r.raw[j];
  s0 = s1 = sb;
  const uint32_t bm = r.ib & 31u;
  if constexpr (FMT == MXP_FMT_MXFP4 || FMT == MXP_FMT_MXFP6) {
#pragma unroll
    for (int j = 0; j < W; ++j) t0[j] = n[j];
  } else if constexpr (FMT == MXP_FMT_MXFP6P) {
    const SixAt at(bm);
    const uint32_t c = at.get(n);                            // s mmmmm -> s 11 m4m3m2 in place, s 00 0m1m0 beside it
#pragma unroll
    for (int j = 0; j < 6; ++j) { t0[j] = n[j]; t1[j] = 0u; }
    at.put(live ? c ^ ((c & 0x20u) | 0x18u | ((c >> 2) & 7u)) : 0u, t0);
    at.put(live ? (c & 0x23u) : 0u, t1);
  } else {
    const FourAt at(bm);
    const uint32_t nib = at.get(n);
    const uint32_t code = ((nib & 8u) << 2) | 0x18u | (nib & 7u);                  // the BM: s 11 mmm
    if constexpr (FMT == MXP_FMT_MXFP4PP) {
      const uint32_t delta = r.ib >> 5, lowered = delta < sb ? sb - delta : 1u;   // (a delta beyond sb - 1 is not written by a conversion)
      s0 = live ? lowered : sb;
      at.put(live ? nib : 0u, n);
#pragma unroll
      for (int j = 0; j < 4; ++j) t0[j] = n[j];
#pragma unroll
      for (int j = 0; j < 6; ++j) t1[j] = 0u;
      SixAt(bm).put(live ? code : 0u, t1);
    } else {
      widen_e2m3(n, t0);
      SixAt(bm).put(live ? (nib << 2) ^ code : 0u, t0);
    }
  }
}

template <int FMT, int TILES, int KS>
__device__ __forceinline__ void store_block(uint8_t* region, uint32_t row, uint32_t kb, const Block<FMT>& r, bool ok) {
  using K = Kind<FMT>;
  using R = Region<FMT, TILES, KS>;
  uint32_t t0[6], t1[6], s0, s1;
  to_terms<FMT>(r, ok, t0, t1, s0, s1);
  const uint32_t rt = row >> 5, rr = row & 31u, run = rt * KS + kb;
  *reinterpret_cast<u32x4*>(region + R::TERM0 + run * kLoRun + rr * 16u) = (u32x4){t0[0], t0[1], t0[2], t0[3]};
  if (K::F0 == kE2M3) *reinterpret_cast<u32x2*>(region + R::TERM0 + R::LO + run * kHiRun + rr * 8u) = (u32x2){t0[4], t0[5]};
  if (K::TERMS == 2) {
    *reinterpret_cast<u32x4*>(region + R::TERM1 + run * kLoRun + rr * 16u) = (u32x4){t1[0], t1[1], t1[2], t1[3]};
    *reinterpret_cast<u32x2*>(region + R::TERM1 + R::LO + run * kHiRun + rr * 8u) = (u32x2){t1[4], t1[5]};
  }
  region[R::SC0 + kb * kScRun + rr * 4u + rt] = (uint8_t)s0;
  if (K::OWN_SCALE) region[R::SC1 + kb * kScRun + rr * 4u + rt] = (uint8_t)s1;
}

// Term T of row tile `rt`, blocks kb (lanes 0 .. 31) and kb + 1 (lanes 32 .. 63), as an MFMA operand
template <int FMT, int TILES, int KS, int T>
__device__ __forceinline__ v8i read_term(const uint8_t* region, uint32_t rt, uint32_t kb, uint32_t rr) {
  using R = Region<FMT, TILES, KS>;
  constexpr int BASE = T == 0 ? R::TERM0 : R::TERM1, F = T == 0 ? Kind<FMT>::F0 : Kind<FMT>::F1;
  const uint32_t run = rt * KS + kb;
  const u32x4 lo = *reinterpret_cast<const u32x4*>(region + BASE + run * kLoRun + rr * 16u);
  u32x2 hi = {0, 0};
  if (F == kE2M3) hi = *reinterpret_cast<const u32x2*>(region + BASE + R::LO + run * kHiRun + rr * 8u);
  return (v8i){(int)lo.x, (int)lo.y, (int)lo.z, (int)lo.w, (int)hi.x, (int)hi.y, 0, 0};
}

struct CanonOperand {
  const uint8_t *el, *sc, *ix;
  int64_t rows;
};

// 2 x 2 wavefronts of WI x WJ MFMA tiles each multiply; kConverting more convert.  The B tile goes in as the MFMA's first operand:
// accumulator register r of lane l is D[m = l % 32][n = 8 (r / 4) + 4 (l / 32) + r % 4] of the 32 x 32 tile.
template <int FA, int FB, int WI, int WJ, int KS>
__global__ void __launch_bounds__(64 * (4 + kConverting)) canon_tiled_kernel(CanonOperand A, CanonOperand B, int nbk, void* __restrict__ Dv, int64_t ldd,
                                                                    int d_bf16, int n_rg, int n_cg) {
  constexpr int TR = 2 * WI, TC = 2 * WJ;
  static_assert(TR <= 4 && TC <= 4, "a scale dword has four tiles");
  using KA = Kind<FA>;
  using KB = Kind<FB>;
  using RA = Region<FA, TR, KS>;
  using RB = Region<FB, TC, KS>;
  constexpr int STAGE = RA::BYTES + RB::BYTES;
  extern __shared__ __attribute__((aligned(16))) uint8_t lds[];
  const uint32_t lane = threadIdx.x & 63u;
  const uint32_t wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);

  // workgroups are dealt round-robin to the XCDs: each takes a contiguous run of positions in bands of 8 tile columns
  const int T = n_rg * n_cg, c = blockIdx.x, x = c & 7, base = T >> 3, rem = T & 7;
  int rg, cg;
  band_decode(x * base + (x < rem ? x : rem) + (c >> 3), n_rg, n_cg, rg, cg, 8);
  const int64_t m0 = (int64_t)rg * (32 * TR), n0 = (int64_t)cg * (32 * TC);
  const int steps = (nbk + KS - 1) / KS;
  // the stage of the next step is written, the present one read: everybody's LDS operations are done
  auto meet = [] { asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory"); };

  if (wave >= 4) {                                           // ---- convert
    constexpr int ROWS_PER_PASS = 64 * kConverting / KS, UA = 32 * TR / ROWS_PER_PASS, UB = 32 * TC / ROWS_PER_PASS;
    static_assert(UA >= 1 && UB >= 1, "every converting thread owns a block of either operand");
    // this thread's blocks; offsets count blocks from the tile's first one (a tile of 128 rows has fewer than 2^24)
    const uint32_t t = threadIdx.x - 256u, kb = t % KS, r0 = t / KS;
    const uint8_t *a_el = A.el + m0 * nbk * KA::BLOCK, *a_sc = A.sc + m0 * nbk, *a_ix = KA::PLUS ? A.ix + m0 * nbk : nullptr;
    const uint8_t *b_el = B.el + n0 * nbk * KB::BLOCK, *b_sc = B.sc + n0 * nbk, *b_ix = KB::PLUS ? B.ix + n0 * nbk : nullptr;
    uint32_t offA[UA], offB[UB];
    bool okA[UA], okB[UB];
#pragma unroll
    for (int u = 0; u < UA; ++u) {
      const uint32_t r = r0 + (uint32_t)(u * ROWS_PER_PASS);
      okA[u] = m0 + r < A.rows;
      offA[u] = okA[u] ? r * (uint32_t)nbk : 0u;
    }
#pragma unroll
    for (int u = 0; u < UB; ++u) {
      const uint32_t r = r0 + (uint32_t)(u * ROWS_PER_PASS);
      okB[u] = n0 + r < B.rows;
      offB[u] = okB[u] ? r * (uint32_t)nbk : 0u;
    }
    struct Step {
      Block<FA> a[UA];
      Block<FB> b[UB];
      bool in_k;
    };
    auto load_step = [&](int s, Step& r) {
      const uint32_t k = (uint32_t)s * KS + kb;
      r.in_k = k < (uint32_t)nbk;
      const uint32_t kc = r.in_k ? k : 0u;
#pragma unroll
      for (int u = 0; u < UA; ++u) r.a[u] = load_block<FA>(a_el, a_sc, a_ix, offA[u] + kc);
#pragma unroll
      for (int u = 0; u < UB; ++u) r.b[u] = load_block<FB>(b_el, b_sc, b_ix, offB[u] + kc);
      __builtin_amdgcn_sched_barrier(0);                     // the loads fly from here on, not from where their values are wanted
    };
    auto store_step = [&](uint8_t* st, const Step& r) {
#pragma unroll
      for (int u = 0; u < UA; ++u) store_block<FA, TR, KS>(st, r0 + (uint32_t)(u * ROWS_PER_PASS), kb, r.a[u], r.in_k && okA[u]);
#pragma unroll
      for (int u = 0; u < UB; ++u) store_block<FB, TC, KS>(st + RA::BYTES, r0 + (uint32_t)(u * ROWS_PER_PASS), kb, r.b[u], r.in_k && okB[u]);
    };
    Step r0s, r1s;
    load_step(0, r1s);
    load_step(1, r0s);
    store_step(lds, r1s);
    load_step(2, r1s);
    meet();
    for (int s = 0; s < steps; s += 2) {                     // while step s is multiplied, step s + 1 is converted and s + 3 loaded
      store_step(lds + STAGE, r0s);
      load_step(s + 3, r0s);
      meet();
      if (s + 1 >= steps) break;
      store_step(lds, r1s);
      load_step(s + 4, r1s);
      meet();
    }
    return;
  }

  // ---- multiply
  const uint32_t wm = wave >> 1, wn = wave & 1u, h = lane >> 5, rr = lane & 31u;
  v16f acc[WI][WJ];
#pragma unroll
  for (int i = 0; i < WI; ++i)
#pragma unroll
    for (int j = 0; j < WJ; ++j)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.0f;
  struct Operands {                                          // of one k-tile
    v8i a0[WI], a1[WI], b0[WJ], b1[WJ];
    uint32_t sa0, sa1, sb0, sb1;
  };
  auto read = [&](const uint8_t* st, uint32_t kt, Operands& o) {
    const uint32_t k2 = 2u * kt + h;
    const uint8_t* stb = st + RA::BYTES;
    o.sb0 = *reinterpret_cast<const uint32_t*>(stb + RB::SC0 + k2 * kScRun + rr * 4u) >> (8u * wn * WJ);
    o.sb1 = KB::OWN_SCALE ? *reinterpret_cast<const uint32_t*>(stb + RB::SC1 + k2 * kScRun + rr * 4u) >> (8u * wn * WJ) : o.sb0;
    o.sa0 = *reinterpret_cast<const uint32_t*>(st + RA::SC0 + k2 * kScRun + rr * 4u) >> (8u * wm * WI);
    o.sa1 = KA::OWN_SCALE ? *reinterpret_cast<const uint32_t*>(st + RA::SC1 + k2 * kScRun + rr * 4u) >> (8u * wm * WI) : o.sa0;
#pragma unroll
    for (int j = 0; j < WJ; ++j) o.b0[j] = read_term<FB, TC, KS, 0>(stb, wn * WJ + j, k2, rr);
#pragma unroll
    for (int i = 0; i < WI; ++i) o.a0[i] = read_term<FA, TR, KS, 0>(st, wm * WI + i, k2, rr);
    if constexpr (KA::TERMS == 2)
#pragma unroll
      for (int i = 0; i < WI; ++i) o.a1[i] = read_term<FA, TR, KS, 1>(st, wm * WI + i, k2, rr);
    if constexpr (KB::TERMS == 2)
#pragma unroll
      for (int j = 0; j < WJ; ++j) o.b1[j] = read_term<FB, TC, KS, 1>(stb, wn * WJ + j, k2, rr);
  };
  // one pair of terms over all tiles, then the next: consecutive MFMAs have different accumulators
  auto tiles = [&](const v8i (&a)[WI], const v8i (&b)[WJ], uint32_t sa, uint32_t sb, auto fa, auto fb) {
    constexpr int Fa = decltype(fa)::value, Fb = decltype(fb)::value;
#define MXP_PAIR(I, J) acc[I][J] = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(b[J], a[I], acc[I][J], Fb, Fa, J, (int)sb, I, (int)sa)
    MXP_PAIR(0, 0);
    if constexpr (WJ > 1) MXP_PAIR(0, 1);
    if constexpr (WI > 1 && WJ > 1) MXP_PAIR(1, 1);
    if constexpr (WI > 1) MXP_PAIR(1, 0);
#undef MXP_PAIR
    static_assert(WI <= 2 && WJ <= 2, "tiles per wavefront");
  };
  auto multiply = [&](const Operands& o) {
    using A0 = std::integral_constant<int, KA::F0>;
    using A1 = std::integral_constant<int, KA::F1>;
    using B0 = std::integral_constant<int, KB::F0>;
    using B1 = std::integral_constant<int, KB::F1>;
    tiles(o.a0, o.b0, o.sa0, o.sb0, A0{}, B0{});
    if constexpr (KA::TERMS == 2) tiles(o.a1, o.b0, o.sa1, o.sb0, A1{}, B0{});
    if constexpr (KB::TERMS == 2) tiles(o.a0, o.b1, o.sa0, o.sb1, A0{}, B1{});
    if constexpr (KA::TERMS == 2 && KB::TERMS == 2) tiles(o.a1, o.b1, o.sa1, o.sb1, A1{}, B1{});
  };
  meet();
  for (int s = 0; s < steps; ++s) {
    const uint8_t* st = lds + (s & 1) * STAGE;
    Operands even, odd;                                      // a k-tile's operands are read while the one before is multiplied
    if constexpr (WI * WJ == 4 && KA::TERMS + KB::TERMS > 2) {   // (two sets of operands do not fit the registers)
#pragma unroll
      for (uint32_t kt = 0; kt < KS / 2; ++kt) {
        read(st, kt, even);
        multiply(even);
      }
      meet();
      continue;
    }
    read(st, 0, even);
#pragma unroll
    for (uint32_t kt = 0; kt < KS / 2; kt += 2) {
      read(st, kt + 1, odd);
      __builtin_amdgcn_sched_barrier(0);
      multiply(even);
      if (kt + 2 < KS / 2) read(st, kt + 2, even);
      __builtin_amdgcn_sched_barrier(0);
      multiply(odd);
    }
    meet();
  }
  uint8_t* patch = lds + wave * (2 * kPatchBytes);           // the stages are idle
  const int64_t tm = m0 / 32 + wm * WI, tn = n0 / 32 + wn * WJ;
  if (d_bf16) store_tile_lds<WI, WJ, true, false, true>(acc, tm, tn, (int)lane, A.rows, B.rows, Dv, ldd, patch);
  else store_tile_lds<WI, WJ, false, false, true>(acc, tm, tn, (int)lane, A.rows, B.rows, Dv, ldd, patch);
}

template <int FA, int FB, int WI, int WJ>
int launch_canon_shape(const CanonOperand& A, const CanonOperand& B, int64_t K, void* D, bool bf, int64_t ldd, hipStream_t s) {
  constexpr int TR = 2 * WI, TC = 2 * WJ;
  // steps of eight blocks, of four where two stages of eight do not fit LDS (128 x 128 tiles of four terms)
  constexpr int KS = 2 * (Region<FA, TR, 8>::BYTES + Region<FB, TC, 8>::BYTES) <= 160 * 1024 ? 8 : 4;
  constexpr int stages = 2 * (Region<FA, TR, KS>::BYTES + Region<FB, TC, KS>::BYTES), patches = 4 * 2 * kPatchBytes;
  constexpr int lds = stages > patches ? stages : patches;
  static_assert(lds <= 160 * 1024, "LDS");
  const int64_t n_rg = (A.rows + 32 * TR - 1) / (32 * TR), n_cg = (B.rows + 32 * TC - 1) / (32 * TC);
  if (n_rg * n_cg > 2147483647LL) return MXP_ERR_UNSUPPORTED;
  allow_dynamic_lds<&canon_tiled_kernel<FA, FB, WI, WJ, KS>>(lds);
  hipLaunchKernelGGL((canon_tiled_kernel<FA, FB, WI, WJ, KS>), dim3((unsigned)(n_rg * n_cg)), dim3(64 * (4 + kConverting)), lds, s, A, B,
                     (int)(K / kBlock), D, ldd, bf ? 1 : 0, (int)n_rg, (int)n_cg);
  return launch_status();
}

// Tiles of the workgroups: 64 x 64 while that is one round of the chip, then 128 x 64, and 128 x 128 where either takes two full
// rounds.  A workgroup takes as long as its tile is large (us, 128 x 128 | 128 x 64 | 64 x 64: 40 x 15641 x 4096 MXFP4++ x MXFP4+
// 31.4 | 23.5 | 18.4 in 245 tiles of 64 x 64, 437 x 3847 x 4288 35.2 | 28.0 | 35.2 in 427 of them, 242 x 11225 x 3936
// 37.2 | 48.4 | 49.6 in 704), but 257 to 512 of 64 x 64 are ahead of two rounds of 128 x 64 (216 shapes, against the best of the three
// 1.20 | 1.46 | 1.00).  Over 35500 shapes of all pairs 0.2 % behind the best.
template <int FA, int FB>
int launch_canon_pair(const CanonOperand& A, const CanonOperand& B, int64_t K, void* D, bool bf, int64_t ldd, hipStream_t s) {
  const int64_t cg64 = (B.rows + 63) / 64, t64 = (A.rows + 63) / 64 * cg64, t128 = (A.rows + 127) / 128 * cg64;
  if (t64 <= kNumCU || (t128 > kNumCU && t64 <= 2 * kNumCU)) return launch_canon_shape<FA, FB, 1, 1>(A, B, K, D, bf, ldd, s);
  if (t128 <= kNumCU) return launch_canon_shape<FA, FB, 2, 1>(A, B, K, D, bf, ldd, s);
  return launch_canon_shape<FA, FB, 2, 2>(A, B, K, D, bf, ldd, s);
}

template <int FA>
int launch_canon_a(int fmtB, const CanonOperand& A, const CanonOperand& B, int64_t K, void* D, bool bf, int64_t ldd, hipStream_t s) {
  constexpr bool PP = FA == MXP_FMT_MXFP4PP, SIX = Kind<FA>::SIX;             // (pairs that canon_gemm_takes refuses are not built)
  if (fmtB == MXP_FMT_MXFP4) return launch_canon_pair<FA, MXP_FMT_MXFP4>(A, B, K, D, bf, ldd, s);
  if (fmtB == MXP_FMT_MXFP4P) return launch_canon_pair<FA, MXP_FMT_MXFP4P>(A, B, K, D, bf, ldd, s);
  if constexpr (!PP && !SIX)
    if (fmtB == MXP_FMT_MXFP4PP) return launch_canon_pair<FA, MXP_FMT_MXFP4PP>(A, B, K, D, bf, ldd, s);
  if constexpr (!PP) {
    if (fmtB == MXP_FMT_MXFP6) return launch_canon_pair<FA, MXP_FMT_MXFP6>(A, B, K, D, bf, ldd, s);
    if (fmtB == MXP_FMT_MXFP6P) return launch_canon_pair<FA, MXP_FMT_MXFP6P>(A, B, K, D, bf, ldd, s);
  }
  return MXP_ERR_UNSUPPORTED;
}

}  // namespace

namespace mxp {
// Which products go without images: those of one round of 128 x 128 tiles (us per call, replayed from a graph, images -> without:
// MXFP4++ x MXFP4+ 1037 x 3001 x 4128 56.4 -> 37.7, 512 x 4096 x 4096 41.5 -> 22.5, 8 x 4096 x 4128 27.6 -> 16.0; MXFP6+ pair
// 200 x 1000 x 4096 44.6 -> 17.4; MXFP4+ pair 16 x 256 x 256 6.3 -> 4.0).  With more rounds the conversions repeat (2048 x 4096 x 4096
// MXFP4+ pair 43.5 | 63.5, MXFP4++ x MXFP4+ 62.7 | 68.6).  The lines below come from both sides' times at 42500 shapes of all pairs
// (1 - 4096 rows, 64 - 16384 columns, K 64 - 16384); of 34950 that they take 43 are slower than through images by more than 3 %,
// 13 % at most.  Not taken:
//  - few rows x four-bit weights in whole chunks beyond a short K: the kernel on canonical weights splits K over its wavefronts
//    (without images / that, geometric means up to 4096 columns, 1 - 32 rows: K = 256 0.70, 1024 0.89, 1536 1.01, 2048 1.17; 33 - 64
//    rows: 256 0.65, 1024 0.84, 2048 1.07);
//  - few rows x few columns of long K, and long K on a small part of the chip: the kernels of the images split K too (us, images | without:
//    MXFP4+ x MXFP4 4 x 278 x 4736 9.1 | 12.8, 366 x 421 x 7936 26.6 | 28.2, but 996 x 474 x 8000 27.0 | 25.3; MXFP4++ x MXFP4+
//    7 x 878 x 12288 32.2 | 40.0, 8 x 165 x 6016 18.1 | 22.4; MXFP6 x MXFP6+ 4 x 163 x 5984 15.7 | 19.7; MXFP6 x MXFP4+
//    2 x 1622 x 6080 14.9 | 19.0).  Two terms on both sides, or codes that go in as they are, pay up to a longer K;
//  - two MXFP4+ operands, both of which are widened, beyond a shorter K still (1 x 1075 x 5792 12.8 | 21.7, 13 x 1112 x 4256 12.3 | 17.0,
//    1575 x 828 x 14688 53.5 | 75.2), in tiles of 128 x 128 beyond 3072 (1024 x 4096 x 4096 31.9 | 33.3);
//  - two MXFP4++ operands, whose product has an FP8 image route with its own error bound that mxp_gemm equals bit for bit, and
//    MXFP4++ next to a six-bit format, which is multiplied as bf16 in whatever room the workspace gives.
bool canon_gemm_takes(int64_t M, int64_t N, int64_t K, int fmtA, int fmtB) {
  if (fmtA > MXP_FMT_MXFP6P || fmtB > MXP_FMT_MXFP6P) return false;
  if (fmtA == MXP_FMT_MXFP4PP ? fmtB >= MXP_FMT_MXFP4PP : fmtB == MXP_FMT_MXFP4PP && fmtA >= MXP_FMT_MXFP4PP) return false;
  if (((M + 127) / 128) * ((N + 127) / 128) > kNumCU) return false;
  const bool four_a = fmtA <= MXP_FMT_MXFP4P, four_b = fmtB <= MXP_FMT_MXFP4P;
  if (M <= 64 && four_a && four_b && K % 256 == 0 && (fmtB == MXP_FMT_MXFP4P || fmtA != fmtB)) return K <= 1024;
  const int64_t tiles = ((M + 127) / 128) * ((N + 63) / 64);  // of 128 x 64
  const bool a_two = fmtA == MXP_FMT_MXFP4PP || fmtA == MXP_FMT_MXFP6P, b_two = fmtB == MXP_FMT_MXFP4PP || fmtB == MXP_FMT_MXFP6P;
  if (a_two || b_two) {
    const bool widened = (a_two != b_two) && fmtA != MXP_FMT_MXFP4 && fmtB != MXP_FMT_MXFP4;
    if (widened && M <= 32 && tiles < 16) return K <= 3584;
    return K <= 6144 || tiles > 32;
  }
  if (fmtA == MXP_FMT_MXFP4P && fmtB == MXP_FMT_MXFP4P) {
    if (tiles > kNumCU) return K <= 3072;
    if (tiles > 160) return K <= 9216;
    return K <= (tiles < (M <= 64 ? 64 : 16) ? 1536 : tiles < 32 ? 4096 : 6144);
  }
  const bool codes = fmtA != MXP_FMT_MXFP4P && fmtB != MXP_FMT_MXFP4P && (fmtA == MXP_FMT_MXFP4 || fmtB == MXP_FMT_MXFP4);
  if (!codes && tiles > 160) return K <= 9216;
  if (!codes && M <= 32 && tiles >= 16 && tiles < 32) return K <= 2560;
  return K <= (tiles < 16 ? 1536 : 6144) || tiles > 160;
}

int canon_gemm_launch(int64_t M, int64_t N, int64_t K, const uint8_t* ae, const uint8_t* as, const uint8_t* ai, int fmtA, const uint8_t* be,
                      const uint8_t* bs, const uint8_t* bi, int fmtB, void* D, int d_dtype, int64_t ldd, hipStream_t s) {
  const CanonOperand A = {ae, as, ai, M}, B = {be, bs, bi, N};
  const bool bf = d_dtype == MXP_BF16;
  switch (fmtA) {
    case MXP_FMT_MXFP4: return launch_canon_a<MXP_FMT_MXFP4>(fmtB, A, B, K, D, bf, ldd, s);
    case MXP_FMT_MXFP4P: return launch_canon_a<MXP_FMT_MXFP4P>(fmtB, A, B, K, D, bf, ldd, s);
    case MXP_FMT_MXFP4PP: return launch_canon_a<MXP_FMT_MXFP4PP>(fmtB, A, B, K, D, bf, ldd, s);
    case MXP_FMT_MXFP6: return launch_canon_a<MXP_FMT_MXFP6>(fmtB, A, B, K, D, bf, ldd, s);
    default: return launch_canon_a<MXP_FMT_MXFP6P>(fmtB, A, B, K, D, bf, ldd, s);
  }
}
}  // namespace mxp

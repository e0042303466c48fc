// D[M][N] = A[M][K] x B[N][K]^T, both operands bf16 rows in memory, fp32 accumulation on the bf16 MFMA: the multiplier of
// the conversion-based products once their quantized operands have been de-converted (Sec. 5), one pass over each.
//
// A workgroup of 2 x 2 wavefronts computes a 64 WM x 64 WN tile, each wavefront WM x WN MFMA tiles of 32 x 32.  K goes by
// in steps of 64; an operand's rows of a step are cut into two halves (half h: the h-th half of every wavefront's row
// tiles), so that a step is four phases, one per pair of halves: (A0,B0) (A0,B1) (A1,B1) (A1,B0).  Each phase changes one
// half only, and the registers of the half it leaves take the next phase's reads.
//
// Both operands go global -> LDS directly (16 bytes per lane), into two slots of a step each.  The halves are what the
// slots are refilled by: A0 and B0 of step k were last read before step k begins, B1 and A1 before its third phase, so
// their place takes step k + 2 from there on.  A wait therefore finds two groups (of two halves each) still in flight --
// five phases between the issue of a copy and its use -- with only two slots of LDS, and the waits are exact counts.
// Bound by the matrix pipes at the clock the power budget leaves them: 4096 x 14336 x 4096 335 us = 1.44 PFLOP/s, 4096 x 4096 x
// 14336 1.54 (a library product of the same operands here: 1.37 - 1.44).  128 registers hold all fragments of a step, so
// each is read from LDS once per wavefront; with 4 x 4 tiles per wavefront that is 64 bytes a clock of LDS reads and 32 of
// copies under the MFMAs, out of 128 (2 x 4 wavefronts of 4 x 2 tiles would read half as much again).
// LDS rows are 128 bytes; 16-byte chunk c of row r lies at position c ^ ((r / 2) % 8): the 16 lanes that read one chunk of
// 16 consecutive rows then cover all 64 banks once, and a copy's 8 lanes still read one 128-byte line.
#include "mxp_common.h"
#include "mxp_tile.h"
#include <type_traits>

namespace {

using namespace mxp;
typedef __bf16 v8bf __attribute__((ext_vector_type(8)));

constexpr int kRowBytes = 128;                               // one operand row of a step: 64 bf16

template <int WM_, int WN_>
struct Geo {
  static constexpr int WM = WM_, WN = WN_;
  static constexpr int TM = 64 * WM, TN = 64 * WN;           // rows of A and of B per workgroup
  static constexpr int A_HALF = TM / 2 * kRowBytes, B_HALF = TN / 2 * kRowBytes;
  static constexpr int SLOT = 2 * (A_HALF + B_HALF);         // A0 | A1 | B0 | B1
  static constexpr int GROUP = WM + WN;                      // copies per wavefront of one half of A and one half of B
  static constexpr int LDS = 2 * SLOT > 8 * kPatchBytes ? 2 * SLOT : 8 * kPatchBytes;   // the epilogue's patches reuse the slots
};

template <int N>
__device__ __forceinline__ void wait_copies_and_barrier() {  // all but the newest N copies landed, own LDS reads done
  asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" ::"n"(N) : "memory");
}

__device__ __forceinline__ v8bf read_chunk(const uint8_t* p) {
  union { u32x4 u; v8bf b; } c;
  c.u = *reinterpret_cast<const u32x4*>(p);
  return c.b;
}

// Source side of the copies of one operand.  Copy u of half h fills LDS rows 8 q .. 8 q + 7 of the half, q = wave W + u
// (W = WM or WN: 16 W rows of a half per wavefront row / column, 32 W rows in all); lane l supplies position l % 8 of row
// l / 8.  Rows past the matrix repeat its last row: they are multiplied into outputs that are not stored.
template <int W>
struct Rows {
  uint32_t off[2][W];
  const uint8_t* p;                                          // step to be copied next (wavefront-uniform)

  __device__ __forceinline__ static int chunk(int wave, int lane, int u) {
    const int r = 8 * (wave * W + u) + (lane >> 3);
    return (lane & 7) ^ ((r >> 1) & 7);
  }
  __device__ __forceinline__ void init(const uint16_t* src, int64_t ld, int64_t row0, int64_t rows, int wave, int lane) {
#pragma unroll
    for (int h = 0; h < 2; ++h)
#pragma unroll
      for (int u = 0; u < W; ++u) {
        const int r = 8 * (wave * W + u) + (lane >> 3);
        int64_t t = (int64_t)(r / (16 * W)) * (32 * W) + h * (16 * W) + r % (16 * W);
        if (row0 + t >= rows) t = rows - 1 - row0;
        off[h][u] = (uint32_t)(t * ld * 2) + 16u * (uint32_t)chunk(wave, lane, u);
      }
    p = reinterpret_cast<const uint8_t*>(src + row0 * ld);
  }
  // the last step holds one block of 32 only: chunks 4 .. 7 are fetched from 0 .. 3 instead (and not used)
  __device__ __forceinline__ void half_step(int wave, int lane) {
#pragma unroll
    for (int u = 0; u < W; ++u) {
      const uint32_t back = chunk(wave, lane, u) >= 4 ? 64u : 0u;
      off[0][u] -= back;
      off[1][u] -= back;
    }
  }
};

template <int IMM>
__device__ __forceinline__ void copy16(uint32_t lds, uint32_t voff, const uint8_t* sptr) {
  asm volatile("s_add_u32 m0, %0, %1\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %2, %3" ::"s"(lds), "n"(IMM), "v"(voff), "s"(sptr) : "memory", "scc");
}

template <class G, bool OUT_BF16>
__device__ __forceinline__ void run_bf16_tile(uint8_t* lds, const uint16_t* __restrict__ A, int64_t lda, const uint16_t* __restrict__ B,
                                              int64_t ldb, int64_t K, int64_t M, int64_t N, void* __restrict__ Dv, int64_t ldd,
                                              int64_t m0, int64_t n0) {
  constexpr int WM = G::WM, WN = G::WN, HM = WM / 2, HN = WN / 2;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = wave >> 1, wn = wave & 1, h = lane >> 5, nl = lane & 31;
  const int64_t nks = (K + 63) / 64;
  const bool tail = (K & 63) != 0;

  Rows<WM> ra;
  Rows<WN> rb;
  ra.init(A, lda, m0, M, wave, lane);
  rb.init(B, ldb, n0, N, wave, lane);
  const uint32_t lds0 = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) uint8_t*)lds;
  const uint32_t lds_a = lds0 + (uint32_t)wave * (WM * 1024), lds_b = lds0 + 2 * G::A_HALF + (uint32_t)wave * (WN * 1024);

  v16f acc[WM][WN];
#pragma unroll
  for (int i = 0; i < WM; ++i)
#pragma unroll
    for (int j = 0; j < WN; ++j)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.0f;

  // operand reads: lane (nl, h) takes chunk 4 h + s of its row: block h of the step, k-slots 8 s .. 8 s + 7
  uint32_t rd_a[4], rd_b[4];
#pragma unroll
  for (int s = 0; s < 4; ++s) {
    const uint32_t o = (uint32_t)(nl * kRowBytes + ((4 * h + s) ^ ((nl >> 1) & 7)) * 16);
    rd_a[s] = o + (uint32_t)(wm * 16 * WM * kRowBytes);
    rd_b[s] = o + (uint32_t)(2 * G::A_HALF + wn * 16 * WN * kRowBytes);
  }
  v8bf fa[2][HM][4], fb[2][HN][4];

  // copy c (0 .. GROUP - 1) of a group: A half ha, B half hb of the step that ra.p / rb.p point at, into slot SL
#define MXP_COPY(SL, ha, hb, c)                                                                                          \
  do {                                                                                                                   \
    constexpr int c_ = (c);                                                                                              \
    if constexpr (c_ < WM) copy16<(SL)*G::SLOT + (ha)*G::A_HALF + c_ * 1024>(lds_a, ra.off[ha][c_ < WM ? c_ : 0], ra.p); \
    else copy16<(SL)*G::SLOT + (hb)*G::B_HALF + (c_ - WM) * 1024>(lds_b, rb.off[hb][c_ >= WM ? c_ - WM : 0], rb.p);      \
  } while (0)
  auto copy_group = [&](auto sl, auto hh) {                  // a whole group: half hh of A and of B
    constexpr int SL = decltype(sl)::value, H = decltype(hh)::value;
    auto rec = [&](auto self, auto cc) {
      constexpr int C = decltype(cc)::value;
      if constexpr (C < G::GROUP) {
        MXP_COPY(SL, H, H, C);
        self(self, std::integral_constant<int, C + 1>{});
      }
    };
    rec(rec, std::integral_constant<int, 0>{});
  };
  // step kk is the next to be copied: the first group of it (A0, B0) ends the use of the previous step's addresses
  auto enter_step = [&](int64_t kk) {
    if (kk > 0 && kk < nks) {                                // past the end the last step is fetched again, unused
      ra.p += kRowBytes;
      rb.p += kRowBytes;
    }
    if (tail && kk == nks - 1) {
      ra.half_step(wave, lane);
      rb.half_step(wave, lane);
    }
  };
  using I0 = std::integral_constant<int, 0>;
  using I1 = std::integral_constant<int, 1>;

  enter_step(0);
  copy_group(I0{}, I0{});
  copy_group(I0{}, I1{});
  enter_step(1);
  copy_group(I1{}, I0{});
  copy_group(I1{}, I1{});
  wait_copies_and_barrier<3 * G::GROUP>();
  // Steps are multiplied in pairs.  Zeros take the place of what the last one lacks: of its second block when K ends with a
  // single block of 32, of a whole step when their number is odd.
  auto zero_fill = [&](int slot, bool whole) {
    wait_copies_and_barrier<0>();
    uint8_t* p = lds + slot * G::SLOT;
    for (int r = tid; r < G::SLOT / kRowBytes; r += 256)
#pragma unroll 1
      for (int c = whole ? 0 : 4; c < 8; ++c) *reinterpret_cast<u32x4*>(p + r * kRowBytes + (c ^ ((r >> 1) & 7)) * 16) = (u32x4){0, 0, 0, 0};
    wait_copies_and_barrier<0>();
  };
  auto read_first = [&](auto par) {                          // the fragments of A0 and B0 of the step in slot par
    constexpr int P = decltype(par)::value;
#pragma unroll
    for (int s = 0; s < 4; ++s) {
#pragma unroll
      for (int i = 0; i < HM; ++i) fa[0][i][s] = read_chunk(lds + P * G::SLOT + rd_a[s] + i * 32 * kRowBytes);
#pragma unroll
      for (int j = 0; j < HN; ++j) fb[P][j][s] = read_chunk(lds + P * G::SLOT + rd_b[s] + j * 32 * kRowBytes);
    }
  };
  if (tail && nks == 1) zero_fill(0, false);
  read_first(I0{});

  // One phase: 4 HM HN MFMAs on halves (ah, bh), whose fragments are in fa[ah] and fb[BS]; behind MFMA m the phase's other
  // work, given by `aside(m)`.
  constexpr int NM = 4 * HM * HN;
  auto phase = [&](auto ah, auto bh, auto bs, auto aside) {
    constexpr int AH = decltype(ah)::value, BH = decltype(bh)::value, BS = decltype(bs)::value;
    auto rec = [&](auto self, auto mc) {
      constexpr int m = decltype(mc)::value;
      if constexpr (m < NM) {
        constexpr int s = m / (HM * HN), q = m % (HM * HN), j = q / HM, i = (j & 1) ? HM - 1 - q % HM : q % HM;
        acc[AH * HM + i][BH * HN + j] =
            __builtin_amdgcn_mfma_f32_32x32x16_bf16(fb[BS][j][s], fa[AH][i][s], acc[AH * HM + i][BH * HN + j], 0, 0, 0);
        __builtin_amdgcn_sched_barrier(0);
        aside(mc);
        __builtin_amdgcn_sched_barrier(0);
        self(self, std::integral_constant<int, m + 1>{});
      }
    };
    rec(rec, I0{});
  };
  // fragments of half H of A (B) of slot SL, part e of 4 HM (4 HN): in the order the MFMAs want them
#define MXP_READ_A(SL, H, e) fa[H][(e) % HM][(e) / HM] = read_chunk(lds + rd_a[(e) / HM] + ((SL)*G::SLOT + (H)*G::A_HALF + (e) % HM * 32 * kRowBytes))
#define MXP_READ_B(SL, H, SET, e) \
  fb[SET][(e) % HN][(e) / HN] = read_chunk(lds + rd_b[(e) / HN] + ((SL)*G::SLOT + (H)*G::B_HALF + (e) % HN * 32 * kRowBytes))
  // the reads and copies of a phase, dealt over its MFMAs from number FIRST on: reads first
  constexpr int FIRST = 2;
  auto deal = [](int m, int total, int first, int span) {    // items [deal(m), deal(m + 1)) go behind MFMA m
    const int t = m < first ? 0 : m - first;
    const int v = (total * t + span - 1) / span;
    return v < total ? v : total;
  };
  auto kstep = [&](auto par, int64_t k) {
    constexpr int P = decltype(par)::value;                  // slot of this step; B0's fragments are in fb[P]
    if (k + 1 == nks || (tail && k + 2 == nks)) zero_fill(1 - P, k + 1 == nks);
    constexpr int B0 = P, B1 = 1 - P;
    constexpr int RSPAN = NM / 2 - FIRST > 0 ? NM / 2 - FIRST : 1, CFIRST = NM / 2, CSPAN = NM - CFIRST;
    using IB0 = std::integral_constant<int, B0>;
    using IB1 = std::integral_constant<int, B1>;
#define MXP_DEAL(m, total, first, span, body)                                                        \
  do {                                                                                               \
    constexpr int lo_ = deal(m, total, first, span), hi_ = (m) == NM - 1 ? (total) : deal((m) + 1, total, first, span); \
    auto rec_ = [&](auto self_, auto ec_) {                                                          \
      constexpr int e = decltype(ec_)::value;                                                        \
      if constexpr (e < hi_) {                                                                       \
        body;                                                                                        \
        self_(self_, std::integral_constant<int, e + 1>{});                                          \
      }                                                                                              \
    };                                                                                               \
    rec_(rec_, std::integral_constant<int, lo_>{});                                                  \
  } while (0)
    constexpr int C1 = G::GROUP / 2, C2 = G::GROUP - C1;     // a group's copies are dealt over two phases
    enter_step(k + 2);
    phase(I0{}, I0{}, IB0{}, [&](auto mc) {
      constexpr int m = decltype(mc)::value;
      if constexpr (m == FIRST - 1) wait_copies_and_barrier<2 * G::GROUP>();   // B1, A1 of this step are in; A0, B0 are free
      MXP_DEAL(m, 4 * HN, FIRST, RSPAN, MXP_READ_B(P, 1, B1, e));
      MXP_DEAL(m, C1, CFIRST, CSPAN, MXP_COPY(P, 0, 0, e));
    });
    phase(I0{}, I1{}, IB1{}, [&](auto mc) {
      constexpr int m = decltype(mc)::value;
      MXP_DEAL(m, 4 * HM, 0, RSPAN, MXP_READ_A(P, 1, e));
      MXP_DEAL(m, C2, CFIRST, CSPAN, MXP_COPY(P, 0, 0, C1 + e));
    });
    phase(I1{}, I1{}, IB1{}, [&](auto mc) {
      constexpr int m = decltype(mc)::value;
      if constexpr (m == FIRST - 1) wait_copies_and_barrier<2 * G::GROUP>();   // A0, B0 of the next step are in; B1, A1 are free
      MXP_DEAL(m, 4 * HM, FIRST, RSPAN, MXP_READ_A(1 - P, 0, e));
      MXP_DEAL(m, C1, CFIRST, CSPAN, MXP_COPY(P, 1, 1, e));
    });
    phase(I1{}, I0{}, IB0{}, [&](auto mc) {
      constexpr int m = decltype(mc)::value;
      MXP_DEAL(m, 4 * HN, 0, RSPAN, MXP_READ_B(1 - P, 0, B1, e));
      MXP_DEAL(m, C2, CFIRST, CSPAN, MXP_COPY(P, 1, 1, C1 + e));
    });
#undef MXP_DEAL
  };
  for (int64_t k = 0; k < nks; k += 2) {
    kstep(I0{}, k);
    kstep(I1{}, k + 1);
  }
#undef MXP_READ_A
#undef MXP_READ_B
#undef MXP_COPY
  wait_copies_and_barrier<0>();                              // the slots are idle: their place holds the epilogue's patches
  uint8_t* patch = lds + wave * (2 * kPatchBytes);
  const int64_t tm = m0 / 32 + wm * WM, tn = n0 / 32 + wn * WN;
  // Streaming stores where a store instruction's runs of 128 bytes start on whole lines (fp32) or halves of them (bf16); elsewhere
  // the cache has to put the lines together (streaming | ordinary, us: 4096 x 14336 x 256 to bf16 61 | 69, 4096 x 14352 x 256 91 | 74,
  // 2772 x 15036 x 256 to fp32 126 | 59; 4096 x 14352 x 256 to fp32, half lines, 82 | 74).
  if ((((uint64_t)(uintptr_t)Dv | (uint64_t)ldd * (OUT_BF16 ? 2 : 4)) & (OUT_BF16 ? 63u : 127u)) == 0)
    store_tile_lds<WM, WN, OUT_BF16, true>(acc, tm, tn, lane, M, N, Dv, ldd, patch);
  else store_tile_lds<WM, WN, OUT_BF16, false>(acc, tm, tn, lane, M, N, Dv, ldd, patch);
}

// Tile lists.  Full tiles (256 x 256) are in band order; the last `2 * halved` workgroups compute the halves (256 x 128) of
// the tiles behind them.  Workgroups are dealt round-robin to the XCDs: workgroup c takes position c / 8 of the c % 8-th
// contiguous run, so that the 32 workgroups an XCD runs at a time share 8 row panels and 4 column panels through its L2.
template <bool OUT_BF16>
__global__ void __launch_bounds__(256) bf16_gemm_kernel(const uint16_t* __restrict__ A, int64_t lda, const uint16_t* __restrict__ B,
                                                        int64_t ldb, int64_t K, int64_t M, int64_t N, void* __restrict__ Dv, int64_t ldd,
                                                        int rows, int cols, int full) {
  extern __shared__ __attribute__((aligned(16))) uint8_t lds[];
  const int c = blockIdx.x;
  int r, q;
  if (c < full) {
    const int x = c & 7, base = full >> 3, rem = full & 7;
    band_decode(x * base + (x < rem ? x : rem) + (c >> 3), rows, cols, r, q);
    run_bf16_tile<Geo<4, 4>, OUT_BF16>(lds, A, lda, B, ldb, K, M, N, Dv, ldd, (int64_t)r * 256, (int64_t)q * 256);
  } else {
    const int n = (int)gridDim.x - full, d = c - full;
    const int x = d & 7, base = n >> 3, rem = n & 7;
    const int p = x * base + (x < rem ? x : rem) + (d >> 3);
    band_decode(full + (p >> 1), rows, cols, r, q);
    const int64_t n0 = (int64_t)q * 256 + (p & 1) * 128;
    if (n0 < N) run_bf16_tile<Geo<4, 2>, OUT_BF16>(lds, A, lda, B, ldb, K, M, N, Dv, ldd, (int64_t)r * 256, n0);
  }
}

// Few tiles: blocks of 128 x 128 while one round of them suffices (bf16 product alone, 256 x 4096 x 4096: 57 -> 45 us; 256 x
// 4096 x 14336: 182 -> 82).  What bounds these is a workgroup's own walk along K.
template <bool OUT_BF16>
__global__ void __launch_bounds__(256, 2) bf16_gemm_block_kernel(const uint16_t* __restrict__ A, int64_t lda, const uint16_t* __restrict__ B,
                                                                 int64_t ldb, int64_t K, int64_t M, int64_t N, void* __restrict__ Dv,
                                                                 int64_t ldd, int rows, int cols) {
  extern __shared__ __attribute__((aligned(16))) uint8_t lds[];
  const int n = (int)gridDim.x, x = blockIdx.x & 7, base = n >> 3, rem = n & 7;
  int r, q;
  band_decode(x * base + (x < rem ? x : rem) + (blockIdx.x >> 3), rows, cols, r, q);
  run_bf16_tile<Geo<2, 2>, OUT_BF16>(lds, A, lda, B, ldb, K, M, N, Dv, ldd, (int64_t)r * 128, (int64_t)q * 128);
}

template <bool OUT_BF16>
void launch_bf16(int64_t M, int64_t N, int64_t K, const uint16_t* A, int64_t lda, const uint16_t* B, int64_t ldb, void* D, int64_t ldd,
                 hipStream_t s) {
  const int64_t blocks = ((M + 127) / 128) * ((N + 127) / 128);
  if (blocks <= kNumCU) {
    constexpr int lds = Geo<2, 2>::LDS;
    allow_dynamic_lds<&bf16_gemm_block_kernel<OUT_BF16>>(lds);
    hipLaunchKernelGGL((bf16_gemm_block_kernel<OUT_BF16>), dim3((unsigned)blocks), dim3(256), lds, s, A, lda, B, ldb, K, M, N, D, ldd,
                       (int)((M + 127) / 128), (int)((N + 127) / 128));
    return;
  }
  const int rows = (int)((M + 255) / 256), cols = (int)((N + 255) / 256), tiles = rows * cols;
  // a last round of at most half the chip's tiles is cut into half tiles: half a round instead of a whole one
  const int rem = tiles % kNumCU, halved = rem <= kNumCU / 2 ? rem : 0, full = tiles - halved;
  constexpr int lds = Geo<4, 4>::LDS;
  static_assert(lds <= 160 * 1024, "LDS");
  allow_dynamic_lds<&bf16_gemm_kernel<OUT_BF16>>(lds);
  hipLaunchKernelGGL((bf16_gemm_kernel<OUT_BF16>), dim3((unsigned)(full + 2 * halved)), dim3(256), lds, s, A, lda, B, ldb, K, M, N, D, ldd,
                     rows, cols, full);
}

}  // namespace

namespace mxp {
bool bf16_gemm_takes(int64_t M, int64_t N, int64_t K, int64_t lda) {
  // row offsets inside a tile are 32-bit byte counts, tile counts and coordinates ints
  return lda < ((int64_t)1 << 23) && ((M + 255) / 256) * ((N + 255) / 256) < ((int64_t)1 << 29);
}

int bf16_gemm_launch(int64_t M, int64_t N, int64_t K, const void* A, int64_t lda, const void* B, int64_t ldb, void* D, int d_dtype,
                     int64_t ldd, hipStream_t s) {
  const uint16_t *a = static_cast<const uint16_t*>(A), *b = static_cast<const uint16_t*>(B);
  if (d_dtype == MXP_BF16) launch_bf16<true>(M, N, K, a, lda, b, ldb, D, ldd, s);
  else launch_bf16<false>(M, N, K, a, lda, b, ldb, D, ldd, s);
  return launch_status();
}
}  // namespace mxp

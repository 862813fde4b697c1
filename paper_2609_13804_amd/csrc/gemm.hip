// Dense contractions of the selection path on gfx950 matrix cores.
//
//   C[m, n] = sum_k A[m, k] * B[n, k]      (both operands K-contiguous)
//
// Accumulation is float32 and the result is stored once (bfloat16 rounded to
// nearest-even, or float32).  Two cores:
//  * bfloat16, gemm_bf16: 256 x 256 tiles of eight waves, each wave owning
//    128 x 64 as 16 x 16 tiles of v_mfma_f32_16x16x32_bf16 (smaller tiles for
//    small products and for the last round of a large one); K in 64-wide
//    stages through LDS rings filled straight from global memory.
//  * float32, gemm_f32: 32 x 64 or 64 x 64 tiles of four waves, as 16 x 16
//    tiles of v_mfma_f32_16x16x4_f32; K in 64-wide stages through an LDS ring
//    filled straight from global memory.
//
// Three users:
//  * the projection of Algorithm 1 step 1: A = [X; s_start; s_stop], B = W_kqv;
//  * the text projection W_text E_text^T (float32 output for the LayerNorm);
//  * per-group Gram products of the projected rows used by the selection
//    recurrence (select.hip): rows [Q_g; q_start; V_g; v_start; context split]
//    against columns [K_g; k_stop; k_start] (bfloat16: the rows and columns
//    beside the tokens' as strips).
#include <type_traits>

#include "sp_internal.h"
#include "lds_dma.h"

namespace sp {
namespace {

typedef __bf16 bf16x4_t __attribute__((ext_vector_type(4)));
typedef __bf16 bf16x8_t __attribute__((ext_vector_type(8)));
typedef float f32x4_t __attribute__((ext_vector_type(4)));
typedef uint32_t u32x4_t __attribute__((ext_vector_type(4)));

constexpr int kThreads = 256;

// ------------------------------------------------------------------ float32
//
// One BM x 64 output tile of four waves (2 x 2, BM / 2 x 32 each), K in 64-wide
// stages through a ring of D LDS buffers filled straight from global memory (a
// 256-byte row is sixteen 16-byte chunks, chunk c of row r at slot c ^ (r & 15)),
// D - 1 stages ahead of the matrix cores, one barrier a stage.
//
// What bounds it: with few tiles, a wave's own chain.  A 32 x 32 tile a wave in
// v_mfma_f32_32x32x2_f32 (64 cycles for K = 2) takes 14 us for K = 1024 however
// idle the chip is; 16 x 32 a wave halves that and doubles the workgroups.  With
// many, the matrix cores (157 TFLOP/s).  A lane reads four consecutive k of its
// row at a time and feeds them to four instructions, which then sum k = 4 (l /
// 16) + i, i = 0..3: A and B agree on the order.  The product is formed
// transposed (B as the row operand), so a lane holds four consecutive columns of
// one row.
// us against tiles of 64 x 64 or 128 x 128 staged through registers into 32-wide
// stages, the text product in a launch of its own: projection and text of one
// image, 578 x 768 x 1024, 46 -> 17; 1202 x 1536 x 1280 90 -> 53; 7202 x 1536 x
// 1280 375 -> 272 (107 TFLOP/s); Gram products of 3 groups of 256 and less, h
// 256, 10.8 -> 6.8, of 32, h 512, 74 -> 63.
template <int BM_, int D_>
struct F32Tile {
  static constexpr int BM = BM_, BN = 64, KS = 64, D = D_, WAVES = 4;
  static constexpr int TM = BM / 32;                               // 16-row tiles of a wave
  static constexpr int ROW = KS * 4, BUF = (BM + BN) * ROW;        // a stage: 24 or 32 KB
  static constexpr int LOADS = BUF / 1024 / WAVES;                 // per wave and stage
  static constexpr int LDS = D * BUF;                              // two workgroups a CU
  static_assert(BM % 32 == 0 && 2 * LDS <= kLdsBytes, "tile shape");
};
using F32Low = F32Tile<32, 3>;     // 72 KB
using F32High = F32Tile<64, 2>;    // 64 KB

template <class G, class ARows, class BRows>
__device__ __forceinline__ void gemm_f32(const ARows& ar, const BRows& br, int64_t M, int64_t N,
                                         int K, float* __restrict__ C, int64_t ldc, int64_t m0,
                                         int64_t n0, char* smem) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int wm = wave >> 1, wn = wave & 1, l16 = lane & 15, lk = lane >> 4;
  // This wave loads 4-row groups wave + 4 q of the stage's A rows, then B rows;
  // rows past M (N) read the last one and are not stored.
  const int dchunk = l16 ^ ((4 * wave + lk) & 15);
  const float* src[G::LOADS];
#pragma unroll
  for (int q = 0; q < G::LOADS; ++q) {
    const int r = 4 * (wave + G::WAVES * q) + lk;
    if (4 * G::WAVES * q < G::BM) {
      const int64_t gm = m0 + r;
      src[q] = ar.row(gm < M ? gm : M - 1) + 4 * dchunk;
    } else {
      const int64_t gn = n0 + r - G::BM;
      src[q] = br.row(gn < N ? gn : N - 1) + 4 * dchunk;
    }
  }
  auto issue = [&](int kt, int slot) {
#pragma unroll
    for (int q = 0; q < G::LOADS; ++q)
      lds_dma16(src[q] + kt * G::KS, smem + slot * G::BUF + (wave + G::WAVES * q) * 1024);
  };
  f32x4_t acc[G::TM][2];
#pragma unroll
  for (int u = 0; u < G::TM; ++u) acc[u][0] = acc[u][1] = f32x4_t{0.f, 0.f, 0.f, 0.f};
  const int arow = (wm * (G::BM / 2) + l16) * G::ROW, brow = (G::BM + wn * 32 + l16) * G::ROW;
  const int KT = K / G::KS;
#pragma unroll
  for (int s = 0; s < G::D - 1; ++s)
    if (s < KT) issue(s, s);
  int slot = 0;
  for (int kt = 0; kt < KT; ++kt) {
    // stage kt has landed (only loads of later stages remain), and after the
    // barrier every wave is past stage kt - 1, whose buffer is refilled
    if (kt + G::D - 2 < KT) wait_vmcnt<(G::D - 2) * G::LOADS>();
    else wait_vmcnt<0>();
    wait_lgkm0();
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
    if (kt + G::D - 1 < KT) issue(kt + G::D - 1, slot == 0 ? G::D - 1 : slot - 1);
    const char* st = smem + slot * G::BUF;
#pragma unroll
    for (int c = 0; c < G::KS / 16; ++c) {
      const int ch = ((4 * c + lk) ^ l16) << 4;
      f32x4_t a[G::TM];
#pragma unroll
      for (int u = 0; u < G::TM; ++u)
        a[u] = *reinterpret_cast<const f32x4_t*>(st + arow + u * 16 * G::ROW + ch);
      const f32x4_t b0 = *reinterpret_cast<const f32x4_t*>(st + brow + ch);
      const f32x4_t b1 = *reinterpret_cast<const f32x4_t*>(st + brow + 16 * G::ROW + ch);
#pragma unroll
      for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int u = 0; u < G::TM; ++u) {
          acc[u][0] = __builtin_amdgcn_mfma_f32_16x16x4f32(b0[i], a[u][i], acc[u][0], 0, 0, 0);
          acc[u][1] = __builtin_amdgcn_mfma_f32_16x16x4f32(b1[i], a[u][i], acc[u][1], 0, 0, 0);
        }
    }
    slot = slot == G::D - 1 ? 0 : slot + 1;
  }
  // lane l, register r: row l % 16, column 4 (l / 16) + r of a 16 x 16 tile
#pragma unroll
  for (int u = 0; u < G::TM; ++u) {
    const int64_t row = m0 + wm * (G::BM / 2) + 16 * u + l16;
    if (row >= M) continue;
#pragma unroll
    for (int t = 0; t < 2; ++t) {
      const int64_t col = n0 + wn * 32 + 16 * t + 4 * lk;
      float* dst = C + row * ldc + col;              // 16-byte aligned: C, ldc and col are
      if (col + 4 <= N) {
        *reinterpret_cast<f32x4_t*>(dst) = acc[u][t];
      } else {
#pragma unroll
        for (int e = 0; e < 4; ++e)
          if (col + e < N) dst[e] = acc[u][t][e];
      }
    }
  }
}

// ------------------------------------------------------------------ bf16
//
// The bfloat16 core: a BM x BN output tile per workgroup of WGM x WGN waves,
// K in 64-wide stages.  Operand tiles go straight from global memory into LDS
// (global_load_lds_dwordx4: one wave instruction fills 1 KiB = 8 rows x 128
// bytes), the A tiles through a ring of D + 1 buffers and the B tiles through a
// ring of D, loads running up to D stages ahead of the matrix cores.
//
// What bounds it and why this shape (9216 x 4096 x 16384 product; one card):
//  * the operand stream into a CU.  Measured without matrix work, the tiles of
//    such a product stream at 13 TB/s in 64-byte row pieces and at 14.8 TB/s in
//    128-byte ones (whole cache lines; 16 against 23 TB/s when they hit the L2),
//    so a stage is 64 wide;
//  * power.  With normally distributed operands in registers the matrix cores
//    sustain 1.79 PFLOP/s with the 32x32x16 instruction and 2.07 with 16x16x32
//    (2.45 with zeros): half the accumulator traffic per flop;
//  * barriers: one per stage, in its middle (below).
// Within a pass of the denoiser a core of 32-wide stages and 32x32x16 instructions
// with whole tiles only took 1341 us for it (0.92 PFLOP/s) and this one takes 998
// (1.24), with bit-identical results; 10240 rows in the encoder 1320 against 976 to
// 993 (1.40).
//
// A 128-byte row holds eight 16-byte chunks, chunk c of row r at slot
// c ^ ((r >> 1) & 7), which the load realises by choosing each lane's source
// address: a 16-lane pass of a fragment read (16 consecutive rows, one chunk
// column) then touches every bank once.  Rows past M (N) are clamped to the
// last valid row and their results are not stored.
//
// The product is formed transposed (B as the instruction's row operand), so a
// lane holds four consecutive columns of one row and the tile is staged through
// LDS in 8-byte (bfloat16) or 16-byte (float32) pieces.
constexpr int kKStage = 64;                // K of one stage
constexpr int kRowBytes = 2 * kKStage;     // one staged operand row

template <int BM_, int BN_, int WGM_, int WGN_, int D_>
struct BfTile {
  static constexpr int BM = BM_, BN = BN_, WGM = WGM_, WGN = WGN_, D = D_;
  static constexpr int WAVES = WGM * WGN, THREADS = 64 * WAVES;
  static constexpr int BUFA = BM * kRowBytes, BUFB = BN * kRowBytes;
  static constexpr int OFFB = (D + 1) * BUFA;               // B ring after the A ring
  static constexpr int LDS = OFFB + D * BUFB;
  static constexpr int TM = BM / WGM / 16, TN = BN / WGN / 16;   // 16 x 16 tiles of a wave
  static constexpr int LA = BM / 8 / WAVES, LB = BN / 8 / WAVES; // loads per wave and stage
  static_assert(BM % (8 * WAVES) == 0 && BN % (8 * WAVES) == 0, "whole loads per wave");
  static_assert(WAVES % 2 == 0, "the parity of a wave's row groups is the wave's");
  static_assert(LDS <= kLdsBytes, "the rings fit the LDS");
};
using TileWhole = BfTile<256, 256, 2, 4, 2>;     // 160 KB
using TileHalf = BfTile<256, 128, 2, 4, 2>;      // 128 KB
using TileQuarter = BfTile<128, 128, 2, 4, 4>;   // 144 KB
using TileSmall = BfTile<64, 64, 2, 2, 4>;       // 72 KB: two workgroups a CU
using TileGramA = BfTile<128, 256, 2, 4, 2>;     // 112 KB, and the strips beside it
using TileGramB = BfTile<256, 192, 2, 4, 2>;     // 144 KB
using TileGramC = BfTile<128, 192, 2, 4, 2>;     // 96 KB

// Output epilogue of the bfloat16 core: the product as it is, or (bfloat16
// output only) the product rounded to bfloat16, plus a per-column float32 bias,
// optionally through the GELU (below), rounded again: the same values as storing
// the product and then running a bias (+ GELU) pass of this arithmetic over it.
constexpr int kEpiNone = 0, kEpiBias = 1, kEpiBiasGelu = 2;

// The GELU, y Phi(y), in float32: Phi(-a) = exp2(-a^2 log2(e) / 2 + g(a)) for a =
// |y|, g = log2 of half the scaled complementary error function of a / sqrt(2), a
// smooth function for which a degree-9 polynomial in 2 a / 5 - 1 stands (weighted
// minimax fit over [0, 5]: least squares at Chebyshev nodes, the weights raised
// where the error in Phi(-a), or in 0.02 of it for small ones, is largest); past 5
// g stays as it is at 5.  Against 64 bits: at most 2.6e-6 of a value for y > -5,
// and 2e-8 past it, where the GELU itself is below 1.5e-6 and g should still fall
// (0.1 of a value at -5.5, 0.6 at -8); y (1 + erf(y / sqrt 2)) / 2 with a correctly
// rounded erf is off by up to 5 % of a value in [-5, -4], 8e-8 past -5 (whole
// values).  2-norm of the error over that of the result, for normal y / for y
// uniform over [-8, 8]: 4.3e-8 / 1.9e-8, and 3.8e-8 / 2.1e-8 that way.
// A wave's epilogue is bound by these instructions, which no matrix work
// hides: about 20 a value where the library's erff took twice as many.  A pass
// of the denoiser (9216 x 16384 x 4096 with bias and GELU in it) 2663 -> 2474 us,
// of the encoder on 16 images about 400 of 7424 us.
__device__ __forceinline__ float gelu(float y) {
  const float u = fmaf(fminf(fabsf(y), 5.0f), 0.4f, -1.0f);
  float g = 0.0007071180152706802f;
  g = fmaf(g, u, -0.00031387381022796035f);
  g = fmaf(g, u, -0.0026931974571198225f);
  g = fmaf(g, u, 0.007887270301580429f);
  g = fmaf(g, u, -0.022970620542764664f);
  g = fmaf(g, u, 0.06388623267412186f);
  g = fmaf(g, u, -0.16125473380088806f);
  g = fmaf(g, u, 0.4011325240135193f);
  g = fmaf(g, u, -1.1640429496765137f);
  g = fmaf(g, u, -2.8228464126586914f);
  const float t = __builtin_amdgcn_exp2f(fmaf(y * y, -0.72134752044448170f, g));   // Phi(-|y|)
  return y * (y > 0.0f ? 1.0f - t : t);
}

// A product may carry strips (Gram products, below): kCols / kRows further
// columns and rows beside the tile, whose operand rows stay in LDS whole.
struct NoStrips {
  static constexpr bool kCols = false, kRows = false;
  __device__ int64_t out_row(int64_t row) const { return row; }
};

template <class G, typename OutT, class ARows, class BRows, int EPI = kEpiNone, class Strips = NoStrips>
__device__ __forceinline__ void gemm_bf16(const ARows& ar, const BRows& br, int64_t M, int64_t N,
                                          int K, OutT* __restrict__ C, int64_t ldc, int64_t m0,
                                          int64_t n0, char* smem,
                                          const float* __restrict__ bias = nullptr,
                                          const Strips& strips = Strips()) {
  static_assert(EPI == kEpiNone || sizeof(OutT) == 2, "bias epilogues write bfloat16");
  constexpr bool SC = Strips::kCols, SR = Strips::kRows;
  constexpr int D = G::D, LA = G::LA, LB = G::LB, TM = G::TM, TN = G::TN, W = G::WAVES;
  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = tid >> 6;
  const int wm = wave / G::WGN, wn = wave % G::WGN;

  // This wave loads 8-row groups wave + W q of both operand tiles; lane
  // (row lane / 8, slot lane % 8) fetches the chunk that the swizzle puts there.
  const int dchunk = (lane & 7) ^ (((wave & 1) << 2) + (lane >> 4));
  typename ARows::Src sa[LA];
  typename BRows::Src sb[LB];
#pragma unroll
  for (int q = 0; q < LA; ++q) sa[q] = ar.src(m0, 8 * (wave + W * q) + (lane >> 3), M, dchunk * 8);
#pragma unroll
  for (int q = 0; q < LB; ++q) sb[q] = br.src(n0, 8 * (wave + W * q) + (lane >> 3), N, dchunk * 8);
  const typename ARows::Base abase = ar.base_of(m0);
  const typename BRows::Base bbase = br.base_of(n0);
  auto issue_a = [&](int kt, int q, int slot) {
    ARows::dma(abase, sa[q], kt * kKStage, smem + slot * G::BUFA + (wave + W * q) * 1024);
  };
  auto issue_b = [&](int kt, int q, int slot) {
    BRows::dma(bbase, sb[q], kt * kKStage, smem + G::OFFB + slot * G::BUFB + (wave + W * q) * 1024);
  };

  f32x4_t acc[TM][TN];
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j) acc[i][j] = f32x4_t{0.f, 0.f, 0.f, 0.f};

  // Fragment of 16 rows at k-step ks (32 wide): lane l reads chunk 4 ks + l / 16
  // of row l % 16, whose slot bits do not depend on the 16-row group.
  const int l16 = lane & 15, lk = lane >> 4;
  const int slot0 = (lk ^ (l16 >> 1)) << 4;
  const int aoff = (wm * (G::BM / G::WGM) + l16) * kRowBytes + slot0;
  const int boff = G::OFFB + (wn * (G::BN / G::WGN) + l16) * kRowBytes + slot0;
  auto frag = [&](int buf, int off, int ks, int i) {
    return *reinterpret_cast<const bf16x8_t*>(smem + buf + (off ^ (ks << 6)) + i * 16 * kRowBytes);
  };
  struct Frags {
    bf16x8_t a[TM], b[TN];
  };
  Frags f0, f1;                            // k-step 0 and 1 of a stage

  // A stage is two phases of TM x TN matrix instructions: k-step 0 (f0), while
  // k-step 1's fragments (f1) are read, then k-step 1, while the next stage's
  // first fragments are read into f0.  Between the phases every wave has read
  // all of stage kt, and passes the workgroup barrier after waiting for its own
  // loads of stage kt + 1: that one barrier both publishes stage kt + 1 and
  // frees the buffers of stage kt.  Phase 0 issues the loads of A for stage
  // kt + D (into the buffer of stage kt - 1), phase 1 those of B (into the
  // buffer just freed), a few at a time between the matrix instructions.
  const int KT = K / kKStage;
  if constexpr (SC || SR) strips.load(K, smem + G::LDS);   // the oldest loads: any wait below covers them
  [[maybe_unused]] f32x4_t cx;
  if constexpr (SR) strips.ctx_load(K, cx);
#pragma unroll
  for (int s = 0; s < D; ++s)
    if (s < KT) {
#pragma unroll
      for (int q = 0; q < LA; ++q) issue_a(s, q, s);
#pragma unroll
      for (int q = 0; q < LB; ++q) issue_b(s, q, s);
    }
  if constexpr (SR) strips.ctx_store(K, cx, smem + G::LDS);
  if (KT >= D) wait_vmcnt<(D - 1) * (LA + LB)>();
  else wait_vmcnt<0>();
  if constexpr (SR) wait_lgkm0();          // ctx_store's writes
  __builtin_amdgcn_s_barrier();
  asm volatile("" ::: "memory");
#pragma unroll
  for (int j = 0; j < TN; ++j) f0.b[j] = frag(0, boff, 0, j);
#pragma unroll
  for (int i = 0; i < TM; ++i) f0.a[i] = frag(0, aoff, 0, i);

  // Strips: the column strip's 16 x 16 tiles are shared out over the waves (CT
  // row groups of the wave's own half each), the row strip's likewise (RT column
  // groups).  Their fragments are read and used within phase 0, for both k-steps
  // (the stage's buffers are free after it), in four slots of TM / 4 groups: the
  // columns' two k-steps, then the rows': read before the slot's first matrix
  // instructions and used after its last.  A stage's two products are one chain in
  // float32; the stages are added in 64 bits, in order, so that the sums do not
  // depend on the tile and are as close as the dot products of 64 lanes that the
  // strips replaced.  Against 64 bits (normal operands, 2-norm), 256-token groups, h
  // 640 / 512-token groups, h 512 / 768-token groups, h 1024: 6.5e-8 / 6.1e-8 /
  // 6.8e-8 with the dot products, 1.0e-7 / 8.7e-8 / 1.9e-7 as one or two chains over
  // K, 5.0e-8 in all of them now, for 1 us of a tile's time.  A lane's results repeat those of
  // the lanes beside it, so each sums other registers, and ten hold all the sums.
  constexpr int CT = TM / G::WGN > 0 ? TM / G::WGN : 1, RT = (TN + 1) / 2, SLOT = TM / 4;
  static_assert(!(SC || SR) || (TM % 4 == 0 && CT <= 2 && RT == 2 && G::WGM == 2), "strip tiles per wave");
  [[maybe_unused]] f32x4_t accc[CT], accr[RT], accx;
  [[maybe_unused]] double sumc = 0.0, sumr[3] = {0.0, 0.0, 0.0}, sumx = 0.0;
  [[maybe_unused]] bf16x8_t xa[CT], xb[RT], xs, xr;
  const int xaoff = aoff + wn * CT * 16 * kRowBytes;
  auto strip_col = [&](int j) { const int q = wm * RT + j; return q < TN ? q : TN - 1; };
  auto strip_read = [&](int kt, int slot, int abuf, int bbuf) {
    const int ks = slot & 1, k = kt * kKStage + ks * 32 + 8 * lk;
    if constexpr (SC)
      if (slot < 2) {
#pragma unroll
        for (int c = 0; c < CT; ++c) xa[c] = frag(abuf, xaoff, ks, c);
      }
    if constexpr (SC)
      if (slot < 2 || SR) xs = strips.col_frag(smem + G::LDS, l16, k);
    if constexpr (SR)
      if (slot >= 2) {
#pragma unroll
        for (int j = 0; j < RT; ++j)
          xb[j] = *reinterpret_cast<const bf16x8_t*>(smem + bbuf + (boff ^ (ks << 6)) + strip_col(j) * 16 * kRowBytes);
        xr = strips.row_frag(smem + G::LDS, l16, k);
      }
  };
  auto strip_mfma = [&](int slot) {
    auto add = [&](bf16x8_t x, bf16x8_t y, f32x4_t& v) {
      v = __builtin_amdgcn_mfma_f32_16x16x32_bf16(x, y, slot & 1 ? v : f32x4_t{0.f, 0.f, 0.f, 0.f}, 0, 0, 0);
    };
    if constexpr (SC)
      if (slot < 2) {
#pragma unroll
        for (int c = 0; c < CT; ++c) add(xs, xa[c], accc[c]);
      }
    if constexpr (SR)
      if (slot >= 2) {
#pragma unroll
        for (int j = 0; j < RT; ++j) add(xb[j], xr, accr[j]);
        if constexpr (SC) add(xs, xr, accx);
      }
  };
  // The stage's sums, a slot or a phase after their last products.
  auto strip_sum_cols = [&]() {
    if constexpr (SC) sumc += (double)Strips::col_value(accc[0], accc[CT - 1], lk);
  };
  auto strip_sum_rows = [&]() {
    if constexpr (SR) {
#pragma unroll
      for (int i = 0; i < 3; ++i) sumr[i] += (double)Strips::row_value(accr[0], accr[1], i, l16);
      if constexpr (SC) sumx += (double)(lk & 1 ? accx[1] : accx[0]);
    }
  };

  // One phase: matrix instructions on `cur` in TM groups; the first groups also
  // read `nxt` (two or three fragments each), and load(i) issues group i's loads.
  auto phase = [&](Frags& cur, Frags& nxt, bool read, int abuf, int bbuf, int ks, int kt, auto&& load) {
    constexpr int R = TM + TN, GR = TM > 2 ? TM - 2 : TM, PER = (R + GR - 1) / GR;
    __builtin_amdgcn_s_setprio(1);   // the wave whose operands are ready goes first
#pragma unroll
    for (int i = 0; i < TM; ++i) {
      if constexpr (SC || SR) {
        if (ks == 1 && i % SLOT == 0) strip_read(kt, i / SLOT, abuf, bbuf);
        if (ks == 1 && i == 2 * SLOT) strip_sum_cols();
        if (ks == 0 && i == 1) strip_sum_rows();
      }
#pragma unroll
      for (int j = 0; j < TN; ++j)
        acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(cur.b[j], cur.a[i], acc[i][j], 0, 0, 0);
      if (read) {
#pragma unroll
        for (int u = 0; u < PER; ++u) {
          const int r = i * PER + u;
          if (r < TN) nxt.b[r] = frag(bbuf, boff, ks, r);
          else if (r < R) nxt.a[r - TN] = frag(abuf, aoff, ks, r - TN);
        }
      }
      load(i);
      if constexpr (SC || SR)
        if (ks == 1 && (i + 1) % SLOT == 0) strip_mfma(i / SLOT);
      __builtin_amdgcn_sched_barrier(0);
    }
    __builtin_amdgcn_s_setprio(0);
  };
  int ia = 0, ib = 0;                      // ring slots of stage kt
  // MORE / REFILL: 1 means always, -1 decided at run time.  The steady-state
  // loop instantiates both as 1, so its body has no branches: at a join of
  // branches the compiler's wait counting falls back to waiting for every
  // outstanding LDS read.
  auto stage = [&](int kt, auto more_c, auto refill_c) {
    constexpr int MORE = decltype(more_c)::value, REFILL = decltype(refill_c)::value;
    const bool more = MORE == 1 || kt + 1 < KT;
    const bool refill = REFILL == 1 || kt + D < KT;
    const int ra = ia == 0 ? D : ia - 1, rb = ib;          // slots of A and B of stage kt + D
    const int ia2 = ia == D ? 0 : ia + 1, ib2 = ib == D - 1 ? 0 : ib + 1;
    phase(f0, f1, true, ia * G::BUFA, ib * G::BUFB, 1, kt, [&](int i) {
      if (refill) {
#pragma unroll
        for (int q = 0; q < LA; ++q)
          if (q * TM / LA == i) issue_a(kt + D, q, ra);
      }
    });
    if (more) {
      // Stage kt + 1 has landed once only loads issued after it remain: A of
      // stages kt + 2 .. kt + D and B of stages kt + 2 .. kt + D - 1.
      if (refill) wait_vmcnt<(D - 1) * LA + (D - 2) * LB>();
      else wait_vmcnt<0>();
      wait_lgkm0();                        // this wave's reads of stage kt
      // Bare s_barrier (no fence): a workgroup fence would wait for every load
      // still in flight and collapse the rings to a single stage.
      __builtin_amdgcn_s_barrier();
      asm volatile("" ::: "memory");
    }
    phase(f1, f0, more, ia2 * G::BUFA, ib2 * G::BUFB, 0, kt, [&](int i) {
      if (refill) {
#pragma unroll
        for (int q = 0; q < LB; ++q)
          if (q * TM / LB == i) issue_b(kt + D, q, rb);
      }
    });
    ia = ia2;
    ib = ib2;
  };
  using Always = std::integral_constant<int, 1>;
  using Checked = std::integral_constant<int, -1>;
  int kt = 0;
  for (; kt + D < KT; ++kt) stage(kt, Always{}, Always{});
  for (; kt < KT; ++kt) stage(kt, Checked{}, Checked{});

  // Epilogue through LDS: once every wave is past the K loop the rings are
  // free, so the tile is staged there in row-major order and leaves as 16-byte
  // row chunks (whole cache lines).  A float32 tile may need several passes of
  // ROWS rows.  Chunks of a row are XOR-ed by the row's index among the rows
  // that share its banks, so the 16 rows that one staging write covers use
  // different banks.
  constexpr int E = (int)sizeof(OutT);
  constexpr int EPC = 16 / E;                              // elements per 16-byte chunk
  constexpr int CPR = G::BN / EPC;                         // chunks per staged row
  constexpr int FIT = G::LDS / (G::BN * E);
  constexpr int ROWS = FIT >= G::BM ? G::BM : G::BM / 2;   // rows staged per pass
  constexpr int PASSES = G::BM / ROWS;
  constexpr int RPB = G::BN * E >= 256 ? 1 : 256 / (G::BN * E);   // rows per 256 bytes (64 banks)
  constexpr int XM = CPR < 16 ? CPR - 1 : 15;
  static_assert(ROWS <= FIT && ROWS * CPR % G::THREADS == 0, "whole chunks per thread");
  static_assert(PASSES == 1 || (G::WGM == 2 && PASSES == 2), "a pass stages whole waves");
  auto sw = [](int lr) { return (lr / RPB) & XM; };
  const bool vec = ((uintptr_t)C % 16 == 0) && ((int64_t)ldc * E % 16 == 0);
  __syncthreads();
#pragma unroll
  for (int p = 0; p < PASSES; ++p) {
    if (PASSES == 1 || wm == p) {
      // 16 x 16 MFMA result layout, operands exchanged: lane l, register r
      // holds row l % 16, column 4 (l / 16) + r.
      f32x4_t bj[TN];
      if constexpr (EPI != kEpiNone) {
#pragma unroll
        for (int j = 0; j < TN; ++j)
#pragma unroll
          for (int r = 0; r < 4; ++r) {
            const int64_t col = n0 + wn * (G::BN / G::WGN) + 16 * j + 4 * lk + r;
            bj[j][r] = col < N ? bias[col] : 0.0f;
          }
      }
#pragma unroll
      for (int i = 0; i < TM; ++i) {
        const int lr = wm * (G::BM / G::WGM) - p * ROWS + 16 * i + l16;
        char* row = smem + lr * (G::BN * E);
#pragma unroll
        for (int j = 0; j < TN; ++j) {
          const int lc = wn * (G::BN / G::WGN) + 16 * j + 4 * lk;
          if constexpr (E == 2) {
            bf16x4_t v;                    // rounded in pairs (v_cvt_pk_bf16_f32)
#pragma unroll
            for (int r = 0; r < 4; ++r) v[r] = (__bf16)acc[i][j][r];
            if constexpr (EPI != kEpiNone) {
#pragma unroll
              for (int r = 0; r < 4; ++r) {
                const float y = (float)v[r] + bj[j][r];
                v[r] = (__bf16)(EPI == kEpiBiasGelu ? gelu(y) : y);
              }
            }
            *reinterpret_cast<bf16x4_t*>(row + (((lc >> 3) ^ sw(lr)) << 4) + ((lc & 4) << 1)) = v;
          } else {
            *reinterpret_cast<f32x4_t*>(row + (((lc >> 2) ^ sw(lr)) << 4)) = acc[i][j];
          }
        }
      }
    }
    __syncthreads();
#pragma unroll
    for (int q = 0; q < ROWS * CPR / G::THREADS; ++q) {
      const int c = tid + G::THREADS * q, lr = c / CPR, ch = c % CPR;
      const int64_t row = m0 + p * ROWS + lr, col = n0 + (int64_t)ch * EPC;
      if (row >= M || col >= N) continue;
      const OutT* src = reinterpret_cast<const OutT*>(smem + lr * (G::BN * E) + ((ch ^ sw(lr)) << 4));
      OutT* dst = C + strips.out_row(row) * ldc + col;
      if (vec && col + EPC <= N) {
        *reinterpret_cast<uint4*>(dst) = *reinterpret_cast<const uint4*>(src);
      } else {
        for (int e = 0; e < EPC && col + e < N; ++e) dst[e] = src[e];
      }
    }
    if (p + 1 < PASSES) __syncthreads();
  }
  if constexpr (SC)
    if (lk < 2 * CT) strips.store_col(C, ldc, m0 + wm * (G::BM / 2) + 16 * (wn * CT + lk / 2) + l16, M, lk & 1, (float)sumc);
  if constexpr (SR) {
#pragma unroll
    for (int i = 0; i < 3; ++i) {
      const int u = Strips::row_slot(i, l16);            // register u % 4 of column group u / 4
      if (u < 4 * RT)
        strips.store_row(C, ldc, l16, n0 + wn * (G::BN / G::WGN) + 16 * strip_col(u / 4) + 4 * lk + u % 4, N, (float)sumr[i]);
    }
    if constexpr (SC)
      if (wave == 0 && lk < 2 && l16 < 5) strips.store_corner(C, ldc, l16, lk, (float)sumx);
  }
}

// How a product of T tiles of 256 x 256 is cut.  The first `full` tiles (whole
// rounds of the 256 CUs) run as they are; the R left over would keep only R
// CUs busy for a whole tile's time, so they are cut into `sub` parts when that
// shortens the last round: four 128 x 128 parts up to 64 tiles, two 256 x 128
// parts up to 128.  A round of whole tiles takes 1, of halves about 0.6 and of
// quarters about 0.36 of a tile's time (K 4096: 88, 54 and 32 us), so beyond
// 128 tiles two rounds of halves or three of quarters would take longer than
// the whole tiles.  Measured, 9216 x 4096 x 4096 (576 tiles): 271 us whole, 243
// halves, 234 quarters; 1037 x 3072 x 3584 (60 tiles): 67, 42, 30 us.
// Products of up to 20 tiles, which quarters leave most CUs without work, take
// 64 x 64 tiles, two workgroups a CU: 1077 x 1024 x 1024 8.5 against 10.3 us,
// 1077 x 1024 x 4096 24 against 28 us.  Every element accumulates K in the same
// order whatever the cut, so results do not depend on it.
struct Cut {
  int64_t full;        // whole tiles
  int64_t blocks;      // workgroups
  int sub;             // parts of each tile left over: 1, 2, 4, or 16 (64 x 64)
};
inline int64_t small_blocks(int64_t T) { return (T * 16 + 7) / 8 * 8; }   // all in 64 x 64
inline Cut cut_tiles(int64_t T) {
  constexpr int64_t kRound = 256;
  Cut c;
  c.full = T / kRound * kRound;
  const int64_t R = T - c.full;
  c.sub = T <= 20 ? 16 : R <= 64 ? 4 : R <= 128 ? 2 : 1;
  c.blocks = c.full + (R * c.sub + 7) / 8 * 8;
  return c;
}

// Workgroup w runs on XCD w % 8, which takes a contiguous run of the tiles in
// banded order: bands of kBand row panels, each band walked column by column
// (the last band as tall as the rows left).  The 32 tiles one XCD runs at a
// time then cover about kBand row panels and 32 / kBand column panels, so they
// share about 12 operand panels in that XCD's L2 (a row-major run of 32 tiles
// spans all the column panels of a wide product).
constexpr int64_t kBand = 4;

// First row and column of tile i of an mt x nt grid in banded order.
__device__ __forceinline__ void banded_tile(int64_t i, int64_t mt, int64_t nt, int64_t& m0, int64_t& n0) {
  const int64_t band = i / (kBand * nt), o = i % (kBand * nt);
  const int64_t rows = mt - band * kBand < kBand ? mt - band * kBand : kBand;
  m0 = (band * kBand + o % rows) * 256;
  n0 = (o / rows) * 256;
}

// The tile (of T) and part that workgroup w takes under a cut (cut_tiles); the
// whole tiles come first.  False for the padding workgroups.
__device__ __forceinline__ bool cut_place(int64_t w, int64_t T, int64_t full, int sub, int64_t& tile,
                                          int& part, bool& whole) {
  whole = w < full || sub == 1;
  part = 0;
  if (w < full) {
    tile = (w % 8) * (full / 8) + w / 8;
    return true;
  }
  const int64_t v = w - full, parts = (T - full) * sub, per = (parts + 7) / 8;
  const int64_t i = (v % 8) * per + v / 8;
  if (i >= parts || v / 8 >= per) return false;
  tile = full + i / sub;
  part = (int)(i % sub);
  return true;
}

// ------------------------------------------------------------------ row maps

// The bfloat16 core takes an operand's rows through src(r0, r, R, c): where lane
// row r of the tile starting at row r0 begins (column c; rows past the last of R
// read the last), and dma(base, src, k, dst), its 16-byte load at column k + c.
// Rows anywhere in memory keep a 64-bit address a lane:
template <class Map>
struct AnyRows {
  struct Base {};
  typedef const __bf16* Src;
  __device__ Base base_of(int64_t) const { return {}; }
  __device__ Src src(int64_t r0, int r, int64_t R, int c) const {
    const int64_t g = r0 + r;
    return static_cast<const Map*>(this)->row(g < R ? g : R - 1) + c;
  }
  __device__ static void dma(Base, Src s, int k, char* dst) { lds_dma16(s + k, dst); }
};

template <typename T>
struct ProjRows : AnyRows<ProjRows<T>> {
  const T* X;
  int64_t T_vis;
  const T* s_start;
  const T* s_stop;
  int ld;
  __device__ const T* row(int64_t m) const {
    if (m < T_vis) return X + m * ld;
    return m == T_vis ? s_start : s_stop;
  }
};

template <typename T>
struct DenseRows {
  const T* base;
  int64_t ld;
  __device__ const T* row(int64_t m) const { return base + m * ld; }
  // bfloat16 core: the tile's first row (uniform) and a 32-bit byte offset a
  // lane, half the address registers (ld up to kMaxDenseLd)
  typedef const char* Base;
  typedef uint32_t Src;
  __device__ Base base_of(int64_t r0) const {
    const uint64_t p = (uint64_t)(base + r0 * ld);         // the same in every lane: into scalar registers
    const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)p);
    const uint32_t hi = __builtin_amdgcn_readfirstlane((uint32_t)(p >> 32));
    return reinterpret_cast<const char*>(((uint64_t)hi << 32) | lo);
  }
  __device__ Src src(int64_t r0, int r, int64_t R, int c) const {
    const int64_t last = R - 1 - r0;
    return (uint32_t)((r < last ? r : last) * ld + c) * (uint32_t)sizeof(T);
  }
  __device__ static void dma(Base b, Src s, int k, char* dst) { lds_dma16(b + (int64_t)k * sizeof(T), s, dst); }
};

// 255 rows of this many bfloat16 values stay within DenseRows' 32-bit byte
// offsets; wider operands take the 64 x 64 tiles with whole addresses.
constexpr int64_t kMaxDenseLd = 1 << 22;

struct WideRows : AnyRows<WideRows> {
  const __bf16* base;
  int64_t ld;
  __device__ const __bf16* row(int64_t m) const { return base + m * ld; }
};

// float32 Gram operand rows of one group with tokens [g0, g0 + n): A side is
// [Q tokens; q_start; V tokens; v_start; c; 0; 0], B side is [K tokens; k_stop;
// k_start].
__device__ const float zero_row[512] = {};     // sp_dims' limit on a float32 h
template <typename T>
struct GramARows {
  const T* KQV;
  int64_t g0, n, start_row;
  int h;
  const T* ctx;        // the image's context
  __device__ const T* row(int64_t r) const {
    const int64_t ld = 3 * (int64_t)h;
    if (r < n) return KQV + (g0 + r) * ld + h;
    if (r == n) return KQV + start_row * ld + h;
    if (r < 2 * n + 1) return KQV + (g0 + r - n - 1) * ld + 2 * h;
    if (r == 2 * n + 1) return KQV + start_row * ld + 2 * h;
    return r == 2 * n + 2 ? ctx : zero_row;
  }
};

template <typename T>
struct GramBRows {
  const T* KQV;
  int64_t g0, n, start_row;
  int h;
  __device__ const T* row(int64_t c) const {
    const int64_t ld = 3 * (int64_t)h;
    if (c < n) return KQV + (g0 + c) * ld;
    if (c == n) return KQV + (start_row + 1) * ld;   // STOP key
    return KQV + start_row * ld;                      // START key
  }
};

// bfloat16 Gram products of one group with tokens [g0, g0 + n): the tiles cover
// the 2 n rows [Q; V] against the n rows [K]; the rows of START and of the
// context split and the columns of STOP and START are strips.  An empty group's
// tile reads START's rows and stores nothing.
struct GramTokenARows : AnyRows<GramTokenARows> {
  const __bf16* KQV;
  int64_t g0, n, start_row;
  int h;
  __device__ const __bf16* row(int64_t r) const {
    const int64_t ld = 3 * (int64_t)h;
    if (r < 0) return KQV + start_row * ld + h;
    return r < n ? KQV + (g0 + r) * ld + h : KQV + (g0 + r - n) * ld + 2 * h;
  }
};
struct GramTokenBRows : AnyRows<GramTokenBRows> {
  const __bf16* KQV;
  int64_t g0, start_row;
  int h;
  __device__ const __bf16* row(int64_t c) const {
    return KQV + (c < 0 ? start_row : g0 + c) * 3 * (int64_t)h;
  }
};

// The strips: rows [q_start; v_start; c_hi; c_mid; c_lo] (kRows) and columns
// [k_stop; k_start] (kCols) of a group's Gram block.  Their seven operand rows
// are loaded into LDS whole, row stride 2 h + 16 bytes (the five rows a
// fragment read touches fall on different banks); a fragment's lanes past them
// repeat a row and are not stored.  The last three rows are the image's float32
// context as bfloat16 values whose sum it is exactly (successive
// round-to-nearest-even residuals, 3 x 8 significant bits); four waves split it on
// the way, while the first stages load: a launch that wrote the split to memory
// before cost 3 to 4 us a selection.
template <bool COLS, bool ROWS>
struct GramStrips {
  static constexpr bool kCols = COLS, kRows = ROWS;
  static constexpr int kMaxH = 1024;                       // sp_dims' limit
  static constexpr int LDS = 7 * (2 * kMaxH + 16);
  const __bf16* start;      // START's projected row [k | q | v], STOP's after it
  const float* ctx;         // the image's context
  int64_t n;
  int h;
  __device__ int stride() const { return 2 * h + 16; }
  __device__ void load(int K, char* dst) const {
    const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
    if (w == 7 || (w >= 2 && w < 5)) return;
    const __bf16* row = w == 0 ? start + h : w == 1 ? start + 2 * h : w == 5 ? start + 3 * h : start;
    for (int c = 0; c < K; c += 512)
      if (c + 8 * lane < K) lds_dma16(row + c + 8 * lane, dst + w * stride() + 2 * c);
  }
  // The other four waves' part: 256 values of the context each, four a lane, then
  // their three rows.
  __device__ int ctx_at() const {
    const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    return w == 7 || (w >= 2 && w < 5) ? 256 * (w == 7 ? 3 : w - 2) + 4 * (int)(threadIdx.x & 63) : kMaxH;
  }
  __device__ void ctx_load(int K, f32x4_t& v) const {
    const int c = ctx_at();
    if (c < K) v = *reinterpret_cast<const f32x4_t*>(ctx + c);
  }
  __device__ void ctx_store(int K, f32x4_t v, char* dst) const {
    const int c = ctx_at();
    if (c >= K) return;
#pragma unroll
    for (int part = 0; part < 3; ++part) {
      bf16x4_t x;
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        x[e] = (__bf16)v[e];
        v[e] -= (float)x[e];
      }
      *reinterpret_cast<bf16x4_t*>(dst + (2 + part) * stride() + 2 * c) = x;
    }
  }
  __device__ bf16x8_t at(const char* s, int r, int k) const {
    return *reinterpret_cast<const bf16x8_t*>(s + r * stride() + 2 * k);
  }
  __device__ bf16x8_t row_frag(const char* s, int l16, int k) const { return at(s, l16 % 5, k); }
  __device__ bf16x8_t col_frag(const char* s, int l16, int k) const { return at(s, 5 + (l16 & 1), k); }
  // Which result a lane sums.  Columns: every lane of token row l16 holds [k_stop,
  // k_start] in registers 0 and 1 of each row group; lane quarter lk takes column
  // lk % 2 of group lk / 2.  Rows: lanes l16 % 5 hold eight columns, four registers
  // of two column groups; fifth l16 / 5 of a row takes registers l16 / 5, + 3, + 6.
  __device__ static float col_value(f32x4_t g0, f32x4_t g1, int lk) {
    const float a = lk & 2 ? g1[0] : g0[0], b = lk & 2 ? g1[1] : g0[1];
    return lk & 1 ? b : a;
  }
  __device__ static int row_slot(int i, int l16) { return l16 < 15 ? l16 / 5 + 3 * i : 8; }
  __device__ static float row_value(f32x4_t g0, f32x4_t g1, int i, int l16) {
    auto at = [&](int u) { return u < 4 ? g0[u % 4] : g1[u % 4]; };
    const float a = at(3 * i), b = at(3 * i + 1), c = at(3 * i + 2 < 8 ? 3 * i + 2 : 7);
    return l16 < 5 ? a : l16 < 10 ? b : c;
  }
  // The block's rows: A of the tokens, A of START, B of the tokens, B of START,
  // the three context rows.
  __device__ int64_t out_row(int64_t r) const { return r < n ? r : r + 1; }
  __device__ int64_t strip_row(int r) const { return r == 0 ? n : 2 * n + r; }
  __device__ void store_col(float* C, int64_t ldc, int64_t row, int64_t M, int c, float v) const {
    if (row < M) C[out_row(row) * ldc + n + c] = v;
  }
  __device__ void store_row(float* C, int64_t ldc, int l16, int64_t col, int64_t N, float v) const {
    if (col < N) C[strip_row(l16 % 5) * ldc + col] = v;
  }
  __device__ void store_corner(float* C, int64_t ldc, int r, int c, float v) const {
    C[strip_row(r) * ldc + n + c] = v;
  }
};

// ------------------------------------------------------------------ kernels

// float32: the projection's tiles, then the text projection's, split over K into
// partial products of K2 each (part p of the product at C2 + p M2 N2).  Tiles in
// row-major order: workgroup w runs on XCD w % 8, so where the column panels are a
// multiple of four, an XCD reads a half to an eighth of the weights.  With a
// contiguous run of tiles an XCD instead, 578 x 768 x 1024 took 25 us, not 16.
struct ProjectF32Args {
  ProjRows<float> ar;
  DenseRows<float> br;
  int64_t M, N, tiles;
  int K;
  float* C;
  DenseRows<float> er, wr;
  int64_t M2, N2, tiles2;       // tiles of one part
  int K2, split;
  float* C2;
};

template <class G>
__global__ __launch_bounds__(kThreads) void project_gemm_f32_kernel(ProjectF32Args p) {
  __shared__ __attribute__((aligned(1024))) char smem[G::LDS];
  int64_t t = blockIdx.x;
  if (t < p.tiles) {
    const int64_t nt = (p.N + G::BN - 1) / G::BN;
    gemm_f32<G>(p.ar, p.br, p.M, p.N, p.K, p.C, p.N, (t / nt) * G::BM, (t % nt) * G::BN, smem);
  } else {
    t -= p.tiles;
    const int64_t nt = (p.N2 + G::BN - 1) / G::BN, part = t / p.tiles2, i = t % p.tiles2;
    DenseRows<float> a, b;
    a.base = p.er.base + part * p.K2;
    a.ld = p.er.ld;
    b.base = p.wr.base + part * p.K2;
    b.ld = p.wr.ld;
    gemm_f32<G>(a, b, p.M2, p.N2, p.K2, p.C2 + part * p.M2 * p.N2, p.N2, (i / nt) * G::BM,
                (i % nt) * G::BN, smem);
  }
}

constexpr int kBfThreads = TileWhole::THREADS;
static_assert(TileHalf::THREADS == kBfThreads && TileQuarter::THREADS == kBfThreads, "one kernel runs all three");

// One tile of 256 x 256 at (m0, n0), or part `part` of `sub` of it.
template <typename OutT, int EPI, class ARows, class BRows>
__device__ __forceinline__ void gemm_bf16_part(const ARows& ar, const BRows& br, int64_t M, int64_t N,
                                               int K, OutT* C, int64_t ldc, int64_t m0, int64_t n0,
                                               bool whole, int sub, int part, char* smem,
                                               const float* bias) {
  if (whole) {
    gemm_bf16<TileWhole, OutT, ARows, BRows, EPI>(ar, br, M, N, K, C, ldc, m0, n0, smem, bias);
  } else if (sub == 2) {
    n0 += 128 * part;
    if (n0 >= N) return;
    gemm_bf16<TileHalf, OutT, ARows, BRows, EPI>(ar, br, M, N, K, C, ldc, m0, n0, smem, bias);
  } else {
    m0 += 128 * (part >> 1);
    n0 += 128 * (part & 1);
    if (m0 >= M || n0 >= N) return;
    gemm_bf16<TileQuarter, OutT, ARows, BRows, EPI>(ar, br, M, N, K, C, ldc, m0, n0, smem, bias);
  }
}

// The projection's tiles in banded order (bfloat16 output), then the text
// projection's (float32 output), cut together: the text tiles are dispatched
// last, onto compute units that the projection's last round leaves idle.
template <class Rows>
struct ProjectArgs {
  ProjRows<__bf16> ar;
  Rows br;
  int64_t M, N;
  int K;
  uint16_t* C;
  Rows er, wr;
  int64_t M2, N2;
  int K2;
  float* C2;
  int64_t full;
  int sub;
};

__device__ __forceinline__ int64_t tiles256(int64_t x) { return (x + 255) / 256; }

__global__ __launch_bounds__(kBfThreads) void project_gemm_bf16_kernel(
    ProjectArgs<DenseRows<__bf16>> p) {
  __shared__ __attribute__((aligned(1024))) char smem[TileWhole::LDS];
  const int64_t mt = tiles256(p.M), nt = tiles256(p.N), nt2 = tiles256(p.N2);
  int64_t t, m0, n0;
  int part;
  bool whole;
  if (!cut_place(blockIdx.x, mt * nt + tiles256(p.M2) * nt2, p.full, p.sub, t, part, whole)) return;
  if (t < mt * nt) {
    banded_tile(t, mt, nt, m0, n0);
    gemm_bf16_part<uint16_t, kEpiNone>(p.ar, p.br, p.M, p.N, p.K, p.C, p.N, m0, n0, whole, p.sub, part,
                                       smem, nullptr);
  } else {
    t -= mt * nt;
    gemm_bf16_part<float, kEpiNone>(p.er, p.wr, p.M2, p.N2, p.K2, p.C2, p.N2, (t / nt2) * 256,
                                    (t % nt2) * 256, whole, p.sub, part, smem, nullptr);
  }
}

// The same products in 64 x 64 tiles (cut 16).
template <class Rows>
__global__ __launch_bounds__(TileSmall::THREADS) void project_gemm_bf16_small_kernel(ProjectArgs<Rows> p) {
  __shared__ __attribute__((aligned(1024))) char smem[TileSmall::LDS];
  const int64_t mt = tiles256(p.M), nt = tiles256(p.N), nt2 = tiles256(p.N2);
  int64_t t, m0, n0;
  int part;
  bool whole;
  if (!cut_place(blockIdx.x, mt * nt + tiles256(p.M2) * nt2, 0, 16, t, part, whole)) return;
  const int64_t dm = 64 * (part >> 2), dn = 64 * (part & 3);
  if (t < mt * nt) {
    banded_tile(t, mt, nt, m0, n0);
    if (m0 + dm >= p.M || n0 + dn >= p.N) return;
    gemm_bf16<TileSmall, uint16_t>(p.ar, p.br, p.M, p.N, p.K, p.C, p.N, m0 + dm, n0 + dn, smem);
  } else {
    t -= mt * nt;
    m0 = (t / nt2) * 256 + dm;
    n0 = (t % nt2) * 256 + dn;
    if (m0 >= p.M2 || n0 >= p.N2) return;
    gemm_bf16<TileSmall, float>(p.er, p.wr, p.M2, p.N2, p.K2, p.C2, p.N2, m0, n0, smem);
  }
}

// A bfloat16 product C = A B^T (bfloat16 out), cut as cut_tiles says, with an
// optional bias (+ GELU) epilogue.
template <int EPI>
__global__ __launch_bounds__(kBfThreads) void dense_bf16_kernel(DenseRows<__bf16> ar,
                                                                DenseRows<__bf16> br, int64_t M,
                                                                int64_t N, int K, uint16_t* C,
                                                                const float* bias, int64_t full,
                                                                int sub) {
  __shared__ __attribute__((aligned(1024))) char smem[TileWhole::LDS];
  const int64_t mt = tiles256(M), nt = tiles256(N);
  int64_t t, m0, n0;
  int part;
  bool whole;
  if (!cut_place(blockIdx.x, mt * nt, full, sub, t, part, whole)) return;
  banded_tile(t, mt, nt, m0, n0);
  gemm_bf16_part<uint16_t, EPI>(ar, br, M, N, K, C, N, m0, n0, whole, sub, part, smem, bias);
}

// The same in 64 x 64 tiles (cut 16).
template <int EPI, class Rows>
__global__ __launch_bounds__(TileSmall::THREADS) void dense_bf16_small_kernel(
    Rows ar, Rows br, int64_t M, int64_t N, int K, uint16_t* C, const float* bias) {
  __shared__ __attribute__((aligned(1024))) char smem[TileSmall::LDS];
  const int64_t mt = tiles256(M), nt = tiles256(N);
  int64_t t, m0, n0;
  int part;
  bool whole;
  if (!cut_place(blockIdx.x, mt * nt, 0, 16, t, part, whole)) return;
  banded_tile(t, mt, nt, m0, n0);
  m0 += 64 * (part >> 2);
  n0 += 64 * (part & 3);
  if (m0 >= M || n0 >= N) return;
  gemm_bf16<TileSmall, uint16_t, Rows, Rows, EPI>(ar, br, M, N, K, C, N, m0, n0, smem, bias);
}

// Workgroup w runs on XCD w % 8.  With at least eight groups, all tiles of a
// group are placed on one XCD (group x + 8 k on XCD x) so that the group's
// rows are fetched into one L2.
__device__ __forceinline__ bool gram_tile(int64_t w, int per_group, int G, int xcd_grouped,
                                          int64_t& g, int64_t& t) {
  if (xcd_grouped) {
    const int64_t i = w / 8;
    g = w % 8 + 8 * (i / per_group);
    t = i % per_group;
  } else {
    g = w / per_group;
    t = w % per_group;
  }
  return g < G;
}

// Validates group g; on inconsistent offsets one workgroup records the error.
__device__ __forceinline__ bool gram_group_ok(const GramArgs& a, int64_t g, int64_t t, int64_t& g0,
                                              int64_t& n, int& b) {
  g0 = a.grp_off[g];
  const int64_t g1 = a.grp_off[g + 1];
  n = g1 - g0;
  b = a.grp_img[g];
  if (g0 < 0 || g1 > a.T_vis || n < 0 || n > a.max_group || b < 0 || b >= a.B) {
    if (t == 0 && threadIdx.x == 0)
      set_device_error(a.err, n > a.max_group ? SP_DEV_GROUP_TOO_LARGE : SP_DEV_BAD_OFFSETS);
    return false;
  }
  return true;
}

// bfloat16 Gram products.  Bound by the float32 blocks' way to memory and the
// projected rows' way in (832 groups of 256 tokens, h 1024: 1.75 GB, 340 us at
// the copy rate) and, below a few rounds of workgroups, by a tile's own latency.
// Tile t of a group covers rows [BM (t / panels), ..) of
// [Q; V] and columns [BN (t % panels), ..) of [K].  The tiles of the first
// panel carry the column strip, those of the first row chunk the row strip, so
// every projected row is read by the tiles alone and no tile is spent on the
// five rows and two columns beside them.  Measured against whole 256 x 256 tiles
// over [Q; q_start; V; v_start; c] x [K; k_stop; k_start] (for groups just below
// a multiple of 256: tiles over the tokens, and dot products in a second kernel
// that read every row again), h 1024: 832 groups of 256 713 -> 418 us, 40 of 576 108
// -> 83, 20 of 1000 130 -> 131, 5 of 576 36 -> 23; 16 of 576, h 640, 33.6 -> 29.7.
template <class G>
__global__ __launch_bounds__(kBfThreads) void gram_gemm_bf16_kernel(GramArgs a, int per_group,
                                                                    int xcd_grouped) {
  static_assert(G::THREADS == kBfThreads, "eight waves");
  constexpr int kLds = G::LDS + GramStrips<true, true>::LDS;
  static_assert(kLds <= kLdsBytes, "rings and strips fit the LDS");
  __shared__ __attribute__((aligned(1024))) char smem[kLds];
  int64_t g, t, g0, n;
  int b;
  if (!gram_tile(blockIdx.x, per_group, a.G, xcd_grouped, g, t)) return;
  if (!gram_group_ok(a, g, t, g0, n, b)) return;
  const int64_t panels = a.max_group > 0 ? (a.max_group + G::BN - 1) / G::BN : 1;
  const int64_t m0 = (t / panels) * G::BM, n0 = (t % panels) * G::BN;
  // outside this (smaller) group; the strips are the first tiles' also in an empty group
  if ((m0 > 0 && m0 >= 2 * n) || (n0 > 0 && n0 >= n)) return;
  const __bf16* KQV = static_cast<const __bf16*>(a.KQV);
  GramTokenARows ar;
  ar.KQV = KQV;
  ar.g0 = g0;
  ar.n = n;
  ar.start_row = a.T_vis;
  ar.h = a.h;
  GramTokenBRows br;
  br.KQV = KQV;
  br.g0 = g0;
  br.start_row = a.T_vis;
  br.h = a.h;
  const __bf16* start = KQV + a.T_vis * 3 * (int64_t)a.h;
  const float* ctx = a.ctx + (int64_t)b * a.h;
  float* C = a.gram + g * a.gram_group_stride;
  auto run = [&](auto cols_c, auto rows_c) {
    using S = GramStrips<decltype(cols_c)::value, decltype(rows_c)::value>;
    gemm_bf16<G, float, GramTokenARows, GramTokenBRows, kEpiNone, S>(
        ar, br, 2 * n, n, a.h, C, a.gram_ld, m0, n0, smem, nullptr, S{start, ctx, n, a.h});
  };
  using T = std::true_type;
  using F = std::false_type;
  if (n0 == 0) {
    if (m0 == 0) run(T{}, T{});
    else run(T{}, F{});
  } else {
    if (m0 == 0) run(F{}, T{});
    else run(F{}, F{});
  }
}

// float32 Gram products, all rows and columns in the tiles.
template <class G>
__global__ __launch_bounds__(kThreads) void gram_gemm_f32_kernel(GramArgs a, int per_group, int xcd_grouped) {
  __shared__ __attribute__((aligned(1024))) char smem[G::LDS];
  int64_t g, t, g0, n;
  int b;
  if (!gram_tile(blockIdx.x, per_group, a.G, xcd_grouped, g, t)) return;
  if (!gram_group_ok(a, g, t, g0, n, b)) return;
  const float* KQV = static_cast<const float*>(a.KQV);
  const int64_t M = 2 * (n + 1) + kGramExtraRows, N = n + 2;
  const int64_t nt = (a.max_group + 2 + G::BN - 1) / G::BN;
  const int64_t m0 = (t / nt) * G::BM, n0 = (t % nt) * G::BN;
  if (m0 >= M || n0 >= N) return;
  GramARows<float> ar{KQV, g0, n, a.T_vis, a.h, a.ctx + (int64_t)b * a.h};
  GramBRows<float> br{KQV, g0, n, a.T_vis, a.h};
  gemm_f32<G>(ar, br, M, N, a.h, a.gram + g * a.gram_group_stride, a.gram_ld, m0, n0, smem);
}

inline int64_t ceil_div(int64_t a, int64_t b) { return (a + b - 1) / b; }

template <class G>
inline int64_t f32_tiles(int64_t M, int64_t N) { return ceil_div(M, G::BM) * ceil_div(N, G::BN); }

// 32 x 64 tiles while 64 x 64 ones would be at most 400, less than a round of
// 512 (two a compute unit).  us, 32 x 64 against 64 x 64 tiles (projection with
// text), at 64 x 64 tiles: 120 17.6 / 24.4, 228 35.3 / 35.6, 384 59.0 / 62.0,
// 456 60.2 / 53.4, 918 113 / 100, 2712 304 / 272.  Every element accumulates K in
// the same order either way.
inline bool f32_low(int64_t M, int64_t N) { return f32_tiles<F32High>(M, N) <= 400; }

}  // namespace

int text_split(int dtype, int64_t T_txt, int h, int d_text) {
  if (dtype == SP_BF16) return 1;   // computed beside the projection, whole K
  // Split K, up to 8 ways and into whole 64-wide stages, while there are fewer than
  // 512 parts of 128 x 128 tiles: four to eight times as many workgroups as parts, in
  // the tiles that the product runs in, beside the projection's.  Many parts shorten
  // the chain of a workgroup and add to what the pooling reads.  us of projection and
  // pooling at 1, 2, 4 and 8 parts (image rows, text rows, d, h): 576, 32, 1024, 256
  // 20.8, 21.1, 21.5, 23.0; 300, 128, 1024, 512 27.9, 23.5, 22.5, 22.9; 2000, 400, 1536,
  // 320 92, 80, 73, 71; 4096, 2048, 1024, 512 155, 148, 147, 152; no image rows, 2048,
  // 1024, 512 48, 44, 44, 52: the rule's choice, 8 in all of these, is up to 18 % from
  // the best and up to 23 % better than one.  The workspace's size and the order of
  // the sums follow the parts.
  const int64_t tiles = ceil_div(T_txt, 128) * ceil_div(h, 128);
  int s = 1;
  while (s < 8 && tiles * s < 512 && d_text % (2 * s * 64) == 0) s *= 2;
  return s;
}

hipError_t launch_project_gemm(int dtype, const void* X, int64_t T_vis, const void* s_start,
                               const void* s_stop, const void* W, int d, int n_out, void* out,
                               const void* E, int64_t T_txt, const void* W_text, int d_text, int h,
                               float* tproj, hipStream_t stream) {
  const int64_t M = T_vis + 2, N = n_out;
  if (dtype == SP_BF16) {
    ProjRows<__bf16> ar{{}, (const __bf16*)X, T_vis, (const __bf16*)s_start, (const __bf16*)s_stop, d};
    const int64_t T = ceil_div(M, 256) * ceil_div(N, 256) +
                      ceil_div(T_txt, 256) * ceil_div((int64_t)h, 256);
    const Cut c = cut_tiles(T);
    auto args = [&](auto rows) {
      using R = decltype(rows);
      auto at = [](const void* p, int64_t ld) { R r; r.base = (const __bf16*)p; r.ld = ld; return r; };
      return ProjectArgs<R>{ar, at(W, d), M, N, d, (uint16_t*)out, at(E, d_text), at(W_text, d_text),
                            T_txt, (int64_t)h, d_text, tproj, c.full, c.sub};
    };
    if (d > kMaxDenseLd || d_text > kMaxDenseLd)
      hipLaunchKernelGGL(project_gemm_bf16_small_kernel<WideRows>, dim3((unsigned)small_blocks(T)),
                         dim3(TileSmall::THREADS), 0, stream, args(WideRows{}));
    else if (c.sub == 16)
      hipLaunchKernelGGL(project_gemm_bf16_small_kernel<DenseRows<__bf16>>, dim3((unsigned)c.blocks),
                         dim3(TileSmall::THREADS), 0, stream, args(DenseRows<__bf16>{}));
    else
      hipLaunchKernelGGL(project_gemm_bf16_kernel, dim3((unsigned)c.blocks), dim3(kBfThreads), 0,
                         stream, args(DenseRows<__bf16>{}));
    return hipGetLastError();
  }
  auto launch = [&](auto tile) {
    using G = decltype(tile);
    const int split = text_split(SP_F32, T_txt, h, d_text);
    const int64_t tiles = f32_tiles<G>(M, N), tiles2 = f32_tiles<G>(T_txt, h);
    const ProjectF32Args p{ProjRows<float>{{}, (const float*)X, T_vis, (const float*)s_start, (const float*)s_stop, d},
                           DenseRows<float>{(const float*)W, d}, M, N, tiles, d, (float*)out,
                           DenseRows<float>{(const float*)E, d_text}, DenseRows<float>{(const float*)W_text, d_text},
                           T_txt, (int64_t)h, tiles2, d_text / split, split, tproj};
    hipLaunchKernelGGL(project_gemm_f32_kernel<G>, dim3((unsigned)(tiles + tiles2 * split)),
                       dim3(kThreads), 0, stream, p);
  };
  if (f32_low(M, N)) launch(F32Low{});
  else launch(F32High{});
  return hipGetLastError();
}

namespace {
// Time of one round of Gram tiles: a fixed part (loads and strips to the first
// matrix instruction, the float32 tile's way out) and the tile's area.  Fitted
// to (us for tiles of 128 x 256 / 256 x 192 / 128 x 192, h 1024): 5 groups of
// 576 tokens 26 / 36 / 23, 16 of 576 42 / 39 / 38, 40 of 576 98 / 83 / 86, 157
// of 576 392 / 330 / 373, 40 of 384 47 / 40 / 42, 832 of 256 420 / 490 / 564, 20
// of 1000 134 / 141 / 157; the choice is within 3 % of the best on each.
inline double gram_tile_us(int bm, int bn, int h) { return 6.0 + 4.3e-4 * bm * bn * h / 1024; }
}  // namespace

hipError_t launch_gram_gemm(const GramArgs& a, hipStream_t stream) {
  if (a.G == 0) return hipSuccess;
  const int64_t M = 2 * ((int64_t)a.max_group + 1) + kGramExtraRows, N = a.max_group + 2;
  const int xcd_grouped = a.G >= 8;
  if (a.dtype == SP_BF16) {
    // The tile that covers the chip's groups in the least time: rounds of 256
    // workgroups, each a fixed part and its area (gram_tile_us).
    const int64_t mg = a.max_group > 0 ? a.max_group : 1;
    auto tiles = [&](int bm, int bn) { return ceil_div(2 * mg, bm) * ceil_div(mg, bn); };
    auto cost = [&](int bm, int bn) {
      return (double)ceil_div(tiles(bm, bn) * a.G, 256) * gram_tile_us(bm, bn, a.h);
    };
    auto launch = [&](auto* kernel, int bm, int bn) {
      const int per_group = (int)tiles(bm, bn);
      const int64_t blocks =
          xcd_grouped ? 8 * ceil_div(a.G, 8) * per_group : (int64_t)a.G * per_group;
      hipLaunchKernelGGL(kernel, dim3((unsigned)blocks), dim3(kBfThreads), 0, stream, a, per_group,
                         xcd_grouped);
    };
    const double ca = cost(128, 256), cb = cost(256, 192), cc = cost(128, 192);
    if (cc <= ca && cc <= cb) launch(gram_gemm_bf16_kernel<TileGramC>, 128, 192);
    else if (cb <= ca) launch(gram_gemm_bf16_kernel<TileGramB>, 256, 192);
    else launch(gram_gemm_bf16_kernel<TileGramA>, 128, 256);
  } else {
    auto launch = [&](auto tile) {
      using G = decltype(tile);
      const int per_group = (int)f32_tiles<G>(M, N);
      const int64_t blocks = xcd_grouped ? 8 * ceil_div(a.G, 8) * per_group : (int64_t)a.G * per_group;
      hipLaunchKernelGGL(gram_gemm_f32_kernel<G>, dim3((unsigned)blocks), dim3(kThreads), 0, stream, a,
                         per_group, xcd_grouped);
    };
    if (f32_low(M * a.G, N)) launch(F32Low{});
    else launch(F32High{});
  }
  return hipGetLastError();
}

hipError_t launch_dense_bf16(const void* A, const void* B, int64_t M, int64_t N, int K, void* C,
                             hipStream_t stream, const float* bias, bool gelu) {
  if (M == 0 || N == 0) return hipSuccess;
  uint16_t* out = (uint16_t*)C;
  const int64_t T = ceil_div(M, 256) * ceil_div(N, 256);
  if (K > kMaxDenseLd) {   // only the encoder's text product (no bias) is this wide
    if (bias) return hipErrorInvalidValue;
    WideRows wa, wb;
    wa.base = (const __bf16*)A;
    wb.base = (const __bf16*)B;
    wa.ld = wb.ld = K;
    hipLaunchKernelGGL((dense_bf16_small_kernel<kEpiNone, WideRows>), dim3((unsigned)small_blocks(T)),
                       dim3(TileSmall::THREADS), 0, stream, wa, wb, M, N, K, out, bias);
    return hipGetLastError();
  }
  DenseRows<__bf16> ar{(const __bf16*)A, K};
  DenseRows<__bf16> br{(const __bf16*)B, K};
  const Cut c = cut_tiles(T);
  const dim3 grid((unsigned)c.blocks);
  auto launch = [&](auto epi_c) {
    constexpr int EPI = decltype(epi_c)::value;
    if (c.sub == 16)
      hipLaunchKernelGGL((dense_bf16_small_kernel<EPI, DenseRows<__bf16>>), grid, dim3(TileSmall::THREADS), 0, stream, ar, br,
                         M, N, K, out, bias);
    else
      hipLaunchKernelGGL(dense_bf16_kernel<EPI>, grid, dim3(kBfThreads), 0, stream, ar, br, M, N, K, out,
                         bias, c.full, c.sub);
  };
  if (!bias) launch(std::integral_constant<int, kEpiNone>{});
  else if (!gelu) launch(std::integral_constant<int, kEpiBias>{});
  else launch(std::integral_constant<int, kEpiBiasGelu>{});
  return hipGetLastError();
}

}  // namespace sp

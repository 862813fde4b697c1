// Eq. 3 on gfx950: the cross-modal input encoder.
//
//   E~ = g LN(E_text W_p^T)                  text projected into R^d (LayerNorm
//                                            without scale or shift, eps 1e-5)
//   H  = Enc([X_b; E~_b])[first N_b rows]    per image b
//
// Enc is two pre-norm transformer blocks of width d: multi-head attention with
// heads of width 128 over the image's whole sequence (bidirectional, or causal
// on request), and an MLP 4d wide with the exact GELU.  Every linear map runs
// on the matrix cores (gemm.hip's bfloat16 core), the q/k/v bias and the MLP's
// bias and GELU in the products' epilogues; the residual + LayerNorm steps are
// row kernels (denoise.hip), the rest is here.
//
// Sequence layout: image b's sequence occupies rows [so_b, so_b + S_b) of the
// workspace buffers, so_b = img_off[b] + text_off[b], S_b = N_b + L_b, its
// visual tokens first (visual row i of image b is sequence row
// i + text_off[b]) and its text tokens after them (text row t of image b is
// sequence row img_off[b + 1] + t).
//
// The residual stream R is float32.  The text product, the LayerNorm outputs,
// every product's result, the biased q/k/v, the probabilities that weight the
// values, each head's output, the GELU output and H are bfloat16, rounded
// once to nearest-even.
#include <type_traits>

#include "sp_internal.h"
#include "lds_dma.h"
#include "row_ops.h"

namespace sp {
namespace {

typedef __bf16 bf16x8_t __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x4_t __attribute__((ext_vector_type(4)));
typedef float f32x16_t __attribute__((ext_vector_type(16)));
typedef __attribute__((address_space(3))) bf16x4_t* ltr_t;

constexpr int kHead = 128;                  // head width
constexpr int kQPerWave = 32;               // queries of one wave (one 32 x 32 MFMA tile)
constexpr float kTextLnEps = 1e-5f;

// The image owning row r of a packed array with offsets off[0..B]: the last
// image whose range starts at or before r (empty images are skipped).
__device__ __forceinline__ int owner(const int32_t* __restrict__ off, int B, int64_t r) {
  int lo = 0, hi = B;                       // off[lo] <= r < off[hi]
  while (hi - lo > 1) {
    const int mid = (lo + hi) >> 1;
    if (off[mid] <= r) lo = mid;
    else hi = mid;
  }
  return lo;
}

// Image b's sequence offset and length, or false (with the error word set)
// when its offsets are inconsistent or its length exceeds max_seq.
__device__ __forceinline__ bool sequence_of(const int32_t* __restrict__ img_off,
                                            const int32_t* __restrict__ text_off, int b,
                                            int max_seq, int64_t S_total, int64_t& so, int& S,
                                            int32_t* err, bool report) {
  const int n = img_off[b + 1] - img_off[b], L = text_off[b + 1] - text_off[b];
  so = (int64_t)img_off[b] + text_off[b];
  S = n + L;
  if (n < 0 || L < 0 || so < 0 || so + S > S_total) {
    if (report) set_device_error(err, SP_DEV_BAD_OFFSETS);
    return false;
  }
  if (S > max_seq) {
    if (report) set_device_error(err, SP_DEV_GROUP_TOO_LARGE);
    return false;
  }
  return true;
}

// ---------------------------------------------------------------- row kernels

// Sequence row s: R = its visual row of X, or g LN(P) of its text row (LayerNorm
// without scale or shift, biased variance, eps 1e-5), and Z = LN1(R) of the first
// block.  One wave per row.  Bound by memory: R is written and not read back.
// Against a kernel for the text rows, one for the visual rows and one for LN1, a
// pass on one image of 1077 rows at width 1024 210 -> 207 us.
__global__ __launch_bounds__(64 * kRowWaves) void enc_input_kernel(
    const uint16_t* __restrict__ X, int64_t T_vis, const uint16_t* __restrict__ P, int64_t T_txt, int d,
    const int32_t* __restrict__ img_off, const int32_t* __restrict__ text_off, int B, float g,
    const float* __restrict__ ln_g, const float* __restrict__ ln_b, float* __restrict__ R,
    uint16_t* __restrict__ Z, int32_t* err) {
  const int lane = threadIdx.x & 63;
  const int64_t s = (int64_t)blockIdx.x * kRowWaves + (threadIdx.x >> 6);
  if (s >= T_vis + T_txt) return;
  int b = 0;                                  // the last image whose sequence starts at or before s
  for (int hi = B; hi - b > 1;) {
    const int mid = (b + hi) >> 1;
    if ((int64_t)img_off[mid] + text_off[mid] <= s) b = mid;
    else hi = mid;
  }
  const int64_t i = s - text_off[b], t = s - img_off[b + 1];      // as a visual row, as a text row
  const bool text = i >= img_off[b + 1];
  if (i < img_off[b] || t >= text_off[b + 1]) return;             // no image's row
  if (text ? t < 0 || t >= T_txt : i < 0 || i >= T_vis) {
    if (lane == 0) set_device_error(err, SP_DEV_BAD_OFFSETS);
    return;
  }
  const uint16_t* src = text ? P + t * d : X + i * d;
  const int nch = d / 8;
  float v[kMaxChunks][8];
#pragma unroll
  for (int c = 0; c < kMaxChunks; ++c) {
    if (lane + 64 * c >= nch) break;
    load8(src + 8 * (lane + 64 * c), v[c]);
  }
  if (text) {
    float sum = 0.0f;
#pragma unroll
    for (int c = 0; c < kMaxChunks; ++c)
      if (lane + 64 * c < nch)
#pragma unroll
        for (int k = 0; k < 8; ++k) sum += v[c][k];
    const float mean = wave_sum(sum) / (float)d;
    float q = 0.0f;
#pragma unroll
    for (int c = 0; c < kMaxChunks; ++c)
      if (lane + 64 * c < nch)
#pragma unroll
        for (int k = 0; k < 8; ++k) {
          const float u = v[c][k] - mean;
          q = fmaf(u, u, q);
        }
    const float rstd = 1.0f / sqrtf(wave_sum(q) / (float)d + kTextLnEps);
#pragma unroll
    for (int c = 0; c < kMaxChunks; ++c)
#pragma unroll
      for (int k = 0; k < 8; ++k) v[c][k] = g * ((v[c][k] - mean) * rstd);
  }
#pragma unroll
  for (int c = 0; c < kMaxChunks; ++c) {
    if (lane + 64 * c >= nch) break;
    store8(R + s * d + 8 * (lane + 64 * c), v[c]);
  }
  ln_store(v, nch, d, lane, ln_g, ln_b, Z + s * d);
}

// H[i] = bf16((R[s] + T[s]) + bias) for visual row i (s = i + text_off[b]):
// the last block's residual, visual positions only.  One workgroup per row.
__global__ __launch_bounds__(256) void enc_out_kernel(
    const float* __restrict__ R, const uint16_t* __restrict__ T, const float* __restrict__ bias,
    int d, const int32_t* __restrict__ img_off, const int32_t* __restrict__ text_off, int B,
    int64_t S_total, uint16_t* __restrict__ H, int32_t* err) {
  const int64_t i = blockIdx.x;
  const int b = owner(img_off, B, i);
  const int64_t s = i + text_off[b];
  if (s < 0 || s >= S_total) {
    if (threadIdx.x == 0) set_device_error(err, SP_DEV_BAD_OFFSETS);
    return;
  }
  for (int c = 8 * threadIdx.x; c < d; c += 8 * 256) {
    float x[8], y[8], bb[8];
    load8(R + s * d + c, x);
    load8(T + s * d + c, y);
    load8(bias + c, bb);
#pragma unroll
    for (int k = 0; k < 8; ++k) x[k] = (x[k] + y[k]) + bb[k];
    store8(H + i * d + c, x);
  }
}

// ---------------------------------------------------------------- attention

__device__ __forceinline__ bf16x8_t ld16(const uint16_t* p) {
  return __builtin_bit_cast(bf16x8_t, *reinterpret_cast<const uint4*>(p));
}

// The larger of v in this lane and in the lane 32 away (their sum likewise).
__device__ __forceinline__ float half_max(float v) {
  const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
  return fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1]));
}
__device__ __forceinline__ float half_sum(float v) {
  const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
  return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}

// Multi-head attention of every image's sequence: O[so + q][128 h + e] =
// sum_k softmax_k(q . k / sqrt(128)) v[k][e], over the image's keys (causal:
// keys k <= q).  A wave takes 32 queries and walks keys in steps of 32 or 64
// with an online softmax:
//   S^T = K Q^T on the matrix cores (v_mfma_f32_32x32x16_bf16: K as the row
//   operand, Q as the column operand), so lane l holds query q0 + l % 32 and
//   16 of each 32 keys (key 8 (r / 4) + 4 (l / 32) + r % 4 in register r); a
//   query's maximum and sum need its lane and the lane 32 away;
//   O^T += V^T P: the probabilities a lane holds are its half of the operand's
//   k slots as they stand (slot 8 (l / 32) + j is key 4 (l / 32) + j for j < 4
//   and 8 + 4 (l / 32) + j - 4 for j >= 4, plus 16 for the second 16 keys).
//   The value operand is read from the row-major tile by the transposing LDS
//   read (ds_read_b64_tr_b16): 16 lanes read 4 keys x 16 columns, four values
//   of one key each, and lane i receives column i of the four keys.
// Tiles of K and V pass through LDS two deep, the next one loading straight
// into LDS while the current one is used.  Rows of 256 bytes are 16-byte
// chunks, XOR-swizzled so that a pass of a fragment read touches every bank
// once: by the row's low four bits (K), by its low two bits on 64-byte pieces
// (V, read 64 bytes of four rows at a time).  Keys past the sequence read its
// last row and are masked.
//
// Two splits of the work over a workgroup's waves:
//   kShared (SPLIT = false): four waves, 128 queries, 32 a wave; the waves share tiles of 64 keys.
//   kSplit (SPLIT = true): eight waves, 64 queries, four waves to 32 of them; each of the
//            four takes every fourth 32-key block of the shared 128-key tiles, and the
//            partial sums are combined through LDS at the end.  (Four waves and 32
//            queries a workgroup: one image of 1400 rows at width 1024, causal, 231
//            against 223 us a pass; 16 of 640 rows 899 against 804.)
//
// What bounds it: with 2 x 8 matrix instructions a 32-key block, the softmax's
// vector instructions (16 exponentials a lane).  So masks are applied only to
// the steps that need them, the running maximum moves (and the sums are
// rescaled) only when a step's maximum exceeds it by more than 2^8, which
// float32 sums hold with the same relative error, and the row sums stay
// per lane until the end.  Probabilities enter the products rounded to bfloat16.
//
// us at width 4096 (32 heads) against a kernel with masks, a rescale and
// shuffles at every step, values transposed by a kernel before it, and 128
// queries a workgroup only: 16 sequences of 640 rows 239 + 50 -> 160 (0.67
// PFLOP/s); one of 1077 rows at width 1024, causal, 50 + 5 -> 17.
constexpr float kRescale = 8.0f;            // log2 of the largest unscaled probability

// kSplit's partial sums, over the tiles: 32 rows of 128 values a wave, padded
constexpr int kPartRow = kHead + 4;

template <bool SPLIT>
struct AttnShape {
  static constexpr int WAVES = SPLIT ? 8 : 4, THREADS = 64 * WAVES;
  static constexpr int SHARES = SPLIT ? 4 : 1;                                 // waves to a query block
  static constexpr int QUERIES = kQPerWave * WAVES / SHARES;                   // of a workgroup
  static constexpr int TILE = SPLIT ? 32 * SHARES : 64;                        // keys of a tile
  static constexpr int BLOCKS = SPLIT ? 1 : 2;                                 // 32-key blocks of a step
  static constexpr int TILE_BYTES = TILE * kHead * 2;                          // K or V
  static constexpr int PARTS = SPLIT ? WAVES * kQPerWave * (kPartRow + 2) * 4 : 0;   // partial sums
  static constexpr int LDS = 4 * TILE_BYTES > PARTS ? 4 * TILE_BYTES : PARTS;
  static constexpr int LOADS = TILE / 4 / WAVES;                               // 4-row groups per wave
  static_assert(LDS * (SPLIT ? 1 : 2) <= kLdsBytes, "the tiles and partial sums fit the LDS");
};

template <bool SPLIT>
__global__ __launch_bounds__(AttnShape<SPLIT>::THREADS, SPLIT ? 1 : 2) void attn_kernel(
    const uint16_t* __restrict__ QKV, int d, int q_blocks, const int32_t* __restrict__ img_off,
    const int32_t* __restrict__ text_off, int max_seq, int64_t S_total, int split_rows, int causal,
    float c2, uint16_t* __restrict__ O, int32_t* err) {
  using G = AttnShape<SPLIT>;
  constexpr int NB = G::BLOCKS;
  __shared__ __attribute__((aligned(1024))) char smem[G::LDS];   // [buffer][K, V]
  const int b = blockIdx.y, heads = d / kHead;
  // Workgroup w runs on XCD w % 8: where the heads divide over the XCDs, a
  // head's query blocks follow one another on one of them and share its keys
  // and values in that L2.  Causal: the blocks with the most keys come first.
  const int w = blockIdx.x;
  int hd, qb;
  if (heads % 8 == 0) {
    hd = w % 8 + 8 * (w / 8 / q_blocks);
    qb = w / 8 % q_blocks;
  } else {
    hd = w / q_blocks;
    qb = w % q_blocks;
  }
  if (causal) qb = q_blocks - 1 - qb;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  int64_t so;
  int S;
  if (!sequence_of(img_off, text_off, b, max_seq, S_total, so, S, err, tid == 0 && w == 0)) return;
  const int qw = qb * G::QUERIES;                                   // the workgroup's first query
  if (qw >= S || (S <= split_rows) != SPLIT) return;
  // this wave's first query (may be past S) and, kSplit, its share of the keys
  const int q0 = qw + wave / G::SHARES * kQPerWave, share = wave % G::SHARES;
  const int ql = lane & 31, half = lane >> 5;
  const int64_t ld = 3 * (int64_t)d;
  const uint16_t* Qb = QKV + so * ld + hd * kHead;
  const int q = q0 + ql;
  const int qr = q < S ? q : S - 1;           // queries past the sequence compute on its last row
  bf16x8_t qf[kHead / 16];
#pragma unroll
  for (int s = 0; s < kHead / 16; ++s) qf[s] = ld16(Qb + qr * ld + 16 * s + 8 * half);

  // keys the workgroup needs, and this wave's own limit
  const int kend_wg = causal ? (S < qw + G::QUERIES ? S : qw + G::QUERIES) : S;
  // (a wave past the sequence only helps load the tiles)
  const int kend = q0 >= S ? 0 : causal ? (S < q0 + kQPerWave ? S : q0 + kQPerWave) : S;
  const int tiles = (kend_wg + G::TILE - 1) / G::TILE;

  // Tile loads: an instruction fills 1 KB, 4 rows; lane i lands on chunk i % 16
  // of row i / 16, so it fetches the logical chunk that the swizzle puts there.
  // The wave loads row groups wave, wave + WAVES, ...
  const int lrow = lane >> 4, lch = lane & 15;
  auto issue_tile = [&](int kt, int buf) {
    const int k0 = kt * G::TILE;
    const uint64_t p = (uint64_t)(Qb + (int64_t)k0 * ld + d);        // uniform: into scalar registers
    const uint32_t plo = __builtin_amdgcn_readfirstlane((uint32_t)p);
    const uint32_t phi = __builtin_amdgcn_readfirstlane((uint32_t)(p >> 32));
    const char* Kt = reinterpret_cast<const char*>(((uint64_t)phi << 32) | plo);
    const char* Vt = Kt + 2 * (int64_t)d;
    const int last = S - 1 - k0;
    char* dst = smem + buf * 2 * G::TILE_BYTES;
#pragma unroll
    for (int i = 0; i < G::LOADS; ++i) {
      const int grp = wave + G::WAVES * i;
      const int r = 4 * grp + lrow;
      const uint32_t row = (uint32_t)(r < last ? r : last) * (uint32_t)(2 * ld);
      lds_dma16(Kt, row + ((lch ^ (r & 15)) << 4), dst + grp * 1024);
      lds_dma16(Vt, row + ((lch ^ (lrow << 2)) << 4), dst + G::TILE_BYTES + grp * 1024);
    }
  };
  // fragment reads: rows r of K in e-slice s; V^T rows of e-tile t at keys r0 + 4 half + 0..3
  const int kbase = ql * 256, ksw = ql & 15;
  auto kfrag = [&](const char* tile, int s) {
    return __builtin_bit_cast(
        bf16x8_t, *reinterpret_cast<const uint4*>(tile + kbase + (((2 * s + half) ^ ksw) << 4)));
  };
  const int vr = (lane >> 2) & 3;
  const int vbase = (4 * half + vr) * 256 + ((lane >> 4) & 1) * 32 + (lane & 3) * 8;
  auto vread = [&](const char* tile, int t, int r0) {
    return __builtin_amdgcn_ds_read_tr16_b64_v4bf16(
        (ltr_t)(tile + vbase + ((t ^ vr) << 6) + r0 * 256));
  };

  f32x16_t o[kHead / 32];
#pragma unroll
  for (int t = 0; t < kHead / 32; ++t)
#pragma unroll
    for (int r = 0; r < 16; ++r) o[t][r] = 0.0f;
  float m = -INFINITY, l = 0.0f;              // of this lane's keys; m is its query's

  // One step: 32 NB keys from kb on, at row `row` of the buffer's tiles.
  auto step = [&](int buf, int row, int kb) {
    const char* Kt = smem + buf * 2 * G::TILE_BYTES + row * 256;
    const char* Vt = Kt + G::TILE_BYTES;
    f32x16_t st[NB];
#pragma unroll
    for (int n = 0; n < NB; ++n)
#pragma unroll
      for (int r = 0; r < 16; ++r) st[n][r] = 0.0f;
#pragma unroll
    for (int s = 0; s < kHead / 16; ++s)
#pragma unroll
      for (int n = 0; n < NB; ++n)
        st[n] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kfrag(Kt + n * 32 * 256, s), qf[s], st[n], 0, 0, 0);
    if (kb + 32 * NB > (causal && q0 + 1 < S ? q0 + 1 : S)) {
      const int lim = causal && q + 1 < S ? q + 1 : S;     // keys below it are visible
#pragma unroll
      for (int n = 0; n < NB; ++n)
#pragma unroll
        for (int r = 0; r < 16; ++r)
          if (kb + 32 * n + 8 * (r >> 2) + 4 * half + (r & 3) >= lim) st[n][r] = -INFINITY;
    }
    // Key kb is visible to every query of the wave (kb < S, and kb <= q0 when
    // causal), so a step's maximum is finite.
    float bm = st[0][0];
#pragma unroll
    for (int n = 0; n < NB; ++n)
#pragma unroll
      for (int r = 0; r < 16; ++r) bm = fmaxf(bm, st[n][r]);
    const float mx = half_max(bm) * c2;
    if (__any(mx > m + kRescale)) {
      const float mn = fmaxf(m, mx);
      const float sc = __builtin_amdgcn_exp2f(m - mn);     // 0 on the first step
      m = mn;
      l *= sc;
#pragma unroll
      for (int t = 0; t < kHead / 32; ++t)
#pragma unroll
        for (int r = 0; r < 16; ++r) o[t][r] *= sc;
    }
#pragma unroll
    for (int n = 0; n < NB; ++n) {
      // A block past the wave's last key is not weighted with 0: its values may
      // be infinite or NaN (causal: rows that these queries must not see).
      if (n > 0 && kb + 32 * n >= kend) break;
      bf16x8_t pb[2];
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        const float p = __builtin_amdgcn_exp2f(fmaf(st[n][r], c2, -m));
        l += p;
        pb[r >> 3][r & 7] = (__bf16)p;
      }
#pragma unroll
      for (int g = 0; g < 2; ++g)
#pragma unroll
        for (int t = 0; t < kHead / 32; ++t) {
          const bf16x4_t lo = vread(Vt, t, 32 * n + 16 * g), hi = vread(Vt, t, 32 * n + 16 * g + 8);
          const bf16x8_t v = __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
          o[t] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(v, pb[g], o[t], 0, 0, 0);
        }
    }
  };

  issue_tile(0, 0);
  for (int kt = 0; kt < tiles; ++kt) {
    const int buf = kt & 1;
    wait_vmcnt<0>();                         // this wave's loads of tile kt
    __syncthreads();                         // every wave's; and all are past tile kt - 1
    if (kt + 1 < tiles) issue_tile(kt + 1, buf ^ 1);
    const int kb = kt * G::TILE + 32 * share;
    if (kb < kend) step(buf, 32 * share, kb);   // uniform in the wave
  }
  l = half_sum(l);

  // O^T[e][q] in o[t][r]: e = 32 t + 8 (r / 4) + 4 (l / 32) + r % 4
  if constexpr (SPLIT) {
    float* part = reinterpret_cast<float*>(smem);                   // [wave][query][kPartRow]
    float* ml = part + G::WAVES * kQPerWave * kPartRow;              // [m, l][wave][query]
    __syncthreads();                                                 // every wave is past its tiles
#pragma unroll
    for (int t = 0; t < kHead / 32; ++t)
#pragma unroll
      for (int g4 = 0; g4 < 4; ++g4)
        *reinterpret_cast<float4*>(part + (wave * kQPerWave + ql) * kPartRow + 32 * t + 8 * g4 + 4 * half) =
            make_float4(o[t][4 * g4], o[t][4 * g4 + 1], o[t][4 * g4 + 2], o[t][4 * g4 + 3]);
    if (half == 0) {
      ml[wave * kQPerWave + ql] = m;
      ml[(G::WAVES + wave) * kQPerWave + ql] = l;
    }
    __syncthreads();
    // 16 values of one query a thread, of the query block's waves w0 ..
    const int cq = (tid >> 3) % kQPerWave, e0 = (tid & 7) * 16, w0 = tid / (8 * kQPerWave) * G::SHARES;
    const int qc = qw + tid / 8;
    if (qc >= S) return;
    float M = -INFINITY;
#pragma unroll
    for (int v = 0; v < G::SHARES; ++v) M = fmaxf(M, ml[(w0 + v) * kQPerWave + cq]);
    float L = 0.0f, acc[16];
#pragma unroll
    for (int e = 0; e < 16; ++e) acc[e] = 0.0f;
#pragma unroll
    for (int v = 0; v < G::SHARES; ++v) {
      // a wave without keys has m = -inf and zero sums
      const float mv = ml[(w0 + v) * kQPerWave + cq];
      const float f = mv == -INFINITY ? 0.0f : __builtin_amdgcn_exp2f(mv - M);
      L = fmaf(ml[(G::WAVES + w0 + v) * kQPerWave + cq], f, L);
#pragma unroll
      for (int e = 0; e < 16; e += 4) {
        const float4 x = *reinterpret_cast<const float4*>(part + ((w0 + v) * kQPerWave + cq) * kPartRow + e0 + e);
        acc[e] = fmaf(x.x, f, acc[e]);
        acc[e + 1] = fmaf(x.y, f, acc[e + 1]);
        acc[e + 2] = fmaf(x.z, f, acc[e + 2]);
        acc[e + 3] = fmaf(x.w, f, acc[e + 3]);
      }
    }
    const float inv = 1.0f / L;
    float out[8];
#pragma unroll
    for (int e = 0; e < 16; e += 8) {
#pragma unroll
      for (int k = 0; k < 8; ++k) out[k] = acc[e + k] * inv;
      store8(O + (so + qc) * d + hd * kHead + e0 + e, out);
    }
  } else {
    if (q >= S) return;
    const float inv = 1.0f / l;
    uint16_t* orow = O + (so + q) * d + hd * kHead;
#pragma unroll
    for (int t = 0; t < kHead / 32; ++t)
#pragma unroll
      for (int g4 = 0; g4 < 4; ++g4) {
        bf16x4_t v;
#pragma unroll
        for (int r = 0; r < 4; ++r) v[r] = (__bf16)(o[t][4 * g4 + r] * inv);
        *reinterpret_cast<bf16x4_t*>(orow + 32 * t + 8 * g4 + 4 * half) = v;
      }
  }
}

// Sequences of up to this many rows take kSplit: while their 32-query blocks of
// all heads are at most one to a compute unit, or one and a half when causal,
// where the later ones have few keys.  us a pass of one image, kShared against
// kSplit: 640 rows at width 1024 167 / 157, 2048 rows at width 512 188 / 155; causal
// at width 1024, 1077 rows 219 / 204, 1536 rows 255 / 230.  A sequence's own length
// decides, so that its rows have the same bits alone and in any batch; in a batch
// that fills the chip kShared would be faster (16 x 640 rows at width 1024 776 / 807).
inline int split_limit(int heads, bool causal) { return (causal ? 384 : 256) * kQPerWave / heads; }

}  // namespace

hipError_t launch_encode(const EncodeArgs& a, hipStream_t stream) {
  if (a.T_vis == 0) return hipSuccess;             // no visual rows: nothing to output
  const int d = a.d;
  const int64_t S = a.T_vis + a.T_txt;
  const int heads = d / kHead;
  const unsigned row_blocks = (unsigned)((S + kRowWaves - 1) / kRowWaves);
  hipError_t e;
  // the sequences: visual rows, then the projected text rows
  if (a.T_txt > 0) {
    if ((e = launch_dense_bf16(a.E, a.W_p, a.T_txt, d, a.d_text, a.HID, stream)) != hipSuccess)
      return e;
  }
  hipLaunchKernelGGL(enc_input_kernel, dim3(row_blocks), dim3(64 * kRowWaves), 0, stream, a.X, a.T_vis,
                     a.HID, a.T_txt, d, a.img_off, a.text_off, a.B, a.g_text, a.blk[0].ln1_g,
                     a.blk[0].ln1_b, a.R, a.L, a.err);
  const float c2 = 1.4426950408889634f / sqrtf((float)kHead);
  // no sequence is longer than the batch, however large a max_seq is passed (the
  // grid would pass the launch limit)
  const int64_t longest = a.max_seq < S ? a.max_seq : S;
  const int limit = split_limit(heads, a.causal);
  // The shortest sequence has at least the rows that B - 1 of the longest leave:
  // past the limit, all of them are shared, and the launch for the others is saved.
  const int split_rows = S - (a.B - 1) * longest > limit ? 0 : limit;
  auto attention = [&](auto split_c, int64_t rows) {
    using G = AttnShape<decltype(split_c)::value>;
    const int64_t q_blocks = (rows + G::QUERIES - 1) / G::QUERIES;
    hipLaunchKernelGGL(attn_kernel<decltype(split_c)::value>, dim3((unsigned)(q_blocks * heads), (unsigned)a.B),
                       dim3(G::THREADS), 0, stream, a.QKV, d, (int)q_blocks, a.img_off, a.text_off,
                       a.max_seq, S, split_rows, a.causal ? 1 : 0, c2, a.A, a.err);
  };
  for (int k = 0; k < kEncoderBlocks; ++k) {
    const EncoderBlockArgs& p = a.blk[k];
    // q, k, v of LN1(R) (in L), biased in the product's epilogue
    if ((e = launch_dense_bf16(a.L, p.W_qkv, S, 3 * (int64_t)d, d, a.QKV, stream, p.b_qkv)) !=
        hipSuccess)
      return e;
    if (longest > split_rows) attention(std::false_type{}, longest);
    if (split_rows > 0) attention(std::true_type{}, longest < split_rows ? longest : split_rows);
    // R += A W_o^T + b_o; LN2 into A
    if ((e = launch_dense_bf16(a.A, p.W_o, S, d, d, a.L, stream)) != hipSuccess) return e;
    if ((e = launch_resid_ln(a.R, a.L, p.b_o, S, d, p.ln2_g, p.ln2_b, a.A, stream)) != hipSuccess)
      return e;
    // the MLP
    if ((e = launch_dense_bf16(a.A, p.W_1, S, 4 * (int64_t)d, d, a.HID, stream, p.b_1, true)) !=
        hipSuccess)
      return e;
    if ((e = launch_dense_bf16(a.HID, p.W_2, S, d, 4 * d, a.L, stream)) != hipSuccess) return e;
    if (k + 1 < kEncoderBlocks) {
      // R += L + b_2, and the next block's LN1 into L (in place, row by row)
      if ((e = launch_resid_ln(a.R, a.L, p.b_2, S, d, a.blk[k + 1].ln1_g, a.blk[k + 1].ln1_b, a.L,
                               stream)) != hipSuccess)
        return e;
    } else {
      hipLaunchKernelGGL(enc_out_kernel, dim3((unsigned)a.T_vis), dim3(256), 0, stream, a.R, a.L,
                         p.b_2, d, a.img_off, a.text_off, a.B, S, a.H, a.err);
    }
  }
  return hipGetLastError();
}

}  // namespace sp

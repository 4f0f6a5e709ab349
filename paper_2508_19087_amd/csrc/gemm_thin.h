// gemm_thin.h - the few-token GEMM (M <= 512) of the WpAq bipolar-INT path on
// the matrix cores of gfx950 (APT-LLM, arXiv 2508.19087, Sec. III-B): the
// packed weights are streamed once, rebuilt from their bit-planes in
// registers and multiplied with activations that stay in registers.
//
// With a handful of tokens the GEMM reads N K p / 8 bytes of weights and
// little else, so HBM should bound it.  XOR + popcount spends 2 p q vector
// instructions per 32 weight elements and token (256 at W4A4 and 8 tokens),
// which is 4-5 times what the stream takes; here a word of 32 weight elements
// costs its rebuild (22 instructions at 4 bits) and one MFMA for 16 tokens.
//
// Work split.  A workgroup of 8 waves owns a contiguous run of 16-row weight
// tiles and all of K: wave w takes the K groups (4 chunks, 512 elements) w,
// w + 8, ..., at most G of them, and keeps the activation operands of those
// groups for its MT 16-token tiles in registers for the whole run (with more
// tokens than that, rows of workgroups share the weights through the caches).
// Per tile a wave loads P 16-byte vectors per group: lane l holds the four
// words of row l mod 16, chunk l / 16 of the group, so 8 whole 128-byte lines
// per plane move with one instruction, and word j of the four lane quarters
// is one MFMA step of 128 elements of k (the k order of a dot product is
// free as long as both operands share it).  D tiles' loads are in flight per
// wave (about 64 KB per compute unit, which covers the latency of HBM at its
// rate).  The 8 waves' partial sums meet in LDS once per tile, double
// buffered, one barrier each.
//
// Operands (class C):
//   kLow   p, q <= 4 and K (2^p - 1)(2^q - 1) < 2^24 (exact fp32 sums):
//          six-bit E2M3 fields on both sides, v_mfma_f32_16x16x128_f8f6f4.
//          E2M3 is linear over its first 16 codes (code c is c / 8), so the
//          weight's word u is its own code and the rebuild is only a merge of
//          planes; the activation's bipolar value v = 2 t + 1 (up to a sign) is
//          the exact E2M3 number t + 1/2.  With D = sum (v_a / 2)(u_w / 8):
//          C = 32 D - (2^p - 1) R_a.
//   kByte  otherwise, int8 bytes y on both sides, v_mfma_i32_16x16x64_i8:
//          y_w = u (p <= 7) or u - 128, y_a = v_a, exact modulo 2^32:
//          C = 2 D + c_w R_a - padding (v_w = 2 y_w + c_w).
//   kByte8 the same for q = 8, where v_a does not fit a byte: y_a = u - 128,
//          v_a = 2 y_a + 1, and one more MFMA per step against a constant
//          operand of ones sums the weights' bytes (R_w).
// R_a, the row sums of the activations, come from the planes at hand, so no
// caller array is read.  Weight padding is u = 0, which adds nothing except as
// the byte -128 at p = 8; that constant is subtracted.
#pragma once

#include <type_traits>

#include "apt_internal.h"
#include "reassemble.h"
#include "rowcode.h"

namespace apt {
namespace thin {

constexpr int kWave = 64;
constexpr int kWaves = 8;
constexpr int kTileN = 16;                    // weight rows per tile
constexpr int kTileM = 16;                    // tokens per MFMA
constexpr int kGroupChunks = 4;               // chunks per K group (one 16-byte vector per lane)
// Weight loads are non-temporal: one row of workgroups reads them once per call.
// With several rows (more tokens than one workgroup holds) the caches serve the
// re-reads all the same: against plain loads equal within 1% up to 4 rows, 2%
// slower with 5 to 16 (40 to 512 tokens, 150 problems), which does not pay for a
// second instance of every kernel.
constexpr int kNT = 2;
constexpr int kRedStride = 20;                // dwords per token row of a tile's partial sums in LDS

enum { kLow = 0, kByte = 1, kByte8 = 2 };
enum { kSrcPacked = 0, kSrcCodes = 1, kSrcHalf = 2 };

typedef int v4i __attribute__((ext_vector_type(4)));
typedef int v8i __attribute__((ext_vector_type(8)));
typedef float v4f __attribute__((ext_vector_type(4)));
typedef uint32_t v4u __attribute__((ext_vector_type(4)));

struct ThinParams {
  GemmArgs g;
  int nchunks;
  int groups;        // 8-row groups of the packed weights
  int tiles;         // 16-row weight tiles
  uint32_t w_bytes;  // bytes of the packed weights (below 2^31)
  uint32_t a_bytes;  // bytes of the packed activations (kSrcPacked)
  const void* a_src; // kSrcCodes / kSrcHalf: [M][K]
  int src;
  int a_vec;         // 16-byte source loads allowed
  uint16_t* a_scale_out;
  int rows_off;      // byte offset of the converted rows in LDS
  int ones;          // byte offset of 32 bytes of ones, from the rows
};

// Items (tile, group) whose weight loads are in flight per wave.  The depth
// divides (or is divided by) the groups of a few tiles so that the ring's
// registers are named statically, and is kept small: the loop over tiles is
// unrolled until the ring's positions repeat, and a workgroup runs only a few
// tiles, so longer code costs more in instruction fetches than deeper loads give
// (MI355X, cold, 8 tokens, W4A4 22016 x 4096: 11.9, 12.3 and 13.8 us at 2, 3
// and 6 tiles).
template <int P, int G>
__host__ __device__ constexpr int depth() {
  return G >= 3 ? G : 2;
}
// Tiles per unrolled loop pass: the ring position of an item repeats after them.
template <int P, int G>
__host__ __device__ constexpr int unroll() {
  constexpr int d = depth<P, G>();
  for (int u = 1;; ++u)
    if (u * G % d == 0) return u;
}

__device__ __forceinline__ __amdgpu_buffer_rsrc_t rsrc_of(const void* base, uint32_t bytes) {
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(base), 0, bytes, 0x00020000);
}

constexpr uint32_t kNowhere = 0x80000000u;  // past the end of every buffer: reads zeros

// The E2M3 operand of one activation word: q <= 4 planes of u.  With s the
// top plane (set: positive) and t the lower bits, complemented where s is
// clear, the value 2u - (2^q - 1) is +-(2 t + 1), so its half is +-(t + 1/2)
// and each bit of its code is a function of t's bits.  (Uniform masks, not
// branches, on q.)
__device__ __forceinline__ void low_operand(const uint32_t u[4], int q, uint32_t out[6]) {
  uint32_t s = 0u;
#pragma unroll
  for (int i = 0; i < 4; ++i) s |= u[i] & (i == q - 1 ? ~0u : 0u);
  const uint32_t t0 = ~(u[0] ^ s) & (q > 1 ? ~0u : 0u);
  const uint32_t t1 = ~(u[1] ^ s) & (q > 2 ? ~0u : 0u);
  const uint32_t t2 = ~(u[2] ^ s) & (q > 3 ? ~0u : 0u);
  const uint32_t m0 = t2, m1 = (t2 & t0) | (~t2 & t1), m2 = (t2 & t1) | (~t2 & (~t1 | t0));
  const uint32_t e0 = t2 | (~t1 & t0), e1 = t2 | t1;
  const uint32_t code[6] = {m0, m1, m2, e0, e1, ~s};
  six_bit_fields(code, out);
}

// The int8 operand of one activation word: v = 2u - (2^q - 1) for q <= 7 (no
// carry leaves a byte: 2u + 128 - (2^q - 1) < 256), u - 128 for q = 8.
__device__ __forceinline__ void byte_operand(const uint32_t u[8], int q, uint32_t out[8]) {
  reassemble_word<8>(u, out);  // u - 128
  if (q < 8) {
    const uint32_t bias = (0x80u - ((1u << q) - 1u)) * 0x01010101u;
#pragma unroll
    for (int t = 0; t < 8; ++t) out[t] = (((out[t] ^ 0x80808080u) << 1) + bias) ^ 0x80808080u;
  }
}

template <int P, int C, int MT, int G, bool FUSED>
__global__ __launch_bounds__(kWaves* kWave, 2) void gemm_thin_kernel(ThinParams prm) {
  extern __shared__ __attribute__((aligned(16))) uint8_t lds[];
  constexpr int D = depth<P, G>();
  constexpr int U = unroll<P, G>();
  static_assert(!FUSED || (MT == 1 && C != kByte8), "unpacked rows: at most 8 tokens, the ones' row for R_w");
  constexpr int QV = C == kLow ? 4 : 8;               // activation planes, at most
  constexpr int AR = C == kLow && !FUSED ? 6 : 8;     // operand registers per word
  constexpr int kRedFloats = MT * kTileM * kRedStride;
  __shared__ uint32_t s_max[kWaves];
  __shared__ float s_rows[MT * kTileM];               // the rows' scales
  __shared__ int32_t s_part[kWaves][MT * kTileM];     // row sums of the activations' words per wave
  __shared__ int32_t s_ra[MT * kTileM];

  const GemmArgs& g = prm.g;
  const int NC = prm.nchunks, q = g.q;
  const int m0 = blockIdx.y * (MT * kTileM);       // this row of workgroups' tokens
  const int M = min(g.M - m0, MT * kTileM);
  const int tid = threadIdx.x, lane = tid % kWave;
  const int wave = __builtin_amdgcn_readfirstlane(tid / kWave);
  const int row = lane % 16, quarter = lane / 16;
  const int t_begin = (int)((int64_t)blockIdx.x * prm.tiles / gridDim.x);
  const int t_end = (int)((int64_t)(blockIdx.x + 1) * prm.tiles / gridDim.x);
  // LDS: partial sums of two tiles, the run's column scales, the converted rows
  uint32_t* const red = reinterpret_cast<uint32_t*>(lds);
  float* const s_ws = reinterpret_cast<float*>(lds + 2 * kWaves * kRedFloats * 4);
  uint8_t* const rows = lds + prm.rows_off;

  // ---- 1. the activations' loads leave first (loads complete in order)
  v4u araw[FUSED ? 1 : G * MT][QV];
  if constexpr (!FUSED) {
    const __amdgpu_buffer_rsrc_t a_rsrc = rsrc_of(g.a_packed, prm.a_bytes);
#pragma unroll
    for (int gm = 0; gm < G * MT; ++gm) {
      const int c = (wave + kWaves * (gm / MT)) * kGroupChunks + quarter;
      const int m = (gm % MT) * kTileM + row;
      // (the host keeps packed activations below 2^31 bytes)
      const uint32_t off = c < NC && m < M ? (uint32_t)plane_words(m0 + m, c, 0, NC, q) * 4u : kNowhere;
#pragma unroll
      for (int i = 0; i < QV; ++i)
        if (i < q) araw[gm][i] = __builtin_amdgcn_raw_buffer_load_b128(a_rsrc, off, i * kPlaneStride * 4, 0);
    }
  }
  // Unpacked rows: wpr waves share a row; lane l of sub-wave s takes the
  // 32-element words 64 (r wpr + s) + l, at most 2 G of them.
  const int wpr = M == 1 ? 8 : M == 2 ? 4 : M <= 4 ? 2 : 1;
  const int src_row = wave / wpr, sub = wave % wpr;
  const int words = NC * kWordsPerPlane;
  const int rounds = src_row < M ? (words - sub * kWave + wpr * kWave - 1) / (wpr * kWave) : 0;
  auto word_of = [&](int r) { return (r * wpr + sub) * kWave + lane; };
  using Half = std::integral_constant<bool, true>;
  using Code = std::integral_constant<bool, false>;
  const int src_bytes = prm.src == kSrcHalf ? 2 : 1;
  const uint8_t* const src_base =
      static_cast<const uint8_t*>(prm.a_src) + (int64_t)(src_row < M ? src_row : 0) * g.K * src_bytes;
  const __amdgpu_buffer_rsrc_t s_rsrc = rsrc_of(src_base, (uint32_t)g.K * src_bytes);
  auto load_word = [&](auto half, int r, uint32_t (&d)[2][8]) __attribute__((always_inline)) {
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      const int k0 = word_of(r) * 32 + h * rowcode::kLaneElems;
      if constexpr (half.value) {
        if (prm.a_vec) rowcode::HalfRow<true, 8>::load(s_rsrc, k0, d[h]);
        else rowcode::HalfRow<false, 8>::load_row(s_rsrc, src_base, g.K, k0, d[h]);
      } else {
        if (prm.a_vec) rowcode::CodeRow<true, 8>::load(s_rsrc, k0, d[h]);
        else rowcode::CodeRow<false, 8>::load_row(s_rsrc, src_base, g.K, k0, d[h]);
      }
    }
  };
  // all of them before the weights, held in registers (the operands that come
  // after them take as many)
  constexpr int kHeld = FUSED ? 2 * G : 1;
  uint32_t held[kHeld][2][8];
  if constexpr (FUSED) {
    if (prm.src == kSrcHalf) {
#pragma unroll
      for (int r = 0; r < kHeld; ++r)
        if (r < rounds) load_word(Half(), r, held[r]);
    } else {
#pragma unroll
      for (int r = 0; r < kHeld; ++r)
        if (r < rounds) load_word(Code(), r, held[r]);
    }
  }

  // ---- 2. the first D items of the weight stream
  const __amdgpu_buffer_rsrc_t w_rsrc = rsrc_of(g.w_packed, prm.w_bytes);
  v4u ring[D][P];
  const uint32_t row_bytes = (uint32_t)NC * P * kPlaneStride * 4u;  // bytes of a row group
  auto load_w = [&](v4u (&wv)[P], int tile, int gi) __attribute__((always_inline)) {
    const int c = (wave + kWaves * gi) * kGroupChunks + quarter;
    const int rg = tile * 2 + row / kRowGroup;
    const uint32_t off = c < NC && rg < prm.groups && tile < t_end
                             ? (uint32_t)rg * row_bytes + (uint32_t)(c * P * kPlaneStride + (row % kRowGroup) * kWordsPerPlane) * 4u
                             : kNowhere;
#pragma unroll
    for (int i = 0; i < P; ++i)
      wv[i] = __builtin_amdgcn_raw_buffer_load_b128(w_rsrc, off, i * kPlaneStride * 4, kNT);
  };
#pragma unroll
  for (int d = 0; d < D; ++d) load_w(ring[d], t_begin + d / G, d % G);

  // the run's column scales and (unless the source gives them) the rows': read
  // here, since a wait for a load issued between the weights' would wait for
  // all of those before it
  if (g.c_fp16 != nullptr) {
    if (prm.src != kSrcHalf && tid < M) s_rows[tid] = __half2float(g.a_scale[m0 + tid]);
    for (int i = tid; i < (t_end - t_begin) * kTileN; i += kWaves * kWave) {
      const int n = t_begin * kTileN + i;
      s_ws[i] = n < g.N ? __half2float(g.w_scale[n]) : 0.0f;
    }
  }

  // ---- 3. unpacked rows: the bipolar words u of the packer's arithmetic
  // (Sec. III-A conversion), one operand byte each, in LDS.  Word w of row m
  // is 32 bytes at (w M + m) 32, in the element order of the weight operand:
  // kLow, the 16 even then the 16 odd elements in the order of
  // six_bit_merge's fields; else the byte tree's.
  uint32_t a_op[G * MT][4][AR];
  if constexpr (FUSED) {
    uint32_t usum = 0u;
    // the operand's bytes from the words' bytes in element order
    auto order = [&](const uint32_t (&c)[8], uint32_t (&o)[8]) __attribute__((always_inline)) {
      if constexpr (C == kLow) {
        six_bit_order(c, o);
      } else {
        // o[t], byte j = element 8 j + t = byte t mod 4 of c[2 j + t / 4]
#pragma unroll
        for (int h = 0; h < 2; ++h)
#pragma unroll
          for (int tp = 0; tp < 4; tp += 2) {
            const uint32_t sel = (uint32_t)(tp | (4 + tp) << 8 | (tp + 1) << 16 | (5 + tp) << 24);
            const uint32_t lo = __builtin_amdgcn_perm(c[2 + h], c[h], sel);
            const uint32_t hi = __builtin_amdgcn_perm(c[6 + h], c[4 + h], sel);
            o[4 * h + tp] = __builtin_amdgcn_perm(hi, lo, 0x05040100u);
            o[4 * h + tp + 1] = __builtin_amdgcn_perm(hi, lo, 0x07060302u);
          }
      }
    };
    auto store_word = [&](int w, const uint32_t (&o)[8]) __attribute__((always_inline)) {
      if (w < words) {
        v4u* dst = reinterpret_cast<v4u*>(rows + (w * M + src_row) * 32);
        dst[0] = v4u{o[0], o[1], o[2], o[3]};
        dst[1] = v4u{o[4], o[5], o[6], o[7]};
      }
    };
    // words in element order (any width, any tail), then the operand's order
    auto convert = [&](auto half, const rowcode::Quantizer& qz, int r) __attribute__((always_inline)) {
      const int w = word_of(r), k0 = w * 32;
      uint32_t c[8], o[8];  // byte b of c[i]: u of element 4 i + b
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        if constexpr (half.value) qz.exact_words(held[r][h], c + 4 * h);
        else rowcode::code_words(held[r][h], q, c + 4 * h);
      }
#pragma unroll
      for (int t = 0; t < 8; ++t) {
        const int nv = g.K - (k0 + 4 * t);  // elements past K: u = 0, and the operand byte 0
        const uint32_t keep = nv >= 4 ? 0xFFFFFFFFu : (nv <= 0 ? 0u : ((1u << (8 * nv)) - 1u));
        c[t] &= keep;
        usum = __builtin_amdgcn_sad_u8(c[t], 0u, usum);
        if (C != kLow && q == 8) c[t] ^= 0x80808080u & keep;  // y = u - 128
      }
      order(c, o);
      store_word(w, o);
    };
    // whole words with the quantizer's short form, which gathers its results
    // straight into the operand's order
    auto convert_quick = [&](const rowcode::Quantizer& qz, int r) __attribute__((always_inline)) {
      uint32_t f[32], o[8], sum = 0u;
      if (C != kLow && q == 8) {
        qz.quick_bits<true>(held[r][0], f);
        qz.quick_bits<true>(held[r][1], f + 16);
      } else {
        qz.quick_bits<false>(held[r][0], f);
        qz.quick_bits<false>(held[r][1], f + 16);
      }
#pragma unroll
      for (int t = 0; t < 8; ++t) {
        constexpr int kField[16] = {0, 6, 12, 18, 24, 30, 4, 10, 16, 22, 28, 2, 8, 14, 20, 26};
        uint32_t e[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) e[i] = f[C == kLow ? kField[4 * (t % 4) + i] + t / 4 : 8 * i + t];
        o[t] = rowcode::Quantizer::gather(e);
        sum = __builtin_amdgcn_sad_u8(o[t], 0u, sum);
        if (C != kLow && q == 8) o[t] ^= 0x80808080u;  // y = u - 128
      }
      usum += word_of(r) < words ? sum : 0u;
      store_word(word_of(r), o);
    };
    rowcode::Quantizer qz{};
    if (prm.src == kSrcHalf) {
      rowcode::HalfExtremes ex;
#pragma unroll
      for (int r = 0; r < kHeld; ++r)
        if (r < rounds) {
          ex.fold(held[r][0]);
          ex.fold(held[r][1]);
        }
      const uint32_t top = rowcode::wave_max(ex.largest_magnitude());
      if (lane == 0) s_max[wave] = top;
      __syncthreads();
      uint32_t v = 0u;
      for (int w = 0; w < wpr; ++w) v = max(v, s_max[src_row * wpr + w]);
      qz.set(v, q);
      qz.quick = __builtin_amdgcn_readfirstlane(qz.quick);
      if (sub == 0 && lane == 0 && src_row < M) {
        s_rows[src_row] = __half2float(__ushort_as_half(qz.scale));
        if (prm.a_scale_out != nullptr && blockIdx.x == 0) prm.a_scale_out[src_row] = qz.scale;
      }
      if (qz.quick && g.K % kChunk == 0) {
#pragma unroll
        for (int r = 0; r < kHeld; ++r)
          if (r < rounds) convert_quick(qz, r);
      } else {
#pragma unroll
        for (int r = 0; r < kHeld; ++r)
          if (r < rounds) convert(Half(), qz, r);
      }
    } else {
#pragma unroll
      for (int r = 0; r < kHeld; ++r)
        if (r < rounds) convert(Code(), qz, r);
    }
    const uint32_t us = rowcode::wave_sum(usum);
    if (lane == 0) s_part[wave][0] = (int32_t)us;
    if (tid < 8) reinterpret_cast<uint32_t*>(rows + prm.ones)[tid] = 0x01010101u;
    __syncthreads();
    if (tid < M) {
      int32_t t = 0;
      for (int w = 0; w < wpr; ++w) t += s_part[tid * wpr + w][0];
      s_ra[tid] = t - (C != kLow && q == 8 ? 128 * g.K : 0);  // sum of y
    }
    // ---- 4. the operands: row 15 holds ones, so that its products are the
    // weights' own sums.  kLow: an FP8 operand's lane quarter b meets k
    // 16 b .. 16 b + 15 and 64 + 16 b .. in its two halves, an FP6 operand's
    // 32 b .. 32 b + 31, so bytes 0..15 belong to weight quarter b / 2 and
    // bytes 16..31 to quarter 2 + b / 2, fields 16 (b mod 2) on.
    // (Row 15's lanes read 32 bytes of ones with a stride of 0; a chunk past
    // the last meets zero weights, or at p = 8 must be zero itself.)
    const uint8_t* const a_base = row == 15 ? rows + prm.ones : rows + min(row, M - 1) * 32;
    const int a_step = row == 15 ? 0 : M * 32;
#pragma unroll
    for (int gi = 0; gi < G; ++gi)
#pragma unroll
      for (int j = 0; j < 4; ++j)
#pragma unroll
        for (int h = 0; h < 2; ++h) {
          const int c = (wave + kWaves * gi) * kGroupChunks + (C == kLow ? 2 * h + quarter / 2 : quarter);
          const int part = C == kLow ? quarter % 2 : h;
          v4u v = *reinterpret_cast<const v4u*>(a_base + (min(c, NC - 1) * 4 + j) * a_step + part * 16);
#pragma unroll
          for (int t = 0; t < 4; ++t) a_op[gi][j][4 * h + t] = P < 8 || c < NC || row == 15 ? v[t] : 0u;
        }
  } else {
    // ---- 4. packed rows: the operands and row sums from the planes
#pragma unroll
    for (int gm = 0; gm < G * MT; ++gm) {
#pragma unroll
      for (int i = 0; i < QV; ++i)
        if (i >= q) araw[gm][i] = v4u{0u, 0u, 0u, 0u};
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        uint32_t u[QV];
#pragma unroll
        for (int i = 0; i < QV; ++i) u[i] = araw[gm][i][j];
        if constexpr (C == kLow) low_operand(u, q, a_op[gm][j]);
        else byte_operand(u, q, a_op[gm][j]);
      }
    }
#pragma unroll
    for (int mt = 0; mt < MT; ++mt) {
      uint32_t t = 0u;
#pragma unroll
      for (int gi = 0; gi < G; ++gi)
#pragma unroll
        for (int i = 0; i < QV; ++i) {
          const v4u v = araw[gi * MT + mt][i];
          t += (__builtin_popcount(v[0]) + __builtin_popcount(v[1]) + __builtin_popcount(v[2]) + __builtin_popcount(v[3])) << i;
        }
      t += __shfl_xor(t, 16);
      t += __shfl_xor(t, 32);
      if (quarter == 0) s_part[wave][mt * kTileM + row] = (int32_t)t;
    }
    __syncthreads();
    if (tid < MT * kTileM) {
      int32_t t = 0;
#pragma unroll
      for (int w = 0; w < kWaves; ++w) t += s_part[w][tid];
      s_ra[tid] = 2 * t - ((1 << q) - 1) * g.K;  // R_a, the sum of 2u - (2^q - 1)
    }
  }
  // (s_ra and s_rows are read after the first tile's barrier)

  // ---- 5. the tiles
  // Unpacked rows: v = 2y + c on both sides, so C = 4 D + 2 c_w sum y_a +
  // 2 c_a sum y_w + c_a c_w K (D has no padding: its activation bytes are 0).
  // Packed rows: C = 2 (D - pad) + c_w R_a, pad being the products of the
  // padding bytes over every element the groups cover past K; kByte8 below.
  constexpr int32_t cw = P == 8 ? 1 : 1 - (1 << P);
  const int32_t ca = C != kLow && q == 8 ? 1 : 1 - (1 << q);
  const int32_t npad = kWaves * G * kGroupChunks * kChunk - g.K;
  constexpr int32_t pad_w = C != kLow && P == 8 ? -128 : 0;
  const int32_t pad = npad * pad_w * (q == 8 ? -128 : 1 - (1 << q));

  auto finish = [&](const v4f (&accf)[MT], const v4i (&acci)[MT], const v4i& ones, int tile) __attribute__((always_inline)) {
    uint32_t* const buf = red + (tile & 1) * kWaves * kRedFloats;
#pragma unroll
    for (int mt = 0; mt < MT; ++mt) {
      v4i v;
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        // sum of u_a u_w (codes u 2^-9 and u 2^-3), or of v_a u_w (v / 2 and u / 8)
        if constexpr (C == kLow) v[r] = (int32_t)(accf[mt][r] * (FUSED ? 4096.0f : 16.0f));
        else if constexpr (C == kByte8) v[r] = 2 * acci[mt][r] + ones[r];
        else v[r] = acci[mt][r];
      }
      // D[n = 4 (lane / 16) + r][m = lane mod 16]
      *reinterpret_cast<v4i*>(buf + wave * kRedFloats + (mt * kTileM + row) * kRedStride + 4 * quarter) = v;
    }
    __syncthreads();
    const int nl = tid % kTileN, n = tile * kTileN + nl;
    for (int m = tid / kTileN; m < M; m += kWaves * kWave / kTileN) {
      uint32_t d = 0u;
#pragma unroll
      for (int w = 0; w < kWaves; ++w) d += buf[w * kRedFloats + m * kRedStride + nl];
      uint32_t cv;
      if constexpr (FUSED) {
        uint32_t wn = 0u;
#pragma unroll
        for (int w = 0; w < kWaves; ++w) wn += buf[w * kRedFloats + 15 * kRedStride + nl];
        wn -= (uint32_t)(npad * pad_w);
        cv = 4u * d + (uint32_t)(2 * cw) * (uint32_t)s_ra[m] + (uint32_t)(2 * ca) * wn +
             (uint32_t)(ca * cw) * (uint32_t)g.K;
      } else if constexpr (C == kByte8) {
        // d = 2 D + sum y_w per wave, and v_a = 2 y_a + 1:
        // C = 4 (D - pad) + 2 c_w sum y_a + sum (2 y_w + c_w), 2 sum y_a = R_a - K
        cv = 2u * d - 4u * (uint32_t)pad - 2u * (uint32_t)(npad * pad_w) + (uint32_t)cw * (uint32_t)s_ra[m];
      } else {
        cv = 2u * (d - (uint32_t)pad) + (uint32_t)cw * (uint32_t)s_ra[m];
      }
      if (n < g.N) {
        const int64_t o = (int64_t)(m0 + m) * g.N + n;
        const int32_t c = (int32_t)cv;
        if (g.c_int32) g.c_int32[o] = c;
        if (g.c_fp16) {
          float f;
          if (g.a_zero) {
            const float sw = __half2float(g.w_scale[n]), zw = __half2float(g.w_zero[n]);
            f = affine_value(c, s_rows[m], sw, zw, (float)g.a_rowsum[m0 + m], __half2float(g.a_zero[m0 + m]),
                             sw * (float)g.w_rowsum[n] + (float)g.K * zw);
          } else {
            f = (float)c * s_rows[m];
            f = f * s_ws[(tile - t_begin) * kTileN + nl];
          }
          g.c_fp16[o] = __float2half_rn(f);
        }
      }
    }
  };

  for (int t0 = t_begin; t0 < t_end; t0 += U) {
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int tile = t0 + u;
      if (tile >= t_end) break;  // uniform
      v4f accf[MT];
      v4i acci[MT], ones = {0, 0, 0, 0};
#pragma unroll
      for (int mt = 0; mt < MT; ++mt) {
        accf[mt] = v4f{0.0f, 0.0f, 0.0f, 0.0f};
        acci[mt] = v4i{0, 0, 0, 0};
      }
#pragma unroll
      for (int gi = 0; gi < G; ++gi) {
        constexpr int kSteps = 4;
        v4u(&wv)[P] = ring[(u * G + gi) % D];
#pragma unroll
        for (int j = 0; j < kSteps; ++j) {
          uint32_t pw[P];
#pragma unroll
          for (int i = 0; i < P; ++i) pw[i] = wv[i][j];
          if constexpr (C == kLow) {
            uint32_t o[6];
            six_bit_word<P>(pw, o);
            const v8i wa = {(int)o[0], (int)o[1], (int)o[2], (int)o[3], (int)o[4], (int)o[5], 0, 0};
#pragma unroll
            for (int mt = 0; mt < MT; ++mt) {
              const uint32_t* a = a_op[gi * MT + mt][j];
              // E2M3 weights (format code 2), no scales
              if constexpr (FUSED) {  // E4M3 activations (code 0)
                const v8i ab = {(int)a[0], (int)a[1], (int)a[2], (int)a[3], (int)a[4], (int)a[5], (int)a[AR - 2], (int)a[AR - 1]};
                accf[mt] = __builtin_amdgcn_mfma_scale_f32_16x16x128_f8f6f4(wa, ab, accf[mt], 2, 0, 0, 0, 0, 0);
              } else {  // E2M3 activations
                const v8i ab = {(int)a[0], (int)a[1], (int)a[2], (int)a[3], (int)a[4], (int)a[5], 0, 0};
                accf[mt] = __builtin_amdgcn_mfma_scale_f32_16x16x128_f8f6f4(wa, ab, accf[mt], 2, 2, 0, 0, 0, 0);
              }
            }
          } else {
            uint32_t o[8];
            reassemble_word<P>(pw, o);
            const v4i w0 = {(int)o[0], (int)o[1], (int)o[2], (int)o[3]};
            const v4i w1 = {(int)o[4], (int)o[5], (int)o[6], (int)o[7]};
#pragma unroll
            for (int mt = 0; mt < MT; ++mt) {
              const uint32_t* a = a_op[gi * MT + mt][j];
              const v4i a0 = {(int)a[0], (int)a[1], (int)a[2], (int)a[3]};
              const v4i a1 = {(int)a[4], (int)a[5], (int)a[6], (int)a[7]};
              acci[mt] = __builtin_amdgcn_mfma_i32_16x16x64_i8(w0, a0, acci[mt], 0, 0, 0);
              acci[mt] = __builtin_amdgcn_mfma_i32_16x16x64_i8(w1, a1, acci[mt], 0, 0, 0);
            }
            if constexpr (C == kByte8) {
              const v4i one = {0x01010101, 0x01010101, 0x01010101, 0x01010101};
              ones = __builtin_amdgcn_mfma_i32_16x16x64_i8(w0, one, ones, 0, 0, 0);
              ones = __builtin_amdgcn_mfma_i32_16x16x64_i8(w1, one, ones, 0, 0, 0);
            }
          }
        }
        load_w(wv, t0 + (u * G + gi + D) / G, (u * G + gi + D) % G);
      }
      finish(accf, acci, ones, tile);
    }
  }
}

struct ThinLaunch {
  int cls, mt, gk;     // operand class, 16-token tiles, K groups per wave
  int grid, blocks;    // workgroups along N, rows of workgroups along M
  size_t lds_bytes;
  int run, rows_off;
};

// The shapes built: those whose operands, ring and sums fit the 256 registers
// of a wave (two waves per SIMD); gk = K groups per wave.
inline bool shape_built(int p, int cls, int mt, int gk) {
  if (cls == kLow) return (mt == 1 && gk <= 4) || (mt == 2 && gk <= 2) || (mt == 4 && gk == 1);
  return (mt == 1 && gk <= (p <= 4 ? 3 : 2)) || (mt == 2 && gk == 1);
}

template <int P, int C, int MT, int G, bool FUSED>
inline hipError_t launch_one(const ThinParams& prm, const ThinLaunch& L, hipStream_t s) {
  auto kern = gemm_thin_kernel<P, C, MT, G, FUSED>;
  if (L.lds_bytes > 48 * 1024) {
    const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(kern),
                                             hipFuncAttributeMaxDynamicSharedMemorySize, (int)L.lds_bytes);
    if (e != hipSuccess) return e;
  }
  return launch_kernel(kern, dim3(L.grid, L.blocks), dim3(kWaves * kWave), L.lds_bytes, s, prm);
}

template <int P, int C, bool FUSED>
inline hipError_t launch_cls(const ThinParams& prm, const ThinLaunch& L, hipStream_t s) {
  if (L.mt == 1 && L.gk == 1) return launch_one<P, C, 1, 1, FUSED>(prm, L, s);
  if (L.mt == 1 && L.gk == 2) return launch_one<P, C, 1, 2, FUSED>(prm, L, s);
  if constexpr (P <= 4) {
    if (L.mt == 1 && L.gk == 3) return launch_one<P, C, 1, 3, FUSED>(prm, L, s);
  }
  if constexpr (C == kLow) {
    if (L.mt == 1 && L.gk == 4) return launch_one<P, C, 1, 4, FUSED>(prm, L, s);
  }
  if constexpr (!FUSED) {
    if (L.mt == 2 && L.gk == 1) return launch_one<P, C, 2, 1, false>(prm, L, s);
    if constexpr (C == kLow) {
      if (L.mt == 2 && L.gk == 2) return launch_one<P, C, 2, 2, false>(prm, L, s);
      if (L.mt == 4 && L.gk == 1) return launch_one<P, C, 4, 1, false>(prm, L, s);
    }
  }
  return hipErrorInvalidValue;
}

// Launch for weight bits P; instantiated once per width in gemm_thin_inst.hip.
template <int P>
hipError_t launch_for_p(const ThinParams& prm, const ThinLaunch& L, hipStream_t s);

}  // namespace thin
}  // namespace apt

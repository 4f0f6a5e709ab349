// gemm_direct.h - the reassembled MFMA GEMM for operands of at most 4 bits, with
// the weights rebuilt straight into operand registers (APT-LLM, arXiv
// 2508.19087, Sec. III-B), for gfx950.  The int8 MFMA route's 256 x 128 shape
// with 4 x 1 waves runs it where p, q <= 4 and K (2^p - 1)(2^q - 1) < 2^24 (exact
// fp32 sums), on tiles of 128 x 256.
//
// Operands are the words u themselves as six-bit E2M3 codes, u / 8 (six_bit_word
// in reassemble.h), on v_mfma_f32_32x32x64_f8f6f4: twice the int8 rate, fewer
// rebuild instructions and three quarters of the activation bytes.  The sum is
// gemm_int8.h's D = sum of u_a u_w and the epilogue its affine correction.
//
// gemm_int8.h rebuilds each weight tile into LDS, where every wave reads all of
// it back, and each wave loads its own activation fragments past LDS; with the
// matrix cores twice as fast that path would be all there is.  Here the roles
// are swapped.  Each of the 4 waves owns 64 of the tile's 256 columns for all
// 128 rows: it loads the packed planes of its own columns (16 bytes per lane and
// plane: the four words of one row and chunk, lanes 0..31 the first chunk of a
// pair, lanes 32..63 the second) and rebuilds word j of both chunks in registers
// as the MFMA operand of 4 row blocks.  The activation fragments of a chunk
// pair go to LDS by direct loads (no registers), double buffered, and every
// wave reads them.  One barrier per chunk pair; two workgroups per compute unit
// fill each other's waits.
//
// What bounds it (MI355X, 2048 x 8192, chunk pair of two workgroups on a compute
// unit, us): 1.32 at W2A2 and 1.92 at W4A4, against 1.0 of MFMA issue at 2 GHz
// and 3.1-3.6 for the int8 shape.  Without the weight loads 1.50 at W4A4, without
// the MFMAs 1.12, without the rebuild 1.88, without the activation loads 1.84:
// the weight loads' returns to registers hold up the MFMAs.  A burst of all the
// loads at the pair's start cost 2.28 (they now leave one per slot), the
// fragment reads one slot ahead instead of at their use took it from 2.04 to
// 1.99, and two slots ahead measured the same.
//
// The k order inside a chunk pair is word j of chunk c from lane half 0 with
// word j of chunk c + 1 from lane half 1, on both sides.
#pragma once

#include "gemm_int8.h"

namespace apt {
namespace direct {

using int8::Int8Params;
using int8::keep_here;
using int8::make_rsrc;
using int8::store_block;
using int8::v16f;
using int8::v16i;
using int8::v2i;
using int8::v4f;
using int8::v4i;
using int8::v4u;
using int8::v8i;

constexpr int kWave = 64, kWaves = 4;
constexpr int kBM = 128, kBN = 256;
constexpr int kMF = kBM / 32, kNF = kBN / kWaves / 32;  // 32 x 32 blocks per wave
constexpr int kPairWords = 8;                           // words of a chunk pair

constexpr int kFrag = kSixBytes;                  // LDS bytes of a fragment (32 rows of one word)

template <int P>
__global__ __launch_bounds__(kWaves* kWave, 2) void gemm_direct_kernel(Int8Params prm) {
  static_assert(P <= 4, "six-bit codes hold words of at most 4 bits");
  constexpr int kStage = kMF * kPairWords * kFrag;
  constexpr int kParts = kPairWords * kFrag / 1024;  // direct loads (1 KB each) per wave and stage
  __shared__ __attribute__((aligned(16))) uint8_t stage0[kStage];
  __shared__ __attribute__((aligned(16))) uint8_t stage1[kStage];

  const GemmArgs& g = prm.g;
  const int NC = prm.nchunks, pairs = (NC + 1) / 2;
  const int tid = threadIdx.x, lane = tid % kWave;
  const int wave = __builtin_amdgcn_readfirstlane(tid / kWave);
  const int r = lane % 32, h = lane / 32;

  // Tile of this workgroup: workgroups are dealt round-robin to the 8 XCDs,
  // each of which takes a contiguous run of tiles in panels of 8 tile rows,
  // walked column by column, so that the tiles in flight on an XCD share both
  // operands in its L2.
  const int tiles_m = prm.tiles / prm.tiles_n;
  int t;
  {
    const int x = blockIdx.x % 8, i = blockIdx.x / 8;
    t = x * (prm.tiles / 8) + min(x, prm.tiles % 8) + i;
  }
  const int panel = t / (8 * prm.tiles_n), rest = t % (8 * prm.tiles_n);
  const int ph = min(8, tiles_m - panel * 8);
  const int m0 = (panel * 8 + rest % ph) * kBM, n0 = rest / ph * kBN;

  // ---- operand sources
  const __amdgpu_buffer_rsrc_t w_rsrc = make_rsrc(g.w_packed, prm.w_bytes);
  const __amdgpu_buffer_rsrc_t a_rsrc = make_rsrc(prm.a_frag, prm.a_bytes);
  uint32_t w_off[kNF];
#pragma unroll
  for (int b = 0; b < kNF; ++b)  // (rows past the edge: the last row, their outputs are not stored)
    w_off[b] = (uint32_t)plane_words(min(n0 + wave * 64 + b * 32 + r, g.N - 1), h, 0, NC, P) * 4u;
  // (the second chunk of the last pair when NC is odd, whatever it reads, meets
  // all-zero activation fragments; past the buffer's end loads give zeros)
  auto load_w1 = [&](v4u (&raw)[kNF][P], int pair, int x) __attribute__((always_inline)) {
    const uint32_t so = (uint32_t)pair * (uint32_t)(2 * P * kPlaneStride * 4);
    raw[x / P][x % P] = __builtin_amdgcn_raw_buffer_load_b128(w_rsrc, w_off[x / P] + x % P * kPlaneStride * 4, so, 0);
  };
  auto load_w = [&](v4u (&raw)[kNF][P], int pair) __attribute__((always_inline)) {
#pragma unroll
    for (int x = 0; x < kNF * P; ++x) load_w1(raw, pair, x);
  };
  // wave w moves row block w of the tile: its 8 words of the pair are contiguous
  const uint32_t a_base = (uint32_t)min(m0 / 32 + wave, prm.mblocks - 1) * (uint32_t)prm.nsteps * (uint32_t)kFrag;
  auto load_a1 = [&](uint8_t* stage, int pair, int k) __attribute__((always_inline)) {
    const uint32_t so = a_base + (uint32_t)pair * (uint32_t)(kPairWords * kFrag);
    __builtin_amdgcn_raw_ptr_buffer_load_lds(
        a_rsrc, (__attribute__((address_space(3))) void*)(stage + (wave * kParts + k) * 1024), 16, lane * 16,
        so + k * 1024, 0, 0);
  };
  auto load_a = [&](uint8_t* stage, int pair) __attribute__((always_inline)) {
#pragma unroll
    for (int k = 0; k < kParts; ++k) load_a1(stage, pair, k);
  };

  v16f acc[kNF][kMF];
#pragma unroll
  for (int b = 0; b < kNF; ++b)
#pragma unroll
    for (int a = 0; a < kMF; ++a)
#pragma unroll
      for (int v = 0; v < 16; ++v) acc[b][a][v] = 0.0f;

  // One chunk pair from `cur`; the next pair's loads leave first.
  auto step = [&](uint8_t* cur, uint8_t* nxt, v4u (&raw)[kNF][P], v4u (&raw_nxt)[kNF][P], int pair) __attribute__((always_inline)) {
    const int next = min(pair + 1, pairs - 1);
    // this wave's direct loads into `cur` and its reads of `nxt` are done
    // (vmcnt 0, lgkmcnt 0), then every wave's
    __builtin_amdgcn_s_waitcnt(0x0070);
    __builtin_amdgcn_s_barrier();
    // the next pair's loads leave one or two at a time behind the MFMAs of each
    // row block (a burst of them holds the wave at its issue), all in the first
    // three quarters of the pair
    constexpr int kLoads = kParts + kNF * P, kSlots = 3 * kMF;
    const uint8_t* const lane_a = cur + h * 4 * kFrag + r * 16;
    const uint8_t* const lane_a8 = cur + h * 4 * kFrag + 512 + r * 8;
    // Slot (j, a): the MFMAs of word j and row block a.  Behind them, the
    // fragment of the next slot is read, a quarter of the next word's rebuild
    // is done and the slot's share of the loads is issued.
    uint32_t af[2][6], w[2][kNF][6];
    auto read_a = [&](int s, uint32_t (&f)[6]) __attribute__((always_inline)) {
      const int off = (s % kMF * kPairWords + s / kMF) * kFrag;
      const v4i lo = *reinterpret_cast<const v4i*>(lane_a + off);
      const v2i hi = *reinterpret_cast<const v2i*>(lane_a8 + off);
#pragma unroll
      for (int i = 0; i < 4; ++i) f[i] = (uint32_t)lo[i];
      f[4] = (uint32_t)hi[0];
      f[5] = (uint32_t)hi[1];
    };
    // half x of word j of column block b
    auto rebuild = [&](int j, int b, int x, uint32_t (&o)[6]) __attribute__((always_inline)) {
      uint32_t pw[P];
#pragma unroll
      for (int i = 0; i < P; ++i) pw[i] = raw[b][i][j];
      six_bit_half<P>(pw, x, o + 3 * x);
    };
    read_a(0, af[0]);
#pragma unroll
    for (int b = 0; b < kNF; ++b)
#pragma unroll
      for (int x = 0; x < 2; ++x) rebuild(0, b, x, w[0][b]);
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int s = 0; s < 4 * kMF; ++s) {
      const int j = s / kMF, a = s % kMF;
      if (s + 1 < 4 * kMF) read_a(s + 1, af[(s + 1) % 2]);
      if (j < 3) rebuild(j + 1, a / 2, a % 2, w[(j + 1) % 2][a / 2]);
      const uint32_t* const f = af[s % 2];
      const v8i ab = {(int)f[0], (int)f[1], (int)f[2], (int)f[3], (int)f[4], (int)f[5], 0, 0};
#pragma unroll
      for (int b = 0; b < kNF; ++b) {
        const uint32_t* const o = w[j % 2][b];
        const v8i wa = {(int)o[0], (int)o[1], (int)o[2], (int)o[3], (int)o[4], (int)o[5], 0, 0};
        // E2M3 on both sides (format code 2), no scales
        acc[b][a] = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(wa, ab, acc[b][a], 2, 2, 0, 0, 0, 0);
      }
#pragma unroll
      for (int x = 0; x < kLoads; ++x)
        if (x * kSlots / kLoads == s) {
          if (x < kNF * P) load_w1(raw_nxt, next, x);
          else load_a1(nxt, next, x - kNF * P);
        }
      __builtin_amdgcn_sched_barrier(0);
    }
    // (an empty use of every accumulator: the pair's MFMAs stay in it)
#pragma unroll
    for (int b = 0; b < kNF; ++b)
#pragma unroll
      for (int a = 0; a < kMF; ++a) keep_here(__builtin_bit_cast(v16i, acc[b][a]));
    __builtin_amdgcn_sched_barrier(0);  // nothing of the next pair waits for its loads in this one
  };

  {
    v4u raw0[kNF][P], raw1[kNF][P];
    load_a(stage0, 0);
    load_w(raw0, 0);
    int pair = 0;
    for (; pair + 1 < pairs; pair += 2) {
      step(stage0, stage1, raw0, raw1, pair);
      step(stage1, stage0, raw1, raw0, pair + 1);
    }
    if (pair < pairs) step(stage0, stage1, raw0, raw1, pair);
  }

  // ---- epilogue (gemm_int8.h's): column terms c_a R_w[n] and row terms c_w R_a[m]
  // - const, and the scales, in stage1; each 32 x 32 block goes through the
  // wave's slot in stage0 and comes back as whole 128-byte rows
  constexpr int kEpiStride = 32 * 4 + 16;
  static_assert(kWaves * 32 * kEpiStride <= kStage && (kBN + kBM) * 16 <= kStage, "the stages hold the epilogue");
  const int q = g.q;
  const uint32_t ca = (uint32_t)(1 - (1 << q)), cw = (uint32_t)int8::offset_of(P);
  const uint32_t const_term = ca * cw * (uint32_t)g.K;  // (padding words are 0 and add nothing)
  const bool fp16 = g.c_fp16 != nullptr, affine = g.a_zero != nullptr, stream = prm.stream_out != 0;
  uint32_t* const s_term = reinterpret_cast<uint32_t*>(stage1);       // columns, then rows
  float* const s_scale = reinterpret_cast<float*>(s_term + kBN + kBM);
  float* const s_zero = s_scale + kBN + kBM;                          // z_w[n] | float(R_a[m])
  float* const s_cross = s_zero + kBN + kBM;                          // s_w R_w[n] + K z_w[n] | z_a[m]
  uint8_t* const slot = stage0 + wave * 32 * kEpiStride;
  __builtin_amdgcn_s_waitcnt(0x0070);  // the last (unused) direct loads have landed
  __builtin_amdgcn_s_barrier();
  for (int i = tid; i < kBN + kBM; i += kWaves * kWave) {
    const bool col = i < kBN;
    const int n = min(n0 + i, g.N - 1), m = min(m0 + i - kBN, g.M - 1);
    const uint32_t rs = (uint32_t)(col ? g.w_rowsum[n] : g.a_rowsum[m]);
    s_term[i] = col ? ca * rs : cw * rs - const_term;
    if (fp16) {
      const float s = __half2float(col ? g.w_scale[n] : g.a_scale[m]);
      s_scale[i] = s;
      if (affine) {
        const float z = __half2float(col ? g.w_zero[n] : g.a_zero[m]);
        s_zero[i] = col ? z : (float)(int32_t)rs;
        s_cross[i] = col ? s * (float)(int32_t)rs + (float)g.K * z : z;
      }
    }
  }
  __syncthreads();
  if (fp16 && g.c_int32 == nullptr && g.N % 8 == 0 && (reinterpret_cast<uintptr_t>(g.c_fp16) & 15) == 0) {
    // fp16 alone: the values are finished where the MFMA leaves them and go
    // through the slot as halves, so that a wave's 64 columns come back as whole
    // 128-byte rows (as 32-column blocks they leave as half lines: W2A2 1024 x
    // 11008 x 4096 4 us more)
    constexpr int kHalfStride = 64 * 2 + 16;
#pragma unroll
    for (int a = 0; a < kMF; ++a) {
      if (m0 + a * 32 >= g.M || n0 + wave * 64 >= g.N) continue;  // uniform: no output here
      const int ml = a * 32 + r;
      const uint32_t at = s_term[kBN + ml];
      const float sa = s_scale[kBN + ml];
      const float ra = affine ? s_zero[kBN + ml] : 0.0f, za = affine ? s_cross[kBN + ml] : 0.0f;
#pragma unroll
      for (int b = 0; b < kNF; ++b) {
        const v16i d = __builtin_convertvector(acc[b][a] * 64.0f, v16i);  // sum of u_a u_w
#pragma unroll
        for (int gi = 0; gi < 4; ++gi) {
          const int nl = b * 32 + gi * 8 + h * 4;
          const v4u wt = *reinterpret_cast<const v4u*>(s_term + wave * 64 + nl);
          const v4f ws = *reinterpret_cast<const v4f*>(s_scale + wave * 64 + nl);
          float f[4];
          if (affine) {
            const v4f zw = *reinterpret_cast<const v4f*>(s_zero + wave * 64 + nl);
            const v4f col = *reinterpret_cast<const v4f*>(s_cross + wave * 64 + nl);
#pragma unroll
            for (int j = 0; j < 4; ++j)
              f[j] = affine_value((int32_t)(4u * (uint32_t)d[gi * 4 + j] + at + wt[j]), sa, ws[j], zw[j], ra, za, col[j]);
          } else {
#pragma unroll
            for (int j = 0; j < 4; ++j)
              f[j] = (float)(int32_t)(4u * (uint32_t)d[gi * 4 + j] + at + wt[j]) * sa * ws[j];
          }
          uint32_t hb[2];
#pragma unroll
          for (int j = 0; j < 4; j += 2)
            hb[j / 2] = __half_as_ushort(__float2half_rn(f[j])) |
                        ((uint32_t)__half_as_ushort(__float2half_rn(f[j + 1])) << 16);
          *reinterpret_cast<uint2*>(slot + r * kHalfStride + nl * 2) = make_uint2(hb[0], hb[1]);
        }
      }
      __builtin_amdgcn_s_waitcnt(0xc07f);  // this wave's LDS writes are done
      __builtin_amdgcn_wave_barrier();
      const int ncol = n0 + wave * 64 + lane % 8 * 8;
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const int row = i * 8 + lane / 8, m = m0 + a * 32 + row;
        const v4i v = *reinterpret_cast<const v4i*>(slot + row * kHalfStride + lane % 8 * 16);
        if (m < g.M && ncol < g.N)
          __builtin_nontemporal_store(v, reinterpret_cast<v4i*>(g.c_fp16 + (int64_t)m * g.N + ncol));
      }
      __builtin_amdgcn_s_waitcnt(0xc07f);  // reads done before the slot is rewritten
      __builtin_amdgcn_wave_barrier();
    }
    return;
  }
  const int er = lane / 8, ec = (lane % 8) * 4;
#pragma unroll
  for (int a = 0; a < kMF; ++a) {
#pragma unroll
    for (int b = 0; b < kNF; ++b) {
      if (m0 + a * 32 >= g.M || n0 + wave * 64 + b * 32 >= g.N) continue;  // uniform: no output here
      const v16i d = __builtin_convertvector(acc[b][a] * 64.0f, v16i);  // sum of u_a u_w
#pragma unroll
      for (int gi = 0; gi < 4; ++gi)
        *reinterpret_cast<v4i*>(slot + r * kEpiStride + (gi * 8 + h * 4) * 4) =
            v4i{d[gi * 4], d[gi * 4 + 1], d[gi * 4 + 2], d[gi * 4 + 3]};
      __builtin_amdgcn_s_waitcnt(0xc07f);  // this wave's LDS writes are done
      __builtin_amdgcn_wave_barrier();
      const int nl = wave * 64 + b * 32 + ec, ncol = n0 + nl;
      const v4u wt = *reinterpret_cast<const v4u*>(s_term + nl);
      const v4f ws = *reinterpret_cast<const v4f*>(s_scale + nl);
      v4i dv[4];
      uint32_t atv[4];
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        dv[i] = *reinterpret_cast<const v4i*>(slot + (er + 8 * i) * kEpiStride + ec * 4);
        atv[i] = s_term[kBN + a * 32 + er + 8 * i];
      }
#pragma unroll
      for (int i = 0; i < 4; ++i) keep_here(dv[i], atv[i]);
      int32_t cv[4][4];
#pragma unroll
      for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int j = 0; j < 4; ++j) cv[i][j] = (int32_t)(4u * (uint32_t)dv[i][j] + atv[i] + wt[j]);
      const int row0 = a * 32 + er;
      const bool inside = m0 + a * 32 + 32 <= g.M && n0 + wave * 64 + b * 32 + 32 <= g.N;
      if (g.c_int32 != nullptr) store_block(g, cv, m0 + row0, ncol, inside, stream);
      if (fp16) {
        uint32_t hb[4][2];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const int ml = row0 + 8 * i;
          const float sa = s_scale[kBN + ml];
          float f[4];
          if (affine) {
            const v4f zw = *reinterpret_cast<const v4f*>(s_zero + nl);
            const v4f col = *reinterpret_cast<const v4f*>(s_cross + nl);
            const float ra = s_zero[kBN + ml], za = s_cross[kBN + ml];
#pragma unroll
            for (int j = 0; j < 4; ++j) f[j] = affine_value(cv[i][j], sa, ws[j], zw[j], ra, za, col[j]);
          } else {
#pragma unroll
            for (int j = 0; j < 4; ++j) f[j] = (float)cv[i][j] * sa * ws[j];
          }
#pragma unroll
          for (int j = 0; j < 4; j += 2)
            hb[i][j / 2] = __half_as_ushort(__float2half_rn(f[j])) |
                           ((uint32_t)__half_as_ushort(__float2half_rn(f[j + 1])) << 16);
        }
        store_block(g, hb, m0 + row0, ncol, inside);
      }
      __builtin_amdgcn_s_waitcnt(0xc07f);  // reads done before the slot is rewritten
      __builtin_amdgcn_wave_barrier();
    }
  }
}

// Launch for weight bits P <= 4; instantiated once per width in
// gemm_direct_inst.hip.
template <int P>
hipError_t launch_for_p(const Int8Params& prm, hipStream_t s);

}  // namespace direct
}  // namespace apt

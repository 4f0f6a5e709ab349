// gemm_thin.hip - the rule, launch geometry and dispatch of the few-token GEMM
// (gemm_thin.h).
#include <algorithm>
#include <cmath>

#include "gemm_thin.h"

namespace apt {

namespace {

using thin::ThinLaunch;
using thin::ThinParams;

// LDS of a workgroup, at most (the kernel's static arrays take 2.4 KB more of the 160 KB).
constexpr size_t kMaxLds = 150 * 1024;

constexpr int kMaxTokens = 512;

// Whether the kernel takes (M, N, K, p, q) from source src, and its launch.
bool plan(int M, int N, int K, int p, int q, int src, ThinLaunch* L) {
  if (M > (src == thin::kSrcPacked ? kMaxTokens : APT_DECODE_MAX_M)) return false;
  const int nc = num_chunks(K);
  // 32-bit offsets below kNowhere
  if (apt_packed_bytes(N, K, p) >= thin::kNowhere || apt_packed_bytes(M, K, q) >= thin::kNowhere) return false;
  L->cls = six_bit_ok(K, p, q) ? thin::kLow : q == 8 ? thin::kByte8 : thin::kByte;
  const int kgroups = (nc + thin::kGroupChunks - 1) / thin::kGroupChunks;
  L->gk = (kgroups + thin::kWaves - 1) / thin::kWaves;
  // the most tokens per workgroup that its registers hold, no more than needed
  L->mt = M <= 16 ? 1 : M <= 32 ? 2 : 4;
  while (L->mt > 1 && !thin::shape_built(p, L->cls, L->mt, L->gk)) L->mt /= 2;
  if (!thin::shape_built(p, L->cls, L->mt, L->gk)) return false;
  L->blocks = (M + L->mt * thin::kTileM - 1) / (L->mt * thin::kTileM);
  const int tiles = (N + thin::kTileN - 1) / thin::kTileN;
  // one workgroup per compute unit in all; with several rows of workgroups a
  // multiple of 8 along N, so that those of one run of tiles sit on one XCD and
  // share its L2
  L->grid = std::max(1, compute_units() / L->blocks);
  if (L->blocks > 1 && L->grid >= 8) L->grid = L->grid / 8 * 8;
  L->grid = std::min(tiles, L->grid);
  L->run = (tiles + L->grid - 1) / L->grid;
  const size_t red = (size_t)2 * thin::kWaves * L->mt * thin::kTileM * thin::kRedStride * 4;
  const size_t scales = ((size_t)L->run * thin::kTileN * 4 + 15) / 16 * 16;
  const size_t rows = src == thin::kSrcPacked ? 0 : (size_t)nc * kChunk * M + 32;
  L->rows_off = (int)(red + scales);
  L->lds_bytes = red + scales + rows;
  return L->lds_bytes <= kMaxLds;
}

hipError_t launch(const GemmArgs& g, const void* a_src, int src, uint16_t* a_scale_out, hipStream_t s) {
  ThinLaunch L;
  if (!plan(g.M, g.N, g.K, g.p, g.q, src, &L)) return hipErrorInvalidValue;
  ThinParams prm;
  prm.g = g;
  prm.nchunks = num_chunks(g.K);
  prm.groups = padded_rows(g.N) / kRowGroup;
  prm.tiles = (g.N + thin::kTileN - 1) / thin::kTileN;
  prm.w_bytes = (uint32_t)apt_packed_bytes(g.N, g.K, g.p);
  prm.a_bytes = src == thin::kSrcPacked ? (uint32_t)apt_packed_bytes(g.M, g.K, g.q) : 0u;
  prm.a_src = a_src;
  prm.src = src;
  prm.a_vec = (reinterpret_cast<uintptr_t>(a_src) & 15u) == 0 && g.K % 16 == 0;
  prm.a_scale_out = a_scale_out;
  prm.rows_off = L.rows_off;
  prm.ones = prm.nchunks * kChunk * g.M;
  switch (g.p) {
    case 1: return thin::launch_for_p<1>(prm, L, s);
    case 2: return thin::launch_for_p<2>(prm, L, s);
    case 3: return thin::launch_for_p<3>(prm, L, s);
    case 4: return thin::launch_for_p<4>(prm, L, s);
    case 5: return thin::launch_for_p<5>(prm, L, s);
    case 6: return thin::launch_for_p<6>(prm, L, s);
    case 7: return thin::launch_for_p<7>(prm, L, s);
    case 8: return thin::launch_for_p<8>(prm, L, s);
  }
  return hipErrorInvalidValue;
}

}  // namespace

// Modelled microseconds on packed activations, infinity where the kernel does
// not take the problem: the launch, the operands' build (per 16-token tile and
// K group), the items' work (a word's rebuild, which grows with the weight bits,
// and the MFMAs of each token tile) and the weight stream (re-reads by further
// rows of workgroups are served by the caches).  Least squares on the relative
// error over cold timings on MI355X: six-bit operands M = 2..512, N and K =
// 512..11008 (median error 6%); bytes M = 2..512, N = 128..22016, K = 128..8192,
// weights of 1 to 8 bits (median error 5% over 1405 problems, up to 32 rows of
// workgroups among them: W4A8 400 x 1024 x 8192 17.6 us modelled, 16.4 measured;
// a word of 1 bit costs what one of 2 does).
double thin_us(int M, int N, int K, int p, int q, bool unpacked) {
  ThinLaunch L;
  if (!plan(M, N, K, p, q, unpacked ? thin::kSrcHalf : thin::kSrcPacked, &L)) return HUGE_VAL;
  const double mb = (double)N * K * p / 8e6, ops = (double)L.mt * L.gk, items = (double)L.run * L.gk;
  constexpr double kRebuild[5] = {0, 7, 10, 18, 22};
  return L.cls == thin::kLow
             ? 2.61 + 0.886 * ops + items * (0.0115 * kRebuild[p] + 0.233 * L.mt) + 0.178 * mb
             : 3.26 + 1.28 * ops + items * (0.106 * std::max(p, 2) + 0.287 * L.mt) + 0.085 * mb;
}

hipError_t launch_gemm_thin(const GemmArgs& g, hipStream_t s) {
  return launch(g, nullptr, thin::kSrcPacked, nullptr, s);
}

hipError_t launch_gemm_thin_act(const GemmArgs& g, const void* a_src, bool fp16_src, uint16_t* a_scale_out,
                                hipStream_t s) {
  return launch(g, a_src, fp16_src ? thin::kSrcHalf : thin::kSrcCodes, fp16_src ? a_scale_out : nullptr, s);
}

}  // namespace apt

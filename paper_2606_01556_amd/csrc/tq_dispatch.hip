// Kernel selection for the fused layer by token count: the decode kernel for
// m <= 16 (bound by the weight bytes; H formed in every work-group), the mid kernel
// (32- or 64-token blocks, H formed per block) up to 512 tokens, then the large
// kernel (128 x 256 blocks, 16 wavefronts), or once its blocks take more
// than one round over the CUs the prefill kernel (H shared by runs of column
// blocks) -- for r <= 64 only where a run is long enough to carry its H pass;
// past 512 tokens the mid kernel again where the large kernel's blocks would
// leave most CUs idle.
#include <algorithm>

#include "tq_kernels.hpp"

namespace tq {

// Past 512 tokens, where Y's fp32 sums may be split over K (the mid kernel's
// plans of one or two column tiles): rounds of 32-token work-groups x (3 + rank
// tiles + column tiles) below this many units per round of large blocks, for
// 64- and 128-wide groups.  The units are those of an earlier mid kernel; the line
// still lies where the times cross: the mid kernel's best plan takes 0.56 of the
// faster block kernel's time below 28 units a round, 0.85 from 28 to 34, 1.02
// from 34 to 50 and 1.28 above (means of 4000 calls, K 512 to 16384, N 256 to
// 16384, M 513 to 4096, r 0 to 128).  30 of 1882 calls below the line are more
// than 10 % slower than on the large kernel, all with K <= 1536.  Between 28 and
// 34 with 128-wide groups the exact plans below take most of what is left.
constexpr int kLargeRound64 = 34, kLargeRound128 = 28;
int split_units(const GemmArgs &a) {
  const int rt = a.geo.r_pad32 / 32, ct32 = a.geo.n_pad / 32, n_rb = a.ms / 32;
  int best = 1 << 30;
  for (int ct : {1, 2, 4})
    best = std::min(best, (n_rb * ((ct32 + ct - 1) / ct) + 255) / 256 * (3 + rt + ct));
  return best;
}
// K-groups per prefill work-group run from which it beats the large kernel at r <= 64
constexpr int kPrefillMinRun = 256;

int choose_kernel(const GemmArgs &a) {
  if (a.force_kernel >= 0) return a.force_kernel;   // validated by the caller
  // the activation code format follows the same token-count split
  if (a.m <= kDecodeMaxTokens && decode_fits(a.m, a.geo.k)) return kKernelDecode;
  if (!act_codes_fp8(a.m)) return kKernelMid;
  // 128 x 256 blocks: the large kernel (16 wavefronts, H formed in the main
  // loop of every block) is faster while its blocks fit in one round over the
  // 256 CUs; beyond, the prefill kernel forms H once per run of column blocks
  // (one work-group per CU).  For ranks up to 64 the large kernel's H share
  // is at most a quarter of a block's work, so the prefill kernel wins only
  // where its run (cpw column blocks of KG groups each) is long -- at least
  // kPrefillMinRun groups -- for its H pass and per-block fills to amortize.
  const int m_tiles = (a.m + 127) / 128, n_tiles = (a.geo.n_pad + 255) / 256;
  const int blocks = m_tiles * n_tiles;
  const int runs = m_tiles >= 256 ? 1 : 256 / m_tiles;
  const int cpw = (n_tiles + runs - 1) / runs;
  const bool long_run = cpw * (a.geo.k / 64) >= kPrefillMinRun;   // 64-wide K-groups
  // With 128-wide groups the large kernel chains two dependent products per H
  // tile in its main loop, and the prefill kernel applies half the scale
  // products per K block: the prefill kernel wins past one round of blocks
  // at every rank but 0 -- there the large kernel took 273 us and it 288 (4096 ->
  // 14336, M = 4096) when the line was drawn, 266 and 233 now; the name stays
  // where callers find it, and the two return the same bits.
  const bool prefill_wins = a.geo.gk == 1 ? a.geo.r_pad32 > 64 || long_run : a.geo.r_pad32 > 0;
  const bool large = blocks <= 256 || !prefill_wins;
  // few large blocks leave most CUs idle
  const int rounds = (blocks + 255) / 256;
  const int large_round = a.geo.gk == 1 ? kLargeRound64 : kLargeRound128;
  const bool mid = large && split_units(a) < rounds * large_round;
  if (mid) return kKernelMid;
  return large ? kKernelLarge : kKernelPrefill;
}

// Time of a large or prefill launch in ns, to compare with the mid kernel's
// plans that sum Y in the same ascending order, by group width and rank (0, up
// to 64, 128): rounds of blocks x a part of its own and a time per 64-wide K
// block for the large kernel; the H pass and the run's blocks for the prefill
// kernel.  Fitted to 2600 calls with K 512 to 16384, N 256 to 16384 and M 513 to
// 4096, 95 % of them within 12 %.
int64_t block_kernel_ns(const GemmArgs &a, int kernel) {
  const int64_t m_tiles = (a.m + 127) / 128, n_tiles = (a.geo.n_pad + 255) / 256;
  const int rt = a.geo.r_pad32 / 32, c = rt == 0 ? 0 : (rt <= 2 ? 1 : 2), g2 = a.geo.gk == 2;
  const int64_t kg = a.geo.k / 64;
  if (kernel == kKernelLarge) {
    constexpr int kRound[2][3] = {{6000, 7600, 10400}, {4500, 7300, 9900}};
    constexpr int kBlock[2][3] = {{620, 700, 885}, {466, 790, 756}};
    return 900 + (m_tiles * n_tiles + 255) / 256 * (kRound[g2][c] + kg * kBlock[g2][c]);
  }
  // launch, column block, H pass and column block per K block
  constexpr int kNs[2][3][4] = {{{3400, 3900, -100, 565}, {8100, 5300, 150, 570}, {12700, 5400, 310, 563}},
                                {{3000, 4000, -80, 468}, {8100, 5300, 140, 448}, {12600, 5000, 255, 465}}};
  const int *t = kNs[g2][c];
  const int64_t runs = m_tiles >= 256 ? 1 : 256 / m_tiles, cpw = (n_tiles + runs - 1) / runs;
  return (t[0] + t[1] * cpw + kg * (t[2] + t[3] * cpw)) * ((m_tiles + 255) / 256);
}

// Whether the mid kernel's blocks take the place of `kernel`'s (same sums).  They
// have to be 2 % cheaper by the model: a third of the calls named large or
// prefill is then replaced; all of these take 0.935 of the block kernels' time on
// average, 55 of 2133 more than 1.02, three more than 1.05.
bool mid_in_place(const GemmArgs &a, int kernel) {
  return a.force_kernel < 0 && a.mid_ct == 0 && 50 * dual_gemm_mid_ns(a) < 49 * block_kernel_ns(a, kernel);
}

int dual_gemm_block(const GemmArgs &a) {
  const int kernel = choose_kernel(a);
  if (kernel == kKernelDecode) {   // (a token block's room for 8 tokens, or half of 9 to 16)
    const int b = dual_gemm_decode_block(a);
    return std::min(a.m, b >> 16) << 16 | (b & 0xffff);
  }
  const bool exact = kernel != kKernelMid;
  return !exact || mid_in_place(a, kernel) ? dual_gemm_mid_block(a, exact) : 128 << 16 | 256;
}

hipError_t launch_dual_gemm(const GemmArgs &a, hipStream_t s) {
  const int kernel = choose_kernel(a);
  switch (kernel) {
    case kKernelDecode: return launch_dual_gemm_decode(a, nullptr, s);
    case kKernelMid: return launch_dual_gemm_mid(a, false, s);
    default:
      // 128 x 256 blocks, or the mid kernel's smaller ones with Y in the same
      // ascending order where they take less time (few blocks, or a last round
      // that is nearly empty): LLaMA3-8B q/o_proj, r = 128 in 128-wide groups,
      // M = 576: 58 -> 43 us.  A forced tile count has a plan of its own, which
      // may sum in parts: it applies where the mid kernel runs under its own name.
      if (mid_in_place(a, kernel)) return launch_dual_gemm_mid(a, true, s);
      return kernel == kKernelLarge ? launch_dual_gemm_large(a, s) : launch_dual_gemm_prefill(a, s);
  }
}

}  // namespace tq

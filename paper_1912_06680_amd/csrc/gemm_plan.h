// GEMM planning and dispatch: engine, tile and split-K for a problem shape.
#pragma once

#include <type_traits>

#include "gemm_f32.h"
#include "gemm_kk.h"

namespace o5 {

// --------------------------------------------------------------- planning

struct GemmPlan {
  BfTile tile;
  int splits;
  int bm, bn;  // tile of the K-contiguous engine: 256 x 256, 256 x 128 or 320 x 256
};

inline int cdiv(long long a, long long b) { return static_cast<int>((a + b - 1) / b); }

// The fp32 engine's K split: two blocks per CU, every split with at least 128 k.
inline GemmPlan plan_gemm_f32(int M, int N, int K) {
  const long long tiles = f32_tiles(M, N);
  const int s = static_cast<int>(std::min<long long>((512 + tiles - 1) / tiles, std::max(1, K / 128)));
  return {BfTile::kDma256, std::max(1, std::min(s, 16)), 256, 256};
}

// K split of the LSTM's and the loss's products in bf16.  A partial sum
// ends where a split ends, so the split decides the rounding of h, the gates
// and dG; a step's results over several updates amplify a difference there
// (Adam's first updates take the sign of gradients near zero), so it is a
// function of the sizes alone and does not follow the tile.
inline int k_splits(int M, int N, int K) {
  const int nkt = cdiv(K, 64);
  const long long t256 = static_cast<long long>(cdiv(M, 256)) * cdiv(N, 256);
  long long t = t256, least = 16;
  if (t256 < 64) {
    t = static_cast<long long>(cdiv(M, 128)) * cdiv(N, 128);
    least = 8;
  } else if (N % 256 != 0 && N % 256 <= 128) {
    t = static_cast<long long>(cdiv(M, 256)) * cdiv(N, 128);
  }
  const long long s = std::min<long long>((256 + t - 1) / t, std::max<long long>(1, nkt / least));
  return static_cast<int>(std::max<long long>(1, std::min<long long>(s, 8)));
}

// Tile, and K split between s_min and s_max, of a bf16 product of two
// K-contiguous operands, by the time each choice takes: rounds of 256 blocks
// (one per CU), each of ceil(K tiles / splits) K tiles and about 5 us of
// prologue and epilogue, plus the split partial sums, stored at about 2.2
// TB/s (a round stores at once) and read back at 4.5.  A K tile of 64 takes
// 1.75 us on 256 x 256 tiles (M = 2048, N = 4096, K = 16640 in two splits:
// 229 us for 130), 1.1 on 256 x 128 (half the products for 3/4 of the operand
// bytes) and 2.1 on 320 x 256.  (A 128 x 128 register-staged tile takes as
// long for a K tile of a quarter of the products: M = 600, N = 4096, K =
// 16384 took 202 us on it and takes 80 as 32 tiles of 320 x 256 in eight
// splits.)  Products of a few dozen columns follow the same estimate: whole
// calls over 75 logits in us, on 128 x 128 tiles or one fixed 256-wide tile
// and with the choice, H = 4096: sampler (splits freely) 21.8 / 18.3 for 60
// rows, 32.2 / 26.0 for 4096, 61.0 / 49.2 for 12000; loss (the step's split)
// 77.4 / 71.4 for 600 rows, 153 / 137 for 9600.
inline GemmPlan plan_gemm_kk(int M, int N, int K, int s_min, int s_max) {
  GemmPlan best{BfTile::kDma256, s_min, 256, 256};
  const int nkt = cdiv(K, 64);
  // One or two K tiles leave nothing to pipeline: a small grid then takes four
  // times the blocks on 128 x 128 tiles.  A pre-LSTM layer's forward in us, 128
  // x 128 against the tiles below: K = 64 13.6 / 15.0 (M = 600, N = 512), 15.6 /
  // 16.8 (1025, 1024); K = 128 14.8 / 15.9 (1025, 512); K = 192 15.5 / 16.3 (600,
  // 512) but 15.4 / 15.1 (60, 4096); K = 384 18.4 / 18.0 (600, 512).
  if (nkt <= 2 && static_cast<long long>(cdiv(M, 256)) * cdiv(N, 256) < 64) return {BfTile::k128x128, s_min, 256, 256};
  double t_best = 1e30;
  const struct {
    int bm, bn;
    double per_tile;
  } shapes[3] = {{256, 256, 1.75}, {256, 128, 1.1}, {320, 256, 2.1}};
  for (const auto& sh : shapes) {
    const long long tiles = static_cast<long long>(cdiv(M, sh.bm)) * cdiv(N, sh.bn);
    for (int s = s_min; s <= s_max && (s == s_min || nkt / s >= 4); ++s) {
      const double rounds = static_cast<double>((tiles * s + 255) / 256);
      const double bytes = 4.0 * s * M * N;
      const double t =
          rounds * (cdiv(nkt, s) * sh.per_tile + 5.0) + bytes / 2.2e6 + (s > 1 ? bytes / 4.5e6 : 0.0);
      if (t < t_best) {
        t_best = t;
        best = {BfTile::kDma256, s, sh.bm, sh.bn};
      }
    }
  }
  return best;
}

// A product of K-contiguous operands (KRows2) in either type: split as the
// optimizer step's, unsplit, or split as is fastest.
enum class Split { kStep, kOne, kFree };
inline GemmPlan plan_gemm(bool bf16, int M, int N, int K, Split split) {
  if (bf16) {
    const int s = split == Split::kStep ? k_splits(M, N, K) : 1;
    return plan_gemm_kk(M, N, K, s, split == Split::kFree ? 8 : s);
  }
  GemmPlan p = plan_gemm_f32(M, N, K);
  if (split == Split::kOne) p.splits = 1;
  return p;
}

// The same, unsplit, where an operand is I-contiguous (bf16: the
// direct-to-LDS engine, or its register-staged sibling for small grids).
inline GemmPlan plan_gemm_icols(bool bf16, int M, int N) {
  const long long t256 = static_cast<long long>(cdiv(M, 256)) * cdiv(N, 256);
  return {bf16 && t256 < 64 ? BfTile::k128x128 : BfTile::kDma256, 1, 256, 256};
}

template <class AL, class BL, class Epi>
inline void run_gemm(const GemmPlan& p, const AL& al, const BL& bl, const Epi& epi, int M, int N, int K,
                     hipStream_t s) {
  static_assert(AL::kBf16 == BL::kBf16, "operands of one type");
  if constexpr (AL::kBf16) {
    if constexpr (std::is_same_v<AL, KRows2<uint16_t>> && std::is_same_v<BL, KRows2<uint16_t>>) {
      if (p.tile == BfTile::kDma256 && kk_fits(al) && kk_fits(bl)) {
        if (p.bn == 128)
          launch_gemm_kk<256, 128>(al, bl, epi, M, N, K, p.splits, s);
        else if (p.bm == 320)
          launch_gemm_kk<320, 256>(al, bl, epi, M, N, K, p.splits, s);
        else
          launch_gemm_kk<256, 256>(al, bl, epi, M, N, K, p.splits, s);
        return;
      }
    }
    if (p.tile == BfTile::kDma256)
      launch_gemm_bf16_dma(al, bl, epi, M, N, K, p.splits, s);
    else
      launch_gemm_bf16(al, bl, epi, M, N, K, p.splits, s);
  } else {
    launch_gemm_f32(al, bl, epi, M, N, K, p.splits, s);
  }
}

}  // namespace o5

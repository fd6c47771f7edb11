// K-split contraction of few token rows: which problems it takes and the tile
// it runs them on (the kernel is in skinny_impl.h, instantiated per epilogue
// in skinny_<epilogue>.hip).
#include "skinny_impl.h"

namespace mmf {

constexpr int64_t kSkinnyMaxRows = 40000;  // measured

SkinnyPlan skinny_plan(int64_t M, int K, int64_t N, Epilogue ep, int cus) {
  // Estimated cost in KB through one compute unit: the rows and the packed
  // columns of a workgroup's tile plus what a workgroup costs beside them
  // (its first loads' latency and the sum of the eight partial tiles, about
  // kFixed KB), times the rounds of workgroups over the chip.
  //  - One-block tiles (FN = 1) read 64-byte pieces of the weight rows, half a
  //    cache line each: their weight bytes count twice.
  //  - Tiles of 4 x 8 (and 4 x 4) blocks take the registers of a whole compute
  //    unit: whole rounds, and a quarter more per byte since one workgroup
  //    cannot cover another's latency (1.45 times for 4 x 16, whose waves read
  //    each row twice).  The others run two per unit.
  constexpr double kFixed = 60.0;
  const double c = cus > 0 ? cus : 256;
  SkinnyPlan best;
  for (int fn = 1; fn <= 16; fn *= 2) {
    if (ep == Epilogue::kGluF32 && fn < 2) continue;
    for (int fm = 1; fm <= 4; ++fm) {
      if (fn == 16 && fm != 4) continue;  // the one form built: smaller ones never measured best
      const int64_t mb = (M + 16 * fm - 1) / (16 * fm), nb = (N + 16 * fn - 1) / (16 * fn);
      if (fm > 1 && 16 * (fm - 1) >= M) continue;  // a block with no row
      const double rows = static_cast<double>(M) / static_cast<double>(mb);
      const double kb = (rows + 16.0 * fn * (fn == 1 ? 0.5 : 0.25)) * K / 1024.0 + kFixed;
      double rounds = static_cast<double>(mb * nb) / c;
      const bool alone = fm * fn >= 16 && fm > 2;
      if (alone) rounds = (fn == 16 ? 1.45 : 1.25) * static_cast<double>(static_cast<int64_t>(rounds + 0.999999));
      if (rounds < 1.0) rounds = 1.0;
      const double cost = rounds * kb;
      if (best.fm == 0 || cost < best.cost) best = {fm, fn, cost, alone ? rounds : 0.0};
    }
  }
  return best;
}

// Estimated microseconds on the plan's tiles, fitted like gemm_us, without the
// outputs' share: per KB through a compute unit, per round of whole-unit tiles
// the sum of their partial tiles, which no other workgroup covers, and the
// packed weights through HBM.  From rows of q a KB takes 1.2 to 1.35 times as
// long as from tiled q.
static double skinny_us(const SkinnyPlan& p, int K, int64_t N, bool tiled) {
  const double us_per_kb = p.rounds == 0.0 ? (tiled ? 0.0212 : 0.0249)
                           : p.fn < 16     ? (tiled ? 0.0162 : 0.0212)
                                           : (tiled ? 0.0150 : 0.0202);
  return 0.7 + us_per_kb * p.cost + 1.8 * p.rounds + 0.02e-6 * static_cast<double>(K) * static_cast<double>(N);
}

bool skinny_fits(int64_t M, int K, int64_t N, Epilogue ep) {
  // 32-bit offsets: the packed weights
  if (M < 1 || N < 1 || static_cast<int64_t>(K / 16) * N * 4 >= (int64_t(1) << 31)) return false;
  return ep == Epilogue::kGluF32 ? N % 32 == 0 : ep == Epilogue::kAffineF32 ? N % 4 == 0 : true;
}

bool skinny_beats_gemm(int64_t M, int K, int64_t N, Epilogue ep, bool tiled, int cus) {
  if (M <= kDecodeMaxTokens) return true;
  // Beyond 16 rows: where it is estimated 5 % faster than the tiled kernel, up
  // to the rows that were measured.  Over 610 shapes of 65 to 36000 rows (K =
  // 64 to 13824, N = 64 to 27648), with weights that no cache holds, the chosen
  // kernel takes 1.003 times the better one's time on average (rows of q:
  // 1.005); 7 run this kernel, 11 the tiled one, and are 3 to 18 % slower for
  // it.  With weights and outputs in the last-level cache: 1.003.
  // Forward calls from bf16 x on either side of the line, K-split / tiled, us:
  //   K = 1024, N = 1024:  M = 1024 9.2 / 10.6, 1536 11.7 / 11.5, 2048 14.0 / 11.8
  //   K = 2048, N = 2048:  M = 64 6.7 / 16.4, 1024 14.7 / 18.3, 2048 21.5 / 21.1, 3072 30.4 / 26.8
  //   K = 2048, N = 6144:  M = 32 7.2 / 16.6, 384 15.7 / 18.7, 640 17.9 / 19.6, 768 25.6 / 22.6
  //   K = 2048, N = 11264: M = 128 12.4 / 18.2, 320 17.2 / 19.3, 384 21.2 / 22.1, 512 28.2 / 22.3
  //   K = 5120, N = 2048:  M = 1024 22.5 / 35.8, 2048 31.7 / 38.1, 3072 60.3 / 46.4
  //   K = 5120, N = 15360: M = 128 19.3 / 33.7, 256 27.6 / 35.4, 320 36.6 / 40.9, 384 45.8 / 40.9
  //   K = 2048, N = 2050:  M = 256 9.7 / 43.2, 768 13.7 / 18.5, 2048 27.1 / 24.4 (N % 4 != 0)
  if (M > kSkinnyMaxRows) return false;
  return skinny_us(skinny_plan(M, K, N, ep, cus), K, N, tiled) < 0.95 * gemm_us(M, K, N, cus);
}

hipError_t launch_skinny(const ContractArgs& a, bool tiled, hipStream_t stream) {
  const SkinnyPlan p = skinny_plan(a.M, a.K, a.N, a.epilogue, device_cus());
  switch (a.epilogue) {
    case Epilogue::kDequantF32: return launch_skinny_dequant(a, p.fm, p.fn, tiled, stream);
    case Epilogue::kRawI32: return launch_skinny_raw(a, p.fm, p.fn, tiled, stream);
    case Epilogue::kGluF32: return launch_skinny_glu(a, p.fm, p.fn, tiled, stream);
    case Epilogue::kAffineF32: return launch_skinny_affine(a, p.fm, p.fn, tiled, stream);
  }
  return hipErrorInvalidValue;
}

}  // namespace mmf

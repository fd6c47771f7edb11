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
  // to the rows that were measured.  Over 2001 shapes of the fit and 1500 drawn
  // ones (K = 16 to 16384, N = 16 to 125000) the chosen kernel takes 1.003 times
  // the better one's time on average; 29 take this kernel and are 3 to 24 %
  // slower for it, 41 the tiled one (3 to 62 %: row-layout q of few features).
  // Forward calls from bf16 x on either side of the line, K-split / tiled, us:
  //   K = 1024, N = 1024:  M = 1024 8.9 / 11.1, 2048 14.4 / 12.0
  //   K = 2048, N = 2048:  M = 64 6.2 / 13.4, 1024 14.3 / 15.7, 1536 19.5 / 17.6
  //   K = 2048, N = 6144:  M = 32 6.5 / 13.3, 384 14.7 / 15.6, 512 16.2 / 16.2, 768 22.1 / 20.7
  //   K = 2048, N = 11264: M = 128 11.3 / 14.4, 256 15.6 / 15.6, 512 26.0 / 20.9
  //   K = 5120, N = 2048:  M = 1024 21.2 / 29.4, 2048 30.7 / 31.7, 4096 55.4 / 45.5
  //   K = 5120, N = 15360: M = 128 19.3 / 33.9, 256 27.4 / 35.3, 512 48.6 / 42.3
  //   K = 2048, N = 2050:  M = 256 9.3 / 40.7, 768 13.0 / 15.9, 1536 20.1 / 18.1 (N % 4 != 0)
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

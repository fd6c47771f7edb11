// K-split contraction of few token rows: which problems it takes and the tile
// it runs them on (the kernel is in skinny_impl.h, instantiated per epilogue
// in skinny_<epilogue>.hip).
#include "skinny_impl.h"

namespace mmf {

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
      if (best.fm == 0 || cost < best.cost) best = {fm, fn, cost};
    }
  }
  return best;
}

bool skinny_takes(int64_t M, int K, int64_t N, Epilogue ep, bool tiled, int cus) {
  // 32-bit offsets: the packed weights, and a tile's rows of q
  if (M < 1 || N < 1 || static_cast<int64_t>(K / 16) * N * 4 >= (int64_t(1) << 31)) return false;
  if (ep == Epilogue::kGluF32 && N % 32 != 0) return false;
  if (ep == Epilogue::kAffineF32 && N % 4 != 0) return false;
  if (M <= kDecodeMaxTokens) return true;
  // Microseconds of a forward from x (act-quant included), fitted to 150
  // shapes (K = 1024 to 13824, N = 1024 to 27648, M = 17 to 1536): this kernel
  // within about 15 %, the tiled one by its tile's k loop when it runs alone.
  // Its k loop slows down beyond K = 4096 when many tiles stream weights at
  // once (33 instead of 24 us at K = 5120), hence the larger margin there.
  // Measured on either side of the line (this kernel / tiled, us):
  //   K = 2048, N = 6144:  M = 33 7.4 / 13.8, 128 9.0 / 14.2, 384 14.4 / 15.7, 640 19.8 / 17.1
  //   K = 2048, N = 11264: M = 256 14.5 / 15.7, 320 19.2 / 16.3
  //   K = 5632, N = 2048:  M = 64 8.1 / 25.9, 512 15.2 / 28.6, 1536 32.2 / 32.4
  //   K = 5120, N = 15360: M = 128 19.5 / 33.7, 256 31.8 / 34.9, 512 58.1 / 41.7
  //   K = 2992, N = 3998:  M = 64 8.1 / 39.0, 1024 27.7 / 57.2 (N % 4 != 0)
  // From rows of q it takes up to 1.4 times as long as from tiled q.
  const double mine = 4.5 + (tiled ? 0.0216 : 0.029) * skinny_plan(M, K, N, ep, cus).cost;
  const double margin = !tiled ? 1.0 : K > 4096 ? 1.3 : 1.15;
  return mine < margin * (3.0 + gemm_alone_us(M, K, N, cus));
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

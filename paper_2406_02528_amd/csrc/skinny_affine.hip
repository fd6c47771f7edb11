// K-split contraction of few token rows: the affine (bias and per-segment activation) epilogue.
#include "skinny_impl.h"

namespace mmf {

hipError_t launch_skinny_affine(const ContractArgs& a, int fm, int fn, bool tiled, hipStream_t stream) {
  return skinny::dispatch<Epilogue::kAffineF32>(a, fm, fn, tiled, stream);
}

}  // namespace mmf

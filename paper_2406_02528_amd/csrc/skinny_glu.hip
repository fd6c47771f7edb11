// K-split contraction of few token rows: the GLU (SiLU(g) * u) epilogue.
#include "skinny_impl.h"

namespace mmf {

hipError_t launch_skinny_glu(const ContractArgs& a, int fm, int fn, bool tiled, hipStream_t stream) {
  return skinny::dispatch<Epilogue::kGluF32>(a, fm, fn, tiled, stream);
}

}  // namespace mmf

// K-split contraction of few token rows: the dequantising epilogue.
#include "skinny_impl.h"

namespace mmf {

hipError_t launch_skinny_dequant(const ContractArgs& a, int fm, int fn, bool tiled, hipStream_t stream) {
  return skinny::dispatch<Epilogue::kDequantF32>(a, fm, fn, tiled, stream);
}

}  // namespace mmf

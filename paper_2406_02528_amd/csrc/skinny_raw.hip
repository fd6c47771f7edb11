// K-split contraction of few token rows: the raw int32 epilogue.
#include "skinny_impl.h"

namespace mmf {

hipError_t launch_skinny_raw(const ContractArgs& a, int fm, int fn, bool tiled, hipStream_t stream) {
  return skinny::dispatch<Epilogue::kRawI32>(a, fm, fn, tiled, stream);
}

}  // namespace mmf

// Where the int8 rows of q lie and which offsets the kernels load them with:
// plain integer arithmetic, shared by the kernels that write and read them and
// compiled by the host compiler alone in the tests.
//
// A buffer load checks its lane offset against the resource's size less the
// scalar offset.  What that check does when the scalar offset is past the end
// is not documented, so every scalar offset here stays inside its resource and
// only lane offsets go past it.
#pragma once
#include <stdint.h>

#ifdef __HIPCC__
#define MMF_HOST_DEVICE __host__ __device__ __attribute__((always_inline))
#else
#define MMF_HOST_DEVICE
#endif

namespace mmf {

// The TiledQ layout of q (M * K bytes, as the rows): row blocks of 16 rows at
// 16 b K; in a block of mr rows (16, or M % 16 in the last) the 64-byte pieces
// of step s = k / 64 at 64 s mr, row r's at 64 r within them (K % 64 bytes per
// row in a last step of less than 64).  Byte offset of row r of a block of mr
// rows, feature k, from the block:
MMF_HOST_DEVICE inline int tiled_q_piece(int r, int mr, int k, int K) {
  const int at = k & 63, rest = K - (k - at), piece = rest < 64 ? rest : 64;
  return (k - at) * mr + r * piece + at;
}

// The scalar offset base + s step of 16-row block fm at k64 step s, from the
// first row of a tile of `rows` rows of q.  A block past the tile's rows reads
// the first block's first step instead (its sums are dropped).
struct QBlock {
  uint32_t base, step;
};
MMF_HOST_DEVICE inline QBlock q_block(int rows, int fm, int K, bool tiled) {
  const int live = rows - 16 * fm < 16 ? rows - 16 * fm : 16;
  if (live <= 0) return {0u, 0u};
  return {static_cast<uint32_t>(16 * fm) * static_cast<uint32_t>(K), tiled ? static_cast<uint32_t>(64 * live) : 64u};
}

// The lane offset of bytes 16 g .. 16 g + 15 of a step of row r in its block;
// `last`: of the last step, whose tiled pieces may be shorter.
MMF_HOST_DEVICE inline uint32_t q_lane(int r, int g, int K, bool tiled, bool last) {
  const uint32_t rest = static_cast<uint32_t>(K) & 63u;  // no branch: a kernel starts with these
  const uint32_t piece = last && rest != 0 ? rest : 64u, pitch = tiled ? piece : static_cast<uint32_t>(K);
  return static_cast<uint32_t>(r) * pitch + 16u * static_cast<uint32_t>(g);
}

// 16-byte vector v of a row of MLGRU gates (f, c and g, K floats each, side by
// side): the resource over the row, the lane offset (past it for vectors past
// K) and the scalar offsets of the three.
struct GateRow {
  uint32_t bytes, lane, f, c, g;
};
MMF_HOST_DEVICE inline GateRow gate_row(int v, int K) {
  const uint32_t part = 4u * static_cast<uint32_t>(K);
  return {3u * part, 4 * v < K ? 16u * static_cast<uint32_t>(v) : 0x80000000u, 0u, part, 2u * part};
}

}  // namespace mmf

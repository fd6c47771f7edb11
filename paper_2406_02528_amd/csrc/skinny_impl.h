// Contraction of few token rows (the ternary sum from quantised activations
// for a batch of running sequences or a short prompt): the K dimension split
// over the waves of each workgroup.  Included by the skinny_*.hip files, one
// per epilogue, which compile in parallel.
//
// With few rows the contraction is bound by how fast the packed weights (and
// the int8 rows, from L2) reach the compute units, and one compute unit can
// only have so many bytes in flight: a tile wide enough for operand reuse
// leaves most of the chip idle (45 rows by 6144 columns are 24 tiles of
// 64 x 256: 15 us for 3 MB of weights).  So the tile here is narrow enough
// that a launch covers the chip, 16 FM rows by 16 FN columns, and the 8 waves
// of a workgroup each take a contiguous eighth of the k64 steps of the whole
// tile.  No operand is read twice inside a workgroup, so nothing is staged
// through LDS and the k loop has no barrier: every wave loads its fragments
// from memory into the registers the matrix instruction reads, D steps ahead.
// The eight partial tiles are then added in LDS (int32, exact) and leave
// through the epilogue.  Wide outputs with many rows have more tiles than the
// chip holds and are bound by the rows every column strip reads again: there
// WN = 2 halves of the waves take 128 columns each and a quarter of the steps
// (64 x 256 tiles; 128 x 5120 x 27648: 27.1 -> 24.1 us).
//
// Fragments: one k64 step is 4 word rows of the packed weights and 64 bytes
// of each row of q.  Lane (g, l16) loads bytes 16 g .. 16 g + 15 of row l16 of
// each 16-row block (one 16-byte load), and the words of word row 4 s + g of
// its F consecutive columns F l16 .. F l16 + F - 1 in each of the NG column
// groups (one 4-, 8- or 16-byte load).  Word rows past K / 16 fall outside the
// buffer resource and read as zero, so what the row fragments hold there (and
// in rows past M, whose sums are dropped) does not matter.
//
// q comes in one of two layouts: rows ([M][K], the public one), or tiled as
// the library's own act-quant launch writes it for this kernel, each 16-row
// block's 64-byte pieces of a k64 step next to each other (TiledQ in
// q_layout.h), so that a fragment is 1 KB of consecutive memory instead of
// 16 half cache lines K bytes apart: with K a multiple of 1024 those fall on
// few L2 channels.  Measured from rows -> tiled, us: 48 x 5632 x 2048
// 7.7 -> 5.3, 128 x 5120 x 15360 20.1 -> 15.9, 128 x 13824 x 5120
// 24.0 -> 16.7, 48 x 2048 x 6144 5.0 -> 4.3.
#pragma once
#include "gemm_common.h"
#include "mmf_device.h"
#include "mmf_launch.h"
#include "q_layout.h"

namespace mmf {
namespace skinny {

constexpr int kWaves = 8;  // per workgroup: kWaves / WN shares of the k64 steps
constexpr int kThreads = kWaves * kWave;

struct Params {
  const int8_t* q;          // [M][K]
  const float* a_scale;     // [M]
  const int32_t* q_rowsum;  // [M]
  const uint32_t* Wp;       // [K/16][N]
  const float* w_scale;
  void* out;
  int64_t M, N;
  int K;
  int mblocks;              // row blocks of 16 FM
  bool tiled;               // layout of q
  Affine affine;
};

// 16-row blocks whose partial sums are in LDS at once (8 partial tiles of
// 16 R rows: about 70 KB, so that two workgroups fit a compute unit).
constexpr int rows_per_round(int fm, int fn) {
  const int r = fn >= 8 ? 1 : fn >= 4 ? 2 : 4;
  return r < fm ? r : fm;
}

// Whether a tile shape keeps four steps of fragments in flight instead of two
// (the wide tiles measured level or faster with two, and four would cost them
// the second workgroup on a compute unit).
constexpr bool skinny_deep(int fm, int fn) { return fn <= 2 || fm == 1 || (fm == 2 && fn == 4); }

// VEC: N % 4 == 0.  Otherwise the word rows start on any dword (buffer loads
// need dword alignment only and are range-checked dword by dword; columns past
// N read the next word row or zero and are dropped), and the outputs that
// cross a row's end are stored one by one.
template <int FM, int NG, int F, int WN, int D, bool VEC, Epilogue EP>
__global__ __launch_bounds__(kThreads) __attribute__((amdgpu_waves_per_eu(2))) void skinny_kernel(const Params p) {
  constexpr int kSplit = kWaves / WN;
  constexpr int FN = NG * F, WC = 16 * FN, BN = WC * WN;  // blocks and columns of a wave, columns of the tile
  constexpr int R = rows_per_round(FM, FN);
  constexpr int kStride = BN + 4;  // padded row of a partial tile: conflict-free 16-byte writes of 16 rows
  constexpr int kPart = 16 * R * kStride;
  static_assert(EP != Epilogue::kGluF32 || (FN >= 2 && VEC), "whole gate/up block pairs per workgroup");
  static_assert(EP != Epilogue::kAffineF32 || VEC, "affine output needs N % 4 == 0");
  __shared__ __attribute__((aligned(16))) int part[kSplit * kPart];
  __shared__ float s_scale[16 * FM];
  __shared__ int s_rsum[16 * FM];

  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int l16 = lane & 15, g = lane >> 4;
  const int kw = wave / WN, nw = wave % WN;  // the wave's share of the steps, its columns
  const int K = p.K, J = K / 16;
  const int64_t N = p.N;

  // Tile order: workgroups are dealt round-robin to the 8 XCDs; each XCD gets
  // a contiguous run of tiles with the row blocks of one column strip next to
  // each other, so that a strip's weights come from HBM once per XCD.
  int64_t L = blockIdx.x;
  {
    const int64_t per = gridDim.x / kXcds;
    if (L < per * kXcds) L = (L % kXcds) * per + L / kXcds;
  }
  const int64_t mb = L % p.mblocks, nb = L / p.mblocks;
  const int64_t m0 = mb * (16 * FM);
  const int64_t n0 = nb * BN;
  const int rows = static_cast<int>(p.M - m0 < 16 * FM ? p.M - m0 : 16 * FM);

  const __amdgpu_buffer_rsrc_t arsrc = __builtin_amdgcn_make_buffer_rsrc(
      const_cast<int8_t*>(p.q + m0 * K), 0, rows * K, kBufferFlags);
  const __amdgpu_buffer_rsrc_t brsrc = __builtin_amdgcn_make_buffer_rsrc(
      const_cast<uint32_t*>(p.Wp), 0, static_cast<int>(static_cast<uint32_t>(J) * 4u * static_cast<uint32_t>(N)),
      kBufferFlags);
  const uint32_t row_bytes = 4u * static_cast<uint32_t>(N);
  // A fragment of block fm and step s: a lane offset (another one in a last
  // step of less than 64 bytes per row) and a wave-uniform one, both inside
  // the resource or past it by the lane offset alone (q_layout.h).
  const uint32_t a_lane = q_lane(l16, g, K, p.tiled, false), a_lane_last = q_lane(l16, g, K, p.tiled, true);
  QBlock a_at[FM];
  uint32_t b_off[NG];
#pragma unroll
  for (int fm = 0; fm < FM; ++fm) a_at[fm] = q_block(rows, fm, K, p.tiled);
#pragma unroll
  for (int c = 0; c < NG; ++c) {
    const int64_t col = n0 + nw * WC + c * 16 * F + F * l16;
    b_off[c] = col < N ? static_cast<uint32_t>(g) * row_bytes + 4u * static_cast<uint32_t>(col) : kOutOfRange;
  }

  // this wave's share of the k64 steps: [sb, sb + ns)
  const int steps = (J + 3) / 4;
  const int base = steps / kSplit, extra = steps % kSplit;
  const int sb = kw * base + (kw < extra ? kw : extra);
  const int ns = base + (kw < extra ? 1 : 0);

  struct Frag {
    v4i a[FM];
    Words<F> b[NG];
  };
  auto load = [&](Frag& f, int i) __attribute__((always_inline)) {
    const int s = sb + (i < ns ? i : ns - 1);  // past the share: its last step again (loaded, not used)
    const uint32_t bs = static_cast<uint32_t>(s) * 4u * row_bytes;
#pragma unroll
    for (int c = 0; c < NG; ++c) f.b[c] = load_words<F>(brsrc, b_off[c], bs);
    const uint32_t al = s == steps - 1 ? a_lane_last : a_lane;
#pragma unroll
    for (int fm = 0; fm < FM; ++fm)
      f.a[fm] = __builtin_bit_cast(v4i, __builtin_amdgcn_raw_buffer_load_b128(
                                            arsrc, al, a_at[fm].base + static_cast<uint32_t>(s) * a_at[fm].step, 0));
  };
  v4i acc[FM][FN];
#pragma unroll
  for (int a = 0; a < FM; ++a)
#pragma unroll
    for (int b = 0; b < FN; ++b) acc[a][b] = v4i{0, 0, 0, 0};
  auto contract = [&](const Frag& f) __attribute__((always_inline)) {
#pragma unroll
    for (int c = 0; c < NG; ++c)
#pragma unroll
      for (int k = 0; k < F; ++k) {
        const uint32_t x = f.b[c].w[k];
        const v4i cw = {static_cast<int>(codes4(x, 0)), static_cast<int>(codes4(x, 1)),
                        static_cast<int>(codes4(x, 2)), static_cast<int>(codes4(x, 3))};
#pragma unroll
        for (int fm = 0; fm < FM; ++fm)
          acc[fm][c * F + k] = __builtin_amdgcn_mfma_i32_16x16x64_i8(cw, f.a[fm], acc[fm][c * F + k], 0, 0, 0);
      }
  };

  Frag fr[D];
#pragma unroll
  for (int d = 0; d < D; ++d) load(fr[d], d);
  // per-row and per-column factors, behind the first fragments
  float my_scale = 0.0f;
  int my_rsum = 0;
  if (tid < 16 * FM && tid < rows) {
    my_rsum = p.q_rowsum[m0 + tid];
    if constexpr (EP != Epilogue::kRawI32) my_scale = p.a_scale[m0 + tid];
  }
  const float ws = (EP == Epilogue::kDequantF32 || EP == Epilogue::kGluF32) ? p.w_scale[0] : 0.0f;
  const float ws_u = EP == Epilogue::kGluF32 ? p.w_scale[1] : 0.0f;
  ColAffine4 col{};
  if constexpr (EP == Epilogue::kAffineF32) {
    static_assert(kThreads % (BN / 4) == 0, "a thread keeps its column quad over the epilogue");
    const int64_t n = n0 + 4 * (tid % (BN / 4));
    col = load_col_affine4(p.affine, p.w_scale, static_cast<uint32_t>(N), n < N ? static_cast<uint32_t>(n) : 0u);
  }

  int i = 0;
  for (; i + D < ns; i += D) {
#pragma unroll
    for (int d = 0; d < D; ++d) {
      contract(fr[d]);
      __builtin_amdgcn_sched_barrier(0);
      load(fr[d], i + D + d);
      __builtin_amdgcn_sched_barrier(0);
    }
  }
#pragma unroll
  for (int d = 0; d < D; ++d)
    if (i + d < ns) contract(fr[d]);

  if (tid < 16 * FM) {
    s_rsum[tid] = my_rsum;
    s_scale[tid] = my_scale;
  }
  // The partial tiles in LDS, R blocks of 16 rows at a time: lane (g, l16)
  // holds row l16 and columns F (4 g + r) + k of each column group.
#pragma unroll
  for (int f0 = 0; f0 < FM; f0 += R) {
    if (f0 > 0) lds_barrier();
    int* mine = part + kw * kPart + nw * WC;
#pragma unroll
    for (int fm = f0; fm < f0 + R && fm < FM; ++fm) {
      int* row = mine + ((fm - f0) * 16 + l16) * kStride;
#pragma unroll
      for (int c = 0; c < NG; ++c) {
        if constexpr (F == 4) {
#pragma unroll
          for (int r = 0; r < 4; ++r)
            *reinterpret_cast<v4i*>(row + c * 64 + 16 * g + 4 * r) =
                v4i{acc[fm][4 * c][r], acc[fm][4 * c + 1][r], acc[fm][4 * c + 2][r], acc[fm][4 * c + 3][r]};
        } else if constexpr (F == 2) {
#pragma unroll
          for (int r = 0; r < 4; r += 2)
            *reinterpret_cast<v4i*>(row + c * 32 + 8 * g + 2 * r) =
                v4i{acc[fm][2 * c][r], acc[fm][2 * c + 1][r], acc[fm][2 * c][r + 1], acc[fm][2 * c + 1][r + 1]};
        } else {
          *reinterpret_cast<v4i*>(row + c * 16 + 4 * g) = acc[fm][c];
        }
      }
    }
    lds_barrier();
    constexpr int kW = EP == Epilogue::kGluF32 ? BN / 2 : BN;  // output columns of the tile
    constexpr int kQuads = kW / 4;
    const int live = (FM - f0 < R ? FM - f0 : R) * 16 * kQuads;
    const int64_t ow = EP == Epilogue::kGluF32 ? N / 2 : N;
    auto total = [&](int row, int c) -> v4i {
      v4i t = v4i{0, 0, 0, 0};
#pragma unroll
      for (int w = 0; w < kSplit; ++w) t += *reinterpret_cast<const v4i*>(part + w * kPart + row * kStride + c);
      return t;
    };
#pragma unroll 2
    for (int e = tid; e < live; e += kThreads) {
      const int lr = e / kQuads, cq = e % kQuads;
      const int tr = f0 * 16 + lr;  // row of the tile
      const int rs = s_rsum[tr];
      const float as = s_scale[tr];
      v4i v;
      if constexpr (EP == Epilogue::kGluF32) {
        const int cg = (cq / 4) * 32 + 4 * (cq % 4);  // gate columns; the up columns follow 16 later
        const v4i tg = total(lr, cg), tu = total(lr, cg + 16);
        const float sg = as * ws, su = as * ws_u;
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const float gv = static_cast<float>(tg[r] - rs) * sg;
          const float uv = static_cast<float>(tu[r] - rs) * su;
          v[r] = __float_as_int(gv * sigmoid_hw(gv) * uv);
        }
      } else {
        const v4i t = total(lr, 4 * cq);
        const float sc = as * ws;
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const int d = t[r] - rs;
          if constexpr (EP == Epilogue::kAffineF32) {
            const float z = static_cast<float>(d) * (as * col.ws) + col.bias[r];
            v[r] = __float_as_int(affine_act(z, col.act, col.lb[r]));
          } else {
            v[r] = EP == Epilogue::kDequantF32 ? __float_as_int(static_cast<float>(d) * sc) : d;
          }
        }
      }
      if (tr < rows) {
        const int64_t n = (EP == Epilogue::kGluF32 ? n0 / 2 : n0) + 4 * cq;
        int* dst = static_cast<int*>(p.out) + (m0 + tr) * ow + n;
        if constexpr (VEC) {
          if (n < ow) *reinterpret_cast<v4i*>(dst) = v;
        } else if (n + 3 < ow) {
          typedef int v4i_dword __attribute__((ext_vector_type(4), aligned(4)));
          *reinterpret_cast<v4i_dword*>(dst) = v;
        } else {
#pragma unroll
          for (int r = 0; r < 3; ++r)
            if (n + r < ow) dst[r] = v[r];
        }
      }
    }
  }
}

template <int FM, int NG, int F, int WN, int D, bool VEC, Epilogue EP>
hipError_t launch_one(const ContractArgs& a, bool tiled, hipStream_t stream) {
  constexpr int kBM = 16 * FM, kBN = 16 * NG * F * WN;
  const int64_t mblocks = (a.M + kBM - 1) / kBM, nblocks = (a.N + kBN - 1) / kBN;
  const Params p{a.q, a.a_scale, a.q_rowsum, a.Wpacked, a.w_scale, a.out, a.M, a.N, a.K,
                 static_cast<int>(mblocks), tiled, a.affine};
  hipLaunchKernelGGL((skinny_kernel<FM, NG, F, WN, D, VEC, EP>), dim3(static_cast<unsigned>(mblocks * nblocks)),
                     dim3(kThreads), 0, stream, p);
  return hipGetLastError();
}

template <int FM, int NG, int F, bool VEC, Epilogue EP>
hipError_t dispatch_d(const ContractArgs& a, bool tiled, hipStream_t stream) {
  if constexpr (skinny_deep(FM, NG * F)) {
    // more than two steps per wave
    if (a.K > 2 * 64 * kWaves) return launch_one<FM, NG, F, 1, 4, VEC, EP>(a, tiled, stream);
  }
  return launch_one<FM, NG, F, 1, 2, VEC, EP>(a, tiled, stream);
}

template <int FM, Epilogue EP>
hipError_t dispatch_fn(const ContractArgs& a, int fn, bool tiled, hipStream_t stream) {
  if constexpr (EP == Epilogue::kDequantF32 || EP == Epilogue::kRawI32) {
    if (a.N % 4 != 0) {
      switch (fn) {
        case 1: return dispatch_d<FM, 1, 1, false, EP>(a, tiled, stream);
        case 2: return dispatch_d<FM, 1, 2, false, EP>(a, tiled, stream);
        case 4: return dispatch_d<FM, 1, 4, false, EP>(a, tiled, stream);
        case 8: return dispatch_d<FM, 2, 4, false, EP>(a, tiled, stream);
        case 16:
          if constexpr (FM == 4) return launch_one<FM, 2, 4, 2, 2, false, EP>(a, tiled, stream);
          return hipErrorInvalidValue;
        default: return hipErrorInvalidValue;
      }
    }
  }
  if (a.N % 4 != 0) return hipErrorInvalidValue;
  switch (fn) {
    case 1:
      if constexpr (EP != Epilogue::kGluF32) return dispatch_d<FM, 1, 1, true, EP>(a, tiled, stream);
      return hipErrorInvalidValue;
    case 2: return dispatch_d<FM, 1, 2, true, EP>(a, tiled, stream);
    case 4: return dispatch_d<FM, 1, 4, true, EP>(a, tiled, stream);
    case 8: return dispatch_d<FM, 2, 4, true, EP>(a, tiled, stream);
    case 16:
      if constexpr (FM == 4) return launch_one<FM, 2, 4, 2, 2, true, EP>(a, tiled, stream);
      return hipErrorInvalidValue;
    default: return hipErrorInvalidValue;
  }
}

template <Epilogue EP>
hipError_t dispatch(const ContractArgs& a, int fm, int fn, bool tiled, hipStream_t stream) {
  switch (fm) {
    case 1: return dispatch_fn<1, EP>(a, fn, tiled, stream);
    case 2: return dispatch_fn<2, EP>(a, fn, tiled, stream);
    case 3: return dispatch_fn<3, EP>(a, fn, tiled, stream);
    case 4: return dispatch_fn<4, EP>(a, fn, tiled, stream);
    default: return hipErrorInvalidValue;
  }
}

}  // namespace skinny

// One per epilogue, in skinny_<epilogue>.hip.
hipError_t launch_skinny_dequant(const ContractArgs& a, int fm, int fn, bool tiled, hipStream_t stream);
hipError_t launch_skinny_raw(const ContractArgs& a, int fm, int fn, bool tiled, hipStream_t stream);
hipError_t launch_skinny_glu(const ContractArgs& a, int fm, int fn, bool tiled, hipStream_t stream);
hipError_t launch_skinny_affine(const ContractArgs& a, int fm, int fn, bool tiled, hipStream_t stream);

}  // namespace mmf

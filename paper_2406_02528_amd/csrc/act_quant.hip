// Fused RMSNorm + per-token absmax int8 quantisation (Algorithm 1,
// rms_norm_fwd + activation_quant; RMSNorm with the mean of squares and
// eps = 1e-6, learned scale gamma), optionally keeping rstd for the backward.
// One to sixteen wave64s per token row; the row is read from HBM once and
// kept in registers while the two row statistics (sum of squares, then
// absmax of the normalised values) are reduced across the row's lanes.
#include "mmf_device.h"
#include "mmf_launch.h"
#include "q_layout.h"

namespace mmf {
namespace {

// Waves of a block: 256 threads, or one row of more than 4 waves.
constexpr int block_waves(int w) { return w > 4 ? w : 4; }
constexpr int kBufferFlags = 0x00020000;  // gfx9 buffer descriptor word 3

// 16-byte vector of activations: 8 bf16 or 4 fp32.
template <typename XT> struct Vec;
template <> struct Vec<uint16_t> {
  static constexpr int kElems = 8;
  using Raw = uint4;
  __device__ static void to_f32(const Raw& r, float* f) {
    const uint32_t w[4] = {r.x, r.y, r.z, r.w};
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      f[2 * i] = __uint_as_float(w[i] << 16);
      f[2 * i + 1] = __uint_as_float(w[i] & 0xFFFF0000u);
    }
  }
};
template <> struct Vec<float> {
  static constexpr int kElems = 4;
  using Raw = float4;
  __device__ static void to_f32(const Raw& r, float* f) {
    f[0] = r.x; f[1] = r.y; f[2] = r.z; f[3] = r.w;
  }
};

// q of one 16-byte vector (E values) into its row: E / 4 packed words, and
// their byte sum added to rs
template <int E>
__device__ __forceinline__ void quantise_store(int8_t* dst, const float* y, float s, int& rs) {
  uint32_t w[E / 4];
#pragma unroll
  for (int g = 0; g < E / 4; ++g) {
    w[g] = quantise4(y + 4 * g, s);
    rs = byte_sum4(w[g], rs);
  }
  if constexpr (E == 8)
    *reinterpret_cast<uint2*>(dst) = make_uint2(w[0], w[1]);
  else
    *reinterpret_cast<uint32_t*>(dst) = w[0];
}

__device__ __forceinline__ float row_rstd(double ss, int K) { return rms_rstd(ss, K); }

// MLGRU decode step: the activations are the output gate o' = g sigmoid(h'),
// h' = f h + (1 - f) c, formed on load from the gates fcg [M][3K] and the state
// h_in [M][K] (nullptr: 0); the new state h' goes to h_out (nullptr: not
// stored), which may be h_in: each element is read and written by one lane.
struct Mlgru {
  const float* fcg;
  const float* h_in;
  float* h_out;
};

// One row per W waves (W = 1 to 16; blocks of 4 waves hold 4 / W rows).
// MLGRU: x is not read (VPL > 0 only).
// VPL > 0: each lane keeps VPL 16-byte vectors of its row in registers (rows
// of at most 64 W VPL vectors), so the row is read from HBM once; with W > 1
// the row's statistics are combined across its waves through LDS, in a fixed
// order (the fp64 sum of squares is therefore deterministic).  VPL == 0: any
// K; the row is re-read from memory (L2) for each of the three passes.
template <typename XT, int W, int VPL, bool TILED, bool MLGRU>
__global__ __launch_bounds__(kWave* block_waves(W)) void act_quant_kernel(
    const XT* __restrict__ x, const float* __restrict__ gamma,
    int8_t* __restrict__ q, float* __restrict__ a_scale,
    int32_t* __restrict__ q_rowsum, float* __restrict__ rstd, int64_t M, int K, const Mlgru step) {
  using V = Vec<XT>;
  constexpr int E = V::kElems;
  static_assert(!MLGRU || (E == 4 && VPL > 0), "fp32 gates, the row in registers");
  constexpr int kBlockWaves = block_waves(W);
  constexpr int kRows = kBlockWaves / W;  // rows per block
  const int lane = threadIdx.x & 63;
  const int wave = threadIdx.x >> 6;
  const int rw = wave % W;                   // wave within the row
  const int rl = rw * kWave + lane;          // lane within the row
  const int64_t row = static_cast<int64_t>(blockIdx.x) * kRows + wave / W;
  const bool live = row < M;                 // uniform per wave (and per row)
  // per-row statistics of the W waves: [row in block][wave in row]
  __shared__ double s_ss[kBlockWaves];
  __shared__ float s_amax[kBlockWaves];
  __shared__ int s_rs[kBlockWaves];
  const int slot0 = (wave / W) * W;
  auto combine_f64 = [&](double v) -> double {
    if constexpr (W == 1) {
      return v;
    } else {
      if (lane == 0) s_ss[wave] = v;
      __syncthreads();
      double t = 0.0;
#pragma unroll
      for (int w = 0; w < W; ++w) t += s_ss[slot0 + w];
      return t;
    }
  };
  auto combine_max = [&](float v) -> float {
    if constexpr (W == 1) {
      return v;
    } else {
      if (lane == 0) s_amax[wave] = v;
      __syncthreads();
      float t = 0.0f;
#pragma unroll
      for (int w = 0; w < W; ++w) t = fmaxf(t, s_amax[slot0 + w]);
      return t;
    }
  };
  auto combine_i32 = [&](int v) -> int {
    if constexpr (W == 1) {
      return v;
    } else {
      if (lane == 0) s_rs[wave] = v;
      __syncthreads();
      int t = 0;
#pragma unroll
      for (int w = 0; w < W; ++w) t += s_rs[slot0 + w];
      return t;
    }
  };
  if constexpr (W == 1) {
    if (!live) return;  // whole wave leaves together
  }
  // a block's rows past M read nothing (a resource of size 0) and store nothing;
  // their waves still take part in the block's barriers
  const int64_t srow = live ? row : 0;
  const int nvec = K / E;
  const typename V::Raw* xr = reinterpret_cast<const typename V::Raw*>(x + srow * K);
  // where a vector of E values starting at feature k goes (pieces of 64 bytes
  // hold whole vectors)
  const int64_t t16 = srow / 16 * 16;
  const int trows = static_cast<int>(M - t16 < 16 ? M - t16 : 16);
  int8_t* const qr = q + (TILED ? t16 : srow) * K;
  auto q_at = [&](int k) -> int8_t* {
    return qr + (TILED ? tiled_q_piece(static_cast<int>(srow - t16), trows, k, K) : k);
  };

  if constexpr (VPL > 0) {
    // Every load of the row and of gamma is issued at once, without branches:
    // both go through buffer resources of the row's (gamma's) size, so the
    // vectors past the row's end read as zero (and gamma == NULL as a
    // resource of size 0).  Guarded loads would each wait for the last.
    const __amdgpu_buffer_rsrc_t grsrc = __builtin_amdgcn_make_buffer_rsrc(
        const_cast<float*>(gamma), 0, gamma != nullptr ? K * 4 : 0, kBufferFlags);
    typename V::Raw raw[VPL];
    float4 gv[VPL][E / 4];
    if constexpr (MLGRU) {
      // f, c and g side by side in the row of fcg (a row past M reads the
      // first one's); the state through a resource of size 0 when there is none
      const __amdgpu_buffer_rsrc_t frsrc = __builtin_amdgcn_make_buffer_rsrc(
          const_cast<float*>(step.fcg + srow * 3 * K), 0, static_cast<int>(gate_row(0, K).bytes), kBufferFlags);
      const __amdgpu_buffer_rsrc_t hrsrc = __builtin_amdgcn_make_buffer_rsrc(
          const_cast<float*>(step.h_in + (step.h_in != nullptr ? srow * K : 0)), 0,
          live && step.h_in != nullptr ? K * 4 : 0, kBufferFlags);
      float4 fv[VPL], cv[VPL], hv[VPL];
#pragma unroll
      for (int i = 0; i < VPL; ++i) {
        const GateRow at = gate_row(rl + W * kWave * i, K);
        fv[i] = __builtin_bit_cast(float4, __builtin_amdgcn_raw_buffer_load_b128(frsrc, at.lane, at.f, 0));
        cv[i] = __builtin_bit_cast(float4, __builtin_amdgcn_raw_buffer_load_b128(frsrc, at.lane, at.c, 0));
        raw[i] = __builtin_bit_cast(float4, __builtin_amdgcn_raw_buffer_load_b128(frsrc, at.lane, at.g, 0));
        hv[i] = __builtin_bit_cast(float4, __builtin_amdgcn_raw_buffer_load_b128(hrsrc, at.lane, 0, 0));
      }
#pragma unroll
      for (int i = 0; i < VPL; ++i) {
        const int v = rl + W * kWave * i;
        const bool ok = v < nvec;
        const float4 hn = {mlgru_step(hv[i].x, fv[i].x, cv[i].x), mlgru_step(hv[i].y, fv[i].y, cv[i].y),
                           mlgru_step(hv[i].z, fv[i].z, cv[i].z), mlgru_step(hv[i].w, fv[i].w, cv[i].w)};
        raw[i] = {ok ? mlgru_out_gate(raw[i].x, hn.x) : 0.0f, ok ? mlgru_out_gate(raw[i].y, hn.y) : 0.0f,
                  ok ? mlgru_out_gate(raw[i].z, hn.z) : 0.0f, ok ? mlgru_out_gate(raw[i].w, hn.w) : 0.0f};
        if (ok && live && step.h_out != nullptr)
          *reinterpret_cast<float4*>(step.h_out + srow * K + 4 * v) = hn;
      }
    } else {
      const __amdgpu_buffer_rsrc_t xrsrc = __builtin_amdgcn_make_buffer_rsrc(
          const_cast<XT*>(x + srow * K), 0, live ? static_cast<int>(K * sizeof(XT)) : 0, kBufferFlags);
#pragma unroll
      for (int i = 0; i < VPL; ++i)
        raw[i] = __builtin_bit_cast(typename V::Raw, __builtin_amdgcn_raw_buffer_load_b128(
                                                         xrsrc, static_cast<uint32_t>((rl + W * kWave * i) * 16), 0, 0));
    }
#pragma unroll
    for (int i = 0; i < VPL; ++i)
#pragma unroll
      for (int e4 = 0; e4 < E / 4; ++e4)
        gv[i][e4] = __builtin_bit_cast(
            float4, __builtin_amdgcn_raw_buffer_load_b128(
                        grsrc, static_cast<uint32_t>(((rl + W * kWave * i) * E + 4 * e4) * 4), 0, 0));
    __builtin_amdgcn_sched_barrier(0);  // all loads before the first wait
    float xf[VPL][E];
    double ss = 0.0;
#pragma unroll
    for (int i = 0; i < VPL; ++i) {
      V::to_f32(raw[i], xf[i]);  // zero past the row's end
#pragma unroll
      for (int e = 0; e < E; ++e) ss = sum_sq(ss, xf[i][e]);
    }
    ss = combine_f64(wave_sum_f64(ss));
    const float r = row_rstd(ss, K);

    float amax = 0.0f;
#pragma unroll
    for (int i = 0; i < VPL; ++i) {
      if (gamma != nullptr) {  // uniform
#pragma unroll
        for (int e4 = 0; e4 < E / 4; ++e4) {
          xf[i][4 * e4 + 0] = (xf[i][4 * e4 + 0] * r) * gv[i][e4].x;
          xf[i][4 * e4 + 1] = (xf[i][4 * e4 + 1] * r) * gv[i][e4].y;
          xf[i][4 * e4 + 2] = (xf[i][4 * e4 + 2] * r) * gv[i][e4].z;
          xf[i][4 * e4 + 3] = (xf[i][4 * e4 + 3] * r) * gv[i][e4].w;
        }
      } else {
#pragma unroll
        for (int e = 0; e < E; ++e) xf[i][e] = xf[i][e] * r;
      }
#pragma unroll
      for (int e = 0; e < E; ++e) amax = fmaxf(amax, fabsf(xf[i][e]));
    }
    amax = fmaxf(combine_max(wave_max_f32(amax)), 1e-5f);
    const float s = 127.0f / amax;

    int rs = 0;
#pragma unroll
    for (int i = 0; i < VPL; ++i) {
      const int v = rl + W * kWave * i;
      if (live && v < nvec) quantise_store<E>(q_at(v * E), xf[i], s, rs);
    }
    rs = combine_i32(wave_sum_i32(rs));
    if (live && rl == 0) {
      a_scale[row] = amax / 127.0f;
      if (q_rowsum != nullptr) q_rowsum[row] = rs;
      if (rstd != nullptr) rstd[row] = r;
    }
  } else {
    // pass 1: sum of squares
    double ss = 0.0;
    if (live) {
      for (int v = rl; v < nvec; v += W * kWave) {
        float f[E];
        V::to_f32(xr[v], f);
#pragma unroll
        for (int e = 0; e < E; ++e) ss = sum_sq(ss, f[e]);
      }
    }
    ss = combine_f64(wave_sum_f64(ss));
    const float r = row_rstd(ss, K);
    // pass 2: absmax of the normalised row
    float amax = 0.0f;
    if (live) {
      for (int v = rl; v < nvec; v += W * kWave) {
        float f[E];
        V::to_f32(xr[v], f);
#pragma unroll
        for (int e = 0; e < E; ++e) {
          float y = f[e] * r;
          if (gamma != nullptr) y = y * gamma[v * E + e];
          amax = fmaxf(amax, fabsf(y));
        }
      }
    }
    amax = fmaxf(combine_max(wave_max_f32(amax)), 1e-5f);
    const float s = 127.0f / amax;
    // pass 3: quantise
    int rs = 0;
    if (live) {
      for (int v = rl; v < nvec; v += W * kWave) {
        float f[E];
        V::to_f32(xr[v], f);
#pragma unroll
        for (int e = 0; e < E; ++e) {
          f[e] = f[e] * r;
          if (gamma != nullptr) f[e] = f[e] * gamma[v * E + e];
        }
        quantise_store<E>(q_at(v * E), f, s, rs);
      }
    }
    rs = combine_i32(wave_sum_i32(rs));
    if (live && rl == 0) {
      a_scale[row] = amax / 127.0f;
      if (q_rowsum != nullptr) q_rowsum[row] = rs;
      if (rstd != nullptr) rstd[row] = r;
    }
  }
}

struct Args {
  const void* x;
  const float* gamma;
  int8_t* q;
  float* a_scale;
  int32_t* q_rowsum;
  float* rstd;
  int64_t M;
  int K;
  bool tiled;
  Mlgru step;
};

template <typename XT, int W, int VPL, bool TILED, bool MLGRU>
hipError_t launch_kernel(const Args& a, hipStream_t stream) {
  constexpr int kRows = block_waves(W) / W;
  const dim3 grid(static_cast<unsigned>((a.M + kRows - 1) / kRows));
  const dim3 block(kWave * block_waves(W));
  hipLaunchKernelGGL((act_quant_kernel<XT, W, VPL, TILED, MLGRU>), grid, block, 0, stream, static_cast<const XT*>(a.x),
                     a.gamma, a.q, a.a_scale, a.q_rowsum, a.rstd, a.M, a.K, a.step);
  return hipGetLastError();
}
template <typename XT, int W, int VPL, bool MLGRU>
hipError_t launch_one(const Args& a, hipStream_t stream) {
  return a.tiled ? launch_kernel<XT, W, VPL, true, MLGRU>(a, stream) : launch_kernel<XT, W, VPL, false, MLGRU>(a, stream);
}

// The number of vectors per lane is the smallest compiled value that holds
// the row (loads past the row's end return zeros but cost nearly a real load
// each).
template <typename XT, int W>
hipError_t launch_w(const Args& a, int vpl, hipStream_t stream) {
  switch (vpl) {
    case 1: return launch_one<XT, W, 1, false>(a, stream);
    case 2: return launch_one<XT, W, 2, false>(a, stream);
    case 3: return launch_one<XT, W, 3, false>(a, stream);
    case 4: return launch_one<XT, W, 4, false>(a, stream);
    case 5: case 6: return launch_one<XT, W, 6, false>(a, stream);
    case 7: case 8: return launch_one<XT, W, 8, false>(a, stream);
    default: return launch_one<XT, W, 0, false>(a, stream);
  }
}

template <int W>
hipError_t launch_mlgru_w(const Args& a, int vpl, hipStream_t stream) {
  switch (vpl) {
    case 1: return launch_one<float, W, 1, true>(a, stream);
    case 2: return launch_one<float, W, 2, true>(a, stream);
    case 3: case 4: return launch_one<float, W, 4, true>(a, stream);
    default: return hipErrorInvalidValue;
  }
}

// Waves per row: one while a lane holds at most 4 vectors of the row, else 2,
// 4, 8 or 16, so that rows up to 64 x 16 x 8 vectors stay in registers (bf16
// K <= 65536, fp32 K <= 32768; read three times from memory instead, a row of
// 13824 fp32 took 16.3 us and 4096 of them 158 us, now 3.7 and 49 us).  With
// so few rows that most of the chip idles anyway, up to 4 waves share what one
// or two would hold (45 rows of 2048 bf16: 2.7 -> 2.5 us; at 256 rows it
// measured slower, 2.3 -> 2.6 us at K = 1024, as did 16 waves per row).
constexpr int64_t kFewRows = 64;
int waves_per_row(int64_t M, int nvec) {
  int w = 1;
  while (w < 4 && nvec > w * kWave * 4) w *= 2;
  while (w < 16 && nvec > w * kWave * 8) w *= 2;
  while (w < 4 && nvec > w * kWave && M <= kFewRows) w *= 2;
  return w;
}

template <typename XT>
hipError_t launch_typed(const Args& a, hipStream_t stream) {
  const int nvec = a.K / Vec<XT>::kElems;
  const int w = waves_per_row(a.M, nvec);
  const int vpl = (nvec + w * kWave - 1) / (w * kWave);
  switch (w) {
    case 1: return launch_w<XT, 1>(a, vpl, stream);
    case 2: return launch_w<XT, 2>(a, vpl, stream);
    case 4: return launch_w<XT, 4>(a, vpl, stream);
    case 8: return launch_w<XT, 8>(a, vpl, stream);
    default: return launch_w<XT, 16>(a, vpl <= 8 ? vpl : 0, stream);
  }
}

}  // namespace

hipError_t launch_act_quant(const void* x, bool x_is_f32, const float* gamma, int8_t* q,
                            float* a_scale, int32_t* q_rowsum, int64_t M, int K,
                            hipStream_t stream, float* rstd, bool tiled) {
  if (M == 0) return hipSuccess;
  const Args a{x, gamma, q, a_scale, q_rowsum, rstd, M, K, tiled, {}};
  return x_is_f32 ? launch_typed<float>(a, stream) : launch_typed<uint16_t>(a, stream);
}

bool act_quant_mlgru_fits(int K) { return K / 4 <= 16 * kWave * 4; }

hipError_t launch_act_quant_mlgru(const float* fcg, const float* h_in, float* h_out, const float* gamma, int8_t* q,
                                  float* a_scale, int32_t* q_rowsum, int64_t M, int K, hipStream_t stream,
                                  bool tiled) {
  if (M == 0) return hipSuccess;
  const Args a{nullptr, gamma, q, a_scale, q_rowsum, nullptr, M, K, tiled, {fcg, h_in, h_out}};
  // four arrays per vector: at most 4 vectors per lane
  const int nvec = K / 4;
  int w = waves_per_row(M, nvec);
  while (w < 16 && nvec > w * kWave * 4) w *= 2;
  const int vpl = (nvec + w * kWave - 1) / (w * kWave);
  switch (w) {
    case 1: return launch_mlgru_w<1>(a, vpl, stream);
    case 2: return launch_mlgru_w<2>(a, vpl, stream);
    case 4: return launch_mlgru_w<4>(a, vpl, stream);
    case 8: return launch_mlgru_w<8>(a, vpl, stream);
    default: return launch_mlgru_w<16>(a, vpl, stream);
  }
}

}  // namespace mmf

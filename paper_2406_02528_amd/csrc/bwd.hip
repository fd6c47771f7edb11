// Final sums of the BitLinear backward (Algorithm 1, backward_pass): the
// fp64 partials of column sums (db from the dY kernel's row tiles, dgamma's)
// added in a fixed order, and the fixed-order fp64 sum of the token-range
// parts of dW when its contraction is split (the two products and the
// partials themselves are in bwd_gemm.hip).
#include "mmf_device.h"
#include "mmf_launch.h"

namespace mmf {
namespace {

constexpr int kBlock = 256;

unsigned blocks_for(int64_t threads) { return static_cast<unsigned>((threads + kBlock - 1) / kBlock); }

// Two arrays of column sums in one launch (the first a_blocks workgroups are
// a's).  out[c] = sum of partials [nparts][cols] over p: 8 columns per workgroup,
// 32 lanes per column, lane l taking the partials l, l + 32, ... (their loads
// issued together), then the 32 lane sums of a column added in lane order.
// Both orders are fixed, so the result is the same bits on every call.
constexpr int kCols = 8, kLanes = kBlock / kCols;
__global__ __launch_bounds__(kBlock) void col_final_kernel(const ColSums a, const ColSums b, unsigned a_blocks) {
  __shared__ double red[kCols][kLanes + 1];
  const int c = threadIdx.x % kCols, l = threadIdx.x / kCols;
  const bool second = blockIdx.x >= a_blocks;  // uniform
  const double* partials = second ? b.partials : a.partials;
  const int64_t nparts = second ? b.nparts : a.nparts, cols = second ? b.cols : a.cols;
  float* out = second ? b.out : a.out;
  const int64_t col = static_cast<int64_t>(blockIdx.x - (second ? a_blocks : 0u)) * kCols + c;
  double acc = 0.0;
  if (col < cols) {
#pragma unroll 4
    for (int64_t p = l; p < nparts; p += kLanes) acc += partials[p * cols + col];
  }
  red[c][l] = acc;
  __syncthreads();
  if (l == 0 && col < cols) {
    double s = 0.0;
    for (int i = 0; i < kLanes; ++i) s += red[c][i];
    out[col] = static_cast<float>(s);
  }
}

// Sum of S partial products [S][n] into out [n] (n % 4 == 0), in order, in
// fp64: four elements per thread, four parts' loads in flight.
__global__ __launch_bounds__(kBlock) void sum_parts_kernel(const float* __restrict__ parts, int64_t S, int64_t n,
                                                           float* __restrict__ out) {
  const int64_t i = 4 * (static_cast<int64_t>(blockIdx.x) * kBlock + threadIdx.x);
  if (i >= n) return;
  double acc[4] = {0.0, 0.0, 0.0, 0.0};
  auto add = [&](float4 v) {
    acc[0] += static_cast<double>(v.x);
    acc[1] += static_cast<double>(v.y);
    acc[2] += static_cast<double>(v.z);
    acc[3] += static_cast<double>(v.w);
  };
  int64_t s = 0;
  for (; s + 4 <= S; s += 4) {
    float4 v[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) v[u] = *reinterpret_cast<const float4*>(parts + (s + u) * n + i);
#pragma unroll
    for (int u = 0; u < 4; ++u) add(v[u]);
  }
  for (; s < S; ++s) add(*reinterpret_cast<const float4*>(parts + s * n + i));
  *reinterpret_cast<float4*>(out + i) = make_float4(static_cast<float>(acc[0]), static_cast<float>(acc[1]),
                                                    static_cast<float>(acc[2]), static_cast<float>(acc[3]));
}

}  // namespace

hipError_t launch_col_final(const ColSums& a, const ColSums& b, hipStream_t stream) {
  const unsigned na = a.out ? static_cast<unsigned>((a.cols + kCols - 1) / kCols) : 0u;
  const unsigned nb = b.out ? static_cast<unsigned>((b.cols + kCols - 1) / kCols) : 0u;
  if (na + nb == 0) return hipSuccess;
  hipLaunchKernelGGL(col_final_kernel, dim3(na + nb), dim3(kBlock), 0, stream, a, b, na);
  return hipGetLastError();
}

hipError_t launch_sum_parts(const float* parts, int64_t S, int64_t n, float* out, hipStream_t stream) {
  if (n == 0) return hipSuccess;
  hipLaunchKernelGGL(sum_parts_kernel, dim3(blocks_for(n / 4)), dim3(kBlock), 0, stream, parts, S, n, out);
  return hipGetLastError();
}

}  // namespace mmf

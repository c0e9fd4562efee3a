// Helper kernels of the runtime: clearing C before split-K accumulation, the
// plain reference product the search checks candidates against, and a
// normwise difference reduction.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstdint>

#include "aux_kernels.h"

namespace gt {
namespace {

__global__ void fill_zero_kernel(float* __restrict__ p, int64_t n) {
  const int64_t stride = static_cast<int64_t>(gridDim.x) * blockDim.x;
  for (int64_t i = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x; i < n; i += stride)
    p[i] = 0.0f;
}

__device__ __forceinline__ float load_in(const void* p, int64_t i, int dtype) {
  if (dtype == 0) return reinterpret_cast<const float*>(p)[i];
  const uint32_t bits = static_cast<uint32_t>(reinterpret_cast<const uint16_t*>(p)[i]) << 16;
  return __builtin_bit_cast(float, bits);
}

// One thread per output (grid-stride over rows and columns, so any M and N
// fit the grid's limits); k ascending, fp32 fused multiply-add. dtype 0/1
// (fp32/bf16), plus 16 when A is K-major (element (m, k) at A[k·M + m]).
__global__ void reference_kernel(const void* __restrict__ A, const void* __restrict__ B,
                                 float* __restrict__ C, int64_t M, int64_t N, int64_t K,
                                 int dtype) {
  const int dt = dtype & 15;
  const int64_t sr = (dtype & 16) ? 1 : K, sk = (dtype & 16) ? M : 1;
  const int64_t rstep = static_cast<int64_t>(gridDim.y) * blockDim.y;
  const int64_t cstep = static_cast<int64_t>(gridDim.x) * blockDim.x;
  for (int64_t row = static_cast<int64_t>(blockIdx.y) * blockDim.y + threadIdx.y; row < M;
       row += rstep)
    for (int64_t col = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x; col < N;
         col += cstep) {
      float s = 0.0f;
      for (int64_t l = 0; l < K; ++l)
        s = fmaf(load_in(A, row * sr + l * sk, dt), load_in(B, l * N + col, dt), s);
      C[row * N + col] = s;
    }
}

// out[2b], out[2b + 1] = block b's max |C − R| and max |R| as bits
// (non-negative floats order like their bit patterns; a NaN difference wins
// the max, a NaN of R alone does not count). Bound by HBM. One pair per
// block, reduced by the caller: every wavefront adding its maxima to two
// shared words with atomics took 374 µs for 2^20 elements (32,768 atomics on
// one line); this takes 29 µs per gt_compare call, copy back included, and
// 53 µs for 2^24. VEC: both arrays 16-byte aligned, four elements a load.
template <bool VEC>
__global__ void __launch_bounds__(256)
    compare_kernel(const float* __restrict__ C, const float* __restrict__ R, int64_t n,
                   unsigned* __restrict__ out) {
  unsigned ud = 0;
  float mr = 0.0f;
  auto take = [&](float c, float r) __attribute__((always_inline)) {
    ud = max(ud, __builtin_bit_cast(unsigned, fabsf(c - r)));
    mr = fmaxf(mr, fabsf(r));
  };
  const int64_t first = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x;
  const int64_t stride = static_cast<int64_t>(gridDim.x) * blockDim.x;
  if constexpr (VEC) {
    const float4* C4 = reinterpret_cast<const float4*>(C);
    const float4* R4 = reinterpret_cast<const float4*>(R);
    const int64_t n4 = n >> 2;
    auto take4 = [&](const float4& c, const float4& r) __attribute__((always_inline)) {
      take(c.x, r.x);
      take(c.y, r.y);
      take(c.z, r.z);
      take(c.w, r.w);
    };
    int64_t i = first;
    for (; i + 3 * stride < n4; i += 4 * stride) {
      float4 c[4], r[4];
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        c[u] = C4[i + u * stride];
        r[u] = R4[i + u * stride];
      }
#pragma unroll
      for (int u = 0; u < 4; ++u) take4(c[u], r[u]);
    }
    for (; i < n4; i += stride) take4(C4[i], R4[i]);
    if (first < (n & 3)) take(C[(n4 << 2) + first], R[(n4 << 2) + first]);
  } else {
    for (int64_t i = first; i < n; i += stride) take(C[i], R[i]);
  }
  unsigned ur = __builtin_bit_cast(unsigned, mr);
  for (int off = 32; off > 0; off >>= 1) {
    ud = max(ud, static_cast<unsigned>(__shfl_xor(static_cast<int>(ud), off)));
    ur = max(ur, static_cast<unsigned>(__shfl_xor(static_cast<int>(ur), off)));
  }
  __shared__ unsigned part[4][2];
  if ((threadIdx.x & 63) == 0) {
    part[threadIdx.x >> 6][0] = ud;
    part[threadIdx.x >> 6][1] = ur;
  }
  __syncthreads();
  if (threadIdx.x < 2)
    out[2 * blockIdx.x + threadIdx.x] = max(max(part[0][threadIdx.x], part[1][threadIdx.x]),
                                            max(part[2][threadIdx.x], part[3][threadIdx.x]));
}

}  // namespace

hipError_t launch_fill_zero(float* p, int64_t n, hipStream_t s) {
  if (n <= 0) return hipSuccess;
  const int64_t blocks = (n + 255) / 256;
  const unsigned g = static_cast<unsigned>(blocks < 65536 ? blocks : 65536);
  hipLaunchKernelGGL(fill_zero_kernel, dim3(g), dim3(256), 0, s, p, n);
  return hipGetLastError();
}

hipError_t launch_reference(const void* A, const void* B, float* C, int64_t M, int64_t N, int64_t K,
                            int dtype, hipStream_t s) {
  if (M <= 0 || N <= 0) return hipSuccess;  // an empty C: nothing to write
  const dim3 block(64, 4);
  // grid.y is limited to 65535 blocks; the kernel strides over what is left
  const dim3 grid(static_cast<unsigned>(std::min<int64_t>((N + 63) / 64, int64_t{1} << 20)),
                  static_cast<unsigned>(std::min<int64_t>((M + 3) / 4, 65535)));
  hipLaunchKernelGGL(reference_kernel, grid, block, 0, s, A, B, C, M, N, K, dtype);
  return hipGetLastError();
}

hipError_t launch_compare(const float* C, const float* R, int64_t n, unsigned* out, int* blocks,
                          hipStream_t s) {
  // 16 elements a thread where that fills the partial-result array or less
  const int64_t want = (n + 4095) / 4096;
  *blocks = static_cast<int>(std::max<int64_t>(1, std::min<int64_t>(want, kCompareBlocks)));
  const bool vec = ((reinterpret_cast<uintptr_t>(C) | reinterpret_cast<uintptr_t>(R)) & 15u) == 0;
  const dim3 grid(static_cast<unsigned>(*blocks)), block(256);
  if (vec)
    hipLaunchKernelGGL(compare_kernel<true>, grid, block, 0, s, C, R, n, out);
  else
    hipLaunchKernelGGL(compare_kernel<false>, grid, block, 0, s, C, R, n, out);
  return hipGetLastError();
}

}  // namespace gt

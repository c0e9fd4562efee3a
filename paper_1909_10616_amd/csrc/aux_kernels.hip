// Helper kernels of the runtime: clearing C before split-K accumulation, the
// plain reference product the search checks candidates against, and a
// normwise difference reduction.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstdint>
#include <type_traits>

#include "aux_kernels.h"

namespace gt {
namespace {

// Clears C before a split-K launch. Bound by its launch up to about 4 MiB and
// by the memory beyond; with 16 bytes a lane instead of 4 (VEC: p is 16-byte
// aligned) 1 MiB took 2.0 µs instead of 2.2, 4 MiB 2.5 instead of 3.0, 64 MiB
// 10.3 instead of 17.8 (6.5 TB/s).
template <bool VEC>
__global__ void __launch_bounds__(256) fill_zero_kernel(float* __restrict__ p, int64_t n) {
  const int64_t first = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x;
  const int64_t stride = static_cast<int64_t>(gridDim.x) * blockDim.x;
  if constexpr (VEC) {
    float4* const p4 = reinterpret_cast<float4*>(p);
    const int64_t n4 = n >> 2;
    for (int64_t i = first; i < n4; i += stride) p4[i] = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
    if (first < (n & 3)) p[(n4 << 2) + first] = 0.0f;
  } else {
    for (int64_t i = first; i < n; i += stride) p[i] = 0.0f;
  }
}

__device__ __forceinline__ float load_in(const void* p, int64_t i, int dtype) {
  if (dtype == 0) return reinterpret_cast<const float*>(p)[i];
  const uint32_t bits = static_cast<uint32_t>(reinterpret_cast<const uint16_t*>(p)[i]) << 16;
  return __builtin_bit_cast(float, bits);
}

// The check product: a T×T tile of C per 256 threads (16×16, each thread
// R = T/16 rows and columns of it), K in chunks of KC through LDS as fp32.
// Every output is one chain of fp32 fused multiply-adds with k ascending,
// whatever the tile, so the values do not depend on it. It stays off the
// matrix cores: what it checks runs there.
// It takes about the sum of its FMAs and of the LDS reads that feed them: R·R FMAs
// a lane against 2·R LDS values per k, which for the 128×128 tile, four
// wavefronts and one k is 136 cycles of a CU's FMAs (a register-only loop of
// v_fmac_f32 reaches 148 TFLOP/s from two wavefronts a SIMD on) and 128 of its LDS
// (128 bytes a cycle). 4096³ bf16: 42.6 ms with one thread per output reading
// A and B through the caches, 1.75 ms (78 TFLOP/s, half of that loop) with
// 128×128 tiles; 1024³ 0.47 -> 0.08 ms. Rows,
// columns and k past the edges are clamped for the loads (any size, any
// alignment, scalar coalesced loads: 2·T·KC of them per T·T·KC FMAs) and
// their products are not formed (k) or not stored (rows, columns).
// AK: A is K-major (element (m, k) at A[k·M + m]).
constexpr int kRefKC = 16;

template <int DT, bool AK, int T>
__global__ void __launch_bounds__(256)
    reference_kernel(const void* __restrict__ Av, const void* __restrict__ Bv,
                     float* __restrict__ C, int64_t M, int64_t N, int64_t K, int64_t tilesN,
                     int64_t tiles) {
  constexpr int KC = kRefKC, R = T / 16, LD = T + 4, NL = T * KC / 256;
  constexpr int V = R < 4 ? R : 4, NV = R / V;  // a thread's rows: NV runs of V, T/NV apart
  __shared__ __align__(16) float as[2][KC][LD], bs[2][KC][LD];
  const int tid = threadIdx.x, tx = tid & 15, ty = tid >> 4;
  constexpr int KS = 256 / T;  // k rows one pass of [k][T] loads covers
  for (int64_t tile = blockIdx.x; tile < tiles; tile += gridDim.x) {
    const int64_t row0 = tile / tilesN * T, col0 = tile % tilesN * T;
    // element offsets of this thread's loads at k = 0; load i of a chunk is
    // row (tid / 16) + 16·i, k tid % 16 of a row-major A, and column tid % T,
    // k tid / T + KS·i of B (and of a K-major A)
    const int64_t bcol = min(col0 + tid % T, N - 1);
    int64_t arow[AK ? 1 : NL];
    if constexpr (AK) {
      arow[0] = min(row0 + tid % T, M - 1);
    } else {
#pragma unroll
      for (int i = 0; i < NL; ++i) arow[i] = min(row0 + ty + 16 * i, M - 1) * K;
    }
    float ra[NL], rb[NL];
    auto gload = [&](int64_t k0) __attribute__((always_inline)) {
#pragma unroll
      for (int i = 0; i < NL; ++i) {
        const int64_t kb = min(k0 + tid / T + KS * i, K - 1);
        rb[i] = load_in(Bv, kb * N + bcol, DT);
        if constexpr (AK)
          ra[i] = load_in(Av, kb * M + arow[0], DT);
        else
          ra[i] = load_in(Av, arow[i] + min(k0 + tx, K - 1), DT);
      }
    };
    auto lstore = [&](int buf) __attribute__((always_inline)) {
#pragma unroll
      for (int i = 0; i < NL; ++i) {
        bs[buf][tid / T + KS * i][tid % T] = rb[i];
        if constexpr (AK)
          as[buf][tid / T + KS * i][tid % T] = ra[i];
        else
          as[buf][tx][ty + 16 * i] = ra[i];
      }
    };
    float acc[R][R];
#pragma unroll
    for (int i = 0; i < R; ++i)
#pragma unroll
      for (int j = 0; j < R; ++j) acc[i][j] = 0.0f;
    auto step = [&](int buf, int kk) __attribute__((always_inline)) {
      float a[R], b[R];
#pragma unroll
      for (int v = 0; v < NV; ++v) {
        __builtin_memcpy(a + v * V, &as[buf][kk][v * (T / NV) + ty * V], V * 4);
        __builtin_memcpy(b + v * V, &bs[buf][kk][v * (T / NV) + tx * V], V * 4);
      }
#pragma unroll
      for (int i = 0; i < R; ++i)
#pragma unroll
        for (int j = 0; j < R; ++j) acc[i][j] = fmaf(a[i], b[j], acc[i][j]);
    };
    gload(0);
    lstore(0);
    __syncthreads();
    int buf = 0;
    int64_t k0 = 0;
    for (; k0 + KC < K; k0 += KC, buf ^= 1) {
      gload(k0 + KC);
#pragma unroll
      for (int kk = 0; kk < KC; ++kk) step(buf, kk);
      lstore(buf ^ 1);
      __syncthreads();
    }
    const int left = static_cast<int>(K - k0);
    for (int kk = 0; kk < left; ++kk) step(buf, kk);
    __syncthreads();  // the next tile's first store reuses a buffer
#pragma unroll
    for (int i = 0; i < R; ++i) {
      const int64_t r = row0 + i / V * (T / NV) + ty * V + i % V;
#pragma unroll
      for (int j = 0; j < R; ++j) {
        const int64_t c = col0 + j / V * (T / NV) + tx * V + j % V;
        if (r < M && c < N) C[r * N + c] = acc[i][j];
      }
    }
  }
}

// The same for a C of few rows and many columns, where a square tile is mostly
// empty: a thread per column and kThinRows rows (blockIdx.y steps over them), B
// read once per that many rows, A by broadcast. The same chain per output.
// Bound by B's bytes and the launch.
constexpr int kThinRows = 4;

template <int DT, bool AK>
__global__ void __launch_bounds__(256)
    reference_thin_kernel(const void* __restrict__ Av, const void* __restrict__ Bv,
                          float* __restrict__ C, int64_t M, int64_t N, int64_t K) {
  constexpr int U = 8;  // k per round of loads
  const int64_t row0 = static_cast<int64_t>(blockIdx.y) * kThinRows;
  int64_t arow[kThinRows];
#pragma unroll
  for (int r = 0; r < kThinRows; ++r) arow[r] = min(row0 + r, M - 1) * (AK ? 1 : K);
  const int64_t stride = static_cast<int64_t>(gridDim.x) * blockDim.x;
  for (int64_t col = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x; col < N;
       col += stride) {
    float acc[kThinRows] = {};
    auto step = [&](int64_t k, float b) __attribute__((always_inline)) {
#pragma unroll
      for (int r = 0; r < kThinRows; ++r)
        acc[r] = fmaf(load_in(Av, arow[r] + k * (AK ? M : 1), DT), b, acc[r]);
    };
    int64_t k = 0;
    for (; k + U <= K; k += U) {
      float b[U];
#pragma unroll
      for (int u = 0; u < U; ++u) b[u] = load_in(Bv, (k + u) * N + col, DT);
#pragma unroll
      for (int u = 0; u < U; ++u) step(k + u, b[u]);
    }
    for (; k < K; ++k) step(k, load_in(Bv, k * N + col, DT));
#pragma unroll
    for (int r = 0; r < kThinRows; ++r)
      if (row0 + r < M) C[(row0 + r) * N + col] = acc[r];
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
  const bool vec = (reinterpret_cast<uintptr_t>(p) & 15u) == 0;
  const int64_t blocks = vec ? (n / 4 + 256) / 256 : (n + 255) / 256;
  const dim3 grid(static_cast<unsigned>(std::min<int64_t>(blocks, 65536))), block(256);
  if (vec)
    hipLaunchKernelGGL(fill_zero_kernel<true>, grid, block, 0, s, p, n);
  else
    hipLaunchKernelGGL(fill_zero_kernel<false>, grid, block, 0, s, p, n);
  return hipGetLastError();
}

namespace {

template <int DT, bool AK>
void launch_reference_tiled(const void* A, const void* B, float* C, int64_t M, int64_t N, int64_t K,
                            hipStream_t s) {
  // The largest tile that gives more than one workgroup for most of the 256
  // compute units, else the smallest: one workgroup alone on a CU is one
  // wavefront a SIMD, which waits for LDS. 256 tiles against four times as many
  // of half the size: 1024³ 107 and 79 µs, 2048³ 365 and 290 µs; 418 tiles
  // (1360×1200×720) 78 and 91 µs.
  constexpr int64_t kEnough = 384;
  // Up to 8 rows against at least a column per thread of one workgroup a CU:
  // 1×1000003 with K = 1 the tiles took 28 µs, one thread per output 8 and the
  // thin form 6; 4×1000003 with K = 64 187, 197 and 44; 8×65536 with K = 4096
  // (fp32) 818, 1841 and 330. Up to 16 rows where K is short: 16×1000003 with
  // K = 1 37, 33 and 18; with K = 256 720, 3631 and 775. At 16384 columns and
  // K = 4096 it is the tiles: 4 rows (K-major) 191, 1117 and 297.
  if (N >= 65536 && (M <= 8 || (M <= 16 && K <= 64))) {
    const dim3 grid(static_cast<unsigned>(std::min<int64_t>((N + 255) / 256, int64_t{1} << 20)),
                    static_cast<unsigned>((M + kThinRows - 1) / kThinRows));
    hipLaunchKernelGGL((reference_thin_kernel<DT, AK>), grid, dim3(256), 0, s, A, B, C, M, N, K);
    return;
  }
  const auto tiles = [&](int64_t t) { return (M + t - 1) / t * ((N + t - 1) / t); };
  const auto run = [&](auto tag) {
    constexpr int T = decltype(tag)::value;
    const int64_t nt = tiles(T);
    const dim3 grid(static_cast<unsigned>(std::min<int64_t>(nt, int64_t{1} << 20)));
    hipLaunchKernelGGL((reference_kernel<DT, AK, T>), grid, dim3(256), 0, s, A, B, C, M, N, K,
                       (N + T - 1) / T, nt);
  };
  if (tiles(128) >= kEnough)
    run(std::integral_constant<int, 128>{});
  else if (tiles(64) >= kEnough)
    run(std::integral_constant<int, 64>{});
  else
    run(std::integral_constant<int, 32>{});
}

}  // namespace

hipError_t launch_reference(const void* A, const void* B, float* C, int64_t M, int64_t N, int64_t K,
                            int dtype, hipStream_t s) {
  if (M <= 0 || N <= 0) return hipSuccess;  // an empty C: nothing to write
  const bool ak = (dtype & 16) != 0;
  if ((dtype & 15) == 0)
    ak ? launch_reference_tiled<0, true>(A, B, C, M, N, K, s)
       : launch_reference_tiled<0, false>(A, B, C, M, N, K, s);
  else
    ak ? launch_reference_tiled<1, true>(A, B, C, M, N, K, s)
       : launch_reference_tiled<1, false>(A, B, C, M, N, K, s);
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

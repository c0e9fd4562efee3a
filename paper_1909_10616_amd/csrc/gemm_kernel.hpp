// Tiling-parameterised GEMM kernel family for gfx950 (CDNA4).
//
// C (M×N, fp32, row-major) = A (M×K, row-major) · B (K×N, row-major), the
// operator whose loop-tiling configuration the search tunes (§3.2, §3.3).
// A configuration's levels map to the launch as follows (level 0 outermost):
//   rows    = ((gridM·wavesM + wm)·repM + rep)·blkM + b
//   k index = ((kLoop·kSplit + z)·kSub + s)·kBlk + b
// Compile-time parameters: input dtype, MFMA size I (16/32), MFMA tiles per
// wavefront TM × TN, and the path:
//   generic — any legitimate configuration: wavefronts that read their own
//             operands (gemm_stream), or, where blocks, alignment or LDS do not
//             allow that, stages shared through LDS in the natural row-major
//             layout, blocks smaller than the MFMA instruction zero-padded in
//             registers (gemm_generic);
//   fast    — blocks that are multiples of the instruction, direct
//             global→LDS loads into a ring of stages: gemm_fast_dl for bf16
//             stages whose loads divide evenly over the wavefronts into the
//             counts it is built for, gemm_ring for all others and for fp32.
// Everything else (grid, waves, block extents, stage depth, split-K, double
// buffering) is a runtime argument.
#pragma once
#include <hip/hip_runtime.h>

#include <atomic>
#include <cstdint>
#include <type_traits>

namespace gt {

struct KArgs {
  const void* A;
  const void* B;
  float* C;
  int64_t M, N, K;
  int32_t gridM, gridN;
  int32_t wavesM, wavesN;
  int32_t blkM, blkN;
  int32_t lgTpbM, lgTpbN;  // log2 of MFMA tiles per block (blk ≥ I) else 0
  int32_t kLoop, kSplit, kSub, kBlk;
  int32_t BM, BN, BK;
  int32_t WM, WN;          // wavefront tile
  int32_t lgBK, lgBN;
  int32_t dbuf;
  int32_t atomic;          // split-K: accumulate with fp32 atomics
  int32_t remap;           // XCD-aware workgroup order
  int32_t aVec, bVec;      // generic path: 1 or 16-byte vector tile loads
  int32_t dl;              // bf16 fast path: loads in whole equal shares (reported only)
  int32_t dlk;             // … that gemm_fast_dl takes
  int32_t ns;              // ring stages (fast path)
  int32_t aKM;             // A given K-major (K×M row-major, element (m, k) at A[k·M + m])
  int32_t lgBM;
  int32_t stream;          // generic path: wavefronts read their own operands
  int32_t wide;            // gemm_ring: a stage's offsets from its origins exceed 32 bits,
                           // the loads step 64-bit addresses
};

typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
// A 16-byte chunk as a native vector (HIP's u32x4 struct is copied by memcpy,
// which keeps staging arrays out of registers).
typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));

template <int DT>
struct Elem;
template <>
struct Elem<0> {  // fp32
  using T = float;
  static constexpr int VEC = 4;  // elements per 16-byte chunk
  static constexpr int EPL = 1;  // elements per lane per MFMA operand
};
template <>
struct Elem<1> {  // bf16 (stored as raw 16-bit patterns)
  using T = uint16_t;
  static constexpr int VEC = 8;
  static constexpr int EPL = 8;
};

template <int I>
struct AccT;
template <>
struct AccT<32> {
  using type = f32x16;
  static constexpr int N = 16;
};
template <>
struct AccT<16> {
  using type = f32x4;
  static constexpr int N = 4;
};

// Row (inside the I×I output tile) of accumulator element i held by lane;
// the column is lane % I.
template <int I>
__device__ __forceinline__ int out_row(int lane, int i) {
  if constexpr (I == 32)
    return 8 * (i >> 2) + 4 * (lane >> 5) + (i & 3);
  else
    return 4 * (lane >> 4) + i;
}

__device__ __forceinline__ f32x16 mfma_bf16(bf16x8 a, bf16x8 b, f32x16 c) {
  return __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b, c, 0, 0, 0);
}
__device__ __forceinline__ f32x4 mfma_bf16(bf16x8 a, bf16x8 b, f32x4 c) {
  return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, c, 0, 0, 0);
}
__device__ __forceinline__ f32x16 mfma_f32(float a, float b, f32x16 c) {
  return __builtin_amdgcn_mfma_f32_32x32x2f32(a, b, c, 0, 0, 0);
}
__device__ __forceinline__ f32x4 mfma_f32(float a, float b, f32x4 c) {
  return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
}

// Workgroup → (tile row, tile column). Consecutive workgroups are dispatched
// round-robin over the 8 XCDs; with `remap` each XCD receives a contiguous
// run of tiles, ordered in groups of 4 tile rows so that the tiles sharing
// an XCD's L2 share A row-blocks and B column-blocks.
__device__ __forceinline__ void tile_of(const KArgs& a, int& gm, int& gn) {
  const int nt = a.gridM * a.gridN;
  int t = static_cast<int>(blockIdx.x);
  if (a.remap) t = (t & 7) * (nt >> 3) + (t >> 3);
  constexpr int G = 4;
  const int per_group = G * a.gridN;
  const int group = t / per_group;
  const int first = group * G;
  const int gsize = min(a.gridM - first, G);
  const int r = t - group * per_group;
  gm = first + r % gsize;
  gn = r / gsize;
}

__device__ __forceinline__ void put(bool atomic, float* p, float v) {
  if (atomic)
    unsafeAtomicAdd(p, v);
  else
    *p = v;
}

// Writes a wavefront's accumulators: TM × TN tiles of I×I from Cw, the
// wavefront tile's origin in C. One 64-bit address per row, stepped by N, and
// one branch for the atomic form: with the address and the branch of every
// element worked out on its own, an element cost about ten instructions.
template <int I, int TM, int TN, typename acc_t>
__device__ __forceinline__ void store_tile(const KArgs& a, float* Cw, int lane,
                                           const acc_t (&acc)[TM][TN]) {
  const int64_t N = a.N;
  float* const first = Cw + static_cast<int64_t>(out_row<I>(lane, 0)) * N + lane % I;
  auto rows = [&](auto put_one) __attribute__((always_inline)) {
    float* p = first;
#pragma unroll
    for (int i = 0; i < TM; ++i) {
#pragma unroll
      for (int e = 0; e < AccT<I>::N; ++e) {
#pragma unroll
        for (int j = 0; j < TN; ++j) put_one(p + j * I, acc[i][j][e]);
        // the lane's next row: the accumulator's, or the next tile's first
        const int here = out_row<I>(0, e);
        p += (e + 1 < AccT<I>::N ? out_row<I>(0, e + 1) - here : I - here) * N;
      }
    }
  };
  if (a.atomic)
    rows([](float* p, float v) __attribute__((always_inline)) { unsafeAtomicAdd(p, v); });
  else
    rows([](float* p, float v) __attribute__((always_inline)) { *p = v; });
}

// ---------------------------------------------------------------------------
// Generic path
// ---------------------------------------------------------------------------

template <typename T, int VEC>
__device__ __forceinline__ void copy_tile(T* lds, const T* g, int64_t ld, int rows, int cols,
                                          int lgcols, int vec, int tid, int nthr) {
  if (vec > 1) {
    constexpr int LGV = VEC == 8 ? 3 : 2;
    const int lgcpr = lgcols - LGV;
    const int chunks = (rows * cols) >> LGV;
    for (int e = tid; e < chunks; e += nthr) {
      const int r = e >> lgcpr;
      const int c = (e & ((1 << lgcpr) - 1)) << LGV;
      *reinterpret_cast<u32x4*>(lds + (r << lgcols) + c) =
          *reinterpret_cast<const u32x4*>(g + r * ld + c);
    }
  } else {
    const int total = rows * cols;
    for (int e = tid; e < total; e += nthr) {
      const int r = e >> lgcols;
      const int c = e & (cols - 1);
      lds[e] = g[r * ld + c];
    }
  }
}

template <int DT, int I, int TM, int TN>
__device__ void gemm_generic(const KArgs& a, char* smem) {
  using T = typename Elem<DT>::T;
  using acc_t = typename AccT<I>::type;
  constexpr int NACC = AccT<I>::N;
  constexpr int EPL = Elem<DT>::EPL;
  constexpr int G = 64 / I;
  constexpr int IK = EPL * G;
  const int tid = threadIdx.x;
  const int nthr = blockDim.x;
  const int lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = wave % a.wavesM;
  const int wn = wave / a.wavesM;
  int gm, gn;
  tile_of(a, gm, gn);
  const int z = blockIdx.y;

  T* As0 = reinterpret_cast<T*>(smem);
  const int stage = (a.BM + a.BN) * a.BK;
  // A K-major: the tile is BK rows of BM contiguous m, kept as [k][m] in LDS
  const bool akm = a.aKM != 0;
  const T* Ag = reinterpret_cast<const T*>(a.A) +
                (akm ? static_cast<int64_t>(gm) * a.BM : static_cast<int64_t>(gm) * a.BM * a.K);
  const T* Bg = reinterpret_cast<const T*>(a.B) + static_cast<int64_t>(gn) * a.BN;
  // LDS element offsets of A (row r, k) = r·sr + k·sk
  const int sr = akm ? 1 : a.BK, sk = akm ? a.BM : 1;

  // Rows of A / columns of B this lane feeds into each MFMA tile.
  int arow[TM], bcol[TN];
  bool aok[TM], bok[TN];
  const int tpbM = 1 << a.lgTpbM, tpbN = 1 << a.lgTpbN;
#pragma unroll
  for (int t = 0; t < TM; ++t) {
    const int in = (t & (tpbM - 1)) * I + (lane % I);
    aok[t] = in < a.blkM;
    arow[t] = wm * a.WM + (t >> a.lgTpbM) * a.blkM + in;
  }
#pragma unroll
  for (int t = 0; t < TN; ++t) {
    const int in = (t & (tpbN - 1)) * I + (lane % I);
    bok[t] = in < a.blkN;
    bcol[t] = wn * a.WN + (t >> a.lgTpbN) * a.blkN + in;
  }

  acc_t acc[TM][TN];
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j) acc[i][j] = acc_t{};

  auto load_stage = [&](int l, int buf) __attribute__((always_inline)) {
    const int64_t kbase = (static_cast<int64_t>(l) * a.kSplit + z) * a.BK;
    T* as = As0 + buf * stage;
    T* bs = as + a.BM * a.BK;
    if (akm)
      copy_tile<T, Elem<DT>::VEC>(as, Ag + kbase * a.M, a.M, a.BK, a.BM, a.lgBM, a.aVec, tid, nthr);
    else
      copy_tile<T, Elem<DT>::VEC>(as, Ag + kbase, a.K, a.BM, a.BK, a.lgBK, a.aVec, tid, nthr);
    copy_tile<T, Elem<DT>::VEC>(bs, Bg + kbase * a.N, a.N, a.BK, a.BN, a.lgBN, a.bVec, tid, nthr);
  };

  auto compute = [&](int buf) __attribute__((always_inline)) {
    const T* as = As0 + buf * stage;
    const T* bs = as + a.BM * a.BK;
    const int nkk = (a.kBlk + IK - 1) / IK;
    for (int s = 0; s < a.kSub; ++s) {
      for (int kk = 0; kk < nkk; ++kk) {
        const int kl0 = kk * IK + (lane / I) * EPL;  // this lane's first k in the sub-step
        if constexpr (DT == 1) {
          bf16x8 af[TM], bfv[TN];
#pragma unroll
          for (int t = 0; t < TM; ++t) {
            uint16_t v[8];
#pragma unroll
            for (int e = 0; e < 8; ++e) {
              const int kl = kl0 + e;
              v[e] = (aok[t] && kl < a.kBlk) ? as[arow[t] * sr + (s * a.kBlk + kl) * sk] : uint16_t(0);
            }
            af[t] = __builtin_bit_cast(bf16x8, v);
          }
#pragma unroll
          for (int t = 0; t < TN; ++t) {
            uint16_t v[8];
#pragma unroll
            for (int e = 0; e < 8; ++e) {
              const int kl = kl0 + e;
              v[e] = (bok[t] && kl < a.kBlk) ? bs[(s * a.kBlk + kl) * a.BN + bcol[t]] : uint16_t(0);
            }
            bfv[t] = __builtin_bit_cast(bf16x8, v);
          }
#pragma unroll
          for (int i = 0; i < TM; ++i)
#pragma unroll
            for (int j = 0; j < TN; ++j) acc[i][j] = mfma_bf16(af[i], bfv[j], acc[i][j]);
        } else {
          float af[TM], bfv[TN];
          const bool kin = kl0 < a.kBlk;
#pragma unroll
          for (int t = 0; t < TM; ++t)
            af[t] = (aok[t] && kin) ? as[arow[t] * sr + (s * a.kBlk + kl0) * sk] : 0.0f;
#pragma unroll
          for (int t = 0; t < TN; ++t)
            bfv[t] = (bok[t] && kin) ? bs[(s * a.kBlk + kl0) * a.BN + bcol[t]] : 0.0f;
#pragma unroll
          for (int i = 0; i < TM; ++i)
#pragma unroll
            for (int j = 0; j < TN; ++j) acc[i][j] = mfma_f32(af[i], bfv[j], acc[i][j]);
        }
      }
    }
  };

  load_stage(0, 0);
  __syncthreads();
  for (int l = 0; l < a.kLoop; ++l) {
    const int cur = a.dbuf ? (l & 1) : 0;
    const bool next = l + 1 < a.kLoop;
    if (a.dbuf && next) load_stage(l + 1, cur ^ 1);
    compute(cur);
    __syncthreads();
    if (!a.dbuf && next) {
      load_stage(l + 1, 0);
      __syncthreads();
    }
  }

  float* Cw = a.C + static_cast<int64_t>(gm) * a.BM * a.N + static_cast<int64_t>(gn) * a.BN;
#pragma unroll
  for (int i = 0; i < TM; ++i) {
#pragma unroll
    for (int j = 0; j < TN; ++j) {
#pragma unroll
      for (int e = 0; e < NACC; ++e) {
        const int ri = (i & (tpbM - 1)) * I + out_row<I>(lane, e);
        const int ci = (j & (tpbN - 1)) * I + (lane % I);
        if (ri < a.blkM && ci < a.blkN) {
          const int r = wm * a.WM + (i >> a.lgTpbM) * a.blkM + ri;
          const int c = wn * a.WN + (j >> a.lgTpbN) * a.blkN + ci;
          put(a.atomic != 0, Cw + static_cast<int64_t>(r) * a.N + c, acc[i][j][e]);
        }
      }
    }
  }
}

// 16-byte chunk q of a tile → its LDS slot: XOR inside each 128-byte line
// (8 chunks) with a hash of the line index, so that the 8 or 16 lanes served
// together by a 16-byte LDS read hit distinct banks.
__device__ __forceinline__ int swz(int q) { return q ^ (((q >> 3) ^ (q >> 6)) & 7); }

template <int V>
constexpr int ilog2c() {
  return V <= 1 ? 0 : 1 + ilog2c<V / 2>();
}

// ---------------------------------------------------------------------------
// Fast path with direct global→LDS loads (bf16)
// ---------------------------------------------------------------------------
//
// Each global_load_lds_dwordx4 of a wavefront writes 64 consecutive 16-byte
// LDS slots (lane j → slot base + j) from 64 per-lane global addresses, so
// tiles reach LDS without passing through registers and a ring of ns stages
// keeps ns − 1 stages of loads in flight. A sits in LDS as [m][k] chunks,
// XOR-swizzled by swz(); with 16×16 MFMA and stages of two or more
// chunk-steps (64- and 128-deep) it is split into planes instead, one per
// chunk-step: plane cs holds the G = 4 chunks that step reads of every one of
// the BM rows, as [m][4] swizzled by swz(). Each fragment read then covers
// one aligned 1 KiB block, which the 16-byte LDS reads serve without bank
// conflicts; the stage-wide layout conflicts 2-way at those depths (with
// 32×32 MFMA, or 32-deep stages, it does not, and is kept). B stays [k][n]
// with the chunks of row k XOR-ed by bswz(k), and its MFMA operands are read
// with the transposing LDS read: inside a 16-lane group, lane l receives
// element (l & 3) of the 8 bytes addressed by lane 4j + (l >> 2) as its j-th
// value, so lanes addressing rows k0 + (i >> 2), columns n0 + 4(i & 3) hand
// lane l four consecutive k of column n0 + l.

typedef short s16x4 __attribute__((ext_vector_type(4)));
// Direct-load instructions per wavefront and stage the kernel keeps offsets
// for: 8 where the accumulator size admits 8 wavefronts (the register budget
// per lane is then 256), 16 otherwise.
constexpr int dl_inst_cap(int64_t acc) { return acc + 96 <= 256 ? 8 : 16; }

// Whether the main loop writes a load's m0 ahead of the MFMA that the load
// follows (ni: loads per wavefront and stage that the loop is built for, tiles:
// MFMAs a chunk-step). With s_nop between two MFMAs instead, 256×256×32 tiles (32
// MFMAs) lose 1 to 3 % (three boxes: 4096³ 112.2 against 111.2, 115.5 against
// 112.7 µs, 2.08 M cycles a launch against 2.01 M; 4096×11008×4096 328 against 323,
// 323 against 317 µs) and 16 MFMAs up to 0.5 %; with 2 and 4 the nop is the faster
// (64×4096×4096 13.7 against 13.9 µs, 128×2624×3456 28.6 against 31.0 µs).
constexpr bool dl_split(int ni, int tiles) { return ni > 0 && tiles >= 16; }

// XOR applied to the 16-byte chunk index of B row k in LDS. A transposing
// read touches rows k0 … k0+3 (k0 ≡ 0 mod 4) and, per 16-lane group, two
// adjacent chunks (four per 32 lanes with 32×32 MFMA; with 16×16 MFMA the
// second 16-lane group reads rows k0+8 … k0+11 instead). f(k mod 4) ∈
// {0, 6, 10, 12}, XOR-ed with 8 when bit 3 of k is set, sends those accesses
// to distinct 16-byte bank slots mod 128 B (16 lanes) and mod 256 B (32 lanes).
__device__ __forceinline__ int bswz(int k, int cprb) {
  const int j = k & 3;
  return (((j << 2) | (((j ^ (j >> 1)) & 1) << 1)) ^ (((k >> 3) & 1) << 3)) & (cprb - 1);
}

// vmcnt field of s_waitcnt on gfx9: bits [3:0] and [15:14]; lgkmcnt [11:8], expcnt [6:4].
template <int N>
__device__ __forceinline__ void waitcnt_vm() {
  __builtin_amdgcn_s_waitcnt((N & 15) | ((N >> 4) << 14) | (0x7 << 4) | (0xf << 8));
}

__device__ __forceinline__ void waitcnt_lgkm0() {
  __builtin_amdgcn_s_waitcnt(0xf | (0x3 << 14) | (0x7 << 4));  // lgkmcnt(0) only
}

// s_waitcnt takes its count as an immediate: wait for the largest of
// {0, 1, 2, 3, 4, 6, 8, 12, 16, 24, 32, 48} that is at most n (a uniform
// value), chosen by a balanced comparison tree.
__device__ __forceinline__ void wait_vm_at_most(int n) {
  if (n >= 12) {
    if (n >= 24) {
      if (n >= 48) waitcnt_vm<48>();
      else if (n >= 32) waitcnt_vm<32>();
      else waitcnt_vm<24>();
    } else {
      if (n >= 16) waitcnt_vm<16>();
      else waitcnt_vm<12>();
    }
  } else if (n >= 4) {
    if (n >= 8) waitcnt_vm<8>();
    else if (n >= 6) waitcnt_vm<6>();
    else waitcnt_vm<4>();
  } else {
    if (n >= 2) {
      if (n >= 3) waitcnt_vm<3>();
      else waitcnt_vm<2>();
    } else if (n >= 1) {
      waitcnt_vm<1>();
    } else {
      waitcnt_vm<0>();
    }
  }
}

// One 16-byte-per-lane direct global→LDS load: lane j reads 16 bytes at
// base + off (base uniform, off this lane's byte offset) and writes them to
// LDS byte address lds_base + 16·j. Written as inline assembly so that the
// compiler does not see an LDS write it would have to wait for before every
// LDS read (it cannot tell the ring slots apart); the ring's vmcnt accounting
// is done explicitly. A load to LDS needs one wait state after a scalar write
// of m0, which the compiler adds for its own loads but not inside an assembly
// statement: s_nop 0 here, other instructions in the forms below.
__device__ __forceinline__ void dma_load16(uint32_t off, uint64_t base, uint32_t lds_base) {
  // base and lds_base are uniform; reading them from the first lane keeps
  // them in scalar registers whatever the compiler inferred
  const uint64_t sb =
      static_cast<uint64_t>(static_cast<uint32_t>(__builtin_amdgcn_readfirstlane(static_cast<int>(base)))) |
      (static_cast<uint64_t>(static_cast<uint32_t>(
           __builtin_amdgcn_readfirstlane(static_cast<int>(base >> 32))))
       << 32);
  asm volatile("s_mov_b32 m0, %2\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, %1"
               :
               : "v"(off), "s"(sb), "s"(__builtin_amdgcn_readfirstlane(static_cast<int>(lds_base)))
               : "memory", "m0");
}

// The same in two parts with an MFMA between them, which is the wait state and
// hides the write of m0. Nothing else in these kernels uses m0, which the
// compiler reserves (checked on the disassembly).
__device__ __forceinline__ void dma_set_lds(uint32_t lds_base) {
  asm volatile("s_mov_b32 m0, %0"
               :
               : "s"(__builtin_amdgcn_readfirstlane(static_cast<int>(lds_base)))
               : "memory", "m0");
}
__device__ __forceinline__ void dma_load16_set(uint32_t off, uint64_t base) {
  const uint64_t sb =
      static_cast<uint64_t>(static_cast<uint32_t>(__builtin_amdgcn_readfirstlane(static_cast<int>(base)))) |
      (static_cast<uint64_t>(static_cast<uint32_t>(
           __builtin_amdgcn_readfirstlane(static_cast<int>(base >> 32))))
       << 32);
  asm volatile("global_load_lds_dwordx4 %0, %1" : : "v"(off), "s"(sb) : "memory");
}

// The same from a 64-bit address of each lane's own.
__device__ __forceinline__ void dma_load16_at(uint64_t addr, uint32_t lds_base) {
  asm volatile("s_mov_b32 m0, %1\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, off"
               :
               : "v"(addr), "s"(__builtin_amdgcn_readfirstlane(static_cast<int>(lds_base)))
               : "memory", "m0");
}

// dma_load16 when n (a uniform value) is above i, and otherwise with no lane
// enabled: the instruction then moves nothing but still counts in vmcnt, in its
// place in the order (measured: after one load of cold memory and eight masked
// ones, vmcnt(8) waited for the first in each of 4096 wavefronts). A scalar
// select instead of a branch. (The instructions after the write of m0
// are its wait state.)
__device__ __forceinline__ void dma_load16_if(int n, int i, uint32_t off, uint64_t base,
                                              uint32_t lds_base) {
  asm volatile(
      "s_mov_b32 m0, %2\n\ts_cmp_gt_i32 %3, %4\n\ts_cselect_b64 exec, -1, 0\n\t"
      "global_load_lds_dwordx4 %0, %1\n\ts_mov_b64 exec, -1"
      :
      : "v"(off), "s"(base), "s"(__builtin_amdgcn_readfirstlane(static_cast<int>(lds_base))),
        "s"(__builtin_amdgcn_readfirstlane(n)), "n"(i)
      : "memory", "m0", "scc");
}

// A wavefront-uniform pointer as a 64-bit scalar (each half taken from the
// first active lane and zero-extended).
__device__ __forceinline__ uint64_t uniform_ptr(const void* p) {
  const uint64_t b = reinterpret_cast<uintptr_t>(p);
  const uint32_t lo = static_cast<uint32_t>(__builtin_amdgcn_readfirstlane(static_cast<int>(b)));
  const uint32_t hi = static_cast<uint32_t>(__builtin_amdgcn_readfirstlane(static_cast<int>(b >> 32)));
  return static_cast<uint64_t>(lo) | (static_cast<uint64_t>(hi) << 32);
}

// Byte offset inside LDS of a pointer into the kernel's dynamic LDS.
__device__ __forceinline__ uint32_t lds_off(const void* p) {
  return static_cast<uint32_t>(reinterpret_cast<uintptr_t>(
      (const __attribute__((address_space(3))) char*)(p)));
}

// Workgroup barrier that no LDS access is moved across.
__device__ __forceinline__ void ring_barrier() {
  asm volatile("" ::: "memory");
  __builtin_amdgcn_s_barrier();
  asm volatile("" ::: "memory");
}

template <int I, int TM, int TN, int CPR>
__device__ __forceinline__ void gemm_fast_dl(const KArgs& a, char* smem) {
  using T = uint16_t;
  using acc_t = typename AccT<I>::type;
  constexpr int NACC = AccT<I>::N;
  constexpr int G = 64 / I;
  constexpr int NCS = CPR / G;
  constexpr int LGCPR = ilog2c<CPR>();
  constexpr int NLINE = CPR >= 8 ? CPR / 8 : 1;
  static_assert(NCS >= 1, "stage shallower than one MFMA K step");
  constexpr int kMaxDlInst = dl_inst_cap(TM * TN * I * I / 64);
  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int nw = blockDim.x >> 6;
  const int wm = wave % a.wavesM;
  const int wn = wave / a.wavesM;
  int gm, gn;
  tile_of(a, gm, gn);
  const int z = blockIdx.y;

  const int BM = a.BM, BN = a.BN, BK = a.BK;
  const int cprb = BN >> 3;                 // 16-byte chunks per B row
  const int achunks = BM << LGCPR;
  const int bchunks = BK * cprb;
  const int stage = achunks + bchunks;      // 16-byte slots per stage
  const int pa = achunks >> 6, pb = bchunks >> 6;
  const int ninst = (pa + pb) / nw;         // load instructions per wavefront per stage
  const int ns = a.ns;
  u32x4* lds = reinterpret_cast<u32x4*>(smem);
  const T* Ag = reinterpret_cast<const T*>(a.A) + static_cast<int64_t>(gm) * BM * a.K;
  const T* Bg = reinterpret_cast<const T*>(a.B) + static_cast<int64_t>(gn) * BN;

  // Load instruction p of a stage fills slots p·64 … p·64+63; wavefront w
  // issues p = w, w + nw, … (A instructions first, then B). Each lane works
  // out the chunk its slot holds: A slot s holds chunk swz(s) (swz is an
  // involution) of the [m][k] layout, or in the plane layout chunk-step
  // s / (4·BM) and in-plane chunk swz(s mod 4·BM) of its [m][4]; B slot
  // (k, cs) holds row k, chunk cs ^ bswz(k). The lane's byte offset from the
  // stage's A (or B) origin is the same for every stage, so it is computed
  // once (it fits 32 bits: BM·K and BK·N are below 2^31).
  constexpr bool PLANES = I == 16 && NCS >= 2;
  const int lgcprb = a.lgBN - 3;
  const int na_w = pa / nw;
  uint32_t doff[kMaxDlInst];
#pragma unroll
  for (int i = 0; i < kMaxDlInst; ++i) {
    doff[i] = 0;
    if (i < na_w) {
      if constexpr (PLANES) {
        const int s = ((wave + i * nw) << 6) + lane;
        const int lgp = a.lgBM + 2;  // slots per plane: BM·4
        const int q = swz(s & ((1 << lgp) - 1));
        doff[i] = (static_cast<uint32_t>(q >> 2) * static_cast<uint32_t>(a.K) +
                   static_cast<uint32_t>((((s >> lgp) << 2) + (q & 3)) << 3)) * 2u;
      } else {
        const int q = swz(((wave + i * nw) << 6) + lane);
        doff[i] = (static_cast<uint32_t>(q >> LGCPR) * static_cast<uint32_t>(a.K) +
                   static_cast<uint32_t>((q & (CPR - 1)) << 3)) * 2u;
      }
    } else if (i < ninst) {
      const int sidx = ((wave + (i - na_w) * nw) << 6) + lane;
      const int k = sidx >> lgcprb, cs = sidx & (cprb - 1);
      doff[i] = (static_cast<uint32_t>(k) * static_cast<uint32_t>(a.N) +
                 static_cast<uint32_t>((cs ^ bswz(k, cprb)) << 3)) * 2u;
    }
  }
  const int lds0 = __builtin_amdgcn_readfirstlane(static_cast<int>(lds_off(lds)));
  const uint32_t stage16 = static_cast<uint32_t>(stage) * 16u;  // bytes per ring slot
  // bytes between the A (B) origins of consecutive stages of this split-K slice
  const uint64_t stepA = static_cast<uint64_t>(a.kSplit) * static_cast<uint64_t>(BK) * 2u;
  const uint64_t stepB = stepA * static_cast<uint64_t>(a.N);
  // Instruction i (< ninst) of this wavefront for stage l into ring slot
  // `slot`; ga, gb: the stage's A and B origins as uniform scalars.
  // A or B is picked with scalar selects, not branches.
  auto dma = [&](uint64_t ga, uint64_t gb, uint32_t sbase, int i) __attribute__((always_inline)) {
    const bool isa = i < na_w;
    const uint32_t da = static_cast<uint32_t>(wave + i * nw) * 1024u;
    const uint32_t db = static_cast<uint32_t>(achunks + ((wave + (i - na_w) * nw) << 6)) * 16u;
    dma_load16(doff[i], isa ? ga : gb, sbase + (isa ? da : db));
  };
  // where instruction i writes (dma's lds_base)
  auto dma_lds = [&](uint32_t sbase, int i) __attribute__((always_inline)) {
    const uint32_t da = static_cast<uint32_t>(wave + i * nw) * 1024u;
    const uint32_t db = static_cast<uint32_t>(achunks + ((wave + (i - na_w) * nw) << 6)) * 16u;
    return sbase + (i < na_w ? da : db);
  };
  // Uniform origins of stage l's A and B tiles and LDS byte base of ring slot `slot`.
  struct StageBase {
    uint64_t ga, gb;
    uint32_t sb;
  };
  auto stage_base = [&](int l, int slot) __attribute__((always_inline)) {
    const int64_t kbase = (static_cast<int64_t>(l) * a.kSplit + z) * BK;
    StageBase r;
    r.ga = uniform_ptr(Ag + kbase);
    r.gb = uniform_ptr(Bg + kbase * a.N);
    r.sb = static_cast<uint32_t>(
        __builtin_amdgcn_readfirstlane(static_cast<int>(lds0 + slot * stage * 16)));
    return r;
  };
  // All of this wavefront's instructions of stage l, back to back.
  auto issue = [&](int l, int slot) __attribute__((always_inline)) {
    const StageBase b = stage_base(l, slot);
#pragma unroll
    for (int i = 0; i < kMaxDlInst; ++i)
      if (i < ninst) dma(b.ga, b.gb, b.sb, i);
  };

  acc_t acc[TM][TN];
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j) acc[i][j] = acc_t{};

  // A fragment slots: in the [m][k] layout a per-row base, to which a
  // chunk-step adds its XOR and line; in the plane layout, this lane's slot in
  // plane 0 (plane cs adds 4·BM·cs).
  const int grp = lane / I;
  int xa[TM][NLINE];
#pragma unroll
  for (int t = 0; t < TM; ++t)
#pragma unroll
    for (int j = 0; j < NLINE; ++j) {
      if constexpr (PLANES) {
        xa[t][j] = swz(((wm * a.WM + t * I + (lane % I)) << 2) + grp);
      } else {
        const int q0 = ((wm * a.WM + t * I + (lane % I)) << LGCPR) + grp + 8 * j;
        xa[t][j] = swz(q0) - 8 * j;
      }
    }
  const int plane_slots = BM << 2;
  // B operand addressing: in 16-lane group g16, input lane i covers row
  // k0 + (i >> 2) (+4 for the second read), columns n0 + 4(i & 3).
  const int i16 = lane & 15, g16 = lane >> 4;
  const int kgrp = I == 32 ? (g16 >> 1) : g16;           // which 8-k group of the step
  const int ncol0 = (I == 32 ? 16 * (g16 & 1) : 0) + 4 * (i16 & 3);
  int bcol[TN];
#pragma unroll
  for (int t = 0; t < TN; ++t) bcol[t] = wn * a.WN + t * I + ncol0;  // column of this lane's 4 values
  const int krow_l = kgrp * 8 + (i16 >> 2);

  u32x4 fa[2][TM];
  u32x4 fb[2][TN];
  auto load_frags = [&](const u32x4* as, int cs, int fs) __attribute__((always_inline)) {
    const int c = cs * G;
    const int j = CPR >= 8 ? (c >> 3) : 0;
#pragma unroll
    for (int t = 0; t < TM; ++t) {
      if constexpr (PLANES)
        fa[fs][t] = as[cs * plane_slots + xa[t][0]];
      else
        fa[fs][t] = as[(xa[t][j] ^ (c & 7)) + (c & ~7)];
    }
    const char* bs = reinterpret_cast<const char*>(as + achunks);
#pragma unroll
    for (int t = 0; t < TN; ++t) {
      s16x4 h[2];
#pragma unroll
      for (int hh = 0; hh < 2; ++hh) {
        const int k = cs * (G * 8) + krow_l + 4 * hh;
        const int col = bcol[t];
        const int chunk = (col >> 3) ^ bswz(k, cprb);
        const char* addr = bs + (k * cprb + chunk) * 16 + (col & 4) * 2;
        h[hh] = __builtin_amdgcn_ds_read_tr16_b64_v4i16(
            (__attribute__((address_space(3))) s16x4*)(addr));
      }
      fb[fs][t] = __builtin_bit_cast(u32x4, __builtin_shufflevector(h[0], h[1], 0, 1, 2, 3, 4, 5, 6, 7));
    }
  };
  auto mfma1 = [&](int fs, int q) __attribute__((always_inline)) {
    const int i = q / TN, j = q % TN;
    acc[i][j] = mfma_bf16(__builtin_bit_cast(bf16x8, fa[fs][i]),
                          __builtin_bit_cast(bf16x8, fb[fs][j]), acc[i][j]);
  };

  // Ring schedule. Stage s is loaded into slot s mod ns. Its loads are issued
  // in a window of NCS chunk-steps of MFMAs: the last chunk-step of stage
  // s − ns (which runs after the barrier that ends stage s − ns, once every
  // wavefront has stopped reading slot s mod ns) and chunk-steps 0 … NCS−2 of
  // stage s − ns + 1, so the whole set is out before the boundary that ends
  // stage s − ns + 1. Inside the window the wavefront's ninst instructions go
  // one at a time, one after every R-th MFMA: a wavefront waiting for room in
  // the memory pipeline cannot issue MFMAs, so loads go out in small doses,
  // and the last of them leaves half a chunk-step before the window closes.
  // Stages 0 … ns−2 (and the part of stage ns − 1's window that would precede
  // stage 0) are issued up front. The boundary (wait for stage l + 1, barrier,
  // first fragments of stage l + 1) sits in front of stage l's last
  // chunk-step of MFMAs.
  constexpr int TMTN = TM * TN;
  constexpr int SPOS = NCS * TMTN;  // MFMA slots in a window
  // The loop is instantiated for NI = cap and cap/2 instructions per
  // wavefront and stage (NI = 0: any other count, guarded per load), so the
  // common cases carry no per-load branch. Load i of a window goes after MFMA
  // slot i·R + R − 1 (slots past the window go out with its last slot). With
  // the full cap (the 64-deep stages of a two-slot ring, where a load has at
  // most one stage to land) the loads go out back to back from the window's
  // start (R = 1); with half the cap (the shallower stages of deeper rings)
  // they are spread over the first half of the window; otherwise they end
  // half a chunk-step before it closes. Measured at 4096³: front-loading
  // gains 3 % on the two-slot rings, spreading 3 % on the five-slot rings.
  // Both parts of every window use the same R.
  auto run = [&](auto ni) __attribute__((always_inline)) {
    constexpr int NI = decltype(ni)::value;
    constexpr int NIE = NI ? NI : kMaxDlInst;
    constexpr int RR = NI == kMaxDlInst ? 1 : (NI ? (SPOS / 2) / (NI ? NI : 1) : (SPOS - TMTN / 2) / NIE);
    constexpr int R = RR > 1 ? RR : 1;
    // open: the window is open for every load of this stage (no guard on it)
    auto dma_at = [&](const StageBase& sb, bool on, int pos, auto open) __attribute__((always_inline)) {
      constexpr bool OPEN = decltype(open)::value;
      const int i = pos / R;
      if (pos % R == R - 1 && i < NIE && i * R + R - 1 < SPOS) {
        if ((OPEN || on) && (NI > 0 || i < ninst)) {
          __builtin_amdgcn_sched_barrier(0);
          dma(sb.ga, sb.gb, sb.sb, i);
          __builtin_amdgcn_sched_barrier(0);
        }
      }
      if (pos == SPOS - 1) {
#pragma unroll
        for (int j = SPOS / R; j < NIE; ++j)
          if ((OPEN || on) && (NI > 0 || j < ninst)) dma(sb.ga, sb.gb, sb.sb, j);
      }
    };
    const int npro = min(ns - 1, a.kLoop);
    for (int l = 0; l < npro; ++l) issue(l, l);
    wait_vm_at_most(__builtin_amdgcn_readfirstlane((npro - 1) * ninst));
    __builtin_amdgcn_s_barrier();
    if (ns - 1 < a.kLoop) {
      // the part of stage ns − 1's window before stage 0 (slot ns − 1 is unused so far)
      const StageBase sb0 = stage_base(ns - 1, ns - 1);
#pragma unroll
      for (int pos = 0; pos < TMTN; ++pos) dma_at(sb0, true, pos, std::true_type{});
    }
    load_frags(lds, 0, 0);
    // One stage; OPEN: both windows it touches are open (all but the last ns stages).
    // cur = l mod ns and its LDS byte address cur_b, and the global origins
    // (ga2, gb2) of stage l + ns, are carried from stage to stage.
    auto stage_step = [&](int l, int cur, uint32_t cur_b, uint64_t ga2, uint64_t gb2,
                          auto open) __attribute__((always_inline)) {
      constexpr bool OPEN = decltype(open)::value;
      const u32x4* as = reinterpret_cast<const u32x4*>(smem + (cur_b - lds0));
      const int ld = l + ns - 1;  // stage whose window ends with this stage's boundary
      const bool load = OPEN || ld < a.kLoop;
      StageBase sbs{0, 0, 0};
      if (load && NCS > 1)  // stage l + ns − 1 goes into slot (cur − 1) mod ns
        sbs = StageBase{ga2 - stepA, gb2 - stepB, cur == 0 ? lds0 + (ns - 1) * stage16 : cur_b - stage16};
#pragma unroll
      for (int cs = 0; cs + 1 < NCS; ++cs) {
        load_frags(as, cs + 1, (cs + 1) & 1);
#pragma unroll
        for (int q = 0; q < TMTN; ++q) {
          if constexpr (dl_split(NI, TMTN) && OPEN) {
            const int pos = TMTN + cs * TMTN + q, i = pos / R;
            if (pos % R == R - 1 && i < NIE && pos + 1 < SPOS) {
              __builtin_amdgcn_sched_barrier(0);
              dma_set_lds(dma_lds(sbs.sb, i));
              __builtin_amdgcn_sched_barrier(0);
              mfma1(cs & 1, q);
              __builtin_amdgcn_sched_barrier(0);
              dma_load16_set(doff[i], i < na_w ? sbs.ga : sbs.gb);
              __builtin_amdgcn_sched_barrier(0);
            } else {
              mfma1(cs & 1, q);
              dma_at(sbs, load, pos, open);
            }
          } else {
            mfma1(cs & 1, q);
            dma_at(sbs, load, TMTN + cs * TMTN + q, open);
          }
        }
      }
      const bool more = OPEN || l + 1 < a.kLoop;
      const uint32_t nx_b = cur + 1 == ns ? lds0 : cur_b + stage16;
      const u32x4* nx = reinterpret_cast<const u32x4*>(smem + (nx_b - lds0));
      if (more) {
        // stages issued after stage l + 1: l + 2 … min(l + ns − 1, kLoop − 1)
        const int pending = OPEN ? ns - 2 : min(ns - 2, a.kLoop - 2 - l);
        wait_vm_at_most(__builtin_amdgcn_readfirstlane(pending * ninst));
        waitcnt_lgkm0();  // this wavefront's reads of slot cur are complete
        // every wavefront: stage l + 1 landed, done reading slot cur
        __builtin_amdgcn_s_barrier();
        if constexpr (NCS >= 2) load_frags(nx, 0, 0);  // the last chunk-step uses slot 1
      }
      // last chunk-step; its slots open the window of stage l + ns (into slot cur)
      const bool load2 = OPEN || l + ns < a.kLoop;
      StageBase sb2{0, 0, 0};
      if (load2) sb2 = StageBase{ga2, gb2, cur_b};
#pragma unroll
      for (int q = 0; q < TMTN; ++q) {
        if constexpr (dl_split(NI, TMTN) && OPEN) {
          const int i = q / R;
          if (q % R == R - 1 && i < NIE && q + 1 < SPOS) {
            __builtin_amdgcn_sched_barrier(0);
            dma_set_lds(dma_lds(sb2.sb, i));
            __builtin_amdgcn_sched_barrier(0);
            mfma1((NCS - 1) & 1, q);
            __builtin_amdgcn_sched_barrier(0);
            dma_load16_set(doff[i], i < na_w ? sb2.ga : sb2.gb);
            __builtin_amdgcn_sched_barrier(0);
          } else {
            mfma1((NCS - 1) & 1, q);
            dma_at(sb2, load2, q, open);
          }
        } else {
          mfma1((NCS - 1) & 1, q);
          dma_at(sb2, load2, q, open);
        }
      }
      if constexpr (NCS == 1) {
        if (more) load_frags(nx, 0, 0);
      }
    };
    int l = 0, cur = 0;
    uint32_t cur_b = static_cast<uint32_t>(lds0);
    // origins of stage ns (as integers: stage ns may lie past the end of K,
    // then only stage ns − 1 = ga2 − stepA is ever loaded from them)
    const uint64_t zA = static_cast<uint64_t>(z) * static_cast<uint64_t>(BK) * 2u;
    uint64_t ga2 = uniform_ptr(Ag) + zA + static_cast<uint64_t>(ns) * stepA;
    uint64_t gb2 = uniform_ptr(Bg) + zA * static_cast<uint64_t>(a.N) + static_cast<uint64_t>(ns) * stepB;
    auto advance = [&]() __attribute__((always_inline)) {
      ++l;
      ga2 += stepA;
      gb2 += stepB;
      if (++cur == ns) {
        cur = 0;
        cur_b = static_cast<uint32_t>(lds0);
      } else {
        cur_b += stage16;
      }
    };
    while (l + ns < a.kLoop) {
      stage_step(l, cur, cur_b, ga2, gb2, std::true_type{});
      advance();
    }
    while (l < a.kLoop) {
      stage_step(l, cur, cur_b, ga2, gb2, std::false_type{});
      advance();
    }
  };
  if (ninst == kMaxDlInst)
    run(std::integral_constant<int, kMaxDlInst>{});
  else if (ninst == kMaxDlInst / 2)
    run(std::integral_constant<int, kMaxDlInst / 2>{});
  else
    run(std::integral_constant<int, 0>{});

  float* Cw = a.C + static_cast<int64_t>(gm) * BM * a.N + static_cast<int64_t>(gn) * BN;
#pragma unroll
  for (int i = 0; i < TM; ++i) {
#pragma unroll
    for (int j = 0; j < TN; ++j) {
#pragma unroll
      for (int e = 0; e < NACC; ++e) {
        const int r = wm * a.WM + i * I + out_row<I>(lane, e);
        const int c = wn * a.WN + j * I + (lane % I);
        put(a.atomic != 0, Cw + static_cast<int64_t>(r) * a.N + c, acc[i][j][e]);
      }
    }
  }
}

// ---------------------------------------------------------------------------
// Fast path with direct global→LDS loads, any stage (fp32, bf16)
// ---------------------------------------------------------------------------
//
// Tiles reach LDS by global_load_lds_dwordx4 (64 consecutive 16-byte slots a
// wavefront instruction), never through registers, into a ring of ns stages
// that keeps ns − 1 stages of loads in flight; one barrier a stage. The loads
// of a stage need not divide evenly over the wavefronts.
// A row-major: [m][k] chunks of 16 bytes, row r's chunks XOR-ed by fswz(r) (bf16
// with 16×16 MFMA and two or more chunk-steps: the planes of gemm_fast_dl), read
// 16 bytes a lane. B (and a K-major A) keep their [k][n] rows, split into one
// panel per wavefront column of WN = TN·I columns so that every row stride is a
// compile-time constant. bf16 panels are read with the transposing LDS read
// (chunks of row k XOR-ed by bswz(k)). fp32: the 4 k of a chunk of A feed 4
// MFMAs, lane group g holding chunk cs·G + g, and a lane reads its column of
// the same 4 k with 4-byte reads (consecutive lanes, consecutive banks); fp32
// MFMAs take 32 (16×16×4) or 64 cycles (32×32×2), so the extra LDS
// instructions stay below the matrix pipe's time: with one wavefront a SIMD and
// one MFMA tile each, 16 of 128 (16×16) or 256 (32×32) cycles per chunk-step.
// With 16×16 MFMA the two lane groups of a half-wavefront read rows 4 apart,
// a multiple of 256 bytes: odd groups' 16 columns are stored in the other half
// of a 128-byte line.
//
// Bound by the matrix pipe where the tiles fill the chip (fp32), by the operand
// stream into LDS (bf16), by the launch and one trip to memory (about 5 µs)
// where K is short. Against the register-staged form it replaced (loads one
// stage ahead, transposed in registers, spilled from 64 accumulators on): fp32
// 2048³ 158 -> 126 µs (137 TFLOP/s), 1024³ 31.3 -> 20.4 µs, K-major 31.7 ->
// 20.8 µs; bf16 3136×4096×1024 in 64×256×32 tiles, 8 wavefronts, 186 -> 55 µs,
// 1024×512×4096 in 64×32×64 tiles 78 -> 28 µs. Against gemm_fast_dl's loop
// with a branch per load: 512×4096×4096 in 128×64×64 tiles (6 loads a
// wavefront and stage) 34.8 -> 29.6 µs; at 2 and 3 loads that loop is up to 12 %
// faster (128×2624×3456 in 32×32×32 tiles 32.3 against 36.6 µs), and at the
// counts it is specialised for 8 % (4096³ in 256×256×32 tiles 115 against
// 131 µs), so those stay there.

// XOR of a row-major A row's chunk index: 8 consecutive rows read at the same
// chunk hit the 8 distinct 16-byte slots of 128 bytes.
template <int CPR>
__device__ __forceinline__ int fswz(int row) {
  return (row >> (CPR >= 8 ? 0 : (CPR == 4 ? 1 : 2))) & ((CPR < 8 ? CPR : 8) - 1);
}

// Whether a [k][n] panel of CW chunks a row stores the rows k with bit 2 set
// with the halves of each 128 bytes swapped: with 16×16 MFMA, where every lane
// holds rows of one instruction and the swap is the same for all of them or
// alternates (panels of 32 and 64 columns; wider ones, of 8 MFMA tiles a
// wavefront or more, keep the 2-way conflict).
template <int I, int CW>
constexpr bool flip_panel() {
  return I == 16 && (CW == 8 || CW == 16);
}

// Whether some wavefront layout (powers of two, up to 8 wavefronts) of this
// kernel has nh / 2 < (the most loads of one operand per wavefront) ≤ nh, or
// at most 2 for nh = 2.
template <int I, int TM, int TN, int CPR>
constexpr bool ring_needs(int nh) {
  for (int wm = 1; wm <= 8; wm *= 2)
    for (int wn = 1; wm * wn <= 8; wn *= 2) {
      const int na = (wm * TM * I * CPR / 64 + wm * wn - 1) / (wm * wn);
      const int nb = (wn * TN * I * CPR / 64 + wm * wn - 1) / (wm * wn);
      const int most = na > nb ? na : nb;
      if (most <= nh && (nh == 2 || most > nh / 2)) return true;
    }
  return false;
}

// Whether the accumulators, the fragments of two chunk-steps and their offsets
// (9 registers a tile row and column) and some 80 for the loads and addresses
// pass what the launch bound gives a lane (256, or 512 for kernels of at most 4
// wavefronts): then a chunk-step holds the fragments of the shorter side of
// the wavefront's tile and a few of the longer one's, read that many tiles ahead
// (ring_stream_step). (16×16 MFMA; no tile of 32×32 ones spills. Not 4×16 and
// 16×4 fp32 tiles in 64-deep stages, which fit without: the compiler then moves
// their 256 accumulators about, 440 against 298 µs at 2048×2048×1024.)
template <int DT, int I, int TM, int TN, int CPR>
constexpr bool ring_streams() {
  constexpr int acc = TM * TN * I * I / 64, spare = DT == 0 && CPR == 16 && acc == 256 ? 32 : 80;
  return I == 16 && acc + 9 * (TM + TN) + spare > (acc + 96 > 256 ? 512 : 256);
}

// One chunk-step of such a kernel: fragments from the stage at st, MFMAs in the
// order of the longer side's tiles, between(g) after each quarter of them.
template <int DT, int I, int TM, int TN, int CPR, bool AK, typename acc_t, typename F>
__device__ __forceinline__ void ring_stream_step(acc_t (&acc)[TM][TN], const char* st, int cs,
                                                 const uint32_t (&xa)[TM], const uint32_t (&xb)[TN],
                                                 int af, int plane, F between) {
  constexpr int G = 64 / I, WM = TM * I, WN = TN * I;
  constexpr bool PLANES = DT == 1 && I == 16 && CPR / G >= 2;
  constexpr bool BL = TN >= TM;  // B's side is the longer one
  constexpr int S = BL ? TM : TN, L = BL ? TN : TM;
  constexpr int D = S >= 4 ? 4 : 8;  // tiles of the longer side read ahead
  static_assert(L >= D, "a streamed tile has a long side");
  auto read = [&](bool b, int t) __attribute__((always_inline)) {
    u32x4 v;
    if (b && DT == 1) {
      s16x4 h[2];
#pragma unroll
      for (int hh = 0; hh < 2; ++hh)
        h[hh] = __builtin_amdgcn_ds_read_tr16_b64_v4i16(
            (__attribute__((address_space(3))) s16x4*)(st + xb[t] + (cs * G * 8 + 4 * hh) * WN * 2));
      v = __builtin_bit_cast(u32x4, __builtin_shufflevector(h[0], h[1], 0, 1, 2, 3, 4, 5, 6, 7));
    } else if (b || AK) {
#pragma unroll
      for (int q = 0; q < 4; ++q)
        v[q] = *reinterpret_cast<const unsigned*>(st + (b ? xb[t] : xa[t]) + (cs * G * 4 + q) * (b ? WN : WM) * 4);
    } else if (PLANES) {
      v = *reinterpret_cast<const u32x4*>(st + cs * plane + xa[t]);
    } else {
      v = *reinterpret_cast<const u32x4*>(st + xa[t] + ((af ^ (cs * G)) << 4));
    }
    return v;
  };
  u32x4 fs[S], fl[D];
#pragma unroll
  for (int t = 0; t < S; ++t) fs[t] = read(!BL, t);
#pragma unroll
  for (int t = 0; t < D; ++t) fl[t] = read(BL, t);
  __builtin_amdgcn_sched_barrier(0);
#pragma unroll
  for (int t = 0; t < L; ++t) {
#pragma unroll
    for (int q = 0; q < (DT == 1 ? 1 : 4); ++q)
#pragma unroll
      for (int s = 0; s < S; ++s) {
        const u32x4 va = BL ? fs[s] : fl[t % D], vb = BL ? fl[t % D] : fs[s];
        acc_t& c = acc[BL ? s : t][BL ? t : s];
        if constexpr (DT == 1)
          c = mfma_bf16(__builtin_bit_cast(bf16x8, va), __builtin_bit_cast(bf16x8, vb), c);
        else
          c = mfma_f32(__builtin_bit_cast(f32x4, va)[q], __builtin_bit_cast(f32x4, vb)[q], c);
      }
    if (t + D < L) fl[t % D] = read(BL, t + D);
    if ((t + 1) % (L / 4) == 0) between((t + 1) / (L / 4) - 1);
    __builtin_amdgcn_sched_barrier(0);
  }
}

template <int DT, int I, int TM, int TN, int CPR, bool AK>
__device__ __forceinline__ void gemm_ring(const KArgs& a, char* smem) {
  static_assert(DT == 0 || !AK, "the K-major-A ring is fp32 only");
  using acc_t = typename AccT<I>::type;
  constexpr int VEC = Elem<DT>::VEC, SZ = 16 / VEC;
  constexpr int G = 64 / I;
  constexpr int NCS = CPR / G;  // chunk-steps per stage
  constexpr int LGCPR = ilog2c<CPR>();
  constexpr int BK = CPR * VEC;
  constexpr int WM = TM * I, WN = TN * I;
  constexpr bool PLANES = DT == 1 && I == 16 && NCS >= 2;
  static_assert(NCS >= 1, "stage shallower than one MFMA K step");
  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int nw = blockDim.x >> 6;
  const int wm = wave % a.wavesM;
  const int wn = wave / a.wavesM;
  int gm, gn;
  tile_of(a, gm, gn);
  const int z = blockIdx.y;
  const int BM = a.BM, BN = a.BN, ns = a.ns, kLoop = a.kLoop;
  const uint32_t bbase = static_cast<uint32_t>(BM << LGCPR) * 16u;  // B inside a slot, bytes
  const uint32_t stage16 = bbase + (static_cast<uint32_t>(BN << LGCPR) * 16u);
  const uint32_t lds0 = static_cast<uint32_t>(
      __builtin_amdgcn_readfirstlane(static_cast<int>(lds_off(smem))));

  // Origins of this workgroup's tiles in bytes, and the strides of consecutive
  // stages of this split-K slice.
  const uint64_t lda = static_cast<uint64_t>(AK ? a.M : a.K) * SZ;
  const uint64_t ldb = static_cast<uint64_t>(a.N) * SZ;
  const uint64_t stepA = static_cast<uint64_t>(a.kSplit) * BK * (AK ? lda : SZ);
  const uint64_t stepB = static_cast<uint64_t>(a.kSplit) * BK * ldb;
  const uint64_t orgA = uniform_ptr(a.A) + static_cast<uint64_t>(gm) * BM * (AK ? SZ : lda) +
                        static_cast<uint64_t>(z) * BK * (AK ? lda : SZ);
  const uint64_t orgB = uniform_ptr(a.B) + static_cast<uint64_t>(gn) * BN * SZ +
                        static_cast<uint64_t>(z) * BK * ldb;

  // A wavefront's loads of one operand of a stage: instructions b0, b0 + db, …
  // of a block of LDS slots, 64 of them each. The block is a row-major A's
  // whole tile or one panel; consecutive wavefronts take the same instruction
  // of consecutive panels (never more than there are wavefronts), then the
  // next. B's start with the last wavefront, so that a short A and a short B
  // are not both on the first ones.
  struct Share {
    int cnt, b0, db, block;
  };
  auto share = [&](int w, int blocks, int insts) __attribute__((always_inline)) {
    const int b0 = w / blocks, db = nw / blocks;
    return Share{(insts - b0 + db - 1) / db, b0, db, w % blocks};
  };
  constexpr int NPA = CPR * WM / 64, NPB = CPR * WN / 64;  // instructions per panel
  const Share ha = AK ? share(wave, a.wavesM, NPA) : share(wave, 1, (BM << LGCPR) >> 6);
  const Share hb = share(nw - 1 - wave, a.wavesN, NPB);
  const int cnt = ha.cnt + hb.cnt;
  // Where load j reads, from the stage's origin: a uniform part and a lane's
  // (an instruction spans at most 32 rows), and where it writes in the slot.
  struct Place {
    uint64_t at;
    uint32_t lane, dst;
  };
  auto panel_place = [&](const Share& h, int j, uint64_t ld, auto wtag, int insts) __attribute__((always_inline)) {
    constexpr int C = decltype(wtag)::value / VEC;  // chunks per row of the panel
    const int s = (h.b0 + j * h.db) << 6;
    const int r0 = s / C, row = C >= 64 ? 0 : lane / C;
    const int pos = C >= 64 ? s % C + lane : lane % C;
    const int k = r0 + row;
    const int x = DT == 1 ? bswz(k, C) : (flip_panel<I, C>() ? k & 4 : 0);
    return Place{static_cast<uint64_t>(r0) * ld + static_cast<uint64_t>(h.block * C) * 16u,
                 static_cast<uint32_t>(row) * static_cast<uint32_t>(ld) + static_cast<uint32_t>(pos ^ x) * 16u,
                 static_cast<uint32_t>(h.block * insts + h.b0 + j * h.db) * 1024u};
  };
  auto place_a = [&](int j) __attribute__((always_inline)) {
    if constexpr (AK) {
      return panel_place(ha, j, lda, std::integral_constant<int, WM>{}, NPA);
    } else {
      const int b = ha.b0 + j * ha.db, s = b << 6;
      Place p;
      p.dst = static_cast<uint32_t>(b) * 1024u;
      if constexpr (PLANES) {
        const int lgp = a.lgBM + 2, in = s & ((1 << lgp) - 1);  // slots per plane: 4·BM
        const int q = swz(in + lane);
        p.at = static_cast<uint64_t>(in >> 2) * lda + static_cast<uint64_t>(s >> lgp) * 64u;
        p.lane = static_cast<uint32_t>((q >> 2) - (in >> 2)) * static_cast<uint32_t>(lda) +
                 static_cast<uint32_t>(q & 3) * 16u;
      } else {
        const int r0 = s >> LGCPR, row = lane >> LGCPR;
        p.at = static_cast<uint64_t>(r0) * lda;
        p.lane = static_cast<uint32_t>(row) * static_cast<uint32_t>(lda) +
                 static_cast<uint32_t>((lane & (CPR - 1)) ^ fswz<CPR>(r0 + row)) * 16u;
      }
      return p;
    }
  };
  auto place_b = [&](int j) __attribute__((always_inline)) {
    Place p = panel_place(hb, j, ldb, std::integral_constant<int, WN>{}, NPB);
    p.dst += bbase;
    return p;
  };
  // All of this wavefront's loads of a stage, back to back, at any distance:
  // every lane steps a 64-bit address of its own. What changes from load to
  // load is added up, not worked out from the load's number, which with 16 and
  // more of them cost more than the stage's MFMAs. (The lane's number is made
  // opaque, so that what follows from it is not kept in registers between
  // stages: spilled, its reload waits for every load on its way.)
  auto issue_panel = [&](const Share& h, uint64_t g, uint64_t ld, uint32_t slot, auto wtag, int insts) __attribute__((always_inline)) {
    constexpr int C = decltype(wtag)::value / VEC;
    constexpr int RI = C >= 64 ? 1 : 64 / C, IR = C >= 64 ? C / 64 : 1;  // rows an instruction, instructions a row
    int ln = lane;
    asm volatile("" : "+v"(ln));
    uint32_t dst = slot + static_cast<uint32_t>(h.block * insts + h.b0) * 1024u;
    int b = h.b0, k = b / IR * RI + (C >= 64 ? 0 : ln / C);
    uint64_t at = g + static_cast<uint64_t>(h.block * C) * 16u + static_cast<uint64_t>(k) * ld;
    const uint64_t step = static_cast<uint64_t>(h.db * RI) * ld;
    for (int j = 0; j < h.cnt; ++j) {
      const int x = DT == 1 ? bswz(k, C) : (flip_panel<I, C>() ? k & 4 : 0);
      const int pos = (C >= 64 ? b % IR * 64 + ln : ln % C) ^ x;
      dma_load16_at(at + static_cast<uint64_t>(pos) * 16u, dst);
      dst += static_cast<uint32_t>(h.db) * 1024u;
      b += h.db;
      if constexpr (IR == 1) {
        k += h.db * RI;
        at += step;
      } else {
        at += static_cast<uint64_t>(b / IR - k) * ld;
        k = b / IR;
      }
    }
  };
  auto issue_all = [&](uint64_t ga, uint64_t gb, uint32_t slot) __attribute__((always_inline)) {
    if constexpr (AK) {
      issue_panel(ha, ga, lda, slot, std::integral_constant<int, WM>{}, NPA);
    } else {
      int ln = lane;
      asm volatile("" : "+v"(ln));
      uint32_t dst = slot + static_cast<uint32_t>(ha.b0) * 1024u;
      int s = (ha.b0 << 6) + ln;
      for (int j = 0; j < ha.cnt; ++j) {
        if constexpr (PLANES) {
          const int lgp = a.lgBM + 2, q = swz(s & ((1 << lgp) - 1));  // slots per plane: 4·BM
          dma_load16_at(ga + static_cast<uint64_t>(q >> 2) * lda + static_cast<uint64_t>(s >> lgp) * 64u +
                            static_cast<uint64_t>(q & 3) * 16u, dst);
        } else {
          const int row = s >> LGCPR;
          dma_load16_at(ga + static_cast<uint64_t>(row) * lda +
                            static_cast<uint64_t>((s & (CPR - 1)) ^ fswz<CPR>(row)) * 16u, dst);
        }
        s += ha.db << 6;
        dst += static_cast<uint32_t>(ha.db) * 1024u;
      }
    }
    issue_panel(hb, gb, ldb, slot + bbase, std::integral_constant<int, WN>{}, NPB);
  };

  acc_t acc[TM][TN];
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j) acc[i][j] = acc_t{};

  // This lane's read offsets inside a slot. fp32 [k][n] panels: rows
  // (cs·G + grp)·4 + q, column t·I + lane % I of the wavefront's panel; bf16:
  // the transposing read's (input lane i of a 16-lane group covers row
  // k0 + (i >> 2), 4 rows further for the second read, columns 4(i & 3) on).
  const int grp = lane / I, l0 = lane % I;
  auto panel_read = [&](int wi, int t, auto w) __attribute__((always_inline)) {
    constexpr int W = decltype(w)::value, C = W / VEC;
    const int block = wi * (BK * W) * SZ;
    if constexpr (DT == 1) {
      const int i16 = lane & 15, g16 = lane >> 4;
      const int k = (I == 32 ? (g16 >> 1) : g16) * 8 + (i16 >> 2);
      const int col = t * I + (I == 32 ? 16 * (g16 & 1) : 0) + 4 * (i16 & 3);
      return static_cast<uint32_t>(block + (k * C + ((col >> 3) ^ bswz(k, C))) * 16 + (col & 4) * 2);
    } else {
      int col = t * I + l0;
      if constexpr (flip_panel<I, C>()) col ^= (grp & 1) << 4;
      return static_cast<uint32_t>(block + (grp * 4 * W + col) * 4);
    }
  };
  uint32_t xa[TM], xb[TN];
  const int af = fswz<CPR>(l0) ^ grp;  // I and the tile's rows are multiples of 16
  const int plane = BM << 6;           // bytes of one chunk-step's plane
#pragma unroll
  for (int t = 0; t < TM; ++t) {
    const int row = wm * WM + t * I + l0;
    if constexpr (AK)
      xa[t] = panel_read(wm, t, std::integral_constant<int, WM>{});
    else if constexpr (PLANES)
      xa[t] = static_cast<uint32_t>(swz((row << 2) + grp)) * 16u;
    else
      xa[t] = static_cast<uint32_t>(row) * (CPR * 16u);
  }
#pragma unroll
  for (int t = 0; t < TN; ++t) xb[t] = bbase + panel_read(wn, t, std::integral_constant<int, WN>{});

  u32x4 fa[2][TM], fb[2][TN];
  auto load_frags = [&](const char* st, int cs, int fs) __attribute__((always_inline)) {
#pragma unroll
    for (int t = 0; t < TM; ++t) {
      if constexpr (AK) {
#pragma unroll
        for (int q = 0; q < 4; ++q)
          fa[fs][t][q] = *reinterpret_cast<const unsigned*>(st + xa[t] + (cs * G * 4 + q) * WM * 4);
      } else if constexpr (PLANES) {
        fa[fs][t] = *reinterpret_cast<const u32x4*>(st + cs * plane + xa[t]);
      } else {
        fa[fs][t] = *reinterpret_cast<const u32x4*>(st + xa[t] + ((af ^ (cs * G)) << 4));
      }
    }
#pragma unroll
    for (int t = 0; t < TN; ++t) {
      if constexpr (DT == 1) {
        s16x4 h[2];
#pragma unroll
        for (int hh = 0; hh < 2; ++hh)
          h[hh] = __builtin_amdgcn_ds_read_tr16_b64_v4i16(
              (__attribute__((address_space(3))) s16x4*)(st + xb[t] + (cs * G * 8 + 4 * hh) * WN * 2));
        fb[fs][t] = __builtin_bit_cast(u32x4, __builtin_shufflevector(h[0], h[1], 0, 1, 2, 3, 4, 5, 6, 7));
      } else {
#pragma unroll
        for (int q = 0; q < 4; ++q)
          fb[fs][t][q] = *reinterpret_cast<const unsigned*>(st + xb[t] + (cs * G * 4 + q) * WN * 4);
      }
    }
  };
  // A chunk-step's MFMAs in SG groups: fp32, one per element of the chunks;
  // bf16, runs of the TM·TN tiles.
  constexpr int SG = DT == 0 || TM * TN >= 4 ? 4 : TM * TN;
  auto mfmas = [&](int fs, int g) __attribute__((always_inline)) {
    if constexpr (DT == 1) {
#pragma unroll
      for (int q = 0; q < TM * TN; ++q)
        if (q * SG / (TM * TN) == g)
          acc[q / TN][q % TN] = mfma_bf16(__builtin_bit_cast(bf16x8, fa[fs][q / TN]),
                                          __builtin_bit_cast(bf16x8, fb[fs][q % TN]), acc[q / TN][q % TN]);
    } else {
#pragma unroll
      for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j)
          acc[i][j] = mfma_f32(__builtin_bit_cast(f32x4, fa[fs][i])[g], __builtin_bit_cast(f32x4, fb[fs][j])[g],
                               acc[i][j]);
    }
  };

  if (ns == 1) {
    // a stage that leaves no room for a second one, or the only one
    uint64_t ga = orgA, gb = orgB;
    for (int l = 0; l < kLoop; ++l, ga += stepA, gb += stepB) {
      issue_all(ga, gb, lds0);
      waitcnt_vm<0>();
      ring_barrier();
      if constexpr (ring_streams<DT, I, TM, TN, CPR>()) {
#pragma unroll
        for (int cs = 0; cs < NCS; ++cs)
          ring_stream_step<DT, I, TM, TN, CPR, AK>(acc, smem, cs, xa, xb, af, plane, [](int) {});
      } else {
        load_frags(smem, 0, 0);
#pragma unroll
        for (int cs = 0; cs < NCS; ++cs) {
          if (cs + 1 < NCS) load_frags(smem, cs + 1, (cs + 1) & 1);
          __builtin_amdgcn_sched_barrier(0);
#pragma unroll
          for (int g = 0; g < SG; ++g) mfmas(cs & 1, g);
          __builtin_amdgcn_sched_barrier(0);
        }
      }
      waitcnt_lgkm0();
      ring_barrier();
    }
  } else {
    // Stage s goes into slot s mod ns. The boundary (wait for stage l + 1,
    // barrier, its first fragments) comes before stage l's last chunk-step of
    // MFMAs; the loads of stage l + ns, into the slot that every wavefront has
    // read by then, are issued from that chunk-step on, over a window of NCS
    // chunk-steps that ends before the next boundary.
    const uint32_t ring = ns * stage16;

    // NH: the loads of A, and of B, that a wavefront issues per stage, evenly
    // spread over a window's NCS·SG MFMA groups as straight-line code; a
    // wavefront with fewer (and every one after the last stage) issues the
    // rest with no lane enabled, so the count is the same everywhere. With one
    // wavefront a SIMD a branch in every group cost a fifth of the loop (fp32
    // 1024³, 64×64×64 tiles: 20.8 µs per 1024 of K with branches, 16.9 µs
    // without, 14 µs of MFMA). NH = 0: more loads than the offsets kept for
    // them, or offsets past 32 bits: all at once after the boundary.
    auto run = [&](auto nh) __attribute__((always_inline)) {
      constexpr int NH = decltype(nh)::value;
      uint32_t oa[NH ? NH : 1], ob[NH ? NH : 1];
#pragma unroll
      for (int i = 0; i < NH; ++i) {
        const Place p = place_a(i), q = place_b(i);
        oa[i] = p.lane + static_cast<uint32_t>(p.at);
        ob[i] = q.lane + static_cast<uint32_t>(q.at);
      }
      struct Window {
        uint64_t ga, gb;
        uint32_t da, db;  // the next load's place in the slot
        int na, nb;       // loads with their lanes enabled
      };
      const uint32_t fa0 = place_a(0).dst, fb0 = place_b(0).dst;
      const uint32_t sda = static_cast<uint32_t>(ha.db) * 1024u, sdb = static_cast<uint32_t>(hb.db) * 1024u;
      auto window = [&](uint64_t ga, uint64_t gb, uint32_t slot, bool on) __attribute__((always_inline)) {
        if (NH == 0 && on) issue_all(ga, gb, slot);
        return Window{ga, gb, slot + fa0, slot + fb0, on ? ha.cnt : 0, on ? hb.cnt : 0};
      };
      // the loads that follow MFMA group u of a window (u < 0: all of them)
      auto group = [&](Window& w, int u) __attribute__((always_inline)) {
#pragma unroll
        for (int i = 0; i < NH; ++i) {
          if (u < 0 || i * NCS * SG / NH == u) {
            dma_load16_if(w.na, i, oa[i], w.ga, w.da);
            w.da += sda;
          }
          if (u < 0 || (2 * i + 1) * NCS * SG / (2 * NH) == u) {
            dma_load16_if(w.nb, i, ob[i], w.gb, w.db);
            w.db += sdb;
          }
        }
      };
      // at most `after` stages past the one wanted may still be on their way
      const int keep = __builtin_amdgcn_readfirstlane((ns - 2) * 2 * NH);
      auto wait_stage = [&](int l) __attribute__((always_inline)) {
        if constexpr (NH == 0)
          wait_vm_at_most(__builtin_amdgcn_readfirstlane(max(min(ns - 2, kLoop - 2 - l), 0) * cnt));
        else if (ns == 3)
          waitcnt_vm<2 * NH>();
        else
          wait_vm_at_most(keep);
      };
      Window w{};
      for (int l = 0; l + 1 < ns; ++l) {
        w = window(orgA + l * stepA, orgB + l * stepB, lds0 + l * stage16, l < kLoop);
        group(w, -1);
      }
      wait_stage(-1);
      ring_barrier();
      if constexpr (ring_streams<DT, I, TM, TN, CPR>()) {
        // The boundary comes after a stage's last chunk-step, and the loads of
        // stage l + ns − 1, into the slot of stage l − 1, are issued during stage l.
        uint32_t cur_b = 0, free_b = ring - stage16;
        for (int l = 0; l < kLoop; ++l) {
          w = window(w.ga + stepA, w.gb + stepB, lds0 + free_b, l + ns - 1 < kLoop);
#pragma unroll
          for (int cs = 0; cs < NCS; ++cs)
            ring_stream_step<DT, I, TM, TN, CPR, AK>(acc, smem + cur_b, cs, xa, xb, af, plane,
                                                     [&](int g) __attribute__((always_inline)) { group(w, SG * cs + g); });
          waitcnt_lgkm0();
          if (l + 1 < kLoop) {
            wait_stage(l);
            ring_barrier();
          }
          free_b = cur_b;
          cur_b = cur_b + stage16 == ring ? 0u : cur_b + stage16;
        }
      } else {
        w = window(orgA + static_cast<uint64_t>(ns - 1) * stepA, orgB + static_cast<uint64_t>(ns - 1) * stepB,
                   lds0 + (ns - 1) * stage16, ns - 1 < kLoop);
        load_frags(smem, 0, 0);
#pragma unroll
        for (int g = 0; g < SG; ++g) group(w, g);
        uint32_t cur_b = 0;  // this stage's slot, bytes from the ring's start
        for (int l = 0; l < kLoop; ++l) {
          const char* st = smem + cur_b;
          const uint32_t nx_b = cur_b + stage16 == ring ? 0u : cur_b + stage16;
#pragma unroll
          for (int cs = 0; cs + 1 < NCS; ++cs) {
            load_frags(st, cs + 1, (cs + 1) & 1);
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int g = 0; g < SG; ++g) {
              mfmas(cs & 1, g);
              group(w, SG + SG * cs + g);
            }
          }
          const bool more = l + 1 < kLoop;
          // (outside the branch: past it the compiler would wait for the next
          // stage's fragments too)
          waitcnt_lgkm0();
          if (more) {
            wait_stage(l);
            ring_barrier();
            if constexpr (NCS >= 2) load_frags(smem + nx_b, 0, 0);
          }
          w = window(w.ga + stepA, w.gb + stepB, lds0 + cur_b, l + ns < kLoop);
#pragma unroll
          for (int g = 0; g < SG; ++g) {
            mfmas((NCS - 1) & 1, g);
            group(w, g);
          }
          if constexpr (NCS == 1) {
            if (more) load_frags(smem + nx_b, 0, 0);
          }
          cur_b = nx_b;
        }
      }
    };
    // The most loads of one operand that any wavefront of the workgroup has.
    const int most = max(((BM << LGCPR) + 64 * nw - 1) / (64 * nw), ((BN << LGCPR) + 64 * nw - 1) / (64 * nw));
    auto run_if = [&](auto nh) __attribute__((always_inline)) {
      if constexpr (ring_needs<I, TM, TN, CPR>(decltype(nh)::value)) run(nh);
    };
    if (a.wide || most > 8)
      run(std::integral_constant<int, 0>{});
    else if (most > 4)
      run_if(std::integral_constant<int, 8>{});
    else if (most > 2)
      run_if(std::integral_constant<int, 4>{});
    else
      run_if(std::integral_constant<int, 2>{});
  }

  store_tile<I, TM, TN>(a,
                        a.C + (static_cast<int64_t>(gm) * BM + wm * WM) * a.N +
                            (static_cast<int64_t>(gn) * BN + wn * WN),
                        lane, acc);
}

// ---------------------------------------------------------------------------
// Generic path without shared stages ("stream"): every wavefront reads its own
// operands, so there are no barriers, and a K step takes IK consecutive k
// whatever kBlk and the stage depth are (the K levels only say where a slice's
// stages lie: one run of all K, or runs of BK with a K split).
//   fp32: 16-byte (row-major A) and 4-byte loads straight into MFMA operands;
//   bf16: a row-major A is loaded the same way, 8 k a lane; B, and a K-major A,
//   pass through a piece of LDS of the wavefront's own, written 16 bytes a
//   lane and read back with the transposing read (chunks of row k XOR-ed by
//   bswz(k)). LDS operations of a wavefront complete in order, so one buffer
//   serves every step.
// Loads run PF steps ahead in registers. Rows and columns that a block smaller
// than I lacks read the block's last ones; their products are not stored. Past
// the end of K both operands are zero.
// Bound by the loads themselves (each wavefront fetches (WM + WN)·K elements
// through its CU's L1) where blocks are small. Against the shared stages of
// gemm_generic, which gather bf16 operands from LDS 2 bytes at a time, pad
// every sub-step to the instruction's K and cross two barriers a stage:
// 1360×1200×720 bf16 in 16×16 tiles 131 -> 33 µs, 2048³ bf16 with a K-major A
// in 128×128 tiles 224 -> 38 µs, 1440×968×176 fp32 in 32×8 tiles 32 -> 21 µs.
template <int TM, int TN>
constexpr bool has_stream() {
  return TM + TN <= 10;
}

template <int DT, int I, int TM, int TN, bool AK>
__device__ __forceinline__ void gemm_stream(const KArgs& a, char* smem) {
  using T = typename Elem<DT>::T;
  using acc_t = typename AccT<I>::type;
  constexpr int NACC = AccT<I>::N;
  constexpr int G = 64 / I;
  constexpr int SZ = sizeof(T);
  constexpr int KL = 16 / SZ;  // consecutive k a lane holds of a step: 8 bf16, 4 fp32
  constexpr int KS = KL * G;   // k per step
  constexpr int PF = TM + TN <= 4 ? 4 : 2;  // steps of loads in flight (even)
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(static_cast<int>(threadIdx.x) >> 6);
  const int wm = wave % a.wavesM;
  const int wn = wave / a.wavesM;
  int gm, gn;
  tile_of(a, gm, gn);
  const int z = blockIdx.y;
  const int grp = lane / I, l0 = lane % I;
  const int tpbM = 1 << a.lgTpbM, tpbN = 1 << a.lgTpbN;
  const int64_t row0 = static_cast<int64_t>(gm) * a.BM + wm * a.WM;
  const int64_t col0 = static_cast<int64_t>(gn) * a.BN + wn * a.WN;
  const int64_t k0 = static_cast<int64_t>(z) * a.BK;
  const int64_t lda = AK ? a.M : a.K;
  const char* pa = reinterpret_cast<const char*>(a.A) + (AK ? k0 * lda + row0 : row0 * lda + k0) * SZ;
  const char* pb = reinterpret_cast<const char*>(a.B) + (k0 * a.N + col0) * SZ;
  const int64_t stepa = (AK ? lda : 1) * KS * SZ, stepb = a.N * KS * SZ;
  // steps of this slice: runs of `run` k, `skip` k apart
  const int64_t run = a.kSplit == 1 ? a.K : a.BK;
  const int64_t skip = a.kSplit == 1 ? 0 : static_cast<int64_t>(a.kSplit - 1) * a.BK;
  const int64_t skipa = skip * (AK ? lda : 1) * SZ, skipb = skip * a.N * SZ;
  const int per_run = static_cast<int>(run / KS);
  const int full = per_run * (a.kSplit == 1 ? 1 : a.kLoop);
  const int left = static_cast<int>(run - static_cast<int64_t>(per_run) * KS);  // kSplit 1 only

  // Row (column) of the wavefront's tile that MFMA tile t has at in-tile row l.
  auto row_of = [&](int t, int l) {
    return (t >> a.lgTpbM) * a.blkM + min((t & (tpbM - 1)) * I + l, a.blkM - 1);
  };
  auto col_of = [&](int t, int l) {
    return (t >> a.lgTpbN) * a.blkN + min((t & (tpbN - 1)) * I + l, a.blkN - 1);
  };

  // One operand given with K as its rows ([k][x], x contiguous, ld long).
  // bf16: TX loads of 64 chunks cover the KS × width panel; fp32: 4 rows a lane.
  struct Panel {
    uint32_t off[8];    // bytes from the step's origin of the lane's loads
    uint32_t put[8];    // bf16: where they go in the wavefront's LDS
    uint32_t get[8];    // bf16: this lane's transposing reads (first of two)
    int row[8];         // first k row of each load, for the end of K
  };
  auto panel = [&](Panel& p, auto txt, int64_t ld, int width, char* lds, auto xof) __attribute__((always_inline)) {
    constexpr int TX = decltype(txt)::value;
    if constexpr (DT == 1) {
      const int cw = width >> 3;  // a power of two
      const int lgcw = 31 - __builtin_clz(cw);
      const int i16 = lane & 15, g16 = lane >> 4;
      const int kgrp = I == 32 ? (g16 >> 1) : g16;
      const int ncol = (I == 32 ? 16 * (g16 & 1) : 0) + 4 * (i16 & 3);
#pragma unroll
      for (int t = 0; t < TX; ++t) {
        const int c = min(lane + 64 * t, KS * cw - 1);
        const int k = c >> lgcw, x = c & (cw - 1);
        p.row[t] = k;
        p.off[t] = (static_cast<uint32_t>(k) * static_cast<uint32_t>(ld) + static_cast<uint32_t>(x * 8)) * 2u;
        p.put[t] = lds_off(lds) + static_cast<uint32_t>((k << lgcw) + (x ^ bswz(k, cw))) * 16u;
        const int kr = kgrp * 8 + (i16 >> 2);
        const int col = min(xof(t, 0) + ncol, width - 4);
        // the second read is 4 rows on: bswz depends on k mod 4 and bit 3 only
        p.get[t] = lds_off(lds) + static_cast<uint32_t>((kr << lgcw) + ((col >> 3) ^ bswz(kr, cw))) * 16u +
                   static_cast<uint32_t>(col & 4) * 2u;
      }
    } else {
#pragma unroll
      for (int t = 0; t < TX; ++t) {
        p.row[t] = grp * 4;
        p.off[t] = (static_cast<uint32_t>(grp * 4) * static_cast<uint32_t>(ld) +
                    static_cast<uint32_t>(xof(t, l0))) * 4u;
      }
    }
  };
  Panel fb, fa;
  const uint32_t ldb4 = static_cast<uint32_t>(a.N) * 4u, lda4 = static_cast<uint32_t>(lda) * 4u;
  // the wavefront's piece of LDS, for its B panel and then for its A panel
  char* const mine = smem + wave * (KS * (AK ? max(a.WM, a.WN) : a.WN) * 2);
  panel(fb, std::integral_constant<int, TN>{}, a.N, a.WN, mine, col_of);
  const int bgap = (a.WN >> 3) * 64, agap = (a.WM >> 3) * 64;  // bytes between a fragment's two reads
  if constexpr (AK) {
    panel(fa, std::integral_constant<int, TM>{}, lda, a.WM, mine, row_of);
  } else {
#pragma unroll
    for (int t = 0; t < TM; ++t)
      fa.off[t] = (static_cast<uint32_t>(row_of(t, l0)) * static_cast<uint32_t>(lda) +
                   static_cast<uint32_t>(grp * KL)) * static_cast<uint32_t>(SZ);
  }

  acc_t acc[TM][TN];
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j) acc[i][j] = acc_t{};

  u32x4 ra[PF][TM], rb[PF][TN];
  // kv: k of this step that exist, KS inside K (`end` false)
  auto load_panel = [&](u32x4& v, const char* base, const Panel& p, int t, uint32_t ld4, int kv,
                        auto end) __attribute__((always_inline)) {
    if constexpr (DT == 1) {
      const bool in = !decltype(end)::value || p.row[t] < kv;
      v = *reinterpret_cast<const u32x4*>(base + (in ? p.off[t] : 0u));
      if (!in) v = u32x4{0, 0, 0, 0};
    } else {
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const bool in = !decltype(end)::value || p.row[t] + q < kv;
        const unsigned x = *reinterpret_cast<const unsigned*>(base + (in ? p.off[t] + q * ld4 : 0u));
        v[q] = in ? x : 0u;
      }
    }
  };
  auto load = [&](int s, int kv, auto end) __attribute__((always_inline)) {
#pragma unroll
    for (int t = 0; t < TM; ++t) {
      if constexpr (AK) {
        load_panel(ra[s][t], pa, fa, t, lda4, kv, end);
      } else {
        const bool in = !decltype(end)::value || grp * KL < kv;  // K is a multiple of KL here
        ra[s][t] = *reinterpret_cast<const u32x4*>(pa + (in ? fa.off[t] : 0u));
        if (!in) ra[s][t] = u32x4{0, 0, 0, 0};
      }
    }
#pragma unroll
    for (int t = 0; t < TN; ++t) load_panel(rb[s][t], pb, fb, t, ldb4, kv, end);
  };
  int in_run = 0;
  auto advance = [&]() __attribute__((always_inline)) {
    pa += stepa;
    pb += stepb;
    // (a select, not a branch, between the loads)
    const bool over = ++in_run == per_run;
    in_run = over ? 0 : in_run;
    pa += over ? skipa : 0;
    pb += over ? skipb : 0;
  };
  typedef __attribute__((address_space(3))) u32x4 lds_u32x4;
  typedef __attribute__((address_space(3))) s16x4 lds_s16x4;
  auto fetch = [&](u32x4& v, const Panel& p, int t, int gap) __attribute__((always_inline)) {
    s16x4 h[2];
    h[0] = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4*)(uintptr_t)(p.get[t]));
    h[1] = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4*)(uintptr_t)(p.get[t] + gap));
    v = __builtin_bit_cast(u32x4, __builtin_shufflevector(h[0], h[1], 0, 1, 2, 3, 4, 5, 6, 7));
  };
  // bf16: a loaded step's panels through LDS into MFMA operands (f = 0 or 1)
  u32x4 af[2][TM], bf[2][TN];
  auto transpose = [&](int s, int f) __attribute__((always_inline)) {
    if constexpr (DT == 1) {
#pragma unroll
      for (int t = 0; t < TN; ++t) *(lds_u32x4*)(uintptr_t)(fb.put[t]) = rb[s][t];
#pragma unroll
      for (int t = 0; t < TN; ++t) fetch(bf[f][t], fb, t, bgap);
      if constexpr (AK) {
#pragma unroll
        for (int t = 0; t < TM; ++t) *(lds_u32x4*)(uintptr_t)(fa.put[t]) = ra[s][t];
#pragma unroll
        for (int t = 0; t < TM; ++t) fetch(af[f][t], fa, t, agap);
      }
    }
  };
  auto multiply = [&](int s, int f) __attribute__((always_inline)) {
    if constexpr (DT == 1) {
#pragma unroll
      for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j)
          acc[i][j] = mfma_bf16(__builtin_bit_cast(bf16x8, AK ? af[f][i] : ra[s][i]),
                                __builtin_bit_cast(bf16x8, bf[f][j]), acc[i][j]);
    } else {
#pragma unroll
      for (int q = 0; q < 4; ++q)
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
          for (int j = 0; j < TN; ++j)
            acc[i][j] = mfma_f32(__builtin_bit_cast(f32x4, ra[s][i])[q],
                                 __builtin_bit_cast(f32x4, rb[s][j])[q], acc[i][j]);
    }
  };

  int issued = 0, done = 0;
#pragma unroll
  for (int s = 0; s < PF; ++s)
    if (issued < full) {
      load(s, KS, std::false_type{});
      advance();
      ++issued;
    }
  if (full) transpose(0, 0);
  // Step `done` is in slot s; the next one's panels pass through LDS while its
  // MFMAs run, then its slot is loaded again. Without a branch between them
  // the compiler counts the loads in flight and waits for the one it needs;
  // the last steps check what is left.
  for (; done + 2 * PF <= full; done += PF) {
#pragma unroll
    for (int s = 0; s < PF; ++s) {
      transpose((s + 1) % PF, (s + 1) & 1);
      multiply(s, s & 1);
      load(s, KS, std::false_type{});
      advance();
    }
    issued += PF;
  }
  while (done < full) {
#pragma unroll
    for (int s = 0; s < PF; ++s)
      if (done < full) {
        ++done;
        if (done < full) transpose((s + 1) % PF, (s + 1) & 1);
        multiply(s, s & 1);
        if (issued < full) {
          load(s, KS, std::false_type{});
          advance();
          ++issued;
        }
      }
  }
  if (left) {
    load(0, left, std::true_type{});
    transpose(0, 0);
    multiply(0, 0);
  }

  float* Cw = a.C + row0 * a.N + col0;
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int e = 0; e < NACC; ++e) {
      const int ri = (i & (tpbM - 1)) * I + out_row<I>(lane, e);
      float* const p = Cw + static_cast<int64_t>((i >> a.lgTpbM) * a.blkM + ri) * a.N;
#pragma unroll
      for (int j = 0; j < TN; ++j) {
        const int ci = (j & (tpbN - 1)) * I + l0;
        if (ri < a.blkM && ci < a.blkN)
          put(a.atomic != 0, p + (j >> a.lgTpbN) * a.blkN + ci, acc[i][j][e]);
      }
    }
}

// Launch bound: the largest wavefront count the legitimacy rule admits for
// this accumulator size (acc + 96 ≤ 512 / ⌈waves/4⌉); the fast path is used
// with at most 8 wavefronts.
template <int I, int TM, int TN>
constexpr int max_waves() {
  constexpr int acc = TM * TN * I * I / 64;
  return acc + 96 <= 128 ? 16 : (acc + 96 <= 256 ? 8 : 4);
}

template <int I, int TM, int TN, int CPR>
constexpr int launch_threads() {
  return 64 * (CPR > 0 && max_waves<I, TM, TN>() > 8 ? 8 : max_waves<I, TM, TN>());
}

// CPR = 0: generic path; CPR > 0: fast path with BK = CPR·VEC.
template <int DT, int I, int TM, int TN, int CPR>
__global__ void __launch_bounds__((launch_threads<I, TM, TN, CPR>())) gemm_kernel(KArgs a) {
  extern __shared__ u32x4 gt_smem[];
  char* smem = reinterpret_cast<char*>(gt_smem);
  if constexpr (CPR == 0) {
    gemm_generic<DT, I, TM, TN>(a, smem);
  } else {
    gemm_ring<DT, I, TM, TN, CPR, false>(a, smem);
  }
}

// Generic path whose wavefronts read their own operands, at most 8 of them.
template <int DT, int I, int TM, int TN, bool AK>
__global__ void __launch_bounds__((launch_threads<I, TM, TN, 1>())) gemm_kernel_stream(KArgs a) {
  extern __shared__ u32x4 gt_smem[];
  gemm_stream<DT, I, TM, TN, AK>(a, reinterpret_cast<char*>(gt_smem));
}

// fp32 fast path for a K-major A.
template <int DT, int I, int TM, int TN, int CPR>
__global__ void __launch_bounds__((launch_threads<I, TM, TN, CPR>())) gemm_kernel_akm(KArgs a) {
  static_assert(DT == 0, "the K-major-A fast path is fp32 only");
  extern __shared__ u32x4 gt_smem[];
  gemm_ring<0, I, TM, TN, CPR, true>(a, reinterpret_cast<char*>(gt_smem));
}

// bf16 fast path with evenly shared loads: a kernel of its own, so that its
// register allocation does not inherit the general ring's.
template <int I, int TM, int TN, int CPR>
__global__ void __launch_bounds__((launch_threads<I, TM, TN, CPR>())) gemm_kernel_dl(KArgs a) {
  extern __shared__ u32x4 gt_smem[];
  gemm_fast_dl<I, TM, TN, CPR>(a, reinterpret_cast<char*>(gt_smem));
}

using LaunchFn = hipError_t (*)(const KArgs&, dim3, dim3, size_t, hipStream_t);

// Raises the kernel's dynamic LDS limit once per device (bit d of `attr_devs`
// for device d < 64; beyond that on every launch), then launches. Concurrent
// callers may both set the attribute, which is idempotent.
template <class F>
hipError_t launch_one(F fn, std::atomic<uint64_t>& attr_devs, const KArgs& a, dim3 grid,
                      dim3 block, size_t lds, hipStream_t s) {
  int dev = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return e;
  const uint64_t bit = dev >= 0 && dev < 64 ? uint64_t{1} << dev : 0;
  if (!bit || !(attr_devs.load(std::memory_order_acquire) & bit)) {
    e = hipFuncSetAttribute(reinterpret_cast<const void*>(fn),
                            hipFuncAttributeMaxDynamicSharedMemorySize, 163840);
    if (e != hipSuccess) return e;
    attr_devs.fetch_or(bit, std::memory_order_release);
  }
  hipLaunchKernelGGL(fn, grid, block, lds, s, a);
  return hipGetLastError();
}

// AKM: the translation unit instantiates the K-major-A fast path (it then
// serves only launches with a.aKM set; the generic path handles both layouts).
template <int DT, int I, int TM, int TN, int CPR, bool AKM = false>
hipError_t launch_gemm(const KArgs& a, dim3 grid, dim3 block, size_t lds, hipStream_t s) {
  if constexpr (AKM) {
    static_assert(CPR > 0, "the K-major-A kernel is a fast-path kernel");
    static std::atomic<uint64_t> attr_akm{0};
    return launch_one(gemm_kernel_akm<DT, I, TM, TN, CPR>, attr_akm, a, grid, block, lds, s);
  } else {
    if constexpr (DT == 1 && CPR > 0) {
      if (a.dlk) {
        static std::atomic<uint64_t> attr_dl{0};
        return launch_one(gemm_kernel_dl<I, TM, TN, CPR>, attr_dl, a, grid, block, lds, s);
      }
    }
    if constexpr (CPR == 0 && has_stream<TM, TN>()) {
      if (a.stream) {
        static std::atomic<uint64_t> attr_s{0}, attr_sk{0};
        return a.aKM ? launch_one(gemm_kernel_stream<DT, I, TM, TN, true>, attr_sk, a, grid, block, lds, s)
                     : launch_one(gemm_kernel_stream<DT, I, TM, TN, false>, attr_s, a, grid, block, lds, s);
      }
    }
    static std::atomic<uint64_t> attr{0};
    return launch_one(gemm_kernel<DT, I, TM, TN, CPR>, attr, a, grid, block, lds, s);
  }
}

// (TM, TN) pairs with TM·TN ≤ 16 (I = 32) and ≤ 64 (I = 16): the register
// rule acc = TM·TN·I²/64 ≤ 256.
#define GT_PAIRS_16(X)                                                                      \
  X(1, 1) X(1, 2) X(2, 1) X(1, 4) X(2, 2) X(4, 1) X(1, 8) X(2, 4) X(4, 2) X(8, 1) X(1, 16) \
      X(2, 8) X(4, 4) X(8, 2) X(16, 1)
#define GT_PAIRS_64(X)                                                                       \
  GT_PAIRS_16(X)                                                                             \
  X(1, 32) X(2, 16) X(4, 8) X(8, 4) X(16, 2) X(32, 1) X(1, 64) X(2, 32) X(4, 16) X(8, 8)     \
      X(16, 4) X(32, 2) X(64, 1)

// Chunks per LDS row with a fast-path instantiation (BK = CPR·VEC).
constexpr int kFastCpr[] = {2, 4, 8, 16};

// Kernel of (dtype, I, CPR, TM, TN), CPR = 0 for the generic path, akm for
// the K-major-A fast path (f32 only); nullptr when not instantiated.
LaunchFn find_gemm_kernel(int dtype, int I, int cpr, int TM, int TN, bool akm);

}  // namespace gt

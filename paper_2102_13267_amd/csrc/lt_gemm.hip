// fp32 contraction region: C = post(A * B) on the MFMA matrix cores (gfx950), fp32 operands and
// accumulation (bf16 operands: lt_gemm_bf16.hip).  Operands are addressed through element strides,
// so transposed, batched and head-split layouts need no copies.  The elementwise chain that
// consumes the product (bias, activation, residual, optimiser update, cast ...) is interpreted on
// the accumulator tile before anything is written: the product itself never travels to HBM unless
// asked for.
//
// Structure: workgroup tile 128 x 128 (or 64 x 64 for small problems so that more compute units
// get a tile), four wavefronts in a 2 x 2 arrangement, each owning a quarter as MFMA 32x32x2
// blocks.  K is walked in slices of 32 that travel from global memory straight into LDS (lt_dma.h), four
// stages, so that the loop holds nothing but LDS reads, MFMAs and one barrier per slice: the matrix
// cores bound it (fp32 MFMA 157 TFLOP/s; the vendor library reaches 141 to 154).  Measured against
// staging the same tiles through registers (transposing stores, the same four slices ahead):
// [1024, 2048] x [2048, 2048] with bias and GELU 90.5 -> 70 us, a head's three products of 2048 x 1024 x 1000, ragged, 67 / 62 / 75 -> 44 /
// 42 / 45; with reads and copies put between the MFMAs by hand (below) 64.5 (133 TFLOP/s) and 37 / 36 / 34, in a row.  A tile over the operand's edge takes the same
// path; what is left of k behind the last whole slice is one checked slice; rows that are not
// 16-byte aligned go through registers.  A long k over few tiles is split over workgroups (partial
// products to a workspace, summed by a second launch).
// Small products take another kernel further down (lt_gemm_small_kernel: no LDS staging, k split
// inside the workgroup and, for a long k, over a few workgroups that meet inside the launch).
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstdio>

#include "lt_dma.h"
#include "lt_gemm_epilogue.h"
#include "lt_launch.h"
#include "lt_reduce.h"

namespace ltk {

// ---- operand staging --------------------------------------------------------------------------
// A "group" is what one lane fetches with one 16-byte load: G consecutive elements along the
// operand's contiguous dimension (4 fp32 or 8 bf16).  For element type T the raw group travels
// as uint4.
template <typename T> struct Elem;
template <> struct Elem<float> { static constexpr int G = 4; static constexpr int BK = 32; };

// LDS layout: tile[k][x] (x = m or n contiguous); an MFMA 32x32x2 lane reads one float.  Row stride:
// BX + 4 for an operand that arrives x-contiguous (16-byte row writes stay aligned).  An operand
// that arrives k-contiguous is transposed by scalar writes, eight lanes of a wave writing rows
// 4 apart: BX + 1 puts those rows 4 banks apart, so a wave's 32 writes per cycle hit 32 banks
// (with BX + 4 they hit 8: counters showed as many bank-conflict cycles as LDS cycles).  ELEMS is
// sized for the wider one, so buffers are interchangeable.
template <typename T, int BX> struct Tile;
template <int BX> struct Tile<float, BX> {
  static constexpr int BK = 32, ELEMS = BK * (BX + 4);
  static constexpr int stride(bool kc) { return kc ? BX + 1 : BX + 4; }
};
// Number of 16-byte groups per lane and k-slice for an operand tile of BX x BK elements.
template <typename T, int BX> struct Groups {
  static constexpr int N = BX * Elem<T>::BK / Elem<T>::G / kGemmThreads;   // 128: 4, 64: 2
};

// (a native vector type, not HIP's uint4 struct: sets of the struct kind that are only ever moved
// whole were left in scratch memory by the compiler)
typedef uint32_t U32x4 __attribute__((ext_vector_type(4)));
template <uint32_t N> struct Num {
  static constexpr uint32_t value = N;
};

template <int N> struct GroupRegs {
  U32x4 g[N];
};

// Fetch this lane's groups of the slice starting at k0, element by element at addresses clamped into the
// operand (branch-free: all of a lane's loads are in flight together).  k past the end reads as zero;
// rows or columns past the edge are copies of the last one and are never stored.  KC: the contraction
// dimension is the operand's contiguous one.  x0: first row (A) / column (B) of the tile.
template <typename T, int BX, bool KC>
__device__ __forceinline__ void fetch_tile(GroupRegs<Groups<T, BX>::N>& gr, const T* base, int64_t s_x, int64_t s_k, uint32_t x0,
                                           uint32_t k0, uint32_t nx, uint32_t nk) {
  constexpr uint32_t G = Elem<T>::G, per_row = (KC ? Elem<T>::BK : BX) / G;
#pragma unroll
  for (int it = 0; it < Groups<T, BX>::N; ++it) {
    const uint32_t e = it * kGemmThreads + threadIdx.x % kGemmThreads, o = e / per_row, i = (e % per_row) * G;
#pragma unroll
    for (uint32_t j = 0; j < G; ++j) {
      const uint32_t x = x0 + (KC ? o : i + j), k = k0 + (KC ? i + j : o);
      const T v = base[(int64_t)min(x, nx - 1u) * s_x + (int64_t)min(k, nk - 1u) * s_k];
      gr.g[it][j] = k < nk ? __float_as_uint(v) : 0u;
    }
  }
}

template <int BX, bool KC>
__device__ __forceinline__ void stash_tile(const GroupRegs<Groups<float, BX>::N>& gr, float* tile) {
  constexpr int G = 4, BK = Elem<float>::BK, STRIDE = Tile<float, BX>::stride(KC), NG = Groups<float, BX>::N;
  const uint32_t t = threadIdx.x % kGemmThreads;
#pragma unroll
  for (int it = 0; it < NG; ++it) {
    const uint32_t e = it * kGemmThreads + t;
    if (KC) {   // transposing: four scalar writes
      const uint32_t x = e / (BK / G), kq = e % (BK / G);
      tile[(kq * G + 0) * STRIDE + x] = __uint_as_float(gr.g[it].x);
      tile[(kq * G + 1) * STRIDE + x] = __uint_as_float(gr.g[it].y);
      tile[(kq * G + 2) * STRIDE + x] = __uint_as_float(gr.g[it].z);
      tile[(kq * G + 3) * STRIDE + x] = __uint_as_float(gr.g[it].w);
    } else {
      const uint32_t k = e / (BX / G), xq = e % (BX / G);
      *(U32x4*)&tile[k * STRIDE + xq * G] = gr.g[it];
    }
  }
}

// ---- whole slices ---------------------------------------------------------------------------------
// Element offset, from the panel's start, of the 16-byte chunk at (outer, inner) of a slice: the same for
// every slice.  Rows (KC) or chunks of four columns past the operand's edge (`left` rows or columns from
// the panel's start) become copies of the last one: in bounds, and their products are never stored.
template <bool KC>
__device__ __forceinline__ int64_t chunk_offset(uint32_t outer, uint32_t inner, int64_t s_x, int64_t s_k, uint32_t left) {
  return KC ? (int64_t)min(outer, left - 1u) * s_x + inner : (int64_t)outer * s_k + min(inner, (left - 1u) & ~3u);
}

// Rows that start at any element: through registers into the padded tiles above, 16-byte loads at
// 4-byte boundaries.
template <int BX> struct Offsets {
  int64_t o[Groups<float, BX>::N];
};
template <int BX, bool KC>
__device__ __forceinline__ Offsets<BX> unaligned_offsets(int64_t s_x, int64_t s_k, uint32_t left) {
  constexpr uint32_t per_row = (KC ? Elem<float>::BK : BX) / 4;
  Offsets<BX> off;
#pragma unroll
  for (int it = 0; it < Groups<float, BX>::N; ++it) {
    const uint32_t e = it * kGemmThreads + threadIdx.x % kGemmThreads;
    off.o[it] = chunk_offset<KC>(e / per_row, (e % per_row) * 4u, s_x, s_k, left);
  }
  return off;
}
template <int BX>
__device__ __forceinline__ void fetch_unaligned(GroupRegs<Groups<float, BX>::N>& gr, const float* panel, const Offsets<BX>& off) {
  typedef uint32_t V __attribute__((ext_vector_type(4), aligned(4)));
#pragma unroll
  for (int it = 0; it < Groups<float, BX>::N; ++it) {
    const V v = *(const V*)(panel + off.o[it]);
    gr.g[it] = U32x4{v.x, v.y, v.z, v.w};
  }
}

// 16-byte aligned rows: straight into LDS (lt_dma.h), dense tiles whose bank conflicts a swizzle avoids.
//   [x][k] tile (k contiguous): rows of 128 bytes, the chunk c of row x at position c ^ ((x >> 1) & 7) --
//     sixteen rows of a ds_read_b128 then cover all 64 banks;
//   [k][x] tile: rows of BX floats; an MFMA lane reads single floats, 32 consecutive ones per half wave,
//     and the half waves read rows four apart: those are exchanged by 32 columns.
template <int BX, bool KC> struct Dense {
  static constexpr uint32_t kBytes = BX * 128, kInstr = BX / 32, kPerRow = KC ? 8 : BX / 4;
  __device__ static __forceinline__ uint32_t swz(uint32_t row) { return KC ? (row >> 1) & 7u : ((row >> 2) & 1u) << 3; }
  // this lane's byte offset for wave instruction `it` of a slice
  __device__ static __forceinline__ uint32_t lane_offset(uint32_t it, int64_t s_x, int64_t s_k, uint32_t left) {
    const uint32_t e = it * (uint32_t)kGemmThreads + threadIdx.x % kGemmThreads, row = e / kPerRow, c = (e % kPerRow) ^ swz(row);
    return (uint32_t)(4 * chunk_offset<KC>(row, c * 4u, s_x, s_k, left));
  }
  __device__ static __forceinline__ void copy(const float* src, const uint32_t (&off)[kInstr], uint32_t tile, uint32_t wave) {
#pragma unroll
    for (uint32_t it = 0; it < kInstr; ++it) copy_part(src, off, it, tile, wave);
  }
  __device__ static __forceinline__ void copy_part(const float* src, const uint32_t (&off)[kInstr], uint32_t it, uint32_t tile, uint32_t wave) {
    copy_1k(src, off[it], tile + (it * (uint32_t)kGemmThreads + wave * 64u) * 16u);
  }
  // This lane's values of row / column x for the k of group g (eight k: four for each half wave).  Which
  // k goes into which of a group's four MFMAs is free as long as both operands agree.
  __device__ static __forceinline__ RawVec group(const char* tile, uint32_t x, uint32_t g, uint32_t h) {
    if (KC) return *(const RawVec*)(tile + x * 128u + (((2u * g + h) ^ swz(x)) << 4));
    const char* p = tile + (8u * g + 4u * h) * (BX * 4u) + (x ^ (h << 5)) * 4u;
    return RawVec{*(const float*)p, *(const float*)(p + BX * 4), *(const float*)(p + BX * 8), *(const float*)(p + BX * 12)};
  }
};

// MFMAs of one k-slice, in groups of four k-steps: the fragments of the next group are read from
// LDS BEFORE the MFMAs of the current one are issued (two register sets; scheduling barriers keep
// the compiler from sinking the reads to their first use), so the matrix cores never wait for an
// LDS round trip inside a slice.
// acc has NCH accumulator sets ("chains"); k-step s adds into set s % NCH.  A wave that owns a
// single 32 x 32 block would otherwise issue nothing but MFMAs that each wait for the one before.
template <int BM, int BN, int MB, int NB, bool AKC, bool BKC, int NCH>
__device__ __forceinline__ void mma_slice(v16f (&acc)[NCH][MB][NB], const float* As, const float* Bs, uint32_t wave_m, uint32_t wave_n,
                                          uint32_t lane) {
  constexpr int SA = Tile<float, BM>::stride(AKC), SB = Tile<float, BN>::stride(BKC), BK = Elem<float>::BK;
  constexpr int KG = 4, NGRP = BK / 2 / KG;   // k-steps per group, groups per slice
  const float* ap = As + (lane >> 5) * SA + wave_m * (MB * 32) + (lane & 31);
  const float* bp = Bs + (lane >> 5) * SB + wave_n * (NB * 32) + (lane & 31);
  float af[2][KG][MB], bf[2][KG][NB];
  auto read_group = [&](int set, int g) {
#pragma unroll
    for (int s = 0; s < KG; ++s) {
      const int kk = (g * KG + s) * 2;
#pragma unroll
      for (int i = 0; i < MB; ++i) af[set][s][i] = ap[kk * SA + i * 32];
#pragma unroll
      for (int j = 0; j < NB; ++j) bf[set][s][j] = bp[kk * SB + j * 32];
    }
  };
  read_group(0, 0);
#pragma unroll
  for (int g = 0; g < NGRP; ++g) {
    if (g + 1 < NGRP) read_group((g + 1) & 1, g + 1);
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int s = 0; s < KG; ++s)
#pragma unroll
      for (int i = 0; i < MB; ++i)
#pragma unroll
        for (int j = 0; j < NB; ++j)
          acc[s % NCH][i][j] = __builtin_amdgcn_mfma_f32_32x32x2f32(af[g & 1][s][i], bf[g & 1][s][j], acc[s % NCH][i][j], 0, 0, 0);
    __builtin_amdgcn_sched_barrier(0);
  }
}

template <typename T, int BM, int BN> struct Smem {
  static constexpr size_t kOperands = 2 * (Tile<T, BM>::ELEMS + Tile<T, BN>::ELEMS) * sizeof(T);   // double buffered
  static constexpr size_t kC = (size_t)BM * (BN + kCPad) * sizeof(float);
  static constexpr size_t kDense = 4 * (size_t)(BM + BN) * 128;   // four dense stages
  static constexpr size_t kMax2 = kOperands > kC ? kOperands : kC;
  static constexpr size_t kBytes = kMax2 > kDense ? kMax2 : kDense;
};

// T: float.  AKC / BKC: the operand's contiguous dimension is k.  AL: both operands' rows are 16-byte
// aligned (the launcher looks).
// KS: halves of the workgroup that share its k (GemmArgs::halves); each has LDS stages of its own, and they
// walk their slices side by side.
// CS: column sums of B ride along (GemmArgs::col_sum; AKC and BKC false).  The workgroups of the first tile row take them from
// the B fragments that they multiply anyway, half of each slice by either wave row.  A slice's values are added pairwise before
// they join a running sum: one of four, which join the total every 32 slices, or in the loop of unaligned rows one, which joins it every
// eight.  However many rows: the total keeps what its additions lose (ColTotal).
template <typename T, int BM, int BN, bool AKC, bool BKC, bool AL, int KS, bool CS>
__global__ __launch_bounds__(kGemmThreads * KS, BM == 64 ? 2 : 1) void lt_gemm_kernel(const GemmArgs a) {
  static_assert(!CS || (!AKC && !BKC), "a weight gradient");
  constexpr int MB = BM / 64, NB = BN / 64, BK = Elem<T>::BK;
  constexpr size_t kHalf = Smem<T, BM, BN>::kBytes;
  __shared__ __attribute__((aligned(16))) char smem_all[KS * kHalf];
  __shared__ __attribute__((aligned(16))) float col_lds[CS ? KS * 2 * BN : 4];   // [half][wave row][column]
  const uint32_t touched = touch_args<GemmArgs>();
  const uint32_t half = KS > 1 ? __builtin_amdgcn_readfirstlane(threadIdx.x / kGemmThreads) : 0u;
  char* const smem = smem_all + half * kHalf;
  // LDS map: A buffer 0, A buffer 1, B buffer 0, B buffer 1 (the C tile of the epilogue reuses it)
  T* const lds = (T*)smem;
  auto As = [&](uint32_t buf) { return lds + buf * Tile<T, BM>::ELEMS; };
  auto Bs = [&](uint32_t buf) { return lds + 2 * Tile<T, BM>::ELEMS + buf * Tile<T, BN>::ELEMS; };
  const uint32_t tid = threadIdx.x % kGemmThreads, lane = tid & 63, wave = tid >> 6;
  const uint32_t wave_m = wave >> 1, wave_n = wave & 1;
  const uint32_t tile_m = blockIdx.y * BM, tile_n = blockIdx.x * BN;
  const uint32_t batch = blockIdx.z / a.splits, split = blockIdx.z % a.splits;
  // this workgroup's share of k: whole slices, split evenly
  const uint32_t slices = (a.k + BK - 1) / BK, per = (slices + a.splits - 1) / a.splits;
  const uint32_t k_begin = min(a.k, split * per * BK), k_end = min(a.k, (split + 1) * per * BK);
  const uint32_t b0 = batch / a.batch1, b1 = batch % a.batch1;
  const T* A = (const T*)a.a.ptr + (int64_t)b0 * a.a.s_b0 + (int64_t)b1 * a.a.s_b1;
  const T* B = (const T*)a.b.ptr + (int64_t)b0 * a.b.s_b0 + (int64_t)b1 * a.b.s_b1;
  const int64_t a_outer = AKC ? a.a.s_row : a.a.s_col, b_outer = BKC ? a.b.s_col : a.b.s_row;
  constexpr int NCH = MB * NB == 1 ? 2 : 1;   // independent accumulator chains per block
  v16f accs[NCH][MB][NB];
#pragma unroll
  for (int c = 0; c < NCH; ++c)
#pragma unroll
    for (int i = 0; i < MB; ++i)
#pragma unroll
      for (int j = 0; j < NB; ++j)
#pragma unroll
        for (int r = 0; r < 16; ++r) accs[c][i][j][r] = 0.0f;

  const bool summing = CS && tile_m == 0u;
  float csum[4][NB];
  ColTotal ctot[NB];
#pragma unroll
  for (int j = 0; j < NB; ++j) csum[0][j] = csum[1][j] = csum[2][j] = csum[3][j] = 0.0f;
  auto join_columns = [&]() __attribute__((always_inline)) {
#pragma unroll
    for (int j = 0; j < NB; ++j) {
      ctot[j].add((csum[0][j] + csum[1][j]) + (csum[2][j] + csum[3][j]));
      csum[0][j] = csum[1][j] = csum[2][j] = csum[3][j] = 0.0f;
    }
  };
  // this wave row's half of a slice in a padded tile: eight k for each half wave
  auto add_columns = [&](const T* tile) {
    const T* p = tile + ((lane >> 5) * 16u + wave_m * 8u) * Tile<T, BN>::stride(false) + wave_n * (NB * 32) + (lane & 31u);
#pragma unroll
    for (int j = 0; j < NB; ++j) {
      float t[8];
#pragma unroll
      for (int e = 0; e < 8; ++e) t[e] = p[e * Tile<T, BN>::stride(false) + j * 32];
      csum[0][j] += ((t[0] + t[1]) + (t[2] + t[3])) + ((t[4] + t[5]) + (t[6] + t[7]));
    }
  };
  GroupRegs<Groups<T, BM>::N> ga;
  GroupRegs<Groups<T, BN>::N> gb;
  // Whole slices of k are fetched in 16-byte chunks with no checks; what is left of k goes through the
  // checked path below.  The last chunk of a tile over the edge may reach up to three elements past its
  // row, into the next one (in bounds if rows are at least that far apart): then the slice with the
  // operand's last row has to be a checked one.
  const uint32_t left_m = a.m - tile_m, left_n = a.n - tile_n;
  const bool a_over = !AKC && left_m < (uint32_t)BM && (a.m & 3u) != 0u, b_over = !BKC && left_n < (uint32_t)BN && (a.n & 3u) != 0u;
  uint32_t n = (k_end - k_begin) / BK;   // whole slices
  if ((a_over && a_outer < 4) || (b_over && b_outer < 4)) n = 0u;
  else if ((a_over || b_over) && n > 0u && k_begin + n * BK == a.k) --n;
  // The halves walk theirs in the same n steps, between the same barriers.  Of an odd number the first takes one more; the
  // second has nothing to multiply in the last step: as a slice of the rest it took 1 to 2 us (1000 x 1024 x 800 21.6 -> 20.2, 600 x 768
  // x 800 19.8 -> 17.7).  (A single slice is left to the rest.)
  if (KS > 1 && n < 2u) n = 0u;
  const uint32_t both = KS > 1 ? n / 2u : n, k_rest = k_begin + n * BK;   // steps in which every half multiplies
  if (KS > 1) n -= both;
  const uint32_t mine = half == 0u ? n : both, k_first = k_begin + half * n * BK;
  const T* const pa = A + (int64_t)tile_m * a.a.s_row + (int64_t)k_first * a.a.s_col;
  const T* const pb = B + (int64_t)tile_n * a.b.s_col + (int64_t)k_first * a.b.s_row;
  const int64_t step_a = BK * a.a.s_col, step_b = BK * a.b.s_row;   // elements per slice of k
  if (AL && n > 0u) {
    // Four LDS stages: the MFMAs of slice j run from registers, the fragments of slice j + 1 are read from
    // its stage, slices j + 2 .. j + 4 are on their way from global memory into theirs.  Behind the
    // barrier of slice j slice j + 1 has landed for every wave, and every wave's reads of slice j's stage,
    // which is copied into next, have returned.  (Copies past the end: the last slice again, unused.)
    typedef Dense<BM, AKC> DA;
    typedef Dense<BN, BKC> DB;
    constexpr uint32_t kStage = DA::kBytes + DB::kBytes, kPer = DA::kInstr + DB::kInstr;
    const uint32_t wave_u = __builtin_amdgcn_readfirstlane(wave), h = lane >> 5;
    const uint32_t lds0 = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) char*)smem;
    uint32_t a_off[DA::kInstr], b_off[DB::kInstr];
#pragma unroll
    for (uint32_t it = 0; it < DA::kInstr; ++it) a_off[it] = DA::lane_offset(it, a.a.s_row, a.a.s_col, left_m);
#pragma unroll
    for (uint32_t it = 0; it < DB::kInstr; ++it) b_off[it] = DB::lane_offset(it, a.b.s_col, a.b.s_row, left_n);
    struct Frags {
      RawVec a[BK / 8][MB], b[BK / 8][NB];
    };
    // this lane's part of group g of the slice in `stage`, of A or of B
    auto read_a = [&](Frags& f, uint32_t stage, int g) {
#pragma unroll
      for (int i = 0; i < MB; ++i) f.a[g][i] = DA::group(smem + stage * kStage, wave_m * (BM / 2) + i * 32u + (lane & 31u), (uint32_t)g, h);
    };
    auto read_b = [&](Frags& f, uint32_t stage, int g) {
#pragma unroll
      for (int j = 0; j < NB; ++j) f.b[g][j] = DB::group(smem + stage * kStage + DA::kBytes, wave_n * (BN / 2) + j * 32u + (lane & 31u), (uint32_t)g, h);
    };
    // k step e of group g
    auto mma = [&](const Frags& f, int g, int e) {
#pragma unroll
      for (int i = 0; i < MB; ++i)
#pragma unroll
        for (int j = 0; j < NB; ++j)
          accs[e % NCH][i][j] = __builtin_amdgcn_mfma_f32_32x32x2f32(f.a[g][i][e], f.b[g][j][e], accs[e % NCH][i][j], 0, 0, 0);
    };
#define LT_COPY(I, STAGE)                                                                  \
  {                                                                                       \
    const int64_t sl = min((uint32_t)(I), mine - 1u);                                     \
    DA::copy(pa + sl * step_a, a_off, lds0 + (STAGE) * kStage, wave_u);                   \
    DB::copy(pb + sl * step_b, b_off, lds0 + (STAGE) * kStage + DA::kBytes, wave_u);      \
  }
    auto add_frags = [&](const Frags& f, auto sum, int set) __attribute__((always_inline)) {
      constexpr int g = decltype(sum)::value > 0 ? 2 * (int)decltype(sum)::value - 2 : 0;
#pragma unroll
      for (int j = 0; j < NB; ++j) {
        const RawVec x = f.b[g][j], y = f.b[g + 1][j];
        csum[set][j] += ((x.x + x.y) + (x.z + x.w)) + ((y.x + y.y) + (y.z + y.w));
      }
    };
    // One slice.  A wave issues in order, and the compiler, left alone, put the LDS reads of the next slice behind the
    // MFMAs and waited for them, twice a slice.  So every MFMA step is followed by one piece of the other work, and nothing
    // moves across: first the reads of the next slice, which have to be back at its barrier, then the copies.  Of the two
    // workgroups of 1024 x 2048 x 2048 on a compute unit the hardware serves the older one first: its loop 41 -> 33.5 us, the
    // other's 70 -> 66, which is what all their MFMAs take at the 2.0 GHz that the card keeps under them; twelve such layers
    // 850 -> 812 us, a head's three products (2048 x 1024 x 1000) 131.6 -> 124.7.
    // (sum: not 0: this wave adds up the columns of groups 2 sum - 2 and 2 sum - 1 as well.)
    auto slice = [&](const Frags& cur, Frags& next, uint32_t next_stage, uint32_t copy_slice, uint32_t copy_stage, auto sum, int set) __attribute__((always_inline)) {
      constexpr int kSum = (int)decltype(sum)::value;
      const int64_t sl = min(copy_slice, mine - 1u);   // (past the end: the last slice again, unused)
      const float* const ca = pa + sl * step_a;
      const float* const cb = pb + sl * step_b;
      const uint32_t at = lds0 + copy_stage * kStage;
#pragma unroll
      for (int s = 0; s < BK / 2; ++s) {
        mma(cur, s / 4, s % 4);
        if (s < BK / 4 && s % 2 == 0) read_a(next, next_stage, s / 2);
        if (s < BK / 4 && s % 2 == 1) read_b(next, next_stage, s / 2);
        if (s >= BK / 4) {
#pragma unroll
          for (uint32_t it = 0; it < kPer; ++it)
            if (it * 8u / kPer == (uint32_t)s - BK / 4) {
              if (it < DA::kInstr) DA::copy_part(ca, a_off, it, at, wave_u);
              else DB::copy_part(cb, b_off, it - DA::kInstr, at + DA::kBytes, wave_u);
            }
        }
        if (kSum > 0 && s == BK / 2 - 2) add_frags(cur, sum, set);
        __builtin_amdgcn_sched_barrier(0);
      }
    };
#define LT_SLICE(J, CUR, NEXT)                                                       \
  {                                                                                  \
    landed_and_read<2 * kPer>();                                                     \
    __syncthreads();                                                                 \
    __builtin_amdgcn_sched_barrier(0);                                               \
    slice(CUR, NEXT, ((J) + 1) & 3, i + (J) + 4u, (J) & 3, sum, (J));                \
  }
// the last ones: a half may have nothing left to multiply
#define LT_LAST(J, CUR, NEXT)                      \
  {                                                \
    landed_and_read<0>();                          \
    __syncthreads();                               \
    if (i + (J) < mine) {                          \
      _Pragma("unroll") for (int g = 0; g < BK / 8; ++g) { \
        read_a(NEXT, ((J) + 1) & 3, g);            \
        read_b(NEXT, ((J) + 1) & 3, g);            \
      }                                            \
      _Pragma("unroll") for (int s = 0; s < BK / 2; ++s) mma(CUR, s / 4, s % 4); \
      if (kSum > 0) add_frags(CUR, sum, J);        \
    }                                              \
  }
    LT_COPY(0, 0);
    LT_COPY(1, 1);
    LT_COPY(2, 2);
    LT_COPY(3, 3);
    landed<3 * kPer>();
    __syncthreads();
    // (every version has the same barriers)
    auto pipeline = [&](auto sum) __attribute__((always_inline)) {
      constexpr int kSum = (int)decltype(sum)::value;
      Frags f0, f1;
#pragma unroll
      for (int g = 0; g < BK / 8; ++g) {
        read_a(f0, 0, g);
        read_b(f0, 0, g);
      }
      uint32_t i = 0;
      for (; i + 4u <= both; i += 4u) {
        LT_SLICE(0, f0, f1);
        LT_SLICE(1, f1, f0);
        LT_SLICE(2, f0, f1);
        LT_SLICE(3, f1, f0);
        if (kSum > 0 && (i & 31u) == 28u) join_columns();
      }
      if (i < n) {   // (everything has been copied by now)
        LT_LAST(0, f0, f1);
        LT_LAST(1, f1, f0);
        LT_LAST(2, f0, f1);
        if (KS > 1 && i + 3u < n) LT_LAST(3, f1, f0);   // (the first half's odd one)
      }
    };
    if (!CS || !summing) pipeline(Num<0>());
    else if (wave_m == 0u) pipeline(Num<1>());
    else pipeline(Num<2>());
    landed<0>();   // nothing may still be on its way into LDS when it is used again
#undef LT_LAST
#undef LT_SLICE
#undef LT_COPY
  }
  if (!AL && n > 0u) {
    // the loads of slice j + 1 under the MFMAs of slice j, two padded buffers, one barrier per slice
    const Offsets<BM> a_off = unaligned_offsets<BM, AKC>(a.a.s_row, a.a.s_col, left_m);
    const Offsets<BN> b_off = unaligned_offsets<BN, BKC>(a.b.s_col, a.b.s_row, left_n);
    fetch_unaligned<BM>(ga, pa, a_off);
    fetch_unaligned<BN>(gb, pb, b_off);
    auto step = [&](uint32_t j, bool multiply) {
      stash_tile<BM, AKC>(ga, As(j & 1u));
      stash_tile<BN, BKC>(gb, Bs(j & 1u));
      const int64_t nx = min(j + 1u, mine - 1u);
      fetch_unaligned<BM>(ga, pa + nx * step_a, a_off);
      fetch_unaligned<BN>(gb, pb + nx * step_b, b_off);
      __syncthreads();
      if (multiply) {
        mma_slice<BM, BN, MB, NB, AKC, BKC, NCH>(accs, As(j & 1u), Bs(j & 1u), wave_m, wave_n, lane);
        if (summing) add_columns(Bs(j & 1u));
      }
    };
    // (a loop inside a loop: 8192 rows, 1030 x 1032, 312 us, with a branch in each step 316; 307 in one chain, 312 with the sums in a
    // launch of their own)
    for (uint32_t j = 0; j < both;) {
      const uint32_t to = CS ? min(j + 8u, both) : both;
#pragma unroll 1
      for (; j < to; ++j) step(j, true);
      if (summing) join_columns();
    }
    if (KS > 1 && both < n) step(both, half == 0u);   // (the first half's odd one)
  }
  // the rest of k: every access checked, one slice at a time, by the first half
#pragma unroll 1
  for (uint32_t k0 = k_rest; k0 < k_end; k0 += BK) {
    if (half == 0u) {
      fetch_tile<T, BM, AKC>(ga, A, a.a.s_row, a.a.s_col, tile_m, k0, a.m, k_end);
      fetch_tile<T, BN, BKC>(gb, B, a.b.s_col, a.b.s_row, tile_n, k0, a.n, k_end);
    }
    __syncthreads();
    if (half == 0u) {
      stash_tile<BM, AKC>(ga, As(0));
      stash_tile<BN, BKC>(gb, Bs(0));
    }
    __syncthreads();
    if (half == 0u) {
      mma_slice<BM, BN, MB, NB, AKC, BKC, NCH>(accs, As(0), Bs(0), wave_m, wave_n, lane);
      if (summing) add_columns(Bs(0));
    }
  }
  v16f (&acc)[MB][NB] = accs[0];
  if (NCH > 1) {
#pragma unroll
    for (int i = 0; i < MB; ++i)
#pragma unroll
      for (int j = 0; j < NB; ++j)
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[i][j][r] += accs[NCH - 1][i][j][r];
  }
  if (summing) {
    join_columns();
    // (read behind the epilogue's barriers)
#pragma unroll
    for (int j = 0; j < NB; ++j) {
      float t = ctot[j].value();
      t += __shfl_xor(t, 32);
      if (lane < 32u) col_lds[(half * 2u + wave_m) * BN + wave_n * (BN / 2) + j * 32u + lane] = t;
    }
  }
  // split-K: this workgroup's partial product goes to its own fp32 copy of the output, row major
  float* const raw = a.split_ws ? a.split_ws + (size_t)split * ((size_t)a.batch0 * a.batch1 * a.m * a.n) : nullptr;
  epilogue<false, BM, BN, MB, NB, KS, kHalf>(a, acc, (float*)smem_all, tile_m, tile_n, wave_m, wave_n, lane, batch, raw);
  if (summing) finish_columns<BN, 2 * KS>(a, col_lds, tile_n, split);
  args_touched(touched);
}

// ---- small contractions -------------------------------------------------------------------------
// A product of a few dozen 64 x 64 tiles leaves most compute units idle, and splitting its k over
// workgroups costs a second launch that adds the partial products up (for a 128 x 784 x 512 layer
// two launches of 5 to 7 microseconds each, most of it launch and memory latency).  Here a
// workgroup of eight wavefronts owns a 32 x 32 tile of the output and splits k INSIDE the
// workgroup: every wave contracts an eighth of k (whole groups of 8) for the whole tile, with its
// operands fetched from global memory straight into the MFMA 32x32x2 register layout -- lane
// (x, h) supplies A[x][k] and B[k][x] for the k of half h, and which k of a group goes into which
// of its four MFMAs is free as long as both operands agree, so a lane takes four CONSECUTIVE k
// (4 h .. 4 h + 3): one 16-byte load where k is the operand's contiguous dimension, four 4-byte
// loads that neighbouring lanes coalesce where it is not.  No LDS staging and no barrier in the
// loop; two groups (16 k) or kSmallG (32 k) are in flight per wave while as many are multiplied (launch_small).  The
// partial tiles of the waves meet in LDS, are added in a fixed order, and the post program runs on
// the sum: one launch.  (A tile may also be two blocks of 32 x 32: then two times four waves.)
// A long k over very few tiles (a batch of 8 rows against a 2048 x 2048 weight: 64 tiles) would
// leave three quarters of the compute units idle and every wave with several dependent round trips
// to memory, so there `splits` workgroups share a tile, each with a slice of k.  Their partial
// tiles (4 KB each) go to a scratch with relaxed device-scope stores, each workgroup takes a ticket
// of its tile, and the one that draws the last ticket adds the partial tiles up in split order
// (deterministic) and runs the post program -- the same exchange as in the reductions, still one
// launch.
constexpr int kSmallThreads = 512, kSmallWaves = 8, kSmallG = 4, kSmallStride = 32 + kCPad;

// Which tile a workgroup works on: grid = (column tiles x workgroups per tile, row tiles, batch), so that
// nothing is divided in the usual case (an integer division costs some 250 cycles at a kernel's start,
// and one flat index took five of them).  The workgroups of a tile are neighbours.
struct SmallTile {
  uint32_t number, row, col, split, b0, b1;
};
__device__ __forceinline__ SmallTile small_tile(const GemmArgs& a) {
  // everything the operands' addresses need, read in one go (field by field, each behind the use of the one
  // before, it is one wait per field)
  asm volatile("" : : "s"(a.splits), "s"(a.batch1), "s"(a.tiles_n), "s"(a.m), "s"(a.n), "s"(a.k), "s"(a.a.ptr), "s"(a.a.s_row), "s"(a.a.s_col),
               "s"(a.a.s_b0), "s"(a.b.ptr), "s"(a.b.s_row), "s"(a.b.s_col), "s"(a.b.s_b0), "s"(a.o_row), "s"(a.post.fast), "s"(a.post.n_in),
               "s"(a.post.n_slots), "s"(a.post.full_vec_ok), "s"(a.post.in[0].ptr), "s"(a.post.in[0].mode), "s"(a.post.in[0].dtype), "s"(a.post.in[0].fetch));
  SmallTile t;
  t.row = blockIdx.y;
  t.col = blockIdx.x;
  t.split = 0u;
  if (a.splits > 1u) {
    t.col = blockIdx.x / a.splits;
    t.split = blockIdx.x - t.col * a.splits;
  }
  t.b0 = blockIdx.z;
  t.b1 = 0u;
  if (a.batch1 > 1u) {
    t.b0 = blockIdx.z / a.batch1;
    t.b1 = blockIdx.z - t.b0 * a.batch1;
  }
  t.number = (blockIdx.z * gridDim.y + t.row) * a.tiles_n + t.col;
  return t;
}

// The sum of a tile's partial quads, `stride` floats apart, in split order (deterministic).  They are all asked for before
// the first is added: read one by one, each waits for its own way to memory and back.  (And no more of them than there are, to the
// next power of two: these loads pass by the caches.)
constexpr int kMaxShare = 8;
template <int N>
__device__ __forceinline__ float4 sum_parts_of(const float* parts, uint32_t stride, uint32_t splits) {
  float4 t[N];
#pragma unroll
  for (uint32_t sp = 0; sp < (uint32_t)N; ++sp) t[sp] = published4(parts + (size_t)min(sp, splits - 1u) * stride);
  float4 sum = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
#pragma unroll
  for (uint32_t sp = 0; sp < (uint32_t)N; ++sp)
    if (sp < splits) {
      sum.x += t[sp].x; sum.y += t[sp].y; sum.z += t[sp].z; sum.w += t[sp].w;
    }
  return sum;
}
__device__ __forceinline__ float4 sum_parts(const float* parts, uint32_t stride, uint32_t splits) {
  if (splits <= 2u) return sum_parts_of<2>(parts, stride, splits);
  if (splits <= 4u) return sum_parts_of<4>(parts, stride, splits);
  return sum_parts_of<kMaxShare>(parts, stride, splits);
}

template <bool V, int G>
__device__ __forceinline__ void small_fetch(float (&v)[G][4], const float* base, int64_t s_k, uint32_t k0, uint32_t k_end) {
#pragma unroll
  for (int g = 0; g < G; ++g) {
    const uint32_t kg = k0 + (uint32_t)g * 8u;
    if (V) {   // k is contiguous and a multiple of 4: the four are valid together
      const bool ok = kg < k_end;
      const float4 t = *(const float4*)(base + (ok ? kg : 0u));
      v[g][0] = ok ? t.x : 0.0f; v[g][1] = ok ? t.y : 0.0f; v[g][2] = ok ? t.z : 0.0f; v[g][3] = ok ? t.w : 0.0f;
    } else {
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const bool ok = kg + (uint32_t)j < k_end;
        const float t = base[(int64_t)(ok ? kg + (uint32_t)j : 0u) * s_k];   // (past the end: element 0 again, in bounds, zeroed)
        v[g][j] = ok ? t : 0.0f;
      }
    }
  }
}

template <int G>
__device__ __forceinline__ void small_mma(v16f& acc0, v16f& acc1, const float (&av)[G][4], const float (&bv)[G][4]) {
#pragma unroll
  for (int g = 0; g < G; ++g) {
    acc0 = __builtin_amdgcn_mfma_f32_32x32x2f32(av[g][0], bv[g][0], acc0, 0, 0, 0);
    acc1 = __builtin_amdgcn_mfma_f32_32x32x2f32(av[g][1], bv[g][1], acc1, 0, 0, 0);
    acc0 = __builtin_amdgcn_mfma_f32_32x32x2f32(av[g][2], bv[g][2], acc0, 0, 0, 0);
    acc1 = __builtin_amdgcn_mfma_f32_32x32x2f32(av[g][3], bv[g][3], acc1, 0, 0, 0);
  }
}

template <int G>
__device__ __forceinline__ float small_colsum(float s, const float (&bv)[G][4]) {
#pragma unroll
  for (int g = 0; g < G; ++g) s += (bv[g][0] + bv[g][1]) + (bv[g][2] + bv[g][3]);
  return s;
}

// Programs whose inputs are fp32 and read in full, by column or as one value: an output whose rows are no whole vectors
// (n = 10) still has its inputs asked for under the contraction, element by element.
__device__ __forceinline__ bool single_elements(const EwProg& p) {
  if (p.n_in > 2u || p.n_slots > 16u) return false;
  bool ok = true;
  for (uint32_t k = 0; k < p.n_in; ++k) ok = ok && p.in[k].dtype == kF32 && (p.in[k].mode == kFull || p.in[k].mode == kRowVec || p.in[k].mode == kScalar);
  return ok;
}
// `i`: the quad's flat index in the output, `col` its column, n columns (what would be past the row's end: its last element again)
template <int N>
__device__ __forceinline__ void fetch_elements(Staged<N>& st, const EwProg& p, uint32_t i, uint32_t col, uint32_t n) {
#pragma unroll
  for (int k = 0; k < 2; ++k) {
    if ((uint32_t)k < p.n_in) {
      const EwIn& in = p.in[k];
      const float* src = (const float*)in.ptr;
#pragma unroll
      for (uint32_t e = 0; e < (uint32_t)kVec; ++e) {
        const uint32_t c = min(e, n - 1u - col);
        st.vec[k][e] = src[in.mode == kFull ? i + c : in.mode == kRowVec ? col + c : 0u];
      }
    }
  }
}
template <int NS, int N>
__device__ __forceinline__ RF<NS> place_elements(RF<NS> f, const EwProg& p, const Staged<N>& st) {
#pragma unroll
  for (int k = 0; k < 2; ++k)
#pragma unroll
    for (int v = 0; v < kVec; ++v) f.e[v][k] = st.vec[k][v];
  return f;
}

// TM x TN: blocks of 32 x 32 per workgroup tile (1 x 1, 2 x 1 or 2 x 2); the eight waves are NB =
// TM * TN blocks times 8 / NB shares of k.  AV / BV: k is the operand's contiguous dimension and
// every group of four is a whole, 16-byte aligned vector (the launcher checks the pointer, the
// strides and k % 4).  CS: the column sums of B ride along (GemmArgs::col_sum); a variant of its own, because the
// second program costs 40 registers that the plain product does not have to carry.
// FOUR: four groups of k in flight, not two (launch_small).
template <int TM, int TN, bool AV, bool BV, bool CS, bool FOUR>
__device__ __forceinline__ void small_tile32(const GemmArgs& a) {
  constexpr uint32_t NB = TM * TN, KW = kSmallWaves / NB;      // blocks, k shares inside the workgroup
  static_assert(!CS || NB == 1, "column sums ride with tiles of 32 x 32");
  static_assert(!CS || !FOUR, "two chunks to a column sum's four groups");
  constexpr int G = NB > 1 || FOUR ? kSmallG : 2;              // groups of 8 k in flight, and as many being multiplied
  constexpr uint32_t kQuads = NB * 256u, QT = (kQuads + kSmallThreads - 1u) / kSmallThreads;   // quads of the tile, per thread
  __shared__ __attribute__((aligned(16))) float Cs[kSmallWaves * 32 * kSmallStride];
  __shared__ uint32_t is_last;
  __shared__ float colp[CS ? kSmallThreads : 1];
  __shared__ __attribute__((aligned(16))) float coltot[CS ? 32 : 4];
  const uint32_t lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  constexpr uint32_t kColWave = kQuads / 64u % (uint32_t)kSmallWaves;
  const uint32_t block = wave % NB, kway = wave / NB, bm = block / TN, bn = block % TN;
  const SmallTile st = small_tile(a);
  const uint32_t tile = st.number, split = st.split, tile_m = st.row * (32u * TM), tile_n = st.col * (32u * TN), b0 = st.b0, b1 = st.b1;
  const float* A = (const float*)a.a.ptr + (int64_t)b0 * a.a.s_b0 + (int64_t)b1 * a.a.s_b1;
  const float* B = (const float*)a.b.ptr + (int64_t)b0 * a.b.s_b0 + (int64_t)b1 * a.b.s_b1;
  // this workgroup's slice of k, and this wave's share of it: whole groups of 8
  const uint32_t per_wg = (((a.k + 7u) / 8u) + a.splits - 1u) / a.splits;
  const uint32_t wg_begin = min(a.k, split * per_wg * 8u), wg_end = min(a.k, (split + 1u) * per_wg * 8u);
  const uint32_t groups = (wg_end - wg_begin + 7u) / 8u, per = (groups + KW - 1u) / KW;
  const uint32_t k_begin = min(wg_end, wg_begin + kway * per * 8u), k_end = min(wg_end, wg_begin + (kway + 1u) * per * 8u);
  const uint32_t x = lane & 31u, h = lane >> 5;
  // rows and columns over the edge are read as copies of the last one (in bounds; never stored)
  const float* ap = A + (int64_t)min(tile_m + bm * 32u + x, a.m - 1u) * a.a.s_row;
  const float* bp = B + (int64_t)min(tile_n + bn * 32u + x, a.n - 1u) * a.b.s_col;
  // The post program and, where every quad of the tile is a whole aligned vector inside the
  // output, its inputs for this thread's quads are asked for now, so that they travel under the
  // contraction.  Quad q of the tile: block q / 256, row (q % 256) / 8 of it, columns 4 (q % 8) ..
  // (the program lives in the lanes of two registers: fetched while every lane is active)
  const EwProg& p = a.post;
  const ProgRegs pr = load_prog_regs(p);
  // column sums of B ride along in the first tile row (every column block exactly once)
  const bool cols_here = CS && tile_m == 0u;                    // (workgroup-uniform)
  // ... and the column program runs on a wave that has no quads of the tile
  const bool col_wave = cols_here && wave == kColWave;
  const uint32_t col_at = tile_n + (lane & 7u) * (uint32_t)kVec;   // (its first eight lanes)
  const EwProg& cp = a.col_post;
  const bool col_fast = CS && cp.fast && cp.full_vec_ok && cp.n_in <= 4u && cp.n_slots <= 8u && (a.n & 3u) == 0u;
  const ProgRegs cpr = CS ? load_prog_regs(a.col_post) : ProgRegs{0u, 0.0f};
  float csum = 0.0f;
  // (a tile over the edge: quads past it read the last row's or column's inputs and are not stored)
  const bool fast = p.fast && p.full_vec_ok && p.n_in <= 4u && p.n_slots <= 8u && (a.n & 3u) == 0u;
  uint32_t qrow[QT], qcol[QT], qi[QT];
#pragma unroll
  for (uint32_t j = 0; j < QT; ++j) {
    const uint32_t q = (threadIdx.x + j * kSmallThreads) % kQuads, qb = q >> 8;   // (threads past the last quad: a copy, never used)
    qrow[j] = tile_m + (qb / TN) * 32u + ((q & 255u) >> 3);
    qcol[j] = tile_n + (qb % TN) * 32u + (q & 7u) * (uint32_t)kVec;
    qi[j] = (uint32_t)((int64_t)b0 * a.o_b0 + (int64_t)b1 * a.o_b1 + (int64_t)qrow[j] * a.o_row + qcol[j]);
  }
  const bool has_quad = threadIdx.x < kQuads;   // (wave-uniform: kQuads is a multiple of 64)
#pragma clang diagnostic push
#pragma clang diagnostic ignored "-Wuninitialized"
#pragma clang diagnostic ignored "-Wsometimes-uninitialized"
  Staged<4> staged[QT];
  if (fast && has_quad) {
#pragma unroll
    for (uint32_t j = 0; j < QT; ++j) {
      const uint32_t r = min(qrow[j], a.m - 1u), c = min(qcol[j], a.n - 4u);
      staged[j] = fetch_inputs_at<4, false, false>(p, (uint32_t)((int64_t)b0 * a.o_b0 + (int64_t)b1 * a.o_b1 + (int64_t)r * a.o_row + c), (b0 * a.batch1 + b1) * a.m + r, c);
    }
  }
#pragma clang diagnostic pop
  // (an output whose rows are no whole vectors: the inputs element by element, but all at once and as early)
  const bool loose = !fast && single_elements(p);
  if (loose && has_quad) {
#pragma unroll
    for (uint32_t j = 0; j < QT; ++j)
      fetch_elements(staged[j], p, qi[j] - qcol[j] + min(qcol[j], a.n - 1u) - (qrow[j] < a.m ? 0u : (uint32_t)((qrow[j] - (a.m - 1u)) * a.o_row)), min(qcol[j], a.n - 1u), a.n);
  }
  if (col_wave && col_fast) staged[0] = fetch_inputs_at<4, false, false>(cp, min(col_at, a.n - 4u), 0u, min(col_at, a.n - 4u));
  v16f acc0, acc1;
#pragma unroll
  for (int r = 0; r < 16; ++r) acc0[r] = acc1[r] = 0.0f;
  constexpr uint32_t kChunk = (uint32_t)G * 8u;
  const uint32_t nch = (k_end - k_begin + kChunk - 1u) / kChunk;   // (wave-uniform)
  float a0[G][4], b0v[G][4], a1[G][4], b1v[G][4];
  const uint32_t kl = k_begin + 4u * h;   // this lane's first k
  if (nch > 0u) {
    small_fetch<AV, G>(a0, ap, a.a.s_col, kl, k_end);
    small_fetch<BV, G>(b0v, bp, a.b.s_row, kl, k_end);
  }
  for (uint32_t c = 0; c < nch; c += 2u) {
    if (c + 1u < nch) {
      small_fetch<AV, G>(a1, ap, a.a.s_col, kl + (c + 1u) * kChunk, k_end);
      small_fetch<BV, G>(b1v, bp, a.b.s_row, kl + (c + 1u) * kChunk, k_end);
    }
    small_mma<G>(acc0, acc1, a0, b0v);
    // (a wave's column sum: four groups, two chunks, at a time, which then join its running sum: with a chunk at a time
    // 1000 rows of N(0, 1) were 1.04e-7 from 64 bits instead of 0.92e-7)
    float four = cols_here ? small_colsum<G>(0.0f, b0v) : 0.0f;
    if (c + 2u < nch) {
      small_fetch<AV, G>(a0, ap, a.a.s_col, kl + (c + 2u) * kChunk, k_end);
      small_fetch<BV, G>(b0v, bp, a.b.s_row, kl + (c + 2u) * kChunk, k_end);
    }
    if (c + 1u < nch) {
      small_mma<G>(acc0, acc1, a1, b1v);
      if (cols_here) four = small_colsum<G>(four, b1v);
    }
    csum += four;
  }
  if (CS) colp[threadIdx.x] = csum;
  float* mine = Cs + wave * (32u * kSmallStride);   // (wave = kway * NB + block)
#pragma unroll
  for (int r = 0; r < 16; ++r) mine[((uint32_t)(r >> 2) * 8u + h * 4u + (uint32_t)(r & 3)) * kSmallStride + x] = acc0[r] + acc1[r];
  __syncthreads();
  float4 sum[QT];
#pragma unroll
  for (uint32_t j = 0; j < QT; ++j) {
    const uint32_t q = (threadIdx.x + j * kSmallThreads) % kQuads;
    const float* src = Cs + (q >> 8) * (32u * kSmallStride) + ((q & 255u) >> 3) * kSmallStride + (q & 7u) * (uint32_t)kVec;
    sum[j] = *(const float4*)src;
#pragma unroll
    for (uint32_t w = 1; w < KW; ++w) {   // share order: deterministic
      const float4 t = *(const float4*)(src + w * NB * (32u * kSmallStride));
      sum[j].x += t.x; sum[j].y += t.y; sum[j].z += t.z; sum[j].w += t.w;
    }
  }
  if (col_wave) {
    // the shares of k in order, lower half of the wave before the upper (deterministic); then the column program on quads of
    // four columns.  (One wave: its LDS accesses are in order.)
    if (lane < 32u) {
      float t = 0.0f;
#pragma unroll
      for (uint32_t w = 0; w < KW; ++w) {
        t += colp[w * 64u + lane];
        t += colp[w * 64u + 32u + lane];
      }
      if (a.col_red == kRedMean) t = t / (float)a.k;
      coltot[lane] = t;
    }
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    if (lane < 8u && col_at < a.n) {
      const uint32_t nv = a.n - col_at >= (uint32_t)kVec ? (uint32_t)kVec : a.n - col_at;
      Quad q;
#pragma unroll
      for (int e = 0; e < kVec; ++e) q.v[e] = coltot[lane * (uint32_t)kVec + (uint32_t)e];
      RF<16> f = col_fast ? place_inputs<16, 4, true, false, 0>(rf_zero<16>(), cp, staged[0], kVec) : load_inputs<16, kMaxIn, false, false>(rf_zero<16>(), cp, 0, col_at, nv);
      f = rf_set<16>(f, cp.anchor_slot, q);
      f = interp<16>(f, cpr, cp.n_code);
      store_outputs<16, false, false>(f, cp, 0, col_at, nv);
    }
  }
  if (a.splits > 1u) {
    // leave this workgroup's partial tile, take a ticket; whoever draws the last one goes on
    float* const parts = a.split_ws + (size_t)tile * a.splits * (NB * 1024u);
    if (has_quad) {
#pragma unroll
      for (uint32_t j = 0; j < QT; ++j)
        publish4(parts + (size_t)split * (NB * 1024u) + (size_t)((threadIdx.x + j * kSmallThreads) % kQuads) * 4u, sum[j]);
      all_published();
    }
    __syncthreads();
    if (threadIdx.x == 0u) {
      const uint32_t t = atomicAdd(&a.tickets[tile], 1u);
      is_last = (t == a.splits - 1u) ? 1u : 0u;
      if (t == a.splits - 1u) a.tickets[tile] = 0u;   // (every workgroup of the tile has been here)
    }
    __syncthreads();
    if (!is_last) return;
    if (has_quad) {
#pragma unroll
      for (uint32_t j = 0; j < QT; ++j) sum[j] = sum_parts(parts + (size_t)((threadIdx.x + j * kSmallThreads) % kQuads) * 4u, NB * 1024u, a.splits);
    }
  }
  if (!has_quad) return;
  const uint32_t n_code = p.n_code;
#pragma unroll
  for (uint32_t j = 0; j < QT; ++j) {
    Quad anchor;
    anchor.v[0] = sum[j].x; anchor.v[1] = sum[j].y; anchor.v[2] = sum[j].z; anchor.v[3] = sum[j].w;
    if (fast) {
      RF<16> f = place_inputs<16, 4, true, false, 0>(rf_zero<16>(), p, staged[j], kVec);
      f = rf_set<16>(f, p.anchor_slot, anchor);
      f = interp<16>(f, pr, n_code);
      if (qrow[j] < a.m && qcol[j] < a.n) store_outputs<16, true, false, 0>(f, p, 0, qi[j], kVec);
    } else if (qrow[j] < a.m && qcol[j] < a.n) {
      const uint32_t nvalid = a.n - qcol[j] >= (uint32_t)kVec ? (uint32_t)kVec : a.n - qcol[j];
      RF<16> f = loose ? place_elements(rf_zero<16>(), p, staged[j]) : load_inputs<16, kMaxIn, false, false>(rf_zero<16>(), p, 0, qi[j], nvalid);
      f = rf_set<16>(f, p.anchor_slot, anchor);
      f = interp<16>(f, pr, n_code);
      store_outputs<16, false, false>(f, p, 0, qi[j], nvalid);
    }
  }
}

// ---- tiny contractions --------------------------------------------------------------------------
// The same for products whose 32 x 32 tiles would number a few dozen (a layer of a small classifier, a few
// rows against a wide weight): tiles of 16 rows by 16 (or 64) columns on MFMA 16x16x4, so that four times as
// many compute units get one and a wave's share of k is a handful of loads that are all in flight at once.  What
// bounds it is launch and memory latency and the number of instructions a wave walks through: counters on
// 128 x 512 x 784 in 32 x 32 tiles (64 workgroups) gave 1350 instructions per wave, a fifth of its cycles, and as
// long again waiting for the matrix cores of a quarter of the chip.  Lane (x, q) supplies A[x][k] and B[k][x] for the four
// consecutive k at 16 g + 4 q of group g.
// BMODE: 0 = B element by element, 1 = four k at once (k contiguous), 2 = four columns at once (columns
// contiguous; the tile is then 64 columns wide, column 4 x + j in accumulator j).
template <bool AV, int BMODE>
__device__ __forceinline__ void small_tile16(const GemmArgs& a) {
  constexpr uint32_t NB = BMODE == 2 ? 4 : 1, kCols = 16u * NB, kStride = kCols + 4u, kQuads = 64u * NB;
  constexpr uint32_t G = BMODE == 2 ? 2 : 4;   // groups of 16 k in flight (and as many being multiplied)
  __shared__ __attribute__((aligned(16))) float Cs[kSmallWaves * 16 * kStride];
  __shared__ uint32_t is_last;
  const uint32_t lane = threadIdx.x & 63u, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), kw = blockDim.x >> 6;
  const SmallTile st = small_tile(a);
  const uint32_t split = st.split, tile_m = st.row * 16u, tile_n = st.col * kCols, b0 = st.b0, b1 = st.b1, x = lane & 15u, q = lane >> 4;
  const float* A = (const float*)a.a.ptr + (int64_t)b0 * a.a.s_b0 + (int64_t)b1 * a.a.s_b1;
  const float* B = (const float*)a.b.ptr + (int64_t)b0 * a.b.s_b0 + (int64_t)b1 * a.b.s_b1;
  // rows and columns over the edge are read as copies of the last one (in bounds; never stored)
  const float* ap = A + (int64_t)min(tile_m + x, a.m - 1u) * a.a.s_row;
  const float* bp = BMODE == 2 ? B + min(tile_n + 4u * x, a.n - 4u) : B + (int64_t)min(tile_n + x, a.n - 1u) * a.b.s_col;
  // this workgroup's slice of k and this wave's share of it: whole groups of 16
  const uint32_t per_wg = ((a.k + 15u) / 16u + a.splits - 1u) / a.splits;
  const uint32_t wg_begin = min(a.k, split * per_wg * 16u), wg_end = min(a.k, (split + 1u) * per_wg * 16u);
  const uint32_t per = ((wg_end - wg_begin + 15u) / 16u + kw - 1u) / kw;
  const uint32_t k_begin = min(wg_end, wg_begin + wave * per * 16u), k_end = min(wg_end, wg_begin + (wave + 1u) * per * 16u);
  float av[2][G][4], bv[2][G][4][NB];
  // (whole steps: a lane's own pointer plus a wave-uniform offset; the last step checks every k)
  const float *al = ap + (int64_t)(4u * q) * a.a.s_col, *bl = bp + (int64_t)(4u * q) * a.b.s_row;
  constexpr uint32_t kStep = G * 16u;
  typedef float V4 __attribute__((ext_vector_type(4), aligned(4)));   // (rows may start at any element)
  auto fetch = [&](int set, uint32_t k0) {
    const bool whole = k0 + kStep <= k_end;
#pragma unroll
    for (uint32_t g = 0; g < G; ++g) {
      const uint32_t kg = k0 + g * 16u + 4u * q;
      const bool in = kg < k_end;
      if (AV) {   // (k is a multiple of 4: the four are valid together)
        const RawVec t = *(const RawVec*)(in ? al + (k0 + g * 16u) : ap);
#pragma unroll
        for (int e = 0; e < 4; ++e) av[set][g][e] = t[e];
      } else {
#pragma unroll
        for (uint32_t e = 0; e < 4u; ++e) av[set][g][e] = *(whole || kg + e < k_end ? al + (int64_t)(k0 + g * 16u + e) * a.a.s_col : ap);
      }
      if (BMODE == 1) {
        const RawVec t = *(const RawVec*)(in ? bl + (k0 + g * 16u) : bp);
#pragma unroll
        for (int e = 0; e < 4; ++e) bv[set][g][e][0] = t[e];
      } else {
#pragma unroll
        for (uint32_t e = 0; e < 4u; ++e) {
          const float* src = whole || kg + e < k_end ? bl + (int64_t)(k0 + g * 16u + e) * a.b.s_row : bp;
          if (BMODE == 2) {
            const V4 t = *(const V4*)src;
#pragma unroll
            for (uint32_t j = 0; j < NB; ++j) bv[set][g][e][j] = t[j];
          } else {
            bv[set][g][e][0] = *src;
          }
        }
      }
    }
  };
  // The post program (its registers live in all lanes of a wave) and its inputs travel under the contraction.
  const EwProg& p = a.post;
  const ProgRegs pr = load_prog_regs(p);
  const uint32_t qrow = tile_m + (threadIdx.x % kQuads) / (4u * NB), qcol = tile_n + (threadIdx.x % (4u * NB)) * (uint32_t)kVec;
  // (a quad past an edge reads the last row's or column's inputs and is not stored)
  const uint32_t in_row = min(qrow, a.m - 1u), in_col = (a.n & 3u) == 0u ? min(qcol, a.n - 4u) : qcol;
  const uint32_t qi = (uint32_t)((int64_t)b0 * a.o_b0 + (int64_t)b1 * a.o_b1 + (int64_t)in_row * a.o_row + in_col);
  const bool has_quad = threadIdx.x < kQuads;   // (wave-uniform)
  const bool fast = p.fast && p.full_vec_ok && p.n_in <= 4u && p.n_slots <= 8u && (a.n & 3u) == 0u;
#pragma clang diagnostic push
#pragma clang diagnostic ignored "-Wuninitialized"
#pragma clang diagnostic ignored "-Wsometimes-uninitialized"
  Staged<4> staged;
  if (k_begin < k_end) fetch(0, k_begin);
  if (fast && has_quad) staged = fetch_inputs_at<4, false, false>(p, qi, (b0 * a.batch1 + b1) * a.m + in_row, in_col);
#pragma clang diagnostic pop
  typedef float v4f __attribute__((ext_vector_type(4)));
  v4f acc[2][NB];
#pragma unroll
  for (int c = 0; c < 2; ++c)
#pragma unroll
    for (uint32_t j = 0; j < NB; ++j) acc[c][j] = v4f{0.0f, 0.0f, 0.0f, 0.0f};
  auto mma = [&](int set, uint32_t k0) {
    if (k0 + kStep > k_end) {   // k past this wave's share: zero on both sides
#pragma unroll
      for (uint32_t g = 0; g < G; ++g)
#pragma unroll
        for (uint32_t e = 0; e < 4u; ++e) {
          const bool ok = k0 + g * 16u + 4u * q + e < k_end;
          av[set][g][e] = ok ? av[set][g][e] : 0.0f;
#pragma unroll
          for (uint32_t j = 0; j < NB; ++j) bv[set][g][e][j] = ok ? bv[set][g][e][j] : 0.0f;
        }
    }
#pragma unroll
    for (uint32_t g = 0; g < G; ++g)
#pragma unroll
      for (uint32_t e = 0; e < 4u; ++e)
#pragma unroll
        for (uint32_t j = 0; j < NB; ++j)
          acc[e & 1u][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(av[set][g][e], bv[set][g][e][j], acc[e & 1u][j], 0, 0, 0);
  };
  for (uint32_t k0 = k_begin; k0 < k_end; k0 += 2u * kStep) {
    if (k0 + kStep < k_end) fetch(1, k0 + kStep);
    mma(0, k0);
    if (k0 + 2u * kStep < k_end) fetch(0, k0 + 2u * kStep);
    if (k0 + kStep < k_end) mma(1, k0 + kStep);
  }
  float* mine = Cs + wave * (16u * kStride);
#pragma unroll
  for (uint32_t r = 0; r < 4u; ++r)
#pragma unroll
    for (uint32_t j = 0; j < NB; ++j) mine[(4u * q + r) * kStride + NB * x + j] = acc[0][j][r] + acc[1][j][r];
  __syncthreads();
  float4 sum = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
  if (has_quad) {
    const float* src = Cs + (qrow - tile_m) * kStride + (qcol - tile_n);
    sum = *(const float4*)src;
    if (kw == (uint32_t)kSmallWaves) {   // (all at once: a read behind the other costs an LDS latency each)
      float4 t[kSmallWaves];
#pragma unroll
      for (uint32_t w = 1; w < (uint32_t)kSmallWaves; ++w) t[w] = *(const float4*)(src + w * (16u * kStride));
#pragma unroll
      for (uint32_t w = 1; w < (uint32_t)kSmallWaves; ++w) {   // share order: deterministic
        sum.x += t[w].x; sum.y += t[w].y; sum.z += t[w].z; sum.w += t[w].w;
      }
    } else {
      for (uint32_t w = 1; w < kw; ++w) {
        const float4 t = *(const float4*)(src + w * (16u * kStride));
        sum.x += t.x; sum.y += t.y; sum.z += t.z; sum.w += t.w;
      }
    }
  }
  if (a.splits > 1u) {
    // leave this workgroup's partial tile, take a ticket; whoever draws the last one goes on
    float* const parts = a.split_ws + (size_t)st.number * a.splits * (kQuads * 4u);
    if (has_quad) {
      publish4(parts + (size_t)split * (kQuads * 4u) + threadIdx.x * 4u, sum);
      all_published();
    }
    __syncthreads();
    if (threadIdx.x == 0u) {
      const uint32_t t = atomicAdd(&a.tickets[st.number], 1u);
      is_last = (t == a.splits - 1u) ? 1u : 0u;
      if (t == a.splits - 1u) a.tickets[st.number] = 0u;   // (every workgroup of the tile has been here)
    }
    __syncthreads();
    if (!is_last) return;
    if (has_quad) sum = sum_parts(parts + threadIdx.x * 4u, kQuads * 4u, a.splits);
  }
  if (!has_quad) return;
  Quad anchor;
  anchor.v[0] = sum.x; anchor.v[1] = sum.y; anchor.v[2] = sum.z; anchor.v[3] = sum.w;
  const uint32_t n_code = p.n_code;
  if (fast) {
    RF<16> f = place_inputs<16, 4, true, false, 0>(rf_zero<16>(), p, staged, kVec);
    f = rf_set<16>(f, p.anchor_slot, anchor);
    f = interp<16>(f, pr, n_code);
    if (qrow < a.m && qcol < a.n) store_outputs<16, true, false, 0>(f, p, 0, qi, kVec);
  } else if (qrow < a.m && qcol < a.n) {
    const uint32_t nvalid = a.n - qcol >= (uint32_t)kVec ? (uint32_t)kVec : a.n - qcol;
    RF<16> f = load_inputs<16, kMaxIn, false, false>(rf_zero<16>(), p, 0, qi, nvalid);
    f = rf_set<16>(f, p.anchor_slot, anchor);
    f = interp<16>(f, pr, n_code);
    store_outputs<16, false, false>(f, p, 0, qi, nvalid);
  }
}

// TM x TN: the workgroup's tile in units of 16 (2 x 2, 4 x 2, 1 x 1, 1 x 4).
template <int TM, int TN, bool AV, bool BV, bool CS, bool FOUR>
__global__ __launch_bounds__(kSmallThreads) void lt_gemm_small_kernel(const GemmArgs a) {
  const uint32_t t = touch_args<GemmArgs>();
  if constexpr (TM == 1) small_tile16<AV, TN == 4 ? 2 : BV ? 1 : 0>(a);
  else small_tile32<TM / 2, TN / 2, AV, BV, CS, FOUR>(a);
  args_touched(t);
}

// four: groups of k in flight in tiles of 32 x 32 (those of other sizes come in one version)
template <int TM, int TN, bool CS>
static void launch_small_tile(const GemmArgs& a, bool av, bool bv, bool four, dim3 grid, uint32_t threads, hipStream_t s) {
  const dim3 block(threads);
  constexpr bool one = TM != 2 || TN != 2;
  if (TN == 4) bv = false;   // (columns contiguous, four at a time)
  if (av && bv) LT_LAUNCH((lt_gemm_small_kernel<TM, TN, true, true && TN != 4, CS, !CS>), grid, block, s, a);
  else if (av) LT_LAUNCH((lt_gemm_small_kernel<TM, TN, true, false, CS, one>), grid, block, s, a);
  else if (bv) LT_LAUNCH((lt_gemm_small_kernel<TM, TN, false, true && TN != 4, CS, !CS>), grid, block, s, a);
  else if (four && !CS) LT_LAUNCH((lt_gemm_small_kernel<TM, TN, false, false, CS, !CS>), grid, block, s, a);
  else LT_LAUNCH((lt_gemm_small_kernel<TM, TN, false, false, CS, one>), grid, block, s, a);
  char name[64];
  snprintf(name, sizeof(name), "lt_gemm_small_kernel<%d, %d, %s, %s, %s>", TM, TN, av ? "true" : "false", bv ? "true" : "false", CS ? "true" : "false");
  note_kernel(name);
}

static hipError_t launch_small(const GemmArgs& args, hipStream_t s) {
  GemmArgs a = args;
  // (64 x 64 tiles lost to the split pair on every shape measured and are not built)
  const bool t22 = a.tile_m == 32u && a.tile_n == 32u, t42 = a.tile_m == 64u && a.tile_n == 32u;
  const bool t11 = a.tile_m == 16u && a.tile_n == 16u, t14 = a.tile_m == 16u && a.tile_n == 64u;
  if (!t22 && !t42 && !t11 && !t14) return hipErrorInvalidValue;
  a.tiles_m = (a.m + a.tile_m - 1u) / a.tile_m;
  a.tiles_n = (a.n + a.tile_n - 1u) / a.tile_n;
  const uint64_t wgs = (uint64_t)a.tiles_m * a.tiles_n * a.batch0 * a.batch1;
  if (a.splits == 0u || wgs * a.splits > 0x7fffffffull || a.tiles_m > 65535u || (uint64_t)a.batch0 * a.batch1 > 65535u) return hipErrorInvalidValue;
  if (a.splits > 1u && (a.splits > (uint32_t)kMaxShare || !a.split_ws || !a.tickets)) return hipErrorInvalidValue;
  // column sums ride along only with an unshared, unbatched product whose B is [k, n] with rows contiguous
  if (a.col_sum && (!t22 || a.splits != 1u || a.batch0 * a.batch1 != 1u || a.b.s_col != 1 || a.col_post.n_slots > 16u)) return hipErrorInvalidValue;
  if (wgs == 0u) return hipSuccess;
  auto aligned = [&](const GemmOperand& o, int64_t s_outer) {
    return (((uintptr_t)o.ptr) & 15u) == 0u && (s_outer % 4) == 0 && (o.s_b0 % 4) == 0 && (o.s_b1 % 4) == 0;
  };
  const bool av = a.a.s_col == 1 && (a.k % 4u) == 0u && aligned(a.a, a.a.s_row), bv = a.b.s_row == 1 && (a.k % 4u) == 0u && aligned(a.b, a.b.s_col);
  const dim3 grid(a.tiles_n * a.splits, a.tiles_m, a.batch0 * a.batch1);
  // Two groups of k in flight or four, in tiles of 32 x 32.  Four where B's rows are read along k, 16 bytes a lane, so that a chunk is
  // a whole cache line of each; and in unshared products with both operands read across k, where a wave's share fills chunks of four
  // as well as chunks of two (nothing is fetched past it).  us, two / four: B transposed, whole vectors, 32 x 2048 x 2048 11.6 / 11.0, 8 x 4096 x
  // 4096 24.3 / 23.1, 32 x 4096 x 4096 27.5 / 26.3; across, with an input of the output's size, 512: 256 x 100 8.4 / 8.0, 200: 512 x 512 7.0 / 6.5, but 128: 784 x 512 7.2 / 8.7,
  // 300: 512 x 512 7.0 / 8.3, shared 8000: 30 x 30 12.8 / 13.2; k of no whole vectors, single values, 32 x 2047 x 1000 11.1 / 12.6, B transposed
  // 12.5 / 15.3.
  const uint32_t per = ((a.k + 7u) / 8u + (uint32_t)kSmallWaves - 1u) / (uint32_t)kSmallWaves;   // (groups of a wave, unshared)
  const bool four = a.splits == 1u && a.a.s_col != 1 && a.b.s_row != 1 && (per + 3u) / 4u * 2u == (per + 1u) / 2u;
  if (t22 && a.col_sum) launch_small_tile<2, 2, true>(a, av, bv, false, grid, kSmallThreads, s);
  else if (t22) launch_small_tile<2, 2, false>(a, av, bv, four, grid, kSmallThreads, s);
  else if (t42) launch_small_tile<4, 2, false>(a, av, bv, true, grid, kSmallThreads, s);
  else {
    // a wave per group of 16 k that a workgroup has to do: at most eight, and the four that a tile of 64
    // columns needs for its epilogue
    const uint32_t groups = ((a.k + 15u) / 16u + a.splits - 1u) / a.splits;
    const uint32_t waves = std::max(std::min(groups, (uint32_t)kSmallWaves), t14 ? 4u : 1u);
    if (t14) {
      if (a.b.s_col != 1 || a.n < 4u || a.n % 4u != 0u) return hipErrorInvalidValue;   // (four columns at a time)
      launch_small_tile<1, 4, false>(a, av, false, true, grid, 64u * waves, s);
    } else {
      launch_small_tile<1, 1, false>(a, av, bv, true, grid, 64u * waves, s);
    }
  }
  return hipGetLastError();
}

template <typename T, int BM, int BN, bool AL, int KS>
static void launch_variant(const GemmArgs& a, const dim3 grid, hipStream_t s) {
  const dim3 block(kGemmThreads * KS);
  const bool akc = a.a.s_col == 1, bkc = a.b.s_row == 1;
  char name[64];
  if (a.col_sum) {
    LT_LAUNCH((lt_gemm_kernel<T, BM, BN, false, false, AL, KS, true>), grid, block, s, a);
    snprintf(name, sizeof(name), "lt_gemm_kernel<float,%d,%d,sums,%s,%d>", BM, BN, AL ? "true" : "false", KS);
    note_kernel(name);
    return;
  }
  if (akc && bkc) LT_LAUNCH((lt_gemm_kernel<T, BM, BN, true, true, AL, KS, false>), grid, block, s, a);
  else if (akc) LT_LAUNCH((lt_gemm_kernel<T, BM, BN, true, false, AL, KS, false>), grid, block, s, a);
  else if (bkc) LT_LAUNCH((lt_gemm_kernel<T, BM, BN, false, true, AL, KS, false>), grid, block, s, a);
  else LT_LAUNCH((lt_gemm_kernel<T, BM, BN, false, false, AL, KS, false>), grid, block, s, a);
  snprintf(name, sizeof(name), "lt_gemm_kernel<float,%d,%d,%s,%s,%s,%d>", BM, BN, akc ? "true" : "false", bkc ? "true" : "false", AL ? "true" : "false", KS);
  note_kernel(name);
}

hipError_t launch_gemm(const GemmArgs& a, hipStream_t s) {
  // an operand must have unit stride along one of its two dimensions
  if ((a.a.s_col != 1 && a.a.s_row != 1) || (a.b.s_col != 1 && a.b.s_row != 1)) return hipErrorInvalidValue;
  if (a.in_dtype == kBF16) return launch_gemm_bf16(a, s);
  const uint32_t batch = a.batch0 * a.batch1;
  if (a.direct) return launch_small(a, s);
  if (a.tile_m != a.tile_n || (a.tile_m != 64u && a.tile_m != 128u)) return hipErrorInvalidValue;
  if (a.col_sum && !columns_ride(a, batch)) return hipErrorInvalidValue;
  const bool big = a.tile_m == 128u;   // the host picks big tiles only when they still give every compute unit work
  const uint32_t bm = a.tile_m;
  if (a.halves != 1u && (a.halves != 2u || big)) return hipErrorInvalidValue;
  if (a.splits == 0u || (a.splits > 1u && !a.split_ws)) return hipErrorInvalidValue;
  const dim3 grid((a.n + bm - 1) / bm, (a.m + bm - 1) / bm, batch * a.splits);
  if (grid.y > 65535u || grid.z > 65535u) return hipErrorInvalidValue;
  // (a lane's offset into a panel is a 32-bit number of bytes: 128 rows of less than 2^23 elements)
  auto aligned = [](const GemmOperand& o, int64_t outer) {
    return ((uintptr_t)o.ptr & 15u) == 0 && outer % 4 == 0 && outer < (1 << 23) && o.s_b0 % 4 == 0 && o.s_b1 % 4 == 0;
  };
  const bool al = aligned(a.a, a.a.s_col == 1 ? a.a.s_row : a.a.s_col) && aligned(a.b, a.b.s_row == 1 ? a.b.s_col : a.b.s_row);
  if (big && al) launch_variant<float, 128, 128, true, 1>(a, grid, s);
  else if (big) launch_variant<float, 128, 128, false, 1>(a, grid, s);
  else if (al && a.halves == 2u) launch_variant<float, 64, 64, true, 2>(a, grid, s);
  else if (al) launch_variant<float, 64, 64, true, 1>(a, grid, s);
  else if (a.halves == 2u) launch_variant<float, 64, 64, false, 2>(a, grid, s);
  else launch_variant<float, 64, 64, false, 1>(a, grid, s);
  return hipGetLastError();
}

}  // namespace ltk

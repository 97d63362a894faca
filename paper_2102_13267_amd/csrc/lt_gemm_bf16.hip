// bf16 contraction on the gfx950 matrix cores: C = post(A * B), fp32 accumulation.
//
// Workgroup tile 128 x 128 (128 x 64 for narrow outputs), k walked in slices of 32, four
// wavefronts in a 2 x 2 arrangement, each owning 64 x 64 (64 x 32) as blocks of
// v_mfma_f32_32x32x16_bf16.  What bounds this kernel is the way into the matrix cores, not the
// matrix cores: per slice a workgroup brings 16 KiB through the L1 (64 bytes per cycle and compute
// unit: 256 cycles) and reads 32 KiB of fragments from LDS for 32 MFMAs (256 cycles per SIMD) --
// at the matrix cores' peak a 128 x 128 tile needs all of the L1's bandwidth.  Two workgroups
// share a compute unit, so one's matrix instructions run under the other's copies, LDS traffic,
// barriers and epilogue.
//
// Whole, 16-byte aligned tiles go from global memory into LDS without touching registers
// (global_load_lds_dwordx4), into dense tiles whose bank conflicts a swizzle takes care of; four
// stages, copies two to three slices ahead, in pairs of slices when an operand's rows are half
// cache lines (see "whole tiles" below).  An MFMA lane wants 8 consecutive k of one row (A) or
// column (B):
//  * k is the operand's contiguous dimension: the tile is [x][k] and a fragment is one
//    ds_read_b128;
//  * x (m or n) is the contiguous dimension: the tile stays as it arrives, [k][x], and the
//    transpose happens in the LDS read: ds_read_b64_tr_b16 hands each lane of a 16-lane group one
//    column of a 4 x 16 sub-tile (lane i gets element i of each of the four rows that lanes
//    4j .. 4j+3 point at), so two such reads give the 8 k values of one x.
// Nothing is transposed by scalar code.  A tile that hangs over the edge of its operand takes the same
// path (rows and chunks past the edge are copies of the last one, never stored); what is left of k
// behind the last whole slice is fetched element by element, one slice.  Rows that are not 16-byte
// aligned (odd lengths) go through registers into padded LDS tiles, 16 bytes at a time, one slice
// ahead.  128 heads of 200 x 64: q k^T 10.7 us, p v 10.3 us (with every access checked element by element: 14.4
// and 14.9).
//
// Epilogue (lt_gemm_epilogue.h): the accumulators leave the MFMA layout through LDS, the whole tile
// at once, and are then walked in row-major 4-element quads by the interpreter (bias, activation,
// residual, optimiser update, cast ...), so the product itself never travels to HBM unless
// asked for.
//
// Split-K: when a problem has few output tiles but a long k, `splits` workgroups share a tile and
// each leaves its fp32 partial product in a workspace; a second, elementwise launch adds them in
// split order and runs the post program at full occupancy (an interpreted epilogue run by one
// workgroup per tile would leave most of the chip idle).
//
// Tile order: workgroups are handed to the eight XCDs round robin, so consecutive workgroup
// numbers are remapped to make each XCD's share a contiguous block of tiles (one set of A and B
// panels per L2).
#include <hip/hip_runtime.h>

#include <cstdio>

#include "lt_dma.h"
#include "lt_gemm_epilogue.h"
#include "lt_launch.h"

namespace ltk {

namespace bf {
constexpr int BK = 32;
constexpr int kStrideKC = 80;    // bytes per row of an [x][k] tile: 64 + 16 of padding

typedef short v4s __attribute__((ext_vector_type(4)));
typedef short v8s __attribute__((ext_vector_type(8)));
typedef __attribute__((address_space(3))) v4s* lds_v4s_ptr;

// Geometry of one padded operand tile of BX rows/columns by 32 k (ragged-tile path).
template <int BX> struct Geo {
  static constexpr int kChunks = BX / 64;              // 16-byte chunks per lane and slice
  static constexpr int kStrideXC = BX * 2 + 32;        // bytes per row of a [k][x] tile
  static constexpr int kBytes = BX * kStrideKC;        // >= 32 * kStrideXC
};

template <uint32_t N> struct Num {
  static constexpr uint32_t value = N;
};

template <int N> struct Chunks {
  uint4 g[N];
};

// (outer, inner) coordinates inside the tile of this lane's chunk number `it`.  KC: rows are x,
// 4 chunks of 8 k each; otherwise rows are k, BX/8 chunks of 8 x each.
template <int BX, bool KC>
__device__ __forceinline__ void chunk_pos(uint32_t it, uint32_t* outer, uint32_t* inner) {
  const uint32_t e = it * kGemmThreads + threadIdx.x % kGemmThreads;
  if (KC) {
    *outer = e >> 2;
    *inner = (e & 3u) * 8u;
  } else {
    *outer = e / (BX / 8);
    *inner = (e % (BX / 8)) * 8u;
  }
}

// Global -> registers for a slice that may run over the end of k (or touch the operand's last row, see
// the kernel): element by element at addresses clamped into the operand, branch-free so that all of
// a lane's loads are in flight together.  k past the end reads as zero; rows or columns past the
// edge are copies of the last one and are never stored.
template <int BX, bool KC>
__device__ __forceinline__ Chunks<Geo<BX>::kChunks> fetch_checked(const uint16_t* base, int64_t s_x, int64_t s_k, uint32_t x0,
                                                                  uint32_t k0, uint32_t nx, uint32_t nk) {
  Chunks<Geo<BX>::kChunks> c;
#pragma unroll
  for (int it = 0; it < Geo<BX>::kChunks; ++it) {
    uint32_t o, i;
    chunk_pos<BX, KC>(it, &o, &i);
    uint32_t e[8];
#pragma unroll
    for (uint32_t j = 0; j < 8u; ++j) {
      const uint32_t x = KC ? x0 + o : x0 + i + j, k = KC ? k0 + i + j : k0 + o;
      e[j] = (uint32_t)base[(int64_t)min(x, nx - 1u) * s_x + (int64_t)min(k, nk - 1u) * s_k];
    }
#pragma unroll
    for (uint32_t j = 0; j < 8u; ++j)
      if ((KC ? k0 + i + j : k0 + o) >= nk) e[j] = 0u;
    c.g[it] = make_uint4(e[0] | e[1] << 16, e[2] | e[3] << 16, e[4] | e[5] << 16, e[6] | e[7] << 16);
  }
  return c;
}

// This lane's element offset of its chunk at (outer, inner) from the (wave-uniform) start of the panel at x0, k0 = 0: the
// same for every slice.  Rows (KC) or chunks of eight columns past the operand's edge become copies
// of the last one.
template <int BX, bool KC>
__device__ __forceinline__ int64_t chunk_offset(uint32_t outer, uint32_t inner, int64_t s_x, int64_t s_k, uint32_t left) {
  return KC ? (int64_t)min(outer, left - 1u) * s_x + inner : (int64_t)outer * s_k + min(inner, (left - 1u) & ~7u);
}

// Global -> registers for a whole slice of an operand whose rows start at any element: 16-byte
// loads at 2-byte boundaries (the hardware takes them; half the rate of aligned ones at worst).
typedef uint32_t U32x4u __attribute__((ext_vector_type(4), aligned(2)));
template <int BX, bool KC>
__device__ __forceinline__ Chunks<Geo<BX>::kChunks> fetch_unaligned(const uint16_t* panel, const int64_t (&off)[Geo<BX>::kChunks]) {
  Chunks<Geo<BX>::kChunks> c;
#pragma unroll
  for (int it = 0; it < Geo<BX>::kChunks; ++it) {
    const U32x4u v = *(const U32x4u*)(panel + off[it]);
    c.g[it] = make_uint4(v.x, v.y, v.z, v.w);
  }
  return c;
}

template <int BX, bool KC>
__device__ __forceinline__ void stash(const Chunks<Geo<BX>::kChunks>& c, char* tile) {
#pragma unroll
  for (int it = 0; it < Geo<BX>::kChunks; ++it) {
    uint32_t o, i;
    chunk_pos<BX, KC>(it, &o, &i);
    *(uint4*)(tile + o * (KC ? kStrideKC : Geo<BX>::kStrideXC) + i * 2u) = c.g[it];
  }
}

// The MFMA fragment of a 32-row (or 32-column) block starting at x_blk for k16 step kk.
template <int BX, bool KC>
__device__ __forceinline__ v8bf fragment(const char* tile, uint32_t x_blk, uint32_t kk, uint32_t lane) {
  const uint32_t kb = kk * 16u + (lane >> 5) * 8u;   // first of this lane's 8 k
  if (KC) {
    return *(const v8bf*)(tile + (x_blk + (lane & 31u)) * kStrideKC + kb * 2u);
  } else {
    constexpr int S = Geo<BX>::kStrideXC;
    const uint32_t i16 = lane & 15u;
    const uint32_t xb = x_blk + ((lane & 31u) >> 4) * 16u;
    const char* p = tile + (kb + (i16 >> 2)) * S + (xb + 4u * (i16 & 3u)) * 2u;
    const v4s lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_v4s_ptr)p);
    const v4s hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_v4s_ptr)(p + 4 * S));
    v8s r;
    r[0] = lo[0]; r[1] = lo[1]; r[2] = lo[2]; r[3] = lo[3];
    r[4] = hi[0]; r[5] = hi[1]; r[6] = hi[2]; r[7] = hi[3];
    return __builtin_bit_cast(v8bf, r);
  }
}

// ---- whole tiles: global memory -> LDS without passing through registers -----------------------
// `global_load_lds_dwordx4`: every lane names its own 16 global bytes, the hardware writes them to
// LDS at a wave-uniform base + lane * 16 (checked with an in-bounds probe), so a wave instruction
// fills 1 KiB of consecutive LDS.  Tiles are therefore dense (no row padding), and bank conflicts
// of the fragment reads are avoided by a swizzle instead: the 16-byte chunk at (row, c) lives at
// position c ^ f(row) of its row.  The swizzle costs nothing in the loop: it is folded into each
// lane's global offset (which chunk it fetches for its LDS slot) and into the fragment addresses.
//   [x][k] tile (k contiguous in memory): rows of 64 bytes, f(x) = (x >> 2) & 3 -- the sixteen rows
//     that one cycle of a ds_read_b128 touches then cover all sixteen 16-byte bank groups;
//   [k][x] tile (x contiguous): rows of BX * 2 bytes, f(k) = (k & 3) << 2 for 256-byte rows
//     (((k >> 1) & 1) << 2 for 128-byte rows): the four k rows of a transposing read land in four
//     different 64-byte bank ranges.
template <int BX, bool KC> struct Dense {
  static constexpr uint32_t kBytes = BX * 64;            // BX x 32 bf16
  static constexpr uint32_t kInstr = BX / 64;            // wave instructions per slice (4 waves x 1 KiB each)
  static constexpr uint32_t kPerRow = BX / 8;            // chunks per k row of a [k][x] tile
  static constexpr uint32_t kRowsPer256 = 256 / (BX * 2) ? 256 / (BX * 2) : 1;   // [k][x] rows per 256 bytes
  __device__ static __forceinline__ uint32_t swz_k(uint32_t k) { return ((k / kRowsPer256) & (4u / kRowsPer256 - 1u)) << 2; }
  __device__ static __forceinline__ uint32_t swz_x(uint32_t x) { return (x >> 2) & 3u; }
};

// This lane's byte offset, for wave instruction `it` of a slice, from the (wave-uniform) start of the
// panel at x0: the same for every slice.  `left`: rows or columns from x0 to the operand's edge.
template <int BX, bool KC>
__device__ __forceinline__ uint32_t dma_lane_offset(uint32_t it, int64_t s_x, int64_t s_k, uint32_t left) {
  typedef Dense<BX, KC> D;
  const uint32_t t = threadIdx.x % kGemmThreads;
  if (KC) {
    const uint32_t row = it * 64u + (t >> 2), c = (t & 3u) ^ D::swz_x(row);
    return (uint32_t)(2 * chunk_offset<BX, KC>(row, c * 8u, s_x, s_k, left));
  }
  const uint32_t k = t / D::kPerRow, xc = (t % D::kPerRow) ^ D::swz_k(k);
  return (uint32_t)(2 * chunk_offset<BX, KC>(it * ((uint32_t)kGemmThreads / D::kPerRow) + k, xc * 8u, s_x, s_k, left));
}

// Start the copy of a slice (`src`: the panel's start at the slice's first k) into the tile at LDS
// address `tile`.
template <int BX, bool KC>
__device__ __forceinline__ void dma_tile(const uint16_t* src, const uint32_t (&off)[Dense<BX, KC>::kInstr], uint32_t tile, uint32_t wave) {
#pragma unroll
  for (uint32_t it = 0; it < Dense<BX, KC>::kInstr; ++it)
    copy_1k(src, off[it], tile + (it * (uint32_t)kGemmThreads + wave * 64u) * 16u);
}

// Two consecutive slices (ka, kb = ka + 32 unless clamped) at once, instruction by instruction.
// A row of an [x][k] slice is 64 bytes, half a cache line; fetched one slice per iteration, the
// second half comes a whole iteration's traffic later, misses the L1 again and costs a second
// request to L2 (measured: 1.8 times the L2 requests, the address unit stalled by the cache for
// 40 % of the kernel).  Back to back, the second access finds the line already on its way.
template <int BX, bool KC>
__device__ __forceinline__ void dma_tile2(const uint16_t* src_a, const uint16_t* src_b, const uint32_t (&off)[Dense<BX, KC>::kInstr],
                                          uint32_t tile_a, uint32_t tile_b, uint32_t wave) {
#pragma unroll
  for (uint32_t it = 0; it < Dense<BX, KC>::kInstr; ++it) {
    const uint32_t dst = (it * (uint32_t)kGemmThreads + wave * 64u) * 16u;
    copy_1k(src_a, off[it], tile_a + dst);
    copy_1k(src_b, off[it], tile_b + dst);
  }
}

// The MFMA fragment of a 32-row (or 32-column) block of a dense, swizzled tile.
template <int BX, bool KC>
__device__ __forceinline__ v8bf fragment_dense(const char* tile, uint32_t x_blk, uint32_t kk, uint32_t lane) {
  typedef Dense<BX, KC> D;
  if (KC) {
    const uint32_t row = x_blk + (lane & 31u), c = kk * 2u + (lane >> 5);
    return *(const v8bf*)(tile + row * 64u + ((c ^ D::swz_x(row)) << 4));
  } else {
    constexpr uint32_t S = BX * 2;
    const uint32_t i16 = lane & 15u;
    const uint32_t k = kk * 16u + (lane >> 5) * 8u + (i16 >> 2);
    const uint32_t col = (x_blk + ((lane & 31u) >> 4) * 16u + 4u * (i16 & 3u)) * 2u;   // byte column
    const char* p = tile + k * S + (((col >> 4) ^ D::swz_k(k)) << 4) + (col & 15u);
    const v4s lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_v4s_ptr)p);
    const v4s hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_v4s_ptr)(p + 4 * S));   // k + 4: same swizzle
    v8s r;
    r[0] = lo[0]; r[1] = lo[1]; r[2] = lo[2]; r[3] = lo[3];
    r[4] = hi[0]; r[5] = hi[1]; r[6] = hi[2]; r[7] = hi[3];
    return __builtin_bit_cast(v8bf, r);
  }
}

// ---- slabs: whole tiles of a workgroup in halves ----------------------------------------------------
// The halves of a workgroup walk its k together, slabs of 64 that all eight waves copy: the first half multiplies
// the first 32 k of each, the other one the rest.  A row of an [x][k] slab is then a whole cache line, four slabs fit in LDS and
// copies go out three slabs ahead.  (With stages of their own, contiguous shares of k and pairs of half lines, two slices
// ahead, the halves waited: 4096 x 1024 x 4096 with k contiguous kept the matrix cores 48 % busy; its loop 35 -> 28.7 us, the
// launch 45.4 -> 39.8.  With both operands across k, whose stages were four slices deep already, nothing changes: 28.7.)
//   [x][k] slab: rows of 128 bytes, chunk c of row x at position c ^ ((x >> 1) & 7);  [k][x] slab: as above, 64 rows.
template <int BX, bool KC> struct Slab {
  static constexpr uint32_t kBytes = BX * 128, kInstr = BX / 64, kPerRow = KC ? 8 : BX / 8;   // (wave instructions: 8 waves x 1 KiB each)
  __device__ static __forceinline__ uint32_t swz(uint32_t row) { return KC ? (row >> 1) & 7u : Dense<BX, false>::swz_k(row); }
  // byte offset of this lane's chunk for wave instruction `it`; *second: how far to go back if it lies in the second half of k
  // and the slab has only the first
  __device__ static __forceinline__ uint32_t lane_offset(uint32_t it, int64_t s_x, int64_t s_k, uint32_t left, uint32_t* second) {
    const uint32_t e = it * 2u * (uint32_t)kGemmThreads + threadIdx.x, row = e / kPerRow, c = (e % kPerRow) ^ swz(row);
    *second = KC ? (c >= 4u ? 64u : 0u) : (row >= 32u ? (uint32_t)(64 * s_k) : 0u);
    return (uint32_t)(2 * chunk_offset<BX, KC>(row, c * 8u, s_x, s_k, left));
  }
  // the fragment of a 32-row (or 32-column) block, k16 step kk of the given half
  __device__ static __forceinline__ v8bf fragment(const char* slab, uint32_t half, uint32_t x_blk, uint32_t kk, uint32_t lane) {
    if (KC) {
      const uint32_t row = x_blk + (lane & 31u), c = half * 4u + kk * 2u + (lane >> 5);
      return *(const v8bf*)(slab + row * 128u + ((c ^ swz(row)) << 4));
    }
    return fragment_dense<BX, false>(slab + half * (BX * 64u), x_blk, kk, lane);   // (32 rows on: the same swizzle)
  }
};

template <int BM, int BN> struct Smem {
  static constexpr size_t kStage = Geo<BM>::kBytes + Geo<BN>::kBytes;
  static constexpr size_t kStripBytes = (size_t)BM * (BN + kCPad) * sizeof(float);   // the whole tile
  static constexpr size_t kDense = 4 * (size_t)(BM + BN) * 64;                        // four dense stages
  static constexpr size_t kMax2 = 2 * kStage > kStripBytes ? 2 * kStage : kStripBytes;   // (unaligned rows: two padded stages)
  static constexpr size_t kBytes = kMax2 > kDense ? kMax2 : kDense;
};

// AL: both operands' rows are 16-byte aligned (the launcher looks).  Two instances, because the path
// that the other one takes costs registers in the main loop.
// KS: halves of the workgroup that share its k (GemmArgs::halves): slabs, above; unaligned rows: each has LDS stages
// and a contiguous share of its own.
// CS: column sums of B ride along (GemmArgs::col_sum; AKC and BKC false).  The workgroups of the first tile row take them
// from the B fragments that they multiply anyway: each of a wave row's two k16 steps of a slice by one of the two
// wave rows, a dot product with ones per register, eight next to a wave's eight MFMAs.  A slice's sum starts afresh and joins
// a running sum, one of two (unaligned rows: one), and these join a total every 128 (64) slices.  65536 columns of N(1, 1), unsplit,
// root mean square error: 0.41e-7 (unaligned 0.40e-7), without a total 0.88e-7 (2.1e-7), in a launch of their own 0.50e-7; 4096 x 1024 x 4096
// 42.3 us as without (joined every 32 slices 43.1: the loop is one of straight-line code).
template <int BM, int BN, bool AKC, bool BKC, bool AL, int KS, bool CS>
__global__ __launch_bounds__(kGemmThreads * KS, 2) void lt_gemm_bf16_kernel(const GemmArgs a) {
  static_assert(!CS || (!AKC && !BKC && BM == 128), "a weight gradient");
  constexpr int MB = BM / 64, NB = BN / 64;   // 32 x 32 blocks per wave: rows, columns
  constexpr size_t kHalf = Smem<BM, BN>::kBytes;
  __shared__ __attribute__((aligned(16))) char smem_all[KS * kHalf];
  __shared__ __attribute__((aligned(16))) float col_lds[CS ? KS * 2 * BN : 4];   // [half][wave row][column]
  const uint32_t touched = touch_args<GemmArgs>();   // (0.4 to 1 us of a launch of 7 to 20)
  const uint32_t half = KS > 1 ? __builtin_amdgcn_readfirstlane(threadIdx.x / kGemmThreads) : 0u;
  char* const smem = smem_all + half * kHalf;
  const uint32_t tid = threadIdx.x % kGemmThreads, lane = tid & 63u, wave = tid >> 6;
  const uint32_t wave_m = wave >> 1, wave_n = wave & 1u;
  // tile number: remap so that each XCD (workgroup number mod 8) owns a contiguous range
  const uint32_t nt = gridDim.x;
  uint32_t t = blockIdx.x;
  if ((nt & 7u) == 0u) t = (blockIdx.x & 7u) * (nt >> 3) + (blockIdx.x >> 3);
  // and, where they number 256 or more, walks it eight rows of tiles at a time, column by column: the 64 tiles that
  // an XCD works on at a time then share eight panels of A and eight of B (row by row, 32 columns: two and 32).
  // 8192 x 4096 x 1024 with bias, GELU and both results 117 -> 103.5 us, 1024 x 4096 from 4096 rows 58.7 -> 50; fewer
  // tiles run at once anyway and lose (300 x 4096 x 1024: 22.9 -> 25.9).
  uint32_t row = t / a.tiles_n, col = t - row * a.tiles_n;
  if (nt >= 256u) {
    const uint32_t strip = row / 8u, rows = min(8u, a.tiles_m - strip * 8u), in_strip = t - strip * (8u * a.tiles_n);
    col = in_strip / rows;
    row = strip * 8u + in_strip - col * rows;
  }
  const uint32_t tile_m = row * BM, tile_n = col * BN;
  const uint32_t batch = blockIdx.y / a.splits, split = blockIdx.y % a.splits;
  const uint32_t b0 = batch / a.batch1, b1 = batch % a.batch1;
  const uint16_t* A = (const uint16_t*)a.a.ptr + (int64_t)b0 * a.a.s_b0 + (int64_t)b1 * a.a.s_b1;
  const uint16_t* B = (const uint16_t*)a.b.ptr + (int64_t)b0 * a.b.s_b0 + (int64_t)b1 * a.b.s_b1;
  // this workgroup's share of k: whole slices, split evenly
  const uint32_t slices = (a.k + BK - 1) / BK;
  const uint32_t per = (slices + a.splits - 1) / a.splits;
  const uint32_t k_begin = min(a.k, split * per * BK), k_end = min(a.k, (split + 1) * per * BK);
  const int64_t a_outer = AKC ? a.a.s_row : a.a.s_col, b_outer = BKC ? a.b.s_col : a.b.s_row;

  constexpr uint32_t kStage = (uint32_t)Smem<BM, BN>::kStage;   // padded layout (ragged tiles): A tile then B tile
  v16f acc[MB][NB];
#pragma unroll
  for (int i = 0; i < MB; ++i)
#pragma unroll
    for (int j = 0; j < NB; ++j)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.0f;

  // fragments of one slice: every MFMA operand of this wave, both k16 steps
  struct Frags {
    v8bf a[BK / 16][MB], b[BK / 16][NB];
  };
  auto load_frags = [&](uint32_t stage) {
    const char* As = smem + stage * kStage;
    const char* Bs = As + Geo<BM>::kBytes;
    Frags f;
#pragma unroll
    for (uint32_t kk = 0; kk < BK / 16; ++kk) {
#pragma unroll
      for (int i = 0; i < MB; ++i) f.a[kk][i] = fragment<BM, AKC>(As, wave_m * (BM / 2) + i * 32u, kk, lane);
#pragma unroll
      for (int j = 0; j < NB; ++j) f.b[kk][j] = fragment<BN, BKC>(Bs, wave_n * (BN / 2) + j * 32u, kk, lane);
    }
    return f;
  };
  auto mma = [&](const Frags& f) {
#pragma unroll
    for (uint32_t kk = 0; kk < BK / 16; ++kk)
#pragma unroll
      for (int i = 0; i < MB; ++i)
#pragma unroll
        for (int j = 0; j < NB; ++j) acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(f.a[kk][i], f.b[kk][j], acc[i][j], 0, 0, 0);
  };
  const bool summing = CS && tile_m == 0u;
  float csum[2][NB];
  ColTotal ctot[NB];
#pragma unroll
  for (int j = 0; j < NB; ++j) csum[0][j] = csum[1][j] = 0.0f;
  auto join_columns = [&]() __attribute__((always_inline)) {
#pragma unroll
    for (int j = 0; j < NB; ++j) {
      ctot[j].add(AL ? csum[0][j] + csum[1][j] : csum[0][j]);   // (unaligned rows: one set)
      csum[0][j] = csum[1][j] = 0.0f;
    }
  };
  // the sums of the B fragments of k16 step kk
  auto add_columns = [&](const Frags& f, int kk, int set) {
    typedef __bf16 V2 __attribute__((ext_vector_type(2)));
    const V2 ones = {(__bf16)1.0f, (__bf16)1.0f};
#pragma unroll
    for (int j = 0; j < NB; ++j) {
      float t = 0.0f;
#pragma unroll
      for (int q = 0; q < 4; ++q) t = __builtin_amdgcn_fdot2_f32_bf16(V2{f.b[kk][j][2 * q], f.b[kk][j][2 * q + 1]}, ones, t, false);
      csum[set][j] += t;
    }
  };
  auto mma_and_sum = [&](const Frags& f) {
    mma(f);
    if (summing) {
      if (wave_m == 0u) add_columns(f, 0, 0);
      else add_columns(f, 1, 0);
    }
  };
  // Whole slices of k are fetched in 16-byte chunks with no checks; what is left of k goes through
  // fetch_checked as one last slice.  A tile that hangs over the operand's edge is filled with copies
  // of the last row (k contiguous), or of the last chunk of eight columns.  That chunk may reach up
  // to seven elements past its row, into the next one (in bounds if rows are at least that far
  // apart): then the slice with the operand's last row has to be the checked one.
  const uint32_t left_m = a.m - tile_m, left_n = a.n - tile_n;
  const bool a_over = !AKC && left_m < (uint32_t)BM && (a.m & 7u) != 0u, b_over = !BKC && left_n < (uint32_t)BN && (a.n & 7u) != 0u;
  uint32_t n = (k_end - k_begin) / BK;   // whole slices
  if ((a_over && a_outer < 8) || (b_over && b_outer < 8)) n = 0u;
  else if ((a_over || b_over) && n > 0u && k_begin + n * BK == a.k) --n;
  // The halves walk theirs in the same n steps, between the same barriers.  Of an odd number the first takes one more; the
  // second has nothing to multiply in the last step: as a slice of the rest it took 2 to 4 us (512 x 768 x 700 17.7 -> 13.2, 768 x 768 x
  // 4096 28.6 -> 23.3).  (A single slice is left to the rest.)
  if (KS > 1 && n < 2u) n = 0u;
  const uint32_t both = KS > 1 ? n / 2u : n, k_rest = k_begin + n * BK;   // steps in which every half multiplies
  if (KS > 1) n -= both;
  const uint32_t mine = half == 0u ? n : both, k_first = KS > 1 && AL ? k_begin : k_begin + half * n * BK;   // (AL: in slabs, below)
  const uint16_t* const pa = A + (int64_t)tile_m * a.a.s_row + (int64_t)k_first * a.a.s_col;
  const uint16_t* const pb = B + (int64_t)tile_n * a.b.s_col + (int64_t)k_first * a.b.s_row;
  const int64_t step_a = BK * a.a.s_col, step_b = BK * a.b.s_row;   // elements per slice of k
  if constexpr (AL && KS == 2) {
    if (n > 0u) {
      // Slabs 0 .. n-1, four stages: the MFMAs of slab j run from fragment registers, the fragments of slab j + 1 are read
      // from its stage, later ones are on their way.  Behind the barrier of slab j slab j + 1 has landed for every wave, and every
      // wave's reads of slab j's stage, which is copied into next, have returned.  (Copies past the end: the last slab again, unused.)
      typedef Slab<BM, AKC> SA;
      typedef Slab<BN, BKC> SB;
      constexpr uint32_t kStageBytes = SA::kBytes + SB::kBytes, kPer = SA::kInstr + SB::kInstr;
      static_assert(4 * kStageBytes <= KS * kHalf, "four slabs fit the tile's LDS");
      const uint32_t wave8 = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
      const uint32_t lds0 = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) char*)smem_all;
      const bool odd = both < n;
      uint32_t a_off[SA::kInstr], a_back[SA::kInstr], b_off[SB::kInstr], b_back[SB::kInstr];
#pragma unroll
      for (uint32_t it = 0; it < SA::kInstr; ++it) a_off[it] = SA::lane_offset(it, a.a.s_row, a.a.s_col, left_m, &a_back[it]);
#pragma unroll
      for (uint32_t it = 0; it < SB::kInstr; ++it) b_off[it] = SB::lane_offset(it, a.b.s_col, a.b.s_row, left_n, &b_back[it]);
      auto copy = [&](uint32_t slab, uint32_t stage) __attribute__((always_inline)) {
        const uint32_t sl = min(slab, n - 1u), cut = odd && sl == n - 1u ? ~0u : 0u;   // (the last one may have only its first half)
        const uint16_t* const ca = pa + (int64_t)sl * (2 * step_a);
        const uint16_t* const cb = pb + (int64_t)sl * (2 * step_b);
        const uint32_t at = lds0 + stage * kStageBytes;
#pragma unroll
        for (uint32_t it = 0; it < SA::kInstr; ++it) copy_1k(ca, a_off[it] - (a_back[it] & cut), at + (it * 2u * (uint32_t)kGemmThreads + wave8 * 64u) * 16u);
#pragma unroll
        for (uint32_t it = 0; it < SB::kInstr; ++it)
          copy_1k(cb, b_off[it] - (b_back[it] & cut), at + SA::kBytes + (it * 2u * (uint32_t)kGemmThreads + wave8 * 64u) * 16u);
      };
      auto frags = [&](uint32_t stage) {
        const char* As = smem_all + stage * kStageBytes;
        const char* Bs = As + SA::kBytes;
        Frags f;
#pragma unroll
        for (uint32_t kk = 0; kk < BK / 16; ++kk) {
#pragma unroll
          for (int i = 0; i < MB; ++i) f.a[kk][i] = SA::fragment(As, half, wave_m * (BM / 2) + i * 32u, kk, lane);
#pragma unroll
          for (int j = 0; j < NB; ++j) f.b[kk][j] = SB::fragment(Bs, half, wave_n * (BN / 2) + j * 32u, kk, lane);
        }
        return f;
      };
      copy(0, 0);
      copy(1, 1);
      copy(2, 2);
      copy(3, 3);
      landed<3 * kPer>();
      __syncthreads();
      // (sum: the k16 step, plus one, of which this wave adds up the columns; every version has the same barriers)
      auto pipeline = [&](auto sum) __attribute__((always_inline)) {
        constexpr int kSum = (int)decltype(sum)::value;
        Frags f0 = frags(0), f1;
#define LT_SLAB(J, CUR, NEXT, GUARD)                           \
  {                                                            \
    landed_and_read<2 * kPer>();                               \
    __syncthreads();                                           \
    copy(i + (J) + 4u, (J) & 3);                               \
    NEXT = frags(((J) + 1) & 3);                               \
    if (!(GUARD) || i + (J) < mine) {                          \
      mma(CUR);                                                \
      if (kSum > 0) add_columns(CUR, kSum - 1, (J) & 1);       \
    }                                                          \
  }
        uint32_t i = 0;
        while (i + 4u <= both) {
          const uint32_t to = kSum > 0 ? min(i + 128u, both) : both;
          for (; i + 4u <= to; i += 4u) {
            LT_SLAB(0, f0, f1, false);
            LT_SLAB(1, f1, f0, false);
            LT_SLAB(2, f0, f1, false);
            LT_SLAB(3, f1, f0, false);
          }
          if (kSum > 0) join_columns();
        }
        if (i < n) {
          LT_SLAB(0, f0, f1, true);
          LT_SLAB(1, f1, f0, true);
          LT_SLAB(2, f0, f1, true);
          if (i + 3u < n) LT_SLAB(3, f1, f0, true);   // (the first half's odd one)
        }
#undef LT_SLAB
      };
      if (!CS || !summing) pipeline(Num<0>());
      else if (wave_m == 0u) pipeline(Num<1>());
      else pipeline(Num<2>());
      landed<0>();   // nothing may still be on its way into LDS when it is used again
    }
  }
  if (AL && KS == 1 && n > 0u) {
    // Software pipeline over slices j = 0 .. n-1, four LDS stages: the MFMAs of slice j run from
    // fragment registers, the fragments of slice j+1 are read from the stage that holds it, and
    // later slices are on their way from global memory straight into their stages -- no
    // registers, no LDS write instructions, two iterations for a copy to land.  (Copies past the
    // end are clamped to the last slice: in bounds, unused.)
    constexpr uint32_t kDenseStage = Dense<BM, AKC>::kBytes + Dense<BN, BKC>::kBytes;
    constexpr uint32_t kPer = Dense<BM, AKC>::kInstr + Dense<BN, BKC>::kInstr;   // copy instructions per wave and slice
    static_assert(4 * kDenseStage <= Smem<BM, BN>::kBytes, "four dense stages fit the tile's LDS");
    const uint32_t wave_u = __builtin_amdgcn_readfirstlane(wave);
    const uint32_t lds0 = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) char*)smem;
    uint32_t a_off[Dense<BM, AKC>::kInstr], b_off[Dense<BN, BKC>::kInstr];
#pragma unroll
    for (uint32_t it = 0; it < Dense<BM, AKC>::kInstr; ++it) a_off[it] = dma_lane_offset<BM, AKC>(it, a.a.s_row, a.a.s_col, left_m);
#pragma unroll
    for (uint32_t it = 0; it < Dense<BN, BKC>::kInstr; ++it) b_off[it] = dma_lane_offset<BN, BKC>(it, a.b.s_col, a.b.s_row, left_n);
#define LT_COPY(I, STAGE)                                                                                  \
  {                                                                                                       \
    const int64_t sl = min((uint32_t)(I), mine - 1u);                                                     \
    dma_tile<BM, AKC>(pa + sl * step_a, a_off, lds0 + (STAGE) * kDenseStage, wave_u);                     \
    dma_tile<BN, BKC>(pb + sl * step_b, b_off, lds0 + (STAGE) * kDenseStage + Dense<BM, AKC>::kBytes, wave_u); \
  }
#define LT_COPY2(I0, S0, I1, S1)                                                                           \
  {                                                                                                       \
    const int64_t sa = min((uint32_t)(I0), mine - 1u), sb = min((uint32_t)(I1), mine - 1u);               \
    dma_tile2<BM, AKC>(pa + sa * step_a, pa + sb * step_a, a_off, lds0 + (S0) * kDenseStage, lds0 + (S1) * kDenseStage, wave_u); \
    dma_tile2<BN, BKC>(pb + sa * step_b, pb + sb * step_b, b_off, lds0 + (S0) * kDenseStage + Dense<BM, AKC>::kBytes, \
                       lds0 + (S1) * kDenseStage + Dense<BM, AKC>::kBytes, wave_u);                       \
  }
    auto dense_frags = [&](uint32_t stage) {
      const char* As = smem + stage * kDenseStage;
      const char* Bs = As + Dense<BM, AKC>::kBytes;
      Frags f;
#pragma unroll
      for (uint32_t kk = 0; kk < BK / 16; ++kk) {
#pragma unroll
        for (int i = 0; i < MB; ++i) f.a[kk][i] = fragment_dense<BM, AKC>(As, wave_m * (BM / 2) + i * 32u, kk, lane);
#pragma unroll
        for (int j = 0; j < NB; ++j) f.b[kk][j] = fragment_dense<BN, BKC>(Bs, wave_n * (BN / 2) + j * 32u, kk, lane);
      }
      return f;
    };
    if (n <= 3u) {
      // a short k (attention scores and contexts: k = 64) fits the stages at once: every slice is
      // copied, one wait, one barrier, and the slices are multiplied straight from LDS
      LT_COPY(0, 0);
      if (n > 1u) LT_COPY(1, 1);
      if (n > 2u) LT_COPY(2, 2);
      landed<0>();
      __syncthreads();
      for (uint32_t j = 0; j < mine; ++j) {
        const Frags f = j == 0u ? dense_frags(0) : j == 1u ? dense_frags(1) : dense_frags(2);
        mma_and_sum(f);
      }
    } else {
    // Four slices per trip: stage numbers and the two fragment sets are compile-time.
    //  * Some operand has k contiguous (64-byte rows per slice): copies go out in pairs, at odd
    //    slices: slices i+J+3 and i+J+4 into the stages of slices i+J-1 (long read) and i+J (read
    //    one iteration ago).  Waits and barriers are then needed at odd slices only: behind the
    //    barrier of slice j (odd) the pair copied two slices earlier -- slices j+1 and j+2, whose
    //    fragments are read in this iteration and the next -- has landed for every wave, and every
    //    wave's reads of the two stages about to be overwritten have returned (each wave waits for
    //    its own LDS reads before the barrier).
    //  * Otherwise (rows of a slice are whole cache lines) pairs gain nothing and their bursts cost
    //    a few percent: one copy per slice, slice i+J+4 into the stage of slice i+J behind the
    //    barrier of slice i+J, which also tells that slice i+J+1 has landed for every wave.
    // Past the end the body copies into stages nobody reads and reads fragments nobody uses; only
    // the MFMAs are guarded.
    constexpr bool kPairs = AKC || BKC;
    if (kPairs) {
      LT_COPY2(0, 0, 1, 1);
      LT_COPY2(2, 2, 3, 3);
      landed<2 * kPer>();   // slices 0 and 1
    } else {
      LT_COPY(0, 0);
      LT_COPY(1, 1);
      LT_COPY(2, 2);
      LT_COPY(3, 3);
      landed<3 * kPer>();   // slice 0
    }
    __syncthreads();
    // (SUM: the k16 step, plus one, of which this wave adds up the columns; every version has the same barriers)
    auto pipeline = [&](auto sum) __attribute__((always_inline)) {
    constexpr int kSum = (int)decltype(sum)::value;
    Frags f0 = dense_frags(0), f1;
#define LT_SLICE(J, CUR, NEXT, GUARD)                                            \
  {                                                                            \
    if (kPairs) {                                                              \
      if ((J) & 1) {                                                           \
        landed_and_read<0>();                                                  \
        __syncthreads();                                                       \
        LT_COPY2(i + (J) + 3u, ((J) + 3) & 3, i + (J) + 4u, (J) & 3);          \
      }                                                                        \
    } else {                                                                   \
      landed_and_read<2 * kPer>();                                             \
      __syncthreads();                                                         \
      LT_COPY(i + (J) + 4u, (J) & 3);                                          \
    }                                                                          \
    NEXT = dense_frags(((J) + 1) & 3);                                         \
    if (!(GUARD) || i + (J) < mine) {                                          \
      mma(CUR);                                                                \
      if (kSum > 0) add_columns(CUR, kSum - 1, (J) & 1);                       \
    }                                                                          \
  }
    uint32_t i = 0;
    while (i + 4u <= n) {
      const uint32_t to = kSum > 0 ? min(i + 128u, n) : n;
      for (; i + 4u <= to; i += 4u) {   // straight-line code: copies, LDS reads and MFMAs interleave
        LT_SLICE(0, f0, f1, false);
        LT_SLICE(1, f1, f0, false);
        LT_SLICE(2, f0, f1, false);
        LT_SLICE(3, f1, f0, false);
      }
      if (kSum > 0) join_columns();
    }
    if (i < n) {                     // one to three left
      LT_SLICE(0, f0, f1, true);
      LT_SLICE(1, f1, f0, true);
      LT_SLICE(2, f0, f1, true);
    }
    };
    if (!CS || !summing) pipeline(Num<0>());
    else if (wave_m == 0u) pipeline(Num<1>());
    else pipeline(Num<2>());
    landed<0>();   // nothing may still be on its way into LDS when it is used again
    }
#undef LT_SLICE
#undef LT_COPY2
#undef LT_COPY
  }
  if (!AL && n > 0u) {
    // an operand whose rows are not 16-byte aligned: through registers into padded LDS tiles, the
    // loads of slice j+1 under the MFMAs of slice j, two buffers and one barrier per slice
    int64_t a_off[Geo<BM>::kChunks], b_off[Geo<BN>::kChunks];
#pragma unroll
    for (int it = 0; it < Geo<BM>::kChunks; ++it) {
      uint32_t o, i;
      chunk_pos<BM, AKC>(it, &o, &i);
      a_off[it] = chunk_offset<BM, AKC>(o, i, a.a.s_row, a.a.s_col, left_m);
    }
#pragma unroll
    for (int it = 0; it < Geo<BN>::kChunks; ++it) {
      uint32_t o, i;
      chunk_pos<BN, BKC>(it, &o, &i);
      b_off[it] = chunk_offset<BN, BKC>(o, i, a.b.s_col, a.b.s_row, left_n);
    }
    Chunks<Geo<BM>::kChunks> ca = fetch_unaligned<BM, AKC>(pa, a_off);
    Chunks<Geo<BN>::kChunks> cb = fetch_unaligned<BN, BKC>(pb, b_off);
    auto step = [&](uint32_t j, bool multiply) {
      char* const st = smem + (j & 1u) * kStage;
      stash<BM, AKC>(ca, st);
      stash<BN, BKC>(cb, st + Geo<BM>::kBytes);
      const int64_t nx = min(j + 1u, mine - 1u);   // (past the end: the last slice again, unused)
      ca = fetch_unaligned<BM, AKC>(pa + nx * step_a, a_off);
      cb = fetch_unaligned<BN, BKC>(pb + nx * step_b, b_off);
      __syncthreads();
      if (multiply) mma_and_sum(load_frags(j & 1u));
    };
    for (uint32_t j = 0; j < both;) {
      const uint32_t to = CS ? min(j + 64u, both) : both;
#pragma unroll 1
      for (; j < to; ++j) step(j, true);
      if (summing) join_columns();
    }
    if (KS > 1 && both < n) step(both, half == 0u);   // (the first half's odd one)
  }
  if (k_rest < k_end) {
    // the rest of k: every address checked, one slice at a time, by the first half
#pragma unroll 1
    for (uint32_t k0 = k_rest; k0 < k_end; k0 += BK) {
      Chunks<Geo<BM>::kChunks> ca;
      Chunks<Geo<BN>::kChunks> cb;
      if (half == 0u) {
        ca = fetch_checked<BM, AKC>(A, a.a.s_row, a.a.s_col, tile_m, k0, a.m, k_end);
        cb = fetch_checked<BN, BKC>(B, a.b.s_col, a.b.s_row, tile_n, k0, a.n, k_end);
      }
      __syncthreads();
      if (half == 0u) {
        stash<BM, AKC>(ca, smem);
        stash<BN, BKC>(cb, smem + Geo<BM>::kBytes);
      }
      __syncthreads();
      if (half == 0u) mma_and_sum(load_frags(0));
    }
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
  epilogue<true, BM, BN, MB, NB, KS, kHalf>(a, acc, (float*)smem_all, tile_m, tile_n, wave_m, wave_n, lane, batch, raw);
  if (summing) finish_columns<BN, 2 * KS>(a, col_lds, tile_n, split);
  args_touched(touched);
}

template <int BM, int BN, bool AL, int KS>
static void launch_layout(const GemmArgs& a, dim3 grid, hipStream_t s) {
  const dim3 block(kGemmThreads * KS);
  const bool akc = a.a.s_col == 1, bkc = a.b.s_row == 1;
  char name[64];   // (no spaces: a launch record holds 47 characters, all but the last bracket)
  if (a.col_sum) {
    if constexpr (BN == 128) {
      LT_LAUNCH((lt_gemm_bf16_kernel<BM, BN, false, false, AL, KS, true>), grid, block, s, a);
      snprintf(name, sizeof(name), "lt_gemm_bf16_kernel<%d,%d,sums,%s,%d>", BM, BN, AL ? "true" : "false", KS);
      note_kernel(name);
    }
    return;
  }
  if (akc && bkc) LT_LAUNCH((lt_gemm_bf16_kernel<BM, BN, true, true, AL, KS, false>), grid, block, s, a);
  else if (akc) LT_LAUNCH((lt_gemm_bf16_kernel<BM, BN, true, false, AL, KS, false>), grid, block, s, a);
  else if (bkc) LT_LAUNCH((lt_gemm_bf16_kernel<BM, BN, false, true, AL, KS, false>), grid, block, s, a);
  else LT_LAUNCH((lt_gemm_bf16_kernel<BM, BN, false, false, AL, KS, false>), grid, block, s, a);
  snprintf(name, sizeof(name), "lt_gemm_bf16_kernel<%d,%d,%s,%s,%s,%d>", BM, BN, akc ? "true" : "false", bkc ? "true" : "false", AL ? "true" : "false", KS);
  note_kernel(name);
}

template <int BM, int BN>
static void launch_tile(const GemmArgs& a, dim3 grid, hipStream_t s) {
  // (a lane's offset into a panel is a 32-bit number of bytes: 128 rows of less than 2^24 elements)
  auto aligned = [](const GemmOperand& o, int64_t outer) {
    return ((uintptr_t)o.ptr & 15u) == 0 && outer % 8 == 0 && outer < (1 << 24) && o.s_b0 % 8 == 0 && o.s_b1 % 8 == 0;
  };
  const bool al = aligned(a.a, a.a.s_col == 1 ? a.a.s_row : a.a.s_col) && aligned(a.b, a.b.s_row == 1 ? a.b.s_col : a.b.s_row);
  if (al && a.halves == 2u) launch_layout<BM, BN, true, 2>(a, grid, s);
  else if (al) launch_layout<BM, BN, true, 1>(a, grid, s);
  else if (a.halves == 2u) launch_layout<BM, BN, false, 2>(a, grid, s);
  else launch_layout<BM, BN, false, 1>(a, grid, s);
}

}  // namespace bf

// a.tile_m, a.tile_n: rows and columns per workgroup tile (128 x 128, or 128 x 64 for narrow outputs).  A
// 256 x 128 tile needs more than the 256 registers that two wavefronts per SIMD leave each, and
// measured slower both ways (two workgroups per compute unit with spills, or one with 385 registers).
// A 256 x 256 tile (128 x 128 per wave, one workgroup per compute unit, 512 registers) runs its main
// loop at twice the matrix-core utilisation of this one (54 % against 28 %), but the layer's shapes
// give it 128 to 512 tiles for 256 compute units and its epilogue has nothing to overlap with:
// 8192 x 4096 x 1024 gains 8 %, 8192 x 1024 x k loses.  Worth it only inside a persistent kernel
// that overlaps one tile's epilogue with the next tile's main loop.
hipError_t launch_gemm_bf16(const GemmArgs& a, hipStream_t s) {
  const uint32_t batch = a.batch0 * a.batch1;
  const uint32_t tiles = a.tiles_m * a.tiles_n;
  if (a.splits == 0u || (a.splits > 1u && !a.split_ws) || (uint64_t)batch * a.splits > 65535u) return hipErrorInvalidValue;
  if (a.halves != 1u && a.halves != 2u) return hipErrorInvalidValue;
  if (a.tile_m != 128u || (a.tile_n != 128u && a.tile_n != 64u)) return hipErrorInvalidValue;
  if (a.tiles_m != (a.m + a.tile_m - 1) / a.tile_m || a.tiles_n != (a.n + a.tile_n - 1) / a.tile_n) return hipErrorInvalidValue;
  if (a.col_sum && !(a.tile_n == 128u && columns_ride(a, batch))) return hipErrorInvalidValue;
  const dim3 grid(tiles, batch * a.splits);
  if (a.tile_n == 64u) bf::launch_tile<128, 64>(a, grid, s);
  else bf::launch_tile<128, 128>(a, grid, s);
  return hipGetLastError();
}

}  // namespace ltk

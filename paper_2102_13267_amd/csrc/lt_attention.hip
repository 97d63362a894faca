// The attention core as it is found in a trace: p = softmax(q k^T), o = p v, and backward
// ds = softmax_grad(dy v^T, p), dq = ds k, dk = ds^T q, dv = p^T dy, for a batch of heads of 32, 64 or 128
// columns.  Scores, probabilities and their gradients never leave the registers; three launches
// (forward, dq, dk + dv) stand for the eight of the parts (lt_lower.cpp finds the pattern).
//
// What bounded the parts: they move the [heads, s, s] tensors through memory six times, their
// products contract 32 to 128 deep (all prologue and epilogue), and rows of odd s defeat vector
// access.  Measured with events, bf16, 128 heads of 200 x 64: forward 11.3, dq 11.2, dk + dv 14.5 us; the eight parts
// take 80 us (107 before their ragged tiles had a path of their own).
//
// One workgroup of four waves takes 128 rows of one head (queries; keys in the dk / dv pass), each wave
// 32 of them, and walks the other side in blocks of TK rows that all four share through LDS, the next block
// on its way into registers meanwhile.  Everything is an MFMA 32x32: scores are computed transposed,
// s^T = k q^T (A: 32 keys from LDS, B: this wave's 32 queries, held in registers), so that a lane owns
// one query's column: row maxima and sums are sums over its registers and one exchange with the
// other half of the wave.  The second product contracts over the rows of that result, and which
// k of an MFMA stands for which row is free as long as both operands agree: the accumulator's
// registers are, converted, the B operand as they are, and A is read from LDS in the matching order
// (bf16: transposing reads, fp32: one row per half wave).  The dk / dv pass is the same with the sides
// swapped.  The forward pass keeps each row's maximum and reciprocal sum, from which the backward passes
// rebuild p exactly.  The correction in ds = p (dp - sum p dp) is summed in a walk of its own over the keys, from the
// very p and dp that the second walk uses: as the row sum of dy * o, with o rounded to bf16, it left the
// rows of ds with a sum that is not zero, which a key bias's gradient (exactly zero) showed.
//
// Rows past the end are copies of the last one on the register side (never stored) and zero in LDS, with
// their scores at minus infinity (forward) or their probabilities at zero (dq).  The dk / dv pass has a copy of the last
// query and its maximum there, but a reciprocal sum of zero: a probability of at most 1, times zero.  (Zeros in
// the query's place meet a key with an infinity as 0 * inf.)
#include <hip/hip_runtime.h>

#include <cstdio>

#include "lt_gemm_epilogue.h"
#include "lt_launch.h"

namespace ltk {

namespace at {
constexpr int kThreads = 256;
constexpr uint32_t kTile = 128;   // rows per workgroup
constexpr float kLog2e = 1.44269504088896340736f;

typedef uint32_t U4 __attribute__((ext_vector_type(4)));
typedef float F4 __attribute__((ext_vector_type(4)));
typedef short S4 __attribute__((ext_vector_type(4)));
typedef short S8 __attribute__((ext_vector_type(8)));
typedef __attribute__((address_space(3))) S4* lds_s4;

template <typename T, int D> struct Geo {
  static constexpr bool BF = sizeof(T) == 2;
  static constexpr int TK = !BF && D == 128 ? 32 : 64;      // rows per block
  static constexpr int NB = TK / 32;
  static constexpr int CH = D * (int)sizeof(T) / 16;        // 16-byte chunks per row
  static constexpr int SB = D * (int)sizeof(T) + 16;        // bytes per LDS row (16 of padding: consecutive rows 4 banks apart)
  static constexpr int N = TK * CH / kThreads;              // chunks per thread and block
  static constexpr int NF = CH / 2;                         // 16-byte fragments of one row per half wave
  static constexpr int DB = D / 32;
};

template <typename T, int D> using Frags = U4[Geo<T, D>::NF];    // one row, half of it per half wave
template <typename T, int D> using Acc = v16f[Geo<T, D>::DB];    // [d][x], d in blocks of 32

// 16 bytes from any element boundary
template <typename T> __device__ __forceinline__ U4 load16(const T* p);
template <> __device__ __forceinline__ U4 load16<uint16_t>(const uint16_t* p) {
  typedef uint32_t V __attribute__((ext_vector_type(4), aligned(2)));
  const V v = *(const V*)p;
  return U4{v.x, v.y, v.z, v.w};
}
template <> __device__ __forceinline__ U4 load16<float>(const float* p) {
  typedef uint32_t V __attribute__((ext_vector_type(4), aligned(4)));
  const V v = *(const V*)p;
  return U4{v.x, v.y, v.z, v.w};
}

template <typename T> __device__ __forceinline__ const T* head(const GemmOperand& o, uint32_t b0, uint32_t b1) {
  return (const T*)o.ptr + (int64_t)b0 * o.s_b0 + (int64_t)b1 * o.s_b1;
}

// one lane's fragments of a row, as the MFMA's B operand: chunk 2 t + h
template <typename T, int D>
__device__ __forceinline__ void row_frags(Frags<T, D>& f, const T* row, uint32_t h) {
#pragma unroll
  for (int t = 0; t < Geo<T, D>::NF; ++t) f[t] = load16<T>(row + (2 * t + h) * (16 / sizeof(T)));
}

// A workgroup's `threads` fetch `count` chunks each: rows from row0 on
template <typename T, int D, int count, int threads>
__device__ __forceinline__ void block_fetch(U4 (&r)[count], const T* base, int64_t s_row, uint32_t row0, uint32_t rows) {
  typedef Geo<T, D> G;
#pragma unroll
  for (int i = 0; i < count; ++i) {
    const uint32_t e = i * threads + threadIdx.x, row = row0 + e / G::CH, c = e % G::CH;
    r[i] = load16<T>(base + (int64_t)min(row, rows - 1u) * s_row + c * (16 / sizeof(T)));
  }
}

template <typename T, int D, int count, int threads>
__device__ __forceinline__ void block_stash(const U4 (&r)[count], char* tile, uint32_t row0, uint32_t rows) {
  typedef Geo<T, D> G;
#pragma unroll
  for (int i = 0; i < count; ++i) {
    const uint32_t e = i * threads + threadIdx.x, row = e / G::CH, c = e % G::CH;
    *(U4*)(tile + row * G::SB + c * 16) = row0 + row < rows ? r[i] : U4{0, 0, 0, 0};
  }
}

// The halves of a workgroup exchange accumulators through LDS (kSwap<D> bytes for one from each of a half's four waves)
template <int D> constexpr int kSwap = 4 * (D / 32) * 16 * 64 * 4;
template <typename T, int D>
__device__ __forceinline__ void swap_put(char* lds, const Acc<T, D>& acc, uint32_t group, uint32_t lane) {
#pragma unroll
  for (int d = 0; d < Geo<T, D>::DB; ++d)
#pragma unroll
    for (int g = 0; g < 4; ++g)
      *(F4*)(lds + (((group * Geo<T, D>::DB + d) * 4 + g) * 64 + lane) * 16) = F4{acc[d][4 * g], acc[d][4 * g + 1], acc[d][4 * g + 2], acc[d][4 * g + 3]};
}
// acc * own + (what the other half put) * theirs
template <typename T, int D>
__device__ __forceinline__ void swap_add(const char* lds, Acc<T, D>& acc, float own, float theirs, uint32_t group, uint32_t lane) {
#pragma unroll
  for (int d = 0; d < Geo<T, D>::DB; ++d)
#pragma unroll
    for (int g = 0; g < 4; ++g) {
      const F4 o = *(const F4*)(lds + (((group * Geo<T, D>::DB + d) * 4 + g) * 64 + lane) * 16);
#pragma unroll
      for (int e = 0; e < 4; ++e) acc[d][4 * g + e] = acc[d][4 * g + e] * own + o[e] * theirs;
    }
}

// x * scale in the type's precision
template <typename T, int count>
__device__ __forceinline__ void scale_chunks(U4 (&x)[count], float scale) {
  if (scale == 1.0f) return;
#pragma unroll
  for (int i = 0; i < count; ++i)
#pragma unroll
    for (int j = 0; j < 4; ++j)
      x[i][j] = sizeof(T) == 2 ? f32_to_bf16_pair(__uint_as_float(x[i][j] << 16) * scale, __uint_as_float(x[i][j] & 0xffff0000u) * scale)
                               : __float_as_uint(__uint_as_float(x[i][j]) * scale);
}

// 32 x 32 block of (LDS rows) . (register rows)^T
template <typename T, int D>
__device__ __forceinline__ v16f dot_rows(const char* tile, uint32_t blk, const Frags<T, D>& f, uint32_t lane) {
  typedef Geo<T, D> G;
  v16f acc;
#pragma unroll
  for (int r = 0; r < 16; ++r) acc[r] = 0.0f;
  const char* p = tile + (blk * 32u + (lane & 31u)) * G::SB + (lane >> 5) * 16u;
#pragma unroll
  for (int t = 0; t < G::NF; ++t) {
    const U4 a = *(const U4*)(p + t * 32);
    if (G::BF) {
      acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(v8bf, a), __builtin_bit_cast(v8bf, f[t]), acc, 0, 0, 0);
    } else {
      const F4 x = __builtin_bit_cast(F4, a), y = __builtin_bit_cast(F4, f[t]);
#pragma unroll
      for (int j = 0; j < 4; ++j) acc = __builtin_amdgcn_mfma_f32_32x32x2f32(x[j], y[j], acc, 0, 0, 0);
    }
  }
  return acc;
}

// acc[d][x] += sum over the 32 rows r of the block: tile[r][d] * p[r][x], p as an accumulator holds it
// (register r of half h: row (r / 4) * 8 + 4 h + r % 4)
template <typename T, int D>
__device__ __forceinline__ void add_rows(Acc<T, D>& acc, const char* tile, uint32_t blk, const v16f& p, uint32_t lane) {
  typedef Geo<T, D> G;
  const uint32_t h = lane >> 5;
  if (G::BF) {
    const uint32_t i16 = lane & 15u;
    const char* base = tile + (blk * 32u + 4u * h + (i16 >> 2)) * G::SB + (((lane & 31u) >> 4) * 16u + 4u * (i16 & 3u)) * 2u;
#pragma unroll
    for (int t = 0; t < 2; ++t) {
      U4 b;
#pragma unroll
      for (int j = 0; j < 4; ++j) b[j] = f32_to_bf16_pair(p[8 * t + 2 * j], p[8 * t + 2 * j + 1]);
#pragma unroll
      for (int d = 0; d < G::DB; ++d) {
        const char* q = base + t * 16 * G::SB + d * 64;
        const S4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s4)q);
        const S4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s4)(q + 8 * G::SB));
        const S8 a = {lo[0], lo[1], lo[2], lo[3], hi[0], hi[1], hi[2], hi[3]};
        acc[d] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(v8bf, a), __builtin_bit_cast(v8bf, b), acc[d], 0, 0, 0);
      }
    }
  } else {
    const char* base = tile + (blk * 32u + 4u * h) * G::SB + (lane & 31u) * 4u;
#pragma unroll
    for (int r = 0; r < 16; ++r)
#pragma unroll
      for (int d = 0; d < G::DB; ++d)
        acc[d] = __builtin_amdgcn_mfma_f32_32x32x2f32(*(const float*)(base + ((r >> 2) * 8 + (r & 3)) * G::SB + d * 128), p[r], acc[d], 0, 0, 0);
  }
}

// acc[d][x] * scale, rounded, * post to row x (= this lane's) of a head's output
template <typename T, int D>
__device__ __forceinline__ void row_store(const Acc<T, D>& acc, float scale, T* row, uint32_t h, float post = 1.0f) {
  const bool twice = post != 1.0f;
#pragma unroll
  for (int d = 0; d < Geo<T, D>::DB; ++d)
#pragma unroll
    for (int g = 0; g < 4; ++g) {
      Quad q;
#pragma unroll
      for (int e = 0; e < 4; ++e) q.v[e] = acc[d][4 * g + e] * scale;
      if (twice) {
#pragma unroll
        for (int e = 0; e < 4; ++e) q.v[e] = (sizeof(T) == 2 ? bf16_to_f32(f32_to_bf16(q.v[e])) : q.v[e]) * post;
      }
      store_vec4_any(row, sizeof(T) == 2 ? kBF16 : kF32, (uint64_t)(d * 32 + g * 8 + 4 * h), q);
    }
}

template <typename T, int D>
__device__ __forceinline__ void clear(Acc<T, D>& acc) {
#pragma unroll
  for (int d = 0; d < Geo<T, D>::DB; ++d)
#pragma unroll
    for (int r = 0; r < 16; ++r) acc[d][r] = 0.0f;
}

__device__ __forceinline__ float other_half(float x) { return __shfl_xor(x, 32); }

template <typename T, int D>
__global__ __launch_bounds__(kThreads, D == 128 ? 1 : 2) void lt_attention_kernel(const AttnArgs a) {
  typedef Geo<T, D> G;
  constexpr int kTileB = G::TK * G::SB;
  __shared__ __attribute__((aligned(16))) char lds[2 * kTileB];
  char *Ks = lds, *Vs = lds + kTileB;
  const uint32_t lane = threadIdx.x & 63u, h = lane >> 5, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const uint32_t tiles = (a.sq + kTile - 1u) / kTile, bh = blockIdx.x / tiles, b0 = bh / a.batch1, b1 = bh % a.batch1;
  const uint32_t q0 = (blockIdx.x % tiles) * kTile + wave * 32u, q = q0 + (lane & 31u);
  const bool busy = q0 < a.sq;
  const T *kp = head<T>(a.k, b0, b1), *vp = head<T>(a.v, b0, b1);
  U4 kr[G::N], vr[G::N];
  block_fetch<T, D, G::N, kThreads>(kr, kp, a.k.s_row, 0, a.sk);
  block_fetch<T, D, G::N, kThreads>(vr, vp, a.v.s_row, 0, a.sk);
  U4 qf[G::NF];
  row_frags<T, D>(qf, head<T>(a.q, b0, b1) + (int64_t)min(q, a.sq - 1u) * a.q.s_row, h);
  scale_chunks<T, G::NF>(qf, a.q_scale);
  v16f acc[G::DB];
  clear<T, D>(acc);
  float m = -INFINITY, l = 0.0f;   // of this lane's query; l over this half's rows
  // (a power of two of at most 1 / keys on every term, in l as well: unnormalised, values of the type's highest few
  // powers of two would add up to infinity)
  const float shrink = __builtin_amdgcn_ldexpf(1.0f, -(32 - (int)__clz((int)(a.sk - 1u))));
  for (uint32_t k0 = 0; k0 < a.sk; k0 += G::TK) {
    __syncthreads();
    block_stash<T, D, G::N, kThreads>(kr, Ks, k0, a.sk);
    block_stash<T, D, G::N, kThreads>(vr, Vs, k0, a.sk);
    __syncthreads();
    block_fetch<T, D, G::N, kThreads>(kr, kp, a.k.s_row, k0 + G::TK, a.sk);   // (past the end: the last row, unused)
    block_fetch<T, D, G::N, kThreads>(vr, vp, a.v.s_row, k0 + G::TK, a.sk);
    if (!busy) continue;
    v16f s[G::NB];
    float mx = m;
#pragma unroll
    for (int b = 0; b < G::NB; ++b) {
      s[b] = dot_rows<T, D>(Ks, b, qf, lane);
      if (k0 + b * 32u + 32u > a.sk) {
#pragma unroll
        for (int r = 0; r < 16; ++r)
          if (k0 + b * 32u + (r >> 2) * 8u + 4u * h + (r & 3) >= a.sk) s[b][r] = -INFINITY;
      }
#pragma unroll
      for (int r = 0; r < 16; ++r) mx = fmaxf(mx, s[b][r]);
    }
    mx = fmaxf(mx, other_half(mx));
    const float base = mx == -INFINITY ? 0.0f : mx;   // (nothing but minus infinity so far: every term is 0)
    const float fade = __builtin_amdgcn_exp2f((m - base) * kLog2e);
    m = mx;
    l *= fade;
#pragma unroll
    for (int d = 0; d < G::DB; ++d)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[d][r] *= fade;
#pragma unroll
    for (int b = 0; b < G::NB; ++b) {
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        s[b][r] = __builtin_amdgcn_exp2f((s[b][r] - base) * kLog2e) * shrink;
        l += s[b][r];
      }
      add_rows<T, D>(acc, Vs, b, s[b], lane);
    }
  }
  l += other_half(l);
  if (q >= a.sq) return;
  const float inv = 1.0f / l;
  row_store<T, D>(acc, inv, (T*)head<T>(a.o, b0, b1) + (int64_t)q * a.o.s_row, h);
  if (a.stats && h == 0u) {
    const uint64_t i = (uint64_t)bh * a.sq + q, n = (uint64_t)a.batch0 * a.batch1 * a.sq;
    a.stats[i] = m;
    a.stats[n + i] = inv * shrink;
  }
}

template <typename T, int D>
__global__ __launch_bounds__(kThreads, D == 128 ? 1 : 2) void lt_attention_dq_kernel(const AttnArgs a) {
  typedef Geo<T, D> G;
  constexpr int kTileB = G::TK * G::SB;
  __shared__ __attribute__((aligned(16))) char lds[2 * kTileB];
  char *Ks = lds, *Vs = lds + kTileB;
  const uint32_t lane = threadIdx.x & 63u, h = lane >> 5, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const uint32_t tiles = (a.sq + kTile - 1u) / kTile, bh = blockIdx.x / tiles, b0 = bh / a.batch1, b1 = bh % a.batch1;
  const uint32_t q0 = (blockIdx.x % tiles) * kTile + wave * 32u, q = q0 + (lane & 31u);
  const uint32_t qc = min(q, a.sq - 1u);
  const bool busy = q0 < a.sq;
  const T *kp = head<T>(a.k, b0, b1), *vp = head<T>(a.v, b0, b1);
  U4 kr[G::N], vr[G::N];
  block_fetch<T, D, G::N, kThreads>(kr, kp, a.k.s_row, 0, a.sk);
  block_fetch<T, D, G::N, kThreads>(vr, vp, a.v.s_row, 0, a.sk);
  U4 qf[G::NF], df[G::NF];
  row_frags<T, D>(qf, head<T>(a.q, b0, b1) + (int64_t)qc * a.q.s_row, h);
  row_frags<T, D>(df, head<T>(a.dy, b0, b1) + (int64_t)qc * a.dy.s_row, h);
  const uint64_t i = (uint64_t)bh * a.sq + qc, n = (uint64_t)a.batch0 * a.batch1 * a.sq;
  const float m = a.stats[i], inv = a.stats[n + i];
  scale_chunks<T, G::NF>(qf, a.q_scale);
  float delta = 0.0f;   // of this lane's query; this half's rows until the first walk is over
  v16f acc[G::DB];
  clear<T, D>(acc);
  const uint32_t blocks = (a.sk + G::TK - 1u) / G::TK;
  // two walks over the keys: the row sum of p * (dy v^T) first, then the gradient
  for (uint32_t it = 0; it < 2u * blocks; ++it) {
    const uint32_t k0 = (it < blocks ? it : it - blocks) * G::TK, k1 = (it + 1u < blocks ? it + 1u : it + 1u - blocks) * G::TK;
    if (it == blocks) delta += other_half(delta);
    __syncthreads();
    block_stash<T, D, G::N, kThreads>(kr, Ks, k0, a.sk);
    block_stash<T, D, G::N, kThreads>(vr, Vs, k0, a.sk);
    __syncthreads();
    block_fetch<T, D, G::N, kThreads>(kr, kp, a.k.s_row, k1, a.sk);
    block_fetch<T, D, G::N, kThreads>(vr, vp, a.v.s_row, k1, a.sk);
    const bool first = it < blocks;
    if (it == blocks && h == 0u && q < a.sq) a.stats[2u * n + i] = delta;
    if (!busy) continue;
#pragma unroll
    for (int b = 0; b < G::NB; ++b) {
      if (k0 + b * 32u >= a.sk) continue;
      v16f s = dot_rows<T, D>(Ks, b, qf, lane);
      const v16f dp = dot_rows<T, D>(Vs, b, df, lane);
#pragma unroll
      for (int r = 0; r < 16; ++r) s[r] = __builtin_amdgcn_exp2f((s[r] - m) * kLog2e) * inv;
      if (k0 + b * 32u + 32u > a.sk) {
#pragma unroll
        for (int r = 0; r < 16; ++r)
          if (k0 + b * 32u + (r >> 2) * 8u + 4u * h + (r & 3) >= a.sk) s[r] = 0.0f;
      }
      if (first) {
#pragma unroll
        for (int r = 0; r < 16; ++r) delta = fmaf(s[r], dp[r], delta);
      } else {
#pragma unroll
        for (int r = 0; r < 16; ++r) s[r] *= dp[r] - delta;
        add_rows<T, D>(acc, Ks, b, s, lane);
      }
    }
  }
  if (q < a.sq) row_store<T, D>(acc, 1.0f, (T*)head<T>(a.dq, b0, b1) + (int64_t)q * a.dq.s_row, h, a.dq_scale);
}

template <typename T, int D>
__global__ __launch_bounds__(kThreads, D == 128 ? 1 : 2) void lt_attention_dkv_kernel(const AttnArgs a) {
  typedef Geo<T, D> G;
  constexpr int kTileB = G::TK * G::SB;
  __shared__ __attribute__((aligned(16))) char lds[2 * kTileB];
  __shared__ __attribute__((aligned(16))) float st[3][G::TK];
  char *Qs = lds, *Ds = lds + kTileB;
  const uint32_t lane = threadIdx.x & 63u, h = lane >> 5, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const uint32_t tiles = (a.sk + kTile - 1u) / kTile, bh = blockIdx.x / tiles, b0 = bh / a.batch1, b1 = bh % a.batch1;
  const uint32_t k0 = (blockIdx.x % tiles) * kTile + wave * 32u, key = k0 + (lane & 31u);
  const uint32_t kc = min(key, a.sk - 1u);
  const bool busy = k0 < a.sk;
  const T *qp = head<T>(a.q, b0, b1), *dp = head<T>(a.dy, b0, b1);
  const float* sp = a.stats + (uint64_t)bh * a.sq;
  const uint64_t n = (uint64_t)a.batch0 * a.batch1 * a.sq;
  U4 qr[G::N], dr[G::N];
  float sr[3] = {0.0f, 0.0f, 0.0f};
  auto fetch = [&](uint32_t q0) {
    block_fetch<T, D, G::N, kThreads>(qr, qp, a.q.s_row, q0, a.sq);
    block_fetch<T, D, G::N, kThreads>(dr, dp, a.dy.s_row, q0, a.sq);
    const uint32_t q = q0 + threadIdx.x;
    if (threadIdx.x < (uint32_t)G::TK) {
#pragma unroll
      for (int j = 0; j < 3; ++j) sr[j] = j == 0 || q < a.sq ? sp[(uint64_t)j * n + min(q, a.sq - 1u)] : 0.0f;
    }
  };
  fetch(0);
  U4 kf[G::NF], vf[G::NF];
  row_frags<T, D>(kf, head<T>(a.k, b0, b1) + (int64_t)kc * a.k.s_row, h);
  row_frags<T, D>(vf, head<T>(a.v, b0, b1) + (int64_t)kc * a.v.s_row, h);
  v16f dk[G::DB], dv[G::DB];
  clear<T, D>(dk);
  clear<T, D>(dv);
  for (uint32_t q0 = 0; q0 < a.sq; q0 += G::TK) {
    __syncthreads();
    scale_chunks<T, G::N>(qr, a.q_scale);
    block_stash<T, D, G::N, kThreads>(qr, Qs, q0, ~0u);   // (past the end: the last query again, see the top)
    block_stash<T, D, G::N, kThreads>(dr, Ds, q0, a.sq);
    if (threadIdx.x < (uint32_t)G::TK) {
#pragma unroll
      for (int j = 0; j < 3; ++j) st[j][threadIdx.x] = sr[j];
    }
    __syncthreads();
    fetch(q0 + G::TK);
    if (!busy) continue;
#pragma unroll
    for (int b = 0; b < G::NB; ++b) {
      if (q0 + b * 32u >= a.sq) continue;
      v16f s = dot_rows<T, D>(Qs, b, kf, lane);
      v16f ds = dot_rows<T, D>(Ds, b, vf, lane);
#pragma unroll
      for (int g = 0; g < 4; ++g) {
        const uint32_t r0 = b * 32u + g * 8u + 4u * h;
        const F4 m = *(const F4*)&st[0][r0], inv = *(const F4*)&st[1][r0], delta = *(const F4*)&st[2][r0];
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const int r = 4 * g + e;
          s[r] = __builtin_amdgcn_exp2f((s[r] - m[e]) * kLog2e) * inv[e];
          ds[r] = s[r] * (ds[r] - delta[e]);
        }
      }
      add_rows<T, D>(dv, Ds, b, s, lane);
      add_rows<T, D>(dk, Qs, b, ds, lane);
    }
  }
  if (key >= a.sk) return;
  row_store<T, D>(dk, 1.0f, (T*)head<T>(a.dk, b0, b1) + (int64_t)key * a.dk.s_row, h);
  row_store<T, D>(dv, 1.0f, (T*)head<T>(a.dv, b0, b1) + (int64_t)key * a.dv.s_row, h);
}

// Up to 256 keys (bf16, heads of up to 64), few workgroups: the walk's cost is its chain of barriers, loads and, in the
// backward pass, the second computation of everything, with one wave per SIMD.  Here all keys are in LDS at once, eight waves share
// them (a group of 32 queries has two, one for every other block of 32 keys), and what the first use of a block computes stays in
// registers for the second.  The halves' sums meet in LDS.  With events around the launch, us, walking / this: 128 heads of
// 200 x 64 forward 12.3 / 11.3, dq 16.9 / 11.2; of 200 x 32 10.1 / 9.1 and 13.3 / 9.1.  Where the launches run which, and why: launch_d.
// (Long walks gain nothing from two halves: at 200 x 64 forward 11.6, dk + dv 15.2 / 14.6, at 256 x 64 and 512 heads dk + dv 40 / 53:
// the registers of both halves fit a compute unit only once.)
template <typename T, int D, int KB>
__global__ __launch_bounds__(2 * kThreads, 4) void lt_attention_kernel_short(const AttnArgs a) {
  typedef Geo<T, D> G;
  constexpr int kT = 2 * kThreads, kRows = 64 * KB, kCount = kRows * G::CH / kT < 1 ? 1 : kRows * G::CH / kT, kTileB = kRows * G::SB;
  static_assert(kRows * G::CH % kT == 0 || kRows * G::CH < kT, "chunks per thread");
  __shared__ __attribute__((aligned(16))) char lds[2 * kTileB > kSwap<D> ? 2 * kTileB : kSwap<D>];
  __shared__ float st[2][kThreads];
  char *Ks = lds, *Vs = lds + kTileB;
  const uint32_t lane = threadIdx.x & 63u, h = lane >> 5, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), group = wave & 3u, half = wave >> 2;
  const uint32_t tiles = (a.sq + kTile - 1u) / kTile, bh = blockIdx.x / tiles, b0 = bh / a.batch1, b1 = bh % a.batch1;
  const uint32_t q0 = (blockIdx.x % tiles) * kTile + group * 32u, q = q0 + (lane & 31u);
  const bool busy = q0 < a.sq;
  {
    U4 kr[kCount], vr[kCount];
    block_fetch<T, D, kCount, kT>(kr, head<T>(a.k, b0, b1), a.k.s_row, 0, a.sk);
    block_fetch<T, D, kCount, kT>(vr, head<T>(a.v, b0, b1), a.v.s_row, 0, a.sk);
    if (kRows * G::CH >= kT || threadIdx.x < (uint32_t)(kRows * G::CH)) {
      block_stash<T, D, kCount, kT>(kr, Ks, 0, a.sk);
      block_stash<T, D, kCount, kT>(vr, Vs, 0, a.sk);
    }
  }
  v16f acc[G::DB];
  clear<T, D>(acc);
  float m = -INFINITY, l = 0.0f;
  const float shrink = __builtin_amdgcn_ldexpf(1.0f, -(32 - (int)__clz((int)(a.sk - 1u))));   // (see above)
  U4 qf[G::NF];
  row_frags<T, D>(qf, head<T>(a.q, b0, b1) + (int64_t)min(q, a.sq - 1u) * a.q.s_row, h);
  scale_chunks<T, G::NF>(qf, a.q_scale);
  __syncthreads();
  if (busy && half * 32u < a.sk) {
    v16f s[KB];
#pragma unroll
    for (int b = 0; b < KB; ++b) {
      const uint32_t blk = 2u * b + half;
      if (blk * 32u >= a.sk) continue;
      s[b] = dot_rows<T, D>(Ks, blk, qf, lane);
      if (blk * 32u + 32u > a.sk) {
#pragma unroll
        for (int r = 0; r < 16; ++r)
          if (blk * 32u + (r >> 2) * 8u + 4u * h + (r & 3) >= a.sk) s[b][r] = -INFINITY;
      }
#pragma unroll
      for (int r = 0; r < 16; ++r) m = fmaxf(m, s[b][r]);
    }
    m = fmaxf(m, other_half(m));
    const float base = m == -INFINITY ? 0.0f : m;
#pragma unroll
    for (int b = 0; b < KB; ++b) {
      const uint32_t blk = 2u * b + half;
      if (blk * 32u >= a.sk) continue;
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        s[b][r] = __builtin_amdgcn_exp2f((s[b][r] - base) * kLog2e) * shrink;
        l += s[b][r];
      }
      add_rows<T, D>(acc, Vs, blk, s[b], lane);
    }
  }
  l += other_half(l);
  __syncthreads();   // (the tiles have been read)
  const uint32_t i = group * 64u + lane;
  if (half == 1u) {
    swap_put<T, D>(lds, acc, group, lane);
    st[0][i] = m;
    st[1][i] = l;
  }
  __syncthreads();
  if (half == 1u || q >= a.sq) return;
  const float m1 = st[0][i], mx = fmaxf(m, m1), base = mx == -INFINITY ? 0.0f : mx;
  const float own = __builtin_amdgcn_exp2f((m - base) * kLog2e), theirs = __builtin_amdgcn_exp2f((m1 - base) * kLog2e);
  l = l * own + st[1][i] * theirs;
  swap_add<T, D>(lds, acc, own, theirs, group, lane);
  const float inv = 1.0f / l;
  row_store<T, D>(acc, inv, (T*)head<T>(a.o, b0, b1) + (int64_t)q * a.o.s_row, h);
  if (a.stats && h == 0u) {
    const uint64_t j = (uint64_t)bh * a.sq + q, n = (uint64_t)a.batch0 * a.batch1 * a.sq;
    a.stats[j] = mx;
    a.stats[n + j] = inv * shrink;
  }
}

// The backward half of it: a block's probabilities and their gradients wait in registers for the row sum
template <typename T, int D, int KB>
__global__ __launch_bounds__(2 * kThreads, 2) void lt_attention_dq_kernel_short(const AttnArgs a) {
  typedef Geo<T, D> G;
  constexpr int kT = 2 * kThreads, kRows = 64 * KB, kCount = kRows * G::CH / kT < 1 ? 1 : kRows * G::CH / kT, kTileB = kRows * G::SB;
  static_assert(kRows * G::CH % kT == 0 || kRows * G::CH < kT, "chunks per thread");
  __shared__ __attribute__((aligned(16))) char lds[2 * kTileB > kSwap<D> ? 2 * kTileB : kSwap<D>];
  __shared__ float st[2][kThreads];
  char *Ks = lds, *Vs = lds + kTileB;
  const uint32_t lane = threadIdx.x & 63u, h = lane >> 5, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), group = wave & 3u, half = wave >> 2;
  const uint32_t tiles = (a.sq + kTile - 1u) / kTile, bh = blockIdx.x / tiles, b0 = bh / a.batch1, b1 = bh % a.batch1;
  const uint32_t q0 = (blockIdx.x % tiles) * kTile + group * 32u, q = q0 + (lane & 31u);
  const uint32_t qc = min(q, a.sq - 1u);
  const bool busy = q0 < a.sq;
  U4 kr[kCount], vr[kCount], qf[G::NF], df[G::NF];
  block_fetch<T, D, kCount, kT>(kr, head<T>(a.k, b0, b1), a.k.s_row, 0, a.sk);
  block_fetch<T, D, kCount, kT>(vr, head<T>(a.v, b0, b1), a.v.s_row, 0, a.sk);
  row_frags<T, D>(qf, head<T>(a.q, b0, b1) + (int64_t)qc * a.q.s_row, h);
  row_frags<T, D>(df, head<T>(a.dy, b0, b1) + (int64_t)qc * a.dy.s_row, h);
  const uint64_t i = (uint64_t)bh * a.sq + qc, n = (uint64_t)a.batch0 * a.batch1 * a.sq;
  const float m = a.stats[i], inv = a.stats[n + i];
  scale_chunks<T, G::NF>(qf, a.q_scale);
  if (kRows * G::CH >= kT || threadIdx.x < (uint32_t)(kRows * G::CH)) {
    block_stash<T, D, kCount, kT>(kr, Ks, 0, a.sk);
    block_stash<T, D, kCount, kT>(vr, Vs, 0, a.sk);
  }
  __syncthreads();
  v16f s[KB], dp[KB], acc[G::DB];
  clear<T, D>(acc);
  float delta = 0.0f;
  if (busy) {
#pragma unroll
    for (int b = 0; b < KB; ++b) {
      const uint32_t blk = 2u * b + half;
      if (blk * 32u >= a.sk) continue;
      s[b] = dot_rows<T, D>(Ks, blk, qf, lane);
      dp[b] = dot_rows<T, D>(Vs, blk, df, lane);
#pragma unroll
      for (int r = 0; r < 16; ++r) s[b][r] = __builtin_amdgcn_exp2f((s[b][r] - m) * kLog2e) * inv;
      if (blk * 32u + 32u > a.sk) {
#pragma unroll
        for (int r = 0; r < 16; ++r)
          if (blk * 32u + (r >> 2) * 8u + 4u * h + (r & 3) >= a.sk) s[b][r] = 0.0f;
      }
#pragma unroll
      for (int r = 0; r < 16; ++r) delta = fmaf(s[b][r], dp[b][r], delta);
    }
  }
  delta += other_half(delta);
  st[half][group * 64u + lane] = delta;
  __syncthreads();
  delta = st[0][group * 64u + lane] + st[1][group * 64u + lane];
  if (half == 0u && h == 0u && q < a.sq) a.stats[2u * n + i] = delta;
  if (busy) {
#pragma unroll
    for (int b = 0; b < KB; ++b) {
      const uint32_t blk = 2u * b + half;
      if (blk * 32u >= a.sk) continue;
#pragma unroll
      for (int r = 0; r < 16; ++r) s[b][r] *= dp[b][r] - delta;
      add_rows<T, D>(acc, Ks, blk, s[b], lane);
    }
  }
  __syncthreads();
  if (half == 1u) swap_put<T, D>(lds, acc, group, lane);
  __syncthreads();
  if (half == 1u) return;
  swap_add<T, D>(lds, acc, 1.0f, 1.0f, group, lane);
  if (q < a.sq) row_store<T, D>(acc, 1.0f, (T*)head<T>(a.dq, b0, b1) + (int64_t)q * a.dq.s_row, h, a.dq_scale);
}

// Which of the two is faster depends on how many workgroups a compute unit gets: few wait for latency, and the short kernels wait
// less; many overlap, and then twice the waves and the exchange of the halves are work on top.  With events round the launch, us,
// walking / short, over 144 to 256 keys and 128 to 1024 queries (heads of 64 unless said otherwise):
//   forward, more than 128 keys: 128 workgroups 9.8 to 11.5 / 9.4 to 10.7, 256 10.8 to 12.8 / 10.3 to 12.9, 384 13.2 to 16.0 / 12.8 to 15.8
//   (on average 3 % less), 512 13.8 to 16.8 / 13.5 to 18.0 (1 % more), 768 17.6 to 21.0 / 19.0 to 23.8, 2048 33 to 42 / 37 to 49.  Up to 128 keys the
//   walk is a step or two: at 16 to 1024 heads of 64 x 64 6.3 to 11.0 / 6.9 to 11.5, of 128 x 64 8.2 to 18.5 / 8.3 to 20.8.
//   dq, more than 128 keys: 256 13.5 to 17.5 / 10.3 to 12.0, 512 17.6 to 25.2 / 17.6 to 23.4, 768 26.6 to 33.3 / 26.4 to 32.8, 1024 31.8 to 44.4 /
//   33.8 to 41.8 (3 % more on average), 2048 53 to 72 / 58 to 78; heads of 32: 1024 16 to 39 / 16 to 34, 2048 36 to 61 / 36 to 59, 4096 55 to 113 / 65 to
//   107.  Up to 128 keys the second walk is what costs: 6.6 to 131 / 6.6 to 132, from 512 workgroups on up to a fifth less.
template <int D>
static bool short_walk(const AttnArgs& a, uint64_t wgs) {
  if (a.pass == kAttnForward) return a.sk > 128u && a.sk <= 256u && wgs <= 384u;
  return a.pass == kAttnDq && (a.sk <= 128u || (a.sk <= 256u && wgs <= (D == 32 ? 2048u : 768u)));
}

template <typename T, int D>
static int launch_short(const AttnArgs& a, dim3 grid, hipStream_t s) {   // (returns KB)
  const dim3 block(2 * kThreads);
  if (a.pass == kAttnForward) {
    LT_LAUNCH((lt_attention_kernel_short<T, D, 4>), grid, block, s, a);
    return 4;
  }
  const int kb = a.sk <= 64u ? 1 : a.sk <= 128u ? 2 : 4;
  if (kb == 1) LT_LAUNCH((lt_attention_dq_kernel_short<T, D, 1>), grid, block, s, a);
  else if (kb == 2) LT_LAUNCH((lt_attention_dq_kernel_short<T, D, 2>), grid, block, s, a);
  else LT_LAUNCH((lt_attention_dq_kernel_short<T, D, 4>), grid, block, s, a);
  return kb;
}

template <typename T, int D>
static hipError_t launch_d(const AttnArgs& a, hipStream_t s) {
  const uint64_t wgs = (uint64_t)a.batch0 * a.batch1 * (((a.pass == kAttnDkv ? a.sk : a.sq) + kTile - 1u) / kTile);
  if (wgs > 0x7fffffffull) return hipErrorInvalidValue;
  const dim3 grid((uint32_t)wgs), block(kThreads);
  const char* const pass = a.pass == kAttnForward ? "" : a.pass == kAttnDq ? "_dq" : "_dkv";
  char name[64];
  int kb = 0;
  if constexpr (sizeof(T) == 2 && D <= 64) {
    if (short_walk<D>(a, wgs)) kb = launch_short<T, D>(a, grid, s);
  }
  if (kb > 0) {
    snprintf(name, sizeof(name), "lt_attention%s_kernel_short<bf16, %d, %d>", pass, D, kb);
  } else {
    if (a.pass == kAttnForward) LT_LAUNCH((lt_attention_kernel<T, D>), grid, block, s, a);
    else if (a.pass == kAttnDq) LT_LAUNCH((lt_attention_dq_kernel<T, D>), grid, block, s, a);
    else LT_LAUNCH((lt_attention_dkv_kernel<T, D>), grid, block, s, a);
    snprintf(name, sizeof(name), "lt_attention%s_kernel<%s, %d>", pass, sizeof(T) == 2 ? "bf16" : "float", D);
  }
  note_kernel(name);
  return hipGetLastError();
}

template <typename T>
static hipError_t launch_t(const AttnArgs& a, hipStream_t s) {
  if (a.d == 32u) return launch_d<T, 32>(a, s);
  if (a.d == 64u) return launch_d<T, 64>(a, s);
  if (a.d == 128u) return launch_d<T, 128>(a, s);
  return hipErrorInvalidValue;
}
}  // namespace at

hipError_t launch_attention(const AttnArgs& a, hipStream_t s) {
  if (a.pass > kAttnDkv || a.sq == 0u || a.sk == 0u || a.batch1 == 0u || a.batch0 == 0u) return hipErrorInvalidValue;
  if (a.pass != kAttnForward && !a.stats) return hipErrorInvalidValue;
  return a.dtype == kBF16 ? at::launch_t<uint16_t>(a, s) : a.dtype == kF32 ? at::launch_t<float>(a, s) : hipErrorInvalidValue;
}

}  // namespace ltk

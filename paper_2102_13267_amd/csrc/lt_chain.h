// Epilogue of a contraction whose post program is a chain (lt_kernels.h): a strip of the product lies in
// LDS, row major, and NT lanes walk it in 16-byte chunks of the output's type, up to 32 elements of a
// lane at a time.
//
// What an epilogue costs is exposed -- the workgroups of a launch reach theirs together -- and in the general
// interpreter it is mostly not the arithmetic: operands are copied out of an indexed register file and the
// result back, element by element, and the slots a program may name keep 128 registers.  Here the running
// values stay where they are, an operand is at most copied once, a bias is loaded once per lane (a lane's
// columns are the same in all its rows), and loads and stores are 16 bytes wide.  8192 x 4096 x 1024 in bf16 with bias,
// GELU and both results stored, tiles of 128 x 128: 124.8 -> 108.2 us, with bias alone 101.5 -> 89.5 (stored as it is:
// 87 to 89), through GELU's gradient 117.2 -> 103.9.  With 16 elements of a lane per trip the first takes 2 us
// longer, with 8 or 4 it takes 12.
#ifndef LT_CHAIN_H_
#define LT_CHAIN_H_
#include <hip/hip_runtime.h>

#include "lt_interp.h"

namespace ltk {

constexpr int kChainN = 32;   // elements of a lane per trip
constexpr int kCPad = 4;   // floats of padding behind a row of the strip

// One 16-byte chunk of a bf16 or fp32 array: as loaded, and as floats.
template <bool BF> struct ChainChunk {
  static constexpr int W = BF ? 8 : 4;
  typedef uint32_t Raw __attribute__((ext_vector_type(4)));
  __device__ static __forceinline__ Raw load(const void* p, uint32_t i) { return *(const Raw*)((const char*)p + (size_t)i * (BF ? 2u : 4u)); }
  __device__ static __forceinline__ float get(const Raw& r, int e) {
    if (BF) return __uint_as_float((e & 1) ? r[e >> 1] & 0xffff0000u : r[e >> 1] << 16);
    return __uint_as_float(r[e]);
  }
  __device__ static __forceinline__ void store(void* p, uint32_t i, const float* v) {
    Raw r;
#pragma unroll
    for (int e = 0; e < 4; ++e) r[e] = BF ? f32_to_bf16_pair(v[2 * e], v[2 * e + 1]) : __float_as_uint(v[e]);
    store_through((char*)p + (size_t)i * (BF ? 2u : 4u), r);
  }
};

struct ChainRegs {
  uint32_t step;   // lane j: step[j]
  float scal;      // lane j: scal[j]
};
// (while every lane of the wave is active)
__device__ __forceinline__ ChainRegs load_chain_regs(const GemmArgs& a) {
  const uint32_t lane = threadIdx.x & 63u;
  ChainRegs r;
  r.step = lane < (uint32_t)kMaxChain ? a.chain.step[lane] : 0u;
  r.scal = lane < (uint32_t)kMaxScal ? a.post.scal[lane] : 0.0f;
  return r;
}

#define LT_CHAIN(EXPR)                                   \
  _Pragma("unroll") for (int e = 0; e < N; ++e) {        \
    const float x = v[e], y = o[e];                      \
    (void)y;                                             \
    v[e] = (EXPR);                                       \
  }
#define LT_CHAIN_SERIAL(EXPR)                            \
  _Pragma("unroll") for (int e = 0; e < N; ++e) {        \
    const float x = v[e], y = o[e];                      \
    (void)y;                                             \
    v[e] = (EXPR);                                       \
    __builtin_amdgcn_sched_barrier(0);                   \
  }

// The strip: ROWS x COLS floats at Cs (rows COLS + kCPad apart), output rows row0 .., columns col0 ..; `t` numbers
// the NT lanes that share it.  base: element offset of the batch's output.  a.n and a.o_row are whole chunks.
template <bool BF, int ROWS, int COLS, int NT>
__device__ __forceinline__ void run_chain(const GemmArgs& a, const ChainRegs cr, const float* Cs, uint32_t t, uint32_t row0, uint32_t col0, int64_t base) {
  typedef ChainChunk<BF> CC;
  typedef typename CC::Raw Raw;
  constexpr int W = CC::W, kStride = COLS + kCPad;
  constexpr uint32_t kLanes = COLS / W, kStep = NT / kLanes, kChunks = ROWS / kStep;   // lanes per row, rows per step, chunks per lane
  constexpr int T = kChunks < kChainN / W ? kChunks : kChainN / W, N = T * W;                    // chunks and elements of a lane per trip
  static_assert(NT % kLanes == 0 && ROWS % kStep == 0 && kChunks % T == 0, "a lane's chunks make whole trips");
  const Chain& ch = a.chain;
  const uint32_t r0 = t / kLanes, c = (t % kLanes) * W, steps = ch.n - 1u;
  // (rows and columns past the edge read the last ones' inputs and store nothing)
  const uint32_t col = min(col0 + c, a.n - (uint32_t)W);
  const bool col_ok = col0 + c < a.n;
  const void* const f0p = a.post.in[ch.full[0]].ptr;
  const void* const f1p = a.post.in[ch.full[1]].ptr;
  Raw row[2];
  row[0] = row[1] = Raw{0u, 0u, 0u, 0u};
  if (ch.n_row > 0u) row[0] = CC::load(a.post.in[ch.row[0]].ptr, col);
  if (ch.n_row > 1u) row[1] = CC::load(a.post.in[ch.row[1]].ptr, col);
#pragma unroll 1
  for (uint32_t trip = 0; trip < kChunks / T; ++trip) {
    uint32_t idx[T];
#pragma unroll
    for (int j = 0; j < T; ++j) idx[j] = (uint32_t)(base + (int64_t)min(row0 + r0 + (trip * T + (uint32_t)j) * kStep, a.m - 1u) * a.o_row + col);
    Raw f0[T], f1[T];
#pragma unroll
    for (int j = 0; j < T; ++j) f0[j] = f1[j] = Raw{0u, 0u, 0u, 0u};
    if (ch.n_full > 0u) {
#pragma unroll
      for (int j = 0; j < T; ++j) f0[j] = CC::load(f0p, idx[j]);
    }
    if (ch.n_full > 1u) {
#pragma unroll
      for (int j = 0; j < T; ++j) f1[j] = CC::load(f1p, idx[j]);
    }
    float v[N];
#pragma unroll
    for (int j = 0; j < T; ++j)
#pragma unroll
      for (int q = 0; q < W / 4; ++q) {
        const float4 x = *(const float4*)&Cs[(r0 + (trip * T + (uint32_t)j) * kStep) * kStride + c + 4 * q];
        v[j * W + 4 * q] = x.x; v[j * W + 4 * q + 1] = x.y; v[j * W + 4 * q + 2] = x.z; v[j * W + 4 * q + 3] = x.w;
      }
    auto store = [&](uint32_t out) {
      void* const p = a.post.out[out].ptr;
#pragma unroll
      for (int j = 0; j < T; ++j)
        if (col_ok && row0 + r0 + (trip * T + (uint32_t)j) * kStep < a.m) CC::store(p, idx[j], &v[j * W]);
    };
    if (ch.first_out != kNoOut) store(ch.first_out);
#pragma unroll 1
    for (uint32_t s = 0; s < steps; ++s) {
      const uint32_t w = (uint32_t)__builtin_amdgcn_readlane((int)cr.step, (int)s);
      const uint32_t op = w & 0xffu, src = (w >> 8) & 15u, out = (w >> 20) & 0xffu;
      const float sc = __uint_as_float((uint32_t)__builtin_amdgcn_readlane((int)__float_as_uint(cr.scal), (int)((w >> 12) & 31u)));
      float o[N];
      switch (src) {
        case kSrcRow0:
#pragma unroll
          for (int e = 0; e < N; ++e) o[e] = CC::get(row[0], e % W);
          break;
        case kSrcRow1:
#pragma unroll
          for (int e = 0; e < N; ++e) o[e] = CC::get(row[1], e % W);
          break;
        case kSrcFull0:
#pragma unroll
          for (int e = 0; e < N; ++e) o[e] = CC::get(f0[e / W], e % W);
          break;
        case kSrcFull1:
#pragma unroll
          for (int e = 0; e < N; ++e) o[e] = CC::get(f1[e / W], e % W);
          break;
        default:
#pragma unroll
          for (int e = 0; e < N; ++e) o[e] = sc;
          break;
      }
      switch (op) {
        case kAdd: LT_CHAIN(x + y) break;
        case kSub: LT_CHAIN(x - y) break;
        case kRsub: LT_CHAIN(y - x) break;
        case kMul: LT_CHAIN(x * y) break;
        case kFma: LT_CHAIN(fmaf(x, sc, y)) break;
        case kRfma: LT_CHAIN(fmaf(y, sc, x)) break;
        case kDiv: LT_CHAIN(fast_div(x, y)) break;
        case kRdiv: LT_CHAIN(fast_div(y, x)) break;
        case kMax: LT_CHAIN((x != x || y != y) ? (x + y) : fmaxf(x, y)) break;
        case kMin: LT_CHAIN((x != x || y != y) ? (x + y) : fminf(x, y)) break;
        case kReluGrad: LT_CHAIN(y > 0.0f ? x : 0.0f) break;
        case kRreluGrad: LT_CHAIN(x > 0.0f ? y : 0.0f) break;
        case kGeluGrad: LT_CHAIN_SERIAL(op_gelu_grad(x, y)) break;
        case kRgeluGrad: LT_CHAIN_SERIAL(op_gelu_grad(y, x)) break;
        case kNeg: LT_CHAIN(-x) break;
        case kAbs: LT_CHAIN(fabsf(x)) break;
        case kSquare: LT_CHAIN(x * x) break;
        case kRelu: LT_CHAIN(x > 0.0f ? x : 0.0f) break;
        case kSqrt: LT_CHAIN(__builtin_amdgcn_sqrtf(x)) break;
        case kRsqrt: LT_CHAIN(__builtin_amdgcn_rsqf(x)) break;
        case kRecip: LT_CHAIN(__builtin_amdgcn_rcpf(x)) break;
        case kGelu: LT_CHAIN_SERIAL(op_gelu(x)) break;
        case kRoundBf16: LT_CHAIN(bf16_to_f32(f32_to_bf16(x))) break;
        default: break;
      }
      if (out != kNoOut) store(out);
    }
  }
}
#undef LT_CHAIN
#undef LT_CHAIN_SERIAL

}  // namespace ltk
#endif  // LT_CHAIN_H_

// Row operators with a fixed body (softmax, layer norm, cross-entropy and their gradients): one
// workgroup or wavefront per row, the row held in registers between passes, LDS only for the
// cross-wave step of the reductions.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstdio>

#include "lt_launch.h"
#include "lt_reduce.h"

namespace ltk {

// ---- fixed-body row operators: the row is held in registers between passes ----------------------
constexpr int kRowVecs = 4;   // 4-vectors per thread: rows up to threads_per_row * 16 columns

struct RowRegs {
  float4 v[kRowVecs];
};

// IO: 0 = element types read from the arguments at run time, 1 = every row-wide tensor is fp32,
// 2 = every row-wide tensor is bf16 (the type branches fold away).
template <int IO>
__device__ __forceinline__ uint32_t io_dtype(uint32_t dtype) {
  return IO == 1 ? (uint32_t)kF32 : IO == 2 ? (uint32_t)kBF16 : dtype;
}

template <int TPR, int IO>
__device__ __forceinline__ RowRegs row_load(const void* ptr, uint32_t dtype_rt, uint64_t base, uint32_t cols, uint32_t lane,
                                            bool vec_ok, float pad) {
  const uint32_t dtype = io_dtype<IO>(dtype_rt);
  RowRegs r;
  if (vec_ok) {
    RawVec raw[kRowVecs];
#pragma unroll
    for (int k = 0; k < kRowVecs; ++k) {   // all loads first, conversions afterwards
      const uint32_t c = (k * TPR + lane) * kVec;
      if (c < cols) raw[k] = fetch_vec4(ptr, dtype, base, c);
    }
#pragma unroll
    for (int k = 0; k < kRowVecs; ++k) {
      const uint32_t c = (k * TPR + lane) * kVec;
      float4 q = make_float4(pad, pad, pad, pad);
      if (c < cols) {
        const Quad t = finish_vec4(dtype, raw[k]);
        q = make_float4(t.v[0], t.v[1], t.v[2], t.v[3]);
      }
      r.v[k] = q;
    }
    return r;
  }
#pragma unroll
  for (int k = 0; k < kRowVecs; ++k) {
    const uint32_t c = (k * TPR + lane) * kVec;
    float4 q = make_float4(pad, pad, pad, pad);
    if (c < cols) {
      q.x = load_elem(ptr, dtype, base + c);
      if (c + 1 < cols) q.y = load_elem(ptr, dtype, base + c + 1);
      if (c + 2 < cols) q.z = load_elem(ptr, dtype, base + c + 2);
      if (c + 3 < cols) q.w = load_elem(ptr, dtype, base + c + 3);
    }
    r.v[k] = q;
  }
  return r;
}

template <int TPR, int IO>
__device__ __forceinline__ void row_store(void* ptr, uint32_t dtype_rt, uint64_t base, uint32_t cols, uint32_t lane, bool vec_ok,
                                          const RowRegs& r) {
  const uint32_t dtype = io_dtype<IO>(dtype_rt);
#pragma unroll
  for (int k = 0; k < kRowVecs; ++k) {
    const uint32_t c = (k * TPR + lane) * kVec;
    if (c >= cols) continue;
    const float4 q = r.v[k];
    if (vec_ok) {
      if (dtype == kBF16) {
        uint2 u;
        u.x = f32_to_bf16_pair(q.x, q.y);
        u.y = f32_to_bf16_pair(q.z, q.w);
        *(uint2*)((uint16_t*)ptr + base + c) = u;
      } else {
        *(float4*)((float*)ptr + base + c) = q;
      }
    } else {
      store_elem(ptr, dtype, base + c, q.x);
      if (c + 1 < cols) store_elem(ptr, dtype, base + c + 1, q.y);
      if (c + 2 < cols) store_elem(ptr, dtype, base + c + 2, q.z);
      if (c + 3 < cols) store_elem(ptr, dtype, base + c + 3, q.w);
    }
  }
}

// Reduce over the TPR lanes that share a row: 16 (a quarter wavefront), 64 or the workgroup.
template <int TPR>
__device__ __forceinline__ float row_reduce_regs(uint32_t red, const RowRegs& r, float* lds) {
  float acc = red_identity(red);
#pragma unroll
  for (int k = 0; k < kRowVecs; ++k) {
    acc = red_combine(red, acc, red_combine(red, red_combine(red, r.v[k].x, r.v[k].y),
                                            red_combine(red, r.v[k].z, r.v[k].w)));
  }
  return TPR == 16 ? row16_reduce(red, acc) : TPR == 64 ? wave_reduce(red, acc) : block_reduce(red, acc, lds);
}

#define LT_ROW_FOREACH(BODY)                                   \
  _Pragma("unroll") for (int k = 0; k < kRowVecs; ++k) {       \
    { float& e = x.v[k].x; const int j = 0; (void)j; BODY }    \
    { float& e = x.v[k].y; const int j = 1; (void)j; BODY }    \
    { float& e = x.v[k].z; const int j = 2; (void)j; BODY }    \
    { float& e = x.v[k].w; const int j = 3; (void)j; BODY }    \
  }

__device__ __forceinline__ float comp(const float4& q, int j) { return j == 0 ? q.x : j == 1 ? q.y : j == 2 ? q.z : q.w; }

template <int OP, int TPR, int IO>
__global__ __launch_bounds__(kBlock) void lt_row_op_kernel(const RowOpArgs a) {
  __shared__ float lds[kBlock / 64];
  constexpr uint32_t tpr = TPR;
  constexpr uint32_t rows_per_block = kBlock / tpr;
  const uint32_t lane = threadIdx.x % tpr, sub = threadIdx.x / tpr;
  const uint32_t cols = a.cols;
  const bool vec_ok = (cols % kVec) == 0;
  const uint32_t nblocks = (a.rows + rows_per_block - 1) / rows_per_block;
  float total = 0.0f;   // losses of this thread's rows
  for (uint32_t blk = blockIdx.x; blk < nblocks; blk += gridDim.x) {
    const uint32_t row = blk * rows_per_block + sub;
    // with 256 threads per row every thread of the workgroup works on the same row, so the
    // workgroup barriers inside block_reduce are reached uniformly; with 64 there are none
    const bool live = row < a.rows;
    const uint64_t base = (uint64_t)(live ? row : 0) * cols;
    const uint32_t ecols = live ? cols : 0u;
    switch (OP) {
      case kSoftmax: {
        RowRegs x = row_load<TPR, IO>(a.in[0], a.in_dtype[0], base, ecols, lane, vec_ok, -INFINITY);
        const float m = row_reduce_regs<TPR>(kRedMax, x, lds);
        LT_ROW_FOREACH(e = __expf(e - m);)
        const float s = row_reduce_regs<TPR>(kRedSum, x, lds);
        const float inv = 1.0f / s;
        LT_ROW_FOREACH(e = e * inv;)
        row_store<TPR, IO>(a.out[0], a.out_dtype[0], base, ecols, lane, vec_ok, x);
      } break;
      case kSoftmaxGrad: {
        RowRegs x = row_load<TPR, IO>(a.in[0], a.in_dtype[0], base, ecols, lane, vec_ok, 0.0f);   // dy
        RowRegs y = row_load<TPR, IO>(a.in[1], a.in_dtype[1], base, ecols, lane, vec_ok, 0.0f);
        RowRegs t = x;
#pragma unroll
        for (int k = 0; k < kRowVecs; ++k) {
          t.v[k].x *= y.v[k].x; t.v[k].y *= y.v[k].y; t.v[k].z *= y.v[k].z; t.v[k].w *= y.v[k].w;
        }
        const float dot = row_reduce_regs<TPR>(kRedSum, t, lds);
        LT_ROW_FOREACH(e = comp(y.v[k], j) * (e - dot);)
        row_store<TPR, IO>(a.out[0], a.out_dtype[0], base, ecols, lane, vec_ok, x);
      } break;
      case kLayerNorm: {
        RowRegs x = row_load<TPR, IO>(a.in[0], a.in_dtype[0], base, ecols, lane, vec_ok, 0.0f);
        // scale and shift are asked for together with the row: their (cache) latency passes under
        // the two reductions instead of after them
        RowRegs g = row_load<TPR, IO>(a.in[1], a.in_dtype[1], 0, ecols, lane, vec_ok, 0.0f);
        RowRegs b = row_load<TPR, IO>(a.in[2], a.in_dtype[2], 0, ecols, lane, vec_ok, 0.0f);
        const float mean = row_reduce_regs<TPR>(kRedSum, x, lds) / (float)cols;
        RowRegs d = x;
#pragma unroll
        for (int k = 0; k < kRowVecs; ++k) {
          const uint32_t c = (k * tpr + lane) * kVec;
          d.v[k].x = (c + 0 < ecols) ? (x.v[k].x - mean) * (x.v[k].x - mean) : 0.0f;
          d.v[k].y = (c + 1 < ecols) ? (x.v[k].y - mean) * (x.v[k].y - mean) : 0.0f;
          d.v[k].z = (c + 2 < ecols) ? (x.v[k].z - mean) * (x.v[k].z - mean) : 0.0f;
          d.v[k].w = (c + 3 < ecols) ? (x.v[k].w - mean) * (x.v[k].w - mean) : 0.0f;
        }
        const float var = row_reduce_regs<TPR>(kRedSum, d, lds) / (float)cols;
        const float rstd = 1.0f / sqrtf(var + a.eps);
        LT_ROW_FOREACH(e = (e - mean) * rstd * comp(g.v[k], j) + comp(b.v[k], j);)
        row_store<TPR, IO>(a.out[0], a.out_dtype[0], base, ecols, lane, vec_ok, x);
        if (lane == 0 && live) {
          store_elem(a.out[1], a.out_dtype[1], row, mean);
          store_elem(a.out[2], a.out_dtype[2], row, rstd);
        }
      } break;
      case kLayerNormGrad: {
        // in: dy, x, gamma, mean, rstd
        RowRegs x = row_load<TPR, IO>(a.in[0], a.in_dtype[0], base, ecols, lane, vec_ok, 0.0f);   // dy -> g
        RowRegs xh = row_load<TPR, IO>(a.in[1], a.in_dtype[1], base, ecols, lane, vec_ok, 0.0f);
        RowRegs gm = row_load<TPR, IO>(a.in[2], a.in_dtype[2], 0, ecols, lane, vec_ok, 0.0f);
        const float mean = live ? load_elem(a.in[3], a.in_dtype[3], row) : 0.0f;
        const float rstd = live ? load_elem(a.in[4], a.in_dtype[4], row) : 0.0f;
        LT_ROW_FOREACH(e = e * comp(gm.v[k], j);)
#pragma unroll
        for (int k = 0; k < kRowVecs; ++k) {
          const uint32_t c = (k * tpr + lane) * kVec;
          xh.v[k].x = (c + 0 < ecols) ? (xh.v[k].x - mean) * rstd : 0.0f;
          xh.v[k].y = (c + 1 < ecols) ? (xh.v[k].y - mean) * rstd : 0.0f;
          xh.v[k].z = (c + 2 < ecols) ? (xh.v[k].z - mean) * rstd : 0.0f;
          xh.v[k].w = (c + 3 < ecols) ? (xh.v[k].w - mean) * rstd : 0.0f;
        }
        const float mg = row_reduce_regs<TPR>(kRedSum, x, lds) / (float)cols;
        RowRegs t = x;
#pragma unroll
        for (int k = 0; k < kRowVecs; ++k) {
          t.v[k].x *= xh.v[k].x; t.v[k].y *= xh.v[k].y; t.v[k].z *= xh.v[k].z; t.v[k].w *= xh.v[k].w;
        }
        const float mgx = row_reduce_regs<TPR>(kRedSum, t, lds) / (float)cols;
        LT_ROW_FOREACH(e = rstd * (e - mg - comp(xh.v[k], j) * mgx);)
        row_store<TPR, IO>(a.out[0], a.out_dtype[0], base, ecols, lane, vec_ok, x);
      } break;
      case kXent:
      case kXentGrad: {
        RowRegs x = row_load<TPR, IO>(a.in[0], a.in_dtype[0], base, ecols, lane, vec_ok, -INFINITY);
        const int32_t label = live ? ((const int32_t*)a.in[1])[row] : 0;
        const float m = row_reduce_regs<TPR>(kRedMax, x, lds);
        RowRegs ex = x;
#pragma unroll
        for (int k = 0; k < kRowVecs; ++k) {
          ex.v[k].x = expf(x.v[k].x - m); ex.v[k].y = expf(x.v[k].y - m);
          ex.v[k].z = expf(x.v[k].z - m); ex.v[k].w = expf(x.v[k].w - m);
        }
        const float s = row_reduce_regs<TPR>(kRedSum, ex, lds);
        // A loss and its gradient read the same logits and need the same maximum and sum: one launch and one pass for
        // both (128 x 10: 6.2 + 6.1 -> 6.3 us with events around them, 2048 x 1000: 7.1 + 7.9 -> 8.9).
        void* const loss = OP == kXent ? a.out[0] : a.out[1];
        if (loss) {
          // the picked logit: only the lane holding column `label` contributes
          float picked = 0.0f;
#pragma unroll
          for (int k = 0; k < kRowVecs; ++k) {
            const int32_t c = (int32_t)((k * tpr + lane) * kVec);
            if (label == c) picked = x.v[k].x;
            if (label == c + 1) picked = x.v[k].y;
            if (label == c + 2) picked = x.v[k].z;
            if (label == c + 3) picked = x.v[k].w;
          }
          RowRegs pk;
#pragma unroll
          for (int k = 0; k < kRowVecs; ++k) pk.v[k] = make_float4(0.f, 0.f, 0.f, 0.f);
          pk.v[0].x = picked;
          const float pv = row_reduce_regs<TPR>(kRedSum, pk, lds);
          if (lane == 0 && live) {
            const float l = logf(s) + m - pv;
            store_elem(loss, a.out_dtype[OP == kXent ? 0 : 1], row, l);
            total += l;
          }
        }
        if (OP == kXentGrad) {
          const float inv = 1.0f / s;
#pragma unroll
          for (int k = 0; k < kRowVecs; ++k) {
            const int32_t c = (int32_t)((k * tpr + lane) * kVec);
            ex.v[k].x = (ex.v[k].x * inv - (label == c ? 1.0f : 0.0f)) * a.scale;
            ex.v[k].y = (ex.v[k].y * inv - (label == c + 1 ? 1.0f : 0.0f)) * a.scale;
            ex.v[k].z = (ex.v[k].z * inv - (label == c + 2 ? 1.0f : 0.0f)) * a.scale;
            ex.v[k].w = (ex.v[k].w * inv - (label == c + 3 ? 1.0f : 0.0f)) * a.scale;
          }
          row_store<TPR, IO>(a.out[0], a.out_dtype[0], base, ecols, lane, vec_ok, ex);
        }
      } break;
      default: break;
    }
  }
  // The mean loss as a launch of its own is a launch's latency for a handful of values: 128 x 10 with events around the
  // launches 6.3 + 6.0 us, here 7.2.
  if constexpr (OP == kXent || OP == kXentGrad) {
    if (!a.has_total) return;
    __shared__ uint32_t is_last;
    float r = block_reduce(kRedSum, total, lds);
    if (gridDim.x > 1u) {
      if (threadIdx.x == 0u) {
        publish(&a.total_parts[blockIdx.x], r);
        all_published();
        const uint32_t t = atomicAdd(a.total_ticket, 1u);
        is_last = t == gridDim.x - 1u ? 1u : 0u;
        if (t == gridDim.x - 1u) *a.total_ticket = 0u;   // (every workgroup has been here)
      }
      __syncthreads();
      if (!is_last) return;
      total = 0.0f;
      for (uint32_t i = threadIdx.x; i < gridDim.x; i += (uint32_t)kBlock) total += published(&a.total_parts[i]);
      r = block_reduce(kRedSum, total, lds);
    }
    if (threadIdx.x == 0u) *a.total = a.total_red == kRedMean ? r / (float)a.rows : r;
  }
}


// ---- layer norm and its gradient, streamed ------------------------------------------------------
// Rows whose wide tensors share one element type: a wave per row, 16 bytes per lane and load (twice
// what the general kernel fetches of a bf16 row at once), scale and shift kept in registers over the rows that a
// wave walks, and the next row on its way while this one is reduced.  NV: 16-byte chunks per lane, so
// rows of up to 512 NV (bf16) or 256 NV (fp32) columns in whole chunks.  Memory bounds it, then the
// two chained reductions of a row; 8192 x 1024 in bf16: 8.2 us forward, 9.4 backward (14.5 and 15.4).
template <bool BF> struct Wide;
template <> struct Wide<true> { static constexpr int E = 8; typedef uint16_t T; };
template <> struct Wide<false> { static constexpr int E = 4; typedef float T; };
typedef uint32_t Raw16 __attribute__((ext_vector_type(4)));

template <bool BF>
__device__ __forceinline__ Raw16 wide_load(const void* p, uint64_t elem) {   // from any element boundary
  if (BF) {
    typedef uint32_t V __attribute__((ext_vector_type(4), aligned(2)));
    const V v = *(const V*)((const uint16_t*)p + elem);
    return Raw16{v.x, v.y, v.z, v.w};
  }
  typedef uint32_t V __attribute__((ext_vector_type(4), aligned(4)));
  const V v = *(const V*)((const float*)p + elem);
  return Raw16{v.x, v.y, v.z, v.w};
}
template <bool BF>
__device__ __forceinline__ float wide_get(const Raw16& r, int e) {
  if (!BF) return __uint_as_float(r[e]);
  return __uint_as_float((e & 1) ? r[e >> 1] & 0xffff0000u : r[e >> 1] << 16);
}
template <bool BF>
__device__ __forceinline__ void wide_store(void* p, uint64_t elem, const float* v) {
  if (BF) {
    typedef uint32_t V __attribute__((ext_vector_type(4), aligned(2)));
    *(V*)((uint16_t*)p + elem) = V{f32_to_bf16_pair(v[0], v[1]), f32_to_bf16_pair(v[2], v[3]), f32_to_bf16_pair(v[4], v[5]), f32_to_bf16_pair(v[6], v[7])};
  } else {
    typedef float V __attribute__((ext_vector_type(4), aligned(4)));
    *(V*)((float*)p + elem) = V{v[0], v[1], v[2], v[3]};
  }
}

// CS > 0 (gradient only): the weight gradient's sums over the rows of dy * xhat, and with CS = 2 the bias gradient's of dy,
// ride along.  Both read what this pass has in registers, and a lane's columns are the same in all its rows, so a row costs
// two additions per element; as a launch of their own they are a second pass over both tensors.  Workgroups are
// twice the size and walk more rows each (RowOpArgs::col_rows of them), so that fewer partial sums are left for the
// launch that adds them up.  Norm forward, gradient and sums, us a pass (28 to 31 of it are the
// host's time): 8192 x 1024 in bf16 35.4 -> 31.5, fp32 52.8 -> 36.5, 16000 x 2048 in bf16 118.6 -> 70.1, 131072 x 256 216 -> 90.
template <int OP, int NV, bool BF, int CS>
__global__ __launch_bounds__(CS ? 2 * kBlock : kBlock) void lt_norm_stream_kernel(const RowOpArgs a) {
  constexpr uint32_t kWaves = (CS ? 2 * kBlock : kBlock) / 64;
  constexpr int E = Wide<BF>::E, N = NV * E;
  constexpr bool kGrad = OP == kLayerNormGrad;   // in: dy, x, gain, mean, rstd; otherwise x, gain, shift
  const uint32_t lane = threadIdx.x & 63u, wave = blockIdx.x * kWaves + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), waves = gridDim.x * kWaves;
  const uint32_t cols = a.cols;
  uint32_t col[NV];
  bool in[NV];
#pragma unroll
  for (int k = 0; k < NV; ++k) {
    in[k] = (k * 64u + lane) * E < cols;
    col[k] = in[k] ? (k * 64u + lane) * E : 0u;   // (a lane past the end: the row's first chunk, left out of everything)
  }
  Raw16 r0[NV], r1[NV], g[NV], b[NV];
  auto fetch = [&](uint32_t row) {
    const uint64_t base = (uint64_t)min(row, a.rows - 1u) * cols;
#pragma unroll
    for (int k = 0; k < NV; ++k) {
      r0[k] = wide_load<BF>(a.in[0], base + col[k]);
      if (kGrad) r1[k] = wide_load<BF>(a.in[1], base + col[k]);
    }
  };
  float mean_n = 0.0f, rstd_n = 0.0f;
  auto fetch_stats = [&](uint32_t row) {
    const uint32_t r = min(row, a.rows - 1u);
    mean_n = load_elem(a.in[3], a.in_dtype[3], r);
    rstd_n = load_elem(a.in[4], a.in_dtype[4], r);
  };
  fetch(wave);
  if (kGrad) fetch_stats(wave);
  float sum[CS > 0 ? CS : 1][CS > 0 ? N : 1];
  if (CS > 0) {
#pragma unroll
    for (int c = 0; c < CS; ++c)
#pragma unroll
      for (int i = 0; i < N; ++i) sum[c][CS > 0 ? i : 0] = 0.0f;
  }
#pragma unroll
  for (int k = 0; k < NV; ++k) {
    g[k] = wide_load<BF>(a.in[kGrad ? 2 : 1], col[k]);
    if (!kGrad) b[k] = wide_load<BF>(a.in[2], col[k]);
  }
  for (uint32_t row = wave; row < a.rows; row += waves) {
    float x[N], t[N];
    float s = 0.0f, s2 = 0.0f;
    const uint64_t base = (uint64_t)row * cols;
    if (!kGrad) {
#pragma unroll
      for (int k = 0; k < NV; ++k)
#pragma unroll
        for (int e = 0; e < E; ++e) {
          x[k * E + e] = wide_get<BF>(r0[k], e);
          s += in[k] ? x[k * E + e] : 0.0f;
        }
      fetch(row + waves);
      const float mean = wave_reduce(kRedSum, s) / (float)cols;
#pragma unroll
      for (int k = 0; k < NV; ++k)
#pragma unroll
        for (int e = 0; e < E; ++e) {
          x[k * E + e] -= mean;
          s2 += in[k] ? x[k * E + e] * x[k * E + e] : 0.0f;
        }
      const float var = wave_reduce(kRedSum, s2) / (float)cols;
      const float rstd = 1.0f / sqrtf(var + a.eps);
#pragma unroll
      for (int k = 0; k < NV; ++k) {
#pragma unroll
        for (int e = 0; e < E; ++e) t[k * E + e] = x[k * E + e] * rstd * wide_get<BF>(g[k], e) + wide_get<BF>(b[k], e);
        if (in[k]) wide_store<BF>(a.out[0], base + col[k], t + k * E);
      }
      if (lane == 0u) {
        store_elem(a.out[1], a.out_dtype[1], row, mean);
        store_elem(a.out[2], a.out_dtype[2], row, rstd);
      }
    } else {
      const float mean = mean_n, rstd = rstd_n;
#pragma unroll
      for (int k = 0; k < NV; ++k)
#pragma unroll
        for (int e = 0; e < E; ++e) {
          const int i = k * E + e;
          x[i] = wide_get<BF>(r0[k], e) * wide_get<BF>(g[k], e);
          t[i] = (wide_get<BF>(r1[k], e) - mean) * rstd;
          s += in[k] ? x[i] : 0.0f;
          s2 += in[k] ? x[i] * t[i] : 0.0f;
          if (CS > 0) sum[0][CS > 0 ? i : 0] += wide_get<BF>(r0[k], e) * t[i];
          if (CS > 1) sum[CS > 1 ? 1 : 0][CS > 1 ? i : 0] += wide_get<BF>(r0[k], e);
        }
      fetch(row + waves);
      fetch_stats(row + waves);
      const float mg = wave_reduce(kRedSum, s) / (float)cols, mgx = wave_reduce(kRedSum, s2) / (float)cols;
#pragma unroll
      for (int k = 0; k < NV; ++k) {
#pragma unroll
        for (int e = 0; e < E; ++e) t[k * E + e] = rstd * (x[k * E + e] - mg - t[k * E + e] * mgx);
        if (in[k]) wide_store<BF>(a.out[0], base + col[k], t + k * E);
      }
    }
  }
  if (CS > 0) {   // the waves' sums meet in LDS, in order
    __shared__ float4 meet[CS > 0 ? kWaves * 64 * N / 4 : 1];
    constexpr uint32_t kQuads = 64u * N / 4u;   // of a row of NV chunks per lane
#pragma unroll
    for (int c = 0; c < CS; ++c) {
      if (c > 0) __syncthreads();
#pragma unroll
      for (int i = 0; i < N; i += 4)
        meet[(threadIdx.x >> 6) * kQuads + ((uint32_t)(i / E) * 64u + lane) * (E / 4) + (uint32_t)(i % E) / 4u] =
            make_float4(sum[c][CS > 0 ? i : 0], sum[c][CS > 0 ? i + 1 : 0], sum[c][CS > 0 ? i + 2 : 0], sum[c][CS > 0 ? i + 3 : 0]);
      __syncthreads();
      for (uint32_t q = threadIdx.x; q < cols / 4u; q += blockDim.x) {
        float4 v = meet[q];
#pragma unroll
        for (uint32_t w = 1; w < kWaves; ++w) {
          const float4 o = meet[w * kQuads + q];
          v.x += o.x; v.y += o.y; v.z += o.z; v.w += o.w;
        }
        *(float4*)(a.col_parts + ((uint64_t)blockIdx.x * CS + c) * cols + q * 4u) = v;
      }
    }
  }
}

template <int OP, int NV, bool BF, int CS = 0>
static hipError_t launch_norm(const RowOpArgs& a, hipStream_t s) {
  // (a wave per row until the chip holds four waves per SIMD; then each walks a few)
  const uint32_t grid = CS ? a.col_rows : std::min((a.rows + kBlock / 64u - 1u) / (kBlock / 64u), 1024u);
  LT_LAUNCH((lt_norm_stream_kernel<OP, NV, BF, CS>), dim3(grid), dim3(CS ? 2 * kBlock : kBlock), s, a);
  char name[48];
  snprintf(name, sizeof(name), "lt_norm_stream_kernel<%d, %d, %s, %d>", (int)OP, NV, BF ? "true" : "false", CS);
  note_kernel(name);
  return hipGetLastError();
}
template <int OP, bool BF>
static hipError_t launch_norm_cols(const RowOpArgs& a, hipStream_t s) {
  const uint32_t per = 64u * Wide<BF>::E;
  if constexpr (OP == kLayerNormGrad) {
    if (a.col_sums > 2u || (a.col_sums && (!a.col_parts || a.col_rows == 0u || a.cols > 4u * per))) return hipErrorInvalidValue;
    if (a.col_sums == 1u) return a.cols <= per ? launch_norm<OP, 1, BF, 1>(a, s) : a.cols <= 2u * per ? launch_norm<OP, 2, BF, 1>(a, s) : launch_norm<OP, 4, BF, 1>(a, s);
    if (a.col_sums == 2u) return a.cols <= per ? launch_norm<OP, 1, BF, 2>(a, s) : a.cols <= 2u * per ? launch_norm<OP, 2, BF, 2>(a, s) : launch_norm<OP, 4, BF, 2>(a, s);
  }
  if (a.cols <= per) return launch_norm<OP, 1, BF>(a, s);
  if (a.cols <= 2u * per) return launch_norm<OP, 2, BF>(a, s);
  if (a.cols <= 4u * per) return launch_norm<OP, 4, BF>(a, s);
  return launch_norm<OP, 8, BF>(a, s);
}

template <int OP, int TPR>
static void launch_io(const RowOpArgs& a, int io, uint32_t grid, hipStream_t s) {
  if (io == 1) LT_LAUNCH((lt_row_op_kernel<OP, TPR, 1>), dim3(grid), dim3(kBlock), s, a);
  else if (io == 2) LT_LAUNCH((lt_row_op_kernel<OP, TPR, 2>), dim3(grid), dim3(kBlock), s, a);
  else LT_LAUNCH((lt_row_op_kernel<OP, TPR, 0>), dim3(grid), dim3(kBlock), s, a);
  char name[48];
  snprintf(name, sizeof(name), "lt_row_op_kernel<%d, %d, %d>", (int)OP, (int)TPR, io == 1 ? 1 : io == 2 ? 2 : 0);
  note_kernel(name);
}

template <int OP>
static hipError_t launch_tpr(const RowOpArgs& a, int io, uint32_t grid, hipStream_t s) {
  if (a.threads_per_row == 16u) launch_io<OP, 16>(a, io, grid, s);
  else if (a.threads_per_row == 64u) launch_io<OP, 64>(a, io, grid, s);
  else if (a.threads_per_row == 256u) launch_io<OP, 256>(a, io, grid, s);
  else return hipErrorInvalidValue;
  return hipGetLastError();
}

// Which tensors of an operator are read or written a whole row at a time (the others are one
// value per row and keep their run-time type).
hipError_t launch_row_op(const RowOpArgs& a, uint32_t grid, hipStream_t s) {
  uint32_t wide_in = 0, wide_out = 1;
  if (a.has_total && ((a.op != kXent && a.op != kXentGrad) || !a.total || !a.total_parts || !a.total_ticket)) return hipErrorInvalidValue;
  switch (a.op) {
    case kSoftmax: wide_in = 1; break;
    case kSoftmaxGrad: wide_in = 2; break;
    case kLayerNorm: wide_in = 3; break;
    case kLayerNormGrad: wide_in = 3; break;
    case kXent: wide_in = 1; wide_out = 0; break;
    case kXentGrad: wide_in = 1; break;
    default: return hipErrorInvalidValue;
  }
  bool f32 = true, bf16 = true;
  for (uint32_t i = 0; i < wide_in; ++i) { f32 &= a.in_dtype[i] == kF32; bf16 &= a.in_dtype[i] == kBF16; }
  for (uint32_t i = 0; i < wide_out; ++i) { f32 &= a.out_dtype[i] == kF32; bf16 &= a.out_dtype[i] == kBF16; }
  const int io = f32 ? 1 : bf16 ? 2 : 0;
  // rows of whole 16-byte chunks, at most eight to a lane: the streamed layer norm
  if ((a.op == kLayerNorm || a.op == kLayerNormGrad) && io != 0 && a.rows > 0u && a.cols > 0u && a.cols % (io == 2 ? 8u : 4u) == 0u &&
      a.cols <= (io == 2 ? 4096u : 2048u)) {
    if (a.op == kLayerNorm) return io == 2 ? launch_norm_cols<kLayerNorm, true>(a, s) : launch_norm_cols<kLayerNorm, false>(a, s);
    return io == 2 ? launch_norm_cols<kLayerNormGrad, true>(a, s) : launch_norm_cols<kLayerNormGrad, false>(a, s);
  }
  if (a.col_sums) return hipErrorInvalidValue;   // (only the streamed gradient takes sums along)
  switch (a.op) {
    case kSoftmax: return launch_tpr<kSoftmax>(a, io, grid, s);
    case kSoftmaxGrad: return launch_tpr<kSoftmaxGrad>(a, io, grid, s);
    case kLayerNorm: return launch_tpr<kLayerNorm>(a, io, grid, s);
    case kLayerNormGrad: return launch_tpr<kLayerNormGrad>(a, io, grid, s);
    case kXent: return launch_tpr<kXent>(a, io, grid, s);
    default: return launch_tpr<kXentGrad>(a, io, grid, s);
  }
}

}  // namespace ltk

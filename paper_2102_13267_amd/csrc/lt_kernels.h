// Kernel argument blocks shared by the host lowering pass and the HIP kernels.
//
// Every fused region is run by one kernel family.  What varies per region -- the
// elementwise chain -- is not compiled: it is a small bytecode program that lives in
// the kernel-argument segment (read through scalar loads) and is interpreted with the
// value slots held in vector registers.  The paper leaves code generation to its
// backend compiler (section 4, "lowering"); this build replaces that compiler with an
// interpreter so that a cache miss costs microseconds, not a JIT run.
#ifndef LT_KERNELS_H_
#define LT_KERNELS_H_

#include <stdint.h>

namespace ltk {

constexpr int kMaxIn = 8;       // array inputs of one program
constexpr int kMaxOut = 8;      // outputs of one program
constexpr int kMaxScal = 32;    // scalar table: dynamic scalars and immediates
constexpr int kMaxCode = 48;    // instructions
constexpr int kSlots = 32;      // value slots a program may name (kernels hold 16 or 32)
constexpr int kVec = 4;         // elements handled per lane and interpreted instruction

// device dtypes of loads / stores
enum : uint32_t { kF32 = 0, kBF16 = 1, kI32 = 2, kI64 = 3 };

// how an input is addressed from the flat index i of the iteration space [rows, cols]
enum : uint32_t {
  kFull = 0,     // element i
  kRowVec = 1,   // element i % cols   (a vector broadcast along rows, e.g. a bias)
  kColVec = 2,   // element i / cols   (one value per row)
  kScalar = 3,   // element 0
  kStrided = 4   // sum_k coord_k(i) * stride[k] over the (<= 4-d) iteration space
};

// interpreter opcodes.  Unary ops come first: the interpreter reads operand b only for
// op >= kAdd.  Operand a is always a value slot; a scalar-table operand can only be b (or c of
// kFma), so non-commutative ops have a reversed form ("kRsub": b - a).
enum : uint32_t {
  kMov = 0, kNeg, kAbs, kExp, kLog, kTanh, kSqrt, kRsqrt, kRecip, kRelu, kGelu, kSquare,
  kSigmoid, kRoundBf16,
  kAdd, kSub, kRsub, kMul, kDiv, kRdiv, kMax, kMin,
  kReluGrad,     // b > 0 ? a : 0     (a = dy, b = x)
  kRreluGrad,    // a > 0 ? b : 0
  kGeluGrad,     // a * gelu'(b)
  kRgeluGrad,    // b * gelu'(a)
  kFma,          // a*b + c
  kSplat,        // b (a scalar-table entry) replicated
  kNumOps
};

// instruction word: op[7:0] dst[12:8] a[18:13] b[24:19] c[30:25];
// operand < 32: value slot; operand >= 32: scal[operand - 32]
inline uint32_t encode(uint32_t op, uint32_t dst, uint32_t a, uint32_t b = 0, uint32_t c = 0) {
  return op | (dst << 8) | (a << 13) | (b << 19) | (c << 25);
}

// how the kernels fetch an input on their fast path (full 4-vectors)
enum : uint32_t {
  kFetchVec4 = 0,   // one 16-byte (8-byte for bf16) load of four consecutive elements
  kFetchBcast = 1,  // one element, replicated to the four lanes
  kFetchSlow = 2    // element by element through the general addressing code
};

struct EwIn {
  const void* ptr;
  uint32_t mode;
  uint32_t dtype;
  uint32_t fetch;      // kFetch*: decided by the host from mode, cols and alignment
  uint32_t pad;
  int64_t stride[4];   // kStrided only, in elements
};

struct EwOut {
  void* ptr;
  uint32_t dtype;
  uint32_t slot;       // value slot stored
  uint32_t scalar;     // 1: a rank-0 result, written once (by flat index 0)
  uint32_t pad;
};

struct EwProg {
  uint32_t n_in, n_out, n_code, anchor_slot;  // anchor_slot: where a reduction / GEMM result enters
  uint32_t vec_ok;     // 1: cols % 4 == 0, so a 4-vector never straddles a row
  uint32_t full_vec_ok;  // 1: every 4-vector of the flat space starts at a multiple of 4
  uint32_t cols;       // last dimension of the iteration space (>= 1)
  uint32_t n_slots;    // value slots the program uses (selects the 16- or 32-slot kernel)
  uint32_t needs_divmod;  // 1: some input is addressed by i / cols or i % cols
  uint32_t fast;       // 1: n % 4 == 0, every input fetches as vec4 / broadcast, outputs contiguous
  uint32_t all_f32;    // 1: every input and output is fp32
  uint32_t pad2;
  uint64_t n;          // elements of the iteration space
  uint32_t dims[4];    // iteration space collapsed to 4 dims (kStrided addressing)
  EwIn in[kMaxIn];
  EwOut out[kMaxOut];
  float scal[kMaxScal];
  uint32_t code[kMaxCode];
};

// ---- elementwise region -----------------------------------------------------------
struct EwArgs {
  EwProg prog;
};

// ---- reductions ---------------------------------------------------------------------
enum : uint32_t { kRedSum = 0, kRedMax = 1, kRedMean = 2 };

// row reduction: out[r] = post(reduce_c pro(x[r, c]))
struct RowArgs {
  EwProg pro;          // iteration space [rows, cols]; its result is slot pro.anchor_slot
  EwProg post;         // iteration space [rows]
  uint32_t rows, cols, red, threads_per_row;
  // filled in by launch_row_reduce for the streamed variant: input numbers of the (up to two) fp32
  // inputs read in full and of the (up to one) fp32 vector broadcast along rows; counts
  uint32_t vin[2], rin, n_vin, n_rin, pad;
};

// global reduction, single launch: per-workgroup partials, the last workgroup to finish
// combines them, then runs the post program (scalar epilogue and optional finaliser)
struct AllArgs {
  EwProg pro;          // iteration space = the reduced tensor, flat
  EwProg post;         // iteration space: 1 element, or the finaliser's shape
  float* partials;     // [gridDim.x]
  uint32_t* ticket;    // zero before launch; reset by the kernel
  uint32_t red, pad;
  uint64_t count;      // elements reduced (for mean)
};

// column reduction over axis 0 of [rows, cols]
struct ColArgs {
  EwProg pro;          // iteration space [rows, cols]
  EwProg post;         // iteration space [cols]
  float* partials;     // [gridDim.y, cols]
  uint32_t* tickets;   // [gridDim.x], zero before launch; reset by the kernel
  uint32_t rows, cols, red;
  uint32_t narrow;     // set by launch_col_reduce: at most 64 columns and 65536 elements, one workgroup (see the kernel)
  // filled in by launch_col_reduce for the streamed variants (by the lowering if norm_grad): input
  // numbers of the (up to two) inputs read in full and of the (up to two) per-row inputs (kColVec),
  // padded with the first
  uint32_t vin[2], cin[2];
  // 1: the program is input vin[0] * ((input vin[1] - input cin[0]) * input cin[1]), a layer norm's
  // weight gradient before its sum, and is not interpreted
  uint32_t norm_grad;
  // 1 (with norm_grad and a sum): the column sums of input vin[0] (the norm's bias gradient) ride along;
  // their partials follow the others', post2 runs on them
  uint32_t sum2;
  EwProg post2;        // iteration space [cols]
  // Not null: the launch that computed the norm's gradient, or a contraction that reads the summed tensor, has left
  // `parts_rows` partial sums of every column here (rows of [1 + sum2][cols] floats: a norm's weight gradient's, then its
  // bias gradient's), and this one only adds them up.
  const float* parts;
  uint32_t parts_rows, pad;
};

// ---- row operators with a fixed body ---------------------------------------------------
enum : uint32_t { kSoftmax = 0, kSoftmaxGrad, kLayerNorm, kLayerNormGrad, kXent, kXentGrad };

struct RowOpArgs {
  uint32_t op, rows, cols, threads_per_row;
  const void* in[5];
  uint32_t in_dtype[5];
  void* out[3];        // (out[1] of xent_grad: null, or the losses, which ride along)
  uint32_t out_dtype[3];
  float eps;           // layer norm
  float scale;         // xent_grad
  // layer_norm_grad: column sums that ride along (0 none, 1 of dy * xhat, 2 of dy as well); col_rows workgroups leave theirs in
  // col_parts, a row of [col_sums][cols] floats each (ColArgs::parts)
  uint32_t col_sums, col_rows;
  float* col_parts;
  // xent and xent_grad: the sum or mean (kRedSum, kRedMean) of the losses goes to `total` as well; the workgroups exchange
  // theirs through total_parts[gridDim.x] and the ticket (zero before the launch; reset by the kernel)
  uint32_t has_total, total_red;
  float* total;
  float* total_parts;
  uint32_t* total_ticket;
};

// ---- contraction ------------------------------------------------------------------------
// C[b] = post(A[b] * B[b]); A is M x K, B is K x N, element (i, j) of an operand is at
// base + b0*sb0 + b1*sb1 + i*s_row + j*s_col (element strides), so transposes, batched
// operands and head-split layouts are all addressing, never copies.
struct GemmOperand {
  const void* ptr;
  int64_t s_row, s_col, s_b0, s_b1;
};

//
// A post program that is a chain -- one running value per element, each step combining it with nothing, a scalar
// or an input, results stored on the way -- is also laid out as such.  The epilogues then evaluate it with the
// running values in registers the compiler has numbered: no slot is looked up, copied out or copied back, and
// 32 elements of a lane share the decoding of a step.
constexpr int kMaxChain = 8;
enum : uint32_t { kSrcNone = 0, kSrcScal, kSrcRow0, kSrcRow1, kSrcFull0, kSrcFull1 };
constexpr uint32_t kNoOut = 0xff;
// step word: op[7:0] src[11:8] scal[19:12] out[27:20].  With v the running value, s the source and c the scalar: an op's
// first operand is v, its second s, and its reversed form takes them the other way round; kFma: v * c + s, kRfma: s * c + v.
constexpr uint32_t kRfma = kNumOps;
struct Chain {
  uint32_t n;                  // steps + 1; 0: the program is no chain
  uint32_t n_row, n_full;      // inputs addressed by column, inputs addressed like the output (up to two of each),
  uint32_t row[2], full[2];    // their input numbers
  uint32_t first_out;          // the output that is the product itself, or kNoOut
  uint32_t step[kMaxChain];    // out: the output that is the running value after the step, or kNoOut
};

struct GemmArgs {
  GemmOperand a, b;
  uint32_t m, n, k;
  uint32_t batch0, batch1;   // batch = batch0 * batch1 (b = b0 * batch1 + b1)
  uint32_t in_dtype;         // kF32 or kBF16 (both operands)
  uint32_t tiles_m, tiles_n;
  // where output element (b0, b1, row, col) goes: b0*o_b0 + b1*o_b1 + row*o_row + col (elements).
  // Contiguous [batch, m, n] by default; a permuted layout when the product's only reader is a
  // permutation (head merge), which then costs nothing.
  int64_t o_b0, o_b1, o_row;
  // Split-K (the LDS-staged kernels): `splits` workgroups share an output tile, each contracting a
  // slice of k and leaving its fp32 partial product, row major, in split_ws[split]; the post
  // program then runs in a second launch (SplitPostArgs) that adds the partials up in split order.
  // With splits = 1 and split_ws set the product goes there as it is, for the second launch.
  // Workgroup tile: bf16 128 x 128 or 128 x 64; fp32 128 x 128 or 64 x 64, and for direct = 1, the one-launch
  // kernel for small products, 16 x 16, 16 x 64, 32 x 32 or 64 x 32.
  // halves = 2 (the LDS-staged kernels): a workgroup of twice the size, each half of it contracting half of the
  // workgroup's k; the two products meet in LDS.
  uint32_t splits, tile_m, tile_n, halves;
  uint32_t direct;
  float* split_ws;           // [splits][batch * m * n] floats
  // The one-launch small kernel (direct = 1) with splits > 1: `splits` workgroups share a tile;
  // split_ws then holds [tile][split][tile_m x tile_n] partial tiles and tickets[tile]
  // counts the workgroups that have left theirs (zero before the launch; the last one adds the
  // partials up in split order, runs the post program and resets the ticket).
  uint32_t* tickets;
  EwProg post;               // iteration space = the output
  // post as a chain, for the LDS-staged kernels: every input and output has the operands' type, columns come in
  // whole 16-byte chunks
  Chain chain;
  // The one-launch small kernel can carry the column sums of its B operand ([k, n], rows
  // contiguous) along: a weight gradient x^T dy and the bias gradient sum_rows(dy) read the same
  // dy.  col_sum = 1: the workgroups of the first tile row add up the columns of B they fetch
  // anyway (col_red: kRedSum or kRedMean) and run col_post on them, iteration space [n].
  // The LDS-staged kernels do so too where A is [k, m] and B [k, n], rows contiguous, in an unbatched product (bf16: tiles of 128
  // columns).  With col_parts set (k splits; n a multiple of four) each split leaves its sums there, [splits][n], for
  // ColArgs::parts, and col_post is not used.
  uint32_t col_sum, col_red;
  float* col_parts;
  EwProg col_post;
};

// second launch of a split-K contraction: anchor = sum over splits of ws[split][i], then the
// contraction's post program over the flat output, exactly like an elementwise region
struct SplitPostArgs {
  EwProg prog;
  const float* ws;
  uint32_t splits, pad;
  uint64_t stride;           // floats between consecutive splits (= elements of the output)
};

// ---- attention core ------------------------------------------------------------------------
// o = softmax(q k^T) v over batch0 x batch1 heads, q and o [sq, d], k and v [sk, d], and its gradients
// for dy [sq, d].  Rows contiguous (s_col = 1), any row and head strides.
enum : uint32_t { kAttnForward = 0, kAttnDq, kAttnDkv };

struct AttnArgs {
  uint32_t pass, dtype, d, sq, sk, batch0, batch1, pad;
  // q is taken as q * q_scale, rounded to its type; dq, rounded, is stored times dq_scale
  float q_scale, dq_scale;
  GemmOperand q, k, v, o, dy;
  GemmOperand dq, dk, dv;
  // [3][batch0 * batch1 * sq]: row maxima and reciprocal row sums (written by the forward pass unless
  // null), row sums of p * (dy v^T) (written by kAttnDq, read by kAttnDkv)
  float* stats;
};

// ---- window update -------------------------------------------------------------------------
// out = base with the window [start, start + len) along one axis replaced by upd.  The tensors are
// seen as [outer, dim, inner] (base, out) and [outer, len, inner] (upd), dense.  window_only: out
// is base's own buffer (updated in place), so only the window is written.
struct SliceArgs {
  const void* base;
  const void* upd;
  void* out;
  uint64_t n;              // elements this launch walks: the window (window_only) or all of out
  uint64_t dim, inner, start, len;
  uint32_t elem_bytes;     // 2, 4 or 8
  uint32_t window_only;
};

// Argument blocks travel by value in the kernel argument segment, which holds 4 KiB.
static_assert(sizeof(EwArgs) <= 4096 && sizeof(RowArgs) <= 4096 && sizeof(AllArgs) <= 4096 && sizeof(ColArgs) <= 4096 &&
                  sizeof(GemmArgs) <= 4096 && sizeof(SplitPostArgs) <= 4096 && sizeof(SliceArgs) <= 4096 &&
                  sizeof(AttnArgs) <= 4096,
              "a kernel's argument block must fit the kernel argument segment");

}  // namespace ltk
#endif  // LT_KERNELS_H_

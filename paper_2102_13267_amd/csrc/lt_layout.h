// Programs laid out for the kernels that evaluate them with their values in fixed registers (Chain, lt_kernels.h):
// host side, no device code.
#ifndef LT_LAYOUT_H_
#define LT_LAYOUT_H_

#include "lt_kernels.h"

namespace ltk {

// The opcode that does the same with its operands exchanged (two-operand instructions).
inline uint32_t reversed_op(uint32_t op) {
  switch (op) {
    case kAdd: case kMul: case kMax: case kMin: return op;
    case kSub: return kRsub;
    case kRsub: return kSub;
    case kDiv: return kRdiv;
    case kRdiv: return kDiv;
    case kReluGrad: return kRreluGrad;
    case kRreluGrad: return kReluGrad;
    case kGeluGrad: return kRgeluGrad;
    default: return kGeluGrad;   // kRgeluGrad
  }
}

// The post program of a contraction as a chain (Chain), where it is one: every instruction takes the running
// value and at most one input or scalar besides, nothing reads an earlier value again, and every result is the
// running value at some step.  Inputs are whole 16-byte chunks of the operands' type, read like the output
// or by column; operations are those of one or a few instructions and GELU (what a chain kernel unrolls 32
// times).  Everything else stays with the interpreter.
inline void make_chain(GemmArgs* a) {
  const EwProg& p = a->post;
  Chain& ch = a->chain;
  ch = Chain{};
  const int64_t w = a->in_dtype == kBF16 ? 8 : 4;
  if (a->n % w || a->o_row % w || a->o_b0 % w || a->o_b1 % w || p.n_out == 0u || p.n_code > (uint32_t)kMaxChain) return;
  for (uint32_t i = 0; i < p.n_in; ++i)
    if (p.in[i].dtype != a->in_dtype || p.in[i].fetch != kFetchVec4 || (p.in[i].mode != kFull && p.in[i].mode != kRowVec)) return;
  for (uint32_t o = 0; o < p.n_out; ++o)
    if (p.out[o].dtype != a->in_dtype || p.out[o].scalar) return;
  // what a slot holds: nothing, an input, a scalar, or the running value after so many steps
  enum { NONE, INPUT, SCAL, VALUE };
  struct Held { int kind; uint32_t i; };
  Held slot[kSlots];
  for (Held& h : slot) h = Held{NONE, 0};
  for (uint32_t i = 0; i < p.n_in; ++i) slot[i] = Held{INPUT, i};
  slot[p.anchor_slot] = Held{VALUE, 0};
  uint32_t steps = 0;
  auto operand = [&](uint32_t x) { return x < 32u ? slot[x] : Held{SCAL, x - 32u}; };
  auto running = [&](const Held& h) { return h.kind == VALUE && h.i == steps; };
  // the source code of an input or scalar (kSrcNone: neither)
  auto source = [&](const Held& h) -> uint32_t {
    if (h.kind == SCAL) return kSrcScal;
    if (h.kind != INPUT) return kSrcNone;
    const bool r = p.in[h.i].mode == kRowVec;
    uint32_t* list = r ? ch.row : ch.full;
    uint32_t& n = r ? ch.n_row : ch.n_full;
    uint32_t at = 0;
    while (at < n && list[at] != h.i) ++at;
    if (at == 2u) return kSrcNone;
    if (at == n) list[n++] = h.i;
    return (r ? kSrcRow0 : kSrcFull0) + at;
  };
  for (uint32_t pc = 0; pc < p.n_code; ++pc) {
    const uint32_t word = p.code[pc], d = (word >> 8) & 31u;
    uint32_t op = word & 0xffu, src = kSrcNone, sc = 0;
    const Held A = operand((word >> 13) & 63u), B = operand((word >> 19) & 63u), C = operand((word >> 25) & 63u);
    if (op == kSplat) {
      if (B.kind != SCAL) return;
      slot[d] = B;
      continue;
    }
    if (op == kMov) {
      slot[d] = A;
      continue;
    }
    if (op == kExp || op == kLog || op == kTanh || op == kSigmoid) return;
    if (op == kFma) {
      if (B.kind != SCAL) return;
      sc = B.i;
      if (running(A) && C.kind == INPUT) src = source(C);
      else if (running(C) && A.kind == INPUT) src = source(A), op = kRfma;
      if (src == kSrcNone) return;
    } else if (op < kAdd) {
      if (!running(A)) return;
    } else {
      const Held* s = nullptr;
      if (running(A) && !running(B)) s = &B;
      else if (running(B) && !running(A)) s = &A, op = reversed_op(op);
      if (!s || (src = source(*s)) == kSrcNone) return;
      if (src == kSrcScal) sc = s->i;
    }
    ch.step[steps++] = op | (src << 8) | (sc << 12) | (kNoOut << 20);
    slot[d] = Held{VALUE, steps};
  }
  ch.first_out = kNoOut;
  for (uint32_t o = 0; o < p.n_out; ++o) {
    const Held h = slot[p.out[o].slot];
    if (h.kind != VALUE) return;
    if (h.i == 0u) {
      if (ch.first_out != kNoOut) return;
      ch.first_out = o;
    } else {
      uint32_t& s = ch.step[h.i - 1u];
      if (((s >> 20) & 0xffu) != kNoOut) return;
      s = (s & ~(0xffu << 20)) | (o << 20);
    }
  }
  ch.n = steps + 1u;
}

}  // namespace ltk
#endif  // LT_LAYOUT_H_

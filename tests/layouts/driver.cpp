// Random programs, evaluated as the interpreter does and from their layouts (lt_layout.h), value by value.
#include <cmath>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <random>
#include <vector>

#include "../../paper_2102_13267_amd/csrc/lt_layout.h"

using namespace ltk;

static float unary(uint32_t op, float x) {
  switch (op) {
    case kNeg: return -x;
    case kAbs: return std::fabs(x);
    case kExp: return std::exp(std::fmin(x, 3.0f));
    case kLog: return std::log(std::fabs(x) + 1.0f);
    case kTanh: return std::tanh(x);
    case kSqrt: return std::sqrt(std::fabs(x));
    case kRsqrt: return 1.0f / std::sqrt(std::fabs(x) + 1.0f);
    case kRecip: return 1.0f / (std::fabs(x) + 1.0f);
    case kRelu: return x > 0 ? x : 0;
    case kGelu: return 0.5f * x;
    case kSquare: return x * x;
    case kSigmoid: return 1.0f / (1.0f + std::exp(-x));
    default: return x;   // kMov, kRoundBf16
  }
}
static float binary(uint32_t op, float a, float b) {
  switch (op) {
    case kAdd: return a + b;
    case kSub: return a - b;
    case kRsub: return b - a;
    case kMul: return a * b;
    case kDiv: return a / (b * b + 1);
    case kRdiv: return b / (a * a + 1);
    case kMax: return a > b || (a == b && !std::signbit(a)) ? a : b;
    case kMin: return a < b || (a == b && std::signbit(a)) ? a : b;
    case kReluGrad: return b > 0 ? a : 0;
    case kRreluGrad: return a > 0 ? b : 0;
    case kGeluGrad: return a * 0.5f + b * 0.25f;
    default: return b * 0.5f + a * 0.25f;   // kRgeluGrad
  }
}
// One element through the program as written; slots hold what they hold.
static void run(const EwProg& p, const std::vector<float>& in, float anchor, float* slot) {
  for (uint32_t i = 0; i < p.n_in; ++i) slot[i] = in[i];
  slot[p.anchor_slot] = anchor;
  for (uint32_t pc = 0; pc < p.n_code; ++pc) {
    const uint32_t w = p.code[pc], op = w & 0xff, d = (w >> 8) & 31;
    auto val = [&](uint32_t x) { return x < 32 ? slot[x] : p.scal[x - 32]; };
    const uint32_t a = (w >> 13) & 63, b = (w >> 19) & 63, c = (w >> 25) & 63;
    if (op == kSplat) slot[d] = val(b);
    else if (op == kFma) slot[d] = std::fma(val(a), val(b), val(c));
    else if (op >= kAdd) slot[d] = binary(op, val(a), val(b));
    else slot[d] = unary(op, val(a));
  }
}
static float step(uint32_t op, float v, float s, float sc) {
  if (op == kFma) return std::fma(v, sc, s);
  if (op == kRfma) return std::fma(s, sc, v);
  return op >= kAdd ? binary(op, v, s) : unary(op, v);
}
static bool same(float a, float b) { return std::memcmp(&a, &b, 4) == 0 || (a != a && b != b); }

// Instructions over slots below 8; operands are slots that hold something (mostly the latest) or scalars.
static EwProg program(std::mt19937& g, uint32_t n_in, uint32_t n_code) {
  EwProg p;
  std::memset(&p, 0, sizeof(p));
  p.n_in = n_in;
  p.n_code = n_code;
  auto rnd = [&](uint32_t n) { return (uint32_t)(g() % n); };
  for (int i = 0; i < kMaxScal; ++i) p.scal[i] = (float)rnd(1000) / 250.0f - 2.0f;
  std::vector<uint32_t> live;
  for (uint32_t i = 0; i < n_in; ++i) live.push_back(i);
  live.push_back(p.anchor_slot = n_in);
  uint32_t last = live.back();
  for (uint32_t pc = 0; pc < n_code; ++pc) {
    auto slot = [&]() { return rnd(3) ? last : live[rnd((uint32_t)live.size())]; };
    const uint32_t d = rnd(8);
    uint32_t op = rnd(kNumOps), a = slot(), b = rnd(4) == 0 ? 32 + rnd(kMaxScal) : slot(), c = slot();
    if (op == kSplat && rnd(4)) op = kAdd;
    if (op == kSplat) b = 32 + rnd(kMaxScal);
    if (op == kFma && rnd(8)) b = 32 + rnd(kMaxScal);
    p.code[pc] = encode(op, d, a, b, c);
    bool known = false;
    for (uint32_t s : live) known |= s == d;
    if (!known) live.push_back(d);
    last = d;
  }
  p.n_slots = 8;
  return p;
}

int main() {
  std::mt19937 g(12345);
  int chains = 0;
  for (int it = 0; it < 200000; ++it) {
    // a contraction's post program; its outputs are slots that hold something when it ends
    GemmArgs q;
    std::memset(&q, 0, sizeof(q));
    const uint32_t m_in = g() % 4;
    q.post = program(g, m_in, g() % 6);
    q.in_dtype = kF32;
    q.n = 8;
    q.o_row = 8;
    std::vector<uint32_t> held;
    for (uint32_t i = 0; i <= m_in; ++i) held.push_back(i);
    for (uint32_t pc = 0; pc < q.post.n_code; ++pc) held.push_back((q.post.code[pc] >> 8) & 31);
    q.post.n_out = 1 + g() % 2;
    for (uint32_t o = 0; o < q.post.n_out; ++o) q.post.out[o].slot = o == 0 ? held.back() : held[g() % held.size()];
    for (uint32_t k = 0; k < m_in; ++k) q.post.in[k].mode = g() % 2 ? kFull : kRowVec;
    make_chain(&q);
    if (!q.chain.n) continue;
    ++chains;
    std::vector<float> in;
    for (uint32_t k = 0; k < m_in; ++k) in.push_back((float)(g() % 2000) / 500.0f - 2.0f);
    const float product = (float)(g() % 2000) / 500.0f - 2.0f;
    float slot[32] = {0}, out[kMaxOut];
    run(q.post, in, product, slot);
    for (float& o : out) o = NAN;
    float v = product;
    if (q.chain.first_out != kNoOut) out[q.chain.first_out] = v;
    for (uint32_t s = 0; s + 1 < q.chain.n; ++s) {
      const uint32_t w = q.chain.step[s], src = (w >> 8) & 15, o = (w >> 20) & 0xff;
      const float sc = q.post.scal[(w >> 12) & 31];
      const float y = src == kSrcFull0 ? in[q.chain.full[0]] : src == kSrcFull1 ? in[q.chain.full[1]] : src == kSrcRow0 ? in[q.chain.row[0]] : src == kSrcRow1 ? in[q.chain.row[1]] : sc;
      v = step(w & 0xff, v, y, sc);
      if (o != kNoOut) out[o] = v;
    }
    for (uint32_t o = 0; o < q.post.n_out; ++o)
      if (!same(out[o], slot[q.post.out[o].slot])) return std::printf("chain of program %d: %g, interpreted %g\n", it, out[o], slot[q.post.out[o].slot]), 1;
  }
  std::printf("%d chains\n", chains);
  return chains > 10000 ? 0 : 1;
}

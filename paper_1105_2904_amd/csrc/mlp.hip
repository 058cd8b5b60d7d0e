// Inference and training kernels of the near-contact closure network
// (mlp_core.h) behind the C ABI of include/lbm.h.
//
//   k_mlp_forward  persistent grid, one 16-sample tile per wave at a time,
//                  weights staged once per workgroup in LDS.
//   k_mlp_train    one workgroup of sixteen waves, a loop over Adam steps:
//                  each wave takes a 16-sample tile of the mini-batch through
//                  forward, loss and backward, then owns one 16 x 16 tile of
//                  the weight gradients, contracted over every sample of the
//                  batch, and the Adam state of those weights.
//   k_mlp_grad     the same pass without the update, on as many workgroups
//                  as the rows fill; k_mlp_grad_sum adds their sums in a
//                  fixed order.
// Loss over B rows: L = (1/B) sum_rows sum_o (y - t)^2.  The backward signals
// are multiplied by the loss scale S before their FP16 rounding and the
// weight gradients divided by S again, in FP32.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstdint>

#include "lbm.h"
#include "mlp_core.h"

namespace {

using mlp::f4;
using mlp::h4;

constexpr int kWaves = 4;

// Bound by its vector instructions: per 16-row tile 32 tanh a lane, each an
// exponential, a reciprocal and four ordinary operations, against 24 MFMAs and
// 640 bytes.  So everything else is kept off the vector unit: the weight
// operands and biases stay in registers, and the tile index and with it every
// address and bound in scalar ones.  The launch bound leaves the compiler 168
// registers a lane, of which it takes 119 (four waves a SIMD all the same);
// bound to 128 it put the products in accumulators, one more move each before
// the tanh.  4,194,304 rows: 179 -> 160 us (253 TFLOP/s of the products).
__global__ __launch_bounds__(256, 3) void k_mlp_forward(const float* __restrict__ P, const float* __restrict__ X,
                                                        float* __restrict__ Y, int64_t n) {
  __shared__ mlp::Weights w;
  const int tid = threadIdx.x, lane = tid & 63, wv = __builtin_amdgcn_readfirstlane(tid >> 6);
  mlp::load_weights(w, P, tid, 256);
  __syncthreads();
  const int r = lane & 15, g = lane >> 4;
  h4 w1[4], w2[4][4], w3[4];
  float b1[4][4], b2[4][4];
#pragma unroll
  for (int mt = 0; mt < 4; mt++) {
    w1[mt] = mlp::ld4(&w.w1t[16 * mt + r][4 * g]);
    w3[mt] = mlp::ld4(&w.w3t[r][16 * mt + 4 * g]);
#pragma unroll
    for (int kt = 0; kt < 4; kt++) w2[mt][kt] = mlp::ld4(&w.w2t[16 * mt + r][16 * kt + 4 * g]);
#pragma unroll
    for (int i = 0; i < 4; i++) {
      b1[mt][i] = w.b1[16 * mt + 4 * g + i];
      b2[mt][i] = w.b2[16 * mt + 4 * g + i];
    }
  }
  const float b30 = w.b3[0], b31 = w.b3[1];
  // one tile: lane (r, g < 2) holds inputs 4g .. 4g+3 of row 16 t + r
  auto tile = [&](f4 xc) {
    h4 xb, h1[4], h2[4];
#pragma unroll
    for (int i = 0; i < 4; i++) xb[i] = (_Float16)xc[i];
    const f4 zero = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int mt = 0; mt < 4; mt++) {
      const f4 acc = mlp::mma(w1[mt], xb, zero);
#pragma unroll
      for (int i = 0; i < 4; i++) h1[mt][i] = (_Float16)mlp::tanh_fast(acc[i] + b1[mt][i]);
    }
#pragma unroll
    for (int mt = 0; mt < 4; mt++) {
      f4 acc = zero;
#pragma unroll
      for (int kt = 0; kt < 4; kt++) acc = mlp::mma(w2[mt][kt], h1[kt], acc);
#pragma unroll
      for (int i = 0; i < 4; i++) h2[mt][i] = (_Float16)mlp::tanh_fast(acc[i] + b2[mt][i]);
    }
    f4 y = zero;
#pragma unroll
    for (int kt = 0; kt < 4; kt++) y = mlp::mma(w3[kt], h2[kt], y);
    return y;
  };
  // whole tiles, the next one's inputs loaded while this one runs
  const int64_t whole = n / 16;
  const int64_t stride = (int64_t)gridDim.x * kWaves;
  const int xoff = r * mlp::kIn + 4 * g, yoff = r * mlp::kOut;
  int64_t t = (int64_t)blockIdx.x * kWaves + wv;
  f4 xn = {0.f, 0.f, 0.f, 0.f};  // stays zero where g >= 2
  if (t < whole && g < 2) xn = *(const f4*)(X + t * 16 * mlp::kIn + xoff);
  for (; t < whole; t += stride) {
    const f4 xc = xn;
    if (t + stride < whole && g < 2) xn = *(const f4*)(X + (t + stride) * 16 * mlp::kIn + xoff);
    const f4 y = tile(xc);
    if (g == 0) {
      float* const out = Y + t * 16 * mlp::kOut;
      out[yoff] = y[0] + b30;
      out[yoff + 1] = y[1] + b31;
    }
  }
  // the rows past the last whole tile, in the wave whose turn it is
  if (t == whole && n % 16 != 0) {
    const bool has = r < (int)(n % 16);
    f4 xc = {0.f, 0.f, 0.f, 0.f};
    if (has && g < 2) xc = *(const f4*)(X + whole * 16 * mlp::kIn + xoff);
    const f4 y = tile(xc);
    if (has && g == 0) {
      float* const out = Y + whole * 16 * mlp::kOut;
      out[yoff] = y[0] + b30;
      out[yoff + 1] = y[1] + b31;
    }
  }
}

// ---------------------------------------------------------------------------
// Gradient pass: kTiles waves, one 16-sample tile each, then one output tile
// of the weight gradients each.
//
// Bound: the latency of one CU's dependent phases, not its units.  With four
// waves, each holding every weight-gradient tile and adding them to a shared
// sum one wave after the other, a step of 256 rows took 56 us; sixteen waves
// (four per SIMD) hide the tanh and LDS latencies of each other, and a wave
// that owns an output tile needs no cross-wave sum at all.  The activations
// and backward signals of every tile pass through LDS once, transposed there
// into the operand order of the gradient products (the samples are the
// contraction).  500 steps of 256 rows: 28.4 -> 5.0 ms (9.9 us a step: about
// 14k cycles of tiles, 4k of products, 5k of Adam); the gradient of 44,672
// rows on 233 workgroups 4,982 -> 17.4 us.
// ---------------------------------------------------------------------------
constexpr int kTiles = 16;              // tiles of a pass, and waves of the workgroup
constexpr int kTrainThreads = 64 * kTiles;
constexpr int kChains = 4;              // partial sums per output: tile t adds to chain t % kChains

// One tile's part in the gradient products.  Activations and signals lie as
// their lanes hold them, [sample][4 consecutive features], and are read back
// with the LDS unit's transposing loads as [feature][4 consecutive samples]:
// one 8-byte write per lane and 16 features, where writes already transposed
// were four of 2 bytes (a training step of 256 rows 11.5 -> 10.4 us).  A sample's
// quads of features trade places (at_quad) so that neither side meets a bank
// conflict: a write takes one quad of each of 16 samples, a read four quads of
// each of four.
struct TileSignals {
  h4 h1[16][mlp::kHid / 4], h2[16][mlp::kHid / 4];  // hidden activations
  h4 g1[16][mlp::kHid / 4], g2[16][mlp::kHid / 4];  // dL/dz1, dL/dz2 (scaled by S)
  _Float16 x[mlp::kIn][16];                         // inputs, [feature][sample]
  _Float16 gy[mlp::kOut][16];                       // dL/dy (scaled by S)
  float e[mlp::kOut][16];                           // y - t
};
struct TrainShared {
  mlp::Weights w;
  TileSignals t[kTiles];
};
static_assert(sizeof(TrainShared) <= 160 * 1024, "one workgroup's LDS");

// Place of feature quad q in sample s's row.
__device__ __forceinline__ int at_quad(int s, int q) { return q ^ (4 * ((s >> 1) & 3) + 2 * (s >> 3)); }

// A tile in accumulator layout (lane l: features 16 mt + 4 (l/16) + i of sample l%16).
__device__ __forceinline__ void put_tile(h4 (*dst)[mlp::kHid / 4], int mt, h4 v, int lane) {
  const int r = lane & 15, g = lane >> 4;
  dst[r][at_quad(r, 4 * mt + g)] = v;
}
// A transposing read: the lanes of each 16-lane group read 16 quads, lane c the
// one at src; lane m gets element m%4 of the quads read by lanes m/4, 4 + m/4,
// 8 + m/4 and 12 + m/4.
__device__ __forceinline__ h4 read_transposed(const h4* src) {
  typedef short s4 __attribute__((ext_vector_type(4)));
  typedef __attribute__((address_space(3))) s4 lds4;
  return __builtin_bit_cast(h4, __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds4*)src));
}
// What lane l reads (as an index into an array's quads) so that it gets
// features 16 mt + l%16 of samples 4 (l/16) .. + 3, an operand of the products
// over samples.
__device__ __forceinline__ int operand_quad(int mt, int lane) {
  const int s = 4 * (lane >> 4) + ((lane & 15) >> 2);
  return s * (mlp::kHid / 4) + at_quad(s, 4 * mt + (lane & 3));
}
// And so that it gets feature 4 q + l%4 of samples 4 ((l/4)%4) .. + 3.
__device__ __forceinline__ int bias_quad(int q, int lane) {
  const int s = 4 * (lane & 3) + ((lane & 15) >> 2);
  return s * (mlp::kHid / 4) + at_quad(s, q);
}

// The inputs and targets of one tile's rows as the lanes of its wave hold
// them: features 4g .. 4g+3 (g < 2) and, at g = 0, the targets of row `row`.
struct TileRows {
  f4 x;
  float t[2];
};
__device__ __forceinline__ TileRows load_rows(const float* __restrict__ X, const float* __restrict__ T, int64_t row,
                                              bool valid, int lane) {
  const int g = lane >> 4;
  TileRows v = {{0.f, 0.f, 0.f, 0.f}, {0.f, 0.f}};
  if (valid && g < 2) {
    const float* p = X + row * mlp::kIn + 4 * g;
    v.x = f4{p[0], p[1], p[2], p[3]};
  }
  if (valid && g == 0) {
    v.t[0] = T[row * mlp::kOut];
    v.t[1] = T[row * mlp::kOut + 1];
  }
  return v;
}

// a b rounded to FP16 once (a fused multiply-add to half precision; adding
// zero keeps the compiler from rounding the product to FP32 first).
__device__ __forceinline__ _Float16 half_product(float a, float b) { return (_Float16)__builtin_fmaf(a, b, 0.0f); }
// a b rounded to FP32 and then to FP16 (the empty statement keeps the compiler
// from fusing the two).  The error signals of the second layer are rounded this
// way where they feed the first layer's and once where they are summed: both
// are results of half an ulp, and a training run keeps its every bit only as
// long as each stays where it is.
__device__ __forceinline__ _Float16 float_product(float a, float b) {
  float p = a * b;
  asm volatile("" : "+v"(p));
  return (_Float16)p;
}

// v, of which the compiler knows nothing: what a loop derives from it (LDS
// addresses, above all) is computed there again and not kept in registers, of
// which sixteen waves leave each lane 128 (without it 33 loads and 9
// stores of spilled values in a training step, now 13 of each in the whole
// kernel: a step of 256 rows 10.3 -> 9.9 us, of 64 7.1 -> 5.6; the gradient
// spilled 24 and spills none now: 44,672 rows 21.3 -> 17.4 us, 512 14.1 -> 11.2).
// Batches of more than 256 rows, whose sums live across the tile phase, still
// spill 77 registers (512 rows 20.2 -> 19.8 us).
__device__ __forceinline__ int fresh(int v) {
  asm volatile("" : "+v"(v));
  return v;
}

// Forward, loss and backward of one tile; its signals to `ts`.
__device__ __forceinline__ void tile_signals(const mlp::Weights& w, TileSignals& ts, const TileRows& in, bool valid,
                                             float S, float Btot, int lane) {
  const int r = lane & 15, g = lane >> 4;
  h4 xb;
#pragma unroll
  for (int i = 0; i < 4; i++) xb[i] = (_Float16)in.x[i];
  h4 h1[4], h2[4];
  f4 y;
  mlp::forward_tile(w, xb, h1, h2, y, lane);
  // output error, scaled for the FP16 backward signals (lanes 0..15)
  h4 gy = {(_Float16)0.0f, (_Float16)0.0f, (_Float16)0.0f, (_Float16)0.0f};
  if (g == 0) {
#pragma unroll
    for (int i = 0; i < 2; i++) {
      const float e = valid ? y[i] + w.b3[i] - in.t[i] : 0.0f;
      if (valid) gy[i] = (_Float16)(S * 2.0f * e / Btot);
      ts.e[i][r] = e;
      ts.gy[i][r] = gy[i];
    }
  }
  if (g < 2) {
#pragma unroll
    for (int i = 0; i < 4; i++) ts.x[4 * g + i][r] = xb[i];
  }
#pragma unroll
  for (int mt = 0; mt < 4; mt++) {
    put_tile(ts.h1, mt, h1[mt], lane);
    put_tile(ts.h2, mt, h2[mt], lane);
  }
  __builtin_amdgcn_sched_barrier(0);
  // dL/dz2 = (W3 dL/dy) * (1 - h2^2),  dL/dz1 = (W2 dL/dz2) * (1 - h1^2)
  h4 gz2[4];
#pragma unroll
  for (int mt = 0; mt < 4; mt++) {
    f4 acc = {0.f, 0.f, 0.f, 0.f};
    acc = mlp::mma(mlp::ld4(&w.w3[16 * mt + r][4 * g]), gy, acc);
    h4 sum;
#pragma unroll
    for (int i = 0; i < 4; i++) {
      const float hv = (float)h2[mt][i];
      const float slope = 1.0f - hv * hv;
      gz2[mt][i] = float_product(acc[i], slope);
      sum[i] = half_product(acc[i], slope);
    }
    put_tile(ts.g2, mt, sum, lane);
    __builtin_amdgcn_sched_barrier(0);
  }
#pragma unroll
  for (int mt = 0; mt < 4; mt++) {
    f4 acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int kt = 0; kt < 4; kt++) acc = mlp::mma(mlp::ld4(&w.w2[16 * mt + r][16 * kt + 4 * g]), gz2[kt], acc);
    h4 gz1;
#pragma unroll
    for (int i = 0; i < 4; i++) {
      const float hv = (float)h1[mt][i];
      gz1[i] = half_product(acc[i], 1.0f - hv * hv);
    }
    put_tile(ts.g1, mt, gz1, lane);
    __builtin_amdgcn_sched_barrier(0);
  }
}

// The gradient sums one thread owns (scaled by S), in kChains partial sums
// each: a 16 x 16 tile of W2 per wave (f4 per lane), a tile of W1 in waves
// 0..3 and of W3 in waves 4..7, the bias sums and the loss.
struct GradSums {
  f4 w2[kChains], w13[kChains];
};
// Bias sums: lane = 16 chain + 4 quad + feature of a wave sums, over the tiles
// of its chain, samples 4 quad .. 4 quad + 3 of bias feature 64 layer +
// 4 wave + feature (layer 0: b1, layer 1: b2); wave 8 also b3 and the loss.
struct BiasSums {
  f4 b[2], b3;
  float loss[4];
};

__device__ __forceinline__ f4 widen(h4 v) { return f4{(float)v[0], (float)v[1], (float)v[2], (float)v[3]}; }

// Adds tiles 0 .. nt-1 of a pass (nt a multiple of kChains).  The loop over
// groups of tiles stays a loop: unrolled, the addresses of every tile, which
// lie past an LDS instruction's 64 KiB offset, were kept in registers.
__device__ __forceinline__ void add_tiles(const TrainShared& sh, int nt, int wv, int lane, GradSums& s, BiasSums& b) {
  const int r = lane & 15, g = lane >> 4;
  const int mt = wv >> 2, kt = wv & 3;
  const h4 zero = {(_Float16)0.0f, (_Float16)0.0f, (_Float16)0.0f, (_Float16)0.0f};
  const int qa = operand_quad(mt, lane), qb = operand_quad(kt, lane), qw = operand_quad(wv & 3, lane);
  const int ch = lane >> 4, q = (lane >> 2) & 3, fe = lane & 3;
  const int qf = bias_quad(wv, lane);
#pragma unroll 1
  for (int t0 = 0; t0 < nt; t0 += kChains) {
    const TileSignals* ts = sh.t + t0;
    const TileSignals& tb = ts[ch];
    const h4 b1 = read_transposed(&tb.g1[0][qf]), b2 = read_transposed(&tb.g2[0][qf]);
#pragma unroll
    for (int c = 0; c < kChains; c++)
      s.w2[c] = mlp::mma(read_transposed(&ts[c].g2[0][qa]), read_transposed(&ts[c].h1[0][qb]), s.w2[c]);
    if (wv < 4) {
#pragma unroll
      for (int c = 0; c < kChains; c++) {
        const h4 x = mlp::ld4(&ts[c].x[r & 7][4 * g]);
        s.w13[c] = mlp::mma(read_transposed(&ts[c].g1[0][qw]), r < mlp::kIn ? x : zero, s.w13[c]);
      }
    } else if (wv < 8) {
#pragma unroll
      for (int c = 0; c < kChains; c++) {
        const h4 gy = mlp::ld4(&ts[c].gy[r & 1][4 * g]);
        s.w13[c] = mlp::mma(r < mlp::kOut ? gy : zero, read_transposed(&ts[c].h2[0][qw]), s.w13[c]);
      }
    } else if (wv == 8) {
      b.b3 += widen(mlp::ld4(&tb.gy[fe & 1][4 * q]));  // features 0 and 1; the rest is not used
#pragma unroll
      for (int k = 0; k < 4; k++)
#pragma unroll
        for (int i = 0; i < mlp::kOut; i++) b.loss[k] += tb.e[i][4 * q + k] * tb.e[i][4 * q + k];
    }
    b.b[0] += widen(b1);
    b.b[1] += widen(b2);
  }
}

// The chains of one output added in order.
__device__ __forceinline__ float chain_sum(const f4 (&s)[kChains], int i) {
  float v = 0.f;
#pragma unroll
  for (int c = 0; c < kChains; c++) v += s[c][i];
  return v;
}
// Sum over the 16 samples (quads, then within the quad) and then over the
// chains in order, of a per-lane quad of sample sums; every lane of a feature
// gets it.
__device__ __forceinline__ float sample_sum(f4 v, int lane) {
#pragma unroll
  for (int o = 8; o > 2; o >>= 1)
#pragma unroll
    for (int k = 0; k < 4; k++) v[k] += __shfl_xor(v[k], o);
  const float s = (v[0] + v[2]) + (v[1] + v[3]);
  float tot = 0.f;
#pragma unroll
  for (int c = 0; c < kChains; c++) tot += __shfl(s, 16 * c + (lane & 15));
  return tot;
}

// Parameters a thread owns, as flat indices: W2[kr][4 consecutive columns]
// from w2; four consecutive columns of a W1 row (waves 0..3, r < 8) or the two
// columns of a W3 row (waves 4..7, g = 0) from w13, n13 of them; and one bias
// (b, -1 for none): in the lanes of chain 0, quad 0 of a feature holds its b1,
// quad 1 its b2, and in wave 8 quad 2 of the first two features b3 (lane =
// 16 chain + 4 quad + feature).
struct Owned {
  int w2, w13, n13, b;
};
__device__ __forceinline__ Owned owned_params(int wv, int lane) {
  const int r = lane & 15, g = lane >> 4;
  Owned o;
  o.w2 = mlp::oW2 + (16 * (wv & 3) + r) * mlp::kHid + 16 * (wv >> 2) + 4 * g;
  o.w13 = wv < 4 ? mlp::oW1 + r * mlp::kHid + 16 * wv + 4 * g : mlp::oW3 + (16 * (wv & 3) + r) * mlp::kOut;
  o.n13 = wv < 4 ? (r < mlp::kIn ? 4 : 0) : (wv < 8 && g == 0 ? mlp::kOut : 0);
  const int q = lane >> 2, fe = lane & 3;
  o.b = -1;
  if (lane < 16) {
    if (q == 0) o.b = mlp::oB1 + 4 * wv + fe;
    if (q == 1) o.b = mlp::oB2 + 4 * wv + fe;
    if (q == 2 && wv == 8 && fe < mlp::kOut) o.b = mlp::oB3 + fe;
  }
  return o;
}
// The sum of the bias a lane owns (see Owned; every lane of a feature holds
// all of its sums).
__device__ __forceinline__ float bias_sum(const BiasSums& bs, int wv, int lane) {
  const float s1 = sample_sum(bs.b[0], lane), s2 = sample_sum(bs.b[1], lane);
  const float s3 = wv == 8 ? sample_sum(bs.b3, lane) : 0.f;
  const int q = (lane >> 2) & 3;
  return q == 0 ? s1 : q == 1 ? s2 : s3;
}

__device__ __forceinline__ void clear(GradSums& s, BiasSums& b) {
  const f4 z = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int c = 0; c < kChains; c++) s.w2[c] = s.w13[c] = z;
  b.b[0] = b.b[1] = b.b3 = z;
#pragma unroll
  for (int k = 0; k < 4; k++) b.loss[k] = 0.f;
}

// x / d for a divisor shared by many: inv is 1/d correctly rounded, and one
// remainder step corrects the quotient (Markstein, IBM J. Res. Dev. 34, 1990),
// fewer instructions than a division.  From |x| = 2^-102 on that is the
// correctly rounded quotient, below (the remainder is subnormal) possibly its
// neighbour.  A quotient past the FP32 range has no remainder (infinity less
// infinity) and is returned as it stands, as a division gives it.
__device__ __forceinline__ float div_by(float x, float d, float inv) {
  const float q = x * inv;
  const float r = __builtin_fmaf(__builtin_fmaf(-q, d, x), inv, q);
  return __builtin_isinf(q) ? q : r;
}
// Constants of one Adam step (Kingma & Ba 2015): learning rate, the bias
// corrections and their reciprocals.
struct AdamStep {
  float lr, c1, c2, i1, i2;
};
// One FP32 master weight and its moments.
struct AdamState {
  float p, m, v;
};
__device__ __forceinline__ void adam(AdamState& a, float gk, const AdamStep& s) {
#pragma clang fp contract(off)
  a.m = __builtin_fmaf(0.9f, a.m, 0.1f * gk);
  a.v = __builtin_fmaf(0.999f, a.v, 0.001f * gk * gk);
  a.p = a.p - s.lr * div_by(a.m, s.c1, s.i1) / (sqrtf(div_by(a.v, s.c2, s.i2)) + 1e-8f);
}

__device__ __forceinline__ AdamState load_state(const float* P, const float* Mo, const float* Vo, int k, bool has) {
  return has ? AdamState{P[k], Mo[k], Vo[k]} : AdamState{0.f, 0.f, 0.f};
}
__device__ __forceinline__ void store_state(float* P, float* Mo, float* Vo, int k, const AdamState& a) {
  P[k] = a.p;
  Mo[k] = a.m;
  Vo[k] = a.v;
}

// `steps` Adam steps: step s takes rows (s * batch + j) mod n.  The master
// weights and moments stay in the registers of their owners; the FP16 tiles
// in LDS follow every update.  ONE: the batch is one pass of tiles, so the
// sums need not live across the tile phase.
template <bool ONE>
__global__ __launch_bounds__(kTrainThreads) void k_mlp_train(float* __restrict__ P, float* __restrict__ Mo,
                                                             float* __restrict__ Vo, const float* __restrict__ X,
                                                             const float* __restrict__ T, int n, int batch, int steps,
                                                             int step0, float lr, float S,
                                                             float* __restrict__ loss_out) {
  __shared__ TrainShared sh;
  const int tid = threadIdx.x, lane = tid & 63, wv = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int tiles = batch / 16;
  const float Btot = (float)batch;
  const Owned own = owned_params(wv, lane);
  AdamState s2[4], s13[4];
#pragma unroll
  for (int i = 0; i < 4; i++) {
    s2[i] = load_state(P, Mo, Vo, own.w2 + i, true);
    s13[i] = load_state(P, Mo, Vo, own.w13 + i, i < own.n13);
  }
  AdamState sb = load_state(P, Mo, Vo, own.b, own.b >= 0);
  // a division by a power of two is the multiplication by its reciprocal
  const bool s_pow2 = __float_as_uint(S) % (1u << 23) == 0 && S >= 0x1p-100f && S <= 0x1p100f;
  const float s_inv = 1.0f / S;
  auto unscale = [&](float v) { return s_pow2 ? v * s_inv : v / S; };
  AdamStep ahead = {};  // of step s - s % 64 + lane
  mlp::load_weights(sh.w, P, tid, kTrainThreads);
  // the row of this lane's sample in tile `tile` of the step whose first row is `from`
  auto row_of = [&](uint32_t from, int tile, int lane) {
    return (int64_t)((from + (uint32_t)(16 * tile + (lane & 15))) % (uint32_t)n);
  };
  uint32_t base = (uint32_t)(((uint64_t)step0 * (uint32_t)batch) % (uint32_t)n);
  TileRows next = load_rows(X, T, row_of(base, wv, lane), wv < tiles, lane);
  __syncthreads();
  for (int s = 0; s < steps; s++) {
    GradSums gs;
    BiasSums bs;
    if constexpr (!ONE) clear(gs, bs);
    const uint32_t base1 = (base + (uint32_t)batch) % (uint32_t)n;
    for (int t0 = 0; t0 < tiles; t0 += kTiles) {
      const TileRows in = next;
      // the next pass's rows, or the next step's first, load meanwhile
      const bool last = ONE || t0 + kTiles >= tiles;
      const int tn = last ? wv : t0 + kTiles + wv;
      const int lt = fresh(lane);
      next = load_rows(X, T, row_of(last ? base1 : base, tn, lt), tn < tiles, lt);
      if (t0 + wv < tiles) tile_signals(sh.w, sh.t[wv], in, true, S, Btot, lt);
      __syncthreads();
      if constexpr (ONE) clear(gs, bs);
      add_tiles(sh, min(kTiles, tiles - t0), wv, fresh(lane), gs, bs);
      if (last) break;
      __syncthreads();  // the tiles are free again
    }
    base = base1;
    if (wv == 8) {
      const float loss = sample_sum(f4{bs.loss[0], bs.loss[1], bs.loss[2], bs.loss[3]}, lane) / Btot;
      if (lane == 0 && loss_out) loss_out[s] = loss;
    }
    // the constants of 64 steps at a time, one per lane
    if (s % 64 == 0) {
      const float tstep = (float)((int64_t)step0 + s + lane + 1);
      ahead.c1 = 1.0f - powf(0.9f, tstep);
      ahead.c2 = 1.0f - powf(0.999f, tstep);
      ahead.i1 = 1.0f / ahead.c1;
      ahead.i2 = 1.0f / ahead.c2;
    }
    auto of_step = [&](float v) {
      return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), s % 64));
    };
    const AdamStep as = {lr, of_step(ahead.c1), of_step(ahead.c2), of_step(ahead.i1), of_step(ahead.i2)};
    const int la = fresh(lane), r = la & 15, g = la >> 4;
#pragma unroll
    for (int i = 0; i < 4; i++) {
      adam(s2[i], unscale(chain_sum(gs.w2, i)), as);
      const _Float16 h = (_Float16)s2[i].p;
      const int kr = 16 * (wv & 3) + r, c = 16 * (wv >> 2) + 4 * g + i;  // W2[kr][c]
      sh.w.w2t[c][kr] = h;
      sh.w.w2[kr][c] = h;
    }
    if (wv < 8) {
#pragma unroll
      for (int i = 0; i < 4; i++) {
        if (i >= own.n13) break;
        adam(s13[i], unscale(chain_sum(gs.w13, i)), as);
        const _Float16 h = (_Float16)s13[i].p;
        if (wv < 4) {
          sh.w.w1t[16 * wv + 4 * g + i][r] = h;
        } else {
          sh.w.w3t[i][16 * (wv & 3) + r] = h;
          sh.w.w3[16 * (wv & 3) + r][i] = h;
        }
      }
    }
    const float db = bias_sum(bs, wv, la);
    if (own.b >= 0) {
      adam(sb, unscale(db), as);
      const int q = la >> 2, fe = la & 3;
      float* const dst = q == 0 ? sh.w.b1 : q == 1 ? sh.w.b2 : sh.w.b3;
      dst[q == 2 ? fe : 4 * wv + fe] = sb.p;
    }
    __syncthreads();
  }
  const Owned to = owned_params(wv, fresh(lane));
#pragma unroll
  for (int i = 0; i < 4; i++) {
    store_state(P, Mo, Vo, to.w2 + i, s2[i]);
    if (i < to.n13) store_state(P, Mo, Vo, to.w13 + i, s13[i]);
  }
  if (to.b >= 0) store_state(P, Mo, Vo, to.b, sb);
}

// Gradient sums (scaled by S) and squared errors of the rows of passes b,
// b + gridDim.x, ... (`per` tiles each) into row b of part: kParams values,
// then the loss sum.  WHOLE (one workgroup, passes of kTiles tiles): the
// finished gradient and loss instead.
constexpr int kPartStride = mlp::kParams + 2;
template <bool WHOLE>
__global__ __launch_bounds__(kTrainThreads) void k_mlp_grad(const float* __restrict__ P, const float* __restrict__ X,
                                                            const float* __restrict__ T, int n, int tiles_per_pass, float S,
                                                            float* __restrict__ part, float* __restrict__ grad,
                                                            float* __restrict__ loss_out) {
  __shared__ TrainShared sh;
  const int tid = threadIdx.x, lane = tid & 63, wv = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int tiles = (int)(((int64_t)n + 15) / 16);
  const float Btot = (float)n;
  const int per = WHOLE ? kTiles : tiles_per_pass;
  const int stride = (WHOLE ? 1 : (int)gridDim.x) * per;
  auto load = [&](int tile) {
    const int64_t row = (int64_t)tile * 16 + (lane & 15);
    return load_rows(X, T, row, wv < per && tile < tiles && row < n, lane);
  };
  int t0 = WHOLE ? 0 : (int)blockIdx.x * per;
  TileRows next = load(t0 + wv);
  mlp::load_weights(sh.w, P, tid, kTrainThreads);
  __syncthreads();
  GradSums gs;
  BiasSums bs;
  clear(gs, bs);
  for (; t0 < tiles; t0 += stride) {
    const TileRows in = next;
    const int lt = fresh(lane);
    if (t0 + stride < tiles) next = load(t0 + stride + wv);
    // whole groups of kChains tiles: the ones past the last row add zeros
    const int nt = min(per, (tiles - t0 + kChains - 1) / kChains * kChains);
    if (wv < nt) tile_signals(sh.w, sh.t[wv], in, (int64_t)(t0 + wv) * 16 + (lt & 15) < n, S, Btot, lt);
    __syncthreads();
    add_tiles(sh, nt, wv, fresh(lane), gs, bs);
    __syncthreads();  // the tiles are free again
  }
  float* const out = WHOLE ? grad : part + (size_t)blockIdx.x * kPartStride;
  const float scale = WHOLE ? S : 1.0f;
  const Owned own = owned_params(wv, lane);
#pragma unroll
  for (int i = 0; i < 4; i++) {
    out[own.w2 + i] = chain_sum(gs.w2, i) / scale;
    if (i < own.n13) out[own.w13 + i] = chain_sum(gs.w13, i) / scale;
  }
  const float db = bias_sum(bs, wv, lane);
  if (own.b >= 0) out[own.b] = db / scale;
  if (wv == 8) {
    const float ls = sample_sum(f4{bs.loss[0], bs.loss[1], bs.loss[2], bs.loss[3]}, lane);
    if (lane == 0) {
      if (!WHOLE)
        out[mlp::kParams] = ls;
      else if (loss_out)
        loss_out[0] = ls / Btot;
    }
  }
}

// Sums of the np (at most kGradMax) partial rows, in a fixed order: workgroup b
// takes values 64 b .. 64 b + 63; its 16 waves add every 16th row each, all
// loaded before the first addition (44,672 rows 22.9 -> 21.4 us at the time), then wave by
// wave.
constexpr int kGradMax = 256;
__global__ __launch_bounds__(1024) void k_mlp_grad_sum(const float* __restrict__ part, int np, float S, float Btot,
                                                       float* __restrict__ grad, float* __restrict__ loss_out) {
  __shared__ float s_sum[16][64];
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  const int k = (int)blockIdx.x * 64 + lane;
  float v = 0.f;
  if (k <= mlp::kParams) {
    float p[kGradMax / 16];
#pragma unroll
    for (int i = 0; i < kGradMax / 16; i++)
      p[i] = wv + 16 * i < np ? part[(size_t)(wv + 16 * i) * kPartStride + k] : 0.0f;
#pragma unroll
    for (int i = 0; i < kGradMax / 16; i++) v += p[i];
  }
  s_sum[wv][lane] = v;
  __syncthreads();
  if (wv > 0 || k > mlp::kParams) return;
  v = 0.f;
#pragma unroll
  for (int w = 0; w < 16; w++) v += s_sum[w][lane];
  if (k < mlp::kParams)
    grad[k] = v / S;
  else if (loss_out)
    loss_out[0] = v / Btot;
}

// Tiles of a gradient's workgroup per pass: the fewest whole groups of kChains
// with which kGradShare workgroups cover the rows, at most kTiles (then up to
// one workgroup per CU, whose LDS it fills).  Fewer tiles share a CU's vector
// units among fewer waves; more workgroups leave more partial rows to add.  4,
// 8, 12, 16 tiles: 512 rows 11.2, 12.2, 13.6, 15.1 us; 8,000 12.9, 13.0, 14.1,
// 15.4; 16,000 14.8, 14.0, 14.6, 15.8; 30,000 18.5, 15.8, 16.0, 16.9; 44,672
// 22.0, 20.9, 17.3, 17.8.  Rows past one pass of every CU spread evenly over
// the passes they need.
constexpr int kGradShare = 240;
int grad_tiles(int64_t tiles) {
  if (tiles <= kTiles) return kTiles;
  const int64_t passes = (tiles + kGradMax * kTiles - 1) / (kGradMax * kTiles);
  const int64_t share = passes > 1 ? passes * kGradMax : kGradShare;
  const int64_t per = (tiles + share - 1) / share;
  return (int)std::min<int64_t>((per + kChains - 1) / kChains * kChains, kTiles);
}
int grad_groups(int32_t n) {
  const int64_t tiles = ((int64_t)n + 15) / 16, per = grad_tiles(tiles);
  return (int)std::min<int64_t>((tiles + per - 1) / per, kGradMax);
}

}  // namespace

extern "C" {

int lbm_mlp_param_count(int32_t* n) {
  if (!n) return LBM_EINVAL;
  *n = mlp::kParams;
  return LBM_OK;
}

int lbm_mlp_forward(const float* d_params, const float* d_x, float* d_y, int64_t n, void* hip_stream) {
  if (!d_params || !d_x || !d_y || n < 0) return LBM_EINVAL;
  if (n == 0) return LBM_OK;
  const int64_t tiles = (n + 15) / 16;
  // every workgroup first stages the weights (about 5 us), so up to 2^17 tiles
  // there are only as many as fit the chip at once (4 per CU: 200,000 rows 14
  // us, against 18 with 2,048 and 26 with 4,096); beyond, twice as many share
  // out the CUs' unequal speed (4,194,304 rows: 160 us, against 168 and 163; at
  // the line itself 2,097,152 rows 85.8 us with 1,024, 16 rows more 82.7 with
  // 2,048)
  const int64_t most = tiles <= (int64_t)1 << 17 ? 1024 : 2048;
  const int64_t blocks = std::min<int64_t>((tiles + kWaves - 1) / kWaves, most);
  k_mlp_forward<<<(unsigned)blocks, 256, 0, (hipStream_t)hip_stream>>>(d_params, d_x, d_y, n);
  return hipGetLastError() == hipSuccess ? LBM_OK : LBM_EHIP;
}

static int gradient_impl(const float* d_params, const float* d_x, const float* d_t, int32_t n, float loss_scale,
                         float* d_grad, float* d_loss, float* work, int groups, hipStream_t stream) {
  if (groups == 1) {
    k_mlp_grad<true><<<1, kTrainThreads, 0, stream>>>(d_params, d_x, d_t, n, kTiles, loss_scale, work, d_grad, d_loss);
  } else {
    k_mlp_grad<false><<<groups, kTrainThreads, 0, stream>>>(d_params, d_x, d_t, n, grad_tiles(((int64_t)n + 15) / 16),
                                                            loss_scale, work, d_grad, d_loss);
    k_mlp_grad_sum<<<(mlp::kParams + 64) / 64, 1024, 0, stream>>>(work, groups, loss_scale, (float)n, d_grad, d_loss);
  }
  return hipGetLastError() == hipSuccess ? LBM_OK : LBM_EHIP;
}

int lbm_mlp_gradient(const float* d_params, const float* d_x, const float* d_t, int32_t n, float loss_scale,
                     float* d_grad, float* d_loss, void* hip_stream) {
  if (!d_params || !d_x || !d_t || !d_grad || n < 1 || !(loss_scale > 0)) return LBM_EINVAL;
  return gradient_impl(d_params, d_x, d_t, n, loss_scale, d_grad, d_loss, nullptr, 1, (hipStream_t)hip_stream);
}

int lbm_mlp_gradient_work_size(int32_t n, size_t* bytes) {
  if (!bytes || n < 1) return LBM_EINVAL;
  const int g = grad_groups(n);
  *bytes = g > 1 ? sizeof(float) * (size_t)kPartStride * g : 0;
  return LBM_OK;
}

int lbm_mlp_gradient_in(const float* d_params, const float* d_x, const float* d_t, int32_t n, float loss_scale,
                        float* d_grad, float* d_loss, void* d_work, size_t bytes, void* hip_stream) {
  if (!d_params || !d_x || !d_t || !d_grad || n < 1 || !(loss_scale > 0)) return LBM_EINVAL;
  size_t need = 0;
  (void)lbm_mlp_gradient_work_size(n, &need);
  if (need > 0 && (!d_work || (uintptr_t)d_work % sizeof(float) || bytes < need)) return LBM_EWORKSPACE;
  return gradient_impl(d_params, d_x, d_t, n, loss_scale, d_grad, d_loss, (float*)d_work, grad_groups(n),
                       (hipStream_t)hip_stream);
}

int lbm_mlp_train(float* d_params, float* d_adam_m, float* d_adam_v, const float* d_x, const float* d_t, int32_t n,
                  int32_t batch, int32_t steps, int32_t step0, float lr, float loss_scale, float* d_loss,
                  void* hip_stream) {
  if (!d_params || !d_adam_m || !d_adam_v || !d_x || !d_t || n < 1 || steps < 0 || step0 < 0) return LBM_EINVAL;
  if (batch < 64 || batch % 64 || !(lr > 0) || !(loss_scale > 0)) return LBM_EINVAL;
  if (steps == 0) return LBM_OK;
  if (batch <= 16 * kTiles)
    k_mlp_train<true><<<1, kTrainThreads, 0, (hipStream_t)hip_stream>>>(d_params, d_adam_m, d_adam_v, d_x, d_t, n, batch,
                                                                        steps, step0, lr, loss_scale, d_loss);
  else
    k_mlp_train<false><<<1, kTrainThreads, 0, (hipStream_t)hip_stream>>>(d_params, d_adam_m, d_adam_v, d_x, d_t, n,
                                                                         batch, steps, step0, lr, loss_scale, d_loss);
  return hipGetLastError() == hipSuccess ? LBM_OK : LBM_EHIP;
}

}  // extern "C"

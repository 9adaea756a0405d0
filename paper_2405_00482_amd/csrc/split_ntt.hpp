// A limb of 2^13 or 2^14 transformed by S = N / 2^12 workgroups, for calls
// with few limbs: one limb on one CU is bound by that CU's issue rate (8 - 16
// waves of 2000 operations) while the others idle.
//
// After the first log2 S forward stages (before the last log2 S inverse ones)
// the transform falls into S blocks of 4096 coefficients, each a 2^12
// transform of its own.  A chain inverse -> conversion -> forward takes two
// launches: the first makes the S blocks of the inverse and writes them as
// they are; in the second every workgroup reads all S blocks, finishes the
// inverse (radix S on the thread's own S values), converts, does the first
// forward stages for the one block it makes, and transforms that.
//
// Block h holds the slots of exponents e = 2 k + 1 with k mod S = brv(h): at S =
// 2 half h of the orbit; at S = 4, as 5^t is 1 or 5 mod 8 for even or odd t,
// the even (h = 0) and odd (1) slots of the first half, the odd (2) and even
// (3) ones of the second.
#pragma once
#include "ntt_core.hpp"

namespace pvfl {

template <int LOGN>
struct SplitNtt {
  static_assert(LOGN == 13 || LOGN == 14, "two or four blocks");
  static constexpr int N = 1 << LOGN, S = N >> 12, T = 256, G = S / 2;  // G: stride of a block's slots
  static constexpr int LDS = NttShape<12>::LDS;

  int h, odd;
  uint32_t e0;  // 5^t of the thread's first slot
  __device__ __forceinline__ explicit SplitNtt(int block) : h(block), odd(S == 4 && (block == 1 || block == 2)) {
    const uint32_t mask = 2u * N - 1u, t = G * threadIdx.x + odd;
    uint32_t r = 1, b = 5;
#pragma unroll
    for (int k = 0; k < 9; ++k) {
      if ((t >> k) & 1u) r = (r * b) & mask;
      b = (b * b) & mask;
    }
    e0 = r;
  }
  // slot w of the thread, and its place in LDS (e: step() applied w times to e0)
  __device__ __forceinline__ int slot(int w) const { return (h >= G ? N / 2 : 0) + G * ((int)threadIdx.x + w * T) + odd; }
  __device__ __forceinline__ int place(uint32_t e) const {
    const uint32_t i = __brev(e >> 1) >> (32 - LOGN);
    return lds_pad((int)((h >= G ? ~i : i) & 4095u));
  }
  static constexpr uint32_t stride() {  // 5^(G T) mod 2N
    uint32_t r = 1;
    for (int i = 0; i < G * T; ++i) r = (r * 5u) & (2u * N - 1u);
    return r;
  }
  __device__ __forceinline__ static uint32_t step(uint32_t e) {
    return (e * std::integral_constant<uint32_t, stride()>::value) & (2u * N - 1u);
  }

  // this block of the inverse transform of in(t), before the last log2 S
  // stages: value threadIdx.x + w T in c[w], centred
  template <class In>
  __device__ __forceinline__ void inverse(double* s, In in, const double* __restrict__ itw, ModQ m, double (&c)[16]) const {
    double v[16];
#pragma unroll
    for (int w = 0; w < 16; ++w) v[w] = in(slot(w));
    uint32_t e = e0;
#pragma unroll
    for (int w = 0; w < 16; ++w) {
      s[place(e)] = reduce(v[w], m);
      e = step(e);
    }
    __syncthreads();
    ntt_inv_regs<12, true>(s, c, itw, m, 0.0, S + h);
  }

  // the coefficients j + k 4096 from the blocks' values j, y[k 4096 + j]
  __device__ __forceinline__ static void finish(const double (&y)[S], const double* __restrict__ itw, ModQ m, double ninv,
                                                double w1, double (&x)[S]) {  // w1 = itw[1] / N
    if constexpr (S == 2) {
      x[0] = mulmod(y[0] + y[1], ninv, m);
      x[1] = mulmod(y[0] - y[1], w1, m);
    } else {
      const double u0 = y[0] + y[1], u1 = mulmod(y[0] - y[1], itw[2], m);
      const double u2 = y[2] + y[3], u3 = mulmod(y[2] - y[3], itw[3], m);
      x[0] = mulmod(u0 + u2, ninv, m);
      x[1] = mulmod(u1 + u3, ninv, m);
      x[2] = mulmod(u0 - u2, w1, m);
      x[3] = mulmod(u1 - u3, w1, m);
    }
  }
  // block h's value of the first log2 S forward stages
  __device__ __forceinline__ double first(const double (&x)[S], const double* __restrict__ tw, ModQ m) const {
    if constexpr (S == 2) {
      const double v = mulmod(x[1], tw[1], m);
      return h ? x[0] - v : x[0] + v;
    } else {
      const double a = mulmod(x[2], tw[1], m), b = mulmod(x[3], tw[1], m);
      const double p = h & 2 ? x[0] - a : x[0] + a;
      const double v = mulmod(h & 2 ? x[1] - b : x[1] + b, tw[2 + (h >> 1)], m);
      return h & 1 ? p - v : p + v;
    }
  }
  // forward transform of the block; slot w of the thread in v[w], centred
  __device__ __forceinline__ void forward(double* s, const double (&c)[16], const double* __restrict__ tw, ModQ m,
                                          double (&v)[16]) const {
    ntt_fwd_regs<12, true>(s, c, tw, m, S + h);
    uint32_t e = e0;
#pragma unroll
    for (int w = 0; w < 16; ++w) {
      v[w] = s[place(e)];
      e = step(e);
    }
  }

  // y: a limb's blocks of the inverse modulo prime ps; conv(x) turns its
  // coefficients into those modulo prime pt; block h of their transform in v
  template <class Y, class Conv>
  __device__ __forceinline__ void chain(double* s, Y y, int ps, int pt, const DevTabs& tb, Conv conv, double (&v)[16]) const {
    const ModQ m = tb.mods[ps], mt = tb.mods[pt];
    const double* itw = tb.inv_tw + (size_t)ps * N;
    const double* tw = tb.fwd_tw + (size_t)pt * N;
    const double ninv = tb.ninv[ps], w1 = reduce(mulmod(itw[1], ninv, m), m);
    double c[16];
#pragma unroll
    for (int w = 0; w < 16; ++w) {
      double in[S], x[S];
#pragma unroll
      for (int k = 0; k < S; ++k) in[k] = y[k * 4096 + (int)threadIdx.x + w * T];
      finish(in, itw, m, ninv, w1, x);
#pragma unroll
      for (int k = 0; k < S; ++k) x[k] = conv(x[k]);
      c[w] = first(x, tw, mt);
    }
    forward(s, c, tw, mt, v);
  }
};

}  // namespace pvfl

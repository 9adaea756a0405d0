// Device helpers shared by the HIP kernel files: the counter-based
// generator and samplers, the orbit shift of a rotation, LDS write-out.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "kernels.hpp"
#include "ntt_core.hpp"
#include "split_ntt.hpp"

namespace pvfl {

// ---------------------------------------------------------------------------
// Philox4x32-10 counter-based generator (Salmon et al., SC'11) and samplers.
// Word idx of stream `stream` under key `seed`: counter = (idx>>1, stream),
// key = seed, word (0,1) for even idx and (2,3) for odd idx, low word first.
// ---------------------------------------------------------------------------
// words 2 `pair` and 2 `pair` + 1
struct PhiloxPair {
  uint64_t w0, w1;
};
__device__ __forceinline__ PhiloxPair philox_pair(uint64_t seed, uint64_t stream, uint64_t pair) {
  uint32_t c0 = (uint32_t)pair, c1 = (uint32_t)(pair >> 32);
  uint32_t c2 = (uint32_t)stream, c3 = (uint32_t)(stream >> 32);
  uint32_t k0 = (uint32_t)seed, k1 = (uint32_t)(seed >> 32);
#pragma unroll
  for (int round = 0; round < 10; ++round) {
    if (round) { k0 += 0x9E3779B9u; k1 += 0xBB67AE85u; }
    const uint32_t lo0 = 0xD2511F53u * c0, hi0 = __umulhi(0xD2511F53u, c0);
    const uint32_t lo1 = 0xCD9E8D57u * c2, hi1 = __umulhi(0xCD9E8D57u, c2);
    const uint32_t n0 = hi1 ^ c1 ^ k0, n2 = hi0 ^ c3 ^ k1;
    c0 = n0; c1 = lo1; c2 = n2; c3 = lo0;
  }
  return PhiloxPair{(uint64_t)c0 | ((uint64_t)c1 << 32), (uint64_t)c2 | ((uint64_t)c3 << 32)};
}
__device__ __forceinline__ uint64_t philox_word(uint64_t seed, uint64_t stream, uint64_t idx) {
  const PhiloxPair p = philox_pair(seed, stream, idx >> 1);
  return (idx & 1) ? p.w1 : p.w0;
}

// floor(u * q / 2^64) for q < 2^49: the high 64 bits of a 64x64 product.
__device__ __forceinline__ uint64_t mul_hi64(uint64_t a, uint64_t b) { return __umul64hi(a, b); }

__device__ __forceinline__ double uniform_res(uint64_t word, uint64_t q) { return u64_to_f64(mul_hi64(word, q)); }
__device__ __forceinline__ int ternary(uint64_t word) { return (int)mul_hi64(word, 3ull) - 1; }
__device__ __forceinline__ int cbd21(uint64_t word) {
  return __popcll(word & 0x1FFFFFull) - __popcll((word >> 21) & 0x1FFFFFull);
}
__device__ __forceinline__ double sample_uniform_res(uint64_t seed, uint64_t stream, uint64_t idx, uint64_t q) {
  return uniform_res(philox_word(seed, stream, idx), q);
}
__device__ __forceinline__ int sample_ternary(uint64_t seed, uint64_t stream, uint64_t idx) {
  return ternary(philox_word(seed, stream, idx));
}
__device__ __forceinline__ int sample_cbd21(uint64_t seed, uint64_t stream, uint64_t idx) {
  return cbd21(philox_word(seed, stream, idx));
}

// c[w] = f(word j, j) for a thread's coefficients j = tid + w T.  A generator
// call yields the words of two neighbouring coefficients, which two
// neighbouring lanes own: each lane calls it for every other w and hands the
// partner its word (quad permutation), half the calls of one per coefficient.
template <int LOGN, class F>
__device__ __forceinline__ void sample_coeffs(uint64_t seed, uint64_t stream, double (&c)[NttShape<LOGN>::PER], F f) {
  constexpr int T = NttShape<LOGN>::T, PER = NttShape<LOGN>::PER;
  const int tid = opaque_tid(), odd = tid & 1;
  auto swap = [](uint64_t x) {
    const int lo = __builtin_amdgcn_mov_dpp((int)(uint32_t)x, 0xB1, 0xf, 0xf, true);
    const int hi = __builtin_amdgcn_mov_dpp((int)(uint32_t)(x >> 32), 0xB1, 0xf, 0xf, true);
    return (uint64_t)(uint32_t)lo | ((uint64_t)(uint32_t)hi << 32);
  };
#pragma unroll
  for (int w = 0; w < PER; w += 2) {
    const PhiloxPair p = philox_pair(seed, stream, (uint64_t)((tid >> 1) + (w + odd) * (T / 2)));
    const uint64_t got = swap(odd ? p.w0 : p.w1);
    c[w] = f(odd ? got : p.w0, tid + w * T);
    c[w + 1] = f(odd ? p.w1 : got, tid + (w + 1) * T);
  }
}

__device__ __forceinline__ int orbit_shift(int t, int rot, int half) {
  return (t & half) | ((t + rot) & (half - 1));
}

// Base conversion of a thread's coefficients j = tid + w T: the sum over `n`
// limbs of y_u[j] hat(u) mod m, less `h`, centred.  Source by source, so that
// a source's loads are in flight together; one limb alone has hat = 1.
template <int LOGN, class Y, class Hat>
__device__ __forceinline__ void convert_coeffs(Y y, int n, Hat hat, double h, ModQ m, double (&x)[NttShape<LOGN>::PER]) {
  constexpr int N = 1 << LOGN, T = NttShape<LOGN>::T, PER = NttShape<LOGN>::PER;
#pragma unroll
  for (int w = 0; w < PER; ++w) x[w] = y[(int)opaque_tid() + w * T];
  if (n > 1) {
    const double h0 = hat(0);
#pragma unroll
    for (int w = 0; w < PER; ++w) x[w] = mulmod(x[w], h0, m);
    for (int u = 1; u < n; ++u) {
      const double hu = hat(u);
#pragma unroll
      for (int w = 0; w < PER; ++w) x[w] += mulmod(y[(size_t)u * N + (int)opaque_tid() + w * T], hu, m);
    }
  }
#pragma unroll
  for (int w = 0; w < PER; ++w) x[w] = reduce(x[w] - h, m);
}

// Key switching with one special prime: the conversions between its two
// transforms.  A digit is one limb and P one prime, so that the products over
// the other primes of a digit or of P are empty: nothing to multiply by.
struct ModUpOne {  // coefficients |x| < q of limb task.src0 to the target limb's prime
  ModQ ms, m;
  __device__ __forceinline__ ModUpOne(const KsTask& task, const DevTabs& tb) : ms(tb.mods[task.src0]), m(tb.mods[task.prime]) {}
  __device__ __forceinline__ double operator()(double x) const { return reduce(x < 0.0 ? x + ms.q : x, m); }
};
struct ModDownOne {  // coefficients of the special limb, less its half, to limb i's prime
  int prime;
  ModQ mp, m;
  double hp, h, pinv;
  __device__ __forceinline__ ModDownOne(int i, const KsLevel* __restrict__ kl, const DevTabs& tb)
      : prime(kl->n_q_total), mp(tb.mods[kl->n_q_total]), m(tb.mods[i]), hp(kl->down_half[kl->lv + 1]),
        h(kl->down_half[i]), pinv(kl->down_pinv[i]) {}
  __device__ __forceinline__ double operator()(double x) const { return reduce(canon(x + hp, mp) - h, m); }
  __device__ __forceinline__ double result(double u, double v) const { return reduce(mulmod(u - v, pinv, m), m); }
};

// Both transforms of a step in one workgroup (N <= 2^14).
// ModUp: coefficients x of limb task.src0 (slots in(t)), converted.  Barrier
// before writing LDS again (the transforms do).
template <int LOGN, class In>
__device__ __forceinline__ void modup_source(double* s, In in, const KsTask& task, const DevTabs& tb, double (&x)[16]) {
  constexpr int N = 1 << LOGN;
  const int si = task.src0;
  const ModUpOne conv(task, tb);
  ntt_inv_in_regs<LOGN>(s, in, tb.inv_tw + (size_t)si * N, conv.ms, tb.ninv[si], x);
#pragma unroll
  for (int w = 0; w < 16; ++w) x[w] = conv(x[w]);
}
// ModDown of ciphertext limb i: the special limb's slots in(t), the limb's own
// slots u (as slots_from_lds orders them), results to out(t, v).
template <int LOGN, class In, class Out>
__device__ __forceinline__ void moddown_limb(double* s, In in, const double (&u)[16], int i,
                                             const KsLevel* __restrict__ kl, const DevTabs& tb, Out out) {
  constexpr int N = 1 << LOGN, T = NttShape<LOGN>::T;
  const ModDownOne conv(i, kl, tb);
  double c[16], v[16];
  ntt_inv_in_regs<LOGN>(s, in, tb.inv_tw + (size_t)conv.prime * N, conv.mp, tb.ninv[conv.prime], c);
#pragma unroll
  for (int w = 0; w < 16; ++w) c[w] = conv(c[w]);
  ntt_fwd_regs<LOGN>(s, c, tb.fwd_tw + (size_t)i * N, conv.m);
  slots_from_lds<LOGN>(s, v);
#pragma unroll
  for (int w = 0; w < 16; ++w) out((int)opaque_tid() + (w >> 1) * T + (w & 1) * (N / 2), conv.result(u[w], v[w]));
}

// One block of a split limb's inverse (SplitNtt), to y[h 4096 ...].
template <int LOGN, class In>
__device__ __forceinline__ void split_inverse(double* s, int h, In in, int pi, const DevTabs& tb, double* __restrict__ y) {
  const SplitNtt<LOGN> sp(h);
  double c[16];
  sp.inverse(s, in, tb.inv_tw + ((size_t)pi << LOGN), tb.mods[pi], c);
#pragma unroll
  for (int w = 0; w < 16; ++w) y[h * 4096 + (int)threadIdx.x + w * 256] = c[w];
}
// Block h of a ModUp target limb from the source limb's blocks y.
template <int LOGN, class Y>
__device__ __forceinline__ void split_modup(double* s, int h, Y y, const KsTask& task, const DevTabs& tb,
                                            double* __restrict__ dst) {
  const SplitNtt<LOGN> sp(h);
  double v[16];
  sp.chain(s, y, task.src0, task.prime, tb, ModUpOne(task, tb), v);
#pragma unroll
  for (int w = 0; w < 16; ++w) dst[sp.slot(w)] = v[w];
}
// Block h of ciphertext limb i after ModDown: the limb's own slots u, the
// special limb's blocks y.
template <int LOGN, class U, class Y>
__device__ __forceinline__ void split_moddown(double* s, int h, U u, Y y, int i, const KsLevel* __restrict__ kl,
                                              const DevTabs& tb, double* __restrict__ out) {
  const SplitNtt<LOGN> sp(h);
  const ModDownOne conv(i, kl, tb);
  double uv[16], v[16];
#pragma unroll
  for (int w = 0; w < 16; ++w) uv[w] = u[sp.slot(w)];
  sp.chain(s, y, conv.prime, i, tb, conv, v);
#pragma unroll
  for (int w = 0; w < 16; ++w) out[sp.slot(w)] = conv.result(uv[w], v[w]);
}

}  // namespace pvfl

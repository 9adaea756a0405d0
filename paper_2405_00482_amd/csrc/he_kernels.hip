// HIP kernels of the RNS-CKKS ciphertext x plaintext matrix product for gfx950.
// Residues are exact binary64 integers (fp64_mod.hpp); evaluation-domain limbs
// are stored in the orbit order of ntt_core.hpp.
// Key generation, encryption and the key-switching kernels loop over limbs
// in registers: keep their thread-index arithmetic inside the loops (see
// opaque_tid in ntt_core.hpp).
#define PVFL_OPAQUE_TID 1

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "he_dev.hpp"
#include "kernels.hpp"
#include "ntt_core.hpp"

namespace pvfl {

#define NTT_KERNEL(LOGN) __global__ __launch_bounds__(NttShape<LOGN>::T)
#define NTT_LDS(LOGN) __shared__ double s[NttShape<LOGN>::LDS]

// ---------------------------------------------------------------------------
// plain batched transforms over contiguous limbs.  Block b handles limb
// b % nl of polynomial b / nl; limb l uses prime map.idx[l].
// ---------------------------------------------------------------------------
template <int LOGN>
NTT_KERNEL(LOGN) void k_ntt_fwd(const double* __restrict__ in, double* __restrict__ out, LimbMap map, DevTabs tb) {
  constexpr int N = 1 << LOGN;
  NTT_LDS(LOGN);
  const int b = blockIdx.x, pi = map.idx[b % map.n];
  const ModQ m = tb.mods[pi];
  const double* src = in + (size_t)b * N;
  double* dst = out + (size_t)b * N;
  ntt_fwd_out<LOGN>(s, [&](int j) { return src[j]; }, tb.fwd_tw + (size_t)pi * N, m,
                    [&](int t, double v) { dst[t] = v; });
}

template <int LOGN>
NTT_KERNEL(LOGN) void k_ntt_inv(const double* __restrict__ in, double* __restrict__ out, LimbMap map, DevTabs tb) {
  constexpr int N = 1 << LOGN;
  NTT_LDS(LOGN);
  const int b = blockIdx.x, pi = map.idx[b % map.n];
  const ModQ m = tb.mods[pi];
  const double* src = in + (size_t)b * N;
  double* dst = out + (size_t)b * N;
  ntt_inv_in<LOGN>(s, [&](int t) { return src[t]; }, tb.inv_tw + (size_t)pi * N, m, tb.ninv[pi],
                   [&](int j, double v) { dst[j] = v; });
}

// signed integer coefficients [count][N] -> evaluation-domain residues
// [count][nl][N]: every limb of polynomial c is the same integer vector.
template <int LOGN>
NTT_KERNEL(LOGN) void k_import_i64(const int64_t* __restrict__ in, double* __restrict__ out, LimbMap map, DevTabs tb) {
  constexpr int N = 1 << LOGN;
  NTT_LDS(LOGN);
  const int b = blockIdx.x, c = b / map.n, pi = map.idx[b % map.n];
  const ModQ m = tb.mods[pi];
  const double t32 = tb.two32[pi];
  const int64_t* src = in + (size_t)c * N;
  double* dst = out + (size_t)b * N;
  ntt_fwd_out<LOGN>(s, [&](int j) { return i64_to_res(src[j], m, t32); }, tb.fwd_tw + (size_t)pi * N, m,
                    [&](int t, double v) { dst[t] = v; });
}

// The same at N <= 2^14 with one workgroup per polynomial: the integer row is
// read once, into registers, and every limb is reduced from it and
// transformed in turn, so the row's memory latency is paid once per
// polynomial instead of once per limb.
template <int LOGN>
LIMBS_KERNEL(LOGN) void k_import_i64_poly(const int64_t* __restrict__ in, double* __restrict__ out, LimbMap map,
                                        DevTabs tb) {
  static_assert(LOGN <= 14, "one LDS-resident limb");
  constexpr int N = 1 << LOGN, T = NttShape<LOGN>::T;
  NTT_LDS(LOGN);
  const int c = blockIdx.x;
  const int64_t* src = in + (size_t)c * N;
  // v = hi 2^32 + lo, both parts exact in binary64
  const unsigned tid = opaque_tid();
  int hi[16];
  unsigned lo[16];
#pragma unroll
  for (int w = 0; w < 16; ++w) {
    const int64_t v = scalar_base(src + w * T)[tid];
    hi[w] = (int)(v >> 32);
    lo[w] = (unsigned)v;
  }
  const OrbitIndex<LOGN> oi = OrbitIndex<LOGN>::make();
  for (int l = 0; l < map.n; ++l) {
    const int pi = map.idx[l];
    const ModQ m = tb.mods[pi];
    const double t32 = tb.two32[pi];
    double x[16];
    // |hi| <= 2^31 and |t32| <= q/2 as mulmod needs, q + 2^32 < 2^51 as the transform
#pragma unroll
    for (int w = 0; w < 16; ++w) {
      asm volatile("" : "+v"(hi[w]), "+v"(lo[w]));  // converted for every limb: half the registers
      x[w] = mulmod((double)hi[w], t32, m) + (double)lo[w];
    }
    double* dst = out + ((size_t)c * map.n + l) * N;
    // nothing in this kernel reads the output again: stream it past L2
    ntt_fwd_regs_out<LOGN>(s, x, tb.fwd_tw + (size_t)pi * N, m,
                           [&](unsigned b, unsigned t, double y) { __builtin_nontemporal_store(y, scalar_base(dst + b) + t); },
                           oi.opaque());
  }
}

// evaluation-domain residues -> canonical coefficient residues as uint64
template <int LOGN>
NTT_KERNEL(LOGN) void k_export_u64(const double* __restrict__ in, uint64_t* __restrict__ out, LimbMap map, DevTabs tb) {
  constexpr int N = 1 << LOGN;
  NTT_LDS(LOGN);
  const int b = blockIdx.x, pi = map.idx[b % map.n];
  const ModQ m = tb.mods[pi];
  const double* src = in + (size_t)b * N;
  uint64_t* dst = out + (size_t)b * N;
  ntt_inv_in<LOGN>(s, [&](int t) { return src[t]; }, tb.inv_tw + (size_t)pi * N, m, tb.ninv[pi],
                   [&](int j, double v) { dst[j] = f64_to_u64(canon(v, m)); });
}

// The same at N <= 2^14 with one workgroup per polynomial: while one limb is
// transformed, the next limb's values are already being loaded into
// registers (its slots go to LDS only after this limb's transform is done).
template <int LOGN>
LIMBS_KERNEL(LOGN) void k_export_u64_poly(const double* __restrict__ in, uint64_t* __restrict__ out, LimbMap map,
                                        DevTabs tb) {
  static_assert(LOGN <= 14, "one LDS-resident limb");
  constexpr int N = 1 << LOGN, T = NttShape<LOGN>::T;
  NTT_LDS(LOGN);
  const int c = blockIdx.x;
  const double* src = in + (size_t)c * map.n * N;
  const unsigned tid = opaque_tid();
  // v[2w], v[2w+1]: orbit slots t = tid + w T and t + N/2 of the current limb
  double v[16];
#pragma unroll
  for (int w = 0; w < 8; ++w) {
    v[2 * w] = scalar_base(src + w * T)[tid];
    v[2 * w + 1] = scalar_base(src + w * T + N / 2)[tid];
  }
  const OrbitIndex<LOGN> oi = OrbitIndex<LOGN>::make();
  for (int l = 0; l < map.n; ++l) {
    const int pi = map.idx[l];
    const ModQ m = tb.mods[pi];
    slots_to_lds<LOGN>(s, v, m, oi.opaque());
    if (l + 1 < map.n) {
      const double* nsrc = src + (size_t)(l + 1) * N;
#pragma unroll
      for (int w = 0; w < 8; ++w) {
        v[2 * w] = scalar_base(nsrc + w * T)[tid];
        v[2 * w + 1] = scalar_base(nsrc + w * T + N / 2)[tid];
      }
    }
    __syncthreads();
    double cf[16];
    ntt_inv_regs<LOGN>(s, cf, tb.inv_tw + (size_t)pi * N, m, tb.ninv[pi]);
    uint64_t* dst = out + ((size_t)c * map.n + l) * N;
#pragma unroll
    for (int w = 0; w < 16; ++w)
      __builtin_nontemporal_store(f64_to_u64(cf[w] < 0.0 ? cf[w] + m.q : cf[w]), scalar_base(dst + w * T) + tid);
    __syncthreads();  // other threads may still read this limb from LDS
  }
}

// ---------------------------------------------------------------------------
// keys and encryption
// ---------------------------------------------------------------------------
// secret key: ternary s, transformed for every prime of the context.
template <int LOGN>
NTT_KERNEL(LOGN) void k_keygen(uint64_t seed, double* __restrict__ sk, DevTabs tb) {
  constexpr int N = 1 << LOGN;
  NTT_LDS(LOGN);
  const int pi = blockIdx.x;
  const ModQ m = tb.mods[pi];
  double* dst = sk + (size_t)pi * N;
  ntt_fwd_out<LOGN>(s, [&](int j) { return (double)sample_ternary(seed, kStreamSecret, (uint64_t)j); },
                    tb.fwd_tw + (size_t)pi * N, m, [&](int t, double v) { dst[t] = v; });
}

// Secret-key encryption of integer coefficients m (c1 = a, c0 = -a s + m + e)
// at level lv; ciphertext c uses msg[c] and seed + c.  The two transforms:
// a, uniform in the coefficient domain, and m + e.
template <int LOGN, class Out>
__device__ __forceinline__ void encrypt_a(double* s, uint64_t seed, int i, const DevTabs& tb, Out out) {
  constexpr int N = 1 << LOGN;
  const ModQ m = tb.mods[i];
  const uint64_t qi = (uint64_t)m.q;
  double c[NttShape<LOGN>::PER];
  sample_coeffs<LOGN>(seed, kStreamEncA | (uint64_t)i, c, [&](uint64_t u, int) { return uniform_res(u, qi); });
  ntt_fwd_regs_out<LOGN>(s, c, tb.fwd_tw + (size_t)i * N, m, out);
}
template <int LOGN, class Out>
__device__ __forceinline__ void encrypt_message(double* s, const int64_t* __restrict__ msg, uint64_t seed, uint64_t stream,
                                                int i, const DevTabs& tb, Out out) {
  constexpr int N = 1 << LOGN;
  const ModQ m = tb.mods[i];
  const double t32 = tb.two32[i];
  double c[NttShape<LOGN>::PER];
  sample_coeffs<LOGN>(seed, stream, c,
                      [&](uint64_t u, int j) { return reduce(i64_to_res(msg[j], m, t32) + (double)cbd21(u), m); });
  ntt_fwd_regs_out<LOGN>(s, c, tb.fwd_tw + (size_t)i * N, m, out);
}

// block (c, i): ciphertext c, limb i
template <int LOGN>
NTT_KERNEL(LOGN) void k_encrypt(const int64_t* __restrict__ msg, const double* __restrict__ sk, uint64_t seed0,
                                 int lv, double* __restrict__ ct_all, double* const* __restrict__ ct_tab, DevTabs tb) {
  constexpr int N = 1 << LOGN;
  NTT_LDS(LOGN);
  const int i = blockIdx.x % (lv + 1), c = blockIdx.x / (lv + 1);
  double* ct = ct_tab ? ct_tab[c] : ct_all + (size_t)c * 2 * (lv + 1) * N;
  const ModQ m = tb.mods[i];
  double* c0 = ct + (size_t)i * N;
  double* c1 = ct + (size_t)(lv + 1 + i) * N;
  encrypt_a<LOGN>(s, seed0 + (uint64_t)c, i, tb, [&](int t, double v) { c1[t] = v; });
  const double* sk_i = sk + (size_t)i * N;
  // slot t of a is read back from what this thread wrote above
  encrypt_message<LOGN>(s, msg + (size_t)c * N, seed0 + (uint64_t)c, kStreamEncE, i, tb,
                        [&](int t, double v) { c0[t] = reduce(v - mulmod(c1[t], sk_i[t], m), m); });
}

// Few ciphertexts: block (c, i, h) makes one of the two transforms, into the
// half h of the ciphertext, and k_encrypt_join subtracts a s.  The sampling
// and the transform of a limb on one CU are the whole time, so the two halves
// side by side take half of it.  One ciphertext at 2^12 / 2^14 / 2^15: 19 ->
// 9 + 2, 54 -> 23 + 3, 127 -> 53 + 15 us (of it 4 / 9 / 10 through
// sample_coeffs).
template <int LOGN>
NTT_KERNEL(LOGN) void k_encrypt_half(const int64_t* __restrict__ msg, uint64_t seed0, int lv, double* __restrict__ ct_all,
                                     double* const* __restrict__ ct_tab, DevTabs tb) {
  constexpr int N = 1 << LOGN;
  NTT_LDS(LOGN);
  const int h = blockIdx.x & 1, b = blockIdx.x >> 1, i = b % (lv + 1), c = b / (lv + 1);
  double* ct = ct_tab ? ct_tab[c] : ct_all + (size_t)c * 2 * (lv + 1) * N;
  double* o = ct + (size_t)(h * (lv + 1) + i) * N;
  if (h)
    encrypt_a<LOGN>(s, seed0 + (uint64_t)c, i, tb, [&](int t, double v) { o[t] = v; });
  else
    encrypt_message<LOGN>(s, msg + (size_t)c * N, seed0 + (uint64_t)c, kStreamEncE, i, tb,
                          [&](int t, double v) { o[t] = v; });
}
// grid (N / 256, limbs, ciphertexts)
__global__ __launch_bounds__(256) void k_encrypt_join(const double* __restrict__ sk, int lv, int N,
                                                      double* __restrict__ ct_all, double* const* __restrict__ ct_tab,
                                                      const ModQ* __restrict__ mods) {
  const int i = blockIdx.y, c = blockIdx.z;
  const size_t t = (size_t)i * N + blockIdx.x * 256 + threadIdx.x;
  double* ct = ct_tab ? ct_tab[c] : ct_all + (size_t)c * 2 * (lv + 1) * N;
  const ModQ m = mods[i];
  ct[t] = reduce(ct[t] - mulmod(ct[(size_t)(lv + 1) * N + t], sk[t], m), m);
}

// public key: block i (limb i < nl): a uniform, b = -a s + e (Sec. 2.2, the
// public-key form of RLWE encryption)
template <int LOGN>
NTT_KERNEL(LOGN) void k_pk_gen(const double* __restrict__ sk, uint64_t seed, int nl, double* __restrict__ pk, DevTabs tb) {
  constexpr int N = 1 << LOGN;
  NTT_LDS(LOGN);
  const int i = blockIdx.x;
  const ModQ m = tb.mods[i];
  const uint64_t qi = (uint64_t)m.q;
  double* b = pk + (size_t)i * N;
  double* a = pk + (size_t)(nl + i) * N;
  ntt_fwd_out<LOGN>(s, [&](int j) { return sample_uniform_res(seed, kStreamPkA | (uint64_t)i, j, qi); },
                    tb.fwd_tw + (size_t)i * N, m, [&](int t, double v) { a[t] = v; });
  const double* sk_i = sk + (size_t)i * N;
  // slot t of a is read back from what this thread wrote above
  ntt_fwd_out<LOGN>(s, [&](int j) { return (double)sample_cbd21(seed, kStreamPkE, (uint64_t)j); },
                    tb.fwd_tw + (size_t)i * N, m,
                    [&](int t, double v) { b[t] = reduce(v - mulmod(a[t], sk_i[t], m), m); });
}

// public-key encryption of integer coefficients m at level lv: v ternary,
// c0 = v b + m + e0, c1 = v a + e1; ciphertext c uses seed + c.  Block (c, i):
// ciphertext c, limb i, three transforms.  Few ciphertexts (SPLIT): block
// (c, i, h) makes half h of the ciphertext and transforms v for itself, two
// transforms in a row instead of three: one ciphertext at 2^13 45 -> 26 us.
template <int LOGN, bool SPLIT>
NTT_KERNEL(LOGN) void k_encrypt_pk(const int64_t* __restrict__ msg, const double* __restrict__ pk, int pk_nl,
                                    uint64_t seed0, int lv, double* __restrict__ ct_all, DevTabs tb) {
  constexpr int N = 1 << LOGN;
  NTT_LDS(LOGN);
  const int b = SPLIT ? blockIdx.x >> 1 : blockIdx.x, i = b % (lv + 1), c = b / (lv + 1);
  const bool h0 = !SPLIT || !(blockIdx.x & 1), h1 = !SPLIT || (blockIdx.x & 1);
  const uint64_t seed = seed0 + (uint64_t)c;
  double* ct = ct_all + (size_t)c * 2 * (lv + 1) * N;
  const ModQ m = tb.mods[i];
  const double* tw = tb.fwd_tw + (size_t)i * N;
  double* c0 = ct + (size_t)i * N;
  double* c1 = ct + (size_t)(lv + 1 + i) * N;
  const double* kb = pk + (size_t)i * N;
  const double* ka = pk + (size_t)(pk_nl + i) * N;
  // v in the evaluation domain, parked in the last half that needs it; every
  // later read of slot t is by the thread that wrote it
  double* vt = h1 ? c1 : c0;
  double x[NttShape<LOGN>::PER];
  sample_coeffs<LOGN>(seed, kStreamPkV, x, [&](uint64_t u, int) { return (double)ternary(u); });
  ntt_fwd_regs_out<LOGN>(s, x, tw, m, [&](int t, double v) { vt[t] = v; });
  if (h0)
    encrypt_message<LOGN>(s, msg + (size_t)c * N, seed, kStreamPkE0, i, tb,
                          [&](int t, double v) { c0[t] = reduce(v + mulmod(vt[t], kb[t], m), m); });
  if (h1) {
    sample_coeffs<LOGN>(seed, kStreamPkE1, x, [&](uint64_t u, int) { return (double)cbd21(u); });
    ntt_fwd_regs_out<LOGN>(s, x, tw, m, [&](int t, double v) { c1[t] = reduce(v + mulmod(c1[t], ka[t], m), m); });
  }
}

// Slot pairs of c0 + c1 s whose loads a thread has in flight, three a slot.  At 2^14 one
// pair: all at once read 48 rows side by side, whose strides are powers of two where the
// limb count is, and with every CU at it 128 ciphertexts of 2 / 4 / 3 limbs took 37 /
// 71 / 55 us instead of 30 / 58 / 51 (one ciphertext 19 either way).  Smaller limbs read
// shorter rows, several workgroups to a CU: there all at once is as fast for many and
// faster for one (the exchange of 16 x 256 at 2^12 66.6 against 67.3 us).
template <int LOGN>
constexpr int kDecryptFlight = LOGN == 14 ? 1 : 8;

// c0 + c1 s -> canonical coefficient residues (uint64), block i = limb i
template <int LOGN>
NTT_KERNEL(LOGN) void k_decrypt_u64(const double* __restrict__ ct, const double* __restrict__ sk, int lv,
                                     uint64_t* __restrict__ out, DevTabs tb) {
  constexpr int N = 1 << LOGN;
  NTT_LDS(LOGN);
  const int i = blockIdx.x;
  const ModQ m = tb.mods[i];
  const double* c0 = ct + (size_t)i * N;
  const double* c1 = ct + (size_t)(lv + 1 + i) * N;
  const double* sk_i = sk + (size_t)i * N;
  uint64_t* dst = out + (size_t)i * N;
  ntt_inv_in<LOGN, kDecryptFlight<LOGN>>(s, [&](int t) { return c0[t] + mulmod(c1[t], sk_i[t], m); }, tb.inv_tw + (size_t)i * N,
                   m, tb.ninv[i], [&](int j, double v) { dst[j] = f64_to_u64(canon(v, m)); });
}

// c0 + c1 s -> canonical coefficient residues (binary64), for the CRT decoder;
// block (c, i) = ciphertext c, limb i
template <int LOGN>
NTT_KERNEL(LOGN) void k_decrypt_f64(const double* __restrict__ ct, const double* const* __restrict__ ct_tab,
                                     const double* __restrict__ sk, int lv, double* __restrict__ out, DevTabs tb) {
  constexpr int N = 1 << LOGN;
  NTT_LDS(LOGN);
  const int i = blockIdx.x % (lv + 1), c = blockIdx.x / (lv + 1);
  const ModQ m = tb.mods[i];
  const double* base = ct_tab ? ct_tab[c] : ct + (size_t)c * 2 * (lv + 1) * N;
  const double* c0 = base + (size_t)i * N;
  const double* c1 = base + (size_t)(lv + 1 + i) * N;
  const double* sk_i = sk + (size_t)i * N;
  double* dst = out + ((size_t)c * (lv + 1) + i) * N;
  ntt_inv_in<LOGN, kDecryptFlight<LOGN>>(s, [&](int t) { return c0[t] + mulmod(c1[t], sk_i[t], m); }, tb.inv_tw + (size_t)i * N,
                   m, tb.ninv[i], [&](int j, double v) { dst[j] = canon(v, m); });
}

// Rotation (Galois) keys.  Block = (key kk, digit j, limb r of Q_L u P):
//   a uniform (coefficient domain) -> NTT;  b = -a s + e_j + [r in D_j] P phi_g(s)
// with phi_g(s) read as an orbit shift of the transformed secret.
// Layout: keys[kk][j][0 = b | 1 = a][r][N].
template <int LOGN>
NTT_KERNEL(LOGN) void k_rotkey_gen(const double* __restrict__ sk, RotKeyList list, uint64_t seed, RotKeyArgs ka,
                                    double* __restrict__ keys, DevTabs tb) {
  constexpr int N = 1 << LOGN;
  NTT_LDS(LOGN);
  const int nlimb = ka.n_limbs;
  const int r = blockIdx.x % nlimb;
  const int j = (blockIdx.x / nlimb) % ka.beta;
  const int kk = blockIdx.x / (nlimb * ka.beta);
  const ModQ m = tb.mods[r];  // limbs of Q_L u P are exactly the context's prime order
  const uint64_t g = list.galois[kk];
  const int rot = list.rot[kk];
  const uint64_t sa = kStreamKeyA | ((uint64_t)j << 40) | ((uint64_t)r << 24) | g;
  const uint64_t se = kStreamKeyE | ((uint64_t)j << 40) | g;
  double* kb = keys + ((((size_t)kk * ka.beta + j) * 2 + 0) * nlimb + r) * N;
  double* kaout = keys + ((((size_t)kk * ka.beta + j) * 2 + 1) * nlimb + r) * N;
  ntt_fwd_out<LOGN>(s, [&](int k) { return sample_uniform_res(seed, sa, k, (uint64_t)m.q); },
                    tb.fwd_tw + (size_t)r * N, m, [&](int t, double v) { kaout[t] = v; });
  const double* sk_r = sk + (size_t)r * N;
  const bool in_digit = (r < ka.n_q) && (r / ka.alpha == j);
  const double pmod = ka.P_mod[r];
  const int half = N / 2;
  // b = e - a s (+ P phi_g(s) on the digit's own limbs); a read back from this thread's writes
  ntt_fwd_out<LOGN>(s, [&](int k) { return (double)sample_cbd21(seed, se, (uint64_t)k); }, tb.fwd_tw + (size_t)r * N,
                    m, [&](int t, double e) {
                      double v = e - mulmod(kaout[t], sk_r[t], m);
                      if (in_digit) v += mulmod(pmod, sk_r[orbit_shift(t, rot, half)], m);
                      kb[t] = reduce(v, m);
                    });
}

// ---------------------------------------------------------------------------
// ModUp (hoisted once per input ciphertext).  Input ciphertext c of a batch
// is at ct + c*ct_stride; its digits go to digits + c*dig_stride.
// step 1: INTT of every limb of c1; y_i = [x_i * (Q_j/q_i)^-1]_{q_i} (canonical)
// step 2: per (digit j, target limb r not in D_j):
//         Conv = sum_{i in D_j} y_i [Q_j/q_i]_r  -> NTT -> digits[j][r]
// ---------------------------------------------------------------------------
template <int LOGN>
NTT_KERNEL(LOGN) void k_modup_intt(const double* __restrict__ ct, const double* const* __restrict__ ct_tab,
                                    size_t ct_stride, int lv, const KsLevel* __restrict__ kl, double* __restrict__ y,
                                    DevTabs tb) {
  constexpr int N = 1 << LOGN;
  NTT_LDS(LOGN);
  const int i = blockIdx.x % (lv + 1), c = blockIdx.x / (lv + 1);
  const ModQ m = tb.mods[i];
  const double* c1 = (ct_tab ? ct_tab[c] : ct + (size_t)c * ct_stride) + (size_t)(lv + 1 + i) * N;
  const double ih = kl->up_inv_hat[i];
  double* dst = y + ((size_t)c * (lv + 1) + i) * N;
  ntt_inv_in<LOGN>(s, [&](int t) { return c1[t]; }, tb.inv_tw + (size_t)i * N, m, tb.ninv[i],
                   [&](int j, double v) { dst[j] = canon(mulmod(canon(v, m), ih, m), m); });
}

template <int LOGN>
NTT_KERNEL(LOGN) void k_modup_conv(const double* __restrict__ y, const double* __restrict__ ct,
                                    const double* const* __restrict__ ct_tab, size_t ct_stride,
                                    const KsLevel* __restrict__ kl, double* __restrict__ digits, size_t dig_stride,
                                    DevTabs tb) {
  constexpr int N = 1 << LOGN, T = NttShape<LOGN>::T;
  NTT_LDS(LOGN);
  const int nt = kl->n_tasks;
  const KsTask& task = kl->up_task[blockIdx.x % nt];  // by reference: a copy indexed at run time would go to scratch memory
  const int nsrc = task.nsrc, src0 = task.src0;
  const int c = blockIdx.x / nt;
  const int K = kl->K, lv = kl->lv;
  const int pi = task.prime;
  const ModQ m = tb.mods[pi];
  double* dst = digits + (size_t)c * dig_stride + ((size_t)task.digit * K + task.limb) * N;
  if (nsrc == 0) {  // limb of the digit itself: residues kept as they are
    const double* src = (ct_tab ? ct_tab[c] : ct + (size_t)c * ct_stride) + (size_t)(lv + 1 + task.limb) * N;
    for (int t = threadIdx.x; t < N; t += T) dst[t] = src[t];
    return;
  }
  double x[NttShape<LOGN>::PER];
  convert_coeffs<LOGN>(gmem(y + (size_t)(c * (lv + 1) + src0) * N), nsrc, [&](int u) { return task.hat[u]; }, 0.0, m, x);
  ntt_fwd_regs_out<LOGN>(s, x, tb.fwd_tw + (size_t)pi * N, m, [&](int t, double v) { dst[t] = v; });
}

// Both steps in one launch for alpha = 1 (a digit is one limb): every target
// limb's workgroup makes the source limb's inverse transform again.  Where the
// transforms leave CUs idle the repeated work costs nothing and one launch with
// its memory round trip is saved (see fuse_transforms).
template <int LOGN>
NTT_KERNEL(LOGN) void k_modup_one(const double* __restrict__ ct, const double* const* __restrict__ ct_tab,
                                   size_t ct_stride, const KsLevel* __restrict__ kl, double* __restrict__ digits,
                                   size_t dig_stride, DevTabs tb) {
  static_assert(LOGN <= 14, "one LDS-resident limb");
  constexpr int N = 1 << LOGN, T = NttShape<LOGN>::T;
  NTT_LDS(LOGN);
  const int nt = kl->n_tasks;
  const KsTask& task = kl->up_task[blockIdx.x % nt];
  const int c = blockIdx.x / nt, lv = kl->lv, pi = task.prime;
  const double* c1 = (ct_tab ? ct_tab[c] : ct + (size_t)c * ct_stride) + (size_t)(lv + 1) * N;
  double* dst = digits + (size_t)c * dig_stride + ((size_t)task.digit * kl->K + task.limb) * N;
  const double* src = c1 + (size_t)task.src0 * N;
  if (task.nsrc == 0) {  // limb of the digit itself: residues kept as they are
    for (int t = threadIdx.x; t < N; t += T) dst[t] = src[t];
    return;
  }
  double x[16];
  modup_source<LOGN>(s, [&](int t) { return src[t]; }, task, tb, x);
  ntt_fwd_regs_out<LOGN>(s, x, tb.fwd_tw + (size_t)pi * N, tb.mods[pi], [&](int t, double v) { dst[t] = v; });
}

// The same with each limb on N / 2^12 workgroups (SplitNtt): the inverses'
// blocks of every source limb, then the blocks of every target limb.
#define SPLIT_KERNEL __global__ __launch_bounds__(256)
template <int LOGN>
SPLIT_KERNEL void k_modup_split_inv(const double* __restrict__ ct, const double* const* __restrict__ ct_tab,
                                    size_t ct_stride, int lv, double* __restrict__ y, DevTabs tb) {
  using Sp = SplitNtt<LOGN>;
  __shared__ double s[Sp::LDS];
  const int h = blockIdx.x % Sp::S, b = blockIdx.x / Sp::S, i = b % (lv + 1), c = b / (lv + 1);
  const double* src = (ct_tab ? ct_tab[c] : ct + (size_t)c * ct_stride) + (size_t)(lv + 1 + i) * Sp::N;
  split_inverse<LOGN>(s, h, [&](int t) { return src[t]; }, i, tb, y + (size_t)b * Sp::N);
}
template <int LOGN>
SPLIT_KERNEL void k_modup_split(const double* __restrict__ y, const double* __restrict__ ct,
                                const double* const* __restrict__ ct_tab, size_t ct_stride,
                                const KsLevel* __restrict__ kl, double* __restrict__ digits, size_t dig_stride, DevTabs tb) {
  using Sp = SplitNtt<LOGN>;
  constexpr int N = Sp::N;
  __shared__ double s[Sp::LDS];
  const int nt = kl->n_tasks, h = blockIdx.x % Sp::S, b = blockIdx.x / Sp::S;
  const KsTask& task = kl->up_task[b % nt];
  const int c = b / nt, lv = kl->lv;
  double* dst = digits + (size_t)c * dig_stride + ((size_t)task.digit * kl->K + task.limb) * N;
  if (task.nsrc == 0) {  // limb of the digit itself: residues kept as they are
    const double* src = (ct_tab ? ct_tab[c] : ct + (size_t)c * ct_stride) + (size_t)(lv + 1 + task.src0) * N;
#pragma unroll
    for (int w = 0; w < 16; ++w) dst[h * 4096 + threadIdx.x + w * 256] = src[h * 4096 + threadIdx.x + w * 256];
    return;
  }
  split_modup<LOGN>(s, h, gmem(y + (size_t)(c * (lv + 1) + task.src0) * N), task, tb, dst);
}

// ---------------------------------------------------------------------------
// ModDown Q_l u P -> Q_l with coefficient-wise rounding, on `npoly` polys
// stored [npoly][K][N] (evaluation domain); output [npoly][l+1][N].
// step 1 (P limbs): INTT, add floor(P/2), y_k = [x_k (P/p_k)^-1]_{p_k}
// step 2 (Q limbs): t_i = Conv_{P->q_i}(y) - floor(P/2) (coefficient domain)
//                   -> NTT -> out_i = (u_i - t_i) * P^-1 mod q_i
// ---------------------------------------------------------------------------
template <int LOGN>
NTT_KERNEL(LOGN) void k_moddown_p(const double* __restrict__ u, const KsLevel* __restrict__ kl,
                                   double* __restrict__ y, DevTabs tb) {
  constexpr int N = 1 << LOGN;
  NTT_LDS(LOGN);
  const int alpha = kl->alpha, K = kl->K, lv = kl->lv;
  const int k = blockIdx.x % alpha, x = blockIdx.x / alpha;
  const int pi = kl->n_q_total + k;
  const ModQ m = tb.mods[pi];
  const double* src = u + ((size_t)x * K + lv + 1 + k) * N;
  const double h = kl->down_half[lv + 1 + k];
  const double ih = kl->down_inv_hat[k];
  double* dst = y + ((size_t)x * alpha + k) * N;
  ntt_inv_in<LOGN>(s, [&](int t) { return src[t]; }, tb.inv_tw + (size_t)pi * N, m, tb.ninv[pi],
                   [&](int c, double v) { dst[c] = canon(mulmod(canon(v + h, m), ih, m), m); });
}

template <int LOGN>
NTT_KERNEL(LOGN) void k_moddown_q(const double* __restrict__ u, const double* __restrict__ y,
                                   const KsLevel* __restrict__ kl, double* __restrict__ out,
                                   double* const* __restrict__ out_tab, DevTabs tb) {
  constexpr int N = 1 << LOGN;
  NTT_LDS(LOGN);
  const int alpha = kl->alpha, K = kl->K, lv = kl->lv;
  const int i = blockIdx.x % (lv + 1), x = blockIdx.x / (lv + 1);
  const ModQ m = tb.mods[i];
  const double h = kl->down_half[i];
  const double* yx = y + (size_t)x * alpha * N;
  const double pinv = kl->down_pinv[i];
  const double* ui = u + ((size_t)x * K + i) * N;
  double* oi = out_tab ? out_tab[x >> 1] + ((size_t)(x & 1) * (lv + 1) + i) * N : out + ((size_t)x * (lv + 1) + i) * N;
  double c[NttShape<LOGN>::PER];
  auto conv = [&] {
    convert_coeffs<LOGN>(gmem(yx), alpha, [&](int k) { return kl->down_hat[k * kMaxLimbs + i]; }, h, m, c);
  };
  if constexpr (LOGN <= 14) {
    constexpr int T = NttShape<LOGN>::T;
    double v[16], uv[16];  // u loaded before the transform: one memory latency instead of eight
#pragma unroll
    for (int w = 0; w < 16; ++w) uv[w] = ui[(int)opaque_tid() + (w >> 1) * T + (w & 1) * (N / 2)];
    conv();
    ntt_fwd_regs<LOGN>(s, c, tb.fwd_tw + (size_t)i * N, m);
    slots_from_lds<LOGN>(s, v);
#pragma unroll
    for (int w = 0; w < 16; ++w)
      oi[(int)opaque_tid() + (w >> 1) * T + (w & 1) * (N / 2)] = reduce(mulmod(uv[w] - v[w], pinv, m), m);
  } else {
    conv();
    ntt_fwd_regs_out<LOGN>(s, c, tb.fwd_tw + (size_t)i * N, m,
                           [&](int t, double v) { oi[t] = reduce(mulmod(ui[t] - v, pinv, m), m); });
  }
}

// Both steps in one launch for alpha = 1, as k_modup_one
template <int LOGN>
NTT_KERNEL(LOGN) void k_moddown_one(const double* __restrict__ u, const KsLevel* __restrict__ kl, double* __restrict__ out,
                                     double* const* __restrict__ out_tab, DevTabs tb) {
  static_assert(LOGN <= 14, "one LDS-resident limb");
  constexpr int N = 1 << LOGN, T = NttShape<LOGN>::T;
  NTT_LDS(LOGN);
  const int K = kl->K, lv = kl->lv;
  const int i = blockIdx.x % (lv + 1), x = blockIdx.x / (lv + 1);
  const double* up = u + ((size_t)x * K + lv + 1) * N;
  const double* ui = u + ((size_t)x * K + i) * N;
  double* oi = out_tab ? out_tab[x >> 1] + ((size_t)(x & 1) * (lv + 1) + i) * N : out + ((size_t)x * (lv + 1) + i) * N;
  double uv[16];
#pragma unroll
  for (int w = 0; w < 16; ++w) uv[w] = ui[(int)opaque_tid() + (w >> 1) * T + (w & 1) * (N / 2)];
  moddown_limb<LOGN>(s, [&](int t) { return up[t]; }, uv, i, kl, tb, [&](int t, double v) { oi[t] = v; });
}

// Each limb on N / 2^12 workgroups, as k_modup_split
template <int LOGN>
SPLIT_KERNEL void k_moddown_split_inv(const double* __restrict__ u, const KsLevel* __restrict__ kl, double* __restrict__ y,
                                      DevTabs tb) {
  using Sp = SplitNtt<LOGN>;
  __shared__ double s[Sp::LDS];
  const int h = blockIdx.x % Sp::S, x = blockIdx.x / Sp::S;
  const double* src = u + ((size_t)x * kl->K + kl->lv + 1) * Sp::N;
  split_inverse<LOGN>(s, h, [&](int t) { return src[t]; }, kl->n_q_total, tb, y + (size_t)x * Sp::N);
}
template <int LOGN>
SPLIT_KERNEL void k_moddown_split(const double* __restrict__ u, const double* __restrict__ y, const KsLevel* __restrict__ kl,
                                  double* __restrict__ out, double* const* __restrict__ out_tab, DevTabs tb) {
  using Sp = SplitNtt<LOGN>;
  constexpr int N = Sp::N;
  __shared__ double s[Sp::LDS];
  const int lv = kl->lv, h = blockIdx.x % Sp::S, b = blockIdx.x / Sp::S, i = b % (lv + 1), x = b / (lv + 1);
  double* oi = out_tab ? out_tab[x >> 1] + ((size_t)(x & 1) * (lv + 1) + i) * N : out + ((size_t)x * (lv + 1) + i) * N;
  split_moddown<LOGN>(s, h, gmem(u + ((size_t)x * kl->K + i) * N), gmem(y + (size_t)x * N), i, kl, tb, oi);
}

// Rescale by q_lv (drop the last limb, coefficient-wise rounding) on polys
// x = 2 pair + half, limbs [lv+1][N] at in + pair in_stride + half (lv+1) N,
// out [x][lv][N].  Same formula as ModDown with P = q_lv.  With pt, the input
// is ct * pt (pt at pt + pair pt_stride): the product never goes to memory.
template <int LOGN>
NTT_KERNEL(LOGN) void k_rescale(const double* __restrict__ in, size_t in_stride, const double* __restrict__ pt,
                                 size_t pt_stride, int lv, const RescaleArgs ra, double* __restrict__ out, DevTabs tb) {
  constexpr int N = 1 << LOGN, PER = NttShape<LOGN>::PER, T = NttShape<LOGN>::T;
  NTT_LDS(LOGN);
  const int i = blockIdx.x % lv, x = blockIdx.x / lv;
  const ModQ ml = tb.mods[lv];
  const ModQ m = tb.mods[i];
  const double* poly = in + (size_t)(x >> 1) * in_stride + (size_t)(x & 1) * (lv + 1) * N;
  const double* pp = pt ? pt + (size_t)(x >> 1) * pt_stride : nullptr;
  // INTT of the dropped limb (every block recomputes it; the limb is L2-resident)
  const double* last = poly + (size_t)lv * N;
  const double* plast = pp + (size_t)lv * N;
  double c[PER];
  if (pp)
    ntt_inv_in_regs<LOGN>(s, [&](int t) { return mulmod(last[t], plast[t], ml); }, tb.inv_tw + (size_t)lv * N,
                          ml, tb.ninv[lv], c);
  else
    ntt_inv_in_regs<LOGN>(s, [&](int t) { return last[t]; }, tb.inv_tw + (size_t)lv * N, ml, tb.ninv[lv], c);
  const double hl = ra.half_mod_last, hi = ra.half_mod[i];
  // [c + h]_{q_l} lifted to q_i, minus h mod q_i
#pragma unroll
  for (int w = 0; w < PER; ++w) c[w] = reduce(canon(c[w] + hl, ml) - hi, m);
  const double inv = ra.inv_last[i];
  const double* ui = poly + (size_t)i * N;
  const double* pi = pp + (size_t)i * N;
  double* oi = out + ((size_t)x * lv + i) * N;
  if constexpr (LOGN <= 14) {
    double u[16], v[16];  // loaded before the transform: one memory latency instead of eight
#pragma unroll
    for (int w = 0; w < 16; ++w) {
      const int t = (int)opaque_tid() + (w >> 1) * T + (w & 1) * (N / 2);
      u[w] = pp ? mulmod(ui[t], pi[t], m) : ui[t];
    }
    ntt_fwd_regs<LOGN>(s, c, tb.fwd_tw + (size_t)i * N, m);
    slots_from_lds<LOGN>(s, v);
#pragma unroll
    for (int w = 0; w < 16; ++w)
      oi[(int)opaque_tid() + (w >> 1) * T + (w & 1) * (N / 2)] = reduce(mulmod(u[w] - v[w], inv, m), m);
  } else {
    ntt_fwd_regs_out<LOGN>(s, c, tb.fwd_tw + (size_t)i * N, m, [&](int t, double v) {
      const double u = pp ? mulmod(ui[t], pi[t], m) : ui[t];
      oi[t] = reduce(mulmod(u - v, inv, m), m);
    });
  }
}

// sum n partials: part[n][2][K][N] -> acc[2][K][N]
__global__ __launch_bounds__(256) void k_sum_partials(const double* __restrict__ part, int n, int K, int N,
                                                       LimbMap limb_prime, const ModQ* __restrict__ mods,
                                                       double* __restrict__ acc) {
  const size_t idx = (size_t)blockIdx.x * 256 + threadIdx.x;
  const size_t tot = (size_t)2 * K * N;
  if (idx >= tot) return;
  const int r = (int)((idx / N) % K);
  const ModQ m = mods[limb_prime.idx[r]];
  double v = 0.0;
  int c = 0;
  for (; c + 4 <= n; c += 4) {  // four loads in flight; |v| < 4.5 q between re-centrings
    double t[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) t[u] = part[(size_t)(c + u) * tot + idx];
    v = reduce(v + t[0] + t[1] + t[2] + t[3], m);
  }
  for (; c < n; ++c) v += part[(size_t)c * tot + idx];
  acc[idx] = reduce(v, m);
}

// P * (c0, c1) on the Q limbs, [2][lv+1][N]
__global__ __launch_bounds__(256) void k_scale_by_p(const double* __restrict__ ct, const double* const* __restrict__ ct_tab,
                                                    int lv, int N, const double* __restrict__ pmod,
                                                    const ModQ* __restrict__ mods, double* __restrict__ out) {
  const size_t idx = (size_t)blockIdx.x * 256 + threadIdx.x;
  const size_t tot = (size_t)2 * (lv + 1) * N;
  if (idx >= tot) return;
  const int c = blockIdx.y;
  const double* src = ct_tab ? ct_tab[c] : ct + (size_t)c * tot;
  const int i = (int)((idx / N) % (lv + 1));
  out[(size_t)c * tot + idx] = reduce(mulmod(src[idx], pmod[i], mods[i]), mods[i]);
}

// ---------------------------------------------------------------------------
// element-wise ciphertext operations (evaluation domain)
// ---------------------------------------------------------------------------
// out[x][i] = in[x][i] * pt[i] for x in {0,1}; pt has >= lv+1 limbs
__global__ __launch_bounds__(256) void k_ct_mul_pt(const double* __restrict__ ct, const double* __restrict__ pt, int lv, int N,
                                                   const ModQ* __restrict__ mods, double* __restrict__ out) {
  const size_t idx = (size_t)blockIdx.x * 256 + threadIdx.x;
  const size_t tot = (size_t)2 * (lv + 1) * N;
  if (idx >= tot) return;
  const size_t within = idx % ((size_t)(lv + 1) * N);
  const int i = (int)(within / N);
  out[idx] = mulmod(ct[idx], pt[within], mods[i]);
}

__global__ __launch_bounds__(256) void k_ct_add(const double* __restrict__ a, const double* __restrict__ b, int lv, int N,
                                                const ModQ* __restrict__ mods, double* __restrict__ out) {
  const size_t idx = (size_t)blockIdx.x * 256 + threadIdx.x;
  const size_t tot = (size_t)2 * (lv + 1) * N;
  if (idx >= tot) return;
  const int i = (int)((idx / N) % (lv + 1));
  out[idx] = reduce(a[idx] + b[idx], mods[i]);
}

// ---------------------------------------------------------------------------
// host-side launchers
// ---------------------------------------------------------------------------
template <int LOGN>
static void launch_ntt_all(const LaunchCtx& L, NttOp op, const void* in, void* out, int nblocks, LimbMap map) {
  const dim3 grid(nblocks), block(NttShape<LOGN>::T);
  switch (op) {
    case NttOp::Fwd: hipLaunchKernelGGL(k_ntt_fwd<LOGN>, grid, block, 0, L.stream, (const double*)in, (double*)out, map, L.tb); break;
    case NttOp::Inv: hipLaunchKernelGGL(k_ntt_inv<LOGN>, grid, block, 0, L.stream, (const double*)in, (double*)out, map, L.tb); break;
    case NttOp::ImportI64:
      if constexpr (LOGN <= 14)  // one workgroup per polynomial (nblocks = polynomials x limbs)
        hipLaunchKernelGGL(k_import_i64_poly<LOGN>, dim3(nblocks / map.n), block, 0, L.stream, (const int64_t*)in,
                           (double*)out, map, L.tb);
      else
        hipLaunchKernelGGL(k_import_i64<LOGN>, grid, block, 0, L.stream, (const int64_t*)in, (double*)out, map, L.tb);
      break;
    case NttOp::ExportU64:
      if constexpr (LOGN <= 14)  // one workgroup per polynomial (nblocks = polynomials x limbs)
        hipLaunchKernelGGL(k_export_u64_poly<LOGN>, dim3(nblocks / map.n), block, 0, L.stream, (const double*)in,
                           (uint64_t*)out, map, L.tb);
      else
        hipLaunchKernelGGL(k_export_u64<LOGN>, grid, block, 0, L.stream, (const double*)in, (uint64_t*)out, map, L.tb);
      break;
  }
}

#define DISPATCH_LOGN(L, FN, ...)                         \
  switch ((L).logN) {                                     \
    case 12: FN<12>(__VA_ARGS__); break;                  \
    case 13: FN<13>(__VA_ARGS__); break;                  \
    case 14: FN<14>(__VA_ARGS__); break;                  \
    case 15: FN<15>(__VA_ARGS__); break;                  \
    default: return hipErrorInvalidValue;                 \
  }

hipError_t launch_ntt(const LaunchCtx& L, NttOp op, const void* in, void* out, int nblocks, LimbMap map) {
  if (nblocks <= 0) return hipSuccess;
  DISPATCH_LOGN(L, launch_ntt_all, L, op, in, out, nblocks, map);
  return hipGetLastError();
}

template <int LOGN>
static void keygen_impl(const LaunchCtx& L, uint64_t seed, double* sk, int n_mod) {
  hipLaunchKernelGGL(k_keygen<LOGN>, dim3(n_mod), dim3(NttShape<LOGN>::T), 0, L.stream, seed, sk, L.tb);
}
hipError_t launch_keygen(const LaunchCtx& L, uint64_t seed, double* sk, int n_mod) {
  DISPATCH_LOGN(L, keygen_impl, L, seed, sk, n_mod);
  return hipGetLastError();
}

template <int LOGN>
static void pk_gen_impl(const LaunchCtx& L, const double* sk, uint64_t seed, int nl, double* pk) {
  hipLaunchKernelGGL(k_pk_gen<LOGN>, dim3(nl), dim3(NttShape<LOGN>::T), 0, L.stream, sk, seed, nl, pk, L.tb);
}
hipError_t launch_pk_gen(const LaunchCtx& L, const double* sk, uint64_t seed, int nl, double* pk) {
  DISPATCH_LOGN(L, pk_gen_impl, L, sk, seed, nl, pk);
  return hipGetLastError();
}
template <int LOGN>
static void encrypt_pk_impl(const LaunchCtx& L, const int64_t* msg, int nct, const double* pk, int pk_nl, uint64_t seed,
                            int lv, double* ct) {
  const dim3 block(NttShape<LOGN>::T);
  if (few_transforms(2 * nct * (lv + 1)))
    hipLaunchKernelGGL((k_encrypt_pk<LOGN, true>), dim3(2 * nct * (lv + 1)), block, 0, L.stream, msg, pk, pk_nl, seed, lv,
                       ct, L.tb);
  else
    hipLaunchKernelGGL((k_encrypt_pk<LOGN, false>), dim3(nct * (lv + 1)), block, 0, L.stream, msg, pk, pk_nl, seed, lv, ct,
                       L.tb);
}
hipError_t launch_encrypt_pk(const LaunchCtx& L, const int64_t* msg, int nct, const double* pk, int pk_nl,
                             uint64_t seed, int lv, double* ct) {
  if (nct <= 0) return hipSuccess;
  DISPATCH_LOGN(L, encrypt_pk_impl, L, msg, nct, pk, pk_nl, seed, lv, ct);
  return hipGetLastError();
}

template <int LOGN>
static void encrypt_impl(const LaunchCtx& L, const int64_t* msg, int nct, const double* sk, uint64_t seed, int lv,
                         double* ct, double* const* ct_tab) {
  const dim3 block(NttShape<LOGN>::T);
  if (few_transforms(2 * nct * (lv + 1))) {
    hipLaunchKernelGGL(k_encrypt_half<LOGN>, dim3(2 * nct * (lv + 1)), block, 0, L.stream, msg, seed, lv, ct, ct_tab, L.tb);
    hipLaunchKernelGGL(k_encrypt_join, dim3((1 << LOGN) / 256, lv + 1, nct), dim3(256), 0, L.stream, sk, lv, 1 << LOGN, ct,
                       ct_tab, L.tb.mods);
  } else {
    hipLaunchKernelGGL(k_encrypt<LOGN>, dim3(nct * (lv + 1)), block, 0, L.stream, msg, sk, seed, lv, ct, ct_tab, L.tb);
  }
}
hipError_t launch_encrypt(const LaunchCtx& L, const int64_t* msg, int nct, const double* sk, uint64_t seed, int lv,
                          double* ct, double* const* ct_tab) {
  if (nct <= 0) return hipSuccess;
  DISPATCH_LOGN(L, encrypt_impl, L, msg, nct, sk, seed, lv, ct, ct_tab);
  return hipGetLastError();
}

template <int LOGN>
static void decrypt_u64_impl(const LaunchCtx& L, const double* ct, const double* sk, int lv, uint64_t* out) {
  hipLaunchKernelGGL(k_decrypt_u64<LOGN>, dim3(lv + 1), dim3(NttShape<LOGN>::T), 0, L.stream, ct, sk, lv, out, L.tb);
}
hipError_t launch_decrypt_u64(const LaunchCtx& L, const double* ct, const double* sk, int lv, uint64_t* out) {
  DISPATCH_LOGN(L, decrypt_u64_impl, L, ct, sk, lv, out);
  return hipGetLastError();
}

template <int LOGN>
static void decrypt_f64_impl(const LaunchCtx& L, const double* ct, const double* const* ct_tab, int nct, const double* sk,
                             int lv, double* out) {
  hipLaunchKernelGGL(k_decrypt_f64<LOGN>, dim3(nct * (lv + 1)), dim3(NttShape<LOGN>::T), 0, L.stream, ct, ct_tab, sk, lv,
                     out, L.tb);
}
hipError_t launch_decrypt_f64(const LaunchCtx& L, const double* ct, int nct, const double* sk, int lv, double* out,
                              const double* const* ct_tab) {
  DISPATCH_LOGN(L, decrypt_f64_impl, L, ct, ct_tab, nct, sk, lv, out);
  return hipGetLastError();
}

template <int LOGN>
static void rotkey_impl(const LaunchCtx& L, const double* sk, const RotKeyList& list, int nkeys, uint64_t seed,
                        const RotKeyArgs& ka, double* keys) {
  hipLaunchKernelGGL(k_rotkey_gen<LOGN>, dim3(nkeys * ka.beta * ka.n_limbs), dim3(NttShape<LOGN>::T), 0, L.stream,
                     sk, list, seed, ka, keys, L.tb);
}
hipError_t launch_rotkey_gen(const LaunchCtx& L, const double* sk, const RotKeyList& list, int nkeys, uint64_t seed,
                             const RotKeyArgs& ka, double* keys) {
  if (nkeys <= 0) return hipSuccess;
  if (nkeys > kKeysPerLaunch) return hipErrorInvalidValue;
  DISPATCH_LOGN(L, rotkey_impl, L, sk, list, nkeys, seed, ka, keys);
  return hipGetLastError();
}

template <int LOGN>
static void modup_impl(const LaunchCtx& L, const double* ct, const double* const* ct_tab, size_t ct_stride, int nct,
                       int lv, int alpha, const KsLevel* kl_dev, int n_tasks, double* y, double* digits, size_t dig_stride) {
  if constexpr (LOGN == 13 || LOGN == 14) {
    constexpr int S = SplitNtt<LOGN>::S;
    if (split_transforms(alpha, nct * n_tasks * S)) {
      hipLaunchKernelGGL(k_modup_split_inv<LOGN>, dim3(nct * (lv + 1) * S), dim3(256), 0, L.stream, ct, ct_tab, ct_stride, lv,
                         y, L.tb);
      hipLaunchKernelGGL(k_modup_split<LOGN>, dim3(nct * n_tasks * S), dim3(256), 0, L.stream, y, ct, ct_tab, ct_stride,
                         kl_dev, digits, dig_stride, L.tb);
      return;
    }
  }
  if constexpr (LOGN <= 14) {
    if (fuse_transforms(alpha, nct * n_tasks)) {
      hipLaunchKernelGGL(k_modup_one<LOGN>, dim3(nct * n_tasks), dim3(NttShape<LOGN>::T), 0, L.stream, ct, ct_tab, ct_stride,
                         kl_dev, digits, dig_stride, L.tb);
      return;
    }
  }
  hipLaunchKernelGGL(k_modup_intt<LOGN>, dim3(nct * (lv + 1)), dim3(NttShape<LOGN>::T), 0, L.stream, ct, ct_tab, ct_stride,
                     lv, kl_dev, y, L.tb);
  hipLaunchKernelGGL(k_modup_conv<LOGN>, dim3(nct * n_tasks), dim3(NttShape<LOGN>::T), 0, L.stream, y, ct, ct_tab,
                     ct_stride, kl_dev, digits, dig_stride, L.tb);
}
hipError_t launch_modup(const LaunchCtx& L, const double* ct, size_t ct_stride, int nct, int lv, int alpha,
                        const KsLevel* kl_dev, int n_tasks, double* y, double* digits, size_t dig_stride, const double* const* ct_tab) {
  if (nct <= 0) return hipSuccess;
  DISPATCH_LOGN(L, modup_impl, L, ct, ct_tab, ct_stride, nct, lv, alpha, kl_dev, n_tasks, y, digits, dig_stride);
  return hipGetLastError();
}

template <int LOGN>
static void moddown_impl(const LaunchCtx& L, const double* u, int npoly, int lv, int alpha, const KsLevel* kl_dev,
                         double* y, double* out, double* const* out_tab) {
  if constexpr (LOGN == 13 || LOGN == 14) {
    constexpr int S = SplitNtt<LOGN>::S;
    if (split_transforms(alpha, npoly * (lv + 1) * S)) {
      hipLaunchKernelGGL(k_moddown_split_inv<LOGN>, dim3(npoly * S), dim3(256), 0, L.stream, u, kl_dev, y, L.tb);
      hipLaunchKernelGGL(k_moddown_split<LOGN>, dim3(npoly * (lv + 1) * S), dim3(256), 0, L.stream, u, y, kl_dev, out,
                         out_tab, L.tb);
      return;
    }
  }
  if constexpr (LOGN <= 14) {
    if (fuse_transforms(alpha, npoly * (lv + 1))) {
      hipLaunchKernelGGL(k_moddown_one<LOGN>, dim3(npoly * (lv + 1)), dim3(NttShape<LOGN>::T), 0, L.stream, u, kl_dev, out,
                         out_tab, L.tb);
      return;
    }
  }
  hipLaunchKernelGGL(k_moddown_p<LOGN>, dim3(npoly * alpha), dim3(NttShape<LOGN>::T), 0, L.stream, u, kl_dev, y, L.tb);
  hipLaunchKernelGGL(k_moddown_q<LOGN>, dim3(npoly * (lv + 1)), dim3(NttShape<LOGN>::T), 0, L.stream, u, y, kl_dev, out,
                     out_tab, L.tb);
}
hipError_t launch_moddown(const LaunchCtx& L, const double* u, int npoly, int lv, int alpha, const KsLevel* kl_dev,
                          double* y, double* out, double* const* out_tab) {
  DISPATCH_LOGN(L, moddown_impl, L, u, npoly, lv, alpha, kl_dev, y, out, out_tab);
  return hipGetLastError();
}

template <int LOGN>
static void rescale_impl(const LaunchCtx& L, const double* in, int npoly, int lv, const RescaleArgs& ra, double* out,
                         size_t in_stride, const double* pt, size_t pt_stride) {
  hipLaunchKernelGGL(k_rescale<LOGN>, dim3(npoly * lv), dim3(NttShape<LOGN>::T), 0, L.stream, in, in_stride, pt, pt_stride,
                     lv, ra, out, L.tb);
}
hipError_t launch_rescale(const LaunchCtx& L, const double* in, int npoly, int lv, const RescaleArgs& ra, double* out,
                          size_t in_stride, const double* pt, size_t pt_stride) {
  if (npoly <= 0) return hipSuccess;
  DISPATCH_LOGN(L, rescale_impl, L, in, npoly, lv, ra, out, in_stride, pt, pt_stride);
  return hipGetLastError();
}

static inline unsigned blocks_for(size_t n) { return (unsigned)((n + 255) / 256); }

hipError_t launch_sum_partials(const LaunchCtx& L, const double* part, int n, int K, int N, LimbMap limb_prime,
                               double* acc) {
  const size_t tot = (size_t)2 * K * N;
  hipLaunchKernelGGL(k_sum_partials, dim3(blocks_for(tot)), dim3(256), 0, L.stream, part, n, K, N, limb_prime, L.tb.mods,
                     acc);
  return hipGetLastError();
}

hipError_t launch_scale_by_p(const LaunchCtx& L, const double* ct, int lv, int N, const double* pmod_dev, double* out,
                             int nct, const double* const* ct_tab) {
  const size_t tot = (size_t)2 * (lv + 1) * N;
  hipLaunchKernelGGL(k_scale_by_p, dim3(blocks_for(tot), nct), dim3(256), 0, L.stream, ct, ct_tab, lv, N, pmod_dev,
                     L.tb.mods, out);
  return hipGetLastError();
}

hipError_t launch_ct_mul_pt(const LaunchCtx& L, const double* ct, const double* pt, int lv, int N, double* out) {
  const size_t tot = (size_t)2 * (lv + 1) * N;
  hipLaunchKernelGGL(k_ct_mul_pt, dim3(blocks_for(tot)), dim3(256), 0, L.stream, ct, pt, lv, N, L.tb.mods, out);
  return hipGetLastError();
}

hipError_t launch_ct_add(const LaunchCtx& L, const double* a, const double* b, int lv, int N, double* out) {
  const size_t tot = (size_t)2 * (lv + 1) * N;
  hipLaunchKernelGGL(k_ct_add, dim3(blocks_for(tot)), dim3(256), 0, L.stream, a, b, lv, N, L.tb.mods, out);
  return hipGetLastError();
}

}  // namespace pvfl

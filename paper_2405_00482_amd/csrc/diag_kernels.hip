// Fused hoisted rotations x plaintext diagonals of one product, lazy ModDown
// (gfx950), and the same sum grouped by giant steps.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "he_dev.hpp"
#include "kernels.hpp"

namespace pvfl {

// The pair (P phi_i(c0) + sum_j phi_i(D_j) b_{i,j}, sum_j phi_i(D_j) a_{i,j})
// of rotation i at one index t of limb r, i > 0, as exact sums of products
// (fp64_mod.hpp).  With B = 2^b > q: c0 and a digit's own limb are below q, the
// other digit limbs, P and the keys are centred, so four digits and P c0 stay
// below 1.75 B^2 < 0.43 * 2^(2b + 3) and fold to less than 3 B.  More than four
// digits are folded four at a time and the sum is centred.
struct Rotated {
  const double* digits;  // limb r of digit 0, [beta][K][N]
  const double* keys;
  const int* slot_of_rot;
  const double* c0;      // limb r of the input (null on the special limbs)
  size_t key_stride, key_digit, dig_digit;  // doubles between keys, a key's digits, digits
  int klimb_off, a_off, half, beta;
  double pmod, cin;
  ModQ m;

  template <int BETA>
  __device__ __forceinline__ void at(int i, int t, double& u0, double& u1) const {
    const int ts = orbit_shift(t, i, half);
    const auto* key = gmem(keys) + (size_t)slot_of_rot[i] * key_stride + klimb_off + t;
    if constexpr (BETA > 0) {
      double d[BETA], kb[BETA], ka[BETA];
#pragma unroll
      for (int j = 0; j < BETA; ++j) {
        d[j] = gmem(digits)[(size_t)j * dig_digit + ts];
        kb[j] = key[(size_t)j * key_digit];
        ka[j] = key[(size_t)j * key_digit + a_off];
      }
      const double c = c0 ? gmem(c0)[ts] : 0.0;
      double h0, l0, h1, l1;
      acc_first(d[0], kb[0], cin, h0, l0);
      acc_first(d[0], ka[0], cin, h1, l1);
#pragma unroll
      for (int j = 1; j < BETA; ++j) {
        acc_mac(d[j], kb[j], h0, l0);
        acc_mac(d[j], ka[j], h1, l1);
      }
      acc_mac(c, pmod, h0, l0);
      u0 = acc_fold(h0, l0, m);
      u1 = acc_fold(h1, l1, m);
    } else {
      u0 = c0 ? mulmod(gmem(c0)[ts], pmod, m) : 0.0;
      u1 = 0.0;
      for (int j0 = 0; j0 < beta; j0 += 4) {
        double h0 = cin, l0 = 0.0, h1 = cin, l1 = 0.0;
        for (int j = j0; j < min(beta, j0 + 4); ++j) {
          const double d = gmem(digits)[(size_t)j * dig_digit + ts];
          acc_mac(d, key[(size_t)j * key_digit], h0, l0);
          acc_mac(d, key[(size_t)j * key_digit + a_off], h1, l1);
        }
        u0 = reduce(u0 + acc_fold(h0, l0, m), m);
        u1 = reduce(u1 + acc_fold(h1, l1, m), m);
      }
    }
  }
};

__device__ __forceinline__ Rotated rotated_of(const DiagArgs& a, int r, ModQ m) {
  const int N = a.N;
  const bool isq = r <= a.lv;
  return Rotated{a.digits + (size_t)r * N, a.keys, a.slot_of_rot, isq ? a.ct + (size_t)r * N : nullptr, a.key_stride,
                 (size_t)2 * a.key_limbs * N, (size_t)a.K * N, a.limb_prime[r] * N, a.key_limbs * N, N >> 1, a.beta,
                 isq ? a.pmod[r] : 0.0, acc_offset(m.q, 3), m};
}

// acc0 = sum_i pt_i (P phi_i(c0) + sum_j phi_i(D_j) b_{i,j})
// acc1 = sum_i pt_i (               sum_j phi_i(D_j) a_{i,j})
// over Q_l u P; the i = 0 term is pt_0 (P c0, P c1) on the Q limbs.
// Workgroup = 64 indices of one limb; its waves share the diagonals [z0, z1)
// of grid slice z (wave w takes z0 + w, z0 + w + waves, ...) and add up in LDS,
// so that a product needs no partial sums in memory unless the indices alone
// leave the chip idle (slices > 1: part[z][2][K][N], summed by the caller).
// Bound by memory: every key and plaintext limb is read once (128 diagonals
// at N = 2^14, 4 + 1 primes: 750 MB, 124 us at the read rate).  One
// workgroup per chunk of diagonals, a sum over 12 partial sums and P c in a
// launch of its own took 145 + 7 + 5 us; this takes 135.
template <int BETA>
__global__ __launch_bounds__(1024) void k_diag_lazy(DiagArgs a) {
  __shared__ double red[2][16][64];
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6, nw = blockDim.x >> 6;
  const int t = blockIdx.x * 64 + lane, r = blockIdx.y;
  const int N = a.N, K = a.K;
  const bool isq = r <= a.lv;
  const ModQ m = a.mods[a.limb_prime[r]];
  const size_t limbN = (size_t)r * N, KN = (size_t)K * N;
  const int z0 = blockIdx.z * a.chunk, z1 = min(z0 + a.chunk, a.mprime);
  const Rotated rot = rotated_of(a, r, m);
  // plaintexts below q times sums below 3 B: nine terms stay below 27 B^2 < 0.43 * 2^(2b + 6)
  const double cout = acc_offset(m.q, 6);
  double hi0 = cout, lo0 = 0.0, hi1 = cout, lo1 = 0.0;
  int cnt = 0;
  const auto* pt = gmem(a.pt) + limbN + t;
  for (int i = z0 + w; i < z1; i += nw) {
    const double p = __builtin_nontemporal_load(pt + (size_t)i * KN);
    double u0, u1;
    if (i > 0) {
      rot.at<BETA>(i, t, u0, u1);
    } else {
      u0 = isq ? mulmod(gmem(a.ct)[limbN + t], rot.pmod, m) : 0.0;
      u1 = isq ? mulmod(gmem(a.ct)[(size_t)(a.lv + 1) * N + limbN + t], rot.pmod, m) : 0.0;
    }
    acc_mac(p, u0, hi0, lo0);
    acc_mac(p, u1, hi1, lo1);
    if (++cnt == 8) {
      lo0 = reduce(acc_fold(hi0, lo0, m), m);
      lo1 = reduce(acc_fold(hi1, lo1, m), m);
      hi0 = hi1 = cout;
      cnt = 0;
    }
  }
  red[0][w][lane] = reduce(acc_fold(hi0, lo0, m), m);
  red[1][w][lane] = reduce(acc_fold(hi1, lo1, m), m);
  __syncthreads();
  for (int h = w; h < 2; h += nw) {
    double* out = a.part + ((size_t)2 * blockIdx.z + h) * KN + limbN + t;
    double v = a.add ? *out : 0.0;
    for (int k = 0; k < nw; ++k) v += red[h][k][lane];
    *out = reduce(v, m);
  }
}

// The baby-step/giant-step sums: giant step g's inner sum over the baby
// rotations, out[g][2][K][N] = sum_k pt_{g bs + k} (rotated pair of k), k < bs.
// A workgroup holds the sums of kGiants giant steps at 64 indices of one limb
// and its waves share the baby rotations, so that a rotation's key product is
// made once per kGiants giant steps instead of once per diagonal.  Diagonal by
// diagonal, 512 diagonals with 32 baby steps at N = 2^14 took 376 us and
// another 12 us for their partial sums; this takes 121 (plaintexts and keys
// alone: 82 us at the read rate).  Whole products of 256 diagonals at 2^14, 4 + 1
// primes, with kGiants 8, 4 and 2, us: 16 giant steps 240, 241, 282; 8 of them 187, 199,
// 241; 4 of them 226, 208, 272; 2 of them 303, 276, 266 (sums past the last giant step are
// made and dropped).  8 to 16 giant steps are the fastest splits of these diagonals.
constexpr int kGiants = 8;
template <int BETA>
__global__ __launch_bounds__(512) void k_diag_bsgs(DiagArgs a, int bs, int g) {
  __shared__ double red[2 * kGiants][8][64];
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6, nw = blockDim.x >> 6;
  const int t = blockIdx.x * 64 + lane, r = blockIdx.y, g0 = blockIdx.z * kGiants;
  const int N = a.N, K = a.K, ng = min(kGiants, g - g0);
  const bool isq = r <= a.lv;
  const ModQ m = a.mods[a.limb_prime[r]];
  const size_t limbN = (size_t)r * N, KN = (size_t)K * N;
  const Rotated rot = rotated_of(a, r, m);
  const double cout = acc_offset(m.q, 6);  // as in k_diag_lazy
  double hi0[kGiants], lo0[kGiants], hi1[kGiants], lo1[kGiants];
#pragma unroll
  for (int u = 0; u < kGiants; ++u) {
    hi0[u] = hi1[u] = cout;
    lo0[u] = lo1[u] = 0.0;
  }
  int cnt = 0;
  const auto* pt = gmem(a.pt) + (size_t)g0 * bs * KN + limbN + t;
  for (int k = w; k < bs; k += nw) {
    double p[kGiants];
#pragma unroll
    for (int u = 0; u < kGiants; ++u)  // past the last giant step: the first one's again, never stored
      p[u] = __builtin_nontemporal_load(pt + ((size_t)(u < ng ? u : 0) * bs + k) * KN);
    double u0, u1;
    if (k > 0) {
      rot.at<BETA>(k, t, u0, u1);
    } else {
      u0 = isq ? mulmod(gmem(a.ct)[limbN + t], rot.pmod, m) : 0.0;
      u1 = isq ? mulmod(gmem(a.ct)[(size_t)(a.lv + 1) * N + limbN + t], rot.pmod, m) : 0.0;
    }
#pragma unroll
    for (int u = 0; u < kGiants; ++u) {
      acc_mac(p[u], u0, hi0[u], lo0[u]);
      acc_mac(p[u], u1, hi1[u], lo1[u]);
    }
    if (++cnt == 8) {
#pragma unroll
      for (int u = 0; u < kGiants; ++u) {
        lo0[u] = reduce(acc_fold(hi0[u], lo0[u], m), m);
        lo1[u] = reduce(acc_fold(hi1[u], lo1[u], m), m);
        hi0[u] = hi1[u] = cout;
      }
      cnt = 0;
    }
  }
#pragma unroll
  for (int u = 0; u < kGiants; ++u) {
    red[2 * u][w][lane] = reduce(acc_fold(hi0[u], lo0[u], m), m);
    red[2 * u + 1][w][lane] = reduce(acc_fold(hi1[u], lo1[u], m), m);
  }
  __syncthreads();
  for (int h = w; h < 2 * ng; h += nw) {
    double v = 0.0;
    for (int k = 0; k < nw; ++k) v += red[h][k][lane];
    a.part[((size_t)2 * g0 + h) * KN + limbN + t] = reduce(v, m);
  }
}

// Alg. 3 ciphertext-matrix product (and the column-order one): out_k = sum_i
// ct_i pt_{i,k}, i < nct, k < nout.  A workgroup holds the sums of OUTS outputs
// at 64 indices of one limb and its NW waves share the ciphertexts, so that a
// ciphertext is read once per OUTS outputs; sums are exact (fp64_mod.hpp):
// eight products of residues below q stay below 8 B^2 < 0.43 * 2^(2b + 5).
// Bound by memory, each plaintext limb read once.  64 ciphertexts, 8 outputs,
// 6 limbs at N = 2^14 (0.50 GB, 83 us at the read rate): one output per thread
// 128 us, this 83.  Both counts are compile-time constants: the registers and
// the LDS are those of the waves there are (two waves with the LDS of eight
// took 2 ciphertexts, 9 outputs, 8 limbs at N = 2^15 from 14 to 50 us).
// STREAM: plaintext loads bypass the caches.
template <int OUTS, int NW, bool STREAM>
__global__ __launch_bounds__(64 * NW) void k_ctmat(const double* __restrict__ ct, const double* __restrict__ pt, int nct,
                                                   int nout, int lv, int N, const ModQ* __restrict__ mods,
                                                   double* __restrict__ out) {
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  const int r = blockIdx.y, k0 = blockIdx.z * OUTS, nk = min(OUTS, nout - k0);
  const ModQ m = mods[r];
  const size_t Q = (size_t)(lv + 1) * N, off = (size_t)r * N + blockIdx.x * 64 + lane;
  const double c = acc_offset(m.q, 5);
  double hi0[OUTS], lo0[OUTS], hi1[OUTS], lo1[OUTS];
#pragma unroll
  for (int u = 0; u < OUTS; ++u) {
    hi0[u] = hi1[u] = c;
    lo0[u] = lo1[u] = 0.0;
  }
  int cnt = 0;
  for (int i = w; i < nct; i += NW) {
    const auto* pi = gmem(pt) + ((size_t)i * nout + k0) * Q + off;
    const auto* ci = gmem(ct) + (size_t)i * 2 * Q + off;
    double p[OUTS];
#pragma unroll
    for (int u = 0; u < OUTS; ++u) {  // past the last output: the first one's again, never stored
      const auto* pu = pi + (size_t)(u < nk ? u : 0) * Q;
      p[u] = STREAM ? __builtin_nontemporal_load(pu) : *pu;
    }
    const double x0 = ci[0], x1 = ci[Q];
    __builtin_amdgcn_sched_barrier(0);  // every load issued before the first is waited for
#pragma unroll
    for (int u = 0; u < OUTS; ++u) {
      acc_mac(x0, p[u], hi0[u], lo0[u]);
      acc_mac(x1, p[u], hi1[u], lo1[u]);
    }
    if (++cnt == 8) {
#pragma unroll
      for (int u = 0; u < OUTS; ++u) {
        lo0[u] = reduce(acc_fold(hi0[u], lo0[u], m), m);
        lo1[u] = reduce(acc_fold(hi1[u], lo1[u], m), m);
        hi0[u] = hi1[u] = c;
      }
      cnt = 0;
    }
  }
  if constexpr (NW == 1) {
#pragma unroll
    for (int u = 0; u < OUTS; ++u) {
      if (u >= nk) break;
      out[(size_t)(2 * (k0 + u)) * Q + off] = reduce(acc_fold(hi0[u], lo0[u], m), m);
      out[(size_t)(2 * (k0 + u) + 1) * Q + off] = reduce(acc_fold(hi1[u], lo1[u], m), m);
    }
  } else {
    __shared__ double red[2 * OUTS][NW][64];
#pragma unroll
    for (int u = 0; u < OUTS; ++u) {
      red[2 * u][w][lane] = reduce(acc_fold(hi0[u], lo0[u], m), m);
      red[2 * u + 1][w][lane] = reduce(acc_fold(hi1[u], lo1[u], m), m);
    }
    __syncthreads();
    for (int h = w; h < 2 * nk; h += NW) {
      double v = 0.0;
#pragma unroll
      for (int k = 0; k < NW; ++k) v += red[h][k][lane];
      out[(size_t)(2 * k0 + h) * Q + off] = reduce(v, m);
    }
  }
}

// One ciphertext: out_k = ct pt_k, thread = (index t, limb r, output k).  There
// is no sum, so nothing to share and no exact sum's offset to make.
__global__ __launch_bounds__(256) void k_ctmat_one(const double* __restrict__ ct, const double* __restrict__ pt, int lv,
                                                   int N, const ModQ* __restrict__ mods, double* __restrict__ out) {
  const int r = blockIdx.y, k = blockIdx.z;
  const ModQ m = mods[r];
  const size_t Q = (size_t)(lv + 1) * N, off = (size_t)r * N + blockIdx.x * 256 + threadIdx.x;
  const double p = pt[(size_t)k * Q + off];
  out[(size_t)k * 2 * Q + off] = reduce(mulmod(ct[off], p, m), m);
  out[(size_t)k * 2 * Q + Q + off] = reduce(mulmod(ct[Q + off], p, m), m);
}

// ---------------------------------------------------------------------------
#define DISPATCH_BETA(KERNEL, BETA_RT, GRID, BLOCK, ...)                                              \
  switch (BETA_RT) {                                                                                  \
    case 1: hipLaunchKernelGGL(KERNEL<1>, GRID, BLOCK, 0, L.stream, __VA_ARGS__); break;              \
    case 2: hipLaunchKernelGGL(KERNEL<2>, GRID, BLOCK, 0, L.stream, __VA_ARGS__); break;              \
    case 3: hipLaunchKernelGGL(KERNEL<3>, GRID, BLOCK, 0, L.stream, __VA_ARGS__); break;              \
    case 4: hipLaunchKernelGGL(KERNEL<4>, GRID, BLOCK, 0, L.stream, __VA_ARGS__); break;              \
    default: hipLaunchKernelGGL(KERNEL<0>, GRID, BLOCK, 0, L.stream, __VA_ARGS__); break;             \
  }

// waves of a workgroup that share n items: a power of two, no more than most
static int waves_for(int n, int most) {
  int w = 1;
  while (w < n && w < most) w *= 2;
  return w;
}

hipError_t launch_diag_lazy(const LaunchCtx& L, const DiagArgs& a, int slices) {
  const dim3 grid(a.N / 64, a.K, slices), block(64 * waves_for(a.chunk, 16));
  DISPATCH_BETA(k_diag_lazy, a.beta, grid, block, a);
  return hipGetLastError();
}

hipError_t launch_diag_bsgs(const LaunchCtx& L, const DiagArgs& a, int bs, int g) {
  const dim3 grid(a.N / 64, a.K, (g + kGiants - 1) / kGiants), block(64 * waves_for(bs, 8));
  DISPATCH_BETA(k_diag_bsgs, a.beta, grid, block, a, bs, g);
  return hipGetLastError();
}

template <int OUTS, bool STREAM>
static void ctmat_run(const LaunchCtx& L, const double* ct, const double* pt, int nct, int nout, int lv, int N, int nw,
                      double* out) {
  const dim3 grid(N / 64, lv + 1, (nout + OUTS - 1) / OUTS), block(64 * nw);
  auto* k = nw == 1 ? k_ctmat<OUTS, 1, STREAM> : nw == 2 ? k_ctmat<OUTS, 2, STREAM>
          : nw == 4 ? k_ctmat<OUTS, 4, STREAM> : k_ctmat<OUTS, 8, STREAM>;
  hipLaunchKernelGGL(k, grid, block, 0, L.stream, ct, pt, nct, nout, lv, N, L.tb.mods, out);
}
template <int OUTS>
static void ctmat_outs(const LaunchCtx& L, const double* ct, const double* pt, int nct, int nout, int lv, int N, int nw,
                       bool stream, double* out) {
  if (stream)
    ctmat_run<OUTS, true>(L, ct, pt, nct, nout, lv, N, nw, out);
  else
    ctmat_run<OUTS, false>(L, ct, pt, nct, nout, lv, N, nw, out);
}

// The outputs fall into as few equal parts of at most eight as they can: 9 of
// 64 ciphertexts with 6 limbs at 2^14 take 85 us as 5 + 4, 128 as 8 + 1.  Waves
// share the ciphertexts until the chip has 2048 of them, eight on a CU, and only
// while each still has four: 256 ciphertexts, one output, 2 limbs at 2^12 take
// 113 us with one wave per workgroup, 19 with eight; beyond the line 16
// ciphertexts, one output, 8 limbs at 2^15 take 16.7 with one, 21 with eight.  One
// ciphertext takes the kernel that shares nothing (9 outputs, 8 limbs at 2^15: 10.8
// against 13.0 us).  Large plaintexts are streamed past the caches: beyond 64
// MiB where many ciphertexts keep the loads at the memory's rate (the 403 MB of 64 x 8
// with 6 limbs at 2^14: 83 us against 94; 101 MB of 64 x 2 just encoded: a transposed
// product 465 against 468); with few, products from the same plaintexts find them in
// the 256 MB last-level cache (107 MB of 3 x 17 with 8 limbs at 2^15: 32 us against 36).
hipError_t launch_ctmat(const LaunchCtx& L, const double* ct, const double* pt, int nct, int nout, int lv, int N,
                        double* out) {
  if (nct == 1) {
    hipLaunchKernelGGL(k_ctmat_one, dim3(N / 256, lv + 1, nout), dim3(256), 0, L.stream, ct, pt, lv, N, L.tb.mods, out);
    return hipGetLastError();
  }
  const int parts = (nout + 7) / 8, outs = (nout + parts - 1) / parts;
  const long waves = (long)(N / 64) * (lv + 1) * ((nout + outs - 1) / outs);
  const size_t mib = (sizeof(double) * (size_t)nct * nout * (lv + 1) * N) >> 20;
  const bool stream = mib >= (nct >= 16 ? 64 : 200);
  int nw = 1;
  while (nw < 8 && waves * nw < 2048 && nct >= 8 * nw) nw *= 2;
  switch (outs) {
    case 1: ctmat_outs<1>(L, ct, pt, nct, nout, lv, N, nw, stream, out); break;
    case 2: ctmat_outs<2>(L, ct, pt, nct, nout, lv, N, nw, stream, out); break;
    case 3: ctmat_outs<3>(L, ct, pt, nct, nout, lv, N, nw, stream, out); break;
    case 4: ctmat_outs<4>(L, ct, pt, nct, nout, lv, N, nw, stream, out); break;
    case 5: ctmat_outs<5>(L, ct, pt, nct, nout, lv, N, nw, stream, out); break;
    case 6: ctmat_outs<6>(L, ct, pt, nct, nout, lv, N, nw, stream, out); break;
    case 7: ctmat_outs<7>(L, ct, pt, nct, nout, lv, N, nw, stream, out); break;
    default: ctmat_outs<8>(L, ct, pt, nct, nout, lv, N, nw, stream, out); break;
  }
  return hipGetLastError();
}

}  // namespace pvfl

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
// alone: 82 us at the read rate).
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
// at 64 indices of one limb and its waves share the ciphertexts, so that a
// ciphertext is read once per OUTS outputs; sums are exact (fp64_mod.hpp):
// eight products of residues below q stay below 8 B^2 < 0.43 * 2^(2b + 5).
// Bound by memory, each plaintext limb read once.  64 ciphertexts, 8 outputs,
// 6 limbs at N = 2^14 (0.50 GB, 83 us at the read rate): one output per thread
// 126 us, this 82.
template <int OUTS>
__global__ __launch_bounds__(512) void k_ctmat(const double* __restrict__ ct, const double* __restrict__ pt, int nct,
                                               int nout, int lv, int N, const ModQ* __restrict__ mods,
                                               double* __restrict__ out) {
  __shared__ double red[2 * OUTS][8][64];
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6, nw = blockDim.x >> 6;
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
  for (int i = w; i < nct; i += nw) {
    const auto* pi = gmem(pt) + ((size_t)i * nout + k0) * Q + off;
    const auto* ci = gmem(ct) + (size_t)i * 2 * Q + off;
    double p[OUTS];
#pragma unroll
    for (int u = 0; u < OUTS; ++u)  // past the last output: the first one's again, never stored
      p[u] = __builtin_nontemporal_load(pi + (size_t)(u < nk ? u : 0) * Q);
    const double x0 = ci[0], x1 = ci[Q];
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
#pragma unroll
  for (int u = 0; u < OUTS; ++u) {
    red[2 * u][w][lane] = reduce(acc_fold(hi0[u], lo0[u], m), m);
    red[2 * u + 1][w][lane] = reduce(acc_fold(hi1[u], lo1[u], m), m);
  }
  __syncthreads();
  for (int h = w; h < 2 * nk; h += nw) {
    double v = 0.0;
    for (int k = 0; k < nw; ++k) v += red[h][k][lane];
    out[(size_t)(2 * k0 + h) * Q + off] = reduce(v, m);
  }
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

hipError_t launch_ctmat(const LaunchCtx& L, const double* ct, const double* pt, int nct, int nout, int lv, int N,
                        double* out) {
  const int outs = nout >= 5 ? 8 : nout >= 3 ? 4 : nout;
  const dim3 grid(N / 64, lv + 1, (nout + outs - 1) / outs), block(64 * waves_for(nct, 8));
  switch (outs) {
    case 1: hipLaunchKernelGGL(k_ctmat<1>, grid, block, 0, L.stream, ct, pt, nct, nout, lv, N, L.tb.mods, out); break;
    case 2: hipLaunchKernelGGL(k_ctmat<2>, grid, block, 0, L.stream, ct, pt, nct, nout, lv, N, L.tb.mods, out); break;
    case 4: hipLaunchKernelGGL(k_ctmat<4>, grid, block, 0, L.stream, ct, pt, nct, nout, lv, N, L.tb.mods, out); break;
    default: hipLaunchKernelGGL(k_ctmat<8>, grid, block, 0, L.stream, ct, pt, nct, nout, lv, N, L.tb.mods, out); break;
  }
  return hipGetLastError();
}

}  // namespace pvfl

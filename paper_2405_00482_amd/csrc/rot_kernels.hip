// Batched single rotations (O3 / O4) for gfx950: up to kRotsPerLaunch
// ciphertexts, each with its own rotation and key, go through key switching
// in four launches.
//
// What bounds a rotation on its own is latency, not arithmetic or bandwidth:
// a limb transform is one workgroup, so one ciphertext occupies 2 to 18 of
// the 256 CUs and every launch takes one transform's latency (13-35 us).  A
// plan that rotates many ciphertexts therefore runs them side by side, and
// the element-wise kernels of a rotation (automorphism, key product, the
// sums) are folded into the transforms that read or write the same limb:
//   k_rot_modup_intt  INTT of c1, read through the rotation where it precedes
//                     the ModUp (O3)
//   k_rot_modup_conv  the converted digit limbs (a digit's own limbs are read
//                     from c1 itself)
//   k_rot_down_p      key product on the special limbs, INTT
//   k_rot_down_q      ModDown's NTT, key product on the ciphertext limbs, the
//                     rotated c0 and (accumulating form) the unrotated input
// Before: seven launches per rotation, one rotation after the other.  Measured
// then and now: the transposed conversion of 256 x 64 with its product at 2^14,
// 6 + 3 primes (63 rotations) 8.14 -> 0.55 ms; Alg. 1's 256 x 512 product at
// 2^13 (31 rotations) 1.16 -> 0.11 ms; the row method's 12 x 64 at 2^13 (83
// rotations in 7 dependent steps) 6.60 -> 0.52 ms.
#define PVFL_OPAQUE_TID 1

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "he_dev.hpp"
#include "kernels.hpp"
#include "ntt_core.hpp"

namespace pvfl {

// Value of (digit j, limb r) of a rotation at slot t: a limb of the digit
// itself is c1's residue, every other limb was converted (k_rot_modup_conv).
// Both are read through the rotation, except converted limbs of an already
// rotated c1 (O3).
struct RotDigits {
  const double* dig;  // [beta][K][N]
  const double* c1;   // [lv+1][N]
  int K, lv, alpha, N, rot, dig_rot;
  __device__ __forceinline__ const double* row(int j, int r, int* shift) const {
    const bool own = r <= lv && r / alpha == j;
    *shift = own ? rot : dig_rot;
    return own ? c1 + (size_t)r * N : dig + ((size_t)j * K + r) * N;
  }
};

// sum_j D_j[r][t] key_j[t] at one slot; key = this half's limb of digit 0
__device__ __forceinline__ double rot_inner_at(const RotDigits& d, int r, const double* key, size_t key_digit, int beta,
                                               int t, ModQ m) {
  double u = 0.0;
  for (int j = 0; j < beta; ++j) {
    int sh;
    const double* row = d.row(j, r, &sh);
    u += mulmod(gmem(row)[orbit_shift(t, sh, d.N >> 1)], gmem(key)[(size_t)j * key_digit + t], m);
  }
  return u;
}

// The same for all slots of a thread (N <= 2^14): u[2w], u[2w + 1] at slots
// t = tid + w T and t + N/2, the loads of a digit all in flight together.
template <int LOGN>
__device__ __forceinline__ void rot_inner(double (&u)[16], const RotDigits& d, int r, const double* key,
                                          size_t key_digit, int beta, ModQ m) {
  constexpr int N = 1 << LOGN, H = N / 2, T = NttShape<LOGN>::T;
  const int tid = opaque_tid();
#pragma unroll
  for (int w = 0; w < 16; ++w) u[w] = 0.0;
#pragma unroll 1
  for (int j = 0; j < beta; ++j) {
    int sh;
    const auto* row = gmem(d.row(j, r, &sh));
    const auto* kj = gmem(key) + (size_t)j * key_digit;
    double a[16], k[16];
#pragma unroll
    for (int w = 0; w < 8; ++w) {
      const int t = tid + w * T, ts = (t + sh) & (H - 1);
      a[2 * w] = row[ts];
      a[2 * w + 1] = row[ts + H];
      k[2 * w] = kj[t];
      k[2 * w + 1] = kj[t + H];
    }
#pragma unroll
    for (int w = 0; w < 16; ++w) u[w] += mulmod(a[w], k[w], m);
  }
}

// The key products of every rotation and limb on their own, one thread per
// index: u[item][x][r][N], x = 0 with P phi(c0) added, with add = 1 both with P
// times the unrotated input.  See launch_rotations for when this is done.
__global__ __launch_bounds__(256) void k_rot_inner(RotBatch b, int pre, int add, const KsLevel* __restrict__ kl,
                                                   const double* __restrict__ digits, size_t dig_stride, int key_limbs,
                                                   int N, const ModQ* __restrict__ mods, double* __restrict__ u) {
  const int t = blockIdx.x * 256 + threadIdx.x, r = blockIdx.y, it = blockIdx.z;
  const int lv = kl->lv, K = kl->K;
  const bool isq = r <= lv;
  const int pi = isq ? r : kl->n_q_total + r - lv - 1;
  const ModQ m = mods[pi];
  const int rot = b.it[it].rot;
  const double* ct = b.it[it].ct;
  const RotDigits d{digits + (size_t)it * dig_stride, ct + (size_t)(lv + 1) * N, K, lv, kl->alpha, N, rot, pre ? 0 : rot};
  const double* key = b.it[it].key + (size_t)pi * N;
  const size_t key_digit = (size_t)2 * key_limbs * N;
  double u0 = 0.0, u1 = 0.0;
  for (int j = 0; j < kl->beta; ++j) {
    int sh;
    const double* row = d.row(j, r, &sh);
    const double x = gmem(row)[orbit_shift(t, sh, N >> 1)];
    u0 += mulmod(x, gmem(key)[(size_t)j * key_digit + t], m);
    u1 += mulmod(x, gmem(key)[(size_t)j * key_digit + (size_t)key_limbs * N + t], m);
  }
  if (isq) {
    const double pmod = kl->p_mod[r];
    u0 += mulmod(gmem(ct)[(size_t)r * N + orbit_shift(t, rot, N >> 1)], pmod, m);
    if (add) {
      u0 += mulmod(gmem(ct)[(size_t)r * N + t], pmod, m);
      u1 += mulmod(gmem(ct)[(size_t)(lv + 1 + r) * N + t], pmod, m);
    }
  }
  double* dst = u + ((size_t)it * 2 * K + r) * N + t;
  *dst = reduce(u0, m);
  dst[(size_t)K * N] = reduce(u1, m);
}

#define ROT_KERNEL(LOGN) __global__ __launch_bounds__(NttShape<LOGN>::T)

// block (item, i): y[item][i] = [c1_i (Q_j/q_i)^-1]_{q_i}, canonical; pre = 1
// reads c1 through the rotation
template <int LOGN>
ROT_KERNEL(LOGN) void k_rot_modup_intt(RotBatch b, int pre, const KsLevel* __restrict__ kl, double* __restrict__ y,
                                       DevTabs tb) {
  constexpr int N = 1 << LOGN;
  __shared__ double s[NttShape<LOGN>::LDS];
  const int lv = kl->lv;
  const int i = blockIdx.x % (lv + 1), it = blockIdx.x / (lv + 1);
  const ModQ m = tb.mods[i];
  const auto* c1 = gmem(b.it[it].ct) + (size_t)(lv + 1 + i) * N;
  const int rot = pre ? b.it[it].rot : 0;
  const double ih = kl->up_inv_hat[i];
  double* dst = y + ((size_t)it * (lv + 1) + i) * N;
  ntt_inv_in<LOGN>(s, [&](int t) { return c1[orbit_shift(t, rot, N / 2)]; }, tb.inv_tw + (size_t)i * N, m,
                   tb.ninv[i], [&](int j, double v) { dst[j] = canon(mulmod(canon(v, m), ih, m), m); });
}

// block (item, task): one converted limb of one digit
template <int LOGN>
ROT_KERNEL(LOGN) void k_rot_modup_conv(const double* __restrict__ y, const KsLevel* __restrict__ kl,
                                       double* __restrict__ digits, size_t dig_stride, DevTabs tb) {
  constexpr int N = 1 << LOGN;
  __shared__ double s[NttShape<LOGN>::LDS];
  const int nt = kl->n_tasks, it = blockIdx.x / nt;
  const KsTask* __restrict__ task = kl->up_task + blockIdx.x % nt;
  const int nsrc = task->nsrc;
  if (nsrc == 0) return;  // the digit's own limb: read from c1
  const int pi = task->prime;
  const ModQ m = tb.mods[pi];
  double* dst = digits + (size_t)it * dig_stride + ((size_t)task->digit * kl->K + task->limb) * N;
  double x[NttShape<LOGN>::PER];
  convert_coeffs<LOGN>(gmem(y + ((size_t)it * (kl->lv + 1) + task->src0) * N), nsrc, [&](int u) { return task->hat[u]; },
                       0.0, m, x);
  ntt_fwd_regs_out<LOGN>(s, x, tb.fwd_tw + (size_t)pi * N, m, [&](int t, double v) { dst[t] = v; });
}

// block (item, task), alpha = 1: both ModUp transforms (k_modup_one)
template <int LOGN>
ROT_KERNEL(LOGN) void k_rot_modup_one(RotBatch b, int pre, const KsLevel* __restrict__ kl, double* __restrict__ digits,
                                      size_t dig_stride, DevTabs tb) {
  constexpr int N = 1 << LOGN;
  __shared__ double s[NttShape<LOGN>::LDS];
  const int nt = kl->n_tasks, it = blockIdx.x / nt;
  const KsTask& task = kl->up_task[blockIdx.x % nt];
  if (task.nsrc == 0) return;  // the digit's own limb: read from c1
  const int pi = task.prime, rot = pre ? b.it[it].rot : 0;
  const auto* src = gmem(b.it[it].ct) + (size_t)(kl->lv + 1 + task.src0) * N;
  double* dst = digits + (size_t)it * dig_stride + ((size_t)task.digit * kl->K + task.limb) * N;
  double x[16];
  modup_source<LOGN>(s, [&](int t) { return src[orbit_shift(t, rot, N / 2)]; }, task, tb, x);
  ntt_fwd_regs_out<LOGN>(s, x, tb.fwd_tw + (size_t)pi * N, tb.mods[pi], [&](int t, double v) { dst[t] = v; });
}

// block (item, half x, limb i), alpha = 1, key products made apart: both
// ModDown transforms
template <int LOGN>
ROT_KERNEL(LOGN) void k_rot_down_one(RotBatch b, const KsLevel* __restrict__ kl, const double* __restrict__ inner,
                                     DevTabs tb) {
  constexpr int N = 1 << LOGN, T = NttShape<LOGN>::T;
  __shared__ double s[NttShape<LOGN>::LDS];
  const int lv = kl->lv;
  const int i = blockIdx.x % (lv + 1), x = (blockIdx.x / (lv + 1)) & 1, it = blockIdx.x / (2 * (lv + 1));
  const auto* u = gmem(inner) + (size_t)(2 * it + x) * kl->K * N;
  double* o = b.it[it].out + (size_t)(x * (lv + 1) + i) * N;
  double uv[16];
#pragma unroll
  for (int w = 0; w < 16; ++w) uv[w] = u[(size_t)i * N + (int)opaque_tid() + (w >> 1) * T + (w & 1) * (N / 2)];
  moddown_limb<LOGN>(s, [&](int t) { return u[(size_t)(lv + 1) * N + t]; }, uv, i, kl, tb,
                     [&](int t, double v) { o[t] = v; });
}

// block (item, half x, special limb k): the key product on limb p_k, then
// ModDown's first step
template <int LOGN>
ROT_KERNEL(LOGN) void k_rot_down_p(RotBatch b, int pre, const KsLevel* __restrict__ kl, const double* __restrict__ digits,
                                   size_t dig_stride, int key_limbs, const double* __restrict__ inner,
                                   double* __restrict__ y, DevTabs tb) {
  constexpr int N = 1 << LOGN, T = NttShape<LOGN>::T;
  __shared__ double s[NttShape<LOGN>::LDS];
  const int alpha = kl->alpha, lv = kl->lv;
  const int k = blockIdx.x % alpha, x = (blockIdx.x / alpha) & 1, it = blockIdx.x / (2 * alpha);
  const int pi = kl->n_q_total + k;
  const ModQ m = tb.mods[pi];
  const double h = kl->down_half[lv + 1 + k], ih = kl->down_inv_hat[k];
  const int rot = b.it[it].rot;
  const RotDigits d{digits + (size_t)it * dig_stride, b.it[it].ct + (size_t)(lv + 1) * N, kl->K, lv, alpha, N, rot,
                    pre ? 0 : rot};
  const double* key = b.it[it].key + ((size_t)x * key_limbs + pi) * N;
  const size_t key_digit = (size_t)2 * key_limbs * N;
  double* dst = y + ((size_t)(2 * it + x) * alpha + k) * N;
  auto store = [&](int c, double v) { dst[c] = canon(mulmod(canon(v + h, m), ih, m), m); };
  if (inner) {
    const auto* src = gmem(inner) + ((size_t)(2 * it + x) * kl->K + lv + 1 + k) * N;
    ntt_inv_in<LOGN>(s, [&](int t) { return src[t]; }, tb.inv_tw + (size_t)pi * N, m, tb.ninv[pi], store);
  } else if constexpr (LOGN <= 14) {
    double u[16], c[16];
    rot_inner<LOGN>(u, d, lv + 1 + k, key, key_digit, kl->beta, m);
    slots_to_lds<LOGN>(s, u, m);
    __syncthreads();
    ntt_inv_regs<LOGN>(s, c, tb.inv_tw + (size_t)pi * N, m, tb.ninv[pi]);
#pragma unroll
    for (int w = 0; w < 16; ++w) store((int)opaque_tid() + w * T, c[w]);
  } else {
    ntt_inv_in<LOGN>(s, [&](int t) { return rot_inner_at(d, lv + 1 + k, key, key_digit, kl->beta, t, m); },
                     tb.inv_tw + (size_t)pi * N, m, tb.ninv[pi], store);
  }
}

// block (item, half x, limb i): out_x = (sum_j D_j key_j - t) P^-1, plus the
// rotated c0 (x = 0), plus the unrotated input with add = 1.  The addends
// join the key product times P, so that one product with P^-1 ends the sum.
template <int LOGN>
ROT_KERNEL(LOGN) void k_rot_down_q(RotBatch b, int pre, int add, const KsLevel* __restrict__ kl,
                                   const double* __restrict__ digits, size_t dig_stride, int key_limbs,
                                   const double* __restrict__ inner, const double* __restrict__ y, DevTabs tb) {
  constexpr int N = 1 << LOGN, H = N / 2, T = NttShape<LOGN>::T;
  __shared__ double s[NttShape<LOGN>::LDS];
  const int alpha = kl->alpha, lv = kl->lv;
  const int i = blockIdx.x % (lv + 1), x = (blockIdx.x / (lv + 1)) & 1, it = blockIdx.x / (2 * (lv + 1));
  const ModQ m = tb.mods[i];
  const double h = kl->down_half[i], pinv = kl->down_pinv[i], pmod = kl->p_mod[i];
  const int rot = b.it[it].rot;
  const double* ct = b.it[it].ct;
  const RotDigits d{digits + (size_t)it * dig_stride, ct + (size_t)(lv + 1) * N, kl->K, lv, alpha, N, rot, pre ? 0 : rot};
  const double* key = b.it[it].key + ((size_t)x * key_limbs + i) * N;
  const size_t key_digit = (size_t)2 * key_limbs * N;
  const double* yx = y + (size_t)(2 * it + x) * alpha * N;
  const auto* c0 = gmem(ct) + (size_t)i * N;
  const auto* cx = gmem(ct) + (size_t)(x * (lv + 1) + i) * N;
  const auto* in = gmem(inner) + ((size_t)(2 * it + x) * kl->K + i) * N;
  double* o = b.it[it].out + (size_t)(x * (lv + 1) + i) * N;
  double c[NttShape<LOGN>::PER];
  auto conv = [&] {
    convert_coeffs<LOGN>(gmem(yx), alpha, [&](int k) { return kl->down_hat[k * kMaxLimbs + i]; }, h, m, c);
  };
  if constexpr (LOGN <= 14) {
    double u[16];
    if (inner) {
#pragma unroll
      for (int w = 0; w < 16; ++w) u[w] = in[(int)opaque_tid() + (w >> 1) * T + (w & 1) * H];
    } else {
      rot_inner<LOGN>(u, d, i, key, key_digit, kl->beta, m);
    }
    if (!inner && x == 0) {
#pragma unroll
      for (int w = 0; w < 16; ++w)
        u[w] += mulmod(c0[(((int)opaque_tid() + (w >> 1) * T + rot) & (H - 1)) + (w & 1) * H], pmod, m);
    }
    if (!inner && add) {
#pragma unroll
      for (int w = 0; w < 16; ++w) u[w] += mulmod(cx[(int)opaque_tid() + (w >> 1) * T + (w & 1) * H], pmod, m);
    }
    recentre(u, m);
    double v[16];
    conv();
    ntt_fwd_regs<LOGN>(s, c, tb.fwd_tw + (size_t)i * N, m);
    slots_from_lds<LOGN>(s, v);
#pragma unroll
    for (int w = 0; w < 16; ++w)
      o[(int)opaque_tid() + (w >> 1) * T + (w & 1) * H] = reduce(mulmod(u[w] - v[w], pinv, m), m);
  } else {
    conv();
    ntt_fwd_regs_out<LOGN>(s, c, tb.fwd_tw + (size_t)i * N, m, [&](int t, double v) {
      double u;
      if (inner) {
        u = in[t];
      } else {
        u = rot_inner_at(d, i, key, key_digit, kl->beta, t, m);
        if (x == 0) u += mulmod(c0[orbit_shift(t, rot, H)], pmod, m);
        if (add) u += mulmod(cx[t], pmod, m);
      }
      o[t] = reduce(mulmod(reduce(u, m) - v, pinv, m), m);
    });
  }
}

// out = (out_add ? out : 0) + sum_k ct_k pt_k over n ciphertexts of lv+1
// limbs: ct_k at ct + k ct_stride, pt_k at pt + k pt_stride (pt null: plain
// sum).  Thread = one residue of c0 and of c1.
__global__ __launch_bounds__(256) void k_sum_cts(const double* __restrict__ ct, size_t ct_stride,
                                                 const double* __restrict__ pt, size_t pt_stride, int n, int lv, int N,
                                                 const ModQ* __restrict__ mods, int out_add, double* __restrict__ out) {
  const size_t Q = (size_t)(lv + 1) * N;
  const size_t idx = (size_t)blockIdx.x * 256 + threadIdx.x;
  if (idx >= Q) return;
  const ModQ m = mods[(blockIdx.x * 256) / N];
  double a0 = out_add ? out[idx] : 0.0, a1 = out_add ? out[Q + idx] : 0.0;
  int k = 0;
  // four terms' loads in flight; re-centred after every four: |a| < 5 q
  for (; k + 4 <= n; k += 4) {
    double c0[4], c1[4], p[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const double* c = ct + (size_t)(k + u) * ct_stride;
      c0[u] = c[idx];
      c1[u] = c[Q + idx];
      p[u] = pt ? pt[(size_t)(k + u) * pt_stride + idx] : 0.0;
    }
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      a0 += pt ? mulmod(c0[u], p[u], m) : c0[u];
      a1 += pt ? mulmod(c1[u], p[u], m) : c1[u];
    }
    a0 = reduce(a0, m);
    a1 = reduce(a1, m);
  }
  for (; k < n; ++k) {
    const double* c = ct + (size_t)k * ct_stride;
    const double p = pt ? pt[(size_t)k * pt_stride + idx] : 0.0;
    a0 += pt ? mulmod(c[idx], p, m) : c[idx];
    a1 += pt ? mulmod(c[Q + idx], p, m) : c[Q + idx];
  }
  out[idx] = reduce(a0, m);
  out[Q + idx] = reduce(a1, m);
}

// ---------------------------------------------------------------------------
template <int LOGN>
static void rotations_impl(const LaunchCtx& L, const RotBatch& b, const RotRun& r) {
  const dim3 block(NttShape<LOGN>::T);
  const KsLevel* kl = r.kl_dev;
  const bool one = LOGN <= 14 && fuse_transforms(r.alpha, b.n * r.n_tasks);
  const bool down_one = LOGN <= 14 && r.inner && fuse_transforms(r.alpha, b.n * 2 * (r.lv + 1));
  if constexpr (LOGN <= 14) {
    if (!r.shared_digits && one)
      hipLaunchKernelGGL(k_rot_modup_one<LOGN>, dim3(b.n * r.n_tasks), block, 0, L.stream, b, r.pre, kl, r.digits,
                         r.dig_stride, L.tb);
  }
  if (!r.shared_digits && !one) {
    hipLaunchKernelGGL(k_rot_modup_intt<LOGN>, dim3(b.n * (r.lv + 1)), block, 0, L.stream, b, r.pre, kl, r.yup, L.tb);
    hipLaunchKernelGGL(k_rot_modup_conv<LOGN>, dim3(b.n * r.n_tasks), block, 0, L.stream, r.yup, kl, r.digits,
                       r.dig_stride, L.tb);
  }
  if (r.inner)
    hipLaunchKernelGGL(k_rot_inner, dim3((1 << LOGN) / 256, r.lv + 1 + r.alpha, b.n), dim3(256), 0, L.stream, b, r.pre, r.add,
                       kl, r.digits, r.dig_stride, r.key_limbs, 1 << LOGN, L.tb.mods, r.inner);
  if constexpr (LOGN <= 14) {
    if (down_one) {
      hipLaunchKernelGGL(k_rot_down_one<LOGN>, dim3(b.n * 2 * (r.lv + 1)), block, 0, L.stream, b, kl, r.inner, L.tb);
      return;
    }
  }
  hipLaunchKernelGGL(k_rot_down_p<LOGN>, dim3(b.n * 2 * r.alpha), block, 0, L.stream, b, r.pre, kl, r.digits,
                     r.dig_stride, r.key_limbs, r.inner, r.ydown, L.tb);
  hipLaunchKernelGGL(k_rot_down_q<LOGN>, dim3(b.n * 2 * (r.lv + 1)), block, 0, L.stream, b, r.pre, r.add, kl, r.digits,
                     r.dig_stride, r.key_limbs, r.inner, r.ydown, L.tb);
}

hipError_t launch_rotations(const LaunchCtx& L, const RotBatch& b, const RotRun& r) {
  if (b.n <= 0) return hipSuccess;
  if (b.n > kRotsPerLaunch) return hipErrorInvalidValue;
  switch (L.logN) {
    case 12: rotations_impl<12>(L, b, r); break;
    case 13: rotations_impl<13>(L, b, r); break;
    case 14: rotations_impl<14>(L, b, r); break;
    case 15: rotations_impl<15>(L, b, r); break;
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

hipError_t launch_sum_cts(const LaunchCtx& L, const double* ct, size_t ct_stride, const double* pt, size_t pt_stride,
                          int n, int lv, int N, bool out_add, double* out) {
  const size_t Q = (size_t)(lv + 1) * N;
  hipLaunchKernelGGL(k_sum_cts, dim3((unsigned)(Q / 256)), dim3(256), 0, L.stream, ct, ct_stride, pt, pt_stride, n, lv, N,
                     L.tb.mods, out_add ? 1 : 0, out);
  return hipGetLastError();
}

}  // namespace pvfl

// Canonical-embedding encode/decode (FP64, gfx950) and the plaintext packing
// of the plans.
//
// Slots z_j (j < N/2) are the values at zeta^(5^j), zeta = exp(i pi / N).  With
// e_j = 5^j mod 2N = 4 f_j + 1 and w_k = m_k + i m_(k+N/2) (k < N/2):
//     z_j = sum_k (w_k zeta^k) W^(-k f_j),   W = exp(-2 pi i / (N/2)),
// a length-N/2 DFT of the twisted w, read at index f_j.  Encoding inverts it:
// place scale*z_j at f_j, forward DFT / (N/2), untwist by zeta^-k, round the
// real and imaginary parts half away from zero to m_k and m_(k+N/2).
// The complex transform runs in LDS (N/2 complex doubles = 8N bytes) as a
// radix-2 decimation-in-frequency FFT (natural order in, bit-reversed out).
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "encode_dev.hpp"
#include "ring15.hpp"

namespace pvfl {

// `parts` workgroups per plaintext (encode_parts): pack, encode, then each its
// share of the limbs reduced and transformed.  out[k][limb][N].
template <int LOGN>
LIMBS_KERNEL(LOGN) void k_encode_pt(EncodeArgs a, EncTabs et, LimbMap map, int parts,
                                                                 DevTabs tb, double* __restrict__ out) {
  __shared__ double2 s2[NttShape<LOGN>::LDS / 2];
  const int k = blockIdx.x / parts;
  const LimbRange lr = limb_part(map.n, blockIdx.x % parts, parts);
  if (lr.l0 >= lr.l1) return;
  encode_pt_body<LOGN>(a, k, et, map, lr, tb, s2, out + (size_t)k * map.n * (1 << LOGN));
}

// Input ciphertext messages: one workgroup per ciphertext, int64 coefficients
template <int LOGN>
__global__ __launch_bounds__(NttShape<LOGN>::T) void k_encode_ct_msg(EncodeArgs a, EncTabs et, int64_t* __restrict__ msg) {
  __shared__ double2 s2[NttShape<LOGN>::LDS / 2];
  encode_ct_body<LOGN>(a, (int)blockIdx.x, et, s2, msg + (size_t)blockIdx.x * (1 << LOGN));
}

// Output idx of a plan from its decoded slots slot(c, j) (output ciphertext
// c, slot j): the lazy rotate-and-sum of Sec. 4.3, added in slot order.
template <class Slot>
__device__ __forceinline__ double readout_value(const EncodeArgs& a, int ras_in_ct, int idx, Slot slot) {
  int c = 0, j0 = idx, step = 0, cnt = 1;
  switch (a.kind) {
    case 0: {
      const int rr = idx % a.bm;
      c = idx / a.bm;
      j0 = (rr / a.mprime) * a.bn + rr % a.mprime;
      step = a.mprime;
      cnt = a.bn / a.mprime;
      break;
    }
    case 1:
      if (a.bm < a.bn && !ras_in_ct) {
        step = a.bm;
        cnt = a.bn / a.bm;
      }
      break;
    case 3: {
      const int col = idx % a.n_out;
      c = col / a.pack;
      j0 = (col % a.pack) * a.width + idx / a.n_out;
      if (a.bm < a.bn) {
        step = a.bm;
        cnt = a.bn / a.bm;
      }
      break;
    }
    case 4:  // COL: row block c of N/2 rows, no rotate-and-sum
      c = idx / a.bm;
      j0 = idx % a.bm;
      break;
  }
  if (step == 0) return slot(c, j0);
  return sum_in_order(cnt, [&](int t) { return slot(c, j0 + t * step); });
}

// Decode and read-out of one output ciphertext per workgroup, N <= 2^14:
// centred CRT lift of the decrypted coefficient residues [nct][l+1][N]
// (canonical, binary64), twist, DFT with sign +1; the slots stay in LDS and
// the outputs that this ciphertext holds are summed from them.
template <int LOGN>
__global__ __launch_bounds__(NttShape<LOGN>::T) void k_decode_readout(const double* __restrict__ res, int lv, CrtTabs ct,
                                                                      EncTabs et, double inv_scale, EncodeArgs a,
                                                                      int ras_in_ct, double* __restrict__ y) {
  constexpr int N = 1 << LOGN, T = NttShape<LOGN>::T;
  __shared__ double2 w[NttShape<LOGN>::LDS / 2];
  const int c = blockIdx.x;
  decode_to_lds<LOGN>(res + (size_t)c * (lv + 1) * N, lv + 1, ct, et, w);
  const double* z = slots_in_order<LOGN>(w, et, inv_scale);
  auto slot = [&](int, int j) { return z[j]; };
  if (a.kind == 3) {  // the columns of this ciphertext, all rows
    const int col0 = c * a.pack, cols = min(a.pack, a.n_out - col0);
    for (int l = threadIdx.x; l < a.m * cols; l += T) {
      const int idx = (l / cols) * a.n_out + col0 + l % cols;
      y[idx] = readout_value(a, ras_in_ct, idx, slot);
    }
  } else {  // HYBRID and COL: row block c; DIAG and ROW have one ciphertext
    const int per = a.kind == 0 || a.kind == 4 ? a.bm : a.m, lo = c * per, hi = min(a.m, lo + per);
    for (int idx = lo + (int)threadIdx.x; idx < hi; idx += T) y[idx] = readout_value(a, ras_in_ct, idx, slot);
  }
}

template <int LOGN>
LIMBS_KERNEL(LOGN) void k_encode_out(EncodeArgs a, const double* __restrict__ v, int mode,
                                                                  int ras_in_ct, OutFactors fac, EncTabs et, LimbMap map,
                                                                  int parts, DevTabs tb, double* __restrict__ out) {
  __shared__ double2 s2[NttShape<LOGN>::LDS / 2];
  const int b = blockIdx.x / parts;
  const LimbRange lr = limb_part(map.n, blockIdx.x % parts, parts);
  if (lr.l0 >= lr.l1) return;
  encode_out_body<LOGN>(a, v, mode, ras_in_ct, b, fac, et, map, lr, tb, s2, out + (size_t)b * map.n * (1 << LOGN));
}

// out c0 = ct c0 + sign * pt, c1 copied, on nct ciphertexts of lv+1 limbs
__global__ __launch_bounds__(256) void k_out_add_pt(const double* __restrict__ ct, const double* __restrict__ pt, double sign,
                                                    int nct, int lv, int N, const ModQ* __restrict__ mods,
                                                    double* __restrict__ out) {
  const size_t Q = (size_t)(lv + 1) * N;
  const size_t idx = (size_t)blockIdx.x * 256 + threadIdx.x;
  if (idx >= (size_t)nct * 2 * Q) return;
  const size_t c = idx / (2 * Q), r = idx % (2 * Q);
  if (r >= Q) {
    out[idx] = ct[idx];
    return;
  }
  const int i = (int)(r / N);
  out[idx] = reduce(ct[idx] + sign * pt[c * Q + r], mods[i]);
}

// lazy rotate-and-sum / read-out of the decoded slots (Sec. 4.3)
__global__ __launch_bounds__(256) void k_readout(const double* __restrict__ z, EncodeArgs a, int ras_in_ct, int count,
                                                 double* __restrict__ y) {
  const int idx = blockIdx.x * 256 + threadIdx.x;
  if (idx >= count) return;
  y[idx] = readout_value(a, ras_in_ct, idx, [&](int c, int j) { return z[(size_t)c * a.slots + j]; });
}

// ---------------------------------------------------------------------------
template <int LOGN>
static void encode_pt_impl(const LaunchCtx& L, const EncodeArgs& a, const EncTabs& et, LimbMap map, int count, double* out) {
  const int parts = encode_parts(LOGN, count, map.n);
  if constexpr (LOGN == 15)
    launch15_encode_pt(L, a, et, map, count, parts, out);
  else
    hipLaunchKernelGGL(k_encode_pt<LOGN>, dim3(count * parts), dim3(NttShape<LOGN>::T), 0, L.stream, a, et, map, parts,
                       L.tb, out);
}
template <int LOGN>
static void encode_out_impl(const LaunchCtx& L, const EncodeArgs& a, const double* v, int mode, int ras_in_ct,
                            const OutFactors& fac, const EncTabs& et, LimbMap map, int count, double* out) {
  const int parts = encode_parts(LOGN, count, map.n);
  if constexpr (LOGN == 15)
    launch15_encode_out(L, a, v, mode, ras_in_ct, fac, et, map, count, parts, out);
  else
    hipLaunchKernelGGL(k_encode_out<LOGN>, dim3(count * parts), dim3(NttShape<LOGN>::T), 0, L.stream, a, v, mode, ras_in_ct,
                       fac, et, map, parts, L.tb, out);
}
template <int LOGN>
static void encode_ct_impl(const LaunchCtx& L, const EncodeArgs& a, const EncTabs& et, int count, int64_t* msg) {
  if constexpr (LOGN == 15)
    launch15_encode_ct(L, a, nullptr, et, count, msg);
  else
    hipLaunchKernelGGL(k_encode_ct_msg<LOGN>, dim3(count), dim3(NttShape<LOGN>::T), 0, L.stream, a, et, msg);
}
template <int LOGN>
static void decode_readout_impl(const LaunchCtx& L, const double* res, int nct, int lv, const CrtTabs& ct,
                                const EncTabs& et, double inv_scale, const EncodeArgs& a, int ras_in_ct, double* y) {
  if constexpr (LOGN <= 14)
    hipLaunchKernelGGL(k_decode_readout<LOGN>, dim3(nct), dim3(NttShape<LOGN>::T), 0, L.stream, res, lv, ct, et, inv_scale,
                       a, ras_in_ct, y);
}

#define DISPATCH_LOGN(L, FN, ...)                         \
  switch ((L).logN) {                                     \
    case 12: FN<12>(__VA_ARGS__); break;                  \
    case 13: FN<13>(__VA_ARGS__); break;                  \
    case 14: FN<14>(__VA_ARGS__); break;                  \
    case 15: FN<15>(__VA_ARGS__); break;                  \
    default: return hipErrorInvalidValue;                 \
  }

hipError_t launch_encode_pt(const LaunchCtx& L, const EncodeArgs& a, const EncTabs& et, LimbMap map, int count,
                            double* out) {
  if (count <= 0) return hipSuccess;
  DISPATCH_LOGN(L, encode_pt_impl, L, a, et, map, count, out);
  return hipGetLastError();
}
hipError_t launch_encode_ct(const LaunchCtx& L, const EncodeArgs& a, const EncTabs& et, int count, int64_t* msg) {
  DISPATCH_LOGN(L, encode_ct_impl, L, a, et, count, msg);
  return hipGetLastError();
}
hipError_t launch_decode_readout(const LaunchCtx& L, const double* res, int nct, int lv, const CrtTabs& ct,
                                 const EncTabs& et, double inv_scale, const EncodeArgs& a, int ras_in_ct, double* y) {
  if (L.logN > 14) return hipErrorInvalidValue;
  DISPATCH_LOGN(L, decode_readout_impl, L, res, nct, lv, ct, et, inv_scale, a, ras_in_ct, y);
  return hipGetLastError();
}
hipError_t launch_encode_out(const LaunchCtx& L, const EncodeArgs& a, const double* v, int mode, int ras_in_ct,
                             const OutFactors& fac, const EncTabs& et, LimbMap map, int count, double* out) {
  if (count <= 0) return hipSuccess;
  DISPATCH_LOGN(L, encode_out_impl, L, a, v, mode, ras_in_ct, fac, et, map, count, out);
  return hipGetLastError();
}
hipError_t launch_out_add_pt(const LaunchCtx& L, const double* ct, const double* pt, double sign, int nct, int lv, int N,
                             double* out) {
  const size_t tot = (size_t)nct * 2 * (lv + 1) * N;
  if (tot == 0) return hipSuccess;
  hipLaunchKernelGGL(k_out_add_pt, dim3((unsigned)((tot + 255) / 256)), dim3(256), 0, L.stream, ct, pt, sign, nct, lv, N,
                     L.tb.mods, out);
  return hipGetLastError();
}
hipError_t launch_readout(const LaunchCtx& L, const double* z, const EncodeArgs& a, int ras_in_ct, int count, double* y) {
  hipLaunchKernelGGL(k_readout, dim3((count + 255) / 256), dim3(256), 0, L.stream, z, a, ras_in_ct, count, y);
  return hipGetLastError();
}

}  // namespace pvfl

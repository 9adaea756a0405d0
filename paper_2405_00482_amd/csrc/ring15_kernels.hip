// Encoder and decoder kernels of the 2^15 ring.  They are a source file of
// their own for PVFL_OPAQUE_TID: a thread has 32 coefficients here, and the
// index arithmetic that the compiler would keep live across the limb loop does
// not fit beside them (512 plaintexts of 10 limbs: 1.20 ms with it and the
// coefficients kept in registers, 0.9 KiB of scratch memory per thread; 1.42
// with the coefficients parked in memory; 0.91 with both.  Messages of 16
// ciphertexts: 118, 68 and 48 us).
#define PVFL_OPAQUE_TID 1

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "encode_dev.hpp"
#include "ring15.hpp"

namespace pvfl {

constexpr int kT15 = NttShape<15>::T;
#define KERNEL15 __global__ __launch_bounds__(kT15)
#define LDS15 __shared__ double2 s2[NttShape<15>::LDS / 2]

// SPLIT: parts > 1 (a limb range known only at run time costs registers here:
// 512 plaintexts 0.98 instead of 0.92 ms)
template <bool SPLIT>
KERNEL15 void k_encode_pt15(EncodeArgs a, EncTabs et, LimbMap map, int parts, DevTabs tb, double* __restrict__ out) {
  LDS15;
  const int k = SPLIT ? blockIdx.x / parts : blockIdx.x;
  const LimbRange lr = SPLIT ? limb_part(map.n, blockIdx.x % parts, parts) : LimbRange{0, map.n};
  if (lr.l0 >= lr.l1) return;
  encode_pt_body<15>(a, k, et, map, lr, tb, s2, out + (size_t)k * map.n * (1 << 15));
}

KERNEL15 void k_encode_pt_batch15(const EncodeArgs* __restrict__ args, const int2* __restrict__ work, int nwork,
                                  const BatchProd* __restrict__ prods, EncTabs et, LimbMap map, DevTabs tb) {
  LDS15;
  const int per_xcd = (nwork + 7) / 8;  // as k_encode_pt_batch
  const int vt = (blockIdx.x & 7) * per_xcd + (blockIdx.x >> 3);
  if (vt >= nwork) return;
  const int2 wk = work[vt];
  encode_pt_body<15>(args[wk.x], wk.y, et, map, LimbRange{0, map.n}, tb, s2,
                     prods[wk.x].pt_out + (size_t)wk.y * map.n * (1 << 15));
}

KERNEL15 void k_encode_ct15(EncodeArgs a, const EncodeArgs* __restrict__ args, EncTabs et, int64_t* __restrict__ msg) {
  LDS15;
  int64_t* dst = msg + (size_t)blockIdx.x * (1 << 15);
  if (args)
    encode_ct_body<15>(args[blockIdx.x], 0, et, s2, dst);
  else
    encode_ct_body<15>(a, (int)blockIdx.x, et, s2, dst);
}

KERNEL15 void k_encode_out15(EncodeArgs a, const double* __restrict__ v, int mode, int ras_in_ct, OutFactors fac,
                             EncTabs et, LimbMap map, int parts, DevTabs tb, double* __restrict__ out) {
  LDS15;
  const int b = blockIdx.x / parts;
  const LimbRange lr = limb_part(map.n, blockIdx.x % parts, parts);
  if (lr.l0 >= lr.l1) return;
  encode_out_body<15>(a, v, mode, ras_in_ct, b, fac, et, map, lr, tb, s2, out + (size_t)b * map.n * (1 << 15));
}

// Decode alone at N = 2^15: slots z[c][j] = Re(.)/scale.  The first DIF stage
// (pairs k, k + M/2) runs in registers, then the two halves in LDS.
KERNEL15 void k_decode15(const double* __restrict__ res, int lv, CrtTabs ct,
                                                              EncTabs et, double inv_scale, double* __restrict__ z) {
  constexpr int LOGN = 15, N = 1 << LOGN, M = N / 2, T = NttShape<LOGN>::T, HM = M / 2;
  __shared__ double2 w[NttShape<LOGN>::LDS / 2];
  const int c = blockIdx.x;
  const double* base = res + (size_t)c * (lv + 1) * N;
  const int nl = lv + 1;
  double* zc = z + (size_t)c * M;
  double2 v0[HM / T];
  with_limbs(nl, [&](auto nl_c) {
    constexpr int NL = decltype(nl_c)::value;
    // twisted w_k = (m_k + i m_(k+N/2)) zeta^k
    auto twisted = [&](int k) {
      return cmul(make_double2(crt_lift<NL>(base, k, N, ct, nl), crt_lift<NL>(base, k + M, N, ct, nl)), et.twist[k]);
    };
#pragma unroll
    for (int u = 0; u < HM / T; ++u) {
      const int k = threadIdx.x + u * T;
      const double2 a0 = twisted(k), b0 = twisted(k + HM);
      w[cpad(k)] = make_double2(a0.x + b0.x, a0.y + b0.y);
      v0[u] = cmul(make_double2(a0.x - b0.x, a0.y - b0.y), cconj(et.fft_tw[k]));
    }
  });
#pragma unroll 1
  for (int h = 0; h < 2; ++h) {
    if (h) {
      __syncthreads();  // half 0's read-out is done
#pragma unroll
      for (int u = 0; u < HM / T; ++u) w[cpad(threadIdx.x + u * T)] = v0[u];
    }
    __syncthreads();
    fft_dif_half15(w, et.fft_tw, true);
    for (int j = threadIdx.x; j < M; j += T) {
      const int r = brev(et.slot2f[j], LOGN - 1);
      if ((r >> (LOGN - 2)) == h) zc[j] = w[cpad(r - h * HM)].x * inv_scale;
    }
  }
}

void launch15_encode_pt(const LaunchCtx& L, const EncodeArgs& a, const EncTabs& et, LimbMap map, int count, int parts,
                        double* out) {
  if (parts > 1)
    hipLaunchKernelGGL(k_encode_pt15<true>, dim3(count * parts), dim3(kT15), 0, L.stream, a, et, map, parts, L.tb, out);
  else
    hipLaunchKernelGGL(k_encode_pt15<false>, dim3(count), dim3(kT15), 0, L.stream, a, et, map, 1, L.tb, out);
}
void launch15_encode_pt_batch(const LaunchCtx& L, const EncodeArgs* args, const int2* work, int nwork,
                              const BatchProd* prods, const EncTabs& et, LimbMap map) {
  hipLaunchKernelGGL(k_encode_pt_batch15, dim3(8 * ((nwork + 7) / 8)), dim3(kT15), 0, L.stream, args, work, nwork, prods,
                     et, map, L.tb);
}
void launch15_encode_ct(const LaunchCtx& L, const EncodeArgs& a, const EncodeArgs* args, const EncTabs& et, int count,
                        int64_t* msg) {
  hipLaunchKernelGGL(k_encode_ct15, dim3(count), dim3(kT15), 0, L.stream, a, args, et, msg);
}
void launch15_encode_out(const LaunchCtx& L, const EncodeArgs& a, const double* v, int mode, int ras_in_ct,
                         const OutFactors& fac, const EncTabs& et, LimbMap map, int count, int parts,
                        double* out) {
  hipLaunchKernelGGL(k_encode_out15, dim3(count * parts), dim3(kT15), 0, L.stream, a, v, mode, ras_in_ct, fac, et, map, parts,
                     L.tb, out);
}
hipError_t launch_decode15(const LaunchCtx& L, const double* res, int nct, int lv, const CrtTabs& ct, const EncTabs& et,
                           double inv_scale, double* z) {
  if (L.logN != 15) return hipErrorInvalidValue;
  hipLaunchKernelGGL(k_decode15, dim3(nct), dim3(kT15), 0, L.stream, res, lv, ct, et, inv_scale, z);
  return hipGetLastError();
}

}  // namespace pvfl

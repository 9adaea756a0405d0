// Encoder/decoder argument structures (canonical embedding, plan packing).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "kernels.hpp"

namespace pvfl {

struct EncTabs {
  const uint32_t* slot2f;   // [N/2] slot j -> DFT index f_j = (5^j mod 2N - 1) / 4
  const uint32_t* f2slot;   // [N/2] the inverse permutation
  const double2* fft_tw;    // [N/4] exp(-2 pi i t / (N/2))
  const double2* twist;     // [N/2] zeta^k = exp(i pi k / N)
};

struct CrtTabs {
  const ModQ* mods;
  const double* garner_inv; // [kMaxLimbs][kMaxLimbs]: q_j^-1 mod q_i (centred), j < i
};

// Plan geometry as the packing kernels see it (all sizes padded to 2^k).
struct EncodeArgs {
  int kind;        // 0 HYBRID, 1 DIAG, 2 ROW, 3 CTMAT
  int m, n, ld;    // operand shape; ld = row stride of X (elements)
  const double* X; // plaintext matrix (pt encode) or encrypted operand (ct encode)
  int bm, bn, mprime, col_blocks, width, pack, n_out, n_out_cts, slots;
  int lbn, lmp, lw;  // log2 of bn, mprime, width (all powers of two)
  double scale;    // encoding scale
  double ind_scale;  // ROW: scale of the indicator plaintext
  int bsgs;          // HYBRID: baby-step size; diagonal i is stored rotated right by (i / bsgs) * bsgs
};

// per-limb factors (centred residues) of a plaintext encoded at a lower scale
struct OutFactors {
  double f[kMaxLimbs];
};

// Workgroups that share one plaintext's nl limbs, each repeating its FFT (worth
// 1.5 limbs' transforms): the number for which `count` plaintexts take the
// least time on 256 CUs holding 4, 2 or 1 workgroups at N = 2^12, 2^13, 2^14+.
// With more than a few rounds of workgroups it is one.  64 plaintexts of 4
// limbs at 2^13: 38 -> 23 us; 128 of 6 limbs at 2^14: 87 -> 62 us; one
// cleartext of 3 limbs at 2^13: 29 -> 16 us.
inline int encode_parts(int logN, int count, int nl) {
  const long slots = 256L * (logN <= 12 ? 4 : logN == 13 ? 2 : 1);
  int best = 1;
  double least = 0.0;
  for (int p = 1; p <= nl; ++p) {
    const double t = (double)(((long)count * p + slots - 1) / slots) * (1.5 + (nl + p - 1) / p);
    if (p == 1 || t < least) {
      best = p;
      least = t;
    }
  }
  return best;
}
hipError_t launch_encode_pt(const LaunchCtx& L, const EncodeArgs& a, const EncTabs& et, LimbMap map, int count,
                            double* out);
// cleartext at the plan's output scale (pvfl_encode_out): out[count][map.n][N]
hipError_t launch_encode_out(const LaunchCtx& L, const EncodeArgs& a, const double* v, int mode, int ras_in_ct,
                             const OutFactors& fac, const EncTabs& et, LimbMap map, int count, double* out);
// out c0 = ct c0 + sign * pt (c1 copied) on nct ciphertexts
hipError_t launch_out_add_pt(const LaunchCtx& L, const double* ct, const double* pt, double sign, int nct, int lv, int N,
                             double* out);
hipError_t launch_encode_ct(const LaunchCtx& L, const EncodeArgs& a, const EncTabs& et, int count, int64_t* msg);
// decode and lazy read-out of a plan's outputs (N <= 2^14); decode alone into slots z[nct][N/2] (N = 2^15)
hipError_t launch_decode_readout(const LaunchCtx& L, const double* res, int nct, int lv, const CrtTabs& ct,
                                 const EncTabs& et, double inv_scale, const EncodeArgs& a, int ras_in_ct, double* y);
hipError_t launch_decode15(const LaunchCtx& L, const double* res, int nct, int lv, const CrtTabs& ct, const EncTabs& et,
                           double inv_scale, double* z);
hipError_t launch_readout(const LaunchCtx& L, const double* z, const EncodeArgs& a, int ras_in_ct, int count, double* y);

}  // namespace pvfl

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
// least time when the busiest of 256 CUs has w workgroups.  Each beyond its
// first adds to the CU's time 0.4 of a workgroup alone at N = 2^12, 0.7 at 2^13
// (they run side by side but share its vector units) and a whole one from 2^14
// (256, 512, 1024 plaintexts of one workgroup each: 13.8, 19.1, 28.7 us with 2
// limbs at 2^12; 27.6, 42.7, 80.0 with 3 at 2^13; 60, 114, 223 with 4 at 2^14).
// With more than a few workgroups to a CU it is one.  64 plaintexts of 3 limbs at 2^13:
// 26 us with one workgroup each, 16 with three; 256 of them: 28 with one, 32 with
// two; 128 of 4 limbs at 2^14: 53 with one, 40 with two.
inline int encode_parts(int logN, int count, int nl) {
  const double beside = logN <= 12 ? 0.4 : logN == 13 ? 0.7 : 1.0;
  int best = 1;
  double least = 0.0;
  for (int p = 1; p <= nl; ++p) {
    const long w = ((long)count * p + 255) / 256;
    const double t = (1.5 + (nl + p - 1) / p) * (1.0 + beside * (w - 1));
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

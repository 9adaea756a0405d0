// Kernel argument structures and launcher declarations shared by the HIP
// kernels and the host side of the library.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "ntt_core.hpp"

namespace pvfl {

constexpr int kMaxLimbs = 24;   // primes of Q_L u P
constexpr int kMaxTasks = 128;  // ModUp (digit, limb) tasks per level
constexpr int kMaxAlpha = 4;    // special primes

// counter-based generator streams (top byte = purpose)
constexpr uint64_t kStreamSecret = 0x01ull << 56;
constexpr uint64_t kStreamEncA = 0x02ull << 56;  // | limb
constexpr uint64_t kStreamEncE = 0x03ull << 56;
constexpr uint64_t kStreamKeyA = 0x04ull << 56;  // | j<<40 | r<<24 | g
constexpr uint64_t kStreamKeyE = 0x05ull << 56;  // | j<<40 | g
constexpr uint64_t kStreamPkA = 0x06ull << 56;   // | limb: public key a
constexpr uint64_t kStreamPkE = 0x07ull << 56;   // public key error
constexpr uint64_t kStreamPkV = 0x08ull << 56;   // public-key encryption: ternary v
constexpr uint64_t kStreamPkE0 = 0x09ull << 56;  // public-key encryption: e0
constexpr uint64_t kStreamPkE1 = 0x0Aull << 56;  // public-key encryption: e1

struct LimbMap {
  int n;
  int idx[kMaxLimbs];
};

struct LaunchCtx {
  hipStream_t stream;
  DevTabs tb;
  int logN;
};

enum class NttOp { Fwd, Inv, ImportI64, ExportU64 };

struct KsTask {
  int digit, limb, prime, nsrc, src0;
  double hat[kMaxAlpha];  // [Q_j / q_src]_{prime}
};

// key-switching constants of one level l (device resident)
struct KsLevel {
  int lv, alpha, beta, K, n_q_total, n_tasks;
  double up_inv_hat[kMaxLimbs];              // limb i <= l: [(Q_j/q_i)^-1]_{q_i}, j = digit of i
  KsTask up_task[kMaxTasks];
  double down_inv_hat[kMaxAlpha];            // [(P/p_k)^-1]_{p_k}
  double down_hat[kMaxAlpha * kMaxLimbs];    // [k][i]: [P/p_k]_{q_i}
  double down_pinv[kMaxLimbs];               // [P^-1]_{q_i}
  double down_half[kMaxLimbs];               // floor(P/2) mod limb r of Q_l u P
  double p_mod[kMaxLimbs];                   // P mod q_i, centred
};

struct RotKeyArgs {
  int n_limbs, beta, alpha, n_q;
  double P_mod[kMaxLimbs];
};

// Up to kKeysPerLaunch rotation keys of one generation launch, passed by
// value: rotation amount and Galois element of each.
constexpr int kKeysPerLaunch = 64;
struct RotKeyList {
  int rot[kKeysPerLaunch];
  uint32_t galois[kKeysPerLaunch];
};

// Single rotations run side by side: rotation `it[k]` reads ciphertext ct
// [2][lv+1][N], writes out (not overlapping any input), uses key
// [beta][2][key_limbs][N] of its Galois element.  Passed by value.
constexpr int kRotsPerLaunch = 64;
struct RotItem {
  const double* ct;
  double* out;
  const double* key;
  int rot, pad;
};
struct RotBatch {
  int n;
  RotItem it[kRotsPerLaunch];
};
struct RotRun {
  const KsLevel* kl_dev;
  int lv, alpha, n_tasks, key_limbs;
  int pre;             // 1: the automorphism precedes the ModUp (O3); 0: hoisted order (O4)
  int add;             // 1: out = ct + RotL(ct); 0: out = RotL(ct)
  bool shared_digits;  // digits already hold the ModUp of the one ciphertext every item rotates (dig_stride 0)
  double* yup;         // [n][lv+1][N]
  double* digits;      // item k at digits + k * dig_stride, [beta][K][N]
  size_t dig_stride;
  double* ydown;       // [n][2][alpha][N]
  double* inner;       // [n][2][K][N]: the key products in a launch of their own; null: inside the transforms
};

struct RescaleArgs {
  double half_mod_last;            // floor(q_l / 2)
  double half_mod[kMaxLimbs];      // floor(q_l / 2) mod q_i
  double inv_last[kMaxLimbs];      // q_l^-1 mod q_i
};

struct DiagArgs {
  int N, K, lv, beta, mprime, chunk, key_limbs;  // chunk: diagonals per grid slice
  int add;                 // 1: add to what `part` holds
  size_t key_stride;
  const ModQ* mods;
  int limb_prime[kMaxLimbs];
  const double* pmod;      // P mod q_i, centred
  const double* pt;        // [n_pts][K][N]
  const int* slot_of_rot;  // [N/2] rotation amount -> key index
  const double* keys;
  const double* digits;    // [beta][K][N]
  const double* ct;        // [2][lv+1][N]
  double* part;            // [slices][2][K][N]
};

// Whether `blocks` workgroups of one transform each are one round, one
// workgroup per CU: then a transform repeated or moved to a workgroup of its
// own costs nothing.
inline bool few_transforms(int blocks) { return blocks <= 256; }

// Whether a key-switching step with `alpha` special primes and `blocks` target
// limbs makes both of its transforms in one launch, each target repeating the
// transform of its source limb: while one round of workgroups, one per CU,
// holds the targets.  Two launches and one, us: ModUp of one ciphertext at
// 2^12 / 2^13 / 2^14 15 -> 11, 29 -> 20, 54 -> 36, ModDown 17 -> 11, 31 -> 20,
// 47 -> 38 (since then, without products by one, 10, 17, 31 and 10, 18, 33);
// beyond the line, 300 targets at 2^14 62 -> 70, 372 at 2^13 no gain.  With
// alpha > 1 a target would repeat alpha transforms.
inline bool fuse_transforms(int alpha, int blocks) { return alpha == 1 && few_transforms(blocks); }

// Whether it splits every limb over N / 2^12 workgroups, `blocks` in all
// (SplitNtt): again while one round holds them.  One ciphertext, one launch
// and the split's two, us: ModUp at 2^13 / 2^14 17 -> 9 + 7, 31 -> 14 + 9,
// ModDown 18 -> 10 + 7, 33 -> 16 + 8 (the rotations' steps gain nothing at 2^13
// and stay in one launch).
inline bool split_transforms(int alpha, int blocks) { return alpha == 1 && blocks <= 256; }

hipError_t launch_ntt(const LaunchCtx& L, NttOp op, const void* in, void* out, int nblocks, LimbMap map);
hipError_t launch_keygen(const LaunchCtx& L, uint64_t seed, double* sk, int n_mod);
// nct ciphertexts [nct][2][lv+1][N] from messages [nct][N]; ciphertext c uses seed + c
// public key (b, a) = (-a s + e, a) over the nl = L+1 ciphertext primes: pk [2][nl][N]
hipError_t launch_pk_gen(const LaunchCtx& L, const double* sk, uint64_t seed, int nl, double* pk);
// public-key encryption at level lv: c = v (b, a) + (m + e0, e1); pk_stride = limbs per pk half
hipError_t launch_encrypt_pk(const LaunchCtx& L, const int64_t* msg, int nct, const double* pk, int pk_nl,
                             uint64_t seed, int lv, double* ct);
hipError_t launch_encrypt(const LaunchCtx& L, const int64_t* msg, int nct, const double* sk, uint64_t seed, int lv,
                          double* ct, double* const* ct_tab = nullptr);
hipError_t launch_decrypt_u64(const LaunchCtx& L, const double* ct, const double* sk, int lv, uint64_t* out);
hipError_t launch_decrypt_f64(const LaunchCtx& L, const double* ct, int nct, const double* sk, int lv, double* out,
                              const double* const* ct_tab = nullptr);
hipError_t launch_rotkey_gen(const LaunchCtx& L, const double* sk, const RotKeyList& list, int nkeys, uint64_t seed,
                             const RotKeyArgs& ka, double* keys);
// ModUp of the c1 halves of nct ciphertexts (ct + c*ct_stride); y holds
// [nct][lv+1][N] coefficient scratch; digits of ciphertext c at digits + c*dig_stride
hipError_t launch_modup(const LaunchCtx& L, const double* ct, size_t ct_stride, int nct, int lv, int alpha,
                        const KsLevel* kl_dev, int n_tasks, double* y, double* digits, size_t dig_stride,
                        const double* const* ct_tab = nullptr);
// out_tab (optional): output of poly x at out_tab[x/2] + (x%2)*(lv+1)*N
hipError_t launch_moddown(const LaunchCtx& L, const double* u, int npoly, int lv, int alpha, const KsLevel* kl_dev,
                          double* y, double* out, double* const* out_tab = nullptr);
// npoly polys (pairs of one ciphertext at in + pair * in_stride; 0 polys apart = one shared ciphertext), each
// limb times pt + pair * pt_stride first when pt is given
hipError_t launch_rescale(const LaunchCtx& L, const double* in, int npoly, int lv, const RescaleArgs& ra, double* out,
                          size_t in_stride, const double* pt = nullptr, size_t pt_stride = 0);
hipError_t launch_rotations(const LaunchCtx& L, const RotBatch& b, const RotRun& r);
// out = (out_add ? out : 0) + sum_k ct_k pt_k (pt null: plain sum), ct_k at ct + k ct_stride, pt_k at pt + k pt_stride
hipError_t launch_sum_cts(const LaunchCtx& L, const double* ct, size_t ct_stride, const double* pt, size_t pt_stride,
                          int n, int lv, int N, bool out_add, double* out);
// one product's diagonals in `slices` slices of a.chunk
hipError_t launch_diag_lazy(const LaunchCtx& L, const DiagArgs& a, int slices);
// baby-step/giant-step inner sums of every giant step, a.part = [g][2][K][N]
hipError_t launch_diag_bsgs(const LaunchCtx& L, const DiagArgs& a, int bs, int g);
// part[n][2][K][N] summed into acc[2][K][N]
hipError_t launch_sum_partials(const LaunchCtx& L, const double* part, int n, int K, int N, LimbMap limb_prime,
                               double* acc);
// Alg. 3: out[k] = sum_i ct[i] * pt[i][k]   (ct [nct][2][lv+1][N], pt [nct][nout][lv+1][N])
hipError_t launch_ctmat(const LaunchCtx& L, const double* ct, const double* pt, int nct, int nout, int lv, int N,
                        double* out);
hipError_t launch_scale_by_p(const LaunchCtx& L, const double* ct, int lv, int N, const double* pmod_dev, double* out,
                             int nct = 1, const double* const* ct_tab = nullptr);
hipError_t launch_ct_mul_pt(const LaunchCtx& L, const double* ct, const double* pt, int lv, int N, double* out);
hipError_t launch_ct_add(const LaunchCtx& L, const double* a, const double* b, int lv, int N, double* out);
}  // namespace pvfl

// Batched execution of many independent products (uneven shapes) sharing one
// context, level and rotation-key set: every phase of the path is one launch
// over all products, and the fused diagonal kernel streams each rotation key
// once per group of products instead of once per product.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "batch.hpp"
#include "encode_dev.hpp"
#include "he_dev.hpp"
#include "ring15.hpp"

namespace pvfl {

// ---------------------------------------------------------------------------
// fused hoisted rotations x diagonals, lazy ModDown, shared keys.
// Block (tile, limb r, work item w): work item = (product group, diagonals
// [i0, i1)); the tile holds 256 consecutive evaluation indices (one half of
// the orbit order), one per thread.  For each diagonal the key limbs
// (b_j, a_j)[r][t] are loaded once and applied to every product of the group
// that has it:
//   acc0_p += pt_{p,i} (P phi_i(c0_p) + sum_j phi_i(D_{p,j}) b_{i,j})
//   acc1_p += pt_{p,i} (                sum_j phi_i(D_{p,j}) a_{i,j})
// phi_i is a shift by i inside the orbit half, so every digit (and P c0) row
// a work item reads is the window [t0 + i0, t0 + tile + i1) of that row: it
// is staged in LDS once and the shifted reads of the loop become LDS reads.
// Partial sums per (product, chunk) go to part[prod.part0 + i0 / CH].
//
// What bounds it: per (product, diagonal, index) 47 binary64 operations, 40
// bytes from LDS and, over PG products, 8 plaintext bytes plus 16 BETA / PG
// key bytes through the vector cache, which takes one wave load per 16
// cycles whatever its width.  Four products of one index share the key
// loads; two products of two indices (half the products per key load)
// measured slower.  A load takes 16 bytes per lane and brings a wave's values
// of two diagonals (swap_halves), half the vector cache's work for two
// vector instructions; with 8-byte loads of one diagonal that cache was the
// busiest unit, 2.5 of 3.5 ms.  64 products at N = 2^14, BETA = 4 (15.6 GB from
// memory, 2.6 ms at the read rate): 3.83 -> 3.48 (exact sums, four products)
// -> 3.25 ms; 16 products of 512 diagonals at 2^15 (keys from L2, operations
// 4.7 ms): 8.6 -> 6.9 -> 6.3 (shared plaintexts) -> 6.2 ms.  Tried on the form
// of 8-byte loads: loads one, two and three diagonals ahead of their use
// (3.5 - 3.8 and 6.7 - 7.6 ms), two indices per thread (3.6 - 4.3 and 7.4 - 9.2).
// ---------------------------------------------------------------------------
// Row stride of the staged windows (doubles): a compile-time constant for the
// usual chunk lengths, so that every row of the stage is one LDS address plus
// an immediate offset.
template <int CHX>
__host__ __device__ constexpr int stage_row(int ch) {
  return (256 + (CHX ? CHX : ch) + 1) & ~1;
}

typedef double PairOfDoubles __attribute__((ext_vector_type(2), aligned(8)));
typedef const __attribute__((address_space(1))) PairOfDoubles* GlobalPair;
// A wave's 64 values of two rows from one 16-byte load per lane: lanes 0..31
// loaded the value pairs of the first row, lanes 32..63 those of the second.
// Swapping the upper half of x with the lower half of y leaves in x the first
// row and in y the second, value 2 l in lane l < 32 and value 2 (l - 32) + 1 in
// lane l >= 32.
__device__ __forceinline__ void swap_halves(PairOfDoubles v, double& r0, double& r1) {
  const uint64_t x = (uint64_t)__double_as_longlong(v.x), y = (uint64_t)__double_as_longlong(v.y);
  const auto lo = __builtin_amdgcn_permlane32_swap((uint32_t)x, (uint32_t)y, false, false);
  const auto hi = __builtin_amdgcn_permlane32_swap((uint32_t)(x >> 32), (uint32_t)(y >> 32), false, false);
  r0 = __longlong_as_double((long long)((uint64_t)lo[0] | ((uint64_t)hi[0] << 32)));
  r1 = __longlong_as_double((long long)((uint64_t)lo[1] | ((uint64_t)hi[1] << 32)));
}

template <int PG, int BETA, int CHX, bool SHARED>
__global__ __launch_bounds__(256) void k_diag_batch(BatchDiagArgs a) {
  extern __shared__ double stage[];  // [PG][BETA + 1][win]
  constexpr int TILE = 256;
  // Workgroups are dispatched round-robin over the 8 XCDs; give each XCD a
  // contiguous range of the task list so that tasks sharing a key tile (same
  // chunk, tile and limb, different product groups) run on one L2.
  const int bid = blockIdx.x;
  const int vt = (bid & 7) * a.per_xcd + (bid >> 3);
  if (vt >= a.n_tasks) return;
  const DiagTask task = a.tasks[vt];
  const int r = task.limb;
  const DiagWork w = a.work[task.work];
  const DiagGroup& G = a.groups[w.grp];
  const int N = a.N, half = N >> 1, K = a.K;
  const int t0 = task.tile * TILE;
  const unsigned tid = threadIdx.x;
  // the thread's index of the tile (swap_halves), and where its value pairs start
  const bool upper = tid & 32u;
  const unsigned pair = (tid & ~63u) + 2 * (tid & 31u), tl = pair + (upper ? 1u : 0u);
  const size_t limbN = (size_t)r * N;
  const int pi = a.limb_prime[r];
  const int klimb = a.key_limb[r];
  const bool isq = r <= a.lv;
  const ModQ m = a.mods[pi];
  const int np = G.np;
  const int win = stage_row<CHX>(a.CH);
  const int span = TILE + (w.i1 - w.i0);
  const size_t KN = (size_t)K * N;
  const size_t Qoff = (size_t)(a.lv + 1) * N;
  // Stage the digit rows and P c0 (zero on the special limbs) of every
  // product: all of a thread's loads are issued before any is stored, so that
  // a task waits once for its windows and not once per row.
  // Even and odd places of a row lie in separate halves: the shifted reads of
  // the two half-waves are then stride one.
  const int oddrow = win >> 1;
  for (int x = (int)tid; x < span; x += TILE) {
    const size_t at = (size_t)((t0 & half) | ((t0 + w.i0 + x) & (half - 1)));
    double v[PG][BETA + 1];
#pragma unroll
    for (int p = 0; p < PG; ++p) {
      const int prod = G.prod[p < np ? p : 0];
      const double* dig = a.digits + (size_t)prod * a.dig_stride + limbN;
      // read once per task: streamed past L2 as well
#pragma unroll
      for (int j = 0; j < BETA; ++j) v[p][j] = __builtin_nontemporal_load(gmem(dig + (size_t)j * KN) + at);
      v[p][BETA] = isq ? __builtin_nontemporal_load(gmem(a.pc + (size_t)prod * a.pc_stride + limbN) + at) : 0.0;
    }
#pragma unroll
    for (int p = 0; p < PG; ++p)
#pragma unroll
      for (int j = 0; j <= BETA; ++j) stage[(size_t)(p * (BETA + 1) + j) * win + (x & 1) * oddrow + (x >> 1)] = v[p][j];
  }
  __syncthreads();
  int mp[PG];
  const double* ptp[PG];
#pragma unroll
  for (int p = 0; p < PG; ++p) {
    const BatchProd& B = a.prods[G.prod[p < np ? p : 0]];
    mp[p] = p < np ? B.mprime : 0;
    ptp[p] = B.pt + limbN + t0;
  }
  int mp_all = mp[0];
#pragma unroll
  for (int p = 1; p < PG; ++p) mp_all = min(mp_all, mp[p]);
  // Exact sums of products (fp64_mod.hpp).  Bounds with B = 2^b > q, b <= 48:
  // keys and converted digits are centred, a digit's own limb is below q, so
  // |sum_j D_j key_j| <= 1.25 B^2 < 0.43 * 2^(2b + 2) (BETA <= 4) and its fold
  // is below 1.5 B, 2 B with P c0.  Plaintexts are below q: nine terms stay
  // below 18 B^2 < 0.43 * 2^(2b + 6), their rounding errors below 9 * 2^49.
  const double cin = acc_offset(m.q, 2), cout = acc_offset(m.q, 6);
  double hi0[PG], lo0[PG], hi1[PG], lo1[PG];
#pragma unroll
  for (int p = 0; p < PG; ++p) {
    hi0[p] = hi1[p] = cout;
    lo0[p] = lo1[p] = 0.0;
  }
  int cnt = 0;
  int i = w.i0;
  if (i == 0) {  // diagonal 0: no rotation; P c0 on the Q limbs
    if (isq) {
#pragma unroll
      for (int p = 0; p < PG; ++p) {
        if (p >= np) continue;
        const double* pcs = stage + (size_t)(p * (BETA + 1) + BETA) * win;
        const double pv = gmem(ptp[p])[tl];
        acc_mac(pv, pcs[(upper ? oddrow : 0) + (pair >> 1)], hi0[p], lo0[p]);
        acc_mac(pv, gmem(a.pc)[(size_t)G.prod[p] * a.pc_stride + Qoff + limbN + t0 + tl], hi1[p], lo1[p]);
      }
    }
    ++i;
    ++cnt;
  }
  // The slots of a chunk of at most 64 diagonals sit in one register across
  // the wave: a scalar load per diagonal would have to be waited for together
  // with the LDS reads.
  const int lane_slot = CHX && a.slot_of_rot ? a.slot_of_rot[min(w.i0 + (int)(tid & 63u), w.i1 - 1)] : 0;
  // a row's place idx + o (o = i - i0): even o at `even` + o / 2, odd o at `odd` + (o - 1) / 2
  const unsigned even = (upper ? oddrow : 0) + (pair >> 1), odd = (upper ? 1 : oddrow) + (pair >> 1);
  const double* keyl = a.keys + (size_t)klimb * N + t0;
  const unsigned pair_next = pair + (upper ? (unsigned)KN : 0u);
  for (; i < w.i1; i += 2) {
    // Diagonals i and i + 1 (the last one alone: i again, unused).  Key limbs
    // (b_j, a_j) of both rotations, whose keys sit at these slots of the key set
    const bool two = i + 1 < w.i1;
    const int i1 = two ? i + 1 : i;
    const int slot0 = CHX ? __builtin_amdgcn_readlane(lane_slot, i - w.i0) : a.slot_of_rot[i];
    const int slot1 = CHX ? __builtin_amdgcn_readlane(lane_slot, i1 - w.i0) : a.slot_of_rot[i1];
    const auto* key0 = scalar_base(keyl + (size_t)slot0 * a.key_stride);
    const auto* key1 = scalar_base(keyl + (size_t)slot1 * a.key_stride);
    const auto* key = (upper ? key1 : key0) + pair;
    double kb[2][BETA], ka[2][BETA], pv[2][PG];
    PairOfDoubles lb[BETA], la[BETA], lp[PG];
#pragma unroll
    for (int j = 0; j < BETA; ++j) {
      lb[j] = *(GlobalPair)(key + (size_t)(2 * j) * a.key_limbs * N);
      la[j] = *(GlobalPair)(key + (size_t)(2 * j + 1) * a.key_limbs * N);
    }
    // Plaintexts of the diagonals (row 0 for a product without one, so that the
    // loads are unconditional).  They are read once: streamed past L2, so that
    // they do not evict the key tile the other product groups still need.
    auto row = [&](int p) {
      const bool next = two && i1 < mp[p];  // else both halves read the one row
      return (GlobalPair)(scalar_base(ptp[p] + (size_t)(i < mp[p] ? i : 0) * KN) + (next ? pair_next : pair));
    };
    if constexpr (SHARED) {  // one load for the group, from L2 for the groups after the first
      lp[0] = *row(0);
    } else {
#pragma unroll
      for (int p = 0; p < PG; ++p) lp[p] = __builtin_nontemporal_load(row(p));
    }
#pragma unroll
    for (int j = 0; j < BETA; ++j) {
      swap_halves(lb[j], kb[0][j], kb[1][j]);
      swap_halves(la[j], ka[0][j], ka[1][j]);
    }
#pragma unroll
    for (int p = 0; p < PG; ++p) {
      if (!SHARED || p == 0) {
        swap_halves(lp[p], pv[0][p], pv[1][p]);
      } else {
        pv[0][p] = pv[0][0];
        pv[1][p] = pv[1][0];
      }
    }
    const int o = i - w.i0;
    const double* st0 = stage + ((o & 1 ? odd : even) + (unsigned)(o >> 1));
    const double* st1 = stage + ((o & 1 ? even : odd) + (unsigned)((o + 1) >> 1));
    auto term = [&](int p, int d) {
      const double* st = d ? st1 : st0;
      const double d0 = st[(p * (BETA + 1)) * win];
      double h0, l0, h1, l1;
      acc_first(d0, kb[d][0], cin, h0, l0);
      acc_first(d0, ka[d][0], cin, h1, l1);
#pragma unroll
      for (int j = 1; j < BETA; ++j) {
        const double dj = st[(p * (BETA + 1) + j) * win];
        acc_mac(dj, kb[d][j], h0, l0);
        acc_mac(dj, ka[d][j], h1, l1);
      }
      l0 += st[(p * (BETA + 1) + BETA) * win];
      acc_mac(pv[d][p], acc_fold(h0, l0, m), hi0[p], lo0[p]);
      acc_mac(pv[d][p], acc_fold(h1, l1, m), hi1[p], lo1[p]);
    };
    if (two && i1 < mp_all) {  // both diagonals of every product: one block without branches
#pragma unroll
      for (int d = 0; d < 2; ++d)
#pragma unroll
        for (int p = 0; p < PG; ++p) term(p, d);
    } else {
#pragma unroll
      for (int p = 0; p < PG; ++p) {
        if (i < mp[p]) term(p, 0);
        if (two && i1 < mp[p]) term(p, 1);
      }
    }
    if ((cnt += 2) >= 8) {  // fold the sums after 8 (9 in the chunk holding diagonal 0) terms
#pragma unroll
      for (int p = 0; p < PG; ++p) {
        lo0[p] = reduce(acc_fold(hi0[p], lo0[p], m), m);
        lo1[p] = reduce(acc_fold(hi1[p], lo1[p], m), m);
        hi0[p] = hi1[p] = cout;
      }
      cnt = 0;
    }
  }
  const int chunk = w.i0 / a.CH;
#pragma unroll
  for (int p = 0; p < PG; ++p) {
    if (p >= np || w.i0 >= mp[p]) continue;
    double* part = a.part + (size_t)(a.prods[G.prod[p]].part0 + chunk) * 2 * KN + limbN + t0 + tl;
    // summed by a later launch: keep them out of L2
    __builtin_nontemporal_store(reduce(acc_fold(hi0[p], lo0[p], m), m), part);
    __builtin_nontemporal_store(reduce(acc_fold(hi1[p], lo1[p], m), m), part + KN);
  }
}

// acc[p] = sum of the chunk partials of product p;  acc [count][2][K][N]
__global__ __launch_bounds__(256) void k_sum_partials_batch(const double* __restrict__ part, const BatchProd* __restrict__ prods,
                                                           int CH, int K, int N, LimbMap limb_prime,
                                                           const ModQ* __restrict__ mods, double* __restrict__ acc) {
  const size_t tot = (size_t)2 * K * N;
  const size_t idx = (size_t)blockIdx.x * 256 + threadIdx.x;
  if (idx >= tot) return;
  const int p = blockIdx.y;
  const BatchProd B = prods[p];
  const int nch = (B.mprime + CH - 1) / CH;
  const int r = (int)((idx / N) % K);
  const ModQ m = mods[limb_prime.idx[r]];
  // eight partials' loads in flight at a time, added in chunk order with a
  // re-centring after every eighth (|v| < 8.5 q): the per-call form's sum
  const double* src = part + (size_t)B.part0 * tot + idx;
  double v = 0.0;
  int c = 0;
  for (; c + 8 <= nch; c += 8) {
    double t[8];
#pragma unroll
    for (int u = 0; u < 8; ++u) t[u] = __builtin_nontemporal_load(gmem(src) + (size_t)(c + u) * tot);
#pragma unroll
    for (int u = 0; u < 8; ++u) v += t[u];
    v = reduce(v, m);
  }
  for (; c < nch; ++c) v += __builtin_nontemporal_load(gmem(src) + (size_t)c * tot);
  acc[(size_t)p * tot + idx] = reduce(v, m);
}

// Workgroups go round-robin over the 8 XCDs; each XCD takes a contiguous
// range of the (product, diagonal) list so that neighbouring diagonals of one
// product, which read neighbouring columns of X, share its L2.
template <int LOGN>
LIMBS_KERNEL(LOGN) void k_encode_pt_batch(const EncodeArgs* __restrict__ args,
                                                                       const int2* __restrict__ work, int nwork,
                                                                       const BatchProd* __restrict__ prods, EncTabs et,
                                                                       LimbMap map, DevTabs tb) {
  __shared__ double2 s2[NttShape<LOGN>::LDS / 2];
  const int per_xcd = (nwork + 7) / 8;
  const int vt = (blockIdx.x & 7) * per_xcd + (blockIdx.x >> 3);
  if (vt >= nwork) return;
  const int2 wk = work[vt];
  const EncodeArgs a = args[wk.x];
  double* out = prods[wk.x].pt_out + (size_t)wk.y * map.n * (1 << LOGN);
  encode_pt_body<LOGN>(a, wk.y, et, map, LimbRange{0, map.n}, tb, s2, out);
}

template <int LOGN>
__global__ __launch_bounds__(NttShape<LOGN>::T) void k_encode_ct_batch(const EncodeArgs* __restrict__ args, EncTabs et,
                                                                       int64_t* __restrict__ msg) {
  __shared__ double2 s2[NttShape<LOGN>::LDS / 2];
  encode_ct_body<LOGN>(args[blockIdx.x], 0, et, s2, msg + (size_t)blockIdx.x * (1 << LOGN));
}

// output row idx of a product from its decoded slots slot(j): the lazy
// rotate-and-sum, added in slot order
template <class Slot>
__device__ __forceinline__ double readout_row(const EncodeArgs& a, int idx, Slot slot) {
  if (a.kind == 0) {
    const int rr = idx, g = rr / a.mprime, rho = rr % a.mprime;
    return sum_in_order(a.bn / a.mprime, [&](int t) { return slot(g * a.bn + rho + t * a.mprime); });
  }
  if (a.bm >= a.bn) return slot(idx);
  return sum_in_order(a.bn / a.bm, [&](int t) { return slot(idx + t * a.bm); });
}

__global__ __launch_bounds__(256) void k_readout_batch(const double* __restrict__ z, const EncodeArgs* __restrict__ args,
                                                       const BatchProd* __restrict__ prods, int slots) {
  const int p = blockIdx.y;
  const EncodeArgs a = args[p];
  const int idx = blockIdx.x * 256 + threadIdx.x;
  if (idx >= a.m) return;
  const double* zp = z + (size_t)p * slots;
  prods[p].y[idx] = readout_row(a, idx, [&](int j) { return zp[j]; });
}

// Decode and read-out in one workgroup per product (N <= 2^14): the slots
// stay in LDS and each row's sum reads them there, in the order of additions of
// k_readout_batch.
template <int LOGN>
__global__ __launch_bounds__(NttShape<LOGN>::T) void k_decode_readout_batch(const double* __restrict__ res, int lv,
                                                                            CrtTabs ct, EncTabs et, double inv_scale,
                                                                            const EncodeArgs* __restrict__ args,
                                                                            const BatchProd* __restrict__ prods) {
  constexpr int N = 1 << LOGN, T = NttShape<LOGN>::T;
  __shared__ double2 w[NttShape<LOGN>::LDS / 2];
  const int p = blockIdx.x;
  decode_to_lds<LOGN>(res + (size_t)p * (lv + 1) * N, lv + 1, ct, et, w);
  const EncodeArgs a = args[p];
  double* y = prods[p].y;
  const double* z = slots_in_order<LOGN>(w, et, inv_scale);
  for (int idx = threadIdx.x; idx < a.m; idx += T) y[idx] = readout_row(a, idx, [&](int j) { return z[j]; });
}

// ---------------------------------------------------------------------------
#define DISPATCH_LOGN(L, FN, ...)                         \
  switch ((L).logN) {                                     \
    case 12: FN<12>(__VA_ARGS__); break;                  \
    case 13: FN<13>(__VA_ARGS__); break;                  \
    case 14: FN<14>(__VA_ARGS__); break;                  \
    case 15: FN<15>(__VA_ARGS__); break;                  \
    default: return hipErrorInvalidValue;                 \
  }

template <int PG, int BETA, int CHX, bool SHARED>
static hipError_t diag_batch_run(const LaunchCtx& L, const BatchDiagArgs& a) {
  const size_t lds = sizeof(double) * (size_t)PG * (BETA + 1) * stage_row<CHX>(a.CH);
  if (lds > kDiagMaxLds) return hipErrorInvalidValue;
  // dynamic LDS above the default limit must be opted in once per kernel instance
  static const hipError_t opt_in = hipFuncSetAttribute((const void*)k_diag_batch<PG, BETA, CHX, SHARED>,
                                                       hipFuncAttributeMaxDynamicSharedMemorySize, (int)kDiagMaxLds);
  if (opt_in != hipSuccess) return opt_in;
  hipLaunchKernelGGL((k_diag_batch<PG, BETA, CHX, SHARED>), dim3(8 * a.per_xcd), dim3(256), lds, L.stream, a);
  return hipGetLastError();
}
// Products that share their plaintexts (the columns of one matrix) load them
// once per group: 16 products of 512 diagonals at 2^15 6.64 -> 6.29 ms (9 loads
// per diagonal and index of four products instead of 12).
template <int PG, int BETA>
static hipError_t diag_batch_ch(const LaunchCtx& L, const BatchDiagArgs& a) {
  if (a.CH > kDiagFixedChunk) return diag_batch_run<PG, BETA, 0, false>(L, a);
  if constexpr (PG > 1)
    if (a.shared_pt) return diag_batch_run<PG, BETA, kDiagFixedChunk, true>(L, a);
  return diag_batch_run<PG, BETA, kDiagFixedChunk, false>(L, a);
}
template <int PG>
static hipError_t diag_batch_pg(const LaunchCtx& L, const BatchDiagArgs& a, int beta) {
  switch (beta) {
    case 1: return diag_batch_ch<PG, 1>(L, a);
    case 2: return diag_batch_ch<PG, 2>(L, a);
    case 3: return diag_batch_ch<PG, 3>(L, a);
    case 4: return diag_batch_ch<PG, 4>(L, a);
  }
  return hipErrorInvalidValue;
}

hipError_t launch_diag_batch(const LaunchCtx& L, const BatchDiagArgs& a, int pg, int beta) {
  if (a.n_tasks <= 0) return hipSuccess;
  switch (pg) {
    case 1: return diag_batch_pg<1>(L, a, beta);
    case 2: return diag_batch_pg<2>(L, a, beta);
    case 4: return diag_batch_pg<4>(L, a, beta);
  }
  return hipErrorInvalidValue;
}

hipError_t launch_sum_partials_batch(const LaunchCtx& L, const double* part, const BatchProd* prods, int count, int CH,
                                     int K, int N, LimbMap limb_prime, double* acc) {
  const size_t tot = (size_t)2 * K * N;
  hipLaunchKernelGGL(k_sum_partials_batch, dim3((unsigned)((tot + 255) / 256), count), dim3(256), 0, L.stream, part, prods,
                     CH, K, N, limb_prime, L.tb.mods, acc);
  return hipGetLastError();
}

template <int LOGN>
static void enc_pt_batch_impl(const LaunchCtx& L, const EncodeArgs* args, const int2* work, int nwork,
                              const BatchProd* prods, const EncTabs& et, LimbMap map) {
  if constexpr (LOGN == 15)
    launch15_encode_pt_batch(L, args, work, nwork, prods, et, map);
  else
    hipLaunchKernelGGL(k_encode_pt_batch<LOGN>, dim3(8 * ((nwork + 7) / 8)), dim3(NttShape<LOGN>::T), 0, L.stream, args,
                       work, nwork, prods, et, map, L.tb);
}
hipError_t launch_encode_pt_batch(const LaunchCtx& L, const EncodeArgs* args, const int2* work, int nwork,
                                  const BatchProd* prods, const EncTabs& et, LimbMap map) {
  if (nwork <= 0) return hipSuccess;
  DISPATCH_LOGN(L, enc_pt_batch_impl, L, args, work, nwork, prods, et, map);
  return hipGetLastError();
}

template <int LOGN>
static void enc_ct_batch_impl(const LaunchCtx& L, const EncodeArgs* args, int count, const EncTabs& et, int64_t* msg) {
  if constexpr (LOGN == 15)
    launch15_encode_ct(L, EncodeArgs{}, args, et, count, msg);
  else
    hipLaunchKernelGGL(k_encode_ct_batch<LOGN>, dim3(count), dim3(NttShape<LOGN>::T), 0, L.stream, args, et, msg);
}
hipError_t launch_encode_ct_batch(const LaunchCtx& L, const EncodeArgs* args, int count, const EncTabs& et, int64_t* msg) {
  DISPATCH_LOGN(L, enc_ct_batch_impl, L, args, count, et, msg);
  return hipGetLastError();
}

template <int LOGN>
static void decode_readout_impl(const LaunchCtx& L, const double* res, int count, int lv, const CrtTabs& ct,
                                const EncTabs& et, double inv_scale, const EncodeArgs* args, const BatchProd* prods) {
  if constexpr (LOGN <= 14)
    hipLaunchKernelGGL(k_decode_readout_batch<LOGN>, dim3(count), dim3(NttShape<LOGN>::T), 0, L.stream, res, lv, ct, et,
                       inv_scale, args, prods);
}
hipError_t launch_decode_readout_batch(const LaunchCtx& L, const double* res, int count, int lv, const CrtTabs& ct,
                                       const EncTabs& et, double inv_scale, const EncodeArgs* args,
                                       const BatchProd* prods) {
  if (L.logN > 14) return hipErrorInvalidValue;
  DISPATCH_LOGN(L, decode_readout_impl, L, res, count, lv, ct, et, inv_scale, args, prods);
  return hipGetLastError();
}
hipError_t launch_readout_batch(const LaunchCtx& L, const double* z, const EncodeArgs* args, const BatchProd* prods,
                                int count, int max_rows, int slots) {
  hipLaunchKernelGGL(k_readout_batch, dim3((max_rows + 255) / 256, count), dim3(256), 0, L.stream, z, args, prods, slots);
  return hipGetLastError();
}

}  // namespace pvfl

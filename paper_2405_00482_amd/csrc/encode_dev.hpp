// Device helpers of the canonical-embedding encoder/decoder and the plan
// packing, shared by the single-plan and the batched kernels.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "encode.hpp"
#include "ntt_core.hpp"

#include <type_traits>

namespace pvfl {

__device__ __forceinline__ double2 cmul(double2 a, double2 b) {
  return make_double2(a.x * b.x - a.y * b.y, a.x * b.y + a.y * b.x);
}
__device__ __forceinline__ double2 cconj(double2 a) { return make_double2(a.x, -a.y); }

// padded index of complex element i in LDS (one pad slot every 16): breaks
// the bank conflicts of strided and bit-reversed access
__device__ __forceinline__ int cpad(int i) { return i + (i >> 4); }

__device__ __forceinline__ double round_half_away(double x) {
  const double r = __builtin_trunc(x + (x >= 0.0 ? 0.5 : -0.5));
  return r;
}

// S radix-2 DIF stages S0 .. S0+S-1 of the M = N/2 point FFT, on register
// sets of 2^S elements {base + u * stride} (stride = half-length of the last
// stage).  Each thread owns 8 elements (M = 8 T), i.e. 8 / 2^S sets; the sets
// partition the array, so a set is loaded, transformed and written back in
// place without a barrier in between.  At stage s a butterfly pairs elements
// half_s = M >> (s+1) apart with twiddle W_M^(j 2^s), j = index mod half_s,
// which for element u of a set is off + (u mod 2^(S-1-st)) * stride.
// A pass is wave-local when a wave's 64 threads own one contiguous run of
// 512 elements: one set of 8 per thread with a stride of at most 64.
template <int LOGN, int S, int S0>
constexpr bool fft_pass_wave_local() {
  return S == 3 && LOGN - 1 - S0 - S <= 6;
}

// Ends with a workgroup barrier, or only a wave-level LDS fence when this
// pass and the next one (NEXT_LOCAL) are both wave-local: the next pass then
// reads only what the same wave wrote.
template <int LOGN, int S, int S0, int TWSH, bool NEXT_LOCAL>
__device__ __forceinline__ void fft_pass(double2* a, const double2* __restrict__ tw, bool conj) {
  constexpr int LOGM = LOGN - 1, M = 1 << LOGM, T = NttShape<LOGN>::T;
  constexpr int SET = 1 << S, NS = 8 >> S;
  static_assert(M == 8 * T, "eight FFT points per thread");
  constexpr int LS = LOGM - S0 - S;  // log2 stride
  constexpr unsigned stride = 1u << LS;
  const unsigned tid = opaque_tid();
  if (tid < (unsigned)T) {  // a transform of M < 8 * blockDim points leaves the other threads idle
  int base[NS], off[NS];
  double2 x[8];
#pragma unroll
  for (int q = 0; q < NS; ++q) {
    const unsigned c = (unsigned)(q * T) + tid;
    off[q] = (int)(c & (stride - 1u));
    base[q] = (int)(((c >> LS) << (LS + S)) | (unsigned)off[q]);
#pragma unroll
    for (int u = 0; u < SET; ++u) x[q * SET + u] = a[cpad(base[q] + (u << LS))];
  }
#pragma unroll
  for (int st = 0; st < S; ++st) {
    const int s = S0 + st;
    const int hs = SET >> (st + 1);
#pragma unroll
    for (int q = 0; q < NS; ++q) {
#pragma unroll
      for (int u = 0; u < SET; ++u) {
        if (u & hs) continue;
        double2 w = tw[((off[q] + ((u & (hs - 1)) << LS)) << s) << TWSH];
        if (conj) w = cconj(w);
        const double2 U = x[q * SET + u], V = x[q * SET + u + hs];
        x[q * SET + u] = make_double2(U.x + V.x, U.y + V.y);
        x[q * SET + u + hs] = cmul(make_double2(U.x - V.x, U.y - V.y), w);
      }
    }
  }
#pragma unroll
  for (int q = 0; q < NS; ++q)
#pragma unroll
    for (int u = 0; u < SET; ++u) a[cpad(base[q] + (u << LS))] = x[q * SET + u];
  }
  if constexpr (fft_pass_wave_local<LOGN, S, S0>() && NEXT_LOCAL)
    wave_lds_sync();
  else
    __syncthreads();
}

// TWSH = 1 runs the 2^(LOGN-1)-point transform with the table of twice that
// size (every second entry), as the halves of the 2^15 ring's FFT do
template <int LOGN, int S0, int TWSH = 0>
__device__ __forceinline__ void fft_passes(double2* a, const double2* __restrict__ tw, bool conj) {
  constexpr int LEFT = LOGN - 1 - S0;
  if constexpr (LEFT >= 3) {
    constexpr int NLEFT = LEFT - 3;  // stages after this pass
    constexpr bool next_local = NLEFT >= 3 && fft_pass_wave_local<LOGN, 3, S0 + 3>();
    fft_pass<LOGN, 3, S0, TWSH, next_local>(a, tw, conj);
    fft_passes<LOGN, S0 + 3, TWSH>(a, tw, conj);
  } else if constexpr (LEFT > 0) {
    fft_pass<LOGN, LEFT, S0, TWSH, false>(a, tw, conj);
  }
}

// In-place DIF FFT over M = N/2 points in LDS (padded by cpad), sign -1
// (conj = false) or +1; the result is left in bit-reversed order.  The input
// must be complete in LDS (barrier before the call); the call ends with a
// barrier.  Radix-8 register passes: ceil(log2(M) / 3) LDS round trips.
template <int LOGN>
__device__ __forceinline__ void fft_dif_lds(double2* a, const double2* __restrict__ tw, bool conj) {
  static_assert(LOGN <= 14, "the 2^15 ring's FFT is split in halves (encode15, k_decode15)");
  fft_passes<LOGN, 0>(a, tw, conj);
}

// Half h of the 2^15 ring's M = 2^14 point DIF FFT, already past its first
// stage and placed in LDS: stages 1.. of the full transform restricted to
// the half are a 2^13-point DIF FFT with twiddle indices doubled.
__device__ __forceinline__ void fft_dif_half15(double2* a, const double2* __restrict__ tw, bool conj) {
  fft_passes<14, 0, 1>(a, tw, conj);
}

__device__ __forceinline__ int brev(int x, int bits) { return (int)(__brev((unsigned)x) >> (32 - bits)); }

// Centred CRT lift (Garner mixed radix) of coefficient kk from its residues
// base[i N + kk], i < nl.  NL > 0 fixes the limb count at compile time; NL = 0
// takes nl at run time, its loops unrolled to the largest count under uniform
// conditions: either way the mixed-radix digits have fixed places and stay in
// registers (indexed at run time they would go to scratch memory, which took
// 16 ciphertexts at N = 2^15 with 8 limbs 0.49 ms instead of 0.17 ms).
template <int NL>
struct CrtResidues {  // of one coefficient
  static constexpr int MAXL = NL > 0 ? NL : kMaxLimbs;
  double v[MAXL];
  __device__ __forceinline__ void load(const double* __restrict__ base, int kk, int N, int nl_rt) {
#pragma unroll
    for (int i = 0; i < MAXL; ++i) v[i] = i < (NL > 0 ? NL : nl_rt) ? gmem(base)[(size_t)i * N + kk] : 0.0;
  }
};
template <int NL>
__device__ __forceinline__ double crt_lift(CrtResidues<NL>& r, const CrtTabs& ct, int nl_rt) {
  constexpr int MAXL = CrtResidues<NL>::MAXL;
  const int nl = NL > 0 ? NL : nl_rt;
  double(&v)[MAXL] = r.v;
#pragma unroll
  for (int i = 0; i < MAXL; ++i) {
    if (i < nl) {
      const ModQ m = ct.mods[i];
      double x = v[i];
#pragma unroll
      for (int j = 0; j < i; ++j) x = mulmod(x - v[j], ct.garner_inv[j * kMaxLimbs + i], m);
      v[i] = canon(x, m);
    }
  }
  // sign: compare with the mixed-radix digits of (Q-1)/2 from the top
  int cmp = 0;
#pragma unroll
  for (int i = MAXL - 1; i >= 0; --i) {
    if (i < nl) {
      const double h2 = 0.5 * (ct.mods[i].q - 1.0);
      if (cmp == 0) cmp = (v[i] > h2) ? 1 : ((v[i] < h2) ? -1 : 0);
    }
  }
  double acc = 0.0;
#pragma unroll
  for (int i = MAXL - 1; i >= 0; --i) {
    if (i == nl - 1) acc = (cmp > 0) ? v[i] - ct.mods[i].q : v[i];
    if (i < nl - 1) acc = acc * ct.mods[i].q + v[i];
  }
  return acc;
}
template <int NL>
__device__ __forceinline__ double crt_lift(const double* __restrict__ base, int kk, int N, const CrtTabs& ct,
                                           int nl_rt) {
  CrtResidues<NL> r;
  r.load(base, kk, N, nl_rt);
  return crt_lift<NL>(r, ct, nl_rt);
}

// f(std::integral_constant<int, NL>) for the limb count nl: one to six and eight by
// number, 0 (loops unrolled to kMaxLimbs under uniform conditions) for the others.
// One / 512 ciphertexts, by number and through the general form, us: 3 limbs at 2^13
// 27 and 66 / 114 and 185, 8 limbs at 2^15 179 and 238 / 1335 and 1409.  Each number is
// one more copy of the loop, and the kernels' other copies pay for it: with seven of its
// own (2^15: 160 instead of 214 / 1193 instead of 1262) the three-limb read-out of one
// ciphertext at 2^13 takes 15.8 instead of 14.9.
template <class F>
__device__ __forceinline__ void with_limbs(int nl, F f) {
  switch (nl) {
    case 1: f(std::integral_constant<int, 1>()); break;
    case 2: f(std::integral_constant<int, 2>()); break;
    case 3: f(std::integral_constant<int, 3>()); break;
    case 4: f(std::integral_constant<int, 4>()); break;
    case 5: f(std::integral_constant<int, 5>()); break;
    case 6: f(std::integral_constant<int, 6>()); break;
    case 8: f(std::integral_constant<int, 8>()); break;
    default: f(std::integral_constant<int, 0>()); break;
  }
}

// Decode of one ciphertext's coefficient residues base[i N + k] (i < nl,
// canonical) up to the slot values, N <= 2^14: CRT lift, twist, DFT with sign
// +1; the spectrum is left in LDS (w, padded, bit-reversed order) for
// decoded_slot().  Ends with a barrier.
template <int LOGN>
__device__ __forceinline__ void decode_to_lds(const double* __restrict__ base, int nl, const CrtTabs& ct,
                                              const EncTabs& et, double2* w) {
  static_assert(LOGN <= 14, "the 2^15 ring's decode splits its FFT in halves");
  constexpr int N = 1 << LOGN, M = N / 2, T = NttShape<LOGN>::T;
  // twisted w_k = (m_k + i m_(k+N/2)) zeta^k
  with_limbs(nl, [&](auto nl_c) {
    constexpr int NL = decltype(nl_c)::value;
    // the residues of U of the thread's 8 points (at most 32 values) in flight
    // together: one ciphertext's decode with read-out at 2^12 11.0 -> 10.2 us,
    // at 2^13 15.8 -> 14.8.  At 2^14 at most 16 values: of 2 limbs, 512 ciphertexts take
    // 65 us with them and 77 with 32, one takes 20 either way
    constexpr int U = NL == 0 ? 1 : NL <= 2 && LOGN < 14 ? 8 : NL <= 4 ? 4 : 2;
#pragma unroll 1
    for (int k0 = opaque_tid(); k0 < M; k0 += U * T) {
      CrtResidues<NL> re[U], im[U];
#pragma unroll
      for (int u = 0; u < U; ++u) {
        re[u].load(base, k0 + u * T, N, nl);
        im[u].load(base, k0 + u * T + M, N, nl);
      }
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const int k = k0 + u * T;
        w[cpad(k)] = cmul(make_double2(crt_lift<NL>(re[u], ct, nl), crt_lift<NL>(im[u], ct, nl)), et.twist[k]);
      }
    }
  });
  __syncthreads();
  fft_dif_lds<LOGN>(w, et.fft_tw, true);
}

// The spectrum decode_to_lds left in LDS becomes the cleartext values of the
// slots in slot order, in the same LDS; ends with a barrier.  The read-out's
// sums then read consecutive places instead of looking every slot's place up
// (decode and read-out at N = 2^12, rows of 128 additions: 14 us with the look-up, 11 us without).
template <int LOGN>
__device__ __forceinline__ const double* slots_in_order(double2* w, const EncTabs& et, double inv_scale) {
  constexpr int M = (1 << LOGN) / 2, T = NttShape<LOGN>::T;
  const int tid = opaque_tid();
  double v[M / T];
#pragma unroll
  for (int u = 0; u < M / T; ++u) v[u] = w[cpad(brev(et.slot2f[tid + u * T], LOGN - 1))].x * inv_scale;
  __syncthreads();
  double* z = (double*)w;
#pragma unroll
  for (int u = 0; u < M / T; ++u) z[tid + u * T] = v[u];
  __syncthreads();
  return z;
}

// z(0) + z(1) + ... + z(cnt - 1) in this order, eight reads in flight at a time
template <class Z>
__device__ __forceinline__ double sum_in_order(int cnt, Z z) {
  double acc = 0.0;
  int t = 0;
  for (; t + 8 <= cnt; t += 8) {
    double v[8];
#pragma unroll
    for (int u = 0; u < 8; ++u) v[u] = z(t + u);
#pragma unroll
    for (int u = 0; u < 8; ++u) acc += v[u];
  }
  for (; t < cnt; ++t) acc += z(t);
  return acc;
}

// Element of X that slot s of plaintext k holds (a KIND plan), or -1 where the
// slot is zero (padding, outside the matrix).
template <int KIND>
__device__ __forceinline__ long pt_slot_index(const EncodeArgs& a, int k, int s) {
  if constexpr (KIND == 0) {  // HYBRID: block (b, c), diagonal i; slot s = g bn + j
    // bn, bm and m' are powers of two (zero padding, Sec. 3): shifts and masks
    const int per = a.col_blocks * a.mprime;
    const int b = k / per, c = (k >> a.lmp) % a.col_blocks, i = k & (a.mprime - 1);
    if (a.bsgs > 0) s = (s - (i & -a.bsgs) + a.slots) & (a.slots - 1);  // pre-rotation by the giant step
    const int g = s >> a.lbn, j = s & (a.bn - 1);
    const int rr = (g << a.lmp) + (j & (a.mprime - 1));
    const int row = b * a.bm + rr, col = c * a.bn + ((i + j) & (a.bn - 1));
    return (rr < a.bm && row < a.m && col < a.n) ? (long)row * a.ld + col : -1;
  } else if constexpr (KIND == 1) {  // DIAG: Eq. 5 over max(m,n) slots
    const int row = s & (a.bm - 1), col = (k + s) & (a.bn - 1);
    return (s < a.width && row < a.m && col < a.n) ? (long)row * a.ld + col : -1;
  } else if constexpr (KIND == 2) {  // ROW: row k in slots 0..n-1
    return (s < a.n && k < a.m) ? (long)k * a.ld + s : -1;
  } else if constexpr (KIND == 3) {  // CTMAT: W (n x n_out); plaintext k = i * n_out_cts + kc
    const int i = k / a.n_out_cts, kc = k % a.n_out_cts;
    const int blk = s >> a.lw, j = s & (a.width - 1);
    const int r = (i + j) & (a.bn - 1), col = kc * a.pack + blk;
    return (blk < a.pack && r < a.n && col < a.n_out) ? (long)r * a.ld + col : -1;
  } else {  // COL: plaintext k = j * row_blocks + b holds rows b bm .. of column j
    const int j = k / a.n_out_cts, b = k % a.n_out_cts;
    const int row = b * a.bm + s;
    return (s < a.bm && row < a.m && j < a.n) ? (long)row * a.ld + j : -1;
  }
}

// Element of the encrypted operand that slot t of input ciphertext c holds, or -1.
template <int KIND>
__device__ __forceinline__ long ct_slot_index(const EncodeArgs& a, int c, int t) {
  if constexpr (KIND == 0) {  // HYBRID: column block c of y, period bn
    const int col = c * a.bn + (t & (a.bn - 1));
    return col < a.n ? col : -1;
  } else if constexpr (KIND == 1 || KIND == 2) {  // DIAG / ROW: y with period n_pad
    const int col = t & (a.bn - 1);
    return col < a.n ? col : -1;
  } else if constexpr (KIND == 3) {  // CTMAT: diagonal c of A (m x n), replicated over pack blocks
    const int blk = t >> a.lw, j = t & (a.width - 1);
    const int row = j & (a.bm - 1), col = (c + j) & (a.bn - 1);
    return (blk < a.pack && row < a.m && col < a.n) ? (long)row * a.ld + col : -1;
  } else {  // COL: ciphertext c holds y_c in every slot
    return c < a.n ? (long)c : -1;
  }
}

// v[u] = scale * (value of slot slot_of(u)), u < CNT.  Every load is issued
// before any value is used (a zero slot loads X[0], which exists, and selects
// 0), so the gather pays one memory latency instead of one per slot.
template <bool CT, int KIND, int CNT, class SlotOf>
__device__ __forceinline__ void gather_kind(const EncodeArgs& a, int k, double scale, SlotOf slot_of,
                                            double (&v)[CNT]) {
  long id[CNT];
#pragma unroll
  for (int u = 0; u < CNT; ++u) id[u] = CT ? ct_slot_index<KIND>(a, k, slot_of(u)) : pt_slot_index<KIND>(a, k, slot_of(u));
  double x[CNT];
#pragma unroll
  for (int u = 0; u < CNT; ++u) x[u] = gmem(a.X)[id[u] < 0 ? 0 : id[u]];
#pragma unroll
  for (int u = 0; u < CNT; ++u) v[u] = id[u] < 0 ? 0.0 : x[u] * scale;
}

template <bool CT, int CNT, class SlotOf>
__device__ __forceinline__ void gather_slots(const EncodeArgs& a, int k, double scale, SlotOf slot_of,
                                             double (&v)[CNT]) {
  switch (a.kind) {
    case 0: gather_kind<CT, 0>(a, k, scale, slot_of, v); break;
    case 1: gather_kind<CT, 1>(a, k, scale, slot_of, v); break;
    case 2: gather_kind<CT, 2>(a, k, scale, slot_of, v); break;
    case 3: gather_kind<CT, 3>(a, k, scale, slot_of, v); break;
    default: gather_kind<CT, 4>(a, k, scale, slot_of, v); break;
  }
}

// The slot values v[u] of slots j = tid + u T (u < 8, N <= 2^14) -> FFT ->
// rounded coefficients in registers, as encode_to_regs_v describes.  Slot j
// is DFT input f = (5^j mod 2N - 1) / 4, i.e. component f mod 2 of y[f / 2].
// Begins by writing LDS (barrier before the call if LDS is in use); ends
// with a barrier.
template <int LOGN>
__device__ __forceinline__ void fft_split_regs(const double (&v)[8], double2* z, double* mreg, const EncTabs& et) {
  static_assert(LOGN <= 14, "the 2^15 ring's encoder splits its FFT in halves");
  constexpr int N = 1 << LOGN, M = N / 2, T = NttShape<LOGN>::T, HM = M / 2, QH = HM / T;
  const int tid = opaque_tid();
  const double inv_m = 1.0 / (double)M;
  {
    OrbitWalk ow = OrbitWalk::start<LOGN>();
    double* zd = (double*)z;
#pragma unroll
    for (int u = 0; u < 2 * QH; ++u) {
      const int f = (int)(ow.e >> 2);
      zd[2 * cpad(f >> 1) + (f & 1)] = v[u];
      ow.next<LOGN>();
    }
  }
  __syncthreads();
  fft_passes<LOGN - 1, 0, 1>(z, et.fft_tw, false);
#pragma unroll
  for (int u = 0; u < QH; ++u) {
    const int k = tid + u * T;
    const double2 Yk = z[cpad(brev(k, LOGN - 2))];
    const double2 Yc = z[cpad(brev((HM - k) & (HM - 1), LOGN - 2))];
    const double2 E = make_double2(0.5 * (Yk.x + Yc.x), 0.5 * (Yk.y - Yc.y));
    const double2 O = make_double2(0.5 * (Yk.y + Yc.y), -0.5 * (Yk.x - Yc.x));
    const double2 wo = cmul(O, et.fft_tw[k]);
    const double2 w0 = cmul(make_double2(E.x + wo.x, E.y + wo.y), cconj(et.twist[k]));
    const double2 w1 = cmul(make_double2(E.x - wo.x, E.y - wo.y), cconj(et.twist[k + HM]));
    mreg[2 * u] = round_half_away(w0.x * inv_m);
    mreg[2 * u + 1] = round_half_away(w0.y * inv_m);
    mreg[2 * (u + QH)] = round_half_away(w1.x * inv_m);
    mreg[2 * (u + QH) + 1] = round_half_away(w1.y * inv_m);
  }
  __syncthreads();
}

// slots -> FFT -> rounded coefficients in registers, N <= 2^14: mreg[2u] = m_k
// and mreg[2u+1] = m_(k+N/2) for k = tid + u T, u < M/T.  gather(slot_of, v)
// fills v[u] with the scaled value of slot slot_of(u) for every u of v.
template <int LOGN, class Gather>
__device__ __forceinline__ void encode_to_regs_v(Gather gather, double2* z, double* mreg, const EncTabs& et) {
  constexpr int N = 1 << LOGN, M = N / 2, T = NttShape<LOGN>::T;
  const int tid = opaque_tid();
  // The DFT input x[f] (slot value at f = f_j) is real: pack y[n] = x[2n] +
  // i x[2n+1], transform M/2 points, and split (real-input FFT):
  //   E[k] = (Y[k] + conj Y[M/2-k]) / 2,  O[k] = (Y[k] - conj Y[M/2-k]) / 2i,
  //   X[k] = E[k] + W^k O[k],  X[k + M/2] = E[k] - W^k O[k],  W = exp(-2 pi i / M).
  // The half transform runs on the first half of the threads with every
  // other twiddle of the M-point table.
  constexpr int HM = M / 2, QH = HM / T;  // QH = 4 complex inputs per thread
  double v[2 * QH];
  gather([&](int u) { return tid + u * T; }, v);
  fft_split_regs<LOGN>(v, z, mreg, et);
}

// The same at N = 2^15, coefficient tid + w T handed to put(w, m) as it is
// made.  The first DIF stage (pairs i, i + M/2, owned by one thread) runs in
// registers and the two halves in LDS one after the other; half h yields the
// coefficients with k = h mod 2.  A thread's 32 coefficients do not stay in
// registers: beside the transform's own values they would spill.  All of a thread's slots are gathered at once.
template <class Gather, class Put>
__device__ __forceinline__ void encode15(Gather gather, double2* z, const EncTabs& et, Put put) {
  constexpr int LOGN = 15, N = 1 << LOGN, M = N / 2, T = NttShape<LOGN>::T, HM = M / 2, PH = M / T, U = HM / T;
  const int tid = opaque_tid();
  const double inv_m = 1.0 / (double)M;
  double2 v0[U];
  {
    int slot[2 * U];
#pragma unroll
    for (int q = 0; q < 2 * U; ++q) slot[q] = (int)et.f2slot[tid + (q >> 1) * T + (q & 1) * HM];
    double ab[2 * U];
    gather([&](int q) { return slot[q]; }, ab);
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int i = tid + u * T;
      const double a0 = ab[2 * u], b0 = ab[2 * u + 1];
      z[cpad(i)] = make_double2(a0 + b0, 0.0);
      v0[u] = cmul(make_double2(a0 - b0, 0.0), et.fft_tw[i]);
    }
  }
#pragma unroll 1
  for (int h = 0; h < 2; ++h) {
    if (h) {
      __syncthreads();  // half 0's read-out is done
#pragma unroll
      for (int u = 0; u < U; ++u) z[cpad(tid + u * T)] = v0[u];
    }
    __syncthreads();
    fft_dif_half15(z, et.fft_tw, false);
    if ((tid & 1) == h) {  // k = tid + u T has the parity of tid
#pragma unroll 4
      for (int u = 0; u < PH; ++u) {
        const int kk = tid + u * T;
        const double2 w = cmul(z[cpad(brev(kk, LOGN - 1) - h * HM)], cconj(et.twist[kk]));
        put(u, round_half_away(w.x * inv_m));
        put(u + PH, round_half_away(w.y * inv_m));
      }
    }
  }
  __syncthreads();
}

template <int LOGN, bool CT>
__device__ __forceinline__ void encode_to_regs(const EncodeArgs& a, int k, double2* z, double* mreg, const EncTabs& et,
                                               double scale) {
  encode_to_regs_v<LOGN>([&](auto slot_of, auto& v) { gather_slots<CT>(a, k, scale, slot_of, v); }, z, mreg, et);
}

// Message of input ciphertext c as int64 coefficients.
template <int LOGN>
__device__ __forceinline__ void encode_ct_body(const EncodeArgs& a, int c, const EncTabs& et, double2* s2,
                                               int64_t* __restrict__ dst) {
  constexpr int N = 1 << LOGN, T = NttShape<LOGN>::T, PH = N / 2 / T;
  if constexpr (LOGN <= 14) {
    double mreg[2 * PH];
    encode_to_regs<LOGN, true>(a, c, s2, mreg, et, a.scale);
#pragma unroll
    for (int u = 0; u < PH; ++u) {
      const int kk = threadIdx.x + u * T;
      dst[kk] = (int64_t)mreg[2 * u];
      dst[kk + N / 2] = (int64_t)mreg[2 * u + 1];
    }
  } else {
    encode15([&](auto slot_of, auto& v) { gather_slots<true>(a, c, a.scale, slot_of, v); }, s2, et,
             [&](int w, double m) { dst[threadIdx.x + w * T] = (int64_t)m; });
  }
}

// Part of a plaintext's limbs [l0, l1) that one workgroup makes.
struct LimbRange {
  int l0, l1;
};
// part `p` of `parts` of n limbs
__device__ __forceinline__ LimbRange limb_part(int n, int p, int parts) {
  const int per = (n + parts - 1) / parts;
  return LimbRange{min(n, p * per), min(n, (p + 1) * per)};
}

// Encodes the slots that gather() yields and transforms the limbs `lr` of
// `map`, to out[limb][N]; first(c, l) turns the integer coefficients into limb l's
// input (|x| < 2^51).  s2: LDS of NttShape<LOGN>::LDS doubles.
template <int LOGN, class Gather, class First, class Store>
__device__ __forceinline__ void encode_limbs(Gather gather, const EncTabs& et, const LimbMap& map, LimbRange lr,
                                             const DevTabs& tb, double2* s2, double* __restrict__ out, First first,
                                             Store store) {
  constexpr int N = 1 << LOGN, T = NttShape<LOGN>::T, PH = N / 2 / T, PER = NttShape<LOGN>::PER;
  double* s = (double*)s2;
  if constexpr (LOGN <= 14) {
    double mreg[2 * PH];
    encode_to_regs_v<LOGN>(gather, s2, mreg, et);
    const OrbitIndex<LOGN> oi = OrbitIndex<LOGN>::make();
    // coefficient tid + w T: w < PH -> m_k (real part), w >= PH -> m_(k+N/2) (imaginary part)
    for (int l = lr.l0; l < lr.l1; ++l) {
      const int pi = map.idx[l];
      double c[PER];
#pragma unroll
      for (int w = 0; w < PER; ++w) c[w] = first(w < PH ? mreg[2 * w] : mreg[2 * (w - PH) + 1], l);
      double* dst = out + (size_t)l * N;
      ntt_fwd_regs_out<LOGN>(s, c, tb.fwd_tw + (size_t)pi * N, tb.mods[pi],
                             [&](unsigned b, unsigned t, double v) { store(scalar_base(dst + b) + t, v); }, oi.opaque());
    }
  } else {
    // the integer coefficients wait in the last limb's place, where each thread
    // reads back only what it wrote; that limb is transformed last, and its
    // first barrier stands between the reads and the output's writes
    double* park = out + (size_t)(lr.l1 - 1) * N;
    encode15(gather, s2, et, [&](int w, double m) { park[opaque_tid() + w * T] = m; });
    for (int l = lr.l0; l < lr.l1; ++l) {
      const int pi = map.idx[l];
      double c[PER];
#pragma unroll
      for (int w = 0; w < PER; ++w) c[w] = first(park[opaque_tid() + w * T], l);
      double* dst = out + (size_t)l * N;
      ntt_fwd_regs_out<LOGN>(s, c, tb.fwd_tw + (size_t)pi * N, tb.mods[pi],
                             [&](int t, double v) { store(dst + t, v); });
    }
  }
}

// Plaintext k of a plan: pack, encode, then the limbs `lr` of `map` reduced and
// transformed; written to out_pt[limb][N].  |m| < 2^51, which the transform
// reduces on entry.
template <int LOGN>
__device__ __forceinline__ void encode_pt_body(const EncodeArgs& a, int k, const EncTabs& et, const LimbMap& map,
                                               LimbRange lr, const DevTabs& tb, double2* s2, double* __restrict__ out_pt) {
  auto same = [](double m, int) { return m; };
  // the plaintext buffer is device memory: global stores (unlike flat stores
  // they do not count against the LDS wait counter of the gather before
  // them), nontemporal because nothing in this kernel reads them again --
  // they would only push the twiddle tables and X out of L2
  auto stream = [](auto* p, double v) {
    __builtin_nontemporal_store(v, (__attribute__((address_space(1))) double*)p);
  };
  if (a.kind == 2 && k == a.m) {
    // ROW indicator plaintext: 1 in slot 0 at scale q_(l-1)
    const double ind = a.ind_scale;
    encode_limbs<LOGN>(
        [&](auto slot_of, auto& v) {
#pragma unroll
          for (int u = 0; u < (int)(sizeof(v) / sizeof(v[0])); ++u) v[u] = slot_of(u) == 0 ? ind : 0.0;
        },
        et, map, lr, tb, s2, out_pt, same, stream);
  } else {
    encode_limbs<LOGN>([&](auto slot_of, auto& v) { gather_slots<false>(a, k, a.scale, slot_of, v); }, et, map, lr,
                       tb, s2, out_pt, same, stream);
  }
}

// Value of slot s of output ciphertext b for a cleartext added to the plan's
// result (mode 0: the m outputs spread by the cleartext inverse RaS of Sec.
// 5.2, each split into equal parts over the slots its row's lazy RaS adds;
// mode 1: slot values [ct_out][N/2] as given).  The parts are powers-of-two
// fractions of v, so the split is exact.
__device__ __forceinline__ double out_slot_value(const EncodeArgs& a, const double* __restrict__ v, int mode,
                                                 int ras_in_ct, int b, int s) {
  if (mode == 1) return v[(size_t)b * a.slots + s];
  switch (a.kind) {
    case 0: {  // HYBRID: slot g bn + j adds into row g m' + (j mod m') of block b
      const int g = s >> a.lbn, j = s & (a.bn - 1);
      const int row = b * a.bm + (g << a.lmp) + (j & (a.mprime - 1));
      return row < a.m ? ldexp(v[row], a.lmp - a.lbn) : 0.0;
    }
    case 1: {  // DIAG over max(m,n) slots
      if (a.bm >= a.bn || ras_in_ct) return s < a.m ? v[s] : 0.0;
      const int r = s & (a.bm - 1);
      return (s < a.bn && r < a.m) ? ldexp(v[r], __builtin_ctz(a.bm) - a.lbn) : 0.0;
    }
    case 4: {  // COL: slot s of output ciphertext b is row b bm + s
      const int row = b * a.bm + s;
      return (s < a.bm && row < a.m) ? v[row] : 0.0;
    }
    case 3: {  // CTMAT: output ciphertext b, column block blk = s / width
      const int blk = s >> a.lw, j = s & (a.width - 1), col = b * a.pack + blk;
      if (blk >= a.pack || col >= a.n_out) return 0.0;
      if (a.bm >= a.bn) return j < a.m ? v[(size_t)j * a.n_out + col] : 0.0;
      const int r = j & (a.bm - 1);
      return (j < a.bn && r < a.m) ? ldexp(v[(size_t)r * a.n_out + col], __builtin_ctz(a.bm) - a.lbn) : 0.0;
    }
  }
  return 0.0;
}

// Output ciphertext b's cleartext at scale a.scale, rounded, then every limb's
// residues times fac[l] (2^e mod q) and transformed, to out[limb][N].
template <int LOGN>
__device__ __forceinline__ void encode_out_body(const EncodeArgs& a, const double* __restrict__ v, int mode,
                                                int ras_in_ct, int b, const OutFactors& fac, const EncTabs& et,
                                                const LimbMap& map, LimbRange lr, const DevTabs& tb, double2* s2,
                                                double* __restrict__ out) {
  encode_limbs<LOGN>(
      [&](auto slot_of, auto& val) {
#pragma unroll
        for (int u = 0; u < (int)(sizeof(val) / sizeof(val[0])); ++u)
          val[u] = out_slot_value(a, v, mode, ras_in_ct, b, slot_of(u)) * a.scale;
      },
      et, map, lr, tb, s2, out, [&](double m, int l) { return mulmod(m, fac.f[l], tb.mods[map.idx[l]]); },
      [](auto* p, double x) { *p = x; });
}

}  // namespace pvfl

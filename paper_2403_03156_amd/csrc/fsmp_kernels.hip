// fsmp_kernels.hip -- gfx950 kernels of libfsmp.so.
//
//  * prologue_kernel: per waveform, the matched filter c(g) = sum_n w[n] V(n - g/sub)
//    over the solution space T (FP64 accumulation) and a scan for non-finite samples.
//  * the Gibbs / RJMCMC chains (Sec. 2.4): chain_lds_kernel (one element of a chain's vectors
//    per lane, H in LDS: the lowest latency of a sweep) where the chains fit the LDS of the
//    chip, chain_kernel (LPC lanes per chain, H in device memory) and chain_lane_kernel (one
//    lane) for more of them.  Per chain they hold the inverse PE-space Gram matrix H = G^{-1},
//    G = A^T A + rho I (symmetric, KCAP x KCAP), the matched-filter terms b, the charge means
//    x = H b and the PE grid indices.  With H at hand
//      birth  : eta = H gamma (one mat-vec), delta^2 = d - gamma^T eta,
//               u+ = (beta - gamma^T x) / delta,
//               delta-nu = -1/2 [-log rho + log delta^2 + (rho m^2 - u+^2) / s];
//      death  : omega = H_jj, delta-nu = 1/2 [-log rho - log omega + (rho m^2 - x_j^2/omega) / s];
//      update : one mat-vec with gamma' (zero at j) and O(1) corrections;
//    accepted moves are rank-one (birth, death) or rank-two (update) edits of H.
//    These are the determinant lemma and Woodbury identity applied in PE space to the
//    normal law of App. A (eq. mgauss); they give the same delta-nu as the paper's
//    N_w x N_w rank-2 form (eqs. 11-18) at O(K^2) instead of O(N_w^2) per step.
//  * posterior_kernel: per waveform, pooled mean / variance / batch-means MCSE.
//
// Random numbers: Philox4x32-10 (Salmon, Moraes, Dror, Shaw, SC'11), key = seed,
// counter = (step, block, uid lo, uid hi).  Words of one step: r0,r1 Box-Muller pair
// (t0 step, update shift), r2 t0 accept, r3 move, r4 (r5) index or 53-bit birth
// uniform, r6 jump accept, r7 the mixture component of a born or updated PE (MCP-PMT law).
// Where a chain owns a whole wavefront (and in the FP64 form's 32-lane groups), its lanes
// make these values LPC sweeps at a time, lane l of its group those of sweep LPC m + l, and
// each sweep reads its own by lane reads.

#include <math.h>

#include <algorithm>
#include <type_traits>

#include "fsmp_internal.h"

namespace fsmp {
namespace {

constexpr int kWave = 64;
// FP32 form: the largest error bound, relative to max(1, |delta-nu|), with which a
// proposal is decided from the corrected FP32 evaluation (above it: the FP64 rebuild)
constexpr double kF32Tol = 1e-5;

// Intra-wavefront ordering of LDS traffic between lanes: the LDS executes one
// wavefront's instructions in order; the fences keep the compiler from moving
// memory operations across this point.
#define WAVE_SYNC()                                        \
  do {                                                     \
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront"); \
    __builtin_amdgcn_wave_barrier();                       \
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront"); \
  } while (0)

__device__ inline void philox4x32_10(uint32_t c0, uint32_t c1, uint32_t c2, uint32_t c3, uint32_t k0, uint32_t k1,
                                     uint32_t *out) {
#pragma unroll
  for (int r = 0; r < 10; ++r) {
    // each 32 x 32 -> 64-bit product is one v_mad_u64_u32 (high and low halves together)
    const uint64_t p0 = (uint64_t)0xD2511F53u * c0, p1 = (uint64_t)0xCD9E8D57u * c2;
    const uint32_t n0 = (uint32_t)(p1 >> 32) ^ c1 ^ k0, n2 = (uint32_t)(p0 >> 32) ^ c3 ^ k1;
    c0 = n0;
    c1 = (uint32_t)p1;
    c2 = n2;
    c3 = (uint32_t)p0;
    k0 += 0x9E3779B9u;
    k1 += 0xBB67AE85u;
  }
  out[0] = c0;
  out[1] = c1;
  out[2] = c2;
  out[3] = c3;
}

__device__ inline double u01(uint32_t r) { return ((double)r + 0.5) * 0x1p-32; }

__device__ inline double u53(uint32_t lo, uint32_t hi) {
  const uint64_t v = ((uint64_t)hi << 32) | lo;
  return (double)(v >> 11) * 0x1p-53 + 0x1p-54;
}

// Standard normal k of the charge draw at `step`: Philox block 2 + k/2, Box-Muller of
// words 0 and 1, the cosine branch for even k and the sine branch for odd k.
__device__ inline double charge_normal(int step, int k, uint32_t uid0, uint32_t uid1, uint32_t key0, uint32_t key1) {
  uint32_t r[4];
  philox4x32_10((uint32_t)step, 2u + (uint32_t)(k >> 1), uid0, uid1, key0, key1, r);
  const double R = sqrt(-2.0 * log(u01(r[0])));
  const double th = 2.0 * M_PI * u01(r[1]);
  return (k & 1) ? R * sin(th) : R * cos(th);
}

// log phi(x); -inf where phi vanishes (x < 0, and x = 0 for BIEXP)
__device__ inline double log_phi(const ModelDev &md, double x) {
  if (md.kind == FSMP_PHI_EXP) return x < 0.0 ? -INFINITY : -x * md.inv_tau2 - md.log_tau2;
  if (!(x > 0.0)) return -INFINITY;
  return md.logC - x * md.inv_tau2 + log(-expm1(-x * md.inv_tau1));
}

// v from the lane the DPP control CTRL selects, for a double (its two halves moved alike)
template <int CTRL>
__device__ inline double dpp_move(double v) {
  const int lo = __builtin_amdgcn_update_dpp(0, __double2loint(v), CTRL, 0xF, 0xF, false);
  const int hi = __builtin_amdgcn_update_dpp(0, __double2hiint(v), CTRL, 0xF, 0xF, false);
  return __hiloint2double(hi, lo);
}

// log2, 2^x and 1 / x in FP32 to an ulp by the hardware's own instructions (first guesses only;
// the library's functions where the source is compiled for the host)
#if defined(__AMDGCN__)
__device__ inline float fast_log2(float x) { return __builtin_amdgcn_logf(x); }
__device__ inline float fast_exp2(float x) { return __builtin_amdgcn_exp2f(x); }
__device__ inline float fast_rcp(float x) { return __builtin_amdgcn_rcpf(x); }
#else
inline float fast_log2(float x) { return log2f(x); }
inline float fast_exp2(float x) { return exp2f(x); }
inline float fast_rcp(float x) { return 1.0f / x; }
#endif

// v of lane L of the wavefront, in scalar registers
__device__ inline double lane_value(double v, int L) {
  const int lo = __builtin_amdgcn_readlane(__double2loint(v), L);
  const int hi = __builtin_amdgcn_readlane(__double2hiint(v), L);
  return __hiloint2double(hi, lo);
}

// v of lane L of the caller's group of W lanes (group index grp; W >= 16, so at most four
// groups): one lane read per group, the caller's own picked by a select
template <int W>
__device__ inline uint32_t group_lane_u32(uint32_t v, int L, int grp) {
  uint32_t out = (uint32_t)__builtin_amdgcn_readlane((int)v, L);
#pragma unroll
  for (int g = 1; g < kWave / W; ++g) {
    const uint32_t x = (uint32_t)__builtin_amdgcn_readlane((int)v, g * W + L);
    out = grp == g ? x : out;
  }
  return out;
}
template <int W>
__device__ inline double group_lane(double v, int L, int grp) {
  const uint32_t lo = group_lane_u32<W>((uint32_t)__double2loint(v), L, grp);
  const uint32_t hi = group_lane_u32<W>((uint32_t)__double2hiint(v), L, grp);
  return __hiloint2double((int)hi, (int)lo);
}

// The value of lane K of the caller's group of W lanes (groups aligned to W, every lane of
// the group active): a DPP broadcast inside a quad (W = 4: quad_perm [K, K, K, K]) or a row
// (W = 16: row_newbcast:K), a lane read into scalar registers for a whole wavefront, else a
// lane permute from lane base + K
template <int W, int K>
__device__ inline double group_bcast(double v, int base) {
  if constexpr (W == 4) return dpp_move<K * 0x55>(v);
  else if constexpr (W == 16) return dpp_move<0x150 + K>(v);
  else if constexpr (W == kWave) return lane_value(v, K);
  else return __shfl(v, base + K, kWave);
}
template <int W, int K>
__device__ inline uint32_t group_bcast(uint32_t v, int base) {
  if constexpr (W == 4) return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, K * 0x55, 0xF, 0xF, false);
  else if constexpr (W == 16) return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x150 + K, 0xF, 0xF, false);
  else if constexpr (W == kWave) return (uint32_t)__builtin_amdgcn_readlane((int)v, K);
  else return (uint32_t)__shfl((int)v, base + K, kWave);
}

// The partial sums of phi over the grid points at or after t0 are geometric series:
// with xs = (first point) dt - t0, the sum over the first k points is
//   EXP:   e^{-xs/tau2} (1 - e^{-k dt/tau2}) / (1 - e^{-dt/tau2}) / tau2,
//   BIEXP: C [e^{-xs/tau2} (1 - e^{-k dt/tau2}) / (1 - e^{-dt/tau2})
//             - e^{-xs/tau12} (1 - e^{-k dt/tau12}) / (1 - e^{-dt/tau12})].
// The t0-dependent factors are computed once per use (XsExp); the count-dependent ones,
// (1 - e^{-k dt/tau}) / (1 - e^{-dt/tau}), come from the table md.ptab ([k][2], k up to the
// longest T, divided on the host), which turns each evaluation of a search into two loads
// and two multiplies.
struct XsExp {
  double e2, e12;
};

__device__ inline XsExp xs_exp(const ModelDev &md, double xs) {
  XsExp x;
  x.e2 = exp(-xs * md.inv_tau2);
  x.e12 = md.kind == FSMP_PHI_EXP ? 0.0 : exp(-xs * md.inv_tau12);
  return x;
}

__device__ inline double phi_partial(const ModelDev &md, const XsExp &x, int64_t k) {
  const double a = x.e2 * md.ptab[2 * k];
  if (md.kind == FSMP_PHI_EXP) return a * md.inv_tau2;
  return md.C * fma(-x.e12, md.ptab[2 * k + 1], a);
}

struct GridPos {
  int64_t gs;  // first grid point of T with g dt >= t0
  int64_t n;   // points of T from gs on (<= 0: none)
  double xs;   // gs dt - t0
};

__device__ inline GridPos grid_pos(const ModelDev &md, double t0, int glo, int ghi) {
  GridPos p;
  int64_t gs = (int64_t)ceil(t0 / md.dt);
  if (gs < glo) gs = glo;
  p.gs = gs;
  p.n = (int64_t)ghi - gs + 1;
  p.xs = (double)gs * md.dt - t0;
  return p;
}

__device__ inline double phi_total(const ModelDev &md, double t0, int glo, int ghi) {
  const GridPos p = grid_pos(md, t0, glo, ghi);
  return p.n > 0 ? phi_partial(md, xs_exp(md, p.xs), p.n) : 0.0;
}

// (1 - e^{-y}) / y for 0 <= y <= 1/4 by its Taylor series (thirteen terms: the rest is below
// 2^-56 of the value), all terms in one chain of multiply-adds
__device__ inline double one_minus_exp_series(double y) {
  const double x = -y;
  double p = 1.0 / 6227020800.0;
  p = fma(p, x, 1.0 / 479001600.0);
  p = fma(p, x, 1.0 / 39916800.0);
  p = fma(p, x, 1.0 / 3628800.0);
  p = fma(p, x, 1.0 / 362880.0);
  p = fma(p, x, 1.0 / 40320.0);
  p = fma(p, x, 1.0 / 5040.0);
  p = fma(p, x, 1.0 / 720.0);
  p = fma(p, x, 1.0 / 120.0);
  p = fma(p, x, 1.0 / 24.0);
  p = fma(p, x, 1.0 / 6.0);
  p = fma(p, x, 0.5);
  return fma(p, x, 1.0);
}

// What a light-curve start t0 contributes to a sweep, the same in all lanes of a chain's group:
// the factors of the partial sums from the first grid point of T at or after t0 (xs_exp), its
// index gs, the number n of points from there on, the sum over them, and for the rise factors
// of the PEs (rise_at) the first grid point g0 at or after t0 (not clipped to T) with
// q1 = 1 - e^{-(g0 dt - t0) / tau_rise}.
struct T0Terms {
  double e2, e12, q1, Phi;
  double p2, p12;  // the count-dependent factors at n (md.ptab), loaded before Phi is formed
  int g0, gs, n;
};

// Phi of a t0's terms: apart from them, so that the loads of its two factors overlap with the
// work in between
__device__ inline void t0_phi(const ModelDev &md, T0Terms &t) {
  const double a = t.e2 * t.p2;
  const double v = md.kind == FSMP_PHI_EXP ? a * md.inv_tau2 : md.C * (a - t.e12 * t.p12);
  t.Phi = t.n > 0 ? v : 0.0;
}

// T0Terms for a chain's lane group (t0, glo <= ghi the same in all its lanes, every lane
// active).  The distance g0 dt - t0 is below one grid step, so with dt / tau <= 1/4 all three
// exponentials are one short series (lane 0 tau2, lane 1 tau12, the others tau_rise): 13
// multiply-adds where the library's exp and expm1 take about 70 instructions.  Other light
// curves, and a T that starts after t0 (the two sums then start at its first point), take the
// library functions.
template <int W>
__device__ inline T0Terms t0_terms(const ModelDev &md, double t0, int glo, int ghi, int lane, int base) {
  T0Terms t;
  const double gd = ceil(md.sub_shift >= 0 ? t0 * md.sub : t0 / md.dt);
  t.g0 = (int)fmin(fmax(gd, -1073741824.0), 1073741824.0);
  t.gs = t.g0 < glo ? glo : t.g0;
  t.n = ghi - t.gs + 1;
  const double *pt = md.ptab + 2 * (t.n > 0 ? t.n : 0);
  t.p2 = pt[0];
  t.p12 = pt[1];
  const double f = (double)t.g0 * md.dt - t0;
  const double y = f * (lane == 0 ? md.inv_tau2 : lane == 1 ? md.inv_tau12 : md.inv_tau1);
  double v, e;
  if (md.small_dt && f <= md.dt) {
    const double p = one_minus_exp_series(y);
    v = y * p;
    e = fma(-y, p, 1.0);
  } else {
    v = -expm1(-y);
    e = exp(-y);
  }
  if (t.g0 < glo) e = exp(-((double)glo * md.dt - t0) * (lane == 0 ? md.inv_tau2 : md.inv_tau12));
  t.e2 = group_bcast<W, 0>(e, base);
  t.e12 = md.kind == FSMP_PHI_EXP ? 0.0 : group_bcast<W, 1>(e, base);
  t.q1 = group_bcast<W, 2>(v, base);
  return t;
}

// Sum over a group of W lanes (W a power of two, groups aligned to W): a butterfly over lane
// offsets W/2, ..., 2, 1, each lane adding the value of lane (its index xor the offset), so
// every lane ends with the same sum.  Offsets of 16 and more go through lane permutes; the
// rest are DPP moves inside a row of 16: xor 8 is a rotation of the row by 8, xor 4 after it
// a rotation by 4 (the values then depend only on the lane index mod 8, where a rotation by
// 4 and xor 4 agree), xor 2 and xor 1 quad permutations.  The pairs, and so the sums, are
// the same as with lane permutes for every offset.  A whole wavefront (W = 64) sums its four
// rows of 16 so and adds the row sums, read from lanes 0, 16, 32 and 48 into scalar
// registers, in that order (no lane permutes, and the result is a scalar).
template <int W>
__device__ inline double group_sum(double v) {
  if constexpr (W == kWave) {
    // a whole wavefront: the rows of 16 lanes by DPP, then their four sums from lanes 0, 16,
    // 32 and 48 into scalar registers, added in that order
    v += dpp_move<0x128>(v);  // row_ror:8
    v += dpp_move<0x124>(v);  // row_ror:4
    v += dpp_move<0x4E>(v);   // quad_perm [2, 3, 0, 1]: xor 2
    v += dpp_move<0xB1>(v);   // quad_perm [1, 0, 3, 2]: xor 1
    return ((lane_value(v, 0) + lane_value(v, 16)) + lane_value(v, 32)) + lane_value(v, 48);
  }
#pragma unroll
  for (int o = W / 2; o >= 16; o >>= 1) v += __shfl_xor(v, o, W);
  if constexpr (W >= 16) {
    v += dpp_move<0x128>(v);  // row_ror:8
    v += dpp_move<0x124>(v);  // row_ror:4
  } else if constexpr (W == 8) {
    v += __shfl_xor(v, 4, W);
  }
  if constexpr (W >= 4) v += dpp_move<0x4E>(v);  // quad_perm [2, 3, 0, 1]: xor 2
  if constexpr (W >= 2) v += dpp_move<0xB1>(v);  // quad_perm [1, 0, 3, 2]: xor 1
  return v;
}

// v times the v of the lane whose index differs by S (16 or 32): gfx950's swaps of rows and of the
// halves of a wavefront, with the same register on both sides, leave both factors in every lane
template <int S>
__device__ inline double lane_xor_product(double v) {
#if defined(__AMDGCN__)
  const unsigned lo = (unsigned)__double2loint(v), hi = (unsigned)__double2hiint(v);
  if constexpr (S == 32) {
    const auto l = __builtin_amdgcn_permlane32_swap(lo, lo, false, false);
    const auto h = __builtin_amdgcn_permlane32_swap(hi, hi, false, false);
    return __hiloint2double((int)h[0], (int)l[0]) * __hiloint2double((int)h[1], (int)l[1]);
  } else {
    const auto l = __builtin_amdgcn_permlane16_swap(lo, lo, false, false);
    const auto h = __builtin_amdgcn_permlane16_swap(hi, hi, false, false);
    return __hiloint2double((int)h[0], (int)l[0]) * __hiloint2double((int)h[1], (int)l[1]);
  }
#else
  return v * __shfl_xor(v, S, kWave);
#endif
}

// The product of v over the lanes of a group of W whose index is the same mod RO, by halves: lane
// offsets W/2, ..., RO (below 16 as in group_sum: a rotation by 4 after one by 8 pairs as xor 4)
template <int W, int RO>
__device__ inline double class_product(double v) {
  static_assert(RO == 4 || RO >= 16, "offsets below 16 come in a pair");
  if constexpr (W >= 64 && RO < 64) v = lane_xor_product<32>(v);
  if constexpr (W >= 32 && RO < 32) v = lane_xor_product<16>(v);
  if constexpr (RO == 4) {
    v *= dpp_move<0x128>(v);  // row_ror:8
    v *= dpp_move<0x124>(v);  // row_ror:4
  }
  return v;
}

// x / b from inv = 1 / b: the quotient's own rounding but for rare ties
__device__ inline double ratio(double x, double b, double inv) {
  const double q = x * inv;
  return fma(fma(-q, b, x), inv, q);
}

template <int W>
__device__ inline int group_or(int v) {
#pragma unroll
  for (int o = W / 2; o > 0; o >>= 1) v |= __shfl_xor(v, o, W);
  return v;
}

template <int W>
__device__ inline int group_min(int v) {
#pragma unroll
  for (int o = W / 2; o > 0; o >>= 1) {
    const int u = __shfl_xor(v, o, W);
    v = u < v ? u : v;
  }
  return v;
}

// The logs of two values that are the same in every lane of a chain's group, in one
// evaluation: the group's first lane takes x0, its second x1, and both results go to the
// whole group (base = the group's first lane; every lane of the group must be active)
template <int W>
__device__ inline void group_log2(double x0, double x1, int lane, int base, double &l0, double &l1) {
  const double v = log(lane == 0 ? x0 : x1);
  l0 = group_bcast<W, 0>(v, base);
  l1 = group_bcast<W, 1>(v, base);
}

// the same for three values (the group's lanes 0, 1 and 2 on)
template <int W>
__device__ inline void group_log3(double x0, double x1, double x2, int lane, int base, double &l0, double &l1,
                                  double &l2) {
  const double v = log(lane == 0 ? x0 : lane == 1 ? x1 : x2);
  l0 = group_bcast<W, 0>(v, base);
  l1 = group_bcast<W, 1>(v, base);
  l2 = group_bcast<W, 2>(v, base);
}

// BIEXP rise factor 1 - e^{-(t - t0) / tau_rise}, in (0, 1) for t > t0; t - t0 is at least an ulp
// of t0, so a product of eight factors stays far above the FP64 underflow threshold
__device__ inline double rise_factor(const ModelDev &md, int g, double t0) {
  return -expm1(-((double)g * md.dt - t0) * md.inv_tau1);
}

// The rise factor of the PE at grid point g from the table rt of md.rise_n entries (LDS):
// with n = g - g0 >= 0 and r_n = 1 - e^{-n dt / tau_rise},
//   1 - e^{-(g dt - t0) / tau_rise} = r_n + (1 - r_n) q1
// (every term positive: no cancellation, however close the PE is to t0).  One LDS read and two
// multiply-adds instead of an expm1 (about 45 instructions) per PE and sweep.
__device__ inline double rise_at(const ModelDev &md, const double *rt, const T0Terms &t, double t0, int g) {
  const int n = g - t.g0;
  // no table; or the rounding of g dt and ceil(t0 / dt) (dt not a power of two) disagrees
  if (md.rise_n == 0 || n < 0) return rise_factor(md, g, t0);
  const double r = rt[n < md.rise_n ? n : md.rise_n - 1];
  return fma(t.q1, 1.0 - r, r);
}

// v / sub and v % sub for v >= 0 (grid indices): shifts when sub is a power of two
__device__ inline int sub_div(const ModelDev &md, int v) { return md.sub_shift >= 0 ? v >> md.sub_shift : v / md.sub; }
__device__ inline int sub_mod(const ModelDev &md, int v) {
  return md.sub_shift >= 0 ? v & (md.sub - 1) : v % md.sub;
}

// overlap sum_{n < Lw} V(n - g1/sub) V(n - g2/sub): the stationary table unless both
// columns run past the window end, then the direct sum over the samples left
__device__ inline double overlap(const ModelDev &md, const double *vt, const double *ov, int g1, int g2, int Lw) {
  const int lo = g1 < g2 ? g1 : g2, hi = g1 < g2 ? g2 : g1;
  const int d = hi - lo;
  if (d >= md.M) return 0.0;
  const int nhi = sub_div(md, lo + md.M - 1);  // last sample of the earlier column
  if (nhi < Lw) return ov[sub_mod(md, lo) * md.M + d];
  double s = 0.0;
  const int n0 = sub_div(md, hi + md.sub - 1);
  for (int n = n0; n < Lw; ++n) s += vt[md.sub * n - lo] * vt[md.sub * n - hi];
  return s;
}

// Birth position: smallest g in T with sum_{g' <= g} phi(g' dt - t0) > target.  The partial sum
// over the first k points is Cd2 e2 (1 - a^k) - Cd12 e12 (1 - b^k), a = e^{-dt / tau2},
// b = e^{-dt / tau12}; with R the whole series less the target, it reaches the target where
//   k dt / tau2 = log(Cd2 e2 / R) + log(1 - w0 e^{-k dt / tau_rise}),   w0 = Cd12 e12 / (Cd2 e2).
// Two Newton steps in FP32 from the large-k solution land on the point or the one after it
// (measured: 99.7% on it, the rest one off, over the light curves of the workloads and rises
// from 0.3 to 20 ns); the group's lanes then evaluate the exact FP64 partial sums at that many
// neighbours and pick the first above the target, so the result is the search's own.  A guess
// outside the neighbourhood falls back to an LPC-ary search of the side it lies on.  One
// round trip to the table instead of log_LPC(points): 1 against 6 for 4-lane groups on
// 1,024-sample windows.
template <int LPC>
__device__ inline int birth_draw(const ModelDev &md, const T0Terms &t, double target, int lane, int grp) {
  const XsExp xe{t.e2, t.e12};
  const uint64_t gmask = (LPC == 64) ? ~0ull : ((1ull << (LPC & 63)) - 1ull);
  const int last = t.n - 1;
  int lo = 0, hi = last;
  {
    const double a2 = md.Cd2 * t.e2, a12 = md.Cd12 * t.e12;
    const double R = fma(md.Cd2, t.e2, -a12) - target;
    const float L = 0.69314718f * (fast_log2((float)a2) - fast_log2((float)R));
    const float w0 = (float)a12 * fast_rcp((float)a2);
    float k = L * md.ga_inv;
    if (md.kind != FSMP_PHI_EXP) {
#pragma unroll
      for (int it = 0; it < 2; ++it) {
        const float w = w0 * fast_exp2(-1.44269504f * md.gb * k);
        const float u = fmaxf(1.0f - w, 1e-6f);
        const float g = k * md.ga - L - 0.69314718f * fast_log2(u);
        const float gp = fmaxf(md.ga - w * md.gb * fast_rcp(u), 0.02f * md.ga);
        k = fmaxf(k - g * fast_rcp(gp), 0.0f);
      }
    }
    // R <= 0 (rounding, the last point), an overflow or a NaN: the guess is the last point
    int kg = R > 0.0 && k < (float)last ? (int)k : last;
    // the neighbours kg - LPC/2 .. kg + LPC/2 - 1, moved inside [0, last]
    int k0 = kg - LPC / 2;
    k0 = k0 > last - (LPC - 1) ? last - (LPC - 1) : k0;
    k0 = k0 < 0 ? 0 : k0;
    const int kl = k0 + lane > last ? last : k0 + lane;
    const bool pred = phi_partial(md, xe, kl + 1) > target;
    const uint64_t bal = (__ballot(pred) >> (grp * LPC)) & gmask;
    if (bal == 0) {
      lo = k0 + LPC > last ? last : k0 + LPC;  // past the neighbourhood (or the last point)
    } else {
      const int l = __ffsll((unsigned long long)bal) - 1;
      hi = k0 + l > last ? last : k0 + l;
      lo = l > 0 || k0 == 0 ? hi : 0;
    }
  }
  while (hi > lo) {
    const int span = hi - lo + 1;
    const int step = (span + LPC - 1) / LPC;
    int kl = lo + (lane + 1) * step - 1;
    if (kl > hi) kl = hi;
    const bool pred = phi_partial(md, xe, kl + 1) > target;
    const uint64_t bal = (__ballot(pred) >> (grp * LPC)) & gmask;
    if (bal == 0) {
      lo = hi;
      break;
    }
    const int l = __ffsll((unsigned long long)bal) - 1;
    int khi = lo + (l + 1) * step - 1;
    if (khi > hi) khi = hi;
    lo = (l == 0) ? lo : lo + l * step;
    hi = khi;
  }
  return t.gs + lo;
}

// ------------------------------------------------------------------ grid occupancy
// The occupancy row of waveform w (grid_sub * L_w points from grid_sub * offsets[w]) counts,
// over its chains' recorded sweeps, the PEs at every grid point.  It is accumulated by
// residence instead of per sweep: a PE that arrives in sweep s is present at the end of
// the sweeps s .. n_steps - 1, so it adds the recorded ones among them, n_steps - max(s,
// burn); one that leaves in sweep s removes the same amount.  The sum over a PE's arrival
// and departure is its number of recorded sweeps at that point, PEs still present at the
// end keep their arrival's count, and a chain starts empty.  Edits that cancel (both before
// burn-in) cost two atomics; nothing waits for the adds.
__device__ inline void occ_edit(const ChainArgs &a, int64_t c, int move, int gj, int gnew, int step, int burn,
                                int n_steps) {
  const int rem = n_steps - (step > burn ? step : burn);
  if (!a.occ || rem <= 0) return;
  // the row is looked up here rather than kept live across the sweep loop
  int32_t *row = a.occ + a.md.sub * a.woff[c / a.n_chains];
  if (move != 1) atomicAdd(row + gj, -rem);
  if (move != 2) atomicAdd(row + gnew, rem);
}

// ------------------------------------------------------------------ prologue
__global__ void __launch_bounds__(256) prologue_kernel(PrologueArgs a) {
  extern __shared__ double vt[];
  const ModelDev &md = a.md;
  for (int i = threadIdx.x; i < md.M; i += blockDim.x) vt[i] = a.vtab[i];
  __syncthreads();
  for (int64_t w = blockIdx.x; w < a.n_wave; w += gridDim.x) {
    const float *x = a.wave + a.woff[w];
    const int Lw = (int)(a.woff[w + 1] - a.woff[w]);
    int bad = 0;
    for (int n = threadIdx.x; n < Lw; n += blockDim.x)
      if (!isfinite(x[n])) bad = 1;
    bad = __syncthreads_or(bad);
    if (threadIdx.x == 0) a.wflags[w] = bad ? FSMP_ST_NONFINITE : 0u;
    if (a.occ)
      for (int64_t g = threadIdx.x; g < (int64_t)md.sub * Lw; g += blockDim.x) a.occ[md.sub * a.woff[w] + g] = 0;
    const int glo = a.grange[2 * w], ghi = a.grange[2 * w + 1];
    double *out = a.mf + a.mfoff[w];
    // four consecutive grid points per thread share each sample load; every point sums its
    // own samples n0(g) .. n1(g) in increasing n (both bounds nondecreasing in g)
    for (int g0 = glo + 4 * (int)threadIdx.x; g0 <= ghi; g0 += 4 * (int)blockDim.x) {
      int n0[4], n1[4];
      double s[4];
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        const int g = g0 + u;
        n0[u] = g <= ghi ? sub_div(md, g + md.sub - 1) : INT32_MAX;
        n1[u] = g <= ghi ? sub_div(md, g + md.M - 1) : -1;
        if (n1[u] > Lw - 1) n1[u] = Lw - 1;
        s[u] = 0.0;
      }
      const int gl = ghi - g0 < 3 ? ghi - g0 : 3;
      // samples that all four points take (four points in T) need no range checks
      const int blo = gl == 3 ? n0[3] : INT32_MAX, bhi = n1[0];
      int n = n0[0];
      for (; n <= n1[gl] && n < blo; ++n) {
        const double xv = (double)x[n];
#pragma unroll
        for (int u = 0; u < 4; ++u)
          if (n >= n0[u] && n <= n1[u]) s[u] += xv * vt[md.sub * n - (g0 + u)];
      }
      for (; n <= bhi; ++n) {
        const double xv = (double)x[n];
#pragma unroll
        for (int u = 0; u < 4; ++u) s[u] += xv * vt[md.sub * n - (g0 + u)];
      }
      for (; n <= n1[gl]; ++n) {
        const double xv = (double)x[n];
#pragma unroll
        for (int u = 0; u < 4; ++u)
          if (n >= n0[u] && n <= n1[u]) s[u] += xv * vt[md.sub * n - (g0 + u)];
      }
#pragma unroll
      for (int u = 0; u < 4; ++u)
        if (g0 + u <= ghi) out[g0 + u - glo] = s[u];
    }
  }
}

// ------------------------------------------------------------------ chains
// LDS block of one chain (its H lives in device memory): x, two scratch vectors (six
// and b in the FP32 form; b and the residual b - G x in the corrected FP64 form), the
// accumulators (kAcc doubles: 12 sums, 3 open batch sums, 5 work counters, then 8 int
// proposal / accept counts and the current run of N: value, first step), then the int grid
// indices.  The accumulators live in LDS, updated by the group's first lane, to keep
// registers free; the N histogram is kept in the output row by run lengths.
//
// kCorr, the corrected FP64 form (H in device memory, capacities from 48 up): FP64 arithmetic through an explicit inverse leaves x = G^-1 b with an error of about
// kappa(G) eps, which u+ = beta - gamma^T x and x_j carry into delta-nu magnified by
// 1 / (sigma_eps^2 delta^2) -- about 1e-8 of delta-nu on pile-up windows at K ~ 100, with or
// without rebuilds of G^-1.  That form keeps the exact G in device memory and the residual
// s = b - G x (recomputed after every accepted move), and evaluates
// gamma^T G^-1 b = gamma^T x + eta^T s and x_j = x_j + h^T s (eta = H gamma, h = row j of H),
// exact to first order in the error of H; the other quantities (delta^2, omega) need no
// correction at this precision.
template <int KCAP, bool F32 = false, bool MCP = false>
struct ChainLayout {
  static constexpr int LD = KCAP;
  static constexpr int kAcc = 25;
  static constexpr bool kCorr = !F32 && KCAP >= 48;
  static constexpr bool kKeepG = F32 || kCorr;  // the exact G in device memory, b per PE
  // the FP32 form keeps b (matched filter + rho mu_q per PE) for its residuals and refresh,
  // and the vectors of its corrected proposals; the mixture form the PEs' components after
  // their grid indices
  static constexpr int kVec = F32 ? 8 : (kCorr ? 5 : 3);
  static constexpr int kDoubles = kVec * KCAP + kAcc + (KCAP + 1) / 2 + (MCP ? (KCAP + 1) / 2 : 0);
};

// Column i of H owned by one lane: element (k, i) at H[(k * LD + i) * HS] (HS = 1 in LDS;
// the number of chains of a wavefront in device memory, where the wavefront's chains are
// interleaved element by element).  Loads go in chunks of 16 rows with one chain per
// wavefront and of 8 with several (whose kernels are short of registers: the smaller chunk
// keeps their spills down), issued unconditionally (rows below the capacity, a multiple of
// 16) with the rows past N dropped by a select, so a chunk costs one memory round trip;
// terms are summed in row order.
template <int LD, int HS, typename MT>
__device__ inline double grp_col_dot(const MT *H, const double *g, int i, int N) {
  constexpr int RC = HS > 1 ? 8 : 16;
  double e = 0.0;
  for (int k0 = 0; k0 < N; k0 += RC) {
    double h[RC], v[RC];
#pragma unroll
    for (int u = 0; u < RC; ++u) {
      h[u] = (double)H[((k0 + u) * LD + i) * HS];
      v[u] = g[k0 + u];
    }
#pragma unroll
    for (int u = 0; u < RC; ++u) e = (k0 + u < N) ? fma(h[u], v[u], e) : e;
  }
  return e;
}

// One element of an edit of G^-1, rounded as written here in every kernel (so a chain's state is the
// same bits in each): h + [(ui uk) cu + (vi vk) cv], of a single vector h + (ui uk) cu with the term
// rounded (what two vectors give with cv = 0); fused into h where a list is built.  Which of the two
// products is rounded first has no meaning; `first`, the first row of a chunk of eight, rounds the
// other one than the rest, so that chains keep the bits they have always had.
__device__ inline double edit_two(double h, double ui, double uk, double cu, double vi, double vk, double cv,
                                  bool first) {
  const double tu = ui * uk * cu, tv = vi * vk * cv;
  return h + (first ? fma(vi * vk, cv, tu) : fma(ui * uk, cu, tv));
}
__device__ inline double edit_one(double h, double ui, double uk, double cu) {
  const double t = ui * uk * cu;
  return h + t;
}
__device__ inline double edit_build(double h, double ui, double uk, double cu) { return fma(ui * uk, cu, h); }

// H(k, i) += ai A_k cA + bi B_k cB for k < N (TWO; edit_two), or the step of a list's build (loads of a
// chunk unconditional, stores guarded; an FP32 H is read into FP64 and written back rounded)
template <int LD, int HS, bool TWO, typename MT>
__device__ inline void grp_col_update(MT *H, int i, int N, double ai, const double *A, double cA, double bi,
                                      const double *B, double cB) {
  for (int k0 = 0; k0 < N; k0 += 8) {
    double h[8], av[8], bw[8];
#pragma unroll
    for (int u = 0; u < 8; ++u) {
      h[u] = (double)H[((k0 + u) * LD + i) * HS];
      av[u] = A[k0 + u];
      if (TWO) bw[u] = B[k0 + u];
    }
#pragma unroll
    for (int u = 0; u < 8; ++u) {
      double v;
      if constexpr (!TWO) {
        v = edit_build(h[u], ai, av[u], cA);
      } else if constexpr (HS > 1) {
        v = edit_two(h[u], ai, av[u], cA, bi, bw[u], cB, u == 0);
      } else {
        // one chain per wavefront: no other kernel repeats its rounding, which is left to the code
        // generator (168 and 232 ms for the launches of 128 and 160 in a batch of 250,000 tuned windows,
        // 174 and 240 with the products fused as in edit_two)
#pragma clang fp contract(fast)
        v = h[u] + (ai * av[u] * cA + bi * bw[u] * cB);
      }
      if (k0 + u < N) H[((k0 + u) * LD + i) * HS] = (MT)v;
    }
  }
}

// Residuals against the exact Gram matrix G = A^T A + rho I of the PE list (FP64, kept in
// device memory in the layout of H), for the rows i owned by this lane of the group:
//   r1 = g1 - G v1 (if v1),  r2 = e_u2 - G v2 (if v2; e_u2 the unit vector at u2),
//   r3 = t3 - G v3.
// Loads in chunks of 8 rows, terms in row order.
template <int LPC, int LD, int HS>
__device__ inline void gram_resid3(const double *Gm, int N, int lane, const double *g1, const double *v1, int u2,
                                   const double *v2, const double *t3, const double *v3, double *r1, double *r2,
                                   double *r3) {
  for (int i = lane; i < N; i += LPC) {
    double a = 0.0, b = 0.0, c = 0.0;
    for (int k0 = 0; k0 < N; k0 += 8) {
      double g[8], x1[8], x2[8], x3[8];
#pragma unroll
      for (int u = 0; u < 8; ++u) {
        g[u] = Gm[((k0 + u) * LD + i) * HS];
        x1[u] = v1 ? v1[k0 + u] : 0.0;
        x2[u] = v2 ? v2[k0 + u] : 0.0;
        x3[u] = v3[k0 + u];
      }
#pragma unroll
      for (int u = 0; u < 8; ++u) {
        const bool in = k0 + u < N;
        a = in ? a + g[u] * x1[u] : a;
        b = in ? b + g[u] * x2[u] : b;
        c = in ? c + g[u] * x3[u] : c;
      }
    }
    if (v1) r1[i] = g1[i] - a;
    if (v2) r2[i] = (i == u2 ? 1.0 : 0.0) - b;
    r3[i] = t3[i] - c;
  }
}

// s = b - G x against the exact G, for the rows i owned by this lane of the group
template <int LPC, int LD, int HS>
__device__ inline void gram_resid_b(const double *Gm, const double *bv, const double *xv, double *rs, int N,
                                    int lane) {
  for (int i = lane; i < N; i += LPC) rs[i] = bv[i] - grp_col_dot<LD, HS>(Gm, xv, i, N);
}

// column i of G (overlap tables, plus the PE's own ridge rho_g on the diagonal) for the PE at
// grid point g against the list zg[0..N), written as row and column i of Gm by the lanes of
// the group (g's own entry by the first lane); zg[i] is not read
template <int LPC, int LD, int HS>
__device__ inline void gram_set(const ModelDev &md, const double *vt, const double *ov, int Lw, double *Gm,
                                const int *zg, int N, int i, int g, double rho_g, int lane) {
  for (int k = lane; k < N; k += LPC) {
    if (k == i) continue;
    const double v = overlap(md, vt, ov, g, zg[k], Lw);
    Gm[(i * LD + k) * HS] = v;
    Gm[(k * LD + i) * HS] = v;
  }
  if (lane == 0) Gm[(i * LD + i) * HS] = overlap(md, vt, ov, g, g, Lw) + rho_g;
}

// A lane's part of a sum of products over the PEs of a chain.  SPLIT: 4 lanes in the order of 16 with
// an element each (group_sum<16>): products rounded, elements l and l + 8, l + 4 and l + 12 of lane l
// (its first and third, second and fourth), then the two; the parts change places at each element.
template <bool SPLIT>
struct LaneSum {
  double a = 0.0, b = 0.0;
  __device__ inline void term(double x) {
    const double t = a + x;
    a = SPLIT ? b : t;
    if (SPLIT) b = t;
  }
  __device__ inline void mac(double x, double y) {
    if constexpr (SPLIT) {
      const double p = x * y;
      term(p);
    } else {
      a = fma(x, y, a);
    }
  }
  template <int LPC>
  __device__ inline double sum() const {
    return group_sum<LPC>(SPLIT ? a + b : a);
  }
};

template <int W>
__device__ inline double group_max(double v) {
#pragma unroll
  for (int o = W / 2; o > 0; o >>= 1) v = fmax(v, __shfl_xor(v, o, W));
  return v;
}

// G^-1 of the PE list zg[0..N) by bordering, in FP64 into M (layout of the lane-group
// kernels; M may hold the old G^-1: only its leading block built so far is read), each step
// the birth update of the inverse of the leading block, its columns owned by the group's
// lanes: false if a Schur complement is not positive.  ek: the PEs' mixture components (their
// own ridge rho_e on the diagonal), or null for the single charge law.  s1, s2: scratch.
template <int LPC, int LD, int HS, bool SPLIT = false>
__device__ bool grp_build(const ModelDev &md, const double *vt, const double *ov, int Lw, double *M, double *s1,
                          double *s2, const int *zg, int N, int lane, const int *ek = nullptr) {
  for (int k = 0; k < N; ++k) {
    const int gk = zg[k];
    for (int i = lane; i < k; i += LPC) s1[i] = overlap(md, vt, ov, gk, zg[i], Lw);
    const double d = overlap(md, vt, ov, gk, gk, Lw) + (ek ? md.mix_rho[ek[k]] : md.rho);
    WAVE_SYNC();
    LaneSum<SPLIT> q;
    for (int i = lane; i < k; i += LPC) {
      const double e = grp_col_dot<LD, HS>(M, s1, i, k);
      s2[i] = e;
      q.mac(s1[i], e);
    }
    const double delta2 = d - q.template sum<LPC>();
    if (!(delta2 > 0.0)) return false;
    const double inv = 1.0 / delta2;
    WAVE_SYNC();
    for (int i = lane; i < k; i += LPC) {
      const double ei = s2[i];
      grp_col_update<LD, HS, false>(M, i, k, ei, s2, inv, 0.0, s2, 0.0);
      M[(k * LD + i) * HS] = -ei * inv;
      M[(i * LD + k) * HS] = -ei * inv;
    }
    if (lane == 0) M[(k * LD + k) * HS] = inv;
    WAVE_SYNC();
  }
  return true;
}

// Precision form: rebuild G^-1 of the current PE list in FP64 into W, recompute x = G^-1 b in
// FP64 and round W into the FP32 H.  False if a Schur complement is not positive.  `drift` =
// the largest change of a charge mean, relative to max(1, |x|).  s1, s2 are scratch.
template <int LPC, int LD, int HS, bool SPLIT, typename HT>
__device__ bool grp_refresh(const ModelDev &md, const double *vt, const double *ov, int Lw, double *W, HT *H,
                            double *xv, const double *bv, double *s1, double *s2, const int *zg, int N, int lane,
                            double &drift) {
  if (!grp_build<LPC, LD, HS, SPLIT>(md, vt, ov, Lw, W, s1, s2, zg, N, lane)) return false;
  double dr = 0.0;
  for (int i = lane; i < N; i += LPC) {
    const double xi = grp_col_dot<LD, HS>(W, bv, i, N);
    dr = fmax(dr, fabs(xi - xv[i]) / fmax(1.0, fabs(xi)));
    xv[i] = xi;
  }
  drift = group_max<LPC>(dr);
  for (int i = lane; i < N; i += LPC)
    for (int k = 0; k < N; ++k) H[(k * LD + i) * HS] = (HT)W[(k * LD + i) * HS];
  WAVE_SYNC();
  return true;
}

// H in device memory (a.dws, the chains of a wavefront interleaved element by element), which
// leaves the LDS to the tables and the vectors and so fits many more chains per CU than
// chain_lds_kernel does.  FORCE (replay): every step follows the recorded proposal of a.force
// (t0 after the half-step, move, index, grid point, accept bit) instead of the chain's
// own draws, and writes the delta-nu and log-acceptance it computes to a.rdnu / a.rla.
// MCP: the Gaussian-mixture charge law, every PE with its component.
template <int KCAP, int LPC, int WPB, bool FORCE, bool F32, bool MCP>
__global__ void __launch_bounds__(kWave *WPB) __attribute__((amdgpu_waves_per_eu(2))) chain_kernel(ChainArgs a) {
  static_assert(!F32 || !FORCE, "the FP32 form does not replay");
  static_assert(!MCP || (!FORCE && !F32), "the mixture form runs FP64 and does not replay");
  static_assert(KCAP % 16 == 0, "the column loads go in chunks of 16 rows below the capacity");
  using HT = typename std::conditional<F32, float, double>::type;
  // The FP32 form runs capacity 16 in groups of 16 lanes or, with many chains, of 4: the 4 lanes take
  // their sums in the order of the 16, and the 16 their t0 products by the classes of the 4, so that a
  // chain is the same bits in either.  (In the 4 lanes 64,000 chains x 400 sweeps take 22.4 ms, 21.8 in
  // an order of their own.)
  constexpr bool SPLIT = F32 && KCAP == 16 && LPC == 4;
  constexpr int TRO = F32 && LPC == 16 ? 4 : LPC;
  constexpr int CPW = kWave / LPC;
  using CL = ChainLayout<KCAP, F32, MCP>;
  constexpr int LD = CL::LD;
  constexpr int HS = CPW;
  extern __shared__ double smem[];
  const ModelDev &md = a.md;
  double *vt = smem;
  double *ov = smem + md.M;
  for (int i = threadIdx.x; i < md.M; i += blockDim.x) vt[i] = a.vtab[i];
  for (int i = threadIdx.x; i < md.sub * md.M; i += blockDim.x) ov[i] = a.ovl[i];
  double *lgn = ov + md.sub * md.M;  // log k, k = 0..KCAP + 1
  for (int i = threadIdx.x; i < KCAP + 2; i += blockDim.x) lgn[i] = log((double)i);
  double *rt = lgn + KCAP + 2;  // rise factors at whole grid steps (rise_at)
  for (int i = threadIdx.x; i < md.rise_n; i += blockDim.x) rt[i] = md.rtab[i];
  __syncthreads();

  // the wavefront's index is the same in all its lanes: taken from the first, it and what
  // follows from it (the tile, and with one chain per wavefront the chain and its waveform's
  // parameters) are held in scalar registers, which keeps those kernels free of spills
  const int wv = __builtin_amdgcn_readfirstlane((int)(threadIdx.x / kWave)), l64 = threadIdx.x % kWave;
  const int grp = l64 / LPC, lane = l64 % LPC;
  const int gbase = grp * LPC;  // the group's first lane in the wavefront
  const int64_t tile = (int64_t)blockIdx.x * WPB + wv;
  const int64_t slot = tile * CPW + grp;
  if (slot >= a.n_list) return;

  double *cb = smem + md.M * (1 + md.sub) + (KCAP + 2) + md.rise_n + (int64_t)(wv * CPW + grp) * CL::kDoubles;
  // device memory of a tile (the wavefront's chains interleaved element by element): H in its
  // storage type; in the FP32 form then the FP64 refresh matrix W and the exact G (FP64), in
  // the corrected FP64 form the exact G
  constexpr bool CORR = CL::kCorr, KEEPG = CL::kKeepG;
  constexpr int64_t kHD = (int64_t)KCAP * LD * CPW * (int64_t)sizeof(HT) / 8;
  constexpr int64_t kTile = kHD + (F32 ? 2 : CORR ? 1 : 0) * (int64_t)KCAP * LD * CPW;
  HT *H = (HT *)(a.dws + tile * kTile) + grp;
  double *W = F32 ? a.dws + tile * kTile + kHD + grp : nullptr;
  double *Gm = F32    ? a.dws + tile * kTile + kHD + (int64_t)KCAP * LD * CPW + grp
               : CORR ? a.dws + tile * kTile + kHD + grp
                      : nullptr;
  double *xv = cb;
  double *s1 = xv + KCAP;
  double *s2 = s1 + KCAP;
  // FP32 form: four more scratch vectors and b of each PE; corrected FP64 form: b and the
  // residual s = b - G x
  double *s3 = F32 ? s2 + KCAP : nullptr;
  double *s4 = F32 ? s3 + KCAP : nullptr;
  double *s5 = F32 ? s4 + KCAP : nullptr;
  double *s6 = F32 ? s5 + KCAP : nullptr;
  double *bv = F32 ? s6 + KCAP : CORR ? s2 + KCAP : nullptr;
  double *rs = CORR ? bv + KCAP : nullptr;
  double *acc = xv + CL::kVec * KCAP;  // [0..11] sums, [12..14] open batch sums, [15..19] work counters
  int *cnt = (int *)(acc + 20);
  int *run = cnt + 8;  // N of the current run among the recorded steps (-1: none yet), its first step
  int *zg = (int *)(acc + CL::kAcc);
  int *ek = zg + 2 * ((KCAP + 1) / 2);  // mixture form: the PEs' components

  const int64_t c = a.chains[slot];
  const int64_t w = c / a.n_chains;
  const int ch = (int)(c % a.n_chains);
  const int Lw = (int)(a.woff[w + 1] - a.woff[w]);
  const double lam = a.lam[w];
  const int kmax = a.kmax[w];
  const int glo = a.grange[2 * w], ghi = a.grange[2 * w + 1];
  const double *mf = a.mf + a.mfoff[w];
  const uint64_t uid = a.wid[w] * (uint64_t)a.n_chains + (uint64_t)ch;
  const uint32_t uid0 = (uint32_t)uid, uid1 = (uint32_t)(uid >> 32);
  uint32_t st = a.wflags[w];
  if (glo > ghi) st |= FSMP_ST_EMPTY_T;
  // this waveform's sweeps and burn-in (the configured burn-in fraction), batch means
  const int steps_w = a.wsteps ? a.wsteps[w] : a.n_steps;
  const int burn = a.wsteps ? (int)((int64_t)steps_w * a.burn_in / a.n_steps) : a.burn_in;
  const int n_steps = (st & FSMP_ST_NONFINITE) ? 0 : steps_w;
  const int S_rec = n_steps > burn ? n_steps - burn : 0;
  const int nb = S_rec > 0 ? (int)floor(sqrt((double)S_rec)) : 0;
  const int lb = nb > 0 ? S_rec / nb : 0;

  // N histogram: the output row, zeroed here, receives the length of every run of equal
  // N among the recorded steps (atomic adds that nothing waits for)
  for (int k = lane; k <= a.kz; k += LPC) a.nhist[c * (a.kz + 1) + k] = 0;
  if (lane == 0) {
    run[0] = -1;
    run[1] = 0;
  }
  WAVE_SYNC();

  double t0 = a.t0init[w];
  int N = 0;
  // the light curve's terms at t0; Lambda_T changes only with t0 (its log is taken with the
  // jump's own log); gmin = the smallest PE grid index (phi must stay positive at every PE)
  T0Terms tc{};
  if (glo <= ghi) {
    tc = t0_terms<LPC>(md, t0, glo, ghi, lane, gbase);
    t0_phi(md, tc);
  }
  double Lam = lam * md.dt * tc.Phi;
  const bool biexp = md.kind == FSMP_PHI_BIEXP;
  int gmin = INT32_MAX;
  if (lane == 0) {
    for (int i = 0; i < 20; ++i) acc[i] = 0.0;
    for (int i = 0; i < 8; ++i) cnt[i] = 0;
  }
  WAVE_SYNC();

  // a caller-supplied initial PE list: G^-1 (FP64, by bordering) and x = G^-1 b of the
  // list before the first sweep; no random numbers are drawn for it
  if (a.zinit && n_steps > 0) {
    const int n0 = (int)(a.zinit_off[c + 1] - a.zinit_off[c]);
    if (n0 > 0) {
      const int32_t *z0 = a.zinit + a.zinit_off[c];
      for (int k = lane; k < n0; k += LPC) zg[k] = z0[k];
      WAVE_SYNC();
      double *M = F32 ? W : (double *)H;
      if (grp_build<LPC, LD, HS, SPLIT>(md, vt, ov, Lw, M, s1, s2, zg, n0, lane)) {
        for (int k = lane; k < n0; k += LPC) s1[k] = mf[zg[k] - glo] + md.rhom;  // b
        WAVE_SYNC();
        for (int i = lane; i < n0; i += LPC) {
          xv[i] = grp_col_dot<LD, HS>(M, s1, i, n0);
          if constexpr (KEEPG) {
            bv[i] = s1[i];
            for (int k = 0; k < n0; ++k) {
              if constexpr (F32) H[(k * LD + i) * HS] = (HT)W[(k * LD + i) * HS];
              Gm[(k * LD + i) * HS] = overlap(md, vt, ov, zg[k], zg[i], Lw) + (k == i ? md.rho : 0.0);
            }
          }
        }
        if constexpr (CORR) {
          WAVE_SYNC();
          gram_resid_b<LPC, LD, HS>(Gm, bv, xv, rs, n0, lane);
        }
        N = n0;
        int m = INT32_MAX;
        for (int i = lane; i < N; i += LPC) {
          m = zg[i] < m ? zg[i] : m;
          occ_edit(a, c, 1, -1, zg[i], 0, burn, n_steps);
        }
        gmin = group_min<LPC>(m);
      } else {
        st |= FSMP_ST_FACTOR;
      }
      WAVE_SYNC();
    }
  }
  // with one chain per wavefront, or in the FP64 form's 32-lane groups, lane l of a chain's
  // group keeps the random values of its sweep LPC m + l
  constexpr bool kStash = LPC == kWave || (LPC == 32 && !F32 && !MCP);
  uint32_t st_r3 = 0, st_r4 = 0, st_r5 = 0, st_r7 = 0;
  double st_l2 = 0.0, st_l6 = 0.0, st_xt = 0.0, st_xs = 0.0;
  for (int step = 0; step < n_steps; ++step) {
    if (a.refresh_M > 0 && step > 0 && step % a.refresh_M == 0 && N > 0) {
      if constexpr (F32) {
        // precision form: FP64 rebuild of G^{-1} every refresh_M sweeps
        double drift;
        if (!grp_refresh<LPC, LD, HS, SPLIT>(md, vt, ov, Lw, W, H, xv, bv, s1, s2, zg, N, lane, drift)) st |= FSMP_ST_FACTOR;
        else if (drift > a.drift_bound) st |= FSMP_ST_DRIFT;
      } else if constexpr (!CORR) {
        // FP64 form: G^-1 rebuilt in place by bordering and x = G^-1 b recomputed, against the
        // rounding the rank-one and rank-two edits accumulate (the corrected form needs none:
        // the residual against the exact G takes up what the edits leave in x, and over 4,000
        // sweeps at K ~ 100 its delta-nu is as close to the exact one without rebuilds as with)
        if (grp_build<LPC, LD, HS>(md, vt, ov, Lw, (double *)H, s1, s2, zg, N, lane, MCP ? ek : nullptr)) {
          for (int i = lane; i < N; i += LPC) s1[i] = mf[zg[i] - glo] + (MCP ? md.mix_rhom[ek[i]] : md.rhom);
          WAVE_SYNC();
          for (int i = lane; i < N; i += LPC) xv[i] = grp_col_dot<LD, HS>((double *)H, s1, i, N);
          WAVE_SYNC();
        } else {
          st |= FSMP_ST_FACTOR;
        }
      }
    }
    // The step's random words and the logs of its three uniforms (Box-Muller radius, t0
    // acceptance, jump acceptance) do not depend on the chain's state: the group's first
    // lane makes Philox block 0 and its second lane block 1, its first three lanes one log
    // each, and the values go to the whole group by lane permutes (the same values as
    // computing all of it in every lane, with a third of the VALU work)
    static_assert(LPC >= 4, "a chain's group needs at least three lanes");
    uint32_t r[8];
    double lg2, lg6;      // log u01(r2), log u01(r6)
    double xi_t0, xi_sh;  // the Box-Muller pair of (r0, r1)
    if constexpr (kStash) {
      // every LPC sweeps each lane of a chain's group makes the random values of one of the
      // group's next LPC sweeps (both Philox blocks, the three logs, the Box-Muller pair), the
      // same functions of the same words as below, so the same values; a sweep reads its own
      // by lane reads (one per group of the wavefront, its own picked), off the sweep's
      // dependent path
      const int sl = step & (LPC - 1);
      if (sl == 0) {
        uint32_t q0[4], q1[4];
        philox4x32_10((uint32_t)(step + lane), 0u, uid0, uid1, a.key0, a.key1, q0);
        philox4x32_10((uint32_t)(step + lane), 1u, uid0, uid1, a.key0, a.key1, q1);
        const double R = sqrt(-2.0 * log(u01(q0[0])));
        const double th = 2.0 * M_PI * u01(q0[1]);
        st_xt = R * cos(th);
        st_xs = R * sin(th);
        st_l2 = log(u01(q0[2]));
        st_l6 = log(u01(q1[2]));
        st_r3 = q0[3];
        st_r4 = q1[0];
        st_r5 = q1[1];
        st_r7 = q1[3];
      }
      r[0] = r[1] = r[2] = r[6] = 0u;  // consumed by the values above
      r[3] = group_lane_u32<LPC>(st_r3, sl, grp);
      r[4] = group_lane_u32<LPC>(st_r4, sl, grp);
      r[5] = group_lane_u32<LPC>(st_r5, sl, grp);
      r[7] = group_lane_u32<LPC>(st_r7, sl, grp);
      lg2 = group_lane<LPC>(st_l2, sl, grp);
      lg6 = group_lane<LPC>(st_l6, sl, grp);
      xi_t0 = group_lane<LPC>(st_xt, sl, grp);
      xi_sh = group_lane<LPC>(st_xs, sl, grp);
    } else {
      double lg0;  // log u01(r0)
      {
        const int base = gbase;
        uint32_t q[4];
        philox4x32_10((uint32_t)step, (uint32_t)(lane & 1), uid0, uid1, a.key0, a.key1, q);
#pragma unroll
        for (int u = 0; u < 4; ++u) {
          r[u] = group_bcast<LPC, 0>(q[u], base);
          r[4 + u] = group_bcast<LPC, 1>(q[u], base);
        }
        const double lv = log(u01(lane == 0 ? r[0] : lane == 1 ? r[2] : r[6]));
        lg0 = group_bcast<LPC, 0>(lv, base);
        lg2 = group_bcast<LPC, 1>(lv, base);
        lg6 = group_bcast<LPC, 2>(lv, base);
      }
      const double R = sqrt(-2.0 * lg0);
      const double th = 2.0 * M_PI * u01(r[1]);
      xi_t0 = R * cos(th);
      xi_sh = R * sin(th);
    }

    // ---- Gibbs half-step 1: t0 by Metropolis-Hastings
    const double t0p = t0 + md.t0_sd * xi_t0;
    bool t0acc = false;
    if (lane == 0) cnt[0]++;
    fsmp_logrec rec{};
    if (FORCE) {
      rec = a.force[c * (int64_t)a.n_steps + step];
      t0acc = (rec.flags & 4) != 0;
      if (rec.t0 != t0) {
        t0 = rec.t0;
        if (glo <= ghi) {
          tc = t0_terms<LPC>(md, t0, glo, ghi, lane, gbase);
          t0_phi(md, tc);
        }
        Lam = lam * md.dt * tc.Phi;
      }
    } else if (t0p >= md.t0_min && t0p <= md.t0_max) {
      const double xmin = (N > 0) ? (double)gmin * md.dt - t0p : 1.0;
      if (biexp ? (xmin > 0.0) : (xmin >= 0.0)) {
        T0Terms tp = tc;
        if (glo <= ghi) tp = t0_terms<LPC>(md, t0p, glo, ghi, lane, gbase);
        double S = 0.0;  // sum over the PEs of log r(t0p) / r(t0), r the rise factor
        if (biexp && N > 0) {
          // the rise factors of a lane's PEs at both t0 multiplied (each at least an ulp of t0 over
          // tau_rise: eight are far from underflow), one log per lane.  PEs m and m + H of a lane
          // first, then every other of those, then the two halves: the order of class_product
          constexpr int E = (KCAP + LPC - 1) / LPC, H = (E + 1) / 2;
          static_assert(E <= 8, "one log per lane");
          double pn[2] = {1.0, 1.0}, pc[2] = {1.0, 1.0};
          int i = lane;
          for (int m = 0; m < H && i < N; ++m, i += LPC) {
            double n0 = rise_at(md, rt, tp, t0p, zg[i]), c0 = rise_at(md, rt, tc, t0, zg[i]);
            if (i + H * LPC < N) {
              const int g = zg[i + H * LPC];
              n0 *= rise_at(md, rt, tp, t0p, g);
              c0 *= rise_at(md, rt, tc, t0, g);
            }
            if (m & 1) {
              pn[1] *= n0;
              pc[1] *= c0;
            } else {
              pn[0] *= n0;
              pc[0] *= c0;
            }
          }
          if constexpr (TRO < LPC) {
            S = group_sum<TRO>(log(class_product<LPC, TRO>(pn[0] * pn[1]) / class_product<LPC, TRO>(pc[0] * pc[1])));
          } else {
            S = group_sum<LPC>(log((pn[0] * pn[1]) / (pc[0] * pc[1])));
          }
        }
        if (glo <= ghi) t0_phi(md, tp);
        const double part = (double)N * (t0p - t0) * md.inv_tau2 + S;
        const double la0 = part - (lam * md.dt * tp.Phi - lam * md.dt * tc.Phi);
        if (lg2 < la0) {
          t0 = t0p;
          tc = tp;
          Lam = lam * md.dt * tc.Phi;
          t0acc = true;
          if (lane == 0) cnt[1]++;
        }
      }
    }

    // ---- Gibbs half-step 2: one RJMCMC jump
    const double um = u01(r[3]);
    const int move = FORCE ? rec.move : ((N == 0 || um < md.J) ? 1 : (um < 2.0 * md.J ? 2 : 3));
    // replay: only the recorded valid proposals are evaluated, and only well-formed ones
    const bool consider =
        !FORCE || ((rec.flags & 1) && (move == 1 ? (rec.g >= glo && rec.g <= ghi)
                                                 : (move == 2 || move == 3) && rec.j >= 0 && rec.j < N));
    // A wavefront carries several chains whose moves differ; the expensive parts are
    // written once so that it executes them once: the proposal evaluation shared by
    // births and time shifts, and one rank-two edit for every accepted move.
    int j = -1, gnew = -1, sh = 0;
    // need_mv: a birth part (births, shifts); need_dp: in the FP32 form, a death part
    // (deaths, shifts) evaluated with the residual correction
    bool valid = false, need_mv = false, need_dp = false;
    // lpd: log phi at a shift's new position less that at its old one; pr_sh: the ratio of their
    // rise factors, whose log is part of it
    double dnu = 0.0, la = -INFINITY, lpd = 0.0, pr_sh = 1.0;
    // xjp: x_j as stored (the corrected FP64 form evaluates with xj = x_j + h^T s and edits x
    // with the stored value, which keeps x = H b along the edits)
    double delta2 = 1.0, up = 0.0, om = 1.0, xj = 0.0, xjp = 0.0, ej = 0.0, beta = 0.0;
    // mixture form: the component of a born or updated PE from word r7 (inverse CDF of the
    // weights); rho, its log, rho mu, rho mu^2 of the new and of the removed / moved PE
    int enew = 0;
    double rn = md.rho, lrn = md.log_rho, rmn = md.rhom, rm2n = md.rhom2;
    double lro = md.log_rho, rm2o = md.rhom2;
    if constexpr (MCP) {
      const double ue = u01(r[7]);
      enew = md.n_mix - 1;
      for (int q = md.n_mix - 2; q >= 0; --q)
        if (ue < md.mix_cdf[q]) enew = q;
      rn = md.mix_rho[enew];
      lrn = md.mix_lrho[enew];
      rmn = md.mix_rhom[enew];
      rm2n = md.mix_rhom2[enew];
    }
    if (move == 1) {
      if (lane == 0) cnt[2]++;
      if (N >= kmax) {
        st |= FSMP_ST_KMAX;
      } else if (tc.Phi > 0.0 && consider) {
        gnew = FORCE ? rec.g : birth_draw<LPC>(md, tc, u53(r[4], r[5]) * tc.Phi, lane, grp);
        need_mv = Lam > 0.0;
      }
    } else {
      j = FORCE ? rec.j : (int)(((uint64_t)r[4] * (uint64_t)N) >> 32);
      if (!consider) {
        j = -1;  // replay: not a recorded valid proposal
      } else if (move == 2) {
        if (lane == 0) cnt[4]++;
        if constexpr (F32) {
          need_dp = true;
        } else {
          om = H[(j * LD + j) * HS];
          xj = xjp = xv[j];
          if constexpr (CORR) {
            double xc = 0.0;
            for (int i = lane; i < N; i += LPC) xc = fma(H[(j * LD + i) * HS], rs[i], xc);
            xj += group_sum<LPC>(xc);
          }
          if constexpr (MCP) {
            lro = md.mix_lrho[ek[j]];
            rm2o = md.mix_rhom2[ek[j]];
          }
          if (om > 0.0) {
            double lom, lLam;
            group_log2<LPC>(om, Lam, lane, gbase, lom, lLam);
            const double v = -lro - lom + (rm2o - ratio(xj * xj, om, 1.0 / om)) * md.inv_s;
            dnu = 0.5 * v;
            la = fma(0.5, v, -lLam) + lgn[N] - (N == 1 ? md.logJ : 0.0);
            valid = true;
          } else {
            st |= FSMP_ST_FACTOR;
          }
        }
      } else {
        if (lane == 0) cnt[6]++;
        sh = FORCE ? rec.g - zg[j] : (int)rint(xi_sh * md.shift_sd / md.dt);
        gnew = zg[j] + sh;
        if (gnew >= glo && gnew <= ghi) {
          const double xnew = (double)gnew * md.dt - t0;
          if (biexp ? xnew > 0.0 : xnew >= 0.0) {
            if constexpr (FORCE) {
              // a recorded t0 may lie after the old position (log phi = -inf there)
              lpd = log_phi(md, xnew) - log_phi(md, (double)zg[j] * md.dt - t0);
            } else {
              lpd = (double)(zg[j] - gnew) * md.dt * md.inv_tau2;
              if (biexp && sh != 0) pr_sh = rise_at(md, rt, tc, t0, gnew) / rise_at(md, rt, tc, t0, zg[j]);
              if constexpr (F32) lpd += log(pr_sh);
            }
            if constexpr (MCP) {
              lro = md.mix_lrho[ek[j]];
              rm2o = md.mix_rhom2[ek[j]];
            }
            if (sh == 0 && (!MCP || enew == ek[j])) {
              valid = true;
              dnu = 0.0;
              la = 0.0;
            } else {
              need_mv = true;
              need_dp = F32;
            }
          }
        }
      }
    }
    // birth or time shift: gamma = overlaps of the new position with the PEs (zero at the
    // shifted one), eta = M gamma, q = gamma^T eta, p = gamma^T x, for M = H or (precision
    // form, near the threshold) its FP64 rebuild W
    auto eval_mv = [&](auto *M) {
      valid = false;
      const int jz = move == 3 ? j : -1;
      for (int i = lane; i < N; i += LPC) s1[i] = (i == jz) ? 0.0 : overlap(md, vt, ov, gnew, zg[i], Lw);
      const double d = overlap(md, vt, ov, gnew, gnew, Lw) + rn;
      beta = mf[gnew - glo] + rmn;
      WAVE_SYNC();
      double q = 0.0, p = 0.0, pc = 0.0, xc = 0.0;
      for (int i = lane; i < N; i += LPC) {
        const double e = grp_col_dot<LD, HS>(M, s1, i, N);
        s2[i] = e;
        q = fma(s1[i], e, q);
        p = fma(s1[i], xv[i], p);
        if constexpr (CORR) {
          pc = fma(e, rs[i], pc);
          if (move == 3) xc = fma((double)M[(j * LD + i) * HS], rs[i], xc);
        }
      }
      q = group_sum<LPC>(q);
      p = group_sum<LPC>(p);
      if constexpr (CORR) {
        p += group_sum<LPC>(pc);
        if (move == 3) xc = group_sum<LPC>(xc);
      }
      if (move == 1) {
        delta2 = d - q;
        if (delta2 > 0.0) {
          up = beta - p;
          double ld2, lLam;
          group_log2<LPC>(delta2, Lam, lane, gbase, ld2, lLam);
          const double v = -lrn + ld2 + (rm2n - ratio(up * up, delta2, 1.0 / delta2)) * md.inv_s;
          dnu = -0.5 * v;
          la = fma(-0.5, v, lLam) - lgn[N + 1] + (N == 0 ? md.logJ : 0.0);
          valid = true;
        } else {
          st |= FSMP_ST_FACTOR;
        }
      } else {
        WAVE_SYNC();
        om = (double)M[(j * LD + j) * HS];
        xj = xjp = xv[j];
        if constexpr (CORR) xj += xc;
        ej = s2[j];
        delta2 = d - (q - ej * ej / om);
        up = beta - (p - ej * xj / om);
        if (delta2 > 0.0 && om > 0.0) {
          double lom, ld2, lpr;
          group_log3<LPC>(om, delta2, pr_sh, lane, gbase, lom, ld2, lpr);
          dnu = 0.5 * (-lom - ld2 + (ratio(up * up, delta2, 1.0 / delta2) - ratio(xj * xj, om, 1.0 / om)) * md.inv_s);
          // mixture form: the removed and the added PE carry their own rho and rho mu^2
          if constexpr (MCP) dnu += 0.5 * (lrn - lro + (rm2o - rm2n) * md.inv_s);
          la = dnu + (lpd + lpr);
          valid = true;
        } else {
          st |= FSMP_ST_FACTOR;
        }
      }
    };
    // The FP32 form evaluates a proposal from its FP32 H with a two-term correction against
    // the exact G (FP64 in device memory, kept with the list).  For a vector f and its
    // approximate solve a = H f, the residual r = f - G a and the correction H r, the bilinear
    // form f'^T G^-1 f is f'^T a + a^T r' + r^T H r' to second order in the error of H (the
    // first term of the correction cancels the first-order error exactly; the last term is
    // the size of what is corrected at second order, taken as the bound of what is left, as
    // the error contracts by |I - H G| per term).  The vectors are gamma (the new position's
    // overlaps, 0 at j for a shift: births and shifts), e_j (deaths and shifts) and b:
    //   Qgg = gamma^T G^-1 gamma, Qjg = e_j^T G^-1 gamma, omega = (G^-1)_jj,
    //   Pg = gamma^T G^-1 b, xj = e_j^T G^-1 b,
    // from one pass over H (eta = H gamma, h = row j), one over G (r_eta, r_h, s = b - G x)
    // and one over H again (H r_eta, H r_h).  A shift's birth part is on the PEs without j, by
    // the identities (G without j)^-1 = (G^-1 - u u^T / omega) there, u = G^-1 e_j:
    //   delta^2 = d - (Qgg - Qjg^2 / omega),  u+ = beta - (Pg - Qjg xj / omega),
    // with each bound carried through them.  bnd is the bound of delta-nu to first order, times
    // four.  Vectors left for the edit: u = h + H r_h in s1, eta + H r_eta (for a shift minus
    // u Qjg / omega, 0 at j) in s3.
    double bnd = 0.0;
    bool inexact = false;
    auto f32_dnu = [&](double Bom, double Bxj, double Bq, double Bp) {
      const double s = md.s;
      if (move == 1) {
        double ld2, lLam;
        group_log2<LPC>(delta2, Lam, lane, gbase, ld2, lLam);
        dnu = -0.5 * (-md.log_rho + ld2 + (md.rhom2 - up * up / delta2) * md.inv_s);
        la = dnu + lLam - lgn[N + 1] + (N == 0 ? md.logJ : 0.0);
      } else if (move == 2) {
        double lom, lLam;
        group_log2<LPC>(om, Lam, lane, gbase, lom, lLam);
        dnu = 0.5 * (-md.log_rho - lom + (md.rhom2 - xj * xj / om) * md.inv_s);
        la = dnu - lLam + lgn[N] - (N == 1 ? md.logJ : 0.0);
      } else {
        double lom, ld2;
        group_log2<LPC>(om, delta2, lane, gbase, lom, ld2);
        dnu = 0.5 * (-lom - ld2 + (up * up / delta2 - xj * xj / om) * md.inv_s);
        la = dnu + lpd;
      }
      double b = 0.0;
      if (move != 2) b += 0.5 * fabs(1.0 / delta2 + up * up / (delta2 * delta2 * s)) * Bq + fabs(up) / (delta2 * s) * Bp;
      if (move != 1) b += 0.5 * fabs(1.0 / om - xj * xj / (om * om * s)) * Bom + fabs(xj) / (om * s) * Bxj;
      bnd = 4.0 * b;
      valid = true;
    };
    auto f32_eval = [&]() {
      valid = false;
      const bool wg = need_mv, wj = need_dp;  // gamma (births, shifts), e_j (deaths, shifts)
      const int jz = move == 3 ? j : -1;
      double d = 0.0;
      if (wg) {
        for (int i = lane; i < N; i += LPC) s2[i] = (i == jz) ? 0.0 : overlap(md, vt, ov, gnew, zg[i], Lw);
        d = overlap(md, vt, ov, gnew, gnew, Lw) + md.rho;
        beta = mf[gnew - glo] + md.rhom;
      }
      WAVE_SYNC();
      // pass 1 over H: eta = H gamma, h = row j; gamma^T eta, gamma^T x
      LaneSum<SPLIT> sqa, spa;
      for (int i = lane; i < N; i += LPC) {
        if (wg) {
          const double e = grp_col_dot<LD, HS>(H, s2, i, N);
          s3[i] = e;
          sqa.mac(s2[i], e);
          spa.mac(s2[i], xv[i]);
        }
        if (wj) s1[i] = (double)H[(j * LD + i) * HS];
      }
      double qa = 0.0, pa = 0.0;
      if (wg) {
        qa = sqa.template sum<LPC>();
        pa = spa.template sum<LPC>();
      }
      WAVE_SYNC();
      // the residuals against G: r_eta = gamma - G eta (s5), r_h = e_j - G h (s4), s = b - G x (s6)
      gram_resid3<LPC, LD, HS>(Gm, N, lane, s2, wg ? s3 : nullptr, j, wj ? s1 : nullptr, bv, xv, s5, s4, s6);
      WAVE_SYNC();
      double eta_j = 0.0, h_j = 0.0, x_j = 0.0;
      if (wj) {
        eta_j = wg ? s3[j] : 0.0;
        h_j = s1[j];
        x_j = xv[j];
      }
      // first correction terms
      LaneSum<SPLIT> sqb, spb, sjb, sob, sxb;
      for (int i = lane; i < N; i += LPC) {
        if (wg) {
          sqb.mac(s3[i], s5[i]);
          spb.mac(s3[i], s6[i]);
        }
        if (wj) {
          if (wg) sjb.mac(s1[i], s5[i]);
          sob.mac(s1[i], s4[i]);
          sxb.mac(s1[i], s6[i]);
        }
      }
      double qb = 0.0, pb = 0.0, jb = 0.0, ob = 0.0, xb = 0.0;
      if (wg) {
        qb = sqb.template sum<LPC>();
        pb = spb.template sum<LPC>();
      }
      if (wj) {
        if (wg) jb = sjb.template sum<LPC>();
        ob = sob.template sum<LPC>();
        xb = sxb.template sum<LPC>();
      }
      // pass 2 over H: H r_eta, H r_h; the second terms, then eta and h corrected in place
      LaneSum<SPLIT> sqc, spc, sjc, soc, sxc;
      for (int i = lane; i < N; i += LPC) {
        double te = 0.0, th = 0.0;
        if (wg) {
          te = grp_col_dot<LD, HS>(H, s5, i, N);
          sqc.mac(s5[i], te);
          spc.mac(te, s6[i]);
        }
        if (wj) {
          th = grp_col_dot<LD, HS>(H, s4, i, N);
          if (wg) sjc.mac(s4[i], te);
          soc.mac(s4[i], th);
          sxc.mac(th, s6[i]);
        }
        if (wg) s3[i] += te;
        if (wj) s1[i] += th;
      }
      double Qgg = 0.0, Pg = 0.0, Qjg = 0.0, Bgg = 0.0, Bp = 0.0, Bjg = 0.0, Bom = 0.0, Bxj = 0.0;
      if (wg) {
        const double qc = sqc.template sum<LPC>(), pc = spc.template sum<LPC>();
        Qgg = qa + qb + qc;
        Pg = pa + pb + pc;
        Bgg = fabs(qc);
        Bp = fabs(pc);
      }
      if (wj) {
        const double jc = wg ? sjc.template sum<LPC>() : 0.0;
        const double oc = soc.template sum<LPC>(), xc = sxc.template sum<LPC>();
        om = h_j + ob + oc;
        xj = x_j + xb + xc;
        Qjg = eta_j + jb + jc;
        Bom = fabs(oc);
        Bxj = fabs(xc);
        Bjg = fabs(jc);
        if (!(om > 0.0) || !(Bom < 0.1 * om)) {
          inexact = true;
          return;
        }
      }
      WAVE_SYNC();
      double Bq = Bgg;
      if (move == 1) {
        delta2 = d - Qgg;
        up = beta - Pg;
      } else if (move == 3) {
        const double cj = Qjg / om, cx = xj / om;
        delta2 = d - (Qgg - Qjg * cj);
        up = beta - (Pg - Qjg * cx);
        Bq = Bgg + 2.0 * fabs(cj) * Bjg + cj * cj * Bom;
        Bp = Bp + fabs(cx) * Bjg + fabs(cj) * Bxj + fabs(cj * cx) * Bom;
        // v = eta - u Qjg / omega on the PEs without j
        for (int i = lane; i < N; i += LPC) s3[i] = (i == j) ? 0.0 : s3[i] - s1[i] * cj;
        WAVE_SYNC();
      }
      if (move != 2 && (!(delta2 > 0.0) || !(Bq < 0.1 * delta2))) {
        inexact = true;
        return;
      }
      f32_dnu(Bom, Bxj, Bq, Bp);
    };
    // the same proposal from the FP64 rebuild W (exact to FP64 rounding), vectors as above
    auto f64_eval_W = [&]() {
      valid = false;
      if (need_dp) {
        for (int i = lane; i < N; i += LPC) s1[i] = W[(j * LD + i) * HS];
        WAVE_SYNC();
        om = s1[j];
        xj = xv[j];
      }
      if (need_mv) {
        const int jz = move == 3 ? j : -1;
        for (int i = lane; i < N; i += LPC) s2[i] = (i == jz) ? 0.0 : overlap(md, vt, ov, gnew, zg[i], Lw);
        const double d = overlap(md, vt, ov, gnew, gnew, Lw) + md.rho;
        beta = mf[gnew - glo] + md.rhom;
        WAVE_SYNC();
        LaneSum<SPLIT> sq, sp;
        for (int i = lane; i < N; i += LPC) {
          const double e = grp_col_dot<LD, HS>(W, s2, i, N);
          s3[i] = e;
          sq.mac(s2[i], e);
          sp.mac(s2[i], xv[i]);
        }
        double q = sq.template sum<LPC>(), p = sp.template sum<LPC>();
        if (move == 3) {
          WAVE_SYNC();
          const double e = s3[j];
          q -= e * e / om;
          p -= e * xj / om;
          WAVE_SYNC();
          for (int i = lane; i < N; i += LPC) s3[i] = (i == j) ? 0.0 : s3[i] - s1[i] * e / om;
          WAVE_SYNC();
        }
        delta2 = d - q;
        up = beta - p;
      }
      if ((move != 1 && !(om > 0.0)) || (move != 2 && !(delta2 > 0.0))) {
        st |= FSMP_ST_FACTOR;
        return;
      }
      f32_dnu(0.0, 0.0, 0.0, 0.0);
      bnd = 0.0;
    };

    const double logu = lg6;
    if constexpr (F32) {
      if (need_mv || need_dp) {
        f32_eval();
        // an estimate above the tolerance, or a decision the error could turn: decide with
        // the FP64 rebuild
        if (inexact || (valid && (bnd > kF32Tol * fmax(1.0, fabs(dnu)) || fabs(logu - la) <= bnd))) {
          double drift;
          if (N == 0 || grp_refresh<LPC, LD, HS, SPLIT>(md, vt, ov, Lw, W, H, xv, bv, s1, s2, zg, N, lane, drift)) {
            f64_eval_W();
          } else {
            valid = false;
            st |= FSMP_ST_FACTOR;
          }
          if (lane == 0) acc[19] += 1.0;
        } else if (!valid) {
          st |= FSMP_ST_FACTOR;
        }
        if (lane == 0) acc[17] += (double)N * N * (need_dp ? 1.0 : 0.0) + (double)N * N * (need_mv ? 2.0 : 0.0) +
                                  (need_dp ? (double)N : 0.0);
      }
    } else if (need_mv) {
      // (the corrected form also reads row j of H for a shift's x_j)
      if (lane == 0) acc[17] += (double)N * N + (CORR && move == 3 ? (double)N : 0.0);
      eval_mv(H);
    } else if (move == 2 && valid && lane == 0) {
      acc[17] += CORR ? (double)N : 1.0;
    }
    // the word count of the proposal in a packed Cholesky factor: birth K(K+1)/2 +
    // 2K + 3, death (K - j)(K - j + 1)/2 + 1, update both (the birth on K - 1 PEs)
    if (lane == 0 && (valid || need_mv || need_dp)) {
      const double K = N, r = N - j;
      const double wb = move == 1 ? K * (K + 1) / 2 + 2 * K + 3 : (K - 1) * K / 2 + 2 * (K - 1) + 3;
      const double wd = r * (r + 1) / 2 + 1;
      acc[15] += move == 1 ? wb : move == 2 ? wd : (need_mv ? wd + wb : 0.0);
    }

    bool accepted = false;
    if (valid && (FORCE ? (rec.flags & 2) != 0 : logu < la)) {
      accepted = true;
      if (lane == 0) cnt[2 * move + 1]++;
      WAVE_SYNC();
      // an accepted zero shift changes nothing (unless it changes the PE's component)
      const bool shift = move == 3 && (sh != 0 || (MCP && enew != ek[j]));
      if (lane == 0) {
        // the word count of the edit in a packed Cholesky factor: birth K + 3, death
        // (K - 1 - j)(K - j) + K(K + 1)/2, update both; and the G^-1 elements this kernel reads
        // and writes in its rank-one or rank-two edit
        const double K = N, r = N - j;
        const double eb = move == 1 ? K + 3 : (K - 1) + 3, ed = (r - 1) * r + K * (K + 1) / 2;
        acc[16] += move == 1 ? eb : move == 2 ? ed : (shift ? ed + eb : 0.0);
        if (move != 3 || shift) acc[18] += 2.0 * K * K;
      }
      if (move != 3 || shift) {
        const double inv_d2 = move == 2 ? 0.0 : 1.0 / delta2;
        const double inv_om = move == 1 ? 0.0 : 1.0 / om;
        const double xn = up * inv_d2;
        const int gj = move == 1 ? -1 : zg[j];
        // the FP32 form has its corrected vectors at hand: u (column j of G^-1) in s1, eta or v
        // in s3
        if constexpr (!F32) {
          if (move != 1) {
            for (int i = lane; i < N; i += LPC) s1[i] = H[(j * LD + i) * HS];  // h = row j of H
            WAVE_SYNC();
          }
          if (shift) {
            for (int i = lane; i < N; i += LPC) s2[i] = (i == j) ? 0.0 : s2[i] - s1[i] * ej * inv_om;
            WAVE_SYNC();
          }
        }
        double *EV = F32 ? s3 : s2;  // eta (birth) or v (shift)
        // H(k, i) += cu u_i u_k + cv v_i v_k for i, k < N:
        //   birth: u = eta, cu = 1/delta^2; death: u = h, cu = -1/omega;
        //   shift: u = h, cu = -1/omega, and v = eta (zero at j), cv = 1/delta^2
        const double *U = move == 1 ? EV : s1;
        const double *V = shift ? EV : U;
        const double cu = move == 1 ? inv_d2 : -inv_om, cv = shift ? inv_d2 : 0.0;
        const double xe = CORR ? xjp : xj;
        for (int i = lane; i < N; i += LPC) {
          const double ui = U[i], vi = V[i];
          if (move == 1) xv[i] -= ui * xn;
          else if (move == 2) xv[i] -= ui * xe * inv_om;
          else xv[i] = (i == j) ? xn : xv[i] - ui * xe * inv_om - vi * xn;
          grp_col_update<LD, HS, true>(H, i, N, ui, U, cu, vi, V, cv);
          if (move == 1) {
            H[(N * LD + i) * HS] = -ui * inv_d2;
            H[(i * LD + N) * HS] = -ui * inv_d2;
          }
        }
        WAVE_SYNC();
        // the exact G follows the list: the new PE's row and column, or the last PE's moved
        // into a freed slot (s2 is free once the edit is done)
        if constexpr (KEEPG) {
          if (move == 1) {
            gram_set<LPC, LD, HS>(md, vt, ov, Lw, Gm, zg, N, N, gnew, rn, lane);
          } else if (move == 3) {
            gram_set<LPC, LD, HS>(md, vt, ov, Lw, Gm, zg, N, j, gnew, rn, lane);
          } else if (j != N - 1) {
            const int last = N - 1;
            for (int i = lane; i < N; i += LPC) s2[i] = Gm[(last * LD + i) * HS];
            WAVE_SYNC();
            const double gd = s2[last];
            for (int i = lane; i < N; i += LPC) {
              if (i == j) {
                Gm[(j * LD + j) * HS] = gd;
              } else {
                Gm[(j * LD + i) * HS] = s2[i];
                Gm[(i * LD + j) * HS] = s2[i];
              }
            }
          }
        }
        if (move == 1) {
          if (lane == 0) {
            H[(N * LD + N) * HS] = inv_d2;
            zg[N] = gnew;
            if constexpr (MCP) ek[N] = enew;
            xv[N] = xn;
            if (KEEPG) bv[N] = beta;
          }
          N++;
          gmin = gnew < gmin ? gnew : gmin;
        } else if (move == 2) {
          const int last = N - 1;
          if (j != last) {
            for (int i = lane; i < N; i += LPC) s1[i] = H[(last * LD + i) * HS];
            WAVE_SYNC();
            const double vd = s1[last];
            for (int i = lane; i < N; i += LPC) {
              if (i == j) {
                H[(j * LD + j) * HS] = vd;
              } else {
                H[(j * LD + i) * HS] = s1[i];
                H[(i * LD + j) * HS] = s1[i];
              }
            }
            if (lane == 0) {
              zg[j] = zg[last];
              if constexpr (MCP) ek[j] = ek[last];
              xv[j] = xv[last];
              if (KEEPG) bv[j] = bv[last];
            }
          }
          N--;
        } else {
          for (int i = lane; i < N; i += LPC) {
            if (i == j) {
              H[(j * LD + j) * HS] = inv_d2;
            } else {
              const double v = -EV[i] * inv_d2;
              H[(j * LD + i) * HS] = v;
              H[(i * LD + j) * HS] = v;
            }
          }
          if (lane == 0) {
            zg[j] = gnew;
            if constexpr (MCP) ek[j] = enew;
            if (KEEPG) bv[j] = beta;
          }
        }
        WAVE_SYNC();
        // the corrected FP64 form: the residual of the new x against the new G
        if constexpr (CORR) {
          gram_resid_b<LPC, LD, HS>(Gm, bv, xv, rs, N, lane);
          if (lane == 0) acc[18] += (double)N * N;
          WAVE_SYNC();
        }
        if (move != 1) {
          if (move == 3 && gnew < gmin) {
            gmin = gnew;
          } else if (gj == gmin) {
            int m = INT32_MAX;
            for (int i = lane; i < N; i += LPC) m = zg[i] < m ? zg[i] : m;
            gmin = group_min<LPC>(m);
          }
        }
        if (lane == 0) occ_edit(a, c, move, gj, gnew, step, burn, n_steps);
      }
    }

    if (a.log && lane == 0) {
      fsmp_logrec *lr = a.log + c * (int64_t)a.n_steps + step;
      lr->move = move;
      lr->flags = (valid ? 1 : 0) | (accepted ? 2 : 0) | (t0acc ? 4 : 0);
      lr->j = j;
      lr->g = gnew;
      lr->t0 = t0;
      lr->dnu = valid ? dnu : 0.0;
      lr->log_alpha = valid ? la : -INFINITY;
    }
    if (FORCE && lane == 0) {
      a.rdnu[c * (int64_t)a.n_steps + step] = valid ? dnu : 0.0;
      a.rla[c * (int64_t)a.n_steps + step] = valid ? la : -INFINITY;
    }

    // ---- record after burn-in
    if (step >= burn) {
      LaneSum<SPLIT> sQ;
      for (int i = lane; i < N; i += LPC) sQ.term(xv[i]);
      const double Q = sQ.template sum<LPC>();
      const double v0 = (double)N, v1 = Q, v2 = t0;
      const int64_t i = step - burn;
      if (lane == 0) {
        acc[0] += v0;
        acc[1] += v0 * v0;
        acc[2] += v1;
        acc[3] += v1 * v1;
        acc[4] += v2;
        acc[5] += v2 * v2;
        if (nb > 0 && i < (int64_t)nb * lb) {
          acc[12] += v0;
          acc[13] += v1;
          acc[14] += v2;
          if ((i + 1) % lb == 0) {
            acc[6] += acc[12];
            acc[7] += acc[12] * acc[12];
            acc[8] += acc[13];
            acc[9] += acc[13] * acc[13];
            acc[10] += acc[14];
            acc[11] += acc[14] * acc[14];
            acc[12] = acc[13] = acc[14] = 0.0;
          }
        }
        if (N != run[0]) {
          if (run[0] >= 0) atomicAdd(a.nhist + c * (a.kz + 1) + run[0], step - run[1]);
          run[0] = N;
          run[1] = step;
        }
      }
      if (a.trace && a.thin > 0 && (i % a.thin) == 0 && lane == 0) {
        double *tr = a.trace + (c * a.n_rec + i / a.thin) * 3;
        tr[0] = v0;
        tr[1] = v2;
        tr[2] = v1;
      }
      if (a.qdraw && a.thin > 0 && (i % a.thin) == 0) {
        // charge draw q = x + sigma_eps R xi, H = R R^T with R upper triangular: the
        // factorisation runs from the last PE backwards on a copy of H's lower triangle
        // in the chain's device-memory scratch; y = R xi accumulates column by column.  The
        // FP32 form draws from its FP64 rebuild W (and the x it recomputes).
        const int64_t rec = c * a.n_rec + i / a.thin;
        double *Ad = a.dscr + slot * (int64_t)(KCAP * KCAP + KCAP);
        double *Av = Ad + KCAP * KCAP;  // the column being eliminated
        WAVE_SYNC();
        bool ok = true;
        if constexpr (F32) {
          double drift;
          if (N > 0 && !grp_refresh<LPC, LD, HS, SPLIT>(md, vt, ov, Lw, W, H, xv, bv, s1, s2, zg, N, lane, drift)) ok = false;
        }
        for (int r = lane; r < N; r += LPC) {
          for (int k = 0; k <= r; ++k) {
            if constexpr (F32) Ad[r * KCAP + k] = W[(k * LD + r) * HS];
            else Ad[r * KCAP + k] = H[(k * LD + r) * HS];
          }
          s1[r] = charge_normal(step, r, uid0, uid1, a.key0, a.key1);
          s2[r] = 0.0;
        }
        WAVE_SYNC();
        for (int jj = N - 1; jj >= 0 && ok; --jj) {
          const double ajj = Ad[jj * KCAP + jj];
          if (!(ajj > 0.0)) {
            ok = false;
            break;
          }
          const double d = sqrt(ajj), xij = s1[jj];
          for (int r = lane; r < jj; r += LPC) {
            const double v = Ad[jj * KCAP + r] / d;
            Av[r] = v;
            s2[r] += v * xij;
          }
          if (lane == 0) s2[jj] += d * xij;
          WAVE_SYNC();
          for (int r = lane; r < jj; r += LPC) {
            const double vr = Av[r];
            for (int k = 0; k <= r; ++k) Ad[r * KCAP + k] -= vr * Av[k];
          }
          WAVE_SYNC();
        }
        if (!ok) st |= FSMP_ST_FACTOR;
        for (int r = lane; r < a.kz; r += LPC) {
          a.zdraw[rec * a.kz + r] = r < N ? zg[r] : -1;
          a.qdraw[rec * a.kz + r] = r < N ? (ok ? xv[r] + a.sigma_eps * s2[r] : NAN) : 0.0;
        }
        WAVE_SYNC();
      }
    }
  }

  WAVE_SYNC();
  const int kz = a.kz;
  for (int k = lane; k < kz; k += LPC) {
    a.z[c * kz + k] = k < N ? zg[k] : -1;
    a.charge[c * kz + k] = k < N ? xv[k] : 0.0;
    if (MCP && a.comp) a.comp[c * kz + k] = k < N ? ek[k] : -1;
  }
  if (lane == 0 && run[0] >= 0) atomicAdd(a.nhist + c * (a.kz + 1) + run[0], n_steps - run[1]);
  if (lane == 0) {
    a.n_pe[c] = N;
    a.t0[c] = t0;
    if (a.rec_steps) a.rec_steps[c] = S_rec;
    for (int i = 0; i < 12; ++i) a.acc[c * 12 + i] = acc[i];
    for (int i = 0; i < 8; ++i) a.counts[c * 8 + i] = cnt[i];
    a.status[c] = st;
    if (a.work) {
      for (int i = 0; i < 5; ++i) a.work[c * 5 + i] = acc[15 + i];
    }
  }
}


// ------------------------------------------------------------------ chains, G^-1 in LDS
// The LDS design: one chain per group of LPC lanes, each lane one element of the vectors (a
// whole wavefront at capacities 48 and 64, a workgroup of two or three above), with G^-1, the
// vectors and the PE list in LDS.  A sweep of the device-memory groups waits for
// 10-40 dependent memory round trips (the columns of G^-1 in chunks, then their edits); here an
// element costs an LDS read, and no more chains than the LDS holds are in flight, so this is the
// design for batches that do not fill the chip with the other ones: a sweep's latency, not the
// chip's throughput, then sets the time.
//
// Capacities up to 64 keep G^-1 full.  From 96 up the symmetric matrix is kept once, by wrapped
// diagonals: row d (0 .. KCAP / 2) holds the elements (i, (i + d) mod KCAP) at column i, so that
// consecutive lanes read consecutive words whichever triangle an element is in (a packed
// triangle would scatter them over the banks); the last row holds every element twice.  That
// halves the LDS a chain takes (the chains in flight) and the words an edit writes.
//
// Elements at and past N of the vectors are kept zero and the matrices start zeroed, so products
// run over whole chunks without selects.
//
// CORR, the corrected FP64 form (capacities from 48 up, see ChainLayout), keeps its exact G in
// device memory and reads it once per accepted move, for the residual.  (Taking its elements
// from the overlap table in LDS instead was slower: 27.7 -> 36.5 ms for 873 chains of 500 sweeps
// at capacity 128; the lanes' gathers conflict.)
//
// MCP: the Gaussian-mixture charge law, every PE with its component (el).
template <int KCAP, int LPC, bool CORR, bool MCP>
struct LdsLayout {
  static constexpr bool kSym = KCAP >= 96;
  static constexpr int kW = LPC > kWave ? LPC / kWave : 1;  // wavefronts of a chain
  static constexpr int kMat = kSym ? (KCAP / 2 + 1) * KCAP : KCAP * KCAP;
  static constexpr int kVec = kSym ? 2 * KCAP : KCAP;  // the two scratch vectors (twice in a row when wrapped)
  // Lanes over which a vector's sums are taken: element i belongs to lane i mod kRO, which adds its
  // elements in order before the butterfly over the kRO lanes.  Every wavefront of a chain forms
  // the whole sum so, from LDS (no exchange of partial sums).  Up to capacity 64 these are the
  // orders of the narrow device-memory groups, whose chains this design repeats bit for bit
  // there (products and edits too are taken in the same order and rounding): a chain's result
  // does not depend on which of the two its launch is given.
  static constexpr int kRO = KCAP <= 32 ? 4 : KCAP == 48 ? 16 : 32;
  // matrix, two scratch vectors, x (b and the residual too in the corrected form), the PE list (and
  // the components).  With the logs a workgroup takes 10 KB at 16 (four chains), 18 at 32 (two), 21 at 48,
  // 36 at 64, 44 at 96 (three on a CU), 75 at 128 (two), 115 at 160 and 162 at 192 (one), and the rise
  // table beside it, which has no room at 192: every PE takes an expm1 in a t0 step there.
  static constexpr int kDoubles = kMat + 2 * kVec + (CORR ? 3 : 1) * KCAP + (KCAP + 1) / 2 * (MCP ? 2 : 1);
};

// the overlap of two columns, as overlap(), with the window-edge sums from the table of partial
// sums ovp where the model has one (else from the response in device memory)
__device__ inline double overlap_edge(const ModelDev &md, const double *vtab, const double *ov, int g1, int g2,
                                      int Lw) {
  const int lo = g1 < g2 ? g1 : g2, hi = g1 < g2 ? g2 : g1;
  const int d = hi - lo;
  if (d >= md.M) return 0.0;
  const int nhi = sub_div(md, lo + md.M - 1);  // last sample of the earlier column
  const int p = sub_mod(md, lo);
  if (nhi < Lw) return ov[p * md.M + d];
  const int n0 = sub_div(md, hi + md.sub - 1);
  if (md.ovp) {
    const int m = Lw - n0;
    return m > 0 ? md.ovp[((int64_t)p * md.M + d) * (md.LV + 1) + m] : 0.0;
  }
  double s = 0.0;
  for (int n = n0; n < Lw; ++n) s += vtab[md.sub * n - lo] * vtab[md.sub * n - hi];
  return s;
}

// partial sums of the stationary overlaps, [sub][M][LV + 1]: entry m sums the first m samples
// that both columns see (in increasing order, as the direct sum)
__global__ void __launch_bounds__(64) overlap_partial_kernel(const double *vtab_g, double *out, int sub, int M, int LV) {
  extern __shared__ double smem[];
  double *vtab = smem;
  for (int i = threadIdx.x; i < M; i += blockDim.x) vtab[i] = vtab_g[i];
  __syncthreads();
  const int t = blockIdx.x * 64 + threadIdx.x;
  if (t >= sub * M) return;
  const int p = t / M, d = t % M;
  const int n0 = (p + d + sub - 1) / sub, n1 = (p + M - 1) / sub;
  double *row = out + (int64_t)t * (LV + 1);
  double s = 0.0;
  row[0] = 0.0;
  for (int m = 1; m <= LV; ++m) {
    const int n = n0 + m - 1;
    if (n <= n1) s += vtab[sub * n - p] * vtab[sub * n - (p + d)];
    row[m] = s;
  }
}

// element (a, b) of the matrix at D
template <int KCAP, bool SYM>
__device__ inline int lds_at(int a, int b) {
  if constexpr (SYM) {
    int d = b - a;
    d = d < 0 ? d + KCAP : d;
    return d <= KCAP / 2 ? d * KCAP + a : (KCAP - d) * KCAP + b;
  } else {
    return a * KCAP + b;
  }
}
template <int KCAP, bool SYM>
__device__ inline void lds_set(double *D, int a, int b, double v) {
  if constexpr (SYM) {
    D[lds_at<KCAP, true>(a, b)] = v;
    const int d = b - a;
    if (d == KCAP / 2 || d == -KCAP / 2) D[KCAP / 2 * KCAP + b] = v;
    if (d == KCAP / 2 || d == -KCAP / 2) D[KCAP / 2 * KCAP + a] = v;
  } else {
    D[a * KCAP + b] = v;
    D[b * KCAP + a] = v;
  }
}

// element i of a scratch vector (both copies when wrapped)
template <int KCAP, bool SYM>
__device__ inline void lds_vec(double *v, int i, double x) {
  v[i] = x;
  if constexpr (SYM) v[i + KCAP] = x;
}

// element i (< KCAP) of H v for the leading N x N block; v zero from N on
template <int KCAP, bool SYM>
__device__ inline double lds_dot(const double *D, const double *v, int i, int N) {
  double e = 0.0;
  if constexpr (SYM) {
    const int dm = N - 1 < KCAP / 2 - 1 ? N - 1 : KCAP / 2 - 1;
    e = D[i] * v[i];  // the diagonal; then the two triangles, each a chain of its own
    double e1 = 0.0;
    for (int d0 = 0; d0 <= dm; d0 += 8) {
      double h0[8], h1[8], v0[8], v1[8];
#pragma unroll
      for (int u = 0; u < 8; ++u) {
        const int d = d0 + u;
        h0[u] = D[d * KCAP + i];
        v0[u] = v[i + d];
        h1[u] = D[d * KCAP + i - d + (d > i ? KCAP : 0)];
        v1[u] = v[i - d + KCAP];
      }
#pragma unroll
      for (int u = 0; u < 8; ++u) {
        if (u > 0) e = fma(h0[u], v0[u], e);
        else e = d0 > 0 ? fma(h0[u], v0[u], e) : e;
        if (u > 0) e1 = fma(h1[u], v1[u], e1);
        else e1 = d0 > 0 ? fma(h1[u], v1[u], e1) : e1;
      }
    }
    e += e1;
    if (N > KCAP / 2) e = fma(D[KCAP / 2 * KCAP + i], v[i + KCAP / 2], e);
  } else {
    for (int k0 = 0; k0 < N; k0 += 8) {
      double h[8], g[8];
#pragma unroll
      for (int u = 0; u < 8; ++u) {
        h[u] = D[(k0 + u) * KCAP + i];
        g[u] = v[k0 + u];
      }
#pragma unroll
      for (int u = 0; u < 8; ++u) e = fma(h[u], g[u], e);
    }
  }
  return e;
}

// one element of an edit by one vector, or by two, or of the step of a list's build
template <bool TWO, bool BUILD>
__device__ inline double lds_edited(double h, double ui, double uk, double cu, double vi, double vk, double cv,
                                    bool first) {
  if constexpr (BUILD) return edit_build(h, ui, uk, cu);
  else if constexpr (TWO) return edit_two(h, ui, uk, cu, vi, vk, cv, first);
  else return edit_one(h, ui, uk, cu);
}

// H += cu u u^T [+ cv v v^T], element i's share (i < N; u, v zero from N on)
template <int KCAP, bool SYM, bool TWO, bool BUILD>
__device__ inline void lds_edit(double *D, const double *u, const double *v, double ui, double cu, double vi,
                                double cv, int i, int N) {
  if constexpr (SYM) {
    const int dm = N - 1 < KCAP / 2 - 1 ? N - 1 : KCAP / 2 - 1;
    for (int d0 = 0; d0 <= dm; d0 += 8) {
      double h[8], a[8], b[8];
#pragma unroll
      for (int q = 0; q < 8; ++q) {
        h[q] = D[(d0 + q) * KCAP + i];
        a[q] = u[i + d0 + q];
        b[q] = TWO ? v[i + d0 + q] : 0.0;
      }
#pragma unroll
      for (int q = 0; q < 8; ++q)
        D[(d0 + q) * KCAP + i] = lds_edited<TWO, BUILD>(h[q], ui, a[q], cu, vi, b[q], cv, q == 0);
    }
    if (N > KCAP / 2) {
      double *e = D + KCAP / 2 * KCAP + i;
      *e = lds_edited<TWO, BUILD>(*e, ui, u[i + KCAP / 2], cu, vi, TWO ? v[i + KCAP / 2] : 0.0, cv, false);
    }
  } else {
    for (int k0 = 0; k0 < N; k0 += 8) {
      double h[8], a[8], b[8];
#pragma unroll
      for (int q = 0; q < 8; ++q) {
        h[q] = D[(k0 + q) * KCAP + i];
        a[q] = u[k0 + q];
        b[q] = TWO ? v[k0 + q] : 0.0;
      }
#pragma unroll
      for (int q = 0; q < 8; ++q)
        D[(k0 + q) * KCAP + i] = lds_edited<TWO, BUILD>(h[q], ui, a[q], cu, vi, b[q], cv, q == 0);
    }
  }
}

// a value that is the same in the lanes of a chain's group, as a scalar where the group is a
// whole wavefront (branches on it then are scalar branches)
template <int LPC>
__device__ inline int group_uniform(int v) {
  if constexpr (LPC >= kWave) return __builtin_amdgcn_readfirstlane(v);
  else return v;
}

// LDS written by a chain's lanes becomes visible to all of them (one wavefront or less: the LDS
// runs its instructions in order; several: a barrier that waits for LDS traffic only, so that
// loads from device memory stay in flight across it)
template <int LPC>
__device__ inline void chain_sync() {
  if constexpr (LPC > kWave) {
#if defined(__AMDGCN__)
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
#else
    __syncthreads();
#endif
  } else {
    WAVE_SYNC();
  }
}

// the same for device memory too
template <int LPC>
__device__ inline void chain_sync_mem() {
  if constexpr (LPC > kWave) __syncthreads();
  else WAVE_SYNC();
}

// Sum over a chain's elements of f(i, sum so far): lane i mod RO adds its elements in order, then
// the butterfly over RO lanes; every wavefront of the chain forms it from LDS
template <int KCAP, int RO, typename F>
__device__ inline double chain_sum(int gl, F f) {
  double t = 0.0;
#pragma unroll
  for (int q = 0; q < KCAP / RO; ++q) t = f((gl & (RO - 1)) + q * RO, t);
  return group_sum<RO>(t);
}

// G^-1 of the PE list zl[0..N) by bordering into the (finite) matrix D, each step the birth
// update of the inverse of the leading block; va, vb: the scratch vectors.  False if a Schur
// complement is not positive.  el: the PEs' mixture components, or null.
template <int KCAP, int LPC, bool SYM, int RO>
__device__ bool lds_build(const ModelDev &md, const double *vtab, const double *ov, int Lw, double *D, double *va,
                          double *vb, const int *zl, int N, int lane, int gl, const int *el) {
  const bool own = KCAP % LPC == 0 || lane < KCAP;  // a lane with an element
  for (int k = 0; k < N; ++k) {
    const int gk = zl[k];
    chain_sync<LPC>();
    if (own) lds_vec<KCAP, SYM>(va, lane, lane < k ? overlap_edge(md, vtab, ov, gk, zl[lane], Lw) : 0.0);
    const double d = overlap_edge(md, vtab, ov, gk, gk, Lw) + (el ? md.mix_rho[el[k]] : md.rho);
    chain_sync<LPC>();
    const double e = lane < k ? lds_dot<KCAP, SYM>(D, va, lane, k) : 0.0;
    if (own) lds_vec<KCAP, SYM>(vb, lane, e);
    chain_sync<LPC>();
    const double q = chain_sum<KCAP, RO>(gl, [&](int i, double t) { return fma(va[i], vb[i], t); });
    const double delta2 = d - q;
    if (!(delta2 > 0.0)) return false;
    const double inv = 1.0 / delta2;
    if (lane < k) lds_edit<KCAP, SYM, false, true>(D, vb, vb, e, inv, 0.0, 0.0, lane, k);
    chain_sync<LPC>();
    if (lane < k) lds_set<KCAP, SYM>(D, k, lane, -e * inv);
    if (lane == 0) lds_set<KCAP, SYM>(D, k, k, inv);
    chain_sync<LPC>();
  }
  return true;
}

// The Gibbs / RJMCMC chains of chain_kernel (the same moves, acceptances and random numbers;
// FP64) with G^-1 in LDS.
// bk: the launch's chains; block: the workgroup's index among theirs.
struct LdsBucket {
  const int32_t *chains;
  int64_t n_list;
  double *dws, *dscr;
};
template <int KCAP, int LPC, bool CORR, bool MCP>
__device__ __attribute__((always_inline)) inline void chain_lds_body(const ChainArgs &a, const LdsBucket &bk, int64_t block, double *smem) {
  using CL = LdsLayout<KCAP, LPC, CORR, MCP>;
  constexpr bool SYM = CL::kSym;
  constexpr int RO = CL::kRO;
  constexpr int W = CL::kW, CPW = LPC < kWave ? kWave / LPC : 1;
  static_assert(LPC >= 16 && LPC >= KCAP, "one element of the vectors per lane");
  const ModelDev &md = a.md;
  // A workgroup is one wavefront (or one chain of several), so that chains of every capacity pack
  // into the LDS of a CU side by side; the overlap table stays in device memory (a few reads per
  // sweep, from the caches), only the rise factors and the logs are copied.  (Workgroups of four
  // wavefronts around one copy of the tables filled a CU each: the launches of a call ran one
  // after the other, 10.9 ms for 8,000 windows of the mixture law, 8.9 ms now.)
  double *rt = smem;
  double *lgn = rt + md.rise_n;
  const double *ov = a.ovl;
  for (int i = threadIdx.x; i < md.rise_n; i += blockDim.x) rt[i] = md.rtab[i];
  for (int i = threadIdx.x; i < KCAP + 2; i += blockDim.x) lgn[i] = log((double)i);
  __syncthreads();
  // lane: the index in the chain's group (its element of the vectors); l64 in the wavefront
  // (gl in the part of a wavefront that the group is)
  const int l64 = threadIdx.x % kWave;
  const int grp = LPC < kWave ? l64 / LPC : 0, gbase = grp * LPC;
  const int lane = W > 1 ? (int)threadIdx.x : l64 % LPC, gl = W > 1 ? l64 : lane;
  constexpr int GW = LPC < kWave ? LPC : kWave;  // lanes that share the per-chain scalars' work
  const int64_t slot = block * CPW + grp;
  if (slot >= bk.n_list) return;
  double *D = lgn + (KCAP + 2) + grp * CL::kDoubles;
  double *va = D + CL::kMat, *vb = va + CL::kVec, *xl = vb + CL::kVec;
  double *bl = CORR ? xl + KCAP : nullptr, *sl = CORR ? bl + KCAP : nullptr;
  int *zl = (int *)(xl + (CORR ? 3 : 1) * KCAP);
  int *el = zl + 2 * ((KCAP + 1) / 2);  // (the mixture form's components)
  double *Gm = CORR ? bk.dws + slot * (int64_t)(KCAP * KCAP) : nullptr;

  const int64_t c = bk.chains[slot];
  const int64_t w = c / a.n_chains;
  const int Lw = (int)(a.woff[w + 1] - a.woff[w]);
  const double lam = a.lam[w];
  const int kmax = a.kmax[w];
  const int glo = a.grange[2 * w], ghi = a.grange[2 * w + 1];
  const double *mf = a.mf + a.mfoff[w];
  const uint64_t uid = a.wid[w] * (uint64_t)a.n_chains + (uint64_t)(c % a.n_chains);
  const uint32_t uid0 = (uint32_t)uid, uid1 = (uint32_t)(uid >> 32);
  uint32_t st = a.wflags[w];
  if (glo > ghi) st |= FSMP_ST_EMPTY_T;
  const int steps_w = a.wsteps ? a.wsteps[w] : a.n_steps;
  const int burn = a.wsteps ? (int)((int64_t)steps_w * a.burn_in / a.n_steps) : a.burn_in;
  const int n_steps = (st & FSMP_ST_NONFINITE) ? 0 : steps_w;
  const int S_rec = n_steps > burn ? n_steps - burn : 0;
  const int nb = S_rec > 0 ? (int)floor(sqrt((double)S_rec)) : 0;
  const int lb = nb > 0 ? S_rec / nb : 0;

  for (int k = lane; k <= a.kz; k += LPC) a.nhist[c * (a.kz + 1) + k] = 0;
  for (int k = lane; k < CL::kMat + 2 * CL::kVec + (CORR ? 3 : 1) * KCAP; k += LPC) D[k] = 0.0;
  for (int k = lane; k < KCAP * (MCP ? 2 : 1); k += LPC) zl[k] = 0;
  if constexpr (CORR)
    for (int k = lane; k < KCAP * KCAP; k += LPC) Gm[k] = 0.0;
  chain_sync_mem<LPC>();

  double t0 = a.t0init[w];
  int N = 0;
  // (an empty T has no points at or after t0: Phi is 0)
  T0Terms tc = t0_terms<GW>(md, t0, glo, ghi, gl, gbase);
  t0_phi(md, tc);
  double Lam = lam * md.dt * tc.Phi;
  const bool biexp = md.kind == FSMP_PHI_BIEXP;
  int gmin = INT32_MAX;  // smallest PE grid index
  double Q = 0.0;        // sum of the charge means, changes with accepted moves only

  // After the list has changed: the residual s = b - G x against the exact G (corrected form) and
  // Q.  Rows of G in chunks of RG, the loads of a chunk in flight together (rows and elements
  // past N are zero or meet a zero x; chunks of 32 measured no faster).  From capacity 96 up every kRefine changes x first takes
  // up H s: an edit leaves about kappa eps in x, and without the refinement those add up over the
  // chain (at N ~ 30 the total charge after 600 sweeps is 3.5e-15 off instead of 3.2e-14).
  constexpr int RG = 16;
  constexpr int kRefine = 16;
  int to_refine = kRefine;
  auto residual = [&]() {
    if constexpr (CORR) {
      const double *gp = Gm + (KCAP % LPC && lane >= KCAP ? KCAP - 1 : lane);
      const bool refine = SYM && --to_refine == 0;
      for (int pass = refine ? 0 : 1; pass < 2; ++pass) {
        double r = 0.0;
        for (int k0 = 0; k0 < N; k0 += RG) {
          double g[RG];
#pragma unroll
          for (int u = 0; u < RG; ++u) g[u] = gp[(k0 + u) * KCAP];
#pragma unroll
          for (int u = 0; u < RG; ++u) r = fma(g[u], xl[k0 + u], r);
        }
        const double rs = lane < N ? bl[lane] - r : 0.0;
        if (pass == 0) {
          to_refine = kRefine;
          if (KCAP % LPC == 0 || lane < KCAP) lds_vec<KCAP, SYM>(va, lane, rs);
          chain_sync<LPC>();
          if (lane < N) xl[lane] += lds_dot<KCAP, SYM>(D, va, lane, N);
          chain_sync<LPC>();
        } else if (KCAP % LPC == 0 || lane < KCAP) {
          sl[lane] = rs;
        }
      }
    }
    chain_sync<LPC>();
    Q = chain_sum<KCAP, RO>(gl, [&](int i, double t) { return t + xl[i]; });
  };

  // a caller-supplied initial PE list: G^-1 and x = G^-1 b of the list before the first sweep
  if (a.zinit && n_steps > 0) {
    const int n0 = (int)(a.zinit_off[c + 1] - a.zinit_off[c]);
    if (n0 > 0) {
      const int32_t *z0 = a.zinit + a.zinit_off[c];
      if (lane < n0) zl[lane] = z0[lane];
      chain_sync<LPC>();
      if (lds_build<KCAP, LPC, SYM, RO>(md, a.vtab, ov, Lw, D, va, vb, zl, n0, lane, gl, nullptr)) {
        const double b = lane < n0 ? mf[zl[lane] - glo] + md.rhom : 0.0;
        if (KCAP % LPC == 0 || lane < KCAP) lds_vec<KCAP, SYM>(va, lane, b);
        chain_sync<LPC>();
        if (lane < n0) {
          xl[lane] = lds_dot<KCAP, SYM>(D, va, lane, n0);
          if constexpr (CORR) {
            bl[lane] = b;
            for (int k = 0; k < n0; ++k)
              Gm[k * KCAP + lane] = overlap_edge(md, a.vtab, ov, zl[k], zl[lane], Lw) + (k == lane ? md.rho : 0.0);
          }
          occ_edit(a, c, 1, -1, zl[lane], 0, burn, n_steps);
        }
        N = n0;
        for (int k = 0; k < n0; ++k) gmin = zl[k] < gmin ? zl[k] : gmin;
        chain_sync<LPC>();
        residual();
      } else {
        st |= FSMP_ST_FACTOR;
      }
      chain_sync<LPC>();
    }
  }

  // the accumulators live in the group's first lanes: lanes 0, 1, 2 the sums of N, Q, t0 (sum,
  // sum of squares, open batch sum, sum and sum of squares of the closed ones); lanes 0 .. 3 the
  // proposals and accepts of t0, birth, death, update.  work: the counters, LDS-free, lane 0
  double a_s = 0.0, a_q = 0.0, a_b = 0.0, a_bs = 0.0, a_bq = 0.0;
  int c_p = 0, c_a = 0;
  double wk0 = 0.0, wk1 = 0.0, wk2 = 0.0, wk3 = 0.0;
  int run_n = -1, run_s = 0;  // N of the current run among the recorded steps, its first step
  int b_left = lb, in_batch = nb * lb;
  int ref_left = a.refresh_M;
  uint32_t st_r3 = 0, st_r4 = 0, st_r5 = 0, st_r7 = 0;
  double st_l2 = 0.0, st_l6 = 0.0, st_xt = 0.0, st_xs = 0.0;

  for (int step = 0; step < n_steps; ++step) {
    if constexpr (!CORR) {
      // G^-1 rebuilt and x = G^-1 b recomputed every refresh_M sweeps, against the rounding the
      // edits accumulate (the corrected form needs none)
      if (a.refresh_M > 0) {
        if (ref_left == 0) {
          ref_left = a.refresh_M;
          if (N > 0) {
            if (lds_build<KCAP, LPC, SYM, RO>(md, a.vtab, ov, Lw, D, va, vb, zl, N, lane, gl, MCP ? el : nullptr)) {
              if (KCAP % LPC == 0 || lane < KCAP)
                lds_vec<KCAP, SYM>(va, lane, lane < N ? mf[zl[lane] - glo] + (MCP ? md.mix_rhom[el[lane]] : md.rhom) : 0.0);
              chain_sync<LPC>();
              if (lane < N) xl[lane] = lds_dot<KCAP, SYM>(D, va, lane, N);
              residual();
            } else {
              st |= FSMP_ST_FACTOR;
            }
          }
        }
        --ref_left;
      }
    }
    // ---- random values: every GW sweeps each lane makes those of one of the next GW (both
    // Philox blocks, the three logs, the Box-Muller pair); a sweep reads its own, by lane reads
    // from a wavefront per chain up, else by lane permutes
    const int sl_ = step & (GW - 1);
    if (sl_ == 0) {
      uint32_t q0[4], q1[4];
      philox4x32_10((uint32_t)(step + gl), 0u, uid0, uid1, a.key0, a.key1, q0);
      philox4x32_10((uint32_t)(step + gl), 1u, uid0, uid1, a.key0, a.key1, q1);
      const double R = sqrt(-2.0 * log(u01(q0[0])));
      const double th = 2.0 * M_PI * u01(q0[1]);
      st_xt = R * cos(th);
      st_xs = R * sin(th);
      st_l2 = log(u01(q0[2]));
      st_l6 = log(u01(q1[2]));
      st_r3 = q0[3];
      st_r4 = q1[0];
      st_r5 = q1[1];
      st_r7 = q1[3];
    }
    uint32_t r3, r4, r5, r7 = 0;
    double lg2, lg6, xi_t0, xi_sh;
    if constexpr (LPC >= kWave) {
      r3 = (uint32_t)__builtin_amdgcn_readlane((int)st_r3, sl_);
      r4 = (uint32_t)__builtin_amdgcn_readlane((int)st_r4, sl_);
      r5 = (uint32_t)__builtin_amdgcn_readlane((int)st_r5, sl_);
      if constexpr (MCP) r7 = (uint32_t)__builtin_amdgcn_readlane((int)st_r7, sl_);
      lg2 = lane_value(st_l2, sl_);
      lg6 = lane_value(st_l6, sl_);
      xi_t0 = lane_value(st_xt, sl_);
      xi_sh = lane_value(st_xs, sl_);
    } else {
      const int from = gbase + sl_;
      r3 = (uint32_t)__shfl((int)st_r3, from, kWave);
      r4 = (uint32_t)__shfl((int)st_r4, from, kWave);
      r5 = (uint32_t)__shfl((int)st_r5, from, kWave);
      if constexpr (MCP) r7 = (uint32_t)__shfl((int)st_r7, from, kWave);
      lg2 = __shfl(st_l2, from, kWave);
      lg6 = __shfl(st_l6, from, kWave);
      xi_t0 = __shfl(st_xt, from, kWave);
      xi_sh = __shfl(st_xs, from, kWave);
    }

    // ---- Gibbs half-step 1: t0 by Metropolis-Hastings
    const double t0p = t0 + md.t0_sd * xi_t0;
    bool t0acc = false;
    if (t0p >= md.t0_min && t0p <= md.t0_max) {
      const double xmin = (N > 0) ? (double)gmin * md.dt - t0p : 1.0;
      if (biexp ? (xmin > 0.0) : (xmin >= 0.0)) {
        T0Terms tp = t0_terms<GW>(md, t0p, glo, ghi, gl, gbase);
        double S = 0.0;  // sum over the PEs of log r(t0p) / r(t0), r the rise factor
        if (biexp && N > 0) {
          double pn = 1.0, pc = 1.0;
#pragma unroll
          for (int q = 0; q < (KCAP + GW - 1) / GW; ++q) {
            const int i = gl + q * GW;
            if (i < N) {
              const int g = zl[i];
              pn *= rise_at(md, rt, tp, t0p, g);
              pc *= rise_at(md, rt, tc, t0, g);
            }
          }
          if constexpr (SYM) {
            S = group_sum<GW>(log(pn / pc));
          } else {
            // one log for the PEs that share a lane of the narrow device-memory groups
            S = group_sum<RO>(log(class_product<GW, RO>(pn) / class_product<GW, RO>(pc)));
          }
        }
        t0_phi(md, tp);
        const double part = (double)N * (t0p - t0) * md.inv_tau2 + S;
        const double la0 = part - (lam * md.dt * tp.Phi - lam * md.dt * tc.Phi);
        if (lg2 < la0) {
          t0 = t0p;
          tc = tp;
          Lam = lam * md.dt * tc.Phi;
          t0acc = true;
        }
      }
    }

    // ---- Gibbs half-step 2: one RJMCMC jump
    const double um = u01(r3);
    const int move = group_uniform<LPC>((N == 0 || um < md.J) ? 1 : (um < 2.0 * md.J ? 2 : 3));
    int j = -1, gnew = -1, sh = 0;
    bool valid = false, need_mv = false;
    double dnu = 0.0, la = -INFINITY, lpd = 0.0, pr_sh = 1.0;
    // mixture form: the component of a born or updated PE from word r7 (inverse CDF of the
    // weights); rho, its log, rho mu, rho mu^2 of the new and of the removed / moved PE
    int enew = 0;
    bool same = true;  // an update keeps the PE's component
    double rn = md.rho, lrn = md.log_rho, rmn = md.rhom, rm2n = md.rhom2;
    double lro = md.log_rho, rm2o = md.rhom2;
    if constexpr (MCP) {
      const double ue = u01(r7);
      enew = md.n_mix - 1;
      for (int q = md.n_mix - 2; q >= 0; --q)
        if (ue < md.mix_cdf[q]) enew = q;
      rn = md.mix_rho[enew];
      lrn = md.mix_lrho[enew];
      rmn = md.mix_rhom[enew];
      rm2n = md.mix_rhom2[enew];
    }
    if (move == 1) {
      if (N >= kmax) {
        st |= FSMP_ST_KMAX;
      } else if (tc.Phi > 0.0) {
        gnew = birth_draw<GW>(md, tc, u53(r4, r5) * tc.Phi, gl, grp);
        need_mv = Lam > 0.0;
      }
    } else {
      j = group_uniform<LPC>((int)(((uint64_t)r4 * (uint64_t)N) >> 32));
      if constexpr (MCP) {
        lro = md.mix_lrho[el[j]];
        rm2o = md.mix_rhom2[el[j]];
        same = move != 3 || enew == el[j];
      }
      if (move == 3) {
        const int gj = zl[j];
        sh = (int)rint(xi_sh * md.shift_sd / md.dt);
        gnew = gj + sh;
        const double xnew = (double)gnew * md.dt - t0;
        if (gnew >= glo && gnew <= ghi && (biexp ? xnew > 0.0 : xnew >= 0.0)) {
          if (sh == 0 && same) {
            valid = true;
            la = 0.0;
          } else {
            lpd = (double)(gj - gnew) * md.dt * md.inv_tau2;
            if (biexp && sh != 0) pr_sh = rise_at(md, rt, tc, t0, gnew) / rise_at(md, rt, tc, t0, gj);
            need_mv = true;
          }
        }
      }
    }
    // birth or shift: gamma = overlaps of the new position with the PEs (zero at the shifted one)
    // in va, eta = H gamma; death or shift: h = row j of H
    double eta = 0.0, hj = 0.0;
    double delta2 = 1.0, up = 0.0, om = 1.0, xj = 0.0, xjp = 0.0, ej = 0.0, beta = 0.0;
    double inv_om = 0.0, inv_d2 = 0.0;
    const bool removes = move == 2 || (move == 3 && need_mv);
    double mfv = 0.0, gam = 0.0;
    if (need_mv) {
      mfv = mf[gnew - glo];
      if (lane < N && lane != j) gam = overlap_edge(md, a.vtab, ov, gnew, zl[lane], Lw);
      chain_sync<LPC>();  // (the last proposal's sums are done with va and vb)
      if (KCAP % LPC == 0 || lane < KCAP) lds_vec<KCAP, SYM>(va, lane, gam);
      chain_sync<LPC>();
    }
    if (removes) {
      om = D[lds_at<KCAP, SYM>(j, j)];
      xj = xjp = xl[j];
      if (lane < N) hj = D[lds_at<KCAP, SYM>(j, lane)];
      // (elements of H past N may be left over from removed PEs: they meet a zero of s)
      if constexpr (CORR)
        xj += chain_sum<KCAP, RO>(gl, [&](int i, double t) { return fma(D[lds_at<KCAP, SYM>(j, i)], sl[i], t); });
      inv_om = 1.0 / om;
    }
    if (need_mv) {
      const double d = overlap_edge(md, a.vtab, ov, gnew, gnew, Lw) + rn;
      if (lane < N) eta = lds_dot<KCAP, SYM>(D, va, lane, N);
      double q, p;
      if (KCAP % LPC == 0 || lane < KCAP) vb[lane] = eta;
      chain_sync<LPC>();
      q = chain_sum<KCAP, RO>(gl, [&](int i, double t) { return fma(va[i], vb[i], t); });
      p = chain_sum<KCAP, RO>(gl, [&](int i, double t) { return fma(va[i], xl[i], t); });
      if constexpr (CORR) p += chain_sum<KCAP, RO>(gl, [&](int i, double t) { return fma(vb[i], sl[i], t); });
      if (move == 3) ej = vb[j];
      if (move == 3) {
        q -= ej * ej / om;
        p -= ej * xj / om;
      }
      beta = mfv + rmn;
      delta2 = d - q;
      up = beta - p;
      inv_d2 = 1.0 / delta2;
    }
    if (need_mv || move == 2) {
      if (delta2 > 0.0 && om > 0.0) {
        // birth: log delta^2, log Lambda; death: log omega, log Lambda; shift: log omega, log
        // delta^2 and the log of the rise factors' ratio
        double l0, l1, l2;
        group_log3<GW>(move == 1 ? delta2 : om, move == 3 ? delta2 : Lam, pr_sh, gl, gbase, l0, l1, l2);
        if (move == 1) {
          const double v = -lrn + l0 + (rm2n - ratio(up * up, delta2, inv_d2)) * md.inv_s;
          dnu = -0.5 * v;
          la = fma(-0.5, v, l1) - lgn[N + 1] + (N == 0 ? md.logJ : 0.0);
        } else if (move == 2) {
          const double v = -lro - l0 + (rm2o - ratio(xj * xj, om, inv_om)) * md.inv_s;
          dnu = 0.5 * v;
          la = fma(0.5, v, -l1) + lgn[N] - (N == 1 ? md.logJ : 0.0);
        } else {
          dnu = 0.5 * (-l0 - l1 + (ratio(up * up, delta2, inv_d2) - ratio(xj * xj, om, inv_om)) * md.inv_s);
          // mixture form: the removed and the added PE carry their own rho and rho mu^2
          if constexpr (MCP) dnu += 0.5 * (lrn - lro + (rm2o - rm2n) * md.inv_s);
          la = dnu + (lpd + l2);
        }
        valid = true;
      } else {
        st |= FSMP_ST_FACTOR;
      }
    }
    const bool accepted = group_uniform<LPC>(valid && lg6 < la) != 0;
    const bool edits = accepted && (move != 3 || sh != 0 || !same);
    c_p += (lane == 0) | (lane == move);
    c_a += (lane == 0 && t0acc) | (lane == move && accepted);
    if (a.work) {
      // the word counts in a packed Cholesky factor of the proposal (birth K(K+1)/2 + 2K + 3,
      // death (K - j)(K - j + 1)/2 + 1, update both, the birth on K - 1 PEs) and of the edit (birth
      // K + 3, death (K - 1 - j)(K - j) + K(K + 1)/2, update both); the elements of G^-1 read by the
      // proposal; the elements of G^-1 and G the edit reads and writes
      const double K = N, r = N - j;
      const double wb = move == 1 ? K * (K + 1) / 2 + 2 * K + 3 : (K - 1) * K / 2 + 2 * (K - 1) + 3;
      const double wd = r * (r + 1) / 2 + 1;
      if (valid || need_mv) wk0 += move == 1 ? wb : move == 2 ? wd : (need_mv ? wd + wb : 0.0);
      if (need_mv) wk2 += K * K + (CORR && move == 3 ? K : 0.0);
      else if (move == 2 && valid) wk2 += CORR ? K : 1.0;
      if (edits) {
        const double eb = move == 1 ? K + 3 : (K - 1) + 3, ed = (r - 1) * r + K * (K + 1) / 2;
        wk1 += move == 1 ? eb : move == 2 ? ed : ed + eb;
        const double Kn = move == 1 ? K + 1 : move == 2 ? K - 1 : K;
        wk3 += 2.0 * K * K + (CORR ? Kn * Kn : 0.0);
      }
    }
    if (edits) {
      // H += cu u u^T + cv v v^T: birth u = eta, cu = 1 / delta^2; death u = h, cu = -1 / omega;
      // shift both, v = eta - h ej / omega (zero at j) with cv = 1 / delta^2
      const double xn = up * inv_d2;
      const int gj = move == 1 ? -1 : zl[j];
      const bool two = move == 3;
      const double cu = move == 1 ? inv_d2 : -inv_om, cv = two ? inv_d2 : 0.0;
      const int last = N - 1;
      const double uu = move == 1 ? eta : hj;
      const double vv = two && lane != j ? eta - hj * ej * inv_om : 0.0;
      chain_sync<LPC>();
      if (KCAP % LPC == 0 || lane < KCAP) {
        lds_vec<KCAP, SYM>(va, lane, uu);
        if (two || LPC < kWave) lds_vec<KCAP, SYM>(vb, lane, vv);
      }
      chain_sync<LPC>();
      if (lane < N) {
        // one edit code for the groups that share a wavefront, a shorter one for a single vector
        if (LPC < kWave || two) lds_edit<KCAP, SYM, true, false>(D, va, vb, uu, cu, vv, cv, lane, N);
        else lds_edit<KCAP, SYM, false, false>(D, va, vb, uu, cu, 0.0, 0.0, lane, N);
        const double xe = CORR ? xjp : xj;
        if (move == 1) xl[lane] -= uu * xn;
        else if (move == 2) xl[lane] -= uu * xe * inv_om;
        else xl[lane] = (lane == j) ? xn : xl[lane] - uu * xe * inv_om - vv * xn;
      }
      chain_sync<LPC>();
      if (move != 2) {
        // the new PE's row: -w / delta^2 with w = eta or v, 1 / delta^2 on the diagonal
        const int r = move == 1 ? N : j;
        if (lane < N && lane != r) {
          lds_set<KCAP, SYM>(D, r, lane, -(move == 1 ? uu : vv) * inv_d2);
          if constexpr (CORR) {
            Gm[r * KCAP + lane] = gam;
            Gm[lane * KCAP + r] = gam;
          }
        }
        if (lane == r) {
          lds_set<KCAP, SYM>(D, r, r, inv_d2);
          if (move == 1) xl[r] = xn;
          zl[r] = gnew;
          if constexpr (MCP) el[r] = enew;
          if constexpr (CORR) {
            bl[r] = beta;
            Gm[r * KCAP + r] = overlap_edge(md, a.vtab, ov, gnew, gnew, Lw) + rn;
          }
        }
        if (move == 1) N++;
      } else {
        // the last PE moves into the freed slot
        double hl = 0.0, gv = 0.0, xlast = 0.0, blast = 0.0;
        int zlast = 0;
        if (lane < N) {
          hl = D[lds_at<KCAP, SYM>(last, lane)];
          if constexpr (CORR) gv = Gm[last * KCAP + lane];
        }
        zlast = zl[last];
        const int elast = MCP ? el[last] : 0;
        xlast = xl[last];
        if constexpr (CORR) blast = bl[last];
        chain_sync<LPC>();
        if (j != last) {
          // row `last` in place of row j: its element at j is the one at the diagonal
          const int at = lane == last ? j : lane;
          if (lane < N && lane != j) {
            lds_set<KCAP, SYM>(D, j, at, hl);
            if constexpr (CORR) {
              Gm[j * KCAP + at] = gv;
              Gm[at * KCAP + j] = gv;
            }
          }
          if (lane == j) {
            zl[j] = zlast;
            if constexpr (MCP) el[j] = elast;
            xl[j] = xlast;
            if constexpr (CORR) bl[j] = blast;
          }
        }
        if (lane == last) xl[last] = 0.0;
        N--;
      }
      N = group_uniform<LPC>(N);
      chain_sync_mem<LPC>();  // (the edits of G too)
      residual();
      if (move != 2 && gnew < gmin) {
        gmin = gnew;
      } else if (move != 1 && gj == gmin) {
        gmin = INT32_MAX;
        for (int i = gl; i < N; i += GW) gmin = zl[i] < gmin ? zl[i] : gmin;
        gmin = group_min<GW>(gmin);
      }
      if (lane == 0) occ_edit(a, c, move, gj, gnew, step, burn, n_steps);
    }

    if (a.log && lane == 0) {
      fsmp_logrec *lr = a.log + c * (int64_t)a.n_steps + step;
      lr->move = move;
      lr->flags = (valid ? 1 : 0) | (accepted ? 2 : 0) | (t0acc ? 4 : 0);
      lr->j = j;
      lr->g = gnew;
      lr->t0 = t0;
      lr->dnu = valid ? dnu : 0.0;
      lr->log_alpha = valid ? la : -INFINITY;
    }

    // ---- record after burn-in
    if (step >= burn) {
      const double v = lane == 0 ? (double)N : lane == 1 ? Q : t0;
      a_s += v;
      a_q += v * v;
      if (in_batch > 0) {
        --in_batch;
        a_b += v;
        if (--b_left == 0) {
          b_left = lb;
          a_bs += a_b;
          a_bq += a_b * a_b;
          a_b = 0.0;
        }
      }
      if (N != run_n) {
        if (run_n >= 0 && lane == 0) atomicAdd(a.nhist + c * (a.kz + 1) + run_n, step - run_s);
        run_n = N;
        run_s = step;
      }
      const int i = step - burn;
      if (a.trace && a.thin > 0 && (i % a.thin) == 0 && lane == 0) {
        double *tr = a.trace + (c * a.n_rec + i / a.thin) * 3;
        tr[0] = (double)N;
        tr[1] = t0;
        tr[2] = Q;
      }
      if (a.qdraw && a.thin > 0 && (i % a.thin) == 0) {
        // charge draw q = x + sigma_eps R xi, H = R R^T with R upper triangular: the
        // factorisation runs from the last PE backwards on a copy of H's lower triangle in the
        // chain's device-memory scratch; y = R xi accumulates column by column
        const int64_t rec = c * a.n_rec + i / a.thin;
        double *Ad = bk.dscr + slot * (int64_t)(KCAP * KCAP + KCAP);
        double *Av = Ad + KCAP * KCAP;  // the column being eliminated
        chain_sync_mem<LPC>();
        bool ok = true;
        for (int r = lane; r < N; r += LPC) {
          for (int k = 0; k <= r; ++k) Ad[r * KCAP + k] = D[lds_at<KCAP, SYM>(k, r)];
          va[r] = charge_normal(step, r, uid0, uid1, a.key0, a.key1);
          vb[r] = 0.0;
        }
        chain_sync_mem<LPC>();
        for (int jj = N - 1; jj >= 0 && ok; --jj) {
          const double ajj = Ad[jj * KCAP + jj];
          if (!(ajj > 0.0)) {
            ok = false;
            break;
          }
          const double dd = sqrt(ajj), xij = va[jj];
          for (int r = lane; r < jj; r += LPC) {
            const double x = Ad[jj * KCAP + r] / dd;
            Av[r] = x;
            vb[r] += x * xij;
          }
          if (lane == 0) vb[jj] += dd * xij;
          chain_sync_mem<LPC>();
          for (int r = lane; r < jj; r += LPC) {
            const double vr = Av[r];
            for (int k = 0; k <= r; ++k) Ad[r * KCAP + k] -= vr * Av[k];
          }
          chain_sync_mem<LPC>();
        }
        if (!ok) st |= FSMP_ST_FACTOR;
        for (int r = lane; r < a.kz; r += LPC) {
          a.zdraw[rec * a.kz + r] = r < N ? zl[r] : -1;
          a.qdraw[rec * a.kz + r] = r < N ? (ok ? xl[r] + a.sigma_eps * vb[r] : NAN) : 0.0;
        }
        chain_sync_mem<LPC>();
      }
    }
  }

  chain_sync_mem<LPC>();
  const int kz = a.kz;
  for (int k = lane; k < kz; k += LPC) {
    a.z[c * kz + k] = k < N ? zl[k] : -1;
    a.charge[c * kz + k] = k < N ? xl[k] : 0.0;
    if (MCP && a.comp) a.comp[c * kz + k] = k < N ? el[k] : -1;
  }
  if (lane < 3) {
    double *ac = a.acc + c * 12;
    ac[2 * lane] = a_s;
    ac[2 * lane + 1] = a_q;
    ac[6 + 2 * lane] = a_bs;
    ac[7 + 2 * lane] = a_bq;
  }
  if (lane < 4) {
    a.counts[c * 8 + 2 * lane] = c_p;
    a.counts[c * 8 + 2 * lane + 1] = c_a;
  }
  if (lane == 0) {
    if (run_n >= 0) atomicAdd(a.nhist + c * (a.kz + 1) + run_n, n_steps - run_s);
    a.n_pe[c] = N;
    a.t0[c] = t0;
    if (a.rec_steps) a.rec_steps[c] = S_rec;
    a.status[c] = st;
    if (a.work) {
      double *wk = a.work + c * 5;
      wk[0] = wk0;
      wk[1] = wk1;
      wk[2] = wk2;
      wk[3] = wk3;
      wk[4] = 0.0;
    }
  }
}

template <int KCAP, int LPC, bool CORR, bool MCP>
__global__ void __launch_bounds__(LPC > kWave ? LPC : kWave) __attribute__((amdgpu_waves_per_eu(2)))
chain_lds_kernel(ChainArgs a) {
  extern __shared__ double smem[];
  chain_lds_body<KCAP, LPC, CORR, MCP>(a, LdsBucket{a.chains, a.n_list, a.dws, a.dscr}, blockIdx.x, smem);
}

// The buckets of capacities up to 64 in one launch, for calls whose workgroups all fit the chip at
// once: as launches of their own they need a hardware queue each to run side by side, and streams
// share queues as HIP deals them (one server event of 1,200 channels: two of its three launches
// ran one after the other: 8.4 ms the call, 4.7 in one launch; 1,000 short windows 7.4, 6.5).
template <bool CORR>
__global__ void __launch_bounds__(kWave) __attribute__((amdgpu_waves_per_eu(2)))
chain_lds_mix_kernel(ChainArgs a, LdsMix m) {
  extern __shared__ double smem[];
  const int64_t b = blockIdx.x;
  if (b < m.end[0])
    chain_lds_body<64, 64, CORR, false>(a, LdsBucket{m.chains[0], m.n_list[0], m.dws[0], m.dscr[0]}, b, smem);
  else if (b < m.end[1])
    chain_lds_body<48, 64, CORR, false>(a, LdsBucket{m.chains[1], m.n_list[1], m.dws[1], m.dscr[1]}, b - m.end[0], smem);
  else if (b < m.end[2])
    chain_lds_body<32, 32, false, false>(a, LdsBucket{m.chains[2], m.n_list[2], m.dws[2], m.dscr[2]}, b - m.end[1], smem);
  else
    chain_lds_body<16, 16, false, false>(a, LdsBucket{m.chains[3], m.n_list[3], m.dws[3], m.dscr[3]}, b - m.end[2], smem);
}

// ------------------------------------------------------------------ chains, one lane each
// birth position for one lane: EXP by the closed-form inverse, BIEXP by bisection on the
// closed-form partial sums (same rule as birth_draw: smallest g with F(g) > target)
__device__ inline int birth_draw_lane(const ModelDev &md, double t0, int glo, int ghi, double target) {
  const GridPos p = grid_pos(md, t0, glo, ghi);
  const XsExp xe = xs_exp(md, p.xs);
  int64_t k;
  if (md.kind == FSMP_PHI_EXP) {
    const double c = target * exp(p.xs * md.inv_tau2) * md.den2 / md.inv_tau2;
    if (c >= 1.0) {
      k = p.n - 1;
    } else {
      const double L = -log1p(-c) / (md.dt * md.inv_tau2);
      k = (int64_t)floor(L);
      if (k < 0) k = 0;
      if (k > p.n - 1) k = p.n - 1;
      if (k > 0 && phi_partial(md, xe, k) > target) k -= 1;
      else if (k < p.n - 1 && !(phi_partial(md, xe, k + 1) > target)) k += 1;
    }
  } else {
    // bisection: the same number of steps in every lane (a Newton inverse with per-lane
    // iteration counts measured slower on the GPU)
    int64_t lo = 0, hi = p.n - 1;
    while (lo < hi) {
      const int64_t mid = lo + (hi - lo) / 2;
      if (phi_partial(md, xe, mid + 1) > target) hi = mid;
      else lo = mid + 1;
    }
    k = lo;
  }
  return (int)(p.gs + k);
}


// Interleaved per-lane state helpers: element e of this lane's chain is p[e * 64].
// Every loop below issues a chunk of independent loads before any store, so one
// memory round trip covers kChunk elements.  Matrices are read into FP64 whatever
// their storage type (FP64, or FP32 in the precision form) and written back rounded.
constexpr int kChunk = 8;

// eta = M gamma over the first n rows; q = gamma^T eta and, when X is given,
// p = gamma^T x, both summed in row order.  Rows go in blocks of 4 and columns in
// chunks of 4: the 20 loads of a chunk are issued unconditionally (indices stay below
// KCAP, a multiple of 4) and the columns past n are dropped by a select, so a chunk
// costs one memory round trip; each row still sums its terms in column order.
template <int KCAP, typename MT>
__device__ inline void lane_matvec(const MT *Mp, const double *G, double *E, const double *X, int n, double &q,
                                   double &p) {
  static_assert(KCAP % 8 == 0, "capacity must be a multiple of 8");
  q = 0.0;
  p = 0.0;
  for (int i0 = 0; i0 < n; i0 += 4) {
    double e[4] = {0.0, 0.0, 0.0, 0.0};
    for (int k0 = 0; k0 < n; k0 += 4) {
      double g[4], h[4][4];
#pragma unroll
      for (int kk = 0; kk < 4; ++kk) {
        g[kk] = G[(k0 + kk) * 64];
#pragma unroll
        for (int u = 0; u < 4; ++u) h[kk][u] = (double)Mp[((k0 + kk) * KCAP + i0 + u) * 64];
      }
#pragma unroll
      for (int kk = 0; kk < 4; ++kk)
#pragma unroll
        for (int u = 0; u < 4; ++u) e[u] = (k0 + kk < n) ? e[u] + h[kk][u] * g[kk] : e[u];
    }
#pragma unroll
    for (int u = 0; u < 4; ++u)
      if (i0 + u < n) {
        E[(i0 + u) * 64] = e[u];
        const double gi = G[(i0 + u) * 64];
        q += gi * e[u];
        if (X) p += gi * X[(i0 + u) * 64];
      }
  }
}

// M(k, i) += (A_i A_k) cA [+ (B_i B_k) cB] for i, k < n.  Loads of a chunk of 8 columns
// are unconditional (below KCAP), stores are guarded.
template <int KCAP, bool TWO, typename MT>
__device__ inline void lane_rank_update(MT *Mp, const double *A, double cA, const double *B, double cB, int n) {
  for (int k = 0; k < n; ++k) {
    const double ak = A[k * 64];
    const double bk = TWO ? B[k * 64] : 0.0;
    for (int i0 = 0; i0 < n; i0 += kChunk) {
      double h[kChunk], av[kChunk], bv[kChunk];
#pragma unroll
      for (int u = 0; u < kChunk; ++u) {
        h[u] = (double)Mp[(k * KCAP + i0 + u) * 64];
        av[u] = A[(i0 + u) * 64];
        if (TWO) bv[u] = B[(i0 + u) * 64];
      }
#pragma unroll
      for (int u = 0; u < kChunk; ++u) {
        double v = h[u] + av[u] * ak * cA;
        if (TWO) v += bv[u] * bk * cB;
        if (i0 + u < n) Mp[(k * KCAP + i0 + u) * 64] = (MT)v;
      }
    }
  }
}

// n elements src[e * 64] -> dst[e * 64] (chunked, loads unconditional below the
// capacity of both rows), converting the type
template <typename DT, typename ST>
__device__ inline void lane_copy(DT *dst, const ST *src, int n) {
  for (int i0 = 0; i0 < n; i0 += kChunk) {
    double v[kChunk];
#pragma unroll
    for (int u = 0; u < kChunk; ++u) v[u] = (double)src[(i0 + u) * 64];
#pragma unroll
    for (int u = 0; u < kChunk; ++u)
      if (i0 + u < n) dst[(i0 + u) * 64] = (DT)v[u];
  }
}

// Charge draw of one lane's chain (q = x + sigma_eps R xi, H = R R^T, R upper
// triangular): the same backward factorisation as the lane-group kernels on a copy of
// H's lower triangle in the interleaved scratch Ap, y = R xi accumulated in S2.  Not
// inlined: it runs only at recorded steps and stays out of the sweep's registers.
template <int KCAP, typename HT>
__device__ __attribute__((noinline)) bool lane_charge_draw(double *Ap, const HT *Hp, const double *Xp, double *S1,
                                                           double *S2, double *S3, const int32_t *Zp, int N, int step,
                                                           uint32_t uid0, uint32_t uid1, uint32_t key0, uint32_t key1,
                                                           double sig, double *q, int32_t *zq, int kz) {
  for (int r = 0; r < N; ++r) {
    for (int k = 0; k <= r; ++k) Ap[(r * KCAP + k) * 64] = (double)Hp[(k * KCAP + r) * 64];
    S1[r * 64] = charge_normal(step, r, uid0, uid1, key0, key1);
    S2[r * 64] = 0.0;
  }
  bool ok = true;
  for (int jj = N - 1; jj >= 0; --jj) {
    const double ajj = Ap[(jj * KCAP + jj) * 64];
    if (!(ajj > 0.0)) {
      ok = false;
      break;
    }
    const double d = sqrt(ajj), xij = S1[jj * 64];
    for (int r = 0; r < jj; ++r) {
      const double v = Ap[(jj * KCAP + r) * 64] / d;
      S3[r * 64] = v;
      S2[r * 64] += v * xij;
    }
    S2[jj * 64] += d * xij;
    for (int r = 0; r < jj; ++r) {
      const double vr = S3[r * 64];
      for (int k = 0; k <= r; ++k) Ap[(r * KCAP + k) * 64] -= vr * S3[k * 64];
    }
  }
  for (int r = 0; r < kz; ++r) {
    zq[r] = r < N ? Zp[r * 64] : -1;
    q[r] = r < N ? (ok ? Xp[r * 64] + sig * S2[r * 64] : NAN) : 0.0;
  }
  return ok;
}

// Workspace of one tile of 64 chains, in doubles: the inverse Gram matrix, five vectors
// (b, x and three scratch); grid indices and the N histogram are in the int workspace.
template <int KCAP>
struct LaneLayout {
  static constexpr int HD = KCAP * KCAP;  // doubles per chain for H
  static constexpr int ED = HD + 5 * KCAP;
  static constexpr int EI = 2 * KCAP + 1;
};

// The inverse Gram matrix of the PE list Zp[0..N) in FP64 by bordering (each step is the
// birth update of the PE-space factor: the exact inverse of the leading block), into Wp.
// Returns false if a Schur complement is not positive.
template <int KCAP>
__device__ bool lane_build(const ModelDev &md, const double *vt, const double *ov, int Lw, double *Wp, double *S1,
                           double *S2, const int32_t *Zp, int N) {
  for (int k = 0; k < N; ++k) {
    const int gk = Zp[k * 64];
    for (int i = 0; i < k; ++i) S1[i * 64] = overlap(md, vt, ov, gk, Zp[i * 64], Lw);
    const double d = overlap(md, vt, ov, gk, gk, Lw) + md.rho;
    double q, p;
    lane_matvec<KCAP, double>(Wp, S1, S2, nullptr, k, q, p);
    const double delta2 = d - q;
    if (!(delta2 > 0.0)) return false;
    const double inv = 1.0 / delta2;
    lane_rank_update<KCAP, false, double>(Wp, S2, inv, nullptr, 0.0, k);
    for (int i = 0; i < k; ++i) {
      const double v = -S2[i * 64] * inv;
      Wp[(k * KCAP + i) * 64] = v;
      Wp[(i * KCAP + k) * 64] = v;
    }
    Wp[(k * KCAP + k) * 64] = inv;
  }
  return true;
}

// Delta-nu and log-acceptance of a birth or update proposal from the inverse Gram
// matrix M (gamma in S1 with a zero at the moved PE, eta = M gamma written to S2).
struct MvResult {
  bool valid;
  double dnu, la, delta2, up, om, xj, ej;
};

template <int KCAP, typename MT>
__device__ inline MvResult lane_propose(const ModelDev &md, const MT *Mp, const double *S1, double *S2,
                                        const double *Xp, int N, int move, int j, double d, double beta, double logLam,
                                        double logN1, double la_ratio) {
  MvResult r;
  r.valid = false;
  r.dnu = 0.0;
  r.la = -INFINITY;
  r.om = 1.0;
  r.xj = 0.0;
  r.ej = 0.0;
  double q, p;
  lane_matvec<KCAP, MT>(Mp, S1, S2, Xp, N, q, p);
  if (move == 1) {
    r.delta2 = d - q;
    r.up = beta - p;
    if (r.delta2 > 0.0) {
      r.dnu = -0.5 * (-md.log_rho + log(r.delta2) + (md.rhom2 - r.up * r.up / r.delta2) * md.inv_s);
      r.la = r.dnu + logLam - logN1 + (N == 0 ? md.logJ : 0.0);
      r.valid = true;
    }
  } else {
    r.om = (double)Mp[(j * KCAP + j) * 64];
    r.xj = Xp[j * 64];
    r.ej = S2[j * 64];
    r.delta2 = d - (q - r.ej * r.ej / r.om);
    r.up = beta - (p - r.ej * r.xj / r.om);
    if (r.delta2 > 0.0 && r.om > 0.0) {
      r.dnu = 0.5 * (-log(r.om) - log(r.delta2) + (r.up * r.up / r.delta2 - r.xj * r.xj / r.om) * md.inv_s);
      r.la = r.dnu + la_ratio;
      r.valid = true;
    }
  }
  return r;
}

// One chain per lane.  The chain's H = G^{-1} (full, KCAP x KCAP, FP64), x, b, scratch and
// PE list live in device memory, interleaved across the 64 chains of a tile so that every
// access of a wavefront is one contiguous segment.  Two wavefronts per SIMD at the least
// (the register budget halves): with one, nothing hides the device-memory round trips of
// the state (measured 21% slower at capacity 16).
template <int KCAP>
__global__ void __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(2))) chain_lane_kernel(ChainArgs a) {
  using LL = LaneLayout<KCAP>;
  extern __shared__ double smem[];
  const ModelDev &md = a.md;
  double *vt = smem;
  double *ov = smem + md.M;
  for (int i = threadIdx.x; i < md.M; i += blockDim.x) vt[i] = a.vtab[i];
  for (int i = threadIdx.x; i < md.sub * md.M; i += blockDim.x) ov[i] = a.ovl[i];
  double *lgn = ov + md.sub * md.M;  // log k, k = 0..KCAP + 1
  for (int i = threadIdx.x; i < KCAP + 2; i += blockDim.x) lgn[i] = log((double)i);
  __syncthreads();
  const int64_t slot = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (slot >= a.n_list) return;

  const int64_t tile = slot >> 6;
  const int ln = (int)(slot & 63);
  double *base = a.dws + tile * (int64_t)LL::ED * 64;
  double *Hp = base + ln;
  double *Xp = base + (int64_t)LL::HD * 64 + ln;
  double *Bp = Xp + KCAP * 64;
  double *S1 = Bp + KCAP * 64;
  double *S2 = S1 + KCAP * 64;
  double *S3 = S2 + KCAP * 64;
  int32_t *Zp = a.iws + tile * (int64_t)LL::EI * 64 + ln;
  int32_t *Hs = Zp + KCAP * 64;
#define HM(k, i) Hp[((k) * KCAP + (i)) * 64]
#define XV(i) Xp[(i) * 64]
#define BV(i) Bp[(i) * 64]
#define G1(i) S1[(i) * 64]
#define G2(i) S2[(i) * 64]
#define G3(i) S3[(i) * 64]
#define ZG(i) Zp[(i) * 64]
#define HIST(i) Hs[(i) * 64]

  const int64_t c = a.chains[slot];
  const int64_t w = c / a.n_chains;
  const int ch = (int)(c % a.n_chains);
  const int Lw = (int)(a.woff[w + 1] - a.woff[w]);
  const double lam = a.lam[w];
  const int kmax = a.kmax[w];
  const int glo = a.grange[2 * w], ghi = a.grange[2 * w + 1];
  const double *mf = a.mf + a.mfoff[w];
  const uint64_t uid = a.wid[w] * (uint64_t)a.n_chains + (uint64_t)ch;
  const uint32_t uid0 = (uint32_t)uid, uid1 = (uint32_t)(uid >> 32);
  uint32_t st = a.wflags[w];
  if (glo > ghi) st |= FSMP_ST_EMPTY_T;
  // this waveform's sweeps and burn-in (the configured burn-in fraction), batch means
  const int steps_w = a.wsteps ? a.wsteps[w] : a.n_steps;
  const int burn = a.wsteps ? (int)((int64_t)steps_w * a.burn_in / a.n_steps) : a.burn_in;
  const int n_steps = (st & FSMP_ST_NONFINITE) ? 0 : steps_w;
  const int S_rec = n_steps > burn ? n_steps - burn : 0;
  const int nb = S_rec > 0 ? (int)floor(sqrt((double)S_rec)) : 0;
  const int lb = nb > 0 ? S_rec / nb : 0;
  for (int k = 0; k <= KCAP; ++k) HIST(k) = 0;

  double t0 = a.t0init[w];
  int N = 0;
  int gmin = INT32_MAX;  // smallest PE grid index (phi must stay positive at every PE)
  double S_cur = 0.0;    // BIEXP: sum_k log(1 - e^{-(t_k - t0)/tau_rise})
  double Phi = (glo <= ghi) ? phi_total(md, t0, glo, ghi) : 0.0;
  double logLam = log(lam * md.dt * Phi);  // changes only with t0
  double acc[12];
#pragma unroll
  for (int i = 0; i < 12; ++i) acc[i] = 0.0;
  double bs0 = 0.0, bs1 = 0.0, bs2 = 0.0;
  int cnt[8];
#pragma unroll
  for (int i = 0; i < 8; ++i) cnt[i] = 0;
  double wk0 = 0.0, wk1 = 0.0, wk2 = 0.0, wk3 = 0.0;
  const bool biexp = md.kind == FSMP_PHI_BIEXP;

  // a caller-supplied initial PE list: G^-1 (FP64, by bordering) and x = G^-1 b of the
  // list before the first sweep; no random numbers are drawn for it
  if (a.zinit && n_steps > 0) {
    const int n0 = (int)(a.zinit_off[c + 1] - a.zinit_off[c]);
    if (n0 > 0) {
      const int32_t *z0 = a.zinit + a.zinit_off[c];
      for (int k = 0; k < n0; ++k) ZG(k) = z0[k];
      if (lane_build<KCAP>(md, vt, ov, Lw, Hp, S1, S2, Zp, n0)) {
        for (int k = 0; k < n0; ++k) BV(k) = mf[ZG(k) - glo] + md.rhom;
        for (int i = 0; i < n0; ++i) {
          double xi = 0.0;
          for (int k = 0; k < n0; ++k) xi += Hp[(i * KCAP + k) * 64] * BV(k);
          XV(i) = xi;
        }
        N = n0;
        for (int i = 0; i < N; ++i) {
          if (biexp) S_cur += log(-expm1(-((double)ZG(i) * md.dt - t0) * md.inv_tau1));
          gmin = ZG(i) < gmin ? ZG(i) : gmin;
          occ_edit(a, c, 1, -1, ZG(i), 0, burn, n_steps);
        }
      } else {
        st |= FSMP_ST_FACTOR;
      }
    }
  }
  for (int step = 0; step < n_steps; ++step) {
    if (a.refresh_M > 0 && step > 0 && step % a.refresh_M == 0 && N > 0) {
      // G^-1 rebuilt by bordering and x = G^-1 b recomputed, against the rounding the edits
      // accumulate
      if (lane_build<KCAP>(md, vt, ov, Lw, Hp, S1, S2, Zp, N)) {
        for (int i = 0; i < N; ++i) {
          double xi = 0.0;
          for (int k = 0; k < N; ++k) xi += Hp[(i * KCAP + k) * 64] * BV(k);
          XV(i) = xi;
        }
      } else {
        st |= FSMP_ST_FACTOR;
      }
    }
    uint32_t r[8];
    philox4x32_10((uint32_t)step, 0u, uid0, uid1, a.key0, a.key1, r);
    philox4x32_10((uint32_t)step, 1u, uid0, uid1, a.key0, a.key1, r + 4);
    const double R = sqrt(-2.0 * log(u01(r[0])));
    const double th = 2.0 * M_PI * u01(r[1]);
    const double xi_t0 = R * cos(th), xi_sh = R * sin(th);

    // ---- Gibbs half-step 1: t0 by Metropolis-Hastings
    const double t0p = t0 + md.t0_sd * xi_t0;
    bool t0acc = false;
    cnt[0]++;
    if (t0p >= md.t0_min && t0p <= md.t0_max) {
      const double xmin = (N > 0) ? (double)gmin * md.dt - t0p : 1.0;
      const bool ok = biexp ? (xmin > 0.0) : (xmin >= 0.0);
      if (ok) {
        double S_new = 0.0;
        if (biexp)
        {
          // the rise factors multiplied in runs of up to eight, one log per run
          double pr = 1.0;
          int m = 0;
          for (int i = 0; i < N; ++i) {
            pr *= rise_factor(md, ZG(i), t0p);
            if (++m == 8) {
              S_new += log(pr);
              pr = 1.0;
              m = 0;
            }
          }
          S_new += log(pr);
        }
        const double part = (double)N * (t0p - t0) * md.inv_tau2 + (S_new - S_cur);
        const double Phip = (glo <= ghi) ? phi_total(md, t0p, glo, ghi) : 0.0;
        const double la0 = part - (lam * md.dt * Phip - lam * md.dt * Phi);
        if (log(u01(r[2])) < la0) {
          t0 = t0p;
          Phi = Phip;
          logLam = log(lam * md.dt * Phi);
          S_cur = S_new;
          t0acc = true;
          cnt[1]++;
        }
      }
    }

    // ---- Gibbs half-step 2: one RJMCMC jump
    const double Lam = lam * md.dt * Phi;
    const double um = u01(r[3]);
    const int move = (N == 0 || um < md.J) ? 1 : (um < 2.0 * md.J ? 2 : 3);
    int j = -1, gnew = -1, sh = 0;
    bool valid = false;
    double dnu = 0.0, la = -INFINITY;
    double delta2 = 1.0, up = 0.0, om = 1.0, xj = 0.0, ej = 0.0, beta = 0.0, dself = 0.0, la_ratio = 0.0;
    bool need_mv = false;
    if (move == 1) {
      cnt[2]++;
      if (N >= kmax) {
        st |= FSMP_ST_KMAX;
      } else if (Phi > 0.0) {
        gnew = birth_draw_lane(md, t0, glo, ghi, u53(r[4], r[5]) * Phi);
        need_mv = Lam > 0.0;
      }
    } else {
      j = (int)(((uint64_t)r[4] * (uint64_t)N) >> 32);
      if (move == 2) {
        cnt[4]++;
        om = HM(j, j);
        xj = XV(j);
        if (om > 0.0) {
          dnu = 0.5 * (-md.log_rho - log(om) + (md.rhom2 - xj * xj / om) * md.inv_s);
          la = dnu - logLam + lgn[N] - (N == 1 ? md.logJ : 0.0);
          valid = true;
          const double r = N - j;
          wk0 += r * (r + 1) / 2 + 1;
          wk2 += 1.0;
        } else {
          st |= FSMP_ST_FACTOR;
        }
      } else {
        cnt[6]++;
        sh = (int)rint(xi_sh * md.shift_sd / md.dt);
        gnew = ZG(j) + sh;
        if (gnew >= glo && gnew <= ghi) {
          const double lpn = log_phi(md, (double)gnew * md.dt - t0);
          if (lpn > -INFINITY) {
            const double lpo = log_phi(md, (double)ZG(j) * md.dt - t0);
            if (sh == 0) {
              valid = true;
              dnu = 0.0;
              la = lpn - lpo;
            } else {
              need_mv = true;
              la_ratio = lpn - lpo;
            }
          }
        }
      }
    }
    if (need_mv) {
      for (int i = 0; i < N; ++i) G1(i) = (i == j) ? 0.0 : overlap(md, vt, ov, gnew, ZG(i), Lw);
      dself = overlap(md, vt, ov, gnew, gnew, Lw) + md.rho;
      beta = mf[gnew - glo] + md.rhom;
      // the word count of the proposal in a packed Cholesky factor, and the G^-1 elements read
      {
        const double K = N, r = N - j;
        wk0 += move == 1 ? K * (K + 1) / 2 + 2 * K + 3 : r * (r + 1) / 2 + 1 + (K - 1) * K / 2 + 2 * (K - 1) + 3;
        wk2 += K * K;
      }
      const MvResult mr =
          lane_propose<KCAP, double>(md, Hp, S1, S2, Xp, N, move, j, dself, beta, logLam, lgn[N + 1], la_ratio);
      valid = mr.valid;
      dnu = mr.dnu;
      la = mr.la;
      delta2 = mr.delta2;
      up = mr.up;
      om = mr.om;
      xj = mr.xj;
      ej = mr.ej;
      if (!valid) st |= FSMP_ST_FACTOR;
    }

    const double logu = log(u01(r[6]));
    bool accepted = false;
    if (valid && logu < la) {
      accepted = true;
      cnt[2 * move + 1]++;
      // One edit path for every accepted move (the wavefront's 64 chains run whichever
      // moves they drew; one path is executed once): with h = row j of H and eta from the
      // proposal, M(k, i) += cu u_i u_k + cv v_i v_k over i, k < N with
      //   birth: u = eta, cu = 1/delta^2; death: u = h, cu = -1/omega;
      //   shift: u = h, cu = -1/omega and v = eta (zero at j), cv = 1/delta^2.
      const bool shift = move == 3 && sh != 0;  // an accepted zero shift changes nothing
      {
        const double K = N, r = N - j;
        const double eb = move == 1 ? K + 3 : (K - 1) + 3, ed = (r - 1) * r + K * (K + 1) / 2;
        wk1 += move == 1 ? eb : move == 2 ? ed : (shift ? ed + eb : 0.0);
      }
      if (move != 3 || shift) {
        wk3 += 2.0 * (double)N * N;
        const double inv_d2 = move == 2 ? 0.0 : 1.0 / delta2;
        const double inv_om = move == 1 ? 0.0 : 1.0 / om;
        const double xn = up * inv_d2;
        const int gj = move == 1 ? -1 : ZG(j);
        occ_edit(a, c, move, gj, gnew, step, burn, n_steps);
        if (move != 1) lane_copy(S3, Hp + (int64_t)j * KCAP * 64, N);  // h = row j of H
        if (shift)
          for (int i = 0; i < N; ++i) G2(i) = (i == j) ? 0.0 : G2(i) - G3(i) * ej * inv_om;
        const double *U = move == 1 ? S2 : S3;
        const double *V = shift ? S2 : U;
        const double cu = move == 1 ? inv_d2 : -inv_om, cv = shift ? inv_d2 : 0.0;
        for (int i = 0; i < N; ++i) {
          const double ui = U[i * 64], vi = V[i * 64];
          XV(i) = move == 1 ? XV(i) - ui * xn
                  : move == 2 ? XV(i) - ui * xj * inv_om
                              : ((i == j) ? xn : XV(i) - ui * xj * inv_om - vi * xn);
        }
        lane_rank_update<KCAP, true, double>(Hp, U, cu, V, cv, N);
        if (move == 1) {
          for (int i = 0; i < N; ++i) {
            const double v = -G2(i) * inv_d2;
            HM(N, i) = v;
            HM(i, N) = v;
          }
          HM(N, N) = inv_d2;
          ZG(N) = gnew;
          BV(N) = beta;
          XV(N) = xn;
          if (biexp) S_cur += log(-expm1(-((double)gnew * md.dt - t0) * md.inv_tau1));
          gmin = gnew < gmin ? gnew : gmin;
          N++;
        } else if (move == 2) {
          const int last = N - 1;
          if (j != last) {
            lane_copy(S3, Hp + (int64_t)last * KCAP * 64, N);  // row `last` moves into slot j
            const double vd = G3(last);
            lane_copy(Hp + (int64_t)j * KCAP * 64, S3, N);
            for (int i = 0; i < N; ++i) HM(i, j) = G3(i);
            HM(j, j) = vd;
            ZG(j) = ZG(last);
            BV(j) = BV(last);
            XV(j) = XV(last);
          }
          N--;
          if (biexp) S_cur -= log(-expm1(-((double)gj * md.dt - t0) * md.inv_tau1));
        } else {
          for (int i = 0; i < N; ++i) {
            if (i == j) {
              HM(j, j) = inv_d2;
            } else {
              const double v = -G2(i) * inv_d2;
              HM(j, i) = v;
              HM(i, j) = v;
            }
          }
          ZG(j) = gnew;
          BV(j) = beta;
          if (biexp)
            S_cur += log(-expm1(-((double)gnew * md.dt - t0) * md.inv_tau1)) -
                     log(-expm1(-((double)gj * md.dt - t0) * md.inv_tau1));
        }
        if (move != 1) {
          if (move == 3 && gnew < gmin) {
            gmin = gnew;
          } else if (gj == gmin) {
            gmin = INT32_MAX;
            for (int i = 0; i < N; ++i) gmin = ZG(i) < gmin ? ZG(i) : gmin;
          }
        }
      }
    }

    if (a.log) {
      fsmp_logrec *lr = a.log + c * (int64_t)a.n_steps + step;
      lr->move = move;
      lr->flags = (valid ? 1 : 0) | (accepted ? 2 : 0) | (t0acc ? 4 : 0);
      lr->j = j;
      lr->g = gnew;
      lr->t0 = t0;
      lr->dnu = valid ? dnu : 0.0;
      lr->log_alpha = valid ? la : -INFINITY;
    }

    // ---- record after burn-in
    if (step >= burn) {
      double Q = 0.0;
      for (int i = 0; i < N; ++i) Q += XV(i);
      const double v0 = (double)N, v1 = Q, v2 = t0;
      acc[0] += v0;
      acc[1] += v0 * v0;
      acc[2] += v1;
      acc[3] += v1 * v1;
      acc[4] += v2;
      acc[5] += v2 * v2;
      const int64_t i = step - burn;
      if (nb > 0 && i < (int64_t)nb * lb) {
        bs0 += v0;
        bs1 += v1;
        bs2 += v2;
        if ((i + 1) % lb == 0) {
          acc[6] += bs0;
          acc[7] += bs0 * bs0;
          acc[8] += bs1;
          acc[9] += bs1 * bs1;
          acc[10] += bs2;
          acc[11] += bs2 * bs2;
          bs0 = bs1 = bs2 = 0.0;
        }
      }
      HIST(N) += 1;
      if (a.trace && a.thin > 0 && (i % a.thin) == 0) {
        double *tr = a.trace + (c * a.n_rec + i / a.thin) * 3;
        tr[0] = v0;
        tr[1] = v2;
        tr[2] = v1;
      }
      if (a.qdraw && a.thin > 0 && (i % a.thin) == 0) {
        const int64_t rec = c * a.n_rec + i / a.thin;
        if (!lane_charge_draw<KCAP, double>(a.dscr + tile * (int64_t)KCAP * KCAP * 64 + ln, Hp, Xp, S1, S2, S3, Zp, N,
                                        step, uid0, uid1, a.key0, a.key1, a.sigma_eps, a.qdraw + rec * a.kz,
                                        a.zdraw + rec * a.kz, a.kz))
          st |= FSMP_ST_FACTOR;
      }
    }
  }

  const int kz = a.kz;
  for (int k = 0; k < kz; ++k) {
    a.z[c * kz + k] = k < N ? ZG(k) : -1;
    a.charge[c * kz + k] = k < N ? XV(k) : 0.0;
  }
  for (int k = 0; k <= kz; ++k) a.nhist[c * (kz + 1) + k] = k <= KCAP ? HIST(k) : 0;
  a.n_pe[c] = N;
  a.t0[c] = t0;
  if (a.rec_steps) a.rec_steps[c] = S_rec;
  for (int i = 0; i < 12; ++i) a.acc[c * 12 + i] = acc[i];
  for (int i = 0; i < 8; ++i) a.counts[c * 8 + i] = cnt[i];
  a.status[c] = st;
  if (a.work) {
    a.work[c * 5 + 0] = wk0;
    a.work[c * 5 + 1] = wk1;
    a.work[c * 5 + 2] = wk2;
    a.work[c * 5 + 3] = wk3;
    a.work[c * 5 + 4] = 0.0;
  }
#undef HM
#undef XV
#undef BV
#undef G1
#undef G2
#undef G3
#undef ZG
#undef HIST
}

// ------------------------------------------------------------------ posterior
// Expected number of PEs at every grid point: the occupancy counts of a waveform's chains
// over its recorded (chain, sweep) pairs; one workgroup per waveform, coalesced over its row.
__global__ void __launch_bounds__(256) occupancy_kernel(PosteriorArgs a) {
  for (int64_t w = blockIdx.x; w < a.n_wave; w += gridDim.x) {
    const int S = a.rec_steps ? a.rec_steps[w * a.n_chains] : a.n_steps - a.burn_in;
    const double inv = S > 0 ? 1.0 / ((double)S * a.n_chains) : 0.0;
    const int64_t b = (int64_t)a.sub * a.woff[w], e = (int64_t)a.sub * a.woff[w + 1];
    for (int64_t g = b + threadIdx.x; g < e; g += blockDim.x) a.occupancy[g] = (double)a.occ[g] * inv;
  }
}

// One wavefront per waveform: lanes 0 .. 2 the moments of N, Q and t0, lanes 0 .. 3 the
// acceptance rates, all lanes the histogram (coalesced; one thread per waveform walked its rows
// word by word).
__global__ void __launch_bounds__(256) posterior_kernel(PosteriorArgs a) {
  const int64_t w = (int64_t)blockIdx.x * (blockDim.x / kWave) + threadIdx.x / kWave;
  const int lane = threadIdx.x % kWave;
  if (w >= a.n_wave) return;
  // the chains of one waveform ran the same number of sweeps
  const int S = a.rec_steps ? a.rec_steps[w * a.n_chains] : a.n_steps - a.burn_in;
  const int nb = S > 0 ? (int)floor(sqrt((double)S)) : 0;
  const int lb = nb > 0 ? S / nb : 0;
  const int C = a.n_chains;
  if (lane < 3) {
    const int v = lane;
    double s1 = 0.0, s2 = 0.0, b1 = 0.0, b2 = 0.0;
    for (int ch = 0; ch < C; ++ch) {
      const double *ac = a.acc + (w * C + ch) * 12;
      s1 += ac[2 * v];
      s2 += ac[2 * v + 1];
      b1 += ac[6 + 2 * v];
      b2 += ac[7 + 2 * v];
    }
    const double n = (double)S * C;
    const double mean = S > 0 ? s1 / n : 0.0;
    const double var = S > 0 ? fmax(s2 / n - mean * mean, 0.0) : 0.0;
    const double B = (double)nb * C;
    double mcse = 0.0;
    if (nb > 0 && B > 1.0) {
      const double bm = b1 / (B * lb);
      const double bv = fmax((b2 / ((double)lb * lb) - B * bm * bm) / (B - 1.0), 0.0);
      mcse = sqrt(bv / B);
    }
    a.mean[w * 3 + v] = mean;
    a.var[w * 3 + v] = var;
    a.mcse[w * 3 + v] = mcse;
  }
  if (lane < 4) {
    double prop = 0.0, acc = 0.0;
    uint32_t st = 0;
    for (int ch = 0; ch < C; ++ch) {
      prop += a.counts[(w * C + ch) * 8 + 2 * lane];
      acc += a.counts[(w * C + ch) * 8 + 2 * lane + 1];
      st |= a.cstatus[w * C + ch];
    }
    a.accept[w * 4 + lane] = prop > 0 ? acc / prop : 0.0;
    if (lane == 0) a.status[w] = st;
  }
  if (a.p_n) {
    const int kz = a.kz;
    const int32_t *nh = a.nhist + w * C * (kz + 1);
    double tot = 0.0;  // whole numbers: exact in any order
    for (int k = lane; k <= kz; k += kWave) {
      double s = 0.0;
      for (int ch = 0; ch < C; ++ch) s += nh[ch * (kz + 1) + k];
      tot += s;
    }
    tot = group_sum<kWave>(tot);
    for (int k = lane; k <= kz; k += kWave) {
      double s = 0.0;
      for (int ch = 0; ch < C; ++ch) s += nh[ch * (kz + 1) + k];
      a.p_n[w * (kz + 1) + k] = tot > 0 ? s / tot : 0.0;
    }
  }
}

// ---- posterior extras: chain diagnostics and the lambda estimates, one wavefront per waveform

// d(lambda) = m(lambda) - lambda, m the mean of k under the weights h_k (lambda / lambda0)^k
// (computed from the largest log-weight down); with `f` also the log-likelihood estimate
// f(lambda) = -(lambda - lambda0) + log sum_k h_k (lambda / lambda0)^k.  lambda = 0 keeps k = 0.
// lh(k): log h_k, -inf for h_k = 0.
template <typename LH>
__device__ inline double lam_tilt(LH lh, int k_lo, int k_hi, double lam, double lam0, double *f) {
  const double lr = lam > 0.0 ? log(lam / lam0) : 0.0;
  const int top = lam > 0.0 ? k_hi : 0;
  double mx = -INFINITY;
  for (int k = k_lo; k <= top; ++k) {
    const double l = lh(k);
    if (l > -INFINITY) mx = fmax(mx, l + k * lr);
  }
  double se = 0.0, sk = 0.0;
  for (int k = k_lo; k <= top; ++k) {
    const double l = lh(k);
    if (l > -INFINITY) {
      const double e = exp(l + k * lr - mx);
      se += e;
      sk += k * e;
    }
  }
  if (f) *f = -(lam - lam0) + mx + log(se);
  return sk / se - lam;
}

// lambda-hat: the + to - crossings of d on 64 grid points of [k_lo, k_hi], each refined to the
// root, and lambda = 0 when k_lo = 0 and d <= 0 at the second point; the largest f wins.  Each
// lane evaluates one point: the grid is one evaluation, and a refinement cuts its interval into
// 65 per evaluation (9 of them where bisecting by one thread took 52).
template <typename LH>
__device__ inline double lambda_mle(LH lh, int k_lo, int k_hi, double lam0, int lane) {
  if (k_lo < 0) return NAN;
  if (k_lo == k_hi) return k_lo;
  constexpr int kGrid = kWave;
  const double span = (double)(k_hi - k_lo);
  const double x = k_lo + span * lane / (kGrid - 1);
  const double dx = lam_tilt(lh, k_lo, k_hi, x, lam0, nullptr);
  const double xp = __shfl(x, lane > 0 ? lane - 1 : 0, kWave), dp = __shfl(dx, lane > 0 ? lane - 1 : 0, kWave);
  const bool zero = k_lo == 0 && (__ballot(lane == 1 && dx <= 0.0) != 0);
  uint64_t cross = __ballot(lane > 0 && dp > 0.0 && dx <= 0.0);
  double est = NAN, best_f = -INFINITY;
  if (zero) {
    double f0;
    (void)lam_tilt(lh, k_lo, k_hi, 0.0, lam0, &f0);
    if (f0 > best_f) {
      best_f = f0;
      est = 0.0;
    }
  }
  while (cross) {
    const int i = __ffsll((unsigned long long)cross) - 1;
    cross &= cross - 1;
    double lo = __shfl(xp, i, kWave), hi = __shfl(x, i, kWave);
    double cand = hi;
    if (__shfl(dx, i, kWave) != 0.0) {
      for (int it = 0; it < 40; ++it) {
        const double mid = 0.5 * (lo + hi);
        if (!(mid > lo && mid < hi)) break;
        const double p = lo + (hi - lo) * (lane + 1) / (kWave + 1);
        const bool neg = !(lam_tilt(lh, k_lo, k_hi, p, lam0, nullptr) > 0.0) || p >= hi;
        const uint64_t bal = __ballot(neg);
        const int l = bal ? __ffsll((unsigned long long)bal) - 1 : kWave;
        const double nlo = __shfl(p, l > 0 ? l - 1 : 0, kWave), nhi = __shfl(p, l < kWave ? l : 0, kWave);
        if (l > 0 && nlo > lo) lo = nlo;
        if (l < kWave && nhi < hi) hi = nhi;
      }
      cand = 0.5 * (lo + hi);
    }
    double fc;
    (void)lam_tilt(lh, k_lo, k_hi, cand, lam0, &fc);
    if (fc > best_f) {
      best_f = fc;
      est = cand;
    }
  }
  return est;
}

// The logs of the waveform's histogram in LDS (lds_k entries per wavefront; 0: rows too long for
// it, taken from device memory at each use).  What bounds it is the chain of exponentials: about
// 11 evaluations of K terms per waveform, each point by a lane of its own (8,000 waveforms of
// four chains, with posterior_kernel: 18 ms with a thread per waveform, under 1 ms now).
__global__ void __launch_bounds__(256) posterior_extra_kernel(PosteriorArgs a, int lds_k) {
  extern __shared__ double smem[];
  const int64_t w = (int64_t)blockIdx.x * (blockDim.x / kWave) + threadIdx.x / kWave;
  const int lane = threadIdx.x % kWave;
  if (w >= a.n_wave) return;
  const int C = a.n_chains;
  const int S = a.rec_steps ? a.rec_steps[w * C] : a.n_steps - a.burn_in;
  // Gelman-Rubin R and the Monte Carlo error from the spread of the chain means
  if (lane < 3) {
    const int v = lane;
    double msum = 0.0;
    for (int ch = 0; ch < C; ++ch) msum += a.acc[(w * C + ch) * 12 + 2 * v] / S;
    const double mbar = msum / C;
    double dev2 = 0.0, wsum = 0.0;
    for (int ch = 0; ch < C; ++ch) {
      const double *ac = a.acc + (w * C + ch) * 12;
      const double m = ac[2 * v] / S;
      dev2 += (m - mbar) * (m - mbar);
      wsum += fmax((ac[2 * v + 1] - S * m * m) / (S - 1), 0.0);
    }
    double r = NAN, mc = NAN;
    if (C >= 2 && S >= 1) mc = sqrt(dev2 / ((double)C * (C - 1)));
    if (C >= 2 && S >= 2) {
      const double W = wsum / C;
      const double B = S * dev2 / (C - 1);
      const double V = (double)(S - 1) / S * W + B / S;
      r = W > 0.0 ? sqrt(V / W) : (V > 0.0 ? INFINITY : 1.0);
    }
    if (a.rhat) a.rhat[w * 3 + v] = r;
    if (a.mcse_chains) a.mcse_chains[w * 3 + v] = mc;
  }
  if (!a.lambda_hat) return;
  const int kz1 = a.kz + 1;
  const int32_t *nh = a.nhist + w * C * kz1;
  double *lg = smem + (int64_t)(threadIdx.x / kWave) * lds_k;
  int k_lo = INT32_MAX, k_hi = -1;
  for (int k = lane; k < kz1; k += kWave) {
    double h = 0.0;
    for (int ch = 0; ch < C; ++ch) h += nh[ch * kz1 + k];
    if (lds_k > 0) lg[k] = log(h);
    if (h > 0.0) {
      k_lo = k < k_lo ? k : k_lo;
      k_hi = k;
    }
  }
  k_lo = group_min<kWave>(k_lo);
  k_hi = -group_min<kWave>(-k_hi);
  WAVE_SYNC();
  if (k_hi < 0) k_lo = -1;
  const double est =
      lds_k > 0 ? lambda_mle([&](int k) { return lg[k]; }, k_lo, k_hi, a.lam0[w], lane)
                : lambda_mle(
                      [&](int k) {
                        double h = 0.0;
                        for (int ch = 0; ch < C; ++ch) h += nh[ch * kz1 + k];
                        return log(h);
                      },
                      k_lo, k_hi, a.lam0[w], lane);
  if (lane == 0) {
    a.lambda_hat[w * 2] = est;
    a.lambda_hat[w * 2 + 1] = a.mean[w * 3 + 1] / a.mu_q;  // lambda-hat_Q = E[Q] / mu_q
  }
}

template <int KCAP, int LPC, int WPB, bool FORCE = false, bool F32 = false, bool MCP = false>
hipError_t launch_chain_t(const ChainArgs &args, hipStream_t st, int32_t *lanes, int64_t *blocks) {
  constexpr int CPB = WPB * (kWave / LPC);
  ChainArgs a = args;
  const int64_t nb = (a.n_list + CPB - 1) / CPB;
  size_t lds = sizeof(double) * ((size_t)a.md.M * (1 + a.md.sub) + (KCAP + 2) +
                                 (size_t)CPB * ChainLayout<KCAP, F32, MCP>::kDoubles);
  // The rise table where it fits beside what the host has checked and costs no workgroup of a CU: two
  // wavefronts per SIMD by their registers, the LDS in units of 1,280 bytes.  (Narrow groups of 96, 2.4
  // KB of table: two workgroups of three are left, 16,000 chains x 60 sweeps 11.4 ms with the table and
  // 9.5 without.)
  auto resident = [](size_t bytes) { return std::min<size_t>(8 / WPB, 160 * 1024 / ((bytes + 1279) / 1280 * 1280)); };
  const size_t with_rise = lds + sizeof(double) * a.md.rise_n;
  if (with_rise > 160 * 1024 || resident(with_rise) < resident(lds)) a.md.rise_n = 0;
  lds += sizeof(double) * a.md.rise_n;
  *lanes = LPC;
  *blocks = nb;
  if (nb == 0) return hipSuccess;
  if (a.dws == nullptr) return hipErrorInvalidValue;
  if (lds > 160 * 1024) return hipErrorInvalidValue;  // the host checks the configurations against this
  if (lds > 64 * 1024) {
    // lift the default dynamic-LDS limit; gfx950 has 160 KB per workgroup
    (void)hipFuncSetAttribute((const void *)chain_kernel<KCAP, LPC, WPB, FORCE, F32, MCP>,
                              hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    (void)hipGetLastError();
  }
  if (FORCE && (a.force == nullptr || a.rdnu == nullptr || a.rla == nullptr)) return hipErrorInvalidValue;
  hipLaunchKernelGGL((chain_kernel<KCAP, LPC, WPB, FORCE, F32, MCP>), dim3((unsigned)nb), dim3(kWave * WPB), lds,
                     st, a);
  return hipGetLastError();
}


template <int KCAP>
hipError_t launch_chain_lane_t(const ChainArgs &a, hipStream_t st, int32_t *lanes, int64_t *blocks) {
  const int64_t nb = (a.n_list + 255) / 256;
  const size_t lds = sizeof(double) * ((size_t)a.md.M * (1 + a.md.sub) + KCAP + 2);
  *lanes = 1;
  *blocks = nb;
  if (nb == 0) return hipSuccess;
  hipLaunchKernelGGL((chain_lane_kernel<KCAP>), dim3((unsigned)nb), dim3(256), lds, st, a);
  return hipGetLastError();
}

// ------------------------------------------------------------------ Lucy-Richardson
// Initial PE sequence by deconvolution (Sec. 2.3): one workgroup per waveform, all arrays
// in LDS, FP64.  Both sums of an iteration are correlations of an LDS array with the
// kernel, out[i] = sum_s X[i + s] k[s]:
//   w^r(t)  = sum_s u[t + s] K[LV - 1 - s]          (u indexed by tau + LV - 1)
//   c(tau)  = sum_s rp[tau + LV - 1 + s] K[s]        (rp: the ratio d / w^r, zero-padded)
// each thread computes R consecutive outputs from a sliding window of X in registers:
// one LDS read of X per R FMAs.  The kernel k is the same for every lane: it is read from
// a read-only device array by scalar loads (eight values per load, through the scalar
// cache), which costs no LDS bandwidth and no vector issue slot.  The lanes of a wavefront
// read X R elements apart, so X is stored skewed by one pad element per R (element e at
// e + e / R): the lanes' reads then fall in different banks.  The first sum uses R = 8;
// the second, which has L_V - 1 more outputs, R = 6, which fills whole wavefronts at the
// usual window lengths (1,024 samples: 128 and 187 chunks, three wavefronts).
constexpr int kLucyR1 = 8, kLucyR2 = 6;

template <int R>
__device__ inline int lsk(int e) {
  return e + e / R;
}

// the read-only kernel array, seen through the constant address space so that its
// wavefront-uniform reads compile to scalar loads
typedef const __attribute__((address_space(4))) double *ConstD;

template <int R>
__device__ inline void lucy_corr(const double *X, ConstD k, int LVp, int i0, double *acc) {
  // i0 and LVp are multiples of R, so every R-element block of X starts at (R + 1) * block
  double xw[R];
  const double *xb = X + (R + 1) * (i0 / R);
#pragma unroll
  for (int j = 0; j < R; ++j) {
    xw[j] = xb[j];
    acc[j] = 0.0;
  }
  const double *nb = xb + (R + 1);  // the next block; one block further per R taps
  for (int s = 0; s < LVp; s += R, nb += R + 1) {
#pragma unroll
    for (int u = 0; u < R; ++u) {
      const double ks = k[s + u];
#pragma unroll
      for (int j = 0; j < R; ++j) acc[j] = fma(xw[j], ks, acc[j]);
#pragma unroll
      for (int j = 0; j < R - 1; ++j) xw[j] = xw[j + 1];
      xw[R - 1] = nb[u];
    }
  }
}

// The data are float32: they are kept so in LDS (half the bytes of a double, one more window of
// 2,048 samples per CU).
__global__ void __launch_bounds__(512) lucy_kernel(LucyArgs a) {
  extern __shared__ double lds[];
  const int LV = a.LV, LVp = a.LVp;
  const ConstD K = (ConstD)a.kern;       // [LVp] K[s], zero beyond LV
  const ConstD Kr = (ConstD)a.kern_rev;  // [LVp] K[LV - 1 - s], zero beyond LV
  __shared__ double redl[8];  // (at most eight wavefronts)
  __shared__ int redc[8];
  constexpr int R1 = kLucyR1, R2 = kLucyR2;
  for (int64_t wi = blockIdx.x; wi < a.n_wave; wi += gridDim.x) {
    const int64_t w = a.order[wi];
    const int Lw = (int)(a.woff[w + 1] - a.woff[w]);
    const int ntau = Lw + LV - 1;
    const int nd = (Lw + R1 - 1) / R1 * R1;       // d zero-padded to whole first-sum chunks
    const int n2 = (ntau + R2 - 1) / R2 * R2;     // outputs of the second sum, whole chunks
    const int nu = n2 + LVp + R1;                 // elements of u (zero beyond ntau)
    const int nrp = n2 + LVp + R2;                // elements of rp: LV - 1 zeros | ratio | zeros
    double *u = lds;                              // skewed by R1
    double *rp = u + lsk<R1>(nu) + 1;             // skewed by R2
    float *d = (float *)(rp + lsk<R2>(nrp) + 1);  // [nd], plain layout
    const float *x = a.wave + a.woff[w];
    __syncthreads();
    double sd = 0.0;
    for (int t = threadIdx.x; t < nd; t += blockDim.x) {
      const float v = t < Lw ? fmaxf(x[t], 0.0f) : 0.0f;
      d[t] = v;
      sd += (double)v;
    }
    for (int o = 32; o > 0; o >>= 1) sd += __shfl_xor(sd, o);
    if ((threadIdx.x & 63) == 0) redl[threadIdx.x >> 6] = sd;
    __syncthreads();
    double tot = 0.0;
    for (int i = 0; i < (int)(blockDim.x >> 6); ++i) tot += redl[i];
    const double u0 = tot / ntau;
    for (int i = threadIdx.x; i < nu; i += blockDim.x) u[lsk<R1>(i)] = i < ntau ? u0 : 0.0;
    for (int i = threadIdx.x; i < nrp; i += blockDim.x) rp[lsk<R2>(i)] = 0.0;
    __syncthreads();
    for (int it = 0; it < a.n_iter; ++it) {
      // w^r and the ratio d / w^r (0 where w^r is not positive).  The writes need no
      // bounds: d is zero past L_w, so the ratios written past the window stay 0
      for (int c0 = threadIdx.x * R1; c0 < Lw; c0 += blockDim.x * R1) {
        double acc[R1];
        lucy_corr<R1>(u, Kr, LVp, c0, acc);
#pragma unroll
        for (int j = 0; j < R1; ++j) {
          // exact division: w^r decays to denormals where d is 0 (0 / w^r must stay 0)
          const double v = acc[j];
          const double q = (double)d[c0 + j] / v;
          rp[lsk<R2>(LV - 1 + c0 + j)] = v > 0.0 ? q : 0.0;
        }
      }
      __syncthreads();
      // u(tau) *= sum_t ratio(t) K(t - tau); u stays 0 past tau = L_w - 1 (a select, no branch)
      for (int c0 = threadIdx.x * R2; c0 < ntau; c0 += blockDim.x * R2) {
        double acc[R2];
        lucy_corr<R2>(rp, K, LVp, c0, acc);
#pragma unroll
        for (int j = 0; j < R2; ++j) {
          double *ue = u + lsk<R1>(c0 + j);
          *ue = c0 + j < ntau ? *ue * acc[j] : 0.0;
        }
      }
      __syncthreads();
    }
    // qhat in PE-charge units (back into a plain layout in rp); candidates tau >= 0 above the
    // threshold (flags in d)
    double lam = 0.0;
    int cnt = 0;
    for (int i = threadIdx.x; i < ntau; i += blockDim.x) {
      const double q = u[lsk<R1>(i)] * a.inv_area;
      rp[i] = q;
      lam += q;
      if (a.qhat) a.qhat[a.woff[w] + w * (int64_t)(LV - 1) + i] = q;
    }
    __syncthreads();
    const double *qh = rp;
    double *flag = u;  // plain layout from here on
    for (int i = threadIdx.x; i < Lw; i += blockDim.x) {
      const bool c = qh[i + LV - 1] > a.threshold;   // tau = i >= 0
      d[i] = c ? 1.0f : 0.0f;
      cnt += c;
    }
    for (int o = 32; o > 0; o >>= 1) {
      lam += __shfl_xor(lam, o);
      cnt += __shfl_xor(cnt, o);
    }
    __syncthreads();
    if ((threadIdx.x & 63) == 0) {
      redl[threadIdx.x >> 6] = lam;
      redc[threadIdx.x >> 6] = cnt;
    }
    __syncthreads();
    lam = 0.0;
    cnt = 0;
    for (int i = 0; i < (int)(blockDim.x >> 6); ++i) {
      lam += redl[i];
      cnt += redc[i];
    }
    const int kmax = a.kmax[w];
    if (cnt > kmax) {
      // keep the kmax largest qhat (ties: earlier tau): rank every candidate
      for (int i = threadIdx.x; i < Lw; i += blockDim.x) {
        if (d[i] == 0.0f) {
          flag[i] = 0.0;
          continue;
        }
        const double qi = qh[i + LV - 1];
        int rank = 0;
        for (int j = 0; j < Lw; ++j) {
          const double qj = qh[j + LV - 1];
          rank += (qj > a.threshold) && (qj > qi || (qj == qi && j < i));
        }
        flag[i] = rank < kmax ? 1.0 : 0.0;
      }
      __syncthreads();
      for (int i = threadIdx.x; i < Lw; i += blockDim.x) d[i] = (float)flag[i];
      __syncthreads();
    }
    if (threadIdx.x == 0) {
      int t_min = -1, t_max = -1;
      for (int i = 0; i < Lw; ++i)
        if (d[i] != 0.0f) {
          if (t_min < 0) t_min = i;
          t_max = i;
        }
      int n = 0;
      double t0 = 0.5 * (a.t0_min + a.t0_max);
      const int sub = a.sub;
      if (t_min < 0) {
        a.g_range[2 * w] = 1;
        a.g_range[2 * w + 1] = 0;
        a.cut[2 * w] = 0;
        a.cut[2 * w + 1] = Lw - 1;
      } else {
        t0 = fmin(fmax(t_min - 0.5 / sub, a.t0_min), a.t0_max);
        for (int i = t_min; i <= t_max; ++i)
          if (d[i] != 0.0f && i - t0 > 0.0 && n < a.kz) a.z[w * (int64_t)a.kz + n++] = sub * i;
        a.g_range[2 * w] = max(0, sub * (t_min - a.margin));
        a.g_range[2 * w + 1] = min(sub * Lw - 1, sub * (t_max + a.margin));
        a.cut[2 * w] = max(0, t_min - a.margin);
        a.cut[2 * w + 1] = min(Lw - 1, t_max + a.margin + LV);
      }
      for (int k = n; k < a.kz; ++k) a.z[w * (int64_t)a.kz + k] = -1;
      a.n_pe[w] = n;
      a.t0[w] = t0;
      a.lam[w] = lam;
    }
    __syncthreads();
  }
}

}  // namespace

hipError_t launch_prologue(const PrologueArgs &a, hipStream_t st) {
  if (a.n_wave == 0) return hipSuccess;
  const int64_t nb = a.n_wave < 65535 * 8 ? a.n_wave : 65535 * 8;
  hipLaunchKernelGGL(prologue_kernel, dim3((unsigned)nb), dim3(256), sizeof(double) * a.md.M, st, a);
  return hipGetLastError();
}

size_t lucy_lds_bytes(int64_t Lw, int LVp) {
  const int64_t R1 = kLucyR1, R2 = kLucyR2;
  const int64_t ntau = Lw + LVp - 1;
  const int64_t nd = (Lw + R1 - 1) / R1 * R1, n2 = (ntau + R2 - 1) / R2 * R2;
  const int64_t nu = n2 + LVp + R1, nrp = n2 + LVp + R2;
  // u and rp, each skewed by one pad element per window width, then d
  return sizeof(double) * (size_t)((nu + nu / R1 + 1) + (nrp + nrp / R2 + 1)) + sizeof(float) * (size_t)((nd + 1) / 2 * 2);
}

hipError_t launch_lucy(const LucyArgs &a, int64_t max_len, hipStream_t st) {
  if (a.n_wave == 0) return hipSuccess;
  const size_t lds = lucy_lds_bytes(max_len, a.LVp);
  // enough threads for the longer pass of the longest window, in whole wavefronts
  const int64_t chunks = std::max((max_len + kLucyR1 - 1) / kLucyR1, (max_len + a.LV - 1 + kLucyR2 - 1) / kLucyR2);
  int threads = (int)((chunks + 63) / 64 * 64);
  threads = threads < 64 ? 64 : (threads > 512 ? 512 : threads);
  if (lds > 64 * 1024) {
    (void)hipFuncSetAttribute((const void *)lucy_kernel, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    (void)hipGetLastError();
  }
  const int64_t nb = a.n_wave < 65535 * 8 ? a.n_wave : 65535 * 8;
  hipLaunchKernelGGL(lucy_kernel, dim3((unsigned)nb), dim3(threads), lds, st, a);
  return hipGetLastError();
}

hipError_t launch_posterior(const PosteriorArgs &a, hipStream_t st) {
  if (a.n_wave == 0) return hipSuccess;
  const int64_t nb = (a.n_wave + 3) / 4;  // four wavefronts, one waveform each
  hipLaunchKernelGGL(posterior_kernel, dim3((unsigned)nb), dim3(256), 0, st, a);
  hipError_t e = hipGetLastError();
  if (e == hipSuccess && (a.rhat || a.mcse_chains || a.lambda_hat)) {
    const int lds_k = a.lambda_hat && a.kz + 1 <= 2048 ? a.kz + 1 : 0;
    hipLaunchKernelGGL(posterior_extra_kernel, dim3((unsigned)nb), dim3(256), sizeof(double) * 4 * lds_k, st, a, lds_k);
    e = hipGetLastError();
  }
  if (e == hipSuccess && a.occupancy) {
    const int64_t nw = a.n_wave < 65535 * 8 ? a.n_wave : 65535 * 8;
    hipLaunchKernelGGL(occupancy_kernel, dim3((unsigned)nw), dim3(256), 0, st, a);
    e = hipGetLastError();
  }
  return e;
}

int chain_kcap_for(int kmax) {
  for (int b = 0; b < kNumCaps; ++b)
    if (kmax <= kCaps[b]) return kCaps[b];
  return 0;
}

// lane-group instances: PE capacity, lanes per chain, wavefronts per workgroup.  With H
// in LDS the LDS bounds the chains per CU (one chain per wavefront at capacity 64); with H
// in device memory each chain keeps only its vectors in LDS, so groups can be narrow and a
// CU holds 8-16x more chains: the narrow table, for launches that throughput bounds (chains
// of equal length).  The wide table (FSMP_DESIGN_GROUP_DEVMEM_WIDE) gives each chain 2-4x the
// lanes, a whole wavefront from capacity 64 up: for launches whose longest chains set their
// duration (per-waveform sweep counts up to 8x the shortest), where a wider group shortens
// each of their sweeps (measured on the uneven-window workload: 1.38 s per step narrow, 0.92 s
// wide from capacity 96 up).
struct GroupCfg {
  int kcap, lpc, wpb;
};
static const GroupCfg kGroupDM[] = {{16, 4, 4},  {32, 4, 4},   {48, 16, 2},  {64, 32, 4},
                                    {96, 16, 2}, {128, 32, 4}, {160, 32, 4}, {192, 32, 2}};
static const GroupCfg kGroupDMWide[] = {{32, 16, 4}, {48, 32, 4},  {64, 64, 4},  {96, 64, 4},
                                        {128, 64, 4}, {160, 64, 4}, {192, 64, 2}};
// the FP32 form keeps eight vectors per chain in LDS: two wavefronts per workgroup at the
// capacities of 4-lane groups (at four, capacity 32 would need 168 KB)
static const GroupCfg kGroupDMF32[] = {{16, 4, 2},  {32, 4, 2},   {64, 32, 4},  {96, 64, 4},
                                       {128, 64, 4}, {160, 64, 4}, {192, 64, 2}};
// its wide groups: 16 lanes per chain at the two smallest capacities (a quarter of the sweep
// latency of the 4-lane groups, which matters where one event's chains finish together);
// from capacity 64 up its groups are already 32-64 lanes wide
static const GroupCfg kGroupDMF32Wide[] = {{16, 16, 4}, {32, 16, 4}};

// the vectors of a chain's LDS block (ChainLayout::kVec); the corrected FP64 form (and with it
// group_dm_ws_doubles' exact G) from capacity 48 up
static_assert(ChainLayout<48>::kCorr && !ChainLayout<32>::kCorr && ChainLayout<64, false, true>::kCorr,
              "the host's sizes assume the corrected FP64 form at capacities 48 and up");
static int chain_vectors(int kcap, bool f32) {
  if (f32) return ChainLayout<64, true>::kVec;
  return kcap >= 48 ? ChainLayout<64>::kVec : ChainLayout<16>::kVec;
}

static size_t chain_lds_bytes(const GroupCfg &g, int M, int sub, bool f32, bool mcp) {
  const int cpb = g.wpb * (64 / g.lpc);
  const size_t per = (size_t)ChainLayout<16>::kAcc + (size_t)chain_vectors(g.kcap, f32) * (size_t)g.kcap +
                     ((size_t)g.kcap + 1) / 2 * (mcp ? 2 : 1);
  return sizeof(double) * ((size_t)M * (1 + sub) + (size_t)g.kcap + 2 + (size_t)cpb * per);
}

// lanes per chain and LDS doubles of one chain of the LDS instances (0: no such instance); `corr`
// means what it does in launch_chain_lds
template <bool MCP>
static int lds_chain_doubles_t(int kcap, bool corr) {
  switch (kcap) {
    case 16: return corr ? 0 : LdsLayout<16, 16, false, MCP>::kDoubles;
    case 32: return corr ? 0 : LdsLayout<32, 32, false, MCP>::kDoubles;
    case 48: return LdsLayout<48, 64, true, MCP>::kDoubles;  // (the uncorrected form takes less)
    case 64: return LdsLayout<64, 64, true, MCP>::kDoubles;
    case 96: return corr ? LdsLayout<96, 128, true, MCP>::kDoubles : 0;
    case 128: return corr ? LdsLayout<128, 128, true, MCP>::kDoubles : 0;
    case 160: return corr ? LdsLayout<160, 192, true, MCP>::kDoubles : 0;
    case 192: return corr ? LdsLayout<192, 192, true, MCP>::kDoubles : 0;
    default: return 0;
  }
}
static int lds_chain_doubles(int kcap, bool corr, bool mcp, int *lpc) {
  *lpc = kcap <= 32 ? kcap : kcap <= 64 ? 64 : kcap <= 128 ? 128 : 192;
  if (!mcp && !corr && kcap == 48) return LdsLayout<48, 64, false, false>::kDoubles;
  if (!mcp && !corr && kcap == 64) return LdsLayout<64, 64, false, false>::kDoubles;
  if (mcp && !corr && kcap >= 48) return 0;
  return mcp ? lds_chain_doubles_t<true>(kcap, corr) : lds_chain_doubles_t<false>(kcap, corr);
}

// LDS bytes of a workgroup (one wavefront, or one chain of several) without the rise table
static size_t lds_block_bytes(int kcap, bool corr, bool mcp) {
  int lpc;
  const int per = lds_chain_doubles(kcap, corr, mcp, &lpc);
  return sizeof(double) * ((size_t)kcap + 2 + (size_t)(lpc < kWave ? kWave / lpc : 1) * per);
}

size_t lds_ws_doubles(int kcap, bool corr, int64_t n_list) { return corr ? (size_t)n_list * kcap * kcap : 0; }

bool chain_lds_supported(int kcap, bool corr, bool mcp) {
  int lpc;
  return lds_chain_doubles(kcap, corr, mcp, &lpc) > 0 && lds_block_bytes(kcap, corr, mcp) <= 160 * 1024;
}

template <int KCAP, int LPC, bool CORR, bool MCP = false>
static hipError_t launch_chain_lds_t(const ChainArgs &args, hipStream_t st, int32_t *lanes, int64_t *blocks) {
  ChainArgs a = args;
  constexpr int W = LdsLayout<KCAP, LPC, CORR, MCP>::kW, CPW = LPC < kWave ? kWave / LPC : 1;
  *lanes = LPC;
  *blocks = (a.n_list + CPW - 1) / CPW;
  if (*blocks == 0) return hipSuccess;
  if (CORR && a.dws == nullptr) return hipErrorInvalidValue;
  // the rise table where it fits
  const size_t kLds = 160 * 1024;
  size_t lds = lds_block_bytes(KCAP, CORR, MCP);
  if (lds + sizeof(double) * a.md.rise_n > kLds) a.md.rise_n = 0;
  lds += sizeof(double) * a.md.rise_n;
  if (lds > kLds) return hipErrorInvalidValue;  // the host checks the configurations against this
  if (lds > 64 * 1024) {
    (void)hipFuncSetAttribute((const void *)chain_lds_kernel<KCAP, LPC, CORR, MCP>,
                              hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    (void)hipGetLastError();
  }
  hipLaunchKernelGGL((chain_lds_kernel<KCAP, LPC, CORR, MCP>), dim3((unsigned)*blocks), dim3(kWave * W), lds, st, a);
  return hipGetLastError();
}

hipError_t launch_chain_lds(int kcap, bool corr, const ChainArgs &a, hipStream_t st, int32_t *lanes,
                            int64_t *blocks) {
  if (a.md.n_mix > 0) {
    switch (kcap) {
      case 16: return launch_chain_lds_t<16, 16, false, true>(a, st, lanes, blocks);
      case 32: return launch_chain_lds_t<32, 32, false, true>(a, st, lanes, blocks);
      case 48: return launch_chain_lds_t<48, 64, true, true>(a, st, lanes, blocks);
      case 64: return launch_chain_lds_t<64, 64, true, true>(a, st, lanes, blocks);
      case 96: return launch_chain_lds_t<96, 128, true, true>(a, st, lanes, blocks);
      case 128: return launch_chain_lds_t<128, 128, true, true>(a, st, lanes, blocks);
      case 160: return launch_chain_lds_t<160, 192, true, true>(a, st, lanes, blocks);
      case 192: return launch_chain_lds_t<192, 192, true, true>(a, st, lanes, blocks);
      default: return hipErrorInvalidValue;
    }
  }
  if (corr) {
    switch (kcap) {
      case 48: return launch_chain_lds_t<48, 64, true>(a, st, lanes, blocks);
      case 64: return launch_chain_lds_t<64, 64, true>(a, st, lanes, blocks);
      case 96: return launch_chain_lds_t<96, 128, true>(a, st, lanes, blocks);
      case 128: return launch_chain_lds_t<128, 128, true>(a, st, lanes, blocks);
      case 160: return launch_chain_lds_t<160, 192, true>(a, st, lanes, blocks);
      case 192: return launch_chain_lds_t<192, 192, true>(a, st, lanes, blocks);
      default: return hipErrorInvalidValue;
    }
  }
  switch (kcap) {
    case 16: return launch_chain_lds_t<16, 16, false>(a, st, lanes, blocks);
    case 32: return launch_chain_lds_t<32, 32, false>(a, st, lanes, blocks);
    case 48: return launch_chain_lds_t<48, 64, false>(a, st, lanes, blocks);
    case 64: return launch_chain_lds_t<64, 64, false>(a, st, lanes, blocks);
    default: return hipErrorInvalidValue;
  }
}

static constexpr int kMixCap[4] = {64, 48, 32, 16};

int lds_mix_index(int kcap) {
  for (int q = 0; q < 4; ++q)
    if (kMixCap[q] == kcap) return q;
  return -1;
}

// LDS of a workgroup of the mixed launch: its largest bucket's
static size_t lds_mix_bytes(const LdsMix &m, bool corr, int rise_n) {
  size_t lds = 0;
  for (int q = 0; q < 4; ++q)
    if (m.n_list[q] > 0) lds = std::max(lds, lds_block_bytes(kMixCap[q], corr && kMixCap[q] >= 48, false));
  return lds + sizeof(double) * rise_n;
}

int64_t lds_mix_blocks(const LdsMix &m, bool corr, int rise_n, int64_t *at_once) {
  int64_t nb = 0;
  for (int q = 0; q < 4; ++q) {
    const int64_t cpw = q < 2 ? 1 : kWave / kMixCap[q];
    nb += (m.n_list[q] + cpw - 1) / cpw;
  }
  *at_once = 256 * std::min<int64_t>(8, (int64_t)(160 * 1024 / (lds_mix_bytes(m, corr, rise_n) + 256)));
  return nb;
}

hipError_t launch_chain_lds_mix(bool corr, const ChainArgs &a, LdsMix m, hipStream_t st, int64_t *blocks) {
  int64_t nb = 0;
  for (int q = 0; q < 4; ++q) {
    const int64_t cpw = q < 2 ? 1 : kWave / kMixCap[q];
    nb += (m.n_list[q] + cpw - 1) / cpw;
    m.end[q] = nb;
    if (corr && q < 2 && m.n_list[q] > 0 && m.dws[q] == nullptr) return hipErrorInvalidValue;
  }
  *blocks = nb;
  if (nb == 0) return hipSuccess;
  const size_t lds = lds_mix_bytes(m, corr, a.md.rise_n);  // (the tables fit beside every one of these)
  if (lds > 160 * 1024) return hipErrorInvalidValue;
  if (corr) hipLaunchKernelGGL((chain_lds_mix_kernel<true>), dim3((unsigned)nb), dim3(kWave), lds, st, a, m);
  else hipLaunchKernelGGL((chain_lds_mix_kernel<false>), dim3((unsigned)nb), dim3(kWave), lds, st, a, m);
  return hipGetLastError();
}

hipError_t launch_overlap_partial(const double *vtab, double *out, int sub, int M, int LV, hipStream_t st) {
  hipLaunchKernelGGL(overlap_partial_kernel, dim3((unsigned)((sub * M + 63) / 64)), dim3(64), sizeof(double) * M, st,
                     vtab, out, sub, M, LV);
  return hipGetLastError();
}

bool chain_dm_supported(int kcap, int M, int sub, bool f32, bool mcp, bool wide) {
  if (f32 && mcp) return false;
  if (wide && f32) {
    for (const GroupCfg &g : kGroupDMF32Wide)
      if (g.kcap == kcap) return chain_lds_bytes(g, M, sub, true, false) <= 160 * 1024;
    return false;
  }
  if (wide) {
    if (mcp) return false;
    for (const GroupCfg &g : kGroupDMWide)
      if (g.kcap == kcap) return chain_lds_bytes(g, M, sub, false, false) <= 160 * 1024;
    return false;
  }
  if (f32) {
    // no capacity 48: the precision form runs it at 64
    for (const GroupCfg &g : kGroupDMF32)
      if (g.kcap == kcap) return chain_lds_bytes(g, M, sub, true, false) <= 160 * 1024;
    return false;
  }
  for (const GroupCfg &g : kGroupDM)
    if (g.kcap == kcap) return chain_lds_bytes(g, M, sub, false, mcp) <= 160 * 1024;
  return false;
}

// H (FP64, with the exact G from capacity 48 up; or FP32 plus the FP64 refresh matrix and the
// exact G) of every chain, in tiles of a wavefront
size_t group_dm_ws_doubles(int kcap, int64_t n_list, bool f32, bool wide) {
  const GroupCfg *t = f32 ? (wide ? kGroupDMF32Wide : kGroupDMF32) : wide ? kGroupDMWide : kGroupDM;
  const int nt = f32    ? (wide ? (int)(sizeof kGroupDMF32Wide / sizeof *kGroupDMF32Wide)
                                : (int)(sizeof kGroupDMF32 / sizeof *kGroupDMF32))
                 : wide ? (int)(sizeof kGroupDMWide / sizeof *kGroupDMWide)
                        : (int)(sizeof kGroupDM / sizeof *kGroupDM);
  for (int q = 0; q < nt; ++q)
    if (t[q].kcap == kcap) {
      const int64_t cpw = 64 / t[q].lpc;
      const size_t k2 = (size_t)kcap * kcap;
      return (size_t)((n_list + cpw - 1) / cpw) * cpw * (f32 ? k2 / 2 + 2 * k2 : kcap >= 48 ? 2 * k2 : k2);
    }
  return 0;
}

size_t lane_ws_doubles(int kcap, int64_t n_list) {
  const size_t tiles = (size_t)((n_list + 63) / 64);
  return tiles * 64 * ((size_t)kcap * kcap + 5 * (size_t)kcap);
}

size_t lane_ws_ints(int kcap, int64_t n_list) {
  const size_t tiles = (size_t)((n_list + 63) / 64);
  return tiles * 64 * (2 * (size_t)kcap + 1);
}

hipError_t launch_chain_lane(int kcap, const ChainArgs &a, hipStream_t st, int32_t *lanes, int64_t *blocks) {
  // one lane per chain pays off only for small PE counts: instances at capacities 16 and 32
  switch (kcap) {
    case 16: return launch_chain_lane_t<16>(a, st, lanes, blocks);
    case 32: return launch_chain_lane_t<32>(a, st, lanes, blocks);
    default: return hipErrorInvalidValue;
  }
}

// instances must match kGroupDM (kGroupDMWide for `wide`, kGroupDMF32 and kGroupDMF32Wide for
// the FP32 form; no wide groups for the mixture law)
hipError_t launch_chain_dm(int kcap, bool fp32, bool wide, const ChainArgs &a, hipStream_t st, int32_t *lanes,
                           int64_t *blocks) {
  if (wide && fp32) {
    if (a.md.n_mix > 0 || a.force) return hipErrorInvalidValue;
    switch (kcap) {
      case 16: return launch_chain_t<16, 16, 4, false, true>(a, st, lanes, blocks);
      case 32: return launch_chain_t<32, 16, 4, false, true>(a, st, lanes, blocks);
      default: return hipErrorInvalidValue;
    }
  }
  if (wide) {
    if (a.md.n_mix > 0) return hipErrorInvalidValue;
    if (a.force) {
      // replay with the wide groups, capacities from 64 up
      switch (kcap) {
        case 64: return launch_chain_t<64, 64, 4, true>(a, st, lanes, blocks);
        case 96: return launch_chain_t<96, 64, 4, true>(a, st, lanes, blocks);
        case 128: return launch_chain_t<128, 64, 4, true>(a, st, lanes, blocks);
        case 160: return launch_chain_t<160, 64, 4, true>(a, st, lanes, blocks);
        case 192: return launch_chain_t<192, 64, 2, true>(a, st, lanes, blocks);
        default: return hipErrorInvalidValue;
      }
    }
    // sampling: the LDS chains are the faster ones at the other capacities whatever their number
    switch (kcap) {
      case 96: return launch_chain_t<96, 64, 4>(a, st, lanes, blocks);
      case 128: return launch_chain_t<128, 64, 4>(a, st, lanes, blocks);
      case 160: return launch_chain_t<160, 64, 4>(a, st, lanes, blocks);
      default: return hipErrorInvalidValue;
    }
  }
  if (a.md.n_mix > 0) {
    if (a.force || fp32) return hipErrorInvalidValue;
    switch (kcap) {
      case 16: return launch_chain_t<16, 4, 4, false, false, true>(a, st, lanes, blocks);
      case 32: return launch_chain_t<32, 4, 4, false, false, true>(a, st, lanes, blocks);
      case 48: return launch_chain_t<48, 16, 2, false, false, true>(a, st, lanes, blocks);
      case 64: return launch_chain_t<64, 32, 4, false, false, true>(a, st, lanes, blocks);
      case 96: return launch_chain_t<96, 16, 2, false, false, true>(a, st, lanes, blocks);
      case 128: return launch_chain_t<128, 32, 4, false, false, true>(a, st, lanes, blocks);
      case 160: return launch_chain_t<160, 32, 4, false, false, true>(a, st, lanes, blocks);
      case 192: return launch_chain_t<192, 32, 2, false, false, true>(a, st, lanes, blocks);
      default: return hipErrorInvalidValue;
    }
  }
  if (a.force) {
    switch (kcap) {
      case 16: return launch_chain_t<16, 4, 4, true>(a, st, lanes, blocks);
      case 32: return launch_chain_t<32, 4, 4, true>(a, st, lanes, blocks);
      case 48: return launch_chain_t<48, 16, 2, true>(a, st, lanes, blocks);
      case 64: return launch_chain_t<64, 32, 4, true>(a, st, lanes, blocks);
      case 96: return launch_chain_t<96, 16, 2, true>(a, st, lanes, blocks);
      case 128: return launch_chain_t<128, 32, 4, true>(a, st, lanes, blocks);
      case 160: return launch_chain_t<160, 32, 4, true>(a, st, lanes, blocks);
      case 192: return launch_chain_t<192, 32, 2, true>(a, st, lanes, blocks);
      default: return hipErrorInvalidValue;
    }
  }
  if (fp32) {
    // instances must match kGroupDMF32
    switch (kcap) {
      case 16: return launch_chain_t<16, 4, 2, false, true>(a, st, lanes, blocks);
      case 32: return launch_chain_t<32, 4, 2, false, true>(a, st, lanes, blocks);
      case 64: return launch_chain_t<64, 32, 4, false, true>(a, st, lanes, blocks);
      case 96: return launch_chain_t<96, 64, 4, false, true>(a, st, lanes, blocks);
      case 128: return launch_chain_t<128, 64, 4, false, true>(a, st, lanes, blocks);
      case 160: return launch_chain_t<160, 64, 4, false, true>(a, st, lanes, blocks);
      case 192: return launch_chain_t<192, 64, 2, false, true>(a, st, lanes, blocks);
      default: return hipErrorInvalidValue;
    }
  }
  switch (kcap) {
    case 16: return launch_chain_t<16, 4, 4>(a, st, lanes, blocks);
    case 32: return launch_chain_t<32, 4, 4>(a, st, lanes, blocks);
    case 48: return launch_chain_t<48, 16, 2>(a, st, lanes, blocks);
    case 64: return launch_chain_t<64, 32, 4>(a, st, lanes, blocks);
    case 96: return launch_chain_t<96, 16, 2>(a, st, lanes, blocks);
    case 128: return launch_chain_t<128, 32, 4>(a, st, lanes, blocks);
    case 160: return launch_chain_t<160, 32, 4>(a, st, lanes, blocks);
    case 192: return launch_chain_t<192, 32, 2>(a, st, lanes, blocks);
    default: return hipErrorInvalidValue;
  }
}

}  // namespace fsmp

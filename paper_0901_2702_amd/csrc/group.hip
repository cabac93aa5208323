// The group inverter: the Levenberg-Marquardt fit of kernels.hip with the
// lanes of a wave on one pixel's synthesis points instead of on 64 pixels.
//
// lm_kernel keeps a pixel per lane, so a launch takes as long as one lane's
// fit however few pixels it has: up to 51 passes of 59 (HMI) or 460 (fine
// spectra) synthesis points one after the other.  Here a wave works on a few
// pixels (slots).  Lane k owns slot k: it keeps the pixel's model, takes the
// decisions and solves the damped system; the synthesis passes of the slots
// follow one another with a point per lane, and the sums over the points are
// formed in the order in which lm_kernel forms them: every row sum adds the
// points in record order, chi^2 the rows in slot order, H and g the residuals
// in the same order.  The dense row sums (59 points, every row sees nearly all
// of them) run on the matrix cores: v_mfma_f32_16x16x4_f32 adds its four
// products one after the other, each with one float32 rounding, as a chain of
// fmaf does, so rows x quantities over 4 points are one instruction and the
// same bits.  The banded rows see 16 points each and are summed on the vector
// ALUs: 38 matrix instructions per chunk, three quarters of them on zero
// taps, hold a wave up for longer (100,003 fine spectra 38.3 ms, now 30.5).
// All products, sums and decisions being those of lm_kernel, so are the
// results, bit for bit.
//
// Trials run without derivatives; only a start and an accepted model that
// does not end its fit get their Jacobian (Fig. 6), with no wave-mates to
// wait for.  The normal equations are equilibrated once per Jacobian and stay
// in LDS for the rejected trials after it.
//
// Few pixels are bound by one fit's serial chain (points, row sums, chi^2,
// Cholesky: 7 us per trial of an HMI pixel), many by VALU issue (79% of the
// cycles at 65,536 HMI pixels, 88% at as many fine spectra), at about 620 wave
// instructions per trial of an HMI pixel (lm_kernel: 500, with lanes and
// derivative passes that wait for each other).  Eight slots share the solve,
// the decisions and the set-up of a turn, which one lane each would otherwise
// run alone (two pixels per wave, 32 lanes each: 1,750 instructions per
// trial, 131,072 pixels in 18.2 ms instead of 6.9).  Measured, default
// options: 37 HMI pixels 3.77 ms (lm_kernel) -> 0.32 ms, 4,096 4.25 -> 0.57,
// 65,536 4.6 -> 3.56; 1,000 fine spectra 30.3 -> 1.42 ms, 100,003 64.0 -> 29.6.
// A chunk costs its 64 points' time however many of them there are, so fits
// through few points, and those of few trials, whose set-up counts, are slower
// here from fewer pixels on (routes.h).
#include <hip/hip_runtime.h>

#include "group.h"
#include "me_device.h"

namespace vfisv {

namespace {

// Orders this wave's LDS accesses (a workgroup is one wave, whose LDS
// operations complete in order: the compiler alone must not move them).
__device__ __forceinline__ void wave_fence() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

constexpr int NEQ = 64;               // chains of the normal equations
constexpr int CSTR = GROUP_PTS + 4;   // a quantity's points in LDS
constexpr int CN = NACC * CSTR;       // floats of a chunk's contributions
constexpr int ASTR = 33;              // row sums of a row
// dense: J [10], r, W J [10] over the 24 residuals (padded), JB pixels at a time
constexpr int DJ = 28, JB = 3, JPIX = (2 * NPAR + 1) * DJ;
static_assert(JB * JPIX <= CN, "J and W J fit the contributions' space");
// banded: a chunk's window is its 64 points behind the last 12 of the chunk
// before; J, r and W J over its 16 rows; VB slots' values summed together
constexpr int BROWS = 16, BJ = 4 * BROWS + 4, BPREV = BAND_S * (BAND_R - 1);
constexpr int WSTR = BPREV + GROUP_PTS + 8, WN = NACC * WSTR, VB = 4;
constexpr int BASTR = 36;  // row sums of a row: 16-byte rows on distinct banks
static_assert((2 * NPAR + 1) * BJ <= WN, "J and W J fit the window's space");

// Equilibrated normal equations of a slot's best model.
struct EqLds {
  double c[55];     // sc_p H_pq sc_q below the diagonal
  double b[NPAR];   // sc_p g_p
  double sc[NPAR];  // 1 / sqrt(H_pp), 0 for a frozen parameter
  float hg[66];     // H (packed) and g
};
struct alignas(16) ModelLds {
  float px[18];  // the fields of Pix that Weideman's series needs
  float rf[10];  // RowFactors
};
struct SlotLds : ModelLds {
  EqLds eq;
};

template <bool BAND>
struct Lds;
template <>
struct Lds<false> {
  double2 c2[(CN + 3) / 4];  // contributions [29][CSTR]; chi^2 terms; J and W J
  float a[JB * NOBS_HMI * ASTR];  // row sums
  float obs[GROUP_SLOTS[KIND_DENSE6]][2 * 4 * NOBS_HMI];  // observations, weights
  SlotLds slot[GROUP_SLOTS[KIND_DENSE6]];
};
template <>
struct Lds<true> {
  double2 c2[WN / 4];  // the window; values only: VB windows, or chi^2 terms, and the tails
  float a[BROWS * BASTR];  // row sums
  SlotLds slot[GROUP_SLOTS[KIND_BAND]];
};
constexpr int TSTR_D = 4 * NOBS_HMI + 1, TSTR_B = 4 * BROWS + 1;  // chi^2 terms of a slot
constexpr int TAIL_B = VB * 4 * WSTR;  // first tail: a slot's last 12 points, four quantities
static_assert(GROUP_SLOTS[KIND_DENSE6] * TSTR_D <= CN / 4, "chi^2 terms");
static_assert(4 * VB * TSTR_B <= TAIL_B && VB * BROWS * 4 <= BROWS * BASTR, "chi^2 terms");
static_assert(TAIL_B + GROUP_SLOTS[KIND_BAND] * 4 * BPREV <= WN, "values-only tails");
static_assert(GROUP_SLOTS[KIND_DENSE6] * NOBS_HMI <= 64 &&
                  GROUP_SLOTS[KIND_DENSE6] * NOBS_HMI * 4 <= JB * NOBS_HMI * ASTR,
              "values-only row sums of every slot");
static_assert(4 * CN >= (int)sizeof(double) * WS_DOUBLES, "the eigen fallback's record fits");
static_assert(sizeof(Lds<false>) <= 20480 && sizeof(Lds<true>) <= 20480, "eight waves on a CU");

// The normal equations as 64 independent chains of sums over the residuals:
// chain e < 55 is H's packed entry e = (p, q), chain 55 + p is g[p]; H's
// entry 30 (azimuth x S0) is zero by construction and its chain takes g[9].
// Column 10 of J is the residual itself.
__device__ __forceinline__ void chain_of(int e, int& p, int& q) {
  if (e == 30) {
    p = 9;
    q = NPAR;
  } else if (e >= 55) {
    p = e - 55;
    q = NPAR;
  } else {
    p = 0;
    while ((p + 1) * (p + 2) / 2 <= e) ++p;
    q = e - p * (p + 1) / 2;
  }
}
static_assert(pk_row(30) == 7 && pk_col(30) == 2 && hzero(0, 30) && hzero(1, 30) && hzero(2, 30) &&
                  hzero(3, 30),
              "entry 30 of H is zero");

__device__ __forceinline__ float fma4(float4 w, float4 c, float s) {
  return fmaf(w.w, c.w, fmaf(w.z, c.z, fmaf(w.y, c.y, fmaf(w.x, c.x, s))));
}
__device__ __forceinline__ float4 ld4(const float* p) { return *reinterpret_cast<const float4*>(p); }
__device__ __forceinline__ void st4(float* p, float a, float b, float c, float d) {
  *reinterpret_cast<float4*>(p) = make_float4(a, b, c, d);
}
// Nothing is scheduled across: the LDS loads of a block are all issued before
// their first use.  (Left to itself the compiler loads one value, waits out
// the LDS and uses it: 62 cycles per term of chi^2.)
__device__ __forceinline__ void issued() { __builtin_amdgcn_sched_barrier(0); }

// chi += the N terms term(0 ..), one after the other; the next LB are loaded meanwhile
template <int N, class F>
__device__ __forceinline__ double chi_chain(double chi, F term) {
  constexpr int LB = 8;
  static_assert(N % LB == 0, "whole blocks");
  double2 t[2][LB];
#pragma unroll
  for (int i = 0; i < LB; ++i) t[0][i] = term(i);
#pragma unroll
  for (int b = 0; b < N / LB; ++b) {
    if (b + 1 < N / LB) {
#pragma unroll
      for (int i = 0; i < LB; ++i) t[(b + 1) & 1][i] = term((b + 1) * LB + i);
    }
    issued();
#pragma unroll
    for (int i = 0; i < LB; ++i) chi = fma(t[b & 1][i].x, t[b & 1][i].y, chi);
    issued();
  }
  return chi;
}
// The same for an entry of H or g: N residuals, four of J and W J per load.
template <int N>
__device__ __forceinline__ float eq_chain(float h, const float* WJ, const float* J) {
  constexpr int LB = 4;
  float4 w[2][LB], j[2][LB];
  const auto load = [&](int b) {
#pragma unroll
    for (int i = 0; i < LB; ++i) {
      if (b * LB + i >= N / 4) continue;
      w[b & 1][i] = ld4(WJ + 4 * (b * LB + i));
      j[b & 1][i] = ld4(J + 4 * (b * LB + i));
    }
  };
  load(0);
#pragma unroll
  for (int b = 0; b * LB < N / 4; ++b) {
    if ((b + 1) * LB < N / 4) load(b + 1);
    issued();
#pragma unroll
    for (int i = 0; i < LB; ++i)
      if (b * LB + i < N / 4) h = fma4(w[b & 1][i], j[b & 1][i], h);
    issued();
  }
  return h;
}
__device__ __forceinline__ f32x4 mfma4(float a, float b, f32x4 c) {
  return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
}

__device__ __forceinline__ void put_model(ModelLds& S, const Pix& p, const RowFactors& f) {
  const float px[18] = {p.vsi, p.invD, p.zs, p.a,      p.denr, p.denr2, p.c0,  p.hs2,  p.hc,
                        p.hI,  p.hq,   p.hsin2g, p.hsg, p.s2h,  p.cgh,   p.eta0, p.alpha, p.oma};
  const float rf[10] = {f.S0, f.S1, f.alpha, f.S1a, f.c2p, f.s2p, f.fB, f.fg, f.fv, f.fD};
#pragma unroll
  for (int k = 0; k < 18; ++k) S.px[k] = px[k];
#pragma unroll
  for (int k = 0; k < 10; ++k) S.rf[k] = rf[k];
}
__device__ __forceinline__ Pix get_pix(const ModelLds& S) {
  Pix p;
  float* const f[18] = {&p.vsi, &p.invD, &p.zs,     &p.a,   &p.denr, &p.denr2, &p.c0,   &p.hs2,
                        &p.hc,  &p.hI,   &p.hq,     &p.hsin2g, &p.hsg, &p.s2h, &p.cgh,  &p.eta0,
                        &p.alpha, &p.oma};
#pragma unroll
  for (int k = 0; k < 18; ++k) *f[k] = S.px[k];
  p.ja = 0;
  p.a0 = p.da = 0.f;
  return p;
}
__device__ __forceinline__ RowFactors get_rf(const ModelLds& S) {
  RowFactors r;
  r.S0 = S.rf[0];
  r.S1 = S.rf[1];
  r.alpha = S.rf[2];
  r.S1a = S.rf[3];
  r.c2p = S.rf[4];
  r.s2p = S.rf[5];
  r.fB = S.rf[6];
  r.fg = S.rf[7];
  r.fv = S.rf[8];
  r.fD = S.rf[9];
  return r;
}

// Scale of parameter p in the equilibration of solve_cholesky.
__device__ __forceinline__ double scale_of(const EqLds& E, uint32_t free_mask, int p) {
  double maxd = 0.0;
#pragma unroll
  for (int k = 0; k < NPAR; ++k)
    if ((free_mask >> k) & 1u) maxd = fmax(maxd, (double)E.hg[pk(k, k)]);
  const double d = (double)E.hg[p * (p + 3) / 2];
  const bool act = ((free_mask >> p) & 1u) && maxd > 0.0 && d > 1e-30 * maxd;
  return act ? root_of(d).rl : 0.0;
}
// This lane's chain (p, q) of the equilibrated system.
__device__ __forceinline__ void scale_entry(EqLds& E, int e, int p, int q) {
  if (q < NPAR) E.c[e] = E.sc[p] * (double)E.hg[e] * E.sc[q];
  else E.b[p] = E.sc[p] * (double)E.hg[55 + p];
}

// The step of solve_cholesky from an equilibrated system.  Returns 0, 1 (left
// to solve_wave) or 2 (nothing free).
__device__ __forceinline__ int solve_equilibrated(const EqLds& E, double eps, double* delta) {
  double L[55], y[NPAR];
  bool any = false;
#pragma unroll
  for (int p = 0; p < NPAR; ++p) {
    const double sc = E.sc[p];
    any = any || sc != 0.0;
    delta[p] = 0.0;
    y[p] = E.b[p];
#pragma unroll
    for (int q = 0; q < p; ++q) L[pk(p, q)] = E.c[pk(p, q)];
    L[pk(p, p)] = (sc != 0.0) ? 1.0 + eps : 1.0;
  }
  if (!any) return 2;
  if (factor_solve(L, y) != 0) return 1;
#pragma unroll
  for (int p = 0; p < NPAR; ++p) delta[p] = rounded(E.sc[p] * y[p]);
  return 0;
}

// Slots of a mask, lowest first (wave-uniform), and its b-th slot per lane
// (b < 4; -1 if there is none).
__device__ __forceinline__ int first_slot(unsigned m) {
  return __builtin_amdgcn_readfirstlane(__ffs((int)m) - 1);
}
__device__ __forceinline__ int nth_slot(unsigned m, int b) {
#pragma unroll
  for (int i = 0; i < 3; ++i)
    if (b > i) m &= m - 1u;
  return __ffs((int)m) - 1;
}

// Residual and Jacobian row of Stokes parameter s (lane-dependent) of one
// observed sample from its row sums a: assemble_sample's operations for it.
__device__ __forceinline__ float assemble_one(const float* a, float rs, const RowFactors& f, int s,
                                              float ob, float* J) {
  const bool lin = s == 1 || s == 2;
  const float a2 = a[2], a3 = a[3], as = a[s == 0 ? 0 : 4];
  const float Q0 = f.S1a * a2, U0 = f.S1a * a3;
  const float SQ = fmaf(f.c2p, Q0, -f.s2p * U0), SU = fmaf(f.s2p, Q0, f.c2p * U0);
  const float cx = s == 1 ? f.c2p : f.s2p, cy = s == 1 ? -f.s2p : f.c2p;
  const float fx = s == 0 ? f.S1 : f.S1a;
  const float* d = a + 5 + (lin ? 1 : s);
  const float qf[6] = {f.fB, f.fg, f.fv, f.fD, 2.f, 1.f};
  const int qidx[6] = {0, 1, 3, 4, 5, 6};
#pragma unroll
  for (int q = 0; q < 6; ++q) {
    const float x = d[4 * q] * fx * qf[q];
    const float y = a[5 + 4 * q + 2] * f.S1a * qf[q];
    const float xy = fmaf(cx, x, cy * y);
    J[qidx[q]] = lin ? xy : x;
  }
  const float dpsi = s == 1 ? -2.f * DEG * SU : 2.f * DEG * SQ;
  J[2] = lin ? dpsi : 0.f;
  J[7] = s == 0 ? rs : 0.f;
  const float j8 = fmaf(cx, f.alpha * a2, cy * (f.alpha * a3));
  J[8] = lin ? j8 : s == 0 ? as : f.alpha * as;
  const float j9 = fmaf(cx, f.S1 * a2, cy * (f.S1 * a3));
  J[9] = lin ? j9 : f.S1 * a[s == 0 ? 1 : 4];
  const float SI = fmaf(f.S0, rs, f.S1 * as);
  const float r = ob - (lin ? (s == 1 ? SQ : SU) : SI);
  return s == 3 ? fmaf(-f.S1a, as, ob) : r;
}

// This lane's entry of H or g (keep: H stays).
__device__ __forceinline__ void store_entry(EqLds& E, float h, bool keep, int e, int p, int q) {
  if (q == NPAR) E.hg[55 + p] = h;
  else if (!keep) E.hg[e] = h;
  if (e == 0) E.hg[30] = 0.f;
}

// Equilibrates the slots of a mask, six at a time.
__device__ __forceinline__ void equilibrate(SlotLds* slot, unsigned jm, uint32_t free_mask,
                                            int lane, int ep, int eq) {
  wave_fence();
  for (unsigned m = jm; m != 0u;) {
    unsigned mk = m;
    const int i = lane / NPAR, p = lane - i * NPAR;
    for (int b = 0; b < i; ++b) mk &= mk - 1u;
    if (mk != 0u && i < 6) {
      EqLds& E = slot[__ffs((int)mk) - 1].eq;
      E.sc[p] = scale_of(E, free_mask, p);
    }
    wave_fence();
    for (int b = 0; b < 6 && m != 0u; ++b, m &= m - 1u) {
      EqLds& E = slot[first_slot(m)].eq;
      scale_entry(E, lane, ep, eq);
      if (lane == 0) E.c[30] = 0.0;
    }
  }
  wave_fence();
}

// The lane's number, recomputed from here on: what a pass derives from it (LDS
// addresses, rows) is not carried through the other passes in registers.
__device__ __forceinline__ int afresh(int lane) {
  asm volatile("" : "+v"(lane));
  return lane;
}

template <bool BAND>
struct Layout;

// ---- dense layout ----------------------------------------------------------
// At most 64 synthesis points: one per lane.  Values only, four slots' four
// quantities are the columns (with the five that a pass with derivatives sums,
// three slots: 65,536 pixels 3.73 ms instead of 3.58).  MFMA lane (col, kq) =
// (lane % 16, lane / 16) feeds tap A[row = col][point 4 i + kq] and quantity B[col] at that
// point in step i, and receives rows 4 kq .. + 3 of quantity col.
// The row sums of a launch in lane pairs (lm_kernel with two lanes per pixel)
// are those of the even and of the odd records, added: the odd ones take MFMA
// rows 8 .. 13.
template <>
struct Layout<false> {
  Lds<false>& S;
  const GroupArgs& ga;
  int lane, col, kq;
  float* const c;
  bool pair;
  float dl, tap[16], rs;
  int row;  // filter row in row slot lane % 6

  __device__ __forceinline__ int row_of(int q) const {
    const Consts& C = ga.A.C;
    int r = q;
    if (C.sw_k >= 0 && !pair) {
#pragma unroll
      for (int k = 0; k < NOBS_HMI; ++k)
        if (q == k) r = C.slot_row[k];
    }
    return r;
  }

  __device__ __forceinline__ Layout(Lds<false>& S_, const GroupArgs& g, int lane_, bool pair_)
      : S(S_), ga(g), lane(lane_), col(lane_ & 15), kq(lane_ >> 4),
        c(reinterpret_cast<float*>(S_.c2)), pair(pair_) {
    row = row_of(lane % NOBS_HMI);
    rs = g.A.C.row_sum[0];
#pragma unroll
    for (int k = 1; k < NOBS_HMI; ++k)
      if (row == k) rs = g.A.C.row_sum[k];
    dl = g.T.dl[lane];
    const int q = col & 7;
    const bool mine = q < NOBS_HMI && (col < 8 || pair);
    const float* w = g.T.taps + (mine ? row_of(q) : 0) * GROUP_PTS;
#pragma unroll
    for (int i = 0; i < 16; ++i)
      tap[i] = mine && (!pair || (kq & 1) == (col >> 3)) ? w[4 * i + kq] : 0.f;
  }

  __device__ __forceinline__ bool take(int k, int64_t pix) {
    constexpr int R = 4 * NOBS_HMI;
    const float* W = ga.A.W_pp ? ga.A.W + pix * R : ga.A.W;
    if (lane < R) S.obs[k][lane] = ga.A.stokes[pix * R + lane];
    else if (lane < 2 * R) S.obs[k][lane] = W[lane - R];
    return false;
  }

  __device__ __forceinline__ void store_rows(f32x4 v, float* a, int astr, int m, bool ok) const {
    if (pair) {
#pragma unroll
      for (int r = 0; r < 4; ++r) v[r] += __shfl_xor(v[r], 32);
    }
    if (ok && kq < 2) {
#pragma unroll
      for (int r = 0; r < 4; ++r)
        if (4 * kq + r < NOBS_HMI) a[(4 * kq + r) * astr + m] = v[r];
    }
  }

  // chi^2 (without 1/dof) of the slots in lm, each in its owner's lane
  __device__ __forceinline__ double values(unsigned lm, bool, int64_t, double) {
    lane = afresh(lane);
    col = lane & 15;
    kq = lane >> 4;
    for (unsigned m = lm; m != 0u;) {
      // four slots share the 16 columns of the MFMA
      const unsigned m0 = m;
#pragma unroll 1
      for (int b = 0; b < 4 && m != 0u; ++b, m &= m - 1u) {
        const Pix px = get_pix(S.slot[first_slot(m)]);
        float v[NACC];
        point_contrib<false>(dl, px, ga.A.C, v);
        const float u[4] = {v[0], v[2], v[3], v[4]};  // what the Stokes values need
#pragma unroll
        for (int k = 0; k < 4; ++k) c[(4 * b + k) * CSTR + lane] = u[k];
      }
      wave_fence();
      // columns without a slot read the first slot's points
      const int k = nth_slot(m0, col >> 2);
      const float* src = c + (k >= 0 ? col : 0) * CSTR + kq;
      float x[16];
#pragma unroll
      for (int i = 0; i < 16; ++i) x[i] = src[4 * i];
      issued();
      f32x4 acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int i = 0; i < 16; ++i) acc = mfma4(tap[i], x[i], acc);
      wave_fence();
      store_rows(acc, S.a + (k >= 0 ? k : 0) * (NOBS_HMI * 4), 4, col & 3, k >= 0);
    }
    wave_fence();
    double2* T = S.c2;
    const int k = lane / NOBS_HMI, q = lane - k * NOBS_HMI;
    if ((lm >> k) & 1u) {
      const float4 h = ld4(S.a + (k * NOBS_HMI + q) * 4);
      const float av[5] = {h.x, 0.f, h.y, h.z, h.w};
      const RowFactors rf = get_rf(S.slot[k]);
      float Sv[4], J[4][NPAR];
      assemble_sample<false>(av, rs, rf, Sv, J);
#pragma unroll
      for (int s = 0; s < 4; ++s) {
        const float r = S.obs[k][s * NOBS_HMI + row] - Sv[s];
        const float w = S.obs[k][(4 + s) * NOBS_HMI + row];
        T[k * TSTR_D + 4 * q + s] = make_double2((double)w * (double)r, (double)r);
      }
    }
    wave_fence();
    double chi = 0.0;
    if (lane < 32 && ((lm >> lane) & 1u)) {
      const double2* t = T + lane * TSTR_D;
      chi = chi_chain<4 * NOBS_HMI>(0.0, [&](int i) { return t[i]; });
    }
    wave_fence();
    return chi;
  }

  // Jacobian and equilibrated normal equations of the slots in jm; those in
  // keep leave H as it is (Sect. 4.4) and take the new gradient
  __device__ __forceinline__ void normal(unsigned jm, unsigned keep, int64_t, int cp, int cq) {
    lane = afresh(lane);
    col = lane & 15;
    kq = lane >> 4;
    for (unsigned m = jm; m != 0u;) {
      const unsigned m0 = m;
      int nb = 0;
#pragma unroll 1
      for (; nb < JB && m != 0u; ++nb, m &= m - 1u) {
        const Pix px = get_pix(S.slot[first_slot(m)]);
        {
          float v[NACC];
          point_contrib<true>(dl, px, ga.A.C, v);
#pragma unroll
          for (int k = 0; k < NACC; ++k) c[k * CSTR + lane] = v[k];
        }
        wave_fence();
        const float* s0 = c + col * CSTR + kq;
        const float* s1 = c + (col + 16 < NACC ? col + 16 : col) * CSTR + kq;
        f32x4 a0 = {0.f, 0.f, 0.f, 0.f}, a1 = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int h = 0; h < 16; h += 8) {
          float x[8], y[8];
#pragma unroll
          for (int i = 0; i < 8; ++i) {
            x[i] = s0[4 * (h + i)];
            y[i] = s1[4 * (h + i)];
          }
          issued();
#pragma unroll
          for (int i = 0; i < 8; ++i) {
            a0 = mfma4(tap[h + i], x[i], a0);
            a1 = mfma4(tap[h + i], y[i], a1);
          }
        }
        wave_fence();
        float* a = S.a + nb * (NOBS_HMI * ASTR);
        store_rows(a0, a, ASTR, col, true);
        store_rows(a1, a, ASTR, col + 16, col + 16 < NACC);
      }
      wave_fence();
      const int b = lane / NOBS_HMI, q = lane - b * NOBS_HMI;
      if (b < nb) {
        unsigned mb = m0;
        if (b > 0) mb &= mb - 1u;
        if (b > 1) mb &= mb - 1u;
        const int k = __ffs((int)mb) - 1;
        float a[NACC];
#pragma unroll
        for (int i = 0; i < NACC; ++i) a[i] = S.a[lane * ASTR + i];
        const RowFactors rf = get_rf(S.slot[k]);
        float Sv[4], J[4][NPAR], w[4];
        assemble_sample<true>(a, rs, rf, Sv, J);
#pragma unroll
        for (int s = 0; s < 4; ++s) w[s] = S.obs[k][(4 + s) * NOBS_HMI + row];
        float* Jt = c + b * JPIX + 4 * q;
        float* WJt = Jt + (NPAR + 1) * DJ;
#pragma unroll
        for (int p = 0; p < NPAR; ++p) {
          st4(Jt + p * DJ, J[0][p], J[1][p], J[2][p], J[3][p]);
          st4(WJt + p * DJ, w[0] * J[0][p], w[1] * J[1][p], w[2] * J[2][p], w[3] * J[3][p]);
        }
        float r[4];
#pragma unroll
        for (int s = 0; s < 4; ++s) r[s] = S.obs[k][s * NOBS_HMI + row] - Sv[s];
        st4(Jt + NPAR * DJ, r[0], r[1], r[2], r[3]);
      }
      wave_fence();
      unsigned mb = m0;
      for (int i = 0; i < nb; ++i, mb &= mb - 1u) {
        const float* Jt = c + i * JPIX + cq * DJ;
        const float* WJt = c + i * JPIX + (NPAR + 1 + cp) * DJ;
        const float h = eq_chain<4 * NOBS_HMI>(0.f, WJt, Jt);
        const int k0 = first_slot(mb);
        EqLds& E = S.slot[k0].eq;
        if (cq == NPAR || !((keep >> k0) & 1u)) E.hg[cq < NPAR ? lane : 55 + cp] = h;
        if (lane == 0) E.hg[30] = 0.f;
      }
      wave_fence();
      {
        const int i = lane / NPAR, p = lane - i * NPAR;
        if (i < nb) {
          unsigned mk = m0;
          if (i > 0) mk &= mk - 1u;
          if (i > 1) mk &= mk - 1u;
          EqLds& E = S.slot[__ffs((int)mk) - 1].eq;
          E.sc[p] = scale_of(E, ga.A.free_mask, p);
        }
      }
      wave_fence();
      mb = m0;
      for (int i = 0; i < nb; ++i, mb &= mb - 1u) {
        EqLds& E = S.slot[first_slot(mb)].eq;
        scale_entry(E, lane, cp, cq);
        if (lane == 0) E.c[30] = 0.0;
      }
      wave_fence();
    }
  }
};

// ---- banded layout ---------------------------------------------------------
// A chunk of 64 points is 16 blocks and completes 16 rows, whose 16 points
// each lie in the chunk's window.  Lane (jr, s) = (lane % 16, lane / 16) sums
// row jr over its points, a share s of the quantities, on the vector ALUs (a
// matrix product would spend its time on the zero taps of 76 points).
template <>
struct Layout<true> {
  Lds<true>& S;
  const GroupArgs& ga;
  int lane, jr, s;
  float* const c;

  __device__ __forceinline__ Layout(Lds<true>& S_, const GroupArgs& g, int lane_, bool)
      : S(S_), ga(g), lane(lane_), jr(lane_ & 15), s(lane_ >> 4),
        c(reinterpret_cast<float*>(S_.c2)) {}

  // Whether no weight of the pixel is negative (the running chi^2 never
  // falls then).
  __device__ __forceinline__ bool take(int, int64_t pix) {
    const int rows = 4 * ga.A.C.n_obs;
    const float* W = ga.A.W_pp ? ga.A.W + pix * rows : ga.A.W;
    bool ok = true;
    for (int r = lane; r < rows; r += 64) ok = ok && W[r] >= 0.f;
    return __ballot(!ok) == 0ull;
  }

  // Observed row that row jr of chunk ch completes, -1 if there is none.
  __device__ __forceinline__ int row_of(int ch) const {
    const int j = ch * BROWS - (BAND_R - 1) + jr;
    return j >= 0 && j < ga.A.C.n_obs ? j : -1;
  }
  struct Taps {
    float4 w[4];
  };
  __device__ __forceinline__ Taps load_taps(int j) const {
    Taps T;
#pragma unroll
    for (int i = 0; i < 4; ++i) T.w[i] = ld4(ga.T.taps + (j >= 0 ? j : 0) * 16 + 4 * i);
    return T;
  }
  // this lane's row summed over the window of one quantity
  __device__ __forceinline__ float row_sum(const Taps& T, const float* window) const {
    float a = 0.f;
#pragma unroll
    for (int i = 0; i < 4; ++i) a = fma4(T.w[i], ld4(window + 4 * (jr + i)), a);
    return a;
  }
  __device__ __forceinline__ int64_t pix_of(int64_t pix, int k) const {
    const unsigned lo = __shfl((unsigned)(pix & 0xffffffffll), k);
    const unsigned hi = __shfl((unsigned)(pix >> 32), k);
    return (int64_t)(((unsigned long long)hi << 32) | lo);
  }

  // chi^2 (without 1/dof) of the slots in lm, each in its owner's lane.  A
  // slot whose running sum has reached its bound (chi^2 of its best model) is
  // left there: with weights >= 0 the rest cannot bring it back below.
  __device__ __forceinline__ double values(unsigned lm, bool monotone, int64_t pix, double bound) {
    lane = afresh(lane);
    jr = lane & 15;
    s = lane >> 4;
    const int no = ga.A.C.n_obs;
    double2* T = S.c2;
    double chi = 0.0;
    float* const tail = c + TAIL_B;
    for (int i = lane; i < GROUP_SLOTS[KIND_BAND] * 4 * BPREV; i += 64) tail[i] = 0.f;
    const int pq = lane / BPREV, pp = lane - pq * BPREV;  // lanes < 48: a point of a tail
#pragma unroll 1
    for (int ch = 0; ch < ga.T.n_chunk && lm != 0u; ++ch) {
      const float dl = ga.T.dl[ch * GROUP_PTS + lane];
      const int j = row_of(ch);
      const Taps taps = load_taps(j);
      const float rs = j >= 0 ? ga.A.row_sums[j] : 0.f;
#pragma unroll 1
      for (unsigned m = lm; m != 0u;) {
        const unsigned m0 = m;
        // lane (jr, s) assembles row jr of the batch's slot s
        const int kb = nth_slot(m0, s);
        const int64_t pb = pix_of(pix, kb >= 0 ? kb : 0);
        float ob[4] = {}, wb[4] = {};
        if (kb >= 0 && j >= 0) {
          const float* o = ga.A.stokes + pb * (int64_t)(4 * no) + j;
          const float* W = (ga.A.W_pp ? ga.A.W + pb * (int64_t)(4 * no) : ga.A.W) + j;
#pragma unroll
          for (int i = 0; i < 4; ++i) {
            ob[i] = o[i * no];
            wb[i] = W[i * no];
          }
        }
        int nb = 0;
#pragma unroll 1
        for (; nb < VB && m != 0u; ++nb, m &= m - 1u) {
          const int k = first_slot(m);
          const Pix px = get_pix(S.slot[k]);
          float v[NACC];
          point_contrib<false>(dl, px, ga.A.C, v);
          // the quantities that the Stokes values need
          const float u[4] = {v[0], v[2], v[3], v[4]};
          float* const win = c + 4 * nb * WSTR;
          float* const last = tail + k * (4 * BPREV);
          if (lane < 4 * BPREV) win[pq * WSTR + pp] = last[lane];
#pragma unroll
          for (int i = 0; i < 4; ++i) {
            win[i * WSTR + BPREV + lane] = u[i];
            if (lane >= GROUP_PTS - BPREV) last[i * BPREV + lane - (GROUP_PTS - BPREV)] = u[i];
          }
        }
        wave_fence();
#pragma unroll 1
        for (int b = 0; b < nb; ++b)
          S.a[(b * BROWS + jr) * 4 + s] = row_sum(taps, c + (4 * b + s) * WSTR);
        wave_fence();
        if (kb >= 0) {
          const float4 h = ld4(S.a + lane * 4);
          const float a[5] = {h.x, 0.f, h.y, h.z, h.w};
          const RowFactors rf = get_rf(S.slot[kb]);
          float Sv[4], J[4][NPAR];
          assemble_sample<false>(a, rs, rf, Sv, J);
#pragma unroll
          for (int i = 0; i < 4; ++i) {
            const float r = ob[i] - Sv[i];
            T[s * TSTR_B + BROWS * i + jr] = j >= 0 ? make_double2((double)wb[i] * (double)r, (double)r)
                                                : make_double2(0.0, 0.0);
          }
        }
        wave_fence();
        const bool mine = lane < 32 && (((m0 & ~m) >> lane) & 1u);
        if (mine) {
          const double2* t = T + __popc(m0 & ((1u << lane) - 1u)) * TSTR_B;
#pragma unroll 1
          for (int b = 0; b < BROWS; b += 2)
            chi = chi_chain<8>(chi, [&](int i) { return t[BROWS * (i & 3) + (i >> 2) + b]; });
        }
        wave_fence();
        lm &= ~(unsigned)__ballot(mine && monotone && rounded(chi * ga.A.inv_dof) >= bound);
      }
    }
    return chi;
  }

  __device__ __forceinline__ void normal(unsigned jm, unsigned keep, int64_t pix, int ep, int eq) {
    lane = afresh(lane);
    jr = lane & 15;
    s = lane >> 4;
    const int no = ga.A.C.n_obs;
    const float* Jc = c + eq * BJ;
    const float* WJ = c + (NPAR + 1 + ep) * BJ;
    for (unsigned m = jm; m != 0u; m &= m - 1u) {
      const int k = first_slot(m);
      const int64_t pk_ = pix_of(pix, k);
      const float* o = ga.A.stokes + pk_ * (int64_t)(4 * no) + s * no;
      const float* W = (ga.A.W_pp ? ga.A.W + pk_ * (int64_t)(4 * no) : ga.A.W) + s * no;
      float h = 0.f;
      // the last 12 points of the chunk before, two float4 per lane
      const int i1 = lane + 64 < NACC * (BPREV / 4) ? lane + 64 : lane;
      float* const p0 = c + (lane / 3) * WSTR + 4 * (lane % 3);
      float* const p1 = c + (i1 / 3) * WSTR + 4 * (i1 % 3);
      float4 t0 = make_float4(0.f, 0.f, 0.f, 0.f), t1 = t0;
#pragma unroll 1
      for (int ch = 0; ch < ga.T.n_chunk; ++ch) {
        // lane (jr, s) assembles residual s of row jr
        const int j = row_of(ch);
        const Taps taps = load_taps(j);
        float ob = 0.f, w = 0.f, rs = 0.f;
        if (j >= 0) {
          ob = o[j];
          w = W[j];
          rs = ga.A.row_sums[j];
        }
        *reinterpret_cast<float4*>(p0) = t0;
        *reinterpret_cast<float4*>(p1) = t1;
        {
          const Pix px = get_pix(S.slot[k]);
          float v[NACC];
          point_contrib<true>(ga.T.dl[ch * GROUP_PTS + lane], px, ga.A.C, v);
#pragma unroll
          for (int i = 0; i < NACC; ++i) c[i * WSTR + BPREV + lane] = v[i];
        }
        wave_fence();
        {
          float v[8];
#pragma unroll
          for (int i = 0; i < 8; ++i) {
            const int q = 8 * s + i < NACC ? 8 * s + i : NACC - 1;
            v[i] = row_sum(taps, c + q * WSTR);
          }
          float* const a = S.a + jr * BASTR + 8 * s;
          st4(a, v[0], v[1], v[2], v[3]);
          st4(a + 4, v[4], v[5], v[6], v[7]);
        }
        t0 = ld4(p0 + GROUP_PTS);
        t1 = ld4(p1 + GROUP_PTS);
        wave_fence();
        {
          const RowFactors rf = get_rf(S.slot[k]);
          float J[NPAR];
          const float r = assemble_one(S.a + jr * BASTR, rs, rf, s, ob, J);
          float* Jt = c + 4 * jr + s;
#pragma unroll
          for (int p = 0; p < NPAR; ++p) {
            Jt[p * BJ] = j >= 0 ? J[p] : 0.f;
            Jt[(NPAR + 1 + p) * BJ] = j >= 0 ? w * J[p] : 0.f;
          }
          Jt[NPAR * BJ] = j >= 0 ? r : 0.f;
        }
        wave_fence();
        h = eq_chain<4 * BROWS>(h, WJ, Jc);
        wave_fence();
      }
      store_entry(S.slot[k].eq, h, (keep >> k) & 1u, lane, ep, eq);
    }
    equilibrate(S.slot, jm, ga.A.free_mask, lane, ep, eq);
  }
};

__device__ __forceinline__ unsigned long long wave_total(unsigned v) {
  for (int off = 32; off >= 1; off >>= 1) v += __shfl_xor(v, off);
  return v;
}

}  // namespace

template <bool BAND>
__global__ __launch_bounds__(64, 2) void lm_group_kernel(const GroupArgs ga) {
  __shared__ Lds<BAND> S;
  const LMArgs& A = ga.A;
  const unsigned long long n_total = A.n_dev ? *A.n_dev : (unsigned long long)A.n;
  const int lane = threadIdx.x;
  const bool serve = n_total <= (unsigned long long)ga.n_max;
  if (A.n_dev && blockIdx.x == 0 && lane == 0) A.work[GROUP_LEFT_SLOT] = serve ? 0ull : n_total;
  if (!serve) return;
  // the launch's own rule for lane pairs, whose sums differ by rounding
  const bool pair = A.lpp_max >= 2 && n_total <= (unsigned long long)A.pair_max;
  Layout<BAND> lay(S, ga, lane, pair);
  // as many slots as the launch's pixels fill: a wave's slots share its turns
  const unsigned long long fill = (n_total + gridDim.x - 1) / gridDim.x;
  const int slots = fill < (unsigned)GROUP_SLOTS[BAND] ? (int)fill : GROUP_SLOTS[BAND];
  const int rows = 4 * A.C.n_obs;
  int cp, cq;
  chain_of(lane, cp, cq);
  bool live = false, fresh = false, need_fb = false;
  // (waves beyond the pixels touch no queue and no counter)
  const bool idle = blockIdx.x >= n_total;
  bool exhausted = idle || lane >= slots;
  bool monotone = false;
  int64_t pix = 0;
  float Mb[NPAR], Mc[NPAR];
#pragma unroll
  for (int k = 0; k < NPAR; ++k) Mb[k] = Mc[k] = 0.f;
  double chib = 0.0, eps = 0.0;
  int it = 0;
  unsigned n_pix = 0, n_trial = 0, n_acc = 0, n_pass = 0, n_fb = 0, n_jac = 0, n_hess = 0;

  for (;;) {
    // ---- slots whose pixel has finished take the next -----------------------
    const unsigned long long nm = __ballot(!live && !exhausted);
    if (nm != 0ull) {
      unsigned long long k0 = 0;
      if (lane == 0) k0 = atomicAdd(&A.work[A.qbase], (unsigned long long)__popcll(nm));
      const unsigned k_lo = __builtin_amdgcn_readfirstlane((unsigned)(k0 & 0xffffffffull));
      const unsigned k_hi = __builtin_amdgcn_readfirstlane((unsigned)(k0 >> 32));
      if (!live && !exhausted) {
        const unsigned long long pos = (((unsigned long long)k_hi << 32) | k_lo) +
                                       (unsigned)__popcll(nm & ((1ull << lane) - 1ull));
        if (pos >= n_total) {
          exhausted = true;
        } else {
          pix = A.idx ? (int64_t)A.idx[pos] : (int64_t)pos;
          double M0[NPAR];
          if (A.init) {
#pragma unroll
            for (int k = 0; k < NPAR; ++k) M0[k] = (double)A.init[pix * NPAR + k];
          } else {
            const double d0[NPAR] = {1500.0, 90.0, 90.0, 0.0, 35.0, 0.25, 15.5, 0.3, 0.7, 0.6};
#pragma unroll
            for (int k = 0; k < NPAR; ++k) M0[k] = d0[k];
          }
          project(M0);
#pragma unroll
          for (int k = 0; k < NPAR; ++k) Mc[k] = (float)M0[k];
          live = true;
          fresh = true;
          eps = A.eps0;
          it = 0;
        }
      }
      for (unsigned m = (unsigned)__ballot(live && fresh); m != 0u; m &= m - 1u) {
        const int k = first_slot(m);
        const unsigned lo = __builtin_amdgcn_readlane((unsigned)(pix & 0xffffffffll), k);
        const unsigned hi = __builtin_amdgcn_readlane((unsigned)(pix >> 32), k);
        const bool f = lay.take(k, (int64_t)(((unsigned long long)hi << 32) | lo));
        if (lane == k) monotone = f;
      }
    }
    // ---- steps left by the solve, one slot at a time ------------------------
    for (unsigned fbm = (unsigned)__ballot(need_fb); fbm != 0u; fbm &= fbm - 1u) {
      const int L = first_slot(fbm);
      double* sws = reinterpret_cast<double*>(S.c2);
      const float* hg = S.slot[L].eq.hg;
      const bool eigen = solve_wave(hg, 1, hg + 55, 1, __shfl(eps, L), A.free_mask, sws, lane);
      if (lane == L) {
        if (eigen) ++n_fb;
        double Mt[NPAR];
#pragma unroll
        for (int k = 0; k < NPAR; ++k) Mt[k] = (double)Mb[k] + sws[200 + k];
        project(Mt);
#pragma unroll
        for (int k = 0; k < NPAR; ++k) Mc[k] = (float)Mt[k];
        need_fb = false;
      }
      __syncthreads();  // the step is read before the record is reused
    }
    const unsigned lm = (unsigned)__ballot(live);
    if (lm == 0u) break;

    // ---- the trials (or starts): chi^2 without derivatives ------------------
    if (live) {
      Pix px;
      RowFactors rf;
      pix_setup(Mc, A.C, px);
      row_factors(Mc, px, A.C, rf);
      put_model(S.slot[lane], px, rf);
    }
    wave_fence();
    const double chi =
        rounded(lay.values(lm, monotone, pix, fresh ? (double)INFINITY : chib) * A.inv_dof);
    bool want_j = false, keep_h = false;
    if (live) {
      ++n_pass;
      int done = -1;
      bool bad_input = false, new_best = true;
      if (fresh) {
        if (!isfinite(chi)) {
          done = 3;
          // a non-finite observation or weight: the pixel is not fitted
          const float* obs = A.stokes + pix * rows;
          const float* W = A.W_pp ? A.W + pix * rows : A.W;
          for (int r = 0; r < rows; ++r)
            bad_input = bad_input || !isfinite(obs[r]) || !isfinite(W[r]);
          if (bad_input) --n_pass;
        }
        chib = chi;
      } else {
        ++it;
        ++n_trial;
        new_best = isfinite(chi) && chi < chib;
        if (new_best) {
          const double dec = chib - chi;
          keep_h = chib < A.hess_reuse;
          chib = chi;
          eps = eps_down(eps);
          ++n_acc;
          if (dec < A.rel_tol * (chi + dec)) done = 0;
        } else {
          eps = eps_up(eps);
          if (eps > A.eps_max) done = 2;
        }
      }
      fresh = false;
      if (new_best) {
#pragma unroll
        for (int k = 0; k < NPAR; ++k) Mb[k] = Mc[k];
      }
      if (done < 0 && it >= A.max_iter) done = 1;
      if (done >= 0) {
        if (bad_input) {
#pragma unroll
          for (int k = 0; k < NPAR; ++k) A.params[pix * NPAR + k] = __builtin_nanf("");
          A.chi2[pix] = __builtin_nan("");
          A.iters[pix] = 0;
          if (A.status) A.status[pix] = 3;
        } else {
#pragma unroll
          for (int k = 0; k < NPAR; ++k) A.params[pix * NPAR + k] = Mb[k];
          A.chi2[pix] = chib;
          A.iters[pix] = it;
          if (A.status) A.status[pix] = done;
        }
        ++n_pix;
        if (it == 0) ++n_pass;  // ended at its start: see the passes below
        live = false;
      }
      want_j = live && new_best;
    }
    // ---- derivatives and normal equations of the new best models ------------
    const unsigned jm = (unsigned)__ballot(want_j);
    const unsigned keep = (unsigned)__ballot(want_j && keep_h);
    if (want_j) {
      ++n_jac;
      if (!keep_h) ++n_hess;
    }
    if (jm != 0u) lay.normal(jm, keep, pix, cp, cq);
    // ---- damped float64 steps from the best models --------------------------
    if (live) {
      double delta[NPAR];
      if (solve_equilibrated(S.slot[lane].eq, eps, delta) == 1) {
        need_fb = true;  // taken at the top of the next turn, by the whole wave
      } else {
        double Mt[NPAR];
#pragma unroll
        for (int k = 0; k < NPAR; ++k) Mt[k] = (double)Mb[k] + delta[k];
        project(Mt);
#pragma unroll
        for (int k = 0; k < NPAR; ++k) Mc[k] = (float)Mt[k];
      }
    }
    wave_fence();
  }
  const unsigned long long tp = wave_total(n_pix), tt = wave_total(n_trial), ta = wave_total(n_acc),
                           ts = wave_total(n_pass), tf = wave_total(n_fb), tj = wave_total(n_jac),
                           th = wave_total(n_hess);
  if (lane == 0 && !idle) {
    atomicAdd(&A.work[0], tj);
    atomicAdd(&A.work[1], tp);
    atomicAdd(&A.work[2], tt);
    atomicAdd(&A.work[3], ta);
    // trials, starts and Jacobians, of which a start's is no pass of its own
    atomicAdd(&A.work[4], ts + tj - tp);
    if (tf) atomicAdd(&A.work[5], tf);
    atomicAdd(&A.work[6], 1ull);
    atomicAdd(&A.work[7], th);
    atomicAdd(&A.work[8], tj);
  }
}

// ---- synthesis -------------------------------------------------------------
// The filtered Stokes vectors (and Jacobians) of given models by the same
// split: a point per lane, `per` models per wave, whose set-up the lanes share
// out.  A model per lane (synth_kernel) takes one lane's pass over all points
// however few models there are, one wave per SIMD that waits out its own
// latencies up to 65,536 models.  Bound by VALU issue from there on (620 wave
// instructions per HMI model with its Jacobian, 2,100 per fine spectrum).
// Measured, a model per lane -> here: 1,000 HMI models with Jacobian 66 -> 11
// us, 65,537 170 -> 88; 30,011 fine spectra 425 -> 97, with Jacobian 599 ->
// 363.  (Jacobian rows through LDS, to store whole lines, take as long.)
// Through filters that leave a chunk partly empty a model per lane is faster
// from some thousands of models on (routes.h).
namespace {

constexpr int SYNTH_PER[2] = {32, 16};  // most models of a wave, per layout
constexpr int DV = 8;                   // dense, values only: models assembled together
static_assert(DV * NOBS_HMI <= 64 && DV % 4 == 0, "lanes of the assembly");

// Row sums over the points with taps alone, for models whose contributions
// are not all finite (a zero tap is no tap); columns m < n of c, rows of a.
__device__ __noinline__ void sums_of_taps(const float* taps, const float* c, int n, float* a,
                                          int astr, int cols, int lane) {
  const int m = lane & 31;
  if (m < n) {
#pragma unroll 1
    for (int r = lane >> 5; r < NOBS_HMI; r += 2) {
      float s = 0.f;
#pragma unroll 1
      for (int k = 0; k < GROUP_PTS; ++k) {
        const float w = taps[r * GROUP_PTS + k];
        if (w != 0.f) s = fmaf(w, c[m * CSTR + k], s);
      }
      a[(m / cols) * (NOBS_HMI * astr) + r * astr + m % cols] = s;
    }
  }
}
__device__ __forceinline__ bool all_finite(f32x4 v) {
  return __ballot(!isfinite((v[0] + v[1]) + (v[2] + v[3]))) == 0ull;
}

__device__ __forceinline__ void setup_models(const SynthArgs& A, ModelLds* rec, int64_t first,
                                             int n, int lane) {
  if (lane < n) {
    float M[NPAR];
#pragma unroll
    for (int q = 0; q < NPAR; ++q) M[q] = A.params[(first + lane) * NPAR + q];
    Pix px;
    RowFactors rf;
    pix_setup(M, A.C, px);
    row_factors(M, px, A.C, rf);
    put_model(rec[lane], px, rf);
  }
  wave_fence();
}

__device__ __forceinline__ void store_jac(float* J, const float* v) {
#pragma unroll
  for (int p = 0; p < NPAR; ++p) J[p] = v[p];
}

}  // namespace

// Dense: the rows of four models' values, or of one model's 29 quantities,
// are one or two chains of 16 MFMAs (Layout<false>).
template <bool DERIV>
__global__ __launch_bounds__(64, DERIV ? 3 : 4) void synth_group_kernel(const SynthArgs A,
                                                                        const GroupTables T,
                                                                        int per) {
  constexpr int NB = DERIV ? 2 : DV, NC = DERIV ? NACC : 16, AS = DERIV ? ASTR : 4;
  __shared__ __align__(16) float c[NC * CSTR];
  __shared__ __align__(16) float a[NB * NOBS_HMI * AS];
  __shared__ ModelLds rec[SYNTH_PER[KIND_DENSE6]];
  const int lane = threadIdx.x, col = lane & 15, kq = lane >> 4;
  const int64_t first = (int64_t)blockIdx.x * per;
  const int n = (int)(A.n - first < per ? A.n - first : per);
  const float dl = T.dl[lane];
  float tap[16];
#pragma unroll
  for (int i = 0; i < 16; ++i) {
    const float w = T.taps[(col < NOBS_HMI ? col : 0) * GROUP_PTS + 4 * i + kq];
    tap[i] = col < NOBS_HMI ? w : 0.f;
  }
  // assembly: lane (model, Stokes parameter, row), the order of the outputs,
  // or (model, row) without derivatives
  constexpr int LM = DERIV ? 4 * NOBS_HMI : NOBS_HMI;
  const int b = lane / LM, t = lane - b * LM, st = t / NOBS_HMI, row = t - st * NOBS_HMI;
  float rs = A.C.row_sum[0];
#pragma unroll
  for (int k = 1; k < NOBS_HMI; ++k)
    if (row == k) rs = A.C.row_sum[k];
  setup_models(A, rec, first, n, lane);
#pragma unroll 1
  for (int k0 = 0; k0 < n; k0 += NB) {
    const bool mine = b < NB && k0 + b < n;
    const int64_t out = (first + k0 + b) * (4 * NOBS_HMI) + t;
    float noise[DERIV ? 1 : 4] = {};
    if (A.noise && mine) {
#pragma unroll
      for (int i = 0; i < (DERIV ? 1 : 4); ++i) noise[i] = A.noise[out + i * NOBS_HMI];
    }
    if constexpr (DERIV) {
#pragma unroll 1
      for (int i = 0; i < NB && k0 + i < n; ++i) {
        {
          const Pix px = get_pix(rec[k0 + i]);
          float v[NACC];
          point_contrib<true>(dl, px, A.C, v);
#pragma unroll
          for (int q = 0; q < NACC; ++q) c[q * CSTR + lane] = v[q];
        }
        wave_fence();
        const float* s0 = c + col * CSTR + kq;
        const float* s1 = c + (col + 16 < NACC ? col + 16 : col) * CSTR + kq;
        f32x4 a0 = {0.f, 0.f, 0.f, 0.f}, a1 = a0;
#pragma unroll
        for (int h = 0; h < 16; h += 8) {
          float x[8], y[8];
#pragma unroll
          for (int j = 0; j < 8; ++j) {
            x[j] = s0[4 * (h + j)];
            y[j] = s1[4 * (h + j)];
          }
          issued();
#pragma unroll
          for (int j = 0; j < 8; ++j) {
            a0 = mfma4(tap[h + j], x[j], a0);
            a1 = mfma4(tap[h + j], y[j], a1);
          }
        }
        float* const ai = a + i * (NOBS_HMI * AS);
        if (kq < 2) {
#pragma unroll
          for (int r = 0; r < 4; ++r) {
            if (4 * kq + r >= NOBS_HMI) continue;
            ai[(4 * kq + r) * AS + col] = a0[r];
            if (col + 16 < NACC) ai[(4 * kq + r) * AS + col + 16] = a1[r];
          }
        }
        if (!all_finite(a0) || !all_finite(a1))
          sums_of_taps(T.taps, c, NACC, ai, AS, NACC, lane);
        wave_fence();
      }
      if (mine) {
        const RowFactors rf = get_rf(rec[k0 + b]);
        float J[NPAR];
        const float r = assemble_one(a + (b * NOBS_HMI + row) * AS, rs, rf, st, 0.f, J);
        A.stokes[out] = A.noise ? plus_noise(-r, noise[0]) : -r;
        store_jac(A.jac + out * NPAR, J);
      }
    } else {
#pragma unroll 1
      for (int h = 0; h < NB && k0 + h < n; h += 4) {
#pragma unroll 1
        for (int i = 0; i < 4 && k0 + h + i < n; ++i) {
          const Pix px = get_pix(rec[k0 + h + i]);
          float v[NACC];
          point_contrib<false>(dl, px, A.C, v);
          const float u[4] = {v[0], v[2], v[3], v[4]};  // what the Stokes values need
#pragma unroll
          for (int q = 0; q < 4; ++q) c[(4 * i + q) * CSTR + lane] = u[q];
        }
        wave_fence();
        const int cols = 4 * (n - k0 - h < 4 ? n - k0 - h : 4);
        const float* src = c + (col < cols ? col : 0) * CSTR + kq;
        float x[16];
#pragma unroll
        for (int j = 0; j < 16; ++j) x[j] = src[4 * j];
        issued();
        f32x4 s = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int j = 0; j < 16; ++j) s = mfma4(tap[j], x[j], s);
        float* const ah = a + h * (NOBS_HMI * AS);
        if (kq < 2 && col < cols) {
#pragma unroll
          for (int r = 0; r < 4; ++r)
            if (4 * kq + r < NOBS_HMI)
              ah[((col >> 2) * NOBS_HMI + 4 * kq + r) * AS + (col & 3)] = s[r];
        }
        if (!all_finite(s)) sums_of_taps(T.taps, c, cols, ah, AS, 4, lane);
        wave_fence();
      }
      if (mine) {
        const float4 h = ld4(a + lane * AS);
        const float av[5] = {h.x, 0.f, h.y, h.z, h.w};
        const RowFactors rf = get_rf(rec[k0 + b]);
        float Sv[4], J[4][NPAR];
        assemble_sample<false>(av, rs, rf, Sv, J);
#pragma unroll
        for (int i = 0; i < 4; ++i)
          A.stokes[out + i * NOBS_HMI] = A.noise ? plus_noise(Sv[i], noise[i]) : Sv[i];
      }
    }
    wave_fence();
  }
}

// Banded: a chunk's 16 rows over its window (Layout<true>), the values of VB
// models at a time.
template <bool DERIV>
__global__ __launch_bounds__(64, DERIV ? 3 : 4) void synth_group_band_kernel(const SynthArgs A,
                                                                             const GroupTables T,
                                                                             int per) {
  constexpr int NB = DERIV ? 1 : VB, NW = DERIV ? NACC : 4 * VB;
  __shared__ __align__(16) float c[NW * WSTR];
  __shared__ __align__(16) float tail[NW * BPREV];
  __shared__ __align__(16) float a[BROWS * (DERIV ? BASTR : 4 * VB)];
  __shared__ ModelLds rec[SYNTH_PER[KIND_BAND]];
  const int lane = threadIdx.x, jr = lane & 15, s = lane >> 4, no = A.C.n_obs;
  const int64_t first = (int64_t)blockIdx.x * per;
  const int n = (int)(A.n - first < per ? A.n - first : per);
  setup_models(A, rec, first, n, lane);
#pragma unroll 1
  for (int k0 = 0; k0 < n; k0 += NB) {
    for (int i = lane; i < NW * BPREV; i += 64) tail[i] = 0.f;
    wave_fence();
    const int nb = n - k0 < NB ? n - k0 : NB;
    // values: lane (jr, s) assembles row jr of model s; derivatives: row jr of
    // Stokes parameter s
    const int kb = DERIV ? k0 : k0 + (s < nb ? s : 0);
    const int64_t base = (first + kb) * (int64_t)(4 * no) + (DERIV ? s * no : 0);
#pragma unroll 1
    for (int ch = 0; ch < T.n_chunk; ++ch) {
      const float dl = T.dl[ch * GROUP_PTS + lane];
      const int j0 = ch * BROWS - (BAND_R - 1) + jr;
      const bool valid = j0 >= 0 && j0 < no, mine = valid && (DERIV || s < nb);
      const int j = valid ? j0 : 0;
      float4 w[4];
#pragma unroll
      for (int i = 0; i < 4; ++i) w[i] = ld4(T.taps + j * 16 + 4 * i);
      const float rs = A.row_sums[j];
      float noise[DERIV ? 1 : 4] = {};
      if (A.noise && mine) {
#pragma unroll
        for (int i = 0; i < (DERIV ? 1 : 4); ++i) noise[i] = A.noise[base + i * no + j];
      }
      for (int i = lane; i < NW * (BPREV / 4); i += 64)
        *reinterpret_cast<float4*>(c + (i / (BPREV / 4)) * WSTR + 4 * (i % (BPREV / 4))) =
            ld4(tail + 4 * i);
      wave_fence();
      const auto row_sum = [&](const float* window) {
        float4 x[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) x[i] = ld4(window + 4 * (jr + i));
        float r = 0.f;
#pragma unroll
        for (int i = 0; i < 4; ++i) r = fma4(w[i], x[i], r);
        return r;
      };
#pragma unroll 1
      for (int b = 0; b < nb; ++b) {
        const Pix px = get_pix(rec[k0 + b]);
        float v[NACC];
        point_contrib<DERIV>(dl, px, A.C, v);
        if constexpr (!DERIV) {  // what the Stokes values need
          v[1] = v[2];
          v[2] = v[3];
          v[3] = v[4];
        }
        constexpr int NQ = DERIV ? NACC : 4;
#pragma unroll
        for (int i = 0; i < NQ; ++i) c[(NQ * b + i) * WSTR + BPREV + lane] = v[i];
        if (lane >= GROUP_PTS - BPREV) {
#pragma unroll
          for (int i = 0; i < NQ; ++i)
            tail[(NQ * b + i) * BPREV + lane - (GROUP_PTS - BPREV)] = v[i];
        }
      }
      wave_fence();
      if constexpr (DERIV) {
        float r[8];
#pragma unroll
        for (int i = 0; i < 8; ++i) r[i] = row_sum(c + (8 * s + i < NACC ? 8 * s + i : NACC - 1) * WSTR);
        st4(a + jr * BASTR + 8 * s, r[0], r[1], r[2], r[3]);
        st4(a + jr * BASTR + 8 * s + 4, r[4], r[5], r[6], r[7]);
        wave_fence();
        if (mine) {
          const RowFactors rf = get_rf(rec[k0]);
          float J[NPAR];
          const float x = assemble_one(a + jr * BASTR, rs, rf, s, 0.f, J);
          A.stokes[base + j] = A.noise ? plus_noise(-x, noise[0]) : -x;
          store_jac(A.jac + (base + j) * NPAR, J);
        }
      } else {
#pragma unroll 1
        for (int b = 0; b < nb; ++b)
          a[(b * BROWS + jr) * 4 + s] = row_sum(c + (4 * b + s) * WSTR);
        wave_fence();
        if (mine) {
          const float4 h = ld4(a + lane * 4);
          const float av[5] = {h.x, 0.f, h.y, h.z, h.w};
          const RowFactors rf = get_rf(rec[kb]);
          float Sv[4], J[4][NPAR];
          assemble_sample<false>(av, rs, rf, Sv, J);
#pragma unroll
          for (int i = 0; i < 4; ++i)
            A.stokes[base + i * no + j] = A.noise ? plus_noise(Sv[i], noise[i]) : Sv[i];
        }
      }
      wave_fence();
    }
  }
}

template <class K>
static void launch_synth_pieces(K kernel, const SynthArgs& a, const GroupTables& t, int64_t per,
                                hipStream_t s) {
  // (a launch takes less than 2^32 lanes)
  constexpr int64_t MAX_GRID = (int64_t)1 << 25;
  const int64_t row = 4 * (int64_t)a.C.n_obs;
  for (int64_t first = 0; first < a.n; first += MAX_GRID * per) {
    SynthArgs p = a;
    p.n = a.n - first < MAX_GRID * per ? a.n - first : MAX_GRID * per;
    p.params += first * NPAR;
    p.stokes += first * row;
    if (p.noise) p.noise += first * row;
    if (p.jac) p.jac += first * row * NPAR;
    kernel<<<(int)((p.n + per - 1) / per), 64, 0, s>>>(p, t, (int)per);
  }
}

hipError_t launch_synth_group(const SynthArgs& a, const GroupTables& t, int kind, bool deriv,
                              int num_cus, hipStream_t s) {
  // as many models per wave as leave the chip its waves (12 or 16 with
  // Jacobian: 65,537 HMI models 106 or 119 us instead of 100)
  const int64_t waves = (int64_t)num_cus * (deriv ? 8 : 16);
  int64_t per = (a.n + waves - 1) / waves;
  if (per > SYNTH_PER[kind]) per = SYNTH_PER[kind];
  if (kind == KIND_BAND) {
    if (deriv) launch_synth_pieces(synth_group_band_kernel<true>, a, t, per, s);
    else launch_synth_pieces(synth_group_band_kernel<false>, a, t, per, s);
  } else {
    if (deriv) launch_synth_pieces(synth_group_kernel<true>, a, t, per, s);
    else launch_synth_pieces(synth_group_kernel<false>, a, t, per, s);
  }
  return hipGetLastError();
}

hipError_t launch_lm_group(const GroupArgs& a, int kind, int grid, hipStream_t s) {
  if (kind == KIND_BAND) lm_group_kernel<true><<<grid, 64, 0, s>>>(a);
  else lm_group_kernel<false><<<grid, 64, 0, s>>>(a);
  return hipGetLastError();
}

hipError_t lm_group_blocks_per_cu(int kind, int* out) {
  return hipOccupancyMaxActiveBlocksPerMultiprocessor(
      out, kind == KIND_BAND ? (const void*)lm_group_kernel<true> : (const void*)lm_group_kernel<false>,
      64, 0);
}

}  // namespace vfisv

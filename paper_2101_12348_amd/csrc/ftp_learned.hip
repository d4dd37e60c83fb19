// Learned root proposal (a project addition to the method): Newton on the
// real phase polynomial from network seeds, verified by a Sturm count.
//
// For each frequency:
//   * the number of distinct real roots of R is counted with a Sturm sequence
//     of the Cayley polynomial f(x) (theta = phi0 + 2 atan x) over the whole
//     real line;
//   * if the count is well determined, 2H network seeds plus evenly spaced
//     starts (only evenly spaced starts for the ablation without network) are
//     refined by FP64 Newton on R(theta) = 2 MM dYM/dtheta - YM dMM/dtheta
//     (Eq. theta2cond written as R(theta) = i e^{-i K theta} p(e^{i theta})),
//     each step evaluated on the Cayley polynomial f with the iterate kept as
//     tan((theta - phi0) / 2) or its reciprocal (newton_u_step); converged
//     roots closer than 1e-8 rad are merged, one root per pass, after every
//     iteration from the second that leaves as many converged, and Newton stops
//     once the merged roots reach the count;
//   * if they do, the Newton roots are the candidate set; otherwise the
//     frequency goes to the Aberth iteration (then, if that does not
//     converge, to the companion-matrix solve) through device work lists.
// For H <= 10 a wavefront takes up to eight frequencies (k_newton_sturm4): their
// Sturm sequences run one per group of eight or sixteen lanes with up to eight
// coefficients per lane in registers, and Newton runs on two of them at a time (32
// starts each, at most D).  For H = 11 a wavefront takes one (k_newton_sturm, 4H
// starts), its Sturm sequence one coefficient per lane (the degree-64 coefficient
// carried as a scalar; see sturm_begin); above, up to four whose sequences run in
// double-double, a 16-lane row each (sturm_count_dd).
#include <hip/hip_ext.h>
#include "ftp_solve_common.h"
#include "ftp_args.h"

namespace ftp {

__device__ __forceinline__ void lwave_sync() {
  __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
  __builtin_amdgcn_wave_barrier();
}

__device__ __forceinline__ double lrdlane(double v, int src) {
  const unsigned long long u = (unsigned long long)__double_as_longlong(v);
  const int lo = __builtin_amdgcn_readlane((int)(unsigned)(u & 0xffffffffull), src);
  const int hi = __builtin_amdgcn_readlane((int)(unsigned)(u >> 32), src);
  return __longlong_as_double((long long)(((unsigned long long)(unsigned)hi << 32) | (unsigned)lo));
}

__device__ __forceinline__ double sgn(double x) { return x > 0.0 ? 1.0 : (x < 0.0 ? -1.0 : 0.0); }

__device__ __forceinline__ int hiword(double x) {
  return (int)((unsigned long long)__double_as_longlong(x) >> 32);
}
__device__ __forceinline__ double from_hiword(int h) {
  return __longlong_as_double((long long)((unsigned long long)(unsigned)h << 32));
}

// Thresholds of the Sturm test, applied to high words of positive doubles: a
// difference of high words is 2^20 log2 of the ratio to within 0.09 (the
// mantissa enters linearly), so "ratio above 1e-12" reads hi(x) - hi(y) >
// hi(1) - hi(1e-12), to within 7% of the bound.  hi(NaN) and hi(inf) are at
// least 0x7ff00000.
constexpr int kHi1 = 0x3ff00000;
constexpr int kHiT12 = kHi1 - 0x3d719799;   // hi(1) - hi(1e-12)
constexpr int kHiT13 = kHi1 - 0x3d3c25c2;   // hi(1) - hi(1e-13)

// Maximum of an int over the wavefront (row stages, then row_bcast:15 and
// row_bcast:31 into lane 63).
__device__ __forceinline__ int wave_max_int(int h) {
  h = max(h, dpp_i<0xB1, 0xf>(h));
  h = max(h, dpp_i<0x4E, 0xf>(h));
  h = max(h, dpp_i<0x141, 0xf>(h));
  h = max(h, dpp_i<0x140, 0xf>(h));
  h = max(h, dpp_i<0x142, 0xa>(h));
  h = max(h, dpp_i<0x143, 0xc>(h));
  return __builtin_amdgcn_readlane(h, 63);
}

// The test of one Sturm step on high words: hr = hi(max |t|) of the
// remainder, hl = hi(|leading coefficient of t|), hM = hi of the larger of
// the two members' largest coefficient magnitudes.  The remainder must not
// vanish against the members (max |t| above 1e-12 of theirs: else a gcd of
// positive degree, repeated or nearly repeated roots) nor lose its leading
// term to cancellation (above 1e-13 of max |t|), and must be finite.
__device__ __forceinline__ bool sturm_step_ok(int hr, int hl, int hM) {
  return (hr < 0x7ff00000) & (hr - hM > -kHiT12) & (hl - hr > -kHiT13);
}
// hi(max |P_q|) of the scaled member P_q = -t / |lead|: hr - hl + hi(1)
// (bounded so that a failed chain's value stays an int)
__device__ __forceinline__ int sturm_member_hi(int hr, int hl) { return min(hr - hl, 0x40000000) + kHi1; }

// Sturm sequence of a degree-D polynomial g over the whole real line, D + 1
// <= 64, in registers: P_0 = g, P_1 = g', P_q = -rem(P_{q-2}, P_{q-1}), lane c
// holding coefficient c (the shift by one power of x is a DPP lane shift).
// Each member is scaled by the reciprocal of its leading coefficient's
// magnitude (P_0 and P_1 with their leading lane set to +-1): a positive scale
// leaves the signs, and so the count, unchanged, and the quotient of each
// division is taken as al bl x + (next coefficient) bl with al, bl = +-1 and no
// division (a member's leading coefficient is +-1 to within the reciprocal's
// few ulp, which perturbs the quotient by as much: the size of the rounding
// already present).  Every member of a generic sequence has degree D - q, so
// its signs at +inf and -inf are those of its leading coefficient (times
// (-1)^(D - q) at -inf), and the count V(-inf) - V(+inf) accumulates as the
// members are formed; consecutive members differ in degree by one, so at -inf
// a sign change occurs exactly where none occurs at +inf, and with V(+inf) =
// vp over the D transitions of a full chain the count is D - 2 vp.  Each step
// is tested (sturm_step_ok); a chain that fails is not trusted.
struct SturmChain {
  double A, B, al, bl;  // the last two members and their leading coefficients (+-1)
  int hMA, hMB;         // hi(max |coefficient|) of A and B
  int sp;               // last member positive at +inf (0 / 1)
  int vp;               // sign changes at +inf so far
  bool ok;
};

// gv: coefficient `lane` of g (lanes 0..min(D, 63)); gtop = g[D].  For D = 64
// the top coefficient has no lane: it is carried as the scalar leading
// coefficient only, which is all the chain needs of it (the first remainder
// cancels it exactly and the shifted derivative reaches lane 63 at most).
__device__ __forceinline__ SturmChain sturm_begin(double gv, double gtop, int D, int lane) {
  SturmChain c;
  const double gnext = lane_shl1(gv);   // g[lane + 1], taken with every lane active
  const double g1 = lane == 63 ? gtop : gnext;
  const double dv = lane < D ? (lane + 1) * g1 : 0.0;
  const double ag = fabs(gtop), sgn = gtop > 0.0 ? 1.0 : -1.0;
  const double sa = fast_rcp_d(ag + 1e-300), sb = fast_rcp_d(D * ag + 1e-300);
  c.ok = ag > 0.0 && ag < INFINITY;
  c.A = lane == D ? sgn : gv * sa;
  c.B = lane == D - 1 ? sgn : dv * sb;
  c.al = sgn;
  c.bl = sgn;
  c.hMA = max(wave_max_int(hiword(c.A) & 0x7fffffff), kHi1);   // the top of A is +-1 (no lane at D = 64)
  c.hMB = wave_max_int(hiword(c.B) & 0x7fffffff);
  c.vp = 0;
  c.sp = gtop > 0.0 ? 1 : 0;
  return c;
}

// Member q (2 <= q <= D) from the last two (every lane holds one chain).
// Branch-free, so that two chains stepped side by side interleave.
__device__ __forceinline__ void sturm_step(SturmChain& c, int D, int q, int lane) {
  const int db = D - q + 1;
  double t = c.A - (c.al * c.bl) * lane_shr1(c.B);
  const double q0 = lrdlane(t, db) * c.bl;
  t = lane < db ? t - q0 * c.B : 0.0;
  const double lead = lrdlane(t, db - 1);
  const int hl = hiword(lead), hla = hl & 0x7fffffff;
  const int hr = wave_max_int(hiword(t) & 0x7fffffff);
  c.ok = c.ok && sturm_step_ok(hr, hla, max(c.hMA, c.hMB));
  // P_q = -t / |lead|: positive at +inf when lead < 0 (sign bit of hl)
  const int tp = (int)((unsigned)hl >> 31);
  c.vp += tp ^ c.sp;
  c.sp = tp;
  const double s = fast_rcp_d(fabs(lead) + 1e-300);
  c.A = c.B;
  c.al = c.bl;
  c.hMA = c.hMB;
  c.B = -t * s;
  c.bl = from_hiword((hl & 0x80000000) ^ 0xbff00000);   // -sign(lead)
  c.hMB = sturm_member_hi(hr, hla);
}

// Distinct real roots of g (coefficient `gv` in lane c, gtop = g[D] != 0,
// D <= 64), or -1; `raw` receives the count whether or not the chain passed
// its tests (a diagnostic).
__device__ int sturm_count_line_reg(double gv, double gtop, int D, int lane, int& raw) {
  SturmChain c = sturm_begin(gv, gtop, D, lane);
  for (int q = 2; q <= D; ++q) sturm_step(c, D, q, lane);
  raw = D - 2 * c.vp;
  return c.ok ? raw : -1;
}

// ---- double-double arithmetic (value hi + lo, |lo| <= ulp(hi) / 2): the
// error-free transformations of Knuth (TAOCP vol. 2, two-sum) and Dekker
// (1971, the product, here through the fused multiply-add).  Contraction of
// a product into a later sum is off in these helpers: the error terms assume
// each operation rounded on its own (a fused p + e in the product's
// normalisation drops the double-double precision to double's).
struct dd { double hi, lo; };
__device__ __forceinline__ dd dd_two_sum(double a, double b) {
#pragma clang fp contract(off)
  const double s = a + b, bb = s - a;
  return dd{s, (a - (s - bb)) + (b - bb)};
}
__device__ __forceinline__ dd dd_quick(double a, double b) {   // |a| >= |b|
#pragma clang fp contract(off)
  const double s = a + b;
  return dd{s, b - (s - a)};
}
__device__ __forceinline__ dd dd_add(dd x, dd y) {
#pragma clang fp contract(off)
  dd s = dd_two_sum(x.hi, y.hi);
  const dd t = dd_two_sum(x.lo, y.lo);
  s.lo += t.hi;
  s = dd_quick(s.hi, s.lo);
  s.lo += t.lo;
  return dd_quick(s.hi, s.lo);
}
__device__ __forceinline__ dd dd_neg(dd x) { return dd{-x.hi, -x.lo}; }
__device__ __forceinline__ dd dd_mul(dd x, dd y) {
#pragma clang fp contract(off)
  const double p = x.hi * y.hi;
  double e = fma(x.hi, y.hi, -p);
  e = fma(x.hi, y.lo, fma(x.lo, y.hi, e));
  return dd_quick(p, e);
}
// 1 / y: the double reciprocal and one correction (y hi + lo).
__device__ __forceinline__ dd dd_rcp(dd y) {
#pragma clang fp contract(off)
  const double r = fast_rcp_d(y.hi);
  const double e = fma(-y.lo, r, fma(-y.hi, r, 1.0));   // relative error of r, about an ulp
  return dd_quick(r, r * e);
}
__device__ __forceinline__ dd dd_ldexp(dd x, int e) { return dd{ldexp(x.hi, e), ldexp(x.lo, e)}; }
// v from lane addr / 4 (ds_bpermute, all lanes active)
__device__ __forceinline__ double bperm_d(int addr, double v) {
  const unsigned long long u = (unsigned long long)__double_as_longlong(v);
  const int lo = __builtin_amdgcn_ds_bpermute(addr, (int)(unsigned)(u & 0xffffffffull));
  const int hi = __builtin_amdgcn_ds_bpermute(addr, (int)(unsigned)(u >> 32));
  return __longlong_as_double((long long)(((unsigned long long)(unsigned)hi << 32) | (unsigned)lo));
}
__device__ __forceinline__ dd dd_bperm(int addr, dd v) { return dd{bperm_d(addr, v.hi), bperm_d(addr, v.lo)}; }
// Value of the previous lane of the 16-lane row.
__device__ __forceinline__ dd dd_ror1(dd v) { return dd{dpp_d<0x121>(v.hi), dpp_d<0x121>(v.lo)}; }   // row_ror:1

// Sturm chains for 64 < D < 96 in double-double, four per wavefront, one per
// 16-lane row: coefficient c = l + 16 s of a member in register s of lane l.
// Each remainder is the exact-arithmetic step (quotient q1 x + q0 from the two
// leading coefficients, by the double-double reciprocal of the divisor's) and each
// member is scaled by a power of two that brings its leading coefficient into [1,
// 2) (exact).  The chain is trusted when every remainder's largest coefficient
// exceeds 1e-24 of the larger of its two members' and its leading coefficient
// 1e-24 of its largest, all finite: in double precision the spread of the Cayley
// polynomial's coefficients at these degrees (1e-15 .. 1e-19) defeats the 1e-13
// test of the other chains, while 106 bits leave room (a 106-bit emulation of this
// chain trusted and matched the exact count on every polynomial tried at H =
// 12..15, also where a double-precision chain with a relaxed test was wrong).
//
// Bound by vector issue: a step is ~70 instructions per register in use and ~110
// for the quotients, maxima and tests, which the four chains share; the registers
// in use fall with the degree.  Against one chain per wavefront with two
// registers and two divisions per step, the Newton round at D = 76 (50 thousand
// frequencies) 1977 -> 753 us.
struct DdState {
  dd at, bt, rb;      // leading coefficients of the last two members, 1 / bt
  double mA, mB;      // their largest coefficients (high words)
  int sp, vp;         // last member positive at +inf; sign changes so far
  bool ok;
};

__device__ __forceinline__ double row_max_hi(int h) {
  h = max(h, dpp_i<0xB1, 0xf>(h));
  h = max(h, dpp_i<0x4E, 0xf>(h));
  h = max(h, dpp_i<0x141, 0xf>(h));
  h = max(h, dpp_i<0x140, 0xf>(h));
  return from_hiword(h);
}

// A (degree db + 1) becomes the next member, -rem(A, B) scaled, of degree db - 1;
// registers 0..R - 1 hold both members (16 (R - 2) <= db - 1).
template <int R>
__device__ __forceinline__ void sturm_dd_step(dd (&A)[6], const dd (&B)[6], DdState& S, int db, int l, int row4) {
#pragma clang fp contract(off)
  const dd q1 = dd_mul(S.at, S.rb);
  // t = A - q1 x B (the coefficient db + 1 cancels)
  dd prev{0.0, 0.0};
#pragma unroll
  for (int s = 0; s < R; ++s) {
    const dd ro = dd_ror1(B[s]);
    const dd sh = l == 0 ? prev : ro;
    prev = ro;
    A[s] = dd_add(A[s], dd_neg(dd_mul(q1, sh)));
  }
  const dd ct = dd_bperm(row4 + ((db & 15) << 2), (R == 1 || (db >> 4) == R - 1) ? A[R - 1] : A[R > 1 ? R - 2 : 0]);
  const dd q0 = dd_mul(ct, S.rb);
  // rem = -(t - q0 B): coefficients below db
  int h = 0;
#pragma unroll
  for (int s = 0; s < R; ++s) {
    dd v = dd_neg(dd_add(A[s], dd_neg(dd_mul(q0, B[s]))));
    if (s >= R - 2) {
      const bool in = l + 16 * s < db;
      v.hi = in ? v.hi : 0.0;
      v.lo = in ? v.lo : 0.0;
    }
    A[s] = v;
    h = max(h, hiword(v.hi) & 0x7fffffff);
  }
  const dd lead = dd_bperm(row4 + (((db - 1) & 15) << 2),
                           (R == 1 || ((db - 1) >> 4) == R - 1) ? A[R - 1] : A[R > 1 ? R - 2 : 0]);
  const double mr = row_max_hi(h);
  S.ok = S.ok && isfinite(mr) && mr > 1e-24 * fmax(S.mA, S.mB) && fabs(lead.hi) > 1e-24 * mr;
  const int tp = lead.hi > 0.0 ? 1 : 0;
  S.vp += tp ^ S.sp;
  S.sp = tp;
  int e = __builtin_amdgcn_frexp_exp(lead.hi);
  if (!(lead.hi != 0.0 && isfinite(lead.hi))) e = 0;
#pragma unroll
  for (int s = 0; s < R; ++s) A[s] = dd_ldexp(A[s], 1 - e);
  S.at = S.bt;
  S.bt = dd_ldexp(lead, 1 - e);
  S.rb = dd_rcp(S.bt);
  S.mA = S.mB;
  S.mB = ldexp(mr, 1 - e);
}

template <int R>
__device__ __forceinline__ void sturm_dd_run(dd (&A)[6], dd (&B)[6], DdState& S, int& db, int l, int row4) {
  // two steps at a time, so that the members' roles are fixed; the registers
  // of the first serve both
#pragma unroll 1
  for (; db >= 2 && db + 1 >= 16 * (R - 1); db -= 2) {
    sturm_dd_step<R>(A, B, S, db, l, row4);
    sturm_dd_step<R>(B, A, S, db - 1, l, row4);
  }
}

// Distinct real roots of the degree-D polynomial f of this lane's row (D even),
// or -1 when a step fails its test (`raw`: the count regardless).  All lanes
// must be active; `on` is uniform in a row.
__device__ int sturm_count_dd(const double* f, bool on, int D, int lane, int& raw) {
#pragma clang fp contract(off)
  const int l = lane & 15, row4 = (lane & ~15) << 2;
  dd A[6], B[6];
  int hA = 0, hB = 0;
  const double fD = on ? f[D] : 1.0, dD = (double)D * fD;
  // scales that bring the leading coefficients into [1, 2) in magnitude
  const int eA = 1 - __builtin_amdgcn_frexp_exp(fD), eB = 1 - __builtin_amdgcn_frexp_exp(dD);
#pragma unroll
  for (int s = 0; s < 6; ++s) {
    // g and g' (exact in double-double: (c + 1) g_{c+1} is one product)
    const int c = l + 16 * s;
    const double g = on && c <= D ? f[c] : 0.0, g1 = on && c < D ? f[c + 1] : 0.0;
    const double p = (double)(c + 1) * g1;
    A[s] = dd_ldexp(dd{g, 0.0}, eA);
    B[s] = dd_ldexp(dd{p, fma((double)(c + 1), g1, -p)}, eB);
    hA = max(hA, hiword(A[s].hi) & 0x7fffffff);
    hB = max(hB, hiword(B[s].hi) & 0x7fffffff);
  }
  DdState S;
  S.at = dd_ldexp(dd{fD, 0.0}, eA);
  S.bt = dd_ldexp(dd{dD, fma((double)D, fD, -dD)}, eB);
  S.rb = dd_rcp(S.bt);
  S.ok = S.at.hi != 0.0 && isfinite(S.at.hi) && S.bt.hi != 0.0;
  S.mA = row_max_hi(hA);
  S.mB = row_max_hi(hB);
  S.sp = S.bt.hi > 0.0 ? 1 : 0;
  S.vp = S.sp ^ (S.at.hi > 0.0 ? 1 : 0);
  int db = D - 1;   // B has degree db, A degree db + 1
  sturm_dd_run<6>(A, B, S, db, l, row4);
  sturm_dd_run<5>(A, B, S, db, l, row4);
  sturm_dd_run<4>(A, B, S, db, l, row4);
  sturm_dd_run<3>(A, B, S, db, l, row4);
  sturm_dd_run<2>(A, B, S, db, l, row4);
  sturm_dd_run<1>(A, B, S, db, l, row4);
  sturm_dd_step<1>(A, B, S, 1, l, row4);
  raw = D - 2 * S.vp;
  return S.ok ? raw : -1;
}

// Sturm chains, one per group of G lanes (8: eight per wavefront; 16: four), D <
// 64.  Lane l of a group holds R consecutive coefficients R l .. R l
// + R - 1 of each member in registers, so the shift by one power of x moves one
// register between lanes (DPP row_shr:1) and the rest by name; R falls from 8
// or 4 to 2 and 1 as the members' degree falls (sturm_repack).  The two
// coefficients a step needs from its own chain (the quotient's and the new
// leading one) come by ds_bpermute.  Per coefficient the arithmetic is that of
// sturm_begin / sturm_step (scaled members with leading coefficient +-1,
// quotients without division).  Coefficients above a member's degree are not
// cleared: they only ever move upwards, and the maxima leave them out.
//
// The tests of the steps (sturm_step_ok, as margins) are taken G steps at a
// time: lane j of a group keeps step j's two high words (largest coefficient,
// leading coefficient with its sign), and sturm_flush forms the margins and sign
// changes of all of them at once.  A step is ~52 vector instructions at R = 8,
// 35 at R = 4 and 22 at R = 1 for 64 / G chains; with the coefficients strided over the lanes
// and the tests in every step it was 66 (36) for four.
template <int G>
struct SturmTests {
  int hrS, hlS;     // this lane's step: hi(max |t|), high word of the leading coefficient
  int n;            // steps held (wave-uniform)
  int c1, c2;       // hi(max |coefficient|) of the last two members before them
  int sp;           // sign of the last member before them at +inf (1: positive)
  int m12, m13;     // smallest margins of the two tests so far (per lane)
  int hmax;         // largest hi(max |t|) so far (finiteness; per lane)
  int vp;           // sign changes at +inf so far (per lane)
};

__device__ __forceinline__ int bperm_i(int addr, int v) { return __builtin_amdgcn_ds_bpermute(addr, v); }

// maximum of an int over each group, left in every lane of the group
template <int G>
__device__ __forceinline__ int group_max_int(int h) {
  h = max(h, dpp_i<0xB1, 0xf>(h));    // quad_perm [1, 0, 3, 2]
  h = max(h, dpp_i<0x4E, 0xf>(h));    // quad_perm [2, 3, 0, 1]
  if constexpr (G == 8) return max(h, dpp_i<0x141, 0xf>(h));   // row_half_mirror
  h = max(h, dpp_i<0x124, 0xf>(h));   // row_ror:4
  return max(h, dpp_i<0x128, 0xf>(h));   // row_ror:8
}
template <int G>
__device__ __forceinline__ int group_sum_int(int h) {
  h += dpp_i<0xB1, 0xf>(h);
  h += dpp_i<0x4E, 0xf>(h);
  if constexpr (G == 8) return h + dpp_i<0x141, 0xf>(h);
  h += dpp_i<0x124, 0xf>(h);
  return h + dpp_i<0x128, 0xf>(h);
}

// Tests and sign changes of the T.n steps held; gb4: byte address (4 x lane) of
// the group's first lane.
template <int G>
__device__ __forceinline__ void sturm_flush(SturmTests<G>& T, int l, int gb4) {
  const int ha = T.hlS & 0x7fffffff, hM = sturm_member_hi(T.hrS, ha), s = (int)((unsigned)T.hlS >> 31);
  const int a1 = gb4 + (((l - 1) & (G - 1)) << 2), a2 = gb4 + (((l - 2) & (G - 1)) << 2);
  const int x1 = bperm_i(a1, hM), x2 = bperm_i(a2, hM), xs = bperm_i(a1, s);
  const int p1 = l >= 1 ? x1 : T.c1, p2 = l >= 2 ? x2 : (l == 1 ? T.c1 : T.c2), ps = l >= 1 ? xs : T.sp;
  if (l < T.n) {
    T.m12 = min(T.m12, T.hrS - max(p1, p2));
    T.m13 = min(T.m13, ha - T.hrS);
    T.hmax = max(T.hmax, T.hrS);
    T.vp += s ^ ps;
  }
  // (a partial flush is the last: the carried values are those of full ones)
  T.c1 = bperm_i(gb4 + ((G - 1) << 2), hM);
  T.c2 = bperm_i(gb4 + ((G - 2) << 2), hM);
  T.sp = bperm_i(gb4 + ((G - 1) << 2), s);
  T.n = 0;
}

// Signs of the last two members' leading coefficients as sign bits.
struct SturmSigns { int b, ab; };   // newer member; product with the older
__device__ __forceinline__ double with_sign(double v, int signbit) {
  const unsigned long long u = (unsigned long long)__double_as_longlong(v);
  return __longlong_as_double((long long)(u ^ ((unsigned long long)(unsigned)signbit << 32)));
}

// One step: from A (older, degree db + 1) and B (degree db), A becomes the
// new member.  RQ = db % R.
template <int G, int R, int RQ, int N>
__device__ __forceinline__ void sturm_rows_step(double (&A)[N], const double (&B)[N], SturmSigns& S, SturmTests<G>& T,
                                                int db, int l, int gb4) {
#pragma clang fp contract(off)
  constexpr int RL = (RQ + R - 1) % R;
  const int lq = db / R, ll = (db - 1) / R;   // (R a power of two)
  const double ab = from_hiword(S.ab ^ kHi1);
  double t[R];
  {
    double sh = dpp_d<0x111>(B[R - 1]);   // row_shr:1, zero into lane 0
    if (G == 8) sh = l == 0 ? 0.0 : sh;
    t[0] = fma(-ab, sh, A[0]);
#pragma unroll
    for (int r = 1; r < R; ++r) t[r] = fma(-ab, B[r - 1], A[r]);
  }
  const double q0 = with_sign(bperm_d(gb4 + (lq << 2), t[RQ]), S.b);
#pragma unroll
  for (int r = 0; r < R; ++r) t[r] = fma(-q0, B[r], t[r]);
  const double lead = bperm_d(gb4 + (ll << 2), t[RL]);
  // largest of the coefficients below db: all of a lane's, in lane lq its first RQ
  double part = 0.0, all = fabs(t[0]);
#pragma unroll
  for (int r = 1; r < R; ++r) {
    if (r == RQ) part = all;
    all = fmax(all, fabs(t[r]));
  }
  int h = l < lq ? hiword(all) : 0;
  if (RQ > 0) h = l == lq ? hiword(part) : h;
  const int hr = group_max_int<G>(h), hlead = hiword(lead);
  const bool mine = l == T.n;
  T.hrS = mine ? hr : T.hrS;
  T.hlS = mine ? hlead : T.hlS;
  if (++T.n == G) sturm_flush<G>(T, l, gb4);
  // P_q = -t / |lead|, its leading coefficient -sign(lead)
  const double sc = fast_rcp_d(fabs(lead) + 1e-300);
#pragma unroll
  for (int r = 0; r < R; ++r) A[r] = -t[r] * sc;
  const int nb = ~hlead & (int)0x80000000;
  S.ab = S.b ^ nb;
  S.b = nb;
}

// R to R / 2 coefficients per lane.
template <int R, int N>
__device__ __forceinline__ void sturm_repack(double (&X)[N], int l, int gb4) {
  const int src = gb4 + ((l >> 1) << 2);
  const bool odd = l & 1;
#pragma unroll
  for (int r = 0; r < R / 2; ++r) {
    const double lo = bperm_d(src, X[r]), hi = bperm_d(src, X[r + R / 2]);
    X[r] = odd ? hi : lo;
  }
}

// Distinct real roots of the degree-D polynomial of this lane's group (D even,
// D + 1 <= RM G, RM = 4 or 8; C[r] = coefficient RM l + r, zero above D; gtop =
// coefficient D), or -1 when a step fails its test (`raw`: the count regardless).
// All lanes must be active.
template <int G, int RM>
__device__ __forceinline__ int sturm_count_groups(const double (&C)[RM], double gtop, int D, int lane, int& raw) {
  // (a chain that ends near the thresholds of its tests turns on its last bits: no
  // contraction, which known signs and degrees would open or close)
#pragma clang fp contract(off)
  const int l = lane & (G - 1), gb4 = (lane & ~(G - 1)) << 2;
  double A[RM], B[RM];
  SturmSigns S;
  SturmTests<G> T;
  bool ok;
  {
    const double ag = fabs(gtop), sgn = gtop > 0.0 ? 1.0 : -1.0;
    const double sa = fast_rcp_d(ag + 1e-300), sb = fast_rcp_d(fma((double)D, ag, 1e-300));
    ok = ag > 0.0 && ag < INFINITY;
    int hA = 0, hB = 0;
    const double up = dpp_d<0x101>(C[0]);   // row_shl:1: coefficient RM (l + 1) (used up to coefficient D)
#pragma unroll
    for (int r = 0; r < RM; ++r) {
      const int k = RM * l + r;
      const double g1 = r < RM - 1 ? C[r < RM - 1 ? r + 1 : RM - 1] : up;   // coefficient k + 1
      const double dv = k < D ? (k + 1) * g1 : 0.0;
      A[r] = k == D ? sgn : C[r] * sa;
      B[r] = k == D - 1 ? sgn : dv * sb;
      hA = max(hA, hiword(A[r]) & 0x7fffffff);
      hB = max(hB, hiword(B[r]) & 0x7fffffff);
    }
    T.c2 = max(group_max_int<G>(hA), kHi1);
    T.c1 = group_max_int<G>(hB);
    T.m12 = T.m13 = 0x7fffffff;
    T.hmax = T.vp = T.n = T.hrS = T.hlS = 0;
    T.sp = gtop > 0.0 ? 1 : 0;
    S.b = gtop > 0.0 ? 0 : (int)0x80000000;
    S.ab = 0;
  }
  int db = D - 1;   // degree of the newer member (odd)
  if constexpr (RM == 8) {
    if (db > 4 * G - 5) {
      // to a multiple of eight coefficients, then whole rounds of them
      const int q = db & 7;
      if (q == 5) {
        sturm_rows_step<G, 8, 5>(A, B, S, T, db, l, gb4);
        sturm_rows_step<G, 8, 4>(B, A, S, T, db - 1, l, gb4);
        db -= 2;
      }
      if (q == 5 || q == 3) {
        sturm_rows_step<G, 8, 3>(A, B, S, T, db, l, gb4);
        sturm_rows_step<G, 8, 2>(B, A, S, T, db - 1, l, gb4);
        db -= 2;
      }
      if (q != 7) {
        sturm_rows_step<G, 8, 1>(A, B, S, T, db, l, gb4);
        sturm_rows_step<G, 8, 0>(B, A, S, T, db - 1, l, gb4);
        db -= 2;
      }
#pragma unroll 1
      for (; db > 4 * G - 5; db -= 8) {
        sturm_rows_step<G, 8, 7>(A, B, S, T, db, l, gb4);
        sturm_rows_step<G, 8, 6>(B, A, S, T, db - 1, l, gb4);
        sturm_rows_step<G, 8, 5>(A, B, S, T, db - 2, l, gb4);
        sturm_rows_step<G, 8, 4>(B, A, S, T, db - 3, l, gb4);
        sturm_rows_step<G, 8, 3>(A, B, S, T, db - 4, l, gb4);
        sturm_rows_step<G, 8, 2>(B, A, S, T, db - 5, l, gb4);
        sturm_rows_step<G, 8, 1>(A, B, S, T, db - 6, l, gb4);
        sturm_rows_step<G, 8, 0>(B, A, S, T, db - 7, l, gb4);
      }
    }
    sturm_repack<8>(A, l, gb4);
    sturm_repack<8>(B, l, gb4);
  }
  if (db > 2 * G - 5) {
    if ((db & 3) == 1) {
      sturm_rows_step<G, 4, 1>(A, B, S, T, db, l, gb4);
      sturm_rows_step<G, 4, 0>(B, A, S, T, db - 1, l, gb4);
      db -= 2;
    }
#pragma unroll 1
    for (; db > 2 * G - 5; db -= 4) {
      sturm_rows_step<G, 4, 3>(A, B, S, T, db, l, gb4);
      sturm_rows_step<G, 4, 2>(B, A, S, T, db - 1, l, gb4);
      sturm_rows_step<G, 4, 1>(A, B, S, T, db - 2, l, gb4);
      sturm_rows_step<G, 4, 0>(B, A, S, T, db - 3, l, gb4);
    }
  }
  sturm_repack<4>(A, l, gb4);
  sturm_repack<4>(B, l, gb4);
#pragma unroll 1
  for (; db > G - 3; db -= 2) {
    sturm_rows_step<G, 2, 1>(A, B, S, T, db, l, gb4);
    sturm_rows_step<G, 2, 0>(B, A, S, T, db - 1, l, gb4);
  }
  sturm_repack<2>(A, l, gb4);
  sturm_repack<2>(B, l, gb4);
#pragma unroll 1
  for (; db > 1; db -= 2) {
    sturm_rows_step<G, 1, 0>(A, B, S, T, db, l, gb4);
    sturm_rows_step<G, 1, 0>(B, A, S, T, db - 1, l, gb4);
  }
  sturm_rows_step<G, 1, 0>(A, B, S, T, 1, l, gb4);
  if (T.n) sturm_flush<G>(T, l, gb4);
  const int m12 = -group_max_int<G>(-T.m12), m13 = -group_max_int<G>(-T.m13);
  ok = ok && group_max_int<G>(T.hmax) < 0x7ff00000 && m12 > -kHiT12 && m13 > -kHiT13;
  raw = D - 2 * group_sum_int<G>(T.vp);
  return ok ? raw : -1;
}

// Coefficients per lane at first of a Sturm chain on G lanes, D < 64 (eight lanes
// throughout, or sixteen above degree 31).
__host__ __device__ inline constexpr int sturm_coefs(int D, int G) { return D < 4 * G ? 4 : 8; }

// C[r] = coefficient R l + r of f (zero above D), l the lane's index in its group.
template <int R>
__device__ __forceinline__ void load_coefficients(const double* f, bool on, int D, int l, double (&C)[R]) {
#pragma unroll
  for (int r = 0; r < R; ++r) C[r] = (on && R * l + r <= D) ? f[R * l + r] : 0.0;
}

// Newton on R(theta) carried out on the Cayley polynomial.  With x = tan((theta
// - phi0) / 2), f(x) = (1 + x^2)^K R(theta), so R'/R = ((1 + x^2) f'/f - 2 K x)
// / 2 and the Newton step of R in theta is d = 2 f / ((1 + x^2) f' - 2 K x f).
// For |x| > 1 the iterate is kept as y = 1 / x and the reversed polynomial
// g(y) = y^D f(1 / y) = (1 + y^2)^K R(theta) serves the same way, with theta
// decreasing in y, so the formula (in g, y) gives -d.  Either way the iterate u
// = x or y has |u| <= 1, and the step (clamped to 0.5 rad as in theta) is
// applied by the tangent addition formula u <- (u - t) / (1 + u t), t = tan(s
// / 2) from its series to fifth order (the clamp bounds the relative error of
// t by 1.3e-5 and it vanishes as the step does, so convergence stays quadratic);
// if the result leaves [-1, 1] its reciprocal is taken and the representation
// flips.  One Newton step costs a real Horner pass of degree D for f and f'
// (2D multiply-adds) in place of K complex multiply-adds for R and R' plus a
// sine and cosine.  cp: coefficients of f (sg > 0) or of g (sg < 0) in
// ascending order, followed by zeros up to c = newton_top(D): zero leading
// coefficients change no result, and with them every degree runs the four-step
// body below without a remainder loop (at H = 4 two of ten steps, whose loads
// and branches cost more than two whole steps).  Returns the signed step s (theta
// moves by sg * s, clamped); ok drops on a zero or non-finite step.
__host__ __device__ inline constexpr int newton_top(int D) { return ((D - 2 + 7) & ~7) + 2; }
__device__ __forceinline__ double newton_u_step(const double* cp, int DP, int K, double& u, int& sg, bool& ok) {
  // f = E(v) + u O(v), v = u^2 (D even: E has the even powers up to D, O the
  // odd ones up to D - 1), f' = 2u E'(v) + O(v) + 2v O'(v): four independent
  // Horner chains of D/2 steps in place of two of D
  const double v = u * u;
  double E = cp[DP], dE = 0.0, O = cp[DP - 1], dO = 0.0;
  // (the new E and O are formed in the loaded coefficients' registers and the
  // derivatives in the old ones', so no step needs a register copy)
  for (int c = DP - 2; c >= 8; c -= 8) {
#pragma unroll
    for (int i = 0; i < 8; i += 2) {
      const double a = cp[c - i], b = cp[c - i - 1];
      const double nE = fma(E, v, a), nO = fma(O, v, b);
      dE = fma(dE, v, E);
      dO = fma(dO, v, O);
      E = nE;
      O = nO;
    }
  }
  dE = fma(dE, v, E);
  E = fma(E, v, cp[0]);
  const double F = fma(u, O, E);
  const double dF = fma(2.0 * u, dE, fma(2.0 * v, dO, O));
  const double den = fma(fma(u, u, 1.0), dF, -(2.0 * K) * u * F);
  const double d = 2.0 * F * fast_rcp_d(den);
  ok = den != 0.0 && isfinite(d);
  const double sc = fmax(-0.5, fmin(0.5, d));
  const double h = 0.5 * sc, h2 = h * h;
  const double t = h * fma(h2, fma(h2, 0.13333333333333333333, 0.33333333333333333333), 1.0);
  const double num = u - t, dd = fma(u, t, 1.0);
  const bool flip = fabs(num) > fabs(dd);
  u = (flip ? dd : num) * fast_rcp_d(flip ? num : dd);
  sg = flip ? -sg : sg;
  return sc;
}

// Convergence of a Newton lane from its step sizes: a step below 1e-12, or,
// in the quadratic regime, a step small enough that the iterate it produced
// is already within ~1e-14 of the root.  With steps s_{k-1}, s_k and the
// error after step k about C s_k^2, C ~ s_k / s_{k-1}^2, the second test is
// s_k^3 < 1e-14 s_{k-1}^2 (with s_k < 1e-6 and s_{k-1} < 1e-3, so that both
// steps are local ones, not a clamped jump); a slowly (linearly) converging
// lane, as near a double root, passes only the first.  Saves the step that
// would merely confirm convergence.
__device__ __forceinline__ bool newton_settled(double sc, double& prev) {
  const double a = fabs(sc);
  const bool c = a < 1e-12 || (a < 1e-6 && prev < 1e-3 && a * a * a < 1e-14 * prev * prev);
  prev = a;
  return c;
}

// Eight frequencies per wavefront (where there are few, four for H > 5 and down to two
// for H <= 5, newton_per), consecutive ones of the list.  Their Sturm chains run side by side, a group of lanes each
// (sturm_count_groups); then Newton runs on two of them at a time, lanes
// 0..31 for the first and 32..63 for the second, each half with min(32, D)
// starts: the 2H network seeds and min(32, D) - 2H evenly spaced phases (all
// evenly spaced without network, tabulated).  The Newton steps are those of R in
// theta, evaluated on the Cayley polynomial (newton_u_step); converged roots are
// merged one root of each half per pass, and a half that has reached its count is
// frozen while the other goes on.
//
// Bound by vector issue and the latency of its serial chains (67 % of the
// slots at six wavefronts per SIMD), so H is a template parameter: strides, loop
// counts and LDS offsets are immediates and few registers spill (see OCC below).  The
// six-wave build moves 1.37 GB at H = 10 (300 thousand frequencies), where 0.29 are
// needed, in the same time as the five-wave one: the traffic hides behind the issue.
// That, the merge of both halves per pass (its scalar half
// shortened in a second step, 6 %), the tabulated starts, phases left to the
// scoring and eight lanes per Sturm chain also above degree 31 (10 %): H = 10, 300
// thousand frequencies 985 -> 775 us; H = 6, 250 thousand 575 -> 420 us; H = 4, 4.2
// million 5.4 -> 4.3 ms.
// Starts of the first round for each frequency.
__host__ __device__ inline constexpr int first_starts(int H, bool equal) {
  return equal ? 2 * H : (6 * H - 2 < 32 ? 6 * H - 2 : 32);
}
// Evenly spaced starts of the first round for the sixteen rotations phi0 = 2
// pi k / 16: entry 32 k + i the iterate (u, sg) of phase (i + 1/2) 2 pi / NS.
__global__ __launch_bounds__(512) void k_start_table(double2* out, int NS) {
  const int k = threadIdx.x >> 5, i = threadIdx.x & 31;
  double s1, c1, u;
  int sg;
  const double phi0 = kTwoPi * k / 16.0;
  double ang = (i + 0.5) * (kTwoPi / NS);
  asm volatile("" : "+v"(ang));   // rounded before the difference
  sincos_small(ang - phi0, s1, c1);
  u_from_dir(c1, s1, u, sg);
  out[threadIdx.x] = make_double2(u, (double)sg);
}

struct NewtonAcc {
  int iters;   // this lane's
  unsigned long long roots, fb;
};

// Newton on frequencies wA (lanes 0..31) and wA + 1 (lanes 32..63, if hasB)
// with Sturm counts cA, cB (-2 inactive, -1 untrusted); f of each half and its
// reversal in fb (LDS, 2 FS doubles per half).
template <int H>
__device__ __forceinline__ void newton_pair(const LearnArgs& L, const RecLayout& RL, int64_t wA, int cA, int cB,
                                            const double* fb, int lane, NewtonAcc& acc) {
  const int half = lane >> 5, hl = lane & 31;
  // starts per frequency: every lane of the half (at most D), or only 2H
  // (flag bit 1: the equal-starts comparison of seeds and evenly spaced phases)
  constexpr int K = 3 * H - 1, D = 2 * K, S = 2 * H, DP = newton_top(D), FS = DP + 2;
  const int NS = first_starts(H, L.flags & 2u);
  const unsigned long long lo32 = 0xffffffffull;
  if (cA == -2 && cB == -2) return;
  double* Rh = L.rec + (wA + half) * (int64_t)RL.stride;   // this lane's frequency (unused when inactive)
  const int64_t wh = wA + half;
  const int cnt = half ? cB : cA;
  const double phi0 = cnt != -2 ? Rh[RL.meta + M_PHI0] : 0.0;
  double u = 0.0;
  int sg = 1;
  bool conv = false, live = cnt >= 0 && hl < NS;
  int its = 0;
  double prev_step = 1.0;
  if (!L.seeds_out) {
    // evenly spaced phases less phi0: tabulated for the sixteen rotations
    const int k0 = (int)rint(phi0 * (16.0 / kTwoPi)) & 15;
    const double2 t = L.starts[32 * k0 + hl];
    u = t.x;
    sg = (int)t.y;
  } else if (live) {
    // start direction relative to phi0: a network seed (its output vector
    // is the root's direction in the canonical frame, rotated here by
    // -(canon + phi0)) or an evenly spaced phase less phi0
    double bc = 1.0, bs = 0.0, ang;
    if (hl < S) {
      const float* o = L.seeds_out + wh * 2 * S;
      bc = (double)o[2 * hl];
      bs = (double)o[2 * hl + 1];
      ang = -(Rh[RL.meta + M_CANON] + phi0);
    } else {
      ang = (hl - S + 0.5) * (kTwoPi / (NS - S)) - phi0;
    }
    double s1, c1;
    sincos_small(ang, s1, c1);
    u_from_dir(fma(bc, c1, -bs * s1), fma(bc, s1, bs * c1), u, sg);
  }
  const double* fbase = fb + 2 * FS * half;
  bool doneA = cA < 0, doneB = cB < 0;
  unsigned long long um = 0ull, merged = 0ull, U = 0ull;   // U: unique converged lanes
  for (int it = 1; it <= 12 && !(doneA && doneB); ++it) {
    if (live && !conv) {
      bool ok;
      const double sc = newton_u_step(sg > 0 ? fbase : fbase + FS, DP, K, u, sg, ok);
      if (!ok) {
        live = false;
      } else {
        ++its;
        if (newton_settled(sc, prev_step)) conv = true;
      }
    }
    if (it >= 2) {   // merges are incremental, so every iteration from the second checks
      const unsigned long long cm = __ballot(conv);
      // (each half on its own count alone: what it settles, and so the lane that
      // stands for a root, does not depend on the other's)
      const bool needA = !doneA && (__popcll(cm & lo32) >= cA || it == 12);
      const bool needB = !doneB && (__popcll(cm >> 32) >= cB || it == 12);
      if (!needA && !needB) continue;
      const unsigned long long need = (needA ? lo32 : 0ull) | (needB ? ~lo32 : 0ull);
      // distinct converged roots of each half: converged lanes of one root lie
      // within 1e-8 rad of each other.
      // Compared on key = u (sg > 0) or sign(u) 2 - u (sg < 0), which
      // increases with theta - phi0 over (-pi, pi) and moves by |du| where
      // theta moves by 2 |du| / (1 + u^2) (the cut at theta - phi0 = pi
      // sits where R is largest, far from any root).  Converged lanes no
      // longer move, so each check settles only the lanes converged since
      // the last: one pass takes the lowest pending lane of each half, counts it
      // as a new root unless a root settled before lies within the tolerance, and
      // settles every converged lane of the half that does.  (Both halves per
      // pass, the keys broadcast through LDS: against one half per pass
      // through scalar registers, with the lowest lane kept as each root's, it
      // takes half the passes and a quarter of the vector instructions.)
      const double key = sg > 0 ? u : copysign(2.0, u) - u;
      const double tol = 0.5e-8 * fma(u, u, 1.0);
      for (unsigned long long pend = cm & ~merged & need; pend;) {
        const unsigned pA = (unsigned)pend, pB = (unsigned)(pend >> 32);
        const unsigned bA = pA & (0u - pA), bB = pB & (0u - pB);   // 0: none pending
        const int jA = __builtin_ctz(pA | 0x80000000u), jB = __builtin_ctz(pB | 0x80000000u);
        const double kj = bperm_d((half ? 32 + jB : jA) << 2, key);
        const unsigned long long same = __ballot(fabs(key - kj) < tol) & cm;
        const unsigned sA = (unsigned)same, sB = (unsigned)(same >> 32);
        const unsigned uA = (unsigned)U, uB = (unsigned)(U >> 32);
        U |= (sA & uA ? 0u : bA) | ((unsigned long long)(sB & uB ? 0u : bB) << 32);
        pend &= ~((sA | bA) | ((unsigned long long)(sB | bB) << 32));
      }
      merged |= cm & need;
      um = U;
      if (__popcll(um & lo32) == cA) doneA = true;
      if (__popcll(um >> 32) == cB) doneB = true;
      if (half ? doneB : doneA) live = false;
    }
  }
  acc.iters += its;
  const int nuA = __popcll(um & lo32), nuB = __popcll(um >> 32);
  const bool okA = cA >= 0 && nuA == cA, okB = cB >= 0 && nuB == cB;
  const bool ok = half ? okB : okA;
  const int nu = half ? nuB : nuA;
  double* cand = Rh + RL.cand;
  // confirmed roots: their keys to the front of the half in lane order (a
  // permutation of the half's lanes), NaN behind them; one store of the slots the
  // scoring reads, which takes the phase only of the winner
  const unsigned uh = half ? (unsigned)(um >> 32) : (unsigned)um, below = (1u << hl) - 1u;
  const bool uniq = (uh >> hl) & 1u;
  const int rank = uniq ? __popc(uh & below) : nu + __popc(~uh & below);
  {
    const unsigned long long v = (unsigned long long)__double_as_longlong(sg > 0 ? u : copysign(2.0, u) - u);
    const int to = (32 * half + rank) << 2;
    const int lo = __builtin_amdgcn_ds_permute(to, (int)(unsigned)(v & 0xffffffffull));
    const int hi = __builtin_amdgcn_ds_permute(to, (int)(unsigned)(v >> 32));
    const double r = __longlong_as_double((long long)(((unsigned long long)(unsigned)hi << 32) | (unsigned)lo));
    if (cnt != -2 && ok && hl < D) cand[hl] = hl < nu ? r : __longlong_as_double(0x7ff8000000000000ll);
  }
  // else the phases of the distinct roots found, which start the later tiers
  if ((cA != -2 && !okA) || (cB != -2 && !okB)) {
    const double thw = theta_from_u(phi0, u, sg);
    if (cnt != -2 && !ok && uniq) cand[rank] = thw;
  }
  if (cnt != -2 && !ok && hl == 0) {
    Rh[RL.meta + M_WARM] = (double)nu;
    Rh[RL.meta + M_COUNT] = (double)cnt;
    Rh[RL.meta + M_FALLBACK] = 1.0;
    const unsigned slot = atomicAdd(L.fb_count, 1u);
    L.fb_list[slot] = wh;
  }
  acc.roots += (unsigned long long)((okA ? nuA : 0) + (okB ? nuB : 0));
  acc.fb += (unsigned long long)((cA != -2 && !okA) + (cB != -2 && !okB));
  lwave_sync();
}

// OCC: resident wavefronts per SIMD the register allocation is made for (5: up
// to 96 VGPRs, 6: up to 80); which is faster depends on the workload and the grid
// (512 lightcurves at H = 4 37.5 ms at five, 36.9 at six; H = 10 the same), so the
// launch shape picks it (4 takes the former).  Spilled registers at five / six: 6-8 /
// 14-20 with sixteen lanes per chain or H <= 5, 20-28 / 32-53 with eight above.
// FEW: L.per frequencies per wavefront instead of one per group (the loop bounds and
// strides as arguments cost a few spills, 0.5 % of the time).
template <int H, int OCC, int G, bool FEW>
__global__ __launch_bounds__(64) __attribute__((amdgpu_waves_per_eu(OCC))) void k_newton_sturm4(SolveArgs a, LearnArgs L) {
  extern __shared__ double sml[];
  constexpr int D = 6 * H - 2, RM = sturm_coefs(D, G);
  constexpr int DP = newton_top(D), FS = DP + 2;   // f and its reversal of the two at hand, 16-byte aligned
  const int lane = threadIdx.x & 63, row = lane / G, l = lane & (G - 1);
  const RecLayout RL(H);
  NewtonAcc acc{0, 0, 0};
  const int half = lane >> 5, hl = lane & 31;
  double* fh = sml + 2 * FS * half;
  for (int k = D + 1 + hl; k <= DP; k += 32) fh[k] = fh[FS + k] = 0.0;
  const int per = FEW ? L.per : 64 / G;   // frequencies per wavefront, even
  for (int64_t w0 = per * (int64_t)blockIdx.x; w0 < L.np; w0 += per * (int64_t)gridDim.x) {
    // this group's frequency (inactive: no turn, past the end, rejected lightcurve,
    // or P constant in theta_2)
    bool mine = row < per && w0 + row < L.np;
    double* Rr = L.rec + (w0 + (mine ? row : 0)) * (int64_t)RL.stride;
    const int st = (int)Rr[RL.meta + M_STATUS];
    mine = mine && st != ST_BAD_LC && st != ST_CONSTANT;
    const unsigned long long act = __ballot(mine);
    if (!act) continue;
    if (L.flags & 1u) {   // forced fallback
      if (l == 0 && mine) {
        const unsigned slot = atomicAdd(L.fb_count, 1u);
        L.fb_list[slot] = w0 + row;
        Rr[RL.meta + M_FALLBACK] = 1.0;
        Rr[RL.meta + M_WARM] = 0.0;
        Rr[RL.meta + M_COUNT] = -1.0;
      }
      acc.fb += (unsigned long long)(__popcll(act) / G);
      continue;
    }
    const double* f = Rr + RL.f;
    double C[RM];
    load_coefficients(f, mine, D, l, C);
    const double gtop = mine ? f[D] : 0.0;
    int raw;
    int cnt = sturm_count_groups<G>(C, gtop, D, lane, raw);
    if (cnt < 2) cnt = -1;
    if (!mine) cnt = -2;
    // Newton two frequencies at a time; each half's coefficients come again, from
    // the cache, ahead of its turn (all eight pairs of rows would take 8 KB of LDS)
    auto fetch = [&](int p, double& v0, double& v1) {
      const int64_t w = w0 + 2 * p + half;
      const double* fw = L.rec + (w < L.np ? w : w0) * (int64_t)RL.stride + RL.f;
      v0 = fw[hl < D ? hl : D];
      v1 = D >= 32 ? fw[hl + 32 < D ? hl + 32 : D] : 0.0;
    };
    double v0, v1;
    fetch(0, v0, v1);
#pragma unroll 1
    for (int p = 0; p < per / 2; ++p) {
      if (hl <= D) fh[hl] = fh[FS + D - hl] = v0;
      if (D >= 32 && hl + 32 <= D) fh[hl + 32] = fh[FS + D - 32 - hl] = v1;
      lwave_sync();
      if (p + 1 < per / 2) fetch(p + 1, v0, v1);
      newton_pair<H>(L, RL, w0 + 2 * p, __builtin_amdgcn_readlane(cnt, 2 * p * G),
                     __builtin_amdgcn_readlane(cnt, (2 * p + 1) * G), sml, lane, acc);
    }
  }
  const unsigned long long iters = (unsigned long long)wave_sum((double)acc.iters);
  if (lane == 0 && a.counters) {
    SolveCounters* c = counter_slot(a.counters);
    if (iters) atomicAdd(&c->newton_iters, iters);
    if (acc.roots) atomicAdd(&c->roots_found, acc.roots);
    if (acc.fb) atomicAdd(&c->fallback, acc.fb);
  }
}

// Above H = 10: one frequency per wavefront at H = 11 (NC = 1, D = 64: the Sturm
// chain of f in registers, the degree-64 coefficient as a scalar), up to four above
// (NC = 4: their double-double chains run side by side), then for each of them Newton
// from 4H starts (the 2H network seeds and 2H evenly spaced phases; all evenly
// spaced without network), stepped on the Cayley polynomial and merged one root
// per pass, with the stop rule of k_newton_sturm4.
__host__ __device__ inline size_t learn_lds_bytes(int H) {
  const int D = 6 * H - 2;
  return (size_t)(2 * (newton_top(D) + 2)) * sizeof(double);   // f and its reversal
}

template <int NC, bool FEW>
__global__ __launch_bounds__(64) __attribute__((amdgpu_waves_per_eu(4))) void k_newton_sturm(SolveArgs a, LearnArgs L) {
  extern __shared__ double sml[];
  const int lane = threadIdx.x & 63;
  const int H = a.H, K = 3 * H - 1, D = 2 * K, S = 2 * H, NS = 2 * S;
  const int DP = newton_top(D), FS = DP + 2;
  const RecLayout RL(H);
  const unsigned long long below = (1ull << lane) - 1ull;
  unsigned long long iters_acc = 0, roots_acc = 0, fb_acc = 0;
  const int per = FEW ? L.per : NC;
  for (int64_t w0 = per * (int64_t)blockIdx.x; w0 < L.np; w0 += per * (int64_t)gridDim.x) {
    // Sturm counts first: an ill-determined count (or fewer than the two real
    // roots every non-constant P has) sends the frequency on without Newton
    const int row = NC > 1 ? lane >> 4 : 0;
    bool mine = row < per && w0 + row < L.np;
    double* Rr = L.rec + (w0 + (mine ? row : 0)) * (int64_t)RL.stride;
    const int st = (int)Rr[RL.meta + M_STATUS];
    mine = mine && st != ST_BAD_LC && st != ST_CONSTANT;
    if (__ballot(mine) == 0ull) continue;
    int cnts = -1, raw;
    if (!(L.flags & 1u)) {
      if constexpr (NC > 1) {
        cnts = sturm_count_dd(Rr + RL.f, mine, D, lane, raw);
      } else {
        const double gv = lane <= D ? Rr[RL.f + lane] : 0.0;
        cnts = sturm_count_line_reg(gv, Rr[RL.f + D], D, lane, raw);
      }
    }
    if (cnts < 2) cnts = -1;
    if (!mine) cnts = -2;
#pragma unroll 1
    for (int p = 0; p < per; ++p) {
      const int cnt = __builtin_amdgcn_readlane(cnts, 16 * p);
      if (cnt == -2) continue;
      const int64_t w = w0 + p;
      double* R = L.rec + w * (int64_t)RL.stride;
      if (L.flags & 1u) {   // forced fallback
        if (lane == 0) {
          const unsigned slot = atomicAdd(L.fb_count, 1u);
          L.fb_list[slot] = w;
          R[RL.meta + M_FALLBACK] = 1.0;
          R[RL.meta + M_WARM] = 0.0;
          R[RL.meta + M_COUNT] = -1.0;
        }
        ++fb_acc;
        continue;
      }
      for (int c = lane; c <= DP; c += 64) {
        const double fc = c <= D ? R[RL.f + c] : 0.0;
        sml[c] = fc;
        sml[FS + (c <= D ? D - c : c)] = fc;
      }
      lwave_sync();
      const double phi0 = R[RL.meta + M_PHI0];
      double u = 0.0;
      int sg = 1;
      bool conv = false, live = cnt >= 0 && lane < NS;
      int its = 0;
      double prev_step = 1.0;
      if (live) {
        const bool seeded = L.seeds_out && lane < S;
        double bc = 1.0, bs = 0.0, ang;
        if (seeded) {
          const float* o = L.seeds_out + w * 2 * S;
          bc = (double)o[2 * lane];
          bs = (double)o[2 * lane + 1];
          ang = -(R[RL.meta + M_CANON] + phi0);
        } else {
          ang = (L.seeds_out ? (lane - S + 0.5) * (kTwoPi / (NS - S)) : (lane + 0.5) * (kTwoPi / NS)) - phi0;
        }
        double s1, c1;
        sincos_small(ang, s1, c1);
        u_from_dir(fma(bc, c1, -bs * s1), fma(bc, s1, bs * c1), u, sg);
      }
      bool done = cnt < 0;
      unsigned long long um = 0ull, merged = 0ull, U = 0ull;
      for (int it = 1; it <= 12 && !done; ++it) {
        if (live && !conv) {
          bool ok;
          const double sc = newton_u_step(sg > 0 ? sml : sml + FS, DP, K, u, sg, ok);
          if (!ok) {
            live = false;
          } else {
            ++its;
            if (newton_settled(sc, prev_step)) conv = true;
          }
        }
        if (it >= 2) {
          const unsigned long long cm = __ballot(conv);
          // fewer converged lanes than the count cannot reach it (the last
          // check always runs: its roots seed the fallback)
          if (__popcll(cm) < cnt && it < 12) continue;
          const double key = sg > 0 ? u : copysign(2.0, u) - u;
          for (unsigned long long pend = cm & ~merged; pend;) {
            const int jj = __builtin_ctzll(pend);
            const double kj = lrdlane(key, jj), uj = lrdlane(u, jj);
            const double tol = 0.5e-8 * fma(uj, uj, 1.0);
            const unsigned long long bit = 1ull << jj;
            const unsigned long long same = __ballot(fabs(key - kj) < tol) & cm;
            const unsigned long long upto = (bit << 1) - 1ull;
            U &= upto | ~same;
            U = (same & (bit - 1ull)) ? (U & ~bit) : (U | bit);
            pend &= ~(same | bit);
          }
          merged = cm;
          um = U;
          if (__popcll(um) == cnt) {
            done = true;
            live = false;
          }
        }
      }
      iters_acc += (unsigned long long)wave_sum((double)(lane < NS ? its : 0));
      const double thw = theta_from_u(phi0, u, sg);
      const int nu = __popcll(um);
      const bool uniq = (um >> lane) & 1ull;
      if (cnt >= 0 && cnt == nu) {
        double* cand = R + RL.cand;
        for (int c = lane; c < D; c += 64) cand[c] = __longlong_as_double(0x7ff8000000000000ll);
        lwave_sync();
        if (uniq) cand[__popcll(um & below)] = thw;
        roots_acc += (unsigned long long)nu;
      } else {
        // the distinct roots Newton did find start the Aberth iteration
        if (uniq) R[RL.cand + __popcll(um & below)] = thw;
        if (lane == 0) {
          R[RL.meta + M_WARM] = (double)nu;
          R[RL.meta + M_COUNT] = (double)cnt;
          R[RL.meta + M_FALLBACK] = 1.0;
          const unsigned slot = atomicAdd(L.fb_count, 1u);
          L.fb_list[slot] = w;
        }
        ++fb_acc;
      }
      lwave_sync();
    }
  }
  if (lane == 0 && a.counters) {
    SolveCounters* c = counter_slot(a.counters);
    if (iters_acc) atomicAdd(&c->newton_iters, iters_acc);
    if (roots_acc) atomicAdd(&c->roots_found, roots_acc);
    if (fb_acc) atomicAdd(&c->fallback, fb_acc);
  }
}

// Lanes per Sturm chain up to H = 10: eight, so eight frequencies per wavefront, where
// that leaves the device two rounds of resident wavefronts; with fewer frequencies
// sixteen (four per wavefront) fill it more evenly, except up to degree 31, where
// eight lanes are also the shorter chain.  Measured with 8 / 16 lanes, whole
// periodograms: H = 6 311 / 305 us at 50 thousand frequencies, 475 / 473 at 100, 755 /
// 810 at 200; H = 10 418 / 405, 655 / 675 and 1140 / 1170.
constexpr int64_t kEightLanesFrom = 100000;
__host__ constexpr int sturm_lanes(int H, int64_t np) { return 6 * H - 2 < 32 || np >= kEightLanesFrom ? 8 : 16; }

// Root counts of a record chunk (diagnostic of the count the learned and
// uniform solvers trust): per pair, the Sturm count of the Cayley polynomial
// f by the device code the Newton kernels use on such a chunk
// (sturm_count_groups for H <= 10, with G = sturm_lanes lanes per pair;
// sturm_count_line_reg, G = 64, for H = 11; sturm_count_dd, DD, above), -1000 - n
// when the chain fails its test (n: the count it reached regardless), -2 for an
// inactive pair; and the number of real
// eigenvalues the companion QR (run before this kernel) marked in M_REAL_LO,
// M_REAL_HI and M_REAL_X (-1 when the QR did not converge).
template <int G, bool DD>
__global__ __launch_bounds__(64) void k_root_counts(const double* rec, int H, int64_t np, int* sturm, int* real) {
  constexpr int per = 64 / G;
  const int lane = threadIdx.x & 63, row = lane / G, l = lane & (G - 1);
  const int D = 6 * H - 2;
  const RecLayout RL(H);
  for (int64_t w0 = per * (int64_t)blockIdx.x; w0 < np; w0 += per * (int64_t)gridDim.x) {
    const bool in = w0 + row < np;
    const double* f = rec + (w0 + (in ? row : 0)) * (int64_t)RL.stride + RL.f;
    int cnt, raw;
    if constexpr (DD) {
      cnt = sturm_count_dd(f, in, D, lane, raw);
    } else if constexpr (G == 64) {
      cnt = sturm_count_line_reg(f[lane], f[D], D, lane, raw);
    } else {
      const double gtop = in ? f[D] : 0.0;
      if (G == 16 || sturm_coefs(D, G) == 4) {
        double C[4];
        load_coefficients(f, in, D, l, C);
        cnt = sturm_count_groups<G>(C, gtop, D, lane, raw);
      } else {
        double C[8];
        load_coefficients(f, in, D, l, C);
        cnt = sturm_count_groups<G>(C, gtop, D, lane, raw);
      }
    }
    if (cnt < 0) cnt = -1000 - raw;
    cnt = __shfl(cnt, (lane * G) & 63);   // pair `lane` of the wavefront to lane `lane`
    if (lane < per && w0 + lane < np) {
      const double* Rq = rec + (w0 + lane) * (int64_t)RL.stride;
      const int st = (int)Rq[RL.meta + M_STATUS];
      const bool act = st != ST_BAD_LC && st != ST_CONSTANT;
      const unsigned lo = (unsigned)Rq[RL.meta + M_REAL_LO], hi = (unsigned)Rq[RL.meta + M_REAL_HI];
      const unsigned x = D > 64 ? (unsigned)Rq[RL.meta + M_REAL_X] : 0u;
      const int nreal = __popcll(((unsigned long long)hi << 32) | lo) + __popc(x);
      sturm[w0 + lane] = act ? cnt : -2;
      real[w0 + lane] = act ? (st == ST_NO_CONVERGE ? -1 : nreal) : -2;
    }
  }
}

hipError_t launch_root_counts(const double* rec, int H, int64_t np, int* sturm, int* real, int waves,
                              hipStream_t st) {
  const dim3 grid((unsigned)waves), block(64);
  if (H > 11) hipLaunchKernelGGL((k_root_counts<16, true>), grid, block, 0, st, rec, H, np, sturm, real);
  else if (H == 11) hipLaunchKernelGGL((k_root_counts<64, false>), grid, block, 0, st, rec, H, np, sturm, real);
  else if (sturm_lanes(H, np) == 16) hipLaunchKernelGGL((k_root_counts<16, false>), grid, block, 0, st, rec, H, np, sturm, real);
  else hipLaunchKernelGGL((k_root_counts<8, false>), grid, block, 0, st, rec, H, np, sturm, real);
  return hipGetLastError();
}

// Second Newton round (project addition) for the frequencies the first left
// unconfirmed: one frequency per wavefront.  Lanes 0..nu - 1 hold the nu
// distinct roots the first round found (converged, not stepped); lanes
// nu..63 start from new phases: the network's 2H seeds first when the
// learned solver supplies them (row i of `seeds` for list entry i), then
// evenly spaced phases offset from the first round's grid.  Newton steps, the
// merge of converged roots and the stop rule are those of the first round,
// against the Sturm count it kept in M_COUNT; a frequency that reaches its
// count is settled (its roots become the candidates), the others go on to
// the Aberth tier through out_list with the roots found as its warm start.
__global__ __launch_bounds__(64) __attribute__((amdgpu_waves_per_eu(4))) void k_newton_retry(RetryArgs A) {
  // the fallback tiers run beside the side stream's scoring: their waves
  // take issue priority over it on a shared SIMD (the tiers are few, latency-bound
  // waves on the step's critical path)
  __builtin_amdgcn_s_setprio(2);
  extern __shared__ double sml[];
  const int lane = threadIdx.x & 63;
  const int H = A.H, K = 3 * H - 1, D = 2 * K, S = 2 * H;
  const int DP = newton_top(D), FS = DP + 2;
  const RecLayout RL(H);
  const unsigned long long below = (1ull << lane) - 1ull;
  const int64_t n = (int64_t)*A.count;
  unsigned long long iters_acc = 0, left_acc = 0;
  for (int64_t i = blockIdx.x; i < n; i += gridDim.x) {
    const int64_t w = A.list[i];
    double* R = A.rec + w * (int64_t)RL.stride;
    const int cnt = (int)R[RL.meta + M_COUNT];
    if (cnt < 2) {   // no trusted count (or a forced fallback): straight on
      if (lane == 0) {
        const unsigned slot = atomicAdd(A.out_count, 1u);
        A.out_list[slot] = w;
      }
      ++left_acc;
      continue;
    }
    for (int c = lane; c <= DP; c += 64) {
      const double fc = c <= D ? R[RL.f + c] : 0.0;
      sml[c] = fc;
      sml[FS + (c <= D ? D - c : c)] = fc;
    }
    const int nu0 = (int)R[RL.meta + M_WARM];
    const double phi0 = R[RL.meta + M_PHI0];
    lwave_sync();
    double u = 0.0;
    int sg = 1;
    bool conv = false, live = false;
    int its = 0;
    double prev_step = 1.0;
    {
      double bc = 1.0, bs = 0.0, ang;
      const int k = lane - nu0, nst = 64 - nu0;
      if (lane < nu0) {
        ang = R[RL.cand + lane] - phi0;   // a root the first round found
        conv = true;
      } else if (A.seeds && k < S) {
        const float* o = A.seeds + i * 2 * S;
        bc = (double)o[2 * k];
        bs = (double)o[2 * k + 1];
        ang = -(R[RL.meta + M_CANON] + phi0);
        live = true;
      } else {
        const int kk = A.seeds ? k - S : k, nn = A.seeds ? nst - S : nst;
        ang = (kk + 0.25) * (kTwoPi / nn) - phi0;
        live = true;
      }
      double s1, c1;
      sincos_small(ang, s1, c1);
      u_from_dir(fma(bc, c1, -bs * s1), fma(bc, s1, bs * c1), u, sg);
    }
    bool done = false;
    unsigned long long um = 0ull, merged = 0ull, U = 0ull;
    for (int it = 1; it <= 12 && !done; ++it) {
      if (live && !conv) {
        bool ok;
        const double sc = newton_u_step(sg > 0 ? sml : sml + FS, DP, K, u, sg, ok);
        if (!ok) {
          live = false;
        } else {
          ++its;
          if (newton_settled(sc, prev_step)) conv = true;
        }
      }
      const unsigned long long cm = __ballot(conv);
      if (__popcll(cm) < cnt && it < 12) continue;
      const double key = sg > 0 ? u : copysign(2.0, u) - u;
      for (unsigned long long pend = cm & ~merged; pend;) {
        const int jj = __builtin_ctzll(pend);
        const double kj = lrdlane(key, jj), uj = lrdlane(u, jj);
        const double tol = 0.5e-8 * fma(uj, uj, 1.0);
        const unsigned long long bit = 1ull << jj;
        const unsigned long long same = __ballot(fabs(key - kj) < tol) & cm;
        const unsigned long long upto = (bit << 1) - 1ull;
        U &= upto | ~same;
        U = (same & (bit - 1ull)) ? (U & ~bit) : (U | bit);
        pend &= ~(same | bit);
      }
      merged = cm;
      um = U;
      if (__popcll(um) == cnt) done = true;
    }
    iters_acc += (unsigned long long)wave_sum((double)its);
    const double thw = theta_from_u(phi0, u, sg);
    const int nu = __popcll(um);
    const bool uniq = (um >> lane) & 1ull;
    lwave_sync();
    if (done) {
      double* cand = R + RL.cand;
      for (int c = lane; c < D; c += 64) cand[c] = __longlong_as_double(0x7ff8000000000000ll);
      lwave_sync();
      if (uniq) cand[__popcll(um & below)] = thw;
    } else {
      if (uniq) R[RL.cand + __popcll(um & below)] = thw;
      if (lane == 0) {
        R[RL.meta + M_WARM] = (double)nu;
        const unsigned slot = atomicAdd(A.out_count, 1u);
        A.out_list[slot] = w;
      }
      ++left_acc;
    }
    lwave_sync();
  }
  if (lane == 0 && A.counters) {
    SolveCounters* c = counter_slot(A.counters);
    if (iters_acc) atomicAdd(&c->newton_iters, iters_acc);
    if (left_acc) atomicAdd(&c->fallback_aberth, left_acc);
  }
}

hipError_t launch_newton_retry(const RetryArgs& A, int waves, hipStream_t st) {
  hipLaunchKernelGGL(k_newton_retry, dim3((unsigned)waves), dim3(64), learn_lds_bytes(A.H), st, A);
  return hipGetLastError();
}

bool newton_four_per_wave(int H) { return 6 * H - 2 < 64; }

// Frequencies per wavefront of the first round: nc (a group of lanes each), fewer
// where that would leave less than `waves` wavefronts: their Newton iterations follow
// one another in a wavefront, so that few frequencies in few wavefronts wait for
// each other on an idle device.  A multiple of `step`, the frequencies Newton takes
// at once.  Measured on given sums, 2 / 4 / 8 per wavefront: H = 5 71 / 76 / 82 us at
// 100 frequencies, 91 / 97 / 106 at 4000, 104 / 104 / 111 at 8000, 128 / 121 / 126 at
// 16000.  H = 12, 1 / 2 / 3 / 4 per wavefront: 124 / 133 / 139 / 149 us at 100, 133 /
// 139 / 149 / 155 at 1000, 164 / 142 / 151 / 160 at 2000, 242 / 191 / 204 / 179 at 4000.
// So the line lies at eight wavefronts per compute unit up to H = 5 and at four above
// H = 11.
static int newton_per(int64_t np, int nc, int step, int64_t waves) {
  const int64_t per = (np + waves - 1) / waves;
  return (int)std::min<int64_t>(nc, (per + step - 1) / step * step);
}

template <int H, int G, bool FEW>
static void launch_newton_f(const SolveArgs& a, const LearnArgs& L, int waves, int occ, hipStream_t st, hipEvent_t done) {
  const size_t lds = (size_t)4 * (newton_top(6 * H - 2) + 2) * sizeof(double);   // f and its reversal of two frequencies
  const dim3 grid((unsigned)waves), block(64);
  if (occ == 6) hipExtLaunchKernelGGL((k_newton_sturm4<H, 6, G, FEW>), grid, block, lds, st, nullptr, done, 0, a, L);
  else hipExtLaunchKernelGGL((k_newton_sturm4<H, 5, G, FEW>), grid, block, lds, st, nullptr, done, 0, a, L);
}
template <int H, int G>
static void launch_newton_g(const SolveArgs& a, LearnArgs L, int waves, int occ, int n_cu, hipStream_t st,
                            hipEvent_t done) {
  if constexpr (6 * H - 2 < 32) {
    L.per = newton_per(L.np, 64 / G, 2, 8 * (int64_t)n_cu);
    if (L.per < 64 / G) return launch_newton_f<H, G, true>(a, L, waves, occ, st, done);
  }
  launch_newton_f<H, G, false>(a, L, waves, occ, st, done);
}

template <int H>
static void launch_newton_h(const SolveArgs& a, const LearnArgs& L, int waves, int occ, int n_cu, hipStream_t st,
                            hipEvent_t done) {
  if constexpr (sturm_lanes(H, 0) == 16) {
    if (sturm_lanes(H, L.np) == 16) return launch_newton_g<H, 16>(a, L, waves, occ, n_cu, st, done);
  }
  launch_newton_g<H, 8>(a, L, waves, occ, n_cu, st, done);
}

hipError_t launch_start_table(double2* out, int H, bool equal, hipStream_t st) {
  hipLaunchKernelGGL(k_start_table, dim3(1), dim3(512), 0, st, out, first_starts(H, equal));
  return hipGetLastError();
}

hipError_t launch_newton_sturm(const SolveArgs& a, LearnArgs L, int waves, int occ, int n_cu, hipStream_t st,
                               hipEvent_t done) {
  switch (a.H) {
#define FTP_NEWTON(h) case h: launch_newton_h<h>(a, L, waves, occ, n_cu, st, done); break;
    FTP_NEWTON(1) FTP_NEWTON(2) FTP_NEWTON(3) FTP_NEWTON(4) FTP_NEWTON(5)
    FTP_NEWTON(6) FTP_NEWTON(7) FTP_NEWTON(8) FTP_NEWTON(9) FTP_NEWTON(10)
#undef FTP_NEWTON
    default:
      const dim3 grid((unsigned)waves);
      const size_t lds = learn_lds_bytes(a.H);
      L.per = newton_per(L.np, 4, 1, 4 * (int64_t)n_cu);
      if (a.H == 11) hipExtLaunchKernelGGL((k_newton_sturm<1, false>), grid, dim3(64), lds, st, nullptr, done, 0, a, L);
      else if (L.per < 4) hipExtLaunchKernelGGL((k_newton_sturm<4, true>), grid, dim3(64), lds, st, nullptr, done, 0, a, L);
      else hipExtLaunchKernelGGL((k_newton_sturm<4, false>), grid, dim3(64), lds, st, nullptr, done, 0, a, L);
  }
  return hipGetLastError();
}

}  // namespace ftp

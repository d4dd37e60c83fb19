// All roots of the Cayley polynomial f by the Aberth-Ehrlich simultaneous
// iteration (O. Aberth, Math. Comp. 27 (1973); L. W. Ehrlich, Comm. ACM 10
// (1967)), one root per lane of a wavefront.  A project addition to the
// method: the paper takes the roots of the phase polynomial (Eq. finalpoly)
// from a companion-matrix eigensolver; this kernel reaches the same root set
// by a different iteration and feeds the same candidate scoring.
//
// Used as the second tier of the learned solve (frequencies whose Newton
// roots the Sturm count did not confirm) and as a solver of its own over all
// frequencies.  Stopping rule: a lane stops when its correction is at the
// rounding level of |z| or when |f(z)| is within 4 D u of sum |f_k| |z|^k (the
// root is exact for a polynomial perturbed at rounding level, the backward
// error test of Bini and Fiorentino's MPSolve).  Frequencies whose roots do
// not all stop within kAberthMaxIt sweeps go to the companion-matrix solve.
//
// Candidates: each root x maps back to the phase
//   theta = phi0 + atan2(Re x, 1 - Im x) + atan2(Re x, 1 + Im x),
// the argument of psi = e^{i phi0} (1 + i x) / (1 - i x), i.e. the projection
// of psi onto the unit circle (Section 2, after Eq. finalpoly); a conjugate pair gives the same
// phase twice.
#include "ftp_solve_common.h"
#include "ftp_args.h"

namespace ftp {

constexpr int kAberthMaxIt = 60;

__host__ __device__ inline size_t aberth_lds_bytes(int H) {
  const int D = 6 * H - 2;
  return (size_t)((D + 2) + 2 * D) * sizeof(double);
}

__device__ __forceinline__ void awave_sync() {
  __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
  __builtin_amdgcn_wave_barrier();
}

__global__ __launch_bounds__(64) void k_aberth(AberthArgs A) {
  // the fallback tiers run beside the side stream's scoring: their waves
  // take issue priority over it on a shared SIMD (the tiers are few, latency-bound
  // waves on the step's critical path)
  __builtin_amdgcn_s_setprio(2);
  extern __shared__ double sab[];
  const int lane = threadIdx.x & 63;
  const int H = A.H, D = 6 * H - 2;
  const RecLayout RL(H);
  double* fc = sab;                                         // D + 1 coefficients
  double2* zs = reinterpret_cast<double2*>(sab + (D + 2));  // D roots (16-byte aligned: D even)
  const int64_t n = A.list ? (int64_t)(*A.count) : A.np;
  constexpr double u = 1.1102230246251565e-16;
  unsigned long long its_acc = 0, qr_acc = 0;
  for (int64_t i = first_item(A.queue, lane); i < n; i = next_item(A.queue, lane, i)) {
    const int64_t w = A.list ? A.list[i] : i;
    double* R = A.rec + w * (int64_t)RL.stride;
    if (!A.list) {
      const int st = (int)R[RL.meta + M_STATUS];
      if (st == ST_BAD_LC || st == ST_CONSTANT) continue;
    }
    if (A.flags & 1u) {
      if (lane == 0) {
        const unsigned slot = atomicAdd(A.qr_count, 1u);
        A.qr_list[slot] = w;
        R[RL.meta + M_FALLBACK] = A.mark;
        ++qr_acc;
      }
      continue;
    }
    double fmaxabs = 0.0;
    for (int c = lane; c <= D; c += 64) fmaxabs = fmax(fmaxabs, fabs(R[RL.f + c]));
    fmaxabs = wave_max(fmaxabs);
    const double fs = fmaxabs > 0.0 ? 1.0 / fmaxabs : 1.0;
    for (int c = lane; c <= D; c += 64) fc[c] = R[RL.f + c] * fs;
    awave_sync();
    const double f0 = fc[0], fD = fc[D];
    double rho = pow(fabs(f0 / fD), 1.0 / D);
    if (!(rho > 1e-8 && rho < 1e8)) rho = 1.0;
    const bool act = lane < D;
    // starting points: the real roots a Newton tier already found
    // (x = tan((theta - phi0) / 2)), the others on a circle of radius rho
    const int nw = A.list ? (int)R[RL.meta + M_WARM] : 0;
    const double phi0s = R[RL.meta + M_PHI0];
    double zr = 0.0, zi = 0.0;
    if (act && lane < nw) {
      zr = tan(0.5 * (R[RL.cand + lane] - phi0s));
      if (!isfinite(zr)) zr = 1e8;
    } else if (act) {
      double sn, cs;
      sincos(kTwoPi * (lane - nw + 0.25) / (D - nw), &sn, &cs);
      zr = rho * cs;
      zi = rho * sn;
    }
    bool done = !act;
    int it = 0;
    for (; it < kAberthMaxIt; ++it) {
      if (act) zs[lane] = make_double2(zr, zi);
      awave_sync();
      if (!done) {
        const double az = sqrt(zr * zr + zi * zi);
        double rr = 0.0, ri = 0.0;   // f'(z) / f(z)
        // one Horner loop for every lane (no divergent branches): inside the
        // unit circle f at x = z; outside, the reversed polynomial
        // g(y) = y^D f(1/y) at x = y = 1/z, with f'/f = y (D - y g'/g)
        const bool inside = az <= 1.0;
        double xr = zr, xi = zi, ax = az;
        if (!inside) {
          const double iz2 = 1.0 / (az * az);
          xr = zr * iz2;
          xi = -zi * iz2;
          ax = 1.0 / az;
        }
        const int c0 = inside ? D : 0, cs = inside ? -1 : 1;   // coefficient of x^D, then step
        double pr = fc[c0], pi = 0.0, dr = 0.0, di = 0.0, ab = fabs(fc[c0]);
        for (int k = 1; k <= D; ++k) {
          const double c = fc[c0 + cs * k];
          const double tr = dr * xr - di * xi + pr;
          di = dr * xi + di * xr + pi;
          dr = tr;
          const double qr = pr * xr - pi * xi + c;
          pi = pr * xi + pi * xr;
          pr = qr;
          ab = ab * ax + fabs(c);
        }
        const double pm2 = pr * pr + pi * pi;
        const bool exact = !(sqrt(pm2) > 4.0 * D * u * ab);
        if (!exact) {
          const double inv = 1.0 / pm2;
          const double qr = (dr * pr + di * pi) * inv, qi = (di * pr - dr * pi) * inv;   // p'/p at x
          if (inside) {
            rr = qr;
            ri = qi;
          } else {
            const double sr = D - (xr * qr - xi * qi), si = -(xr * qi + xi * qr);       // D - y g'/g
            rr = xr * sr - xi * si;
            ri = xr * si + xi * sr;
          }
        }
        if (exact) {
          done = true;
        } else {
          // sum_{j != lane} 1 / (z - z_j): the j = lane term is 1/0 -> skipped
          // by a select, so the loop body has no branch and unrolls
          double sr = 0.0, si = 0.0;
#pragma unroll 4
          for (int j = 0; j < D; ++j) {
            const double2 zj = zs[j];
            const double er = zr - zj.x, ei = zi - zj.y;
            const double inv = j == lane ? 0.0 : fast_rcp_d(er * er + ei * ei);
            sr += er * inv;
            si -= ei * inv;
          }
          const double br = rr - sr, bi = ri - si;
          const double inv = fast_rcp_d(br * br + bi * bi);
          const double cr = br * inv, ci = -bi * inv;   // correction 1 / (f'/f - S)
          if (isfinite(cr) && isfinite(ci)) {
            zr -= cr;
            zi -= ci;
            if (sqrt(cr * cr + ci * ci) <= 4.0 * u * sqrt(zr * zr + zi * zi)) done = true;
          } else {
            done = true;   // coincident estimates: leave to the verdict below
          }
        }
      }
      awave_sync();
      if (__ballot(!done) == 0ull) break;
    }
    // verdict: every lane stopped with a finite root, and the roots add up to
    // -f_{D-1} / f_D (Vieta), which two estimates stuck on one root would break
    const bool finite = !act || (isfinite(zr) && isfinite(zi));
    double sx = act ? zr : 0.0, sy = act ? zi : 0.0, sa = act ? sqrt(zr * zr + zi * zi) : 0.0;
    sx = wave_sum(sx);
    sy = wave_sum(sy);
    sa = wave_sum(sa);
    const double ex = sx + fc[D - 1] / fD;
    const bool vieta = sqrt(ex * ex + sy * sy) <= 1e-8 * (sa + fabs(fc[D - 1] / fD)) + 1e-12;
    const bool ok = it < kAberthMaxIt && __ballot(!finite) == 0ull && vieta;
    its_acc += (unsigned long long)(it < kAberthMaxIt ? it + 1 : it);
    if (ok) {
      const double phi0 = R[RL.meta + M_PHI0];
      double* cand = R + RL.cand;
      if (act) cand[lane] = phi0 + atan2(zr, 1.0 - zi) + atan2(zr, 1.0 + zi);
    } else if (lane == 0) {
      const unsigned slot = atomicAdd(A.qr_count, 1u);
      A.qr_list[slot] = w;
      R[RL.meta + M_FALLBACK] = A.mark;
      ++qr_acc;
    }
    awave_sync();
  }
  if (lane == 0 && A.counters) {
    if (its_acc) atomicAdd(&counter_slot(A.counters)->aberth_iters, its_acc);
    if (qr_acc) atomicAdd(&counter_slot(A.counters)->fallback_qr, qr_acc);
  }
}

// The same iteration for the fallback tier (a list of a few frequencies, D <
// 64), eight lanes per root and a workgroup of ceil(D / 8) wavefronts per
// frequency: the GPU is otherwise idle while the tier runs, and its time is the
// slowest frequency's sweeps, a serial chain, so each sweep is split as finely
// as the reductions repay.  Lane q of a root's eight evaluates the powers c = q
// mod 8 of the polynomial (a_c = f_c inside the unit circle, f_{D-c} for the
// reversed one outside) by Horner in y = x^8, V = sum_q x^q P_q(y), V' = sum_q (q
// x^(q-1) P_q + 8 x^(q+7) P_q'), and sums 1 / (z - z_j) over j = q mod 8; the
// partials meet by DPP.  The roots are exchanged through LDS (two copies in turn,
// so that one barrier per sweep is enough).
//
// Bound by latency, and a tier of two frequencies by fetching its own code (a
// cold 64-byte line costs ~0.1 us): phases, radii and tests use the short forms
// that the bounds of a starting value or a test need, not the library's.  Two frequencies at
// D = 34 44 -> 34 us (13 sweeps each); 339 at D = 58 beside the scoring 111 -> 98 us.
// (Four wavefronts with one lane per root, partials through LDS, before, which took 6.2
// ms for 37700 frequencies at D = 58: so long a list fills the device, and the
// instructions of eight wavefronts per frequency, not their latency, count: 7.4 ms.)
constexpr int kAbL = 8;   // lanes per root
__host__ __device__ inline constexpr int aberth_waves(int D) { return (D + kAbL - 1) / kAbL; }

// Lists that give every resident wavefront (4096) more than five frequencies' shares
// this way are swept a wavefront per frequency instead (aberth_long): half the
// instructions for a frequency, whose roots share the powers of x and fill the lanes,
// in a chain four times as long.  Measured a workgroup / a wavefront per frequency:
// D = 58 51 / 213 us at 225 frequencies, 282 / 250 at 1900, 500 / 410 at 3800, 7.2 / 3.3
// ms at 37700; D = 46 512 / 441 at 4100; D = 34 195 / 246 at 1900, 376 / 404 at 3800, 907
// / 923 at 9300.
constexpr int64_t kAberthLong = 20480;

// Sum over a root's eight lanes, in all of them.
__device__ __forceinline__ double sum8(double v) {
  v += dpp_d<0xB1>(v);    // quad_perm [1, 0, 3, 2]
  v += dpp_d<0x4E>(v);    // quad_perm [2, 3, 0, 1]
  return v + dpp_d<0x141>(v);   // row_half_mirror
}

// The pieces of a sweep, with every rounding spelled out: a list is swept in one of
// two forms (below) by its length, and a frequency's roots are the same in both.
__device__ __forceinline__ double2 amul(double2 a, double2 b) {
  return make_double2(fma(a.x, b.x, -(a.y * b.y)), fma(a.x, b.y, a.y * b.x));
}
__device__ __forceinline__ double2 pick(bool c, double2 a, double2 b) { return make_double2(c ? a.x : b.x, c ? a.y : b.y); }

// The argument of a root's polynomial (z inside the unit circle, 1 / z of the
// reversed one outside) and the powers of it the residue classes share.
struct AberthPoint {
  bool inside;
  double2 x1, x2, x3, x4, x7, y;   // y = x^8
  double ay;                       // |y|
  __device__ __forceinline__ AberthPoint(double2 z) {
#pragma clang fp contract(off)
    const double az2 = fma(z.x, z.x, z.y * z.y);
    inside = az2 <= 1.0;
    x1 = z;
    double ax2 = az2;
    if (!inside) {
      ax2 = fast_rcp_d(az2);
      x1 = make_double2(z.x * ax2, -z.y * ax2);
    }
    x2 = amul(x1, x1);
    x4 = amul(x2, x2);
    y = amul(x4, x4);
    x3 = amul(x1, x2);
    x7 = amul(x3, x4);
    ay = (ax2 * ax2) * (ax2 * ax2);
  }
};

struct AberthPoly { double vr, vi, dr, di, ab; };   // V, V', sum |a_c| |x|^c

// Residue class q of the polynomial: xq = x^q, xm = x^(q-1) (anything for q = 0); a =
// coefficients q, q + 8, ..
__device__ __forceinline__ AberthPoly aberth_poly(const AberthPoint& X, double2 xq, double2 xm, int q, const double* a) {
#pragma clang fp contract(off)
  double2 p = make_double2(a[56], 0.0), d = make_double2(0.0, 0.0);
  double ab = fabs(a[56]);
#pragma unroll
  for (int c = 48; c >= 0; c -= 8) {
    const double cc = a[c];
    d = make_double2(fma(d.x, X.y.x, fma(-d.y, X.y.y, p.x)), fma(d.x, X.y.y, fma(d.y, X.y.x, p.y)));
    p = make_double2(fma(p.x, X.y.x, fma(-p.y, X.y.y, cc)), fma(p.x, X.y.y, p.y * X.y.x));
    ab = fma(ab, X.ay, fabs(cc));
  }
  const double2 v = amul(xq, p), m = amul(xm, p), h = amul(amul(xq, X.x7), d);
  return AberthPoly{v.x, v.y, fma(8.0, h.x, (double)q * m.x), fma(8.0, h.y, (double)q * m.y),
                    __builtin_amdgcn_sqrt(fma(xq.x, xq.x, xq.y * xq.y)) * ab};
}

// Residue class q of sum 1 / (z - z_j): zj(k) = root 8 k + q; the root itself (`self`)
// and j >= D, zeros there, are skipped; eight reciprocals side by side.
template <typename Z>
__device__ __forceinline__ double2 aberth_others(Z zj, double2 z, int q, int self, int D) {
#pragma clang fp contract(off)
  double2 e[8];
  double inv[8];
#pragma unroll
  for (int k = 0; k < 8; ++k) {
    const double2 o = zj(k);
    e[k] = make_double2(z.x - o.x, z.y - o.y);
  }
#pragma unroll
  for (int k = 0; k < 8; ++k) inv[k] = fast_rcp_d(fma(e[k].x, e[k].x, e[k].y * e[k].y));
  double2 s = make_double2(0.0, 0.0);
#pragma unroll
  for (int k = 0; k < 8; ++k) {
    const int j = 8 * k + q;
    const double iv = (j == self || j >= D) ? 0.0 : inv[k];
    s = make_double2(fma(e[k].x, iv, s.x), fma(-e[k].y, iv, s.y));
  }
  return s;
}

// Moves a root by its correction 1 / (f'/f - S); true once it has settled.
__device__ __forceinline__ bool aberth_move(const AberthPoint& X, const AberthPoly& S, double2 o, int D, double2& z) {
#pragma clang fp contract(off)
  constexpr double u = 1.1102230246251565e-16;
  const double pm2 = fma(S.vr, S.vr, S.vi * S.vi);
  const double tol = 4.0 * D * u * S.ab;
  if (!(pm2 > tol * tol)) return true;
  const double inv = fast_rcp_d(pm2);
  const double2 qq = make_double2(fma(S.dr, S.vr, S.di * S.vi) * inv, fma(S.di, S.vr, -(S.dr * S.vi)) * inv);   // q'/q at x
  double2 r = qq;
  if (!X.inside) {
    const double2 g = amul(X.x1, qq);
    r = amul(X.x1, make_double2(D - g.x, -g.y));      // x (D - x q'/q)
  }
  const double br = r.x - o.x, bi = r.y - o.y;
  const double inv2 = fast_rcp_d(fma(br, br, bi * bi));
  const double cr = br * inv2, ci = -bi * inv2;
  if (!(isfinite(cr) && isfinite(ci))) return true;   // coincident estimates: left to the verdict
  z.x -= cr;
  z.y -= ci;
  return fma(cr, cr, ci * ci) <= (16.0 * u * u) * fma(z.x, z.x, z.y * z.y);
}

// Scale of f, and the starting point of root `root` (the roots Newton left, tan of
// half their phase, then a circle), zero from D on.
__device__ __forceinline__ double aberth_scale(double fmaxabs) { return fmaxabs > 0.0 ? fast_rcp_d(fmaxabs) : 1.0; }
__device__ __forceinline__ double2 aberth_start(const double* R, const RecLayout& RL, double f0, double fD, int root, int D) {
  const int nw = (int)R[RL.meta + M_WARM];
  const double phi0 = R[RL.meta + M_PHI0];
  // |f_0 / f_D|^(1 / D), the radius of the starting circle (to single precision)
  const double rat = fabs(f0 * fast_rcp_d(fD));
  const float lg = __builtin_amdgcn_logf((float)__builtin_amdgcn_frexp_mant(rat)) + (float)__builtin_amdgcn_frexp_exp(rat);
  double rho = (double)__builtin_amdgcn_exp2f(lg / (float)D);
  if (!(rho > 1e-8 && rho < 1e8)) rho = 1.0;
  const bool warm = root < nw;
  const double ang = warm ? 0.5 * (R[RL.cand + root] - phi0) : kTwoPi * (root - nw + 0.25) * fast_rcp_d((double)(D - nw));
  double sn, cs;
  sincos_small(ang, sn, cs);
  double2 z = make_double2(0.0, 0.0);
  if (root < D) {
    z = warm ? make_double2(sn * fast_rcp_d(cs), 0.0) : make_double2(rho * cs, rho * sn);
    if (warm && !isfinite(z.x)) z.x = 1e8;
  }
  return z;
}

// The verdict on the roots (a lane each): all finite and their sum that of the
// polynomial's roots (Vieta).
__device__ __forceinline__ bool aberth_accept(double2 z, int lane, double fD1, double fD, int D) {
#pragma clang fp contract(off)
  const bool al = lane < D;
  const bool finite = !al || (isfinite(z.x) && isfinite(z.y));
  double sx = al ? z.x : 0.0, sy = al ? z.y : 0.0, sa = al ? __builtin_amdgcn_sqrt(fma(z.x, z.x, z.y * z.y)) : 0.0;
  sx = wave_sum(sx);
  sy = wave_sum(sy);
  sa = wave_sum(sa);
  const double ratio = fD1 * fast_rcp_d(fD), ex = sx + ratio;
  const bool vieta = __builtin_amdgcn_sqrt(fma(ex, ex, sy * sy)) <= fma(1e-8, sa + fabs(ratio), 1e-12);
  return __ballot(!finite) == 0ull && vieta;
}

// The candidates of accepted roots, phi0 + arg((1 - z.y + i z.x) (1 + z.y + i z.x)); a
// refused frequency goes to the companion solve's list.  All lanes of one wave.
__device__ __forceinline__ void aberth_finish(const AberthArgs& A, double* R, const RecLayout& RL, int64_t w, double2 z,
                                              int lane, int D, bool ok, unsigned long long& qr_acc) {
  if (ok) {
    double ud;
    int sg;
    u_from_dir(1.0 - fma(z.x, z.x, z.y * z.y), 2.0 * z.x, ud, sg);
    if (lane < D) R[RL.cand + lane] = theta_from_u(R[RL.meta + M_PHI0], ud, sg);
  } else if (lane == 0) {
    const unsigned slot = atomicAdd(A.qr_count, 1u);
    A.qr_list[slot] = w;
    R[RL.meta + M_FALLBACK] = A.mark;
    ++qr_acc;
  }
}

// A long list: a wavefront per frequency, a lane per root and the residue classes in
// turn, added in the order of sum8 (pairs, quads, both quads).
__device__ __forceinline__ void aberth_long(const AberthArgs& A, const RecLayout& RL, int D, int64_t n, double (*fc)[64],
                                            double2* zs, int lane, int64_t first, int64_t step,
                                            unsigned long long& its_acc, unsigned long long& qr_acc) {
  for (int64_t i = first; i < n; i += step) {
    const int64_t w = A.list[i];
    double* R = A.rec + w * (int64_t)RL.stride;
    const double fv = lane <= D ? R[RL.f + lane] : 0.0;
    const double fs = aberth_scale(wave_max(fabs(fv)));
    fc[0][lane] = fv * fs;
    fc[1][lane <= D ? D - lane : lane] = fv * fs;
    awave_sync();
    const double fD = fc[0][D];
    double2 z = aberth_start(R, RL, fc[0][0], fD, lane, D);
    bool done = lane >= D;
    int it = 0;
    for (; it < kAberthMaxIt; ++it) {
      zs[lane] = z;
      awave_sync();
      const AberthPoint X(z);
      const double* a = fc[X.inside ? 0 : 1];
      double2 to = make_double2(0.0, 0.0);
#pragma unroll 1
      for (int q4 = 0; q4 < 8; q4 += 4) {
        double2 qo = make_double2(0.0, 0.0);
#pragma unroll 1
        for (int q2 = q4; q2 < q4 + 4; q2 += 2) {
          double2 po = make_double2(0.0, 0.0);
#pragma unroll 1
          for (int q = q2; q < q2 + 2; ++q) po = cadd(po, aberth_others([&](int k) { return zs[8 * k + q]; }, z, q, lane, D));
          qo = cadd(qo, po);
        }
        to = cadd(to, qo);
      }
      auto add = [](AberthPoly& s, const AberthPoly& t) {
        s.vr += t.vr; s.vi += t.vi; s.dr += t.dr; s.di += t.di; s.ab += t.ab;
      };
      AberthPoly T{};
#pragma unroll 1
      for (int q4 = 0; q4 < 8; q4 += 4) {
        AberthPoly Q{};
#pragma unroll 1
        for (int q2 = q4; q2 < q4 + 4; q2 += 2) {
          AberthPoly P{};
#pragma unroll 1
          for (int q = q2; q < q2 + 2; ++q) {
            // (q is uniform; the products are those of the lanes' selections below)
            const double2 one = make_double2(1.0, 0.0);
            auto low = [&](int e) { return pick(e & 2, pick(e & 1, X.x3, X.x2), pick(e & 1, X.x1, one)); };
            const int qm = q > 0 ? q - 1 : 0;
            const double2 lo = low(q), lm = low(qm);
            const double2 xq = (q & 4) ? amul(lo, X.x4) : lo, xm = (qm & 4) ? amul(lm, X.x4) : lm;
            add(P, aberth_poly(X, xq, xm, q, a + q));
          }
          add(Q, P);
        }
        add(T, Q);
      }
      if (!done) done = aberth_move(X, T, to, D, z);
      awave_sync();
      if (__ballot(!done) == 0ull) break;
    }
    const bool ok = it < kAberthMaxIt && aberth_accept(z, lane, fc[0][D - 1], fD, D);
    if (lane == 0) its_acc += (unsigned long long)(it < kAberthMaxIt ? it + 1 : it);
    aberth_finish(A, R, RL, w, z, lane, D, ok, qr_acc);
    awave_sync();
  }
}

__global__ __launch_bounds__(64 * 8) __attribute__((amdgpu_waves_per_eu(4))) void k_aberth_split(AberthArgs A) {
  // the fallback tiers run beside the side stream's scoring: their waves
  // take issue priority over it on a shared SIMD (the tiers are few, latency-bound
  // waves on the step's critical path)
  __builtin_amdgcn_s_setprio(2);
  __shared__ double fcs[8][2][64];   // f and its reversal, zeros above D (per wave of a long list)
  __shared__ double2 zss[8][64];     // the roots (a short list: two copies)
  __shared__ int busy[2][8];         // wavefronts with roots still moving
  const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6, nwv = blockDim.x >> 6;
  const int root = tid >> 3, q = tid & 7;
  const int H = A.H, D = 6 * H - 2;
  const RecLayout RL(H);
  const int64_t n = (int64_t)(*A.count);
  unsigned long long its_acc = 0, qr_acc = 0;
  if (A.flags & 1u) {   // forced fallback
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + tid; i < n; i += (int64_t)gridDim.x * blockDim.x) {
      const int64_t w = A.list[i];
      const unsigned slot = atomicAdd(A.qr_count, 1u);
      A.qr_list[slot] = w;
      A.rec[w * (int64_t)RL.stride + RL.meta + M_FALLBACK] = A.mark;
      ++qr_acc;
    }
    if (qr_acc && A.counters) atomicAdd(&counter_slot(A.counters)->fallback_qr, qr_acc);
    return;
  }
  if (n * aberth_waves(D) > kAberthLong) {
    aberth_long(A, RL, D, n, fcs[wv], zss[wv], lane, (int64_t)blockIdx.x * nwv + wv, (int64_t)gridDim.x * nwv, its_acc, qr_acc);
    if (lane == 0 && A.counters) {
      if (its_acc) atomicAdd(&counter_slot(A.counters)->aberth_iters, its_acc);
      if (qr_acc) atomicAdd(&counter_slot(A.counters)->fallback_qr, qr_acc);
    }
    return;
  }
  double (*fc)[64] = fcs[0];
  double2 (*zs)[64] = zss;
  // (places of no root: zeros, made visible by the first barrier below)
  if (wv == 0) zs[0][lane] = zs[1][lane] = make_double2(0.0, 0.0);
  for (int64_t i = blockIdx.x; i < n; i += gridDim.x) {
    const int64_t w = A.list[i];
    double* R = A.rec + w * (int64_t)RL.stride;
    // every wave forms the same scale, starting points and verdict
    const double fv = lane <= D ? R[RL.f + lane] : 0.0;
    const double fs = aberth_scale(wave_max(fabs(fv)));
    if (wv == 0) {
      fc[0][lane] = fv * fs;
      fc[1][lane <= D ? D - lane : lane] = fv * fs;
    }
    __syncthreads();
    const double fD = fc[0][D];
    double2 z = aberth_start(R, RL, fc[0][0], fD, root, D);
    if (q == 0) zs[0][root] = z;
    __syncthreads();
    bool done = root >= D;
    int it = 0;
    for (; it < kAberthMaxIt; ++it) {
      const double2* zc = zs[it & 1];
      const AberthPoint X(z);
      const double2 one = make_double2(1.0, 0.0);
      const double2 xa = (q & 1) ? X.x1 : one, xb = (q & 2) ? X.x2 : one, xc = (q & 4) ? X.x4 : one;
      const int qm = q > 0 ? q - 1 : 0;
      const double2 ya = (qm & 1) ? X.x1 : one, yb = (qm & 2) ? X.x2 : one, yc = (qm & 4) ? X.x4 : one;
      double2 o = aberth_others([&](int k) { return zc[8 * k + q]; }, z, q, root, D);
      AberthPoly S = aberth_poly(X, amul(amul(xa, xb), xc), amul(amul(ya, yb), yc), q, fc[X.inside ? 0 : 1] + q);
      S.vr = sum8(S.vr);
      S.vi = sum8(S.vi);
      S.dr = sum8(S.dr);
      S.di = sum8(S.di);
      S.ab = sum8(S.ab);
      o = make_double2(sum8(o.x), sum8(o.y));
      if (!done) done = aberth_move(X, S, o, D, z);
      const int nb = (it + 1) & 1;
      if (q == 0) zs[nb][root] = z;
      const bool moving = __ballot(!done) != 0ull;
      if (lane == 0) busy[nb][wv] = moving;
      __syncthreads();
      int any = 0;
      for (int k = 0; k < nwv; ++k) any |= busy[nb][k];
      if (!any) break;   // the same in every wave
    }
    // the verdict, on the roots of the last sweep, a lane each
    const double2 zl = zs[(it < kAberthMaxIt ? it + 1 : it) & 1][lane];
    const bool ok = it < kAberthMaxIt && aberth_accept(zl, lane, fc[0][D - 1], fD, D);
    if (wv == 0) {
      its_acc += (unsigned long long)(it < kAberthMaxIt ? it + 1 : it);
      aberth_finish(A, R, RL, w, zl, lane, D, ok, qr_acc);
    }
    __syncthreads();   // LDS reused by the next frequency
  }
  if (tid == 0 && A.counters) {
    if (its_acc) atomicAdd(&counter_slot(A.counters)->aberth_iters, its_acc);
    if (qr_acc) atomicAdd(&counter_slot(A.counters)->fallback_qr, qr_acc);
  }
}

hipError_t launch_aberth(const AberthArgs& A, int waves, hipStream_t st) {
  if (6 * A.H - 2 > 64) {
    // degree above 64 (one root per lane does not fit): the tier hands its
    // list to the companion solve (the Aberth solver is refused at plan
    // creation for such H)
    AberthArgs F = A;
    F.flags |= 1u;
    hipLaunchKernelGGL(k_aberth, dim3((unsigned)waves), dim3(64), 0, st, F);
    return hipGetLastError();
  }
  if (A.list && 6 * A.H - 2 < 64) {
    // fallback tier: a workgroup per frequency, grid-strided over the list
    const int wpf = aberth_waves(6 * A.H - 2);
    hipLaunchKernelGGL(k_aberth_split, dim3((unsigned)std::max(1, waves / wpf)), dim3(64 * wpf), 0, st, A);
  } else {
    hipLaunchKernelGGL(k_aberth, dim3((unsigned)waves), dim3(64), aberth_lds_bytes(A.H), st, A);
  }
  return hipGetLastError();
}

}  // namespace ftp

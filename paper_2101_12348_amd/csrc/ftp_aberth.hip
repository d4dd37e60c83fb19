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
// (Four wavefronts with one lane per root, partials through LDS, before.)
constexpr int kAbL = 8;   // lanes per root
__host__ __device__ inline constexpr int aberth_waves(int D) { return (D + kAbL - 1) / kAbL; }

// Sum over a root's eight lanes, in all of them.
__device__ __forceinline__ double sum8(double v) {
  v += dpp_d<0xB1>(v);    // quad_perm [1, 0, 3, 2]
  v += dpp_d<0x4E>(v);    // quad_perm [2, 3, 0, 1]
  return v + dpp_d<0x141>(v);   // row_half_mirror
}

__global__ __launch_bounds__(64 * 8) void k_aberth_split(AberthArgs A) {
  // the fallback tiers run beside the side stream's scoring: their waves
  // take issue priority over it on a shared SIMD (the tiers are few, latency-bound
  // waves on the step's critical path)
  __builtin_amdgcn_s_setprio(2);
  __shared__ double fc[2][64];      // f and its reversal, zeros above D
  __shared__ double2 zs[2][64];     // the roots
  __shared__ int busy[2][8];        // wavefronts with roots still moving
  const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6, nwv = blockDim.x >> 6;
  const int root = tid >> 3, q = tid & 7;
  const int H = A.H, D = 6 * H - 2;
  const RecLayout RL(H);
  const int64_t n = (int64_t)(*A.count);
  constexpr double u = 1.1102230246251565e-16;
  unsigned long long its_acc = 0, qr_acc = 0;
  // (places of no root: zeros, made visible by the first barrier below)
  if (wv == 0) zs[0][lane] = zs[1][lane] = make_double2(0.0, 0.0);
  for (int64_t i = blockIdx.x; i < n; i += gridDim.x) {
    const int64_t w = A.list[i];
    double* R = A.rec + w * (int64_t)RL.stride;
    if (A.flags & 1u) {
      if (tid == 0) {
        const unsigned slot = atomicAdd(A.qr_count, 1u);
        A.qr_list[slot] = w;
        R[RL.meta + M_FALLBACK] = A.mark;
        ++qr_acc;
      }
      continue;
    }
    // every wave forms the same scale, starting points and verdict
    const double fv = lane <= D ? R[RL.f + lane] : 0.0;
    const int nw = (int)R[RL.meta + M_WARM];
    const double phi0 = R[RL.meta + M_PHI0];
    const double fmaxabs = wave_max(fabs(fv));
    const double fs = fmaxabs > 0.0 ? fast_rcp_d(fmaxabs) : 1.0;
    if (wv == 0) {
      fc[0][lane] = fv * fs;
      fc[1][lane <= D ? D - lane : lane] = fv * fs;
    }
    const bool act = root < D;
    double zr = 0.0, zi = 0.0;
    __syncthreads();
    const double f0 = fc[0][0], fD = fc[0][D];
    // |f_0 / f_D|^(1 / D), the radius of the starting circle (to single precision)
    const double rat = fabs(f0 * fast_rcp_d(fD));
    const float lg = __builtin_amdgcn_logf((float)__builtin_amdgcn_frexp_mant(rat)) + (float)__builtin_amdgcn_frexp_exp(rat);
    double rho = (double)__builtin_amdgcn_exp2f(lg / (float)D);
    if (!(rho > 1e-8 && rho < 1e8)) rho = 1.0;
    {
      // the roots Newton left (tan of half their phase), then the circle
      const bool warm = root < nw;
      const double ang = warm ? 0.5 * (R[RL.cand + root] - phi0) : kTwoPi * (root - nw + 0.25) * fast_rcp_d((double)(D - nw));
      double sn, cs;
      sincos_small(ang, sn, cs);
      if (act) {
        zr = warm ? sn * fast_rcp_d(cs) : rho * cs;
        zi = warm ? 0.0 : rho * sn;
        if (warm && !isfinite(zr)) zr = 1e8;
      }
    }
    if (q == 0) zs[0][root] = make_double2(zr, zi);
    __syncthreads();
    bool done = !act;
    int it = 0;
    for (; it < kAberthMaxIt; ++it) {
      const double2* zc = zs[it & 1];
      const double az2 = zr * zr + zi * zi;
      const bool inside = az2 <= 1.0;
      double xr = zr, xi = zi, ax2 = az2;
      if (!inside) {
        const double iz2 = fast_rcp_d(az2);
        xr = zr * iz2;
        xi = -zi * iz2;
        ax2 = iz2;
      }
      // x^q, x^(q-1) (0 for q = 0), x^(q+7), y = x^8 and the moduli
      const double2 x1 = make_double2(xr, xi), x2 = cmul(x1, x1), x4 = cmul(x2, x2), y = cmul(x4, x4);
      const double2 one = make_double2(1.0, 0.0);
      const double2 xa = (q & 1) ? x1 : one, xb = (q & 2) ? x2 : one, xc = (q & 4) ? x4 : one;
      const double2 xq = cmul(cmul(xa, xb), xc), x7 = cmul(cmul(x1, x2), x4);
      const int qm = q > 0 ? q - 1 : 0;
      const double2 ya = (qm & 1) ? x1 : one, yb = (qm & 2) ? x2 : one, yc = (qm & 4) ? x4 : one;
      const double2 xm = cmul(cmul(ya, yb), yc), xh = cmul(xq, x7);
      const double ay = (ax2 * ax2) * (ax2 * ax2), axq = __builtin_amdgcn_sqrt(xq.x * xq.x + xq.y * xq.y);
      const double* a = fc[inside ? 0 : 1] + q;
      double pr = a[56], pi = 0.0, dr = 0.0, di = 0.0, ab = fabs(a[56]);
#pragma unroll
      for (int c = 48; c >= 0; c -= 8) {
        const double cc = a[c];
        const double tr = dr * y.x - di * y.y + pr;
        di = dr * y.y + di * y.x + pi;
        dr = tr;
        const double qr = pr * y.x - pi * y.y + cc;
        pi = pr * y.y + pi * y.x;
        pr = qr;
        ab = ab * ay + fabs(cc);
      }
      // the roots' sum (j = root and j >= D, zeros here, skipped), eight reciprocals
      // side by side
      double sr = 0.0, si = 0.0;
      double2 e[8];
      double inv[8];
#pragma unroll
      for (int k = 0; k < 8; ++k) {
        const double2 zj = zc[8 * k + q];
        e[k] = make_double2(zr - zj.x, zi - zj.y);
      }
#pragma unroll
      for (int k = 0; k < 8; ++k) inv[k] = fast_rcp_d(e[k].x * e[k].x + e[k].y * e[k].y);
#pragma unroll
      for (int k = 0; k < 8; ++k) {
        const int j = 8 * k + q;
        const double iv = (j == root || j >= D) ? 0.0 : inv[k];
        sr += e[k].x * iv;
        si -= e[k].y * iv;
      }
      const double2 p = make_double2(pr, pi);
      const double2 v = cmul(xq, p);
      const double2 vd = cadd(cscale(cmul(xm, p), (double)q), cscale(cmul(xh, make_double2(dr, di)), 8.0));
      pr = sum8(v.x);
      pi = sum8(v.y);
      dr = sum8(vd.x);
      di = sum8(vd.y);
      sr = sum8(sr);
      si = sum8(si);
      ab = sum8(axq * ab);
      if (!done) {
        const double pm2 = pr * pr + pi * pi;
        const double tol = 4.0 * D * u * ab;
        const bool exact = !(pm2 > tol * tol);
        if (exact) {
          done = true;
        } else {
          const double inv = fast_rcp_d(pm2);
          const double qr = (dr * pr + di * pi) * inv, qi = (di * pr - dr * pi) * inv;   // q'/q at x
          double rr = qr, ri = qi;
          if (!inside) {
            const double s2r = D - (xr * qr - xi * qi), s2i = -(xr * qi + xi * qr);      // D - y g'/g
            rr = xr * s2r - xi * s2i;
            ri = xr * s2i + xi * s2r;
          }
          const double br = rr - sr, bi = ri - si;
          const double inv2 = fast_rcp_d(br * br + bi * bi);
          const double cr = br * inv2, ci = -bi * inv2;   // correction 1 / (f'/f - S)
          if (isfinite(cr) && isfinite(ci)) {
            zr -= cr;
            zi -= ci;
            if (cr * cr + ci * ci <= (16.0 * u * u) * (zr * zr + zi * zi)) done = true;
          } else {
            done = true;   // coincident estimates: leave to the verdict below
          }
        }
      }
      const int nb = (it + 1) & 1;
      if (q == 0) zs[nb][root] = make_double2(zr, zi);
      const bool moving = __ballot(!done) != 0ull;
      if (lane == 0) busy[nb][wv] = moving;
      __syncthreads();
      int any = 0;
      for (int k = 0; k < nwv; ++k) any |= busy[nb][k];
      if (!any) break;   // the same in every wave
    }
    // the verdict, on the roots of the last sweep, a lane each
    const double2 z = zs[(it < kAberthMaxIt ? it + 1 : it) & 1][lane];
    const bool al = lane < D;
    const bool finite = !al || (isfinite(z.x) && isfinite(z.y));
    double sx = al ? z.x : 0.0, sy = al ? z.y : 0.0, sa = al ? __builtin_amdgcn_sqrt(z.x * z.x + z.y * z.y) : 0.0;
    sx = wave_sum(sx);
    sy = wave_sum(sy);
    sa = wave_sum(sa);
    const double fD1 = fc[0][D - 1];
    const double ratio = fD1 * fast_rcp_d(fD), ex = sx + ratio;
    const bool vieta = __builtin_amdgcn_sqrt(ex * ex + sy * sy) <= 1e-8 * (sa + fabs(ratio)) + 1e-12;
    const bool ok = it < kAberthMaxIt && __ballot(!finite) == 0ull && vieta;
    if (wv == 0) {
      its_acc += (unsigned long long)(it < kAberthMaxIt ? it + 1 : it);
      if (ok) {
        // phi0 + arg((1 - z.y + i z.x) (1 + z.y + i z.x))
        double ud;
        int sg;
        u_from_dir(1.0 - (z.x * z.x + z.y * z.y), 2.0 * z.x, ud, sg);
        if (al) R[RL.cand + lane] = theta_from_u(phi0, ud, sg);
      } else if (lane == 0) {
        const unsigned slot = atomicAdd(A.qr_count, 1u);
        A.qr_list[slot] = w;
        R[RL.meta + M_FALLBACK] = A.mark;
        ++qr_acc;
      }
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

// Companion-matrix root step of the fast template periodogram (Section 2,
// after Eq. finalpoly): the eigenvalues of the real companion matrix of the
// Cayley polynomial f by Francis double-shift QR in LDS, each mapped back to
// psi and projected onto the unit circle (a complex pair gives one candidate).
#include <type_traits>

#include "ftp_solve_common.h"

namespace ftp {

namespace {

__device__ __forceinline__ void qr_sync() {
  __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
  __builtin_amdgcn_wave_barrier();
}

// 1/sqrt(s) and 1/d from the hardware estimates (better than 2^-22) refined
// by one third-order step each (a shorter dependent chain than two Newton
// steps; error a few ulp, the level to which a Householder step is backward
// stable).
__device__ __forceinline__ double rsq_refined(double s) {
  const double y = __builtin_amdgcn_rsq(s);
  const double e = fma(-(s * y), y, 1.0);
  return fma(y * e, fma(e, 0.375, 0.5), y);
}
__device__ __forceinline__ double rcp_refined(double d) {
  const double r = __builtin_amdgcn_rcp(d);
  const double e = fma(-d, r, 1.0);
  return fma(r, fma(e, e, e), r);
}

// Offset of a lane among its group's columns or rows.  A group of 32 lanes is
// two rows of 16; lanes 16..18 repeat lanes 0..2, so that a row broadcast
// reaches the whole group from lanes 0, 1 and 2.  kSpan: distinct offsets.
template <int G>
__device__ __forceinline__ int lane_offset(int hl) {
  if constexpr (G == 32) return hl < 16 ? hl : (hl < 19 ? hl - 16 : hl - 3);
  return hl;
}
template <int G>
constexpr int kSpan = G == 32 ? 29 : G;

// Value of the lanes with offset C (C <= 2) of each group, in every lane of
// the group: DPP row_newbcast within 16 lanes, v_readlane for the wavefront.
template <int G, int C>
__device__ __forceinline__ int group_bcast_i(int v) {
  if constexpr (G == 64) return __builtin_amdgcn_readlane(v, C);
  return __builtin_amdgcn_mov_dpp(v, 0x150 + C, 0xf, 0xf, true);
}
template <int G, int C>
__device__ __forceinline__ double group_bcast(double v) {
  const long long u = __double_as_longlong(v);
  const int lo = group_bcast_i<G, C>((int)u), hi = group_bcast_i<G, C>((int)(u >> 32));
  return __longlong_as_double(((long long)hi << 32) | (long long)(unsigned)lo);
}

// A value that is the same in all 64 lanes, as a scalar (G = 64: one matrix
// per wavefront, so its loop state is uniform).
template <int G>
__device__ __forceinline__ int uni(int v) {
  if constexpr (G == 64) return __builtin_amdgcn_readfirstlane(v);
  return v;
}

// Ballot over the lanes of this lane's group, bit hl = the group's lane hl.
template <int G>
__device__ __forceinline__ unsigned long long group_ballot(bool p, int lane) {
  const unsigned long long b = __ballot(p);
  if constexpr (G == 64) return b;
  return (b >> (lane & ~(G - 1))) & ((1ull << G) - 1ull);
}

// Reflector I - beta u u^T, u = (x - al, y, z), which takes (x, y, z) to
// (al, 0, 0), al = -sign(x) |(x, y, z)|; the identity when the column vanishes
// or `on` is false.
struct Reflector {
  double u0, u1, u2, beta, al;
  __device__ __forceinline__ Reflector(double x, double y, double z, bool on) : u1(y), u2(z) {
    const double s2 = fma(z, z, fma(y, y, x * x));
    const bool nz = s2 > 1e-290 && on;
    const double nrm = nz ? s2 * rsq_refined(s2) : 0.0;
    al = copysign(nrm, -x);
    u0 = x - al;
    beta = nz ? rcp_refined(fma(nrm, fabs(x), s2)) : 0.0;
  }
  __device__ __forceinline__ double dot(double a, double b, double c) const {
    return beta * fma(u0, a, fma(u1, b, u2 * c));
  }
  __device__ __forceinline__ void apply(double& a, double& b, double& c) const {
    const double w = dot(a, b, c);
    a = fma(-w, u0, a);
    b = fma(-w, u1, b);
    c = fma(-w, u2, c);
  }
  __device__ __forceinline__ double first(double a, double b, double c) const { return fma(-dot(a, b, c), u0, a); }
};

// Word of LDS at a byte address.
typedef __attribute__((address_space(3))) double lds_double;
__device__ __forceinline__ lds_double& lds(unsigned byte) { return *(lds_double*)byte; }

}  // namespace

// Storage of an N x N upper Hessenberg matrix in LDS: column j holds rows 0 ..
// j + 3 at hcol(j) + i, the Hessenberg band and the bulge of the chase (zero
// below the subdiagonal outside the bulge).
__host__ __device__ inline constexpr int hcol(int j) { return j * (j + 7) / 2; }
// doubles per matrix: the columns, N words that stay zero in place of the
// columns past the last (a sweep's last steps) and words that idle lanes read
// and write, each lane its own
__host__ __device__ inline constexpr int qr_doubles(int N, int G) { return (hcol(N) + N + G + 3 + 1) & ~1; }

// Eigenvalues of companion matrices for the pairs of a chunk (or of a list of
// them), one matrix per group of G lanes, 64 / G per wavefront.  Candidates
// theta_rel (relative to t_ref) go to rec.cand; NaN marks none.  Every matrix
// sees the same arithmetic whatever G is.
//
// The matrix of f (first row -f[N-1-j] / f[N], ones below the diagonal) is
// balanced by powers of two before the iteration (without it the Cayley
// polynomial's spread of coefficients, binomial growth with N, costs the
// roots their accuracy).  For a companion matrix the balanced scaling is
// known: with E_j the upper concave hull of log2 |coefficients| in falling
// degree, the diagonal 2^-E_j leaves in row and column j the moduli the hull's
// slopes give the j-th and next largest roots, so every row and column norm
// agrees within a small factor.  The hull is raised from the points by
// midpoint steps at halving strides, which is enough for a scaling (the roots
// come out as accurate as after iterated balancing, N = 4 .. 88).
//
// The iteration is EISPACK hqr's (eigenvalues only): deflation at negligible
// subdiagonals, double shifts from the trailing 2 x 2, exceptional shifts at 10
// and 20 sweeps.  A pass of the chase takes two steps (rows k..k+3, then
// columns k..k+3), a lane on one column of the row update and one row of the
// column update, so a window of up to G columns needs one pass, and the next
// bulge column comes from three lanes of the group.  Groups are independent:
// each carries its own window, a group between sweeps looks for deflations
// (phase A) while the others wait, and one instruction stream chases every
// group's bulge (phase B).
//
// Bound: a pass is one serial chain (two reflectors, an LDS round trip, the
// broadcasts) of ~170 instructions that a lone wavefront issues in ~1700
// cycles, so throughput is the matrices in flight (LDS capacity: ten per CU at
// N = 58) until the vector issue limits it (near half of its slots are used).
// Two steps per pass halve the LDS traffic and share the addressing; packed
// columns double the matrices in flight against a dense matrix.  Measured
// against one dense or packed matrix per wavefront with one step per pass
// (50 000 frequencies, whole periodogram): N = 16 3.24 -> 1.19 ms, N = 28 8.1 ->
// 3.4, N = 34 11.4 -> 5.8, N = 58 50.7 -> 25.3, N = 70 160 -> 44.5, N = 88 481 ->
// 100 ms; 497 matrices of N = 16 (one per wavefront) 202 -> 120 us.
template <int N, int G>
__global__ __launch_bounds__(64) void k_qr(double* rec, int stride, int64_t np, const int64_t* list,
                                           const unsigned int* list_count, SolveCounters* counters,
                                           unsigned* queue) {
  // the fallback tiers run beside the side stream's scoring: their waves
  // take issue priority over it on a shared SIMD (the tiers are few, latency-bound
  // waves on the step's critical path)
  __builtin_amdgcn_s_setprio(2);
  extern __shared__ double smq[];
  constexpr int NG = 64 / G, SL = (N + G - 1) / G, MD = qr_doubles(N, G);
  const int lane = threadIdx.x & 63, hl = lane & (G - 1), g = lane / G, ho = lane_offset<G>(hl);
  double* P = smq + g * MD;
  const RecLayout RL((N + 2) / 6);
  const int64_t total = list ? (int64_t)*list_count : np;
  const int64_t units = (total + NG - 1) / NG;
  unsigned long long sweeps_acc = 0;
  for (int64_t u = first_item(queue, lane); u < units; u = next_item(queue, lane, u)) {
    const int64_t item = u * NG + g;
    bool have = item < total;
    const int64_t q = have ? (list ? list[item] : item) : 0;
    double* R = rec + q * (int64_t)stride;
    const int st = have ? (int)R[RL.meta + M_STATUS] : (int)ST_BAD_LC;
    have = have && st != ST_BAD_LC && st != ST_CONSTANT;
    if (__ballot(have) == 0ull) continue;
    // ---- the balanced companion matrix
    {
      const double* f = R + RL.f;
      const double lead = have ? f[N] : 1.0;
      double a[SL];
      float* E = reinterpret_cast<float*>(P);   // E[j + 1] = log2 |a_j|, E[0] = 0, raised to the hull
      float ev[SL];
#pragma unroll
      for (int s = 0; s < SL; ++s) {
        const int j = hl + G * s;
        a[s] = (have && j < N) ? -f[N - 1 - j] / lead : 0.0;
        const float m = (float)fabs(__builtin_amdgcn_frexp_mant(a[s]));
        ev[s] = fminf(fmaxf((float)__builtin_amdgcn_frexp_exp(a[s]) + __log2f(m), -4000.f), 4000.f);
        if (j < N) E[j + 1] = ev[s];
      }
      if (hl == 0) E[0] = 0.f;
      qr_sync();
      constexpr int S0 = N >= 64 ? 32 : N >= 32 ? 16 : N >= 16 ? 8 : N >= 8 ? 4 : N >= 4 ? 2 : 1;   // <= N / 2
#pragma unroll 1
      for (int t = 2 * S0; t > 1; t >>= 1) {
        const int s0 = t >> 1;
#pragma unroll 1
        for (int rep = 0; rep < 2; ++rep) {
#pragma unroll
          for (int s = 0; s < SL; ++s) {
            const int j = hl + G * s + 1;
            if (j >= s0 && j + s0 <= N) ev[s] = fmaxf(ev[s], 0.5f * (E[j - s0] + E[j + s0]));
          }
          qr_sync();
#pragma unroll
          for (int s = 0; s < SL; ++s) {
            const int j = hl + G * s + 1;
            if (j <= N) E[j] = ev[s];
          }
          qr_sync();
        }
      }
      int e0[SL], e1[SL];
#pragma unroll
      for (int s = 0; s < SL; ++s) {
        const int j = hl + G * s;
        e0[s] = j <= N ? (int)rintf(E[j]) : 0;
        e1[s] = j < N ? (int)rintf(ev[s]) : 0;
      }
      qr_sync();
      for (int i = hl; i < MD; i += G) P[i] = 0.0;
      qr_sync();
#pragma unroll
      for (int s = 0; s < SL; ++s) {
        const int j = hl + G * s;
        if (j < N) {
          P[hcol(j)] = ldexp(a[s], -e0[s]);
          if (j + 1 < N) P[hcol(j) + j + 1] = ldexp(1.0, e1[s] - e0[s]);
        }
      }
      qr_sync();
    }
    // ---- QR iteration: window [l, m] of each group, bulge at k.  mm = m while
    // a bulge is chased, -1 between sweeps, -2 once the matrix is done.
    // Addresses are LDS byte addresses that a pass advances by adding: ra of
    // (k, k + ho), the row update's first word; ca of (k + 4 - ho, k), the
    // column update's; za of that row in column N; kv = 8 (k + 4) is the distance
    // of columns k and k + 1.
    const unsigned gb = (unsigned)(uintptr_t)(lds_double*)P;
    const unsigned gt = gb + 8u * (unsigned)(hcol(N) + N + hl), h16 = 16u * (unsigned)ho + 24u;
    int m = have ? N - 1 : -1, mm = have ? -1 : -2, lo = 0, l = 0, k = 0, its = 0, sweeps = 0;
    int lw = 0;   // l in the lanes of offset 0, past every k in the others
    unsigned ra = gt, ca = gt, za = gt, kv = 32u;
    constexpr int maxit = 30 * N;
    bool failed = false;
    double x = 0.0, y = 0.0, z = 0.0;
    for (;;) {
      mm = uni<G>(mm);
      // phase A: deflation, shifts, the next bulge
      if (mm == -1) {
        m = uni<G>(m);
        const int m1 = m > 0 ? m - 1 : 0;
        const double d = P[hcol(m) + m], b = P[hcol(m) + m1];
        const double aa = P[hcol(m1) + m1], c = P[hcol(m1) + m1 + 1];
        // the entries a sweep from lo starts with, in case the block holds
        int q0 = hcol(lo) + lo, q1 = q0 + lo + 4;
        double all = P[q0], al1 = P[q0 + 1], f0 = P[q1], f1 = P[q1 + 1], f2 = P[q1 + 2];
        // largest row of the block with a negligible subdiagonal entry
        l = lo;
#pragma unroll
        for (int p = SL - 1; p >= 0; --p) {
          const int top = m - G * p, i = top - hl;
          if (p > 0 && __ballot(top > lo) == 0ull) continue;
          const int ii = i > lo ? i : 1;
          const int qi = hcol(ii - 1) + ii;
          const double s1 = fabs(P[qi - 1]) + fabs(P[qi + ii + 3]);   // X(i-1, i-1), X(i, i)
          // both diagonal entries zero: against the matrix's scale, which
          // balancing brings near 1
          const bool ok = i > lo && fabs(P[qi]) <= kEps * (s1 == 0.0 ? 1.0 : s1);
          const unsigned long long hit = group_ballot<G>(ok, lane);
          l = hit ? top - (__ffsll((long long)hit) - 1) : l;
        }
        l = uni<G>(l);
        const int lo0 = lo;
        lo = l;
        if (l >= m - 1) {
          // one or two eigenvalues: real part on the diagonal, imaginary
          // part below it (column m is not touched any more)
          double r1 = d, i1 = 0.0;
          if (l < m) {
            const double p = 0.5 * (aa - d), qd = fma(p, p, b * c);
            const double zq = fabs(qd) > 1e-290 ? fabs(qd) * rsq_refined(fabs(qd)) : 0.0;
            double r0, i0 = 0.0;
            if (qd >= 0.0) {
              const double zz = p + copysign(zq, p);
              r0 = d + zz;
              r1 = zz != 0.0 ? fma(-b * c, rcp_refined(zz), d) : r0;
            } else {
              r0 = r1 = d + p;
              i0 = zq;
              i1 = -zq;
            }
            if (hl == 0) {
              P[hcol(m1) + m1] = r0;
              P[hcol(m1) + m1 + 1] = i0;
            }
          }
          if (hl == 0) {
            P[hcol(m) + m] = r1;
            P[hcol(m) + m + 1] = i1;
          }
          // what is left of the block, or everything above it
          m = l - 1;
          its = 0;
          lo = m >= lo0 ? lo0 : 0;
          mm = m >= 0 ? -1 : -2;
        } else if (sweeps >= maxit) {
          // the remaining diagonal serves as estimates (real)
          for (int i = hl; i <= m; i += G) P[hcol(i) + i + 1] = 0.0;
          failed = true;
          mm = -2;
        } else {
          double S = aa + d, T = aa * d - b * c;
          if (its == 10 || its == 20) {
            const double sx = fabs(c) + fabs(P[hcol(m - 2) + m - 1]);
            const double cc = d + 0.75 * sx;
            S = 2.0 * cc;
            T = cc * cc - 0.4375 * sx * sx;
          }
          ++its;
          ++sweeps;
          if (l != lo0) {
            q0 = hcol(l) + l;
            q1 = q0 + l + 4;
            all = P[q0];
            al1 = P[q0 + 1];
            f0 = P[q1];
            f1 = P[q1 + 1];
            f2 = P[q1 + 2];
          }
          x = all * all + f0 * al1 - S * all + T;
          y = al1 * (all + f1 - S);
          z = f2 * al1;
          k = l;
          lw = ho == 0 ? l : N;
          mm = m;
          ra = gb + 8u * (unsigned)(hcol(l + ho) + l);
          ca = gb + 8u * (unsigned)(q0 + 4 - ho);
          za = gb + 8u * (unsigned)(hcol(N) + l + 4 - ho);
          kv = 8u * (unsigned)(l + 4);
        }
      }
      qr_sync();
      mm = uni<G>(mm);
      if (__ballot(mm != -2) == 0ull) break;
      do {
        k = uni<G>(k);
        kv = (unsigned)uni<G>((int)kv);
        mm = uni<G>(mm);
        // phase B: two chase steps (k and k + 1) of every group that has a bulge:
        // both reflectors are applied to the rows, then both to the columns
        // (products from the left and from the right commute).
        // Row update of rows k..k+3: a lane on column k + ho
        const bool rv = k + ho <= mm;
        const unsigned ar = rv ? ra : gt;
        double b0 = lds(ar), b1 = lds(ar + 8), b2 = lds(ar + 16), b3 = lds(ar + 24);
        __builtin_amdgcn_sched_barrier(0);   // the loads' latency under the reflector's
        const Reflector r1(x, y, z, true);
        r1.apply(b0, b1, b2);
        // the second bulge column, rows k+1..k+3 of column k after the first step:
        // the 3 x 3 block below row k after its row update, from the lanes of
        // columns k, k+1 and k+2 (row k + 3 is zero at k and k + 1), then its
        // column update.  No second step at k = m - 1; no row k + 3 at k = m - 2.
        const bool two = k + 2 <= mm, three = k + 3 <= mm;
        double x2, y2, z2;
        {
          const double p1 = group_bcast<G, 0>(b1), q1 = group_bcast<G, 1>(b1), t1 = group_bcast<G, 2>(b1);
          const double p2 = group_bcast<G, 0>(b2), q2 = group_bcast<G, 1>(b2), t2 = group_bcast<G, 2>(b2);
          const double h = group_bcast<G, 2>(b3);
          x2 = r1.first(p1, q1, t1);
          y2 = r1.first(p2, q2, t2);
          z2 = three ? -(r1.beta * z * h) * r1.u0 : 0.0;
        }
        const Reflector r2(x2, y2, z2, two);
        r2.apply(b1, b2, b3);
        lds(ar) = b0;
        lds(ar + 8) = b1;
        lds(ar + 16) = b2;
        lds(ar + 24) = b3;
        auto row_pass = [&](auto self, auto P1) -> void {
          constexpr int p = decltype(P1)::value, W = kSpan<G> * p;
          if constexpr (W < N) {
            if (__ballot(k + W <= mm)) {
              const unsigned a = k + ho + W <= mm ? ra + 8u * (unsigned)(W * (k + ho) + W * (W + 7) / 2) : gt;
              double e0 = lds(a), e1 = lds(a + 8), e2 = lds(a + 16), e3 = lds(a + 24);
              r1.apply(e0, e1, e2);
              r2.apply(e1, e2, e3);
              lds(a) = e0;
              lds(a + 8) = e1;
              lds(a + 16) = e2;
              lds(a + 24) = e3;
              self(self, std::integral_constant<int, p + 1>{});
            }
          }
        };
        row_pass(row_pass, std::integral_constant<int, 1>{});
        // the bulge column k - 1 becomes (al, 0, 0) (none in the first step: the
        // negligible entry at (l, l - 1) marks where the block ends)
        {
          const unsigned a = rv && k > lw ? ra - kv : gt - 8u;
          lds(a + 8) = r1.al;
          lds(a + 16) = 0.0;
          lds(a + 24) = 0.0;
        }
        qr_sync();
        // column update of columns k..k+3, rows l..min(k + 4, m): a lane on row
        // k + 4 - ho.  (Row k + 4 has no word at column k and zeros at k + 1 and
        // k + 2; columns past m meet zero components of the reflectors and stay
        // as they are.)  Column k is left with its second reflector's value at
        // row k + 1 and zeros below.
        double c1n = 0.0;
        const int i = k + 4 - ho;
        if (i >= l && i <= mm) {
          const unsigned a0 = ho == 0 ? za : ca, a1 = ca + kv, a2u = a1 + kv + 8u;
          const unsigned a2 = min(a2u, za), a3 = min(a2u + kv + 16u, za);
          double c0 = lds(a0), c2 = lds(a2), c3 = lds(a3);
          c1n = lds(a1);
          r1.apply(c0, c1n, c2);
          r2.apply(c1n, c2, c3);
          lds(a0) = ho < 3 ? 0.0 : c0;
          lds(a1) = c1n;
          lds(a2) = c2;
          lds(a3) = c3;
        }
        auto col_pass = [&](auto self, auto P1) -> void {
          constexpr int p = decltype(P1)::value, W = kSpan<G> * p;
          if constexpr (W < N + 4) {
            if (__ballot(mm >= 0 && k + 4 - W >= l)) {
              if (mm >= 0 && i - W >= l) {
                const unsigned a0 = ca - 8u * W, a1 = a0 + kv, a2u = a1 + kv + 8u;
                const unsigned a2 = min(a2u, za - 8u * W), a3 = min(a2u + kv + 16u, za - 8u * W);
                double c0 = lds(a0), c1 = lds(a1), c2 = lds(a2), c3 = lds(a3);
                r1.apply(c0, c1, c2);
                r2.apply(c1, c2, c3);
                lds(a0) = c0;
                lds(a1) = c1;
                lds(a2) = c2;
                lds(a3) = c3;
              }
              self(self, std::integral_constant<int, p + 1>{});
            }
          }
        };
        col_pass(col_pass, std::integral_constant<int, 1>{});
        qr_sync();
        // next bulge column: rows k+2..k+4 of column k+1 (a row past the window:
        // zero)
        x = group_bcast<G, 2>(c1n);
        y = group_bcast<G, 1>(c1n);
        z = group_bcast<G, 0>(c1n);
        ra += 2u * kv + h16;
        ca += 2u * kv + 24u;
        za += 16u;
        kv += 16u;
        k += 2;
        mm = k < mm ? mm : (mm < -1 ? mm : -1);
      } while (__ballot(mm == -1) == 0ull);
    }
    qr_sync();
    // ---- eigenvalues to candidates
    sweeps_acc += (unsigned long long)(have && hl == 0 ? sweeps : 0);
    if (have && failed && hl == 0) R[RL.meta + M_STATUS] = (double)ST_NO_CONVERGE;
    const double phi0 = have ? R[RL.meta + M_PHI0] : 0.0;
    unsigned long long rm = 0ull;
    unsigned rx = 0u;
#pragma unroll
    for (int s = 0; s < SL; ++s) {
      const int c = hl + G * s;
      bool real = false;
      if (have && c < N) {
        const double xr = P[hcol(c) + c], xi = P[hcol(c) + c + 1];
        double th = __longlong_as_double(0x7ff8000000000000ll);
        if (xi >= 0.0 && isfinite(xr) && isfinite(xi)) th = phi0 + atan2(xr, 1.0 - xi) + atan2(xr, 1.0 + xi);
        real = xi == 0.0 && isfinite(xr);
        R[RL.cand + c] = th;
      }
      const unsigned long long b = group_ballot<G>(real, lane);
      if (G * s < 64) rm |= b << ((G * s) & 63);
      else rx |= (unsigned)b << ((G * s - 64) & 31);
    }
    if (have && hl == 0) {
      R[RL.meta + M_REAL_LO] = (double)(unsigned)(rm & 0xffffffffull);
      R[RL.meta + M_REAL_HI] = (double)(unsigned)(rm >> 32);
      R[RL.meta + M_REAL_X] = (double)rx;
    }
    qr_sync();
  }
  if (counters && hl == 0 && sweeps_acc) atomicAdd(&counter_slot(counters)->qr_sweeps, sweeps_acc);
}

template <int N, int G>
static hipError_t launch_qr_g(double* rec, int stride, int64_t np, const int64_t* list, const unsigned* list_count,
                              SolveCounters* counters, unsigned* queue, int waves, hipStream_t st) {
  const int64_t units = (np + 64 / G - 1) / (64 / G);
  const unsigned grid = (unsigned)(waves < units ? waves : units);
  hipLaunchKernelGGL((k_qr<N, G>), dim3(grid), dim3(64), (64 / G) * qr_doubles(N, G) * sizeof(double), st, rec, stride, np,
                     list, list_count, counters, queue);
  return hipGetLastError();
}

// Lanes per matrix when there are many: the fewest for which a window still
// fits a pass or two and the LDS still holds several wavefronts per SIMD.
// Measured on 50 000 frequencies with 16 / 32 / 64 lanes: N = 28 3.39 / 3.80 /
// 6.08 ms, N = 34 6.00 / 5.84 / 8.42, N = 58 43.7 / 25.3 / 25.5, N = 64 55.0 /
// 36.7 / 33.5.
constexpr int qr_group(int N) { return N <= 28 ? 16 : N <= 58 ? 32 : 64; }

template <int N>
static hipError_t launch_qr_n(double* rec, int stride, int64_t np, const int64_t* list, const unsigned* list_count,
                              SolveCounters* counters, unsigned* queue, int waves, bool many, hipStream_t st) {
  if (many) return launch_qr_g<N, qr_group(N)>(rec, stride, np, list, list_count, counters, queue, waves, st);
  return launch_qr_g<N, 64>(rec, stride, np, list, list_count, counters, queue, waves, st);
}

// `many`: enough matrices to fill the device with several per wavefront; else
// one wavefront per matrix.
hipError_t launch_qr(int H, double* rec, int stride, int64_t np, const int64_t* list, const unsigned* list_count,
                     SolveCounters* counters, unsigned* queue, int waves, bool many, hipStream_t st) {
#define FTP_QR_CASE(h) \
  case h: return launch_qr_n<6 * h - 2>(rec, stride, np, list, list_count, counters, queue, waves, many, st)
  switch (H) {
    FTP_QR_CASE(1);
    FTP_QR_CASE(2);
    FTP_QR_CASE(3);
    FTP_QR_CASE(4);
    FTP_QR_CASE(5);
    FTP_QR_CASE(6);
    FTP_QR_CASE(7);
    FTP_QR_CASE(8);
    FTP_QR_CASE(9);
    FTP_QR_CASE(10);
    FTP_QR_CASE(11);
    FTP_QR_CASE(12);
    FTP_QR_CASE(13);
    FTP_QR_CASE(14);
    FTP_QR_CASE(15);
    default: return hipErrorInvalidValue;
  }
#undef FTP_QR_CASE
}

}  // namespace ftp

// Per-frequency stage of the fast template periodogram: the method's phase
// polynomial (Section 2, Eq. finalpoly), its roots as the eigenvalues of a
// companion matrix, and the scoring of every root (Section 2: the phase
// condition is necessary, not sufficient, so each solution is scored).
//
// Three kernels, each with as many trial frequencies per wavefront as fill it,
// exchanging a per-pair record through HBM (RecLayout):
//   k_assemble : gather and deconvolve the NFFT sums (or read given sums);
//                assemble mu (MM), eta (YM) and the trig coefficients r_d of
//                R(theta) = i psi^{-K} p(psi), K = 3H - 1; pick a rotation
//                phi0 among 16 that maximises |R(phi0 + pi)|; expand the
//                Cayley polynomial f(x) = (1 + x^2)^K R(phi0 + 2 atan x), a real
//                polynomial of degree D = 6H - 2 whose real roots are the real
//                phases (leading coefficient R(phi0 + pi));
//   k_qr       : eigenvalues of the real companion matrix of f (ftp_qr.hip);
//   k_score    : P = YM^2 / (YY MM) at every candidate, best by P with the
//                documented tie rule, Newton polish on R(theta) kept only if P
//                does not drop, outputs theta_2, theta_1, theta_3 (k_score4: the
//                same for Newton's roots up to H = 10, without the polish).
#include <hip/hip_ext.h>
#include "ftp_solve_common.h"

namespace ftp {

__device__ __forceinline__ int wave_lane() { return threadIdx.x & 63; }

// Orders this wave's LDS accesses (LDS operations of one wavefront are
// performed in program order, so a compiler fence at wavefront scope is
// enough; every workgroup here is a single wave).
__device__ __forceinline__ void wave_sync() {
  __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
  __builtin_amdgcn_wave_barrier();
}

// f_c = sum_j rc[j] T[c][j], j = 0..K, over row c of the Cayley table (rows of
// cayley_row(K) doubles, 16-byte aligned like rc), in two sums, even and odd j.
__device__ __forceinline__ double cayley_dot(const double* rc, const double* row, int K) {
  double acc0 = 0.0, acc1 = 0.0;
  const double2* r2 = reinterpret_cast<const double2*>(rc);
  const double2* t2 = reinterpret_cast<const double2*>(row);
  const int n2 = (K + 1) >> 1;
#pragma unroll 4
  for (int i = 0; i < n2; ++i) {
    const double2 r = r2[i], t = t2[i];
    acc0 = fma(r.x, t.x, acc0);
    acc1 = fma(r.y, t.y, acc1);
  }
  if (!(K & 1)) acc0 = fma(rc[K], row[K], acc0);
  return acc0 + acc1;
}

// ------------------------------------------------------------- assemble

// Per-frequency working set of k_assemble:
// Z, mu, eta, r and a scratch of 8H + 2 complex values (assemble_r's MM and YM
// coefficient rows; later the rotated 2 rho_j, two rows of cayley_row(K)).
__host__ __device__ inline int asm2_doubles(int H) {
  return 2 * ((3 * H + 1) + (2 * H + 1) + (H + 1) + 3 * H + (8 * H + 2));
}
__device__ __forceinline__ FreqWork asm2_layout(double* sm, int H, double2*& scr) {
  FreqWork W;
  double2* q = reinterpret_cast<double2*>(sm);
  W.Z = q; q += 3 * H + 1;
  W.mu = q; q += 2 * H + 1;
  W.eta = q; q += H + 1;
  W.r = q; q += 3 * H;
  W.al = nullptr;
  scr = q;
  return W;
}
// Waves per workgroup of k_assemble: they share one LDS copy of the Cayley
// table (14 KB at H = 10) and of the template's products, which the loops read
// with LDS latency instead of the L2's.
constexpr int kAsmWaves = 4;
// Lanes per frequency of k_assemble: sixteen where 3H and 2H + 1 fit them.
__host__ __device__ inline constexpr int asm_group(int H) { return H <= 5 ? 16 : 32; }
// Doubles of the Cayley table in LDS (none above H = 10, whose f comes by Horner).
__host__ __device__ inline int cayley_doubles(int H) {
  const int K = 3 * H - 1;
  return 2 * K < 64 ? (2 * K + 1) * cayley_row(K) : 0;
}
__host__ __device__ inline int asm2_table_doubles(int H) {
  return cayley_doubles(H) + 2 * template_products(H) + 2 * H;
}
// nb > 0 (shared-phase bands): the Cayley table, then per band the 2H + 1
// template products, the template and the weight share; per frequency the
// bands' sums as well.
__host__ __device__ inline int asm2_band_doubles(int H, int nb) {
  return cayley_doubles(H) + 2 * nb * (3 * H + 2);
}
__host__ __device__ inline size_t asm2_lds_bytes(int H, int nb, int waves) {
  const int tab = nb ? asm2_band_doubles(H, nb) : asm2_table_doubles(H);
  return ((size_t)tab + (size_t)waves * (64 / asm_group(H)) * (asm2_doubles(H) + nb * 6 * H)) * sizeof(double);
}

// mu_e, e = 0..2H, of MM from the sums, on a group of nl
// lanes, lane per e.  The pairs (n, m) of e are run in one loop: n + m = e first,
// then n - m = e (m = |e - n|; conjugating Z_m turns the first form into the
// second), with the template's factors alpha_n alpha_m and 2 alpha_n conj(alpha_m)
// from the table `prod` in that order (row e - 1, H entries, zero where e has
// fewer pairs).  e = 0: s = sum_n |alpha_n|^2 (1 - |Z_n|^2), whose terms the
// lanes form and lane 0 adds in order (scr: H complex; pn: |alpha_n|^2).
__device__ __forceinline__ void assemble_mu(const FreqWork& W, int H, int lane, int nl, const double2* prod,
                                            const double* pn, double2* scr) {
#pragma clang fp contract(off)
  for (int n = lane; n < H; n += nl) {
    const double2 z = W.Z[n + 1];
    scr[n] = make_double2(pn[n], 1.0 - fma(z.x, z.x, z.y * z.y));
  }
  for (int e = lane + 1; e <= 2 * H; e += nl) {
    const double2 Ze = W.Z[e];
    const double2* P = prod + (e - 1) * H;
    const int n0 = e > H ? e - H : 1;
    double2 acc = make_double2(0.0, 0.0);
#pragma unroll 2
    for (int i = 0; i < H; ++i) {
      int n = n0 + i;
      n += n >= e ? 1 : 0;
      const int m = abs(e - n);
      const double2 a = W.Z[n], zm = W.Z[m], p = P[i];
      const double by = n > e ? -zm.y : zm.y;
      const double tx = Ze.x - fma(a.x, zm.x, -(a.y * by));
      const double ty = Ze.y - fma(a.y, zm.x, a.x * by);
      acc.x += fma(tx, p.x, ty * p.y);
      acc.y += fma(tx, p.y, -(ty * p.x));
    }
    W.mu[e] = acc;
  }
  __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
  __builtin_amdgcn_wave_barrier();
  if (lane == 0) {
    double t = 0.0;
#pragma unroll 4
    for (int n = 0; n < H; ++n) t = fma(scr[n].x, scr[n].y, t);
    W.mu[0] = make_double2(2.0 * t, 0.0);
  }
}

// Shared-phase bands (Appendix A): trig coefficients of MM and YM from the
// sums of every band.  With Z^b_n (weights normalised over all bands, Z^b_0 =
// W_b the band's share) and Zy^b_n:
//   B_n = sum_b alpha^b_n conj(Z^b_n)            (psi^n coefficient of Mbar),
//   eta_n = sum_b alpha^b_n conj(Zy^b_n),
//   mu_e = sum_b conj(Z^b_e) T^b_e - C_e,
// T^b_e = sum_{n+m=e} alpha^b_n alpha^b_m + 2 sum_{n-m=e} alpha^b_n conj(alpha^b_m)
// (T^b_0 = 2 sum_n |alpha^b_n|^2) the band's sum of M^2, and C_e the same
// products of B (Mbar^2).  One band reduces to assemble_mu.  W.Z[1..H]
// receive conj(B_n), which the scoring uses with unit alpha for Mbar.
struct BandTables { const double2 *Zb, *T, *alb, *wsb; };
__device__ __forceinline__ void band_tables(double2* alb, double2* wsb, double2* T, const SolveArgs& a, int tid, int nt) {
  const int H = a.H, nb = a.n_band;
  for (int q = tid; q < nb * H; q += nt) alb[q] = a.alpha[q];
  for (int b = tid; b < nb; b += nt) wsb[b] = make_double2(a.lcs[b].wsum, 0.0);
  __syncthreads();
  for (int q = tid; q < nb * (2 * H + 1); q += nt) {
    const int b = q / (2 * H + 1), e = q % (2 * H + 1);
    const double2* al = alb + b * H;
    double2 acc = make_double2(0.0, 0.0);
    if (e == 0) {
      for (int n = 0; n < H; ++n) acc.x += 2.0 * cabs2(al[n]);
    } else {
      const int nlo = e - H > 1 ? e - H : 1;
      const int nhi = e - 1 < H ? e - 1 : H;
      for (int n = nlo; n <= nhi; ++n) acc = cadd(acc, cmul(al[n - 1], al[e - n - 1]));
      for (int n = e + 1; n <= H; ++n) acc = cadd(acc, cscale(cmul(al[n - 1], cconj(al[n - e - 1])), 2.0));
    }
    T[q] = acc;
  }
}
__device__ __forceinline__ void assemble_shared(const BandTables& S, const FreqWork& W, int nb, int H, int lane, int nl) {
  for (int q = lane; q < 2 * H; q += nl) {
    const int n = (q % H) + 1;
    const bool isy = q >= H;
    double2 acc = make_double2(0.0, 0.0);
    for (int b = 0; b < nb; ++b) {
      const double2 z = S.Zb[b * 3 * H + (isy ? 2 * H + n - 1 : n - 1)];
      acc = cadd(acc, cmul(S.alb[b * H + n - 1], cconj(z)));
    }
    if (isy) W.eta[n] = acc;
    else W.Z[n] = cconj(acc);
  }
  if (lane == 0) W.eta[0] = make_double2(0.0, 0.0);
  wave_sync();
  for (int e = lane; e <= 2 * H; e += nl) {
    double2 acc = make_double2(0.0, 0.0);
    for (int b = 0; b < nb; ++b) {
      const double2 ze = e == 0 ? S.wsb[b] : S.Zb[b * 3 * H + e - 1];
      acc = cadd(acc, cmul(cconj(ze), S.T[b * (2 * H + 1) + e]));
    }
    double2 c = make_double2(0.0, 0.0);
    if (e == 0) {
      for (int n = 1; n <= H; ++n) c.x += 2.0 * cabs2(W.Z[n]);
    } else {
      const int nlo = e - H > 1 ? e - H : 1;
      const int nhi = e - 1 < H ? e - 1 : H;
      for (int n = nlo; n <= nhi; ++n) c = cadd(c, cmul(cconj(W.Z[n]), cconj(W.Z[e - n])));
      for (int n = e + 1; n <= H; ++n) c = cadd(c, cscale(cmul(cconj(W.Z[n]), W.Z[n - e]), 2.0));
    }
    W.mu[e] = csub(acc, c);
  }
  wave_sync();
}

// Maximum over a group of GL lanes (16 or 32), in every lane of it: of an int,
// and of a double.
template <int GL>
__device__ __forceinline__ int group_max_i(int h, int half) {
  h = max(h, dpp_i<0xB1, 0xf>(h));
  h = max(h, dpp_i<0x4E, 0xf>(h));
  h = max(h, dpp_i<0x141, 0xf>(h));
  h = max(h, dpp_i<0x140, 0xf>(h));
  if constexpr (GL == 16) return h;
  h = max(h, dpp_i<0x142, 0xa>(h));
  const int lo = __builtin_amdgcn_readlane(h, 31), hi = __builtin_amdgcn_readlane(h, 63);
  return half ? hi : lo;
}
template <int GL>
__device__ __forceinline__ double group_max_d(double v, int half) {
  if constexpr (GL == 16) {
    v = fmax(v, dpp_d<0xB1>(v));
    v = fmax(v, dpp_d<0x4E>(v));
    v = fmax(v, dpp_d<0x141>(v));
    return fmax(v, dpp_d<0x140>(v));
  } else {
    double lo, hi;
    half_max_d(v, lo, hi);
    return half ? hi : lo;
  }
}
__device__ __forceinline__ int abs2_hi(double2 z) {
  return (int)((unsigned long long)__double_as_longlong(cabs2(z)) >> 32) & 0x7fffffff;
}

// Above H = 10 the products of the Cayley table would not be exact; f(x) = sum_j
// rho_{j-K} u^j v^(D-j), u = 1 + i x, v = 1 - i x, comes by homogeneous Horner, h <-
// u h + rho_{K-l} v^l.  With the powers of i taken out (h_c = i^c g_c, v^l's
// coefficient c = i^c V_c) both recurrences are real shifts: g_c += g_{c-1},
// V_c -= V_{c-1}, then g_c += rho V_c.  Lane hl of 32 holds c = 3 hl..3 hl + 2 (D <
// 95, so the next group's first lane receives V = 0 by itself).  Against 64 lanes
// exchanging h and v through LDS for one frequency: the assembly of 50 thousand
// frequencies at H = 13 806 -> 203 us.
__device__ __forceinline__ void f_by_horner(const FreqWork& W, double2* rho, int K, int D, int hl, int k0, double tab_c,
                                            double tab_s, bool write, double* f) {
#pragma clang fp contract(off)
  for (int l0 = 0; l0 <= D; l0 += 32) {
    const int l = l0 + hl, d = K - l;
    const double ec = __shfl(tab_c, (d * k0) & 15), es = __shfl(tab_s, (d * k0) & 15);
    if (l <= D) {
      const double2 r = W.r[d < 0 ? -d : d], rd = make_double2(r.x, d < 0 ? -r.y : r.y);
      rho[l] = make_double2(fma(rd.x, ec, -(rd.y * es)), fma(rd.y, ec, rd.x * es));
    }
  }
  wave_sync();
  const double2 r0 = rho[0];
  double v0 = hl == 0 ? 1.0 : 0.0, v1 = 0.0, v2 = 0.0;
  double x0 = hl == 0 ? r0.x : 0.0, x1 = 0.0, x2 = 0.0, y0 = hl == 0 ? r0.y : 0.0, y1 = 0.0, y2 = 0.0;
#pragma unroll 2
  for (int l = 1; l <= D; ++l) {
    const double2 r = rho[l];
    const double xs = lane_shr1(x2), ys = lane_shr1(y2), vp = lane_shr1(v2);
    const double xp = hl == 0 ? 0.0 : xs, yp = hl == 0 ? 0.0 : ys;
    v2 = v2 - v1;
    v1 = v1 - v0;
    v0 = v0 - vp;
    x2 = (x2 + x1) + r.x * v2;
    x1 = (x1 + x0) + r.x * v1;
    x0 = (x0 + xp) + r.x * v0;
    y2 = (y2 + y1) + r.y * v2;
    y1 = (y1 + y0) + r.y * v1;
    y0 = (y0 + yp) + r.y * v0;
  }
  // f_c = Re(i^c g_c)
  const double gx[3] = {x0, x1, x2}, gy[3] = {y0, y1, y2};
#pragma unroll
  for (int s = 0; s < 3; ++s) {
    const int c = 3 * hl + s;
    const double v = (c & 1) ? gy[s] : gx[s];
    if (write && c <= D) f[c] = ((c + 1) & 2) ? -v : v;
  }
  wave_sync();
}

// Several frequencies per wavefront (sums from the grids, given, or of
// shared-phase bands), one per group of GL lanes with its own LDS working set: two of 32 lanes,
// or four of 16 where the template has at most five harmonics.  The assembly's
// per-frequency loops have 3H, 2H + 1, K + 1 or 16 lanes of work, which a group
// holds (the Cayley dot products, D + 1 columns, take two rounds), so one
// instruction stream serves all of them; maxima and the rotation argmax are
// reduced per group.  A pair with status "constant" or from a rejected lightcurve
// still runs the (cheap) rotation and dot products, whose results are not
// written.
//
// Bound by vector issue (60-65 % of the slots) and, up to H = 5, by writing the
// records (750 bytes each at H = 4), so the loops are laid out for few
// instructions: mu's pairs in one loop over the template's tabulated products,
// rows of the Cayley table contiguous per lane, the rotation's sixteen phases
// formed once, and for the grids H as a template parameter (loops and LDS
// offsets unroll; 10-14 % of the time).  Large H = 10 lightcurve (300 thousand
// frequencies) 575 -> 402 us; a batch round at H = 4 (4.2 million), sixteen lanes
// per frequency instead of 32 as well, 3.87 -> 1.65 ms; three bands at H = 6 (50
// thousand frequencies), one per wavefront before, 184 -> 84 us.
// HT: H, or 0 to take it from the arguments.  MODE: the sums' source.
enum { kFromGrids = 0, kFromSums = 1, kFromBands = 2 };
template <typename R, int GL, int HT, int MODE>
__global__ __launch_bounds__(64 * kAsmWaves) __attribute__((amdgpu_waves_per_eu(4))) void k_assemble(SolveArgs a, double* rec,
                                                                                          int64_t p0, int64_t np) {
  extern __shared__ double sma[];
  constexpr int NG = 64 / GL;
  const int lane = wave_lane(), half = lane >> 5, g = lane / GL, hl = lane & (GL - 1), wv = threadIdx.x >> 6;
  if (a.clear8 && blockIdx.x == 0 && threadIdx.x < 8) a.clear8[threadIdx.x] = 0u;
  const int H = HT ? HT : a.H, K = 3 * H - 1, D = 2 * K;
  const RecLayout RL(H);
  const int nwv = MODE == kFromBands ? blockDim.x >> 6 : kAsmWaves, nt = 64 * nwv;
  const int nb = MODE == kFromBands ? a.n_band : 0;
  // the Cayley table, the template's products and squares (or the bands'),
  // shared by the workgroup's waves
  const int LR = cayley_row(K), nct = cayley_doubles(H);
  const int ntab = MODE == kFromBands ? asm2_band_doubles(H, nb) : asm2_table_doubles(H);
  for (int i = threadIdx.x; i < (MODE == kFromBands ? nct : ntab); i += nt) sma[i] = a.ctab[i];
  const double* ctab = sma;
  const double2* prod = reinterpret_cast<const double2*>(sma + nct);
  const double* pn = sma + nct + 2 * template_products(H);
  double2* scr;
  double* const work = sma + ntab + (NG * wv + g) * (asm2_doubles(H) + nb * 6 * H);
  const FreqWork W = asm2_layout(work, H, scr);
  double2* const Zb = reinterpret_cast<double2*>(work + asm2_doubles(H));
  double2* const bt = reinterpret_cast<double2*>(sma + nct);
  const BandTables B{Zb, bt, bt + nb * (2 * H + 1), bt + nb * (3 * H + 1)};
  if (MODE == kFromBands) band_tables(bt + nb * (2 * H + 1), bt + nb * (3 * H + 1), bt, a, threadIdx.x, nt);
  __syncthreads();
  double tab_c, tab_s;
  sincos(kTwoPi * (lane & 15) / 16.0, &tab_s, &tab_c);
  // the rotation's candidate phases (lanes 0..15 of a group)
  double2 rot;
  sincos_small(kTwoPi * hl / 16.0 + kPi, rot.y, rot.x);
  const double2 alk = hl < H ? a.alpha[hl] : make_double2(0.0, 0.0);
  // MM, YM of order one: the squared threshold of the constant test below
  const double ctol = 64.0 * kEps * (6.0 * H) * (2.0 * H + 1.0), ctol2 = ctol * ctol;
  const typename Cplx<R>::T* grids = reinterpret_cast<const typename Cplx<R>::T*>(a.grids);
  const int64_t gw = (int64_t)blockIdx.x * nwv + wv, nw = (int64_t)gridDim.x * nwv;
  for (int64_t w0 = NG * gw; w0 < np; w0 += NG * nw) {
    const bool has = w0 + g < np;                    // an empty group repeats the first
    const int64_t w = has ? w0 + g : w0;
    const int64_t pidx = p0 + w;
    double* Rr = rec + w * (int64_t)RL.stride;
    const int64_t lc = pair_lc(a, pidx);
    const LcInfo& L = a.lcs[lc];
    const int64_t j = pidx - a.freq_off[lc] + 1;
    const bool bad = L.status != 0;
    if constexpr (MODE == kFromBands) {
      // every band's sums of this frequency (grids of lightcurves 0..nb-1)
      for (int q = hl; q < nb * 3 * H; q += GL) {
        const int b = q / (3 * H), qq = q % (3 * H);
        const int gr = qq < 2 * H ? 0 : 1;
        const int k = gr == 0 ? qq + 1 : qq - 2 * H + 1;
        Zb[q] = bad ? make_double2(0.0, 0.0) : gather_mode<R>(a.lcs[b], gr, (int64_t)k * j, grids);
      }
      wave_sync();
      assemble_shared(B, W, nb, H, hl, GL);
    } else {
      if (hl == 0) W.Z[0] = make_double2(1.0, 0.0);
      for (int q = hl; q < 3 * H; q += GL) {
        double2 z = make_double2(0.0, 0.0);
        if (!bad) {
          if constexpr (MODE == kFromSums) {
            z = reinterpret_cast<const double2*>(a.sums_in)[pidx * 3 * H + q];
            if (q >= 2 * H) z = cscale(z, L.inv_sqrt_yy);
          } else {
            const int gr = q < 2 * H ? 0 : 1;
            const int k = gr == 0 ? q + 1 : q - 2 * H + 1;
            z = gather_mode<R>(L, gr, (int64_t)k * j, grids);
          }
        }
        W.Z[q + 1] = z;
      }
      wave_sync();
      assemble_mu(W, H, hl, GL, prod, pn, scr);
      if (hl < H) {
#pragma clang fp contract(off)
        const double2 z = W.Z[2 * H + 1 + hl];   // eta_k = alpha_k conj(Zy_k)
        W.eta[hl + 1] = make_double2(fma(alk.x, z.x, alk.y * z.y), fma(alk.y, z.x, -(alk.x * z.y)));
      }
    }
    if (hl == 0) W.eta[0] = make_double2(0.0, 0.0);
    wave_sync();
    assemble_r(W, H, hl, scr, GL);
    const double ref = ref_cycles(j, L.df, L.tref);
    // R = 0 against rounding noise: largest squared magnitudes by their high
    // words (within 2^-20)
    int rmax = 0, mumax = 0, etamax = 0;
    for (int d = hl; d <= K; d += GL) rmax = max(rmax, abs2_hi(W.r[d]));
    for (int e = hl; e <= 2 * H; e += GL) mumax = max(mumax, abs2_hi(W.mu[e]));
    if (hl <= H) etamax = abs2_hi(W.eta[hl]);
    rmax = group_max_i<GL>(rmax, half);
    mumax = group_max_i<GL>(mumax, half);
    etamax = group_max_i<GL>(etamax, half);
    auto from_hi = [](int h) { return __longlong_as_double((long long)((unsigned long long)(unsigned)h << 32)); };
    const bool constant = !(from_hi(rmax) > ctol2 * (from_hi(mumax) * from_hi(etamax)));
    // rotation phi0: the 16 candidates of each group on its lanes 0..15
    double Rv = -1.0;
    if (GL == 16 || hl < 16) {
      double2 q = W.r[K];
#pragma unroll 4
      for (int d = K - 1; d >= 1; --d) q = cfma(q, rot, W.r[d]);
      Rv = fabs(fma(2.0, fma(rot.x, q.x, -(rot.y * q.y)), W.r[0].x));
    }
    const double rm = group_max_d<GL>(Rv, half);
    const unsigned long long mask = __ballot((GL == 16 || hl < 16) && Rv == rm);
    const unsigned hm = (unsigned)(mask >> (lane & ~(GL - 1))) & 0xffffu;
    const int k0 = hm ? __ffs(hm) - 1 : 0;
    const double phi0 = constant ? 0.0 : kTwoPi * k0 / 16.0;
    const bool write = has && !bad;
    if (HT == 0 && D >= 64) {
      f_by_horner(W, scr, K, D, hl, k0, tab_c, tab_s, write && !constant, Rr + RL.f);
    } else {
      // 2 rho_j = 2 r_{j-K} e^{i (j-K) phi0}, j = 0..K - 1, and rho_K (every lane
      // takes part in the table reads), then the dot products over j <= K (the
      // terms j and D - j are equal)
      double* rx = reinterpret_cast<double*>(scr);
      double* ry = rx + LR;
      for (int jx = hl; jx < ((K + GL) & ~(GL - 1)); jx += GL) {
#pragma clang fp contract(off)
        const int d = jx - K;
        const int m = (d * k0) & 15;
        const double ec = __shfl(tab_c, m), es = __shfl(tab_s, m);
        if (jx <= K) {
          const double2 rd = W.r[-d];
          const double wgt = jx < K ? 2.0 : 1.0;
          rx[jx] = wgt * fma(rd.x, ec, rd.y * es);
          ry[jx] = wgt * fma(rd.x, es, -(rd.y * ec));
        }
      }
      wave_sync();
      for (int c = hl; c <= D; c += GL) {
        const double fc = cayley_dot((c & 1) ? ry : rx, ctab + c * LR, K);
        if (write && !constant) Rr[RL.f + c] = fc;
      }
    }
    if (write) {
      double2* r2 = reinterpret_cast<double2*>(Rr);
      for (int d = hl; d <= K; d += GL) r2[RL.r / 2 + d] = W.r[d];
      for (int e = hl; e <= 2 * H; e += GL) r2[RL.mu / 2 + e] = W.mu[e];
      if (hl < H) {
        r2[RL.eta / 2 + hl] = W.eta[hl + 1];
        r2[RL.zw / 2 + hl] = W.Z[hl + 1];
      }
      if (hl == 0) {
        Rr[RL.meta + M_PHI0] = phi0;
        Rr[RL.meta + M_REF] = ref;
        Rr[RL.meta + M_STATUS] = constant ? (double)ST_CONSTANT : (double)ST_OK;
        Rr[RL.meta + M_LC] = (double)lc;
        Rr[RL.meta + M_FALLBACK] = 0.0;
        Rr[RL.meta + M_WARM] = 0.0;
      }
    } else if (has && hl == 0) {
      Rr[RL.meta + M_STATUS] = (double)ST_BAD_LC;
      Rr[RL.meta + M_LC] = (double)lc;
      Rr[RL.meta + M_FALLBACK] = 0.0;
      Rr[RL.meta + M_WARM] = 0.0;
    }
    wave_sync();
  }
}

// ---------------------------------------------------------------- score

// Best-candidate selection across the wave: max P; near ties (1e-12 relative)
// prefer theta_1 > 0, then the smallest absolute theta_2.
struct Best { double P, th_rel, th_abs, amp_sign; int lane; };

__device__ __forceinline__ Best select_best(double P, double th_rel, double th_abs, double ym, bool valid,
                                            int lane) {
  const double pv = valid ? P : -1.0;
  const double pmax = wave_max(pv);
  const bool near = valid && pv >= pmax - 1e-12 * fmax(pmax, 1e-300);
  double key = near ? ((ym > 0.0 ? 0.0 : 8.0) + th_abs) : 1e30;
  const double kmin = -wave_max(-key);
  const unsigned long long mask = __ballot(near && key == kmin);
  Best b;
  b.lane = mask ? __ffsll((long long)mask) - 1 : 0;
  b.P = __shfl(pv, b.lane);
  b.th_rel = __shfl(th_rel, b.lane);
  b.th_abs = __shfl(th_abs, b.lane);
  b.amp_sign = __shfl(ym, b.lane);
  return b;
}

// select_best over two candidates per lane (candidate c = lane + 64 slot,
// degree D > 64); `slot` receives the winner's slot, Best.lane its lane.
__device__ __forceinline__ Best select_best2(const double (&P)[2], const double (&th_rel)[2],
                                             const double (&th_abs)[2], const double (&ym)[2],
                                             const bool (&valid)[2], int& slot) {
  const double p0 = valid[0] ? P[0] : -1.0, p1 = valid[1] ? P[1] : -1.0;
  const double pmax = wave_max(fmax(p0, p1));
  const double lo = pmax - 1e-12 * fmax(pmax, 1e-300);
  const bool n0 = valid[0] && p0 >= lo, n1 = valid[1] && p1 >= lo;
  const double k0 = n0 ? ((ym[0] > 0.0 ? 0.0 : 8.0) + th_abs[0]) : 1e30;
  const double k1 = n1 ? ((ym[1] > 0.0 ? 0.0 : 8.0) + th_abs[1]) : 1e30;
  const double kmin = -wave_max(-fmin(k0, k1));
  const unsigned long long m0 = __ballot(n0 && k0 == kmin), m1 = __ballot(n1 && k1 == kmin);
  slot = m0 ? 0 : (m1 ? 1 : 0);
  const unsigned long long mask = m0 ? m0 : m1;
  Best b;
  b.lane = mask ? __ffsll((long long)mask) - 1 : 0;
  b.P = slot ? __shfl(p1, b.lane) : __shfl(p0, b.lane);
  b.th_rel = slot ? __shfl(th_rel[1], b.lane) : __shfl(th_rel[0], b.lane);
  b.th_abs = slot ? __shfl(th_abs[1], b.lane) : __shfl(th_abs[0], b.lane);
  b.amp_sign = slot ? __shfl(ym[1], b.lane) : __shfl(ym[0], b.lane);
  return b;
}

__device__ __forceinline__ double wrap_2pi(double x) {
  // a phase plus a rotation, both in [0, 2 pi): the difference is exact
  if (x >= 0.0 && x < 2.0 * kTwoPi) return x >= kTwoPi ? x - kTwoPi : x;
  x = fmod(x, kTwoPi);
  if (x < 0.0) x += kTwoPi;
  if (x >= kTwoPi) x -= kTwoPi;
  return x;
}

// Degeneracy threshold: MM <= tau sum |alpha|^2 at every candidate, with tau
// set by the precision of the sums (exact sums 1e-14, FP64 NFFT 1e-9, FP32
// NFFT 1e-5: a few hundred times the sums' error relative to sum|g|).
__device__ __forceinline__ double mm_floor(const FreqWork& W, int H, double tau) {
  double s = 0.0;
  for (int n = 0; n < H; ++n) s += cabs2(W.al[n]);
  return tau * s;
}

__host__ __device__ inline size_t score_lds_bytes(int H) {
  const int K = 3 * H - 1;
  return (size_t)(2 * ((3 * H + 1) + (2 * H + 1) + (H + 1) + (K + 1) + H)) * sizeof(double);
}

// Scores all candidates of pairs [p0, p0 + np) and writes the outputs.  At
// least four waves per SIMD (at most 128 VGPRs, no spills; measured faster
// than five waves with spills, or than the uncapped allocation).
// `list` (device, *list_n entries): score only those pairs of the chunk.
// NSL: candidates per lane (2 for degree D > 64).
template <int NSL>
__global__ __launch_bounds__(64) __attribute__((amdgpu_waves_per_eu(4))) void k_score(SolveArgs a, const double* rec, int64_t p0, int64_t np,
                                                                                      const int64_t* list,
                                                                                      const unsigned* list_n) {
  // On a list this is the last of the fallback tiers, whose waves take issue priority
  // over the side stream's scoring on a shared SIMD (the tiers are few, latency-bound
  // waves on the step's critical path).  Above H = 10 it is that scoring as well, at
  // the tiers' own priority: 2.68 ms for a periodogram at H = 13 (50 thousand
  // frequencies) against 2.71 with the priority on lists only.
  __builtin_amdgcn_s_setprio(2);
  extern __shared__ double sms[];
  const int lane = wave_lane();
  const int H = a.H, K = 3 * H - 1, D = 2 * K;
  const RecLayout RL(H);
  FreqWork W;
  {
    double2* q = reinterpret_cast<double2*>(sms);
    W.Z = q; q += 3 * H + 1;
    W.mu = q; q += 2 * H + 1;
    W.eta = q; q += H + 1;
    W.r = q; q += K + 1;
    W.al = q;
  }
  // shared phase: the record holds conj(B_n) in place of Z_n, so unit alpha
  // gives Mbar; the degeneracy scale comes from the bands' templates
  for (int q = lane; q < H; q += 64) W.al[q] = a.n_band ? make_double2(1.0, 0.0) : a.alpha[q];
  wave_sync();
  const double floor_mm = a.n_band ? a.mm_tau * a.lcs[0].mm_scale : mm_floor(W, H, a.mm_tau);
  // the record fields each lane needs (lane d <= K: r_d; e <= 2H: mu_e;
  // k < H: eta, Z_w; candidates c = lane + 64 s < D) are loaded one pair
  // ahead, so their latency overlaps the scoring of the current pair
  struct Fields { double2 r, mu, eta, zw; double cand[NSL]; };
  const int64_t n = list ? (int64_t)*list_n : np;
  auto item = [&](int64_t i) { return list ? list[i] : i; };
  auto fetch = [&](int64_t i) {
    Fields f;
    f.r = f.mu = f.eta = f.zw = make_double2(0.0, 0.0);
#pragma unroll
    for (int sl = 0; sl < NSL; ++sl) f.cand[sl] = 0.0;
    if (i < n) {
      const double* R = rec + item(i) * (int64_t)RL.stride;
      if (lane <= K) f.r = make_double2(R[RL.r + 2 * lane], R[RL.r + 2 * lane + 1]);
      if (lane <= 2 * H) f.mu = make_double2(R[RL.mu + 2 * lane], R[RL.mu + 2 * lane + 1]);
      if (lane < H) {
        f.eta = make_double2(R[RL.eta + 2 * lane], R[RL.eta + 2 * lane + 1]);
        f.zw = make_double2(R[RL.zw + 2 * lane], R[RL.zw + 2 * lane + 1]);
      }
#pragma unroll
      for (int sl = 0; sl < NSL; ++sl)
        if (lane + 64 * sl < D) f.cand[sl] = R[RL.cand + 64 * sl + lane];
    }
    return f;
  };
  Fields nxt = fetch(blockIdx.x);
  for (int64_t i = blockIdx.x; i < n; i += gridDim.x) {
    const Fields cur = nxt;
    nxt = fetch(i + gridDim.x);
    const int64_t w = item(i);
    const int64_t pidx = p0 + w;
    const double* Rr = rec + w * (int64_t)RL.stride;
    const int st = (int)Rr[RL.meta + M_STATUS];
    if (a.newton_cands == 2 && Rr[RL.meta + M_FALLBACK] != 0.0) continue;   // the fallback list's scoring takes it
    const int64_t lc = (int64_t)Rr[RL.meta + M_LC];
    const LcInfo& L = a.lcs[lc];
    if (st == ST_BAD_LC) {
      if (lane == 0) {
        a.power[pidx] = 0.0; a.phase[pidx] = 0.0; a.amp[pidx] = 0.0; a.offset[pidx] = 0.0;
        if (a.status) a.status[pidx] = ST_BAD_LC;
      }
      continue;
    }
    const double ref = Rr[RL.meta + M_REF];
    if (lane <= K) W.r[lane] = cur.r;
    if (lane <= 2 * H) W.mu[lane] = cur.mu;
    if (lane < H) {
      W.eta[lane + 1] = cur.eta;
      // the conjugated psi^k coefficient of Mbar, conj(alpha_k conj(Z_k))
      W.Z[lane + 1] = cconj(cmul(W.al[lane], cconj(cur.zw)));
    }
    if (lane == 0) W.eta[0] = make_double2(0.0, 0.0);
    wave_sync();
    double th[NSL];
    bool valid[NSL];
    Cand c[NSL];
#pragma unroll
    for (int sl = 0; sl < NSL; ++sl) {
      th[sl] = 0.0;
      valid[sl] = false;
      if (st == ST_CONSTANT) {
        // P does not depend on the phase: score theta_2 = 0 (absolute)
        th[sl] = -kTwoPi * ref;
        valid[sl] = lane == 0 && sl == 0;
      } else if (lane + 64 * sl < D) {
        th[sl] = cur.cand[sl];
        valid[sl] = !isnan(th[sl]);
        if (!valid[sl]) th[sl] = 0.0;
      }
      c[sl] = eval_candidate(W, H, th[sl]);
    }
    double mml = valid[0] ? c[0].MM : -1.0;
    if (NSL > 1) mml = fmax(mml, valid[NSL - 1] ? c[NSL - 1].MM : -1.0);
    const double mmmax = wave_max(mml);
    int stout = st;
    if (mmmax <= floor_mm) stout = ST_DEGENERATE;
    // positive-amplitude variant: only candidates with theta_1 = YM/MM > 0
    const bool pos = (a.flags & kFlagPositiveAmp) != 0u;
    bool ok[NSL];
    bool any_ok = false;
#pragma unroll
    for (int sl = 0; sl < NSL; ++sl) {
      ok[sl] = valid[sl] && (c[sl].MM > floor_mm || stout == ST_DEGENERATE) && (!pos || c[sl].YM > 0.0);
      any_ok = any_ok || ok[sl];
    }
    const bool none = pos && stout != ST_DEGENERATE && __ballot(any_ok) == 0ull;
    Best b;
    int bslot = 0;
    if constexpr (NSL == 1) {
      b = select_best(c[0].P, th[0], wrap_2pi(th[0] + kTwoPi * ref), c[0].YM, ok[0], lane);
    } else {
      const double P2[2] = {c[0].P, c[NSL - 1].P}, ym2[2] = {c[0].YM, c[NSL - 1].YM};
      const double th2[2] = {th[0], th[NSL - 1]};
      const double ta2[2] = {wrap_2pi(th[0] + kTwoPi * ref), wrap_2pi(th[NSL - 1] + kTwoPi * ref)};
      const bool ok2[2] = {ok[0], ok[NSL - 1]};
      b = select_best2(P2, th2, ta2, ym2, ok2, bslot);
    }
    // Newton polish of the winner on R(theta) (Eq. theta2cond): a step is
    // kept only if it is small and P does not drop; a step below 1e-13 rad
    // changes P by O(1e-26) and ends the polish without re-scoring
    double best_th = b.th_rel;
    const Cand& cw = c[0];
    Cand cb = {__shfl(cw.P, b.lane), __shfl(cw.YM, b.lane), __shfl(cw.MM, b.lane), __shfl(cw.Mbar, b.lane)};
    if (NSL > 1 && bslot) {
      const Cand& cx = c[NSL - 1];
      cb = Cand{__shfl(cx.P, b.lane), __shfl(cx.YM, b.lane), __shfl(cx.MM, b.lane), __shfl(cx.Mbar, b.lane)};
    }
    // roots that Newton already converged (steps below 1e-12 rad, learned and
    // uniform solvers) are not polished: the polish step would be rounding noise
    const bool newton_root = a.newton_cands && Rr[RL.meta + M_FALLBACK] == 0.0;
    if (stout != ST_DEGENERATE && stout != ST_CONSTANT && !none && !newton_root) {
      for (int it = 0; it < 3; ++it) {
        double Rv, dR;
        eval_R(W, H, best_th, Rv, dR);
        if (!(dR != 0.0) || !isfinite(Rv / dR)) break;
        const double step = Rv / dR;
        if (fabs(step) > 1e-3 || fabs(step) < 1e-13) break;
        const double nt = best_th - step;
        const Cand nc = eval_candidate(W, H, nt);
        if (!(nc.P >= cb.P)) break;
        best_th = nt;
        cb = nc;
      }
    }
    if (lane == 0) {
      const double sq = sqrt(L.yy);
      double P = cb.P, amp = cb.MM > 0.0 ? cb.YM / cb.MM * sq : 0.0;
      double off = L.ybar - cb.Mbar * amp;
      double th_abs = wrap_2pi(best_th + kTwoPi * ref);
      if (stout == ST_DEGENERATE || none) { P = 0.0; amp = 0.0; off = L.ybar; th_abs = 0.0; }
      a.power[pidx] = P;
      a.phase[pidx] = th_abs;
      a.amp[pidx] = amp;
      a.offset[pidx] = off;
      const double fb = Rr[RL.meta + M_FALLBACK];
      const int fbits = fb >= 2.0 ? (ST_FALLBACK | ST_FALLBACK_QR) : (fb != 0.0 ? ST_FALLBACK : 0);
      if (a.status) a.status[pidx] = (uint8_t)(stout | fbits);
    }
    wave_sync();
  }
}

// Maximum of a double over each 16-lane row, in every lane of the row.
__device__ __forceinline__ double row_max_d(double v) {
  v = fmax(v, dpp_d<0xB1>(v));    // quad_perm [1, 0, 3, 2]
  v = fmax(v, dpp_d<0x4E>(v));    // quad_perm [2, 3, 0, 1]
  v = fmax(v, dpp_d<0x141>(v));   // row_half_mirror
  v = fmax(v, dpp_d<0x140>(v));   // row_mirror
  return v;
}

// e^{i (theta - phi0)} of a root's key (see newton_pair): key = u = tan((theta -
// phi0) / 2) for |key| <= 1, else sign(u) 2 - u with u its reciprocal.
__device__ __forceinline__ double2 dir_from_key(double key) {
  const bool in = fabs(key) <= 1.0;
  const double u = in ? key : copysign(2.0, key) - key;
  const double i = fast_rcp_d(fma(u, u, 1.0)), c = fma(-u, u, 1.0) * i;
  return make_double2(in ? c : -c, 2.0 * u * i);
}
__device__ __forceinline__ double theta_from_key(double phi0, double key) {
  const bool in = fabs(key) <= 1.0;
  return theta_from_u(phi0, in ? key : copysign(2.0, key) - key, in ? 1 : -1);
}

// Scoring of the first round's Newton-root pairs (M_FALLBACK = 0), four
// frequencies per wavefront, one per 16-lane row: the roots (at most 32 per
// frequency, its starts) are scored 16 at a time, and the candidates 16..31
// of a row take a second evaluation only when some row of the wavefront has
// more than 16 roots (a frequency has ~12 real roots at H = 10).  The
// candidates, tie rule and outputs of k_score, without the polish (the roots
// are Newton-converged).  The roots come as keys: e^{i theta} of a candidate is
// rational in its key, and only winners need their phase (near ties, which
// the smallest phase decides, form all of them).
//
// A wavefront takes `per` consecutive frequencies (4..64, a multiple of 4).
// Their winners wait in LDS and are finished together, a lane each: phase,
// amplitude and the stores, which are contiguous.  The record fields a row's
// lanes read (meta; mu_e, e = l, l + 16; eta_k and Z_w k, k = l + 1;
// candidates l, l + 16) are loaded one iteration ahead.
//
// Bound by vector issue and LDS latency: H is a template parameter so that
// the Horner chains unroll with their loads ahead of them.  Against one kernel
// for all H that formed every candidate's phase by a sine and cosine and finished
// each frequency by itself, with spills: large H = 10 (300 thousand frequencies)
// 168 -> 98 us alone, batch round at H = 4 (4.2 million) 1.25 -> 0.71 ms.  Three
// wavefronts per SIMD from H = 8 (their chains' loads would spill at four).
struct Score4Fetch {
  double st, fb, lc, ref, phi0, c0, c1;
  double mu0[2], mu1[2], eta[2], zw[2];
};

template <int H>
__device__ __forceinline__ void score4_fetch(const double* rec, int64_t np, int64_t w0, int row, int l, Score4Fetch& F) {
  constexpr int D = 6 * H - 2, NC = D < 32 ? D : 32;   // NC: the first round's starts per frequency
  const RecLayout RL(H);
  const bool has = w0 + row < np;
  const double* Rr = rec + (has ? w0 + row : w0) * (int64_t)RL.stride;
  const double qnan = __longlong_as_double(0x7ff8000000000000ll);
  F.st = Rr[RL.meta + M_STATUS];
  F.fb = has ? Rr[RL.meta + M_FALLBACK] : 1.0;   // past the end: scored, never written
  F.lc = Rr[RL.meta + M_LC];
  F.ref = Rr[RL.meta + M_REF];
  F.phi0 = Rr[RL.meta + M_PHI0];
  const double2* mu = reinterpret_cast<const double2*>(Rr + RL.mu);
  const int lh = l < H ? l : H - 1;
  auto get = [](double (&d)[2], const double2* p) {
    const double2 v = *p;
    d[0] = v.x;
    d[1] = v.y;
  };
  get(F.mu0, mu + (l < 2 * H ? l : 2 * H));
  if constexpr (2 * H >= 16) get(F.mu1, mu + (l + 16 < 2 * H ? l + 16 : 2 * H));
  get(F.eta, reinterpret_cast<const double2*>(Rr + RL.eta) + lh);
  get(F.zw, reinterpret_cast<const double2*>(Rr + RL.zw) + lh);
  F.c0 = Rr[RL.cand + (l < NC ? l : NC - 1)];
  F.c1 = qnan;
  if (l >= NC) F.c0 = qnan;
  if (NC > 16) {
    F.c1 = Rr[RL.cand + (l + 16 < NC ? l + 16 : NC - 1)];
    if (l + 16 >= NC) F.c1 = qnan;
  }
}

constexpr int kScorePer = 64;   // frequencies a wavefront takes at most
// LDS of k_score4: per row MM's, YM's and Mbar's coefficients (4H + 1 complex: an
// odd count, so that the rows' broadcasts meet distinct banks), then the winners.
__host__ __device__ inline size_t score4_lds_bytes(int H) {
  return (size_t)(4 * 2 * (4 * H + 1) + 7 * kScorePer) * sizeof(double) + kScorePer * sizeof(int);
}

template <int H>
__global__ __launch_bounds__(64) __attribute__((amdgpu_waves_per_eu(H >= 8 ? 3 : 4))) void k_score4(SolveArgs a, const double* rec,
                                                                                       int64_t p0, int64_t np, int per) {
  extern __shared__ double sms[];
  const int lane = wave_lane(), row = lane >> 4, l = lane & 15;
  double2* mu = reinterpret_cast<double2*>(sms) + row * (4 * H + 1);
  double2* eta = mu + 2 * H;    // eta[k], k = 1..H
  double2* zb = eta + H;        // zb[k] = alpha_k conj(Z_k), k = 1..H
  double* fin = sms + 4 * 2 * (4 * H + 1);
  int* fcode = reinterpret_cast<int*>(fin + 7 * kScorePer);
  const double2 alk = l < H && !a.n_band ? a.alpha[l] : make_double2(1.0, 0.0);
  double floor_mm;
  {
    double s = 0.0;
    if (!a.n_band)
      for (int n = 0; n < H; ++n) s += cabs2(a.alpha[n]);
    floor_mm = a.n_band ? a.mm_tau * a.lcs[0].mm_scale : a.mm_tau * s;
  }
  const bool pos = (a.flags & kFlagPositiveAmp) != 0u;
  double tab_c, tab_s;
  sincos(kTwoPi * l / 16.0, &tab_s, &tab_c);
  const int64_t wb = (int64_t)blockIdx.x * per, we = wb + per < np ? wb + per : np;
  Score4Fetch F;
  score4_fetch<H>(rec, we, wb, row, l, F);
  for (int64_t w0 = wb; w0 < we; w0 += 4) {
    // this iteration's fields into LDS and registers, then the next
    // iteration's loads
    const int st = (int)F.st;
    const bool mine = F.fb == 0.0;
    const double lc = F.lc, ref = F.ref, phi0 = F.phi0;
    if (l <= 2 * H) mu[l] = make_double2(F.mu0[0], F.mu0[1]);
    if constexpr (2 * H >= 16) {
      if (l + 16 <= 2 * H) mu[l + 16] = make_double2(F.mu1[0], F.mu1[1]);
    }
    if (l < H) {
      eta[l + 1] = make_double2(F.eta[0], F.eta[1]);
      zb[l + 1] = cmul(alk, make_double2(F.zw[0], -F.zw[1]));
    }
    const double k0v = F.c0, k1v = F.c1;
    const bool roots = st != ST_CONSTANT && st != ST_BAD_LC;
    const bool valid0 = roots ? !isnan(k0v) : st == ST_CONSTANT && l == 0, valid1 = roots && !isnan(k1v);
    if (w0 + 4 < we) score4_fetch<H>(rec, we, w0 + 4, row, l, F);
    wave_sync();
    // (the evaluation reads mu, eta and Z: the Newton roots take no polish on R)
    const bool second = __ballot(valid1) != 0ull;   // wave-uniform
    const int kr = (int)rint(phi0 * (16.0 / kTwoPi)) & 15;
    const double rc = __shfl(tab_c, kr), rs = __shfl(tab_s, kr);
    // P does not depend on the phase: theta_2 = 0 (absolute) is scored
    const double th_const = -kTwoPi * ref;
    const bool any_const = __ballot(st == ST_CONSTANT) != 0ull;
    Cand c0 = Cand{0.0, 0.0, 0.0, 0.0}, c1 = c0;
#pragma unroll 1
    for (int sl = second ? 1 : 0; sl >= 0; --sl) {
      const bool v = (sl ? valid1 : valid0) && roots;
      const double2 d = dir_from_key(v ? (sl ? k1v : k0v) : 0.0);
      double2 psi = make_double2(fma(d.x, rc, -(d.y * rs)), fma(d.x, rs, d.y * rc));
      if (any_const && st == ST_CONSTANT) sincos_small(th_const, psi.y, psi.x);
      c1 = c0;
      double2 m = mu[2 * H];
#pragma unroll
      for (int k = 2 * H - 1; k >= 1; --k) m = cfma(m, psi, mu[k]);
      double2 y = eta[H], b = zb[H];
#pragma unroll
      for (int k = H - 1; k >= 1; --k) {
        y = cfma(y, psi, eta[k]);
        b = cfma(b, psi, zb[k]);
      }
      // the sums above stop at psi^1: one more factor psi
      c0.MM = fma(2.0, m.x * psi.x - m.y * psi.y, mu[0].x);
      c0.YM = 2.0 * (y.x * psi.x - y.y * psi.y);
      c0.Mbar = 2.0 * (b.x * psi.x - b.y * psi.y);
      c0.P = c0.MM > 0.0 ? c0.YM * c0.YM / c0.MM : 0.0;
    }
    auto row_bits = [&](bool x) { return (unsigned)(__ballot(x) >> (16 * row)) & 0xffffu; };
    const bool above0 = valid0 && c0.MM > floor_mm, above1 = valid1 && c1.MM > floor_mm;
    int stout = st;
    if (st != ST_BAD_LC && row_bits(above0 || above1) == 0u) stout = ST_DEGENERATE;
    const bool degen = stout == ST_DEGENERATE;
    const bool ok0 = valid0 && (above0 || degen) && (!pos || c0.YM > 0.0);
    const bool ok1 = valid1 && (above1 || degen) && (!pos || c1.YM > 0.0);
    const bool none = pos && !degen && row_bits(ok0 || ok1) == 0u;
    // the winner of each row, as select_best over its candidates in index order
    const double v0 = ok0 ? c0.P : -1.0, v1 = ok1 ? c1.P : -1.0;
    const double pmax = row_max_d(fmax(v0, v1));
    const double lo = pmax - 1e-12 * fmax(pmax, 1e-300);
    unsigned m0 = row_bits(ok0 && v0 >= lo), m1 = row_bits(ok1 && v1 >= lo);
    if (__ballot(__popc(m0) + __popc(m1) > 1)) {
      double kmin = 1e30, kk0 = 1e30, kk1 = 1e30;
#pragma unroll 1
      for (int sl = 0; sl < 2; ++sl) {
        const double t = roots ? theta_from_key(phi0, sl ? (valid1 ? k1v : 0.0) : (valid0 ? k0v : 0.0)) : th_const;
        const double kv = ((sl ? c1.YM : c0.YM) > 0.0 ? 0.0 : 8.0) + wrap_2pi(t + kTwoPi * ref);
        if (sl) kk1 = ((m1 >> l) & 1u) ? kv : 1e30;
        else kk0 = ((m0 >> l) & 1u) ? kv : 1e30;
      }
      kmin = -row_max_d(-fmin(kk0, kk1));
      m0 = row_bits(((m0 >> l) & 1u) && kk0 == kmin);
      m1 = row_bits(((m1 >> l) & 1u) && kk1 == kmin);
    }
    const unsigned mb = m0 ? m0 : m1;
    const int bl = mb ? __ffs(mb) - 1 : 0;
    if (l == bl) {
      const bool s1 = m0 == 0u && m1 != 0u;
      const int i = (int)(w0 - wb) + row;
      fin[i] = s1 ? c1.P : c0.P;
      fin[kScorePer + i] = s1 ? c1.YM : c0.YM;
      fin[2 * kScorePer + i] = s1 ? c1.MM : c0.MM;
      fin[3 * kScorePer + i] = s1 ? c1.Mbar : c0.Mbar;
      fin[4 * kScorePer + i] = s1 ? k1v : k0v;
      fin[5 * kScorePer + i] = ref;
      fin[6 * kScorePer + i] = lc;
      fcode[i] = stout | (none ? 256 : 0) | (mine ? 512 : 0) | (roots ? 1024 : 0) | (kr << 12);
    }
    wave_sync();
  }
  if (lane < (int)(we - wb)) {
    const int code = fcode[lane], stout = code & 255;
    if (!(code & 512)) return;
    const int64_t pidx = p0 + wb + lane;
    if (stout == ST_BAD_LC) {
      a.power[pidx] = 0.0; a.phase[pidx] = 0.0; a.amp[pidx] = 0.0; a.offset[pidx] = 0.0;
    } else {
      const LcInfo& L = a.lcs[(int64_t)fin[6 * kScorePer + lane]];
      const double YM = fin[kScorePer + lane], MM = fin[2 * kScorePer + lane], ref = fin[5 * kScorePer + lane];
      const double th = (code & 1024) ? theta_from_key(kTwoPi * (code >> 12) / 16.0, fin[4 * kScorePer + lane]) : -kTwoPi * ref;
      double P = fin[lane], amp = MM > 0.0 ? YM / MM * sqrt(L.yy) : 0.0;
      double off = L.ybar - fin[3 * kScorePer + lane] * amp;
      double th_abs = wrap_2pi(th + kTwoPi * ref);
      if (stout == ST_DEGENERATE || (code & 256)) { P = 0.0; amp = 0.0; off = L.ybar; th_abs = 0.0; }
      a.power[pidx] = P;
      a.phase[pidx] = th_abs;
      a.amp[pidx] = amp;
      a.offset[pidx] = off;
    }
    if (a.status) a.status[pidx] = (uint8_t)stout;
  }
}

// Writes the deconvolved sums of every pair (3H complex per pair: Z_w(k j),
// k = 1..2H, then Z_y(k j), k = 1..H with the 1/sqrt(YY) normalisation undone).
template <typename R>
__global__ __launch_bounds__(64) void k_gather_sums(SolveArgs a, double* out) {
  const int lane = wave_lane();
  const int H = a.H;
  const typename Cplx<R>::T* grids = reinterpret_cast<const typename Cplx<R>::T*>(a.grids);
  for (int64_t pidx = blockIdx.x; pidx < a.total; pidx += gridDim.x) {
    const int64_t lc = pair_lc(a, pidx);
    const LcInfo& L = a.lcs[lc];
    const int64_t j = pidx - a.freq_off[lc] + 1;
    for (int q = lane; q < 3 * H; q += 64) {
      const int g = q < 2 * H ? 0 : 1;
      const int k = g == 0 ? q + 1 : q - 2 * H + 1;
      double2 v = L.status ? make_double2(0.0, 0.0) : gather_mode<R>(L, g, (int64_t)k * j, grids);
      if (g == 1) v = cscale(v, sqrt(L.yy));
      out[(pidx * 3 * H + q) * 2] = v.x;
      out[(pidx * 3 * H + q) * 2 + 1] = v.y;
    }
  }
}

// chi^2_0 of each lightcurve of a chunk (Section 2.2): sum (y - ybar)^2 /
// sigma^2 = YY / w_inv with YY = sum w (y - ybar)^2, sum w = 1 (unit weights:
// w_inv = 1/N); 0 for a rejected lightcurve.
__global__ __launch_bounds__(256) void k_lc_chi2(const LcInfo* lcs, int64_t n_lc, double* out) {
  const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (i < n_lc) out[i] = lcs[i].status == 0 ? lcs[i].yy / lcs[i].winv : 0.0;
}

// Multi-phase multi-band combination (Section 2.2, Eq.
// multibandmultiphase): power[j] = sum_k chi2[k] P_k[j] / sum_k chi2[k] over
// the band periodograms P_k = bp[k n_f + j]; 0 when every band was rejected.
__global__ __launch_bounds__(256) void k_mb_combine(const double* bp, int64_t n_band, int64_t n_f,
                                                    const double* chi2, double* power) {
  const int64_t j = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (j >= n_f) return;
  double num = 0.0, den = 0.0;
  for (int64_t k = 0; k < n_band; ++k) {
    num += chi2[k] * bp[k * n_f + j];
    den += chi2[k];
  }
  power[j] = den > 0.0 ? num / den : 0.0;
}

// Clears n counters (a kernel rather than a memset node, so that captured
// graphs replay it like any other launch).
__global__ __launch_bounds__(256) void k_zero_u32(unsigned* p, int64_t n, unsigned* p2) {
  for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < n; i += (int64_t)gridDim.x * 256) {
    p[i] = 0u;
    if (p2) p2[i] = 0u;
  }
}

// lc_stats[0..3] = t_ref, ybar, YY, status bits of the first lightcurve.
__global__ void k_export_stats(const LcInfo* lcs, double* out) {
  if (threadIdx.x == 0) {
    out[0] = lcs[0].tref;
    out[1] = lcs[0].ybar;
    out[2] = lcs[0].yy;
    out[3] = (double)lcs[0].status;
  }
}

// ------------------------------------------------------------ launchers

template <typename R>
static void launch_assemble_r(const SolveArgs& a, double* rec, int64_t p0, int64_t np, unsigned wg, int nw,
                             hipStream_t st) {
  const dim3 grid(wg), block(64 * nw);
  const size_t lds = asm2_lds_bytes(a.H, a.n_band, nw);
  const bool g16 = asm_group(a.H) == 16;
  if (a.sums_in) {
    if (g16) hipLaunchKernelGGL((k_assemble<double, 16, 0, kFromSums>), grid, block, lds, st, a, rec, p0, np);
    else hipLaunchKernelGGL((k_assemble<double, 32, 0, kFromSums>), grid, block, lds, st, a, rec, p0, np);
    return;
  }
  switch (a.H) {
#define FTP_ASM(h)                                                                                                  \
  case h:                                                                                                           \
    if (a.n_band) hipLaunchKernelGGL((k_assemble<R, asm_group(h), h, kFromBands>), grid, block, lds, st, a, rec, p0, np); \
    else hipLaunchKernelGGL((k_assemble<R, asm_group(h), h, kFromGrids>), grid, block, lds, st, a, rec, p0, np);     \
    break;
    FTP_ASM(1) FTP_ASM(2) FTP_ASM(3) FTP_ASM(4) FTP_ASM(5)
    FTP_ASM(6) FTP_ASM(7) FTP_ASM(8) FTP_ASM(9) FTP_ASM(10)
#undef FTP_ASM
    default:   // (H as an argument costs 3 % here, where f's recurrence dominates)
      if (a.n_band) hipLaunchKernelGGL((k_assemble<R, 32, 0, kFromBands>), grid, block, lds, st, a, rec, p0, np);
      else hipLaunchKernelGGL((k_assemble<R, 32, 0, kFromGrids>), grid, block, lds, st, a, rec, p0, np);
  }
}

hipError_t launch_assemble(int precision, const SolveArgs& a, double* rec, int64_t p0, int64_t np, int waves,
                           hipStream_t st) {
  // several frequencies per wavefront, kAsmWaves wavefronts per workgroup (one where
  // many bands of many harmonics would not fit its LDS: at most 44 KB)
  const int per = 64 / asm_group(a.H);
  const int nw = asm2_lds_bytes(a.H, a.n_band, kAsmWaves) <= ((size_t)64 << 10) ? kAsmWaves : 1;
  const int64_t w2 = std::max<int64_t>(1, std::min<int64_t>(waves, (np + per - 1) / per));
  if (precision == 1) launch_assemble_r<double>(a, rec, p0, np, (unsigned)((w2 + nw - 1) / nw), nw, st);
  else launch_assemble_r<float>(a, rec, p0, np, (unsigned)((w2 + nw - 1) / nw), nw, st);
  return hipGetLastError();
}

hipError_t launch_score(const SolveArgs& a, const double* rec, int64_t p0, int64_t np, int waves,
                        hipStream_t st, const int64_t* list, const unsigned* list_n) {
  if (6 * a.H - 2 > 64)
    hipLaunchKernelGGL(k_score<2>, dim3((unsigned)waves), dim3(64), score_lds_bytes(a.H), st, a, rec, p0, np, list,
                       list_n);
  else
    hipLaunchKernelGGL(k_score<1>, dim3((unsigned)waves), dim3(64), score_lds_bytes(a.H), st, a, rec, p0, np, list,
                       list_n);
  return hipGetLastError();
}

// Newton-candidate pairs, four per wavefront (see k_score4), one above H = 10 (the
// pairs the fallback tiers work on beside it are skipped); `done` (nullable): an
// event the launch itself records at the kernel's end.
hipError_t launch_score_newton(const SolveArgs& a0, const double* rec, int64_t p0, int64_t np, int waves, hipStream_t st,
                         hipEvent_t done) {
  SolveArgs a = a0;
  a.newton_cands = 2;
  if (a.H > 10) {
    const dim3 g((unsigned)waves);
    if (a.H == 11)
      hipExtLaunchKernelGGL(k_score<1>, g, dim3(64), score_lds_bytes(a.H), st, nullptr, done, 0, a, rec, p0, np,
                            (const int64_t*)nullptr, (const unsigned*)nullptr);
    else
      hipExtLaunchKernelGGL(k_score<2>, g, dim3(64), score_lds_bytes(a.H), st, nullptr, done, 0, a, rec, p0, np,
                            (const int64_t*)nullptr, (const unsigned*)nullptr);
    return hipGetLastError();
  }
  // consecutive frequencies per wavefront: more amortise the finish, fewer fill
  // the chip (twice over at four wavefronts per SIMD)
  const int w = std::max(1, std::min(waves, 8192));
  const int64_t want = (np + w - 1) / w;
  const int per = (int)std::min<int64_t>(kScorePer, std::max<int64_t>(4, (want + 3) & ~(int64_t)3));
  const dim3 grid((unsigned)((np + per - 1) / per));
  const size_t lds = score4_lds_bytes(a.H);
  switch (a.H) {
#define FTP_SCORE4(h) case h: hipExtLaunchKernelGGL((k_score4<h>), grid, dim3(64), lds, st, nullptr, done, 0, a, rec, p0, np, per); break;
    FTP_SCORE4(1) FTP_SCORE4(2) FTP_SCORE4(3) FTP_SCORE4(4) FTP_SCORE4(5)
    FTP_SCORE4(6) FTP_SCORE4(7) FTP_SCORE4(8) FTP_SCORE4(9) FTP_SCORE4(10)
#undef FTP_SCORE4
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

hipError_t launch_gather_sums(int precision, const SolveArgs& a, double* out, int blocks, hipStream_t st) {
  if (precision == 1)
    hipLaunchKernelGGL(k_gather_sums<double>, dim3((unsigned)blocks), dim3(64), 0, st, a, out);
  else
    hipLaunchKernelGGL(k_gather_sums<float>, dim3((unsigned)blocks), dim3(64), 0, st, a, out);
  return hipGetLastError();
}

hipError_t launch_lc_chi2(const LcInfo* lcs, int64_t n_lc, double* out, hipStream_t st) {
  hipLaunchKernelGGL(k_lc_chi2, dim3((unsigned)((n_lc + 255) / 256)), dim3(256), 0, st, lcs, n_lc, out);
  return hipGetLastError();
}

hipError_t launch_mb_combine(const double* bp, int64_t n_band, int64_t n_f, const double* chi2, double* power,
                             hipStream_t st) {
  hipLaunchKernelGGL(k_mb_combine, dim3((unsigned)((n_f + 255) / 256)), dim3(256), 0, st, bp, n_band, n_f, chi2,
                     power);
  return hipGetLastError();
}

// Clears p[0..n) and, when given, p2[0..n) in one launch.
hipError_t launch_zero_u32(unsigned* p, int64_t n, hipStream_t st, unsigned* p2) {
  if (n <= 0) return hipSuccess;
  const int64_t blocks = (n + 255) / 256 < 4096 ? (n + 255) / 256 : 4096;
  hipLaunchKernelGGL(k_zero_u32, dim3((unsigned)blocks), dim3(256), 0, st, p, n, p2);
  return hipGetLastError();
}

hipError_t launch_export_stats(const LcInfo* lcs, double* out, hipStream_t st) {
  hipLaunchKernelGGL(k_export_stats, dim3(1), dim3(64), 0, st, lcs, out);
  return hipGetLastError();
}

}  // namespace ftp

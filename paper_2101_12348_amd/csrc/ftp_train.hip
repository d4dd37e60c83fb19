// Training kernels of the root-proposal network: loss and gradient of a batch.
// Rows of the batch are independent through the forward pass, the loss and
// the backward pass, so one kernel takes a tile of rows through all of them
// with the activations in LDS (k_train_rows); the weight gradients are one
// split-K launch for the four layers (k_wgrad), and one launch adds the
// partial sums of weights and biases in a fixed order (k_grad_reduce).
#include <algorithm>

#include "ftp_args.h"
#include "ftp_mlp_tile.h"
#include "ftp_solve_common.h"

namespace ftp {

namespace {

__device__ __forceinline__ bool bf16_positive(uint16_t b) { return !(b & 0x8000u) && (b & 0x7fffu); }

// v of the other 16-lane row of the half-wave (v_permlane16_swap exchanges the
// odd rows of its first operand with the even rows of its second).
__device__ __forceinline__ float other_row(float v, int lane) {
  const unsigned u = __float_as_uint(v);
  const auto r = __builtin_amdgcn_permlane16_swap(u, u, false, false);
  return __uint_as_float((lane & 16) ? (unsigned)r[0] : (unsigned)r[1]);
}
template <int CTRL>
__device__ __forceinline__ float dpp_f(float v) {
  return __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(v), CTRL, 0xf, 0xf, true));
}
// Minimum and sum over the 32 lanes of a half-wave, in each of them: quad
// permutes and mirrors within the rows, then the two rows.
__device__ __forceinline__ float half_min(float v, int lane) {
  v = fminf(v, dpp_f<0xB1>(v));
  v = fminf(v, dpp_f<0x4E>(v));
  v = fminf(v, dpp_f<0x141>(v));
  v = fminf(v, dpp_f<0x140>(v));
  return fminf(v, other_row(v, lane));
}
__device__ __forceinline__ float half_sum(float v, int lane) {
  v += dpp_f<0xB1>(v);
  v += dpp_f<0x4E>(v);
  v += dpp_f<0x141>(v);
  v += dpp_f<0x140>(v);
  return v + other_row(v, lane);
}

// Chamfer loss on the circle of one sample (see k_chamfer) on a half-wave: lane
// k holds seed (ou, ov); the roots' directions are computed a root per lane and
// read back from LDS (dir, 32 of them, this half-wave's own).  (gu, gv)
// receives dL/d(u, v) of the lane's seed; returns L.  As in k_chamfer, a root
// that no seed is within 3.4e38 of (seeds not finite) counts as nearest to seed
// 0, so the gradients of a network that has diverged are not finite either, and
// the terms are divided before they are added, so that none overflows early.
__device__ __forceinline__ float chamfer_half(float ou, float ov, int Kseeds, const float* roots, int n, float lam,
                                              int lane, float2* dir, float& gu, float& gv) {
  const int hl = lane & 31, hb = lane & 32;
  const bool on = hl < Kseeds;
  float L = 0.f, best = 3.4e38f, bu = 0.f, bv = 0.f;
  gu = gv = 0.f;
  // x / n by the correctly rounded reciprocal and one residual step
  // (Markstein: the correctly rounded quotient); the residual of an infinite x is
  // NaN, which the maximum drops
  const float fn = (float)(n > 0 ? n : 1), rn = 1.f / fn;
  auto over_n = [&](float x) {
    const float q = x * rn;
    return fmaf(fmaxf(fmaf(-q, fn, x), -3.4e38f), rn, q);
  };
  // (both halves run as many roots as the longer of the two samples has)
  const int nmax = max(n, __shfl_xor(n, 32));
  for (int j0 = 0; j0 < nmax; j0 += 32) {
    float sn = 0.f, cs = 0.f;
    if (j0 + hl < n) sincosf(roots[j0 + hl], &sn, &cs);
    dir[hl] = make_float2(cs, sn);
    __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
    __builtin_amdgcn_wave_barrier();
#pragma unroll 4
    for (int q = 0; q < min(32, nmax - j0); ++q) {
      const float2 d = dir[q];
      const bool has = j0 + q < n;
      const float du = ou - d.x, dv = ov - d.y;
      const float d2 = du * du + dv * dv;
      // nearest seed of the root (the lowest index among equals)
      const float db = half_min(on ? d2 : 3.4e38f, lane);
      const unsigned hit = (unsigned)(__ballot(on && d2 == db) >> hb);
      if (has) {
        L = fmaf(db, rn, L);
        const bool mine = hl == __ffs(hit ? hit : 1u) - 1;
        gu += mine ? over_n(2.f * du) : 0.f;
        gv += mine ? over_n(2.f * dv) : 0.f;
        // nearest root of the seed
        if (d2 < best) {
          best = d2;
          bu = du;
          bv = dv;
        }
      }
    }
    __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
    __builtin_amdgcn_wave_barrier();
  }
  const float back = half_sum(on ? lam * best / Kseeds : 0.f, lane);
  if (n > 0) {
    L += back;
    gu += lam * 2.f * bu / Kseeds;
    gv += lam * 2.f * bv / Kseeds;
  }
  return L;
}

// Rows of the LDS tile (W columns, a multiple of 8) to global rows row0 ..: two
// rows per wave, 16 bytes per lane.
__device__ __forceinline__ void store_rows(const uint16_t* t, uint16_t* out, int W, int64_t row0, int64_t B, int wave,
                                           int lane) {
  const int i = 2 * wave + (lane >> 5), c = 8 * (lane & 31);
  if (row0 + i < B && c < W)
    *reinterpret_cast<uint4*>(out + (row0 + i) * W + c) = *reinterpret_cast<const uint4*>(t + i * kTileLd + c);
}

}  // namespace

// Forward, loss and backward of kTileRows samples per workgroup: activations,
// masks and upstream gradients stay in LDS, each wave owns one 16-column tile
// of every layer (ftp_mlp_tile.h).  Written out: the hidden activations and the
// gradients at every layer's output in bf16 (the operands of k_wgrad), the
// loss, and per tile the column sums of the FP32 gradients (bias gradients).
// Same operands, K order and rounding points as one k_gemm_bf16 launch per
// layer, so activations and gradients equal those bit for bit.  Bound by the
// latency of seven layers in a row, each one round of weight loads from L2
// (issued a layer ahead) and eight MFMA steps per wave: 45 us for 8192 rows of a
// 118-256-256-256-40 network, a seventh of it the loss.
__global__ __launch_bounds__(64 * kTileWaves) void k_train_rows(TrainArgs a) {
  __shared__ __align__(16) uint16_t xa[kTileRows * kTileLd];       // X, then the upstream gradients
  __shared__ __align__(16) uint16_t hh[3][kTileRows * kTileLd];    // hidden activations
  __shared__ float of[kTileRows * kTileOutLd];
  __shared__ float2 dir[kTileRows][32];                             // directions of the roots
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int mrow = lane & 15, n = 16 * wave + mrow;   // this lane's column of a layer
  const int64_t tile = a.tile0 + blockIdx.x, row0 = tile * kTileRows;
  const int W = a.width;
  float* part = a.bias_part + tile * (3 * W + a.dout);
  bf16x8_t f0[8], f1[8];
  tile_load_b(a.w + a.oW[0], a.din, a.din, W, n, lane, f0);
  // rows of X, zero-padded to whole K slices and past the batch
  {
    const int kp = (a.din + 31) & ~31;
#pragma unroll
    for (int r = 0; r < 2; ++r) {
      const int i = 2 * wave + r;
      for (int c = lane; c < kp; c += 64)
        xa[i * kTileLd + c] = (row0 + i < a.B && c < a.din) ? a.X[(row0 + i) * a.din + c] : (uint16_t)0;
    }
  }
  __syncthreads();
  f32x4_t acc[2];
  // forward
#pragma unroll 1
  for (int l = 0; l < 3; ++l) {
    tile_load_b(a.w + a.oW[l + 1], W, W, l == 2 ? a.dout : W, n, lane, f1);
    const uint16_t* in = l == 0 ? xa : hh[l - 1];
    if (16 * wave < W) {
      tile_mfma(in, l == 0 ? (a.din + 31) >> 5 : W >> 5, f0, lane, acc);
      const float bn = a.w32[a.ob[l] + n];
#pragma unroll
      for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int v = 0; v < 4; ++v)
          hh[l][(16 * i + 4 * (lane >> 4) + v) * kTileLd + n] = bf16_rne(fmaxf(acc[i][v] + bn, 0.f));
    }
    __syncthreads();
    store_rows(hh[l], a.h[l], W, row0, a.B, wave, lane);
#pragma unroll
    for (int s = 0; s < 8; ++s) f0[s] = f1[s];
  }
  // (the first backward layer's weights while the loss is formed)
  tile_load_b(a.wt[2], a.ldt[2], a.ldt[2], W, n, lane, f1);
  if (16 * wave < a.dout) {
    tile_mfma(hh[2], W >> 5, f0, lane, acc);
    if (n < a.dout) {
      const float bn = a.w32[a.ob[3] + n];
#pragma unroll
      for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int v = 0; v < 4; ++v) of[(16 * i + 4 * (lane >> 4) + v) * kTileOutLd + n] = acc[i][v] + bn;
    }
  }
  __syncthreads();
  // loss: one sample per half-wave
  {
    const int i = 2 * wave + (lane >> 5), hl = lane & 31, Ks = a.dout / 2;
    const int64_t b = row0 + i;
    const bool in = b < a.B;
    const int nr = in ? min(a.nroots[b], a.R) : 0;
    float* o = of + i * kTileOutLd;
    const float ou = hl < Ks ? o[2 * hl] : 0.f, ov = hl < Ks ? o[2 * hl + 1] : 0.f;
    float gu, gv;
    const float L = chamfer_half(ou, ov, Ks, a.roots + (in ? b : 0) * a.R, nr, a.lam, lane, dir[i], gu, gv);
    if (in && hl == 0) a.loss[b] = L;
    const float invB = 1.f / (float)a.B;
    gu *= invB;
    gv *= invB;
    if (hl < Ks) {
      o[2 * hl] = gu;
      o[2 * hl + 1] = gv;
    }
    // bf16 operand row, zero-padded to whole K slices
    const int kp = (a.dout + 31) & ~31;
    for (int c = hl; c < kp / 2; c += 32) {
      const unsigned u = c < Ks ? bf16_rne(gu) : 0u, v = c < Ks ? bf16_rne(gv) : 0u;
      reinterpret_cast<unsigned*>(xa + i * kTileLd)[c] = u | (v << 16);
      if (c < Ks && in) reinterpret_cast<unsigned*>(a.g[3] + b * a.dout)[c] = u | (v << 16);
    }
  }
  __syncthreads();
  if (tid < a.dout) {
    float s = 0.f;
    for (int i = 0; i < kTileRows; ++i) s += of[i * kTileOutLd + tid];
    part[3 * W + tid] = s;
  }
  // backward: gradient at the output of layer l - 1 from that of layer l (rows past
  // the batch stay zero also where a weight is not finite)
  const int rows = (int)min((int64_t)kTileRows, a.B - row0);
#pragma unroll 1
  for (int l = 3; l >= 1; --l) {
#pragma unroll
    for (int s = 0; s < 8; ++s) f0[s] = f1[s];
    if (l > 1) tile_load_b(a.wt[l - 2], a.ldt[l - 2], a.ldt[l - 2], W, n, lane, f1);
    if (16 * wave < W) tile_mfma(xa, (l == 3 ? a.dout + 31 : W) >> 5, f0, lane, acc);
    __syncthreads();   // every wave has read this layer's operand
    if (16 * wave < W) {
      float cs = 0.f;
#pragma unroll
      for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int v = 0; v < 4; ++v) {
          const int r = 16 * i + 4 * (lane >> 4) + v;
          const float x = r < rows && bf16_positive(hh[l - 1][r * kTileLd + n]) ? acc[i][v] : 0.f;
          cs += x;
          xa[r * kTileLd + n] = bf16_rne(x);
        }
      cs += __shfl_xor(cs, 16);
      cs += __shfl_xor(cs, 32);
      if (lane < 16) part[(l - 1) * W + n] = cs;
    }
    __syncthreads();
    store_rows(xa, a.g[l - 1], W, row0, a.B, wave, lane);
  }
}

// Partial weight gradients of every layer: dW_l[o, i] = sum_b g_l[b, o] in_l[b, i]
// over rows [s rows, (s + 1) rows) of the batch for each split s, one 64 x 64 tile
// of one layer per workgroup, FP32 sums written to wpart + s n_params.  Both
// operands have the batch as their leading dimension, so slices of 32 rows are
// loaded along the columns, two rows per thread, and turned on the way into
// LDS; the next two slices' loads are in flight during the MFMAs.  The split gives a few hundred
// workgroups where the 44 tiles alone (H = 10) would leave the device idle (24
// us for 8192 rows; one unsplit GEMM per layer took 4.9 ms).
__global__ __launch_bounds__(256) void k_wgrad(WgradArgs a) {
  __shared__ __align__(16) unsigned As[2][64 * 20];
  __shared__ __align__(16) unsigned Bs[2][64 * 20];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  // workgroups go to the eight XCDs in turn: the tiles of one split, which read
  // the same rows, stay on one (its L2 then fetches them once)
  const int ntile = a.tiles[0] + a.tiles[1] + a.tiles[2] + a.tiles[3];
  const int within = blockIdx.x >> 3, split = (blockIdx.x & 7) + 8 * (within / ntile);
  if (split >= a.splits) return;
  int l = 0, t = within % ntile;
  while (l < 3 && t >= a.tiles[l]) t -= a.tiles[l++];
  const int nout = a.nout[l], nin = a.nin[l];
  const int ti = (nin + 63) / 64;
  const int o0 = (t / ti) * 64, i0 = (t % ti) * 64;
  const uint16_t* G = a.g[l];
  const uint16_t* I = a.in[l];
  const int64_t b0 = (int64_t)split * a.rows, b1 = min(a.B, b0 + a.rows);
  const int wm = (wave >> 1) * 32, wn = (wave & 1) * 32;
  f32x4_t acc[2][2];
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int j = 0; j < 2; ++j) acc[i][j] = f32x4_t{0.f, 0.f, 0.f, 0.f};
  // loader: rows 2 rp and 2 rp + 1 of a slice, columns c .. c + 3; row pairs
  // become 32-bit words, word rp of LDS row (column) c + q.  The 16-byte chunk
  // of a word is exchanged by the column's multiple of 16, so that neither
  // these writes nor the fragment reads meet bank conflicts.
  const int rp = tid >> 4, lc = (tid & 15) * 4;
  const int wdst = lc * 20 + (((rp >> 2) ^ (lc >> 4)) << 2) + (rp & 3);
  union V { uint2 u; uint16_t e[4]; };
  V va[2][2], vb[2][2];   // two slices of 32 rows
  // Columns past the operand feed only outputs that are not stored, so their
  // loads are merely kept in bounds; rows past the split must count as zero (in
  // one operand).
  auto load4 = [&](const uint16_t* S, int ld, int c0, int64_t b) {
    V v;
    const int c = c0 + lc;
    const uint16_t* p = S + b * ld;
    if (c + 4 <= ld || c >= ld) {
      __builtin_memcpy(&v, p + (c + 4 <= ld ? c : 0), 8);
    } else {
#pragma unroll
      for (int q = 0; q < 4; ++q) v.e[q] = p[min(c + q, ld - 1)];
    }
    return v;
  };
  const bool in_a = o0 + 64 <= nout, in_b = i0 + 64 <= nin;
  const bool wide = nout >= 4 && nin >= 4;
  auto fetch = [&](int64_t b) {
    if (in_a && in_b && b + 64 <= b1) {   // (uniform) whole slices of whole tiles
      const uint16_t* pa = G + (b + 2 * rp) * nout + o0 + lc;
      const uint16_t* pb = I + (b + 2 * rp) * nin + i0 + lc;
#pragma unroll
      for (int s = 0; s < 2; ++s)
#pragma unroll
        for (int r = 0; r < 2; ++r) {
          __builtin_memcpy(&va[s][r], pa + (32 * s + r) * nout, 8);
          __builtin_memcpy(&vb[s][r], pb + (32 * s + r) * nin, 8);
        }
      return;
    }
#pragma unroll
    for (int s = 0; s < 2; ++s)
#pragma unroll
      for (int r = 0; r < 2; ++r) {
        const int64_t row = b + 32 * s + 2 * rp + r, rc = min(row, b1 - 1);
        if (wide) {
          va[s][r] = load4(G, nout, o0, rc);
          vb[s][r] = load4(I, nin, i0, rc);
        } else {
#pragma unroll
          for (int q = 0; q < 4; ++q) {
            va[s][r].e[q] = G[rc * nout + min(o0 + lc + q, nout - 1)];
            vb[s][r].e[q] = I[rc * nin + min(i0 + lc + q, nin - 1)];
          }
        }
        if (row >= b1) va[s][r].u = make_uint2(0u, 0u);
      }
  };
  if (b0 < b1) fetch(b0);
  for (int64_t b = b0; b < b1; b += 64) {
#pragma unroll
    for (int s = 0; s < 2; ++s)
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        As[s][wdst + 20 * q] = va[s][0].e[q] | ((unsigned)va[s][1].e[q] << 16);
        Bs[s][wdst + 20 * q] = vb[s][0].e[q] | ((unsigned)vb[s][1].e[q] << 16);
      }
    __syncthreads();
    if (b + 64 < b1) fetch(b + 64);
#pragma unroll
    for (int s = 0; s < 2; ++s) {
      bf16x8_t af[2], bf[2];
      auto frag = [&](const unsigned* S, int c16) {
        const int c = 16 * c16 + (lane & 15);
        return *reinterpret_cast<const bf16x8_t*>(S + c * 20 + (((lane >> 4) ^ c16) << 2));
      };
#pragma unroll
      for (int i = 0; i < 2; ++i) {
        af[i] = frag(As[s], (wm >> 4) + i);
        bf[i] = frag(Bs[s], (wn >> 4) + i);
      }
#pragma unroll
      for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j)
          acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(af[i], bf[j], acc[i][j], 0, 0, 0);
    }
    __syncthreads();
  }
  float* out = a.wpart + (int64_t)split * a.n_params + a.oW[l];
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        const int o = o0 + wm + 16 * i + 4 * (lane >> 4) + v, c = i0 + wn + 16 * j + (lane & 15);
        if (o < nout && c < nin) out[(int64_t)o * nin + c] = acc[i][j][v];
      }
}

// Column sums over 32-row tiles of the FP32 gradient at a layer's output (the
// layer-by-layer path; k_train_rows forms them itself): part[t][n].
__global__ __launch_bounds__(256) void k_col_part(const float* G, int64_t M, int N, int64_t ld, float* part,
                                                  int ld_part) {
  const int n = blockIdx.y * 256 + threadIdx.x;
  if (n >= N) return;
  const int64_t m0 = (int64_t)blockIdx.x * kTileRows, m1 = min(M, m0 + kTileRows);
  float s = 0.f;
  for (int64_t m = m0; m < m1; ++m) s += G[m * ld + n];
  part[(int64_t)blockIdx.x * ld_part + n] = s;
}

// Gradients from the partial sums, in a fixed order: workgroups below a.wblocks
// take 256 weights each (the splits in turn), the others a bias per wavefront
// (the tiles strided over the lanes, then the lanes by halving).
__global__ __launch_bounds__(256) void k_grad_reduce(WgradArgs a, float* grad) {
  if ((int)blockIdx.x < a.wblocks) {
    int64_t p = (int64_t)blockIdx.x * 256 + threadIdx.x;   // index among the weights
    int l = 0;
    for (; l < 4; ++l) {
      const int64_t c = (int64_t)a.nin[l] * a.nout[l];
      if (p < c) break;
      p -= c;
    }
    if (l == 4) return;
    const float* w = a.wpart + a.oW[l] + p;
    float s = 0.f;
#pragma unroll 4
    for (int k = 0; k < a.splits; ++k) s += w[(int64_t)k * a.n_params];
    grad[a.oW[l] + p] = s;
    return;
  }
  const int lane = threadIdx.x & 63;
  const int nb = a.nout[0] + a.nout[1] + a.nout[2] + a.nout[3];
  int c = (blockIdx.x - a.wblocks) * 4 + (threadIdx.x >> 6);
  if (c >= nb) return;
  float s = 0.f;
  for (int t = lane; t < a.btiles; t += 64) s += a.bias_part[(int64_t)t * nb + c];
  for (int o = 32; o > 0; o >>= 1) s += __shfl_xor(s, o);
  int l = 0;
  while (c >= a.nout[l]) c -= a.nout[l++];
  if (lane == 0) grad[a.ob[l] + c] = s;
}

// Tiles of a launch: a grid of 2^32 threads and more is cut short without an
// error, so larger batches take several launches.
constexpr int64_t kLaunchTiles = 1 << 21;

hipError_t launch_train_rows(TrainArgs a, hipStream_t st) {
  const int64_t tiles = (a.B + kTileRows - 1) / kTileRows;
  for (a.tile0 = 0; a.tile0 < tiles; a.tile0 += kLaunchTiles)
    hipLaunchKernelGGL(k_train_rows, dim3((unsigned)std::min(kLaunchTiles, tiles - a.tile0)), dim3(64 * kTileWaves), 0,
                       st, a);
  return hipGetLastError();
}

hipError_t launch_col_part(const float* G, int64_t M, int N, int64_t ld, float* part, int ld_part, hipStream_t st) {
  const int64_t tiles = (M + kTileRows - 1) / kTileRows;
  for (int64_t t = 0; t < tiles; t += kLaunchTiles)
    hipLaunchKernelGGL(k_col_part, dim3((unsigned)std::min(kLaunchTiles, tiles - t), (unsigned)((N + 255) / 256)),
                       dim3(256), 0, st, G + t * kTileRows * ld, M - t * kTileRows, N, ld, part + t * ld_part, ld_part);
  return hipGetLastError();
}

// Fills in the tile counts of `a` and launches the weight gradients and the
// final sums into `grad`.
hipError_t launch_wgrad(WgradArgs a, float* grad, hipStream_t st) {
  int tiles = 0, nb = 0;
  int64_t nw = 0;
  for (int l = 0; l < 4; ++l) {
    a.tiles[l] = ((a.nout[l] + 63) / 64) * ((a.nin[l] + 63) / 64);
    tiles += a.tiles[l];
    nb += a.nout[l];
    nw += (int64_t)a.nin[l] * a.nout[l];
  }
  a.wblocks = (int)((nw + 255) / 256);
  hipLaunchKernelGGL(k_wgrad, dim3((unsigned)(tiles * ((a.splits + 7) & ~7))), dim3(256), 0, st, a);
  hipLaunchKernelGGL(k_grad_reduce, dim3((unsigned)(a.wblocks + (nb + 3) / 4)), dim3(256), 0, st, a, grad);
  return hipGetLastError();
}

}  // namespace ftp

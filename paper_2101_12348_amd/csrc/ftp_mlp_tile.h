// Building blocks of the network kernels that keep a tile of rows in LDS and
// take it through the layers: 32 rows per workgroup of sixteen waves, each wave
// on one 16-column tile of a layer (width <= 256), K <= 256.  A wave's weight
// fragments of a whole layer (eight 16-byte loads) are issued together, so a
// layer costs one round of memory latency at most.
#pragma once

#include "ftp_internal.h"

namespace ftp {

typedef __attribute__((__vector_size__(8 * sizeof(__bf16)))) __bf16 bf16x8_t;
typedef __attribute__((__vector_size__(4 * sizeof(float)))) float f32x4_t;

// float -> bf16 bits by the hardware conversion (round to nearest even, one
// instruction on gfx950; equal to f2bf for finite values)
__device__ __forceinline__ uint16_t bf16_rne(float x) { return __builtin_bit_cast(uint16_t, (__bf16)x); }

constexpr int kTileWaves = 16;
constexpr int kTileLd = 256 + 8;      // LDS row of one sample's activations (bf16)
constexpr int kTileOutLd = 64 + 4;    // LDS row of one sample's outputs (FP32)

// B fragments of the wave's column tile: column n (row n of W, clamped to the
// last), k = 32 s + 8 (lane / 16) .. + 7 of slice s, zero from K on.  Rows of W
// have stride ld; slices past K are not loaded (K is wave-uniform, so the
// whole slices are unconditional loads).
__device__ __forceinline__ void tile_load_b(const uint16_t* W, int ld, int K, int nout, int n, int lane,
                                            bf16x8_t (&f)[8]) {
  const uint16_t* row = W + (int64_t)min(n, nout - 1) * ld + 8 * (lane >> 4);
  const int full = K >> 5;
#pragma unroll
  for (int s = 0; s < 8; ++s) {
    if (s < full) {
      __builtin_memcpy(&f[s], row + 32 * s, 16);
    } else if (s == full && (K & 31)) {
      union { bf16x8_t v; uint4 u; uint16_t e[8]; } x;
      x.u = make_uint4(0u, 0u, 0u, 0u);
#pragma unroll
      for (int q = 0; q < 8; ++q)
        if (32 * s + 8 * (lane >> 4) + q < K) x.e[q] = row[32 * s + q];
      f[s] = x.v;
    }
  }
}

// acc[i] = rows 16 i .. + 15 of `in` (LDS) times the fragments, ns slices; lane
// holds rows 16 i + 4 (lane / 16) + v of column lane % 16 of the wave's tile.
__device__ __forceinline__ void tile_mfma(const uint16_t* in, int ns, const bf16x8_t (&f)[8], int lane,
                                          f32x4_t (&acc)[2]) {
  acc[0] = f32x4_t{0.f, 0.f, 0.f, 0.f};
  acc[1] = f32x4_t{0.f, 0.f, 0.f, 0.f};
  const uint16_t* a0 = in + (lane & 15) * kTileLd + 8 * (lane >> 4);
#pragma unroll
  for (int s = 0; s < 8; ++s) {
    if (s < ns) {
      const bf16x8_t x0 = *reinterpret_cast<const bf16x8_t*>(a0 + 32 * s);
      const bf16x8_t x1 = *reinterpret_cast<const bf16x8_t*>(a0 + 16 * kTileLd + 32 * s);
      acc[0] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(x0, f[s], acc[0], 0, 0, 0);
      acc[1] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(x1, f[s], acc[1], 0, 0, 0);
    }
  }
}

}  // namespace ftp

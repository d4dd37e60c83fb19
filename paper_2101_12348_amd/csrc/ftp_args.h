// Argument blocks of the per-frequency kernels that the host runtime
// launches, shared by the kernels' sources and ftp_capi.hip (one definition).
#pragma once

#include "ftp_internal.h"

namespace ftp {

// Newton + Sturm (first round): pairs [0, np) of a record chunk.
struct LearnArgs {
  double* rec;
  int64_t np;
  const float* seeds_out;   // network output, np x 4H (u, v pairs); nullptr = evenly spaced starts
  int64_t* fb_list;         // pairs the round leaves unconfirmed
  unsigned int* fb_count;
  unsigned flags;           // bit 0: forced fallback (every pair to the list); bit 1: 2H starts only
  const double2* starts;    // H <= 10: evenly spaced starts per rotation (k_start_table)
  int per;                  // H <= 5 and H >= 12: frequencies per wavefront (newton_per)
};

// Second Newton round over the first round's list (k_newton_retry).
struct RetryArgs {
  double* rec;
  int H;
  const int64_t* list;       // first-round fallback list
  const unsigned* count;     // its length
  const float* seeds;        // nullable: network output rows in list order
  int64_t* out_list;         // pairs left to the Aberth tier
  unsigned* out_count;
  SolveCounters* counters;
};

// Aberth tier (or the Aberth solver over every pair).
struct AberthArgs {
  double* rec;
  int64_t np;
  const int64_t* list;       // pairs to solve; nullptr = every pair of the chunk
  const unsigned* count;     // length of `list`
  int64_t* qr_list;          // pairs left to the companion-matrix solve
  unsigned* qr_count;
  SolveCounters* counters;
  int H;
  double mark;               // M_FALLBACK value written for pairs sent on
  unsigned flags;            // bit 0: send every pair on (companion solve only)
  unsigned* queue;           // work counter (zeroed), or nullptr for grid striding
};

// The four network layers in one kernel (k_mlp_fused).
struct FusedMlpArgs {
  const uint16_t* X;     // np x kp[0] bf16 features (zero padded)
  int64_t np;
  const uint16_t* wi;    // padded bf16 weights, layer l at wi + oWi[l], rows of kp[l]
  const float* w32;      // FP32 parameters (biases at w32 + ob[l])
  int64_t oWi[4], ob[4];
  int kp[4], nout[4];
  float* out;            // np x nout[3]
  const unsigned* np_dev;   // nullable: rows past *np_dev (on the device) are skipped
};

// Rows of a training batch per workgroup of k_train_rows, and per partial sum
// of the bias gradients.
constexpr int kTileRows = 32;

// Transposed bf16 weights of layers 1..3 of a network whose training runs
// through k_train_rows: layer l + 1 at p[l], `nin` rows of ld[l] (nout[l] padded
// with zeros to whole K slices); p[0] == nullptr for other networks.
struct TransposedWeights {
  uint16_t* p[3];
  int64_t oW[3];            // offsets of these layers in the parameters
  int nin, nout[3], ld[3];
};

// Forward, loss and backward of a batch (k_train_rows): width a multiple of 32
// up to 256, din up to 256.
struct TrainArgs {
  const uint16_t* X;        // B x din bf16
  int64_t B;
  int64_t tile0;            // first tile of the launch (filled in by the launcher)
  int din, width, dout;
  const uint16_t* w;        // bf16 weights, layer l at w + oW[l]
  const float* w32;         // FP32 parameters (biases at w32 + ob[l])
  int64_t oW[4], ob[4];
  const uint16_t* wt[3];    // transposed weights of layers 1..3 (TransposedWeights), rows of ldt[l]
  int ldt[3];
  const float* roots;       // B x R
  const int* nroots;
  int R;
  float lam;
  uint16_t* h[3];           // hidden activations, B x width
  uint16_t* g[4];           // gradients at the layers' outputs (bf16), B x width (layer 3: B x dout)
  float* loss;              // B
  float* bias_part;         // per tile of kTileRows rows: 3 width + dout column sums
};

// Weight gradients of a batch (k_wgrad) and the final sums (k_grad_reduce).
struct WgradArgs {
  const uint16_t* g[4];     // gradients at the layers' outputs, B x nout[l]
  const uint16_t* in[4];    // the layers' inputs, B x nin[l]
  int nin[4], nout[4];
  int64_t oW[4], ob[4];
  int64_t B, rows;          // rows per split (a multiple of 32)
  int splits;
  float* wpart;             // splits x n_params
  int64_t n_params;
  const float* bias_part;   // btiles x (sum of nout)
  int btiles;
  int tiles[4], wblocks;    // filled in by the launcher
};

}  // namespace ftp

// Launch interface between the training step (k_train.hip) and the fused
// forward and backward chains (k_chain.hip).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "blob_layout.h"
#include "train_layout.h"

namespace nedf {

constexpr int HEAD_PART = 520;  // 512 weight grads, 2 bias grads, 3 loss terms (total, mse, bce)

struct ChainLineArgs {
  const float *o_l, *d_l, *depth;
  const uint8_t* hit;
  int B, enc_L, n_hidden;
  float bound, w_hit;
  const uint8_t* w[NEDF_MAX_LAYERS];   // packed weights of the hidden layers
  const uint8_t* wt[NEDF_MAX_LAYERS];  // packed transposes (layers 1 ..)
  const float* bias[NEDF_MAX_LAYERS];
  const float *head_w, *head_b;        // [2][256], [2]
  uint16_t* Hin;                       // [B][16 K0] encoded input
  uint16_t* H;                         // [n_hidden][B][256] activations (the last one not written)
  uint16_t* G;                         // [n_hidden][B][256] gradients at the pre-activations
  uint8_t* bits;                       // [n_hidden][B / 32][4][64] words: signs of H (two blocks per lane)
  float* hpart;                        // [B / 128][HEAD_PART]
};

struct ChainPointsArgs {
  int B, n_blocks;
  float w_hit;
  const uint8_t* w[NEDF_TRAIN_MAX_LAYERS];   // packed weights (the head's with K outermost)
  const uint8_t* wt[NEDF_TRAIN_MAX_LAYERS];  // packed transposes (layers 1 ..)
  const float* bias[NEDF_TRAIN_MAX_LAYERS];
  const uint16_t* X;                         // [B][1024] encoded input, in 32 x 32 tiles
  const float *mu, *alpha;                   // [B]
  uint16_t *H, *A;                           // [n_blocks + 1][B][256] stream, [n_blocks][B][256] inner activations
  uint16_t* G;                               // [layers][B][256] gradients at the pre-activations
  uint8_t* bits;                             // [2 n_blocks + 1] sign arrays as in ChainLineArgs
  float* lpart;                              // [workgroups][3] loss sums (total, bins, hit)
};

// Waves per workgroup (each 32 rows) for a batch of B rows on `cus` compute
// units: a round of 8-wave workgroups takes about 1.8 times a round of 4-wave
// ones and holds twice the rows.
int chain_line_waves(int B, int cus);
void launch_chain_line(const ChainLineArgs& a, int n_comp, int k0, int waves, hipStream_t s);
// Two waves per workgroup while that is no more rounds than four (the chain
// of 16 blocks: 421 against 432 us at 16,384 rows, where four waves leave
// half of the compute units empty; 584 us with four at 32,768 rows, two
// rounds of 415 with two).
int chain_points_waves(int B, int cus);
void launch_chain_points(const ChainPointsArgs& a, int waves, hipStream_t s);

int cu_count();

}  // namespace nedf

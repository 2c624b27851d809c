// tt_mlp.h -- the screen network's inference over the wave pass's
// candidates compacted first (tt_mlp.hip), for tt_screen_infer, and its
// training step in one call, for tt_mlp_train_step.
#pragma once

#include <hip/hip_runtime.h>
#include <stddef.h>
#include <stdint.h>

#include "tt.h"

namespace tt {

// Candidates per span of the compaction pass (one block each), and the most
// spans the inference blocks' prefix sums hold (n up to 2^21).
constexpr int kGateSpan = 512;
constexpr int kGateMaxSpans = 4096;

// int32 elements of the work buffer for n candidates: the compacted list
// (kGateSpan per span) and one count per span.
inline size_t gate_work_ints(int n) {
  const size_t spans = ((size_t)n + kGateSpan - 1) / kGateSpan;
  return spans * kGateSpan + spans;
}

// Gated inference in two launches: a pass that compacts the candidates the
// screen's wave pass takes, span by span, into work; then the network over
// that list in chunks of 128 rows by a persistent grid of `blocks` blocks
// (one per CU: every block but the last gets a full chunk).  Requires
// n <= kGateSpan * kGateMaxSpans.  Weights and biases as mlp_infer; logits
// rows of the other candidates are not written.
hipError_t mlp_infer_gated_list(const tt_neuron* desc, int n, const uint16_t* const* w, const float* const* b,
                                float* logits, int32_t* work, int blocks, hipStream_t s);

// Parameters of the network: weights of the four layers, then biases.
constexpr int kTrainWeights = 32 * 256 + 2 * 256 * 256 + 256 * 12;
constexpr int kTrainParams = kTrainWeights + 3 * 256 + 12;
struct TrainArgs {
  const uint16_t* x;    // [batch][32]
  const float *y, *m, *h;
  const uint16_t* w[4];
  const float* b[4];
  uint16_t *act[3], *dh[3];  // [batch][256]
  float* z;             // [batch][12]
  uint16_t* dz;         // [batch][12]
  float* loss;
  float *p[8], *g[8], *am[8], *av[8];  // weights of the layers, then biases
  uint16_t* wb[4];      // == w, written by the update
  int batch;
  // in the scratch, set by train_step
  uint16_t* dzp;        // [batch][16]: dz, columns 12.. zero
  float* loss_part;
  int row_blocks;
  // weight gradients of layer l: slices[l] partial sums over kslice[l] rows
  // each, [slices][out][in] at part[l], and of its biases, [slices][out] at
  // dbp[l]
  int slices[4], kslice[4];
  float *part[4], *dbp[4];
};
// scratch of a step on `batch` rows; most: of one on any batch up to it
size_t train_scratch_floats(int batch, bool most);
hipError_t train_step(TrainArgs a, float* scratch, float lr, float b1, float b2, float eps, float bc1, float bc2,
                      hipStream_t s);

}  // namespace tt

// Launch interface of the verifier-head kernels (internal).
#pragma once

#include "device_util.h"

namespace pr {

constexpr int kHeadD = 64;        // model width
constexpr int kHeadFF = 128;      // feed-forward width
constexpr int kHeadHeads = 4;     // attention heads (16 dimensions each)
constexpr int kHeadLayers = 2;    // encoder layers
constexpr int kHeadWeights = 67329;

// Consecutive rows r0 .. of request req, whose rows are [lo, hi).
struct HeadBlock {
  int32_t r0, lo, hi, req;
};

struct HeadArgs {
  const float* X;          // [n_rows][4] input sequence (l, m, h, rho)
  int64_t n_rows;
  const int32_t* offsets;  // [n_req + 1]
  int32_t n_req;
  int32_t max_len;         // longest request that is scored
  const float* weights;    // [kHeadWeights]
  float* scores;           // [n_req]
  void* ws;                // workspace
  // the workspace's arrays, set by launch_head; np padded rows each
  int64_t np;
  __bf16* Ws;              // the weight matrices' three bfloat16 terms, in operand order
  float* H;                // [np][64] activations
  __bf16* Q;               // [4][np / 16] groups of 16 queries by head, three terms, in operand order
  __bf16* K[kHeadLayers];  // the keys of a layer, likewise
  float* V[kHeadLayers];   // the values of a layer by head and group of 16, in operand order
  float* z;                // [np] rows' products with the output map
  HeadBlock* items;        // [cap] row blocks of the requests, the heaviest first
  int32_t cap;
  int32_t* ctl;            // [0] number of blocks listed
};

// The head as one kernel per layer (head.hip) with head_workspace_bytes at
// a.ws, or as separate tile kernels (head_tiles.hip) with the smaller
// head_tiles_workspace_bytes.
size_t head_workspace_bytes(int64_t n_rows);
hipError_t launch_head(const HeadArgs& a, hipStream_t stream);
size_t head_tiles_workspace_bytes(int64_t n_rows);
hipError_t launch_head_tiles(const HeadArgs& a, hipStream_t stream);

}  // namespace pr

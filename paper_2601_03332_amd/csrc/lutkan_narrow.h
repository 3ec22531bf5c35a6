// The one-launch forward of narrow LUT layers (lutkan_narrow.hip), called by the dispatch in lutkan_kernels.hip.
#pragma once

#include <cstddef>
#include <cstdint>

#include "lutkan.h"

namespace lutkan {

struct NarrowPlan {
  int waves;           // per work-group; 0: the kernel does not serve the layer
  int n_split, chunk;  // chunks of inputs, inputs per chunk
  int stage;           // inputs whose slices are staged together
  double cost;         // estimate, microseconds
};
// The launch shape for B rows, with at most workspace_bytes of partial sums.
NarrowPlan narrow_plan(const lutkan_dev_layer *layer, int64_t B, size_t workspace_bytes);
int narrow_forward(const lutkan_dev_layer *layer, const NarrowPlan &plan, const float *x, int64_t B, float *y, void *workspace, void *hip_stream);

}  // namespace lutkan

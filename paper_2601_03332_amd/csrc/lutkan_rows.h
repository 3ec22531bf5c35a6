// The one-launch forward of a few rows (lutkan_rows.hip), called by the dispatch in lutkan_kernels.hip.
#pragma once

#include <cstdint>

#include "lutkan.h"

namespace lutkan {

struct RowsPlan {
  int waves_per_row;   // 16 or 4; 0: the kernel does not serve the layer
  double cost;         // estimate, microseconds
  double against_passes;   // what the passes must be priced above
};
RowsPlan rows_plan(const lutkan_dev_layer *layer, int64_t B);
int rows_forward(const lutkan_dev_layer *layer, const RowsPlan &plan, const float *x, int64_t B, float *y, void *hip_stream);

}  // namespace lutkan

// The B-spline layer on the matrix cores (bspline_matrix.hip), called by the dispatch in bspline_kernels.hip.
#pragma once

#include <cstddef>
#include <cstdint>

#include "lutkan.h"

namespace lutkan {

// Layers the matrix kernel serves: phi edges, at most 13 segments on the domain grid, one knot vector whose neighbouring gaps
// differ by less than a factor of about 3.
bool bspline_matrix_fits(const bspline_dev_layer *layer);
// The whole forward of a layer that fits.  `workspace` takes the partial sums when the inputs are split into chunks, as many
// chunks as it has room for.
int bspline_matrix_forward(const bspline_dev_layer *layer, const float *x, int64_t B, float *y, void *workspace, size_t workspace_bytes,
                           void *hip_stream);

}  // namespace lutkan

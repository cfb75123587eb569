// Launch interface of the top-p (nucleus) feature kernels (internal).
#pragma once

#include "row_features.h"

namespace pr {

size_t topp_workspace(pr_dtype dtype, int64_t n_rows, int32_t V);
// Workspace with which a small batch's rows are spread over several workgroups
// each (0: none is used); one workgroup per row with less.
size_t topp_split_workspace(int64_t n_rows, int32_t V, bool seq);
hipError_t launch_topp(const RowArgs& a, pr_dtype dtype, void* workspace, size_t workspace_bytes, hipStream_t stream);

}  // namespace pr

// Weight gradient of fp32 layers on the bf16 matrix cores (conv_wsplit.hip).
#pragma once
#include "common.h"

namespace distdl {

// Layers with channel counts that are multiples of 4 and tensors below 2 GiB whose staged rows fit in LDS; expects
// 16-byte aligned tensors and the plan's pointer tables (tab_x, tab_dy) uploaded.
bool wgrad_split_supported(const distdl_plan* p);
int wgrad_split_chunks(const distdl_plan* p);  // partials per worker; 0 where not supported
double wgrad_split_us(const distdl_plan* p);    // estimated time of its matrix instructions and steps
int conv_wgrad_split(distdl_plan* p, float* partial, hipStream_t st);

}  // namespace distdl

// Convolution of fp32 tensors on the bf16 matrix cores (conv_split.hip).  The entry points expect the plan's pointer
// tables to be uploaded; the tensors that are read, and (channel counts that are multiples of 4) those that are written,
// are 16-byte aligned.
#pragma once
#include "common.h"
#include "weight_job.h"

namespace distdl {

bool corr_split_supported(const distdl_plan* p, bool backward);
double corr_split_used(const distdl_plan* p, bool backward);  // part of its windows that are outputs
double corr_split_us(const distdl_plan* p, bool backward);  // estimated time
void corr_split_shape(const distdl_plan* p, bool backward, int32_t out[5]);  // see distdl_debug_conv_split
// The job that has to be done before either of the following.
int split_weight_job(distdl_plan* p, bool backward, const float* w, hipStream_t st, WeightJob& job);
int conv_fwd_split(distdl_plan* p, const float* w, const float* bias, hipStream_t st);
int conv_bwd_data_split(distdl_plan* p, const float* w, hipStream_t st);

}  // namespace distdl

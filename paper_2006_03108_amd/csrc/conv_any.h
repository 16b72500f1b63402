// Convolution kernels for any shape whose tensors are addressed by 31-bit byte offsets (conv_any.hip).  The entry
// points expect the plan's pointer tables to be uploaded; `aligned`: the arrays that are read are 16-byte aligned.
#pragma once
#include "common.h"
#include "weight_job.h"

namespace distdl {

bool conv_any_supported(const distdl_plan* p);
// The job that has to be done before either of the following.
int any_weight_job(distdl_plan* p, bool backward, const void* w, bool aligned, hipStream_t st, WeightJob& job);
int conv_fwd_any(distdl_plan* p, const void* w, const void* bias, bool aligned, hipStream_t st);
int conv_bwd_data_any(distdl_plan* p, const void* w, bool aligned, hipStream_t st);
double corr_any_us(const distdl_plan* p, bool backward, bool aligned);  // estimated time
int wgrad_any_chunks(const distdl_plan* p);
int wgrad_any_rows(const distdl_plan* p);       // of a tile: 64 or 256
bool wgrad_any_unsure(const distdl_plan* p);    // the estimate is one of 64 rows alone
double wgrad_any_us(const distdl_plan* p);  // estimated time
int conv_wgrad_any(distdl_plan* p, float* partial, hipStream_t st);

}  // namespace distdl

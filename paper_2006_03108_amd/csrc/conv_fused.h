// Small convolution layers: the forward pass in one launch, the adjoint in one or two (conv_fused.hip).
#pragma once
#include "common.h"

namespace distdl {

// Both directions are calls with their halo exchange.  vec: channel counts are multiples of 4 and all arrays 16-byte aligned.
double conv_fused_us(const distdl_plan* p, bool backward, bool vec);  // estimated time; infinite: not taken
void conv_fused_make_tables(const distdl_plan* p, bool backward);  // on the host
int conv_fused_records(const distdl_plan* p, bool backward);        // of 176 bytes, in those tables
// The tables that have been made, for the copy that a plan's first call makes.
void conv_fused_add_tables(const distdl_plan* p, HostTables& t);
bool conv_fused_ready(const distdl_plan* p, bool backward, hipStream_t st);
// x <- H x and y; the pointer tables are uploaded.  wide: the buffers take the 16-byte box tasks.
int conv_fwd_fused(distdl_plan* p, const void* w, const void* bias, bool vec, bool wide, hipStream_t st);
// dx with H* applied, and dw, db or (*partials > 0) so many partial sums of them in `partial`, whose reduction is the caller's
int conv_bwd_fused(distdl_plan* p, const void* w, void* dw, void* db, float* partial, bool vec, hipStream_t st, int* partials);

}  // namespace distdl

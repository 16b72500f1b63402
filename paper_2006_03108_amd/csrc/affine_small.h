// Small affine layers: one launch forward, one for dx, dW and db (affine_small.hip).
#pragma once
#include <vector>

#include "gemm_mfma.h"

namespace distdl {

// Estimated time of a call (us), given the host's time for its arrays.  All of them take what gemm_split_usable says: up to eight
// segments, 31-bit byte offsets.
double affine_small_fwd_us(const std::vector<GemmBlock>& blocks, bool bf16, double arrays);
double affine_small_bwd_us(const std::vector<GemmBlock>& bx, const std::vector<GemmBlock>& bw, bool bf16, double arrays);
// Whether bf16 rows and lines are whole 4-byte words: others move value by value, which the estimates ask for
bool affine_small_words(const std::vector<GemmBlock>& blocks);
int launch_affine_small_fwd(const GemmBlock* d_blocks, const std::vector<GemmBlock>& blocks, bool bf16, hipStream_t st);
int launch_affine_small_bwd(const GemmBlock* d_bx, const std::vector<GemmBlock>& bx, const GemmBlock* d_bw, const std::vector<GemmBlock>& bw,
                            const ColsumBlock* d_cs, int n_cs, int max_f, bool bf16, hipStream_t st);

}  // namespace distdl

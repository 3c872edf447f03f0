// fused_launch.h -- launchers of the fused kernel (persistent) and of the
// small-call kernel, one of each per operand precision.
// Each is defined in its own translation unit (fused_launch.hip built with
// KVX_LAUNCH_PREC = 0, 1, 2), so the kernel's instantiations compile in
// parallel.
#pragma once

#include "kernel_mfma.h"
#include "kernel_small.h"

namespace kvx {

void launch_fused_bf16x2(bool identity, bool ds128, int grid, hipStream_t st, const FusedArgs& a);
void launch_fused_bf16(bool identity, bool ds128, int grid, hipStream_t st, const FusedArgs& a);
void launch_fused_f16(bool identity, bool ds128, int grid, hipStream_t st, const FusedArgs& a);
// row tiles of kSRows rows; grid = row_tiles * n_tiles * 2 * lt
void launch_small_bf16x2(bool identity, int grid, hipStream_t st, const FusedArgs& a);
void launch_small_bf16(bool identity, int grid, hipStream_t st, const FusedArgs& a);
void launch_small_f16(bool identity, int grid, hipStream_t st, const FusedArgs& a);

}  // namespace kvx

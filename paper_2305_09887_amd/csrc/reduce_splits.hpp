// Shape of the second stage of a split reduction (gemm_weight.hip, gemm_tf.hip).
#pragma once

namespace tma {

// Second stage of the split reduction, fixed order.  A block owns 16 groups of four
// consecutive outputs; its 16 lanes-by-split slices each add up 1/16 of the splits (all
// their 16-byte loads in flight together), then the slices are combined in slice order
// through LDS.
constexpr int kRedCols = 16;    // float4 columns per block
constexpr int kRedSlices = 16;  // split slices per block

}  // namespace tma

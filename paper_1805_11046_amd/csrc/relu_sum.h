// Optional last step of a layer-gradient convolution's epilogue (network plumbing, not from the paper): the
// gradient that leaves a residual block towards its input, res = act > 0 ? dx + other : 0, with dx the value the
// epilogue is about to store, other the gradient of the block's other branch (nullable: nothing added) and act the
// block's input, whose rectifier the gradient passes (nullable: nothing is masked).  One fp32 addition, as
// q8t_relu_bwd_sum performs it, so the fused call and the two separate ones agree bit for bit.  Both NULL: nothing
// happens.
#pragma once

struct Q8tReluSum {
    const float *other;
    const float *act;
};

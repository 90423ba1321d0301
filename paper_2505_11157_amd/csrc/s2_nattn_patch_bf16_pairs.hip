// Patch kernels of bf16 tensors, staging mode kPairs.
#include "s2_nattn_patch_impl.h"

template struct PatchKernels<bf16raw, kPairs>;

// Patch kernels of bf16 tensors whose wavefronts share patches, staging mode kHalves.
#include "s2_nattn_patch_impl.h"

template struct PatchKernels<unsigned short, kHalves, true>;

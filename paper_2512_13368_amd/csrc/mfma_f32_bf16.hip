// The small-head kernels for bf16 storage: a translation unit of its own, so that the two storage types are compiled side by side.
#define BLOSSOM_SMALL_BF16
#include "mfma_f32.hip"

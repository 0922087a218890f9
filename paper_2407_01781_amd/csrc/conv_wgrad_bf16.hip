// The matrix-unit weight gradient for bf16.
#include "conv_wgrad.h"

template hipError_t fx::launch_wgrad_tiles<__bf16>(const fx_kmap*, const void*, const void*, int, int, float*, int, bool, hipStream_t);

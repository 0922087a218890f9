// The matrix-unit weight gradient for f16.
#include "conv_wgrad.h"

template hipError_t fx::launch_wgrad_tiles<_Float16>(const fx_kmap*, const void*, const void*, int, int, float*, int, bool, hipStream_t);

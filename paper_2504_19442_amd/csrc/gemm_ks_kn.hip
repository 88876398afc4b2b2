// K-split GEMM kernels that read a B stored [K][N] in place.
#include "gemm_ks.h"

AGG_KN_INSTANCE(64, 64, 2, 8, 1)
AGG_KN_INSTANCE(64, 128, 4, 6, 1)
AGG_KN_INSTANCE(128, 128, 4, 4, 2)

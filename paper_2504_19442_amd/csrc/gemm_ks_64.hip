// K-split GEMM kernels, tiles of 64 rows.
#include "gemm_ks.h"

AGG_KS_INSTANCE(false, 64, 32, 4, 3, KS_DENSE)
AGG_KS_INSTANCE(true, 64, 64, 4, 8, KS_DENSE | KS_MOE)
AGG_KS_INSTANCE(true, 64, 128, 4, 6, KS_DENSE | KS_MOE)

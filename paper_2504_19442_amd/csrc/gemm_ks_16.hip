// K-split GEMM kernels, tiles of 16 and 32 rows.
#include "gemm_ks.h"

AGG_KS_INSTANCE(false, 16, 16, 8, 4, KS_DENSE)
AGG_KS_INSTANCE(false, 16, 32, 8, 3, KS_DENSE | KS_MOE)
AGG_KS_INSTANCE(false, 16, 64, 4, 3, KS_MOE)
AGG_KS_INSTANCE(false, 32, 32, 8, 2, KS_DENSE | KS_MOE)

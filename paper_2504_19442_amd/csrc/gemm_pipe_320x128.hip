// The grouped GEMM with 320 x 128 tiles, as one stream of K stages over a workgroup's tiles.
#include "gemm_pipe.h"

AGG_PIPE_INSTANCE(320, 128)

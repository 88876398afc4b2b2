// The grouped GEMM with 128 x 192 tiles, as one stream of K stages over a workgroup's tiles.
#include "gemm_pipe.h"

AGG_PIPE_INSTANCE(128, 192)

// Dispatch of a GEMM launch to the translation unit that holds the kernels of its tile configuration.
#include "agg_internal.h"

namespace agg {

#define AGG_DECL(BM, BN, MF) hipError_t launch_gemm_##BM##x##BN##_mf##MF(const GemmParams& p, bool grouped, int grid, hipStream_t s);
AGG_DECL(256, 224, 32) AGG_DECL(256, 256, 32) AGG_DECL(128, 256, 32) AGG_DECL(128, 128, 32)
AGG_DECL(256, 224, 16) AGG_DECL(256, 256, 16) AGG_DECL(128, 256, 16) AGG_DECL(128, 128, 16)
#undef AGG_DECL
#define AGG_DECL(BM, BN) hipError_t launch_gemm_pipe_##BM##x##BN(const GemmParams& p, bool grouped, int grid, hipStream_t s);
AGG_DECL(128, 192) AGG_DECL(128, 224) AGG_DECL(192, 192) AGG_DECL(320, 128)
#undef AGG_DECL
#define AGG_DECL(BM, BN) hipError_t launch_gemm_ks_##BM##x##BN(const GemmParams& p, bool grouped, int grid, hipStream_t s);
AGG_DECL(16, 16) AGG_DECL(16, 32) AGG_DECL(16, 64) AGG_DECL(32, 32) AGG_DECL(64, 32) AGG_DECL(64, 64) AGG_DECL(64, 128)
#undef AGG_DECL

static hipError_t launch_any(const GemmParams& p, bool grouped, int cfg, int grid, hipStream_t stream)
{
    switch (cfg) {
        case TILE_256x224: return launch_gemm_256x224_mf32(p, grouped, grid, stream);
        case TILE_256x256: return launch_gemm_256x256_mf32(p, grouped, grid, stream);
        case TILE_128x256: return launch_gemm_128x256_mf32(p, grouped, grid, stream);
        case TILE_128x128: return launch_gemm_128x128_mf32(p, grouped, grid, stream);
        case TILE_256x224 | TILE_K32: return launch_gemm_256x224_mf16(p, grouped, grid, stream);
        case TILE_256x256 | TILE_K32: return launch_gemm_256x256_mf16(p, grouped, grid, stream);
        case TILE_128x256 | TILE_K32: return launch_gemm_128x256_mf16(p, grouped, grid, stream);
        case TILE_128x128 | TILE_K32: return launch_gemm_128x128_mf16(p, grouped, grid, stream);
        case PIPE_128x192: return launch_gemm_pipe_128x192(p, grouped, grid, stream);
        case PIPE_128x224: return launch_gemm_pipe_128x224(p, grouped, grid, stream);
        case PIPE_192x192: return launch_gemm_pipe_192x192(p, grouped, grid, stream);
        case PIPE_320x128: return launch_gemm_pipe_320x128(p, grouped, grid, stream);
        case KS_16x16: return launch_gemm_ks_16x16(p, grouped, grid, stream);
        case KS_16x32: return launch_gemm_ks_16x32(p, grouped, grid, stream);
        case KS_16x64: return launch_gemm_ks_16x64(p, grouped, grid, stream);
        case KS_32x32: return launch_gemm_ks_32x32(p, grouped, grid, stream);
        case KS_64x32: return launch_gemm_ks_64x32(p, grouped, grid, stream);
        case KS_64x64: return launch_gemm_ks_64x64(p, grouped, grid, stream);
        case KS_64x128: return launch_gemm_ks_64x128(p, grouped, grid, stream);
        default: return hipErrorInvalidValue;
    }
}

hipError_t launch_gemm_kn_64x64(const GemmParams& p, int grid, hipStream_t s);
hipError_t launch_gemm_kn_64x128(const GemmParams& p, int grid, hipStream_t s);
hipError_t launch_gemm_kn_128x128(const GemmParams& p, int grid, hipStream_t s);

hipError_t launch_gemm(const GemmParams& p, int cfg, int grid, hipStream_t stream)
{
    if (p.b_kn) {
        switch (cfg) {
            case KN_64x64: return launch_gemm_kn_64x64(p, grid, stream);
            case KN_64x128: return launch_gemm_kn_64x128(p, grid, stream);
            case KN_128x128: return launch_gemm_kn_128x128(p, grid, stream);
            default: return hipErrorInvalidValue;
        }
    }
    return launch_any(p, false, cfg, grid, stream);
}

hipError_t launch_gemm_grouped(const GemmParams& p, int cfg, int grid, hipStream_t stream)
{
    return launch_any(p, true, cfg, grid, stream);
}

}  // namespace agg

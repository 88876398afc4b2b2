// B given as [K][N] (N contiguous) -> the [N][K] (K contiguous) form the GEMM kernels load whole 128-byte lines of.
#include "agg_internal.h"

namespace agg {

typedef __attribute__((__vector_size__(4 * sizeof(unsigned)))) unsigned u32x4;

// 16 bytes at any even address: B's rows start wherever its leading dimension puts them (one load instruction here, whose
// address the hardware allows to be unaligned)
__device__ inline u32x4 load8(const uint16_t* p)
{
    u32x4 v;
    __builtin_memcpy(&v, p, sizeof v);
    return v;
}

// A wave moves a 64 x 64 tile by itself: a lane
// loads 8 k-rows x 8 columns (8 lanes cover 128 bytes of a row), turns the 8 x 8 block in registers (a byte permute per
// pair of elements), and the wave swaps the 16-byte pieces through 8 KiB of LDS so that the stores, too, are 128 bytes of a
// row per 8 consecutive lanes.  Bound: memory traffic (K x N x 2 bytes read and written); eight 16-byte loads in flight
// per lane, no workgroup barrier.  Against two-byte accesses (us, kernel trace): 4096 x 3584, aligned rows (59 MB) 18.9 -> 11.3;
// 5824 x 4111, odd rows (96 MB) with the GEMM of 16 rows behind it 76.8 -> 39.3 (of which the GEMM 25 -> 9).
__global__ __launch_bounds__(256) void transpose_kn_kernel(const uint16_t* __restrict__ B_kn, long long ldb, int K, int N,
                                                                uint16_t* __restrict__ B_nk)
{
    __shared__ u32x4 tile[4][512];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int k0 = (blockIdx.y * 2 + (wave & 1)) * 64, n0 = (blockIdx.x * 2 + (wave >> 1)) * 64;
    if (k0 >= K || n0 >= N) return;
    const int kg = lane >> 3, ng = lane & 7;
    const int n = n0 + ng * 8;
    u32x4 v[8];
#pragma unroll
    for (int i = 0; i < 8; ++i) {
        const uint16_t* src = B_kn + (long long)(k0 + kg * 8 + i) * ldb + n;
        if (n + 8 <= N) {
            v[i] = load8(src);
        } else {                              // the ragged end of the row: nothing behind column N is read
            unsigned e[8];
#pragma unroll
            for (int j = 0; j < 8; ++j) e[j] = n + j < N ? src[j] : 0u;
            v[i] = u32x4{e[0] | e[1] << 16, e[2] | e[3] << 16, e[4] | e[5] << 16, e[6] | e[7] << 16};
        }
    }
    // piece (column ng * 8 + j, k-group kg): its eight k values; pieces of a column are spread over the banks by the column
#pragma unroll
    for (int j = 0; j < 8; ++j) {
        u32x4 o;
#pragma unroll
        for (int w = 0; w < 4; ++w)
            o[w] = __builtin_amdgcn_perm(v[2 * w + 1][j >> 1], v[2 * w][j >> 1], (j & 1) ? 0x07060302u : 0x05040100u);
        tile[wave][(ng * 8 + j) * 8 + (kg ^ ng)] = o;
    }
    // (the wave reads what it wrote itself: LDS keeps a wave's operations in order)
#pragma unroll
    for (int i = 0; i < 8; ++i) {
        const int c = i * 8 + kg;                          // this lane's column of step i, and k-group ng of it
        const u32x4 o = tile[wave][c * 8 + (ng ^ i)];
        if (n0 + c < N) *(u32x4*)(B_nk + (long long)(n0 + c) * K + k0 + ng * 8) = o;
    }
}

hipError_t launch_transpose_kn(const uint16_t* B_kn, long long ldb, int K, int N, uint16_t* B_nk, hipStream_t stream)
{
    if (K % 64 != 0) return hipErrorInvalidValue;              // (no GEMM of this library takes such a K)
    hipLaunchKernelGGL(transpose_kn_kernel, dim3((N + 127) / 128, (K + 127) / 128), dim3(256), 0, stream, B_kn, ldb, K, N, B_nk);
    return hipGetLastError();
}

}  // namespace agg

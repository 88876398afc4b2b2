// Rules by which the host picks grids.  Plain C++, so that they can be checked without a GPU.
#pragma once

namespace agg {

// Workgroups of a reducer launch over n_vec4 float4 whose caller leaves the size to the library.  Persistent, each walking
// many blocks of 256 (one acquire per workgroup, not per block).
//   beside_gemm: one per CU; a CU that runs a GEMM has room for one (one wave of at most 64 registers per SIMD).
//   W = 8: two per CU.  Its kernel takes 83 registers per lane, so that a CU with one of its workgroups has no room for the
//     large GEMM tiles (448 of 512) whatever the grid, and with two of them still room for the K-split ones (208).
//   Other worlds (41 to 57 registers): three per two CUs.  The reducer may have to wait for a GEMM that is launched after
//     it: half of the CUs keep room for any GEMM workgroup of this library, and three such reducers leave all CUs room for
//     the K-split ones.  With two per CU a large tile finds no room anywhere, and a GEMM that comes late runs into the
//     time limit of the reducer's wait.
// Measured with slots that are in no cache (us at 1 / 1.25 / 1.5 / 2 per CU): eight slots of 1024 x 8192 59.0 / 61.8 / 57.5 /
// 54.7, two 32.8 / 29.9 / 27.5 / 25.1, three 45.8 / 41.1 / 37.1 / 32.0, four 46.5 / 43.1 / 39.5 / 35.2, six 46.2 / 48.4 /
// 46.4 / 46.3, sixteen 95.5 / 109 / 104 / 99.1; below 60 MB of slots all within 10 %.
inline int reduce_workgroups(int W, int num_cus, long long n_vec4, bool beside_gemm)
{
    const long long need = (n_vec4 + 255) / 256;
    const long long want = beside_gemm ? num_cus : W == 8 ? num_cus * 2ll : num_cus * 3ll / 2;
    const long long n = need < want ? need : want;
    return n < 1 ? 1 : (int)n;
}

}  // namespace agg

// bat_cube.hip -- ahead-of-time kernels of the sub-cube sweep (bat_cube.hpp).
//
//  k_cube_fwd     : the sweep, graph read from the kernel arguments
//  k_cube_finish  : fixed-order double-double sum of the blocks' partials
//                   and the results
#include <hip/hip_runtime.h>

#include "bat_launch.hpp"

using bat::u32;
using bat::u64;

namespace {
// the launch's one argument, read in place: indexing a by-value copy by a
// run-time index would put it in scratch memory
__device__ __forceinline__ bat::CubeArgs *cube_args()
{
    return (bat::CubeArgs *)__builtin_amdgcn_kernarg_segment_ptr();
}
}  // namespace

__global__ void __launch_bounds__(bat::kCubeWaves *bat::kWave) k_cube_fwd(bat::CubeParams)
{
    __shared__ bat::CubeTables T;
    __shared__ bat::CubeWave W[bat::kCubeWaves];
    bat::CubeArgs *P = cube_args();
    bat::cube_kernel(P, T, W, bat::CubeDyn{P, 0u});
}

constexpr int kFinishThreads = 1024;
__global__ void __launch_bounds__(kFinishThreads) k_cube_finish(bat::CubeParams, u32)
{
    bat::CubeArgs *P = cube_args();
    const u32 n = *(const __attribute__((address_space(4))) u32 *)(P + 1);
    __shared__ double sh[kFinishThreads / 64][2];
    __shared__ u64 sc[kFinishThreads / 64];
    const u32 tid = threadIdx.x;
    if (tid == 0) bat::cube_clock(P, 1);
    double h = 0.0, l = 0.0;
    u64 c = 0;
    for (u32 k = tid; k < n; k += kFinishThreads) {
        const bat::double2_t x = P->part[k];
        bat::dd_add(h, l, x.x, x.y);
        c += P->pcount[k];
    }
    bat::wave_sum_dd(h, l);
    c = bat::wave_sum_u64(c);
    if ((tid & 63u) == 0) {
        sh[tid >> 6][0] = h;
        sh[tid >> 6][1] = l;
        sc[tid >> 6] = c;
    }
    __syncthreads();
    if (tid == 0) {
        h = l = 0.0;
        c = 0;
        for (int k = 0; k < kFinishThreads / 64; ++k) {
            bat::dd_add(h, l, sh[k][0], sh[k][1]);
            c += sc[k];
        }
        bat::cube_results(P, h, l, c);
    }
}

namespace batk {

hipError_t cube_sweep(hipStream_t st, unsigned blocks, int waves, const bat::CubeParams &P)
{
    hipLaunchKernelGGL(k_cube_fwd, dim3(blocks), dim3((unsigned)waves * bat::kWave), 0, st, P);
    return hipGetLastError();
}

hipError_t cube_finish(hipStream_t st, unsigned blocks, const bat::CubeParams &P)
{
    hipLaunchKernelGGL(k_cube_finish, dim3(1), dim3(kFinishThreads), 0, st, P, blocks);
    return hipGetLastError();
}

}  // namespace batk

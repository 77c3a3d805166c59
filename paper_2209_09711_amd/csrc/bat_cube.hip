// bat_cube.hip -- ahead-of-time kernels of the sub-cube sweep (bat_cube.hpp).
//
//  k_cube_fwd     : the sweep, graph read from the kernel arguments
//  k_cube_grad    : the same with T1_i and T0_i of every arc
//  k_cube_finish  : fixed-order double-double sum of the blocks' partials
//                   and the results
//  k_cube_grad_finish : the same of the blocks' columns, a block per arc
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
    bat::cube_kernel(P, T, W, bat::CubeDyn<bat::CubeArgs>{P, 0u});
}

__global__ void __launch_bounds__(bat::kCubeWaves *bat::kWave) __attribute__((amdgpu_waves_per_eu(2, 2)))
k_cube_grad(bat::CubeParams)
{
    __shared__ bat::CubeSumTables T;
    __shared__ bat::CubeGradTables X;
    __shared__ bat::CubeGradWave W[bat::kCubeWaves];
    __shared__ bat::double2_t cols[bat::grad_units(batk::kCubeMaxBits)][1 + 2 * batk::kCubeMaxBits];
    bat::CubeArgs *P = cube_args();
    bat::cube_grad_kernel(P, T, X, W, cols, bat::CubeDyn<bat::CubeArgs>{P, 0u});
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
#pragma unroll 4
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

// Block 0: R and the count; block 1 + a: T1, T0 and dR/dp of arc a (both R
// for an arc that is not enumerated).  The last block to end publishes.
constexpr int kGradFinishThreads = 256;
__global__ void __launch_bounds__(kGradFinishThreads) k_cube_grad_finish(bat::CubeParams, u32)
{
    bat::CubeArgs *P = cube_args();
    const u32 n = *(const __attribute__((address_space(4))) u32 *)(P + 1);
    __shared__ double sh[kGradFinishThreads / 64][4];
    __shared__ u64 sc[kGradFinishThreads / 64];
    const u32 tid = threadIdx.x, b = blockIdx.x;
    if (b == 0 && tid == 0) bat::cube_clock(P, 1);
    u32 bit = P->M;  // the arc's counter bit
    if (b > 0)
        for (u32 c = 0; c < P->M; ++c) bit = P->arc_of_bit[c] == b - 1u ? c : bit;
    const bool own = b > 0 && bit < P->M;
    const u32 c0 = own ? 1u + 2u * bit : 0u, c1 = own ? c0 + 1u : 0u;
    double h[2] = {0.0, 0.0}, l[2] = {0.0, 0.0};
    u64 cnt = 0;
    for (u32 k = tid; k < n; k += kGradFinishThreads) {
        const bat::double2_t x = P->part[(u64)c0 * n + k];
        bat::dd_add(h[0], l[0], x.x, x.y);
        if (own) {
            const bat::double2_t y = P->part[(u64)c1 * n + k];
            bat::dd_add(h[1], l[1], y.x, y.y);
        }
        if (b == 0) cnt += P->pcount[k];
    }
    bat::wave_sum_dd(h[0], l[0]);
    bat::wave_sum_dd(h[1], l[1]);
    cnt = bat::wave_sum_u64(cnt);
    if ((tid & 63u) == 0) {
        sh[tid >> 6][0] = h[0];
        sh[tid >> 6][1] = l[0];
        sh[tid >> 6][2] = h[1];
        sh[tid >> 6][3] = l[1];
        sc[tid >> 6] = cnt;
    }
    __syncthreads();
    if (tid != 0) return;
    h[0] = l[0] = h[1] = l[1] = 0.0;
    cnt = 0;
    for (int k = 0; k < kGradFinishThreads / 64; ++k) {
        bat::dd_add(h[0], l[0], sh[k][0], sh[k][1]);
        bat::dd_add(h[1], l[1], sh[k][2], sh[k][3]);
        cnt += sc[k];
    }
    const int st = P->done[1] ? -1 : 0;
    if (b == 0) {
        bat::cube_store(P, h[0], l[0], cnt, st);
    } else {
        if (!own) {
            h[1] = h[0];
            l[1] = l[0];
        }
        if (P->res) {
            double *r = P->res + 2 + 4 * (b - 1u);
            r[0] = h[0];
            r[1] = l[0];
            r[2] = h[1];
            r[3] = l[1];
        }
        const double nan = __builtin_nan("");
        if (P->dRdp) P->dRdp[b - 1u] = st ? nan : (h[1] - h[0]) + (l[1] - l[0]);
        if (P->T1) P->T1[b - 1u] = st ? nan : h[1] + l[1];
        if (P->T0) P->T0[b - 1u] = st ? nan : h[0] + l[0];
    }
    __threadfence_system();
    if (atomicAdd(P->done, 1u) == gridDim.x - 1u) bat::cube_publish(P);
}

namespace batk {

hipError_t cube_grad(hipStream_t st, unsigned blocks, int waves, const bat::CubeParams &P)
{
    hipLaunchKernelGGL(k_cube_grad, dim3(blocks), dim3((unsigned)waves * bat::kWave), 0, st, P);
    return hipGetLastError();
}

hipError_t cube_grad_finish(hipStream_t st, unsigned blocks, const bat::CubeParams &P)
{
    hipLaunchKernelGGL(k_cube_grad_finish, dim3(1u + P.m), dim3(kGradFinishThreads), 0, st, P, blocks);
    return hipGetLastError();
}

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

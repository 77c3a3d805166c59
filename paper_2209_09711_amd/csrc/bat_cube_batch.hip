// bat_cube_batch.hip -- sub-cube sweeps (bat_cube.hpp) of many graphs, each
// with several probability vectors, in one launch.
//
//  k_cube_batch<PW>     : the sweeps; a block takes a run of one entry's work
//                         items (entry: a graph with up to PW vectors)
//  k_cube_batch_finish  : fixed-order double-double sums of the blocks'
//                         partials, written to the host, a block per entry
//
// A word's verdicts are the same for every probability vector, so an entry's
// closures run once, with 64 words in the 64 lanes; its sums then run
// transposed: the words with anything in them are listed, and a lane forms,
// for one probability vector, the sum over half of a word (64 / PW lanes per
// vector, so 32 / PW words at a time).  The tables are [index][PW], read
// without bank conflicts by neighbouring lanes.
//
// What bounds it: with 32 vectors the LDS reads of the sums (two byte sums
// and a prefix factor per word and vector) and the ends of blocks (byte
// tables leave room for one block of 16 wavefronts per CU), with few the
// closures.  256 graphs of 16 to 28 arcs: 0.67 ms with 3 vectors, 0.95 ms
// with 16, 1.5 ms with 32 (the words' values read from LDS by every lane and
// one word at a time: 2.1 ms; nibble sums, four reads, in blocks of 8
// wavefronts, two per CU: 2.2 ms; every n-th item to a wavefront instead of
// a counter: 2.5 ms).
#include <hip/hip_runtime.h>

#include "bat_launch.hpp"

using bat::kCubeGroup;
using bat::kWave;
using bat::u32;
using bat::u64;
using bat::BatchCube;
using bat::BatchCubes;

namespace bat {

typedef const __attribute__((address_space(4))) BatchCube BatchArgs;
__device__ __forceinline__ double cube_p(BatchArgs *P, u32 a) { return P->p[a]; }
__device__ __forceinline__ const __attribute__((address_space(4))) u32 *cube_steps(BatchArgs *P)
{
    return (const __attribute__((address_space(4))) u32 *)P->step;
}

__device__ __forceinline__ u32 cube_window(BatchArgs *P, u32 base)
{
    const u32 lo = P->win_lo, last = P->win_last;
    u32 m = ~0u;
    if (lo > base) m = lo - base >= 32u ? 0u : ~0u << (lo - base);
    if (last < base) m = 0u;
    else if (last - base < 31u) m &= (2u << (last - base)) - 1u;
    return m;
}

template <int PW>
struct BatchTables {
    double tb[256][PW];  // word 0: bits 0..2, by byte
    double a4[4][PW];    // bits 3..4
    double q5[32][PW];   // word 1 (with one level: 1)
    double n1[16][PW];   // bits 0..1, by nibble
    double c1[8][PW];    // bits 2..4
    double ql[kWave][PW];  // lane bits
    double pr[32][PW];
};

constexpr int kBatchWaves = batk::kCubeBatchWaves;
constexpr int kBatchQueue = 512;
constexpr int kBatchPlaces = 64;  // sums of a block
constexpr int kBatchWords = 4;    // words in flight with 32 vectors
struct BatchWave {
    unsigned short queue[kBatchQueue];
    u32 V[kWave], x[kWave];
};

template <int PW>
__device__ __forceinline__ double batch_q(const BatchTables<PW> &T, u32 M, u32 cb, u32 x, u32 p)
{
    if (cb >= M) return x ? 0.0 : 1.0;  // a bit past the last arc: never set
    const double q = T.pr[cb][p];
    return x ? q : 1.0 - q;
}

template <int PW>
__device__ __forceinline__ void batch_tables(BatchArgs *P, BatchTables<PW> &T)
{
    const u32 tid = threadIdx.x, nt = blockDim.x, M = P->M, levels = P->levels;
    const u32 p = tid % PW, row = tid / PW, rows = nt / PW;  // (nt is a multiple of PW)
    for (u32 cb = row; cb < M; cb += rows) T.pr[cb][p] = p < P->n_p ? P->p[(u64)p * P->m + P->arc_of_bit[cb]] : 0.0;
    __syncthreads();
    {
        double q[8];
#pragma unroll
        for (u32 k = 0; k < 8; ++k)
            q[k] = batch_q(T, M, 0, k & 1u, p) * batch_q(T, M, 1, (k >> 1) & 1u, p) * batch_q(T, M, 2, k >> 2, p);
        for (u32 y = row; y < 256u; y += rows) {
            double s = 0.0;
#pragma unroll
            for (u32 k = 0; k < 8; ++k) s += ((y >> k) & 1u) ? q[k] : 0.0;
            T.tb[y][p] = s;
        }
    }
    for (u32 h = row; h < 4u; h += rows) T.a4[h][p] = batch_q(T, M, 3, h & 1u, p) * batch_q(T, M, 4, h >> 1, p);
    for (u32 j = row; j < 32u; j += rows) {
        double q = 1.0;
        for (u32 k = 0; levels > 1u && k < 5u; ++k) q *= batch_q(T, M, 5 + k, (j >> k) & 1u, p);
        T.q5[j][p] = q;
    }
    if (levels > 1u) {
        for (u32 y = row; y < 16u; y += rows) {
            double s = 0.0;
#pragma unroll
            for (u32 k = 0; k < 4; ++k)
                s += ((y >> k) & 1u) ? batch_q(T, M, 5, k & 1u, p) * batch_q(T, M, 6, k >> 1, p) : 0.0;
            T.n1[y][p] = s;
        }
        for (u32 h = row; h < 8u; h += rows)
            T.c1[h][p] = batch_q(T, M, 7, h & 1u, p) * batch_q(T, M, 8, (h >> 1) & 1u, p) * batch_q(T, M, 9, h >> 2, p);
    }
    for (u32 j = row; j < (u32)kWave; j += rows) {
        double q = 1.0;
        for (u32 b = 0; b < P->lane_bits; ++b) q *= batch_q(T, M, kCubeGroup * levels + b, (j >> b) & 1u, p);
        T.ql[j][p] = q;
    }
    __syncthreads();
}

template <int PW>
struct BatchSweep {
    BatchArgs *P;
    const BatchTables<PW> &T;
    BatchWave &W;
    CubeDyn<BatchArgs> clo;
    u32 lane;
    u64 cnt;
    double acc;  // of the current item, without the item's own bits
    // 32 vectors and two levels: sum under the prefix `own` of word 1
    double under;
    u32 own;

    // List the words V that hold anything, in lane order.
    __device__ __forceinline__ u32 list(u32 V, u32 x)
    {
        const u64 nz = __ballot(V != 0u);
        const u32 at = __builtin_amdgcn_mbcnt_hi((u32)(nz >> 32), __builtin_amdgcn_mbcnt_lo((u32)nz, 0u));
        if (V) {
            W.V[at] = V;
            W.x[at] = x;
        }
        wave_lds_sync();
        return (u32)__popcll(nz);
    }

    // Half of word v for the lane's vector.
    __device__ __forceinline__ double half_word(u32 v, double a0, double a1, u32 p) const
    {
        return __builtin_fma(a1, T.tb[(v >> 8) & 255u][p], a0 * T.tb[v & 255u][p]);
    }

    // What is under the prefix so far goes up to it.
    __device__ __forceinline__ void flush()
    {
        if constexpr (PW == 32) {
            acc = __builtin_fma(T.ql[own][lane % PW], under, acc);
            under = 0.0;
        }
    }

    // Words of single vectors, each under the prefix x: lane << 5 | index in
    // word 1 (TWO levels; else that index has no meaning).
    template <bool TWO>
    __device__ __forceinline__ void words(u32 V, u32 x)
    {
        constexpr u32 step = 32 / PW;
        cnt += (u64)__popc(V);
        if constexpr (PW == 32) {
            // one word at a time, the same for all lanes: it stays scalar, and
            // a prefix's factor is read once for all words under it
            const u32 p = lane % PW, half = lane / PW;
            const double a0 = T.a4[2 * half][p], a1 = T.a4[2 * half + 1][p];
            for (u64 nz = __ballot(V != 0u); nz != 0ull;) {
                // kBatchWords at a time (the last ones perhaps none), so that
                // their LDS reads overlap: 1.9 ms one by one, 1.5 ms by 4,
                // 1.57 ms by 8, which spill
                u32 v[kBatchWords], y[kBatchWords];
                int i = 0;
#pragma unroll
                for (int k = 0; k < kBatchWords; ++k) {
                    i = nz ? __builtin_ctzll(nz) : i;
                    v[k] = nz ? (u32)__builtin_amdgcn_readlane((int)V, i) : 0u;
                    y[k] = (u32)__builtin_amdgcn_readlane((int)x, i);
                    nz &= nz - 1ull;
                }
                double F[kBatchWords], q[kBatchWords];
#pragma unroll
                for (int k = 0; k < kBatchWords; ++k) {
                    F[k] = half_word(v[k] >> (16 * half), a0, a1, p);
                    q[k] = TWO ? T.q5[y[k] & 31u][p] : T.ql[y[k] >> 5][p];
                }
#pragma unroll
                for (int k = 0; k < kBatchWords; ++k) {
                    if constexpr (TWO) {
                        if (y[k] >> 5 != own) {
                            flush();
                            own = y[k] >> 5;
                        }
                        under = __builtin_fma(q[k], F[k], under);
                    } else {
                        acc = __builtin_fma(q[k], F[k], acc);
                    }
                }
            }
            return;
        }
        const u32 n = list(V, x), p = lane % PW, half = (lane / PW) & 1u, first = lane / (2 * PW);
        const double a0 = T.a4[2 * half][p], a1 = T.a4[2 * half + 1][p];
#pragma unroll 4
        for (u32 i = first; i < n + first; i += step) {
            const bool on = i < n;
            const u32 k = on ? i : n - 1u, v = W.V[k] >> (16 * half), y = W.x[k];
            const double F = half_word(v, a0, a1, p);
            double q = T.ql[y >> 5][p];
            if (TWO) q *= T.q5[y & 31u][p];
            acc = __builtin_fma(on ? q : 0.0, F, acc);
        }
        wave_lds_sync();
    }

    // The cubes S of the lanes' words of level 1.
    __device__ __forceinline__ void cubes(u32 S)
    {
        constexpr u32 step = 32 / PW;
        cnt += (u64)__popc(S) << kCubeGroup;
        const u32 n = list(S, lane), p = lane % PW, half = (lane / PW) & 1u, first = lane / (2 * PW);
#pragma unroll 2
        for (u32 i = first; i < n + first; i += step) {
            const bool on = i < n;
            const u32 k = on ? i : n - 1u, v = W.V[k] >> (16 * half);
            double F = 0.0;
#pragma unroll
            for (u32 h = 0; h < 4; ++h) F = __builtin_fma(T.c1[4 * half + h][p], T.n1[(v >> (4 * h)) & 15u][p], F);
            acc = __builtin_fma(on ? T.ql[W.x[k]][p] : 0.0, F, acc);
        }
        wave_lds_sync();
    }

    // The sum of a work item for the lane's vector (over all lanes of it),
    // added to h + l.
    __device__ __forceinline__ void item(u64 block, double &h, double &l)
    {
        const u32 levels = P->levels, lane_bits = P->lane_bits, M = P->M, rb = kCubeGroup * levels + lane_bits;
        clo.item(block);
        const bool live = (lane >> lane_bits) == 0u;
        acc = under = 0.0;
        own = 0u;
        if (levels == 1u) {
            u32 V = clo.close(0u, lane << kCubeGroup, live);
            if (M < 5u) V &= (1u << (1u << M)) - 1u;  // bits past the last arc
            words<false>(V & cube_window(P, ((u32)block << rb) | lane << kCubeGroup), lane << 5);
        } else {
            const u32 rel = lane << (2 * kCubeGroup);
            const u32 up = clo.close(1u, rel, live);
            if (__ballot(up != 0u) == 0ull) return;
            const u32 down = clo.close(2u, rel, live && up != 0u);
            cubes(down);
            u32 total;
            const u32 U = up & ~down, e = wave_excl_popc(U, total);
            for (u32 w0 = 0; w0 < total; w0 += kBatchQueue) {
                cube_enqueue<kBatchQueue>(W.queue, U, e, w0, lane);
                const u32 end = min(total, w0 + (u32)kBatchQueue);
                for (u32 r = w0; r < end; r += (u32)kWave) {
                    const bool on = r + lane < end;
                    const u32 x = W.queue[(on ? r + lane : end - 1u) - w0];
                    words<true>(clo.close(0u, x << kCubeGroup, on), x);
                }
            }
            flush();
        }
        double s, e;
        two_sum(acc, shfl_xor_d(acc, PW), s, e);
#pragma unroll
        for (int off = 2 * PW; off < kWave; off <<= 1) {
            const double y = shfl_xor_d(s, off), z = shfl_xor_d(e, off);
            double t;
            two_sum(s, y, s, t);
            e = (e + z) + t;
        }
        double q = 1.0;
        const u32 p = lane % PW;
#pragma unroll 4
        for (u32 b = rb; b < M; ++b) {
            const double x = T.pr[b][p];
            q *= (block >> (b - rb)) & 1u ? x : 1.0 - x;
        }
        dd_add(h, l, q * s, q * e);
    }
};

// The wavefronts of a block take its work items from a counter, some in a
// run where they are many; a run's sums have a place of their own and are
// added in a fixed order.
template <int PW>
__device__ __forceinline__ void batch_block(BatchArgs *P, const BatchCubes &L, u32 blk)
{
    __shared__ BatchTables<PW> T;
    __shared__ BatchWave Ws[kBatchWaves];
    __shared__ double2_t su[kBatchPlaces][PW];
    __shared__ u64 sc[kBatchWaves];
    __shared__ u32 next;
    if (threadIdx.x == 0) next = 0u;
    batch_tables<PW>(P, T);
    const u32 lane = threadIdx.x & (kWave - 1);
    const u32 wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    BatchSweep<PW> S{P, T, Ws[wave], CubeDyn<BatchArgs>{P, 0u}, lane, 0ull, 0.0, 0.0, 0u};
    const u64 first = (u64)(blk - P->first_block) * P->units;
    const u32 n = (u32)min((u64)P->units, P->n_items - first), run = (n + kBatchPlaces - 1u) / kBatchPlaces;
    for (;;) {
        __builtin_amdgcn_wave_barrier();  // (see cube_kernel)
        const u32 k = __builtin_amdgcn_readfirstlane(atomicAdd(&next, 1u)) / kWave;
        if (k * run >= n) break;
        double h = 0.0, l = 0.0;
        for (u32 i = k * run; i < min(n, (k + 1u) * run); ++i)
            S.item(((first + i) * P->item_mul) & P->item_mask, h, l);
        if (lane < (u32)PW) su[k][lane] = {h, l};
    }
    const u64 c = wave_sum_u64(S.cnt);
    if (lane == 0) sc[wave] = c;
    __syncthreads();  // the tables' place takes the sums of the places
    static_assert(sizeof(T) >= sizeof(double2_t) * kBatchWaves * kWave / 2 && PW * kBatchPlaces >= 64, "");
    double2_t *red = (double2_t *)&T;
    constexpr u32 rows = 16;
    const u32 p = threadIdx.x % PW, row = threadIdx.x / PW;
    double h = 0.0, l = 0.0;
    if (row < rows) {
        for (u32 k = row; k * run < n; k += rows) dd_add(h, l, su[k][p].x, su[k][p].y);
        red[threadIdx.x] = {h, l};
    }
    for (u32 s = rows / 2; s; s >>= 1) {
        __syncthreads();
        if (row < s) {
            dd_add(h, l, red[threadIdx.x + s * PW].x, red[threadIdx.x + s * PW].y);
            red[threadIdx.x] = {h, l};
        }
    }
    if (row == 0) L.part[(u64)blk * PW + p] = {h, l};
    if (threadIdx.x == 0) {
        u64 n = 0;
        for (int w = 0; w < kBatchWaves; ++w) n += sc[w];
        L.pcount[blk] = n;
    }
}

// One vector per entry: the lanes that hold the words sum them too.
__device__ __forceinline__ void batch_block_1(BatchArgs *P, const BatchCubes &L, u32 blk)
{
    __shared__ CubeTables T;
    __shared__ CubeWave Ws[kCubeWaves];
    __shared__ double2_t su[kCubeWaves];
    __shared__ u64 sc[kCubeWaves];
    cube_tables(P, T);
    const u32 lane = threadIdx.x & (kWave - 1);
    const u32 wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    CubeSweep<CubeDyn<BatchArgs>, BatchArgs> S{P, T, Ws[wave], CubeDyn<BatchArgs>{P, 0u}, lane, 0.0, 0.0, 0ull};
    const u64 first = (u64)(blk - P->first_block) * P->units;
    for (u32 k = wave; k < P->units && first + k < P->n_items; k += kCubeWaves)
        S.item(((first + k) * P->item_mul) & P->item_mask, 0u);
    wave_sum_dd(S.hi, S.lo);
    const u64 c = wave_sum_u64(S.cnt);
    if (lane == 0) {
        su[wave] = {S.hi, S.lo};
        sc[wave] = c;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        double h = 0.0, l = 0.0;
        u64 n = 0;
        for (int w = 0; w < kCubeWaves; ++w) {
            dd_add(h, l, su[w].x, su[w].y);
            n += sc[w];
        }
        L.part[blk] = {h, l};
        L.pcount[blk] = n;
    }
}

}  // namespace bat

template <int PW>
__global__ void __launch_bounds__(PW == 1 ? bat::kCubeWaves *kWave : bat::kBatchWaves *kWave) k_cube_batch(BatchCubes L)
{
    const u32 blk = L.block0 + blockIdx.x;
    if (blk == 0 && threadIdx.x == 0) {
        L.diag[0] = wall_clock64();
        *L.done = 0u;
    }
    const u32 e = ((const __attribute__((address_space(4))) u32 *)L.block_entry)[blk];
    bat::BatchArgs *P = (bat::BatchArgs *)(L.entries + (u64)e * L.stride);
    if constexpr (PW == 1) bat::batch_block_1(P, L, blk);
    else bat::batch_block<PW>(P, L, blk);
}

constexpr int kBatchFinish = 256;
__global__ void __launch_bounds__(kBatchFinish) k_cube_batch_finish(BatchCubes L, u32 pw)
{
    __shared__ bat::double2_t sh[kBatchFinish];
    __shared__ u64 sc[kBatchFinish / kWave];
    const u32 tid = threadIdx.x, e = blockIdx.x, p = tid % pw, row = tid / pw, rows = kBatchFinish / pw;
    if (e == 0 && tid == 0) L.diag[1] = wall_clock64();
    const BatchCube &E = *(const BatchCube *)(L.entries + (u64)e * L.stride);
    double h = 0.0, l = 0.0;
    u64 n = 0;
    for (u32 b = row; b < E.n_blocks; b += rows) {
        const bat::double2_t x = L.part[(u64)(E.first_block + b) * pw + p];
        bat::dd_add(h, l, x.x, x.y);
    }
    for (u32 b = tid; b < E.n_blocks; b += kBatchFinish) n += L.pcount[E.first_block + b];
    // a tree over the rows (one thread after them all took 8 us here)
    sh[tid] = {h, l};
    n = bat::wave_sum_u64(n);
    if ((tid & (kWave - 1)) == 0) sc[tid / kWave] = n;
    for (u32 r = rows / 2; r; r >>= 1) {
        __syncthreads();
        if (row < r) {
            bat::dd_add(h, l, sh[tid + r * pw].x, sh[tid + r * pw].y);
            sh[tid] = {h, l};
        }
    }
    if (tid < pw) L.sums[(u64)e * pw + tid] = {h, l};
    __syncthreads();
    if (tid == 0) {
        n = 0;
        for (int w = 0; w < kBatchFinish / kWave; ++w) n += sc[w];
        L.counts[e] = n << (E.m - E.M);
    }
    __threadfence_system();
    __syncthreads();
    if (tid == 0 && atomicAdd(L.done, 1u) == gridDim.x - 1u) {
        L.diag[2] = wall_clock64();
        __hip_atomic_store(L.diag + 3, L.seq, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_SYSTEM);
    }
}

namespace batk {

hipError_t cube_batch(hipStream_t st, unsigned blocks, int pw, const BatchCubes &L)
{
    const dim3 g(blocks), b((unsigned)(kWave * (pw == 1 ? bat::kCubeWaves : bat::kBatchWaves)));
    switch (pw) {
    case 1: hipLaunchKernelGGL(k_cube_batch<1>, g, b, 0, st, L); break;
    case 4: hipLaunchKernelGGL(k_cube_batch<4>, g, b, 0, st, L); break;
    case 8: hipLaunchKernelGGL(k_cube_batch<8>, g, b, 0, st, L); break;
    case 16: hipLaunchKernelGGL(k_cube_batch<16>, g, b, 0, st, L); break;
    default: hipLaunchKernelGGL(k_cube_batch<32>, g, b, 0, st, L); break;
    }
    return hipGetLastError();
}

hipError_t cube_batch_finish(hipStream_t st, unsigned entries, int pw, const BatchCubes &L)
{
    hipLaunchKernelGGL(k_cube_batch_finish, dim3(entries), dim3(kBatchFinish), 0, st, L, (u32)pw);
    return hipGetLastError();
}

}  // namespace batk

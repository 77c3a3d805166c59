// bat_ms_cube.hpp -- device code of the bit-sliced multi-state sweep by
// cubes (demands 1 to 3, whole spaces).
//
// Included as text after bat_device.hpp and bat_cube.hpp by the kernels
// compiled at run time; includes no header.
//
// The slots (slot 0 least significant) are split into
//     prefix | word 1: slots KW .. KW+KW1-1 | word 0: slots 0 .. KW-1
// with words of at most 32 vectors.  A lane holds a prefix.  Its word 1
// stands for B1 cubes, each free in the slots of word 0; the maximum flow
// never falls when a capacity rises, so the flow test with the free slots at
// their least capacities gives the cubes that meet the demand for certain
// (added whole), with them at their greatest those that can.  The undecided
// ones are queued and taken 64 at a time, one per lane, as word 0's.
//
// The test is the one described at ms_bits_kernel (max-flow min-cut), with
// its closures by removal of the nodes (see bat_cube_plan.hpp), exact in one
// pass.  Slots are ordered by distance from the nearer terminal, the farthest
// lowest: on 3^18 vectors at demand 2 one word 0 in 40 is left to test.
//
// What bounds it: the issue of the closures, up to one per slot and word, and
// on small spaces one wavefront's chain of them.  Kernel times against every
// word tested by itself: 3^18 vectors at demand 1, 2, 3: 25 us, 40 us, 0.48 ms
// against 137 us, 0.76 ms, 3.1 ms.
//
// G (compiled for one graph and one set of states): M, D, KW, KW1, B0, FULL0,
// B1, FULL1, LOOP (more items than wavefronts), SLOTS, RESULT (a slot, or
// 255: never connected), per slot SIG, OFF, C1 / CE1 / CE12 (bit k: state k
// has capacity >= 1 / exactly 1 / 1 or 2), per word slot P1 / PE1 / PE12 (its
// word's vectors whose state has such a capacity), per slot of word 0 LO / HI
// (the same three, bits 0..2, of its least and greatest capacity), steps(r).

namespace bat {

constexpr int kMsCubeWaves = 4;  // wavefronts of a block
constexpr int kMsCubeQueue = 512;

struct MsCubeParams {
    u64 n_prefix, n_items;  // 64 prefixes an item
    u64 n_waves;            // wavefronts, at most the items: each takes every n_waves-th
    const double *tb;       // [2][4][256]: word 0, word 1 (times word 0's probability)
    const double *q1;       // [32] word 1's vectors
    const u32 *m1;          // [3][32] capacity bits of word 1's slots, per vector
    const double *w;        // probability of (slot, state)
    double *part;           // [n_waves][2]
    u64 *pcount;            // [n_waves]
    u64 *diag;              // [0]: the device clock at the start
};

struct MsCubeWave {
    unsigned short queue[kMsCubeQueue];
    u32 bits[3][kWave];  // the lanes' prefixes: capacity >= 1, exactly 1, 1 or 2, by slot
    double q[kWave];
};
struct MsCubeLds {
    double tb[2][4][256];
    double q1[32];
    u32 m1[3][32];
    MsCubeWave wave[kMsCubeWaves];
};

// s-t connected over the slots' masks without slots a and b.
template <class G>
__device__ __forceinline__ u32 ms_joined(const u32 (&W)[G::M], int a)
{
    if constexpr (G::RESULT == 255u) return 0u;
    u32 r[G::SLOTS];
#pragma unroll
    for (int j = 0; j < G::M; ++j) r[j] = j == a ? 0u : W[j];
    G::steps(r);
    return r[G::RESULT];
}

// The vectors of `full` whose maximum flow is at least D.  LEVEL: whose word
// varies; bits: the capacities of the slots outside it, by slot.
template <class G, int LEVEL>
__device__ __forceinline__ u32 ms_meets(const u32 (&bits)[3], u32 full)
{
    auto mask = [&](int j, int kind) -> u32 {
        const bool word = LEVEL == 0 ? j < (int)G::KW : j >= (int)G::KW && j < (int)(G::KW + G::KW1);
        if (word) return kind == 0 ? G::P1[j] : kind == 1 ? G::PE1[j] : G::PE12[j];
        return (u32)__builtin_amdgcn_sbfe((int)bits[kind], j, 1);
    };
    u32 W[G::M];
#pragma unroll
    for (int j = 0; j < G::M; ++j) {
        W[j] = mask(j, 0);
        asm volatile("" : "+v"(W[j]));
    }
    u32 V = ms_joined<G>(W, -1) & full;
    if constexpr (G::D >= 2) {
#pragma unroll
        for (int j = 0; j < G::M; ++j) {
            if ((G::D == 2 ? G::CE1[j] : G::CE12[j]) == 0u) continue;
            const u32 need = V & mask(j, G::D == 2 ? 1 : 2);
            if (__ballot(need != 0u) != 0ull) V &= ~need | ms_joined<G>(W, j);
        }
    }
    if constexpr (G::D == 3) {
        auto unit = [&](u32 j) -> u32 {
            const bool word = LEVEL == 0 ? j < G::KW : j >= G::KW && j < G::KW + G::KW1;
            return word ? G::PE1[j] : 0u - ((bits[1] >> j) & 1u);
        };
        for (u32 m1 = G::UPAIR; m1 != 0u; m1 &= m1 - 1u) {
            const u32 j1 = (u32)__builtin_ctz(m1), u1 = unit(j1);
            if (__ballot((V & u1) != 0u) == 0ull) continue;
            for (u32 m2 = m1 & (m1 - 1u); m2 != 0u; m2 &= m2 - 1u) {
                const u32 j2 = (u32)__builtin_ctz(m2), need = V & u1 & unit(j2);
                if (__ballot(need != 0u) == 0ull) continue;
                u32 Wp[G::M];
#pragma unroll
                for (int j = 0; j < G::M; ++j) {
                    Wp[j] = ((u32)j == j1 || (u32)j == j2) ? 0u : W[j];
                    asm volatile("" : "+v"(Wp[j]));
                }
                V &= ~need | ms_joined<G>(Wp, -1);
            }
        }
    }
    return V;
}

template <class G>
__device__ void ms_cube_kernel(const MsCubeParams &P, MsCubeLds &L)
{
    const u32 tid = threadIdx.x, lane = tid & (kWave - 1), wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    if (blockIdx.x == 0 && tid == 0) P.diag[0] = wall_clock64();
    for (u32 i = tid; i < 2048u; i += blockDim.x) L.tb[i >> 10][(i >> 8) & 3u][i & 255u] = P.tb[i];
    if (tid < 32u) L.q1[tid] = P.q1[tid];
    if (tid < 96u) L.m1[tid >> 5][tid & 31u] = P.m1[tid];
    __syncthreads();
    MsCubeWave &W = L.wave[wave];
    u32 low[3] = {0u, 0u, 0u}, high[3] = {0u, 0u, 0u};  // word 0's slots at their least, greatest
#pragma unroll
    for (int j = 0; j < (int)G::KW; ++j)
#pragma unroll
        for (int k = 0; k < 3; ++k) {
            low[k] |= ((G::LO[j] >> k) & 1u) << j;
            high[k] |= ((G::HI[j] >> k) & 1u) << j;
        }
    const u64 first = (u64)blockIdx.x * kMsCubeWaves + wave;
    if (first >= P.n_waves) return;
    double hi = 0.0, lo = 0.0;
    u64 cnt = 0;
    auto add = [&](int level, double p, u32 V) {
        if (__ballot(V != 0u) == 0ull) return;
        const double(&tb)[4][256] = L.tb[level];
        const double F = ((tb[0][V & 255u] + tb[1][(V >> 8) & 255u]) + tb[2][(V >> 16) & 255u]) + tb[3][V >> 24];
        double s, e;
        two_sum(hi, p * F, s, e);
        hi = s;
        lo += e;
    };
    auto take = [&](u64 item) {
        // neighbouring prefixes lie in different items
        const u64 prefix = item + (u64)lane * P.n_items;
        const bool live = prefix < P.n_prefix;
        u64 r = prefix;
        u32 up[3] = {0u, 0u, 0u};
        double q = 1.0, qe = 0.0;
#pragma unroll
        for (int j = (int)(G::KW + G::KW1); j < (int)G::M; ++j) {
            const u32 x = (u32)(r % G::SIG[j]);
            r /= G::SIG[j];
            up[0] |= ((G::C1[j] >> x) & 1u) << j;
            up[1] |= ((G::CE1[j] >> x) & 1u) << j;
            up[2] |= ((G::CE12[j] >> x) & 1u) << j;
            dd_mul(q, qe, P.w[G::OFF[j] + x]);
        }
        q += qe;
        const u32 most[3] = {up[0] | high[0], up[1] | high[1], up[2] | high[2]};
        const u32 can = ms_meets<G, 1>(most, live ? G::FULL1 : 0u);
        if (__ballot(can != 0u) != 0ull) {
            const u32 least[3] = {up[0] | low[0], up[1] | low[1], up[2] | low[2]};
            const u32 sure = ms_meets<G, 1>(least, can), U = can & ~sure;
            cnt += (u64)__popc(sure) * G::B0;
            add(1, q, sure);
            u32 total;
            const u32 e = wave_excl_popc(U, total);
#pragma unroll
            for (int k = 0; k < 3; ++k) W.bits[k][lane] = up[k];
            W.q[lane] = q;
            for (u32 w0 = 0; w0 < total; w0 += kMsCubeQueue) {
                cube_enqueue<kMsCubeQueue>(W.queue, U, e, w0, lane);
                const u32 end = min(total, w0 + (u32)kMsCubeQueue);
                for (u32 i = w0; i < end; i += (u32)kWave) {
                    const bool on = i + lane < end;
                    const u32 x = W.queue[(on ? i + lane : end - 1u) - w0], own = x >> 5, y = x & 31u;
                    const u32 bits[3] = {W.bits[0][own] | L.m1[0][y], W.bits[1][own] | L.m1[1][y],
                                         W.bits[2][own] | L.m1[2][y]};
                    const u32 V = ms_meets<G, 0>(bits, on ? G::FULL0 : 0u);
                    cnt += (u64)__popc(V);
                    add(0, W.q[own] * L.q1[y], V);
                }
                wave_lds_sync();
            }
        }
    };
    // (the loop costs the small spaces, whose items fit the wavefronts, 10% of
    // their kernel time)
    if constexpr (G::LOOP != 0u) {
        for (u64 item = first; item < P.n_items; item += P.n_waves) take(item);
    } else {
        take(first);
    }
    wave_sum_dd(hi, lo);
    const u64 c = wave_sum_u64(cnt);
    if (lane == 0) {
        P.part[2 * first] = hi;
        P.part[2 * first + 1] = lo;
        P.pcount[first] = c;
    }
}

}  // namespace bat

// bat_ms.hip -- multi-state arcs: the BAT over a mixed-radix solution space
// (Section 4.1: arcs with sigma_i states give prod_i sigma_i vectors) with a
// demand-level flow test per state vector.
//
// What is computed: arc i is in state k in 0..sigma_i-1 with probability
// w_i(k), and carries at most cap_i(k) units (either way for an undirected
// arc).  A vector X meets demand d when the maximum s-t flow is at least d;
// R_d = sum of prod_i w_i(x_i) over those X, and count = their number.  The
// paper defines reliability for binary arcs only (Eq. 1) and names the
// multi-state problem as the next one to solve; with two states of capacity
// 0 and 1 and d = 1 this is exactly Eq. 1.
//
// Mapping onto the machine.  The kernel sees the arcs in slots; slot 0 is
// the fastest-changing coordinate of the mixed-radix index.  The vectors are
// decided as cubes: a node (K, states of the slots from K on) stands for all
// states of the slots below K.  The maximum flow never falls when a capacity
// rises, so two tests bound the whole cube: with the free slots at their
// least capacities a flow of d settles it (met: its weight is added whole),
// with them at their greatest one short of d does (not met); else the cube
// splits into one node per state of slot K-1.  A flow found with the least
// capacities stays feasible with the greatest, so the second test goes on
// from the first.  A child whose slot has the least capacity has failed its
// first test already (its parent's), one with the greatest has met its
// second.  An undecided cube of slot 0 alone is not split (unless the range
// ends inside it): as a function of one arc's capacity c the maximum flow is
// min(A + c, B), the smaller of the least cut through the arc and the least
// one that avoids it, so where it is short of d by x at the least capacity
// and meets d at the greatest, it meets d from x units more on.  (Split into
// its states, one test each: 3^15 vectors at demand 4 0.35 ms a call, now
// 0.29; 16^7 at demand 14 45 ms, now 6.2, against 8.3 ms with a run of
// vectors per lane.)
//
// A wavefront takes 64 cubes of the `L` lowest slots, one per lane, and from
// there its lanes share one stack of nodes in LDS: a lane whose node is
// decided takes the next one, so that no lane waits for another's deep cube
// (lanes run in lockstep: which lane takes which node, and with it the sum,
// is fixed).  A lane that finds no more room on the stack keeps its children
// to itself and goes through them in order, which needs no memory.  (With
// room for all 64 lanes' children asked of it, arcs of more than 8 states
// never shared any: 10^8 vectors at demand 9 30 ms, 3.5 with what room there
// is.)
//
// The flow test pushes augmenting paths found on node bitmasks: a search
// sweeps the slots in order, adding the far end of every arc with residual
// capacity out of the reached set, until t is reached or a sweep adds
// nothing (no augmenting path: the flow is maximal); the arcs that first
// reached each node form a tree rooted at s, whose path to t reverse sweeps
// collect; the smaller of its bottleneck and the missing demand is pushed,
// so a test takes at most d pushes.  A loop step is one sweep out and back
// and, where it reaches t, one push.
//
// The host pads the slots past the last arc up to MM with one-state self-
// loops at s (capacity 0, probability 1), which change nothing, so every
// sweep is straight-line code over MM slots with no test of the arc count,
// and orders a whole space's slots by distance from the nearer terminal, the
// farthest lowest: the arcs that rarely matter are free in the cubes.
//
// What bounds it: the sweeps' instructions, some 30 steps of 1100 per
// wavefront at half its lanes on 3^15 vectors and demand 4: 0.26 ms against
// 1.22 ms with a run of vectors per lane, each tested by itself.  (Before
// slot 0's bound: an item of 64 neighbouring cubes 0.63 ms against 0.32; one
// sweep, one way, per step 1.15 ms; slots ordered outward from s leave twice
// as many cubes undecided.)
#include <hip/hip_runtime.h>

#include "bat_launch.hpp"

using bat::u32;
using bat::u64;

constexpr int kMsWaves = bat::kWavesPerBlock;
constexpr u32 kMsStack = 512;  // nodes of a wavefront's stack

// A node: 5 bits per state of the slots below L, then K, the lane whose root
// it lies under, and what its parent's tests say.
constexpr u32 kMsAtK = 5 * batk::kMsTreeSlots, kMsAtRoot = kMsAtK + 4;
constexpr u64 kMsLowFails = 1ull << (kMsAtRoot + 6), kMsHighMeets = 1ull << (kMsAtRoot + 7);
static_assert(kMsAtRoot + 8 <= 64 && batk::kMsTreeSlots < 16, "");

// Up to 16 slots the per-slot registers leave room for 4 wavefronts per SIMD
// (128 VGPRs), up to 20 for 3; the compiler is held to that.
template <int MM>
__global__ void __launch_bounds__(64 * kMsWaves) __attribute__((amdgpu_waves_per_eu(MM <= 16 ? 4 : MM <= 20 ? 3 : 1, MM <= 16 ? 4 : MM <= 20 ? 3 : 8)))
k_ms_flow(batk::MsParams P)
{
    __shared__ int capt[batk::kMsMaxTable + batk::kMsMaxArcs];
    __shared__ double wt[batk::kMsMaxTable + batk::kMsMaxArcs];
    __shared__ u64 stacks[kMsWaves][kMsStack];
    __shared__ unsigned char roots[kMsWaves][64][MM];  // states of the slots from L on
    __shared__ int sig[MM], off[MM], least[MM], most[MM];
    __shared__ u64 size[batk::kMsTreeSlots + 1];       // vectors of a cube
    __shared__ double weight[batk::kMsTreeSlots + 1];  // and its free slots' probability
    const u32 tid = threadIdx.x, lane = tid & 63u, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    if (blockIdx.x == 0 && tid == 0) P.diag[0] = wall_clock64();
    for (u32 i = tid; i < P.n_table; i += blockDim.x) {
        capt[i] = P.cap[i];
        wt[i] = P.w[i];
    }
    if (tid == 0) {
#pragma unroll
        for (int i = 0; i < MM; ++i) {
            sig[i] = (int)P.sig[i];
            off[i] = (int)P.off[i];
            least[i] = P.least[i];
            most[i] = P.most[i];
        }
        for (u32 k = 0; k <= P.L; ++k) {
            size[k] = P.size[k];
            weight[k] = P.weight[k];
        }
    }
    __syncthreads();
    const u64 item = (u64)blockIdx.x * kMsWaves + wave;
    if (item >= P.n_items) return;
    const u32 s = P.s, t = P.t, L = P.L;
    const int d = (int)P.d;
    const bool dir = P.directed != 0;
    u64 *stack = stacks[wave];

    // the item's roots lie apart (neighbours share most slots' states, and a
    // hard one has hard neighbours)
    const u64 root0 = P.root_lo + item, root = root0 + lane * P.n_items, size_L = P.size[L];
    // the item holds an end of the range inside a root's cube
    const bool ends = (item == 0ull && P.root_lo * size_L < P.c_lo) ||
                      ((P.root_hi - 1ull - root0) % P.n_items == 0ull && P.root_hi * size_L > P.c_hi);
    {
        // (64-bit divisions only while needed)
        u64 r = root;
        u32 i = L;
        for (; i < P.m && (P.root_hi >> 31) != 0ull && __ballot((r >> 32) != 0ull) != 0ull; ++i) {
            roots[wave][lane][i] = (unsigned char)(r % (u64)(u32)sig[i]);
            r /= (u64)(u32)sig[i];
        }
        for (u32 q = (u32)r; i < (u32)MM; ++i) {
            const u32 x = (u32)sig[i];
            roots[wave][lane][i] = (unsigned char)(i < P.m ? q % x : 0u);
            q = i < P.m ? q / x : 0u;
        }
    }
    double hi = 0.0, lo = 0.0;
    u64 cnt = 0;
    u64 node = (u64)L << kMsAtK | (u64)lane << kMsAtRoot;
    u32 K = L, top = L;  // its K; the lane's own cubes end at `top`
    bool busy = root < P.root_hi, fresh = busy;
    u32 sp = 0u;  // nodes on the stack

    int rf[MM], rb[MM];  // residual capacity of each slot's arc, u -> v and v -> u
#pragma unroll
    for (int i = 0; i < MM; ++i) rf[i] = rb[i] = 0;
    const bool two = sig[0] <= 2;  // slot 0's states are its least and its greatest
    int total = 0, base = 0;       // the flow; its greatest with the least capacities
    bool high = false;             // testing the greatest capacities
    u32 reach = 0u, tf = 0u, tb = 0u;

    auto state = [&](u32 i) -> u32 {
        return i < (u32)batk::kMsTreeSlots && i < L ? (u32)(node >> (5u * i)) & 31u
                                                    : (u32)roots[wave][(node >> kMsAtRoot) & 63u][i];
    };
    // the cube's weight (need: only its states of slot 0 of that capacity)
    auto met = [&](u64 nd, u32 k, int need) {
        double pr = weight[k];
        u64 number = size[k];
        if (need > 0) {
            pr = 0.0;
            number = 0ull;
            for (int x = 0; x < sig[0]; ++x) {
                const bool on = capt[x] >= need;
                pr += on ? wt[x] : 0.0;
                number += on ? 1ull : 0ull;
            }
        }
#pragma unroll
        for (u32 i = 0; i < (u32)MM; ++i) {
            const u32 x = i < (u32)batk::kMsTreeSlots && i < L ? (u32)(nd >> (5u * i)) & 31u
                                                              : (u32)roots[wave][(nd >> kMsAtRoot) & 63u][i];
            pr *= i < k ? 1.0 : wt[P.off[i] + x];
        }
        double s_, e_;
        bat::two_sum(hi, pr, s_, e_);
        hi = s_;
        lo += e_;
        cnt += number;
    };
    // the child of `nd` (of cube k) with state x in slot k - 1
    auto child = [&](u64 nd, u32 k, u32 x) -> u64 {
        const int c = capt[off[k - 1u] + (int)x];
        u64 r = (nd & ~(15ull << kMsAtK | kMsLowFails | kMsHighMeets)) | (u64)(k - 1u) << kMsAtK | (u64)x << (5u * (k - 1u));
        if (!ends) {
            r |= c == least[k - 1u] ? kMsLowFails : 0ull;
            r |= c == most[k - 1u] ? kMsHighMeets : 0ull;
        }
        return r;
    };

    for (;;) {
        __builtin_amdgcn_wave_barrier();
        const u64 idle = __ballot(!busy);
        if (idle == ~0ull && sp == 0u) break;
        if (idle != 0ull && sp != 0u) {
            const u32 n = min((u32)__popcll(idle), sp);
            const u32 k = __builtin_amdgcn_mbcnt_hi((u32)(idle >> 32), __builtin_amdgcn_mbcnt_lo((u32)idle, 0u));
            if (!busy && k < n) {
                node = stack[sp - 1u - k];
                K = top = (u32)(node >> kMsAtK) & 15u;
                busy = fresh = true;
            }
            sp -= n;
        }
        // -1: the test goes on; 0: not met; 1: met; 2: split; 3: met from
        // some capacity of slot 0 on
        int out = -1;
        if (fresh) {
            fresh = false;
            if (ends) {
                u64 c = (root0 + ((node >> kMsAtRoot) & 63u) * P.n_items) * size_L;
                for (u32 i = 0; i < L; ++i) c += ((node >> (5u * i)) & 31u) * size[i];
                const u64 e = c + size[K];
                if (e <= P.c_lo || c >= P.c_hi) out = 0;
                else if (c < P.c_lo || e > P.c_hi) out = 2;
            }
            if ((node & kMsLowFails) && (node & kMsHighMeets) && (K != 1u || two)) out = K == 1u ? 3 : 2;
            high = (node & kMsLowFails) && (K != 1u || two);
#pragma unroll
            for (u32 i = 0; i < (u32)MM; ++i) {
                const int c = capt[P.off[i] + state(i)];
                rf[i] = i < K ? (high ? P.most[i] : P.least[i]) : c;
                rb[i] = dir ? 0 : rf[i];
            }
            total = 0;
            reach = 1u << s;
            tf = tb = 0u;
        }
        if (busy && out < 0) {
            // reach grows from {s} over arcs with residual capacity, from
            // the slots near the terminals to the far ones and back: the way
            // a path takes them; tf / tb mark the arc that first reached a
            // node, used u -> v or v -> u
            const u32 before = reach;
            auto search = [&](int i) {
                const u32 u = P.u[i], v = P.v[i], ru = reach >> u, rv = reach >> v;
                const u32 fw = ru & ~rv & (u32)min(rf[i], 1), bw = rv & ~ru & (u32)min(rb[i], 1);
                reach |= (fw << v) | (bw << u);
                tf |= fw << i;
                tb |= bw << i;
            };
#pragma unroll
            for (int i = MM - 1; i >= 0; --i) search(i);
#pragma unroll
            for (int i = 1; i < MM; ++i) search(i);
            const bool found = (reach >> t) & 1u;
            if (!found && reach == before) {
                // no augmenting path: the flow is maximal
                if (high || K == 0u) {
                    out = 0;
                } else if (node & kMsHighMeets) {
                    out = K == 1u ? 3 : 2;
                    base = total;
                } else {
                    // the greatest capacities, from this flow and reach
                    high = true;
                    base = total;
#pragma unroll
                    for (u32 i = 0; i < (u32)MM; ++i) {
                        const int more = i < K ? P.most[i] - P.least[i] : 0;
                        rf[i] += more;
                        rb[i] += dir ? 0 : more;
                    }
                }
            }
            if (found) {
                // the marked arcs form a tree rooted at s: collect its path
                // to t, an arc joining when the node it reached is on the
                // path, in the reverse of the search's order
                u32 on = 1u << t, pf = 0u, pb = 0u;
                auto collect = [&](int i) {
                    const u32 u = P.u[i], v = P.v[i];
                    const u32 jf = (tf >> i) & (on >> v) & 1u;
                    const u32 jb = (tb >> i) & (on >> u) & 1u;
                    on |= (jf << u) | (jb << v);
                    pf |= jf << i;
                    pb |= jb << i;
                };
                do {
#pragma unroll
                    for (int i = MM - 1; i >= 0; --i) collect(i);
#pragma unroll
                    for (int i = 1; i < MM; ++i) collect(i);
                } while (!((on >> s) & 1u));
                // push its bottleneck (at least one unit), at most what the
                // demand lacks
                int b = d - total;
#pragma unroll
                for (int i = 0; i < MM; ++i) {
                    b = (pf >> i) & 1u ? min(b, rf[i]) : b;
                    b = (pb >> i) & 1u ? min(b, rb[i]) : b;
                }
#pragma unroll
                for (int i = 0; i < MM; ++i) {
                    const int df = ((pf >> i) & 1u) ? b : 0, db = ((pb >> i) & 1u) ? b : 0;
                    rf[i] += db - df;
                    rb[i] += df - db;
                }
                total += b;
                reach = 1u << s;
                tf = tb = 0u;
                if (total >= d) out = !high ? 1 : K == 1u ? 3 : 2;
            }
        }
        if (out == 1) met(node, K, 0);
        if (out == 3) met(node, 1u, two ? most[0] : least[0] + d - base);
        // the cubes that split: children on the stack while there is room,
        // else the lane goes to the first of its own
        if (__ballot(out == 2) != 0ull) {
            const u64 split = __ballot(out == 2);
            const u32 rank = __builtin_amdgcn_mbcnt_hi((u32)(split >> 32), __builtin_amdgcn_mbcnt_lo((u32)split, 0u));
            const bool room = sp + (rank + 1u) * P.most_states <= kMsStack;
            bool more = out == 2;
            if (!room && more) {
                node = child(node, K, 0u);
                --K;
                fresh = true;
                out = -1;
                more = false;
            }
            for (u32 x = 0;; ++x) {
                more = more && x < (u32)sig[K ? K - 1u : 0u];
                if (__ballot(more) == 0ull) break;
                const u64 w = __ballot(more);
                if (more)
                    stack[sp + __builtin_amdgcn_mbcnt_hi((u32)(w >> 32), __builtin_amdgcn_mbcnt_lo((u32)w, 0u))] =
                        child(node, K, x);
                sp += (u32)__popcll(w);
            }
            bat::wave_lds_sync();
        }
        if (out >= 0) {
            // decided, or its children are on the stack: the next of the
            // lane's own cubes
            busy = false;
            while (K < top) {
                const u32 x = ((u32)(node >> (5u * K)) & 31u) + 1u;
                node &= ~(31ull << (5u * K));
                if (x < (u32)sig[K]) {
                    node = child(node, K + 1u, x);
                    busy = fresh = true;
                    break;
                }
                ++K;
            }
        }
    }
    bat::wave_sum_dd(hi, lo);
    const u64 csum = bat::wave_sum_u64(cnt);
    if (lane == 0) {
        P.part[2 * item] = hi;
        P.part[2 * item + 1] = lo;
        P.pcount[item] = csum;
    }
}

template __global__ void k_ms_flow<16>(batk::MsParams);
template __global__ void k_ms_flow<20>(batk::MsParams);
template __global__ void k_ms_flow<24>(batk::MsParams);
template __global__ void k_ms_flow<32>(batk::MsParams);

namespace batk {

hipError_t ms_sweep(hipStream_t st, unsigned blocks, const MsParams &P)
{
    const dim3 g(blocks), b(64 * kMsWaves);
    switch (ms_slots((int)P.m)) {
    case 16: hipLaunchKernelGGL(k_ms_flow<16>, g, b, 0, st, P); break;
    case 20: hipLaunchKernelGGL(k_ms_flow<20>, g, b, 0, st, P); break;
    case 24: hipLaunchKernelGGL(k_ms_flow<24>, g, b, 0, st, P); break;
    default: hipLaunchKernelGGL(k_ms_flow<32>, g, b, 0, st, P); break;
    }
    return hipGetLastError();
}

}  // namespace batk

// bat_cube_plan.hpp -- host side of the sub-cube sweep (bat_cube.hpp): which
// arcs it enumerates, in which order they take the counter bits, and the
// steps of its closures.
//
// Arcs on no simple s-t path never change a verdict, so they are left out of
// the sweep's counter: each contributes the factor q(0) + q(1) = 1 to the
// sums and 2 to the count.  The others take the counter bits by influence:
// the arc most often pivotal (over vectors drawn evenly) is the most
// significant bit, so that the low bits, free while a sub-cube is decided
// as a whole, are the arcs that least often matter.  On the 5x5 grid 4% of
// the cubes of 5 low arcs, 12% of those of 10 and 23% of those of 15 are
// left undecided this way; in breadth-first order it is 30%, 38% and 42%.
#pragma once
#include <algorithm>
#include <cstdint>
#include <cstring>
#include <vector>

#include "bat.h"
#include "bat_launch.hpp"

namespace batcube {

using bat::u32;
using bat::u64;

// One step of a closure on its words ("slots"; slot c < M holds the working
// mask of the arc at counter bit c): d = a & b (assign), or d |= a & b.
struct Step {
    int a, b, d;
    bool assign;
};

// A closure as straight-line steps: the nodes other than s and t are removed
// one by one, and removing k joins each pair of its neighbours i, j by the
// word "i - k - j works", added to theirs.  What is left between s and t is
// the verdict.  Exact in one pass, with no test for a fixed point: the node
// with the fewest pairs goes first (then the fewest new ones), and the
// networks here take 20 to 135 steps where sweeps over the relaxations until
// nothing changes take about 5 x 2 per arc and a popcount test each.
struct Program {
    std::vector<Step> step;
    int result = -1;  // slot of the verdict; -1: never connected, -2: always
    int slots = 0;    // slots used, the arcs' included
};

struct CubePlan {
    int m = 0, M = 0;                   // arcs, arcs enumerated
    int levels = 1, lane_bits = 0;      // see bat_cube.hpp
    bool directed = false;
    std::vector<int> arc_of_bit;        // [M]
    int slots = 0;                      // the most slots of a closure
    int steps = 0;                      // steps of all closures
    // [0]: the whole graph; [2 l - 1], [2 l]: level l with the arcs below
    // its word all up, all down
    Program prog[2 * bat::kCubeLevels - 1];
    int rel_bits() const { return bat::kCubeGroup * levels + lane_bits; }
};

// How often each arc is pivotal over 1024 vectors drawn evenly (a fixed
// sequence: the order, and with it the rounding, is the same every call),
// bit-sliced, 512 vectors to a block.  An arc u - v that is down is pivotal
// when s reaches u and v reaches t (or the other way round) and s does not
// reach t.  (Twice the vectors left the number of undecided cubes within 2%
// on the 36-arc random graph and the 5x5 grid.)
typedef u64 Words __attribute__((vector_size(64)));
constexpr int kSampleBlocks = 2;

struct Sampler {
    Words up[BAT_MAX_ARCS], rs[BAT_MAX_NODES], rt[BAT_MAX_NODES];
    int u[BAT_MAX_ARCS], v[BAT_MAX_ARCS];
    int arcs = 0;
};

// (hipcc also parses this file for the device, which has no such versions)
#if defined(__HIP_DEVICE_COMPILE__)
#define BAT_HOST_CLONES
#else
#define BAT_HOST_CLONES __attribute__((target_clones("avx2", "default")))
#endif

// One block: reach from s and to t over the block's working arcs, then the
// pivotal vectors of each arc added to count.
BAT_HOST_CLONES inline void sample_block(Sampler &X, int n, int s, int t, bool directed, u64 &seed, u32 *count)
{
    const Words none = {0, 0, 0, 0, 0, 0, 0, 0}, all = ~none;
    for (int i = 0; i < X.arcs; ++i)
        for (int k = 0; k < 8; ++k) {  // splitmix64
            u64 z = (seed += 0x9E3779B97F4A7C15ull);
            z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ull;
            z = (z ^ (z >> 27)) * 0x94D049BB133111EBull;
            X.up[i][k] = z ^ (z >> 31);
        }
    for (int x = 0; x < n; ++x) X.rs[x] = X.rt[x] = none;
    X.rs[s] = X.rt[t] = all;
    for (int side = 0; side < 2; ++side) {
        Words *r = side ? X.rt : X.rs;
        // a digraph's reach to t runs against the arcs
        const int *hu = side && directed ? X.v : X.u, *hv = side && directed ? X.u : X.v;
        for (bool fwd = true;; fwd = !fwd) {
            Words grew = none;
            for (int q = 0; q < X.arcs; ++q) {
                const int i = fwd ? q : X.arcs - 1 - q;
                const Words a = r[hu[i]], c = r[hv[i]], w = X.up[i];
                const Words nc = c | (a & w), na = directed ? a : a | (c & w);
                grew |= (nc ^ c) | (na ^ a);
                r[hv[i]] = nc;
                r[hu[i]] = na;
            }
            u64 any = 0;
            for (int k = 0; k < 8; ++k) any |= grew[k];
            if (!any) break;
        }
    }
    for (int i = 0; i < X.arcs; ++i) {
        Words p = X.rs[X.u[i]] & X.rt[X.v[i]];
        if (!directed) p |= X.rs[X.v[i]] & X.rt[X.u[i]];
        p &= ~X.up[i] & ~X.rs[t];
        for (int k = 0; k < 8; ++k) count[i] += (u32)__builtin_popcountll(p[k]);
    }
}

inline void influence(int n, int m, const bat_arc *arcs, const std::vector<char> &rel, int s, int t, bool directed,
                      std::vector<u32> &count)
{
    count.assign(m, 0);
    Sampler X;
    int arc[BAT_MAX_ARCS];
    for (int i = 0; i < m; ++i)
        if (rel[i]) {
            arc[X.arcs] = i;
            X.u[X.arcs] = arcs[i].u;
            X.v[X.arcs++] = arcs[i].v;
        }
    u32 c[BAT_MAX_ARCS] = {};
    u64 seed = 0x9E3779B97F4A7C15ull;
    for (int b = 0; b < kSampleBlocks; ++b) sample_block(X, n, s, t, directed, seed, c);
    for (int k = 0; k < X.arcs; ++k) count[arc[k]] = c[k];
}

// The steps of one closure.  Arcs below counter bit `low` are all up (joined
// into one node each; a digraph's stay, with a full mask) or all down (left
// out).
inline Program make_program(int n, const bat_arc *arcs, const std::vector<int> &arc_of_bit, int s, int t, int low,
                            bool up, bool directed)
{
    std::vector<int> root(n);
    for (int x = 0; x < n; ++x) root[x] = x;
    auto find = [&](int x) {
        while (root[x] != x) x = root[x] = root[root[x]];
        return x;
    };
    const int M = (int)arc_of_bit.size();
    if (up && !directed)
        for (int c = 0; c < low && c < M; ++c) root[find(arcs[arc_of_bit[c]].u)] = find(arcs[arc_of_bit[c]].v);
    s = find(s);
    t = find(t);
    Program P;
    P.slots = M;
    if (s == t) {
        P.result = -2;
        return P;
    }
    // slot[i * n + j]: the word of i -> j, or -1 (the same both ways for
    // undirected arcs); to[i], from[j]: the nodes at its other end; spare:
    // slots freed by removed nodes
    std::vector<int> slot((size_t)n * n, -1), spare;
    u64 to[BAT_MAX_NODES] = {}, from[BAT_MAX_NODES] = {};
    auto at = [&](int i, int j) -> int & { return slot[(size_t)i * n + j]; };
    auto set = [&](int i, int j, int x) {
        at(i, j) = x;
        to[i] |= 1ull << j;
        from[j] |= 1ull << i;
        if (!directed) {
            at(j, i) = x;
            to[j] |= 1ull << i;
            from[i] |= 1ull << j;
        }
    };
    for (int c = M - 1; c >= 0; --c) {
        if (c < low && !(up && directed)) break;
        const int u = find(arcs[arc_of_bit[c]].u), v = find(arcs[arc_of_bit[c]].v);
        if (u == v || (directed && (v == s || u == t))) continue;
        if (at(u, v) >= 0) P.step.push_back({c, c, at(u, v), false});  // parallel arcs: one word
        else set(u, v, c);
    }
    u64 left = 0;
    for (int x = 0; x < n; ++x)
        if (find(x) == x && x != s && x != t) left |= 1ull << x;
    while (left) {
        int k = -1, best_pairs = 0, best_new = 0;
        for (u64 w = left; w; w &= w - 1) {
            const int x = __builtin_ctzll(w);
            const u64 in = from[x], out = to[x];
            const int ni = __builtin_popcountll(in), no = __builtin_popcountll(out);
            const int pairs = directed ? ni * no - __builtin_popcountll(in & out) : ni * (ni - 1) / 2;
            if (k >= 0 && pairs > best_pairs) continue;
            int fresh = 0;
            for (u64 q = in; q; q &= q - 1) {
                const int i = __builtin_ctzll(q);
                fresh += __builtin_popcountll(out & ~to[i] & ~(1ull << i));
            }
            if (k < 0 || pairs < best_pairs || fresh < best_new) {
                k = x;
                best_pairs = pairs;
                best_new = fresh;
            }
        }
        left &= ~(1ull << k);
        const u64 in = from[k], out = to[k];
        for (u64 q = in; q; q &= q - 1) {
            const int i = __builtin_ctzll(q);
            for (u64 z = directed ? out : out & (~0ull << i); z; z &= z - 1) {
                const int j = __builtin_ctzll(z);
                if (i == j) continue;
                const int a = at(i, k), b = at(k, j), d = at(i, j);
                if (d >= 0) {
                    P.step.push_back({a, b, d, false});
                    continue;
                }
                int x = P.slots;
                if (spare.empty()) {
                    ++P.slots;
                } else {
                    x = spare.back();
                    spare.pop_back();
                }
                P.step.push_back({a, b, x, true});
                set(i, j, x);
            }
        }
        for (u64 q = in; q; q &= q - 1) {
            const int i = __builtin_ctzll(q);
            spare.push_back(at(i, k));
            to[i] &= ~(1ull << k);
        }
        for (u64 q = out; q; q &= q - 1) {
            const int j = __builtin_ctzll(q);
            if (directed) spare.push_back(at(k, j));
            from[j] &= ~(1ull << k);
        }
    }
    P.result = at(s, t);
    return P;
}

// rel[i]: arc i lies on a relevant path.  levels: 0 = by size.
inline void make_cube_plan(int n, int m, const bat_arc *arcs, const std::vector<char> &rel, int s, int t, bool directed,
                           int levels, CubePlan &P)
{
    P.m = m;
    P.directed = directed;
    P.arc_of_bit.clear();
    for (int i = m - 1; i >= 0; --i)
        if (rel[i]) P.arc_of_bit.push_back(i);
    P.M = (int)P.arc_of_bit.size();
    constexpr int G = bat::kCubeGroup;
    P.levels = std::max(1, std::min(levels, std::min(bat::kCubeLevels, P.M / G)));
    if (P.levels > 1) {  // one level decides every vector by itself: any order does
        std::vector<u32> cnt;
        influence(n, m, arcs, rel, s, t, directed, cnt);
        std::stable_sort(P.arc_of_bit.begin(), P.arc_of_bit.end(), [&](int a, int b) { return cnt[a] < cnt[b]; });
    }
    P.lane_bits = std::max(0, std::min(bat::kLaneBits, P.M - G * P.levels));
    P.slots = P.steps = 0;
    for (int k = 0; k < 2 * P.levels - 1; ++k) {
        const int lev = (k + 1) / 2;
        P.prog[k] = make_program(n, arcs, P.arc_of_bit, s, t, G * lev, (k & 1) != 0, directed);
        P.slots = std::max(P.slots, P.prog[k].slots);
        P.steps += (int)P.prog[k].step.size();
    }
}

}  // namespace batcube

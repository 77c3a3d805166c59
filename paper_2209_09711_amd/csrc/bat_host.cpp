// bat_host.cpp -- the C ABI declared in include/bat.h.
//
// Per call: validate -> plan (which arcs can matter, sweep order, launch
// shape) -> queue on one stream: probability tables from p (on the device),
// the enumeration kernel over the counter range, a fixed-order reduction of
// the per-work-item partials, and either a copy back (synchronous entry
// points) or a finalize kernel into the caller's device buffers (_async).
//
// The enumeration kernel is the template in bat_device.hpp, instantiated
// either ahead of time with the graph read at run time (k_fwd_dyn /
// k_grad_dyn) or at run time through hiprtc with the graph's arcs as
// compile-time constants, so that every node's reach word lives in a fixed
// register (bat_fwd_jit / bat_grad_jit).  Compiled modules are cached per
// (device, graph structure, kernel kind).
#include <hip/hip_runtime.h>
#include <hip/hiprtc.h>

#include <algorithm>
#include <atomic>
#include <cerrno>
#include <chrono>
#include <cmath>
#include <cstdarg>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <map>
#include <mutex>
#include <string>
#include <thread>
#include <tuple>
#include <vector>

#include <dlfcn.h>
#include <spawn.h>
#include <sys/stat.h>
#include <sys/wait.h>
#include <unistd.h>

#include "bat.h"
#include "bat_launch.hpp"
#include "bat_cube_plan.hpp"

using bat::u32;
using bat::u64;


namespace {

const char *kVersion = "bat-mi355x 0.1.0";

#include "bat_device_embed.inc"  // kDeviceSource: bat_device.hpp as text

// ------------------------------------------------------------ errors
thread_local std::string t_err;

int fail(int code, const char *fmt, ...)
{
    char buf[1024];
    va_list ap;
    va_start(ap, fmt);
    vsnprintf(buf, sizeof buf, fmt, ap);
    va_end(ap);
    t_err = buf;
    return code;
}

#define HIPCHK(expr)                                                                         \
    do {                                                                                     \
        hipError_t e_ = (expr);                                                              \
        if (e_ != hipSuccess)                                                                \
            return fail(e_ == hipErrorOutOfMemory ? BAT_ENOMEM : BAT_EDEVICE, "%s: %s (%s:%d)", \
                        #expr, hipGetErrorString(e_), __FILE__, __LINE__);                   \
    } while (0)

// ------------------------------------------------------------ options
struct Options {
    std::atomic<int64_t> jit{2}, chunk_log2{0}, seg_log2{6}, check_every{1}, autotune{1}, perm{-1}, chain_log2{-1}, item_order{-1},
        window_test{1}, block_waves{-1}, super_restart{-1}, simd_waves{-1}, keep_bottom{-1}, series{1},
        grad_keep_bottom{2}, ms_run{0}, jit_procs{16}, batch_jit_arcs{-1}, batch_streams{-1}, ms_bits{1}, batch_acc{1}, jit_flush_req{0},
        cubes{-1}, cube_levels{0}, cube_split{0};
    Options()
    {
        auto rd = [](const char *k, std::atomic<int64_t> &v) {
            const char *e = getenv(k);
            if (e && *e) v = strtoll(e, nullptr, 10);
        };
        rd("BAT_JIT", jit);
        rd("BAT_CHUNK_LOG2", chunk_log2);
        rd("BAT_SEG_LOG2", seg_log2);
        rd("BAT_CHECK_EVERY", check_every);
        rd("BAT_AUTOTUNE", autotune);
        rd("BAT_PERM", perm);
        rd("BAT_CHAIN_LOG2", chain_log2);
        rd("BAT_ITEM_ORDER", item_order);
        rd("BAT_WINDOW_TEST", window_test);
        rd("BAT_BLOCK_WAVES", block_waves);
        rd("BAT_SUPER_RESTART", super_restart);
        rd("BAT_SIMD_WAVES", simd_waves);
        rd("BAT_KEEP_BOTTOM", keep_bottom);
        rd("BAT_SERIES", series);
        rd("BAT_GRAD_KEEP_BOTTOM", grad_keep_bottom);
        rd("BAT_MS_RUN", ms_run);
        rd("BAT_JIT_PROCS", jit_procs);
        rd("BAT_BATCH_JIT_ARCS", batch_jit_arcs);
        rd("BAT_BATCH_STREAMS", batch_streams);
        rd("BAT_MS_BITS", ms_bits);
        rd("BAT_BATCH_ACC", batch_acc);
        rd("BAT_CUBES", cubes);
        rd("BAT_CUBE_LEVELS", cube_levels);
        rd("BAT_CUBE_SPLIT", cube_split);
    }
    std::atomic<int64_t> *find(const char *k)
    {
        if (!k) return nullptr;
        if (!strcmp(k, "BAT_JIT")) return &jit;
        if (!strcmp(k, "BAT_CHUNK_LOG2")) return &chunk_log2;
        if (!strcmp(k, "BAT_SEG_LOG2")) return &seg_log2;
        if (!strcmp(k, "BAT_CHECK_EVERY")) return &check_every;
        if (!strcmp(k, "BAT_AUTOTUNE")) return &autotune;
        if (!strcmp(k, "BAT_PERM")) return &perm;
        if (!strcmp(k, "BAT_CHAIN_LOG2")) return &chain_log2;
        if (!strcmp(k, "BAT_ITEM_ORDER")) return &item_order;
        if (!strcmp(k, "BAT_WINDOW_TEST")) return &window_test;
        if (!strcmp(k, "BAT_BLOCK_WAVES")) return &block_waves;
        if (!strcmp(k, "BAT_SUPER_RESTART")) return &super_restart;
        if (!strcmp(k, "BAT_SIMD_WAVES")) return &simd_waves;
        if (!strcmp(k, "BAT_KEEP_BOTTOM")) return &keep_bottom;
        if (!strcmp(k, "BAT_SERIES")) return &series;
        if (!strcmp(k, "BAT_GRAD_KEEP_BOTTOM")) return &grad_keep_bottom;
        if (!strcmp(k, "BAT_MS_RUN")) return &ms_run;
        if (!strcmp(k, "BAT_JIT_PROCS")) return &jit_procs;
        if (!strcmp(k, "BAT_BATCH_JIT_ARCS")) return &batch_jit_arcs;
        if (!strcmp(k, "BAT_BATCH_STREAMS")) return &batch_streams;
        if (!strcmp(k, "BAT_MS_BITS")) return &ms_bits;
        if (!strcmp(k, "BAT_BATCH_ACC")) return &batch_acc;
        if (!strcmp(k, "BAT_JIT_FLUSH")) return &jit_flush_req;
        if (!strcmp(k, "BAT_CUBES")) return &cubes;
        if (!strcmp(k, "BAT_CUBE_LEVELS")) return &cube_levels;
        if (!strcmp(k, "BAT_CUBE_SPLIT")) return &cube_split;
        return nullptr;
    }
    // whether every knob of the plain sweep's launch is at its default
    bool plain_shape_default() const
    {
        return jit == 2 && perm < 0 && chain_log2 < 0 && chunk_log2 <= 0 && seg_log2 == 6 && check_every == 1 &&
               item_order < 0 && window_test == 1 && block_waves < 0 && super_restart < 0 && simd_waves < 0 &&
               keep_bottom < 0 && series == 1 && grad_keep_bottom == 2;
    }
};
Options &opts()
{
    static Options o;
    return o;
}

// ------------------------------------------------------------ validation
int validate(int32_t n, int32_t m, const bat_arc *arcs, const double *p_host, int32_t s, int32_t t)
{
    if (n < 2) return fail(BAT_EINVAL, "n_nodes must be >= 2 (got %d)", n);
    if (m < 0) return fail(BAT_EINVAL, "n_arcs must be >= 0 (got %d)", m);
    if (n > BAT_MAX_NODES) return fail(BAT_ETOOBIG, "n_nodes %d exceeds %d", n, BAT_MAX_NODES);
    if (m > BAT_MAX_ARCS) return fail(BAT_ETOOBIG, "n_arcs %d exceeds %d", m, BAT_MAX_ARCS);
    if (s < 0 || s >= n || t < 0 || t >= n) return fail(BAT_EINVAL, "s=%d or t=%d outside [0,%d)", s, t, n);
    if (s == t) return fail(BAT_EINVAL, "s and t must differ (both %d)", s);
    if (m > 0 && !arcs) return fail(BAT_EINVAL, "arcs is NULL");
    for (int32_t i = 0; i < m; ++i)
        if (arcs[i].u < 0 || arcs[i].u >= n || arcs[i].v < 0 || arcs[i].v >= n)
            return fail(BAT_EINVAL, "arc %d = (%d,%d) has a node outside [0,%d)", i, arcs[i].u, arcs[i].v, n);
    if (p_host)
        for (int32_t i = 0; i < m; ++i)
            if (!(p_host[i] >= 0.0 && p_host[i] <= 1.0))
                return fail(BAT_EINVAL, "p[%d] = %g is not a probability", i, p_host[i]);
    return BAT_OK;
}

// ------------------------------------------------------------ planning
// Arcs that lie on some simple s-t path: exactly those in the biconnected
// component of the graph plus a virtual arc (s, t) that contains the
// virtual arc (two edges share a biconnected component iff a simple cycle
// passes through both).  Every other arc never changes whether s reaches t,
// so the sweeps skip it; its state is still enumerated and weighted.
struct Bcc {
    int n, m;
    std::vector<std::vector<std::pair<int, int>>> adj;
    std::vector<int> disc, low, stk;
    std::vector<char> rel;
    int timer = 0;
    void dfs(int u, int pe)
    {
        disc[u] = low[u] = ++timer;
        for (auto [v, e] : adj[u]) {
            if (e == pe) continue;
            if (!disc[v]) {
                stk.push_back(e);
                dfs(v, e);
                low[u] = std::min(low[u], low[v]);
                if (low[v] >= disc[u]) {
                    std::vector<int> comp;
                    for (;;) {
                        int x = stk.back();
                        stk.pop_back();
                        comp.push_back(x);
                        if (x == e) break;
                    }
                    bool has_virtual = false;
                    for (int x : comp) has_virtual |= (x == m);
                    if (has_virtual)
                        for (int x : comp)
                            if (x < m) rel[x] = 1;
                }
            } else if (disc[v] < disc[u]) {
                stk.push_back(e);
                low[u] = std::min(low[u], disc[v]);
            }
        }
    }
};

struct Plan {
    int n = 0, m = 0, s = 0, t = 0;
    int perm = 0;                         // arc -> counter bit assignment kind (0 = the paper's order)
    bool directed = false;                // arcs are u -> v
    bool identity = true;                 // cb_of_arc is the paper's backward order
    std::vector<int> cb_of_arc;           // counter bit of each arc
    std::vector<unsigned char> row;       // row[j] = arc at counter bit m-1-j
    int N = 0, S = 0, T = 0;              // relevant nodes, renumbered
    std::vector<int> ru, rv, rb, rd;      // relaxations (forward order): nodes, counter bit, discovers rv
    std::vector<u32> code, wconst;        // the same for the generic kernel
    // The graph-specialised kernel's relaxations: as above, after series
    // contraction (undirected graphs), so a relaxation may stand for two
    // arcs in series; rb2 is the second arc's counter bit, -1 for one arc.
    int jN = 0, jS = 0, jT = 0;
    std::vector<int> jru, jrv, jrb, jrb2, jrd;
    std::vector<u32> prog;                // code/wconst pairs, groups of 4, forward then backward
    std::string structure;                // JIT key (graph structure only)
};

// Which arc sits at which counter bit.  Kind 0 is the paper's backward
// order (arc i at bit m-1-i) and kind kPermForward its forward BAT order
// (arc i at bit i): the range entry points use one of these two, since
// their indices are the paper's.  The others only reorder a full sweep (R
// and the count are sums over all vectors):
//   1: the 11 in-wavefront bits (word + lane) on the relevant arcs latest in
//      BFS order (nearest t), the 3 chained iteration bits on pruned arcs
//      first (their warm steps are free), then on the next-latest arcs;
//   2: in-wavefront bits as in kind 0, chained bits on pruned arcs, then on
//      arcs from the middle of the BFS order;
//   3: in-wavefront bits as in kind 1, chained bits as in kind 2.
// Every other arc keeps the relative order of kind 0.
constexpr int kPermKinds = 4;
constexpr int kDefaultPerm = 3;  // untuned whole sweeps
constexpr int kPermForward = 4;  // the forward BAT order (ranges only; never tuned)
constexpr int kPermInfluence = 5;  // the sub-cube sweep's order (bat_cube_plan.hpp); no sweep of the plain kernels
constexpr int kGradThreeWaveNodes = 28;  // gradient sweeps of graphs up to this size run 3 waves/SIMD
constexpr int kSuperMaxNodes = 28;       // forward sweeps keep super-block bottoms in LDS up to this size

void assign_bits(int m, const std::vector<int> &rel_bfs, const std::vector<char> &rel, int kind,
                 std::vector<int> &cb_of_arc)
{
    cb_of_arc.assign(m, -1);
    if (kind == kPermForward) {  // forward BAT (Section 4.2): arc i on counter bit i
        for (int i = 0; i < m; ++i) cb_of_arc[i] = i;
        return;
    }
    if (kind == 0 || m <= bat::kWordBits) {
        for (int i = 0; i < m; ++i) cb_of_arc[i] = m - 1 - i;
        return;
    }
    std::vector<int> by_cb;
    std::vector<char> used(m, 0);
    auto take = [&](int a) {
        if (a >= 0 && a < m && !used[a]) {
            used[a] = 1;
            by_cb.push_back(a);
        }
    };
    const int nr = (int)rel_bfs.size();
    // in-wavefront bits
    if (kind == 2) {
        for (int c = 0; c < bat::kWordBits; ++c) take(m - 1 - c);
    } else {
        for (int k = nr - 1; k >= 0 && (int)by_cb.size() < bat::kWordBits; --k) take(rel_bfs[k]);
        for (int i = m - 1; i >= 0 && (int)by_cb.size() < bat::kWordBits; --i) take(i);
    }
    // chained iteration bits
    const size_t want = bat::kWordBits + 3;
    for (int i = m - 1; i >= 0 && by_cb.size() < want; --i)
        if (!rel[i]) take(i);
    if (kind == 1) {
        for (int k = nr - 1; k >= 0 && by_cb.size() < want; --k) take(rel_bfs[k]);
    } else {
        for (int d = 0; d < nr && by_cb.size() < want; ++d) {
            int k = nr / 2 + ((d & 1) ? -(d + 1) / 2 : d / 2);
            if (k >= 0 && k < nr) take(rel_bfs[k]);
        }
    }
    for (int i = m - 1; i >= 0; --i) take(i);
    for (int c = 0; c < m; ++c) cb_of_arc[by_cb[c]] = c;
}

// The specialised kernel's relaxation list.  In an undirected graph a
// node other than s and t with exactly two relevant arcs, to two different
// neighbours u and w, only ever passes reach between them: it is reached
// from u through its first arc or from w through its second, and it passes
// on nothing else.  Removing it and joining u and w by one relaxation whose
// working mask is the AND of the two arcs' masks leaves every other node's
// reach, t's in particular, exactly as it was.  Only pairs of real arcs are
// joined (a relaxation stands for at most two arcs).  Digraphs keep the
// plain list.
void contract_series(int32_t n, int32_t m, const bat_arc *arcs, int32_t s, int32_t t, const std::vector<char> &rel,
                     Plan &P)
{
    struct VArc {
        int u, v, b1, b2;
    };
    std::vector<VArc> va;
    std::vector<std::vector<int>> inc(n);  // relevant arcs at each node
    for (int i = 0; i < m; ++i)
        if (rel[i] && arcs[i].u != arcs[i].v) {
            inc[arcs[i].u].push_back(i);
            inc[arcs[i].v].push_back(i);
        }
    std::vector<char> used(m, 0), gone(n, 0);
    if (!P.directed && opts().series.load() != 0) {
        for (int v = 0; v < n; ++v) {
            if (v == s || v == t || inc[v].size() != 2) continue;
            const int a = inc[v][0], b = inc[v][1];
            if (used[a] || used[b]) continue;
            const int u = arcs[a].u == v ? arcs[a].v : arcs[a].u;
            const int w = arcs[b].u == v ? arcs[b].v : arcs[b].u;
            if (u == w || gone[u] || gone[w]) continue;
            used[a] = used[b] = 1;
            gone[v] = 1;
            va.push_back({u, w, P.cb_of_arc[a], P.cb_of_arc[b]});
        }
    }
    for (int i = 0; i < m; ++i)
        if (rel[i] && !used[i] && arcs[i].u != arcs[i].v) va.push_back({arcs[i].u, arcs[i].v, P.cb_of_arc[i], -1});
    // BFS from s in arc-list order, as for the plain list
    std::vector<int> id(n, -1), order{s};
    std::vector<char> listed(va.size(), 0);
    id[s] = 0;
    P.jru.clear(); P.jrv.clear(); P.jrb.clear(); P.jrb2.clear(); P.jrd.clear();
    for (size_t h = 0; h < order.size(); ++h) {
        const int x = order[h];
        for (size_t k = 0; k < va.size(); ++k) {
            if (listed[k]) continue;
            const VArc &e = va[k];
            if (P.directed ? e.u != x : (e.u != x && e.v != x)) continue;
            const int y = e.u == x ? e.v : e.u;
            int disc = 0;
            if (id[y] < 0) {
                id[y] = (int)order.size();
                order.push_back(y);
                disc = 1;
            }
            listed[k] = 1;
            P.jru.push_back(id[x]);
            P.jrv.push_back(id[y]);
            P.jrb.push_back(e.b1);
            P.jrb2.push_back(e.b2);
            P.jrd.push_back(disc);
        }
    }
    if (id[t] < 0) {
        id[t] = (int)order.size();
        order.push_back(t);
    }
    P.jN = (int)order.size();
    P.jS = 0;
    P.jT = id[t];
}

// rel[i]: arc i may lie on a simple s-t path (exactly, for undirected arcs).
std::vector<char> relevance(int32_t n, int32_t m, const bat_arc *arcs, int32_t s, int32_t t, bool directed)
{
    Bcc B;
    B.n = n;
    B.m = m;
    B.rel.assign(m + 1, 0);
    if (!directed) {
        B.adj.assign(n, {});
        for (int i = 0; i < m; ++i) {
            int u = arcs[i].u, v = arcs[i].v;
            if (u == v) continue;  // a self-loop never joins two nodes
            B.adj[u].push_back({v, i});
            B.adj[v].push_back({u, i});
        }
        B.adj[s].push_back({t, m});
        B.adj[t].push_back({s, m});
        B.disc.assign(n, 0);
        B.low.assign(n, 0);
        B.dfs(s, -1);
    } else {
        // arc u -> v can only matter when s reaches u and v reaches t, and
        // it neither enters s nor leaves t (a superset of the arcs on simple
        // s -> t paths, which is hard to decide exactly for digraphs)
        std::vector<char> from_s(n, 0), to_t(n, 0);
        std::vector<int> q{s};
        from_s[s] = 1;
        for (size_t h = 0; h < q.size(); ++h)
            for (int i = 0; i < m; ++i)
                if (arcs[i].u == q[h] && !from_s[arcs[i].v]) {
                    from_s[arcs[i].v] = 1;
                    q.push_back(arcs[i].v);
                }
        q.assign(1, t);
        to_t[t] = 1;
        for (size_t h = 0; h < q.size(); ++h)
            for (int i = 0; i < m; ++i)
                if (arcs[i].v == q[h] && !to_t[arcs[i].u]) {
                    to_t[arcs[i].u] = 1;
                    q.push_back(arcs[i].u);
                }
        for (int i = 0; i < m; ++i) {
            const int u = arcs[i].u, v = arcs[i].v;
            B.rel[i] = u != v && v != s && u != t && from_s[u] && to_t[v];
        }
    }
    return B.rel;
}

void make_plan(int32_t n, int32_t m, const bat_arc *arcs, int32_t s, int32_t t, Plan &P, int perm_kind = 0,
               bool directed = false)
{
    P.n = n;
    P.m = m;
    P.s = s;
    P.t = t;
    P.perm = perm_kind;
    P.directed = directed;
    const std::vector<char> Brel = relevance(n, m, arcs, s, t, directed);

    // BFS from s over relevant arcs: node numbering and sweep order
    std::vector<int> id(n, -1), order, rel_bfs, disc_flag;
    std::vector<char> listed(m, 0);
    std::vector<std::pair<int, int>> ends;
    id[s] = 0;
    order.push_back(s);
    for (size_t h = 0; h < order.size(); ++h) {
        int u = order[h];
        for (int i = 0; i < m; ++i) {
            if (!Brel[i] || listed[i]) continue;
            int a = arcs[i].u, b = arcs[i].v;
            if (directed ? a != u : (a != u && b != u)) continue;  // directed: leave by the tail
            int w = (a == u) ? b : a;
            int discovers = 0;
            if (id[w] < 0) {
                id[w] = (int)order.size();
                order.push_back(w);
                discovers = 1;
            }
            listed[i] = 1;
            rel_bfs.push_back(i);
            ends.push_back({id[u], id[w]});
            disc_flag.push_back(discovers);
        }
    }
    if (id[t] < 0) {  // s and t never connected: keep both as nodes, no arcs
        id[t] = (int)order.size();
        order.push_back(t);
    }
    // relevant = swept: an arc the search from s never lists cannot matter
    std::vector<char> rel(m, 0);
    for (int i = 0; i < m; ++i) rel[i] = listed[i];
    assign_bits(m, rel_bfs, rel, perm_kind, P.cb_of_arc);
    {  // must be a bijection onto [0, m); otherwise use the paper's order
        std::vector<char> hit(std::max(m, 1), 0);
        bool ok = true;
        for (int i = 0; i < m; ++i) {
            int c = P.cb_of_arc[i];
            if (c < 0 || c >= m || hit[c]) ok = false;
            else hit[c] = 1;
        }
        if (!ok) {
            P.perm = 0;
            for (int i = 0; i < m; ++i) P.cb_of_arc[i] = m - 1 - i;
        }
    }
    P.identity = true;  // the paper's backward order: arc i on counter bit m - 1 - i
    for (int i = 0; i < m; ++i)
        if (P.cb_of_arc[i] != m - 1 - i) P.identity = false;
    P.row.assign(std::max(m, 1), 0);
    for (int i = 0; i < m; ++i) P.row[m - 1 - P.cb_of_arc[i]] = (unsigned char)i;
    P.ru.clear(); P.rv.clear(); P.rb.clear(); P.rd.clear();
    for (size_t k = 0; k < rel_bfs.size(); ++k) {
        P.ru.push_back(ends[k].first);
        P.rv.push_back(ends[k].second);
        P.rb.push_back(P.cb_of_arc[rel_bfs[k]]);
        P.rd.push_back(disc_flag[k]);
    }
    P.N = (int)order.size();
    P.S = 0;
    P.T = id[t];
    P.code.resize(P.ru.size());
    P.wconst.resize(P.ru.size());
    for (size_t k = 0; k < P.ru.size(); ++k) {
        P.code[k] = (u32)P.ru[k] | ((u32)P.rv[k] << 6) | ((u32)P.rb[k] << 12);
        P.wconst[k] = P.rb[k] < bat::kSliceBits ? bat::slice_pattern(P.rb[k]) : 0u;
    }
    // the generic kernel's program: (code, pattern) pairs in sweep order,
    // each direction padded to whole groups of 4 with (0, 0), which relaxes
    // node 0 against itself with an empty mask (a no-op)
    {
        const size_t nr = P.code.size(), ng = (nr + 3) / 4;
        P.prog.assign(2 * ng * 8 + 8, 0u);  // + the spare group read ahead of the last
        for (size_t k = 0; k < nr; ++k) {
            P.prog[2 * k] = P.code[k];
            P.prog[2 * k + 1] = P.wconst[k];
            const size_t kb = nr - 1 - k;  // backward sweep position of relaxation k
            P.prog[ng * 8 + 2 * kb] = P.code[k];
            P.prog[ng * 8 + 2 * kb + 1] = P.wconst[k];
        }
    }
    contract_series(n, m, arcs, s, t, rel, P);
    std::string sdesc = std::string(directed ? "D " : "") + "N" + std::to_string(P.jN) + " S" + std::to_string(P.jS) +
                        " T" + std::to_string(P.jT) + " m" + std::to_string(m) + " :";
    for (size_t k = 0; k < P.jru.size(); ++k)
        sdesc += " " + std::to_string(P.jru[k]) + "," + std::to_string(P.jrv[k]) + "," + std::to_string(P.jrb[k]) +
                 (P.jrb2[k] >= 0 ? "&" + std::to_string(P.jrb2[k]) : std::string()) + (P.jrd[k] ? "d" : "");
    P.structure = sdesc;
}

// Relaxation code of each chained counter bit 11 + b (b = 0..5), ~0 where
// that arc is pruned (no relaxation) or absent.
void chain_codes(const Plan &P, u32 out[6])
{
    for (int b = 0; b < 6; ++b) out[b] = ~0u;
    for (size_t k = 0; k < P.code.size(); ++k)
        if (P.rb[k] >= bat::kWordBits && P.rb[k] < bat::kWordBits + 6) out[P.rb[k] - bat::kWordBits] = P.code[k];
}

// ------------------------------------------------------------ device state
struct DeviceInfo {
    int id = -1;
    int cus = 0;
    int clock_khz = 0;  // of the device clock kernels read (wall_clock64)
    std::string arch;
};

int current_device(DeviceInfo &D)
{
    static std::mutex mu;
    static std::map<int, DeviceInfo> cache;
    int dev = 0;
    HIPCHK(hipGetDevice(&dev));
    std::lock_guard<std::mutex> lk(mu);
    auto it = cache.find(dev);
    if (it == cache.end()) {
        hipDeviceProp_t prop;
        HIPCHK(hipGetDeviceProperties(&prop, dev));
        DeviceInfo d;
        d.id = dev;
        d.cus = prop.multiProcessorCount;
        d.arch = prop.gcnArchName;
        HIPCHK(hipDeviceGetAttribute(&d.clock_khz, hipDeviceAttributeWallClockRate, dev));
        it = cache.emplace(dev, d).first;
    }
    D = it->second;
    return BAT_OK;
}

// Per thread and device: a device workspace and a pinned host staging
// buffer the synchronous calls reuse (grown, never shrunk), so a small call
// makes one host-to-device and one device-to-host copy and no allocation.
struct Scratch {
    char *dev = nullptr;
    size_t dev_cap = 0;
    char *host = nullptr;
    size_t host_cap = 0;
};

// What exiting threads leave behind, for later threads to take over. A
// thread's destructor makes no HIP call (the runtime may already be torn
// down at process exit), so its streams, events and scratch come here
// instead of being freed; the pool itself lives until the process ends.
// Side streams of a thread on one device, for launches that may overlap
// (the batched sweep's graph-specialised kernels), with the events that
// fork them from and join them to the thread's stream.
constexpr int kSideStreams = 4;
struct SideStreams {
    hipStream_t s[kSideStreams] = {};
    hipEvent_t fork = nullptr;
    hipEvent_t join[kSideStreams] = {};
};

// Where a thread's sub-cube sweeps report to (pinned host memory, never
// freed): the device clocks and sequence number of its last kDiagSlots
// asynchronous launches, then of its last synchronous one, [start, swept,
// done, seq] each.
constexpr u64 kDiagSlots = 16;
struct Diag {
    u64 *slots = nullptr;
    u64 seq = 0;
};

struct ResourcePool {
    std::mutex mu;
    std::vector<Diag> diag;
    std::multimap<int, hipStream_t> streams;
    std::multimap<int, Scratch> scratch;
    std::vector<std::vector<hipEvent_t>> events;
    std::multimap<int, SideStreams> side;
};
ResourcePool &pool()
{
    static ResourcePool *P = new ResourcePool;  // never destroyed
    return *P;
}

struct ThreadState {
    std::map<int, hipStream_t> streams;
    std::map<int, SideStreams> side;
    std::map<int, Scratch> scratch;
    hipEvent_t ev[4] = {nullptr, nullptr, nullptr, nullptr};
    Diag diag;
    bool have_launch = false;
    u64 cube_seq = 0;  // the last launch was this sub-cube sweep (0: another kernel)
    u64 *cube_slot = nullptr;  // which reports here (null: it was captured)
    hipStream_t cube_stream = nullptr;
    int cube_dev = 0, cube_khz = 0;
    bat_launch_info info{};
    ~ThreadState()
    {
        ResourcePool &P = pool();
        std::lock_guard<std::mutex> g(P.mu);
        for (auto &kv : streams) P.streams.emplace(kv.first, kv.second);
        for (auto &kv : side) P.side.emplace(kv.first, kv.second);
        for (auto &kv : scratch)
            if (kv.second.dev || kv.second.host) P.scratch.emplace(kv.first, kv.second);
        if (ev[0]) P.events.emplace_back(ev, ev + 4);
        if (diag.slots) P.diag.push_back(diag);
    }
};
thread_local ThreadState t_state;

int thread_stream(int dev, hipStream_t &s)
{
    auto it = t_state.streams.find(dev);
    if (it == t_state.streams.end()) {
        hipStream_t st = nullptr;
        {
            ResourcePool &P = pool();
            std::lock_guard<std::mutex> g(P.mu);
            auto pit = P.streams.find(dev);
            if (pit != P.streams.end()) {
                st = pit->second;
                P.streams.erase(pit);
            }
        }
        if (!st) HIPCHK(hipStreamCreateWithFlags(&st, hipStreamNonBlocking));
        it = t_state.streams.emplace(dev, st).first;
    }
    s = it->second;
    return BAT_OK;
}

int side_streams(int dev, SideStreams *&out)
{
    auto it = t_state.side.find(dev);
    if (it == t_state.side.end()) {
        SideStreams S;
        bool have = false;
        {
            ResourcePool &P = pool();
            std::lock_guard<std::mutex> g(P.mu);
            auto pit = P.side.find(dev);
            if (pit != P.side.end()) {
                S = pit->second;
                P.side.erase(pit);
                have = true;
            }
        }
        if (!have) {
            // default priority, like every stream of the library
            for (int k = 0; k < kSideStreams; ++k) HIPCHK(hipStreamCreateWithFlags(&S.s[k], hipStreamNonBlocking));
            HIPCHK(hipEventCreateWithFlags(&S.fork, hipEventDisableTiming));
            for (int k = 0; k < kSideStreams; ++k) HIPCHK(hipEventCreateWithFlags(&S.join[k], hipEventDisableTiming));
        }
        it = t_state.side.emplace(dev, S).first;
    }
    out = &it->second;
    return BAT_OK;
}

// Make the thread's scratch on device `dev` at least this large; growing
// waits for the stream first (the old buffers may still be in use).
int scratch_reserve(int dev, hipStream_t st, size_t dev_bytes, size_t host_bytes, Scratch *&S)
{
    auto sit = t_state.scratch.find(dev);
    if (sit == t_state.scratch.end()) {
        Scratch taken;
        {
            ResourcePool &P = pool();
            std::lock_guard<std::mutex> g(P.mu);
            auto pit = P.scratch.find(dev);
            if (pit != P.scratch.end()) {
                taken = pit->second;
                P.scratch.erase(pit);
            }
        }
        sit = t_state.scratch.emplace(dev, taken).first;
    }
    S = &sit->second;
    if (S->dev_cap < dev_bytes) {
        HIPCHK(hipStreamSynchronize(st));
        if (S->dev) HIPCHK(hipFree(S->dev));
        S->dev = nullptr;
        S->dev_cap = 0;
        const size_t cap = std::max<size_t>(dev_bytes, 1 << 20);
        HIPCHK(hipMalloc((void **)&S->dev, cap));
        S->dev_cap = cap;
    }
    if (S->host_cap < host_bytes) {
        HIPCHK(hipStreamSynchronize(st));
        if (S->host) HIPCHK(hipHostFree(S->host));
        S->host = nullptr;
        S->host_cap = 0;
        const size_t cap = std::max<size_t>(host_bytes, 64 << 10);
        HIPCHK(hipHostMalloc((void **)&S->host, cap, hipHostMallocDefault));
        S->host_cap = cap;
    }
    return BAT_OK;
}

int events_ready()
{
    if (!t_state.ev[0]) {
        {
            ResourcePool &P = pool();
            std::lock_guard<std::mutex> g(P.mu);
            if (!P.events.empty()) {
                for (int i = 0; i < 4; ++i) t_state.ev[i] = P.events.back()[i];
                P.events.pop_back();
            }
        }
        if (!t_state.ev[0])
            for (auto &e : t_state.ev) HIPCHK(hipEventCreate(&e));
    }
    return BAT_OK;
}

// The next launch's report slot (null: `stream` is being captured; a replay
// could write to the slot at any time).  Synchronous calls, which wait on
// theirs, have one that no launch still running can write to.  A call that
// must allocate nothing has none (null) on a thread without slots.
enum class Report { sync, async, noalloc };
int diag_next(hipStream_t stream, u64 *&slot, u64 &seq, Report kind, bool *captured = nullptr)
{
    Diag &G = t_state.diag;
    if (!G.slots) {
        ResourcePool &P = pool();
        std::lock_guard<std::mutex> g(P.mu);
        if (!P.diag.empty()) {
            G = P.diag.back();
            P.diag.pop_back();
        }
    }
    slot = nullptr;
    if (captured) *captured = false;
    if (kind != Report::sync && stream) {
        hipStreamCaptureStatus cs = hipStreamCaptureStatusNone;
        HIPCHK(hipStreamIsCapturing(stream, &cs));
        if (cs != hipStreamCaptureStatusNone) {
            if (captured) *captured = true;
            return BAT_OK;
        }
    }
    if (!G.slots) {
        if (kind == Report::noalloc) return BAT_OK;
        void *h = nullptr;
        HIPCHK(hipHostMalloc(&h, sizeof(u64) * 4 * (kDiagSlots + 1), hipHostMallocDefault));
        memset(h, 0, sizeof(u64) * 4 * (kDiagSlots + 1));
        G.slots = (u64 *)h;
    }
    seq = ++G.seq;
    slot = G.slots + 4 * (kind == Report::sync ? kDiagSlots : seq % kDiagSlots);
    return BAT_OK;
}

bool diag_done(const u64 *slot, u64 seq) { return __atomic_load_n(slot + 3, __ATOMIC_ACQUIRE) == seq; }

// ------------------------------------------------- fixed device scratch
// The workspace of bat_reliability_noalloc: a fixed array in device memory,
// one copy per GPU the library runs on, held until the process ends.  In
// host code `scratch` names the symbol, not a device address: the address
// of a GPU's copy comes from hipGetSymbolAddress with that GPU current, once
// per device, and only that address is passed to kernels and copies.
constexpr size_t kNoAllocScratchBytes = BAT_NOALLOC_SCRATCH_BYTES;
static __device__ __align__(256) char scratch[kNoAllocScratchBytes];

int noalloc_scratch(int dev, char *&ptr)
{
    static std::mutex mu;
    static std::map<int, char *> addr;  // device -> its copy of `scratch`
    std::lock_guard<std::mutex> lk(mu);
    auto it = addr.find(dev);
    if (it == addr.end()) {
        void *a = nullptr;
        HIPCHK(hipGetSymbolAddress(&a, HIP_SYMBOL(scratch)));
        if (!a) return fail(BAT_EDEVICE, "no device address for the fixed scratch on device %d", dev);
        it = addr.emplace(dev, (char *)a).first;
    }
    ptr = it->second;
    return BAT_OK;
}

// ------------------------------------------------------------ JIT cache
struct JitEntry {
    hipModule_t mod = nullptr;
    hipFunction_t fn = nullptr;
    uint64_t id = 0;  // hash of the compiled code object
};
std::mutex g_jit_mu;
std::map<std::string, JitEntry> g_jit;

// Drop every compiled kernel of this process (modules unloaded) after the
// current device has finished its work.
// Code objects compiled before their first launch (the autotuner compiles
// its candidates' kernels side by side), by the key of their source text.
std::mutex g_pre_mu;
std::map<std::pair<uint64_t, uint64_t>, std::vector<char>> g_precompiled;

void jit_flush()
{
    (void)hipDeviceSynchronize();
    {
        std::lock_guard<std::mutex> lk(g_pre_mu);
        g_precompiled.clear();
    }
    std::lock_guard<std::mutex> lk(g_jit_mu);
    for (auto &kv : g_jit)
        if (kv.second.mod) (void)hipModuleUnload(kv.second.mod);
    g_jit.clear();
}

// ---------------------------------------------------- on-disk code cache
// Compiled code objects are kept across processes, keyed by two
// independent 64-bit hashes of the whole source text, the target and the
// compile options, so a changed kernel is never served stale.  Directory:
// BAT_JIT_CACHE_DIR, else $XDG_CACHE_HOME/bat-mi355x, else
// $HOME/.cache/bat-mi355x; BAT_JIT_CACHE=0 turns it off.  Anything that
// fails to read, write or load falls back to compiling.
struct CacheKey {
    uint64_t h1, h2, len;
};
CacheKey cache_key(const std::string &text)
{
    uint64_t a = 1469598103934665603ull, b = 0x9E3779B97F4A7C15ull;
    for (unsigned char c : text) {
        a = (a ^ c) * 1099511628211ull;           // FNV-1a
        b = (b + c) * 0xBF58476D1CE4E5B9ull;       // multiply-add, then mix
        b ^= b >> 31;
    }
    return {a, b, (uint64_t)text.size()};
}
// Identity of a code object's machine code: a hash of its .text and
// .rodata sections. The rest of the object varies between compilations of
// the same source (the compilation-unit id symbol), the code does not. A
// blob that does not parse as a 64-bit ELF is hashed whole.
uint64_t machine_code_id(const std::vector<char> &co)
{
    const size_t n = co.size();
    auto rd = [&](size_t off, size_t len, uint64_t &v) {
        if (off + len > n) return false;
        v = 0;
        for (size_t i = 0; i < len; ++i) v |= (uint64_t)(unsigned char)co[off + i] << (8 * i);
        return true;
    };
    uint64_t shoff = 0, shentsize = 0, shnum = 0, shstrndx = 0;
    const bool elf = n > 64 && co[0] == 0x7f && co[1] == 'E' && co[2] == 'L' && co[3] == 'F' && co[4] == 2 &&
                     rd(0x28, 8, shoff) && rd(0x3A, 2, shentsize) && rd(0x3C, 2, shnum) && rd(0x3E, 2, shstrndx) &&
                     shentsize >= 64 && shstrndx < shnum && shoff + shnum * shentsize <= n;
    if (!elf) return cache_key(std::string(co.begin(), co.end())).h1;
    uint64_t stroff = 0;
    if (!rd(shoff + shstrndx * shentsize + 0x18, 8, stroff)) return cache_key(std::string(co.begin(), co.end())).h1;
    std::string text;
    for (uint64_t i = 0; i < shnum; ++i) {
        const size_t h = shoff + i * shentsize;
        uint64_t name = 0, type = 0, off = 0, size = 0;
        if (!rd(h, 4, name) || !rd(h + 4, 4, type) || !rd(h + 0x18, 8, off) || !rd(h + 0x20, 8, size)) continue;
        if (type == 8 || off + size > n || stroff + name >= n) continue;  // no bits in the file
        const char *nm = co.data() + stroff + name;
        const size_t room = n - (stroff + name);
        if (strnlen(nm, room) == room) continue;
        if (!strcmp(nm, ".text") || !strcmp(nm, ".rodata")) text.append(co.data() + off, size);
    }
    if (text.empty()) return cache_key(std::string(co.begin(), co.end())).h1;
    return cache_key(text).h1;
}

// Identity of an ahead-of-time kernel instance: the digest of the sources
// it was compiled from, the kernel and its node-count class.
uint64_t aot_kernel_id(const char *kernel, int nodes, bool directed)
{
    const int nmax = nodes <= 16 ? 16 : nodes <= 32 ? 32 : 64;
    return cache_key(std::string(kAotKernelDigest) + " " + kernel + " " + std::to_string(nmax) +
                     (directed ? " directed" : ""))
        .h1;
}

std::string cache_dir()
{
    const char *on = getenv("BAT_JIT_CACHE");
    if (on && !strcmp(on, "0")) return "";
    std::string d;
    if (const char *e = getenv("BAT_JIT_CACHE_DIR"); e && *e) {
        d = e;
    } else if (const char *x = getenv("XDG_CACHE_HOME"); x && *x) {
        d = std::string(x) + "/bat-mi355x";
    } else if (const char *h = getenv("HOME"); h && *h) {
        d = std::string(h) + "/.cache";
        mkdir(d.c_str(), 0755);
        d += "/bat-mi355x";
    } else {
        return "";
    }
    mkdir(d.c_str(), 0755);  // may exist already
    struct stat st;
    if (stat(d.c_str(), &st) != 0 || !S_ISDIR(st.st_mode)) return "";
    return d;
}
std::string cache_path(const std::string &dir, const CacheKey &k)
{
    char name[64];
    snprintf(name, sizeof name, "/%016llx.co", (unsigned long long)k.h1);
    return dir + name;
}
constexpr char kCacheMagic[8] = {'B', 'A', 'T', 'J', 'I', 'T', '1', '\n'};
bool cache_read(const std::string &path, const CacheKey &k, std::vector<char> &code)
{
    FILE *f = fopen(path.c_str(), "rb");
    if (!f) return false;
    char magic[8];
    uint64_t hdr[3], n = 0;
    bool ok = fread(magic, 1, 8, f) == 8 && !memcmp(magic, kCacheMagic, 8) && fread(hdr, 8, 3, f) == 3 &&
              hdr[0] == k.h1 && hdr[1] == k.h2 && hdr[2] == k.len && fread(&n, 8, 1, f) == 1 && n > 0 &&
              n < (1ull << 30);
    if (ok) {
        code.resize(n);
        ok = fread(code.data(), 1, n, f) == n;
    }
    fclose(f);
    return ok;
}
void cache_write(const std::string &path, const CacheKey &k, const std::vector<char> &code)
{
    const std::string tmp = path + ".tmp" + std::to_string((long long)getpid());
    FILE *f = fopen(tmp.c_str(), "wb");
    if (!f) return;
    const uint64_t hdr[4] = {k.h1, k.h2, k.len, (uint64_t)code.size()};
    bool ok = fwrite(kCacheMagic, 1, 8, f) == 8 && fwrite(hdr, 8, 4, f) == 4 &&
              fwrite(code.data(), 1, code.size(), f) == code.size();
    ok = (fclose(f) == 0) && ok;
    if (!ok || rename(tmp.c_str(), path.c_str()) != 0) unlink(tmp.c_str());
}

// Launch shape of a specialised kernel: wavefronts per block and whether
// forward sweeps keep super-block bottoms in LDS.  The gradient sweep
// always runs 4 wavefronts per block and no super-block store.
struct JitShape {
    int waves = bat::kWavesPerBlock;
    bool super_restart = false;
    int simd_waves = 0;  // > 0: ask the compiler to fit this many wavefronts per SIMD
    bool keep_bottom = true;  // chain starts resume from the kept block bottom
    bool bottom_lds = false;  // ... kept in LDS instead of registers
};

// Default shape of the forward sweep: 4 wavefronts per block, kept block
// bottoms, no super-block store, compiled to fit 6 wavefronts per SIMD.
// The kernel is latency-bound: on the 5x5 grid, fitting 6 wavefronts (80
// registers, spills outside the innermost loops) instead of the compiler's
// 4 (109 registers) takes the sweep from 161 to 141 ms.  Bigger plans
// spill inside the sweeps at that budget but still gained (a 29-word
// plan: 11.6 ms against 13.5 ms with the compiler's budget).
constexpr int kDefaultSimdWaves = 6;

// waves: 1, 2 or 4 (anything else: 4); super_restart: 1 on, else off;
// simd_waves: 5 to 8, 0 = the compiler's own register budget, else the
// default; keep_bottom: 0 off, else on
JitShape jit_shape(bool grad, int waves, int super_restart, int simd_waves, int keep_bottom)
{
    JitShape sh;
    if (grad) {
        // the gradient sweep of a graph of up to kGradThreeWaveNodes nodes
        // fits 3 wavefronts per SIMD without spilling; on the 36-arc random
        // graph 4 (128 registers, spilling) took 32 ms against 20 ms
        sh.simd_waves = 3;
        // the gradient's registers are full: a kept bottom lives in LDS
        sh.keep_bottom = opts().grad_keep_bottom.load() == 2;
        sh.bottom_lds = sh.keep_bottom;
    } else {
        sh.keep_bottom = keep_bottom != 0;
        sh.bottom_lds = keep_bottom == 2;
        sh.waves = waves == 1 ? 1 : waves == 2 ? 2 : 4;
        sh.super_restart = super_restart == 1;
        sh.simd_waves = (simd_waves >= 5 && simd_waves <= 8) ? simd_waves : simd_waves == 0 ? 0 : kDefaultSimdWaves;
    }
    return sh;
}

// batch_np > 0: instead of the forward or gradient sweep, the batched
// sweep of batch_np probability vectors, in blocks of batch_jit_waves
// wavefronts: 3 per SIMD (168 registers) keep the sweep loops free of
// spills up to 16 p-vectors, beyond that 2 per SIMD (256 registers); at 3
// per SIMD 32 accumulators spill inside the sweeps
constexpr int batch_jit_waves(int np) { return np > 16 ? 8 : 12; }
// the transposed accumulation (option BAT_BATCH_ACC 1, 9..32 p-vectors:
// two lanes per p-vector above 16, else four): one accumulator per lane,
// blocks of kBatchTWaves wavefronts
constexpr int kBatchTWaves = 16;
static_assert(kBatchTWaves <= bat::kBatchTMaxWaves, "one LDS row per wavefront");
bool batch_transposed(int np) { return np > 8 && np <= bat::kBatchCols && opts().batch_acc.load() == 1; }
int batch_waves(int np) { return batch_transposed(np) ? kBatchTWaves : batch_jit_waves(np); }
// p-vectors per specialised entry: 32 (blocks of 8 wavefronts) measured
// faster than two entries of 16 (blocks of 12) on 256 graphs x 32
// p-vectors, 18.7 against 19.4 ms: the closure then runs once
constexpr int kBatchSpecP = 32;

std::string jit_source(const Plan &P, bool grad, const JitShape &sh, int batch_np = 0)
{
    std::string s;
    s.reserve(strlen(kDeviceSource) + 4096);
    s += kDeviceSource;
    s += "\nstruct JitGraph {\n";
    s += "  static constexpr int N = " + std::to_string(P.jN) + ";\n";
    s += "  static constexpr int S = " + std::to_string(P.jS) + ";\n";
    s += "  static constexpr int T = " + std::to_string(P.jT) + ";\n";
    size_t nr = P.jru.size();
    s += "  static constexpr int NR = " + std::to_string(nr) + ";\n";
    auto arr = [&](const char *name, const std::vector<int> &v) {
        s += std::string("  static constexpr unsigned char ") + name + "[" + std::to_string(nr ? nr : 1) + "] = {";
        if (nr == 0) s += "0";
        for (size_t k = 0; k < nr; ++k) s += (k ? "," : "") + std::to_string(v[k]);
        s += "};\n";
    };
    arr("RU", P.jru);
    arr("RV", P.jrv);
    arr("RB", P.jrb);
    arr("RD", P.jrd);
    // second counter bit of a relaxation that joins two arcs in series
    // (255: one arc)
    {
        std::vector<int> b2(nr);
        for (size_t k = 0; k < nr; ++k) b2[k] = P.jrb2[k] < 0 ? 255 : P.jrb2[k];
        arr("RB2", b2);
    }
    s += std::string("  static constexpr bool DIR = ") + (P.directed ? "true" : "false") + ";\n";
    // forward sweeps of graphs small enough for the LDS store (4 blocks of
    // 4 wavefronts per CU keep (N + 2) words per lane each) also resume
    // block bottoms from the kept bottom of their 2^6-aligned super-block
    s += std::string("  static constexpr bool SUPER = ") +
         (!grad && sh.super_restart && P.jN <= kSuperMaxNodes ? "true" : "false") + ";\n";
    // wavefronts per block (the launch uses the same)
    s += "  static constexpr int WAVES = " + std::to_string(sh.waves) + ";\n";
    s += std::string("  static constexpr bool KEEPB = ") + (sh.keep_bottom ? "true" : "false") + ";\n";
    s += std::string("  static constexpr bool BOTTOM_LDS = ") + (sh.bottom_lds ? "true" : "false") + ";\n";
    // relaxations of counter bits 11..16 (the chained iteration arcs)
    int ck[6] = {-1, -1, -1, -1, -1, -1};
    for (size_t k = 0; k < nr; ++k)
        for (int b : {P.jrb[k], P.jrb2[k]})
            if (b >= bat::kWordBits && b < bat::kWordBits + 6) ck[b - bat::kWordBits] = (int)k;
    s += "  static constexpr int CK[6] = {";
    for (int b = 0; b < 6; ++b) s += (b ? "," : "") + std::to_string(ck[b]);
    s += "};\n";
    s += "};\n";
    // the gradient sweep of a small graph fits three wavefronts per SIMD
    // with spills confined to once-per-segment code; larger graphs keep the
    // compiler's register budget
    if (grad && P.jN <= kGradThreeWaveNodes && sh.simd_waves)
        s += "extern \"C\" __global__ void __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(" +
             std::to_string(sh.simd_waves) + ", " + std::to_string(sh.simd_waves) + ")))\n"
             "bat_grad_jit(bat::KParams P) {\n"
             "  __shared__ bat::LdsTables L; __shared__ bat::LdsGrad LG;\n"
             "  bat::sweep_kernel<bat::StaticClosure<JitGraph>, true>(P, L, &LG);\n}\n";
    else if (batch_np > 0 && batch_transposed(batch_np))
        s += "extern \"C\" __global__ void __launch_bounds__(" + std::to_string(bat::kWave * kBatchTWaves) +
             ") bat_batch_jit(bat::KParams P) {\n"
             "  __shared__ bat::LdsBatchT<" + std::to_string(batch_np) + "> L;\n"
             "  bat::batch_kernel_t<bat::StaticClosure<JitGraph>, " + std::to_string(batch_np) + ">(P, L);\n}\n";
    else if (batch_np > 0)
        s += "extern \"C\" __global__ void __launch_bounds__(" + std::to_string(bat::kWave * batch_jit_waves(batch_np)) +
             ") bat_batch_jit(bat::KParams P) {\n"
             "  __shared__ bat::LdsBatch<" + std::to_string(batch_np) + "> L;\n"
             "  bat::batch_kernel<bat::StaticClosure<JitGraph>, " + std::to_string(batch_np) + ">(P, L);\n}\n";
    else if (grad)
        s += "extern \"C\" __global__ void __launch_bounds__(256) bat_grad_jit(bat::KParams P) {\n"
             "  __shared__ bat::LdsTables L; __shared__ bat::LdsGrad LG;\n"
             "  bat::sweep_kernel<bat::StaticClosure<JitGraph>, true>(P, L, &LG);\n}\n";
    else
        s += "extern \"C\" __global__ void __launch_bounds__(" + std::to_string(bat::kWave * sh.waves) + ")" +
             (sh.simd_waves ? " __attribute__((amdgpu_waves_per_eu(" + std::to_string(sh.simd_waves) + ", " +
                                  std::to_string(sh.simd_waves) + ")))"
                            : std::string()) +
             " bat_fwd_jit(bat::KParams P) {\n"
             "  __shared__ bat::LdsTables L;\n"
             "  bat::sweep_kernel<bat::StaticClosure<JitGraph>, false>(P, L, nullptr);\n}\n";
    return s;
}

// One hiprtc compilation of a specialised kernel's source (no shared state:
// several may run at once on host threads).
const char *const kJitOpts[] = {"-O3", "-std=c++17", "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops"};

std::string jit_key_text(const std::string &src, const std::string &arch)
{
    std::string keytext = src;
    keytext += "\n//--offload-arch=" + arch;
    for (const char *opt : kJitOpts) keytext += std::string("\n//") + opt;
    return keytext;
}

bool jit_compile(const std::string &src, const std::string &arch, std::vector<char> &code, std::string &err)
{
    const std::string a = "--offload-arch=" + arch;
    std::vector<const char *> o{a.c_str()};
    for (const char *opt : kJitOpts) o.push_back(opt);
    hiprtcProgram prog;
    if (hiprtcCreateProgram(&prog, src.c_str(), "bat_jit.hip", 0, nullptr, nullptr) != HIPRTC_SUCCESS) {
        err = "hiprtcCreateProgram failed";
        return false;
    }
    hiprtcResult rc = hiprtcCompileProgram(prog, (int)o.size(), o.data());
    if (rc != HIPRTC_SUCCESS) {
        size_t ls = 0;
        hiprtcGetProgramLogSize(prog, &ls);
        std::string log(ls + 1, '\0');
        hiprtcGetProgramLog(prog, &log[0]);
        hiprtcDestroyProgram(&prog);
        err = std::string(hiprtcGetErrorString(rc)) + ": " + log.substr(0, 800);
        return false;
    }
    size_t sz = 0;
    hiprtcGetCodeSize(prog, &sz);
    code.assign(sz, 0);
    hiprtcGetCode(prog, code.data());
    hiprtcDestroyProgram(&prog);
    return true;
}

// The compile helper (bat_jitc) installed beside this library, or "".
std::string jitc_path()
{
    Dl_info di;
    if (!dladdr((const void *)&jitc_path, &di) || !di.dli_fname) return "";
    std::string p = di.dli_fname;
    const size_t slash = p.rfind('/');
    p = (slash == std::string::npos ? std::string(".") : p.substr(0, slash)) + "/bat_jitc";
    return access(p.c_str(), X_OK) == 0 ? p : "";
}

// The file of the hiprtc library this process compiles with, or "".
std::string hiprtc_path()
{
    Dl_info di;
    if (!dladdr((const void *)&hiprtcCompileProgram, &di) || !di.dli_fname) return "";
    return di.dli_fname;
}

// Compile the kernels of these sources that are neither precompiled nor
// on disk.  hiprtc runs one compilation at a time per process, so they run
// in child processes of the compile helper, up to option BAT_JIT_PROCS at
// once; their first launch then only loads the code.  Whatever does not
// come back (no helper, a failed child) is compiled in-process by that
// launch as usual.
void jit_precompile_sources(const DeviceInfo &D, const std::vector<std::string> &sources);

// The same for the kernels of these (plan, gradient?, shape) launches.
void jit_precompile(const DeviceInfo &D, const std::vector<std::tuple<const Plan *, bool, JitShape>> &want)
{
    std::vector<std::string> sources;
    for (const auto &w : want) sources.push_back(jit_source(*std::get<0>(w), std::get<1>(w), std::get<2>(w)));
    jit_precompile_sources(D, sources);
}

void jit_precompile_sources(const DeviceInfo &D, const std::vector<std::string> &sources)
{
    const int64_t procs = std::min<int64_t>(opts().jit_procs.load(), 64);
    if (procs < 1) return;
    const std::string helper = jitc_path(), rtc = hiprtc_path();
    if (helper.empty() || rtc.empty()) return;
    struct Job {
        std::string src;
        CacheKey ck;
        std::string src_path, out_path;
        pid_t pid = -1;
    };
    std::vector<Job> jobs;
    const std::string cdir = cache_dir();
    for (const std::string &src : sources) {
        Job j;
        j.src = src;
        j.ck = cache_key(jit_key_text(j.src, D.arch));
        {
            std::lock_guard<std::mutex> lk(g_pre_mu);
            if (g_precompiled.count({j.ck.h1, j.ck.h2})) continue;
        }
        if (!cdir.empty()) {
            struct stat st;
            if (stat(cache_path(cdir, j.ck).c_str(), &st) == 0) continue;  // on disk already
        }
        bool dup = false;
        for (const Job &o : jobs) dup = dup || (o.ck.h1 == j.ck.h1 && o.ck.h2 == j.ck.h2);
        if (!dup) jobs.push_back(std::move(j));
    }
    if (jobs.empty()) return;
    const char *tenv = getenv("TMPDIR");
    std::string dir = std::string(tenv && *tenv ? tenv : "/tmp") + "/bat_jitc.XXXXXX";
    if (!mkdtemp(&dir[0])) return;
    const std::string arch = "--offload-arch=" + D.arch;
    for (size_t i0 = 0; i0 < jobs.size(); i0 += (size_t)procs) {
        const size_t i1 = std::min(jobs.size(), i0 + (size_t)procs);
        for (size_t i = i0; i < i1; ++i) {
            Job &j = jobs[i];
            j.src_path = dir + "/" + std::to_string(i) + ".hip";
            j.out_path = dir + "/" + std::to_string(i) + ".co";
            FILE *f = fopen(j.src_path.c_str(), "wb");
            if (!f) continue;
            const bool ok = fwrite(j.src.data(), 1, j.src.size(), f) == j.src.size();
            if (fclose(f) != 0 || !ok) continue;
            std::vector<char *> argv{(char *)helper.c_str(), (char *)rtc.c_str(), (char *)j.src_path.c_str(),
                                     (char *)j.out_path.c_str(), (char *)arch.c_str()};
            for (const char *opt : kJitOpts) argv.push_back((char *)opt);
            argv.push_back(nullptr);
            pid_t pid;
            if (posix_spawn(&pid, helper.c_str(), nullptr, nullptr, argv.data(), environ) == 0) j.pid = pid;
        }
        for (size_t i = i0; i < i1; ++i) {
            Job &j = jobs[i];
            if (j.pid > 0) {
                int st = 0;
                pid_t r;
                while ((r = waitpid(j.pid, &st, 0)) < 0 && errno == EINTR) {
                }
                std::vector<char> code;
                if (r == j.pid && WIFEXITED(st) && WEXITSTATUS(st) == 0) {
                    if (FILE *f = fopen(j.out_path.c_str(), "rb")) {
                        char buf[1 << 16];
                        size_t k;
                        while ((k = fread(buf, 1, sizeof buf, f)) > 0) code.insert(code.end(), buf, buf + k);
                        fclose(f);
                    }
                }
                if (!code.empty()) {
                    if (!cdir.empty()) cache_write(cache_path(cdir, j.ck), j.ck, code);
                    std::lock_guard<std::mutex> lk(g_pre_mu);
                    g_precompiled[{j.ck.h1, j.ck.h2}] = std::move(code);
                }
            }
            unlink(j.src_path.c_str());
            unlink(j.out_path.c_str());
        }
    }
    rmdir(dir.c_str());
}

// A kernel loaded before, without the text of its source.
bool jit_ready(const std::string &key, hipFunction_t &fn, uint64_t &id)
{
    std::lock_guard<std::mutex> lk(g_jit_mu);
    auto it = g_jit.find(key);
    if (it == g_jit.end()) return false;
    fn = it->second.fn;
    id = it->second.id;
    return true;
}

// The kernel `kname` of source `src`, loaded once per process under `key`:
// from the precompiled table, else the disk cache, else compiled here.
int jit_load(const DeviceInfo &D, const std::string &key, const std::string &src, const char *kname,
             hipFunction_t &fn, double &compile_ms, uint64_t &id)
{
    compile_ms = 0.0;
    std::lock_guard<std::mutex> lk(g_jit_mu);
    auto it = g_jit.find(key);
    if (it != g_jit.end()) {
        fn = it->second.fn;
        id = it->second.id;
        return BAT_OK;
    }
    auto t0 = std::chrono::steady_clock::now();
    const CacheKey ck = cache_key(jit_key_text(src, D.arch));
    const std::string cdir = cache_dir();
    std::vector<char> code;
    // the kernel's identity: its machine code, so that edits which leave
    // the code alone (comments) keep it
    auto code_id = [&]() { return machine_code_id(code); };
    bool pre = false;
    {
        std::lock_guard<std::mutex> lk2(g_pre_mu);
        auto pit = g_precompiled.find({ck.h1, ck.h2});
        if (pit != g_precompiled.end()) {
            code = std::move(pit->second);
            g_precompiled.erase(pit);
            pre = true;
        }
    }
    if (!pre && !cdir.empty() && cache_read(cache_path(cdir, ck), ck, code)) {
        JitEntry e;
        e.id = id = code_id();
        if (hipModuleLoadData(&e.mod, code.data()) == hipSuccess && hipModuleGetFunction(&e.fn, e.mod, kname) == hipSuccess) {
            g_jit.emplace(key, e);
            fn = e.fn;
            compile_ms = std::chrono::duration<double, std::milli>(std::chrono::steady_clock::now() - t0).count();
            return BAT_OK;
        }
        if (e.mod) (void)hipModuleUnload(e.mod);
        (void)hipGetLastError();  // a stale or damaged entry: compile afresh
    }
    if (!pre) {
        std::string err;
        if (!jit_compile(src, D.arch, code, err)) return fail(BAT_EDEVICE, "hiprtc compile failed (%s)", err.c_str());
        if (!cdir.empty()) cache_write(cache_path(cdir, ck), ck, code);
    }
    JitEntry e;
    e.id = id = code_id();
    HIPCHK(hipModuleLoadData(&e.mod, code.data()));
    HIPCHK(hipModuleGetFunction(&e.fn, e.mod, kname));
    g_jit.emplace(key, e);
    fn = e.fn;
    compile_ms = std::chrono::duration<double, std::milli>(std::chrono::steady_clock::now() - t0).count();
    return BAT_OK;
}

int jit_get(const DeviceInfo &D, const Plan &P, bool grad, const JitShape &sh, hipFunction_t &fn, double &compile_ms,
            uint64_t &id)
{
    compile_ms = 0.0;
    const std::string key = std::to_string(D.id) + (grad ? " grad " : " fwd ") + std::to_string(sh.waves) +
                            (sh.super_restart ? "s" : "") + (sh.keep_bottom ? (sh.bottom_lds ? "K" : "k") : "") + "/" +
                            std::to_string(sh.simd_waves) + " " + P.structure;
    {
        std::lock_guard<std::mutex> lk(g_jit_mu);
        auto it = g_jit.find(key);
        if (it != g_jit.end()) {
            fn = it->second.fn;
            id = it->second.id;
            return BAT_OK;
        }
    }
    return jit_load(D, key, jit_source(P, grad, sh), grad ? "bat_grad_jit" : "bat_fwd_jit", fn, compile_ms, id);
}

// ------------------------------------------------------------ autotune cache
struct TuneChoice {
    int chunk_log2, check_every, jit, perm, chain = -1, order = -1;
    // specialised forward launch shape (-1: default)
    int waves = -1, super_restart = -1, simd_waves = -1, keep_bottom = -1;
};
std::mutex g_tune_mu;
std::map<std::string, TuneChoice> g_tune;

// The graph itself (node count, arcs, terminals): what tuned choices are
// remembered under.
std::string graph_key(int32_t n, int32_t m, const bat_arc *arcs, int32_t s, int32_t t, bool directed = false)
{
    std::string k = std::string(directed ? "D" : "") + std::to_string(n) + "/" + std::to_string(s) + "/" +
                    std::to_string(t) + ":";
    for (int32_t i = 0; i < m; ++i) k += std::to_string(arcs[i].u) + "-" + std::to_string(arcs[i].v) + ",";
    return k;
}

// ------------------------------------------------------------ the sweep
struct Request {
    int32_t n, m, s, t;
    const bat_arc *arcs;
    const double *p_dev;    // device probabilities
    u64 c_lo, c_hi;
    bool grad;
    // forced knobs (autotuner); -1 = from options / the tuned choice
    int force_chunk_log2 = -1, force_check = -1, force_jit = -1, force_perm = -1, force_chain = -1,
        force_order = -1, force_waves = -1, force_super = -1, force_simd = -1, force_keep = -1;
    // timing sample (autotuner): sweep only this many work items, spread
    // over the whole counter by an odd multiplier (0 = everything)
    u64 sample_items = 0;
    // a part of the counter, or the first part of a split sweep: work items
    // no larger than fill_item_log2's size
    bool fill = false;
    // one part of a whole sweep split into split_parts (a power of two):
    // part split_index (0 = no split)
    u64 split_parts = 0, split_index = 0;
};

// Options, then the tuned choice for this graph (if any and enabled), then
// what the request forces.
TuneChoice choose(const DeviceInfo &D, const std::string &gkey, bool grad, const Request *rq)
{
    Options &O = opts();
    TuneChoice tc{(int)O.chunk_log2.load(), (int)O.check_every.load(), (int)O.jit.load(), -1};
    if (O.autotune.load()) {
        std::lock_guard<std::mutex> lk(g_tune_mu);
        auto it = g_tune.find(std::to_string(D.id) + (grad ? " grad " : " fwd ") + gkey);
        if (it != g_tune.end()) tc = it->second;
    }
    if (O.perm.load() >= 0) tc.perm = (int)O.perm.load();
    if (O.chain_log2.load() >= 0) tc.chain = (int)O.chain_log2.load();
    if (O.item_order.load() >= 0) tc.order = (int)O.item_order.load();
    if (O.block_waves.load() >= 0) tc.waves = (int)O.block_waves.load();
    if (O.super_restart.load() >= 0) tc.super_restart = (int)O.super_restart.load();
    if (O.simd_waves.load() >= 0) tc.simd_waves = (int)O.simd_waves.load();
    if (O.keep_bottom.load() >= 0) tc.keep_bottom = (int)O.keep_bottom.load();
    if (rq) {
        if (rq->force_chunk_log2 >= 0) tc.chunk_log2 = rq->force_chunk_log2;
        if (rq->force_check >= 0) tc.check_every = rq->force_check;
        if (rq->force_jit >= 0) tc.jit = rq->force_jit;
        if (rq->force_perm >= 0) tc.perm = rq->force_perm;
        if (rq->force_chain >= 0) tc.chain = rq->force_chain;
        if (rq->force_order >= 0) tc.order = rq->force_order;
        if (rq->force_waves >= 0) tc.waves = rq->force_waves;
        if (rq->force_super >= 0) tc.super_restart = rq->force_super;
        if (rq->force_simd >= 0) tc.simd_waves = rq->force_simd;
        if (rq->force_keep >= 0) tc.keep_bottom = rq->force_keep;
    }
    return tc;
}

struct Launch {
    void *ws = nullptr;     // workspace (stream-ordered; null when the thread's scratch is used)
    double *res = nullptr;  // [ncol][2]
    u64 *count = nullptr;
    int *status = nullptr;
    const unsigned char *cb_of_arc = nullptr;
    u32 ncol = 1;
    // the output block res | count | status, contiguous in the workspace,
    // and where its host copy goes in the thread's staging buffer
    const char *out_dev = nullptr;
    size_t out_bytes = 0, out_host_off = 0;
};

size_t align_up(size_t x, size_t a) { return (x + a - 1) / a * a; }

// Work-item size (log2 iterations) for `iters` iterations in `parts` launches
// (0 or 1: one): ~256 work items per CU per launch, so that the last,
// partly idle round of items is a small share of a launch, but at most 4096
// and, for one launch where the sweep has that many, at least 32 iterations
// per item (a split sweep needs the items to deal out into its parts).
// Measured: the 36-arc graph (2^25 iterations) 6.3 ms at 512 iterations
// per item against 8.4 ms at 2048 (64 items per CU); the 40-arc grid in 16
// parts 127 ms against 154 ms (one launch: 118 ms); items of 8 iterations
// slowed the 30-arc graph's gradient sweep (2.3 against 1.9 ms at 32).
// min_log2: the smallest item for one launch where the sweep has that many
// iterations (32 for the graph-specialised kernels and for gradients; the
// generic forward kernel on small graphs is faster with items of one
// chained block: on 256 graphs of 16 to 28 arcs, 20.9 ms in all at 8
// iterations per item against 42.3 ms at 32)
int fill_item_log2(u64 iters, int cus, u64 parts, int min_log2 = 5)
{
    const u64 target = iters / ((u64)std::max(cus, 1) * 256ull * std::max<u64>(parts, 1));
    int c = 0;
    while (c < 12 && (2ull << c) <= target) ++c;
    if (parts <= 1)
        while (c < min_log2 && (2ull << c) <= iters) ++c;
    return c;
}

// Queue tables + sweep + reduce on `stream`.  Allocates the workspace with
// hipMallocAsync; the caller frees it on the same stream.
// p_host (synchronous calls) is uploaded with the plan through the thread's
// pinned staging buffer into its reused workspace; otherwise rq.p_dev is
// already on the device and the workspace is allocated on the stream.
// fixed_ws (fixed_cap bytes): a caller-provided device workspace instead of
// an allocation.  The ahead-of-time kernels then run (loading a compiled
// kernel module would take device memory), and work items grow until the
// partials fit; BAT_ETOOBIG when even items of 2^kFixedMaxItemLog2
// iterations do not fit.  Every byte the sweep reads is written first by
// this call's own kernels and copy, so the workspace needs no clearing.
constexpr int kFixedMaxItemLog2 = 24;

int queue_sweep(const Request &rq, const Plan &P, const DeviceInfo &D, const TuneChoice &tc, hipStream_t stream,
                Launch &L, const double *p_host = nullptr, char *fixed_ws = nullptr, size_t fixed_cap = 0)
{
    const u32 m = (u32)rq.m;
    const u32 ubits = m > (u32)bat::kWordBits ? m - bat::kWordBits : 0u;
    const u64 g_first = rq.c_lo >> bat::kWordBits;
    const u64 g_last = (rq.c_hi - 1) >> bat::kWordBits;
    Options &O = opts();
    // pick the kernel
    bool use_jit = false;
    if (tc.jit == 1) use_jit = true;
    else if (tc.jit == 2) use_jit = (rq.c_hi - rq.c_lo) >= (1ull << 32) || (P.N > 32 && (rq.c_hi - rq.c_lo) >= (1ull << 22));
    if (fixed_ws) use_jit = false;
    // warm-started chains need >= k iteration bits; k = 3..6 (the gradient
    // sweep keeps at most 4 fast bits: k <= 4)
    u32 ck = tc.chain < 0 ? 3u : (tc.chain >= 6 ? 6u : (tc.chain >= 3 ? (u32)tc.chain : 0u));
    if (rq.grad && ck > (u32)bat::kGradFastMax) ck = bat::kGradFastMax;
    if (ubits < ck) ck = ubits >= 3 ? 3u : 0u;
    const bool chain = ck > 0 && !P.ru.empty();
    const u64 bmask = chain ? (1ull << ck) - 1ull : 0ull;
    const u64 g_base = g_first & ~bmask;
    const u64 g_end = g_last | bmask;
    const u64 iters = g_end - g_base + 1;

    const int clog_fill = fill_item_log2(iters, D.cus, rq.split_parts, use_jit || rq.grad ? 5 : 0);
    int clog = tc.chunk_log2;
    // a size tuned for the whole counter would leave a short range's last
    // round of work items mostly idle
    if (clog <= 0 || (rq.fill && clog > clog_fill)) clog = clog_fill;
    clog = std::min(clog, 20);
    if (chain) clog = std::max(clog, (int)ck);
    u32 f = (u32)std::max<int64_t>(0, std::min<int64_t>(O.seg_log2.load(), bat::kMaxSegLog));
    if (rq.grad) f = std::min<u32>(f, bat::kGradFastMax);
    if (chain) f = std::max<u32>(f, ck);
    if (f > ubits) f = ubits;
    const u32 ncol = rq.grad ? 1u + 2u * m : 1u;
    // workspace: input block (p | row, cb_of_arc maps | relaxation program),
    // then tables | partials | counts | output block (res | count | status)
    auto in_size = [&]() {
        size_t o = 0;
        if (p_host) o = align_up(o + sizeof(double) * (m + 1), 256);
        o = align_up(o + 128, 256);
        return align_up(o + sizeof(u32) * (P.prog.size() + 1), 256);
    };
    auto ws_size = [&](u64 n_chunks) {
        size_t o = in_size();
        o = align_up(o + sizeof(double) * bat::kTables, 256);
        o = align_up(o + sizeof(double) * 2 * ncol * n_chunks, 256);
        o = align_up(o + sizeof(u64) * n_chunks, 256);
        return align_up(o + sizeof(double) * 2 * ncol + sizeof(u64) + 64, 256);
    };
    if (fixed_ws) {
        if (rq.split_parts || rq.sample_items) return fail(BAT_EINVAL, "a fixed workspace sweeps whole ranges only");
        while (ws_size((iters + (1ull << clog) - 1) >> clog) > fixed_cap) {
            if (clog >= kFixedMaxItemLog2)
                return fail(BAT_ETOOBIG,
                            "%llu iterations need %zu bytes of fixed scratch even in work items of 2^%d "
                            "iterations; it holds %zu",
                            (unsigned long long)iters, ws_size((iters + (1ull << clog) - 1) >> clog), clog,
                            fixed_cap);
            ++clog;
        }
    }

    bat::KParams K;
    memset(&K, 0, sizeof K);
    K.c_lo = rq.c_lo;
    K.c_hi = rq.c_hi;
    K.g_first = g_first;
    K.g_last = g_last;
    K.g_base = g_base;
    K.g_end = g_end;
    K.chunk_iters = 1ull << clog;
    K.n_chunks = (iters + K.chunk_iters - 1) >> clog;
    K.chunk_mul = 1;
    K.chunk_mask = ~0ull;
    const bool pow2 = (K.n_chunks & (K.n_chunks - 1)) == 0;
    const bool sample = rq.sample_items && rq.sample_items < K.n_chunks && pow2;
    if (pow2 && (sample || tc.order != 0)) {
        // work item -> chunk through an odd multiplier: a bijection modulo
        // n_chunks that spreads consecutive items over the whole counter
        K.chunk_mul = 0x9E3779B97F4A7C15ull;
        K.chunk_mask = K.n_chunks - 1;
        if (sample) K.n_chunks = rq.sample_items;
    }
    if (rq.split_parts) {
        // Part j of J: the work items whose blocks are j modulo J, visited
        // in spread order (item i sweeps block j + J ((i M) mod S), S = N / J
        // items per part), so every part samples the whole counter the way
        // a whole sweep does.  min(J, N) parts.
        const u64 N = K.n_chunks;
        if (!pow2 || sample || (rq.split_parts & (rq.split_parts - 1)))
            return fail(BAT_EINVAL, "cannot split %llu work items into %llu parts", (unsigned long long)N,
                        (unsigned long long)rq.split_parts);
        const u64 parts = std::min<u64>(rq.split_parts, N);
        if (rq.split_index >= parts)
            return fail(BAT_EINVAL, "part %llu of %llu", (unsigned long long)rq.split_index, (unsigned long long)parts);
        K.g_base = g_base + rq.split_index * K.chunk_iters;
        K.chunk_mul = 0x9E3779B97F4A7C15ull * parts;
        K.chunk_mask = N - 1;
        K.n_chunks = N / parts;
    }
    K.m = m;
    K.ubits = ubits;
    K.seg_log = f;
    K.check_every = tc.check_every >= 2 ? 2u : 1u;
    K.chain = chain ? ck : 0u;
    K.ncol = ncol;
    K.window_test = (chain && O.window_test.load() != 0) ? 1u : 0u;
    K.n_nodes = (u32)P.N;
    K.s = (u32)P.S;
    K.t = (u32)P.T;
    K.n_relax = (u32)P.code.size();
    K.n_groups = (u32)((P.prog.size() - 8) / 16);
    chain_codes(P, K.ck_code);
    L.ncol = K.ncol;

    size_t off = 0;
    const size_t o_p = off;
    if (p_host) off = align_up(off + sizeof(double) * (m + 1), 256);
    const size_t o_map = off;  // row[64] | cb_of_arc[64]
    off = align_up(off + 128, 256);
    const size_t o_rl = off;
    off = align_up(off + sizeof(u32) * (P.prog.size() + 1), 256);
    const size_t in_bytes = off;
    const size_t o_tab = off;
    off = align_up(off + sizeof(double) * bat::kTables, 256);
    const size_t o_part = off;
    off = align_up(off + sizeof(double) * 2 * K.ncol * K.n_chunks, 256);
    const size_t o_pc = off;
    off = align_up(off + sizeof(u64) * K.n_chunks, 256);
    const size_t o_res = off;
    const size_t o_cnt = o_res + sizeof(double) * 2 * K.ncol;
    const size_t o_st = o_cnt + sizeof(u64);
    const size_t out_bytes = o_st + sizeof(int) - o_res;
    off = align_up(o_st + 64, 256);
    char *ws = nullptr;
    Scratch *S = nullptr;
    const size_t out_host_off = align_up(in_bytes, 256);
    if (in_bytes != in_size() || off != ws_size(K.n_chunks))
        return fail(BAT_EDEVICE, "workspace layout mismatch (%zu/%zu, %zu/%zu)", in_bytes, in_size(), off,
                    ws_size(K.n_chunks));
    if (fixed_ws) {
        if (off > fixed_cap) return fail(BAT_ETOOBIG, "needs %zu bytes of fixed scratch; it holds %zu", off, fixed_cap);
        ws = fixed_ws;
    } else if (p_host) {
        int rc = scratch_reserve(D.id, stream, off, out_host_off + out_bytes, S);
        if (rc) return rc;
        ws = S->dev;
    } else {
        HIPCHK(hipMallocAsync((void **)&ws, off, stream));
        L.ws = ws;
    }
    K.tables = (const double *)(ws + o_tab);
    K.status = (const int *)(ws + o_st);
    K.prog = (const u32 *)(ws + o_rl);
    K.part = (double *)(ws + o_part);
    K.pcount = (u64 *)(ws + o_pc);
    L.res = (double *)(ws + o_res);
    L.count = (u64 *)(ws + o_cnt);
    L.status = (int *)(ws + o_st);
    L.out_dev = ws + o_res;
    L.out_bytes = out_bytes;
    L.out_host_off = out_host_off;
    // the input block, built once on the host and copied in one piece
    std::vector<char> local;
    char *in = nullptr;
    if (S) {
        in = S->host;
    } else {
        local.assign(in_bytes, 0);
        in = local.data();
    }
    if (p_host && m > 0) memcpy(in + o_p, p_host, sizeof(double) * m);
    unsigned char *maps = (unsigned char *)(in + o_map);
    memset(maps, 0, 128);
    for (int i = 0; i < P.m; ++i) {
        maps[i] = P.row[i];
        maps[64 + i] = (unsigned char)P.cb_of_arc[i];
    }
    if (!P.prog.empty()) memcpy(in + o_rl, P.prog.data(), sizeof(u32) * P.prog.size());
    HIPCHK(hipMemcpyAsync(ws, in, in_bytes, hipMemcpyHostToDevice, stream));
    // (a copy from pageable memory has read its source when the call returns)
    const double *p_dev = p_host ? (const double *)(ws + o_p) : rq.p_dev;
    const bool identity = P.identity;
    const unsigned char *d_row = identity ? nullptr : (const unsigned char *)(ws + o_map);
    L.cb_of_arc = identity ? nullptr : (const unsigned char *)(ws + o_map + 64);

    hipFunction_t jfn = nullptr;
    double jit_ms = 0.0;
    uint64_t kernel_id = 0;
    const JitShape shape = jit_shape(rq.grad, tc.waves, tc.super_restart, tc.simd_waves, tc.keep_bottom);
    if (use_jit) {
        int rc = jit_get(D, P, rq.grad, shape, jfn, jit_ms, kernel_id);
        if (rc) return rc;
    } else {
        kernel_id = aot_kernel_id(rq.grad ? "k_grad_dyn" : "k_fwd_dyn", (int)P.N, P.directed);
    }

    int rc = events_ready();
    if (rc) return rc;
    HIPCHK(hipEventRecord(t_state.ev[0], stream));
    HIPCHK(batk::build_tables(stream, p_dev, d_row, m, f, (double *)K.tables, (int *)K.status));
    HIPCHK(hipEventRecord(t_state.ev[1], stream));
    // one work item per wavefront
    const u64 wpb = use_jit ? (u64)shape.waves : (u64)bat::kWavesPerBlock;
    const u64 blocks = (K.n_chunks + wpb - 1) / wpb;
    if (blocks > 0x7fffffffull) return fail(BAT_ETOOBIG, "too many work items (%llu)", (unsigned long long)blocks);
    if (use_jit) {
        void *args[] = {&K};
        HIPCHK(hipModuleLaunchKernel(jfn, (unsigned)blocks, 1, 1, (unsigned)(bat::kWave * wpb), 1, 1, 0, stream, args,
                                     nullptr));
    } else {
        HIPCHK(batk::sweep_dyn(stream, (unsigned)blocks, rq.grad, P.N, P.directed, K));
    }
    HIPCHK(hipEventRecord(t_state.ev[2], stream));
    HIPCHK(batk::reduce(stream, (const double *)K.part, (const u64 *)K.pcount, K.n_chunks, K.ncol, L.res, L.count));
    HIPCHK(hipEventRecord(t_state.ev[3], stream));

    bat_launch_info &I = t_state.info;
    memset(&I, 0, sizeof I);
    t_state.cube_seq = 0;
    I.jit_ms = jit_ms;
    I.vectors = std::min<u64>(rq.c_hi - rq.c_lo, K.n_chunks * K.chunk_iters << bat::kWordBits);
    I.specialised = use_jit ? 1 : 0;
    I.chunk_log2 = clog;
    I.n_chunks = (int32_t)std::min<u64>(K.n_chunks, 0x7fffffff);
    I.relaxations = (int32_t)(use_jit ? P.jru.size() : P.code.size());
    I.kernel_id = kernel_id;
    I.perm = P.perm;
    I.chain_log2 = (int32_t)K.chain;
    I.check_every = (int32_t)K.check_every;
    I.item_order = K.chunk_mul != 1 ? 1 : 0;
    I.block_waves = (int32_t)wpb;
    I.keep_bottom =
        (use_jit && shape.keep_bottom && P.jN <= bat::kKeepBottomMaxNodes) ? (shape.bottom_lds ? 2 : 1) : 0;
    I.super_restart = (I.keep_bottom && shape.super_restart && P.jN <= kSuperMaxNodes) ? 1 : 0;
    I.window_test = use_jit ? (int32_t)K.window_test : 0;
    I.simd_waves = (use_jit && !(rq.grad && P.jN > kGradThreeWaveNodes)) ? shape.simd_waves : 0;
    t_state.have_launch = true;
    return BAT_OK;
}

// ------------------------------------------------------- sub-cube sweeps
// Whole sweeps in the form of bat_cube.hpp.  Option BAT_CUBES: -1 (default)
// takes it unless a knob of the plain sweep's launch has been set (those
// describe the plain kernels), 0 never, 1 always where it can run.
bool cubes_wanted()
{
    const int64_t want = opts().cubes.load();
    if (want == 0) return false;
    return want == 1 || opts().plain_shape_default();
}

// The arcs a sub-cube sweep enumerates.
std::vector<char> cube_arcs(int32_t n, int32_t m, const bat_arc *arcs, int32_t s, int32_t t, bool directed)
{
    std::vector<char> rel = relevance(n, m, arcs, s, t, directed);
    for (int32_t i = 0; i < m; ++i)
        if (arcs[i].u == arcs[i].v) rel[i] = 0;
    return rel;
}

// Levels by size.  One level decides every word of 32 vectors by itself: one
// closure deep, so the shortest while the device holds its 2^(M - 11)
// wavefronts (24 arcs: 16 us against 12 us with two levels; 22 arcs: 8 us
// against 10 us).  Three levels decide less (30 arcs: 42 us against 34 us)
// but run longer chains of closures per wavefront; they win from 33 arcs on
// (specialised: 32 arcs 126 us against 94 us, 33 arcs 110 us against 131 us,
// 35 arcs 0.14 ms against 0.39 ms).
void make_cubes(int32_t n, int32_t m, const bat_arc *arcs, int32_t s, int32_t t, bool directed,
                batcube::CubePlan &C, int levels = 0)
{
    const std::vector<char> rel = cube_arcs(n, m, arcs, s, t, directed);
    if (levels <= 0) levels = (int)opts().cube_levels.load();
    int M = 0;
    for (int32_t i = 0; i < m; ++i) M += rel[i] ? 1 : 0;
    if (levels <= 0) levels = M <= 23 ? 1 : M <= 32 ? 2 : 3;
    batcube::make_cube_plan(n, m, arcs, rel, s, t, directed, levels, C);
}

// Work items of a whole sweep.
u64 cube_items(const batcube::CubePlan &C) { return 1ull << std::max(0, C.M - C.rel_bits()); }

// The closures as the ahead-of-time kernels read them.
bool cube_pack(const batcube::CubePlan &C, bat::CubeProg *prog, u32 *step)
{
    u32 at = 0;
    for (int k = 0; k < 2 * C.levels - 1; ++k) {
        const batcube::Program &pr = C.prog[k];
        bat::CubeProg &q = prog[k];
        q.first = at;
        q.octets = (u32)std::max<size_t>(1, (pr.step.size() + 7) / 8);
        q.result = pr.result == -1 ? bat::kCubeNever : pr.result == -2 ? bat::kCubeAlways : (u32)pr.result;
        q.word = (u32)(bat::kCubeGroup * ((k + 1) / 2));
        if (at + 8 * q.octets > (u32)bat::kCubeSteps) return false;
        for (u32 i = 0; i < 8 * q.octets; ++i) {
            if (i < pr.step.size()) {
                const batcube::Step &x = pr.step[i];
                step[at + i] = (u32)x.a | (u32)x.b << 8 | (u32)x.d << 16 | (x.assign ? 0u : 1u << 31);
            } else {
                step[at + i] = 1u << 31;  // slot 0 |= itself
            }
        }
        at += 8 * q.octets;
    }
    return true;
}

// Most blocks a sweep of many work items is cut into (40 arcs: 8192), and the
// work items from which its units are taken in chunks.
constexpr u64 kCubeBlocks = 1ull << 17;
constexpr int64_t kCubeSplitMost = 64;
bool cube_chunked(const batcube::CubePlan &C) { return cube_items(C) > kCubeBlocks * bat::kCubeUnits; }

// Most chunks of units a gradient sweep is cut into, while a block takes no
// more than grad_units of them.
constexpr u64 kGradChunks = 65536;

// How a sweep's items are cut (split: units of an item; units: of a block;
// chunk: units summed in one place): with the plan, the order of its sums.
struct CubeShape {
    u32 split = 0, units = 0, chunk = 0;  // 0: by size
};

// The launch of a cube plan: everything but the result and partial pointers.
// part j of `parts` (a power of two, at most the items): the items that are
// j modulo parts.
int cube_params(const batcube::CubePlan &C, const double *p_host, const double *p_dev, const DeviceInfo &D,
                bat::CubeParams &K, unsigned &blocks, int &waves, bool jit, bool grad, u64 parts = 1, u64 part = 0,
                const CubeShape *want = nullptr)
{
    memset(&K, 0, sizeof K);
    K.m = (u32)C.m;
    K.M = (u32)C.M;
    K.levels = (u32)C.levels;
    K.lane_bits = (u32)C.lane_bits;
    K.n_items = cube_items(C) / parts;
    K.item_mul = 0x9E3779B97F4A7C15ull * parts;  // odd times parts: consecutive items lie apart
    K.item_mask = cube_items(C) - 1;
    K.item_base = part;
    // Items are split into up to 4 units while there are few.  With two
    // levels only to fill the device: 24 arcs, 256 items: 11.0 us in 4 units
    // each, 15.3 us whole; 27 arcs, 2048 items: 37 us in 2, 47 us whole; with
    // gradients, whose units also fold 50 sums, 24 arcs 32 us in 4 and 74 us
    // in 16, 27 arcs 91 us whole and 119 us in 2.  With three levels, where
    // deciding the item's first word again is a small part, until the long
    // items no longer set the end: 36 arcs, 16384 items: 0.57 ms in 4, 1.02
    // ms whole, with gradients 1.6 and 2.6 ms; 40 arcs, 524288 items: 11.9 ms
    // in 4, 9.1 ms whole.
    u64 split = 1;
    const u64 enough = (u64)D.cus * (C.levels == 3 ? 1024 : grad ? 4 : 16);
    if (opts().cube_split.load() > 0) split = (u64)std::min<int64_t>(opts().cube_split.load(), kCubeSplitMost);
    else
        while (split < 4 && K.n_items * split < enough) split *= 2;
    if (C.levels == 1) split = 1;
    if (want && want->split) split = want->split;
    K.split = (u32)split;
    const u64 w = K.n_items * split;
    waves = (int)std::min<u64>(w, bat::kCubeWaves);
    u64 units = (u64)waves;
    if (grad) {
        // a chunk's fold of some 50 columns takes as long as several rounds:
        // chunks of several units once they are many (36 arcs, 65536 units:
        // 1.6 ms one by one, 2.6 ms in chunks of 8 of a block of 64; 40 arcs,
        // 524288 units: 20.4 ms in eights, 26 ms in twos; with columns kept as
        // double-doubles 21.0 ms in eights)
        u64 per = 1;
        while (w / per > kGradChunks) per *= 2;
        if (want && want->chunk) per = want->chunk;
        const u64 chunks = (w + per - 1) / per;
        u64 cb = (u64)waves;
        while (cb < (u64)bat::grad_units(C.M) && chunks / (2 * cb) >= (u64)D.cus * 4) cb *= 2;
        if (want && want->units) cb = want->units;
        K.chunk = (u32)per;
        K.units = (u32)cb;
        blocks = (unsigned)((chunks + cb - 1) / cb);
        K.fused = 0u;
    }
    // units per block: as many as leave every CU some 16 blocks
    while (units < bat::kCubeUnits && w / (2 * units) >= (u64)D.cus * 16) units *= 2;
    if (!grad) {
        if (want && want->units) units = want->units;
        u64 per = 1;
        while (cube_chunked(C) && w / (units * per) > kCubeBlocks) per *= 2;
        if (want && want->chunk) per = want->chunk;
        K.chunk = (u32)per;
        K.units = (u32)units;
        const u64 nb = (w + units * per - 1) / (units * per);
        blocks = (unsigned)nb;
        K.fused = nb == 1 ? 1u : 0u;
    }
    K.p_dev = p_dev;
    if (p_host) memcpy(K.p, p_host, sizeof(double) * C.m);
    for (int c = 0; c < C.M; ++c) K.arc_of_bit[c] = (unsigned char)C.arc_of_bit[c];
    if (!jit && !cube_pack(C, K.prog, K.step)) return fail(BAT_EDEVICE, "sub-cube closures of too many steps");
    return BAT_OK;
}

// Whether a shape that a file names is one this library cuts parts of
// `n_items` items into.
bool cube_shape_ok(const batcube::CubePlan &C, bool grad, const CubeShape &H, u64 n_items)
{
    if (!H.split) return true;
    const u32 most = grad ? (u32)bat::grad_units(C.M) : (u32)bat::kCubeUnits;
    if (H.split > (u32)kCubeSplitMost || (C.levels == 1 && H.split != 1) || H.units < 1 || H.units > most || H.chunk < 1 ||
        (!grad && !cube_chunked(C) && H.chunk != 1))
        return false;
    const u64 w = n_items * H.split, per = (u64)H.units * H.chunk;
    return (w + per - 1) / per <= (kCubeBlocks * (u64)kCubeSplitMost);
}

// Whether the plan runs as a graph-specialised kernel: by the rule of the
// plain sweep (a compile takes about half a second, once per graph).
bool cube_jit(const batcube::CubePlan &C)
{
    const int64_t jit = opts().jit.load();
    return jit == 1 || (jit == 2 && C.m >= 32);
}

// Whether a kernel can run the plan (aot: the ahead-of-time one).
bool cube_fits(const batcube::CubePlan &C, bool aot = false)
{
    if (!aot && cube_jit(C)) return true;
    return C.M <= batk::kCubeMaxBits && C.slots <= bat::kCubeSlots && C.steps + 8 * bat::kCubeProgs <= bat::kCubeSteps;
}

// The partials (none when one block writes the results): per block, or with
// gradients per block and column, and the reduction's block counter.
size_t cube_part_bytes(const bat::CubeParams &K, unsigned blocks, bool grad)
{
    if (grad) return 256 + (16 * (1 + 2 * (size_t)K.M) + 8) * blocks;
    return K.fused ? 0 : 24 * (size_t)blocks;
}
void cube_parts(bat::CubeParams &K, unsigned blocks, bool grad, char *ws)
{
    if (grad) {
        K.done = (u32 *)ws;
        K.part = (bat::double2_t *)(ws + 256);
        K.pcount = (u64 *)(ws + 256 + 16 * (1 + 2 * (size_t)K.M) * blocks);
    } else if (!K.fused) {
        K.part = (bat::double2_t *)ws;
        K.pcount = (u64 *)(ws + 16 * (size_t)blocks);
    }
}

// The hiprtc source of the sweep specialised for a plan.  with_arcs: also
// the arcs at the counter bits, in a comment (the code does not depend on
// them).
std::string cube_source(const batcube::CubePlan &C, bool grad, bool with_arcs = false)
{
    std::string g = "\nnamespace bat {\nstruct JitCube {\n";
    if (with_arcs) {
        g += "  // arcs at counter bits 0, 1, ...:";
        for (int a : C.arc_of_bit) g += " " + std::to_string(a);
        g += "\n";
    }
    auto num = [&](const char *k, int v) { g += std::string("  static constexpr int ") + k + " = " + std::to_string(v) + ";\n"; };
    num("M", C.M);
    num("REL", C.rel_bits());
    num("SLOTS", std::max(C.slots, 1));
    g += "  static constexpr u32 LEVELS = " + std::to_string(C.levels) + "u, LANE_BITS = " + std::to_string(C.lane_bits) +
         "u;\n  static constexpr bool CHUNKED = " + (cube_chunked(C) ? "true" : "false") +
         ";\n  static constexpr u32 RESULT[5] = {";
    for (int k = 0; k < bat::kCubeProgs; ++k) {
        const int r = k < 2 * C.levels - 1 ? C.prog[k].result : -1;
        g += (k ? ", " : "") + std::to_string(r == -1 ? bat::kCubeNever : r == -2 ? bat::kCubeAlways : (u32)r) + "u";
    }
    g += "};\n  template <u32 K> __device__ static __forceinline__ void steps(u32 *r) {\n";
    for (int k = 0; k < 2 * C.levels - 1; ++k) {
        g += "    if constexpr (K == " + std::to_string(k) + "u) {\n";
        for (const batcube::Step &x : C.prog[k].step)
            g += "      r[" + std::to_string(x.d) +
                 (x.assign ? "] = r[" + std::to_string(x.a) + "] & r[" + std::to_string(x.b) + "];\n"
                           : "] = and_or(r[" + std::to_string(x.a) + "], r[" + std::to_string(x.b) + "], r[" +
                                 std::to_string(x.d) + "]);\n");
        g += "    }\n";
    }
    g += "  }\n};\n}\n";
    if (grad)
        g += "extern \"C\" __global__ void __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(3, 3))) "
             "bat_cube_grad_jit(bat::CubeParams) {\n"
             "  __shared__ bat::CubeSumTables T; __shared__ bat::CubeGradTables X;\n"
             "  __shared__ bat::CubeGradWave W[bat::kCubeWaves];\n"
             "  __shared__ bat::double2_t cols[bat::grad_units(bat::JitCube::M)][1 + 2 * bat::JitCube::M];\n"
             "  bat::cube_grad_kernel((bat::CubeArgs *)__builtin_amdgcn_kernarg_segment_ptr(), T, X, W, cols, "
             "bat::CubeStatic<bat::JitCube>{});\n}\n";
    else
        g += "extern \"C\" __global__ void __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(5, 5))) "
             "bat_cube_jit(bat::CubeParams) {\n"
             "  __shared__ bat::CubeTables T; __shared__ bat::CubeWave W[bat::kCubeWaves];\n"
             "  bat::cube_kernel((bat::CubeArgs *)__builtin_amdgcn_kernarg_segment_ptr(), T, W, "
             "bat::CubeStatic<bat::JitCube>{});\n}\n";
    return std::string(kDeviceSource) + kCubeSource + g;
}

// The specialised kernel of a plan, by the bytes its source is made from.
int cube_jit_get(const batcube::CubePlan &C, const DeviceInfo &D, bool grad, hipFunction_t &fn, double &jit_ms, uint64_t &id)
{
    std::string key = std::to_string(D.id) + (grad ? " cubeg " : " cube ") + std::to_string(C.M) + " " + std::to_string(C.levels) + " " +
                      std::to_string(C.lane_bits) + " " + std::to_string(C.slots) + ":";
    for (int k = 0; k < 2 * C.levels - 1; ++k) {
        key += " " + std::to_string(C.prog[k].result) + " ";
        for (const batcube::Step &x : C.prog[k].step) {
            const unsigned char b[4] = {(unsigned char)x.a, (unsigned char)x.b, (unsigned char)x.d,
                                        (unsigned char)(x.assign ? 1 : 0)};
            key.append((const char *)b, sizeof b);
        }
        key += ";";
    }
    if (jit_ready(key, fn, id)) return BAT_OK;
    return jit_load(D, key, cube_source(C, grad), grad ? "bat_cube_grad_jit" : "bat_cube_jit", fn, jit_ms, id);
}

void cube_launch_info(const batcube::CubePlan &C, const bat::CubeParams &K, int waves)
{
    bat_launch_info &I = t_state.info;
    memset(&I, 0, sizeof I);
    t_state.cube_seq = 0;
    I.vectors = (1ull << C.m) / (cube_items(C) / K.n_items);
    I.chunk_log2 = std::max(0, C.rel_bits() + (C.m - C.M) - bat::kWordBits);
    I.n_chunks = (int32_t)std::min<u64>(K.n_items, 0x7fffffff);
    I.relaxations = C.M;
    I.perm = kPermInfluence;
    I.check_every = 1;
    I.item_order = 1;
    I.block_waves = waves;
    t_state.have_launch = true;
}

// Queue the sweep (and its reduction) on `stream`; K's result pointers set.
// No event is recorded where the kernels can report their clocks themselves
// (four event records took a third of a small call's time).
int cube_queue(const batcube::CubePlan &C, bat::CubeParams &K, unsigned blocks, int waves, bool jit, bool grad,
               const DeviceInfo &D, hipStream_t stream, Report kind)
{
    hipFunction_t fn = nullptr;
    double jit_ms = 0.0;
    uint64_t kid = aot_kernel_id(grad ? "k_cube_grad" : "k_cube_fwd", 0, false);
    if (jit) {
        int rc = cube_jit_get(C, D, grad, fn, jit_ms, kid);
        if (rc) return rc;
    }
    u64 *slot = nullptr;
    bool captured = false;
    int rc = diag_next(stream, slot, K.seq, kind, &captured);
    if (rc) return rc;
    K.diag = slot;
    const bool events = !slot && !captured;
    if (events) {
        rc = events_ready();
        if (rc) return rc;
        HIPCHK(hipEventRecord(t_state.ev[0], stream));
        HIPCHK(hipEventRecord(t_state.ev[1], stream));
    }
    if (jit) {
        void *args[] = {&K};
        HIPCHK(hipModuleLaunchKernel(fn, blocks, 1, 1, (unsigned)(waves * bat::kWave), 1, 1, 0, stream, args, nullptr));
    } else if (grad) {
        HIPCHK(batk::cube_grad(stream, blocks, waves, K));
    } else {
        HIPCHK(batk::cube_sweep(stream, blocks, waves, K));
    }
    if (events) HIPCHK(hipEventRecord(t_state.ev[2], stream));
    if (grad) HIPCHK(batk::cube_grad_finish(stream, blocks, K));
    else if (!K.fused) HIPCHK(batk::cube_finish(stream, blocks, K));
    if (events) HIPCHK(hipEventRecord(t_state.ev[3], stream));
    cube_launch_info(C, K, waves);
    t_state.info.specialised = jit ? 1 : 0;
    t_state.info.jit_ms = jit_ms;
    t_state.info.kernel_id = kid;
    t_state.cube_seq = slot ? K.seq : captured ? ~0ull : 0ull;
    t_state.cube_slot = slot;
    t_state.cube_stream = stream;
    t_state.cube_dev = D.id;
    t_state.cube_khz = D.clock_khz;
    return BAT_OK;
}

// Wait for a launch on the thread's stream: a short call's results are
// there some microseconds before the stream counts as idle, so its report
// is polled first.
int cube_wait(const bat::CubeParams &K, hipStream_t stream)
{
    const auto t0 = std::chrono::steady_clock::now();
    for (int k = 0; !diag_done(K.diag, K.seq); ++k) {
        __builtin_ia32_pause();
        if ((k & 63) == 63 && std::chrono::steady_clock::now() - t0 > std::chrono::microseconds(200)) {
            HIPCHK(hipStreamSynchronize(stream));
            if (!diag_done(K.diag, K.seq)) return fail(BAT_EDEVICE, "a sweep ended without its results");
        }
    }
    return BAT_OK;
}

// A whole sweep over host probabilities (validated); res: R as a
// double-double, with gradients followed by T0 and T1 of each arc, written
// by the device into the pinned staging buffer.
// shape: how to cut the items; set to how they were.
int cube_sync(const batcube::CubePlan &C, const double *p, const DeviceInfo &D, bool grad, std::vector<double> &res,
              u64 &count, u64 parts = 1, u64 part = 0, CubeShape *shape = nullptr)
{
    hipStream_t stream;
    int rc = thread_stream(D.id, stream);
    if (rc) return rc;
    bat::CubeParams K;
    unsigned blocks = 0;
    int waves = 0;
    // (a resumed checkpoint may need the specialised kernel whatever BAT_JIT is)
    const bool jit = cube_jit(C) || !cube_fits(C, true);
    rc = cube_params(C, p, nullptr, D, K, blocks, waves, jit, grad, parts, part, shape);
    if (rc) return rc;
    if (shape) *shape = CubeShape{K.split, K.units, K.chunk};
    Scratch *S = nullptr;
    const size_t n = grad ? 2 + 4 * (size_t)C.m : 2;
    rc = scratch_reserve(D.id, stream, cube_part_bytes(K, blocks, grad), 8 * (n + 1), S);
    if (rc) return rc;
    cube_parts(K, blocks, grad, S->dev);
    K.res = (double *)S->host;
    K.count = (u64 *)(S->host + 8 * n);
    rc = cube_queue(C, K, blocks, waves, jit, grad, D, stream, Report::sync);
    if (!rc) rc = cube_wait(K, stream);
    if (rc) {
        (void)hipStreamSynchronize(stream);
        return rc;
    }
    res.assign((const double *)S->host, (const double *)S->host + n);
    memcpy(&count, S->host + 8 * n, 8);
    return BAT_OK;
}

// The same on `stream` over device probabilities, results to device memory.
// ws: a workspace of ws_bytes, or null to take one from the stream's pool.
int cube_async(const batcube::CubePlan &C, const double *p_dev, const DeviceInfo &D, hipStream_t stream, bool grad,
               double *R, u64 *count, double *dRdp, double *T1, double *T0, int *status, char *ws, size_t ws_bytes)
{
    bat::CubeParams K;
    unsigned blocks = 0;
    int waves = 0;
    const bool jit = !ws && cube_jit(C);  // (a fixed workspace: no module is loaded)
    int rc = cube_params(C, nullptr, p_dev, D, K, blocks, waves, jit, grad);
    if (rc) return rc;
    const size_t need = cube_part_bytes(K, blocks, grad);
    void *own = nullptr;
    if (!ws && need) {
        HIPCHK(hipMallocAsync(&own, need, stream));
        ws = (char *)own;
    } else if (ws && need > ws_bytes) {
        return fail(BAT_ETOOBIG, "needs %zu bytes of fixed scratch; it holds %zu", need, ws_bytes);
    }
    cube_parts(K, blocks, grad, ws);
    K.R = R;
    K.count = count;
    K.status = status;
    K.dRdp = dRdp;
    K.T1 = T1;
    K.T0 = T0;
    rc = cube_queue(C, K, blocks, waves, jit, grad, D, stream, own || !ws ? Report::async : Report::noalloc);
    if (own) {
        const hipError_t e = hipFreeAsync(own, stream);
        if (!rc) HIPCHK(e);
    }
    return rc;
}

struct Prepared {
    DeviceInfo D;
    Plan P;
    hipStream_t stream = nullptr;
};

// Validate, pick the launch choices and plan.  full_range: the whole
// counter, where any arc order may be used; otherwise the paper's order.
int prepare(int32_t n, int32_t m, const bat_arc *arcs, const double *p_host, int32_t s, int32_t t, bool grad,
            bool full_range, const Request *forced, Prepared &X, TuneChoice &tc, uint32_t flags = 0)
{
    int rc = validate(n, m, arcs, p_host, s, t);
    if (rc) return rc;
    rc = current_device(X.D);
    if (rc) return rc;
    const bool directed = (flags & BAT_DIRECTED) != 0;
    tc = choose(X.D, graph_key(n, m, arcs, s, t, directed), grad, forced);
    const bool forward = forced && forced->force_perm == kPermForward;
    if (!forward && (tc.perm < 0 || tc.perm >= kPermKinds)) tc.perm = kDefaultPerm;
    if (!full_range && !forward) tc.perm = 0;
    make_plan(n, m, arcs, s, t, X.P, tc.perm, directed);
    return BAT_OK;
}

// Synchronous driver over host p; fills res (ncol double-double pairs),
// count and the plan's arc -> counter bit map (for the gradient columns).
int run_sync(int32_t n, int32_t m, const bat_arc *arcs, const double *p, int32_t s, int32_t t, u64 c_lo,
             u64 c_hi, bool grad, std::vector<double> &res, u64 &count, Request *tmpl = nullptr,
             std::vector<int> *cb_of_arc = nullptr, uint32_t flags = 0)
{
    Prepared X;
    TuneChoice tc;
    const bool full = c_lo == 0 && c_hi == (1ull << m);
    if (!p && m > 0) return fail(BAT_EINVAL, "p is NULL");
    if (full && !tmpl && cubes_wanted()) {
        int rc = validate(n, m, arcs, p, s, t);
        if (!rc) rc = current_device(X.D);
        if (rc) return rc;
        batcube::CubePlan C;
        make_cubes(n, m, arcs, s, t, (flags & BAT_DIRECTED) != 0, C);
        if (cube_fits(C)) {
            if (cb_of_arc) {  // (the columns are in arc order)
                cb_of_arc->resize(m);
                for (int32_t a = 0; a < m; ++a) (*cb_of_arc)[a] = a;
            }
            return cube_sync(C, p, X.D, grad, res, count);
        }
    }
    // any arc order for a whole sweep; a partial range is in the paper's
    // order unless the caller (the autotuner timing a sample) forces one
    const bool allow_perm = full || (tmpl && tmpl->force_perm >= 0);
    int rc = prepare(n, m, arcs, p, s, t, grad, allow_perm, tmpl, X, tc, flags);
    if (rc) return rc;
    rc = thread_stream(X.D.id, X.stream);
    if (rc) return rc;
    Request rq = tmpl ? *tmpl : Request{};
    rq.n = n; rq.m = m; rq.s = s; rq.t = t; rq.arcs = arcs; rq.p_dev = nullptr;
    rq.c_lo = c_lo; rq.c_hi = c_hi; rq.grad = grad;
    Launch L;
    static const double kNoArcs = 0.0;
    rc = queue_sweep(rq, X.P, X.D, tc, X.stream, L, m > 0 ? p : &kNoArcs);
    if (rc) {
        (void)hipStreamSynchronize(X.stream);
        return rc;
    }
    // one copy back: res | count | status, into the pinned staging buffer
    Scratch &S = t_state.scratch[X.D.id];
    char *out = S.host + L.out_host_off;
    HIPCHK(hipMemcpyAsync(out, L.out_dev, L.out_bytes, hipMemcpyDeviceToHost, X.stream));
    HIPCHK(hipStreamSynchronize(X.stream));
    res.assign(2 * L.ncol, 0.0);
    memcpy(res.data(), out, sizeof(double) * 2 * L.ncol);
    memcpy(&count, out + sizeof(double) * 2 * L.ncol, sizeof(u64));
    int st = 0;
    memcpy(&st, out + sizeof(double) * 2 * L.ncol + sizeof(u64), sizeof(int));
    if (st) return fail(BAT_EINVAL, "a probability is outside [0,1]");
    if (cb_of_arc) *cb_of_arc = X.P.cb_of_arc;
    return BAT_OK;
}

void split_grad(const std::vector<double> &res, const std::vector<int> &cb_of_arc, int32_t m, double *dRdp,
                double *T1, double *T0)
{
    for (int32_t a = 0; a < m; ++a) {
        int cb = cb_of_arc[a];
        const double *t0 = &res[2 * (1 + 2 * cb)], *t1 = &res[2 * (1 + 2 * cb + 1)];
        if (dRdp) dRdp[a] = (t1[0] - t0[0]) + (t1[1] - t0[1]);
        if (T1) T1[a] = t1[0] + t1[1];
        if (T0) T0[a] = t0[0] + t0[1];
    }
}

int range_cubes(int32_t n, int32_t m, const bat_arc *arcs, const double *p, int32_t s, int32_t t, const DeviceInfo &D,
                bool forward, u64 c_lo, u64 c_hi, double *R, u64 &count, bool &fits);

// Partial sums over [c_lo, c_hi) of the counter whose bits follow arc-to-bit
// order kind `perm` (0: the paper's backward BAT indices, kPermForward: its
// forward ones); arguments already validated except the probabilities.
int range_in_order(int32_t n, int32_t m, const bat_arc *arcs, const double *p, int32_t s, int32_t t,
                   uint32_t flags, int perm, u64 c_lo, u64 c_hi, double *R_hi, double *R_lo, uint64_t *count_out,
                   double *T1_out, double *T0_out)
{
    const bool grad = T1_out != nullptr;
    if (c_lo == c_hi) {
        int rc = validate(n, m, arcs, p, s, t);
        if (rc) return rc;
        *R_hi = *R_lo = 0.0;
        *count_out = 0;
        if (grad)
            for (int32_t a = 0; a < m; ++a) T1_out[a] = T0_out[a] = 0.0;
        return BAT_OK;
    }
    std::vector<double> res;
    std::vector<int> cba;
    u64 cnt = 0;
    Request order{};
    order.force_perm = perm;
    order.fill = true;
    int rc = run_sync(n, m, arcs, p, s, t, c_lo, c_hi, grad, res, cnt, &order, &cba, flags);
    if (rc) return rc;
    *R_hi = res[0];
    *R_lo = res[1];
    *count_out = cnt;
    if (grad) split_grad(res, cba, m, nullptr, T1_out, T0_out);
    return BAT_OK;
}

// The arc-to-bit order a whole sweep of this graph would take (tuned or
// default); the forward BAT order when the flags ask for it.
int whole_sweep_order(int32_t n, int32_t m, const bat_arc *arcs, int32_t s, int32_t t, uint32_t flags, bool grad,
                      int &perm)
{
    if (flags & BAT_FORWARD_ORDER) {
        perm = kPermForward;
        return BAT_OK;
    }
    DeviceInfo D;
    int rc = current_device(D);
    if (rc) return rc;
    const TuneChoice tc = choose(D, graph_key(n, m, arcs, s, t, (flags & BAT_DIRECTED) != 0), grad, nullptr);
    perm = tc.perm >= 0 && tc.perm < kPermKinds ? tc.perm : kDefaultPerm;
    return BAT_OK;
}

// ------------------------------------------------------------ checkpoints
// A chunked sweep's running sums: R and the per-arc T1 / T0 as unevaluated
// double-doubles (hi, lo), the count exactly.
struct RunningSums {
    // the launch every chunk repeats (-1: no chunk run yet): arc-to-bit
    // order kind, work-item size (log2 iterations), chain length
    int order = -1, items = -1, chain = -1;
    // order kPermInfluence (sub-cube sweeps): items is 32 levels + the bits
    // of an item, bits a hash of the arcs' counter bits, shape how the items
    // are cut (0 in files of before it was kept: by size)
    uint64_t bits = 0;
    CubeShape shape;
    u64 parts = 0;  // chunks: parts of the whole sweep's work items
    u64 done = 0;
    u64 count = 0;
    double R[2] = {0.0, 0.0};
    std::vector<double> T1, T0;  // 2 m each (hi, lo per arc) when kept
};

// hi + lo += x_hi + x_lo (Knuth's two-sum on the high parts)
void dd_acc(double *d, double x_hi, double x_lo)
{
    const double s = d[0] + x_hi;
    const double bb = s - d[0];
    const double e = (d[0] - (s - bb)) + (x_hi - bb);
    const double lo = e + d[1] + x_lo;
    d[0] = s + lo;
    d[1] = lo - (d[0] - s);
}

uint64_t fnv_bytes(uint64_t h, const void *data, size_t len)
{
    const unsigned char *b = (const unsigned char *)data;
    for (size_t i = 0; i < len; ++i) h = (h ^ b[i]) * 1099511628211ull;  // FNV-1a
    return h;
}

// The line that names the problem a checkpoint file belongs to.
std::string checkpoint_problem(int32_t n, int32_t m, const bat_arc *arcs, const double *p, int32_t s, int32_t t,
                               uint32_t flags, int32_t clog, bool grad)
{
    uint64_t ha = fnv_bytes(1469598103934665603ull, arcs, sizeof(bat_arc) * (size_t)m);
    uint64_t hp = fnv_bytes(1469598103934665603ull, p, sizeof(double) * (size_t)m);
    char buf[256];
    snprintf(buf, sizeof buf, "problem n=%d m=%d s=%d t=%d flags=%u chunk_log2=%d grad=%d arcs=%016llx p=%016llx",
             n, m, s, t, flags, clog, grad ? 1 : 0, (unsigned long long)ha, (unsigned long long)hp);
    return buf;
}

const char *kCheckpointMagic = "bat-checkpoint 1";

// Reads `path` into S.  1: no such file (a fresh start), 0: read, < 0: error.
int checkpoint_read(const char *path, const std::string &problem, bool grad, int32_t m, uint32_t flags,
                    RunningSums &S)
{
    FILE *f = fopen(path, "r");
    if (!f) {
        if (errno == ENOENT) return 1;
        return fail(BAT_EIO, "checkpoint %s: cannot open (%s)", path, strerror(errno));
    }
    std::string text;
    char buf[4096];
    size_t got;
    while ((got = fread(buf, 1, sizeof buf, f)) > 0) text.append(buf, got);
    const bool bad_read = ferror(f) != 0;
    fclose(f);
    if (bad_read) return fail(BAT_EIO, "checkpoint %s: read error", path);
    std::vector<std::string> lines;
    for (size_t a = 0, b; a < text.size(); a = b + 1) {
        b = text.find('\n', a);
        if (b == std::string::npos) b = text.size();
        lines.push_back(text.substr(a, b - a));
    }
    if (lines.size() < 2 || lines[0] != kCheckpointMagic)
        return fail(BAT_EIO, "checkpoint %s: not a checkpoint file", path);
    if (lines[1] != problem)
        return fail(BAT_EINVAL, "checkpoint %s belongs to another problem (%s; this call: %s)", path,
                    lines[1].c_str(), problem.c_str());
    if (lines.size() < (grad ? 9u : 7u)) return fail(BAT_EIO, "checkpoint %s: truncated", path);
    unsigned long long parts = 0, done = 0, cnt = 0, bits = 0;
    int order = -1, items = -1, chain = -1;
    char tail;
    CubeShape shape;
    bool cube_line = sscanf(lines[3].c_str(),
                            "launch order=%d items=%d chain=%d split=%u units=%u chunk=%u bits=%llx %c", &order, &items,
                            &chain, &shape.split, &shape.units, &shape.chunk, &bits, &tail) == 7 &&
                     shape.split && shape.units && shape.chunk;
    if (!cube_line) {  // (a file of before the shape was kept)
        shape = CubeShape{};
        cube_line = sscanf(lines[3].c_str(), "launch order=%d items=%d chain=%d bits=%llx %c", &order, &items, &chain,
                           &bits, &tail) == 4;
    }
    const bool cubes = order == kPermInfluence;
    const bool launch_ok =
        cubes ? cube_line
              : sscanf(lines[3].c_str(), "launch order=%d items=%d chain=%d %c", &order, &items, &chain, &tail) == 3;
    if (sscanf(lines[2].c_str(), "parts %llu %c", &parts, &tail) != 1 ||
        !launch_ok ||
        sscanf(lines[4].c_str(), "done %llu %c", &done, &tail) != 1 ||
        sscanf(lines[5].c_str(), "count %llu %c", &cnt, &tail) != 1)
        return fail(BAT_EIO, "checkpoint %s: malformed header", path);
    const int ubits = m > bat::kWordBits ? m - bat::kWordBits : 0;
    const bool fwd = (flags & BAT_FORWARD_ORDER) != 0;
    if (cubes) {
        const int levels = items / 32, rel = items % 32;
        if (fwd || levels < 1 || levels > bat::kCubeLevels || rel < bat::kCubeGroup * levels || chain != 0 ||
            parts == 0 || (parts & (parts - 1)) != 0 || parts > (1ull << std::max(m - rel, 0)) || done > parts)
            return fail(BAT_EIO, "checkpoint %s: bad launch or part counts", path);
    } else if (fwd ? order != kPermForward : (order < 0 || order >= kPermKinds))
        return fail(BAT_EIO, "checkpoint %s: bad arc order %d", path, order);
    if (!cubes && (items < 0 || items > 20 || (chain != 0 && (chain < 3 || chain > 6)) || parts == 0 ||
        (parts & (parts - 1)) != 0 || parts > (1ull << std::max(ubits - items, 0)) || done > parts))
        return fail(BAT_EIO, "checkpoint %s: bad launch or part counts", path);
    // "<tag> hi lo [hi lo ...]" with hexadecimal floats (exact round trip)
    auto doubles = [&](const std::string &ln, const char *tag, size_t want, double *out) {
        const size_t tl = strlen(tag);
        if (ln.compare(0, tl, tag) != 0) return false;
        const char *q = ln.c_str() + tl;
        for (size_t i = 0; i < want; ++i) {
            char *e = nullptr;
            out[i] = strtod(q, &e);
            if (e == q || !std::isfinite(out[i])) return false;
            q = e;
        }
        while (*q == ' ') ++q;
        return *q == '\0';
    };
    RunningSums R;
    R.order = order;
    R.items = items;
    R.chain = chain;
    R.bits = bits;
    R.shape = shape;
    R.parts = parts;
    R.done = done;
    R.count = cnt;
    if (!doubles(lines[6], "R", 2, R.R)) return fail(BAT_EIO, "checkpoint %s: malformed R line", path);
    if (grad) {
        R.T1.assign(2 * (size_t)m, 0.0);
        R.T0.assign(2 * (size_t)m, 0.0);
        if (!doubles(lines[7], "T1", 2 * (size_t)m, R.T1.data()) || !doubles(lines[8], "T0", 2 * (size_t)m, R.T0.data()))
            return fail(BAT_EIO, "checkpoint %s: malformed T1/T0 lines", path);
    }
    S = std::move(R);
    return 0;
}

// Writes S to path + ".tmp", then renames it over `path`, so a reader sees
// either the old file or the new one whole.
int checkpoint_write(const char *path, const std::string &problem, bool grad, const RunningSums &S)
{
    std::string text = std::string(kCheckpointMagic) + "\n" + problem + "\n";
    char buf[256];
    char bits[96] = "";
    if (S.order == kPermInfluence)
        snprintf(bits, sizeof bits, " split=%u units=%u chunk=%u bits=%016llx", S.shape.split, S.shape.units,
                 S.shape.chunk, (unsigned long long)S.bits);
    snprintf(buf, sizeof buf, "parts %llu\nlaunch order=%d items=%d chain=%d%s\ndone %llu\ncount %llu\nR %a %a\n",
             (unsigned long long)S.parts, S.order, S.items, S.chain, bits, (unsigned long long)S.done,
             (unsigned long long)S.count, S.R[0], S.R[1]);
    text += buf;
    if (grad) {
        for (int w = 0; w < 2; ++w) {
            const std::vector<double> &v = w ? S.T0 : S.T1;
            text += w ? "T0" : "T1";
            for (double x : v) {
                snprintf(buf, sizeof buf, " %a", x);
                text += buf;
            }
            text += "\n";
        }
    }
    const std::string tmp = std::string(path) + ".tmp";
    FILE *f = fopen(tmp.c_str(), "w");
    if (!f) return fail(BAT_EIO, "checkpoint %s: cannot create (%s)", tmp.c_str(), strerror(errno));
    const bool ok = fwrite(text.data(), 1, text.size(), f) == text.size() && fflush(f) == 0 && fsync(fileno(f)) == 0;
    if (fclose(f) != 0 || !ok) {
        unlink(tmp.c_str());
        return fail(BAT_EIO, "checkpoint %s: write failed", tmp.c_str());
    }
    if (rename(tmp.c_str(), path) != 0) {
        unlink(tmp.c_str());
        return fail(BAT_EIO, "checkpoint %s: rename failed (%s)", path, strerror(errno));
    }
    return BAT_OK;
}

// Chunk S.done of a checkpointed sweep: one part of the whole sweep's work
// items (queue_sweep's split), under the launch the first chunk took: its
// arc order, work-item size and chain length fix which blocks each part
// holds and how its sums are rounded.
int run_part(int32_t n, int32_t m, const bat_arc *arcs, const double *p, int32_t s, int32_t t, uint32_t flags,
             bool grad, u64 parts_wanted, RunningSums &S, double *R_hl, uint64_t *count, double *T1, double *T0)
{
    Request rq{};
    const bool first = S.order < 0;
    if (first ? cubes_wanted() && !(flags & BAT_FORWARD_ORDER) : S.order == kPermInfluence) {
        // the sub-cube sweep's items
        DeviceInfo D;
        int rc = current_device(D);
        if (rc) return rc;
        batcube::CubePlan C;
        make_cubes(n, m, arcs, s, t, (flags & BAT_DIRECTED) != 0, C, first ? 0 : S.items / 32);
        uint64_t bits = fnv_bytes(1469598103934665603ull, C.arc_of_bit.data(), sizeof(int) * C.arc_of_bit.size());
        if (!first && (bits != S.bits || S.items != 32 * C.levels + C.rel_bits() || S.parts > cube_items(C) ||
                       !cube_shape_ok(C, grad, S.shape, cube_items(C) / S.parts)))
            return fail(BAT_EIO, "the checkpoint's work items are not the ones this library cuts");
        if (!first || cube_fits(C)) {
            if (first) {
                S.order = kPermInfluence;
                S.items = 32 * C.levels + C.rel_bits();
                S.chain = 0;
                S.bits = bits;
                S.parts = std::min<u64>(parts_wanted, cube_items(C));
            }
            u64 c = 0;
            std::vector<double> res;
            rc = cube_sync(C, p, D, grad, res, c, S.parts, S.done, &S.shape);
            if (rc) return rc;
            *count = c;
            R_hl[0] = res[0];
            R_hl[1] = res[1];
            if (grad) {
                std::vector<int> arc(m);
                for (int32_t a = 0; a < m; ++a) arc[a] = a;
                split_grad(res, arc, m, nullptr, T1, T0);
            }
            return BAT_OK;
        }
    }
    if (first) {
        int rc = whole_sweep_order(n, m, arcs, s, t, flags, grad, rq.force_perm);
        if (rc) return rc;
        rq.split_parts = parts_wanted;
        rq.fill = true;
    } else {
        rq.force_perm = S.order;
        rq.force_chunk_log2 = S.items;
        rq.force_chain = S.chain;
        rq.split_parts = S.parts;
    }
    rq.split_index = S.done;
    std::vector<double> res;
    std::vector<int> cba;
    u64 cnt = 0;
    int rc = run_sync(n, m, arcs, p, s, t, 0, 1ull << m, grad, res, cnt, &rq, &cba, flags);
    if (rc) return rc;
    if (first) {
        const bat_launch_info &I = t_state.info;
        const int ubits = m > bat::kWordBits ? m - bat::kWordBits : 0;
        S.order = I.perm;
        S.items = I.chunk_log2;
        S.chain = I.chain_log2;
        S.parts = std::min<u64>(parts_wanted, 1ull << std::max(ubits - S.items, 0));
    }
    R_hl[0] = res[0];
    R_hl[1] = res[1];
    *count = cnt;
    if (grad) split_grad(res, cba, m, nullptr, T1, T0);
    return BAT_OK;
}

}  // namespace

namespace {

// ------------------------------------------------------------ multi-state
// Arcs with sigma_i states (bat_ms.hip): validate, order the arcs for the
// flow searches, and sweep [c_lo, c_hi) of the mixed-radix counter.
int ms_validate(int32_t n, int32_t m, const bat_arc *arcs, const int32_t *sigma, const int32_t *cap, const double *w,
                int32_t s, int32_t t, int32_t d, uint32_t flags, u64 &N, int32_t &n_table)
{
    if (flags & ~(uint32_t)BAT_DIRECTED) return fail(BAT_EINVAL, "unknown flags 0x%x", flags);
    if (n < 2 || m < 0) return fail(BAT_EINVAL, "need n_nodes >= 2 and n_arcs >= 0 (got %d, %d)", n, m);
    if (n > batk::kMsMaxNodes || m > batk::kMsMaxArcs)
        return fail(BAT_ETOOBIG, "multi-state arcs: at most %d nodes and %d arcs (got %d, %d)", batk::kMsMaxNodes,
                    batk::kMsMaxArcs, n, m);
    if (s < 0 || s >= n || t < 0 || t >= n || s == t) return fail(BAT_EINVAL, "bad terminals s=%d t=%d", s, t);
    if (d < 1 || d > batk::kMsMaxDemand) return fail(BAT_EINVAL, "demand %d outside [1, %d]", d, batk::kMsMaxDemand);
    if (m > 0 && (!arcs || !sigma || !w)) return fail(BAT_EINVAL, "NULL arcs, n_states or probabilities");
    N = 1;
    n_table = 0;
    for (int32_t i = 0; i < m; ++i) {
        if (arcs[i].u < 0 || arcs[i].u >= n || arcs[i].v < 0 || arcs[i].v >= n)
            return fail(BAT_EINVAL, "arc %d has a node outside [0, %d)", i, n);
        if (sigma[i] < 1 || sigma[i] > batk::kMsMaxStates)
            return fail(BAT_EINVAL, "arc %d has %d states, outside [1, %d]", i, sigma[i], batk::kMsMaxStates);
        for (int32_t k = 0; k < sigma[i]; ++k) {
            const double x = w[n_table + k];
            if (!(x >= 0.0 && x <= 1.0)) return fail(BAT_EINVAL, "probability of arc %d state %d is %g", i, k, x);
            if (cap && (cap[n_table + k] < 0 || cap[n_table + k] > batk::kMsMaxCapacity))
                return fail(BAT_EINVAL, "capacity of arc %d state %d outside [0, %d]", i, k, batk::kMsMaxCapacity);
        }
        n_table += sigma[i];
        if (n_table > batk::kMsMaxTable)
            return fail(BAT_ETOOBIG, "more than %d (arc, state) pairs", batk::kMsMaxTable);
        if ((u64)sigma[i] > (1ull << 62) / N) return fail(BAT_ETOOBIG, "more than 2^62 state vectors");
        N *= (u64)sigma[i];
    }
    return BAT_OK;
}

// The sums of a multi-state sweep's work items, written by the device to the
// pinned `out` and waited for by its report, as a sub-cube sweep's (four
// events, a copy back and the stream's own wait took half of a small call:
// 3^9 vectors 62 us with them).  Clears the launch info.
int ms_finish(hipStream_t st, const DeviceInfo &D, double *part, u64 *pcount, u64 n_items, u64 *slot, u64 seq, char *out,
              double &R_hi, double &R_lo, u64 &count)
{
    bat::CubeParams K;
    memset(&K, 0, sizeof K);
    K.part = (bat::double2_t *)part;
    K.pcount = pcount;
    K.res = (double *)out;
    K.count = (u64 *)(out + 2 * sizeof(double));
    K.diag = slot;
    K.seq = seq;
    HIPCHK(batk::cube_finish(st, (unsigned)n_items, K));
    const int rc = cube_wait(K, st);
    if (rc) {
        (void)hipStreamSynchronize(st);
        return rc;
    }
    memcpy(&R_hi, out, sizeof(double));
    memcpy(&R_lo, out + sizeof(double), sizeof(double));
    memcpy(&count, out + 2 * sizeof(double), sizeof(u64));
    memset(&t_state.info, 0, sizeof t_state.info);
    t_state.cube_seq = seq;
    t_state.cube_slot = slot;
    t_state.cube_dev = D.id;
    t_state.cube_khz = D.clock_khz;
    t_state.have_launch = true;
    return BAT_OK;
}

// Demand <= 3: the bit-sliced kernel (ms_bits_kernel in bat_device.hpp)
// compiled for the graph and its states, over the vector indices
// [c_lo, c_hi) (slot 0 least significant).  Slots in sweep order: slot j
// joins su[j] and sv[j] and has sig[j] states whose capacities and
// probabilities are capt / wt at off[j].
int ms_bits_run(int32_t n, int32_t m, const int *su, const int *sv, const bat::u32 *sig, const bat::u32 *off,
                const std::vector<int32_t> &capt, const std::vector<double> &wt, int32_t s, int32_t t, int32_t d,
                bool directed, u64 c_lo, u64 c_hi, double &R_hi, double &R_lo, u64 &count, std::string *src_only)
{
    // word slots: the longest prefix whose states fit the 32 bits of a word
    int kw = 0;
    u64 B = 1;
    while (kw < m && B * sig[kw] <= 32) B *= sig[kw++];
    // the words the range touches
    const u64 w_lo = c_lo / B, w_hi = c_hi > c_lo ? (c_hi + B - 1) / B : w_lo;
    // run slots: as many as keep about 2^19 lane runs (32 wavefronts per
    // CU: the kernel is latency-bound; on the 3^18 workload runs of 27
    // steps took 0.94 ms, of 81 steps 1.15 ms, of 9 steps 1.09 ms) and a
    // run within 2^31 steps (option BAT_MS_RUN > 0: runs of at most that
    // many steps)
    const u64 want_run =
        opts().ms_run.load() > 0 ? (u64)opts().ms_run.load() : std::max<u64>(1, (w_hi - w_lo) >> 19);
    int kr = 0;
    u64 run = 1;
    while (kw + kr < m && run * sig[kw + kr] <= std::min<u64>(want_run, 1ull << 31)) run *= sig[kw + kr++];
    const u64 rl_lo = w_lo / run, rl_hi = (w_hi + run - 1) / run;
    const u64 n_lane = rl_hi - rl_lo;
    const u64 n_items = (n_lane + bat::kWave - 1) / bat::kWave;
    const u64 blocks = (n_items + bat::kWavesPerBlock - 1) / bat::kWavesPerBlock;
    if (blocks > 0x7fffffffull) return fail(BAT_ETOOBIG, "too many work items (%llu)", (unsigned long long)n_items);
    auto capof = [&](int j, u32 x) { return capt[off[j] + x]; };
    // the kernel's constants
    std::vector<u32> c1(m, 0u), ce1(m, 0u), ce12(m, 0u), ww1(m, 0u), wu1(m, 0u), wu12(m, 0u);
    u32 upair = 0u;
    for (int j = 0; j < m; ++j)
        for (u32 x = 0; x < sig[j]; ++x) {
            if (capof(j, x) >= 1) c1[j] |= 1u << x;
            if (capof(j, x) == 1) ce1[j] |= 1u << x;
            if (capof(j, x) == 1 || capof(j, x) == 2) ce12[j] |= 1u << x;
        }
    for (int j = 0; j < m; ++j)
        if (ce1[j]) upair |= 1u << j;
    u64 stride = 1;
    for (int j = 0; j < kw; ++j) {
        for (u64 b = 0; b < B; ++b) {
            const u32 x = (u32)((b / stride) % sig[j]);
            if (capof(j, x) >= 1) ww1[j] |= 1u << b;
            if (capof(j, x) == 1) wu1[j] |= 1u << b;
            if (capof(j, x) == 1 || capof(j, x) == 2) wu12[j] |= 1u << b;
        }
        stride *= sig[j];
    }
    const u32 full = B == 32 ? ~0u : (u32)((1ull << B) - 1ull);
    std::string g = "\nstruct JitMs {\n";
    auto num = [&](const char *k, u64 v) { g += std::string("  static constexpr unsigned ") + k + " = " + std::to_string(v) + "u;\n"; };
    num("N", (u64)n);
    num("S", (u64)s);
    num("T", (u64)t);
    num("M", (u64)m);
    num("KW", (u64)kw);
    num("KR", (u64)kr);
    num("D", (u64)d);
    num("B", B);
    num("FULL", full);
    num("RUN", run);
    num("UPAIR", upair);
    g += std::string("  static constexpr bool DIR = ") + (directed ? "true" : "false") + ";\n";
    auto arr = [&](const char *k, auto get) {
        g += std::string("  static constexpr unsigned ") + k + "[" + std::to_string(m) + "] = {";
        for (int j = 0; j < m; ++j) g += (j ? "," : "") + std::to_string((u64)get(j)) + "u";
        g += "};\n";
    };
    arr("NU", [&](int j) { return su[j]; });
    arr("NV", [&](int j) { return sv[j]; });
    arr("SIG", [&](int j) { return sig[j]; });
    arr("OFF", [&](int j) { return off[j]; });
    arr("C1", [&](int j) { return c1[j]; });
    arr("CE1", [&](int j) { return ce1[j]; });
    arr("CE12", [&](int j) { return ce12[j]; });
    arr("WW1", [&](int j) { return ww1[j]; });
    arr("WU1", [&](int j) { return wu1[j]; });
    arr("WU12", [&](int j) { return wu12[j]; });
    g += "};\n";
    g += "extern \"C\" __global__ void __launch_bounds__(256) bat_ms_bits(bat::MsBitsParams P) {\n"
         "  __shared__ double tb[4][256];\n"
         "  bat::ms_bits_kernel<JitMs>(P, tb);\n}\n";
    if (src_only) {
        *src_only = std::string(kDeviceSource) + g;
        return BAT_OK;
    }
    DeviceInfo D;
    int rc = current_device(D);
    if (rc) return rc;
    hipFunction_t fn;
    double jit_ms = 0.0;
    uint64_t kid = 0;
    const std::string key = std::to_string(D.id) + " ms" + g;
    if (!jit_ready(key, fn, kid)) {
        rc = jit_load(D, key, std::string(kDeviceSource) + g, "bat_ms_bits", fn, jit_ms, kid);
        if (rc) return rc;
    }
    hipStream_t st;
    rc = thread_stream(D.id, st);
    if (rc) return rc;
    // F tables of the word slots: Q_in(b) is the product of the word
    // slots' probabilities in vector b, TB_h[x] the sum of Q_in(8h + i)
    // over the bits i of x
    std::vector<double> qin(32, 0.0), tb(1024, 0.0);
    for (u64 b = 0; b < B; ++b) {
        double q = 1.0;
        u64 r = b;
        for (int j = 0; j < kw; ++j) {
            q *= wt[off[j] + (u32)(r % sig[j])];
            r /= sig[j];
        }
        qin[b] = q;
    }
    for (int h = 0; h < 4; ++h)
        for (int x = 0; x < 256; ++x) {
            double a = 0.0;
            for (int i = 0; i < 8; ++i)
                if ((x >> i) & 1) a += qin[8 * h + i];
            tb[256 * h + x] = a;
        }
    // workspace: input (tb | w) | partials | counts | output (res | count)
    const size_t o_tb = 0;
    const size_t o_w = align_up(o_tb + sizeof(double) * tb.size(), 256);
    const size_t in_bytes = align_up(o_w + sizeof(double) * (wt.size() + 1), 256);
    const u64 items = std::max<u64>(n_items, 1);
    const size_t o_part = in_bytes;
    const size_t o_pc = align_up(o_part + sizeof(double) * 2 * items, 256);
    const size_t o_res = align_up(o_pc + sizeof(u64) * items, 256);
    const size_t o_cnt = o_res + 2 * sizeof(double);
    const size_t out_bytes = o_cnt + sizeof(u64) - o_res;
    const size_t total = align_up(o_cnt + sizeof(u64) + 64, 256);
    Scratch *S = nullptr;
    const size_t out_host_off = in_bytes;
    rc = scratch_reserve(D.id, st, total, out_host_off + out_bytes, S);
    if (rc) return rc;
    char *ws = S->dev;
    memcpy(S->host + o_tb, tb.data(), sizeof(double) * tb.size());
    memcpy(S->host + o_w, wt.data(), sizeof(double) * wt.size());
    HIPCHK(hipMemcpyAsync(ws, S->host, in_bytes, hipMemcpyHostToDevice, st));
    bat::MsBitsParams K;
    memset(&K, 0, sizeof K);
    K.n_lane = n_lane;
    K.rl_base = rl_lo;
    K.c_lo = c_lo;
    K.c_hi = c_hi;
    K.n_items = n_items;
    K.tb = (const double *)(ws + o_tb);
    K.w = (const double *)(ws + o_w);
    K.part = (double *)(ws + o_part);
    K.pcount = (u64 *)(ws + o_pc);
    u64 seq = 0;
    rc = diag_next(st, K.diag, seq, Report::sync);
    if (rc) return rc;
    void *args[] = {&K};
    HIPCHK(hipModuleLaunchKernel(fn, (unsigned)std::max<u64>(blocks, 1), 1, 1,
                                 (unsigned)(bat::kWave * bat::kWavesPerBlock), 1, 1, 0, st, args, nullptr));
    rc = ms_finish(st, D, K.part, K.pcount, n_items, K.diag, seq, S->host + out_host_off, R_hi, R_lo, count);
    if (rc) return rc;
    bat_launch_info &I = t_state.info;
    I.vectors = c_hi - c_lo;
    I.n_chunks = (int32_t)std::min<u64>(n_items, 0x7fffffff);
    I.chunk_log2 = -1;
    I.relaxations = m;
    I.specialised = 1;
    I.jit_ms = jit_ms;
    I.kernel_id = kid;
    I.block_waves = bat::kWavesPerBlock;
    return BAT_OK;
}

// Most wavefronts of a multi-state launch, so that neither its threads (HIP's
// limit is 2^32) nor its partials grow with the space: past that each takes
// several work items, or there are several launches.
constexpr u64 kMsLaunchWaves = 65536;

// Fewest prefixes worth their own wavefronts: 3^16 vectors at demand 3 took 66
// us with 59049 prefixes and words of 27 cubes, 97 us with 531441 and words of
// 3; 3^15 98 us with 177147, 114 us with 19683, a wavefront per CU.
constexpr u64 kMsCubePrefixes = 32768;
// Vectors from which the cubes win.  Whole calls, cubes against every word by
// itself (10 nodes): 3^14 52 and 34 us at demand 1, 53 and 42 us at 2, 51 and
// 44 us at 3; 3^15 53 and 44, 56 and 71, 53 and 80 us; 3^17 57 and 74, 67 and
// 181, 282 and 851 us.
constexpr u64 ms_cube_vectors(int d) { return 1ull << (d == 1 ? 26 : 23); }

// A whole space with demand <= 3 by cubes (bat_ms_cube.hpp); slots as above,
// ordered by distance from the nearer terminal.
int ms_cubes_run(int32_t n, int32_t m, const int *su, const int *sv, const bat::u32 *sig, const bat::u32 *off,
                 const std::vector<int32_t> &capt, const std::vector<double> &wt, int32_t s, int32_t t, int32_t d,
                 bool directed, u64 N, double &R_hi, double &R_lo, u64 &count, std::string *src_only)
{
    // the two words: as many slots as fit 32 vectors each
    int kw = 0, kw1 = 0;
    u64 B0 = 1, B1 = 1;
    while (kw < m && B0 * sig[kw] <= 32) B0 *= sig[kw++];
    const u64 fewest = opts().cubes.load() == 1 ? 1 : kMsCubePrefixes;
    while (kw + kw1 < m && B1 * sig[kw + kw1] <= 32 && N / (B0 * B1 * sig[kw + kw1]) >= fewest)
        B1 *= sig[kw + kw1++];
    const u64 n_prefix = N / (B0 * B1), n_items = (n_prefix + bat::kWave - 1) / bat::kWave;
    const u64 n_waves = std::min(n_items, kMsLaunchWaves);
    const u64 blocks = (n_waves + bat::kMsCubeWaves - 1) / bat::kMsCubeWaves;
    auto kinds = [](int32_t c) { return (c >= 1 ? 1u : 0u) | (c == 1 ? 2u : 0u) | (c == 1 || c == 2 ? 4u : 0u); };
    std::vector<u32> c[3], word[3], lo(m, 0u), hi(m, 0u), m1(96, 0u);
    for (int k = 0; k < 3; ++k) {
        c[k].assign(m, 0u);
        word[k].assign(m, 0u);
    }
    // the tables are rounded once, from extended precision: their errors are
    // the same for every cube, and do not average out
    long double sum0 = 1.0L, q[2][32] = {};
    std::vector<double> q1(32, 0.0), tb(2048, 0.0);
    for (u64 b = 0; b < B0; ++b) q[0][b] = 1.0L;
    for (u64 b = 0; b < B1; ++b) q[1][b] = 1.0L;
    u64 stride = 1;
    u32 upair = 0u;
    for (int j = 0; j < m; ++j) {
        int32_t least = capt[off[j]], most = least;
        long double sum = 0.0L;
        for (u32 x = 0; x < sig[j]; ++x) {
            const int32_t cap = capt[off[j] + x];
            least = std::min(least, cap);
            most = std::max(most, cap);
            sum += wt[off[j] + x];
            for (int k = 0; k < 3; ++k) c[k][j] |= ((kinds(cap) >> k) & 1u) << x;
        }
        if (c[1][j]) upair |= 1u << j;
        if (j < kw) {
            lo[j] = kinds(least);
            hi[j] = kinds(most);
            sum0 *= sum;
        }
        if (j == kw) stride = 1;
        if (j < kw + kw1) {
            const int level = j < kw ? 0 : 1;
            for (u64 b = 0; b < (level ? B1 : B0); ++b) {
                const u32 x = (u32)((b / stride) % sig[j]);
                q[level][b] *= wt[off[j] + x];
                for (int k = 0; k < 3; ++k) {
                    word[k][j] |= ((c[k][j] >> x) & 1u) << b;
                    if (level) m1[32 * k + b] |= ((c[k][j] >> x) & 1u) << j;
                }
            }
            stride *= sig[j];
        }
    }
    for (u64 b = 0; b < B1; ++b) {
        q1[b] = (double)q[1][b];
        q[1][b] *= sum0;
    }
    for (int level = 0; level < 2; ++level)
        for (int h = 0; h < 4; ++h) {
            // (bytes of the bits that a word has)
            const int bits = std::max(0, std::min(8, (int)(level ? B1 : B0) - 8 * h));
            double *t = &tb[1024 * level + 256 * h];
            long double acc[256];
            acc[0] = 0.0L;
            for (int b = 0; b < bits; ++b) {
                const long double w = q[level][8 * h + b];
                for (int x = 0; x < 1 << b; ++x) {
                    acc[(1 << b) + x] = acc[x] + w;
                    t[(1 << b) + x] = (double)acc[(1 << b) + x];
                }
            }
        }
    // the closure, on slots
    std::vector<bat_arc> sa(m);
    std::vector<int> bit(m);
    for (int j = 0; j < m; ++j) {
        sa[j].u = su[j];
        sa[j].v = sv[j];
        bit[j] = j;
    }
    const batcube::Program pr = batcube::make_program(n, sa.data(), bit, s, t, 0, false, directed);
    std::string g = "\nstruct JitMs {\n";
    auto num = [&](const char *k, u64 v) { g += std::string("  static constexpr unsigned ") + k + " = " + std::to_string(v) + "u;\n"; };
    num("M", (u64)m);
    num("D", (u64)d);
    num("KW", (u64)kw);
    num("KW1", (u64)kw1);
    num("LOOP", n_items > n_waves ? 1u : 0u);
    num("B0", B0);
    num("FULL0", B0 == 32 ? 0xffffffffull : (1ull << B0) - 1ull);
    num("B1", B1);
    num("FULL1", B1 == 32 ? 0xffffffffull : (1ull << B1) - 1ull);
    num("UPAIR", upair);
    num("SLOTS", (u64)std::max(pr.slots, m));
    num("RESULT", pr.result < 0 ? 255ull : (u64)pr.result);
    auto arr = [&](const char *k, auto get) {
        g += std::string("  static constexpr unsigned ") + k + "[" + std::to_string(m) + "] = {";
        for (int j = 0; j < m; ++j) g += (j ? "," : "") + std::to_string((u64)get(j)) + "u";
        g += "};\n";
    };
    arr("SIG", [&](int j) { return sig[j]; });
    arr("OFF", [&](int j) { return off[j]; });
    arr("C1", [&](int j) { return c[0][j]; });
    arr("CE1", [&](int j) { return c[1][j]; });
    arr("CE12", [&](int j) { return c[2][j]; });
    arr("P1", [&](int j) { return word[0][j]; });
    arr("PE1", [&](int j) { return word[1][j]; });
    arr("PE12", [&](int j) { return word[2][j]; });
    arr("LO", [&](int j) { return lo[j]; });
    arr("HI", [&](int j) { return hi[j]; });
    g += "  __device__ static __forceinline__ void steps(unsigned (&r)[SLOTS]) {\n";
    for (const batcube::Step &x : pr.step) {
        const std::string a = "r[" + std::to_string(x.a) + "]", b = "r[" + std::to_string(x.b) + "]",
                          dd = "r[" + std::to_string(x.d) + "]";
        g += "    " + dd + (x.assign ? " = " + a + " & " + b : " = bat::and_or(" + a + ", " + b + ", " + dd + ")") + ";\n";
    }
    g += "  }\n};\n"
         "extern \"C\" __global__ void __launch_bounds__(256) bat_ms_cubes(bat::MsCubeParams P) {\n"
         "  __shared__ bat::MsCubeLds L;\n"
         "  bat::ms_cube_kernel<JitMs>(P, L);\n}\n";
    auto source = [&]() { return std::string(kDeviceSource) + kCubeSource + kMsCubeSource + g; };
    if (src_only) {
        *src_only = source();
        return BAT_OK;
    }
    DeviceInfo D;
    int rc = current_device(D);
    if (rc) return rc;
    hipFunction_t fn;
    double jit_ms = 0.0;
    uint64_t kid = 0;
    const std::string key = std::to_string(D.id) + " mscube" + g;
    if (!jit_ready(key, fn, kid)) {  // (the source is some 200 KiB)
        rc = jit_load(D, key, source(), "bat_ms_cubes", fn, jit_ms, kid);
        if (rc) return rc;
    }
    hipStream_t st;
    rc = thread_stream(D.id, st);
    if (rc) return rc;
    // workspace: input (tb | q1 | m1 | w) | partials | counts | output (res | count)
    const size_t o_q1 = sizeof(double) * tb.size(), o_m1 = o_q1 + sizeof(double) * 32, o_w = o_m1 + sizeof(u32) * 96;
    const size_t in_bytes = align_up(o_w + sizeof(double) * (wt.size() + 1), 256);
    const size_t o_part = in_bytes, o_pc = align_up(o_part + sizeof(double) * 2 * n_waves, 256);
    const size_t out_bytes = 2 * sizeof(double) + sizeof(u64);
    Scratch *S = nullptr;
    rc = scratch_reserve(D.id, st, o_pc + sizeof(u64) * n_waves, in_bytes + out_bytes, S);
    if (rc) return rc;
    memcpy(S->host, tb.data(), sizeof(double) * tb.size());
    memcpy(S->host + o_q1, q1.data(), sizeof(double) * 32);
    memcpy(S->host + o_m1, m1.data(), sizeof(u32) * 96);
    memcpy(S->host + o_w, wt.data(), sizeof(double) * wt.size());
    char *ws = S->dev;
    HIPCHK(hipMemcpyAsync(ws, S->host, in_bytes, hipMemcpyHostToDevice, st));
    bat::MsCubeParams K;
    memset(&K, 0, sizeof K);
    K.n_prefix = n_prefix;
    K.n_items = n_items;
    K.n_waves = n_waves;
    K.tb = (const double *)ws;
    K.q1 = (const double *)(ws + o_q1);
    K.m1 = (const u32 *)(ws + o_m1);
    K.w = (const double *)(ws + o_w);
    K.part = (double *)(ws + o_part);
    K.pcount = (u64 *)(ws + o_pc);
    u64 seq = 0;
    rc = diag_next(st, K.diag, seq, Report::sync);
    if (rc) return rc;
    void *args[] = {&K};
    HIPCHK(hipModuleLaunchKernel(fn, (unsigned)blocks, 1, 1, (unsigned)(bat::kWave * bat::kMsCubeWaves), 1, 1, 0, st, args,
                                 nullptr));
    rc = ms_finish(st, D, K.part, K.pcount, n_waves, K.diag, seq, S->host + in_bytes, R_hi, R_lo, count);
    if (rc) return rc;
    bat_launch_info &I = t_state.info;
    I.vectors = N;
    I.n_chunks = (int32_t)std::min<u64>(n_items, 0x7fffffff);
    I.chunk_log2 = -1;
    I.relaxations = m;
    I.specialised = 1;
    I.jit_ms = jit_ms;
    I.kernel_id = kid;
    I.perm = kPermInfluence;
    I.block_waves = bat::kMsCubeWaves;
    return BAT_OK;
}

int ms_run(int32_t n, int32_t m, const bat_arc *arcs, const int32_t *sigma, const int32_t *cap, const double *w,
           int32_t s, int32_t t, int32_t d, uint32_t flags, bool whole, u64 c_lo, u64 c_hi, double &R_hi,
           double &R_lo, u64 &count, std::string *src_only = nullptr)
{
    u64 N = 0;
    int32_t n_table = 0;
    int rc = ms_validate(n, m, arcs, sigma, cap, w, s, t, d, flags, N, n_table);
    if (rc) return rc;
    if (whole) {
        c_lo = 0;
        c_hi = N;
    }
    if (c_lo > c_hi || c_hi > N)
        return fail(BAT_EINVAL, "range [%llu, %llu) outside [0, %llu)", (unsigned long long)c_lo,
                    (unsigned long long)c_hi, (unsigned long long)N);
    // Slots: the kernel sweeps arcs in slot order, and slot 0 is the
    // fastest-changing coordinate of its index.  A whole space may take any
    // arc order (R and the count are sums over every vector): for the
    // bit-sliced kernel arcs near s first, by breadth-first distance of their
    // nearer end, so one search sweep reaches far; for the flow kernel, whose
    // cubes leave the lowest slots free, the arcs farthest from both
    // terminals first.  A range reads its indices in the caller's order,
    // arc 0 most significant: slot j is arc m - 1 - j.
    const bool bits = d <= 3 && m > 0 && c_hi > c_lo && opts().ms_bits.load() != 0;
    const int64_t want_cubes = opts().cubes.load();
    const bool cubes = bits && whole && opts().ms_run.load() <= 0 &&
                       (want_cubes == 1 || (want_cubes != 0 && N >= ms_cube_vectors(d)));
    std::vector<int> ord(m);
    for (int i = 0; i < m; ++i) ord[i] = whole ? i : m - 1 - i;
    if (whole && m > 1) {
        auto distances = [&](int from) {
            std::vector<int> dist(n, 1 << 30);
            std::vector<int> q{from};
            dist[from] = 0;
            for (size_t h = 0; h < q.size(); ++h)
                for (int i = 0; i < m; ++i) {
                    const int a = arcs[i].u, b = arcs[i].v, x = q[h];
                    const int y = a == x ? b : (b == x ? a : -1);
                    if (y >= 0 && dist[y] > dist[x] + 1) {
                        dist[y] = dist[x] + 1;
                        q.push_back(y);
                    }
                }
            return dist;
        };
        const std::vector<int> dist = distances(s), back = bits && !cubes ? std::vector<int>() : distances(t);
        auto key = [&](int i) {
            const int a = dist[arcs[i].u], b = dist[arcs[i].v];
            if (!bits || cubes) return std::make_pair(-std::min({a, b, back[arcs[i].u], back[arcs[i].v]}), 0);
            return std::make_pair(std::min(a, b), std::max(a, b));
        };
        std::stable_sort(ord.begin(), ord.end(), [&](int x, int y) { return key(x) < key(y); });
    }
    batk::MsParams K;
    memset(&K, 0, sizeof K);
    K.m = (u32)m;
    K.n = (u32)n;
    K.s = (u32)s;
    K.t = (u32)t;
    K.d = (u32)d;
    K.directed = (flags & BAT_DIRECTED) ? 1u : 0u;
    K.n_table = (u32)n_table + (u32)(batk::ms_slots(m) - m);
    std::vector<int> first(m + 1, 0);
    for (int i = 0; i < m; ++i) first[i + 1] = first[i] + sigma[i];
    // the kernel instance's slot count; the slots past the last arc are
    // one-state self-loops at s (capacity 0, probability 1): no-ops
    const int slots = batk::ms_slots(m);
    std::vector<int32_t> capt(n_table + (slots - m));
    std::vector<double> wt(n_table + (slots - m));
    u32 o = 0;
    for (int j = m; j < slots; ++j) {
        K.sig[j] = 1u;
        K.off[j] = (u32)(n_table + (j - m));
        K.u[j] = K.v[j] = (unsigned char)s;
        capt[n_table + (j - m)] = 0;
        wt[n_table + (j - m)] = 1.0;
    }
    for (int j = 0; j < m; ++j) {
        const int i = ord[j];
        K.sig[j] = (u32)sigma[i];
        K.off[j] = o;
        K.u[j] = (unsigned char)arcs[i].u;
        K.v[j] = (unsigned char)arcs[i].v;
        for (int k = 0; k < sigma[i]; ++k) {
            capt[o + k] = cap ? cap[first[i] + k] : k;
            wt[o + k] = w[first[i] + k];
        }
        o += (u32)sigma[i];
    }
    // demand 1 to 3: the bit-sliced kernel
    if (bits) {
        std::vector<int> su(m), sv(m);
        for (int j = 0; j < m; ++j) {
            su[j] = K.u[j];
            sv[j] = K.v[j];
        }
        if (cubes)
            return ms_cubes_run(n, m, su.data(), sv.data(), K.sig, K.off, capt, wt, s, t, d, K.directed != 0, N, R_hi,
                                R_lo, count, src_only);
        return ms_bits_run(n, m, su.data(), sv.data(), K.sig, K.off, capt, wt, s, t, d, K.directed != 0, c_lo, c_hi,
                           R_hi, R_lo, count, src_only);
    }
    if (src_only) return fail(BAT_EINVAL, "no bit-sliced kernel for this sweep (it needs demand 1 to 3 and arcs)");
    // cubes of the L lowest slots: as large as leave some 1024 work items of
    // 64 (3^15 vectors, demand 4: 0.28 ms with 2768 items, 0.36 ms with 923,
    // 0.39 ms with 8304; option BAT_MS_RUN > 0: of at most that many vectors)
    const u64 span = c_hi - c_lo;
    // The first slot already where that leaves 512: a cube of one free slot is
    // decided whole, by one flow and its bound (6^7 vectors, demand 11: 60 us
    // with 729 items, 75 us with 4374 of single vectors; 8^6: 68 us with 512,
    // 79 us; 5^7 even with 244).
    const u64 most_size = opts().ms_run.load() > 0 ? (u64)opts().ms_run.load()
                                                   : std::max<u64>(1, span / (64 * 1024));
    const u64 first_size = opts().ms_run.load() > 0 ? most_size : std::max<u64>(1, span / (64 * 512));
    K.size[0] = 1;
    K.weight[0] = 1.0;
    for (int j = 0; j < slots; ++j) {
        K.least[j] = K.most[j] = capt[K.off[j]];
        double sum = 0.0;
        for (u32 k = 0; k < K.sig[j]; ++k) {
            K.least[j] = std::min(K.least[j], capt[K.off[j] + k]);
            K.most[j] = std::max(K.most[j], capt[K.off[j] + k]);
            sum += wt[K.off[j] + k];
        }
        if (j == (int)K.L && j < std::min<int>(m, batk::kMsTreeSlots) &&
            K.size[j] * K.sig[j] <= (j ? most_size : first_size)) {
            K.size[j + 1] = K.size[j] * K.sig[j];
            K.weight[j + 1] = K.weight[j] * sum;
            K.most_states = std::max(K.most_states, K.sig[j]);
            K.L = (u32)(j + 1);
        }
    }
    // roots: those cubes.  A launch takes at most kMsLaunchWaves work items of 64;
    // longer ranges go in several, one after the other
    const u64 size_L = K.size[K.L], root_end = span ? (c_hi + size_L - 1) / size_L : c_lo / size_L;
    const u64 n_items = (root_end - c_lo / size_L + 63) / 64;
    DeviceInfo D;
    rc = current_device(D);
    if (rc) return rc;
    hipStream_t st;
    rc = thread_stream(D.id, st);
    if (rc) return rc;
    // workspace: input (cap | w tables) | partials | counts | output (res | count)
    const size_t n_tab = capt.size();
    const size_t o_cap = 0;
    const size_t o_w = align_up(o_cap + sizeof(int32_t) * (n_tab + 1), 256);
    const size_t in_bytes = align_up(o_w + sizeof(double) * (n_tab + 1), 256);
    const u64 items = std::min(std::max<u64>(n_items, 1), kMsLaunchWaves);
    const size_t o_part = in_bytes;
    const size_t o_pc = align_up(o_part + sizeof(double) * 2 * items, 256);
    const size_t total = align_up(o_pc + sizeof(u64) * items, 256);
    const size_t out_bytes = 2 * sizeof(double) + sizeof(u64);
    Scratch *S = nullptr;
    const size_t out_host_off = in_bytes;
    rc = scratch_reserve(D.id, st, total, out_host_off + out_bytes, S);
    if (rc) return rc;
    char *ws = S->dev;
    memcpy(S->host + o_cap, capt.data(), sizeof(int32_t) * n_tab);
    memcpy(S->host + o_w, wt.data(), sizeof(double) * n_tab);
    HIPCHK(hipMemcpyAsync(ws, S->host, in_bytes, hipMemcpyHostToDevice, st));
    K.cap = (const int *)(ws + o_cap);
    K.w = (const double *)(ws + o_w);
    K.part = (double *)(ws + o_part);
    K.pcount = (u64 *)(ws + o_pc);
    double sum[2] = {0.0, 0.0};
    u64 number = 0, start = 0;
    K.root_hi = c_lo / size_L;
    do {
        K.root_lo = K.root_hi;
        K.root_hi = std::min(K.root_lo + 64 * kMsLaunchWaves, root_end);
        K.n_items = (K.root_hi - K.root_lo + 63) / 64;
        K.c_lo = std::max(c_lo, K.root_lo * size_L);
        K.c_hi = std::min(c_hi, K.root_hi * size_L);
        const u64 blocks = (K.n_items + bat::kWavesPerBlock - 1) / bat::kWavesPerBlock;
        u64 seq = 0;
        rc = diag_next(st, K.diag, seq, Report::sync);
        if (rc) return rc;
        HIPCHK(batk::ms_sweep(st, (unsigned)std::max<u64>(blocks, 1), K));
        rc = ms_finish(st, D, K.part, K.pcount, K.n_items, K.diag, seq, S->host + out_host_off, R_hi, R_lo, count);
        if (rc) return rc;
        dd_acc(sum, R_hi, R_lo);
        number += count;
        // the launch report covers all of them
        if (!start) start = K.diag[0];
        K.diag[0] = start;
    } while (K.root_hi < root_end);
    R_hi = sum[0];
    R_lo = sum[1];
    count = number;
    bat_launch_info &I = t_state.info;
    I.vectors = span;
    I.n_chunks = (int32_t)std::min<u64>(n_items, 0x7fffffff);
    I.chunk_log2 = -1;
    I.relaxations = m;
    I.kernel_id = aot_kernel_id("k_ms_flow", batk::ms_slots(m), K.directed != 0);
    I.block_waves = bat::kWavesPerBlock;
    return BAT_OK;
}

}  // namespace

// ====================================================================== C ABI
extern "C" {

const char *bat_version(void) { return kVersion; }

const char *bat_last_error(void) { return t_err.c_str(); }

int bat_set_option(const char *key, int64_t value)
{
    auto *o = opts().find(key);
    if (!o) return fail(BAT_EINVAL, "unknown option '%s'", key ? key : "(null)");
    if (!strcmp(key, "BAT_JIT_FLUSH")) {  // an action, not a setting
        if (value) jit_flush();
        return BAT_OK;
    }
    *o = value;
    return BAT_OK;
}

int bat_get_option(const char *key, int64_t *value)
{
    auto *o = opts().find(key);
    if (!o || !value) return fail(BAT_EINVAL, "unknown option '%s'", key ? key : "(null)");
    *value = o->load();
    return BAT_OK;
}

int bat_reliability_ex(int32_t n, int32_t m, const bat_arc *arcs, const double *p, int32_t s, int32_t t,
                       uint32_t flags, double *R_out, uint64_t *count_out, double *dRdp_out, double *T1_out,
                       double *T0_out)
{
    t_err.clear();
    if (!R_out || !count_out) return fail(BAT_EINVAL, "NULL output pointer");
    if (flags & ~(uint32_t)(BAT_DIRECTED | BAT_FORWARD_ORDER)) return fail(BAT_EINVAL, "unknown flags 0x%x", flags);
    if (m < 0 || m > BAT_MAX_ARCS) return validate(n, m, arcs, p, s, t);
    const bool grad = dRdp_out || T1_out || T0_out;
    std::vector<double> res;
    std::vector<int> cba;
    u64 cnt = 0;
    // a whole sweep: the index order does not matter, any arc order is used
    int rc = run_sync(n, m, arcs, p, s, t, 0, 1ull << m, grad, res, cnt, nullptr, &cba, flags);
    if (rc) return rc;
    *R_out = res[0] + res[1];
    *count_out = cnt;
    if (grad) split_grad(res, cba, m, dRdp_out, T1_out, T0_out);
    return BAT_OK;
}

int bat_reliability(int32_t n, int32_t m, const bat_arc *arcs, const double *p, int32_t s, int32_t t,
                    double *R_out, uint64_t *count_out)
{
    return bat_reliability_ex(n, m, arcs, p, s, t, 0u, R_out, count_out, nullptr, nullptr, nullptr);
}

int bat_reliability_grad(int32_t n, int32_t m, const bat_arc *arcs, const double *p, int32_t s, int32_t t,
                         double *R_out, uint64_t *count_out, double *dRdp_out, double *T1_out, double *T0_out)
{
    t_err.clear();
    if (!dRdp_out && m > 0) return fail(BAT_EINVAL, "NULL output pointer");
    if (m == 0) {  // no arcs: no gradient to write, R = 0 from the forward sweep
        return bat_reliability_ex(n, m, arcs, p, s, t, 0u, R_out, count_out, nullptr, nullptr, nullptr);
    }
    return bat_reliability_ex(n, m, arcs, p, s, t, 0u, R_out, count_out, dRdp_out, T1_out, T0_out);
}

int bat_reliability_range_ex(int32_t n, int32_t m, const bat_arc *arcs, const double *p, int32_t s, int32_t t,
                             uint32_t flags, uint64_t c_lo, uint64_t c_hi, double *R_hi, double *R_lo,
                             uint64_t *count_out, double *T1_out, double *T0_out)
{
    t_err.clear();
    if (!R_hi || !R_lo || !count_out) return fail(BAT_EINVAL, "NULL output pointer");
    if ((T1_out == nullptr) != (T0_out == nullptr)) return fail(BAT_EINVAL, "T1_out and T0_out must both be set or both NULL");
    if (flags & ~(uint32_t)(BAT_DIRECTED | BAT_FORWARD_ORDER)) return fail(BAT_EINVAL, "unknown flags 0x%x", flags);
    if (m < 0 || m > BAT_MAX_ARCS) return validate(n, m, arcs, p, s, t);
    if (c_lo > c_hi || c_hi > (1ull << m)) return fail(BAT_EINVAL, "bad range [%llu, %llu) for m = %d",
                                                     (unsigned long long)c_lo, (unsigned long long)c_hi, m);
    if (!T1_out && !(flags & BAT_DIRECTED) && c_lo < c_hi && (p || m == 0) && cubes_wanted()) {
        int rc = validate(n, m, arcs, p, s, t);
        DeviceInfo D;
        if (!rc) rc = current_device(D);
        if (rc) return rc;
        double R[2];
        u64 count = 0;
        bool fits = false;
        rc = range_cubes(n, m, arcs, p, s, t, D, (flags & BAT_FORWARD_ORDER) != 0, c_lo, c_hi, R, count, fits);
        if (rc) return rc;
        if (fits) {
            *R_hi = R[0];
            *R_lo = R[1];
            *count_out = count;
            return BAT_OK;
        }
    }
    // the indices are the paper's: backward BAT (Eq. 2-3) or forward (Eq. 4-5)
    return range_in_order(n, m, arcs, p, s, t, flags, (flags & BAT_FORWARD_ORDER) ? kPermForward : 0, c_lo, c_hi,
                          R_hi, R_lo, count_out, T1_out, T0_out);
}

int bat_reliability_range(int32_t n, int32_t m, const bat_arc *arcs, const double *p, int32_t s, int32_t t,
                          uint64_t c_lo, uint64_t c_hi, double *R_hi, double *R_lo, uint64_t *count_out,
                          double *T1_out, double *T0_out)
{
    return bat_reliability_range_ex(n, m, arcs, p, s, t, 0u, c_lo, c_hi, R_hi, R_lo, count_out, T1_out, T0_out);
}

int bat_reliability_checkpointed(int32_t n, int32_t m, const bat_arc *arcs, const double *p, int32_t s, int32_t t,
                                 uint32_t flags, int32_t chunk_log2, const char *path, int64_t max_chunks,
                                 double *R_out, uint64_t *count_out, double *dRdp_out, double *T1_out,
                                 double *T0_out)
{
    t_err.clear();
    if (!R_out || !count_out) return fail(BAT_EINVAL, "NULL output pointer");
    if (flags & ~(uint32_t)(BAT_DIRECTED | BAT_FORWARD_ORDER)) return fail(BAT_EINVAL, "unknown flags 0x%x", flags);
    if (chunk_log2 < 0 || chunk_log2 > BAT_MAX_ARCS)
        return fail(BAT_EINVAL, "chunk_log2 %d outside [0, %d]", chunk_log2, BAT_MAX_ARCS);
    if (!p && m > 0) return fail(BAT_EINVAL, "p is NULL");
    int rc = validate(n, m, arcs, p, s, t);
    if (rc) return rc;
    const bool grad = dRdp_out || T1_out || T0_out;
    const int32_t clog = chunk_log2 < m ? chunk_log2 : m;
    const u64 parts_wanted = 1ull << (m - clog);
    const std::string problem = checkpoint_problem(n, m, arcs, p, s, t, flags, chunk_log2, grad);
    RunningSums S;
    if (grad) {
        S.T1.assign(2 * (size_t)m, 0.0);
        S.T0.assign(2 * (size_t)m, 0.0);
    }
    if (path) {
        rc = checkpoint_read(path, problem, grad, m, flags, S);
        if (rc < 0) return rc;
    }
    std::vector<double> t1(m > 0 ? m : 1), t0(m > 0 ? m : 1);
    for (int64_t ran = 0; (S.parts == 0 || S.done < S.parts) && (max_chunks < 0 || ran < max_chunks); ++ran) {
        double hl[2] = {0.0, 0.0};
        uint64_t c = 0;
        rc = run_part(n, m, arcs, p, s, t, flags, grad, parts_wanted, S, hl, &c, grad ? t1.data() : nullptr,
                      grad ? t0.data() : nullptr);
        if (rc) return rc;
        dd_acc(S.R, hl[0], hl[1]);
        S.count += c;
        for (int32_t a = 0; grad && a < m; ++a) {
            dd_acc(&S.T1[2 * a], t1[a], 0.0);
            dd_acc(&S.T0[2 * a], t0[a], 0.0);
        }
        ++S.done;
        if (path) {
            rc = checkpoint_write(path, problem, grad, S);
            if (rc) return rc;
        }
    }
    if (S.parts == 0 || S.done < S.parts) return BAT_PENDING;
    *R_out = S.R[0] + S.R[1];
    *count_out = S.count;
    for (int32_t a = 0; grad && a < m; ++a) {
        const double *a1 = &S.T1[2 * a], *a0 = &S.T0[2 * a];
        if (dRdp_out) dRdp_out[a] = (a1[0] - a0[0]) + (a1[1] - a0[1]);
        if (T1_out) T1_out[a] = a1[0] + a1[1];
        if (T0_out) T0_out[a] = a0[0] + a0[1];
    }
    return BAT_OK;
}

static int async_common(int32_t n, int32_t m, const bat_arc *arcs, const double *p_dev, int32_t s, int32_t t,
                        double *R_dev, uint64_t *count_dev, bool grad, double *dRdp_dev, double *T1_dev,
                        double *T0_dev, int32_t *status_dev, void *stream)
{
    t_err.clear();
    if (!R_dev || !count_dev || (grad && !dRdp_dev && m > 0)) return fail(BAT_EINVAL, "NULL output pointer");
    if (m > 0 && !p_dev) return fail(BAT_EINVAL, "p_dev is NULL");
    Prepared X;
    TuneChoice tc;
    hipStream_t st = (hipStream_t)stream;
    int rc;
    if (cubes_wanted()) {
        rc = validate(n, m, arcs, nullptr, s, t);
        if (!rc) rc = current_device(X.D);
        if (rc) return rc;
        batcube::CubePlan C;
        make_cubes(n, m, arcs, s, t, false, C);
        if (cube_fits(C))
            return cube_async(C, p_dev, X.D, st, grad, R_dev, (u64 *)count_dev, dRdp_dev, T1_dev, T0_dev,
                              (int *)status_dev, nullptr, 0);
    }
    rc = prepare(n, m, arcs, nullptr, s, t, grad, true, nullptr, X, tc);
    if (rc) return rc;
    Request rq{};
    rq.n = n; rq.m = m; rq.s = s; rq.t = t; rq.arcs = arcs; rq.p_dev = p_dev;
    rq.c_lo = 0; rq.c_hi = 1ull << m; rq.grad = grad;
    Launch L;
    rc = queue_sweep(rq, X.P, X.D, tc, st, L);
    if (rc) {
        if (L.ws) (void)hipFreeAsync(L.ws, st);
        return rc;
    }
    HIPCHK(batk::finalize(st, (const double *)L.res, (const u64 *)L.count, (const int *)L.status, L.cb_of_arc,
                          (u32)m, grad, R_dev, (u64 *)count_dev, dRdp_dev, T1_dev, T0_dev, (int *)status_dev));
    HIPCHK(hipFreeAsync(L.ws, st));
    return BAT_OK;
}

int bat_reliability_async(int32_t n, int32_t m, const bat_arc *arcs, const double *p_dev, int32_t s, int32_t t,
                          double *R_dev, uint64_t *count_dev, int32_t *status_dev, void *stream)
{
    return async_common(n, m, arcs, p_dev, s, t, R_dev, count_dev, false, nullptr, nullptr, nullptr, status_dev,
                        stream);
}

int bat_reliability_grad_async(int32_t n, int32_t m, const bat_arc *arcs, const double *p_dev, int32_t s,
                               int32_t t, double *R_dev, uint64_t *count_dev, double *dRdp_dev, double *T1_dev,
                               double *T0_dev, int32_t *status_dev, void *stream)
{
    return async_common(n, m, arcs, p_dev, s, t, R_dev, count_dev, true, dRdp_dev, T1_dev, T0_dev, status_dev,
                        stream);
}

int bat_reliability_noalloc(int32_t n, int32_t m, const bat_arc *arcs, const double *p_dev, int32_t s, int32_t t,
                            double *R_dev, uint64_t *count_dev, int32_t *status_dev, void *stream)
{
    t_err.clear();
    if (!R_dev || !count_dev) return fail(BAT_EINVAL, "NULL output pointer");
    if (m > 0 && !p_dev) return fail(BAT_EINVAL, "p_dev is NULL");
    Prepared X;
    TuneChoice tc;
    int rc = validate(n, m, arcs, nullptr, s, t);
    if (!rc) rc = current_device(X.D);
    if (rc) return rc;
    // set-up on this device's first call: the address of its scratch copy
    char *ws = nullptr;
    rc = noalloc_scratch(X.D.id, ws);
    if (rc) return rc;
    hipStream_t st = (hipStream_t)stream;
    if (cubes_wanted()) {
        batcube::CubePlan C;
        make_cubes(n, m, arcs, s, t, false, C);
        if (cube_fits(C, true))
            return cube_async(C, p_dev, X.D, st, false, R_dev, (u64 *)count_dev, nullptr, nullptr, nullptr,
                              (int *)status_dev, ws, kNoAllocScratchBytes);
    }
    rc = prepare(n, m, arcs, nullptr, s, t, false, true, nullptr, X, tc);
    if (rc) return rc;
    Request rq{};
    rq.n = n; rq.m = m; rq.s = s; rq.t = t; rq.arcs = arcs; rq.p_dev = p_dev;
    rq.c_lo = 0; rq.c_hi = 1ull << m; rq.grad = false;
    Launch L;
    rc = queue_sweep(rq, X.P, X.D, tc, st, L, nullptr, ws, kNoAllocScratchBytes);
    if (rc) return rc;
    HIPCHK(batk::finalize(st, (const double *)L.res, (const u64 *)L.count, (const int *)L.status, L.cb_of_arc,
                          (u32)m, false, R_dev, (u64 *)count_dev, nullptr, nullptr, nullptr, (int *)status_dev));
    return BAT_OK;
}

int bat_ms_reliability(int32_t n, int32_t m, const bat_arc *arcs, const int32_t *n_states, const int32_t *capacity,
                       const double *w, int32_t s, int32_t t, int32_t demand, uint32_t flags, double *R_out,
                       uint64_t *count_out)
{
    t_err.clear();
    if (!R_out || !count_out) return fail(BAT_EINVAL, "NULL output pointer");
    double hi = 0.0, lo = 0.0;
    u64 c = 0;
    int rc = ms_run(n, m, arcs, n_states, capacity, w, s, t, demand, flags, true, 0, 0, hi, lo, c);
    if (rc) return rc;
    *R_out = hi + lo;
    *count_out = c;
    return BAT_OK;
}

int bat_ms_reliability_range(int32_t n, int32_t m, const bat_arc *arcs, const int32_t *n_states,
                             const int32_t *capacity, const double *w, int32_t s, int32_t t, int32_t demand,
                             uint32_t flags, uint64_t c_lo, uint64_t c_hi, double *R_hi, double *R_lo,
                             uint64_t *count_out)
{
    t_err.clear();
    if (!R_hi || !R_lo || !count_out) return fail(BAT_EINVAL, "NULL output pointer");
    double hi = 0.0, lo = 0.0;
    u64 c = 0;
    int rc = ms_run(n, m, arcs, n_states, capacity, w, s, t, demand, flags, false, c_lo, c_hi, hi, lo, c);
    if (rc) return rc;
    *R_hi = hi;
    *R_lo = lo;
    *count_out = c;
    return BAT_OK;
}

int bat_valu_peak(double *lane_ops_per_s)
{
    t_err.clear();
    if (!lane_ops_per_s) return fail(BAT_EINVAL, "NULL output pointer");
    DeviceInfo D;
    int rc = current_device(D);
    if (rc) return rc;
    hipStream_t st;
    rc = thread_stream(D.id, st);
    if (rc) return rc;
    rc = events_ready();
    if (rc) return rc;
    void *sink = nullptr;
    HIPCHK(hipMallocAsync(&sink, 64 * sizeof(u32), st));
    // 64 blocks of 256 threads per CU; 2048 trips of 16 instructions each
    const unsigned blocks = (unsigned)std::max(D.cus, 1) * 64u;
    const u32 iters = 2048;
    const double ops = (double)blocks * 256.0 * iters * batk::kValuPeakOpsPerTrip;
    double best = 0.0;
    hipError_t e = hipSuccess;
    for (int rep = 0; rep < 4 && e == hipSuccess; ++rep) {  // the first is a warm-up
        float ms = 0.0f;
        e = hipEventRecord(t_state.ev[0], st);
        if (e == hipSuccess) e = batk::valu_peak(st, blocks, iters, (u32 *)sink);
        if (e == hipSuccess) e = hipEventRecord(t_state.ev[1], st);
        if (e == hipSuccess) e = hipEventSynchronize(t_state.ev[1]);
        if (e == hipSuccess) e = hipEventElapsedTime(&ms, t_state.ev[0], t_state.ev[1]);
        if (e == hipSuccess && rep > 0 && ms > 0.0f) best = std::max(best, ops / (ms * 1e-3));
    }
    const hipError_t ef = hipFreeAsync(sink, st);
    if (e == hipSuccess) e = ef;
    if (e == hipSuccess) e = hipStreamSynchronize(st);
    if (e != hipSuccess) return fail(BAT_EDEVICE, "bat_valu_peak: %s", hipGetErrorString(e));
    *lane_ops_per_s = best;
    return BAT_OK;
}

int bat_last_launch(bat_launch_info *info)
{
    if (!info) return fail(BAT_EINVAL, "NULL info");
    if (!t_state.have_launch) return fail(BAT_EINVAL, "no launch on this thread yet");
    if (t_state.cube_seq) {
        const u64 *d = t_state.cube_slot;
        if (!d) return fail(BAT_EDEVICE, "the last launch was captured: it has no times");
        if (!diag_done(d, t_state.cube_seq)) {
            // wait for its stream, not for the device, which other streams may
            // keep busy; a stream captured itself cannot be waited for, one
            // destroyed since leaves only the device.  (Relaxed: the thread
            // may be capturing another stream, which this does not touch.)
            hipStreamCaptureMode mode = hipStreamCaptureModeRelaxed;
            HIPCHK(hipThreadExchangeStreamCaptureMode(&mode));
            hipStreamCaptureStatus cs = hipStreamCaptureStatusNone;
            hipError_t e = t_state.cube_stream ? hipStreamIsCapturing(t_state.cube_stream, &cs) : hipSuccess;
            if (e == hipSuccess && cs == hipStreamCaptureStatusNone) e = hipStreamSynchronize(t_state.cube_stream);
            if (e != hipSuccess) {
                (void)hipGetLastError();
                int dev = 0;
                e = hipGetDevice(&dev);
                if (e == hipSuccess) e = hipSetDevice(t_state.cube_dev);
                if (e == hipSuccess) e = hipDeviceSynchronize();
                (void)hipSetDevice(dev);
            }
            (void)hipThreadExchangeStreamCaptureMode(&mode);
            HIPCHK(e);
        }
        // no times where an older launch ended later, in this one's slot
        const u64 t0 = d[0], t1 = d[1], t2 = d[2];
        const bool got = diag_done(d, t_state.cube_seq) && t0 <= t1 && t1 <= t2;
        const double khz = std::max(t_state.cube_khz, 1);
        t_state.info.kernel_ms = got ? (double)(t1 - t0) / khz : 0.0;
        t_state.info.total_ms = got ? (double)(t2 - t0) / khz : 0.0;
        *info = t_state.info;
        return BAT_OK;
    }
    HIPCHK(hipEventSynchronize(t_state.ev[3]));
    float k = 0.f, tot = 0.f;
    HIPCHK(hipEventElapsedTime(&k, t_state.ev[1], t_state.ev[2]));
    HIPCHK(hipEventElapsedTime(&tot, t_state.ev[0], t_state.ev[3]));
    t_state.info.kernel_ms = k;
    t_state.info.total_ms = tot;
    *info = t_state.info;
    return BAT_OK;
}

int bat_jit_source(int32_t n, int32_t m, const bat_arc *arcs, int32_t s, int32_t t, uint32_t flags, int32_t grad,
                   int32_t perm, char *buf, uint64_t *len)
{
    t_err.clear();
    if (!len) return fail(BAT_EINVAL, "len is NULL");
    if (flags & ~(uint32_t)BAT_DIRECTED) return fail(BAT_EINVAL, "unknown flags 0x%x", flags);
    int rc = validate(n, m, arcs, nullptr, s, t);
    if (rc) return rc;
    if ((perm < 0 || perm >= kPermKinds) && perm != kPermInfluence)
        return fail(BAT_EINVAL, "perm %d outside [0, %d)", perm, kPermKinds);
    if (perm == kPermInfluence && grad < 0) return fail(BAT_EINVAL, "no batched sub-cube sweep of one graph");
    if (grad < -batk::kBatchMaxP || grad > 1) return fail(BAT_EINVAL, "grad %d outside [-%d, 1]", grad, batk::kBatchMaxP);
    if (grad < 0 && (flags & BAT_DIRECTED)) return fail(BAT_EINVAL, "the batched sweep is undirected");
    Plan P;
    batcube::CubePlan C;
    if (perm == kPermInfluence) make_cubes(n, m, arcs, s, t, (flags & BAT_DIRECTED) != 0, C);
    else make_plan(n, m, arcs, s, t, P, perm, (flags & BAT_DIRECTED) != 0);
    Options &O = opts();
    const std::string src =
        perm == kPermInfluence ? cube_source(C, grad != 0, true)
        : grad < 0 ? jit_source(P, false, jit_shape(false, 4, 0, 0, 1), -grad)
                 : jit_source(P, grad != 0,
                              jit_shape(grad != 0, (int)O.block_waves.load(), (int)O.super_restart.load(),
                                        (int)O.simd_waves.load(), (int)O.keep_bottom.load()));
    const uint64_t need = (uint64_t)src.size() + 1;
    const uint64_t have = *len;
    *len = need;
    if (!buf) return BAT_OK;
    if (have < need) return fail(BAT_ETOOBIG, "buffer of %llu bytes, need %llu", (unsigned long long)have,
                                 (unsigned long long)need);
    memcpy(buf, src.c_str(), need);
    return BAT_OK;
}

int bat_ms_jit_source(int32_t n, int32_t m, const bat_arc *arcs, const int32_t *n_states, const int32_t *capacity,
                      int32_t s, int32_t t, int32_t demand, uint32_t flags, uint64_t c_lo, uint64_t c_hi, char *buf,
                      uint64_t *len)
{
    t_err.clear();
    if (!len) return fail(BAT_EINVAL, "len is NULL");
    if (m > 0 && !n_states) return fail(BAT_EINVAL, "NULL n_states");
    // the source does not depend on the probabilities: any valid ones
    int64_t pairs = 0;
    for (int32_t i = 0; i < m; ++i) pairs += n_states[i] > 0 ? n_states[i] : 0;
    if (pairs > batk::kMsMaxTable) return fail(BAT_ETOOBIG, "more than %d (arc, state) pairs", batk::kMsMaxTable);
    std::vector<double> w((size_t)pairs + 1, 1.0);
    std::string src;
    double hi = 0.0, lo = 0.0;
    u64 c = 0;
    const bool whole = c_lo == 0 && c_hi == 0;
    int rc = ms_run(n, m, arcs, n_states, capacity, w.data(), s, t, demand, flags, whole, c_lo, c_hi, hi, lo, c, &src);
    if (rc) return rc;
    const uint64_t need = (uint64_t)src.size() + 1;
    const uint64_t have = *len;
    *len = need;
    if (!buf) return BAT_OK;
    if (have < need) return fail(BAT_ETOOBIG, "buffer of %llu bytes, need %llu", (unsigned long long)have,
                                 (unsigned long long)need);
    memcpy(buf, src.c_str(), need);
    return BAT_OK;
}

int bat_autotune(int32_t n, int32_t m, const bat_arc *arcs, const double *p, int32_t s, int32_t t,
                 double *best_ns_per_vector)
{
    t_err.clear();
    int rc = validate(n, m, arcs, p, s, t);
    if (rc) return rc;
    if (!p && m > 0) return fail(BAT_EINVAL, "p is NULL");
    DeviceInfo D;
    rc = current_device(D);
    if (rc) return rc;
    // Each candidate sweeps a sample of its work items spread over the whole
    // counter (an odd-multiplier hash of the item index, so every arc's
    // state varies across the sample), about 2^38 vectors or everything if
    // that is less; candidates are compared by their best time per vector
    // over two timed passes.
    const u64 total = 1ull << m;
    const u32 ubits = m > bat::kWordBits ? (u32)m - bat::kWordBits : 0u;
    // the automatic work-item size (as queue_sweep picks it)
    const int clog_auto = fill_item_log2(1ull << ubits, D.cus, 1);
    struct Cand {
        int clog, check, jit, perm, chain, waves = -1, super_restart = -1, simd_waves = -1, keep_bottom = -1;
    };
    constexpr double kTuneMargin = 0.01;
    auto measure = [&](const Cand &c, double &ns, bool grad = false) -> bool {
        ns = 1e300;
        // the best of at least two timed passes, more for short samples (up
        // to ~40 ms of timed kernel, at most 6 passes), whose times scatter
        // more; a pass whose kernel was compiled or loaded first is not
        // timed (the kernels were compiled ahead, so that is one pass)
        double timed_ms = 0.0;
        int timed = 0;
        for (int rep = 0; rep < 8 && (timed < 2 || (timed < 6 && timed_ms < 40.0)); ++rep) {
            Request tmpl{};
            tmpl.force_chunk_log2 = c.clog;
            tmpl.force_check = c.check;
            tmpl.force_jit = c.jit;
            tmpl.force_perm = c.perm;
            tmpl.force_chain = c.chain;
            tmpl.force_waves = c.waves;
            tmpl.force_super = c.super_restart;
            tmpl.force_simd = c.simd_waves;
            tmpl.force_keep = c.keep_bottom;
            const int cl = c.clog > 0 ? c.clog : std::max(clog_auto, 3);
            const u64 per_item = 1ull << (cl + bat::kWordBits);
            tmpl.sample_items = std::max<u64>(1024, (1ull << 38) / per_item);
            std::vector<double> res;
            u64 cnt = 0;
            bat_launch_info li;
            if (run_sync(n, m, arcs, p, s, t, 0, total, grad, res, cnt, &tmpl) || bat_last_launch(&li)) return false;
            if (li.jit_ms == 0.0) {
                ns = std::min(ns, li.kernel_ms * 1e6 / (double)li.vectors);
                timed_ms += li.kernel_ms;
                ++timed;
            }
        }
        return true;
    };
    double best = 1e300;
    Cand bc{0, 1, 2, kDefaultPerm, 3};
    const char *vb = getenv("BAT_AUTOTUNE_VERBOSE");
    const bool verbose = vb && *vb && *vb != '0';
    auto consider = [&](const Cand &c) {
        double ns;
        const bool ok = measure(c, ns);
        if (verbose)
            fprintf(stderr,
                    "bat_autotune: chunk_log2=%d check=%d jit=%d perm=%d chain=%d waves=%d super=%d simd=%d "
                    "keep=%d -> %s %.6f ns/vector\n",
                    c.clog, c.check, c.jit, c.perm, c.chain, c.waves, c.super_restart, c.simd_waves, c.keep_bottom,
                    ok ? "ok" : "failed", ok ? ns : 0.0);
        // a later candidate must win by a margin: near ties keep the
        // earlier (default-first) choice, so repeated tuning agrees
        if (ok && ns < best * (1.0 - kTuneMargin)) {
            best = ns;
            bc = c;
        }
    };
    // compile the specialised kernels of candidates ahead of their runs, in
    // parallel (their knobs resolved as a launch resolves them)
    const std::string gkey = graph_key(n, m, arcs, s, t);
    auto precompile = [&](const std::vector<std::pair<Cand, bool>> &cands) {
        std::vector<Plan> plans(cands.size());
        std::vector<std::tuple<const Plan *, bool, JitShape>> want;
        for (size_t i = 0; i < cands.size(); ++i) {
            const Cand &c = cands[i].first;
            const bool grad = cands[i].second;
            Request r{};
            r.force_chunk_log2 = c.clog;
            r.force_check = c.check;
            r.force_jit = c.jit;
            r.force_perm = c.perm;
            r.force_chain = c.chain;
            r.force_waves = c.waves;
            r.force_super = c.super_restart;
            r.force_simd = c.simd_waves;
            r.force_keep = c.keep_bottom;
            TuneChoice tc = choose(D, gkey, grad, &r);
            if (tc.jit != 1) continue;
            if (tc.perm < 0 || tc.perm >= kPermKinds) tc.perm = kDefaultPerm;
            make_plan(n, m, arcs, s, t, plans[i], tc.perm);
            want.emplace_back(&plans[i], grad, jit_shape(grad, tc.waves, tc.super_restart, tc.simd_waves, tc.keep_bottom));
        }
        jit_precompile(D, want);
    };
    {
        std::vector<std::pair<Cand, bool>> first;
        for (int i = 0; i < kPermKinds; ++i) first.push_back({{0, 1, 1, i, 3}, false});
        for (int perm : {kDefaultPerm, 0}) first.push_back({{0, 1, 1, perm, 3}, true});
        precompile(first);
    }
    // stage 1: arc-to-bit order x chain length, specialised kernel,
    // automatic work-item size (the two interact); the default order first
    for (int i = 0; i < kPermKinds; ++i) {
        const int perm = (kDefaultPerm + i) % kPermKinds;
        for (int k : {3, 5}) consider({0, 1, 1, perm, k});
    }
    {
        const Cand w1 = bc;
        for (int k : {4, 6})
            if (k != w1.chain) consider({0, 1, 1, w1.perm, k});
    }
    // stage 2: work-item size, convergence-test cadence, generic kernel
    const Cand w = bc;
    for (int d : {-2, 2}) {
        int cl = clog_auto + d;
        if (cl >= 5 && cl <= 14) consider({cl, w.check, w.jit, w.perm, w.chain});
    }
    consider({bc.clog, 2, bc.jit, bc.perm, bc.chain});
    // launch shape of the specialised forward sweep: the register budget
    // (5 wavefronts per SIMD, or the compiler's own), then blocks of 2
    // wavefronts and the super-block store (which takes LDS, so whole
    // 4-wavefront blocks wait for it)
    if (bc.jit != 0) {
        {
            std::vector<std::pair<Cand, bool>> shapes;
            for (int sw : {5, 6, 0}) shapes.push_back({{bc.clog, bc.check, bc.jit, bc.perm, bc.chain, -1, -1, sw}, false});
            shapes.push_back({{bc.clog, bc.check, bc.jit, bc.perm, bc.chain, -1, -1, -1, 2}, false});
            shapes.push_back({{bc.clog, bc.check, bc.jit, bc.perm, bc.chain, 2, 0}, false});
            shapes.push_back({{bc.clog, bc.check, bc.jit, bc.perm, bc.chain, 4, 1}, false});
            shapes.push_back({{bc.clog, bc.check, bc.jit, bc.perm, 3}, true});
            precompile(shapes);
        }
        const Cand w2 = bc;
        // (-1 is the default: 6, or the compiler's budget for big plans)
        for (int sw : {5, 6, 0})
            consider({w2.clog, w2.check, w2.jit, w2.perm, w2.chain, -1, -1, sw});
        const Cand w3 = bc;
        // the kept block bottom in LDS: no spills for it, but fewer blocks fit
        consider({w3.clog, w3.check, w3.jit, w3.perm, w3.chain, -1, -1, w3.simd_waves, 2});
        const Cand w4 = bc;
        consider({w4.clog, w4.check, w4.jit, w4.perm, w4.chain, 2, 0, w4.simd_waves, w4.keep_bottom});
        consider({w4.clog, w4.check, w4.jit, w4.perm, w4.chain, 4, 1, w4.simd_waves, w4.keep_bottom});
    }
    if (total <= (1ull << 32)) consider({bc.clog, 1, 0, 0, 0});
    if (best >= 1e300) return fail(BAT_EDEVICE, "autotune: no candidate ran (%s)", t_err.c_str());
    {
        std::lock_guard<std::mutex> lk(g_tune_mu);
        TuneChoice tc{bc.clog, bc.check, bc.jit, bc.perm, bc.chain};
        tc.waves = bc.waves;
        tc.super_restart = bc.super_restart;
        tc.simd_waves = bc.simd_waves;
        tc.keep_bottom = bc.keep_bottom;
        const std::string gk = graph_key(n, m, arcs, s, t);
        g_tune[std::to_string(D.id) + " fwd " + gk] = tc;
    }
    // the gradient sweep: its own arc order and chain length (it keeps at
    // most 4 chained bits, and its cost is spread differently), starting
    // from the forward's choice; the launch shape is its own and fixed
    {
        Cand gb{bc.clog, bc.check, bc.jit, bc.perm, std::min(bc.chain, 4)};
        double gbest = 1e300;
        auto gconsider = [&](const Cand &c) {
            double ns;
            const bool ok = measure(c, ns, true);
            if (verbose)
                fprintf(stderr, "bat_autotune (gradient): chunk_log2=%d check=%d jit=%d perm=%d chain=%d -> %s %.6f ns/vector\n",
                        c.clog, c.check, c.jit, c.perm, c.chain, ok ? "ok" : "failed", ok ? ns : 0.0);
            if (ok && ns < gbest * (1.0 - kTuneMargin)) {
                gbest = ns;
                gb = c;
            }
        };
        gconsider(gb);
        if (bc.jit != 0) {
            for (int perm : {kDefaultPerm, 0})
                for (int k : {3, 4})
                    if (perm != gb.perm || k != gb.chain) gconsider({bc.clog, bc.check, bc.jit, perm, k});
        }
        std::lock_guard<std::mutex> lk(g_tune_mu);
        TuneChoice tc{gb.clog, gb.check, gb.jit, gb.perm, gb.chain};
        g_tune[std::to_string(D.id) + " grad " + graph_key(n, m, arcs, s, t)] = tc;
    }
    // the time per vector of the sweep that a whole call takes: by sub-cubes,
    // where it does, they have no knobs (the choice above then serves what
    // the plain launch is left with)
    batcube::CubePlan C;
    if (cubes_wanted()) make_cubes(n, m, arcs, s, t, false, C);
    if (cubes_wanted() && cube_fits(C)) {
        best = 1e300;
        for (int rep = 0; rep < 3; ++rep) {
            std::vector<double> res;
            u64 cnt = 0;
            bat_launch_info li;
            rc = cube_sync(C, p, D, false, res, cnt);
            if (!rc) rc = bat_last_launch(&li);
            if (rc) return rc;
            if (rep > 0) best = std::min(best, li.kernel_ms * 1e6 / (double)li.vectors);
        }
        if (verbose) fprintf(stderr, "bat_autotune: sub-cubes -> %.6f ns/vector\n", best);
    }
    if (best_ns_per_vector) *best_ns_per_vector = best;
    t_err.clear();
    return BAT_OK;
}

}  // extern "C"

namespace {

// ------------------------------------------------ batched sub-cube sweeps
// An entry: a graph with probability vectors [n_p][m].
struct CubeJob {
    int graph;  // entries of one graph follow each other
    int32_t n, m, s, t;
    const bat_arc *arcs;
    const double *p;
    int n_p;
    std::vector<char> rel;  // arcs to enumerate
    int M, levels;
    u32 win_lo, win_last;   // (one level) vectors asked for, in arc order
    u64 items;
    u32 units, first_block, n_blocks;
};

// Most enumerated arcs swept with one level: 22 and 23 measured alike (0.67
// and 0.71 ms with 3 vectors, 1.64 and 1.74 ms with 32), 20 and 17 slower.
constexpr int kCubeBatchOneLevel = 22;
constexpr int kCubeBatchP = 32;  // most probability vectors of an entry
// Most work items of a block: the partials of the largest batch then take
// some 20 MiB (64 graphs of 28 to 32 arcs x 32 vectors: 11.3 ms; with at most
// 256 items 11.5 ms and up to 134 MiB), and also with one level forced on
// 1024 entries of 32 arcs a launch has 2^19 blocks of 1024 threads (HIP: fewer
// than 2^32 threads).
constexpr u64 kCubeBatchItems = 4096;
constexpr size_t kCubeBatchJobs = 1024;  // most entries of a sweep (about 12 KiB of staging each)

// Vectors a lane group of the kernel is made for.
int cube_batch_width(int n_p) { return n_p <= 1 ? 1 : n_p <= 4 ? 4 : n_p <= 8 ? 8 : n_p <= 16 ? 16 : 32; }

// All jobs (of at most kCubeMaxBits enumerated arcs, the largest first) in
// one sweep, many of them in two launches so that the device works on the
// largest while the host still plans the others.  sums: [jobs][width]; fits = false
// (nothing to wait for) when a plan needs more than the kernels hold.
// At most kCubeBatchJobs at once, which bounds the buffers.
int cube_batch_run(CubeJob *jobs, size_t n, int width, const DeviceInfo &D, std::vector<bat::double2_t> &sums,
                   std::vector<u64> &counts, bool &fits);
int cube_batch_all(std::vector<CubeJob> &jobs, int width, const DeviceInfo &D, std::vector<bat::double2_t> &sums,
                   std::vector<u64> &counts, bool &fits)
{
    u64 start = 0;
    int32_t blocks = 0, steps = 0;
    for (size_t at = 0; at < jobs.size(); at += kCubeBatchJobs) {
        int rc = cube_batch_run(&jobs[at], std::min(jobs.size() - at, kCubeBatchJobs), width, D, sums, counts, fits);
        if (rc || !fits) return rc;
        // the launch report covers all of them
        u64 *slot = t_state.cube_slot;
        if (at == 0) start = slot[0];
        slot[0] = start;
        t_state.info.n_chunks = blocks += t_state.info.n_chunks;
        t_state.info.relaxations = steps += t_state.info.relaxations;
    }
    return BAT_OK;
}

// Waits for its streams where a sweep is left early, so that nothing queued
// still uses the thread's buffers when its next call does.
struct Drain {
    hipStream_t st = nullptr, side = nullptr;
    bool on = true;
    ~Drain()
    {
        if (!on) return;
        if (side) (void)hipStreamSynchronize(side);
        (void)hipStreamSynchronize(st);
    }
};

int cube_batch_run(CubeJob *jobs, size_t n, int width, const DeviceInfo &D, std::vector<bat::double2_t> &sums,
                   std::vector<u64> &counts, bool &fits)
{
    fits = true;
    hipStream_t st;
    int rc = thread_stream(D.id, st);
    if (rc) return rc;
    const u64 waves = width == 1 ? bat::kCubeWaves : batk::kCubeBatchWaves;
    u64 blocks = 0, items = 0;
    int m_max = 0;
    for (size_t i = 0; i < n; ++i) {
        CubeJob &J = jobs[i];
        const int rb = bat::kCubeGroup * J.levels +
                       std::max(0, std::min(bat::kLaneBits, J.M - bat::kCubeGroup * J.levels));
        J.items = 1ull << std::max(0, J.M - rb);
        items += J.items;
        m_max = std::max(m_max, J.m);
    }
    // items per block: enough to be worth its tables, few enough for an even
    // end (256 graphs x 32 vectors: 1.5 ms with 8 blocks per CU, 1.62 ms with
    // 4, 3.2 ms with 32; one vector, whose blocks are a quarter the size: 0.58
    // ms with 32, 0.72 ms with 8)
    const u64 per_cu = width == 1 ? 32 : 8;
    u64 units = waves;
    while (units < kCubeBatchItems && items / (2 * units) >= per_cu * (u64)D.cus) units *= 2;
    for (size_t i = 0; i < n; ++i) {
        CubeJob &J = jobs[i];
        J.units = (u32)std::min<u64>(J.items, units);
        J.first_block = (u32)blocks;
        J.n_blocks = (u32)((J.items + J.units - 1) / J.units);
        blocks += J.n_blocks;
    }
    // records: the entry, its steps, its probabilities
    const size_t o_step = align_up(sizeof(bat::BatchCube), 64);
    const size_t o_p = o_step + align_up(sizeof(u32) * (bat::kCubeSteps + 4), 64);
    const size_t stride = align_up(o_p + sizeof(double) * (size_t)width * (size_t)m_max, 256);
    const size_t o_ent = align_up(sizeof(u32) * blocks, 256), in_bytes = o_ent + stride * n;
    const size_t o_part = align_up(in_bytes, 256), o_pc = o_part + 16 * (size_t)width * blocks;
    const size_t o_done = o_pc + 8 * blocks, h_sums = in_bytes, h_cnt = h_sums + 16 * (size_t)width * n;
    Scratch *S = nullptr;
    rc = scratch_reserve(D.id, st, o_done + 8, h_cnt + 8 * n, S);
    if (rc) return rc;
    bat::BatchCubes L;
    memset(&L, 0, sizeof L);
    L.entries = S->dev + o_ent;
    L.stride = (u32)stride;
    L.block_entry = (const u32 *)S->dev;
    L.part = (bat::double2_t *)(S->dev + o_part);
    L.pcount = (u64 *)(S->dev + o_pc);
    L.done = (u32 *)(S->dev + o_done);
    L.sums = (bat::double2_t *)(S->host + h_sums);
    L.counts = (u64 *)(S->host + h_cnt);
    u64 *slot = nullptr;
    rc = diag_next(st, slot, L.seq, Report::sync);
    if (rc) return rc;
    L.diag = slot;
    u32 *be = (u32 *)S->host;
    for (size_t i = 0; i < n; ++i)
        for (u32 b = 0; b < jobs[i].n_blocks; ++b) be[jobs[i].first_block + b] = (u32)i;
    batcube::CubePlan C;
    size_t sent = 0, first = 0;
    u64 steps = 0;
    const bool two = n > 64;
    SideStreams *SS = nullptr;
    if (two) {
        rc = side_streams(D.id, SS);
        if (rc) return rc;
    }
    Drain drain{st, SS ? SS->s[0] : nullptr};
    size_t chunk = two ? n / 8 : n;
    for (size_t i = 0; i < n; ++i) {
        CubeJob &J = jobs[i];
        char *rec = S->host + o_ent + stride * i;
        if (i == 0 || J.graph != jobs[i - 1].graph)
            batcube::make_cube_plan(J.n, J.m, J.arcs, J.rel, J.s, J.t, false, J.levels, C);
        bat::BatchCube &E = *(bat::BatchCube *)rec;
        memset(&E, 0, sizeof E);
        E.m = (u32)J.m;
        E.M = (u32)C.M;
        E.levels = (u32)C.levels;
        E.lane_bits = (u32)C.lane_bits;
        E.n_p = (u32)J.n_p;
        E.split = 1;
        E.units = J.units;
        E.first_block = J.first_block;
        E.n_blocks = J.n_blocks;
        E.win_lo = J.win_lo;
        E.win_last = J.win_last;
        E.n_items = J.items;
        E.item_mul = 0x9E3779B97F4A7C15ull;
        E.item_mask = J.items - 1;
        E.p = (const double *)(S->dev + o_ent + stride * i + o_p);
        E.step = (const u32 *)(S->dev + o_ent + stride * i + o_step);
        for (int c = 0; c < C.M; ++c) E.arc_of_bit[c] = (unsigned char)C.arc_of_bit[c];
        bool ok = C.slots <= bat::kCubeSlots && C.levels == J.levels;
        bat::CubeProg prog[bat::kCubeProgs];
        ok = ok && cube_pack(C, prog, (u32 *)(rec + o_step));
        if (!ok) {
            fits = false;
            return BAT_OK;
        }
        memcpy(E.prog, prog, sizeof E.prog);
        if (J.m > 0) memcpy(rec + o_p, J.p, sizeof(double) * (size_t)J.n_p * (size_t)J.m);
        steps += C.M;
        if (i + 1 == n || i + 1 - first >= chunk) {
            const size_t to = o_ent + stride * (i + 1);
            // the later launch runs beside the first one, whose last blocks
            // leave CUs idle; it reads the table of blocks that went up with
            // the first copy, so it waits for that
            const hipStream_t ls = first ? SS->s[0] : st;
            if (first) HIPCHK(hipStreamWaitEvent(ls, SS->fork, 0));
            HIPCHK(hipMemcpyAsync(S->dev + sent, S->host + sent, to - sent, hipMemcpyHostToDevice, ls));
            if (two && !first) HIPCHK(hipEventRecord(SS->fork, st));
            sent = to;
            L.block0 = jobs[first].first_block;
            HIPCHK(batk::cube_batch(ls, (unsigned)(J.first_block + J.n_blocks - L.block0), width, L));
            first = i + 1;
            chunk = n;
        }
    }
    if (SS) {
        HIPCHK(hipEventRecord(SS->join[0], SS->s[0]));
        HIPCHK(hipStreamWaitEvent(st, SS->join[0], 0));
    }
    HIPCHK(batk::cube_batch_finish(st, (unsigned)n, width, L));
    bat::CubeParams K;
    K.diag = L.diag;
    K.seq = L.seq;
    rc = cube_wait(K, st);
    if (rc) return rc;
    drain.on = false;
    sums.insert(sums.end(), L.sums, L.sums + n * (size_t)width);
    counts.insert(counts.end(), L.counts, L.counts + n);
    bat_launch_info &I = t_state.info;
    memset(&I, 0, sizeof I);
    I.n_chunks = (int32_t)std::min<u64>(blocks, 0x7fffffff);
    I.relaxations = (int32_t)std::min<u64>(steps, 0x7fffffff);
    I.perm = kPermInfluence;
    I.check_every = 1;
    I.item_order = 1;
    I.block_waves = (int32_t)waves;
    I.kernel_id = aot_kernel_id("k_cube_batch", width, false);
    t_state.have_launch = true;
    t_state.cube_seq = L.seq;
    t_state.cube_slot = slot;
    t_state.cube_dev = D.id;
    t_state.cube_khz = D.clock_khz;
    return BAT_OK;
}

// ------------------------------------------------- ranges of the counter
// A range of the paper's counter is a few aligned cubes: blocks of vectors
// that share the leading arcs' states.  With those arcs joined (up) or left
// out (down), a cube is a whole sweep of a smaller graph, whose arcs may take
// the counter bits in any order.  The ends of the range, up to 2^20 vectors,
// stay in the counter's order: a one-level sweep of the block that holds the
// end, of which only the words inside the range count.  All of them run in
// one batched launch (2^30 vectors of 36 arcs: 74 us against 2.85 ms with the
// plain sweep; a hundredth of 2^36 from an odd index 0.10 against 2.5 ms;
// 4000 of 2^20 vectors 36 against 99 us; 33 arcs whole 0.37 against 0.94 ms).
constexpr int kRangeEnd = 20;       // log2 of an end's block
constexpr size_t kRangeCubes = 256;  // most cubes

// The cube of `bits` low counter bits under the higher bits `high`, or its
// vectors first to last; scale: the probability of `high`.
void range_job(int32_t n, int32_t m, const bat_arc *arcs, const double *p, int32_t s, int32_t t, bool forward,
               int bits, u64 high, bool whole, u64 first, u64 last, std::vector<CubeJob> &jobs,
               std::vector<std::vector<bat_arc>> &job_arcs, std::vector<std::vector<double>> &job_p,
               std::vector<double> &scale)
{
    std::vector<int> root(n);
    for (int x = 0; x < n; ++x) root[x] = x;
    auto find = [&](int x) {
        while (root[x] != x) x = root[x] = root[root[x]];
        return x;
    };
    double q = 1.0;
    for (int b = bits; b < m; ++b) {
        const int a = forward ? b : m - 1 - b;
        const bool up = (high >> (b - bits)) & 1u;
        q *= up ? p[a] : 1.0 - p[a];
        if (up) root[find(arcs[a].u)] = find(arcs[a].v);
    }
    std::vector<int> id(n, -1);
    int nn = 0;
    auto node = [&](int x) {
        x = find(x);
        if (id[x] < 0) id[x] = nn++;
        return id[x];
    };
    CubeJob J;
    J.s = node(s);
    J.t = node(t);
    std::vector<bat_arc> sub(bits);
    std::vector<double> sp(bits);
    for (int b = 0; b < bits; ++b) {  // job arc i at counter bit bits - 1 - i
        const int a = forward ? b : m - 1 - b;
        sub[bits - 1 - b] = {node(arcs[a].u), node(arcs[a].v)};
        sp[bits - 1 - b] = p[a];
    }
    J.graph = (int)jobs.size();
    J.n = nn;
    J.m = bits;
    J.n_p = 1;
    J.win_lo = 0;
    J.win_last = ~0u;
    if (whole) {
        if (J.s != J.t) J.rel = cube_arcs(J.n, J.m, sub.data(), J.s, J.t, false);
        else J.rel.assign(bits, 0);  // always connected
        J.rel.resize(bits);
        J.M = 0;
        for (char x : J.rel) J.M += x ? 1 : 0;
        J.levels = J.M <= 23 ? 1 : 2;
    } else {
        J.rel.assign(bits, 1);
        J.M = bits;
        J.levels = 1;
        J.win_lo = (u32)first;
        J.win_last = (u32)last;
    }
    job_arcs.push_back(std::move(sub));
    job_p.push_back(std::move(sp));
    J.arcs = job_arcs.back().data();
    J.p = job_p.back().data();
    jobs.push_back(std::move(J));
    scale.push_back(q);
}

int range_cubes(int32_t n, int32_t m, const bat_arc *arcs, const double *p, int32_t s, int32_t t, const DeviceInfo &D,
                bool forward, u64 c_lo, u64 c_hi, double *R, u64 &count, bool &fits)
{
    fits = false;
    std::vector<CubeJob> jobs;
    std::vector<std::vector<bat_arc>> job_arcs;
    std::vector<std::vector<double>> job_p;
    std::vector<double> scale;
    R[0] = R[1] = 0.0;
    count = 0;
    const int g = std::min<int>(m, kRangeEnd);
    const u64 block = 1ull << g;
    auto add = [&](int bits, u64 high, bool whole, u64 first, u64 last) {
        range_job(n, m, arcs, p, s, t, forward, bits, high, whole, first, last, jobs, job_arcs, job_p, scale);
    };
    u64 a = c_lo >> g, b = c_hi >> g;
    size_t cubes = 0;
    if (c_lo % block != 0 || a == b) {  // the first block, not from its start or not to its end
        const u64 end = std::min(c_hi, (a + 1) << g);
        add(g, a, false, c_lo - (a << g), end - 1 - (a << g));
        ++a;
    }
    while (a < b) {
        int k = 0;
        while (g + k < batk::kCubeMaxBits && g + k < m && a % (2ull << k) == 0 && b - a >= 2ull << k) ++k;
        if (++cubes > kRangeCubes) return BAT_OK;
        add(g + k, a >> k, true, 0, 0);
        a += 1ull << k;
    }
    if (a == b && c_hi % block != 0) add(g, b, false, 0, c_hi - 1 - (b << g));
    // the largest first
    std::vector<size_t> order(jobs.size());
    for (size_t i = 0; i < order.size(); ++i) order[i] = i;
    std::stable_sort(order.begin(), order.end(), [&](size_t i, size_t j) { return jobs[i].M > jobs[j].M; });
    std::vector<CubeJob> sorted;
    for (size_t i : order) sorted.push_back(std::move(jobs[i]));
    std::vector<bat::double2_t> sums;
    std::vector<u64> counts;
    int rc = cube_batch_all(sorted, 1, D, sums, counts, fits);
    if (rc || !fits) return rc;
    for (size_t i = 0; i < sorted.size(); ++i) {
        const double q = scale[order[i]], x = q * sums[i].x;
        dd_acc(R, x, std::fma(q, sums[i].x, -x) + q * sums[i].y);
        count += counts[i];
    }
    t_state.info.vectors = c_hi - c_lo;
    return BAT_OK;
}

// A batch in that form; fits = false where a graph is too large for it.
int cube_batched(int32_t n_graphs, const int32_t *n_nodes, const int32_t *arc_offsets, const bat_arc *arcs,
                 const int32_t *s, const int32_t *t, int32_t n_pvec, const double *p, const DeviceInfo &D, double *R_out,
                 uint64_t *counts_out, bool &fits)
{
    fits = false;
    const int groups = (n_pvec + kCubeBatchP - 1) / kCubeBatchP, per = (n_pvec + groups - 1) / groups;
    const int width = cube_batch_width(per);
    std::vector<std::vector<char>> rel(n_graphs);
    std::vector<int> M(n_graphs, 0), order(n_graphs);
    u64 vectors = 0;
    for (int32_t g = 0; g < n_graphs; ++g) {
        const int32_t m = arc_offsets[g + 1] - arc_offsets[g];
        rel[g] = cube_arcs(n_nodes[g], m, arcs + arc_offsets[g], s[g], t[g], false);
        rel[g].resize(m);
        for (char x : rel[g]) M[g] += x ? 1 : 0;
        if (M[g] > batk::kCubeMaxBits) return BAT_OK;
        order[g] = g;
        vectors += 1ull << m;
    }
    std::stable_sort(order.begin(), order.end(), [&](int a, int b) { return M[a] > M[b]; });
    std::vector<CubeJob> jobs;
    std::vector<std::pair<int, int>> of;  // graph, first vector
    for (int g : order)
        for (int b = 0; b < n_pvec; b += per) {
            CubeJob J;
            J.graph = g;
            J.n = n_nodes[g];
            J.m = arc_offsets[g + 1] - arc_offsets[g];
            J.s = s[g];
            J.t = t[g];
            J.arcs = arcs + arc_offsets[g];
            J.p = p + (int64_t)n_pvec * arc_offsets[g] + (int64_t)b * J.m;
            J.n_p = std::min(per, n_pvec - b);
            J.rel = rel[g];
            J.M = M[g];
            J.levels = M[g] <= kCubeBatchOneLevel ? 1 : 2;
            if (opts().cube_levels.load() > 0)
                J.levels = std::max(1, std::min({(int)opts().cube_levels.load(), 2, J.M / bat::kCubeGroup}));
            J.win_lo = 0;
            J.win_last = ~0u;
            jobs.push_back(std::move(J));
            of.push_back({g, b});
        }
    std::vector<bat::double2_t> sums;
    std::vector<u64> counts;
    int rc = cube_batch_all(jobs, width, D, sums, counts, fits);
    if (rc || !fits) return rc;
    for (size_t i = 0; i < jobs.size(); ++i) {
        for (int q = 0; q < jobs[i].n_p; ++q)
            R_out[(size_t)of[i].first * n_pvec + of[i].second + q] = sums[i * width + q].x + sums[i * width + q].y;
        counts_out[of[i].first] = counts[i];
    }
    t_state.info.vectors = vectors;
    return BAT_OK;
}

}  // namespace

// Tuned knobs of the batched launch: chained iteration bits and the
// per-wavefront segment size, cached under the batch's structure.
struct BatchTune {
    int chain = -1;  // -1: option BAT_CHAIN_LOG2 (-1 = 3)
    int seg = -1;    // -1: batk::kBatchSegLog
    int jit_arcs = -1;  // graphs with at least this many arcs run graph-specialised (0: none; -1: option)
    int streams = -1;   // side streams of the specialised kernels (0: the thread's stream; -1: option, else 3)
    int cubes = 0;      // (forced only) sub-cube sweeps
};
std::mutex g_btune_mu;
std::map<std::string, BatchTune> g_btune;

// The batch's structure (graphs, terminals, p-vector count) as a key.
std::string batch_key(int device, int32_t n_graphs, const int32_t *n_nodes, const int32_t *arc_offsets,
                      const bat_arc *arcs, const int32_t *s, const int32_t *t, int32_t n_pvec)
{
    uint64_t h = 1469598103934665603ull;  // FNV-1a over the structure
    auto mix = [&](const void *d, size_t n) {
        const unsigned char *c = (const unsigned char *)d;
        for (size_t i = 0; i < n; ++i) h = (h ^ c[i]) * 1099511628211ull;
    };
    mix(n_nodes, sizeof(int32_t) * n_graphs);
    mix(arc_offsets, sizeof(int32_t) * (n_graphs + 1));
    mix(arcs, sizeof(bat_arc) * arc_offsets[n_graphs]);
    mix(s, sizeof(int32_t) * n_graphs);
    mix(t, sizeof(int32_t) * n_graphs);
    return std::to_string(device) + " batch " + std::to_string(n_graphs) + " " + std::to_string(n_pvec) + " " +
           std::to_string(h);
}

bool batch_cubes_wanted()
{
    const Options &o = opts();
    return cubes_wanted() && (o.cubes.load() == 1 || (o.batch_jit_arcs.load() < 0 && o.batch_streams.load() < 0 &&
                                                      o.batch_acc.load() == 1));
}

int batched_impl(int32_t n_graphs, const int32_t *n_nodes, const int32_t *arc_offsets, const bat_arc *arcs,
                 const int32_t *s, const int32_t *t, int32_t n_pvec, const double *p, double *R_out,
                 uint64_t *counts_out, const BatchTune *force)
{
    t_err.clear();
    if (n_graphs <= 0) return fail(BAT_EINVAL, "n_graphs must be >= 1");
    if (!n_nodes || !arc_offsets || !s || !t || !R_out || !counts_out) return fail(BAT_EINVAL, "NULL argument");
    if (n_pvec < 1 || n_pvec > BAT_MAX_PVEC) return fail(BAT_EINVAL, "n_pvec %d outside [1, %d]", n_pvec, BAT_MAX_PVEC);
    if (arc_offsets[0] != 0) return fail(BAT_EINVAL, "arc_offsets[0] must be 0");
    for (int32_t g = 0; g < n_graphs; ++g) {
        int32_t m = arc_offsets[g + 1] - arc_offsets[g];
        if (m < 0) return fail(BAT_EINVAL, "arc_offsets not ascending at graph %d", g);
        int rc = validate(n_nodes[g], m, m ? arcs + arc_offsets[g] : nullptr, nullptr, s[g], t[g]);
        if (rc) return fail(rc, "graph %d: %s", g, t_err.c_str());
        if (m > 0 && !p) return fail(BAT_EINVAL, "p is NULL");
        const double *pg = p + (int64_t)n_pvec * arc_offsets[g];
        for (int64_t i = 0; i < (int64_t)n_pvec * m; ++i)
            if (!(pg[i] >= 0.0 && pg[i] <= 1.0))
                return fail(BAT_EINVAL, "graph %d: p[%lld] = %g is not a probability", g, (long long)i, pg[i]);
    }
    DeviceInfo D;
    int rc = current_device(D);
    if (rc) return rc;
    // sub-cube sweeps unless a knob of the plain launch has been set; they
    // have none to tune (256 graphs of 16 to 28 arcs x 32 p-vectors: 2.9 ms
    // a call against 11.6 ms with the tuned plain launch, 16 of 8 to 20 arcs
    // x 3: 0.10 ms against 0.9 ms)
    if (force ? force->cubes != 0 : batch_cubes_wanted()) {
        bool fits = false;
        rc = cube_batched(n_graphs, n_nodes, arc_offsets, arcs, s, t, n_pvec, p, D, R_out, counts_out, fits);
        if (rc || fits) return rc;
        if (force) return BAT_PENDING;
    }
    hipStream_t st;
    rc = thread_stream(D.id, st);
    if (rc) return rc;

    // plans, entries (graph x group of <= 32 p-vectors), longest first
    std::vector<Plan> plans(n_graphs);
    std::vector<u32> progs;
    std::vector<u32> prog_off(n_graphs);
    int nmax = 2;
    for (int32_t g = 0; g < n_graphs; ++g) {
        int32_t m = arc_offsets[g + 1] - arc_offsets[g];
        make_plan(n_nodes[g], m, arcs + arc_offsets[g], s[g], t[g], plans[g]);
        prog_off[g] = (u32)progs.size();
        progs.insert(progs.end(), plans[g].prog.begin(), plans[g].prog.end());
        nmax = std::max(nmax, plans[g].N);
    }
    // knobs: forced (autotuner), else the tuned choice, else the options
    BatchTune bt;
    if (force) {
        bt = *force;
    } else if (opts().autotune.load()) {
        std::lock_guard<std::mutex> lk(g_btune_mu);
        auto it = g_btune.find(batch_key(D.id, n_graphs, n_nodes, arc_offsets, arcs, s, t, n_pvec));
        if (it != g_btune.end()) bt = it->second;
    }
    if (!force && opts().chain_log2.load() >= 0) bt.chain = (int)opts().chain_log2.load();
    if (!force && opts().batch_jit_arcs.load() >= 0) bt.jit_arcs = (int)opts().batch_jit_arcs.load();
    const int jit_arcs = bt.jit_arcs > 0 ? bt.jit_arcs : 0;
    // chained iteration bits (-1 = 3, 0 = none, 3..6)
    const int bchain = bt.chain < 0 ? 3 : (bt.chain >= 3 ? std::min(bt.chain, 6) : 0);
    const u32 bseg = bt.seg > 0 ? (u32)std::min(bt.seg, batk::kBatchSegLog) : (u32)batk::kBatchSegLog;
    // graphs of at least jit_arcs arcs (and a full work item) get their own
    // graph-specialised kernel, for at most kBatchSpecP p-vectors per entry;
    // the rest share the generic persistent one
    auto specialised = [&](const batk::BatchEntry &e) {
        return jit_arcs > 0 && (int)e.m >= jit_arcs && e.ubits >= e.f && e.f >= 3;
    };
    std::vector<batk::BatchEntry> ents;
    for (int32_t g = 0; g < n_graphs; ++g) {
        const Plan &P = plans[g];
        u32 m = (u32)P.m;
        u32 ubits = m > (u32)bat::kWordBits ? m - bat::kWordBits : 0u;
        batk::BatchEntry probe;
        memset(&probe, 0, sizeof probe);
        probe.m = m;
        probe.ubits = ubits;
        probe.f = std::min<u32>(ubits, bseg);
        const int32_t per = specialised(probe) ? kBatchSpecP : batk::kBatchMaxP;
        for (int32_t b = 0; b < n_pvec; b += per) {
            batk::BatchEntry e;
            memset(&e, 0, sizeof e);
            e.m = m;
            e.ubits = ubits;
            e.f = std::min<u32>(ubits, bseg);
            e.P = (u32)std::min<int32_t>(per, n_pvec - b);
            e.n_nodes = (u32)P.N;
            e.s = (u32)P.S;
            e.t = (u32)P.T;
            e.n_relax = (u32)P.code.size();
            e.prog_off = prog_off[g];
            e.n_groups = (u32)((P.prog.size() - 8) / 16);
            // warm-started chains over k <= f iteration bits
            e.chain = (bchain >= 3 && e.f >= (u32)bchain) ? (u32)bchain : (e.f >= 3 && bchain >= 3 ? e.f : 0u);
            chain_codes(P, e.ck_code);
            e.graph = (u32)g;
            e.pv_base = (u32)b;
            ents.push_back(e);
        }
    }
    // generic entries first (one queue), then the specialised ones; each
    // part longest first
    std::stable_sort(ents.begin(), ents.end(), [&](const batk::BatchEntry &a, const batk::BatchEntry &b) {
        const bool sa = specialised(a), sb = specialised(b);
        return sa != sb ? sb : a.m > b.m;
    });
    size_t n_gen = 0;
    while (n_gen < ents.size() && !specialised(ents[n_gen])) ++n_gen;
    nmax = 2;
    for (size_t i = 0; i < n_gen; ++i) nmax = std::max(nmax, (int)ents[i].n_nodes);
    // wavefronts per block of the generic kernel: an item is that many
    // segments
    const bool gen_t = opts().batch_acc.load() == 1;
    const int gen_waves = gen_t ? batk::batch_waves_t(nmax) : batk::batch_waves(nmax);
    u64 n_items = 0, n_gen_items = 0, tab = 0;
    std::vector<u64> item_start;
    std::vector<u32> pair_entry, pair_pv;
    std::vector<u64> entry_p_off;
    u64 vectors = 0;
    for (size_t i = 0; i < ents.size(); ++i) {
        batk::BatchEntry &e = ents[i];
        u64 iters = 1ull << e.ubits;
        // a generic item is a block's worth of segments, a specialised one a
        // single segment (one wavefront)
        u64 per_item = i < n_gen ? (u64)gen_waves << e.f : 1ull << e.f;
        e.item_begin = n_items;
        e.n_items = (iters + per_item - 1) / per_item;
        e.tab_off = tab;
        item_start.push_back(n_items);
        n_items += e.n_items;
        if (i < n_gen) n_gen_items = n_items;
        tab += (u64)e.P * bat::kTablesFwd;
        for (u32 q = 0; q < e.P; ++q) {
            pair_entry.push_back((u32)i);
            pair_pv.push_back(q);
        }
        entry_p_off.push_back((u64)n_pvec * (u64)arc_offsets[e.graph]);
        vectors += 1ull << e.m;
    }
    item_start.push_back(n_items);
    const int64_t p_total = (int64_t)n_pvec * arc_offsets[n_graphs];

    // the specialised kernels: one per (graph, p-vectors in the entry),
    // compiled side by side before the first is loaded
    std::vector<hipFunction_t> spec_fn(ents.size(), nullptr);
    uint64_t spec_id = 0;
    double spec_jit_ms = 0.0;
    if (n_gen < ents.size()) {
        const JitShape sh = jit_shape(false, 4, 0, 0, 1);
        auto t0 = std::chrono::steady_clock::now();
        std::vector<std::string> srcs(ents.size()), keys(ents.size()), todo;
        for (size_t i = n_gen; i < ents.size(); ++i) {
            keys[i] = std::to_string(D.id) + " batch" + std::to_string(ents[i].P) +
                      (batch_transposed((int)ents[i].P) ? "t " : " ") + plans[ents[i].graph].structure;
            srcs[i] = jit_source(plans[ents[i].graph], false, sh, (int)ents[i].P);
            std::lock_guard<std::mutex> lk(g_jit_mu);
            if (!g_jit.count(keys[i])) todo.push_back(srcs[i]);
        }
        if (!todo.empty()) jit_precompile_sources(D, todo);
        for (size_t i = n_gen; i < ents.size(); ++i) {
            const std::string &key = keys[i];
            double ms = 0.0;
            uint64_t id = 0;
            rc = jit_load(D, key, srcs[i], "bat_batch_jit", spec_fn[i], ms, id);
            if (rc) return rc;
            spec_id = spec_id * 0x100000001b3ull + id;
        }
        spec_jit_ms = std::chrono::duration<double, std::milli>(std::chrono::steady_clock::now() - t0).count();
    }

    // device buffers (one stream-ordered allocation)
    size_t off = 0;
    auto take = [&](size_t bytes) { size_t o = off; off = align_up(off + bytes, 256); return o; };
    const size_t o_ent = take(sizeof(batk::BatchEntry) * ents.size());
    const size_t o_ist = take(sizeof(u64) * item_start.size());
    const size_t o_prog = take(sizeof(u32) * (progs.size() + 1));
    const size_t o_pe = take(sizeof(u32) * pair_entry.size());
    const size_t o_pp = take(sizeof(u32) * pair_pv.size());
    const size_t o_epo = take(sizeof(u64) * entry_p_off.size());
    const size_t o_p = take(sizeof(double) * (size_t)(p_total + 1));
    const size_t o_tab = take(sizeof(double) * tab);
    const size_t o_part = take(sizeof(double) * 2 * batk::kBatchMaxP * n_items);
    const size_t o_pc = take(sizeof(u64) * n_items);
    const size_t o_ctr = take(sizeof(unsigned long long));
    const size_t o_R = take(sizeof(double) * (size_t)n_graphs * n_pvec);
    const size_t o_cnt = take(sizeof(u64) * (size_t)n_graphs);
    char *ws = nullptr;
    // side streams for the specialised kernels (before anything is queued)
    const size_t n_spec = ents.size() - n_gen;
    SideStreams *SS = nullptr;
    // how many side streams: forced by the option, else tuned, else 3 (with
    // the thread's stream, the 4 hardware queues HIP gives a process by
    // default; which queue a stream shares depends on the streams the
    // process made before it, so the autotuner measures 1 to 3)
    int want_side = bt.streams >= 0 ? bt.streams : 3;
    if (opts().batch_streams.load() >= 0 && (!force || bt.streams < 0)) want_side = (int)opts().batch_streams.load();
    const int n_side = (int)std::min<int64_t>(std::min<int64_t>(want_side, kSideStreams), (int64_t)n_spec);
    if (n_side > 0) {
        rc = side_streams(D.id, SS);
        if (rc) return rc;
    }
    // lanes for the specialised kernels: the thread's stream (lane 0, which
    // runs its share first and the generic persistent kernel after it) and
    // the side streams; each kernel goes to the least-loaded lane, largest
    // first, lane 0 starting with the generic kernel's work (weighted by
    // its slower closure)
    double lane_load[kSideStreams + 1] = {};
    for (size_t i = 0; i < n_gen; ++i) lane_load[0] += 1.5 * (double)ents[i].P * (double)(1ull << ents[i].m);
    HIPCHK(hipMallocAsync((void **)&ws, off, st));
    auto h2d = [&](size_t o, const void *src, size_t bytes) -> hipError_t {
        return bytes ? hipMemcpyAsync(ws + o, src, bytes, hipMemcpyHostToDevice, st) : hipSuccess;
    };
    HIPCHK(h2d(o_ent, ents.data(), sizeof(batk::BatchEntry) * ents.size()));
    HIPCHK(h2d(o_ist, item_start.data(), sizeof(u64) * item_start.size()));
    HIPCHK(h2d(o_prog, progs.data(), sizeof(u32) * progs.size()));
    HIPCHK(h2d(o_pe, pair_entry.data(), sizeof(u32) * pair_entry.size()));
    HIPCHK(h2d(o_pp, pair_pv.data(), sizeof(u32) * pair_pv.size()));
    HIPCHK(h2d(o_epo, entry_p_off.data(), sizeof(u64) * entry_p_off.size()));
    HIPCHK(h2d(o_p, p, sizeof(double) * (size_t)p_total));
    HIPCHK(hipMemsetAsync(ws + o_ctr, 0, sizeof(unsigned long long), st));

    const batk::BatchEntry *d_ent = (const batk::BatchEntry *)(ws + o_ent);
    rc = events_ready();
    if (rc) return rc;
    HIPCHK(hipEventRecord(t_state.ev[0], st));
    HIPCHK(batk::batched_tables(st, d_ent, (const u32 *)(ws + o_pe), (const u32 *)(ws + o_pp),
                                (const u64 *)(ws + o_epo), (const double *)(ws + o_p), (unsigned)pair_entry.size(),
                                (double *)(ws + o_tab)));
    HIPCHK(hipEventRecord(t_state.ev[1], st));
    batk::BatchParams BP;
    memset(&BP, 0, sizeof BP);
    BP.entries = d_ent;
    BP.item_start = (const u64 *)(ws + o_ist);
    BP.n_entries = (u32)n_gen;
    BP.check_every = opts().check_every.load() >= 2 ? 2u : 1u;
    BP.n_items = n_gen_items;
    BP.prog = (const u32 *)(ws + o_prog);
    BP.tables = (const double *)(ws + o_tab);
    BP.part = (double *)(ws + o_part);
    BP.pcount = (u64 *)(ws + o_pc);
    BP.ctr = (unsigned long long *)(ws + o_ctr);
    // the specialised kernels run on side streams forked from the thread's
    // stream after the tables, so that small ones overlap; joined before
    // the reduction
    if (n_side > 0) {
        HIPCHK(hipEventRecord(SS->fork, st));
        for (int k = 0; k < n_side; ++k) HIPCHK(hipStreamWaitEvent(SS->s[k], SS->fork, 0));
    }
    const int window = opts().window_test.load() != 0 ? 1 : 0;
    for (size_t i = n_gen; i < ents.size(); ++i) {
        const batk::BatchEntry &e = ents[i];
        bat::KParams K;
        memset(&K, 0, sizeof K);
        const u64 iters = 1ull << e.ubits;
        K.c_lo = 0;
        K.c_hi = 1ull << e.m;
        K.g_first = 0;
        K.g_last = iters - 1;
        K.g_base = 0;
        K.g_end = iters - 1;
        K.chunk_iters = 1ull << e.f;  // one segment per work item
        K.n_chunks = e.n_items;
        K.chunk_mul = 1;
        K.chunk_mask = ~0ull;
        K.m = e.m;
        K.ubits = e.ubits;
        K.seg_log = e.f;
        K.check_every = BP.check_every;
        K.chain = e.chain;
        K.ncol = 1;
        K.window_test = (e.chain && window) ? 1u : 0u;
        K.n_nodes = e.n_nodes;
        K.s = e.s;
        K.t = e.t;
        K.tables = (const double *)(ws + o_tab) + e.tab_off;
        K.part = (double *)(ws + o_part) + e.item_begin * batk::kBatchMaxP * 2;
        K.pcount = (u64 *)(ws + o_pc) + e.item_begin;
        const u64 wpb = (u64)batch_waves((int)e.P);
        const u64 blocks = std::min<u64>((u64)D.cus, (e.n_items + wpb - 1) / wpb);
        void *args[] = {&K};
        int k_min = 0;
        for (int k = 1; k <= n_side; ++k)
            if (lane_load[k] < lane_load[k_min]) k_min = k;
        lane_load[k_min] += (double)e.P * (double)(1ull << e.m);
        hipStream_t ls = k_min > 0 ? SS->s[k_min - 1] : st;
        HIPCHK(hipModuleLaunchKernel(spec_fn[i], (unsigned)blocks, 1, 1, (unsigned)(bat::kWave * wpb), 1, 1, 0, ls, args,
                                     nullptr));
    }
    // the generic queue after the specialised kernels (the largest graphs)
    // are queued, behind lane 0's: its persistent blocks then fill the CUs
    // the others leave
    if (n_gen_items > 0) {
        unsigned blocks = (unsigned)std::max<u64>(1, std::min<u64>((u64)D.cus, n_gen_items));
        HIPCHK(batk::batched_sweep(st, blocks, nmax, gen_t, BP));
    }
    for (int k = 0; k < n_side; ++k) {
        HIPCHK(hipEventRecord(SS->join[k], SS->s[k]));
        HIPCHK(hipStreamWaitEvent(st, SS->join[k], 0));
    }
    HIPCHK(hipEventRecord(t_state.ev[2], st));
    HIPCHK(batk::batched_reduce(st, d_ent, (unsigned)ents.size(), (const double *)(ws + o_part),
                                (const u64 *)(ws + o_pc), (u32)n_pvec, (double *)(ws + o_R), (u64 *)(ws + o_cnt)));
    HIPCHK(hipEventRecord(t_state.ev[3], st));
    HIPCHK(hipMemcpyAsync(R_out, ws + o_R, sizeof(double) * (size_t)n_graphs * n_pvec, hipMemcpyDeviceToHost, st));
    HIPCHK(hipMemcpyAsync(counts_out, ws + o_cnt, sizeof(u64) * (size_t)n_graphs, hipMemcpyDeviceToHost, st));
    HIPCHK(hipFreeAsync(ws, st));
    HIPCHK(hipStreamSynchronize(st));
    bat_launch_info &I = t_state.info;
    memset(&I, 0, sizeof I);
    t_state.cube_seq = 0;
    I.vectors = vectors;
    I.specialised = n_gen < ents.size() ? 1 : 0;
    I.jit_ms = spec_jit_ms;
    I.chunk_log2 = (int32_t)bseg;
    I.n_chunks = (int32_t)std::min<u64>(n_items, 0x7fffffff);
    {
        size_t nrel = 0;
        for (const Plan &pl : plans) nrel += pl.code.size();
        I.relaxations = (int32_t)nrel;
    }
    I.kernel_id = aot_kernel_id(gen_t ? "k_batched_dyn_t" : "k_batched_dyn", (int)nmax, false) ^
                  spec_id;
    I.perm = -1;
    I.chain_log2 = (int32_t)bchain;
    I.check_every = 1;
    I.item_order = 0;
    I.block_waves = (int32_t)gen_waves;
    I.super_restart = 0;
    I.window_test = 0;
    t_state.have_launch = true;
    return BAT_OK;
}

extern "C" int bat_reliability_batched(int32_t n_graphs, const int32_t *n_nodes, const int32_t *arc_offsets,
                                       const bat_arc *arcs, const int32_t *s, const int32_t *t, int32_t n_pvec,
                                       const double *p, double *R_out, uint64_t *counts_out)
{
    return batched_impl(n_graphs, n_nodes, arc_offsets, arcs, s, t, n_pvec, p, R_out, counts_out, nullptr);
}

extern "C" int bat_autotune_batched(int32_t n_graphs, const int32_t *n_nodes, const int32_t *arc_offsets,
                                    const bat_arc *arcs, const int32_t *s, const int32_t *t, int32_t n_pvec,
                                    const double *p, double *best_kernel_ms)
{
    t_err.clear();
    if (n_graphs <= 0 || !n_nodes || !arc_offsets || !arcs || !s || !t)
        return fail(BAT_EINVAL, "invalid batch description");
    if (n_pvec < 1 || n_pvec > BAT_MAX_PVEC) return fail(BAT_EINVAL, "n_pvec %d outside [1, %d]", n_pvec, BAT_MAX_PVEC);
    DeviceInfo D;
    int rc = current_device(D);
    if (rc) return rc;
    std::vector<double> R((size_t)n_graphs * n_pvec);
    std::vector<uint64_t> cnt((size_t)n_graphs);
    const char *vb = getenv("BAT_AUTOTUNE_VERBOSE");
    const bool verbose = vb && *vb && *vb != '0';
    // the whole batch, each candidate once untimed and then the best of two
    // (a batch is one launch: sampling it would change its load balance)
    double best = 1e300;
    BatchTune bb;
    // sub-cube sweeps have no knobs, so where they are taken the plain
    // launch, slower on every batch measured, is not timed
    if (batch_cubes_wanted()) {
        BatchTune c;
        c.cubes = 1;
        for (int rep = 0; rep < 3; ++rep) {
            rc = batched_impl(n_graphs, n_nodes, arc_offsets, arcs, s, t, n_pvec, p, R.data(), cnt.data(), &c);
            if (rc == BAT_PENDING) break;  // a graph too large for them
            if (rc) return rc;
            bat_launch_info li;
            rc = bat_last_launch(&li);
            if (rc) return rc;
            if (rep > 0) best = std::min(best, li.kernel_ms);
        }
        if (verbose) fprintf(stderr, "bat_autotune_batched: sub-cubes -> %.3f ms\n", best);
        if (rc == BAT_OK) {
            if (best_kernel_ms) *best_kernel_ms = best;
            t_err.clear();
            return BAT_OK;
        }
    }
    for (int seg : {6, 5, 4})
        for (int chain : {0, 3, 4, 5, 6}) {
            if (chain > seg) continue;
            const BatchTune c{chain, seg};
            double ms = 1e300;
            for (int rep = 0; rep < 3; ++rep) {
                rc = batched_impl(n_graphs, n_nodes, arc_offsets, arcs, s, t, n_pvec, p, R.data(), cnt.data(), &c);
                if (rc) return rc;
                bat_launch_info li;
                rc = bat_last_launch(&li);
                if (rc) return rc;
                if (rep > 0) ms = std::min(ms, li.kernel_ms);
            }
            if (verbose) fprintf(stderr, "bat_autotune_batched: seg_log2=%d chain=%d -> %.3f ms\n", seg, chain, ms);
            if (ms < best) {
                best = ms;
                bb = c;
            }
        }
    // then graph-specialised kernels for the largest graphs (thresholds on
    // the arc count: the largest, 2 and 4 below it), with the winning
    // segment size and chain length; a threshold must win by 2% over none.
    // (Smaller segments for the specialised graphs, which spread a graph
    // over more wavefronts, measured slower on 256 graphs x 32 p-vectors.)
    if (bb.chain != 0) {
        int32_t m_max = 0;
        for (int32_t g = 0; g < n_graphs; ++g) m_max = std::max(m_max, arc_offsets[g + 1] - arc_offsets[g]);
        const double base = best;
        const BatchTune gen = bb;
        // each threshold with 3, 2 and 1 side streams: which hardware queue
        // a stream lands on depends on the streams the process made before
        // it (torch's default stream, once used, holds one of HIP's 4), and
        // a threshold measured on shared queues loses to a worse one
        for (int arcs_min : {m_max - 4, m_max - 2, m_max}) {
            if (arcs_min < bat::kWordBits + 3) continue;
            for (int ns : {3, 2, 1}) {
                BatchTune c = gen;
                c.jit_arcs = arcs_min;
                c.streams = ns;
                double ms = 1e300;
                for (int rep = 0; rep < 3; ++rep) {
                    rc = batched_impl(n_graphs, n_nodes, arc_offsets, arcs, s, t, n_pvec, p, R.data(), cnt.data(), &c);
                    if (rc) return rc;
                    bat_launch_info li;
                    rc = bat_last_launch(&li);
                    if (rc) return rc;
                    if (rep > 0) ms = std::min(ms, li.kernel_ms);
                }
                if (verbose)
                    fprintf(stderr,
                            "bat_autotune_batched: seg_log2=%d chain=%d specialised from %d arcs on %d side streams "
                            "-> %.3f ms\n",
                            c.seg, c.chain, arcs_min, ns, ms);
                if (ms < best && ms < base * 0.98) {
                    best = ms;
                    bb = c;
                }
            }
        }
        if (bb.jit_arcs < 0) bb.jit_arcs = 0;  // tuned: none
    }
    {
        std::lock_guard<std::mutex> lk(g_btune_mu);
        g_btune[batch_key(D.id, n_graphs, n_nodes, arc_offsets, arcs, s, t, n_pvec)] = bb;
    }
    if (best_kernel_ms) *best_kernel_ms = best;
    t_err.clear();
    return BAT_OK;
}

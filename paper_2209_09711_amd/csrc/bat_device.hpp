// bat_device.hpp -- device code for exact BAT reliability on CDNA4 (gfx950).
//
// Included twice: by bat_kernels.hip (ahead-of-time kernels that read the
// graph at run time) and, as embedded text, by the graph-specialised
// kernels compiled at run time with hiprtc (graph baked in as constants).
// It therefore includes no header: hiprtc provides the HIP device API.
//
// What is computed (Section 3, Eq. 1): for every arc-state vector X of the
// 2^m generated by the BAT (Section 3.1), whether s and t are connected in
// G(X) (the PLSA question of Section 3.2), the count of such X and the sum
// of Pr(X) = prod_i q_i(x_i) over them; optionally the per-arc sums T1_i,
// T0_i whose difference is dR/dp_i.
//
// Mapping of the enumeration onto the machine.  The counter c (0-based BAT
// index, Eq. 2-3: arc i is bit m-1-i, so counter bit cb belongs to arc
// m-1-cb) is split as
//     c = g << 11 | lane << 5 | j
// j (5 bits, "slice"): the 32 vectors held in the 32 bits of one word;
// lane (6 bits): the wavefront lane; g: the loop iteration, uniform across
// the wavefront.  One wavefront iteration therefore decides 2048 vectors.
// Connectivity is decided bit-sliced: reach[v] is a 32-bit word whose bit j
// says node v is reachable from s in vector j.  Relaxing arc (u, v) is
//     reach[v] |= reach[u] & W;  reach[u] |= reach[v] & W
// where W says in which of the 32 vectors the arc works: a constant bit
// pattern for slice arcs, all-ones/all-zeros per lane for lane arcs, and
// uniform for iteration arcs.  Sweeps in BFS order from s, alternately
// forward and backward, repeat until a sweep changes nothing (the layered
// search's fixed point: no new node can join a layer) or t is reached in
// all 32 vectors (the layered search's early stop at the sink).  Each sweep
// is 2 VALU ops per arc for 2048 vectors.
//
// Probability (Eq. 1) factorises along the same split:
//     Pr(X) = Q_U(g) * Q_L(lane) * Q_S(j),   Q_S(j) = A(j >> 3) * B(j & 7)
// so the connected mass of one word V is
//     F(V) = sum_{h<4} A(h) * TB[byte h of V],   TB[x] = sum_{i in x} B(i)
// read from a 256-entry table in LDS; Q_U(g) = Q_hi(g >> f) * Q_lo(g mod 2^f).
// Lanes accumulate short segments of Q_lo * F, segments are folded into a
// double-double with Q_hi, and the lane totals are multiplied by Q_L and
// reduced across the wavefront in double-double, then across work items in
// fixed order: no floating-point atomics, bitwise deterministic.

namespace bat {

typedef unsigned int u32;
typedef unsigned long long u64;

constexpr int kSliceBits = 5;
constexpr int kLaneBits = 6;
constexpr int kWordBits = 11;  // slice + lane
constexpr int kWave = 64;
constexpr int kWavesPerBlock = 4;  // blocks of the generic and gradient sweeps
constexpr int kBlock = kWave * kWavesPerBlock;
constexpr int kMaxSegLog = 8;
constexpr int kGradFastMax = 4;  // fast iteration bits the gradient sweep keeps per-lane sums for
constexpr int kKeepBottomMaxNodes = 32;  // graphs up to this many relevant nodes keep chained-block bottoms
constexpr int kMaxArcs = 62;

// ---------------------------------------------------------------- tables
// Offsets (in doubles) inside the table block written by build_tables.
constexpr int kTB = 0;                       // [256]  B-sums over slice bits 0..2
constexpr int kA4 = kTB + 256;               // [4]    A over slice bits 3..4
constexpr int kQL = kA4 + 4;                 // [64]   Q_L(lane)
constexpr int kQlo = kQL + 64;               // [256]  Q_lo(g mod 2^f)
constexpr int kQG = kQlo + 256;              // [128]  (q(0), q(1)) of g bit b at 2b, 2b+1
constexpr int kTBG = kQG + 128;              // [6][256] TB_a^x, a = 0..2, x = 0..1
constexpr int kA4M = kTBG + 6 * 256;         // [2][4] A without slice bit 3 / 4
constexpr int kQLM = kA4M + 8;               // [6][64] Q_L without lane bit b
constexpr int kQLOM = kQLM + 6 * 64;         // [8][256] Q_lo without g bit b
constexpr int kTablesFwd = kTBG;             // doubles the forward kernel needs
constexpr int kTables = kQLOM + 8 * 256;     // whole block

// (a & b) | c.  v_bitop3_b32 issues at the full rate (1.7 wave64
// instructions per CU and clock measured), v_and_or_b32, which the compiler
// picks for the plain expression, at half of it (0.95).
__device__ __forceinline__ u32 and_or(u32 a, u32 b, u32 c)
{
#if defined(__HIP_DEVICE_COMPILE__) || defined(__HIPCC_RTC__)
    return __builtin_amdgcn_bitop3_b32(a, b, c, 0xEA);
#else
    return (a & b) | c;  // hipcc's host pass, which parses this and has no such builtin
#endif
}

// The 32-bit word in which slice arc cb works: bit j set iff bit cb of j.
__host__ __device__ constexpr u32 slice_pattern(int cb)
{
    return cb == 0 ? 0xAAAAAAAAu
         : cb == 1 ? 0xCCCCCCCCu
         : cb == 2 ? 0xF0F0F0F0u
         : cb == 3 ? 0xFF00FF00u
                   : 0xFFFF0000u;
}

struct KParams {
    u64 c_lo, c_hi;        // counter range [c_lo, c_hi)
    u64 g_first, g_last;   // inclusive iteration range: g_first = c_lo >> 11 ...
    u64 g_base, g_end;     // iterations actually swept (block-aligned when chained); vectors
                           // outside [c_lo, c_hi) are masked out
    u64 chunk_iters;       // iterations per wavefront work item
    u64 n_chunks;          // work items
    u64 chunk_mul;         // work item w sweeps chunk (w * chunk_mul) & chunk_mask: the identity
    u64 chunk_mask;        // (1, ~0) normally; an odd multiplier spreads a timing sample
    u32 m;                 // arcs
    u32 ubits;             // iteration bits = max(m - 11, 0)
    u32 seg_log;           // f: iteration bits folded through Q_lo
    u32 check_every;       // 1: convergence test after every sweep, 2: every pair
    u32 chain;             // k > 0: warm-started chains over the k (3..6) lowest iteration bits
    u32 ncol;              // result columns: 1 (R) or 1 + 2 m (R, T1/T0 per bit)
    u32 window_test;       // 1: skip chained blocks that no vector of can connect (see window_live)
    // run-time graph (generic kernels only)
    u32 n_nodes, s, t, n_relax;
    u32 n_groups;          // ceil(n_relax / 4)
    u32 ck_code[6];        // relaxation code of counter bit 11 + b (~0: pruned)
    // [2 n_groups + 1][4][2]: the forward sweep's relaxations, then the
    // backward sweep's, each as (u | v << 6 | cb << 12, slice pattern of the
    // arc or 0) pairs in groups of 4, padded with (0, 0) pairs (no-ops),
    // then one spare group of no-ops
    const u32 *prog;
    const double *tables;  // table block
    const int *status;     // 0 if the probabilities were valid
    double *part;          // [n_chunks][ncol][2] double-double partials
    u64 *pcount;           // [n_chunks]
};

// ------------------------------------------------------- double-double
__device__ __forceinline__ void two_sum(double a, double b, double &s, double &e)
{
    s = a + b;
    double bb = s - a;
    e = (a - (s - bb)) + (b - bb);
}

__device__ __forceinline__ void dd_add(double &hi, double &lo, double xh, double xl)
{
    double s, e;
    two_sum(hi, xh, s, e);
    e += lo + xl;
    two_sum(s, e, hi, lo);
}

__device__ __forceinline__ double shfl_xor_d(double x, int m)
{
    return __shfl_xor(x, m, kWave);
}

// Butterfly reduction across the 64 lanes; every lane ends with the total.
__device__ __forceinline__ void wave_sum_dd(double &hi, double &lo)
{
#pragma unroll
    for (int off = kWave / 2; off >= 1; off >>= 1) {
        double oh = shfl_xor_d(hi, off), ol = shfl_xor_d(lo, off);
        dd_add(hi, lo, oh, ol);
    }
}

__device__ __forceinline__ u64 wave_sum_u64(u64 x)
{
#pragma unroll
    for (int off = kWave / 2; off >= 1; off >>= 1) x += __shfl_xor(x, off, kWave);
    return x;
}

// Which of the word's 32 vectors lie in [c_lo, c_hi).
__device__ __forceinline__ u32 edge_mask(u64 c_lo, u64 c_hi, u64 g, u32 lane)
{
    u64 base = (g << kWordBits) | ((u64)lane << kSliceBits);
    u64 lo = c_lo > base ? c_lo - base : 0ull;
    u64 hi = c_hi > base ? c_hi - base : 0ull;
    u32 mlo = lo >= 32 ? ~0u : ((1u << (u32)lo) - 1u);
    u32 mhi = hi >= 32 ? ~0u : ((1u << (u32)hi) - 1u);
    return mhi & ~mlo;
}

__device__ __forceinline__ void relax(u32 &ru, u32 &rv, u32 w)
{
    u32 a = ru, b = rv;
    rv = and_or(a, w, b);
    ru = and_or(b, w, a);
}

// ----------------------------------------------------------- closures
// Chains over the k lowest iteration bits (k = 3..6): a symmetric chain
// decomposition of the 2^k subsets (3, 6, 10, 20 chains).  Each step after a
// chain's first switches one more iteration arc on, so its closure can start
// from the previous one.  Entry: offset in the block (bits 0..5) and the bit
// switched on plus one (bits 6..8; 0 = cold start).
__device__ __constant__ unsigned short kChain3[8] = {
    0, 65, 131, 199, 4, 69, 2, 198};
__device__ __constant__ unsigned short kChain4[16] = {
    0, 65, 131, 199, 271, 8, 73, 139, 4, 69, 269, 12, 2, 198, 270, 10};
__device__ __constant__ unsigned short kChain5[32] = {
    0, 65, 131, 199, 271, 351, 16, 81, 147, 215, 8, 73, 139, 347, 24, 89, 4, 69, 269, 349, 20, 85, 12, 348,
    2, 198, 270, 350, 18, 214, 10, 346};
__device__ __constant__ unsigned short kChain6[64] = {
    0, 65, 131, 199, 271, 351, 447, 32, 97, 163, 231, 303, 16, 81, 147, 215, 439, 48, 113, 179, 8, 73, 139,
    347, 443, 40, 105, 171, 24, 89, 441, 56, 4, 69, 269, 349, 445, 36, 101, 301, 20, 85, 437, 52, 12, 348,
    444, 44, 2, 198, 270, 350, 446, 34, 230, 302, 18, 214, 438, 50, 10, 346, 442, 42};

// A closure policy decides the verdict word for (g, lane): bit j set iff s
// and t are connected in the vector c = g << 11 | lane << 5 | j.

// Sum of the popcounts of the reach words as one dependent chain of
// v_bcnt_u32_b32 (popcount plus accumulate): one instruction per node.  A
// sweep changed nothing exactly when this sum did not grow, because reach
// words only ever gain bits.
__device__ __forceinline__ u32 bcnt_acc(u32 x, u32 acc)
{
    u32 d;
    asm("v_bcnt_u32_b32 %0, %1, %2" : "=v"(d) : "v"(x), "v"(acc));
    return d;
}

// Graph known at compile time (hiprtc): every node is a fixed register.
// G provides N, S, T, NR, DIR (arcs are directed RU -> RV), SUPER (keep
// super-block bottoms in LDS), the arrays RU,
// RV, RB, RD (relaxation endpoints in forward sweep order, the counter bit
// of the relaxed arc, whether the relaxation is the one that first reaches
// RV in BFS order) and CK[6] (the relaxation of counter bits 11..16, or -1
// if that arc is pruned).
//
// State carried between calls: the reach words, the popcount sum at the
// last convergence test and whether the words are a fixed point of the arc
// set.  cold() starts from {s}; warm() starts from the previous state after
// one iteration arc has been switched on.  That is exact because reach is
// monotone in the arc set: the old reach is contained in the new one, and
// sweeping from any such under-approximation reaches the same fixed point.
template <class G, bool KEEP = true>
struct StaticClosure {
    static constexpr bool kWarm = true;
    // Keep the closure of each chained block's bottom (all chained bits
    // off) in registers, so later chain starts resume from it; only for
    // graphs small enough that the copy does not cost occupancy, and not
    // in the gradient sweep (KEEP = false), whose sums need the registers.
    static constexpr bool kKeepBottom = KEEP && G::KEEPB && G::N <= kKeepBottomMaxNodes;
    // ... in LDS (node-major per wavefront, like the super-block store)
    // rather than registers, which the compiler would spill when asked to
    // fit more wavefronts
    static constexpr bool kBottomLds = kKeepBottom && G::BOTTOM_LDS;
    // the reach words but s's (all ones), then prev | fixed << 31 (prev is
    // a popcount sum of at most 32 (N - 1) < 2^31)
    static constexpr int kBottomWords = G::N;
    static constexpr int bottom_slot(int i) { return i > G::S ? i - 1 : i; }
    // Also keep, in LDS, the closure of each 2^6-aligned super-block's
    // bottom: every later block bottom in it resumes from that state.
    static constexpr bool kSuper = kKeepBottom && G::SUPER;
    // Test whole windows of 2048 iterations at once for blocks that cannot
    // connect s and t (both sweeps: a skipped block adds nothing to R, T1
    // or T0).
    static constexpr bool kWindowTest = true;
    static constexpr int kSuperWords = G::N + 2;  // reach words, prev, fixed
    u32 lanew[kLaneBits];
    u32 r[G::N];
    u32 W[G::NR > 0 ? G::NR : 1];
    u32 prev;
    u32 fixed;
    u32 rb[kKeepBottom && !kBottomLds ? G::N : 1];
    u32 prevb, fixedb;

    u32 sbase;  // this lane's first word in the super-block store

    __device__ __forceinline__ void init(u32 lane, const KParams &)
    {
#pragma unroll
        for (int b = 0; b < kLaneBits; ++b) lanew[b] = 0u - ((lane >> b) & 1u);
        prev = 0u;
        fixed = 0u;
        sbase = (threadIdx.x >> 6) * (kSuperWords * kWave) + lane;
    }

    // node-major per wavefront: word i of lane l at [wave][i][l], so each
    // store or load of one word is contiguous across the wavefront
    __device__ static u32 *super_store()
    {
        __shared__ u32 sb[kSuper ? G::WAVES * kSuperWords * kWave : 1];
        return sb;
    }

    // The super-block bottom has just been solved cold: keep its state.
    __device__ __forceinline__ void keep_super()
    {
        if constexpr (kSuper) {
            u32 *sb = super_store() + sbase;
#pragma unroll
            for (int i = 0; i < G::N; ++i) sb[i * kWave] = r[i];
            sb[G::N * kWave] = prev;
            sb[(G::N + 1) * kWave] = fixed;
        }
    }

    // A block bottom inside a super-block whose bottom was kept: that
    // bottom's arc set plus the iteration arcs of the bits set in `off`
    // (bits k..5 of g).  Resume from the kept state.
    __device__ __forceinline__ u32 restart_super(u64 g, u32 off, const KParams &P)
    {
        if constexpr (!kSuper) {
            return cold(g, P);
        } else {
            if (G::NR == 0) return 0u;
            const u32 *sb = super_store() + sbase;
#pragma unroll
            for (int i = 0; i < G::N; ++i) r[i] = sb[i * kWave];
            prev = sb[G::N * kWave];
            fixed = sb[(G::N + 1) * kWave];
            set_masks(g);
            const bool c0 = consistent<G::CK[0]>(), c1 = consistent<G::CK[1]>(), c2 = consistent<G::CK[2]>(),
                       c3 = consistent<G::CK[3]>(), c4 = consistent<G::CK[4]>(), c5 = consistent<G::CK[5]>();
            const bool cons = (!(off & 1u) || c0) && (!(off & 2u) || c1) && (!(off & 4u) || c2) &&
                              (!(off & 8u) || c3) && (!(off & 16u) || c4) && (!(off & 32u) || c5);
            const bool done = (r[G::T] == ~0u) || (fixed && cons);
            if (!done) converge(true, P);
            return r[G::T];
        }
    }

    __device__ __forceinline__ u32 wmask(int cb, u64 g) const
    {
        if (cb < kSliceBits) return slice_pattern(cb);
        if (cb < kWordBits) return lanew[cb - kSliceBits];
        return 0u - (u32)((g >> (cb - kWordBits)) & 1ull);
    }

    // A relaxation standing for two arcs in series (RB2 < 255) works where
    // both do.
    __device__ __forceinline__ void set_masks(u64 g)
    {
#pragma unroll
        for (int k = 0; k < G::NR; ++k)
            W[k] = G::RB2[k] == 255 ? wmask(G::RB[k], g) : wmask(G::RB[k], g) & wmask(G::RB2[k], g);
    }

    // Masks of the window test: every word arc (counter bits 0..10) up;
    // iteration bits 0..10 take the word's place (0..4 the in-word index,
    // 5..10 the lane); the higher iteration bits are those of the window.
    __device__ __forceinline__ u32 wmask_window(int cb, u64 wbase) const
    {
        if (cb < kWordBits) return ~0u;
        if (cb < kWordBits + kSliceBits) return slice_pattern(cb - kWordBits);
        if (cb < 2 * kWordBits) return lanew[cb - kWordBits - kSliceBits];
        return 0u - (u32)((wbase >> (cb - kWordBits)) & 1ull);
    }

    // (s's word is all ones throughout and is left out)
    __device__ __forceinline__ u32 popsum() const
    {
        u32 ps = 0u;
#pragma unroll
        for (int i = 0; i < G::N; ++i)
            if (i != G::S) ps = bcnt_acc(r[i], ps);
        return ps;
    }

    __device__ __forceinline__ void sweep_fwd()
    {
#pragma unroll
        for (int k = 0; k < G::NR; ++k) rel(k);
    }

    // Relaxation k: both directions, or tail to head only for a digraph.
    // Reach that flows into s (already all ones) or out of t (already
    // decides the verdict) changes nothing, so relaxations at s or t run
    // one way only: out of s, into t.
    static constexpr int one_way(int k)
    {
        return G::DIR || G::RU[k] == G::S || G::RV[k] == G::T ? 1 : (G::RV[k] == G::S || G::RU[k] == G::T) ? 2 : 0;
    }

    // Relaxation k: both directions, or one (1: RU to RV, 2: RV to RU).
    // s's word is all ones, so out of s the mask alone flows (and s's
    // word is never read: it needs no register).
    __device__ __forceinline__ void rel(int k)
    {
        if (G::RU[k] == G::S) r[G::RV[k]] |= W[k];
        else if (one_way(k) == 1) r[G::RV[k]] = and_or(r[G::RU[k]], W[k], r[G::RV[k]]);
        else if (one_way(k) == 2) r[G::RU[k]] = and_or(r[G::RV[k]], W[k], r[G::RU[k]]);
        else relax(r[G::RU[k]], r[G::RV[k]], W[k]);
    }

    // Forward sweep from relaxation K0 on (K0 < 0: all of it).
    template <int K0>
    __device__ __forceinline__ void sweep_fwd_from()
    {
        if constexpr (K0 <= 0) {
            sweep_fwd();
        } else {
#pragma unroll
            for (int k = K0; k < G::NR; ++k) rel(k);
        }
    }

    __device__ __forceinline__ void sweep_bwd()
    {
#pragma unroll
        for (int k = G::NR - 1; k >= 0; --k) rel(k);
    }

    // true: stop (t reached in every vector, or the sweep changed nothing)
    __device__ __forceinline__ bool settled(bool test)
    {
        if (r[G::T] == ~0u) {
            fixed = 0u;
            return true;
        }
        if (!test) return false;
        u32 ps = popsum();
        if (ps == prev) {
            fixed = 1u;
            return true;
        }
        prev = ps;
        return false;
    }

    // Alternate sweeps until settled.
    __device__ __forceinline__ void converge(bool fwd_first, const KParams &P)
    {
        const bool every = P.check_every < 2;
        for (int it = 0; it < 32 * G::N + 4; ++it) {
            if (fwd_first) sweep_fwd();
            else sweep_bwd();
            if (settled(every)) break;
            if (fwd_first) sweep_bwd();
            else sweep_fwd();
            if (settled(true)) break;
        }
    }

    // Bit j of lane l: whether iteration wbase + 32 l + j (wbase 2048-
    // aligned) connects s and t with all 11 word arcs up.  Where it does
    // not, none of that iteration's 2048 vectors is connected, since
    // switching arcs off never adds a path; nor is any vector of an
    // iteration whose iteration arcs are a subset of its.
    __device__ __forceinline__ u32 window_live(u64 wbase, const KParams &P)
    {
        if (G::NR == 0) return 0u;
#pragma unroll
        for (int k = 0; k < G::NR; ++k)
            W[k] = G::RB2[k] == 255 ? wmask_window(G::RB[k], wbase)
                                    : wmask_window(G::RB[k], wbase) & wmask_window(G::RB2[k], wbase);
        return solve(P);
    }

    __device__ __forceinline__ u32 cold(u64 g, const KParams &P)
    {
        if (G::NR == 0) return 0u;
        set_masks(g);
        return solve(P);
    }

    // The closure from {s} under the current masks.
    __device__ __forceinline__ u32 solve(const KParams &P)
    {
        // First forward sweep in BFS order: the relaxation that discovers a
        // node is its first write, so it assigns (r[v] = r[u] & W; the
        // reverse direction cannot add anything yet) and nothing needs
        // clearing beforehand.
        r[G::S] = ~0u;
#pragma unroll
        for (int k = 0; k < G::NR; ++k) {
            if (G::RD[k]) r[G::RV[k]] = r[G::RU[k]] & W[k];
            else rel(k);
        }
        if (r[G::T] == ~0u) {
            fixed = 0u;
            return ~0u;
        }
        prev = popsum();
        converge(false, P);
        return r[G::T];
    }

    template <int K>
    __device__ __forceinline__ bool consistent() const
    {
        // a fixed point stays one when the new arc adds nothing: equal
        // reach words, or for a digraph, the tail's inside the head's
        // (a one-way relaxation: the source's inside the target's)
        if constexpr (K < 0) return true;
        else if constexpr (G::RU[K] == G::S) return r[G::RV[K]] == ~0u;
        else if constexpr (one_way(K) == 1) return (r[G::RU[K]] & ~r[G::RV[K]]) == 0u;
        else if constexpr (one_way(K) == 2) return (r[G::RV[K]] & ~r[G::RU[K]]) == 0u;
        else return r[G::RU[K]] == r[G::RV[K]];
    }

    // Iteration bit `bit` (0..5) has just been switched on.  A fixed point
    // of the old arc set stays one exactly when the new arc's endpoints
    // already have equal reach words.  Otherwise every relaxation before
    // the new arc's is still a no-op, so the first forward sweep starts at
    // the new arc.  (Lanes that stopped with t reached in all 32 vectors
    // hold no fixed point but keep that verdict: reach only grows.)
    __device__ __forceinline__ u32 warm(u64 g, u32 bit, const KParams &P)
    {
        if (G::NR == 0) return 0u;
        set_masks(g);
        // all the compares, then a select on the uniform bit (a branch per
        // bit would be folded into a scratch-memory lookup table)
        const bool c0 = consistent<G::CK[0]>(), c1 = consistent<G::CK[1]>(), c2 = consistent<G::CK[2]>(),
                   c3 = consistent<G::CK[3]>(), c4 = consistent<G::CK[4]>(), c5 = consistent<G::CK[5]>();
        const bool cons = bit == 0 ? c0 : bit == 1 ? c1 : bit == 2 ? c2 : bit == 3 ? c3 : bit == 4 ? c4 : c5;
        const bool done = (r[G::T] == ~0u) || (fixed && cons);
        if (!done) {
            switch (bit) {
            case 0: sweep_fwd_from<G::CK[0]>(); break;
            case 1: sweep_fwd_from<G::CK[1]>(); break;
            case 2: sweep_fwd_from<G::CK[2]>(); break;
            case 3: sweep_fwd_from<G::CK[3]>(); break;
            case 4: sweep_fwd_from<G::CK[4]>(); break;
            default: sweep_fwd_from<G::CK[5]>(); break;
            }
            if (!settled(P.check_every < 2)) converge(false, P);
        }
        return r[G::T];
    }

    // The block bottom has just been solved cold: keep its state.
    __device__ static u32 *bottom_store()
    {
        __shared__ u32 bs[kBottomLds ? G::WAVES * kBottomWords * kWave : 1];
        return bs;
    }

    __device__ __forceinline__ void keep_bottom()
    {
        if constexpr (kBottomLds) {
            u32 *bs = bottom_store() + (threadIdx.x >> 6) * (kBottomWords * kWave) + (threadIdx.x & (kWave - 1));
#pragma unroll
            for (int i = 0; i < G::N; ++i)
                if (i != G::S) bs[bottom_slot(i) * kWave] = r[i];
            bs[(G::N - 1) * kWave] = prev | (fixed << 31);
        } else if constexpr (kKeepBottom) {
#pragma unroll
            for (int i = 0; i < G::N; ++i) rb[i] = r[i];
            prevb = prev;
            fixedb = fixed;
        }
    }

    // A chain start at offset `off` inside the block: the bottom's arc set
    // plus the chained arcs whose bits are set in `off`.  Resume from the
    // bottom's state; it stays a fixed point exactly when every one of
    // those arcs joins equal reach words.
    __device__ __forceinline__ u32 restart(u64 g, u32 off, const KParams &P)
    {
        if constexpr (!kKeepBottom) {
            return cold(g, P);
        } else {
            if (G::NR == 0) return 0u;
            if constexpr (kBottomLds) {
                const u32 *bs =
                    bottom_store() + (threadIdx.x >> 6) * (kBottomWords * kWave) + (threadIdx.x & (kWave - 1));
#pragma unroll
                for (int i = 0; i < G::N; ++i) r[i] = i == G::S ? ~0u : bs[bottom_slot(i) * kWave];
                const u32 pf = bs[(G::N - 1) * kWave];
                prev = pf & 0x7fffffffu;
                fixed = pf >> 31;
            } else {
#pragma unroll
                for (int i = 0; i < G::N; ++i) r[i] = rb[i];
                prev = prevb;
                fixed = fixedb;
            }
            set_masks(g);
            const bool c0 = consistent<G::CK[0]>(), c1 = consistent<G::CK[1]>(), c2 = consistent<G::CK[2]>(),
                       c3 = consistent<G::CK[3]>(), c4 = consistent<G::CK[4]>(), c5 = consistent<G::CK[5]>();
            const bool cons = (!(off & 1u) || c0) && (!(off & 2u) || c1) && (!(off & 4u) || c2) &&
                              (!(off & 8u) || c3) && (!(off & 16u) || c4) && (!(off & 32u) || c5);
            const bool done = (r[G::T] == ~0u) || (fixed && cons);
            if (!done) converge(true, P);
            return r[G::T];
        }
    }

    __device__ __forceinline__ u32 verdict(u64 g, const KParams &P) { return cold(g, P); }
};

typedef const __attribute__((address_space(4))) u32 ConstU32;

// Graph read at run time: the relaxation list is uniform, so node ids are
// scalar values and reach[] is indexed through the VGPR-index mode.  The
// reach words persist across the iterations of a work item, so chained
// blocks warm-start here too (chain starts are solved cold: no kept bottom).
template <int NMAX, bool DIR = false>
struct DynClosure {
    static constexpr bool kWarm = false;  // chains run inside sweep_range
    u32 lane;

    __device__ __forceinline__ void init(u32 l, const KParams &) { lane = l; }

    // Iterations g0..g1 (g0 aligned to 2^chain when chain > 0): add(g, V)
    // receives each iteration's verdict word, done(blk, n) follows each
    // block of n iterations starting at blk.  With chain = k > 0 the
    // iterations go in blocks of 2^k along the chain tables and each step
    // that switches one arc on resumes from the previous fixed point (the
    // arc's relaxation code comes with the launch, ~0 = pruned: consistent).
    // The reach words stay a local array so that they live in registers
    // indexed through the VGPR-index mode.
    template <class Add, class Done>
    __device__ __forceinline__ void sweep_range(u64 g0, u64 g1, u32 chain, const KParams &P, Add &&add,
                                                Done &&done) const
    {
        u32 r[NMAX];
        const u32 s = __builtin_amdgcn_readfirstlane(P.s);
        const u32 t = __builtin_amdgcn_readfirstlane(P.t);
        const u32 nr = __builtin_amdgcn_readfirstlane(P.n_relax);
        const u32 ng = __builtin_amdgcn_readfirstlane(P.n_groups);
        // the program does not change during a launch: read it through the
        // constant address space, so uniform reads become scalar loads
        const ConstU32 *prog = (const ConstU32 *)P.prog;
        const bool every = P.check_every < 2;
        u32 ck[6];
#pragma unroll
        for (int b = 0; b < 6; ++b) ck[b] = __builtin_amdgcn_readfirstlane(P.ck_code[b]);
        u32 prev = 0u, fixed = 0u;
        const u32 nst = chain ? 1u << chain : 1u;
        const unsigned short *tab = chain == 6 ? kChain6 : chain == 5 ? kChain5 : chain == 4 ? kChain4 : kChain3;
        for (u64 blk = g0; blk <= g1; blk += nst) {
            for (u32 st = 0; st < nst; ++st) {
                const u32 e = chain ? tab[st] : 0u;
                const u64 g = blk + (e & 63u);
                const u32 bit = e >> 6;  // 0: cold start, else chained bit + 1
                if (nr == 0) {
                    add(g, 0u);
                    continue;
                }
                bool run = true;
                if (bit == 0) {
#pragma unroll
                    for (int i = 0; i < NMAX; ++i) r[i] = 0u;
                    r[s] = ~0u;
                    prev = 32u;
                } else {
                    // uniform select (a run-time index would put the
                    // parameter block in scratch memory)
                    const u32 code = bit == 1u   ? ck[0]
                                     : bit == 2u ? ck[1]
                                     : bit == 3u ? ck[2]
                                     : bit == 4u ? ck[3]
                                     : bit == 5u ? ck[4]
                                                 : ck[5];
                    bool cons = true;
                    if (code != ~0u) {
                        const u32 ru = r[code & 63u], rv = r[(code >> 6) & 63u];
                        cons = DIR ? (ru & ~rv) == 0u : ru == rv;
                    }
                    run = !((r[t] == ~0u) || (fixed && cons));
                }
                if (run) {
                    // alternate sweeps until t is reached in every vector
                    // (fixed = 0) or a sweep changes nothing (fixed = 1)
                    const u64 cbase = (g << kWordBits) | ((u64)lane << kSliceBits);
                    u32 dir = 0u;
                    fixed = 0u;
                    for (int it = 0; it < 2 * (32 * NMAX + 4); ++it) {
                        // the direction is the same in every active lane;
                        // saying so keeps the program reads scalar (inside
                        // this per-lane branch the compiler cannot tell)
                        const u32 d = __builtin_amdgcn_readfirstlane(dir);
                        const ConstU32 *pg = prog + (d ? ng * 8u : 0u);
                        // four relaxations per scalar load; the next group
                        // is loaded while this one runs (the program ends
                        // with a spare group)
                        u32 cur[8];
#pragma unroll
                        for (int j = 0; j < 8; ++j) cur[j] = pg[j];
                        for (u32 q = 0; q < ng; ++q) {
                            u32 nxt[8];
#pragma unroll
                            for (int j = 0; j < 8; ++j) nxt[j] = pg[(q + 1u) * 8u + j];
#pragma unroll
                            for (int j = 0; j < 4; ++j) {
                                const u32 code = cur[2 * j], wc = cur[2 * j + 1];
                                const u32 u = code & 63u, v = (code >> 6) & 63u, cb = (code >> 12) & 63u;
                                const u32 w = wc | (0u - (u32)((cbase >> cb) & 1ull));
                                const u32 ru = r[u], rv = r[v];
                                r[v] = rv | (ru & w);
                                if constexpr (!DIR) r[u] = ru | (rv & w);
                            }
#pragma unroll
                            for (int j = 0; j < 8; ++j) cur[j] = nxt[j];
                        }
                        if (r[t] == ~0u) break;
                        if (d == 1u || every) {
                            u32 ps = 0;
#pragma unroll
                            for (int i = 0; i < NMAX; ++i) ps += __popc(r[i]);
                            if (ps == prev) {
                                fixed = 1u;
                                break;
                            }
                            prev = ps;
                        }
                        dir ^= 1u;
                    }
                }
                add(g, r[t]);
            }
            done(blk, (u64)nst);
        }
    }
};

// ------------------------------------------------------ LDS table copy
struct alignas(16) Pair {
    double x, y;
};
struct LdsTables {
    double tb[256];
    double a4[4];
    double ql[64];
    double qlo[256];
    double qg[128];
};
struct LdsGrad {
    // one 64-byte record per in-word byte value: TB, then TB_a^x for
    // a = 0..2, x = 0..1, then padding, read as four 16-byte loads
    alignas(16) double tbx[256 * 8];
    double a4m[8];
    double qlm[6 * 64];
    // Q_lo without iteration bit b, for the fast bits the gradient keeps
    // (b < kGradFastMax, f <= kGradFastMax): [b][g mod 2^f]
    double qlom[kGradFastMax << kGradFastMax];
};

// tid of nthreads (the block's threads) copies a share
__device__ __forceinline__ void load_tables(const double *T, LdsTables &L, u32 tid, u32 nthreads)
{
    for (u32 i = tid; i < (u32)kTBG; i += nthreads) {
        double v = T[i];
        if (i < 256) L.tb[i] = v;
        else if (i < 260) L.a4[i - 256] = v;
        else if (i < 324) L.ql[i - 260] = v;
        else if (i < 580) L.qlo[i - 324] = v;
        else L.qg[i - 580] = v;
    }
}

__device__ __forceinline__ void load_grad_tables(const double *T, LdsGrad &L, u32 tid, u32 nthreads)
{
    for (u32 i = tid; i < 256 * 8; i += nthreads) {
        const u32 rec = i >> 3, c = i & 7u;
        L.tbx[i] = c == 0 ? T[kTB + rec] : c < 7 ? T[kTBG + (c - 1) * 256 + rec] : 0.0;
    }
    for (u32 i = tid; i < 8; i += nthreads) L.a4m[i] = T[kA4M + i];
    for (u32 i = tid; i < 6 * 64; i += nthreads) L.qlm[i] = T[kQLM + i];
    for (u32 i = tid; i < (u32)(kGradFastMax << kGradFastMax); i += nthreads)
        L.qlom[i] = T[kQLOM + (i >> kGradFastMax) * 256 + (i & ((1u << kGradFastMax) - 1u))];
}

// Q_hi(g): product over the iteration bits >= f, optionally leaving one out.
__device__ __forceinline__ double q_hi(const LdsTables &L, u64 g, u32 f, u32 ubits, u32 skip)
{
    double q = 1.0;
    for (u32 b = f; b < ubits; ++b) {
        double x = L.qg[2 * b + (u32)((g >> b) & 1ull)];
        q = (b == skip) ? q : q * x;
    }
    return q;
}

// ------------------------------------------------------- accumulation
// Per-lane sums of one work item (see the header for the factorisation).
// R: segments of 2^f iterations of Q_lo * F(V), folded with Q_hi into a
// double-double.  Gradient sums go straight into per-work-item totals with
// the uniform factor Q_hi * Q_lo (a work item is at most 4096 iterations,
// so each total adds at most 4096 positive terms).
template <bool GRAD>
struct Accum {
    double tot_hi, tot_lo;  // sum_g Q_U(g) F(V), without Q_L
    u64 cnt;
    double seg, qhi;
    double tot_fast[kGradFastMax][2];
    double tot_sl[3][2];    // slice arcs 0..2 (bits inside a byte)
    double tot_tb[4];       // sum_g Q_U Q_lo TB[byte h of V]: slice arcs 3, 4
    double slow_hi[2], slow_lo[2];

    __device__ __forceinline__ void zero(const KParams &)
    {
        tot_hi = tot_lo = seg = 0.0;
        qhi = 1.0;
        cnt = 0;
        if (GRAD) {
#pragma unroll
            for (int b = 0; b < kGradFastMax; ++b) tot_fast[b][0] = tot_fast[b][1] = 0.0;
#pragma unroll
            for (int a = 0; a < 3; ++a) tot_sl[a][0] = tot_sl[a][1] = 0.0;
#pragma unroll
            for (int h = 0; h < 4; ++h) tot_tb[h] = 0.0;
            slow_hi[0] = slow_hi[1] = slow_lo[0] = slow_lo[1] = 0.0;
        }
    }

    __device__ __forceinline__ void start_segment(const LdsTables &L, u64 g, u32 f, u32 ubits)
    {
        qhi = q_hi(L, g, f, ubits, 0xffffffffu);
    }

    // One verdict word of iteration g (glo = g mod 2^f).
    __device__ __forceinline__ void add(const LdsTables &L, const LdsGrad *LG, u32 V, u32 glo, u32 f)
    {
        cnt += __popc(V);
        const u32 b0 = V & 255u, b1 = (V >> 8) & 255u, b2 = (V >> 16) & 255u, b3 = V >> 24;
        const double ql = L.qlo[glo];
        if constexpr (!GRAD) {
            const double t0 = L.tb[b0], t1 = L.tb[b1], t2 = L.tb[b2], t3 = L.tb[b3];
            double F = L.a4[0] * t0;
            F = __builtin_fma(L.a4[1], t1, F);
            F = __builtin_fma(L.a4[2], t2, F);
            F = __builtin_fma(L.a4[3], t3, F);
            seg = __builtin_fma(ql, F, seg);
        } else {
            // byte by byte: record h holds TB and TB_a^x (a = 0..2, x = 0..1)
            // of byte h's value; one record live at a time
            double F = 0.0, sg[6] = {0.0, 0.0, 0.0, 0.0, 0.0, 0.0}, tb[4];
            const u32 bs[4] = {b0, b1, b2, b3};
#pragma unroll
            for (int h = 0; h < 4; ++h) {
                const Pair *rp = reinterpret_cast<const Pair *>(LG->tbx + bs[h] * 8u);
                const Pair v0 = rp[0], v1 = rp[1], v2 = rp[2], v3 = rp[3];
                const double ah = L.a4[h];
                tb[h] = v0.x;
                F = __builtin_fma(ah, v0.x, F);
                sg[0] = __builtin_fma(ah, v0.y, sg[0]);
                sg[1] = __builtin_fma(ah, v1.x, sg[1]);
                sg[2] = __builtin_fma(ah, v1.y, sg[2]);
                sg[3] = __builtin_fma(ah, v2.x, sg[3]);
                sg[4] = __builtin_fma(ah, v2.y, sg[4]);
                sg[5] = __builtin_fma(ah, v3.x, sg[5]);
            }
            seg = __builtin_fma(ql, F, seg);
            const double qq = qhi * ql;  // uniform
            // slice arcs 3 and 4 select the byte: their sums are fixed
            // combinations of the per-byte totals, formed once per work item
#pragma unroll
            for (int h = 0; h < 4; ++h) tot_tb[h] = __builtin_fma(qq, tb[h], tot_tb[h]);
            // slice arcs 0..2 select bits inside each byte
#pragma unroll
            for (int a = 0; a < 3; ++a) {
                tot_sl[a][0] = __builtin_fma(qq, sg[2 * a], tot_sl[a][0]);
                tot_sl[a][1] = __builtin_fma(qq, sg[2 * a + 1], tot_sl[a][1]);
            }
            // fast iteration arcs: bits below f of g (f <= kGradFastMax)
            const double qF = qhi * F;
            // (bits b >= f are slow arcs: their fast sums are never written;
            // the bit's state is uniform, so a 0/1 factor replaces a branch)
#pragma unroll
            for (int b = 0; b < kGradFastMax; ++b) {
                const double w = LG->qlom[(b << kGradFastMax) + glo] * qF;
                const bool on = (glo >> b) & 1u;
                const double x1 = on ? 1.0 : 0.0, x0 = on ? 0.0 : 1.0;
                tot_fast[b][1] = __builtin_fma(w, x1, tot_fast[b][1]);
                tot_fast[b][0] = __builtin_fma(w, x0, tot_fast[b][0]);
            }
        }
    }

    // Close the segment holding iteration g (its bits >= f are those of g).
    __device__ __forceinline__ void end_segment(const LdsTables &L, u64 g, u32 f, u32 ubits, u32 lane)
    {
        dd_add(tot_hi, tot_lo, qhi * seg, 0.0);
        if (GRAD) {
            // slow iteration arcs (bits >= f): the lane whose id is the bit
            // owns that arc's sums for this work item
            if (ubits > f) {
                double sh = L.ql[lane] * seg, sl = 0.0;
                wave_sum_dd(sh, sl);
                if (lane >= f && lane < ubits) {
                    double qm = q_hi(L, g, f, ubits, lane);
                    u32 x = (u32)((g >> lane) & 1ull);
                    double vh = qm * sh, vl = qm * sl;
                    if (x) dd_add(slow_hi[1], slow_lo[1], vh, vl);
                    else dd_add(slow_hi[0], slow_lo[0], vh, vl);
                }
            }
        }
        seg = 0.0;
    }

    // Fold the wavefront and write the work item's partials.
    __device__ __forceinline__ void write(const KParams &P, const LdsTables &L, const LdsGrad *LG, u64 chunk,
                                          u32 lane, u32 f, u32 ubits)
    {
        double *out = P.part + chunk * (u64)P.ncol * 2ull;
        const double qlane = L.ql[lane];
        double rh = qlane * tot_hi, rl = qlane * tot_lo;
        wave_sum_dd(rh, rl);
        u64 csum = wave_sum_u64(cnt);
        if (lane == 0) {
            out[0] = rh;
            out[1] = rl;
            P.pcount[chunk] = csum;
        }
        if (!GRAD) return;
        const u32 m = P.m;
        // column of counter bit cb, state x
        auto col = [&](u32 cb, u32 x) -> double * { return out + 2 * (1 + 2 * cb + x); };
        // lane arcs (counter bits 5..10)
        const double tot = tot_hi + tot_lo;
#pragma unroll
        for (int b = 0; b < kLaneBits; ++b) {
            const double v = LG->qlm[b * 64 + lane] * tot;
            const u32 x = (lane >> b) & 1u;
            double h1 = x ? v : 0.0, l1 = 0.0, h0 = x ? 0.0 : v, l0 = 0.0;
            wave_sum_dd(h1, l1);
            wave_sum_dd(h0, l0);
            const u32 cb = kSliceBits + b;
            if (lane == 0 && cb < m) {
                double *o1 = col(cb, 1), *o0 = col(cb, 0);
                o1[0] = h1; o1[1] = l1; o0[0] = h0; o0[1] = l0;
            }
        }
        // slice arcs (counter bits 0..4)
#pragma unroll
        for (int a = 0; a < kSliceBits; ++a) {
            double s1, s0;
            if (a < 3) {
                s1 = tot_sl[a][1];
                s0 = tot_sl[a][0];
            } else {
                const double *am = LG->a4m;
                if (a == 3) {
                    s0 = am[0] * tot_tb[0] + am[2] * tot_tb[2];
                    s1 = am[1] * tot_tb[1] + am[3] * tot_tb[3];
                } else {
                    s0 = am[4] * tot_tb[0] + am[5] * tot_tb[1];
                    s1 = am[6] * tot_tb[2] + am[7] * tot_tb[3];
                }
            }
            double h1 = qlane * s1, l1 = 0.0, h0 = qlane * s0, l0 = 0.0;
            wave_sum_dd(h1, l1);
            wave_sum_dd(h0, l0);
            if (lane == 0 && (u32)a < m) {
                double *o1 = col(a, 1), *o0 = col(a, 0);
                o1[0] = h1; o1[1] = l1; o0[0] = h0; o0[1] = l0;
            }
        }
        // fast iteration arcs (counter bits 11 .. 11+f-1)
#pragma unroll
        for (int b = 0; b < kGradFastMax; ++b) {
            if ((u32)b < f) {
                double h1 = qlane * tot_fast[b][1], l1 = 0.0, h0 = qlane * tot_fast[b][0], l0 = 0.0;
                wave_sum_dd(h1, l1);
                wave_sum_dd(h0, l0);
                if (lane == 0) {
                    double *o1 = col(kWordBits + b, 1), *o0 = col(kWordBits + b, 0);
                    o1[0] = h1; o1[1] = l1; o0[0] = h0; o0[1] = l0;
                }
            }
        }
        // slow iteration arcs: lane b owns counter bit 11 + b
        if (lane >= f && lane < ubits) {
            double *o1 = col(kWordBits + lane, 1), *o0 = col(kWordBits + lane, 0);
            o1[0] = slow_hi[1]; o1[1] = slow_lo[1]; o0[0] = slow_hi[0]; o0[1] = slow_lo[0];
        }
    }
};


// ------------------------------------------- batched accumulation
// The graph-specialised batched sweep: one verdict word serves NP
// probability vectors of the same graph (Eq. 1 with NP probability
// assignments).  Its work item is exactly one segment of 2^f iterations
// (f <= 6, the launch sizes it so): the segment's sum of Q_lo * F(V) per
// p-vector is scaled by that p-vector's Q_hi in place, then by Q_L(lane),
// and folded across the wavefront into column q of the item's partials.
constexpr int kBatchCols = 32;  // p-vector columns of a batched partial slot
constexpr int kBatchQlo = 64;   // Q_lo entries: 2^f, f <= 6

template <int NP>
struct LdsBatch {
    double tb[NP][256];
    double a4[NP][4];
    double qlo[NP][kBatchQlo];
    double full[NP];  // F(~0): a word whose 32 vectors all connect
};

// T: NP consecutive forward table blocks
template <int NP>
__device__ __forceinline__ void load_batch_tables(const double *T, LdsBatch<NP> &L, u32 tid, u32 nthreads)
{
    for (u32 i = tid; i < NP * 256u; i += nthreads) L.tb[i >> 8][i & 255u] = T[(u64)(i >> 8) * kTablesFwd + kTB + (i & 255u)];
    for (u32 i = tid; i < NP * 4u; i += nthreads) L.a4[i >> 2][i & 3u] = T[(u64)(i >> 2) * kTablesFwd + kA4 + (i & 3u)];
    for (u32 i = tid; i < NP * (u32)kBatchQlo; i += nthreads)
        L.qlo[i / kBatchQlo][i % kBatchQlo] = T[(u64)(i / kBatchQlo) * kTablesFwd + kQlo + (i % kBatchQlo)];
    __syncthreads();
    // the operations, in their order, of the table path for a word of ones
    for (u32 q = tid; q < (u32)NP; q += nthreads) {
        double F = L.a4[q][0] * L.tb[q][255];
        F = __builtin_fma(L.a4[q][1], L.tb[q][255], F);
        F = __builtin_fma(L.a4[q][2], L.tb[q][255], F);
        L.full[q] = __builtin_fma(L.a4[q][3], L.tb[q][255], F);
    }
    __syncthreads();
}

template <int NP>
struct AccumBatch {
    double tot[NP];  // this segment's sum of Q_lo * F(V), then times Q_hi
    u64 cnt;
    const double *T;

    __device__ __forceinline__ void zero(const KParams &P)
    {
#pragma unroll
        for (int q = 0; q < NP; ++q) tot[q] = 0.0;
        cnt = 0;
        T = P.tables;
    }

    __device__ __forceinline__ void start_segment(const LdsBatch<NP> &, u64, u32, u32) {}

    __device__ __forceinline__ void add(const LdsBatch<NP> &L0, const LdsGrad *, u32 V, u32 glo, u32)
    {
        cnt += __popc(V);
        if (__ballot(V != 0u) == 0ull) return;
        // re-read the per-p-vector factors every time (held in registers
        // they would take 4 NP doubles): an opaque zero offset keeps the
        // compiler from hoisting the reads out of the sweep loop
        u32 zero;
        asm volatile("v_mov_b32 %0, 0" : "=v"(zero));
        const LdsBatch<NP> &L = *(const LdsBatch<NP> *)((const char *)&L0 + zero);
        // words of all ones or all zeros across the wavefront (the five
        // in-word arcs do not matter): F is full or 0, no table reads
        if (__ballot(V != 0u && V != ~0u) == 0ull) {
            const double on = V ? 1.0 : 0.0;
#pragma unroll
            for (int q = 0; q < NP; ++q) tot[q] = __builtin_fma(L.qlo[q][glo], on * L.full[q], tot[q]);
            return;
        }
        const u32 b0 = V & 255u, b1 = (V >> 8) & 255u, b2 = (V >> 16) & 255u, b3 = V >> 24;
#pragma unroll
        for (int q = 0; q < NP; ++q) {
            double F = L.a4[q][0] * L.tb[q][b0];
            F = __builtin_fma(L.a4[q][1], L.tb[q][b1], F);
            F = __builtin_fma(L.a4[q][2], L.tb[q][b2], F);
            F = __builtin_fma(L.a4[q][3], L.tb[q][b3], F);
            tot[q] = __builtin_fma(L.qlo[q][glo], F, tot[q]);
        }
    }

    // the item's one segment ends: its bits >= f are those of g
    __device__ __forceinline__ void end_segment(const LdsBatch<NP> &, u64 g, u32 f, u32 ubits, u32)
    {
#pragma unroll
        for (int q = 0; q < NP; ++q) {
            const double *Tq = T + (u64)q * kTablesFwd + kQG;
            double qh = 1.0;
            for (u32 b = f; b < ubits; ++b) qh *= Tq[2 * b + (u32)((g >> b) & 1ull)];
            tot[q] *= qh;
        }
    }

    __device__ __forceinline__ void write(const KParams &P, const LdsBatch<NP> &, const LdsGrad *, u64 chunk, u32 lane,
                                          u32, u32)
    {
        double *out = P.part + chunk * (u64)kBatchCols * 2ull;
#pragma unroll
        for (int q = 0; q < NP; ++q) {
            double h = tot[q] * T[(u64)q * kTablesFwd + kQL + lane], l = 0.0;
            wave_sum_dd(h, l);
            if (lane == 0) {
                out[2 * q] = h;
                out[2 * q + 1] = l;
            }
        }
        const u64 c = wave_sum_u64(cnt);
        if (lane == 0) P.pcount[chunk] = c;
    }
};

// Transposed accumulation for 9..32 p-vectors.  Above 16, lane (q, h) =
// (lane & 31, lane >> 5) holds p-vector q's share of bytes h and h + 2 of
// every word: F_q(V) = A_q(0) TB_q[b0] + ... + A_q(3) TB_q[b3] is split
// over the lanes q and q + 32; up to 16, lane (q, h) = (lane & 15,
// lane >> 4) holds byte h alone, over four lanes.  Each iteration the
// wavefront classifies its 64 words by ballot: a word of zeros adds
// nothing, a word of ones adds Q_L(src) F_q(~0) (a masked sum of Q_L, or
// the whole sum when all 64 are ones), and only a mixed word (kept in the
// wavefront's LDS row) takes byte-table reads, one per byte the lane
// holds.  The table rows are padded to 257 doubles so that the p-vectors'
// reads of one byte value fall in different banks.  The registers hold one
// accumulator per lane instead of NP, and the item ends with one or two
// exchanges between the lanes of a p-vector instead of NP wavefront folds.
constexpr int kBatchTStride = 257;
constexpr int kBatchTMaxWaves = 16;

template <int NP>
struct LdsBatchT {
    double tb[NP][kBatchTStride];
    double qlo[NP][kBatchQlo + 1];
    double ql[NP][kWave + 1];
    double a4[NP][4];
    double qls[NP];  // sum of Q_L over the 64 lanes
    u32 row[kBatchTMaxWaves][kWave];
};

template <int NP>
__device__ __forceinline__ void load_batch_tables_t(const double *T, LdsBatchT<NP> &L, u32 tid, u32 nthreads)
{
    for (u32 i = tid; i < NP * 256u; i += nthreads) L.tb[i >> 8][i & 255u] = T[(u64)(i >> 8) * kTablesFwd + kTB + (i & 255u)];
    for (u32 i = tid; i < NP * 64u; i += nthreads) {
        L.qlo[i >> 6][i & 63u] = T[(u64)(i >> 6) * kTablesFwd + kQlo + (i & 63u)];
        L.ql[i >> 6][i & 63u] = T[(u64)(i >> 6) * kTablesFwd + kQL + (i & 63u)];
    }
    for (u32 i = tid; i < NP * 4u; i += nthreads) L.a4[i >> 2][i & 3u] = T[(u64)(i >> 2) * kTablesFwd + kA4 + (i & 3u)];
    __syncthreads();
    for (u32 q = tid; q < (u32)NP; q += nthreads) {
        double a = 0.0;
        for (u32 k = 0; k < 64u; ++k) a += L.ql[q][k];
        L.qls[q] = a;
    }
    __syncthreads();
}

template <int NP>
struct AccumBatchT {
    static_assert(NP > 8 && NP <= kBatchCols, "two or four lanes per p-vector");
    // p-vector slots across the wavefront: 32 (two lanes of two bytes each
    // per p-vector) above 16 p-vectors, else 16 (four lanes of one byte)
    static constexpr u32 kQN = NP > 16 ? 32u : 16u;
    static constexpr bool kTwoBytes = kQN == 32u;
    double tot;          // this segment's share of sum Q_lo Q_L F_q, then times Q_hi
    double a0, a1;       // A_q of the lane's bytes (0 for lanes past NP; a1 unused with one byte)
    double fullp, qlsum; // the lane's share of F_q(~0); sum of Q_L
    u64 cnt;
    const double *T;
    u32 lane, q, sh0, sh1;
    u32 *row;            // the wavefront's LDS row of mixed words

    __device__ __forceinline__ void zero(const KParams &P)
    {
        tot = 0.0;
        cnt = 0;
        T = P.tables;
        lane = threadIdx.x & (kWave - 1);
        const u32 qv = lane & (kQN - 1u);
        q = qv < (u32)NP ? qv : 0u;
        sh0 = 8u * (lane / kQN);
        sh1 = sh0 + 16u;
        a0 = a1 = fullp = qlsum = 0.0;
        row = nullptr;
    }

    __device__ __forceinline__ void start_segment(const LdsBatchT<NP> &L, u64, u32, u32)
    {
        const bool live = (lane & (kQN - 1u)) < (u32)NP;
        const u32 h = lane / kQN;
        a0 = live ? L.a4[q][h] : 0.0;
        a1 = (live && kTwoBytes) ? L.a4[q][(h + 2u) & 3u] : 0.0;
        const double t = L.tb[q][255];
        fullp = kTwoBytes ? __builtin_fma(a1, t, a0 * t) : a0 * t;
        qlsum = L.qls[q];
        row = const_cast<u32 *>(L.row[__builtin_amdgcn_readfirstlane(threadIdx.x >> 6)]);
    }

    __device__ __forceinline__ void add(const LdsBatchT<NP> &L, const LdsGrad *, u32 V, u32 glo, u32)
    {
        cnt += __popc(V);
        const u64 nz = __ballot(V != 0u);
        if (nz == 0ull) return;
        const u64 om = __ballot(V == ~0u);
        const u64 mm = nz & ~om;
        double x = 0.0;
        if (om != 0ull) {
            double os = 0.0;
            if (om == ~0ull) {
                os = qlsum;
            } else {
                for (u64 b = om; b != 0ull; b &= b - 1ull) os += L.ql[q][__builtin_ctzll(b)];
            }
            x = os * fullp;
        }
        if (mm != 0ull) {
            // the mixed words through the row: LDS operations of one
            // wavefront complete in order, so the reads see these writes
            row[lane] = V;
            asm volatile("" ::: "memory");
            for (u64 b = mm; b != 0ull; b &= b - 1ull) {
                const u32 s = (u32)__builtin_ctzll(b);
                const u32 Vs = row[s];
                double t = a0 * L.tb[q][(Vs >> sh0) & 255u];
                if constexpr (kTwoBytes) t = __builtin_fma(a1, L.tb[q][(Vs >> sh1) & 255u], t);
                x = __builtin_fma(L.ql[q][s], t, x);
            }
            asm volatile("" ::: "memory");
        }
        tot = __builtin_fma(L.qlo[q][glo], x, tot);
    }

    // the item's one segment ends: its bits >= f are those of g
    __device__ __forceinline__ void end_segment(const LdsBatchT<NP> &, u64 g, u32 f, u32 ubits, u32)
    {
        const double *Tq = T + (u64)q * kTablesFwd + kQG;
        double qh = 1.0;
        for (u32 b = f; b < ubits; ++b) qh *= Tq[2 * b + (u32)((g >> b) & 1ull)];
        tot *= qh;
    }

    __device__ __forceinline__ void write(const KParams &P, const LdsBatchT<NP> &, const LdsGrad *, u64 chunk, u32,
                                          u32, u32)
    {
        double *out = P.part + chunk * (u64)kBatchCols * 2ull;
        double h, l;
        two_sum(tot, shfl_xor_d(tot, 32), h, l);
        if constexpr (!kTwoBytes) {
            const double oh = shfl_xor_d(h, 16), ol = shfl_xor_d(l, 16);
            dd_add(h, l, oh, ol);
        }
        if (lane < (u32)NP) {
            out[2 * lane] = h;
            out[2 * lane + 1] = l;
        }
        const u64 c = wave_sum_u64(cnt);
        if (lane == 0) P.pcount[chunk] = c;
    }
};

// ------------------------------------------------------- the sweep body
// One wavefront processes work item `chunk`: iterations
// [g_base + chunk*chunk_iters, ...] up to g_end.
template <class Closure, bool GRAD, class Acc = Accum<GRAD>, class Tables = LdsTables>
__device__ void run_chunk(const KParams &P, Closure &cl, const Tables &L, const LdsGrad *LG, u64 item,
                          u64 chunk, u32 lane)
{
    const u64 g0 = P.g_base + chunk * P.chunk_iters;
    u64 g1 = g0 + P.chunk_iters - 1;
    if (g1 > P.g_end) g1 = P.g_end;
    const u32 f = P.seg_log;
    const u32 ubits = P.ubits;
    const u64 segmask = (1ull << f) - 1ull;
    Acc A;
    A.zero(P);
    bool chained = false;

    if constexpr (Closure::kWarm) {
        if (P.chain) {
            // blocks of 2^k iterations, aligned; f >= k so a block never
            // straddles a segment
            const u32 nst = 1u << P.chain;
            const unsigned short *tab = P.chain == 6 ? kChain6 : P.chain == 5 ? kChain5 : P.chain == 4 ? kChain4 : kChain3;
            u64 super_blk = ~0ull;  // super-block whose bottom is kept
            u64 wcur = ~0ull;       // window the test word covers
            u32 live = 0u;
            for (u64 blk = g0; blk <= g1; blk += nst) {
                if (blk == g0 || (blk & segmask) == 0) A.start_segment(L, blk, f, ubits);
                if constexpr (Closure::kWindowTest) {
                    if (P.window_test) {
                        // the block's top (every chained bit on) holds the
                        // most arcs of the block: if it cannot connect,
                        // nothing in the block can, and the block adds 0
                        const u64 wb = blk & ~(u64)(kWave * 32 - 1);
                        if (wb != wcur) {
                            live = cl.window_live(wb, P);
                            wcur = wb;
                        }
                        const u64 top = blk + nst - 1u;
                        const u32 w = (u32)__builtin_amdgcn_readlane((int)live, (int)((top >> 5) & 63u));
                        if (((w >> (top & 31u)) & 1u) == 0u) {
                            if (blk + nst > g1 || ((blk + nst) & segmask) == 0) A.end_segment(L, blk, f, ubits, lane);
                            continue;
                        }
                    }
                }
                for (u32 st = 0; st < nst; ++st) {
                    const u32 e = tab[st];
                    const u64 g = blk + (e & 63u);
                    u32 V;
                    if ((e >> 6) != 0) {
                        V = cl.warm(g, (e >> 6) - 1u, P);
                    } else if ((e & 63u) == 0) {
                        // block bottom: resume from the kept bottom of its
                        // 2^6-aligned super-block when this work item swept it
                        if constexpr (Closure::kSuper) {
                            const bool super_start = (blk & 63ull) == 0;
                            if (!super_start && super_blk == (blk & ~63ull)) {
                                V = cl.restart_super(g, (u32)(blk & 63ull), P);
                            } else {
                                V = cl.cold(g, P);
                                if (super_start) {
                                    cl.keep_super();
                                    super_blk = blk;
                                }
                            }
                        } else {
                            V = cl.cold(g, P);
                        }
                        cl.keep_bottom();
                    } else {
                        V = cl.restart(g, e & 63u, P);
                    }
                    if (g <= P.g_first || g >= P.g_last) V &= edge_mask(P.c_lo, P.c_hi, g, lane);
                    A.add(L, LG, V, (u32)(g & segmask), f);
                }
                if (blk + nst > g1 || ((blk + nst) & segmask) == 0) A.end_segment(L, blk, f, ubits, lane);
            }
            chained = true;
        }
    }
    if constexpr (Closure::kWarm) {
        if (!chained) {
            for (u64 g = g0;; ++g) {
                const u32 glo = (u32)(g & segmask);
                if (g == g0 || glo == 0) A.start_segment(L, g, f, ubits);
                u32 V = cl.verdict(g, P);
                if (g <= P.g_first || g >= P.g_last) V &= edge_mask(P.c_lo, P.c_hi, g, lane);
                A.add(L, LG, V, glo, f);
                if (g == g1 || ((g + 1) & segmask) == 0) A.end_segment(L, g, f, ubits, lane);
                if (g == g1) break;
            }
        }
    } else {
        // the run-time graph: its closure drives the iterations (chained
        // blocks or one by one); a block never straddles a segment
        cl.sweep_range(
            g0, g1, P.chain, P,
            [&](u64 g, u32 V) {
                const u32 glo = (u32)(g & segmask);
                if (g == g0 || glo == 0) A.start_segment(L, g, f, ubits);
                if (g <= P.g_first || g >= P.g_last) V &= edge_mask(P.c_lo, P.c_hi, g, lane);
                A.add(L, LG, V, glo, f);
            },
            [&](u64 blk, u64 n) {
                if (blk + n > g1 || ((blk + n) & segmask) == 0) A.end_segment(L, blk, f, ubits, lane);
            });
    }
    // one call site: the wave folds are long and run once per work item
    A.write(P, L, LG, item, lane, f, ubits);
}

// Kernel body: one work item per wavefront, 4 wavefronts per block.
template <class Closure, bool GRAD>
__device__ void sweep_kernel(const KParams &P, LdsTables &L, LdsGrad *LG)
{
    const u32 tid = threadIdx.x;
    // blocks of 1 to 4 wavefronts (the launch decides; the specialised
    // forward sweep may use fewer, so a finished wavefront's slot is not
    // held by the block's slower ones)
    const u32 nthreads = blockDim.x;
    load_tables(P.tables, L, tid, nthreads);
    if (GRAD) load_grad_tables(P.tables, *LG, tid, nthreads);
    __syncthreads();
    const u32 lane = tid & (kWave - 1);
    // wave-uniform: keeps the iteration counter and every quantity derived
    // from it (the iteration arcs' masks) in scalar registers
    const u32 wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const u64 item = (u64)blockIdx.x * __builtin_amdgcn_readfirstlane(nthreads >> 6) + wave;
    if (item >= P.n_chunks) return;
    Closure cl;
    cl.init(lane, P);
    run_chunk<Closure, GRAD>(P, cl, L, LG, item, (item * P.chunk_mul) & P.chunk_mask, lane);
}

// Batched kernel body (graph-specialised): NP probability vectors of one
// graph, their tables loaded once per block; each wavefront takes work
// items (one segment of 2^f iterations each) grid-stride until none is left.
template <class Closure, int NP>
__device__ void batch_kernel(const KParams &P, LdsBatch<NP> &L)
{
    const u32 tid = threadIdx.x;
    load_batch_tables<NP>(P.tables, L, tid, blockDim.x);
    const u32 lane = tid & (kWave - 1);
    const u32 wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const u32 wpb = __builtin_amdgcn_readfirstlane(blockDim.x >> 6);
    const u64 stride = (u64)gridDim.x * wpb;
    Closure cl;
    cl.init(lane, P);
    for (u64 item = (u64)blockIdx.x * wpb + wave; item < P.n_chunks; item += stride)
        run_chunk<Closure, false, AccumBatch<NP>, LdsBatch<NP>>(P, cl, L, nullptr, item, item, lane);
}

// The same with the transposed accumulation (17..32 p-vectors).
template <class Closure, int NP>
__device__ void batch_kernel_t(const KParams &P, LdsBatchT<NP> &L)
{
    const u32 tid = threadIdx.x;
    load_batch_tables_t<NP>(P.tables, L, tid, blockDim.x);
    const u32 lane = tid & (kWave - 1);
    const u32 wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const u32 wpb = __builtin_amdgcn_readfirstlane(blockDim.x >> 6);
    const u64 stride = (u64)gridDim.x * wpb;
    Closure cl;
    cl.init(lane, P);
    for (u64 item = (u64)blockIdx.x * wpb + wave; item < P.n_chunks; item += stride)
        run_chunk<Closure, false, AccumBatchT<NP>, LdsBatchT<NP>>(P, cl, L, nullptr, item, item, lane);
}


// ------------------------------------------ multi-state arcs, demand <= 2
// The multi-state reading (Section 4.1's solution space of prod sigma_i
// vectors, arcs with capacities) asks whether the maximum s-t flow reaches
// the demand d.  For d <= 3 max-flow min-cut gives that test a bit-sliced
// form: the flow is at least 1 when t is reachable from s over the arcs
// whose state gives capacity >= 1; at least 2 when besides no single arc
// of capacity exactly 1 separates them in that graph (a cut of capacity 1
// is one unit arc plus arcs of capacity 0); at least 3 when no single arc
// of capacity 1 or 2 and no two arcs of capacity 1 separate them (a cut of
// capacity 2 holds one arc of capacity 2 or two of capacity 1 besides arcs
// of capacity 0).  A word of up to 32 vectors is therefore decided as a
// binary word is: one closure over the capacity->=1 masks, then one
// closure without each arc (or pair) that could complete such a cut in a
// vector still connected.
//
// Mixed-radix split of a vector's index (slot 0 least significant):
//   word slots 0 .. KW-1       bit b of the word (B = prod of their states)
//   run slots KW .. KW+KR-1    the wavefront's loop step (uniform)
//   lane slots KW+KR .. M-1    the lane's run index
// G (compiled at run time for one graph and one set of states): N, S, T,
// M, DIR, D, KW, KR, B and FULL (the word's B vectors and their bits), RUN
// (steps per lane), UPAIR (bit j: slot j has a unit-capacity state), and
// per slot NU, NV (nodes), SIG (states), OFF (first probability entry), C1
// / CE1 / CE12 (bit k: state k has capacity >= 1 / exactly 1 / 1 or 2),
// WW1 / WU1 / WU12 (word slots: the word's vectors whose state has
// capacity >= 1 / exactly 1 / 1 or 2).  A sweep covers the vector indices [c_lo, c_hi): the
// words at its ends are masked.
struct MsBitsParams {
    u64 n_lane;        // lane runs swept: rl_base .. rl_base + n_lane - 1
    u64 rl_base;       // first lane run
    u64 c_lo, c_hi;    // vector indices swept: [c_lo, c_hi) (word slots least significant)
    u64 n_items;       // wavefront work items, 64 lane runs each
    const double *tb;  // [4][256]: TB_h[x] = sum over the bits i of x of Q_in(8h + i)
    const double *w;   // probability of (slot, state), at OFF[slot] + state
    double *part;      // [n_items][2] double-double partials
    u64 *pcount;       // [n_items]
    u64 *diag;         // [0]: the device clock at the start
};

// Reach from s, in the vectors of `src`, over the slots' masks W (slot E
// left out; -1: none): forward then backward sweeps in slot order until
// every lane's t word holds `need` (tested after each sweep) or a sweep
// pair adds nothing.
template <class G, int E>
__device__ __forceinline__ void ms_closure(const u32 (&W)[G::M], u32 src, u32 need, u32 (&r)[G::N])
{
#pragma unroll
    for (int v = 0; v < G::N; ++v) r[v] = 0u;
    r[G::S] = src;
    u32 before = 0u;
    for (;;) {
#pragma unroll
        for (int j = 0; j < G::M; ++j) {
            if (j == E) continue;
            r[G::NV[j]] = and_or(r[G::NU[j]], W[j], r[G::NV[j]]);
            if (!G::DIR) r[G::NU[j]] = and_or(r[G::NV[j]], W[j], r[G::NU[j]]);
        }
        // the slots run outward from s: a forward sweep often suffices
        if (__ballot((r[G::T] & need) != need) == 0ull) break;
#pragma unroll
        for (int j = G::M - 1; j >= 0; --j) {
            if (j == E) continue;
            r[G::NV[j]] = and_or(r[G::NU[j]], W[j], r[G::NV[j]]);
            if (!G::DIR) r[G::NU[j]] = and_or(r[G::NV[j]], W[j], r[G::NU[j]]);
        }
        if (__ballot((r[G::T] & need) != need) == 0ull) break;
        // reach only grows: an unchanged bit count is a fixed point
        u32 tot = 0u;
#pragma unroll
        for (int v = 0; v < G::N; ++v) tot += __popc(r[v]);
        if (__ballot(tot != before) == 0ull) break;
        before = tot;
    }
}

// Drop from V the vectors in which one arc (slot J onwards) whose state
// the masks U flag (capacity exactly 1 for demand 2; 1 or 2 for demand 3,
// CAP12) cuts s from t.  r0: the reach of the first closure; an arc whose
// tail s does not reach cannot cut.
template <class G, int J, bool CAP12>
struct MsCut {
    __device__ static __forceinline__ void run(const u32 (&W)[G::M], const u32 (&U)[G::M], const u32 (&r0)[G::N],
                                               u32 &V)
    {
        if constexpr (J < G::M) {
            if constexpr ((CAP12 ? G::CE12[J] : G::CE1[J]) != 0u) {
                const u32 need = V & U[J] & r0[G::NU[J]];
                if (__ballot(need != 0u) != 0ull) {
                    u32 r[G::N];
                    ms_closure<G, J>(W, need, need, r);
                    V &= ~need | r[G::T];
                }
            }
            MsCut<G, J + 1, CAP12>::run(W, U, r0, V);
        }
    }
};

// Demand 3: drop from V the vectors in which two arcs of capacity 1 cut s
// from t together.  Pairs of the slots that have a unit-capacity state,
// in uniform loops; ubits: the lane's unit-capacity flags of the run and
// lane slots (bit j), word slots by their constant patterns.  One closure
// serves every pair, on the arc masks with the pair's two cleared.
template <class G>
__device__ __forceinline__ void ms_cut_pairs(const u32 (&W)[G::M], u32 ubits, u32 &V)
{
    auto unit = [&](u32 j) -> u32 {
        return j < G::KW ? G::WU1[j] : (((ubits >> j) & 1u) ? ~0u : 0u);
    };
    for (u32 m1 = G::UPAIR; m1 != 0u; m1 &= m1 - 1u) {
        const u32 j1 = (u32)__builtin_ctz(m1);
        const u32 u1 = unit(j1);
        for (u32 m2 = m1 & (m1 - 1u); m2 != 0u; m2 &= m2 - 1u) {
            const u32 j2 = (u32)__builtin_ctz(m2);
            // (one of the two lies on the first closure's walk to t, but
            // not necessarily both: no reach filter here)
            const u32 need = V & u1 & unit(j2);
            if (__ballot(need != 0u) == 0ull) continue;
            u32 Wp[G::M];
#pragma unroll
            for (int j = 0; j < G::M; ++j) {
                Wp[j] = ((u32)j == j1 || (u32)j == j2) ? 0u : W[j];
                asm volatile("" : "+v"(Wp[j]));
            }
            u32 r[G::N];
            ms_closure<G, -1>(Wp, need, need, r);
            V &= ~need | r[G::T];
        }
    }
}

// One wavefront per work item: 64 lane runs of RUN words each.
template <class G>
__device__ void ms_bits_kernel(const MsBitsParams &P, double (&tb)[4][256])
{
    const u32 tid = threadIdx.x;
    if (blockIdx.x == 0 && tid == 0) P.diag[0] = wall_clock64();
    for (u32 i = tid; i < 1024u; i += blockDim.x) tb[i >> 8][i & 255u] = P.tb[i];
    __syncthreads();
    const u32 lane = tid & (kWave - 1);
    const u64 item = (u64)blockIdx.x * __builtin_amdgcn_readfirstlane(blockDim.x >> 6) +
                     __builtin_amdgcn_readfirstlane(tid >> 6);
    if (item >= P.n_items) return;
    // the lane slots' states are the digits of the lane's run index
    const u64 rl_rel = item * kWave + lane;
    const bool lane_live = rl_rel < P.n_lane;
    const u64 rl_abs = P.rl_base + rl_rel;
    u64 rl = rl_abs;
    u32 W[G::M], U[G::M], U2[G::M];
    u32 ubits_lane = 0u;  // lane slots with a unit-capacity state (bit j)
    double ql = 1.0;
#pragma unroll
    for (int j = 0; j < G::M; ++j) {
        if (j < G::KW) {
            W[j] = G::WW1[j];
            U[j] = G::WU1[j];
            U2[j] = G::WU12[j];
        } else if (j >= G::KW + G::KR) {
            const u32 x = (u32)(rl % G::SIG[j]);
            rl /= G::SIG[j];
            W[j] = ((G::C1[j] >> x) & 1u) ? ~0u : 0u;
            U[j] = ((G::CE1[j] >> x) & 1u) ? ~0u : 0u;
            U2[j] = ((G::CE12[j] >> x) & 1u) ? ~0u : 0u;
            ubits_lane |= ((G::CE1[j] >> x) & 1u) << j;
            // opaque masks: seen as selects, the relaxations would compile
            // to a select and an OR each instead of one AND-OR
            asm volatile("" : "+v"(W[j]));
            ql *= P.w[G::OFF[j] + x];
        } else {
            W[j] = U[j] = U2[j] = 0u;
        }
    }
    u32 xr[G::M];  // run slots' states (uniform); the others unused
#pragma unroll
    for (int j = 0; j < G::M; ++j) xr[j] = 0u;
    double acc_h = 0.0, acc_l = 0.0;
    u64 cnt = 0;
    for (u32 step = 0; step < G::RUN; ++step) {
        double q = ql;
        u32 ubits = ubits_lane;
#pragma unroll
        for (int j = G::KW; j < G::KW + G::KR; ++j) {
            W[j] = ((G::C1[j] >> xr[j]) & 1u) ? ~0u : 0u;
            U[j] = ((G::CE1[j] >> xr[j]) & 1u) ? ~0u : 0u;
            U2[j] = ((G::CE12[j] >> xr[j]) & 1u) ? ~0u : 0u;
            ubits |= ((G::CE1[j] >> xr[j]) & 1u) << j;
            asm volatile("" : "+v"(W[j]));
            q *= P.w[G::OFF[j] + xr[j]];
        }
        // the word's vectors c = (rl RUN + step) B + b inside [c_lo, c_hi)
        u32 full = 0u;
        if (lane_live) {
            const u64 c0 = (rl_abs * G::RUN + step) * (u64)G::B;
            const u64 lo = c0 >= P.c_lo ? 0ull : P.c_lo - c0;
            const u64 hi = c0 + G::B <= P.c_hi ? (u64)G::B : (P.c_hi > c0 ? P.c_hi - c0 : 0ull);
            if (hi > lo) full = G::FULL & (u32)((~0ull << lo) & ((hi >= 64ull ? 0ull : (1ull << hi)) - 1ull));
        }
        u32 r0[G::N];
        ms_closure<G, -1>(W, full, full, r0);
        u32 V = r0[G::T];
        if constexpr (G::D == 2) MsCut<G, 0, false>::run(W, U, r0, V);
        if constexpr (G::D == 3) {
            MsCut<G, 0, true>::run(W, U2, r0, V);
            ms_cut_pairs<G>(W, ubits, V);
        }
        cnt += (u64)__popc(V);
        if (__ballot(V != 0u) != 0ull) {
            const double F = ((tb[0][V & 255u] + tb[1][(V >> 8) & 255u]) + tb[2][(V >> 16) & 255u]) + tb[3][V >> 24];
            double s, e;
            two_sum(acc_h, q * F, s, e);
            acc_h = s;
            acc_l += e;
        }
        // next run state: the run slots count up, KW fastest
#pragma unroll
        for (int j = G::KW; j < G::KW + G::KR; ++j) {
            if (++xr[j] < G::SIG[j]) break;
            xr[j] = 0u;
        }
    }
    wave_sum_dd(acc_h, acc_l);
    const u64 c = wave_sum_u64(cnt);
    if (lane == 0) {
        P.part[2 * item] = acc_h;
        P.part[2 * item + 1] = acc_l;
        P.pcount[item] = c;
    }
}

}  // namespace bat

// bat_cube.hpp -- device code of the sub-cube sweep: whole sweeps of the
// 2^m state vectors in which a cube of vectors that all connect, or that
// all do not, is decided and added as one.
//
// Included by bat_cube.hip and, as text after bat_device.hpp, by the
// graph-specialised kernels compiled at run time; includes no header.
//
// The counter's M bits (the arcs on some s-t path, most often pivotal arc
// most significant) are split, for `levels` = 1 to 3, into
//     item | lane (up to 6 bits) | word of level levels-1 | ... | word 0
// with words of 5 bits.  A wavefront takes an item.  A lane holds one
// prefix; its word of level l > 0 stands for the 32 cubes that the 5 bits
// below the prefix make, each still free in the 5 l bits under it.  Reach
// only grows when an arc comes up, so two bit-sliced closures decide such a
// word: with every free arc down, the cubes connected for certain (S: added
// whole, 2^(5 l) vectors each); with every free arc up, those that can
// connect at all (P).  The cubes of P & ~S become prefixes of the next
// level: the wavefront queues them and takes 64 at a time, one per lane, so
// every lane works however unevenly the undecided cubes lie.  Word 0 has
// nothing free under it: one closure decides its 32 vectors.  Every vector
// thus gets the verdict the plain sweep gives it, from its own word 0 or
// from the cube that holds it.
//
// A closure removes the nodes other than s and t one by one: straight-line
// AND-ORs on the working masks of the arcs and of the node pairs a removed
// node joins (see bat_cube_plan.hpp), exact in one pass.
//
// What bounds it: the issue of those AND-ORs, and the scalar instructions
// that index their registers when the graph is read at run time.  The sums
// are per word: F(V) from the byte tables of the level (see bat_device.hpp),
// times the prefix's probability, a product of one table entry per level.

namespace bat {

constexpr int kCubeGroup = 5;                     // bits of a word
constexpr int kCubeLevels = 3;
constexpr int kCubeProgs = 2 * kCubeLevels - 1;   // closures: word 0, then (up, down) per level
constexpr int kCubeSlots = 64;                    // words of a closure (ahead-of-time kernels)
constexpr int kCubeSteps = 640;                   // steps of all closures, padded
constexpr int kCubeQueue = 1024;                  // prefixes queued at a time (a level can make 2048)
constexpr int kCubeWaves = 4;                     // wavefronts per block
constexpr int kCubeUnits = 64;                    // most units of work a block takes

struct alignas(16) double2_t {
    double x, y;
};

struct CubeProg {
    u32 first;    // its first step in step[]
    u32 octets;   // steps in groups of 8, padded
    u32 result;   // slot of the verdict; kCubeNever, kCubeAlways
    u32 word;     // counter bit of the word's first arc
};
constexpr u32 kCubeNever = 254u, kCubeAlways = 255u;

// Kernel argument (under 4 KiB): the plan travels with the launch, so a call
// makes no copy of it.
struct CubeParams {
    u64 n_items;              // work items of this launch
    u64 item_mul, item_mask;  // work item w is block item_base + ((w item_mul) & item_mask)
    u64 item_base;
    u32 m, M;                 // arcs, arcs enumerated (counter bits)
    u32 levels, lane_bits;
    u32 split;                // units an item is split into (see cube_share)
    u32 units;                // units per block (with gradients and chunked sweeps: chunks)
    u32 chunk;                // with gradients and chunked sweeps: units per chunk
    u32 fused;                // one block: it writes the results itself
    // partials: [blocks] double-doubles and counts; with gradients
    // [1 + 2 M][blocks] (R, then bit cb down and up)
    double2_t *part;
    u64 *pcount;
    u32 *done;                // with gradients: finished blocks of the reduction, whether p_dev is no probability
    const double *p_dev;      // [m] on the device, or null: p below
    // results: dd and count, or R (with the check of p_dev); null where not wanted
    double *res, *R;
    u64 *count;
    int *status;
    double *dRdp, *T1, *T0;   // [m] each
    u64 *diag;                // host, or null: [start, swept, done] device clocks and seq, written last
    u64 seq;
    CubeProg prog[kCubeProgs];
    unsigned char arc_of_bit[64];
    double p[kMaxArcs];
    // a | b << 8 | d << 16, slot d = a & b; bit 31: added to what d holds.
    // (read 16 bytes past the last step)
    u32 step[kCubeSteps + 4];
};

typedef const __attribute__((address_space(4))) CubeParams CubeArgs;

// FIRST: the lowest level whose words are summed by the byte tables
// (gradients have larger records for level 0).
template <u32 FIRST>
struct CubeTablesFrom {
    double tb[kCubeLevels - FIRST][256];  // per level: sums over bits 0..2 of the word's index
    double a4[kCubeLevels][4];    // bits 3..4
    double q5[kCubeLevels][32];   // all five
    double ql[kWave];             // lane bits
    double pr[64];                // working probability of the arc at counter bit cb
};
using CubeTables = CubeTablesFrom<0>;
using CubeSumTables = CubeTablesFrom<1>;
struct CubeWave {
    unsigned short queue[2][kCubeQueue];
    unsigned short from[kWave];  // level 1 prefixes (lane << 5 | word 2 index, or the lane) of the final rounds
    double qp[2][kWave];         // their probabilities
};

// x of another lane through the data-parallel primitives, where there is one
// in a bank of BANKS; else `old`.
template <int CTRL, int BANKS>
__device__ __forceinline__ double dpp_d(double old, double x)
{
    const u64 o = (u64)__double_as_longlong(old), b = (u64)__double_as_longlong(x);
    const u32 lo = (u32)__builtin_amdgcn_update_dpp((int)(u32)o, (int)(u32)b, CTRL, 0xf, BANKS, false);
    const u32 hi = (u32)__builtin_amdgcn_update_dpp((int)(u32)(o >> 32), (int)(u32)(b >> 32), CTRL, 0xf, BANKS, false);
    return __longlong_as_double((long long)((u64)hi << 32 | lo));
}

// Lanes with bit BIT of their number clear keep a and get the a of the lane
// with that bit set, as b; the others keep b (as b) and get that lane's b.
template <int BIT>
__device__ __forceinline__ void exchange(double &a, double &b)
{
#if defined(__HIP_DEVICE_COMPILE__) || defined(__HIPCC_RTC__)
    const u64 x = (u64)__double_as_longlong(a), y = (u64)__double_as_longlong(b);
    if constexpr (BIT >= 4) {
        const auto lo = BIT == 5 ? __builtin_amdgcn_permlane32_swap((u32)x, (u32)y, false, false)
                                 : __builtin_amdgcn_permlane16_swap((u32)x, (u32)y, false, false);
        const auto hi = BIT == 5 ? __builtin_amdgcn_permlane32_swap((u32)(x >> 32), (u32)(y >> 32), false, false)
                                 : __builtin_amdgcn_permlane16_swap((u32)(x >> 32), (u32)(y >> 32), false, false);
        a = __longlong_as_double((long long)((u64)hi[0] << 32 | lo[0]));
        b = __longlong_as_double((long long)((u64)hi[1] << 32 | lo[1]));
    } else if constexpr (BIT == 3) {  // 8 lanes on in the row, either way round
        const double k = dpp_d<0x128, 0xc>(a, b);
        b = dpp_d<0x128, 0x3>(b, a);
        a = k;
    } else if constexpr (BIT == 2) {  // 4 lanes down, 4 lanes up
        const double k = dpp_d<0x114, 0xa>(a, b);
        b = dpp_d<0x104, 0x5>(b, a);
        a = k;
    } else {  // within 4 lanes
        const bool up = (threadIdx.x >> BIT) & 1u;
        const double send = up ? a : b, keep = up ? b : a;
        a = keep;
        b = BIT == 1 ? dpp_d<0x4e, 0xf>(send, send) : dpp_d<0xb1, 0xf>(send, send);
    }
#else
    (void)a, (void)b;  // hipcc's host pass, which parses this and has no such builtins
#endif
}

// The sums over the 64 lanes of N columns (double-doubles h + l): two at a
// time change places so that each half of the lanes adds up one of them,
// then quarters, down to a column per lane: N + 1 additions or so in all,
// where a fold of each column by itself takes 6 N.  Columns below LOW have no
// low parts yet.  wave_column gives the column whose sum a lane ends up with,
// in h[0] and l[0], or N.
template <int N, int LOW, int BIT = 5, int K>
__device__ __forceinline__ void wave_fold(double (&h)[K], double (&l)[K])
{
    constexpr int H = (N + 1) / 2;
#pragma unroll
    for (int i = 0; i < H; ++i) {
        double a = h[i], b = i + H < N ? h[i + H] : 0.0, e;
        exchange<BIT>(a, b);
        two_sum(a, b, h[i], e);
        if (i >= LOW || i + H >= LOW) {
            double c = l[i], d = i + H < N ? l[i + H] : 0.0;
            exchange<BIT>(c, d);
            e += c + d;
        }
        l[i] = e;
    }
    if constexpr (BIT > 0) wave_fold<H, 0, BIT - 1>(h, l);
}
template <int N, int BIT = 5>
__device__ __forceinline__ u32 wave_column(u32 lane)
{
    constexpr u32 H = (N + 1) / 2;
    u32 i = 0u;
    if constexpr (BIT > 0) i = wave_column<(int)H, BIT - 1>(lane);
    i = i < H ? i + ((lane >> BIT) & 1u) * H : (u32)N;
    return i < (u32)N ? i : (u32)N;
}

// LDS written by some lanes of a wavefront and read by others: the LDS
// operations of one wavefront complete in order, so only the compiler must
// keep them so.
__device__ __forceinline__ void wave_lds_sync()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

template <u32 FIRST>
__device__ __forceinline__ double cube_q(const CubeTablesFrom<FIRST> &T, u32 M, u32 cb, u32 x)
{
    if (cb >= M) return x ? 0.0 : 1.0;  // a bit past the last arc: never set
    const double p = T.pr[cb];
    return x ? p : 1.0 - p;
}

// h + l times f.  The gradients' tables of products round them once, not at
// each factor: an error that T1 and T0 do not share stays in their difference.
__device__ __forceinline__ void dd_mul(double &h, double &l, double f)
{
    const double p = h * f;
    l = __builtin_fma(l, f, __builtin_fma(h, f, -p));
    h = p;
}

__device__ __forceinline__ double cube_p(CubeArgs *P, u32 a) { return P->p_dev ? P->p_dev[a] : P->p[a]; }
__device__ __forceinline__ const __attribute__((address_space(4))) u32 *cube_steps(CubeArgs *P) { return P->step; }

// The vectors of word [base, base + 32) that the launch asks for.
__device__ __forceinline__ u32 cube_window(CubeArgs *, u32) { return ~0u; }

// The block's probability tables (all threads).
template <class Args, u32 FIRST>
__device__ __forceinline__ void cube_tables(Args *P, CubeTablesFrom<FIRST> &T)
{
    const u32 tid = threadIdx.x, nt = blockDim.x, M = P->M, levels = P->levels;
    if (tid < M) T.pr[tid] = cube_p(P, P->arc_of_bit[tid]);
    __syncthreads();
    for (u32 i = tid; i + FIRST * 256u < levels * 256u; i += nt) {
        const u32 l = FIRST + (i >> 8), y = i & 255u, c0 = kCubeGroup * l;
        double b[2][3];
#pragma unroll
        for (u32 k = 0; k < 3; ++k) {
            b[0][k] = cube_q(T, M, c0 + k, 0u);
            b[1][k] = cube_q(T, M, c0 + k, 1u);
        }
        double s = 0.0;
#pragma unroll
        for (u32 k = 0; k < 8; ++k) s += ((y >> k) & 1u) ? b[k & 1u][0] * b[(k >> 1) & 1u][1] * b[k >> 2][2] : 0.0;
        T.tb[l - FIRST][y] = s;
    }
    for (u32 i = tid; i < levels * 32u; i += nt) {
        const u32 l = i >> 5, j = i & 31u;
        const double hi = cube_q(T, M, kCubeGroup * l + 3, (j >> 3) & 1u) * cube_q(T, M, kCubeGroup * l + 4, j >> 4);
        double q = 1.0;
        for (u32 k = 0; k < 3; ++k) q *= cube_q(T, M, kCubeGroup * l + k, (j >> k) & 1u);
        T.q5[l][j] = q * hi;
        if ((j & 7u) == 0u) T.a4[l][j >> 3] = hi;
    }
    if (tid < (u32)kWave) {
        double q = 1.0, e = 0.0;
        for (u32 b = 0; b < P->lane_bits; ++b) {
            const double f = cube_q(T, M, kCubeGroup * levels + b, (tid >> b) & 1u);
            if constexpr (FIRST == 0) q *= f;
            else dd_mul(q, e, f);
        }
        T.ql[tid] = q + e;
    }
    __syncthreads();
}

// Number of set bits of x in the lanes below this one, and in all lanes.
__device__ __forceinline__ u32 wave_excl_popc(u32 x, u32 &total)
{
    const u32 c = (u32)__popc(x);
    u32 e = 0u, t = 0u;
#pragma unroll
    for (u32 b = 0; b < 6; ++b) {
        const u64 m = __ballot((c >> b) & 1u);
        e += __builtin_amdgcn_mbcnt_hi((u32)(m >> 32), __builtin_amdgcn_mbcnt_lo((u32)m, 0u)) << b;
        t += (u32)__popcll(m) << b;
    }
    total = t;
    return e;
}

// The rounds of 64 prefixes a unit takes of its item's `total`: every
// split-th from its own, or all of a few rounds for unit 0 and none for the
// others, which end there (long items are what a launch waits for at its
// end; short ones are not worth sharing).
constexpr u32 kCubeShare = 2;
__device__ __forceinline__ bool cube_share(u32 total, u32 sub, u32 split, u32 &first, u32 &step)
{
    const bool few = total <= kCubeShare * (u32)kWave;
    first = few ? 0u : sub;
    step = few ? 1u : split;
    return total != 0u && (!few || sub == 0u);
}

// Entries [w0, w0 + QUEUE) of the wavefront's set bits, in lane order:
// lane << 5 | bit.  e: set bits in the lanes below.
template <u32 QUEUE>
__device__ __forceinline__ void cube_enqueue(unsigned short *q, u32 U, u32 e, u32 w0, u32 lane)
{
    u32 pos = e - w0;
    while (__ballot(U != 0u) != 0ull) {
        if (U) {
            if (pos < QUEUE) q[pos] = (unsigned short)(lane << 5 | (u32)__builtin_ctz(U));
            ++pos;
            U &= U - 1u;
        }
    }
    wave_lds_sync();
}

// Graph read at run time, at most 32 counter bits: the words live in v64 to
// v127 and the steps, read with scalar loads (four each, the next four ahead
// of use), name them through the VGPR-index mode.  Hand-written because
// compiled code leaves and enters that mode around each access: 9
// instructions per step here against about 17.
#define BAT_CUBE_STEP(w)                      \
    "s_set_gpr_idx_on " w ", 0x1\n\t"         \
    "v_mov_b32 %[x], v64\n\t"                 \
    "s_lshr_b32 s72, " w ", 8\n\t"            \
    "s_set_gpr_idx_on s72, 0x1\n\t"           \
    "v_and_b32 %[x], v64, %[x]\n\t"           \
    "s_lshr_b32 s72, " w ", 16\n\t"           \
    "s_ashr_i32 s73, " w ", 31\n\t"           \
    "s_set_gpr_idx_on s72, 0x9\n\t"           \
    "v_and_or_b32 v64, v64, s73, %[x]\n\t"
#define BAT_CUBE_MASK(v, cb) "v_bfe_i32 " v ", %[c], " cb ", 1\n\t"

template <class Args>
struct CubeDyn {
    static constexpr bool kChunked = false;
    Args *P;
    u32 base;  // the item's counter bits

    __device__ __forceinline__ u32 levels() const { return P->levels; }
    __device__ __forceinline__ u32 lane_bits() const { return P->lane_bits; }
    __device__ __forceinline__ u32 arcs() const { return P->M; }
    __device__ __forceinline__ void item(u64 block) { base = (u32)(block << (kCubeGroup * P->levels + P->lane_bits)); }

    // rel: the prefix's counter bits within the item
    __device__ __forceinline__ u32 close(u32 pi, u32 rel, bool live) const
    {
        // free arcs' bits: set when up, as a digraph's closures use them
        const u32 c = base | rel | ((pi & 1u) ? (1u << (kCubeGroup * ((pi + 1u) >> 1))) - 1u : 0u);
        const u32 result = P->prog[pi].result;
        if (result >= (u32)kCubeSlots) return live && result == kCubeAlways ? ~0u : 0u;
        const __attribute__((address_space(4))) u32 *steps = cube_steps(P);
        u32 off = P->prog[pi].first * 4u, n = P->prog[pi].octets, x, out;
        asm volatile(
            "s_mov_b32 s74, m0\n\t"
            "s_load_dwordx4 s[64:67], %[p], %[o]\n\t"
            BAT_CUBE_MASK("v64", "0") BAT_CUBE_MASK("v65", "1") BAT_CUBE_MASK("v66", "2") BAT_CUBE_MASK("v67", "3")
            BAT_CUBE_MASK("v68", "4") BAT_CUBE_MASK("v69", "5") BAT_CUBE_MASK("v70", "6") BAT_CUBE_MASK("v71", "7")
            BAT_CUBE_MASK("v72", "8") BAT_CUBE_MASK("v73", "9") BAT_CUBE_MASK("v74", "10") BAT_CUBE_MASK("v75", "11")
            BAT_CUBE_MASK("v76", "12") BAT_CUBE_MASK("v77", "13") BAT_CUBE_MASK("v78", "14") BAT_CUBE_MASK("v79", "15")
            BAT_CUBE_MASK("v80", "16") BAT_CUBE_MASK("v81", "17") BAT_CUBE_MASK("v82", "18") BAT_CUBE_MASK("v83", "19")
            BAT_CUBE_MASK("v84", "20") BAT_CUBE_MASK("v85", "21") BAT_CUBE_MASK("v86", "22") BAT_CUBE_MASK("v87", "23")
            BAT_CUBE_MASK("v88", "24") BAT_CUBE_MASK("v89", "25") BAT_CUBE_MASK("v90", "26") BAT_CUBE_MASK("v91", "27")
            BAT_CUBE_MASK("v92", "28") BAT_CUBE_MASK("v93", "29") BAT_CUBE_MASK("v94", "30") BAT_CUBE_MASK("v95", "31")
            "s_set_gpr_idx_on %[w], 0x8\n\t"
            "v_mov_b32 v64, 0xaaaaaaaa\n\t"
            "v_mov_b32 v65, 0xcccccccc\n\t"
            "v_mov_b32 v66, 0xf0f0f0f0\n\t"
            "v_mov_b32 v67, 0xff00ff00\n\t"
            "v_mov_b32 v68, 0xffff0000\n\t"
            "s_waitcnt lgkmcnt(0)\n"
            "1:\n\t"
            "s_load_dwordx4 s[68:71], %[p], %[o] offset:0x10\n\t"
            BAT_CUBE_STEP("s64") BAT_CUBE_STEP("s65") BAT_CUBE_STEP("s66") BAT_CUBE_STEP("s67")
            "s_waitcnt lgkmcnt(0)\n\t"
            "s_load_dwordx4 s[64:67], %[p], %[o] offset:0x20\n\t"
            BAT_CUBE_STEP("s68") BAT_CUBE_STEP("s69") BAT_CUBE_STEP("s70") BAT_CUBE_STEP("s71")
            "s_add_u32 %[o], %[o], 32\n\t"
            "s_sub_u32 %[n], %[n], 1\n\t"
            "s_cmp_lg_u32 %[n], 0\n\t"
            "s_waitcnt lgkmcnt(0)\n\t"
            "s_cbranch_scc1 1b\n\t"
            "s_set_gpr_idx_on %[r], 0x1\n\t"
            "v_mov_b32 %[out], v64\n\t"
            "s_set_gpr_idx_off\n\t"
            "s_mov_b32 m0, s74"
            : [o] "+s"(off), [n] "+s"(n), [x] "=&v"(x), [out] "=&v"(out)
            : [p] "s"(steps), [c] "v"(c), [w] "s"(P->prog[pi].word), [r] "s"(result)
            : "scc", "memory", "s64", "s65", "s66", "s67", "s68", "s69", "s70", "s71", "s72", "s73", "s74", "v64", "v65",
              "v66", "v67", "v68", "v69", "v70", "v71", "v72", "v73", "v74", "v75", "v76", "v77", "v78", "v79", "v80",
              "v81", "v82", "v83", "v84", "v85", "v86", "v87", "v88", "v89", "v90", "v91", "v92", "v93", "v94", "v95",
              "v96", "v97", "v98", "v99", "v100", "v101", "v102", "v103", "v104", "v105", "v106", "v107", "v108",
              "v109", "v110", "v111", "v112", "v113", "v114", "v115", "v116", "v117", "v118", "v119", "v120", "v121",
              "v122", "v123", "v124", "v125", "v126", "v127");
        return live ? out : 0u;
    }
};
#undef BAT_CUBE_STEP
#undef BAT_CUBE_MASK

// Graph known at compile time (hiprtc): G holds the plan's sizes and, as
// G::run<k>(r), the steps of closure k on an array that becomes registers.
// The masks of the item's arcs are uniform and stay scalar.
template <class G>
struct CubeStatic {
    static constexpr bool kChunked = G::CHUNKED;
    u32 um[G::M > G::REL ? G::M - G::REL : 1];  // masks of the item's arcs

    __device__ __forceinline__ u32 levels() const { return G::LEVELS; }
    __device__ __forceinline__ u32 lane_bits() const { return G::LANE_BITS; }
    __device__ __forceinline__ u32 arcs() const { return G::M; }
    __device__ __forceinline__ void item(u64 block)
    {
        const u32 b[2] = {(u32)__builtin_amdgcn_readfirstlane((u32)block),
                          (u32)__builtin_amdgcn_readfirstlane((u32)(block >> 32))};
#pragma unroll
        for (int k = 0; k < G::M - G::REL; ++k) {
            um[k] = 0u - ((b[k >> 5] >> (k & 31)) & 1u);
            // opaque: a mask seen as all or nothing would turn each AND-OR
            // into a select and an OR
            asm volatile("" : "+s"(um[k]));
        }
    }

    template <u32 K>
    __device__ __forceinline__ u32 run(u32 rel, bool live) const
    {
        constexpr int word = kCubeGroup * (int)((K + 1u) / 2u);
        if constexpr (K >= 2u * G::LEVELS - 1u || G::RESULT[K] == kCubeNever) {
            return 0u;
        } else if constexpr (G::RESULT[K] == kCubeAlways) {
            return live ? ~0u : 0u;
        } else {
            u32 r[G::SLOTS];
#pragma unroll
            for (int c = 0; c < G::M; ++c) {
                if (c < word) r[c] = (K & 1u) ? ~0u : 0u;
                else if (c < word + kCubeGroup) r[c] = slice_pattern(c - word);
                else if (c < G::REL) {
                    r[c] = (u32)__builtin_amdgcn_sbfe((int)rel, c, 1);
                    asm volatile("" : "+v"(r[c]));
                } else r[c] = um[c - G::REL];
            }
            G::template steps<K>(r);
            return live ? r[G::RESULT[K]] : 0u;
        }
    }

    __device__ __forceinline__ u32 close(u32 pi, u32 rel, bool live) const
    {
        return pi == 0u   ? run<0>(rel, live)
               : pi == 1u ? run<1>(rel, live)
               : pi == 2u ? run<2>(rel, live)
               : pi == 3u ? run<3>(rel, live)
                          : run<4>(rel, live);
    }
};

// One wavefront's share of the sweep.
template <class Clo, class Args = CubeArgs>
struct CubeSweep {
    Args *P;
    const CubeTables &T;
    CubeWave &W;
    Clo clo;
    u32 lane;
    double hi, lo;     // sum of the probabilities
    u64 cnt;

    __device__ __forceinline__ void add(u32 level, double q, u32 V)
    {
        cnt += (u64)__popc(V) << (kCubeGroup * level);
        if (__ballot(V != 0u) == 0ull) return;
        const double *tb = T.tb[level], *a4 = T.a4[level];
        double F = a4[0] * tb[V & 255u];
        F = __builtin_fma(a4[1], tb[(V >> 8) & 255u], F);
        F = __builtin_fma(a4[2], tb[(V >> 16) & 255u], F);
        F = __builtin_fma(a4[3], tb[V >> 24], F);
        double s, e;
        two_sum(hi, q * F, s, e);
        hi = s;
        lo += e;
    }

    // The cubes of the prefix's word: added where they connect for certain
    // (when `mine`), returned where they are undecided.
    __device__ __forceinline__ u32 classify(u32 level, u32 rel, double q, bool live, bool mine)
    {
        const u32 up = clo.close(2u * level - 1u, rel, live);
        if (__ballot(up != 0u) == 0ull) return 0u;
        const u32 down = clo.close(2u * level, rel, live && up != 0u);
        if (mine) add(level, q, down);
        return up & ~down;
    }

    // The vectors under the undecided cubes U of level 1 prefixes (one per
    // lane: `from`, probability q), the share of unit `sub` of `split`.
    __device__ __forceinline__ void finals(u32 U, u32 from, double q, u32 sub, u32 split)
    {
        u32 total, step, round;
        const u32 e = wave_excl_popc(U, total);
        if (!cube_share(total, sub, split, round, step)) return;
        W.from[lane] = (unsigned short)from;
        W.qp[1][lane] = q;
        for (u32 w0 = 0; w0 < total; w0 += kCubeQueue) {
            cube_enqueue<kCubeQueue>(W.queue[1], U, e, w0, lane);
            const u32 end = min(total, w0 + (u32)kCubeQueue);
            for (; (u32)kWave * round < end; round += step) {
                const u32 i = (u32)kWave * round + lane;
                const bool live = i < end;
                const u32 x = W.queue[1][(live ? i : end - 1u) - w0], own = x >> 5;
                const u32 rel = (u32)W.from[own] << (2 * kCubeGroup) | (x & 31u) << kCubeGroup;
                const u32 V = clo.close(0u, rel, live);
                add(0u, W.qp[1][own] * T.q5[1][x & 31u], V);
            }
            wave_lds_sync();
        }
    }

    __device__ __forceinline__ void item(u64 block, u32 sub)
    {
        const u32 levels = clo.levels(), lane_bits = clo.lane_bits(), split = P->split, M = clo.arcs();
        const u32 rb = kCubeGroup * levels + lane_bits;
        clo.item(block);
        const bool live = (lane >> lane_bits) == 0u;
        // the item's probability: one factor per lane, multiplied across
        double q = lane + rb < M ? cube_q(T, M, rb + lane, (u32)(block >> lane) & 1u) : 1.0;
#pragma unroll
        for (int off = kWave / 2; off >= 1; off >>= 1) q *= shfl_xor_d(q, off);
        q *= T.ql[lane];
        if (levels == 1u) {
            u32 V = clo.close(0u, lane << kCubeGroup, live);
            if (M < 5u) V &= (1u << (1u << M)) - 1u;  // bits past the last arc
            add(0u, q, V & cube_window(P, ((u32)block << rb) | lane << kCubeGroup));
            return;
        }
        const u32 U = classify(levels - 1u, lane << (kCubeGroup * levels), q, live, sub == 0u);
        if (levels == 2u) {
            finals(U, lane, q, sub, split);
            return;
        }
        u32 total, step, round;
        const u32 e = wave_excl_popc(U, total);
        if (!cube_share(total, sub, split, round, step)) return;
        W.qp[0][lane] = q;
        for (u32 w0 = 0; w0 < total; w0 += kCubeQueue) {
            cube_enqueue<kCubeQueue>(W.queue[0], U, e, w0, lane);
            const u32 end = min(total, w0 + (u32)kCubeQueue);
            for (; (u32)kWave * round < end; round += step) {
                const u32 i = (u32)kWave * round + lane;
                const bool on = i < end;
                const u32 x = W.queue[0][(on ? i : end - 1u) - w0];
                const double q1 = W.qp[0][x >> 5] * T.q5[2][x & 31u];
                const u32 U1 = classify(1u, x << (2 * kCubeGroup), q1, on, true);
                finals(U1, x, q1, 0u, 1u);
            }
            wave_lds_sync();
        }
    }
};

__device__ __forceinline__ void cube_clock(CubeArgs *P, u32 k)
{
    if (P->diag) P->diag[k] = wall_clock64();
}

// 0, or -1 when a p on the device is no probability.  (By the one thread that
// then writes the outputs, which may lie where p does.)
__device__ __forceinline__ int cube_status(CubeArgs *P)
{
    int st = 0;
    if (P->p_dev)
        for (u32 i = 0; i < P->m; ++i)
            if (!(P->p_dev[i] >= 0.0 && P->p_dev[i] <= 1.0)) st = -1;
    return st;
}

// R and the count from the sums (one thread): as a double-double and the
// count, or as R and the count with the status (NaN and -1).
__device__ __forceinline__ void cube_store(CubeArgs *P, double hi, double lo, u64 cnt, int st)
{
    if (P->res) {
        P->res[0] = hi;
        P->res[1] = lo;
    }
    if (P->R) *P->R = st ? __builtin_nan("") : hi + lo;
    if (P->count) *P->count = st ? 0ull : cnt << (P->m - P->M);
    if (P->status) *P->status = st;
}

// The sequence number goes last: a host that sees it sees the results too,
// so a synchronous call need not wait for the stream.
__device__ __forceinline__ void cube_publish(CubeArgs *P)
{
    cube_clock(P, 2);
    if (P->diag) __hip_atomic_store(P->diag + 3, P->seq, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_SYSTEM);
}

__device__ __forceinline__ void cube_results(CubeArgs *P, double hi, double lo, u64 cnt)
{
    cube_store(P, hi, lo, cnt, cube_status(P));
    cube_publish(P);
}

// A block takes `units` consecutive units; its wavefronts take the next one
// from the block's own counter, so that one wavefront's long unit does not
// leave the others waiting at the end (units differ widely: with a fixed
// unit per wavefront 70% of the resident wavefront cycles of the 5x5 grid
// were spent waiting, and it took 17.9 ms against 12.0 ms with 32 units per
// block; later 8.65 ms with 32, 7.9 ms with 64, 8.6 ms with 128, whose
// blocks are too few for an even end; 8 and 16 wavefronts per block: 8.7
// and 9.7 ms).  Each unit's sum has its own place and they
// are added in unit order, whichever wavefront formed them.  Past 2^23 work
// items a place takes the sum of a chunk of consecutive units, so that
// neither the blocks (HIP launches fewer than 2^32 threads) nor their
// partials grow with the sweep.
template <class Clo>
__device__ __forceinline__ void cube_kernel(CubeArgs *P, CubeTables &T, CubeWave *Ws, Clo clo)
{
    __shared__ double2_t su[kCubeUnits];
    __shared__ u64 sc[kCubeUnits];
    __shared__ u32 next;
    if (blockIdx.x == 0 && threadIdx.x == 0) cube_clock(P, 0);
    if (threadIdx.x == 0) next = 0u;
    cube_tables(P, T);
    const u32 lane = threadIdx.x & (kWave - 1);
    const u32 wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const u32 split = P->split, units = P->units;
    const u64 first = (u64)blockIdx.x * units, all = P->n_items * split;
    for (;;) {
        // Every lane adds 1 (compiled to one add of 64): under an "if lane 0"
        // the compiler joined this branch to the one that ends the loop
        // body, sent the other lanes round the loop past the atomic and
        // never ended it.
        __builtin_amdgcn_wave_barrier();
        const u32 k = __builtin_amdgcn_readfirstlane(atomicAdd(&next, 1u)) / kWave;
        if (k >= units) break;
        CubeSweep<Clo> S{P, T, Ws[wave], clo, lane, 0.0, 0.0, 0ull};
        if constexpr (Clo::kChunked) {
            const u64 c0 = (first + k) * P->chunk, c1 = min(all, c0 + P->chunk);
            for (u64 w = c0; w < c1; ++w)
                S.item(P->item_base + ((w / split * P->item_mul) & P->item_mask), (u32)(w % split));
        } else {
            const u64 w = first + k, it = w / split;
            if (w < all) S.item(P->item_base + ((it * P->item_mul) & P->item_mask), (u32)(w % split));
        }
        wave_sum_dd(S.hi, S.lo);
        const u64 c = wave_sum_u64(S.cnt);
        if (lane == 0) {
            su[k] = {S.hi, S.lo};
            sc[k] = c;
        }
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        double h = 0.0, l = 0.0;
        u64 n = 0;
        for (u32 k = 0; k < units; ++k) {
            dd_add(h, l, su[k].x, su[k].y);
            n += sc[k];
        }
        if (P->fused) {
            cube_clock(P, 1);
            cube_results(P, h, l, n);
        } else {
            P->part[blockIdx.x] = {h, l};
            P->pcount[blockIdx.x] = n;
        }
    }
}

// ------------------------------------------------------------- gradients
// The same sweep with T1_i and T0_i of every arc.  Each decided word adds to
// the arcs of its own bits, by the tables with one bit left out, and a cube
// that connects whole also to the arcs free in it (its whole sum, for either
// state).  What lies under a prefix goes up once: the sums of a round's
// lanes are added per prefix of the level above (a segmented sum, as the
// lanes lie in prefix order), so an arc above a word costs once per prefix,
// not once per word under it.  A wavefront takes chunks of consecutive units
// from the block's counter and folds its columns after each chunk (unless
// nothing connected) into the chunk's own place in LDS, which the block adds
// up in order, so that no sum depends on timing.  (Every n-th unit to a
// wavefront and one fold each left the longest one running: 36 arcs, 3.5
// ms.)  Nothing is divided by a probability: 0 and 1 are exact.
//
// What bounds it: besides the closures, the 64-byte records of the words'
// bytes (16 LDS reads of 16 bytes per 64 words).

struct CubeGradTables {
    alignas(16) double tbx[256 * 8];  // word 0, per byte value: TB, then TB without bit a = 0..2 of state x = 0, 1
    double a4m[8];                    // word 0: A without bit 3, without bit 4
    double q5m[kCubeLevels - 1][5][32];  // words 1, 2: their probability without arc a
};

__device__ __forceinline__ void cube_grad_tables(CubeArgs *P, const CubeSumTables &T, CubeGradTables &X)
{
    const u32 tid = threadIdx.x, nt = blockDim.x, M = P->M;
    for (u32 y = tid; y < 256u; y += nt) {
        double s = 0.0, sg[6] = {0.0, 0.0, 0.0, 0.0, 0.0, 0.0}, b[2][3];
#pragma unroll
        for (u32 k = 0; k < 3; ++k) {
            b[0][k] = cube_q(T, M, k, 0u);
            b[1][k] = cube_q(T, M, k, 1u);
        }
#pragma unroll
        for (u32 i = 0; i < 8; ++i) {
            const double on = (y >> i) & 1u ? 1.0 : 0.0;
            const double q0 = b[i & 1u][0], q1 = b[(i >> 1) & 1u][1], q2 = b[i >> 2][2];
            s += on * q0 * q1 * q2;
            sg[i & 1u] += on * q1 * q2;
            sg[2 + ((i >> 1) & 1u)] += on * q0 * q2;
            sg[4 + (i >> 2)] += on * q0 * q1;
        }
        X.tbx[8 * y] = s;
#pragma unroll
        for (u32 k = 0; k < 6; ++k) X.tbx[8 * y + 1 + k] = sg[k];
        X.tbx[8 * y + 7] = 0.0;
    }
    if (tid < 4u) {
        X.a4m[tid] = cube_q(T, M, 4, tid >> 1);
        X.a4m[4 + tid] = cube_q(T, M, 3, tid & 1u);
    }
    for (u32 i = tid; i < (P->levels - 1u) * 160u; i += nt) {
        const u32 l = i / 160u, a = (i % 160u) >> 5, j = i & 31u;
        double q = 1.0, e = 0.0;
        for (u32 b = 0; b < 5u; ++b)
            if (b != a) dd_mul(q, e, cube_q(T, M, kCubeGroup * (l + 1u) + b, (j >> b) & 1u));
        X.q5m[l][a][j] = q + e;
    }
    __syncthreads();
}

constexpr int kGradQueue = kCubeQueue / 2;
struct CubeGradWave {
    unsigned short queue[kCubeLevels - 1][kGradQueue];
    unsigned short from[kWave];
    // of the prefixes above words 0 and 1: probabilities, the sums under them
    double qp[kCubeLevels - 1][kWave];
    double val[kCubeLevels - 1][kWave];
};

template <class Clo>
struct CubeGradSweep {
    CubeArgs *P;
    const CubeSumTables &T;
    const CubeGradTables &X;
    CubeGradWave &W;
    Clo clo;
    u32 lane;
    double hi, lo;            // R
    u64 cnt;
    double g0[3][2], tb0[4];  // word 0: bits 0..2 by state; per byte for bits 3, 4
    double g1[5][2], g2[5][2];  // words 1, 2
    double free1, free2;      // cubes that connect whole, of words 1 and 2
    double lane_hi, lane_lo;  // all under the lane's prefix, without the lane bits' probability
    double sh[2], sl[2];      // item bit `lane`, by state

    __device__ __forceinline__ void zero()
    {
        hi = lo = free1 = free2 = 0.0;
        cnt = 0;
#pragma unroll
        for (int a = 0; a < 3; ++a) g0[a][0] = g0[a][1] = 0.0;
#pragma unroll
        for (int h = 0; h < 4; ++h) tb0[h] = 0.0;
#pragma unroll
        for (int a = 0; a < 5; ++a) g1[a][0] = g1[a][1] = g2[a][0] = g2[a][1] = 0.0;
        lane_hi = lane_lo = sh[0] = sh[1] = sl[0] = sl[1] = 0.0;
    }

    __device__ __forceinline__ void addR(double x)
    {
        double s, e;
        two_sum(hi, x, s, e);
        hi = s;
        lo += e;
    }

    // A final word under a prefix of probability q: R, the count and word
    // 0's arcs; returns F(V).
    __device__ __forceinline__ double word0(double q, u32 V)
    {
        cnt += (u64)__popc(V);
        double F = 0.0, sg[6] = {0.0, 0.0, 0.0, 0.0, 0.0, 0.0};
#pragma unroll
        for (int h = 0; h < 4; ++h) {
            const Pair *rp = reinterpret_cast<const Pair *>(X.tbx + ((V >> (8 * h)) & 255u) * 8u);
            const Pair v0 = rp[0], v1 = rp[1], v2 = rp[2], v3 = rp[3];
            const double ah = T.a4[0][h];
            tb0[h] = __builtin_fma(q, v0.x, tb0[h]);
            F = __builtin_fma(ah, v0.x, F);
            sg[0] = __builtin_fma(ah, v0.y, sg[0]);
            sg[1] = __builtin_fma(ah, v1.x, sg[1]);
            sg[2] = __builtin_fma(ah, v1.y, sg[2]);
            sg[3] = __builtin_fma(ah, v2.x, sg[3]);
            sg[4] = __builtin_fma(ah, v2.y, sg[4]);
            sg[5] = __builtin_fma(ah, v3.x, sg[5]);
        }
#pragma unroll
        for (int a = 0; a < 3; ++a) {
            g0[a][0] = __builtin_fma(q, sg[2 * a], g0[a][0]);
            g0[a][1] = __builtin_fma(q, sg[2 * a + 1], g0[a][1]);
        }
        addR(q * F);
        return F;
    }

    __device__ __forceinline__ double word_sum(u32 level, u32 V) const
    {
        const double *tb = T.tb[level - 1u], *a4 = T.a4[level];
        double F = a4[0] * tb[V & 255u];
        F = __builtin_fma(a4[1], tb[(V >> 8) & 255u], F);
        F = __builtin_fma(a4[2], tb[(V >> 16) & 255u], F);
        return __builtin_fma(a4[3], tb[V >> 24], F);
    }

    // The cubes S of a word of level 1 or 2 that connect whole: R, the count
    // and the word's arcs g.  An arc's state x left out of the sum is the
    // sum of the cubes of state x taken for both (its two probabilities add
    // to 1).
    __device__ __forceinline__ double cubes(u32 level, double q, u32 S, double (&g)[5][2], double &all)
    {
        cnt += (u64)__popc(S) << (kCubeGroup * level);
        if (__ballot(S != 0u) == 0ull) return 0.0;
#pragma unroll
        for (int a = 0; a < 5; ++a) {
            const u32 pat = slice_pattern(a), s1 = S & pat, s0 = S & ~pat;
            g[a][1] = __builtin_fma(q, word_sum(level, s1 | s1 >> (1 << a)), g[a][1]);
            g[a][0] = __builtin_fma(q, word_sum(level, s0 | s0 << (1 << a)), g[a][0]);
        }
        const double F = word_sum(level, S);
        all = __builtin_fma(q, F, all);
        addR(q * F);
        return F;
    }

    // The sum v under cube j of a word of level 1 or 2 (q: the probability
    // above the word): its arcs g.
    __device__ __forceinline__ void under(u32 level, double q, u32 j, double v, double (&g)[5][2])
    {
        const double qv = q * v;
#pragma unroll
        for (int a = 0; a < 5; ++a) {
            const double w = X.q5m[level - 1u][a][j] * qv;
            const double up = (j >> a) & 1u ? 1.0 : 0.0, down = (j >> a) & 1u ? 0.0 : 1.0;
            g[a][1] = __builtin_fma(w, up, g[a][1]);
            g[a][0] = __builtin_fma(w, down, g[a][0]);
        }
    }

    // The sums of x over the round's lanes of one prefix (own, contiguous)
    // added to val; lanes that are not `on` belong to none.
    __device__ __forceinline__ void to_prefix(double *val, u32 own, double x, bool on)
    {
        own = on ? own : (u32)kWave;
        const u32 before = (u32)__shfl_up((int)own, 1, kWave);
        const u64 heads = __ballot(lane == 0u || own != before);
        const int start = 63 - __builtin_clzll(heads & (~0ull >> (63u - lane)));
#pragma unroll
        for (int off = 1; off <= 16; off <<= 1) {  // at most 32 lanes per prefix
            const double y = __shfl_up(x, off, kWave);
            x += (int)lane - off >= start ? y : 0.0;
        }
        if (on && (lane == 63u || ((heads >> (lane + 1u)) & 1ull))) val[own] += x;
    }

    // Decides a word: returns its undecided cubes; v: the sum of its
    // connected ones (when `mine`).
    __device__ __forceinline__ u32 classify(u32 level, u32 rel, double q, bool live, bool mine, double (&g)[5][2],
                                            double &all, double &v)
    {
        v = 0.0;
        const u32 up = clo.close(2u * level - 1u, rel, live);
        if (__ballot(up != 0u) == 0ull) return 0u;
        const u32 down = clo.close(2u * level, rel, live && up != 0u);
        if (mine) v = cubes(level, q, down, g, all);
        return up & ~down;
    }

    // The vectors under the undecided cubes U of level 1 words (one per
    // lane: `from`, probability q above the word); returns their sums.
    __device__ __forceinline__ double finals(u32 U, u32 from, double q, u32 sub, u32 split)
    {
        u32 total, step, round;
        const u32 e = wave_excl_popc(U, total);
        if (!cube_share(total, sub, split, round, step)) return 0.0;
        W.from[lane] = (unsigned short)from;
        W.qp[0][lane] = q;
        W.val[0][lane] = 0.0;
        for (u32 w0 = 0; w0 < total; w0 += kGradQueue) {
            cube_enqueue<kGradQueue>(W.queue[0], U, e, w0, lane);
            const u32 end = min(total, w0 + (u32)kGradQueue);
            for (; (u32)kWave * round < end; round += step) {
                const u32 i = (u32)kWave * round + lane;
                const bool on = i < end;
                const u32 x = W.queue[0][(on ? i : end - 1u) - w0], own = x >> 5, j = x & 31u;
                const u32 V = clo.close(0u, (u32)W.from[own] << (2 * kCubeGroup) | j << kCubeGroup, on);
                const double qo = W.qp[0][own], qj = T.q5[1][j];
                const double F = word0(qo * qj, V);
                under(1u, qo, j, F, g1);
                to_prefix(W.val[0], own, qj * F, on);
            }
            wave_lds_sync();
        }
        return W.val[0][lane];
    }

    __device__ __forceinline__ void unit(u64 block, u32 sub)
    {
        const u32 levels = clo.levels(), lane_bits = clo.lane_bits(), split = P->split, M = clo.arcs();
        const u32 rb = kCubeGroup * levels + lane_bits;
        clo.item(block);
        const bool live = (lane >> lane_bits) == 0u;
        // the item's probability, and without the item bit `lane`
        double qi = 1.0, qm = 1.0;
#pragma unroll 4
        for (u32 b = rb; b < M; ++b) {
            const double f = cube_q(T, M, b, (u32)(block >> (b - rb)) & 1u);
            qi *= f;
            qm *= b - rb == lane ? 1.0 : f;
        }
        const double q = qi * T.ql[lane];
        double v;  // the sum under the lane's prefix
        if (levels == 1u) {
            u32 V = clo.close(0u, lane << kCubeGroup, live);
            if (M < 5u) V &= (1u << (1u << M)) - 1u;
            v = word0(q, V);
        } else if (levels == 2u) {
            const u32 U = classify(1u, lane << (2 * kCubeGroup), q, live, sub == 0u, g1, free1, v);
            v += finals(U, lane, q, sub, split);
        } else {
            const u32 U = classify(2u, lane << (3 * kCubeGroup), q, live, sub == 0u, g2, free2, v);
            u32 total, step, round;
            const u32 e = wave_excl_popc(U, total);
            if (!cube_share(total, sub, split, round, step)) total = 0u;
            W.qp[1][lane] = q;
            W.val[1][lane] = 0.0;
            for (u32 w0 = 0; w0 < total; w0 += kGradQueue) {
                cube_enqueue<kGradQueue>(W.queue[1], U, e, w0, lane);
                const u32 end = min(total, w0 + (u32)kGradQueue);
                for (; (u32)kWave * round < end; round += step) {
                    const u32 i = (u32)kWave * round + lane;
                    const bool on = i < end;
                    const u32 x = W.queue[1][(on ? i : end - 1u) - w0], own = x >> 5, j = x & 31u;
                    const double qo = W.qp[1][own], qj = T.q5[2][j];
                    double v1;
                    const u32 U1 = classify(1u, x << (2 * kCubeGroup), qo * qj, on, true, g1, free1, v1);
                    v1 += finals(U1, x, qo * qj, 0u, 1u);
                    under(2u, qo, j, v1, g2);
                    to_prefix(W.val[1], own, qj * v1, on);
                }
                wave_lds_sync();
            }
            v += W.val[1][lane];
        }
        wave_lds_sync();
        v = live ? v : 0.0;
        if (__ballot(v != 0.0) == 0ull) return;
        double w = qi * v, e;
        lane_lo += __builtin_fma(qi, v, -w);
        two_sum(lane_hi, w, lane_hi, e);
        lane_lo += e;
        if (rb < M) {
            double h = T.ql[lane] * v, l = 0.0;
            wave_sum_dd(h, l);
            // (the product's own error too: T1 and T0 share most of h, whose
            // rounding would not cancel in their difference)
            const u32 x = (u32)(block >> lane) & 1u;
            const double vh = qm * h, vl = __builtin_fma(qm, h, -vh) + qm * l;
            if (lane + rb < M) {
                double s, e;
                two_sum(x ? sh[1] : sh[0], vh, s, e);
                e += vl;
                sh[1] = x ? s : sh[1];
                sh[0] = x ? sh[0] : s;
                sl[1] += x ? e : 0.0;
                sl[0] += x ? 0.0 : e;
            }
        }
    }

    // Fold the wavefront's columns into the chunk's place (col: [1 + 2 M],
    // R first).
    __device__ __forceinline__ u64 write(double2_t *col)
    {
        const u64 c = wave_sum_u64(cnt);
        if (c == 0ull) return 0ull;  // nothing connected: every sum is 0
        const u32 levels = clo.levels(), lane_bits = clo.lane_bits(), M = clo.arcs();
        const u32 rb = kCubeGroup * levels + lane_bits;
        // the words' arcs (down, up), then the lane bits', then R
        constexpr int words = 10 * kCubeLevels, N = words + 2 * kLaneBits + 1;
        double h[N], l[N];
        const double f0 = free1 + free2, *am = X.a4m;
#pragma unroll
        for (int a = 0; a < 5; ++a)
#pragma unroll
            for (int x = 0; x < 2; ++x) {
                if (a < 3) h[2 * a + x] = g0[a][x] + f0;
                h[10 + 2 * a + x] = g1[a][x] + free2;
                h[20 + 2 * a + x] = g2[a][x];
            }
        h[6] = am[0] * tb0[0] + am[2] * tb0[2] + f0;
        h[7] = am[1] * tb0[1] + am[3] * tb0[3] + f0;
        h[8] = am[4] * tb0[0] + am[5] * tb0[1] + f0;
        h[9] = am[6] * tb0[2] + am[7] * tb0[3] + f0;
        // the lane bits' probability without each: what is below it times
        // what is above
        double f[kLaneBits], above[kLaneBits], ea[kLaneBits], below = 1.0, eb = 0.0;
#pragma unroll
        for (int b = kLaneBits - 1; b >= 0; --b) {
            f[b] = (u32)b < lane_bits ? cube_q(T, M, kCubeGroup * levels + b, (lane >> b) & 1u) : 1.0;
            above[b] = b == kLaneBits - 1 ? 1.0 : above[b + 1];
            ea[b] = b == kLaneBits - 1 ? 0.0 : ea[b + 1];
            if (b < kLaneBits - 1) dd_mul(above[b], ea[b], f[b + 1]);
        }
#pragma unroll
        for (int b = 0; b < kLaneBits; ++b) {
            const double q = below * above[b], e = __builtin_fma(below, above[b], -q) + (below * ea[b] + eb * above[b]);
            const double v = q * lane_hi, w = __builtin_fma(q, lane_hi, -v) + (q * lane_lo + e * lane_hi);
            const bool x = (lane >> b) & 1u;
            h[words + 2 * b] = x ? 0.0 : v;
            l[words + 2 * b] = x ? 0.0 : w;
            h[words + 2 * b + 1] = x ? v : 0.0;
            l[words + 2 * b + 1] = x ? w : 0.0;
            dd_mul(below, eb, f[b]);
        }
#pragma unroll
        for (int i = 0; i < words; ++i) l[i] = 0.0;
        h[N - 1] = hi;
        l[N - 1] = lo;
        wave_fold<N, words>(h, l);
        const u32 i = wave_column<N>(lane), b = i < (u32)words ? i / 2u : kCubeGroup * levels + (i - words) / 2u;
        const bool arc = i < (u32)words ? b < kCubeGroup * levels : i < N - 1u && b < rb;
        if (i == N - 1u) col[0] = {h[0], l[0]};
        else if (arc && b < M) col[1u + 2u * b + (i & 1u)] = {h[0], l[0]};
        if (lane + rb < M) {
            col[1u + 2u * (rb + lane)] = {sh[0], sl[0]};
            col[2u + 2u * (rb + lane)] = {sh[1], sl[1]};
        }
        return c;
    }
};

// cols: [grad_units(M)][COLS], COLS >= 1 + 2 M.
// Most chunks of a block: as many as leave the LDS room for three blocks on a
// CU.
constexpr int grad_units(int M) { return M <= 45 ? 8 : 4; }
template <int UNITS, int COLS, class Clo>
__device__ __forceinline__ void cube_grad_kernel(CubeArgs *P, CubeSumTables &T, CubeGradTables &X, CubeGradWave *Ws,
                                                 double2_t (&cols)[UNITS][COLS], Clo clo)
{
    __shared__ u32 next;
    __shared__ u64 sc[UNITS];
    if (threadIdx.x == 0) next = 0u;
    if (blockIdx.x == 0 && threadIdx.x < (u32)kWave) {
        // p is checked here, not by the finishing kernel, whose blocks write
        // their outputs at different times: an output may lie where p does
        const double p = P->p_dev && threadIdx.x < P->m ? P->p_dev[threadIdx.x] : 0.0;
        const u64 bad = __ballot(!(p >= 0.0 && p <= 1.0));
        if (threadIdx.x == 0) {
            cube_clock(P, 0);
            P->done[0] = 0u;
            P->done[1] = bad ? 1u : 0u;
        }
    }
    cube_tables(P, T);
    cube_grad_tables(P, T, X);
    const u32 lane = threadIdx.x & (kWave - 1);
    const u32 wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const u32 split = P->split, units = P->units, per = P->chunk, M = clo.arcs();
    const u64 all = P->n_items * split;
    CubeGradSweep<Clo> S{P, T, X, Ws[wave], clo, lane};
    for (;;) {
        __builtin_amdgcn_wave_barrier();  // (see cube_kernel)
        const u32 k = __builtin_amdgcn_readfirstlane(atomicAdd(&next, 1u)) / kWave;
        if (k >= units) break;
        S.zero();
        for (u32 i = 0; i < per; ++i) {
            const u64 w = ((u64)blockIdx.x * units + k) * per + i;
            if (w >= all) break;
            const u64 it = w / split;
            S.unit(P->item_base + ((it * P->item_mul) & P->item_mask), (u32)(w % split));
        }
        const u64 c = S.write(cols[k]);
        if (lane == 0) sc[k] = c;
    }
    __syncthreads();
    const u32 n = gridDim.x;
    for (u32 i = threadIdx.x; i < 1u + 2u * M; i += blockDim.x) {
        double h = 0.0, l = 0.0;
        for (u32 k = 0; k < units; ++k)
            if (sc[k]) dd_add(h, l, cols[k][i].x, cols[k][i].y);
        P->part[(u64)i * n + blockIdx.x] = {h, l};
    }
    if (threadIdx.x == 0) {
        u64 c = 0;
        for (u32 k = 0; k < units; ++k) c += sc[k];
        P->pcount[blockIdx.x] = c;
    }
}

}  // namespace bat

// k_knn_fit.hip -- K nearest matches per match on the match graph and the
// per-match interpolation model (Algorithm 1, steps 4-6; Sec. 3.2-3.4).
//
// One wavefront per match s:
//  1. Dijkstra from s on the match graph.  The visited set lives in LDS:
//     entries e (tentative distance, lightest incident edge, CSR range)
//     owned by lane e % 64, and an open-addressing node table whose slots
//     hold a node and its entry in one word.  Several frontier nodes are
//     settled per step: a frontier node v
//     with tentative d(v) is final once d(v) <= dmin + lightest_edge(v),
//     where dmin is the smallest tentative distance on the frontier (no
//     unsettled node can still lower it).  The edges of all nodes settled in
//     a step are relaxed together, one lane per edge, in windows of 64
//     edges: a prefix sum of the settled nodes' degrees places their edge
//     segments, a prefix maximum over marked segment starts tells every lane
//     whose edge it holds, and one 16-byte read of the node table's bucket
//     finds the entry of a neighbour that was visited before.  Every CSR record carries the neighbour's CSR
//     range and lightest edge, so one round of global loads per window is
//     all a step needs.  Float sums are monotone, so the distances equal
//     those of a sequential Dijkstra in the same precision, and a settled
//     distance is never lowered again.
//  2. The search stops once at least K settled nodes lie strictly below the
//     frontier minimum: the K smallest (distance, index) pairs are then all
//     settled.  They are selected by a bitonic sort of packed
//     (distance bits, index) keys, which also fixes the order of the sums
//     below (deterministic results).  s itself is first, at distance 0.
//  3. Weights k = exp(-a d) (Eq. 1).  NW: kernel-weighted mean displacement.
//     LA: weighted least squares of Eq. (2) with weights k^2 (each equation
//     scaled by k) or k, solved about the weighted centroid of the
//     neighbours (a 2x2 system per displacement component).  The fit is
//     done in FP32; when the neighbourhood is ill-conditioned (eigenvalue
//     ratio of the weighted position covariance below fp64_route, or fewer
//     than 3 neighbours) it is re-accumulated and solved in FP64, where a
//     near-collinear neighbourhood (ratio <= deg_tau) falls back to NW.
//  Output per match: b00 b01 b10 b11 c0 c1 with flow(p) = B (p - p_s) + c.
//
// Wave-wide sums, minima and scans use DPP row operations (registers only,
// fixed combination order).  The workgroup is a single wavefront, whose LDS
// instructions execute in issue order, so phases that hand data between
// lanes through LDS only need to keep the compiler from reordering them.
//
// A source whose visited set outgrows the small LDS table is put on an
// overflow list and redone by a second launch with a larger table; if that
// overflows too, the match's model is zero and the pair's counters record
// it (epic_get_stats then reports EPIC_ERR_CAPACITY for the pair).
#include <type_traits>

#include "epic_dev.h"
#include "fit.h"
#include "wave.h"

namespace epic {

namespace {

// Compiler-only ordering of the wavefront's LDS accesses (see above).
__device__ __forceinline__ void lds_order() { __asm__ __volatile__("" ::: "memory"); }

// Node table: an open-addressing hash of the visited nodes.  A slot holds
// the node in the high bits over its entry (EB bits; the all-ones entry
// marks a node that got no entry), all ones when empty.  256-entry tables
// pack both into 32 bits (nodes below 2^23 - 1), larger ones into 64.  The
// slots are read in buckets of 16 bytes (one LDS read): a node sits at the
// first slot that was empty, in slot order, from the start of its home
// bucket on, and slots are never freed, so a bucket with an empty slot ends
// every search that reaches it.  Five of six edges lead to a node that is
// in the table already, and a bucket is seldom full, so most edges find
// their entry with that one read; probing slot by slot with a
// compare-and-swap each cost the wavefront as many round trips as its
// unluckiest lane needed.  With the lane state kept as numbers and the
// window's atomics left to lanes that hold an edge (together 3037 -> 2804
// vector, 1879 -> 1547 scalar instructions a match on 64 mixed pairs of 444
// thousand matches): 64 mixed pairs, 473 thousand matches, K = 100: 2.07 ->
// 1.84 ms; 2048 x 1080 with 40000: 199 -> 174 us; 1024 x 436 with 8000: 55.7 ->
// 48.7 us (kernel trace).
template <int VCAP>
struct NodeSlot {
    using T = typename std::conditional<(VCAP <= 256), u32, u64>::type;
    static constexpr int SLOTS = VCAP + VCAP / 2;            // load at most 2/3
    static constexpr int BW = 16 / (int)sizeof(T);           // slots per bucket
    static constexpr int NB = SLOTS / BW;
    static constexpr int EB = VCAP <= 256 ? 9 : 32;
    static constexpr T EMPTY = ~(T)0;
    static constexpr u32 NO_ENTRY = VCAP <= 256 ? 0x1ffu : 0xffffffffu;
    static_assert(VCAP <= 256 ? VCAP < 0x1ff : true, "entry field");
    static_assert(SLOTS % BW == 0 && SLOTS >= VCAP + 64, "every window's nodes find an empty slot");
    __device__ static T pack(int v, u32 e) { return ((T)(u32)v << EB) | (T)e; }
    __device__ static int node(T w) { return (int)(w >> EB); }
    __device__ static u32 entry(T w) { return (u32)(w & (T)NO_ENTRY); }
    // First slot of node v's home bucket: a multiplicative hash, then the
    // product range reduction (NB need not be a power of two).  Nodes of
    // 32-bit slots take the 24-bit multiplies, which run at the full rate
    // (the compiler would make the first one a 32-bit multiply): the low 24
    // bits of v times the golden ratio are a fraction, its product with NB
    // the bucket.
    __device__ static u32 home(int v) {
        if constexpr (sizeof(T) == 4) {
            u32 h, b;
            __asm__("v_mul_u32_u24 %0, %1, %2" : "=v"(h) : "s"(0x9e3779u), "v"(v));
            __asm__("v_mul_hi_u32_u24 %0, %1, %2" : "=v"(b) : "s"((u32)SLOTS << 8), "v"(h));
            return b & ~(u32)(BW - 1);
        } else {
            return (u32)(((u64)((u32)v * 2654435761u) * (u32)NB) >> 32) * BW;
        }
    }
    // Looks for node v in its home bucket, at slot b: its entry, or a number
    // of VCAP or more when it is not there; `slot` is then the first slot to
    // try (the bucket's first empty one, or the next bucket's when full).
    __device__ static u32 find(const T* htab, u32 b, int v, u32& slot) {
        if constexpr (sizeof(T) == 4) {
            const uint4 w = *reinterpret_cast<const uint4*>(htab + b);
            const u32 t = (u32)v << EB;
            slot = b + (w.x != EMPTY) + (w.y != EMPTY) + (w.z != EMPTY) + (w.w != EMPTY);
            // a slot of v leaves its entry, any other slot more
            return min(min(w.x ^ t, w.y ^ t), min(w.z ^ t, w.w ^ t));
        } else {
            const ulonglong2 w = *reinterpret_cast<const ulonglong2*>(htab + b);
            slot = b + (w.x != EMPTY) + (w.y != EMPTY);
            return w.x != EMPTY && node(w.x) == v ? entry(w.x) : w.y != EMPTY && node(w.y) == v ? entry(w.y) : ~0u;
        }
    }
    // Whether a slot read as w is taken by another node than v.
    __device__ static bool other(T w, int v) {
        if constexpr (sizeof(T) == 4) return min(w ^ ((u32)v << EB), ~w) > NO_ENTRY;     // (one compare)
        else return w != EMPTY && node(w) != v;
    }
};

// FP64: 7.0 KB a match with 256 entries, 23 resident per CU (9.0 KB and 17
// with every field in double and an array of its own), and up to 128
// candidates sorted in registers: 1024 x 436 with 8000 matches 357 -> 346 us
// a call, 1242 x 480 with 9000 380 -> 359 us.
template <int VCAP, bool F64>
struct KnnLds {
    static constexpr int HCAP = NodeSlot<VCAP>::SLOTS;
    static constexpr int TW = 64;                 // edges per relaxation window (one per lane)
    using DT = typename std::conditional<F64, u64, u32>::type;     // distance bits
    using RT = typename std::conditional<F64, double, float>::type;
    using ST = typename NodeSlot<VCAP>::T;
    // FP32, entry e: tentative distance (2e), lightest incident edge (2e + 1:
    // its high 16 float bits over the degree, the CSR record's own word);
    // FP64: tentative distance (e), the lightest edge rounded down to a float
    // in mi (the settle test needs a lower bound) and the degree in dg.  The
    // last entry takes what does not fit.  After the search: the sort keys.
    static constexpr int DS = F64 ? 1 : 2;        // words of dm per entry
    alignas(16) DT dm[DS * (VCAP + 1) + (F64 ? 1 : 0)];
    // entry e: CSR start, once settled less its offset in the step's edges;
    // after the search, the entry's node
    alignas(16) u32 rd[VCAP + 4];
    alignas(16) ST htab[HCAP];    // node table
    alignas(16) u32 head[TW + 4]; // ((1 + position) << 12) | (1 + entry) of the edge segment
                                  // starting at a window position, 0 elsewhere (and one that
                                  // takes the marks beyond the window)
    alignas(16) u32 mi[F64 ? VCAP + 4 : 4];       // (after the search: node of each sort key)
    u32 dg[F64 ? VCAP + 4 : 1];
};

template <bool F64>
__device__ __forceinline__ typename std::conditional<F64, double, float>::type from_bits(
    typename std::conditional<F64, u64, u32>::type b) {
    if constexpr (F64) return dbits(b); else return __uint_as_float(b);
}
template <bool F64>
__device__ __forceinline__ typename std::conditional<F64, u64, u32>::type to_bits(
    typename std::conditional<F64, double, float>::type v) {
    if constexpr (F64) return bitsd(v); else return __float_as_uint(v);
}

// Value of v in lane (this lane xor j); j is a power of two below 64 that
// the callers' unrolled loops make a constant.
__device__ __forceinline__ u64 xor_lane_u64(u64 v, int j) {
    switch (j) {
        case 1: return wave::xor_lane<1>(v);
        case 2: return wave::xor_lane<2>(v);
        case 4: return wave::xor_lane<4>(v);
        case 8: return wave::xor_lane<8>(v);
        case 16: return wave::xor_lane<16>(v);
        default: return wave::xor_lane<32>(v);
    }
}

__device__ __forceinline__ int xor_lane_int(int v, int j) {
    switch (j) {
        case 1: return wave::xor_lane<1>(v);
        case 2: return wave::xor_lane<2>(v);
        case 4: return wave::xor_lane<4>(v);
        case 8: return wave::xor_lane<8>(v);
        case 16: return wave::xor_lane<16>(v);
        default: return wave::xor_lane<32>(v);
    }
}

// Lanes l of a wavefront with bit j of l clear, as a mask (j a power of two
// below 64): 0x5555..., 0x3333..., 0x0f0f..., ...
__device__ __forceinline__ constexpr u64 low_lanes(int j) { return ~0ull / ((1ull << j) + 1ull); }

// Ascending bitonic sort of 64 E keys held in registers, key lane + 64 r in
// v[r] (E = 1 or 2).  Exchanges across lanes go through DPP, swizzle and
// permute moves; the distance-64 exchange swaps the two registers of a lane.
// Which lanes keep the smaller key of a pair is a lane mask fixed by the step.
// PAIR: w[r] goes with v[r]; of two equal keys the lower lane's counts as the
// smaller (without, the keys are distinct, or alike in every way).
template <int E, bool PAIR>
__device__ __forceinline__ void bitonic_regs(u64 (&v)[2], int (&w)[2], int lane) {
#pragma unroll
    for (int k = 2; k <= 64 * E; k <<= 1) {
#pragma unroll
        for (int j = k >> 1; j > 0; j >>= 1) {
            if (j == 64) {                  // k = 128: ascending everywhere
                const u64 a = v[0], b = v[1];
                const bool lt = PAIR ? a <= b : a < b;
                v[0] = lt ? a : b;
                v[1] = lt ? b : a;
                if constexpr (PAIR) {
                    const int wa = w[0], wb = w[1];
                    w[0] = lt ? wa : wb;
                    w[1] = lt ? wb : wa;
                }
            } else {
#pragma unroll
                for (int r = 0; r < E; ++r) {
                    const u64 a = v[r], b = xor_lane_u64(a, j);
                    // the lower index of an ascending pair (or the upper of a
                    // descending one) keeps the smaller key
                    const u64 asc = k < 64 ? low_lanes(k) : (((64 * r) & k) == 0 ? ~0ull : 0ull);
                    const u64 keep_min = ~(low_lanes(j) ^ asc);
                    if constexpr (PAIR) {
                        const int wb = xor_lane_int(w[r], j);
                        const u64 lt = wave::ballot(a < b) | (wave::ballot(a == b) & low_lanes(j));
                        const bool own = __builtin_amdgcn_inverse_ballot_w64(~(lt ^ keep_min));
                        v[r] = own ? a : b;
                        w[r] = own ? w[r] : wb;
                    } else {
                        v[r] = ((a < b) == (bool)__builtin_amdgcn_inverse_ballot_w64(keep_min)) ? a : b;
                    }
                }
            }
        }
    }
}

// Processes source `s` of pair P; returns false when the visited set did not
// fit the table (nothing written then).
template <int VCAP, int KMAX, bool F64>
__device__ __forceinline__ bool knn_fit_one(const PairDev& P, const RunDev& run, int s, KnnLds<VCAP, F64>& S) {
    using LdsT = KnnLds<VCAP, F64>;
    using RT = typename LdsT::RT;
    const RT RINF = (RT)INFINITY;
    constexpr int HCAP = LdsT::HCAP;
    constexpr int TW = LdsT::TW;
    static_assert(TW == 64, "an edge per lane");
    constexpr int R = VCAP / 64;        // entries per lane
    using NS = NodeSlot<VCAP>;
    using ST = typename NS::T;
    static_assert(VCAP < 4096, "head mark layout");
    constexpr int RK = KMAX / 64;
    const int lane = threadIdx.x;
    const int K = P.K;
    const int keff = __builtin_amdgcn_readfirstlane(P.counters[C_KEFF]);
    ST* const htab = S.htab;
    u64* const keys = reinterpret_cast<u64*>(S.dm);       // sort keys, after the search
    EPIC_GLOBAL float* prm = gmem(P.params) + 6LL * s;
    // the match's own row, fetched now so that its latency hides behind the search
    const float4 me = gload(reinterpret_cast<const float4*>(P.matches) + s);
    // read once: the LDS ordering points below would make the compiler
    // reload it from the descriptor at every window
    const uint4* const adj = P.adj;
    const uint4* const adj64 = P.adj64;
    const u32 last_rec = (u32)P.hash_cap - 1u;

    // ------------------------------------------------------------ Dijkstra
    // entries not in use read as distance infinity, lightest edge and degree
    // 0: never the frontier minimum, never settled
    {
        const uint4 ones = make_uint4(~0u, ~0u, ~0u, ~0u), zero = make_uint4(0u, 0u, 0u, 0u);
        uint4* const t = reinterpret_cast<uint4*>(htab);
        for (int i = lane; i < NS::NB; i += 64) t[i] = ones;
        if (lane < TW / 4) reinterpret_cast<uint4*>(S.head)[lane] = zero;
        uint4* const dmq = reinterpret_cast<uint4*>(S.dm);
        constexpr u32 DINF = (u32)(DOUBLE_INF_BITS >> 32);
        const uint4 unused = F64 ? make_uint4(0u, DINF, 0u, DINF) : make_uint4(FLOAT_INF_BITS, 0u, FLOAT_INF_BITS, 0u);
        for (int i = lane; i < VCAP * 8 / 16; i += 64) dmq[i] = unused;
        if constexpr (F64)
            for (int i = lane; i < VCAP / 4; i += 64) reinterpret_cast<uint4*>(S.mi)[i] = zero;
    }
    __syncthreads();
    if (lane == 0) {
        const u32 a = gmem(P.row_ptr)[s], b = gmem(P.row_ptr)[s + 1];
        S.dm[0] = 0;
        if constexpr (F64) {
            S.mi[0] = __float_as_uint(__double2float_rd(dbits(gmem(P.minin64)[s])));
            S.rd[0] = a;
            S.dg[0] = b - a;
        } else {
            // (a degree above 16 bits stops the pair before this kernel)
            S.dm[1] = (gmem(P.minin)[s] & 0xffff0000u) | (b - a);
            S.rd[0] = a;
        }
        htab[NS::home(s)] = NS::pack(s, 0u);
    }
    __syncthreads();

    int nvis = 1;               // entries in use (the same in every lane)
    int nsettled = 0;           // settled entries (the same in every lane)
    // Lane state of group r, entry lane + 64 r: its distance as last read, a
    // mark once it is settled (0 before), its edges in this step (0 unless
    // settled in it) and where they start among the step's edges.  Kept as
    // numbers, not as lane masks: the scalar unit, shared by the CU's four
    // SIMDs, is nearly as busy with this kernel as the SIMDs are.  The mark is
    // all ones in FP32, above an infinity's bits: costs may be any finite
    // numbers, so dmin plus a lightest edge can be infinite, and an entry must
    // not be settled twice.  Sums of FP64 (of at most FLT_MAX a pixel) stay
    // finite; their mark is infinity.
    const RT SETTLED = F64 ? RINF : (RT)__uint_as_float(~0u);
    RT d[R], sf[R];
    u32 dg[R], off[R];
#pragma unroll
    for (int r = 0; r < R; ++r) {
        d[r] = RINF;
        sf[r] = (RT)0;
        dg[r] = off[r] = 0u;
    }
    RT dstop = RINF;
    // One step on the groups in use (RU of them, or with RU = 0 `ru`, known
    // at run time; on the 64-pair batch 1 % faster with RU than with a branch
    // per group): settles the final frontier nodes and marks where their
    // edges start in the step's first window.  Returns the number of edges,
    // or -1 when the search is done.
    auto step = [&](auto ru_c, int ru) -> int {
        constexpr int RU = decltype(ru_c)::value;
        RT mi[R], x[R];          // x: the distance on the frontier, the mark of settled entries
        RT fmin = RINF;
#pragma unroll
        for (int r = 0; r < R; ++r) {
            if (RU ? r >= RU : r >= ru) continue;
            if constexpr (F64) {
                d[r] = dbits(S.dm[lane + 64 * r]);
                mi[r] = (double)__uint_as_float(S.mi[lane + 64 * r]);
                dg[r] = S.dg[lane + 64 * r];
                x[r] = sf[r] > d[r] ? sf[r] : d[r];
                fmin = fmin < x[r] ? fmin : x[r];
            } else {
                const uint2 v = *reinterpret_cast<const uint2*>(&S.dm[2 * (lane + 64 * r)]);
                d[r] = __uint_as_float(v.x);
                mi[r] = __uint_as_float(v.y & 0xffff0000u);
                dg[r] = v.y & 0xffffu;
                x[r] = __uint_as_float(max(__float_as_uint(d[r]), __float_as_uint(sf[r])));
                fmin = __uint_as_float(min(__float_as_uint(fmin), __float_as_uint(x[r])));
            }
        }
        RT dmin;
        if constexpr (F64) dmin = wave::min(fmin); else dmin = wave::min_nonneg(fmin);
        // entries strictly below the frontier minimum are settled (only
        // counted once enough entries are settled at all)
        int below = 0;
        if (nsettled >= keff) {
#pragma unroll
            for (int r = 0; r < R; ++r)
                if (RU ? r < RU : r < ru) below += __popcll(wave::ballot(d[r] < dmin));
        }
        if (below >= keff || !(dmin < RINF)) {
            dstop = dmin;       // nodes settled at this point lie at or above dmin
            return -1;
        }
        // settle the final frontier nodes; their edges are relaxed below
        u32 my_edges = 0u;
        bool newly[R];
#pragma unroll
        for (int r = 0; r < R; ++r) {
            newly[r] = false;
            if (RU ? r >= RU : r >= ru) continue;
            u64 m;
            if constexpr (F64) m = wave::ballot(x[r] <= dmin + mi[r]);
            else m = wave::ballot(__float_as_uint(x[r]) <= __float_as_uint(dmin + mi[r]));     // (in the bits' order)
            newly[r] = __builtin_amdgcn_inverse_ballot_w64(m);
            nsettled += __popcll(m);
            sf[r] = newly[r] ? SETTLED : sf[r];
            dg[r] = newly[r] ? dg[r] : 0u;
            my_edges += dg[r];
        }
        const u32 incl = (u32)wave::incl_scan((int)my_edges);
        // a settled node's CSR start less the start of its edges in this
        // step turns an edge's position into its record's index; positions
        // beyond the first window are marked when their window comes
        u32 o = incl - my_edges;
#pragma unroll
        for (int r = 0; r < R; ++r) {
            if (RU ? r >= RU : r >= ru) continue;
            off[r] = o;
            if (newly[r]) {
                const u32 at = min(o, (u32)TW);
                S.head[at] = (at << 12) + (u32)((1 << 12) + lane + 64 * r + 1);
                atomicSub(&S.rd[lane + 64 * r], o);
            }
            o += dg[r];
        }
        return __builtin_amdgcn_readlane((int)incl, 63);
    };
    for (;;) {
        // nvis and nsettled are the same in every lane; readfirstlane lets
        // the compiler keep them (and the branches on them) scalar
        nvis = __builtin_amdgcn_readfirstlane(nvis);
        nsettled = __builtin_amdgcn_readfirstlane(nsettled);
        const int ru = (nvis + 63) >> 6;
        int T;
        if constexpr (R <= 4) {
            // the groups in use known at compile time: no branch per group
            T = ru == 1 ? step(std::integral_constant<int, 1>{}, ru) : ru == 2 ? step(std::integral_constant<int, 2>{}, ru)
              : ru == 3 ? step(std::integral_constant<int, 3>{}, ru) : step(std::integral_constant<int, R>{}, ru);
        } else {
            T = step(std::integral_constant<int, 0>{}, ru);
        }
        if (T < 0) break;
        u32 carry = 0u;             // 1 + entry of the segment that reaches into the next window
        for (int wb = 0; wb < T && nvis <= VCAP; wb += TW) {
            if (wb > 0) {
                // mark the segments that start in this window (a node reached
                // by an edge has at least that edge, so no two start at one place)
#pragma unroll
                for (int r = 0; r < R; ++r) {
                    const u32 at = off[r] - (u32)wb;
                    if (r < ru && dg[r] != 0u && at < (u32)TW)
                        S.head[at] = (at << 12) + (u32)((1 << 12) + lane + 64 * r + 1);
                }
            }
            lds_order();
            // the last segment start at or before this lane; the marks are
            // taken back as they are read
            const u32 hv = atomicExch(&S.head[lane], 0u);
            const u32 seg = wave::incl_max(max(hv, carry)) & 0xfffu;
            carry = (u32)__builtin_amdgcn_readlane((int)seg, 63);
            // this lane's edge: its source's settled distance and its record
            // (lanes beyond the last edge read some record of the array and
            // look for the source s, which is in the table)
            const bool act = lane < T - wb;
            const u32 qe = seg - 1u;
            const RT du = from_bits<F64>(S.dm[LdsT::DS * qe]);
            const u32 ei = min(S.rd[qe] + (u32)wb + (u32)lane, last_rec);
            // (32-bit slots: nodes below 2^23, so the records lie within 2 GiB)
            const uint4 rec = sizeof(ST) == 4
                                  ? gload(reinterpret_cast<const uint4*>(reinterpret_cast<const char*>(adj) + (ei << 4)))
                                  : gload(adj + ei);
            RT cand;
            u64 nbm = 0ull;
            if constexpr (F64) {
                // (one 16-byte load beside the record's)
                const uint4 r64 = gload(adj64 + ei);
                cand = du + dbits(words_u64(r64.x, r64.y));
                nbm = words_u64(r64.z, r64.w);
            } else {
                cand = du + __uint_as_float(rec.y);
            }
            const int v = act ? (int)rec.x : s;
            // find the neighbour's entry in the node table, or claim the
            // first empty slot, which several lanes of this window may try
            // for (the swap returns the slot's node when it is taken; the
            // table always has an empty slot)
            u32 slot;
            u32 e = NS::find(htab, NS::home(v), v, slot);
            ST prev = 0;
            if (e >= (u32)VCAP) {
                for (;;) {
                    if (slot == (u32)HCAP) slot = 0u;
                    prev = atomicCAS(&htab[slot], NS::EMPTY, NS::pack(v, NS::NO_ENTRY));
                    if (!NS::other(prev, v)) break;
                    ++slot;
                }
            }
            // the nodes claimed here get entries (their distance, lightest
            // edge and CSR range)
            const u64 m = wave::ballot(prev == NS::EMPTY);
            if (__builtin_amdgcn_inverse_ballot_w64(m)) {
                const u32 en = min((u32)(nvis + wave::lanes_below(m)), (u32)VCAP);
                S.dm[LdsT::DS * en] = to_bits<F64>(cand);
                S.rd[en] = rec.z;
                if constexpr (F64) {
                    S.mi[en] = __float_as_uint(__double2float_rd(dbits(nbm)));
                    S.dg[en] = rec.w;
                } else {
                    // lightest edge bits over the degree; the edge was
                    // rounded down to 16 bits: a lower bound, which is all
                    // the settle test needs
                    S.dm[2 * en + 1] = rec.w;
                }
                htab[slot] = NS::pack(v, en);
            }
            nvis += __popcll(m);
            lds_order();
            // relax: nodes claimed in this window have their entries by now
            if (e >= (u32)VCAP) e = NS::entry(htab[slot]);
            // (lanes without an edge stay out: atomics on one address go one by one)
            if (act) atomicMin(&S.dm[LdsT::DS * e], to_bits<F64>(cand));
            lds_order();
        }
        if (nvis > VCAP) return false;
    }

    // ---------------------------------------- select the K nearest (sorted)
    // Candidates: settled entries strictly below dstop, sorted in LDS: FP32
    // as packed (distance bits, index) words, FP64 as (distance bits, index)
    // pairs held in two arrays.
    // each entry's node, from the node table (slot -> node, slot -> entry),
    // into the CSR array, which the search no longer needs
    int* const node_of = reinterpret_cast<int*>(S.rd);
    int* const snode = reinterpret_cast<int*>(S.mi);      // FP64: the node of each sort key
    __syncthreads();
    for (int h = lane; h < HCAP; h += 64) {
        const ST w = htab[h];
        const u32 e = NS::entry(w);
        if (e < (u32)VCAP) node_of[e] = NS::node(w);         // (an empty slot's entry field is no entry)
    }
    __syncthreads();                 // the distances (the keys' space) are in registers from here
    int nc = 0;
#pragma unroll
    for (int r = 0; r < R; ++r) {
        const bool c = d[r] < dstop;         // settled: nothing on the frontier lies below dstop
        const u64 m = wave::ballot(c);
        const int pos = nc + wave::lanes_below(m);
        nc += __popcll(m);
        if (c) {
            const int e = lane + 64 * r;
            if constexpr (F64) {
                keys[pos] = bitsd(d[r]);
                snode[pos] = node_of[e];
            } else {
                keys[pos] = ((u64)__float_as_uint(d[r]) << 32) | (u32)node_of[e];
            }
        }
    }
    int p2 = 64;
    while (p2 < nc) p2 <<= 1;
    int knode[RK];
    RT kdist[RK];
    bool sorted = false;
    if constexpr (F64 && VCAP <= 256) {
        // up to 128 keys: sorted in registers by the distance alone; only
        // equal distances need the nodes in the comparison, and go to the
        // sort in LDS
        static_assert(RK <= 2, "register sort holds two keys per lane");
        if (p2 <= 128) {
            __syncthreads();
            u64 v[2];
            int w[2];
#pragma unroll
            for (int r = 0; r < 2; ++r) {
                const bool in = lane + 64 * r < nc;
                v[r] = in ? keys[lane + 64 * r] : ~0ull;
                w[r] = in ? snode[lane + 64 * r] : 0x7fffffff;
            }
            if (p2 == 64) bitonic_regs<1, true>(v, w, lane); else bitonic_regs<2, true>(v, w, lane);
            // the next key of each lane's keys (the last lane of the first
            // register is followed by the first of the second)
            const u64 n0 = __shfl_down(v[0], 1), n1 = __shfl_down(v[1], 1), h = __shfl(v[1], 0);
            const bool tie = (lane + 1 < nc && v[0] == (lane == 63 ? h : n0)) || (lane + 65 < nc && v[1] == n1);
            if (wave::ballot(tie) == 0ull) {
#pragma unroll
                for (int r = 0; r < RK; ++r) {
                    knode[r] = w[r];
                    kdist[r] = dbits(v[r]);
                }
                sorted = true;
            }
        }
    }
    if constexpr (!F64 && VCAP <= 256) {
        // up to 128 keys (the usual case): sorted in registers
        static_assert(RK <= 2, "register sort holds two keys per lane");
        if (p2 <= 128) {
            __syncthreads();
            u64 v[2];
            v[0] = lane < nc ? keys[lane] : ~0ull;
            v[1] = lane + 64 < nc ? keys[lane + 64] : ~0ull;
            int none[2];
            if (p2 == 64) bitonic_regs<1, false>(v, none, lane); else bitonic_regs<2, false>(v, none, lane);
#pragma unroll
            for (int r = 0; r < RK; ++r) {
                knode[r] = (int)(u32)v[r];
                kdist[r] = __uint_as_float((u32)(v[r] >> 32));
            }
            sorted = true;
        }
    }
    if (!sorted) {
        for (int i = nc + lane; i < p2; i += 64) {
            keys[i] = ~0ull;
            if constexpr (F64) snode[i] = 0x7fffffff;
        }
        __syncthreads();
        // each lane takes compare-exchange pairs (i, i + j): pair t has i = t
        // with a zero bit inserted at the position of j
        for (int k = 2; k <= p2; k <<= 1) {
            for (int j = k >> 1; j > 0; j >>= 1) {
                for (int t = lane; t < (p2 >> 1); t += 64) {
                    const int i = ((t & ~(j - 1)) << 1) | (t & (j - 1));
                    const int ixj = i | j;
                    {
                        const u64 a = keys[i], b = keys[ixj];
                        const bool up = (i & k) == 0;
                        if constexpr (F64) {
                            const int na = snode[i], nb = snode[ixj];
                            const bool gt = a > b || (a == b && na > nb);
                            const bool lt = a < b || (a == b && na < nb);
                            if (up ? gt : lt) {
                                keys[i] = b;
                                keys[ixj] = a;
                                snode[i] = nb;
                                snode[ixj] = na;
                            }
                        } else {
                            // keys are distinct except the padding, whose swap is harmless
                            if ((a > b) == up) {
                                keys[i] = b;
                                keys[ixj] = a;
                            }
                        }
                    }
                }
                __syncthreads();
            }
        }
#pragma unroll
        for (int r = 0; r < RK; ++r) {
            const int jj = lane + 64 * r;
            const u64 kb = jj < p2 ? keys[jj] : ~0ull;
            if constexpr (F64) {
                knode[r] = jj < p2 ? snode[jj] : 0x7fffffff;
                kdist[r] = dbits(kb);
            } else {
                knode[r] = (int)(u32)kb;
                kdist[r] = __uint_as_float((u32)(kb >> 32));
            }
        }
    }
    const int n = min(keff, nc);
    if (P.dbg_knn_idx) {
#pragma unroll
        for (int r = 0; r < RK; ++r) {
            const int jj = lane + 64 * r;
            if (jj < K) {
                const bool ok = jj < n;
                gmem(P.dbg_knn_idx)[(long long)s * K + jj] = ok ? knode[r] : -1;
                gmem(P.dbg_knn_d)[(long long)s * K + jj] = ok ? (float)kdist[r] : __int_as_float(0x7f800000);
            }
        }
    }

    // ----------------------------------------------------------------- fit
    const float xm = me.x, ym = me.y;
    const float um = me.z - xm, vm = me.w - ym;
    // the K nearest rows, all loads in flight at once (lanes beyond n load
    // the match's own row and do not use it)
    float4 mrow[RK];
#pragma unroll
    for (int r = 0; r < RK; ++r) {
        const int node = lane + 64 * r < n ? knode[r] : s;
        mrow[r] = gload(reinterpret_cast<const float4*>(P.matches) + node);
    }
    const bool la = P.mode == 1 && !run.force_nw;
    const FitOut fo = fit_about<RK, F64>(lane, n, kdist, mrow, xm, ym, um, vm, (double)me.z - (double)xm,
                                         (double)me.w - (double)ym, P.a, run.la_wpow, la, run.fp64_route,
                                         run.deg_tau);
    const float* out = fo.p;
    if (fo.fp64) {
        if (F64 && lane < 6) {
            double v = fo.p64[0];
#pragma unroll
            for (int i = 1; i < 6; ++i) v = lane == i ? fo.p64[i] : v;
            gmem(P.params64)[6LL * s + lane] = v;
        }
        if (lane == 0) {
            // (the FP64 path counts them without an atomic each, which at one
            // address take 12 ns: the CSR scan sets the count)
            if (!F64 && la) atomicAdd(&P.counters[C_FP64], 1);
            if (fo.degenerate) atomicAdd(&P.counters[C_DEGENERATE], 1);
        }
    }
    if (lane < 6) {
        float v = out[0];
#pragma unroll
        for (int i = 1; i < 6; ++i) v = lane == i ? out[i] : v;
        prm[lane] = v;
    }
    if (run.prune_px > 0.0f && lane == 0) {
        // consistency check (first, NW pass): the NW field at this match's
        // pixel is its own model's constant, out[4], out[5]
        const double du = ((double)me.z - (double)me.x) - (double)out[4];
        const double dv = ((double)me.w - (double)me.y) - (double)out[5];
        P.fill[s] = sqrt(du * du + dv * dv) <= (double)run.prune_px ? 1u : 0u;
    }
    return true;
}

// Writes the model and debug rows of a match that is not a graph node.
__device__ __forceinline__ void knn_fit_inactive(const PairDev& P, int s) {
    const int lane = threadIdx.x;
    if (lane < 6) P.params[6LL * s + lane] = 0.0f;
    if (lane == 0) P.fill[s] = 0u;        // never kept by the consistency check
    if (P.dbg_knn_idx)
        for (int j = lane; j < P.K; j += 64) {
            P.dbg_knn_idx[(long long)s * P.K + j] = -1;
            P.dbg_knn_d[(long long)s * P.K + j] = __int_as_float(0x7f800000);
        }
}

__device__ __forceinline__ bool knn_active(const PairDev& P, int s) {
    // a pair whose graph overflowed its hash has incomplete adjacency: skip
    // it (its status already reports EPIC_ERR_CAPACITY)
    const bool graph_ok = (P.counters[C_OVERFLOW] & 1) == 0;
    const int sp = P.seed_pix[s];
    return graph_ok && sp >= 0 && label_at(P, sp) == (u32)s && P.counters[C_KEFF] > 0;
}

}  // namespace

// First launch: one block (one wavefront) per match of every pair.
// At most 80 scalar registers: beyond that the hardware's allocation granule
// leaves room for 7 wavefronts per SIMD, not 8 (an earlier form of the search
// took 82, and the dispatcher's SGPR-full stall counter showed the last 832
// of 8000 matches waiting for the first ones to end).
template <int VCAP, int KMAX, bool F64>
__global__ __launch_bounds__(64) __attribute__((amdgpu_num_sgpr(80))) void k_knn_fit(
    const PairDev* __restrict__ pairs, RunDev run) {
    __shared__ KnnLds<VCAP, F64> S;
    const int p = find_pair(run.npairs, (int)blockIdx.x, [&](int i) { return pairs[i].src_block_base; });
    const PairDev& P = pairs[p];
    const int s = (int)blockIdx.x - P.src_block_base;
    if (s >= P.N) return;          // after the consistency check: a match that was removed
    if (!knn_active(P, s)) {
        knn_fit_inactive(P, s);
        return;
    }
    if (!knn_fit_one<VCAP, KMAX, F64>(P, run, s, S) && threadIdx.x == 0)
        run.ovf_list[atomicAdd(run.ovf_count, 1)] = (int)blockIdx.x;
}

// Second launch: the matches whose visited set did not fit, with a larger
// table.  A fixed grid walks the overflow list.
template <int VCAP, int KMAX, bool F64>
__global__ __launch_bounds__(64) void k_knn_fit_retry(const PairDev* __restrict__ pairs, RunDev run) {
    __shared__ KnnLds<VCAP, F64> S;
    const int count = *run.ovf_count;
    for (int i = (int)blockIdx.x; i < count; i += (int)gridDim.x) {
        const int gb = run.ovf_list[i];
        const int p = find_pair(run.npairs, gb, [&](int k) { return pairs[k].src_block_base; });
        const PairDev& P = pairs[p];
        const int s = gb - P.src_block_base;
        if (!knn_fit_one<VCAP, KMAX, F64>(P, run, s, S)) {
            knn_fit_inactive(P, s);
            if (threadIdx.x == 0) {
                atomicOr(&P.counters[C_OVERFLOW], 2);
                if (F64 && P.mode == 1 && !run.force_nw) atomicSub(&P.counters[C_FP64], 1);
            }
        }
        __syncthreads();
    }
}

namespace {
template <bool F64>
void launch_knn_t(const PairDev* d_pairs, const RunDev& run, int total_blocks, int kmax, int nmax, hipStream_t s) {
    const int retry_grid = 512;
    // 256-entry tables keep node and entry in one 32-bit slot (nodes below
    // 2^23 - 1); a call with larger pairs takes the 512-entry kernels
    const bool small_ids = nmax < (1 << 23) - 1;
    if (kmax <= 64 && small_ids) {
        hipLaunchKernelGGL((k_knn_fit<256, 64, F64>), dim3(total_blocks), dim3(64), 0, s, d_pairs, run);
        hipLaunchKernelGGL((k_knn_fit_retry<1024, 64, F64>), dim3(retry_grid), dim3(64), 0, s, d_pairs, run);
    } else if (kmax <= 128 && small_ids) {
        hipLaunchKernelGGL((k_knn_fit<256, 128, F64>), dim3(total_blocks), dim3(64), 0, s, d_pairs, run);
        hipLaunchKernelGGL((k_knn_fit_retry<2048, 128, F64>), dim3(retry_grid), dim3(64), 0, s, d_pairs, run);
    } else {
        hipLaunchKernelGGL((k_knn_fit<512, 256, F64>), dim3(total_blocks), dim3(64), 0, s, d_pairs, run);
        hipLaunchKernelGGL((k_knn_fit_retry<2048, 256, F64>), dim3(retry_grid), dim3(64), 0, s, d_pairs, run);
    }
}
}  // namespace

hipError_t launch_knn_fit(const PairDev* d_pairs, const RunDev& run, int total_blocks, int kmax, int nmax,
                          hipStream_t s) {
    if (run.precision == 1) launch_knn_t<true>(d_pairs, run, total_blocks, kmax, nmax, s);
    else launch_knn_t<false>(d_pairs, run, total_blocks, kmax, nmax, s);
    return hipGetLastError();
}

}  // namespace epic

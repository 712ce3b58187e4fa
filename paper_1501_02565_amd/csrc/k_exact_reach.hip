// k_exact_reach.hip -- the exact per-pixel interpolation (k_exact.hip) with
// one workgroup per match for its bounded single-source distances.
//
// A match matters to about twice the K nearest matches' share of the pixels
// (1024 x 436, 8000 matches, K = 100: 10 thousand of 446 thousand), so its
// distances fit in LDS.  They are kept in pages of 8 x 8 pixels, allocated as
// the relaxation reaches a block of the image; a wavefront relaxes a page,
// one pixel per lane, until nothing in it changes, and marks the neighbouring
// blocks in which a changed border pixel improves a pixel within its bound.
// The marked pages are the next round's work; a round ends at a barrier.  The
// value of a pixel is the minimum over paths of the same left-fold FP32 sums
// as in the tiled transform, whatever the order of relaxation (k_geodesic.hip),
// and the same bound cuts it off, so the distances are the same bits.
//
//   k_exact_reach    per source: the distances, stored as one entry of 64 per
//                    reached block; k_exact_reach_wide the same with a whole
//                    CU's LDS instead of half of it, for the sources that
//                    reach more blocks, and k_exact_reach_big with the pages
//                    in memory, for those that reach more still.
//   k_exact_offsets  the entries of a block are counted as they are stored;
//                    their prefix sums,
//   k_exact_place    and each block's list of (entry, source).
//   k_exact_nearest  a wavefront per pixel: its candidates from the entries of
//                    its block, the K smallest (distance, index) keys of them
//                    sorted in registers, and the fit (fit.h).
//
// Entries go to a pool.  When it is full the remaining sources are put off to
// another round of the same launches, which merges into the pixels' lists;
// the host launches as many rounds as could be needed at most (each source
// reaching every block), and the unneeded ones leave at once.
//
// Measured on 1024 x 436, 8000 matches, K = 100: 5.3 ms for the whole call,
// where the batched transforms and per-pixel heaps (k_exact.hip) took 28.4:
// the distances 3.4 ms (bound by the latency of a page's LDS round trips and
// of the costs it loads), the nearest and fits 1.9 ms (instruction issue).
// Where most matches reach more blocks than LDS holds, the batched form is the
// faster one: exact_plan.h chooses.
#include <algorithm>

#include "epic_dev.h"
#include "fit.h"
#include "wave.h"

namespace epic {

namespace {

constexpr u32 INF_BITS = 0x7f800000u;

// Two workgroups fit a CU's LDS, with 1024 threads at 8 wavefronts per SIMD its
// wave slots too.  512 and 768 threads took 6.9 and 6.1 ms where 1024 take
// 5.7 (1024 x 436, 8000 matches, K = 100); 896, of which one workgroup fits, 7.9.
// (These before the wide form: there the sources that outgrow this one took 0.74
// ms with their pages in memory, 0.35 with all of a CU's LDS; with a table of 40
// blocks there too, 0.35 and 0.54 in memory for those that reach further.  How
// many outgrow it is the scene's: another one of these sizes has wide sources
// of 0.93 ms.)
template <int PAGES_, int TB_>
struct ReachCfg {
    static constexpr int NT = 1024, NW = NT / 64;       // threads, wavefronts
    static constexpr int PAGES = PAGES_;               // pages; page 0 stays infinite
    static constexpr int TB = TB_;                     // blocks across the page table
};
using ReachMost = ReachCfg<272, 40>;
using ReachWide = ReachCfg<544, 60>;     // a CU's LDS

template <class C>
struct ReachLds {
    alignas(16) u32 page[C::PAGES][64];               // distance bits
    u32 tab[C::TB * C::TB];        // block -> page (0: none)
    u32 where[C::PAGES];           // page -> block (x | y << 16)
    u32 req[C::PAGES];             // neighbours to mark, a bit per direction
    unsigned short list[2][C::PAGES];
    u32 stamp[C::PAGES];           // last round the page was listed for
    int npages, n[2], full;
    u32 base;
};
static_assert(2 * sizeof(ReachLds<ReachMost>) <= 160 * 1024, "two workgroups per CU");
static_assert(sizeof(ReachLds<ReachWide>) <= 160 * 1024, "one workgroup per CU");

// Directions: (sx + 1) * 3 + (sy + 1), 4 is the block itself.
template <int CONN>
struct Nb {
    static constexpr int DX[8] = {1, -1, 0, 0, 1, -1, 1, -1};
    static constexpr int DY[8] = {0, 0, 1, -1, 1, 1, -1, -1};
};

// One lane's pixel of a page during its visit.
template <int CONN>
struct Pixel {
    float w[CONN];                 // step costs to the neighbours
    float ub[CONN];                // the neighbours' bounds
    float own_ub;                  // below 0: outside the image
};

template <int CONN>
__device__ __forceinline__ void load_pixel(const ExactArgs& A, int x, int y, Pixel<CONN>& px) {
    const bool in = x < A.W && y < A.H;
    const float2* const cu = A.cu;
    const float2 own = in ? gload(cu + ((long long)y * A.W + x)) : make_float2(0.0f, -1.0f);
    px.own_ub = own.y;
    float2 q[CONN];
#pragma unroll
    for (int k = 0; k < CONN; ++k) {
        const int nx = x + Nb<CONN>::DX[k], ny = y + Nb<CONN>::DY[k];
        const bool ok = in && nx >= 0 && ny >= 0 && nx < A.W && ny < A.H;
        q[k] = ok ? gload(cu + ((long long)ny * A.W + nx)) : make_float2(0.0f, -1.0f);
    }
#pragma unroll
    for (int k = 0; k < CONN; ++k) {
        px.w[k] = step_f32(k < 4 ? 1.0f : 1.41421356237309515f, own.x, q[k].x);
        px.ub[k] = q[k].y;
    }
}

// Relaxes one page to its fixpoint (wavefront-wide); at[k] is where neighbour
// k's distance lies, self the lane's own.  Returns the directions in which a
// changed pixel improves a neighbour outside the page.  Other wavefronts may
// be relaxing the pages around it: values are read and written whole (32-bit
// relaxed atomics), every value is a path's length, and whoever lowers a
// pixel that this page has read too early marks it again.
template <int CONN>
__device__ __forceinline__ u32 relax_page(const Pixel<CONN>& px, u32* self, u32* const (&at)[CONN], int lane) {
    const int lx = lane & 7, ly = lane >> 3;
    u32 d = lds_ld(self);
    const u32 d0 = d;
    u32 nb[CONN];
    for (int it = 0; it < 4096; ++it) {
#pragma unroll
        for (int k = 0; k < CONN; ++k) nb[k] = lds_ld(at[k]);
        u32 best = d;
#pragma unroll
        for (int k = 0; k < CONN; ++k)
            best = min(best, __float_as_uint(relax_f32(__uint_as_float(nb[k]), px.w[k])));
        const bool take = best < d && __uint_as_float(best) <= px.own_ub;
        if (take) {
            d = best;
            lds_st(self, d);
        }
        if (wave::ballot(take) == 0ull) break;
    }
    u32 mask = 0u;
#pragma unroll
    for (int k = 0; k < CONN; ++k) {
        const int nx = lx + Nb<CONN>::DX[k], ny = ly + Nb<CONN>::DY[k];
        const int sx = nx < 0 ? -1 : nx > 7 ? 1 : 0, sy = ny < 0 ? -1 : ny > 7 ? 1 : 0;
        const float cand = relax_f32(__uint_as_float(d), px.w[k]);
        if ((sx != 0 || sy != 0) && d < d0 && __float_as_uint(cand) < nb[k] && cand <= px.ub[k])
            mask |= 1u << ((sx + 1) * 3 + sy + 1);
    }
    u32 all = 0u;
#pragma unroll
    for (int b = 0; b < 9; ++b)
        if (wave::ballot((mask >> b) & 1u) != 0ull) all |= 1u << b;
    return all;
}

// Stores a source's entries, or puts the source off when the pool is full.
// blk(i) is the block of its i-th page, val(i, lane) a distance.
template <int NT, class B, class V>
__device__ __forceinline__ void store_entries(const ExactArgs& A, int src, int m, u32& s_base, B blk, V val) {
    const int tid = threadIdx.x, lane = tid & 63;
    if (tid == 0) s_base = atomicAdd(&A.ctl[X_USED], (u32)m);
    __syncthreads();
    const u32 base = s_base;
    if (base > A.pool_cap || A.pool_cap - base < (u32)m) {
        if (tid == 0) atomicMin(&A.ctl[X_LIMIT], base);
        if (tid == 0) A.pend[A.round & 1 ? 0 : 1][atomicAdd(&A.ctl[X_PEND0 + 16 * (A.round & 1 ? 0 : 1)], 1u)] = (u32)src;
        __syncthreads();
        return;
    }
    for (int i = tid; i < m; i += NT) {
        const u32 b = blk(i);
        A.meta[base + i] = make_uint4(b, atomicAdd(&A.bcount[b], 1u), (u32)src, 0u);
    }
    for (int i = tid >> 6; i < m; i += NT / 64) A.pool[((size_t)base + i) * 64 + lane] = val(i, lane);
    __syncthreads();
}

// Source seeds: the pixel of a match that holds it.
__device__ __forceinline__ void seed_of(const ExactArgs& A, int s, int& sx, int& sy) {
    const float4 m = gload(reinterpret_cast<const float4*>(A.matches) + s);
    sx = (int)floor((double)m.x + 0.5);
    sy = (int)floor((double)m.y + 0.5);
}

}  // namespace

// One source's distances in LDS and their entries; false when it reaches more
// blocks than there are pages, or further than the table.
template <int CONN, class C>
__device__ __forceinline__ bool reach_source(const ExactArgs& A, int s, ReachLds<C>& S) {
    constexpr int NT = C::NT, NW = C::NW, PAGES = C::PAGES, TB = C::TB;
    const int tid = threadIdx.x, lane = tid & 63, wid = tid >> 6;
    int sx, sy;
    seed_of(A, s, sx, sy);
    const int BW = (A.W + 7) >> 3, BH = (A.H + 7) >> 3;
    const int ox = (sx >> 3) - TB / 2, oy = (sy >> 3) - TB / 2;       // table origin (blocks)
    for (int i = tid; i < PAGES * 16; i += NT)
        reinterpret_cast<uint4*>(&S.page[0][0])[i] = make_uint4(INF_BITS, INF_BITS, INF_BITS, INF_BITS);
    for (int i = tid; i < TB * TB; i += NT) S.tab[i] = 0u;
    for (int i = tid; i < PAGES; i += NT) S.stamp[i] = 0u;
    __syncthreads();
    if (tid == 0) {
        S.npages = 2;
        S.n[0] = 1;
        S.n[1] = 0;
        S.full = 0;
        S.list[0][0] = 1;
        S.where[1] = (u32)(sx >> 3) | (u32)(sy >> 3) << 16;
        S.tab[(TB / 2) * TB + TB / 2] = 1u;
        S.page[1][(sy & 7) * 8 + (sx & 7)] = 0u;
    }
    __syncthreads();
    const int lx = lane & 7, ly = lane >> 3;
    bool seeded = false;           // the source's own page: its seed counts as changed
    for (int round = 1;; ++round) {
        const int cur = (round - 1) & 1, n = S.n[cur];
        for (int i = wid; i < n; i += NW) {
            const int p = __builtin_amdgcn_readfirstlane((int)S.list[cur][i]);
            const u32 wh = (u32)__builtin_amdgcn_readfirstlane((int)S.where[p]);
            const int bx = (int)(wh & 0xffffu), by = (int)(wh >> 16);
            Pixel<CONN> px;
            load_pixel<CONN>(A, bx * 8 + lx, by * 8 + ly, px);
            // the pages around it (0, all infinite, where there is none)
            int pg[9];
#pragma unroll
            for (int q = 0; q < 9; ++q) {
                const int cx = bx + q / 3 - 1 - ox, cy = by + q % 3 - 1 - oy;
                pg[q] = (cx >= 0 && cy >= 0 && cx < TB && cy < TB)
                            ? __builtin_amdgcn_readfirstlane((int)lds_ld(&S.tab[cy * TB + cx])) : 0;
            }
            u32* at[CONN];
#pragma unroll
            for (int k = 0; k < CONN; ++k) {
                const int nx = lx + Nb<CONN>::DX[k], ny = ly + Nb<CONN>::DY[k];
                const int qx = nx < 0 ? 0 : nx > 7 ? 2 : 1, qy = ny < 0 ? 0 : ny > 7 ? 2 : 1;
                int page = pg[4];
#pragma unroll
                for (int q = 0; q < 9; ++q)
                    if (q == qx * 3 + qy) page = pg[q];
                at[k] = &S.page[page][(ny & 7) * 8 + (nx & 7)];
            }
            const bool first = !seeded && p == 1 && round == 1;
            u32 mask = relax_page<CONN>(px, &S.page[p][lane], at, lane);
            if (first) {
                // (the seed was not lowered by a relaxation: mark every block
                // next to its pixel's block)
                mask = CONN == 8 ? 0x1efu : 0xaau;
            }
            if (lane == 0) S.req[p] = mask;
        }
        seeded = true;
        __syncthreads();
        if (tid == 0) S.n[cur ^ 1] = 0;
        // pages for the marked blocks (bit 31 of a table entry: being allocated)
        for (int i = tid; i < n * 9; i += NT) {
            const int p = S.list[cur][i / 9], q = i % 9;
            if (!((S.req[p] >> q) & 1u)) continue;
            const int bx = (int)(S.where[p] & 0xffffu) + q / 3 - 1, by = (int)(S.where[p] >> 16) + q % 3 - 1;
            if (bx < 0 || by < 0 || bx >= BW || by >= BH) continue;
            const int cx = bx - ox, cy = by - oy;
            if (cx < 0 || cy < 0 || cx >= TB || cy >= TB) {
                S.full = 1;
                continue;
            }
            u32* const t = &S.tab[cy * TB + cx];
            if (lds_ld(t) == 0u && atomicCAS(t, 0u, 0x80000000u) == 0u) {
                const int page = atomicAdd(&S.npages, 1);
                if (page >= PAGES) {
                    S.full = 1;
                    lds_st(t, 0u);
                } else {
                    S.where[page] = (u32)bx | (u32)by << 16;
                    lds_st(t, (u32)page);
                }
            }
        }
        __syncthreads();
        if (S.full) break;
        for (int i = tid; i < n * 9; i += NT) {
            const int p = S.list[cur][i / 9], q = i % 9;
            if (!((S.req[p] >> q) & 1u)) continue;
            const int bx = (int)(S.where[p] & 0xffffu) + q / 3 - 1, by = (int)(S.where[p] >> 16) + q % 3 - 1;
            if (bx < 0 || by < 0 || bx >= BW || by >= BH) continue;
            const int page = (int)S.tab[(by - oy) * TB + bx - ox];
            if (atomicExch(&S.stamp[page], (u32)round) != (u32)round)
                S.list[cur ^ 1][atomicAdd(&S.n[cur ^ 1], 1)] = (unsigned short)page;
        }
        __syncthreads();
        if (S.n[cur ^ 1] == 0) break;
    }
    if (S.full) return false;
    const int m = S.npages - 1;
    store_entries<NT>(A, s, m, S.base,
                      [&](int i) { return (S.where[i + 1] >> 16) * (u32)BW + (S.where[i + 1] & 0xffffu); },
                      [&](int i, int l) { return S.page[i + 1][l]; });
    return true;
}

template <int CONN>
__global__ __launch_bounds__(ReachMost::NT) __attribute__((amdgpu_waves_per_eu(8))) void k_exact_reach(ExactArgs A) {
    __shared__ ReachLds<ReachMost> S;
    int s = (int)blockIdx.x;
    if (A.round > 0) {
        const u32* const np = &A.ctl[X_PEND0 + 16 * (A.round & 1)];
        if ((u32)s >= *np) return;
        s = (int)A.pend[A.round & 1][s];
    }
    if (A.owner[s] == 0) return;
    if (!reach_source<CONN>(A, s, S) && threadIdx.x == 0) A.wide[atomicAdd(&A.ctl[X_WIDE], 1u)] = (u32)s;
}

// The sources that found no page left, with all of a CU's LDS; workgroup g
// takes every gridDim.x-th of them.
template <int CONN>
__global__ __launch_bounds__(ReachWide::NT) void k_exact_reach_wide(ExactArgs A) {
    __shared__ ReachLds<ReachWide> S;
    const int count = (int)A.ctl[X_WIDE];
    for (int w = (int)blockIdx.x; w < count; w += (int)gridDim.x) {
        const int s = (int)A.wide[w];
        if (!reach_source<CONN>(A, s, S) && threadIdx.x == 0) A.big[atomicAdd(&A.ctl[X_BIG], 1u)] = (u32)s;
        __syncthreads();             // S is set up again
    }
}

// The same with the pages in memory (block b's page at b, page `nblocks` all
// infinite), for the sources of the overflow list: workgroup g takes every
// gridDim.x-th of them, in its own part of the scratch, which it leaves clean.
template <int CONN>
__global__ __launch_bounds__(512) void k_exact_reach_big(ExactArgs A) {
    constexpr int NT = 512, NW = NT / 64;
    __shared__ int s_n[2], s_m;
    __shared__ u32 s_base;
    const int tid = threadIdx.x, lane = tid & 63, wid = tid >> 6;
    const int count = (int)A.ctl[X_BIG];
    if ((int)blockIdx.x >= count) return;
    const int BW = (A.W + 7) >> 3, BH = (A.H + 7) >> 3, NB = BW * BH;
    u32* const page = A.scratch + (size_t)blockIdx.x * A.scratch_words;       // (NB + 1) * 64
    u32* const req = page + (size_t)(NB + 1) * 64;                            // NB
    u32* const stamp = req + NB;                                              // NB: 0 = not reached
    u32* const reached = stamp + NB;                                          // NB: the blocks reached
    u32* const list0 = reached + NB;                                          // 2 * NB
    for (int i = tid; i < (NB + 1) * 64; i += NT) page[i] = INF_BITS;
    for (int i = tid; i < NB; i += NT) stamp[i] = 0u;
    __syncthreads();
    const int lx = lane & 7, ly = lane >> 3;
    for (int w = (int)blockIdx.x; w < count; w += (int)gridDim.x) {
        const int s = (int)A.big[w];
        int sx, sy;
        seed_of(A, s, sx, sy);
        const int b0 = (sy >> 3) * BW + (sx >> 3);
        if (tid == 0) {
            s_n[0] = 1;
            s_n[1] = 0;
            s_m = 1;
            list0[0] = (u32)b0;
            reached[0] = (u32)b0;
            stamp[b0] = 1u;
            page[(size_t)b0 * 64 + (sy & 7) * 8 + (sx & 7)] = 0u;
        }
        __syncthreads();
        for (u32 round = 2;; ++round) {
            const int cur = (int)(round & 1u), n = s_n[cur];
            const u32* const list = list0 + (size_t)cur * NB;
            u32* const next = list0 + (size_t)(cur ^ 1) * NB;
            for (int i = wid; i < n; i += NW) {
                const int b = __builtin_amdgcn_readfirstlane((int)lds_ld(&list[i]));
                const int bx = b % BW, by = b / BW;
                Pixel<CONN> px;
                load_pixel<CONN>(A, bx * 8 + lx, by * 8 + ly, px);
                u32* at[CONN];
#pragma unroll
                for (int k = 0; k < CONN; ++k) {
                    const int nx = bx * 8 + lx + Nb<CONN>::DX[k], ny = by * 8 + ly + Nb<CONN>::DY[k];
                    const int qx = nx >> 3, qy = ny >> 3;
                    const bool in = nx >= 0 && ny >= 0 && qx < BW && qy < BH;
                    at[k] = page + ((size_t)(in ? qy * BW + qx : NB) * 64 + (ny & 7) * 8 + (nx & 7));
                }
                u32 mask = relax_page<CONN>(px, page + ((size_t)b * 64 + lane), at, lane);
                if (round == 2) mask = CONN == 8 ? 0x1efu : 0xaau;
                if (lane == 0) req[b] = mask;
            }
            __syncthreads();
            if (tid == 0) s_n[cur ^ 1] = 0;
            __syncthreads();
            for (int i = tid; i < n * 9; i += NT) {
                const int b = (int)list[i / 9], q = i % 9;
                if (!((req[b] >> q) & 1u)) continue;
                const int bx = b % BW + q / 3 - 1, by = b / BW + q % 3 - 1;
                if (bx < 0 || by < 0 || bx >= BW || by >= BH) continue;
                const int t = by * BW + bx;
                const u32 old = atomicExch(&stamp[t], round);
                if (old != round) next[atomicAdd(&s_n[cur ^ 1], 1)] = (u32)t;
                if (old == 0u) reached[atomicAdd(&s_m, 1)] = (u32)t;
            }
            __syncthreads();
            if (s_n[cur ^ 1] == 0) break;
        }
        const int m = s_m;
        store_entries<NT>(A, s, m, s_base, [&](int i) { return reached[i]; },
                          [&](int i, int l) { return page[(size_t)reached[i] * 64 + l]; });
        for (int i = wid; i < m; i += NW) page[(size_t)reached[i] * 64 + lane] = INF_BITS;
        for (int i = tid; i < m; i += NT) stamp[reached[i]] = 0u;
        __syncthreads();
    }
}

// Prefix sums of the blocks' entry counts (one workgroup of 1024).
__global__ __launch_bounds__(1024) void k_exact_offsets(ExactArgs A) {
    __shared__ u32 s_wave[16];
    const int tid = threadIdx.x, lane = tid & 63, wid = tid >> 6;
    const int NB = ((A.W + 7) >> 3) * ((A.H + 7) >> 3), chunk = (NB + 1023) / 1024;
    const int b = min(NB, tid * chunk), e = min(NB, b + chunk);
    u32 sum = 0;
    for (int i = b; i < e; ++i) sum += A.bcount[i];
    const u32 incl = (u32)wave::incl_scan((int)sum);
    if (lane == 63) s_wave[wid] = incl;
    __syncthreads();
    u32 at = incl - sum;
    for (int w = 0; w < wid; ++w) at += s_wave[w];
    for (int i = b; i < e; ++i) {
        A.offset[i] = at;
        at += A.bcount[i];
    }
}

__global__ __launch_bounds__(256) void k_exact_place(ExactArgs A) {
    const u32 used = min(A.ctl[X_USED], A.ctl[X_LIMIT]);
    for (u32 e = blockIdx.x * 256 + threadIdx.x; e < used; e += gridDim.x * 256) {
        const uint4 m = gload(A.meta + e);
        A.order[A.offset[m.x] + m.y] = make_uint2(e, m.z);
    }
}

namespace {

// Ascending bitonic sort of 128 keys, key lane + 64 r in v[r], and the merge
// of a sorted v into a sorted best (the 128 smallest of both).
__device__ __forceinline__ u64 xor_key(u64 v, int j) {
    switch (j) {
        case 1: return wave::xor_lane<1>(v);
        case 2: return wave::xor_lane<2>(v);
        case 4: return wave::xor_lane<4>(v);
        case 8: return wave::xor_lane<8>(v);
        case 16: return wave::xor_lane<16>(v);
        default: return wave::xor_lane<32>(v);
    }
}
__device__ __forceinline__ constexpr u64 low_half(int j) { return ~0ull / ((1ull << j) + 1ull); }

template <int E>
__device__ __forceinline__ void step_keys(u64 (&v)[2], int k, int j) {
    if (j == 64) {
        const u64 a = v[0], b = v[1];
        v[0] = a < b ? a : b;
        v[1] = a < b ? b : a;
        return;
    }
#pragma unroll
    for (int r = 0; r < E; ++r) {
        const u64 a = v[r], b = xor_key(a, j);
        const u64 asc = k < 64 ? low_half(k) : (((64 * r) & k) == 0 ? ~0ull : 0ull);
        const bool keep_min = __builtin_amdgcn_inverse_ballot_w64(~(low_half(j) ^ asc));
        v[r] = ((a < b) == keep_min) ? a : b;
    }
}
template <int E>
__device__ __forceinline__ void sort_keys(u64 (&v)[2]) {
#pragma unroll
    for (int k = 2; k <= 64 * E; k <<= 1)
#pragma unroll
        for (int j = k >> 1; j > 0; j >>= 1) step_keys<E>(v, k, j);
}
__device__ __forceinline__ void merge_keys(u64 (&best)[2], const u64 (&v)[2], int lane) {
    const u64 r0 = __shfl(v[1], 63 - lane), r1 = __shfl(v[0], 63 - lane);     // v backwards
    best[0] = best[0] < r0 ? best[0] : r0;
    best[1] = best[1] < r1 ? best[1] : r1;
#pragma unroll
    for (int j = 64; j > 0; j >>= 1) step_keys<2>(best, 128, j);
}

}  // namespace

namespace {

// Pixel i of block b, by one wavefront.  Candidates of the block's entries are
// gathered in LDS until more than 64 are there, sorted and merged; a candidate
// that is not among the K smallest so far is dropped when it is read.
template <int RK>
__device__ __forceinline__ void nearest_of(const ExactArgs& A, int b, int i, int lane, bool last, u64* buf) {
    const int BW = (A.W + 7) >> 3;
    const int x = (b % BW) * 8 + (i & 7), y = (b / BW) * 8 + (i >> 3);
    if (x >= A.W || y >= A.H) return;
    const long long p = (long long)y * A.W + x;
    const int K = A.K;
    u64 best[2] = {~0ull, ~0ull};
    if (A.round > 0) {
#pragma unroll
        for (int r = 0; r < 2; ++r)
            if (lane + 64 * r < K) best[r] = gmem(A.lists)[(long long)(lane + 64 * r) * A.HW + p];
    }
    auto kth = [&]() {
        const u64 v = K > 64 ? best[1] : best[0];
        const int l = (K - 1) & 63;
        return words_u64((u32)__builtin_amdgcn_readlane((int)(u32)v, l), (u32)__builtin_amdgcn_readlane((int)(v >> 32), l));
    };
    u64 cut = kth();
    int cnt = 0;
    auto flush = [&]() {
        __syncthreads();
        u64 v[2];
        v[0] = lane < cnt ? buf[lane] : ~0ull;
        v[1] = lane + 64 < cnt ? buf[lane + 64] : ~0ull;
        if (cnt > 64) sort_keys<2>(v); else sort_keys<1>(v);
        merge_keys(best, v, lane);
        cut = kth();
        cnt = 0;
        __syncthreads();
    };
    const int ne = (int)A.bcount[b];
    const u32 off = A.offset[b];
    for (int j0 = 0; j0 < ne; j0 += 64) {
        u64 key = ~0ull;
        if (j0 + lane < ne) {
            const uint2 o = A.order[off + j0 + lane];
            const u32 d = gmem(A.pool)[(size_t)o.x * 64 + i];
            if (d < INF_BITS) key = words_u64(o.y, d);
        }
        const u64 m = wave::ballot(key < cut);
        if (cnt + __popcll(m) > 128) flush();
        if (key < cut) buf[cnt + wave::lanes_below(wave::ballot(key < cut))] = key;
        cnt += __popcll(wave::ballot(key < cut));
        if (cnt > 64 && j0 + 64 < ne) flush();
    }
    if (cnt > 0) flush();
    if (!last) {
#pragma unroll
        for (int r = 0; r < 2; ++r)
            if (lane + 64 * r < K) gmem(A.lists)[(long long)(lane + 64 * r) * A.HW + p] = best[r];
        return;
    }
    int node[RK];
    float kd[RK];
    int n = 0;
#pragma unroll
    for (int r = 0; r < RK; ++r) {
        const u64 v = lane + 64 * r < K ? best[r] : ~0ull;
        node[r] = v != ~0ull ? (int)(u32)v : -1;
        kd[r] = v != ~0ull ? key_dist(v) : 0.0f;
        n += __popcll(wave::ballot(node[r] >= 0));
    }
    float2 f;
    if (n == 0) {
        f.x = f.y = __int_as_float(0x7fc00000);          // no match in the image
    } else {
        const int n0 = __builtin_amdgcn_readfirstlane(node[0]);
        float4 mrow[RK];
#pragma unroll
        for (int r = 0; r < RK; ++r) mrow[r] = gload(reinterpret_cast<const float4*>(A.matches) + (node[r] >= 0 ? node[r] : n0));
        const float4 m0 = gload(reinterpret_cast<const float4*>(A.matches) + n0);
        const FitOut fo = fit_about<RK, false>(lane, n, kd, mrow, (float)x, (float)y, m0.z - m0.x, m0.w - m0.y,
                                               (double)m0.z - (double)m0.x, (double)m0.w - (double)m0.y,
                                               A.a, A.wpow, A.mode == 1, A.fp64_route, A.deg_tau);
        f.x = fo.p[4];
        f.y = fo.p[5];
    }
    if (lane == 0) gstore(reinterpret_cast<float2*>(A.flow) + p, f);
}

}  // namespace

template <int KMAX>
__global__ __launch_bounds__(64) void k_exact_nearest(ExactArgs A) {
    constexpr int RK = KMAX / 64;
    __shared__ u64 buf[128];
    const int lane = threadIdx.x;
    if (A.round > 0 && A.ctl[X_PEND0 + 16 * (A.round & 1)] == 0u) return;     // nothing was put off to this round
    const bool last = A.ctl[X_PEND0 + 16 * ((A.round & 1) ^ 1)] == 0u;
    const int BW = (A.W + 7) >> 3, NB = BW * ((A.H + 7) >> 3);
    // (one pixel per workgroup in the first round; the later ones, which
    // seldom have anything to do, take a small grid)
    for (u32 g = blockIdx.x; g < (u32)NB * 64u; g += gridDim.x)
        nearest_of<RK>(A, (int)(g >> 6), (int)(g & 63u), lane, last, buf);
}
// Before a round: empty counts, pool and lists (the list that the round reads stays).
__global__ __launch_bounds__(256) void k_exact_round(ExactArgs A) {
    const int NB = ((A.W + 7) >> 3) * ((A.H + 7) >> 3);
    const int i = (int)(blockIdx.x * 256 + threadIdx.x);
    if (i < NB) A.bcount[i] = 0u;
    if (i == 0) {
        A.ctl[X_USED] = 0u;
        A.ctl[X_LIMIT] = A.pool_cap;
        A.ctl[X_WIDE] = 0u;
        A.ctl[X_BIG] = 0u;
        A.ctl[X_PEND0 + 16 * ((A.round & 1) ^ 1)] = 0u;
        if (A.round == 0) A.ctl[X_PEND0] = 0u;
    }
}

hipError_t launch_exact_reach(const ExactArgs& A0, int conn, int rounds, int big_groups, hipStream_t s) {
    ExactArgs A = A0;
    const int NB = ((A.W + 7) >> 3) * ((A.H + 7) >> 3);
    for (int r = 0; r < rounds; ++r) {
        A.round = r;
        hipLaunchKernelGGL(k_exact_round, dim3((unsigned)((NB + 255) / 256)), dim3(256), 0, s, A);
        if (conn == 4) {
            hipLaunchKernelGGL(k_exact_reach<4>, dim3((unsigned)A.N), dim3(ReachMost::NT), 0, s, A);
            hipLaunchKernelGGL(k_exact_reach_wide<4>, dim3(256), dim3(ReachWide::NT), 0, s, A);
            hipLaunchKernelGGL(k_exact_reach_big<4>, dim3((unsigned)big_groups), dim3(512), 0, s, A);
        } else {
            hipLaunchKernelGGL(k_exact_reach<8>, dim3((unsigned)A.N), dim3(ReachMost::NT), 0, s, A);
            hipLaunchKernelGGL(k_exact_reach_wide<8>, dim3(256), dim3(ReachWide::NT), 0, s, A);
            hipLaunchKernelGGL(k_exact_reach_big<8>, dim3((unsigned)big_groups), dim3(512), 0, s, A);
        }
        hipLaunchKernelGGL(k_exact_offsets, dim3(1), dim3(1024), 0, s, A);
        hipLaunchKernelGGL(k_exact_place, dim3(2048), dim3(256), 0, s, A);
        const dim3 g(r == 0 ? (unsigned)NB * 64u : std::min((unsigned)NB * 64u, 8192u));
        if (A.K <= 64) hipLaunchKernelGGL(k_exact_nearest<64>, g, dim3(64), 0, s, A);
        else hipLaunchKernelGGL(k_exact_nearest<128>, g, dim3(64), 0, s, A);
    }
    return hipGetLastError();
}

}  // namespace epic

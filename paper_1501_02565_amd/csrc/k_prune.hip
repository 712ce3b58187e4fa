// k_prune.hip -- the consistency check of the matches (Sec. 5.1 of the
// paper, "Pruning of matches"): the interpolation is run once with the
// Nadaraya-Watson estimator, and the matches whose displacement differs from
// that first estimate at their own pixel by more than a threshold are
// removed before the interpolation proper.
//
// At the pixel of match m the NW field is the model of cell m, whose value
// there is its constant c_m, so the test only needs the per-match models of
// the first pass: m is kept when it was placed on its pixel and
// |u_m - c_m| <= threshold (Euclidean norm, evaluated in double from the
// FP32 model).  The K-NN + fit kernel of the first pass takes that decision
// right after the fit and leaves a flag per match; k_prune compacts the
// kept matches in index order (so ties keep breaking towards the lower
// original index) and points the pair's descriptor at them: the second
// pass of every kernel then sees N' matches.  The first pass's drop counts
// and status are saved in counters the second pass keeps.
#include "epic_dev.h"
#include "wave.h"

namespace epic {

// One workgroup of 1024 threads per pair.  The matches are taken in groups of
// PRUNE_R segments of 1024, one match per thread and segment, the flags and
// rows of a group in flight together; ballots count the kept ones of each
// wavefront and segment, and every wavefront scans the group's counts to place
// its own.  Bound by the latency of a group's loads: 10000 matches 7.4 us, where
// threads that owned a contiguous chunk each, match by match, took 18.1.
constexpr int PRUNE_R = 8;

__global__ __launch_bounds__(1024) void k_prune(PairDev* __restrict__ pairs, RunDev run) {
    PairDev& P = pairs[blockIdx.x];
    static_assert(PRUNE_R * 16 == 128, "two counts per lane");
    __shared__ int s_wave[PRUNE_R * 16];
    const int tid = threadIdx.x, lane = tid & 63, wid = __builtin_amdgcn_readfirstlane(tid >> 6);
    const u32 N = (u32)P.N;
    const float4* rows = reinterpret_cast<const float4*>(P.matches);
    int total = 0;
    for (u32 g0 = 0; g0 < N; g0 += PRUNE_R * 1024u) {
        // keep flags left by the first pass's K-NN + fit (0 for matches that
        // were not placed on their pixel)
        u32 flag[PRUNE_R];
        float4 row[PRUNE_R];
#pragma unroll
        for (int r = 0; r < PRUNE_R; ++r) {
            const u32 m = g0 + r * 1024u + tid;
            flag[r] = 0u;
            row[r] = make_float4(0.f, 0.f, 0.f, 0.f);
            if (m < N) {
                flag[r] = P.fill[m];
                row[r] = gload(rows + m);
            }
        }
        u64 kept[PRUNE_R];
#pragma unroll
        for (int r = 0; r < PRUNE_R; ++r) {
            kept[r] = wave::ballot(flag[r] != 0u);
            if (lane == 0) s_wave[r * 16 + wid] = (int)__popcll(kept[r]);
        }
        __syncthreads();
        const int s0 = s_wave[2 * lane], s1 = s_wave[2 * lane + 1];
        const int incl = wave::incl_scan(s0 + s1);
        // kept before count 2 lane + (wid & 1)
        const int e = total + incl - s1 - (wid & 1 ? 0 : s0);
#pragma unroll
        for (int r = 0; r < PRUNE_R; ++r) {
            // (read before the lanes part)
            const int before = __builtin_amdgcn_readlane(e, (r * 16 + wid) >> 1);
            if (flag[r] == 0u) continue;
            const int m = (int)(g0 + r * 1024u) + tid;
            const int pos = before + (int)__popcll(kept[r] & ((1ull << lane) - 1ull));
            gstore(reinterpret_cast<float4*>(P.matches_kept) + pos, row[r]);
            P.kept_idx[pos] = m;
            if (P.dbg_kept) P.dbg_kept[pos] = m;
        }
        total += __builtin_amdgcn_readlane(incl, 63);
        __syncthreads();             // s_wave is written again
    }
    __syncthreads();                 // every thread is done with the first pass's N and rows
    if (tid == 0) {
        int* c = P.counters;
        c[C_PRUNED] = c[C_USED] - total;
        c[C_OUTSIDE0] = c[C_OUTSIDE];
        c[C_DUP0] = c[C_DUPLICATE];
        // a first-pass model that a K-NN overflow left at zero decided a
        // match: report the capacity error of that pass
        c[C_STATUS0] = c[C_STATUS] != 0 ? c[C_STATUS] : ((c[C_OVERFLOW] & 2) ? -6 : 0);
        if (P.dbg_n_kept) *P.dbg_n_kept = total;
        P.N = total;
        P.matches = P.matches_kept;
    }
}

hipError_t launch_prune(PairDev* d_pairs, const RunDev& run, hipStream_t s) {
    hipLaunchKernelGGL(k_prune, dim3(run.npairs), dim3(1024), 0, s, d_pairs, run);
    return hipGetLastError();
}

}  // namespace epic

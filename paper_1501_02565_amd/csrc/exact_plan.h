// exact_plan.h -- which form epic_interp_exact takes after its bounds, and
// where the per-match form (k_exact_reach.hip) keeps its arrays in the
// workspace.  Host code without HIP.
#pragma once

#include <algorithm>
#include <cstddef>
#include <cstdint>

namespace epic {

constexpr size_t kAlign = 256;
inline size_t align_up(size_t v) { return (v + kAlign - 1) & ~(kAlign - 1); }

constexpr int kExactRounds = 8;        // rounds of the per-match form, at most
constexpr int kExactGroups = 256;      // workgroups for the sources that outgrow LDS, at most
constexpr size_t kExactCtl = 96;       // its control words

struct ExactPlan {
    int rounds = 0;                    // 0: the batched transforms (k_exact.hip)
    int big_groups = 0;
    uint32_t pool_cap = 0;             // entries
    size_t scratch_words = 0;          // per workgroup of big_groups
    // offsets in the workspace
    size_t cu = 0, ctl = 0, pend[2] = {0, 0}, wide = 0, big = 0, bcount = 0, offset = 0;
    size_t scratch = 0, meta = 0, order = 0, pool = 0;
};

// begin: the first free byte; used: the end of what the approximated pass
// left there (read by the bounds, over before the entries come); tail: the
// pixels' lists and what follows them.
//
// The entries' pool must take the worst case (every match reaching every
// block of 8 x 8 pixels) in at most kExactRounds rounds.  Given that, the
// form is chosen by how far a match reaches.  A pixel has about 2 K matches
// within its bound, so a match reaches about 2 K / N of the blocks: `reach`
// (all of them when N <= 2 K).  The per-match form keeps a match's distances
// in LDS up to 271, then 543 blocks; one that reaches more is computed in
// memory, by one of kExactGroups workgroups, after both LDS sizes have been
// tried, and that a chip full of other matches has to hide.  Times in us,
// batched against per-match form (layered costs):
//   reach fits LDS   300 x 640,  N = 320, K = 16 (reach 304): 2024, 1261
//   and N >= reach   1024 x 436, N = 640, K = 16 (352): 4032, 2271;
//                    N = 500 (451): 3895, 3591; N = 256, K = 8 (440): 2683, 3160
//   reach more       1024 x 436, N = 768, K = 64 (1173): 12875, 12809; N = 512,
//                    K = 64 (1760): 12916, 13802; N = 64, K = 16 (3520): 5197, 13552;
//                    2048 x 1080, N = 1024, K = 128 (8640): 143730, 127609
//   image of few     96 x 128 (192 blocks), N = 16 .. 64, K = 16: 522, 419 .. 459, 296,
//   blocks           N = 8, K = 16: 436, 535; N = 12, K = 4 (128): 398, 319;
//                    64 x 64 (64), N = 8: 315, 232; 128 x 160 (320), N = 32, K = 16: 599, 758
// Matches that reach much also need the pool and the workgroups in full: a
// second round repeats what did not fit (1024 x 436, N = 768, K = 128 with
// room for 1, 1/2, 1/4, 1/7 of the worst case: 30144, 25627; 32424, 40709;
// 38984, 73250; 47610, 160899), where short reaches leave the pool half empty
// (300 x 640, N = 320, K = 16 with 1/7: 5840, 1380).
inline ExactPlan exact_plan(int H, int W, int N, int K, size_t begin, size_t used, size_t tail) {
    ExactPlan p;
    const ExactPlan batched;
    const long long bw = (W + 7) / 8, bh = (H + 7) / 8, nb = bw * bh;
    const size_t cu_b = align_up(8 * (size_t)H * W);
    if (tail < cu_b + begin) return batched;
    const size_t end = (tail - cu_b) & ~(kAlign - 1);
    size_t cur = begin;
    auto take = [&](size_t bytes) {
        const size_t at = cur;
        cur += align_up(bytes);
        return at;
    };
    p.cu = end;
    p.ctl = take(4 * kExactCtl);
    p.pend[0] = take(4 * (size_t)N);
    p.pend[1] = take(4 * (size_t)N);
    p.wide = take(4 * (size_t)N);
    p.big = take(4 * (size_t)N);
    p.bcount = take(4 * (size_t)nb);
    p.offset = take(4 * (size_t)nb);
    const size_t group_b = align_up(4 * ((size_t)(nb + 1) * 64 + 5 * (size_t)nb));
    p.scratch_words = group_b / 4;
    const size_t left = end > cur ? end - cur : 0;
    p.big_groups = (int)std::min<size_t>(kExactGroups, left / 4 / group_b);
    // 16 + 8 + 256 bytes an entry, and the arrays' alignment
    const size_t entries_b = left - (size_t)p.big_groups * group_b;
    const long long cap = entries_b > 3 * kAlign ? (long long)((entries_b - 3 * kAlign) / 280) : 0;
    const long long per_round = cap / nb - 1;               // matches a round places at least
    if (p.big_groups < 1 || per_round < 1 || end < used) return batched;
    // a launch has fewer than 2^32 threads: 1024 a match, 64 a pixel of the
    // blocks (the batched form takes matches in chunks, and 64 a pixel of the
    // image)
    if (N >= 1 << 22 || nb >= 1 << 20) return batched;
    // 32-bit entries, 16-bit block coordinates
    if (cap >= (1LL << 31) || (long long)N * nb >= (1LL << 31) || bw >= 65536 || bh >= 65536) return batched;
    const long long rounds = (N + per_round - 1) / per_round;
    if (rounds > kExactRounds) return batched;
    const long long reach = N <= 2LL * K ? nb : (2LL * K * nb + N - 1) / N;
    const bool in_lds = N >= 16 ? std::min(nb, 2 * reach) <= 256 : reach <= 128;
    const bool room = reach <= 352 || (p.big_groups == kExactGroups && cap >= 2LL * N * reach);
    if (!in_lds && !(N >= std::min(reach, 768LL) && room)) return batched;
    p.rounds = (int)rounds;
    p.pool_cap = (uint32_t)cap;
    p.scratch = take((size_t)p.big_groups * group_b);
    p.meta = take(16 * (size_t)cap);
    p.order = take(8 * (size_t)cap);
    p.pool = take(256 * (size_t)cap);
    return p;
}

}  // namespace epic

// How a block's two weight gradients share a launch of wgrad_rd_kernel (host side, no HIP: kernels_wgr.hip).
#pragma once
#include <algorithm>
#include <climits>

namespace mbk {

// One of them: 64 x 64 tiles, chunks of the contraction, cycles a chunk takes, and the most splits it may have.
struct WgrSide {
    int tiles, chunks, cost, most;
    // the fewest splits whose longest one takes at most `bound` cycles
    int splits(long long bound) const
    {
        const long long per = bound / cost; // chunks of a split
        return per ? (int)((chunks + per - 1) / per) : INT_MAX;
    }
};

// Of the numbers of splits with which all workgroups are resident at once, the pair whose slower side ends first,
// and of those the one with the fewest workgroups.  Both counts only fall as the time allowed grows, so that
// time is found by halving: a few dozen divisions a call.  (Every pair in turn, up to 640 x 640, is the same answer
// after as much as 1 ms, where the backward pass it plans takes a few hundred microseconds: 8 -> 48 -> 8 on 46 planes of
// 81x81, training step 413 us before such a search, 1039 with it.)
inline void wgr_pair_splits(const WgrSide &a, const WgrSide &b, int resident, int *sa, int *sb)
{
    const auto fits = [&](long long bound) {
        const int i = a.splits(bound), j = b.splits(bound);
        return i <= a.most && j <= b.most && (long long)i * a.tiles + (long long)j * b.tiles <= resident;
    };
    // one split each takes `hi`, and is the answer where even that does not fit
    long long lo = 0, hi = std::max((long long)a.chunks * a.cost, (long long)b.chunks * b.cost);
    while (fits(hi) && hi - lo > 1) {
        const long long mid = lo + (hi - lo) / 2;
        if (fits(mid))
            hi = mid;
        else
            lo = mid;
    }
    *sa = a.splits(hi);
    *sb = b.splits(hi);
}

} // namespace mbk

// The search of one hop of a shard's walk from micro-batch to micro-batch, shared by the plan's kernels.  Nothing in it
// needs the device: where the prefix is probed is the caller's.
#pragma once

namespace dc {

// The end of the micro-batch that opens at slot j of a shard of n slots (j < n): the last e in (j, n] whose prefix fits,
// or j + 1 if there is none (an over-budget slot still advances by one).  sz: slots in the micro-batch before it (0: none).
// G = 1 << lg_G lanes probe at once; the prefix sums do not decrease, so the places that fit come first and their number
// is all that is needed:
//   count(c, step, last, inside): how many of the G places c, c + step, c + 2 step, ... fit, where a place beyond `last`
//   stands for `last` or, with `inside`, does not fit.  No place beyond n is asked for: the words behind a shard's end
//   belong to the next shard, or to nobody.
// The first window probes G slots one by one, placed around the end that a micro-batch as long as the one before would have
// (slots of a shard mostly come in descending length, so it holds a few more; the first one of a shard: the G slots behind
// the start).  Most micro-batches end inside it; if not, the lanes spread evenly over what is left on the side where the
// end lies, then over the stretch between the last probe that fits and the first that does not.
template <typename Count>
__device__ __forceinline__ int next_fit_end(int G, int lg_G, int j, int sz, int n, Count count) {
    const int first = max(j + 1, j + sz + 1 - (G >> 2));
    int lo, hi = n, e = j + 1;                           // candidates [lo, hi]; everything below lo fits
    {
        const int cnt = count(first, 1, n, true);
        if (cnt == 0) { lo = j + 1; hi = min(first - 1, n); }    // it ends before the window (which may lie beyond the shard's end)
        else { e = first + cnt - 1; lo = (cnt == G && first + G <= n) ? first + G : n + 1; }      // n + 1: found
    }
    while (lo <= hi) {
        const int S = (hi - lo + G) >> lg_G;             // ceil(candidates / G) >= 1
        const int cnt = count(lo + S - 1, S, hi, false);
        if (cnt > 0) e = min(lo + cnt * S - 1, hi);
        if (cnt == G) break;                             // the last lane's probe is hi itself
        hi = min(lo + (cnt + 1) * S - 1, hi) - 1;
        lo += cnt * S;
    }
    return e;
}

}  // namespace dc

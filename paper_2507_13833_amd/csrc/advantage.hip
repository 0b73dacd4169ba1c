// Group-relative advantage (the GRPO "advantage" stage, App. B Table 2; advantages
// are part of the payload the Data Coordinator moves, Sec. 1) fused with its
// broadcast over the rollout layout's tokens.
//
// One launch, one wavefront per sequence.  The wave finds the sequence's prompt group,
// recomputes the group's mean and std from its G rewards (float64, in index order;
// cheaper than a second launch or a grid-wide dependency), writes adv_seq[i] and then
// streams the sequence's own token range: 4 mask bytes in, 16 bytes of float32 out per
// lane and step (5 B/token, HBM-bound).  A sequence is one contiguous run in its
// rollout shard, so no lane ever has to search for the sequence a token belongs to.
#include <algorithm>
#include "advantage_device.h"

namespace dc {

constexpr int ADV_BLOCK = 256;
constexpr int ADV_WAVES = ADV_BLOCK / WAVE;

__global__ __launch_bounds__(ADV_BLOCK) void advantage_kernel(AdvArgs a, SourceDesc sd) {
    advantage_wave(a, sd, (int64_t)blockIdx.x * ADV_WAVES + __builtin_amdgcn_readfirstlane((int)(threadIdx.x / WAVE)));   // one wave per sequence
}

// The stage for many short sequences: a wave takes SEQS consecutive ones, lane k finds sequence k's place, group and
// advantage by itself (the same sums in the same order), and the wave then streams their tokens, four sequences' mask
// words in flight at a time, the first four's asked for ahead of the statistics.
// With a wave per sequence every lane of it works out the same statistics, ~350 vector instructions in float64 for a
// sequence whose tokens take ten, and 65 536 of those are the stage's time: 69.0 us for 28 M tokens in 65 536 sequences, 43.3
// with eight to a wave.  A wave waits for nothing but its groups' loads: while the ragged heads and tails, three tokens each,
// were read where they are written, each such read waited for the stores in front of it (31 M tokens in 65 536 sequences 48.0
// us, now 44.1; sequences that all have one length, and no ragged ends, lose 1 to 5 %: 32 768 of 300 18.4, now 19.3).  Below 16 384 sequences there are not enough waves left (8192
// of 57 tokens 10.4 -> 11.4), and longer ones want their tokens spread over more waves; the line is the mean above which
// the stage with a quarter of its sequences past the four steps is slower so (16 384 of 326 18.3 / 18.4, of 469 20.6 / 22.9;
// 24 576 of 416 27.1 / 27.8, of 678 32.2 / 34.8; 32 768 of 792 44.0 / 41.3; 49 152 of 998 69.3 / 68.5).
// Four to a wave where eight leave too few waves (us with eight and with four, groups of 8): 16 384 of 20 tokens 11.3 / 10.4, of
// 300 14.4 / 13.1; 20 480 of 20 12.1 / 11.5, of 300 16.1 / 14.5; 24 576 of 20 12.1 / 12.7, of 300 19.1 / 16.4; 32 760 of 20
// 13.7 / 15.5, of 200 17.2 / 17.8, of 300 21.2 / 20.0; 40 000 of 300 24.0 / 25.3.  Every wave works its groups out for itself, so
// not with large groups: 20 480 of 200 in groups of 16 14.9 / 15.1, of 64 21.7 / 23.8, of 1024 168 / 204.
// Long sequences are not a single wave's: the first ADV_SETS workgroups look for them, each in a set of its own (of
// neighbours, as the answers to one prompt are, every one in another set), and take them with all their waves and
// ADV_UNROLL steps in flight.  16 384 sequences of 190 tokens, 64 of 32 K among them: 28.9 us with a wave per sequence, 17.9
// here (64 at a stretch: 22.4 and 17.2), where the wave that met them took 98 and 450.
constexpr int ADV_GROUP = 4;                           // sequences in flight
constexpr int ADV_STEPS = 4;                           // 4-token chunks per lane of one of them in flight
constexpr int ADV_REST = 8;                            // the same of a longer one's rest
constexpr int ADV_LONG = 4096;                         // tokens from which a sequence is a long one
constexpr int ADV_SETS = 509;                          // (half as many: a Pareto tail of 65 536 of 786 tokens 102 us instead of
                                                       // 83; a prime, so that one long answer to every prompt is in every set)
constexpr int ADV_BRIEF_MIN_SEQ = 16384;               // a wave per sequence fills the chip's wave slots twice
constexpr int ADV_BRIEF_MAX_MEAN = ADV_STEPS * WAVE * 4;       // (what the four steps take)
constexpr int ADV_BRIEF_SEQ_PER_TOKEN = 48;            // sequences per token of the mean length, at least
// Four sequences to a wave instead of eight: below the first line, or below the second if the sequences are not very short;
// not where the groups are large, as every wave works out its groups' sums.
constexpr int ADV_FOUR_MAX_SEQ = 22528, ADV_FOUR_LONGER_MAX_SEQ = 32768;
constexpr int ADV_FOUR_LONGER_MIN_MEAN = 225;
constexpr int ADV_FOUR_MAX_GROUP = 16;                 // responses to a prompt, on average

__device__ __forceinline__ bool adv_long(int32_t ln) { return ln >= ADV_LONG && ln <= DC_MAX_SEQ_LEN; }

// (bounded to eight waves to a SIMD: the long ones' code alone would take the scalar registers of one of them)
template <int SEQS>
__global__ __launch_bounds__(ADV_BLOCK, 8) void advantage_brief_kernel(AdvArgs a, SourceDesc sd) {
    static_assert(SEQS % ADV_GROUP == 0 && SEQS <= WAVE, "a lane per sequence");
    const int lane = threadIdx.x & (WAVE - 1);
    const int w = __builtin_amdgcn_readfirstlane((int)(threadIdx.x / WAVE));
    const int N = a.n_seq;
    if (blockIdx.x < ADV_SETS) {                                     // (uniform) long ones, by the workgroup's waves together
        __shared__ uint64_t found[ADV_WAVES];
        for (int64_t base = blockIdx.x; base < N; base += (int64_t)ADV_BLOCK * ADV_SETS) {
            const int64_t at = base + (int64_t)threadIdx.x * ADV_SETS;
            const uint64_t mine = __ballot(adv_long(at < N ? a.seq_len[at] : 0));
            if (lane == 0) found[w] = mine;
            lds_barrier();
#pragma unroll 1
            for (int q = 0; q < ADV_WAVES; ++q) {
                for (uint64_t left = wave_read_lane(found[q], 0); left != 0ull; left &= left - 1ull)      // (uniform)
                    advantage_sequence<ADV_WAVES>(a, sd, (int)base + (q * WAVE + __ffsll((long long)left) - 1) * ADV_SETS, w);
            }
            lds_barrier();
        }
        return;
    }
    const int64_t first = ((int64_t)(blockIdx.x - ADV_SETS) * ADV_WAVES + w) * SEQS;
    if (lane < SEQS && first + lane <= a.n_groups) {             // group table: [0] = 0, non-decreasing, last = N
        const int g = (int)first + lane;
        const int32_t v = a.group_off[g];
        bool bad = v < 0 || v > N || (g == 0 && v != 0) || (g == a.n_groups && v != N);
        if (g < a.n_groups && a.group_off[g + 1] < v) bad = true;
        if (bad) set_status(a.status, DC_ERR_BAD_LAYOUT);
    }
    if (first >= N) return;
    // ---- lane k: sequence first + k (lanes beyond the last one repeat it and store nothing) ----
    const int n = (int)min((int64_t)SEQS, N - first);            // (uniform)
    const int i = (int)first + min(lane, n - 1);
    const int64_t so = a.src_tok_off[i], so_next = a.src_tok_off[min(i + 1, N - 1)];
    const int32_t ln = a.seq_len[i];
    const bool lng = adv_long(ln), mine = lane < n && !lng;          // (a long one is done above)
    const double ri = (double)a.reward[i];
    int g = min((int)(((int64_t)i * a.n_groups) / N), max(a.n_groups - 1, 0));     // where it is if all groups have the same size
    int g0 = a.group_off[g], g1 = a.group_off[min(g + 1, a.n_groups)];
    if (a.n_groups > 0 && (i < g0 || i >= g1)) {
        int lo = 0, hi = a.n_groups;                    // invariant: group_off[lo] <= i
        while (hi - lo > 1) {
            const int mid = (lo + hi) >> 1;
            if (a.group_off[mid] <= i) lo = mid; else hi = mid;
        }
        g0 = a.group_off[lo];
        g1 = a.group_off[lo + 1];
    }
    int s = 0;                                           // (seq_off[k] = N from k = n_src on)
    int64_t buf_tokens = sd.tokens[0];
    int32_t buf_end = sd.seq_off[1];
#pragma unroll
    for (int k = 1; k < DC_MAX_SRC_SHARDS; ++k)
        if (i >= sd.seq_off[k]) { s = k; buf_tokens = sd.tokens[k]; buf_end = sd.seq_off[k + 1]; }
    const bool bad_len = ln <= 0 || ln > DC_MAX_SEQ_LEN;
    const bool bad_off = !bad_len && (so < 0 || so + ln > buf_tokens || (i + 1 < buf_end && so_next < so + ln));
    if (mine && bad_len) set_status(a.status, DC_ERR_ZERO_LENGTH_SEQ);
    if (mine && bad_off) set_status(a.status, DC_ERR_BAD_LAYOUT);
    const bool none = bad_len || bad_off || lng;                     // nothing to write here
    const int64_t begin = so, end = none ? so : so + ln;

    // ---- the wave's view of sequence k ----
    // (all of it uniform; lanes add 32-bit offsets, so an access costs no address arithmetic of its own)
    struct Seq {
        const uint8_t* mask;                                          // of its first token
        float* out;
        int32_t a4, e4, end;                                          // ragged head up to a4, body in whole 16-byte chunks, ragged tail from e4
    };
    auto seq = [&](int k) {
        Seq q;
        const int sh = __builtin_amdgcn_readlane(s, k);
        const int64_t at = wave_read_lane(begin, k);
        q.mask = a.mask[sh] + at;
        q.out = a.adv_tok[sh] + at;
        q.end = (int32_t)(wave_read_lane(end, k) - at);
        const int32_t head = (int32_t)(-at) & 3;
        q.a4 = min(q.end, head);
        q.e4 = max(q.a4, ((q.end - head) & ~3) + head);
        return q;
    };
    uint32_t mk[ADV_GROUP][ADV_STEPS];
    uint32_t ends[ADV_GROUP];                                        // lanes 0 .. 2: the head's mask bytes, 32 .. 34: the tail's
    auto end_token = [&](const Seq& q) {                             // (-1: none)
        const int32_t t = lane < 32 ? lane : q.e4 + (lane - 32);
        return (lane & 31) < 3 && t < (lane < 32 ? q.a4 : q.end) ? t : -1;
    };
    auto load_group = [&](int k0) {
#pragma unroll
        for (int k = 0; k < ADV_GROUP; ++k) {
            if (k0 + k >= n) continue;                               // (uniform)
            const Seq q = seq(k0 + k);
#pragma unroll
            for (int u = 0; u < ADV_STEPS; ++u) {
                const uint32_t c = (uint32_t)(u * WAVE + lane) * 4u;
                mk[k][u] = (int32_t)c < q.e4 - q.a4 ? load4(q.mask + q.a4 + c) : 0u;
            }
            const int32_t t = end_token(q);
            ends[k] = 0;
            if (t >= 0) ends[k] = q.mask[(uint32_t)t];
        }
    };
    load_group(0);

    // ---- lane k: the advantage of its sequence, float64 in index order ----
    float adv = 0.0f;
    const int G = g1 - g0;
    if (a.n_groups > 0 && g0 >= 0 && g1 <= N && i >= g0 && i < g1) {  // (else a bad group table, flagged above)
        const uint32_t r0 = __float_as_uint(a.reward[g0]);
        bool same = true;
        double sum = 0.0;
        for (int q = g0; q < g1; ++q) {
            const float r = a.reward[q];
            same = same && __float_as_uint(r) == r0;
            sum += (double)r;
        }
        if (!same && G - a.ddof > 0) {
            const double mean = sum / (double)G;
            double ss = 0.0;
            for (int q = g0; q < g1; ++q) {
                const double d = (double)a.reward[q] - mean;
                ss += d * d;
            }
            adv = (float)((ri - mean) / (sqrt(ss / (double)(G - a.ddof)) + a.eps));
        }
    }
    if (mine) a.adv_seq[i] = adv;

    // ---- the tokens ----
#pragma unroll
    for (int k0 = 0; k0 < SEQS; k0 += ADV_GROUP) {
        if (k0 >= n) break;                                           // (uniform)
        if (k0 > 0) load_group(k0);
#pragma unroll
        for (int k = 0; k < ADV_GROUP; ++k) {
            if (k0 + k >= n) continue;                               // (uniform)
            const Seq q = seq(k0 + k);
            const uint32_t av = (uint32_t)__builtin_amdgcn_readlane((int)__float_as_uint(adv), k0 + k);
            const int32_t t = end_token(q);
            if (t >= 0) q.out[(uint32_t)t] = ends[k] ? __uint_as_float(av) : 0.0f;
#pragma unroll
            for (int u = 0; u < ADV_STEPS; ++u) {
                const uint32_t c = (uint32_t)(u * WAVE + lane) * 4u;
                if ((int32_t)c < q.e4 - q.a4) store16(q.out + q.a4 + c, select_by_mask(mk[k][u], av));
            }
            for (int32_t c0 = q.a4 + ADV_STEPS * WAVE * 4; c0 < q.e4; c0 += ADV_REST * WAVE * 4) {       // (uniform) a longer one's rest
                uint32_t more[ADV_REST];
#pragma unroll
                for (int u = 0; u < ADV_REST; ++u) {
                    const uint32_t c = (uint32_t)(u * WAVE + lane) * 4u;
                    more[u] = (int32_t)c < q.e4 - c0 ? load4(q.mask + c0 + c) : 0u;
                }
#pragma unroll
                for (int u = 0; u < ADV_REST; ++u) {
                    const uint32_t c = (uint32_t)(u * WAVE + lane) * 4u;
                    if ((int32_t)c < q.e4 - c0) store16(q.out + c0 + c, select_by_mask(more[u], av));
                }
            }
        }
    }
}

AdvArgs make_adv_args(int32_t n_seq, const SourceDesc& src, const int64_t* d_src_tok_off, const int32_t* d_seq_len,
                      const float* d_reward, const int32_t* d_group_off, int32_t n_groups, double eps, int32_t ddof,
                      const uint8_t* const* mask_base, float* d_adv_seq, float* const* adv_tok_base, int32_t* d_status) {
    AdvArgs a;
    a.n_seq = n_seq; a.n_groups = n_groups; a.ddof = ddof; a.eps = eps;
    a.src_tok_off = d_src_tok_off; a.seq_len = d_seq_len; a.reward = d_reward; a.group_off = d_group_off;
    a.adv_seq = d_adv_seq; a.status = d_status;
    a.per_token = adv_tok_base != nullptr;
    for (int s = 0; s < DC_MAX_SRC_SHARDS; ++s) {
        a.mask[s] = (a.per_token && s < src.n_src) ? mask_base[s] : nullptr;
        a.adv_tok[s] = (a.per_token && s < src.n_src) ? adv_tok_base[s] : nullptr;
    }
    return a;
}

hipError_t launch_advantage(int32_t n_seq, const SourceDesc& src, const int64_t* d_src_tok_off,
                            const int32_t* d_seq_len, const float* d_reward, const int32_t* d_group_off,
                            int32_t n_groups, double eps, int32_t ddof,
                            const uint8_t* const* mask_base, float* d_adv_seq, float* const* adv_tok_base,
                            int32_t* d_status, hipStream_t st) {
    const AdvArgs a = make_adv_args(n_seq, src, d_src_tok_off, d_seq_len, d_reward, d_group_off, n_groups, eps, ddof,
                                    mask_base, d_adv_seq, adv_tok_base, d_status);
    int64_t tokens = 0;
    for (int s = 0; s < src.n_src; ++s) tokens += src.tokens[s];
    if (a.per_token && n_seq >= ADV_BRIEF_MIN_SEQ && tokens / n_seq <= std::min(ADV_BRIEF_MAX_MEAN, n_seq / ADV_BRIEF_SEQ_PER_TOKEN)) {
        auto launch = [&](auto kernel, int seqs) {
            const int64_t blocks = (adv_waves(n_seq, n_groups) + ADV_WAVES * seqs - 1) / (ADV_WAVES * seqs);
            hipLaunchKernelGGL(kernel, dim3((unsigned)blocks + ADV_SETS), dim3(ADV_BLOCK), 0, st, a, src);
        };
        const bool four = (int64_t)n_groups * ADV_FOUR_MAX_GROUP >= n_seq &&
                          (n_seq < ADV_FOUR_MAX_SEQ || (n_seq < ADV_FOUR_LONGER_MAX_SEQ && tokens / n_seq >= ADV_FOUR_LONGER_MIN_MEAN));
        if (four) launch(advantage_brief_kernel<4>, 4);
        else launch(advantage_brief_kernel<8>, 8);
        return hipGetLastError();
    }
    const int64_t grid = (adv_waves(n_seq, n_groups) + ADV_WAVES - 1) / ADV_WAVES;
    hipLaunchKernelGGL(advantage_kernel, dim3((unsigned)grid), dim3(ADV_BLOCK), 0, st, a, src);
    return hipGetLastError();
}

}  // namespace dc

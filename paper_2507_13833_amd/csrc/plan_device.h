// The plan proper (dense prefix of the slot lengths, shard bases, next-fit micro-batches, per-slot outputs)
// as device code of one workgroup of PLAN_BLOCK lanes, shared by plan_kernel (a launch of its own behind
// slots_kernel) and by the launch that runs it as the tail of the balance workgroup.
#pragma once
#include "dc_device.h"
#include "dc_internal.h"
#include "dc_lanes.h"
#include "plan_walk.h"

namespace dc {

constexpr int PLAN_BLOCK = 1024;
constexpr int PLAN_WAVES = PLAN_BLOCK / WAVE;
constexpr int PLAN_IPT = DC_MAX_SEQ / PLAN_BLOCK;        // slots per lane at the size limit
constexpr int PLAN_WORDS = DC_MAX_SEQ / 32;
constexpr int PLAN_NEXT_MAX = DC_MAX_SEQ / 2;            // slots up to which the unused end of the prefix holds a word per slot

// The place of sequence i in the rollout layout, validated, from its length and its element offset as they were read
// (placed: i is a sequence at all); see slot_source.
__device__ __forceinline__ void slot_source_of(const PlanArgs& a, const SourceDesc& sd, int32_t i, bool placed, int32_t ln, int64_t so,
                                               int32_t* ln_out, int64_t* so_out, int32_t* sh_out) {
    int32_t sh = 0;                                      // rollout shard (seq_off[s] = N from s = n_src on)
    if (sd.n_src > 1 && placed) {
#pragma unroll
        for (int s = 1; s < DC_MAX_SRC_SHARDS; ++s) sh += i >= sd.seq_off[s] ? 1 : 0;
    }
    int64_t tokens = sd.tokens[0];
#pragma unroll
    for (int s = 1; s < DC_MAX_SRC_SHARDS; ++s) tokens = sh == s ? sd.tokens[s] : tokens;
    const bool bad_len = placed && (ln <= 0 || ln > DC_MAX_SEQ_LEN);
    const bool bad_off = placed && !bad_len && (so < 0 || so + ln > tokens);
    const bool over = placed && !bad_len && !bad_off && ln > a.budget;   // still laid out, alone in its micro-batch
    const int32_t e = !placed ? DC_ERR_BAD_LAYOUT
                      : bad_len ? DC_ERR_ZERO_LENGTH_SEQ
                      : bad_off ? DC_ERR_BAD_LAYOUT
                      : over ? DC_ERR_SEQ_EXCEEDS_BUDGET : 0;
    if (e != 0) set_status(a.status, e);
    if (!placed || bad_len || bad_off) ln = 0;
    *ln_out = ln;
    *so_out = placed ? so : 0;
    *sh_out = sh;
}

// The sequence behind slot j with its place in the rollout layout, validated (what the gather may rely
// on): ln = tokens to move (0 if a check fails), so = element offset in rollout shard sh.  ln_in < 0: the
// length is taken from a.seq_len; else it is the slot's length as the caller has it already.  Sets the
// device status on a failed check (and on a sequence above the token budget, which is still laid out).
__device__ __forceinline__ void slot_source(const PlanArgs& a, const SourceDesc& sd, int j, int32_t ln_in,
                                            int32_t* ln_out, int64_t* so_out, int32_t* sh_out) {
    const int32_t i = a.perm ? a.perm[j] : j;                                     // no permutation: slot j holds sequence j
    const bool placed = i >= 0 && i < a.n_seq;
    const int32_t ln = placed ? (ln_in < 0 ? a.seq_len[i] : ln_in) : 0;
    const int64_t so = placed ? a.src_tok_off[i] : 0;
    slot_source_of(a, sd, i, placed, ln, so, ln_out, so_out, sh_out);
}

struct PlanLds {
    int64_t  gpre[DC_MAX_SEQ + 1];          // dense exclusive prefix of slot lengths
    uint32_t start_bits[PLAN_WORDS];        // slot opens a micro-batch
    uint32_t seen_bits[PLAN_WORDS];         // sequence already placed (perm must be a permutation)
    int32_t  word_starts[PLAN_WORDS + 1];   // starts in the words before this one
    int32_t  word_last[PLAN_WORDS];         // last start in the words before this one, or -1
    int64_t  wave_pref[PLAN_IPT * PLAN_WAVES];  // tokens before the 64 slots a wave handles in one step
    int64_t  shard_shift[DC_MAX_SHARDS];    // aligned token offset of each shard minus its dense one
    int32_t  shard_off[DC_MAX_SHARDS + 1];  // copy of shard_seq_off
    int64_t  tmp64[16];
    int32_t  tmp32[16];
    int32_t  ok;
    int64_t  end;                           // d_shard_tok_off[P]
};


// The caller holds, per lane, the sequence and the (validated) length of slots tid, tid + PLAN_BLOCK, ...
// (seq = -1, len = 0 beyond N).  check_perm: seq comes from a caller's permutation and must be checked;
// fixed_c > 0: shard p owns slots [p * fixed_c, (p + 1) * fixed_c) and a.shard_seq_off is not read.
// STEPS: how the unrolled passes over a lane's slots treat the steps beyond nb.  STEP_OVER: a test each; ALL: none, there are
// few or none of them (the steps then run into each other: 16 scans at once).  CHAINS = false: for more than PLAN_NEXT_MAX slots,
// without the code that such a batch never takes.
// Every lane of the workgroup must call it (barriers inside).
enum PlanSteps { STEP_OVER, ALL };
template <int IPT, PlanSteps STEPS = ALL, bool CHAINS = true>
__device__ __forceinline__ void plan_body(PlanLds& L, const PlanArgs& a, int32_t (&seq)[IPT], int32_t (&len)[IPT],
                                          bool check_perm, int fixed_c) {
    const int tid = threadIdx.x, lane = tid & (WAVE - 1), w = tid / WAVE;
    const int N = a.n_seq, P = a.n_shards;
    const int nb = (N + PLAN_BLOCK - 1) / PLAN_BLOCK;    // steps of 1024 slots, <= IPT

    for (int i = tid; i < PLAN_WORDS; i += PLAN_BLOCK) { L.start_bits[i] = 0; L.seen_bits[i] = 0; }
    if (tid == 0) L.ok = 1;
    lds_barrier();
    for (int p = tid; p <= P; p += PLAN_BLOCK) {         // P + 1 entries, P up to the block size
        if (fixed_c > 0) { L.shard_off[p] = p * fixed_c; continue; }        // (uniform) N == P * fixed_c: nothing to check
        const int32_t v = a.shard_seq_off[p];
        L.shard_off[p] = v;
        bool bad = v < 0 || v > N || (p == 0 && v != 0) || (p == P && v != N);
        if (p < P && a.shard_seq_off[p + 1] < v) bad = true;
        if (bad) L.ok = 0;
    }
    lds_barrier();
    if (tid == 0) *a.plan_ok = L.ok;                     // read by records_kernel
    if (!L.ok) {                                         // unusable shard table: plan nothing
        if (tid == 0) { set_status(a.status, DC_ERR_BAD_LAYOUT); *a.n_mb = 0; }
        return;
    }

    // ---- 1. permutation check, dense prefix of the slot lengths ----
    uint32_t dup = 0;                                    // bit q: perm repeats an earlier entry at my slot of step q
    if (check_perm) {                                    // (uniform)
#pragma unroll
        for (int q = 0; q < IPT; ++q) {
            const int32_t i = seq[q];                    // -1 beyond N; out-of-range entries were emptied by slots_kernel
            if (i >= 0 && i < N) dup |= ((atomicOr(&L.seen_bits[i >> 5], 1u << (i & 31)) >> (i & 31)) & 1u) << q;
        }
    }
    if (__ballot(dup != 0) != 0ull) {                    // uniform, rare: perm is not a permutation; a repeat moves nothing
        if (dup != 0) set_status(a.status, DC_ERR_BAD_LAYOUT);
#pragma unroll
        for (int q = 0; q < IPT; ++q)
            if ((dup >> q) & 1u) { len[q] = 0; a.slot_len[q * PLAN_BLOCK + tid] = 0; }
    }
    // dense prefix: inclusive scan inside each wave step (a wave's 64 slots hold < 2^31 tokens) ...
    int32_t inc[IPT];
    // (the loops' bodies stand in them, not in lambdas: 15.9 us for 16 384 slots in plan_kernel instead of 16.4)
#pragma unroll
    for (int q = 0; q < IPT; ++q)
        if (STEPS == ALL || q < nb) {
            inc[q] = (int32_t)wave_incl_scan_add_u32((uint32_t)len[q]);
            if (lane == WAVE - 1) L.wave_pref[q * PLAN_WAVES + w] = inc[q];
        }
    lds_barrier();
    // ... an exclusive scan of the 256 step totals in slot order (step q, wave w) ...
    {
        const int64_t v = tid < nb * PLAN_WAVES ? L.wave_pref[tid] : 0;
        int64_t total;
        const int64_t ex = block_excl_scan_add<int64_t>(v, L.tmp64, &total);
        if (tid < PLAN_IPT * PLAN_WAVES) L.wave_pref[tid] = ex;
        if (tid == 0) L.gpre[N] = total;
    }
    lds_barrier();
    // ... and their sum
    const int whole_steps = N / PLAN_BLOCK;              // (uniform) steps in which every lane has a slot
#pragma unroll
    for (int q = 0; q < IPT; ++q) {
        const int j = q * PLAN_BLOCK + tid;
        if (j < N) L.gpre[j] = L.wave_pref[q * PLAN_WAVES + w] + (inc[q] - len[q]);
    }
    lds_barrier();

    // ---- 2. shard bases: lane p takes shard p; exclusive scan of the loads rounded up to the alignment ----
    if (P <= WAVE) {                                     // (uniform) one wave holds every shard: no barrier, the others go on
        if (w == 0) {
            const int64_t first = lane < P ? L.gpre[L.shard_off[lane]] : 0;
            const int64_t load = lane < P ? L.gpre[L.shard_off[lane + 1]] - first : 0;
            const int64_t padded = a.align == 1 ? load : (load + a.align - 1) / a.align * a.align;   // (uniform)
            const int64_t inc = wave_incl_scan_add<int64_t>(padded);
            const int64_t end = (int64_t)(((uint64_t)(uint32_t)__builtin_amdgcn_readlane((int)((uint64_t)inc >> 32), WAVE - 1) << 32) |
                                          (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)inc, WAVE - 1));
            if (lane < P) { L.shard_shift[lane] = inc - padded - first; a.shard_tok_off[lane] = inc - padded; }
            if (lane == 0) {
                L.end = end;
                a.shard_tok_off[P] = end;
                a.dst_tok_off[N] = end;
                if (end > a.capacity) set_status(a.status, DC_ERR_OVERFLOW);
            }
        }
    } else {
        const int64_t first = tid < P ? L.gpre[L.shard_off[tid]] : 0;
        const int64_t load = tid < P ? L.gpre[L.shard_off[tid + 1]] - first : 0;
        const int64_t padded = (load + a.align - 1) / a.align * a.align;
        int64_t end;
        const int64_t base = block_excl_scan_add<int64_t>(padded, L.tmp64, &end);
        if (tid < P) { L.shard_shift[tid] = base - first; a.shard_tok_off[tid] = base; }
        if (tid == 0) {
            L.end = end;
            a.shard_tok_off[P] = end;
            a.dst_tok_off[N] = end;
            if (end > a.capacity) set_status(a.status, DC_ERR_OVERFLOW);
        }
    }

    // ---- 3. micro-batch starts ----
    bool chains = false;                                 // (uniform)
    if constexpr (CHAINS) {
        const uint64_t all_tokens = (uint64_t)L.gpre[N];
        chains = N <= PLAN_NEXT_MAX && all_tokens <= 0xFFFFFFFFull && all_tokens > (uint64_t)(4 + 4 * nb) * (uint64_t)P * (uint64_t)a.budget;
    }
    if (chains) {
        // Few slots and long chains: every slot finds the end of the micro-batch that would start with it (a bisection of
        // the prefix's low words, a lane's slots side by side), and lane p follows shard p's chain, one LDS read a hop.
        // A walk's hop (below) reads the start, probes a window and counts: 620 cycles against 250, but the search takes
        // 1.3 K for every 1024 slots, so it pays from about 4 + 4 hops per 1024 slots on.  2048 slots on 8 shards, 25 hops
        // each: 16.2 K -> 8.7 K cycles; 8192 on 32 shards with 23 hops, which the line leaves to the walk: 15.6 K -> 16.9 K.
        uint16_t* const next = reinterpret_cast<uint16_t*>(&L.gpre[PLAN_NEXT_MAX + 1]);
        const int span = fixed_c > 0 ? fixed_c : N;          // slots of a shard, at most
        const int first_step = 1 << (31 - __clz(max(span, 1)));
        auto low = [&](int at) { return reinterpret_cast<const uint32_t*>(&L.gpre[at])[0]; };
        constexpr int SIDE = 4;
        for (int q0 = 0; q0 < nb; q0 += SIDE) {              // (uniform)
            int lo[SIDE], hi[SIDE];
            uint32_t limit[SIDE];
#pragma unroll
            for (int i = 0; i < SIDE; ++i) {
                const int j = min((q0 + i) * PLAN_BLOCK + tid, N - 1);
                lo[i] = j + 1;
                hi[i] = min(N, j + span);
                limit[i] = (uint32_t)min((uint64_t)low(j) + (uint64_t)a.budget, (uint64_t)0xFFFFFFFFull);
            }
            for (int step = first_step; step >= 1; step >>= 1) {     // (uniform) the last e in (j, hi] that fits, or j + 1
#pragma unroll
                for (int i = 0; i < SIDE; ++i) {
                    const int c = lo[i] + step;
                    const uint32_t g = low(min(c, N));
                    if (c <= hi[i] && g <= limit[i]) lo[i] = c;
                }
            }
#pragma unroll
            for (int i = 0; i < SIDE; ++i) {
                const int j = (q0 + i) * PLAN_BLOCK + tid;
                if (j < N) next[j] = (uint16_t)lo[i];
            }
        }
        lds_barrier();
        if (tid < P) {
            const int b = L.shard_off[tid + 1];
            for (int j = L.shard_off[tid]; j < b;) {
                const int e = min((int)next[j], b);
                atomicOr(&L.start_bits[j >> 5], 1u << (j & 31));
                j = e;
            }
        }
    } else
    // Many shards: lane p walks shard p.
    // Each hop looks for the last slot that still fits under the budget.  Slots of a shard come in
    // descending length, so a micro-batch holds about as many slots as the one before it: the
    // search gallops outwards from that guess and bisects what is left (a few probes of the prefix
    // instead of log2 N per hop; the hops of a shard are one dependent chain).
    if (P <= PLAN_WAVES * 4) {
        // Few shards: a group of 32 or 16 LANES walks a shard (every wave takes 2 or 4 shards).  A
        // hop probes G slots at once, one per lane: the prefix sums do not decrease, so the lanes that still fit
        // are a prefix of the group and a ballot counts them - one LDS round trip per window where the
        // dependent probes of a bisection take six to eight.  (Not a whole wave per shard, even where there are
        // waves enough: a hop costs a wave the same instructions whatever its groups' width, sixteen waves
        // walking at once are bound by the compute unit's issue rate, and eight or fewer by a hop's latency,
        // which is the shorter of the two.)
        const int spw = P <= PLAN_WAVES ? 2 : 4;             // shards per wave
        const int G = WAVE / spw, g = lane / G, gl = lane - g * G;
        const int lg_G = spw == 2 ? 5 : 4;
        const uint64_t group_mask = (G == WAVE ? ~0ull : (1ull << G) - 1ull);
        const int p = w * spw + g;
        if (p < P) {
            const int b = L.shard_off[p + 1];
            int j = L.shard_off[p];
            int sz = 0;                                      // slots in the micro-batch before this one
            while (j < b) {                                  // uniform over the group
                if (gl == 0) atomicOr(&L.start_bits[j >> 5], 1u << (j & 31));
                const int64_t limit = L.gpre[j] + a.budget;
                const int e = next_fit_end(G, lg_G, j, sz, b, [&](int c, int step, int last, bool inside) {
                    c += gl * step;
                    const bool fits = (!inside || c <= last) && L.gpre[min(c, last)] <= limit;
                    return __popcll((__ballot(fits) >> (g * G)) & group_mask);
                });
                sz = e - j;
                j = e;
            }
        }
    } else if (tid < P) {
        const int b = L.shard_off[tid + 1];
        int j = L.shard_off[tid];
        int sz = 1;                                      // slots in the previous micro-batch
        while (j < b) {
            atomicOr(&L.start_bits[j >> 5], 1u << (j & 31));
            const int64_t limit = L.gpre[j] + a.budget;
            int lo = j + 1, hi = b;                      // largest e in [lo, hi] with gpre[e] <= limit; gpre[lo] may
                                                         // exceed it: an over-budget slot still advances by one
            int g = min(j + sz, b);
            if (g > lo) {
                if (L.gpre[g] <= limit) {
                    lo = g;
                    for (int w = 1; lo < hi; w <<= 1) {  // gallop up
                        g = min(lo + w, hi);
                        if (L.gpre[g] <= limit) lo = g; else { hi = g - 1; break; }
                    }
                } else {
                    hi = g - 1;
                    for (int w = 1; lo < hi; w <<= 1) {  // gallop down
                        g = max(hi + 1 - w, lo);
                        if (g == lo) break;
                        if (L.gpre[g] <= limit) { lo = g; break; }
                        hi = g - 1;
                    }
                }
            }
            while (lo < hi) {
                const int mid = (lo + hi + 1) >> 1;
                if (L.gpre[mid] <= limit) lo = mid; else hi = mid - 1;
            }
            sz = lo - j;
            j = lo;
        }
    }
    lds_barrier();

    // ---- 4. micro-batch index per slot, outputs ----
    // per word of 32 slots: starts in the words before it, and the last start before it
    int32_t M;
    {   // (the two scans share their barriers)
        const uint32_t bits = tid < PLAN_WORDS ? L.start_bits[tid] : 0u;
        const int32_t n_here = (int32_t)__popc(bits), last_here = bits ? tid * 32 + 31 - __clz(bits) : -1;
        const int32_t inc_n = wave_incl_scan_add<int32_t>(n_here), inc_l = wave_incl_scan_max(last_here);
        int32_t* tmp_l = reinterpret_cast<int32_t*>(L.tmp64);
        if (lane == WAVE - 1) { L.tmp32[w] = inc_n; tmp_l[w] = inc_l; }
        lds_barrier();
        int32_t before = inc_n - n_here, last = wave_shift_up1(inc_l, -1);
        M = 0;
        for (int i = 0; i < PLAN_WAVES; ++i) {
            const int32_t x = L.tmp32[i];
            if (i < w) { before += x; last = max(last, tmp_l[i]); }
            M += x;
        }
        if (tid < PLAN_WORDS) { L.word_starts[tid] = before; L.word_last[tid] = last; }
        if (tid == 0) L.word_starts[PLAN_WORDS] = M;
    }
    lds_barrier();
    // One slot per lane and step.  Nothing here depends on a lane's own condition except the stores of a last,
    // partial step: every slot of a micro-batch stores the micro-batch's first slot (the same word with the same
    // value), and every slot stores the cu_seqlens entry behind its own, which is either the entry that the next
    // slot stores too or the end of the micro-batch.  Differences of prefix sums inside a micro-batch fit 32 bits,
    // so they are taken between the low words.
    const bool shift_bases = a.align != 1;               // (uniform)
    auto low_word = [&](int at) { return reinterpret_cast<const uint32_t*>(&L.gpre[at])[0]; };
    // (equal shards: slot j stands in shard j / fixed_c; one division per lane, then steps of PLAN_BLOCK slots)
    const bool by_c = shift_bases && fixed_c > 0;        // (uniform)
    const int step_k = by_c ? PLAN_BLOCK / fixed_c : 0, step_r = by_c ? PLAN_BLOCK - step_k * fixed_c : 0;
    int shard = by_c ? tid / fixed_c : 0, in_shard = by_c ? tid - shard * fixed_c : 0;
    auto slot_out = [&](int q, bool whole) {             // whole (uniform): every lane has a slot in this step
        const int jr = q * PLAN_BLOCK + tid, j = whole ? jr : min(jr, N - 1);
        const uint32_t bits = L.start_bits[j >> 5];
        const uint32_t upto = bits & (0xFFFFFFFFu >> (31 - (j & 31)));               // starts at slots <= j of the word
        const int32_t m = L.word_starts[j >> 5] + (int32_t)__popc(upto) - 1;         // my micro-batch
        const int32_t first = upto ? (j & ~31) + 31 - __clz(upto) : L.word_last[j >> 5];     // its first slot (slot 0 starts one)
        const int64_t g = L.gpre[j];
        const uint32_t g_next = low_word(j + 1), g_first = low_word(max(first, 0));
        int64_t d = g;
        if (by_c) {
            d = g + L.shard_shift[min(shard, P - 1)];
            shard += step_k;
            in_shard += step_r;
            if (in_shard >= fixed_c) { in_shard -= fixed_c; shard += 1; }
        } else if (shift_bases) {                        // shard of the slot, then its aligned base
            int lo = 0, hi = P - 1;                      // largest p with shard_off[p] <= j
            while (lo < hi) {
                const int mid = (lo + hi + 1) >> 1;
                if (L.shard_off[mid] <= j) lo = mid; else hi = mid - 1;
            }
            d = g + L.shard_shift[lo];
        }
        if (whole || jr < N) {
            a.dst_tok_off[(uint32_t)j] = d;
            a.mb_seq_off[(uint32_t)m] = first;
            a.cu_seqlens[(uint32_t)(j + m)] = (int32_t)((uint32_t)g - g_first);
            a.cu_seqlens[(uint32_t)(j + m) + 1u] = (int32_t)(g_next - g_first);
        }
    };
#pragma unroll 4
    for (int q = 0; q < whole_steps; ++q) slot_out(q, true);
    if (whole_steps < nb) slot_out(whole_steps, false);
    for (int p = tid; p <= P; p += PLAN_BLOCK) {         // micro-batches before each shard's first slot
        const int js = L.shard_off[p];
        int32_t c = M;
        if (js < N) c = L.word_starts[js >> 5] + (int32_t)__popc(L.start_bits[js >> 5] & ((1u << (js & 31)) - 1u));
        a.shard_mb_off[p] = c;
    }
    if (tid == 0) { *a.n_mb = M; a.mb_seq_off[M] = N; }
}

constexpr int REC_BLOCK = 256;                            // granules of one workgroup

// The first slot j of a token axis (starts(j) as for build_record) whose successor starts after `begin`, or N:
// what build_record's bisection finds, for the REC_BLOCK consecutive granules of a workgroup together (every thread of
// the workgroup must call it; begin must not decrease with the thread index).  A bisection of its own is 14 dependent
// reads of global memory per lane at 16 384 slots.  Here the workgroup reads REC_BLOCK evenly spaced starts at once,
// every lane finds its stretch between two of them in the LDS, the workgroup reads the stretches of all its lanes
// (one run of starts: the granules are neighbours) and every lane bisects its own stretch in the LDS: two reads of
// global memory in a row.  A run longer than REC_STAGE entries is bisected where it lies.
constexpr int REC_STAGE = 1024;
struct RecLds {
    int64_t sample[REC_BLOCK];
    int64_t stage[REC_STAGE];
    int32_t run_lo, run_hi;
};
template <typename Starts>
__device__ __forceinline__ int first_slot_after(RecLds& L, int N, Starts starts, int64_t begin) {
    const int tid = threadIdx.x;
    const int stride = (N + REC_BLOCK - 1) / REC_BLOCK;              // >= 1 (N > 0)
    L.sample[tid] = starts(min(tid * stride, N));
    __syncthreads();
    // the last sample that does not lie after `begin` (the first one if all do)
    int i = 0;
#pragma unroll
    for (int step = REC_BLOCK / 2; step >= 1; step >>= 1)
        if (L.sample[i + step] <= begin) i += step;
    // the answer lies in [lo, hi]: everything before sample i starts at or before `begin`; the slot before sample i + 1
    // has a successor behind `begin` (no sample i + 1: hi = N stands for "none")
    int lo = min(i * stride, N);
    int hi = i + 1 < REC_BLOCK ? min((i + 1) * stride, N) - 1 : N;
    hi = max(hi, lo);
    if (tid == 0) L.run_lo = lo;
    if (tid == REC_BLOCK - 1) L.run_hi = hi;
    __syncthreads();
    const int run_lo = L.run_lo, run_hi = max(L.run_hi, L.run_lo);    // the bisections read starts[run_lo + 1 .. run_hi]
    lo = min(max(lo, run_lo), run_hi);                                // (starts that do not rise with j, a caller's mistake, give
    hi = min(hi, run_hi);                                             // a slot that means nothing, but no place outside the run)
    const bool staged = run_hi - run_lo + 1 <= REC_STAGE;             // (uniform)
    if (staged)
        for (int k = tid; k <= run_hi - run_lo; k += REC_BLOCK) L.stage[k] = starts(min(run_lo + k, N));
    __syncthreads();
    while (lo < hi) {
        const int mid = (lo + hi) >> 1;
        const int64_t next = staged ? L.stage[mid + 1 - run_lo] : starts(mid + 1);
        if (next > begin) hi = mid; else lo = mid + 1;
    }
    return lo;
}

// Tables of granule g of a token axis holding N slots (starts(j), 0 <= j <= N; starts(N): its end);
// usable = false leaves the granule empty.  desc(j, &ln, &so, &sh): the validated source of slot j.
// found >= 0: the first slot whose successor starts after the granule's first token (else it is looked for here).
template <typename Starts, typename Desc>
__device__ __forceinline__ void build_record(int N, bool usable, Starts starts, Desc desc, int64_t g,
                                             int32_t* first_out, GranRec* rec_out, int found = -1) {
    const int64_t begin = g * GATHER_GRAN;
    int first = N;
    if (usable && N > 0) {
        // first j whose successor starts after `begin` ...
        int lo = 0, hi = N;
        if (found >= 0) lo = hi = found;
        while (lo < hi) {
            const int mid = (lo + hi) >> 1;
            if (starts(mid + 1) > begin) hi = mid; else lo = mid + 1;
        }
        // ... and if `begin` lies in the padding behind that slot (or the slot is empty), the next one
        while (lo < N) {
            int32_t ln, sh;
            int64_t so;
            desc(lo, &ln, &so, &sh);
            if (starts(lo) + ln > begin) break;
            ++lo;
        }
        first = lo;
    }
    GranRec rec;
#pragma unroll
    for (int r = 0; r < REC_SLOTS; ++r) {
        rec.e[r].start = REL_FAR; rec.e[r].lensh = 0; rec.e[r].src_off = 0;
        const int j = first + r;
        if (j < N) {
            const int64_t d = starts(j) - begin;
            if (d < GATHER_GRAN) {
                int32_t ln, sh;
                int64_t so;
                desc(j, &ln, &so, &sh);
                rec.e[r].start = (int32_t)max(d, (int64_t)-REL_FAR);
                rec.e[r].lensh = ln | (sh << LENSH_SHIFT);
                rec.e[r].src_off = so;
            }
        }
    }
    *first_out = first;
    u32x4* out = reinterpret_cast<u32x4*>(rec_out);
    const u32x4* in = reinterpret_cast<const u32x4*>(&rec);
#pragma unroll
    for (int r = 0; r < REC_SLOTS; ++r) out[r] = in[r];
}

// The granule tables and the per-slot source descriptors as the tail of the launch that balances and plans (fixed_c > 0,
// behind plan_body), for a batch small enough that one workgroup is quicker with them than a launch of its own is started:
// up to SMALL_REC_SLOTS slots and SMALL_REC_GRANS granules, the slots' starts and sources in the LDS behind the prefix.
// src_off[q]: d_src_tok_off of the slots' sequences, asked for before the plan.
// The line (steps in us, this way against the plan by shards behind it, plan_shards.hip): 48 / 64 / 128 sequences 17.7 / 19.8 /
// 22.5 against 19.2 / 20.1 / 22.8.  Above 128 a shard's walk is what the other way waits for: 192 and 256 on 8 shards 21.5 and
// 22.8 against 22.3 and 23.6, on 4 21.3 and 24.1 against 21.9 and 24.6, on 2 25.2 and 28.2 against 25.4 and 27.8, on one 31.5 and
// 36.3 against 30.7 and 35.0.  Above 256 the two are within 0.8 of each other up to 512 (of 450 tokens; of 1500 the other way
// is up to 0.9 quicker), and 1024 on 8 shards take 31.8 against 30.9, 2048 50.1 against 44.5.  A call between other kernels,
// its code not in the caches, shows the same line (192 and 256 on 8 shards 30.7 and 32.1 against 30.5 and 32.4).
struct SmallRecLds {
    int64_t start[SMALL_REC_SLOTS + 1];     // d_dst_tok_off
    int64_t src_off[SMALL_REC_SLOTS];
    int32_t lensh[SMALL_REC_SLOTS];         // length | rollout shard << LENSH_SHIFT
};
constexpr int SMALL_REC_IPT = (SMALL_REC_SLOTS + PLAN_BLOCK - 1) / PLAN_BLOCK;
static_assert(sizeof(SmallRecLds) <= sizeof(int64_t) * (DC_MAX_SEQ - SMALL_REC_SLOTS), "it fits behind the prefix of as many slots");
__device__ __forceinline__ void small_records(PlanLds& L, const PlanArgs& a, const SourceDesc& sd, const int32_t (&seq)[SMALL_REC_IPT],
                                              const int32_t (&len)[SMALL_REC_IPT], const int64_t (&src_off)[SMALL_REC_IPT], int fixed_c) {
    SmallRecLds& R = *reinterpret_cast<SmallRecLds*>(&L.gpre[SMALL_REC_SLOTS + 1]);
    const int tid = threadIdx.x;
    const int N = a.n_seq;
    lds_barrier();                                       // (the words behind the prefix are not the plan's any more)
#pragma unroll
    for (int q = 0; q < SMALL_REC_IPT; ++q) {
        const int j = q * PLAN_BLOCK + tid;
        if (j < N) {
            int32_t ln, sh;
            int64_t so;
            slot_source_of(a, sd, seq[q], seq[q] >= 0 && seq[q] < N, len[q], src_off[q], &ln, &so, &sh);
            R.start[j] = L.gpre[j] + (a.align != 1 ? L.shard_shift[j / fixed_c] : 0);
            R.src_off[j] = so;
            R.lensh[j] = ln | (sh << LENSH_SHIFT);
            a.slot_src_off[j] = so;
            a.slot_len[j] = ln;
            a.slot_shard[j] = sh;
        }
    }
    if (tid == 0) R.start[N] = L.end;
    lds_barrier();
    for (int64_t g = tid; g < a.n_gran; g += PLAN_BLOCK)
        build_record(N, true, [&](int j) { return R.start[j]; },
                     [&](int j, int32_t* ln, int64_t* so, int32_t* sh) {
                         const int32_t ls = R.lensh[j];
                         *ln = ls & ((1 << LENSH_SHIFT) - 1); *sh = ls >> LENSH_SHIFT; *so = R.src_off[j];
                     },
                     g, a.gran_first + g, a.gran_rec + g);
}

}  // namespace dc

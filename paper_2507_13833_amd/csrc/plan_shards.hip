// The plan, the granule tables and the slots' sources behind a launch that has made perm with Algorithm 1 as printed (every
// shard holds C slots), by a few workgroups per shard.
//
// Bound by latency: two trips to memory (perm; the sequences' lengths and offsets), then a chain of reads of the LDS.  Clocks of
// the last walker on 32 shards of 256 slots (2.4 GHz): lengths and bases 1.3 us, prefix 0.6, every slot's end 1.8, hops 1.3,
// counts 0.6, the others' counts 1.2, outputs 0.6; of a slice: 1.3, 0.6, sources 1.0, granules 1.7.
// A shard's slots, its micro-batches and its stretch of the token axis concern nobody else, but for two sums over
// the shards: where a shard's tokens start (the loads are known before this launch) and how many micro-batches the shards
// before it hold.  So workgroup p walks shard p's micro-batches, P + slice * P + p writes a part of its slots and granules;
// each of them makes the prefix of the shard's lengths for itself, and the only thing that travels between workgroups
// is one count per shard.
// 7.4 to 10.1 us (rocprofv3) on 4 to 128 shards of 64 to 640 slots, 0.2 M to 42 M tokens.  With the plan as the tail of the
// balance workgroup (12 to 13 us, and 2 to 6 for shard_of_seq and the slots' lengths) and the tables in a launch behind it
// (7.4 to 9.8) the two launches took: 2048 sequences on 8 shards 41 us, now 34; 15 360 on 24 112, now 91; 8192 on 32 72, now
// 57; 16 384 on 64 106, now 88; 8192 on 128 66, now 50.
// Shards of more than 2048 slots (up to sixteen to a lane, in loops that keep nothing in registers from one pass to the next:
// unrolled, the walk spilled 94 of them and took 8 to 12 us more), both launches: 16 384 sequences on 4 shards 302 us with
// 4096 tokens to a micro-batch and 296 with 65 536, as the balance workgroup's tail 352 and 316; 8190 on 3 210 and 205, so
// 224 and 215.
#include "plan_device.h"

namespace dc {

struct ShardPlanArgs {
    int32_t        C, slices;
    const int64_t* shard_load;
    int32_t*       shard_of_seq;
    uint32_t*      mb_counts;        // zeroed by the launch before; see publish_count
    int32_t*       gran_first;
    GranRec*       gran_rec;
    int64_t        n_gran;
    int32_t        looks;            // at another shard's count
};

// A shard's number of micro-batches, left where the others look for it: a word each up to 64 shards, above that a byte (a
// shard then holds at most DC_MAX_SEQ / 65 slots).  Zero: not there yet.
__device__ __forceinline__ int count_shift(int P, int p) { return P <= WAVE ? 0 : 8 * (p & 3); }
__device__ __forceinline__ uint32_t* count_word(uint32_t* counts, int P, int p) { return counts + (P <= WAVE ? p : p >> 2); }
__device__ __forceinline__ void publish_count(uint32_t* counts, int P, int p, int n) {
    __hip_atomic_fetch_or(count_word(counts, P, p), (uint32_t)n << count_shift(P, p), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
// The count, or 0 if it has not come after so many looks (PLAN_SHARDS_LOOKS take a few hundred us; it comes within one or two).
// Nothing says that all walkers are on the chip at once, so nobody waits for another without an end: a walker whose look
// stays empty counts that shard itself (with no looks every walker counts all shards before its own: same outputs).
__device__ __forceinline__ int wait_count(uint32_t* counts, int P, int p, int looks) {
    const uint32_t mask = P <= WAVE ? 0xFFFFFFFFu : 0xFFu;
    for (int look = 0; look < looks; ++look) {
        const uint32_t n = (__hip_atomic_load(count_word(counts, P, p), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) >> count_shift(P, p)) & mask;
        if (n != 0) return (int)n;
        __builtin_amdgcn_s_sleep(1);
    }
    return 0;
}
static_assert(DC_MAX_SEQ / (WAVE + 1) < 256, "a count of more than 64 shards fits a byte");
static_assert(MB_COUNT_BYTES >= WAVE * 4 && MB_COUNT_BYTES >= BAL_PLAN_MAX_SHARDS, "a word or a byte per shard");

// Slots behind the shard's last one kept at hand, for the records of its last granules.  A granule that starts in front of the
// next shard's first token has no later first slot than that shard's first: the slot behind the one found starts behind the
// granule's start, whether it passes the checks or not.
constexpr int TAIL_SLOTS = REC_SLOTS;

// Exclusive prefix of the lengths of a shard's slots, in 64 bits (16 384 slots can hold 2^38 tokens, in an arena of any size).
// last_within: e[k] is the last e in [from[k], C] with at(e) <= limit[k] (from[k] is one), a lane's slots side by side.
template <int CAP, bool SPLIT>
struct ShardPrefix {
    int64_t v[CAP + 1];
    __device__ __forceinline__ int64_t at(int r) const { return v[r]; }
    __device__ __forceinline__ uint32_t low(int r) const { return (uint32_t)v[r]; }
    template <int SIDE>
    __device__ __forceinline__ void last_within(int C, const int (&from)[SIDE], const int64_t (&limit)[SIDE], int (&e)[SIDE]) const {
#pragma unroll
        for (int k = 0; k < SIDE; ++k) e[k] = from[k];
        for (int hop = 1 << (31 - __clz(C)); hop >= 1; hop >>= 1) {      // (uniform)
#pragma unroll
            for (int k = 0; k < SIDE; ++k) {
                const int c = e[k] + hop;
                if (v[min(c, C)] <= limit[k] && c <= C) e[k] = c;
            }
        }
    }
};
// SPLIT: the tokens before every 64 slots in 64 bits, those of the slots in front inside the 64 in 32 (below 2^30): 64 for
// every slot of a large shard leave no room for its walk, and 32 alone would make falling sums of 2^32 tokens and more.
template <int CAP>
struct ShardPrefix<CAP, true> {
    int64_t  step[CAP / WAVE + 1];
    uint32_t in[CAP + 1];
    __device__ __forceinline__ int64_t at(int r) const { return step[r / WAVE] + (int64_t)in[r]; }
    __device__ __forceinline__ uint32_t low(int r) const { return (uint32_t)step[r / WAVE] + in[r]; }
    // (the 64 it stands in, then its place there)
    template <int SIDE>
    __device__ __forceinline__ void last_within(int C, const int (&from)[SIDE], const int64_t (&limit)[SIDE], int (&e)[SIDE]) const {
        const int last = C / WAVE;
        int s[SIDE];
        uint32_t left[SIDE];
#pragma unroll
        for (int k = 0; k < SIDE; ++k) s[k] = from[k] / WAVE;
        for (int hop = last > 0 ? 1 << (31 - __clz(last)) : 0; hop >= 1; hop >>= 1) {      // (uniform)
#pragma unroll
            for (int k = 0; k < SIDE; ++k) {
                const int c = s[k] + hop;
                if (step[min(c, last)] <= limit[k] && c <= last) s[k] = c;
            }
        }
#pragma unroll
        for (int k = 0; k < SIDE; ++k) {
            left[k] = (uint32_t)min(limit[k] - step[s[k]], (int64_t)0x7FFFFFFF);
            e[k] = s[k] * WAVE;
        }
#pragma unroll
        for (int hop = WAVE / 2; hop >= 1; hop >>= 1) {
#pragma unroll
            for (int k = 0; k < SIDE; ++k) {
                const int c = e[k] + hop;
                if (in[min(c, C)] <= left[k] && c <= C) e[k] = c;
            }
        }
    }
};

// BLOCK * IPT: slots of a shard at most.  STAGE: the slots' sources and a word of 64 bits for each stand in the LDS too.
template <int BLOCK, int IPT, bool STAGE>
struct ShardPlanLds {
    static constexpr int CAP = BLOCK * IPT, STEPS = CAP / WAVE;
    ShardPrefix<CAP, !STAGE> pre;
    union {
        struct { uint16_t next[2][CAP + 1]; uint8_t opens[CAP]; } walk;
        struct { int64_t src_off[STAGE ? CAP : 1]; int32_t lensh[STAGE ? CAP : 1]; } src;
    };
    int64_t base[BAL_PLAN_MAX_SHARDS + 1];   // aligned token offset of every shard
    uint32_t step_sum[STEPS];
    int32_t step_count[STEPS];
    int64_t tmp64[BLOCK / WAVE];
    int32_t tmp32[BLOCK / WAVE];
    int32_t missing;                         // the first shard whose count has not come
    int64_t tail_start[TAIL_SLOTS], tail_src[TAIL_SLOTS];
    int32_t tail_len[TAIL_SLOTS], tail_lensh[TAIL_SLOTS];
};

__device__ __forceinline__ int32_t sane_len(int32_t s) { return s > 0 && s <= DC_MAX_SEQ_LEN ? s : 1; }      // (the balance's own rule)

template <int BLOCK, int IPT, bool STAGE>
__global__ __launch_bounds__(BLOCK) void plan_shards_kernel(PlanArgs a, SourceDesc sd, ShardPlanArgs s) {
    using Lds = ShardPlanLds<BLOCK, IPT, STAGE>;
    __shared__ Lds L;
    constexpr int WAVES = BLOCK / WAVE, UNROLL = IPT < 4 ? IPT : 4;
    const int tid = threadIdx.x, lane = tid & (WAVE - 1), w = __builtin_amdgcn_readfirstlane(tid / WAVE);
    const int N = a.n_seq, P = a.n_shards, C = s.C;
    const bool walker = (int)blockIdx.x < P;
    const int slice = walker ? -1 : ((int)blockIdx.x - P) / P;
    const int p = (int)blockIdx.x - (slice + 1) * P;
    const int j0 = p * C, j_end = j0 + C;
    const int nq = (C + BLOCK - 1) / BLOCK;                       // (uniform) steps with slots at all, <= IPT

    // ---- the shard's slots, and what a slice needs of the next ones ----
    int32_t seq[IPT], len[IPT];
    int64_t src[IPT];
    const int64_t my_load = tid < P ? s.shard_load[tid] : 0;
#pragma unroll
    for (int q = 0; q < IPT; ++q) seq[q] = q < nq ? a.perm[j0 + min(q * BLOCK + tid, C - 1)] : 0;
    const int tail_j = j_end + tid;
    const bool has_tail = !walker && tid < TAIL_SLOTS && tail_j < N;
    int32_t tail_seq = has_tail ? a.perm[tail_j] : 0;
    tail_seq = min(max(tail_seq, 0), N - 1);
    const int32_t tail_len = has_tail ? sane_len(a.seq_len[tail_seq]) : 0;
    const int64_t tail_src = has_tail ? a.src_tok_off[tail_seq] : 0;
#pragma unroll
    for (int q = 0; q < IPT; ++q) {
        len[q] = 0;
        src[q] = 0;
        if (q < nq) {
            seq[q] = min(max(seq[q], 0), N - 1);
            len[q] = a.seq_len[seq[q]];
            if (STAGE && !walker) src[q] = a.src_tok_off[seq[q]];
        }
    }
    // ---- shard bases: exclusive scan of the loads, each rounded up to the alignment ----
    {
        const int64_t padded = a.align == 1 ? my_load : (my_load + a.align - 1) / a.align * a.align;      // (uniform)
        int64_t end;
        const int64_t b = block_excl_scan_add<int64_t>(padded, L.tmp64, &end);
        if (tid < P) L.base[tid] = b;
        if (tid == 0) L.base[P] = end;
    }
    // ---- prefix of the lengths (whole behind the next barrier) ----
    auto prefix = [&]() {
        uint32_t inc[IPT];
#pragma unroll
        for (int q = 0; q < IPT; ++q) {
            const int r = q * BLOCK + tid;
            len[q] = q < nq && r < C ? sane_len(len[q]) : 0;
            inc[q] = wave_incl_scan_add_u32((uint32_t)len[q]);    // (64 lengths stay below 2^31)
            if (lane == WAVE - 1) L.step_sum[r / WAVE] = inc[q];
            if constexpr (!STAGE)
                if (r <= C) L.pre.in[r] = inc[q] - (uint32_t)len[q];
        }
        lds_barrier();
        if constexpr (STAGE) {
            static_assert(Lds::STEPS <= WAVE, "every wave scans them for itself");
            const int64_t n = lane < Lds::STEPS ? (int64_t)L.step_sum[lane] : 0;
            const int64_t upto = wave_incl_scan_add(n);
#pragma unroll
            for (int q = 0; q < IPT; ++q) {
                const int r = q * BLOCK + tid;
                if (r < C) L.pre.v[r] = wave_read_lane((int64_t)(upto - n), q * WAVES + w) + (int64_t)(inc[q] - (uint32_t)len[q]);
            }
            if (tid == 0) L.pre.v[C] = wave_read_lane(upto, WAVE - 1);
        } else {
            static_assert(Lds::STEPS <= BLOCK, "a thread per step");
            int64_t total;
            const int64_t ex = block_excl_scan_add<int64_t>(tid < Lds::STEPS ? (int64_t)L.step_sum[tid] : 0, L.tmp64, &total);
            if (tid < Lds::STEPS) L.pre.step[tid] = ex;
            if (tid == 0) {
                L.pre.step[Lds::STEPS] = total;
                if (C == Lds::CAP) L.pre.in[Lds::CAP] = 0;
            }
        }
    };
    prefix();

    if (walker) {
        // Every slot finds the end of the micro-batch that would open with it (a bisection, a lane's slots side by side).
        // Then the hops are doubled, slots known to open one naming those 1, 2, 4, ... hops on, until a hop from the first
        // slot leaves the shard: log2 of the number of micro-batches in rounds of two LDS reads, where following the
        // chain takes a read (~130 cycles) for each.
        int target = p;                                           // the shard that is walked: the workgroup's own, unless
        bool published = false;                                   // another's count does not come
        int32_t theirs = 0, mb0 = 0, n_mb = 0;                    // thread k < p: shard k's count
        int32_t opened = 0;
        uint16_t* first_of = nullptr;
        auto opening = [&](int q) {                               // lanes whose slot of step q opens a micro-batch
            const int r = q * BLOCK + tid;
            return __ballot(q < nq && r < C && L.walk.opens[min(r, C - 1)] != 0);
        };
        auto micro_batch = [&](int q, uint64_t opens) {           // the lane's slot's
            const int32_t in_front = Lds::STEPS <= WAVE ? wave_read_lane(opened, q * WAVES + w) : L.step_count[q * WAVES + w];
            return in_front + (int32_t)__popcll(opens & (~0ull >> (WAVE - 1 - lane))) - 1;
        };
        for (;;) {
            lds_barrier();
            constexpr int SIDE = UNROLL;
#pragma unroll 1
            for (int q0 = 0; q0 < nq; q0 += SIDE) {                   // (uniform)
                int from[SIDE], e[SIDE];
                int64_t limit[SIDE];
#pragma unroll
                for (int k = 0; k < SIDE; ++k) {
                    from[k] = min((q0 + k) * BLOCK + tid, C - 1);
                    limit[k] = L.pre.at(from[k]) + a.budget;
                }
                L.pre.last_within(C, from, limit, e);
#pragma unroll
                for (int k = 0; k < SIDE; ++k) {                      // (a sequence above the budget is alone in its micro-batch)
                    const int r = (q0 + k) * BLOCK + tid;
                    if (r < C) { L.walk.next[0][r] = (uint16_t)max(e[k], r + 1); L.walk.opens[r] = r == 0; }
                }
            }
            if (tid == 0) { L.walk.next[0][C] = (uint16_t)C; L.walk.next[1][C] = (uint16_t)C; }
            int cur = 0;
            for (;; cur ^= 1) {                                       // (at most log2(C) + 1 rounds: a hop moves on by a slot at least)
                lds_barrier();
                if ((int)L.walk.next[cur][0] >= C) break;             // (uniform)
#pragma unroll UNROLL
                for (int q = 0; q < IPT; ++q) {
                    const int r = q * BLOCK + tid;
                    if (q < nq && r < C) {
                        const int e = L.walk.next[cur][r];
                        if (L.walk.opens[r] && e < C) L.walk.opens[e] = 1;      // (one that another lane has just named names a true one too)
                        L.walk.next[cur ^ 1][r] = L.walk.next[cur][e];
                    }
                }
            }
            // ---- micro-batches that open in front of every 64 slots ----
#pragma unroll UNROLL
            for (int q = 0; q < IPT; ++q) {
                const uint64_t opens = opening(q);
                if (lane == 0) L.step_count[q * WAVES + w] = (int32_t)__popcll(opens);
            }
            lds_barrier();
            if constexpr (Lds::STEPS <= WAVE) {                       // every wave scans them for itself, lane k keeps step k's
                const int32_t n = lane < Lds::STEPS ? L.step_count[lane] : 0;
                const int32_t upto = wave_incl_scan_add(n);
                opened = upto - n;
                n_mb = wave_read_lane(upto, WAVE - 1);
            } else {
                opened = block_excl_scan_add<int32_t>(tid < Lds::STEPS ? L.step_count[tid] : 0, L.tmp32, &n_mb);
                if (tid < Lds::STEPS) L.step_count[tid] = opened;
                lds_barrier();
            }
            if (!published && tid == 0) publish_count(s.mb_counts, P, p, n_mb);
            first_of = L.walk.next[cur ^ 1];                          // (its last reader is a barrier behind)
#pragma unroll UNROLL
            for (int q = 0; q < IPT; ++q) {
                const uint64_t opens = opening(q);
                if ((opens >> lane) & 1ull) first_of[micro_batch(q, opens)] = (uint16_t)(q * BLOCK + tid);
            }
            // ---- the micro-batches of the shards before this one ----
            // (readfirstlane: without it the compiler sets scratch memory aside that the kernel never touches)
            if (!published) theirs = tid < p ? wait_count(s.mb_counts, P, tid, __builtin_amdgcn_readfirstlane(s.looks)) : 0;
            else if (tid == target && target != p) theirs = n_mb;
            published = true;
            const bool missing = tid < p && theirs == 0;
            int32_t sum;                                              // (the missing ones ride the sum's high bits)
            block_excl_scan_add<int32_t>(missing ? 1 << 20 : theirs, L.tmp32, &sum);
            static_assert(DC_MAX_SEQ < (1 << 20) && BAL_PLAN_MAX_SHARDS <= (1 << 11), "both parts fit");
            if ((sum >> 20) == 0) {                                   // (uniform)
                mb0 = sum;
                if (target == p) break;
                target = p;                                           // (its walk was overwritten)
            } else {
                if (tid == 0) L.missing = P;
                lds_barrier();
                if (missing) atomicMin(&L.missing, tid);
                lds_barrier();
                target = L.missing;
            }
            lds_barrier();
#pragma unroll
            for (int q = 0; q < IPT; ++q) {
                len[q] = 0;
                if (q < nq) len[q] = a.seq_len[min(max(a.perm[target * C + min(q * BLOCK + tid, C - 1)], 0), N - 1)];
            }
            prefix();
        }
        // ---- outputs (see plan_body: a slot stores the entry behind its own as well) ----
#pragma unroll UNROLL
        for (int q = 0; q < IPT; ++q) {
            const int r = q * BLOCK + tid, j = j0 + r;
            const int32_t mine = micro_batch(q, opening(q));
            if (q < nq && r < C) {
                const int first = first_of[mine];
                const uint32_t g_first = L.pre.low(first);        // (differences inside a micro-batch fit 32 bits)
                const uint32_t m = (uint32_t)(mb0 + mine);
                a.mb_seq_off[m] = j0 + first;
                a.cu_seqlens[(uint32_t)j + m] = (int32_t)(L.pre.low(r) - g_first);
                a.cu_seqlens[(uint32_t)j + m + 1u] = (int32_t)(L.pre.low(r + 1) - g_first);
            }
        }
        if (tid == 0) {
            a.shard_mb_off[p] = mb0;
            a.shard_tok_off[p] = L.base[p];
            if (p == 0) *a.plan_ok = 1;
            if (p == P - 1) {
                const int64_t end = L.base[P];
                a.shard_mb_off[P] = mb0 + n_mb;
                *a.n_mb = mb0 + n_mb;
                a.mb_seq_off[mb0 + n_mb] = N;
                a.shard_tok_off[P] = end;
                a.dst_tok_off[N] = end;
                if (end > a.capacity) set_status(a.status, DC_ERR_OVERFLOW);
            }
        }
        return;
    }

    // ---- the slots' sources ----
    if (has_tail) {
        int32_t ln, sh;
        int64_t so;
        slot_source_of(a, sd, tail_seq, true, tail_len, tail_src, &ln, &so, &sh);
        L.tail_len[tid] = tail_len;
        L.tail_lensh[tid] = ln | (sh << LENSH_SHIFT);
        L.tail_src[tid] = so;
    }
    lds_barrier();
    const int64_t base = L.base[p];
    if (has_tail) {
        const int k = tail_j / C;                                 // its shard, whose first slot (behind j_end) is here too
        int64_t at = L.base[k];
        for (int u = k * C - j_end; u < tid; ++u) at += L.tail_len[u];
        L.tail_start[tid] = at;
    }
#pragma unroll
    for (int q = 0; q < IPT; ++q) {
        const int r = q * BLOCK + tid, j = j0 + r;
        const bool mine = q % s.slices == slice;                  // (uniform) this workgroup writes the step's slots
        if (q < nq && r < C && (STAGE || mine)) {
            int32_t ln, sh;
            int64_t so;
            slot_source_of(a, sd, seq[q], true, len[q], STAGE ? src[q] : a.src_tok_off[seq[q]], &ln, &so, &sh);
            if constexpr (STAGE) {
                L.src.src_off[r] = so;
                L.src.lensh[r] = ln | (sh << LENSH_SHIFT);
            }
            if (mine) {
                a.dst_tok_off[j] = base + L.pre.at(r);
                s.shard_of_seq[seq[q]] = p;
                a.slot_src_off[j] = so;
                a.slot_len[j] = ln;
                a.slot_shard[j] = sh;
            }
        }
    }
    lds_barrier();
    // ---- the granules whose first token lies in the shard's stretch ----
    auto starts = [&](int j) { return j < j_end ? base + L.pre.at(j - j0) : L.tail_start[j - j_end]; };      // (j < N)
    auto desc = [&](int j, int32_t* ln, int64_t* so, int32_t* sh) {
        int32_t ls;
        if (j >= j_end) {
            ls = L.tail_lensh[j - j_end];
            *so = L.tail_src[j - j_end];
        } else if constexpr (STAGE) {
            ls = L.src.lensh[j - j0];
            *so = L.src.src_off[j - j0];
        } else {
            slot_source(a, sd, j, (int32_t)(L.pre.low(j - j0 + 1) - L.pre.low(j - j0)), ln, so, sh);
            return;
        }
        *ln = ls & ((1 << LENSH_SHIFT) - 1);
        *sh = ls >> LENSH_SHIFT;
    };
    const int64_t ga = (base + GATHER_GRAN - 1) / GATHER_GRAN;
    const int64_t gb = min(s.n_gran, (L.base[p + 1] + GATHER_GRAN - 1) / GATHER_GRAN);
    for (int64_t g = ga + slice * BLOCK + tid; g < gb; g += s.slices * BLOCK) {
        const int from[1] = {0};
        const int64_t rel[1] = {g * GATHER_GRAN - base};
        int found[1];                                             // the first slot whose end lies behind the granule's first token
        L.pre.last_within(C, from, rel, found);
        build_record(N, true, starts, desc, g, s.gran_first + g, s.gran_rec + g, j0 + found[0]);
    }
    // ---- and the table's end, which no token reaches ----
    const int64_t ge = (L.base[P] + GATHER_GRAN - 1) / GATHER_GRAN;
    for (int64_t g = ge + ((int64_t)blockIdx.x - P) * BLOCK + tid; g < s.n_gran; g += (int64_t)P * s.slices * BLOCK)
        build_record(N, false, starts, desc, g, s.gran_first + g, s.gran_rec + g);
}

hipError_t launch_plan_shards(const PlanArgs& p, const SourceDesc& src, const Workspace& ws, const int64_t* d_shard_load,
                              int32_t* d_shard_of_seq, int looks, hipStream_t st) {
    const int P = p.n_shards, C = p.n_seq / P;
    if (P < 1 || P > BAL_PLAN_MAX_SHARDS || C < 1 || C * P != p.n_seq || p.n_seq > DC_MAX_SEQ || !ws.mb_counts)
        return hipErrorInvalidValue;
    ShardPlanArgs s;
    s.C = C; s.shard_load = d_shard_load; s.shard_of_seq = d_shard_of_seq; s.mb_counts = ws.mb_counts;
    s.gran_first = ws.gran_first; s.gran_rec = ws.gran_rec; s.n_gran = ws.n_gran; s.looks = looks;
    auto launch = [&](auto kernel, int block) {
        // a granule per thread, up to 1024 workgroups
        const int64_t want = (ws.n_gran + (int64_t)P * block - 1) / ((int64_t)P * block);
        s.slices = (int32_t)max((int64_t)1, min(want, (int64_t)(1024 / P)));
        hipLaunchKernelGGL(kernel, dim3((unsigned)(P * (1 + s.slices))), dim3(block), 0, st, p, src, s);
        return hipGetLastError();
    };
    static_assert(512 * 4 == PLAN_SHARDS_STAGED && 1024 * 16 == DC_MAX_SEQ, "what the two kernels hold");
    if (C <= PLAN_SHARDS_STAGED) return launch(plan_shards_kernel<512, 4, true>, 512);
    return launch(plan_shards_kernel<1024, 16, false>, 1024);
}

}  // namespace dc

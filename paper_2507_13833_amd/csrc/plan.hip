// Plan of the packed training layout: destination token offsets of every output
// slot, shard token offsets, next-fit micro-batches under the token budget and the
// per-micro-batch cu_seqlens, plus the gather's workspace (validated per-slot
// source descriptors and, per 1024-token granule of the destination, the first slot
// reaching into it and the record of the slots that do).
//
// O(N) integer work on at most DC_MAX_SEQ slots: latency-bound, so the plan proper runs as
// ONE workgroup of 1024 lanes with everything staged in LDS (behind Algorithm 1 as printed, whose shards are all alike:
// plan_shards.hip).  Lane t handles slots t,
// t + 1024, ... (every global access is coalesced):
//   0. (slots_kernel, many workgroups) len = seq_len[perm[j]] and the rollout offset of every
//      slot, validated: random gathers, which need more loads in flight than one CU has;
//   1. slot lengths, check that perm is a permutation; wave scans + one scan of the 256 wave
//      totals -> dense prefix gpre[0..N] (int64, LDS);
//   2. shard bases: exclusive scan of the shard loads, each rounded up to the alignment (a base is
//      always a multiple of it, so rounding the running sum equals summing the rounded loads);
//   3. micro-batch starts -> start bits: a group of lanes per shard hops from start to start, probing a
//      window of slots at once for the last one that still fits under the budget (above 64 shards one
//      lane per shard, each hop a bisection); where the micro-batches are short, every slot's hop is
//      found first, all slots side by side, and the walk only follows them;
//   4. per 32 slots: starts before the word and the last start before it (two scans over
//      512 words); then every slot reads its micro-batch index and start from those and
//      writes its outputs.
#include "plan_device.h"

namespace dc {


// Per-slot source descriptors (one lane per slot, many workgroups; runs before plan_kernel on
// the same stream): the sequence behind each slot, its length and place in the rollout layout,
// validated; a slot that fails a check gets length 0 and moves nothing.  These are random
// gathers over seq_len / src_tok_off, which one workgroup alone could not keep in flight.
constexpr int SLOTS_BLOCK = 256;

__global__ __launch_bounds__(SLOTS_BLOCK) void slots_kernel(PlanArgs a, SourceDesc sd) {
    const int j = blockIdx.x * SLOTS_BLOCK + threadIdx.x;
    const int N = a.n_seq;
    if (a.own_shard_off && j <= sd.n_src) a.own_shard_off[j] = sd.seq_off[j];     // the plan keeps the rollout shards
    if (j >= N) return;
    int32_t ln, sh;
    int64_t so;
    slot_source(a, sd, j, -1, &ln, &so, &sh);
    a.slot_src_off[j] = so;
    a.slot_len[j] = ln;
    a.slot_shard[j] = sh;
}

// IPT: slots per lane at most, PLAN_IPT (more than PLAN_NEXT_MAX slots) or half of that; either kernel holds the code of its
// sizes alone.  One kernel whose passes are left at the first step without slots took 7.6 us for 64 slots, 10.9 for 2048 on 8
// shards, 16.4 for 8192 on 32 and 16.8 for 16 384 on 64; these take 6.7, 9.8, 15.5 and 15.9.
template <int IPT>
__global__ __launch_bounds__(PLAN_BLOCK) void plan_kernel(PlanArgs a) {
    __shared__ PlanLds L;
    const int tid = threadIdx.x;
    const int N = a.n_seq;
    // the slots' sequences and lengths (validated by slots_kernel): asked for first, so that these loads are in
    // flight while the shard table is fetched and checked
    int32_t seq[IPT], len[IPT];
#pragma unroll
    for (int q = 0; q < IPT; ++q) {
        const int j = q * PLAN_BLOCK + tid;
        seq[q] = j < N ? (a.perm ? a.perm[j] : j) : -1;
        len[q] = j < N ? a.slot_len[j] : 0;
    }
    plan_body<IPT, (IPT < PLAN_IPT ? STEP_OVER : ALL), (IPT < PLAN_IPT)>(L, a, seq, len, true, 0);
}

// Per-granule tables for the gather (one lane per granule, many workgroups; runs after
// plan_kernel on the same stream): F[g] = first slot that ends after the granule's first
// token, found by bisection over the slot starts, and the record of the first REC_SLOTS
// slots from F[g] on that start before the granule's end.
struct RecArgs {
    int32_t        n_seq;
    int64_t        n_gran;
    const int64_t* dst_tok_off;      // [N+1]
    const int64_t* slot_src_off;
    const int32_t* slot_len;
    const int32_t* slot_shard;
    const int32_t* plan_ok;
    int32_t*       gran_first;
    GranRec*       gran_rec;
};

// The descriptors as slots_kernel left them in the workspace.
struct StoredDesc {
    const int64_t* slot_src_off;
    const int32_t* slot_len;
    const int32_t* slot_shard;
    __device__ __forceinline__ void operator()(int j, int32_t* ln, int64_t* so, int32_t* sh) const {
        *ln = slot_len[j]; *so = slot_src_off[j]; *sh = slot_shard[j];
    }
};

__global__ __launch_bounds__(REC_BLOCK) void records_kernel(RecArgs a) {
    __shared__ RecLds L;
    const int64_t g = (int64_t)blockIdx.x * REC_BLOCK + threadIdx.x;
    const bool usable = *a.plan_ok != 0;
    int found = -1;
    if (usable && a.n_seq > 0)                                   // (uniform) lanes behind the last granule look for its slot
        found = first_slot_after(L, a.n_seq, [&](int j) { return a.dst_tok_off[j]; }, min(g, a.n_gran - 1) * GATHER_GRAN);
    if (g >= a.n_gran) return;
    build_record(a.n_seq, usable, [&](int j) { return a.dst_tok_off[j]; }, StoredDesc{a.slot_src_off, a.slot_len, a.slot_shard}, g,
                 a.gran_first + g, a.gran_rec + g, found);
}

hipError_t launch_plan(const dc_params& prm, const SourceDesc& src, const int64_t* d_src_tok_off,
                       const int32_t* d_seq_len, const int32_t* d_perm, const int32_t* d_shard_seq_off,
                       int64_t dst_capacity, int64_t* d_dst_tok_off, int64_t* d_shard_tok_off,
                       int32_t* d_shard_mb_off, int32_t* d_mb_seq_off, int32_t* d_cu_seqlens,
                       int32_t* d_n_mb, const Workspace& ws, int32_t* d_status, hipStream_t st) {
    PlanArgs a = make_plan_args(prm, d_src_tok_off, d_seq_len, d_perm, d_shard_seq_off, dst_capacity, d_dst_tok_off,
                                d_shard_tok_off, d_shard_mb_off, d_mb_seq_off, d_cu_seqlens, d_n_mb, ws, d_status);
    if (!d_shard_seq_off) { a.own_shard_off = ws.own_shard_off; a.shard_seq_off = ws.own_shard_off; }
    hipError_t e;
    if (prm.n_seq > DC_MAX_SEQ) {
        if (!ws.gpre) return hipErrorInvalidValue;
        e = launch_plan_large(a, src, st);
    } else {
        if (prm.n_seq > 0 || a.own_shard_off) {
            hipLaunchKernelGGL(slots_kernel, dim3((unsigned)max(1, (prm.n_seq + SLOTS_BLOCK - 1) / SLOTS_BLOCK)),
                               dim3(SLOTS_BLOCK), 0, st, a, src);
            e = hipGetLastError();
            if (e != hipSuccess) return e;
        }
        static_assert(PLAN_NEXT_MAX == PLAN_IPT / 2 * PLAN_BLOCK, "the line between the two kernels");
        if (prm.n_seq <= PLAN_NEXT_MAX) hipLaunchKernelGGL(plan_kernel<PLAN_IPT / 2>, dim3(1), dim3(PLAN_BLOCK), 0, st, a);
        else hipLaunchKernelGGL(plan_kernel<PLAN_IPT>, dim3(1), dim3(PLAN_BLOCK), 0, st, a);
        e = hipGetLastError();
    }
    if (e != hipSuccess) return e;
    return launch_records(prm.n_seq, d_dst_tok_off, ws, st);
}

hipError_t launch_records(int32_t n_seq, const int64_t* d_dst_tok_off, const Workspace& ws, hipStream_t st) {
    RecArgs r;
    r.n_seq = n_seq; r.n_gran = ws.n_gran; r.dst_tok_off = d_dst_tok_off;
    r.slot_src_off = ws.slot_src_off; r.slot_len = ws.slot_len; r.slot_shard = ws.slot_shard;
    r.plan_ok = ws.plan_ok; r.gran_first = ws.gran_first; r.gran_rec = ws.gran_rec;
    hipLaunchKernelGGL(records_kernel, dim3((unsigned)((ws.n_gran + REC_BLOCK - 1) / REC_BLOCK)), dim3(REC_BLOCK), 0, st, r);
    return hipGetLastError();
}

PlanArgs make_plan_args(const dc_params& prm, const int64_t* d_src_tok_off, const int32_t* d_seq_len,
                        const int32_t* d_perm, const int32_t* d_shard_seq_off, int64_t dst_capacity,
                        int64_t* d_dst_tok_off, int64_t* d_shard_tok_off, int32_t* d_shard_mb_off,
                        int32_t* d_mb_seq_off, int32_t* d_cu_seqlens, int32_t* d_n_mb, const Workspace& ws,
                        int32_t* d_status) {
    PlanArgs a;
    a.n_seq = prm.n_seq; a.n_shards = prm.n_shards; a.align = prm.align_tokens;
    a.budget = prm.token_budget; a.capacity = dst_capacity;
    a.src_tok_off = d_src_tok_off; a.seq_len = d_seq_len; a.perm = d_perm; a.shard_seq_off = d_shard_seq_off;
    a.dst_tok_off = d_dst_tok_off; a.shard_tok_off = d_shard_tok_off; a.shard_mb_off = d_shard_mb_off;
    a.mb_seq_off = d_mb_seq_off; a.cu_seqlens = d_cu_seqlens; a.n_mb = d_n_mb;
    a.slot_src_off = ws.slot_src_off; a.slot_len = ws.slot_len; a.slot_shard = ws.slot_shard;
    a.plan_ok = ws.plan_ok; a.status = d_status;
    a.gpre = ws.gpre; a.start_bits = ws.start_bits; a.tile_tokens = ws.tile_tokens;
    a.own_shard_off = nullptr;
    a.gran_first = nullptr; a.gran_rec = nullptr; a.n_gran = 0;
    return a;
}

}  // namespace dc

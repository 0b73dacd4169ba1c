// The plan of the packed training layout for more slots than one workgroup's LDS holds
// (DC_MAX_SEQ < N <= DC_MAX_SEQ_LARGE): the steps of slots_kernel and plan_kernel over MANY workgroups, each step a
// launch (no workgroup waits for another inside one), the prefix of the slot lengths in the workspace:
//   slots    every slot's source, validated; every sequence notes a slot that claims it;
//   tiles    a slot whose sequence has noted another slot repeats it and is emptied; the prefix inside every tile of
//            PL_TILE slots, and the tile's tokens;
//   walk     workgroup p: the aligned start of shard p (summed over the shards before it), and its next-fit
//            micro-batches, by one wave that probes 64 slots of the prefix at once, the shard's part of it staged in the LDS;
//   outputs  tiles of slots: the micro-batches that open before a tile are counted in the bitmap by every workgroup for
//            itself.
// (Where the last two read the prefix they add the tokens of the tiles before, which every workgroup sums for itself.)
// Bound by launches and by the walk of the longest shard.  65 536 slots on 64 shards: 4.9 + 4.7 + 7.8 + 5.4 us; one
// workgroup doing all of it behind slots_kernel, every probe a read of global memory, took 4.7 + 208 us.
#include "plan_device.h"

namespace dc {

constexpr int PL_TILE = 512;                              // slots of one workgroup (slots, tiles)
constexpr int PL_MAX_TILES = DC_MAX_SEQ_LARGE / PL_TILE;
constexpr int PL_WALK = 256;                              // threads that stage a shard
constexpr int PL_STAGE = 32768;                           // slots of a shard that fit the LDS
constexpr int PL_OUT = 1024;                              // slots of one workgroup (outputs)
constexpr int PL_OUT_WORDS = PL_OUT / 32;
static_assert(PL_TILE % 32 == 0 && DC_MAX_SEQ_LARGE % PL_TILE == 0, "a tile owns whole words of the bitmap");
static_assert(sizeof(int64_t) * 32 <= sizeof(int32_t) * PL_TILE, "a word of the table per 32 slots holds the tiles' tokens");

// `note`: one word per sequence (cu_seqlens serves: the last launch writes all N of them), null without a permutation.
__global__ __launch_bounds__(PL_TILE) void plan_large_slots_kernel(PlanArgs a, SourceDesc sd, int32_t* note) {
    const int j = blockIdx.x * PL_TILE + threadIdx.x;
    const int N = a.n_seq;
    if (a.own_shard_off && j <= sd.n_src) a.own_shard_off[j] = sd.seq_off[j];     // the plan keeps the rollout shards
    if (j >= N) return;
    int32_t ln, sh;
    int64_t so;
    slot_source(a, sd, j, -1, &ln, &so, &sh);
    a.slot_src_off[j] = so;
    a.slot_len[j] = ln;
    a.slot_shard[j] = sh;
    if (note) {
        const int32_t i = a.perm[j];
        if (i >= 0 && i < N) note[i] = j;
    }
}

// Sum of one value per thread over the workgroup, in every thread.
__device__ __forceinline__ int64_t block_sum(int64_t v, int64_t* tmp) {
    int64_t total;
    block_excl_scan_add<int64_t>(v, tmp, &total);
    return total;
}

// gpre[j] becomes the tokens of the slots before slot j of j's own tile (gpre[N]: of the tile that slot N would stand in).
__global__ __launch_bounds__(PL_TILE) void plan_large_tiles_kernel(PlanArgs a, const int32_t* note) {
    __shared__ int64_t tmp[PL_TILE / WAVE];
    const int tid = threadIdx.x, t = blockIdx.x;
    const int j = t * PL_TILE + tid;
    const int N = a.n_seq, P = a.n_shards;
    if (t == 0) {                                         // the shard table
        bool bad = false;
        for (int p = tid; p <= P; p += PL_TILE) {
            const int32_t v = a.shard_seq_off[p];
            bad |= v < 0 || v > N || (p == 0 && v != 0) || (p == P && v != N);
            if (p < P && a.shard_seq_off[p + 1] < v) bad = true;
        }
        const int any = __syncthreads_or(bad ? 1 : 0);
        if (tid == 0) {
            *a.plan_ok = any ? 0 : 1;                     // read by the launches behind this one
            if (any) { set_status(a.status, DC_ERR_BAD_LAYOUT); *a.n_mb = 0; }
        }
    }
    int64_t len = j < N ? a.slot_len[j] : 0;
    if (j < N && note) {
        const int32_t i = a.perm[j];                      // (an entry out of range was emptied and flagged by the launch before)
        if (i >= 0 && i < N && note[i] != j) {            // perm is not a permutation; a repeat moves nothing
            set_status(a.status, DC_ERR_BAD_LAYOUT);
            a.slot_len[j] = 0;
            len = 0;
        }
    }
    int64_t total;
    const int64_t ex = block_excl_scan_add<int64_t>(len, tmp, &total);
    if (j < N) a.gpre[j] = ex;
    if (j == N - 1) a.gpre[N] = N % PL_TILE ? ex + len : 0;
    if (tid == 0) a.tile_tokens[t] = total;
    if (tid < PL_TILE / 32 && t * (PL_TILE / 32) + tid < (N + 31) / 32) a.start_bits[t * (PL_TILE / 32) + tid] = 0;
}

// base[t] = tokens of the tiles before tile t, for every tile and the one behind the last.  Every thread of the workgroup
// must call it (barriers inside, one behind the last write).
template <int BLOCK>
__device__ __forceinline__ void tile_bases(const PlanArgs& a, int64_t* base, int64_t* tmp) {
    const int tiles = (a.n_seq + PL_TILE - 1) / PL_TILE;
    constexpr int PER = (PL_MAX_TILES + BLOCK - 1) / BLOCK;
    const int per = (tiles + BLOCK - 1) / BLOCK, lo = (int)threadIdx.x * per;      // (uniform) per <= PER
    int64_t v[PER], sum = 0;
#pragma unroll
    for (int q = 0; q < PER; ++q) v[q] = q < per && lo + q < tiles ? a.tile_tokens[lo + q] : 0;
#pragma unroll
    for (int q = 0; q < PER; ++q) sum += v[q];
    int64_t total;
    int64_t run = block_excl_scan_add<int64_t>(sum, tmp, &total);
#pragma unroll
    for (int q = 0; q < PER; ++q) {
        if (q < per && lo + q < tiles) base[lo + q] = run;
        run += v[q];
    }
    if (threadIdx.x == 0) base[tiles] = total;
    __syncthreads();
}

// The micro-batches of n slots by next-fit, one wave; at(c): tokens of the shard before its slot c, 0 <= c <= n.
template <typename At>
__device__ __forceinline__ void walk_shard(const PlanArgs& a, int first_slot, int n, At at) {
    const int lane = threadIdx.x;
    int j = 0, sz = 0;
    while (j < n) {                                       // (uniform)
        if (lane == 0) atomicOr(&a.start_bits[(first_slot + j) >> 5], (int32_t)(1u << ((first_slot + j) & 31)));
        const int64_t limit = at(j) + a.budget;
        const int e = next_fit_end(WAVE, 6, j, sz, n, [&](int c, int step, int last, bool inside) {
            c += lane * step;
            return (int)__popcll(__ballot((!inside || c <= last) && at(min(c, last)) <= limit));
        });
        sz = e - j;
        j = e;
    }
}

__global__ __launch_bounds__(PL_WALK) void plan_large_walk_kernel(PlanArgs a) {
    __shared__ uint32_t part[PL_STAGE];
    __shared__ int64_t tile_base[PL_MAX_TILES + 1];
    __shared__ int64_t tmp[PL_WALK / WAVE];
    const int tid = threadIdx.x, p = blockIdx.x;
    const int N = a.n_seq, P = a.n_shards;
    const int ok = *a.plan_ok, s0 = a.shard_seq_off[p], n = a.shard_seq_off[p + 1] - s0;      // (asked for at once)
    tile_bases<PL_WALK>(a, tile_base, tmp);
    if (ok == 0) return;                                  // (uniform)
    auto dense = [&](int j) { return tile_base[j / PL_TILE] + a.gpre[j]; };      // tokens of the slots before slot j
    int64_t mine = 0;                                     // aligned tokens of the shards before mine
    for (int q = tid; q < p; q += PL_WALK) {
        const int64_t load = dense(a.shard_seq_off[q + 1]) - dense(a.shard_seq_off[q]);
        mine += a.align == 1 ? load : (load + a.align - 1) / a.align * a.align;
    }
    const int64_t base = block_sum(mine, tmp);
    const int64_t g0 = dense(s0), load = dense(s0 + n) - g0;
    if (tid == 0) {
        a.shard_tok_off[p] = base;
        if (p == P - 1) {
            const int64_t end = base + (load + a.align - 1) / a.align * a.align;
            a.shard_tok_off[P] = end;
            a.dst_tok_off[N] = end;
            if (end > a.capacity) set_status(a.status, DC_ERR_OVERFLOW);
        }
    }
    const bool staged = n < PL_STAGE && load <= 0xFFFFFFFFLL;        // (uniform)
    if (staged)
        for (int c = tid; c <= n; c += PL_WALK) part[c] = (uint32_t)(dense(s0 + c) - g0);
    __syncthreads();
    if (tid >= WAVE) return;
    if (staged) walk_shard(a, s0, n, [&](int c) { return (int64_t)part[c]; });
    else walk_shard(a, s0, n, [&](int c) { return dense(s0 + c) - g0; });
}

__global__ __launch_bounds__(PL_OUT) void plan_large_out_kernel(PlanArgs a) {
    __shared__ uint32_t bits_of[PL_OUT_WORDS + 1];        // the tile's words and the one behind them
    __shared__ int32_t starts_before[PL_OUT_WORDS + 1], last_before[PL_OUT_WORDS];
    __shared__ int32_t shard_off[DC_MAX_SHARDS + 1];
    __shared__ int64_t shard_shift[DC_MAX_SHARDS];
    __shared__ int64_t tile_base[PL_MAX_TILES + 1];
    __shared__ int64_t tmp64[PL_OUT / WAVE];
    __shared__ int32_t tmp32[PL_OUT / WAVE];
    const int tid = threadIdx.x, t = blockIdx.x;
    const int N = a.n_seq, P = a.n_shards;
    const int n_words = (N + 31) / 32, w0 = t * PL_OUT_WORDS;
    const int ok = *a.plan_ok;
    // starts in the words before the tile, and the last of them
    int64_t n_mine = 0;
    int32_t last_mine = -1;
    for (int i = tid; i < w0; i += PL_OUT) {
        const uint32_t b = (uint32_t)a.start_bits[i];
        n_mine += __popc(b);
        if (b) last_mine = i * 32 + 31 - __clz(b);        // (i grows)
    }
    tile_bases<PL_OUT>(a, tile_base, tmp64);
    if (ok == 0) return;                                  // (uniform)
    auto dense = [&](int j) { return tile_base[j / PL_TILE] + a.gpre[j]; };      // tokens of the slots before slot j
    for (int p = tid; p <= P; p += PL_OUT) {
        shard_off[p] = a.shard_seq_off[p];
        if (p < P) shard_shift[p] = a.align == 1 ? 0 : a.shard_tok_off[p] - dense(a.shard_seq_off[p]);
    }
    if (tid <= PL_OUT_WORDS) bits_of[tid] = w0 + tid < n_words ? (uint32_t)a.start_bits[w0 + tid] : 0u;
    const int32_t m0 = (int32_t)block_sum(n_mine, tmp64);
    last_mine = wave_incl_scan_max(last_mine);
    if ((tid & (WAVE - 1)) == WAVE - 1) tmp32[tid / WAVE] = last_mine;
    __syncthreads();
    if (tid < WAVE) {                                     // one wave: the tile's 32 words
        int32_t l0 = -1;
        for (int i = 0; i < PL_OUT / WAVE; ++i) l0 = max(l0, tmp32[i]);
        const uint32_t b = tid < PL_OUT_WORDS ? bits_of[tid] : 0u;
        const int32_t c = (int32_t)__popc(b);
        const int32_t inc = wave_incl_scan_add<int32_t>(c);
        const int32_t l = wave_incl_scan_max(b ? (w0 + tid) * 32 + 31 - __clz(b) : -1);
        if (tid < PL_OUT_WORDS) {
            starts_before[tid] = m0 + inc - c;
            last_before[tid] = max(l0, wave_shift_up1(l, -1));
        }
        if (tid == PL_OUT_WORDS - 1) starts_before[PL_OUT_WORDS] = m0 + inc;
    }
    __syncthreads();
    const int j = t * PL_OUT + tid;
    const int wl = tid >> 5;
    if (j < N) {
        const uint32_t bits = bits_of[wl];
        const uint32_t upto = bits & (0xFFFFFFFFu >> (31 - (j & 31)));           // starts at slots <= j of the word
        const int32_t m = starts_before[wl] + (int32_t)__popc(upto) - 1;         // my micro-batch
        const int32_t first = upto ? (j & ~31) + 31 - __clz(upto) : max(last_before[wl], 0);
        if ((bits >> (j & 31)) & 1u) a.mb_seq_off[m] = j;
        const int64_t g = dense(j), gs = dense(first);
        int64_t d = g;
        if (a.align != 1) {                               // uniform: shard of the slot, then its aligned base
            int lo = 0, hi = P - 1;                       // largest p with shard_off[p] <= j
            while (lo < hi) {
                const int mid = (lo + hi + 1) >> 1;
                if (shard_off[mid] <= j) lo = mid; else hi = mid - 1;
            }
            d = g + shard_shift[lo];
        }
        a.dst_tok_off[j] = d;
        a.cu_seqlens[j + m] = (int32_t)(g - gs);
        const bool closes = (j + 1 == N) || ((bits_of[(tid + 1) >> 5] >> ((j + 1) & 31)) & 1u);
        if (closes) a.cu_seqlens[j + m + 1] = (int32_t)(dense(j + 1) - gs);
    }
    const bool last_tile = (t + 1) * PL_OUT >= N;
    for (int p = tid; p <= P; p += PL_OUT) {              // micro-batches before each shard's first slot
        const int js = shard_off[p];
        if (js < N ? js / PL_OUT != t : !last_tile) continue;
        const int w = (js - t * PL_OUT) >> 5;
        a.shard_mb_off[p] = js < N ? starts_before[w] + (int32_t)__popc(bits_of[w] & ((1u << (js & 31)) - 1u)) : starts_before[PL_OUT_WORDS];
    }
    if (last_tile && tid == 0) {
        const int32_t M = starts_before[PL_OUT_WORDS];
        *a.n_mb = M;
        a.mb_seq_off[M] = N;
    }
}

hipError_t launch_plan_large(const PlanArgs& a, const SourceDesc& src, hipStream_t st) {
    if (a.n_seq > DC_MAX_SEQ_LARGE || a.n_seq <= 0 || !a.gpre || !a.start_bits || !a.tile_tokens) return hipErrorInvalidValue;
    const unsigned tiles = (unsigned)((a.n_seq + PL_TILE - 1) / PL_TILE);
    int32_t* note = a.perm ? a.cu_seqlens : nullptr;
    hipLaunchKernelGGL(plan_large_slots_kernel, dim3(tiles), dim3(PL_TILE), 0, st, a, src, note);
    hipLaunchKernelGGL(plan_large_tiles_kernel, dim3(tiles), dim3(PL_TILE), 0, st, a, note);
    hipLaunchKernelGGL(plan_large_walk_kernel, dim3((unsigned)a.n_shards), dim3(PL_WALK), 0, st, a);
    hipLaunchKernelGGL(plan_large_out_kernel, dim3((unsigned)((a.n_seq + PL_OUT - 1) / PL_OUT)), dim3(PL_OUT), 0, st, a);
    return hipGetLastError();
}

}  // namespace dc

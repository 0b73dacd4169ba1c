// Argsort of the sequence lengths for more sequences than one workgroup's LDS holds (Algorithm 1's first
// statement above DC_MAX_SEQ sequences): a stable LSD radix sort of the sequence indices by descending
// length over MANY workgroups, three passes of 8 bits (lengths are at most 2^24), each pass three launches:
//   count    every workgroup takes a tile of SORT_TILE positions and counts its digits;
//   scan     workgroup d turns the counts of digit d into running sums over the tiles and notes the digit's total;
//   scatter  every workgroup scans the 256 totals (where each digit starts), ranks its tile again, stably (wave
//            by wave, lanes with equal digits matched by ballots), and moves the indices; the last pass also
//            writes the lengths in sorted order.
// No workgroup ever waits for another inside a launch; the launches of a pass order them.
//
// Up to SORT_PORTIONS * SORT_PORTION sequences two launches take the place of the nine: a workgroup sorts a portion of the
// sequences in its LDS (as dc_balance sorts its own), then every element counts, in each other portion, the elements that
// come before it.  Bound by latency: the nine take 4 to 7 us each whatever they do, 47 us for 65 536 sequences; these two
// take 22 (12 + 10).  A portion more costs every element a search more, a larger one its workgroup a longer sort: dc_balance_ws of
// 98 304 and 131 072 sequences on 64 shards 296 -> 284 and 348 -> 336 us; lengths anywhere up to 2^24, which a portion sorts in three
// passes, 662 -> 666 and 869 -> 875 (65 536: 457 -> 452).
#include "balance_device.h"

namespace dc {

constexpr int SORT_BLOCK = 256;
constexpr int SORT_WAVES = SORT_BLOCK / WAVE;
constexpr int SORT_PER_WAVE = 256;                        // consecutive positions of one wave
constexpr int SORT_TILE = SORT_WAVES * SORT_PER_WAVE;     // positions of one workgroup
constexpr int SORT_LEN_BITS = 24;
static_assert((1 << SORT_LEN_BITS) >= DC_MAX_SEQ_LEN, "three 8-bit passes cover every length");

struct SortArgs {
    int32_t        n;
    int32_t        n_tiles;
    int32_t        shift;             // 0, 8, 16
    const int32_t* seq_len;
    const int32_t* src;               // indices in the order of the pass before (null: the identity)
    int32_t*       dst;
    uint32_t*      counts;            // [256 * n_tiles], digit-major
    uint32_t*      totals;            // [256] items per digit
    int32_t*       len_out;           // last pass: the lengths in the order of dst (else null)
    int32_t*       status;            // first pass: DC_ERR_ZERO_LENGTH_SEQ for a length outside (0, 2^24] (else null)
};

// Key of a sequence: ascending keys = descending lengths; lengths outside (0, 2^24] count as 1, as everywhere.
__device__ __forceinline__ int32_t sort_len(int32_t len) { return (len <= 0 || len > DC_MAX_SEQ_LEN) ? 1 : len; }
__device__ __forceinline__ uint32_t sort_key(int32_t len) { return (uint32_t)(DC_MAX_SEQ_LEN - sort_len(len)); }

// For the wave's positions base .. base + 63 (valid below n_end): my digit, the lanes of this step that hold the
// same digit, and how many of them stand before me.
__device__ __forceinline__ void match_digits(bool valid, uint32_t d, int lane, uint64_t* peers_out, int* before_out) {
    const uint64_t valid_lanes = __builtin_amdgcn_ballot_w64(valid);
    uint32_t peers_lo = (uint32_t)valid_lanes, peers_hi = (uint32_t)(valid_lanes >> 32);
#pragma unroll
    for (int b = 0; b < 8; ++b) {
        const uint64_t bal = __builtin_amdgcn_ballot_w64(((d >> b) & 1u) != 0u);
        const uint32_t mine = (uint32_t)__builtin_amdgcn_sbfe((int)d, (unsigned)b, 1u);      // all ones if my bit is set
        peers_lo &= ~((uint32_t)bal ^ mine);
        peers_hi &= ~((uint32_t)(bal >> 32) ^ mine);
    }
    const uint64_t peers = ((uint64_t)peers_hi << 32) | peers_lo;
    *peers_out = peers;
    *before_out = __popcll(peers & ((1ull << lane) - 1ull));
}

__global__ __launch_bounds__(SORT_BLOCK) void sort_count_kernel(SortArgs a) {
    __shared__ uint32_t cnt[256];
    const int tid = threadIdx.x;
    cnt[tid] = 0;
    __syncthreads();
    const int begin = blockIdx.x * SORT_TILE, end = min(a.n, begin + SORT_TILE);
    for (int pos = begin + tid; pos < end; pos += SORT_BLOCK) {
        const int32_t i = a.src ? a.src[pos] : pos;
        const int32_t raw = a.seq_len[min(max(i, 0), a.n - 1)];
        if (a.status && raw != sort_len(raw)) set_status(a.status, DC_ERR_ZERO_LENGTH_SEQ);
        const uint32_t d = (sort_key(raw) >> a.shift) & 0xFFu;
        atomicAdd(&cnt[d], 1u);                                   // (only the totals matter here)
    }
    __syncthreads();
    a.counts[(size_t)tid * a.n_tiles + blockIdx.x] = cnt[tid];
}

// Workgroup d: exclusive scan of counts[d][0 .. n_tiles) in place; totals[d] = their sum.
__global__ __launch_bounds__(SORT_BLOCK) void sort_scan_kernel(uint32_t* counts, uint32_t* totals, int32_t n_tiles) {
    __shared__ uint32_t tmp[SORT_WAVES];
    const int tid = threadIdx.x;
    uint32_t* row = counts + (size_t)blockIdx.x * n_tiles;
    uint32_t carry = 0;
    for (int base = 0; base < n_tiles; base += SORT_BLOCK) {      // (uniform)
        const int i = base + tid;
        const uint32_t c = i < n_tiles ? row[i] : 0u;
        uint32_t all;
        const uint32_t before = block_excl_scan_add<uint32_t>(c, tmp, &all);
        if (i < n_tiles) row[i] = carry + before;
        carry += all;
    }
    if (tid == 0) totals[blockIdx.x] = carry;
}

__global__ __launch_bounds__(SORT_BLOCK) void sort_scatter_kernel(SortArgs a) {
    constexpr int PITCH = SORT_WAVES + 1;                         // odd: the digits' rows start in different LDS banks
    __shared__ uint32_t cnt[256 * PITCH];                         // [digit][wave]: first counts, then the wave's next place
    __shared__ uint32_t tmp[SORT_WAVES];
    const int tid = threadIdx.x, lane = tid & (WAVE - 1), w = tid / WAVE;
    uint32_t n_all;
    const uint32_t digit_start = block_excl_scan_add<uint32_t>(a.totals[tid], tmp, &n_all);      // tid = digit
    for (int i = tid; i < 256 * PITCH; i += SORT_BLOCK) cnt[i] = 0;
    __syncthreads();
    const int begin = blockIdx.x * SORT_TILE + w * SORT_PER_WAVE, end = min(a.n, begin + SORT_PER_WAVE);
    for (int sweep = 0; sweep < 2; ++sweep) {
        for (int base = begin; base < end; base += WAVE) {       // uniform over the wave; positions in order
            const int pos = base + lane;
            const bool valid = pos < end;
            int32_t i = 0, len = 1;
            uint32_t d = 0;
            if (valid) {
                i = a.src ? a.src[pos] : pos;
                len = sort_len(a.seq_len[min(max(i, 0), a.n - 1)]);
                d = (sort_key(len) >> a.shift) & 0xFFu;
            }
            uint64_t peers;
            int before;
            match_digits(valid, d, lane, &peers, &before);
            const int leader = valid ? (__ffsll((long long)peers) - 1) : lane;
            uint32_t old = 0;
            if (valid && lane == leader) {                        // one lane per distinct digit
                uint32_t* c = &cnt[d * PITCH + w];
                old = *c;
                *c = old + (uint32_t)__popcll(peers);
            }
            old = (uint32_t)__shfl((int)old, leader, WAVE);
            if (sweep == 1 && valid) {
                const uint32_t out = min(old + (uint32_t)before, (uint32_t)(a.n - 1));
                a.dst[out] = i;
                if (a.len_out) a.len_out[out] = len;
            }
        }
        __syncthreads();
        if (sweep == 0) {
            // the wave's first place for every digit: where the digit starts for this tile, plus the waves before
            const uint32_t start = digit_start + a.counts[(size_t)tid * a.n_tiles + blockIdx.x];
            uint32_t run = start;
#pragma unroll
            for (int q = 0; q < SORT_WAVES; ++q) { const uint32_t c = cnt[tid * PITCH + q]; cnt[tid * PITCH + q] = run; run += c; }
            __syncthreads();
        }
    }
}

constexpr int SORT_PORTION = 8192;
constexpr int SORT_PORTIONS = 16;
static_assert(SORT_PORTION <= DC_MAX_SEQ && SORT_PORTION <= 0x10000, "a portion fits the LDS, a place in it 16 bits");

// Workgroup b: portion b by descending length, equal lengths in index order: lengths to len_out, indices to idx_out.
__global__ __launch_bounds__(BAL_BLOCK) void sort_portions_kernel(int32_t n_all, const int32_t* __restrict__ seq_len,
                                                                  int32_t* __restrict__ len_out, int32_t* __restrict__ idx_out,
                                                                  int32_t* status) {
    __shared__ BalLds L;
    const int tid = threadIdx.x, lane = tid & (WAVE - 1), w = tid / WAVE;
    const int first = blockIdx.x * SORT_PORTION, N = min(SORT_PORTION, n_all - first);
    const int rounds = (N + BAL_BLOCK - 1) / BAL_BLOCK;
    constexpr int USED = SORT_PORTION / BAL_BLOCK;
    bin_sort_clear(L);                                            // (the barrier below stands between this and the bins' use)
    int32_t len[BAL_ROUNDS];
#pragma unroll
    for (int q = 0; q < BAL_ROUNDS; ++q) len[q] = q < USED ? seq_len[first + min(bal_item(q, rounds), N - 1)] : 1;
    int32_t mx = 0, mn = INT32_MAX;
#pragma unroll
    for (int q = 0; q < USED; ++q) {
        const bool mine = q < rounds && bal_item(q, rounds) < N;
        const int32_t s = sort_len(len[q]);
        if (mine && s != len[q]) set_status(status, DC_ERR_ZERO_LENGTH_SEQ);
        len[q] = mine ? s : 1;
        mx = max(mx, mine ? s : 0);
        mn = min(mn, mine ? s : INT32_MAX);
    }
    wave_all_reduce([&](auto j) {
        constexpr int J = decltype(j)::value;
        const uint32_t hi = lane_xor<J>((uint32_t)mx), lo = lane_xor<J>((uint32_t)mn);
        mx = max(mx, (int32_t)hi);
        mn = min(mn, (int32_t)lo);
    });
    if (lane == 0) { L.red[w] = mx; L.red[BAL_WAVES + w] = mn; }
    lds_barrier();
    mx = 0; mn = INT32_MAX;
    for (int i = 0; i < BAL_WAVES; ++i) { mx = max(mx, L.red[i]); mn = min(mn, L.red[BAL_WAVES + i]); }
    const uint32_t range = (uint32_t)(mx - mn);
    const int passes = range == 0 ? 0 : (32 - __clz(range) + 7) / 8;
    if ((uint32_t)mx <= PACKED_MAX_LEN) {                         // (uniform) words of length << 16 | place in the portion
        uint32_t* src = reinterpret_cast<uint32_t*>(L.keys);
        uint32_t* dst = reinterpret_cast<uint32_t*>(L.idx_a);
        if (range != 0u && range <= BIN_RANGE_MAX && bin_sort_packed(L, N, (uint32_t)mx, range, len, dst)) {
            src = dst;
        } else {
            lds_barrier();
#pragma unroll
            for (int q = 0; q < USED; ++q) {
                const int i = bal_item(q, rounds);
                if (q < rounds && i < N) src[i] = ((uint32_t)len[q] << 16) | (uint32_t)i;
            }
            lds_barrier();
            for (int pass = 0; pass < passes; ++pass) {
                const int shift = pass * 8;
                counting_pass(L, N, rounds,
                              [&](int pos) { return ((uint32_t)mx - (src[pos] >> 16)) >> shift; },
                              [&](int pos, int out) { dst[out] = src[pos]; });
                uint32_t* t = src; src = dst; dst = t;
            }
        }
        for (int i = tid; i < N; i += BAL_BLOCK) {
            const uint32_t e = src[i];
            len_out[first + i] = (int32_t)(e >> 16);
            idx_out[first + i] = first + (int32_t)(e & 0xFFFFu);
        }
        return;
    }
    lds_barrier();
#pragma unroll
    for (int q = 0; q < USED; ++q) {
        const int i = bal_item(q, rounds);
        if (q < rounds && i < N) { L.keys[i] = len[q]; L.idx_a[i] = (uint16_t)i; }
    }
    uint16_t* src = L.idx_a;
    uint16_t* dst = L.idx_b;
    lds_barrier();
    for (int pass = 0; pass < passes; ++pass) {
        const int shift = pass * 8;
        counting_pass(L, N, rounds,
                      [&](int pos) { return ((uint32_t)(mx - L.keys[src[pos]])) >> shift; },
                      [&](int pos, int out) { dst[out] = src[pos]; });
        uint16_t* t = src; src = dst; dst = t;
    }
    for (int i = tid; i < N; i += BAL_BLOCK) {
        len_out[first + i] = L.keys[src[i]];
        idx_out[first + i] = first + (int32_t)src[i];
    }
}

// Every element's place among all portions: its place in its own, and in each other one the elements before it, which
// are those that are longer, and of an earlier portion those of its length too.  512 evenly spaced lengths of every portion
// stand in the LDS (one read of memory), what lies between two of them is bisected where it is.  PORTIONS: at most; up to eight
// side by side.
template <int PORTIONS>
__global__ __launch_bounds__(SORT_BLOCK) void sort_merge_kernel(int32_t n_all, const int32_t* __restrict__ len_in,
                                                                const int32_t* __restrict__ idx_in, int32_t* __restrict__ len_out,
                                                                int32_t* __restrict__ idx_out) {
    constexpr int SAMPLES = 512, STRIDE = SORT_PORTION / SAMPLES, SIDE = PORTIONS < 8 ? PORTIONS : 8;
    __shared__ int32_t sample[PORTIONS][SAMPLES];
    static_assert(STRIDE * SAMPLES == SORT_PORTION && SAMPLES % SORT_BLOCK == 0 && (STRIDE & (STRIDE - 1)) == 0, "whole stretches");
    const int tid = threadIdx.x;
    const int n_portions = (n_all + SORT_PORTION - 1) / SORT_PORTION;
    {
        int32_t x[PORTIONS][SAMPLES / SORT_BLOCK];                // (every load is issued before the first is looked at)
#pragma unroll
        for (int b = 0; b < PORTIONS; ++b)
#pragma unroll
            for (int s = 0; s < SAMPLES / SORT_BLOCK; ++s)
                x[b][s] = len_in[min(b * SORT_PORTION + (s * SORT_BLOCK + tid) * STRIDE, n_all - 1)];
#pragma unroll
        for (int b = 0; b < PORTIONS; ++b)
#pragma unroll
            for (int s = 0; s < SAMPLES / SORT_BLOCK; ++s)        // (behind the last element: shorter than any)
                sample[b][s * SORT_BLOCK + tid] = b * SORT_PORTION + (s * SORT_BLOCK + tid) * STRIDE < n_all ? x[b][s] : 0;
    }
    const int t = blockIdx.x * SORT_BLOCK + tid;
    const int32_t mine = len_in[min(t, n_all - 1)], idx = idx_in[min(t, n_all - 1)];
    const int own = (int)(blockIdx.x * SORT_BLOCK) / SORT_PORTION;        // (uniform)
    __syncthreads();
    int place = min(t, n_all - 1) - own * SORT_PORTION;
    for (int b0 = 0; b0 < n_portions; b0 += SIDE) {               // (uniform)
        int lo[SIDE], hi[SIDE], size[SIDE];
        int32_t limit[SIDE];                                      // an element comes before mine if it is longer than this
#pragma unroll
        for (int k = 0; k < SIDE; ++k) {
            const int b = min(b0 + k, n_portions - 1);
            limit[k] = b < own ? mine - 1 : mine;
            size[k] = min(SORT_PORTION, n_all - b * SORT_PORTION);
            lo[k] = 0;
        }
#pragma unroll
        for (int step = SAMPLES / 2; step >= 1; step >>= 1) {     // samples before mine, all but the last looked at
#pragma unroll
            for (int k = 0; k < SIDE; ++k)
                if (sample[min(b0 + k, n_portions - 1)][lo[k] + step - 1] > limit[k]) lo[k] += step;
        }
#pragma unroll
        for (int k = 0; k < SIDE; ++k) {
            if (sample[min(b0 + k, n_portions - 1)][lo[k]] > limit[k]) lo[k] += 1;
            hi[k] = min(lo[k] * STRIDE, size[k]);
            lo[k] = min(max(lo[k] * STRIDE - STRIDE + 1, 0), hi[k]);
        }
#pragma unroll
        for (int step = STRIDE; step >= 1; step >>= 1) {          // STRIDE + 1 places at most are left
#pragma unroll
            for (int k = 0; k < SIDE; ++k) {
                const int mid = (lo[k] + hi[k]) >> 1;
                const int32_t x = len_in[min(min(b0 + k, n_portions - 1) * SORT_PORTION + mid, n_all - 1)];
                if (lo[k] < hi[k]) { if (x > limit[k]) lo[k] = mid + 1; else hi[k] = mid; }
            }
        }
#pragma unroll
        for (int k = 0; k < SIDE; ++k)
            if (b0 + k < n_portions && b0 + k != own) place += lo[k];
    }
    if (t < n_all) {
        place = min(place, n_all - 1);
        len_out[place] = mine;
        idx_out[place] = idx;
    }
}

// Bytes of the (digit, tile) table for n sequences.
size_t sort_large_table_bytes(int32_t n_seq) {
    const size_t tiles = ((size_t)n_seq + SORT_TILE - 1) / SORT_TILE;
    return 256 * (tiles + 1) * sizeof(uint32_t);                  // the (digit, tile) counts, then the digits' totals
}

// d_idx_a, d_idx_b, d_sorted_len, d_spare: arrays of n_seq int32; d_counts: sort_large_table_bytes(n_seq).  The passes go
// identity -> b, b -> a, a -> b: the sorted indices end in d_idx_b, their lengths in d_sorted_len, the others are free again.
hipError_t launch_sort_large(int32_t n_seq, const int32_t* d_seq_len, int32_t* d_idx_a, int32_t* d_idx_b,
                             int32_t* d_sorted_len, int32_t* d_spare, uint32_t* d_counts, int32_t* d_status, hipStream_t st) {
    if (n_seq <= SORT_PORTIONS * SORT_PORTION) {
        hipLaunchKernelGGL(sort_portions_kernel, dim3((unsigned)((n_seq + SORT_PORTION - 1) / SORT_PORTION)), dim3(BAL_BLOCK), 0, st,
                           n_seq, d_seq_len, d_spare, d_idx_a, d_status);
        auto merge = [&](auto kernel) {
            hipLaunchKernelGGL(kernel, dim3((unsigned)((n_seq + SORT_BLOCK - 1) / SORT_BLOCK)), dim3(SORT_BLOCK), 0, st, n_seq, d_spare,
                               d_idx_a, d_sorted_len, d_idx_b);
        };
        if (n_seq <= 4 * SORT_PORTION) merge(sort_merge_kernel<4>);
        else if (n_seq <= 8 * SORT_PORTION) merge(sort_merge_kernel<8>);
        else merge(sort_merge_kernel<SORT_PORTIONS>);
        return hipGetLastError();
    }
    SortArgs a;
    a.n = n_seq;
    a.n_tiles = (n_seq + SORT_TILE - 1) / SORT_TILE;
    a.seq_len = d_seq_len;
    a.counts = d_counts;
    a.totals = d_counts + (size_t)256 * a.n_tiles;
    const int32_t* src = nullptr;
    int32_t* dst = d_idx_b;
    for (int pass = 0; pass < SORT_LEN_BITS / 8; ++pass) {
        a.shift = 8 * pass;
        a.src = src;
        a.dst = dst;
        a.status = pass == 0 ? d_status : nullptr;
        a.len_out = pass == SORT_LEN_BITS / 8 - 1 ? d_sorted_len : nullptr;
        hipLaunchKernelGGL(sort_count_kernel, dim3((unsigned)a.n_tiles), dim3(SORT_BLOCK), 0, st, a);
        hipLaunchKernelGGL(sort_scan_kernel, dim3(256), dim3(SORT_BLOCK), 0, st, a.counts, a.totals, a.n_tiles);
        hipLaunchKernelGGL(sort_scatter_kernel, dim3((unsigned)a.n_tiles), dim3(SORT_BLOCK), 0, st, a);
        hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
        src = dst;
        dst = dst == d_idx_b ? d_idx_a : d_idx_b;
    }
    return hipSuccess;                                            // (src == d_idx_b: the order of the last pass)
}

}  // namespace dc

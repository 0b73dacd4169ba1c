// Reverse path: packed training layout -> rollout layout, for per-token fields a stage
// running in the training layout produced (the collect / concat side of a stage transition,
// App. B Table 2; Sec. 6 "Distributed Databuffer" moves data between stages in both
// directions).
//
// A scatter by destination would write the rollout buffers in sequence-random order, which
// costs twice what random reads cost.  Instead the rollout layout is treated as the
// DESTINATION of a gather: sequence i of rollout shard s is "slot" i of that shard, it starts
// at its rollout offset and comes from element dst_tok_off[slot of i] of the training arena.
// One launch inverts the permutation (every sequence notes a slot that claims it), one builds the
// granule tables of every rollout buffer's token axis, taking every sequence's source through its
// note, and writes the per-sequence descriptors that crowded granules read, and one launch of the
// gather's tile mover (the rollout buffers being destination segments of one grid) moves the
// data: linear, aligned 16-byte stores into the rollout buffers, one (mis)aligned load per chunk
// from the arena.  (Clearing the descriptors, claiming them by compare-and-swap and building the tables were three
// launches, the last with a bisection of fourteen dependent reads per granule: 16 us before a gather of 90 us.  Whole calls:
// 24.3 M tokens of 8192 sequences 103 -> 99 us, 632 K of 3108 26.8 -> 17.0 us, 16 M of 35 712 134 -> 82 us, the last two
// with the crowded granules' new path.)
#include "plan_device.h"

namespace dc {

constexpr int SCAT_BLOCK = 256;

struct ScatArgs {
    int32_t        n_seq;
    int64_t        capacity;         // elements of every training arena
    const int64_t* src_tok_off;      // rollout offset of every sequence
    const int32_t* seq_len;
    const int32_t* perm;
    const int64_t* dst_tok_off;      // arena offset of every slot
    int64_t*       r_src_off;
    int32_t*       r_len;
    int32_t*       note;
    int32_t*       gran_first;
    GranRec*       gran_rec;
    int32_t*       status;
};

__device__ __forceinline__ int rollout_shard(const SourceDesc& sd, int i) {
    int sh = 0;                                          // seq_off[s] = N from s = n_src on
    if (sd.n_src > 1) {
#pragma unroll
        for (int s = 1; s < DC_MAX_SRC_SHARDS; ++s) sh += i >= sd.seq_off[s] ? 1 : 0;
    }
    return sh;
}
__device__ __forceinline__ int64_t shard_tokens(const SourceDesc& sd, int sh) {
    int64_t t = sd.tokens[0];
#pragma unroll
    for (int s = 1; s < DC_MAX_SRC_SHARDS; ++s) t = sh == s ? sd.tokens[s] : t;
    return t;
}

// One lane per slot j: the sequence it holds notes it.  Of several slots that name one sequence any is noted (the next
// launch sees that the others are not); a note that nobody writes is checked before it is used.
__global__ __launch_bounds__(SCAT_BLOCK) void scatter_note_kernel(ScatArgs a) {
    const int j = blockIdx.x * SCAT_BLOCK + threadIdx.x;
    if (j >= a.n_seq) return;
    const int32_t i = a.perm[j];
    if (i < 0 || i >= a.n_seq) { set_status(a.status, DC_ERR_BAD_LAYOUT); return; }
    a.note[i] = j;
}

// Tokens to move for sequence i of rollout shard sh and where they stand in the arena: ln = 0 if no slot places it or a
// check fails (the rollout side is written, so nothing unchecked may steer a store).  Returns the error.
__device__ __forceinline__ int32_t back_source(const ScatArgs& a, const SourceDesc& sd, int i, int sh, int32_t* ln_out, int64_t* from_out) {
    *ln_out = 0;
    *from_out = 0;
    const int32_t j = a.note[i];
    const int32_t ln = a.seq_len[i];
    const int64_t so = a.src_tok_off[i], next_off = a.src_tok_off[min(i + 1, a.n_seq - 1)];
    const bool in_range = j >= 0 && j < a.n_seq;
    const int32_t named = a.perm[in_range ? j : 0];
    const int64_t from = a.dst_tok_off[in_range ? j : 0];
    if (!in_range || named != i) return 0;               // no slot names it (and then some slot is wrong: flagged there)
    const int64_t tokens = shard_tokens(sd, sh);
    const int64_t next = i + 1 >= sd.seq_off[sh + 1] ? tokens : next_off;
    if (ln <= 0 || ln > DC_MAX_SEQ_LEN) return DC_ERR_ZERO_LENGTH_SEQ;
    if (so < 0 || so + ln > tokens || so + ln > next) return DC_ERR_BAD_LAYOUT;
    if (from < 0 || from + ln > a.capacity) return DC_ERR_OVERFLOW;
    *ln_out = ln;
    *from_out = from;
    return 0;
}

// The first workgroups: the granule tables of every rollout buffer, one behind the other, each workgroup inside one
// buffer.  The others: one lane per sequence, its descriptor and the errors; one lane per slot, a slot that its sequence
// has not noted (perm names the sequence twice).
static_assert(SCAT_BLOCK == REC_BLOCK, "both parts of the launch");
__global__ __launch_bounds__(REC_BLOCK) void scatter_records_kernel(ScatArgs a, SourceDesc sd, BackSegs bs, uint32_t rec_blocks) {
    if (blockIdx.x < rec_blocks) {                       // (uniform)
        __shared__ RecLds L;
        int s = 0;                                       // my buffer, and my block's number in it
        uint32_t b = blockIdx.x;
        int32_t first_seq = 0, n = 0;
        int64_t gb = 0, n_gran = 0, tokens = 0;
        uint32_t before = 0;
#pragma unroll
        for (int q = 0; q < DC_MAX_SRC_SHARDS; ++q) {
            const int64_t grans = bs.gran_base[q + 1] - bs.gran_base[q];
            const uint32_t blocks = (uint32_t)((grans + REC_BLOCK - 1) / REC_BLOCK);
            if (b >= before && b < before + blocks) {
                s = q; first_seq = bs.first_seq[q]; n = bs.n_seq[q]; gb = bs.gran_base[q]; n_gran = grans; tokens = bs.tokens[q];
                b -= before;
                before = 0x80000000u;                    // found
            }
            if (before < 0x80000000u) before += blocks;
        }
        auto starts = [&](int i) { return i < n ? max((int64_t)0, min(a.src_tok_off[first_seq + i], tokens)) : tokens; };
        const int64_t g = (int64_t)b * REC_BLOCK + threadIdx.x;
        const int found = first_slot_after(L, n, starts, min(g, n_gran - 1) * GATHER_GRAN);
        if (g >= n_gran) return;
        build_record(n, true, starts,
                     [&](int i, int32_t* ln, int64_t* so, int32_t* sh) { back_source(a, sd, first_seq + i, s, ln, so); *sh = 0; },
                     g, a.gran_first + gb + g, a.gran_rec + gb + g, found);
        return;
    }
    const int i = (int)(blockIdx.x - rec_blocks) * REC_BLOCK + (int)threadIdx.x;
    if (i >= a.n_seq) return;
    int32_t ln;
    int64_t from;
    const int32_t e = back_source(a, sd, i, rollout_shard(sd, i), &ln, &from);
    a.r_len[i] = ln;
    a.r_src_off[i] = from;
    const int32_t named = a.perm[i];                     // (as slot i)
    const bool twice = named >= 0 && named < a.n_seq && a.note[named] != i;
    if (e != 0) set_status(a.status, e);
    else if (twice) set_status(a.status, DC_ERR_BAD_LAYOUT);
}

BackSegs make_back_segs(const SourceDesc& src) {
    BackSegs b;
    b.n_seg = src.n_src;
    uint32_t tiles = 0;
    int64_t gran = 0;
    for (int s = 0; s < DC_MAX_SRC_SHARDS; ++s) {
        const bool live = s < src.n_src && src.seq_off[s + 1] > src.seq_off[s] && src.tokens[s] > 0;
        b.first_seq[s] = s < src.n_src ? src.seq_off[s] : 0;
        b.n_seq[s] = live ? src.seq_off[s + 1] - src.seq_off[s] : 0;
        b.tokens[s] = live ? src.tokens[s] : 0;
        b.gran_base[s] = gran;
        if (live) {
            tiles += (uint32_t)((src.tokens[s] + GATHER_TILE_TOKENS - 1) / GATHER_TILE_TOKENS);
            // whole tiles plus the padding the tile mover's table loads need; a multiple of 4 entries
            gran += ((src.tokens[s] + GATHER_GRAN - 1) / GATHER_GRAN + GRAN_TABLE_PAD + 3) / 4 * 4;
        }
        b.tile_end[s] = tiles;
    }
    b.gran_base[DC_MAX_SRC_SHARDS] = gran;
    return b;
}

ScatterWorkspace carve_scatter_workspace(void* base, int32_t n_seq, const SourceDesc& src) {
    auto round_up = [](size_t x, size_t a) { return (x + a - 1) / a * a; };
    ScatterWorkspace w;
    const size_t n = (size_t)(n_seq > 0 ? n_seq : 0);
    char* p = static_cast<char*>(base);
    size_t off = 0;
    w.r_src_off = reinterpret_cast<int64_t*>(p + off); off += round_up(n * sizeof(int64_t), 256);
    w.r_len = reinterpret_cast<int32_t*>(p + off);     off += round_up(n * sizeof(int32_t), 256);
    w.note = reinterpret_cast<int32_t*>(p + off);      off += round_up(n * sizeof(int32_t), 256);
    w.n_gran_all = make_back_segs(src).gran_base[DC_MAX_SRC_SHARDS];
    w.gran_first = reinterpret_cast<int32_t*>(p + off); off += round_up((size_t)w.n_gran_all * sizeof(int32_t), 256);
    w.gran_rec = reinterpret_cast<GranRec*>(p + off);   off += round_up((size_t)w.n_gran_all * sizeof(GranRec), 256);
    w.bytes = off + 256;
    return w;
}

hipError_t launch_scatter(int32_t n_seq, const SourceDesc& src, const int64_t* d_src_tok_off,
                          const int32_t* d_seq_len, const int32_t* d_perm, const FieldTable& ft,
                          int64_t dst_capacity, const int64_t* d_dst_tok_off, const ScatterWorkspace& ws,
                          int32_t* d_status, hipStream_t st) {
    if (n_seq == 0 || ft.n_fields == 0) return hipSuccess;
    ScatArgs a;
    a.n_seq = n_seq; a.capacity = dst_capacity; a.src_tok_off = d_src_tok_off; a.seq_len = d_seq_len;
    a.perm = d_perm; a.dst_tok_off = d_dst_tok_off; a.r_src_off = ws.r_src_off;
    a.r_len = ws.r_len; a.note = ws.note; a.gran_first = ws.gran_first; a.gran_rec = ws.gran_rec; a.status = d_status;
    const unsigned grid = (unsigned)((n_seq + SCAT_BLOCK - 1) / SCAT_BLOCK);
    const BackSegs bs = make_back_segs(src);
    unsigned rec_blocks = 0;
    for (int s = 0; s < DC_MAX_SRC_SHARDS; ++s) rec_blocks += (unsigned)((bs.gran_base[s + 1] - bs.gran_base[s] + REC_BLOCK - 1) / REC_BLOCK);
    hipLaunchKernelGGL(scatter_note_kernel, dim3(grid), dim3(SCAT_BLOCK), 0, st, a);
    hipLaunchKernelGGL(scatter_records_kernel, dim3(rec_blocks + grid), dim3(REC_BLOCK), 0, st, a, src, bs, rec_blocks);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    return launch_gather_back(bs, ft, d_src_tok_off, ws, st);
}

}  // namespace dc

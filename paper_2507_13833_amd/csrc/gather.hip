// Segmented gather: rollout layout -> packed training layout (Sec. 6, "Distributed
// Databuffer": re-partitioning of a stage's outputs when the next stage's DP size
// differs).  HBM-bound; every destination byte is written once with aligned
// 16-byte stores, every source byte is read once.
//
// Work decomposition: FIELD-MAJOR.  The destination token axis is cut into tiles of 4096
// tokens; the grid walks all tiles of field 0, then all tiles of field 1, ...  At any
// moment the chip therefore streams one destination array (and the matching sequences of
// one source array) instead of all fields at once, which keeps DRAM pages open longer than
// a tile that touches every field.  One workgroup owns one tile of one field, one wavefront
// a 1024-token granule of it (1, 2 or 4 16-byte chunks per lane for 1-, 2-, 4-byte
// elements); no two workgroups ever write the same cache line.
//
// Where a chunk comes from:
//   sparse tiles (at most REC_SLOTS slots reach into each granule: the usual case) - every
//     wave works alone: it reads its granule's record (the plan left the first slots of
//     every granule inline) with ONE scalar load, which does not queue behind the bulk
//     traffic in the vector memory pipeline; when one slot covers all 64 chunks of a wave
//     instruction the source address is scalar arithmetic, else every lane selects its
//     slot with a few compares against scalar registers.  No LDS, no barrier;
//   dense granules (more slots than that: short sequences) - the wave stages the granule's slots in
//     LDS words of its own, every lane finds its chunks' slots by bisection, and what is left of the
//     slots' edges is dealt out again, one element per lane.  No barrier here either.
// A chunk inside one slot takes one (mis)aligned 16-byte source load (plus one dword
// and a byte funnel shift for 1- and 2-byte fields) and one aligned 16-byte store;
// a chunk that touches a slot boundary, padding or the arena end is copied element
// by element, all its elements in flight together.
#include <algorithm>
#include <hip/hip_ext.h>
#include "dc_device.h"
#include "dc_internal.h"

namespace dc {

constexpr int GATHER_BLOCK = 256;
static_assert(GRAN_PER_TILE == GATHER_BLOCK / WAVE, "one granule per wave");
// Carrier workgroups from which the narrow fields ride (the chip holds 2048).  A 1-byte field gains by it from about 3000 on, a
// 2-byte one, with half as much in flight as a 4-byte field itself, loses unless there are many workgroups or the others make up
// for it; the line rises with twice the 2-byte fields less the 4-byte and the 1-byte ones.  Us with workgroups of their own ->
// riding, of both directions: one 1-byte field beside one 4-byte one 36.8 -> 35.5 at 3200 workgroups, 53.9 -> 49.8 at 5000, 76.3 ->
// 70.4 at 8000; three 51.6 -> 47.3, 79.5 -> 70.7 and 115.4 -> 99.4; one 2-byte field 31.5 -> 33.5, 58.3 -> 57.6 and 83.3 -> 82.4;
// two 41.2 -> 46.0, 61.8 -> 65.8 and 95.6 -> 97.1; two and a 1-byte one 48.5 -> 54.7, 72.9 -> 76.9 and 128.3 -> 123.4; two 2-byte
// fields beside two 4-byte ones 32.9 -> 34.8, 47.4 -> 50.0 and 85.4 -> 83.1.
constexpr int64_t GATHER_RIDE_MIN_WGS = 3000, GATHER_RIDE_MAX_WGS = 8192, GATHER_RIDE_STEP_WGS = 1700;
static int64_t ride_min_workgroups(int n_four, int n_two, int n_one) {
    const int64_t line = GATHER_RIDE_MIN_WGS + GATHER_RIDE_STEP_WGS * (2 * n_two - n_four - n_one);
    return std::min(std::max(line, GATHER_RIDE_MIN_WGS), GATHER_RIDE_MAX_WGS);
}
constexpr int32_t LEN_MASK = (1 << LENSH_SHIFT) - 1;
static_assert(GATHER_GRAN == WAVE * 16, "a wave covers its granule with 1, 2 or 4 chunks per lane");
static_assert(GRAN_PER_TILE + 1 <= 8, "the tile's slice of the granule table is one 8-dword scalar load");
static_assert(GRAN_TABLE_PAD >= 8, "that load never leaves the table");
static_assert(sizeof(GranEntry) == 16, "one 16-byte load per record entry");

struct GatherArgs {
    int32_t        n_seq;
    int64_t        capacity;                     // elements of every destination arena
    const int64_t* dst_tok_off;
    const int64_t* slot_src_off;
    const int32_t* slot_len;
    const int32_t* slot_shard;
    const int32_t* gran_first;                   // padded: whole tiles plus GRAN_PER_TILE + 1 entries
    const GranRec* gran_rec;                     // same length
    uint32_t       tiles;                        // tiles per field
    uint32_t       n_carriers, n_riders;         // fields the grid walks (first in the field table), fields riding along
};

// Payload pointers are rebuilt from integers (base + offset arithmetic in scalar registers
// or LDS); typing them as global-address-space pointers keeps the accesses global_load /
// global_store instead of flat ones.
#define DC_GLOBAL __attribute__((address_space(1)))
typedef const DC_GLOBAL char* gptr;
typedef DC_GLOBAL char* gptr_w;

// One element of 1 << lg bytes (lg is uniform).
__device__ __forceinline__ uint32_t load_elem(int lg, gptr s) {
    if (lg == 2) return *reinterpret_cast<const DC_GLOBAL uint32_t*>(s);
    if (lg == 1) return *reinterpret_cast<const DC_GLOBAL uint16_t*>(s);
    return *reinterpret_cast<const DC_GLOBAL uint8_t*>(s);
}
__device__ __forceinline__ void store_elem(int lg, gptr_w d, uint32_t v) {
    if (lg == 2) *reinterpret_cast<DC_GLOBAL uint32_t*>(d) = v;
    else if (lg == 1) *reinterpret_cast<DC_GLOBAL uint16_t*>(d) = (uint16_t)v;
    else *reinterpret_cast<DC_GLOBAL uint8_t*>(d) = (uint8_t)v;
}

typedef DC_GLOBAL u32x4 g_u32x4;
typedef DC_GLOBAL u32x4_a4 g_u32x4_a4;
__device__ __forceinline__ u32x4 gload16_a4(gptr p) {
    return __builtin_nontemporal_load(reinterpret_cast<const g_u32x4_a4*>(p));
}
__device__ __forceinline__ uint32_t gload4(gptr p) {
    return __builtin_nontemporal_load(reinterpret_cast<const DC_GLOBAL uint32_t*>(p));
}
__device__ __forceinline__ void gstore16(gptr_w p, u32x4 v) {
    __builtin_nontemporal_store(v, reinterpret_cast<g_u32x4*>(p));
}
__device__ __forceinline__ void gstore4(gptr_w p, uint32_t v) {
    __builtin_nontemporal_store(v, reinterpret_cast<DC_GLOBAL uint32_t*>(p));
}

// 16 source bytes starting at byte address a (any alignment): dword loads from the address
// rounded down to 4, plus the following dword when a is not a multiple of 4; realign()
// shifts them into place (a no-op for aligned sources, e.g. every 4-byte field).
__device__ __forceinline__ void load_chunk(gptr a, u32x4& v, uint32_t& x) {
    const uintptr_t u = reinterpret_cast<uintptr_t>(a);
    gptr a4 = reinterpret_cast<gptr>(u & ~uintptr_t(3));
    v = gload16_a4(a4);
    x = (u & 3) ? gload4(a4 + 16) : 0u;
}
__device__ __forceinline__ u32x4 realign(u32x4 v, uint32_t x, uint32_t sh) {
    u32x4 o;
    o.x = __builtin_amdgcn_alignbyte(v.y, v.x, sh);
    o.y = __builtin_amdgcn_alignbyte(v.z, v.y, sh);
    o.z = __builtin_amdgcn_alignbyte(v.w, v.z, sh);
    o.w = __builtin_amdgcn_alignbyte(x, v.w, sh);
    return o;
}

// ---------------------------------------------------------------- sparse granules: one wave, no LDS
typedef uint32_t u32x8 __attribute__((ext_vector_type(8)));
typedef uint32_t u32x16 __attribute__((ext_vector_type(16)));
#define DC_CONSTANT __attribute__((address_space(4)))

// Uniform loads through the scalar data cache: they do not queue behind the bulk traffic in
// the vector memory pipeline, and their results land in scalar registers.
__device__ __forceinline__ u32x8 sload8(const void* p) {
#pragma clang diagnostic push
#pragma clang diagnostic ignored "-Wold-style-cast"
    return *(const DC_CONSTANT u32x8*)p;
#pragma clang diagnostic pop
}
__device__ __forceinline__ u32x16 sload16(const void* p) {
#pragma clang diagnostic push
#pragma clang diagnostic ignored "-Wold-style-cast"
    return *(const DC_CONSTANT u32x16*)p;
#pragma clang diagnostic pop
}

// One record entry as the selection needs it (all scalar): the slot's first token and end
// relative to the granule, and the source byte address the granule's token 0 would have
// inside the slot.
struct SlotS {
    int32_t st, en;
    int64_t ad;
};

// The 16-byte chunks of a granule that do not lie inside one slot: those that a slot's end (or the arena's) falls into and,
// where slots do not follow each other without a gap, those that a slot's start falls into.  Four of each at most, known from
// the record alone, and moved one element per lane: lane q * (tokens of a chunk) + r picks the end (start) of slot q out of the
// record by itself.  (In scalar registers, eight edges packed into words, the kernels ran out of those, 10 to 48 spilled: 1.8 M
// tokens of four fields in 2048 sequences took 11.2 us instead of 10.7, 22.6 instead of 21.4 back.)
struct EdgeElem {
    uint32_t val;
    int32_t  tok;            // the element's token inside the granule, -1: nothing there
};
template <bool STARTS>
__device__ __forceinline__ EdgeElem edge_load(const SlotS (&e)[REC_SLOTS], int lg, int lane, int32_t limit) {
    const int lg_tpc = 4 - lg, in_chunk = (1 << lg_tpc) - 1, q = lane >> lg_tpc;
    int32_t at = STARTS ? e[0].st : min(e[0].en, limit);
#pragma unroll
    for (int k = 1; k < REC_SLOTS; ++k) at = q == k ? (STARTS ? e[k].st : min(e[k].en, limit)) : at;
    const bool there = q < REC_SLOTS && at > 0 && at < (STARTS ? limit : GATHER_GRAN) && (at & in_chunk) != 0;
    const int32_t t = (at & ~in_chunk) + (lane & in_chunk);
    int32_t e_sel = INT32_MIN;
    int64_t a_sel = 0;
#pragma unroll
    for (int k = 0; k < REC_SLOTS; ++k)
        if (t >= e[k].st) { e_sel = e[k].en; a_sel = e[k].ad; }
    EdgeElem x;
    x.tok = there && t < e_sel && t < limit ? t : -1;
    x.val = 0;
    if (x.tok >= 0) x.val = load_elem(lg, reinterpret_cast<gptr>(a_sel + ((int64_t)t << lg)));
    return x;
}
// (uniform) Whether a slot starts inside the granule behind a gap (else its start is another's end).
__device__ __forceinline__ bool starts_behind_gap(const SlotS (&e)[REC_SLOTS], int32_t limit) {
    bool gap = e[0].st > 0 && e[0].st < limit;
#pragma unroll
    for (int k = 1; k < REC_SLOTS; ++k) gap = gap || (e[k].st != e[k - 1].en && e[k].st < limit);
    return gap;
}
__device__ __forceinline__ void edge_store(gptr_w dst, int lg, const EdgeElem& x) {
    if (x.tok >= 0) store_elem(lg, dst + ((int64_t)x.tok << lg), x.val);
}

// The wave's granule (1024 tokens: es chunks per lane) of one field, on its way from the granule's slots (its record) to
// its place.  MAXU: chunks per lane at most, 4, or 2 for fields of 1- and 2-byte elements.
template <int MAXU>
struct SparseMove {
    static constexpr int NARROWU = 2;                      // chunks per lane of 1- and 2-byte elements
    u32x4    v[MAXU];
    uint32_t x[NARROWU], shift[NARROWU];                   // (4-byte sources are 4-byte aligned)
    uint32_t in_mask;                                      // bit u: chunk u is inside one slot
    bool     part, gap;                                    // (uniform) not every chunk is; a slot starts behind a gap
    EdgeElem edge;
    gptr_w   dst;

    // `limit` = tokens of the granule that exist in the arena (> 0).  BACK: destination and only source are given (back_dst,
    // back_src) instead of fd's.
    template <bool BACK>
    __device__ __forceinline__ void slots(SlotS (&e)[REC_SLOTS], const FieldDesc& fd, int n_src, const char* back_src, int lg,
                                          const u32x16& rec) const {
#pragma unroll
        for (int k = 0; k < REC_SLOTS; ++k) {
            const int32_t st = (int32_t)rec[4 * k], ls = (int32_t)rec[4 * k + 1];
            const int64_t so = (int64_t)((uint64_t)rec[4 * k + 2] | ((uint64_t)rec[4 * k + 3] << 32));
            const char* base = BACK ? back_src : fd.src[0];
            if (!BACK && n_src > 1) base = fd.src[(ls >> LENSH_SHIFT) & (DC_MAX_SRC_SHARDS - 1)];
            e[k].st = st;
            e[k].en = st + (ls & LEN_MASK);
            e[k].ad = reinterpret_cast<int64_t>(base) + ((so - st) << lg);
        }
    }

    template <bool BACK>
    __device__ __forceinline__ void load(const FieldDesc& fd, int n_src, char* back_dst, const char* back_src, int lg,
                                         const u32x16& rec, int64_t wave_begin, int32_t limit) {
        const int es = 1 << lg;
        const int tpc = 16 >> lg;                          // tokens per 16-byte chunk
        const int tpi = WAVE * tpc;                        // tokens one wave instruction covers
        const int lane = threadIdx.x & (WAVE - 1);
        dst = reinterpret_cast<gptr_w>(reinterpret_cast<uintptr_t>(BACK ? back_dst : fd.dst) + (wave_begin << lg));
        SlotS e[REC_SLOTS];
        slots<BACK>(e, fd, n_src, back_src, lg, rec);
        in_mask = 0;
        part = false;
        gptr from[MAXU];
#pragma unroll
        for (int u = 0; u < MAXU; ++u) {
            from[u] = nullptr;
            if (u < es) {                                  // uniform
                const int32_t lo = u * tpi;                // the instruction's first token inside the granule
                const int32_t c0 = lo + lane * tpc;        // my chunk's first token
                // scalar: the slot of the instruction's first token; does it cover all 64 chunks?
                int32_t s_en = INT32_MIN;
                int64_t s_ad = 0;
#pragma unroll
                for (int k = 0; k < REC_SLOTS; ++k)
                    if (lo >= e[k].st) { s_en = e[k].en; s_ad = e[k].ad; }
                if (s_en >= lo + tpi && lo + tpi <= limit) {   // uniform: one slot, no search per lane
                    in_mask |= 1u << u;
                    from[u] = reinterpret_cast<gptr>(s_ad + ((int64_t)c0 << lg));
                } else {
                    part = true;
                    int32_t e_sel = INT32_MIN;
                    int64_t a_sel = 0;
#pragma unroll
                    for (int k = 0; k < REC_SLOTS; ++k)
                        if (c0 >= e[k].st) { e_sel = e[k].en; a_sel = e[k].ad; }
                    if (c0 + tpc <= e_sel && c0 + tpc <= limit) in_mask |= 1u << u;
                    from[u] = reinterpret_cast<gptr>(a_sel + ((int64_t)c0 << lg));
                }
            }
        }
#pragma unroll
        for (int u = 0; u < MAXU; ++u)
            if (in_mask & (1u << u)) {
                if (u < NARROWU) {
                    shift[u] = (uint32_t)reinterpret_cast<uintptr_t>(from[u]) & 3u;
                    load_chunk(from[u], v[u], x[u]);
                } else {
                    v[u] = gload16_a4(from[u]);
                }
            }
        // the edges' elements go out with the loads above, so a wave with a sequence boundary in its granule (two waves in
        // five, or all of them) pays no second round trip
        edge.tok = -1;
        edge.val = 0;
        gap = false;
        if (part) {
            edge = edge_load<false>(e, lg, lane, limit);
            gap = starts_behind_gap(e, limit);
        }
    }

    // The edges in front of the whole chunks, where they wait for the last load: beside the chunks next to them they fill their
    // lines at once.  31 M tokens in 65 536 sequences 146 -> 139 us, 158 -> 150 back; 24 M of two 4-byte fields and a 2-byte one
    // 100.5 -> 98.2 back.
    template <bool BACK>
    __device__ __forceinline__ void store(const FieldDesc& fd, int n_src, const char* back_src, int lg, const u32x16& rec,
                                          int32_t limit) const {
        const int lane = threadIdx.x & (WAVE - 1);
        if (part) edge_store(dst, lg, edge);               // (uniform)
#pragma unroll
        for (int u = 0; u < MAXU; ++u)
            if (in_mask & (1u << u)) gstore16(dst + (u * WAVE + lane) * 16, u < NARROWU ? realign(v[u], x[u], shift[u]) : v[u]);
        if (!gap) return;                                  // (uniform)
        SlotS e[REC_SLOTS];
        slots<BACK>(e, fd, n_src, back_src, lg, rec);
        edge_store(dst, lg, edge_load<true>(e, lg, lane, limit));
    }
};

// ---------------------------------------------------------------- dense granules: one wave, LDS words of its own
// The slots that reach into a granule, relative to its first token, DENSE_SLOTS at a time.  A pass serves the tokens
// before the slot behind its last one, whose start the last entry holds ("no slot" if there is none); a chunk that this
// start falls into is served by both passes, each its own tokens.  Lane k stages slot k.
// Bound by latency: the granule's table entries, the slots' descriptors and the payload are each one trip to memory for
// the whole granule.  The gather kernel takes 6.2 us for 15 550 tokens in 64 sequences and 34 us for 3.3 M tokens in 15 360 (5
// fields).  With the slots staged per tile by the workgroup, one chunk per lane at a time and an edge chunk's elements one
// after the other it took 14.7 and 70 us.
constexpr int DENSE_SLOTS = WAVE - 1;
constexpr int DENSE_CHUNKS = GATHER_GRAN / 4;                  // chunks of a granule of 4-byte elements, the most there are
struct WaveSlots {
    int32_t  start[WAVE];          // first destination token of the slot (REL_FAR: none)
    int32_t  end[WAVE];            // one past its last token
    int64_t  addr[WAVE];           // source byte address of the granule's token 0 (may lie before the buffer)
    uint32_t adv[WAVE];            // (advantage arena) bits of the slot's advantage
    uint32_t edge[DENSE_CHUNKS];   // chunks that do not lie inside one slot: first token | (slot + 1) << 16
};
static_assert(GATHER_GRAN <= (1 << 16), "a token of the granule and a slot share a word");

// Stage slots from `base` on; src0: the only rollout buffer (n_src == 1), else fd.src[] has the slot's.
__device__ __forceinline__ void stage_wave_slots(const GatherArgs& a, WaveSlots& sg, const FieldDesc& fd, int n_src,
                                                 const char* src0, int lg, int lane, int base, int last, int64_t wave_begin) {
    const int j = base + lane;
    int32_t st = REL_FAR, en = REL_FAR;
    int64_t ad = 0;
    if (j <= last) {
        const int64_t d = a.dst_tok_off[j] - wave_begin;
        st = (int32_t)max((int64_t)-REL_FAR, min((int64_t)REL_FAR, d));
        en = st + a.slot_len[j];
        const char* from = src0;
        if (n_src > 1) from = fd.src[a.slot_shard[j] & (DC_MAX_SRC_SHARDS - 1)];
        ad = reinterpret_cast<int64_t>(from) + ((a.slot_src_off[j] - d) << lg);
    }
    __builtin_amdgcn_wave_barrier();                       // (the wave's reads of the pass before come first)
    sg.start[lane] = st; sg.end[lane] = en; sg.addr[lane] = ad;
    __builtin_amdgcn_wave_barrier();
}

// First token behind this pass; *more: the granule has slots left behind it.
__device__ __forceinline__ int32_t dense_pass_end(const WaveSlots& sg, int32_t limit, bool* more) {
    const int32_t next = __builtin_amdgcn_readfirstlane(sg.start[DENSE_SLOTS]);
    *more = next < limit;
    return *more ? next : limit;
}

// Lanes of the mask below this one.
__device__ __forceinline__ int lanes_below(uint64_t mask) {
    return (int)__builtin_amdgcn_mbcnt_hi((uint32_t)(mask >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)mask, 0u));
}

// The probe distance a bisection over n slots starts with (2 p - 1 >= n; n <= DENSE_SLOTS).
__device__ __forceinline__ int dense_first_step(int n) {
    return 1 << (31 - __builtin_clz((uint32_t)max(n, 1)));
}

// The wave's granule of one field, slots first .. last reaching into it (same arguments as SparseMove::load otherwise).
template <bool BACK>
__device__ __forceinline__ void move_wave_dense(const GatherArgs& a, WaveSlots& sg, const FieldDesc& fd, int n_src,
                                                char* back_dst, const char* back_src, int lg, int first, int last,
                                                int64_t wave_begin, int32_t limit) {
    const int es = 1 << lg;
    const int lg_tpc = 4 - lg, tpc = 16 >> lg;             // tokens per 16-byte chunk
    int lane = threadIdx.x & (WAVE - 1);
    gptr_w dst = reinterpret_cast<gptr_w>(reinterpret_cast<uintptr_t>(BACK ? back_dst : fd.dst) + (wave_begin << lg));
    constexpr int MAXU = 4, NARROWU = 2;                   // chunks per lane; of 1- and 2-byte elements
    int base = first;
    int32_t pass_begin = 0;
    for (;;) {
        asm volatile("" : "+v"(lane), "+s"(base));         // (what depends on them is worked out here, not kept across passes and fields)
        stage_wave_slots(a, sg, fd, BACK ? 1 : n_src, BACK ? back_src : fd.src[0], lg, lane, base, last, wave_begin);
        bool more;
        const int32_t pass_end = dense_pass_end(sg, limit, &more);
        // ---- every chunk's slot: the last one that starts at or before it ----
        int k[MAXU];
#pragma unroll
        for (int u = 0; u < MAXU; ++u) k[u] = -1;
#pragma unroll 1
        for (int step = dense_first_step(min(last - base + 1, DENSE_SLOTS)); step >= 1; step >>= 1) {   // (uniform)
#pragma unroll
            for (int u = 0; u < MAXU; ++u)
                if (u < es && sg.start[min(k[u] + step, WAVE - 1)] <= (u * WAVE + lane) * tpc) k[u] += step;
        }
        // ---- chunks inside one slot; the others are listed ----
        uint32_t in_mask = 0;                              // bit u: chunk u is inside one slot
        int n_edge = 0;                                    // (uniform)
#pragma unroll
        for (int u = 0; u < MAXU; ++u) {
            if (u < es) {                                  // uniform
                const int32_t c0 = (u * WAVE + lane) * tpc;
                const bool mine = c0 + tpc > pass_begin && c0 < pass_end;
                const bool in = c0 >= pass_begin && k[u] >= 0 && c0 + tpc <= min(sg.end[max(k[u], 0)], pass_end);
                if (in) in_mask |= 1u << u;
                const uint64_t edges = __ballot(mine && !in);
                if (mine && !in) sg.edge[n_edge + lanes_below(edges)] = (uint32_t)c0 | ((uint32_t)(k[u] + 1) << 16);
                n_edge += __popcll(edges);
            }
        }
        __builtin_amdgcn_wave_barrier();
        u32x4 v[MAXU];
        uint32_t x[NARROWU], shift[NARROWU];               // (4-byte sources are 4-byte aligned)
#pragma unroll
        for (int u = 0; u < MAXU; ++u)
            if (in_mask & (1u << u)) {
                gptr from = reinterpret_cast<gptr>(sg.addr[k[u]] + (u * WAVE + lane) * 16);
                if (u < NARROWU) {
                    shift[u] = (uint32_t)reinterpret_cast<uintptr_t>(from) & 3u;
                    load_chunk(from, v[u], x[u]);
                } else {
                    v[u] = gload16_a4(from);
                }
            }
        // ---- the listed chunks, one element per lane: the first EDGE_MAX elements' loads go out with the loads above ----
        constexpr int EDGE_MAX = 2;
        const int n_items = n_edge << lg_tpc;              // (uniform)
        uint32_t val[EDGE_MAX];
        int32_t tok[EDGE_MAX];                             // the element's token, -1: nothing there
        auto edge_load = [&](int from_item) {
#pragma unroll
            for (int r = 0; r < EDGE_MAX; ++r) {
                tok[r] = -1;
                val[r] = 0;
                const int item = from_item + r * WAVE + lane;
                if (from_item + r * WAVE < n_items) {      // uniform
                    const uint32_t e = sg.edge[min(item >> lg_tpc, DENSE_CHUNKS - 1)];
                    const int32_t t = (int32_t)(e & 0xFFFFu) + (item & (tpc - 1));
                    int q = (int)(e >> 16) - 1;
                    if (item < n_items) {
                        while (q + 1 < WAVE && sg.start[q + 1] <= t) ++q;
                        if (q >= 0 && t >= pass_begin && t < min(sg.end[q], pass_end)) {
                            tok[r] = t;
                            val[r] = load_elem(lg, reinterpret_cast<gptr>(sg.addr[q] + ((int64_t)t << lg)));
                        }
                    }
                }
            }
        };
        auto edge_store = [&]() {
#pragma unroll
            for (int r = 0; r < EDGE_MAX; ++r)
                if (tok[r] >= 0) store_elem(lg, dst + ((int64_t)tok[r] << lg), val[r]);
        };
        if (n_items > 0) edge_load(0);
        asm volatile("" : "+v"(lane));
#pragma unroll
        for (int u = 0; u < MAXU; ++u)
            if (in_mask & (1u << u)) {
                gstore16(dst + (u * WAVE + lane) * 16, u < NARROWU ? realign(v[u], x[u], shift[u]) : v[u]);
            }
        if (n_items > 0) edge_store();
#pragma unroll 1
        for (int item = EDGE_MAX * WAVE; item < n_items; item += EDGE_MAX * WAVE) {
            edge_load(item);
            edge_store();
        }
        if (!more) break;
        base += DENSE_SLOTS;
        pass_begin = pass_end;
    }
}

// ---------------------------------------------------------------- per-token advantage made on the way
// The advantage field of the training layout without its rollout-layout copy: the value of a
// token is its sequence's advantage where the sequence's mask byte is non-zero and +0.0f
// elsewhere (selection, as in the advantage stage), so the gather reads the 1-byte mask where
// it would read a 4-byte field.  These workgroups also move the mask field itself, from the
// bytes they have loaded anyway.
struct AdvSynth {
    const int32_t* perm;          // [N] slot -> sequence
    const float*   adv_seq;       // [N] advantage of every sequence
    float*         dst;           // float32 arena of the training layout
};
// It travels in the field table, in the entry behind the mask's (dst = the arena, src[0] = perm,
// src[1] = adv_seq), and is read from there by the workgroups that need it: as kernel arguments of
// their own the pointers would sit in scalar registers of every workgroup.
__device__ __forceinline__ AdvSynth adv_synth_of(const FieldDesc& fd) {
    AdvSynth s;
    s.perm = reinterpret_cast<const int32_t*>(fd.src[0]);
    s.adv_seq = reinterpret_cast<const float*>(fd.src[1]);
    s.dst = reinterpret_cast<float*>(fd.dst);
    return s;
}

__device__ __forceinline__ uint32_t sload1(const void* p) {
#pragma clang diagnostic push
#pragma clang diagnostic ignored "-Wold-style-cast"
    return *(const DC_CONSTANT uint32_t*)p;
#pragma clang diagnostic pop
}

// Advantage bits of the output slots first .. first + REC_SLOTS - 1 (indices clamped into the
// arrays whatever perm holds).  Two batches of scalar loads: one round trip each.
__device__ __forceinline__ void slot_adv_scalar(const AdvSynth& s, int N, int first, uint32_t (&adv)[REC_SLOTS]) {
    uint32_t q[REC_SLOTS];
#pragma unroll
    for (int k = 0; k < REC_SLOTS; ++k) q[k] = sload1(s.perm + min(first + k, N - 1));
#pragma unroll
    for (int k = 0; k < REC_SLOTS; ++k) adv[k] = sload1(s.adv_seq + min(q[k], (uint32_t)(N - 1)));
}

// The two aligned words that hold the 4 mask bytes at byte address p (any alignment), and the
// output chunk of those 4 tokens.
__device__ __forceinline__ void load_mask4(gptr p, uint32_t& w0, uint32_t& w1) {
    const uintptr_t u = reinterpret_cast<uintptr_t>(p);
    gptr a4 = reinterpret_cast<gptr>(u & ~uintptr_t(3));
    w0 = gload4(a4);
    w1 = (u & 3) ? gload4(a4 + 4) : 0u;
}
__device__ __forceinline__ uint32_t mask4_of(uint32_t w0, uint32_t w1, gptr p) {
    return __builtin_amdgcn_alignbyte(w1, w0, (uint32_t)reinterpret_cast<uintptr_t>(p) & 3u);
}
__device__ __forceinline__ u32x4 select_adv4(uint32_t m, uint32_t adv) {
    u32x4 o;
    o.x = (m & 0x000000FFu) ? adv : 0u;
    o.y = (m & 0x0000FF00u) ? adv : 0u;
    o.z = (m & 0x00FF0000u) ? adv : 0u;
    o.w = (m & 0xFF000000u) ? adv : 0u;
    return o;
}

constexpr int ADV_TPC = 4;                    // tokens per 16-byte chunk of the float32 output
constexpr int ADV_TPI = WAVE * ADV_TPC;       // tokens one wave instruction covers

// The wave's granule of the advantage arena, slots from the granule's record, their advantage
// bits in adv[].  `mk` is the mask field.
__device__ __forceinline__ void adv_wave_sparse(const FieldDesc& mk, int n_src, const AdvSynth& s,
                                                const uint32_t (&adv)[REC_SLOTS], const u32x16& rec, int64_t wave_begin,
                                                int32_t limit) {
    const int lane = threadIdx.x & (WAVE - 1);
    gptr_w dst = reinterpret_cast<gptr_w>(reinterpret_cast<uintptr_t>(s.dst) + (wave_begin << 2));
    gptr_w mdst = reinterpret_cast<gptr_w>(reinterpret_cast<uintptr_t>(mk.dst) + wave_begin);

    const char* base[REC_SLOTS];                           // one batch of scalar loads
#pragma unroll
    for (int k = 0; k < REC_SLOTS; ++k)
        base[k] = n_src > 1 ? mk.src[((int32_t)rec[4 * k + 1] >> LENSH_SHIFT) & (DC_MAX_SRC_SHARDS - 1)] : mk.src[0];
    SlotS e[REC_SLOTS];                                    // ad: byte address of the granule's token 0 in the mask
#pragma unroll
    for (int k = 0; k < REC_SLOTS; ++k) {
        const int32_t st = (int32_t)rec[4 * k], ls = (int32_t)rec[4 * k + 1];
        const int64_t so = (int64_t)((uint64_t)rec[4 * k + 2] | ((uint64_t)rec[4 * k + 3] << 32));
        e[k].st = st;
        e[k].en = st + (ls & LEN_MASK);
        e[k].ad = reinterpret_cast<int64_t>(base[k]) + (so - st);
    }

    constexpr int NU = GATHER_GRAN / ADV_TPI;              // 4 chunks per lane
    uint32_t in_mask = 0, bnd_mask = 0;
    gptr from[NU];
    uint32_t av[NU];
#pragma unroll
    for (int u = 0; u < NU; ++u) {
        const int32_t lo = u * ADV_TPI;
        const int32_t c0 = lo + lane * ADV_TPC;
        int32_t s_en = INT32_MIN;
        int64_t s_ad = 0;
        uint32_t s_av = 0;
#pragma unroll
        for (int k = 0; k < REC_SLOTS; ++k)
            if (lo >= e[k].st) { s_en = e[k].en; s_ad = e[k].ad; s_av = adv[k]; }
        if (s_en >= lo + ADV_TPI && lo + ADV_TPI <= limit) {       // uniform: one slot serves the instruction
            in_mask |= 1u << u;
            from[u] = reinterpret_cast<gptr>(s_ad + c0);
            av[u] = s_av;
        } else {
            int32_t e_sel = INT32_MIN;
            int64_t a_sel = 0;
            uint32_t v_sel = 0;
#pragma unroll
            for (int k = 0; k < REC_SLOTS; ++k)
                if (c0 >= e[k].st) { e_sel = e[k].en; a_sel = e[k].ad; v_sel = adv[k]; }
            const bool in = c0 + ADV_TPC <= e_sel && c0 + ADV_TPC <= limit;
            if (in) in_mask |= 1u << u;
            else if (c0 < limit) bnd_mask |= 1u << u;
            from[u] = reinterpret_cast<gptr>(a_sel + c0);
            av[u] = v_sel;
        }
    }
    uint32_t w0[NU], w1[NU];
#pragma unroll
    for (int u = 0; u < NU; ++u)
        if (in_mask & (1u << u)) load_mask4(from[u], w0[u], w1[u]);
#pragma unroll
    for (int u = 0; u < NU; ++u)
        if (in_mask & (1u << u)) {
            const uint32_t m = mask4_of(w0[u], w1[u], from[u]);
            gstore16(dst + (u * WAVE + lane) * 16, select_adv4(m, av[u]));
            gstore4(mdst + (u * WAVE + lane) * 4, m);      // the mask's own move: the bytes are here already
        }
    // ---- chunks that touch a slot boundary, padding or the arena end: token by token ----
    if (__ballot(bnd_mask != 0) == 0ull) return;                             // uniform
#pragma unroll 1
    for (int u = 0; u < NU; ++u) {
        const bool mine = (bnd_mask >> u) & 1u;
        if (__ballot(mine) == 0ull) continue;                                // uniform
        const int32_t c0 = u * ADV_TPI + lane * ADV_TPC;
        uint32_t val[ADV_TPC], sel[ADV_TPC];
        bool ok[ADV_TPC];
#pragma unroll
        for (int r = 0; r < ADV_TPC; ++r) {
            const int32_t t = c0 + r;
            int32_t e_sel = INT32_MIN;
            int64_t a_sel = 0;
            sel[r] = 0;
#pragma unroll
            for (int k = 0; k < REC_SLOTS; ++k)
                if (t >= e[k].st) { e_sel = e[k].en; a_sel = e[k].ad; sel[r] = adv[k]; }
            ok[r] = mine && t < e_sel && t < limit;
            val[r] = 0;
            if (ok[r]) val[r] = load_elem(0, reinterpret_cast<gptr>(a_sel + t));
        }
#pragma unroll
        for (int r = 0; r < ADV_TPC; ++r)
            if (ok[r]) {
                store_elem(2, dst + ((int64_t)(c0 + r) << 2), val[r] ? sel[r] : 0u);
                store_elem(0, mdst + (c0 + r), val[r]);
            }
    }
}

// The same for a granule with more slots than its record holds: slots and their advantages staged in the wave's LDS words.
__device__ __forceinline__ void adv_wave_dense(const GatherArgs& a, WaveSlots& sg, const FieldDesc& mk, int n_src,
                                               const AdvSynth& s, int first, int last, int64_t wave_begin, int32_t limit) {
    int lane = threadIdx.x & (WAVE - 1);
    const int N = a.n_seq;
    gptr_w dst = reinterpret_cast<gptr_w>(reinterpret_cast<uintptr_t>(s.dst) + (wave_begin << 2));
    gptr_w mdst = reinterpret_cast<gptr_w>(reinterpret_cast<uintptr_t>(mk.dst) + wave_begin);
    constexpr int NU = GATHER_GRAN / ADV_TPI;
    int base = first;
    int32_t pass_begin = 0;
    for (;;) {
        asm volatile("" : "+v"(lane), "+s"(base));
        uint32_t av = 0;
        if (lane < DENSE_SLOTS && base + lane <= last) {
            const uint32_t sq = min((uint32_t)s.perm[base + lane], (uint32_t)(N - 1));
            av = __float_as_uint(s.adv_seq[sq]);
        }
        stage_wave_slots(a, sg, mk, n_src, mk.src[0], 0, lane, base, last, wave_begin);            // addresses in mask bytes
        sg.adv[lane] = av;
        __builtin_amdgcn_wave_barrier();
        bool more;
        const int32_t pass_end = dense_pass_end(sg, limit, &more);
        int k[NU];
#pragma unroll
        for (int u = 0; u < NU; ++u) k[u] = -1;
#pragma unroll 1
        for (int step = dense_first_step(min(last - base + 1, DENSE_SLOTS)); step >= 1; step >>= 1) {   // (uniform)
#pragma unroll
            for (int u = 0; u < NU; ++u)
                if (sg.start[min(k[u] + step, WAVE - 1)] <= (u * WAVE + lane) * ADV_TPC) k[u] += step;
        }
        uint32_t in_mask = 0;
        int n_edge = 0;                                    // (uniform)
        gptr from[NU];
        uint32_t w0[NU], w1[NU], sel[NU];
#pragma unroll
        for (int u = 0; u < NU; ++u) {
            const int32_t c0 = (u * WAVE + lane) * ADV_TPC;
            const int at = max(k[u], 0);
            const bool mine = c0 + ADV_TPC > pass_begin && c0 < pass_end;
            const bool in = c0 >= pass_begin && k[u] >= 0 && c0 + ADV_TPC <= min(sg.end[at], pass_end);
            if (in) in_mask |= 1u << u;
            from[u] = reinterpret_cast<gptr>(sg.addr[at] + c0);
            sel[u] = sg.adv[at];
            const uint64_t edges = __ballot(mine && !in);
            if (mine && !in) sg.edge[n_edge + lanes_below(edges)] = (uint32_t)c0 | ((uint32_t)(k[u] + 1) << 16);
            n_edge += __popcll(edges);
        }
        __builtin_amdgcn_wave_barrier();
#pragma unroll
        for (int u = 0; u < NU; ++u)
            if (in_mask & (1u << u)) load_mask4(from[u], w0[u], w1[u]);
#pragma unroll
        for (int u = 0; u < NU; ++u)
            if (in_mask & (1u << u)) {
                const uint32_t m = mask4_of(w0[u], w1[u], from[u]);
                gstore16(dst + (u * WAVE + lane) * 16, select_adv4(m, sel[u]));
                gstore4(mdst + (u * WAVE + lane) * 4, m);
            }
#pragma unroll 1
        for (int item = lane; item < n_edge * ADV_TPC; item += WAVE) {        // one token per lane
            const uint32_t e = sg.edge[item / ADV_TPC];
            const int32_t t = (int32_t)(e & 0xFFFFu) + (item & (ADV_TPC - 1));
            int q = (int)(e >> 16) - 1;
            while (q + 1 < WAVE && sg.start[q + 1] <= t) ++q;
            if (q >= 0 && t >= pass_begin && t < min(sg.end[q], pass_end)) {
                const uint32_t m = load_elem(0, reinterpret_cast<gptr>(sg.addr[q] + t));
                store_elem(2, dst + ((int64_t)t << 2), m ? sg.adv[q] : 0u);
                store_elem(0, mdst + t, m);
            }
        }
        if (!more) break;
        base += DENSE_SLOTS;
        pass_begin = pass_end;
    }
}

// ---------------------------------------------------------------- the kernel
// What wave w of a tile needs of its granule.  F[g] = first slot ending after granule g's first token; slots F[g] ..
// F[g + 1] are the ones that can reach into granule g.  The tables are padded, so the entries of a whole tile (and one
// more) exist even for the last, partial tile.
struct WaveGran {
    u32x16  rec;
    int     first, last;           // slots that can reach into the granule
    int32_t limit;                 // tokens of it that exist in the arena
};
__device__ __forceinline__ WaveGran wave_granule(const GatherArgs& a, uint32_t tile, int w) {
    const int64_t g0 = (int64_t)tile * GRAN_PER_TILE;
    const u32x8 F = sload8(a.gran_first + g0);
    WaveGran g;
    g.rec = sload16(a.gran_rec + g0 + w);
    g.first = (int)F[0];
    int next = (int)F[1];
#pragma unroll
    for (int i = 1; i < GRAN_PER_TILE; ++i)
        if (w == i) { g.first = (int)F[i]; next = (int)F[i + 1]; }
    g.last = min(max(next, g.first), a.n_seq - 1);
    g.limit = (int32_t)max((int64_t)0, min((int64_t)GATHER_GRAN, a.capacity - (g0 + w) * GATHER_GRAN));
    return g;
}

// The tile `tile` of carrier field fc.  BACK = false: the forward direction, fields as the
// table gives them.  BACK = true: the reverse direction, destination = the field's rollout
// buffer of segment seg, only source = its training arena.
template <bool BACK>
__device__ __forceinline__ void move_tile(const GatherArgs& a, const FieldTable& ft, WaveSlots* slots, uint32_t tile, uint32_t fc,
                                          int seg) {
    const int w = __builtin_amdgcn_readfirstlane((int)(threadIdx.x / WAVE));
    const int N = a.n_seq;
    const int64_t wave_begin = (int64_t)tile * GATHER_TILE_TOKENS + w * GATHER_GRAN;
    const WaveGran g = wave_granule(a, tile, w);
    if (g.limit <= 0 || g.first < 0 || g.first >= N) return;      // behind the arena's end, or nothing reaches into the granule

    // f = fc, then the riders n_carriers + fc, n_carriers + fc + n_carriers, ...  (Two loops rather than a test inside one:
    // the registers of the one path do not add to the other's.)
    const uint32_t n = a.n_carriers + a.n_riders;
    auto next_field = [&](uint32_t f) { return f < a.n_carriers ? a.n_carriers + f : f + a.n_carriers; };
    auto lg_of = [&](const FieldDesc& fd) { return fd.elem_bytes == 4 ? 2 : (fd.elem_bytes == 2 ? 1 : 0); };
    if (g.last - g.first < REC_SLOTS) {
        // (a wave's loads and stores retire in one order, so a field's loads issued behind another's stores wait for those:
        //  the first rider's go out in front of the carrier's stores)
        auto load = [&](auto& m, const FieldDesc& fd) {
            m.template load<BACK>(fd, ft.n_src, BACK ? const_cast<char*>(fd.src[seg]) : nullptr, BACK ? fd.dst : nullptr, lg_of(fd), g.rec,
                                  wave_begin, g.limit);
        };
        auto store = [&](auto& m, const FieldDesc& fd) {
            m.template store<BACK>(fd, ft.n_src, BACK ? fd.dst : nullptr, lg_of(fd), g.rec, g.limit);
        };
        SparseMove<4> m;
        load(m, ft.f[fc]);
        uint32_t f = next_field(fc);
        if (f < n) {                                              // (uniform)
            SparseMove<2> r;
            load(r, ft.f[f]);
            store(m, ft.f[fc]);
            store(r, ft.f[f]);
            for (f = next_field(f); f < n; f = next_field(f)) {
                load(r, ft.f[f]);
                store(r, ft.f[f]);
            }
        } else {
            store(m, ft.f[fc]);
        }
    } else {
        for (uint32_t f = fc; f < n; f = next_field(f)) {
            const FieldDesc& fd = ft.f[f];
            move_wave_dense<BACK>(a, slots[w], fd, ft.n_src, BACK ? const_cast<char*>(fd.src[seg]) : nullptr, BACK ? fd.dst : nullptr,
                                  lg_of(fd), g.first, g.last, wave_begin, g.limit);
        }
    }
}

// One workgroup per tile of GATHER_TILE_TOKENS tokens of one field, field-major.  Waves are short-lived on purpose: a wave that ends right
// after issuing its stores does not hold its slot until they are acknowledged, which a
// looping wave would (loads and stores retire through one in-order counter).
__global__ __launch_bounds__(GATHER_BLOCK) void gather_kernel(GatherArgs a, FieldTable ft) {
    // The grid walks the "carrier" fields, field after field (the 4-byte fields if there are
    // any, else every field).  Narrower fields ride along: rider r is moved by the waves of
    // carrier r mod n_carriers, right after their own data and from the same granule record.
    // A wave of a narrow field has only 1 or 2 KB in flight; as a workgroup of its own it
    // would hold a wave slot as long as a 4 KB one.
    // (the division runs in the vector unit; the wave's place is the same in every lane)
    const uint32_t fc = (uint32_t)__builtin_amdgcn_readfirstlane((int)(blockIdx.x / a.tiles));
    __shared__ WaveSlots slots[GRAN_PER_TILE];
    move_tile<false>(a, ft, slots, blockIdx.x - fc * a.tiles, fc, 0);
}

// The tile `tile` of the advantage arena and of the mask field.
__device__ __forceinline__ void adv_tile(const GatherArgs& a, const FieldTable& ft, WaveSlots* slots, uint32_t mask_field,
                                         uint32_t tile) {
    const int w = __builtin_amdgcn_readfirstlane((int)(threadIdx.x / WAVE));
    const int N = a.n_seq;
    const int64_t wave_begin = (int64_t)tile * GATHER_TILE_TOKENS + w * GATHER_GRAN;
    const WaveGran g = wave_granule(a, tile, w);
    if (g.limit <= 0 || g.first < 0 || g.first >= N) return;

    const FieldDesc& mk = ft.f[mask_field];
    const AdvSynth s = adv_synth_of(ft.f[mask_field + 1]);
    if (g.last - g.first < REC_SLOTS) {
        uint32_t adv[REC_SLOTS];
        slot_adv_scalar(s, N, g.first, adv);
        adv_wave_sparse(mk, ft.n_src, s, adv, g.rec, wave_begin, g.limit);
    } else {
        adv_wave_dense(a, slots[w], mk, ft.n_src, s, g.first, g.last, wave_begin, g.limit);
    }
}

// gather_kernel with one more "carrier" behind the others: the advantage arena, made from the mask.
__global__ __launch_bounds__(GATHER_BLOCK) void gather_adv_kernel(GatherArgs a, FieldTable ft, uint32_t mask_field) {
    // The advantage tiles write four bytes for every byte they read; a run of them at the end of the
    // grid would be a pure write stream, which the memory serves more slowly than a mix.  They are
    // dealt in between the others instead: every (n_carriers + 1)-th workgroup takes one.
    __shared__ WaveSlots slots[GRAN_PER_TILE];
    const uint32_t per = a.n_carriers + 1;
    const uint32_t round = blockIdx.x / per, r = blockIdx.x % per;
    if (r == a.n_carriers) {
        adv_tile(a, ft, slots, mask_field, (uint32_t)__builtin_amdgcn_readfirstlane((int)round));
    } else {
        const uint32_t idx = round * a.n_carriers + r;
        move_tile<false>(a, ft, slots, (uint32_t)__builtin_amdgcn_readfirstlane((int)(idx % a.tiles)),
                         (uint32_t)__builtin_amdgcn_readfirstlane((int)(idx / a.tiles)), 0);
    }
}

// Reverse direction: the same grid over the tiles of all rollout buffers, one behind the other.
// a.dst_tok_off, a.slot_* and the granule tables arrive as the arrays of all segments; the
// workgroup narrows them to its segment's part.
__global__ __launch_bounds__(GATHER_BLOCK) void gather_back_kernel(GatherArgs a, FieldTable ft, BackSegs bs) {
    const uint32_t fc = (uint32_t)__builtin_amdgcn_readfirstlane((int)(blockIdx.x / a.tiles));
    const uint32_t t = blockIdx.x - fc * a.tiles;
    int seg = 0;
#pragma unroll
    for (int q = 0; q + 1 < DC_MAX_SRC_SHARDS; ++q) seg += t >= bs.tile_end[q] ? 1 : 0;   // t < tile_end[last]
    const uint32_t tile = t - (seg > 0 ? bs.tile_end[seg - 1] : 0u);
    const int first_seq = bs.first_seq[seg];
    a.n_seq = bs.n_seq[seg];
    a.capacity = bs.tokens[seg];
    a.dst_tok_off += first_seq;
    a.slot_src_off += first_seq;
    a.slot_len += first_seq;
    a.gran_first += bs.gran_base[seg];
    a.gran_rec += bs.gran_base[seg];
    __shared__ WaveSlots slots[GRAN_PER_TILE];
    move_tile<true>(a, ft, slots, tile, fc, seg);
}

// Field table with the 4-byte fields first (they carry, the others ride) and the grid's shape.
// skip >= 0: that field goes behind all others and neither carries nor rides (its place is returned).
static int order_fields(const FieldTable& ft, int64_t tiles, FieldTable* sorted, GatherArgs* a, int skip = -1) {
    *sorted = ft;
    int n = 0, n_wide = 0;
    for (int pass = 0; pass < 2; ++pass)
        for (int f = 0; f < ft.n_fields; ++f)
            if (f != skip && (ft.f[f].elem_bytes == 4) == (pass == 0)) {
                sorted->f[n++] = ft.f[f];
                if (pass == 0) n_wide = n;
            }
    const int n_moved = n;
    if (skip >= 0) sorted->f[n] = ft.f[skip];
    // riding pays when the carriers alone give the chip several rounds of workgroups; a small
    // batch needs every workgroup it can get
    int n_two = 0;
    for (int f = n_wide; f < n_moved; ++f) n_two += sorted->f[f].elem_bytes == 2 ? 1 : 0;
    const bool ride = n_wide > 0 && tiles * n_wide >= ride_min_workgroups(n_wide, n_two, n_moved - n_wide - n_two);
    a->n_carriers = (uint32_t)(ride ? n_wide : n_moved);
    a->n_riders = (uint32_t)n_moved - a->n_carriers;
    a->tiles = (uint32_t)tiles;
    return n_moved;
}

hipError_t launch_gather(int32_t n_seq, const FieldTable& ft, int64_t dst_capacity,
                         const int64_t* d_dst_tok_off, const Workspace& ws, hipStream_t st,
                         hipEvent_t begins, hipEvent_t ends) {
    if (n_seq == 0 || ft.n_fields == 0 || dst_capacity == 0) return hipSuccess;
    GatherArgs a;
    a.n_seq = n_seq;
    a.capacity = dst_capacity;
    a.dst_tok_off = d_dst_tok_off;
    a.slot_src_off = ws.slot_src_off;
    a.slot_len = ws.slot_len;
    a.slot_shard = ws.slot_shard;
    a.gran_first = ws.gran_first;
    a.gran_rec = ws.gran_rec;
    const int64_t tiles = (dst_capacity + GATHER_TILE_TOKENS - 1) / GATHER_TILE_TOKENS;
    if (tiles * ft.n_fields > 0x7FFFFFFFLL || tiles * GRAN_PER_TILE + GRAN_PER_TILE + 1 > ws.n_gran)
        return hipErrorInvalidValue;
    FieldTable sorted;
    order_fields(ft, tiles, &sorted, &a);
    if (begins || ends)                                   // the dispatch itself carries the two events
        hipExtLaunchKernelGGL(gather_kernel, dim3((unsigned)(tiles * a.n_carriers)), dim3(GATHER_BLOCK), 0, st, begins, ends,
                              0, a, sorted);
    else
        hipLaunchKernelGGL(gather_kernel, dim3((unsigned)(tiles * a.n_carriers)), dim3(GATHER_BLOCK), 0, st, a, sorted);
    return hipGetLastError();
}

hipError_t launch_gather_advantage(int32_t n_seq, const FieldTable& ft, int mask_field, const int32_t* d_perm,
                                   const float* d_adv_seq, float* d_adv_tok_dst, int64_t dst_capacity,
                                   const int64_t* d_dst_tok_off, const Workspace& ws, hipStream_t st) {
    if (n_seq == 0 || dst_capacity == 0) return hipSuccess;
    if (mask_field < 0 || mask_field >= ft.n_fields || ft.f[mask_field].elem_bytes != 1) return hipErrorInvalidValue;
    GatherArgs a;
    a.n_seq = n_seq;
    a.capacity = dst_capacity;
    a.dst_tok_off = d_dst_tok_off;
    a.slot_src_off = ws.slot_src_off;
    a.slot_len = ws.slot_len;
    a.slot_shard = ws.slot_shard;
    a.gran_first = ws.gran_first;
    a.gran_rec = ws.gran_rec;
    const int64_t tiles = (dst_capacity + GATHER_TILE_TOKENS - 1) / GATHER_TILE_TOKENS;
    if (tiles * (ft.n_fields + 1) > 0x7FFFFFFFLL || tiles * GRAN_PER_TILE + GRAN_PER_TILE + 1 > ws.n_gran)
        return hipErrorInvalidValue;
    FieldTable sorted;
    const int at = order_fields(ft, tiles, &sorted, &a, mask_field);          // the mask's place; behind it:
    FieldDesc& syn = sorted.f[at + 1];
    syn.dst = reinterpret_cast<char*>(d_adv_tok_dst);
    syn.elem_bytes = 4;
    syn.src[0] = reinterpret_cast<const char*>(d_perm);
    syn.src[1] = reinterpret_cast<const char*>(d_adv_seq);
    hipLaunchKernelGGL(gather_adv_kernel, dim3((unsigned)(tiles * (a.n_carriers + 1))), dim3(GATHER_BLOCK), 0, st, a,
                       sorted, (uint32_t)at);
    return hipGetLastError();
}

hipError_t launch_gather_back(const BackSegs& bs, const FieldTable& ft, const int64_t* d_src_tok_off, const ScatterWorkspace& ws,
                              hipStream_t st) {
    const int64_t tiles = bs.tile_end[DC_MAX_SRC_SHARDS - 1];
    if (ft.n_fields == 0 || tiles == 0) return hipSuccess;
    if (tiles * ft.n_fields > 0x7FFFFFFFLL) return hipErrorInvalidValue;
    for (int s = 0; s < DC_MAX_SRC_SHARDS; ++s) {           // every segment's tables hold its tiles plus the padding
        const int64_t seg_tiles = bs.tile_end[s] - (s > 0 ? bs.tile_end[s - 1] : 0u);
        if (seg_tiles > 0 && seg_tiles * GRAN_PER_TILE + GRAN_PER_TILE + 1 > bs.gran_base[s + 1] - bs.gran_base[s])
            return hipErrorInvalidValue;
    }
    if (bs.gran_base[DC_MAX_SRC_SHARDS] > ws.n_gran_all) return hipErrorInvalidValue;
    GatherArgs a;
    a.n_seq = 0;
    a.capacity = 0;
    a.dst_tok_off = d_src_tok_off;
    a.slot_src_off = ws.r_src_off;
    a.slot_len = ws.r_len;
    a.slot_shard = nullptr;                                // (the arena is the only source)
    a.gran_first = ws.gran_first;
    a.gran_rec = ws.gran_rec;
    FieldTable sorted;
    order_fields(ft, tiles, &sorted, &a);
    hipLaunchKernelGGL(gather_back_kernel, dim3((unsigned)(tiles * a.n_carriers)), dim3(GATHER_BLOCK), 0, st, a, sorted, bs);
    return hipGetLastError();
}

}  // namespace dc

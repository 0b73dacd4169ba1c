// Generalized advantage estimation (Schulman et al. 2016, arXiv 1506.02438, eqs. 11-16) over the
// loss-bearing tokens of every sequence, in the rollout layout: the advantage stage of PPO
// (Sec. 7.1 evaluates PPO with a critic; App. B Table 2 "advantage"), the counterpart of the
// group-relative advantage.  Outputs per token: the advantage and the value target.
//
// With t_1 < ... < t_m the loss-bearing tokens of a sequence:
//   delta_k = r_k + gamma V[t_{k+1}] - V[t_k]   (V[t_{m+1}] = 0; r_k = KL penalty, plus the score on t_m)
//   A_k     = delta_k + gamma lambda A_{k+1},   ret_k = A_k + V[t_k]
// a first-order linear recurrence running backwards in time.  NW wavefronts share
// one sequence and walk it from the end; per iteration a wave takes 64 * T tokens, a lane T = 8
// or 4 consecutive ones (two aligned 16-byte groups of the value array or one; NW and T by the
// batch, see launch_gae), lane 0 of wave 0 the latest.  Inside an iteration
//   * "gamma V of the next loss-bearing token" is a copy from the nearest earlier lane (or wave)
//     that holds one, not arithmetic;
//   * each lane folds its tokens into one affine map A_after = P A_in + B, the lanes' maps are
//     composed by a 6-step DPP scan, the waves' maps through LDS, and each lane then replays its
//     tokens from the state entering it;
//   * a wave whose tokens all bear loss (the inside of a response) never looks at a mask
//     again; a wave without any loss-bearing token (a prompt) only writes zeros;
//   * the outputs leave through a transpose in LDS, so that a store instruction writes 64
//     consecutive 16-byte chunks (a lane's own 8 tokens are 32 bytes: two instructions that
//     each write every other 16 bytes, which streaming stores handle at a third of the rate; with 4
//     tokens a lane writes one chunk as it is).
// All arithmetic is float64 (the kernel is bound by HBM, not by the vector unit: 13 B per token,
// 21 with the KL penalty); outputs are rounded once to float32.
// Measured rationale: one wave per sequence left the longest sequence (36 K tokens, 141 dependent
// blocks) running alone for 160 us; with two or four waves it is still 36 or 18 dependent iterations, which
// run on alone when the sequence's workgroup starts late, so the first workgroups of the grid
// look for long sequences and start those (with all their waves, where the batch's other sequences get
// a wave each); anything derived from a loaded mask word at load time makes
// the wave wait for the loads it has just issued (the prefetch ring keeps the raw words);
// plain loads with streaming stores beat both all-plain and all-streaming accesses (every line
// of the value array is touched by two load instructions, 32 bytes apart per lane).
#include <algorithm>
#include "dc_device.h"
#include "dc_internal.h"
#include "dc_lanes.h"

namespace dc {

struct GaeArgs {
    int32_t        n_seq, use_kl;
    double         gamma, decay, kl_coef;            // decay = gamma * lambda
    int32_t        n_sets, long_len;                 // sets among which long sequences are looked for; what counts as long
    const int64_t* src_tok_off;
    const int32_t* seq_len;
    const float*   reward;
    int32_t*       status;
    const float*   value[DC_MAX_SRC_SHARDS];
    const uint8_t* mask[DC_MAX_SRC_SHARDS];
    const float*   logp[DC_MAX_SRC_SHARDS];
    const float*   ref[DC_MAX_SRC_SHARDS];
    float*         adv[DC_MAX_SRC_SHARDS];
    float*         ret[DC_MAX_SRC_SHARDS];
};

typedef float f32x4 __attribute__((ext_vector_type(4)));

// One lane's T consecutive tokens, T = 8 or 4: elements x0 .. x0 + T - 1 of the shard's buffers (x0 a multiple of T).
template <bool KL, int T>
struct GaeLane {
    float    v[T];                             // values (0 outside the sequence)
    float    lp[KL ? T : 1], rf[KL ? T : 1];   // log-probabilities, policy and reference (KL penalty only)
    uint32_t m[T / 4];                         // the mask bytes as loaded (0 outside the sequence); nothing is
                                               // derived from them before the lane's turn comes: a use here would make
                                               // the wave wait for the loads it has only just issued
    uint32_t inside;                           // bit t: token t belongs to the sequence
};

__device__ __forceinline__ uint32_t nonzero_bytes(uint32_t m) {
    return ((m & 0x000000FFu) ? 1u : 0u) | ((m & 0x0000FF00u) ? 2u : 0u) |
           ((m & 0x00FF0000u) ? 4u : 0u) | ((m & 0xFF000000u) ? 8u : 0u);
}

template <bool KL, int T>
__device__ __forceinline__ void load_lane(const float* __restrict__ V, const uint8_t* __restrict__ M,
                                          const float* __restrict__ LP, const float* __restrict__ RF,
                                          int64_t x0, bool live, int64_t so, int64_t end, GaeLane<KL, T>& g) {
    if (live && x0 >= so && x0 + T <= end) {              // all tokens inside the sequence: vector loads
        f32x4 v[T / 4], p[T / 4], r[T / 4];
#pragma unroll
        for (int h = 0; h < T / 4; ++h) v[h] = *reinterpret_cast<const f32x4*>(V + x0 + 4 * h);
#pragma unroll
        for (int h = 0; h < T / 4; ++h) g.m[h] = *reinterpret_cast<const uint32_t*>(M + x0 + 4 * h);
        if constexpr (KL) {
#pragma unroll
            for (int h = 0; h < T / 4; ++h) p[h] = *reinterpret_cast<const f32x4*>(LP + x0 + 4 * h);
#pragma unroll
            for (int h = 0; h < T / 4; ++h) r[h] = *reinterpret_cast<const f32x4*>(RF + x0 + 4 * h);
        }
        g.inside = (1u << T) - 1u;
#pragma unroll
        for (int t = 0; t < T; ++t) {
            g.v[t] = v[t >> 2][t & 3];
            if constexpr (KL) { g.lp[t] = p[t >> 2][t & 3]; g.rf[t] = r[t >> 2][t & 3]; }
        }
    } else {                                              // the sequence starts or ends inside, or lies elsewhere
        g.inside = 0;
#pragma unroll
        for (int h = 0; h < T / 4; ++h) g.m[h] = 0;
#pragma unroll
        for (int t = 0; t < T; ++t) g.v[t] = 0.0f;
#pragma unroll
        for (int t = 0; t < (KL ? T : 1); ++t) { g.lp[t] = 0.0f; g.rf[t] = 0.0f; }
        if (live) {
#pragma unroll
            for (int t = 0; t < T; ++t) {
                const int64_t x = x0 + t;
                if (x >= so && x < end) {
                    g.inside |= 1u << t;
                    g.v[t] = V[x];
                    g.m[t >> 2] |= (uint32_t)M[x] << (8 * (t & 3));
                    if constexpr (KL) { g.lp[t] = LP[x]; g.rf[t] = RF[x]; }
                }
            }
        }
    }
}

// ---- cross-lane moves of doubles through DPP (two 32-bit moves; nothing touches LDS) ----
template <int CTRL, int ROW_MASK = 0xF>
__device__ __forceinline__ double dpp_mov_f64(double old, double v) {
    const uint64_t o = (uint64_t)__double_as_longlong(old), x = (uint64_t)__double_as_longlong(v);
    const uint32_t lo = dpp_mov<CTRL, ROW_MASK>((uint32_t)o, (uint32_t)x);
    const uint32_t hi = dpp_mov<CTRL, ROW_MASK>((uint32_t)(o >> 32), (uint32_t)(x >> 32));
    return __longlong_as_double((long long)((uint64_t)lo | ((uint64_t)hi << 32)));
}
// One step of the inclusive scan of affine maps x -> P x + B in lane order: my map is applied
// after the map arriving from the lower lane; lanes that receive nothing see the identity.
template <int CTRL, int ROW_MASK = 0xF>
__device__ __forceinline__ void affine_scan_step(double& P, double& B) {
    const double Pp = dpp_mov_f64<CTRL, ROW_MASK>(1.0, P), Bp = dpp_mov_f64<CTRL, ROW_MASK>(0.0, B);
    B = P * Bp + B;
    P = P * Pp;
}
__device__ __forceinline__ double readlane_f64(double v, int src) {
    const uint64_t x = (uint64_t)__double_as_longlong(v);
    const uint32_t lo = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)x, src);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(x >> 32), src);
    return __longlong_as_double((long long)((uint64_t)lo | ((uint64_t)hi << 32)));
}

constexpr int GAE_SET = 32, GAE_MANY_SET = 64;        // sequences of a set, at most
__device__ __forceinline__ bool gae_is_long(int32_t ln, int32_t long_len) { return ln >= long_len && ln <= DC_MAX_SEQ_LEN; }
// The longest long sequence of a set whose key lies below `below` (its own key goes there), or -1; every wave that asks gets
// the same answer.  Set s of a.n_sets: sequences s, s + n_sets, s + 2 n_sets, ... (up to SET of them, neighbours in different
// sets).  Key: the length, then the lower index.
template <int SET>
__device__ __forceinline__ int gae_longest_of_set(const GaeArgs& a, int set, int lane, int32_t& below) {
    const int k = lane & (SET - 1);
    const int64_t idx = (int64_t)set + (int64_t)k * a.n_sets;
    int32_t ln = 0;
    if (idx < a.n_seq) ln = a.seq_len[idx];
    static_assert((int64_t)DC_MAX_SEQ_LEN * SET + SET <= INT32_MAX && SET <= WAVE, "the key fits 32 bits");
    int32_t key = gae_is_long(ln, a.long_len) ? ln * SET + (SET - 1 - k) : -1;
    if (key >= below) key = -1;
#pragma unroll
    for (int d = SET / 2; d >= 1; d >>= 1) key = max(key, __shfl_xor(key, d, WAVE));
    below = __builtin_amdgcn_readfirstlane(key);
    return below < 0 ? -1 : set + (SET - 1 - (below & (SET - 1))) * a.n_sets;
}

// What the NW waves of a sequence exchange through LDS (one wave: nothing):
// gamma * V of each wave's earliest loss-bearing token (a later wave's first loss-bearing token
// needs it), and each wave's composed map, from which every wave derives the state entering its
// tokens and the state carried to the next iteration.  Two barriers per iteration; every wave
// of a sequence runs the same number of iterations (a wave whose lanes all lie before the
// sequence's start just takes part in the barriers).
template <int NW>
struct GaeLds {
    double  u[NW], P[NW], B[NW];
    int32_t has[NW];
};
// A wave's outputs on their way out (8 tokens to a lane).
template <int T>
struct alignas(16) GaeStage { float x[T == 8 ? 2 * WAVE * T : 4]; };

// What a sequence is, asked for at once: one trip to memory.
struct GaeSeq {
    int32_t ln;
    int64_t so, next;
    float   score;
};
__device__ __forceinline__ GaeSeq gae_fetch(const GaeArgs& a, int i) {
    GaeSeq q;
    q.ln = a.seq_len[i];
    q.so = a.src_tok_off[i];
    q.next = a.src_tok_off[min(i + 1, a.n_seq - 1)];
    q.score = a.reward[i];
    return q;
}

// Sequence i by NW waves, the workgroup's only ones if there is more than one, of which this is number w (uniform): T tokens
// to a lane, the loads of AHEAD iterations in flight ahead of the one worked on.  An iteration covers NW * 64 * T tokens,
// wave 0 the latest 64 * T of them, lane 0 of a wave its latest T.
template <int NW, bool KL, int T, int AHEAD>
__device__ __forceinline__ void gae_sequence(const GaeArgs& a, const SourceDesc& sd, GaeLds<NW>* x, GaeStage<T>& stage, int i,
                                             const GaeSeq& me, int w, int lane) {
    constexpr int UNR = NW > 4 ? 1 : NW;                           // (unrolled over 8 waves it would cost 25 registers)
    const int32_t ln = me.ln;
    const int64_t so = me.so, next = me.next;
    const float score = me.score;
    int s = 0;                                                     // (seq_off[k] = N from k = n_src on)
#pragma unroll
    for (int k = 1; k < DC_MAX_SRC_SHARDS; ++k) s += i >= sd.seq_off[k] ? 1 : 0;
    if (ln <= 0 || ln > DC_MAX_SEQ_LEN) {                          // uniform over the waves
        if (w == 0 && lane == 0) set_status(a.status, DC_ERR_ZERO_LENGTH_SEQ);
        return;
    }
    if (so < 0 || so + ln > sd.tokens[s] || (i + 1 < sd.seq_off[s + 1] && next < so + ln)) {
        if (w == 0 && lane == 0) set_status(a.status, DC_ERR_BAD_LAYOUT);   // outside its buffer or overlapping the next
        return;
    }
    const float* __restrict__ V = a.value[s];
    const uint8_t* __restrict__ M = a.mask[s];
    const float* __restrict__ LP = a.logp[s];
    const float* __restrict__ RF = a.ref[s];
    float* __restrict__ ADV = a.adv[s];
    float* __restrict__ RET = a.ret[s];
    const int64_t end = so + ln;
    constexpr int LG_T = T == 8 ? 3 : 2;
    static_assert(T == 1 << LG_T, "8 or 4 tokens to a lane");
    const int64_t q_lo = so >> LG_T, q_hi = (end - 1) >> LG_T;    // aligned T-token lane groups the sequence touches
    const double gamma = a.gamma, decay = a.decay, klc = a.kl_coef;
    constexpr int STEP = NW * WAVE;                                // lane groups per iteration
    double decay_pow_T = 1.0;                                      // decay^T: a lane's multiplier when all its tokens bear loss
#pragma unroll
    for (int t = 0; t < T; ++t) decay_pow_T *= decay;

    // carried from iteration to iteration (uniform): A of the next loss-bearing token, and gamma * its
    // value, which starts out as the sequence's score (so the score lands on the last such token)
    double A_carry = 0.0, U_carry = (double)score;

    GaeLane<KL, T> ring[AHEAD > 0 ? AHEAD : 1];
#pragma unroll
    for (int k = 0; k < AHEAD; ++k) {
        const int64_t q = q_hi - (int64_t)k * STEP - w * WAVE - lane;
        load_lane<KL, T>(V, M, LP, RF, q * T, q >= q_lo, so, end, ring[k]);
    }
    for (int64_t top = q_hi; top >= q_lo; top -= STEP) {
        const int64_t q = top - w * WAVE - lane;                   // my lane group; lane 0 of wave 0 holds the latest one
        GaeLane<KL, T> cur;
        if constexpr (AHEAD > 0) {
            cur = ring[0];
#pragma unroll
            for (int k = 0; k + 1 < AHEAD; ++k) ring[k] = ring[k + 1];
            const int64_t qn = q - (int64_t)AHEAD * STEP;
            load_lane<KL, T>(V, M, LP, RF, qn * T, qn >= q_lo, so, end, ring[AHEAD - 1]);
        } else {
            load_lane<KL, T>(V, M, LP, RF, q * T, q >= q_lo, so, end, cur);
        }
        uint32_t loss = nonzero_bytes(cur.m[0]);                   // bit t: token t bears loss
        if constexpr (T == 8) loss |= nonzero_bytes(cur.m[1]) << 4;
        const uint64_t holders = __ballot(loss != 0);              // lanes of my wave with a loss-bearing token
        const bool any = holders != 0ull;                          // uniform over the wave
        // uniform: every lane that holds tokens of the sequence at all holds T loss-bearing ones (the
        // inside of a response); then no mask is looked at again
        const bool solid = any && __ballot(loss != (1u << T) - 1u && cur.inside != 0u) == 0ull;

        // ---- gamma * V of my earliest loss-bearing token; the wave's earliest goes to the other waves ----
        double U_last;
        if (solid) {
            U_last = gamma * (double)cur.v[0];
        } else {
            float first = cur.v[T - 1];
#pragma unroll
            for (int t = T - 2; t >= 0; --t)
                if (loss & (1u << t)) first = cur.v[t];
            U_last = gamma * (double)first;
        }
        const double U_wave = readlane_f64(U_last, any ? 63 - __builtin_clzll(holders) : 0);
        double U_w = U_carry, U_next = U_carry;                    // entering my wave / carried to the next iteration
        if constexpr (NW == 1) {
            if (any) U_next = U_wave;
        } else {
            if (lane == 0) { x->has[w] = any ? 1 : 0; x->u[w] = U_wave; }
            lds_barrier();
#pragma unroll UNR
            for (int k = 0; k < NW; ++k) {
                const bool h = x->has[k] != 0;
                const double u = x->u[k];
                if (h && k < w) U_w = u;
                if (h) U_next = u;
            }
        }

        // ---- my tokens, latest first: r[t] = what token t adds to decay * A (its TD residual), and the lane's map
        // A_after = P * A_in + B; then the inclusive scan of the lanes' maps (rows of 16 lanes, then across rows) ----
        double r[T], Pi = 1.0, Bi = 0.0;
        if (solid) {
            double u = dpp_mov_f64<DPP_WAVE_SHR1>(U_w, U_last);    // gamma * V[0] of the lane before mine; lane 0: U_w
            double B = 0.0;
#pragma unroll
            for (int t = T - 1; t >= 0; --t) {
                const double vt = (double)cur.v[t];
                r[t] = u - vt;
                if constexpr (KL) r[t] = __builtin_fma(-klc, (double)cur.lp[t] - (double)cur.rf[t], r[t]);
                B = __builtin_fma(decay, B, r[t]);
                u = gamma * vt;
            }
            Pi = decay_pow_T; Bi = B;
        } else if (any) {
            const uint64_t before = holders & ((1ull << lane) - 1ull);        // lanes with later tokens than mine
            const int from = before ? 63 - __builtin_clzll(before) : 0;
            const double U_from = __shfl(U_last, from, WAVE);
            double u = before ? U_from : U_w, P = 1.0, B = 0.0;
#pragma unroll
            for (int t = T - 1; t >= 0; --t) {
                const double vt = (double)cur.v[t];
                r[t] = u - vt;
                if constexpr (KL) r[t] = __builtin_fma(-klc, (double)cur.lp[t] - (double)cur.rf[t], r[t]);
                if (loss & (1u << t)) {
                    B = __builtin_fma(decay, B, r[t]);
                    P = decay * P;
                    u = gamma * vt;
                }
            }
            Pi = P; Bi = B;
        }
        if (any) {
            affine_scan_step<DPP_ROW_SHR1>(Pi, Bi);
            affine_scan_step<DPP_ROW_SHR2>(Pi, Bi);
            affine_scan_step<DPP_ROW_SHR4>(Pi, Bi);
            affine_scan_step<DPP_ROW_SHR8>(Pi, Bi);
            affine_scan_step<DPP_ROW_BCAST15, 0xA>(Pi, Bi);
            affine_scan_step<DPP_ROW_BCAST31, 0xC>(Pi, Bi);
        }
        double A_w = A_carry, A_next = A_carry;                    // entering my wave / carried to the next iteration
        if constexpr (NW == 1) {
            A_next = __builtin_fma(readlane_f64(Pi, WAVE - 1), A_next, readlane_f64(Bi, WAVE - 1));
        } else {
            if (lane == WAVE - 1) { x->P[w] = Pi; x->B[w] = Bi; }   // the wave's whole map (identity without loss)
            lds_barrier();
#pragma unroll UNR
            for (int k = 0; k < NW; ++k) {
                const double Pk = x->P[k], Bk = x->B[k];
                if (k == w) A_w = A_next;
                A_next = __builtin_fma(Pk, A_next, Bk);
            }
        }

        // ---- outputs: replay my tokens from the state entering my lane ----
        float oa[T], orr[T];
#pragma unroll
        for (int t = 0; t < T; ++t) { oa[t] = 0.0f; orr[t] = 0.0f; }
        if (any) {
            // the maps of all lanes before mine (identity for lane 0), applied to the state entering the wave
            const double Pe = dpp_mov_f64<DPP_WAVE_SHR1>(1.0, Pi), Be = dpp_mov_f64<DPP_WAVE_SHR1>(0.0, Bi);
            double A = __builtin_fma(Pe, A_w, Be);
            if (solid) {
#pragma unroll
                for (int t = T - 1; t >= 0; --t) {
                    A = __builtin_fma(decay, A, r[t]);
                    oa[t] = (float)A;
                    orr[t] = (float)(A + (double)cur.v[t]);
                }
            } else {
#pragma unroll
                for (int t = T - 1; t >= 0; --t)
                    if (loss & (1u << t)) {
                        A = __builtin_fma(decay, A, r[t]);
                        oa[t] = (float)A;
                        orr[t] = (float)(A + (double)cur.v[t]);
                    }
            }
        }
        // ---- stores, through a transpose in LDS: a lane's 8 tokens are 32 bytes, and 16 bytes per lane at a
        // 32-byte stride, the other halves in a second instruction, is a pattern that streaming stores write at
        // a third of the rate of 64 consecutive 16-byte chunks (2.3 against 6.3 TB/s, write-only probe).
        // Memory order runs against lane order; the wave's window starts at lane 63's first token.
        if (__ballot(cur.inside != 0u) != 0ull) {                  // uniform: some token of the window lies inside
            auto store4 = [&](int64_t t0, f32x4 va, f32x4 vr) {
                if (t0 >= so && t0 + 4 <= end) {
                    __builtin_nontemporal_store(va, reinterpret_cast<f32x4*>(ADV + t0));
                    __builtin_nontemporal_store(vr, reinterpret_cast<f32x4*>(RET + t0));
                } else {
#pragma unroll
                    for (int e = 0; e < 4; ++e)
                        if (t0 + e >= so && t0 + e < end) { ADV[t0 + e] = va[e]; RET[t0 + e] = vr[e]; }
                }
            };
            if constexpr (T == 4) {
                f32x4 va, vr;
                va.x = oa[0]; va.y = oa[1]; va.z = oa[2]; va.w = oa[3];
                vr.x = orr[0]; vr.y = orr[1]; vr.z = orr[2]; vr.w = orr[3];
                store4(q * T, va, vr);
            } else {
                float* st_a = stage.x;
                float* st_r = st_a + WAVE * T;
                const int mine = (WAVE - 1 - lane) * T;
                f32x4 o;
                o.x = oa[0]; o.y = oa[1]; o.z = oa[2]; o.w = oa[3];
                *reinterpret_cast<f32x4*>(st_a + mine) = o;
                o.x = oa[T - 4]; o.y = oa[T - 3]; o.z = oa[T - 2]; o.w = oa[T - 1];
                *reinterpret_cast<f32x4*>(st_a + mine + 4) = o;
                o.x = orr[0]; o.y = orr[1]; o.z = orr[2]; o.w = orr[3];
                *reinterpret_cast<f32x4*>(st_r + mine) = o;
                o.x = orr[T - 4]; o.y = orr[T - 3]; o.z = orr[T - 2]; o.w = orr[T - 1];
                *reinterpret_cast<f32x4*>(st_r + mine + 4) = o;
                const int64_t base = (top - (int64_t)w * WAVE - (WAVE - 1)) * T;
#pragma unroll
                for (int u = 0; u < 2; ++u) {
                    const int c = (u * WAVE + lane) * 4;           // my chunk of 4 tokens in this instruction
                    store4(base + c, *reinterpret_cast<const f32x4*>(st_a + c), *reinterpret_cast<const f32x4*>(st_r + c));
                }
            }
        }
        A_carry = A_next;
        U_carry = U_next;
    }
}

// One workgroup of NW waves per sequence, in index order, behind n_sets workgroups that each start the longest sequence of
// a set if it is a long one: a 36 K-token sequence is 36 dependent iterations, and started late it runs on alone after
// the rest.
template <int NW, bool KL, int T, int AHEAD>
__global__ __launch_bounds__(NW * WAVE) void gae_kernel(GaeArgs a, SourceDesc sd) {
    __shared__ GaeLds<NW> x;
    __shared__ GaeStage<T> stage[NW];
    const int lane = threadIdx.x & (WAVE - 1);
    const int w = __builtin_amdgcn_readfirstlane((int)(threadIdx.x / WAVE));
    int i = (int)blockIdx.x - a.n_sets;
    const bool early = i < 0;
    GaeSeq me = {0, 0, 0, 0.0f};
    if (!early) me = gae_fetch(a, i);
    if (early || gae_is_long(me.ln, a.long_len)) {                 // uniform over the workgroup
        int32_t below = INT32_MAX;
        const int longest = gae_longest_of_set<GAE_SET>(a, early ? (int)blockIdx.x : i % a.n_sets, lane, below);
        if (early ? longest < 0 : longest == i) return;            // nothing to start early / started early
        if (early) {
            i = longest;
            me = gae_fetch(a, i);
        }
    }
    gae_sequence<NW, KL, T, AHEAD>(a, sd, &x, stage[w], i, me, w, lane);
}

// One WAVE per sequence, W of them to a workgroup, behind GAE_SHARE * n_sets workgroups that take the long sequences with all
// W waves (alone a wave would be at a 32 K-token sequence for 128 iterations, each waiting for its loads): the r-th
// workgroup of a set takes its r-th longest, (r + GAE_SHARE)-th, ...  The sets' first workgroups come first.
constexpr int GAE_SHARE = 4;
template <int W, bool KL, int T, int AHEAD>
__global__ __launch_bounds__(W * WAVE, T == 4 ? 8 : 4) void gae_many_kernel(GaeArgs a, SourceDesc sd) {
    __shared__ GaeLds<W> x;
    __shared__ GaeStage<T> stage[W];
    const int lane = threadIdx.x & (WAVE - 1);
    const int w = __builtin_amdgcn_readfirstlane((int)(threadIdx.x / WAVE));
    const int n_early = a.n_sets * GAE_SHARE;
    if ((int)blockIdx.x < n_early) {                               // (uniform)
        const int r = (int)blockIdx.x / a.n_sets, set = (int)blockIdx.x - r * a.n_sets;
        int32_t below = INT32_MAX;
        for (int skip = r;; skip = GAE_SHARE - 1) {
            int i = gae_longest_of_set<GAE_MANY_SET>(a, set, lane, below);
            for (int q = 0; q < skip && i >= 0; ++q) i = gae_longest_of_set<GAE_MANY_SET>(a, set, lane, below);
            if (i < 0) return;
            gae_sequence<W, KL, T, AHEAD>(a, sd, &x, stage[w], i, gae_fetch(a, i), w, lane);
        }
    }
    const int i = ((int)blockIdx.x - n_early) * W + w;
    if (i >= a.n_seq) return;
    const GaeSeq me = gae_fetch(a, i);
    if (gae_is_long(me.ln, a.long_len)) return;                    // its set's workgroups do it
    gae_sequence<1, KL, T, 0>(a, sd, nullptr, stage[w], i, me, 0, lane);
}

hipError_t launch_gae(int32_t n_seq, const SourceDesc& src, const int64_t* d_src_tok_off, const int32_t* d_seq_len,
                      const float* d_reward, const float* const* value_base, const uint8_t* const* mask_base,
                      const float* const* logp_base, const float* const* ref_base, double gamma, double lambda,
                      double kl_coef, float* const* adv_base, float* const* ret_base, int32_t* d_status,
                      hipStream_t st) {
    if (n_seq == 0) return hipSuccess;
    GaeArgs a;
    a.n_seq = n_seq; a.use_kl = kl_coef != 0.0 ? 1 : 0;
    a.gamma = gamma; a.decay = gamma * lambda; a.kl_coef = kl_coef;
    a.src_tok_off = d_src_tok_off; a.seq_len = d_seq_len; a.reward = d_reward; a.status = d_status;
    int64_t tokens = 0;
    for (int s = 0; s < src.n_src; ++s) tokens += src.tokens[s];
    const int64_t mean = tokens / n_seq;                           // (the buffers' sizes bound the lengths' sum)
    for (int s = 0; s < DC_MAX_SRC_SHARDS; ++s) {
        const bool on = s < src.n_src;
        a.value[s] = on ? value_base[s] : nullptr;
        a.mask[s] = on ? mask_base[s] : nullptr;
        a.logp[s] = on && a.use_kl ? logp_base[s] : nullptr;
        a.ref[s] = on && a.use_kl ? ref_base[s] : nullptr;
        a.adv[s] = on ? adv_base[s] : nullptr;
        a.ret[s] = on ? ret_base[s] : nullptr;
    }
    using std::integral_constant;
    // (many: gae_many_kernel with that many waves to a workgroup)
    auto launch = [&](auto kl, auto many, auto nw, auto t, auto ahead) {
        constexpr bool KL = decltype(kl)::value, MANY = decltype(many)::value;
        constexpr int NW = decltype(nw)::value, T = decltype(t)::value, AHEAD = decltype(ahead)::value;
        // long: at least twice the mean and 4 iterations; where a wave has a sequence to itself, four times and 8 iterations
        const int64_t long_len = MANY ? std::max<int64_t>(4 * mean, 8 * WAVE * T) : std::max<int64_t>(2 * mean, 4 * NW * WAVE * T);
        a.long_len = (int32_t)std::min<int64_t>(long_len, INT32_MAX);
        if constexpr (MANY) {
            a.n_sets = (n_seq + GAE_MANY_SET - 1) / GAE_MANY_SET;
            // (a long sequence in every prompt's group, at the same place in each, must not fall into a few of the sets: 16 384 of
            // 300 tokens and every 64th of 8192 take 21 us so, 377 with 256 sets)
            auto odd = [](int32_t x) { return x % 2 && x % 3 && x % 5 && x % 7 && x % 11 && x % 13; };
            while (!odd(a.n_sets)) ++a.n_sets;
            const dim3 grid((unsigned)(GAE_SHARE * a.n_sets + (n_seq + NW - 1) / NW)), block(NW * WAVE);
            hipLaunchKernelGGL((gae_many_kernel<NW, KL, T, AHEAD>), grid, block, 0, st, a, src);
        } else {
            a.n_sets = (n_seq + GAE_SET - 1) / GAE_SET;
            const dim3 grid((unsigned)(n_seq + a.n_sets)), block(NW * WAVE);
            hipLaunchKernelGGL((gae_kernel<NW, KL, T, AHEAD>), grid, block, 0, st, a, src);
        }
    };
    // Waves per sequence and tokens per lane, by what the chip holds at once and how long a sequence is (us with two waves of
    // 8 tokens and two iterations ahead for every batch, and so; "+ 1": with one of 32 K tokens among them; KL: with the
    // penalty, whose loads and registers make a wave of its own per sequence pay up to a smaller mean):
    //   up to 1024 sequences, and up to 4096 long ones: four waves of 8, one ahead: the longest sequence's iterations are the
    //   time (1000 of 1499 18.6 -> 13.3, + 1 54 -> 32; 3000 of 2599 KL 39.0 -> 36.4, + 1 61 -> 42);
    //   up to 2048: two waves of 8, two ahead, or four of 4 above 1024 tokens (2000 of 1499 18.7 -> 16.7);
    //   more: a wave that holds few tokens for its registers and its trips to memory is the time.
    //     Short sequences, one wave of 4 each, eight to a workgroup (4096 of 299 14.1 -> 12.2, + 1 54 -> 41; 16 384 of 299
    //     39.7 -> 23.9, + 1 55 -> 44; of 699 52.8 -> 38.7; KL 67.7 -> 50.5; 32 768 of 849 102 -> 78).  Where the lines lie, in
    //     us against four waves of 4: 4096 of 299 11.5 / 13.3, of 499 13.1 / 14.2, of 699 17.5 / 16.1; 8192 of 699 25.0 / 27.4,
    //     of 999 33.2 / 31.4; 16 384 of 849 44 / 50, KL of 599 44.6 / 48.4, of 849 60.3 / 56.0.
    //     Then four waves of 4 (8192 of 1249 39.3 -> 36.3; 16 384 of 1249 KL 95 -> 79, + 1 95 -> 79; of 2599 103 -> 100, of
    //     2620 under a heavy tail, up to 32 K tokens, 82 -> 76; of 3499 155 -> 152); from 2048 tokens on with KL one ahead
    //     (16 384 of 2599 188 -> 184, of 3499 245 / 241 without and with it).  Two waves of 8 without a ring are up to 5 %
    //     faster where no length stands out (16 384 of 1599 66 / 70), but a heavy tail waits for them: of 2620 83 / 76, 9216 of
    //     2300 61 / 50.
    constexpr integral_constant<int, 0> c0; constexpr integral_constant<int, 1> c1; constexpr integral_constant<int, 2> c2;
    constexpr integral_constant<int, 4> c4; constexpr integral_constant<int, 8> c8;
    constexpr std::true_type many; constexpr std::false_type one;
    auto pick = [&](auto kl) {
        constexpr bool KL = decltype(kl)::value;
        if (n_seq <= 1024 || (n_seq <= 4096 && mean > 2048)) launch(kl, one, c4, c8, c1);
        else if (n_seq <= 2048 && mean <= 1024) launch(kl, one, c2, c8, c2);
        else if (n_seq <= 2048) launch(kl, one, c4, c4, c0);
        else if (mean <= (n_seq <= 4096 ? 384 : KL ? 704 : n_seq <= 8192 ? 768 : 960)) launch(kl, many, c8, c4, c0);
        else if (!KL || mean <= 2048) launch(kl, one, c4, c4, c0);
        else if constexpr (KL) launch(kl, one, c4, c4, c1);
    };
    if (a.use_kl) pick(std::true_type{});
    else pick(std::false_type{});
    return hipGetLastError();
}

}  // namespace dc

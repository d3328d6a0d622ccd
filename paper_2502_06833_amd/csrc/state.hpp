// Device-resident decoding state shared by the per-pass kernels and the fused decode kernel.
#pragma once
#include "common.hpp"
#include "entropy.hpp"

namespace ead {

// Per-sequence decoding state, all device arrays indexed by sequence.
struct SeqState {
    int *tokens;            // [max_batch][max_seq] prompt + generated
    int *len;               // tokens present
    int *kvlen;             // [2][max_batch] positions each model has consumed
    int *model, *c, *ngen, *done, *last_step;
    int *goal;              // tokens a sequence may have generated before it pauses (<= the run's bound)
    float *ring;            // [max_batch][w_cap]
    int *out_tok; uint8_t *out_mid; float *out_H; float *out_Hbar; uint8_t *out_dec;   // [max_batch][cap]
    int *forced_tok; uint8_t *forced_mid;                                              // replay, [max_batch][cap]
    int *err;
    int max_batch, max_seq, cap;
};

struct Plan { int *hdr; int *row_seq, *row_pos, *lm_row, *lm_seq; int2 *groups; };      // groups: see PlanArgs::group_rows

struct FinArgs {
    SeqState s; Plan p; GateCfg cfg;
    const EntPartial *partials; int n_part; int unit;
    int score_mode; float *sc_H; int *sc_arg;      // score: indexed by position
    int model_id, max_new, eos_id, replay, n_new, force_model, step;
    int sampling;            // 1: the token is the sampled one (st.gidx), else the arg max
    int *host_model, *host_done;   // pinned host memory, [max_batch]: next model and done flag of the sequences this pass finalizes
};

// What lm_record needs of sequence b's state: tokens it has generated, its dwell counter, tokens present.
struct FinSeq { int n, c, len; };

// Algorithm 1's bookkeeping for sequence b once its entropy and window mean are known and the switch rule
// has been taken (next, c): record the token, its model and entropy, append the token.  Called by one thread.
__device__ __forceinline__ void lm_record(const FinArgs &a, int b, const FinSeq &q, const EntStat &st, float H, float hb, int next, int c) {
    const int n = q.n, cur = a.model_id;
    const size_t o = (size_t)b * a.s.cap + n;
    const int choice = a.sampling ? st.gidx : st.idx;
    a.s.out_tok[o] = choice; a.s.out_mid[o] = (uint8_t)cur; a.s.out_H[o] = H; a.s.out_Hbar[o] = hb;
    a.s.out_dec[o] = (uint8_t)next;
    int tok = choice;
    if (a.replay) {
        tok = a.s.forced_tok[o];
        const int nxt = (n + 1 < a.n_new) ? a.s.forced_mid[o + 1] : cur;
        if (nxt != cur) c = 0;
        next = nxt;
    }
    if (a.force_model >= 0) next = a.force_model;
    a.s.tokens[(size_t)b * a.s.max_seq + q.len] = tok;
    a.s.len[b] = q.len + 1; a.s.ngen[b] = n + 1;
    const int done = (n + 1 >= a.max_new) || (a.eos_id >= 0 && tok == a.eos_id);
    a.s.done[b] = done;
    a.s.model[b] = next; a.s.c[b] = c; a.s.last_step[b] = a.step;
    // what the host's mirror needs after the pass, written where it can read it without a copy
    if (a.host_model) { a.host_model[b] = next; a.host_done[b] = done; }
    if (!isfinite(H)) atomicOr(a.s.err, 1);
}

// The same from the state in memory: push the window, apply the switch rule, record (persistent kernels).
__device__ __forceinline__ void lm_finalize_seq(const FinArgs &a, int b, const EntStat &st, float H) {
    const FinSeq q{a.s.ngen[b], a.s.c[b], a.s.len[b]};
    int next = a.model_id, c = q.c;
    const float hb = gate_update(a.s.ring + (size_t)b * a.cfg.w, q.n, H, a.cfg, &next, &c);
    lm_record(a, b, q, st, H, hb, next, c);
}

// One workgroup per sequence that gets logits this pass: finish entropy and arg max from the LM-head
// partials, then the bookkeeping above.  A chain of latencies and nothing else (24 KB a row are read), so
// every load of a stage is requested at once -- the partials (kFinVecs per thread) with the row's state, the
// window next, by one thread per entry -- and the partials are moved to their common maximum once and added,
// instead of merged pair by pair.  (A single wave that merged 1024 partials in a loop and read the window one
// entry after the other took 11-14 us.)
constexpr int kFinThreads = 256, kFinVecs = 4;

__global__ __launch_bounds__(kFinThreads) void k_lm_finalize(FinArgs a) {
    constexpr int NW = kFinThreads / 64;
    __shared__ float s_m[NW], s_gs[NW], s_Z[NW], s_S[NW];
    __shared__ int s_idx[NW], s_gidx[NW];
    __shared__ float s_win[kFinThreads];
    const int i = blockIdx.x, tid = threadIdx.x, wave = tid >> 6;
    const int count = a.p.hdr[1], b = a.p.lm_seq[i];
    const int nw = min(NW, (a.n_part + 63) >> 6);        // waves that hold partials
    const EntPartial *pp = a.partials + (size_t)i * a.n_part;
    EntPartial e[kFinVecs];
#pragma unroll
    for (int v = 0; v < kFinVecs; ++v) {
        const int j = tid + v * kFinThreads;
        e[v] = pp[min(j, a.n_part - 1)];
        if (j >= a.n_part) e[v].Z = 0.f;
    }
    if (i >= count) return;
    // the row's state and the entries of its window that are already there (oldest first), while the partials arrive
    const FinSeq q{a.s.ngen[b], a.s.c[b], a.s.len[b]};
    const int w = a.cfg.w, cnt = min(q.n + 1, w);
    float *ring = a.s.ring + (size_t)b * w;
    if (!a.score_mode && tid < cnt - 1) s_win[tid] = ring[(q.n + 1 - cnt + tid) % w];
    if (wave < nw) {
        // this wave's partials at their common maximum (empty ones count for nothing)
        float m = -INFINITY, gs = -INFINITY;
#pragma unroll
        for (int v = 0; v < kFinVecs; ++v)
            if (e[v].Z != 0.f) { m = fmaxf(m, e[v].m); gs = fmaxf(gs, e[v].gs); }
        m = wave_max(m);
        if (a.sampling) gs = wave_max(gs);
        float Z = 0.f, S = 0.f;
        int idx = kNoIndex, gidx = kNoIndex;
#pragma unroll
        for (int v = 0; v < kFinVecs; ++v)
            if (e[v].Z != 0.f) {
                const float d = e[v].m - m, x = __expf(d);
                Z += x * e[v].Z; S += x * (e[v].S + d * e[v].Z);
                if (rank_of(e[v].m) == m) idx = min(idx, e[v].idx);      // m is the largest rank: fmaxf drops NaN
                if (e[v].gs == gs) gidx = min(gidx, e[v].gidx);
            }
        Z = wave_sum(Z); S = wave_sum(S);
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) idx = min(idx, __shfl_xor(idx, o, kWave));
        if (a.sampling) {
#pragma unroll
            for (int o = 32; o > 0; o >>= 1) gidx = min(gidx, __shfl_xor(gidx, o, kWave));
        }
        if ((tid & 63) == 0) { s_m[wave] = m; s_Z[wave] = Z; s_S[wave] = S; s_idx[wave] = idx; s_gs[wave] = gs; s_gidx[wave] = gidx; }
    }
    __syncthreads();
    if (tid != 0) return;
    EntStat st; st.init();
    for (int v = 0; v < nw; ++v) {
        EntStat t; t.m = s_m[v]; t.Z = s_Z[v]; t.S = s_S[v]; t.idx = s_idx[v]; t.gs = s_gs[v]; t.gidx = s_gidx[v];
        st.merge(t);
    }
    if (st.gidx == kNoIndex) st.gidx = st.idx;           // no perturbed score above -inf (NaN, or an overflow of l / T): the arg max
    const float H = entropy_from(st, a.unit);
    if (a.score_mode) {
        const int pos = a.p.row_pos[a.p.lm_row[i]];
        a.sc_H[pos] = H; a.sc_arg[pos] = st.idx;
        return;
    }
    // window mean: oldest to newest in fp32, as gate_update sums it
    float sum = 0.f;
    for (int j = 0; j < cnt - 1; ++j) sum = sum + (j < kFinThreads ? s_win[j] : ring[(q.n + 1 - cnt + j) % w]);
    sum = sum + H;
    ring[q.n % w] = H;
    const float hb = sum / (float)cnt;
    int next = a.model_id, c = q.c;
    gate_switch(hb, a.cfg, &next, &c);
    lm_record(a, b, q, st, H, hb, next, c);
}

}  // namespace ead

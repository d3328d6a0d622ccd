// Kernels of the library compiled for the CPU (tests/host_hip stands in for the HIP headers), with a C interface for
// tests/test_host_kernels.py: what they do with inputs that must not reach a GPU before they are known to be handled.
#include <hip/hip_runtime.h>
#undef HOST_SHARED
#define HOST_SHARED
#include "linear.hpp"
#undef HOST_SHARED
#define HOST_SHARED static
#include "rules.hpp"
#include "state.hpp"
#include "stream_list.hpp"
#include "turn.hpp"
#include <atomic>
#include <chrono>

using namespace ead;

extern "C" {

// k_lm_finalize over `rows` sequences of n_part partials each: the token appended, its entropy, and the error flag.
void host_finalize(const EntPartial *partials, int rows, int n_part, int sampling, int *tok, float *H, int *err) {
    std::vector<int> zero(rows, 0), len(rows, 0), seq(rows), out[5];
    for (auto &v : out) v.assign(rows, 0);
    std::vector<float> ring(rows * 5, 0.f), hb(rows);
    std::vector<uint8_t> mid(rows), dec(rows);
    for (int r = 0; r < rows; ++r) seq[r] = r;
    int hdr[4] = {rows, rows, 0, 0};
    FinArgs a{};
    a.s.tokens = tok; a.s.len = len.data(); a.s.model = out[0].data(); a.s.c = out[1].data(); a.s.ngen = zero.data();
    a.s.done = out[2].data(); a.s.last_step = out[3].data(); a.s.ring = ring.data(); a.s.out_tok = out[4].data(); a.s.out_mid = mid.data();
    a.s.out_H = H; a.s.out_Hbar = hb.data(); a.s.out_dec = dec.data(); a.s.err = err; a.s.max_batch = rows; a.s.max_seq = 1; a.s.cap = 1;
    a.p.hdr = hdr; a.p.lm_seq = seq.data();
    a.cfg = GateCfg{5, 0.f, 1};
    a.partials = partials; a.n_part = n_part; a.max_new = 2; a.eos_id = -1; a.force_model = -1; a.sampling = sampling;
    *err = 0;
    host_launch((unsigned)rows, kFinThreads, [=] { k_lm_finalize(a); });
}

// lm_fold over `groups` groups of 8 row blocks, as the lane that holds rows 0..3 of every block; inv_t 0: greedy.
void host_fold(const float *logits /* [groups][8][4] */, int groups, int last_have, float inv_t, EntPartial *out) {
    LinArgs<bf16_t> a{};
    a.samp_inv_t = inv_t;
    EntStat st; st.init();
    for (int g = 0; g < groups; ++g) {
        f32x4_t acc[kLmRows];
        for (int j = 0; j < kLmRows; ++j) for (int e = 0; e < 4; ++e) acc[j][e] = logits[(g * kLmRows + j) * 4 + e];
        lm_fold(a, acc, g * kLmRows * 16, g + 1 == groups ? last_have : kLmRows, 0, true, 0, 0, st);
    }
    out->m = st.m; out->Z = st.Z; out->S = st.S; out->idx = st.idx; out->gs = st.gs; out->gidx = st.gidx;
}

// 1 if ead_entropy_argmax takes one launch for [rows, V] logits of `size` bytes each
int host_entropy_folds(int rows, int V, int size) {
    int chunks, per;
    entropy_split(rows, V, &chunks, &per);
    return entropy_folds(rows, chunks, (size_t)rows * V * size);
}

int host_entropy_row_parts(int rows, int V) { return entropy_row_parts(rows, V); }

int host_attention_chunk(int T, int KV, int hd, int ctx, int mfma, long items) { return attention_chunk(T, KV, hd, ctx, mfma != 0, 256, 16, items); }

int host_prompt_attention(int T, int seqs, long groups, int KV, int ctx) { return prompt_attention(T, seqs, groups, 1, KV, 128, ctx, 256, false); }

int host_score_prompt_attention(int T, long groups, int KV, int ctx) { return prompt_attention(T, 1, groups, 1, KV, 128, ctx, 256, true); }

// `rows` rows each of `seqs` sequences behind `have` keys, G query heads per KV head, 256 compute units
int host_prompt_attention_rows(int seqs, int rows, int have, int G, int KV, int hd) {
    const int rq = 16 / G, gr = 4 * rq, last = have + rows - 1;
    return prompt_attention(seqs * rows, seqs, (long)seqs * (last / rq - have / rq + 1), (long)seqs * (last / gr - have / gr + 1), KV, hd, last + 1, 256, false);
}

// NB row blocks x K, one row, 256 compute units
int host_ring_takes_matrix(int K, int NB, int epi) { return ring_takes(K, NB, 256, (Epilogue)epi); }
int host_ring_takes(int K, int residual, int lm) { return host_ring_takes_matrix(K, 128, residual ? EPI_RES : lm ? EPI_LOGITS : EPI_QKV); }

// the first `terms` bf16 terms of eight floats, added up
void host_bf16_terms(const float *in, int terms, double *sum) {
    float f[8];
    for (int e = 0; e < 8; ++e) { f[e] = in[e]; sum[e] = 0.0; }
    for (int i = 0; i < terms; ++i) {
        const u32x4_t w = __builtin_bit_cast(u32x4_t, take_bf16(f));
        for (int e = 0; e < 8; ++e) sum[e] += __uint_as_float((e & 1 ? w[e / 2] >> 16 : w[e / 2] & 0xFFFFu) << 16);
    }
}

// row blocks, token blocks and slabs of K a workgroup of k_linear_mfma takes, as R * 100 + NT * 10 + KS; 0 if scratch does not hold the slabs
int host_narrow_plan(int NB, int KC, int TB, int split, long floats, int groups) {
    const NarrowPlan p = narrow_plan(NB, KC, TB, 256, split != 0, (size_t)floats, groups);
    const long g = (long)((NB + p.R - 1) / p.R) * ((TB + p.NT - 1) / p.NT);
    if (p.KS > 1 && ((long)p.KS * g * p.R * p.NT * 256 > floats || g > groups || p.KS > KC)) return 0;
    return p.R * 100 + p.NT * 10 + p.KS;
}

int host_gate_up_by_one(int NB) { return gate_up_by_one(NB, 256); }
int host_gate_up_streamed(int NB, int KC, int TB) { return gate_up_streamed(NB, KC, TB, 256); }
int host_lm_by_rings(int NB, int KC, int TB) { return lm_by_rings(NB, KC, TB, 256); }
int host_lm_once(int NB, int KC) { return lm_once(NB, KC, 256); }
int host_tiles_once(int NB, int KC, int rg, int slabs) { return tiles_once((long)NB * KC, rg, slabs != 0); }
int host_gate_up_by_four(int NB, int KC) { return gate_up_by_four(NB, KC, 256); }

// the tile of workgroup `id` as g * 1000000 + sweep * 1000 + ks; -1: none
int host_tile_at(int id, int NG, int SG, int KS, int bs) {
    const TileAt t = tile_at(id, NG, SG, KS, bs);
    return t.g < 0 ? -1 : t.g * 1000000 + t.sweep * 1000 + t.ks;
}

// sweeps in whole tiles * 100 + slabs of the others
int host_tile_plan(int NG, int SG, int KC, int split, long floats) {
    const TilePlan p = tile_plan(NG, SG, KC, 256, split != 0, (size_t)floats);
    return p.whole * 100 + p.KS;
}

// slices of K * 1000 + tiles of a slice; 0: no slice fits
int host_stream_split(int NB, int KC, int most) {
    const StreamSplit p = stream_split(NB, KC, 256, most);
    return p.slices * 1000 + p.tiles;
}
int host_stream_pays_ffn(int d, int F, int KV, int layers, int keys) { return stream_pays(d, F, KV, layers, keys); }
int host_stream_pays(int d, int KV, int layers, int keys) { return stream_pays(d, 4 * d, KV, layers, keys); }

// The fetching waves' list of every workgroup of a model whose matrices lie apart from each other: slots it begins (layers x phases, then the
// ones requested past the end of the list), each of them the slot the multiplying waves read there and every byte inside the unit.  Returns the
// bytes requested outside, or -1 where a slot is another one than is read.
long host_stream_list(int L, const int *NB, const int *KC, const int *ks_log2, const int *KCs, int G) {
    StreamModel sm{};
    sm.L = L;
    size_t at = 0;
    for (int j = 0; j < 4; ++j) {
        sm.m[j] = StreamMat{at, NB[j], KC[j], ks_log2[j], KCs[j]};
        at += (size_t)NB[j] * KC[j] * 512 + 8192;
    }
    sm.layer_stride = at;
    sm.base = (const bf16_t *)0x10000000;
    sm.m[4] = StreamMat{0, NB[4], KC[4], ks_log2[4], KCs[4]};
    sm.lm = sm.base + at * L;
    long outside = 0;
    for (int wg = 0; wg < G; ++wg) {
        StreamList pos;
        pos.enter(sm, 0, 0, wg, G);
        size_t end = 0;
        auto take = [&]() {
            for (int tile = 0; tile < kFusedWaves; ++tile) {
                const size_t last = pos.cur + (size_t)pos.request(tile) * 1024 + 1024;
                if (last > end) outside += (long)(last - end);
            }
            pos.next(sm, wg, G);
        };
        for (int l = 0; l < L; ++l)
            for (int j = 0; j < (l + 1 < L ? 4 : 5); ++j) {
                const StreamShare s = stream_share(sm.m[j], wg, G);
                for (int u = 0; u < s.n; ++u)
                    for (int t = 0; t < s.kcn; t += kFusedWaves) {
                        const size_t tiles = (size_t)(s.rb0 + u * s.step) * sm.m[j].KC + s.kc0;
                        const size_t first = (size_t)(j == 4 ? sm.lm : sm.base + l * sm.layer_stride + sm.m[j].off) + tiles * 1024;
                        if (pos.cur != first + (size_t)t * 1024) return -1;
                        end = first + (size_t)s.kcn * 1024;
                        take();
                    }
            }
        for (int i = 0; i < kStreamDepth - 1; ++i) take();      // the ring is filled to the end
    }
    return outside;
}

// 160 KB of LDS, 256 workgroups: a slice's columns of matrix j, 0 where the model is not taken
int host_stream_slice(int d, int H, int KV, int hd, int F, int j) {
    StreamModel sm{}; StreamExchange ex{};
    return stream_plan(StreamDims{d, H, KV, hd, F, 128256, 16}, 256, (size_t)160 << 10, &sm, &ex) ? sm.m[j].KCs * 32 : 0;
}

// `n` handles in threads of their own, each launching `times` on its stream: launches that another handle's stream was queued after without having
// waited for them, + 1000000 per launch that the last holder had not ended with.
int host_turns(int n, int times) {
    LaunchTurns<int, 2> turns;
    std::vector<std::atomic<int>> queued(n), seen(n);      // launches on a stream; how many of the last one's the stream that waited last has seen
    std::atomic<int> last{-1}, bad{0};
    std::vector<std::thread> pool;
    for (int i = 0; i < n; ++i)
        pool.emplace_back([&, i] {
            for (int k = 0; k < times; ++k) {
                const int rc = turns.launch(1, &queued[i], i, [&](int on) { seen[i] = on * 10000 + queued[on]; return 0; }, [&] {
                    std::this_thread::sleep_for(std::chrono::microseconds(300));       // a launch takes a while before it is queued
                    const int before = last;
                    if (before >= 0 && before != i && seen[i] != before * 10000 + queued[before]) ++bad;
                    ++queued[i]; last = i;
                    return 0;
                });
                if (rc) ++bad;
            }
        });
    for (auto &t : pool) t.join();
    for (int i = 0; i < n; ++i) turns.end(1, &queued[i], [&] { if (last != i) bad += 1000000; last = -1; });
    return bad;
}

// a refused launch leaves the turn where it was, so that the next handle waits for the launch that did run
int host_turn_refused() {
    LaunchTurns<int, 1> turns;
    int a, b, c, waited = -1;
    const auto wait = [&](int on) { waited = on; return 0; };
    turns.launch(0, &a, 7, wait, [] { return 0; });
    if (waited != -1 || turns.launch(0, &b, 8, wait, [] { return 5; }) != 5 || waited != 7) return -1;
    waited = -1;
    turns.launch(0, &c, 9, wait, [] { return 0; });
    return waited;
}

}  // extern "C"

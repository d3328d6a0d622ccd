// k_decode_stream's view of a model: how its matrices are cut, what the workgroups hand over where, and the list of weight
// tiles a workgroup's fetching waves walk.  Sizes and addresses alone.
#pragma once
#include "common.hpp"
#include "rules.hpp"

namespace ead {

constexpr int kStreamDepth = 14;                 // ring slots
constexpr int kStreamSlotBytes = 8192;           // 8 tiles of 1 KB
constexpr int kStreamProducers = 2;
constexpr int kStreamLoads = kFusedWaves / kStreamProducers;   // tile loads per fetching wave and slot
constexpr int kStreamThreads = (kFusedWaves + kStreamProducers) * 64;
static_assert(kStreamLoads * (kStreamDepth - 1) <= 63, "outstanding loads must fit the vector memory counter");
constexpr int kStreamPieces = 3;                 // float4 pieces of the residual stream per thread
constexpr int kStreamMaxWidth = kStreamPieces * 4 * kFusedThreads;      // d_model this kernel serves
constexpr int kStreamMaxSlices = 4;              // slices of K a matrix may be cut into
constexpr int kStreamStage = 8;                  // float4 pieces of the SwiGLU products a thread stages at once
// columns of a slice of matrix j (StreamModel) that the routine staging its activations holds in registers: the attention output comes in as many
// pieces as the residual stream
constexpr int stream_stage_most(int j) { return 4 * kFusedThreads * (j == 3 ? kStreamStage : kStreamPieces); }

// How a matrix is split: row blocks, tiles of a row block, slices of K (a power of two) and tiles of a slice (the last may be shorter).
struct StreamMat { size_t off; int NB, KC, ks_log2, KCs; };
// Where a model's packed weights are: matrix j (0 QKV, 1 output projection, 2 gate/up, 3 down) of layer l starts at
// base + l * layer_stride + m[j].off (elements); m[4] is the LM head, at lm.
struct StreamModel {
    const bf16_t *base, *lm; size_t layer_stride;
    StreamMat m[5];
    int L;
};

// The exchange buffer of a launch and the one to be emptied for the next: regions of a layer, in words.
struct StreamExchange {
    float *now, *next;
    int layer_words, total_words;            // of this model's layers; of both buffers as a whole
    int qkv, att, ml, o, h, down;            // region offsets inside a layer
};

// columns of activations the stage holds beside the ring (three half-precision terms a column), of `lds` bytes a workgroup may have
inline int stream_stage_cols(size_t lds) {
    const size_t rest = (size_t)kStreamDepth * kStreamSlotBytes + (2 * kFusedWaves * 16 + 64) * sizeof(float) + 256;
    return lds > rest ? std::max(0, (int)((lds - rest) / 6) - 8) : 0;
}

struct StreamDims { int d, H, KV, hd, F, V, L; };

// How k_decode_stream takes a model on `grid` workgroups of `lds` bytes (all but where the weights are), and the regions of its exchange; false
// where it does not serve it: the key splits of all KV heads need workgroups of their own, a slice of K has to fit the stage and the
// registers of the routine that stages it, and every workgroup needs a unit of some matrix.
inline bool stream_plan(const StreamDims &q, int grid, size_t lds, StreamModel *sm, StreamExchange *ex) {
    const int NQ = q.H * q.hd, NK = q.KV * q.hd, stage = stream_stage_cols(lds);
    if (q.d > kStreamMaxWidth || q.KV * kFusedMaxSplits > grid) return false;
    sm->L = q.L;
    const int rows[5] = {NQ + 2 * NK, q.d, 2 * q.F, q.d, q.V}, cols[5] = {q.d, NQ, q.d, q.F, q.d};
    for (int j = 0; j < 5; ++j) {
        StreamMat &t = sm->m[j];
        t.off = 0; t.NB = rows[j] / 16; t.KC = cols[j] / 32;
        const int most = std::min(stage, stream_stage_most(j));
        const bool cut = j == 0 || j == 1 || j == 3;      // gate/up and the LM head need whole sums
        const StreamSplit sp = cut ? stream_split(t.NB, t.KC, grid, most) : StreamSplit{1, t.KC};
        if (!sp.slices || sp.tiles * 32 > most) return false;
        t.ks_log2 = sp.slices == 4 ? 2 : sp.slices - 1; t.KCs = sp.tiles;
    }
    if (std::max(sm->m[2].NB, sm->m[4].NB) < grid) return false;      // a workgroup without any unit has nothing to fetch
    ex->qkv = 0; ex->att = (NQ + 2 * NK) << sm->m[0].ks_log2; ex->ml = ex->att + NQ * kFusedMaxSplits; ex->o = ex->ml + q.H * kFusedMaxSplits * 2;
    ex->h = ex->o + (q.d << sm->m[1].ks_log2); ex->down = ex->h + q.F; ex->layer_words = ex->down + (q.d << sm->m[3].ks_log2);
    return true;
}

// A workgroup's share of a matrix: which slice, how many row blocks, from which one on, how far apart; the slice's tiles.
struct StreamShare { int slice, rb0, step, n, kc0, kcn; };
__device__ __forceinline__ StreamShare stream_share(const StreamMat &m, int wg, int G) {
    StreamShare s;
    s.step = G >> m.ks_log2; s.slice = wg & ((1 << m.ks_log2) - 1); s.rb0 = wg >> m.ks_log2;
    s.n = s.rb0 < min(s.step, m.NB) ? (m.NB - s.rb0 + s.step - 1) / s.step : 0;
    s.kc0 = s.slice * m.KCs; s.kcn = min(m.KCs, m.KC - s.kc0);
    return s;
}

// The fetching waves' position in the list of slots of their workgroup.  Everything is the same in all lanes and
// lives in scalar registers; the matrices' descriptions come from the kernel arguments by scalar loads, so that the loop
// around the tile loads touches no vector memory but the weights.  (An array of descriptions that the compiler put into
// scratch memory cost a wait for all outstanding loads at every matrix.)
__device__ __forceinline__ int uni(int v) { return __builtin_amdgcn_readfirstlane(v); }
__device__ __forceinline__ size_t uni(size_t v) {
    const uint32_t lo = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)v);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)(v >> 32));
    return ((size_t)hi << 32) | (size_t)lo;
}
struct StreamList {
    int l, j, units;                 // layer, matrix, units of it still to come (this one included)
    int left, kcn;                   // tiles of this unit from the current slot on; of a whole unit
    size_t cur, unit, step;          // byte addresses: the slot's first tile, the unit's; distance of two units
    // the tile of the slot that is requested in the place of tile `i`: tiles past the end of a unit are its last one again
    __device__ __forceinline__ int request(int i) const { return min(i, min(uni(left), kFusedWaves) - 1); }
    // to the first unit of matrix jj of layer ll or, where the workgroup has none there, of the next one that has; past the end of the list
    // the position stays on its last slot, with the tiles that slot has (the weights may end there)
    __device__ __forceinline__ void enter(const StreamModel &sm, int ll, int jj, int wg, int G) {
        for (;; ++jj) {
            if (jj == 4 && ll < sm.L - 1) { jj = 0; ++ll; }
            if (jj > 4) return;
            const StreamShare s = stream_share(sm.m[jj], wg, G);
            if (s.n == 0) continue;
            l = ll; j = jj; units = s.n; left = kcn = s.kcn;
            const size_t first = (size_t)(jj == 4 ? sm.lm : sm.base + (size_t)ll * sm.layer_stride + sm.m[jj].off);
            unit = cur = uni(first + ((size_t)s.rb0 * sm.m[jj].KC + s.kc0) * 1024);
            step = (size_t)s.step * sm.m[jj].KC * 1024;
            return;
        }
    }
    __device__ __forceinline__ void next(const StreamModel &sm, int wg, int G) {
        if (left > kFusedWaves) { left -= kFusedWaves; cur += kStreamSlotBytes; return; }
        if (units > 1) { --units; unit += step; cur = unit; left = kcn; return; }
        enter(sm, l, j + 1, wg, G);
    }
};

}  // namespace ead

// One decode step of one model for a single token row as ONE persistent kernel whose weight
// stream never stops: bf16 models.
//
// A workgroup is eight consuming waves and two fetching waves.  The fetching waves walk, in
// order, every weight tile their workgroup will need during the whole step (all layers, then
// the LM head) and load it straight from global memory into a ring of 8 KB slots in LDS
// (global_load_lds, 16 bytes per lane); they hold no data in registers and never look at
// LDS, so nothing but the ring's capacity ever stops them.  While the consuming waves wait for
// the other workgroups or run the attention phase, the ring fills with the next matrix, and the first
// units of a phase are multiplied out of LDS the moment their activations are there.
//
// A slot is 8 consecutive tiles of one 16-row block (one per consuming wave: wave w of slot t
// multiplies tile 8 t + w).  Hand-over is ONE hardware barrier per slot: the fetching waves
// arrive when slot i has landed, the consuming waves when they have read slot i - 1; behind it
// the consumers read slot i and the fetchers refill the ring position of slot i - 1.  The
// consuming waves also meet at the hardware barrier for their own reasons (staging, reductions);
// the fetching waves cannot look at LDS without stalling their loads (measured: a
// fetching wave that polls a counter in LDS between its loads streams at 3.8 instead of 6.3 TB/s over
// the chip), so they learn nothing from memory: they replay the fixed sequence of those meetings
// and arrive at each.  Should the consuming waves
// leave early (a wait that was given up), the hardware barrier counts only the surviving waves
// and the fetching waves run their list to its end.
//
// Work split of a phase: units of one 16-row block x one of KS slices of K (stream_split), unit by unit over the
// workgroups; a workgroup's units are all of one slice, so it stages that slice of the activations only.  A unit's
// sums leave as they are; whoever stages the next phase adds the slices in order, and the residual stream, which all
// workgroups add up alike, never leaves their registers.
//
// What one workgroup hands to another goes through an exchange buffer that holds a pattern no published value has
// (kEmptyWord) until the value is there: a reader asks for the words themselves until none of them is empty.  That is one
// trip to memory and one back, 2.0 us for 2048 words read by each of 256 workgroups and 2.9 for 8192, where a grid barrier
// and the reads behind it take 3.2 and 4.6.  Every word is written once per launch; two buffers take turns, and a launch
// empties the one that the next will use.
//
// What bounds it (Llama 1B shape, 330 keys, us of a 36 us layer; 19 of weights at 6.4 TB/s): gate/up and down run at the stream's rate (8.5 and 4.5 of what the ring
// does not hold yet); a hand-over takes 2.3-3.4 of which the ring absorbs the part that it is not full; attention 5 and the hand-overs around it, during which the
// ring is full and nothing streams, are the rest.  Before, per layer: grid barriers, staging behind them and FMAs 43 us; the kernels per layer 42.
// Steps that led there, us a layer: exchange 43, fetching waves' position in scalar registers 37.5, non-temporal tiles and matrix-core products 37.8 (the
// LM head 525 MB 78 -> 72), lane-move reductions 35.6.
#pragma once
#include "fused.hpp"
#include "stream_list.hpp"

namespace ead {

typedef u32x4_t StreamRing[kFusedWaves][64];

// Request this fetching wave's tiles of the slot at the list position into the ring slot at LDS address `lds`.  Tiles past the
// end of a unit re-read its last tile (they meet zeros in the multiply), so that every slot is the same number of loads and the
// wait counts stay fixed; so do the slots requested past the end of the list.
__device__ __forceinline__ void stream_issue(const StreamList &pos, uint32_t lds, int p, int lane) {
    const bf16_t *base = reinterpret_cast<const bf16_t *>(uni(pos.cur));
#pragma unroll
    for (int q = 0; q < kStreamLoads; ++q) {
        const int tile = p + kStreamProducers * q;
        request_tile<true>(base, (uint32_t)(pos.request(tile) * 1024 + lane * 16), (uint32_t)uni((int)(lds + tile * 1024)));
    }
}

// ---- hardware barriers ---------------------------------------------------------------------------
// Every barrier of the workgroup is the hardware barrier and takes all ten waves.  The consuming
// waves meet at it for their own reasons too (staging, reductions): the number of
// such meetings per phase is fixed by the code below (kSync*), and the fetching waves, which have
// nothing to do there, simply arrive as many times (follow).
constexpr int kSyncStage = 2;            // any of the staging routines
constexpr int kSyncAttention = 3;        // stream_attention, or as many lone barriers of a workgroup without a share
constexpr int kSyncRowsEnd = 1;          // stream_rows, when the workgroup owned a unit
constexpr int kSyncGridBarrier = 2;      // bar_arrive + bar_wait, once, at the end

__device__ __forceinline__ void follow(int n) {
    for (int i = 0; i < n; ++i) asm volatile("s_barrier" ::: "memory");
}

// ---- the exchange ----------------------------------------------------------------------------------
constexpr uint32_t kEmptyWord = 0xFFFFFFFFu;      // a NaN: a published NaN of this pattern goes out as another one

__device__ __forceinline__ void publish(float *p, float v) {
    const uint32_t w = __float_as_uint(v);
    __hip_atomic_store(reinterpret_cast<uint32_t *>(p), w == kEmptyWord ? 0x7FC00000u : w, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

constexpr int kCoherentLoad = 16 | (int)0x80000000;      // cache policy of the buffer loads: served past the XCD's L2 (sc1), volatile
typedef __amdgpu_buffer_rsrc_t StreamRsrc;
__device__ __forceinline__ StreamRsrc exchange_rsrc(float *base, int words) {
    return __builtin_amdgcn_make_buffer_rsrc((void *)base, 0, words * 4, 0x00020000);
}

// Waits until the pieces of 16 bytes at byte offsets voff[i] (those that `present` names; a lane that needs none passes an offset another lane
// reads) of the region at `soff` are all published, and returns them.  False: given up, and nothing may be done with the values.
template <int N, typename Present>
__device__ __forceinline__ bool collect(StreamRsrc rsrc, int soff, const int (&voff)[N], Present present, u32x4_t (&v)[N], const GridBar &bar) {
    for (int spins = 0;; ++spins) {
#pragma unroll
        for (int i = 0; i < N; ++i)
            if (present(i)) v[i] = __builtin_amdgcn_raw_buffer_load_b128(rsrc, voff[i], soff, kCoherentLoad);
        bool full = true;
#pragma unroll
        for (int i = 0; i < N; ++i)
            if (present(i)) full = full && v[i].x != kEmptyWord && v[i].y != kEmptyWord && v[i].z != kEmptyWord && v[i].w != kEmptyWord;
        if (__all(full)) return true;
        if (spins >= bar.spin_limit || ((spins & 1023) == 1023 && ld_coherent(bar.abort_flag))) return false;
        asm volatile("" ::: "memory");
    }
}

__device__ __forceinline__ f32x4e_t as_floats(u32x4_t w) { return __builtin_bit_cast(f32x4e_t, w); }

// ---- reductions by lane moves inside a row of sixteen (no trip through LDS, which every phase would wait for several times) ----
template <int CTRL> __device__ __forceinline__ float moved(float v) { return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), CTRL, 0xF, 0xF, true)); }
constexpr int kXor1 = 0xB1, kXor2 = 0x4E, kMirror8 = 0x141, kMirror16 = 0x140;
// the sum over groups of N neighbouring lanes, in all of them
template <int N> __device__ __forceinline__ float lanes_sum(float v) {
    static_assert(N == 4 || N == 8 || N == 16, "a row of sixteen lanes at most");
    v += moved<kXor1>(v); v += moved<kXor2>(v);
    if constexpr (N >= 8) v += moved<kMirror8>(v);
    if constexpr (N >= 16) v += moved<kMirror16>(v);
    return v;
}
__device__ __forceinline__ float lane_value(float v, int l) { return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), l)); }
__device__ __forceinline__ float rows_sum(float v) {
    v = lanes_sum<16>(v);
    return (lane_value(v, 0) + lane_value(v, 16)) + (lane_value(v, 32) + lane_value(v, 48));
}
__device__ __forceinline__ float rows_max(float v) {
    v = fmaxf(v, moved<kXor1>(v)); v = fmaxf(v, moved<kXor2>(v)); v = fmaxf(v, moved<kMirror8>(v)); v = fmaxf(v, moved<kMirror16>(v));
    return fmaxf(fmaxf(lane_value(v, 0), lane_value(v, 16)), fmaxf(lane_value(v, 32), lane_value(v, 48)));
}

// ---- staging -----------------------------------------------------------------------------------------
// The work-item's number, opaque: what these routines derive from it is computed where it is used and not kept, in
// registers or spilled, across the loop over the layers that calls them on the same regions every time.
__device__ __forceinline__ int fresh_tid() {
    int t = threadIdx.x;
    asm volatile("" : "+v"(t));
    return t;
}
// Thread t of the consuming waves keeps elements (t + i * 512) * 4 .. + 3 of the residual stream in x[i].

// x += the KS slices' sums of `n` rows that lie one behind the other at word `off`
__device__ __forceinline__ bool add_sums(f32x4e_t (&x)[kStreamPieces], StreamRsrc rsrc, int off, int n, int KS, const GridBar &bar) {
    constexpr int NS = kStreamMaxSlices;
    const int tid = fresh_tid();
    int voff[kStreamPieces * NS];
    u32x4_t v[kStreamPieces * NS];
#pragma unroll
    for (int i = 0; i < kStreamPieces; ++i)
#pragma unroll
        for (int s = 0; s < NS; ++s) voff[i * NS + s] = (s * n + min((tid + i * kFusedThreads) * 4, n - 4)) * 4;
    if (!collect(rsrc, off * 4, voff, [&](int j) { return j % NS < KS && j / NS * 4 * kFusedThreads < n; }, v, bar)) return false;
#pragma unroll
    for (int i = 0; i < kStreamPieces; ++i)
#pragma unroll
        for (int s = 0; s < NS; ++s)
            if (s < KS && (tid + i * kFusedThreads) * 4 < n) x[i] += as_floats(v[i * NS + s]);
    return true;
}

// ---- activations as half-precision terms ---------------------------------------------------------------
// The products run on the matrix cores, whose sixteen columns a single row leaves idle: three of them take the activations'
// terms, v = hi + mid / 2^11 + lo / 2^22 with halves hi, mid, lo of 11 bits each, which hold a float32's 24 bits.  The vector is
// first scaled by the power of two that brings its largest magnitude to 2^14 .. 2^15, so that no term overflows
// and elements 2^-29 of the largest still keep all their bits.  (With FMAs on float32 activations a slot cost 300 ns, of which half was
// arithmetic and a third reading the activations.)
struct StreamScale { float up, down; };
__device__ __forceinline__ StreamScale scale_for(float largest) {
    int e = (int)((__float_as_uint(largest) >> 23) & 255u);
    e = e == 255 ? 141 : max(e, 15);                       // not finite: as it is; tiny or zero: by 2^126
    return StreamScale{__uint_as_float((uint32_t)(268 - e) << 23), __uint_as_float((uint32_t)(e - 14) << 23)};
}
__device__ __forceinline__ float largest_of(f32x4e_t v) { return fmaxf(fmaxf(fabsf(v.x), fabsf(v.y)), fmaxf(fabsf(v.z), fabsf(v.w))); }

// Where the terms of a slice lie in LDS: term m of column k at xt[m * stride + k].
struct StreamTerms { uint16_t *xt; int stride; };
__device__ __forceinline__ void put_terms(const StreamTerms &x, int k, f32x4e_t v) {
    typedef _Float16 f16x4_t __attribute__((ext_vector_type(4)));
    const f16x4_t hi = __builtin_convertvector(v, f16x4_t);
    const f32x4e_t r = (v - __builtin_convertvector(hi, f32x4e_t)) * 2048.f;
    const f16x4_t mid = __builtin_convertvector(r, f16x4_t);
    const f16x4_t lo = __builtin_convertvector((r - __builtin_convertvector(mid, f32x4e_t)) * 2048.f, f16x4_t);
    *reinterpret_cast<f16x4_t *>(x.xt + k) = hi;
    *reinterpret_cast<f16x4_t *>(x.xt + x.stride + k) = mid;
    *reinterpret_cast<f16x4_t *>(x.xt + 2 * x.stride + k) = lo;
}

// The largest of the threads' values over the consuming waves (one of the two meetings of a staging routine)
__device__ __forceinline__ float block_largest(float v, float *s_max) {
    const int tid = threadIdx.x;
    v = rows_max(v);
    if ((tid & 63) == 0) s_max[tid >> 6] = v;
    __syncthreads();
    float r = 0.f;
#pragma unroll
    for (int w = 0; w < kFusedWaves; ++w) r = fmaxf(r, s_max[w]);
    return r;
}

// The terms of x * gain, of the columns [c0, c0 + cn) of this workgroup's slice; returns the factor (1 / rms, scale taken back) for the sums to come
__device__ __forceinline__ float stage_norm_x(const StreamTerms &xt, float *s_red, float *s_max, const f32x4e_t (&x)[kStreamPieces], const f32x4e_t (&gn)[kStreamPieces],
                                              int n, int c0, int cn, float eps) {
    const int tid = fresh_tid();
    float ss = 0.f, big = 0.f;
#pragma unroll
    for (int i = 0; i < kStreamPieces; ++i) {
        if ((tid + i * kFusedThreads) * 4 < n) {
            ss += x[i].x * x[i].x + x[i].y * x[i].y + x[i].z * x[i].z + x[i].w * x[i].w;
            big = fmaxf(big, largest_of(x[i] * gn[i]));
        }
    }
    ss = rows_sum(ss);
    if ((tid & 63) == 0) s_red[tid >> 6] = ss;
    const StreamScale sc = scale_for(block_largest(big, s_max));
    float tot = 0.f;
#pragma unroll
    for (int w = 0; w < kFusedWaves; ++w) tot += s_red[w];
#pragma unroll
    for (int i = 0; i < kStreamPieces; ++i) {
        const int k = (tid + i * kFusedThreads) * 4;
        if (k < n && k >= c0 && k < c0 + cn) put_terms(xt, k - c0, x[i] * gn[i] * sc.up);
    }
    __syncthreads();
    return sc.down / sqrtf(tot / (float)n + eps);
}

__device__ __forceinline__ void load_gain(f32x4e_t (&gn)[kStreamPieces], const float *gain, int n) {
    const int tid = fresh_tid();
#pragma unroll
    for (int i = 0; i < kStreamPieces; ++i) gn[i] = *(gptr<f32x4e_t>)(gain + min((tid + i * kFusedThreads) * 4, n - 4));
}

// The terms of the words [c0, c0 + cn) of the region at word `off`; *factor: what takes the scale back from the sums
__device__ __forceinline__ bool stage_words(const StreamTerms &xt, float *s_max, StreamRsrc rsrc, int off, int c0, int cn, const GridBar &bar, float *factor) {
    const int tid = fresh_tid();
    int voff[kStreamStage];
    u32x4_t v[kStreamStage];
#pragma unroll
    for (int i = 0; i < kStreamStage; ++i) voff[i] = (c0 + min((tid + i * kFusedThreads) * 4, cn - 4)) * 4;
    if (!collect(rsrc, off * 4, voff, [&](int i) { return i * 4 * kFusedThreads < cn; }, v, bar)) return false;
    float big = 0.f;
#pragma unroll
    for (int i = 0; i < kStreamStage; ++i)
        if (i * 4 * kFusedThreads < cn) big = fmaxf(big, largest_of(as_floats(v[i])));
    const StreamScale sc = scale_for(block_largest(big, s_max));
#pragma unroll
    for (int i = 0; i < kStreamStage; ++i) {
        const int k = (tid + i * kFusedThreads) * 4;
        if (k < cn) put_terms(xt, k, as_floats(v[i]) * sc.up);
    }
    __syncthreads();
    *factor = sc.down;
    return true;
}

// The terms of columns [c0, c0 + cn) of the attention output: the merge of its S splits' un-normalised results.  A thread takes
// four neighbouring dimensions of a head at a time.
template <int HD>
__device__ __forceinline__ bool stage_attention(const StreamTerms &xt, float *s_max, StreamRsrc rsrc, int att, int ml, int c0, int cn, int S, const GridBar &bar,
                                                float *factor) {
    const int tid = fresh_tid();
    f32x4e_t r[kStreamPieces];
    float big = 0.f;
#pragma unroll
    for (int i = 0; i < kStreamPieces; ++i) {
        r[i] = f32x4e_t{0.f, 0.f, 0.f, 0.f};
        if (i * 4 * kFusedThreads >= cn) continue;
        const int kk = c0 + min((tid + i * kFusedThreads) * 4, cn - 4), h = kk / HD, dd = kk % HD;
        // pieces 0 .. 7: the splits' results; 8 .. 11: their maxima and sums, two splits to a piece
        constexpr int NS = kFusedMaxSplits;
        int voff[NS + NS / 2];
        u32x4_t v[NS + NS / 2];
#pragma unroll
        for (int s = 0; s < NS; ++s) voff[s] = (att + (h * NS + s) * HD + dd) * 4;
#pragma unroll
        for (int s = 0; s < NS / 2; ++s) voff[NS + s] = (ml + (h * NS + 2 * s) * 2) * 4;
        if (!collect(rsrc, 0, voff, [&](int j) { return j < NS ? j < S : 2 * (j - NS) < S; }, v, bar)) return false;
        const u32x4_t *m4 = v + NS;
        float M = kNegBig;
#pragma unroll
        for (int s = 0; s < NS; ++s)
            if (s < S) M = fmaxf(M, __uint_as_float(s & 1 ? m4[s >> 1].z : m4[s >> 1].x));
        float L = 0.f;
        f32x4e_t acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int s = 0; s < NS; ++s)
            if (s < S) {
                const float c = __expf(__uint_as_float(s & 1 ? m4[s >> 1].z : m4[s >> 1].x) - M);
                L += __uint_as_float(s & 1 ? m4[s >> 1].w : m4[s >> 1].y) * c;
                acc += as_floats(v[s]) * c;
            }
        r[i] = acc * (1.0f / L);
        big = fmaxf(big, largest_of(r[i]));
    }
    const StreamScale sc = scale_for(block_largest(big, s_max));
#pragma unroll
    for (int i = 0; i < kStreamPieces; ++i) {
        const int k = (tid + i * kFusedThreads) * 4;
        if (k < cn) put_terms(xt, k, r[i] * sc.up);
    }
    __syncthreads();
    *factor = sc.down;
    return true;
}

struct StreamPos { int ri; int nblk; };   // ring position of the next slot; units taken so far (whose turn, which buffer)

// The consuming side of one matrix: this workgroup's units, the activations' terms of its slice in LDS, sums scaled by `scale`.
// SWIGLU publishes the products, LOGITS folds the logits into the entropy statistics, the others publish the sums.
template <int EPI>
__device__ __forceinline__ void stream_rows(const LinArgs<bf16_t> &a, float *out, const StreamRing *ring, const StreamTerms &xt, const uint16_t *xzero,
                                            float *red, const StreamShare &sh, float scale, StreamPos &sp, EntStat &st) {
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int nt = (sh.kcn + 7) >> 3, col = lane & 15;
    const uint16_t *xq = col < 3 ? xt.xt + col * xt.stride + (lane >> 4) * 8 : xzero;
    const int xstep = col < 3 ? kFusedWaves * 32 : 0;            // from a wave's tile to its next
    const float weight = col == 0 ? scale : col == 1 ? scale * (1.f / 2048.f) : col == 2 ? scale * (1.f / 4194304.f) : 0.f;
    int pend = -1, pend_wave = 0, pend_par = 0;
    auto finish = [&]() {          // the row block `pend`: add the waves' partial sums and pass them on
        if (wave == pend_wave && lane < 16) {
            float v = 0.f;
#pragma unroll
            for (int w = 0; w < kFusedWaves; ++w) v += red[(pend_par * kFusedWaves + w) * 16 + lane];
            const int p = pend * 16 + lane;
            if constexpr (EPI == EPI_SWIGLU) {
                const float other = __shfl_xor(v, 1, kWave);       // even lane: gate, odd lane: up
                if (!(lane & 1)) publish(out + (p >> 1), v / (1.f + __expf(-v)) * other);
            } else if constexpr (EPI == EPI_LOGITS) {
                epilogue<bf16_t, EPI_LOGITS>(a, p, 0, v, true, st, EpiPre{});
            } else {
                publish(out + (size_t)sh.slice * a.Np + p, v);
            }
        }
    };
    for (int u = 0, rb = sh.rb0; u < sh.n; ++u, rb += sh.step) {
        const int my_wave = sp.nblk & (kFusedWaves - 1), par = sp.nblk & 1;
        // A slot's tile and activations are read right behind its barrier and multiplied behind the NEXT
        // one, while the next slot's reads are in flight.
        f32x4_t acc = {0.f, 0.f, 0.f, 0.f};
        u32x4_t w{}, x{};
        const uint16_t *xp = xq + (col < 3 ? wave * 32 : 0);
        for (int t = 0; t < nt; ++t) {
            asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
            const u32x4_t wn = ring[sp.ri][wave][lane];
            sp.ri = sp.ri + 1 == kStreamDepth ? 0 : sp.ri + 1;
            const u32x4_t xn = *reinterpret_cast<const u32x4_t *>(t * kFusedWaves + wave < sh.kcn ? xp : xzero);
            xp += xstep;
            if (t == 0 && pend >= 0) finish();
            if (t > 0) acc = __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(f16x8_t, w), __builtin_bit_cast(f16x8_t, x), acc, 0, 0, 0);
            w = wn; x = xn;
        }
        acc = __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(f16x8_t, w), __builtin_bit_cast(f16x8_t, x), acc, 0, 0, 0);
        f32x4e_t sum;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            float v = acc[i] * weight;
            sum[i] = lanes_sum<4>(v);
        }
        if (col == 0) *reinterpret_cast<f32x4e_t *>(red + (par * kFusedWaves + wave) * 16 + (lane >> 4) * 4) = sum;
        pend = rb; pend_wave = my_wave; pend_par = par;
        ++sp.nblk;
    }
    if (pend >= 0) { __syncthreads(); finish(); }     // kSyncRowsEnd
}

// ---- attention of the row, split over (KV head, key split) ---------------------------------------------
// A wave serves one of the G query heads that share the KV head on one slice of the split's keys (wave w: head w % G, slice
// w / G), so the per-lane state is one head's worth.  The first keys and values are requested before the row's query is there, the
// next ones one round ahead.  The newest position's key and value come with the query through the exchange; the workgroup whose
// split holds that position appends them to the caches.
template <int HD, int G>
__device__ __forceinline__ bool stream_attention(const FusedArgs<bf16_t> &a, const FusedLayer<bf16_t> &ly, StreamRsrc rsrc, float *now,
                                                 const StreamExchange &ex, int layer, int KS, int seq, int pos, int S, float *lds) {
    typedef bf16_t KT;
    constexpr int LPK = HD / 8, KPI = 64 / LPK, NI = 4, CH = NI * KPI;
    constexpr int NS = kFusedWaves / G;            // key slices per workgroup
    const int kvh = blockIdx.x / S, split = blockIdx.x % S;
    const int nkeys = pos + 1, per = (nkeys + S - 1) / S;
    const int key0 = split * per, key1 = min(key0 + per, nkeys);
    const int tid = fresh_tid(), lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int slot = lane / LPK, dl = lane % LPK;
    const int g = wave % G, slice = wave / G;
    const bool active = slice < NS, own = pos >= key0 && pos < key1;
    // LDS: the G scaled queries, the new key and value as the caches hold them, then the waves' results
    float *qs = lds;
    bf16_t *kn = reinterpret_cast<bf16_t *>(qs + G * HD), *vn = kn + HD;
    float *wo = qs + (G + 1) * HD, *wm = wo + kFusedWaves * HD, *wl = wm + kFusedWaves;
    const size_t base = ((size_t)seq * a.KV + kvh) * (size_t)a.fin.s.max_seq * HD;
    const KT *kb = ly.kcache + base + dl * 8, *vb = ly.vcache + base + dl * 8;
    Vec8<KT> kx[2][NI], vx[2][NI];
    auto request = [&](Vec8<KT> (&k)[NI], Vec8<KT> (&v)[NI], int c0) {
#pragma unroll
        for (int i = 0; i < NI; ++i) {
            const int kk = min(c0 + i * KPI + slot, key1 - 1);
            k[i].load(kb + (size_t)max(kk, 0) * HD); v[i].load(vb + (size_t)max(kk, 0) * HD);
        }
    };
    const int c00 = key0 + slice * CH;
    if (active) { request(kx[0], vx[0], c00); request(kx[1], vx[1], c00 + NS * CH); }
    // the G query heads, and for the newest position its key and value: four packed rows a thread
    {
        const int NQ = a.H * HD, NK = a.KV * HD, nq4 = G * HD / 4, n4 = own ? nq4 + HD / 2 : nq4;
        const int i4 = min(tid, n4 - 1), part = i4 < nq4 ? 0 : i4 < nq4 + HD / 4 ? 1 : 2;      // query, key, value
        const int r4 = part == 0 ? i4 : part == 1 ? i4 - nq4 : i4 - nq4 - HD / 4;
        const int row = (part == 0 ? kvh * G * HD : part == 1 ? NQ + kvh * HD : NQ + NK + kvh * HD) + r4 * 4;
        const int r = (r4 * 4) % HD, i = r >> 1;       // packed rows (2i, 2i + 1) of a head are its dimensions (i, i + HD / 2)
        const f32x4e_t cs = *(gptr<f32x4e_t>)(reinterpret_cast<const float *>(a.rope + (size_t)pos * (HD / 2) + i));
        int voff[kStreamMaxSlices];
        u32x4_t w[kStreamMaxSlices];
#pragma unroll
        for (int s = 0; s < kStreamMaxSlices; ++s) voff[s] = (s * (NQ + 2 * NK) + row) * 4;
        if (!collect(rsrc, (layer * ex.layer_words + ex.qkv) * 4, voff, [&](int s) { return s < KS; }, w, a.bar)) return false;
        f32x4e_t v = as_floats(w[0]);
#pragma unroll
        for (int s = 1; s < kStreamMaxSlices; ++s)
            if (s < KS) v += as_floats(w[s]);
        if (tid < n4) {
            if (part < 2) v = f32x4e_t{v.x * cs.x - v.y * cs.y, v.x * cs.y + v.y * cs.x, v.z * cs.z - v.w * cs.w, v.z * cs.w + v.w * cs.z};
            if (part == 0) {
                const float scale = 1.0f / sqrtf((float)HD);
                float *q = qs + (r4 * 4) / HD * HD + i;
                q[0] = v.x * scale; q[1] = v.z * scale; q[HD / 2] = v.y * scale; q[HD / 2 + 1] = v.w * scale;
            } else if (part == 1) {
                const KT b0 = from_f32<KT>(v.x), b1 = from_f32<KT>(v.z), b2 = from_f32<KT>(v.y), b3 = from_f32<KT>(v.w);
                KT *d = ly.kcache + base + (size_t)pos * HD + i;
                kn[i] = b0; kn[i + 1] = b1; kn[i + HD / 2] = b2; kn[i + HD / 2 + 1] = b3;
                d[0] = b0; d[1] = b1; d[HD / 2] = b2; d[HD / 2 + 1] = b3;
            } else {
                const size_t tb = ((size_t)seq * a.KV + kvh) * HD * (size_t)a.fin.s.max_seq;
#pragma unroll
                for (int e = 0; e < 4; ++e) {       // rows of V are not permuted
                    const KT b = from_f32<KT>(e == 0 ? v.x : e == 1 ? v.y : e == 2 ? v.z : v.w);
                    vn[r + e] = b;
                    ly.vcache[base + (size_t)pos * HD + r + e] = b;
                    if (ly.vtcache) ly.vtcache[tb + vt_offset(r + e, pos, a.fin.s.max_seq)] = b;
                }
            }
        }
    }
    __syncthreads();
    float o[8], m = kNegBig, l = 0.f;
#pragma unroll
    for (int e = 0; e < 8; ++e) o[e] = 0.f;
    auto round = [&](Vec8<KT> (&k)[NI], Vec8<KT> (&v)[NI], const float (&qv)[8], int c0) {
        float s[NI];
#pragma unroll
        for (int i = 0; i < NI; ++i) {
            const int kk = c0 + i * KPI + slot;
            if (kk == pos) {
                k[i].raw = *reinterpret_cast<const u32x4_t *>(kn + dl * 8);
                v[i].raw = *reinterpret_cast<const u32x4_t *>(vn + dl * 8);
            }
            float kf[8];
            k[i].unpack(kf);
            float d = 0.f;
#pragma unroll
            for (int e = 0; e < 8; ++e) d += qv[e] * kf[e];
            d = lanes_sum<LPK>(d);
            s[i] = kk < key1 ? d : kNegBig;
        }
        float mc = s[0];
#pragma unroll
        for (int i = 1; i < NI; ++i) mc = fmaxf(mc, s[i]);
        const float mn = fmaxf(m, mc);
        const float corr = __expf(m - mn);
        l *= corr;
#pragma unroll
        for (int e = 0; e < 8; ++e) o[e] *= corr;
        m = mn;
#pragma unroll
        for (int i = 0; i < NI; ++i) {
            const bool in = c0 + i * KPI + slot < key1;      // past the split's end the value may be anything
            const float p = in ? __expf(s[i] - mn) : 0.f;
            l += p;
            float vf[8];
            v[i].unpack(vf);
#pragma unroll
            for (int e = 0; e < 8; ++e) o[e] += in ? p * vf[e] : 0.f;
        }
    };
    if (active) {
        float qv[8];
#pragma unroll
        for (int e = 0; e < 8; ++e) qv[e] = qs[g * HD + dl * 8 + e];
        for (int c0 = c00; c0 < key1; c0 += 2 * NS * CH) {
            round(kx[0], vx[0], qv, c0);
            if (c0 + 2 * NS * CH < key1) request(kx[0], vx[0], c0 + 2 * NS * CH);
            if (c0 + NS * CH < key1) {
                round(kx[1], vx[1], qv, c0 + NS * CH);
                if (c0 + 3 * NS * CH < key1) request(kx[1], vx[1], c0 + 3 * NS * CH);
            }
        }
    }
    // merge the key slots of the wave
#pragma unroll
    for (int off = LPK; off < 64; off <<= 1) {
        const float m2 = __shfl_xor(m, off, kWave), l2 = __shfl_xor(l, off, kWave);
        const float M = fmaxf(m, m2);
        const float ca = __expf(m - M), cb = __expf(m2 - M);
        l = l * ca + l2 * cb;
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            const float o2 = __shfl_xor(o[e], off, kWave);
            o[e] = o[e] * ca + o2 * cb;
        }
        m = M;
    }
    // waves meet in LDS: wo[wave][HD], wm[wave], wl[wave]
    if (slot == 0) {
#pragma unroll
        for (int e = 0; e < 8; ++e) wo[wave * HD + dl * 8 + e] = o[e];
        if (dl == 0) { wm[wave] = active ? m : kNegBig; wl[wave] = active ? l : 0.f; }
    }
    __syncthreads();
    float *att = now + (size_t)layer * ex.layer_words + ex.att, *ml = now + (size_t)layer * ex.layer_words + ex.ml;
    for (int e = tid; e < G * HD; e += kFusedThreads) {
        const int gg = e / HD, dd = e % HD, h = kvh * G + gg;
        float M = kNegBig;
#pragma unroll
        for (int sl = 0; sl < NS; ++sl) M = fmaxf(M, wm[sl * G + gg]);
        float L = 0.f, acc = 0.f;
#pragma unroll
        for (int sl = 0; sl < NS; ++sl) {
            const float c = __expf(wm[sl * G + gg] - M);
            L += wl[sl * G + gg] * c;
            acc += wo[(sl * G + gg) * HD + dd] * c;
        }
        publish(att + ((size_t)h * kFusedMaxSplits + split) * HD + dd, acc);
        if (dd == 0) {
            float *q = ml + ((size_t)h * kFusedMaxSplits + split) * 2;
            publish(q, M); publish(q + 1, L);
            // a reader takes two splits at a time: the one past the last is never written by anybody else
            if (split == S - 1 && (S & 1)) { publish(q + 2, kNegBig); publish(q + 3, 0.f); }
        }
    }
    __syncthreads();
    return true;
}

template <int HD, int G>
__global__ __launch_bounds__(kStreamThreads) void k_decode_stream(FusedArgs<bf16_t> a, StreamModel sm, StreamExchange ex) {
    typedef bf16_t WT;
    extern __shared__ __attribute__((aligned(16))) unsigned char smem_raw[];
    StreamRing *ring = reinterpret_cast<StreamRing *>(smem_raw);
    float *smem = reinterpret_cast<float *>(smem_raw + (size_t)kStreamDepth * kStreamSlotBytes);
    __shared__ int s_plan[4];        // seq, pos, token, whether to go on
    __shared__ int s_ok;
    __shared__ float s_red[kFusedWaves], s_max[kFusedWaves];
    float *red = smem, *zeros = red + 2 * kFusedWaves * 16, *xs = zeros + 64;       // 64 zeros
    const uint16_t *xzero = reinterpret_cast<const uint16_t *>(zeros);
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);

    if (wave >= kFusedWaves) {
        // ---- fetching waves ------------------------------------------------------------------
        const int p = wave - kFusedWaves, wg = blockIdx.x, G_ = gridDim.x;
        const uint32_t ring0 = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) unsigned char *)smem_raw;
        StreamList pos;
        pos.enter(sm, 0, 0, wg, G_);        // a workgroup owns a unit of some matrix: the launch has at most as many as the LM head has row blocks
        int ri = 0;
        for (int s = 0; s < kStreamDepth - 1; ++s) {
            stream_issue(pos, ring0 + ri * kStreamSlotBytes, p, lane);
            pos.next(sm, wg, G_);
            ri = ri + 1 == kStreamDepth ? 0 : ri + 1;
        }
        __syncthreads();                    // the consuming waves have set up their constants
        if (!uni(s_plan[3])) { wait_stores(); return; }      // (nothing may land in LDS after the workgroup has gone)
        // the consuming waves' phases, one by one: arrive where they meet, hand over a slot where they read one
        for (int l = 0; l <= sm.L; ++l)
            for (int kind = l < sm.L ? 0 : 5; kind < (l < sm.L ? 5 : 6); ++kind) {
                if (kind == 1) { follow(kSyncAttention); continue; }
                follow(kSyncStage);
                const StreamShare sh = stream_share(sm.m[kind == 0 ? 0 : kind - 1], wg, G_);
                const int n = sh.n * ((sh.kcn + 7) >> 3);
                for (int i = 0; i < n; ++i) {
                    asm volatile("s_waitcnt vmcnt(%0)\n\ts_barrier" ::"n"(kStreamLoads * (kStreamDepth - 2)) : "memory");
                    stream_issue(pos, ring0 + ri * kStreamSlotBytes, p, lane);
                    pos.next(sm, wg, G_);
                    ri = ri + 1 == kStreamDepth ? 0 : ri + 1;
                }
                if (n > 0) follow(kSyncRowsEnd);
            }
        follow(kSyncGridBarrier);
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        return;
    }

    // ---- consuming waves -----------------------------------------------------------------------
    if (tid < 64) zeros[tid] = 0.f;
    const int m = a.fin.model_id, MB = a.fin.s.max_batch;
    // the one sequence this model serves in this step, and its newest position
    if (tid == 0) {
        // Given up, in an earlier launch (the exchange is in no defined state then) or in this one while this workgroup was starting?  One
        // thread looks, for all waves: where each looks by itself, some can leave and others go on with a plan that nobody has written.
        const int given_up = ld_coherent(a.bar.abort_flag);
        int seq = 0;
        for (int b = 0; b < a.batch; ++b)
            if (!a.fin.s.done[b] && a.fin.s.model[b] == m && a.fin.s.last_step[b] != a.fin.step) { seq = b; break; }
        const int pos = a.fin.s.kvlen[m * MB + seq];
        s_plan[0] = seq; s_plan[1] = pos; s_plan[2] = a.fin.s.tokens[(size_t)seq * a.fin.s.max_seq + pos];
        s_plan[3] = !given_up;
    }
    __syncthreads();
    if (!uni(s_plan[3])) return;
    BlockSync sync;
    StreamPos sp{0, 0};
    const int seq = uni(s_plan[0]), pos = uni(s_plan[1]);
    const WT *emb = a.embed + (size_t)s_plan[2] * a.d;
    const int NQ = a.H * HD, NK = a.KV * HD, G_ = gridDim.x, wg = blockIdx.x;
    // key splits of the attention phase: 64 keys or more each, as many workgroups as that gives
    const int S = min(kFusedMaxSplits, max(1, (pos + 1 + 63) / 64));
    const StreamRsrc rsrc = exchange_rsrc(ex.now, ex.layer_words * a.L);
    GridBar bar = a.bar;
    EntStat st; st.init();
    f32x4e_t x[kStreamPieces], gn[kStreamPieces];
#pragma unroll
    for (int i = 0; i < kStreamPieces; ++i) {       // the residual stream starts as the embedding row
        const int k = (tid + i * kFusedThreads) * 4;
        x[i] = f32x4e_t{0.f, 0.f, 0.f, 0.f};
        if (k < a.d) x[i] = f32x4e_t{to_f32(emb[k]), to_f32(emb[k + 1]), to_f32(emb[k + 2]), to_f32(emb[k + 3])};
    }

    // phases: per layer QKV, attention, output projection, gate/up, down; then the LM head.
    // Every workgroup-wide meeting below is counted in the kSync* constants the fetching waves follow.
    const int clear_per = (ex.total_words / 4 + a.L * G_ - 1) / (a.L * G_);      // float4 pieces of the other buffer a workgroup empties per layer
    // the terms' rows start 16 bytes apart from a multiple of the banks
    auto terms = [&](const StreamShare &sh) { return StreamTerms{reinterpret_cast<uint16_t *>(xs), sh.kcn * 32 + 8}; };
    auto share = [&](int j) { return stream_share(sm.m[j], wg, G_); };
    for (int l = 0; l < a.L; ++l) {
        const FusedLayer<WT> ly = a.layers[l];
        const int lo = l * ex.layer_words;
        float *now = ex.now + (size_t)lo;
        LinArgs<WT> p{};
        {                                       // RMSNorm + QKV
            const StreamShare sh = share(0);
            load_gain(gn, ly.g_attn, a.d);
            if (l > 0 && !add_sums(x, rsrc, lo - ex.layer_words + ex.down, a.d, 1 << sm.m[3].ks_log2, a.bar)) { give_up(a.bar); return; }
            const float inv = stage_norm_x(terms(sh), s_red, s_max, x, gn, a.d, sh.kc0 * 32, sh.kcn * 32, a.eps);
            p.Np = NQ + 2 * NK;
            stream_rows<EPI_QKV>(p, now + ex.qkv, ring, terms(sh), xzero, red, sh, inv, sp, st);
        }
        // rotary + KV append + attention
        if (wg < a.KV * S) {
            if (!stream_attention<HD, G>(a, ly, rsrc, ex.now, ex, l, 1 << sm.m[0].ks_log2, seq, pos, S, xs)) { give_up(a.bar); return; }
        } else follow(kSyncAttention);
        {                                       // output projection
            const StreamShare sh = share(1);
            float f = 1.f;
            if (sh.n == 0) follow(kSyncStage);
            else if (!stage_attention<HD>(terms(sh), s_max, rsrc, lo + ex.att, lo + ex.ml, sh.kc0 * 32, sh.kcn * 32, S, a.bar, &f)) { give_up(a.bar); return; }
            p.Np = a.d;
            stream_rows<EPI_RES>(p, now + ex.o, ring, terms(sh), xzero, red, sh, f, sp, st);
        }
        {                                       // residual, RMSNorm + gate/up + SwiGLU
            const StreamShare sh = share(2);
            load_gain(gn, ly.g_ffn, a.d);
            if (!add_sums(x, rsrc, lo + ex.o, a.d, 1 << sm.m[1].ks_log2, a.bar)) { give_up(a.bar); return; }
            const float inv = stage_norm_x(terms(sh), s_red, s_max, x, gn, a.d, sh.kc0 * 32, sh.kcn * 32, a.eps);
            for (int i = tid; i < clear_per; i += kFusedThreads) {
                const int c = (l * G_ + wg) * clear_per + i;
                if (c * 4 < ex.total_words) reinterpret_cast<u32x4_t *>(ex.next)[c] = u32x4_t{kEmptyWord, kEmptyWord, kEmptyWord, kEmptyWord};
            }
            p.Np = 2 * a.F;
            stream_rows<EPI_SWIGLU>(p, now + ex.h, ring, terms(sh), xzero, red, sh, inv, sp, st);
        }
        {                                       // down projection
            const StreamShare sh = share(3);
            float f = 1.f;
            if (sh.n == 0) follow(kSyncStage);
            else if (!stage_words(terms(sh), s_max, rsrc, lo + ex.h, sh.kc0 * 32, sh.kcn * 32, a.bar, &f)) { give_up(a.bar); return; }
            p.Np = a.d;
            stream_rows<EPI_RES>(p, now + ex.down, ring, terms(sh), xzero, red, sh, f, sp, st);
        }
    }
    {                                           // residual, final RMSNorm + LM head, entropy statistics folded in
        const StreamShare sh = share(4);
        load_gain(gn, a.g_final, a.d);
        if (!add_sums(x, rsrc, (a.L - 1) * ex.layer_words + ex.down, a.d, 1 << sm.m[3].ks_log2, a.bar)) { give_up(a.bar); return; }
        const float inv = stage_norm_x(terms(sh), s_red, s_max, x, gn, a.d, 0, a.d, a.eps);
        LinArgs<WT> p{};
        p.Np = a.V;
        stream_rows<EPI_LOGITS>(p, nullptr, ring, terms(sh), xzero, red, sh, inv, sp, st);
        if (lane < 16) {                        // one partial per (workgroup, wave)
            p.partials = a.lm_part + (size_t)wave * gridDim.x;
            logits_flush<WT, true>(p, 0, true, st);
        }
    }
    bar_arrive(bar, sync);
    if (!bar_wait(bar, &s_ok, sync)) return;
    // A wave that gives up leaves alone: the rest of its workgroup goes on, with what that wave would have staged missing, and may arrive here in full
    // number.  The flag was in memory before the wave was gone, and so before its workgroup could arrive without it.
    if (blockIdx.x == 0 && wave == 0 && !ld_coherent(a.bar.abort_flag)) {
        EntStat r; r.init();
        for (int i = lane; i < (int)gridDim.x * kFusedWaves; i += 64) {
            EntStat q;
            q.m = ld_coherent(&a.lm_part[i].m); q.Z = ld_coherent(&a.lm_part[i].Z);
            q.S = ld_coherent(&a.lm_part[i].S); q.idx = ld_coherent(&a.lm_part[i].idx);
            q.gs = -INFINITY; q.gidx = 0x7FFFFFFF;      // this kernel decodes greedily (the host keeps sampled runs off it)
            r.merge(q);
        }
        r = wave_merge(r);
        const float H = entropy_from(r, a.fin.unit);
        if (lane == 0) {
            lm_finalize_seq(a.fin, seq, r, H);
            a.fin.s.kvlen[m * MB + seq] = pos + 1;
        }
    }
}

}  // namespace ead

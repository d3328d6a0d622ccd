// Weight-streaming linear layers: Y[T, N] = X[T, K] * W[N, K]^T with fused prologues
// (RMSNorm) and epilogues (rotary + KV append, residual add, SwiGLU, entropy statistics).
//
// Two paths share the tiled weight layout and the epilogues:
//   k_linear_valu, k_linear_ring  plain FMAs for one or two token rows (and for fp32 weights); activations stay fp32,
//                  staged once per workgroup in LDS.
//   k_linear_mfma, k_linear_mfma_ls, k_lm_ls, k_linear_mfma_gemm, k_linear_mfma_tile (k_linear_mfma_wt: fallback)
//                  16x16x32 f16 products for three rows and more (batched decode, catch-up chunks, prompts);
//                  activations are half-precision tiles.  Which one takes a pass follows the matrix's shape and the
//                  pass's number of token blocks (launch_mfma, launch_lm).
// A workgroup owns 16-row blocks of W.  In k_linear_valu and k_linear_mfma its waves split K, so a wave reads contiguous
// streams of 1 KB (2-byte) tiles; partial sums meet in LDS and are added in wave order.  All sums are taken in an order that
// the matrix's shape and the number of token blocks fix: a row's result does not depend on what the other rows of
// its pass hold, but passes of another width class may add in another order.
#pragma once
#include "common.hpp"
#include "rules.hpp"

namespace ead {

struct EntPartial { float m, Z, S; int idx; float gs; int gidx; };

template <typename WT>
struct LinArgs {
    const WT *W;            // tiled weights, Np x K
    int Np, K;
    const int *count;       // device: number of activation rows this pass
    const int *rowmap;      // optional: activation row r reads x[rowmap[r]] (LM head), else x[r]
    const float *x;         // fp32 activations [*, ldx]        (VALU path)
    int ldx;
    const bf16_t *xp;       // half-precision activation tiles [K/32][ceil(rows/16)][64][8] (MFMA path; the element type only names the width)
    const float *gain;      // RMSNorm gain (VALU path prologue), null = no norm
    float eps;
    // outputs
    float *out;             // RES: residual stream [T, ldo] (+=); SWIGLU: h [T, ldo]; QKV: q [T, ldo]
    int ldo;
    const WT *res_embed;    // RES, optional: the residual is this embedding row instead of out (first layer)
    bf16_t *out_tiles;      // SWIGLU, optional: h as half-precision tiles for the next MFMA layer
    int tbs;                // token blocks of the pass, (count + 15) / 16: the stride of activation tiles (xp, out_tiles) along k
    // QKV
    WT *kcache, *vcache;    // this layer's cache, [seq][kv_head][max_seq][hd]
    WT *vtcache;            // optional second copy of V, transposed in tiles (vt_offset): the matrix-core attention contracts over keys
    const int *row_seq, *row_pos;
    const float2 *rope;     // [max_seq][hd/2] (cos, sin)
    int n_heads, n_kv_heads, hd, max_seq;
    // LOGITS
    EntPartial *partials;   // [rows][gridDim.x]
    float *logits;          // optional dump [rows][Np]
    // LOGITS with sampling: inverse temperature (0 = greedy), generator key, and where to find
    // the sequence of LM row t and its count of generated tokens
    float samp_inv_t; uint32_t samp_k0, samp_k1;
    const int *samp_seq, *samp_ngen;
    // MFMA path with K split over KS workgroups per row-block group
    int tb_base;            // k_linear_mfma_wt with split K, k_sk_merge, k_lm_ls: first token block of the sweep this launch takes
    int sweeps;             // without split K: > 1 = one workgroup per (row-block group, sweep of 128 rows; k_linear_mfma_gemm: 256); k_linear_mfma_tile: sweeps of a band
    int tile_sweeps;        // k_linear_mfma_tile, k_sk_merge<EPI, 0>: sweeps of 256 rows this launch takes, from token block tb_base on
    int KS;
    int once;               // k_linear_mfma_ls, k_lm_ls: weight tiles are requested non-temporally (tiles_once, lm_once)
    float *sk_part;         // [KS][groups][R][NT][256] partial sums
    int *sk_tickets;        // [groups] arrival counters, zero between launches
};

// ------------------------------------------------------------------------------------
// Epilogue for one output element: packed row p of token row t.  Called by 16-lane
// groups whose lanes hold consecutive packed rows, so the rotary / SwiGLU partner is
// the neighbouring lane.
// ------------------------------------------------------------------------------------
template <typename T> __device__ __forceinline__ void put(T *p, T v, bool coherent) {
    if (coherent) st_coherent(p, v); else *p = v;
}

// What an epilogue reads from memory for one output element.  It is fetched ahead (before
// the k loop of the FMA path, before the reduction of the MFMA path) so that the chain
// position -> rotary table, or the residual, is not waited for between two barriers.
struct EpiPre { float res; float2 cs; int pos, seq; };

// COH: outputs are handed to other workgroups inside the same kernel (fused decode).
template <typename WT, int EPI, bool COH = false>
__device__ __forceinline__ EpiPre epi_prefetch(const LinArgs<WT> &a, int p, int t, bool valid) {
    EpiPre e; e.res = 0.f; e.cs = make_float2(1.f, 0.f); e.pos = 0; e.seq = 0;
    if (!valid) return e;
    if constexpr (EPI == EPI_RES) {
        const float *dst = a.out + (size_t)t * a.ldo + p;
        e.res = a.res_embed ? to_f32(a.res_embed[p]) : (COH ? ld_coherent(dst) : *dst);
    } else if constexpr (EPI == EPI_QKV) {
        e.pos = a.row_pos[t]; e.seq = a.row_seq[t];
        const int hd = a.hd, NQ = a.n_heads * hd, NK = a.n_kv_heads * hd;
        if (p < NQ + NK) {
            const int pp = p < NQ ? p : p - NQ;
            e.cs = a.rope[(size_t)e.pos * (hd >> 1) + ((pp % hd) >> 1)];
        }
    } else if constexpr (EPI == EPI_LOGITS) {
        if (a.samp_inv_t > 0.f) { e.seq = a.samp_seq[t]; e.pos = a.samp_ngen[e.seq]; }
    }
    return e;
}

template <typename WT, int EPI, bool COH = false>
__device__ __forceinline__ void epilogue(const LinArgs<WT> &a, int p, int t, float v, bool valid,
                                         EntStat &st, const EpiPre &pre) {
    if constexpr (EPI == EPI_RES) {
        if (valid) put(a.out + (size_t)t * a.ldo + p, pre.res + v, COH);
    } else if constexpr (EPI == EPI_SWIGLU) {
        float other = __shfl_xor(v, 1, kWave);       // even lane: gate, odd lane: up
        if (valid && !(p & 1)) {
            float h = v / (1.f + __expf(-v)) * other;
            int i = p >> 1;
            if (a.out) put(a.out + (size_t)t * a.ldo + i, h, COH);
            if (a.out_tiles) {
                size_t off = act_tile_offset(t >> 4, i >> 5, a.tbs) + (size_t)(((t & 15) + 16 * ((i & 31) >> 3)) * 8 + (i & 7));
                a.out_tiles[off].u = f32_to_f16_sat(h);
            }
        }
    } else if constexpr (EPI == EPI_QKV) {
        float other = __shfl_xor(v, 1, kWave);
        if (!valid) return;
        const int hd = a.hd, NQ = a.n_heads * hd, NK = a.n_kv_heads * hd;
        const int pos = pre.pos;
        if (p < NQ + NK) {                            // rotary: lanes (2i, 2i+1) hold dims (i, i+hd/2)
            int pp = p < NQ ? p : p - NQ;
            int head = pp / hd, r = pp % hd, i = r >> 1, s = r & 1;
            const float2 cs = pre.cs;
            float res = s ? (other * cs.y + v * cs.x) : (v * cs.x - other * cs.y);
            int dim = i + s * (hd >> 1);
            if (p < NQ) put(a.out + (size_t)t * a.ldo + head * hd + dim, res, COH);
            else {
                size_t o = (((size_t)pre.seq * a.n_kv_heads + head) * a.max_seq + pos) * hd + dim;
                put(a.kcache + o, from_f32<WT>(res), COH);
            }
        } else {
            int pp = p - NQ - NK, head = pp / hd, dim = pp % hd;
            size_t o = (((size_t)pre.seq * a.n_kv_heads + head) * a.max_seq + pos) * hd + dim;
            put(a.vcache + o, from_f32<WT>(v), COH);
            if (a.vtcache) put(a.vtcache + ((size_t)pre.seq * a.n_kv_heads + head) * hd * a.max_seq + vt_offset(dim, pos, a.max_seq), from_f32<WT>(v), COH);
        }
    } else {                                          // EPI_LOGITS: fold the logit into (m, Z, S, argmax)
        if (!valid) return;
        if (a.logits) a.logits[(size_t)t * a.Np + p] = v;
        if (a.samp_inv_t > 0.f) {                     // perturbed score l/T + g; rows come in rising order
            const float sc = fmaf(v, a.samp_inv_t, gumbel_noise(a.samp_k0, a.samp_k1, pre.seq, pre.pos, p));
            if (sc > st.gs) { st.gs = sc; st.gidx = p; }
        }
        if (st.Z == 0.f) { st.m = v; st.Z = 1.f; st.S = 0.f; st.idx = p; }
        else if (v > st.m) {
            float d = st.m - v, e = __expf(d);
            st.S = e * (st.S + d * st.Z); st.Z = st.Z * e + 1.f; st.m = v; st.idx = p;
        } else {
            float d = v - st.m, e = __expf(d);
            st.S += e * d; st.Z += e;
        }
    }
}

// After a workgroup has seen all its row blocks: merge the 16 lanes of each token row
// and store one partial per (row, workgroup).
template <typename WT, bool COH = false>
__device__ __forceinline__ void logits_flush(const LinArgs<WT> &a, int t, bool valid, EntStat st) {
#pragma unroll
    for (int o = 8; o > 0; o >>= 1) {
        EntStat q;
        q.m = __shfl_xor(st.m, o, kWave); q.Z = __shfl_xor(st.Z, o, kWave);
        q.S = __shfl_xor(st.S, o, kWave); q.idx = __shfl_xor(st.idx, o, kWave);
        q.gs = __shfl_xor(st.gs, o, kWave); q.gidx = __shfl_xor(st.gidx, o, kWave);
        st.merge(q);
    }
    if (valid && (threadIdx.x & 15) == 0) {
        EntPartial *d = a.partials + (size_t)t * gridDim.x + blockIdx.x;
        put(&d->m, st.m, COH); put(&d->Z, st.Z, COH); put(&d->S, st.S, COH); put(&d->idx, st.idx, COH);
        put(&d->gs, st.gs, COH); put(&d->gidx, st.gidx, COH);
    }
}

// ------------------------------------------------------------------------------------
// FMA path.  TC token rows per pass over the weights; NW waves split K.
// dynamic LDS: xs[TC][K] floats, then red[NW][TC][16] floats.
// A wave's tiles are fetched U at a time, one group ahead of the arithmetic, and the
// first group of the next row block (or of the kernel, before the activations are even
// staged) is already in flight while partial sums are being reduced.
// ------------------------------------------------------------------------------------
template <typename WT, int U>
__device__ __forceinline__ void load_group(Vec8<WT> (&w)[U], const WT *wp, int kc, int kc1) {
#pragma unroll
    for (int u = 0; u < U; ++u) {
        if (kc + u < kc1) w[u].load_stream(wp + (size_t)u * 512);
        else w[u].zero();
    }
}

template <typename WT, int TC, int NW, int EPI>
__global__ __launch_bounds__(NW * 64) void k_linear_valu(LinArgs<WT> a) {
    constexpr int U = sizeof(WT) == 2 ? 8 : 4;
    extern __shared__ float smem[];
    const int K = a.K, KC = K >> 5, NB = a.Np >> 4;
    float *xs = smem;
    float *red = smem + (size_t)TC * K;
    __shared__ float s_ss[NW];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int g = lane >> 4;
    const int T = *a.count;
    const int kc0 = (wave * KC) / NW, kc1 = ((wave + 1) * KC) / NW;

    Vec8<WT> cur[U];
    if ((int)blockIdx.x < NB) load_group<WT, U>(cur, a.W + tile_offset(blockIdx.x, kc0, KC) + lane * 8, kc0, kc1);

    const int tstep = TC * (int)gridDim.y;                // blockIdx.y: one of the groups of TC rows of a pass
    for (int t0 = (int)blockIdx.y * TC; t0 < T; t0 += tstep) {
        // ---- stage (and normalise) TC activation rows ----
        for (int tc = 0; tc < TC; ++tc) {
            const int t = t0 + tc;
            float *xr = xs + (size_t)tc * K;
            if (t < T) {
                const float *src = a.x + (size_t)(a.rowmap ? a.rowmap[t] : t) * a.ldx;
                float ss = 0.f;
                for (int k = tid * 4; k < K; k += NW * 64 * 4) {
                    float4 v = *reinterpret_cast<const float4 *>(src + k);
                    *reinterpret_cast<float4 *>(xr + k) = v;
                    ss += v.x * v.x + v.y * v.y + v.z * v.z + v.w * v.w;
                }
                if (a.gain) {
                    ss = wave_sum(ss);
                    if (lane == 0) s_ss[wave] = ss;
                    __syncthreads();
                    float tot = 0.f;
#pragma unroll
                    for (int w = 0; w < NW; ++w) tot += s_ss[w];
                    const float inv = 1.0f / sqrtf(tot / (float)K + a.eps);
                    for (int k = tid * 4; k < K; k += NW * 64 * 4) {
                        float4 v = *reinterpret_cast<float4 *>(xr + k);
                        float4 gn = *reinterpret_cast<const float4 *>(a.gain + k);
                        v.x *= inv * gn.x; v.y *= inv * gn.y; v.z *= inv * gn.z; v.w *= inv * gn.w;
                        *reinterpret_cast<float4 *>(xr + k) = v;
                    }
                    __syncthreads();
                }
            } else {
                for (int k = tid * 4; k < K; k += NW * 64 * 4)
                    *reinterpret_cast<float4 *>(xr + k) = make_float4(0, 0, 0, 0);
            }
        }
        __syncthreads();

        EntStat st; st.init();
        for (int rb = blockIdx.x; rb < NB; rb += gridDim.x) {
            float acc[TC];
#pragma unroll
            for (int tc = 0; tc < TC; ++tc) acc[tc] = 0.f;
            const WT *wp = a.W + tile_offset(rb, kc0, KC) + lane * 8;
            const float *xq = xs + g * 8;
            // what the epilogue reads is requested now and arrives during the k loop
            const EpiPre pre = epi_prefetch<WT, EPI>(a, rb * 16 + (tid & 15), t0 + (tid >> 4), tid < 16 * TC && t0 + (tid >> 4) < T);
            for (int kc = kc0; kc < kc1; kc += U) {
                // fetch one group ahead: the rest of this row block, else the head of the next
                // one (the next pass over the same block when more token rows follow)
                Vec8<WT> nxt[U];
                if (kc + U < kc1) load_group<WT, U>(nxt, wp + (size_t)U * 512, kc + U, kc1);
                else {
                    int nrb = rb + gridDim.x;
                    if (nrb >= NB && t0 + tstep < T) nrb = blockIdx.x;
                    if (nrb < NB) load_group<WT, U>(nxt, a.W + tile_offset(nrb, kc0, KC) + lane * 8, kc0, kc1);
                    else {
#pragma unroll
                        for (int u = 0; u < U; ++u) nxt[u].zero();
                    }
                }
#pragma unroll
                for (int u = 0; u < U; ++u) {
                    float wf[8];
                    cur[u].unpack_w(wf);
                    const int kk = min(kc + u, kc1 - 1);          // tiles past the end are zero
#pragma unroll
                    for (int tc = 0; tc < TC; ++tc) {
                        const float4 x0 = *reinterpret_cast<const float4 *>(xq + (size_t)tc * K + kk * 32);
                        const float4 x1 = *reinterpret_cast<const float4 *>(xq + (size_t)tc * K + kk * 32 + 4);
                        acc[tc] += wf[0] * x0.x + wf[1] * x0.y + wf[2] * x0.z + wf[3] * x0.w
                                 + wf[4] * x1.x + wf[5] * x1.y + wf[6] * x1.z + wf[7] * x1.w;
                    }
                }
#pragma unroll
                for (int u = 0; u < U; ++u) cur[u] = nxt[u];
                wp += (size_t)U * 512;
            }
#pragma unroll
            for (int tc = 0; tc < TC; ++tc) {
                float v = acc[tc];
                v += __shfl_xor(v, 16, kWave);
                v += __shfl_xor(v, 32, kWave);
                if (lane < 16) red[(wave * TC + tc) * 16 + lane] = v;
            }
            __syncthreads();
            if (tid < 16 * TC) {
                const int tc = tid >> 4, j = tid & 15;
                float v = 0.f;
#pragma unroll
                for (int w = 0; w < NW; ++w) v += red[(w * TC + tc) * 16 + j];
                epilogue<WT, EPI>(a, rb * 16 + j, t0 + tc, v, t0 + tc < T, st, pre);
            }
            __syncthreads();
        }
        if constexpr (EPI == EPI_LOGITS) {
            if (tid < 16 * TC) logits_flush<WT>(a, t0 + (tid >> 4), t0 + (tid >> 4) < T, st);
        }
    }
}

// ------------------------------------------------------------------------------------
// One row of a bf16 model, where this is the faster form (launch_valu): QKV and gate/up of a short K, long residual projections, the LM head.
// A wave needs only its own slice of the activations, so it requests the slice (XV vectors a lane) and its gains before its first weights,
// leaves their product in LDS for itself alone, and the RMSNorm factor, which needs the whole row, is applied to the finished sums: the wait
// for the row's sum of squares between two barriers goes.  Weights run through a ring of D groups of U tiles across the row blocks
// of the workgroup, one barrier per row block.  (The activations must not be loaded in a loop: the compiler then waits for the
// weights requested after them, which cost 1 us a launch.)  k_linear_valu -> this, us: QKV 3072 x 2048 6.0 -> 5.7, 2048 x 1536 6.1 -> 5.2;
// down 2048 x 8192 9.9 -> 9.5, 3072 x 8192 12.2 -> 11.7; LM head 128256 x 2048 87 -> 82, 128256 x 3072 123 -> 116.
// What bounds it: the weight stream, and in launches of some 10 MB the latencies.
// ------------------------------------------------------------------------------------
template <int NW, int EPI, int U, int D, int XV>
__global__ __launch_bounds__(NW * 64) void k_linear_ring(LinArgs<bf16_t> a) {
    extern __shared__ float smem[];
    const int K = a.K, KC = K >> 5, NB = a.Np >> 4;
    float *xs = smem;                                      // [K]: a wave's slice is written and read by the wave alone
    float *zero = smem + K;                                // [32]: what tiles past a slice's end are multiplied with
    float *red = zero + 32;                                // [2][NW][16]
    __shared__ float s_ss[NW];
    const int tid = threadIdx.x, lane = tid & 63, g8 = (lane >> 4) * 8;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const bool valid = tid < 16 && *a.count > 0;
    const int kc0 = (wave * KC) / NW, kc1 = ((wave + 1) * KC) / NW;
    const int ng = max(1, (kc1 - kc0 + U - 1) / U);        // groups of U tiles per row block
    const int nrb = (NB - 1 - (int)blockIdx.x) / (int)gridDim.x + 1, total = nrb * ng;      // the grid is at most NB

    const int ks = kc0 * 32 + lane * 4, ke = kc1 * 32;
    const float *src = a.x + (size_t)(a.rowmap ? a.rowmap[0] : 0) * a.ldx;
    float4 xv[XV], gv[XV];
#pragma unroll
    for (int i = 0; i < XV; ++i) xv[i] = *reinterpret_cast<const float4 *>(src + min(ks + 256 * i, K - 4));
    if (a.gain) {
#pragma unroll
        for (int i = 0; i < XV; ++i) gv[i] = *reinterpret_cast<const float4 *>(a.gain + min(ks + 256 * i, K - 4));
    }
    __builtin_amdgcn_sched_barrier(0);
    Vec8<bf16_t> w[D][U];
    int nj = 0, ngi = 0;                                   // next group to request; past the end the last row block's again, never used
    const bf16_t *wbase = a.W + lane * 8;
    auto request = [&](int s) __attribute__((always_inline)) {
        const bf16_t *p = wbase + tile_offset((int)blockIdx.x + nj * (int)gridDim.x, 0, KC);
#pragma unroll
        for (int u = 0; u < U; ++u) w[s][u].load_stream(p + (size_t)min(kc0 + ngi * U + u, max(kc1 - 1, 0)) * 512);
        if (++ngi == ng) { ngi = 0; if (nj + 1 < nrb) ++nj; }
    };
#pragma unroll
    for (int s = 0; s < D; ++s) { request(s); __builtin_amdgcn_sched_barrier(0); }
    float ss = 0.f;
#pragma unroll
    for (int i = 0; i < XV; ++i) {
        const int k = ks + 256 * i;
        if (k < ke) {
            float4 v = xv[i];
            if (a.gain) {
                ss += v.x * v.x + v.y * v.y + v.z * v.z + v.w * v.w;
                v.x *= gv[i].x; v.y *= gv[i].y; v.z *= gv[i].z; v.w *= gv[i].w;
            }
            *reinterpret_cast<float4 *>(xs + k) = v;
        }
    }
    if (a.gain) { ss = wave_sum(ss); if (lane == 0) s_ss[wave] = ss; }
    if (tid < 32) zero[tid] = 0.f;
    __syncthreads();

    EntStat st; st.init();
    EpiPre pre;
    float acc = 0.f, inv = 1.f;
    int g = 0, rb = blockIdx.x, par = 0;
    for (int i0 = 0; i0 < total; i0 += D) {
#pragma unroll
        for (int s = 0; s < D; ++s) {
            if (i0 + s < total) {                          // uniform over the wave; every wave meets the others once per row block
                if (g == 0) {
                    pre = epi_prefetch<bf16_t, EPI>(a, rb * 16 + (tid & 15), 0, valid);
                    acc = 0.f;
                }
                const int kb = kc0 + g * U;
#pragma unroll
                for (int u = 0; u < U; ++u) {
                    float wf[8];
                    w[s][u].unpack_w(wf);
                    const float *xp = kb + u < kc1 ? xs + (kb + u) * 32 + g8 : zero + g8;
                    const float4 x0 = *reinterpret_cast<const float4 *>(xp), x1 = *reinterpret_cast<const float4 *>(xp + 4);
                    acc += wf[0] * x0.x + wf[1] * x0.y + wf[2] * x0.z + wf[3] * x0.w
                         + wf[4] * x1.x + wf[5] * x1.y + wf[6] * x1.z + wf[7] * x1.w;
                }
                __builtin_amdgcn_sched_barrier(0);
                request(s);
                __builtin_amdgcn_sched_barrier(0);
                if (++g == ng) {
                    float *rd = red + (size_t)par * NW * 16;      // two sets: the next row block's sums may be written while these are read
                    acc += __shfl_xor(acc, 16, kWave);
                    acc += __shfl_xor(acc, 32, kWave);
                    if (lane < 16) rd[wave * 16 + lane] = acc;
                    __syncthreads();
                    if (tid < 16) {
                        if (a.gain && rb == (int)blockIdx.x) {
                            float tot = 0.f;
#pragma unroll
                            for (int q = 0; q < NW; ++q) tot += s_ss[q];
                            inv = 1.0f / sqrtf(tot / (float)K + a.eps);
                        }
                        float v = 0.f;
#pragma unroll
                        for (int q = 0; q < NW; ++q) v += rd[q * 16 + tid];
                        epilogue<bf16_t, EPI>(a, rb * 16 + tid, 0, v * inv, valid, st, pre);
                    }
                    par ^= 1; g = 0; rb += gridDim.x;
                }
            }
        }
    }
    if constexpr (EPI == EPI_LOGITS) {
        if (tid < 16) logits_flush<bf16_t>(a, 0, valid, st);
    }
}

// ------------------------------------------------------------------------------------
// MFMA path (bf16).  A workgroup of NW waves owns R row blocks of W at a time and NT
// blocks of 16 token rows; its waves split K.  For every k tile a wave fetches R weight
// tiles (the stream from memory) and the NT activation tiles (from cache), so an activation
// tile is fetched once for R weight tiles: with R = 1 the activation fetches alone would
// take most of a compute unit's load-issue cycles at a batch of 32.  Fetches run a ring of
// D k tiles ahead of the matrix cores; the ring slots are register arrays indexed by the
// unrolled loop, so nothing is copied and a wave keeps D * R KB of weights in flight.
// Both operands are IEEE halves (common.hpp): the weights keep their bf16 values exactly, the
// activations are rounded to 11 significant bits (with bf16-rounded activations the logits of a
// full-depth model drift well past their tolerance; a bf16 hi + lo pair, which this path used
// first, costs two products and twice the activation traffic per weight tile).  Within a wave every
// output element accumulates its k tiles in ascending order, whatever R, NT and D are, and the waves' sums
// are added in wave order.  Matrices with few row blocks are also split along K over KS workgroups per
// group (SK), whose sums meet in memory and are added in order of the slabs.  NW and KS follow the
// matrix's shape and the number of token blocks (launch_narrow), so they change the order of a row's sums only
// from one width class of passes to another.
// ------------------------------------------------------------------------------------
template <int NW, int R, int NT, int D, int EPI, bool SK = false>
__global__ __launch_bounds__(NW * 64) void k_linear_mfma(LinArgs<bf16_t> a) {
    constexpr int NE = (NT * 256 + NW * 64 - 1) / (NW * 64);     // epilogue elements per thread and row block
    __shared__ float red[NW][NT][64][4];
    __shared__ int s_ticket;
    const int K = a.K, KC = K >> 5, NB = a.Np >> 4, NG = (NB + R - 1) / R;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);     // uniform: keeps the k range in scalar registers
    const int T = *a.count;
    const int TB = (T + 15) >> 4;
    if (TB == 0) return;
    // SK: workgroup (g, ks) takes slab ks of K for row-block group g, and TB <= NT gridDim.y
    const int KS = SK ? a.KS : 1;
    const int ks = SK ? (int)blockIdx.x % KS : 0;
    const int slab0 = (ks * KC) / KS, slab1 = ((ks + 1) * KC) / KS;
    const int kc0 = slab0 + (wave * (slab1 - slab0)) / NW, kc1 = slab0 + ((wave + 1) * (slab1 - slab0)) / NW;
    const int nsteps = kc1 - kc0;
    float *part = SK ? a.sk_part + (size_t)blockIdx.y * KS * NG * R * NT * 256 : nullptr;      // this sweep's partial sums and counters
    int *tickets = SK ? a.sk_tickets + (size_t)blockIdx.y * NG : nullptr;
    // this thread's i-th element in the epilogue: number e of the sweep's NT blocks of 16 x 16, token block e >> 8, token column
    // (e >> 4) & 15 (the same for all i from four waves up), weight row j
    const int j = tid & 15;
    auto elem = [&](int i) __attribute__((always_inline)) { return tid + i * NW * 64; };
    auto column = [&](int i) __attribute__((always_inline)) { return (elem(i) >> 4) & 15; };

    // blockIdx.y: one of the pass's sweeps of NT token blocks
    for (int tb0 = (int)blockIdx.y * NT; tb0 < TB; tb0 += NT * (int)gridDim.y) {
        EntStat st[NE];
#pragma unroll
        for (int i = 0; i < NE; ++i) st[i].init();
        const bf16_t *xh[NT];
#pragma unroll
        for (int b = 0; b < NT; ++b)         // token blocks past the end repeat the last one; their results are dropped
            xh[b] = a.xp + act_tile_offset(min(tb0 + b, TB - 1), kc0, TB) + lane * 8;
        const int gstep = SK ? NG : (int)gridDim.x;
        for (int g = SK ? (int)blockIdx.x / KS : (int)blockIdx.x; g < NG; g += gstep) {
            f32x4_t acc[R][NT];
            const bf16_t *wp[R];
#pragma unroll
            for (int r = 0; r < R; ++r) {
#pragma unroll
                for (int b = 0; b < NT; ++b) acc[r][b] = f32x4_t{0.f, 0.f, 0.f, 0.f};
                wp[r] = a.W + tile_offset(min(g * R + r, NB - 1), kc0, KC) + lane * 8;
            }
            Vec8<bf16_t> wa[D][R], xa[D][NT];
            // k tile i of the wave's range into ring slot s; past the end the last tile is
            // fetched again (from cache) and not used, so no branch surrounds the loads
            auto issue = [&](int s, int i) __attribute__((always_inline)) {
                const size_t off = (size_t)max(min(i, nsteps - 1), 0) * 512, xoff = off * TB;
#pragma unroll
                for (int r = 0; r < R; ++r) wa[s][r].load_stream(wp[r] + off);
#pragma unroll
                for (int b = 0; b < NT; ++b) xa[s][b].load(xh[b] + xoff);
            };
#pragma unroll
            for (int s = 0; s < D; ++s) {    // in slot order: the waits below count on it
                issue(s, s);
                __builtin_amdgcn_sched_barrier(0);
            }
            for (int i0 = 0; i0 < nsteps; i0 += D) {
#pragma unroll
                for (int s = 0; s < D; ++s) {
                    if (i0 + s < nsteps) {
#pragma unroll
                        for (int r = 0; r < R; ++r) {
#pragma unroll
                            for (int b = 0; b < NT; ++b)
                                acc[r][b] = __builtin_amdgcn_mfma_f32_16x16x32_f16(
                                    __builtin_bit_cast(f16x8_t, wa[s][r].raw), __builtin_bit_cast(f16x8_t, xa[s][b].raw), acc[r][b], 0, 0, 0);
                        }
                    }
                    // the slot is refilled only after its last reader has been issued: moved any
                    // earlier, the refill needs registers of its own and a copy that waits for it
                    __builtin_amdgcn_sched_barrier(0);
                    issue(s, i0 + s + D);
                    __builtin_amdgcn_sched_barrier(0);
                }
            }
            // what the epilogues read is requested for all row blocks at once
            EpiPre pre[R][NE];
            if (!SK) {
#pragma unroll
                for (int r = 0; r < R; ++r)
#pragma unroll
                    for (int i = 0; i < NE; ++i) {
                        const int b = elem(i) >> 8, t = (tb0 + b) * 16 + column(i), rb = g * R + r;
                        pre[r][i] = epi_prefetch<bf16_t, EPI>(a, rb * 16 + j, t, b < NT && rb < NB && tb0 + b < TB && t < T);
                    }
            }
            // the waves' partial sums meet in LDS, one row block at a time.  D holds weight
            // row j of token column c in lane c + 16*(j/4), register j%4.
#pragma unroll
            for (int r = 0; r < R; ++r) {
#pragma unroll
                for (int b = 0; b < NT; ++b)
                    *reinterpret_cast<float4 *>(&red[wave][b][lane][0]) = make_float4(acc[r][b][0], acc[r][b][1], acc[r][b][2], acc[r][b][3]);
                __syncthreads();
                const int rb = g * R + r;
#pragma unroll
                for (int i = 0; i < NE; ++i) {
                    const int b = elem(i) >> 8;          // uniform within a wave
                    if (b < NT) {
                        float v = 0.f;
#pragma unroll
                        for (int w = 0; w < NW; ++w) v += red[w][b][column(i) + 16 * (j >> 2)][j & 3];
                        const int t = (tb0 + b) * 16 + column(i);
                        if constexpr (SK)
                            st_coherent(part + ((((size_t)ks * NG + g) * R + r) * NT + b) * 256 + (elem(i) & 255), v);
                        else
                            epilogue<bf16_t, EPI>(a, rb * 16 + j, t, v, rb < NB && tb0 + b < TB && t < T, st[i], pre[r][i]);
                    }
                }
                __syncthreads();
            }
            if constexpr (SK) {
                // the slab's sums are written through to memory; the workgroup that arrives last
                // for this group adds the slabs in order and runs the epilogue.  The counter
                // is left at zero for the next launch.
                wait_stores();
                __syncthreads();
                if (tid == 0) s_ticket = __hip_atomic_fetch_add(tickets + g, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                __syncthreads();
                if (s_ticket == KS - 1) {
                    if (tid == 0) st_coherent(tickets + g, 0);
                    // all slabs of all the group's elements, and what the epilogues read, are
                    // requested before the first sum
#pragma unroll
                    for (int r = 0; r < R; ++r)
#pragma unroll
                        for (int i = 0; i < NE; ++i) {
                            const int b = elem(i) >> 8, t = (tb0 + b) * 16 + column(i), rb = g * R + r;
                            pre[r][i] = epi_prefetch<bf16_t, EPI>(a, rb * 16 + j, t, b < NT && rb < NB && tb0 + b < TB && t < T);
                        }
                    float pv[R][NE][kSplitKMax];
#pragma unroll
                    for (int r = 0; r < R; ++r)
#pragma unroll
                        for (int i = 0; i < NE; ++i) {
                            const int b = min(elem(i) >> 8, NT - 1);
#pragma unroll
                            for (int q = 0; q < kSplitKMax; ++q)
                                pv[r][i][q] = ld_coherent(part + ((((size_t)min(q, KS - 1) * NG + g) * R + r) * NT + b) * 256 + (elem(i) & 255));
                        }
#pragma unroll
                    for (int r = 0; r < R; ++r) {
                        const int rb = g * R + r;
#pragma unroll
                        for (int i = 0; i < NE; ++i) {
                            const int b = elem(i) >> 8;
                            if (b < NT) {
                                float v = 0.f;
#pragma unroll
                                for (int q = 0; q < kSplitKMax; ++q) v += q < KS ? pv[r][i][q] : 0.f;
                                const int t = (tb0 + b) * 16 + column(i);
                                epilogue<bf16_t, EPI>(a, rb * 16 + j, t, v, rb < NB && tb0 + b < TB && t < T, st[i], pre[r][i]);
                            }
                        }
                    }
                }
            }
        }
        if constexpr (EPI == EPI_LOGITS) {
#pragma unroll
            for (int i = 0; i < NE; ++i) {
                const int b = elem(i) >> 8;
                if (b < NT) {
                    const int t = (tb0 + b) * 16 + column(i);
                    logits_flush<bf16_t>(a, t, tb0 + b < TB && t < T, st[i]);
                }
            }
        }
    }
}

// ------------------------------------------------------------------------------------
// The epilogues on the matrix cores' own output layout: lane L of a 16 x 16 block holds weight rows p .. p + 3
// (p = first row of the block + 4 (L / 16)) of token L % 16, so both halves of a rotary pair or of a gate/up pair are
// in the lane and a residual or a rotary table entry is one 16-byte load: no exchange between lanes.
// ------------------------------------------------------------------------------------
struct QuadTok { int pos, seq; };                      // EPI_QKV: of the lane's token

template <int EPI>
__device__ __forceinline__ QuadTok quad_token(const LinArgs<bf16_t> &a, int t, bool ok) {
    QuadTok k{0, 0};
    if constexpr (EPI == EPI_QKV) { if (ok) { k.pos = a.row_pos[t]; k.seq = a.row_seq[t]; } }
    return k;
}
template <int EPI>
__device__ __forceinline__ float4 quad_prefetch(const LinArgs<bf16_t> &a, int p, int t, bool ok, const QuadTok &k) {
    float4 r = make_float4(0.f, 0.f, 0.f, 0.f);
    if (!ok) return r;
    if constexpr (EPI == EPI_RES) r = *reinterpret_cast<const float4 *>(a.out + (size_t)t * a.ldo + p);
    else if constexpr (EPI == EPI_QKV) {
        const int NQ = a.n_heads * a.hd, NK = a.n_kv_heads * a.hd;
        if (p < NQ + NK) r = *reinterpret_cast<const float4 *>(a.rope + (size_t)k.pos * (a.hd >> 1) + (((p < NQ ? p : p - NQ) & (a.hd - 1)) >> 1));
    }
    return r;
}
template <int EPI>
__device__ __forceinline__ void quad_epilogue(const LinArgs<bf16_t> &a, int p, int t, const f32x4_t &v, bool ok, const QuadTok &k, const float4 &pre) {
    if (!ok) return;
    if constexpr (EPI == EPI_RES) {
        *reinterpret_cast<float4 *>(a.out + (size_t)t * a.ldo + p) = make_float4(pre.x + v[0], pre.y + v[1], pre.z + v[2], pre.w + v[3]);
    } else if constexpr (EPI == EPI_SWIGLU) {
        const int i = p >> 1;                          // even: the two outputs are neighbours in a tile
        const float h0 = v[0] / (1.f + __expf(-v[0])) * v[1], h1 = v[2] / (1.f + __expf(-v[2])) * v[3];
        const size_t off = act_tile_offset(t >> 4, i >> 5, a.tbs) + (size_t)(((t & 15) + 16 * ((i & 31) >> 3)) * 8 + (i & 7));
        *reinterpret_cast<uint32_t *>(a.out_tiles + off) = (uint32_t)f32_to_f16_sat(h0) | ((uint32_t)f32_to_f16_sat(h1) << 16);
    } else {
        const int hd = a.hd, sh = 31 - __clz(hd), NQ = a.n_heads * hd, NK = a.n_kv_heads * hd;      // hd: 32, 64 or 128
        if (p < NQ + NK) {                             // rows (2i, 2i + 1) hold dims (i, i + hd/2): here pairs i and i + 1
            const int pp = p < NQ ? p : p - NQ, head = pp >> sh, i = (pp & (hd - 1)) >> 1;
            const float lo0 = v[0] * pre.x - v[1] * pre.y, hi0 = v[0] * pre.y + v[1] * pre.x;
            const float lo1 = v[2] * pre.z - v[3] * pre.w, hi1 = v[2] * pre.w + v[3] * pre.z;
            if (p < NQ) {
                float *q = a.out + (size_t)t * a.ldo + head * hd + i;
                *reinterpret_cast<float2 *>(q) = make_float2(lo0, lo1);
                *reinterpret_cast<float2 *>(q + (hd >> 1)) = make_float2(hi0, hi1);
            } else {
                bf16_t *c = a.kcache + (((size_t)k.seq * a.n_kv_heads + head) * a.max_seq + k.pos) * hd + i;
                *reinterpret_cast<uint32_t *>(c) = (uint32_t)f32_to_bf16(lo0) | ((uint32_t)f32_to_bf16(lo1) << 16);
                *reinterpret_cast<uint32_t *>(c + (hd >> 1)) = (uint32_t)f32_to_bf16(hi0) | ((uint32_t)f32_to_bf16(hi1) << 16);
            }
        } else {
            const int pp = p - NQ - NK, head = pp >> sh, dim = pp & (hd - 1);
            const size_t row = (size_t)k.seq * a.n_kv_heads + head;
            const uint16_t b0 = f32_to_bf16(v[0]), b1 = f32_to_bf16(v[1]), b2 = f32_to_bf16(v[2]), b3 = f32_to_bf16(v[3]);
            *reinterpret_cast<uint2 *>(a.vcache + (row * a.max_seq + k.pos) * hd + dim) = make_uint2((uint32_t)b0 | ((uint32_t)b1 << 16), (uint32_t)b2 | ((uint32_t)b3 << 16));
            if (a.vtcache) {
                bf16_t *vt = a.vtcache + row * hd * a.max_seq + vt_offset(dim, k.pos, a.max_seq);      // dims are 32 elements apart
                vt[0].u = b0; vt[32].u = b1; vt[64].u = b2; vt[96].u = b3;
            }
        }
    }
}

// All blocks of a wave that share a token block: first row block rb of `n` (those below NB count), token block tb.
template <int EPI, int N>
__device__ __forceinline__ void quad_blocks(const LinArgs<bf16_t> &a, const f32x4_t *const (&v)[N], int rb, int NB, int tb, int T, int lane, bool ok) {
    const int t = tb * 16 + (lane & 15), p = rb * 16 + 4 * (lane >> 4);
    ok = ok && t < T;
    const QuadTok k = quad_token<EPI>(a, t, ok);
    float4 pre[N];
#pragma unroll
    for (int j = 0; j < N; ++j) pre[j] = quad_prefetch<EPI>(a, p + 16 * j, t, ok && rb + j < NB, k);
#pragma unroll
    for (int j = 0; j < N; ++j) quad_epilogue<EPI>(a, p + 16 * j, t, *v[j], ok && rb + j < NB, k, pre[j]);
}

constexpr int kWideTok = 8;          // token blocks (of 16 rows) per sweep

// Passes of more than 32 rows: a workgroup takes RG (8; 7 where that fills the compute units better)
// row blocks and 16 NW TPW token rows per sweep; each of its NW waves owns TPW (1 or 2) token blocks
// and all RG row blocks.  NW follows the pass: four waves for up to 64 rows (TPW = 1) and for sweeps of
// 128 (TPW = 2), five to eight waves with one block each for 65-128 rows, so that a pass of 72 rows
// multiplies and fetches five blocks' worth, not eight.  A wave's activation fragments (of its
// blocks) come straight from memory in the matrix cores' operand layout and are never
// shared; the step's RG weight tiles, of which each wave fetches at most two, go through LDS (8 KB read per
// wave and step; sharing the activation tiles instead, with a row-block pair per wave, reads 16 KB
// and is no faster).  SK: workgroup (g, ks) takes slab ks of K for group g (one sweep only: TB <= NW TPW)
// and leaves its sums in memory for k_sk_merge.
template <int DA, int EPI, bool SK = false, int TPW = 2, int RG = 8, int NW = 4>
__global__ __launch_bounds__(NW * 64) void k_linear_mfma_wt(LinArgs<bf16_t> a) {
    static_assert(RG >= 5 && RG <= 8 && NW >= 4 && NW <= 8, "each wave fetches at most two of the workgroup's weight tiles");
    constexpr int NT = NW * TPW;                       // token blocks per sweep (TPW per wave); RG row blocks per workgroup
    constexpr int WPT = (RG + NW - 1) / NW;            // weight tiles a wave fetches per step: tiles wave, wave + NW
    __shared__ __attribute__((aligned(16))) bf16_t s_w[2][8][512];
    const int K = a.K, KCfull = K >> 5, NB = a.Np >> 4, NG = (NB + RG - 1) / RG;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int T = *a.count;
    const int TB = (T + 15) >> 4;
    if (TB == 0) return;
    const int KS = SK ? a.KS : 1;
    int g = SK ? (int)blockIdx.x / KS : (int)blockIdx.x, tb_first = SK ? a.tb_base : 0;
    const int ks = SK ? (int)blockIdx.x % KS : 0;
    const bool one_sweep = SK || a.sweeps > 1;
    if (!SK && a.sweeps > 1) {
        // workgroup id -> (group, sweep) such that the sweeps of one group run at about the same time on
        // one XCD (id % 8) and find the group's weight tiles in its L2
        const int q = (int)blockIdx.x >> 3, r = (int)blockIdx.x & 7;
        g = (q / a.sweeps) * 8 + r; tb_first = (q % a.sweeps) * NT;
        if (g >= NG || tb_first >= TB) return;
    }
    const int kbase = (ks * KCfull) / KS, KC = ((ks + 1) * KCfull) / KS - kbase;     // this workgroup's k tiles

    for (int tb0 = tb_first; tb0 < TB; tb0 += one_sweep ? TB : NT) {
        f32x4_t acc[RG][TPW];
        const bf16_t *wp[WPT], *bp[TPW];
#pragma unroll
        for (int j = 0; j < RG; ++j)
#pragma unroll
            for (int q = 0; q < TPW; ++q) acc[j][q] = f32x4_t{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int q = 0; q < WPT; ++q)      // a wave whose second tile would lie past RG fetches the last tile again and drops it
            wp[q] = a.W + tile_offset(min(g * RG + min(wave + q * NW, RG - 1), NB - 1), kbase, KCfull) + lane * 8;
#pragma unroll
        for (int q = 0; q < TPW; ++q) {
            const int blk = min(tb0 + wave * TPW + q, TB - 1);
            bp[q] = a.xp + act_tile_offset(blk, kbase, TB) + lane * 8;
        }
        Vec8<bf16_t> wa[DA][WPT], ba[DA][TPW];
        auto issue = [&](int s, int i) __attribute__((always_inline)) {
            const size_t off = (size_t)min(i, KC - 1) * 512;
#pragma unroll
            for (int q = 0; q < WPT; ++q) wa[s][q].load_stream(wp[q] + off);
#pragma unroll
            for (int q = 0; q < TPW; ++q) ba[s][q].load(bp[q] + off * TB);
        };
#pragma unroll
        for (int s = 0; s < DA; ++s) {
            issue(s, s);
            __builtin_amdgcn_sched_barrier(0);
        }
        for (int i0 = 0; i0 < KC; i0 += DA) {
#pragma unroll
            for (int s = 0; s < DA; ++s) {
                const int i = i0 + s;
                if (i < KC) {                                  // uniform over the workgroup
                    bf16_t (*buf)[512] = s_w[i & 1];
#pragma unroll
                    for (int q = 0; q < WPT; ++q)
                        if (wave + q * NW < RG)                // uniform over the wave
                            *reinterpret_cast<u32x4_t *>(&buf[wave + q * NW][lane * 8]) = wa[s][q].raw;
                    __syncthreads();
                    u32x4_t fw[RG];
#pragma unroll
                    for (int j = 0; j < RG; ++j) fw[j] = *reinterpret_cast<const u32x4_t *>(&buf[j][lane * 8]);
                    __builtin_amdgcn_sched_barrier(0);
                    // neighbouring products go to different accumulators: none waits for another's result
#pragma unroll
                    for (int j = 0; j < RG; ++j)
#pragma unroll
                        for (int q = 0; q < TPW; ++q)
                            acc[j][q] = __builtin_amdgcn_mfma_f32_16x16x32_f16(
                                __builtin_bit_cast(f16x8_t, fw[j]), __builtin_bit_cast(f16x8_t, ba[s][q].raw), acc[j][q], 0, 0, 0);
                }
                __builtin_amdgcn_sched_barrier(0);
                issue(s, i + DA);
                __builtin_amdgcn_sched_barrier(0);
            }
        }
        if constexpr (!SK) {
#pragma unroll
            for (int q = 0; q < TPW; ++q) {
                const f32x4_t *v[RG];
#pragma unroll
                for (int j = 0; j < RG; ++j) v[j] = &acc[j][q];
                const int tb = tb0 + wave * TPW + q;
                quad_blocks<EPI, RG>(a, v, g * RG, NB, tb, T, lane, tb < TB);
            }
        } else {
            const size_t slab = (size_t)NG * RG * NT * 256;                // floats per slab
#pragma unroll
            for (int j = 0; j < RG; ++j)
#pragma unroll
                for (int q = 0; q < TPW; ++q) {
                    const int rb = g * RG + j, b = wave * TPW + q;
                    if (rb < NB && tb0 + b < TB) {
                        float *dst = a.sk_part + (size_t)ks * slab + ((size_t)rb * NT + b) * 256 + lane;
                        st_coherent(dst, acc[j][q][0]); st_coherent(dst + 64, acc[j][q][1]);
                        st_coherent(dst + 128, acc[j][q][2]); st_coherent(dst + 192, acc[j][q][3]);
                    }
                }
        }
        __syncthreads();                 // the weight buffers are reused by the next sweep
    }
}

// ------------------------------------------------------------------------------------
// Passes of 33-128 rows, and the 128-row sweeps of longer passes, with the weight stream decoupled from the arithmetic.
// In k_linear_mfma_wt every wave fetches weights (from HBM), fetches activations (from L2) and
// multiplies; a wave's loads complete in order, so its slow weight fetches and its fast
// activation fetches wait for each other, and what a wave can keep in flight is bounded by its
// registers (about 40 KB of weights per compute unit, which at 2-3 us of loaded memory latency
// is 3.5-5 TB/s over the chip).  Here a workgroup has two extra waves that do nothing but fetch
// weight tiles, straight into LDS (the load writes LDS itself: no registers, no ds_write), kDepth - 1
// k steps ahead: up to 104 KB of weights in flight per compute unit.  The NW multiplying waves
// (one token block each, all RG row blocks, as in k_linear_mfma_wt with TPW = 1) fetch only
// their activation fragments, and read a step's weight fragments from LDS while they multiply the step
// before (all waves read all RG tiles: the LDS reads of a step take as long as its products).
// One workgroup barrier per k step hands a step's tiles over; the slot a step leaves is refilled
// right after the next barrier, when every wave has read it.
// The order of the sums of an output element is that of k_linear_mfma_wt.
// ------------------------------------------------------------------------------------
constexpr int kLsDepth = 14;                 // k steps of weight tiles LDS holds (8 KB each)
constexpr int kLsProducers = 2;              // fetching waves; each has 4 (kLsDepth - 1) loads of 1 KB in flight (the counter holds 63)
constexpr size_t kLsLdsBytes = (size_t)kLsDepth * 8 * 1024;
// The ring of a kernel with rg row blocks per workgroup: up to four take slots of half the size, and twice as many steps fit.
constexpr int ls_slot_tiles(int rg) { return rg <= 4 ? 4 : 8; }
constexpr int ls_depth(int rg) { return kLsDepth * 8 / ls_slot_tiles(rg); }

// a.once picks one of two fetching loops.  (A fetching wave that chose at every request made passes of several sweeps 7-20 % slower.)
template <int EPI, bool SK, int NW, int RG>
__global__ __launch_bounds__((NW + kLsProducers) * 64) void k_linear_mfma_ls(LinArgs<bf16_t> a) {
    static_assert(RG >= 3 && RG <= 8 && NW >= 1 && NW <= 8, "two producer waves share a step's four or eight tile slots");
    constexpr int SLOT = ls_slot_tiles(RG), PL = SLOT / 2, DEPTH = ls_depth(RG);      // tiles per slot, loads per producer wave and step, k steps in the ring
    static_assert(PL * (DEPTH - 1) <= 63, "the load counter holds 63");
    constexpr int DA = 6;                              // ring of activation fragments per multiplying wave
    extern __shared__ __attribute__((aligned(16))) unsigned char ls_smem[];
    bf16_t (*s_w)[SLOT][512] = reinterpret_cast<bf16_t (*)[SLOT][512]>(ls_smem);                 // [DEPTH][SLOT][512]
    const int K = a.K, KCfull = K >> 5, NB = a.Np >> 4, NG = (NB + RG - 1) / RG;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int T = *a.count;
    const int TB = (T + 15) >> 4;
    if (TB == 0) return;
    const int KS = SK ? a.KS : 1;
    int g = SK ? (int)blockIdx.x / KS : (int)blockIdx.x, tb0 = SK ? a.tb_base : 0;
    const int ks = SK ? (int)blockIdx.x % KS : 0;
    if (!SK && a.sweeps > 1) {
        // passes of more than 128 rows: one workgroup per (group, 128-row sweep), numbered as in
        // k_linear_mfma_wt so that the sweeps of one group run at about the same time on one XCD
        const int q = (int)blockIdx.x >> 3, r = (int)blockIdx.x & 7;
        g = (q / a.sweeps) * 8 + r; tb0 = (q % a.sweeps) * NW;
        if (g >= NG || tb0 >= TB) return;
    }
    const int kbase = (ks * KCfull) / KS, KC = ((ks + 1) * KCfull) / KS - kbase;     // this workgroup's k tiles
    auto kstep = [&](int j) __attribute__((always_inline)) { return min(j, KC - 1); };      // past the end: the last step again

    if (wave >= NW) {
        // ---- fetching wave p: tile slots p, p + 2, .. of every step (slots past RG repeat the last row block) ----
        const int p = wave - NW;
        const bf16_t *wp[PL];
#pragma unroll
        for (int q = 0; q < PL; ++q)
            wp[q] = a.W + tile_offset(min(g * RG + min(p + 2 * q, RG - 1), NB - 1), kbase, KCfull) + lane * 8;
        auto fetch = [&](auto once) __attribute__((always_inline)) {
            auto issue = [&](int j) __attribute__((always_inline)) {      // step j (past the end: the last step again, never read)
                const size_t off = (size_t)kstep(j) * 512;
                bf16_t (*slot)[512] = s_w[j % DEPTH];
#pragma unroll
                for (int q = 0; q < PL; ++q) request_tile_at<decltype(once)::value>(wp[q] + off, &slot[p + 2 * q][0]);
            };
            for (int j = 0; j < DEPTH - 1; ++j) issue(j);
            asm volatile("s_waitcnt vmcnt(%0)" ::"n"(PL * (DEPTH - 2)) : "memory");      // step 0 has landed
            __builtin_amdgcn_s_barrier();                 // the bare barrier: this wave has nothing else to wait for
            for (int i = 0; i < KC; ++i) {
                // the multiplying waves read a step's tiles one step ahead of using them: step i + 1 has to
                // have landed; steps i + 2 .. i + DEPTH - 2 may still be on their way
                asm volatile("s_waitcnt vmcnt(%0)" ::"n"(PL * (DEPTH - 3)) : "memory");
                __builtin_amdgcn_s_barrier();
                issue(i + DEPTH - 1);                  // into the slot of step i - 1, which every wave has read by now
            }
        };
        if (a.once) fetch(std::true_type{}); else fetch(std::false_type{});
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");    // nothing may land in LDS after the workgroup has gone
        return;
    }

    // ---- multiplying wave: token block tb0 + wave, all RG row blocks ----
    f32x4_t acc[RG];
#pragma unroll
    for (int j = 0; j < RG; ++j) acc[j] = f32x4_t{0.f, 0.f, 0.f, 0.f};
    const int blk = min(tb0 + wave, TB - 1);
    const bf16_t *bp = a.xp + act_tile_offset(blk, kbase, TB) + lane * 8;
    Vec8<bf16_t> ba[DA];
    auto issue = [&](int s, int i) __attribute__((always_inline)) {
        ba[s].load(bp + (size_t)kstep(i) * 512 * TB);
    };
#pragma unroll
    for (int s = 0; s < DA; ++s) {
        issue(s, s);
        __builtin_amdgcn_sched_barrier(0);
    }
    // weight fragments of step i + 1 are read from LDS while step i is multiplied (two register sets)
    static_assert(DA % 2 == 0, "the two fragment sets alternate with the unrolled ring slots");
    u32x4_t fw[2][RG];
    __syncthreads();
#pragma unroll
    for (int j = 0; j < RG; ++j) fw[0][j] = *reinterpret_cast<const u32x4_t *>(&s_w[0][j][lane * 8]);
    for (int i0 = 0; i0 < KC; i0 += DA) {
#pragma unroll
        for (int s = 0; s < DA; ++s) {
            const int i = i0 + s;
            if (i < KC) {                                  // uniform over the workgroup
                __syncthreads();
                bf16_t (*nxt)[512] = s_w[(i + 1) % DEPTH];      // past the last step: a slot nobody uses
#pragma unroll
                for (int j = 0; j < RG; ++j) fw[(s + 1) & 1][j] = *reinterpret_cast<const u32x4_t *>(&nxt[j][lane * 8]);
                __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                for (int j = 0; j < RG; ++j)
                    acc[j] = __builtin_amdgcn_mfma_f32_16x16x32_f16(
                        __builtin_bit_cast(f16x8_t, fw[s & 1][j]), __builtin_bit_cast(f16x8_t, ba[s].raw), acc[j], 0, 0, 0);
            }
            __builtin_amdgcn_sched_barrier(0);
            issue(s, i + DA);
            __builtin_amdgcn_sched_barrier(0);
        }
    }
    if constexpr (!SK) {
        const f32x4_t *v[RG];
#pragma unroll
        for (int j = 0; j < RG; ++j) v[j] = &acc[j];
        quad_blocks<EPI, RG>(a, v, g * RG, NB, tb0 + wave, T, lane, tb0 + wave < TB);
    } else {
        const size_t slab = (size_t)NG * RG * NW * 256;                // floats per slab
#pragma unroll
        for (int j = 0; j < RG; ++j) {
            const int rb = g * RG + j, b = wave;
            if (rb < NB && tb0 + b < TB) {
                float *dst = a.sk_part + (size_t)ks * slab + ((size_t)rb * NW + b) * 256 + lane;
                st_coherent(dst, acc[j][0]); st_coherent(dst + 64, acc[j][1]);
                st_coherent(dst + 128, acc[j][2]); st_coherent(dst + 192, acc[j][3]);
            }
        }
    }
}

// ------------------------------------------------------------------------------------
// The LM head of passes of several rows: the weight stream of k_linear_mfma_ls, one workgroup per compute unit that
// walks its share of the row blocks (ranges of equal length, eight blocks at a time) without the stream ever
// stopping -- the fetching waves run 13 k steps ahead across the groups of row blocks, so the ring fills while the
// multiplying waves fold a group's logits into the statistics.  A multiplying wave owns one token block; a lane
// holds 4 consecutive vocabulary entries x 8 row blocks of one token, takes their maximum first and moves its sums
// once per group, and keeps its statistics in registers to the end: no exchange between waves, one partial per
// (token, workgroup).  A perturbed score's noise comes four to a generator call, since a lane's entries are
// exactly the four words of one counter.
// What bounds it: the weight stream from memory (every byte once).
// ------------------------------------------------------------------------------------
constexpr int kLmRows = 8;                            // row blocks per group
constexpr size_t kLmLdsBytes = (size_t)kLsDepth * kLmRows * 1024;

// the 4 x kLmRows logits a lane holds after a group: first vocabulary entry p0 + 16 j of row block j (`have` of them valid)
__device__ __forceinline__ void lm_fold(const LinArgs<bf16_t> &a, const f32x4_t (&acc)[kLmRows], int p0, int have, int t, bool valid,
                                        int seq, int tok, EntStat &st) {
    if (!valid) return;
    if (a.logits) {
#pragma unroll
        for (int j = 0; j < kLmRows; ++j)
            if (j < have) *reinterpret_cast<float4 *>(a.logits + (size_t)t * a.Np + p0 + 16 * j) = make_float4(acc[j][0], acc[j][1], acc[j][2], acc[j][3]);
    }
    if (a.samp_inv_t > 0.f) {
#pragma unroll
        for (int j = 0; j < kLmRows; ++j) {
            if (j >= have) continue;
            const int p = p0 + 16 * j;                // a multiple of 4: the four entries share one counter
            const Philox4 r = philox4x32_10((uint32_t)p >> 2, (uint32_t)tok, (uint32_t)seq, 0u, a.samp_k0, a.samp_k1);
            const uint32_t w[4] = {r.x, r.y, r.z, r.w};
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const float sc = fmaf(acc[j][e], a.samp_inv_t, gumbel_of(w[e]));
                if (sc > st.gs) { st.gs = sc; st.gidx = p + e; }        // entries come in rising order
            }
        }
    }
    float mx = -INFINITY;
#pragma unroll
    for (int j = 0; j < kLmRows; ++j)
        if (j < have) mx = fmaxf(mx, fmaxf(fmaxf(acc[j][0], acc[j][1]), fmaxf(acc[j][2], acc[j][3])));
    if (st.Z == 0.f || mx > st.m) {
        int idx = p0;                                 // of a group of NaN alone: its first entry
#pragma unroll
        for (int j = kLmRows - 1; j >= 0; --j)
#pragma unroll
            for (int e = 3; e >= 0; --e) if (j < have && acc[j][e] == mx) idx = p0 + 16 * j + e;
        if (st.Z != 0.f) {
            const float d = st.m - mx, x = __expf(d);
            st.S = x * (st.S + d * st.Z); st.Z *= x;
        }
        st.m = mx; st.idx = idx;
    }
#pragma unroll
    for (int j = 0; j < kLmRows; ++j)
        if (j < have) {
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const float d = acc[j][e] - st.m, x = __expf(d);
                st.S += x * d; st.Z += x;
            }
        }
}

template <int NW>
__global__ __launch_bounds__((NW + kLsProducers) * 64) void k_lm_ls(LinArgs<bf16_t> a) {
    static_assert(NW >= 1 && NW <= 8 && kLmRows == 8, "a producer wave fetches four of the step's eight tile slots");
    constexpr int DA = 6;                              // ring of activation fragments per multiplying wave
    extern __shared__ __attribute__((aligned(16))) unsigned char ls_smem[];
    bf16_t (*s_w)[kLmRows][512] = reinterpret_cast<bf16_t (*)[kLmRows][512]>(ls_smem);        // [kLsDepth]
    const int KC = a.K >> 5, NB = a.Np >> 4;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int T = *a.count;
    const int TB = (T + 15) >> 4;
    const int rb0 = (int)(((long)blockIdx.x * NB) / gridDim.x), rb1 = (int)(((long)(blockIdx.x + 1) * NB) / gridDim.x);
    if (a.tb_base >= TB || rb0 >= rb1) return;          // the grid is at most NB, so every range holds a row block
    const int groups = (rb1 - rb0 + kLmRows - 1) / kLmRows, total = groups * KC;      // k steps of the whole range

    if (wave >= NW) {
        // ---- fetching wave p: tile slots p, p + 2, p + 4, p + 6 of every step (slots past the range repeat its last row block) ----
        const int p = wave - NW;
        const bf16_t *wp[4];
        int g = 0, k = 0, slot = 0;                    // next step to request
        auto point = [&]() __attribute__((always_inline)) {
#pragma unroll
            for (int q = 0; q < 4; ++q) wp[q] = a.W + tile_offset(min(rb0 + g * kLmRows + p + 2 * q, rb1 - 1), 0, KC) + lane * 8;
        };
        point();
        auto fetch = [&](auto once) __attribute__((always_inline)) {
            auto issue = [&]() __attribute__((always_inline)) {      // past the range: its last step again, never read
                const size_t off = (size_t)k * 512;
#pragma unroll
                for (int q = 0; q < 4; ++q) request_tile_at<decltype(once)::value>(wp[q] + off, &s_w[slot][p + 2 * q][0]);
                slot = slot + 1 == kLsDepth ? 0 : slot + 1;
                if (k + 1 < KC) ++k;
                else if (g + 1 < groups) { k = 0; ++g; point(); }
            };
            for (int j = 0; j < kLsDepth - 1; ++j) issue();
            asm volatile("s_waitcnt vmcnt(%0)" ::"n"(4 * (kLsDepth - 2)) : "memory");      // step 0 has landed
            __builtin_amdgcn_s_barrier();
            for (int i = 0; i < total; ++i) {
                asm volatile("s_waitcnt vmcnt(%0)" ::"n"(4 * (kLsDepth - 3)) : "memory");  // step i + 1 has landed
                __builtin_amdgcn_s_barrier();
                issue();                               // into the slot of step i - 1, which every wave has read by now
            }
        };
        if (a.once) fetch(std::true_type{}); else fetch(std::false_type{});
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");    // nothing may land in LDS after the workgroup has gone
        return;
    }

    // ---- multiplying wave: token block a.tb_base + wave, the range's row blocks in groups of eight ----
    const int tb = a.tb_base + wave, t = tb * 16 + (lane & 15);
    const bool valid = tb < TB && t < T;
    int seq = 0, tok = 0;
    if (a.samp_inv_t > 0.f && valid) { seq = a.samp_seq[t]; tok = a.samp_ngen[seq]; }
    const bf16_t *bp = a.xp + act_tile_offset(min(tb, TB - 1), 0, TB) + lane * 8;
    Vec8<bf16_t> ba[DA];
    auto issue = [&](int s, int k) __attribute__((always_inline)) { ba[s].load(bp + (size_t)min(k, KC - 1) * 512 * TB); };
#pragma unroll
    for (int s = 0; s < DA; ++s) {
        issue(s, s);
        __builtin_amdgcn_sched_barrier(0);
    }
    EntStat st; st.init();
    static_assert(DA % 2 == 0, "the two fragment sets alternate with the unrolled ring slots");
    u32x4_t fw[2][kLmRows];
    __syncthreads();
#pragma unroll
    for (int j = 0; j < kLmRows; ++j) fw[0][j] = *reinterpret_cast<const u32x4_t *>(&s_w[0][j][lane * 8]);
    int slot = 0;                                      // of the step being multiplied
    for (int g = 0; g < groups; ++g) {
        f32x4_t acc[kLmRows];
#pragma unroll
        for (int j = 0; j < kLmRows; ++j) acc[j] = f32x4_t{0.f, 0.f, 0.f, 0.f};
        for (int i0 = 0; i0 < KC; i0 += DA) {
#pragma unroll
            for (int s = 0; s < DA; ++s) {
                const int i = i0 + s;
                if (i < KC) {                          // uniform over the workgroup
                    __syncthreads();
                    slot = slot + 1 == kLsDepth ? 0 : slot + 1;      // past the last step: a slot nobody uses
#pragma unroll
                    for (int j = 0; j < kLmRows; ++j) fw[(s + 1) & 1][j] = *reinterpret_cast<const u32x4_t *>(&s_w[slot][j][lane * 8]);
                    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                    for (int j = 0; j < kLmRows; ++j)
                        acc[j] = __builtin_amdgcn_mfma_f32_16x16x32_f16(
                            __builtin_bit_cast(f16x8_t, fw[s & 1][j]), __builtin_bit_cast(f16x8_t, ba[s].raw), acc[j], 0, 0, 0);
                }
                __builtin_amdgcn_sched_barrier(0);
                issue(s, i + DA);
                __builtin_amdgcn_sched_barrier(0);
            }
        }
        // the next group starts again at activation fragment 0 and at the even fragment set; what it needs is
        // requested before this group's logits are folded
#pragma unroll
        for (int s = 0; s < DA; ++s) issue(s, s);
        if (KC & 1) {
#pragma unroll
            for (int j = 0; j < kLmRows; ++j) fw[0][j] = fw[1][j];
        }
        const int first = rb0 + g * kLmRows;
        lm_fold(a, acc, first * 16 + 4 * (lane >> 4), min(kLmRows, rb1 - first), t, valid, seq, tok, st);
    }
    // the four lanes of a token
#pragma unroll
    for (int o = 16; o < 64; o <<= 1) {
        EntStat q;
        q.m = __shfl_xor(st.m, o, kWave); q.Z = __shfl_xor(st.Z, o, kWave);
        q.S = __shfl_xor(st.S, o, kWave); q.idx = __shfl_xor(st.idx, o, kWave);
        q.gs = __shfl_xor(st.gs, o, kWave); q.gidx = __shfl_xor(st.gidx, o, kWave);
        st.merge(q);
    }
    if (valid && lane < 16) {
        EntPartial e; e.m = st.m; e.Z = st.Z; e.S = st.S; e.idx = st.idx; e.gs = st.gs; e.gidx = st.gidx;
        a.partials[(size_t)t * gridDim.x + blockIdx.x] = e;
    }
}

// ------------------------------------------------------------------------------------
// Passes of more than 128 rows (prompt prefill, scoring) through matrices whose 128 x 256 tiles fill the chip (the
// costs are compared in launch_mfma).  With 128 rows per workgroup every wave of k_linear_mfma_ls reads all of a step's weight tiles from LDS for one
// token block: 8 KB of LDS reads per 8 products, which is LDS-bound at half the matrix cores'
// rate, and every workgroup fetches its activation tiles itself.  Here a workgroup covers
// 8 row blocks x 16 token blocks (128 output rows x 256 token rows); its two fetching waves bring
// both the step's 8 weight tiles and its 16 activation tiles into LDS (24 KB per k step,
// kGemmDepth steps), and each of the eight multiplying waves owns 4 row blocks x 4 token blocks:
// 8 KB of LDS reads per 16 products.  Hand-over, slot reuse and the order of the sums of an
// output element (k tiles in ascending order, one accumulator) are those of k_linear_mfma_ls.
// ------------------------------------------------------------------------------------
constexpr int kGemmDepth = 6;                        // k steps of tiles LDS holds
constexpr int kGemmRows = 8, kGemmTok = 16;          // row blocks and token blocks per workgroup
constexpr int kGemmTiles = kGemmRows + kGemmTok;     // 1 KB tiles per k step; each fetching wave brings half of them
constexpr size_t kGemmLdsBytes = (size_t)kGemmDepth * kGemmTiles * 1024;

template <int EPI>
__global__ __launch_bounds__(640) void k_linear_mfma_gemm(LinArgs<bf16_t> a) {
    constexpr int PL = kGemmTiles / 2;                 // loads per fetching wave and k step
    static_assert(PL * (kGemmDepth - 1) <= 63, "the load counter holds 63");
    extern __shared__ __attribute__((aligned(16))) unsigned char ls_smem[];
    bf16_t (*s_w)[kGemmTiles][512] = reinterpret_cast<bf16_t (*)[kGemmTiles][512]>(ls_smem);    // [kGemmDepth]: weight tiles, then activation tiles
    const int KC = a.K >> 5, NB = a.Np >> 4, NG = (NB + kGemmRows - 1) / kGemmRows;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int T = *a.count;
    const int TB = (T + 15) >> 4;
    if (TB == 0) return;
    // workgroup id -> (group, sweep): the sweeps of one group run at about the same time on one XCD (id % 8)
    const int q = (int)blockIdx.x >> 3, r = (int)blockIdx.x & 7;
    const int g = (q / a.sweeps) * 8 + r, tb0 = (q % a.sweeps) * kGemmTok;
    if (g >= NG || tb0 >= TB) return;
    auto kstep = [&](int j) __attribute__((always_inline)) { return min(j, KC - 1); };      // past the end: the last step again

    if (wave >= 8) {
        // ---- fetching wave p: weight tiles p, p + 2, .. and activation tiles p, p + 2, .. of every step ----
        const int p = wave - 8;
        const bf16_t *wp[kGemmRows / 2], *xp[kGemmTok / 2];
#pragma unroll
        for (int j = 0; j < kGemmRows / 2; ++j) wp[j] = a.W + tile_offset(min(g * kGemmRows + p + 2 * j, NB - 1), 0, KC) + lane * 8;
#pragma unroll
        for (int j = 0; j < kGemmTok / 2; ++j) xp[j] = a.xp + act_tile_offset(min(tb0 + p + 2 * j, TB - 1), 0, TB) + lane * 8;
        auto issue = [&](int j) __attribute__((always_inline)) {      // step j (past the end: the last step again, never read)
            const size_t woff = (size_t)kstep(j) * 512, xoff = woff * TB;
            bf16_t (*slot)[512] = s_w[j % kGemmDepth];
#pragma unroll
            for (int i = 0; i < kGemmRows / 2; ++i)
                __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void *)(wp[i] + woff),
                                                 (__attribute__((address_space(3))) void *)&slot[p + 2 * i][0], 16, 0, 0);
#pragma unroll
            for (int i = 0; i < kGemmTok / 2; ++i)
                __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void *)(xp[i] + xoff),
                                                 (__attribute__((address_space(3))) void *)&slot[kGemmRows + p + 2 * i][0], 16, 0, 0);
        };
        for (int j = 0; j < kGemmDepth - 1; ++j) issue(j);
        asm volatile("s_waitcnt vmcnt(%0)" ::"n"(PL * (kGemmDepth - 2)) : "memory");      // step 0 has landed
        __builtin_amdgcn_s_barrier();
        for (int i = 0; i < KC; ++i) {
            asm volatile("s_waitcnt vmcnt(%0)" ::"n"(PL * (kGemmDepth - 3)) : "memory");  // step i + 1 has landed
            __builtin_amdgcn_s_barrier();
            issue(i + kGemmDepth - 1);                // into the slot of step i - 1, which every wave has read by now
        }
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");    // nothing may land in LDS after the workgroup has gone
        return;
    }

    // ---- multiplying wave: row blocks 4 wr .. + 3 of the group, token blocks 4 wt .. + 3 of the sweep ----
    const int wr = wave & 1, wt = wave >> 1;
    f32x4_t acc[4][4];
#pragma unroll
    for (int j = 0; j < 4; ++j)
#pragma unroll
        for (int b = 0; b < 4; ++b) acc[j][b] = f32x4_t{0.f, 0.f, 0.f, 0.f};
    u32x4_t fw[2][4], fx[2][4];                       // fragments of step i + 1 are read while step i is multiplied
    auto fetch = [&](int set, int slot) __attribute__((always_inline)) {
#pragma unroll
        for (int j = 0; j < 4; ++j) fw[set][j] = *reinterpret_cast<const u32x4_t *>(&s_w[slot][4 * wr + j][lane * 8]);
#pragma unroll
        for (int b = 0; b < 4; ++b) fx[set][b] = *reinterpret_cast<const u32x4_t *>(&s_w[slot][kGemmRows + 4 * wt + b][lane * 8]);
    };
    __syncthreads();
    fetch(0, 0);
    for (int i0 = 0; i0 < KC; i0 += 2) {
#pragma unroll
        for (int s = 0; s < 2; ++s) {
            const int i = i0 + s;
            if (i < KC) {                                  // uniform over the workgroup
                __syncthreads();
                fetch((s + 1) & 1, (i + 1) % kGemmDepth);  // past the last step: a slot nobody uses
                __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                for (int j = 0; j < 4; ++j)
#pragma unroll
                    for (int b = 0; b < 4; ++b)
                        acc[j][b] = __builtin_amdgcn_mfma_f32_16x16x32_f16(
                            __builtin_bit_cast(f16x8_t, fw[s][j]), __builtin_bit_cast(f16x8_t, fx[s][b]), acc[j][b], 0, 0, 0);
            }
            __builtin_amdgcn_sched_barrier(0);
        }
    }
#pragma unroll
    for (int b = 0; b < 4; ++b) {
        const f32x4_t *v[4] = {&acc[0][b], &acc[1][b], &acc[2][b], &acc[3][b]};
        const int tb = tb0 + 4 * wt + b;
        quad_blocks<EPI, 4>(a, v, g * kGemmRows + 4 * wr, NB, tb, T, lane, tb < TB);
    }
}

// ------------------------------------------------------------------------------------
// Long passes, 256 x 256 tiles: 16 row blocks x 16 token blocks per workgroup, eight waves of 8 x 4 blocks (128 accumulator
// registers; 12 KB of LDS reads per 32 products, where the 4 x 4 blocks of k_linear_mfma_gemm read 16 KB and the
// LDS port bounds them).  No separate fetching waves -- two waves per SIMD may use 256 registers each, three would not --
// so every wave requests four of the step's 32 tiles (16 of weights, 16 of activations, 32 KB) straight into a ring
// of five steps.  The requests are written in assembly: they have no output register, and the compiler, which would
// otherwise let every LDS read wait for all of them, is told by the counter waits here instead.
//
// Step i: wait until this wave's tiles of step i + 1 have landed, meet the other waves (theirs have, too, and all have
// read step i - 1), request step i + 4 into the slot of step i - 1, read the fragments of step i + 1, multiply step i.
// Every output element adds its k tiles in ascending order, as in the other kernels without a split of K.
//
// SK: a workgroup takes one of KS slabs of K of a tile and leaves its sums for k_sk_merge.  Serves the sweeps that a whole round of
// workgroups would serve half empty (tile_plan in rules.hpp).
// ------------------------------------------------------------------------------------
constexpr int kTileDepth = 5, kTileBlocks = 16;        // k steps in LDS; row blocks and token blocks per workgroup
constexpr size_t kTileLdsBytes = (size_t)kTileDepth * 2 * kTileBlocks * 1024;
constexpr int kTileBand = 6;                           // most sweeps that run side by side, see launch

// Which tile a workgroup takes: group of 16 row blocks, sweep of 256 tokens, slab of K (g < 0: none), of NG x SG x KS in a grid of those rounded up to a multiple of
// eight.  XCD id % 8 takes an eighth of all tiles, one behind the other: with every eighth group of row blocks instead, 108 groups x 14 sweeps were 196 tiles for
// the 32 units of one XCD and 182 for those of another, seven rounds where 189 are six.  The sweeps of a band of `bs` run side by side for one group after the
// other, so that what runs at a time on an XCD shares weights and activations in L2.
struct TileAt { int g, sweep, ks; };
__device__ __forceinline__ TileAt tile_at(int id, int NG, int SG, int KS, int bs) {
    const int total = NG * SG * KS, per = (total + 7) >> 3, unit = (id & 7) * per + (id >> 3);
    if ((id >> 3) >= per || unit >= total) return TileAt{-1, 0, 0};
    const int ks = unit % KS, tile = unit / KS;
    const int band = min(tile / (NG * bs), (SG - 1) / bs), in = tile - band * NG * bs, width = min(bs, SG - band * bs);
    return TileAt{in / width, band * bs + in % width, ks};
}

template <int EPI, bool SK = false>
__global__ __launch_bounds__(512, 2) void k_linear_mfma_tile(LinArgs<bf16_t> a) {
    constexpr int NWV = 8, WB = 4, PL = 4;             // waves; token blocks of a wave; its requests per step
    extern __shared__ __attribute__((aligned(16))) unsigned char ls_smem[];
    bf16_t (*s_w)[2 * kTileBlocks][512] = reinterpret_cast<bf16_t (*)[2 * kTileBlocks][512]>(ls_smem);       // [kTileDepth]: weight tiles, activation tiles
    const int KCfull = a.K >> 5, NB = a.Np >> 4, NG = (NB + kTileBlocks - 1) / kTileBlocks;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int T = *a.count;
    const int TB = (T + 15) >> 4;
    const int KS = SK ? a.KS : 1, SG = a.tile_sweeps;
    const TileAt at = tile_at((int)blockIdx.x, NG, SG, KS, a.sweeps);
    if (at.g < 0) return;
    const int g = at.g, ks = at.ks, tb0 = a.tb_base + at.sweep * kTileBlocks;
    if (tb0 >= TB) return;
    const int kbase = (ks * KCfull) / KS, KC = ((ks + 1) * KCfull) / KS - kbase;     // this workgroup's k tiles

    // this wave's four tiles of a step: weight tiles wave, wave + 8, activation tiles wave, wave + 8
    const bf16_t *src[PL];
#pragma unroll
    for (int j = 0; j < PL / 2; ++j) {
        src[j] = a.W + tile_offset(min(g * kTileBlocks + wave + NWV * j, NB - 1), kbase, KCfull);
        src[PL / 2 + j] = a.xp + act_tile_offset(min(tb0 + wave + NWV * j, TB - 1), kbase, TB);
    }
    const uint32_t lds0 = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) unsigned char *)ls_smem + (uint32_t)wave * 1024, voff = (uint32_t)lane * 16;
    const size_t xstep = (size_t)TB * 512;
    int next = 0, nslot = 0;                            // step to request next and its slot; past the end the last step again, never read
    auto request = [&]() __attribute__((always_inline)) {
        const uint32_t l = lds0 + (uint32_t)nslot * (2 * kTileBlocks * 1024);
#pragma unroll
        for (int j = 0; j < PL; ++j) request_tile(src[j], voff, l + (uint32_t)j * NWV * 1024);
        nslot = nslot + 1 == kTileDepth ? 0 : nslot + 1;
        if (++next < KC) {
#pragma unroll
            for (int j = 0; j < PL / 2; ++j) { src[j] += 512; src[PL / 2 + j] += xstep; }
        }
    };
    const int wr = wave & 1, wt = wave >> 1;            // row blocks 8 wr .. + 7 of the group, token blocks 4 wt .. + 3 of the sweep
    f32x4_t acc[8][WB];
#pragma unroll
    for (int j = 0; j < 8; ++j)
#pragma unroll
        for (int b = 0; b < WB; ++b) acc[j][b] = f32x4_t{0.f, 0.f, 0.f, 0.f};
    u32x4_t fw[2][8], fx[2][WB];
    auto fetch = [&](int set, int slot) __attribute__((always_inline)) {
#pragma unroll
        for (int b = 0; b < WB; ++b) fx[set][b] = *reinterpret_cast<const u32x4_t *>(&s_w[slot][kTileBlocks + WB * wt + b][lane * 8]);
#pragma unroll
        for (int j = 0; j < 8; ++j) fw[set][j] = *reinterpret_cast<const u32x4_t *>(&s_w[slot][8 * wr + j][lane * 8]);
    };
    for (int j = 0; j < kTileDepth - 1; ++j) request();
    asm volatile("s_waitcnt vmcnt(%0)" ::"n"(PL * (kTileDepth - 2)) : "memory");      // step 0 has landed
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
    fetch(0, 0);
    int slot = 0;
    for (int i0 = 0; i0 < KC; i0 += 2) {
#pragma unroll
        for (int s = 0; s < 2; ++s) {
            if (i0 + s < KC) {                          // uniform over the workgroup
                asm volatile("s_waitcnt vmcnt(%0)" ::"n"(PL * (kTileDepth - 3)) : "memory");
                // step i's fragments, requested a step ago, are here: said before the next ones are requested, or the
                // compiler waits for those as well before the first product
                __builtin_amdgcn_s_waitcnt(kWaitLdsReads);
                __builtin_amdgcn_s_barrier();
                request();
                slot = slot + 1 == kTileDepth ? 0 : slot + 1;
                fetch(s ^ 1, slot);                     // past the last step: a slot nobody uses
                __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                for (int j = 0; j < 8; ++j)
#pragma unroll
                    for (int b = 0; b < WB; ++b)
                        acc[j][b] = __builtin_amdgcn_mfma_f32_16x16x32_f16(
                            __builtin_bit_cast(f16x8_t, fw[s][j]), __builtin_bit_cast(f16x8_t, fx[s][b]), acc[j][b], 0, 0, 0);
                __builtin_amdgcn_sched_barrier(0);
            }
        }
    }
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");    // nothing may land in LDS after the workgroup has gone
    if constexpr (SK) {
        // this slab's sums, for k_sk_merge: blocks of 16 x 16 ordered [slab][row block][token block of the launch]
        const int NT = SG * kTileBlocks;
#pragma unroll
        for (int b = 0; b < WB; ++b) {
            const int tb = tb0 + WB * wt + b;
            if (tb < TB) {
#pragma unroll
                for (int j = 0; j < 8; ++j) {
                    const int rb = g * kTileBlocks + 8 * wr + j;
                    if (rb < NB) {
                        float *dst = a.sk_part + (((size_t)ks * NG * kTileBlocks + rb) * NT + (tb - a.tb_base)) * 256 + lane;
                        dst[0] = acc[j][b][0]; dst[64] = acc[j][b][1]; dst[128] = acc[j][b][2]; dst[192] = acc[j][b][3];
                    }
                }
            }
        }
        return;
    }
#pragma unroll
    for (int b = 0; b < WB; ++b) {
        const f32x4_t *v[8] = {&acc[0][b], &acc[1][b], &acc[2][b], &acc[3][b], &acc[4][b], &acc[5][b], &acc[6][b], &acc[7][b]};
        const int tb = tb0 + WB * wt + b;
        quad_blocks<EPI, 8>(a, v, g * kTileBlocks + 8 * wr, NB, tb, T, lane, tb < TB);
    }
}

// Sum of the K slabs that k_linear_mfma_wt<..., SK = true, TPW> (k_linear_mfma_tile<EPI, true>: NTB = 0) left in memory, in slab order, then
// the epilogue.  One wave per 16 x 16 block; grid = ceil(row blocks * NT / 4) workgroups, NT token blocks.
template <int EPI, int NTB = kWideTok>
__global__ __launch_bounds__(256) void k_sk_merge(LinArgs<bf16_t> a, int NGR /* row blocks incl. padding */) {
    const int NT = NTB ? NTB : a.tile_sweeps * kTileBlocks;
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int NB = a.Np >> 4, T = *a.count, TB = (T + 15) >> 4, KS = a.KS;
    const int blk = blockIdx.x * 4 + wave, rb = blk / NT, b = blk % NT;
    if (rb >= NB || a.tb_base + b >= TB) return;
    const size_t slab = (size_t)NGR * NT * 256;
    const float *src = a.sk_part + ((size_t)rb * NT + b) * 256 + lane;
    const int t = (a.tb_base + b) * 16 + (lane & 15), p = rb * 16 + 4 * (lane >> 4);
    const QuadTok k = quad_token<EPI>(a, t, t < T);
    const float4 pre = quad_prefetch<EPI>(a, p, t, t < T, k);
    float pv[kSplitKMax][4];
#pragma unroll
    for (int q = 0; q < kSplitKMax; ++q) {
        const float *sq = src + (size_t)min(q, KS - 1) * slab;
        pv[q][0] = sq[0]; pv[q][1] = sq[64]; pv[q][2] = sq[128]; pv[q][3] = sq[192];
    }
    f32x4_t d = f32x4_t{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int q = 0; q < kSplitKMax; ++q)
        if (q < KS) { d[0] += pv[q][0]; d[1] += pv[q][1]; d[2] += pv[q][2]; d[3] += pv[q][3]; }
    quad_epilogue<EPI>(a, p, t, d, t < T, k, pre);
}

// ------------------------------------------------------------------------------------
// fp32 activations -> half-precision activation tiles, through RMSNorm.  Rows past `rows` (padding of the last 16-row
// block) are zeroed.  Two launches a layer that do little else than be launched, so what counts is the chain of
// latencies: the row's length is known when the kernel is compiled, so every load is requested at once and nothing branches, and the number of
// rows comes with the launch (12 rows in a graph, us, an empty kernel taking 1.7: K = 896 2.9 -> 2.1, 2048 3.2 -> 2.3, 5120 4.0 ->
// 2.8; before, one kernel for all lengths with 15 predicated pieces, and the count read from the plan).
// ------------------------------------------------------------------------------------
struct PackArgs {
    const float *x; int ldx;
    int rows; const int *rowmap;         // rowmap, optional: row t is x[rowmap[t]]
    const float *gain; float eps;
    bf16_t *out; int K;
};

// pieces tid, tid + stride, .. (V of them) of row t, normalised, into their tiles; a piece past the row repeats its last one and is dropped
template <int V>
__device__ __forceinline__ void pack_load(const PackArgs &a, int t, int tid, int stride, float4 (&v)[V], float4 (&g)[V]) {
    const float *src = a.x + (size_t)(a.rowmap ? a.rowmap[t] : t) * a.ldx;
#pragma unroll
    for (int i = 0; i < V; ++i) v[i] = *reinterpret_cast<const float4 *>(src + min((tid + stride * i) * 4, a.K - 4));
#pragma unroll
    for (int i = 0; i < V; ++i) g[i] = *reinterpret_cast<const float4 *>(a.gain + min((tid + stride * i) * 4, a.K - 4));
}
template <int V>
__device__ __forceinline__ float pack_squares(const PackArgs &a, int tid, int stride, const float4 (&v)[V]) {
    float ss = 0.f;
#pragma unroll
    for (int i = 0; i < V; ++i) {
        const float q = v[i].x * v[i].x + v[i].y * v[i].y + v[i].z * v[i].z + v[i].w * v[i].w;
        ss += (tid + stride * i) * 4 < a.K ? q : 0.f;
    }
    return ss;
}
template <int V>
__device__ __forceinline__ void pack_store(const PackArgs &a, int t, int tid, int stride, float inv, const float4 (&v)[V], const float4 (&g)[V]) {
    const int TB = (a.rows + 15) >> 4;
    const bool real = t < a.rows;
#pragma unroll
    for (int i = 0; i < V; ++i) {
        const int k = (tid + stride * i) * 4;
        if (k < a.K) {
            const float f[4] = {v[i].x * (inv * g[i].x), v[i].y * (inv * g[i].y), v[i].z * (inv * g[i].z), v[i].w * (inv * g[i].w)};
            // four of the eight elements a lane of the consuming product holds: 8 bytes, side by side with the neighbouring thread's
            const size_t off = act_tile_offset(t >> 4, k >> 5, TB) + (size_t)(((t & 15) + 16 * ((k & 31) >> 3)) * 8 + (k & 7));
            uint2 r;
            r.x = real ? (uint32_t)f32_to_f16_sat(f[0]) | ((uint32_t)f32_to_f16_sat(f[1]) << 16) : 0u;
            r.y = real ? (uint32_t)f32_to_f16_sat(f[2]) | ((uint32_t)f32_to_f16_sat(f[3]) << 16) : 0u;
            *reinterpret_cast<uint2 *>(a.out + off) = r;
        }
    }
}

// A workgroup of NT threads per row: V pieces per thread, K <= 4 NT V.  Rows of more than 5120: eight waves (3 and 1024 rows of 8192, us: 3.1
// and 18.9; four waves and eight pieces 3.5 and 19.7; the kernel for all lengths 4.9 and 18.8; of 15360: 4.1 and 33.9, 4.5 and 35.5, 6.9 and 34.0).
template <int V, int NT = 256>
__global__ __launch_bounds__(NT) void k_pack_act(PackArgs a) {
    __shared__ float s_ss[NT / 64];
    const int t = blockIdx.x, tid = threadIdx.x;
    float4 v[V], g[V];
    pack_load<V>(a, min(t, a.rows - 1), tid, NT, v, g);
    const float ss = wave_sum(pack_squares<V>(a, tid, NT, v));
    if ((tid & 63) == 0) s_ss[tid >> 6] = ss;
    __syncthreads();
    float tot = 0.f;
#pragma unroll
    for (int w = 0; w < NT / 64; ++w) tot += s_ss[w];
    const float inv = 1.0f / sqrtf(tot / (float)a.K + a.eps);
    pack_store<V>(a, t, tid, NT, inv, v, g);
}

// Long passes: a wave per row, four rows per workgroup, V pieces per lane, K <= 256 V: nothing to wait for between waves (1024 rows,
// us: K = 896 5.8 -> 2.7, 2048 7.6 -> 3.7, 5120 12.9 -> 7.7; at 96 rows a workgroup per row is the faster: K = 5120 3.4 against 4.3).
template <int V>
__global__ __launch_bounds__(256) void k_pack_rows(PackArgs a) {
    const int t = blockIdx.x * 4 + (int)(threadIdx.x >> 6), lane = threadIdx.x & 63;
    float4 v[V], g[V];
    pack_load<V>(a, min(t, a.rows - 1), lane, 64, v, g);
    const float inv = 1.0f / sqrtf(wave_sum(pack_squares<V>(a, lane, 64, v)) / (float)a.K + a.eps);
    pack_store<V>(a, t, lane, 64, inv, v, g);
}

}  // namespace ead

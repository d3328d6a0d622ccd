// Rules of dispatch that need nothing but sizes: plain host functions.
#pragma once
#include <algorithm>
#include <cstddef>

namespace ead {

enum Epilogue { EPI_QKV = 0, EPI_RES = 1, EPI_SWIGLU = 2, EPI_LOGITS = 3 };      // what becomes of a linear layer's sums

// the persistent kernels of one row: waves (of the streamed one: that multiply) and threads of a workgroup, most splits of a KV head's keys
constexpr int kFusedWaves = 8, kFusedThreads = kFusedWaves * 64, kFusedMaxSplits = 8;

constexpr int kEntMaxChunks = 64;                       // most pieces a row of logits is cut into

// The split of a row into work items depends on (rows, V) alone, so a step's result does not depend on
// how many steps share a launch, nor on which entry point asked for it.  Long chunks (up to 8 vectors
// per thread) amortise the per-workgroup merge; shorter ones only when the rows of one step would
// otherwise give too few workgroups to fill the chip: one per compute unit (with two, rows are cut finer than it pays: both launches
// of 97 x 50264 float32 14.2 -> 12.5 us in a graph, 128 x 32000 12.0 -> 9.7, 40 x 128256 bf16 10.2 -> 9.3; nothing slower at 1-200 rows x 4096-128256).
inline void entropy_split(int rows, int V, int *chunks_out, int *per_out) {
    const int nvec = V / 8;
    int chunks = std::max(1, (nvec + 2047) / 2048);
    while ((long)chunks * rows < 256 && chunks < kEntMaxChunks && nvec / (chunks * 2) >= 256) chunks *= 2;
    int per = (std::max(nvec, 1) + chunks - 1) / chunks;
    while (per > 8 * 256) { ++chunks; per = (nvec + chunks - 1) / chunks; }
    *chunks_out = chunks; *per_out = per;
}

// Whether ead_entropy_argmax merges a row's chunks in the launch that computes them.  The call is bound by the host where a
// second launch is saved (10.3 -> 7.5 us), as long as the chain behind a row's last chunk stays hidden: its chunks
// arrive one after another at a word of their row, and rows share the words' cache lines, so the time grows about
// as rows x chunks^2 (us in one launch against two: 4 chunks x 128 rows 8.1 / 10.4, 8 x 64 9.2 / 10.2, 16 x 16 9.0 / 10.3, 40 x 3
// 8.9 / 10.3, 64 x 1 7.7 / 10.4; but 16 x 24 11.1 / 10.2, 40 x 6 11.8 / 10.3, 40 x 13 14.8 / 10.6, 64 x 4 12.1 / 10.3).  A workgroup that takes one item
// after another waits for the chain each time (2000 rows of one chunk: 16.8 / 15.2; 800: 10.4 / 10.4).  Above 4 MB the kernel
// itself is the longer part.
inline bool entropy_folds(int rows, int chunks, size_t bytes) {
    return bytes <= ((size_t)4 << 20) && (long)rows * chunks <= 600 && (long)rows * chunks * chunks <= 4800;
}

// The same for larger calls: up to 32 MB, at most 600 chunks, eight a row, the second launch still is the longer part (us in one launch
// against two, float32: 97 x 50264 10.5 / 12.6, 128 x 50264 10.1 / 12.6, 64 x 128256 11.1 / 12.5, 256 x 32000 10.8 / 12.6; bf16: 64 x 128256 10.0 /
// 12.5, 128 x 50264 10.1 / 12.5; but 776 chunks, 97 x 128256, 13.4 / 12.5).  That is a call's time where the host bounds it (the Python binding: 64 x 128256 bf16 10.6 a
// call, two launches 13.4); to a caller whose host takes less than the kernel, the chain of eight arrivals costs up to 0.9 (9.3 / 8.4), of four nothing.
inline bool entropy_folds_large(int rows, int chunks, size_t bytes) {
    return bytes <= ((size_t)32 << 20) && (long)rows * chunks <= 600 && chunks <= 8;
}

// Pieces a row is given to workgroups in by k_entropy_rows (1: a workgroup takes whole rows, 2048 vectors at a time), by rows
// and vocabulary alone, so that a step's result does not depend on how many steps share a launch.  One or two rows of
// more than three times 2048 vectors: eight pieces (more where 2048 vectors ask for it), which keep 16 steps of two rows
// at about one workgroup per compute unit
// (2 rows x 151936: one step 19.5 -> 9.9 us, 64 steps 90 -> 58; 37 pieces: 10.4 and 105).  Shorter rows are through
// before a piece's partial and counter are (1 x 32000: whole 7.3 and 45 us, in pieces 9.6 and 50).  From more rows on the pieces'
// merges cost more over 16 steps than the fuller chip gives (8 rows x 151936, 40 steps: 75 whole, 132 in pieces).
inline int entropy_row_parts(int rows, int V) {
    const int nvec = V / 8, least = (nvec + 2047) / 2048;         // at most 8 vectors per thread and piece
    return rows > 2 || nvec <= 3 * 2048 ? 1 : std::max(least, 8);
}

// How k_linear_mfma takes a matrix of NB row blocks x KC k tiles (QKV and residual projections) in a pass of TB token blocks:
// R row blocks and NT token blocks a workgroup, K split into KS slabs (may_split: residual projections).
//
// These passes are a weight stream and a chain of latencies, so what counts is that every compute unit has a workgroup and that a
// workgroup has little to do: the smallest R x NT that is at most one workgroup per unit.  A matrix's second and
// later token blocks find its tiles in L2.  Measured on rotating weights, us, with the former rule (all of up to 64 rows
// in one workgroup, R by matrix size) -> now: 896 x 896 at 32, 64 and 128 rows 4.3 -> 3.5, 5.7 -> 3.5, 5.6 -> 4.3; 1152 x 896 at 64
// rows 7.2 -> 5.1 (one block and one: 4.9); 896 x 4864 at 64: 9.4 -> 7.6; 2048 x 2048 at 32: 6.0 -> 4.9; 3072 x 2048 at 64: 10.2 ->
// 8.6 (R = 1, NT = 2, 384 workgroups: 10.8); 4096 x 4096 at 64: 13.4 -> 12.0.  Of two R x NT of two, the one with more workgroups; of equally many
// two row blocks (2048 x 2048 at 64 rows: 5.6 against 5.9), from 128 k tiles on two token blocks (896 x 4864 at 96: 9.7 against 11.0).
// Eight blocks (3072 x 3072 at 160 rows: 23.4 -> 12.9) and sixteen (at 256: 31.3 -> 17.2) only where that leaves one round of
// workgroups; a QKV projection of fewer than 32 k tiles takes up to three rounds of small ones instead (1152 x 896 at 320 rows 9.6 -> 8.3; in four
// rounds 4096 x 768 at 128 rows 11.2, in tiles of two by four 9.75), of more than one row block per unit only where eight blocks are more than a round,
// too (7168 x 768 at 64 rows 12.1 against 10.2), and four blocks up to three rounds before sixteen (6144 x 896 at 80 rows 12.3, 13.8).  Up to 16 k tiles
// the small ones hold out for six rounds, and sixteen blocks never pay (7168 x 384 at 128 rows: 11.7, in eight 10.8, in sixteen 12.1).
//
// K is split where units would idle and a slab keeps more than 32 k tiles (896 x 4864 at 16 rows: 8.0 -> 6.4; 2048 x 8192: 128
// workgroups 11.8, two slabs 9.9, four of two row blocks 10.3).  Long K (256 k tiles and more) of 17 to 64 rows: two row blocks and two token blocks,
// whose tiles are fetched half as often, and the slabs that fill the chip (2048 x 8192 at 64 rows 14.0, unsplit 15.0; 4096 x
// 14336 at 32 24.5, unsplit 28.0), three token blocks all in one workgroup from a third of a row block per unit on (a layer's two residual projections, 2048 x 9728 at 40
// rows: 23.8, in two by two 25.8; 2048 x 8192 21.9, 23.0; 1536 x 11008 24.6, 25.7; but 1024 x 8192 20.6, 18.4); of few row blocks also at more rows (512 x 14336 at 80: 11.4, unsplit 16.8), but not where even eight slabs leave
// a quarter of the units idle (at 32 rows 768 x 9728 9.3, two row blocks and one token block 8.7; 512 x 11008 9.2, one and one in four slabs 8.1).  Long K of up to 16 rows: two or four row blocks from 3/4 of a row block per unit on (4096 x 14336: 27.9
// -> 21.5, 5120 x 13824: 29.5 -> 26.1), and from half on where that gives three slabs (2560 x 11008 13.8, unsplit 16.3) or K is very long (3072 x
// 14336 19.5 against 20.6, but 3072 x 8192 14.0 against 12.7).
constexpr int kSplitKMax = 8;       // most slabs of K per row-block group

struct NarrowPlan { int R, NT, KS; };

inline NarrowPlan narrow_plan(int NB, int KC, int TB, int n_cu, bool may_split, size_t most_floats, int most_groups) {
    const auto groups = [&](int R, int NT) { return (long)((NB + R - 1) / R) * ((TB + NT - 1) / NT); };
    const auto fits = [&](const NarrowPlan &p) {       // the slabs' sums and the counters have room
        return (size_t)p.KS * groups(p.R, p.NT) * p.R * p.NT * 256 <= most_floats && groups(p.R, p.NT) <= most_groups;
    };
    if (may_split && KC >= 256 && (TB <= 4 || 3 * groups(2, 2) <= n_cu)) {
        NarrowPlan p{0, 0, 1};
        if (TB == 3 && 3 * NB > n_cu) p = NarrowPlan{2, 4, 1};
        else if (TB >= 2 && 4 * kSplitKMax * groups(2, 2) > 3 * n_cu) p = NB > n_cu && TB == 2 ? NarrowPlan{4, 2, 1} : NarrowPlan{2, 2, 1};
        else if (TB >= 2) { if (TB == 2 && kSplitKMax * groups(2, 1) > n_cu) p = NarrowPlan{2, 1, 1}; }
        else if (4 * NB > 3 * n_cu) p = NarrowPlan{NB > n_cu ? 4 : 2, 1, 1};
        else if (2 * NB > n_cu && (3 * groups(2, 1) <= n_cu || KC >= 384)) p = NarrowPlan{2, 1, 1};
        if (p.R) {
            p.KS = std::min<long>(kSplitKMax, n_cu / groups(p.R, p.NT));
            if (p.KS > 1 && fits(p)) return p;
        }
    }
    NarrowPlan p{2, 1, 1};
    const long one = groups(1, 1), rows2 = groups(2, 1), toks2 = groups(1, 2), rows4 = groups(4, 2), toks4 = groups(2, 4);
    if (one <= n_cu || TB <= 1) p = NarrowPlan{one <= n_cu ? 1 : 2, 1, 1};
    else if (std::min(rows2, toks2) <= n_cu) {
        const bool toks = rows2 > n_cu || (toks2 <= n_cu && (toks2 > rows2 || (toks2 == rows2 && KC >= 128)));
        p = toks ? NarrowPlan{1, 2, 1} : NarrowPlan{2, 1, 1};
    } else if (groups(2, 2) <= n_cu) p = NarrowPlan{2, 2, 1};
    else if (!may_split && KC < 32 && (KC <= 16 ? toks2 <= 6 * n_cu : toks2 <= 3 * n_cu && (NB <= n_cu || toks4 > n_cu))) p = NarrowPlan{1, 2, 1};
    else if (toks4 <= n_cu || TB == 2 || KC <= 16) p = NarrowPlan{2, TB > 2 ? 4 : 2, 1};
    else if (rows4 <= n_cu) p = NarrowPlan{4, 2, 1};
    else if (!may_split && KC < 32 && groups(2, 2) <= 3 * n_cu) p = NarrowPlan{2, 2, 1};
    else p = groups(4, 4) <= n_cu ? NarrowPlan{4, 4, 1} : NarrowPlan{2, 4, 1};
    if (may_split && p.R == 1 && p.NT == 1) {          // any larger tile was taken because the smaller ones fill the chip
        while (p.KS < kSplitKMax && (p.KS + 1) * groups(p.R, p.NT) <= n_cu && KC / (p.KS + 1) > 32) ++p.KS;
        while (p.KS > 1 && !fits(p)) --p.KS;
    }
    return p;
}

// Whether gate/up of up to 16 rows goes one row block a workgroup instead of two: where the fullest unit then has fewer blocks to take.  us of two / one:
// 4096 x 2560 7.8 / 6.2 (one block per unit instead of two), 9728 x 896 7.3 / 6.6 (three instead of four), 28672 x 4096 41.2 / 40.6 (seven, eight); but,
// as many either way, 6144 x 2048 7.1 / 8.1, 8192 x 2560 9.0 / 9.9, 21504 x 4096 32.1 / 35.4, 32768 x 5120 53.4 / 54.9.
inline bool gate_up_by_one(int NB, int n_cu) { return (NB + n_cu - 1) / n_cu % 2 == 1; }

// Keys per split of a pass's attention.  A workgroup takes at least 512 keys; more splits only while that helps to fill the
// chip, never more than max_splits (the last one merges them all), bounded scratch (items: rows x splits).  A decode
// step of one or two rows is a chain of latencies: splits of 128 keys, one workgroup per query head and split, spread it
// over more compute units (+3 % tokens/s at batch 1 against 512).
//
// The matrix-core kernel (mfma) from 3/8 of a (row, KV head) pair per compute unit: there are workgroups enough, and a
// launch with splits pays 4-8 us for the partials' way through memory and for workgroups that find nothing to do.
//  * pairs for at most half the units: whole up to 896 keys (head dims below 128: 1664), then two splits, one workgroup per unit
//    (us whole, in 2, 3 and 4 splits at 96 pairs of 5 query heads of 128, every row at 1000 keys 18.8, 18.5, 22.7, 21.3; 1600:
//    30.5, 23.9, 29.6, 26.8; 2000: 33.3, 28.5, 35.4, 31.4; 4000: 59.9, 49.0, 57.1, 53.8; 6000: 81.2, 59.1, 78.0, 68.2; 128
//    pairs, 2000 keys: 34.5, 33.7, 38.4, 34.4; rows of 250-2000 keys 34.5, 29.6, 32.3, 30.9; heads of 64, 96 pairs:
//    2000 keys 17.4, 15.5, 18.9, 16.9; 128 pairs of 7 heads of 64: 1500 keys 14.7 whole, 16.1 in two);
//  * more pairs: whole up to 2048 keys, since two splits are more workgroups than units (160 pairs, 2000 keys 38.2, 47.9, 41.4, 48.1;
//    256 pairs 53.4, 57.4, 66.7, 66.1; 64 rows of the 0.5B shape at 128-1050 keys 10.2 whole, 13.2 split).
// Beyond that, and with fewer pairs (8 rows of the 14B shape at 128-1050 keys: 14.8 against 17.0 whole): the splits that keep
// two workgroups per unit.  The kernel is bound by the latency of its short chains of loads: fewer, longer workgroups.
inline int attention_chunk(int T, int KV, int hd, int ctx_max, bool mfma, int n_cu, int max_splits, long items) {
    const long pairs = (long)T * KV;
    const auto splits = [&](int chunk) { return (ctx_max + chunk - 1) / chunk; };
    int chunk = T <= 2 ? 128 : 512;
    if (mfma && pairs >= 3 * n_cu / 8) {
        if (2 * pairs <= n_cu && ctx_max > (hd >= 128 ? 896 : 1664)) {
            if (ctx_max <= 6144) chunk = ((ctx_max + 1) / 2 + 31) & ~31;      // whole blocks of 32 keys
        } else if (ctx_max <= 2048) chunk = 2048;
    }
    while (pairs * splits(chunk) > 1024 && chunk < 65536) chunk <<= 1;
    while (splits(chunk) > max_splits) chunk <<= 1;
    while (ctx_max > chunk && (long)T * splits(chunk) > items) chunk <<= 1;   // a single split leaves no partials
    if (mfma && T > 2 && pairs * splits(chunk) > 64)
        while (pairs * splits(chunk) > 2 * n_cu && chunk < 65536) chunk <<= 1;
    return chunk;
}

// Whether one row goes through k_linear_ring instead of k_linear_valu (NB row blocks x K).  The ring keeps one workgroup per compute unit (gate/up of
// K < 2048: two) and gains the wait for the row's norm and the gaps between row blocks; it loses where its slices fill its groups badly
// (below 1280 four waves take eight k tiles a group, from there on eight waves take four) or where the other form's many workgroups hide more.
// us of k_linear_valu / ring, rotating weights, 256 units:
//  * QKV: up to one row block per unit (1152 x 896 4.4 / 3.8, 3840 x 1280 6.5 / 5.4; but 4608 x 1536 7.2 / 7.5); K = 2048, where the other form
//    has eight waves, too: up to 3/4 (3072 x 2048 6.1 / 5.8, 4096 x 2048 6.6 / 6.9).  Longer K 5120 x 3072 10.2 / 11.1.
//  * gate/up below 1280: up to one row block per unit (4096 x 1024 4.9 / 4.1) or more than two (9856 x 896 7.0 / 6.3; between them 4160 x 384 4.2 / 4.4,
//    8192 x 1024 6.1 / 6.4).  From 1280 on only 2048, whose slices are whole groups (8192 x 2048 9.2 / 8.7, 16384 x 2048 14.0 / 13.8; but 7680 x 1280
//    7.1 / 8.5, 9216 x 1536 9.8 / 9.9, 15360 x 1920 13.1 / 14.4).
//  * LM head: 1280 to 3776 (128256 x 1536 69 / 59, 128256 x 3072 129 / 116; 256000 x 3776 280 / 277, 256000 x 4064 302 / 308); 896 to 1024 (128256 x 1024 47 / 43;
//    but x 1152 57 / 76, of which up to four row blocks per unit 16000 x 1152 13.9 / 13.3); shorter rows of few blocks (32768 x 640 14.6 / 13.2, 16000 x 384 9.2 / 8.3, 4096 x 64
//    5.0 / 4.7; but 151936 x 512 35 / 47, 50304 x 640 18.2 / 18.7, 32000 x 384 12.3 / 13.0).
//  * residual projections of 6144 to 8192, all that four vectors a lane hold, of up to 3/4 row block per unit (2048 x 8192 9.9 / 9.1, 3072 x 8192
//    12.1 / 11.3, 1024 x 6144 7.7 / 7.35, 3072 x 6912 10.5 / 10.4; but 4096 x 7680 13.2 / 13.8, 2048 x 4864 7.6 / 7.8).
inline bool ring_takes(int K, int NB, int n_cu, Epilogue epi) {
    switch (epi) {
        case EPI_QKV: return K <= 2048 && 4 * NB <= (K < 2048 ? 4 : 3) * n_cu;
        case EPI_SWIGLU: return K < 1280 ? NB <= n_cu || NB > 2 * n_cu : K == 2048;
        case EPI_RES: return K >= 6144 && K <= 8192 && 4 * NB <= 3 * n_cu;
        default: break;
    }
    if (K >= 896) return K <= 1024 || (K < 1280 ? NB <= 4 * n_cu : K <= 3776);
    return NB <= (K >= 640 ? 8 : K >= 128 ? 4 : 2) * n_cu;
}

// Whether a pass's attention goes to k_attn, a workgroup per (row, query head): few rows, which want the lanes.  All its products are
// float32; the kernels of more rows split queries and probabilities into bf16 terms (1e-7 and 2e-6 from 64 bits).
inline bool per_head_attention(int T, int KV, int splits) { return T <= 2 || (long)T * KV * splits <= 64; }

// Whether a pass's attention goes to k_attn_prompt (rows of `seqs` sequences in workgroups of four waves that share K and V and take
// all keys in turn) instead of k_attn_mfma (`groups` workgroups per KV head whose waves split the keys).  The first takes
// 0.55 (head dims up to 64) to 0.76 us per 32 keys of the longest context whatever the number of rows, up to a workgroup per
// unit; the second 0.4 us per 32 keys and round of workgroups.  us of the second against the first (here with queries in two terms; the third adds
// 3-8 %), heads of 128, 5 per KV head, 8 KV heads:
// contexts up to 160: 17 rows 7.6 / 5.7, 130 rows 12.3 / 8.2, 4 rows each of 4 and 12 sequences 7.5 / 5.3 and 8.0 / 5.4;
// rows from key 200 on: 64 rows (176 workgroups) 10.6 / 11.1, 130 (352) 16.6 / 12.5; from 600: 64 rows 14.8 / 19.5, 130 rows 25.0 / 21.1, 11 rows each of
// 12 sequences (384) 23.7 / 20.5, 4 rows each of 40 (640) 50.6 / 24.6; from 2000: 64 rows 29.7 / 49.5, 160 (440) 55.6 / 52.1, 500 rows (1344) 160.6 / 66.3; from 8000: 160 rows 177 /
// 183, 500 rows 538 / 221.  Heads of 64, 7 per KV head, 2 KV heads: from 600 160 rows (160) 13.2 / 16.1, 500 rows (500) 27.2 / 21.7.
//
// A few rows each of many sequences are where the first has more workgroups than units (`own` per KV head) and the second may still have no more than
// two each, all resident: that one is faster then (5 rows each of 40 sequences, 480 workgroups against 320, heads of 64 and 128, from key
// 400: 16.1 / 16.5 and 21.2 / 22.9, 1000: 24.6 / 29.0 and 35.9 / 41.5, 2000: 41.5 / 48.4 and 60.3 / 70.7; but 6 rows each of 33, 528 against 264: 31.6 / 28.4 and 56.3 /
// 41.3), heads of 64 and up to five rows a sequence also a little past it (5 each of 48, 576: 25.5 / 29.1, 6 each of 40, 640: 31.7 / 29.4; from key 400 5 each of 48 16.7 / 15.8).
// Where a sequence's rows are one workgroup of the second, too, and their keys and values more than the caches hold, both read the same bytes (32 KV heads of 128, 5
// rows each of 100 sequences from 600, 1 GB: 193 / 202, of 40 from 1000, 0.66 GB: 130 / 133; of 64 from 300, 0.32 GB: 76 / 75).
//
// Scoring stays with k_attn_mfma.  It returns logits, and the two kernels add a row's keys in another order: behind a few layers of half-precision
// activations that is 9e-4 of the logits' norm (8 layers of the 14B shape, 101 rows; either kernel is 1.4e-3 from 64 bits), where a pass of 101 rows
// with its logits takes 3.7 ms and the other kernel saves 0.03 of them.
constexpr int kGroupSeqs = 1024;                        // most sequences of a batch whose passes k_plan lists in groups
inline bool prompt_attention(int T, int seqs, long groups, long own, int KV, int hd, int ctx, int n_cu, bool scoring) {
    if (scoring || T < 17 || T < 4 * seqs || per_head_attention(T, KV, 1)) return false;
    if (ctx <= 160) return true;
    const long wgs = groups * KV;
    if (ctx > 320 && own * KV > n_cu && wgs <= (hd <= 64 && ctx > 512 && T <= 5 * seqs ? 600 : 2 * n_cu)) return false;
    if (groups == seqs && (size_t)seqs * ctx * KV * hd * 4 >= ((size_t)512 << 20)) return false;
    return wgs >= (ctx <= 320 ? 256 : ctx <= 4096 ? 400 : 512);
}

// Whether a gate/up matrix in a pass of two token blocks goes four row blocks to a workgroup of two waves (launch_narrow: what both ways measured).
inline bool gate_up_by_four(int NB, int KC, int n_cu) { return NB > 6 * n_cu && KC % 64 != 0; }

// Gate/up matrices whose passes of one or two token blocks stream through k_linear_mfma_ls (us in launch_narrow's workgroups / this way).  One
// block: long K and more than four row blocks per compute unit (28672 x 4096 41.5 / 40.0, 27648 x 5120 50.6 / 46.9; but 16384 x 3072 18.1 / 21.1, 16384 x 2048
// 14.5 / 16.9, 9728 x 896 7.4 / 8.4).  Two: K of 3072 and more (28672 x 4096 48.3 / 40.2, 27648 x 5120 55.6 / 47.2, 16384 x 3072 21.8 / 20.4) and more than two row
// blocks per unit, since up to there launch_narrow's workgroups are one round (8192 x 3072 12.8 / 15.8, x 5120 18.2 / 23.6, 2048 x 4096 12.9 / 17.7; 8320 x 3072 17.5 / 15.2,
// 9728 x 5120 29.0 / 23.5).  Shorter ones gain alone
// (17920 x 1536 17.5 / 14.6, 24576 x 1536 18.8 / 16.5, 9728 x 896 9.5 / 8.3; not 16384 x 2048, 16.1 / 16.5) but belong to small models, whose passes run beside the large
// model's: a workgroup of 112 KB of LDS keeps that one's out of its unit (64 rows grouped, 0.5B / 14B shapes: 64.5 ms with them, 63.4 without).  Runs of one
// lane, where nothing runs beside them, go without that gain: the rule does not know the lane.
inline bool gate_up_streamed(int NB, int KC, int TB, int n_cu) {
    return TB == 1 ? KC >= 128 && NB > 4 * n_cu : TB == 2 && KC >= 96 && NB > 2 * n_cu;
}

// Whether k_linear_mfma_ls requests a matrix of `tiles` k tiles (KB) non-temporally, rg row blocks to a workgroup, in slabs of K or not.  A long stream from memory
// gains by it (us with plain requests / this way: 27648 x 5120 at 64 rows 50.3 / 48.0, 5120 x 13824 in slabs 31.7 / 26.9), a shorter one is not bound by memory and
// loses (16384 x 896 at 128 rows 13.1 / 15.0, 4096 x 2048 11.2 / 13.2, 12288 x 1536 in slabs 13.3 / 14.8), and so does a group of five row blocks, whose
// slot repeats three tiles that the vector cache no longer holds (19456 x 5120 37.6 / 42.8), up to some size one of six (20672 x 3328 23.7 / 27.6).  236 gate/up
// shapes at 16 to 128 rows, 22 of slabs.
inline bool tiles_once(long tiles, int rg, bool slabs) {
    return slabs ? tiles >= 80000 : rg != 5 && tiles >= (rg == 6 ? 140000 : 96000);
}

// LM heads of one and two token blocks that stay with k_linear_mfma's register rings (us with them / through k_lm_ls).  A workgroup of k_lm_ls walks its NB / n_cu
// row blocks eight at a time, and slots past their end cost what the others do: rings where that leaves half a group and more empty on every unit
// (8192 x 4096 at 3 rows 15.6 / 31.5, 16384 x 5120 30.3 / 38.7, 40000 x 4096 53 / 73, 100000 x 4096 131 / 151, at 24 rows 40000 x 5120 77 / 94;
// but 24000 x 4096 at 12 rows 36.6 / 35.0, 65536 x 3328 72 / 67, 50256 x 4096 at 24 rows 90 / 77).  Where K is no multiple of 512 the rings' last turn is partly empty and
// more has to be (81920 x 2304 at 12 rows 66 / 65, 114688 x 1792 at 3 rows 72 / 70; 100000 x 3328 111 / 121).  K below 1280, with two blocks to 2048: never.  One block of
// K between 2048 and 4096, whole turns: the two are level, and with few rows that sample the rings are up to 4 % the faster (128256 x 3072 at 3 and 12 rows greedy
// 126 127 / 127 128, sampling 131 141 / 132 133).  (180 shapes at 3 to 32 rows; the one taken is at most 7 % the slower, 1 % in the mean.)
inline bool lm_by_rings(int NB, int KC, int TB, int n_cu) {
    if (TB > 2 || KC < 40 || (TB == 2 && KC <= 64)) return false;
    const long walked = (long)((NB + 8 * n_cu - 1) / (8 * n_cu)) * 8 * n_cu, empty = walked - NB;
    const bool whole = KC % 16 == 0;
    if (TB == 1 && whole && KC > 64 && KC < 128) return true;
    return 2 * empty >= (TB == 1 ? 7 : 8) * n_cu && (whole || 8 * NB <= 5 * walked || (TB == 1 && KC > 64 && empty >= 6 * n_cu));
}

// Whether k_lm_ls requests its tiles non-temporally.  Where its groups of eight row blocks are mostly full it does: the kernel alone then is faster from some 300 MB on (us with
// plain requests / this way: 128256 x 4096 at 32 rows 178 / 159, 32000 x 4096 at 64 rows 51 / 45) and up to 10 % slower below (32000 x 2048 at 3 rows 25.1 / 27.6), but the head
// leaves the caches to the layers' weights, K and V, which gains more (us a step of small models, LM head of 32000 x 1536, 48, 64, 100 and 128 rows: 304 310 361 377 / 288 297 342 363;
// 32000 x 768: 454 486 608 643 / 440 479 603 640).  Where slots past the row blocks' end repeat the last one, which the vector cache then no longer holds, only
// long streams do (8192 x 4096 at 64 rows 28 / 31, 16384 x 5120 34 / 43; 40000 x 4096 at 3 rows 77 / 73).
inline bool lm_once(int NB, int KC, int n_cu) {
    const long walked = (long)((NB + 8 * n_cu - 1) / (8 * n_cu)) * 8 * n_cu;
    return 4 * NB >= 3 * walked || (long)NB * KC >= (KC >= 96 ? 190000 : 290000);
}

// How 256 x 256 tiles take a pass: NG groups of 16 row blocks x SG sweeps of 256 tokens x KC k tiles.  The first `whole` sweeps in tiles of full depth, the
// others, which would leave a round of workgroups partly empty, in tiles of one of KS slabs of K, whose sums another launch adds.  Cost in
// cycles: 1750 per k tile and round, 1950 with the whole chip busy (measured; an eighth of the tiles to each XCD's units), the sums written and read at 5 TB/s, and
// the two launches more; a split has to promise 8 %.  (ms of a 6-layer pair's prompts, Qwen 0.5B / 14B shapes, before -> now: 2600 positions
// 13.2 -> 10.6, 3950 15.4 -> 14.4, 5870 27.3 -> 22.2, 10670 43.8 -> 39.2; of that the numbering of the tiles 42.2.)
struct TilePlan { int whole, KS; long cost; };
inline TilePlan tile_plan(int NG, int SG, int KC, int n_cu, bool may_split, size_t most_floats) {
    const auto cost = [&](long tiles, long steps) {
        const long rounds = ((tiles + 7) / 8 + n_cu / 8 - 1) / (n_cu / 8);
        return rounds * steps * 1750 + 200 * steps * tiles / n_cu;
    };
    TilePlan best{SG, 1, cost((long)NG * SG, KC)};
    if (!may_split || SG < 4) return best;
    for (int whole = 0; whole < SG; ++whole)
        for (int KS = 2; KS <= kSplitKMax && KC / KS >= 32; ++KS) {
            const long floats = (long)NG * (SG - whole) * 65536 * KS;
            if ((size_t)floats > most_floats) break;
            const long c = (cost((long)NG * whole, KC) + cost((long)NG * (SG - whole) * KS, KC / KS + 9) + floats * 8 / 2000 + 12000) * 27 / 25;
            if (c < best.cost) best = TilePlan{whole, KS, c};
        }
    return best;
}

// How k_decode_stream cuts a matrix of NB row blocks x KC tiles into units of one row block x one of `slices` parts of K for G workgroups:
// the fewest slots of eight tiles for the workgroup that has most (a slot is 0.33 us at the stream's rate), where a slice more
// is one more vector of sums for every workgroup to read (0.2 us).  `most`: columns of a slice that fit the stage.
struct StreamSplit { int slices, tiles; };      // slices of K, tiles of each but a shorter last
inline StreamSplit stream_split(int NB, int KC, int G, int most) {
    StreamSplit best{0, 0};
    float cost = 0.f;
    for (int s = 1; s <= 4; s *= 2) {
        if (G % s || KC < 8 * s) continue;
        const int tiles = s == 1 ? KC : ((KC + s - 1) / s + 7) / 8 * 8;
        if (tiles * (s - 1) >= KC || tiles * 32 > most) continue;
        const int rounds = (NB + G / s - 1) / (G / s);
        const float c = 0.33f * (float)(rounds * ((tiles + 7) / 8)) + 0.2f * (float)s;
        if (best.slices == 0 || c < cost) { best = StreamSplit{s, tiles}; cost = c; }
    }
    return best;
}

// Whether a step of one row goes to k_decode_stream: what a layer gains has to pay for the way in and the barrier at the end, 3-18 us a step.
// Measured, us a layer at 330 keys with the kernels per layer / this way: d 896 28.0 / 24.8, 1536 44.0 / 35.9, 2048 42.3 / 35.6, 3072 56.1 / 47.2, 4096 90.9 / 83.5, 5120 114.4 /
// 100.0; at 1200 keys, which eight workgroups per KV head share, 28.9 / 28.2 and 44.3 / 42.9 (two KV heads), 43.9 / 37.6, 58.1 / 50.9, 93.7 / 87.6, 117.1 / 106.1 (eight).
// Those have an FFN of 2.7 to 5.8 d.  The hand-overs cost the same whatever streams between them, so short FFNs gain less or lose (us a step of 12 layers and a vocabulary of
// 8192, per layer / this way, at d_ffn 512, 1024, 2048, 3072, 4864: d 896 278 285 297 322 - / 300 299 300 309 -; 1024 279 287 302 333 365 / 292 292 293 299 318; 1536 330
// 339 357 378 432 / 339 345 350 367 391; 2048 with four KV heads 327 336 368 398 447 / 339 342 342 365 404, with eight 332 346 371 398 447 / 332 333 332 356 396; 3072 432
// 440 473 510 582 / 388 397 402 444 496; 4096 492 506 548 592 681 / 490 492 525 577 657).
inline bool stream_pays(int d, int F, int KV, int layers, int keys) {
    const float f = (float)F, at330 = d <= 1024 ? std::min(2.5f, 0.00093f * f - 1.3f) : d < 2048 ? std::min(6.f, 0.00088f * f - 0.8f) :
                    std::min(6.f, (d <= 3072 ? 0.0016f * f + 0.3f + 0.0035f * (float)(d - 2048) : 0.0004f * f + 1.f) - (KV >= 8 ? 0.f : 1.2f));
    const float gain = at330 - (KV >= 8 ? 0.0015f : 0.006f) * (float)std::max(0, keys - 330);
    return keys <= 2048 && gain * (float)layers > 20.f;
}

}  // namespace ead

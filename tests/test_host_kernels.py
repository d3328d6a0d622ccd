"""CPU: kernels of the library compiled for the host (tests/host_kernels.cpp), on inputs that are shown to be handled before
a GPU sees them: logits that are not finite must leave a token inside the vocabulary.  Also the rules of dispatch, at sizes
where the other side was measured slower."""
import ctypes as C
import os
import subprocess

import numpy as np
import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
CLANG = "/opt/rocm/llvm/bin/clang++"
PARTIAL = np.dtype([("m", "f4"), ("Z", "f4"), ("S", "f4"), ("idx", "i4"), ("gs", "f4"), ("gidx", "i4")])
NONE = 0x7FFFFFFF


@pytest.fixture(scope="module")
def host(tmp_path_factory):
    so = str(tmp_path_factory.mktemp("host") / "host_kernels.so")
    subprocess.run([CLANG, "-x", "c++", "-std=c++17", "-O1", "-fPIC", "-shared", "-w", "-I", os.path.join(HERE, "host_hip"),
                    "-I", os.path.join(os.path.dirname(HERE), "paper_2502_06833_amd", "csrc"),
                    os.path.join(HERE, "host_kernels.cpp"), "-o", so, "-lpthread"], check=True)
    return C.CDLL(so)


def _finalize(host, parts, sampling):
    rows, n = parts.shape
    tok, H, err = np.full(rows, -1, np.int32), np.zeros(rows, np.float32), np.zeros(1, np.int32)
    host.host_finalize(parts.ctypes.data_as(C.c_void_p), rows, n, int(sampling), tok.ctypes.data_as(C.c_void_p),
                       H.ctypes.data_as(C.c_void_p), err.ctypes.data_as(C.c_void_p))
    return tok, H, int(err[0])


def _partials(n, rng):
    p = np.zeros((1, n), PARTIAL)
    p["m"] = rng.integers(0, 5, n); p["Z"] = 1 + rng.random(n); p["S"] = -rng.random(n); p["idx"] = 16 * np.arange(n) + rng.integers(0, 16, n)
    p["gs"] = rng.integers(0, 5, n); p["gidx"] = 16 * np.arange(n) + rng.integers(0, 16, n)
    return p


@pytest.mark.parametrize("n", [1, 37, 64, 65, 256, 512, 1024])
@pytest.mark.parametrize("sampling", [False, True])
def test_finalize_picks_a_token_of_the_vocabulary(host, n, sampling):
    p = _partials(n, np.random.default_rng(n))
    key, idx = ("gs", "gidx") if sampling else ("m", "idx")
    tok, H, err = _finalize(host, p, sampling)                       # finite: the lowest index of the largest value
    assert tok[0] == p[idx][0][p[key][0] == p[key].max()].min() and np.isfinite(H[0]) and err == 0
    for bad in (np.ones(n, bool), np.arange(n) < 64, np.arange(n) >= 64, np.arange(n) % 3 != 1):
        q = p.copy()
        for k in ("m", "Z", "S"):
            q[k][0][bad] = np.nan
        q["gs"][0][bad] = -np.inf                                    # a NaN score never beats the running maximum
        q["gidx"][0][bad] = NONE
        tok, H, err = _finalize(host, q, sampling)
        good = ~bad
        if good.any():
            assert tok[0] == q[idx][0][good][q[key][0][good] == q[key][0][good].max()].min()
        else:
            assert tok[0] == q["idx"].min()
        if bad.any():
            assert np.isnan(H[0]) and err == 1


def test_finalize_without_a_perturbed_score_takes_the_arg_max(host):
    """l / T can overflow to -inf in every entry while the logits are finite."""
    p = _partials(100, np.random.default_rng(0))
    p["gs"] = -np.inf; p["gidx"] = NONE
    tok, H, err = _finalize(host, p, True)
    assert tok[0] == p["idx"][0][p["m"][0] == p["m"].max()].min() and np.isfinite(H[0]) and err == 0


@pytest.mark.parametrize("groups,have", [(1, 8), (1, 1), (3, 5)])
def test_lm_fold_keeps_an_index_of_the_vocabulary(host, groups, have):
    rng = np.random.default_rng(groups)
    blocks = (groups - 1) * 8 + have
    base = rng.normal(size=(groups * 8, 4)).astype(np.float32)
    place = 16 * np.arange(groups * 8)[:, None] + np.arange(4)
    for bad in ("none", "all", "first group", "scattered", "-inf"):
        x = base.copy()
        if bad == "all":
            x[:] = np.nan
        elif bad == "first group":
            x[:8] = np.nan
        elif bad == "scattered":
            x[rng.random(x.shape) < 0.5] = np.nan
        elif bad == "-inf":
            x[:] = -np.inf
        out = np.zeros(1, PARTIAL)
        host.host_fold(x.ctypes.data_as(C.c_void_p), groups, have, C.c_float(0.0), out.ctypes.data_as(C.c_void_p))
        v, where = x[:blocks].ravel(), place[:blocks].ravel()
        finite = v[np.isfinite(v)]
        if len(finite):
            assert out["idx"][0] == where[v == finite.max()].min(), bad
        else:
            assert out["idx"][0] in where, bad
        assert bool(np.isfinite(out["Z"][0])) == (bad == "none" or bool(np.isfinite(v).all())), bad


@pytest.mark.parametrize("rows,V,size,one", [
    (1, 8, 2, 1), (1, 262144, 2, 1), (3, 151936, 2, 1), (16, 50264, 4, 1), (64, 32000, 2, 1), (600, 512, 2, 1),
    (24, 50264, 2, 0), (7, 128256, 2, 0), (13, 151936, 2, 0), (4, 262144, 2, 0), (2000, 512, 2, 0), (4096, 64, 4, 0),      # in one launch: 6-47 % slower
    (97, 50264, 4, 0)])
def test_small_entropy_calls_take_one_launch_where_that_is_faster(host, rows, V, size, one):
    assert host.host_entropy_folds(rows, V, size) == one


@pytest.mark.parametrize("rows,V,parts", [(1, 8192, 1), (2, 32000, 1), (1, 49152, 1), (1, 49160, 8), (2, 131072, 8), (2, 151936, 10), (3, 151936, 1), (1, 1048576, 64)])
def test_gate_rows_go_to_workgroups_in_pieces_where_that_is_faster(host, rows, V, parts):
    assert host.host_entropy_row_parts(rows, V) == parts


@pytest.mark.parametrize("T,KV,hd,ctx,splits", [
    (12, 8, 128, 700, 1), (12, 8, 128, 1000, 2), (12, 8, 128, 2000, 2), (16, 8, 128, 2000, 2), (16, 8, 128, 4000, 2), (12, 8, 128, 6000, 2),
    (12, 8, 64, 1000, 1), (12, 8, 64, 2000, 2), (64, 2, 64, 1050, 1), (64, 2, 64, 2000, 2),
    (18, 8, 128, 2000, 1), (32, 8, 128, 2000, 1), (18, 8, 128, 3000, 3), (20, 8, 128, 3000, 3), (32, 8, 128, 3000, 2),
    (8, 8, 128, 1050, 3), (1, 8, 128, 500, 4)])
def test_attention_splits_follow_the_measured_best(host, T, KV, hd, ctx, splits):
    """Among them the passes that one workgroup per context (12-16 rows at 1000 keys and more) or two splits of 2048 keys
    (18-20 rows at 3000) had made slower."""
    chunk = host.host_attention_chunk(T, KV, hd, ctx, 1, C.c_long(2048))
    assert -(-ctx // chunk) == splits and (splits == 1 or chunk % 32 == 0)


def test_attention_splits_stay_within_the_scratch(host):
    for T in (1, 2, 3, 12, 16, 17, 33, 100, 1024, 4096):
        for KV in (1, 2, 8, 40):
            for ctx in (1, 31, 128, 897, 1665, 2048, 2049, 6145, 70001):
                for mfma in (0, 1):
                    for hd in (32, 128):
                        chunk = host.host_attention_chunk(T, KV, hd, ctx, mfma, C.c_long(2048))
                        splits = -(-ctx // chunk)
                        assert splits == 1 or (splits <= 16 and T * splits <= 2048 and chunk % 32 == 0), (T, KV, ctx, mfma, hd)


@pytest.mark.parametrize("NB,KC,split,plans", [
    (72, 28, 0, {1: 111, 2: 111, 3: 111, 4: 211, 12: 221, 20: 121}), (56, 28, 1, {1: 111, 4: 111, 6: 211, 10: 221, 31: 241}),
    (56, 152, 1, {1: 114, 2: 112, 3: 111, 4: 111, 6: 121}), (128, 256, 1, {1: 112, 2: 224, 4: 222, 6: 221}),
    (192, 96, 1, {1: 111, 2: 211, 4: 221, 8: 241, 10: 421, 16: 441}), (256, 448, 1, {1: 212, 2: 222, 4: 221}),
    (320, 432, 1, {1: 413, 2: 423, 3: 241}), (448, 160, 0, {1: 211, 2: 221, 4: 241})])
def test_narrow_passes_take_the_measured_best(host, NB, KC, split, plans):
    """The rule's choice at matrices it was measured at (times in rules.hpp); of other shapes it says nothing."""
    for TB, plan in plans.items():
        assert host.host_narrow_plan(NB, KC, TB, split, C.c_long(8 << 20), 4096) == plan, TB


def test_narrow_plans_are_instantiated_and_stay_within_the_scratch(host):
    plain = {11, 12, 21, 22, 24, 42, 44}                     # R, NT of the kernels launch_narrow knows without a split of K
    slabs = {11, 21, 22, 24, 41, 42}
    for NB in (1, 2, 5, 16, 63, 64, 96, 128, 171, 192, 193, 256, 257, 320, 512, 513, 960):
        for KC in (1, 4, 28, 33, 66, 128, 255, 256, 300, 448, 480):
            for TB in (1, 2, 3, 4, 5, 8, 9, 16, 17, 31):
                for split in (0, 1):
                    for floats, groups in ((8 << 20, 4096), (1 << 16, 64)):
                        r = host.host_narrow_plan(NB, KC, TB, split, C.c_long(floats), groups)
                        assert r and r // 10 in (plain if r % 10 == 1 else slabs) and (split or r % 10 == 1), (NB, KC, TB, split)
                        assert r % 10 <= 8


@pytest.mark.parametrize("T,seqs,groups,KV,ctx,takes", [
    (17, 1, 6, 8, 17, 1), (130, 1, 44, 8, 130, 1), (16, 4, 8, 8, 4, 0), (48, 12, 24, 8, 4, 1), (48, 48, 48, 8, 100, 0),
    (64, 1, 22, 8, 264, 0), (130, 1, 44, 8, 330, 0), (130, 1, 44, 8, 310, 1), (160, 1, 55, 8, 2160, 1), (160, 1, 55, 8, 8160, 0), (500, 1, 168, 8, 8500, 1),
    (64, 64, 64, 8, 1000, 0), (160, 1, 80, 2, 760, 0), (500, 1, 250, 2, 1100, 1)])
def test_prompt_attention_takes_the_passes_it_is_faster_at(host, T, seqs, groups, KV, ctx, takes):
    """The rule's choice at passes that were measured (times in rules.hpp)."""
    assert host.host_prompt_attention(T, seqs, C.c_long(groups), KV, ctx) == takes


@pytest.mark.parametrize("seqs,rows,have,G,KV,hd,takes", [
    (40, 5, 999, 8, 4, 64, 0), (40, 5, 999, 8, 4, 128, 0), (40, 5, 1999, 6, 4, 128, 0), (40, 5, 399, 8, 4, 128, 0),      # 480 workgroups against 320
    (33, 6, 999, 8, 4, 64, 1), (33, 6, 999, 8, 4, 128, 1), (24, 8, 1999, 8, 4, 64, 1), (64, 5, 999, 7, 4, 64, 1),       # 528 and more; 480 against 192
    (48, 5, 999, 8, 4, 64, 0), (48, 5, 399, 8, 4, 64, 1), (48, 5, 999, 8, 4, 128, 1), (24, 8, 1999, 4, 8, 64, 1), (40, 6, 999, 7, 4, 64, 1),
    (100, 5, 599, 1, 32, 128, 0), (100, 7, 599, 1, 32, 128, 0), (40, 5, 299, 1, 32, 128, 1), (100, 5, 599, 2, 16, 128, 1), (100, 5, 599, 4, 8, 64, 1)])
def test_prompt_attention_of_a_few_rows_of_many_sequences(host, seqs, rows, have, G, KV, hd, takes):
    """The same for catch-ups, where the kernels' numbers of workgroups and the bytes of the caches decide (times in rules.hpp)."""
    assert host.host_prompt_attention_rows(seqs, rows, have, G, KV, hd) == takes


def test_queries_in_three_terms_lose_nothing(host):
    """k_attn_prompt's queries: three bf16 terms are the float32 value itself (two are within 2^-17 of it, which is seen in its sums)."""
    rng = np.random.default_rng(0)
    x = (rng.standard_normal(8000) * 10.0 ** rng.uniform(-8, 8, 8000)).astype(np.float32)
    x[:8] = [0.0, 1.0, -1.0, 1.0 + 2.0 ** -23, 2.0 - 2.0 ** -23, -3.0000002, 65504.0, 1e-20]
    out = np.zeros(8)
    for i in range(0, x.size, 8):
        v = np.ascontiguousarray(x[i:i + 8])
        host.host_bf16_terms(v.ctypes.data_as(C.c_void_p), 3, out.ctypes.data_as(C.c_void_p))
        assert (out == v).all()
        host.host_bf16_terms(v.ctypes.data_as(C.c_void_p), 2, out.ctypes.data_as(C.c_void_p))
        assert (np.abs(out - v) <= 2.0 ** -17 * np.abs(v)).all()


@pytest.mark.parametrize("KV,most", [(1, 64), (2, 32), (3, 21)])
def test_passes_of_few_rows_and_heads_keep_float32_attention(host, KV, most):
    """Up to 64 (row, KV head) pairs are k_attn's, whose queries and probabilities are float32, however short their contexts."""
    for T in range(17, most + 2):
        for G in (1, 2, 4, 7, 8):
            for pos in (0, 40, 95):
                groups = (pos + T - 1) // (16 // G) - pos // (16 // G) + 1
                assert bool(host.host_prompt_attention(T, 1, C.c_long(groups), KV, pos + T)) == (T > most), (T, G, pos)


@pytest.mark.parametrize("G,KV", [(5, 8), (7, 2), (1, 32), (8, 1)])
def test_scoring_keeps_its_attention_kernel(host, G, KV):
    """Logits that a program compares from one version to the next: no scoring pass (up to 160 rows, any context) changes kernels."""
    rq = 16 // G
    for T in (17, 64, 101, 128, 160):
        for pos in (0, 160, 1120, 4800):
            groups = (pos + T - 1) // rq - pos // rq + 1
            assert not host.host_score_prompt_attention(T, C.c_long(groups), KV, pos + T), (T, pos)


@pytest.mark.parametrize("K,residual,lm,takes", [(2048, 0, 0, 1), (3072, 0, 0, 0), (2048, 1, 0, 0), (8192, 1, 0, 1), (14336, 1, 0, 0), (4864, 1, 0, 0),
                                                 (3072, 0, 1, 1), (4096, 0, 1, 0), (32, 0, 0, 1)])
def test_ring_kernel_takes_the_matrices_it_is_faster_at(host, K, residual, lm, takes):
    """The rule's choice by K, at 128 row blocks; by row blocks below."""
    assert host.host_ring_takes(K, residual, lm) == takes


QKV, RES, SWIGLU, LOGITS = range(4)


@pytest.mark.parametrize("epi,N,K,takes", [
    (QKV, 1152, 896, 1), (QKV, 4096, 1536, 1), (QKV, 4608, 1536, 0), (QKV, 3072, 2048, 1), (QKV, 4096, 2048, 0), (QKV, 1024, 2080, 0),
    (SWIGLU, 4096, 1024, 1), (SWIGLU, 8192, 1024, 0), (SWIGLU, 9728, 896, 1), (SWIGLU, 7680, 1280, 0), (SWIGLU, 17920, 1536, 0), (SWIGLU, 15872, 1984, 0), (SWIGLU, 16384, 2048, 1),
    (LOGITS, 151936, 896, 1), (LOGITS, 151936, 864, 0), (LOGITS, 32768, 640, 1), (LOGITS, 32784, 640, 0), (LOGITS, 16384, 512, 1), (LOGITS, 32000, 512, 0), (LOGITS, 8192, 64, 1),
    (LOGITS, 16384, 64, 0), (LOGITS, 128256, 1152, 0), (LOGITS, 16000, 1152, 1), (LOGITS, 256000, 1280, 1), (LOGITS, 151936, 3776, 1), (LOGITS, 151936, 3808, 0),
    (RES, 3072, 8192, 1), (RES, 4096, 8192, 0), (RES, 2048, 6144, 1), (RES, 2048, 6112, 0), (RES, 2048, 8224, 0)])
def test_ring_kernel_by_row_blocks(host, epi, N, K, takes):
    """Matrices on both sides of the rule's edges: where k_linear_valu measured faster, one row is its own."""
    assert host.host_ring_takes_matrix(K, N // 16, epi) == takes


def test_ring_kernel_holds_what_it_takes(host):
    """No rule takes a K whose slices do not fit the instantiation's registers (four, one and two vectors of 256 elements per wave of eight)."""
    for K in range(32, 15361, 32):
        for NB in (1, 72, 192, 193, 256, 257, 512, 513, 1024, 2049, 9496, 16000):
            for epi, most in ((QKV, 2048), (RES, 8192), (SWIGLU, 2048), (LOGITS, 4096)):
                assert K <= most or not host.host_ring_takes_matrix(K, NB, epi), (K, NB, epi)


@pytest.mark.parametrize("NB,KC,split,plans", [
    (448, 24, 0, {3: 241, 4: 241, 5: 221, 8: 441}), (256, 24, 0, {4: 221, 8: 241}), (512, 28, 0, {4: 241, 8: 441}), (288, 16, 0, {4: 121}), (448, 12, 0, {8: 241}), (192, 28, 0, {8: 121}),
    (160, 344, 1, {1: 213}), (192, 256, 1, {1: 111}), (192, 448, 1, {1: 212}), (136, 256, 1, {1: 213}),
    (384, 28, 0, {5: 221, 8: 221}),
    (32, 344, 1, {2: 114, 3: 228, 5: 225, 8: 224}), (48, 448, 1, {2: 215, 6: 223, 8: 121}), (64, 256, 1, {2: 228}), (16, 448, 1, {2: 118, 10: 226}), (384, 16, 1, {6: 241})])
def test_narrow_passes_of_wide_or_small_matrices(host, NB, KC, split, plans):
    """Shapes that no model above has: where the smallest tiles take four rounds of workgroups and more, and long K of few row blocks."""
    for TB, plan in plans.items():
        assert host.host_narrow_plan(NB, KC, TB, split, C.c_long(8 << 20), 4096) == plan, TB


@pytest.mark.parametrize("NB,KC,plan", [(128, 304, 244), (96, 344, 245), (86, 257, 245), (85, 257, 222), (128, 255, 121), (64, 256, 224)])
def test_three_token_blocks_of_long_k_share_a_workgroup(host, NB, KC, plan):
    """Residual projections of 33 to 48 rows: from a third of a row block per unit on, the weights are fetched once (times in rules.hpp)."""
    assert host.host_narrow_plan(NB, KC, 3, 1, C.c_long(8 << 20), 4096) == plan


@pytest.mark.parametrize("NB,one", [(1, 1), (256, 1), (257, 0), (512, 0), (513, 1), (608, 1), (768, 1), (1024, 0), (1120, 1), (1344, 0), (1728, 1), (1792, 1), (2048, 0)])
def test_gate_up_takes_one_row_block_where_the_fullest_unit_has_fewer(host, NB, one):
    assert host.host_gate_up_by_one(NB) == one
    by_one, by_two = -(-NB // 256), 2 * -(-(-(-NB // 2)) // 256)
    assert bool(one) == (by_one < by_two)


@pytest.mark.parametrize("NG,SG,KS,bs", [(1, 1, 1, 1), (20, 12, 1, 6), (20, 2, 6, 2), (108, 14, 1, 5), (17, 1, 3, 1), (28, 13, 1, 5), (5, 16, 8, 6), (7, 11, 2, 4)])
def test_tiles_are_taken_once_each(host, NG, SG, KS, bs):
    grid = (NG * SG * KS + 7) // 8 * 8
    got = [host.host_tile_at(i, NG, SG, KS, bs) for i in range(grid)]
    want = sorted(g * 1000000 + s * 1000 + k for g in range(NG) for s in range(SG) for k in range(KS))
    assert sorted(v for v in got if v >= 0) == want
    per_xcd = [sum(v >= 0 for v in got[x::8]) for x in range(8)]
    assert max(per_xcd) <= (len(want) + 7) // 8


@pytest.mark.parametrize("NG,SG,KC,plan", [(20, 14, 432, 1206), (20, 14, 160, 1205), (20, 4, 432, 3), (17, 16, 96, 1503), (28, 14, 160, 1401), (20, 8, 160, 801), (20, 3, 432, 301)])
def test_last_sweeps_are_cut_along_k_where_a_round_would_be_partly_empty(host, NG, SG, KC, plan):
    host.host_tile_plan.argtypes = [C.c_int] * 4 + [C.c_long]
    assert host.host_tile_plan(NG, SG, KC, 1, 16 << 20) == plan
    assert host.host_tile_plan(NG, SG, KC, 0, 16 << 20) == SG * 100 + 1


def test_tile_plans_stay_within_the_scratch(host):
    host.host_tile_plan.argtypes = [C.c_int] * 4 + [C.c_long]
    for NG in range(1, 70):
        for SG in range(1, 17):
            for KC in (32, 64, 160, 257, 480):
                p = host.host_tile_plan(NG, SG, KC, 1, 16 << 20)
                whole, KS = p // 100, p % 100
                assert 0 <= whole <= SG and 1 <= KS <= 8 and (KS == 1) == (whole == SG)
                assert KS == 1 or (NG * (SG - whole) * 65536 * KS <= 16 << 20 and KC // KS >= 32)


def test_stream_splits_cover_k_and_fit_the_stage(host):
    for NB in (8, 56, 128, 192, 256, 320, 384, 448, 960):
        for KC in range(8, 481):
            for most in (512, 1024, 7680):
                p = host.host_stream_split(NB, KC, most)
                slices, tiles = p // 1000, p % 1000
                if slices == 0:
                    assert KC * 32 > most
                    continue
                assert slices in (1, 2, 4) and tiles * 32 <= most
                assert tiles * (slices - 1) < KC <= tiles * slices and (slices == 1 or tiles % 8 == 0)


@pytest.mark.parametrize("d,KV,layers,keys,pays", [(2048, 8, 16, 330, 1), (896, 2, 24, 330, 1), (4096, 8, 8, 1200, 1), (5120, 8, 48, 2048, 1), (1536, 2, 28, 330, 1),
                                                   (896, 2, 24, 1200, 0), (2048, 8, 1, 330, 0), (896, 2, 6, 330, 0), (2048, 8, 16, 4096, 0)])
def test_one_row_streams_where_that_is_faster(host, d, KV, layers, keys, pays):
    assert host.host_stream_pays(d, KV, layers, keys) == pays


@pytest.mark.parametrize("KC", [1, 7, 8, 9, 28, 31, 33, 34, 35, 37, 38, 64, 161])
@pytest.mark.parametrize("G,NB", [(256, (72, 56, 608, 56, 8192)), (256, (160, 128, 256, 128, 257)), (8, (3, 2, 9, 8, 8)), (8, (24, 17, 31, 1, 9))])
def test_stream_requests_stay_inside_the_matrices(host, KC, G, NB):
    """Every matrix of KC k tiles, whole or in two or four slices; the list ends inside the LM head or, for workgroups without a unit of it, before."""
    host.host_stream_list.restype = C.c_long
    ints = lambda v: (C.c_int * 5)(*v)
    for ks in range(3):
        tiles = KC if ks == 0 else (KC + (8 << ks) - 1) // (8 << ks) * 8
        if tiles * ((1 << ks) - 1) >= KC:
            continue
        cut = [ks, ks, 0, ks, 0]
        assert host.host_stream_list(2, ints(NB), ints([KC] * 5), ints(cut), ints([tiles if c else KC for c in cut]), G) == 0


def test_stream_stages_whole_slices(host):
    """A thread of the 512 that stage holds 3 x 4 columns of the residual stream and of the attention output, 8 x 4 of the SwiGLU products; every
    width of attention output the kernel is built for (heads x head_dim up to 15360), whatever d_model is."""
    taken = 0
    for hd, G in ((64, 4), (128, 4), (64, 7), (128, 3), (128, 5), (128, 6)):
        for KV in range(1, 33):
            if G * KV * hd > 15360:
                continue
            for d in list(range(256, 6145, 448)) + [2048, 3584, 4096, 6144]:
                for F in (1024, 14336, 15360):
                    cols = [host.host_stream_slice(d, G * KV, KV, hd, F, j) for j in range(5)]
                    taken += cols[0] > 0
                    assert max(cols[0], cols[1], cols[2], cols[4]) <= 3 * 4 * 512 and cols[3] <= 8 * 4 * 512, (hd, G, KV, d, F)
    assert taken > 1000
    assert host.host_stream_slice(4096, 56, 14, 128, 1024, 1) == 3584        # two slices where one of 7168 would fit the stage


@pytest.mark.parametrize("handles", [1, 2, 3, 8])
def test_persistent_launches_wait_for_each_other(host, handles):
    """A launch is queued behind all earlier ones on the device, whichever handle made them."""
    assert host.host_turns(handles, 60) == 0
    assert host.host_turn_refused() == 7


@pytest.mark.parametrize("N,K,four", [(27648, 896, 1), (27648, 2560, 1), (30720, 2944, 1), (24576, 896, 0), (24576, 2560, 0), (17920, 1536, 0), (27648, 2048, 0)])
def test_gate_up_of_two_token_blocks_where_four_row_blocks_are_faster(host, N, K, four):
    assert host.host_gate_up_by_four(N // 16, K // 32) == four


@pytest.mark.parametrize("d,F,KV,layers,keys,pays", [
    (896, 4864, 2, 24, 330, 1), (896, 1024, 2, 24, 330, 0), (896, 2048, 2, 24, 330, 0), (1024, 1024, 4, 40, 330, 0), (1024, 4864, 4, 24, 330, 1), (768, 512, 3, 24, 40, 0),
    (1536, 8960, 2, 28, 1200, 1), (1536, 4864, 2, 28, 1200, 0), (1536, 1024, 2, 28, 330, 0), (2048, 512, 4, 40, 330, 0), (2048, 8192, 8, 16, 2048, 1), (3072, 8192, 8, 28, 2048, 1), (3072, 512, 8, 24, 1200, 1),
    (4096, 512, 8, 40, 1200, 0), (4096, 14336, 8, 32, 2048, 1), (5120, 13824, 8, 48, 2048, 1)])
def test_one_row_does_not_stream_where_the_ffn_is_short(host, d, F, KV, layers, keys, pays):
    assert host.host_stream_pays_ffn(d, F, KV, layers, keys) == pays


@pytest.mark.parametrize("N,K,rows,rings,once", [
    (8192, 4096, 3, 1, 0), (8192, 2304, 16, 1, 0), (8192, 4096, 32, 1, 0), (8192, 2048, 32, 0, 0), (8192, 896, 3, 0, 0), (16384, 5120, 24, 1, 0), (16384, 5120, 64, 0, 0),
    (24000, 1024, 64, 0, 0), (24000, 4096, 12, 0, 1), (32000, 768, 3, 0, 1), (32000, 4096, 16, 0, 1), (40000, 2048, 3, 1, 0), (40000, 5120, 24, 1, 1), (50256, 4096, 24, 0, 1),
    (65536, 2048, 24, 0, 1), (81920, 2304, 12, 0, 1), (100000, 4096, 3, 1, 1), (100000, 3328, 12, 1, 1), (128256, 2048, 3, 0, 1), (128256, 2304, 3, 0, 1), (128256, 3072, 3, 1, 1),
    (128256, 3072, 32, 0, 1), (128256, 4096, 16, 0, 1), (151936, 896, 3, 0, 1), (151936, 1536, 3, 0, 1), (151936, 5120, 32, 0, 1), (151936, 5120, 64, 0, 1)])
def test_lm_heads_take_the_kernel_and_the_requests_measured_faster(host, N, K, rows, rings, once):
    TB = (rows + 15) // 16
    assert host.host_lm_by_rings(N // 16, K // 32, TB) == rings and host.host_lm_once(N // 16, K // 32) == once


@pytest.mark.parametrize("N,K,rg,slabs,once", [(27648, 5120, 7, 0, 1), (28672, 4096, 7, 0, 1), (16384, 896, 4, 0, 0), (4096, 2048, 4, 0, 0), (19456, 5120, 5, 0, 0), (20672, 3328, 6, 0, 0),
                                               (24576, 5120, 6, 0, 1), (5120, 13824, 8, 1, 1), (12288, 1536, 8, 1, 0), (7168, 5120, 8, 1, 0)])
def test_tiles_are_requested_as_measured_faster(host, N, K, rg, slabs, once):
    assert host.host_tiles_once(N // 16, K // 32, rg, slabs) == once


@pytest.mark.parametrize("N,K,rows,streamed", [(8192, 3072, 32, 0), (8208, 3072, 32, 1), (2048, 4096, 24, 0), (9728, 5120, 24, 1), (28672, 4096, 3, 1), (16384, 4096, 3, 0), (17920, 1536, 24, 0)])
def test_gate_up_of_few_rows_streams_where_that_is_faster(host, N, K, rows, streamed):
    assert host.host_gate_up_streamed(N // 16, K // 32, (rows + 15) // 16) == streamed

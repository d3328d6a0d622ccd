"""GPU: passes of every width class (1-2, 3-16, 17-32, 33-64, 65-128 rows and beyond) through models whose row-block counts
and depths of K leave remainders in every kernel's split, against the oracle."""
import numpy as np
import pytest

import oracle
import synth_inputs as si
from gpu_helpers import TOL_H, TOL_LOGIT, check_logits, make_pair

pytestmark = pytest.mark.gpu

# odd numbers of k tiles (11 and 13), row blocks that divide evenly by nothing (vocabulary: 513), fewer row blocks than
# compute units; 40 k tiles and a long K that is split (258 tiles); half a row block per compute unit at a long K (2048 x 8192)
ODD = si.ModelShape("odd-k", 2, 352, 11, 11, 416, 8208, 1e-5, 1e4)
LONG = si.ModelShape("long-k", 1, 1280, 10, 2, 8256, 8208, 1e-5, 1e4)
HALF = si.ModelShape("half-chip", 1, 2048, 16, 4, 8192, 1040, 1e-5, 1e4)
WIDE = si.ModelShape("wide-ffn", 1, 256, 4, 2, 15328, 1040, 1e-5, 1e4)          # 1916 row blocks in gate/up
WIDTHS = (1, 2, 3, 16, 17, 32, 33, 64, 70, 128, 131)


@pytest.mark.parametrize("small,large", [(ODD, LONG), (WIDE, HALF)], ids=lambda s: s.name)
def test_score_at_every_pass_width(small, large):
    """Logits within 2e-2 of the row maximum, entropy within 1e-2 nats (the tolerances of all bf16 parity tests)."""
    import paper_2502_06833_amd as ead
    Ws, Wl, os_, ol = make_pair(small, large, lm_sigma=1.5)
    e = ead.EAD(small, Ws, large, Wl, window=5, tau=0.0, d_min=4, max_batch=1, max_seq=160)
    toks = si.prompt_np(0, "widths", max(WIDTHS), small.vocab)
    for which, om in ((0, os_), (1, ol)):
        ref = om.forward_dense(toks)                     # causal: a shorter passage is a prefix
        Hr, ar = oracle.entropy_rows(ref)
        top = np.sort(ref, axis=1)[:, -2:]
        clear = top[:, 1] - top[:, 0] > 2 * TOL_LOGIT * np.abs(ref).max(axis=1)
        for T in WIDTHS:
            print(f"score model {which} width {T}", flush=True)
            out = e.score(which, toks[:T])
            check_logits(out["logits"], ref[:T], TOL_LOGIT)
            assert np.abs(out["H"] - Hr[:T]).max() < TOL_H
            assert (out["argmax"] == ar[:T])[clear[:T]].all()
            assert np.abs(oracle.entropy_rows(out["logits"])[0] - out["H"]).max() < 1e-4      # statistics against the logits they fold
            assert (out["logits"].argmax(1) == out["argmax"]).all()
    e.close()


def test_tiles_of_two_to_sixteen_blocks():
    """Every R x NT of narrow_plan (rules.hpp) that the shapes above do not reach: 192 row blocks at 33 to 150 rows (and one and two: K of 1056 and 3072), scored, and at
    200 as a prompt (four row blocks and four token blocks), whose first generated entropy hangs on it."""
    import paper_2502_06833_amd as ead
    small = si.ModelShape("mid-o", 1, 1056, 33, 11, 416, 1040, 1e-5, 1e4)          # 66 row blocks x 33 k tiles
    large = si.ModelShape("wide-o", 1, 3072, 24, 8, 512, 1040, 1e-5, 1e4)
    Ws, Wl, os_, ol = make_pair(small, large, lm_sigma=1.5)
    e = ead.EAD(small, Ws, large, Wl, window=5, tau=0.0, d_min=4, max_batch=1, max_seq=224)
    toks = si.prompt_np(0, "tiles", 201, small.vocab)
    for which, om in ((0, os_), (1, ol)):
        ref = om.forward_dense(toks)
        for T in (1, 2, 33, 49, 65, 97, 150):
            print(f"score model {which} width {T}", flush=True)
            check_logits(e.score(which, toks[:T])["logits"], ref[:T], TOL_LOGIT)
        out = e.replay([toks], np.array([[5]], np.int32), np.array([[which]], np.uint8))
        assert abs(out["H"][0, 0] - oracle.entropy_rows(ref[-1:])[0][0]) < TOL_H
    e.close()


class WideRow(si.ModelShape):
    """A model of few heads, so that rows of up to 15360 come with small matrices."""
    head_dim = 128


@pytest.mark.parametrize("d", [5152, 6176, 8192, 9248, 12320, 15360])
def test_rows_longer_than_the_models(d):
    """Normalised and packed rows of every length class past 5120 (three to eight pieces a thread, the last ones partly past the row's end):
    passes of 1, 3, 40 and 128 rows scored, and 300 as a prompt, whose first generated entropy hangs on it."""
    import paper_2502_06833_amd as ead
    shape = WideRow(f"row-{d}", 1, d, 4, 2, 64, 528, 1e-5, 1e4)
    other = si.ModelShape("row-other", 1, 128, 4, 4, 128, 528, 1e-5, 1e4)
    W, Wo, om, _ = make_pair(shape, other, gain_std=0.2, lm_sigma=1.5)
    e = ead.EAD(shape, W, other, Wo, window=5, tau=0.0, d_min=4, max_batch=1, max_seq=320)
    toks = si.prompt_np(0, "row", 301, shape.vocab)
    ref = om.forward_dense(toks)
    for T in (1, 3, 40, 128):
        check_logits(e.score(0, toks[:T])["logits"], ref[:T], TOL_LOGIT)
    out = e.replay([toks], np.array([[5]], np.int32), np.array([[0]], np.uint8))
    assert abs(out["H"][0, 0] - oracle.entropy_rows(ref[-1:])[0][0]) < TOL_H
    e.close()


@pytest.mark.parametrize("d,ffn", [(1408, 8192), (1440, 8224), (2048, 9728)])
def test_three_token_blocks_split_along_k(d, ffn):
    """Residual projections of two row blocks and four token blocks a workgroup, in four and five slabs of K, even and uneven: 33 to 48 rows scored."""
    import paper_2502_06833_amd as ead
    shape = WideRow(f"three-{d}", 1, d, 4, 2, ffn, 528, 1e-5, 1e4)
    other = si.ModelShape("three-other", 1, 128, 4, 4, 128, 528, 1e-5, 1e4)
    W, Wo, om, _ = make_pair(shape, other, gain_std=0.2, lm_sigma=1.5)
    e = ead.EAD(shape, W, other, Wo, window=5, tau=0.0, d_min=4, max_batch=1, max_seq=64)
    toks = si.prompt_np(0, "three", 48, shape.vocab)
    ref = om.forward_dense(toks)
    for T in (33, 40, 48):
        check_logits(e.score(0, toks[:T])["logits"], ref[:T], TOL_LOGIT)
    e.close()


@pytest.mark.parametrize("d,heads,kv,ffn", [(1056, 33, 11, 7200), (1312, 41, 41, 6176), (2176, 34, 17, 8160), (2048, 32, 8, 6144), (864, 27, 9, 8192)])
def test_one_row_in_uneven_slices(d, heads, kv, ffn):
    """k_linear_ring where the waves' slices of K differ by a tile, fill their groups partly and end inside an activation vector: 33, 41
    and 68 k tiles over four and eight waves, down projections of 192 to 256; one position scored (a single key, so that only V is
    rounded, to 2^-9) and 12 tokens of one row replayed."""
    import paper_2502_06833_amd as ead
    shape = si.ModelShape(f"one-{d}", 1, d, heads, kv, ffn, 1040, 1e-5, 1e4)
    other = si.ModelShape("one-other", 1, 128, 4, 4, 128, 1040, 1e-5, 1e4)
    W, Wo, om, _ = make_pair(shape, other, gain_std=0.2, lm_sigma=1.5)
    e = ead.EAD(shape, W, other, Wo, window=5, tau=0.0, d_min=4, max_batch=1, max_seq=32)
    toks = si.prompt_np(0, "one", 14, shape.vocab)
    ref = om.forward_dense(toks)
    check_logits(e.score(0, toks[:1])["logits"], ref[:1], 4e-3)
    out = e.replay([toks[:2]], toks[None, 2:], np.zeros((1, 12), np.uint8))
    assert np.abs(out["H"][0] - oracle.entropy_rows(ref[1:13])[0]).max() < TOL_H
    e.close()


@pytest.mark.parametrize("length", [64, 66, 171])
def test_logits_of_many_pieces_arrive_in_their_place(length):
    """Long logits reach the caller in pieces, by several threads (from 64 rows of this vocabulary on: a multiple of the piece,
    a remainder, and two passes): every row's statistics, folded on the device, are those of the row's logits."""
    import paper_2502_06833_amd as ead
    shape = si.ModelShape("pieces", 1, 256, 4, 2, 416, 32768, 1e-5, 1e4)
    Ws, Wl, os_, _ = make_pair(shape, si.ModelShape("other", 1, 128, 4, 4, 128, 32768, 1e-5, 1e4), lm_sigma=1.5)
    e = ead.EAD(shape, Ws, si.ModelShape("other", 1, 128, 4, 4, 128, 32768, 1e-5, 1e4), Wl, window=5, tau=0.0, d_min=4, max_batch=1, max_seq=192)
    toks = si.prompt_np(0, "pieces", length, shape.vocab)
    first = e.score(0, toks)
    again = e.score(0, toks)
    for out in (first, again):
        check_logits(out["logits"], os_.forward_dense(toks), TOL_LOGIT)
        assert np.abs(oracle.entropy_rows(out["logits"])[0] - out["H"]).max() < 1e-4
        assert (out["logits"].argmax(1) == out["argmax"]).all()
    assert (first["logits"] == again["logits"]).all()
    e.close()


def _score_into(e, toks, logits, H):
    import ctypes as C
    import paper_2502_06833_amd as ead
    t = np.ascontiguousarray(toks, np.int32)
    rc = ead.lib().ead_score(e._h, 0, t.ctypes.data_as(C.POINTER(C.c_int32)), t.size, C.cast(logits, C.POINTER(C.c_float)),
                             H.ctypes.data_as(C.POINTER(C.c_float)), None)
    assert rc == 0


def test_logits_into_pinned_memory():
    """A pinned destination, whole or from the middle of the allocation on, gets what a pageable one gets, and nothing beyond it."""
    import torch
    import paper_2502_06833_amd as ead
    shape = si.ModelShape("pinned", 1, 256, 4, 2, 416, 32768, 1e-5, 1e4)
    other = si.ModelShape("other", 1, 128, 4, 4, 128, 32768, 1e-5, 1e4)
    Ws, Wl, _, _ = make_pair(shape, other, lm_sigma=1.5)
    e = ead.EAD(shape, Ws, other, Wl, window=5, tau=0.0, d_min=4, max_batch=1, max_seq=192)
    for length in (40, 66, 171):
        toks = si.prompt_np(0, "pinned", length, shape.vocab)
        want = e.score(0, toks)
        n = length * shape.vocab
        for skip in (0, 48):
            buf = torch.full((n + 96,), -7.0, pin_memory=True)
            H = np.zeros(length, np.float32)
            _score_into(e, toks, buf.data_ptr() + 4 * skip, H)
            got = buf.numpy()
            assert (got[skip:skip + n].reshape(length, -1) == want["logits"]).all() and (H == want["H"]).all()
            assert (got[:skip] == -7.0).all() and (got[skip + n:] == -7.0).all()
    e.close()


def test_scoring_allocates_nothing():
    """Everything a handle needs is allocated when it is created: the first scoring call whose logits leave in pieces maps no
    further memory of the driver's (device or pinned) and leaves no thread behind."""
    import os
    import paper_2502_06833_amd as ead
    shape = si.ModelShape("maps", 1, 256, 4, 2, 416, 32768, 1e-5, 1e4)
    other = si.ModelShape("other", 1, 128, 4, 4, 128, 32768, 1e-5, 1e4)
    Ws, Wl, _, _ = make_pair(shape, other)
    e = ead.EAD(shape, Ws, other, Wl, window=5, tau=0.0, d_min=4, max_batch=1, max_seq=192)
    toks = si.prompt_np(0, "maps", 100, shape.vocab)
    logits, H = np.full(100 * shape.vocab, 1.0, np.float32), np.zeros(100, np.float32)

    def mapped():
        with open("/proc/self/maps") as f:
            rows = [ln.split() for ln in f if "/dev/dri" in ln]
        return sum(int(b, 16) - int(a, 16) for a, b in (r[0].split("-") for r in rows)), len(os.listdir("/proc/self/task"))

    _score_into(e, toks[:40], logits.ctypes.data, H)           # 5 MB: the runtime's copy, whose own staging memory comes with its first use
    before = mapped()
    _score_into(e, toks, logits.ctypes.data, H)
    assert mapped() == before
    e.close()


@pytest.mark.parametrize("batch", [3, 20, 40])
def test_sampled_choice_of_wide_passes(batch):
    """The sampled token of every row of a pass, where the two best perturbed scores are clearly apart."""
    import paper_2502_06833_amd as ead
    other = si.ModelShape("other", 1, 512, 4, 4, 512, ODD.vocab, 1e-5, 1e4)
    Ws, Wl, os_, ol = make_pair(ODD, other, lm_sigma=1.5)
    temperature, n = 0.8, 3
    prompts = [si.prompt_np(0, f"w{b}", 4 + b % 5, ODD.vocab) for b in range(batch)]
    forced = np.stack([si.prompt_np(1, f"w{b}", n, ODD.vocab) for b in range(batch)])
    mid = np.zeros((batch, n), np.uint8)
    mid[1::2, 1:] = 1
    e = ead.EAD(ODD, Ws, other, Wl, window=5, tau=0.0, d_min=2, max_batch=batch, max_seq=32)
    e.set_sampling(temperature, 77)
    rp = e.replay(prompts, forced, mid)
    checked = 0
    for b in range(batch):
        seq = np.concatenate([prompts[b], forced[b]])
        for i in range(n):
            lg = (ol if mid[b, i] else os_).forward_dense(seq[:len(prompts[b]) + i])[-1]
            sc = lg / temperature + oracle.gumbel(77, b, i, ODD.vocab)
            two = np.sort(sc)[-2:]
            if two[1] - two[0] > 2 * TOL_LOGIT * np.abs(lg).max() / temperature:
                checked += 1
                assert rp["choice"][b, i] == int(sc.argmax()), (b, i)
    assert checked >= batch                              # a third of the positions at least
    e.close()

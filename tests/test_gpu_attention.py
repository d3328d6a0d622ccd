"""Matrix-core attention (passes of many rows) at long contexts: several key splits, groups of
rows of one sequence that share a pass over its K/V, ragged group boundaries.  Narrow bf16
models keep the oracle fast; the weights are drawn wider than usual (std 0.05) so that the
attention weights are far from uniform and a wrong key or column mapping shows in the logits.
Head layouts: G = 2 with head dim 32 (8 rows per group) and G = 3 with head dim 64 (5 rows per
group); G = 4, 5, 7 with head dims 64 and 128 are covered at short contexts by the
depth-truncated pairs of test_gpu_models.py."""
import numpy as np
import pytest

import oracle
import synth_inputs as si
from gpu_helpers import make_pair

pytestmark = pytest.mark.gpu

TOL_LOGIT, TOL_H, BAND = 2e-2, 1e-2, 1e-2

ATT_S = si.ModelShape("att-s", 2, 256, 8, 4, 512, 512, 1e-5, 1e4, bf16=True)
ATT_L = si.ModelShape("att-l", 2, 384, 6, 2, 768, 512, 1e-5, 1e4, bf16=True)


@pytest.fixture(scope="module")
def att():
    import paper_2502_06833_amd as ead
    Ws = si.model_weights_torch(ATT_S, 0, "cuda", 0.05)
    Wl = si.model_weights_torch(ATT_L, 0, "cuda", 0.05)
    os_ = oracle.Model(ATT_S, {k: v.float().cpu().numpy() for k, v in Ws.items()})
    ol = oracle.Model(ATT_L, {k: v.float().cpu().numpy() for k, v in Wl.items()})
    e = ead.EAD(ATT_S, Ws, ATT_L, Wl, window=5, tau=0.0, d_min=16, max_batch=3, max_seq=1250)
    yield e, os_, ol
    e.close()


def test_long_context_scoring_against_oracle(att):
    """1100 teacher-forced positions per model in passes of 160 rows: every row group but the
    first and the last of a pass is full, contexts run from 1 to 1100 keys."""
    e, os_, ol = att
    toks = si.prompt_np(2, "att-long", 1100, ATT_S.vocab)
    for which, om in ((0, os_), (1, ol)):
        ref = om.forward_dense(toks)
        out = e.score(which, toks)
        err = np.abs(out["logits"] - ref).max(axis=1) / np.abs(ref).max(axis=1)
        Hr, ar = oracle.entropy_rows(ref)
        print(f"model {which}: logits rel err {err.max():.2e}, H err {np.abs(out['H'] - Hr).max():.2e}, "
              f"H range {Hr.min():.2f}..{Hr.max():.2f}", flush=True)
        assert err.max() < TOL_LOGIT
        assert np.abs(out["H"] - Hr).max() < TOL_H
        top2 = np.sort(ref, axis=1)
        clear = (top2[:, -1] - top2[:, -2]) > 2 * TOL_LOGIT * np.abs(ref).max(axis=1)
        assert (out["argmax"][clear] == ar[clear]).all()
        assert Hr.max() - Hr.min() > 0.05            # the attention is not uniform: the test can see a wrong key


def test_catchups_over_several_key_splits_against_oracle(att):
    """Prompts of 1100, 700 and 37 tokens decoded together along the oracle's trajectories: every
    switch makes the other model catch up 16 or more rows at contexts beyond 1024 keys (three key
    splits of 512, merged by the last workgroup to arrive; row groups cut at multiples of 8 and 5)."""
    e, os_, ol = att
    prompts = [si.prompt_np(3, f"att{b}", n, ATT_S.vocab) for b, n in enumerate((1100, 700, 37))]
    n_new, d_min = 56, 16
    probe = oracle.generate(os_, ol, prompts[0], n_new, 5, 1e30, d_min=d_min)
    tau = float(np.percentile(probe["Hbar"], 45))
    refs = [oracle.generate(os_, ol, p, n_new, 5, tau, d_min=d_min) for p in prompts]
    print("large share per row:", [float(r["model_id"].mean()) for r in refs], flush=True)
    assert any(0.0 < r["model_id"].mean() < 1.0 for r in refs)         # at least one row switches
    e.set_gate(5, tau, d_min)
    rp = e.replay(prompts, np.stack([r["tokens"] for r in refs]), np.stack([r["model_id"] for r in refs]))
    for b, r in enumerate(refs):
        print(f"  row {b}: H err {np.abs(rp['H'][b] - r['H']).max():.2e}", flush=True)
        assert np.abs(rp["H"][b] - r["H"]).max() < TOL_H
        assert np.abs(rp["Hbar"][b] - r["Hbar"]).max() < TOL_H
        safe = np.abs(r["Hbar"] - tau) > BAND
        want_next = np.concatenate([r["model_id"][1:], rp["next_model"][b][-1:]])
        assert (rp["next_model"][b][safe] == want_next[safe]).all()
    st = e.stats()
    assert st["catchup_rows_large"] >= 16


@pytest.mark.parametrize("heads,kv_heads", [(4, 4), (8, 1), (16, 2)])
def test_head_layouts_at_the_ends_of_the_range(heads, kv_heads):
    """G = 1 (16 rows of a sequence per pass over its K/V), G = 8 (2 rows), and G = 8
    with two KV heads at 16 query heads: 300 teacher-forced positions against the oracle."""
    import paper_2502_06833_amd as ead
    shape = si.ModelShape(f"att-{heads}-{kv_heads}", 2, 32 * heads, heads, kv_heads, 256, 512, 1e-5, 1e4, bf16=True)
    W = si.model_weights_torch(shape, 1, "cuda", 0.05)
    om = oracle.Model(shape, {k: v.float().cpu().numpy() for k, v in W.items()})
    e = ead.EAD(shape, W, shape, W, window=5, tau=0.0, d_min=4, max_batch=1, max_seq=320)
    toks = si.prompt_np(5, shape.name, 300, shape.vocab)
    ref = om.forward_dense(toks)
    out = e.score(1, toks)
    err = np.abs(out["logits"] - ref).max(axis=1) / np.abs(ref).max(axis=1)
    Hr, _ = oracle.entropy_rows(ref)
    print(f"{shape.name}: logits rel err {err.max():.2e}, H err {np.abs(out['H'] - Hr).max():.2e}", flush=True)
    assert err.max() < TOL_LOGIT
    assert np.abs(out["H"] - Hr).max() < TOL_H
    e.close()


@pytest.mark.parametrize("heads,kv_heads,hd,rows,lens", [(8, 8, 128, 12, (1003, 897, 30, 520)), (8, 4, 32, 24, (1750, 1409, 733, 60)),
                                                         (16, 8, 64, 16, (1700, 31, 1000, 851))])
def test_decode_rows_in_two_key_splits(heads, kv_heads, hd, rows, lens):
    """96 to 128 (row, KV head) pairs at contexts beyond 896 (head dims below 128: 1664) keys: two splits of an odd number
    of key blocks, short rows that reach only the first."""
    import paper_2502_06833_amd as ead
    shape = si.ModelShape(f"two-{heads}-{kv_heads}-{hd}", 1, heads * hd, heads, kv_heads, 256, 512, 1e-5, 1e4, bf16=True)
    W = si.model_weights_torch(shape, 1, "cuda", 0.05)
    om = oracle.Model(shape, {k: v.float().cpu().numpy() for k, v in W.items()})
    e = ead.EAD(shape, W, shape, W, window=5, tau=0.0, d_min=4, max_batch=rows, max_seq=max(lens) + 8)
    seqs = [si.prompt_np(7, f"two{n}", n + 4, shape.vocab) for n in lens]
    refs = [oracle.entropy_rows(om.forward_dense(q[:-1]))[0][n - 1:] for q, n in zip(seqs, lens)]
    which = [b % len(lens) for b in range(rows)]
    rp = e.replay([seqs[i][:lens[i]] for i in which], np.stack([seqs[i][lens[i]:] for i in which]), np.zeros((rows, 4), np.uint8))
    for b, i in enumerate(which):
        assert np.abs(rp["H"][b] - refs[i]).max() < TOL_H, (b, lens[i])
    e.close()


@pytest.mark.parametrize("heads,kv,hd", [(8, 8, 32), (4, 2, 64), (6, 2, 128), (4, 1, 32), (5, 1, 128), (6, 1, 64), (7, 1, 64), (8, 1, 128), (4, 1, 128)])
def test_prompt_attention_of_every_head_layout(heads, kv, hd):
    """k_attn_prompt: rows cut at multiples of 8 (eight heads share K and V) to 64 positions, last key blocks and last groups partly
    filled.  Prompts of several lengths in one pass (first, middle and last rows of a group), whose first generated entropy hangs on
    every cached key; and passes of the same rows scored, through k_attn_mfma."""
    import paper_2502_06833_amd as ead
    shape = si.ModelShape(f"pa{heads}-{hd}", 2, heads * hd, heads, kv, 256, 512, 1e-5, 1e4, bf16=True)
    tiny = si.ModelShape("pa-other", 1, 128, 4, 4, 128, 512, 1e-5, 1e4, bf16=True)
    W, Wt = si.model_weights_torch(shape, 0, "cuda", 0.05), si.model_weights_torch(tiny, 0, "cuda", 0.05)
    om = oracle.Model(shape, {k: v.float().cpu().numpy() for k, v in W.items()})
    lens = (700, 33, 290, 2, 96, 511)
    e = ead.EAD(shape, W, tiny, Wt, window=5, tau=0.0, d_min=4, max_batch=len(lens), max_seq=704)
    toks = si.prompt_np(4, "pa", 160, 512)
    ref = om.forward_dense(toks)
    for T in (17, 33, 129, 160):
        out = e.score(0, toks[:T])
        assert (np.abs(out["logits"] - ref[:T]).max(axis=1) < TOL_LOGIT * np.abs(ref[:T]).max(axis=1)).all(), T
    e.force_model(0)
    prompts = [si.prompt_np(5, f"pa{n}", n, 512) for n in lens]
    got = e.generate(prompts, 1)
    for b, p in enumerate(prompts):
        assert abs(got["H"][b, 0] - oracle.entropy_rows(om.forward_dense(p)[-1:])[0][0]) < TOL_H, lens[b]
    e.close()


@pytest.mark.parametrize("heads,kv,hd", [(8, 8, 32), (4, 2, 64), (6, 2, 128), (4, 1, 32), (5, 1, 128), (6, 1, 64), (7, 1, 64), (8, 1, 128)])
def test_prompt_attention_from_inside_a_group(heads, kv, hd):
    """k_attn_prompt in passes that start inside a group of rows (leading waves idle, leading columns of a wave masked) and end at each of
    a group's rows: one model generates n tokens after a prompt of 45, then the other takes over and catches up n + 1 rows.  One layer, so
    that the entropy there hangs on the pass's last row, whose attention is the only thing that scoring the same tokens does in another
    kernel (k_attn_mfma).  The LM head of one row keeps float32 activations and that of a scoring pass rounds them to 11 bits, 2e-4 each over
    512 logits of deviation 1.5: 5e-4 between the two seen, 1e-3 allowed; one wrong key moves them by 1e-2 and more in the median, the worst of a case by 0.09."""
    import paper_2502_06833_amd as ead
    shape = si.ModelShape(f"pc{heads}-{hd}", 1, heads * hd, heads, kv, 256, 512, 1e-5, 1e4, bf16=True)
    tiny = si.ModelShape("pc-other", 1, 128, 4, 4, 128, 512, 1e-5, 1e4, bf16=True)
    W, Wt, om, _ = make_pair(shape, tiny, lm_sigma=1.5)
    e = ead.EAD(shape, W, tiny, Wt, window=5, tau=0.0, d_min=4, max_batch=1, max_seq=160)
    toks = si.prompt_np(6, "inside", 160, 512)
    ref = oracle.entropy_rows(om.forward_dense(toks))[0]
    scored = e.score(0, toks)["H"]
    worst = 0.0
    for n in range(max(17, 65 // kv), min(max(17, 65 // kv) + 66, 114)):
        mids = np.ones((1, n + 1), np.uint8)
        mids[0, n] = 0
        H = e.replay([toks[:45]], toks[None, 45:45 + n + 1], mids)["H"][0, n]
        worst = max(worst, abs(H - scored[44 + n]))
        assert abs(H - ref[44 + n]) < TOL_H, n
    print(f"heads {heads} kv {kv} hd {hd}: {worst:.1e} from scoring", flush=True)
    assert worst < 1e-3
    e.close()

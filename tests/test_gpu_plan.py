"""GPU: the row plan and the finalisation kernel where their per-sequence work wraps around (more than 64
sequences, more prompt positions than a pass takes, windows longer than a workgroup), against the oracle."""
import numpy as np
import pytest

import oracle
import synth_inputs as si

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("batch,w,n,hi", [(64, 5, 14, 40), (65, 5, 14, 40), (130, 3, 14, 24), (1, 300, 290, 8)])
def test_wide_batches_and_long_windows_follow_the_oracle(batch, w, n, hi):
    import paper_2502_06833_amd as ead
    ss, sl = si.TINY_S, si.TINY_L
    Ws, Wl = si.model_weights_torch(ss, 0, "cuda"), si.model_weights_torch(sl, 0, "cuda")
    os_ = oracle.Model(ss, {k: v.float().cpu().numpy() for k, v in Ws.items()})
    ol = oracle.Model(sl, {k: v.float().cpu().numpy() for k, v in Wl.items()})
    prompts = [si.prompt_np(0, f"plan{b}", 1 + (b * 7) % hi, ss.vocab) for b in range(batch)]
    probe = oracle.generate(os_, ol, prompts[batch // 2], n, w, 1e30)
    tau = float(np.percentile(probe["Hbar"], 50))
    e = ead.EAD(ss, Ws, sl, Wl, window=w, tau=tau, d_min=4, max_batch=batch, max_seq=max(32, hi + n))
    # every row along the oracle's trajectory: fp32 sums of at most 1024 terms in another order (1e-4 nats as for
    # the fp32 pair elsewhere)
    rows = range(batch) if batch == 1 else sorted({0, 1, 62, 63, batch - 2, batch - 1, batch // 3})
    refs = {b: oracle.generate(os_, ol, prompts[b], n, w, tau, d_min=4) for b in rows}
    tok = np.stack([refs[b]["tokens"] if b in refs else refs[0]["tokens"] for b in range(batch)])
    mid = np.stack([refs[b]["model_id"] if b in refs else refs[0]["model_id"] for b in range(batch)])
    rp = e.replay(prompts, tok, mid)
    for b in rows:
        assert np.abs(rp["H"][b] - refs[b]["H"]).max() < 1e-4, b
        assert np.abs(rp["Hbar"][b] - refs[b]["Hbar"]).max() < 1e-4, b
        assert (rp["argmax"][b] == refs[b]["tokens"]).all(), b
    e.close()


def test_prompts_of_many_sequences_cut_between_passes():
    """130 prompts of 20-79 tokens, 6300 positions to consume: more than a prompt pass takes (4096 rows), so both models take two
    passes of about equal length and the cut falls inside a sequence beyond the first 64, whose rows, like its
    neighbours' and the last sequences', follow the oracle (tolerance as above)."""
    import paper_2502_06833_amd as ead
    ss, sl = si.TINY_S, si.TINY_L
    Ws, Wl = si.model_weights_torch(ss, 0, "cuda"), si.model_weights_torch(sl, 0, "cuda")
    os_ = oracle.Model(ss, {k: v.float().cpu().numpy() for k, v in Ws.items()})
    ol = oracle.Model(sl, {k: v.float().cpu().numpy() for k, v in Wl.items()})
    batch, n, w = 130, 6, 3
    prompts = [si.prompt_np(0, f"cut{b}", 20 + (b * 7) % 60, ss.vocab) for b in range(batch)]
    ends = np.cumsum([len(p) - 1 for p in prompts])
    assert 4096 < ends[-1] <= 2 * 4096
    first = -(-(ends[-1] // 2 + ends[-1] % 2) // 256) * 256              # rows of the first pass
    cut = int(np.searchsorted(ends, first, side="right"))
    assert cut >= 64 and ends[cut] > first > ends[cut - 1]
    e = ead.EAD(ss, Ws, sl, Wl, window=w, tau=0.0, d_min=4, max_batch=batch, max_seq=96)
    forced = np.stack([si.prompt_np(1, f"cut{b}", n, ss.vocab) for b in range(batch)])
    mid = np.zeros((batch, n), np.uint8)
    mid[:, 3:] = 1
    rp = e.replay(prompts, forced, mid)
    for b in sorted({0, 63, 64, cut - 1, cut, cut + 1, 127, 128, batch - 1}):
        seq = np.concatenate([prompts[b], forced[b]])
        for which, om in ((0, os_), (1, ol)):
            H, am = oracle.entropy_rows(om.forward_dense(seq[:-1])[len(prompts[b]) - 1:])
            at = mid[b] == which
            assert np.abs(rp["H"][b] - H)[at].max() < 1e-4, (b, which)
            assert (rp["argmax"][b] == am)[at].all(), (b, which)
    e.close()


def test_results_of_a_batch_that_takes_several_fetch_rounds():
    """40 sequences of up to 8192 tokens exceed the staging buffer of one round (36 rows): same results as with room for
    64 tokens, bit for bit."""
    import paper_2502_06833_amd as ead
    ss, sl = si.TINY_S, si.TINY_L
    Ws, Wl = si.model_weights_torch(ss, 0, "cuda"), si.model_weights_torch(sl, 0, "cuda")
    prompts = [si.prompt_np(0, f"fetch{b}", 1 + b % 9, ss.vocab) for b in range(40)]
    got = []
    for room in (64, 8192):
        e = ead.EAD(ss, Ws, sl, Wl, window=5, tau=6.2, d_min=2, max_batch=40, max_seq=room)
        got.append(e.generate(prompts, 11))
        e.close()
    for k in got[0]:
        assert (got[0][k] == got[1][k]).all(), k
    assert (got[0]["lens"] == 11).all()

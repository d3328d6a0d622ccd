"""Parity at the benchmark's full sizes and in its launch configuration.

The oracle can afford a few positions of the full-depth Llama-shaped pair (its fp32 weights
take 35 GB of host memory), so logits / entropy / arg max are compared there position by
position; everything longer is checked through properties that hold at any size (catch-up
invariance, batch independence) or on depth-truncated pairs (same widths, heads and vocab).
"""
import math

import numpy as np
import pytest
import torch

import oracle
import synth_inputs as si

pytestmark = pytest.mark.gpu

TOL_LOGIT, TOL_H, BAND = 2e-2, 1e-2, 1e-2


def _ead():
    import paper_2502_06833_amd as ead
    return ead


@pytest.fixture(scope="module")
def llama_full():
    ead = _ead()
    ss, sl = si.PAIRS["llama"]
    Ws = si.model_weights_torch(ss, 0, "cuda")
    Wl = si.model_weights_torch(sl, 0, "cuda")
    e = ead.EAD(ss, Ws, sl, Wl, window=5, tau=0.0, d_min=10, max_batch=2, max_seq=640)
    yield e, Ws, Wl
    e.close()


def test_llama_full_depth_sampled_positions_against_oracle(llama_full):
    e, Ws, Wl = llama_full
    ss, sl = si.PAIRS["llama"]
    toks = si.prompt_np(0, "full", 5, ss.vocab)
    for which, shape, W in ((0, ss, Ws), (1, sl, Wl)):
        print(f"full-depth {shape.name}: oracle on {len(toks)} positions", flush=True)
        om = oracle.Model(shape, {k: v.float().cpu().numpy() for k, v in W.items()})
        ref = om.forward_dense(toks)
        del om
        for n in (len(toks), 2):                 # 5 rows: MFMA kernels; 2 rows: FMA kernels
            out = e.score(which, toks[:n])
            err = np.abs(out["logits"] - ref[:n]).max(axis=1) / np.abs(ref[:n]).max(axis=1)
            Hr, ar = oracle.entropy_rows(ref[:n])
            rms = float(np.sqrt(np.mean((out["logits"] - ref[:n]) ** 2) / np.mean(ref[:n] ** 2)))
            print(f"  rows={n}: logits rel err {err.max():.2e} (RMS-relative {rms:.2e}), H err {np.abs(out['H'] - Hr).max():.2e}", flush=True)
            assert err.max() < TOL_LOGIT
            assert np.abs(out["H"] - Hr).max() < TOL_H
            top2 = np.sort(ref[:n], axis=1)
            clear = (top2[:, -1] - top2[:, -2]) > 2 * TOL_LOGIT * np.abs(ref[:n]).max(axis=1)
            assert (out["argmax"][clear] == ar[clear]).all()
        sigma = 0.02 * math.sqrt(shape.d_model)          # logits ~ N(0, sigma^2): H ~ ln V - sigma^2/2
        assert abs(Hr.mean() - (math.log(shape.vocab) - sigma * sigma / 2)) < 0.1


def test_qwen_full_depth_sampled_positions_against_oracle():
    """The Qwen-0.5B / Qwen-14B shaped pair at full depth (48 layers of width 5120; G = 7 and 5):
    logits, entropy and arg max of a few positions against the oracle, through the MFMA kernels
    (5 rows) and the FMA kernels (2 rows); then four rows decoded together against the same
    rows decoded alone (the batched workload's launch configuration)."""
    ead = _ead()
    ss, sl = si.PAIRS["qwen"]
    Ws = si.model_weights_torch(ss, 0, "cuda")
    Wl = si.model_weights_torch(sl, 0, "cuda")
    e = ead.EAD(ss, Ws, sl, Wl, window=5, tau=0.0, d_min=3, max_batch=4, max_seq=96)
    toks = si.prompt_np(0, "qfull", 5, ss.vocab)
    for which, shape, W in ((0, ss, Ws), (1, sl, Wl)):
        print(f"full-depth {shape.name}: oracle on {len(toks)} positions", flush=True)
        om = oracle.Model(shape, {k: v.float().cpu().numpy() for k, v in W.items()})
        ref = om.forward_dense(toks)
        del om
        for n in (len(toks), 2):
            out = e.score(which, toks[:n])
            err = np.abs(out["logits"] - ref[:n]).max(axis=1) / np.abs(ref[:n]).max(axis=1)
            Hr, ar = oracle.entropy_rows(ref[:n])
            rms = float(np.sqrt(np.mean((out["logits"] - ref[:n]) ** 2) / np.mean(ref[:n] ** 2)))
            print(f"  rows={n}: logits rel err {err.max():.2e} (RMS-relative {rms:.2e}), H err {np.abs(out['H'] - Hr).max():.2e}", flush=True)
            assert err.max() < TOL_LOGIT
            assert np.abs(out["H"] - Hr).max() < TOL_H
            top2 = np.sort(ref[:n], axis=1)
            clear = (top2[:, -1] - top2[:, -2]) > 2 * TOL_LOGIT * np.abs(ref[:n]).max(axis=1)
            assert (out["argmax"][clear] == ar[clear]).all()
    del Ws, Wl
    torch.cuda.empty_cache()
    prompts = [si.prompt_np(1, f"qrow{b}", n, ss.vocab) for b, n in enumerate((40, 9, 64, 23))]
    e.set_gate(5, 11.7525, 3)
    both = e.generate(prompts, 10)
    for b, p in enumerate(prompts):
        one = e.generate([p], 10)
        assert np.abs(one["H"][0] - both["H"][b]).max() < TOL_H
    e.close()


def test_qwen_full_depth_wide_passes_and_what_the_bf16_cache_costs():
    """The 14B-shaped model at full depth through passes of 72, 40, 5 and 2 rows (fetching-wave kernels with five
    and four token blocks, narrow matrix-core kernels, FMA kernels) against the oracle on 72 positions.

    What holds at every position: the entropy within 1e-2 nats, and the same logits whichever pass computed
    them (passes served by one kernel family agree bit for bit; families differ by the order of their fp32
    sums and by where the half-precision rounding of the matrix-core kernels' activations falls, amplified by
    48 layers to 7e-3 of the row maximum, several times below the error against the oracle).  The logits
    themselves stay within 2e-2 of
    the row maximum only for the first positions: the kernels keep K and V in bf16 (the oracle in fp32), each
    cached element carries a relative rounding error of up to 2^-9 (1.1e-3 rms), a layer's attention output
    inherits about 2.5e-3 of that through scores and values, and 48 layers of a randomly initialised network
    add up and amplify it to 2.5-3.5e-2 rms of the logits from about 20 cached positions on -- by the same
    amount position by position in every pass width, which is what identifies the cache and not a kernel.
    The bound asserted for those positions is 6e-2."""
    ead = _ead()
    ss, sl = si.PAIRS["qwen"]
    Ws = si.model_weights_torch(ss.truncated(1), 0, "cuda")        # the small model is not under test here
    Wl = si.model_weights_torch(sl, 0, "cuda")
    e = ead.EAD(ss.truncated(1), Ws, sl, Wl, window=5, tau=0.0, d_min=3, max_batch=1, max_seq=96)
    toks = si.prompt_np(0, "qwide", 72, ss.vocab)
    print("full-depth qwen-14b: oracle on 72 positions", flush=True)
    om = oracle.Model(sl, {k: v.float().cpu().numpy() for k, v in Wl.items()})
    ref = om.forward_dense(toks)
    del om
    Hr, ar = oracle.entropy_rows(ref)
    top = np.abs(ref).max(axis=1)
    outs = {}
    for n in (72, 40, 5, 2):
        out = outs[n] = e.score(1, toks[:n])
        err = np.abs(out["logits"] - ref[:n]).max(axis=1) / top[:n]
        print(f"  rows={n}: logits err / row max: first 5 positions {err[:5].max():.2e}, all {err.max():.2e}; "
              f"H err {np.abs(out['H'] - Hr[:n]).max():.2e}", flush=True)
        assert np.abs(out["H"] - Hr[:n]).max() < TOL_H
        assert err[:5].max() < TOL_LOGIT
        assert err.max() < 6e-2
        gap = np.sort(ref[:n], axis=1)
        clear = (gap[:, -1] - gap[:, -2]) > 2 * 6e-2 * top[:n]
        assert (out["argmax"][clear] == ar[:n][clear]).all()
    for n in (40, 5, 2):                                       # the same logits whichever pass computed them
        d = np.abs(outs[72]["logits"][:n] - outs[n]["logits"]).max(axis=1) / top[:n]
        print(f"  72-row pass against {n}-row pass: {d.max():.2e} of the row maximum", flush=True)
        assert d.max() < 1e-2
    e.close()


def test_llama_full_size_catchup_and_paths_agree(llama_full):
    """512-token prompt, the benchmark's launch configuration: after 10 small-model tokens the
    large model catches up (11 rows through the MFMA kernels); its entropy there equals the
    one it gives when scoring the same tokens from scratch; the fused single-row kernel and
    the per-layer kernels agree."""
    e, _, _ = llama_full
    ss, _ = si.PAIRS["llama"]
    prompt = si.prompt_np(0, "row0", 512, ss.vocab)
    e.set_gate(5, 0.0, 10)
    outs = []
    for fused in (False, 1, 2):            # per-layer kernels; streamed persistent kernel; register-buffered one
        e.set_fused(fused)
        outs.append(e.generate([prompt], 14))
    e.set_fused(False)
    a, b, c = outs
    assert list(a["model_id"][0]) == [0] * 10 + [1] * 4
    assert np.abs(a["H"] - b["H"]).max() < TOL_H
    assert np.abs(a["H"] - c["H"]).max() < TOL_H
    seq = np.concatenate([prompt, a["tokens"][0]])
    sc = e.score(1, seq[:-1], want_logits=False)
    for i in range(10, 14):
        assert abs(sc["H"][512 + i - 1] - a["H"][0, i]) < TOL_H
    st = e.stats()
    assert st["tokens_small"] == 10 and st["tokens_large"] == 4


def test_llama_full_size_batch_rows_independent(llama_full):
    e, _, _ = llama_full
    ss, _ = si.PAIRS["llama"]
    prompts = [si.prompt_np(0, "row0", 300, ss.vocab), si.prompt_np(1, "row1", 77, ss.vocab)]
    tau = 11.3526
    e.set_gate(5, tau, 3)
    both = e.generate(prompts, 12)
    assert both["model_id"].min() == 0 and both["model_id"].max() == 1          # rows switch, at different steps
    # each row alone along the trajectory it took in the batch (a free-running single run may take the
    # other branch where a window mean falls on the threshold to the last bit): the same entropies,
    # and the same decisions wherever the mean is not within rounding of the threshold
    for b, p in enumerate(prompts):
        one = e.replay([p], both["tokens"][b], both["model_id"][b])
        assert np.abs(one["H"][0] - both["H"][b]).max() < TOL_H
        assert np.abs(one["Hbar"][0] - both["Hbar"][b]).max() < TOL_H
        clear = np.abs(both["Hbar"][b] - tau)[:-1] > 1e-3
        assert (one["next_model"][0][:-1][clear] == both["model_id"][b][1:][clear]).all()


def test_qwen_truncated_batch_with_ragged_prompts_and_catchups():
    """Qwen-shaped widths (2 layers each), 8 rows with prompts of 5-40 tokens decoded together:
    rows switch at different times, so small- and large-model rows mix within a step and each
    row gets its own catch-up.  Four rows are checked against the oracle token by token."""
    ead = _ead()
    ss, sl = (s.truncated(2) for s in si.PAIRS["qwen"])
    Ws = si.model_weights_torch(ss, 0, "cuda")
    Wl = si.model_weights_torch(sl, 0, "cuda")
    os_ = oracle.Model(ss, {k: v.float().cpu().numpy() for k, v in Ws.items()})
    ol = oracle.Model(sl, {k: v.float().cpu().numpy() for k, v in Wl.items()})
    B, n_new, d_min = 8, 20, 3
    lens = si.prompt_lengths(3, B, 5, 40)
    prompts = [si.prompt_np(3, f"q{b}", int(lens[b]), ss.vocab) for b in range(B)]
    probe = oracle.generate(os_, ol, prompts[0], n_new, 5, 1e30, d_min=d_min)
    tau = float(np.percentile(probe["Hbar"], 40))
    checked = [0, 2, 5, 7]
    refs = {b: oracle.generate(os_, ol, prompts[b], n_new, 5, tau, d_min=d_min) for b in checked}
    print("large share per checked row:", [float(refs[b]["model_id"].mean()) for b in checked], flush=True)
    e = ead.EAD(ss, Ws, sl, Wl, window=5, tau=tau, d_min=d_min, max_batch=B, max_seq=64)
    free = e.generate(prompts, n_new)                    # mixed small/large rows, device-side decisions
    st = e.stats()
    assert st["tokens_small"] + st["tokens_large"] == B * n_new
    assert st["catchup_rows_large"] > 0
    # teacher-forced along the oracle trajectories (unchecked rows replay the GPU's own run)
    ft = free["tokens"].copy(); fm = free["model_id"].copy()
    for b in checked:
        ft[b], fm[b] = refs[b]["tokens"], refs[b]["model_id"]
    rp = e.replay(prompts, ft, fm)
    n_dec = 0
    for b in checked:
        r = refs[b]
        assert np.abs(rp["H"][b] - r["H"]).max() < TOL_H, b
        assert np.abs(rp["Hbar"][b] - r["Hbar"]).max() < TOL_H, b
        safe = np.abs(r["Hbar"] - tau) > BAND
        want_next = np.concatenate([r["model_id"][1:], rp["next_model"][b][-1:]])
        assert (rp["next_model"][b][safe] == want_next[safe]).all(), b
        n_dec += int(safe.sum())
    print(f"decisions checked outside the band: {n_dec}/{len(checked) * n_new}", flush=True)
    # unchecked rows: replaying the GPU's own trajectory reproduces its entropies
    for b in range(B):
        if b not in checked:
            assert np.abs(rp["H"][b] - free["H"][b]).max() < 2e-3
    # the grouped schedule (small-model rows run ahead, large-model rows served together)
    # replays the same trajectories to the same entropies and decisions
    e.set_schedule(True, 0.5, 0.25)
    rg = e.replay(prompts, ft, fm)
    sg = e.stats()
    assert sg["tokens_small"] + sg["tokens_large"] == B * n_new
    for b in checked:
        r = refs[b]
        assert np.abs(rg["H"][b] - r["H"]).max() < TOL_H, b
        safe = np.abs(r["Hbar"] - tau) > BAND
        want_next = np.concatenate([r["model_id"][1:], rg["next_model"][b][-1:]])
        assert (rg["next_model"][b][safe] == want_next[safe]).all(), b
    assert np.abs(rg["H"] - rp["H"]).max() < 2e-3
    lock_large, grouped_large = st["steps_large"], sg["steps_large"]
    print(f"large-model passes: lock step {lock_large}, grouped {grouped_large}", flush=True)
    e.close()


def test_qwen_truncated_1024_row_prefill_against_oracle():
    """Qwen-shaped widths (2 layers each, gains 1 + N(0, 0.3^2)): a 1025-token prompt is prefilled in one pass of
    1024 rows per model (four sweeps of 256 x 256 tiles through the gate/up matrices, of 128 x 256 tiles through the
    large model's others, eight 128-row sweeps through the small model's others; attention over up to 1024 keys in row groups); then
    Algorithm 1 runs along the oracle's own trajectory: ten small-model tokens, the large model's catch-up of
    eleven rows on top of its 1024 cached positions, two large-model tokens.  Entropies, window means and clear
    arg maxes of all twelve tokens against the oracle."""
    from gpu_helpers import check_replay_row, make_pair, trajectory_logit_stats
    ead = _ead()
    ss, sl = (s.truncated(2) for s in si.PAIRS["qwen"])
    Ws, Wl, os_, ol = make_pair(ss, sl, seed=6, gain_std=0.3, lm_sigma=1.5)
    prompt = si.prompt_np(6, "q1025", 1025, ss.vocab)
    print("1024-row prefill: oracle run over 1037 positions", flush=True)
    ref = oracle.generate(os_, ol, prompt, 12, 5, 0.0, d_min=10)
    assert list(ref["model_id"]) == [0] * 10 + [1] * 2
    stats = trajectory_logit_stats(os_, ol, prompt, ref["tokens"], ref["model_id"])
    e = ead.EAD(ss, Ws, sl, Wl, window=5, tau=0.0, d_min=10, max_batch=1, max_seq=1056)
    rp = e.replay([prompt], ref["tokens"], ref["model_id"])
    n_dec, n_arg = check_replay_row(rp, 0, ref, 0.0, 12, stats)
    print(f"  H err {np.abs(rp['H'][0] - ref['H']).max():.2e}; decisions checked {n_dec}/12, clear arg maxes {n_arg}/12", flush=True)
    assert n_dec == 12                                   # tau = 0: every window mean is far from the threshold
    free = e.generate([prompt], 12)
    assert list(free["model_id"][0]) == [0] * 10 + [1] * 2
    assert np.abs(free["H"][0, :1] - ref["H"][:1]).max() < TOL_H     # the first token follows the prefill directly
    e.close()


def test_ragged_row_block_counts_in_a_1024_row_prefill_against_oracle():
    """Widths whose row-block counts are not multiples of what a workgroup takes (gate/up of the large model: 740
    row blocks in groups of 16 through the 256 x 256 tiles; the small model's: 372 row blocks in groups of 8 through the 128 x 256
    tiles): the last group of these launches holds row blocks that do not exist (128-row sweeps with such a group:
    test_gpu_long_prefill.py).  A 1025-token prompt is prefilled in one pass of 1024 rows per model and
    Algorithm 1 then runs along the oracle's trajectory (ten small-model tokens, the large model's catch-up,
    two large-model tokens); entropies, window means and clear arg maxes against the oracle."""
    from gpu_helpers import check_replay_row, make_pair, trajectory_logit_stats
    ead = _ead()
    ss = si.ModelShape("ragged-s", 2, 1024, 8, 2, 2976, 4096, 1e-5, 1e4)
    sl = si.ModelShape("ragged-l", 2, 2048, 16, 4, 5920, 4096, 1e-5, 1e4)
    Ws, Wl, os_, ol = make_pair(ss, sl, seed=8, gain_std=0.3, lm_sigma=1.5)
    prompt = si.prompt_np(8, "r1025", 1025, ss.vocab)
    ref = oracle.generate(os_, ol, prompt, 12, 5, 0.0, d_min=10)
    assert list(ref["model_id"]) == [0] * 10 + [1] * 2
    stats = trajectory_logit_stats(os_, ol, prompt, ref["tokens"], ref["model_id"])
    e = ead.EAD(ss, Ws, sl, Wl, window=5, tau=0.0, d_min=10, max_batch=1, max_seq=1056)
    rp = e.replay([prompt], ref["tokens"], ref["model_id"])
    n_dec, n_arg = check_replay_row(rp, 0, ref, 0.0, 12, stats)
    print(f"  H err {np.abs(rp['H'][0] - ref['H']).max():.2e}; decisions checked {n_dec}/12, clear arg maxes {n_arg}/12", flush=True)
    assert n_dec == 12
    e.close()


def test_qwen_truncated_long_prefill_agrees_with_scoring():
    """Qwen-shaped widths (2 layers each): a 600-token prompt is prefilled in one pass of 599 rows
    (38 token blocks: three sweeps of the tiled kernels or five 128-row sweeps per matrix, the last of them
    partly empty; row groups of 2 and 3 in the attention); the entropies of the following tokens -- small
    model, then the large one after a 10-row catch-up -- equal those of scoring the same tokens in passes of
    160 rows (two sweeps, one launch pair per sweep where K is split)."""
    ead = _ead()
    ss, sl = (s.truncated(2) for s in si.PAIRS["qwen"])
    Ws = si.model_weights_torch(ss, 0, "cuda")
    Wl = si.model_weights_torch(sl, 0, "cuda")
    e = ead.EAD(ss, Ws, sl, Wl, window=5, tau=0.0, d_min=10, max_batch=1, max_seq=640)
    prompt = si.prompt_np(4, "qlong", 600, ss.vocab)
    out = e.generate([prompt], 14)
    assert list(out["model_id"][0]) == [0] * 10 + [1] * 4
    seq = np.concatenate([prompt, out["tokens"][0]])
    for which, rng in ((0, range(0, 10)), (1, range(10, 14))):
        sc = e.score(which, seq[:-1], want_logits=False)
        for i in rng:
            assert abs(sc["H"][600 + i - 1] - out["H"][0, i]) < TOL_H, (which, i)
    e.close()


def test_qwen_full_depth_batch64_grouped_rows_follow_the_oracle():
    """The default benchmark's launch configuration at full size: the Qwen-0.5B / Qwen-14B shaped pair at full
    depth (24 and 48 layers), 64 ragged rows, grouped two-lane schedule.  The prompts are short (5-12 tokens) so
    that the oracle can follow three rows through the 14B shape token by token; those rows are teacher-forced
    along the oracle's trajectories (entropy, window mean, switch decision, arg max), the other 61 replay the
    library's own free run.  Gains 1 + N(0, 0.3^2) and wide LM heads spread the entropies enough for most
    decisions to fall outside the exemption band."""
    from gpu_helpers import check_replay_row, make_pair, trajectory_logit_stats
    ead = _ead()
    ss, sl = si.PAIRS["qwen"]
    n_new, d_min, w, batch, checked = 12, 3, 5, 64, (0, 21, 47)
    print("full-depth batch 64: weights and oracle models", flush=True)
    Ws, Wl, os_, ol = make_pair(ss, sl, seed=4, gain_std=0.3, lm_sigma=1.5)
    lens = si.prompt_lengths(4, batch, 5, 12)
    prompts = [si.prompt_np(4, f"fb{b}", int(lens[b]), ss.vocab) for b in range(batch)]
    hb = np.concatenate([oracle.generate(os_, ol, prompts[b], n_new, w, 1e30, d_min=d_min)["Hbar"] for b in checked])
    tau = float(np.percentile(hb, 55))
    refs, stats = {}, {}
    for b in checked:
        print(f"full-depth batch 64: oracle row {b} (prompt of {len(prompts[b])})", flush=True)
        refs[b] = oracle.generate(os_, ol, prompts[b], n_new, w, tau, d_min=d_min)
        stats[b] = trajectory_logit_stats(os_, ol, prompts[b], refs[b]["tokens"], refs[b]["model_id"])
    shares = [float(refs[b]["model_id"].mean()) for b in checked]
    print(f"tau {tau:.4f}; large share per checked row {shares}", flush=True)
    assert 0.0 < np.mean(shares) < 1.0
    del os_, ol
    e = ead.EAD(ss, Ws, sl, Wl, window=w, tau=tau, d_min=d_min, max_batch=batch, max_seq=32)
    del Ws, Wl
    torch.cuda.empty_cache()
    e.set_schedule(True, 0.5, 0.25)
    free = e.generate(prompts, n_new)
    st = e.stats()
    assert (free["lens"] == n_new).all() and st["switches"] > 0 and st["catchup_rows_large"] > 0
    print(f"  free run: passes large/small {st['steps_large']}/{st['steps_small']}, large share {st['large_share']:.2f}", flush=True)
    ft, fm = free["tokens"].copy(), free["model_id"].copy()
    for b in checked:
        ft[b], fm[b] = refs[b]["tokens"], refs[b]["model_id"]
    rp = e.replay(prompts, ft, fm)
    n_dec = n_arg = 0
    for b in checked:
        print(f"  row {b}: H err {np.abs(rp['H'][b] - refs[b]['H']).max():.2e}, window mean err {np.abs(rp['Hbar'][b] - refs[b]['Hbar']).max():.2e}", flush=True)
        d, a = check_replay_row(rp, b, refs[b], tau, n_new, stats[b], tol_logit=6e-2)
        n_dec += d; n_arg += a
    total = len(checked) * n_new
    print(f"  decisions checked outside the band {n_dec}/{total}, arg maxes with a clear gap {n_arg}/{total}", flush=True)
    assert n_dec >= total // 3
    others = [b for b in range(batch) if b not in checked]
    assert np.abs(rp["H"][others] - free["H"][others]).max() < TOL_H
    e.set_schedule(False)
    e.close()

"""GPU: single-row decode steps through the persistent streaming kernel (k_decode_stream), asked for and taken by itself, against the per-layer kernels."""
import ctypes as C
import threading

import numpy as np
import pytest

import oracle
import synth_inputs as si
from gpu_helpers import TOL_H, make_pair

pytestmark = pytest.mark.gpu

# heads x head_dim x query heads per KV head of every instantiation; row blocks and k tiles that leave remainders in the units and slots (33 to 161 k
# tiles, 2 to 4 slices of K); a vocabulary of 257 row blocks
CASES = [("g4", 2, 2048, 32, 8, 5152), ("g7", 3, 896, 14, 2, 4864), ("g3", 2, 3072, 24, 8, 2080), ("g5", 1, 5120, 40, 8, 2048),
         ("g6", 2, 1536, 12, 2, 8960), ("g4-128", 1, 4096, 32, 8, 4192)]


@pytest.mark.parametrize("name,layers,d,heads,kv,ffn", CASES, ids=[c[0] for c in CASES])
def test_replay_matches_the_oracle_and_the_per_layer_kernels(name, layers, d, heads, kv, ffn):
    """Entropies along a trajectory within 1e-2 nats of the oracle, from the first key on and across 64-key splits, and within 2e-3 of the per-layer kernels: both keep
    float32 activations, but another order of sums moves a cached key or value to its other bf16 neighbour (2^-8 of it), and what two kernel families differ by
    for that reason is bounded by 7e-3 of the row maximum in the logits, 2e-3 nats."""
    _check_replay(si.ModelShape("stream-" + name, layers, d, heads, kv, ffn, 4112, 1e-5, 1e4))


class Head128(si.ModelShape):
    head_dim = 128


@pytest.mark.parametrize("d,heads,kv", [(4096, 56, 14), (2048, 100, 25)])
def test_attention_output_of_more_columns_than_a_workgroup_stages_at_once(d, heads, kv):
    """7168 and 12800 columns, in two slices of the output projection's K and in four."""
    _check_replay(Head128(f"stream-wide-{heads}", 1, d, heads, kv, 1056, 4112, 1e-5, 1e4))


def _check_replay(shape):
    import paper_2502_06833_amd as ead
    other = si.ModelShape("stream-other", 1, 128, 4, 4, 128, 4112, 1e-5, 1e4)
    W, Wo, om, _ = make_pair(shape, other, gain_std=0.2, lm_sigma=1.5)
    e = ead.EAD(shape, W, other, Wo, window=5, tau=0.0, d_min=4, max_batch=1, max_seq=160)
    e.set_fused(1)
    e.profile(True)
    e.replay([si.prompt_np(0, "taken", 1, shape.vocab)], np.zeros((1, 2), np.int32), np.zeros((1, 2), np.uint8))
    assert any("decode_fused" in p["name"] for p in e.profile_read())      # the kernel serves this shape
    e.profile(False)
    for P, n in ((1, 6), (60, 8), (125, 10)):
        toks = si.prompt_np(0, f"s{P}", P + n, shape.vocab)
        got = {}
        for mode in (0, 1):
            e.set_fused(mode)
            got[mode] = e.replay([toks[:P]], toks[None, P:], np.zeros((1, n), np.uint8))["H"][0]
        ref = oracle.entropy_rows(om.forward_dense(toks)[P - 1:P + n - 1])[0]
        assert np.abs(got[1] - ref).max() < TOL_H
        assert np.abs(got[1] - got[0]).max() < 2e-3
    e.close()


DEEP = si.ModelShape("stream-deep", 20, 2048, 32, 8, 512, 4112, 1e-5, 1e4)
FLAT = si.ModelShape("stream-flat", 20, 1536, 12, 2, 512, 4112, 1e-5, 1e4)


def _pair():
    return [si.model_weights_torch(s, 0, "cuda", lm_std=1.5 / np.sqrt(s.d_model)) for s in (DEEP, FLAT)]


def test_taken_by_itself_and_switched_off():
    """A run of both models, switching: the default takes the kernel, as the profile says, set_fused(False) does not; two default runs agree bit for bit, and the
    entropies before the first token that differs (two logits may be close) are within 2e-3 (see above)."""
    import paper_2502_06833_amd as ead
    Ws, Wl = _pair()
    e = ead.EAD(DEEP, Ws, FLAT, Wl, window=3, tau=7.2, d_min=2, max_batch=1, max_seq=96)
    prompt = si.prompt_np(0, "auto", 40, DEEP.vocab)
    e.profile(True)
    runs = [e.generate([prompt], 24)]
    names = {p["name"] for p in e.profile_read() if p["launches"]}
    e.profile(False)
    assert any("decode_fused" in n for n in names)
    runs.append(e.generate([prompt], 24))
    e.set_fused(False)
    runs.append(e.generate([prompt], 24))
    e.set_fused(-1)                                     # the default again
    runs.append(e.generate([prompt], 24))
    assert (runs[3]["H"] == runs[0]["H"]).all() and (runs[3]["tokens"] == runs[0]["tokens"]).all()
    assert (runs[0]["H"] == runs[1]["H"]).all() and (runs[0]["tokens"] == runs[1]["tokens"]).all()
    same = (runs[2]["tokens"] == runs[0]["tokens"])[0].cumprod().astype(bool) & (runs[2]["model_id"] == runs[0]["model_id"])[0].cumprod().astype(bool)
    assert same[:4].all() and np.abs(runs[2]["H"] - runs[0]["H"])[0][same].max() < 2e-3
    e.close()


def _spin_limit(e, polls):
    """Polls after which a wait inside the kernel is given up (-1: as many as ever; -2: its launches are refused); every kernel ends normally."""
    import paper_2502_06833_amd as ead
    fn = ead.lib().ead_test_spin_limit
    fn.argtypes = [C.c_void_p, C.c_int32]
    assert fn(e._h, polls) == 0


@pytest.mark.parametrize("polls", [0, 1, 2, 4])
def test_a_launch_given_up_leaves_no_token(polls):
    """Waves that give up leave one by one while the rest of their workgroups go on, at other places for every limit and run: the kernels per layer finish the
    run from the last token that was whole.  Entropies within 2e-3 of those kernels' own run, as long as the tokens are the same (two logits may be close)."""
    import paper_2502_06833_amd as ead
    Ws, Wl = _pair()
    e = ead.EAD(DEEP, Ws, FLAT, Wl, window=3, tau=7.2, d_min=2, max_batch=1, max_seq=96)
    e.force_model(0)
    prompt = si.prompt_np(0, "given-up", 40, DEEP.vocab)
    e.set_fused(False)
    want = e.generate([prompt], 24)
    e.close()
    for _ in range(4):
        e = ead.EAD(DEEP, Ws, FLAT, Wl, window=3, tau=7.2, d_min=2, max_batch=1, max_seq=96)
        e.force_model(0)
        e.begin([prompt], 24)
        e.decode(3)
        _spin_limit(e, polls)
        e.decode(21)
        got = e.fetch()
        assert got["lens"][0] == 24
        same = (got["tokens"] == want["tokens"])[0].cumprod().astype(bool)
        assert same[:4].all() and np.abs(got["H"] - want["H"])[0][same].max() < 2e-3
        e.close()


@pytest.mark.parametrize("polls", [0, 2])
@pytest.mark.parametrize("max_batch", [1, 2], ids=["one-lane", "two-lanes"])
def test_switches_after_a_launch_given_up(polls, max_batch):
    """Passes of the kernels per layer that follow a launch that was given up (the other model's catch-up after a switch, here dictated by a trajectory and by
    the window) find the device where the host counts it.  Without a single poll no launch gets through: bit for bit the run of the kernels per layer."""
    import paper_2502_06833_amd as ead
    Ws, Wl = _pair()
    args = dict(window=3, tau=7.2, d_min=2, max_batch=max_batch, max_seq=96)
    prompt, forced = si.prompt_np(0, "given-up", 30, DEEP.vocab), si.prompt_np(0, "forced", 24, DEEP.vocab)
    for mid in (np.arange(24) // 5 % 2, 1 - np.arange(24) // 3 % 2):
        got, stats = {}, {}
        for limit in (None, polls):
            e = ead.EAD(DEEP, Ws, FLAT, Wl, **args)
            if limit is None:
                e.set_fused(False)
            else:
                _spin_limit(e, limit)
            got[limit] = e.replay([prompt], forced[None], mid[None].astype(np.uint8))
            stats[limit] = e.stats()
            e.close()
        assert _counts(stats[polls]) == _counts(stats[None])
        assert np.abs(got[polls]["H"] - got[None]["H"]).max() < (1e-9 if polls == 0 else 2e-3)
    got = {}
    for limit in (None, polls):
        e = ead.EAD(DEEP, Ws, FLAT, Wl, **args)
        if limit is None:
            e.set_fused(False)
        else:
            _spin_limit(e, limit)
        got[limit] = e.generate([prompt], 24)
        stats[limit] = e.stats()
        assert stats[limit]["tokens_small"] + stats[limit]["tokens_large"] == 24
        if limit is not None:
            assert (e.generate([prompt], 24)["lens"] == 24).all()        # the handle goes on with the kernels per layer
        e.close()
    assert len(set(got[None]["model_id"][0])) == 2 and got[polls]["lens"][0] == 24
    if polls == 0:
        assert all((got[0][k] == got[None][k]).all() for k in ("tokens", "model_id", "H", "Hbar"))
        assert _counts(stats[0]) == _counts(stats[None])


def _counts(stats):
    """What a run's statistics say of its tokens, not of how often the host waited."""
    return {k: v for k, v in stats.items() if k != "host_syncs"}


def test_a_launch_refused_leaves_the_run_to_the_kernels_per_layer():
    import paper_2502_06833_amd as ead
    Ws, Wl = _pair()
    prompt = si.prompt_np(0, "given-up", 30, DEEP.vocab)
    e = ead.EAD(DEEP, Ws, FLAT, Wl, window=3, tau=7.2, d_min=2, max_batch=1, max_seq=96)
    e.set_fused(1)
    runs = [e.generate([prompt], 24)]
    e.set_fused(-1)
    _spin_limit(e, -2)
    runs.append(e.generate([prompt], 24))
    _spin_limit(e, -1)
    e.set_fused(False)
    runs.append(e.generate([prompt], 24))
    assert all((runs[1][k] == runs[2][k]).all() for k in ("tokens", "model_id", "H", "Hbar"))
    e.set_fused(1)
    _spin_limit(e, -2)
    with pytest.raises(ead.EadError):                                  # asked for: an error
        e.generate([prompt], 24)
    _spin_limit(e, -1)
    again = e.generate([prompt], 24)
    assert all((again[k] == runs[0][k]).all() for k in ("tokens", "model_id", "H", "Hbar"))
    e.close()


def test_a_kernel_asked_for_that_gives_up_is_an_error():
    import paper_2502_06833_amd as ead
    Ws, Wl = _pair()
    prompt = si.prompt_np(0, "given-up", 30, DEEP.vocab)
    for mode, grouped in ((1, False), (2, False), (1, True)):
        e = ead.EAD(DEEP, Ws, FLAT, Wl, window=3, tau=7.2, d_min=2, max_batch=2, max_seq=96)
        e.set_schedule(grouped)
        e.set_fused(False)
        want = e.generate([prompt], 24)
        e.set_fused(mode)
        _spin_limit(e, 0)
        with pytest.raises(ead.EadError) as err:
            e.generate([prompt], 24)
        assert err.value.status == 7                                   # EAD_ERR_DEVICE
        got = e.generate([prompt], 24)                                 # the kernels per layer from then on
        assert all((got[k] == want[k]).all() for k in ("tokens", "model_id", "H"))
        _spin_limit(e, -1)
        e.set_fused(mode)                                              # asked for once more: its buffers are as at the start
        again = e.generate([prompt], 24)
        same = (again["tokens"] == want["tokens"])[0].cumprod().astype(bool) & (again["model_id"] == want["model_id"])[0].cumprod().astype(bool)
        assert same[:4].all() and np.abs(again["H"] - want["H"])[0][same].max() < 2e-3
        e.close()


@pytest.mark.parametrize("other", ["streamed", "register-buffered"])
def test_two_handles_in_two_threads(other):
    """Persistent kernels of two handles on streams of their own: one starts after the other's has ended, and both finish with the tokens of a run alone."""
    import torch
    import paper_2502_06833_amd as ead
    Ws, Wl = _pair()
    prompts = [si.prompt_np(0, f"thread{i}", 30 + i, DEEP.vocab) for i in range(2)]
    handles, streams = [], [torch.cuda.Stream() for _ in range(2)]
    for i in range(2):
        with torch.cuda.stream(streams[i]):
            handles.append(ead.EAD(DEEP, Ws, FLAT, Wl, window=3, tau=7.2, d_min=2, max_batch=1, max_seq=96))
    for i in range(2):
        handles[i].set_fused(2 if other == "register-buffered" and i else 1)      # not taken by itself with two streams
    want = [handles[i].generate([prompts[i]], 32) for i in range(2)]
    got = [[], []]

    def work(i):
        for _ in range(4):
            got[i].append(handles[i].generate([prompts[i]], 32))

    threads = [threading.Thread(target=work, args=(i,)) for i in range(2)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    for i in range(2):
        assert len(got[i]) == 4
        for r in got[i]:
            assert (r["tokens"] == want[i]["tokens"]).all() and (r["H"] == want[i]["H"]).all()
        handles[i].close()


def test_not_taken_by_itself_beside_a_handle_on_another_stream():
    """The kernel takes the whole chip, so runs of handles on streams of their own keep to the per-layer kernels, which share it; on one stream they take it."""
    import torch
    import paper_2502_06833_amd as ead
    Ws, Wl = _pair()
    prompt = si.prompt_np(0, "beside", 40, DEEP.vocab)

    def handle(stream):
        with torch.cuda.stream(stream):
            return ead.EAD(DEEP, Ws, FLAT, Wl, window=3, tau=7.2, d_min=2, max_batch=1, max_seq=96)

    def run(e):
        e.profile(True)
        out = e.generate([prompt], 16)
        names = {p["name"] for p in e.profile_read() if p["launches"]}
        e.profile(False)
        return out, any("decode_fused" in n for n in names)

    one, two = torch.cuda.Stream(), torch.cuda.Stream()
    a, same = handle(one), handle(one)
    alone, taken = run(a)
    assert taken and run(same)[1]
    b = handle(two)
    beside, taken = run(a)
    assert not taken and not run(b)[1]
    a.set_fused(False)
    layers, _ = run(a)
    assert all((beside[k] == layers[k]).all() for k in ("tokens", "model_id", "H"))
    a.set_fused(-1)
    b.close()
    again, taken = run(a)
    assert taken and all((again[k] == alone[k]).all() for k in ("tokens", "model_id", "H"))
    a.close()
    same.close()

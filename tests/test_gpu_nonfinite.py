"""GPU: weights that make the logits NaN end a run with the documented error, and every token handed on stays inside the
vocabulary (the rule itself is checked on the CPU in test_host_kernels.py)."""
import numpy as np
import pytest

import synth_inputs as si

pytestmark = pytest.mark.gpu

BF16_S = si.ModelShape("nan-s", 1, 128, 4, 2, 256, 512, 1e-5, 1e4)
BF16_L = si.ModelShape("nan-l", 1, 256, 4, 2, 512, 512, 1e-5, 1e4)


@pytest.mark.parametrize("small,large,batch", [(si.TINY_S, si.TINY_L, 1), (si.TINY_S, si.TINY_L, 5), (BF16_S, BF16_L, 1)],
                         ids=["fp32-1", "fp32-5", "bf16-1"])
@pytest.mark.parametrize("temperature", [0.0, 0.7])
def test_nan_gain_ends_a_run_with_the_error(small, large, batch, temperature):
    import paper_2502_06833_amd as ead
    Ws, Wl = si.model_weights_torch(small, 0, "cuda"), si.model_weights_torch(large, 0, "cuda")
    Wl["norm_final"][3] = float("nan")
    e = ead.EAD(small, Ws, large, Wl, window=2, tau=0.0, d_min=2, max_batch=batch, max_seq=32)      # tau 0: the large model takes over
    e.set_sampling(temperature, 5)
    prompts = [si.prompt_np(0, f"nan{b}", 2 + b, small.vocab) for b in range(batch)]
    with pytest.raises(ead.EadError) as err:
        e.generate(prompts, 12)
    assert err.value.status == 6                                   # EAD_ERR_NONFINITE
    for n in (1, 2):
        out = e.score(1, prompts[0][:n])
        assert np.isnan(out["H"]).all() and ((out["argmax"] >= 0) & (out["argmax"] < small.vocab)).all()
    e.force_model(0)                                             # the handle still serves the model that is sound
    out = e.generate(prompts, 12)
    assert np.isfinite(out["H"]).all() and (out["lens"] == 12).all()
    e.close()

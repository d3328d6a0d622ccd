"""GPU: prompt passes long enough for the tiled kernels (128-row sweeps, 128 x 256 and 256 x 256 tiles, several bands of
sweeps), with row-block counts and row counts that leave partly empty tiles, against teacher-forced scoring of the
same prompts in passes of at most 160 rows.  (Of a model of one layer the prompt's first entropy sees the QKV projections' sums alone; the
residual projections of these shapes are compared with the oracle in test_gpu_wide_batches.py.)"""
import numpy as np
import pytest

import synth_inputs as si

pytestmark = pytest.mark.gpu

# 4096 wide with 40 + 16 heads' worth of QKV row blocks: residual and QKV projections reach the 256 x 256 tiles from about
# 2100 rows; 1914 row blocks in the narrow model's gate/up do from 257
WIDE = si.ModelShape("wide-d", 1, 4096, 32, 8, 544, 1040, 1e-5, 1e4)
FFN = si.ModelShape("wide-f", 2, 256, 4, 2, 15312 // 32 * 32, 1040, 1e-5, 1e4)

# 136 row blocks in the residual projections: 128-row sweeps of five row blocks from about 900 rows, the last group with one
FIVES = si.ModelShape("wide-r", 1, 2176, 17, 17, 544, 1040, 1e-5, 1e4)


@pytest.mark.parametrize("lens,large", [((130,), WIDE), ((258,), WIDE), ((301, 2), WIDE), ((520, 505), WIDE), ((1101, 900, 310), WIDE),
                                        ((1500, 1400, 1301, 1200), WIDE), ((1025,), FIVES)])
def test_prompt_passes_agree_with_scoring(lens, large):
    """First entropy of every row within 2e-3 nats of the scored one (kernel families differ by 7e-3 of the row maximum in
    the logits, which is 2e-3 nats in the entropy), same token unless the scored logits are close."""
    import paper_2502_06833_amd as ead
    W = {s.name: si.model_weights_torch(s, 0, "cuda", lm_std=1.5 / np.sqrt(s.d_model)) for s in (large, FFN)}
    e = ead.EAD(FFN, W[FFN.name], large, W[large.name], window=5, tau=0.0, d_min=4, max_batch=len(lens), max_seq=max(lens) + 2)
    prompts = [si.prompt_np(0, f"long{i}", n, 1040) for i, n in enumerate(lens)]
    for which in (0, 1):
        e.force_model(which)
        got = e.generate(prompts, 1)
        for b, p in enumerate(prompts):
            ref = e.score(which, p)
            two = np.sort(ref["logits"][-1])[-2:]
            assert abs(got["H"][b, 0] - ref["H"][-1]) < 2e-3, (which, b)
            if two[1] - two[0] > 2e-2 * np.abs(ref["logits"][-1]).max():
                assert got["tokens"][b, 0] == ref["argmax"][-1], (which, b)
    e.close()

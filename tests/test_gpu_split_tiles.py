"""GPU: long passes whose last sweeps are cut along K (tile_plan in rules.hpp), against teacher-forced scoring of the same prompts in passes of at most 160
rows: residual projections of 17 groups of row blocks, 15 sweeps whole and a partly filled one in 3 and 4 slabs; all sweeps in 8 slabs, the last token block
partly filled; row blocks that fill their groups partly, uneven slabs of 257 k tiles; QKV projections, 10 sweeps whole and two in slabs.  In models of one layer the first
entropy after a prompt follows the QKV projections' sums alone; test_gpu_wide_batches.py compares all of them, row by row, with the oracle."""
import numpy as np
import pytest

import synth_inputs as si

pytestmark = pytest.mark.gpu

SHAPES = [(si.ModelShape("whole-and-slabs", 1, 4352, 34, 17, 3072, 1040, 1e-5, 1e4), (1400, 1301, 1330)),
          (si.ModelShape("slabs", 1, 1024, 8, 4, 8192, 1040, 1e-5, 1e4), (500, 480)),
          (si.ModelShape("uneven-slabs", 1, 1056, 33, 11, 8224, 1040, 1e-5, 1e4), (1400, 1301, 1330)),
          (si.ModelShape("qkv-slabs", 1, 4096, 32, 8, 544, 1040, 1e-5, 1e4), (1500, 1480))]
OTHER = si.ModelShape("split-other", 1, 128, 4, 4, 128, 1040, 1e-5, 1e4)


@pytest.mark.parametrize("shape,lens", SHAPES, ids=lambda v: getattr(v, "name", None))
def test_split_tiles_agree_with_scoring(shape, lens):
    """First entropy of every row within 2e-3 nats of the scored one (the kernel families differ by 7e-3 of the row maximum in the logits, which is 2e-3 nats
    in the entropy), same token unless the scored logits are close."""
    import paper_2502_06833_amd as ead
    W = {s.name: si.model_weights_torch(s, 0, "cuda", lm_std=1.5 / np.sqrt(s.d_model)) for s in (shape, OTHER)}
    e = ead.EAD(shape, W[shape.name], OTHER, W[OTHER.name], window=5, tau=0.0, d_min=4, max_batch=len(lens), max_seq=max(lens) + 2)
    prompts = [si.prompt_np(0, f"split{i}", n, 1040) for i, n in enumerate(lens)]
    e.force_model(0)
    got = e.generate(prompts, 1)
    for b, p in enumerate(prompts):
        ref = e.score(0, p)
        two = np.sort(ref["logits"][-1])[-2:]
        assert abs(got["H"][b, 0] - ref["H"][-1]) < 2e-3, b
        if two[1] - two[0] > 2e-2 * np.abs(ref["logits"][-1]).max():
            assert got["tokens"][b, 0] == ref["argmax"][-1], b
    e.close()

"""GPU: decode passes of 978 to 4028 sequences at once, every row against the oracle.  All rows' logits come out of the pass, so each of its matrices' sums counts
(a prompt pass leaves keys and values alone, in a model of one layer those of its QKV projection).  The shapes of test_gpu_split_tiles.py, at the row
counts of its prompt passes, whose last sweeps are cut along K (tile_plan in rules.hpp), and those of test_gpu_long_prefill.py (whole tiles, sweeps of five
row blocks with one in the last group)."""
import numpy as np
import pytest

import oracle
import synth_inputs as si
from gpu_helpers import TOL_H, TOL_LOGIT, make_pair
from test_gpu_long_prefill import FIVES, WIDE
from test_gpu_split_tiles import OTHER, SHAPES

pytestmark = pytest.mark.gpu

CASES = [(shape, sum(lens) - len(lens)) for shape, lens in SHAPES] + [(WIDE, 2308), (FIVES, 1024)]


@pytest.mark.parametrize("shape,rows", CASES, ids=lambda v: getattr(v, "name", None))
def test_every_row_of_a_wide_batch(shape, rows):
    """37 prompts of three tokens take turns over the rows, so that no two rows a tile, a sweep or a slab apart hold the same one.  Entropy within 1e-2 nats, arg max
    where the oracle's two best logits are further apart than twice the logit tolerance (the tolerances of all bf16 parity tests)."""
    import paper_2502_06833_amd as ead
    W, Wo, om, _ = make_pair(shape, OTHER, gain_std=0.2, lm_sigma=1.5)
    prompts = [si.prompt_np(0, f"wide{i}", 3, shape.vocab) for i in range(37)]
    ref = np.stack([om.forward_dense(p)[-1] for p in prompts])
    H, arg = oracle.entropy_rows(ref)
    two = np.sort(ref, axis=1)
    clear = two[:, -1] - two[:, -2] > 2 * TOL_LOGIT * np.abs(ref).max(axis=1)
    assert clear.sum() >= 10 and np.ptp(H) > 10 * TOL_H
    e = ead.EAD(shape, W, OTHER, Wo, window=5, tau=0.0, d_min=4, max_batch=rows, max_seq=32)
    e.force_model(0)
    got = e.generate([prompts[r % 37] for r in range(rows)], 1)
    e.close()
    which = np.arange(rows) % 37
    assert np.abs(got["H"][:, 0] - H[which]).max() < TOL_H
    assert (got["tokens"][:, 0] == arg[which])[clear[which]].all()

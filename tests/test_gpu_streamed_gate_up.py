"""GPU: gate/up matrices and LM heads of passes of one and two token blocks through the fetching-wave kernels and the register rings, on both sides of their rules
(gate_up_streamed, lm_by_rings, tiles_once and lm_once in rules.hpp): 1028 row blocks (a last group of three in five) x 128 and 129 k tiles from three rows on, 1024 x 128 and
544 x 96 from 17, 128 x 96 that stay with the other kernel; 1540 row blocks x 29, two waves to four of them from 17 to 32; LM heads of 1000 to 2000 row blocks."""
import numpy as np
import pytest

import oracle
import synth_inputs as si
from gpu_helpers import TOL_H, TOL_LOGIT, check_logits, make_pair

pytestmark = pytest.mark.gpu


class FewHeads(si.ModelShape):
    head_dim = 128


@pytest.mark.parametrize("d,ffn", [(4096, 8224), (4128, 8224), (3072, 1024), (4096, 8192), (928, 12320), (2336, 512), (2560, 512), (3072, 4352)])
def test_gate_up_of_one_and_two_token_blocks(d, ffn):
    """Logits within 2e-2 of the row maximum, entropy within 1e-2 nats (the tolerances of all bf16 parity tests)."""
    _check_scores(FewHeads(f"gu-{d}", 1, d, 4, 2, ffn, 1040, 1e-5, 1e4))


@pytest.mark.parametrize("vocab,d", [(24000, 4096), (32000, 1280), (23984, 1280), (16400, 2336), (16368, 2336), (16384, 2560)])
def test_lm_heads_of_one_and_two_token_blocks(vocab, d):
    """1500 row blocks x 128 and 2000 x 40 non-temporally, 1499 x 40 plainly through k_lm_ls; 1025 x 73 through the rings up to 16 rows, 1023 x 73 (whose last workgroup has three row
    blocks of four) and 1024 x 80 up to 32."""
    _check_scores(FewHeads(f"lm-{vocab}", 1, d, 4, 2, 256, vocab, 1e-5, 1e4))


def _check_scores(shape):
    import paper_2502_06833_amd as ead
    other = si.ModelShape("gu-other", 1, 128, 4, 4, 128, shape.vocab, 1e-5, 1e4)
    W, Wo, om, _ = make_pair(shape, other, gain_std=0.2, lm_sigma=1.5)
    e = ead.EAD(shape, W, other, Wo, window=5, tau=0.0, d_min=4, max_batch=1, max_seq=64)
    toks = si.prompt_np(0, "gu", 33, shape.vocab)
    ref = om.forward_dense(toks)
    for T in (3, 16, 17, 32, 33):
        out = e.score(0, toks[:T])
        check_logits(out["logits"], ref[:T], TOL_LOGIT)
        assert np.abs(out["H"] - oracle.entropy_rows(ref[:T])[0]).max() < TOL_H
        assert np.abs(oracle.entropy_rows(out["logits"])[0] - out["H"]).max() < 1e-4      # statistics against the logits they fold
    e.close()

"""GPU: steps of the stand-alone gate that share a launch: what a step yields does not depend on how many do, up to the 64 of a launch, past
them, and where the rows bound them (4096 row steps a launch)."""
import pytest

import synth_inputs as si

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("rows,vocab,steps,window", [(1, 50264, 65, 5), (2, 2048, 129, 64), (5, 1000, 64, 3), (70, 512, 59, 5), (3, 512, 33, 65)])
def test_steps_sharing_a_launch_match_single_steps(rows, vocab, steps, window):
    import torch
    import paper_2502_06833_amd as ead
    tensors = [si.logits_torch(i, "steps", rows, vocab, torch.bfloat16, "cuda") for i in range(7)]
    many = ead.Gate(rows, window, 5.0, 2)
    one = ead.Gate(rows, window, 5.0, 2)
    for _ in range(2):                                  # the second run begins with a full window
        H, am, mid, hb = many.run_logits(tensors, steps)
        for s in range(steps):
            h1, a1, m1, w1, _ = one.step_logits(tensors[s % 7])
            assert torch.equal(H[s], h1) and torch.equal(am[s], a1) and torch.equal(mid[s], m1) and torch.equal(hb[s], w1), s
    many.close()
    one.close()

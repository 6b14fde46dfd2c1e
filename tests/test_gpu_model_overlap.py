"""Model step with each layer's AdamW update inside its backward
(Model.train_step_overlapped) against the plain step (train_step: the
backward of every layer, then one AdamW over all parameters).

Every sum of a step is taken in a fixed order, so both give the same bits: every
parameter, master weight, moment and gradient, the embedding's among them.
"""
import pytest

import forge_inputs as fi
from gpu_util import banner

pytestmark = pytest.mark.gpu

CASES = {
    # layers below 2^20 token x hidden elements: everything in order
    "tiny_untied": lambda: fi.config("tiny", n_layers=2, seed=41),
    # 512 x 2048: side streams and the optimizer stream, tied head
    "two_layers_tied": lambda: fi.config("dense1b", batch=1, seq=512, vocab=1024, n_layers=2,
                                         seed=43),
}


@pytest.mark.parametrize("case", list(CASES))
def test_overlapped_model_step_equals_plain_step(case):
    import torch
    from paper_2609_13645_amd import runtime
    cfg = CASES[case]()
    banner(f"model step: per-layer overlapped updates vs one AdamW ({case})")
    inp = fi.model_inputs(cfg)
    plain = runtime.Model(cfg, inp)
    over = runtime.Model(cfg, inp)
    plain.train_step()
    over.train_step_overlapped()
    torch.cuda.synchronize()
    assert torch.equal(plain.loss, over.loss)
    for n in plain.flat.offsets:
        for buf in ("param", "master", "m", "v", "grad"):
            a = plain.flat.view(getattr(plain.flat, buf), n)
            b = over.flat.view(getattr(over.flat, buf), n)
            assert torch.equal(a, b), (n, buf)
    plain.train_step()
    over.train_step_overlapped()
    torch.cuda.synchronize()
    assert int(plain.dev_step.item()) == int(over.dev_step.item()) == 2
    assert torch.equal(over.loss, plain.loss)
    for buf in ("param", "master", "m", "v", "grad"):
        assert torch.equal(getattr(over.flat, buf), getattr(plain.flat, buf)), buf
    # the update moved the weights
    assert not torch.equal(over.flat.master, runtime.Model(cfg, inp).flat.master)

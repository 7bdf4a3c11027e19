"""Recompute mode on a batch of one chunk: dS formed from the logits the forward kept.  The default mode against the explicit one, which
recomputes them in bf16 (same arithmetic: same bits), and f32 against the oracle."""
import pytest
import torch

from paper_2603_16435_amd import synth
from parity_util import compare_all, run_gpu, run_oracle

pytestmark = pytest.mark.gpu
OUT = ("loss", "seq_loss", "logprob", "lse", "entropy", "coeff", "d_hidden", "d_weight", "target_col", "target_logit")


# one token, a tile of tokens less one / exactly / plus one, several tiles; vocabulary one past a tile, one short of one, less than one
@pytest.mark.parametrize("H,V,lengths,tau", [(456, 513, [1, 0, 0, 0], 0.0), (512, 2559, [100, 99, 1, 55], 0.8), (640, 255, [256, 0, 0, 0], 0.0),
                                             (1160, 3000, [200, 57, 0, 0], 0.7), (776, 5000, [300, 301, 2, 64], 0.0)])
@pytest.mark.parametrize("layout", ["packed", "padded"])
def test_bf16_kept_logits_give_the_bits_of_recomputed_ones(H, V, lengths, tau, layout):
    cfg = synth.RolloutConfig("kept", 2, 2, 1, 64, H, V, "bf16", 0.5, seed=81)
    b = synth.make_rollouts(cfg, "cuda", layout, lengths=lengths, temperature=tau or 1.0)
    want, got = (run_gpu(b, "flow", temperature=tau, backward_mode=m) for m in ("recompute", "auto"))
    for name in OUT:
        assert torch.equal(getattr(got, name), getattr(want, name)), name


# a few tokens in many rows: a block of 16 tokens less one / exactly / plus one, tokens of the second tile alone past its border
@pytest.mark.parametrize("tokens", [15, 16, 17, 257])
def test_bf16_few_tokens_in_many_rows(tokens):
    cfg = synth.RolloutConfig("kept", 2, 2, 1, 64, 520, 2559, "bf16", 0.5, seed=85)
    b = synth.make_rollouts(cfg, "cuda", "packed", lengths=[400, 300, 1, 300])
    on = b.mask.nonzero().flatten()
    b.mask[on[torch.randperm(len(on), generator=torch.Generator().manual_seed(1)).cuda()[tokens:]]] = 0
    want, got = (run_gpu(b, "flow", backward_mode=m) for m in ("recompute", "auto"))
    for name in OUT:
        assert torch.equal(getattr(got, name), getattr(want, name)), name


def test_bf16_no_row_counts():
    cfg = synth.RolloutConfig("kept", 1, 2, 1, 8, 512, 600, "bf16", 0.5, seed=82)
    b = synth.make_rollouts(cfg, "cuda", "packed", lengths=[8, 8])
    b.mask.zero_()
    r = run_gpu(b, "grpo")
    assert not r.d_hidden.any() and not r.d_weight.any() and r.loss.item() == 0.0


@pytest.mark.parametrize("H,V,lengths", [(64, 300, [1, 0, 0, 0]), (64, 257, [64, 0, 63, 1]), (132, 1000, [65, 10, 0, 2]),
                                         (36, 33001, [63, 66, 0, 1])])               # (the last: wide tiles)
def test_f32_kept_logits(H, V, lengths):
    cfg = synth.RolloutConfig("kept", 2, 2, 1, 64, H, V, "f32", 0.5, seed=83)
    b = synth.make_rollouts(cfg, "cuda", "padded", lengths=lengths)
    ref = run_oracle(b, "grpo", temperature=0.9)
    print(compare_all(b, run_gpu(b, "grpo", temperature=0.9), ref, temperature=0.9, loss_tol=1e-5, logp_atol=2e-5, grad_tol=1e-4), flush=True)

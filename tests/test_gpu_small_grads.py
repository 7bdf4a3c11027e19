"""Small f32 batches: dX and dW in one launch out of the kept logits, the combine inside the loss launch.  Against the oracle, and the log-probs to
the bit against the scoring call, which combines in a launch of its own."""
import pytest
import torch

from paper_2603_16435_amd import binding, synth
from parity_util import compare_all, run_gpu, run_oracle
from test_gpu_f32_tiles import F32_TOL, off_grid

pytestmark = pytest.mark.gpu


# tokens one short of a block of 16, a block, one past it, one; vocabularies of one tile, one past two, the last that takes the path and the first that does
# not; columns one piece past a block of 32 or 64; more rows than the combine in the loss launch takes, blocks of 64 columns in dX
@pytest.mark.parametrize("H,V,lengths", [(4, 5, [1, 0, 0, 0]), (36, 255, [15, 0, 0, 0]), (68, 513, [16, 17, 1, 300]), (128, 2048, [100, 99, 1, 55]),
                                         (128, 2049, [100, 99, 1, 55]), (260, 1000, [256, 257, 3, 500]), (64, 1793, [1000, 1, 15, 1016])])
@pytest.mark.parametrize("objective", ["grpo", "flow"])
def test_small_f32_batches(H, V, lengths, objective):
    cfg = synth.RolloutConfig("small", 2, 2, 1, 64, H, V, "f32", 0.5, seed=91)
    b = synth.make_rollouts(cfg, "cuda", "padded", lengths=lengths, temperature=0.9)
    b.hidden[b.mask == 0] = float("inf")                                    # rows that do not count reach no sum
    got = run_gpu(b, objective, temperature=0.9)
    b.hidden[b.mask == 0] = 0.0
    # the flow weight is exp of a sum of n f32 log-probs of magnitude below 8, each rounded by up to 2^-22: with n = 1016 at random signs
    # 4 sqrt(n / 3) 2^-22 = 1.8e-5 of a term, and the terms of d_log_z (up to 9 here, differences of which remain) and of the loss have that error: 1.6e-4
    tol = F32_TOL if objective == "grpo" else dict(F32_TOL, loss_tol=1.6e-4)
    print(compare_all(b, got, run_oracle(b, objective, temperature=0.9), temperature=0.9, **tol), flush=True)
    logp, lse = binding.rl_token_logprob_tempered(b.hidden, b.weight, b.token_ids, b.mask, 0.9, b.cu_seqlens)
    assert torch.equal(got.logprob, logp) and torch.equal(got.lse, lse)
    b.weight, b.hidden = off_grid(b.weight), off_grid(b.hidden)
    again = run_gpu(b, objective, temperature=0.9)
    assert torch.equal(again.d_hidden, got.d_hidden) and torch.equal(again.d_weight, got.d_weight)


def test_no_row_counts():
    b = synth.make_rollouts(synth.RolloutConfig("small", 1, 2, 1, 8, 64, 600, "f32", 0.5, seed=92), "cuda", "packed", lengths=[8, 8])
    b.mask.zero_()
    r = run_gpu(b, "grpo")
    assert not r.d_hidden.any() and not r.d_weight.any() and r.loss.item() == 0.0


# two workgroups a CU at the most, one launch; more, of a small vocabulary; more, of a larger one: the pair of contractions
@pytest.mark.parametrize("V,rows", [(1000, 1700), (700, 2000), (1000, 2000)])
def test_many_rows(V, rows):
    b = synth.make_rollouts(synth.RolloutConfig("small", 2, 2, 1, 8, 4, V, "f32", 0.5, seed=93), "cuda", "packed", lengths=[rows, rows, rows - 3, rows])
    print(compare_all(b, run_gpu(b, "grpo"), run_oracle(b, "grpo"), **F32_TOL), flush=True)

"""The f32 contraction kernel of aligned operands: against the oracle, and to the bit against the general kernel that unaligned ones take."""
import pytest
import torch

from paper_2603_16435_amd import binding, synth
from parity_util import compare_all, run_gpu, run_oracle

pytestmark = pytest.mark.gpu
F32_TOL = dict(loss_tol=1e-5, logp_atol=2e-5, grad_tol=1e-4)          # the tolerances of the parity tests
OUT = ("loss", "seq_loss", "logprob", "lse", "entropy", "coeff", "d_hidden", "d_weight", "target_col", "target_logit")


def off_grid(t):
    buf = torch.empty(t.numel() + 1, dtype=t.dtype, device=t.device)
    buf[1:].copy_(t.flatten())
    return buf[1:].view(t.shape)


# wide tiles in the logits from 512 tiles of 256 x 64 on; one, two, three, five slabs of K, whole or with a tail
@pytest.mark.parametrize("H,V,lengths", [(4, 33001, [130, 1, 0, 99]), (32, 33001, [64, 64, 64, 64]), (36, 33001, [129, 0, 3, 61]),
                                         (96, 40000, [193, 1, 1, 1]), (132, 33001, [200, 1, 0, 99])])
@pytest.mark.parametrize("chunk", [0, 256])                  # the logits kept, or (more than 256 tokens) formed again for dS; in scoring neither
def test_aligned_and_unaligned_operands_give_the_same_bits(H, V, lengths, chunk):
    cfg = synth.RolloutConfig("edge", 2, 2, 1, 64, H, V, "f32", 0.5, seed=71)
    b = synth.make_rollouts(cfg, "cuda", "packed", lengths=lengths)
    want = run_gpu(b, "flow", chunk_rows=chunk)
    scored = binding.rl_token_logprob_tempered(b.hidden, b.weight, b.token_ids, b.mask, 1.0, b.cu_seqlens)
    b.weight, b.hidden = off_grid(b.weight), off_grid(b.hidden)
    got = run_gpu(b, "flow", chunk_rows=chunk)
    for name in OUT:
        assert torch.equal(getattr(got, name), getattr(want, name)), name
    again = binding.rl_token_logprob_tempered(b.hidden, b.weight, b.token_ids, b.mask, 1.0, b.cu_seqlens)
    for lp, lse in (scored, again):
        assert torch.equal(lp, want.logprob) and torch.equal(lse, want.lse)


@pytest.mark.parametrize("chunk", [0, 1024])
def test_wide_tiles_in_every_contraction(chunk):
    cfg = synth.RolloutConfig("edge", 2, 2, 1, 64, 228, 33001, "f32", 0.5, seed=72)
    b = synth.make_rollouts(cfg, "cuda", "packed", lengths=[900, 0, 893, 9])        # K of dW 1802: 26 past a slab
    ref = run_oracle(b, "grpo")
    print(compare_all(b, run_gpu(b, "grpo", chunk_rows=chunk), ref, **F32_TOL), flush=True)

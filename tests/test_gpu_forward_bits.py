"""A token's log-prob, lse and entropy are the same bits however many rows are staged with it: the f32 forward takes square, wide or narrow
tiles by the size of the chunk, and all add in the same order."""
import pytest
import torch

from paper_2603_16435_amd import binding, synth
from parity_util import run_gpu

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("V,rows,tau", [(1000, 9000, 0.0), (300, 17000, 0.8),       # wide tiles from 8192 / 16384 staged rows on
                                          (30000, 8000, 0.0)])                     # square ones, fifteen rounds of them; wide; narrow
def test_f32_log_probs_do_not_depend_on_the_chunk(V, rows, tau):
    cfg = synth.RolloutConfig("bits", 2, 4, 1, rows // 8, 68, V, "f32", 0.5, seed=61)
    b = synth.make_rollouts(cfg, "cuda", "packed", lengths=[rows // 8] * 8)
    want = run_gpu(b, "grpo", backward=False, temperature=tau)
    for chunk in (4096, 256):
        got = run_gpu(b, "grpo", chunk_rows=chunk, backward=False, temperature=tau)
        for name in ("logprob", "lse", "entropy", "target_logit", "loss", "coeff"):
            assert torch.equal(getattr(got, name), getattr(want, name)), (chunk, name)


def test_f32_static_scoring_call_in_smaller_chunks_gives_the_same_bits():
    # a million rows: the plan fits the static array with 4096-row chunks (narrow tiles), the workspace call takes 32768 (wide)
    cfg = synth.RolloutConfig("bits", 1, 8, 1, 129400, 4, 1000, "f32", 0.5, seed=62)
    b = synth.make_rollouts(cfg, "cuda", "packed", lengths=[129400] * 8)
    logp, lse = (torch.empty(b.R, dtype=torch.float32, device="cuda") for _ in range(2))
    binding.rl_token_logprob_static(b.hidden, b.weight, b.token_ids, b.mask, b.cu_seqlens, logp, lse)
    ref_lp, ref_lse = binding.rl_token_logprob(b.hidden, b.weight, b.token_ids, b.mask, b.cu_seqlens)
    assert torch.equal(logp, ref_lp) and torch.equal(lse, ref_lse)

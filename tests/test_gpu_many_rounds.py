"""dX + dW of chunks beyond 32768 rows at a head whose dW comes in more than 24 rounds of tiles: two launches, of which the chunk's number of tokens
picks one on the device."""
import dataclasses

import pytest
import torch

from paper_2603_16435_amd import synth
from parity_util import run_gpu

pytestmark = pytest.mark.gpu
H, V = 2816, 152064                                  # 11 x 594 tiles of dW: 25.5 rounds


@pytest.mark.parametrize("mode", ["recompute", "stash"])
def test_few_tokens_in_many_rows(mode):
    """The bits of the same tokens in a batch of few rows, which reads W as it is stored."""
    cfg = synth.RolloutConfig("rounds", 1, 2, 1, 8, H, V, "bf16", 0.5, seed=95)
    few = synth.make_rollouts(cfg, "cuda", "packed", lengths=[40, 300])
    R = 32768 + 300
    many = dataclasses.replace(few)
    at = torch.cat([torch.arange(40), torch.arange(R - 300, R)]).cuda()
    for name in ("hidden", "token_ids", "mask", "old_logprob", "ref_logprob"):
        v = getattr(few, name)
        w = torch.zeros(R, *v.shape[1:], dtype=v.dtype, device="cuda")
        w[at] = v
        setattr(many, name, w)
    many.cu_seqlens = torch.tensor([0, 40, R], dtype=torch.int32, device="cuda")
    want, got = run_gpu(few, "grpo", mode=mode), run_gpu(many, "grpo", mode=mode)
    for name in ("loss", "seq_loss", "d_weight"):
        assert torch.equal(getattr(got, name), getattr(want, name)), name
    for name in ("logprob", "lse", "coeff", "d_hidden"):
        assert torch.equal(getattr(got, name)[at], getattr(want, name)), name


@pytest.mark.parametrize("tokens", [33280, 33281])   # the last chunk of the one form, the first of the other
def test_one_chunk_of_many_tokens(tokens):
    """Against the same batch in two chunks.  dX does not depend on the chunks; dW is one sum of `tokens` products in f32 or two added up:
    1e-4 of the largest entry, as between any two orders of such sums here."""
    cfg = synth.RolloutConfig("rounds", 2, 4, 1, 8, H, V, "bf16", 0.5, seed=96)
    n = tokens // 8
    b = synth.make_rollouts(cfg, "cuda", "packed", lengths=[n] * 7 + [tokens - 7 * n])
    want, got = run_gpu(b, "flow", mode="stash", chunk_rows=16896), run_gpu(b, "flow", mode="stash")
    assert torch.equal(got.loss, want.loss) and torch.equal(got.d_hidden, want.d_hidden)
    assert bool(got.d_weight.isfinite().all()) and float((got.d_weight - want.d_weight).abs().max()) <= 1e-4 * float(want.d_weight.abs().max())

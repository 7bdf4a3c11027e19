"""Hidden states that span 4 GiB or more take another form of load addresses in the bf16 logits: same bits as the same rows close together."""
import dataclasses

import pytest
import torch

from paper_2603_16435_amd import synth
from parity_util import run_gpu

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("H,kw", [(512, dict(mode="recompute")), (512, dict(mode="stash", chunk_rows=1 << 22)), (520, dict(mode="recompute"))])
def test_rows_more_than_4_gib_apart(H, kw):
    cfg = synth.RolloutConfig("far", 1, 2, 1, 8, H, 300, "bf16", 0.5, seed=91)
    near = synth.make_rollouts(cfg, "cuda", "packed", lengths=[40, 300])
    R = (1 << 32) // (2 * H) + 512                              # 512 rows past the 4 GiB
    far = dataclasses.replace(near)
    at = torch.cat([torch.arange(40), torch.arange(R - 300, R)]).cuda()
    for name in ("hidden", "token_ids", "mask", "old_logprob", "ref_logprob"):
        v = getattr(near, name)
        w = torch.zeros(R, *v.shape[1:], dtype=v.dtype, device="cuda")
        w[at] = v
        setattr(far, name, w)
    far.cu_seqlens = torch.tensor([0, 40, R], dtype=torch.int32, device="cuda")
    kw = dict(kw)
    want = run_gpu(near, "grpo", mode=kw["mode"])
    got = run_gpu(far, "grpo", **kw)
    for name in ("loss", "seq_loss", "d_weight"):
        assert torch.equal(getattr(got, name), getattr(want, name)), name
    for name in ("logprob", "lse", "entropy", "coeff", "d_hidden"):
        assert torch.equal(getattr(got, name)[at], getattr(want, name)), name
    assert int((got.d_hidden != 0).any(dim=1).sum()) <= 340

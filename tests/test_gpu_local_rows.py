"""The preparation inside the launch of the logits: each workgroup works out by itself which rows count.  Against the same rows at the head of a batch that is
too large for it (the preparation in launches of its own), to the bit; offsets that decrease, empty sequences, bad tokens, prompts that do not exist."""
import numpy as np
import pytest
import torch

from paper_2603_16435_amd import synth
from parity_util import run_gpu
from test_gpu_f32_tiles import OUT

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype,V,R,B", [("bf16", 1000, 128, 5), ("bf16", 1000, 64, 64), ("bf16", 300, 1, 1), ("bf16", 1000, 129, 5), ("f32", 1000, 1024, 64),
                                         ("f32", 1000, 1025, 64), ("f32", 300, 65, 3), ("f32", 20000, 200, 7)])
def test_rows_worked_out_by_every_workgroup(dtype, V, R, B):
    rng = np.random.default_rng(R * 101 + B)
    cu = np.concatenate([[0], np.sort(rng.integers(0, R + 1, B - 1)), [R]]).astype(np.int32)
    if B > 3:
        cu[2] = max(int(cu[1]) - 3, 0)                                       # goes back: that sequence keeps nothing
    P = 3
    group = rng.integers(0, P, B).astype(np.int32)
    if B > 4:
        group[4] = -1
    ids = rng.integers(0, V, R).astype(np.int32)
    ids[rng.random(R) < 0.1] = V
    mask = (rng.random(R) < 0.8).astype(np.uint8)
    b = synth.make_rollouts(synth.RolloutConfig("local", P, 1, 1, 4, 64, V, dtype, 0.5, seed=6), "cuda", "packed", lengths=[R + 4096, 0, 0])
    d = lambda a: torch.from_numpy(a).cuda()
    pad = lambda a: np.concatenate([a, np.zeros(4096, a.dtype)])
    b.cu_seqlens, b.group_idx, b.rewards = d(cu), d(group), torch.from_numpy(rng.random(B).astype(np.float32)).cuda()
    b.mask, b.token_ids = d(pad(mask)), d(pad(ids))
    want = run_gpu(b, "grpo", backward=False)
    for name in ("hidden", "mask", "token_ids", "old_logprob", "ref_logprob"):
        setattr(b, name, getattr(b, name)[:R].contiguous())
    b.R = R
    got = run_gpu(b, "grpo", backward=False)
    assert got.stats_dict() == want.stats_dict()
    assert R == 1 or got.stats_dict()["n_bad_token"] > 0
    assert torch.equal(got.seq_len, want.seq_len) and torch.equal(got.loss, want.loss) and torch.equal(got.advantages, want.advantages)
    for name in OUT:
        a, w = getattr(got, name), getattr(want, name)
        if a is not None and a.shape[:1] == (R,):
            assert torch.equal(a, w[:R]), name
    lp = run_gpu(b, "grpo")                                                    # with the backward
    for name in ("logprob", "lse", "coeff"):
        assert torch.equal(getattr(lp, name), getattr(got, name)), name

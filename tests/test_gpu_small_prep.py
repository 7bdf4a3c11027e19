"""The one-launch preparation of small batches, at its edges: sequences that begin and end inside, at and across 64-row words, rows of no
sequence, bad tokens, prompts without members; and the batch one row, one sequence or one prompt beyond its range."""
import numpy as np
import pytest
import torch

from oracle import policy_oracle as orc
from paper_2603_16435_amd import synth
from parity_util import np_bits, run_gpu

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("B,R,P", [(1, 1, 0), (1, 4096, 0), (3, 200, 0), (15, 4096, 0), (16, 4095, 0), (17, 1000, 0), (64, 4096, 0), (64, 130, 32), (64, 2049, 33),
                                   (65, 1025, 32), (128, 4096, 0), (128, 130, 0), (129, 4096, 0), (5, 4097, 0)])
def test_index_work_of_small_batches(B, R, P):
    rng = np.random.default_rng(B * 10007 + R)
    cuts = np.sort(rng.integers(0, R + 1, B - 1))
    if R > 128:
        cuts = np.sort(np.where(rng.random(B - 1) < 0.4, cuts // 64 * 64, cuts))        # some at words' borders, some sequences empty
    cu = np.concatenate([[0], cuts, [R if B % 2 else R - R // 10]]).astype(np.int32)      # rows behind the last sequence
    P = P or max(1, B // 3)
    cfg = synth.RolloutConfig("prep", P, 1, 1, 4, 8, 300, "f32", 0.5, seed=5)
    b = synth.make_rollouts(cfg, "cuda", "packed", lengths=[R] + [0] * (P - 1))
    mask = (rng.random(R) < 0.8).astype(np.uint8)
    ids = rng.integers(0, 300, R).astype(np.int32)
    ids[rng.random(R) < 0.05] = 300
    group = rng.integers(0, P, B).astype(np.int32)
    if B > 4:
        group[2] = P                                                                   # names no prompt
    d = lambda a: torch.from_numpy(a).cuda()
    b.mask, b.token_ids, b.cu_seqlens, b.group_idx = d(mask), d(ids), d(cu), d(group)
    b.rewards = torch.from_numpy(rng.random(B).astype(np.float32)).cuda()
    got = run_gpu(b, "grpo", backward=False)
    want = orc.compact_rows(mask, ids, cu, 300, group, P)
    T = want["row_map"].size
    np.testing.assert_array_equal(got.row_map.cpu().numpy()[:T], want["row_map"])
    assert (got.row_map.cpu().numpy()[T:] == -1).all()
    np.testing.assert_array_equal(got.seq_len.cpu().numpy(), want["seq_len"])
    np.testing.assert_array_equal(got.group_count.cpu().numpy(), orc.group_count(group, P))
    counts = np.zeros(R, bool); counts[want["row_map"]] = True
    col = got.target_col.cpu().numpy()
    np.testing.assert_array_equal(col, np.where(counts, ids, -1))
    assert not np_bits(got.logprob)[~counts].any()
    adv = np.zeros(B)
    rew = b.rewards.cpu().numpy().astype(np.float64)
    for p in range(P):
        m = group == p
        if m.any():
            adv[m] = (rew[m] - rew[m].mean()) / (rew[m].std() + 1e-6)
    np.testing.assert_allclose(got.advantages.cpu().numpy(), adv, rtol=1e-6, atol=1e-6)    # f32 rounding of an f64 value of order one

"""Row compaction and advantages where their launches change form: as many sequences as one workgroup adds up, and one more."""
import numpy as np
import pytest
import torch

from paper_2603_16435_amd import synth
from parity_util import compare_all, run_gpu, run_oracle

pytestmark = pytest.mark.gpu
BF16_TOL = dict(loss_tol=1e-2, logp_atol=2e-3, grad_tol=2e-2)          # the tolerances of the parity tests


@pytest.mark.parametrize("P,G", [(256, 4), (205, 5), (300, 1), (1, 257)])      # 1024 and 1025 sequences; more prompts, more members than a workgroup has threads
def test_many_short_sequences(P, G):
    rng = np.random.default_rng(9)
    lengths = rng.integers(0, 4, P * G).tolist()
    cfg = synth.RolloutConfig("many", P, G, 1, 4, 128, 300, "bf16", 0.5, seed=41)
    b = synth.make_rollouts(cfg, "cuda", "padded", lengths=lengths)
    for objective in ("grpo", "flow"):
        ref = run_oracle(b, objective)
        for mode in ("recompute", "stash"):
            print(objective, mode, compare_all(b, run_gpu(b, objective, chunk_rows=512, mode=mode), ref, **BF16_TOL), flush=True)

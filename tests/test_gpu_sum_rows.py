"""Sums over the vocabulary tiles by workgroups of 16 rows: rows one short of a workgroup, one, one past it; tiles fewer and more than there are slices."""
import pytest

from paper_2603_16435_amd import synth
from parity_util import compare_all, run_gpu, run_oracle

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("V", [300, 16384, 16640, 33000])
@pytest.mark.parametrize("lengths", [[15, 0], [16, 1], [100, 29]])
@pytest.mark.parametrize("mode", ["stash", "recompute"])
def test_sums(V, lengths, mode):
    b = synth.make_rollouts(synth.RolloutConfig("sums", 1, 2, 1, 64, 128, V, "bf16", 0.5, seed=98), "cuda", "packed", lengths=lengths)
    print(compare_all(b, run_gpu(b, "grpo", mode=mode), run_oracle(b, "grpo"), loss_tol=1e-2, logp_atol=2e-3, grad_tol=2e-2), flush=True)      # as in the parity tests

"""dX of f32 batches out of dS^T and W as they are stored: to the bit what the transposed copies give (a weight off the 16-byte grid takes those), and against
the oracle."""
import pytest
import torch

from paper_2603_16435_amd import synth
from parity_util import compare_all, run_gpu, run_oracle
from test_gpu_f32_tiles import F32_TOL, off_grid

pytestmark = pytest.mark.gpu


# vocabularies of whole tiles, one entry past one (255 rows of W that do not exist), two slabs short of one; columns one piece past a tile of 64, and one
# piece in all; few slabs of K in a slice; tokens one past and one short of a tile
@pytest.mark.parametrize("H,V,lengths", [(68, 33024, [130, 1, 0, 126]), (4, 33025, [64, 0, 64, 127]), (64, 32960, [1, 0, 0, 0]),
                                         (708, 600, [1000, 300, 0, 621]), (1024, 257, [600, 600, 600, 247])])
@pytest.mark.parametrize("chunk", [0, 1024])
def test_dx_reads_its_operands_k_major(H, V, lengths, chunk):
    cfg = synth.RolloutConfig("kmajor", 2, 2, 1, 64, H, V, "f32", 0.5, seed=75)
    b = synth.make_rollouts(cfg, "cuda", "packed", lengths=lengths)
    got = run_gpu(b, "grpo", chunk_rows=chunk)
    if H * V <= 1 << 20:
        print(compare_all(b, got, run_oracle(b, "grpo"), **F32_TOL), flush=True)
    b.weight = off_grid(b.weight)
    want = run_gpu(b, "grpo", chunk_rows=chunk)
    assert torch.equal(got.d_hidden, want.d_hidden) and torch.equal(got.d_weight, want.d_weight)

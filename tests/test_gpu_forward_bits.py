"""A token's log-prob, lse and entropy are the same bits however many rows are staged with it: the f32 forward takes wide or narrow tiles by the
size of the chunk, square ones where operands off the 16-byte grid come in many rounds of them, and all add in the same order."""
import pytest
import torch

from paper_2603_16435_amd import binding, synth
from parity_util import run_gpu
from test_gpu_f32_tiles import OUT, off_grid

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("V,rows,tau", [(1000, 9000, 0.0), (300, 17000, 0.8),       # wide tiles from 8192 / 16384 staged rows on
                                          (30000, 8000, 0.0)])                     # wide in many rounds; narrow
def test_f32_log_probs_do_not_depend_on_the_chunk(V, rows, tau):
    cfg = synth.RolloutConfig("bits", 2, 4, 1, rows // 8, 68, V, "f32", 0.5, seed=61)
    b = synth.make_rollouts(cfg, "cuda", "packed", lengths=[rows // 8] * 8)
    want = run_gpu(b, "grpo", backward=False, temperature=tau)
    for chunk in (4096, 256):
        got = run_gpu(b, "grpo", chunk_rows=chunk, backward=False, temperature=tau)
        for name in ("logprob", "lse", "entropy", "target_logit", "loss", "coeff"):
            assert torch.equal(getattr(got, name), getattr(want, name)), (chunk, name)


# narrow tiles one short of and at a CU each, one past it (two on some), at two each, one past that; one, two and broken bands of rows of tiles; a K tail.  The same
# tokens among 9000 rows take wide tiles
@pytest.mark.parametrize("V,tiles_n", [(2048, 31), (2048, 32), (2000, 33), (2048, 64), (2048, 65), (4096, 17), (4096, 32), (3000, 22), (10240, 7)])
def test_f32_log_probs_do_not_depend_on_how_the_tiles_fill_the_chip(V, tiles_n):
    cfg = synth.RolloutConfig("bits", 1, 1, 1, 8, 292, V, "f32", 0.5, seed=64)
    b = synth.make_rollouts(cfg, "cuda", "packed", lengths=[9000])
    n = 16 * tiles_n - 5
    score = lambda r: binding.rl_token_logprob_tempered(b.hidden[:r], b.weight, b.token_ids[:r], b.mask[:r], 0.9, torch.tensor([0, r], dtype=torch.int32, device="cuda"))
    for got, want in zip(score(n), score(9000)):
        assert torch.equal(got, want[:n])


@pytest.mark.parametrize("backward", [False, True])                        # True: the logits are kept as well
def test_f32_square_tiles_of_unaligned_operands_give_the_same_bits(backward):
    cfg = synth.RolloutConfig("bits", 2, 4, 1, 1000, 68, 30000, "f32", 0.5, seed=63)          # 118 x 32 square tiles: fifteen rounds
    b = synth.make_rollouts(cfg, "cuda", "packed", lengths=[1000] * 7 + [937])
    want = run_gpu(b, "flow", backward=backward)
    b.weight, b.hidden = off_grid(b.weight), off_grid(b.hidden)
    got = run_gpu(b, "flow", backward=backward)
    for name in OUT:
        if backward or not name.startswith("d_"):
            assert torch.equal(getattr(got, name), getattr(want, name)), name


def test_f32_static_scoring_call_in_smaller_chunks_gives_the_same_bits():
    # a million rows: the plan fits the static array with 4096-row chunks (narrow tiles), the workspace call takes 32768 (wide)
    cfg = synth.RolloutConfig("bits", 1, 8, 1, 129400, 4, 1000, "f32", 0.5, seed=62)
    b = synth.make_rollouts(cfg, "cuda", "packed", lengths=[129400] * 8)
    logp, lse = (torch.empty(b.R, dtype=torch.float32, device="cuda") for _ in range(2))
    binding.rl_token_logprob_static(b.hidden, b.weight, b.token_ids, b.mask, b.cu_seqlens, logp, lse)
    ref_lp, ref_lse = binding.rl_token_logprob(b.hidden, b.weight, b.token_ids, b.mask, b.cu_seqlens)
    assert torch.equal(logp, ref_lp) and torch.equal(lse, ref_lse)

"""The loss of a batch is added up by the workgroup that forms its last sequence's loss (up to 64 sequences) or by a launch of its own: either
side of the border, and on replays of a captured call."""
import pytest
import torch

from paper_2603_16435_amd import binding, synth
from parity_util import compare_all, run_gpu, run_oracle

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("P,G", [(16, 4), (13, 5), (1, 64), (65, 1)])
@pytest.mark.parametrize("dtype,mode", [("f32", None), ("bf16", "stash"), ("bf16", "recompute")])
def test_as_many_sequences_as_finish_inline_and_one_more(P, G, dtype, mode):
    cfg = synth.RolloutConfig("finish", P, G, 1, 4, 128, 300, dtype, 0.5, seed=43)
    b = synth.make_rollouts(cfg, "cuda", "packed", lengths=[(3 * i) % 5 for i in range(P * G)])
    tol = dict(loss_tol=1e-5, logp_atol=2e-5, grad_tol=1e-4) if dtype == "f32" else dict(loss_tol=1e-2, logp_atol=2e-3, grad_tol=2e-2)
    for objective in ("grpo", "flow"):
        print(objective, compare_all(b, run_gpu(b, objective, mode=mode), run_oracle(b, objective), **tol), flush=True)


@pytest.mark.parametrize("dtype,H", [("f32", 64), ("bf16", 512)])
def test_replays_of_a_captured_call(dtype, H):
    cfg = synth.RolloutConfig("graph", 2, 4, 1, 40, H, 600, dtype, 0.5, seed=44)
    b = synth.make_rollouts(cfg, "cuda", "packed", lengths=[40, 1, 0, 17, 33, 8, 25, 40])
    batch = binding.make_batch(b.hidden, b.weight, b.token_ids, b.mask, b.cu_seqlens, b.group_idx, b.rewards, b.old_logprob, b.ref_logprob, b.log_z, 2)
    plan = binding.PolicyLossPlan(batch, binding.make_params(), "cuda:0", b.hidden.dtype)
    names = ("loss", "seq_loss", "d_log_z", "logprob", "d_hidden", "d_weight")
    stream = torch.cuda.Stream()
    with torch.cuda.stream(stream):
        r = plan.run(binding.RL_OBJ_FLOW)
    torch.cuda.synchronize()
    want = {n: getattr(r, n).clone() for n in names}
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=stream):
        plan.run(binding.RL_OBJ_FLOW)
    for _ in range(4):
        for n in names:
            getattr(r, n).fill_(7.0)                     # eager work between the replays
        graph.replay()
        torch.cuda.synchronize()
        for n in names:
            assert torch.equal(getattr(r, n), want[n]), n

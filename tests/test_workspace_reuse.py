"""The room for kept logits is optional: a workspace sized for a larger batch, or for the recomputing backward, serves the default mode."""
import ctypes as C
import itertools
import os

import pytest
import torch

from paper_2603_16435_amd import binding, synth
from parity_util import run_gpu

built = pytest.mark.skipif(not os.path.exists(binding.LIB_PATH), reason="library not built")
FAKE = 0x100000


def _size(R, H, V, dtype, **prm):
    b, n = binding.rl_batch(), C.c_size_t(0)
    b.R, b.H, b.V, b.B, b.P, b.dtype = R, H, V, 4, 2, dtype
    p = binding.make_params(**prm)
    assert binding.lib().rl_workspace_bytes(C.byref(b), C.byref(p), 1, C.byref(n)) == 0
    return n.value


@built
@pytest.mark.skipif(torch.cuda.is_available(), reason="the accepted calls would run, on pointers that are none")
@pytest.mark.parametrize("dtype,H,V", [("bf16", 3584, 152064), ("bf16", 512, 32000), ("bf16", 520, 50257), ("bf16", 128, 1000), ("f32", 768, 50257)])
def test_a_workspace_for_more_rows_or_for_recomputing_is_accepted(dtype, H, V):
    dt = binding.RL_BF16 if dtype == "bf16" else binding.RL_F32

    def accepted(R, nbytes, **prm):
        b, out = binding.rl_batch(), binding.rl_outputs()
        b.R, b.H, b.V, b.B, b.P, b.dtype = R, H, V, 4, 2, dt
        for f in ("hidden", "weight", "token_ids", "mask", "cu_seqlens", "group_idx", "rewards", "old_logprob", "ref_logprob"):
            setattr(b, f, FAKE)
        out.loss = out.d_hidden = out.d_weight = FAKE
        status = binding.lib().rl_policy_loss_fwd_bwd(C.byref(b), C.byref(binding.make_params(**prm)), 0, C.byref(out), FAKE, nbytes, None)
        assert status in (5, 6)                      # refused for its workspace, or past all checks and then stopped by the missing GPU
        return status == 6

    rows = (1, 100, 256, 257, 5000, 11540, 12000, 16128, 16384, 16385, 20000, 32768, 32769, 100000)
    for R in rows:
        need = _size(R, H, V, dt, backward_mode="recompute")
        assert need <= _size(R, H, V, dt)
        assert accepted(R, need) and accepted(R, need, backward_mode="recompute") and not accepted(R, need - 256), R
    for small, large in itertools.combinations(rows, 2):
        assert accepted(small, _size(large, H, V, dt)), (small, large)


@built
def test_the_plan_takes_a_small_workspace_when_memory_is_short(monkeypatch):
    b = binding.rl_batch()
    b.R, b.H, b.V, b.B, b.P, b.dtype = 300, 512, 1000, 4, 2, binding.RL_BF16
    small = _size(300, 512, 1000, binding.RL_BF16, backward_mode="recompute")
    real = binding._workspace

    def short(nbytes, device):
        if nbytes > small:
            raise torch.OutOfMemoryError("no memory")
        return real(nbytes, device)

    monkeypatch.setattr(binding, "_workspace", short)
    assert binding.PolicyLossPlan(b, binding.make_params(), "cpu", torch.bfloat16).ws.numel() == small
    with pytest.raises(torch.OutOfMemoryError):
        binding.PolicyLossPlan(b, binding.make_params(max_seq_len=300, backward_mode="stash"), "cpu", torch.bfloat16)


@pytest.mark.gpu
@pytest.mark.parametrize("H,V", [(512, 700), (776, 5000)])
def test_without_room_for_kept_logits_they_are_recomputed(H, V):
    cfg = synth.RolloutConfig("room", 2, 2, 1, 64, H, V, "bf16", 0.5, seed=84)
    b = synth.make_rollouts(cfg, "cuda", "packed", lengths=[300, 1, 0, 64])
    want = run_gpu(b, "flow")
    c = b.cfg
    batch = binding.make_batch(b.hidden, b.weight, b.token_ids, b.mask, b.cu_seqlens, b.group_idx, b.rewards, b.old_logprob, b.ref_logprob, b.log_z, c.P)
    plan = binding.PolicyLossPlan(batch, binding.make_params(c.clip_eps, c.kl_coef, c.beta, c.adv_eps, c.adv_std_ddof), "cuda", torch.bfloat16)
    need = _size(b.R, H, V, binding.RL_BF16, backward_mode="recompute")
    assert need < plan.ws.numel()
    whole = plan.ws
    plan.ws = whole[:need]
    whole[need:] = 0x5A
    got = plan.run(binding.RL_OBJ_FLOW)
    torch.cuda.synchronize()
    for name in ("loss", "seq_loss", "logprob", "lse", "entropy", "coeff", "d_hidden", "d_weight"):
        assert torch.equal(getattr(got, name), getattr(want, name)), name
    assert bool((whole[need:] == 0x5A).all())

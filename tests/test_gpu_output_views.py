"""Tensors that share memory: gradients that start at any element of a buffer, a weight off the 16-byte grid, outputs in the place of inputs."""
import pytest
import torch

from paper_2603_16435_amd import binding, synth
from parity_util import compare_all, run_oracle
from test_gpu_f32_tiles import F32_TOL

pytestmark = pytest.mark.gpu


def _plan(b, mode, chunk):
    c = b.cfg
    batch = binding.make_batch(b.hidden, b.weight, b.token_ids, b.mask, b.cu_seqlens, b.group_idx, b.rewards, b.old_logprob,
                               b.ref_logprob, b.log_z, c.P)
    prm = binding.make_params(chunk_rows=chunk, backward_mode=mode, max_seq_len=int(b.lengths.max()) if mode == "stash" else 0)
    return binding.PolicyLossPlan(batch, prm, "cuda", b.hidden.dtype)


@pytest.mark.parametrize("dtype,H,V,mode,chunk", [
    ("bf16", 384, 20001, "stash", 0),           # dX in slices, whole tiles and edges
    ("bf16", 384, 20001, "recompute", 0),
    ("bf16", 136, 600, "recompute", 256),       # two chunks: dW is read and added to
    ("bf16", 256, 700, "stash", 256),
    ("f32", 68, 900, "recompute", 256),
])
@pytest.mark.parametrize("off", [1, 3])
def test_gradients_may_start_at_any_element(dtype, H, V, mode, chunk, off):
    cfg = synth.RolloutConfig("views", 2, 2, 1, 64, H, V, dtype, 0.5, seed=71)
    b = synth.make_rollouts(cfg, "cuda", "padded", lengths=[200, 56, 1, 160])
    plan = _plan(b, mode, chunk)
    want = plan.run(binding.RL_OBJ_FLOW)
    dX = torch.full((b.R * H + 2 * off + 8,), 7.0, dtype=b.hidden.dtype, device="cuda")      # one guard on either side
    dW = torch.full((V * H + 2 * off + 8,), 7.0, dtype=torch.float32, device="cuda")
    plan.out.d_hidden, plan.out.d_weight = dX[off:].data_ptr(), dW[off:].data_ptr()
    plan.run(binding.RL_OBJ_FLOW)
    torch.cuda.synchronize()
    assert dX[off:].data_ptr() % 16 and dW[off:].data_ptr() % 16
    assert torch.equal(dX[off:off + b.R * H], want.d_hidden.flatten()) and torch.equal(dW[off:off + V * H], want.d_weight.flatten())
    for g, n in ((dX, b.R * H), (dW, V * H)):
        assert bool((g[:off] == 7.0).all()) and bool((g[off + n:] == 7.0).all())


@pytest.mark.parametrize("H,mode", [(136, "auto"), (256, "auto"), (256, "recompute")])
def test_a_workspace_sized_for_an_aligned_weight_serves_one_that_is_not(H, mode):
    cfg = synth.RolloutConfig("views", 2, 2, 1, 64, H, 700, "bf16", 0.5, seed=72)
    b = synth.make_rollouts(cfg, "cuda", "packed", lengths=[20, 3, 0, 40])
    plan = _plan(b, mode, 0)
    buf = torch.empty(b.weight.numel() + 1, dtype=torch.bfloat16, device="cuda")
    buf[1:].copy_(b.weight.flatten())
    plan.batch.weight = buf[1:].data_ptr()
    got = plan.run(binding.RL_OBJ_GRPO)
    b.weight = buf[1:].view(b.weight.shape)
    want = _plan(b, mode, 0).run(binding.RL_OBJ_GRPO)
    torch.cuda.synchronize()
    assert torch.equal(got.d_weight, want.d_weight) and torch.equal(got.d_hidden, want.d_hidden) and torch.equal(got.loss, want.loss)


@pytest.mark.parametrize("P,G", [(300, 3), (8, 4)])       # the preparation and the finish of the loss in launches of their own, or with others
@pytest.mark.parametrize("dtype,mode,objective", [("bf16", "recompute", "GRPO"), ("bf16", "stash", "GRPO"), ("bf16", "auto", "FLOW"), ("bf16", "stash", "FLOW"),
                                                  ("f32", "auto", "FLOW")])
def test_outputs_in_the_place_of_inputs(P, G, dtype, mode, objective):
    """Rewards turn into advantages, token ids into target columns (or target logits, entropies), log-Z into its gradient in place: an input is
    only overwritten when the call has read it everywhere.  300 prompts: the advantages of more than one workgroup."""
    objective = getattr(binding, "RL_OBJ_" + objective)
    cfg = synth.RolloutConfig("views", P, G, 1, 4, 128, 300, dtype, 0.5, seed=73)
    b = synth.make_rollouts(cfg, "cuda", "padded", lengths=[(7 * i) % 5 for i in range(P * G)])
    plan = _plan(b, mode, 0)
    plan.res.target_col, plan.res.target_logit = torch.empty(b.R, dtype=torch.int32, device="cuda"), torch.empty(b.R, device="cuda")
    plan.out.target_col, plan.out.target_logit = plan.res.target_col.data_ptr(), plan.res.target_logit.data_ptr()
    names = ("loss", "seq_loss", "logprob", "advantages", "seq_len", "target_col", "target_logit", "entropy", "d_hidden", "d_weight", "d_log_z")
    res = plan.run(objective)
    want = {n: getattr(res, n).clone() for n in names}
    for field, inp in (("advantages", "rewards"), ("seq_len", "cu_seqlens"), ("target_col", "token_ids"), ("target_logit", "token_ids"),
                       ("entropy", "token_ids"), ("d_log_z", "log_z")):
        keep, own = getattr(b, inp).clone(), getattr(plan.out, field)
        setattr(plan.out, field, getattr(b, inp).data_ptr())
        for n in names:
            getattr(plan.res, n).zero_()
        plan.run(objective)
        torch.cuda.synchronize()
        assert torch.equal(getattr(b, inp)[:want[field].numel()].view(want[field].dtype), want[field]), field
        for n in names:
            assert n == field or torch.equal(getattr(plan.res, n), want[n]), (field, n)
        getattr(b, inp).copy_(keep)
        setattr(plan.out, field, own)


# a small batch, whose one launch for both gradients reads the inputs themselves and steps aside; K-major operands of dX; rows that do not count become zero in place
@pytest.mark.parametrize("H,V,lengths,layout", [(128, 1024, [100, 99, 1, 156], "packed"), (64, 300, [30, 0, 1, 12], "padded"), (68, 33024, [130, 1, 0, 126], "packed")])
def test_gradients_in_the_place_of_inputs(H, V, lengths, layout):
    b = synth.make_rollouts(synth.RolloutConfig("views", 2, 2, 1, 64, H, V, "f32", 0.5, seed=74), "cuda", layout, lengths=lengths)
    ref = run_oracle(b, "flow")
    # the flow weight is exp of a sum of n <= 156 f32 log-probs below 16, each rounded by up to 2^-21: at random signs 4 sqrt(n / 3) 2^-21 = 1.4e-5 of a term, and the
    # terms of d_log_z, whose differences remain, are up to 2 x 1.2 x 16 / B = 9.6: 1.4e-4
    tol = dict(F32_TOL, loss_tol=1.4e-4)
    hidden, weight = b.hidden.clone(), b.weight.clone()
    got = {}
    for name, inp in (("d_hidden", "hidden"), ("d_weight", "weight")):
        plan = _plan(b, "auto", 0)
        setattr(plan.out, name, getattr(b, inp).data_ptr())
        setattr(plan.res, name, getattr(b, inp))
        res = plan.run(binding.RL_OBJ_FLOW)
        torch.cuda.synchronize()
        got[name] = (res.d_hidden.clone(), res.d_weight.clone())
        b.hidden.copy_(hidden), b.weight.copy_(weight)
        res.d_hidden, res.d_weight = got[name]
        print(name, compare_all(b, res, ref, **tol), flush=True)
    for a, c in zip(*got.values()):
        assert torch.equal(a, c)

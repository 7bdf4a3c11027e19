"""Scoring a few tokens takes a kernel of its own: to the bit what the same tokens get among more rows, and close to the oracle."""
import pytest
import torch

from paper_2603_16435_amd import binding, synth

pytestmark = pytest.mark.gpu


def offsets(R, seqs=1):
    """One sequence of R rows behind empty ones; of more than 64 sequences the preparation is in launches of its own."""
    return torch.tensor([0] * seqs + [R], dtype=torch.int32, device="cuda")


def score(b, hidden, ids, tau, static=False, seqs=1):
    R = hidden.shape[0]
    mask = torch.ones(R, dtype=torch.uint8, device="cuda")
    mask[b.T:] = 0
    cu = offsets(R, seqs)
    if static:
        out = tuple(torch.empty(R, device="cuda") for _ in range(2))
        binding.rl_token_logprob_static(hidden, b.weight, ids, mask, cu, *out, tau)
        return out
    return binding.rl_token_logprob_tempered(hidden, b.weight, ids, mask, tau, cu)


# hidden sizes of one slab, two, a few with and without a tail; vocabularies inside a half tile, at its border, past it, the largest of one round, three rounds
@pytest.mark.parametrize("H,V", [(64, 100), (128, 128), (384, 129), (456, 5000), (576, 32768), (1160, 257), (512, 65537)])
@pytest.mark.parametrize("T", [1, 16, 63, 64, 65, 128])
def test_few_tokens(H, V, T):
    cfg = synth.RolloutConfig("few", 1, 1, 1, 8, H, V, "bf16", 0.5, seed=95)
    b = synth.make_rollouts(cfg, "cuda", "packed", lengths=[T])
    b.token_ids[0], b.token_ids[T - 1] = 0, V - 1
    pad = 300 - T                                                  # the same tokens among rows that do not count: the hot kernel
    hidden = torch.cat([b.hidden, torch.randn(pad, H, device="cuda").to(torch.bfloat16)])
    ids = torch.cat([b.token_ids, torch.zeros(pad, dtype=torch.int32, device="cuda")])
    for tau in (1.0, 0.7):
        want = score(b, hidden, ids, tau)
        for got in (score(b, b.hidden, b.token_ids, tau), score(b, b.hidden, b.token_ids, tau, static=True),
                    score(b, b.hidden, b.token_ids, tau, seqs=70)):
            assert torch.equal(got[0], want[0][:T]) and torch.equal(got[1], want[1][:T])
        assert not want[0][T:].any()
    z = b.hidden.double().cpu() @ b.weight.double().cpu().t()
    ref = torch.log_softmax(z / 0.7, 1).gather(1, b.token_ids.long().cpu()[:, None])[:, 0]
    assert (got[0].double().cpu() - ref).abs().max() < 2e-3         # the tolerance of the parity tests


def test_rows_scattered_and_none_counting():
    cfg = synth.RolloutConfig("few", 1, 1, 1, 8, 256, 3000, "bf16", 0.5, seed=96)
    b = synth.make_rollouts(cfg, "cuda", "packed", lengths=[120])
    full = score(b, b.hidden, b.token_ids, 1.0)
    cu = torch.tensor([0, 50, 120], dtype=torch.int32, device="cuda")
    mask = (torch.arange(120, device="cuda") % 3 == 1).to(torch.uint8)
    lp, lse = binding.rl_token_logprob_tempered(b.hidden, b.weight, b.token_ids, mask, 1.0, cu)
    assert torch.equal(lp, full[0] * mask) and torch.equal(lse, full[1] * mask)
    lp, lse = binding.rl_token_logprob_tempered(b.hidden, b.weight, b.token_ids, torch.zeros_like(mask), 1.0, cu)
    assert not lp.any() and not lse.any()


# a weight larger than the memory-side cache: non-temporal loads, but where its rows are off the lines; more rounds of workgroups than prepare for themselves
@pytest.mark.parametrize("H,V,T", [(4104, 32768, 3), (4160, 32768, 3), (5120, 32000, 100), (1024, 140000, 64), (960, 140000, 65)])
def test_large_weight(H, V, T):
    g = torch.Generator(device="cuda").manual_seed(97)
    n = lambda *s: torch.randn(*s, generator=g, device="cuda", dtype=torch.bfloat16)
    W, X = n(V, H) * H ** -0.5, n(300, H)
    ids = torch.randint(0, V, (300,), generator=g, device="cuda", dtype=torch.int32)
    mask = (torch.arange(300, device="cuda") < T).to(torch.uint8)
    want = binding.rl_token_logprob_tempered(X, W, ids, mask, 1.0, offsets(300))
    for seqs in (1, 70):
        got = binding.rl_token_logprob_tempered(X[:T], W, ids[:T], mask[:T], 1.0, offsets(T, seqs))
        assert torch.equal(got[0], want[0][:T]) and torch.equal(got[1], want[1][:T])

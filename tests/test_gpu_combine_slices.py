"""The softmax partials of a row are added up in 4, 8 or 16 slices, by the number of vocabulary tiles: log-probs, lse and entropy on either side
of each line, for few and for many rows, against 64 bits."""
import pytest
import torch

from paper_2603_16435_amd import synth
from parity_util import run_gpu

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("V", [1, 256, 2048, 2049, 16384, 16385])           # one, one, eight, nine, 64, 65 tiles
def test_partials_in_slices(V, dtype):
    cfg = synth.RolloutConfig("slices", 2, 2, 1, 64, 128, V, dtype, 0.5, seed=97)
    few = None
    for lengths in ([20, 1, 3, 40], [20, 1, 3, 600]):
        b = synth.make_rollouts(cfg, "cuda", "packed", lengths=lengths)
        got = run_gpu(b, "grpo", backward=False)
        z = b.hidden.double() @ b.weight.double().T
        lse = torch.logsumexp(z, 1)
        p = torch.softmax(z, 1)
        want = {"logprob": z.gather(1, b.token_ids.long()[:, None])[:, 0] - lse, "lse": lse, "entropy": lse - (p * z).sum(1)}
        on = b.mask.bool()
        for name, w in want.items():
            # f32 sums of 128 products and of 256 exponentials of a tile: the tolerance of the parity tests
            assert float((getattr(got, name).double() - w)[on].abs().max()) <= (2e-5 if dtype == "f32" else 2e-3), (name, lengths)
        if few is None:
            few = [getattr(got, n)[:24].clone() for n in want]
    assert all(torch.equal(f, getattr(got, n)[:24]) for f, n in zip(few, want))      # the first sequences are the same ones

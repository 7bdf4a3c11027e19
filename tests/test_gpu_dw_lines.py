"""dW in whole lines: lane pairs swap halves, and arrays whose rows lie on 128-byte lines are written past the caches.  Against the oracle, and to the bit
against an array that starts one element later."""
import pytest
import torch

from paper_2603_16435_amd import binding, synth
from parity_util import f64, run_oracle
from test_gpu_output_views import _plan

pytestmark = pytest.mark.gpu


# vocabularies of whole tiles, one short of one (a pair of rows of which one exists) and one past it; rows on lines, or not; one piece of columns in the last
# tile; one chunk, and chunks that are added up
@pytest.mark.parametrize("H,V", [(256, 512), (288, 511), (512, 513), (264, 257), (520, 512)])
@pytest.mark.parametrize("chunk", [0, 256])
def test_dw_in_lines(H, V, chunk):
    cfg = synth.RolloutConfig("lines", 2, 2, 1, 64, H, V, "bf16", 0.5, seed=74)
    b = synth.make_rollouts(cfg, "cuda", "padded", lengths=[200, 56, 1, 160])
    plan = _plan(b, "recompute", chunk)
    buf = torch.full((V * H + 65,), 7.0, dtype=torch.float32, device="cuda")
    got = []
    for off in (32, 33):
        plan.out.d_weight = buf[off:].data_ptr()
        plan.run(binding.RL_OBJ_GRPO)
        torch.cuda.synchronize()
        got.append(buf[off:off + V * H].clone())
        assert bool((buf[:off] == 7.0).all()) and bool((buf[off + V * H:] == 7.0).all())
        buf.fill_(7.0)
    assert torch.equal(got[0], got[1])
    ref = run_oracle(b, "grpo")["d_weight"]
    assert abs(f64(got[0].view(V, H)) - ref).max() <= 2e-2 * abs(ref).max()          # dS in bf16, as in the parity tests

"""log Z added up by the last workgroup of the hidden layer: group borders of 16 prompts and 16 units, the fewest units that take the path and the most that do
not, one workgroup and many, the same workspace used again (the counts start from nothing on every call)."""
import numpy as np
import pytest
import torch

from oracle import logz_head_oracle as lzo
from paper_2603_16435_amd import binding
from parity_util import np_bits
from test_gpu_logz_head import _head

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("P,H,M", [(1, 16, 1), (16, 20, 31), (1, 16, 32), (15, 24, 33), (16, 40, 48), (17, 64, 520), (64, 36, 32), (33, 100, 1024), (2, 8, 1025)])
def test_log_z_sum(P, H, M):
    X, cu, W1, b1, w2, b2, d = _head(P + M, P, H, M, tuple(1 + (7 * i) % 90 for i in range(P)), torch.float32)
    f = lzo.logz_head_forward(np_bits(X), cu.numpy(), W1.numpy(), b1.numpy(), w2.numpy(), float(b2))
    g = [t.cuda() for t in (X, cu, W1, b1, w2, b2)]
    z, ws = binding.rl_logz_head_forward(*g)
    again, _ = binding.rl_logz_head_forward(*g, workspace=ws)
    assert torch.equal(z, again)                                                     # whichever workgroup is last: the same order of sums
    assert np.abs(z.double().cpu().numpy() - f["log_z"]).max() <= 2e-5 * max(1.0, np.abs(f["log_z"]).max())      # the tolerance of the parity tests

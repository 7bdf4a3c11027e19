"""The encode of a few vectors per group: rounds of entries in two buffers, whatever their number.  Codes and residuals equal the float64 oracle's."""
import pytest
import torch

from paper_2603_16435_amd import binding, synth
from test_gpu_rvq_encode import _compare

pytestmark = pytest.mark.gpu


# one round in all; an odd number of rounds, of one and of three a stage; a round that is partly past the stage's end; the largest stages that the scores have room for;
# one vector, a block of 16, one past it, 32; more workgroups than CUs; more entries than there is room for (the kernel of many vectors)
@pytest.mark.parametrize("G,L,N,S", [(1, 1, 1, 64), (3, 16, 3, 256), (2, 5, 3, 704), (9, 16, 2, 320), (1, 16, 3, 2048),
                                     (8, 17, 1, 128), (8, 32, 3, 320), (1, 32, 2, 1024), (8, 20, 5, 192),
                                     (264, 33, 2, 64), (17, 650, 2, 64), (1, 300, 2, 2048)])
def test_rounds(G, L, N, S):
    x, cb = synth.make_rvq_case(G, L, N, S, seed=5, device="cuda")
    codes, res = binding.rl_rvq_encode(x, cb)
    torch.cuda.synchronize()
    _compare(x, cb, codes, res)

"""Cutting a contraction along K: the rule on the host, and the contractions that use it at the edges of their tiles."""
import ctypes as C
import os

import pytest
import torch

from paper_2603_16435_amd import binding, synth
from parity_util import compare_all, run_gpu, run_oracle

F32_TOL = dict(loss_tol=1e-5, logp_atol=2e-5, grad_tol=1e-4)          # the tolerances of the parity tests


@pytest.mark.skipif(not os.path.exists(binding.LIB_PATH), reason="library not built")
@pytest.mark.parametrize("slots", [256, 512])
def test_slices_cover_k_once_and_stay_within_the_partial_buffer(slots):
    lib = binding.lib()
    s, per = C.c_int32(0), C.c_int32(0)
    for tiles in (1, 2, 3, 14, 16, 42, 108, 255, 256, 257, 511, 512, 700, 1024, 1025, 100000):
        for slabs in (0, 1, 3, 4, 5, 7, 8, 32, 63, 64, 65, 257, 1576, 2376):
            assert lib.rl_debug_split_k(tiles, slabs, slots, C.byref(s), C.byref(per)) == 0
            s_, p_ = s.value, per.value
            assert 1 <= s_ <= 64 and p_ >= 1
            assert s_ * p_ >= slabs and (s_ - 1) * p_ < max(slabs, 1)         # no slab left out, no slice empty
            if s_ > 1:
                assert p_ >= 4 and tiles * s_ <= 2 * slots
    lib.rl_debug_split_k(42, 2376, 256, C.byref(s), C.byref(per))
    assert s.value >= 6                                                        # few tiles of a long K are cut


@pytest.mark.gpu
@pytest.mark.parametrize("H,V,lengths", [
    (36, 300, [1, 0, 2, 1]),               # one narrow tile, K tail of the logits, K of dX too short for many slices
    (132, 2600, [17, 16, 15, 40]),         # narrow tiles with remainders in every extent, dX in slices
    (64, 33001, [130, 1, 100, 99]),        # wide tiles, ragged vocabulary, dX in many slices
])
def test_f32_contractions_at_the_edges_of_their_tiles(H, V, lengths):
    cfg = synth.RolloutConfig("edge", 2, 2, 1, 64, H, V, "f32", 0.5, seed=31)
    b = synth.make_rollouts(cfg, "cuda", "packed", lengths=lengths)
    for objective in ("grpo", "flow"):
        ref = run_oracle(b, objective)
        for chunk in (0, 256):
            print(objective, chunk, compare_all(b, run_gpu(b, objective, chunk_rows=chunk), ref, **F32_TOL), flush=True)

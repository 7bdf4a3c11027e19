"""Cutting a contraction along K: the rule on the host, and the contractions that use it at the edges of their tiles."""
import ctypes as C
import itertools
import os

import pytest
import torch

from paper_2603_16435_amd import binding, synth
from parity_util import compare_all, run_gpu, run_oracle

F32_TOL = dict(loss_tol=1e-5, logp_atol=2e-5, grad_tol=1e-4)          # the tolerances of the parity tests
BF16_TOL = dict(loss_tol=1e-2, logp_atol=2e-3, grad_tol=2e-2)


@pytest.mark.skipif(not os.path.exists(binding.LIB_PATH), reason="library not built")
@pytest.mark.parametrize("slots", [256, 512])
def test_slices_cover_k_once_and_stay_within_the_partial_buffer(slots):
    lib = binding.lib()
    s, per, rows = C.c_int32(0), C.c_int32(0), C.c_int32(0)

    def cut(tm, tn, steps, fill):
        assert lib.rl_debug_split_k(tm, tn, steps, slots, fill, C.byref(s), C.byref(per), C.byref(rows)) == 0
        return s.value, per.value, rows.value

    for tn, steps, fill in itertools.product((1, 2, 3, 14, 56, 300, 600), (0, 1, 3, 4, 5, 7, 8, 32, 63, 64, 65, 157, 158, 257, 1188, 1576),
                                             (0, 1000, 1 << 33)):
        used = 0
        for tm in (*range(1, 40), 127, 128, 160, 256, 257, 511, 512, 5000):
            n, p, bound = cut(tm, tn, steps, fill)
            assert 1 <= n <= 64 and p >= 1
            assert n * p >= steps and (n - 1) * p < max(steps, 1)             # no step left out, no slice empty
            if n > 1:
                assert p >= 4 and tm * tn * n <= 2 * slots
                used = max(used, tm * n)
            assert used <= bound                                              # whatever fewer tokens there are than the launch allows for
    assert cut(3, 14, 1188, 0)[0] >= 6                                        # few tiles of a long K are cut ...
    assert cut(3, 14, 1188, 1 << 30)[0] == 1                                  # ... unless enough other work runs beside them


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


@pytest.mark.gpu
@pytest.mark.parametrize("H,V,lengths,modes", [
    (128, 513, [1, 0, 2, 1], ("recompute", "stash")),         # three vocabulary tiles: a K of six steps
    (384, 20001, [200, 56, 1, 60], ("recompute", "stash")),   # two M-tiles, ragged vocabulary, many slices, H not a multiple of the tile
    (136, 20001, [257, 0, 0, 0], ("recompute",)),             # hidden size off the hot kernel's grid for the logits
])
def test_bf16_dx_in_slices(H, V, lengths, modes):
    cfg = synth.RolloutConfig("edge", 2, 2, 1, 64, H, V, "bf16", 0.5, seed=32)
    b = synth.make_rollouts(cfg, "cuda", "padded", lengths=lengths)
    for objective in ("grpo", "flow"):
        ref = run_oracle(b, objective)
        for mode in modes:
            for chunk in (0, 512):
                print(objective, mode, chunk, compare_all(b, run_gpu(b, objective, chunk_rows=chunk, mode=mode), ref, **BF16_TOL), flush=True)


@pytest.mark.gpu
@pytest.mark.parametrize("H,V,lengths", [
    (8, 257, [3, 0, 1, 2]),             # general kernel: one 16-byte chunk of K, one row past a vocabulary tile
    (120, 512, [40, 1, 0, 30]),         # ... its second slab ends one chunk early
    (136, 300, [100, 100, 57, 3]),      # ... the last chunk alone in a third
    (192, 700, [10, 0, 90, 31]),        # ... the last size with dS there
    (200, 700, [10, 0, 90, 31]),        # dS in the hot kernel, two slab pairs
    (264, 1000, [5, 300, 0, 9]),        # ... three pairs: all of them in the tail loop, the last chunk alone
    (320, 1000, [5, 300, 0, 9]),        # the last size with the forward in the general kernel
    (328, 500, [33, 1, 64, 0]),         # both in the hot kernel, all of K in the tail loop
    (448, 500, [33, 1, 64, 0]),         # forward in the general kernel once more
    (456, 500, [33, 1, 64, 0]),
    (520, 769, [64, 64, 64, 64]),       # five pairs: plain loop and tail loop
    (1160, 2000, [31, 2, 200, 1]),
])
def test_bf16_hidden_sizes_off_the_slab_grid(H, V, lengths):
    cfg = synth.RolloutConfig("edge", 2, 2, 1, 64, H, V, "bf16", 0.5, seed=33)
    b = synth.make_rollouts(cfg, "cuda", "packed", lengths=lengths)
    for objective in ("grpo", "flow"):
        ref = run_oracle(b, objective)
        print(objective, compare_all(b, run_gpu(b, objective), ref, **BF16_TOL), flush=True)


@pytest.mark.gpu
@pytest.mark.parametrize("V", [512, 513, 575, 576, 577, 767, 1024 + 129])      # rows of W past the last slab: none, one, all but one, a whole slab, ...
def test_dx_reads_w_to_its_last_row_and_no_further(V):
    cfg = synth.RolloutConfig("edge", 2, 2, 1, 64, 384, V, "bf16", 0.5, seed=34)
    b = synth.make_rollouts(cfg, "cuda", "packed", lengths=[20, 3, 0, 40])
    # W in front of a block of NaN: whatever is read past its last row shows
    buf = torch.full((V + 300, 384), float("nan"), dtype=torch.bfloat16, device="cuda")
    buf[:V] = b.weight
    b.weight = buf[:V]
    ref = run_oracle(b, "grpo")
    for mode in ("recompute", "stash"):
        print(mode, compare_all(b, run_gpu(b, "grpo", mode=mode), ref, **BF16_TOL), flush=True)


@pytest.mark.skipif(not os.path.exists(binding.LIB_PATH), reason="library not built")
def test_workspace_sized_for_aligned_or_no_pointers_serves_any_alignment():
    """A call whose weight or hidden states lie off the 16-byte grid takes other kernels; a workspace sized without pointers, or for
    aligned ones, is large enough for those too."""
    lib = binding.lib()

    def size(hidden, weight, R, H, V, dtype, bwd, prm):
        b = binding.rl_batch()
        b.R, b.H, b.V, b.B, b.P, b.dtype, b.weight, b.hidden = R, H, V, 4, 2, dtype, weight, hidden
        n = C.c_size_t(0)
        assert lib.rl_workspace_bytes(C.byref(b), C.byref(prm), bwd, C.byref(n)) == 0
        return n.value

    shapes = itertools.product((1, 300, 1000, 32768, 32769, 50000, 140000), (8, 128, 136, 3584), (300, 5000, 152064),
                               (binding.RL_BF16, binding.RL_F32), (0, 1), (0, 512, 70000), (0, 1, 5000))
    for R, H, V, dtype, bwd, chunk, promise in shapes:
        prm = binding.make_params(chunk_rows=chunk, max_seq_len=promise)
        n = {p: size(*p, R, H, V, dtype, bwd, prm) for p in itertools.product((None, 0x1000, 0x1002), repeat=2)}
        enough = n[0x1000, 0x1000]
        assert n[None, None] >= enough and max(n.values()) == n[None, None] and enough == max(n.values()), (R, H, V, dtype, bwd, chunk, promise)


@pytest.mark.gpu
@pytest.mark.parametrize("off", [(1, 0), (0, 1), (1, 1)])      # hidden / weight off the 16-byte grid: the general kernel, W^T in memory
def test_bf16_operands_off_the_16_byte_grid(off):
    cfg = synth.RolloutConfig("edge", 2, 2, 1, 64, 136, 600, "bf16", 0.5, seed=35)
    b = synth.make_rollouts(cfg, "cuda", "packed", lengths=[20, 3, 0, 40])
    for name, o in zip(("hidden", "weight"), off):
        t = getattr(b, name)
        buf = torch.empty(t.numel() + o, dtype=t.dtype, device="cuda")
        buf[o:].copy_(t.flatten())
        setattr(b, name, buf[o:].view(t.shape))
    ref = run_oracle(b, "flow")
    print(compare_all(b, run_gpu(b, "flow"), ref, **BF16_TOL), flush=True)

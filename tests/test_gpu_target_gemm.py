"""The target's projections where the row tiles of a launch can go wrong, against the oracle: float32 trees around every count
of 16-row tiles, and more than 64 rows at the widths where a workgroup takes eight, ten or sixteen row blocks of the weights,
with ragged tiles, ragged stages and several row groups."""
import numpy as np
import pytest
import torch

import synth_inputs as si
from paper_2406_13170_amd import device as D

from gpu_common import say
from test_gpu_step import check_target, run_target

pytestmark = pytest.mark.gpu

# 2063 and 2052 row blocks (the head and gate/up): ten a workgroup, the last one ragged (W_down then has 513 steps, an odd number, in
# eight splits)
TEN = si.with_(si.MINI, name="mini_ten_blocks", vocab=33003, d_ffn=16416)
# 2000 row blocks: eight a workgroup, or sixteen over two row groups
EIGHT = si.with_(si.MINI, name="mini_eight_blocks", vocab=32000, d_ffn=16000)
# 960 row blocks of Q, K and V: eight a workgroup over two row groups; W_o splits its axis in two, ten blocks a workgroup
QKV = si.with_(si.MINI, name="mini_wide_qkv", d_model=5120, n_heads=40, d_ffn=512, vocab=512)
TEN_F32 = si.with_(si.TINY, name="tiny_ten_blocks", vocab=33003, d_ffn=16416)


@pytest.mark.parametrize("cfg,T,caps,L,Bsz", [
    (TEN, 13, (10,) * 4, 40, 5),        # 65 rows: three tiles, one row in the last (gate/up and the head)
    (TEN, 96, (10,) * 5, 30, 3),        # 288 rows: one group of nine tiles, the first wave has three
    (EIGHT, 64, (10,) * 4, 20, 2),      # 128 rows: a tile a wave (gate/up and the head)
    (EIGHT, 64, (10,) * 4, 20, 6),      # 384 rows: one group of twelve tiles, three a wave
    (EIGHT, 43, (10,) * 4, 33, 9),      # 387 rows: thirteen tiles, two groups of seven, two a wave and one
    (QKV, 64, (10,) * 4, 20, 8),        # 512 rows: two groups of eight tiles, two a wave
    (TEN_F32, 32, (10,) * 4, 17, 6),    # float32, 192 rows
])
def test_target_forward_over_wide_matrices(cfg, T, caps, L, Bsz):
    say(f"target_forward {cfg.name} T={T} L={L} batch={Bsz} (M = {T * Bsz})")
    cfgx, refs, got, _ = run_target(cfg, 1, T, caps, L, Bsz=Bsz, tiled=True)
    check_target(cfgx, refs, got)


# 65 to 128 rows, where each matrix goes to the kernel that suits it (gemm_is_wide).  Of the projections into Q, K and V, W_o,
# gate/up, W_down and the LM head, those of tiled weights on the wide kernel:
DOWN = si.with_(si.MINI, name="mini_down", d_model=1664, n_heads=13, d_ffn=4608, vocab=512)


@pytest.mark.parametrize("cfg,n_layers,T,caps,L,Bsz", [
    (si.MINI, 2, 64, (10,) * 4, 40, 2),    # none
    (EIGHT, 1, 32, (10,) * 4, 33, 4),      # gate/up, which then writes rows for a skinny W_down, and the head
    (TEN, 2, 13, (10,) * 4, 40, 5),        # the same over 65 rows, two layers
    (QKV, 1, 13, (10,) * 4, 20, 5),        # Q, K, V and W_o
    (QKV, 1, 64, (10,) * 4, 20, 2),        # Q, K, V
    (DOWN, 1, 13, (10,) * 4, 20, 5),       # none: W_down would be, but its input comes from a skinny gate/up
    (si.V7B, 1, 40, (10,) * 4, 64, 2),     # all but W_o
    (TEN_F32, 1, 16, (10,) * 4, 17, 5),    # float32: none
    (si.TINY, 2, 16, (4, 2, 2, 2), 9, 8),  # the same, 128 rows
])
def test_target_forward_over_two_blocks_of_rows(cfg, n_layers, T, caps, L, Bsz):
    """Against the oracle, and tiled against row-major weights: the same bits, whichever kernel took which matrix."""
    say(f"target_forward {cfg.name} T={T} batch={Bsz} (M = {T * Bsz})")
    runs = {}
    for tiled in (True, False):
        cfgx, refs, got, _ = run_target(cfg, n_layers, T, caps, L, Bsz=Bsz, tiled=tiled, oracle=tiled)
        if tiled:
            check_target(cfgx, refs, got)
        runs[tiled] = got
    for key in ("hidden", "logits", "tgt"):
        assert np.array_equal(runs[True][key], runs[False][key]), key
    bits = lambda t: t.view(torch.int16 if t.element_size() == 2 else torch.int32)
    for key in ("k_caches", "v_caches"):
        rows = [D.unpack_kv(r["ctx"], r["k_caches"], r["v_caches"])[key == "v_caches"][:, :, :, L:L + T] for r in runs.values()]
        assert torch.equal(bits(rows[0]), bits(rows[1])), key


@pytest.mark.parametrize("cfg,keys", [(EIGHT, ("gate_up",)), (EIGHT, ("down", "wo")), (QKV, ("qkv", "down")), (DOWN, ("down",))])
def test_partly_tiled_weights_over_two_blocks_of_rows(cfg, keys):
    """Whichever matrices are tiled, the results are those of row-major weights."""
    say(f"target_forward {cfg.name}, 65 rows, tiled copies of {keys}")
    runs = [run_target(cfg, 2, 13, (10,) * 4, 20, Bsz=5, tiled=tiled, tiled_keys=keys if tiled else None, oracle=False)[2]
            for tiled in (True, False)]
    for key in ("hidden", "logits", "tgt"):
        assert np.array_equal(runs[0][key], runs[1][key]), key


@pytest.mark.parametrize("T", [2, 16, 17, 32, 33, 48, 49, 64])
@pytest.mark.parametrize("tiled", [True, False])
def test_float32_target_forward_over_few_rows(T, tiled):
    say(f"target_forward tiny T={T} tiled={tiled}")
    cfgx, refs, got, _ = run_target(si.TINY, 1, T, (10,) * 4, 21, tiled=tiled)
    check_target(cfgx, refs, got)

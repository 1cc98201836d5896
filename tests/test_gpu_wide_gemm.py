"""The wide GEMM where its groups of row tiles, its waves' shares of them, its weight stages and its row argmax can go wrong,
against the oracle: one to thirteen tiles of 32 rows in a group of up to three a wave, ragged stages (43 steps of the reduction
axis), a ragged last tile of weights, with and without the logits."""
import numpy as np
import pytest

import synth_inputs as si

from gpu_common import say
from test_gpu_step import check_target, run_target

pytestmark = pytest.mark.gpu

# 172 and 688 steps' worth of blocks: W_down has 43 steps of 64 bytes, the head 2063 row blocks (the last one ragged)
RAGGED = si.with_(si.MINI, name="mini_ragged", vocab=33003, d_ffn=1376)


@pytest.mark.parametrize("T,Bsz", [(43, 3),     # 129 rows: five tiles, one row in the last
                                   (32, 5),     # 160: five tiles, two of them with the first wave
                                   (24, 8),     # 192: six
                                   (64, 4),     # 256: eight, two a wave
                                   (43, 6),     # 258: nine, three of them with the first wave
                                   (88, 4),     # 352: eleven
                                   (96, 4),     # 384: twelve, three a wave
                                   (59, 7)])    # 413: thirteen, two groups
def test_wide_gemm_row_groups(T, Bsz):
    say(f"target_forward {RAGGED.name} T={T} batch={Bsz} (M = {T * Bsz})")
    cfgx, refs, got, _ = run_target(RAGGED, 1, T, (10,) * 5, 37, Bsz=Bsz, tiled=True)
    check_target(cfgx, refs, got)
    # the argmax that the kernel takes from its registers is that of the logits it writes, ties to the lower token
    assert np.array_equal(np.asarray(got["tgt"]).reshape(-1), np.asarray(got["logits"]).reshape(T * Bsz, -1).argmax(1))

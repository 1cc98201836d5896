"""The sampling draw's run sums at vocabularies around the thread count and its multiples, and the commit at the deepest
paths, the other head widths and fewer heads than gathered rows."""
import numpy as np
import pytest

import synth_inputs as si

import test_gpu_loop
from gpu_common import say
from test_gpu_typical import run_case

pytestmark = pytest.mark.gpu

LAST = np.float32(1.0) - np.float32(2.0 ** -24)               # u * Z may reach the rounded total: the last live token


# one token a run and fewer, two with an empty tail of runs, eight exactly and nine, 31 and 32 with a ragged last run
@pytest.mark.parametrize("V", [5, 63, 1023, 1024, 1025, 8191, 8192, 8193, 31745, 32000])
def test_draw_at_run_edges(V):
    say(f"draw at run edges V={V}")
    T, caps = (1, (4, 4, 4, 4)) if V < 16 else (16, (4, 2, 2, 2))
    run_case(V, T, caps, 4, 9, 0.7, 0.09, 0.3, spread=1.5, us=np.array([0.0, 0.31, 0.77, LAST], dtype=np.float32))


def test_draw_falls_back_to_the_last_token_of_non_zero_probability():
    """Half of the vocabulary has probability zero; u = 1 lies at or above every cumulative sum."""
    V = 3000
    logits = np.random.default_rng(4).standard_normal((2, 1, V)).astype(np.float32)
    logits[0, 0, 1501:] = -np.inf
    logits[1, 0, ::2] = -1.0e30
    run_case(V, 1, (4, 4, 4, 4), 2, 5, 1.0, 0.09, 0.3, logits=logits, toks=np.zeros((2, 1), dtype=np.int32),
             us=np.array([LAST, LAST], dtype=np.float32))


@pytest.mark.parametrize("cfg,T,caps,L,B_", [
    (si.with_(si.MINI, name="mini_deep"), 40, (2,) * 8, 50, 2),                                    # K = 8 rows in bf16
    (si.with_(si.TINY, name="tiny_deep_dh128", d_model=512, head_dim=128), 33, (2,) * 8, 27, 2),   # ... 128 wide in float32
    (si.with_(si.MINI, name="mini_dh64", d_model=256, head_dim=64), 64, (10,) * 4, 63, 1),
    (si.with_(si.TINY, name="tiny_one_head", d_model=64, n_heads=1), 16, (4, 2, 2, 2), 5, 1),      # one head gathers K + 1 rows
])
def test_commit_of_deep_paths_and_other_head_widths(cfg, T, caps, L, B_):
    test_gpu_loop.test_commit_moves_the_accepted_rows_and_gathers_the_next_draft_inputs(cfg, T, caps, L, B_)

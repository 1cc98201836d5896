"""Whole drafts against the oracle where the adaptation layers' attention cuts its keys into splits or shares cache rows
between positions: float32 and bf16, both head widths, lengths from one row to a full cache, unequal over the batch, with dead
positions inside a group."""
import numpy as np
import pytest
import torch

import synth_inputs as si
from oracle import amphista_oracle as orc
from paper_2406_13170_amd import binding as B
from paper_2406_13170_amd import device as D

from gpu_common import DEV, TOL, assert_rows_close, cfg_tensor_to_dev, draft_f32, f32_to_dev, i32_to_dev, make_ctx, np_of, say, topk_consistent

pytestmark = pytest.mark.gpu


def check_draft(cfg, n_new, max_kv, lens, live, check=None, seed=17):
    """amph_draft over n_new positions of len(lens) sequences of which live[b] count; `check`: elements held against the oracle."""
    batch, n_h, d_h, d, V, K = len(lens), cfg.n_heads, cfg.head_dim, cfg.d_model, cfg.vocab, cfg.K
    cfg = si.with_(cfg, batch=batch)
    say(f"draft {cfg.name} batch {batch} n_new {n_new} max_kv {max_kv} lengths {lens} live {live}")
    ctx = make_ctx(cfg, max_kv=max_kv)
    dw = si.draft_weights(cfg, seed)
    dwd, dwo = D.draft_to_device(dw, DEV), draft_f32(dw)
    h = si.as_f32_exact(cfg, seed, "da.h", (batch, n_new, d), 1.0)
    tok = si.tokens(cfg, seed, "da.tok", (batch, n_new))
    top = max(lens)
    rows = [[si.normal(cfg, seed, f"da.sal{s}.{kv}", (batch, n_h, max(top, 1), d_h), 1.0) for kv in "kv"] for s in range(2)]
    sal = torch.full((2, batch, 2, n_h, max_kv, d_h), float("nan"), dtype=D.torch_dtype(cfg.dtype), device=DEV)
    for s in range(2):
        for kv in range(2):
            t = cfg_tensor_to_dev(rows[s][kv])
            for b, n in enumerate(lens):
                sal[s, b, kv, :, :n] = t[b, :, :n]
    sal_len = i32_to_dev(lens)
    idx = torch.full((batch, K, cfg.topk), -7, dtype=torch.int32, device=DEV)
    val = torch.full((batch, K, cfg.topk), float("nan"), device=DEV)
    logits = torch.full((batch, K, V), float("nan"), device=DEV)
    ctx.amph_draft(B.Context.draft_struct(dwd), f32_to_dev(h), i32_to_dev(tok), sal, sal_len, idx, val, logits, n_new=n_new,
                   n_valid=i32_to_dev(live))
    assert ctx.device_status() == 0
    assert list(np_of(sal_len)) == [n + r for n, r in zip(lens, live)]
    lg, tol = np_of(logits), TOL[cfg.dtype]
    for b in (range(batch) if check is None else check):
        k0 = [rows[s][0].f32[b][:, :lens[b]] for s in range(2)]
        v0 = [rows[s][1].f32[b][:, :lens[b]] for s in range(2)]
        ref, k1, v1 = orc.draft_catchup(dwo, h[b, :live[b]], tok[b, :live[b]], k0, v0, n_h, cfg.topk, cfg.rms_eps, cfg.rope_theta)
        # float32 sums; in bf16 also the live new rows of the cache, rounded to 2^-9 of their values (the oracle keeps them whole),
        # whose part in an attention over n rows of like weight goes with the root of their share
        tight = 1e-5 if cfg.dtype == "f32" else 1e-5 + 3 * 2.0 ** -9 * (live[b] / (lens[b] + live[b])) ** 0.5
        worst = assert_rows_close(lg[b], ref["logits"], tight, f"logits of element {b}")
        say(f"  element {b}: worst row error of the logits {worst:.2e}")
        for r in range(K):
            ok, bad = topk_consistent(np_of(idx)[b, r], np.asarray(ref["logits"][r]), cfg.topk, tol * np.abs(ref["logits"][r]).max())
            assert ok, bad
        new = slice(lens[b], lens[b] + live[b])
        for s in range(2):
            assert_rows_close(np_of(sal[s, b, 0, :, new]).reshape(-1, d_h), k1[s][:, new].reshape(-1, d_h), tol, "keys")
            assert_rows_close(np_of(sal[s, b, 1, :, new]).reshape(-1, d_h), v1[s][:, new].reshape(-1, d_h), tol, "values")
        assert torch.isnan(sal[:, b, :, :, lens[b] + live[b]:].float()).all()


# Few heads: eight key splits, whose partial results W_o folds while it stages its rows: one row, two, and as many as share a
# launch; lengths that leave splits empty (0 to 6 rows), with one row, full ones.
TINY_128 = si.with_(si.TINY, name="tiny_dh128", d_model=256, n_heads=2, head_dim=128)
TINY_TWO = si.with_(si.TINY, name="tiny_two_heads", d_model=128, n_heads=2)
MINI_64 = si.with_(si.MINI, name="mini_dh64", d_model=256, n_heads=4, head_dim=64)


@pytest.mark.parametrize("cfg,n_new,lens,live", [
    (si.TINY, 1, [0], [1]), (si.TINY, 1, [6], [1]), (si.TINY, 1, [1023], [1]),
    (si.TINY, 5, [2], [5]), (si.TINY, 5, [700], [3]), (si.TINY, 3, [129], [3]),
    (si.TINY, 1, [7, 500], [1, 1]), (si.TINY, 1, [900, 3, 64, 0, 511], [1] * 5),
    (TINY_TWO, 1, [5, 1023, 128, 0, 77, 640, 1, 9], [1] * 8), (TINY_TWO, 3, [800, 2], [2, 3]),
    (TINY_128, 4, [333], [4]), (si.MINI, 1, [0], [1]), (si.MINI, 1, [1023], [1]), (si.MINI, 1, [600, 12], [1, 1]),
    (si.MINI, 5, [400, 30], [2, 5]), (MINI_64, 1, [250, 1000], [1, 1]), (MINI_64, 5, [1000], [4]),
])
def test_draft_with_key_splits(cfg, n_new, lens, live):
    check_draft(cfg, n_new, 1024, lens, live)


# Many (head, sequence, position) triples: three or six positions share a workgroup's cache rows.
def wide(name, n_h, d_h, base=si.MINI, K=4):
    return si.with_(base, name=name, d_model=n_h * d_h, n_heads=n_h, head_dim=d_h, d_ffn=512, vocab=512, K=K)


H16_64, H16_128 = wide("mini_16x64", 16, 64), wide("mini_16x128", 16, 128)
F16_64, F16_128 = wide("tiny_16x64", 16, 64, si.TINY), wide("tiny_16x128", 16, 128, si.TINY)
H16_K8 = wide("mini_16x64_k8", 16, 64, K=8)


@pytest.mark.parametrize("cfg,n_new,max_kv,lens,live,check", [
    # three positions together, one key split
    (H16_64, 3, 96, [93, 0, 5, 31, 64, 17], [3, 3, 1, 2, 3, 2], None),
    (H16_128, 3, 96, [40, 93, 1, 7, 15, 33], [2, 3, 3, 1, 3, 3], None),
    (F16_64, 3, 96, [93, 0, 5, 31, 64, 17], [3, 3, 1, 2, 3, 2], None),
    (F16_128, 3, 96, [40, 93, 1, 7, 15, 33], [2, 3, 3, 1, 3, 3], None),
    # six (four, five of them taken), over four, two and one key splits
    (H16_64, 5, 1024, [1019, 0, 700, 129], [5, 4, 1, 3], None),
    (H16_128, 5, 512, [507, 2, 130, 61], [5, 5, 2, 4], None),
    (F16_64, 4, 512, [508, 0, 63, 64, 200], [4, 4, 3, 2, 1], None),
    (F16_128, 5, 256, [251, 33, 0, 128], [5, 3, 5, 1], None),
    (H16_128, 5, 96, [91, 16, 17, 0], [5, 1, 4, 5], None),
    # two groups of rows: six and one, six and three
    (H16_K8, 9, 512, [503, 70], [9, 7], None),
    (H16_K8, 9, 512, [100, 500], [6, 3], None),
    (H16_K8, 7, 128, [121, 0, 50], [7, 6, 2], None),
    # a batch of eight with 32 heads; one sequence of 52 heads on a long cache
    (wide("mini_32x64", 32, 64), 5, 256, [251, 3, 100, 0, 64, 199, 17, 130], [5, 5, 1, 2, 3, 4, 5, 5], [0, 2, 3, 7]),
    (wide("mini_52x64", 52, 64, K=5), 6, 1024, [700], [6], None),
    (wide("mini_52x64", 52, 64, K=5), 6, 1024, [1018], [4], None),
])
def test_draft_with_positions_that_share_cache_rows(cfg, n_new, max_kv, lens, live, check):
    check_draft(cfg, n_new, max_kv, lens, live, check)

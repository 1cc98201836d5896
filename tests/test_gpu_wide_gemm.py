"""The wide GEMM where its groups of row tiles, its waves' shares of them, its weight stages and its row argmax can go wrong,
against the oracle: one to thirteen tiles of 32 rows in a group of up to three a wave, ragged stages (43 steps of the reduction
axis), a ragged last tile of weights, with and without the logits."""
import numpy as np
import pytest
import torch

import synth_inputs as si
from paper_2406_13170_amd import binding as B
from paper_2406_13170_amd import device as D

from gpu_common import DEV, i32_to_dev, make_ctx, say
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


@pytest.mark.parametrize("cfg,T,Bsz", [(si.MINI, 64, 3), (RAGGED, 43, 3), (si.TINY, 64, 3)])
def test_wide_gemm_writes_logits_that_begin_anywhere(cfg, T, Bsz):
    """logits_out on a 4-byte boundary only: the same logits, and not a float before or behind them."""
    say(f"target_forward {cfg.name} T={T} batch={Bsz} (M = {T * Bsz}), logits off a 16-byte boundary")
    L = 37
    cfgx, _, got, (ctx, tree, otree) = run_target(cfg, 1, T, (10,) * 5, L, Bsz=Bsz, tiled=True, oracle=False)
    dev, n = got["dev"], Bsz * T * cfgx.vocab
    tok = i32_to_dev(si.tokens(cfgx, 0, "tree.tok", (Bsz, T)))
    pos = i32_to_dev(np.stack([L + otree.depth for _ in range(Bsz)]))
    for off in (1, 2, 3):
        buf = torch.full((n + 8,), -7.0, device=DEV)
        tgt = torch.full((Bsz, T), -1, dtype=torch.int32, device=DEV)
        ctx.amph_target_forward(tree, dev["structs"], dev["embed_d"], dev["fn_d"], None, tok, pos, got["k_caches"], got["v_caches"],
                                i32_to_dev(np.full(Bsz, L)), None, buf[off:off + n], tgt, tiled_structs=dev["tiled_structs"],
                                lm_head_tiled=dev["lm_t"])
        out = buf.cpu().numpy()
        assert np.array_equal(out[off:off + n], got["logits"].reshape(-1)) and np.array_equal(tgt.cpu().numpy(), got["tgt"])
        assert np.all(out[:off] == -7.0) and np.all(out[off + n:] == -7.0)


@pytest.mark.parametrize("cfg,V", [(si.MINI, 2048), (si.MINI, 16003), (si.MINI, 32000), (si.MINI, 33003), (si.TINY, 1024), (si.TINY, 1003)])
@pytest.mark.parametrize("T,Bsz", [(43, 3), (64, 4), (96, 4)])
def test_wide_gemm_argmax_of_ties(cfg, V, T, Bsz):
    """A head of five different rows over and over, and one of zeros: equal logits in a lane, in its partner, in other tiles and
    in a ragged last one.  The lowest token wins."""
    say(f"argmax of ties {cfg.name} V={V} T={T} batch={Bsz} (M = {T * Bsz})")
    cfgx = si.with_(cfg, vocab=V, batch=Bsz, K=5, topk=10)
    ctx = make_ctx(cfgx, T=T, batch=Bsz, max_kv=128)
    tree = B.Tree(si.tree_paths(T, (10,) * 5), 5)
    tdt = D.torch_dtype(cfg.dtype)
    g = torch.Generator().manual_seed(3)
    embed = torch.randn((V, cfg.d_model), generator=g).to(tdt).to(DEV)
    norm = torch.ones((cfg.d_model,), dtype=tdt, device=DEV)
    few = torch.randn((5, cfg.d_model), generator=g).to(tdt).to(DEV)
    tok = torch.randint(0, V, (Bsz, T), generator=g, dtype=torch.int32).to(DEV)
    for head in (few[torch.arange(V, device=DEV) % 5].contiguous(), torch.zeros((V, cfg.d_model), dtype=tdt, device=DEV)):
        lm_t = D.pack_lm_head(ctx, head)
        tgt = {}
        for with_logits in (True, False):
            logits = torch.full((Bsz, T, V), float("nan"), device=DEV) if with_logits else None
            tgt[with_logits] = torch.full((Bsz, T), -1, dtype=torch.int32, device=DEV)
            ctx.amph_target_forward(tree, [], embed, norm, None, tok, torch.zeros_like(tok), None, None, i32_to_dev(np.zeros(Bsz)), None,
                                    logits, tgt[with_logits], tiled_structs=None, lm_head_tiled=lm_t)
            if with_logits:
                want = logits.cpu().numpy().argmax(-1)             # (the first of equal ones)
        assert want.max() < 5
        for t in tgt.values():
            assert np.array_equal(t.cpu().numpy(), want)

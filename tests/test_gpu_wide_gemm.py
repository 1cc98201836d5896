"""The wide GEMM against the oracle: the head's groups of five to thirteen row tiles (up to three a wave) beside a layer whose W_down
has ragged stages (43 steps of the reduction axis in two slabs); the row argmax; logits that begin anywhere; and every instance that the
plan selects, on narrow matrices that it gives them."""
import numpy as np
import pytest
import torch

import synth_inputs as si
from oracle import amphista_oracle as orc
from paper_2406_13170_amd import binding as B
from paper_2406_13170_amd import device as D

import wide_plan as wp
from gpu_common import DEV, cfg_tensor_to_dev, f32_layers, i32_to_dev, make_ctx, np_of, say
from test_gpu_step import check_target, run_target

pytestmark = pytest.mark.gpu

# W_down has 43 steps of 64 bytes, the head 2063 row blocks (the last one ragged)
RAGGED = si.with_(si.MINI, name="mini_ragged", vocab=33003, d_ffn=1376)


# the head's groups; the layer's matrices form groups of three tiles (gate/up of four over 256 rows), a tile a wave
@pytest.mark.parametrize("T,Bsz", [(43, 3),     # 129 rows: five tiles, one row in the last, two tiles with the first wave
                                   (32, 5),     # 160: five tiles
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


# ---- every instance of the kernel, on narrow matrices that the plan gives it -----------------------------------------------
def run_twins(case, n_layers, d, d_ffn, vocab):
    """A pass over many sequences of which only two are different: those against the oracle, the others against their twins, bit by
    bit (a row of a GEMM does not depend on the rows beside it)."""
    dtype, T, Bsz, _, d_h, _, _ = case
    L, K, seed = 20, 5, 3
    cfg = si.with_(si.MINI if dtype == "bf16" else si.TINY, name=f"twins_{dtype}_{d}", d_model=d, n_heads=d // d_h, head_dim=d_h, d_ffn=d_ffn,
                   vocab=vocab, batch=Bsz, K=K, topk=10)
    n_h, max_kv = cfg.n_heads, (L + T + 31) // 32 * 32
    ctx = make_ctx(cfg, T=T, max_kv=max_kv)
    paths = si.tree_paths(T, (10,) * K)
    tree, otree = B.Tree(paths, K), orc.tree_from_paths(paths, K)
    tw = si.target_weights(cfg, seed, n_layers)
    layers_d = [D.layer_to_device(lw, DEV) for lw in tw["layers"]]
    packed = [D.pack_layer(ctx, l) for l in layers_d]
    structs = [B.amph_layer_w(rms1=l["rms1"].data_ptr(), rms2=l["rms2"].data_ptr()) for l in layers_d]
    lm_t = D.pack_lm_head(ctx, cfg_tensor_to_dev(tw["lm_head"]))
    kv = [[si.normal(cfg, seed, f"twins{li}.{n}", (2, n_h, L, d_h), 1.0) for li in range(n_layers)] for n in "kv"]
    caches = []
    for rows in kv:
        t = torch.zeros((max(n_layers, 1), Bsz, n_h, max_kv, d_h), dtype=D.torch_dtype(cfg.dtype), device=DEV)
        for li, r in enumerate(rows):
            t[li, :, :, :L] = cfg_tensor_to_dev(r)[torch.arange(Bsz) % 2]
        caches.append(t)
    k_caches, v_caches = D.pack_kv(ctx, *caches)
    del caches
    tok = si.tokens(cfg, seed, "twins.tok", (2, T))
    pos = (L + otree.depth).astype(np.int32)
    hidden = torch.full((Bsz, T, d), float("nan"), device=DEV)
    logits = torch.full((Bsz, T, vocab), float("nan"), device=DEV)
    tgt = torch.full((Bsz, T), -1, dtype=torch.int32, device=DEV)
    ctx.amph_target_forward(tree, structs, cfg_tensor_to_dev(tw["embed"]), cfg_tensor_to_dev(tw["final_norm"]), None,
                            i32_to_dev(tok[np.arange(Bsz) % 2]), i32_to_dev(np.tile(pos, (Bsz, 1))), k_caches, v_caches,
                            i32_to_dev(np.full(Bsz, L)), hidden, logits, tgt, tiled_structs=[p[0] for p in packed], lm_head_tiled=lm_t)
    torch.cuda.synchronize()
    assert ctx.device_status() == 0
    bits = lambda t: t.view(torch.int16 if t.element_size() == 2 else torch.int32)  # noqa: E731
    rows = [t[:, :, :, L:L + T].transpose(0, 1) for t in D.unpack_kv(ctx, k_caches, v_caches)] if n_layers else []
    for t in [hidden, logits, tgt] + rows:
        t = bits(t.contiguous())
        for b in range(2, Bsz):
            assert torch.equal(t[b], t[b % 2]), f"sequence {b} differs from its twin"
    two = dict(embed=tw["embed"].f32, layers=f32_layers(tw["layers"]), final_norm=tw["final_norm"].f32, lm_head=tw["lm_head"].f32)
    refs = [orc.target_forward(two, tok[b], pos, otree.mask, [r.f32[b] for r in kv[0]], [r.f32[b] for r in kv[1]], n_h, cfg.rms_eps,
                               cfg.rope_theta, keep=True) for b in range(2)]
    check_target(cfg, refs, dict(hidden=np_of(hidden[:2]), logits=np_of(logits[:2]), tgt=np_of(tgt[:2]), k_caches=k_caches, v_caches=v_caches,
                                 L=L, T=T, ctx=ctx))
    assert torch.equal(logits.argmax(-1).to(torch.int32), tgt)


ids = lambda c: "-".join(str(x) for x in c[:6])  # noqa: E731


@pytest.mark.parametrize("case", wp.LAYERS, ids=ids)
def test_wide_gemm_instances_of_a_layer(case):
    say(f"wide GEMM instances {sorted(case[-1])}: {case[:6]}, M = {case[1] * case[2]}")
    assert case[-1] <= {wp.instance(*g) for g in wp.gemms(case)}
    run_twins(case, 1, case[3], case[5], 512)


@pytest.mark.parametrize("case", wp.HEADS, ids=ids)
def test_wide_gemm_instances_of_the_head(case):
    say(f"wide GEMM instances {sorted(case[-1])}: {case[:6]}, M = {case[1] * case[2]}")
    assert case[-1] <= {wp.instance(*g) for g in wp.gemms(case)}
    run_twins(case, 0, case[3], 320, case[5])


@pytest.mark.parametrize("cfg,T,Bsz", [(si.V7B, 64, 8), (si.V13B, 64, 2)])
def test_wide_gemm_at_model_width(cfg, T, Bsz):
    say(f"one layer of {cfg.name} over {T * Bsz} rows")
    run_twins((cfg.dtype, T, Bsz, cfg.d_model, cfg.head_dim, cfg.d_ffn, set()), 1, cfg.d_model, cfg.d_ffn, cfg.vocab)


def test_wide_gemm_over_more_than_4_gib_of_activations():
    """W_down of 128 x 278,528 over 8,192 rows, 4.6 GB of them."""
    case = ("bf16", 128, 64, 128, 64, 278528, set())
    down = wp.instance("bf16", wp.STORE, 128, 278528, 8192)
    say(f"one layer of 128 x 278528 over 8192 rows: W_down on {down}")
    assert down
    run_twins(case, 1, 128, 278528, 512)

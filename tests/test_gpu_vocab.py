"""Vocabularies up to the largest one, 65536 tokens: sampling acceptance whose runs come through LDS in several pieces, the
argmax of given logits, and the draft's top-k over up to 1024 candidate lists, ties included.  Then the cache layouts of the
head widths that no model configuration here has."""
import numpy as np
import pytest
import torch

import synth_inputs as si
from oracle import amphista_oracle as orc
from paper_2406_13170_amd import binding as B

from gpu_common import DEV, f32_to_dev, i32_to_dev, make_ctx, np_of, say
from test_gpu_draft_mm import device_draft_weights, to_float
import test_gpu_kernels
from test_gpu_typical import run_case

pytestmark = pytest.mark.gpu


# 32 tokens a thread fill one piece; 33 leave one token for the second, 64 fill two
@pytest.mark.parametrize("V", [32767, 32768, 32769, 33003, 65535, 65536])
def test_accept_typical_over_large_vocabularies(V):
    say(f"accept_typical V={V}")
    last = np.float32(1.0) - np.float32(2.0 ** -24)
    run_case(V, 22, (10,) * 4, 3, 1, 0.7, 0.09, 0.3, spread=2.0, us=np.array([0.0, 0.37, last], dtype=np.float32))
    run_case(V, 5, (4, 2, 2, 2), 3, 2, 1.0, 0.05, 0.6, spread=1.0, us=np.array([0.02, 0.5, 0.98], dtype=np.float32))


@pytest.mark.parametrize("V", [33003, 65536])
def test_draw_lands_in_every_piece_of_a_run(V):
    """A tree of one node whose distribution is all on one token: it is drawn, wherever in a thread's run it lies."""
    say(f"draw V={V}")
    C = (V + 1023) // 1024
    tokens = [0, 1, 31, 32, C - 1, C, 7 * C + 31, 7 * C + 32, 500 * C + C - 1, V // 2, V - 2, V - 1]
    logits = np.full((len(tokens), 1, V), -50.0, dtype=np.float32)
    for b, t in enumerate(tokens):
        logits[b, 0, t] = 20.0
    run_case(V, 1, (4, 4, 4, 4), len(tokens), 3, 0.7, 0.09, 0.3, logits=logits, toks=np.zeros((len(tokens), 1), dtype=np.int32),
             us=np.linspace(0.01, 0.99, len(tokens)).astype(np.float32))


@pytest.mark.parametrize("V", [1, 5, 1024, 1025, 8192, 8193, 16384, 16385, 32768, 32769, 65535, 65536])
def test_accept_takes_the_argmax_of_given_logits(V):
    """The root alone: next_tok is the row's argmax, ties to the lowest id, whatever NaN or infinities stand beside it."""
    say(f"accept from logits V={V}")
    Bn = 7
    rng = np.random.default_rng(V)
    logits = rng.standard_normal((Bn, 1, V)).astype(np.float32)
    tie = sorted(int(t) for t in rng.integers(0, V, size=3))
    logits[0, 0, V - 1] = 9.0
    logits[1, 0, 0] = 9.0
    logits[2, 0, tie] = 9.0                                    # up to three equal maxima
    logits[3, 0, :] = 0.0                                      # all equal ...
    logits[3, 0, V // 2:] = -0.0                               # ... in both signs
    logits[4, 0, :] = -np.inf
    logits[4, 0, V // 3] = -3.0e38                             # the type's end next to infinities
    logits[5, 0, tie[1]] = np.inf
    logits[6, 0, :] = -np.inf                                  # nothing but infinities: the lowest id
    want = [orc.row_argmax(logits[b, 0]) for b in range(Bn)]
    if V > 8:
        logits[0, 0, 3] = np.nan                               # NaN is never the best
    cfg = si.with_(si.TINY, vocab=V, batch=Bn, topk=1)
    ctx = make_ctx(cfg, T=1, batch=Bn)
    out = [torch.full(s, -7, dtype=torch.int32, device=DEV) for s in ((Bn,), (Bn, 5), (Bn,), (Bn,))]
    ctx.amph_accept(B.Tree([], 4), i32_to_dev(np.zeros((Bn, 1))), None, f32_to_dev(logits), *out)
    assert list(np_of(out[2])) == [int(w) for w in want] and list(np_of(out[0])) == [0] * Bn


@pytest.mark.parametrize("V,topk", [(40, 16), (16383, 10), (32769, 10), (33003, 16), (65535, 1), (65536, 10)])
@pytest.mark.parametrize("dtype,batch", [("bf16", 1), ("bf16", 2), ("f32", 1), ("f32", 3)])
def test_draft_top_k_over_large_vocabularies(V, topk, dtype, batch):
    """The chosen tokens are the best of the logits that the same call returns: descending, ties to the lower token."""
    d, n_h, f, K = 256, 4, 256, 4
    say(f"draft top-{topk} V={V} {dtype} batch {batch}")
    w = device_draft_weights(d, n_h, f, V, K, V)
    half = V // 2
    w["lm_head"][half:2 * half] = w["lm_head"][:half]          # every logit twice, half a vocabulary apart
    w["lm_head"][1:min(V, 90)] = w["lm_head"][0]               # and a run of equal ones across the first lists
    if dtype == "f32":
        w = to_float(w)
    ctx = B.Context(d_model=d, n_heads=n_h, head_dim=64, d_ffn=f, vocab=V, K=K, topk=topk, max_tree=16, max_kv=32, batch=batch,
                    dtype=B.AMPH_F32 if dtype == "f32" else B.AMPH_BF16, rms_eps=1e-6, rope_theta=10000.0, device=DEV)
    g = torch.Generator(device=DEV).manual_seed(V + batch)
    h = torch.randn((batch, 1, d), generator=g, device=DEV)
    tok = torch.randint(0, V, (batch, 1), generator=g, device=DEV, dtype=torch.int32)
    kv = torch.zeros((2, batch, 2, n_h, 32, 64), dtype=w["embed"].dtype, device=DEV)
    idx = torch.full((batch, K, topk), -7, dtype=torch.int32, device=DEV)
    val, logits = torch.zeros((batch, K, topk), device=DEV), torch.full((batch, K, V), float("nan"), device=DEV)
    ctx.amph_draft(B.Context.draft_struct(w), h, tok, kv, i32_to_dev([0] * batch), idx, val, logits, n_new=1)
    assert ctx.device_status() == 0
    lg = np_of(logits).reshape(-1, V)
    for r in range(lg.shape[0]):
        order = np.lexsort((np.arange(V), -lg[r]))[:topk]
        assert list(np_of(idx).reshape(-1, topk)[r]) == list(order)
        assert np.array_equal(np_of(val).reshape(-1, topk)[r], lg[r][order])


@pytest.mark.parametrize("cfg,max_kv,lead", [
    (si.with_(si.MINI, name="mini_dh64", d_model=256, head_dim=64), 96, (2, 1, 4)),
    (si.with_(si.TINY, name="tiny_dh128", d_model=512, head_dim=128), 64, (1, 2, 4)),
    (si.with_(si.MINI, name="mini_one_step"), 128, (1, 1, 4)),
])
def test_cache_layouts_of_other_head_widths(cfg, max_kv, lead):
    test_gpu_kernels.test_pack_and_unpack_kv_follow_the_header_formulas(cfg, max_kv, lead)

"""The draft's projections on the matrix cores (float32 rows against bf16 weights): their error against 64 bits at the edges
of blocks, tiles and stages, non-finite activations, and whole drafts over row counts around the edges of a launch."""
import numpy as np
import pytest
import torch

import synth_inputs as si
from oracle import amphista_oracle as orc
from paper_2406_13170_amd import binding as B
from paper_2406_13170_amd import device as D

from gpu_common import DEV, TOL, assert_rows_close, draft_f32, f32_to_dev, i32_to_dev, make_ctx, np_of, say, topk_consistent

pytestmark = pytest.mark.gpu


# N: one block, a ragged one, ragged last workgroups of every height; K: one piece, ragged and whole stages, long axes
@pytest.mark.parametrize("M", [1, 3, 5, 8])
@pytest.mark.parametrize("N,K", [(16, 8), (5, 40), (40, 264), (515, 520), (4096, 1032), (4100, 1016), (6000, 4096), (12300, 1024),
                                 (1024, 17920), (22016, 512)])
def test_projection_error_against_64_bits(M, N, K):
    say(f"projection M={M} N={N} K={K}")
    g = torch.Generator(device=DEV).manual_seed(N * 31 + K)
    W = (torch.randn((N, K), generator=g, device=DEV) * 0.02).bfloat16()
    x = torch.randn((M, K), generator=g, device=DEV)
    y = torch.full((M, N), float("nan"), device=DEV)
    make_ctx(si.MINI).amph_gemv(x, W, y, M, N, K)
    ref = x.double() @ W.double().t()
    # float32 sums of K random terms in chains of at most 280: about sqrt(280) / 2 half-ulps of the running sum
    err = float((y.double() - ref).norm() / ref.norm())
    assert err < 5e-7, err


def test_projection_of_more_than_4_gib_of_rows():
    """Eight rows of 134,218,752 floats against sixteen of bf16."""
    M, N, K = 8, 16, (1 << 27) + 1024
    say(f"projection M={M} N={N} K={K}")
    g = torch.Generator(device=DEV).manual_seed(7)
    W = torch.empty((N, K), dtype=torch.bfloat16, device=DEV).normal_(0.0, 0.02, generator=g)
    x = torch.empty((M, K), device=DEV).normal_(0.0, 1.0, generator=g)
    y = torch.full((M, N), float("nan"), device=DEV)
    make_ctx(si.MINI).amph_gemv(x, W, y, M, N, K)
    ref = torch.zeros((M, N), dtype=torch.float64, device=DEV)
    for c in range(0, K, 1 << 22):
        ref += x[:, c:c + (1 << 22)].double() @ W[:, c:c + (1 << 22)].double().t()
    # a wave adds 524,292 steps up in runs of 16: chains of 32,768 rounded sums, about sqrt(32768) / 2 half-ulps of the running sum
    err = float((y.double() - ref).norm() / ref.norm())
    assert err < 1.1e-5, err


# rows that begin at any float: one matrix that is small, one that is not
@pytest.mark.parametrize("N,K", [(515, 520), (4100, 1032)])
@pytest.mark.parametrize("M", [1, 5, 8])
@pytest.mark.parametrize("shift", [1, 2, 3])
def test_projection_of_rows_off_the_16_byte_grid(M, N, K, shift):
    say(f"projection M={M} N={N} K={K} shift={shift}")
    g = torch.Generator(device=DEV).manual_seed(N + K + shift)
    W = (torch.randn((N, K), generator=g, device=DEV) * 0.02).bfloat16()
    x = torch.randn((M * K + shift,), generator=g, device=DEV)[shift:].view(M, K)
    assert x.data_ptr() % 16 == 4 * shift
    y = torch.full((M, N), float("nan"), device=DEV)
    make_ctx(si.MINI).amph_gemv(x, W, y, M, N, K)
    ref = x.double() @ W.double().t()
    err = float((y.double() - ref).norm() / ref.norm())
    assert err < 5e-7, err                                    # the bound of the aligned rows above


@pytest.mark.parametrize("M", [5])
def test_projection_of_infinities_and_nan(M):
    N, K = 48, 520
    W = si.normal(si.MINI, 3, "dm.inf", (N, K), 0.02).f32
    x = si.as_f32_exact(si.MINI, 3, "dm.x", (M, K), 1.0)
    x[0, 7], x[1, 300], x[2, 519], x[3, 0], x[3, 1] = np.inf, -np.inf, np.nan, 3.0e38, 1.0e-38
    W[0, 7] = 0.0                                             # 0 * inf
    y = torch.zeros((M, N), device=DEV)
    ctx = make_ctx(si.MINI)
    ctx.amph_gemv(f32_to_dev(x), torch.from_numpy(W).to(DEV).bfloat16(), y, M, N, K)
    got = np_of(y).astype(np.float64)
    with np.errstate(invalid="ignore"):
        ref = x.astype(np.float64) @ W.astype(np.float64).T
    assert np.array_equal(np.isnan(got), np.isnan(ref))
    assert np.array_equal(got[np.isinf(ref)], ref[np.isinf(ref)])
    fin = np.isfinite(ref)
    assert np.all(np.abs(got - ref)[fin] <= 1e-5 * np.maximum(np.abs(ref[fin]), 1.0))


# rows of a launch: one tile exactly, one more than a tile, three tiles, more than a launch takes; 4 * B rows in the heads
@pytest.mark.parametrize("batch,n_new", [(4, 4), (17, 1), (9, 5), (10, 5), (13, 4)])
def test_draft_over_many_rows_matches_the_oracle(batch, n_new):
    cfg = si.with_(si.MINI, batch=batch)
    seed, Ls = 13, 21
    n_h, d_h, d, V, K = cfg.n_heads, cfg.head_dim, cfg.d_model, cfg.vocab, cfg.K
    max_kv = 64
    ctx = make_ctx(cfg, max_kv=max_kv)
    dw = si.draft_weights(cfg, seed)
    dwd, dwo = D.draft_to_device(dw, DEV), draft_f32(dw)
    h = si.as_f32_exact(cfg, seed, "dm.h", (batch, n_new, d), 1.0)
    tok = si.tokens(cfg, seed, "dm.tok", (batch, n_new))
    live = [1 + (3 * b) % n_new for b in range(batch)]
    lens = [Ls - b % 5 for b in range(batch)]
    rows = [[si.normal(cfg, seed, f"dm.sal{s}.{kv}", (batch, n_h, Ls, d_h), 1.0) for kv in "kv"] for s in range(2)]
    sal = torch.zeros((2, batch, 2, n_h, max_kv, d_h), dtype=torch.bfloat16, device=DEV)
    for s in range(2):
        for kv in range(2):
            sal[s, :, kv, :, :Ls] = D.to_device(rows[s][kv], DEV)
    before = np_of(sal)
    sal_len = i32_to_dev(lens)
    idx = torch.zeros((batch, K, cfg.topk), dtype=torch.int32, device=DEV)
    val = torch.zeros((batch, K, cfg.topk), device=DEV)
    logits = torch.zeros((batch, K, V), device=DEV)
    args = (B.Context.draft_struct(dwd), f32_to_dev(h), i32_to_dev(tok), sal, sal_len, idx, val, logits)
    ctx.amph_draft(*args, n_new=n_new, n_valid=i32_to_dev(live))
    assert ctx.device_status() == 0
    assert list(np_of(sal_len)) == [n + r for n, r in zip(lens, live)]
    after, lg = np_of(sal), np_of(logits)
    for b in sorted({0, 1, batch // 2, batch - 1}):
        say(f"batch {batch} n_new {n_new} element {b} live {live[b]}")
        k0 = [rows[s][0].f32[b][:, :lens[b]] for s in range(2)]
        v0 = [rows[s][1].f32[b][:, :lens[b]] for s in range(2)]
        ref, k1, v1 = orc.draft_catchup(dwo, h[b, :live[b]], tok[b, :live[b]], k0, v0, n_h, cfg.topk, cfg.rms_eps, cfg.rope_theta)
        assert_rows_close(lg[b], ref["logits"], TOL["bf16"], "logits")
        for r in range(K):
            ok, bad = topk_consistent(np_of(idx)[b, r], np.asarray(ref["logits"][r]), cfg.topk, 1e-2 * np.abs(ref["logits"][r]).max())
            assert ok, bad
        end = lens[b] + live[b]
        for s in range(2):
            assert_rows_close(after[s, b, 0, :, lens[b]:end].reshape(-1, d_h), k1[s][:, lens[b]:].reshape(-1, d_h), TOL["bf16"], "keys")
            assert_rows_close(after[s, b, 1, :, lens[b]:end].reshape(-1, d_h), v1[s][:, lens[b]:].reshape(-1, d_h), TOL["bf16"], "values")
        assert np.array_equal(after[:, b, :, :, end:], before[:, b, :, :, end:])          # rows of dead positions stay
    # a token outside the vocabulary is reported
    tok[batch - 1, 0] = V
    sal_len.copy_(i32_to_dev(lens))
    args = (*args[:2], i32_to_dev(tok), *args[3:])
    ctx.amph_draft(*args, n_new=n_new, n_valid=i32_to_dev(live))
    assert ctx.device_status() == B.AMPH_DEV_BAD_TOKEN


# Whole drafts at the widths where the launch rule takes two to six row blocks a workgroup and splits the axis, over one, two
# and three tiles of 16 rows and over two launches.  The same values as a float32 model run on the vector kernels (which the
# oracle's tests hold); what may differ is the bf16 rounding of the new cache rows.  Queries and keys of the adaptation layers
# are of size 0.4, so that every row of a cache has a like weight and the new rows' rounding counts with their share; those of
# the self-attention over the heads are small too (its softmax over rows of size 10 would magnify any difference).
def device_draft_weights(d, n_h, f, V, K, seed):
    g = torch.Generator(device=DEV).manual_seed(seed)
    w = lambda *shape, std=0.02: torch.empty(shape, dtype=torch.bfloat16, device=DEV).normal_(0.0, std, generator=g)
    small = 0.4 * d ** -0.5
    gain = lambda: (1.0 + w(d).float() * 5).bfloat16()
    layer = lambda: dict(rms1=gain(), wq=w(d, d, std=small), wk=w(d, d, std=small), wv=w(d, d), wo=w(d, d), rms2=gain(), w_gate=w(f, d), w_up=w(f, d), w_down=w(d, f))
    return dict(embed=w(V, d), fc=[w(d, 2 * d) for _ in range(2)], sal=[layer() for _ in range(2)], mlp=w(K, d, d), pe=w(K, d),
                aeb_wq=w(d, d, std=small / 10), aeb_wk=w(d, d, std=small / 10), aeb_wv=w(d, d), aeb_wo=w(d, d), lm_head=w(V, d))


def to_float(x):
    if isinstance(x, dict):
        return {k: to_float(v) for k, v in x.items()}
    return [to_float(v) for v in x] if isinstance(x, list) else x.float()


@pytest.mark.parametrize("d,n_h,f,K,sizes", [
    (2560, 20, 6912, 4, [(8, 5), (1, 3)]),
    (3072, 24, 8192, 4, [(12, 4), (4, 5)]),
    (4096, 32, 11008, 4, [(4, 5), (8, 5), (12, 4), (10, 5), (8, 1), (2, 1)]),
    (5120, 40, 13824, 4, [(3, 5), (7, 5)]),
    (6656, 52, 17920, 5, [(4, 6), (8, 6), (3, 1)]),
], ids=["2560", "3072", "4096", "5120", "6656"])
def test_draft_on_the_matrix_cores_against_the_vector_kernels(d, n_h, f, K, sizes):
    V, topk, max_kv, d_h = 1000, 10, 416, d // n_h
    wb = device_draft_weights(d, n_h, f, V, K, d)
    models = {B.AMPH_BF16: wb, B.AMPH_F32: to_float(wb)}
    for batch, n_new in sizes:
        say(f"draft width {d}, {batch} sequences of {n_new} positions")
        g = torch.Generator(device=DEV).manual_seed(batch * 100 + n_new)
        lens = [400 - 37 * (b % 7) for b in range(batch)]
        live = [1 + (3 * b + n_new - 1) % n_new for b in range(batch)]
        h = torch.randn((batch, n_new, d), generator=g, device=DEV)
        tok = torch.randint(0, V, (batch, n_new), generator=g, device=DEV, dtype=torch.int32)
        cache = torch.randn((2, batch, 2, n_h, max_kv, d_h), generator=g, device=DEV).bfloat16()
        got = {}
        for code, w in models.items():
            ctx = B.Context(d_model=d, n_heads=n_h, head_dim=d_h, d_ffn=f, vocab=V, K=K, topk=topk, max_tree=16, max_kv=max_kv,
                            batch=batch, dtype=code, rms_eps=1e-6, rope_theta=10000.0, device=DEV)
            kv, sal_len = cache.to(w["embed"].dtype), i32_to_dev(lens)
            idx = torch.zeros((batch, K, topk), dtype=torch.int32, device=DEV)
            val, logits = torch.zeros((batch, K, topk), device=DEV), torch.full((batch, K, V), float("nan"), device=DEV)
            ctx.amph_draft(B.Context.draft_struct(w), h, tok, kv, sal_len, idx, val, logits, n_new=n_new, n_valid=i32_to_dev(live))
            assert ctx.device_status() == 0
            got[code] = (logits.double(), kv, val, idx, sal_len)
        (lb, kb, vb, ib, nb), (lf, kf, _, _, nf) = got[B.AMPH_BF16], got[B.AMPH_F32]
        assert torch.equal(nb, nf) and [int(n) for n in nb] == [n + r for n, r in zip(lens, live)]
        # relative to a row's largest logit: float32 sums, and 2^-9 (three deviations) of the new rows' values by the root of their
        # share in the attention, whose output over hundreds of rows is below a tenth of what it is added to
        err = ((lb - lf).abs().amax(-1) / lf.abs().amax(-1)).amax()
        say(f"  logits differ by {float(err):.2e}")
        assert float(err) < 1e-5 + 0.1 * 3 * 2.0 ** -9 * (n_new / (min(lens) + n_new)) ** 0.5
        assert torch.equal(vb.double(), torch.gather(lb, 2, ib.long())) and torch.equal(vb.double(), lb.topk(topk, -1).values)
        for b in range(batch):
            end = lens[b] + live[b]
            a, c = kb[:, b, :, :, lens[b]:end].double(), kf[:, b, :, :, lens[b]:end].double()
            assert float((a - c).abs().max()) <= 2.0 ** -8 * float(c.abs().max())          # the rounding to bf16 (half of it)
            assert float((a - c).norm() / c.norm()) < 2.0 ** -8
            assert torch.equal(kb[:, b, :, :, end:], cache[:, b, :, :, end:])              # rows of dead positions stay

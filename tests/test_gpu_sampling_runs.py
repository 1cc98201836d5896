"""The sampling draw's run sums at vocabularies around the thread count and its multiples, and the commit at the deepest
paths, the other head widths and fewer heads than gathered rows, and of nothing."""
import numpy as np
import pytest
import torch

import synth_inputs as si
from oracle import amphista_oracle as orc
from paper_2406_13170_amd import binding as B
from paper_2406_13170_amd import device as D

import test_gpu_loop
from gpu_common import DEV, f32_to_dev, i32_to_dev, make_ctx, say
from test_gpu_typical import run_case

pytestmark = pytest.mark.gpu

LAST = np.float32(1.0) - np.float32(2.0 ** -24)               # u * Z may reach the rounded total: the last live token


# one token a run and fewer, two with an empty tail of runs, eight exactly and nine, 31 and 32 with a ragged last run
@pytest.mark.parametrize("V", [5, 63, 1023, 1024, 1025, 8191, 8192, 8193, 31745, 32000])
def test_draw_at_run_edges(V):
    say(f"draw at run edges V={V}")
    T, caps = (1, (4, 4, 4, 4)) if V < 16 else (16, (4, 2, 2, 2))
    run_case(V, T, caps, 4, 9, 0.7, 0.09, 0.3, spread=1.5, us=np.array([0.0, 0.31, 0.77, LAST], dtype=np.float32))


def test_draw_at_the_end_of_the_live_tokens():
    """Half of the vocabulary has probability zero; u is the largest below 1, the draw one of the last live tokens."""
    V = 3000
    logits = np.random.default_rng(4).standard_normal((2, 1, V)).astype(np.float32)
    logits[0, 0, 1501:] = -np.inf
    logits[1, 0, ::2] = -1.0e30
    run_case(V, 1, (4, 4, 4, 4), 2, 5, 1.0, 0.09, 0.3, logits=logits, toks=np.zeros((2, 1), dtype=np.int32),
             us=np.array([LAST, LAST], dtype=np.float32))


def emulated_draw(x):
    """Z and the scan's total in float32, in the kernels' orders: 1024 threads a strided and a consecutive share of the exponentials."""
    n = 1024
    e = np.exp(x - x.max(), dtype=np.float32)
    C = (len(e) + n - 1) // n
    e = np.pad(e, (0, C * n - len(e)))
    z, run = np.zeros(n, dtype=np.float32), np.zeros(n, dtype=np.float32)
    for j in range(C):
        z += e.reshape(C, n)[j]
        run += e.reshape(n, C)[:, j]
    z, inc = z.reshape(16, 64), run.reshape(16, 64)
    lane = np.arange(64)
    for off in (32, 16, 8, 4, 2, 1):
        z = z + z[:, lane ^ off]
    for off in (1, 2, 4, 8, 16, 32):
        inc = np.where(lane >= off, inc + inc[:, np.maximum(lane - off, 0)], inc)
    add = lambda v: np.add.accumulate(v, dtype=np.float32)[-1]  # noqa: E731
    base = np.float32(0) if len(inc) == 1 else add(inc[:-1, 63])
    return add(z[:, 0]), inc[-1, 63] + base


@pytest.mark.parametrize("live", [65536, 65000, 64576])
def test_draw_that_no_run_reaches_takes_the_last_live_token(live):
    """One token of probability near 1 ahead of 63 small ones in its run, which it swallows there and not in the strided order of
    Z: the run sums end 16 float32 steps and more below u * Z, no run crosses, and the last token of non-zero probability counts."""
    V = 65536
    x = np.full(V, -17.33, dtype=np.float32)
    x[64512] = 0.0
    x[live:] = -np.inf
    z, total = emulated_draw(x)
    assert total < LAST * z - 4 * np.spacing(z)                # (the device's exponentials may differ in the last place)
    cfg = si.with_(si.TINY, vocab=V, batch=1, K=4, topk=4)
    ctx = make_ctx(cfg, T=1, batch=1)
    tree = B.Tree([], 4)
    out = [torch.full((n,), -7, dtype=torch.int32, device=DEV) for n in (1, 5, 1, 1)]
    ctx.amph_accept_typical(tree, i32_to_dev([0]), f32_to_dev(x[None, None]), 1.0, 0.09, 0.3, f32_to_dev(np.array([LAST])), out[0], out[1],
                            out[2], out[3])
    a_len, path, nxt, best = (t.tolist() for t in out)
    assert a_len == [0] and best == [0] and path == [0, -1, -1, -1, -1]
    assert nxt == [live - 1]


@pytest.mark.parametrize("cfg,T,caps,L,B_", [
    (si.with_(si.MINI, name="mini_deep"), 40, (2,) * 8, 50, 2),                                    # K = 8 rows in bf16
    (si.with_(si.TINY, name="tiny_deep_dh128", d_model=512, head_dim=128), 33, (2,) * 8, 27, 2),   # ... 128 wide in float32
    (si.with_(si.MINI, name="mini_dh64", d_model=256, head_dim=64), 64, (10,) * 4, 63, 1),
    (si.with_(si.TINY, name="tiny_one_head", d_model=64, n_heads=1), 16, (4, 2, 2, 2), 5, 1),      # one head gathers K + 1 rows
])
def test_commit_of_deep_paths_and_other_head_widths(cfg, T, caps, L, B_):
    test_gpu_loop.test_commit_moves_the_accepted_rows_and_gathers_the_next_draft_inputs(cfg, T, caps, L, B_)


@pytest.mark.parametrize("cfg", [
    si.with_(si.MINI, name="mini_every_length"),                                                   # 128 wide, two value rows at a time
    si.with_(si.MINI, name="mini_every_length_dh64", d_model=256, head_dim=64),                    # ... and four
    si.with_(si.TINY, name="tiny_every_length_dh128", d_model=512, head_dim=128),
    si.with_(si.TINY, name="tiny_every_length"),
])
def test_commit_of_every_length(cfg):
    """Ten sequences of one call: number b of nine accepted b nodes, the tenth has no room for its tree.  Data movement: exact."""
    T, K, L, n_layers = 17, 8, 29, 2
    cfgx = si.with_(cfg, batch=10, K=K, topk=2)
    max_kv = 96
    say(f"commit {cfg.name}: every accepted length")
    ctx = make_ctx(cfgx, T=T, max_kv=max_kv)
    tree = B.Tree([(1,) * m + (r,) for m in range(K) for r in range(2)], K)
    chain = [2 * m for m in range(K + 1)]                          # the second child of every node on the way
    assert tree.T == T and [int(tree.parent[n]) for n in chain] == [-1] + chain[:-1]
    a = list(range(K + 1)) + [3]
    lens = [L] * (K + 1) + [max_kv - T + 1]                       # the last has no room for the tree: nothing moves
    path = [chain[:n + 1] + [-1] * (K - n) for n in a]
    shape = (n_layers, cfgx.batch, cfg.n_heads, max_kv, cfg.head_dim)
    rows = [torch.randn(shape, generator=torch.Generator().manual_seed(i)).to(D.torch_dtype(cfg.dtype)).to(DEV) for i in range(2)]
    k_caches, v_caches = D.pack_kv(ctx, *rows)
    kv_len = i32_to_dev(lens)
    ctx.amph_commit(tree, n_layers, k_caches, v_caches, kv_len, i32_to_dev(a), i32_to_dev(path))
    assert kv_len.tolist() == [n + x + 1 for n, x in zip(lens[:-1], a)] + lens[-1:]
    for got, src in zip(D.unpack_kv(ctx, k_caches, v_caches), rows):
        want = src.clone()
        for b in range(K + 1):
            for j in range(1, a[b] + 1):
                want[:, b, :, L + j] = src[:, b, :, L + chain[j]]
        assert torch.equal(got, want)                             # the rows past the accepted ones keep what they held


def test_commit_takes_time_for_what_was_accepted_only():
    """Deep caches (60 layers, four sequences, 52 heads): with nothing accepted there is nothing to read.  A commit of nothing takes
    0.24 of one of a row a sequence (9.2 of 38.2 us); it took 0.51 (28.8 of 56.2) where it read rows that nobody had accepted."""
    T, L, n_layers = 96, 63, 60
    cfg = si.with_(si.V33B, batch=4)
    K = cfg.K
    ctx = make_ctx(cfg, T=T, max_kv=160)
    otree = orc.tree_from_paths(si.tree_paths(T, (10,) * K), K)
    tree = B.Tree(si.tree_paths(T, (10,) * K), K)
    chain = [int(n) for n in max(otree.retrieve, key=lambda r: sum(n >= 0 for n in r))]
    shape = (n_layers, cfg.batch, cfg.n_heads, 160, cfg.head_dim)
    k_caches = torch.randint(-2 ** 15, 2 ** 15, shape, dtype=torch.int16, device=DEV)
    v_caches = torch.randint(-2 ** 15, 2 ** 15, shape, dtype=torch.int16, device=DEV)
    before = k_caches.clone(), v_caches.clone()
    kv_len = torch.empty((cfg.batch,), dtype=torch.int32, device=DEV)
    us = {}
    for a in (0, 1):
        a_len = i32_to_dev([a] * cfg.batch)
        path = i32_to_dev([chain[:a + 1] + [-1] * (K - a)] * cfg.batch)
        times = []
        for _ in range(30):
            kv_len.fill_(L)
            ev = [torch.cuda.Event(enable_timing=True) for _ in range(2)]
            ev[0].record()
            ctx.amph_commit(tree, n_layers, k_caches, v_caches, kv_len, a_len, path)
            ev[1].record()
            torch.cuda.synchronize()
            times.append(ev[0].elapsed_time(ev[1]) * 1e3)
        us[a] = min(times)
        assert kv_len.tolist() == [L + a + 1] * cfg.batch
        if a == 0:                                             # not a byte of the caches moves
            assert torch.equal(k_caches, before[0]) and torch.equal(v_caches, before[1])
    say(f"commit of nothing {us[0]:.1f} us, of one row a sequence {us[1]:.1f} us")
    assert us[0] < 0.38 * us[1]

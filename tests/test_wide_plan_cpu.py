"""The wide GEMM's plan on the host: the shapes that its instances are tested on take these instances, and no call takes another."""
import random

import pytest

import synth_inputs as si
import test_gpu_target_gemm as tg
import wide_plan as wp


@pytest.mark.parametrize("case", wp.LAYERS + wp.HEADS, ids=lambda c: "-".join(str(x) for x in c[:6]))
def test_cases_take_the_instances_they_are_there_for(case):
    got = {wp.instance(*g) for g in wp.gemms(case) if wp.instance(*g) and wp.ragged(*g)}
    assert case[-1] <= got, (case[-1] - got, got)


def test_every_instance_that_the_plan_selects_has_a_case():
    """2,500 models and row counts over what amph_create accepts, of each storage type."""
    have = {dt: set().union(*(c[-1] for c in wp.LAYERS + wp.HEADS if c[0] == dt)) for dt in wp.ELEM}
    assert {dt: len(s) for dt, s in have.items()} == {"bf16": 56, "f32": 16}
    rng = random.Random(5)
    for dt in wp.ELEM:
        for _ in range(2500):
            d, f, V = 64 * rng.randint(1, 160), 32 * rng.randint(1, 1024), rng.randint(16, 65536)
            M = rng.choice([rng.randint(65, 1024), rng.randint(65, 8192)])
            for epi, rows, Kd in wp.layer_gemms(d, f) + [(wp.ARGMAX, V, d)]:
                p, got = wp.plan(dt, epi, rows, Kd, M), wp.instance(dt, epi, rows, Kd, M)
                assert got is None or got in have[dt], (dt, epi, rows, Kd, M, got)
                if got:                                        # groups cover the rows, waves their group's tiles, the slices are not empty
                    tiles = (M + 31) // 32
                    assert p.mgroups * p.gt >= tiles > (p.mgroups - 1) * p.gt and p.tw == (p.gt + 3) // 4 <= 3
                    assert p.tiles * p.nb >= p.blocks > (p.tiles - 1) * p.nb and Kd * wp.ELEM[dt] // 64 >= p.split


@pytest.mark.parametrize("cfg,M,wide", [
    (si.MINI, 128, ""), (tg.EIGHT, 128, "gate_up head"), (tg.TEN, 65, "gate_up head"), (tg.QKV, 65, "qkv wo"), (tg.QKV, 128, "qkv"),
    (tg.DOWN, 65, "down"),                                     # (its input comes from a skinny gate/up: the pass leaves it to that kernel)
    (si.V7B, 80, "qkv gate_up down head"), (tg.TEN_F32, 80, ""), (si.TINY, 128, ""),
], ids=lambda x: getattr(x, "name", str(x)))
def test_two_blocks_of_rows_as_their_test_says(cfg, M, wide):
    gemms = zip(["qkv", "wo", "gate_up", "down", "head"], wp.layer_gemms(cfg.d_model, cfg.d_ffn) + [(wp.ARGMAX, cfg.vocab, cfg.d_model)])
    assert [n for n, g in gemms if wp.instance(cfg.dtype, *g, M)] == wide.split()


@pytest.mark.parametrize("dt,epi", [("bf16", wp.STORE), ("bf16", wp.QKV), ("bf16", wp.SWIGLU), ("bf16", wp.ARGMAX), ("f32", wp.STORE)])
def test_large_operands(dt, epi):
    """Activations of 2 GiB and more, and of more than 4, are the wide kernel's; its offsets in a workgroup's weights have 32 bits: what
    sixteen blocks would need more for is the skinny one's."""
    for M in (129, 8192):
        for row_bytes in ((1 << 18) - 64, 1 << 18, (1 << 18) + 64, 1 << 19, (1 << 19) + 64, (1 << 24) - 64):
            assert wp.plan(dt, epi, 256, row_bytes // wp.ELEM[dt], M).wide, (M, row_bytes)
        assert not wp.plan(dt, epi, 256, (1 << 24) // wp.ELEM[dt], M).wide


# What launches in a row took (us) with some of their plans (row blocks a workgroup, groups of rows): groups of five, six, nine and ten
# tiles, whose busiest wave has three or five sixteens of rows; float32.
MEASURED = [
    ("bf16", wp.QKV, 5120, 5120, 352, 1, {(8, 2): 60.1, (4, 1): 70.2}),
    ("bf16", wp.STORE, 5120, 13824, 144, 4, {(6, 1): 36.9, (10, 2): 42.8}),
    ("bf16", wp.STORE, 5120, 13824, 256, 1, {(4, 3): 75.7, (4, 2): 87.7}),
    ("bf16", wp.STORE, 6656, 17920, 352, 2, {(8, 2): 94.0, (4, 1): 108.7}),
    ("bf16", wp.STORE, 6656, 17920, 640, 4, {(8, 2): 139.4, (10, 3): 158.1}),
    ("bf16", wp.STORE, 6656, 6656, 512, 1, {(8, 4): 58.1, (4, 2): 65.8}),
    ("f32", wp.QKV, 2048, 2048, 336, 1, {(4, 2): 93.0, (8, 3): 121.9}),
    ("f32", wp.SWIGLU, 5632, 2048, 144, 1, {(4, 1): 92.6, (8, 2): 118.0}),
    ("f32", wp.STORE, 4096, 11008, 576, 1, {(4, 4): 460.7, (8, 6): 610.1}),
]


@pytest.mark.parametrize("dt,epi,rows,Kd,M,split,us", MEASURED, ids=lambda x: str(x) if not isinstance(x, dict) else "")
def test_picks_are_the_fast_plans(dt, epi, rows, Kd, M, split, us):
    p = wp.plan(dt, epi, rows, Kd, M, split)
    assert us.get((p.nb, p.mgroups)) == min(us.values()), (p.nb, p.mgroups)
    assert abs(p.cost / min(us.values()) - 1) < 0.2                    # (it deviates by 6 % over thousands of them)


@pytest.mark.parametrize("shapes", [[(2048, 8160), (2048, 8192)], [(4096, 4064), (4096, 4096), (4096, 4128)]], ids=str)
def test_slabs_do_not_jump_between_like_shapes(shapes):
    for M in (144, 256, 384, 512, 768):
        assert len({wp.plan("bf16", wp.STORE, rows, Kd, M).split for rows, Kd in shapes}) == 1, M

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

"""Verification attention on both sides of the line up to which one workgroup walks a head's cache alone, and its key splits and their
fold under several query groups."""
import pytest

import synth_inputs as si
from gpu_common import say
from test_gpu_kernels import verify_case
from test_verify_plan_cpu import splits

pytestmark = pytest.mark.gpu

MINI64 = si.with_(si.MINI, name="mini_64_wide", d_model=256, head_dim=64)


@pytest.mark.parametrize("cfg,T,max_kv,n", [
    (si.MINI, 64, 512, 1), (si.MINI, 64, 544, 5),                # 128-wide heads in bf16: four key steps a wave, and five
    (si.MINI, 61, 512, 1), (si.MINI, 1, 512, 1), (si.MINI, 1, 544, 5),
    (MINI64, 64, 768, 1), (MINI64, 64, 800, 7),                  # 64-wide ones: six, and seven
    (si.TINY, 96, 192, 1), (si.TINY, 96, 224, 4),                # float32: three, and four
    (si.TINY, 16, 256, 1), (si.TINY, 16, 288, 5),                # over few queries four, and five
    (si.MINI, 96, 576, 5), (si.MINI, 128, 576, 5),               # splits under three and four query groups, ragged in both
    (si.MINI, 113, 640, 5), (si.TINY, 96, 352, 6), (si.TINY, 128, 352, 6),
])
def test_short_caches(cfg, T, max_kv, n):
    """The cache full to its last row, and two sequences, one of them short, of which the longer leaves a ragged last key step."""
    say(f"verify_attn {cfg.name} T={T}, caches of {max_kv} rows, register kernel")
    assert splits(cfg.dtype, cfg.head_dim, cfg.n_heads, 1, T, max_kv) == n
    say(f"  worst row error {verify_case(cfg, T, (10,) * 8, max_kv - T, kernel=0, max_kv=max_kv):.2e}")
    L = max_kv - T - 5
    say(f"  batch of two, one short: {verify_case(cfg, T, (10,) * 8, L, B_=2, lens=[L, 3], kernel=0, max_kv=max_kv):.2e}")

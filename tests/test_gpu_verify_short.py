"""Verification attention on both sides of the line up to which one workgroup walks a head's cache alone (256 KB of bf16, 128 KB of float32)."""
import pytest

import synth_inputs as si
from gpu_common import say
from test_gpu_kernels import verify_case

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("cfg,T,L", [
    (si.MINI, 64, 448), (si.MINI, 64, 449),     # 512 rows of 128 dims, and a key step more
    (si.MINI, 61, 387),                         # ragged queries and keys
    (si.TINY, 16, 240), (si.TINY, 16, 241),     # 256 rows of 64 dims in float32, and more
    (si.MINI, 1, 511),
])
def test_short_caches(cfg, T, L):
    say(f"verify_attn {cfg.name} T={T} L={L}, kernel by shape")
    say(f"  worst row error {verify_case(cfg, T, (10,) * 4, L):.2e}")
    say(f"  batch of two, one short: {verify_case(cfg, T, (10,) * 4, L, B_=2, lens=[L, 3]):.2e}")

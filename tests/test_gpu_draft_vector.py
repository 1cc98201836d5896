"""Drafts on the vector kernels where their rows no longer fit in LDS whole, against the oracle: Eq. 1 over half its columns at a
time, W_down over slices of the reduction axis, the head MLPs one source at a time; and one or two bf16 rows against matrices
that the matrix cores do not take."""
import pytest

import synth_inputs as si

from test_gpu_draft_attn import check_draft

pytestmark = pytest.mark.gpu


def model(name, base, n_h, d_h, f, V=512):
    return si.with_(base, name=name, d_model=n_h * d_h, n_heads=n_h, head_dim=d_h, d_ffn=f, vocab=V)


@pytest.mark.parametrize("cfg,n_new,lens,live", [
    # float32: five rows of [h ; e] are 140 KB, of the FFN 160 and 320
    (model("f32_wide_fc", si.TINY, 56, 64, 512), 5, [20], [4]),
    (model("f32_wide_ffn", si.TINY, 8, 64, 8192), 5, [20], [5]),
    (model("f32_wider_ffn", si.TINY, 8, 64, 16384), 5, [3], [2]),
    # six rows of both head sources are 172 KB, of one 86; two launches of rows with eleven
    (model("f32_heads_by_source", si.TINY, 56, 64, 256), 1, [20, 0, 5, 31, 1, 9], [1] * 6),
    (model("f32_heads_by_source", si.TINY, 56, 64, 256), 1, [20, 0, 5, 31, 1, 9, 2, 3, 4, 17, 22], [1] * 11),
    # bf16: Eq. 1 at widths that are no multiple of 256, its rows whole and in halves
    (model("bf16_odd_fc", si.MINI, 9, 64, 512), 5, [20], [5]),
    (model("bf16_wide_odd_fc", si.MINI, 57, 64, 512), 5, [20], [4]),
    # one and two rows against more than 4 M weights in every projection; W_down over slices
    (model("bf16_two_rows", si.MINI, 18, 128, 2304, V=2304), 1, [20], [1]),
    (model("bf16_two_rows", si.MINI, 18, 128, 2304, V=2304), 1, [20, 7], [1, 1]),
    (model("bf16_two_rows", si.MINI, 18, 128, 2304, V=2304), 2, [20], [2]),
    (model("bf16_sliced_ffn", si.MINI, 4, 128, 17920), 1, [20, 7], [1, 1]),
], ids=lambda v: v.name if isinstance(v, si.Config) else None)
def test_draft_on_the_vector_kernels(cfg, n_new, lens, live):
    check_draft(cfg, n_new, 64, lens, live)

"""Where the verification attention's register kernel stops walking a head's cache with one workgroup and splits its keys, as the
library plans it: by the key steps of a wave, for each storage type and head width."""
import ctypes as C

import pytest

from paper_2406_13170_amd import binding as B

ELEM = {"bf16": 2, "f32": 4}
REGS = 0

# dtype, head_dim, heads, sequences, tree nodes, cache rows, key splits of the register kernel
EDGES = [
    ("bf16", 128, 4, 1, 64, 512, 1), ("bf16", 128, 4, 1, 64, 544, 5), ("bf16", 128, 52, 2, 48, 512, 1), ("bf16", 128, 52, 2, 48, 544, 1),
    ("bf16", 128, 52, 1, 48, 512, 1), ("bf16", 128, 52, 1, 48, 544, 2),
    ("bf16", 64, 32, 1, 64, 768, 1), ("bf16", 64, 32, 1, 64, 800, 4), ("bf16", 64, 32, 1, 64, 1024, 4), ("bf16", 64, 4, 1, 16, 1024, 8),
    ("f32", 128, 8, 1, 96, 128, 1), ("f32", 128, 8, 1, 96, 160, 3), ("f32", 128, 8, 1, 16, 160, 3),
    ("f32", 64, 4, 1, 96, 192, 1), ("f32", 64, 4, 1, 96, 224, 4), ("f32", 64, 4, 1, 16, 256, 1), ("f32", 64, 4, 1, 17, 256, 4),
    ("f32", 64, 4, 1, 16, 288, 5), ("f32", 64, 24, 1, 96, 256, 1), ("f32", 64, 24, 1, 96, 288, 3),
]


def splits(dtype, d_h, heads, Bsz, T, max_kv, kernel=REGS):
    f = B.lib()["_ZN4amph22verify_partials_floatsEiiiiiii"]       # amph::verify_partials_floats(B, T, heads, d_h, max_kv, element bytes, kernel)
    f.restype, f.argtypes = C.c_size_t, [C.c_int] * 7
    groups = ((T + 15) // 16 + 1) // 2
    nq = ((T + 15) // 16 + groups - 1) // groups * 16
    one = Bsz * groups * heads * (nq * d_h + 2 * nq)              # floats of one split's partials (without splits there are none)
    n = f(Bsz, T, heads, d_h, max_kv, ELEM[dtype], kernel)
    assert n % one == 0
    return n // one or 1


@pytest.mark.parametrize("case", EDGES, ids=lambda c: "-".join(str(x) for x in c))
def test_key_splits_begin_where_a_wave_walks_too_far(case):
    assert splits(*case[:-1]) == case[-1]

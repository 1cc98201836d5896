"""Which instance of the wide GEMM a matrix takes, as the library plans it, and small shapes that between them take every one.

A GEMM is (epilogue, pairs of weight row blocks a workgroup, tiles of 32 activation rows a wave).  A case is (storage type, tree nodes,
sequences, d_model, head_dim, d_ffn or vocabulary) with the instances that it is here for; each of these has a reduction axis of at least
nine steps of 64 bytes that ends inside a round of eight (two LDS stages), and most have ragged tiles of rows and of weights."""
import ctypes as C

from paper_2406_13170_amd import binding as B

STORE, QKV, SWIGLU, ARGMAX = 0, 2, 3, 4
ELEM = {"bf16": 2, "f32": 4}


class Plan(C.Structure):
    _fields_ = [(n, C.c_int) for n in ("nb", "split", "tiles", "blocks")] + [("wide", C.c_bool)] + \
               [(n, C.c_int) for n in ("mgroups", "tw", "gt")] + [("cost", C.c_double)]


def plan(dtype, epi, rows, Kd, M, split=0) -> Plan:
    f = B.lib()["_ZN4amph9gemm_planEiiiiiib"]                 # amph::gemm_plan(epi, rows, Kd, element bytes, M, split, tiled)
    f.restype, f.argtypes = Plan, [C.c_int] * 6 + [C.c_bool]
    return f(epi, rows, Kd, ELEM[dtype], M, split if epi == STORE else 1, True)


def instance(dtype, epi, rows, Kd, M):
    """(epilogue, pairs, tiles a wave), or None where the skinny kernel takes it."""
    p = plan(dtype, epi, rows, Kd, M)
    return (epi, p.nb // 2, p.tw) if p.wide else None


def layer_gemms(d, f):
    """(epilogue, rows, reduction length): Q, K and V; W_o; gate and up; W_down."""
    return [(QKV, d, d), (STORE, d, d), (SWIGLU, f, d), (STORE, d, f)]


def ragged(dtype, epi, rows, Kd, M):
    p, steps = plan(dtype, epi, rows, Kd, M), Kd * ELEM[dtype] // 64
    n = [steps * (s + 1) // p.split - steps * s // p.split for s in range(p.split)]
    return min(n) >= 9 and any(x % 8 for x in n)


LAYERS = [
    ("bf16", 12, 11, 320, 64, 288, {(STORE, 2, 1), (QKV, 2, 1), (SWIGLU, 2, 1)}),
    ("bf16", 50, 41, 832, 64, 416, {(STORE, 2, 2), (QKV, 2, 3), (SWIGLU, 2, 2)}),
    ("bf16", 38, 54, 320, 64, 1120, {(STORE, 3, 1), (SWIGLU, 3, 2)}),
    ("bf16", 41, 32, 384, 64, 832, {(QKV, 3, 1)}),
    ("bf16", 49, 53, 384, 64, 7040, {(STORE, 3, 2), (SWIGLU, 5, 2)}),
    ("bf16", 77, 27, 384, 64, 1280, {(QKV, 2, 2), (SWIGLU, 2, 3)}),
    ("bf16", 85, 31, 448, 64, 544, {(QKV, 3, 2)}),
    ("bf16", 70, 44, 576, 64, 832, {(QKV, 4, 2), (SWIGLU, 4, 2)}),
    ("bf16", 89, 39, 832, 64, 4928, {(STORE, 4, 2), (QKV, 5, 2), (SWIGLU, 5, 3)}),
    ("bf16", 114, 25, 2432, 64, 1056, {(STORE, 5, 2), (SWIGLU, 3, 3)}),
    ("bf16", 77, 46, 1088, 64, 1408, {(STORE, 5, 1), (QKV, 5, 3), (SWIGLU, 6, 2)}),
    ("bf16", 72, 54, 1088, 64, 1568, {(QKV, 8, 2), (SWIGLU, 8, 2)}),
    ("bf16", 77, 41, 2688, 128, 320, {(STORE, 4, 3), (SWIGLU, 3, 1)}),
    ("bf16", 95, 41, 2688, 128, 320, {(STORE, 6, 2)}),
    ("bf16", 81, 38, 3200, 128, 320, {(STORE, 5, 3), (QKV, 4, 3)}),
    ("bf16", 100, 40, 3200, 128, 256, {(STORE, 8, 2)}),
    ("bf16", 100, 41, 832, 64, 352, {(STORE, 2, 3)}),
    ("bf16", 61, 42, 576, 64, 4736, {(STORE, 3, 3)}),
    ("bf16", 61, 51, 448, 64, 1792, {(STORE, 4, 1)}),
    ("bf16", 96, 43, 448, 64, 384, {(QKV, 3, 3)}),
    ("bf16", 100, 31, 320, 64, 256, {(QKV, 4, 1)}),
    ("bf16", 53, 58, 384, 64, 256, {(QKV, 5, 1)}),
    ("bf16", 114, 25, 896, 128, 288, {(QKV, 6, 2)}),
    ("bf16", 37, 7, 320, 64, 4160, {(SWIGLU, 4, 1)}),
    ("bf16", 27, 29, 320, 64, 4640, {(SWIGLU, 4, 3)}),
    ("bf16", 65, 4, 320, 64, 6176, {(SWIGLU, 5, 1)}),
    ("f32", 11, 13, 320, 64, 320, {(STORE, 2, 1), (QKV, 2, 1), (SWIGLU, 2, 1)}),
    ("f32", 56, 14, 704, 64, 1216, {(QKV, 2, 2), (SWIGLU, 2, 2)}),
    ("f32", 97, 8, 576, 64, 3008, {(SWIGLU, 4, 2)}),
    ("f32", 31, 30, 2112, 64, 256, {(QKV, 4, 2)}),
    ("f32", 43, 3, 1088, 64, 2208, {(STORE, 2, 2)}),
    ("f32", 18, 15, 2112, 64, 3904, {(STORE, 4, 1)}),
    ("f32", 62, 28, 640, 64, 4416, {(STORE, 4, 2)}),
    ("f32", 25, 21, 1728, 64, 256, {(QKV, 4, 1)}),
    ("f32", 11, 24, 320, 64, 4224, {(SWIGLU, 4, 1)}),
]

HEADS = [
    ("bf16", 47, 3, 320, 64, 1140, {(ARGMAX, 2, 1)}),
    ("bf16", 15, 54, 320, 64, 2103, {(ARGMAX, 3, 1)}),
    ("bf16", 18, 61, 320, 64, 2338, {(ARGMAX, 2, 2)}),
    ("bf16", 101, 13, 320, 64, 2580, {(ARGMAX, 3, 2)}),
    ("bf16", 38, 42, 320, 64, 4215, {(ARGMAX, 3, 3)}),
    ("bf16", 58, 27, 320, 64, 4627, {(ARGMAX, 5, 2)}),
    ("bf16", 27, 57, 320, 64, 5391, {(ARGMAX, 4, 3)}),
    ("bf16", 81, 22, 320, 64, 5285, {(ARGMAX, 6, 2)}),
    ("bf16", 65, 24, 320, 64, 6161, {(ARGMAX, 5, 3)}),
    ("bf16", 110, 21, 320, 64, 5434, {(ARGMAX, 8, 2)}),
    ("bf16", 57, 36, 320, 64, 1544, {(ARGMAX, 2, 3)}),
    ("bf16", 35, 44, 320, 64, 1541, {(ARGMAX, 4, 1)}),
    ("bf16", 95, 27, 320, 64, 1538, {(ARGMAX, 4, 2)}),
    ("bf16", 115, 27, 320, 64, 1029, {(ARGMAX, 5, 1)}),
    ("f32", 31, 6, 320, 64, 1112, {(ARGMAX, 2, 1)}),
    ("f32", 32, 25, 320, 64, 2427, {(ARGMAX, 2, 2)}),
    ("f32", 18, 59, 320, 64, 3664, {(ARGMAX, 4, 2)}),
    ("f32", 19, 27, 320, 64, 5128, {(ARGMAX, 4, 1)}),
]


def gemms(case):
    dtype, T, Bsz, d, _, n, _ = case
    return [(dtype, epi, rows, Kd, T * Bsz) for epi, rows, Kd in (layer_gemms(d, n) if case in LAYERS else [(ARGMAX, n, d)])]

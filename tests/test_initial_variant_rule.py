"""The rule that picks a new context's collide-stream variant, compiled from
its header: on the shapes timed on either side of each line it gives the variant
that was the faster one there (or one within 1 %)."""
import ctypes as C
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
BYTES = {"fp64": 8, "fp32": 4, "fp16": 2, "bf16": 2}

# boxes' sites, storage, lattice, walls, nx of a single box -> variant
CASES = [
    (96 ** 3, "fp32", 19, False, 96, 3),
    (118 ** 3, "fp32", 19, False, 118, 3),
    (64 ** 3, "fp16", 19, True, 64, 3),
    (120 ** 3, "fp32", 19, False, 120, 12),
    (162 ** 3, "fp32", 19, False, 162, 12),
    (144 ** 3, "fp32", 27, False, 144, 12),
    (172 ** 3, "fp16", 19, False, 172, 12),
    (168 ** 3, "fp32", 19, False, 168, 15),        # 12: 166 us against 140
    (172 ** 3, "fp32", 19, False, 172, 15),        # 12: 152 against 145
    (4_485_000, "fp32", 19, False, 0, 15),         # 36 boxes, 12: 131 against 117
    (136 ** 3, "fp64", 19, False, 136, 15),
    (154 ** 3, "fp32", 27, False, 154, 0),         # 12: 167 against 153
    (116 ** 3, "fp64", 27, False, 116, 0),         # 12: 137 against 130
    (256 ** 3, "fp32", 27, False, 256, 0),
    (256 ** 3, "fp16", 19, False, 256, 15),
    (256 ** 3, "fp32", 19, True, 256, 15),
    (64 * 480 * 512, "fp32", 19, False, 64, 1),    # 15: 481 against 459
    (64 * 512 * 512, "fp64", 19, False, 64, 15),
    (64 * 512 * 512, "fp16", 19, True, 64, 15),
    (256 ** 3, "fp16", 19, True, 256, 1),          # 15: 334 against 277
    (256 ** 3, "bf16", 19, True, 256, 1),
    (128 * 256 * 256, "fp16", 19, True, 128, 1),   # 15: 184 against 168
    (256 * 64 * 64, "fp16", 19, True, 256, 1),
    (256 * 32 * 64, "fp16", 19, True, 256, 3),
    (152 ** 3, "fp16", 19, True, 152, 3),          # 12: 63 against 55
    (136 ** 3, "fp16", 27, True, 136, 3),          # 12: 86 against 76
    (154 ** 3, "fp16", 19, True, 154, 12),
    (256 * 128 * 128, "fp16", 19, True, 256, 12),
]


@pytest.fixture(scope="module")
def rule(tmp_path_factory):
    d = tmp_path_factory.mktemp("rule")
    src = d / "rule.cpp"
    src.write_text('#include "initial_variant.h"\n'
                   'extern "C" int rule(int lattice, int bytes, double mb, int rows_k, int walls) {\n'
                   '    return lbd::initial_variant(lattice, bytes, mb, rows_k, walls != 0);\n}\n')
    so = d / "rule.so"
    subprocess.run(["g++", "-std=c++17", "-shared", "-fPIC", "-I",
                    os.path.join(ROOT, "paper_2403_05443_amd", "csrc"), str(src), "-o", str(so)], check=True)
    f = C.CDLL(str(so)).rule
    f.argtypes = [C.c_int, C.c_int, C.c_double, C.c_int, C.c_int]
    return f


@pytest.mark.parametrize("sites,storage,lattice,walls,nx,variant", CASES)
def test_variant_on_either_side_of_each_line(rule, sites, storage, lattice, walls, nx, variant):
    mb = sites * lattice * BYTES[storage] / 1e6
    rows_k = nx // 64 if lattice == 19 and nx in (64, 128, 256) else 0
    assert rule(lattice, BYTES[storage], mb, rows_k, walls) == variant

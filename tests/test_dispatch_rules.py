"""The rules of csrc/dispatch.hpp, compiled by themselves: which launches a call makes at sizes on both sides of each line.
The times behind them stand beside the rules."""
import ctypes
import os
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2401_09149_amd", "csrc")
SHIM = """
#include "dispatch.hpp"
extern "C" int one_launch(int64_t B, int64_t S, int64_t Hq, int64_t Hkv, int causal, int64_t docs) {
  return ie::bwd64_in_one_launch(B, S, Hq, Hkv, causal != 0, docs, 256, 512);
}
"""


@pytest.fixture(scope="module")
def rules(tmp_path_factory):
    d = tmp_path_factory.mktemp("dispatch")
    src, lib = str(d / "shim.cpp"), str(d / "shim.so")
    with open(src, "w") as f:
        f.write(SHIM)
    subprocess.run(["g++", "-std=c++17", "-O1", "-Wall", "-Werror", "-shared", "-fPIC", "-I", CSRC, src, "-o", lib], check=True)
    return ctypes.CDLL(lib)


@pytest.mark.parametrize("B,S,Hq,Hkv,causal,docs,one", [
    (1, 512, 2, 2, 1, 0, True),       # everything resident
    (1, 4096, 8, 8, 0, 0, True),      # exactly
    (1, 700, 48, 48, 1, 0, False),    # 576 short items
    (1, 640, 80, 80, 1, 0, True),
    (1, 1600, 24, 24, 1, 0, True),
    (1, 4096, 16, 8, 0, 0, True),     # fewer dK/dV items than CUs
    (1, 8192, 8, 2, 0, 0, False),
    (1, 8192, 8, 1, 0, 0, False),
    (1, 8192, 16, 8, 1, 0, True),     # one to two rounds
    (1, 6000, 24, 12, 0, 0, True),
    (4, 2000, 16, 16, 0, 0, True),    # several rounds
    (4, 4096, 16, 16, 1, 0, True),
    (2, 8192, 16, 16, 0, 0, False),
    (4, 8192, 16, 16, 1, 0, False),
    (4, 8192, 16, 16, 0, 0, False),
    (1, 65536, 16, 16, 1, 35, False),  # packed: by the mean document
    (1, 16384, 16, 16, 1, 31, True),
])
def test_bwd64_launches(rules, B, S, Hq, Hkv, causal, docs, one):
    i64 = ctypes.c_int64
    assert bool(rules.one_launch(i64(B), i64(S), i64(Hq), i64(Hkv), causal, i64(docs))) == one

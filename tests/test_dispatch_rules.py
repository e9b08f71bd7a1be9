"""The rules of csrc/dispatch.hpp, compiled by themselves: which launches a call makes at sizes on both sides of each line.
The times behind them stand beside the rules."""
import ctypes
import os
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2401_09149_amd", "csrc")
SHIM = """
#include "dispatch.hpp"
extern "C" int route_64(int64_t B, int64_t S, int64_t Hq, int64_t Hkv, int causal, int64_t docs) {
  return (int)ie::bwd64_route(B, S, Hq, Hkv, causal != 0, docs, 256, 512);
}
extern "C" int one_launch_128(int64_t B, int64_t S, int64_t Hq, int64_t Hkv, int causal, int64_t docs) {
  return ie::bwd128_in_one_launch(B, S, Hq, Hkv, causal != 0, docs, 256);
}
extern "C" int fwd_128(int64_t B, int64_t S, int64_t Hq, int causal, int64_t docs, int narrow) {
  return (int)ie::fwd128_route(B, S, Hq, causal != 0, docs, 256, narrow != 0);
}
extern "C" int deals(int64_t items, int one_list, int grouped, int stores) { return ie::dkdv_deals(items, one_list != 0, grouped != 0, stores != 0, 256); }
extern "C" int flips(int64_t items, int64_t tiles, int causal, int packed) { return ie::fwd_flips(items, tiles, causal != 0, packed != 0, 256); }
extern "C" int lazy_64(int64_t items, int causal, int packed, int64_t tiles) { return ie::fwd64_is_lazy(items, causal != 0, packed != 0, 256, tiles); }
extern "C" int by_head(int64_t items, int64_t tiles, int causal, int packed, int d64) {
  return ie::fwd_head_by_head(tiles, items, causal != 0, packed != 0, d64 != 0, 256, false, 1, 0, 128);
}
extern "C" int by_head_of(int64_t B, int64_t S, int64_t Hq, int64_t Hkv, int causal, int64_t D) {
  const int64_t tiles = (S + 127) / 128;
  return ie::fwd_head_by_head(tiles, tiles * B * Hq, causal != 0, false, D == 64, 256, B * Hq % 8 != 0, Hq / Hkv, B * S * Hkv * D * 4, S - (tiles - 1) * 128);
}
extern "C" int bwd_by_head(int64_t S, int64_t heads, int causal, int packed) {
  const int64_t tiles = (S + 127) / 128;
  return ie::bwd_head_by_head(tiles, S - (tiles - 1) * 128, tiles * heads, causal != 0, packed != 0, 256);
}
extern "C" int dq16(int64_t items_128, int64_t items_256, int wide, int causal, int packed) {
  return ie::dq128_on_16x16x32(items_128, items_256, wide != 0, causal != 0, packed != 0, 256);
}
extern "C" int own(int64_t I, int64_t J, int64_t R) {
  float us;
  const ie::Tile tile = ie::pick_tile(I, J, R, 0, 256, &us);
  return ie::pick_own(I, J, R, 256, us, ie::kCost[tile].ti);
}
extern "C" int tile(int64_t I, int64_t J, int64_t R, int product) { return ie::pick_tile(I, J, R, product, 256); }
"""
TILES = [(256, 256), (256, 128), (128, 256), (128, 128), (64, 128), (64, 64), (32, 32)]   # enum Tile


@pytest.fixture(scope="module")
def rules(tmp_path_factory):
    d = tmp_path_factory.mktemp("dispatch")
    src, lib = str(d / "shim.cpp"), str(d / "shim.so")
    with open(src, "w") as f:
        f.write(SHIM)
    subprocess.run(["g++", "-std=c++17", "-O1", "-Wall", "-Werror", "-shared", "-fPIC", "-I", CSRC, src, "-o", lib], check=True)
    return ctypes.CDLL(lib)


WIDE, NARROW, SEQ = 0, 1, 2   # enum Fwd128


@pytest.mark.parametrize("B,S,Hq,causal,docs,narrow,route", [
    (1, 8192, 8, 1, 0, 1, SEQ),         # up to two items per CU
    (1, 8192, 4, 1, 0, 1, SEQ),
    (1, 30000, 1, 1, 0, 0, SEQ),
    (1, 3000, 8, 0, 0, 1, SEQ),
    *((1, s, 2, c, 0, 1, SEQ) for s in (385, 449, 512, 513, 640, 641) for c in (1,)),
    *((1, s, 2, 0, 0, 1, SEQ) for s in (897, 960, 1024, 1025)),   # the GPU test's sizes (test_gpu_fwd_routes.py)
    (2, 700, 3, 1, 0, 1, SEQ), (1, 1100, 4, 0, 0, 1, SEQ), (1, 2500, 2, 1, 4, 0, SEQ), (1, 2300, 2, 0, 4, 0, SEQ),
    (2, 430, 40, 1, 0, 1, NARROW),      # short items, a second round
    (1, 3720, 16, 1, 2, 0, NARROW),     # a few long documents
    (1, 7756, 4, 0, 6, 0, NARROW),
    (1, 12790, 19, 0, 6, 0, WIDE),      # and of more items
    (1, 21359, 17, 0, 12, 0, WIDE),
    (1, 19894, 17, 1, 9, 0, NARROW),   # causal up to twelve items per CU
    (1, 11892, 15, 1, 4, 0, NARROW),
    (1, 24000, 17, 1, 9, 0, WIDE),
    (1, 18616, 8, 1, 8, 0, NARROW),
    (1, 3000, 16, 0, 0, 1, NARROW),
    (1, 3001, 32, 1, 0, 1, NARROW),
    (1, 4129, 17, 0, 0, 1, NARROW),     # a last round of a few items
    (1, 5747, 14, 0, 0, 1, NARROW),
    (1, 6917, 14, 0, 0, 1, WIDE),       # and one of many
    (1, 555, 47, 0, 0, 1, NARROW),      # short items on nearly every CU
    (2, 413, 31, 1, 0, 1, NARROW),
    (1, 555, 8, 1, 0, 1, SEQ),
    (2, 652, 27, 1, 0, 1, NARROW),      # and a second one on some
    (1, 4096, 32, 1, 0, 1, NARROW),
    (1, 32768, 32, 1, 0, 0, WIDE),
    (1, 16384, 16, 1, 0, 0, WIDE),
    (1, 8000, 100, 1, 63, 0, NARROW),   # packed: short documents
    (1, 2222, 2, 1, 4, 0, SEQ),
    (1, 65536, 8, 1, 17, 0, WIDE),      # long ones
    (1, 50671, 9, 0, 35, 0, WIDE),
    (4, 4621, 36, 1, 0, 0, WIDE),       # many items
])
def test_fwd128_route(rules, B, S, Hq, causal, docs, narrow, route):
    i64 = ctypes.c_int64
    assert rules.fwd_128(i64(B), i64(S), i64(Hq), causal, i64(docs), narrow) == route


@pytest.mark.parametrize("B,S,H,causal,packed,flips", [
    (1, 4096, 32, 1, 0, True),
    (2, 4096, 32, 1, 0, True),     # eight items per CU
    (1, 4096, 65, 1, 0, False),
    (1, 1024, 33, 1, 0, True),     # eight tiles
    (1, 1024, 32, 1, 0, False),    # one item per CU
    (4, 647, 36, 1, 0, False),     # short items
    (4, 263, 41, 1, 0, False),
    (1, 896, 60, 1, 0, False),
    (1, 4096, 32, 0, 0, False),
    (1, 4096, 32, 1, 1, False),
    (1, 1100, 60, 1, 0, True),     # the GPU test's sizes (test_gpu_fwd_routes.py)
    (1, 1100, 20, 1, 0, False),
])
def test_forward_order(rules, B, S, H, causal, packed, flips):
    i64, tiles = ctypes.c_int64, -(-S // 128)
    assert bool(rules.flips(i64(B * tiles * H), i64(tiles), causal, packed)) == flips


@pytest.mark.parametrize("items,tiles,causal,packed,d64,share", [
    (512, 8, 0, 0, 0, 0), (520, 8, 0, 0, 0, 8), (5000, 1, 0, 0, 0, 0), (5000, 2, 0, 0, 1, 2), (5000, 8, 0, 1, 0, 0),
    (2048, 8, 1, 0, 0, 0), (2056, 8, 1, 0, 0, 5), (2056, 8, 1, 0, 1, 0), (3080, 8, 1, 0, 1, 5), (9000, 2, 1, 0, 0, 0),
    (4096, 32, 1, 0, 0, 0), (4104, 17, 1, 0, 1, 11), (9000, 3, 1, 0, 0, 3), (9000, 4, 1, 0, 0, 3), (9000, 6, 1, 0, 0, 5), (9000, 5, 1, 1, 0, 0),
])
def test_forward_head_by_head(rules, items, tiles, causal, packed, d64, share):
    assert rules.by_head(ctypes.c_int64(items), ctypes.c_int64(tiles), causal, packed, d64) == share


def by_head(rules, B, S, Hq, Hkv, causal, D):
    return rules.by_head_of(*map(ctypes.c_int64, (B, S, Hq, Hkv)), causal, ctypes.c_int64(D))


@pytest.mark.parametrize("B,S,Hq,Hkv,causal,D,share", [
    (43, 256, 31, 31, 0, 128, 0),       # one list, two to four tiles: K and V of all heads stay in the last-level cache
    (25, 192, 28, 14, 0, 128, 0),
    (17, 301, 12, 12, 0, 128, 0),
    (45, 512, 4, 4, 0, 64, 0),
    (1537, 256, 1, 1, 0, 128, 2),       # 192 MiB and more
    (1535, 256, 1, 1, 0, 128, 0),
    (3074, 256, 2, 1, 0, 128, 2),
    (3, 713, 36, 36, 0, 128, 0),        # five to eight tiles, few items per CU
    (5, 896, 20, 20, 0, 128, 0),
    (6, 896, 30, 30, 0, 64, 0),
    (307, 513, 1, 1, 0, 128, 0),
    (309, 513, 1, 1, 0, 128, 5),
    (86, 1152, 1, 1, 0, 64, 9),         # nine and more
    (85, 1152, 1, 1, 0, 64, 0),
    (31, 2176, 1, 1, 0, 128, 17),
    (54, 163, 32, 32, 0, 128, 0),       # lists, two tiles of which one is not half full
    (54, 192, 32, 32, 0, 128, 0),
    (54, 193, 32, 32, 0, 128, 2),
    (54, 163, 32, 32, 0, 64, 2),
    (16, 163, 32, 32, 0, 64, 0),        # up to four items per CU at head dimension 64
    (159, 190, 24, 24, 0, 128, 2),      # K and V of all heads outgrow the last-level cache
    (82, 190, 24, 24, 0, 128, 0),
    (69, 538, 4, 1, 0, 128, 5),         # one list, grouped heads
    (49, 512, 4, 1, 0, 128, 4),
    (47, 512, 4, 1, 0, 128, 0),
    (49, 512, 4, 2, 0, 128, 0),
    (49, 512, 4, 1, 0, 64, 0),
    (39, 538, 4, 2, 0, 128, 5),
    (39, 538, 4, 2, 0, 64, 0),
    (378, 975, 4, 4, 0, 128, 8),
    (83, 544, 36, 36, 1, 128, 5),
    (118, 2230, 5, 5, 1, 64, 13),
])
def test_forward_head_by_head_by_shape(rules, B, S, Hq, Hkv, causal, D, share):
    assert by_head(rules, B, S, Hq, Hkv, causal, D) == share


@pytest.mark.parametrize("S,heads,causal,packed,share", [
    (161, 1544, 0, 0, 0), (192, 1544, 0, 0, 0), (193, 1544, 0, 0, 2), (202, 360, 0, 0, 2),   # two tiles: 33 to 74 rows in the last, many items
    (202, 256, 0, 0, 0), (224, 256, 0, 0, 0), (202, 264, 0, 0, 2),   # two dQ items per CU
    (225, 64, 0, 0, 2), (256, 64, 0, 0, 2), (257, 64, 0, 0, 3), (384, 1208, 0, 0, 3), (384, 1208, 1, 0, 0), (384, 1208, 0, 1, 0), (100, 64, 0, 0, 1),
])
def test_backward_head_by_head(rules, S, heads, causal, packed, share):
    assert rules.bwd_by_head(ctypes.c_int64(S), ctypes.c_int64(heads), causal, packed) == share


def test_gpu_cases_of_many_heads(rules):
    """test_many_heads_in_head_by_head_order: the kernel with that order, the share of tiles it names and, with a backward
    pass, the shared launch, in that order in one of them."""
    from test_gpu_fwd_routes import MANY_HEADS
    for S, heads, D, causal, backward, H, group, share in MANY_HEADS:
        B, Hkv = heads // H, H // group
        assert heads % H == 0 and by_head(rules, B, S, H, Hkv, causal, D) == share, (S, heads)
        if D == 128:
            assert rules.fwd_128(*map(ctypes.c_int64, (B, S, H)), causal, ctypes.c_int64(0), 1) == NARROW, (S, heads)   # (sizes alone: 4096 tokens and fewer)
        if backward:
            assert rules.one_launch_128(*map(ctypes.c_int64, (B, S, H, Hkv)), causal, ctypes.c_int64(0)) == 1, (S, heads)
    assert any(backward and heads % 8 == 0 and rules.bwd_by_head(ctypes.c_int64(S), ctypes.c_int64(heads), causal, 0) > 1 for S, heads, _, causal, backward, *_ in MANY_HEADS)
    assert {(D, causal, B_H % 8 != 0) for _, B_H, D, causal, _, _, _, share in MANY_HEADS if share} >= {
        (64, False, False), (64, False, True), (64, True, False), (128, False, False), (128, False, True), (128, True, False), (128, True, True)}


@pytest.mark.parametrize("S,H,causal,packed,lazy", [
    (512, 2, 1, 0, False),       # the smallest calls: a wave per SIMD
    (4096, 8, 0, 0, False),      # 256 items
    (4096, 9, 0, 0, True),
    (8192, 12, 1, 0, False),     # 768
    (8192, 13, 1, 0, True),
    (2000, 64, 0, 0, True),
    (8192, 12, 1, 1, False),
    (8192, 12, 0, 1, False),
    (8192, 13, 0, 1, True),
    (512, 400, 1, 0, False),     # four tiles
    (513, 400, 1, 0, True),
    (500, 400, 0, 0, False),
])
def test_fwd64_search(rules, S, H, causal, packed, lazy):
    i64, tiles = ctypes.c_int64, -(-S // 128)
    assert bool(rules.lazy_64(i64(tiles * H), causal, packed, i64(tiles))) == lazy


def test_cases_of_both_forward_bodies_at_head_dimension_64(rules):
    from test_gpu_fwd_routes import LAZY_64, SEARCHING_64
    for cases, lazy in ((LAZY_64, True), (SEARCHING_64, False)):
        for S, H, causal, lens in cases:
            tiles = S // 128 + len(lens) if lens else -(-S // 128)
            mean = S // 128 // len(lens) if lens else tiles
            assert bool(rules.lazy_64(ctypes.c_int64(tiles * H), int(causal), int(lens is not None), ctypes.c_int64(mean))) == lazy, (S, H)


TWO, DEALT, QUEUED = 0, 1, 2   # enum Bwd64


@pytest.mark.parametrize("B,S,Hq,Hkv,causal,docs,route", [
    (1, 700, 48, 48, 1, 0, DEALT),      # a little over one round of short items
    (1, 640, 80, 80, 1, 0, DEALT),
    (1, 8192, 8, 1, 0, 0, DEALT),       # fewer dK/dV items than CUs
    (1, 8192, 8, 2, 0, 0, DEALT),
    (1, 8192, 16, 8, 1, 0, DEALT),      # one to two rounds
    (1, 1000, 80, 80, 1, 0, DEALT),     # the GPU test's sizes (test_gpu_bwd_both.py)
    (1, 1300, 80, 20, 0, 0, DEALT),
    (4, 2000, 16, 16, 0, 0, TWO),       # several rounds
    (4, 4096, 16, 16, 1, 0, TWO),
    (4, 8192, 16, 16, 0, 0, TWO),
    (1, 13900, 24, 3, 0, 0, QUEUED),    # long items of grouped heads
    (1, 6400, 56, 14, 0, 0, QUEUED),
    (1, 6400, 64, 16, 0, 0, QUEUED),
    (1, 6400, 136, 17, 0, 0, TWO),      # dK/dV items that nearly fill their last round
    (1, 2020, 192, 6, 0, 0, DEALT),     # fewer dK/dV items than CUs
    (1, 13900, 24, 3, 0, 1, DEALT),     # packed
    (1, 13900, 24, 3, 1, 0, DEALT),
    (153, 886, 24, 24, 1, 0, TWO),      # many short batch entries
    (1127, 193, 16, 16, 1, 0, TWO),
    (1127, 100, 16, 16, 1, 0, DEALT),   # of one tile
    (100, 193, 16, 16, 1, 0, DEALT),    # not so many
    (1, 16384, 16, 16, 1, 31, DEALT),
    (1, 52129, 8, 2, 1, 53, DEALT),     # packed: the longest document's tail
    (1, 15593, 24, 6, 1, 11, DEALT),
    (1, 10106, 40, 10, 1, 6, DEALT),
    (1, 65065, 136, 34, 1, 261, TWO),   # and rounds enough to hide it
    (1, 38376, 136, 34, 1, 74, TWO),
])
def test_bwd64_route(rules, B, S, Hq, Hkv, causal, docs, route):
    i64 = ctypes.c_int64
    assert rules.route_64(i64(B), i64(S), i64(Hq), i64(Hkv), causal, i64(docs)) == route


@pytest.mark.parametrize("B,S,Hq,Hkv,causal,docs,one", [
    (1, 2048, 16, 16, 1, 0, True),     # a dK/dV item and a dQ item per CU
    (1, 4096, 8, 8, 1, 0, True),
    (1, 8192, 4, 4, 1, 0, True),
    (1, 300, 128, 128, 1, 0, True),    # the GPU test's sizes (test_gpu_bwd_both.py)
    (2, 200, 160, 40, 0, 0, True),
    (1, 260, 150, 150, 1, 2, True),
    (1, 3001, 32, 8, 1, 0, True),      # fewer dK/dV items than CUs, each of 4 heads
    (1, 14426, 16, 2, 1, 0, True),
    (1, 4096, 32, 32, 1, 0, False),
    (2, 4096, 32, 32, 1, 0, False),
    (1, 32768, 32, 32, 1, 0, False),
    (2, 6144, 10, 10, 0, 0, False),
    (1, 65536, 8, 8, 1, 20, False),
    (102, 689, 24, 24, 1, 0, False),   # many short batch entries
    (387, 141, 16, 16, 0, 0, False),
    (561, 161, 8, 8, 0, 0, False),
    (735, 100, 22, 22, 1, 0, True),    # of one tile
    (1, 50000, 8, 8, 1, 180, False),   # packed: short documents, many items
    (1, 35000, 4, 4, 1, 12, True),     # long ones on few heads
    (1, 13439, 36, 9, 1, 2, False),    # two documents: neither is three times their mean
    (1, 18080, 28, 7, 1, 2, False),
    (1, 13880, 19, 19, 0, 0, False),   # equal items: a gain of 4 % at least
    (1, 2568, 20, 10, 0, 0, False),
    (1, 12173, 17, 17, 0, 0, False),
])
def test_bwd128_launches(rules, B, S, Hq, Hkv, causal, docs, one):
    i64 = ctypes.c_int64
    assert bool(rules.one_launch_128(i64(B), i64(S), i64(Hq), i64(Hkv), causal, i64(docs))) == one


@pytest.mark.parametrize("B,S,Hq,Hkv,causal,docs", [
    (2 ** 20, 1, 8, 8, 1, 0),              # 2^24 backward items, 2^23 in the forward
    (2 ** 19, 100, 24, 12, 0, 0),
    (1, 2 ** 22, 32, 32, 1, 2 ** 19),      # packed: 2^19 short documents
])
def test_more_items_than_a_launch_has_workgroups(rules, B, S, Hq, Hkv, causal, docs):
    """A launch that the hardware deals out has fewer than 2^32 threads (2^24 workgroups); queues take what is beyond."""
    i64 = ctypes.c_int64
    args = (i64(B), i64(S), i64(Hq), i64(Hkv), causal, i64(docs))
    items = B * (S // 128 + docs if docs else -(-S // 128))
    assert items * (Hq + Hkv) >= 2 ** 24
    assert rules.route_64(*args) != DEALT and not rules.one_launch_128(*args)
    if items * Hq >= 2 ** 24:
        assert rules.fwd_128(i64(B), i64(S), i64(Hq), causal, i64(docs), 0) == WIDE


@pytest.mark.parametrize("S,Hq,Hkv,stores,deals", [
    (9984, 6, 6, 1, False),      # one list, dS stored
    (3328, 15, 15, 1, False),
    (8192, 5, 5, 1, True),       # 320 items
    (9984, 6, 6, 0, True),
    (4096, 16, 16, 1, True),     # eight lists
    (32046, 16, 2, 0, False),    # one list of grouped heads
    (32046, 64, 8, 0, True),
])
def test_first_dkdv_items(rules, S, Hq, Hkv, stores, deals):
    i64 = ctypes.c_int64
    assert bool(rules.deals(i64(-(-S // 128) * Hkv), int(Hkv % 8 != 0), int(Hq != Hkv), stores)) == deals


@pytest.mark.parametrize("S,H,wide,causal,packed,on16", [
    (32768, 16, 1, 1, 0, True),
    (4096, 32, 1, 0, 0, True),
    (2048, 40, 1, 1, 0, True),     # 320 items of 256 rows
    (3001, 24, 1, 1, 0, False),    # 288
    (6000, 8, 1, 1, 0, False),
    (2048, 32, 1, 0, 0, True),     # 256
    (3001, 16, 1, 0, 0, False),    # 192
    (8192, 8, 0, 1, 0, True),
    (12000, 3, 0, 1, 0, False),
    (8192, 6, 0, 0, 0, True),
    (12000, 3, 0, 0, 0, False),
    (65536, 8, 1, 1, 1, True),
    (16384, 4, 1, 1, 1, False),
    (128, 250, 1, 0, 0, False),    # no 128-row item for every CU
])
def test_dq128_form(rules, S, H, wide, causal, packed, on16):
    i64 = ctypes.c_int64
    assert bool(rules.dq16(i64(-(-S // 128) * H), i64(-(-S // 256) * H), wide, causal, packed)) == on16


def linear_tile(rules, product, M, N, K):
    """Output tile of a product of y = x w^T (x [M,K], w [N,K]) on 256 CUs."""
    I, J, R = {"fwd": (M, N, K), "dx": (M, K, N), "dw": (N, K, M)}[product]
    i64 = ctypes.c_int64
    return TILES[rules.tile(i64(I), i64(J), i64(R), ["fwd", "dx", "dw"].index(product))]


@pytest.mark.parametrize("product,M,N,K,tile", [
    # weight gradients over a few tokens: the outputs' way to memory, for which larger tiles do better
    ("dw", 128, 8192, 8192, (256, 256)),
    ("dw", 64, 4096, 4096, (256, 256)),
    ("dw", 192, 30720, 5120, (256, 256)),
    ("dw", 8192, 9600, 3200, (256, 256)),
    ("dw", 512, 2048, 2048, (128, 128)),
    ("dx", 4096, 17152, 3200, (256, 256)),
    ("fwd", 8192, 12288, 4096, (256, 256)),
    ("fwd", 200, 4096, 4096, (64, 64)),
    ("fwd", 1, 4096, 11008, (32, 32)),
])
def test_linear_tile(rules, product, M, N, K, tile):
    assert linear_tile(rules, product, M, N, K) == tile


def own(rules, M, N, K):
    return rules.own(ctypes.c_int64(M), ctypes.c_int64(N), ctypes.c_int64(K))


@pytest.mark.parametrize("M,N,K,kernel", [
    (200, 12288, 4096, 3), (200, 4096, 4096, 1), (200, 4096, 11008, 1), (200, 22016, 4096, 0),
    (31, 4096, 4096, 0), (1537, 2368, 2368, 0), (1, 22016, 4096, 0), (8192, 4096, 4096, 0),
    (48, 6144, 1024, 1), (48, 6144, 960, 0), (60, 69632, 1280, 2), (60, 131080, 1280, 0), (1111, 5328, 14848, 3),
    (1200, 256, 4096, 1), (1500, 328, 8192, 1), (270, 10912, 65536, 3), (270, 10912, 65600, 0),
    (362, 11088, 768, 0),      # few steps, several rounds
    (318, 13312, 1024, 0), (131, 16128, 768, 0),
    (85, 33288, 1792, 0),      # one row tile, two rounds of weights that are read once
    (113, 33000, 2496, 0), (127, 39936, 2304, 0),
    (83, 12360, 9856, 0),      # and one round of them
    (84, 12544, 6912, 0),
    (683, 3584, 768, 0),       # few steps
    (132, 11776, 768, 0),
])
def test_forward_tiles_of_independent_waves(rules, M, N, K, kernel):
    assert own(rules, M, N, K) == kernel


def test_gpu_cases_of_independent_waves(rules):
    """They take the kernels they name, each also with more tiles than CUs; the ring's cases are left to the ring."""
    from test_gpu_linear_tiles import FORWARD, OWN
    assert [own(rules, M, N, K) for M, N, K, _ in OWN] == [k for *_, k in OWN]
    for kernel, (ti, tj) in {1: (64, 64), 2: (64, 96), 3: (128, 96)}.items():
        assert any(k == kernel and -(-M // ti) * -(-N // tj) > 256 for M, N, _, k in OWN), kernel
    assert {(k, K // 64 % 4 != 0) for _, _, K, k in OWN} >= {(1, True), (2, True), (3, True), (1, False), (2, False), (3, False)}
    assert all(own(rules, M, N, K) == 0 for M, N, K, _ in FORWARD)


def test_every_linear_route_has_a_gpu_case(rules):
    """The cases of test_gpu_linear_tiles take the tiles they name, and together every kernel of every product."""
    from test_gpu_linear_tiles import BACKWARD, FORWARD
    cases = [("fwd", M, N, K, t) for M, N, K, t in FORWARD]
    cases += [(p, M, N, K, t) for M, N, K, dx, dw in BACKWARD for p, t in (("dx", dx), ("dw", dw)) if t]
    for p, M, N, K, t in cases:
        assert linear_tile(rules, p, M, N, K) == t, (p, M, N, K)
    routes = {(p, t) for p in ("fwd", "dx", "dw") for t in TILES} - {("dx", (32, 32)), ("dw", (32, 32))}
    assert {(p, t) for p, *_, t in cases} == routes


def test_dq_full_chip_cases_take_the_16x16x32_form(rules):
    from test_gpu_dq_full_chip import CASES
    i64 = ctypes.c_int64
    for name, (B, S, Hq, Hkv, causal, lens) in CASES.items():
        packed = lens is not None
        items = [-(-S // rows) * B * Hq for rows in (128, 256)]
        assert not packed or sum(lens) == S
        for wide in (0, 1):
            assert rules.dq16(i64(items[0]), i64(items[1]), wide, int(causal), int(packed)), (name, wide)


def backward_form(rules, B, S, Hq, Hkv, D, causal, docs):
    """"two" launches, one that the hardware deals out, or one with queues, as launch_bwd_d (csrc/attn_bwd.hip) chooses."""
    i64 = ctypes.c_int64
    items = B * (S // 128 + docs if docs else -(-S // 128)) * (Hq + Hkv)
    if items <= (512 if D == 64 else 256):   # all resident
        return "dealt"
    args = (i64(B), i64(S), i64(Hq), i64(Hkv), int(causal), i64(docs))
    return ("two", "dealt", "queued")[rules.route_64(*args) if D == 64 else rules.one_launch_128(*args)]


def test_launches_of_the_shared_launch_cases(rules):
    """The cases of test_gpu_bwd_both take the launches that they are there for."""
    from test_gpu_bwd_both import DEALT as dealt, MORE, QUEUED as queued
    for B, S, Hq, Hkv, D, causal, lens in dealt + MORE:
        assert backward_form(rules, B, S, Hq, Hkv, D, causal, len(lens) if lens else 0) == "dealt", (B, S, Hq)
    B, S, Hq, Hkv, D, causal, _ = queued
    assert backward_form(rules, B, S, Hq, Hkv, D, causal, 0) == "queued"


def test_fused_sequence_parallel_cases_take_every_form(rules):
    """The cases of test_gpu_sp_fused take the kernels that they name, and together every one that has a chunked form."""
    from test_gpu_sp_fused import CASES
    i64, seen = ctypes.c_int64, set()
    for B, Sl, Hq, Hkv, D, P, causal, fwd, bwd in CASES:
        S, Hql, Hkvl = P * Sl, Hq // P, Hkv // P
        assert backward_form(rules, B, S, Hql, Hkvl, D, causal, 0) == bwd, (Sl, Hq, D)
        if D == 128:
            narrow = S <= 4096 or (S <= 8192 and -(-S // 256) * B * Hql < 512)   # fwd_prefers_128_rows (csrc/launch.hpp)
            assert ("wide", "narrow", "seq")[rules.fwd_128(i64(B), i64(S), i64(Hql), int(causal), i64(0), int(narrow))] == fwd, (Sl, Hq)
        seen |= {(D, "fwd", fwd), (D, "bwd", bwd)}
    assert seen == {(64, "fwd", "narrow"), *((128, "fwd", f) for f in ("wide", "narrow", "seq")),
                    *((64, "bwd", b) for b in ("two", "dealt", "queued")), *((128, "bwd", b) for b in ("two", "dealt"))}

"""The linear kernels' tile sizes at their edges: every route of the size rule (pick_tile in csrc/dispatch.hpp), with
one output index less and more than whole tiles, contractions that fill the copy ring partly, exactly and with a partial
last step, and more tiles than workgroups.  The tiles named here are what the rule gives on 256 CUs; test_dispatch_rules
holds it to them, and holds this file to all routes.  Oracle, tolerance and its derivation are test_gpu_linear's."""
import pytest

from test_gpu_linear import run_all

pytestmark = pytest.mark.gpu

FORWARD = [   # M, N, K, tile
    (1, 8, 64, (32, 32)),            # one tile with one row and eight columns, a quarter of one step
    (33, 2056, 320, (32, 32)),       # one step and a quarter
    (1, 9736, 768, (32, 32)),        # more tiles than CUs: the ring runs on across tiles
    (31, 9608, 576, (64, 64)),       # one tile row, ragged in both indices
    (250, 4040, 2112, (64, 64)),     # 33 steps, more row tiles than one
    (1543, 520, 2112, (64, 64)),
    (129, 8200, 128, (64, 128)),     # fewer steps than ring stages
    (130, 20488, 320, (64, 128)),    # more tiles than CUs
    (255, 12296, 192, (128, 128)),
    (640, 9224, 192, (128, 256)),
    (2047, 2056, 1024, (256, 128)),
    (2300, 7432, 1088, (256, 256)),  # more tiles than CUs
    (2049, 4104, 64, (256, 256)),
]
BACKWARD = [   # M, N, K, dx tile, dw tile
    (64, 64, 8, (64, 128), (64, 128)),          # one output chunk per row
    (64, 1536, 520, (64, 64), (64, 128)),
    (448, 320, 2056, (64, 64), (64, 64)),
    (1088, 192, 2056, (128, 128), (64, 64)),
    (2304, 64, 7176, (256, 128), (64, 64)),     # dx with a single step per tile
    (128, 3840, 2056, (64, 64), (256, 128)),    # dx with 60 steps
    (320, 1920, 4352, (64, 128), (128, 256)),
    (320, 6400, 4104, (64, 128), (256, 256)),   # dw with five steps per tile
    (2304, 1088, 4104, (256, 256), (128, 256)),
    (1088, 320, 4104, (128, 256), (64, 128)),
    (320, 1544, 1544, None, (128, 128)),        # dw ragged in both indices (N is not a multiple of 64: no dx)
]


@pytest.mark.parametrize("M,N,K,tile", FORWARD)
def test_forward_tiles(M, N, K, tile):
    print(f"case M{M} N{N} K{K} {tile}", flush=True)
    run_all(M, N, K, seed=M + N + K, which=("fwd",))


@pytest.mark.parametrize("M,N,K,dx,dw", BACKWARD)
def test_backward_tiles(M, N, K, dx, dw):
    print(f"case M{M} N{N} K{K} {dx} {dw}", flush=True)
    run_all(M, N, K, seed=M + N + K, which=("dx", "dw") if dx else ("dw",))


OWN = [   # M, N, K, kernel of enum Own: the forward tiles whose waves share nothing (pick_own in csrc/dispatch.hpp)
    (35, 4552, 1024, 1),      # four steps per wave, one tile per workgroup, ragged in both indices
    (449, 2008, 1792, 1),     # the 256th tile of 256
    (394, 624, 2112, 1),      # 33 steps: one wave has a ninth
    (1478, 1296, 1280, 1),    # two rounds: the rings run on across tiles
    (1250, 264, 2112, 1),     # a narrow output
    (65, 8320, 1856, 2),
    (33, 68312, 1728, 2),     # three rounds, with a step less in one wave
    (604, 1608, 1024, 2),
    (65, 16736, 1984, 3),
    (1218, 1624, 1536, 3),
    (130, 12224, 1536, 3),    # 256 tiles
    (260, 11032, 5632, 3),    # two rounds: the rings, one step of A and two of B, run on across tiles
    (266, 10912, 6336, 3),    # and with a step less in one wave
]


@pytest.mark.parametrize("M,N,K,own", OWN)
def test_forward_tiles_of_independent_waves(M, N, K, own):
    print(f"case M{M} N{N} K{K} {own}", flush=True)
    run_all(M, N, K, seed=M + N + K, which=("fwd",))

"""The linear kernels' tile sizes at their edges: every route of the size rule (pick_tile in csrc/linear_gemm.hip), with
one output index less and more than whole tiles, contractions that fill the copy ring partly, exactly and with a partial
last step, and more tiles than workgroups.  Oracle, tolerance and its derivation are test_gpu_linear's."""
import pytest

from test_gpu_linear import run_all

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("M,N,K", [
    (1, 8, 64),          # one 32 x 32 tile with one row and eight columns, a quarter of one step
    (33, 2056, 320),     # 32 x 32 tiles, one step and a quarter
    (31, 9608, 576),     # 32 x 32, more tiles than CUs: the ring runs on across tiles
    (250, 4040, 2112),   # 64 x 64
    (129, 8200, 128),    # 64 x 128, fewer steps than ring stages
    (130, 20488, 320),   # 64 x 128, more tiles than CUs
    (255, 12296, 192),   # 128 x 128
    (640, 9224, 192),    # 128 x 256
    (2047, 2056, 1024),  # 256 x 128
    (2300, 7432, 1088),  # 256 x 256, more tiles than CUs
])
def test_forward_tiles(M, N, K):
    print(f"case M{M} N{N} K{K}", flush=True)
    run_all(M, N, K, seed=M + N + K, which=("fwd",))


@pytest.mark.parametrize("M,N,K", [
    # (dx tile, dw tile)
    (64, 64, 8),         # 64 x 128 both: one output chunk per row
    (64, 1536, 520),     # 64 x 64, 64 x 128
    (448, 320, 2056),    # 64 x 128, 64 x 64
    (1088, 192, 2056),   # 128 x 128, 64 x 64
    (2304, 64, 7176),    # 128 x 256 with a single step per tile, 64 x 64
    (128, 3840, 2056),   # 64 x 64 with 60 steps, 256 x 128
    (320, 1920, 4352),   # 64 x 128, 128 x 256
    (320, 6400, 4104),   # 64 x 128, 256 x 256 with five steps per tile
    (2304, 1088, 4104),  # 256 x 256, 128 x 256
])
def test_backward_tiles(M, N, K):
    print(f"case M{M} N{N} K{K}", flush=True)
    run_all(M, N, K, seed=M + N + K, which=("dx", "dw"))

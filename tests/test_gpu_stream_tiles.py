"""Importance, stream kernels: blocks of stationary rows that end after each of their tiles (a wavefront with two tiles has an
early and a late one, some of which lie past the end), one tile per wavefront and two groups of wavefronts; against fp64."""
import pytest

from test_gpu_launch_shapes import run_importance_on_gpu

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("B,L,H,Hkv,N,D", [
    (5, 1, 41, 41, 1025, 128), (5, 1, 41, 41, 1056, 64), (5, 1, 41, 41, 1089, 128),      # 64 rows per wavefront, five blocks
    (5, 1, 41, 41, 1152, 128), (5, 1, 41, 41, 1185, 64), (5, 1, 41, 41, 1217, 128), (5, 1, 41, 41, 1249, 128),
    (1, 1, 8, 2, 801, 128), (1, 1, 8, 8, 833, 64), (1, 1, 6, 3, 865, 128), (1, 1, 8, 4, 896, 128),   # two groups
    (1, 10, 40, 8, 161, 128), (1, 10, 40, 8, 225, 64),                                   # one group, 800 blocks
])
def test_tiles(B, L, H, Hkv, N, D):
    run_importance_on_gpu(B, L, H, Hkv, N, D)
